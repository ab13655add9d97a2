// Forward product of the N:M-sparse ternary linear layer in block tiles of middle size (Section 2.2 forward-pass equation):
// a layer or a few with some 200 to 1500 tokens, where tiles of 64 x 32 whose wavefronts share nothing (sbn_tile.hip) bring too many
// bytes per product and pieces of 512 rows (sbn_gemm.hip) leave most multiprocessors with one short piece.
//
// A block owns R rows of W and T tokens over the whole input dimension; a ring of stages 512 weights deep (four chunks: 128 bytes of
// a weight row, 512 of a token row) is filled by LDS-DMA, and the wavefronts share the stage: NW of them side by side over the
// rows, KS rows of them over the stage's chunks.  The fragments of the next stage are read, and the stage after the ring asked
// for, between the matrix instructions of the current one; one barrier per stage.
// What bounds it: the operand bytes, of which a multiprocessor takes in 45 to 57 per ns while they come from memory or the
// last-level cache (every XCD fetches the rows the quantizer has just written; on operands in the L2 777 x 2560 -> 2560 takes 9.0 us
// instead of 11.1), on top of 3.5 us for launch, first stage and result.  So tiles are chosen for few bytes and few rounds.  Three other
// schedules of the main loop (fragments read where they are used, a quarter stage ahead, stages of 256) were no faster.
// Measured, us per launch behind the quantizer, weights from memory, 2:4 (the faster of tiles and pieces -> this one):
//   tokens          256           384           512           640           777
//   2560 -> 2560    8.5 -> 7.6    9.0 -> 8.0    11.1 -> 9.6   13.5 -> 10.0  13.7 -> 11.2
//   2560 -> 6912   12.7 -> 9.4   16.0 -> 14.3  (15.9 / 16.4) (17.2 / 21.0)
//   6912 -> 2560   13.8 -> 13.5  15.8 -> 14.7  20.4 -> 15.8  23.7 -> 17.6  24.8 -> 21.0
//   4096 -> 4096   10.7 -> 9.5   13.9 -> 11.6  17.2 -> 13.7
#include <algorithm>

#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

struct BlockItem {
    const int8_t *xq;
    const float *sx;
    const uint8_t *packed;
    const float *gamma;
    const float *bias;
    float *Y;
    int32_t *acc_out;
    int d_in, d_out, tokens;
    int tiles_r, tiles_t;   // row and token tiles
    int group;              // token tiles that are walked before the next row tile
};
constexpr int BLOCK_ITEMS = 8;   // problems of a launch
struct BlockTable {
    BlockItem it[BLOCK_ITEMS];
    int tile0[BLOCK_ITEMS + 1];   // first tile of each problem; entries past the last problem hold the total
};

// NW wavefronts side by side over the rows, each 32 RW rows and all 32 TW tokens; KS of these rows of wavefronts split every
// stage's 512 weights; NS stages
template <int NW_, int KS_, int RW_, int TW_, int NS_> struct BlockShape {
    static constexpr int NW = NW_, KS = KS_, RW = RW_, TW = TW_, NS = NS_;
    static constexpr int R = 32 * RW * NW, T = 32 * TW, WAVES = NW * KS, THREADS = 64 * WAVES;
    static constexpr int ABYTES = R * 128, BBYTES = T * 512, STAGE = ABYTES + BBYTES;   // one stage: 512 weights deep
    static constexpr int NA = R / 8 / WAVES, NB = T / 2 / WAVES, DMA = NA + NB;   // LDS-DMA instructions of a wavefront per stage
    static constexpr int PITCH = R + 4;                       // words between the token rows of a staged tile of sums
    static constexpr int SUMS = 32 * PITCH;                   // words of 32 token rows
    static constexpr int SUMBUF = TW > 1 ? 2 : 1;             // buffers of them
    static constexpr int LDS = NS * STAGE > SUMBUF * KS * SUMS * 4 ? NS * STAGE : SUMBUF * KS * SUMS * 4;   // the ring, later the sums
    static_assert(NA * WAVES * 8 == R && NB * WAVES * 2 == T, "every wavefront brings the same number of rows");
    static_assert(R + T <= THREADS, "a thread for every scale and bias of the tile");
    static_assert((NS - 1) * DMA < 64, "the wait counter holds what may be outstanding");
    static_assert(LDS + 4 * (R + T) <= 160 * 1024, "a multiprocessor's LDS");
};

template <class S, bool DENSE>
__global__ void __launch_bounds__(S::THREADS) gemm_block_kernel(BlockTable tab)
{
    constexpr int R = S::R, T = S::T, RW = S::RW, TW = S::TW, NS = S::NS, KS = S::KS, PITCH = S::PITCH;
    extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
    __shared__ __attribute__((aligned(16))) float scale_s[T], bias_s[R];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD x takes the x-th of eight runs of consecutive tiles
    const int total = (int)gridDim.x, x8 = (int)blockIdx.x & 7, q8 = total >> 3, rem8 = total & 7;
    const int tile = x8 * q8 + (x8 < rem8 ? x8 : rem8) + ((int)blockIdx.x >> 3);
    int p = 0;
    while (p + 1 < BLOCK_ITEMS && tile >= tab.tile0[p + 1]) ++p;
    const BlockItem &g = tab.it[p];
    int to, tt;
    {
        const int local = tile - tab.tile0[p], per = g.tiles_r * g.group, gi = local / per, in = local % per;
        const int left = g.tiles_t - gi * g.group, wide = left < g.group ? left : g.group;
        to = in / wide;
        tt = gi * g.group + in % wide;
    }
    const int row0 = to * R, t0 = tt * T;
    const int r = lane & 31, c = lane >> 5;
    const int wr = wave % S::NW, kg = wave / S::NW;
    const uint32_t ones = vgpr_ones();
    const int K = g.d_in, nchunks = K / CHUNK, nstage = (nchunks + 3) >> 2;
    const uint32_t lds0 = lds_address(lds);

    float pre = 0.0f, gamma = 0.0f;
    const bool has_bias = g.bias != nullptr;
    if (tid < T) {
        pre = g.sx[t0 + tid < g.tokens ? t0 + tid : g.tokens - 1];
        gamma = *g.gamma;
    } else if (has_bias && tid - T < R) {
        pre = g.bias[row0 + tid - T < g.d_out ? row0 + tid - T : g.d_out - 1];
    }

    const uint8_t *const wbase = g.packed + (int64_t)row0 * nchunks * 32;
    const int8_t *const xbase = g.xq + (int64_t)t0 * K;
    // weights: one instruction fills 8 rows of 128 bytes (four chunks), slot l % 8 of a row holds granule (l % 8) ^ ((row >> 1) & 7);
    // tokens: 2 rows of 512 bytes, slot l % 32 holds granule (l % 32) ^ (row & 15)
    uint32_t woff[S::NA], xoff[S::NB];
#pragma unroll
    for (int i = 0; i < S::NA; ++i) {
        const int row = 8 * (S::NA * wave + i) + (lane >> 3), o = row0 + row < g.d_out ? row : g.d_out - 1 - row0;
        woff[i] = (uint32_t)o * (uint32_t)(nchunks * 32) + 16u * ((lane & 7) ^ ((row >> 1) & 7));
    }
#pragma unroll
    for (int i = 0; i < S::NB; ++i) {
        const int row = 2 * (S::NB * wave + i) + (lane >> 5), t = t0 + row < g.tokens ? row : g.tokens - 1 - t0;
        xoff[i] = (uint32_t)t * (uint32_t)K + 16u * ((lane & 31) ^ (row & 15));
    }
    auto request_one = [&](int s, int slot, int k) {   // k-th of a wavefront's DMA instructions of a stage
        const uint32_t dst = lds0 + slot * S::STAGE;
        const int left = nchunks - 4 * s;   // chunks that do not exist: the stage's first in their place (meets zero codes)
        if (k < S::NA) {
            const int row = 8 * (S::NA * wave + k) + (lane >> 3), chunk = ((lane & 7) ^ ((row >> 1) & 7)) >> 1;
            lds_dma16(wbase + (int64_t)s * 128, chunk < left ? woff[k] : woff[k] - 32u * (uint32_t)chunk, dst + 1024 * (S::NA * wave + k));
        } else {
            const int i = k - S::NA, row = 2 * (S::NB * wave + i) + (lane >> 5), chunk = ((lane & 31) ^ (row & 15)) >> 3;
            lds_dma16(xbase + (int64_t)s * 512, chunk < left ? xoff[i] : xoff[i] - 128u * (uint32_t)chunk, dst + S::ABYTES + 1024 * (S::NB * wave + i));
        }
    };
    auto request = [&](int s, int slot) {
#pragma unroll
        for (int k = 0; k < S::DMA; ++k) request_one(s, slot, k);
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nstage) request(s, s);

    v16i acc[RW][TW];
#pragma unroll
    for (int a = 0; a < RW; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0;

    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef __attribute__((address_space(3))) const v2u *lds_v2u;
    typedef __attribute__((address_space(3))) const v4u *lds_v4u;
    // [chunk of the stage this wavefront walks][sub-step][lower, upper 16 bytes] and [chunk]
    constexpr int NH = 4 / KS;   // chunks of a stage that a wavefront multiplies
    uint32_t baddr[NH][2][2], iaddr[NH], caddr[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const int h = NH * kg + i;
        const uint32_t brow = lds0 + S::ABYTES + r * 512, arow = lds0 + (32 * RW * wr + r) * 128, asw = (r >> 1) & 7;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            baddr[i][u][0] = brow + 16 * ((8 * h + 2 * u + c) ^ (r & 15));
            baddr[i][u][1] = brow + 16 * ((8 * h + 4 + 2 * u + c) ^ (r & 15));
        }
        iaddr[i] = DENSE ? arow + 16 * ((2 * h + c) ^ asw) : arow + 8 * c + 16 * ((2 * h) ^ asw);
        caddr[i] = DENSE ? 0 : arow + 8 * c + 16 * ((2 * h + 1) ^ asw);
    }
    // the fragments of a stage: [chunk][sub-step][token tile], [chunk][row tile]
    struct Frag {
        v8i x[NH][2][TW];
        v4u w[NH][RW];
    };
    constexpr int NREAD = NH * (RW + 2 * TW);
    auto read_one = [&](Frag &f, uint32_t at, int k) {   // k-th of NREAD reads
        const int i = k / (RW + 2 * TW), j = k % (RW + 2 * TW);
        if (j < RW) {
            if constexpr (DENSE) {
                f.w[i][j] = ((lds_v4u)(uintptr_t)(iaddr[i] + at))[32 * j * 128 / 16];
            } else {
                const v2u iv = ((lds_v2u)(uintptr_t)(iaddr[i] + at))[32 * j * 128 / 8], cv = ((lds_v2u)(uintptr_t)(caddr[i] + at))[32 * j * 128 / 8];
                f.w[i][j] = v4u{iv.x, iv.y, cv.x, cv.y};
            }
        } else {
            const int u = (j - RW) / TW, b = (j - RW) % TW;
            f.x[i][u][b].lo = ((lds_v4i)(uintptr_t)(baddr[i][u][0] + at))[32 * b * 512 / 16];
            f.x[i][u][b].hi = ((lds_v4i)(uintptr_t)(baddr[i][u][1] + at))[32 * b * 512 / 16];
        }
    };
    constexpr int SLOTS = (DENSE ? 2 : 1) * NH * 2 * RW * TW;
    // the matrix instructions of a stage; side(k) goes out behind the k-th, where a scheduling barrier holds it
    auto multiply = [&](Frag &f, int s, auto &&side) {
        int k = 0;
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            // chunks past the last have zero codes
            const bool none = 4 * s + NH * kg + i >= nchunks;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int a = 0; a < RW; ++a) {
                    if constexpr (DENSE) {
                        v4i a01, a23;
                        expand_dense_codes(none ? 0 : f.w[i][a][2 * u], none ? 0 : f.w[i][a][2 * u + 1], a01, a23);
#pragma unroll
                        for (int b = 0; b < TW; ++b) {
                            acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(a01, f.x[i][u][b], acc[a][b], 0x44444444, 0, 0);
                            side(k++);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                        for (int b = 0; b < TW; ++b) {
                            acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(a23, f.x[i][u][b], acc[a][b], (int)0xeeeeeeeeu, 0, 0);
                            side(k++);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        const v4i av = expand_codes(none ? 0 : f.w[i][a][2 + u], ones);
#pragma unroll
                        for (int b = 0; b < TW; ++b) {
                            acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(av, f.x[i][u][b], acc[a][b], (int)f.w[i][a][u], 0, 0);
                            side(k++);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
        }
    };
    auto wait_for = [&](int later) {   // all but `later` of the requested stages have landed
        if (later >= NS - 1) SBN_WAIT_VMCNT((NS - 1) * S::DMA);
        else if (NS > 5 && later == 4) SBN_WAIT_VMCNT((NS > 5 ? 4 : 0) * S::DMA);
        else if (NS > 4 && later == 3) SBN_WAIT_VMCNT((NS > 4 ? 3 : 0) * S::DMA);
        else if (NS > 3 && later == 2) SBN_WAIT_VMCNT((NS > 3 ? 2 : 0) * S::DMA);
        else if (NS > 2 && later == 1) SBN_WAIT_VMCNT((NS > 2 ? 1 : 0) * S::DMA);
        else SBN_WAIT_VMCNT(0);
    };
    // One stage: its fragments lie in `now`, stage s + 1 has landed (slot `slot`) and nobody reads the slot of stage s any
    // more.  The fragments of stage s + 1 are read under the matrix instructions of stage s.
    int slot = 0;
    auto step = [&](Frag &now, Frag &next, int s) {
        const int free = slot;
        slot = slot + 1 == NS ? 0 : slot + 1;
        const uint32_t at = (uint32_t)(slot * S::STAGE);
        const bool more = s + NS < nstage;
        multiply(now, s, [&](int m) {
            constexpr int NOPS = NREAD + S::DMA;
#pragma unroll
            for (int k = 0; k < NOPS; ++k) {
                if ((NOPS <= SLOTS ? k : k * SLOTS / NOPS) != m) continue;
                if (k < NREAD) read_one(next, at, k);
                else if (more) request_one(s + NS, free, k - NREAD);
            }
        });
        if (s + 2 < nstage) wait_for(nstage - 3 - s < NS - 2 ? nstage - 3 - s : NS - 2);
        __syncthreads();
    };
    Frag f0, f1;
    wait_for(nstage - 1);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NREAD; ++k) read_one(f0, 0, k);
    if (nstage > 1) wait_for(nstage - 2 < NS - 2 ? nstage - 2 : NS - 2);
    __syncthreads();
    int s = 0;
    for (; s + 2 < nstage; s += 2) {
        step(f0, f1, s);
        step(f1, f0, s + 1);
    }
    if (s + 1 < nstage) {
        step(f0, f1, s);
        multiply(f1, s + 1, [](int) {});
    } else {
        multiply(f0, s, [](int) {});
    }

    // ---- the sums go through LDS, 32 tokens at a time, and leave as whole rows of the tile
    __syncthreads();
    if (tid < T) scale_s[tid] = __fdiv_rn(gamma, pre);
    else if (tid - T < R) bias_s[tid - T] = pre;
    int *const red = reinterpret_cast<int *>(lds);
    const bool vec = (g.d_out & 3) == 0;
#pragma unroll
    for (int b = 0; b < TW; ++b) {
        int *const sums = red + (b & 1) * KS * S::SUMS;
#pragma unroll
        for (int a = 0; a < RW; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<v4i *>(&sums[kg * S::SUMS + r * PITCH + 32 * (RW * wr + a) + 8 * q + 4 * c]) =
                    v4i{acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
        __syncthreads();
        if (vec) {
#pragma unroll
            for (int v = tid; v < 32 * R / 4; v += S::THREADS) {
                const int tl = v / (R / 4), o = row0 + 4 * (v % (R / 4)), t = t0 + 32 * b + tl;
                if (t >= g.tokens || o >= g.d_out) continue;
                v4i sum = *reinterpret_cast<const v4i *>(&sums[tl * PITCH + 4 * (v % (R / 4))]);
#pragma unroll
                for (int k = 1; k < KS; ++k) sum += *reinterpret_cast<const v4i *>(&sums[k * S::SUMS + tl * PITCH + 4 * (v % (R / 4))]);
                const float scale = scale_s[32 * b + tl];
                v4f y = {(float)sum[0] * scale, (float)sum[1] * scale, (float)sum[2] * scale, (float)sum[3] * scale};
                if (has_bias) y += *reinterpret_cast<const v4f *>(&bias_s[o - row0]);
                __builtin_nontemporal_store(y, reinterpret_cast<v4f *>(g.Y + (int64_t)t * g.d_out + o));
                if (g.acc_out) *reinterpret_cast<v4i *>(g.acc_out + (int64_t)t * g.d_out + o) = sum;
            }
        } else {   // token rows of no whole 16 bytes leave word by word, neighbouring lanes side by side
            for (int v = tid; v < 32 * R; v += S::THREADS) {
                const int tl = v / R, o = row0 + v % R, t = t0 + 32 * b + tl;
                if (t >= g.tokens || o >= g.d_out) continue;
                int sum = 0;
#pragma unroll
                for (int k = 0; k < KS; ++k) sum += sums[k * S::SUMS + tl * PITCH + v % R];
                const float y = (float)sum * scale_s[32 * b + tl];
                g.Y[(int64_t)t * g.d_out + o] = has_bias ? y + bias_s[o - row0] : y;
                if (g.acc_out) g.acc_out[(int64_t)t * g.d_out + o] = sum;
            }
        }
    }
}

template <class S, bool DENSE>
sbn_status launch_block_as(int count, const LinearItem *items, hipStream_t stream)
{
    BlockTable tab;
    int tiles = 0;
    for (int i = 0; i < count; ++i) {
        const LinearItem &li = items[i];
        BlockItem &g = tab.it[i];
        g.xq = li.xq; g.sx = li.sx; g.packed = static_cast<const uint8_t *>(li.packed); g.gamma = li.gamma; g.bias = li.bias;
        g.Y = li.Y; g.acc_out = li.acc_out;
        g.d_in = (int)li.d_in; g.d_out = (int)li.d_out; g.tokens = (int)li.tokens;
        g.tiles_r = (int)ceil_div(li.d_out, S::R);
        g.tiles_t = (int)ceil_div(li.tokens, S::T);
        // token tiles whose int8 rows take 1.5 MB of an XCD's L2 while the weights pass
        g.group = std::min(g.tiles_t, (int)std::max<int64_t>(1, (3 << 19) / (li.d_in * S::T)));
        tab.tile0[i] = tiles;
        tiles += g.tiles_r * g.tiles_t;
    }
    for (int i = count; i <= BLOCK_ITEMS; ++i) tab.tile0[i] = tiles;
    for (int i = count; i < BLOCK_ITEMS; ++i) tab.it[i] = tab.it[0];
    static thread_local bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_block_kernel<S, DENSE>), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
        if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
        raised = true;
    }
    hipLaunchKernelGGL((gemm_block_kernel<S, DENSE>), dim3(tiles), dim3(S::THREADS), S::LDS, stream, tab);
    return check_launch("gemm_block_kernel");
}

template <class S>
sbn_status launch_block_shape(int count, const LinearItem *items, bool dense, hipStream_t stream)
{
    for (int first = 0; first < count; first += BLOCK_ITEMS) {
        const int n = std::min(count - first, BLOCK_ITEMS);
        sbn_status st = dense ? launch_block_as<S, true>(n, items + first, stream) : launch_block_as<S, false>(n, items + first, stream);
        if (st != SBN_OK) return st;
    }
    return SBN_OK;
}

// 64 x 32 (two blocks on a multiprocessor), 128 x 32 (two), 128 x 64 (one, sixteen wavefronts).  A launch of one round of blocks, for
// the first two also of two: the time is a constant and one per stage, the latter growing with the part of the device that is
// busy, for dense codes and with the outputs, and the token rows, which every XCD fetches, up to 2 MB of them.  Fitted to 220 calls
// of 96 to 2048 tokens through eleven layers (all kernels measured): 3 to 4 % off.
struct BlockFit { int R, T, rounds; float fixed, stage, busy, dense, out_mb, rows_mb; };
constexpr BlockFit BLOCK_FITS[] = {
    {64, 32, 1, 3.17f, 0.364f, 0.0f, 0.50f, 0.27f, 1.03f}, {64, 32, 2, 3.47f, 0.499f, 0.08f, 0.61f, 0.14f, 1.34f},
    {128, 32, 1, 3.27f, 0.715f, 0.09f, 0.36f, 0.10f, 1.14f}, {128, 32, 2, 4.55f, 0.798f, 0.22f, 0.73f, 0.0f, 1.68f},
    {128, 64, 1, 4.82f, 0.532f, 0.26f, 0.67f, 0.05f, 1.31f},
};

int choose_block(int count, const LinearItem *items, bool dense, float &us)
{
    us = 1e30f;
    int best = 0;
    if (count > BLOCK_ITEMS) return best;
    int64_t depth = 0, rows = 0;
    double out_mb = 0, word_mb = 0;
    for (int i = 0; i < count; ++i) {
        if (items[i].d_out % 4 != 0) word_mb += 4e-6 * (double)items[i].tokens * (double)items[i].d_out;
        depth = std::max(depth, ceil_div(items[i].d_in, 4 * CHUNK));
        rows = std::max(rows, items[i].tokens * items[i].d_in);
        out_mb += 4e-6 * (double)items[i].tokens * (double)items[i].d_out;
    }
    const int64_t cus = device_cus();
    for (const BlockFit &f : BLOCK_FITS) {
        int64_t tiles = 0;
        for (int i = 0; i < count; ++i) tiles += ceil_div(items[i].d_out, f.R) * ceil_div(items[i].tokens, f.T);
        if (ceil_div(tiles, cus) != f.rounds) continue;
        const float load = (float)(tiles - (f.rounds - 1) * cus) / (float)cus;
        const float e = f.fixed + f.stage * (float)depth * (1.0f + f.busy * load) * (dense ? 1.0f + f.dense : 1.0f) + f.out_mb * (float)out_mb + 0.3f * (float)word_mb +
                        f.rows_mb * std::min(2.0f, 1e-6f * (float)rows);
        if (e < us) { us = e; best = f.R == 64 ? 0 : f.T == 32 ? 1 : 2; }
    }
    return best;
}

}  // namespace

float gemm_block_estimate_us(int count, const LinearItem *items, bool dense)
{
    float us;
    choose_block(count, items, dense, us);
    return us;
}

int block_form_count() { return 3; }

int block_form(int count, const LinearItem *items, bool dense)
{
    float us;
    return choose_block(count, items, dense, us);
}

sbn_status launch_gemm_block(int count, const LinearItem *items, bool dense, hipStream_t stream, int form)
{
    if (form < 0) form = block_form(count, items, dense);
    switch (form) {
    case 0: return launch_block_shape<BlockShape<2, 4, 1, 1, 3>>(count, items, dense, stream);
    case 1: return launch_block_shape<BlockShape<4, 2, 1, 1, 2>>(count, items, dense, stream);
    case 2: return launch_block_shape<BlockShape<4, 4, 1, 2, 3>>(count, items, dense, stream);
    }
    return SBN_EINVAL;
}

}  // namespace sbn
