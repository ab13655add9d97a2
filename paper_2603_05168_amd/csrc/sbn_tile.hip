// Forward product of the N:M-sparse ternary linear layer in small block tiles (Section 2.2 forward-pass equation): decode
// batches and short prompts through a layer or a few, where the large tiles of the streaming and the GEMM kernel leave most
// multiprocessors idle (a 2560 x 2560 layer is 20 strips or 5 row tiles to them).
//
// A block owns 16 RT rows of W and 16 TT tokens over the whole input dimension, and its wavefronts split that dimension:
// stage s (256 weights) goes to wavefront s % NW.  A wavefront brings its stages into a part of LDS of its own (LDS-DMA,
// whole lines of the token rows), reads the fragments into registers, asks for its next stage at once and multiplies; no
// wavefront waits for another before the end, where the partial sums meet in LDS.
// What bounds it: up to some 300 blocks the chain request - stage - reduce - store of a single block (about 2.5 us, on top
// of 2 us that any launch costs), beyond that the 105 bytes/ns that LDS-DMA deposits per multiprocessor, reached to 65 %:
// the time a block waits for its first stage and for its last store is covered by other blocks only, so four wavefronts
// (48 KB) per block, three blocks per multiprocessor, beat eight of them with one (40 against 23.5 us at 777 x 2560 ->
// 6912).  Operands loaded straight into registers in the instruction's layout (consecutive lanes = rows) pass the vector
// L1 at 16 bytes per clock and were up to twice as slow (57 us there).
// Measured, us per launch behind the quantizer, weights from memory, 2:4 (the faster of the two kernels named in
// launch_gemm_smfmac -> this one; in brackets where that one is chosen):
//   tokens               32           64          128          256            512            777           1024
//   2560 -> 2560   9.7 -> 4.7  12.9 -> 5.2  13.7 -> 6.3  14.0 -> 8.3    14.0 -> 11.1  (13.8 -> 14.9) (14.1 -> 18.0)
//   2560 -> 6912  10.4 -> 6.0  14.2 -> 7.3  17.4 -> 8.7  17.8 -> 13.5  (17.8 -> 20.5) (19.7 -> 27.2) (21.3 -> 33.4)
//   6912 -> 2560  18.4 -> 7.0  27.1 -> 8.6  40.8 -> 10.5 41.5 -> 14.1   40.2 -> 21.1   38.8 -> 26.3   39.8 -> 29.8
#include <algorithm>

#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

struct TileItem {
    const int8_t *xq;
    const float *sx;
    const uint8_t *packed;
    const float *gamma;
    const float *bias;
    float *Y;
    int32_t *acc_out;
    int d_in, d_out, tokens;
    int strips8;           // row strips of an XCD
};
template <int NI>
struct TileTable {
    TileItem it[NI];
    int block0[NI + 1];   // first block of each problem; entries past the last problem hold the total
};
constexpr int TILE_FEW = 4, TILE_MANY = 40;
static_assert(sizeof(TileTable<TILE_MANY>) <= 4096, "the table travels as a kernel argument");
constexpr int TILE_NW = 8;   // wavefronts of a block at most

template <int RT, int TT> struct TileShape {
    static constexpr int R = 16 * RT, T = 16 * TT;      // rows of W and tokens of a block
    static constexpr int ABYTES = R * 64, BBYTES = T * 256, STAGE = ABYTES + BBYTES;   // one stage of one wavefront: 256 weights deep
    static constexpr int PITCH = R + 4;                 // 32-bit words between the token rows of a partial tile in LDS
    static_assert(T * PITCH * 4 <= STAGE, "a wavefront's partial sums fit where its operands were");
};

template <int RT, int TT, bool DENSE, int NI>
__global__ void __launch_bounds__(64 * TILE_NW) gemm_tile_kernel(TileTable<NI> tab)
{
    using S = TileShape<RT, TT>;
    constexpr int R = S::R, PITCH = S::PITCH;
    extern __shared__ __attribute__((aligned(1024))) int8_t lds[];   // [wavefront][stage], later [wavefront][token][PITCH] words
    __shared__ __attribute__((aligned(16))) float scale_s[S::T], bias_s[R];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
    int p = 0;
    while (p + 1 < NI && (int)blockIdx.x >= tab.block0[p + 1]) ++p;
    const TileItem &g = tab.it[p];
    // Blocks go round-robin to the eight XCDs, each with an L2 of its own: an XCD takes every eighth row strip, all of its
    // strips for one token tile before the next tile, so its share of the weights (an eighth of 4.4 MB for 2560 x 6912)
    // stays in its L2 and the activations pass through it once.  With the tiles of a strip following each other instead,
    // 777 x 6912 int8 rows (5.4 MB) went through every L2 once per strip: 36 us against 22.6.
    const int local = (int)blockIdx.x - tab.block0[p], strip = (local & 7) + 8 * ((local >> 3) % g.strips8), tt = (local >> 3) / g.strips8;
    const int row0 = strip * R, t0 = tt * S::T;
    if (row0 >= g.d_out) return;
    const int r = lane & 15, q = lane >> 4;
    const uint32_t ones = vgpr_ones();
    const int K = g.d_in, nchunks = K / CHUNK, nstage = (nchunks + 1) >> 1;
    const uint32_t lds0 = lds_address(lds) + wave * S::STAGE;
    // gamma / s_x of the block's tokens and the bias of its rows: asked for in front of everything else, put into LDS for
    // the epilogue once the main loop is over
    float pre = 0.0f, gamma = 0.0f;
    const int tid = (int)threadIdx.x;
    const bool has_bias = g.bias != nullptr;
    if (tid < S::T) {
        pre = g.sx[t0 + tid < g.tokens ? t0 + tid : g.tokens - 1];
        gamma = *g.gamma;
    } else if (has_bias && tid - S::T < R) {
        pre = g.bias[row0 + tid - S::T < g.d_out ? row0 + tid - S::T : g.d_out - 1];
    }

    // DMA roles.  Weights: one instruction fills 16 rows of 64 bytes (two chunks), slot l % 4 of a row holds granule
    // (l % 4) ^ ((row >> 2) & 3).  Tokens: one instruction fills 4 rows of 256 bytes, slot l % 16 holds granule
    // (l % 16) ^ (row & 15).  Rows past the matrix: its last row again (never stored).
    const uint8_t *wbase = g.packed + (int64_t)row0 * nchunks * 32;
    const int8_t *xbase = g.xq + (int64_t)t0 * K;
    uint32_t woff[RT], xoff[4 * TT];
    uint32_t wgran[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int row = 16 * i + (lane >> 2), o = row0 + row < g.d_out ? row : g.d_out - 1 - row0;
        wgran[i] = (lane & 3) ^ ((row >> 2) & 3);
        woff[i] = (uint32_t)o * (uint32_t)(nchunks * 32) + 16u * wgran[i];
    }
#pragma unroll
    for (int i = 0; i < 4 * TT; ++i) {
        const int row = 4 * i + (lane >> 4), t = t0 + row < g.tokens ? row : g.tokens - 1 - t0;
        xoff[i] = (uint32_t)t * (uint32_t)K + 16u * ((lane & 15) ^ (row & 15));
    }
    auto request = [&](int s) {
        const uint8_t *wb = wbase + (int64_t)s * 64;
        const int8_t *xb = xbase + (int64_t)s * 256;
        const bool half = 2 * s + 1 >= nchunks;   // the stage's second chunk does not exist: its first again (meets zero codes)
#pragma unroll
        for (int i = 0; i < RT; ++i) lds_dma16(wb, half && wgran[i] >= 2 ? woff[i] - 32u : woff[i], lds0 + 1024 * i);
#pragma unroll
        for (int i = 0; i < 4 * TT; ++i) {
            const uint32_t gran = (lane & 15) ^ ((4 * i + (lane >> 4)) & 15);
            lds_dma16(xb, half && gran >= 8 ? xoff[i] - 128u : xoff[i], lds0 + S::ABYTES + 1024 * i);
        }
    };

    v4i acc[RT][TT];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int b = 0; b < TT; ++b) acc[a][b] = v4i{0, 0, 0, 0};

    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v2u *lds_v2u;
    typedef __attribute__((address_space(3))) const v4u *lds_v4u;
    if (wave < nstage) request(wave);
    for (int s = wave; s < nstage; s += nw) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        v4u w4[RT];          // 2:4: index words 2 (q & 1) + {0, 1} of chunk q >> 1, then the code words; dense: words of granule q
        v4i x[TT][4];
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            const uint32_t row = lds0 + (16 * a + r) * 64;
            const uint32_t sw = (r >> 2) & 3;
            if constexpr (DENSE) {
                w4[a] = *(lds_v4u)(uintptr_t)(row + 16 * (q ^ sw));
            } else {
                const v2u iv = *(lds_v2u)(uintptr_t)(row + 16 * ((2 * (q >> 1)) ^ sw) + 8 * (q & 1));
                const v2u cv = *(lds_v2u)(uintptr_t)(row + 16 * ((2 * (q >> 1) + 1) ^ sw) + 8 * (q & 1));
                w4[a] = v4u{iv.x, iv.y, cv.x, cv.y};
            }
        }
#pragma unroll
        for (int b = 0; b < TT; ++b) {
            const uint32_t row = lds0 + S::ABYTES + (16 * b + r) * 256;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // 2:4: j = 2 u + upper: 16 bytes at 64 (q >> 1) + 16 (q & 1) + 32 u + 128 upper; dense: at 64 q + 16 j
                const uint32_t gran = DENSE ? 4 * q + j : 4 * (q >> 1) + (q & 1) + 2 * (j >> 1) + 8 * (j & 1);
                x[b][j] = *(lds_v4i)(uintptr_t)(row + 16 * (gran ^ (r & 15)));
            }
        }
        if (2 * s + 1 >= nchunks && q >= 2) {
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                w4[a].z = w4[a].w = 0;
                if constexpr (DENSE) w4[a].x = w4[a].y = 0;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // everything is in registers: the stage can be filled again
        if (s + nw < nstage) request(s + nw);
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            if constexpr (DENSE) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const v4i av = expand_codes(w4[a][j], ones);
#pragma unroll
                    for (int b = 0; b < TT; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, x[b][j], acc[a][b], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const v4i av = expand_codes(w4[a][2 + u], ones);
#pragma unroll
                    for (int b = 0; b < TT; ++b) {
                        const v4i l = x[b][2 * u], h = x[b][2 * u + 1];
                        const v8i bv = {l[0], l[1], l[2], l[3], h[0], h[1], h[2], h[3]};
                        acc[a][b] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(av, bv, acc[a][b], (int)w4[a][u], 0, 0);
                    }
                }
            }
        }
    }
    int *const red = reinterpret_cast<int *>(lds);
    constexpr int WRED = S::STAGE / 4;                 // words between two wavefronts' partial sums
    constexpr int VECS = S::T * R / 4;                 // 16-byte vectors of the tile's sums

    // ---- the wavefronts' partial sums meet in LDS; whole token rows of the strip leave
    if (tid < S::T) scale_s[tid] = __fdiv_rn(gamma, pre);
    else if (tid - S::T < R) bias_s[tid - S::T] = pre;
    const bool vec = (g.d_out & 3) == 0;
#pragma unroll
    for (int b = 0; b < TT; ++b)
#pragma unroll
        for (int a = 0; a < RT; ++a)   // lane: token r of its tile, rows 4 q .. + 3
            *reinterpret_cast<v4i *>(&red[wave * WRED + (16 * b + r) * PITCH + 16 * a + 4 * q]) = acc[a][b];
    __syncthreads();
    for (int v = threadIdx.x; v < VECS; v += (int)blockDim.x) {
        const int tl = v / (R / 4), o = row0 + 4 * (v % (R / 4)), t = t0 + tl;
        if (t >= g.tokens || o >= g.d_out) continue;
        v4i sum = *reinterpret_cast<const v4i *>(&red[tl * PITCH + 4 * (v % (R / 4))]);
        for (int w = 1; w < nw; ++w) sum += *reinterpret_cast<const v4i *>(&red[w * WRED + tl * PITCH + 4 * (v % (R / 4))]);
        const float scale = scale_s[tl];
        v4f y = {(float)sum[0] * scale, (float)sum[1] * scale, (float)sum[2] * scale, (float)sum[3] * scale};
        float *dst = g.Y + (int64_t)t * g.d_out + o;
        if (vec) {
            if (has_bias) y += *reinterpret_cast<const v4f *>(&bias_s[o - row0]);
            *reinterpret_cast<v4f *>(dst) = y;
            if (g.acc_out) *reinterpret_cast<v4i *>(g.acc_out + (int64_t)t * g.d_out + o) = sum;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (o + i < g.d_out) {
                    dst[i] = has_bias ? y[i] + bias_s[o - row0 + i] : y[i];
                    if (g.acc_out) g.acc_out[(int64_t)t * g.d_out + o + i] = sum[i];
                }
        }
    }
}

template <int RT, int TT, bool DENSE, int NI>
sbn_status launch_tile_as(int count, const LinearItem *items, int max_nw, hipStream_t stream)
{
    TileTable<NI> tab;
    using S = TileShape<RT, TT>;
    int blocks = 0, most = 1;
    for (int i = 0; i < count; ++i) {
        const LinearItem &li = items[i];
        TileItem &g = tab.it[i];
        g.xq = li.xq; g.sx = li.sx; g.packed = static_cast<const uint8_t *>(li.packed); g.gamma = li.gamma; g.bias = li.bias;
        g.Y = li.Y; g.acc_out = li.acc_out;
        g.d_in = (int)li.d_in; g.d_out = (int)li.d_out; g.tokens = (int)li.tokens;
        g.strips8 = (int)ceil_div(ceil_div(li.d_out, 16 * RT), 8);
        tab.block0[i] = blocks;
        blocks += 8 * g.strips8 * (int)ceil_div(li.tokens, 16 * TT);
        const int nstage = (int)ceil_div(li.d_in, 2 * CHUNK);
        most = nstage > most ? nstage : most;
    }
    for (int i = count; i <= NI; ++i) tab.block0[i] = blocks;
    for (int i = count; i < NI; ++i) tab.it[i] = tab.it[0];
    // as few wavefronts as walk the stages in the same number of rounds, but a thread for every scale and bias of the tile (a
    // wavefront without a stage adds zeros)
    const int rounds = (int)ceil_div(most, max_nw), nw = std::max((int)ceil_div(most, rounds), (S::T + S::R + 63) / 64);
    const size_t lds = (size_t)nw * S::STAGE;
    static thread_local bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_tile_kernel<RT, TT, DENSE, NI>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TILE_NW * S::STAGE);
        if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
        raised = true;
    }
    hipLaunchKernelGGL((gemm_tile_kernel<RT, TT, DENSE, NI>), dim3(blocks), dim3(64 * nw), lds, stream, tab);
    return check_launch("gemm_tile_kernel");
}

template <int RT, int TT>
sbn_status launch_tile_shape(int count, const LinearItem *items, bool dense, int max_nw, hipStream_t stream)
{
    for (int first = 0; first < count; first += TILE_MANY) {
        const int n = count - first < TILE_MANY ? count - first : TILE_MANY;
        const LinearItem *it = items + first;
        // a launch of a few problems carries a short table: the 3 KB of a long one cost the host a microsecond
        sbn_status st = n <= TILE_FEW ? (dense ? launch_tile_as<RT, TT, true, TILE_FEW>(n, it, max_nw, stream) : launch_tile_as<RT, TT, false, TILE_FEW>(n, it, max_nw, stream))
                                      : (dense ? launch_tile_as<RT, TT, true, TILE_MANY>(n, it, max_nw, stream) : launch_tile_as<RT, TT, false, TILE_MANY>(n, it, max_nw, stream));
        if (st != SBN_OK) return st;
    }
    return SBN_OK;
}

// tiles of 64 rows x 32 tokens
int64_t wide_tiles(const LinearItem &li) { return ceil_div(li.d_out, 64) * ceil_div(li.tokens, 32); }

}  // namespace

// Estimated time of a call on this kernel in us: the chain of one block (768 weights 3.6 us, from 1620 on 4.5); per tile of 64 x
// 32 and multiprocessor 0.59 us for its sums and outputs and 1.46 us (dense codes 1.54) per 2560 weights for its deposits; the
// weights once from memory at 6 TB/s; and the activations, which the quantizer or another kernel has just written and which every
// XCD fetches from memory before its L2 has them, 1.3 us per MB up to 2.6 us, from where on the rounds of tiles cover it.  (Behind
// a quantizer, its own time subtracted: 512 / 777 / 1024 tokens 2560 -> 2560 11.1 / 14.9 / 18.0 us; on rows that lie in the L2 9.5 / 12.3 / 14.5.)
// With up to eight row tiles in all, the rounds are too short to cover it: another 0.4 us per MB beyond 2 MB (4000 tokens, 2560 ->
// 512: 20.6 us, 6912 -> 512 35.5; with 24 row tiles, 2560 -> 1500, nothing).  Outputs stored in single words: 0.1 us per MB.
float gemm_tile_estimate_us(int count, const LinearItem *items, bool dense)
{
    double us = 0, chain = 0, rows_mb = 0;
    int64_t row_tiles = 0;
    for (int i = 0; i < count; ++i) {
        const double k = (double)items[i].d_in;
        row_tiles += ceil_div(items[i].d_out, 64);
        if (items[i].d_out % 4 != 0) us += 0.4e-6 * (double)items[i].tokens * (double)items[i].d_out;
        chain = std::max(chain, 2.7 + std::min(1.8, k / 900.0));
        rows_mb = std::max(rows_mb, 1e-6 * k * (double)items[i].tokens);
        us += (double)wide_tiles(items[i]) / (double)device_cus() * (0.59 + (dense ? 1.54 : 1.46) * k / 2560.0) + (double)items[i].d_out * k / 4 / 6e6;
    }
    if (row_tiles <= 8) us += 0.4 * std::max(0.0, rows_mb - 2.0);
    return (float)(us + chain + std::min(2.6, 1.3 * rows_mb));
}

// Tile shape: 64 x 32 moves the fewest bytes per product and takes over where it gives most multiprocessors a tile
// (from 25 for 32 multiprocessors on, 200 on 256; 128 tokens, 6912 -> 2560: 160 tiles, 8.3 us against 9.2 with 32 x 32, but 2560 -> 2560 6.1 against 5.5 with
// 32 x 16); below that smaller tiles, 32 x 16 up to 32 tokens (32 tokens, 6912 -> 2560: 5.7 us against 6.7 with 32 x 32), 32 x 32
// beyond (64 tokens: 6.7 against 7.6 with 32 x 16).  Eight wavefronts walk the stages in fewer rounds and are faster while a
// multiprocessor has one block (64 tokens, 6912 -> 2560: 6.7 us against 7.3 with four), four leave room for more blocks
// (256 tokens, 2560 -> 2560: 7.4 us against 9.6).
sbn_status launch_gemm_tile(int count, const LinearItem *items, bool dense, hipStream_t stream)
{
    int64_t wide = 0, tokens = 0, square = 0;
    for (int i = 0; i < count; ++i) {
        wide += wide_tiles(items[i]);
        square += ceil_div(items[i].d_out, 32) * ceil_div(items[i].tokens, 32);
        tokens = items[i].tokens > tokens ? items[i].tokens : tokens;
    }
    if (32 * wide >= 25 * (int64_t)device_cus()) return launch_tile_shape<4, 2>(count, items, dense, 4, stream);
    if (tokens <= 32) return launch_tile_shape<2, 1>(count, items, dense, 8, stream);
    return launch_tile_shape<2, 2>(count, items, dense, square <= device_cus() ? 8 : 4, stream);
}

}  // namespace sbn
