// Decode batches and short prompts in one launch, the activation quantizer inside (Section 2.1 quantizer, Section 2.2
// forward-pass equation): calls that want nothing but Y (and the accumulators) and need no quantized rows back.
//
// A block owns R rows of W and T = 4, 8 or 16 tokens over the whole input dimension.  A wavefront reads one whole token row (its
// largest magnitude needs no other wavefront and no barrier), quantizes it into LDS, and after the one barrier multiplies its
// part of the weights, which LDS-DMA has brought into a part of LDS of its own; the partial sums meet in LDS and leave as whole
// rows of the strip.  Every block repeats the quantizer for its tokens: 24 vector instructions per eight values, 0.5 us per
// block at 16 tokens of 2560 values, against a launch in front (2.5 us on the device, 2.5 to 3 on the host).
// What bounds it: the chain launch - row - quantize - barrier - multiply - sums - store (3 us), then the bytes of a block, which
// a multiprocessor takes in at 45 to 55 bytes/ns while they come from memory or the last-level cache.  Hence
//   * LDS-DMA of 128 contiguous bytes of a weight row (512 weights).  Pieces of 64 bytes cost the same time as whole lines (62
//     against 108 bytes/ns out of the L2, 31 against 44 from memory), and loads into registers in the instruction's layout, where
//     consecutive lanes are different rows, 20 bytes/ns: 2560 -> 2560 at 32 tokens 7.5 us with those, 5.9 with 64-byte pieces, 5.7;
//   * the weights are asked for behind the maxima: the compiler waits for the last token values with everything that was
//     asked for since, so in front of them the weights would be waited for too (64 tokens, 2560 -> 2560: 6.1 against 5.8 us);
//   * blocks whose bytes and quantizing balance and which fill the device once (the shapes below and choose()).
// Measured, us per call, quantizer included, weights from memory, 2:4 (before: quantizer launch and the kernels of
// launch_gemm_smfmac, up to 16 tokens gemv_self_kernel -> now):
//   tokens              8            16           32           64           128          256
//   2560 -> 2560        4.8 -> 4.5   6.1 -> 4.5   7.2 -> 4.9   7.8 -> 5.8   8.8 -> 6.3   11.0 -> 8.0
//   2560 -> 3 x 2560    5.3 -> 4.8   6.5 -> 5.1   7.7 -> 6.1   9.2 -> 6.5   10.6 -> 7.9  16.7 -> 14.4
//   2560 -> 2 x 6912    6.9 -> 5.4   9.2 -> 6.4   9.5 -> 6.6   10.6 -> 8.0  15.1 -> 13.7 (21.8 / 25.9)
//   6912 -> 2560        6.9 -> 6.8   9.4 -> 7.0   8.9 -> 8.4   11.0 -> 9.6  (13.3 / 14.0)
#include <algorithm>
#include <type_traits>

#include "sbn_decode.hpp"
#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

constexpr int SELF_ITEMS = 8;   // problems of a launch
struct SelfItem {
    const uint4 *X;
    const uint8_t *packed;
    const float *gamma;
    const float *bias;
    float *Y;
    int32_t *acc_out;
    int d_in, d_out, tokens;
    int nvec;              // 16-byte vectors of a row of X
    int groups;            // token groups of a block's size
    int depth;             // super-steps of weights that a wavefront's part of LDS holds
};
struct SelfTable {
    SelfItem it[SELF_ITEMS];
    int unit0[SELF_ITEMS + 1];   // first block of each problem; entries past the last problem hold the total
};
constexpr size_t SELF_LDS = 160 * 1024 - 256;   // beside the scales
constexpr int SELF_MAX_ROW = 8192;              // values of a row of X at most: 16 vectors of a lane

// bytes between the int8 rows in LDS: whole super-steps, and 16 more so that 16 rows lie in different banks
constexpr int self_pitch(int64_t d_in) { return (int)((d_in + 511) / 512 * 512 + 16); }

// RT row tiles of 16 for each of G groups of wavefronts, whose KS wavefronts split the input dimension; T tokens, one or TPW for
// each wavefront to quantize; XV = 16-byte vectors of a row per lane at most
template <int RT_, int G_, int T_, int WAVES_, int XV_> struct SelfShape {
    static constexpr int RT = RT_, G = G_, T = T_, WAVES = WAVES_, XV = XV_;
    static constexpr int R = 16 * RT * G, KS = WAVES / G, TPW = T / WAVES, PITCH = R + 4;
    static constexpr int STAGE = 16 * RT * 128;   // bytes of a wavefront's super-step: 512 weights of its rows
    static_assert(KS * G == WAVES && TPW * WAVES == T, "every wavefront has rows and tokens");
};

template <int DPP> __device__ __forceinline__ uint32_t dpp_max(uint32_t m)
{
    const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)m, DPP, 0xf, 0xf, true);
    return o > m ? o : m;
}

template <class S, bool DENSE>
__global__ void __launch_bounds__(64 * S::WAVES) gemm_self_kernel(SelfTable tab)
{
    constexpr int R = S::R, T = S::T, RT = S::RT, KS = S::KS, TPW = S::TPW, XV = S::XV, PITCH = S::PITCH;
    extern __shared__ __attribute__((aligned(16))) int8_t dyn[];   // int8 rows, the wavefronts' weights; later [K part][token][PITCH] sums
    __shared__ float scale_s[T];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // blocks go round-robin to the eight XCDs: XCD x takes the x-th of eight runs of consecutive units, in which the token groups
    // of a row strip follow each other, so that its weights come from memory once
    const int total = (int)gridDim.x, x8 = (int)blockIdx.x & 7, rem8 = total & 7;
    const int unit = x8 * (total >> 3) + (x8 < rem8 ? x8 : rem8) + ((int)blockIdx.x >> 3);
    int p = 0;
    while (p + 1 < SELF_ITEMS && unit >= tab.unit0[p + 1]) ++p;
    const SelfItem &it = tab.it[p];
    const int local = unit - tab.unit0[p], row0 = local / it.groups * R, t0 = T * (local % it.groups);
    const int K = it.d_in, nchunks = K / CHUNK, nvec = it.nvec, xpitch = self_pitch(K);
    const int r = lane & 15, c4 = lane >> 4;
    const int group = wave % S::G, part = wave / S::G;
    const uint32_t ones = vgpr_ones();

    // The token rows of this wavefront, unconditional: past the row and past the tokens the loads lie past the end of the buffer,
    // where they return zeros and fetch nothing.
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(it.X) + (int64_t)t0 * nvec, (short)0, (it.tokens - t0) * nvec * 16, 0x00027000);
    uint4 xv[TPW][XV];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            const int vec = 64 * i + lane;
            const uint32_t at = vec < nvec ? 16u * (uint32_t)((TPW * wave + t) * nvec + vec) : 0x7ffffff0u;
            xv[t][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rows, at, 0, 0));
        }
    const float gamma = *it.gamma;

    // Weights: super-step j of this wavefront (part + KS j of all) is 512 weights of its rows in a part of LDS of its own, filled by
    // LDS-DMA instructions of 8 rows x 128 bytes (slot l % 8 of a row holds granule (l % 8) ^ ((row >> 1) & 7)).
    const int nsuper = (nchunks + 3) >> 2, steps = nsuper > part ? (nsuper - part + KS - 1) / KS : 0;
    const int prow = row0 + 16 * RT * group < it.d_out ? row0 + 16 * RT * group : it.d_out - 1;   // a group past the matrix: its last row
    const uint8_t *const wbase = it.packed + (int64_t)prow * nchunks * 32;
    int8_t *const wdyn = dyn + T * xpitch + wave * (it.depth * S::STAGE);
    const uint32_t wlds = lds_address(wdyn);
    uint32_t woff[2 * RT], wchunk[2 * RT];
#pragma unroll
    for (int i = 0; i < 2 * RT; ++i) {
        const int row = 8 * i + (lane >> 3), left = it.d_out - prow, gran = (lane & 7) ^ ((row >> 1) & 7);
        woff[i] = (uint32_t)((row < left ? row : left - 1) * nchunks * 32 + 16 * gran);
        wchunk[i] = gran >> 1;
    }
    auto request = [&](int j, int slot) {
        const int st = part + KS * j;
#pragma unroll
        for (int i = 0; i < 2 * RT; ++i)   // chunks past the row: the super-step's first again (meets zero codes)
            lds_dma16(wbase + (int64_t)st * 128, 4 * st + (int)wchunk[i] < nchunks ? woff[i] : woff[i] - 32u * wchunk[i], wlds + slot * S::STAGE + 1024 * i);
    };

    // ---- the rows' scales and int8 values
    float s[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        uint32_t m2 = 0;
#pragma unroll
        for (int i = 0; i < XV; ++i) m2 = max_u16x2(m2, absmax_pair_bf16x8(xv[t][i]));
        uint32_t m = m2 >> 16 > (m2 & 0xffffu) ? m2 >> 16 : m2 & 0xffffu;
        m = dpp_max<0x121>(m);   // row_ror 1, 2, 4, 8
        m = dpp_max<0x122>(m);
        m = dpp_max<0x124>(m);
        m = dpp_max<0x128>(m);
        const auto x16 = __builtin_amdgcn_permlane16_swap(m, m, false, false);
        m = x16[0] > x16[1] ? x16[0] : x16[1];
        const auto x32 = __builtin_amdgcn_permlane32_swap(m, m, false, false);
        m = x32[0] > x32[1] ? x32[0] : x32[1];
        asm volatile("" : "+v"(m));   // the requests below stand behind the maxima
        s[t] = scale_from_absmax_bits(m);
    }
    for (int j = 0; j < it.depth; ++j)
        if (j < steps) request(j, j);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        if (lane == 0) scale_s[TPW * wave + t] = __fdiv_rn(gamma, s[t]);
        int8_t *const xs = dyn + (TPW * wave + t) * xpitch + 8 * lane;
#pragma unroll
        for (int i = 0; i < XV; ++i)
            if (64 * i + lane < nvec) *reinterpret_cast<uint2 *>(xs + 512 * i) = quantize_bf16x8(xv[t][i], s[t]);
    }
    __syncthreads();

    v4i acc[RT];
#pragma unroll
    for (int a = 0; a < RT; ++a) acc[a] = v4i{0, 0, 0, 0};
    const int8_t *const xr = dyn + (r & (T - 1)) * xpitch;   // columns past the tokens repeat them (not stored)
    int slot = 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (int j = 0; j < steps; ++j) {
        const int st = part + KS * j;
        if (j >= it.depth) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        uint4 idx4[RT], code4[RT];   // the lane's chunk
        const bool in = 4 * st + c4 < nchunks;
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            const int8_t *row = wdyn + slot * S::STAGE + (16 * a + r) * 128;
            idx4[a] = *reinterpret_cast<const uint4 *>(row + 16 * ((2 * c4) ^ ((r >> 1) & 7)));
            code4[a] = *reinterpret_cast<const uint4 *>(row + 16 * ((2 * c4 + 1) ^ ((r >> 1) & 7)));
            if (!in) {   // past the row zero codes
                if constexpr (DENSE) idx4[a] = make_uint4(0, 0, 0, 0);
                code4[a] = make_uint4(0, 0, 0, 0);
            }
        }
        if (j + it.depth < steps) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // in registers: the slot can be filled again
            request(j + it.depth, slot);
        }
        slot = slot + 1 == it.depth ? 0 : slot + 1;
        gemv_super_step<DENSE ? GEMV_DENSE : GEMV_2OF4, RT>(idx4, code4, xr + 512 * st, c4, ones, [](int k) { return k; }, acc);
    }

    // ---- sums through LDS, whole rows of the strip leave
    int *const red = reinterpret_cast<int *>(dyn);
    __syncthreads();
#pragma unroll
    for (int a = 0; a < RT; ++a)   // lane: token r, rows 4 c4 ..
        if (r < T) *reinterpret_cast<v4i *>(&red[(part * T + r) * PITCH + 16 * (RT * group + a) + 4 * c4]) = acc[a];
    __syncthreads();
    const bool has_bias = it.bias != nullptr;
    if ((it.d_out & 3) == 0) {
        for (int v = tid; v < T * R / 4; v += 64 * S::WAVES) {
            const int tl = v / (R / 4), o = row0 + 4 * (v % (R / 4)), t = t0 + tl;
            if (t >= it.tokens || o >= it.d_out) continue;
            v4i sum = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < KS; ++k) sum += *reinterpret_cast<const v4i *>(&red[(k * T + tl) * PITCH + 4 * (v % (R / 4))]);
            const float scale = scale_s[tl];
            v4f y = {(float)sum[0] * scale, (float)sum[1] * scale, (float)sum[2] * scale, (float)sum[3] * scale};
            if (has_bias)
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] += it.bias[o + i];
            *reinterpret_cast<v4f *>(it.Y + (int64_t)t * it.d_out + o) = y;
            if (it.acc_out) *reinterpret_cast<v4i *>(it.acc_out + (int64_t)t * it.d_out + o) = sum;
        }
    } else {   // token rows of no whole 16 bytes leave word by word, neighbouring lanes side by side
        for (int v = tid; v < T * R; v += 64 * S::WAVES) {
            const int tl = v / R, o = row0 + v % R, t = t0 + tl;
            if (t >= it.tokens || o >= it.d_out) continue;
            int sum = 0;
#pragma unroll
            for (int k = 0; k < KS; ++k) sum += red[(k * T + tl) * PITCH + v % R];
            const float y = (float)sum * scale_s[tl];
            it.Y[(int64_t)t * it.d_out + o] = has_bias ? y + it.bias[o] : y;
            if (it.acc_out) it.acc_out[(int64_t)t * it.d_out + o] = sum;
        }
    }
}

template <class S, bool DENSE>
sbn_status launch_self_as(int count, const LinearItem *items, hipStream_t stream)
{
    SelfTable tab;
    int blocks = 0, pitch = 0, depth = 1;
    for (int i = 0; i < count; ++i) {
        const LinearItem &li = items[i];
        SelfItem &g = tab.it[i];
        g.X = static_cast<const uint4 *>(li.X); g.packed = static_cast<const uint8_t *>(li.packed); g.gamma = li.gamma; g.bias = li.bias;
        g.Y = li.Y; g.acc_out = li.acc_out;
        g.d_in = (int)li.d_in; g.d_out = (int)li.d_out; g.tokens = (int)li.tokens;
        g.nvec = (int)li.row_values() / 8;
        g.groups = (int)ceil_div(li.tokens, S::T);
        tab.unit0[i] = blocks;
        blocks += (int)ceil_div(li.d_out, S::R) * g.groups;
        pitch = std::max(pitch, self_pitch(li.d_in));
        depth = std::max(depth, (int)ceil_div(ceil_div(li.d_in, 4 * CHUNK), S::KS));
    }
    // all super-steps of the weights where they fit; more blocks than multiprocessors leave room for a second block if the rows allow it
    const size_t rows = (size_t)S::T * pitch, stages = S::WAVES * S::STAGE;
    const size_t room = blocks > device_cus() && rows + stages <= SELF_LDS / 2 ? SELF_LDS / 2 : SELF_LDS;
    if (rows + stages > room) return SBN_EUNSUPPORTED;   // cannot happen: choose() has looked at the same sum
    depth = std::min(depth, (int)((room - rows) / stages));
    for (int i = 0; i < count; ++i) tab.it[i].depth = depth;
    for (int i = count; i <= SELF_ITEMS; ++i) tab.unit0[i] = blocks;
    for (int i = count; i < SELF_ITEMS; ++i) tab.it[i] = tab.it[0];
    const size_t lds = std::max(rows + depth * stages, (size_t)S::KS * S::T * S::PITCH * 4);
    static thread_local bool raised = false;
    if (!raised) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_self_kernel<S, DENSE>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)SELF_LDS);
        if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
        raised = true;
    }
    hipLaunchKernelGGL((gemm_self_kernel<S, DENSE>), dim3(blocks), dim3(64 * S::WAVES), lds, stream, tab);
    return check_launch("gemm_self_kernel");
}

template <int RT, int G, int T, int WAVES>
sbn_status launch_self_shape(int count, const LinearItem *items, bool dense, hipStream_t stream)
{
    int64_t longest = 0;
    for (int i = 0; i < count; ++i) longest = std::max(longest, items[i].row_values());
    auto launch = [&](auto xv) {
        using S = SelfShape<RT, G, T, WAVES, xv()>;
        return dense ? launch_self_as<S, true>(count, items, stream) : launch_self_as<S, false>(count, items, stream);
    };
    return longest <= 2560   ? launch(std::integral_constant<int, 5>())
           : longest <= 4096 ? launch(std::integral_constant<int, 8>())
                             : launch(std::integral_constant<int, 16>());
}

// The shapes, rows x tokens; the comment says where each is the fastest (2:4, weights from memory).
struct SelfForm { int RT, G, T, WAVES; };
constexpr SelfForm SELF_FORMS[] = {
    {1, 1, 4, 4},     // 16 x 4: few rows and tokens (1280 -> 512 at 16 tokens 3.0 us, 3.4 with the next)
    {2, 2, 4, 4},     // 64 x 4: wider ones (512 -> 8192 at 8 tokens 3.5)
    {2, 1, 8, 8},     // 32 x 8: one group of tokens (2560 -> 2560 at 16 tokens 4.5, 4.8 with the next)
    {2, 2, 8, 8},     // 64 x 8
    {3, 2, 8, 8},     // 96 x 8: long rows at 64 tokens (6912 -> 2560 9.6, 11.0 with 64 x 8 or 128 x 8)
    {2, 4, 8, 8},     // 128 x 8
    {2, 4, 16, 16},   // 128 x 16: 64 tokens, 2560 -> 3 x 2560 6.5 (7.6 with 128 x 8)
    {2, 8, 16, 16},   // 256 x 16: 64 tokens, 2560 -> 2 x 6912 8.0 (more than one round of the device with the others)
};

// Estimated time in us of a call in one shape: the chain; the rows of a block's tokens (of which the quantizer is a part) and its
// weights, which take up to 1.6 times as long with the whole device reading; the steps of a wavefront; a further block of
// a multiprocessor, 0.7 of the first where two are resident, 1.1 where not; the outputs, more where they are stored in
// single words.  Fitted to 315 calls of 1 to 384
// tokens, 512 to 8192 values and 512 to 28672 outputs, all shapes measured: 8 % off, and the shape it picks is 0.9 % from the fastest.
float self_estimate_us(const SelfForm &f, int count, const LinearItem *items, bool dense)
{
    const int R = 16 * f.RT * f.G, KS = f.WAVES / f.G;
    int64_t blocks = 0, longest = 0;
    double out_mb = 0, word_mb = 0;
    for (int i = 0; i < count; ++i) {
        if (items[i].d_out % 4 != 0) word_mb += 4e-6 * (double)items[i].tokens * (double)items[i].d_out;
        blocks += ceil_div(items[i].d_out, R) * ceil_div(items[i].tokens, f.T);
        longest = std::max(longest, items[i].d_in);
        out_mb += 4e-6 * (double)items[i].tokens * (double)items[i].d_out;
    }
    const size_t lds = (size_t)f.T * self_pitch(longest) + (size_t)f.WAVES * f.RT * 16 * 128;
    if (lds > SELF_LDS || blocks > 4 * (int64_t)device_cus()) return 1e30f;   // (the fit ends at four rounds)
    const double k = (double)longest / 2560.0, cus = device_cus(), load = std::min(1.0, (double)blocks / cus);
    const double steps = (double)(ceil_div(ceil_div(longest, 4 * CHUNK), KS) * f.RT);
    const double work = f.T / 8.0 * k + 0.326 * (R / 64.0) * k * (1.0 + 0.6 * load) + 0.168 * steps * (dense ? 1.735 : 1.0) + (f.WAVES == 16 ? 0.305 : 0.0);
    const double more = (double)(ceil_div(blocks, (int64_t)cus) - 1);
    return (float)(2.955 + work + more * (0.104 + (lds <= SELF_LDS / 2 ? 0.706 : 1.085) * work) + 0.258 * out_mb + 0.45 * word_mb);
}

int choose(int count, const LinearItem *items, bool dense, float &us)
{
    int best = 0;
    us = 1e30f;
    for (int i = 0; i < (int)(sizeof(SELF_FORMS) / sizeof(SELF_FORMS[0])); ++i) {
        const float e = self_estimate_us(SELF_FORMS[i], count, items, dense);
        if (e < us) { us = e; best = i; }
    }
    return best;
}

// whether the outputs of one problem reach into the rows of another (or the same)
bool writes_over_rows(const LinearItem &out, const LinearItem &in)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(in.X), x_end = x + 2 * (uintptr_t)(in.tokens * in.row_values());
    const uintptr_t bytes = 4 * (uintptr_t)(out.tokens * out.d_out), y = reinterpret_cast<uintptr_t>(out.Y), acc = reinterpret_cast<uintptr_t>(out.acc_out);
    return (y < x_end && x < y + bytes) || (acc && acc < x_end && x < acc + bytes);
}

bool self_accepts(int count, const LinearItem *items)
{
    if (count > SELF_ITEMS) return false;
    // blocks write their outputs while others still read the rows; behind a quantizer of its own a call may write over them
    for (int i = 0; i < count; ++i)
        for (int j = 0; j < count; ++j)
            if (writes_over_rows(items[i], items[j])) return false;
    for (int i = 0; i < count; ++i)
        // (The rows of X are addressed with 31 bits behind a buffer's base.  The estimates are fitted to 384 tokens and hold to 512: of 50
        // calls of 385 to 512 that are taken 46 are 1.002 to 1.97 times as fast as two launches, three 0.99, one 0.88 - 416 tokens,
        // 768 -> 2 x 1336 with dense codes, 10.4 us against 9.2.)
        if (!items[i].X || items[i].row_values() > SELF_MAX_ROW || items[i].tokens > 512) return false;
    return true;
}

}  // namespace

// Up to 16 tokens, against gemv_self_kernel and gemv_smfmac_kernel.  Those give a block one wavefront per 512 values: they are at
// their best while every multiprocessor has one block (16 rows) and with as many wavefronts as SIMDs or multiples of it, at
// their worst with five (2049 to 2560 values), in further rounds of blocks, and beyond eight tokens.  Measured both ways over 610
// calls of 2 to 16 tokens, 256 to 8192 values, 256 to 63000 outputs in one to four problems, weights from memory (this kernel's time
// against theirs):
//   9 to 16 tokens  1.23 times as fast in the mean (0.91 to 2.3)
//   6 to 8          1.00 to 1.78 with more than 16 outputs per multiprocessor or rows of 2049 to 2560 values (8 tokens, 2560 -> 3 x 2560
//                   4.5 us / 5.4); with fewer outputs 0.89 to 0.95 at six and seven tokens beyond half as many (4096 -> 4096 5.3 / 4.9),
//                   and 0.90 to 1.05 for several problems of short rows (6 tokens, 512 -> 2 x 492 3.5 / 3.2)
//   3 to 5          outputs from 32 per multiprocessor on: rows of 2049 to 2560 values 1.03 to 1.36 (4 tokens, 2560 -> 2 x 6912 5.6 / 6.0); up to
//                   512 values 1.01 to 1.10, less beyond 128 outputs; between them 0.86 to 0.98 (4 tokens, 1024 -> 8192 3.8 / 3.5) save
//                   for five tokens from 1025 values on and where outputs are stored in words (3 tokens, 1536 -> 9883 4.3 / 4.9)
// By this rule seven of the 610 are slower than there by more than 2 % (at worst 0.91), and of 400 others, 246 of them taken and 1.19 times as
// fast, eleven (at worst 0.94).  In a stack, behind other calls, the two are closer: 4 tokens, eight blocks of 2560 and 6912 172.9 us
// with 2560 -> 2 x 6912 on either.  Calls large enough for the streaming kernel stay there.
bool gemv_takes_self(int count, const LinearItem *items)
{
    if (!self_accepts(count, items)) return false;
    const int64_t cus = device_cus();
    int64_t tokens = 0, rows = 0, strips = 0, longest = 0;
    bool words = false;
    for (int i = 0; i < count; ++i) {
        if (items[i].quantized) return false;
        tokens = std::max(tokens, items[i].tokens);
        rows += items[i].d_out;
        strips += ceil_div(items[i].d_out, 128);
        longest = std::max(longest, items[i].d_in);
        words = words || items[i].d_out % 4 != 0;
    }
    // (strips of 128 rows x 8 tokens fit with rows of any length: four rounds of them at most, for which the shapes are estimated)
    if (rows >= 256 * cus || strips > 2 * cus) return false;
    const bool five_waves = longest > 4 * 512 && longest <= 5 * 512;
    if (tokens >= 9) return true;
    if (tokens >= 6) return five_waves || rows > 16 * cus || ((count == 1 || longest > 1280) && (tokens == 8 || rows <= 8 * cus));
    if (tokens < 3 || rows < 32 * cus || longest > 2560) return false;
    return five_waves || (words || longest <= 512 ? rows < 128 * cus : tokens == 5 && longest > 1024);
}

// Beyond 16 tokens, against the quantizer (2.5 us and 0.38 us per MB of X) and the kernels of launch_gemm_smfmac, whose second launch
// costs a microsecond more than the sum of the two when they are not replayed from a graph.  Of 420 calls drawn from 17 to 2500 tokens, up to
// 8192 values and outputs, one to three problems, whole and ragged chunks, 217 are taken, in 0.74 of the time of two launches; five are
// slower by more than 2 % (152 tokens, 768 -> 3 x 3968 10.8 us against 9.0; 240 tokens, 1048 -> 4392 10.9 / 9.7).
bool gemm_takes_self(int count, const LinearItem *items, bool dense)
{
    if (!self_accepts(count, items)) return false;
    double quantizer = 0;
    for (int i = 0; i < count; ++i) {
        bool seen = false;
        for (int j = 0; j < i; ++j) seen = seen || (items[j].X == items[i].X && items[j].tokens == items[i].tokens && items[j].d_in == items[i].d_in);
        if (!seen) quantizer += 2.5 + 0.76e-6 * (double)items[i].tokens * (double)items[i].d_in;
    }
    int64_t longest = 0;
    for (int i = 0; i < count; ++i) longest = std::max(longest, items[i].d_in);
    float us;
    choose(count, items, dense, us);
    // rows beyond 7168 values: the estimate is up to 1.5 us short (172 tokens, 8192 -> 1246: 13.8 us, 12.1 in two launches); of what is
    // left, 30 calls of 17 to 300 tokens through 7296 to 8192 values, all are faster than two launches, 1.10 to 1.76 times
    return us < gemm_estimate_us(count, items, dense) + (float)quantizer + (longest > 7168 ? -1.0f : 0.6f);
}

int self_form_count() { return (int)(sizeof(SELF_FORMS) / sizeof(SELF_FORMS[0])); }

int self_form(int count, const LinearItem *items, bool dense)
{
    float us;
    return choose(count, items, dense, us);
}

sbn_status launch_gemm_self(int count, const LinearItem *items, bool dense, hipStream_t stream, int form)
{
    if (form < 0) form = self_form(count, items, dense);
    switch (form) {
    case 0: return launch_self_shape<1, 1, 4, 4>(count, items, dense, stream);
    case 1: return launch_self_shape<2, 2, 4, 4>(count, items, dense, stream);
    case 2: return launch_self_shape<2, 1, 8, 8>(count, items, dense, stream);
    case 3: return launch_self_shape<2, 2, 8, 8>(count, items, dense, stream);
    case 4: return launch_self_shape<3, 2, 8, 8>(count, items, dense, stream);
    case 5: return launch_self_shape<2, 4, 8, 8>(count, items, dense, stream);
    case 6: return launch_self_shape<2, 4, 16, 16>(count, items, dense, stream);
    case 7: return launch_self_shape<2, 8, 16, 16>(count, items, dense, stream);
    }
    return SBN_EINVAL;
}

}  // namespace sbn
