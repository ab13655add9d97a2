// Forward of the N:M-sparse ternary linear layer: activation quantizer, decode GEMV, generic path.
// Section 2.1 (per-token absmax int8 activations), Section 2.2 (forward-pass equation),
// Appendix B listing (forward()).
#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <type_traits>
#include <vector>

#include "sbn_decode.hpp"
#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

// ---- activation quantizer -----------------------------------------------------------------------
// TPT threads share one token (256 = a block of four wavefronts per token for prefill, 1024 = a larger
// block per token for decode, where only a handful of tokens exist).  A thread keeps its 16-byte vectors of the row
// in registers, so X is read once; the maximum magnitude is taken on the bf16 bit patterns (exact).
// s_x = 127 / max(amax, 1e-5) is one IEEE fp32 division, x * s_x one fp32 multiply, rounding is
// half-to-even.  Rows longer than VMAX * TPT vectors take the two-pass kernel below.
// The int8 rows lie ldq bytes apart.  xq2 (or null) takes the same rows ld2 bytes apart: an input dimension that is no
// multiple of 128 gives the caller its dense rows and the matrix kernels rows of whole chunks in one pass.
template <int TPT, int VMAX>
__global__ void __launch_bounds__(TPT < 256 ? 256 : TPT) act_quant_kernel(const uint4 *__restrict__ X, int64_t tokens, int nvec,
                                                                         int8_t *__restrict__ xq, int64_t ldq, float *__restrict__ sx,
                                                                         int8_t *__restrict__ xq2, int64_t ld2)
{
    constexpr int BLOCK = TPT < 256 ? 256 : TPT;
    constexpr int TOK_PER_BLOCK = BLOCK / TPT;
    __shared__ uint32_t wave_max[BLOCK / 64];
    const int sub = threadIdx.x % TPT;
    const int64_t t = (int64_t)blockIdx.x * TOK_PER_BLOCK + threadIdx.x / TPT;
    const bool live = t < tokens;
    const uint4 *row = X + (live ? t : 0) * nvec;
    uint4 v[VMAX];
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < VMAX; ++i) {
        const int idx = sub + i * TPT;
        v[i] = (live && idx < nvec) ? row[idx] : make_uint4(0, 0, 0, 0);
        m = absmax_bits_bf16x8(v[i], m);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)m, off, 64);
        m = o > m ? o : m;
    }
    if constexpr (TPT > 64) {
        if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < TPT / 64; ++w) {
            const uint32_t o = wave_max[w];
            m = o > m ? o : m;
        }
    }
    const float s = scale_from_absmax_bits(m);
    if (!live) return;
    if (sub == 0) sx[t] = s;
    uint2 *out = reinterpret_cast<uint2 *>(xq + t * ldq);
    uint2 *out2 = reinterpret_cast<uint2 *>(xq2 + t * ld2);
#pragma unroll
    for (int i = 0; i < VMAX; ++i) {
        const int idx = sub + i * TPT;
        if (idx >= nvec) break;
        const uint2 q = quantize_bf16x8(v[i], s);
        out[idx] = q;
        if (xq2) out2[idx] = q;
    }
}

// any row length: one wavefront per token, the row is read twice (the second read is cache resident)
__global__ void __launch_bounds__(256) act_quant_two_pass_kernel(const uint4 *__restrict__ X, int64_t tokens, int nvec,
                                                                int8_t *__restrict__ xq, int64_t ldq, float *__restrict__ sx,
                                                                int8_t *__restrict__ xq2, int64_t ld2)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= tokens) return;
    const uint4 *row = X + t * nvec;
    uint32_t m = 0;
    for (int v = lane; v < nvec; v += 64) {
        m = absmax_bits_bf16x8(row[v], m);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)m, off, 64);
        m = o > m ? o : m;
    }
    const float s = scale_from_absmax_bits(m);
    if (lane == 0) sx[t] = s;
    uint2 *out = reinterpret_cast<uint2 *>(xq + t * ldq);
    uint2 *out2 = reinterpret_cast<uint2 *>(xq2 + t * ld2);
    for (int v = lane; v < nvec; v += 64) {
        const uint2 q = quantize_bf16x8(row[v], s);
        out[v] = q;
        if (xq2) out2[v] = q;
    }
}

// int8 rows of d_in values (a multiple of 8) -> the same rows ldq bytes apart; what lies between is left as it is
__global__ void __launch_bounds__(256) spread_rows_kernel(const uint2 *__restrict__ src, int64_t tokens, int nvec, int8_t *__restrict__ dst, int64_t ldq)
{
    const int64_t t = blockIdx.x;
    for (int v = threadIdx.x; v < nvec; v += 256) reinterpret_cast<uint2 *>(dst + t * ldq)[v] = src[t * nvec + v];
}

// ---- RMS normalisation fused in front of the quantizer (Algorithm 1: x~ <- Q_a(Norm(x))) ---------
// Same ownership of a token row as act_quant_kernel, the row held in registers throughout, X read
// once.  The mean of squares is summed in double (every square of a bf16 value is exact), r =
// 1/sqrt(mean + eps) is rounded to fp32 once, n = bf16(fp32(x * r) * g) replaces the row in the
// registers, and the quantizer runs on it as it would on a stored bf16 tensor.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;   // round to nearest even; finite inputs
}

template <int TPT, int VMAX>
__global__ void __launch_bounds__(TPT < 256 ? 256 : TPT) rmsnorm_act_quant_kernel(const uint4 *__restrict__ X, const float *__restrict__ gain,
                                                                                 float eps, int64_t tokens, int nvec, int8_t *__restrict__ xq,
                                                                                 float *__restrict__ sx, uint4 *__restrict__ xn)
{
    constexpr int BLOCK = TPT < 256 ? 256 : TPT;
    constexpr int TOK_PER_BLOCK = BLOCK / TPT;
    __shared__ double wave_ssq[BLOCK / 64];
    __shared__ uint32_t wave_max[BLOCK / 64];
    const int sub = threadIdx.x % TPT;
    const int64_t t = (int64_t)blockIdx.x * TOK_PER_BLOCK + threadIdx.x / TPT;
    const bool live = t < tokens;
    const uint4 *row = X + (live ? t : 0) * nvec;
    uint4 v[VMAX];
    double ssq = 0.0;
#pragma unroll
    for (int i = 0; i < VMAX; ++i) {
        const int idx = sub + i * TPT;
        v[i] = (live && idx < nvec) ? row[idx] : make_uint4(0, 0, 0, 0);
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double lo = (double)__uint_as_float(w[k] << 16), hi = (double)__uint_as_float(w[k] & 0xffff0000u);
            ssq += lo * lo;
            ssq += hi * hi;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ssq += __shfl_xor(ssq, off, 64);
    if constexpr (TPT > 64) {
        if ((threadIdx.x & 63) == 0) wave_ssq[threadIdx.x >> 6] = ssq;
        __syncthreads();
        ssq = 0.0;
#pragma unroll
        for (int w = 0; w < TPT / 64; ++w) ssq += wave_ssq[w];
    }
    const float r = (float)(1.0 / sqrt(ssq / (double)(nvec * 8) + (double)eps));
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < VMAX; ++i) {
        const int idx = sub + i * TPT;
        if (idx >= nvec) break;
        float g[8];
        if (gain) {
            const float4 g0 = *reinterpret_cast<const float4 *>(gain + (int64_t)idx * 8);
            const float4 g1 = *reinterpret_cast<const float4 *>(gain + (int64_t)idx * 8 + 4);
            g[0] = g0.x; g[1] = g0.y; g[2] = g0.z; g[3] = g0.w; g[4] = g1.x; g[5] = g1.y; g[6] = g1.z; g[7] = g1.w;
        }
        uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float lo = __fmul_rn(__uint_as_float(w[k] << 16), r), hi = __fmul_rn(__uint_as_float(w[k] & 0xffff0000u), r);
            if (gain) {
                lo = __fmul_rn(lo, g[2 * k]);
                hi = __fmul_rn(hi, g[2 * k + 1]);
            }
            w[k] = f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
        }
        v[i] = make_uint4(w[0], w[1], w[2], w[3]);
        m = absmax_bits_bf16x8(v[i], m);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)m, off, 64);
        m = o > m ? o : m;
    }
    if constexpr (TPT > 64) {
        if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < TPT / 64; ++w) {
            const uint32_t o = wave_max[w];
            m = o > m ? o : m;
        }
    }
    const float s = scale_from_absmax_bits(m);
    if (!live) return;
    if (sub == 0) sx[t] = s;
    uint2 *out = reinterpret_cast<uint2 *>(xq + t * (int64_t)nvec * 8);
#pragma unroll
    for (int i = 0; i < VMAX; ++i) {
        const int idx = sub + i * TPT;
        if (idx >= nvec) break;
        out[idx] = quantize_bf16x8(v[i], s);
        if (xn) xn[t * nvec + idx] = v[i];
    }
}

// ---- decode GEMV on the sparse MFMA (tokens <= 16, 2:4) -----------------------------------------
// A block owns 16 RT rows of W.  Its wavefronts split the input dimension in super-steps of 512
// weights: for such a super-step a lane (row r = lane % 16, quarter c = lane / 16) loads the whole
// 32-byte chunk c of its row (one 16-byte index load, one 16-byte code load; a wavefront reads
// 128 contiguous bytes per row), then issues four v_smfmac_i32_16x16x128_i8, the j-th using index
// word j and code word j.  The tokens are the B operand (16 columns; columns >= tokens are not stored).
// Partial accumulators of the wavefronts are summed through LDS, rescaled and stored.
struct GemvItem {
    const int8_t *xq;
    const float *sx;
    const uint8_t *packed;
    const float *gamma;
    const float *bias;
    float *Y;
    int32_t *acc_out;
    const uint4 *X;   // bf16 activations of a block that quantizes them itself (then xq and sx are unused)
    int d_in, d_out, tokens;
    int d_x;          // values in a row of X (d_in rounded down to what X holds: d_in counts whole chunks)
};
template <int NI>
struct GemvTable {
    GemvItem it[NI];  // problem = blockIdx.y; row tile = blockIdx.x (surplus blocks exit at once)
};
// A launch of a few problems carries a short table: the 3 KB of the long one cost the host half a microsecond.
constexpr int GEMV_FEW = 4, GEMV_MAX_ITEMS = 40;
static_assert(sizeof(GemvTable<GEMV_MAX_ITEMS>) <= 4096, "the table travels as a kernel argument");

// the lane's chunk of super-step s of its row in each row tile; zero codes past the row
template <int FORM, int RT>
__device__ __forceinline__ void gemv_fetch(const uint8_t *const (&wrow)[RT], int s, int c4, int nchunks, uint4 (&idx4)[RT], uint4 (&code4)[RT])
{
    constexpr int CB = FORM == GEMV_1OF4 ? 16 : 32;   // bytes of a chunk
    const int chunk = 4 * s + c4;
#pragma unroll
    for (int a = 0; a < RT; ++a) {
        idx4[a] = code4[a] = make_uint4(0, 0, 0, 0);
        if (chunk < nchunks) {
            idx4[a] = *reinterpret_cast<const uint4 *>(wrow[a] + (int64_t)chunk * CB);
            if constexpr (FORM != GEMV_1OF4) code4[a] = *reinterpret_cast<const uint4 *>(wrow[a] + (int64_t)chunk * CB + 16);
        }
    }
}

// A block's wavefronts in groups of four, their number as a compile-time value: what is read of all wavefronts is asked for at
// once (a loop over a number known at run time waits for each of its reads: 0.05 us apiece)
constexpr int GEMV_WAVE_GROUPS = 4;
constexpr int gemv_groups(int nwaves) { return (nwaves + 3) / 4; }
template <class F> __device__ __forceinline__ void with_wave_groups(int nwaves, F &&f)
{
    const int n = gemv_groups(nwaves);
    if (n == 1) f(std::integral_constant<int, 1>());
    else if (n == 2) f(std::integral_constant<int, 2>());
    else if (n == 3) f(std::integral_constant<int, 3>());
    else f(std::integral_constant<int, 4>());
}
constexpr size_t gemv_red_lds(int nwaves, int rt) { return (size_t)4 * gemv_groups(nwaves) * rt * 1024; }

// Sums the wavefronts' partial accumulators (red: [wavefront, whole groups][row tile][lane]), rescales and stores: wavefront a
// takes row tile a.  Lane: token lane % 16 with the factor `scale`, rows 4 * (lane / 16) + i.
template <int RT>
__device__ __forceinline__ void gemv_finish(const GemvItem &it, const v4i (&acc)[RT], v4i *red, int row0, float scale, int wave, int nwaves, int lane)
{
#pragma unroll
    for (int a = 0; a < RT; ++a) {
        red[(wave * RT + a) * 64 + lane] = acc[a];
        for (int w = nwaves + wave; w < 4 * gemv_groups(nwaves); w += nwaves) red[(w * RT + a) * 64 + lane] = v4i{0, 0, 0, 0};
    }
    __syncthreads();
    for (int a = wave; a < RT; a += nwaves) {
        v4i sum = {0, 0, 0, 0};
        with_wave_groups(nwaves, [&](auto groups) {
            // half of them at a time from twelve on: with all in registers a multiprocessor would not hold two such blocks
            constexpr int BATCH = groups() == 4 ? 8 : groups() == 3 ? 6 : 4 * groups();
#pragma unroll
            for (int w0 = 0; w0 < 4 * groups(); w0 += BATCH) {
                v4i part[BATCH];
#pragma unroll
                for (int w = 0; w < BATCH; ++w) part[w] = red[((w0 + w) * RT + a) * 64 + lane];
#pragma unroll
                for (int w = 0; w < BATCH; ++w) sum += part[w];
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        const int tok = lane & 15, o = row0 + 16 * a + 4 * (lane >> 4);
        if (tok >= it.tokens || o >= it.d_out) continue;
        v4f y = {(float)sum[0] * scale, (float)sum[1] * scale, (float)sum[2] * scale, (float)sum[3] * scale};
        float *dst = it.Y + (int64_t)tok * it.d_out + o;
        if ((it.d_out & 3) == 0 && !it.bias && !it.acc_out) {
            *reinterpret_cast<v4f *>(dst) = y;
            continue;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (o + i < it.d_out) {
                dst[i] = it.bias ? y[i] + it.bias[o + i] : y[i];
                if (it.acc_out) it.acc_out[(int64_t)tok * it.d_out + o + i] = sum[i];
            }
    }
}

// on activations that are quantized already
template <int FORM, int RT, int NI>
__global__ void __launch_bounds__(1024) gemv_smfmac_kernel(GemvTable<NI> tab)
{
    constexpr int CB = FORM == GEMV_1OF4 ? 16 : 32;
    extern __shared__ __attribute__((aligned(16))) int8_t dyn[];
    const GemvItem &it = tab.it[blockIdx.y];
    const int row0 = (int)blockIdx.x * 16 * RT;
    if (row0 >= it.d_out) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int r = lane & 15, c4 = lane >> 4;
    const uint32_t ones = vgpr_ones();
    const int K = it.d_in, nchunks = K / CHUNK, nsuper = (nchunks + 3) / 4;
    const uint8_t *wrow[RT];
#pragma unroll
    for (int a = 0; a < RT; ++a) {
        const int row = row0 + 16 * a + r;
        wrow[a] = it.packed + (int64_t)(row < it.d_out ? row : it.d_out - 1) * nchunks * CB;   // rows past the end are computed and dropped
    }
    const int tok = r < it.tokens ? r : 0;   // as B operand the lane holds token r
    const int8_t *xrow = it.xq + (int64_t)tok * K;
    const float gamma = *it.gamma, sx = it.sx[tok];
    uint4 idx4[RT], code4[RT];
    gemv_fetch<FORM, RT>(wrow, wave, c4, nchunks, idx4, code4);
    v4i acc[RT];
#pragma unroll
    for (int a = 0; a < RT; ++a) acc[a] = v4i{0, 0, 0, 0};
    for (int s = wave; s < nsuper; s += nwaves) {
        uint4 ic[RT], cc[RT];
#pragma unroll
        for (int a = 0; a < RT; ++a) { ic[a] = idx4[a]; cc[a] = code4[a]; }
        gemv_fetch<FORM, RT>(wrow, s + nwaves, c4, nchunks, idx4, code4);   // the next super-step of this wavefront (zeros past the end)
        gemv_super_step<FORM, RT>(ic, cc, xrow + s * 512, c4, ones, [&](int k) { return s * 512 + k < K ? k : K - 16 - s * 512; }, acc);
    }
    gemv_finish<RT>(it, acc, reinterpret_cast<v4i *>(dyn), row0, __fdiv_rn(gamma, sx), wave, nwaves, lane);
}

// The same with the quantizer inside, for rows of at most 16 super-steps: wavefront w owns super-step w of the weights AND of
// the token rows.  Its 8 KB of weights and its 512 values of every token (one 16-byte load per lane and token) are asked
// for together, the largest magnitude of each row meets in LDS behind one barrier, every wavefront quantizes its own
// values (the quantizer's arithmetic) into its own part of LDS and reads the operand from there.  Two barriers in all, and
// the quantizer's work is split over all wavefronts; a wavefront per token row left the other wavefronts waiting.
// What bounds it: the chain of one load, two barriers and a store on top of the 1.9 us of any launch, and the vector work of
// every wavefront (four of them share a SIMD), of the quantizer above all: 0.3 us per token at 14 wavefronts.  Measured, weights from
// memory, us at 1 / 4 / 8 / 12 / 16 tokens: 2560 -> 2560 3.3 / 3.9 / 4.5 / 5.1 / 5.7 (a wavefront per token row: 5.4 / 5.9 / 6.1 / 7.6 / 8.3),
// 6912 -> 2560 5.0 / 6.2 / 7.6 / 8.8 / 9.9 (6.7 / 7.0 / 7.7 / 8.6 / 10.0), 2560 -> 13824 5.7 / 6.5 / 7.5 / 8.7 / 9.7 (10.7 / 12.1 / 14.8 / 19.6 / 22.1).
constexpr int GEMV_SELF_SUPER = 16;       // super-steps at most = wavefronts of a block
static_assert(GEMV_SELF_SUPER <= 4 * GEMV_WAVE_GROUPS, "as many groups as with_wave_groups knows");
constexpr int GEMV_SELF_PITCH = 512 + 16; // bytes between the token rows of a wavefront's part of LDS
constexpr size_t gemv_self_lds(int64_t tokens, int nwaves, int ss, int rt) { return (size_t)nwaves * ss * (size_t)tokens * GEMV_SELF_PITCH + gemv_red_lds(nwaves, rt); }

template <int CTRL> __device__ __forceinline__ uint32_t dpp_max_u16x2(uint32_t mine, uint32_t theirs)
{
    return max_u16x2(mine, (uint32_t)__builtin_amdgcn_mov_dpp((int)theirs, CTRL, 0xf, 0xf, true));
}
// Exchange between two lanes of which one keeps the first half of the registers and the other (upper) the second: half as
// many registers, each the maximum over both lanes.
template <int CTRL, int H> __device__ __forceinline__ void halve_max_u16x2(uint32_t *m, bool upper)
{
#pragma unroll
    for (int j = 0; j < H; ++j) m[j] = dpp_max_u16x2<CTRL>(upper ? m[j + H] : m[j], upper ? m[j] : m[j + H]);
}
// TM = token slots, SS = super-steps per wavefront: wavefront w owns the super-steps w, w + nwaves, ...  Up to four slots the
// registers are held to what lets a multiprocessor run two blocks of 16 wavefronts (8192 -> 16384 at one token: 12.5 us without).
template <int FORM, int RT, int NI, int TM, int SS>
__global__ void __launch_bounds__(1024, TM * SS <= 4 ? 8 : 4) gemv_self_kernel(GemvTable<NI> tab)
{
    constexpr int CB = FORM == GEMV_1OF4 ? 16 : 32;
    extern __shared__ __attribute__((aligned(16))) int8_t dyn[];      // [wavefront][super-step][tokens][pitch], then the partial accumulators
    constexpr int PAIRS = TM <= 2 ? 1 : TM <= 4 ? 2 : TM <= 8 ? 4 : 8;
    __shared__ __attribute__((aligned(16))) uint32_t amax[PAIRS][4 * GEMV_SELF_SUPER + 4];   // [tokens 2 p, 2 p + 1][wavefront, row of 16 lanes]
    const GemvItem &it = tab.it[blockIdx.y];
    const int row0 = (int)blockIdx.x * 16 * RT;
    if (row0 >= it.d_out) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int r = lane & 15, c4 = lane >> 4, T = it.tokens;
    const uint32_t ones = vgpr_ones();
    const int K = it.d_in, nchunks = K / CHUNK, nvec = it.d_x / 8;
    // The token values first, they are needed first, then the weights, without a branch in between: behind a branch the wait
    // for the first value would be one for everything.  Rows past the tokens lie past the end of the buffer, where a load
    // returns zeros and fetches nothing.
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4 *>(it.X), (short)0, T * nvec * 16, 0x00027000);
    uint4 xv[SS][TM];
#pragma unroll
    for (int ss = 0; ss < SS; ++ss) {
        const int vec = 64 * (wave + ss * nwaves) + lane;
        const uint32_t at = 16u * (uint32_t)(vec < nvec ? vec : nvec - 1);   // past the row its last vector again: the maximum is the same, the codes are zero
#pragma unroll
        for (int t = 0; t < TM; ++t)
            xv[ss][t] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rows, at + 16u * (uint32_t)(t * nvec), 0, 0));
    }
    constexpr int WS = SS < 2 || (RT == 2 && TM * SS <= 4) ? 1 : 2;   // super-steps whose weights are asked for ahead
    uint4 idx4[WS][RT], code4[WS][RT];
    const uint8_t *const wbase = it.packed + (int64_t)row0 * nchunks * CB;
    const auto chunk_of = [&](int ss) { return 4 * (wave + ss * nwaves) + c4; };
    const auto fetch = [&](int ss) {
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            // rows past the end are computed and dropped; the offsets within the block's rows (at most 256 chunks each) are small
            const int row = 16 * a + r < it.d_out - row0 ? 16 * a + r : it.d_out - row0 - 1;
            const uint8_t *src = wbase + (uint32_t)(row * nchunks + (chunk_of(ss) < nchunks ? chunk_of(ss) : nchunks - 1)) * (uint32_t)CB;
            idx4[ss % WS][a] = *reinterpret_cast<const uint4 *>(src);
            code4[ss % WS][a] = make_uint4(0, 0, 0, 0);
            if constexpr (FORM != GEMV_1OF4) code4[ss % WS][a] = *reinterpret_cast<const uint4 *>(src + 16);
        }
    };
#pragma unroll
    for (int ss = 0; ss < WS; ++ss) fetch(ss);
    const float gamma = *it.gamma;
    // largest magnitudes, two tokens in a register; rows of 16 lanes are reduced here, the rest through LDS.  Lanes that exchange
    // keep half of the pairs each, so that a row ends with pair r % PAIRS in lane r: for 16 tokens 30 operations where
    // reducing every pair over all lanes takes 64 (and eight stores).
    uint32_t m[PAIRS];
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        m[p] = 0;
        if (2 * p >= TM || 2 * p >= T) continue;
        uint32_t m0 = 0, m1 = 0;
#pragma unroll
        for (int ss = 0; ss < SS; ++ss) {
            const uint32_t a0 = absmax_pair_bf16x8(xv[ss][2 * p < TM ? 2 * p : 0]), a1 = absmax_pair_bf16x8(xv[ss][2 * p < TM ? 2 * p + 1 : 1]);
            m0 = ss ? max_u16x2(m0, a0) : a0;
            m1 = ss ? max_u16x2(m1, a1) : a1;
        }
        m[p] = max_u16x2(__builtin_amdgcn_perm(m1, m0, 0x05040100u), __builtin_amdgcn_perm(m1, m0, 0x07060302u));   // low halves, high halves
    }
    if constexpr (PAIRS >= 8) halve_max_u16x2<0x141, 4>(m, (r & 4) != 0);   // row_half_mirror
    if constexpr (PAIRS >= 4) halve_max_u16x2<0x4e, 2>(m, (r & 2) != 0);    // quad_perm 2 3 0 1
    if constexpr (PAIRS >= 2) halve_max_u16x2<0xb1, 1>(m, (r & 1) != 0);    // quad_perm 1 0 3 2
    if constexpr (PAIRS < 2) m[0] = dpp_max_u16x2<0x121>(m[0], m[0]);       // row_ror 1, 2, 4, 8: lanes with the same pair
    if constexpr (PAIRS < 4) m[0] = dpp_max_u16x2<0x122>(m[0], m[0]);
    if constexpr (PAIRS < 8) m[0] = dpp_max_u16x2<0x124>(m[0], m[0]);
    m[0] = dpp_max_u16x2<0x128>(m[0], m[0]);
    if (r < PAIRS) amax[r][4 * wave + c4] = m[0];
    __syncthreads();
    // lane: the scale of token lane % 16
    float s;
    {
        // quarter c4 reads what wavefronts c4, c4 + 4, ... found (past the last one that one again), then the quarters meet
        const uint4 *col = reinterpret_cast<const uint4 *>(amax[(r >> 1) % PAIRS]);
        uint32_t m2 = 0;
        with_wave_groups(nwaves, [&](auto groups) {
            uint4 v[groups()];
#pragma unroll
            for (int i = 0; i < groups(); ++i) v[i] = col[i + 1 < groups() || 4 * i + c4 < nwaves ? 4 * i + c4 : nwaves - 1];
#pragma unroll
            for (int i = 0; i < groups(); ++i) m2 = max_u16x2(m2, max_u16x2(max_u16x2(v[i].x, v[i].y), max_u16x2(v[i].z, v[i].w)));
        });
        uint32_t m = r & 1 ? m2 >> 16 : m2 & 0xffffu;
        const auto x16 = __builtin_amdgcn_permlane16_swap(m, m, false, false);   // neighbouring quarters
        m = x16[0] > x16[1] ? x16[0] : x16[1];
        const auto x32 = __builtin_amdgcn_permlane32_swap(m, m, false, false);   // halves of the wavefront
        m = x32[0] > x32[1] ? x32[0] : x32[1];
        s = scale_from_absmax_bits(m);
    }
    int8_t *const xs = dyn + wave * SS * T * GEMV_SELF_PITCH;
#pragma unroll
    for (int ss = 0; ss < SS; ++ss)
#pragma unroll
        for (int t = 0; t < TM; ++t)
            if (t < T)
                *reinterpret_cast<uint2 *>(xs + (ss * T + t) * GEMV_SELF_PITCH + 8 * lane) =
                    quantize_bf16x8(xv[ss][t], __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(s), t)));
    v4i acc[RT];
#pragma unroll
    for (int a = 0; a < RT; ++a) acc[a] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int ss = 0; ss < SS; ++ss) {
#pragma unroll
        for (int a = 0; a < RT; ++a) {   // past the row zero codes (the code words of 1:4 are the upper half of its one vector)
            if (chunk_of(ss) < nchunks) continue;
            if constexpr (FORM == GEMV_DENSE) idx4[ss % WS][a] = make_uint4(0, 0, 0, 0);
            else if constexpr (FORM == GEMV_1OF4) idx4[ss % WS][a].z = idx4[ss % WS][a].w = 0;
            code4[ss % WS][a] = make_uint4(0, 0, 0, 0);
        }
        // what the wavefront wrote itself: its LDS operations complete in order
        gemv_super_step<FORM, RT, RT == 2 && TM * SS <= 4>(idx4[ss % WS], code4[ss % WS], xs + (ss * T + (r < T ? r : 0)) * GEMV_SELF_PITCH, c4, ones, [](int k) { return k; }, acc);
        if constexpr (WS < SS) __builtin_amdgcn_sched_barrier(0);   // not in front of the step: no registers for it there
        if (ss + WS < SS) fetch(ss + WS);
    }
    gemv_finish<RT>(it, acc, reinterpret_cast<v4i *>(dyn + nwaves * SS * T * GEMV_SELF_PITCH), row0, __fdiv_rn(gamma, s), wave, nwaves, lane);
}

// ---- streaming decode GEMV for grouped calls ---------------------------------------------------
// Persistent blocks, one per multiprocessor: the rows of all problems are cut into units of 16*RT
// rows x the whole input dimension (a contiguous range of packed bytes); every block takes a
// contiguous run of units and hands them to its NW wavefronts one at a time.  The int8 activations
// of the current problem (tokens x d_in) are staged in LDS once per block and problem; the packed weights
// go straight from HBM to registers through a queue of DEPTH super-steps (512 weights each) per
// wavefront, so that several 16-byte loads per lane are always in flight.  No cross-wave reduction.
// The blocks' shares are equal and fixed.  Measured with timestamps (64 x (2560 x 6912), eight tokens, 52 us): the
// blocks finish between 43 and 52 us - multiprocessors in alternate positions of an XCD run about 10 % apart, and so
// do the older and the younger wavefronts of a SIMD - and the wavefronts idle 7 us on average before the kernel ends.
// Holding back a sixth of the units as a device-wide pool for wavefronts out of work did not recover that (52.7 us):
// a unit of 16 rows is 10 us of one wavefront's time at K = 6912, as coarse as the imbalance itself, and a counter
// that 2048 wavefronts ask per unit is far too hot (5800 returning atomics on one word: 55 us), so the pool had to be
// drawn per block, eight units at a time.  Finer balancing would need units split along K across wavefronts.
struct GemvStreamItem {
    const int8_t *xq;
    const float *sx;
    const uint8_t *packed;
    const float *gamma;
    float *Y;
    int d_in, d_out, tokens;
    int input;   // index into GemvStreamTable::in when the kernel quantizes the activations itself, else -1
};
// A distinct activation matrix of the call that the kernel quantizes itself: the first blocks of the
// grid take one token row each (same arithmetic as the quantizer kernels), write the int8 row and its
// scale to the workspace and raise a per-token flag; every block waits for the flags of an input, with
// its first weight loads already in flight, before it stages that input - the quantizer then costs no
// launch of its own.  Rows and scales are ordinary stores and loads; the flag is stored with release
// and, once seen, followed by an acquire fence, both at device scope, so the hand-over rests on the
// language's memory model alone (one L2 write-back per producer block, one invalidation per consumer).
// The wait is bounded: a block out of polls quantizes the rows itself into LDS (same result).
struct GemvStreamInput {
    const uint4 *X;              // bf16 [tokens, d_in]
    unsigned long long *xq;      // workspace, int8 [tokens, d_in] as 8-byte words
    unsigned *sx;                // workspace, fp32 bits [tokens]
    unsigned long long *flags;   // workspace, one per token
    int tokens, d_in;
};
constexpr int GEMV_STREAM_MAX = 64;
constexpr int GEMV_STREAM_INPUTS = 4;
constexpr int GEMV_QUANT_VEC = 4;    // 16-byte vectors of a row per thread when a block quantizes it
constexpr int STAGE_BATCH = 8;       // activation loads a thread has in flight while it stages a block's input in LDS
constexpr int GEMV_OWN_VEC = 14;     // 16-byte vectors of a token row per lane when a wavefront quantizes a row for its own block
struct GemvStreamTable {
    GemvStreamItem it[GEMV_STREAM_MAX];
    int unit0[GEMV_STREAM_MAX + 1];   // first unit of each problem
    int count;
    GemvStreamInput in[GEMV_STREAM_INPUTS];
    int tok0[GEMV_STREAM_INPUTS + 1]; // first producer block of each input
    int nin;
    unsigned epoch;                   // distinguishes this launch's flags from whatever the workspace held
    int spin_limit;
    int share, share_rem;             // units per block: the first share_rem blocks take share + 1, the others share
    int pad;
};
static_assert(sizeof(GemvStreamTable) <= 4096 && sizeof(GemvStreamTable) % 8 == 0, "the table travels as a kernel argument");

// A value every lane holds alike, moved to a scalar register: what is read from the LDS copy of a launch table decides
// loop bounds and branches, which must stay scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned uni(unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); }
template <typename T> __device__ __forceinline__ T *uni(T *p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    // rebuilt as a pointer into global memory, so that what is read through it stays a global (not a flat) access
    typedef T __attribute__((address_space(1))) *global_ptr;
    return (T *)(global_ptr)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ unsigned long long gemv_flag_value(unsigned epoch, int t)
{
    return ((unsigned long long)epoch << 32) | (0x5bd1e995u ^ (unsigned)t);
}

template <int RT, int DEPTH, int NW, int FORM>
__global__ void __launch_bounds__(64 * NW) gemv_stream_kernel(GemvStreamTable tab_arg)
{
    constexpr bool DENSE = FORM == GEMV_DENSE, ONE4 = FORM == GEMV_1OF4;
    constexpr int CB = ONE4 ? 16 : 32;   // bytes of a chunk: the 1:4 form is one 16-byte load per lane and super-step
    extern __shared__ __attribute__((aligned(16))) int8_t xlds[];   // [tokens][d_in + 16]
    // The launch table is fetched once, by the whole block in one round trip, into LDS.  Read through the kernel
    // argument it costs a chain of dependent scalar loads before the first weight load can go out (which problem, its
    // shape, its pointers: a dozen, each a trip to memory: measured 5.6 us from the block's start to its first load).
    __shared__ __attribute__((aligned(16))) GemvStreamTable tab;
    {
        (void)tab_arg;
        const uint2 *src = (const uint2 *)__builtin_amdgcn_kernarg_segment_ptr();   // the table is the only argument
        uint2 *dst = reinterpret_cast<uint2 *>(&tab);
        for (int i = threadIdx.x; i < (int)(sizeof(GemvStreamTable) / 8); i += 64 * NW) dst[i] = src[i];
        __syncthreads();
    }
    __shared__ int unit_ctr;                                        // next unit of the current problem nobody has taken
    __shared__ float sx_lds[16];                                    // s_x of the staged tokens of a self-quantized input
    __shared__ uint32_t wave_amax[NW];
    __shared__ int stage_ok;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // quantize token row t of an input with the whole block: to the workspace (publish) or to the LDS copy
    auto quantize_row = [&](const GemvStreamInput &in, int t, int8_t *lds_row, bool publish) {
        const int nvec = in.d_in / 8;
        const uint4 *row = in.X + (int64_t)t * nvec;
        uint4 v[GEMV_QUANT_VEC];
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < GEMV_QUANT_VEC; ++i) {
            const int idx = threadIdx.x + i * 64 * NW;
            v[i] = idx < nvec ? row[idx] : make_uint4(0, 0, 0, 0);
            m = absmax_bits_bf16x8(v[i], m);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)m, off, 64);
            m = o > m ? o : m;
        }
        __syncthreads();   // wave_amax is free again
        if (lane == 0) wave_amax[wave] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) m = wave_amax[w] > m ? wave_amax[w] : m;
        const float s = scale_from_absmax_bits(m);
        if (threadIdx.x == 0) {
            if (publish) in.sx[t] = __float_as_uint(s);
            else sx_lds[t] = s;
        }
#pragma unroll
        for (int i = 0; i < GEMV_QUANT_VEC; ++i) {
            const int idx = threadIdx.x + i * 64 * NW;
            if (idx >= nvec) continue;
            const uint2 q = quantize_bf16x8(v[i], s);
            if (publish)
                reinterpret_cast<uint2 *>(in.xq)[(int64_t)t * nvec + idx] = q;
            else
                reinterpret_cast<uint2 *>(lds_row)[idx] = q;
        }
    };
    auto load_input = [&](int j) {
        const GemvStreamInput &src = tab.in[j];
        GemvStreamInput d;
        d.X = uni(src.X); d.xq = uni(src.xq); d.sx = uni(src.sx); d.flags = uni(src.flags);
        d.tokens = uni(src.tokens); d.d_in = uni(src.d_in);
        return d;
    };
    auto load_item = [&](int i) {
        const GemvStreamItem &src = tab.it[i];
        GemvStreamItem d;
        d.xq = uni(src.xq); d.sx = uni(src.sx); d.packed = uni(src.packed); d.gamma = uni(src.gamma); d.Y = uni(src.Y);
        d.d_in = uni(src.d_in); d.d_out = uni(src.d_out); d.tokens = uni(src.tokens); d.input = uni(src.input);
        return d;
    };
    auto unit0 = [&](int i) { return uni(tab.unit0[i]); };
    // What stands between a block's start and its first requests is a chain of dependent reads of this table, so the
    // chain is kept short: the block's share from two numbers the host divided out, its first problem from one read
    // of all problem boundaries and a vote.
    const unsigned epoch = uni(tab.epoch);
    const int spin_limit = uni(tab.spin_limit);
    const int share = uni(tab.share), share_rem = uni(tab.share_rem);
    const int bound = tab.unit0[1 + lane];   // boundaries past the last problem hold the total
    if ((int)blockIdx.x < uni(tab.tok0[GEMV_STREAM_INPUTS])) {   // producer role: one token row of one input
        int j = 0;
        while ((int)blockIdx.x >= uni(tab.tok0[j + 1])) ++j;
        const GemvStreamInput in = load_input(j);
        const int t = (int)blockIdx.x - uni(tab.tok0[j]);
        quantize_row(in, t, nullptr, true);
        // The row and its scale are ordinary stores. The barrier orders every thread's part before thread 0,
        // whose release store of the flag makes all of it visible to the whole device before the flag is.
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(&in.flags[t], gemv_flag_value(epoch, t), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int b0 = share * (int)blockIdx.x + ((int)blockIdx.x < share_rem ? (int)blockIdx.x : share_rem);
    const int b1 = b0 + share + ((int)blockIdx.x < share_rem ? 1 : 0);
    const int r = lane & 15, c4 = lane >> 4;
    const uint32_t ones = vgpr_ones();
    // the block's first problem: as many problems end at or before its first unit
    int item = __builtin_popcountll(__ballot(bound <= b0));
    int u = b0;
    const int8_t *staged_xq = nullptr;   // what the LDS copy currently holds (block-uniform)
    int staged_tokens = 0, staged_k = 0;
    bool first_problem = true;
    while (u < b1) {
        while (u >= unit0(item + 1)) ++item;
        const GemvStreamItem it = load_item(item);
        const int item_u0 = unit0(item), item_u1 = unit0(item + 1);
        const int seg_end = b1 < item_u1 ? b1 : item_u1;
        const int ua = u - item_u0, ub = seg_end - item_u0;   // units of this problem for the block
        u = seg_end;
        const int K = it.d_in, nchunks = K / CHUNK, nsuper = (nchunks + 3) / 4, pitch = K + 16;
        const bool tok_ok = r < it.tokens;
        const int xoff = (tok_ok ? r : 0) * pitch + (DENSE ? 128 * c4 : 128 * (c4 >> 1) + 16 * (c4 & 1));
        const bool ragged = (nchunks & 3) != 0;   // the last super-step of a unit then covers fewer than four chunks

        // Wavefronts of a block advance at very different speeds (measured: the first one to finish
        // an equal share is done in half the time of the last), so the units of the block are handed
        // out one at a time from a counter in LDS: wavefront w starts with unit ua + w and takes the
        // next free one whenever its load stream reaches the end of a unit.  The loads run DEPTH
        // super-steps ahead of the arithmetic; with nsuper > DEPTH they are at most one unit ahead,
        // so one register (nu) carries the unit number from the load side to the arithmetic.  Shorter
        // rows fall back to equal contiguous shares.
        const bool dyn = nsuper > DEPTH;
        const int wa = dyn ? ua + wave : ua + (int)((int64_t)(ub - ua) * wave / NW);
        const int wb = dyn ? ub : ua + (int)((int64_t)(ub - ua) * (wave + 1) / NW);   // first unit number that is not this wavefront's
        __syncthreads();   // nobody still uses the previous problem's counter or activations
        if (threadIdx.x == 0) unit_ctr = ua + NW;
        int iu = wa, is = 0, cu = wa, cs = 0, nu = wb;
        int grabbed = wb;   // prefetched from the counter one unit ahead of its use
        uint4 qi[DEPTH][RT], qc[DEPTH][RT];
        // Every load is unconditional, so the loop below is straight-line code and the wait the
        // compiler places before a slot is consumed leaves the DEPTH - 1 younger super-steps in
        // flight (a load inside a branch makes it wait for everything).  Past the end of the
        // wavefront's work the last unit is fetched again (cache hits, no HBM traffic) and ignored.
        // The lane's packed rows of the unit being loaded: the 64-bit address arithmetic runs once per unit, a load
        // adds the chunk's offset (the vector unit is the scarce resource of the 1:4 form).
        const uint8_t *prow[RT];
        auto locate = [&](int unit) {
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                int row = unit * 16 * RT + 16 * a + r;
                row = row < it.d_out ? row : it.d_out - 1;
                prow[a] = it.packed + (int64_t)row * nchunks * CB;
            }
        };
        locate(wa < wb ? wa : ub - 1);
        auto issue = [&](uint4(&ib)[RT], uint4(&cb)[RT]) {
            int ch = 4 * is + c4;
            ch = ch < nchunks ? ch : nchunks - 1;
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                const uint8_t *p = prow[a] + (uint32_t)ch * CB;
                ib[a] = *reinterpret_cast<const uint4 *>(p);        // plain loads: nontemporal ones measured 30 % slower
                if constexpr (ONE4) cb[a] = make_uint4(0, 0, 0, 0);
                else cb[a] = *reinterpret_cast<const uint4 *>(p + 16);
            }
            if (++is == nsuper) {
                is = 0;
                if (dyn) {
                    iu = nu = __builtin_amdgcn_readfirstlane(grabbed);
                    if (lane == 0) grabbed = atomicAdd(&unit_ctr, 1);
                } else {
                    ++iu;
                }
                locate(iu < wb ? iu : ub - 1);
            }
        };
        // Activations are staged only when they differ from what the block already holds (projections
        // that share an input, Q/K/V or up/gate, come one after the other).
        const bool restage = it.xq != staged_xq || it.tokens != staged_tokens || K != staged_k;
        const bool self_quant = it.input >= 0;
        // The input of a block's FIRST problem is quantized by the block itself, a wavefront per token row with the
        // whole row in registers: one trip to memory for the bf16 rows (requested before the weight queue fills),
        // a wavefront-level maximum, the int8 row written straight into LDS.  Waiting for the producer blocks
        // instead put the staged activations 8-10 us behind the block's start (row read, release, poll, acquire,
        // staging read: five trips in a row) with only the DEPTH queued super-steps of weights to cover them.
        // Inputs that a block meets later were published by the producer blocks long before.
        const bool own = restage && self_quant && first_problem && K <= 8 * 64 * GEMV_OWN_VEC;
        first_problem = false;
        uint4 xv[GEMV_OWN_VEC];
        const uint4 *own_X = nullptr;
        auto own_request = [&](int t) {
            const uint4 *row = own_X + (int64_t)t * (K / 8);
#pragma unroll
            for (int i = 0; i < GEMV_OWN_VEC; ++i) {
                if (64 * i >= K / 8) break;   // the same for every lane
                const int idx = lane + 64 * i;
                xv[i] = row[idx < K / 8 ? idx : K / 8 - 1];   // past the end the last vector again: the maximum is the same
            }
        };
        auto own_quantize = [&](int t) {
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < GEMV_OWN_VEC; ++i) {
                if (64 * i >= K / 8) break;
                m = absmax_bits_bf16x8(xv[i], m);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const uint32_t o = (uint32_t)__shfl_xor((int)m, off, 64);
                m = o > m ? o : m;
            }
            const float s = scale_from_absmax_bits(m);
            if (lane == 0) sx_lds[t] = s;
            uint2 *lds_row = reinterpret_cast<uint2 *>(xlds + t * pitch);
#pragma unroll
            for (int i = 0; i < GEMV_OWN_VEC; ++i) {
                if (64 * i >= K / 8) break;
                const int idx = lane + 64 * i;
                if (idx < K / 8) lds_row[idx] = quantize_bf16x8(xv[i], s);
            }
        };
        if (own) {
            own_X = uni(tab.in[it.input].X);
            if (wave < it.tokens) own_request(wave);
        }
        // copy tokens x K quantized activations into the LDS rows; the loads go out in batches so that
        // their latencies overlap instead of adding up
        auto stage = [&](const int8_t *src, int tokens) {
            const int n16 = tokens * (K / 16);
            for (int v0 = threadIdx.x; v0 < n16; v0 += 64 * NW * STAGE_BATCH) {
                uint4 q[STAGE_BATCH];
#pragma unroll
                for (int b = 0; b < STAGE_BATCH; ++b) {
                    const int v = v0 + 64 * NW * b;
                    q[b] = *reinterpret_cast<const uint4 *>(src + (int64_t)(v < n16 ? v : n16 - 1) * 16);
                }
#pragma unroll
                for (int b = 0; b < STAGE_BATCH; ++b) {
                    // past the end the last vector is written again (same bytes, same place): no branch, so the batch
                    // stays in registers
                    const int v = v0 + 64 * NW * b < n16 ? v0 + 64 * NW * b : n16 - 1;
                    *reinterpret_cast<uint4 *>(&xlds[(v / (K / 16)) * pitch + (v % (K / 16)) * 16]) = q[b];
                }
            }
        };
        if (restage && !self_quant) stage(it.xq, it.tokens);
        __syncthreads();   // counter and activations in place
        if (dyn && lane == 0) grabbed = atomicAdd(&unit_ctr, 1);
        if (wa < wb) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) issue(qi[d], qc[d]);
        }
        if (own) {
            for (int t = wave; t < it.tokens; t += NW) {
                if (t != wave) own_request(t);
                own_quantize(t);
            }
            __syncthreads();
        } else if (restage && self_quant) {
            // the first weight loads are in flight; now wait (bounded) for the blocks that quantize this input
            const GemvStreamInput in = load_input(it.input);
            if (threadIdx.x == 0) stage_ok = 1;
            __syncthreads();
            if ((int)threadIdx.x < in.tokens) {
                const unsigned long long want = gemv_flag_value(epoch, threadIdx.x);
                int spins = 0, ok = spin_limit >= 0;
                while (ok && __hip_atomic_load(&in.flags[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != want) {
                    if (++spins > spin_limit) ok = 0;
                    else __builtin_amdgcn_s_sleep(4);
                }
                if (!ok) stage_ok = 0;   // several lanes may write the same value
                // acquire: what the producers stored before their flags is what the loads below see; the
                // barrier hands that on to the block's other threads
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            }
            __syncthreads();
            if (!stage_ok) {   // out of patience: quantize the rows here, straight into LDS (same arithmetic, same result)
                for (int t = 0; t < in.tokens; ++t) quantize_row(in, t, xlds + t * pitch, false);
            } else {
                if ((int)threadIdx.x < in.tokens) sx_lds[threadIdx.x] = __uint_as_float(in.sx[threadIdx.x]);
                stage(reinterpret_cast<const int8_t *>(in.xq), in.tokens);
            }
            __syncthreads();
        }
        if (restage) {
            staged_xq = it.xq;
            staged_tokens = it.tokens;
            staged_k = K;
        }
        const float scale = tok_ok ? __fdiv_rn(*it.gamma, self_quant ? sx_lds[r] : it.sx[r]) : 0.0f;

        v4i acc[RT];
#pragma unroll
        for (int a = 0; a < RT; ++a) acc[a] = v4i{0, 0, 0, 0};
        // Lanes of absent tokens read token 0's activations (their accumulator columns are never
        // stored); activations past the input dimension are read from the slack behind the staged
        // rows and meet zero codes.
        while (cu < wb) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                uint4 ic[RT], cc[RT];
#pragma unroll
                for (int a = 0; a < RT; ++a) { ic[a] = qi[d][a]; cc[a] = qc[d][a]; }
                issue(qi[d], qc[d]);
                if ((ragged && cs == nsuper - 1 && 4 * cs + c4 >= nchunks) || cu >= wb) {
#pragma unroll
                    for (int a = 0; a < RT; ++a) {
                        cc[a] = make_uint4(0, 0, 0, 0);
                        if constexpr (DENSE) ic[a] = make_uint4(0, 0, 0, 0);   // all eight words are codes
                        if constexpr (ONE4) ic[a].z = ic[a].w = 0;             // the chunk's two code words
                    }
                }
                if constexpr (DENSE) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const v4i b = *reinterpret_cast<const v4i *>(&xlds[xoff + cs * 512 + 16 * j]);
#pragma unroll
                        for (int a = 0; a < RT; ++a) {
                            const uint4 &half = j < 4 ? ic[a] : cc[a];
                            const uint32_t cw = (j & 3) == 0 ? half.x : (j & 3) == 1 ? half.y : (j & 3) == 2 ? half.z : half.w;
                            acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(expand_codes(cw, ones), b, acc[a], 0, 0, 0);
                        }
                    }
                }
                // sparse forms: the super-step's activations are asked for first, so that the LDS latency passes under
                // the vector work that builds the A operands
                v8i bq[DENSE ? 1 : 4];
#pragma unroll
                for (int j = 0; j < (DENSE ? 0 : 4); ++j) {
                    const uint4 blo = *reinterpret_cast<const uint4 *>(&xlds[xoff + cs * 512 + 32 * j]);
                    const uint4 bhi = *reinterpret_cast<const uint4 *>(&xlds[xoff + cs * 512 + 32 * j + 256]);
                    bq[j] = v8i{(int)blo.x, (int)blo.y, (int)blo.z, (int)blo.w, (int)bhi.x, (int)bhi.y, (int)bhi.z, (int)bhi.w};
                }
                uint32_t iw1[RT][2][2];
                v4i a1[RT][2][2];
                if constexpr (ONE4) {
#pragma unroll
                    for (int a = 0; a < RT; ++a) {
                        expand_1of4(ic[a].x, ic[a].z, ones, iw1[a][0], a1[a][0]);
                        expand_1of4(ic[a].y, ic[a].w, ones, iw1[a][1], a1[a][1]);
                    }
                }
#pragma unroll
                for (int j = 0; j < (DENSE ? 0 : 4); ++j) {
#pragma unroll
                    for (int a = 0; a < RT; ++a) {
                        if constexpr (ONE4) {
                            acc[a] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(a1[a][j >> 1][j & 1], bq[j], acc[a], (int)iw1[a][j >> 1][j & 1], 0, 0);
                            continue;
                        }
                        const uint32_t cw = j == 0 ? cc[a].x : j == 1 ? cc[a].y : j == 2 ? cc[a].z : cc[a].w;
                        const uint32_t iw = j == 0 ? ic[a].x : j == 1 ? ic[a].y : j == 2 ? ic[a].z : ic[a].w;
                        acc[a] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(expand_codes(cw, ones), bq[j], acc[a], (int)iw, 0, 0);
                    }
                }
                if (++cs == nsuper) {
                    // unit cu complete: lane holds token r, rows 4 * c4 + i of each row tile
                    if (tok_ok && cu < wb) {
#pragma unroll
                        for (int a = 0; a < RT; ++a) {
                            const int o = cu * 16 * RT + 16 * a + 4 * c4;
                            if (o + 3 < it.d_out && (it.d_out & 3) == 0) {
                                const v4f y = {(float)acc[a][0] * scale, (float)acc[a][1] * scale, (float)acc[a][2] * scale,
                                               (float)acc[a][3] * scale};
                                // streaming store: Y is not read again here and should not displace the weight stream in L2
                                __builtin_nontemporal_store(y, reinterpret_cast<v4f *>(it.Y + (int64_t)r * it.d_out + o));
                            } else {
                                for (int i = 0; i < 4; ++i)
                                    if (o + i < it.d_out) it.Y[(int64_t)r * it.d_out + o + i] = (float)acc[a][i] * scale;
                            }
                        }
                    }
#pragma unroll
                    for (int a = 0; a < RT; ++a) acc[a] = v4i{0, 0, 0, 0};
                    cs = 0;
                    cu = dyn ? nu : cu + 1;
                }
            }
        }
    }
}

// ---- generic path: any supported pattern, plain integer arithmetic ---------------------------------
// One thread per output row, eight tokens per block row; decodes every slot of the packed row.
__global__ void __launch_bounds__(128) linear_generic_kernel(const int8_t *__restrict__ xq, const float *__restrict__ sx,
                                                            const uint8_t *__restrict__ packed, const float *gamma,
                                                            const float *bias, float *Y, int32_t *acc_out,
                                                            int64_t tokens, int d_in, int d_out, Pattern pat)
{
    const int o = blockIdx.x * 128 + threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.y * 8;
    if (o >= d_out) return;
    const int nchunks = (d_in + CHUNK - 1) / CHUNK;
    int acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int c = 0; c < nchunks; ++c) {
        const uint8_t *idx_field = packed + ((int64_t)o * nchunks + c) * pat.chunk_bytes;
        const uint8_t *code_field = idx_field + pat.idx_bytes;
        for (int s = 0; s < pat.slots; ++s) {
            const int v = s & 15;
            const int cp = 32 * (s >> 4) + 8 * (v & 3) + 2 * (v >> 2);
            const uint32_t code = (code_field[cp >> 3] >> (cp & 7)) & 3u;
            if (code == 0) continue;
            int j = s % pat.N;
            if (pat.b) {
                const int p = s * pat.b;
                const uint32_t two = (uint32_t)idx_field[p >> 3] | ((uint32_t)idx_field[(p >> 3) + ((p >> 3) + 1 < pat.idx_bytes ? 1 : 0)] << 8);
                j = (two >> (p & 7)) & ((1u << pat.b) - 1u);
            }
            const int col = c * CHUNK + (s / pat.N) * pat.M + j;
            if (col >= d_in) continue;
            const int w = code == 1u ? 1 : -1;
#pragma unroll
            for (int tt = 0; tt < 8; ++tt)
                if (t0 + tt < tokens) acc[tt] += w * (int)xq[(t0 + tt) * d_in + col];
        }
    }
    const float g = *gamma;
#pragma unroll
    for (int tt = 0; tt < 8; ++tt) {
        if (t0 + tt >= tokens) break;
        float y = (float)acc[tt] * __fdiv_rn(g, sx[t0 + tt]);
        if (bias) y += bias[o];
        Y[(t0 + tt) * d_out + o] = y;
        if (acc_out) acc_out[(t0 + tt) * d_out + o] = acc[tt];
    }
}

}  // namespace

size_t linear_workspace_bytes(int64_t tokens, int64_t d_out, int64_t d_in)
{
    // int8 activations in rows of whole chunks + per-token scales + the weights in another form: dense int8 for the
    // comparison path, or at most two bits per weight of whole chunks
    const int64_t kp = ceil_div(d_in, CHUNK) * CHUNK;
    return align_up((size_t)tokens * kp, 256) + align_up((size_t)tokens * sizeof(float), 256) +
           align_up((size_t)d_out * (d_in > kp / 4 ? d_in : kp / 4), 256);
}

sbn_status launch_act_quant(const void *X, int64_t tokens, int64_t d_in, int8_t *xq, float *sx, hipStream_t stream, int64_t ldq,
                            int8_t *xq2, int64_t ld2)
{
    const uint4 *x = static_cast<const uint4 *>(X);
    const int nvec = (int)(d_in / 8);
    if (ldq == 0) ldq = d_in;
    if (tokens <= 64 && nvec <= 2 * 1024) {
        hipLaunchKernelGGL((act_quant_kernel<1024, 2>), dim3((unsigned)tokens), dim3(1024), 0, stream, x, tokens, nvec, xq, ldq, sx, xq2, ld2);
    } else if (nvec <= 2 * 256) {
        // a block of four wavefronts per token (measured against one or two wavefronts per token with longer loops: same
        // kernel time, but the step that follows starts 1-2 % earlier)
        hipLaunchKernelGGL((act_quant_kernel<256, 2>), dim3((unsigned)tokens), dim3(256), 0, stream, x, tokens, nvec, xq, ldq, sx, xq2, ld2);
    } else if (nvec <= 4 * 256) {
        hipLaunchKernelGGL((act_quant_kernel<256, 4>), dim3((unsigned)tokens), dim3(256), 0, stream, x, tokens, nvec, xq, ldq, sx, xq2, ld2);
    } else {
        hipLaunchKernelGGL(act_quant_two_pass_kernel, dim3((unsigned)ceil_div(tokens, 4)), dim3(256), 0, stream, x, tokens, nvec, xq, ldq, sx, xq2, ld2);
    }
    return check_launch("act_quant_kernel");
}

sbn_status launch_spread_rows(const int8_t *src, int64_t tokens, int64_t d_in, int8_t *dst, int64_t ldq, hipStream_t stream)
{
    hipLaunchKernelGGL(spread_rows_kernel, dim3((unsigned)tokens), dim3(256), 0, stream, reinterpret_cast<const uint2 *>(src), tokens,
                       (int)(d_in / 8), dst, ldq);
    return check_launch("spread_rows_kernel");
}

sbn_status launch_rmsnorm_act_quant(const void *X, const float *gain, float eps, int64_t tokens, int64_t d_in, int8_t *xq,
                                    float *sx, void *xn, hipStream_t stream)
{
    const uint4 *x = static_cast<const uint4 *>(X);
    uint4 *n = static_cast<uint4 *>(xn);
    const int nvec = (int)(d_in / 8);
    if (nvec <= 2 * 256 && tokens > 64) {
        hipLaunchKernelGGL((rmsnorm_act_quant_kernel<256, 2>), dim3((unsigned)tokens), dim3(256), 0, stream, x, gain, eps, tokens, nvec,
                           xq, sx, n);
    } else if (nvec <= 4 * 256 && tokens > 64) {
        hipLaunchKernelGGL((rmsnorm_act_quant_kernel<256, 4>), dim3((unsigned)tokens), dim3(256), 0, stream, x, gain, eps, tokens, nvec,
                           xq, sx, n);
    } else if (nvec <= 2 * 1024) {
        hipLaunchKernelGGL((rmsnorm_act_quant_kernel<1024, 2>), dim3((unsigned)tokens), dim3(1024), 0, stream, x, gain, eps, tokens,
                           nvec, xq, sx, n);
    } else {
        return SBN_EUNSUPPORTED;   // rows longer than 16384 do not fit the registers of a block
    }
    return check_launch("rmsnorm_act_quant_kernel");
}

static void fill_gemv_item(GemvItem &g, const LinearItem &li)
{
    g.xq = li.xq; g.sx = li.sx; g.packed = static_cast<const uint8_t *>(li.packed);
    g.gamma = li.gamma; g.bias = li.bias; g.Y = li.Y; g.acc_out = li.acc_out;
    g.d_in = (int)li.d_in; g.d_out = (int)li.d_out; g.tokens = (int)li.tokens; g.d_x = (int)li.row_values();
    g.X = nullptr;
}

// multiprocessors of the current device (cached per thread)
int device_cus()
{
    static thread_local int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) cus = prop.multiProcessorCount;
        if (cus <= 0) cus = 256;
    }
    return cus;
}

template <int FORM>
static sbn_status launch_gemv_as(int count, const LinearItem *items, hipStream_t stream);

sbn_status launch_gemv(int count, const LinearItem *items, GemvForm form, hipStream_t stream)
{
    if (form != GEMV_1OF4 && gemv_takes_self(count, items)) return launch_gemm_self(count, items, form == GEMV_DENSE, stream);
    switch (form) {
    case GEMV_2OF4: return launch_gemv_as<GEMV_2OF4>(count, items, stream);
    case GEMV_DENSE: return launch_gemv_as<GEMV_DENSE>(count, items, stream);
    case GEMV_1OF4: return launch_gemv_as<GEMV_1OF4>(count, items, stream);
    }
    return SBN_EINVAL;
}

// Launch number of the streaming kernel with the fused quantizer: it tags the per-token flags a launch raises in
// the caller's workspace (never cleared), so that flags left by any earlier launch - of either instantiation of
// the kernel, on any workspace - can never be taken for this launch's.  One counter for the whole library.
static std::atomic<unsigned> g_gemv_stream_epoch{1};

// true while `stream` records into a graph (or when that cannot be told)
static bool stream_is_capturing(hipStream_t stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return status != hipStreamCaptureStatusNone;
}

constexpr size_t GEMV_SELF_LDS = 152 * 1024;   // next to 4 KB of maxima
// Row tiles of 16 from which a block takes two of them, in sixteenths of a multiprocessor: it then has more than one block either
// way, and the quantizer's work is done half as often (480 tiles, eight tokens: 5.9 us against 6.4; 160 tiles, one token: 4.1
// against 3.7).
constexpr int64_t GEMV_PAIR_TILES = 25;
// Every block quantizes all token rows, 0.04 to 0.06 us per 1000 values and block of a multiprocessor, where a launch of the
// quantizer in front costs 2.2 us on the device and another launch on the host.  Measured in this form and with the quantizer in
// front: 8192 -> 8192 9.9 us against 11.2 at eight tokens, 13.3 against 13.4 at 16; 4096 -> 28672 (three blocks per multiprocessor)
// 13.0 against 16.2 at eight, 25.5 against 20.6 at 16; 8192 -> 28672 33 against 29 at eight.
constexpr int64_t GEMV_SELF_VALUES = 16 * 8192;

// one launch of the row-tile kernels; tm = 0: on quantized activations, else the token slots of the kernel that quantizes
template <int FORM, int RT, int NI>
static sbn_status launch_gemv_rows(int n, const LinearItem *items, int nwaves, int ss, int tm, hipStream_t stream)
{
    GemvTable<NI> tab;
    int blocks = 0;
    int64_t tokens = 1;
    for (int i = 0; i < n; ++i) {
        fill_gemv_item(tab.it[i], items[i]);
        tab.it[i].X = static_cast<const uint4 *>(items[i].X);
        const int nb = (int)ceil_div(items[i].d_out, 16 * RT);
        blocks = nb > blocks ? nb : blocks;
        tokens = items[i].tokens > tokens ? items[i].tokens : tokens;
    }
    for (int i = n; i < NI; ++i) tab.it[i] = tab.it[0];
    const dim3 grid(blocks, n), block(64 * nwaves);
    if (tm == 0) {
        hipLaunchKernelGGL((gemv_smfmac_kernel<FORM, RT, NI>), grid, block, gemv_red_lds(nwaves, RT), stream, tab);
        return check_launch("gemv_smfmac_kernel");
    }
    const size_t lds = gemv_self_lds(tokens, nwaves, ss, RT);
    auto launch = [&](auto slots, auto steps) -> sbn_status {
        constexpr auto kernel = &gemv_self_kernel<FORM, RT, NI, slots(), steps()>;
        static thread_local bool raised = false;   // one for each kernel: the types of the arguments tell them apart
        if (!raised) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)GEMV_SELF_LDS);
            if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
            raised = true;
        }
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, tab);
        return check_launch("gemv_self_kernel");
    };
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    const std::integral_constant<int, 4> four;
    if (ss > 1) return tm == 2 ? (ss == 2 ? launch(two, two) : launch(two, four)) : ss == 2 ? launch(four, two) : launch(four, four);
    return tm == 2   ? launch(two, one)
           : tm == 4 ? launch(four, one)
           : tm == 8 ? launch(std::integral_constant<int, 8>(), one)
           : tm == 12 ? launch(std::integral_constant<int, 12>(), one)
                      : launch(std::integral_constant<int, 16>(), one);
}

template <int FORM>
static sbn_status launch_gemv_as(int count, const LinearItem *items, hipStream_t stream)
{
    constexpr int RT = 1;
    static thread_local std::vector<const int8_t *> written;   // xq buffers a quantizer kernel of this call has filled
    written.clear();
    // quantizer launches for the problems first .. first + n - 1 that still need one (shared inputs once)
    auto quantize_run = [&](int first, int n) -> sbn_status {
        for (int i = 0; i < n; ++i) {
            const LinearItem &li = items[first + i];
            if (li.quantized || std::find(written.begin(), written.end(), li.xq) != written.end()) continue;
            sbn_status st = launch_act_quant(li.X, li.tokens, li.row_values(), li.xq, li.sx, stream, li.d_in);
            if (st != SBN_OK) return st;
            written.push_back(li.xq);
        }
        return SBN_OK;
    };
    int first = 0;
    while (first < count) {
        // --- persistent streaming kernel when a run of problems holds enough rows to keep every block busy
        int n = count - first < GEMV_STREAM_MAX ? count - first : GEMV_STREAM_MAX;
        int64_t units = 0, lds_need = 16;
        bool plain = true;
        for (int i = 0; i < n; ++i) {
            const LinearItem &li = items[first + i];
            units += ceil_div(li.d_out, 16 * RT);
            const int64_t b = li.tokens * (li.d_in + 16) + 512;   // slack: reads past a ragged input dimension stay inside
            lds_need = b > lds_need ? b : lds_need;
            if (li.bias || li.acc_out) plain = false;
        }
        // one block of NW wavefronts per multiprocessor, sharing one staged copy of the activations
        const int nblocks = device_cus();
        constexpr int GEMV_STREAM_LDS = 160 * 1024 - 4608;   // the kernel's copy of the launch table, its counter and scales are static LDS
        if (plain && lds_need <= GEMV_STREAM_LDS && units >= 16 * (int64_t)nblocks) {
            // One row tile per unit, DEPTH 5 and 8 wavefronts per block measured best among one or two row tiles,
            // depths 2..8 and 6..16 wavefronts (more wavefronts finish their shares further apart, fewer leave too
            // few loads in flight; units of 16 rows balance the wavefronts better than units of 32: +2.5 to +4 %)
            // (the 1:4 form has half the bytes per super-step: twice the depth keeps the same bytes in flight)
            constexpr int DEPTH = FORM == GEMV_1OF4 ? 10 : 5, NW = 8;
            GemvStreamTable tab;
            tab.count = n;
            tab.nin = 0;
            for (int j = 0; j <= GEMV_STREAM_INPUTS; ++j) tab.tok0[j] = 0;
            // the kernel quantizes up to GEMV_STREAM_INPUTS distinct inputs itself; more than that (or rows too
            // long for one block's registers) go through the quantizer kernel first
            // Not under stream capture: the flags carry a per-launch number that the host hands out, and a replayed
            // graph would present the previous replay's flags again.  A captured launch takes the quantizer kernels.
            // One case needs neither flags nor producer blocks and is taken under capture as well: every problem of
            // the launch reads the same unquantized input and its rows fit a wavefront's registers; each block then
            // quantizes that input once, for itself, in front of its first problem and never stages anything else.
            bool fuse = true, one_input = true;
            int nin = 0;
            const int8_t *in_xq[GEMV_STREAM_INPUTS];
            for (int i = 0; i < n && fuse; ++i) {
                const LinearItem &li = items[first + i];
                if (li.quantized || std::find(written.begin(), written.end(), li.xq) != written.end()) { one_input = false; continue; }
                if (li.d_in > 8 * GEMV_QUANT_VEC * 64 * NW || li.tokens > 16 || li.row_values() != li.d_in) { fuse = false; break; }
                if (li.d_in > 8 * 64 * GEMV_OWN_VEC) one_input = false;
                bool seen = false;
                for (int j = 0; j < nin; ++j) seen = seen || in_xq[j] == li.xq;
                if (seen) continue;
                if (nin == GEMV_STREAM_INPUTS) { fuse = false; break; }
                in_xq[nin++] = li.xq;
            }
            one_input = one_input && fuse && nin == 1;
            if (fuse && !one_input && stream_is_capturing(stream)) fuse = false;
            if (!fuse) {
                sbn_status st = quantize_run(first, n);
                if (st != SBN_OK) return st;
                nin = 0;
            }
            int u = 0;
            for (int i = 0; i < n; ++i) {
                const LinearItem &li = items[first + i];
                GemvStreamItem &g = tab.it[i];
                g.xq = li.xq; g.sx = li.sx; g.packed = static_cast<const uint8_t *>(li.packed); g.gamma = li.gamma; g.Y = li.Y;
                g.d_in = (int)li.d_in; g.d_out = (int)li.d_out; g.tokens = (int)li.tokens; g.input = -1;
                for (int j = 0; j < nin; ++j)
                    if (in_xq[j] == li.xq) {
                        g.input = j;
                        if (j == tab.nin) {   // first problem with this input: describe it
                            GemvStreamInput &in = tab.in[j];
                            in.X = static_cast<const uint4 *>(li.X);
                            in.xq = reinterpret_cast<unsigned long long *>(li.xq);
                            in.sx = reinterpret_cast<unsigned *>(li.sx);
                            // the scales of at most 16 tokens fill 64 bytes of their 256-byte region; the flags take its second half
                            in.flags = reinterpret_cast<unsigned long long *>(reinterpret_cast<uint8_t *>(li.sx) + 128);
                            in.tokens = (int)li.tokens; in.d_in = (int)li.d_in;
                            tab.tok0[j + 1] = tab.tok0[j] + in.tokens;
                            ++tab.nin;
                        }
                    }
                tab.unit0[i] = u;
                u += (int)ceil_div(li.d_out, 16 * RT);
            }
            for (int i = n; i <= GEMV_STREAM_MAX; ++i) tab.unit0[i] = u;
            tab.share = u / nblocks;
            tab.share_rem = u % nblocks;
            tab.pad = 0;
            for (int j = tab.nin; j < GEMV_STREAM_INPUTS; ++j) tab.tok0[j + 1] = tab.tok0[tab.nin];
            if (one_input)   // no producer blocks: nobody would read what they publish
                for (int j = 0; j <= GEMV_STREAM_INPUTS; ++j) tab.tok0[j] = 0;
            tab.epoch = g_gemv_stream_epoch.fetch_add(1, std::memory_order_relaxed);
            tab.spin_limit = gemv_spin_limit();
            static thread_local bool raised = false;
            if (!raised) {
                hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemv_stream_kernel<RT, DEPTH, NW, FORM>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, GEMV_STREAM_LDS);
                if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
                raised = true;
            }
            hipLaunchKernelGGL((gemv_stream_kernel<RT, DEPTH, NW, FORM>), dim3(nblocks), dim3(64 * NW), (size_t)lds_need, stream, tab);
            sbn_status st = check_launch("gemv_stream_kernel");
            if (st != SBN_OK) return st;
            first += n;
            continue;
        }
        // --- otherwise: blocks of 16 or 32 rows, wavefronts split the input dimension (lowest latency)
        n = count - first < GEMV_MAX_ITEMS ? count - first : GEMV_MAX_ITEMS;
        int most_super = 1;
        int64_t tiles = 0, most_tokens = 1;
        bool self_quant = true;
        for (int i = 0; i < n; ++i) {
            const LinearItem &li = items[first + i];
            const int nsuper = (int)ceil_div(li.d_in, 4 * CHUNK);
            most_super = nsuper > most_super ? nsuper : most_super;
            most_tokens = li.tokens > most_tokens ? li.tokens : most_tokens;
            tiles += ceil_div(li.d_out, 16);
            if (li.quantized || std::find(written.begin(), written.end(), li.xq) != written.end()) self_quant = false;
        }
        // one wavefront per super-step up to 16, so that every wavefront has loads in flight at once
        const int nwaves = most_super < GEMV_SELF_SUPER ? most_super : GEMV_SELF_SUPER;
        const int rt = 16 * tiles >= GEMV_PAIR_TILES * device_cus() ? 2 : 1;
        const int64_t per_cu = std::max<int64_t>(1, tiles / rt / device_cus());
        // Longer rows: two or four super-steps per wavefront while their values fit the registers, up to four tokens.  us in this
        // form and with the separate quantizer: 14336 -> 4096 at 1 / 2 / 3 tokens 7.7 / 8.4 / 9.3 against 10.3 / 10.7 / 11.1, 28672 -> 8192
        // 17 / 18 / 20 against 44 / 46 / 49 (the other form reads rows this long past the vector L1 again and again); but with two row tiles
        // per block and two super-steps, at one token 9216 -> 16384 15.1 against 16.6, at three 21.2 against 17.4.
        const int rounds = (int)ceil_div(most_super, GEMV_SELF_SUPER), ss = rounds <= 2 ? rounds : 4;
        if (rounds > 4 || (rounds > 1 && most_tokens > (rounds == 2 && rt == 2 ? 2 : 4)) || most_tokens * most_super * 512 * per_cu > GEMV_SELF_VALUES ||
            gemv_self_lds(most_tokens, nwaves, ss, rt) > GEMV_SELF_LDS)
            self_quant = false;
        if (!self_quant) {
            sbn_status st = quantize_run(first, n);
            if (st != SBN_OK) return st;
        }
        const int tm = !self_quant ? 0 : most_tokens <= 2 ? 2 : most_tokens <= 4 ? 4 : most_tokens <= 8 ? 8 : most_tokens <= 12 ? 12 : 16;
        sbn_status st = n <= GEMV_FEW ? (rt == 2 ? launch_gemv_rows<FORM, 2, GEMV_FEW>(n, items + first, nwaves, ss, tm, stream) : launch_gemv_rows<FORM, 1, GEMV_FEW>(n, items + first, nwaves, ss, tm, stream))
                                      : (rt == 2 ? launch_gemv_rows<FORM, 2, GEMV_MAX_ITEMS>(n, items + first, nwaves, ss, tm, stream) : launch_gemv_rows<FORM, 1, GEMV_MAX_ITEMS>(n, items + first, nwaves, ss, tm, stream));
        if (st != SBN_OK) return st;
        first += n;
    }
    return SBN_OK;
}

sbn_status launch_linear_generic(const LinearItem &it, const Pattern &pat, hipStream_t stream)
{
    dim3 grid((unsigned)ceil_div(it.d_out, 128), (unsigned)ceil_div(it.tokens, 8));
    hipLaunchKernelGGL(linear_generic_kernel, grid, dim3(128), 0, stream, it.xq, it.sx,
                       static_cast<const uint8_t *>(it.packed), it.gamma, it.bias, it.Y, it.acc_out, it.tokens,
                       (int)it.d_in, (int)it.d_out, pat);
    return check_launch("linear_generic_kernel");
}

}  // namespace sbn
