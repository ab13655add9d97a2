// Backward products of the sparse ternary linear layer under the dual straight-through estimator
// (Section 2.3; Appendix B listing, backward()):
//   dX[t,k] = gamma * sum_o dY[t,o] * W_eff[o,k]          contraction over d_out
//   dW[o,k] = sum_t (dY[t,o] / s_x[t]) * xq[t,k]          contraction over tokens; dense, unmasked
// Both run on the dense bf16 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation): the 2:4
// structure lies along d_in, which is not the contracted dimension of either product, so the sparse
// instruction does not apply.  One GEMM kernel serves both: dY, and dY / s_x in the same layout, are read as they lie (dW
// contracts their slow dimension: the transposing LDS read), one kernel writes dY / s_x and puts W_eff^T (a byte per weight) and x~^T
// (exact in bf16) contraction-major first.
#include <algorithm>
#include <vector>

#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

// two values rounded to bf16 (to nearest, ties to even), lo in the low half: v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2bf));
}

// ---- layout kernels -------------------------------------------------------------------------------
// One quarter (32 weights, quarter P of its chunk) of a packed row: put(k, code) for every slot, k = weight inside the quarter.
template <int N, int M, int P, class Put>
__device__ __forceinline__ void decode_quarter(const uint32_t *chunk, Put &&put)
{
    constexpr int B = N == M ? 0 : M == 2 ? 1 : M == 4 ? 2 : 3;
    constexpr int SLOTS = 32 * N / M, FIRST = SLOTS * P;                 // slots of the quarter, its first one
    constexpr int IDX_WORDS = 128 * N / M * B / 32;                      // words of the chunk's index field (a whole number here)
    constexpr int I0 = FIRST * B / 32, I1 = B ? ((FIRST + SLOTS) * B - 1) / 32 : I0, C0 = FIRST / 16, C1 = (FIRST + SLOTS - 1) / 16;
    uint32_t iw[I1 - I0 + 2], cw[C1 - C0 + 1];
#pragma unroll
    for (int i = 0; i <= I1 - I0; ++i) iw[i] = B ? chunk[I0 + i] : 0u;
    iw[I1 - I0 + 1] = 0;
#pragma unroll
    for (int i = 0; i <= C1 - C0; ++i) cw[i] = chunk[IDX_WORDS + C0 + i];
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) {
        const int slot = FIRST + i, v = slot & 15, bit = slot * B - 32 * I0;
        const uint32_t code = (cw[slot / 16 - C0] >> (8 * (v & 3) + 2 * (v >> 2))) & 3u;
        uint32_t j = (uint32_t)(i % N);
        if (B) j = ((bit & 31) + B <= 32 ? iw[bit >> 5] >> (bit & 31) : __funnelshift_r(iw[bit >> 5], iw[(bit >> 5) + 1], bit & 31)) & ((1u << B) - 1u);
        put(i / N * M + (int)j, code);
    }
}

// W_eff^T for dX: a byte per weight, the high half of the bf16 value +-0.5 or 0 (the low half is zero).  [d_in, ld], ld >= d_out a
// multiple of 128, zeros for rows of W past d_out.  One tile is 128 rows of W x 128 weights, so that whole cache lines leave.
constexpr int TB = 128 + 16;   // pitch of a row of the tile
constexpr uint32_t code_byte(uint32_t code) { return code == 0 ? 0u : code == 1 ? 0x3fu : 0xbfu; }

__device__ __forceinline__ void write_code_tile(const uint8_t *tile, uint8_t *__restrict__ dst, int64_t ld, int64_t k0, int64_t o0, int64_t kmax)
{
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = threadIdx.x + 256 * i, row = v >> 3, col = (v & 7) * 16;
        if (k0 + row < kmax) *reinterpret_cast<uint4 *>(dst + (k0 + row) * ld + o0 + col) = *reinterpret_cast<const uint4 *>(tile + row * TB + col);
    }
}

// from packed weights, a wavefront per quarter of the chunk
template <int N, int M>
__device__ __forceinline__ void unpack_transpose_tile(const uint8_t *__restrict__ packed, int d_out, int d_in, uint8_t *__restrict__ wt, int64_t ld,
                                                      int chunk, int o0, uint8_t *tile)
{
    constexpr int B = N == M ? 0 : M == 2 ? 1 : M == 4 ? 2 : 3, CHUNK_WORDS = 128 * N / M * (2 + B) / 32;
    const int nchunks = (d_in + CHUNK - 1) / CHUNK;
    const int quarter = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = threadIdx.x & 63; k < 32 * 8; k += 64) *reinterpret_cast<uint4 *>(tile + (32 * quarter + (k >> 3)) * TB + 16 * (k & 7)) = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int ro = 64 * half + (threadIdx.x & 63), o = o0 + ro;
        uint8_t *const col = tile + 32 * quarter * TB + ro;
        if (o >= d_out) continue;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(packed) + ((int64_t)o * nchunks + chunk) * CHUNK_WORDS;
        auto put = [&](int k, uint32_t code) {
            if (code) col[k * TB] = (uint8_t)(code == 1u ? code_byte(1) : code_byte(3));
        };
        if (quarter == 0) decode_quarter<N, M, 0>(src, put);
        else if (quarter == 1) decode_quarter<N, M, 1>(src, put);
        else if (quarter == 2) decode_quarter<N, M, 2>(src, put);
        else decode_quarter<N, M, 3>(src, put);
    }
    write_code_tile(tile, wt, ld, (int64_t)chunk * CHUNK, o0, d_in);
}

// from int8 W_eff [rows, cols] (patterns without a decoder here), cols a multiple of 8.  Bound by the bytes in and out: rows go into LDS as
// they are read, their granules of 16 bytes XOR-swizzled with row / 16; a thread takes four weights of 16 rows back, 16 words, and
// transposes them with byte permutations, so that whole 128 bytes leave.  Byte by byte the launch took 24.5 us at 2560 x 2560 and
// 3:4, a byte per weight and half the bytes of the bf16 form that took 9.7; this way 6.7.
__device__ __forceinline__ void transpose_codes_tile(const int8_t *__restrict__ src, int64_t rows, int64_t cols, uint8_t *__restrict__ wt, int64_t ld,
                                                     int64_t k0, int64_t o0, uint8_t *tile)
{
    const int g = threadIdx.x & 7;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = 32 * i + (int)(threadIdx.x >> 3);
        uint2 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t k = k0 + 16 * g + 8 * h;
            v[h] = o0 + o < rows && k < cols ? *reinterpret_cast<const uint2 *>(src + (o0 + o) * cols + k) : make_uint2(0, 0);
        }
        // 0, 1, -1 -> 0x00, 0x3f, 0xbf: 63 times the lowest bit, and the sign
        auto coded = [](uint32_t w) { const uint32_t n = w & 0x01010101u; return ((n << 6) - n) | (w & 0x80808080u); };
        *reinterpret_cast<uint4 *>(tile + o * 128 + 16 * (g ^ ((o >> 4) & 7))) = make_uint4(coded(v[0].x), coded(v[0].y), coded(v[1].x), coded(v[1].y));
    }
    static_assert(code_byte(1) == 0x3f && code_byte(3) == 0xbf, "as above");
    __syncthreads();
    const int kg = threadIdx.x >> 3;   // rows 16 g .. + 15, weights 4 kg .. + 3
    if (k0 + 4 * kg >= cols) return;
    uint32_t out[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const uint32_t *>(tile + (16 * g + 4 * q + i) * 128 + 16 * ((kg >> 2) ^ g) + 4 * (kg & 3));
        const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
        const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
        out[0][q] = __builtin_amdgcn_perm(c, a, 0x05040100u);
        out[1][q] = __builtin_amdgcn_perm(c, a, 0x07060302u);
        out[2][q] = __builtin_amdgcn_perm(d, b, 0x05040100u);
        out[3][q] = __builtin_amdgcn_perm(d, b, 0x07060302u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        *reinterpret_cast<uint4 *>(wt + (k0 + 4 * kg + j) * ld + o0 + 16 * g) = make_uint4(out[j][0], out[j][1], out[j][2], out[j][3]);
}

// int8 [rows, cols] -> bf16 transposed: dst [cols, ld] with dst[c, r] = src[r, c], zeros for r in [rows, ld), ld a multiple of 64;
// one tile of 64 rows x 128 columns, so that reads and writes are whole cache lines (rows of 64 bytes were asked for by two
// XCDs each).  Rows go into LDS as they are read; a thread takes eight rows of a pair of columns back (a word each) and
// sorts them into two vectors.  Pitch of 65 words: the 64 words of a read lie in different banks.
constexpr int TQ = 128 + 2;
__device__ __forceinline__ void transpose_i8_tile(const int8_t *__restrict__ src, int64_t rows, int64_t cols, uint16_t *__restrict__ dst,
                                                  int64_t ld, int64_t c0, int64_t r0, uint16_t *tile)
{
    const int cv = (threadIdx.x & 7) * 16;   // one 16-byte vector of two source rows per thread
    __attribute__((aligned(16))) int8_t q[2][16];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t row = r0 + 32 * h + (threadIdx.x >> 3);
        const bool row_ok = row < rows;
        if (row_ok && c0 + cv + 16 <= cols && (cols & 15) == 0) {
            *reinterpret_cast<uint4 *>(q[h]) = *reinterpret_cast<const uint4 *>(src + row * cols + c0 + cv);
        } else {
            for (int e = 0; e < 16; ++e) q[h][e] = (row_ok && c0 + cv + e < cols) ? src[row * cols + c0 + cv + e] : (int8_t)0;
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 16; e += 2)   // |q| <= 128: exact in bf16, the high half of the fp32 value
            *reinterpret_cast<uint32_t *>(&tile[(32 * h + (threadIdx.x >> 3)) * TQ + cv + e]) =
                __builtin_amdgcn_perm(__float_as_uint((float)q[h][e + 1]), __float_as_uint((float)q[h][e]), 0x07060302u);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int v = threadIdx.x + 256 * h, b = (v >> 3) * 2, av = (v & 7) * 8;
        if (c0 + b >= cols) continue;
        uint32_t w[8], lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = *reinterpret_cast<const uint32_t *>(&tile[(av + i) * TQ + b]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x05040100u);
            hi[i] = __builtin_amdgcn_perm(w[2 * i + 1], w[2 * i], 0x07060302u);
        }
        uint16_t *d = dst + (c0 + b) * ld + r0 + av;   // columns are a multiple of 8: both of a pair exist
        *reinterpret_cast<uint4 *>(d) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        *reinterpret_cast<uint4 *>(d + ld) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    }
}

// dY [tokens, 8 nvec] bf16 -> dY[t, :] / s_x[t], rounded to bf16 (the one rounding of an operand of dW), same layout.  It is the
// gradient that is rounded and not x~ / s_x, of which a row has 255 values at most: the error of a gradient is another one in
// every token, that of a level would be the same wherever tokens share s_x (saturated or clipped activations) and add up over
// them, and it would depend on where the levels lie between two powers of two, i.e. on the amplitude of the activations.
// Four rows from t0 on, vector i of 8 values; the quotient is the IEEE one for all operands.  Zeros and |a| in [2^-90, 2^100) over s in
// [2^-20, 2^30) (s_x of rows whose largest value lies between 2^-23 and 2^26) take Markstein's form: with r = 1 / s rounded once
// per row, a r and one correction by the remainder.  There the quotient is normal and the remainder exact, so the result depends
// on the two significands alone, and for all 2^7 of a bf16 times 2^23 of an fp32 it is the rounded quotient (compared one by one
// on the CPU).  Outside that range the form is not the quotient (a r = inf is corrected to NaN, a remainder that underflows loses
// its end), and a lane that has met any such operand divides.  The range check is a minimum and a maximum per two values; a
// training step's time does not show it (1024 tokens 2560 x 6912 313.0 us without and 313.2 with it, a block at 16384 5798 and 5802).
constexpr unsigned QUOT_A_MIN = (127 - 90) << 7;     // bf16 magnitude
constexpr float QUOT_A_END = 0x1p100f;
constexpr unsigned QUOT_S_MIN = (127u - 20) << 23, QUOT_S_END = (127u + 30) << 23;
__device__ __forceinline__ void scale_four_rows(const uint4 *__restrict__ dY, const float *__restrict__ sx, int64_t tokens, int nvec,
                                                uint4 *__restrict__ dst, int64_t t0, int i)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    uint4 v[4];
    float s[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + r < tokens ? t0 + r : tokens - 1;   // past the end the last row again (not stored)
        v[r] = dY[t * nvec + i];
        s[r] = sx[t];
    }
    float most = 0.0f;               // largest magnitude, NaN for any NaN
    u16x2 least = {0xffff, 0xffff};  // smallest of twice the magnitude less one, of which zeros have the largest
    unsigned scales = 0;
    uint32_t o[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t w[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
        const float inv = __fdiv_rn(1.0f, s[r]);
        auto over_s = [&](float a) {
            const float q = a * inv;
            return __builtin_fmaf(__builtin_fmaf(-q, s[r], a), inv, q);   // of zeros without the sign: a sum of dW begins with +0
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float lo = __uint_as_float(w[k] << 16), hi = __uint_as_float(w[k] & 0xffff0000u);
            uint32_t twice;
            asm("v_pk_mad_u16 %0, %1, 2, -1 op_sel_hi:[1,0,0]" : "=v"(twice) : "v"(w[k]));
            least = __builtin_elementwise_min(least, __builtin_bit_cast(u16x2, twice));
            asm("v_maximum3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(lo), "v"(hi));
            o[r][k] = pack_bf16(over_s(lo), over_s(hi));
        }
        scales = max(scales, __float_as_uint(s[r]) - QUOT_S_MIN);
    }
    if (scales < QUOT_S_END - QUOT_S_MIN && most < QUOT_A_END && min(least.x, least.y) >= 2 * QUOT_A_MIN - 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (t0 + r < tokens) dst[(t0 + r) * nvec + i] = make_uint4(o[r][0], o[r][1], o[r][2], o[r][3]);
        return;
    }
#pragma unroll 1
    for (int64_t t = t0; t < t0 + 4 && t < tokens; ++t) {
        const uint4 d = dY[t * nvec + i];
        const float st = sx[t];
        auto over = [&](uint32_t w) { return pack_bf16(__fdiv_rn(__uint_as_float(w << 16), st), __fdiv_rn(__uint_as_float(w & 0xffff0000u), st)); };
        dst[t * nvec + i] = make_uint4(over(d.x), over(d.y), over(d.z), over(d.w));
    }
}

// All operands of a call's products in one launch: W_eff^T (128 rows of W x one chunk per block), the transpose of x~ (64 x 128
// per block) and dY / s_x (256 x four rows of eight values per block).  Bound by the bytes that they move; the decoders, which wait for their LDS, run beside the streams.
// One launch per layer for W_eff^T and one for the other two left the device in a tail seven to fourteen times per training
// step, and a block with 256 vectors of one row quad alone left a third of its lanes idle at 2560 outputs.  us per step of a block at
// 16384 tokens, before and then: 617 -> 462 (5.6 to 5.8 TB/s; less by the half of W_eff^T since that is a byte per weight); 6912 x 2560 at 1024 tokens (6:8) 23.0 -> 17.8.
enum OperandKind { OPERAND_UNPACK, OPERAND_CODES, OPERAND_TRANSPOSE, OPERAND_SCALE };   // W_eff^T from packed weights, from int8; x~^T; dY / s_x
struct OperandJob {
    const void *src;
    const float *sx;
    void *dst;
    int64_t ld;        // row length of dst (all but scale)
    int rows, cols;    // of src; scale: tokens and vectors of eight values per token
    int across;        // blocks along the columns of src, 128 each
    int kind;
};
constexpr int OPERAND_JOBS_MAX = 24;
struct OperandGroup {
    OperandJob job[OPERAND_JOBS_MAX];
    int block0[OPERAND_JOBS_MAX + 1];
    int count;
};

template <int N, int M>   // 0, 0: no unpacking among the jobs
__global__ void __launch_bounds__(256) operands_kernel(OperandGroup grp)
{
    __shared__ __attribute__((aligned(16))) uint8_t tile[128 * TB > 128 * TQ ? 128 * TB : 128 * TQ];
    int j = 0;
    while (j + 1 < grp.count && (int)blockIdx.x >= grp.block0[j + 1]) ++j;
    const OperandJob &job = grp.job[j];
    const unsigned b = blockIdx.x - grp.block0[j];
    if (job.kind == OPERAND_SCALE) {
        // the vectors of a row quad one after another; a block starts at vector `first` of quad `quad`
        const unsigned nvec = job.cols;
        unsigned quad = b * 256 / nvec;   // vectors of a whole dY / 4: below 2^32 for any that fits the device
        unsigned i = b * 256 - quad * nvec + threadIdx.x;
        if (nvec >= 256) {
            if (i >= nvec) { i -= nvec; ++quad; }
        } else {
            quad += i / nvec;
            i %= nvec;
        }
        if (quad < (unsigned)(job.rows + 3) / 4)
            scale_four_rows(static_cast<const uint4 *>(job.src), job.sx, job.rows, (int)nvec, static_cast<uint4 *>(job.dst), 4 * (int64_t)quad, (int)i);
        return;
    }
    const int across = (int)(b % job.across), down = (int)(b / job.across);
    if constexpr (N != 0) {
        if (job.kind == OPERAND_UNPACK) {
            unpack_transpose_tile<N, M>(static_cast<const uint8_t *>(job.src), job.rows, job.cols, static_cast<uint8_t *>(job.dst), job.ld, across, 128 * down,
                                        tile);
            return;
        }
    }
    if (job.kind == OPERAND_CODES) {
        transpose_codes_tile(static_cast<const int8_t *>(job.src), job.rows, job.cols, static_cast<uint8_t *>(job.dst), job.ld, 128 * (int64_t)across,
                             128 * (int64_t)down, tile);
        return;
    }
    transpose_i8_tile(static_cast<const int8_t *>(job.src), job.rows, job.cols, static_cast<uint16_t *>(job.dst), job.ld, 128 * (int64_t)across,
                      64 * (int64_t)down, reinterpret_cast<uint16_t *>(tile));
}

// The jobs of a call, unpacking first (their blocks take longest), dealt out in launches of OPERAND_JOBS_MAX.
sbn_status launch_operands(const std::vector<OperandJob> &jobs, const Pattern &pat, hipStream_t stream)
{
    for (size_t first = 0; first < jobs.size(); first += OPERAND_JOBS_MAX) {
        OperandGroup grp;
        grp.count = (int)std::min(jobs.size() - first, (size_t)OPERAND_JOBS_MAX);
        std::copy_n(jobs.begin() + first, grp.count, grp.job);
        std::stable_sort(grp.job, grp.job + grp.count, [](const OperandJob &a, const OperandJob &b) { return a.kind < b.kind; });
        int64_t blocks = 0;
        for (int i = 0; i < grp.count; ++i) {
            const OperandJob &j = grp.job[i];
            grp.block0[i] = (int)blocks;
            blocks += j.kind == OPERAND_SCALE ? ceil_div(ceil_div(j.rows, 4) * (int64_t)j.cols, 256) : j.across * (j.ld / (j.kind == OPERAND_TRANSPOSE ? 64 : 128));
        }
        for (int i = grp.count; i <= OPERAND_JOBS_MAX; ++i) grp.block0[i] = (int)blocks;
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, grp); };
        if (grp.job[0].kind != OPERAND_UNPACK) launch(operands_kernel<0, 0>);
        else if (pat.N == pat.M) launch(operands_kernel<8, 8>);   // dense codes look the same for every M
        else if (pat.N == 2 && pat.M == 4) launch(operands_kernel<2, 4>);
        else if (pat.N == 6) launch(operands_kernel<6, 8>);
        else if (pat.N == 1) launch(operands_kernel<1, 4>);
        else launch(operands_kernel<2, 8>);
        const sbn_status st = check_launch("operands_kernel");
        if (st != SBN_OK) return st;
    }
    return SBN_OK;
}

// patterns that operands_kernel decodes itself
bool has_unpack(const Pattern &pat)
{
    return pat.N == pat.M || (pat.N == 2 && pat.M == 4) || (pat.N == 6 && pat.M == 8) || (pat.N == 1 && pat.M == 4) || (pat.N == 2 && pat.M == 8);
}

// ---- bf16 GEMM -------------------------------------------------------------------------------------------
// C[m, n] (+)= alpha * sum_k Q[m, k] * P[n, k], C bf16 [M, ldc].  P is [N, ldp] with k contiguous and K a multiple of 64
// (the layout kernels pad it with zeros).  Q has k contiguous as well ([M, ldq], dX), or lies the other way round
// ([k, ldq] with m contiguous, transposed: dW reads dY / s_x as it lies); it may end before K.
// P supplies the rows of the MFMA result so that a lane ends up with four consecutive n of one C row (one 8-byte store).
struct GemmBf16Args {
    const void *P;        // bf16, or (not transposed) a byte per value: see bf16_dx_body
    const uint16_t *Q;
    uint16_t *C;
    const float *alpha;   // device scalar or null (= 1)
    int64_t ldp, ldq, ldc;
    int N, M, K;
    int kq;               // k that Q has (<= K)
    int transposed;       // Q is [k, ldq]
    int accumulate;
    int tiles_n, tiles_m;
    const uint8_t *mask;    // null, or one bit per element of C (rows of mask_pitch bytes): zero bits block the new term
    int mask_pitch;
};

// Tile order.  Blocks go to the eight XCDs round-robin and every XCD has its own L2, so XCD x takes
// a contiguous eighth of an order in which consecutive tiles form compact rectangles: super-tiles of
// 8 x 8 tiles (3072 operand rows for 64 tiles instead of up to all of them), bands of eight tile rows,
// super-tiles left to right in a band, the row index fastest inside a super-tile.  With plain row-major
// order the L2s missed on two thirds of their requests.  bid = block index inside the product's
// range; returns false for the blocks that pad the range to a multiple of eight.
__device__ __forceinline__ bool bf16_tile_of_block(const GemmBf16Args &g, int bid, int &tn, int &tm)
{
    const int nb = g.tiles_n * g.tiles_m;
    const int per = (nb + 7) >> 3;
    const int id = (bid & 7) * per + (bid >> 3);
    if ((bid >> 3) >= per || id >= nb) return false;
    const int band_tiles = 8 * g.tiles_n;
    const int nbands = (g.tiles_m + 7) >> 3;
    int band = id / band_tiles;
    band = band < nbands - 1 ? band : nbands - 1;
    const int h = band == nbands - 1 ? g.tiles_m - 8 * band : 8;      // tile rows of this band
    const int rem = id - band * band_tiles;
    const int ncols = (g.tiles_n + 7) >> 3;
    int col = rem / (8 * h);
    col = col < ncols - 1 ? col : ncols - 1;
    const int rem2 = rem - col * 8 * h;
    tn = 8 * col + rem2 / h;
    tm = 8 * band + rem2 % h;
    return true;
}

// Result of a wavefront: WP x WQ tiles of 32 x 32 at rows (of C) mw + 32 b + .., columns nw + 32 a + ..; tile (a, b): lane
// holds m = column r, n = rows 8q + 4c + i.  Stored from there, an instruction would touch 32 rows with 16 bytes each
// (16 us of a tile of 256 x 256, next to 60 us of matrix work at 2560 k).  So 32 rows at a time go through the wavefront's
// 16 KB of the idle stages in fp32 (granules of 16 bytes XOR-swizzled with the row) and leave as whole rows of the
// wavefront's tile, 16 bytes per lane.  N is a multiple of 8.  A wavefront's LDS operations complete in order, so the next 32 rows
// are written behind the reads of the last ones without a wait, and what is already in C is asked for in front of them.
template <int WP, int WQ>
__device__ __forceinline__ void bf16_wave_epilogue(const GemmBf16Args &g, const v16f (&acc)[WP][WQ], const float alpha, uint8_t *stg, int nw, int mw, int lane)
{
    constexpr int ROW = WP * 128, LPR = ROW / 32, J = 32 * LPR / 64;     // bytes of a staged row, lanes per row, stores of 32 rows
    const int r = lane & 31, c = lane >> 5;
    const int h = lane % LPR, n = nw + 8 * h;
    const int m0 = mw + lane / LPR, rows = n < g.N ? g.M - m0 : 0;     // of C, from the lane's first on
    const int64_t step = (int64_t)(64 / LPR) * g.ldc;
    uint16_t *dst = g.C + (int64_t)m0 * g.ldc + n;
    auto inside = [&](const int b, const int j) { return 32 * b + (64 / LPR) * j < rows; };
    auto at = [&](uint16_t *&p) {   // address by address: all of them at once would not fit the registers
        uint4 *const here = reinterpret_cast<uint4 *>(p);
        p += step;
        asm volatile("" : "+v"(p));
        return here;
    };
    v4f lo[J], hi[J];
    auto read = [&](const int first, const int n) {   // staged rows of stores [first, first + n)
#pragma unroll
        for (int j = first; j < first + n; ++j) {
            const int row = (64 / LPR) * j + lane / LPR;
            lo[j] = *reinterpret_cast<const v4f *>(stg + row * ROW + 16 * ((2 * h) ^ (row & 15)));
            hi[j] = *reinterpret_cast<const v4f *>(stg + row * ROW + 16 * ((2 * h + 1) ^ (row & 15)));
        }
        asm volatile("" ::: "memory");   // the next rows' writes stay behind them
    };
    auto stage = [&](const int b) {
#pragma unroll
        for (int a = 0; a < WP; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<v4f *>(stg + r * ROW + 16 * ((8 * a + 2 * q + c) ^ (r & 15))) =
                    v4f{acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
        asm volatile("" ::: "memory");   // the reads are of what other lanes have written
    };
    if (!g.accumulate && !g.mask) {
#pragma unroll
        for (int b = 0; b < WQ; ++b) {
            stage(b);
            read(0, J);
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint4 o = make_uint4(pack_bf16(lo[j][0] * alpha, lo[j][1] * alpha), pack_bf16(lo[j][2] * alpha, lo[j][3] * alpha),
                                           pack_bf16(hi[j][0] * alpha, hi[j][1] * alpha), pack_bf16(hi[j][2] * alpha, hi[j][3] * alpha));
                uint4 *const out = at(dst);
                if (inside(b, j)) *out = o;
            }
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < WQ; ++b) {
        uint4 old[J];
        uint16_t *from = dst;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint4 *const in = at(from);
            old[j] = make_uint4(0, 0, 0, 0);
            if (g.accumulate && inside(b, j)) old[j] = *in;
        }
        stage(b);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (j % (J / 2) == 0) read(j, J / 2);   // in two parts, beside what is in C already
            uint4 *const out = at(dst);
            if (!inside(b, j)) continue;
            float v[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] = lo[j][i] * alpha; v[4 + i] = hi[j][i] * alpha; }
            if (g.mask) {   // n is a multiple of 8: its mask bits sit in one byte
                const int m = m0 + 32 * b + (64 / LPR) * j;
                const uint32_t mb = g.mask[(int64_t)m * g.mask_pitch + (n >> 3)];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = (mb >> i) & 1u ? v[i] : 0.0f;
            }
            if (g.accumulate) {
                const uint32_t w[4] = {old[j].x, old[j].y, old[j].z, old[j].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[2 * i] += __uint_as_float(w[i] << 16);
                    v[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
                }
            }
            *out = make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        }
    }
}

// One launch covers the tiles of up to GB_GROUP_MAX products (dW and dX of the layers of a call): product p owns the blocks
// [block0[p], block0[p + 1]), longest contraction first, so that the short tiles fill the multiprocessors the long ones
// leave idle.  Each range starts at a multiple of 8 (the blocks in between exit at once), which keeps block index
// mod 8 = XCD for the tile order above.
constexpr int GB_GROUP_MAX = 8;
struct GemmBf16Group {
    GemmBf16Args g[GB_GROUP_MAX];
    int block0[GB_GROUP_MAX + 1];
    int count;
};

__device__ __forceinline__ int bf16_product_of_block(const GemmBf16Group &grp)
{
    int prob = 0;
    while (prob + 1 < grp.count && (int)blockIdx.x >= grp.block0[prob + 1]) ++prob;
    return prob;
}

// Block tile 256 x 256 with eight wavefronts of 128 (n) x 64 (m), or 128 x 128 with four of 64 x 64 (two blocks per
// multiprocessor), stages of 64 k filled by LDS-DMA: a ring of five slots that the two operands take in turns, so that P lies in
// LDS two stages ahead and Q one.  A stage is consumed in quarters of 16 k; the fragments of the next quarter are read under the
// matrix instructions of the current one, also across the barrier between two stages, and the requests for later stages
// stand there as well, so a wavefront always has matrix instructions to issue: 1.42 us per stage of the large tile of dW, 1.38 of
// dX, where one barrier, eight requests and a first read in front of every stage's matrix instructions took 1.9 us.  What bounds
// it now: the matrix pipe at the clock the board's power holds (1.85 to 1.89 PFLOP/s on operands from registers for dW, 1.95 to 2.03
// for the ternary operand of dX) inside a tile, 2.5 us per tile for its first stages and 3.2 for its result, which nothing covers, and
// rounds of tiles that end unevenly: 1.2 to 1.4 PFLOP/s over a launch of a training step.
// The fifth slot is what LDS has left beside two whole stages.  With two, all requests of a stage had three quarters of one to
// arrive in: three layers of 2560 x 2560 at 16384 tokens 943 us then and 927 now (the products alone), two of 6912 x 2560 1844
// and 1806, a training step of 6912 x 2560 in two parts of 1024 tokens (small tiles) 324 and 306.
constexpr int GD_K = 64;     // k per stage
template <bool BIG> struct Bf16Tile {
    static constexpr int N = BIG ? 256 : 128, M = BIG ? 256 : 128;
    static constexpr int WAVES = BIG ? 8 : 4, WN = 2, WM = WAVES / WN;       // wavefronts along n and m
    static constexpr int WP = N / WN / 32, WQ = M / WM / 32;                 // 32 x 32 tiles of a wavefront: 4 x 2 or 2 x 2
    static constexpr int SLOT = N * GD_K * 2, SLOTS = 5;                     // one operand's share of a stage
    static constexpr int LDS = SLOTS * SLOT, STAGING = 4 * SLOT / WAVES;     // the last: of a wavefront, for its result
    static_assert(M == N, "the two operands take turns in the slots");
};

// dW: P bf16, Q transposed.
template <bool BIG>
__device__ __forceinline__ void bf16_dw_body(const GemmBf16Args &g, uint8_t *dlds, int n0, int m0)
{
    using S = Bf16Tile<BIG>;
    constexpr int WP = S::WP, WQ = S::WQ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;
    const int r = lane & 31, c = lane >> 5;
    const uint32_t lds0 = lds_address(dlds);
    const int nk = g.K / GD_K;
    const float alpha = g.alpha ? *g.alpha : 1.0f;   // here it is a scalar load: in front of everything that writes memory

    // DMA roles, four instructions per operand and wavefront.  P: one instruction fills 8 rows x 128 bytes (lane l:
    // row l / 8, slot l % 8 holding global column slot ^ ((row >> 1) & 7)).  Q: a stage is 64 k rows of M values,
    // one instruction fills 1024 bytes of them, slot s of row k holds the eight values of granule s ^ f(k),
    // f = 4 (k & 3) | 2 ((k >> 2) & 1): the four k rows that a transposing read of 16 lanes takes lie in different banks.
    // Operands are buffers that move on with the stages: rows and k rows past the matrix, and stages past the last, read as zeros and fetch
    // nothing.  Their size has 32 bits: of P it ends with the last row's part of the stage, of Q with the stage's rows unless those are longer
    // than anything that is asked for (launch_backward_grouped sees to the rest).
    constexpr int QROW = S::M * 2;                        // bytes of a k row of a stage
    const int kleft = g.kq - (nk - 1) * GD_K;             // k of the last stage that Q has
    const int prows = g.N - n0 < S::N ? g.N - n0 : S::N;
    const uint32_t ppitch = 2u * (uint32_t)g.ldp;
    const uint32_t qpitch = 2u * (uint32_t)g.ldq, pbytes = (uint32_t)(prows - 1) * ppitch + GD_K * 2;
    auto up_to_end = [&](const int k) { return (uint32_t)std::min((uint64_t)k * qpitch - 2u * (uint32_t)m0, (uint64_t)0xfffffff0u); };   // of k rows
    const uint32_t qbytes = up_to_end(GD_K), qbytes_last = up_to_end(kleft);
    v4i pbuffer = buffer_of(static_cast<const uint16_t *>(g.P) + (int64_t)n0 * g.ldp, pbytes);
    v4i qbuffer = buffer_of(g.Q + m0, nk > 1 ? qbytes : qbytes_last);
    uint64_t qstep = (uint64_t)g.ldq * (GD_K * 2);
    asm volatile("" : "+s"(qstep));                       // in a register: loaded again in every step it would be waited for with all LDS reads
    uint32_t poff[4], qoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3);
        const int col = (lane & 7) ^ ((row >> 1) & 7);
        poff[i] = (uint32_t)row * ppitch + 16u * col;
        constexpr int GPR = S::M / 8, RPI = 64 / GPR;          // granules of a k row, k rows per instruction
        const int k = RPI * (4 * wave + i) + lane / GPR;
        const int gran = (lane % GPR) ^ (4 * (k & 3) | 2 * ((k >> 2) & 1));
        qoff[i] = (uint32_t)k * qpitch + 16u * gran;
    }
    // the four instructions of a wavefront and slot one by one, so that they can stand between matrix instructions; the fourth moves
    // the operand on to its next stage, kt + 1
    auto move_on = [](v4i &buffer, const uint64_t step) {
        const uint64_t base = ((uint64_t)(uint32_t)buffer[1] << 32 | (uint32_t)buffer[0]) + step;
        buffer[0] = (int)(uint32_t)base;
        buffer[1] = (int)(uint32_t)(base >> 32);
    };
    auto dma_p = [&](const int kt, const uint32_t slot, const int i) {
        lds_dma16_buffer(pbuffer, poff[i], 0, lds0 + slot + wave * 4096 + i * 1024);
        if (i < 3) return;
        move_on(pbuffer, GD_K * 2);
        pbuffer[2] = kt + 1 < nk ? (int)pbytes : 0;
    };
    auto dma_q = [&](const int kt, const uint32_t slot, const int i) {
        lds_dma16_buffer(qbuffer, qoff[i], 0, lds0 + slot + wave * 4096 + i * 1024);
        if (i < 3) return;
        move_on(qbuffer, qstep);
        qbuffer[2] = kt + 2 < nk ? (int)qbytes : kt + 2 == nk ? (int)qbytes_last : 0;
    };
    // LDS read addresses: P: row * 128 + 16 * ((2u + c) ^ ((row >> 1) & 7)); (row >> 1) & 7 = (r >> 1) & 7 for every
    // tile of the wavefront, so one lane address per u, tiles are immediate offsets; the addresses move on with the slot.  Q: lane l of a
    // group of 16 supplies the address of row k0 + (l >> 2), columns 4 (l & 3) .. + 3 and gets four k of column l; two
    // reads (h = 0, 1) make the eight k of a fragment.
    uint32_t pa[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int slot = (2 * u + c) ^ ((r >> 1) & 7);
        pa[u] = lds0 + (wn * 32 * WP + r) * 128 + 16 * slot;
    }
    uint32_t qt[WQ][2];
    const int rr = (lane & 15) >> 2;
#pragma unroll
    for (int b = 0; b < WQ; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int gran = (wm * 32 * WQ + 32 * b) / 8 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
            qt[b][h] = lds0 + S::SLOT + (8 * c + 4 * h + rr) * QROW + 16 * (gran ^ (4 * rr | 2 * h)) + 8 * (lane & 1);
        }
    typedef __attribute__((address_space(3))) const v8bf *lds_v8bf;
    typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4bf *lds_v4bf;

    v16f acc[WP][WQ];
#pragma unroll
    for (int a = 0; a < WP; ++a)
#pragma unroll
        for (int b = 0; b < WQ; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    v8bf fp[2][WP], fq[2][WQ];
    constexpr int READS = WP + 2 * WQ;         // LDS reads of a quarter step
    auto read_one = [&](const int u, const int i) {
        const int set = u & 1;
        if (i < WP) {
            fp[set][i] = *(lds_v8bf)(uintptr_t)(pa[u] + i * 32 * 128);
        } else {
            const int b = (i - WP) >> 1, h = (i - WP) & 1;
            const v4bf v = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4bf)(uintptr_t)(qt[b][h] + 16 * u * QROW));
            if (h == 0) fq[set][b].lo = v; else fq[set][b].hi = v;
        }
    };
    // byte offset of the slot two further on in the ring
    auto advance = [](const uint32_t slot) { return slot < 3u * S::SLOT ? slot + 2u * S::SLOT : slot - 3u * S::SLOT; };
    // A quarter step: WP x WQ matrix instructions; side(s) is issued after instruction s.  The source order is the intended
    // issue order, a scheduling barrier after every matrix instruction keeps it.
    constexpr int SLOTS = WP * WQ;
    auto quarter = [&](const int u, auto &&side) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int a = s / WQ, b = s % WQ;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp[u & 1][a], fq[u & 1][b], acc[a][b], 0, 0, 0);
            side(s);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // operations [0, n) spread over the slots of a quarter step
    auto spread = [&](const int s, const int n, auto &&op) {
#pragma unroll
        for (int k = 0; k < n; ++k)
            if (k * SLOTS / n == s) op(k);
    };
    // The slots are a ring in the order P(0), Q(0), P(1), Q(1), ...  Step kt: quarters 0 to 2 read the fragments of the next
    // quarter under their matrix instructions; then stage kt + 1 must have landed and every wavefront holds the last fragments of
    // stage kt, so behind the barrier the last quarter reads the first fragments of stage kt + 1 and asks for Q(kt + 2) in the slot of
    // P(kt), and the first two quarters of the next step for P(kt + 3) in that of Q(kt): all of them in one quarter are more
    // than a multiprocessor's input path takes in.
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (j & 1) dma_q(j >> 1, j * S::SLOT, i);
            else dma_p(j >> 1, j * S::SLOT, i);
        }
    SBN_WAIT_VMCNT(8);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < READS; ++i) read_one(0, i);
    uint32_t sp = 0, sq = S::SLOT;
    for (int kt = 0; kt < nk; ++kt) {
        const uint32_t sp_next = advance(sp), sq_next = advance(sq);
        const uint32_t free = advance(sp_next);   // of Q(kt - 1)
#pragma unroll
        for (int u = 0; u < 3; ++u)
            quarter(u, [&](const int s) {
                spread(s, READS, [&](const int k) { read_one(u + 1, k); });
                if (u < 2) spread(s, 2, [&](const int k) { dma_p(kt + 2, free, 2 * u + k); });
            });
        SBN_WAIT_VMCNT(4);   // P(kt + 2) may fly
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) pa[u] += sp_next - sp;
#pragma unroll
        for (int b = 0; b < WQ; ++b) { qt[b][0] += sq_next - sq; qt[b][1] += sq_next - sq; }
        quarter(3, [&](const int s) {
            spread(s, READS, [&](const int k) { read_one(0, k); });
            spread(s, 4, [&](const int k) { dma_q(kt + 2, sp, k); });
        });
        sp = sp_next;
        sq = sq_next;
    }
    SBN_WAIT_VMCNT(0);   // the surplus stages have landed
    __syncthreads();
    bf16_wave_epilogue<WP, WQ>(g, acc, alpha, dlds + wave * S::STAGING, n0 + wn * 32 * WP, m0 + wm * 32 * WQ, lane);
}

// dX: P holds a byte per value, the high half of a bf16 (see write_code_tile): half the bytes of a stage to bring and to read, and a
// register of two values is one byte permutation, four for the eight of a fragment.  A matrix instruction executes in 61 to 75 % of
// the SIMD cycles of a training step's products, first stages, results and last rounds included, at the 1.6 GHz that the board's power
// holds; of that power the operands' way through the L2 and LDS is the part that can be saved.
// A slot of P lasts for two stages (rows of 128 bytes), of Q for one: two slots of P and three of Q.  P(j) serves the stages 2j and
// 2j + 1.  Half c of the lanes multiplies in quarter u the eight k at 32 (u / 2) + 16 c + 8 (u & 1), so that the bytes of two quarters
// are one read of 16.
template <bool BIG>
__device__ __forceinline__ void bf16_dx_body(const GemmBf16Args &g, uint8_t *dlds, int n0, int m0)
{
    using S = Bf16Tile<BIG>;
    constexpr int WP = S::WP, WQ = S::WQ;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;
    const int r = lane & 31, c = lane >> 5;
    const uint32_t lds0 = lds_address(dlds);
    const int nk = g.K / GD_K;
    // a scalar load: in front of everything that writes memory.  Twice that, for weights of +-0.5, unless it has no double
    const float gamma = g.alpha ? *g.alpha : 1.0f;
    const bool no_double = fabsf(gamma) >= 0x1p127f;
    const float alpha = no_double ? gamma : 2.0f * gamma;

    // DMA roles, four instructions per slot and wavefront: one fills 8 rows x 128 bytes (lane l: row l / 8, slot l % 8 holding global column
    // slot ^ ((row >> 1) & 7)).  Rows past the matrix and stages past the last read as zeros and fetch nothing.
    const int kleft = g.kq - (nk - 1) * GD_K;             // k of the last stage that Q has
    const int prows = g.N - n0 < S::N ? g.N - n0 : S::N, qrows = g.M - m0 < S::M ? g.M - m0 : S::M;
    const uint32_t ppitch = (uint32_t)g.ldp, qpitch = 2u * (uint32_t)g.ldq;
    const uint32_t pbytes = (uint32_t)prows * ppitch, qbytes = (uint32_t)qrows * qpitch;
    v4i pbuffer = buffer_of(static_cast<const uint8_t *>(g.P) + (int64_t)n0 * g.ldp, pbytes);
    v4i qbuffer = buffer_of(g.Q + (int64_t)m0 * g.ldq, qbytes);
    uint32_t at = 0, qat = 0;                             // bytes into a row of P and Q
    uint32_t poff[4], qoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 32 * wave + 8 * i + (lane >> 3), col = (lane & 7) ^ ((row >> 1) & 7);
        poff[i] = (uint32_t)row * ppitch + 16u * col;
        qoff[i] = (uint32_t)row * qpitch + 16u * col;
    }
    constexpr uint32_t QRING = 2 * S::SLOT;               // slots 0, 1: P; 2, 3, 4: Q
    // the instructions of a wavefront and slot one by one; the fourth moves the operand on
    auto dma_p = [&](const int slot, const int i) {
        lds_dma16_buffer(pbuffer, poff[i], at, lds0 + slot * S::SLOT + wave * 4096 + i * 1024);
        if (i < 3) return;
        at += 128;
        pbuffer[2] = at < ppitch ? (int)pbytes : 0;
    };
    auto dma_q = [&](const uint32_t ring, const int i) {
        lds_dma16_buffer(qbuffer, qoff[i], qat, lds0 + QRING + ring + wave * 4096 + i * 1024);
        if (i < 3) return;
        qat += 128;
        qbuffer[2] = qat < 128u * nk ? (int)qbytes : 0;
    };
    // k of the last stage past the end of a row of Q: what was fetched in their place is the next row, which may be infinite, and zeros
    // of P do not cancel that.
    // A lane overwrites what it asked for itself, behind its own wait and in front of the barrier that publishes the stage.
    auto zero_tail = [&](const uint32_t slot) {
        typedef __attribute__((address_space(3))) v4i *lds_v4i;
        asm volatile("" ::: "memory");   // not in front of the wait
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 8 * ((lane & 7) ^ (((32 * wave + 8 * i + (lane >> 3)) >> 1) & 7));
            if (k >= kleft) *(lds_v4i)(uintptr_t)(lds0 + slot + wave * 4096 + i * 1024 + 16 * lane) = v4i{0, 0, 0, 0};
        }
    };
    // LDS read addresses: row * 128 + 16 * (granule ^ ((row >> 1) & 7)); (row >> 1) & 7 = (r >> 1) & 7 for every tile of the wavefront, so
    // tiles are immediate offsets.  P: [stage parity][quarter / 2], Q: [quarter], moving on with the slots
    uint32_t pa[2][2], qa[4];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < 2; ++v) pa[e][v] = lds0 + (wn * 32 * WP + r) * 128 + 16 * ((4 * e + 2 * v + c) ^ ((r >> 1) & 7));
#pragma unroll
    for (int u = 0; u < 4; ++u) qa[u] = lds0 + QRING + (wm * 32 * WQ + r) * 128 + 16 * ((4 * (u >> 1) + 2 * c + (u & 1)) ^ ((r >> 1) & 7));
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v4u *lds_v4u;
    typedef __attribute__((address_space(3))) const v8bf *lds_v8bf;

    v16f acc[WP][WQ];
#pragma unroll
    for (int a = 0; a < WP; ++a)
#pragma unroll
        for (int b = 0; b < WQ; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    v4u raw[2][WP];                 // [quarter / 2][tile]: bytes of two quarters
    v8bf fp[2], fq[2][WQ];          // fragments of the tile at hand and of the next
    auto widen = [&](const int u, const int a) {   // eight bytes to bf16
        const uint32_t w0 = raw[u >> 1][a][2 * (u & 1)], w1 = raw[u >> 1][a][2 * (u & 1) + 1];
        return __builtin_bit_cast(v8bf, v4u{__builtin_amdgcn_perm(w0, w0, 0x010c000cu), __builtin_amdgcn_perm(w0, w0, 0x030c020cu),
                                            __builtin_amdgcn_perm(w1, w1, 0x010c000cu), __builtin_amdgcn_perm(w1, w1, 0x030c020cu)});
    };
    uint32_t pslot = 0, qring = 0;  // bytes to the slots of the stage at hand
    auto read_p = [&](const int e, const int v, const int a) { raw[v][a] = ((lds_v4u)(uintptr_t)pa[e][v])[a * 32 * 128 / 16]; };
    auto read_q = [&](const int u, const int b) { fq[u & 1][b] = ((lds_v8bf)(uintptr_t)qa[u])[b * 32 * 128 / 16]; };
    constexpr int SLOTS = WP * WQ;
    // A quarter step: WP x WQ matrix instructions; side(s) is issued after instruction s, and the next tile's bytes are widened there.
    auto quarter = [&](const int u, auto &&side) {
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            const int a = s / WQ, b = s % WQ;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fp[a & 1], fq[u & 1][b], acc[a][b], 0, 0, 0);
            side(s);
            // (of the next quarter's first tile behind this quarter's last instruction but one: its bytes have long been there, or
            // were read a quarter ago)
            if (b == 0 && a + 1 < WP) fp[(a + 1) & 1] = widen(u, a + 1);
            if (b == 0 && a + 1 == WP) fp[(a + 1) & 1] = widen((u + 1) & 3, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto spread = [&](const int s, const int n, auto &&op) {
#pragma unroll
        for (int k = 0; k < n; ++k)
            if (k * SLOTS / n == s) op(k);
    };
    static_assert(WP % 2 == 0, "a quarter ends on the set of fragments that the next begins with");
    // Step kt of parity e: quarters 0 to 2 read the fragments of the next quarter (P: of two quarters) under their matrix instructions;
    // then stage kt + 1 must have landed and every wavefront holds the last fragments of stage kt, so behind the barrier the last
    // quarter reads the first fragments of stage kt + 1.  The slot of Q(kt) takes Q(kt + 3), asked for in the last quarter and the
    // first of the next step; the slot of P(kt / 2), after an odd kt, P(kt / 2 + 2) in the next step's second and third.
    // Requests in flight at the wait behind Q(kt + 1): Q(kt + 2) and one P; behind the P that an even stage begins: Q(kt + 2).
    auto step = [&](const int kt, const int e) {
        quarter(0, [&](const int s) {
            spread(s, WQ, [&](const int k) { read_q(1, k); });
            spread(s, WP, [&](const int k) { read_p(e, 1, k); });
            spread(s, 2, [&](const int k) { dma_q(qring >= S::SLOT ? qring - S::SLOT : 2u * S::SLOT, 2 + k); });
        });
        quarter(1, [&](const int s) {
            spread(s, WQ, [&](const int k) { read_q(2, k); });
            if (e == 0) spread(s, 2, [&](const int k) { dma_p(pslot ? 0 : 1, k); });
        });
        quarter(2, [&](const int s) {
            spread(s, WQ, [&](const int k) { read_q(3, k); });
            if (e == 0) spread(s, 2, [&](const int k) { dma_p(pslot ? 0 : 1, 2 + k); });
        });
        if (e == 0) SBN_WAIT_VMCNT(8); else SBN_WAIT_VMCNT(4);
        const uint32_t left = qring;
        qring = qring < 2u * S::SLOT ? qring + S::SLOT : 0;
        if (kt == nk - 2 && kleft < GD_K) zero_tail(QRING + qring);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) qa[u] += qring - left;
        if (e == 1) {
            const uint32_t other = pslot ? 0u : (uint32_t)S::SLOT;
#pragma unroll
            for (int i = 0; i < 4; ++i) pa[i >> 1][i & 1] += other - pslot;
            pslot = other;
        }
        quarter(3, [&](const int s) {
            spread(s, WQ, [&](const int k) { read_q(0, k); });
            spread(s, WP, [&](const int k) { read_p(e ^ 1, 0, k); });
            spread(s, 2, [&](const int k) { dma_q(left, k); });
        });
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) dma_p(0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) dma_q(0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) dma_q(S::SLOT, i);
#pragma unroll
    for (int i = 0; i < 2; ++i) dma_q(2 * S::SLOT, i);
    SBN_WAIT_VMCNT(6);
    if (nk == 1 && kleft < GD_K) zero_tail(QRING);
    __syncthreads();
#pragma unroll
    for (int a = 0; a < WP; ++a) read_p(0, 0, a);
#pragma unroll
    for (int b = 0; b < WQ; ++b) read_q(0, b);
    fp[0] = widen(0, 0);
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
        step(kt, 0);
        step(kt + 1, 1);
    }
    if (kt < nk) step(kt, 0);
    SBN_WAIT_VMCNT(0);   // requests past the last stage deposit zeros
    __syncthreads();
    if (no_double) {
#pragma unroll
        for (int a = 0; a < WP; ++a)
#pragma unroll
            for (int b = 0; b < WQ; ++b) acc[a][b] *= 2.0f;
    }
    bf16_wave_epilogue<WP, WQ>(g, acc, alpha, dlds + wave * S::STAGING, n0 + wn * 32 * WP, m0 + wm * 32 * WQ, lane);
}

template <bool BIG>
__global__ void __launch_bounds__(64 * Bf16Tile<BIG>::WAVES) gemm_bf16_kernel(GemmBf16Group grp)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t dlds[];
    const int prob = bf16_product_of_block(grp);
    const GemmBf16Args &g = grp.g[prob];
    int tn, tm;
    if (!bf16_tile_of_block(g, (int)blockIdx.x - grp.block0[prob], tn, tm)) return;
    const int n0 = tn * Bf16Tile<BIG>::N, m0 = tm * Bf16Tile<BIG>::M;
    if (g.transposed) bf16_dw_body<BIG>(g, dlds, n0, m0);
    else bf16_dx_body<BIG>(g, dlds, n0, m0);
}

template <bool BIG>
sbn_status launch_gemm_bf16_as(int count, const GemmBf16Args *args, hipStream_t stream)
{
    using S = Bf16Tile<BIG>;
    for (int first = 0; first < count; first += GB_GROUP_MAX) {
        GemmBf16Group grp;
        grp.count = count - first < GB_GROUP_MAX ? count - first : GB_GROUP_MAX;
        int order[GB_GROUP_MAX];
        for (int i = 0; i < grp.count; ++i) order[i] = first + i;
        std::stable_sort(order, order + grp.count, [&](int a, int b) { return args[a].K > args[b].K; });
        int blocks = 0;
        for (int i = 0; i < grp.count; ++i) {
            grp.g[i] = args[order[i]];
            grp.g[i].tiles_n = (int)ceil_div(grp.g[i].N, S::N);
            grp.g[i].tiles_m = (int)ceil_div(grp.g[i].M, S::M);
            grp.block0[i] = blocks;
            blocks += (grp.g[i].tiles_n * grp.g[i].tiles_m + 7) / 8 * 8;   // eight equal shares, one per XCD
        }
        for (int i = grp.count; i <= GB_GROUP_MAX; ++i) grp.block0[i] = blocks;
        for (int i = grp.count; i < GB_GROUP_MAX; ++i) grp.g[i] = grp.g[0];
        static thread_local bool raised = false;
        if (!raised) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_bf16_kernel<BIG>), hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
            if (e != hipSuccess) { set_hip_error(e, "hipFuncSetAttribute"); return SBN_EHIP; }
            raised = true;
        }
        hipLaunchKernelGGL(gemm_bf16_kernel<BIG>, dim3(blocks), dim3(64 * S::WAVES), S::LDS, stream, grp);
        sbn_status st = check_launch("gemm_bf16_kernel");
        if (st != SBN_OK) return st;
    }
    return SBN_OK;
}

// Estimated time in us of the products of a call with the tiles of one size: every multiprocessor's share of all tiles, or the
// longest tile.  256 x 256 counts 1.45 us per stage of 64 k (1.2 while most multiprocessors idle) and 10 us for its first stages
// and its result; of 128 x 128 a multiprocessor holds two, 1.05 us per stage (0.6) and 7 us.  Both take less by now, the large
// tile 1.4 and 6, but in proportion: over 70 calls of 128 to 8192 tokens with both sizes measured the choice costs 0.38 % against
// the faster one of each (at worst 1.10, 2048 tokens 2560 -> 6912: 163 us against 148).
template <bool BIG>
float gemm_bf16_estimate_us(int count, const GemmBf16Args *args)
{
    using S = Bf16Tile<BIG>;
    const float step = BIG ? 1.45f : 1.05f, alone = BIG ? 1.2f : 0.6f, fixed = BIG ? 10.0f : 7.0f;
    float total = 0, longest = 0;
    for (int i = 0; i < count; ++i) {
        const float tiles = (float)(ceil_div(args[i].N, S::N) * ceil_div(args[i].M, S::M)), stages = (float)(args[i].K / GD_K);
        total += tiles * (stages * step + fixed);
        longest = std::max(longest, stages * alone + fixed);
    }
    return std::max(longest, total / (float)((BIG ? 1 : 2) * device_cus()));
}

// Large tiles move half the operand bytes per product; small ones share the device better where there are few (us per call,
// 6912 x 2560 at 1024 tokens 144 with large, 97 with small tiles; 1024 x 1024 at 512 tokens 35 / 18; 2560 x 2560 at 16384 tokens 390 / 450).
sbn_status launch_gemm_bf16(int count, const GemmBf16Args *args, hipStream_t stream)
{
    return gemm_bf16_estimate_us<true>(count, args) <= gemm_bf16_estimate_us<false>(count, args) ? launch_gemm_bf16_as<true>(count, args, stream)
                                                                                               : launch_gemm_bf16_as<false>(count, args, stream);
}

inline int64_t pad64(int64_t x) { return (x + 63) / 64 * 64; }

// The products read their operands through buffers whose size has 32 bits: a whole tile's rows of both operands of dX, the last row's stage
// behind the other rows of P of dW, and 63 rows of a stage of its Q.  Where the rows are so long that those of a large tile do not fit, the
// product is cut into products of `fit` rows (a multiple of `unit`), of which it does the first and more in turn.
constexpr int64_t OPERAND_END = (int64_t)1 << 32;
constexpr int64_t rows_fit(int64_t pitch) { return (OPERAND_END - 1) / pitch; }
constexpr int64_t rows_fit_moving(int64_t pitch) { return (OPERAND_END - 1 - GD_K * 2) / pitch + 1; }
template <class Each>
void cut_rows(int64_t rows, int64_t fit, int64_t unit, Each &&each)   // each(first, count)
{
    const int64_t most = fit >= Bf16Tile<true>::N ? rows : fit / unit * unit;
    for (int64_t first = 0; first < rows; first += most) each(first, std::min(most, rows - first));
}

}  // namespace

// Eight rows (the least that a product has columns) of x~^T and of W_eff^T, one of dY for dX, 63 for dW: some 306 million tokens and 34
// million outputs for dW, 536 million outputs for dX.
bool backward_takes(int64_t tokens, int64_t d_out, bool dx, bool dw)
{
    return (!dx || (rows_fit(ceil_div(d_out, 128) * 128) >= 8 && rows_fit(2 * d_out) >= 1)) &&
           (!dw || (rows_fit_moving(2 * pad64(tokens)) >= 8 && (GD_K - 1) * 2 * d_out + 2 * Bf16Tile<true>::M < OPERAND_END));
}

size_t backward_workspace_bytes(int64_t tokens, int64_t d_out, int64_t d_in)
{
    // W_eff^T [d_in, 2 pad64(d_out)] bytes (a byte per weight in rows of whole 128 lies in it) + int8 W_eff (generic patterns) + x~^T bf16 [d_in, pad64(tokens)]
    // + dY / s_x bf16 [tokens, d_out] + the mask bit plane of the gradient-masked variant
    return align_up((size_t)d_in * pad64(d_out) * 2, 256) + align_up((size_t)d_out * d_in, 256) +
           align_up((size_t)d_in * pad64(tokens) * 2, 256) + align_up((size_t)tokens * d_out * 2, 256) +
           align_up((size_t)d_out * ((d_in + 31) / 32) * 4, 256);
}

// Backward products of `count` layers in one pass: the operands of all layers in ONE launch, then ONE matrix-multiply
// launch (per GB_GROUP_MAX products) over all dW and dX tiles.  Layers that share their quantized input (Q/K/V,
// up/gate) share its transpose.
sbn_status launch_backward_grouped(int count, const BackwardItem *items, const Pattern &pat, int flags, hipStream_t stream)
{
    const int accumulate = (flags & SBN_BWD_ACCUMULATE) != 0;
    std::vector<GemmBf16Args> products;
    std::vector<const uint16_t *> xt_of(count, nullptr);
    products.reserve(2 * count);
    std::vector<OperandJob> jobs;
    jobs.reserve(3 * count);
    sbn_status st;
    for (int i = 0; i < count; ++i) {
        const BackwardItem &it = items[i];
        const int64_t tokens = it.tokens, d_in = it.d_in, d_out = it.d_out;
        uint8_t *ws = static_cast<uint8_t *>(it.workspace);
        uint8_t *wt = ws;   // a byte per weight in rows of whole 128, which the region for 2 bytes in rows of whole 64 holds
        ws += align_up((size_t)d_in * pad64(d_out) * 2, 256);
        int8_t *w8 = reinterpret_cast<int8_t *>(ws);
        ws += align_up((size_t)d_out * d_in, 256);
        uint16_t *xt = reinterpret_cast<uint16_t *>(ws);
        ws += align_up((size_t)d_in * pad64(tokens) * 2, 256);
        uint16_t *dys = reinterpret_cast<uint16_t *>(ws);
        ws += align_up((size_t)tokens * d_out * 2, 256);
        uint32_t *mask_bits = reinterpret_cast<uint32_t *>(ws);
        const uint16_t *dy = static_cast<const uint16_t *>(it.dY);

        if (it.dX) {
            const int64_t ldw = ceil_div(d_out, 128) * 128;
            if (has_unpack(pat)) {
                jobs.push_back({it.packed, nullptr, wt, ldw, (int)d_out, (int)d_in, (int)ceil_div(d_in, CHUNK), OPERAND_UNPACK});
            } else {
                st = launch_expand_groups(it.packed, d_out, d_in, pat, w8, stream);
                if (st != SBN_OK) return st;
                jobs.push_back({w8, nullptr, wt, ldw, (int)d_out, (int)d_in, (int)ceil_div(d_in, 128), OPERAND_CODES});
            }
            // dX[t, k] = gamma * sum_o dY[t, o] * W_eff^T[k, o]
            GemmBf16Args a{};
            a.P = wt; a.ldp = ldw; a.N = (int)d_in;
            a.Q = dy; a.ldq = d_out; a.M = (int)tokens; a.kq = (int)d_out;
            a.K = (int)pad64(d_out);
            a.C = static_cast<uint16_t *>(it.dX); a.ldc = d_in; a.alpha = it.gamma;
            cut_rows(tokens, rows_fit(2 * d_out), 1, [&](int64_t m0, int64_t m) {
                cut_rows(d_in, rows_fit(ldw), 8, [&](int64_t n0, int64_t n) {
                    GemmBf16Args part = a;
                    part.P = wt + n0 * ldw; part.N = (int)n;
                    part.Q = a.Q + m0 * d_out; part.M = (int)m;
                    part.C = a.C + m0 * d_in + n0;
                    products.push_back(part);
                });
            });
        }
        if (it.dW) {
            const int64_t ldt = pad64(tokens);
            const uint16_t *xts = nullptr;   // an earlier layer of the call already transposed the same activations
            for (int j = 0; j < i && !xts; ++j)
                if (xt_of[j] && items[j].xq == it.xq && items[j].tokens == tokens && items[j].d_in == d_in) xts = xt_of[j];
            if (!xts) {
                xts = xt;
                jobs.push_back({it.xq, nullptr, xt, ldt, (int)tokens, (int)d_in, (int)ceil_div(d_in, 128), OPERAND_TRANSPOSE});
            }
            xt_of[i] = xts;
            jobs.push_back({dy, it.sx, dys, 0, (int)tokens, (int)(d_out / 8), 0, OPERAND_SCALE});
            // dW[o, k] = sum_t (dY / s_x)[t, o] * x~[t, k]; x~^T is zero for t in [tokens, ldt)
            GemmBf16Args a{};
            a.P = xts; a.ldp = ldt; a.N = (int)d_in;
            a.Q = dys; a.ldq = d_out; a.M = (int)d_out; a.kq = (int)tokens; a.transposed = 1;
            a.K = (int)ldt;
            a.C = static_cast<uint16_t *>(it.dW); a.ldc = d_in; a.accumulate = accumulate;
            if (flags & SBN_BWD_MASK_DW) {
                // ablation variant: only the weights of the current mask receive the new gradient term
                st = launch_mask_bitplane(it.packed, d_out, d_in, pat, mask_bits, stream);
                if (st != SBN_OK) return st;
                a.mask = reinterpret_cast<const uint8_t *>(mask_bits);
                a.mask_pitch = (int)((d_in + 31) / 32 * 4);
            }
            cut_rows(d_in, rows_fit_moving(2 * ldt), 8, [&](int64_t n0, int64_t n) {
                GemmBf16Args part = a;
                part.P = xts + n0 * ldt; part.N = (int)n;
                part.C = a.C + n0;
                if (a.mask) part.mask = a.mask + n0 / 8;
                products.push_back(part);
            });
        }
    }
    st = launch_operands(jobs, pat, stream);
    if (st != SBN_OK) return st;
    // all products are independent of each other (dX reads W_eff^T and dY, dW reads x~^T and dY / s_x)
    return launch_gemm_bf16((int)products.size(), products.data(), stream);
}

sbn_status launch_backward(const void *dY, int64_t tokens, int64_t d_in, int64_t d_out, const Pattern &pat,
                           const void *packed, const float *gamma, const int8_t *xq, const float *sx, void *dX,
                           void *dW, int flags, void *workspace, size_t ws_bytes, hipStream_t stream)
{
    (void)ws_bytes;
    BackwardItem it{dY, tokens, d_in, d_out, packed, gamma, xq, sx, dX, dW, workspace};
    return launch_backward_grouped(1, &it, pat, flags, stream);
}

}  // namespace sbn
