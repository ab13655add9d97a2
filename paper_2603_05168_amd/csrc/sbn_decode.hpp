// Pieces shared by the kernels that quantize activations and by the decode kernels: the quantizer's arithmetic on bf16 vectors,
// and one super-step (512 weights) of the product on the 16-row matrix instructions.
#pragma once
#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

// ---- pieces of the activation quantizer shared by its kernels -------------------------------------
// largest 15-bit magnitude pattern among eight bf16 values and a running maximum (bf16 magnitudes order like integers);
// the two halves of a word are compared as a pair of 16-bit integers
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t absmax_bits_bf16x8(const uint4 &d, uint32_t m)
{
    const uint32_t w[4] = {d.x, d.y, d.z, d.w};
    ushort2_t best = {0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t mag = w[k] & 0x7fff7fffu;
        best = __builtin_elementwise_max(best, __builtin_bit_cast(ushort2_t, mag));
    }
    const uint32_t both = __builtin_bit_cast(uint32_t, best), lo = both & 0xffffu, hi = both >> 16;
    m = lo > m ? lo : m;
    m = hi > m ? hi : m;
    return m;
}

// s_x from the largest magnitude pattern: 127 / max(amax, 1e-5), one IEEE division
__device__ __forceinline__ float scale_from_absmax_bits(uint32_t m)
{
    float amax = __uint_as_float(m << 16);
    amax = amax < 1e-5f ? 1e-5f : amax;
    return __fdiv_rn(127.0f, amax);
}

// eight bf16 values of a row -> eight int8: clip(rint(x * s)) with one fp32 multiply and half-to-even rounding, s the
// scale of that same row.  The rounding is an addition of 1.5 * 2^23: the sum has an ulp of 1, so the (round-to-nearest-
// even) addition rounds the product exactly as rint does, and the low byte of the sum's bit pattern is the integer in
// two's complement.  No clip is needed: |x| <= amax <= max(amax, 1e-5) and s = fl(127 / max(amax, 1e-5)), so
// |fl(x * s)| <= 127 (1 + 2^-24)^2 < 127.5 and the rounded value already lies in [-127, 127].
__device__ __forceinline__ uint2 quantize_bf16x8(const uint4 &d, float s)
{
    // The addition writes the low byte of its result straight into byte i of the packed word (SDWA destination select), so the
    // four bytes of a word are put together by the additions themselves.
    const uint32_t w[4] = {d.x, d.y, d.z, d.w};
    const float magic = 12582912.0f;
    uint32_t packed[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float p0 = __fmul_rn(__uint_as_float(w[2 * h] << 16), s), p1 = __fmul_rn(__uint_as_float(w[2 * h] & 0xffff0000u), s);
        const float p2 = __fmul_rn(__uint_as_float(w[2 * h + 1] << 16), s), p3 = __fmul_rn(__uint_as_float(w[2 * h + 1] & 0xffff0000u), s);
        uint32_t z;
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_0 dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:DWORD" : "=v"(z) : "v"(p0), "v"(magic));
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_1 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(z) : "v"(p1), "v"(magic));
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_2 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(z) : "v"(p2), "v"(magic));
        asm("v_add_f32_sdwa %0, %1, %2 dst_sel:BYTE_3 dst_unused:UNUSED_PRESERVE src0_sel:DWORD src1_sel:DWORD" : "+v"(z) : "v"(p3), "v"(magic));
        packed[h] = z;
    }
    return make_uint2(packed[0], packed[1]);
}

__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a), __builtin_bit_cast(ushort2_t, b)));
}
// largest magnitude patterns of the even and of the odd ones of eight bf16 values
__device__ __forceinline__ uint32_t absmax_pair_bf16x8(const uint4 &d)
{
    return max_u16x2(max_u16x2(d.x & 0x7fff7fffu, d.y & 0x7fff7fffu), max_u16x2(d.z & 0x7fff7fffu, d.w & 0x7fff7fffu));
}

// ---- a super-step of the decode kernels: --------------------------------------------------
// for a super-step a lane (row r = lane % 16, quarter c4 = lane / 16) holds the 32-byte chunk c4 of its row.
// One super-step of one wavefront and row tile: idx4 / code4 = the lane's chunk, bfrag(j, x) = the lane's token operand.
// FORM = GEMV_DENSE: weights stored as dense 2-bit codes (the packed form of N = M, and what other patterns are
// rewritten to for decode): a chunk is eight code words, every word is the A operand of one v_mfma_i32_16x16x64_i8
// (lane quarter c holds k = 16c .. 16c+15 of the instruction on both operands).  FORM = GEMV_1OF4 reads the 1:4 packed
// form as stored (16-byte chunks, one load per lane and super-step) and builds the sparse instruction's operands in
// registers (expand_1of4): half the weight bytes for three times the vector work.
// x0 = the lane's token row at the super-step's first value; inside(k) = k, or an offset inside the row where k lies past
// it (zero codes meet what is read there).  The operand loads stand in front, unconditional, so that all are in flight together;
// HALVES: in two batches, from LDS, where the registers of one are short.
template <int FORM, int RT, bool HALVES = false, class Inside>
__device__ __forceinline__ void gemv_super_step(const uint4 (&idx4)[RT], const uint4 (&code4)[RT], const int8_t *x0, const int c4,
                                                const uint32_t ones, Inside &&inside, v4i (&acc)[RT])
{
    uint4 x[8];
    const auto load = [&](int j) {
        x[j] = *reinterpret_cast<const uint4 *>(x0 + inside(FORM == GEMV_DENSE ? 128 * c4 + 16 * j : 128 * (c4 >> 1) + 16 * (c4 & 1) + 32 * (j >> 1) + 256 * (j & 1)));
    };
    const auto second_half = [&]() {
        if constexpr (HALVES) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 4; j < 8; ++j) load(j);
        }
    };
#pragma unroll
    for (int j = 0; j < (HALVES ? 4 : 8); ++j) load(j);
    if constexpr (FORM == GEMV_DENSE) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j == 4) second_half();
            const v4i b = __builtin_bit_cast(v4i, x[j]);
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                const uint4 &h = j < 4 ? idx4[a] : code4[a];
                const uint32_t w = (j & 3) == 0 ? h.x : (j & 3) == 1 ? h.y : (j & 3) == 2 ? h.z : h.w;
                acc[a] = __builtin_amdgcn_mfma_i32_16x16x64_i8(expand_codes(w, ones), b, acc[a], 0, 0, 0);
            }
        }
    } else {
        uint32_t iw1[RT][2][2];
        v4i a1[RT][2][2];
        if constexpr (FORM == GEMV_1OF4) {   // the chunk is two index words and two code words
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                expand_1of4(idx4[a].x, idx4[a].z, ones, iw1[a][0], a1[a][0]);
                expand_1of4(idx4[a].y, idx4[a].w, ones, iw1[a][1], a1[a][1]);
            }
        }
        // B operand: elements 0..15 pair with the A lanes of quarters 0/1, elements 16..31 with
        // quarters 2/3 (measured operand layout of the instruction)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j == 2) second_half();
            const uint4 &blo = x[2 * j], &bhi = x[2 * j + 1];
            const v8i b = {(int)blo.x, (int)blo.y, (int)blo.z, (int)blo.w, (int)bhi.x, (int)bhi.y, (int)bhi.z, (int)bhi.w};
#pragma unroll
            for (int a = 0; a < RT; ++a) {
                if constexpr (FORM == GEMV_1OF4) {
                    acc[a] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(a1[a][j >> 1][j & 1], b, acc[a], (int)iw1[a][j >> 1][j & 1], 0, 0);
                } else {
                    const uint32_t cw = j == 0 ? code4[a].x : j == 1 ? code4[a].y : j == 2 ? code4[a].z : code4[a].w;
                    const uint32_t iw = j == 0 ? idx4[a].x : j == 1 ? idx4[a].y : j == 2 ? idx4[a].z : idx4[a].w;
                    acc[a] = __builtin_amdgcn_smfmac_i32_16x16x128_i8(expand_codes(cw, ones), b, acc[a], (int)iw, 0, 0);
                }
            }
        }
    }
}

}  // namespace sbn
