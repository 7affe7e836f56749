// Device helpers for gfx950: MXINT block arithmetic on 64-wide wavefronts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lqer {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// an 8-byte load from a 4-byte aligned address (exponent words of the compact weight records)
typedef u32x2 u32x2_a4 __attribute__((aligned(4)));

union Frag {            // one bf16 MFMA operand (16x16x32 or 32x32x16): 8 bf16 per lane
    bf16x8 v;
    u32x4 u;
    bf16x2 h[4];
};

__device__ __forceinline__ float f32_from_bits(uint32_t b) { return __builtin_bit_cast(float, b); }
__device__ __forceinline__ uint32_t f32_bits(float f) { return __builtin_bit_cast(uint32_t, f); }

// fp32 scale 2^(eb - 127 - 2 + 9) for a W block with exponent byte eb: the +9 undoes the 2^-9 of
// the fp8 subnormal encoding, the -2 is the MXINT4 fraction.  eb <= 247 is checked at import.
__device__ __forceinline__ float w_scale(uint32_t eb) { return f32_from_bits((eb + 7u) << 23); }

// 8 sign-magnitude 4-bit codes (layout in lqer_internal.h) -> 8 bf16 values code * 2^(e-2).
__device__ __forceinline__ bf16x8 unpack_w8(uint32_t w, float scale) {
    const uint32_t r0 = w & 0x87878787u;
    const uint32_t r1 = __builtin_amdgcn_alignbit(w, w, 4) & 0x87878787u;
    Frag f;
    f.h[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r0, scale, false);
    f.h[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r0, scale, true);
    f.h[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r1, scale, false);
    f.h[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r1, scale, true);
    return f.v;
}

// 2-bit weights: fp32 scale 2^(eb - 127 + 9) for a block with exponent byte eb (no fraction bits; the +9 undoes the
// 2^-9 of the fp8 subnormal encoding).  eb <= 245 is checked at import.
__device__ __forceinline__ float w2_scale(uint32_t eb) { return f32_from_bits((eb + 9u) << 23); }

// Eight of the 16 sign-and-magnitude 2-bit codes of a block word (layout in lqer_internal.h) -> 8 bf16 values
// code * 2^e: elements 8 half .. 8 half + 7.
__device__ __forceinline__ bf16x8 unpack_w8_b2(uint32_t w, int half, float scale) {
    const uint32_t r0 = (half ? __builtin_amdgcn_alignbit(w, w, 4) : w) & 0x81818181u;
    const uint32_t r1 = __builtin_amdgcn_alignbit(w, w, half ? 6 : 2) & 0x81818181u;
    Frag f;
    f.h[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r0, scale, false);
    f.h[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r0, scale, true);
    f.h[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r1, scale, false);
    f.h[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r1, scale, true);
    return f.v;
}

// Two fp32 values that are exactly representable in bf16 -> packed pair (a low, b high).
__device__ __forceinline__ uint32_t pack_bf16_exact(float a, float b) {
    return __builtin_amdgcn_perm(f32_bits(b), f32_bits(a), 0x07060302u);
}

// 4 int8 codes in a word, times an exact power-of-two scale -> 4 bf16 (exact), as two packed pairs.
__device__ __forceinline__ u32x2 int8x4_to_bf16(uint32_t w, float scale) {
    const float f0 = (float)(int)(int8_t)(w & 0xFF) * scale;
    const float f1 = (float)(int)(int8_t)((w >> 8) & 0xFF) * scale;
    const float f2 = (float)(int)(int8_t)((w >> 16) & 0xFF) * scale;
    const float f3 = (float)(int)(int8_t)(w >> 24) * scale;
    return u32x2{pack_bf16_exact(f0, f1), pack_bf16_exact(f2, f3)};
}

// One MXINT8 block (16 int8 codes) -> the two MFMA operands of its two K steps.
__device__ __forceinline__ void int8x16_to_frags(u32x4 cw, float scale, Frag& f0, Frag& f1) {
    const u32x2 a = int8x4_to_bf16(cw[0], scale), b = int8x4_to_bf16(cw[1], scale);
    const u32x2 c = int8x4_to_bf16(cw[2], scale), d = int8x4_to_bf16(cw[3], scale);
    f0.u = u32x4{a[0], a[1], b[0], b[1]};
    f1.u = u32x4{c[0], c[1], d[0], d[1]};
}

// fp32 scale 2^(eb - 127 - 6) of an MXINT8 block.  Below the normal range (eb < 7) the value is
// produced by a second exact multiply.
__device__ __forceinline__ float h_scale(uint32_t eb) {
    return (eb >= 7u) ? f32_from_bits((eb - 6u) << 23)
                      : f32_from_bits((eb + 18u) << 23) * 0x1p-24f;
}

// fp32 scale 2^(eb - 127 - frac) of an MXINT block with `frac` fraction bits (6 for 8-bit codes, 4 for 6-bit).
__device__ __forceinline__ float x_scale(uint32_t eb, int frac) {
    return (eb > (uint32_t)frac) ? f32_from_bits((eb - frac) << 23)
                                 : f32_from_bits((eb + 24u - frac) << 23) * 0x1p-24f;
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// D[i][j] += sum_k A[i][k] B[k][j], 32 x 32 x 16.  Lane (l % 32, l / 32) supplies A[l % 32][8 (l/32) ..+7]
// and B[8 (l/32) ..+7][l % 32]; accumulator register r of lane l is D[8 (r/4) + 4 (l/32) + r % 4][l % 32].
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// ---- both operands as fp6 -------------------------------------------------------------------------------------------------
// The block-scaled MFMA on fp6 operands (E2M3: integers 0 to 16 in units of 1/8 carry their own value as code, above that the
// even ones to 32 and the multiples of 4 to 60) runs at four times bf16's rate.  An MXINT8 code x = 16 h + l (h and l with x's
// sign, |h| <= 7, |l| <= 15) against an MXINT4 code w is (8 h) (2 w) + l w: two fp6 products, all four factors exact, and
// a block of 16 of both operands is one scaled block of 32 - the instruction's own size - [8 h | l] against [2 w | w].  The
// scales are the blocks' exponent bytes.  Half of four times bf16's rate is left: a loop of these MFMAs on random operands
// delivers 5170 to 5580 TFLOP/s of fp6 products (2600 to 2800 of the product's own), bf16's 1610 to 1850.
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// D[i][j] += 2^(sa + sb - 254) sum_k A[i][k] B[k][j], 32 x 32 x 64: lane (l % 32, l / 32) supplies the 32 elements k = 32 (l / 32) .. of
// its row of A and column of B, element i at bit 6 i, and their scales as byte BYTE of a word each; D as of mfma32.
template <int BYTE>
__device__ __forceinline__ f32x16 mfma32_six(u32x6 a, u32x6 b, f32x16 c, uint32_t sa, uint32_t sb) {
    const i32x8 av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)a[4], (int)a[5], 0, 0};
    const i32x8 bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], (int)b[4], (int)b[5], 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 2, 2, BYTE, (int)sa, BYTE, (int)sb);
}

// The same with fp4 (E2M1) as the first operand: element i at bit 4 i.
template <int BA, int BB>
__device__ __forceinline__ f32x16 mfma32_four(u32x4 a, u32x6 b, f32x16 c, uint32_t sa, uint32_t sb) {
    const i32x8 av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
    const i32x8 bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], (int)b[4], (int)b[5], 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, c, 4, 2, BA, (int)sa, BB, (int)sb);
}

// Where element e of a block lies among an operand's 16 fields of each half: 0, 8, 1, 9 .. 3, 11, 4, 12 .., the order in which
// expand_four finds 2-bit codes.
constexpr int six_field(int e) { return (e & 3) * 2 + ((e >> 3) & 1) + ((e >> 2) & 1) * 8; }

// The 2-bit codes of a block (layout in lqer_internal.h) -> the operand [w | w / 2] in fp4, where 1 is code 2 and 1/2 code 1.  Against
// [8 h | l], whose values are h and l / 8, the sum is x w / 16; with 4 bits it is x w / 64 for weights w / 4, so both take the block's
// exponent byte less 2 as the weights' scale.  Nine instructions for 16 codes, from the records the other kernels read.
__device__ __forceinline__ u32x4 expand_four(uint32_t p) {
    const uint32_t r = (p & 0x55555555u) | (__builtin_amdgcn_alignbit(p, p, 4) & 0xAAAAAAAAu);     // signs three above magnitudes
    const uint32_t l0 = r & 0x99999999u, l1 = __builtin_amdgcn_alignbit(r, r, 2) & 0x99999999u;
    return u32x4{l0 + (l0 & 0x11111111u), l1 + (l1 & 0x11111111u), l0, l1};
}

// Bit g of three words, g mod 6 in the set given by `six` (bits 0 to 5), as the mask of word j.
constexpr uint32_t six_mask(uint32_t six, int j) {
    uint32_t m = 0;
    for (int p = 0; p < 32; ++p)
        if ((six >> ((32 * j + p) % 6)) & 1u) m |= 1u << p;
    return m;
}

// A lane's two blocks of one chunk (layout in lqer_internal.h) -> the operand [2 w | w] of its block S.
template <int S>
__device__ __forceinline__ u32x6 expand_six(u32x4 c) {
    const uint32_t sg = S == 0 ? c[3] : c[3] << 1;
    u32x6 r;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const uint32_t sign = sg & six_mask(0x20, j);
        const uint32_t lo = j > 0 ? c[j - 1] : 0u, hi = j < 2 ? c[j + 1] : 0u;      // neighbours in the run of 96 bits
        const uint32_t one = S == 0 ? c[j] : __builtin_amdgcn_alignbit(hi, c[j], 3);
        const uint32_t two = S == 0 ? __builtin_amdgcn_alignbit(c[j], lo, 31) : __builtin_amdgcn_alignbit(hi, c[j], 2);
        r[j] = (two & six_mask(0x0E, j)) | sign;
        r[3 + j] = (one & six_mask(0x07, j)) | sign;
    }
    return r;
}

// 16 codes of a block (as floats, times `up` at most 128 in size) -> the operand [8 h | l], its fields as six_field orders them.  (|h| <= 7 also
// for a code of -128, whose l is then -16.)  The conversion takes its 32 values alternately from two registers' runs.
template <bool CLAMP>
__device__ __forceinline__ u32x6 codes_to_six(const float (&r)[16], float up) {
    const float per16 = 0.0625f * up, per8 = 0.125f * up;
    f32x16 even, odd;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        float h = __builtin_truncf(r[i] * per16);
        if (CLAMP) h = __builtin_fmaxf(h, -7.0f);
        const float l = __builtin_fmaf(h, -2.0f, r[i] * per8);
        const int f = six_field(i);
        if (f & 1) { odd[f >> 1] = h; odd[8 + (f >> 1)] = l; }
        else { even[f >> 1] = h; even[8 + (f >> 1)] = l; }
    }
    return __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(even, odd, 1.0f);
}

// Back: the codes times `scale` (a power of two).
__device__ __forceinline__ void six_to_values(u32x6 v, float scale, float (&r)[16]) {
    typedef float f32x32 __attribute__((ext_vector_type(32)));
    const f32x32 e = __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(v, 1.0f);
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = __builtin_fmaf(e[six_field(i)], 16.0f, e[16 + six_field(i)] * 8.0f) * scale;
}

// Eight values of one MXINT8 block held by this lane (the other eight sit in lane ^ 32): the block's
// exponent byte from the maximum over both lanes, and this lane's codes as two words of four bytes.
__device__ __forceinline__ uint32_t requant_half_block(const float (&v)[8], uint32_t& w0, uint32_t& w1) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(v[i]));
    m = __builtin_fmaxf(m, __shfl_xor(m, 32));
    const uint32_t eb = (f32_bits(m) >> 23) & 0xFFu;
    const int e = (int)eb - 127;
    uint32_t w[2] = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float r = __builtin_rintf(__builtin_amdgcn_ldexpf(v[i], 6 - e));
        r = __builtin_fminf(__builtin_fmaxf(r, -127.0f), 127.0f);
        w[i >> 2] |= ((uint32_t)(int)r & 0xFFu) << (8 * (i & 3));
    }
    w0 = w[0];
    w1 = w[1];
    return eb;
}

// MXINT8 quantization of one value given the block's exponent byte: code = sat(rne(v * 2^(6-e))).
__device__ __forceinline__ int mx8_code(float v, int e_unbiased) {
    float r = __builtin_rintf(__builtin_amdgcn_ldexpf(v, 6 - e_unbiased));
    r = __builtin_fminf(__builtin_fmaxf(r, -127.0f), 127.0f);
    return (int)r;
}

// ---- per-token INT8 codes ---------------------------------------------------------------------------------------------
// rint(x / s) in [-127, 127], the quotient rounded to fp32 as a division rounds it, in three instructions instead of ten
// (P. Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor", 1990): with y = 1 / s correctly
// rounded and q = x y, the remainder r = x - q s is exact in one fused multiply-add, and q + r y is within 2^-47 of the quotient
// before it is rounded.  s is an fp16 value of 11 significant bits, so no quotient lies within 2^-36 of the middle between two
// fp32 values: the rounding is the division's.  (Where x y underflows the code is 0 either way.)  Scales that are zero or
// infinite - row maxima below 127 2^-25 or from 127 65520 on - keep the division.
struct Int8Coder {
    float s, y;
    __device__ __forceinline__ explicit Int8Coder(float scale) : s(scale), y(__fdiv_rn(1.0f, scale)) {}
    __device__ __forceinline__ Int8Coder(float scale, float inverse) : s(scale), y(inverse) {}   // inverse: 1 / scale, correctly rounded
    static __device__ __forceinline__ uint32_t clamp(float q) {
        q = __builtin_rintf(q);
        return (uint32_t)(int)__builtin_fminf(__builtin_fmaxf(q, -127.0f), 127.0f) & 0xFFu;
    }
    template <int N>
    __device__ __forceinline__ void codes(const f32x4 (&x)[N], uint32_t (&c)[N][4]) const {
        if (__builtin_expect(!(s > 0.f && s < __builtin_inff()), 0)) {
            asm volatile("");                        // (a branch: left alone, the divisions are done everywhere and one of two results taken)
#pragma unroll
            for (int i = 0; i < 4 * N; ++i) c[i >> 2][i & 3] = clamp(__fdiv_rn(x[i >> 2][i & 3], s));
            return;
        }
#pragma unroll
        for (int i = 0; i < 4 * N; ++i) {
            const float v = x[i >> 2][i & 3], q = v * y;
            c[i >> 2][i & 3] = clamp(__builtin_fmaf(__builtin_fmaf(-q, s, v), y, q));
        }
    }
};

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// the maximum over the wavefront, in every lane: within 16 lanes by lane permutations of the instruction itself, then the four
__device__ __forceinline__ float wave_max(float m) {
    m = __builtin_fmaxf(m, dpp_move<0xB1>(m));       // quad_perm [1,0,3,2]
    m = __builtin_fmaxf(m, dpp_move<0x4E>(m));       // quad_perm [2,3,0,1]
    m = __builtin_fmaxf(m, dpp_move<0x141>(m));      // row_half_mirror
    m = __builtin_fmaxf(m, dpp_move<0x140>(m));      // row_mirror
    float r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = f32_from_bits((uint32_t)__builtin_amdgcn_readlane((int)f32_bits(m), 16 * i));
    return __builtin_fmaxf(__builtin_fmaxf(r[0], r[1]), __builtin_fmaxf(r[2], r[3]));
}

// ---- buffer loads -----------------------------------------------------------------------------------------------------
// A load whose offset lies past the buffer's end accesses no memory and returns zeros.
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
constexpr int kNoOffset = (int)0x80000000;           // or-ed to an offset: past the end of any buffer of at most 2 GiB
__device__ __forceinline__ BufferRsrc buffer_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 buffer_load16(BufferRsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }
__device__ __forceinline__ u32x4 buffer_load16_nt(BufferRsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 2); }
__device__ __forceinline__ u32x2 buffer_load8(BufferRsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0); }
__device__ __forceinline__ uint32_t buffer_load4(BufferRsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }
__device__ __forceinline__ uint32_t buffer_load1(BufferRsrc r, int off) { return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0); }

// ---- direct-to-LDS loads ----------------------------------------------------------------------------------------------
// 1 KiB (64 lanes x 16 bytes) or 256 B from `base` + this lane's byte offset to LDS address at + ADD + 16 (4) * lane.
// Written as asm because the compiler answers its own builtin with a full drain of the loads in flight in front of every
// LDS read; nothing is returned in registers, and the kernel counts these loads itself (staged_wait).  M0 has no other use.
template <int ADD>
__device__ __forceinline__ void lds_dma16(uint32_t at, uint32_t off, const uint8_t* base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(at), "v"(off), "s"(base), "n"(ADD) : "memory", "scc");
}
template <int ADD>
__device__ __forceinline__ void lds_dma4(uint32_t at, uint32_t off, const uint8_t* base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(at), "v"(off), "s"(base), "n"(ADD) : "memory", "scc");
}
// All but this wavefront's newest LEFT loads have landed, all but its newest READS reads of LDS have returned, and so have everybody's.
template <int LEFT, int READS = 0>
__device__ __forceinline__ void staged_wait() {
    static_assert(LEFT >= 0 && LEFT < 64 && READS >= 0 && READS < 16, "a 6-bit and a 4-bit counter");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" ::"n"(LEFT), "n"(READS) : "memory");
}

}  // namespace lqer
