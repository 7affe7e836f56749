// The scaled-integer variant (kernels_int.hip) for few tokens: two launches that are bound by memory latency, not by
// bytes (4096 x 4096: 8.4 MB of nibbles, 1.7 us at the copy rate), so each is built to be one chain of as few dependent
// memory round trips as the step allows.
//
//   int_few_prep_kernel   a workgroup per K slice and block of 32 tokens: row maxima over all of K (every workgroup finds
//                         them anew: a launch of its own would cost more than reading the few rows again), the slice's
//                         codes in operand order, and the slice's share of T = X_q A_k
//   int_few_kernel        a workgroup per 32 columns and block of 32 tokens, eight wavefronts that take the K groups in
//                         turn; their sums, the token scales and the correction - a rank block of 16 per wavefront -
//                         meet in LDS in wavefront order
//
// Five launches (quantizer, projection in planes and their sum, product in planes and their sum) before; 4096 x 4096 at
// 16 tokens 23.2 -> 13.4 us a call in a stream of them, 8192 x 28672 at 16 tokens 80 -> 49 us.  How far up these two are the
// faster ones: few_tokens in int_host.cpp.
#include "lqer_internal.h"
#include "mx_device.h"

namespace lqer {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kFewWaves = 8;

__device__ __forceinline__ i32x16 i8_products(const i32x4 (&x)[4], const i32x4 (&w)[4]) {
    i32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) s = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[q], w[q], s, 0, 0, 0);
    return s;
}

// Register r of a 32x32 result is row 8 (r / 4) + 4 (lane / 32) + r % 4.
__device__ __forceinline__ int result_row(int r, int hh) { return 8 * (r >> 2) + 4 * hh + (r & 3); }

// LDS: [slice groups][8 cells][32 rows][16 B] codes, then [8 wavefronts][16][64] fp32 partial sums of T
__global__ __launch_bounds__(64 * kFewWaves) void int_few_prep_kernel(IntFewArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ float smax[32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane & 31, hh = lane >> 5;
    const int64_t row0 = (int64_t)blockIdx.y * 32;
    const int rows = a.M - row0 < 32 ? (int)(a.M - row0) : 32;
    const int gb = blockIdx.x * a.slice_groups;
    const int count = a.G - gb < a.slice_groups ? (int)a.G - gb : a.slice_groups;
    float* red = reinterpret_cast<float*>(lds + a.slice_groups * 4096);

    // A_k's records of this wavefront's first group are asked for ahead of everything else
    i32x4 aw[4];
    float asc = 0.f;
    auto load_a = [&](int rg, int g) {
        const uint8_t* rec = a.At + ((int64_t)rg * a.G + gb + g) * 4096 + lane * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) aw[q] = *reinterpret_cast<const i32x4*>(rec + q * 1024);
        asc = a.Asc[((int64_t)rg * a.G + gb + g) * 32 + t];
    };
    if (a.kp32 > 0 && wave < count) load_a(0, wave);

    // row maxima: wavefront w takes rows w, w + 8, ..
    const int64_t n4 = a.G * 32;                     // float4 per row
    for (int r = wave; r < rows; r += kFewWaves) {
        const float* x = a.X + (row0 + r) * a.ldx;
        float m = 0.f;
        for (int64_t i0 = 0; i0 < n4; i0 += 512) {   // eight loads in flight
            f32x4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int64_t i = i0 + 64 * j + lane;
                v[j] = *reinterpret_cast<const f32x4*>(x + 4 * (i < n4 ? i : n4 - 1));
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[j][0]), __builtin_fabsf(v[j][1])),
                                                       __builtin_fmaxf(__builtin_fabsf(v[j][2]), __builtin_fabsf(v[j][3]))));
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, off));
        // s = fp16(amax / 127), the division in fp32 and correctly rounded; 1 for an all-zero row
        const _Float16 sh = (m == 0.f) ? (_Float16)1.0f : (_Float16)__fdiv_rn(m, 127.0f);
        if (lane == 0) {
            smax[r] = (float)sh;
            if (blockIdx.x == 0) a.Xs[row0 + r] = (float)sh;
        }
    }
    __syncthreads();

    // codes of the slice: an item is half a run of 32 elements of one row, half of two cells (its even elements, its odd ones);
    // whole runs left half of the threads idle behind the other half's 32 exact divisions:
    // 16 x 4096 x 4096 whole call 13.3 -> 12.6 us, 1 token 10.5 -> 9.7, 16 x 11008 x 4096 23.7 -> 22.6
    uint8_t* xc = a.Xc + (int64_t)blockIdx.y * a.K * 32;
    for (int item = tid; item < rows * count * 8; item += 64 * kFewWaves) {
        const int half = item & 1, run = (item >> 1) % (count * 4), r = (item >> 1) / (count * 4);
        const float* x = a.X + (row0 + r) * a.ldx + (int64_t)gb * 128 + run * 32 + half * 16;
        const float s = smax[r];
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const f32x4*>(x + 4 * j);
        u32x2 ev = u32x2{0, 0}, od = u32x2{0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float q = __builtin_rintf(__fdiv_rn(v[j][e], s));
                q = __builtin_fminf(__builtin_fmaxf(q, -127.0f), 127.0f);
                const uint32_t c = (uint32_t)(int)q & 0xFFu;
                const int k = 2 * j + (e >> 1);      // position among the half's even or odd elements
                if (e & 1) od[k >> 2] |= c << (8 * (k & 3));
                else ev[k >> 2] |= c << (8 * (k & 3));
            }
        *reinterpret_cast<u32x2*>(lds + (2 * run * 32 + r) * 16 + half * 8) = ev;
        *reinterpret_cast<u32x2*>(lds + ((2 * run + 1) * 32 + r) * 16 + half * 8) = od;
        uint8_t* dst = xc + (((int64_t)gb * 8 + 2 * run) << (a.lr + 4)) + r * 16 + half * 8;
        *reinterpret_cast<u32x2*>(dst) = ev;
        *reinterpret_cast<u32x2*>(dst + (16 << a.lr)) = od;
    }
    if (a.kp32 == 0) return;
    __syncthreads();

    // the slice's share of T: MFMA (sp, p) of a group uses cell 4 sp + 2 hh + p; rows past the last repeat it
    const int row = t < rows ? t : rows - 1;
    for (int rg = 0; rg < a.kp32; ++rg) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int g = wave; g < count; g += kFewWaves) {
            if (rg > 0 || g >= kFewWaves) load_a(rg, g);
            i32x4 x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                x[q] = *reinterpret_cast<const i32x4*>(lds + ((g * 8 + 4 * (q >> 1) + 2 * hh + (q & 1)) * 32 + row) * 16);
            const i32x16 s = i8_products(x, aw);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += (float)s[r] * asc;
        }
        if (rg > 0) __syncthreads();                 // the sums of the rank group before have been read
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {                // wavefront w finishes registers 2 w and 2 w + 1
            const int r = 2 * wave + i, orow = result_row(r, hh);
            float v = red[r * 64 + lane];
#pragma unroll
            for (int w = 1; w < kFewWaves; ++w) v += red[(w * 16 + r) * 64 + lane];
            if (orow < rows) a.T[((int64_t)blockIdx.x * a.M + row0 + orow) * a.kp32 * 32 + rg * 32 + t] = v * smax[orow];
        }
    }
}

// LDS: [8 wavefronts][2: product, correction][16][64] fp32
__global__ __launch_bounds__(64 * kFewWaves) void int_few_kernel(IntFewArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    float* red = reinterpret_cast<float*>(lds);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane & 31, hh = lane >> 5;
    const int64_t cg = blockIdx.x, row0 = (int64_t)blockIdx.y * 32;
    const int rows = a.M - row0 < 32 ? (int)(a.M - row0) : 32;
    const int row = t < rows ? t : rows - 1;         // rows past the last repeat it and are never stored
    const int G = (int)a.G;
    const uint8_t* wp = a.Wt + cg * a.G * 2048 + lane * 16;
    const float* sp = a.Wsc + cg * a.G * 32 + t;
    const uint8_t* xp = a.Xc + (int64_t)blockIdx.y * a.K * 32 + row * 16 + ((2 * hh) << (a.lr + 4));
    const int cell = 16 << a.lr;                     // bytes from one cell column to the next

    struct Set { u32x4 c[2]; i32x4 x[4]; float s; };
    auto load = [&](Set& d, int g) {
        d.c[0] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wp + (int64_t)g * 2048));
        d.c[1] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wp + (int64_t)g * 2048 + 1024));
        d.s = sp[(int64_t)g * 32];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            d.x[q] = *reinterpret_cast<const i32x4*>(xp + ((int64_t)g * 8 + 4 * (q >> 1) + (q & 1)) * cell);
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    auto use = [&](const Set& d) {
        i32x4 w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[q][e] = (int)(((q & 1) ? d.c[q >> 1][e] : d.c[q >> 1][e] << 4) & 0xF0F0F0F0u);
        const i32x16 s = i8_products(d.x, w);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += (float)s[r] * d.s;
    };
    // wavefront w takes groups w, w + 8, ..; four sets in flight
    Set s0, s1, s2, s3;
    const int last = G - 1;
    auto at = [&](int g) { return g < last ? g : last; };          // (clamped: loads stay unconditional)
    load(s0, at(wave));
    load(s1, at(wave + 8));
    load(s2, at(wave + 16));
    load(s3, at(wave + 24));
    // the correction's operands: rank block `wave` of B_k and of the S partial sums of T, added in slice order
    const bool tail = wave < a.kp16;
    u32x4 bw = u32x4{0, 0, 0, 0};
    f32x4 p0 = f32x4{0.f, 0.f, 0.f, 0.f}, p1 = p0;
    if (tail) {
        bw = *reinterpret_cast<const u32x4*>(a.Bt + (cg * a.kp16 + wave) * kBRecordBytes + t * 16);
        const int64_t ldt = (int64_t)a.kp32 * 32, stride = a.M * ldt;
        const float* src = a.T + (row0 + row) * ldt + wave * 16 + 8 * hh;
        for (int z0 = 0; z0 < a.S; z0 += 8) {
            f32x4 q0[8], q1[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int z = z0 + j < a.S ? z0 + j : a.S - 1;
                q0[j] = *reinterpret_cast<const f32x4*>(src + z * stride);
                q1[j] = *reinterpret_cast<const f32x4*>(src + z * stride + 4);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < a.S) { p0 += q0[j]; p1 += q1[j]; }
        }
    }
    for (int g = wave; g < G; g += 32) {
        use(s0);
        load(s0, at(g + 32));
        if (g + 8 < G) use(s1);
        load(s1, at(g + 40));
        if (g + 16 < G) use(s2);
        load(s2, at(g + 48));
        if (g + 24 < G) use(s3);
        load(s3, at(g + 56));
    }
    f32x16 ta;
#pragma unroll
    for (int r = 0; r < 16; ++r) ta[r] = 0.f;
    if (tail) {
        Frag hi, lo, f0, f1;
        int8x16_to_frags(bw, 1.0f, f0, f1);
        const Frag bf = hh ? f1 : f0;                // lane half hh takes ranks 8 hh .. + 7 of the block on both sides
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t h2[2], l2[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float v = e < 2 ? p0[(2 * e + j) & 3] : p1[(2 * e + j) & 3];
                const uint32_t hb = f32_bits(v) & 0xFFFF0000u;
                h2[j] = hb >> 16;
                l2[j] = f32_bits(v - f32_from_bits(hb)) >> 16;
            }
            hi.u[e] = h2[0] | (h2[1] << 16);
            lo.u[e] = l2[0] | (l2[1] << 16);
        }
        ta = mfma32(hi.v, bf.v, ta);
        ta = mfma32(lo.v, bf.v, ta);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        red[((wave * 2) * 16 + r) * 64 + lane] = acc[r];
        if (tail) red[((wave * 2 + 1) * 16 + r) * 64 + lane] = ta[r];
    }
    __syncthreads();
    const int64_t n = cg * 32 + t;
    const float sb = a.kp16 > 0 ? a.Bsc[n] : 0.f;
    const int nt = a.kp16 < kFewWaves ? a.kp16 : kFewWaves;
#pragma unroll
    for (int i = 0; i < 2; ++i) {                    // wavefront w finishes registers 2 w and 2 w + 1
        const int r = 2 * wave + i, orow = result_row(r, hh);
        float v = red[r * 64 + lane];
#pragma unroll
        for (int w = 1; w < kFewWaves; ++w) v += red[((w * 2) * 16 + r) * 64 + lane];
        float c = 0.f;
        for (int w = 0; w < nt; ++w) c += red[((w * 2 + 1) * 16 + r) * 64 + lane];
        if (orow < rows && n < a.N) a.Y[(row0 + orow) * a.ldy + n] = v * a.Xs[row0 + orow] + c * sb;
    }
}

hipError_t launch_int_few(const IntFewArgs& a, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.M + 31) / 32);
    const size_t prep_lds = (size_t)a.slice_groups * 4096 + kFewWaves * 4096;
    hipLaunchKernelGGL(int_few_prep_kernel, dim3((unsigned)a.S, blocks), dim3(64 * kFewWaves), prep_lds, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(int_few_kernel, dim3((unsigned)a.N32, blocks), dim3(64 * kFewWaves), (size_t)kFewWaves * 8192, s, a);
    return hipGetLastError();
}

}  // namespace lqer
