// The scaled-integer variant (kernels_int.hip) for few tokens: two launches that are bound by memory latency, not by
// bytes (4096 x 4096: 8.4 MB of nibbles, 1.7 us at the copy rate), so each is built to be one chain of as few dependent
// memory round trips as the step allows.
//
//   int_few_prep_kernel   a workgroup per K slice and block of 32 tokens: row maxima over all of K (every workgroup finds
//                         them anew: a launch of its own would cost more than reading the few rows again), the slice's
//                         codes in operand order, and the slice's share of T = X_q A_k.  The rows, the values to quantize and
//                         A_k are all asked for at the start
//   int_few_kernel        a workgroup per 32 columns and block of 32 tokens, eight wavefronts that take the K groups in
//                         turn; their sums, the token scales and the correction - a rank block of 16 per wavefront -
//                         meet in LDS in wavefront order
//
// Five launches (quantizer, projection in planes and their sum, product in planes and their sum) before; 8192 x 28672 at 16
// tokens 80 -> 49 us.  What is kept off the chain: divisions (Int8Coder - sixteen of a thread's, done by every wavefront, were
// most of the first launch), rows read one after the other, waits for T ahead of the product, reads of scales behind it.  Whole
// calls replayed from a graph, rank 32, with and without those: 4096 x 4096 at 1 token 10.7 -> 9.5 us, at 16 14.6 -> 13.0, at 32
// 20.2 -> 18.3, 1024 x 1024 at 4 9.8 -> 8.1, 4096 x 11008 at 16 21.3 -> 18.6.  How far up these two are the faster ones:
// few_tokens in int_host.cpp.
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

// LDS: [slice groups][8 cells][32 rows][16 B] codes, then [slice groups][16][64] fp32 sums of T, one per wavefront with a group
// NW wavefronts: 8 for up to 8 tokens, a row and up to 16 of its loads each, and 16 beyond.
constexpr int kFewSliceGroups = 7;
template <int NW>
__global__ __launch_bounds__(64 * NW) void int_few_prep_kernel(IntFewArgs a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ float smax[32], pmax[NW][32];
    static_assert(kFewSliceGroups <= NW && (NW == 8 || NW == 16), "a K group of the slice per wavefront");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane & 31, hh = lane >> 5;
    const int64_t row0 = (int64_t)blockIdx.y * 32;
    const int rows = a.M - row0 < 32 ? (int)(a.M - row0) : 32;
    const int gb = blockIdx.x * a.slice_groups;
    const int count = a.G - gb < a.slice_groups ? (int)a.G - gb : a.slice_groups;
    float* red = reinterpret_cast<float*>(lds + a.slice_groups * 4096);

    // What does not wait for the maxima is asked for first: the values of this thread's first codes (a wavefront quantizes rows
    // w, w + NW, .., a lane half a run of 32 elements), and A_k's records of the wavefront's group.
    const int per_row = count * 8, in = lane < per_row ? lane : per_row - 1;
    f32x4 iv[4];
    auto load_item = [&](int r) {
        const float* x = a.X + (row0 + r) * a.ldx + (int64_t)gb * 128 + in * 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) iv[j] = *reinterpret_cast<const f32x4*>(x + 4 * j);
    };
    if (wave < rows) load_item(wave);
    i32x4 aw[4];
    float asc = 0.f;
    auto load_a = [&](int rg) {
        const uint8_t* rec = a.At + ((int64_t)rg * a.G + gb + wave) * 4096 + lane * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) aw[q] = *reinterpret_cast<const i32x4*>(rec + q * 1024);
        asc = a.Asc[((int64_t)rg * a.G + gb + wave) * 32 + t];
    };
    if (a.kp32 > 0 && wave < count) load_a(0);

    // Row maxima: up to eight rows are shared by several wavefronts; a batch of loads covers 4096 values.
    const int wl = rows > 8 ? (NW == 16 ? 4 : 3) : (rows > 4 ? 3 : (rows > 2 ? 2 : rows - 1)), parts = NW >> wl;
    {
        constexpr int NB = 16;                       // float4 per lane and batch
        const int n4 = (int)a.G * 32;                // float4 per row, a multiple of `parts`
        const int part = wave >> wl, len = (n4 << wl) / NW, begin = part * len;
        for (int r = wave & ((1 << wl) - 1); r < rows; r += 1 << wl) {
            const uint8_t* x = reinterpret_cast<const uint8_t*>(a.X + (row0 + r) * a.ldx) + (int64_t)begin * 16;
            float m = 0.f;
            for (int b0 = 0; b0 < len; b0 += 64 * NB) {
                f32x4 v[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int i = b0 + j * 64 + lane;
                    v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (b0 + j * 64 < len) v[j] = *reinterpret_cast<const f32x4*>(x + (uint32_t)((i < len ? i : len - 1) * 16));
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[j][0]), __builtin_fabsf(v[j][1])),
                                                           __builtin_fmaxf(__builtin_fabsf(v[j][2]), __builtin_fabsf(v[j][3]))));
            }
            m = wave_max(m);
            if (lane == 0) pmax[part][r] = m;
        }
    }
    __syncthreads();

    // codes of the slice
    uint8_t* xc = a.Xc + (int64_t)blockIdx.y * a.K * 32;
    for (int r = wave; r < rows; r += NW) {
        if (r != wave) load_item(r);
        float m = pmax[0][r];
        for (int p = 1; p < parts; ++p) m = __builtin_fmaxf(m, pmax[p][r]);
        // s = fp16(amax / 127), the division in fp32 and correctly rounded; 1 for an all-zero row
        float s = (m == 0.f) ? 1.0f : (float)(_Float16)__fdiv_rn(m, 127.0f);
        s = f32_from_bits(__builtin_amdgcn_readfirstlane(f32_bits(s)));
        if (lane == 0) {
            smax[r] = s;
            if (blockIdx.x == 0) a.Xs[row0 + r] = s;
        }
        uint32_t c4[4][4];
        Int8Coder(s).codes(iv, c4);
        const int half = in & 1, run = in >> 1;
        u32x2 ev = u32x2{0, 0}, od = u32x2{0, 0};    // half of two cells: the half run's even elements, and its odd ones
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t c = c4[j][e];
                const int k = 2 * j + (e >> 1);      // position among the half's even or odd elements
                if (e & 1) od[k >> 2] |= c << (8 * (k & 3));
                else ev[k >> 2] |= c << (8 * (k & 3));
            }
        if (lane >= per_row) continue;
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
        if (rg > 0) __syncthreads();                 // the sums of the rank group before have been read
        if (wave < count) {
            if (rg > 0) load_a(rg);
            i32x4 x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                x[q] = *reinterpret_cast<const i32x4*>(lds + ((wave * 8 + 4 * (q >> 1) + 2 * hh + (q & 1)) * 32 + row) * 16);
            const i32x16 s = i8_products(x, aw);
#pragma unroll
            for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = (float)s[r] * asc;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16 / NW; ++i) {          // wavefront w finishes register w (and w + 8)
            const int reg = wave + 8 * i, orow = result_row(reg, hh);
            float v = red[reg * 64 + lane];
            for (int w = 1; w < count; ++w) v += red[(w * 16 + reg) * 64 + lane];
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
    // Buffers of the workgroup's column group and token block: a K group past the last lies past their end (no access, zeros)
    const BufferRsrc wbuf = buffer_rsrc(a.Wt + cg * a.G * 2048, (uint32_t)G * 2048u), sbuf = buffer_rsrc(a.Wsc + cg * a.G * 32, (uint32_t)G * 128u);
    const int cell = 16 << a.lr;                     // bytes from one cell column to the next
    const BufferRsrc xbuf = buffer_rsrc(a.Xc + (int64_t)blockIdx.y * a.K * 32, (uint32_t)(G * 8 * cell));

    struct Set { u32x4 c[2]; i32x4 x[4]; float s; };
    auto load = [&](Set& d, int g) {
        d.c[0] = buffer_load16_nt(wbuf, g * 2048 + lane * 16);
        d.c[1] = buffer_load16_nt(wbuf, g * 2048 + 1024 + lane * 16);
        d.s = f32_from_bits(buffer_load4(sbuf, g * 128 + t * 4));
#pragma unroll
        for (int q = 0; q < 4; ++q)
            d.x[q] = __builtin_bit_cast(i32x4, buffer_load16(xbuf, (g * 8 + 4 * (q >> 1) + 2 * hh + (q & 1)) * cell + row * 16));
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
    load(s0, wave);
    load(s1, wave + 8);
    load(s2, wave + 16);
    load(s3, wave + 24);
    __builtin_amdgcn_sched_barrier(0);
    // what is needed after the product: scales of this thread's two results, rank block `wave` of B_k and the first eight
    // partial sums of T
    const int64_t n = cg * 32 + t;
    const float sb = a.kp16 > 0 ? a.Bsc[n] : 0.f;
    float st[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int orow = result_row(2 * wave + i, hh);
        st[i] = a.Xs[row0 + (orow < rows ? orow : rows - 1)];
    }
    const bool tail = wave < a.kp16;
    u32x4 bw;                                        // (given a value here, it would be copied - and waited for - where the branch ends)
    f32x4 p0 = f32x4{0.f, 0.f, 0.f, 0.f}, p1 = p0;
    f32x4 q0[8], q1[8];
    const int64_t ldt = (int64_t)a.kp32 * 32, stride = a.M * ldt;
    const float* src = a.T + (row0 + row) * ldt + wave * 16 + 8 * hh;
    auto load_t = [&](int z0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int z = z0 + j < a.S ? z0 + j : a.S - 1;
            q0[j] = *reinterpret_cast<const f32x4*>(src + z * stride);
            q1[j] = *reinterpret_cast<const f32x4*>(src + z * stride + 4);
        }
    };
    if (tail) {
        bw = *reinterpret_cast<const u32x4*>(a.Bt + (cg * a.kp16 + wave) * kBRecordBytes + t * 16);
        load_t(0);
    }
    int g = wave;
    for (; g + 32 < G; g += 32) {
        use(s0);
        load(s0, g + 32);
        use(s1);
        load(s1, g + 40);
        use(s2);
        load(s2, g + 48);
        use(s3);
        load(s3, g + 56);
    }
    if (g < G) use(s0);
    if (g + 8 < G) use(s1);
    if (g + 16 < G) use(s2);
    if (g + 24 < G) use(s3);
    if (tail) {                                      // the partial sums in slice order
        for (int z0 = 0;;) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (z0 + j < a.S) { p0 += q0[j]; p1 += q1[j]; }
            z0 += 8;
            if (z0 >= a.S) break;
            load_t(z0);
        }
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
    for (int r = 0; r < 16; ++r) red[((wave * 2) * 16 + r) * 64 + lane] = acc[r];
    if (tail) {
#pragma unroll
        for (int r = 0; r < 16; ++r) red[((wave * 2 + 1) * 16 + r) * 64 + lane] = ta[r];
    }
    __syncthreads();
    const int nt = a.kp16 < kFewWaves ? a.kp16 : kFewWaves;
#pragma unroll
    for (int i = 0; i < 2; ++i) {                    // wavefront w finishes registers 2 w and 2 w + 1
        const int r = 2 * wave + i, orow = result_row(r, hh);
        float v = red[r * 64 + lane];
#pragma unroll
        for (int w = 1; w < kFewWaves; ++w) v += red[((w * 2) * 16 + r) * 64 + lane];
        float c = 0.f;
        for (int w = 0; w < nt; ++w) c += red[((w * 2 + 1) * 16 + r) * 64 + lane];
        if (orow < rows && n < a.N) a.Y[(row0 + orow) * a.ldy + n] = v * st[i] + c * sb;
    }
}

hipError_t launch_int_few(const IntFewArgs& a, hipStream_t s) {
    const unsigned blocks = (unsigned)((a.M + 31) / 32);
    if (a.slice_groups > kFewSliceGroups) return hipErrorInvalidValue;
    const size_t prep_lds = (size_t)a.slice_groups * 8192;
    if (a.M <= 8) hipLaunchKernelGGL(int_few_prep_kernel<8>, dim3((unsigned)a.S, blocks), dim3(64 * 8), prep_lds, s, a);
    else hipLaunchKernelGGL(int_few_prep_kernel<16>, dim3((unsigned)a.S, blocks), dim3(64 * 16), prep_lds, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(int_few_kernel, dim3((unsigned)a.N32, blocks), dim3(64 * kFewWaves), (size_t)kFewWaves * 8192, s, a);
    return hipGetLastError();
}

}  // namespace lqer
