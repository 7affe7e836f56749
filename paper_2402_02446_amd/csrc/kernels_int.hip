// The scaled-integer variant of the layer (Table 2, "L2QER-INT": INT4 weights in groups of 128 with FP16 scales,
// INT8 activations with one scale per token, INT8 rank-k factors; Sec. 2.1 for the form of such formats):
//   Y[t][n] = s_t sum_g sW[n][g] I_W[t][n][g]  +  sum_r T[t][r] Bc[r][n] sB[n],   T[t][r] = s_t sum_g sA[r][g] I_A[t][r][g]
// with I the exact integer inner product of one group of 128 codes.  An FP16 scale times a code is no bf16 number, so
// the scales cannot be folded into the operands the way MXINT's powers of two are; instead the integer products run on
// the int8 matrix cores (32x32x32, exact in i32) and every group's sum is converted and scaled once, in fp32.
//
//   quant_token_kernel   per-token INT8 quantizer (one workgroup per token row: row maximum, then codes)
//   int_prep_kernel      the quantizer and the projection T = X_q A_k in one launch, 8 tokens per workgroup: ranks up to 64, smaller calls
//   int_main_kernel      the main product with the rank-k correction (T_hi | T_lo against B_k's codes on the bf16 matrix
//                        cores, one scale per column) in the epilogue; operands by direct-to-LDS loads.  Few tiles: K in
//                        planes, one more for the correction, that int_reduce_planes_kernel adds and scales per token
//   int_gemm_kernel      the projection T = X_q A_k, A_k as 8-bit "weights": 128 tokens x 128 ranks per workgroup, four
//                        wavefronts of 64 x 64, one K group per step, all of it asked for one group ahead
//
// Weight codes keep their canonical nibbles: of a 32-bit word (8 elements) `(w << 4) & 0xF0F0F0F0` are the even
// elements times 16 as int8 and `w & 0xF0F0F0F0` the odd ones - two instructions per 8 weights; the factor 16 is
// folded into the scale table.  A lane's 16 bytes (32 consecutive K) thus feed two MFMAs, one with the even and one
// with the odd elements, and the activation codes are stored in the same order: every run of 32 as its 16 even
// elements followed by its 16 odd ones (the contraction does not care about the order, only that both sides agree).
#include <mutex>

#include "lqer_internal.h"
#include "mx_device.h"

namespace lqer {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

// ---- per-token INT8 quantizer ----------------------------------------------------------------------------------
// PERM: codes in the order the product kernel reads them (see above); otherwise canonical.  The first NB x 1024 values of a row
// stay in registers between the two passes over it; a longer row's others are read again.  2048 tokens of 11008 x 4096, whole
// call, with a division per value and two reads 161 us, now 149; of 4096 x 11008 153 and 150.
template <bool PERM, int NB>
__global__ __launch_bounds__(256) void quant_token_kernel(const float* __restrict__ X, int64_t ldx, int64_t K,
                                                          int8_t* __restrict__ codes, int64_t ldc, float* scale_f32,
                                                          uint16_t* scale_f16) {
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const float* x = X + row * ldx;
    const int64_t n4 = K >> 2;
    auto load = [&](f32x4 (&v)[NB], int64_t i0) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int64_t i = i0 + 256 * j + threadIdx.x;
            v[j] = *reinterpret_cast<const f32x4*>(x + 4 * (i < n4 ? i : n4 - 1));
        }
    };
    float m = 0.f;
    auto look = [&](const f32x4 (&v)[NB]) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
            m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[j][0]), __builtin_fabsf(v[j][1])),
                                                   __builtin_fmaxf(__builtin_fabsf(v[j][2]), __builtin_fabsf(v[j][3]))));
    };
    f32x4 first[NB];
    load(first, 0);
    look(first);
    for (int64_t i0 = 256 * NB; i0 < n4; i0 += 256 * NB) {
        f32x4 v[NB];
        load(v, i0);
        look(v);
    }
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
    // s = fp16(amax / 127), the division in fp32 and correctly rounded; 1 for an all-zero row
    const _Float16 sh = (m == 0.f) ? (_Float16)1.0f : (_Float16)__fdiv_rn(m, 127.0f);
    const Int8Coder coder((float)sh);
    if (threadIdx.x == 0) {
        if (scale_f32) scale_f32[row] = (float)sh;
        if (scale_f16) scale_f16[row] = __builtin_bit_cast(uint16_t, sh);
    }
    int8_t* c = codes + row * ldc;
    auto store = [&](const f32x4 (&v)[NB], int64_t i0) {
        uint32_t q4[NB][4];
        coder.codes(v, q4);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int64_t i = i0 + 256 * j + threadIdx.x;
            if (i >= n4) continue;
            const uint32_t (&q)[4] = q4[j];
            if (PERM) {
                const int64_t e0 = 4 * i, span = e0 & ~(int64_t)31, h = (e0 & 31) >> 1;   // elements e0, e0+2 even; e0+1, e0+3 odd
                *reinterpret_cast<uint16_t*>(c + span + h) = (uint16_t)(q[0] | (q[2] << 8));
                *reinterpret_cast<uint16_t*>(c + span + 16 + h) = (uint16_t)(q[1] | (q[3] << 8));
            } else {
                *reinterpret_cast<uint32_t*>(c + 4 * i) = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
            }
        }
    };
    store(first, 0);
    for (int64_t i0 = 256 * NB; i0 < n4; i0 += 256 * NB) {
        f32x4 v[NB];
        load(v, i0);
        store(v, i0);
    }
}

template <bool PERM>
static void launch_quant_token_t(const float* X, int64_t rows, int64_t K, int64_t ldx, int8_t* codes, int64_t ldc,
                                 float* scale_f32, uint16_t* scale_f16, hipStream_t s) {
    // rows of up to 1024, 4096 values, longer ones: a batch's loads beyond a short row's end are clamped, not left out, and cost as
    // much as the row's own (5664 rows of 88 values 7.6 us in batches of four, 5.1 of one)
    if (K <= 1024) hipLaunchKernelGGL((quant_token_kernel<PERM, 1>), dim3((unsigned)rows), dim3(256), 0, s, X, ldx, K, codes, ldc, scale_f32, scale_f16);
    else if (K <= 4096) hipLaunchKernelGGL((quant_token_kernel<PERM, 4>), dim3((unsigned)rows), dim3(256), 0, s, X, ldx, K, codes, ldc, scale_f32, scale_f16);
    else hipLaunchKernelGGL((quant_token_kernel<PERM, 12>), dim3((unsigned)rows), dim3(256), 0, s, X, ldx, K, codes, ldc, scale_f32, scale_f16);
}

hipError_t launch_quant_token(const float* X, int64_t rows, int64_t K, int64_t ldx, int8_t* codes, int64_t ldc,
                              float* scale_f32, uint16_t* scale_f16, bool perm, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (perm) launch_quant_token_t<true>(X, rows, K, ldx, codes, ldc, scale_f32, scale_f16, s);
    else launch_quant_token_t<false>(X, rows, K, ldx, codes, ldc, scale_f32, scale_f16, s);
    return hipGetLastError();
}

// ---- quantizer and projection in one launch ------------------------------------------------------------------------
// A workgroup has 8 tokens, its wavefronts the K groups in turn: row maxima, then codes to the workspace and from LDS, as operands, into
// T = X_q A_k, summed over the wavefronts in wavefront order.  The first kKeep groups of a wavefront stay in registers between the two
// passes; later ones are read again.  A wavefront's loads cover two rows of a group each; its codes change hands through 1 KB of LDS, from
// where a lane takes one cell of 16.  The 32 rows of an MFMA's operand are the tokens four times, each time with another cell of every
// lane half: four MFMAs with a group's four A_k operands, of each of which one block of rows is the tokens' share of the sum.
// Bound by latency and by A_k's way from L2 (32 bytes per K and rank group, a workgroup): which calls take it, fused_prep in int_host.cpp.
// Beside quantizer, projection in planes and their sum (8.4 + 7.9 + 4.7 us and the gaps at 2048 tokens of 4096, rank 32), whole calls, N = 512:
// 130 tokens of 512 21.3 -> 14.2 us, of 4096 23.8 -> 18.5, 2048 tokens of 4096 41.1 -> 34.2, of 11008 64.3 -> 56.4.  With 16 tokens
// a workgroup 15.2, 23.2, 40.4 and 64.8: half the workgroups, each with twice the vector work.
constexpr int kIntPrepRows = 8, kIntPrepRun = 32 * 16 + 32;     // bytes of LDS per run of 32 of K, 8 banks apart

template <int NW, int RG>
__global__ __launch_bounds__(64 * NW) void int_prep_kernel(IntPrepArgs a) {
    constexpr int ROWS = kIntPrepRows, J = ROWS / 2, kKeep = 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[NW * 4 * kIntPrepRun];       // a tile of codes, then 256 sums, per wavefront
    __shared__ float pmax[ROWS][2 * NW], scale[ROWS], inverse[ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), t = lane & 31, hh = lane >> 5;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int rows = a.M - row0 < ROWS ? (int)(a.M - row0) : ROWS;
    const int G = (int)(a.K >> 7);
    const float* src[J];                             // rows 2 j + hh (past the last: that one again)
#pragma unroll
    for (int j = 0; j < J; ++j) src[j] = a.X + (row0 + (2 * j + hh < rows ? 2 * j + hh : rows - 1)) * a.ldx + 4 * t;
    auto load = [&](f32x4 (&v)[J], int g) {
#pragma unroll
        for (int j = 0; j < J; ++j) v[j] = *reinterpret_cast<const f32x4*>(src[j] + (int64_t)g * 128);
    };
    float m[J];
#pragma unroll
    for (int j = 0; j < J; ++j) m[j] = 0.f;
    auto look = [&](const f32x4 (&v)[J]) {
#pragma unroll
        for (int j = 0; j < J; ++j)
            m[j] = __builtin_fmaxf(m[j], __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[j][0]), __builtin_fabsf(v[j][1])),
                                                         __builtin_fmaxf(__builtin_fabsf(v[j][2]), __builtin_fabsf(v[j][3]))));
    };
    f32x4 kept[kKeep][J];
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (wave + i * NW < G) load(kept[i], wave + i * NW);
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (wave + i * NW < G) look(kept[i]);
    for (int g = wave + kKeep * NW; g < G; g += NW) {
        f32x4 v[J];
        load(v, g);
        look(v);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        float x = m[j];                              // over 16 lanes, as in wave_max
        x = __builtin_fmaxf(x, dpp_move<0xB1>(x));
        x = __builtin_fmaxf(x, dpp_move<0x4E>(x));
        x = __builtin_fmaxf(x, dpp_move<0x141>(x));
        x = __builtin_fmaxf(x, dpp_move<0x140>(x));
        if ((lane & 15) == 0) pmax[2 * j + hh][2 * wave + ((lane >> 4) & 1)] = x;
    }
    __syncthreads();
    if (tid < 16 * ROWS) {                           // 16 lanes per row
        const int row = tid >> 4, part = tid & 15;
        float x = 2 * NW >= 16 || part < 2 * NW ? pmax[row][part] : 0.f;
        if (2 * NW > 16) x = __builtin_fmaxf(x, pmax[row][(part + 16) % (2 * NW)]);
        x = __builtin_fmaxf(x, dpp_move<0xB1>(x));
        x = __builtin_fmaxf(x, dpp_move<0x4E>(x));
        x = __builtin_fmaxf(x, dpp_move<0x141>(x));
        x = __builtin_fmaxf(x, dpp_move<0x140>(x));
        // s = fp16(amax / 127), the division in fp32 and correctly rounded; 1 for an all-zero row
        const float s = (x == 0.f) ? 1.0f : (float)(_Float16)__fdiv_rn(x, 127.0f);
        if (part == 0) {
            scale[row] = s;
            inverse[row] = __fdiv_rn(1.0f, s);
            if (row < rows) a.Xs[row0 + row] = s;
        }
    }
    __syncthreads();

    float acc[RG][4];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[rg][r] = 0.f;
    uint8_t* tile = lds + wave * 4 * kIntPrepRun;
    uint8_t* put = tile + (t >> 3) * kIntPrepRun + hh * 16 + 2 * (t & 7);            // [run of 32][even, odd][row][16 B]
    const int row = t & 7, run = 2 * (t >> 4) + hh, odd = (t >> 3) & 1;              // as operand: row t % 8, cell 4 sp + 2 hh + p, 2 sp + p = t / 8
    const uint8_t* get = tile + run * kIntPrepRun + odd * 256 + row * 16;
    int8_t* dst = a.Xc + (row0 + row) * a.K + run * 32 + odd * 16;
    auto group = [&](const f32x4 (&v)[J], int g) {
        i32x4 w[4];
        float sc;
        auto load_a = [&](int rg) {
            const uint8_t* rec = a.At + ((int64_t)rg * G + g) * 4096 + lane * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = *reinterpret_cast<const i32x4*>(rec + q * 1024);
            sc = a.Asc[((int64_t)rg * G + g) * 32 + t];
        };
        load_a(0);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const f32x4 one[1] = {v[j]};
            uint32_t c[1][4];
            Int8Coder(scale[2 * j + hh], inverse[2 * j + hh]).codes(one, c);
            *reinterpret_cast<uint16_t*>(put + 32 * j) = (uint16_t)(c[0][0] | (c[0][2] << 8));
            *reinterpret_cast<uint16_t*>(put + 32 * j + 256) = (uint16_t)(c[0][1] | (c[0][3] << 8));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                           // (only this wavefront's lanes read them)
        const i32x4 x = *reinterpret_cast<const i32x4*>(get);
        asm volatile("" ::: "memory");
        if (row < rows) *reinterpret_cast<i32x4*>(dst + (int64_t)g * 128) = x;
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) {
            if (rg > 0) load_a(rg);
            i32x16 s[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
#pragma unroll
                for (int r = 0; r < 16; ++r) s[b][r] = 0;
                s[b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x, w[b], s[b], 0, 0, 0);
            }
            // rows 8 b .. + 7 of the product with w[b] are in its registers 4 b .. + 3
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rg][r] += (float)(s[0][r] + s[1][4 + r] + s[2][8 + r] + s[3][12 + r]) * sc;
        }
    };
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (wave + i * NW < G) group(kept[i], wave + i * NW);
    for (int g = wave + kKeep * NW; g < G; g += NW) {
        f32x4 v[J];
        load(v, g);
        group(v, g);
    }
    // register r of lane (t, hh): token 4 hh + r, rank t
    float* red = reinterpret_cast<float*>(lds);
    static_assert(64 * 4 * 4 <= 4 * kIntPrepRun, "a wavefront's sums in its tile's place");
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
        __syncthreads();                             // the tiles, or the sums before these, have been read
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(wave * 4 + r) * 64 + lane] = acc[rg][r];
        __syncthreads();
        for (int item = tid; item < 256; item += 64 * NW) {
            float v = red[item];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += red[w * 256 + item];
            const int orow = 4 * ((item >> 5) & 1) + (item >> 6);
            if (orow < rows) a.T[(row0 + orow) * a.ldt + rg * 32 + (item & 31)] = v * scale[orow];
        }
    }
}

template <int NW>
static void launch_int_prep_t(const IntPrepArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)((a.M + kIntPrepRows - 1) / kIntPrepRows)), block(64 * NW);
    if (a.ldt == 32) hipLaunchKernelGGL((int_prep_kernel<NW, 1>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((int_prep_kernel<NW, 2>), grid, block, 0, s, a);
}

// Ranks up to 64.  About two K groups a wavefront: more wavefronts would be idle, fewer longer chains.
hipError_t launch_int_prep(const IntPrepArgs& a, hipStream_t s) {
    if (a.M == 0) return hipSuccess;
    if (a.K <= 1024) launch_int_prep_t<4>(a, s);
    else if (a.K <= 2048) launch_int_prep_t<8>(a, s);
    else launch_int_prep_t<16>(a, s);
    return hipGetLastError();
}

// ---- the product kernel ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void int_gemm_kernel(IntGemmArgs a) {
    constexpr int TM = 2, TN = 2;
    constexpr int NL = 4;                            // 16-byte loads per lane, column group and K group
    constexpr int REC = NL * 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t xs[2][128 * 128];
    __shared__ __attribute__((aligned(16))) float ss[2][128];      // the K group's scales of the tile's 128 columns

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int t = lane & 31, hh = lane >> 5;
    const int64_t m0 = (int64_t)blockIdx.y * 128;
    const int64_t g0 = ((int64_t)blockIdx.x * 2 + wc) * TN;        // first column group of this wavefront
    auto clamp_group = [&](int64_t g) { return g < a.N32 ? g : a.N32 - 1; };   // (the store is masked)
    auto group_of = [&](int tn) { return clamp_group(g0 + tn); };
    // activation loader: thread -> four 16-byte cells of a 128 x 128 byte tile
    const int ld_row = tid >> 3, ld_cell = tid & 7;
    const int8_t* ld_src = a.Xc + (m0 + ld_row) * a.ldxc + ld_cell * 16;
    const int ld_dst = ld_row * 128 + ((ld_cell ^ ((ld_row >> 1) & 7)) << 4);   // rows 32 apart share the swizzle term
    // scale loader: the first 32 threads bring the 4 x 32 scales of the tile's column groups (four floats each)
    const float* sc_src = a.Wsc + clamp_group((int64_t)blockIdx.x * 4 + ((tid >> 3) & 3)) * a.G * 32 + (tid & 7) * 4;
    const int sc_dst = ((tid >> 3) & 3) * 32 + (tid & 7) * 4;
    struct XStage { u32x4 x[4]; f32x4 s; };
    auto fetch_x = [&](XStage& st, int64_t g) {
#pragma unroll
        for (int j = 0; j < 4; ++j) st.x[j] = *reinterpret_cast<const u32x4*>(ld_src + (int64_t)j * 32 * a.ldxc + g * 128);
        st.s = *reinterpret_cast<const f32x4*>(sc_src + g * 32);     // (every thread: the wavefronts beyond the first ask for the same lines again)
    };
    auto store_x = [&](const XStage& st, int buf) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4*>(&xs[buf][ld_dst + j * 32 * 128]) = st.x[j];
        if (tid < 32) *reinterpret_cast<f32x4*>(&ss[buf][sc_dst]) = st.s;
    };
    struct WSet { u32x4 c[TN][NL]; };
    auto load_w = [&](WSet& w, int64_t g) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint8_t* rec = a.Wt + (group_of(tn) * a.G + g) * REC + lane * 16;
#pragma unroll
            for (int l = 0; l < NL; ++l) w.c[tn][l] = *reinterpret_cast<const u32x4*>(rec + l * 1024);
        }
    };
    // operand read: MFMA (sp, p) of a group uses bytes 64 sp + 32 hh + 16 p .. + 15 of the token's 128: cell 4 sp + 2 hh + p
    const int rd_row = wr * 64 + t;
    auto read_x = [&](int buf, int tm, int sp, int p) {
        const int row = rd_row + tm * 32;
        const int cell = (4 * sp + 2 * hh + p) ^ ((row >> 1) & 7);   // rows are 128 B = half of the banks: 16 rows of a read hit 16 different bank groups
        return *reinterpret_cast<const i32x4*>(&xs[buf][row * 128 + (cell << 4)]);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tm][tn][r] = 0.f;

    float st[TM];                                    // token scales (for the epilogue; asked for here, ahead of the loop)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) st[tm] = a.Xs[m0 + wr * 64 + tm * 32 + t];

    // this workgroup's K groups [gb, ge)
    const int64_t gb = (int64_t)blockIdx.z * a.g_per_z;
    const int64_t ge = gb + a.g_per_z < a.G ? gb + a.g_per_z : a.G;
    WSet w0, w1;
    XStage stx;
    fetch_x(stx, gb);
    load_w(w0, gb);
    store_x(stx, 0);

    // One K group.  The next group's activations, scales and weights are asked for first and stay in flight through the
    // step (they land in LDS / become `cur` at its end); the column groups are worked one after the other, so that the
    // conversion and scaling of one's sums can run beside the MFMAs of the other.
    auto step = [&](const WSet& cur, WSet& nxt, int64_t g) {
        __syncthreads();                             // tile g is complete; the other buffer is free again
        const int buf = (int)((g - gb) & 1);
        const int64_t gn = g + 1 < ge ? g + 1 : g;   // clamped: loads stay unconditional
        fetch_x(stx, gn);
        load_w(nxt, gn);
        __builtin_amdgcn_sched_barrier(0);           // (not to be sunk towards their uses: that would put the round trip on the step's path)
        i32x4 xb[2][2][TM];
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) xb[sp][p][tm] = read_x(buf, tm, sp, p);
        auto products = [&](i32x16 (&ia)[TM], int tn) {
#pragma unroll
            for (int sp = 0; sp < 2; ++sp)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const i32x4 wv = __builtin_bit_cast(i32x4, cur.c[tn][2 * sp + p]);
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) {
                        if (sp == 0 && p == 0) {
                            i32x16 z;
#pragma unroll
                            for (int r = 0; r < 16; ++r) z[r] = 0;
                            ia[tm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv, xb[sp][p][tm], z, 0, 0, 0);
                        } else {
                            ia[tm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv, xb[sp][p][tm], ia[tm], 0, 0, 0);
                        }
                    }
                }
        };
        // the group's exact integer sums, scaled once: register r of a lane is column 8 (r / 4) + 4 hh + r % 4
        auto fold = [&](const i32x16 (&ia)[TM], int tn) {
            f32x4 sc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) sc[q] = *reinterpret_cast<const f32x4*>(&ss[buf][(wc * 2 + tn) * 32 + 8 * q + 4 * hh]);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[tm][tn][r] += (float)ia[tm][r] * sc[r >> 2][r & 3];
        };
        // (the empty asm statements keep the arithmetic where it is written: nothing else orders pure instructions
        // against the scheduling barriers, and left alone they all sink to the end of the step)
        i32x16 ia0[TM], ia1[TM];
        products(ia0, 0);
        asm volatile("" : "+v"(ia0[0]), "+v"(ia0[1]));
        __builtin_amdgcn_sched_barrier(0);
        // the second column group's MFMAs run while the first one's sums are converted and scaled
        products(ia1, 1);
        fold(ia0, 0);
        asm volatile("" : "+v"(ia1[0]), "+v"(ia1[1]), "+v"(acc[0][0]), "+v"(acc[1][0]));
        __builtin_amdgcn_sched_barrier(0);
        fold(ia1, 1);
        asm volatile("" : "+v"(acc[0][1]), "+v"(acc[1][1]));
        __builtin_amdgcn_sched_barrier(0);
        store_x(stx, buf ^ 1);                       // last read two barriers ago (a clamped re-write of the last tile is harmless)
    };
    for (int64_t g = gb; g < ge; g += 2) {
        step(w0, w1, g);
        if (g + 1 < ge) step(w1, w0, g + 1);
    }

    // ---- epilogue: token scale, store (padded rows too: the main kernel reads them) ----------------------------------------------------------
    if (!a.planes) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[tm][tn][r] *= st[tm];
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t row = m0 + wr * 64 + tm * 32 + t;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int64_t cg = g0 + tn;
            if (cg >= a.N32) continue;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int64_t n = cg * 32 + 8 * r4 + 4 * hh;
                float* dst = a.Out + (int64_t)blockIdx.z * a.out_z_stride + row * a.ldo + n;
                const f32x4 v = f32x4{acc[tm][tn][4 * r4], acc[tm][tn][4 * r4 + 1], acc[tm][tn][4 * r4 + 2], acc[tm][tn][4 * r4 + 3]};
                if (n + 3 < a.N) {
                    *reinterpret_cast<f32x4*>(dst) = v;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (n + j < a.N) dst[j] = v[j];
                }
            }
        }
    }
}

// ---- the main product ----------------------------------------------------------------------------------------------
// Y = s_t sum_g sW I_W + T B_k on 128 tokens x 128 columns per workgroup, four wavefronts of 128 x 32, one K group of 128
// at a time.  Beside the int8 matrix pipe (16 MFMAs of 32 cycles a group and wavefront) it is bound by vector
// instructions: converting and scaling the group's exact sums costs two per accumulator register, 128 a group (the FP16
// group scales leave no way round it), the nibbles' expansion 24.  A loop of just these, two wavefronts on a SIMD, takes
// 0.90 us a group against 0.67 us of its MFMAs alone (at the clock each of them sustains).  So
//   * activations, nibbles and scales reach LDS by direct loads two groups ahead (three stages of 25 KB, two workgroups on
//     a compute unit), counted by the kernel itself: no registers, no address arithmetic per load;
//   * a wavefront owns all 128 tokens of 32 columns, so a nibble is expanded once per workgroup;
//   * tokens are the rows and columns the lanes of the MFMA's result: a lane needs one scale per group;
//   * the sums of two 32 x 32 tiles are folded beside the MFMAs of the other two, laced instruction by instruction.
// Whole calls at rank 32, by int_gemm_kernel's tiles -> so: 2048 tokens of 4096 x 11008 162 -> 141 us, of 11008 x 4096
// 163 -> 149, 65536 tokens of 4096 x 4096 1849 -> 1672.  Left out one at a time, the loads cost 8 % of the time, the folding 12 %, the LDS reads 22 %,
// three quarters of the MFMAs 24 %: what was left was the phases of a group waiting for each other, the two workgroups of a compute unit
// in step.  So a wavefront's priority is raised while it has MFMAs to issue, the earlier half of a group above the later, and
// falls for the wait, the reads and the folding before them: its neighbour then does these beside its MFMAs, and reads never hold up a
// wavefront that could issue.  2048 tokens of 4096 x 11008, whole call, no priorities 150.5 us, raised for the later half 140.5, for both
// alike 138.5, so 138.0; raised from the reads on 151.  (With X all zeros 138 -> 125: it is waiting that went, not power.)
constexpr int kIntStages = 3, kIntStage = 128 * 128 + 4 * (2048 + 256);

__global__ __launch_bounds__(256, 2) void int_main_kernel(IntGemmArgs a) {
    constexpr int NW = 4, BN = 32 * NW, WOFF = 128 * 128, SOFF = WOFF + NW * 2048;
    constexpr int XL = 16 / NW, L = XL + 3;          // loads per wavefront and group: 4 activations, 2 nibbles, 1 scales
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane & 31, hh = lane >> 5;

    // workgroup -> K plane and output tile, in bands of eight tile rows.  Consecutive positions land on one XCD, which then shares
    // activations or weights - but where one tile row is all there is and its tiles alone fill the chip's XCDs, that only crowds
    // each XCD's part of the weights: 64 tokens of 2048 x 16384 take 27.2 us so and 22.7 as numbered, of 1920 x 20848 1 to 4 %
    // more (as numbered everywhere up to 1000 tokens, 50 layers took 1.4 % longer on average, 800 tokens of 11008 x 800 18 %).
    // (Both numbers, and a select: a branch here or at the token scales below changes the order the compiler gives the loop's
    // LDS reads and MFMAs, up to 4 % of a prefill call.)
    const int grid_n = (int)((a.N + BN - 1) / BN), grid_m = (int)((a.M + 127) / 128);
    int lin;
    {
        const int nwg = gridDim.x, pid = blockIdx.x;
        const int xcd = pid & 7, local = pid >> 3, per = nwg >> 3, rem = nwg & 7;
        const int walk = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
        lin = __builtin_amdgcn_readfirstlane(grid_m == 1 && grid_n >= 96 ? pid : walk);
    }
    const int plane = lin / (grid_m * grid_n);
    lin -= plane * (grid_m * grid_n);
    int tile_m, tile_n;
    {
        const int width = 8 * grid_n, grp = lin / width, in = lin - grp * width, first_m = grp * 8;
        const int gsize = (grid_m - first_m < 8) ? grid_m - first_m : 8;
        tile_m = first_m + in % gsize;
        tile_n = in / gsize;
    }
    const int64_t m0 = (int64_t)tile_m * 128;
    const int64_t cg = (int64_t)tile_n * NW + wave, cgc = cg < a.N32 ? cg : a.N32 - 1;   // this wavefront's column group (the store is masked)
    const int gb = plane * (int)a.g_per_z;                         // K groups [gb, gb + count)
    const int count = gb + (int)a.g_per_z < (int)a.G ? (int)a.g_per_z : (gb < (int)a.G ? (int)a.G - gb : 0);   // (0: a plane for the correction only)

    // ---- loads: activations 8 rows each (cells XOR-swizzled by row), codes and scales of the wavefront's column group
    uint32_t x_off[XL];
#pragma unroll
    for (int j = 0; j < XL; ++j)
        x_off[j] = (uint32_t)((8 * (NW * j + wave) + (lane >> 3)) * (int)a.ldxc) +
                   (((uint32_t)(lane & 7) ^ (uint32_t)(((wave & 1) * 4 + (lane >> 4)) & 7)) << 4);
    const uint32_t w_off = lane * 16;
    const uint32_t s_off = t * 4;                    // (both lane halves bring the same 32 scales)
    const uint8_t* x_ptr = reinterpret_cast<const uint8_t*>(a.Xc + m0 * a.ldxc + (int64_t)gb * 128);
    const uint8_t* w_ptr = a.Wt + (cgc * a.G + gb) * 2048;
    const uint8_t* s_ptr = reinterpret_cast<const uint8_t*>(a.Wsc + (cgc * a.G + gb) * 32);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)lds);
    auto issue = [&](uint32_t stage) {               // the next group -> the stage at that byte offset
        const uint32_t at_x = lds0 + stage + wave * 1024, at_w = lds0 + stage + wave * 2048, at_s = lds0 + stage + wave * 256;
        lds_dma16<0>(at_x, x_off[0], x_ptr);
        lds_dma16<NW * 1024>(at_x, x_off[1], x_ptr);
        lds_dma16<2 * NW * 1024>(at_x, x_off[2], x_ptr);
        lds_dma16<3 * NW * 1024>(at_x, x_off[3], x_ptr);
        lds_dma16<WOFF>(at_w, w_off, w_ptr);
        lds_dma16<WOFF + 1024>(at_w, w_off, w_ptr + 1024);
        lds_dma4<SOFF>(at_s, s_off, s_ptr);
        x_ptr += 128;
        w_ptr += 2048;
        s_ptr += 128;
    };

    // ---- operands: MFMA (sp, p) of a group uses bytes 64 sp + 32 hh + 16 p .. + 15 of the token's 128: cell 4 sp + 2 hh + p
    int rd_x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) rd_x[q] = t * 128 + (((4 * (q >> 1) + 2 * hh + (q & 1)) ^ ((t >> 1) & 7)) << 4);
    const int rd_w = WOFF + wave * 2048 + lane * 16, rd_s = SOFF + wave * 256 + t * 4;

    f32x16 acc[4];                                   // [tm]: register r = token 8 (r / 4) + 4 hh + r % 4, lane t = column
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
    i32x16 pend[2];                                  // sums of tiles 2 and 3 of the group before, not folded yet
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) pend[i][r] = 0;
    float pend_sc = 0.f;
    auto fold = [&](f32x16& c, const i32x16& i, float s) {
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] += (float)i[r] * s;
    };
    // the 128 products of two tiles, one K quarter after the other
    auto products = [&](i32x16 (&s)[2], const i32x4 (&x)[2][4], const i32x4 (&w)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                i32x16 z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0;
                s[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[i][q], w[q], q == 0 ? z : s[i], 0, 0, 0);
            }
    };
    auto expand = [&](i32x4 (&w)[4], const u32x4 (&c)[2]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[q][e] = (int)(((q & 1) ? c[q >> 1][e] : c[q >> 1][e] << 4) & 0xF0F0F0F0u);
    };
    auto group = [&](const uint8_t* st, bool more, uint32_t st_in) {   // more: the group two behind goes to the stage at st_in
        u32x4 cw[2];
        i32x4 x0[2][4], x1[2][4], w[4];
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) cw[sp] = *reinterpret_cast<const u32x4*>(st + rd_w + sp * 1024);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) x0[i][q] = *reinterpret_cast<const i32x4*>(st + rd_x[q] + i * 4096);
        const float sc = *reinterpret_cast<const float*>(st + rd_s);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i) x1[i][q] = *reinterpret_cast<const i32x4*>(st + rd_x[q] + (2 + i) * 4096);
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue(st_in);                      // (behind the reads, which the group is waiting for: 1 us of 139)
        __builtin_amdgcn_sched_barrier(0);
        fold(acc[2], pend[0], pend_sc);              // while the reads are on their way
        __builtin_amdgcn_sched_barrier(0);
        // behind every MFMA a few vector instructions: the rest of the group before, then the first two tiles
        __builtin_amdgcn_s_setprio(2);
        i32x16 s[2];
        expand(w, cw);
        products(s, x0, w);
        fold(acc[3], pend[1], pend_sc);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x2, 7, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        products(pend, x1, w);
        fold(acc[0], s[0], sc);
        fold(acc[1], s[1], sc);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        pend_sc = sc;
    };
    auto next_stage = [](uint32_t s) { return s + kIntStage == kIntStages * kIntStage ? 0u : s + kIntStage; };
    if (count > 0) issue(0);
    if (count > 1) issue(kIntStage);
    uint32_t st = 0, st_in = 2 * kIntStage;
    for (int g = 0; g < count; ++g) {
        // group g has landed; the stage of group g - 1 has been read by everybody and takes group g + 2
        if (g + 1 < count) staged_wait<L>();
        else staged_wait<0>();
        group(lds + st, g + 2 < count, st_in);
        if (g + 2 < count) st_in = next_stage(st_in);
        st = next_stage(st);
    }
    // ---- token scales, rank-k correction (by one plane), store --------------------------------------------------
    const bool tail = a.kp16 > 0 && plane == a.tail_plane;
    const int64_t n = cg * 32 + t;
    const float sb = tail ? a.Bsc[cgc * 32 + t] : 0.f;
    float* dst = a.Out + (int64_t)plane * a.out_z_stride + n;
    // Its operands: wavefront w asks for T of token tile w (the others need the same tiles: split into two bf16 terms once,
    // through LDS) and for B_k's codes of its own columns, all rank blocks in flight together.  With every wavefront fetching
    // and splitting all four tiles block by block, 16 tokens of 512 x 2048 at rank 128 took 30 us by this path, now 24, and
    // 1024 tokens of 4096 x 4096 at rank 64 55, now 52.
    constexpr int RB = 8;                            // rank blocks of 16
    f32x4 p[RB][2];
    u32x4 bw[RB];
    if (tail) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb >= a.kp16) continue;
            const float* src = a.T + (m0 + wave * 32 + t) * a.ldt + rb * 16 + 8 * hh;
            p[rb][0] = *reinterpret_cast<const f32x4*>(src);
            p[rb][1] = *reinterpret_cast<const f32x4*>(src + 4);
            bw[rb] = *reinterpret_cast<const u32x4*>(a.Bt + (cgc * a.kp16 + rb) * kBRecordBytes + t * 16);
        }
    }
    fold(acc[2], pend[0], pend_sc);
    fold(acc[3], pend[1], pend_sc);
    f32x16 ta[4];
#pragma unroll
    for (int tm = 0; tm < 4; ++tm)
#pragma unroll
        for (int r = 0; r < 16; ++r) ta[tm][r] = 0.f;
    if (tail) {                                      // (the same for the whole workgroup)
        static_assert(RB * 2 * 4 * 1024 <= kIntStages * kIntStage, "[rank block][term][token tile][64 lanes][16 B]");
        __syncthreads();                             // every wavefront is done with the stages
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb >= a.kp16) continue;
            Frag hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t h2[2], l2[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float v = p[rb][e >> 1][(2 * e + j) & 3];
                    const uint32_t hb = f32_bits(v) & 0xFFFF0000u;
                    h2[j] = hb >> 16;
                    l2[j] = f32_bits(v - f32_from_bits(hb)) >> 16;
                }
                hi.u[e] = h2[0] | (h2[1] << 16);
                lo.u[e] = l2[0] | (l2[1] << 16);
            }
            *reinterpret_cast<u32x4*>(lds + (((rb * 2 + 0) * 4 + wave) * 64 + lane) * 16) = hi.u;
            *reinterpret_cast<u32x4*>(lds + (((rb * 2 + 1) * 4 + wave) * 64 + lane) * 16) = lo.u;
        }
        __syncthreads();
        // one 32x32x16 step per rank block and bf16 term of T: lane half hh takes ranks 8 hh .. + 7 of the block on both sides
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb >= a.kp16) continue;
            Frag f0, f1;
            int8x16_to_frags(bw[rb], 1.0f, f0, f1);
            const Frag bf = hh ? f1 : f0;
#pragma unroll
            for (int term = 0; term < 2; ++term)
#pragma unroll
                for (int tm = 0; tm < 4; ++tm) {
                    Frag x;
                    x.u = *reinterpret_cast<const u32x4*>(lds + (((rb * 2 + term) * 4 + tm) * 64 + lane) * 16);
                    ta[tm] = mfma32(x.v, bf.v, ta[tm]);
                }
        }
    }
#pragma unroll
    for (int tm = 0; tm < 4; ++tm) {
        const int64_t row0 = m0 + tm * 32;
        // (a select, not a branch: see above)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 s4 = *reinterpret_cast<const f32x4*>(a.Xs + row0 + 8 * q + 4 * hh);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[tm][4 * q + j] *= a.planes ? 1.0f : s4[j];
        }
        if (tail) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tm][r] += ta[tm][r] * sb;
        }
        if (cg >= a.N32 || n >= a.N) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t row = row0 + 8 * (r >> 2) + 4 * hh + (r & 3);
            if (row < a.M) dst[row * a.ldo] = acc[tm][r];
        }
    }
}

// Few-token calls split the K groups of the projection and of the main product over planes of workgroups, each leaving
// its share of T or Y in the workspace; this adds the planes in plane order (the same bits on every run).
// The sum of the K planes gets its token scale here, once (scaled plane by plane, 200 tokens of 512 x 11008 were 3.7e-8 from
// the 64-bit result, now 2.5e-8, one rounding), and then the correction's plane, if there is one (tail = 1).
// Y may be the first plane itself (a thread reads all of its elements before it writes them).
__global__ __launch_bounds__(256) void int_reduce_planes_kernel(const float* P, int planes, int64_t plane_stride,
                                                                int64_t M, int64_t N, int64_t ldp, float* Y, int64_t ldy,
                                                                const float* Xs, int tail) {
    const int64_t n4 = (N + 3) / 4;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M * n4) return;
    const int64_t r = i / n4, c = 4 * (i - r * n4);
    const float* src = P + r * ldp + c;
    f32x4 v = *reinterpret_cast<const f32x4*>(src), corr = f32x4{0.f, 0.f, 0.f, 0.f};
    if (tail != 0) corr = *reinterpret_cast<const f32x4*>(src + planes * plane_stride);
    const float s = Xs[r];
    for (int z0 = 1; z0 < planes; z0 += 8) {         // eight loads in flight, added in plane order
        f32x4 q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = *reinterpret_cast<const f32x4*>(src + (z0 + j < planes ? z0 + j : planes - 1) * plane_stride);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (z0 + j < planes) v += q[j];
    }
    v = v * s + corr;
    float* dst = Y + r * ldy + c;
    if (c + 3 < N) {
        *reinterpret_cast<f32x4*>(dst) = v;
    } else {
        for (int j = 0; c + j < N; ++j) dst[j] = v[j];
    }
}

// `planes` K planes, and tail (0 or 1) of the correction behind them
hipError_t launch_int_reduce_planes(const float* P, int planes, int64_t plane_stride, int64_t M, int64_t N, int64_t ldp,
                                    float* Y, int64_t ldy, const float* Xs, int tail, hipStream_t s) {
    const int64_t items = M * ((N + 3) / 4);
    hipLaunchKernelGGL(int_reduce_planes_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, P, planes, plane_stride, M, N, ldp, Y, ldy, Xs, tail);
    return hipGetLastError();
}

// Projection T = X_q A_k: Out = T, N = padded rank.
hipError_t launch_int_projection(const IntGemmArgs& a, hipStream_t s) {
    if (a.M == 0) return hipSuccess;
    const unsigned planes = (unsigned)((a.G + a.g_per_z - 1) / a.g_per_z);
    const dim3 grid((unsigned)((a.N + 127) / 128), (unsigned)((a.M + 127) / 128), planes), block(256);
    hipLaunchKernelGGL(int_gemm_kernel, grid, block, 0, s, a);
    return hipGetLastError();
}

// Main product with the correction, in ceil(G / g_per_z) K planes (and one more where the correction has its own).
hipError_t launch_int_main(const IntGemmArgs& a, hipStream_t s) {
    if (a.M == 0) return hipSuccess;
    constexpr int LDS_BYTES = kIntStages * kIntStage;
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(int_main_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    });
    if (attr_err != hipSuccess) return attr_err;
    int64_t planes = (a.G + a.g_per_z - 1) / a.g_per_z;
    if (a.tail_plane >= planes) planes = a.tail_plane + 1;
    const int64_t wgs = ((a.M + 127) / 128) * ((a.N + 127) / 128) * planes;
    hipLaunchKernelGGL(int_main_kernel, dim3((unsigned)wgs), dim3(256), LDS_BYTES, s, a);
    return hipGetLastError();
}

}  // namespace lqer
