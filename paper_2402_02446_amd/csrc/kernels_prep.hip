// Stage 1 of the forward pass: quantize activations to MXINT8 (Sec. 4.1, block [1,16]; MXINT6 for the
// W4A6 setup of Table 2) and compute the low-rank projection T = X_q A_k (Eq. 3 / Eq. 6, first small
// matmul).
//
// One workgroup owns 16 token rows and a K slice; its wavefronts take the quarters (64 columns) of the
// slice's 256-wide K tiles in turn (its tiles, quarter by quarter, where the row-wise form below exists beside it).  Lane (t = lane % 16, q = lane / 16) owns block q of a quarter for
// token t: it finds the block maximum, quantizes, and keeps the dequantized values
// code * 2^(e-6) - exact in bf16 - both for the store to the bf16 activation matrix the main
// kernels read and as its MFMA operand.  A_k arrives already dequantized to bf16 (exactly, at
// import), so every product entering the fp32 MFMA accumulator is exact.
//
// Few-token calls are bound by the latency of this step, mid-sized ones nearly so: it is one memory round trip and one
// block's arithmetic per wavefront.  With whole tiles per wavefront and each quarter's loads behind a branch it was four round
// trips and 64 values' arithmetic one after the other; whole calls replayed from a graph (4-bit weights, rank 32):
// 4096 x 4096 at 1 token 9.4 -> 8.4 us, at 16 11.4 -> 10.4, at 40 20.6 -> 16.9, 2048 x 2048 at 64 19.0 -> 15.3,
// 4096 x 11008 at 128 36.6 -> 32.7.  Launches of 256 and more row blocks x K slices take as many wavefronts as tiles, four quarters each:
// there the chip is full, and 16 wavefronts of a quarter each were 3 % slower for a call of 2048 tokens at rank 256.
//
// S == 1: T is final; it is split into two bf16 terms T_hi + T_lo and stored behind the
//         activations of the same row, where the main kernel treats it as 2*kp more K columns.
// S  > 1: each K slice stores an fp32 partial T; the main kernel adds the slices in a fixed order.
// For the streaming kernel the activations are stored as 16-byte cells [K / 8][token row] instead
// (or as the codes themselves, see the store below); extra workgroups clear Y or the tiled
// kernel's flags where the main kernel needs that.
#include <type_traits>

#include "lqer_internal.h"
#include "mx_device.h"

namespace lqer {

struct PrepArgs {
    const float* X; int64_t ldx;
    const int8_t* Xc; const uint8_t* Xe;
    int64_t M, K;
    int64_t KT;            // K tiles
    int tiles_per_slice;
    int kp, kp16;
    int groups_per_wg;     // rank groups one plane of grid.z computes: at most 4 (the last plane may have fewer)
    int g_first;           // first rank group of plane 0
    const uint8_t* At;
    uint16_t* Xh; int64_t ldxh;
    uint16_t* Xt; int64_t ldxt;   // T_hi | T_lo | zero padding, row by row
    int64_t tail_cols;     // its columns
    uint8_t* Xe6;          // SIX: exponent bytes of the fp6 blocks (Xh: the images)
    float* Tpart;
    int64_t tp_rows;       // rows per slice of Tpart
    int lr;                // CELLS: log2 of the token rows per 16-byte cell column
    int act_frac;          // fraction bits of the activation codes: 6 (MXINT8) or 4 (MXINT6)
    bool x8;               // CELLS: store MXINT8 codes [block][row][16] and exponent bytes [block][row] instead of bf16 cells
    float* Yz; int64_t ldy, N;   // Yz != null: extra workgroups clear Y[M][N] for a main kernel that adds into it
    int nslices;                 // K slices = the part of grid.y that does the projection
    bool by_tiles;               // a wavefront takes whole tiles, otherwise quarters of them
    int nwaves;                  // wavefronts of a workgroup (an argument: blockDim costs a vector load ahead of everything else)
    uint32_t* flags; int nflags; // flags != null: words the first workgroup clears for the main kernel
};

__device__ __forceinline__ void split_bf16(float t, uint16_t& hi, uint16_t& lo) {
    const uint32_t hb = f32_bits(t) & 0xFFFF0000u;
    hi = (uint16_t)(hb >> 16);
    const float rem = t - f32_from_bits(hb);              // exact
    lo = (uint16_t)(f32_bits(rem) >> 16);
}

constexpr int kPrepWaves = 16;     // quarter-tile form, at most
constexpr int kPrepRowWaves = 8;   // row-wise form

// LDS of a workgroup: a wavefront's sums of up to maxg rank groups, or its 16 x 256 tile in the row-wise form.  By the wavefronts there
// are: room for 16 of them where a launch has one to eight leaves two workgroups to a compute unit (ranks above 64; 24734 x 224
// x 144 rank 144 65 us a call, 53 like this).
static_assert(4 * 64 * 16 <= 8192 && kPrepWaves * 4 * 64 * 16 <= 64 * 1024, "the sums fit the tiles, and the default limit");
constexpr int prep_lds_bytes(int nwaves, int maxg, bool rowwise) { return nwaves * (rowwise ? 8192 : maxg * 64 * 16); }

// CELLS: the activations are stored for the streaming kernel, as 16-byte cells (8 consecutive K
// elements) ordered [K / 8][token row]; otherwise row-major for the tiled kernel.
// SRC: where the activations come from: 0 = fp32 X (quantized here), 1 = MXINT codes and exponent bytes,
// 2 = the bf16 matrix an earlier launch on the same X left in the workspace (nothing is stored again: only T
// is computed, for another layer applied to the same activations).
template <int CTRL>
__device__ __forceinline__ float dpp_quad(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// SIX: the activations are stored as fp6 operands (layout in lqer_internal.h) instead of bf16, and read back so by SRC 2.
template <int SRC, bool FINAL, int MAXG, bool CELLS, bool RW = false, bool SIX = false>
__device__ __forceinline__ void prep_body(const PrepArgs& a) {
    static_assert(!RW || (SRC == 0 && !CELLS && !SIX), "the row-wise form reads fp32 rows and writes row-major bf16");
    static_assert(!SIX || !CELLS, "the streaming kernel takes no fp6 operands");
    // ROWWISE (fp32 X in, row-major bf16 out: the prefill case, bound by HBM): a wavefront reads and writes whole rows
    // of its 16 x 256 tile - 1 KiB per load, 512 B per store, every cache line touched by one instruction - with the
    // four lanes of a quad sharing a block, and turns the tile into the MFMA operand order (lane = token, 16-byte
    // runs of one block) through 8 KB of LDS of its own; the sums of T go through the same memory afterwards.
    // Chosen by the launcher for launches of many workgroups; with few (prefill calls of a few thousand tokens, where K
    // is split over workgroups) the longer chain load - quantize - LDS - MFMA per tile and the two workgroups per
    // compute unit cost more than the coalescing gains (measured: 8192 wide, 4096 tokens 46 -> 52 us; 65536 tokens of
    // 4096 channels 373 -> 308 us), and the lane-per-block form below is used.
    constexpr bool ROWWISE = RW;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];    // prep_lds_bytes of it
    float (*red)[MAXG][64][4] = reinterpret_cast<float (*)[MAXG][64][4]>(smem);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = a.nwaves, nthreads = 64 * nwaves;
    const int t = lane & 15, q = lane >> 4;
    const int64_t row = (int64_t)blockIdx.x * 16 + t;
    const bool row_ok = row < a.M;
    const int slice = blockIdx.y;
    const int g0 = a.g_first + blockIdx.z * a.groups_per_wg;
    const int ng = (a.kp16 - g0 < a.groups_per_wg) ? a.kp16 - g0 : a.groups_per_wg;   // rank groups of this plane
    const bool store_x = (blockIdx.z == 0) && SRC != 2;
    const int64_t nblk = a.K / 16;

    f32x4 acc[MAXG];
#pragma unroll
    for (int g = 0; g < MAXG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (a.flags != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        for (int i = threadIdx.x; i < a.nflags; i += nthreads) a.flags[i] = 0u;

    // Workgroups behind the a.nslices K slices (grid.y) only clear Y for a main kernel that adds into it,
    // so the clearing runs beside the projection instead of in front of it.
    if ((int)blockIdx.y >= a.nslices) {
        if (blockIdx.z != 0) return;                 // one plane of grid.z clears
        const int64_t n4 = (a.N + 3) / 4;
        const int64_t all = (int64_t)gridDim.x * (gridDim.y - a.nslices) * nthreads;
        const int64_t me = ((int64_t)(blockIdx.y - a.nslices) * gridDim.x + blockIdx.x) * nthreads + threadIdx.x;
        for (int64_t i = me; i < a.M * n4; i += all) {
            const int64_t r = i / n4, c = 4 * (i - r * n4);
            float* dst = a.Yz + r * a.ldy + c;
            if (c + 3 < a.N) {
                *reinterpret_cast<f32x4*>(dst) = f32x4{0.f, 0.f, 0.f, 0.f};
            } else {
                for (int64_t j = c; j < a.N; ++j) a.Yz[r * a.ldy + j] = 0.f;
            }
        }
        return;
    }

    const int64_t tile_begin = (int64_t)slice * a.tiles_per_slice;
    int64_t tile_end = tile_begin + a.tiles_per_slice;
    if (tile_end > a.KT) tile_end = a.KT;

    if constexpr (ROWWISE) {
        for (int64_t tile = tile_begin + wave; tile < tile_end; tile += nwaves) {
            Frag xf[4][2];                                   // [p][half]
            uint8_t* tl = smem + wave * 8192;                 // [16 rows][32 cells of 16 B], cell index XOR row
            const int64_t col = tile * kTileK + 4 * lane;     // this lane's four columns (K is a multiple of 16: all in or all out)
            const bool col_ok = col < a.K;
            // four batches of four rows: the next batch's loads are on their way while one is quantized.  Rows past M
            // repeat the last one (their stores are skipped); columns past K are zeroed after the load.
            const int64_t row0 = (int64_t)blockIdx.x * 16;
            const int64_t last = a.M - 1 - row0;              // >= 0: the grid covers M
            const int64_t ccol = col_ok ? col : 0;
            const float* xsrc = a.X + row0 * a.ldx + ccol;
            uint16_t* xdst = a.Xh + row0 * a.ldxh + col;
            const float keep = col_ok ? 1.0f : 0.0f;
            auto load_rows = [&](f32x4 (&v)[4], int i0) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t r = (i0 + i) <= last ? (i0 + i) : last;
                    v[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(xsrc + r * a.ldx));
                }
            };
            const float lim = (float)((2 << a.act_frac) - 1);
            auto quantize_rows = [&](const f32x4 (&v)[4], int i0) {
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
                    const int i = i0 + ii;
                    const f32x4 x = v[ii] * keep;
                    float m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(x[0]), __builtin_fabsf(x[1])),
                                              __builtin_fmaxf(__builtin_fabsf(x[2]), __builtin_fabsf(x[3])));
                    m = __builtin_fmaxf(m, dpp_quad<0xB1>(m));    // quad_perm [1,0,3,2]
                    m = __builtin_fmaxf(m, dpp_quad<0x4E>(m));    // quad_perm [2,3,0,1]
                    const uint32_t eb = (f32_bits(m) >> 23) & 0xFFu;
                    const int sh = a.act_frac - ((int)eb - 127);
                    const float scale = x_scale(eb, a.act_frac);
                    float c[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float r = __builtin_rintf(__builtin_amdgcn_ldexpf(x[j], sh));
                        c[j] = __builtin_fminf(__builtin_fmaxf(r, -lim), lim) * scale;
                    }
                    const u32x2 w = u32x2{pack_bf16_exact(c[0], c[1]), pack_bf16_exact(c[2], c[3])};
                    // columns between K and the end of the last tile are written as zeros: the main kernel reads whole tiles
                    if (store_x && i <= last) *reinterpret_cast<u32x2*>(xdst + i * a.ldxh) = w;
                    *reinterpret_cast<u32x2*>(tl + i * 512 + (((lane >> 1) ^ i) << 4) + (lane & 1) * 8) = w;
                }
            };
            f32x4 va[4], vb[4];
            load_rows(va, 0);
            load_rows(vb, 4);
            __builtin_amdgcn_wave_barrier();                  // the previous tile's operand reads are issued before these writes
            quantize_rows(va, 0);
            load_rows(va, 8);
            quantize_rows(vb, 4);
            load_rows(vb, 12);
            quantize_rows(va, 8);
            quantize_rows(vb, 12);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    xf[p][h].u = *reinterpret_cast<const u32x4*>(tl + t * 512 + (((2 * (q + 4 * p) + h) ^ t) << 4));
#pragma unroll
            for (int g = 0; g < MAXG; ++g) {
                if (g < ng) {
                    const uint8_t* rec = a.At + ((int64_t)(g0 + g) * a.KT + tile) * kARecordBytes;
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        Frag af[2];
                        af[0].u = *reinterpret_cast<const u32x4*>(rec + (2 * p) * 1024 + lane * 16);
                        af[1].u = *reinterpret_cast<const u32x4*>(rec + (2 * p + 1) * 1024 + lane * 16);
                        acc[g] = mfma16(af[0].v, xf[p][0].v, acc[g]);
                        acc[g] = mfma16(af[1].v, xf[p][1].v, acc[g]);
                    }
                    // one rank group's eight loads in flight at a time: all of them at once cost the registers of a second workgroup
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    } else {
        // The unit of work is a quarter of a tile (64 columns, one block per lane), so that a wavefront's chain is one round trip
        // to memory and 16 values' arithmetic; the next unit's operands are asked for ahead of it.  No load is conditional: a
        // branch around it would have the compiler wait for it at the branch's end.
        struct Unit {
            u32x4 x[SRC == 0 ? 4 : (SRC == 2 ? 2 : 1)];     // the block: fp32, codes, or bf16
            uint32_t eb;
            Frag af[CELLS ? MAXG : 1][2];
        };
        const int64_t rowc = row_ok ? row : a.M - 1;
        const float* xrow = a.X + rowc * a.ldx;
        const int8_t* crow = a.Xc + rowc * a.K;
        const uint8_t* erow = a.Xe + rowc * nblk;
        const uint16_t* hrow = a.Xh + rowc * a.ldxh;
        const uint8_t* alane = a.At + lane * 16;
        const int units = (int)(tile_end - tile_begin) * 4;
        // fp6 images: this lane's row in one, the image of a unit, the byte of its block's exponent
        const int64_t six_rt = rowc / kX6Rows;
        const int six_lane = (int)(rowc % kX6Rows / 32) * 64 + (q >> 1) * 32 + (int)(rowc % 32);     // row group, hh, row
        const int six_cell = (q & 1) * 256 + six_lane;
        auto six_image = [&](int unit) {
            return reinterpret_cast<uint8_t*>(a.Xh) + ((six_rt * a.KT + tile_begin) * 4 + unit) * kX6Chunk;
        };
        auto six_exp = [&](int unit) {
            return a.Xe6 + (six_rt * a.KT + tile_begin + (unit >> 2)) * kX6Scales + six_lane * 8 + 2 * (unit & 3) + (q & 1);
        };
        auto load_a = [&](Frag (&af)[2], int g, int unit) {
            const int gc = g < ng ? g : 0;
            const uint8_t* rec = alane + ((int64_t)(g0 + gc) * a.KT + tile_begin + (unit >> 2)) * kARecordBytes + (unit & 3) * 2048;
            af[0].u = *reinterpret_cast<const u32x4*>(rec);
            af[1].u = *reinterpret_cast<const u32x4*>(rec + 1024);
        };
        auto load_unit = [&](Unit& u, int unit) {
            const int64_t kb = (tile_begin + (unit >> 2)) * 16 + q + 4 * (unit & 3);
            const int64_t kbc = kb < nblk ? kb : nblk - 1;
            if constexpr (CELLS) {
                if (a.kp > 0) {                              // (the same for the whole launch)
#pragma unroll
                    for (int g = 0; g < MAXG; ++g) load_a(u.af[g], g, unit);
                }
            }
            if constexpr (SRC == 2 && SIX) {
                const uint8_t* img = six_image(unit);
                u.x[0] = *reinterpret_cast<const u32x4*>(img + six_cell * 16);
                const u32x2 w = *reinterpret_cast<const u32x2*>(img + 8192 + six_cell * 8);
                u.x[1] = u32x4{w[0], w[1], 0u, 0u};
                u.eb = *six_exp(unit);
            } else if constexpr (SRC == 2) {
                static_assert(SRC != 2 || !CELLS, "the stored matrix is read back in its row-major form only");
                u.x[0] = *reinterpret_cast<const u32x4*>(hrow + kbc * 16);
                u.x[1] = *reinterpret_cast<const u32x4*>(hrow + kbc * 16 + 8);
            } else if constexpr (SRC == 1) {
                u.x[0] = *reinterpret_cast<const u32x4*>(crow + kbc * 16);
                u.eb = erow[kbc];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) u.x[i] = *reinterpret_cast<const u32x4*>(xrow + kbc * 16 + 4 * i);
            }
        };
        // Where fp32 input takes the row-wise form, a wavefront takes its tiles' four quarters one after the other here too: T is then
        // added up in the same order whatever the activations come from.  (Elsewhere quarters in turn are the faster: 4-bit layers
        // on codes, 8192 tokens, 4096 wide 39.7 us a call, 42.0 by tiles.)
        auto next_unit = [&](int unit) { return a.by_tiles ? unit + ((unit & 3) == 3 ? 4 * nwaves - 3 : 1) : unit + nwaves; };
        // more: the wavefront has another unit behind this one.  (Two instances: where loads may or may not follow, the compiler
        // waits for all of them.)
        auto process = [&](Unit& cur, Unit& nxt, int unit, auto more) {
            Frag af[MAXG][2];
            if constexpr (CELLS) {
#pragma unroll
                for (int g = 0; g < MAXG; ++g) {
                    af[g][0] = cur.af[g][0];
                    af[g][1] = cur.af[g][1];
                }
            } else if (!SIX && a.kp > 0) {
#pragma unroll
                for (int g = 0; g < MAXG; ++g) load_a(af[g], g, unit);
            }
            if constexpr (decltype(more)::value) load_unit(nxt, next_unit(unit));
            __builtin_amdgcn_sched_barrier(0);
            const int64_t blk = (tile_begin + (unit >> 2)) * 16 + q + 4 * (unit & 3);   // block index along K
            const bool ok = row_ok && blk < nblk;
            Frag xf[2];
            float scale = 0.f;
            float r[16];
            u32x4 cw = u32x4{0, 0, 0, 0};                    // the block's 16 codes as bytes (SRC 1, or CELLS of 16+ rows)
            uint32_t eb = 0;
            if constexpr (SRC == 2 && SIX) {
                const u32x6 v = {cur.x[0][0], cur.x[0][1], cur.x[0][2], cur.x[0][3], cur.x[1][0], cur.x[1][1]};
                six_to_values(v, x_scale(cur.eb, 6), r);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) xf[h].u[i] = ok ? pack_bf16_exact(r[8 * h + 2 * i], r[8 * h + 2 * i + 1]) : 0u;
            } else if constexpr (SRC == 2) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) xf[h].u[i] = ok ? cur.x[h][i] : 0u;
            } else if constexpr (SRC == 1) {
#pragma unroll
                for (int i = 0; i < 4; ++i) cw[i] = ok ? cur.x[0][i] : 0u;
                eb = ok ? cur.eb : 0u;
                scale = x_scale(eb, a.act_frac);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = cw[i];
                    r[4 * i + 0] = (float)(int)(int8_t)(w & 0xFF);
                    r[4 * i + 1] = (float)(int)(int8_t)((w >> 8) & 0xFF);
                    r[4 * i + 2] = (float)(int)(int8_t)((w >> 16) & 0xFF);
                    r[4 * i + 3] = (float)(int)(int8_t)(w >> 24);
                }
            } else {
                float v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = ok ? f32_from_bits(cur.x[i >> 2][i & 3]) : 0.f;
                float m = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i += 4)
                    m = __builtin_fmaxf(m, __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[i]), __builtin_fabsf(v[i + 1])),
                                                           __builtin_fmaxf(__builtin_fabsf(v[i + 2]), __builtin_fabsf(v[i + 3]))));
                eb = (f32_bits(m) >> 23) & 0xFFu;
                const int sh = a.act_frac - ((int)eb - 127);
                const float lim = (float)((2 << a.act_frac) - 1);             // 127 or 31
                scale = x_scale(eb, a.act_frac);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float c = __builtin_rintf(__builtin_amdgcn_ldexpf(v[i], sh));
                    r[i] = __builtin_fminf(__builtin_fmaxf(c, -lim), lim);
                }
                if constexpr (CELLS) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        cw[i] = ((uint32_t)(int)r[4 * i] & 0xFFu) | (((uint32_t)(int)r[4 * i + 1] & 0xFFu) << 8) |
                                (((uint32_t)(int)r[4 * i + 2] & 0xFFu) << 16) | ((uint32_t)(int)r[4 * i + 3] << 24);
                }
            }
            if constexpr (SRC != 2) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        xf[h].u[i] = pack_bf16_exact(r[8 * h + 2 * i] * scale, r[8 * h + 2 * i + 1] * scale);
            }
            if (store_x && row_ok) {
                if constexpr (SIX) {
                    // The exponent byte is that of 6 fraction bits.  Beyond 254 (a byte of 255 is a NaN to the matrix instruction) the codes
                    // take the rest, and where they cannot, the block's values are infinities in fp32, which T makes NaNs of as well.
                    int e6 = (int)eb + 6 - a.act_frac;
                    float up = 1.0f;
                    if (__builtin_expect(e6 > 254, 0)) {
                        up = f32_from_bits((uint32_t)(e6 - 254 + 127) << 23);
                        float m = 0.f;
#pragma unroll
                        for (int i = 0; i < 16; ++i) m = __builtin_fmaxf(m, __builtin_fabsf(r[i]));
                        e6 = m * up >= 128.0f ? 255 : 254;
                        if (e6 == 255) up = 1.0f;
                    }
                    const u32x6 w = codes_to_six<SRC == 1>(r, up);
                    uint8_t* img = six_image(unit);
                    *reinterpret_cast<u32x4*>(img + six_cell * 16) = u32x4{w[0], w[1], w[2], w[3]};
                    *reinterpret_cast<u32x2*>(img + 8192 + six_cell * 8) = u32x2{w[4], w[5]};
                    *six_exp(unit) = (uint8_t)e6;
                } else if (CELLS) {
                    if (a.x8) {
                        // 16 token rows and more: MXINT8 as it is, 16 code bytes per (block, row), and the
                        // exponent bytes [block][row] behind all codes; the main kernel converts
                        uint8_t* base = reinterpret_cast<uint8_t*>(a.Xh);
                        const int64_t entry = (blk << a.lr) + row;
                        *reinterpret_cast<u32x4*>(base + entry * 16) = cw;
                        // the main kernel scales codes by 2^(byte - 127 - 6): narrower codes carry the difference in the byte
                        const uint32_t ebs = eb + (6 - a.act_frac);
                        base[((a.KT * 16) << (a.lr + 4)) + entry] = (uint8_t)(ebs < 254u ? ebs : 254u);
                    } else {
                        uint16_t* dst = a.Xh + ((((blk * 2) << a.lr) + row) << 3);
                        *reinterpret_cast<u32x4*>(dst) = xf[0].u;
                        *reinterpret_cast<u32x4*>(dst + (8 << a.lr)) = xf[1].u;
                    }
                } else {
                    uint16_t* dst = a.Xh + row * a.ldxh + blk * 16;
                    *reinterpret_cast<u32x4*>(dst) = xf[0].u;
                    *reinterpret_cast<u32x4*>(dst + 8) = xf[1].u;
                }
            }
            if constexpr (SIX) {
                // (large calls, whose other wavefronts cover these loads; in front they would take the conversion's registers)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int g = 0; g < MAXG; ++g) load_a(af[g], g, unit);
            }
            if (a.kp > 0) {
#pragma unroll
                for (int g = 0; g < MAXG; ++g) {
                    acc[g] = mfma16(af[g][0].v, xf[0].v, acc[g]);
                    acc[g] = mfma16(af[g][1].v, xf[1].v, acc[g]);
                }
            }
        };
        Unit cur, nxt;
        int unit = a.by_tiles ? 4 * wave : wave;
        if (unit < units) {
            load_unit(cur, unit);
            for (; next_unit(unit) < units; unit = next_unit(unit)) {
                process(cur, nxt, unit, std::true_type{});
                cur = nxt;
            }
            process(cur, nxt, unit, std::false_type{});
        }
    }

    if (a.kp == 0) {
        // no low-rank branch: only the zero padding behind K_pad (none) remains
        return;
    }

    // add the wavefronts' partial T in a fixed order
    if constexpr (ROWWISE) __syncthreads();          // the sums reuse the tiles' memory: every wavefront is done with its tile
#pragma unroll
    for (int g = 0; g < MAXG; ++g)
        *reinterpret_cast<f32x4*>(&red[wave][g][lane][0]) = acc[g];
    __syncthreads();
    for (int item = threadIdx.x; item < ng * 64; item += nthreads) {
        const int g = item >> 6, l = item & 63;
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[0][g][l][0]);
        for (int w = 1; w < nwaves; ++w) {
            const f32x4 o = *reinterpret_cast<const f32x4*>(&red[w][g][l][0]);
            s[0] += o[0]; s[1] += o[1]; s[2] += o[2]; s[3] += o[3];
        }
        const int64_t orow = (int64_t)blockIdx.x * 16 + (l & 15);
        const int r0 = (g0 + g) * 16 + 4 * (l >> 4);          // first of this lane's 4 ranks
        if (orow < a.M) {
            if (FINAL) {
                uint16_t hi[4], lo[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) split_bf16(s[j], hi[j], lo[j]);
                uint16_t* base = a.Xt + orow * a.ldxt;
                *reinterpret_cast<u32x2*>(base + r0) =
                    u32x2{(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
                *reinterpret_cast<u32x2*>(base + a.kp + r0) =
                    u32x2{(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
            } else {
                *reinterpret_cast<f32x4*>(a.Tpart + ((int64_t)slice * a.tp_rows + orow) * a.kp + r0) = s;
            }
        }
    }
    // zero the padding behind T_hi | T_lo so the main kernel can read whole 64-column chunks
    if (FINAL && blockIdx.z == 0) {
        const int pad = (int)(a.tail_cols - 2 * a.kp);
        for (int item = threadIdx.x; item < 16 * pad; item += nthreads) {
            const int64_t orow = (int64_t)blockIdx.x * 16 + item / pad;
            if (orow < a.M) a.Xt[orow * a.ldxt + 2 * a.kp + item % pad] = 0;
        }
    }
}

template <int SRC, bool FINAL, int MAXG, bool CELLS, bool RW = false, bool SIX = false>
__global__ __launch_bounds__(64 * (RW ? kPrepRowWaves : kPrepWaves), RW ? 4 : 1) void prep_kernel(PrepArgs a) {
    prep_body<SRC, FINAL, MAXG, CELLS, RW, SIX>(a);
}

// Rank groups beyond the first four (ranks above 64) on the tiled path, large calls (launch_prep says which): T = X_q A_k from the activations the launch above has stored.
// Bound by A_k's way from L2, 2 KiB per 64 of K and rank group: with 16 rows a workgroup, four groups at a time, that was 256 MB at rank
// 256, 4096 wide and 2048 tokens.  Here a wavefront has 16 R rows and GRP groups, all operands of the next 64 of K in flight while it
// multiplies these; the workgroup's eight split its K slice in turn and add up through LDS, in wavefront order, 16 rows at a time.
constexpr int kProjectWaves = 8;
template <bool SIX, int R, int GRP>
__global__ __launch_bounds__(64 * kProjectWaves, 2) void project_kernel(PrepArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = lane & 15, q = lane >> 4;
    const int slice = blockIdx.y, g0 = a.g_first + blockIdx.z * a.groups_per_wg;
    const int ng = a.kp16 - g0 < a.groups_per_wg ? a.kp16 - g0 : a.groups_per_wg;
    const int64_t row0 = (int64_t)blockIdx.x * (16 * R);
    const int64_t tile_begin = (int64_t)slice * a.tiles_per_slice;
    const int64_t tiles = a.KT - tile_begin < a.tiles_per_slice ? a.KT - tile_begin : a.tiles_per_slice;
    const int units = tiles > 0 ? (int)tiles * 4 : 0;          // 64 of K each; a lane owns block q of a row

    struct XRaw { u32x4 p; u32x4 h; uint32_t e; };             // fp6: six words and the exponent; bf16: the 16 values
    struct Set { XRaw x[R]; Frag a[GRP][2]; };
    // (Rows past M are workspace rows; their sums are not stored.)
    auto load_x = [&](XRaw (&x)[R], int unit) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t row = row0 + 16 * r + t;
            if constexpr (SIX) {
                const int six_lane = (int)(row % kX6Rows / 32) * 64 + (q >> 1) * 32 + (int)(row % 32), six_cell = (q & 1) * 256 + six_lane;
                const int64_t tile = row / kX6Rows * a.KT + tile_begin + (unit >> 2);
                const uint8_t* img = reinterpret_cast<const uint8_t*>(a.Xh) + (tile * 4 + (unit & 3)) * kX6Chunk;
                x[r].p = *reinterpret_cast<const u32x4*>(img + six_cell * 16);
                const u32x2 w = *reinterpret_cast<const u32x2*>(img + 8192 + six_cell * 8);
                x[r].h = u32x4{w[0], w[1], 0u, 0u};
                x[r].e = a.Xe6[tile * kX6Scales + six_lane * 8 + 2 * (unit & 3) + (q & 1)];
            } else {
                const uint16_t* src = a.Xh + row * a.ldxh + (tile_begin * 16 + 4 * unit + q) * 16;
                x[r].p = *reinterpret_cast<const u32x4*>(src);
                x[r].h = *reinterpret_cast<const u32x4*>(src + 8);
            }
        }
    };
    auto load_a = [&](Frag (&f)[2], int g, int unit) {
        const uint8_t* rec = a.At + ((int64_t)(g0 + (g < ng ? g : 0)) * a.KT + tile_begin + (unit >> 2)) * kARecordBytes + (unit & 3) * 2048 + lane * 16;
        f[0].u = *reinterpret_cast<const u32x4*>(rec);
        f[1].u = *reinterpret_cast<const u32x4*>(rec + 1024);
    };
    f32x4 acc[R][GRP];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int g = 0; g < GRP; ++g) acc[r][g] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave < units) {
        XRaw x[R];
        Frag af[GRP][2];
        load_x(x, wave);
#pragma unroll
        for (int g = 0; g < GRP; ++g) load_a(af[g], g, wave);
        for (int unit = wave; unit < units; unit += kProjectWaves) {
            const int next = unit + kProjectWaves < units ? unit + kProjectWaves : unit;       // (the last one's once more: no branch)
            Frag xf[R][2];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (SIX) {
                    float v[16];
                    six_to_values(u32x6{x[r].p[0], x[r].p[1], x[r].p[2], x[r].p[3], x[r].h[0], x[r].h[1]}, x_scale(x[r].e, 6), v);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) xf[r][h].u[i] = pack_bf16_exact(v[8 * h + 2 * i], v[8 * h + 2 * i + 1]);
                } else {
                    xf[r][0].u = x[r].p;
                    xf[r][1].u = x[r].h;
                }
            }
            load_x(x, next);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < GRP; ++g) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r][g] = mfma16(af[g][h].v, xf[r][h].v, acc[r][g]);
                load_a(af[g], g, next);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    f32x4* const red = reinterpret_cast<f32x4*>(smem);         // [wave][GRP][64]
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r > 0) __syncthreads();
#pragma unroll
        for (int g = 0; g < GRP; ++g) red[(wave * GRP + g) * 64 + lane] = acc[r][g];
        __syncthreads();
        for (int item = threadIdx.x; item < GRP * 64; item += 64 * kProjectWaves) {
            const int l = item & 63, g = item >> 6;
            const int64_t orow = row0 + 16 * r + (l & 15);
            if (g >= ng || orow >= a.M) continue;
            f32x4 s = red[item];
#pragma unroll
            for (int w = 1; w < kProjectWaves; ++w) s += red[w * GRP * 64 + item];
            const int r0 = (g0 + g) * 16 + 4 * (l >> 4);
            if (a.Tpart == nullptr) {
                uint16_t hi[4], lo[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) split_bf16(s[j], hi[j], lo[j]);
                uint16_t* base = a.Xt + orow * a.ldxt;
                *reinterpret_cast<u32x2*>(base + r0) = u32x2{(uint32_t)hi[0] | ((uint32_t)hi[1] << 16), (uint32_t)hi[2] | ((uint32_t)hi[3] << 16)};
                *reinterpret_cast<u32x2*>(base + a.kp + r0) = u32x2{(uint32_t)lo[0] | ((uint32_t)lo[1] << 16), (uint32_t)lo[2] | ((uint32_t)lo[3] << 16)};
            } else {
                *reinterpret_cast<f32x4*>(a.Tpart + ((int64_t)slice * a.tp_rows + orow) * a.kp + r0) = s;
            }
        }
    }
}

template <bool SIX, int R>
static void launch_project_t(dim3 grid, hipStream_t s, const PrepArgs& a) {
    const dim3 block(64 * kProjectWaves);
    if (a.groups_per_wg <= 4) hipLaunchKernelGGL((project_kernel<SIX, R, 4>), grid, block, kProjectWaves * 4 * 1024, s, a);
    else hipLaunchKernelGGL((project_kernel<SIX, R, 6>), grid, block, kProjectWaves * 6 * 1024, s, a);
}

// Rank groups 4 and on.  64 rows a wavefront where that leaves a workgroup for every compute unit, else 32.
static hipError_t launch_project(PrepArgs a, int S, bool six, hipStream_t s) {
    const int rest = a.kp16 - 4, planes = (rest + 5) / 6;
    a.g_first = 4;
    a.groups_per_wg = (rest + planes - 1) / planes;
    const int64_t tall = (a.M + 63) / 64;
    const bool four = tall * S * planes >= 256;
    const dim3 grid((unsigned)(four ? tall : (a.M + 31) / 32), (unsigned)S, (unsigned)planes);
    if (six) four ? launch_project_t<true, 4>(grid, s, a) : launch_project_t<true, 2>(grid, s, a);
    else four ? launch_project_t<false, 4>(grid, s, a) : launch_project_t<false, 2>(grid, s, a);
    return hipGetLastError();
}

// Several layers applied to the same few tokens: grid.z holds the rank groups of all of them (the first plane stores the
// activations), workgroups behind the K slices clear whichever Y a main kernel adds into.
struct PrepLayer { const uint8_t* At; float* Tpart; float* Yz; int64_t ldy, N; int kp, kp16, z0; };
struct PrepGroup { PrepArgs a; int n; PrepLayer layer[kGroupLayers]; };

__global__ __launch_bounds__(64 * kPrepWaves) void prep_group_kernel(PrepGroup g) {
    if ((int)blockIdx.y >= g.a.nslices) {
        if (blockIdx.z != 0) return;
        const int64_t nthreads = (int64_t)gridDim.x * (gridDim.y - g.a.nslices) * 64 * g.a.nwaves;
        const int64_t me = ((int64_t)(blockIdx.y - g.a.nslices) * gridDim.x + blockIdx.x) * 64 * g.a.nwaves + threadIdx.x;
        for (int li = 0; li < g.n; ++li) {
            const PrepLayer& L = g.layer[li];
            const int64_t n4 = (L.N + 3) / 4;
            for (int64_t i = me; i < g.a.M * n4; i += nthreads) {
                const int64_t r = i / n4, c = 4 * (i - r * n4);
                if (c + 3 < L.N) {
                    *reinterpret_cast<f32x4*>(L.Yz + r * L.ldy + c) = f32x4{0.f, 0.f, 0.f, 0.f};
                } else {
                    for (int64_t j = c; j < L.N; ++j) L.Yz[r * L.ldy + j] = 0.f;
                }
            }
        }
        return;
    }
    int li = 0;
    while (li + 1 < g.n && (int)blockIdx.z >= g.layer[li + 1].z0) ++li;
    const PrepLayer& L = g.layer[li];
    PrepArgs a = g.a;
    a.At = L.At; a.Tpart = L.Tpart; a.kp = L.kp; a.kp16 = L.kp16;
    a.g_first = -L.z0;
    prep_body<0, false, 1, true>(a);
}

template <int SRC, bool FINAL, int MAXG, bool CELLS>
static void launch_prep_t(dim3 grid, dim3 block, hipStream_t s, const PrepArgs& a, bool rowwise, bool six) {
    if constexpr (!CELLS) {
        if (six) {
            hipLaunchKernelGGL((prep_kernel<SRC, FINAL, MAXG, CELLS, false, true>), grid, block, prep_lds_bytes(a.nwaves, MAXG, false), s, a);
            return;
        }
    }
    if constexpr (SRC == 0 && !CELLS) {
        if (rowwise) {
            hipLaunchKernelGGL((prep_kernel<SRC, FINAL, MAXG, CELLS, true>), grid, block, prep_lds_bytes(a.nwaves, MAXG, true), s, a);
            return;
        }
    }
    hipLaunchKernelGGL((prep_kernel<SRC, FINAL, MAXG, CELLS, false>), grid, block, prep_lds_bytes(a.nwaves, MAXG, false), s, a);
}

int prep_slices(const Layer& L, int64_t M, int path, bool least) {
    if (path != 1) {
        // tiled path: one workgroup per 16 token rows; when that leaves compute units idle, split K as well (each slice keeps at least
        // two tiles) and let the main kernel add the partial T.  Either one workgroup of up to 16 wavefronts to a compute unit, where they
        // are at least three quarters of a round; or 384 of eight and more, two to a unit and so three quarters of one as well, if that
        // leaves a slice three tiles: more partial sums cost the main kernel as much whatever K (5072 tokens of 1088 x 6432 rank 16 in two
        // slices 101.6 us, 97.6 in one).
        // 5700 calls of 700 to 9000 tokens, projection and main product: 1.6 % from the best of all slices and wavefront counts on average;
        // the first form wherever it fills 256 units once or more, however empty its last round, 3.3 % (4133 tokens of 10704 x 822 rank
        // 32 152 us, 127 by this), always 512 of the second 2.6 %, with a line at 512 instead of 384 (7823 tokens of 976 x 4707 rank 256
        // 186 us, 160) 1.7 %.
        const int64_t rg = (M + 15) / 16;
        int64_t s = 1;
        auto more = [&] { return s < 8 && L.KT / (2 * s) >= 2; };
        while (2 * rg * s <= 256 && more()) s *= 2;
        if (rg * s >= 192 && rg * s <= 256) return (int)s;
        while (rg * s < 192 && more()) s *= 2;
        while (!least && rg * s < 384 && more() && L.KT >= 6 * s) s *= 2;
        return (int)s;
    }
    // streaming path: at most two row groups, so K is spread over workgroups (the main kernel adds
    // up to 8 partial sums); one wavefront per K tile of a slice, at most kPrepWaves.
    int64_t s = L.KT;
    if (s > 8) s = 8;
    if (s < 1) s = 1;
    return (int)s;
}

// Wavefronts of a workgroup: one per tile of the slice where the launch's workgroups (`wgs`: row blocks x slices) fill the chip anyway,
// eight of two workgroups to a compute unit, or up to 16 where there is exactly one for each; otherwise one per quarter of a tile in
// as few and as even rounds as fit.  Which quarters a wavefront adds up before the wavefronts' sums meet decides the bits of T, so that
// goes by token rows and slices alone: not by the planes of rank groups, which differ between a layer's own call and one that finds its
// activations stored.
static int prep_waves(int tiles, int64_t wgs) {
    if (wgs >= 256) {
        const int most = wgs > 256 ? kPrepRowWaves : kPrepWaves;
        return tiles < most ? (tiles < 1 ? 1 : tiles) : most;
    }
    const int units = 4 * tiles;
    if (units <= kPrepWaves) return units < 1 ? 1 : units;
    const int rounds = (units + kPrepWaves - 1) / kPrepWaves;
    return (units + rounds - 1) / rounds;
}

hipError_t launch_prep(const Layer& L, const float* X, int64_t ldx, const int8_t* Xc, const uint8_t* Xe,
                       int64_t M, const Workspace& ws, float* y_zero, int64_t ldy, hipStream_t s, bool reuse_xh) {
    if (M == 0) return hipSuccess;
    if (reuse_xh && (ws.cells || X != nullptr || Xc != nullptr)) return hipErrorInvalidValue;
    PrepArgs a;
    a.X = X; a.ldx = ldx; a.Xc = Xc; a.Xe = Xe;
    a.M = M; a.K = L.K; a.KT = L.KT;
    a.tiles_per_slice = (int)((L.KT + ws.S - 1) / ws.S);
    a.kp = L.kp; a.kp16 = L.kp16;
    a.groups_per_wg = L.kp16;
    // Few-token calls are bound by the latency of reading A_k (1 MB for K = 8192, kp = 64) with a handful of
    // workgroups: there every rank group gets workgroups of its own (grid.z), each quantizing the few
    // rows again; 1 us less on the 70B-shaped layer.
    int gz = 1;
    if (ws.cells && L.kp16 > 1) { gz = L.kp16; a.groups_per_wg = 1; }
    // More than four rank groups (ranks above 64) on the tiled path: this launch does the first four, a second one the others from
    // the activations this one stores (or an earlier one has; half the bytes, nothing to quantize): project_kernel, or this kernel in planes of
    // four groups.  The line is where A_k's way from L2, a quarter or half of it here, outweighs what the other kernel takes longer to start
    // and end, 2.3 us (138 random calls of ranks 128 and 256): whole calls, 4096 x 4096 rank 256 at 2048 tokens 87 -> 81 us, 0.92 of
    // the time on average from 4096 tokens and K on; below the line up to 1.13 of it.
    const bool two_launches = !ws.cells && L.kp16 > 4;
    const bool project = a.tiles_per_slice >= 4 && (double)M * (double)L.K * (double)(L.kp - 64) > 1.3e9;
    if (two_launches) {
        a.groups_per_wg = 4;
        if (reuse_xh && !project) gz = (L.kp16 + 3) / 4;
    }
    a.g_first = 0;
    a.At = L.At; a.Xh = ws.Xh; a.ldxh = ws.ldxh;
    a.Xt = ws.Xt; a.ldxt = ws.ldxt;
    a.tail_cols = ws.ldxh - L.KT * kTileK;
    a.Xe6 = ws.six ? six_scales(ws, L) : nullptr;
    a.Tpart = ws.Tpart;
    a.tp_rows = ws.tp_rows;
    a.lr = ws.lr;
    a.x8 = ws.x8;
    a.act_frac = L.act_bits - 2;
    a.Yz = y_zero; a.ldy = ldy; a.N = L.N;
    a.nslices = ws.S;
    a.flags = ws.flags; a.nflags = ws.flags ? kTiledFlags : 0;
    const bool cells = ws.cells;
    const int src = reuse_xh ? 2 : (Xc != nullptr ? 1 : 0);
    const int64_t rg = (M + 15) / 16;
    // the row-wise form for fp32 input in row-major layout when the launch has workgroups to spare
    a.by_tiles = !cells && !ws.six && rg * ws.S >= 2048;
    const bool rowwise = a.by_tiles && src == 0;
    a.nwaves = prep_waves(a.tiles_per_slice, cells ? 0 : rg * ws.S);
    dim3 block(64 * a.nwaves);
    // clearing workgroups: about four 16-byte stores per thread
    const int64_t zero_wgs = y_zero ? (M * ((L.N + 3) / 4) + 4 * block.x * rg - 1) / (4 * block.x * rg) : 0;
    dim3 grid((unsigned)rg, (unsigned)(ws.S + zero_wgs), (unsigned)gz);
    const bool fin = (ws.Tpart == nullptr);          // T final (hi/lo behind the row) or partial sums
    if (cells && fin && L.kp > 0) return hipErrorInvalidValue;
    if (a.groups_per_wg > 4) return hipErrorInvalidValue;
#define LQER_PREP(FC, FN, MG, CL) launch_prep_t<FC, FN, MG, CL>(grid, block, s, a, rowwise, ws.six)
#define LQER_PREP_G(FC, FN) do { if (a.groups_per_wg <= 1) LQER_PREP(FC, FN, 1, false); else if (a.groups_per_wg == 2) LQER_PREP(FC, FN, 2, false); else LQER_PREP(FC, FN, 4, false); } while (0)
#define LQER_PREP_C(FN) do { if (src == 1) LQER_PREP_G(1, FN); else LQER_PREP_G(0, FN); } while (0)
    if (cells) {
        if (src == 1) LQER_PREP(1, false, 1, true);
        else LQER_PREP(0, false, 1, true);
    }
    else if (src == 2) { if (fin) LQER_PREP_G(2, true); else LQER_PREP_G(2, false); }
    else if (fin) LQER_PREP_C(true);
    else LQER_PREP_C(false);
    if (two_launches) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (project) return launch_project(a, ws.S, ws.six, s);
        if (!reuse_xh) {
            a.g_first = 4;
            grid.z = (unsigned)((L.kp16 - 4 + 3) / 4);
            grid.y = (unsigned)ws.S;
            if (fin) LQER_PREP_G(2, true); else LQER_PREP_G(2, false);
        }
    }
#undef LQER_PREP_C
#undef LQER_PREP_G
#undef LQER_PREP
    return hipGetLastError();
}

// The projection step of launch_stream_group: what launch_prep does for each layer alone, in one launch.
hipError_t launch_prep_group(const Layer* const* layers, int n, const float* X, int64_t ldx, int64_t M, const Workspace& ws,
                             float* const* Tpart, float* const* Y, const int64_t* ldy, bool zero_y, hipStream_t s) {
    if (M == 0) return hipSuccess;
    if (n < 1 || n > kGroupLayers || !ws.cells) return hipErrorInvalidValue;
    const Layer& L0 = *layers[0];
    PrepGroup g{};
    PrepArgs& a = g.a;
    a.X = X; a.ldx = ldx; a.M = M; a.K = L0.K; a.KT = L0.KT;
    a.tiles_per_slice = (int)((L0.KT + ws.S - 1) / ws.S);
    a.groups_per_wg = 1;
    a.Xh = ws.Xh; a.ldxh = ws.ldxh; a.tp_rows = M; a.lr = ws.lr; a.x8 = ws.x8;
    a.act_frac = L0.act_bits - 2;
    a.nslices = ws.S;
    g.n = n;
    int z = 0;
    int64_t cols4 = 0;
    for (int i = 0; i < n; ++i) {
        const Layer& L = *layers[i];
        g.layer[i] = PrepLayer{L.At, Tpart[i], Y[i], ldy[i], L.N, L.kp, L.kp16, z};
        z += L.kp16;
        cols4 += (L.N + 3) / 4;
    }
    a.by_tiles = false;
    a.nwaves = prep_waves(a.tiles_per_slice, 0);
    const dim3 block(64 * a.nwaves);
    const int64_t rg = (M + 15) / 16;
    const int64_t zero_wgs = zero_y ? (M * cols4 + 4 * block.x * rg - 1) / (4 * block.x * rg) : 0;
    hipLaunchKernelGGL(prep_group_kernel, dim3((unsigned)rg, (unsigned)(ws.S + zero_wgs), (unsigned)(z > 0 ? z : 1)), block,
                       prep_lds_bytes(a.nwaves, 1, false), s, g);
    return hipGetLastError();
}

}  // namespace lqer
