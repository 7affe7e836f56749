// Stage 2, large-M ("prefill") form of Y = X_q W_q + T B_k (Eq. 3 / Eq. 6): an MFMA-bound tiled
// GEMM.  Sec. 2.1 observes that run-time dequantization is what costs weight-only schemes in the
// compute-bound regime, so here the weight expansion is kept to seven VALU instructions per 8
// elements (unpack_w8) and runs beside the matrix pipe.
//
// Workgroup tile BM x BN, WR x WC wavefronts, each owning TM x TN tiles of the 32x32x16 bf16
// MFMA (the shape one wavefront per SIMD can keep close to the matrix pipe's peak).  The
// contraction axis is walked in chunks of 64 = four MFMA steps; lane half hh owns blocks 2hh and
// 2hh+1 of a chunk for every operand, so block scales never cross lanes.
//   activations (bf16, exact dequantized X_q, then T_hi | T_lo): global -> registers two or three
//       chunks ahead -> a ring of four LDS stages of XOR-swizzled 16-byte cells -> ds_read_b128
//       operands shared by the wavefronts of a row;
//   weights: each wavefront loads the packed MXINT4 records of its own columns straight into
//       registers (fully coalesced 16-byte loads), three chunks ahead, into four register sets used
//       by name in turn (a copy between sets would force a wait on the newest load), and expands
//       them there;
//   the rank-kp correction is ceil(2 kp / 64) more chunks behind the others whose weight operand comes from B_k.
// MFMA operands are swapped (weights first) so a lane ends up with runs of four consecutive
// output columns of one token and stores each as one 16-byte write.
//
// Work split.  The launch is either one workgroup per output tile, or - when the tiles do not fill
// whole rounds of the chip - as many workgroups as the chip holds at once, each taking its share of
// whole tiles and, before them, an equal share of the K tiles of the remaining output tiles (those
// are cut wherever a share ends).  A workgroup whose share starts inside an output tile leaves its
// accumulators in a workspace slot of its own and raises a flag; the workgroup that has the start
// of that output tile adds the later pieces in K order and stores.  A share is one contiguous range,
// so only its first piece can be handed over and only its last piece can wait, and the waiting
// piece needs pieces that are computed first by the workgroups they belong to: no wait depends on
// another wait.  The sum order is fixed by the split, so the result has the same bits every run.
//
// Layers mostly run on fp6 operands instead, in a kernel of their own (kernels_six.hip); what is here serves layers of rank 0, those whose
// correction outweighs K, calls of few activations, and 2-bit layers of few K tiles or of exponents that span more than 16 values.
//
// Calls that do not fill the chip for long mostly take staged_kernel (pick_small says which): tiles of 64 rows, every
// operand - activations, packed weights, exponents - brought to LDS by direct loads several chunks ahead, and where
// the tiles are too few, several workgroups per tile, each with an equal range of K ("planes"), that store their partial
// sums of Y in the workspace's slots; reduce_planes_kernel adds them in plane order.  There the correction comes first, by
// the plane with the start of K.  A piece of tiled_kernel that hands
// its accumulators over and another that waits for them cost more than such a call's product.
#include <atomic>
#include <mutex>
#include <type_traits>

#include "lqer_internal.h"
#include "mx_device.h"
#include "tiled_common.h"

namespace lqer {

// MINW = wavefronts per SIMD the register allocation must allow (2 lets two four-wavefront workgroups share a compute unit)
// SPLIT = the workgroup walks a list of pieces (work split); otherwise it computes output tile blockIdx.x
// whole, as straight-line code (the loop over pieces costs the main product a few percent)
// WB = mantissa bits of W_q: 4, or 2 (half the code bytes per record, one 32-bit word per block)
template <int TM, int TN, int WR, int WC, int NS, int MINW, bool SPLIT, int WB>
__global__ __launch_bounds__(64 * WR * WC, MINW) void tiled_kernel(TiledArgs a) {
    static_assert(WB == 4 || WB == 2, "weight mantissas of 4 or 2 bits");
    constexpr int BM = 32 * TM * WR;
    constexpr int NW = WR * WC;
    constexpr int STAGE = BM * 128;                // bytes: BM rows x 64 bf16
    constexpr int NT = 64 * NW;
    constexpr int LPT = BM * 8 / NT;               // 16-byte cells each thread moves per chunk
    // chunks between fetching activations and using them: 3 where the registers allow a second set in flight
    constexpr int XD = (TM * TN * 16 + LPT * 8 <= 144) ? 3 : 2;
    static_assert((BM * 8) % NT == 0, "loader must divide evenly");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform by construction
    const int wr = wave / WC, wc = wave % WC;
    const int t = lane & 31, hh = lane >> 5;

    // ---- workgroup -> position in the work split: consecutive positions land on one XCD ----------
    int lin;
    {
        const int nwg = gridDim.x;
        const int pid = blockIdx.x;
        const int xcd = pid & 7, local = pid >> 3;
        const int per = nwg >> 3, rem = nwg & 7;
        lin = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
    }
    __shared__ int wait_ok;
    const int KT = (int)a.KT;                                  // K tiles and chunks fit 32 bits: scalar compares
    const int nb2 = 2 * a.kp16;
    const int tail_chunks = (nb2 + 3) / 4;
    static_assert(NS == 4, "stage and register-set indices below assume rings of four");
    constexpr int ROWS_PER_PASS = NT / 8;
    static_assert(ROWS_PER_PASS % 16 == 0, "swizzle must not depend on the pass");
    const int ld_row0 = tid >> 3;
    // (row >> 1) & 7 is the same for every pass because ROWS_PER_PASS is a multiple of 16
    const int ld_dst0 = ld_row0 * 128 + (((tid & 7) ^ ((ld_row0 >> 1) & 7)) << 4), ld_col = tid & 7;
    // ---- operand reader: in step s this lane reads logical cell 4 hh + s of its TM rows -----------
    // row = (wr TM + tm) 32 + t, so the swizzle term depends on t only
    int rd_off[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
        rd_off[s4] = (wr * TM * 32 + t) * 128 + (((4 * hh + s4) ^ ((t >> 1) & 7)) << 4);
    const int lane16 = lane * 16;
    // exponent of a block without a branch in the main loop: bytes (16, 8, 0xFF, 0) or nibbles (8, 4, 0xF, bias)
    const bool exp4 = a.exp_bias >= 0;                          // wave-uniform
    const int es1 = exp4 ? 8 : 16, es0 = exp4 ? 4 : 8;
    const uint32_t emask = exp4 ? 0xFu : 0xFFu, ebias = exp4 ? (uint32_t)a.exp_bias : 0u;
    // nibbles sit in front of the codes (lane * 4), bytes behind them (lane * 8)
    const int code_off = exp4 ? kWCompactCodeOffset : 0, exp_off = exp4 ? lane16 >> 2 : w_code_bytes(WB) + (lane16 >> 1);

    int64_t dp_next = lin;                                     // next whole tile of this workgroup
    int64_t u = a.sk_share * lin;                              // its range of the shared K tiles
    int64_t u_end = u + a.sk_share;
    if (u_end > a.sk_units) u_end = a.sk_units;
    bool first_piece = true;
  for (;;) {
    // ---- next piece: output tile and K tiles [kt0, kt1) -------------------------------------------
    int64_t tile_lin;
    int kt0, kt1;
    // The shared K tiles come first: the hand-over between workgroups then overlaps with the whole
    // tiles of other workgroups instead of ending the kernel.
    if constexpr (!SPLIT) {
        tile_lin = lin; kt0 = 0; kt1 = KT;
    } else if (u < u_end) {
        const int64_t rt = u / a.sk_tile_units;
        tile_lin = a.dp_tiles + rt;
        kt0 = (int)(u - rt * a.sk_tile_units);
        const int64_t left = u_end - u;
        if (kt0 >= KT) {                                       // only empty units of this tile are left
            u += (left < a.sk_tile_units - kt0) ? left : a.sk_tile_units - kt0;
            continue;
        }
        kt1 = (left < (int64_t)(KT - kt0)) ? kt0 + (int)left : KT;
        u += (kt1 == KT) ? a.sk_tile_units - kt0 : kt1 - kt0;  // past the tile's empty units as well
        if (u > u_end) u = u_end;
    } else if (dp_next < a.dp_tiles) {
        tile_lin = dp_next; kt0 = 0; kt1 = KT;
        dp_next += gridDim.x;
    } else {
        break;
    }
    const bool owner = !SPLIT || (kt0 == 0);                   // this piece stores the tile
    if constexpr (SPLIT) {
        if (!first_piece) __syncthreads();                     // every wavefront is done with the LDS stages
        first_piece = false;
    }
    // output tiles are walked in bands of group_m tile rows
    int tile_m, tile_n;
    {
        const int64_t width = (int64_t)a.group_m * a.grid_n;
        const int grp = (int)(tile_lin / width);
        const int in = (int)(tile_lin - grp * width);
        const int first_m = grp * a.group_m;
        const int gsize = (a.grid_m - first_m < a.group_m) ? a.grid_m - first_m : a.group_m;
        tile_m = first_m + in % gsize;
        tile_n = in / gsize;
    }
    const int64_t m0 = (int64_t)tile_m * BM;
    // ---- activation loader: thread -> 16-byte cells of a stage -----------------------------------
    // Cell j of this thread is row (tid >> 3) + j * (NT / 8), 16-byte column tid & 7.  Rows past M are
    // read as they are (the workspace rows are padded to the tile height) and never stored.
    const uint16_t* ld_base = a.Xh + (m0 + ld_row0) * a.ldxh + 8 * (tid & 7);
    const int64_t ld_stride = (int64_t)ROWS_PER_PASS * a.ldxh;           // elements between passes
    const int64_t g0 = ((int64_t)tile_n * WC + wc) * TN;       // first column group of this wavefront
    auto group_of = [&](int tn) {
        const int64_t g = g0 + tn;
        return g < a.N32 ? g : a.N32 - 1;                      // clamp; the store is masked
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tm][tn][r] = 0.f;

    typedef typename std::conditional<WB == 2, u32x2, u32x4>::type WVec;   // a lane's two blocks of one chunk
    struct WSet {                // packed codes of one chunk for this wavefront's TN column groups
        WVec c[TN];
    };
    struct ESet {                // exponent bytes of one K tile (four chunks) for the same groups
        u32x2 e[TN];
    };
    auto load_wset = [&](WSet& w, int ch) {
        const int64_t tile = ch >> 2;
        const int cc = ch & 3;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint8_t* rec = a.Wt + (tile * a.N32 + group_of(tn)) * a.rec_bytes;   // wave-uniform
            if constexpr (WB != 2) w.c[tn] = *reinterpret_cast<const u32x4*>(rec + code_off + cc * 1024 + lane16);
            else w.c[tn] = *reinterpret_cast<const u32x2*>(rec + code_off + (cc >> 1) * 1024 + lane16 + (cc & 1) * 8);
        }
    };
    auto load_eset = [&](ESet& x, int tile_i) {
        const int64_t tile = tile_i;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint8_t* rec = a.Wt + (tile * a.N32 + group_of(tn)) * a.rec_bytes;
            // always 8 bytes wide: with nibbles only the first word is used (the buffer is padded behind the last record)
            const u32x2_a4 w = *reinterpret_cast<const u32x2_a4*>(rec + exp_off);
            x.e[tn] = u32x2{w[0], exp4 ? w[0] >> 16 : w[1]};
        }
    };
    auto fetch_x = [&](u32x4 (&st)[LPT], int ch) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) st[j] = *reinterpret_cast<const u32x4*>(ld_base + j * ld_stride + (int64_t)ch * 64);
    };
    // correction chunk tc when T is final
    auto fetch_tail = [&](u32x4 (&st)[LPT], int tc) {
        const uint16_t* src = a.Xt + (m0 + ld_row0) * a.ldxt + 8 * ld_col + tc * 64;
#pragma unroll
        for (int j = 0; j < LPT; ++j) st[j] = *reinterpret_cast<const u32x4*>(src + j * ROWS_PER_PASS * a.ldxt);
    };
    // Correction chunk tc when the projection kernel left T as S partial sums (it split K over
    // workgroups): add them in slice order and form the bf16 term this cell holds - T_hi for tail
    // columns below kp, T_lo for the next kp, zero behind.
    auto fetch_t = [&](u32x4 (&st)[LPT], int tc) {
        const int col = (int)tc * 64 + 8 * ld_col;
        const bool lo = col >= a.kp;
        const int r0 = lo ? col - a.kp : col;
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            float sum[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] = 0.f;
            if (col < 2 * a.kp) {
                const float* src = a.Tpart + (m0 + ld_row0 + j * ROWS_PER_PASS) * a.kp + r0;
                for (int sl = 0; sl < a.S; ++sl) {
                    const f32x4 p0 = *reinterpret_cast<const f32x4*>(src + sl * a.tp_stride);
                    const f32x4 p1 = *reinterpret_cast<const f32x4*>(src + sl * a.tp_stride + 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) { sum[e] += p0[e]; sum[4 + e] += p1[e]; }
                }
            }
            uint32_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t hb = f32_bits(sum[e]) & 0xFFFF0000u;
                h[e] = lo ? f32_bits(sum[e] - f32_from_bits(hb)) >> 16 : hb >> 16;
            }
            st[j] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
        }
    };
    // a correction chunk in either form
    auto fetch_corr = [&](u32x4 (&st)[LPT], int tc) {
        if (a.S <= 1) fetch_tail(st, tc);
        else fetch_t(st, tc);
    };
    auto store_x = [&](const u32x4 (&st)[LPT], int stage) {
#pragma unroll
        for (int j = 0; j < LPT; ++j)
            *reinterpret_cast<u32x4*>(lds + stage * STAGE + ld_dst0 + j * ROWS_PER_PASS * 128) = st[j];
    };
    // one 64-wide chunk of the main product: c = chunk index within its K tile = stage = register set.
    // The activation operands are read one MFMA step ahead: `xa` holds step 0 on entry and step 0
    // of the next chunk on exit (that stage was completed two barriers ago, so it may be read
    // before the next barrier).
    Frag xa[TM];
    auto read_xa = [&](Frag (&dst)[TM], int stage_idx, int s4) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
            dst[tm].u = *reinterpret_cast<const u32x4*>(lds + stage_idx * STAGE + rd_off[s4] + tm * 4096);
    };
    auto mma_chunk = [&](const WSet& w, const ESet& x, int c) {
        float sc[TN][2];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint32_t ew = x.e[tn][c >> 1] >> ((c & 1) * es1);
            sc[tn][0] = (WB == 4) ? w_scale((ew & emask) + ebias) : w2_scale((ew & emask) + ebias);
            sc[tn][1] = (WB == 4) ? w_scale(((ew >> es0) & emask) + ebias) : w2_scale(((ew >> es0) & emask) + ebias);
        }
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            Frag xn[TM];
            if (s4 < 3) read_xa(xn, c, s4 + 1);
            else read_xa(xn, (c + 1) & 3, 0);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                bf16x8 wv;
                if constexpr (WB == 4) wv = unpack_w8(w.c[tn][s4], sc[tn][s4 >> 1]);
                else wv = unpack_w8_b2(w.c[tn][s4 >> 1], s4 & 1, sc[tn][s4 >> 1]);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) acc[tm][tn] = mfma32(wv, xa[tm].v, acc[tm][tn]);
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) xa[tm] = xn[tm];
        }
    };

    // prologue: activations of the piece's first two chunks into stages 0 and 1, the weights of its
    // first three, and (XD == 3) the activations of the third in registers
    // (a K tile is four chunks, so a piece has at least four)
    const int first_ch = kt0 * 4;
    WSet w0, w1, w2, w3;
    ESet ea, eb;
    u32x4 sta[LPT], stb[LPT];                      // activations on their way to LDS (stb: XD == 3 only)
    {
        fetch_x(sta, first_ch);
        load_eset(ea, kt0);
        load_wset(w0, first_ch);
        store_x(sta, 0);
        fetch_x(sta, first_ch + 1);
        load_wset(w1, first_ch + 1);
        store_x(sta, 1);
        if constexpr (XD == 3) fetch_x(sta, first_ch + 2);
        load_wset(w2, first_ch + 2);
    }

    // ---- main product -----------------------------------------------------------------------------
    // chunk ch: barrier; fetch the weights of chunk ch+3 into the register set chunk ch-1 has left,
    // and the activations of chunk ch+XD; arithmetic of chunk ch; write the activations of chunk ch+2
    // into stage (ch+2)%4, which was last read two barriers ago.  With XD == 3 those were fetched
    // during the previous chunk and waited in registers (two sets, used in turn), so both kinds of
    // load have more than two chunks' time to arrive: measured with the loads taken out, a
    // distance of two left a fifth of the kernel's time waiting for them.
    // Exponent bytes of the next tile are fetched during the second chunk of a tile.
    // Every load below is issued unconditionally, with its index clamped at the end of the range:
    // a load inside a branch would make the compiler's wait counts assume the worst case and the
    // LDS write at the end of the chunk would wait for the newest weights as well.
    const int last_main = kt1 * 4 - 1, last_tile = kt1 - 1;
    auto step = [&](const WSet& cur, const ESet& ecur, WSet& fill, ESet& enext, u32x4 (&st_old)[LPT],
                    u32x4 (&st_new)[LPT], int ch, int c) {
        __syncthreads();
        if (ch == first_ch) read_xa(xa, 0, 0);   // later chunks find step 0 already read by the previous one
        fetch_x(st_new, ch + XD < last_main ? ch + XD : last_main);
        // loads retire in order: keep the activation loads ahead of the weight loads, so that the
        // LDS write at the end of this chunk does not have to wait for the weights fetched here
        __builtin_amdgcn_sched_barrier(0);
        load_wset(fill, ch + 3 < last_main ? ch + 3 : last_main);
        if (c == 1) load_eset(enext, (ch >> 2) + 1 < last_tile ? (ch >> 2) + 1 : last_tile);
        mma_chunk(cur, ecur, c);
        store_x(st_old, (c + 2) & 3);  // stage (ch+2)%4: free since two barriers ago, also for a clamped re-write
    };
    // XD == 2: one set, fetched and written in the same chunk
    u32x4 (&st_even_old)[LPT] = sta;
    u32x4 (&st_even_new)[LPT] = (XD == 3) ? stb : sta;
    u32x4 (&st_odd_old)[LPT] = (XD == 3) ? stb : sta;
    u32x4 (&st_odd_new)[LPT] = sta;
    for (int tile = kt0; tile < kt1; tile += 2) {
        step(w0, ea, w3, eb, st_even_old, st_even_new, tile * 4 + 0, 0);
        step(w1, ea, w0, eb, st_odd_old, st_odd_new, tile * 4 + 1, 1);
        step(w2, ea, w1, eb, st_even_old, st_even_new, tile * 4 + 2, 2);
        step(w3, ea, w2, eb, st_odd_old, st_odd_new, tile * 4 + 3, 3);
        if (tile + 1 < kt1) {
            step(w0, eb, w3, ea, st_even_old, st_even_new, tile * 4 + 4, 0);
            step(w1, eb, w0, ea, st_odd_old, st_odd_new, tile * 4 + 5, 1);
            step(w2, eb, w1, ea, st_even_old, st_even_new, tile * 4 + 6, 2);
            step(w3, eb, w2, ea, st_odd_old, st_odd_new, tile * 4 + 7, 3);
        }
    }

    // ---- rank-kp correction: [T_hi | T_lo | 0] against B_k ---------------------------------------
    // The correction chunks are fetched here rather than ahead from the main loop: B_k's
    // records are needed at the same moment and cost the same memory round trip.  Stages 0 and 1 are
    // free: every wavefront is past the barrier of the last main chunk, which reads stage 3.
    // lane half hh owns rank blocks jb = 4 cc + 2 hh + {0, 1} of tail chunk cc
    // Lane indices for everything behind the main loop come through an opaque copy: address terms
    // built from them would otherwise be computed once in front of the loop over pieces and
    // occupy registers all through the main product.
    int t_e = t, hh_e = hh, lane_e = lane;
    if constexpr (SPLIT) asm volatile("" : "+v"(t_e), "+v"(hh_e), "+v"(lane_e));
    const int my_tail = owner ? tail_chunks : 0;              // the piece that stores the tile adds the correction
    // two correction chunks at a time through stages 0 and 1 (ranks up to 64 need one round, 256 four)
    for (int cc0 = 0; cc0 < my_tail; cc0 += 2) {
        {
            u32x4 tst[2][LPT];
            if (cc0 > 0) __syncthreads();                      // every wavefront has read the previous pair of chunks
            fetch_corr(tst[0], cc0);
            if (cc0 + 1 < tail_chunks) fetch_corr(tst[1], cc0 + 1);
            store_x(tst[0], 0);
            if (cc0 + 1 < tail_chunks) store_x(tst[1], 1);
            __syncthreads();
        }
        for (int cc = cc0; cc < cc0 + 2 && cc < my_tail; ++cc) {
            const uint8_t* stage = lds + (cc & 1) * STAGE;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int jb = 4 * cc + 2 * hh_e + j;
                const bool live = jb < nb2;
                const int rb = live ? (jb < a.kp16 ? jb : jb - a.kp16) : 0;
                Frag bf[TN][2];
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    u32x4 cw = u32x4{0, 0, 0, 0};
                    uint32_t eb = 0;
                    if (live) {
                        const uint8_t* rec = a.Bt + (group_of(tn) * a.kp16 + rb) * kBRecordBytes;
                        cw = *reinterpret_cast<const u32x4*>(rec + t_e * 16);
                        eb = rec[512 + t_e];
                    }
                    int8x16_to_frags(cw, h_scale(eb), bf[tn][0], bf[tn][1]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    Frag xa[TM];
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm)
                        xa[tm].u = *reinterpret_cast<const u32x4*>(stage + rd_off[2 * j + h] + tm * 4096);
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int tm = 0; tm < TM; ++tm) acc[tm][tn] = mfma32(bf[tn][h].v, xa[tm].v, acc[tm][tn]);
                }
            }
        }
    }

    // ---- a piece that starts inside the tile hands its accumulators over ---------------------------
    // The slot is written and read with device-scope relaxed atomic accesses of 8 bytes: they pass
    // through the XCD's L2 to where every XCD sees them, so neither side needs a cache write-back or
    // invalidate (which would also throw out the weights and activations other workgroups share there).
    constexpr int64_t PART_FLOATS = (int64_t)NW * TM * TN * 1024;          // = BM x BN
    typedef unsigned long long u64;
    union Pair { u64 q; float f[2]; };
    if (SPLIT && !owner) {
        u64* slot = reinterpret_cast<u64*>(a.Part + (int64_t)lin * PART_FLOATS) + (int64_t)wave * TM * TN * 8 * 64 + lane_e;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int h8 = 0; h8 < 8; ++h8) {
                    Pair p;
                    p.f[0] = acc[tm][tn][2 * h8]; p.f[1] = acc[tm][tn][2 * h8 + 1];
                    __hip_atomic_store(slot + ((tm * TN + tn) * 8 + h8) * 64, p.q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
        // The flag may only be raised once every slot store of every wavefront has been acknowledged by the
        // memory system: a workgroup-scope fence does not wait for outstanding vector stores on this chip
        // (and a device-scope release would write the XCD's L2 back), so each wavefront drains its own
        // store counter explicitly, the barrier collects all wavefronts, and only then is the flag stored.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_store(a.flags + lin, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        continue;
    }
    // ---- the piece with the start of the tile adds the later pieces, in K order --------------------
    if (SPLIT && kt1 < KT) {
        const int64_t rt = tile_lin - a.dp_tiles;
        const int64_t last_wg = (rt * a.sk_tile_units + a.KT - 1) / a.sk_share;   // workgroup with the tile's last K tile
        for (int64_t w = lin + 1; w <= last_wg; ++w) {
            if (tid == 0) {
                int polls = 0;
                while (__hip_atomic_load(a.flags + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u &&
                       polls < a.spin_limit) {
                    __builtin_amdgcn_s_sleep(8);
                    ++polls;
                }
                wait_ok = (polls < a.spin_limit) ? 1 : 0;
            }
            __syncthreads();
            const bool ok = wait_ok != 0;
            const u64* slot = reinterpret_cast<const u64*>(a.Part + w * PART_FLOATS) + (int64_t)wave * TM * TN * 8 * 64 + lane_e;
            // groups of 32 loads: enough in flight to cover the round trip, few enough to fit beside the accumulators
            constexpr int PER = TM * TN * 8;                   // 8-byte words of this lane in the slot
            constexpr int GRP = PER < 32 ? PER : 32;
            static_assert(PER % GRP == 0, "whole groups");
#pragma unroll
            for (int g0 = 0; g0 < PER; g0 += GRP) {
                Pair p[GRP];
#pragma unroll
                for (int i = 0; i < GRP; ++i)
                    p[i].q = __hip_atomic_load(slot + (g0 + i) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int i = 0; i < GRP; ++i) {
                    const int mt = (g0 + i) / 8, h8 = (g0 + i) % 8;
                    // a piece that never arrived must not pass for a result
                    if (!ok) p[i].f[0] = p[i].f[1] = __builtin_nanf("");
                    acc[mt / TN][mt % TN][2 * h8] += p[i].f[0];
                    acc[mt / TN][mt % TN][2 * h8 + 1] += p[i].f[1];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __syncthreads();                                   // wait_ok may be rewritten
        }
    }

    // ---- store: lane (t, hh) holds columns 8 r4 + 4 hh .. + 3 of token t for every MFMA tile ------
    // As MXINT8 for the next layer: block b of a column group is columns 16 b .. 16 b + 15 = accumulator
    // registers 8 b .. 8 b + 7 of this lane and of lane ^ 32 (the same token).
    if (a.Yc != nullptr) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t row = m0 + (wr * TM + tm) * 32 + t_e;
            if (row >= a.M) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int64_t cg = g0 + tn;
                if (cg >= a.N32) continue;
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = acc[tm][tn][8 * b + i];
                    uint32_t w0, w1;
                    const uint32_t eb = requant_half_block(v, w0, w1);
                    const int64_t n0 = cg * 32 + 16 * b;
                    if (n0 < a.N) {
                        int8_t* dst = a.Yc + row * a.ldyc + n0 + 4 * hh_e;
                        *reinterpret_cast<uint32_t*>(dst) = w0;
                        *reinterpret_cast<uint32_t*>(dst + 8) = w1;
                        if (hh_e == 0) a.Ye[row * (a.N >> 4) + (n0 >> 4)] = (uint8_t)eb;
                    }
                }
            }
        }
        if constexpr (!SPLIT) break; else continue;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t row = m0 + (wr * TM + tm) * 32 + t_e;
        if (row >= a.M) continue;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int64_t cg = g0 + tn;
            if (cg >= a.N32) continue;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int64_t n = cg * 32 + 8 * r4 + 4 * hh_e;
                float* dst = a.Y + row * a.ldy + n;
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
    if constexpr (!SPLIT) break;
  }   // pieces
}

// ---- the same product with every operand staged by direct-to-LDS loads -----------------------------------------------
// What bounds these launches is not the loads' latency (three or seven stages ahead measure the same) but one or two
// wavefronts on a SIMD issuing an instruction every four to eight cycles each, and the waits for their LDS reads: 64 x 128 tiles of four
// 64 x 32 wavefronts, two or three workgroups on a compute unit, are the fastest where the launch is a round or two.  A K tile of such
// a workgroup takes 0.83 us alone and 1.5 us beside another (its MFMAs: 0.45 and 0.9), 1.17 and 1.77 by a loop of two chunks
// over five stages with the reads one step ahead (45 scalar instructions a chunk and ten vector ones for addresses: now 18 and none).
// Whole calls, that loop -> this one: 4096 x 4096 at 40 tokens 16.9 -> 15.9 us, 4096 x 11008 at 128 32.7 -> 27.2,
// 4112 x 11000 at 203 44.9 -> 38.9, 4096 x 4096 at 512 36.8 -> 31.2, rank 64 at 1024 57.4 -> 53.9; 2-bit rank 128 at 512 50.0 -> 43.5.
// (The correction's operands are asked for in one go per two chunks: 2-bit weights with rank 256 at 64 tokens 84 -> 30 us.)
// Four stages of 64 K in LDS, one per chunk of a K tile: [BM rows x 64 activations, 16-byte cells XOR-swizzled][wave][TN]
// 1 KiB of codes [wave][TN] 256 B of exponent words; chunk ch + 3 is asked for when chunk ch starts.
template <int TM, int TN, int WR, int WC, int MINW, bool PLANES, int WB>
__global__ __launch_bounds__(64 * WR * WC, MINW) void staged_kernel(TiledArgs a) {
    static_assert(WB == 4 || WB == 2, "weight mantissas of 4 or 2 bits");
    constexpr int BM = 32 * TM * WR, NW = WR * WC, NT = 64 * NW;
    constexpr int XB = BM * 128, WOFF = XB, EOFF = XB + NW * TN * 1024, STAGE = EOFF + NW * TN * 256;
    constexpr int XL = XB / 1024 / NW;             // activation loads per wavefront and chunk
    static_assert(XB % (1024 * NW) == 0 && NW % 2 == 0, "whole loads, and a swizzle that is the same for all of a wavefront's");
    constexpr int L = XL + 2 * TN;                 // loads per wavefront and chunk
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int t = lane & 31, hh = lane >> 5;
    // workgroup -> output tile (and K plane): consecutive positions land on one XCD
    int lin;
    {
        const int nwg = gridDim.x, pid = blockIdx.x;
        const int xcd = pid & 7, local = pid >> 3, per = nwg >> 3, rem = nwg & 7;
        lin = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
    }
    const int KT = (int)a.KT;
    int plane = 0, kt0 = 0, kt1 = KT;
    if constexpr (PLANES) {
        // neighbouring workgroups of one XCD: neighbouring tiles of the same K range, which share activations or weights
        plane = lin / (int)a.dp_tiles;
        lin -= plane * (int)a.dp_tiles;
        kt0 = plane * (int)a.sk_share;
        kt1 = kt0 + (int)a.sk_share < KT ? kt0 + (int)a.sk_share : KT;
    }
    int tile_m, tile_n;                            // bands of group_m tile rows
    {
        const int width = a.group_m * a.grid_n, grp = lin / width, in = lin - grp * width, first_m = grp * a.group_m;
        const int gsize = (a.grid_m - first_m < a.group_m) ? a.grid_m - first_m : a.group_m;
        tile_m = first_m + in % gsize;
        tile_n = in / gsize;
    }
    const int64_t m0 = (int64_t)tile_m * BM;
    const int64_t g0 = ((int64_t)tile_n * WC + wc) * TN;       // first column group of this wavefront
    auto group_of = [&](int tn) { return g0 + tn < a.N32 ? g0 + tn : a.N32 - 1; };   // clamped; the store is masked

    // ---- loads ---------------------------------------------------------------------------------------------------
    // Activations: load j of this wavefront brings rows 8 (NW j + wave) .. + 7; lane -> row lane / 8 of them, LDS cell
    // lane % 8, which holds the row's cell (lane % 8) ^ ((row >> 1) & 7).  (Rows past M are workspace rows: see there.)
    // What differs between the loads of a chunk is in the lanes' offsets, so that one scalar address serves all of a kind.
    uint32_t x_off[XL], w_off[TN], e_off[TN];
#pragma unroll
    for (int j = 0; j < XL; ++j)
        x_off[j] = (uint32_t)((8 * (NW * j + wave) + (lane >> 3)) * (int)a.ldxh * 2) +
                   (((uint32_t)(lane & 7) ^ (uint32_t)(((wave & 1) * 4 + (lane >> 4)) & 7)) << 4);
    const bool exp4 = a.exp_bias >= 0;             // wave-uniform
    const int64_t g_first = group_of(0);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const uint32_t rec = (uint32_t)(group_of(tn) - g_first) * (uint32_t)a.rec_bytes;
        w_off[tn] = rec + lane * 16 + (exp4 ? kWCompactCodeOffset : 0);
        e_off[tn] = rec + (exp4 ? lane * 4 : w_code_bytes(WB) + lane * 8);
    }
    const int64_t tile_stride = a.N32 * a.rec_bytes;
    const uint8_t* x_ptr = reinterpret_cast<const uint8_t*>(a.Xh + m0 * a.ldxh + kt0 * kTileK);
    const uint8_t* w_ptr = a.Wt + g_first * a.rec_bytes + kt0 * tile_stride;       // record of the K tile being asked for
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)lds);
    const uint32_t at_x = lds0 + wave * 1024, at_w = lds0 + wave * (TN * 1024), at_e = lds0 + wave * (TN * 256);
    const uint32_t e_half = exp4 ? 0 : 4;          // exponent words: with nibbles the record's only one, with bytes the first or second four of a lane's eight
    auto issue = [&](auto cc) {                    // the next chunk of the row, number CC of its K tile -> stage CC
        constexpr int CC = decltype(cc)::value, ST = CC * STAGE;
        lds_dma16<ST>(at_x, x_off[0], x_ptr);
        if constexpr (XL > 1) lds_dma16<ST + NW * 1024>(at_x, x_off[1], x_ptr);
        if constexpr (XL > 2) lds_dma16<ST + 2 * NW * 1024>(at_x, x_off[2], x_ptr);
        if constexpr (XL > 3) lds_dma16<ST + 3 * NW * 1024>(at_x, x_off[3], x_ptr);
        const uint8_t* wp = w_ptr + (WB == 2 ? CC >> 1 : CC) * 1024;
        const uint8_t* ep = CC < 2 ? w_ptr : w_ptr + e_half;
        lds_dma16<ST + WOFF>(at_w, w_off[0], wp);
        lds_dma4<ST + EOFF>(at_e, e_off[0], ep);
        if constexpr (TN > 1) {
            lds_dma16<ST + WOFF + 1024>(at_w, w_off[TN - 1], wp);
            lds_dma4<ST + EOFF + 256>(at_e, e_off[TN - 1], ep);
        }
        x_ptr += 128;
        if constexpr (CC == 3) w_ptr += tile_stride;
    };
    static_assert(XL <= 4 && TN <= 2, "issue() spells its loads out");

    // ---- operands ------------------------------------------------------------------------------------------------
    int rd_off[4];                                 // step s: logical cell 4 hh + s of this lane's TM rows
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) rd_off[s4] = (wr * TM * 32 + t) * 128 + (((4 * hh + s4) ^ ((t >> 1) & 7)) << 4);
    auto read_x = [&](Frag (&dst)[TM], const uint8_t* stage, int s4) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) dst[tm].u = *reinterpret_cast<const u32x4*>(stage + rd_off[s4] + tm * 4096);
    };
    typedef typename std::conditional<WB == 2, u32x2, u32x4>::type WVec;   // a lane's two blocks of one chunk
    struct WSet { WVec c[TN]; uint32_t e[TN]; };
    auto read_w = [&](WSet& w, const uint8_t* stage, int cc) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint8_t* src = stage + WOFF + (wave * TN + tn) * 1024 + lane * 16;
            if constexpr (WB != 2) w.c[tn] = *reinterpret_cast<const u32x4*>(src);
            else w.c[tn] = *reinterpret_cast<const u32x2*>(src + (cc & 1) * 8);
            w.e[tn] = *reinterpret_cast<const uint32_t*>(stage + EOFF + (wave * TN + tn) * 256 + lane * 4);
        }
    };
    const int es0 = exp4 ? 4 : 8;
    const uint32_t emask = exp4 ? 0xFu : 0xFFu;
    const uint32_t ebase = ((exp4 ? (uint32_t)a.exp_bias : 0u) + (WB == 4 ? 7u : 9u)) << 23;   // w_scale / w2_scale of exponent 0

    // The terms are summed as two chains - the correction and then the first half of the K range, the second half - since
    // an fp32 chain rounds at the size its sum has reached: the correction's steps come while that is small.  Relative
    // distance from the 64-bit result, 4096 x 4096 at 512 tokens, one chain with the correction last -> so: rank 32 2.29e-7 ->
    // 2.22e-7, rank 128 2.91e-7 -> 2.57e-7, rank 256 3.37e-7 -> 2.72e-7.
    f32x16 acc0[TM][TN], acc1[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc0[tm][tn][r] = acc1[tm][tn][r] = 0.f;

    // ---- main product --------------------------------------------------------------------------------------------
    const int tiles = kt1 - kt0;                   // K tiles of this workgroup
    // Software pipeline of MFMA steps (16 of K), four to a chunk, four chunks to a K tile, all of them spelled out so that
    // every LDS address is a constant behind a lane's: while the MFMAs of one step run, the weights of the next are expanded and
    // the activations of the third one after it (AHEAD) read from LDS.  A wavefront issues an instruction every four to eight
    // cycles and an LDS read takes longer than a step, so what bounds these launches - one or two wavefronts on a SIMD -
    // is the instructions between its MFMAs and the waits for operands: the pattern below puts a few vector instructions
    // behind every MFMA, where they cost nothing.
    constexpr int AHEAD = TN == 1 ? 3 : 2;         // steps (a step of two column groups is twice as long, and short of registers)
    Frag xr[4][TM];                                // activations of step s of this chunk or the next
    bf16x8 wv[TN];
    float sc[TN][2];
    auto scales = [&](const WSet& w, int cc) {
        const int esh = exp4 ? (cc & 3) * 8 : (cc & 1) * 16;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const uint32_t ew = w.e[tn] >> esh;
            sc[tn][0] = f32_from_bits(((ew & emask) << 23) + ebase);
            sc[tn][1] = f32_from_bits((((ew >> es0) & emask) << 23) + ebase);
        }
    };
    auto expand = [&](const WSet& w, int s4) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if constexpr (WB == 4) wv[tn] = unpack_w8(w.c[tn][s4], sc[tn][s4 >> 1]);
            else wv[tn] = unpack_w8_b2(w.c[tn][s4 >> 1], s4 & 1, sc[tn][s4 >> 1]);
        }
    };
    // Chunk CC: on entry xr holds its first AHEAD steps, wv the weights of step 0 and w its codes; on exit the same of the next chunk, in wn its codes.
    auto chunk = [&](f32x16 (&acc)[TM][TN], const WSet& w, WSet& wn, auto cc) {
        constexpr int CC = decltype(cc)::value;
        const uint8_t* const cur = lds + CC * STAGE;
        const uint8_t* const nxt = lds + (CC + 1) % 4 * STAGE;
        read_w(wn, nxt, CC + 1);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            bf16x8 now[TN];
            read_x(xr[(s4 + AHEAD) & 3], s4 + AHEAD < 4 ? cur : nxt, (s4 + AHEAD) & 3);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) now[tn] = wv[tn];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) acc[tm][tn] = mfma32(now[tn], xr[s4][tm].v, acc[tm][tn]);
            if (s4 < 3) {
                expand(w, s4 + 1);
            } else {
                scales(wn, CC + 1);
                expand(wn, 0);
            }
            if (s4 == 0) __builtin_amdgcn_sched_group_barrier(0x100, TM + 2 * TN, 0);              // LDS reads
            else __builtin_amdgcn_sched_group_barrier(0x100, TM, 0);
#pragma unroll
            for (int i = 0; i < TM * TN; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                              // an MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, (10 * TN + TM * TN - 1) / (TM * TN), 0);   // vector instructions
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    constexpr std::integral_constant<int, 0> C0{};
    constexpr std::integral_constant<int, 1> C1{};
    constexpr std::integral_constant<int, 2> C2{};
    constexpr std::integral_constant<int, 3> C3{};
    issue(C0);
    issue(C1);

    // ---- rank-kp correction: [T_hi | T_lo | 0] against B_k, by the workgroup with the start of K -----------------------
    // (its tiles of T take the memory of the last two stages, which the loads on their way do not write)
    const int nb2 = 2 * a.kp16, tail_chunks = (nb2 + 3) / 4;
    const int my_tail = (kt0 == 0) ? tail_chunks : 0;
    constexpr int LPT = BM * 8 / NT;               // 16-byte cells each thread moves per chunk
    constexpr int ROWS_PER_PASS = NT / 8;
    static_assert(ROWS_PER_PASS % 16 == 0, "swizzle must not depend on the pass");
    const int ld_row0 = tid >> 3;
    const int ld_dst0 = ld_row0 * 128 + (((tid & 7) ^ ((ld_row0 >> 1) & 7)) << 4);
    // Asked for beside the first chunks instead of behind the last: rank 128 at 512 tokens 56 -> 54 us, 2-bit rank 256 at 64
    // tokens 51 -> 48 us a call; nothing slower.
    uint8_t* const t_tiles = lds + 2 * STAGE;
    for (int cc0 = 0; cc0 < my_tail; cc0 += 2) {   // two correction chunks at a time (ranks up to 64 need one round)
        u32x4 bw[2][2][TN];                        // B_k's codes and exponents of both chunks: asked for ahead of T
        uint32_t be[2][2][TN];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int jb = 4 * (cc0 + q) + 2 * hh + j;
                const int rb = jb < nb2 ? (jb < a.kp16 ? jb : jb - a.kp16) : 0;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    const uint8_t* rec = a.Bt + (group_of(tn) * a.kp16 + rb) * kBRecordBytes;
                    bw[q][j][tn] = *reinterpret_cast<const u32x4*>(rec + t * 16);
                    be[q][j][tn] = rec[512 + t];
                }
            }
        u32x4 tst[2][LPT];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < LPT; ++j) {
                const int col = (cc0 + q) * 64 + 8 * (tid & 7);
                const int64_t row = m0 + ld_row0 + j * ROWS_PER_PASS;
                tst[q][j] = u32x4{0, 0, 0, 0};
                if (col >= 2 * a.kp) continue;
                if (a.S <= 1) {
                    tst[q][j] = *reinterpret_cast<const u32x4*>(a.Xt + row * a.ldxt + col);
                    continue;
                }
                // T as S fp32 partial sums: added in slice order, then the bf16 term this cell holds
                const bool lo = col >= a.kp;
                const float* src = a.Tpart + row * a.kp + (lo ? col - a.kp : col);
                f32x4 p0[8], p1[8];
#pragma unroll
                for (int sl = 0; sl < 8; ++sl) {   // all slices' loads in flight together
                    const int64_t o = (int64_t)(sl < a.S ? sl : a.S - 1) * a.tp_stride;
                    p0[sl] = *reinterpret_cast<const f32x4*>(src + o);
                    p1[sl] = *reinterpret_cast<const f32x4*>(src + o + 4);
                }
#pragma unroll
                for (int sl = 1; sl < 8; ++sl)
                    if (sl < a.S) { p0[0] += p0[sl]; p1[0] += p1[sl]; }
                uint32_t h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = e < 4 ? p0[0][e & 3] : p1[0][e & 3];
                    const uint32_t hb = f32_bits(v) & 0xFFFF0000u;
                    h[e] = lo ? f32_bits(v - f32_from_bits(hb)) >> 16 : hb >> 16;
                }
                tst[q][j] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
            }
        if (cc0 > 0) __syncthreads();              // every wavefront is done with the previous two chunks
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < LPT; ++j)
                *reinterpret_cast<u32x4*>(t_tiles + q * XB + ld_dst0 + j * ROWS_PER_PASS * 128) = tst[q][j];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (cc0 + q >= my_tail) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int jb = 4 * (cc0 + q) + 2 * hh + j;     // lane half hh owns rank blocks 4 cc + 2 hh + {0, 1}
                Frag bf[TN][2];
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    int8x16_to_frags(jb < nb2 ? bw[q][j][tn] : u32x4{0, 0, 0, 0}, h_scale(be[q][j][tn]), bf[tn][0], bf[tn][1]);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    Frag xt[TM];
                    read_x(xt, t_tiles + q * XB, 2 * j + h);
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int tm = 0; tm < TM; ++tm) acc0[tm][tn] = mfma32(bf[tn][h].v, xt[tm].v, acc0[tm][tn]);
                }
            }
        }
    }
    if (my_tail > 0) __syncthreads();              // the tiles of T have been read by everybody

    issue(C2);
    staged_wait<2 * L>();
    WSet w0, w1;
    read_w(w0, lds, 0);
#pragma unroll
    for (int s4 = 0; s4 < AHEAD; ++s4) read_x(xr[s4], lds, s4);
    scales(w0, 0);
    expand(w0, 0);
    // A K tile.  Chunks CC and CC + 1 have landed when CC starts, for every wavefront; its predecessor has been read by
    // everybody (the RA newest reads are of CC itself), and that stage takes chunk CC + 3: of the same K tile, or of the next
    // one unless this is the last.
    constexpr int RA = AHEAD * TM;
    auto tile = [&](f32x16 (&acc)[TM][TN], auto last) {
        constexpr bool LAST = decltype(last)::value;
        staged_wait<L, RA>();
        issue(C3);
        chunk(acc, w0, w1, C0);
        staged_wait<L, RA>();
        if constexpr (!LAST) issue(C0);
        chunk(acc, w1, w0, C1);
        staged_wait<LAST ? 0 : L, RA>();
        if constexpr (!LAST) issue(C1);
        chunk(acc, w0, w1, C2);
        if constexpr (!LAST) {
            staged_wait<L, RA>();
            issue(C2);
        }
        chunk(acc, w1, w0, C3);                    // (the last one reads ahead what nobody uses)
    };
    const int half = (tiles + 1) / 2;
    int kt = 0;
    for (; kt < half && kt + 1 < tiles; ++kt) tile(acc0, std::false_type{});
    for (; kt + 1 < tiles; ++kt) tile(acc1, std::false_type{});
    tile(acc1, std::true_type{});
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc0[tm][tn][r] += acc1[tm][tn][r];

    // ---- store: lane (t, hh) holds columns 8 r4 + 4 hh .. + 3 of token t for every MFMA tile ------------------------------
    if (!PLANES && a.Yc != nullptr) {              // as MXINT8: block b of a column group is registers 8 b .. + 7 of two lanes
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t row = m0 + (wr * TM + tm) * 32 + t;
            if (row >= a.M) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                if (g0 + tn >= a.N32) continue;
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = acc0[tm][tn][8 * b + i];
                    uint32_t w0, w1;
                    const uint32_t eb = requant_half_block(v, w0, w1);
                    const int64_t n0 = (g0 + tn) * 32 + 16 * b;
                    if (n0 < a.N) {
                        int8_t* dst = a.Yc + row * a.ldyc + n0 + 4 * hh;
                        *reinterpret_cast<uint32_t*>(dst) = w0;
                        *reinterpret_cast<uint32_t*>(dst + 8) = w1;
                        if (hh == 0) a.Ye[row * (a.N >> 4) + (n0 >> 4)] = (uint8_t)eb;
                    }
                }
            }
        }
        return;
    }
    float* out = a.Y;
    int64_t ldo = a.ldy;
    if constexpr (PLANES) {
        ldo = plane_ld(a.N);
        out = a.Part + (int64_t)plane * a.M * ldo;
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int64_t row = m0 + (wr * TM + tm) * 32 + t;
        if (row >= a.M) continue;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if (g0 + tn >= a.N32) continue;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int64_t n = (g0 + tn) * 32 + 8 * r4 + 4 * hh;
                float* dst = out + row * ldo + n;
                const f32x4 v = f32x4{acc0[tm][tn][4 * r4], acc0[tm][tn][4 * r4 + 1], acc0[tm][tn][4 * r4 + 2], acc0[tm][tn][4 * r4 + 3]};
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

// Y = sum of the K planes in plane order (the same bits on every run), as fp32 or as MXINT8 blocks of 16 along N.  Bound
// by the planes' way back from the caches (about 5.7 TB/s written and read, plus 4 us); a thread adds four columns with
// eight planes' loads in flight, and for MXINT8 the four lanes of a quad hold one block (N is then a multiple of 16).
__global__ __launch_bounds__(256) void reduce_planes_kernel(TiledArgs a, int planes) {
    const int64_t ldp = plane_ld(a.N), n4 = ldp / 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.M * n4) return;
    const int64_t r = i / n4, c = 4 * (i - r * n4);
    const float* src = a.Part + r * ldp + c;
    const int64_t stride = a.M * ldp;
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < planes; z0 += 8) {
        f32x4 q[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = *reinterpret_cast<const f32x4*>(src + (z0 + j < planes ? z0 + j : planes - 1) * stride);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (z0 + j < planes) v = (z0 + j == 0) ? q[0] : v + q[j];
    }
    if (a.Yc != nullptr) {
        float m = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(v[0]), __builtin_fabsf(v[1])),
                                  __builtin_fmaxf(__builtin_fabsf(v[2]), __builtin_fabsf(v[3])));
        m = __builtin_fmaxf(m, __shfl_xor(m, 1));
        m = __builtin_fmaxf(m, __shfl_xor(m, 2));
        const uint32_t eb = (f32_bits(m) >> 23) & 0xFFu;
        uint32_t w = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) w |= ((uint32_t)mx8_code(v[j], (int)eb - 127) & 0xFFu) << (8 * j);
        *reinterpret_cast<uint32_t*>(a.Yc + r * a.ldyc + c) = w;
        if ((c & 15) == 0) a.Ye[r * (a.N >> 4) + (c >> 4)] = (uint8_t)eb;
        return;
    }
    float* dst = a.Y + r * a.ldy + c;
    if (c + 3 < a.N) {
        *reinterpret_cast<f32x4*>(dst) = v;
    } else {
        for (int j = 0; c + j < a.N; ++j) dst[j] = v[j];
    }
}

hipError_t launch_reduce_planes(const TiledArgs& a, int planes, hipStream_t s) {
    const int64_t items = a.M * (plane_ld(a.N) / 4);
    hipLaunchKernelGGL(reduce_planes_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, s, a, planes);
    return hipGetLastError();
}

// Time estimates in microseconds for one tile shape, launched as one workgroup per tile or with the
// work split described at the head of this file.
struct TileShape { int id, bm, bn, share; double pair, single, cut; };
// whole-chip TFLOP/s measured on an 8192 x 28672 layer: `pair` with `share` workgroups on every compute unit
// (M = 4096), `single` with one (M = 128), `cut` for the pieces of tiles cut along K (M = 128 .. 2048)
static const TileShape kShapes[] = {
    {11, 128, 512, 1, 1372.0, 1372.0, 1372.0}, {12, 128, 256, 2, 1300.0, 1000.0, 1150.0}, {4, 128, 128, 2, 1058.0, 800.0, 1058.0},
};
constexpr double kPieceUs = 4.0;       // filling the pipeline and storing the tile, per piece
constexpr double kSplitFixedUs = 38.0; // what a split launch was measured to take beyond this, per workgroup sharing a compute unit: the
                                       // pieces' drain and refill, not the slots' way through memory (the time is the same without them)

// one K tile (256 deep) of one output tile, with `share` workgroups on every compute unit
static double unit_us(const TileShape& sh, int share, int cus) {
    const double rate = (share == sh.share) ? sh.pair : sh.single;       // TFLOP/s = flop/us * 1e-6
    return 2.0 * sh.bm * sh.bn * kTileK * (double)cus * share / (rate * 1e6);
}

static double time_whole(const TileShape& sh, int64_t tiles, int64_t KT, int cus) {
    const int64_t n = (tiles + cus - 1) / cus;               // tiles of the busiest compute unit
    const double full = (double)KT * unit_us(sh, sh.share, cus) + kPieceUs;
    const double alone = (double)KT * unit_us(sh, 1, cus) + kPieceUs;
    return (sh.share == 2) ? (double)(n / 2) * full + (double)(n % 2) * alone : (double)n * full;
}

static double time_split(const TileShape& sh, int64_t tiles, int64_t KT, int cus) {
    const Split sp = split_tiles(tiles, KT, (int64_t)cus * sh.share, true);
    const bool one_piece = sp.aligned;                       // cut along tile boundaries: no workgroup gets two pieces
    if (sp.sk_units == 0) return time_whole(sh, tiles, KT, cus);
    const double rounds = (double)(sp.dp_tiles / sp.grid);
    const double whole_part = rounds * (double)KT * unit_us(sh, sh.share, cus);
    const double cut_part = (double)sp.sk_share * unit_us(sh, sh.share, cus) * sh.pair / sh.cut;
    if (!one_piece) return whole_part + cut_part + (rounds + 2.0) * kPieceUs + kSplitFixedUs * sh.share;
    // cut along tiles: one piece per workgroup; the workgroup with a tile's first piece reads the slots of the
    // others one after the other (about 7 us per 256 KiB slot beyond the first, from launches with 2 and 4 pieces)
    const double pieces = (double)(sp.sk_tile_units / sp.sk_share);
    const double slot_us = 7.0 * (double)sh.bm * sh.bn * 4.0 / 262144.0;
    return whole_part + cut_part + (rounds + 1.0) * kPieceUs + 0.5 * kSplitFixedUs + (pieces - 2.0) * slot_us;
}

// the split has to promise a clear gain: its estimate is the rougher of the two
static bool split_pays(const TileShape& sh, int64_t tiles, int64_t KT, int cus) {
    return time_split(sh, tiles, KT, cus) < 0.95 * time_whole(sh, tiles, KT, cus);
}

// ---- calls that do not fill the chip for long: which tile, how many K planes -------------------------------------------
// Time model, in us: a workgroup takes `unit[r - 1]` per K tile when r of them share a compute unit, `round` more per round of
// workgroups, `fixed` per launch; every two chunks of the correction beyond the first two take corr[0] + corr[1] S, S the
// partial sums of T, per round of workgroups that have it, and tile[0] + tile[1] S per output tile of the busiest compute unit
// (two workgroups there share its way to the caches); Y takes `out` per MB; planes take `plane` and `plane_mb` per MB of partial
// sums written and read.  Fitted to 5000 timings of 769 calls (K 256 to 14336, N 256 to 28672, 33 to 65536 tokens, ranks 0 to
// 256), 128 x 512 to 25000 older ones: mean error 4 to 7 % a shape.  Its choice is 0.6 % from the fastest form timed on average, within 4 % on
// 95 % of the calls, 33 % off at the very worst (2.4 %, 17 %, 33 % with the figures of the staged kernel's loop before).
// Main product, best form of tiled_kernel against what is chosen: 4096 x 4096 at 64 tokens 43 us and 12 (64 x 128 in planes),
// 4112 x 11000 at 203 tokens 52 and 33 (64 x 128), 2-bit 4096 x 4096 with rank 256 at 2048 tokens 101 and 80 (64 x 512).  Forms of tiled_kernel belong to the choice as much as the staged ones, also at 2 bits and
// large ranks: best staged form against what is chosen, 384 x 27648 with rank 128 at 4627 tokens 265 us and 243, 2-bit
// 592 x 912 with rank 64 at 63752 tokens 170 and 140.
struct SmallShape { int id, bm, bn, resident; double unit[2], round, fixed, corr[2], tile[2], out, plane, plane_mb; };
static const SmallShape kSmallShapes4[] = {
    {33, 64, 128, 2, {0.83, 1.52}, 2.11, 5.75, {0.99, 0.0}, {0.0, 0.66}, 0.074, 3.6, 0.125},
    {31, 64, 256, 2, {1.62, 2.80}, 1.27, 6.38, {2.48, 0.0}, {0.0, 0.58}, 0.191, 3.6, 0.169},
    {32, 64, 512, 1, {2.61, 0.0}, 2.99, 6.01, {0.0, 0.31}, {3.72, 0.0}, 0.193, 3.5, 0.170},
    {12, 128, 256, 2, {3.07, 5.26}, 2.24, 6.15, {2.03, 1.40}, {0.0, 1.11}, 0.188, 0.0, 0.0},        // tiled_kernel, whole tiles
    {11, 128, 512, 1, {4.69, 0.0}, 2.7, 7.2, {0.0, 0.0}, {4.15, 1.16}, 0.220, 0.0, 0.0},
};
static const SmallShape kSmallShapes2[] = {
    {33, 64, 128, 2, {0.89, 1.52}, 1.18, 6.52, {0.20, 0.04}, {0.0, 0.61}, 0.116, 3.9, 0.148},
    {31, 64, 256, 2, {1.63, 2.77}, 0.90, 6.87, {1.36, 0.02}, {0.0, 0.66}, 0.221, 3.7, 0.183},
    {32, 64, 512, 1, {2.57, 0.0}, 3.85, 5.52, {0.0, 0.46}, {2.51, 0.0}, 0.168, 3.2, 0.189},
    {12, 128, 256, 2, {3.08, 5.22}, 0.38, 8.44, {1.68, 2.03}, {0.0, 0.47}, 0.192, 0.0, 0.0},
    {11, 128, 512, 1, {4.53, 0.0}, 3.2, 7.8, {0.0, 0.0}, {3.50, 1.30}, 0.205, 0.0, 0.0},
};
// The 128 x 512 shape with tiles cut in pieces, for 4 and 2 bits: us per launch, K tile of a piece, K tile and number of whole
// rounds, piece beyond two, the correction per round.  Whole pieces per tile (460 timings, 5 %), and equal shares, whose
// estimate is the rougher one (370 timings, 6 %): it counts only where the launch is long enough for them to pay, and has to
// promise 3 %.
struct SmallPieces { double fixed, share, unit, round, piece, corr, slice; };
static const SmallPieces kSmallWhole[2] = {{24.3, 5.73, 5.17, 12.3, 3.6, 4.5, 1.30}, {24.6, 5.46, 5.23, 10.5, 3.9, 4.4, 1.27}};
static const SmallPieces kSmallShares[2] = {{22.3, 6.11, 6.03, 10.0, 0.0, 3.6, 1.82}, {21.0, 6.14, 6.14, 9.6, 0.0, 3.4, 1.76}};
constexpr double kSharesFlops = 6e10;
constexpr int kMaxPlanes = 16;
// Above this many operations the chip is full long enough to lower its clock, which this model does not know; the estimate
// above is calibrated there (8192 x 28672 at 2048 tokens: its choice 714 us, this model's 770 us; below the line, main product
// of 11008 x 4096 at 1500 tokens, 146 to 149 us by the estimate's forms, 142 by the model's choice).
constexpr double kSmallFlops = 1.5e11;

struct SmallPick { int id, planes, share; double us; };      // share: K tiles per plane; planes 0: tiled_kernel in pieces

// pairs of correction chunks beyond the first
static int more_pairs(int kp) { return kp > 64 ? (kp + 63) / 64 - 1 : 0; }

static double small_us(const SmallShape& sh, const Layer& L, int64_t M, int S, int64_t tiles, int planes, int64_t share, int cus) {
    const int64_t wgs = tiles * planes, per_round = (int64_t)cus * sh.resident;
    const int64_t full = wgs / per_round, rest = wgs - full * per_round;
    const int64_t rounds = full + (rest > 0 ? 1 : 0);
    double t = sh.fixed + (double)full * sh.unit[sh.resident - 1] * (double)share + (double)rounds * sh.round + sh.out * (double)M * (double)L.N * 4e-6;
    if (rest > 0) t += sh.unit[(rest + cus - 1) / cus - 1] * (double)share;
    // the correction, by one plane of a tile
    const int64_t left = tiles % per_round, corr_rounds = tiles / per_round + (left > 0 ? 1 : 0);
    const int64_t on_cu = tiles / per_round * sh.resident + (left + cus - 1) / cus;
    t += more_pairs(L.kp) * ((double)corr_rounds * (sh.corr[0] + sh.corr[1] * (double)S) + (double)on_cu * (sh.tile[0] + sh.tile[1] * (double)S));
    if (planes > 1) t += sh.plane + sh.plane_mb * (double)planes * (double)M * (double)plane_ld(L.N) * 8e-6;
    return t;
}

static double pieces_us(const SmallPieces& c, const Layer& L, int S, const Split& sp) {
    const double rounds = (double)(sp.dp_tiles / sp.grid);
    double t = c.fixed + c.share * (double)sp.sk_share + rounds * (c.unit * (double)L.KT + c.round);
    if (sp.aligned) t += c.piece * (double)(sp.sk_tile_units / sp.sk_share - 2);
    return t + more_pairs(L.kp) * (rounds + 1.0) * (c.corr + c.slice * (double)S);
}

// S: partial sums of T.  part_bytes: room for planes (0: whole tiles only).  only: this shape of the staged kernel, in at
// least min_planes planes (id 0: not to be had).
static SmallPick pick_small(const Layer& L, int64_t M, int S, int64_t part_bytes, int cus, int only = 0, int min_planes = 1) {
    SmallPick best{0, 1, (int)L.KT, 0.0};
    const SmallShape* const table = L.w_bits == 4 ? kSmallShapes4 : kSmallShapes2;
    const int n_shapes = 5;
    for (int i = 0; i < n_shapes; ++i) {
        const SmallShape& sh = table[i];
        if (only != 0 && sh.id != only) continue;
        const int64_t tiles = ((M + sh.bm - 1) / sh.bm) * ((L.N + sh.bn - 1) / sh.bn);
        for (int p = min_planes; p <= kMaxPlanes && p <= L.KT; ++p) {
            const int64_t share = (L.KT + p - 1) / p;
            const int planes = (int)((L.KT + share - 1) / share);
            if (planes != p) continue;                       // the same planes as a smaller p
            if (p > 1 && (sh.bm == 128 || (int64_t)p * M * plane_ld(L.N) * 4 > part_bytes)) continue;
            const double us = small_us(sh, L, M, S, tiles, planes, share, cus);
            if (best.id == 0 || us < best.us) best = SmallPick{sh.id, planes, (int)share, us};
        }
        if (sh.id == 11 && part_bytes > 0) {
            const Split sp = split_tiles(tiles, L.KT, cus, true);
            if (sp.sk_units == 0 || (!sp.aligned && 2.0 * (double)M * (double)L.N * (double)L.K < kSharesFlops)) continue;
            const double us = pieces_us((sp.aligned ? kSmallWhole : kSmallShares)[L.w_bits == 4 ? 0 : 1], L, S, sp);
            if (us * (sp.aligned ? 1.0 : 1.03) < best.us) best = SmallPick{11, 0, (int)sp.sk_share, us};
        }
    }
    return best;
}

// CAN_SPLIT: the shape also exists in the form that walks a list of pieces
template <int WB, int TM, int TN, int WR, int WC, int NS, int MINW = 1, bool CAN_SPLIT = false>
static hipError_t launch_tiled_t(TiledArgs a, int64_t M, int mode, int cus, hipStream_t s) {
    constexpr int BM = 32 * TM * WR, BN = 32 * TN * WC;
    constexpr int LDS_BYTES = NS * BM * 128;
    a.grid_m = (int)((M + BM - 1) / BM);
    a.grid_n = (int)((a.N + BN - 1) / BN);
    a.group_m = 8;
    const int64_t tiles = (int64_t)a.grid_m * a.grid_n;
    TileShape me = {0, BM, BN, MINW, 1.0, 1.0, 1.0};
    for (const TileShape& sh : kShapes)
        if (sh.bm == BM && sh.bn == BN && sh.share == MINW) me = sh;
    static KernelSetup setup_split, setup_whole;
    // The split launches one workgroup per slot and its owners wait for workgroups with higher numbers: all of
    // them must be resident at once.  The number the runtime reports for this instance decides, not the launch
    // bounds; should it ever be lower than the shape assumes, tiles are not cut.
    bool can_split = CAN_SPLIT;
    if constexpr (CAN_SPLIT) {
        const hipError_t e = prepare_kernel(tiled_kernel<TM, TN, WR, WC, NS, MINW, true, WB>, setup_split, LDS_BYTES, 64 * WR * WC);
        if (e != hipSuccess) return e;
        if (setup_split.resident < MINW) can_split = false;
    }
    const int64_t slots = (int64_t)cus * MINW;
    // mode 0: split when the estimate says so; 1: never; 2: whenever there is a remainder to split; 3: the same, always in
    // equal shares of the remaining K tiles (never along tile boundaries); 4 (pick_small): as 2 where this instance can
    bool split = false;
    if (can_split && a.Part != nullptr && (int64_t)BM * BN * 4 * slots <= kTiledPartBytesPerCu * (int64_t)cus && slots <= kTiledFlags) {
        if (mode >= 2) split = true;
        else if (mode == 0) split = split_pays(me, tiles, a.KT, cus);
    }
    if ((mode == 2 || mode == 3) && !split) return hipErrorInvalidValue;      // asked for, not available
    const Split sp = split ? split_tiles(tiles, a.KT, slots, mode != 3) : whole_tiles(tiles, a.KT);
    a.dp_tiles = sp.dp_tiles; a.sk_units = sp.sk_units; a.sk_share = sp.sk_share; a.sk_tile_units = sp.sk_tile_units;
    if constexpr (CAN_SPLIT) {
        if (sp.sk_units > 0)
            return launch_kernel(tiled_kernel<TM, TN, WR, WC, NS, MINW, true, WB>, setup_split, LDS_BYTES, sp.grid, 64 * WR * WC, a, s);
    }
    return launch_kernel(tiled_kernel<TM, TN, WR, WC, NS, MINW, false, WB>, setup_whole, LDS_BYTES, tiles, 64 * WR * WC, a, s);
}

// staged_kernel on whole tiles, or on K planes and then their sum.
template <int WB, int TM, int TN, int WR, int WC, int MINW>
static hipError_t launch_staged_t(TiledArgs a, const SmallPick& pick, hipStream_t s) {
    constexpr int BM = 32 * TM * WR, BN = 32 * TN * WC, NW = WR * WC;
    constexpr int LDS_BYTES = 4 * (BM * 128 + NW * TN * 1280);
    a.grid_m = (int)((a.M + BM - 1) / BM);
    a.grid_n = (int)((a.N + BN - 1) / BN);
    a.dp_tiles = (int64_t)a.grid_m * a.grid_n;
    a.sk_share = pick.share;
    static KernelSetup setup_whole, setup_planes;
    if (pick.planes == 1)
        return launch_kernel(staged_kernel<TM, TN, WR, WC, MINW, false, WB>, setup_whole, LDS_BYTES, a.dp_tiles, 64 * NW, a, s);
    const hipError_t e = launch_kernel(staged_kernel<TM, TN, WR, WC, MINW, true, WB>, setup_planes, LDS_BYTES,
                                       a.dp_tiles * pick.planes, 64 * NW, a, s);
    if (e != hipSuccess) return e;
    return launch_reduce_planes(a, pick.planes, s);
}

template <int WB>
static hipError_t launch_staged(const TiledArgs& a, const SmallPick& pick, hipStream_t s) {
    switch (pick.id) {
        case 31: return launch_staged_t<WB, 2, 2, 1, 4, 2>(a, pick, s);      // 64 x 256, 72 KB: two workgroups per compute unit
        case 32: return launch_staged_t<WB, 2, 2, 1, 8, 2>(a, pick, s);      // 64 x 512, 112 KB
        default: return launch_staged_t<WB, 2, 1, 1, 4, 2>(a, pick, s);      // 64 x 128, 52 KB: two workgroups per compute unit
    }
}

__global__ void clear_flags_kernel(uint32_t* flags, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) flags[i] = 0u;
}

// For a tiled launch that does not follow the projection kernel (which clears the flags itself).
hipError_t launch_clear_flags(const Workspace& ws, hipStream_t s) {
    if (ws.flags == nullptr) return hipSuccess;
    hipLaunchKernelGGL(clear_flags_kernel, dim3((kTiledFlags + 255) / 256), dim3(256), 0, s, ws.flags, kTiledFlags);
    return hipGetLastError();
}

static std::atomic<int> g_wait_limit{1 << 22};
int tiled_wait_limit() { return g_wait_limit.load(); }
void set_tiled_wait_limit(int polls) { g_wait_limit.store(polls); }

int compute_units() {
    static int cus = 0;                                      // one kind of device per process
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cus = n;
    }
    return cus;
}

hipError_t launch_tiled(const Layer& L, int64_t M, const Workspace& ws, float* Y, int64_t ldy, const Requant& rq,
                        int variant, hipStream_t s) {
    if (M == 0) return hipSuccess;
    TiledArgs a;
    a.Wt = L.Wt; a.Bt = L.Bt; a.Xh = ws.Xh; a.ldxh = ws.ldxh; a.Y = Y; a.ldy = ldy;
    a.Yc = rq.codes; a.Ye = rq.exps; a.ldyc = rq.ld;
    a.Xt = ws.Xt; a.ldxt = ws.ldxt; a.Xe6 = nullptr;
    a.Tpart = ws.Tpart; a.S = ws.S; a.tp_stride = ws.tp_rows * L.kp;
    a.M = M; a.N = L.N; a.KT = L.KT; a.N32 = L.N32; a.kp = L.kp; a.kp16 = L.kp16;
    a.grid_m = a.grid_n = 0; a.group_m = 8;
    a.Part = ws.Part; a.flags = ws.flags;
    a.rec_bytes = L.w_rec_bytes; a.exp_bias = L.w_exp_bias;
    a.spin_limit = tiled_wait_limit();                       // by default about a second of polling
    a.dp_tiles = a.sk_units = 0; a.sk_share = 1; a.sk_tile_units = L.KT;
    const int cus = compute_units();
    // variant = 100 * mode + tile shape; mode 0 = split the work when the estimate says so, 1 = never, 2 = always,
    // 3 = always and in equal shares
    int mode = variant / 100;
    variant %= 100;
    if (mode < 0 || mode > 3) return hipErrorInvalidValue;
    if (ws.six) return launch_six(a, L, ws, mode, variant, cus, s);
    if (variant >= 31 && variant <= 33) {
        // a shape of the staged kernel by force: 0 = planes when the estimate says so, 1 = whole tiles, 2 = planes
        if (mode == 3) return hipErrorInvalidValue;
        const int64_t part_bytes = (mode != 1 && ws.Part != nullptr) ? kTiledPartBytesPerCu * (int64_t)cus : 0;
        const SmallPick pick = pick_small(L, M, ws.S, part_bytes, cus, variant, mode == 2 ? 2 : 1);
        if (pick.id == 0) return hipErrorInvalidValue;       // one K tile, or no room: no planes
        return L.w_bits == 4 ? launch_staged<4>(a, pick, s) : launch_staged<2>(a, pick, s);
    }
    if (variant == 0 && mode <= 1 && 2.0 * (double)M * (double)L.N * (double)L.K <= kSmallFlops) {
        const int64_t part_bytes = (mode == 0 && ws.Part != nullptr) ? kTiledPartBytesPerCu * (int64_t)cus : 0;
        const SmallPick pick = pick_small(L, M, ws.S, part_bytes, cus);
        if (pick.id > 12) return L.w_bits == 4 ? launch_staged<4>(a, pick, s) : launch_staged<2>(a, pick, s);
        variant = pick.id;                                   // the launches below: tiles whole, or cut if the instance can
        mode = pick.planes == 0 ? 4 : 1;
    }
    if (variant == 0) {
        // pick the tile shape (and the split) with the lowest estimated time
        double best = 0.0;
        for (const TileShape& entry : kShapes) {
            TileShape sh = entry;
            int64_t KT = L.KT;
            if (L.w_bits == 2) {
                // the 2-bit instances against the table's 4-bit rates, and the correction's extra K columns, which at the
                // ranks such layers come with are no longer small (measured on 4096 x 4096 at 2048 tokens and rank 256:
                // 128 x 512 cut along K 103 us, 128 x 256 114 us, 128 x 128 113 us)
                const double f = sh.id == 11 ? 0.85 : 0.7;
                sh.pair *= f; sh.single *= f; sh.cut *= f;
                KT += (2 * L.kp + kTileK - 1) / kTileK;
            }
            const int64_t tiles = ((M + sh.bm - 1) / sh.bm) * ((L.N + sh.bn - 1) / sh.bn);
            double t = time_whole(sh, tiles, KT, cus);
            if (mode >= 2 && ws.Part != nullptr) t = time_split(sh, tiles, KT, cus);
            else if (mode == 0 && ws.Part != nullptr && split_pays(sh, tiles, KT, cus)) t = time_split(sh, tiles, KT, cus);
            if (variant == 0 || t < best) { best = t; variant = sh.id; }
        }
    }
    if (L.w_bits == 2) {
        // 2-bit weights: the three shapes the automatic choice uses
        switch (variant) {
            case 4: return launch_tiled_t<2, 2, 2, 2, 2, 4, 2, true>(a, M, mode, cus, s);
            case 11: return launch_tiled_t<2, 4, 2, 1, 8, 4, 1, true>(a, M, mode, cus, s);
            case 12: return launch_tiled_t<2, 4, 2, 1, 4, 4, 2, true>(a, M, mode, cus, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (variant) {
        case 1: return launch_tiled_t<4, 4, 4, 2, 2, 4>(a, M, mode, cus, s);      // 256 x 256
        case 3: return launch_tiled_t<4, 2, 4, 2, 2, 4>(a, M, mode, cus, s);      // 128 x 256
        case 4: return launch_tiled_t<4, 2, 2, 2, 2, 4, 2, true>(a, M, mode, cus, s);   // 128 x 128, two workgroups per compute unit
        case 7: return launch_tiled_t<4, 2, 4, 2, 4, 4>(a, M, mode, cus, s);      // 128 x 512, eight wavefronts
        case 8: return launch_tiled_t<4, 2, 4, 2, 2, 4, 2>(a, M, mode, cus, s);   // 128 x 256, two workgroups per compute unit
        case 11: return launch_tiled_t<4, 4, 2, 1, 8, 4, 1, true>(a, M, mode, cus, s);     // 128 x 512, eight wavefronts, each 128 x 64
        case 12: return launch_tiled_t<4, 4, 2, 1, 4, 4, 2, true>(a, M, mode, cus, s);  // 128 x 256, four wavefronts each 128 x 64, two workgroups per compute unit
        case 13: return launch_tiled_t<4, 4, 2, 1, 4, 4>(a, M, mode, cus, s);     // 128 x 256, four wavefronts each 128 x 64
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lqer
