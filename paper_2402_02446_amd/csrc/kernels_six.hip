// Stage 2, large M, on fp6 operands: the form of the main product (Eq. 3 / Eq. 6) that layers with a correction mostly take
// (tiled_takes_six).  An 8-bit activation code in two halves against the 4-bit code, exact, two products on the block-scaled fp6
// MFMA (mfma32_six) for one of codes; 2-bit codes as fp4 (mfma32_four), from their records as they are.
//
// Workgroup tile 32 TM rows x 32 TN NW columns, NW wavefronts side by side, each all the rows of 32 TN columns: TM x TN tiles of the
// 32x32x64 MFMA.  The contraction axis is walked in chunks of 64, two MFMA steps: lane (i = lane % 32, hh = lane / 32) owns block 2 hh + s
// of a chunk in step s, for row or column i of every operand.  Activations (images, ready operands), packed weights and exponents go from memory
// to LDS by direct loads, a chunk in four stages; weights are expanded in registers (14 instructions an operand), each for TM MFMAs.
// A stage takes its next chunk as soon as every wavefront has its operands in registers: behind the barrier that also says the following chunk
// has landed, one a chunk, so a load has three chunks' time.
// The rank-kp correction, T_hi and T_lo against B_k on the 32x32x16 bf16 MFMA, is summed by itself and added once where the tile's
// sums take a wavefront's registers (CHAINS = 1): an fp32 chain rounds at the size its sum has reached, and the product of fp6 operands
// mostly is exact up to the end.  T waits in LDS from the start, B_k is asked for ahead of the last chunk.  Smaller tiles sum two
// chains - the correction and the first half of K, the second half.
//
// Work split: whole tiles; K planes, whose partial sums reduce_planes_kernel adds; or pieces handed from one workgroup to another as
// in tiled_kernel (kernels_tiled.hip says how).
#include <type_traits>

#include "lqer_internal.h"
#include "mx_device.h"
#include "tiled_common.h"

namespace lqer {

// lds_dma16 by the wavefronts below BELOW, and staged_wait with a count of theirs and one of the others'.  (Branches inside one statement: the
// compiler's own would cut the loop's blocks, and cost it copies of what lives across them.)
template <int ADD, int BELOW>
__device__ __forceinline__ void lds_dma16_below(int wave, uint32_t at, uint32_t off, const uint8_t* base) {
    asm volatile("s_cmp_ge_u32 %4, %5\n\ts_cbranch_scc1 .Lsix_issue%=\n\ts_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n.Lsix_issue%=:"
                 ::"s"(at), "v"(off), "s"(base), "n"(ADD), "s"(wave), "n"(BELOW) : "memory", "scc");
}
template <int LEFT, int OTHERS, int BELOW>
__device__ __forceinline__ void staged_wait_by(int wave) {
    static_assert(LEFT < 64 && OTHERS < 64, "a 6-bit counter");
    asm volatile("s_cmp_ge_u32 %2, %3\n\ts_cbranch_scc1 .Lsix_other%=\n\ts_waitcnt vmcnt(%0)\n\ts_branch .Lsix_done%=\n.Lsix_other%=:\n\ts_waitcnt vmcnt(%1)\n"
                 ".Lsix_done%=:\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(LEFT), "n"(OTHERS), "s"(wave), "n"(BELOW) : "memory", "scc");
}

enum { kWhole = 0, kPlanes = 1, kPieces = 2 };

// LDS of a workgroup: four stages of activations and weights, the exponent bytes of a K tile (activations, weights), T of 64 ranks - in the last
// two stages' memory where two workgroups share a compute unit (their correction comes first).
template <int TM, int TN, int NW, int BITS>
struct SixLds {
    static constexpr bool OVER = NW == 4;
    static constexpr int XB = TM * 3072, WB = NW * TN * 1024;                  // a stage
    static constexpr int SX = OVER ? XB + WB : XB, SW = OVER ? XB + WB : WB;   // from one stage to the next
    static constexpr int W_AT = OVER ? XB : 4 * XB;
    static constexpr int XE_AT = 4 * (XB + WB), WE_AT = XE_AT + TM * 512, WE = BITS == 4 ? 512 : 256;     // WE: exponents of a column group
    static constexpr int T_AT = OVER ? 2 * (XB + WB) : WE_AT + NW * TN * WE;
    static constexpr int BYTES = OVER ? WE_AT + NW * TN * WE : T_AT + TM * 8192;
    static_assert(!OVER || 2 * (XB + WB) >= TM * 8192, "T fits two stages");
    static_assert(BYTES <= (OVER ? 80 : 159) * 1024, "one workgroup per compute unit, or two");
};

// What bounds it.  On a full chip the clock, that is, energy: 3.7 us per K tile of 128 x 512 with the values of a product, 2.6 with
// activations of zero, at 1.45 and 2.0 GHz, where the bare MFMA loop's rate would be 2.6; 8 % fewer cycles (5820 to 5330, a chunk's loads
// in three parts instead of one) gave 1 % of time.  Taken out one at a time, the loads cost 9 %, the expansion 8, the reads of activations
// and the barrier 6 each.  On a chip that is not full it is neither: the matrix units are busy for a tenth of 203 tokens of 4112 x 11000 and the vector
// port for a quarter, waits for memory and LDS take a third, and three workgroups on a unit are no faster per K tile than two; what they
// share is not shown yet.  The shape: a block-scaled MFMA holds the vector port for 16 cycles whatever its shape
// (loops of MFMAs with n vector instructions behind each: 32x32x64 max(32, 16 + 4 n) cycles, 16x16x128 16 + 4 n, of 16 bare), so that of the
// two shapes only this one leaves room for the expansion, 3.5 instructions per MFMA where a wavefront has 128 rows.  (With 16x16x128 MFMAs,
// whose bare loop is the faster by 13 % on such operands: 7660 cycles and 4.1 us.)
// Whole calls, operands through registers and the correction's behind the last chunk -> this: 8192 x 28672 rank 64 at 4096 tokens
// 1108 -> 981 us, 11008 x 4096 rank 32 at 2048 154 -> 136, three layers of 4096 x 4096 rank 32 at 8192 587 -> 534, 4112 x 11000 rank 24
// at 203 33.5 -> 32.0.  Distance from the 64-bit result as before: 2.5e-7, 2.4e-7, 2.2e-7, 2.1e-7.
template <int TM, int TN, int NW, int CHAINS, int MODE, int BITS>
__global__ __launch_bounds__(64 * NW, 2) void six_kernel(TiledArgs a) {
    constexpr int BM = 32 * TM, NT = 64 * NW;
    typedef SixLds<TM, TN, NW, BITS> Lds;
    static_assert(BITS == 4 || BITS == 2, "fp6 records, or the 2-bit ones with exponent nibbles");
    constexpr int REC = BITS == 4 ? kW6RecordBytes : w_record_bytes(2, true), CODES = BITS == 4 ? 0 : kWCompactCodeOffset;
    constexpr int EG = BITS == 4 ? 2 : 4;          // column groups whose exponents a load of 1 KiB brings
    constexpr int XB = Lds::XB, WB = Lds::WB, SX = Lds::SX, SW = Lds::SW;
    constexpr int XF = XB / 1024 / NW, XR = XB / 1024 % NW;    // 1 KiB pieces of a stage: every wavefront's, and how many wavefronts take one more
    constexpr int L = XF + TN;                     // loads of a wavefront per chunk (one more in the first XR), and with a K tile's first chunk ...
    constexpr int LE = 2;                          // ... the exponents
    static_assert((TM == 4 || TM == 2) && (TN == 2 || TN == 1) && (NW == 8 || NW == 4) && XF <= 3, "issue() spells the pieces out");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ int wait_ok;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lane = tid & 63;
    // workgroup -> position: consecutive positions land on one XCD
    int lin;
    {
        const int nwg = gridDim.x, pid = blockIdx.x;
        const int xcd = pid & 7, local = pid >> 3, per = nwg >> 3, rem = nwg & 7;
        lin = (xcd < rem) ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
    }
    const int KT = (int)a.KT;
    const int64_t tile_stride = a.N32 * REC;
    constexpr bool XE4 = NW * 256 >= TM * 512;     // exponents of the activations: 256 B from each wavefront, or 1 KiB
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)lds);
    const uint32_t at_x = lds0 + wave * 1024, at_w = lds0 + Lds::W_AT + wave * (TN * 1024);
    const uint32_t at_xe = lds0 + Lds::XE_AT + (XE4 ? wave % (2 * TM) * 256 : (wave & 1) * 1024);
    const uint32_t at_we = lds0 + Lds::WE_AT + wave * TN / EG * 1024;
    uint32_t rd16 = lane * 16, rdw = Lds::W_AT + wave * (TN * 1024) + lane * 16;

    int64_t dp_next = lin;                         // kPieces: the next whole tile of this workgroup, and its range of the shared K tiles
    int64_t u = MODE == kPieces ? a.sk_share * lin : 0;
    int64_t u_end = u + a.sk_share;
    if (u_end > a.sk_units) u_end = a.sk_units;
    bool first_piece = true;
  for (;;) {
    int64_t tile_lin = lin;
    int kt0 = 0, kt1 = KT, plane = 0;
    if constexpr (MODE == kPlanes) {
        // neighbouring workgroups of one XCD: neighbouring tiles of the same K range, which share activations or weights
        plane = lin / (int)a.dp_tiles;
        tile_lin = lin - plane * (int)a.dp_tiles;
        kt0 = plane * (int)a.sk_share;
        kt1 = kt0 + (int)a.sk_share < KT ? kt0 + (int)a.sk_share : KT;
    } else if constexpr (MODE == kPieces) {
        // the shared K tiles first: the hand-over then overlaps with the whole tiles of other workgroups
        if (u < u_end) {
            const int64_t rt = u / a.sk_tile_units;
            tile_lin = a.dp_tiles + rt;
            kt0 = (int)(u - rt * a.sk_tile_units);
            const int64_t left = u_end - u;
            if (kt0 >= KT) {                       // only empty units of this tile are left
                u += (left < a.sk_tile_units - kt0) ? left : a.sk_tile_units - kt0;
                continue;
            }
            kt1 = (left < (int64_t)(KT - kt0)) ? kt0 + (int)left : KT;
            u += (kt1 == KT) ? a.sk_tile_units - kt0 : kt1 - kt0;
            if (u > u_end) u = u_end;
        } else if (dp_next < a.dp_tiles) {
            tile_lin = dp_next;
            dp_next += gridDim.x;
        } else {
            break;
        }
        if (!first_piece) __syncthreads();         // every wavefront is done with the LDS stages
        first_piece = false;
    }
    const bool owner = MODE == kWhole || kt0 == 0; // this piece adds the correction (and stores the tile, unless a plane)
    int tile_m, tile_n;                            // bands of group_m tile rows
    {
        const int64_t width = (int64_t)a.group_m * a.grid_n;
        const int grp = (int)(tile_lin / width), in = (int)(tile_lin - grp * width), first_m = grp * a.group_m;
        const int gsize = (a.grid_m - first_m < a.group_m) ? a.grid_m - first_m : a.group_m;
        tile_m = first_m + in % gsize;
        tile_n = in / gsize;
    }
    const int64_t m0 = (int64_t)tile_m * BM;
    const int64_t n_first = (int64_t)tile_n * (NW * TN);       // first column group of the tile
    const int64_t g0 = n_first + wave * TN;                    // first column group of this wavefront
    auto clamped = [&](int64_t g) { return g < a.N32 ? g : a.N32 - 1; };       // (the store is masked)

    // ---- loads -----------------------------------------------------------------------------------------------------------------
    // Rows past M are workspace rows and hold whatever was there; they reach only their own row of Y.
    const int img = TM == 4 ? tile_m : tile_m >> 1, half = TM == 4 ? 0 : tile_m & 1;
    const uint8_t* x_ptr = reinterpret_cast<const uint8_t*>(a.Xh) + ((int64_t)img * KT + kt0) * (4 * kX6Chunk);
    const uint8_t* xe_ptr = a.Xe6 + ((int64_t)img * KT + kt0) * kX6Scales + half * 1024 + (XE4 ? wave % (2 * TM) * 256 : (wave & 1) * 1024);
    const int64_t g_first = clamped(g0);
    const uint8_t* w_ptr = a.Wt + g_first * REC + (int64_t)kt0 * tile_stride;
    const int64_t w_second = (clamped(g0 + 1) - g_first) * REC;
    // piece p of a stage, in the image: all of it, or the tile's half of each of its four runs
    auto piece = [&](int p) {
        if (TM == 4) return p * 1024;
        return p < 4 ? (p >> 1) * 4096 + (2 * half + (p & 1)) * 1024 : 8192 + (p - 4) * 2048 + half * 1024;
    };
    x_ptr += piece(wave);
    const int x_second = piece(wave + NW) - piece(wave);
    // exponents of EG neighbouring column groups, this wavefront's among them
    const int64_t ge = n_first + wave * TN / EG * EG;
    const int64_t ge_first = clamped(ge);
    const int64_t ge_rel = (ge_first - g_first) * REC;
    uint32_t we_off = (uint32_t)(clamped(ge + lane / (64 / EG)) - ge_first) * REC + (BITS == 4 ? kWExpOffset : 0) + lane % (64 / EG) * 16;
    // (Opaque, so that addresses are one scalar and one of these each: left alone, sums of them take the registers of the product.)
    asm volatile("" : "+v"(we_off), "+v"(rd16), "+v"(rdw));
    // The next chunk, number CC of its K tile -> stage CC, in three parts: a chunk's loads in one go would queue up, and the wavefronts behind them.
    auto issue_part = [&](auto cc, auto pp) {
        constexpr int CC = decltype(cc)::value, P = decltype(pp)::value;
        if constexpr (P == 0) {
            if constexpr (XF > 0) lds_dma16<CC * SX>(at_x, rd16, x_ptr);
            if constexpr (XF > 1) lds_dma16<CC * SX + NW * 1024>(at_x, rd16, x_ptr + NW * 1024);
        }
        if constexpr (P == 1) {
            if constexpr (XF > 2) lds_dma16<CC * SX + 2 * NW * 1024>(at_x, rd16, x_ptr + 2 * NW * 1024);
            if constexpr (XR > 0) lds_dma16_below<CC * SX + XF * NW * 1024, XR>(wave, at_x, rd16, XF == 1 ? x_ptr + x_second : x_ptr);
            lds_dma16<CC * SW>(at_w, rd16, w_ptr + CODES + (BITS == 4 ? CC : CC >> 1) * 1024);
            x_ptr += kX6Chunk;
        }
        if constexpr (P == 2) {
            if constexpr (TN == 2) lds_dma16<CC * SW + 1024>(at_w, rd16, w_ptr + CODES + (BITS == 4 ? CC : CC >> 1) * 1024 + w_second);
            if constexpr (CC == 0) {
                if constexpr (XE4) lds_dma4<0>(at_xe, rd16 >> 2, xe_ptr);
                else lds_dma16<0>(at_xe, rd16, xe_ptr);
                lds_dma16<0>(at_we, we_off, w_ptr + ge_rel);
                xe_ptr += kX6Scales;
            }
            if constexpr (CC == 3) w_ptr += tile_stride;
        }
    };
    constexpr std::integral_constant<int, 0> C0{};
    constexpr std::integral_constant<int, 1> C1{};
    constexpr std::integral_constant<int, 2> C2{};
    constexpr std::integral_constant<int, 3> C3{};
    auto issue = [&](auto cc) {
        issue_part(cc, C0);
        issue_part(cc, C1);
        issue_part(cc, C2);
    };
    static_assert(XF <= 1 || TM == 4, "pieces beyond the second are those of whole images");
    // All loads but those of this wavefront's newest CHUNKS chunks (E: with exponents among them) have landed, and everybody's.
    auto arrive = [&](auto chunks, auto e) {
        constexpr int C = decltype(chunks)::value, E = decltype(e)::value * LE;
        if constexpr (XR > 0) staged_wait_by<C * (L + 1) + E, C * L + E, XR>(wave);
        else staged_wait<C * L + E>();
    };
    f32x16 acc[CHAINS][TM][TN];

    // ---- rank-kp correction ----------------------------------------------------------------------------------------------------
    // 64 ranks a round: T as [row][T_hi of eight octets of ranks | T_lo of them], 16-byte cells XOR-ed with the row; B_k's codes and
    // exponents, of ranks 16 b + 8 hh .. + 7 and this lane's column of a group, in registers.
    const int rounds = owner ? (a.kp + 63) / 64 : 0;
    constexpr int TI = BM * 8 / NT;                // octets of T a thread brings
    auto t_item = [&](int j, int& row, int& oct) {
        const int item = tid + j * NT;
        row = item >> 3;
        oct = item & 7;
    };
    // an octet's two bf16 terms -> its cells.  (Those behind the last rank repeat the first.)
    auto put_octet = [&](int row, int oct, u32x4 hi, u32x4 lo) {
        *reinterpret_cast<u32x4*>(lds + Lds::T_AT + row * 256 + ((oct ^ (row & 15)) << 4)) = hi;
        *reinterpret_cast<u32x4*>(lds + Lds::T_AT + row * 256 + (((8 + oct) ^ (row & 15)) << 4)) = lo;
    };
    auto put_sums = [&](int row, int oct, const f32x4& q0, const f32x4& q1) {
        u32x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t h[2], l[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const float v = e < 2 ? q0[2 * e + k] : q1[2 * (e - 2) + k];
                h[k] = f32_bits(v) & 0xFFFF0000u;
                l[k] = f32_bits(v - f32_from_bits(h[k]));
            }
            hi[e] = (h[0] >> 16) | h[1];
            lo[e] = (l[0] >> 16) | (l[1] & 0xFFFF0000u);
        }
        put_octet(row, oct, hi, lo);
    };
    // T final, or as up to two fp32 partial sums: all of a thread's loads, and later its stores
    struct TSet { f32x4 p0[TI][2], p1[TI][2]; };   // final: [0] are the bits of T_hi, T_lo
    auto fetch_t = [&](TSet& t, int round) {
#pragma unroll
        for (int j = 0; j < TI; ++j) {
            int row, oct;
            t_item(j, row, oct);
            const int r0 = round * 64 + oct * 8 < a.kp ? round * 64 + oct * 8 : 0;
            if (a.S <= 1) {
                const uint16_t* src = a.Xt + (m0 + row) * a.ldxt + r0;
                t.p0[j][0] = *reinterpret_cast<const f32x4*>(src);
                t.p1[j][0] = *reinterpret_cast<const f32x4*>(src + a.kp);
            } else {
                const float* src = a.Tpart + (m0 + row) * a.kp + r0;
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    t.p0[j][sl] = *reinterpret_cast<const f32x4*>(src + sl * a.tp_stride);
                    t.p1[j][sl] = *reinterpret_cast<const f32x4*>(src + sl * a.tp_stride + 4);
                }
            }
        }
    };
    auto put_t = [&](TSet& t) {
#pragma unroll
        for (int j = 0; j < TI; ++j) {
            int row, oct;
            t_item(j, row, oct);
            if (a.S <= 1) put_octet(row, oct, __builtin_bit_cast(u32x4, t.p0[j][0]), __builtin_bit_cast(u32x4, t.p1[j][0]));
            else put_sums(row, oct, t.p0[j][0] + t.p0[j][1], t.p1[j][0] + t.p1[j][1]);
        }
    };
    // more partial sums (few rows): added in slice order, an octet's all in flight together
    auto sum_t = [&](int round) {
        for (int j = 0; j < TI; ++j) {
            int row, oct;
            t_item(j, row, oct);
            const int r0 = round * 64 + oct * 8 < a.kp ? round * 64 + oct * 8 : 0;
            const float* src = a.Tpart + (m0 + row) * a.kp + r0;
            f32x4 p0[8], p1[8];
#pragma unroll
            for (int sl = 0; sl < 8; ++sl) {
                const int64_t o = (int64_t)(sl < a.S ? sl : a.S - 1) * a.tp_stride;
                p0[sl] = *reinterpret_cast<const f32x4*>(src + o);
                p1[sl] = *reinterpret_cast<const f32x4*>(src + o + 4);
            }
#pragma unroll
            for (int sl = 1; sl < 8; ++sl)
                if (sl < a.S) { p0[0] += p0[sl]; p1[0] += p1[sl]; }
            put_sums(row, oct, p0[0], p1[0]);
        }
    };
    auto bring_t = [&](int round) {
        if (a.S > 2) {
            sum_t(round);
        } else {
            TSet t;
            fetch_t(t, round);
            put_t(t);
        }
    };
    struct BSet { u32x2 c[4]; uint32_t e[4]; };    // of one column group
    auto load_b = [&](BSet& b, int tn, int round) {
        uint32_t l = rd16 >> 4;
        asm volatile("" : "+v"(l));
        const uint32_t off = (l & 31) * 16 + (l >> 5) * 8, eoff = 512 + (l & 31);
        const uint8_t* first = a.Bt + clamped(g0 + tn) * a.kp16 * kBRecordBytes;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int blk = 4 * round + j < a.kp16 ? 4 * round + j : a.kp16 - 1;
            b.c[j] = *reinterpret_cast<const u32x2*>(first + blk * kBRecordBytes + off);
            b.e[j] = first[blk * kBRecordBytes + eoff];
        }
    };
    // T B_k of the round's ranks and a column group, on top of `sum`, a tile
    struct BFrag { Frag f[4]; };
    auto expand_b = [&](BFrag& o, const BSet& b, int live) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float sc = h_scale(b.e[j]);
            const uint32_t keep = (uint32_t)((j - live) >> 31);                  // (T holds other ranks behind its last.  A mask: a branch costs the registers.)
            const u32x2 lo = int8x4_to_bf16(b.c[j][0] & keep, sc), hi = int8x4_to_bf16(b.c[j][1] & keep, sc);
            o.f[j].u = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    };
    // (Half a round or a whole one, without branches: B_k is zero behind its last rank.)
    auto correct = [&](f32x16& sum, const BFrag& b, int tm, auto blocks) {
        uint32_t l = rd16 >> 4;
        asm volatile("" : "+v"(l));
        const uint8_t* base = lds + Lds::T_AT + (l & 31) * 256 + tm * 8192;
        const uint32_t cell = ((l >> 5) ^ (l & 15)) << 4;
        constexpr int STEPS = 2 * decltype(blocks)::value;
        auto read_t = [&](int k) { return *reinterpret_cast<const u32x4*>(base + (cell ^ ((8 * (k & 1) + 2 * (k >> 1)) << 4))); };
        Frag t[2];
        t[0].u = read_t(0);
        t[1].u = read_t(1);
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            sum = mfma32(b.f[k >> 1].v, t[k & 1].v, sum);
            if (k + 2 < STEPS) t[k & 1].u = read_t(k + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // T of the first 64 ranks, for the correction behind the product: where it is final, by direct loads as well, ahead of everything else so
    // that the counts below are of what follows.  (Cells behind the last rank repeat the first.)
    if (CHAINS == 1 && a.S <= 1 && owner) {
#pragma unroll
        for (int j = 0; j < TM * 8 / NW; ++j) {
            const int piece_t = wave * (TM * 8 / NW) + j, row = piece_t * 4 + (lane >> 4), cell = (lane & 15) ^ (row & 15), r0 = (cell & 7) * 8;
            lds_dma16<Lds::T_AT>(lds0 + piece_t * 1024, (uint32_t)((row * (int)a.ldxt + (r0 < a.kp ? r0 : 0) + (cell >> 3) * a.kp) * 2),
                                 reinterpret_cast<const uint8_t*>(a.Xt + m0 * a.ldxt));
        }
    }
    // Everything asked for at once.  (What arrives in registers is waited for with all loads behind it.)
    const bool t_in_registers = owner && a.S <= 2 && !(CHAINS == 1 && a.S <= 1);
    TSet t_first;
    BSet b_first[TN];
    if (t_in_registers) fetch_t(t_first, 0);
    if (CHAINS == 2 && owner) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) load_b(b_first[tn], tn, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    issue(C0);
    issue(C1);
    if constexpr (!Lds::OVER) {
        issue(C2);
        issue(C3);
    }
    if (t_in_registers) put_t(t_first);
    else if (owner && a.S > 2) sum_t(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < CHAINS; ++h)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[h][tm][tn][r] = 0.f;
    if constexpr (CHAINS == 2) {
        for (int r = 0; r < rounds; ++r) {
            if (r > 0) {
                __syncthreads();                   // T has been read by everybody
                if (a.S <= 2) put_t(t_first);
                else sum_t(r);
            }
            __syncthreads();
            BFrag bf[TN];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) expand_b(bf[tn], b_first[tn], a.kp16 - 4 * r);
            if (r + 1 < rounds) {                  // the next round's operands, beside this one's arithmetic
                if (a.S <= 2) fetch_t(t_first, r + 1);
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) load_b(b_first[tn], tn, r + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) correct(acc[0][tm][tn], bf[tn], tm, std::integral_constant<int, 4>{});
        }
    }
    if constexpr (Lds::OVER) {
        if (rounds > 0) __syncthreads();           // T has been read by everybody
        issue(C2);
        issue(C3);
    }

    // ---- main product ----------------------------------------------------------------------------------------------------------
    // Two MFMA steps of 32 to a chunk.  Operands are read a chunk ahead, into the registers of those just used; so is what a lane
    // has of the weights' codes, and of the exponents, in a K tile's last chunk.
    typedef typename std::conditional<BITS == 4, u32x6, u32x4>::type WOp;      // a weight operand, and what it is made of
    typedef typename std::conditional<BITS == 4, u32x4, u32x2>::type WRaw;
    u32x6 x[2][TM];
    WOp w;
    u32x2 xe[TM], we[TN];                          // we: byte 2c + s of eight as in xe; BITS = 2: byte c of word s
    WRaw raw[TN];
    auto read_x = [&](int stage, int s, int tm) {
        const u32x4 p = *reinterpret_cast<const u32x4*>(lds + rd16 + (stage * SX + (s * TM + tm) * 1024));
        const u32x2 h = *reinterpret_cast<const u32x2*>(lds + (rd16 >> 1) + (stage * SX + TM * 2048 + (s * TM + tm) * 512));
        return u32x6{p[0], p[1], p[2], p[3], h[0], h[1]};
    };
    // (2 bits: a stage holds two chunks' codes)
    auto read_raw = [&](int stage, int tn) { return *reinterpret_cast<const WRaw*>(lds + rdw + (stage * SW + tn * 1024 + (BITS == 4 ? 0 : (stage & 1) * 8))); };
    auto read_xe = [&](int tm) { return *reinterpret_cast<const u32x2*>(lds + Lds::XE_AT + (rd16 >> 1) + tm * 512); };
    const uint32_t bias4 = (uint32_t)(a.exp_bias - 2) * 0x01010101u;           // BITS = 2 (see expand_four)
    auto read_we = [&](int tn) {
        const uint8_t* at = lds + Lds::WE_AT + (wave * TN + tn) * Lds::WE;
        if constexpr (BITS == 4) {
            return *reinterpret_cast<const u32x2*>(at + (rd16 >> 1));
        } else {
            const uint32_t v = *reinterpret_cast<const uint32_t*>(at + (rd16 >> 2));
            return u32x2{(v & 0x0F0F0F0Fu) + bias4, ((v >> 4) & 0x0F0F0F0Fu) + bias4};
        }
    };
    auto expand = [&](const WRaw& v, auto ss) {
        if constexpr (BITS == 4) return expand_six<decltype(ss)::value>(v);
        else return expand_four(v[decltype(ss)::value]);
    };
    BSet b_last;                                   // CHAINS = 1: B_k for the correction, asked for in the middle of the last chunk
    // Chunk CC of its K tile.  On entry x, raw and w, the first step's and column group's weights, are its own; on exit the next chunk's.  more:
    // there is a K tile behind this one.
    auto chunk = [&](f32x16 (&sum)[TM][TN], auto cc, auto more) {
        constexpr int CC = decltype(cc)::value;
        constexpr bool MORE = decltype(more)::value, NEXT = MORE || CC < 3;
        constexpr int NS = (CC + 1) & 3;
        WRaw rawn;
        u32x2 wen;
        auto phase = [&](auto ss, auto nn) {
            constexpr int S = decltype(ss)::value, N = decltype(nn)::value, BYTE = (2 * CC + S) & 3;
            constexpr bool LAST = N == TN - 1;
            if constexpr (NEXT && S == 0 && LAST) {
                // the next chunk has landed, and this one's stage has been read by everybody
                if constexpr (MORE) arrive(C2, std::integral_constant<int, CC == 1 || CC == 2>{});
                else arrive(std::integral_constant<int, CC < 2 ? 2 - CC : 0>{}, C0);
            }
            if constexpr (MORE && TN == 2 && (S == 1 || N == 1)) {
                issue_part(cc, std::integral_constant<int, S + N - (S == 0)>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (MORE && TN == 1) {
                if constexpr (S == 0) issue_part(cc, C0);
                else { issue_part(cc, C1); issue_part(cc, C2); }
                __builtin_amdgcn_sched_barrier(0);
            }
            int reads = 0;
            if constexpr (TN == 2) {
                if constexpr (NEXT && S == 1) { raw[N] = read_raw(NS, N); reads = 1; }
                if constexpr (NEXT && CC == 3 && S == 1 && N == 1) { we[0] = read_we(0); reads = 2; }
                if constexpr (CC == 0 && S == 0 && N == 0) { we[1] = read_we(1); reads = 1; }
            } else {
                if constexpr (NEXT && S == 0) { rawn = read_raw(NS, 0); reads = 1; }
                if constexpr (NEXT && CC == 3 && S == 1) { wen = read_we(0); reads = 1; }
            }
            if (reads == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            else if (reads == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            const WOp now = w;
            if constexpr (!LAST) w = expand(raw[TN - 1], ss);
            else if constexpr (S == 0) w = expand(raw[0], C1);
            else if constexpr (NEXT) w = expand(TN == 2 ? raw[0] : rawn, C0);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                if constexpr (BITS == 4) sum[tm][N] = mfma32_six<BYTE>(now, x[S][tm], sum[tm][N], we[N][CC >> 1], xe[tm][CC >> 1]);
                else sum[tm][N] = mfma32_four<CC, BYTE>(now, x[S][tm], sum[tm][N], we[N][S], xe[tm][CC >> 1]);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if constexpr (NEXT && LAST) {
                    x[S][tm] = read_x(NS, S, tm);
                    if constexpr (CC == 3 && S == 1) {
                        xe[tm] = read_xe(tm);
                        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                    } else {
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    }
                }
                __builtin_amdgcn_sched_group_barrier(0x002, TM == 4 ? 4 : 7, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        phase(C0, C0);
        if constexpr (TN == 2) phase(C0, C1);
        if constexpr (CHAINS == 1 && !NEXT) {
            load_b(b_last, 0, 0);                  // (into the registers of the first step's activations)
            __builtin_amdgcn_sched_barrier(0);
        }
        phase(C1, C0);
        if constexpr (TN == 2) phase(C1, C1);
        if constexpr (TN == 1 && NEXT) {
            raw[0] = rawn;
            if constexpr (CC == 3) we[0] = wen;
        }
    };
    arrive(C3, C0);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        raw[tn] = read_raw(0, tn);
        we[tn] = read_we(tn);
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        x[0][tm] = read_x(0, 0, tm);
        x[1][tm] = read_x(0, 1, tm);
        xe[tm] = read_xe(tm);
    }
    w = expand(raw[0], C0);
    auto tile = [&](f32x16 (&sum)[TM][TN], auto more) {
        chunk(sum, C0, more);
        chunk(sum, C1, more);
        chunk(sum, C2, more);
        chunk(sum, C3, more);
    };
    const int tiles = kt1 - kt0, first_half = (tiles + 1) / 2;
    int kt = 0;
    if constexpr (CHAINS == 2) {
        for (; kt < first_half && kt + 1 < tiles; ++kt) tile(acc[0], std::true_type{});
    }
    for (; kt + 1 < tiles; ++kt) tile(acc[CHAINS - 1], std::true_type{});
    tile(acc[CHAINS - 1], std::false_type{});
    if constexpr (CHAINS == 2) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[0][tm][tn][r] += acc[1][tm][tn][r];
    } else {
        auto add_round = [&](auto blocks, int r) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                BFrag bf;
                expand_b(bf, b_last, a.kp16 - 4 * r);
                if (tn + 1 < TN) load_b(b_last, tn + 1, r);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    f32x16 corr;
#pragma unroll
                    for (int q = 0; q < 16; ++q) corr[q] = 0.f;
                    correct(corr, bf, tm, blocks);
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[0][tm][tn][q] += corr[q];
                    asm volatile("" : "+v"(acc[0][tm][tn]));       // (here, not in a block behind: the sum's registers are needed)
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (owner) {
            if (a.kp <= 32) add_round(C2, 0);
            else add_round(std::integral_constant<int, 4>{}, 0);
            for (int r = 1; r < rounds; ++r) {
                __syncthreads();                   // T has been read by everybody
                load_b(b_last, 0, r);
                bring_t(r);
                __syncthreads();
                add_round(std::integral_constant<int, 4>{}, r);
            }
        }
    }
    // The product ends here, in front of the stores' conditions: left alone the compiler moves the last MFMAs behind the test of a
    // lane's row, and a matrix instruction takes every lane's operands.
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) asm volatile("" : "+v"(acc[0][tm][tn]));

    // ---- pieces: handed over and added as in tiled_kernel -----------------------------------------------------------------------
    uint32_t le = rd16 >> 4;
    asm volatile("" : "+v"(le));
    if constexpr (MODE == kPieces) {
        constexpr int64_t PART_FLOATS = (int64_t)BM * 32 * TN * NW;
        typedef unsigned long long u64;
        union Pair { u64 q; float f[2]; };
        constexpr int PER = TM * TN * 8;           // 8-byte words of this lane in a slot
        if (!owner) {
            u64* slot = reinterpret_cast<u64*>(a.Part + (int64_t)lin * PART_FLOATS) + (int64_t)wave * PER * 64 + le;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                Pair p;
                p.f[0] = acc[0][i / 8 / TN][i / 8 % TN][2 * (i & 7)];
                p.f[1] = acc[0][i / 8 / TN][i / 8 % TN][2 * (i & 7) + 1];
                __hip_atomic_store(slot + i * 64, p.q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            // the flag goes up once every wavefront's stores are acknowledged (a fence does not wait for them)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) __hip_atomic_store(a.flags + lin, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            continue;
        }
        if (kt1 < KT) {
            const int64_t rt = tile_lin - a.dp_tiles;
            const int64_t last_wg = (rt * a.sk_tile_units + a.KT - 1) / a.sk_share;    // workgroup with the tile's last K tile
            for (int64_t v = lin + 1; v <= last_wg; ++v) {
                if (tid == 0) {
                    int polls = 0;
                    while (__hip_atomic_load(a.flags + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u && polls < a.spin_limit) {
                        __builtin_amdgcn_s_sleep(8);
                        ++polls;
                    }
                    wait_ok = (polls < a.spin_limit) ? 1 : 0;
                }
                __syncthreads();
                const bool ok = wait_ok != 0;
                const u64* slot = reinterpret_cast<const u64*>(a.Part + v * PART_FLOATS) + (int64_t)wave * PER * 64 + le;
                constexpr int GRP = 32;            // loads in flight: enough to cover the round trip, few enough to fit beside the sums
                static_assert(PER % GRP == 0, "whole groups");
#pragma unroll
                for (int i0 = 0; i0 < PER; i0 += GRP) {
                    Pair p[GRP];
#pragma unroll
                    for (int i = 0; i < GRP; ++i) p[i].q = __hip_atomic_load(slot + (i0 + i) * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int i = 0; i < GRP; ++i) {
                        const int at = i0 + i;
                        // a piece that never arrived must not pass for a result
                        if (!ok) p[i].f[0] = p[i].f[1] = __builtin_nanf("");
                        acc[0][at / 8 / TN][at / 8 % TN][2 * (at & 7)] += p[i].f[0];
                        acc[0][at / 8 / TN][at / 8 % TN][2 * (at & 7) + 1] += p[i].f[1];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();                   // wait_ok may be rewritten
            }
        }
    }

    // ---- store: lane (t, hh) holds columns 8 r4 + 4 hh .. + 3 of token t for every MFMA tile ---------------------------------------
    const int t_e = le & 31, hh_e = le >> 5;
    if (MODE != kPlanes && a.Yc != nullptr) {      // as MXINT8 for the next layer: block b of a group is registers 8 b .. + 7 of two lanes
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t row = m0 + tm * 32 + t_e;
            if (row >= a.M) continue;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                if (g0 + tn >= a.N32) continue;
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = acc[0][tm][tn][8 * b + i];
                    uint32_t w0, w1;
                    const uint32_t eb = requant_half_block(v, w0, w1);
                    const int64_t n0 = (g0 + tn) * 32 + 16 * b;
                    if (n0 < a.N) {
                        int8_t* dst = a.Yc + row * a.ldyc + n0 + 4 * hh_e;
                        *reinterpret_cast<uint32_t*>(dst) = w0;
                        *reinterpret_cast<uint32_t*>(dst + 8) = w1;
                        if (hh_e == 0) a.Ye[row * (a.N >> 4) + (n0 >> 4)] = (uint8_t)eb;
                    }
                }
            }
        }
    } else {
        float* out = a.Y;
        int64_t ldo = a.ldy;
        if constexpr (MODE == kPlanes) {
            ldo = plane_ld(a.N);
            out = a.Part + (int64_t)plane * a.M * ldo;
        }
        if (m0 + BM <= a.M && (g0 + TN) * 32 <= a.N && ldo < (1 << 24)) {        // a tile inside: one lane offset, no masks
            float* first = out + m0 * ldo + g0 * 32;
            const uint32_t off = t_e * (uint32_t)ldo + 4 * hh_e;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm, first += 32 * ldo) {
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        *reinterpret_cast<f32x4*>(first + off + (tn * 32 + 8 * r4)) =
                            f32x4{acc[0][tm][tn][4 * r4], acc[0][tm][tn][4 * r4 + 1], acc[0][tm][tn][4 * r4 + 2], acc[0][tm][tn][4 * r4 + 3]};
            }
        } else {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const int64_t row = m0 + tm * 32 + t_e;
                if (row >= a.M) continue;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    if (g0 + tn >= a.N32) continue;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int64_t n = (g0 + tn) * 32 + 8 * r4 + 4 * hh_e;
                        float* dst = out + row * ldo + n;
                        const f32x4 v = f32x4{acc[0][tm][tn][4 * r4], acc[0][tm][tn][4 * r4 + 1], acc[0][tm][tn][4 * r4 + 2], acc[0][tm][tn][4 * r4 + 3]};
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
    }
    if constexpr (MODE != kPieces) break;
  }   // pieces
}

// ---- which tile, cut along K or not -------------------------------------------------------------------------------------
// Time model of the main product in us: a workgroup takes per K tile between unit[r][0] and unit[r][1] when r + 1 of them share a compute unit, by how
// many compute units have that many (a full chip's clock is lower); `fixed` per launch, start[r - 1] more where r + 1 of them start on a
// unit at once, `round` per round of workgroups beyond the first; out[0] per MB of Y, out[1] per MB beyond the 256 that the caches hold,
// out[2] per MB of a Y beyond them whose rows share 128-byte lines (half-written ones go to memory twice); corr[0] + corr[1] S per
// round and 64 ranks of the correction beyond the first, S > 1 the partial sums of T, corr[2] per round above rank 32; planes take
// `plane` and `plane_mb` per MB of partial sums written and read.  Fitted to 130000 timings of 22800 calls of K 64 to 12288, N 256 to 28672, 33
// to 65536 tokens and ranks 8 to 256, planes of every number among them, on a warm chip: mean error 3 to 5 % a shape.  Of the calls that
// take fp6 operands, fitted on one half, the choice on the other is 0.5 % from the fastest form on average, 4 % at the 95th percentile, 26 % at
// the very worst; without `start`, out[1] and out[2] it was 0.7 and 5 %: 129 tokens of 6672 x 1776 rank 32 took 14 planes for 6, 18.2 us for
// 16.0, 8192 of 512 x 16244 rank 32 tiles of 128 x 512, 296 us for 231.
struct SixShape { int id, bm, bn, resident; double unit[3][2], start[2], fixed, round, out[3], corr[3], plane, plane_mb; };
static const SixShape kSixShapes[] = {
    {21, 128, 512, 1, {{2.202, 3.530}}, {0.0}, 13.867, 7.088, {0.155, 0.000, 0.064}, {4.513, 0.375, 2.333}, 0.0, 0.0},
    {22, 128, 256, 1, {{1.345, 2.098}}, {0.0}, 10.971, 4.711, {0.171, 0.000, 0.034}, {2.523, 0.357, 0.152}, 0.0, 0.0},
    {41, 64, 256, 2, {{1.370, 1.575}, {2.032, 2.271}}, {1.574}, 8.721, 1.360, {0.209, 0.029, 0.011}, {2.167, 0.235, 0.077}, 2.482, 0.163},
    {42, 64, 512, 1, {{1.712, 2.233}}, {0.0}, 10.153, 3.804, {0.171, 0.000, 0.017}, {2.427, 0.209, 0.193}, 2.538, 0.154},
    {43, 64, 128, 3, {{0.981, 1.072}, {1.223, 1.421}, {1.854, 1.939}}, {1.396, 0.684}, 7.063, 0.271, {0.205, 0.053, 0.014}, {1.390, 0.228, 0.079}, 2.436, 0.174},
    {44, 128, 128, 2, {{1.133, 1.352}, {1.705, 2.163}}, {1.761}, 9.148, 2.545, {0.211, 0.014, 0.031}, {2.630, 0.372, 0.112}, 2.665, 0.171},
};
// 128 x 512 with the tiles that do not fill a round cut in whole pieces: us per launch, K tile of a piece, K tile and number of whole
// rounds, piece beyond two, 64 ranks of the correction beyond the first, MB of Y, of one beyond the caches with rows that share lines (as
// above).  Of 1600 timings one half fitted: 5 %; with the models above the choice on 4800 other calls is 0.4 % from the fastest form on average, 23 % at
// worst (0.8 % before these).  In equal shares, and 128 x 256 in pieces, by force only: 15 to 20 % from any such model.
struct SixPieces { double fixed, share, unit, round, piece, corr, out[2]; };
static const SixPieces kSixPieces = {29.573, 3.535, 3.600, 11.348, 5.054, 7.626, {0.106, 0.049}};
constexpr int kMostPlanes = 16;

struct SixPick { int id, planes, share; double us; };        // share: K tiles per plane; planes 0: in pieces

// rounds of the correction beyond the first
static int more_rounds(int kp) { return kp > 64 ? (kp + 63) / 64 - 1 : 0; }

// Y, of mb MB, is more than the caches hold, and its rows do not start on 128 bytes (where they are as close as they can be)
static bool ragged_beyond_caches(const Layer& L, double mb) { return mb > 256.0 && ((L.N + 3) / 4 & 7) != 0; }

static double six_us(const SixShape& sh, const Layer& L, int64_t M, int S, int64_t tiles, int planes, int64_t share, int cus) {
    const int64_t wgs = tiles * planes, slots = (int64_t)cus * sh.resident, full = wgs / slots, rest = wgs - full * slots;
    const double mb = (double)M * (double)L.N * 4e-6;
    double t = sh.fixed + sh.round * (double)(full + (rest > 0 ? 1 : 0) - 1) + sh.out[0] * mb + sh.unit[sh.resident - 1][1] * (double)full * (double)share;
    if (mb > 256.0) t += sh.out[1] * (mb - 256.0);
    if (ragged_beyond_caches(L, mb)) t += sh.out[2] * mb;
    for (int r = 1; r < sh.resident; ++r)
        if (wgs > (int64_t)r * cus) t += sh.start[r - 1];
    if (rest > 0) {
        const int64_t r = (rest - 1) / cus;
        const double fill = (double)(rest - r * cus) / (double)cus;
        t += (double)share * (sh.unit[r][0] * (1.0 - fill) + sh.unit[r][1] * fill);
    }
    const double corr_rounds = (double)((tiles + slots - 1) / slots);
    t += corr_rounds * ((double)more_rounds(L.kp) * (sh.corr[0] + sh.corr[1] * (S > 1 ? S : 0)) + (L.kp > 32 ? sh.corr[2] : 0.0));
    if (planes > 1) t += sh.plane + sh.plane_mb * (double)planes * (double)M * (double)plane_ld(L.N) * 8e-6;
    return t;
}

// S: partial sums of T.  part_bytes: room for the pieces' accumulators or the planes (0: whole tiles only).  only: this shape and no
// other, in at least min_planes planes (id 0: not to be had).
static SixPick pick_six(const Layer& L, int64_t M, int S, int64_t part_bytes, int cus, int only = 0, int min_planes = 1) {
    SixPick best{0, 1, (int)L.KT, 0.0};
    for (const SixShape& sh : kSixShapes) {
        if (only != 0 && sh.id != only) continue;
        const int64_t tiles = ((M + sh.bm - 1) / sh.bm) * ((L.N + sh.bn - 1) / sh.bn);
        const bool large = sh.id < 40;                       // (no planes)
        for (int p = large ? 1 : min_planes; p <= (large ? 1 : kMostPlanes) && p <= L.KT; ++p) {
            const int64_t share = (L.KT + p - 1) / p;
            const int planes = (int)((L.KT + share - 1) / share);
            if (planes != p) continue;                       // the same planes as a smaller p
            if (p > 1 && (int64_t)p * M * plane_ld(L.N) * 4 > part_bytes) continue;
            const double us = six_us(sh, L, M, S, tiles, planes, share, cus);
            if (best.id == 0 || us < best.us) best = SixPick{sh.id, planes, (int)share, us};
        }
        if (sh.id == 21 && part_bytes > 0) {
            const Split sp = split_tiles(tiles, L.KT, cus, true);
            if (sp.sk_units == 0 || !sp.aligned) continue;
            const SixPieces& c = kSixPieces;
            const double rounds = (double)(sp.dp_tiles / sp.grid), mb = (double)M * (double)L.N * 4e-6;
            const double us = c.fixed + c.share * (double)sp.sk_share + rounds * (c.unit * (double)L.KT + c.round) +
                              c.piece * (double)(sp.sk_tile_units / sp.sk_share - 2) + c.corr * more_rounds(L.kp) * (rounds + 1.0) +
                              (c.out[0] + (ragged_beyond_caches(L, mb) ? c.out[1] : 0.0)) * mb;
            if (us < best.us) best = SixPick{21, 0, (int)sp.sk_share, us};
        }
    }
    return best;
}

// W_q records -> fp6 records (layouts in lqer_internal.h): a thread turns the 16 bytes of one lane and chunk.
__global__ __launch_bounds__(256) void widen_six_kernel(const uint8_t* Wt, int rec_bytes, int exp_bias, uint8_t* W6, int64_t records) {
    const int64_t rec = blockIdx.x;
    if (rec >= records) return;
    const int lane = threadIdx.x & 63, c = threadIdx.x >> 6;
    const uint8_t* src = Wt + rec * rec_bytes;
    uint8_t* dst = W6 + rec * kW6RecordBytes;
    const u32x4 w = *reinterpret_cast<const u32x4*>(src + (exp_bias >= 0 ? kWCompactCodeOffset : 0) + c * 1024 + lane * 16);
    uint32_t out[4] = {0u, 0u, 0u, 0u}, any[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {                      // the lane's two blocks
        any[b] = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t word = w[2 * b + (e >> 3)];
            const int i = e & 3;
            const uint32_t mag = (e & 4) ? (word >> (8 * i + 4)) & 7u : (word >> (8 * i)) & 7u;
            const uint32_t sg = (e & 4) ? (word >> (8 * ((i + 1) & 3) + 3)) & 1u : (word >> (8 * i + 7)) & 1u;
            any[b] |= mag;
            const int f = six_field(e), bit = 6 * f + 3 * b, at = bit & 31;
            out[bit >> 5] |= mag << at;
            if (at > 29) out[(bit >> 5) + 1] |= mag >> (32 - at);
            out[3] |= sg << (((6 * f + 5) & 31) - b);   // a field's sixth bit: an odd one
        }
    }
    *reinterpret_cast<u32x4*>(dst + c * 1024 + lane * 16) = u32x4{out[0], out[1], out[2], out[3]};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        uint32_t e;
        if (exp_bias >= 0) e = ((src[lane * 4 + c] >> (4 * b)) & 15u) + (uint32_t)exp_bias;
        else e = src[kWExpOffset + lane * 8 + 2 * c + b];
        dst[kWExpOffset + lane * 8 + 2 * c + b] = (uint8_t)(any[b] != 0u && e >= 2u ? e - 2u : 0u);
    }
}

hipError_t launch_widen_six(const Layer& L, hipStream_t s) {
    const int64_t records = L.N32 * L.KT;
    hipLaunchKernelGGL(widen_six_kernel, dim3((unsigned)records), dim3(256), 0, s, L.Wt, L.w_rec_bytes, L.w_exp_bias, L.W6, records);
    return hipGetLastError();
}

// Where a layer's calls take fp6 operands: with at least half as many K tiles as its correction has chunks of 64 columns beyond the first
// (always up to rank 64, from K = 257 at rank 128, from 769 at rank 256), and where the activations are more than next to nothing.  What
// the fp6 form takes longer, it takes to start and to end; of a few K tiles and a small rank (whose chunks the bf16 form has as further
// columns of K) it needs many rows to win that back: M KT^2 above 12500 up to three tiles and rank 32, above 8000 with four, and at one tile whatever the rank.
// From 8 tiles on the bf16 form cuts K and is the faster up to 3e5 activations of such ranks.  On 18000 calls of 33 to 100000 tokens, K 64
// to 11008: fp6 / bf16, rank 8 to 32, one tile 1.12 below 500 tokens, 1.08 at 4000 to 8000, 0.99 beyond 24000; two 1.11, 1.02, 1.00;
// three 1.08, 0.97; rank 64 and above from two tiles on 0.85 to 1.03 everywhere.  Without the two lines calls below them were up to 1.13 of
// the time of the bf16 form: 629 tokens of 320 x 872 rank 24 12.0 us, 10.8 by them, 69 of 4096 x 2430 rank 32 18.3 and 16.6.
// N has no say so that layers of one rank that share their activations share their form, and one quantization.
// 2-bit layers: where their exponents are nibbles (a K tile's eight scales are then two words of bytes, with a bias), and from four K tiles on
// (below, a call is projection and store: both forms within 3 %).  166 random calls of 33 to 8192 tokens, ranks 64 to 256: 0.90 of the
// bf16 form's time on average, 1.04 at worst; 4096 x 4096 rank 256 at 2048 tokens 109 -> 87 us.
bool tiled_takes_six(const Layer& L, int64_t M, int variant) {
    if (L.kp == 0 || (L.w_bits == 4 ? L.W6 == nullptr : L.w_exp_bias < 2)) return false;
    const int shape = variant % 100, mode = variant / 100;
    if (shape != 0) return shape == 21 || shape == 22 || (shape >= 41 && shape <= 44);
    if (mode > 1) return false;                              // cut by force: the bf16 shapes
    if (L.w_bits == 2 && L.KT < 4) return false;
    if (L.KT < 5 && (L.KT == 1 || L.kp <= 32) && M * L.KT * L.KT <= (L.KT == 4 ? 8000 : 12500)) return false;
    if (L.KT >= 8 && L.kp <= 32 && M * L.K <= 300000) return false;
    return M * L.K > 150000 && 2 * L.KT >= (2 * L.kp + 63) / 64 - 1;
}

uint8_t* six_scales(const Workspace& ws, const Layer& L) {
    return reinterpret_cast<uint8_t*>(ws.Xh) + ws.xh_rows / kX6Rows * L.KT * (4 * kX6Chunk);
}

// images, exponent bytes and T in the room the bf16 rows have (400 and 512 bytes per row and K tile)
void set_six_layout(Workspace& ws, const Layer& L) {
    ws.six = true;
    ws.ldxt = ws.ldxh - L.KT * kTileK;
    ws.Xt = reinterpret_cast<uint16_t*>(six_scales(ws, L) + ws.xh_rows / kX6Rows * L.KT * kX6Scales);
}

// ---- launches --------------------------------------------------------------------------------------------------------------------
// pieces: 0 = whole tiles, 2 = cut the tiles that do not fill a round, 3 = the same in equal shares of their K tiles
template <int TM, int TN, int NW, int CHAINS, int BITS>
static hipError_t launch_large(TiledArgs a, int pieces, bool by_force, int cus, hipStream_t s) {
    constexpr int BM = 32 * TM, BN = 32 * TN * NW, LDS = SixLds<TM, TN, NW, BITS>::BYTES;
    a.grid_m = (int)((a.M + BM - 1) / BM);
    a.grid_n = (int)((a.N + BN - 1) / BN);
    const int64_t tiles = (int64_t)a.grid_m * a.grid_n;
    static KernelSetup setup_pieces, setup_whole;
    Split sp = whole_tiles(tiles, a.KT);
    if (pieces != 0) {
        // One workgroup per compute unit, and owners wait for workgroups with higher numbers: all of them must be resident at once.
        const hipError_t e = prepare_kernel(six_kernel<TM, TN, NW, CHAINS, kPieces, BITS>, setup_pieces, LDS, 64 * NW);
        if (e != hipSuccess) return e;
        const bool fits = a.Part != nullptr && setup_pieces.resident >= 1 && (int64_t)BM * BN * 4 <= kTiledPartBytesPerCu && cus <= kTiledFlags;
        if (fits) sp = split_tiles(tiles, a.KT, cus, pieces != 3);
        else if (by_force) return hipErrorInvalidValue;
    }
    a.dp_tiles = sp.dp_tiles; a.sk_units = sp.sk_units; a.sk_share = sp.sk_share; a.sk_tile_units = sp.sk_tile_units;
    if (sp.sk_units > 0) return launch_kernel(six_kernel<TM, TN, NW, CHAINS, kPieces, BITS>, setup_pieces, LDS, sp.grid, 64 * NW, a, s);
    return launch_kernel(six_kernel<TM, TN, NW, CHAINS, kWhole, BITS>, setup_whole, LDS, tiles, 64 * NW, a, s);
}

// whole tiles, or K planes and then their sum
template <int TM, int TN, int NW, int BITS>
static hipError_t launch_small(TiledArgs a, const SixPick& pick, hipStream_t s) {
    constexpr int BM = 32 * TM, BN = 32 * TN * NW, LDS = SixLds<TM, TN, NW, BITS>::BYTES;
    a.grid_m = (int)((a.M + BM - 1) / BM);
    a.grid_n = (int)((a.N + BN - 1) / BN);
    a.dp_tiles = (int64_t)a.grid_m * a.grid_n;
    a.sk_share = pick.share;
    static KernelSetup setup_whole, setup_planes;
    if (pick.planes == 1) return launch_kernel(six_kernel<TM, TN, NW, 2, kWhole, BITS>, setup_whole, LDS, a.dp_tiles, 64 * NW, a, s);
    const hipError_t e = launch_kernel(six_kernel<TM, TN, NW, 2, kPlanes, BITS>, setup_planes, LDS, a.dp_tiles * pick.planes, 64 * NW, a, s);
    if (e != hipSuccess) return e;
    return launch_reduce_planes(a, pick.planes, s);
}

template <int BITS>
static hipError_t launch_pick(const TiledArgs& a, const SixPick& pick, int pieces, bool by_force, int cus, hipStream_t s) {
    switch (pick.id) {
        case 21: return launch_large<4, 2, 8, 1, BITS>(a, pieces, by_force, cus, s);     // 128 x 512
        case 22: return launch_large<4, 1, 8, 2, BITS>(a, pieces, by_force, cus, s);     // 128 x 256
        case 41: return launch_small<2, 2, 4, BITS>(a, pick, s);     // 64 x 256, 61 KB: two workgroups per compute unit
        case 42: return launch_small<2, 2, 8, BITS>(a, pick, s);     // 64 x 512, 113 KB
        case 44: return launch_small<4, 1, 4, BITS>(a, pick, s);     // 128 x 128, 68 KB: two workgroups per compute unit
        default: return launch_small<2, 1, 4, BITS>(a, pick, s);     // 64 x 128, 43 KB: three workgroups per compute unit
    }
}

hipError_t launch_six(TiledArgs a, const Layer& L, const Workspace& ws, int mode, int variant, int cus, hipStream_t s) {
    if (L.w_bits == 4) a.Wt = L.W6;                          // (2-bit weights: the records as they are)
    a.Xe6 = six_scales(ws, L);
    const int64_t part_bytes = (mode != 1 && ws.Part != nullptr) ? kTiledPartBytesPerCu * (int64_t)cus : 0;
    // By force: mode 0 = cut when the estimate says so, 1 = whole tiles, 2 = pieces or planes, 3 = pieces in equal shares
    const bool small = variant >= 41;
    if (small && mode == 3) return hipErrorInvalidValue;
    const SixPick pick = pick_six(L, a.M, ws.S, part_bytes, cus, variant, small && mode == 2 ? 2 : 1);
    if (pick.id == 0) return hipErrorInvalidValue;
    int pieces = pick.planes == 0 ? 2 : 0;
    const bool by_force = variant != 0 && !small && mode >= 2;
    if (by_force) pieces = mode;
    return L.w_bits == 4 ? launch_pick<4>(a, pick, pieces, by_force, cus, s) : launch_pick<2>(a, pick, pieces, by_force, cus, s);
}

}  // namespace lqer
