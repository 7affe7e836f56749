// What the two files of prefill kernels share: kernels_tiled.hip (bf16 operands) and kernels_six.hip (fp6 operands).
#pragma once
#include <mutex>

#include "lqer_internal.h"

namespace lqer {

struct TiledArgs {
    const uint8_t* Wt; const uint8_t* Bt;
    const uint16_t* Xh; int64_t ldxh;                // (fp6 form: the images)
    const uint16_t* Xt; int64_t ldxt;                // T_hi | T_lo | 0, row by row
    const uint8_t* Xe6;                              // fp6 form: exponent bytes of the activations' blocks
    const float* Tpart; int S; int64_t tp_stride;    // S > 1: T as S fp32 partial sums [S][tp_stride / kp rows][kp]
    float* Y; int64_t ldy;
    int8_t* Yc; uint8_t* Ye; int64_t ldyc;           // Yc != null: store Y as MXINT8 (blocks of 16 along N) instead of fp32
    int64_t M, N, KT, N32;
    int kp, kp16;
    int grid_m, grid_n;
    int group_m;
    // work split (the head of kernels_tiled.hip says how)
    int64_t dp_tiles;          // output tiles taken whole, tile i by workgroup i % gridDim.x
    int64_t sk_units;          // K tile units of the remaining output tiles, shared out in ranges of ...
    int64_t sk_share;          // ... this many per workgroup
    int64_t sk_tile_units;     // units per remaining tile: KT, or KT rounded up to whole shares so that no share
                               // crosses a tile (the units past KT are empty)
    float* Part;               // [gridDim.x][BM * BN] accumulators handed over
    uint32_t* flags;           // [gridDim.x], zero before the launch; 1 = slot written
    int spin_limit;            // polls of a flag before the waiting workgroup gives up (and stores NaN)
    int rec_bytes;             // bytes of a weight record
    int exp_bias;              // >= 0: exponent nibbles (byte = nibble + exp_bias); -1: exponent bytes
};

// row stride of a plane of partial sums
__host__ __device__ constexpr int64_t plane_ld(int64_t N) { return (N + 3) / 4 * 4; }

struct Split { int64_t grid, dp_tiles, sk_units, sk_share, sk_tile_units; bool aligned; };

inline Split whole_tiles(int64_t tiles, int64_t KT) { return Split{tiles, tiles, 0, 1, KT, false}; }

// slots = workgroups the chip holds at once.
// aligned: where the chip holds two or more workgroups per remaining tile, every such tile is cut into the same
// whole number of pieces, one per workgroup, instead of equal shares of all remaining K tiles: a share then never
// crosses a tile, so no workgroup gets a second (possibly tiny) piece.  Measured on 11008 x 4096 at M = 2048
// (128 tiles of 43 K tiles on 256 workgroups): 157 us against 172 us with equal shares (tiled_kernel, when it took that call).
inline Split split_tiles(int64_t tiles, int64_t KT, int64_t slots, bool aligned) {
    Split sp;
    sp.grid = slots;
    sp.dp_tiles = (tiles / slots) * slots;
    const int64_t rem = tiles - sp.dp_tiles;
    if (rem == 0) return whole_tiles(tiles, KT);
    const int64_t p = slots / rem;                           // pieces per remaining tile
    if (aligned && p >= 2 && KT / p >= 2) {
        sp.sk_share = (KT + p - 1) / p;
        sp.sk_tile_units = sp.sk_share * p;
        sp.sk_units = rem * sp.sk_tile_units;
        sp.aligned = true;
        return sp;
    }
    sp.aligned = false;
    sp.sk_tile_units = KT;
    sp.sk_units = rem * KT;
    sp.sk_share = (sp.sk_units + slots - 1) / slots;
    if (sp.sk_share < 2) sp.sk_share = 2;                    // a piece is worth its hand-over
    return sp;
}

// What has to be established once per kernel instance and process: the dynamic LDS limit, and how many of its
// workgroups one compute unit really holds (the work split launches exactly as many workgroups as are resident
// at once, because owners wait for flags that later workgroups raise).
struct KernelSetup {
    std::once_flag once;
    hipError_t err = hipSuccess;
    int resident = 0;            // workgroups per compute unit
};

template <typename Kern>
inline hipError_t prepare_kernel(Kern kern, KernelSetup& ks, int lds_bytes, int threads) {
    std::call_once(ks.once, [&] {
        ks.err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (ks.err != hipSuccess) return;
        int n = 0;
        ks.err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, threads, (size_t)lds_bytes);
        ks.resident = n;
    });
    return ks.err;
}

template <typename Kern>
inline hipError_t launch_kernel(Kern kern, KernelSetup& ks, int lds_bytes, int64_t grid_x, int threads, const TiledArgs& a, hipStream_t s) {
    const hipError_t e = prepare_kernel(kern, ks, lds_bytes, threads);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid_x), dim3(threads), lds_bytes, s, a);
    return hipGetLastError();
}

// Y = the sum of `planes` planes of partial sums at a.Part
hipError_t launch_reduce_planes(const TiledArgs& a, int planes, hipStream_t s);
// The main product on fp6 operands (ws.six); mode and variant as in launch_tiled.
hipError_t launch_six(TiledArgs a, const Layer& L, const Workspace& ws, int mode, int variant, int cus, hipStream_t s);

}  // namespace lqer
