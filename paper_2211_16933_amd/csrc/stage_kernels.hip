// The stage kernels of one mode (ELB_STAGE_MODE: MODE_FP64, MODE_FP32, MODE_FP32_MIXED or
// MODE_FP32_FIXUP), compiled once per mode so that the modes build side by side.
#include <hip/hip_runtime.h>

#include <climits>

#include "stage_table.h"

#ifndef ELB_STAGE_MODE
#error "compile with -DELB_STAGE_MODE=0..3"
#endif

namespace elb {

namespace {

constexpr int MODE = ELB_STAGE_MODE;
constexpr int ANY = 1 << 30;  // a tile taken for any number of blocks

template <typename R, int Q, int S, int L, bool RET, bool CL>
void launch_stage(const void *args, int blocks, size_t shm, hipStream_t st)
{
    hipLaunchKernelGGL((k_stage<R, Q, S, L, MODE, RET, CL>), dim3(blocks), dim3(Geometry<R, Q, S, L>::NT), shm, st,
                       *static_cast<const StageArgs<R> *>(args));
}

// The tiles of small problems, by Q: strips, cells per strip, and the largest number of blocks
// for which the tile is taken (pick_stage takes the first that fits; the tile of large
// problems comes last).  A launch of few blocks is a chain of latencies: staging, row and
// cell closures, then the march along a strip, which alone is half of it on 8-cell strips
// (FP64 Q = 16, 128 cells: 9600 of 19500 cycles), while most of the chip idles.  Shorter
// strips and fewer rows per block cut that chain, until the blocks no longer have a compute
// unit each and the 6 halo rows staged and closed again by every block cost more than the
// strips save.  The lines were measured on a shock tube of 128 to 32768 cells; us per launch,
// the large-problem tile against the one taken here:
//   FP64  Q = 8   128 cells 9.2 / 5.0, 8192 9.5 / 5.9, 32768 12.1 / 8.9
//         Q = 16  128 cells 8.5 / 5.4, 8192 9.3 / 6.9, 32768 12.0 / 11.6
//         Q = 48  128 cells 10.8 / 6.7, 2048 11.2 / 7.4, 8192 12.4 / 12.1 (more blocks: 14.5)
//         Q = 96  128 cells 11.5 / 7.4, 2048 12.0 / 9.9 (2 x 2: 11.6)
//         Q = 200 128 cells 23.7 / 17.2, 1024 24.7 / 23.3 (2 x 2: 27.9)
//   mixed Q = 8   128 cells 8.9 / 5.6, 8192 9.3 / 6.2, 32768 11.0 / 8.6
//         Q = 48  128 cells 10.4 / 6.9, 2048 10.9 / 7.3, 8192 11.4 / 9.3
//         Q = 64  128 cells 10.2 / 7.0, 8192 11.4 / 10.0
//         Q = 96  128 cells 10.8 / 8.2, 2048 11.2 / 8.9, 4096 11.5 / 9.8
// Two of them are the better tile at any size: Q = 8 on 4-cell strips (131072 cells: FP64
// 29.6 / 23.9, mixed 22.7 / 21.5) and plain FP32 Q = 64 on 4 x 8 (65536 cells: 37.5 / 34.7;
// mixed 41.1 / 42.5).
// Every tile keeps the strip count's split of a wave into phi or theta items and the lane
// count of the coefficient recurrence (Geometry::RG) of the large one, so all give the same
// bits.  X3: also compiled with the learned closure inside (whole 16-cell tiles, Q <= 16), which
// has a limit of its own: the closure's blocks are fewer per compute unit, and one more round of
// them costs more than the short strips save (Q = 12, us on 4-cell / 8-cell strips: FP64 1032 blocks
// 22.0 / 20.8; mixed 1125 17.9 / 20.4, 1282 23.8 / 20.6).
#if ELB_STAGE_MODE == 0
#define CL12 1024
#define ELB_SMALL_TILES(X2, X3) \
    X2(8, 8, 1, 1024) X3(8, 8, 2, 1024, 1024) X2(8, 8, 4, ANY) \
    X2(12, 8, 1, 256) X3(12, 8, 2, 512, 512) X3(12, 8, 4, 1300, CL12) \
    X2(16, 8, 1, 256) X3(16, 8, 2, 512, 512) X3(16, 8, 4, 1024, 1024) \
    X2(20, 8, 1, 256) X2(20, 8, 2, 512) \
    X2(24, 8, 1, 256) X2(24, 8, 2, 512) \
    X2(32, 4, 2, 256) X2(32, 4, 4, 512) \
    X2(40, 8, 1, 256) X2(40, 8, 2, 512) \
    X2(48, 4, 2, 256) X2(48, 4, 4, 512) \
    X2(64, 4, 2, 256) \
    X2(96, 2, 2, 256) X2(96, 2, 4, 256) \
    X2(200, 2, 2, 128) X2(200, 2, 4, 256)
#else
#define CL12 1280
#define ELB_SMALL_TILES(X2, X3) \
    X2(8, 8, 1, 1024) X3(8, 8, 2, 1024, 1024) X2(8, 8, 4, ANY) \
    X2(12, 8, 1, 256) X3(12, 8, 2, 512, 512) X3(12, 8, 4, 1300, CL12) \
    X3(16, 8, 2, 512, 512) X3(16, 8, 4, 1024, 1024) \
    X2(20, 8, 1, 256) X2(20, 8, 2, 256) X2(20, 8, 4, 1024) \
    X2(24, 16, 1, 256) X2(24, 16, 2, 256) X2(24, 16, 4, 512) \
    X2(32, 8, 1, 256) X2(32, 8, 2, 256) X2(32, 8, 4, 512) \
    X2(40, 8, 1, 256) X2(40, 8, 2, 256) X2(40, 8, 4, 512) \
    X2(48, 8, 1, 256) X2(48, 8, 2, 256) X2(48, 8, 4, 256) \
    X2(64, 4, 2, 256) X2(64, 4, 4, 256) X2(64, 4, 8, MODE == MODE_FP32 ? ANY : 256) \
    X2(96, 4, 2, 256) X2(96, 4, 4, 256) \
    X2(200, 2, 2, 128) X2(200, 2, 4, 128)
#endif

#if ELB_STAGE_MODE == 0
typedef double Real;
#else
typedef float Real;
#endif

#define ELB_ST(QV, SV, LV, CAP, RET, CL) \
    {QV, SV, LV, RET, CL, Geometry<Real, QV, SV, LV>::NT, Geometry<Real, QV, SV, LV>::ROWS, CAP, \
     &launch_stage<Real, QV, SV, LV, RET, CL>},
// chi_SET and chi_RET-FM; and for Q <= 16 with the learned closure inside
#define ELB_S2(QV, SV, LV, CAP) ELB_ST(QV, SV, LV, CAP, false, false) ELB_ST(QV, SV, LV, CAP, true, false)
#define ELB_S3(QV, SV, LV, CAP, CLCAP) ELB_S2(QV, SV, LV, CAP) ELB_ST(QV, SV, LV, CLCAP, false, true)
// the large-problem tile
#define ELB_L2(QV) ELB_S2(QV, (Shape<Real, QV>::S), (Shape<Real, QV>::L), INT_MAX)
#define ELB_L3(QV) ELB_S3(QV, (Shape<Real, QV>::S), (Shape<Real, QV>::L), INT_MAX, INT_MAX)

const StageKernel kStage[] = {
    ELB_SMALL_TILES(ELB_S2, ELB_S3)
    // Q = 8 with the learned closure, 65536 cells: FP64 4-cell strips 29.0 us, 8-cell 36.7; mixed
    // 27.7 and 23.0 (32768 cells: 15.7 and 19.2)
#if ELB_STAGE_MODE == 0
    ELB_ST(8, 8, 4, ANY, false, true)
#else
    ELB_ST(8, 8, 4, 1300, false, true) ELB_ST(8, 8, 8, INT_MAX, false, true)
#endif
    ELB_L3(12) ELB_L3(16) ELB_L2(20) ELB_L2(24) ELB_L2(32)
    ELB_L2(40) ELB_L2(48)
#if ELB_STAGE_MODE != 1  // plain FP32 takes its 4 x 8 tile at any size
    ELB_L2(64)
#endif
    ELB_L2(96) ELB_L2(200)
};

#if ELB_STAGE_MODE != 3
template <typename R, int Q, int S, int L, bool RET>
void launch_batch(const BatchStage &bs, int grid, size_t shm, hipStream_t st)
{
    hipLaunchKernelGGL((k_stage_batch<R, Q, S, L, MODE, RET>), dim3(grid), dim3(Geometry<R, Q, S, L>::NT), shm, st, bs);
}

#define ELB_BKX(QV, SV, LV, CAP, RET) \
    {QV, SV, LV, RET, Geometry<Real, QV, SV, LV>::NT, Geometry<Real, QV, SV, LV>::ROWS, CAP, \
     &launch_batch<Real, QV, SV, LV, RET>},
#define ELB_BK(QV, SV, LV) ELB_BKX(QV, SV, LV, INT_MAX, false)
#define ELB_BKR(QV, SV, LV) ELB_BKX(QV, SV, LV, INT_MAX, true)
#define ELB_BK2(QV, SV, LV, CAP) ELB_BKX(QV, SV, LV, CAP, false) ELB_BKX(QV, SV, LV, CAP, true)
#define ELB_BK3(QV, SV, LV, CAP, CLCAP) ELB_BK2(QV, SV, LV, CAP)

// Variant 0 of every Q is the single-problem shape; the FP32 modes also have the 16-cell strips
// in blocks of up to 384 threads, between which the tuner chooses.  chi_RET-FM: the
// single-problem shape of every Q.  Then the tiles of small problems: indices kept in a tuner
// cache file count the variants of a Q in this order, so new ones come last.
const BatchKernel kBatch[] = {
#if ELB_STAGE_MODE == 0
    ELB_BK(8, 8, 8) ELB_BK(12, 8, 8) ELB_BK(16, 8, 8) ELB_BK(20, 4, 8)
    ELB_BK(24, 4, 8) ELB_BK(32, 4, 8) ELB_BK(40, 8, 8) ELB_BK(48, 4, 8)
    ELB_BK(64, 2, 8) ELB_BK(96, 2, 8) ELB_BK(200, 2, 8)
    ELB_BKR(8, 8, 8) ELB_BKR(12, 8, 8) ELB_BKR(16, 8, 8) ELB_BKR(20, 4, 8)
    ELB_BKR(24, 4, 8) ELB_BKR(32, 4, 8) ELB_BKR(40, 8, 8) ELB_BKR(48, 4, 8)
    ELB_BKR(64, 2, 8) ELB_BKR(96, 2, 8) ELB_BKR(200, 2, 8)
#else
    ELB_BK(8, 8, 8) ELB_BK(12, 8, 8) ELB_BK(16, 8, 8) ELB_BK(16, 16, 8)
    ELB_BK(20, 8, 8) ELB_BK(24, 16, 8) ELB_BK(24, 8, 8) ELB_BK(32, 8, 8)
    ELB_BK(32, 4, 16) ELB_BK(40, 8, 8) ELB_BK(48, 8, 8) ELB_BK(48, 4, 16)
    ELB_BK(64, 6, 8) ELB_BK(96, 4, 8)
#if ELB_STAGE_MODE == 2
    ELB_BK(96, 2, 16)
#endif
    ELB_BK(200, 2, 8)
    ELB_BKR(8, 8, 8) ELB_BKR(12, 8, 8) ELB_BKR(16, 8, 8) ELB_BKR(20, 8, 8)
    ELB_BKR(24, 16, 8) ELB_BKR(32, 8, 8) ELB_BKR(40, 8, 8) ELB_BKR(48, 8, 8)
    ELB_BKR(64, 6, 8) ELB_BKR(96, 4, 8) ELB_BKR(200, 2, 8)
#endif
    ELB_SMALL_TILES(ELB_BK2, ELB_BK3)
};
#endif

}  // namespace

#if ELB_STAGE_MODE == 0
StageTable stage_table_f64()
#elif ELB_STAGE_MODE == 1
StageTable stage_table_f32()
#elif ELB_STAGE_MODE == 2
StageTable stage_table_mixed()
#else
StageTable stage_table_fixup()
#endif
{
    const int n = (int)(sizeof kStage / sizeof kStage[0]);
#if ELB_STAGE_MODE != 3
    return {kStage, n, kBatch, (int)(sizeof kBatch / sizeof kBatch[0])};
#else
    return {kStage, n, nullptr, 0};  // batches do not carry the moment fix-up
#endif
}

}  // namespace elb
