// Batched face-sum kernels: one persistent launch per class over a device
// work list that covers every tile of every problem of the class.
#include "cdugks_device.h"

namespace cdg {

// waves per SIMD the batched face sums are compiled for: 3 for the FP32
// forms of 1-D and 2-D classes, like the single-problem 2-D kernel
template <typename ST, int MAXD>
constexpr int batched_face_waves() { return MAXD <= 2 && !std::is_same<ST, double>::value ? 3 : 1; }

// ACC: the class's problems have an external acceleration (stage 1 of the
// 1-D and 2-D face sums adds its source; 3-D problems load quarter-step
// fields that already carry it)
// SM2: how 2-D problems store their face values
template <typename ST, int MAXD, bool DIR, bool SS, bool ACC, int SM2 = fv_store_mode<2>()>
__global__ __launch_bounds__(WG, (batched_face_waves<ST, MAXD>())) void k_face_sums_batched(const Problem* probs, const WorkItem* items, int nitems,
                                                          int* queue, int* other) {
    // Tile shape 0 for every problem.  (32 x 8 tiles were faster in FP32 while
    // face values were streamed in half lines; with ordinary stores, see
    // st_faces, 16 x 16 takes 2.05 against 2.11 ms per step of 20 uneven
    // problems, as fewer cells of the small ones are padding.)
    using K1 = FaceSumKernel<1, ST, DIR, SS, 0, ACC>;
    using K2 = FaceSumKernel<MAXD >= 2 ? 2 : 1, ST, DIR, SS, 0, ACC, true, MAXD >= 2 ? SM2 : fv_store_mode<1>()>;
    // 3-D FP64 boxes stream their face values whatever the rows: measured (the
    // reason is not known), four problems of 33^3 x 8^3 take 8.66 ms streamed,
    // 9.05 with ordinary stores and 9.20 with the test per store of single
    // problems; of 64 x 32 x 32 cells, whole sectors, 9.41, 9.44 and 9.79.
    using K3 = FaceSumKernel<MAXD >= 3 ? 3 : 1, ST, DIR, SS, 0, false, true,
                             std::is_same<ST, double>::value ? FV_STREAM : FV_EITHER>;
    __shared__ union U {
        typename K1::Smem s1;
        typename K2::Smem s2;
        typename K3::Smem s3;
    } sm;
    __shared__ int slot;
    if (blockIdx.x == 0 && threadIdx.x == 0) *other = 0;
    for (int w = next_item(queue, &slot); w < nitems; w = next_item(queue, &slot)) {
        const WorkItem it = load_uniform(items + w);
        const Problem P = load_uniform(probs + it.prob);
        if (P.D == 1) K1::run(P, it.tile, it.slice, P.nslices, sm.s1);
        else if (MAXD >= 2 && P.D == 2) K2::run(P, it.tile, it.slice, P.nslices, sm.s2);
        else if (MAXD >= 3) K3::run(P, it.tile, it.slice, P.nslices, sm.s3);
    }
}

#define CDG_DISPATCH_MAXD(STORAGE, MAXD, MACRO)                      \
    do {                                                             \
        if ((STORAGE) == 0) {                                        \
            if ((MAXD) == 1) MACRO(double, 1);                       \
            else if ((MAXD) == 2) MACRO(double, 2);                  \
            else MACRO(double, 3);                                   \
        } else if ((STORAGE) == 1) {                                 \
            if ((MAXD) == 1) MACRO(float, 1);                        \
            else if ((MAXD) == 2) MACRO(float, 2);                   \
            else MACRO(float, 3);                                    \
        } else {                                                     \
            if ((MAXD) == 1) MACRO(Bf16Tail, 1);                     \
            else if ((MAXD) == 2) MACRO(Bf16Tail, 2);                \
            else MACRO(Bf16Tail, 3);                                 \
        }                                                            \
    } while (0)

// stream: every 2-D problem of the class has face rows of whole 64-byte
// sectors.  2-D FP64 then streams the face values, as a single problem does
// (see st_faces; steps streamed and not: two of 256^2 x 28^2 3245 and 3270 us,
// forty of 64^2 x 20^2 2666 and 2722), which ragged rows would lose by (sixty
// uneven problems 14.81 ms and 14.20).  With a test per store instead of a
// kernel of its own: 3281 and 2692 us, 14.29 ms.
template <typename ST, int MAXD, bool DIR, bool SS, bool ACC>
static void launch_class(const Problem* probs, const WorkItem* items, int nitems, int grid, bool stream, int* queue,
                         int* other, hipStream_t s) {
    if constexpr (MAXD == 2 && std::is_same<ST, double>::value) {
        if (stream) {
            hipLaunchKernelGGL((k_face_sums_batched<ST, MAXD, DIR, SS, ACC, FV_STREAM>), dim3(grid), dim3(WG), 0, s,
                               probs, items, nitems, queue, other);
            return;
        }
    }
    hipLaunchKernelGGL((k_face_sums_batched<ST, MAXD, DIR, SS, ACC>), dim3(grid), dim3(WG), 0, s, probs, items, nitems,
                       queue, other);
}

hipError_t launch_face_sums_batched(const Problem* probs, const WorkItem* items, int nitems, int grid,
                                    int maxd, int storage, bool dirichlet, bool single_slope, bool accel,
                                    bool stream, int* queue, int* other, hipStream_t s) {
    if (nitems <= 0) return hipSuccess;
#define CDG_B(DIRV, SSV, ACCV)                                                                               \
    do {                                                                                                     \
        if ((STORAGE_) == 0) {                                                                               \
            if (maxd == 1) CDG_LB(double, 1, DIRV, SSV, ACCV);                                                     \
            else if (maxd == 2) CDG_LB(double, 2, DIRV, SSV, ACCV);                                                \
            else CDG_LB(double, 3, DIRV, SSV, ACCV);                                                               \
        } else if ((STORAGE_) == 1) {                                                                        \
            if (maxd == 1) CDG_LB(float, 1, DIRV, SSV, ACCV);                                                      \
            else if (maxd == 2) CDG_LB(float, 2, DIRV, SSV, ACCV);                                                 \
            else CDG_LB(float, 3, DIRV, SSV, ACCV);                                                                \
        } else {                                                                                             \
            if (maxd == 1) CDG_LB(Bf16Tail, 1, DIRV, SSV, ACCV);                                                   \
            else if (maxd == 2) CDG_LB(Bf16Tail, 2, DIRV, SSV, ACCV);                                              \
            else CDG_LB(Bf16Tail, 3, DIRV, SSV, ACCV);                                                             \
        }                                                                                                    \
    } while (0)
#define CDG_LB(TT, MD, DIRV, SSV, ACCV)                                                                      \
    launch_class<TT, MD, DIRV, SSV, ACCV>(probs, items, nitems, grid, stream, queue, other, s)
#define STORAGE_ storage
    // the acceleration never comes with the single-slope option (refused at
    // problem set-up)
    if (dirichlet) {
        if (single_slope) CDG_B(true, true, false);
        else if (accel) CDG_B(true, false, true);
        else CDG_B(true, false, false);
    } else {
        if (single_slope) CDG_B(false, true, false);
        else if (accel) CDG_B(false, false, true);
        else CDG_B(false, false, false);
    }
#undef STORAGE_
#undef CDG_LB
#undef CDG_B
    return hipGetLastError();
}

int batched_face_blocks_per_cu(int maxd, int storage, bool accel) {
    int n = 0;
    hipError_t e = hipSuccess;
    if (accel) {
#define CDG_L(TT, MD) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (k_face_sums_batched<TT, MD, false, false, true>), WG, 0)
        CDG_DISPATCH_MAXD(storage, maxd, CDG_L);
#undef CDG_L
    } else {
#define CDG_L(TT, MD) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (k_face_sums_batched<TT, MD, false, false, false>), WG, 0)
        CDG_DISPATCH_MAXD(storage, maxd, CDG_L);
#undef CDG_L
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return n;
}

}  // namespace cdg
