// Heavy-first work list of a large plan (Section 3.2), in O(T) memory: the
// windows stably sorted by their key, largest first (radix.hip), and every
// window's items written at the position its rank gives (see WorkListShape).
#include "f3s_internal.h"

namespace f3s {
namespace {

// Window order[i] is i-th in the sorted order; one wavefront per window.
__global__ __launch_bounds__(256) void k_place_items(const int32_t *order, const int32_t *key,
                                                     int32_t T, WorkListShape shape,
                                                     WorkItem *items, int32_t *merges,
                                                    int32_t *first)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= T) return;
    const int w = order[i];
    const int pos = key[w] == shape.piece ? i + shape.slot_base[w] - shape.split_idx[w]
                                          : i + shape.n_pieces - shape.n_split;
    if ((threadIdx.x & 63) == 0) first[w] = pos;
    place_window(shape, w, pos, threadIdx.x & 63, 64, items, merges);
}

// heavy[j] += items of the windows whose key exceeds heavy_blocks(j).
__global__ __launch_bounds__(256) void k_heavy_table(const int32_t *key, int32_t T,
                                                     WorkListShape shape, int32_t *heavy)
{
    __shared__ int32_t hist[kHeavySteps + 1];
    if (threadIdx.x <= kHeavySteps) hist[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < T;
         w += (int64_t)gridDim.x * 256) {
        const int level = heavy_level(key[w]);
        const int n = shape.slot_base[w + 1] - shape.slot_base[w];
        if (level) atomicAdd(&hist[level], n ? n : 1);
    }
    __syncthreads();
    if (threadIdx.x < kHeavySteps) {
        int h = 0;
        for (int l = threadIdx.x + 1; l <= kHeavySteps; ++l) h += hist[l];
        if (h) atomicAdd(&heavy[threadIdx.x], h);
    }
}

}  // namespace

hipError_t launch_worklist(const int32_t *key, const WorkListShape &shape, int32_t T,
                           const RadixScratch &radix, WorkItem *items, int32_t *merges,
                           int32_t *pos, int32_t *heavy, hipStream_t s)
{
    if (T == 0) return hipSuccess;
    const int32_t *sorted_keys = nullptr, *order = nullptr;
    // windows above the piece size are split and have it as their key
    hipError_t e = launch_radix_pairs(key, nullptr, T, shape.piece, true, radix, &sorted_keys,
                                      &order, s);
    if (e != hipSuccess) return e;
    k_place_items<<<(unsigned)((T + 3) / 4), 256, 0, s>>>(order, key, T, shape, items, merges,
                                                            pos);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const unsigned g = (unsigned)((T + 255) / 256);
    k_heavy_table<<<g < 64 ? g : 64, 256, 0, s>>>(key, T, shape, heavy);
    return hipGetLastError();
}

}  // namespace f3s
