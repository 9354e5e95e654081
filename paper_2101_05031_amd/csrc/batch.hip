// Work queue of batched slicing.  The paper notes that slicing time follows
// the number of struts meeting a plane (Sec. 6.4), so planes and tiles carry
// very uneven work.  Work items are (slab, tile) buckets; the queue orders
// them by descending cost (bucket length x planes, in 256 logarithmic classes;
// a stable sort keeps tiles of one class in spatial order), so that the field
// launch, which takes them in that order, ends on its smallest items.
#include "kernels.hpp"

namespace lsl {
namespace {

__global__ void k_queue_keys(FieldArgs a, uint32_t n_items, uint32_t* keys, uint32_t* vals) {
    const uint32_t it = blockIdx.x * blockDim.x + threadIdx.x;
    if (it >= n_items) return;
    uint32_t t = it;
    const uint32_t tx = t % (uint32_t)a.ntx;
    t /= (uint32_t)a.ntx;
    const uint32_t ty = t % (uint32_t)a.nty;
    t /= (uint32_t)a.nty;
    const int slab = a.s_lo + (int)t;
    int kb = slab * a.slab, ke = kb + a.slab;
    if (kb < a.k0) kb = a.k0;
    if (ke > a.k0 + a.nk) ke = a.k0 + a.nk;
    const uint32_t bucket = ((uint32_t)(slab - a.group_s0) * (uint32_t)a.nty + ty) *
                                (uint32_t)a.ntx + tx;
    const uint32_t len = a.offsets[bucket + 1] - a.offsets[bucket];
    const float cost = (float)len * (float)(ke - kb);
    int cls = (int)(8.0f * __log2f(1.0f + cost));
    cls = cls < 0 ? 0 : (cls > 255 ? 255 : cls);
    keys[it] = 255u - (uint32_t)cls;          // descending cost
    vals[it] = it;
}

}  // namespace

lsl_status launch_queue_build(const FieldArgs& f, uint32_t* keys, uint32_t* vals,
                              uint32_t* keys_alt, uint32_t* vals_alt, uint32_t n_items,
                              uint32_t* tmp, const uint32_t** queue_out, hipStream_t st) {
    k_queue_keys<<<(n_items + 255) / 256, 256, 0, st>>>(f, n_items, keys, vals);
    LSL_HIP(hipGetLastError());
    int which = 0;
    LSL_TRY(radix_sort_pairs(keys, vals, keys_alt, vals_alt, n_items, 8, tmp, &which, st));
    *queue_out = which ? vals_alt : vals;
    return LSL_OK;
}

}  // namespace lsl
