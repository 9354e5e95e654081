// Field evaluation (Eq. 6 with the closed form of Eq. 7, Sec. 4).
//
// The float32 kernel of the paper's kernel (field_q32.hpp) serves lattices
// whose planes may share reference planes; the method below (field_block.hpp)
// serves float64, the compact Gaussian and float32 lattices whose planes are
// coarse against the smallest support (every plane staged from float64).
//
// One wave owns an 8x8 pixel block of one tile and one slab of planes.  The
// wave walks its tile's bucket list (edge-list order) 64 struts at a time.  Per
// strut and plane that may reach the block it stages, in float64, the foot F
// of the block centre c on the strut's line:
//
//   tc = (c - a).u,  m = a + tc u - c  (m is orthogonal to u),
//
// and drops the strut for that plane when no pixel of the block can be within
// R of the segment: with F* the segment's point nearest to c, D = |F* - c| and
// n = (F* - c)/D, the segment lies in n.(x - F*) >= 0, so a pixel c + d is at
// least D - n.d >= D - (3.5 dx |n_x| + 3.5 dy |n_y|) from it (the block is
// flat, so struts passing above or below it are dropped sooner than by a
// bounding circle).  The surviving struts are compacted into LDS with a
// ballot/mbcnt prefix.  For a pixel p = c + d (d in the plane) the
// arclength coordinates of the strut ends with origin at the foot of p are
//
//   alpha = -tc - d.u,   beta = (L - tc) - d.u,
//   H = R^2 - dist(p, line)^2 = (R^2 - |m|^2) + 2 m.d - |d|^2 + (d.u)^2,
//
// all formed from small quantities, and the term is
//
//   r/R^4 * integral over [clamp(alpha), clamp(beta)] of (H - t^2)^2 dt
//     = r/R^4 * (cb - ca) * (H^2 - 2/3 H S1 + S2/5),
//   S1 = ca^2 + ca cb + cb^2,  S2 = (ca^2 + cb^2) S1 - (ca cb)^2,
//   ca, cb = alpha, beta clamped to [-sqrt(H), sqrt(H)].
//
// Terms outside the support come out as exact zeros (cb - ca = 0).  A strut
// is a candidate of a block and plane only where it passes the distance test
// and its binned pixel and plane ranges cover them, so every tile size, slab
// depth and group split hands the block the same candidates in the same
// order.  Sums are compensated, s' = s + g, e += g - (s' - s): float32 adds
// each run of four consecutive candidates plainly, ((t0 + t1) + t2) + t3, and
// compensates once per run; float64 compensates every term.
#include <type_traits>

#include "field_block.hpp"
#include "field_q32.hpp"

namespace lsl {
namespace {

// Waves per SIMD the kernels are built for: the registers of one or two
// planes fit eight (64 each), of four planes six; eight and more planes are
// fastest with five (96 registers; four and six measured 9% and 3% slower),
// but the float32 kernels of field_block.hpp, which keep less between planes,
// with six (per-strut supports 1.37 -> 1.33 ms, the Gaussian 2.71 -> 2.59 ms).
template <typename T>
constexpr int field_waves(int SZ, int form) {
    const bool small = sizeof(T) == 4 && form == kFormBlock && SZ <= 8;
    return SZ <= 2 ? 8 : SZ <= 4 || small ? 6 : 5;
}

// One wave per workgroup takes one 8x8 block of one (slab, tile) item.  The
// items come in the order of `queue` (descending cost, slice_batch), the
// hardware handing workgroups out as others end, or, without one, in order;
// either way the blocks of an item follow each other on one XCD, whose L2
// then holds the item's records (workgroups go to the 8 XCDs in turn).
//
// Workgroups of one wave: a workgroup's place is taken again only when all
// its waves have ended, so four unequal blocks leave a compute unit partly
// idle; and a grid of persistent workgroups that pull items from a counter
// waits at each item for its slowest wave.  96 planes of 2048^2 of 1M struts:
// persistent workgroups of four waves 8.0 ms, this 7.7 ms;
// 812 float64 struts, 50 planes of 256^2: 54 and 36 us.
template <typename T, int SZ, bool STATS, int K, bool SR, int FORM>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(field_waves<T>(SZ, FORM)))) void
k_field(FieldArgs a, const uint32_t* queue, uint32_t item0, uint32_t n_items) {
    const int nsub = a.tile / kBlockPix, nsub2 = nsub * nsub;
    const uint32_t xcd = blockIdx.x % 8u, u = blockIdx.x / 8u;
    const uint32_t seq = u / (uint32_t)nsub2;
    const int sub = (int)(u % (uint32_t)nsub2);
    uint32_t t;
    if (queue) {
        const uint32_t i = item0 + seq * 8u + xcd;
        if (i >= n_items) return;
        t = queue[i];
    } else {
        // each XCD walks a contiguous range of items
        const uint32_t per = gridDim.x / 8u / (uint32_t)nsub2;
        t = item0 + xcd * per + seq;
        if (t >= n_items) return;
    }
    const int tx = (int)(t % (uint32_t)a.ntx);
    t /= (uint32_t)a.ntx;
    const int ty = (int)(t % (uint32_t)a.nty);
    t /= (uint32_t)a.nty;
    if constexpr (FORM != kFormBlock) {
        __shared__ q32::Lds<SZ> lds;
        q32::field_block<SZ, STATS, SR, FORM == kFormAligned>(a, a.s_lo + (int)t, tx, ty, sub,
                                                              lds);
    } else {
        __shared__ Stage<T> stage[kWave];
        __shared__ T pend[fieldk::pend_elems<T, SZ>()];
        __shared__ fieldk::Pairs<SZ> pairs;
        fieldk::field_block<T, SZ, STATS, K, SR>(a, a.s_lo + (int)t, tx, ty, sub, stage, pend,
                                                 pairs);
    }
}

// Block-major binary image of a field: one wave takes 8 rows x 64 columns
// (8 blocks); each row's ballot gives one byte of each block's word.
template <typename T>
__global__ __launch_bounds__(256) void k_bits_blk(const T* field, int32_t nk, int32_t W,
                                                  int32_t H, T C, uint64_t* out) {
    const int lane = lane_id();
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int nbx = (W + 7) / 8, nby = (H + 7) / 8;
    const int chunks = (W + 63) / 64;
    const uint64_t n = (uint64_t)nk * (uint64_t)nby * (uint64_t)chunks;
    if (wave >= n) return;
    const int c = (int)(wave % (uint64_t)chunks);
    const uint64_t kb = wave / (uint64_t)chunks;           // plane * nby + block row
    const int by = (int)(kb % (uint64_t)nby);
    const uint64_t k = kb / (uint64_t)nby;
    const T* f = field + k * (uint64_t)W * (uint64_t)H;
    const int i = c * 64 + lane;
    uint64_t word = 0;                                     // lane b < 8: block c*8 + b
    // all eight rows are read before the first is used, at clamped places (a
    // load under a condition waits for its own value before the next one:
    // 32 planes of 2048^2 173 -> 99 us, 3.1 -> 5.4 TB/s)
    T v[8];
    const int ic = i < W ? i : W - 1;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int j = by * 8 + r;
        v[r] = f[(size_t)(j < H ? j : H - 1) * W + ic];
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const uint64_t m = ballot64(i < W && by * 8 + r < H && v[r] >= C);
        word |= ((m >> (8 * (lane & 7))) & 0xffull) << (8 * r);
    }
    if (lane < 8 && c * 8 + lane < nbx) out[kb * (uint64_t)nbx + (uint64_t)(c * 8 + lane)] = word;
}

// A launch holds at most 2^25 workgroups (a grid's threads are counted in 32
// bits); larger calls take several.
constexpr uint32_t kMaxGroups = 1u << 25;

uint32_t items_per_launch(int32_t tile) {
    const uint32_t nsub = (uint32_t)(tile / kBlockPix);
    return kMaxGroups / (nsub * nsub) / 8u * 8u;
}

template <typename T, int SZ, int K, bool SR, int FORM>
lsl_status launch_form(const FieldArgs& a, bool stats, const uint32_t* queue, uint32_t n_items,
                       hipStream_t st) {
    const uint32_t nsub2 = (uint32_t)(a.tile / kBlockPix) * (uint32_t)(a.tile / kBlockPix);
    const uint32_t per_launch = items_per_launch(a.tile);
    for (uint32_t i0 = 0; i0 < n_items; i0 += per_launch) {
        const uint32_t n = n_items - i0 < per_launch ? n_items - i0 : per_launch;
        const uint32_t blocks = (n + 7u) / 8u * 8u * nsub2;
        if (stats)
            k_field<T, SZ, true, K, SR, FORM><<<blocks, 64, 0, st>>>(a, queue, i0, i0 + n);
        else
            k_field<T, SZ, false, K, SR, FORM><<<blocks, 64, 0, st>>>(a, queue, i0, i0 + n);
        LSL_HIP(hipGetLastError());
    }
    return LSL_OK;
}

template <typename T, int SZ, int K, bool SR>
lsl_status launch_tk(const FieldArgs& a, bool stats, const uint32_t* queue, uint32_t n,
                     hipStream_t st) {
    if constexpr (std::is_same<T, float>::value && K == LSL_KERNEL_QUARTIC) {
        if constexpr (SZ >= 8) {
            if (field_form(a, SZ) == kFormAligned)
                return launch_form<T, SZ, K, SR, kFormAligned>(a, stats, queue, n, st);
        }
        if (field_form(a, SZ) != kFormBlock)
            return launch_form<T, SZ, K, SR, kFormGeneral>(a, stats, queue, n, st);
    }
    return launch_form<T, SZ, K, SR, kFormBlock>(a, stats, queue, n, st);
}

template <typename T, int SZ>
lsl_status launch_t(const FieldArgs& a, bool stats, const uint32_t* queue, uint32_t n,
                    hipStream_t st) {
    if constexpr (std::is_same<T, float>::value) {
        if (a.kernel == LSL_KERNEL_GAUSS && a.gauss_short)
            return a.strut_R
                       ? launch_tk<T, SZ, fieldk::kGaussShort, true>(a, stats, queue, n, st)
                       : launch_tk<T, SZ, fieldk::kGaussShort, false>(a, stats, queue, n, st);
    }
    if (a.kernel == LSL_KERNEL_GAUSS)
        return a.strut_R ? launch_tk<T, SZ, LSL_KERNEL_GAUSS, true>(a, stats, queue, n, st)
                         : launch_tk<T, SZ, LSL_KERNEL_GAUSS, false>(a, stats, queue, n, st);
    return a.strut_R ? launch_tk<T, SZ, LSL_KERNEL_QUARTIC, true>(a, stats, queue, n, st)
                     : launch_tk<T, SZ, LSL_KERNEL_QUARTIC, false>(a, stats, queue, n, st);
}

template <typename T>
lsl_status launch_dt(const FieldArgs& a, bool stats, const uint32_t* queue, uint32_t n,
                     hipStream_t st) {
    switch (slab_planes(a.slab, a.nk)) {
        case 1: return launch_t<T, 1>(a, stats, queue, n, st);
        case 2: return launch_t<T, 2>(a, stats, queue, n, st);
        case 4: return launch_t<T, 4>(a, stats, queue, n, st);
        case 8: return launch_t<T, 8>(a, stats, queue, n, st);
        default: return launch_t<T, 16>(a, stats, queue, n, st);
    }
}

}  // namespace

lsl_status launch_field(int dtype, const FieldArgs& a, bool stats, const uint32_t* queue,
                        hipStream_t st) {
    const uint64_t n_items = (uint64_t)(a.s_hi - a.s_lo + 1) * (uint64_t)a.ntx * (uint64_t)a.nty;
    if (n_items == 0 || a.nk <= 0) return LSL_OK;
    if (n_items > 0x7fffffffull) {               // (a slab group has fewer buckets)
        set_error("slice_field: too many work items in one launch");
        return LSL_EINTERNAL;
    }
    return dtype == LSL_F32 ? launch_dt<float>(a, stats, queue, (uint32_t)n_items, st)
                            : launch_dt<double>(a, stats, queue, (uint32_t)n_items, st);
}

uint32_t field_launches(int32_t tile, uint64_t n_items) {
    return (uint32_t)((n_items + items_per_launch(tile) - 1) / items_per_launch(tile));
}

lsl_status launch_bits_blk(int dtype, const void* field, int32_t nk, int32_t W, int32_t H,
                           double C, uint64_t* out, hipStream_t st) {
    const uint64_t waves = (uint64_t)nk * (uint64_t)((H + 7) / 8) * (uint64_t)((W + 63) / 64);
    if (waves == 0) return LSL_OK;
    const uint64_t blocks = (waves + 3) / 4;
    if (dtype == LSL_F32)
        k_bits_blk<float><<<(unsigned)blocks, 256, 0, st>>>((const float*)field, nk, W, H,
                                                            (float)C, out);
    else
        k_bits_blk<double><<<(unsigned)blocks, 256, 0, st>>>((const double*)field, nk, W, H, C,
                                                             out);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

}  // namespace lsl
