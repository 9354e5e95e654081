// Device-wide building blocks: fills, exclusive prefix sums and a stable LSD
// radix sort of 32-bit (key, value) pairs.  All stream-ordered, no host
// synchronisation, deterministic.
#include "common.hpp"

namespace lsl {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;   // 2048

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        T o = __shfl_up(v, d, kWave);
        if (lane >= d) v += o;
    }
    return v;
}

// Exclusive scan of one value per thread over a 256-thread block.  Returns
// the exclusive prefix; *block_total receives the block's sum.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* smem4, T* block_total) {
    const int lane = lane_id(), w = threadIdx.x >> 6;
    T inc = wave_inclusive_scan(v);
    if (lane == kWave - 1) smem4[w] = inc;
    __syncthreads();
    T before = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kScanThreads / kWave; ++i) {
        T s = smem4[i];
        if (i < w) before += s;
        tot += s;
    }
    __syncthreads();
    *block_total = tot;
    return before + inc - v;
}

// The thread's kScanItems consecutive values from position base on (zeros
// past n); whole runs are read with 16-byte loads (base is a multiple of
// kScanItems, so they are aligned whenever the array is).
template <typename T>
__device__ __forceinline__ T load_run(const T* in, size_t base, size_t n, T (&v)[kScanItems]) {
    if (base + kScanItems <= n && ((uintptr_t)in & 15u) == 0) {
        constexpr int per = 16 / sizeof(T);
        struct alignas(16) Pack {
            T x[per];
        };
#pragma unroll
        for (int i = 0; i < kScanItems / per; ++i) {
            const Pack p = reinterpret_cast<const Pack*>(in + base)[i];
#pragma unroll
            for (int j = 0; j < per; ++j) v[i * per + j] = p.x[j];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) v[i] = (base + i < n) ? in[base + i] : T(0);
    }
    T s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) s += v[i];
    return s;
}

template <typename T>
__device__ __forceinline__ void store_run(T* out, size_t base, size_t n, T pre,
                                          const T (&v)[kScanItems]) {
    T r[kScanItems];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        r[i] = pre;
        pre += v[i];
    }
    if (base + kScanItems <= n && ((uintptr_t)out & 15u) == 0) {
        constexpr int per = 16 / sizeof(T);
        struct alignas(16) Pack {
            T x[per];
        };
#pragma unroll
        for (int i = 0; i < kScanItems / per; ++i) {
            Pack p;
#pragma unroll
            for (int j = 0; j < per; ++j) p.x[j] = r[i * per + j];
            reinterpret_cast<Pack*>(out + base)[i] = p;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kScanItems; ++i)
            if (base + i < n) out[base + i] = r[i];
    }
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const T* in, size_t n, T* sums,
                                                              const T* also) {
    __shared__ T sm[4];
    if (blockIdx.y) {                  // the second array: its totals follow the first's
        in = also;
        sums += gridDim.x;
    }
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    T v[kScanItems];
    const T s = load_run(in, base, n, v);
    T tot;
    block_exclusive_scan(s, sm, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Single block: exclusive scan of n values, carry across chunks (in may be
// out).
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_one(const T* in, T* out, size_t n, T* also,
                                                           size_t also_step) {
    __shared__ T sm[4];
    if (blockIdx.y) in = out = also ? also : out + also_step;
    T carry = 0;
    for (size_t c = 0; c < n; c += kScanTile) {
        const size_t base = c + (size_t)threadIdx.x * kScanItems;
        T v[kScanItems];
        const T s = load_run((const T*)in, base, n, v);
        T tot;
        const T pre = block_exclusive_scan(s, sm, &tot) + carry;
        store_run(out, base, n, pre, v);
        carry += tot;
    }
}

// The scan of one tile.  RAW: sums holds the tiles' plain totals, and the
// block adds up those before it (a few loads per thread, cheaper than a
// launch of their own); else they have been scanned.
template <typename T, bool RAW>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const T* in, T* out, size_t n,
                                                            const T* sums, T* also) {
    __shared__ T sm[4];
    if (blockIdx.y) {
        in = out = also;
        sums += gridDim.x;
    }
    T before;
    if (RAW) {
        T s = 0;
        for (unsigned i = threadIdx.x; i < blockIdx.x; i += kScanThreads) s += sums[i];
        block_exclusive_scan(s, sm, &before);
    } else {
        before = sums[blockIdx.x];
    }
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    T v[kScanItems];
    const T s = load_run((const T*)in, base, n, v);
    T tot;
    const T pre = block_exclusive_scan(s, sm, &tot) + before;
    store_run(out, base, n, pre, v);
}

// Up to kScanOne values take one block (its chunks are serial, about 1 us
// each, against 2 us and more for another launch); up to kScanRaw tiles each
// block adds up the totals before it; beyond that (8M values) the totals get
// a scan of their own.
constexpr size_t kScanOne = 4 * (size_t)kScanTile;
constexpr size_t kScanRaw = 4096;

template <typename T>
lsl_status scan_impl(const T* in, T* out, size_t n, T* tmp, hipStream_t st, T* also) {
    const size_t nb = (n + kScanTile - 1) / kScanTile;
    const unsigned na = also ? 2u : 1u;
    if (n <= kScanOne) {
        if (n > 0) k_scan_one<T><<<dim3(1, na), kScanThreads, 0, st>>>(in, out, n, also, 0);
        LSL_HIP(hipGetLastError());
        return LSL_OK;
    }
    const dim3 grid((unsigned)nb, na);
    k_scan_reduce<T><<<grid, dim3(kScanThreads), 0, st>>>(in, n, tmp, also);
    if (nb <= kScanRaw) {
        k_scan_down<T, true><<<grid, dim3(kScanThreads), 0, st>>>(in, out, n, tmp, also);
    } else {
        k_scan_one<T><<<dim3(1, na), kScanThreads, 0, st>>>(tmp, tmp, nb, nullptr, nb);
        k_scan_down<T, false><<<grid, dim3(kScanThreads), 0, st>>>(in, out, n, tmp, also);
    }
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

// --------------------------------------------------------------------------
// Radix sort: stable, least significant digit first, 8 bits a pass.  Every
// wave owns a contiguous run of the block's items (64 ITEMS of them, in
// rounds of 64 lanes) and ranks them by itself: the lanes that hold the same
// digit find each other with eight ballots and take the next places of the
// wave's own counter of that digit, so that the ranking needs no barrier.
// The waves' counters are then summed in wave order.
//
//   up to kSortOne items: one block, the items in LDS from pass to pass, one
//     launch for the whole sort;
//   more: per pass a histogram, (above kSortRaw blocks, where every block
//     reading all of it takes longer than a launch: 57 blocks 19 us a pass
//     against 9 + 5) a scan of each digit's row of it, and a scatter that puts
//     its tile in order in LDS first, so that its stores run along the output.
//
// Small sorts are bound by launches and by the ranking's serial chain, large
// ones by the scattered stores.  Against five launches a pass (histogram,
// three of a scan, a scatter with four barriers per 256 items and stores
// straight from the ranks): binning and slicing 812 float64 struts 0.62 ->
// 0.50 ms, the support metrics' gradient over 2M incidences 0.273 -> 0.215 ms.
// --------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;    // 2048 pairs per block
constexpr int kOneThreads = 1024;
constexpr int kOneWaves = kOneThreads / kWave;
constexpr size_t kSortOne = (size_t)kOneThreads * kSortItems;   // 8192
constexpr size_t kSortRaw = 16;                         // blocks

// The wave's lanes with this lane's digit (valid lanes only).
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid) {
    uint64_t peers = ballot64(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = ballot64(bit);
        peers &= bit ? bb : ~bb;
    }
    return peers;
}

// Ranks the wave's items by digit, in item order: rank[r] is the number of
// the wave's earlier items with the digit of item r, and cnt[256] (LDS, the
// wave's own, zero before) the digits' totals.
template <bool DROP>
__device__ __forceinline__ void wave_rank(const uint32_t (&k)[kSortItems], int shift, size_t i0,
                                          size_t n, uint32_t* cnt, uint32_t (&rank)[kSortItems],
                                          int rounds) {
    const uint64_t lt = lanes_below(lane_id());
    volatile uint32_t* c = cnt;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if (r >= rounds) break;
        const bool valid = i0 + (size_t)r * kWave < n && !(DROP && k[r] == kNoKey);
        const uint32_t d = (k[r] >> shift) & 255u;
        const uint64_t peers = same_digit(d, valid);
        const uint32_t before = c[d];
        rank[r] = before + (uint32_t)__popcll(peers & lt);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt) == 0ull) c[d] = before + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
}

// 256 threads, one per digit: exclusive prefix of v over the digits
__device__ __forceinline__ uint32_t digit_scan(uint32_t v, uint32_t* sm4) {
    uint32_t tot;
    return block_exclusive_scan(v, sm4, &tot);
}

__global__ __launch_bounds__(kOneThreads) void k_radix_one(const uint32_t* kin,
                                                           const uint32_t* vin, uint32_t* kout,
                                                           uint32_t* vout, uint32_t n,
                                                           int key_bits) {
    __shared__ uint32_t sk[kSortOne], sv[kSortOne];
    __shared__ uint32_t cnt[kOneWaves][256];
    __shared__ uint32_t dsum[4];
    const int t = threadIdx.x, w = t / kWave;
    // the items in equal runs over all waves: as few rounds as will hold them
    const int rounds = (int)((n + kOneThreads - 1) / kOneThreads);
    const uint32_t i0 = (uint32_t)w * (uint32_t)(kWave * rounds) + (uint32_t)lane_id();
    uint32_t k[kSortItems], v[kSortItems], rank[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = i0 + (uint32_t)r * kWave;
        k[r] = r < rounds && i < n ? kin[i] : 0u;
        v[r] = !vin ? i : r < rounds && i < n ? vin[i] : 0u;
    }
    for (int shift = 0; shift < key_bits; shift += 8) {
        for (int i = t; i < kOneWaves * 256; i += kOneThreads) (&cnt[0][0])[i] = 0u;
        __syncthreads();
        wave_rank<false>(k, shift, i0, n, cnt[w], rank, rounds);
        __syncthreads();
        // digit t: the waves' counts become their first places
        uint32_t tot = 0, inc = 0;
        if (t < 256) {
#pragma unroll
            for (int q = 0; q < kOneWaves; ++q) {
                const uint32_t c = cnt[q][t];
                cnt[q][t] = tot;
                tot += c;
            }
            inc = wave_inclusive_scan(tot);
            if (lane_id() == kWave - 1) dsum[w] = inc;
        }
        __syncthreads();
        if (t < 256) {
            uint32_t base = inc - tot;
            for (int q = 0; q < w; ++q) base += dsum[q];
#pragma unroll
            for (int q = 0; q < kOneWaves; ++q) cnt[q][t] += base;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            if (r < rounds && i0 + (uint32_t)r * kWave < n) {
                const uint32_t pos = cnt[w][(k[r] >> shift) & 255u] + rank[r];
                sk[pos] = k[r];
                sv[pos] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kSortItems; ++r) {
            const uint32_t i = i0 + (uint32_t)r * kWave;
            k[r] = r < rounds && i < n ? sk[i] : 0u;
            v[r] = r < rounds && i < n ? sv[i] : 0u;
        }
    }
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = i0 + (uint32_t)r * kWave;
        if (r < rounds && i < n) {
            kout[i] = k[r];
            vout[i] = v[r];
        }
    }
}

// hist: RAW [block][digit], else [digit][block].  With n_dev the items are
// *n_dev <= n (blocks past them count nothing), with DROP the keys kNoKey are
// left out.
template <bool RAW, bool DROP>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint32_t* keys, size_t n,
                                                             const uint32_t* n_dev, int shift,
                                                             uint32_t* hist, uint32_t nblocks) {
    if (n_dev) n = *n_dev < n ? *n_dev : n;
    __shared__ uint32_t h[kSortWaves][256];
    const int t = threadIdx.x, w = t / kWave;
    const size_t i0 = (size_t)blockIdx.x * kSortTile + (size_t)w * (kWave * kSortItems) +
                      (size_t)lane_id();
    const uint64_t lt = lanes_below(lane_id());
    uint32_t k[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const size_t i = i0 + (size_t)r * kWave;
        k[r] = i < n ? keys[i] : 0u;
    }
    for (int q = 0; q < kSortWaves; ++q) h[q][t] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const bool valid = i0 + (size_t)r * kWave < n && !(DROP && k[r] == kNoKey);
        const uint32_t d = (k[r] >> shift) & 255u;
        const uint64_t peers = same_digit(d, valid);
        // one lane adds the group's size
        if (valid && (peers & lt) == 0ull) atomicAdd(&h[w][d], (uint32_t)__popcll(peers));
    }
    __syncthreads();
    const uint32_t s = (h[0][t] + h[1][t]) + (h[2][t] + h[3][t]);
    if (RAW)
        hist[(size_t)blockIdx.x * 256 + t] = s;
    else
        hist[(size_t)t * nblocks + blockIdx.x] = s;
}

// one block per digit: exclusive scan of its row, and its total
__global__ __launch_bounds__(kScanThreads) void k_radix_rows(uint32_t* hist, uint32_t nblocks,
                                                             uint32_t* dtot) {
    __shared__ uint32_t sm[4];
    uint32_t* row = hist + (size_t)blockIdx.x * nblocks;
    uint32_t carry = 0;
    for (uint32_t c = 0; c < nblocks; c += kScanThreads) {
        const uint32_t i = c + threadIdx.x;
        const uint32_t v = i < nblocks ? row[i] : 0u;
        uint32_t tot;
        const uint32_t pre = block_exclusive_scan(v, sm, &tot);
        if (i < nblocks) row[i] = carry + pre;
        carry += tot;
    }
    if (threadIdx.x == 0) dtot[blockIdx.x] = carry;
}

template <bool RAW, bool DROP>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, size_t n,
    const uint32_t* n_dev, int shift, const uint32_t* hist, const uint32_t* dtot,
    uint32_t nblocks) {
    if (n_dev) n = *n_dev < n ? *n_dev : n;
    if ((size_t)blockIdx.x * kSortTile >= n) return;
    __shared__ uint32_t cnt[kSortWaves][256];
    __shared__ uint32_t gbase[256];          // where the block's items of a digit go, less their
                                             // place in the block's own order
    __shared__ uint32_t sk[kSortTile], sv[kSortTile];
    __shared__ uint32_t sm[4], s_m;
    const int t = threadIdx.x, w = t / kWave;
    const size_t tile0 = (size_t)blockIdx.x * kSortTile;
    const uint32_t l0 = (uint32_t)w * (kWave * kSortItems) + (uint32_t)lane_id();
    const size_t i0 = tile0 + l0;
    uint32_t k[kSortItems], v[kSortItems], rank[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const size_t i = i0 + (size_t)r * kWave;
        k[r] = i < n ? kin[i] : 0u;
        v[r] = !vin ? (uint32_t)i : i < n ? vin[i] : 0u;       // (no values: the places)
    }
    // digit t: items of all blocks, and of the blocks before this one
    uint32_t all = 0, before = 0;
    if (RAW) {
#pragma unroll
        for (uint32_t b = 0; b < (uint32_t)kSortRaw; ++b) {
            const uint32_t x = b < nblocks ? hist[(size_t)b * 256 + t] : 0u;
            before += b < blockIdx.x ? x : 0u;
            all += x;
        }
    } else {
        all = dtot[t];
        before = hist[(size_t)t * nblocks + blockIdx.x];
    }
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) cnt[q][t] = 0u;
    __syncthreads();
    wave_rank<DROP>(k, shift, i0, n, cnt[w], rank, kSortItems);
    const uint32_t first = digit_scan(all, sm) + before;     // (barriers inside)
    uint32_t tot = 0;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) tot += cnt[q][t];
    uint32_t place = digit_scan(tot, sm);
    gbase[t] = first - place;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
        const uint32_t c = cnt[q][t];
        cnt[q][t] = place;
        place += c;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if (i0 + (size_t)r * kWave < n && !(DROP && k[r] == kNoKey)) {
            const uint32_t pos = cnt[w][(k[r] >> shift) & 255u] + rank[r];
            sk[pos] = k[r];
            sv[pos] = v[r];
        }
    }
    if (t == 255) s_m = place;                       // the tile's items
    __syncthreads();
    const uint32_t m = s_m;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const uint32_t i = (uint32_t)r * kSortThreads + (uint32_t)t;
        if (i < m) {
            const uint32_t key = sk[i];
            const uint32_t pos = gbase[(key >> shift) & 255u] + i;
            kout[pos] = key;
            vout[pos] = sv[i];
        }
    }
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_bytes0(uint8_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

unsigned grid_for(size_t n, unsigned threads) {
    size_t g = (n + threads - 1) / threads;
    if (g > 65536u * 4u) g = 65536u * 4u;
    return (unsigned)(g == 0 ? 1 : g);
}

}  // namespace

int scan_form(size_t n) {
    const size_t nb = (n + kScanTile - 1) / kScanTile;
    return n <= kScanOne ? 0 : nb <= kScanRaw ? 1 : 2;
}

int radix_form(size_t n) {
    const size_t nb = (n + kSortTile - 1) / kSortTile;
    return n <= 1 ? 0 : n <= kSortOne ? 1 : nb <= kSortRaw ? 2 : 3;
}

size_t scan_tmp_elems(size_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

lsl_status exclusive_scan_u32(const uint32_t* in, uint32_t* out, size_t n, uint32_t* tmp,
                              hipStream_t st, uint32_t* also) {
    return scan_impl<uint32_t>(in, out, n, tmp, st, also);
}

lsl_status exclusive_scan_u64(const uint64_t* in, uint64_t* out, size_t n, uint64_t* tmp,
                              hipStream_t st) {
    return scan_impl<uint64_t>(in, out, n, tmp, st, nullptr);
}

size_t radix_tmp_elems(size_t n) {
    const size_t nb = (n + kSortTile - 1) / kSortTile;
    return 256 * (nb == 0 ? 1 : nb) + 256;
}

namespace {
template <bool RAW, bool DROP>
void radix_pass(const uint32_t* ki, const uint32_t* vi, uint32_t* ko, uint32_t* vo, size_t n,
                const uint32_t* n_dev, int shift, uint32_t* hist, uint32_t nb, hipStream_t st) {
    uint32_t* dtot = hist + 256 * (size_t)nb;
    k_radix_hist<RAW, DROP><<<nb, kSortThreads, 0, st>>>(ki, n, n_dev, shift, hist, nb);
    if (!RAW) k_radix_rows<<<256, kScanThreads, 0, st>>>(hist, nb, dtot);
    k_radix_scatter<RAW, DROP><<<nb, kSortThreads, 0, st>>>(ki, vi, ko, vo, n, n_dev, shift, hist,
                                                            dtot, nb);
}
}  // namespace

int radix_passes(size_t n, int key_bits) {
    return n <= kSortOne ? 1 : (key_bits + 7) / 8;
}

lsl_status radix_sort_places(const uint32_t* keys, uint32_t* k0, uint32_t* v0, uint32_t* k1,
                             uint32_t* v1, size_t n, int key_bits, uint32_t* tmp,
                             hipStream_t st) {
    if (n == 0) return LSL_OK;
    if (key_bits < 1) key_bits = 1;
    const uint32_t *ki = keys, *vi = nullptr;
    if (n <= kSortOne) {
        k_radix_one<<<1, kOneThreads, 0, st>>>(ki, vi, k0, v0, (uint32_t)n, key_bits);
        LSL_HIP(hipGetLastError());
        return LSL_OK;
    }
    const size_t nb = (n + kSortTile - 1) / kSortTile;
    if (n > 0xffffffffull) {
        set_error("radix sort: too many items");
        return LSL_EINTERNAL;
    }
    uint32_t *ko = k0, *vo = v0, *kn = k1, *vn = v1;
    for (int shift = 0; shift < key_bits; shift += 8) {
        (nb <= kSortRaw ? radix_pass<true, false> : radix_pass<false, false>)(
            ki, vi, ko, vo, n, nullptr, shift, tmp, (uint32_t)nb, st);
        LSL_HIP(hipGetLastError());
        ki = ko;
        vi = vo;
        ko = kn;
        vo = vn;
        kn = (uint32_t*)ki;
        vn = (uint32_t*)vi;
    }
    return LSL_OK;
}

lsl_status radix_sort_pairs(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, size_t n,
                            int key_bits, uint32_t* tmp, int* which, hipStream_t st,
                            const uint32_t* n_keep) {
    *which = 0;
    if (n <= 1 || key_bits <= 0) return LSL_OK;
    if (n <= kSortOne) {
        k_radix_one<<<1, kOneThreads, 0, st>>>(k0, v0, k1, v1, (uint32_t)n, key_bits);
        LSL_HIP(hipGetLastError());
        *which = 1;
        return LSL_OK;
    }
    const size_t nb = (n + kSortTile - 1) / kSortTile;
    if (n > 0xffffffffull) {
        set_error("radix sort: too many items");
        return LSL_EINTERNAL;
    }
    const bool raw = nb <= kSortRaw;
    uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
    for (int shift = 0; shift < key_bits; shift += 8) {
        // the first pass drops the items without a key, the others find fewer
        const bool drop = n_keep && shift == 0;
        const uint32_t* nd = drop ? nullptr : n_keep;
        if (raw)
            (drop ? radix_pass<true, true> : radix_pass<true, false>)(ki, vi, ko, vo, n, nd, shift,
                                                                      tmp, (uint32_t)nb, st);
        else
            (drop ? radix_pass<false, true> : radix_pass<false, false>)(
                ki, vi, ko, vo, n, nd, shift, tmp, (uint32_t)nb, st);
        LSL_HIP(hipGetLastError());
        uint32_t* t;
        t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
        *which ^= 1;
    }
    return LSL_OK;
}

lsl_status fill_u32(uint32_t* p, uint32_t v, size_t n, hipStream_t st) {
    if (n == 0) return LSL_OK;
    k_fill_u32<<<grid_for(n, 256), 256, 0, st>>>(p, v, n);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

lsl_status fill_bytes0(void* p, size_t bytes, hipStream_t st) {
    if (bytes == 0) return LSL_OK;
    if (bytes % 4 == 0 && ((uintptr_t)p % 4) == 0)
        return fill_u32((uint32_t*)p, 0u, bytes / 4, st);
    k_fill_bytes0<<<grid_for(bytes, 256), 256, 0, st>>>((uint8_t*)p, bytes);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

}  // namespace lsl
