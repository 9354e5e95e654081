// Marching squares on the binary slice images (Sec. 4: rough boundary
// curves from the binary image).  The images are block-major: one 64-bit
// word per 8x8 pixel block, bit 8 r + c = pixel (8 bx + c, 8 by + r).
//
// Cell (i, j) has corners (i,j), (i+1,j), (i+1,j+1), (i,j+1) -> bits b0..b3
// of its case code.  For the 64 cells of a block these are four 64-bit masks
// built from the block word and its right, lower and lower-right neighbours
// with shifts, so one lane finds all boundary cells of a block at once:
//   M = (b0|b1|b2|b3) & ~(b0&b1&b2&b3)       cells with one or two segments
//   S = saddles 5 and 10                        cells with two segments
// A strip is 8 pixel rows of one plane, a chunk 64 of its blocks (one per
// lane):
//
//   count: one wave per strip: popcount(M) + popcount(S) per row, kept per
//          chunk and summed per strip
//   scan : exclusive prefix over (plane, strip) -> per-plane offsets
//   emit : one wave per chunk: the rows' places follow from the strip's
//          scanned offset and the counts of the rows above and the chunks to
//          the left; a wave prefix of the per-(row, block) counts ranks every
//          boundary cell in row-major order.
//
// The emit pass lists the chunk's segments in LDS in that order and writes
// one per lane, so that a row's stores run along the output.  One wave per
// strip, walking its chunks in turn and listing cells block by block, was
// bound by its serial chain and by scattered stores: 5.7M sub-pixel segments of
// 32 planes of 2048^2 239 -> 171 us, 40 planes of 2979 x 2983 103 -> 60 us.
//
// Segment ends are edge midpoints in grid units; the inside lies on the left
// of each segment; the saddles 5 and 10 keep the two inside corners apart.
// Outputs are deterministic and written with no atomics.
#include <algorithm>

#include "grid.hpp"
#include "kernels.hpp"
#include "splitters.hpp"

namespace lsl {
namespace {

constexpr int kMThreads = 256;

// chunks of 64 blocks in a strip
size_t strip_chunks(int32_t W) { return (size_t)(((W + 7) / 8 + kWave - 1) / kWave); }

constexpr uint64_t kCol0 = 0x0101010101010101ull;   // column 0 of every row
constexpr uint64_t kCol7 = 0x8080808080808080ull;   // column 7 of every row

// Per case: up to two segments (5 and 10 have two, 0 and 15 none) as
// (x0, y0, x1, y1) in half units of the cell.  The table is folded at
// compile time into register constants (kSegWord), so a lane's lookup by its
// own case is arithmetic, not a memory load.
// edge midpoints in half units: B=(1,0) E=(2,1) T=(1,2) L=(0,1)
constexpr int8_t kSegT[16][2][4] = {
    {{0, 0, 0, 0}, {0, 0, 0, 0}},
    {{1, 0, 0, 1}, {0, 0, 0, 0}},   // 1: B -> L
    {{2, 1, 1, 0}, {0, 0, 0, 0}},   // 2: E -> B
    {{2, 1, 0, 1}, {0, 0, 0, 0}},   // 3: E -> L
    {{1, 2, 2, 1}, {0, 0, 0, 0}},   // 4: T -> E
    {{1, 0, 0, 1}, {1, 2, 2, 1}},   // 5: B -> L, T -> E
    {{1, 2, 1, 0}, {0, 0, 0, 0}},   // 6: T -> B
    {{1, 2, 0, 1}, {0, 0, 0, 0}},   // 7: T -> L
    {{0, 1, 1, 2}, {0, 0, 0, 0}},   // 8: L -> T
    {{1, 0, 1, 2}, {0, 0, 0, 0}},   // 9: B -> T
    {{2, 1, 1, 0}, {0, 1, 1, 2}},   // 10: E -> B, L -> T
    {{2, 1, 1, 2}, {0, 0, 0, 0}},   // 11: E -> T
    {{0, 1, 2, 1}, {0, 0, 0, 0}},   // 12: L -> E
    {{1, 0, 2, 1}, {0, 0, 0, 0}},   // 13: B -> E
    {{0, 1, 1, 0}, {0, 0, 0, 0}},   // 14: L -> B
    {{0, 0, 0, 0}, {0, 0, 0, 0}},
};

// cases 4w .. 4w+3, 16 bits each: segment s in bits 8s .. 8s+7, its
// coordinates (each 0, 1 or 2) in 2 bits apiece, x0 lowest
constexpr uint64_t seg_word(int w) {
    uint64_t r = 0;
    for (int c = 0; c < 4; ++c)
        for (int s = 0; s < 2; ++s)
            for (int e = 0; e < 4; ++e)
                r |= (uint64_t)kSegT[4 * w + c][s][e] << (16 * c + 8 * s + 2 * e);
    return r;
}
constexpr uint64_t kSegWord[4] = {seg_word(0), seg_word(1), seg_word(2), seg_word(3)};

// segment s of case cs as (x0, y0, x1, y1) in half units
__device__ __forceinline__ void seg_points(int cs, int s, int8_t g[4]) {
    const int w = cs >> 2;
    const uint64_t word = w == 0 ? kSegWord[0] : w == 1 ? kSegWord[1]
                        : w == 2 ? kSegWord[2] : kSegWord[3];
    const uint32_t b = (uint32_t)(word >> (16 * (cs & 3) + 8 * s)) & 0xffu;
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = (int8_t)((b >> (2 * e)) & 3u);
}


// The four corner masks of the 64 cells of block (bx, by) of one plane, with
// the cells outside [0, W-1) x [0, H-1) cleared from M and S.
struct CellMasks {
    uint64_t b0, b1, b2, b3, m, s;
};

__device__ __forceinline__ CellMasks cell_masks(const uint64_t* P, int nbx, int nby, int bx,
                                                int by, int32_t W, int32_t H) {
    const size_t row = (size_t)by * (size_t)nbx;
    const bool right = bx + 1 < nbx, down = by + 1 < nby;
    const uint64_t w = P[row + bx];
    const uint64_t wr = right ? P[row + bx + 1] : 0ull;
    const uint64_t wd = down ? P[row + nbx + bx] : 0ull;
    const uint64_t wdr = (right && down) ? P[row + nbx + bx + 1] : 0ull;
    CellMasks c;
    c.b0 = w;
    c.b1 = ((w >> 1) & ~kCol7) | ((wr & kCol0) << 7);              // pixel (i+1, j)
    c.b3 = (w >> 8) | (wd << 56);                                   // pixel (i, j+1)
    const uint64_t b1d = ((wd >> 1) & ~kCol7) | ((wdr & kCol0) << 7);
    c.b2 = (c.b1 >> 8) | (b1d << 56);                               // pixel (i+1, j+1)
    int nc = W - 1 - 8 * bx, nr = H - 1 - 8 * by;                   // valid cell columns / rows
    nc = nc < 0 ? 0 : (nc > 8 ? 8 : nc);
    nr = nr < 0 ? 0 : (nr > 8 ? 8 : nr);
    const uint64_t cols = (uint64_t)((1u << nc) - 1u) * kCol0;
    const uint64_t rows = nr >= 8 ? ~0ull : ((1ull << (8 * nr)) - 1ull);
    const uint64_t valid = cols & rows;
    const uint64_t all = c.b0 & c.b1 & c.b2 & c.b3;
    const uint64_t any = c.b0 | c.b1 | c.b2 | c.b3;
    c.m = any & ~all & valid;
    c.s = ((c.b0 & c.b2 & ~c.b1 & ~c.b3) | (c.b1 & c.b3 & ~c.b0 & ~c.b2)) & valid;
    return c;
}

// v + v of the lane the DPP control selects (0 where it selects none)
template <int CTRL, int ROWS, int BANKS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t acc, uint32_t v) {
    return acc + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, BANKS, false);
}

// inclusive prefix over the wave's lanes with DPP moves: within rows of 16
// (shifts by 1, 2, 3 of the inputs, then by 4 and 8 of the partial sums),
// then across rows (broadcasts of lanes 15 and 31)
__device__ __forceinline__ uint32_t wave_incl32(uint32_t v) {
    const uint32_t v0 = v;
    v = dpp_add<0x111, 0xf, 0xf>(v0, v0);          // row_shr:1
    v = dpp_add<0x112, 0xf, 0xf>(v, v0);           // row_shr:2
    v = dpp_add<0x113, 0xf, 0xf>(v, v0);           // row_shr:3
    v = dpp_add<0x114, 0xf, 0xe>(v, v);            // row_shr:4, lanes 4..15 of a row
    v = dpp_add<0x118, 0xf, 0xc>(v, v);            // row_shr:8, lanes 8..15
    v = dpp_add<0x142, 0xa, 0xf>(v, v);            // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc, 0xf>(v, v);            // row_bcast:31 into rows 2 and 3
    return v;
}

// the same for 64-bit words of packed counts whose fields never carry (the
// low halves' sums stay below 2^32)
__device__ __forceinline__ uint64_t wave_incl(uint64_t v, int) {
    return (uint64_t)wave_incl32((uint32_t)v) | ((uint64_t)wave_incl32((uint32_t)(v >> 32)) << 32);
}

__device__ __forceinline__ uint64_t wave_last(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, kWave - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), kWave - 1);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// total over the wave of packed counts that never carry
__device__ __forceinline__ uint64_t wave_total(uint64_t v) { return wave_last(wave_incl(v, 0)); }

// segments of row r (0..7) of a block: one per boundary cell, two per saddle
__device__ __forceinline__ uint32_t row_count(const CellMasks& c, int r) {
    return (uint32_t)(__popc((uint32_t)(c.m >> (8 * r)) & 0xffu) +
                      __popc((uint32_t)(c.s >> (8 * r)) & 0xffu));
}

// segments of the block's rows 4q .. 4q + 3, 16 bits each
__device__ __forceinline__ uint64_t row_counts4(const CellMasks& c, int q) {
    uint64_t v = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) v |= (uint64_t)row_count(c, 4 * q + h) << (16 * h);
    return v;
}

// rows r, r + 1 (r even) of a pair of 16-bit words as 32-bit halves
__device__ __forceinline__ uint64_t widen2(const uint64_t (&v)[2], int r) {
    const uint64_t w = v[r >> 2] >> (16 * (r & 3));
    return (w & 0xffffull) | ((w & 0xffff0000ull) << 16);
}

// Segments per strip (tot), per row of the strip (rows: two rows per word,
// 32 bits each, lower row in the low half) and per row of each chunk (crows:
// four rows per word, 16 bits each; a row of a chunk holds at most
// 2 x 8 x 64 = 1024 segments).
__global__ __launch_bounds__(kMThreads) void k_strip_count(const uint64_t* img, int32_t nk,
                                                           int32_t W, int32_t H,
                                                           unsigned long long* tot,
                                                           unsigned long long* rows,
                                                           unsigned long long* crows) {
    const int lane = lane_id();
    const int nbx = (W + 7) / 8, nby = (H + 7) / 8, nch = (nbx + kWave - 1) / kWave;
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (wave >= (uint64_t)nk * (uint64_t)nby) return;
    const uint64_t k = wave / (uint64_t)nby;
    const int by = (int)(wave % (uint64_t)nby);
    const uint64_t* P = img + k * (uint64_t)nby * (uint64_t)nbx;
    uint64_t t2[4] = {0, 0, 0, 0};
    for (int ch = 0; ch < nch; ++ch) {
        const int bx = ch * kWave + lane;
        CellMasks c{};
        if (bx < nbx) c = cell_masks(P, nbx, nby, bx, by, W, H);
        uint64_t all[2] = {0, 0};
        if (ballot64(c.m != 0ull) != 0ull) {
#pragma unroll
            for (int q = 0; q < 2; ++q) all[q] = wave_total(row_counts4(c, q));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) t2[q] += widen2(all, 2 * q);
        if (lane == 0) {
            crows[2 * (wave * (uint64_t)nch + (uint64_t)ch)] = all[0];
            crows[2 * (wave * (uint64_t)nch + (uint64_t)ch) + 1] = all[1];
        }
    }
    uint64_t cnt = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) cnt += (t2[q] & 0xffffffffull) + (t2[q] >> 32);
    if (lane == 0) {
        tot[wave] = cnt;
#pragma unroll
        for (int q = 0; q < 4; ++q) rows[4 * wave + q] = t2[q];
    }
}

__global__ void k_ms_offsets(const unsigned long long* scan, uint32_t per_plane, int32_t nk,
                             const unsigned long long* base, int64_t* offsets) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k <= nk) offsets[k] = (int64_t)(scan[(size_t)k * per_plane] + (base ? *base : 0ull));
}

// base += this call's total (the segments of several calls share one array)
__global__ void k_ms_advance(unsigned long long* base, const unsigned long long* scan,
                             size_t n) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *base += scan[n];
}

// Optional outputs of the emit pass for sub-pixel segments and chaining:
// endpoints interpolated on the field, each segment's start and end edge and
// its cell.  Edge ids per plane: 2 (y W + x) for the edge (x,y)-(x+1,y),
// 2 (y W + x) + 1 for (x,y)-(x,y+1).
struct SubPix {
    const void* field;                // [nk][H][W], T
    double C;
    uint32_t* edge_s;                 // [total] start edge of each segment
    uint32_t* edge_e;                 // [total] end edge
    uint32_t* cell;                   // [total] j (W-1) + i
};

// One end of a segment of cell (i, j) at table point g (half units): its
// edge id and, for SUB, the point where g - C interpolates to zero along the
// edge, from its lower-(j, i) grid point P to Q.
template <bool SUB, typename T>
__device__ __forceinline__ float2 seg_end(const int8_t* g, int i, int j, int32_t W, const T* f,
                                          T C, uint32_t* edge) {
    if (!SUB) return make_float2((float)i + 0.5f * g[0], (float)j + 0.5f * g[1]);   // midpoint
    if (!(g[1] & 1)) {                              // horizontal edge at y = j + g/2
        const int y = j + (g[1] >> 1);
        *edge = 2u * ((uint32_t)y * (uint32_t)W + (uint32_t)i);
        const T gp = f[(size_t)y * W + i], gq = f[(size_t)y * W + i + 1];
        return make_float2((float)((T)i + (C - gp) / (gq - gp)), (float)y);
    }
    const int x = i + (g[0] >> 1);                  // vertical edge at x = i + g/2
    *edge = 2u * ((uint32_t)j * (uint32_t)W + (uint32_t)x) + 1u;
    const T gp = f[(size_t)j * W + x], gq = f[(size_t)(j + 1) * W + x];
    return make_float2((float)x, (float)((T)j + (C - gp) / (gq - gp)));
}

constexpr uint32_t kList = 512;        // segments listed per wave and round

template <bool SUB, typename T>
__global__ __launch_bounds__(kMThreads) void k_strip_emit(uint64_t block0, const uint64_t* img,
                                                          uint64_t n_chunks,
                                                          int32_t W, int32_t H,
                                                          const unsigned long long* scan,
                                                          const unsigned long long* rows,
                                                          const unsigned long long* crows,
                                                          const unsigned long long* base,
                                                          float4* segs, int64_t capacity,
                                                          SubPix sp) {
    // a listed segment: column in the chunk | row << 9 | case << 12 | which of
    // the case's two << 16
    __shared__ uint32_t s_list[kMThreads / kWave][kList];
    __shared__ uint64_t s_shift[kMThreads / kWave][8];
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const int nbx = (W + 7) / 8, nby = (H + 7) / 8, nch = (nbx + kWave - 1) / kWave;
    const uint64_t item = (block0 + blockIdx.x) * (kMThreads / kWave) + (uint64_t)w;
    if (item >= n_chunks) return;
    const uint64_t all[2] = {crows[2 * item], crows[2 * item + 1]};
    if ((all[0] | all[1]) == 0ull) return;
    const uint64_t strip = item / (uint64_t)nch;
    const int ch = (int)(item % (uint64_t)nch);
    const uint64_t k = strip / (uint64_t)nby;
    const int by = (int)(strip % (uint64_t)nby);
    const uint64_t* P = img + k * (uint64_t)nby * (uint64_t)nbx;
    const int bx = ch * kWave + lane;
    CellMasks c{};
    if (bx < nbx) c = cell_masks(P, nbx, nby, bx, by, W, H);
    // the counts of the chunks to the left, per row
    uint64_t left[4] = {0, 0, 0, 0};
    for (int q = 0; q < ch; ++q) {
        const uint64_t v[2] = {crows[2 * (item - (uint64_t)ch + (uint64_t)q)],
                               crows[2 * (item - (uint64_t)ch + (uint64_t)q) + 1]};
#pragma unroll
        for (int h = 0; h < 4; ++h) left[h] += widen2(v, 2 * h);
    }
    // row r's segments take places first[r] .. of the list, and list place p
    // of row r goes to position p + shift[r] of the output
    uint32_t first[8], n_seg = 0;
    {
        uint64_t run = scan[strip] + (base ? *base : 0ull);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint32_t lw = (uint32_t)(left[r >> 1] >> (32 * (r & 1)));
            first[r] = n_seg;
            if (lane == 0) s_shift[w][r] = run + lw - (uint64_t)n_seg;
            run += (uint32_t)(rows[4 * strip + (r >> 1)] >> (32 * (r & 1)));
            n_seg += (uint32_t)(all[r >> 2] >> (16 * (r & 3))) & 0xffffu;
        }
    }
    uint64_t ex[2];                    // the lane's places within the rows
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint64_t v = row_counts4(c, q);
        ex[q] = wave_incl(v, lane) - v;
    }
    const T* f = SUB ? (const T*)sp.field + k * (uint64_t)W * (uint64_t)H : nullptr;
    uint32_t* list = s_list[w];
    for (uint32_t R = 0; R < n_seg; R += kList) {
        uint64_t mb = c.m;
        int rcur = -1;
        uint32_t p = 0;
        while (mb) {
            const int bit = __ffsll((unsigned long long)mb) - 1;
            mb &= mb - 1ull;
            const int r = bit >> 3;
            if (r != rcur) {
                uint32_t fr = first[0];
#pragma unroll
                for (int q = 1; q < 8; ++q) fr = r == q ? first[q] : fr;
                p = fr + ((uint32_t)(ex[r >> 2] >> (16 * (r & 3))) & 0xffffu) - R;
                rcur = r;
            }
            const uint32_t cs = (uint32_t)((c.b0 >> bit) & 1ull) |
                                ((uint32_t)((c.b1 >> bit) & 1ull) << 1) |
                                ((uint32_t)((c.b2 >> bit) & 1ull) << 2) |
                                ((uint32_t)((c.b3 >> bit) & 1ull) << 3);
            const uint32_t e = (uint32_t)(8 * lane + (bit & 7)) | ((uint32_t)r << 9) | (cs << 12);
            if (p < kList) list[p] = e;                   // (unsigned: earlier rounds' are skipped)
            ++p;
            if ((c.s >> bit) & 1ull) {
                if (p < kList) list[p] = e | (1u << 16);
                ++p;
            }
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t m = n_seg - R < kList ? n_seg - R : kList;
        for (uint32_t q = (uint32_t)lane; q < m; q += kWave) {
            const uint32_t e = list[q];
            const int r = (int)(e >> 9) & 7, cs = (int)(e >> 12) & 15, sg = (int)(e >> 16);
            const uint64_t os = s_shift[w][r] + (uint64_t)(R + q);
            const int ci = ch * 8 * kWave + (int)(e & 511u), cj = 8 * by + r;
            if ((int64_t)os < capacity) {
                int8_t g[4];
                seg_points(cs, sg, g);
                uint32_t es = 0, ee = 0;
                const float2 a = seg_end<SUB, T>(g, ci, cj, W, f, (T)sp.C, &es);
                const float2 b = seg_end<SUB, T>(g + 2, ci, cj, W, f, (T)sp.C, &ee);
                segs[os] = make_float4(a.x, a.y, b.x, b.y);
                if (SUB) {
                    sp.edge_s[os] = es;
                    sp.edge_e[os] = ee;
                    sp.cell[os] = (uint32_t)cj * (uint32_t)(W - 1) + (uint32_t)ci;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Case code of every cell, [nk][H-1][W-1] bytes (optional output).
__global__ __launch_bounds__(kMThreads) void k_ms_codes(const uint64_t* img, int32_t W, int32_t H,
                                                        uint8_t* codes) {
    const uint32_t k = blockIdx.y;
    const int nbx = (W + 7) / 8, nby = (H + 7) / 8;
    const uint64_t cw = (uint64_t)(W - 1), cps = cw * (uint64_t)(H - 1);
    const uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cps) return;
    const int j = (int)(c / cw), i = (int)(c % cw);
    const uint64_t* P = img + (uint64_t)k * (uint64_t)nby * (uint64_t)nbx;
    auto at = [&](int x, int y) -> uint32_t {
        const uint64_t w = P[(size_t)(y >> 3) * (size_t)nbx + (size_t)(x >> 3)];
        return (uint32_t)(w >> (8 * (y & 7) + (x & 7))) & 1u;
    };
    codes[(uint64_t)k * cps + c] =
        (uint8_t)(at(i, j) | (at(i + 1, j) << 1) | (at(i + 1, j + 1) << 2) | (at(i, j + 1) << 3));
}

// Row-major copy of block-major images: word w of row j holds pixels
// 32 w .. 32 w + 31 (bit x % 32 is pixel x).  A thread reads the four block
// words of one output column and block row once and writes its eight rows
// (byte r of each block word is row r of the block).
__global__ __launch_bounds__(256) void k_bits_rows(const uint64_t* img, uint64_t n, int32_t W,
                                                   int32_t H, uint32_t* out) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int words = (W + 31) / 32, nbx = (W + 7) / 8, nby = (H + 7) / 8;
    const int w = (int)(t % (uint64_t)words);
    const uint64_t kb = t / (uint64_t)words;
    const int by = (int)(kb % (uint64_t)nby);
    const uint64_t k = kb / (uint64_t)nby;
    const uint64_t* row = img + (k * (uint64_t)nby + (uint64_t)by) * (uint64_t)nbx;
    uint64_t q[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int bx = 4 * w + c;
        q[c] = bx < nbx ? row[bx] : 0ull;
    }
    uint32_t* o = out + (k * (uint64_t)H + (uint64_t)(8 * by)) * (uint64_t)words + (uint64_t)w;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (8 * by + r < H) {
            uint32_t v = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) v |= (uint32_t)((q[c] >> (8 * r)) & 0xffull) << (8 * c);
            o[(uint64_t)r * (uint64_t)words] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// Chaining.  Segment s of plane k ends on edge e; the segment that starts on
// e lies in the cell across e and follows s.  In the same row that cell's
// segments are next to s in the list; in the row above or below they are found
// by a binary search of the row, whose place in the list the count pass left.
//
// Chains and ranks.  Jumping pointers over all segments costs a pass over
// the whole list per round (two sets of 1 + log2(longest) rounds), so only
// splitters take part: chain starts, segments smaller than both neighbours
// (so every closed loop has one, its smallest segment among them) and about one
// segment in kSplit by its index (splitters.hpp).
//   1. Each splitter walks to the next one, kSplit steps on average along a
//      chain of scattered indices; the segments it passes learn it and their
//      distance from it.
//   2. Jumping among the splitters: X is the splitter 2^r further on (or the
//      chain's last), dX the distance to it, M the smallest segment index
//      among the next 2^r splitters (-1 once they run past the end of an open
//      chain) and dM the distance to it.  A round that changes no M is the
//      last: M is then -1 all along an open chain, and X its last splitter,
//      and the smallest index of a loop all along the loop (a window's
//      minimum equals the next window's, hence every window's).
//   3. A chain's start leaves its distance to the last splitter there; the
//      smallest segment of a loop finds the loop's length in its own dM.  A
//      splitter's rank is that less its own distance, and a segment's rank
//      its splitter's plus its distance from it.
// All integer: bitwise deterministic (the splitters' numbering is not, and
// no result depends on it).  Bound by gathers over the list: 5.7M segments in
// 32 planes (1.2M splitters, loops of up to 10^5 segments) take 0.49 ms for
// steps 1-3, against 1.76 ms for 2 x 17 rounds over all segments.
constexpr uint32_t kSuccMask = 0x3fffffffu;        // fewer than 2^30 segments
constexpr uint32_t kSuccNone = 0x80000000u;        // end of an open chain
constexpr uint32_t kSuccSplit = 0x40000000u;       // the successor is a splitter

__device__ __forceinline__ uint32_t plane_between(const int64_t* off, uint32_t lo, uint32_t hi,
                                                  uint64_t s) {
    while (hi - lo > 1) {                          // off[lo] <= s < off[hi]
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint64_t)off[mid] <= s) lo = mid; else hi = mid;
    }
    return lo;
}

// position of the first segment of cell row j of plane k, and of the next row
__device__ __forceinline__ void row_span(const unsigned long long* scan,
                                         const unsigned long long* rows, uint32_t nby, uint32_t k,
                                         int j, uint64_t* a, uint64_t* b) {
    const uint64_t strip = (uint64_t)k * nby + (uint64_t)(j >> 3);
    uint64_t pos = scan[strip];
    const int r = j & 7;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t t = rows[4 * strip + q];
        const uint64_t lo = t & 0xffffffffull, hi = t >> 32;
        if (r == 2 * q) {
            *a = pos;
            *b = pos + lo;
        }
        pos += lo;
        if (r == 2 * q + 1) {
            *a = pos;
            *b = pos + hi;
        }
        pos += hi;
    }
}

// Successors.  Bound by the search's serial chain of gathers, so each block
// keeps the cells of its 256 segments and of the 256 before and after them in
// LDS, and rows that lie within are searched there (the row above or below is
// at most two rows' segments away); longer rows in memory.  5.7M segments of 32
// planes of 2048^2 (87 to a row): 117 -> 95 us.
constexpr uint32_t kSuccSide = 256;
__global__ __launch_bounds__(256) void k_poly_succ(const int64_t* off, int32_t nk, uint64_t total,
                                                   int32_t W, int32_t H,
                                                   const unsigned long long* scan,
                                                   const unsigned long long* rows,
                                                   const uint32_t* edge_s, const uint32_t* edge_e,
                                                   const uint32_t* cell, int32_t* succ,
                                                   int32_t* pred) {
    __shared__ uint32_t s_k[2];
    __shared__ uint32_t s_cell[256 + 2 * kSuccSide];
    const uint64_t s0 = (uint64_t)blockIdx.x * 256u;
    if (threadIdx.x < 2) {                         // planes of the block's first and last segment
        const uint64_t q = threadIdx.x == 0 ? s0 : (s0 + 255 < total ? s0 + 255 : total - 1);
        s_k[threadIdx.x] = plane_between(off, 0u, (uint32_t)nk, q);
    }
    // the segments [w0, w1) in s_cell
    const uint64_t w0 = s0 < kSuccSide ? 0 : s0 - kSuccSide;
    const uint64_t w1 = s0 + 256 + kSuccSide < total ? s0 + 256 + kSuccSide : total;
    for (uint64_t q = w0 + threadIdx.x; q < w1; q += 256) s_cell[q - w0] = cell[q];
    __syncthreads();
    const uint64_t s = s0 + threadIdx.x;
    if (s >= total) return;
    const uint32_t k = plane_between(off, s_k[0], s_k[1] + 1, s);
    const uint32_t cw = (uint32_t)(W - 1);
    const uint32_t c = s_cell[s - w0], i = c % cw, j = c / cw;
    const uint32_t e = edge_e[s], at = e >> 1;
    int64_t r = -1;
    if (e & 1u) {                                  // vertical edge: the cell beside, same row
        const int x = (int)(at % (uint32_t)W);
        const bool left = x == (int)i;
        if (left ? i > 0u : i + 1u < cw) {
            const uint64_t lo = (uint64_t)off[k], hi = (uint64_t)off[k + 1];
            const uint32_t nc = left ? c - 1u : c + 1u;
#pragma unroll
            for (uint64_t d = 1; d <= 3; ++d) {    // at most two segments per cell
                const uint64_t q = left ? s - d : s + d;
                if ((left ? s >= lo + d : q < hi) && s_cell[q - w0] == nc && edge_s[q] == e)
                    r = (int64_t)q;
            }
        }
    } else {                                       // horizontal edge: the row above or below
        const int nj = at / (uint32_t)W == j ? (int)j - 1 : (int)j + 1;
        if (nj >= 0 && nj < H - 1) {
            const uint32_t nc = (uint32_t)nj * cw + i;
            uint64_t a = 0, b = 0;
            row_span(scan, rows, (uint32_t)((H + 7) / 8), k, nj, &a, &b);
            const uint64_t end = b;
            if (a >= w0 && b <= w1) {              // first position with cell >= nc
                const uint32_t last = (uint32_t)(b - w0);
                uint32_t x = (uint32_t)(a - w0), y = last;
                while (x < y) {
                    const uint32_t mid = (x + y) >> 1;
                    if (s_cell[mid] < nc) x = mid + 1; else y = mid;
                }
                for (uint32_t q = x; q < last && q < x + 2 && s_cell[q] == nc; ++q)
                    if (edge_s[w0 + q] == e) r = (int64_t)(w0 + q);
            } else {
                while (a < b) {
                    const uint64_t mid = (a + b) >> 1;
                    if (cell[mid] < nc) a = mid + 1; else b = mid;
                }
                for (uint64_t q = a; q < end && q < a + 2 && cell[q] == nc; ++q)
                    if (edge_s[q] == e) r = (int64_t)q;
            }
        }
    }
    succ[s] = (int32_t)r;
    if (r >= 0) pred[r] = (int32_t)s;              // (each edge starts one segment)
}

__device__ __forceinline__ bool is_splitter(int32_t s, int32_t before, int32_t after) {
    if (before < 0) return true;
    if (after >= 0 && s < before && s < after) return true;
    return split_pick((uint32_t)s);
}

// Numbers the splitters (own = {number, 0}, seg = their segments) and marks
// the links that lead to one.  A block takes 2048 segments for one addition
// to the shared count (256 for each: 259 us for 5.7M segments, bound by the
// additions to one address; 50 us).
constexpr uint32_t kMarkItems = 8;

__global__ __launch_bounds__(256) void k_poly_mark(const int32_t* succ, const int32_t* pred,
                                                   uint32_t total, uint32_t cap, uint32_t* link,
                                                   int2* own, uint32_t* seg, uint32_t* count) {
    __shared__ uint32_t wsum[4], s_base;
    const int lane = lane_id(), w = threadIdx.x >> 6;
    // wave w: segments s0 + 64 r + lane
    const uint32_t s0 = blockIdx.x * (256u * kMarkItems) + (uint32_t)w * (64u * kMarkItems) +
                        (uint32_t)lane;
    uint64_t m[kMarkItems];
    uint32_t n = 0;
#pragma unroll
    for (uint32_t r = 0; r < kMarkItems; ++r) {
        const uint32_t s = s0 + 64u * r;
        bool sp = false;
        if (s < total) {
            const int32_t nx = succ[s];
            sp = is_splitter((int32_t)s, pred[s], nx);
            uint32_t l = kSuccNone;
            if (nx >= 0)
                l = (uint32_t)nx | (is_splitter(nx, (int32_t)s, succ[nx]) ? kSuccSplit : 0u);
            link[s] = l;
        }
        m[r] = ballot64(sp);
        n += (uint32_t)__popcll(m[r]);
    }
    if (lane == 0) wsum[w] = n;
    __syncthreads();
    if (threadIdx.x == 0) s_base = atomicAdd(count, wsum[0] + wsum[1] + wsum[2] + wsum[3]);
    __syncthreads();
    uint32_t a = s_base;
    for (int q = 0; q < w; ++q) a += wsum[q];
#pragma unroll
    for (uint32_t r = 0; r < kMarkItems; ++r) {
        const uint32_t i = a + (uint32_t)__popcll(m[r] & lanes_below(lane));
        if (((m[r] >> lane) & 1ull) && i < cap) {
            own[s0 + 64u * r] = make_int2((int)i, 0);
            seg[i] = s0 + 64u * r;
        }
        a += (uint32_t)__popcll(m[r]);
    }
}

// The splitters of one block: a contiguous range, neighbouring ranges on one
// XCD, so that what a plane's splitters gather from each other stays in one L2.
__device__ __forceinline__ void splitter_range(uint32_t n, uint32_t* beg, uint32_t* end) {
    const uint32_t per = ((n + gridDim.x - 1u) / gridDim.x + 255u) & ~255u;
    const uint64_t b = (uint64_t)xcd_remap(blockIdx.x, gridDim.x) * per;
    *beg = b < n ? (uint32_t)b : n;
    *end = b + per < n ? (uint32_t)(b + per) : n;
}

__global__ __launch_bounds__(256) void k_poly_walk(const uint32_t* link, const uint32_t* seg,
                                                   const uint32_t* count, uint32_t cap,
                                                   uint32_t total, int2* own, int4* state) {
    const uint32_t n = *count < cap ? *count : cap;
    uint32_t beg, end;
    splitter_range(n, &beg, &end);
    for (uint32_t a = beg + threadIdx.x; a < end; a += 256u) {
        uint32_t x = seg[a];
        int4 st = make_int4((int)a, -1, 0, 0);     // the last splitter of an open chain
        for (uint32_t d = 1; d <= total; ++d) {    // (a chain holds at most `total` segments)
            const uint32_t l = link[x];
            if (l & kSuccNone) break;
            x = l & kSuccMask;
            if (l & kSuccSplit) {
                st = make_int4(own[x].x, (int)x, (int)d, (int)d);
                break;
            }
            own[x] = make_int2((int)a, (int)d);
        }
        state[a] = st;
    }
}

// One round of jumps, state = (X, M, dM, dX).  changed[r] says whether round
// r has anything to do (round 0 does); the round after the last finds 0.
__global__ __launch_bounds__(256) void k_poly_jump(const int4* in, int4* out,
                                                   const uint32_t* count, uint32_t cap,
                                                   const uint32_t* changed, uint32_t* next) {
    if (changed && *changed == 0u) return;
    const uint32_t n = *count < cap ? *count : cap;
    bool any = false;
    uint32_t beg, end;
    splitter_range(n, &beg, &end);
    for (uint32_t a = beg + threadIdx.x; a < end; a += 256u) {
        int4 s = in[a];
        const int4 x = in[s.x];
        if (x.y < s.y) {
            s.y = x.y;
            s.z = (int)((uint32_t)s.w + (uint32_t)x.z);
            any = true;
        }
        s.x = x.x;
        s.w = (int)((uint32_t)s.w + (uint32_t)x.w);
        out[a] = s;
    }
    if (ballot64(any) != 0ull && lane_id() == 0) *next = 1u;
}

// the buffer that the last round wrote (0 or 1)
__device__ __forceinline__ int last_state(const uint32_t* changed, int32_t rounds) {
    int r = 1;                                     // round 0 always runs
    while (r < rounds && changed[r] != 0u) ++r;
    return r & 1;
}

__global__ __launch_bounds__(256) void k_poly_heads(const int4* s0, const int4* s1,
                                                    const uint32_t* changed, int32_t rounds,
                                                    const uint32_t* seg, const int32_t* pred,
                                                    const uint32_t* count, uint32_t cap,
                                                    int2* head) {
    const int4* st = last_state(changed, rounds) ? s1 : s0;
    const uint32_t n = *count < cap ? *count : cap;
    uint32_t beg, end;
    splitter_range(n, &beg, &end);
    for (uint32_t a = beg + threadIdx.x; a < end; a += 256u) {
        const int4 s = st[a];
        const int32_t p = (int32_t)seg[a];
        if (s.y < 0) {
            if (pred[p] < 0) head[s.x] = make_int2(p, s.w);
        } else if (s.y == p) {
            head[a] = make_int2(p, s.z);
        }
    }
}

// per splitter: its chain's start (index within the plane) and its rank
__global__ __launch_bounds__(256) void k_poly_rank(const int4* s0, const int4* s1,
                                                   const uint32_t* changed, int32_t rounds,
                                                   const int2* own, const int2* head,
                                                   const int64_t* off, int32_t nk,
                                                   const uint32_t* count, uint32_t cap,
                                                   int2* res) {
    const int4* st = last_state(changed, rounds) ? s1 : s0;
    const uint32_t n = *count < cap ? *count : cap;
    uint32_t beg, end;
    splitter_range(n, &beg, &end);
    for (uint32_t a = beg + threadIdx.x; a < end; a += 256u) {
        const int4 s = st[a];
        const int2 h = s.y < 0 ? head[s.x] : head[own[s.y].x];
        const uint32_t k = plane_between(off, 0u, (uint32_t)nk, (uint64_t)h.x);
        res[a] = make_int2(h.x - (int32_t)off[k], h.y - (s.y < 0 ? s.w : s.z));
    }
}

__global__ __launch_bounds__(256) void k_poly_out(const int2* own, const int2* res, uint64_t total,
                                                  int32_t* chain, int32_t* rank) {
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= total) return;
    const int2 o = own[s];
    const int2 r = res[o.x];
    chain[s] = r.x;
    rank[s] = r.y + o.y;
}

}  // namespace

// tmp: per-strip totals (n + 1, scanned in place), the scan's scratch, then
// the per-row totals of every strip (4 words per strip) and of every chunk
// (2 words per chunk)
size_t contour_tmp_elems(int32_t nk, int32_t W, int32_t H) {
    const size_t n = (size_t)nk * (size_t)((H + 7) / 8);
    return (n + 1) + scan_tmp_elems(n + 1) + 4 * n + 2 * n * strip_chunks(W);
}

namespace {
constexpr int32_t kPolyRounds = 32;

// Scratch of slice_polylines, 16-byte aligned parts.  The links and the
// splitters' segments take the place of the emit pass's edge lists, which
// have been read by then.
struct PolyScratch {
    uint32_t *link, *seg;             // [total], [cap]: over edge_s, edge_e
    int32_t *succ, *pred;             // [total]
    int2* res;                        // [cap]
    int2* own;                        // [total]
    int4* state[2];                   // [cap]
    int2* head;                       // [cap]
    uint32_t *count, *changed;        // splitters; one flag per round
};
size_t up4(size_t n) { return (n + 3) & ~(size_t)3; }
PolyScratch poly_scratch(uint32_t* p, uint64_t total, uint32_t cap) {
    const size_t t = up4((size_t)total), c = up4((size_t)cap);
    PolyScratch s;
    s.link = p;
    s.seg = p + t;
    s.succ = (int32_t*)(p + 3 * t);
    s.pred = s.succ + t;
    s.own = (int2*)(p + 5 * t);
    uint32_t* q = p + 7 * t;
    s.state[0] = (int4*)q;
    s.state[1] = (int4*)(q + 4 * c);
    s.head = (int2*)(q + 8 * c);
    s.res = (int2*)(q + 10 * c);
    s.count = q + 12 * c;
    s.changed = s.count + 1;
    return s;
}
}  // namespace

size_t polyline_scratch_elems(uint64_t total, int32_t nk, int32_t W, int32_t H) {
    return 7 * up4((size_t)total) + 12 * up4(poly_splitters(total, nk, W, H)) + kPolyRounds + 8;
}

namespace {
unsigned long long* strip_rows(unsigned long long* tmp, size_t n) {
    return tmp + (n + 1) + scan_tmp_elems(n + 1);
}
unsigned long long* chunk_rows(unsigned long long* tmp, size_t n) {
    return strip_rows(tmp, n) + 4 * n;
}
uint64_t emit_blocks(size_t chunks) { return (chunks + kMThreads / kWave - 1) / (kMThreads / kWave); }

template <bool SUB, typename T>
void emit_launch(const uint64_t* img, size_t n, int32_t W, int32_t H,
                 const unsigned long long* tmp, const unsigned long long* base, float* segs,
                 int64_t capacity, const SubPix& sp, hipStream_t st) {
    unsigned long long* t = (unsigned long long*)tmp;
    const size_t chunks = n * strip_chunks(W);
    for_launches(emit_blocks(chunks), kMThreads, [&](uint64_t block0, uint32_t blocks) {
        k_strip_emit<SUB, T><<<blocks, kMThreads, 0, st>>>(
            block0, img, chunks, W, H, tmp, strip_rows(t, n), chunk_rows(t, n), base,
            (float4*)segs, capacity, sp);
    });
}
}  // namespace

lsl_status launch_contours_count(const uint64_t* img, int32_t nk, int32_t W, int32_t H,
                                 int64_t* offsets, uint8_t* codes, unsigned long long* tmp,
                                 const unsigned long long* base, hipStream_t st) {
    const uint32_t nby = (uint32_t)((H + 7) / 8);
    const size_t n = (size_t)nk * nby;
    if (n > 0x7fffffffull / 4) {
        set_error("slice_contours: too many planes in one call");
        return LSL_EINVAL;
    }
    unsigned long long* tot = tmp;
    unsigned long long* stmp = tmp + n + 1;
    if (W > 1 && H > 1)
        k_strip_count<<<(unsigned)((n + 3) / 4), kMThreads, 0, st>>>(img, nk, W, H, tot,
                                                                     strip_rows(tmp, n),
                                                                     chunk_rows(tmp, n));
    else
        LSL_TRY(fill_bytes0(tot, n * 8, st));
    LSL_HIP(hipGetLastError());
    if (codes && W > 1 && H > 1) {
        const uint64_t cps = (uint64_t)(W - 1) * (uint64_t)(H - 1);
        const uint64_t words = (uint64_t)((H + 7) / 8) * (uint64_t)((W + 7) / 8);
        for (int32_t k = 0; k < nk; k += 65535) {        // grid y holds at most 65535 planes
            const int32_t m = nk - k < 65535 ? nk - k : 65535;
            const dim3 grid((unsigned)((cps + kMThreads - 1) / kMThreads), (unsigned)m);
            k_ms_codes<<<grid, kMThreads, 0, st>>>(img + (uint64_t)k * words, W, H,
                                                   codes + (uint64_t)k * cps);
        }
        LSL_HIP(hipGetLastError());
    }
    // exclusive scan over n + 1 entries: the last one receives the total
    LSL_TRY(fill_bytes0(tot + n, 8, st));
    LSL_TRY(exclusive_scan_u64((const uint64_t*)tot, (uint64_t*)tot, n + 1, (uint64_t*)stmp,
                               st));
    k_ms_offsets<<<(nk + 1 + 255) / 256, 256, 0, st>>>(tot, nby, nk, base, offsets);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

lsl_status launch_contours_emit(const uint64_t* img, int32_t nk, int32_t W, int32_t H,
                                const unsigned long long* tmp, unsigned long long* base,
                                float* segs, int64_t capacity, hipStream_t st) {
    const uint32_t nby = (uint32_t)((H + 7) / 8);
    const size_t n = (size_t)nk * nby;
    if (W > 1 && H > 1)
        emit_launch<false, float>(img, n, W, H, tmp, base, segs, capacity, SubPix{}, st);
    if (base) k_ms_advance<<<1, 64, 0, st>>>(base, tmp, n);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

uint32_t contour_launches(int32_t nk, int32_t W, int32_t H) {
    const size_t n = (size_t)nk * (size_t)((H + 7) / 8);
    return (uint32_t)launch_count(emit_blocks(n * strip_chunks(W)), kMThreads);
}

lsl_status launch_bits_rows(const uint64_t* img, int32_t nk, int32_t W, int32_t H,
                            uint32_t* bits, hipStream_t st) {
    const uint64_t n = (uint64_t)nk * (uint64_t)((H + 7) / 8) * (uint64_t)((W + 31) / 32);
    if (n == 0) return LSL_OK;
    k_bits_rows<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(img, n, W, H, bits);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

lsl_status launch_polylines(const uint64_t* img, const void* field, int dtype, double C,
                            int32_t nk, int32_t W, int32_t H, const unsigned long long* tmp,
                            const int64_t* offsets, uint64_t total, int32_t rounds, float* segs,
                            uint32_t* scratch, int32_t* chain, int32_t* rank, hipStream_t st) {
    if (total == 0 || W < 2 || H < 2) return LSL_OK;
    const uint32_t nby = (uint32_t)((H + 7) / 8);
    const size_t n = (size_t)nk * nby;
    SubPix sp;
    sp.field = field;
    sp.C = C;
    const size_t part = up4((size_t)total);
    sp.edge_s = scratch;
    sp.edge_e = scratch + part;
    sp.cell = scratch + 2 * part;
    if (dtype == LSL_F32)
        emit_launch<true, float>(img, n, W, H, tmp, nullptr, segs, (int64_t)total, sp, st);
    else
        emit_launch<true, double>(img, n, W, H, tmp, nullptr, segs, (int64_t)total, sp, st);
    LSL_HIP(hipGetLastError());
    if (!chain || !rank) return LSL_OK;
    const uint32_t cap = poly_splitters(total, nk, W, H);
    const PolyScratch ps = poly_scratch(scratch, total, cap);
    const unsigned g = (unsigned)((total + 255) / 256);
    // the splitters' passes: enough blocks to fill the GPU, each over several
    const unsigned gs = std::min((cap + 255u) / 256u, 2048u);
    // the search ends after at most ceil(log2(longest chain)) rounds
    const int32_t jumps = std::min(std::max(rounds - 1, 1), kPolyRounds);
    LSL_TRY(fill_u32(ps.count, 0u, 1 + kPolyRounds + 1, st));
    LSL_TRY(fill_u32((uint32_t*)ps.pred, 0xffffffffu, total, st));
    k_poly_succ<<<g, 256, 0, st>>>(offsets, nk, total, W, H, tmp,
                                   strip_rows((unsigned long long*)tmp, n), sp.edge_s, sp.edge_e,
                                   sp.cell, ps.succ, ps.pred);
    k_poly_mark<<<(unsigned)((total + 2047) / 2048), 256, 0, st>>>(ps.succ, ps.pred, (uint32_t)total, cap, ps.link, ps.own, ps.seg,
                                   ps.count);
    k_poly_walk<<<gs, 256, 0, st>>>(ps.link, ps.seg, ps.count, cap, (uint32_t)total, ps.own,
                                    ps.state[0]);
    for (int32_t r = 0; r < jumps; ++r)
        k_poly_jump<<<gs, 256, 0, st>>>(ps.state[r & 1], ps.state[(r + 1) & 1], ps.count, cap,
                                        r > 0 ? ps.changed + r : nullptr, ps.changed + r + 1);
    k_poly_heads<<<gs, 256, 0, st>>>(ps.state[0], ps.state[1], ps.changed, jumps, ps.seg, ps.pred,
                                     ps.count, cap, ps.head);
    k_poly_rank<<<gs, 256, 0, st>>>(ps.state[0], ps.state[1], ps.changed, jumps, ps.own, ps.head,
                                    offsets, nk, ps.count, cap, ps.res);
    k_poly_out<<<g, 256, 0, st>>>(ps.own, ps.res, total, chain, rank);
    LSL_HIP(hipGetLastError());
    return LSL_OK;
}

}  // namespace lsl
