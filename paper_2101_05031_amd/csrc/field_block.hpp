// Per-block field evaluation of the general field kernel (see field.hip for
// the method).
#pragma once

#include "kernels.hpp"

namespace lsl {
namespace fieldk {

template <typename T>
struct Num;

template <>
struct Num<float> {
    static __device__ __forceinline__ float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float clamp_(float v, float lo, float hi) {
        return __builtin_amdgcn_fmed3f(v, lo, hi);
    }
    static __device__ __forceinline__ float fma_(float a, float b, float c) {
        return __builtin_fmaf(a, b, c);
    }
    static __device__ __forceinline__ float max_(float a, float b) { return __builtin_fmaxf(a, b); }
    static __device__ __forceinline__ float erf_(float x) { return erff(x); }
    static __device__ __forceinline__ float exp_(float x) { return expf(x); }
};

template <>
struct Num<double> {
    static __device__ __forceinline__ double sqrt_(double x) { return __builtin_sqrt(x); }
    static __device__ __forceinline__ double clamp_(double v, double lo, double hi) {
        return __builtin_fmin(__builtin_fmax(v, lo), hi);
    }
    static __device__ __forceinline__ double fma_(double a, double b, double c) {
        return __builtin_fma(a, b, c);
    }
    static __device__ __forceinline__ double max_(double a, double b) { return __builtin_fmax(a, b); }
    static __device__ __forceinline__ double erf_(double x) { return erf(x); }
    static __device__ __forceinline__ double exp_(double x) { return exp(x); }
};

// One (pixel, strut) term of the field.
template <typename T>
__device__ __forceinline__ T eval_term(const Stage<T>& e, T dX, T dY, T d2) {
    using N = Num<T>;
    const T du = N::fma_(dX, e.ux, dY * e.uy);                 // d.u
    const T al = e.ntc - du;                                     // alpha
    const T be = e.nbtc - du;                                    // beta
    const T H = N::fma_(du, du, N::fma_(e.mx2, dX, N::fma_(e.my2, dY, e.H0 - d2)));
    const T h = N::sqrt_(N::max_(H, T(0)));
    const T ca = N::clamp_(al, -h, h);
    const T cb = N::clamp_(be, -h, h);
    const T D = cb - ca;
    const T x2 = ca * ca, y2 = cb * cb, xy = ca * cb;
    const T q2 = x2 + y2;
    const T S1 = q2 + xy;
    const T S2 = N::fma_(q2, S1, -(xy * xy));
    const T u = N::fma_(T(-2.0 / 3.0), S1, H);
    const T Q = N::fma_(H, u, T(0.2) * S2);
    return (e.wq * D) * Q;
}

// The Gaussian variant's term: with the same H, h and clamped ends,
//   wq [exp(H k2) c0 (erf(cb k1) - erf(ca k1)) - (cb - ca)],
// wq = r exp(-R^2 k2), k1 = 1/(sigma sqrt 2), k2 = 1/(2 sigma^2),
// c0 = sigma sqrt(pi/2): exp(H k2) wq / r = exp(-dist(p, line)^2 k2).  An
// empty interval gives erf(x) - erf(x) = 0 and cb - ca = 0: an exact zero.
template <typename T>
__device__ __forceinline__ T eval_term_gauss(const Stage<T>& e, T dX, T dY, T d2, T k1, T k2,
                                             T c0) {
    using N = Num<T>;
    const T du = N::fma_(dX, e.ux, dY * e.uy);
    const T al = e.ntc - du;
    const T be = e.nbtc - du;
    const T H = N::fma_(du, du, N::fma_(e.mx2, dX, N::fma_(e.my2, dY, e.H0 - d2)));
    const T h = N::sqrt_(N::max_(H, T(0)));
    const T ca = N::clamp_(al, -h, h);
    const T cb = N::clamp_(be, -h, h);
    const T E = N::erf_(cb * k1) - N::erf_(ca * k1);
    return e.wq * N::fma_(N::exp_(H * k2) * c0, E, ca - cb);
}

// The Gaussian term of lattices whose supports stay within kGaussNear sigma
// (3 sigma is the usual choice), in float32.  Lengths are in units of
// sigma sqrt(2 / log2 e) (the staging scales them in float64), so that H is the
// exponent to base 2 itself, |x| <= h <= 2.577 at the ends, and
//
//   wq [2^H (F(cb) - F(ca)) - (cb - ca)],  F(x) = integral of 2^(-t^2) from 0
//   to x = x P(x^2),
//
// with P of degree 10 about x^2 = 3.4375 (minimax fit of F(x)/x on x^2 <= 6.64;
// of the centres in steps of 1/64 the one whose coefficients' rounding to
// float32 costs least: relative error 5.3e-9, mean 9e-10, so that a sum of
// many terms gains no bias), the difference of the two products rounded
// once, and 2^H from the hardware's exp2 with no rounding before it.  Emulated
// in float32 against float64, the form with erf and exp correctly rounded in
// brackets: at supports of 3 sigma a term is 1.8e-8 of the largest off in the
// mean square (2.1e-8), a sum of 40 terms 3.8e-8 (4.4e-8); no worse than that form
// at any support from 0.1 to 3.03 sigma.  No branches, where erff takes both of
// its own in most waves; bound by its instructions' issue.  16 planes of 2048^2
// of 1M struts: 4.3 ms with erff and expf, 2.5 ms so.
constexpr int kGaussShort = 2;                  // the kernel parameter of this form

__device__ __forceinline__ float gauss_poly(float x) {
    const float t = __builtin_fmaf(x, x, -3.4375f);
    float p = 4.4692621e-11f;
    p = __builtin_fmaf(p, t, -7.0460648e-10f);
    p = __builtin_fmaf(p, t, 9.396974e-09f);
    p = __builtin_fmaf(p, t, -1.2787227e-07f);
    p = __builtin_fmaf(p, t, 1.5704942e-06f);
    p = __builtin_fmaf(p, t, -1.7079133e-05f);
    p = __builtin_fmaf(p, t, 0.00016385793f);
    p = __builtin_fmaf(p, t, -0.0013756008f);
    p = __builtin_fmaf(p, t, 0.010109045f);
    p = __builtin_fmaf(p, t, -0.067659326f);
    return __builtin_fmaf(p, t, 0.55745947f);
}

__device__ __forceinline__ float eval_term_short(const Stage<float>& e, float dX, float dY,
                                                 float d2) {
    using N = Num<float>;
    const float du = N::fma_(dX, e.ux, dY * e.uy);
    const float al = e.ntc - du;
    const float be = e.nbtc - du;
    const float H = N::fma_(du, du, N::fma_(e.mx2, dX, N::fma_(e.my2, dY, e.H0 - d2)));
    const float h = N::sqrt_(N::max_(H, 0.0f));
    const float ca = N::clamp_(al, -h, h);
    const float cb = N::clamp_(be, -h, h);
    const float E = N::fma_(cb, gauss_poly(cb), -(ca * gauss_poly(ca)));
    return e.wq * N::fma_(__builtin_amdgcn_exp2f(H), E, ca - cb);
}

template <typename T>
__device__ __forceinline__ void comp_add(T t, T& s, T& c) {
    const T sn = s + t;
    c += t - (sn - s);
    s = sn;
}

// Terms per compensated add.  float32 adds each run of four consecutive
// candidates of a (block, plane) plainly, ((t0 + t1) + t2) + t3, and
// compensates once per run; float64 compensates every term, and so does the
// Gaussian term (two erf and one exp per pair dwarf the sum, and the runs'
// extra registers would spill).  Runs are counted
// over the whole candidate sequence of the (block, plane), across the 64-entry
// chunks of the bucket list: a run left open at the end of a chunk waits in
// LDS (`pend`, [SZ][64] per wave) for the next one.
template <typename T>
struct Group {
    static constexpr int n = 1;
};
template <>
struct Group<float> {
    static constexpr int n = 4;
};
template <typename T, int SZ>
constexpr int pend_elems() {
    return Group<T>::n > 1 ? SZ * kWave : 1;
}

// Staging works on (strut, plane) pairs.  Most entries of a bucket reach the
// block in few of the slab's planes (a bucket covers a whole tile and slab, and
// planes may lie far apart), so staging every entry for every plane would
// leave most lanes without a candidate.  For 64 entries at a time (one per
// lane) a float32 pre-test, with its rounding added to the support, finds the
// planes whose exact test may pass; those pairs are listed plane by plane in
// LDS, in entry order, and staged in float64, one per lane.  64 planes of 1024^2 of
// 115k struts, 1.6 mm apart: 605 -> 484 us.
template <int SZ>
struct Pairs {
    uint32_t id[kWave];                // the entries' edge-list positions
    uint16_t pair[SZ * kWave];         // entry | plane << 6
};

// One wave evaluates the 8x8 block `sub` of tile (tx, ty) over the planes of
// `slab` that lie in [k0, k0+nk); `stage` is the wave's 64-entry LDS area,
// `pend` its pend_elems<T, SZ>() open-run sums and `pl` its pair list.  K: LSL_KERNEL_QUARTIC, LSL_KERNEL_GAUSS
// or kGaussShort;
// SR: per-strut supports (in the record's pad) instead of one support R.
template <typename T, int SZ, bool STATS, int K, bool SR>
__device__ __forceinline__ void field_block(const FieldArgs& a, int slab, int tx, int ty, int sub,
                                            Stage<T>* stage, T* pend, Pairs<SZ>& pl) {
    constexpr bool kShort = K == kGaussShort;
    constexpr int G = K == LSL_KERNEL_QUARTIC ? Group<T>::n : 1;
    // the unit of length is 1 / lu (1, or the short Gaussian form's)
    const double lu = kShort ? a.gk1 * kSqrtLog2E : 1.0;
    const int lane = lane_id();
    const uint32_t n_binned = a.n_binned, n_pairs = a.n_pairs;
    const int nsub = a.tile / kBlockPix;
    const int i0 = tx * a.tile + (sub % nsub) * kBlockPix;
    const int j0 = ty * a.tile + (sub / nsub) * kBlockPix;
    if (i0 >= a.W || j0 >= a.H) return;
    int kb = slab * a.slab, ke = kb + a.slab;
    if (kb < a.k0) kb = a.k0;
    if (ke > a.k0 + a.nk) ke = a.k0 + a.nk;
    const int nvalid = ke - kb;

    const uint32_t bucket = ((uint32_t)(slab - a.group_s0) * (uint32_t)a.nty + (uint32_t)ty) *
                                (uint32_t)a.ntx + (uint32_t)tx;
    uint32_t beg = a.offsets[bucket], end = a.offsets[bucket + 1];
    if (end > n_pairs) end = n_pairs;
    if (beg > end) beg = end;

    const int lx = lane & 7, ly = lane >> 3;
    const int pi = i0 + lx, pj = j0 + ly;
    const bool pix = pi < a.W && pj < a.H;
    const double cx = a.x0 + ((double)i0 + 4.0) * a.dx;     // centre of the 8x8 centres
    const double cy = a.y0 + ((double)j0 + 4.0) * a.dy;
    const T dX = (T)(((double)lx - 3.5) * a.dx * lu);
    const T dY = (T)(((double)ly - 3.5) * a.dy * lu);
    const T d2 = dX * dX + dY * dY;
    // half extents of the block's pixel centres about c
    const double hx = 3.5 * a.dx, hy = 3.5 * a.dy;
    // one support: the (slightly widened) cull radius and R^2 are uniform
    const double Rc_u = a.R * (1.0 + 1e-7);
    const double Rc2_u = Rc_u * Rc_u;
    const double R2_u = a.R * a.R;
    const T gk1 = (T)a.gk1, gk2 = (T)a.gk2, gc0 = (T)a.gc0;

    // the block's pixel columns and rows (for the range test)
    const int ie = i0 + 7 < a.W - 1 ? i0 + 7 : a.W - 1;
    const int je = j0 + 7 < a.H - 1 ? j0 + 7 : a.H - 1;

    T acc_s[SZ], acc_c[SZ];
    int open[SZ];                       // terms in each plane's open run (wave-uniform)
#pragma unroll
    for (int k = 0; k < SZ; ++k) {
        acc_s[k] = acc_c[k] = T(0);
        open[k] = 0;
    }
    unsigned long long n_cand = 0, n_useful = 0;

    const StrutRec<T>* recs = (const StrutRec<T>*)a.rec;
    constexpr bool kScale = sizeof(T) == 8 || K != LSL_KERNEL_QUARTIC;
    const double sc_u = kScale ? __builtin_ldexp(1.0, -__builtin_amdgcn_frexp_exp(a.R)) : 1.0;
    for (uint32_t cbase = beg; cbase < end; cbase += kWave) {
        // ------------------------------------------------- pairs of 64 entries
        const uint32_t idx = cbase + (uint32_t)lane;
        bool valid = idx < end;
        uint32_t p = valid ? a.ids[idx] : 0u;
        valid = valid && p < n_binned;
        if (!valid) p = 0u;
        uint32_t near = 0u;             // bit k: the strut may reach the block at plane kb + k
        {
            // The strut is a candidate of this block and plane only where its
            // binned pixel and plane ranges cover them: then every tile size,
            // slab depth and group split hands the block the same candidates in
            // the same order, and the runs of four are the same.
            const PRange pr = a.pranges[p];
            valid = valid && (int)pr.i0 <= ie && (int)pr.i1 >= i0 && (int)pr.j0 <= je &&
                    (int)pr.j1 >= j0;
            const int klo = pr.k0 - kb > 0 ? pr.k0 - kb : 0;
            const int khi = pr.k1 - kb < nvalid - 1 ? pr.k1 - kb : nvalid - 1;
            if (valid && klo <= khi) near = (2u << khi) - (1u << klo);
        }
        if (SZ > 1) {
            const StrutRec<T> r = recs[p];
            const double4 ln = a.line[p];
            // Lengths over a power of two near the support: the test's fourth
            // powers of raw lengths leave float32's range from supports of 4e9 and
            // 1e-11 units on, and infinities or zeros compare as out of reach.
            // Scaled, a value that overflows makes err infinite (kept), and one
            // that underflows is far within the support.  (Not where the record's
            // r / R^4 has a narrower range of its own, float32 and the paper's
            // kernel: there the scaling cost 1%.)
            const double Rs = SR ? (double)r.pad : a.R;
            const double sc = !kScale ? 1.0
                              : SR    ? __builtin_ldexp(1.0, -__builtin_amdgcn_frexp_exp(Rs))
                                      : sc_u;
            const double wx = (cx - (double)r.ax) * sc, wy = (cy - (double)r.ay) * sc,
                         wz = (a.z0 + ((double)kb + 0.5) * a.dz - (double)r.az) * sc;
            const double dz = a.dz * sc;
            const float hxf = (float)(hx * sc), hyf = (float)(hy * sc);
            const double tc = fma(wx, ln.x, fma(wy, ln.y, wz * ln.z));
            const double mx = fma(tc, ln.x, -wx), my = fma(tc, ln.y, -wy), mz = fma(tc, ln.z, -wz);
            const float tc0 = (float)tc, L = (float)(ln.w * sc), ux = (float)ln.x, uy = (float)ln.y;
            const float mx0 = (float)mx, my0 = (float)my;
            const float m20 = (float)fma(mx, mx, fma(my, my, mz * mz));
            const float dtc = (float)(dz * ln.z);
            const float vx = (float)(dz * ln.z * ln.x), vy = (float)(dz * ln.z * ln.y);
            const float c1 = (float)(-2.0 * dz * mz), c2 = (float)(dz * dz * (1.0 - ln.z * ln.z));
            const float Rf = (float)(Rs * sc);
            const float Rw2 = Rf * Rf * 1.00002f;
            // what the rounding of the values below may add up to in D^2 and q
            const float T1 = fabsf(tc0) + (float)SZ * fabsf(dtc) + L;
            const float M1 = m20 + (float)SZ * fabsf(c1) + (float)(SZ * SZ) * c2;
            const float err = 4e-6f * (__builtin_fmaf(T1, T1, M1) + hxf * hxf + hyf * hyf);
            uint32_t pass = 0u;
#pragma unroll
            for (int k = 0; k < SZ; ++k) {
                const float kf = (float)k;
                const float tk = __builtin_fmaf(kf, dtc, tc0);
                const float dt = __builtin_amdgcn_fmed3f(tk, 0.0f, L) - tk;
                const float ex = __builtin_fmaf(dt, ux, __builtin_fmaf(kf, vx, mx0));
                const float ey = __builtin_fmaf(dt, uy, __builtin_fmaf(kf, vy, my0));
                const float m2 = __builtin_fmaf(kf * kf, c2, __builtin_fmaf(kf, c1, m20));
                const float D2 = __builtin_fmaf(dt, dt, m2);
                const float q = (D2 - err) - __builtin_fmaf(hxf, fabsf(ex), hyf * fabsf(ey));
                // (not a comparison that a NaN would fail)
                const bool far = q > 0.0f && q * q >= Rw2 * (D2 + err);
                pass |= far ? 0u : 1u << k;
            }
            near &= pass;
        }
        pl.id[lane] = p;
        int np = 0;
#pragma unroll
        for (int k = 0; k < SZ; ++k) {
            const bool on = (near >> k) & 1u;
            const uint64_t m = ballot64(on);
            if (on)
                pl.pair[np + (int)__builtin_amdgcn_mbcnt_hi(
                                 (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    (uint16_t)((uint32_t)lane | ((uint32_t)k << 6));
            np += __popcll(m);
        }
        __builtin_amdgcn_wave_barrier();

        for (int pb = 0; pb < np; pb += kWave) {
            // ------------------------------------------ staging, one pair per lane
            const bool has = pb + lane < np;
            const uint32_t pair = has ? (uint32_t)pl.pair[pb + lane] : 0u;
            const int kk = has ? (int)(pair >> 6) : -1;
            bool pass = false;
            Stage<T> s;
            {
                const uint32_t ps = pl.id[pair & 63u];
                const StrutRec<T> r = recs[ps];
                const double4 ln = a.line[ps];
                const double ux = ln.x, uy = ln.y, uz = ln.z, L = ln.w;
                const double wx = cx - (double)r.ax, wy = cy - (double)r.ay;
                const double txy = fma(wx, ux, wy * uy);
                const double z = a.z0 + ((double)(kb + kk) + 0.5) * a.dz;
                const double wz = z - (double)r.az;
                const double tc = fma(wz, uz, txy);
                const double mx = fma(tc, ux, -wx), my = fma(tc, uy, -wy), mz = fma(tc, uz, -wz);
                const double m2 = fma(mx, mx, fma(my, my, mz * mz));
                // e = F* - c, F* the point of the segment nearest to c, and
                // D = |e|.  The segment lies in the half-space n.(x - F*) >= 0
                // (n = e / D), so a pixel c + d of the block is at least
                // D - n.d >= D - (hx |e_x| + hy |e_y|) / D from it: the strut
                // reaches no pixel when D^2 - hx |e_x| - hy |e_y| >= R D.
                const double dt = fmin(fmax(tc, 0.0), L) - tc;
                const double ex = fma(dt, ux, mx), ey = fma(dt, uy, my);
                const double D2 = fma(dt, dt, m2);
                const double q = D2 - fma(hx, fabs(ex), hy * fabs(ey));
                double Rc2 = Rc2_u, R2 = R2_u;
                if (SR) {               // per-strut supports
                    const double Rs = (double)r.pad;
                    const double Rc = Rs * (1.0 + 1e-7);
                    Rc2 = Rc * Rc;
                    R2 = Rs * Rs;
                }
                pass = has && (q <= 0.0 || q * q < Rc2 * D2);
                s.mx2 = (T)(2.0 * mx * lu);
                s.my2 = (T)(2.0 * my * lu);
                s.ux = (T)ux;
                s.uy = (T)uy;
                s.ntc = (T)(-tc * lu);
                s.nbtc = (T)((L - tc) * lu);
                s.H0 = (T)((R2 - m2) * (lu * lu));
                s.wq = r.wq;
            }
            const uint64_t mask = ballot64(pass);
            if (mask == 0ull) continue;
            if (pass)                   // (its rank: the passing lanes below this one)
                stage[__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = s;
            __builtin_amdgcn_wave_barrier();

            // --------------------------- evaluation, the planes' runs of the list
            int j0s = 0;
#pragma unroll
            for (int k = 0; k < SZ; ++k) {
                const int n_k = __popcll(ballot64(pass && kk == k));
                if (n_k == 0) continue;
                const Stage<T>* st = stage + j0s;
                j0s += n_k;
                const int n = n_k;
                T s_ = acc_s[k], c_ = acc_c[k];
                auto term_at = [&](int j) -> T {
                    T t;
                    if constexpr (kShort)
                        t = eval_term_short(st[j], dX, dY, d2);
                    else if constexpr (K == LSL_KERNEL_GAUSS)
                        t = eval_term_gauss<T>(st[j], dX, dY, d2, gk1, gk2, gc0);
                    else
                        t = eval_term<T>(st[j], dX, dY, d2);
                    if (STATS) n_useful += t > T(0) ? 1ull : 0ull;
                    return t;
                };
                if (G == 1) {
                    for (int j = 0; j < n; ++j) comp_add(term_at(j), s_, c_);
                } else {
                    T* pk = pend + k * kWave + lane;
                    int q = open[k];
                    int j = 0;
                    if (q != 0) {               // complete the run left open
                        T g = *pk;
                        for (; j < n && q < G; ++j, ++q) g += term_at(j);
                        if (q == G) {
                            comp_add(g, s_, c_);
                            q = 0;
                        } else {
                            *pk = g;
                        }
                    }
#pragma unroll 1
                    for (; j + G <= n; j += G) {
                        T g = term_at(j);
#pragma unroll
                        for (int i = 1; i < G; ++i) g += term_at(j + i);
                        comp_add(g, s_, c_);
                    }
                    if (j < n) {                // open a run with the rest
                        T g = term_at(j);
                        for (q = 1, ++j; j < n; ++j, ++q) g += term_at(j);
                        *pk = g;
                    }
                    open[k] = q;
                }
                if (STATS) n_cand += pix ? (unsigned long long)n : 0ull;
                acc_s[k] = s_;
                acc_c[k] = c_;
            }
            __builtin_amdgcn_wave_barrier();
        }
        __builtin_amdgcn_wave_barrier();
    }

    if (G > 1) {
#pragma unroll
        for (int k = 0; k < SZ; ++k)
            if (open[k] != 0) comp_add(pend[k * kWave + lane], acc_s[k], acc_c[k]);
    }

    if (STATS) {
        if (!pix) n_useful = 0;
        for (int d = 32; d >= 1; d >>= 1) {
            n_cand += __shfl_xor(n_cand, d, kWave);
            n_useful += __shfl_xor(n_useful, d, kWave);
        }
        const unsigned long long npx = (unsigned long long)__popcll(ballot64(pix)) * nvalid;
        if (lane == 0) {
            atomicAdd(&a.stats[0], n_cand);
            atomicAdd(&a.stats[1], n_useful);
            atomicAdd(&a.stats[2], npx);
        }
        return;
    }
    if (pix && a.field) {
        T* out = (T*)a.field;
#pragma unroll
        for (int k = 0; k < SZ; ++k)
            if (k < nvalid)
                out[((size_t)(kb + k - a.k0) * (size_t)a.H + (size_t)pj) * (size_t)a.W + (size_t)pi] =
                    acc_s[k] + acc_c[k];
    }
    if (a.bits_blk || a.bits_rows) {
        // binary image: the block's ballot
        const T C = (T)a.C;
#pragma unroll
        for (int k = 0; k < SZ; ++k) {
            const uint64_t m = ballot64(pix && acc_s[k] + acc_c[k] >= C);
            if (lane == k) {                       // (through LDS: one copy of the stores' code)
                pl.id[2 * k] = (uint32_t)m;
                pl.id[2 * k + 1] = (uint32_t)(m >> 32);
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int k = 0; k < nvalid; ++k)
            store_bits(a, kb + k - a.k0, i0, j0,
                       (uint64_t)pl.id[2 * k] | ((uint64_t)pl.id[2 * k + 1] << 32), lane);
    }
}


}  // namespace fieldk
}  // namespace lsl
