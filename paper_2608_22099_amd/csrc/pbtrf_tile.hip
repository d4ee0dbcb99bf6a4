// Band Cholesky for kd <= 144: panels of 16 columns, the trailing triangle on
// the matrix cores (the Cholesky case the paper names beside LU, end of
// Sec. II-B).  (Batches of small systems go by columns: chol_columns().)
//
// What bounds it is the chain of n column steps (update of the next diagonal
// entry, square root, reciprocal, scaling), not the n*kd^2 operations.  One
// workgroup per matrix keeps the 16-row tiles that the band's window covers in
// LDS (lower triangle only; a tile is 16 x 16, column-major) and overlaps the
// chain of one panel with the trailing update of the panel before it:
//   phase 1  (all waves) the tiles of the next panel's columns take the panel's
//            update;
//   phase 2  wave 0 factors the next panel, one row per lane and up to three
//            rows per lane, its 16 columns in registers (a pivot column
//            reaches the lanes by lane reads, so the chain has no LDS trip);
//            the other waves apply the panel to the remaining tiles, store it
//            to the band and bring in the tile row that the panel after next
//            reaches.
// Waves 1-3 and 5-7 do phase 2's matrix work: wave 4 shares its SIMD with
// wave 0, whose step is bound by its instruction issue.
//
// Every entry takes its fused multiply-adds one column step after another
// (v_mfma_f64_16x16x4f64 sums in ascending order with one rounding each), so
// the factor is bitwise that of the unblocked loops.  Rows that only some of a
// panel's columns reach (the band's edge) meet multipliers that are
// structurally zero: a no-op except on a -0.0 or against an infinity or NaN.
// Those, pivots outside the plain square root's range and a pivot that is not
// positive are looked for, and the tile or panel is then redone step by step.
//
// Measured (ms, against the kernel it replaced: one column step at a time for
// the whole workgroup): n = 32768, kd = 140: 206.9 -> 10.9; n = 20000, kd = 100:
// 85.9 -> 5.2; n = 8192, kd = 64: 21.4 -> 1.7; kd = 16: 8.3 -> 1.4; 1024
// systems of n = 256, kd = 16: 0.377 -> 0.124 (two workgroups per CU for
// kd <= 48).  A panel of kd = 140 takes about 14500 cycles: 1100-2400 phase 1,
// then wave 0 700 for its rows, 365 a column step and 1300 for the results,
// beside 12000 of the helpers (3400 the entering row, 1700 a pair of tiles).
#include <algorithm>
#include <climits>

#include "bufio.hpp"
#include "pbtrf_tile.hpp"

namespace bandlu {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kB = 16;          // panel width and tile edge
constexpr int kTile = kB * kB;  // doubles in a tile
constexpr int kThreads = kCholTileThreads;
constexpr int kHelpers = 384;   // threads of the waves that work in phase 2 beside wave 0

// sqrt(d) and 1/sqrt(d) for d in [2^-600, 2^600]: Goldschmidt's iteration from
// the hardware's estimate, then corrections by the exact residual (fma) until the
// root and the quotient are correctly rounded, as sqrt and 1/x are; such values
// need no scaling.
__device__ __forceinline__ void sqrt_recip(double d, double &g, double &r) {
    const double y = __builtin_amdgcn_rsq(d);
    const double s0 = d * y, h0 = y * 0.5;
    const double r0 = __builtin_fma(-h0, s0, 0.5);
    const double h1 = __builtin_fma(h0, r0, h0), s1 = __builtin_fma(s0, r0, s0);
    const double d0 = __builtin_fma(-s1, s1, d);
    const double s2 = __builtin_fma(d0, h1, s1);
    const double d1 = __builtin_fma(-s2, s2, d);
    g = __builtin_fma(d1, h1, s2);
    const double q = __builtin_amdgcn_rcp(g);
    const double e0 = __builtin_fma(-g, q, 1.0);
    const double q1 = __builtin_fma(q, e0, q);
    const double e1 = __builtin_fma(-g, q1, 1.0);
    const double q2 = __builtin_fma(q1, e1, q1);
    const double e2 = __builtin_fma(-g, q2, 1.0);
    r = __builtin_fma(e2, q2, q2);
}

__device__ __forceinline__ bool is_neg_zero(double v) {
    return __double_as_longlong(v) == (1ll << 63);
}

// Keeps an update in its step: the compiler otherwise runs the chain of the
// first row set alone, keeps every pivot column in scalar registers (spilled
// to lanes) and updates the other row sets afterwards.
__device__ __forceinline__ double pin(double v) {
    asm volatile("" : "+v"(v));
    return v;
}

// T: tile rows that a panel reaches, 16 (T - 2) < kd <= 16 (T - 1)
template <int T>
__global__ __launch_bounds__(kThreads, 2) void pbtrf_tile_kernel(CholParams P) {
    extern __shared__ double tiles[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = P.n, kd = P.kd;
    double *AB = P.AB + int64_t(blockIdx.x) * P.strideAB;
    const int64_t ldab = P.ldab;
    constexpr int RPL = (kB * T + 63) / 64;  // rows per lane of wave 0
    constexpr int W = T + 2;                 // tile rows in the window
    constexpr int kPairs = T > 2 ? (T - 1) / 2 * ((T - 1) / 2 + 1) - ((T - 1) % 2 ? 0 : (T - 1) / 2) : 0;
    const int np = (n + kB - 1) / kB;      // panels
    const int edge = (kd + 1) / kB;        // first tile row (from the panel) with rows past kd
    int *const s_info = reinterpret_cast<int *>(tiles + W * (W + 1) / 2 * kTile);
    int *const s_neg = s_info + 1;  // the last tile row that entered with a -0.0
    int *const s_odd = s_info + 2;  // the last panel with an infinity or NaN in L
    // helpers: waves 1, 2, 3, 5, 6, 7
    const int hw = wv == 0 || wv == 4 ? -1 : (wv < 4 ? wv - 1 : wv - 2);
    const int ht = hw * 64 + lane;

    int *const s_pairs = s_info + 4;

    // tile (a, b) of the window whose first tile row is at ring position pm
    auto tile = [&](int pm, int a, int b) __attribute__((always_inline)) -> double * {
        int r = pm + a, c = pm + b;
        r = r >= W ? r - W : r;
        c = c >= W ? c - W : c;
        const int hi = max(r, c), lo = min(r, c);
        return tiles + (hi * (hi + 1) / 2 + lo) * kTile;
    };
    // C(i, c) -= L(i, k) L(c, k), k = 0..15, for H tiles (a, b), (a + 1, b).
    // `Op` holds the operands of one such update, so that the next one's are
    // read while this one's matrix instructions run.
    struct Op {
        double *C[2];
        v4d acc[2];
        double x[4], y[2][4];
    };
    auto read = [&]<int H>(Op &o, int pm, int a, int b) __attribute__((always_inline)) {
        const double *LJ = tile(pm, b, 0) + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) o.x[q] = LJ[64 * q];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            // (past the last tile row: a slot that no tile of the window uses)
            o.C[h] = (h == 0 || a + 1 < T ? tile(pm, a + h, b) : tile(pm, T + 1, 0)) + lane;
            const double *LI = tile(pm, a + h, 0) + lane;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                o.acc[h][q] = o.C[h][64 * q];
                o.y[h][q] = LI[64 * q];
            }
        }
    };
    auto apply = [&]<int H>(Op &o) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < H; ++h)
                o.acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(-o.x[q], o.y[h][q], o.acc[h], 0, 0, 0);
#pragma unroll
        for (int h = 0; h < H; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) o.C[h][64 * q] = o.acc[h][q];
    };
    // the same for one tile step by step, with the band's edge
    auto apply_edge = [&](int pm, int a, int b) __attribute__((always_inline)) {
        double *C = tile(pm, a, b);
        const double *LI = tile(pm, a, 0), *LJ = tile(pm, b, 0);
        const int i = lane & 15, lk = lane >> 4, ri = kB * a + i;
#pragma unroll 1
        for (int q = 0; q < 4; ++q) {
            double v = C[64 * q + lane];
#pragma unroll 1
            for (int k = 0; k < kB; ++k)
                if (ri - k <= kd) v = __builtin_fma(-LI[k * kB + i], LJ[k * kB + 4 * q + lk], v);
            C[64 * q + lane] = v;
        }
    };

    // wave 0: factor panel p (tile column 0 of the window at ring position pm)
    auto factor = [&](int p, int pm) __attribute__((always_inline)) {
        const int nb = min(kB, n - kB * p);
        int ln = lane;
        asm volatile("" : "+v"(ln));  // (its compares are not kept across panels)
        double *base[RPL];
        double x[RPL][kB];
#pragma unroll
        for (int q = 0; q < RPL; ++q) {
            const int ri = 64 * q + lane;
            base[q] = tile(pm, min(ri >> 4, T - 1), 0) + (ri & 15);
        }
        auto load = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < RPL; ++q)
#pragma unroll
                for (int s = 0; s < kB; ++s) x[q][s] = base[q][s * kB];
        };
        load();
        // (rows past kd are as they entered: a -0.0 there would not survive a
        // structurally zero multiplier)
        const bool plain = __builtin_amdgcn_readfirstlane(*s_neg) < p + edge;
        unsigned worst = 0;
        double g, r;  // the step's diagonal entry of L and its reciprocal (lane s)
        sqrt_recip(x[0][0], g, r);
#pragma unroll
        for (int s = 0; s < kB; ++s) {
            // (a scheduling region per step: the next column's update, then its
            // root while the other columns take the step)
            const double rs = readlane_d(r, s);
            const double gs = g;
            // the pivot was positive and in [2^-600, 2^600]: 1/root in [2^-300, 2^300]
            worst = max(worst, unsigned(__double_as_longlong(rs) >> 32) - (723u << 20));
            asm volatile("" : "+v"(worst));
            double l[RPL];
#pragma unroll
            for (int q = 0; q < RPL; ++q) l[q] = x[q][s] * rs;
#pragma unroll
            for (int c = s + 1; c < kB; ++c) {
                const double lc = readlane_d(l[0], c);
#pragma unroll
                for (int q = 0; q < RPL; ++q) x[q][c] = pin(__builtin_fma(-l[q], lc, x[q][c]));
                if (c == s + 1) sqrt_recip(x[0][c], g, r);
            }
            x[0][s] = ln == s ? gs : l[0];
#pragma unroll
            for (int q = 1; q < RPL; ++q) x[q][s] = l[q];
            __builtin_amdgcn_sched_barrier(0);
        }
        // an infinity or NaN in the panel's top block (0 times it is NaN)
        double inf = 0.0;
#pragma unroll
        for (int s = 0; s < kB; ++s) inf = __builtin_fma(x[0][s], 0.0, inf);
        if (!plain || __any(worst >= (600u << 20) || (ln < kB && inf != 0.0))) {
            // ---- step by step: the band's edge by exec mask, a stop at the
            // first pivot that is not positive
            load();
            int lim = nb;
#pragma unroll
            for (int s = 0; s < kB; ++s) {
                if (s >= lim) continue;
                const double d = readlane_d(x[0][s], s);
                if (!(d > 0.0)) {
                    lim = s;
                    continue;
                }
                const double g = __builtin_sqrt(d), r = 1.0 / g;
                double l[RPL];
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                    l[q] = x[q][s] * r;
                    if (64 * q + lane - s <= kd) x[q][s] = q == 0 && lane == s ? g : l[q];
                }
#pragma unroll
                for (int c = s + 1; c < kB; ++c) {
                    const double lc = readlane_d(l[0], c);
#pragma unroll
                    for (int q = 0; q < RPL; ++q)
                        if (64 * q + lane - s <= kd) x[q][c] = __builtin_fma(-l[q], lc, x[q][c]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (lim < nb) {
                // the columns from the failing one on keep their updated
                // values; for the tiles the panel ends here
                if (lane == 0) *s_info = kB * p + lim + 1;
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                    const int ri = 64 * q + lane;
#pragma unroll
                    for (int s = 0; s < kB; ++s)
                        if (s >= lim && s < nb) {
                            if (ri >= s && ri - s <= kd && kB * p + ri < n)
                                AB[(ri - s) + int64_t(kB * p + s) * ldab] = x[q][s];
                        }
                }
            }
#pragma unroll
            for (int q = 0; q < RPL; ++q)
#pragma unroll
                for (int s = 0; s < kB; ++s)
                    if (s >= lim) x[q][s] = 0.0;
        }
#pragma unroll
        for (int q = 0; q < RPL; ++q)
            if (64 * q + lane < kB * T) {
#pragma unroll
                for (int s = 0; s < kB; ++s) base[q][s * kB] = x[q][s];
            }
    };

    if (tid == 0) {
        *s_info = 0;
        *s_neg = -1;
        *s_odd = -1;
    }
    __syncthreads();
    // tile rows 0..T-1
    for (int e = tid; e < T * T * kTile; e += kThreads) {
        const int a = e / (T * kTile), b = e / kTile % T, k = e % kTile;
        const int c = kB * b + k / kB, i = kB * a + k % kB;
        const bool ok = i < n && c <= i && i - c <= kd;
        const double v = AB[ok ? (i - c) + int64_t(c) * ldab : 0];
        if (b <= a) tile(0, a, b)[k] = ok ? v : (i == c && i >= n ? 1.0 : 0.0);
        if (ok && is_neg_zero(v)) atomicMax(s_neg, a);
    }
    // phase 2's pairs of tiles
    for (int e = tid; e < T * T; e += kThreads) {
        const int b = e / T, a = b + 2 * (e % T);
        if (b >= 2 && a < T) {
            int at = (a - b) / 2;
            for (int c = 2; c < b; ++c) at += (T - c + 1) / 2;
            s_pairs[at] = a | b << 8;
        }
    }
    __syncthreads();
    // (each kind of wave has a loop of its own, so that none carries another's
    // registers; all of them meet at the same barriers)
    int pm = 0, info = 0, p = -1;
    auto phase1 = [&]() __attribute__((always_inline)) {
        // (wave 0 last: it is the last to arrive)
        const int first = (wv + 7) & 7;
        const bool neg = __builtin_amdgcn_readfirstlane(*s_neg) >= p + edge;
#pragma unroll 1
        for (int a = 1 + first; a < T; a += kThreads / 64) {
            Op o;
            read.template operator()<1>(o, pm, a, 1);
            // an infinity or NaN in tile rows a and 1 of the panel
            bool odd = false;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                odd |= !__builtin_isfinite(o.x[q]) || !__builtin_isfinite(o.y[0][q]);
            const bool any = __any(odd);
            if (any && lane == 0) *s_odd = p;
            if (a >= edge && (any || neg))
                apply_edge(pm, a, 1);
            else
                apply.template operator()<1>(o);
        }
    };
    if (wv == 0) {
#pragma unroll 1
        for (;;) {
            const int pn = p < 0 ? 0 : (pm + 1 >= W ? 0 : pm + 1);
            if (p >= 0) phase1();
            __syncthreads();
            if (!info && p + 1 < np) factor(p + 1, pn);
            __syncthreads();
            if (info || p + 1 >= np) break;
            ++p;
            pm = pn;
            info = __builtin_amdgcn_readfirstlane(*s_info);
        }
    } else if (hw < 0) {
#pragma unroll 1
        for (;;) {
            const int pn = p < 0 ? 0 : (pm + 1 >= W ? 0 : pm + 1);
            if (p >= 0) phase1();
            __syncthreads();
            __syncthreads();
            if (info || p + 1 >= np) break;
            ++p;
            pm = pn;
            info = __builtin_amdgcn_readfirstlane(*s_info);
        }
    } else {
        // the tile row that enters in phase 2 of panel p, p+1+T: helper thread
        // ht < 256 holds entry ht of its tiles, loaded a panel ahead
        double ent[T];
        const bool loader = hw < 4;
        const int ei = ht % kB, ec = ht / kB;
        auto entering = [&](int p, int u) __attribute__((always_inline)) -> bool {
            const int c = kB * (p + 2 + u) + ec, i = kB * (p + 1 + T) + ei;
            return i < n && c <= i && i - c <= kd;
        };
        auto fetch = [&](int p) __attribute__((always_inline)) {
            const int64_t off = (kB * (p + 1 + T) + ei) + int64_t(kB * (p + 2) + ec) * (ldab - 1);
#pragma unroll
            for (int u = 0; u < T; ++u)
                ent[u] = AB[entering(p, u) ? off + u * kB * (ldab - 1) : 0];
        };
        if (loader) fetch(-1);
#pragma unroll 1
        for (;;) {
            const int pn = p < 0 ? 0 : (pm + 1 >= W ? 0 : pm + 1);
            if (p >= 0) {
                phase1();
            }
            __syncthreads();
            if (loader) {
                bool neg = false;
#pragma unroll
                for (int u = 0; u < T; ++u) {
                    const bool ok = entering(p, u);
                    const bool past = u == T - 1 && ei == ec && kB * (p + 1 + T) + ei >= n;
                    neg |= ok && is_neg_zero(ent[u]);
                    tile(pn, T, 1 + u)[ht] = ok ? ent[u] : (past ? 1.0 : 0.0);
                }
                if (neg) atomicMax(s_neg, p + 1 + T);
                fetch(p + 1);
            }
            if (p >= 0) {
                // tiles (a, b), 2 <= b <= a < T, two of a column at a time, the
                // pairs dealt out in turn
                const bool odd = __builtin_amdgcn_readfirstlane(*s_neg) >= p + edge ||
                                 __builtin_amdgcn_readfirstlane(*s_odd) == p;
                // (dealt out in turn, first to the helpers that bring nothing in)
                auto pair = [&](int t) __attribute__((always_inline)) -> int {
                    return __builtin_amdgcn_readfirstlane(s_pairs[min(t, kPairs - 1)]);
                };
                constexpr int kStep = kHelpers / 64;
                // (with few pairs the order does not matter, and this one lets two
                // workgroups share a CU: 106 registers against 158)
                const int t0 = T > 4 ? kStep - 1 - hw : hw;
                if (odd) {
#pragma unroll 1
                    for (int t = t0; t < kPairs; t += kStep) {
                        const int ab = pair(t), a = ab & 255, b = ab >> 8;
#pragma unroll 1
                        for (int h = a; h < min(a + 2, T); ++h) {
                            if (h >= edge) {
                                apply_edge(pm, h, b);
                            } else {
                                Op o;
                                read.template operator()<1>(o, pm, h, b);
                                apply.template operator()<1>(o);
                            }
                        }
                    }
                } else if (t0 < kPairs) {
                    Op o[2];
                    int ab = pair(t0), an = pair(t0 + kStep);
                    read.template operator()<2>(o[0], pm, ab & 255, ab >> 8);
#pragma unroll 1
                    for (int t = t0;; t += 2 * kStep) {
                        if (t + kStep < kPairs) {
                            ab = an;
                            an = pair(t + 2 * kStep);
                            read.template operator()<2>(o[1], pm, ab & 255, ab >> 8);
                        }
                        apply.template operator()<2>(o[0]);
                        if (t + kStep >= kPairs) break;
                        if (t + 2 * kStep < kPairs) {
                            ab = an;
                            an = pair(t + 3 * kStep);
                            read.template operator()<2>(o[0], pm, ab & 255, ab >> 8);
                        }
                        apply.template operator()<2>(o[1]);
                        if (t + 2 * kStep >= kPairs) break;
                    }
                }
                // the panel's columns (those before a failing one): half the
                // helpers take the even columns, the others the odd ones
                const int cols = info ? info - 1 - kB * p : min(kB, n - kB * p);
                const int t = ht % (kHelpers / 2), c0 = ht / (kHelpers / 2);
                if (t <= kd) {
                    const double *b0 = tile(pm, 0, 0), *b1 = b0;
                    {
                        // (tile() of a row that differs by lane)
                        int r0 = pm + (t >> 4), r1 = pm + min((t >> 4) + 1, T);
                        r0 = r0 >= W ? r0 - W : r0;
                        r1 = r1 >= W ? r1 - W : r1;
                        const int h0 = max(r0, pm), l0 = min(r0, pm);
                        const int h1 = max(r1, pm), l1 = min(r1, pm);
                        b0 = tiles + (h0 * (h0 + 1) / 2 + l0) * kTile + (t & 15);
                        b1 = tiles + (h1 * (h1 + 1) / 2 + l1) * kTile + (t & 15) - kB;
                    }
                    double *col = AB + t + int64_t(kB * p + c0) * ldab;
                    double v[kB / 2];
#pragma unroll
                    for (int u = 0; u < kB / 2; ++u) {
                        const int c = 2 * u + c0;
                        v[u] = ((t & 15) + c < kB ? b0 : b1)[c * (kB + 1)];
                    }
#pragma unroll
                    for (int u = 0; u < kB / 2; ++u) {
                        const int c = 2 * u + c0;
                        if (c < cols && kB * p + c + t < n) col[2 * u * ldab] = v[u];
                    }
                }
            }
            __syncthreads();
            if (info || p + 1 >= np) break;
            ++p;
            pm = pn;
            info = __builtin_amdgcn_readfirstlane(*s_info);
        }
    }
    if (info) {
        // not positive definite: the columns after the panel keep what the
        // steps before the failing one left in them
        for (int e = tid; e < T * T * kTile; e += kThreads) {
            const int a = e / (T * kTile), b = e / kTile % T;
            const int c = kB * (p + b) + e % kTile / kB, i = kB * (p + a) + e % kB;
            if (b >= 1 && b <= a && i < n && c <= i && i - c <= kd)
                AB[(i - c) + int64_t(c) * ldab] = tile(pm, a, b)[e % kTile];
        }
    }
    if (tid == 0) P.info[blockIdx.x] = info;
}

template <int T>
int launch(const CholParams &P, int64_t batch, hipStream_t s) {
    constexpr int W = T + 2;
    // the tiles, three counters and the list of pairs
    constexpr int shm = W * (W + 1) / 2 * kTile * 8 + 16 + T * T * 4;
    static_assert(shm <= 160 * 1024, "LDS of a CU");
    if (shm > 64 * 1024) {
        if (hipError_t e = hipFuncSetAttribute((const void *)pbtrf_tile_kernel<T>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, shm);
            e != hipSuccess)
            return hip_fail(e, "band_pbtrf (LDS window size)");
    }
    hipLaunchKernelGGL(pbtrf_tile_kernel<T>, dim3((unsigned)batch), dim3(kThreads), shm, s, P);
    BANDLU_CHECK_LAUNCH("band_pbtrf");
    return BANDLU_OK;
}

}  // namespace

int launch_pbtrf_tile(const CholParams &P, int64_t batch, hipStream_t s) {
    switch ((P.kd + kB - 1) / kB) {
        case 0:
        case 1: return launch<2>(P, batch, s);
        case 2: return launch<3>(P, batch, s);
        case 3: return launch<4>(P, batch, s);
        case 4: return launch<5>(P, batch, s);
        case 5: return launch<6>(P, batch, s);
        case 6: return launch<7>(P, batch, s);
        case 7: return launch<8>(P, batch, s);
        case 8: return launch<9>(P, batch, s);
        default: return launch<10>(P, batch, s);
    }
}

}  // namespace bandlu
