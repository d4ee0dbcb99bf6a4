// Banded LU with partial pivoting (xGBTRF semantics, m x n) for 1 <= kl <= 31
// and 2kl+ku+1 <= 448, one matrix per workgroup of one pivot wavefront and one
// update wavefront per 64 columns of the window: the single-matrix kernel of
// Sec. III-A's specialised algorithm f(N).
//
// The column steps form one chain of dependent pivot decisions.  A single
// wavefront that also carries the rank-1 updates, the row stores and the
// refills issues a few hundred instructions per step, and one wavefront issues
// at most one instruction every four cycles.  Here the work of a step is split
// between wavefronts that run on different SIMDs:
//   wave P (pivots) holds the pivot column transposed, one row per lane.  At
//     step j it takes column j (rows j-1..j-1+kl, up to date through step j-2)
//     from wave U, applies step j-1 to it (interchange, one fused multiply-add
//     per row) and adds the row that enters, finds the pivot (first largest
//     |a|; a NaN counts only in first position), forms the multipliers in the
//     lanes of their rows, stores ipiv[j], and hands the pivot offset and the
//     multipliers to the waves U;
//   waves U (updates) run one step behind with the band window in registers:
//     column c in lane (c mod M) mod 64 of wave (c mod M) / 64 (M = 64 NU for
//     NU waves, M >= 2kl+ku+1; one wave may hold M = 128, two columns per
//     lane), row r in slot r mod H (H = kl + 1).  At its step
//     j a wave applies the interchange and the rank-1 update of step j-1 to its
//     columns, stores row j-1 of U, refills the freed slot with the row that
//     enters, and the wave that holds them stores the multipliers of column
//     j-1 and hands column j+1 (rows j..j+kl, up to date through step j-1) to
//     wave P.  A column is written by the wave that holds it alone, after that
//     wave's loads of it: wave P reads original entries only, and each of them
//     before the waves U reach the column that holds it.
// The two hand-overs are double buffered in LDS and one workgroup barrier per
// step separates them.  Every entry sees the same operations in the same order
// as in the unblocked algorithm, so the factors are bitwise those of the
// reference loops.
//
// A step is bound by wave P's chain (argmax, reciprocal, hand-over) and, from
// kl = 16 or so on, by a wave U's: the multipliers read from LDS, the selects of
// the interchange and one fused multiply-add per row.  More columns take more
// waves and little more time.  Measured (ns per column, random entries; before:
// the kernel that each of them replaced): n = 4096, kl = ku = 31: 5430 -> 1029
// (one launch per panel of 32 columns); kl = 20, ku = 200: 5600 -> 943;
// kl = 31, ku = 385: 5600 -> 1328; 8192, kl = 12, ku = 90: 864 -> 651 (both
// blocks of 64 columns in one wave); kl = ku = 16: 727 -> 672; 9216 x 8192 with
// kl = ku = 16: 3207 -> 663 (the window in global memory).
#pragma once

#include <cfloat>
#include <utility>

#include "bufio.hpp"
#include "common.hpp"
#include "getrf_window.hpp"
#include "wave.hpp"

namespace bandlu {

// 64-bit lane masks on the scalar unit: `len` lanes from lane `start` on,
// wrapping around (0 <= len <= 63)
__device__ __forceinline__ unsigned long long split_lanes(int start, int len) {
    const unsigned long long ones = (1ull << len) - 1;
    const int s = start & 63;
    return (ones << s) | ((ones >> 1) >> (63 - s));
}

// rotate right by r (0 <= r <= 63)
__device__ __forceinline__ unsigned long long split_rotr(unsigned long long m, int r) {
    return (m >> r) | ((m << 1) << (63 - r));
}

// prefetch depth of a wave U: a multiple of H (so that every register slot
// index is a compile-time constant), at least 16, and even for H <= 16 (so that
// the parity of the LDS buffers is one too; beyond that the registers of twice
// the depth are worth more)
constexpr int split_pf(int H) {
    int m = (16 + H - 1) / H;
    if (H <= 16 && ((m * H) & 1)) ++m;
    return m * H;
}

// Interchange of slots S0 and (S0 + p) % H, 1 <= p < H uniform: a uniform
// branch to the group of eight offsets that holds p, selects within it (all
// offsets as selects cost four instructions each, more than the update).
template <int H, int S0>
__device__ __forceinline__ void split_swap(double (&a)[H], int p) {
    auto group = [&]<int K0>() __attribute__((always_inline)) {
        double a0 = a[S0];
#pragma unroll
        for (int k = K0; k < K0 + 8 && k < H; ++k) {
            const bool hit = p == k;
            const double ak = a[(S0 + k) % H];
            a0 = hit ? ak : a0;
            a[(S0 + k) % H] = hit ? a[S0] : ak;
        }
        a[S0] = a0;
        asm volatile("" ::: "memory");  // (stays a branch)
    };
    if (H <= 9 || p < 9) group.template operator()<1>();
    else if (H <= 17 || p < 17) group.template operator()<9>();
    else if (H <= 25 || p < 25) group.template operator()<17>();
    else group.template operator()<25>();
}

// CPL: columns per lane; NU: waves U (0: as many as the launch has).  One wave U
// has kernels of its own from kl = 7 on: with M known, single matrices of kl = 9..31 took 2-12 %
// less (kl = 16, n = 5000: 3525 -> 3305 us random, 2930 -> 2645 dominant).
// CPL = 2 (one wave U for 65..128 columns) runs batches whose matrices all fit
// the chip at once: see split_two_columns() in getrf.hip.
template <int H, int CPL, int NU>
__global__ __launch_bounds__(CPL == 1 ? 64 * (1 + kSplitMaxU) : 128) void getrf_split_kernel(WinParams P) {
    constexpr int PF = split_pf(H);
    static_assert(H >= 2 && H <= 32, "window of 2..32 rows");
    static_assert(PF % H == 0 && PF + 1 <= 64, "prefetch depth: a multiple of H below 64");
    static_assert(CPL == 1 || NU == 1, "several columns per lane in one wave U");
    constexpr int kl = H - 1;
    const int tid = threadIdx.x;
    const int L = tid & 63;
    const int64_t b = blockIdx.x;  // one matrix per workgroup
    const int ku = P.ku, kv = kl + P.ku, ldab = int(P.ldab);
    const int M = NU ? 64 * CPL * NU : int(blockDim.x) - 64;  // columns that the waves U hold
    int n = P.n, m = P.m;
    double *ABb = P.AB + b * P.strideAB;
    int32_t *ipb = P.ipiv + b * P.strideP;
    int j0 = 0;
    if (P.resume) {
        // after the diagonal-pivot kernel (getrf_diag.hpp): ipiv[n-1] > 0 says
        // it factored the whole band, -(j0+1) that column j0 failed its check.
        // Steps 0..j0-1 interchanged nothing, so the trailing band from column
        // j0 on is a band problem of its own with the same kl and ku.
        const int mark = ipb[n - 1];
        if (mark > 0) return;
        j0 = -mark - 1;
        n -= j0;
        m -= j0;
        ABb += int64_t(j0) * ldab;
        ipb += j0;
    }
    const int steps = min(m, n);
    const Buf ab = make_buf(ABb, uint32_t(int64_t(ldab) * n * 8));
    __shared__ double s_l[2][32];    // multipliers of a step by row offset 1..kl
    __shared__ int s_pv[2][2];       // pivot offset and nonzero-pivot flag of a step
    __shared__ double s_col[2][64];  // a column for wave P, rows by offset from its first

    // original band entry (r, c), else an offset outside the buffer (reads 0)
    auto foff = [&](int r, int c) -> uint32_t {
        const bool ok = c >= 0 && c < n && r >= 0 && r < m && unsigned(r - c + ku) <= unsigned(kl + ku);
        return ok ? uint32_t(c * ldab + kv + r - c) * 8u : kOutside;
    };

    if (tid >= 64) {
        // ----------------------------------------------------------- waves U --
        // first column of this wave
        const int w0 = NU == 1 ? 0 : (__builtin_amdgcn_readfirstlane(tid) >> 6) * 64 - 64;
        // column that this lane holds in sub-slot s at step x: the first c >= x
        // with c mod M = w0 + 64 s + L; xm = x mod M
        auto colof = [&](int s, int x, int xm) -> int {
            if (NU == 1) return x + ((L + 64 * s - x) & (64 * CPL - 1));
            const int d = w0 + L - xm;
            return x + (d < 0 ? d + M : d);
        };
        double a[CPL][H];
        double pf[CPL][PF];
#pragma unroll
        for (int s = 0; s < CPL; ++s) {
#pragma unroll
            for (int r = 0; r < H; ++r)
                a[s][r] = buf_ld(ab, foff(r, r < H - 1 ? colof(s, r - H + 1, M + r - H + 1) : colof(s, 0, 0)));
#pragma unroll
            for (int k = 0; k < PF; ++k) pf[s][k] = buf_ld(ab, foff(k + H, colof(s, k + 1, k + 1)));
        }
        int ju = 0;
        // column 1, rows 0..kl (no step applied yet) for wave P's step 1: it
        // sits in lane 1 of the first wave, slots 0..kl
        if (tid == 64 + 1) {
#pragma unroll
            for (int t = 0; t < H; ++t) s_col[0][t] = a[0][t];
        }
        lds_barrier();
        // (with one wave U they stay in vector registers: one instruction less)
        auto uni = [](int v) __attribute__((always_inline)) -> int {
            return NU == 1 ? v : __builtin_amdgcn_readfirstlane(v);
        };
        bool live = true;
        int odd = 0;  // parity of the block's first step (0 where PF is even)
        int jm = 0;   // jj mod M (several waves U)
        auto ustep = [&]<int U>(int jj) __attribute__((always_inline)) {
            constexpr int S0 = U % H;
            if (!live) return;
            if (jj >= steps) {
                live = false;
                return;
            }
            const int par = PF & 1 ? (U & 1) ^ odd : U & 1;  // jj & 1
            // ---- step jj as decided by wave P
            const int pv = uni(s_pv[par][0]);
            const int nz = uni(s_pv[par][1]);
            int c[CPL];
#pragma unroll
            for (int s = 0; s < CPL; ++s) c[s] = colof(s, jj, jm);
            if (nz) {
                ju = max(ju, min(jj + ku + pv, n - 1));
                if (pv != 0) {
                    // interchange rows jj and jj+pv in columns jj..ju
#pragma unroll
                    for (int s = 0; s < CPL; ++s)
                        if (c[s] <= ju) {
                            if constexpr (CPL == 2 || (NU == 1 && H <= 9)) win_swap<H, S0>(a[s], pv);
                            else split_swap<H, S0>(a[s], pv);
                        }
                }
                double lm[H];
#pragma unroll
                for (int t = 1; t < H; ++t) lm[t] = s_l[par][t];
                // rank-1 update of columns jj+1..ju, under an exec mask (the empty
                // volatile asm keeps the block a branch: as selects it would cost
                // two more instructions per entry)
#pragma unroll
                for (int s = 0; s < CPL; ++s) {
                    if (c[s] > jj && c[s] <= ju) {
                        const double uu = a[s][S0];
#pragma unroll
                        for (int t = 1; t < H; ++t)
                            a[s][(S0 + t) % H] = __builtin_fma(-lm[t], uu, a[s][(S0 + t) % H]);
                        asm volatile("" ::: "memory");
                    }
                }
            }
            // ---- multipliers of column jj (as wave P formed them; for a zero pivot
            // the column as it is) into the band, by the wave that holds the
            // column: no store can overtake a load of an original entry of it
            if (NU == 1 || unsigned(jm - w0) < 64u) {
                const int kmj = min(kl, m - 1 - jj);
                const double lv = s_l[par][L & 31];
                buf_st(ab, (L >= 1 && L <= kmj) ? uint32_t(jj * ldab + kv + L) * 8u : kOutside, lv);
            }
            // ---- row jj of U leaves the window (columns jj..jj+kv; a retired
            // column has c >= jj+M-H+1 > jj+kv), row jj+H enters
#pragma unroll
            for (int s = 0; s < CPL; ++s) {
                const bool ok = c[s] < n && c[s] <= jj + kv;
                buf_st(ab, ok ? uint32_t(c[s] * ldab + kv + jj - c[s]) * 8u : kOutside, a[s][S0]);
                a[s][S0] = pf[s][U];
                pf[s][U] = buf_ld(ab, foff(jj + PF + H, c[s] > jj + PF ? c[s] : c[s] + M));
            }
            // ---- column jj+2, rows jj+1..jj+1+kl (through step jj), for wave P
            if (NU != 1) jm = jm + 1 == M ? 0 : jm + 1;
            if (jj + 2 < steps) {
                const int wc = NU == 1 ? (jj + 2) & (M - 1) : (jm + 1 == M ? 0 : jm + 1) - w0;
                if (L == (CPL == 1 ? wc : wc & 63)) {
                    if (CPL == 1 || wc < 64) {
#pragma unroll
                        for (int t = 0; t < H; ++t) s_col[par ^ 1][t] = a[0][(S0 + 1 + t) % H];
                    } else {
#pragma unroll
                        for (int t = 0; t < H; ++t) s_col[par ^ 1][t] = a[CPL - 1][(S0 + 1 + t) % H];
                    }
                }
            }
            if (jj + 1 < steps) lds_barrier();
        };
        for (int jj0 = 0; live; jj0 += PF) {
            [&]<int... Us>(std::integer_sequence<int, Us...>) {
                (ustep.template operator()<Us>(jj0 + Us), ...);
            }(std::make_integer_sequence<int, PF>{});
            odd ^= PF & 1;
        }
        return;
    }

    // -------------------------------------------------------------- wave P --
    const Buf pb = make_buf(ipb, uint32_t(int64_t(steps) * 4));
    // entering entries a(c+kl, c) of the 64 columns of this and the next block
    double E = buf_ld(ab, foff(L + kl, L));
    double En = buf_ld(ab, foff(64 + L + kl, 64 + L));
    // column 0, rows 0..kl
    double y = buf_ld(ab, L <= kl ? foff(L, 0) : kOutside);
    double lprev = 0.0;
    int pprev = 0, nzprev = 0, juprev = 0;
    int ju = 0, info = 0;
    for (int j = 0; j < steps; ++j) {
        const int u = j & 63;
        if (j > 0) {
            // column j, rows j-1..j-1+kl through step j-2, from wave U
            const int q = (j - 1) & 63;  // lane of row j-1
            double v = s_col[(j - 1) & 1][(L - q) & 63];
            if (nzprev && j <= juprev) {
                // step j-1 on column j: interchange, then one fma per row below
                if (pprev != 0) {
                    const int qp = (q + pprev) & 63;
                    const double vq = readlane_d(v, q), vp = readlane_d(v, qp);
                    v = L == q ? vp : (L == qp ? vq : v);
                }
                const double u0 = readlane_d(v, q);
                const int kmp = min(kl, m - j);
                if (__builtin_amdgcn_inverse_ballot_w64(split_lanes(q + 1, kmp)))
                    v = __builtin_fma(-lprev, u0, v);
            }
            // row j+kl enters the window (no step has touched it yet)
            const double e = readlane_d(E, u);
            y = L == ((j + kl) & 63) ? e : v;
        }
        // ---- pivot: first largest |y| over rows j..j+km.  The maximum is taken
        // over the high 32 bits of |y|; a NaN on the diagonal ranks above
        // everything and one below it with the zeros, so an earlier row wins
        // against it; only rows that tie on the high word compare low words.
        const int km = min(kl, m - 1 - j);
        const unsigned long long cand = split_lanes(u, km + 1);
        const double rall = 1.0 / y;
        const bool nan = __builtin_isnan(y);
        const bool inc = __builtin_amdgcn_inverse_ballot_w64(cand);
        const int toff = (L - u) & 63;
        const unsigned yhi = unsigned(__double_as_longlong(y) >> 32) & 0x7fffffffu;
        const unsigned khi = !inc ? 0u : (nan ? (toff == 0 ? 0x7ff00001u : 0u) : yhi);
        unsigned long long hit = __ballot(khi == wave_max_u32(khi)) & cand;
        if (__popcll(hit) > 1) {
            const bool tied = (hit >> L) & 1;
            const unsigned klo = (tied && !nan) ? unsigned(__double_as_longlong(y)) : 0u;
            hit &= __ballot(klo == wave_max_u32(klo));
        }
        const int p = __builtin_ctzll(split_rotr(hit, u));
        const int lp = (u + p) & 63;
        const double piv = readlane_d(y, lp);
        const double rcp = readlane_d(rall, lp);  // 1/piv, formed beside the reduction
        buf_st_i32(pb, L == 0 ? uint32_t(j) * 4u : kOutside, j0 + j + p + 1);
        const bool nzj = piv != 0.0;
        // the interchange (none for a zero pivot: then every candidate is zero
        // and p = 0)
        const double y0 = readlane_d(y, u);
        y = L == u ? piv : (L == lp ? y0 : y);
        // multipliers; a zero pivot eliminates nothing and the column below the
        // diagonal stays as it is
        double l = nzj ? y * rcp : y;
        if (nzj && !(fabs(piv) >= DBL_MIN)) l = y / piv;
        if (nzj) ju = max(ju, min(j + ku + p, n - 1));
        if (!nzj && info == 0) info = j + 1;
        // ---- hand-over to wave U (which also stores the multipliers)
        const bool mrow = __builtin_amdgcn_inverse_ballot_w64(split_lanes(u + 1, km));
        if (mrow) s_l[j & 1][toff] = l;
        if (L == 0) {
            s_pv[j & 1][0] = p;
            s_pv[j & 1][1] = nzj ? 1 : 0;
        }
        lprev = l;
        pprev = p;
        nzprev = nzj ? 1 : 0;
        juprev = ju;
        lds_barrier();
        if (u == 63) {
            E = En;
            En = buf_ld(ab, foff(j + 65 + L + kl, j + 65 + L));
        }
    }
    if (L == 0) {
        if (!P.resume) P.info[b] = info;
        else if (info != 0 && P.info[b] == 0) P.info[b] = j0 + info;
    }
}

// the kernels for H = LO..HI
template <int LO, int HI, int CPL, int NU>
struct SplitRange {
    template <int... Is>
    static constexpr auto make(std::integer_sequence<int, Is...>) {
        return std::array<WinKernel, HI - LO + 1>{{&getrf_split_kernel<LO + Is, CPL, NU>...}};
    }
};

// any number of waves U; one wave U; one wave U with two columns per lane
WinKernel split_kernel_h2_16(int H);
WinKernel split_kernel_h17_24(int H);
WinKernel split_kernel_h25_32(int H);
WinKernel split_one_h8_16(int H);
WinKernel split_one_h17_24(int H);
WinKernel split_one_h25_32(int H);
WinKernel split_two_h8_16(int H);

}  // namespace bandlu
