// L^T pass of the transposed solve A^T x = b with the band LU factors (the
// general "A \ B" of Listing 1 on A^T; xGBTRS with trans = 'T'):
//   for j = n-2 .. 0:  b_j = fma(-l_t, b_{j+t}, b_j), t = 1..min(kl, n-1-j)
//                      ascending; then the interchange of row j.
// The first term of row j needs the value that row j+1 has just produced, so
// the n*kl fused multiply-adds are one serial chain.  What bounds it is the
// latency of a term: v_mfma_f64_4x4x4f64 sums four terms, in ascending order
// and with one rounding each, in 20 cycles, where a chain of v_fma_f64 whose
// operands come from LDS by broadcast loads (16 bytes for all 64 lanes a term)
// ran at 27 cycles a term.  One 8-byte LDS load feeds an operand of four terms.
//
// One workgroup per right-hand side.  Wave 0 runs the chain: lanes 0, 16, 32
// and 48 hold the four multipliers (operand A) and the four vector entries
// (operand B) of a group; the sum stays in lane 0 of the accumulator, which is
// also the lane of the next row's first operand, so the newest value is never
// waited for in LDS.  Waves 1..3 bring the multipliers of the next NB rows to
// one half of a double buffer (negated, and -0.0 beyond the row's last one)
// while wave 0 works on the other half.  The vector's window is an LDS ring
// that holds every position twice (q mod R and R + q mod R), so that the kl
// positions a row reads are consecutive.
//
// Measured, n = 32768, kl = ku = 256, one right-hand side: 88.5 ms with the
// broadcast loads, 28.9 ms with this kernel (26 cycles per group of four where
// the bare instruction chain takes 20, and about 400 cycles per row around
// it).  Operands held 16 groups ahead instead of 8 ran at 24 cycles a group
// and lost as much on padded rows.  Small systems are bound by what a workgroup
// sets up: with the window, the halves and the loads cut to their size, 65536
// systems (both passes) take 363 us for 390 at n = 8, kl = 1, and 1281 for 1363 at
// n = 64, where the broadcast loads took 356 and 1304.
#include <algorithm>

#include "getrs_lt.hpp"
#include "bufio.hpp"

namespace bandlu {
namespace {

constexpr int kLtThreads = 256;
constexpr int kLtLoaders = kLtThreads - 64;
constexpr int kGroups = 8;              // groups of four terms to a block
constexpr int kBlk = 4 * kGroups;       // terms to a block
// multipliers in one half-buffer: 16 KiB, so that the whole workgroup stays
// below 64 KiB of LDS (a half lasts wave 0 at least 5000 cycles, two trips to HBM)
constexpr int kHalfMax = 2048;
// multipliers that a loader brings to a half: all of the largest half, or those
// of the smaller halves that many systems and few rows take
constexpr int kPerLoader = (kHalfMax + kLtLoaders - 1) / kLtLoaders;
constexpr int kPerLoaderSmall = 3;

// TG: groups of a row's last block; MULTI: rows of more than one block; PL:
// multipliers per loader.
// kps: log2 of the multipliers kept per row; nbs: log2 of the rows per half
template <int TG, bool MULTI, int PL>
__global__ __launch_bounds__(kLtThreads, 2) void lt_mfma_kernel(LtParams P, int kps, int nbs) {
    extern __shared__ double lds_lt[];
    const int tid = threadIdx.x;
    const int64_t sys = blockIdx.x;
    const int64_t b = sys / P.nrhs, k = sys - b * P.nrhs;
    const int n = P.n, kl = P.kl, R = P.R, mask = R - 1;
    const int NB = 1 << nbs, half = NB << kps;
    double *const ring = lds_lt;              // 2R doubles, then 64 that nobody reads
    double *const lbuf = lds_lt + 2 * R + 64; // two halves of NB rows, and room to read one row on
    const int nrow = n - 1;                   // rows n-2 .. 0
    const int nhalf = lt_halves(n, nbs);

    if (tid >= 64) {
        const double *__restrict__ AB = P.AB + b * P.strideAB;
        const int lt = tid - 64;
        auto stage = [&](int h) {
            double *dst = lbuf + (h & 1) * half;
            double v[PL];
#pragma unroll
            for (int i = 0; i < PL; ++i) {
                const int e = lt + kLtLoaders * i;
                const int j = n - 2 - (h << nbs) - (e >> kps);
                const int t = 1 + (e & ((1 << kps) - 1));
                const bool ok = e < half && j >= 0 && t <= min(kl, n - 1 - j);
                v[i] = AB[ok ? P.kv + t + int64_t(j) * P.ldab : 0];
                v[i] = ok ? -v[i] : -0.0;
            }
#pragma unroll
            for (int i = 0; i < PL; ++i) {
                const int e = lt + kLtLoaders * i;
                if (e < half) dst[e] = v[i];
            }
        };
        stage(0);
        for (int h = 0; h < nhalf; ++h) {
            __syncthreads();  // half h staged; the half of h-1 is free
            if (h + 1 < nhalf) stage(h + 1);
        }
        return;
    }

    const int lane = tid, lk = lane >> 4;
    const int32_t *__restrict__ ipiv = P.ipiv + b * P.strideP;
    double *x = P.B + b * P.strideB + k * P.ldb;
    // positions enter the ring in blocks of 64, loaded a block ahead; so does ipiv
    int low = std::max(0, n - 64), pbase = low;
    int hi = n;  // positions >= hi are stored back
    // (positions the ring does not hold yet must be finite: they meet a
    // multiplier of -0.0 near the matrix's end)
    for (int i = lane; i < 2 * R + 64; i += 64) ring[i] = 0.0;
    auto enter = [&](double v) {
        if (low + lane >= 0 && low + lane < n) {
            ring[(low + lane) & mask] = v;
            ring[((low + lane) & mask) + R] = v;
        }
    };
    auto x_at = [&](int base) { return base + lane >= 0 && base + lane < n ? x[base + lane] : 0.0; };
    auto p_at = [&](int base) { return base + lane >= 0 && base + lane < n ? ipiv[base + lane] : 0; };
    enter(x_at(low));
    double xnext = x_at(low - 64);
    int ipv = p_at(low), ipv_next = p_at(low - 64);
    const int nfull = MULTI ? (kl - 1) / kBlk : 0;  // whole blocks before the last
    const int tail = kl - nfull * kBlk;             // terms of the last block, 1..4*TG
    // the operands of the group that is g groups ahead, two by one LDS read
    double a[kGroups], v[kGroups];
    auto pair = [&](double (&d)[kGroups], const double *src, int g) __attribute__((always_inline)) {
        d[g] = src[4 * g];
        d[g + 1] = src[4 * g + 4];
    };
    // lane 0 keeps its value; the other lanes' stores go to the 64 spare words
    double *const spare = ring + 2 * R + lane;
    auto put = [&](int q, double val) __attribute__((always_inline)) {
        double *d = lane == 0 ? ring + (q & mask) : spare;
        double *d2 = lane == 0 ? ring + (q & mask) + R : spare;
        *d = val;
        *d2 = val;
    };
    double prev = ring[(n - 1) & mask];  // position j+1
    double xj = ring[(n - 2) & mask];    // position j
    int j = n - 2, i = 0;
    while (i < nrow) {
        // ---- rows i .. i+seg-1: no staging, no entering positions
        const int c = i & (NB - 1);
        if (j < pbase) {
            pbase -= 64;
            ipv = ipv_next;
            ipv_next = p_at(pbase - 64);
        }
        if (j > 0 && j <= low) {  // (row j reads position j-1 for the next one)
            low -= 64;
            enter(xnext);
            xnext = x_at(low - 64);
        }
        const double *lrow = lbuf + ((i >> nbs) & 1) * half + (c << kps) + lk;
        if (c == 0) {
            __syncthreads();  // the half of these rows is staged
            const double *xw = ring + ((j + 1) & mask) + lk;
#pragma unroll
            for (int g = 0; g < kGroups; g += 2) {
                pair(a, lrow, g);
                pair(v, xw, g);
            }
        }
        int seg = min(min(NB - c, nrow - i), j - pbase + 1);
        if (low > 0) seg = min(seg, j - low);
        i += seg;
        // (where the rows' loop lies in its cache lines is worth up to 4 %: n = 32768,
        // kl = ku = 256, both passes: 42.2 ms on a line, 43.0-43.8 as it fell before)
        asm volatile(".p2align 6");
        for (; seg > 0; --seg, --j) {
            const double xjn = ring[(j - 1) & mask];
            const int p = __builtin_amdgcn_readlane(ipv, j - pbase) - 1;
            double acc = xj;
            v[0] = lane == 0 ? prev : v[0];
            const double *la = lrow, *xv = ring + ((j + 1) & mask) + lk;
            // whole blocks: each operand register takes its value of the next
            // block as soon as its group is done
            for (int bl = 0; bl < nfull; ++bl) {
                la += kBlk;
                xv += kBlk;
#pragma unroll
                for (int g = 0; g < kGroups; g += 2) {
                    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g], v[g], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g + 1], v[g + 1], acc, 0, 0, 0);
                    pair(a, la, g);
                    pair(v, xv, g);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // the last block, and the first operands of row j-1 (position j,
            // its newest, comes from the accumulator)
            lrow += 1 << kps;
            xv = ring + (j & mask) + lk;
            constexpr int kHeld = MULTI ? kGroups : (TG + 1) / 2 * 2;
#pragma unroll
            for (int g = 0; g < kHeld; g += 2) {
                if (g < TG)
                    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g], 4 * g + lk < tail ? v[g] : 0.0,
                                                             acc, 0, 0, 0);
                if (g + 1 < TG)
                    acc = __builtin_amdgcn_mfma_f64_4x4x4f64(
                        a[g + 1], 4 * g + 4 + lk < tail ? v[g + 1] : 0.0, acc, 0, 0, 0);
                pair(a, lrow, g);
                pair(v, xv, g);
                __builtin_amdgcn_sched_barrier(0);
            }
            xj = xjn;
            // the interchange of row j
            if (p > j && p < n) {
                const double vp = ring[p & mask];
                put(p, acc);
                put(j, vp);
                prev = vp;
                // (the operands just read may include position p)
#pragma unroll
                for (int g = 0; g < kHeld; g += 2) pair(v, xv, g);
            } else {
                put(j, acc);
                prev = acc;
            }
        }
        // positions >= (last row) + kl are final
        while (hi - 64 >= j + 1 + kl && hi - 64 >= 0) {
            x[hi - 64 + lane] = ring[(hi - 64 + lane) & mask];
            hi -= 64;
        }
    }
    for (int q = lane; q < hi; q += 64) x[q] = ring[q & mask];
}

template <int TG, bool MULTI>
void lt_launch(const LtParams &P, int64_t systems, size_t shm, int kps, int nbs, hipStream_t s) {
    if ((1 << (nbs + kps)) <= kPerLoaderSmall * kLtLoaders)
        hipLaunchKernelGGL((lt_mfma_kernel<TG, MULTI, kPerLoaderSmall>), dim3((unsigned)systems),
                           dim3(kLtThreads), shm, s, P, kps, nbs);
    else
        hipLaunchKernelGGL((lt_mfma_kernel<TG, MULTI, kPerLoader>), dim3((unsigned)systems),
                           dim3(kLtThreads), shm, s, P, kps, nbs);
}

template <int TG>
void lt_launch(const LtParams &P, int64_t systems, size_t shm, int kps, int nbs, hipStream_t s) {
    if (P.kl > kBlk)
        lt_launch<TG, true>(P, systems, shm, kps, nbs, s);
    else
        lt_launch<TG, false>(P, systems, shm, kps, nbs, s);
}

}  // namespace

int launch_getrs_lt(LtParams P, int64_t systems, hipStream_t s) {
    int kps = 5;
    while ((1 << kps) < P.kl) ++kps;
    // the window, or the whole vector and the kl positions past it (which have
    // to be zero, not the slots of others)
    int R = 64;
    while (R < P.kl + std::min(P.n, 192)) R <<= 1;
    P.R = R;
    // rows per half: few where many systems share a CU (their LDS bounds how
    // many fit), less than the full half where the window is largest, and no
    // more than there are
    const int room = systems >= 512 ? 512 : (R > 1024 ? kHalfMax / 2 : kHalfMax);
    int nbs = 0;
    while (nbs < 6 && (2 << (nbs + kps)) <= room && (1 << nbs) < P.n - 1) ++nbs;
    const size_t shm = (size_t(2) * R + 64 + (size_t(2) << (nbs + kps)) + (size_t(1) << kps) + kBlk) *
                       sizeof(double);
    // groups of the last block, rounded up to one of the compiled counts
    const int groups = ((P.kl - 1) % kBlk) / 4 + 1;
    if (groups <= 1)
        lt_launch<1>(P, systems, shm, kps, nbs, s);
    else if (groups <= 2)
        lt_launch<2>(P, systems, shm, kps, nbs, s);
    else if (groups <= 4)
        lt_launch<4>(P, systems, shm, kps, nbs, s);
    else
        lt_launch<kGroups>(P, systems, shm, kps, nbs, s);
    BANDLU_CHECK_LAUNCH("band_getrs_t (L^T pass)");
    return BANDLU_OK;
}

}  // namespace bandlu
