"""The work that this framework is timed on: what its users call it for, over
the sizes that its workloads, tests and benchmark use.

Every case is one pass through public entry points of
``paper_2608_22099_amd`` on seeded synthetic bands (fp64, the one data type).
Conventions are the binding's: a tensor ``A`` of shape (n, lda) holds the
column-major matrix with ``A[j, i]`` = element (i, j); a band array (n, ldab)
is the xGBTRF layout; right-hand sides are (nrhs, n).

The kinds of pass:

  solve   dense-stored matrix -> structure_aware_lu (detect, host policy,
          convert, band LU) -> solve of one right-hand side
  gbsv    dense-stored matrix -> detect, host policy, convert -> band_gbsv
          (factor and solve in one call)
  batch   the same path for many small systems, by the batched entry points
  spd     dense-stored SPD matrix -> structure_aware_solve (band Cholesky)
  chol    band-stored SPD matrix -> band_pbtrf and band_pbtrs
  trans   factors in hand -> band_getrs_t (A^T X = B)
  rect    band-stored rectangular matrix -> band_getrf_mn
  band    band-stored matrix -> band_getrf and band_getrs, several
          right-hand sides
  fused   dense-stored matrix -> band_detect_convert (one read)
"""
import math

import numpy as np
import torch

from paper_2608_22099_amd import bandlu, policy

F64 = torch.float64


def listed():
    return [
        # a small system solved on its own: launch latency and a short chain
        dict(name="solve_n1000_kl3_ku3", kind="solve", n=1000, kl=3, ku=3, dist="normal",
             shift=0.0),
        # a diagonally dominant narrow band (discretised operators)
        dict(name="solve_n8192_kl16_ku16", kind="solve", n=8192, kl=16, ku=16, dist="normal",
             shift=64.0),
        # very different lower and upper bandwidths, with interchanges (rows
        # swapped in pairs: plain random entries give an unbounded solution
        # where the two bandwidths differ)
        dict(name="solve_n16384_kl2_ku64", kind="solve", n=16384, kl=2, ku=64, dist="uniform",
             shift=64.0, swapped=True),
        # the paper's own example: 10^4 x 10^4 with 100 sub- and 100
        # super-diagonals, random, so that interchanges happen at most steps
        dict(name="solve_n10000_kl100_ku100", kind="solve", n=10000, kl=100, ku=100,
             dist="normal", shift=0.0),
        # the benchmark's default: the largest matrix, a wide dominant band
        dict(name="gbsv_n32768_kl256_ku256", kind="gbsv", n=32768, kl=256, ku=256,
             dist="normal", shift=1024.0, nrhs=1),
        # thousands of independent small systems
        dict(name="batch4096_n256_kl4_ku4", kind="batch", n=256, kl=4, ku=4, dist="normal",
             shift=0.0, batch=4096),
        # a symmetric positive definite system through the dispatch
        dict(name="spd_n8192_kd64", kind="spd", n=8192, kd=64),
        # a large band-stored SPD system
        dict(name="chol_n32768_kd140", kind="chol", n=32768, kd=140, nrhs=1),
        # the transposed system with factors that the program keeps
        dict(name="trans_n32768_kl256_ku256", kind="trans", n=32768, kl=256, ku=256,
             dist="normal", shift=1024.0, nrhs=1),
        # a rectangular band
        dict(name="rect_m9216_n8192_kl16_ku16", kind="rect", m=9216, n=8192, kl=16, ku=16,
             dist="normal", shift=0.0),
        # a medium band kept in band storage, several right-hand sides
        dict(name="band_n4096_kl31_ku31_rhs16", kind="band", n=4096, kl=31, ku=31,
             dist="normal", shift=0.0, nrhs=16),
        # identify and convert in one read, odd size, caps above the band
        dict(name="fused_n12287_kl48_ku32", kind="fused", n=12287, kl=48, ku=32, kl_cap=64,
             ku_cap=64, dist="normal", shift=0.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "gbsv", "batch", "spd", "chol", "trans", "rect", "band",
                       "fused"])
    dist = rng.choice(["normal", "uniform"])
    rows = rng.choice(["dominant", "swapped", "random"])

    def band(lo, hi_l, hi_u):
        """Bandwidths and values: dominant rows, the same in swapped pairs, or
        random entries (no larger than one another, equal bandwidths)."""
        kl, ku = _log(rng, lo, hi_l), _log(rng, lo, hi_u)
        if rows == "random":
            return dict(kl=kl, ku=kl, dist=dist, shift=0.0)
        return dict(kl=kl, ku=ku, dist=dist, shift=float(2 * (kl + ku) + 2),
                    swapped=rows == "swapped")

    if kind == "solve":
        n = _log(rng, 128, 16384)
        return dict(kind=kind, n=n, **band(1, min(128, n // 8), min(128, n // 8)))
    if kind == "gbsv":
        n = _log(rng, 1024, 32768)
        return dict(kind=kind, n=n, nrhs=_log(rng, 1, 8),
                    **band(16, min(256, n // 8), min(256, n // 8)))
    if kind == "batch":
        n = _log(rng, 32, 512)
        return dict(kind=kind, n=n, batch=min(_log(rng, 64, 4096), 2 ** 28 // (n * n)),
                    **band(1, min(16, n // 8), min(16, n // 8)))
    if kind == "spd":
        n = _log(rng, 256, 8192)
        return dict(kind=kind, n=n, kd=_log(rng, 1, min(128, n // 8)))
    if kind == "chol":
        return dict(kind=kind, n=_log(rng, 1024, 32768), kd=_log(rng, 4, 140),
                    nrhs=_log(rng, 1, 4))
    if kind == "trans":
        return dict(kind=kind, n=_log(rng, 1024, 32768), nrhs=_log(rng, 1, 4), **band(1, 256, 256))
    if kind == "rect":
        n = _log(rng, 512, 8192)
        return dict(kind=kind, m=int(n * rng.uniform(0.8, 1.25)), n=n, **band(1, 32, 32))
    if kind == "band":
        return dict(kind=kind, n=_log(rng, 256, 8192), nrhs=_log(rng, 1, 32), **band(1, 31, 64))
    n = _log(rng, 1024, 16384)
    b = band(1, 128, 128)
    return dict(kind="fused", n=n, kl_cap=b["kl"] + rng.randint(0, 32),
                ku_cap=b["ku"] + rng.randint(0, 32), **b)


# ------------------------------------------------------------------ inputs --
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed):
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    return g


def _values(shape, dist, g):
    x = torch.empty(shape, dtype=F64, device=_device())
    return x.normal_(generator=g) if dist == "normal" else x.uniform_(-1.0, 1.0, generator=g)


def _clear_outside(S, m, top):
    """Zero the slots of a band (.., n, h) whose row j + r - top is not in 0..m-1."""
    n, h = S.shape[-2:]
    j = torch.arange(n, device=S.device)[:, None]
    r = torch.arange(h, device=S.device)[None, :]
    i = j + r - top
    S.masked_fill_((i < 0) | (i >= m), 0.0)


def _band(case, g, batch=None):
    """Band array (.., n, 2kl+ku+1) in the xGBTRF layout, fill rows +0.0.

    ``shift`` is added to the diagonal.  With ``swapped``, the matrix has one
    diagonal less on either side, and then about half of its rows change
    places with their neighbour (a band of kl, ku whose pivots are found
    below the diagonal there)."""
    n, kl, ku = case["n"], case["kl"], case["ku"]
    lead = () if batch is None else (batch,)
    S = torch.zeros(lead + (n, 2 * kl + ku + 1), dtype=F64, device=_device())
    S[..., kl:] = _values(lead + (n, kl + ku + 1), case["dist"], g)
    S[..., kl + ku] += case["shift"]
    m = case.get("m", n)
    if case.get("swapped"):
        S[..., kl] = 0.0
        S[..., -1] = 0.0
        # rows i and i+1 (i even) of column j sit at r = kl+ku+i-j and r+1
        pick = torch.rand(m // 2, generator=g, device=S.device) < 0.5
        j = torch.arange(n, device=S.device)[:, None]
        i = j + torch.arange(kl, 2 * kl + ku, device=S.device)[None, :] - (kl + ku)
        take = (i >= 0) & (i % 2 == 0) & (i + 1 < m)
        take &= pick[(i // 2).clamp(0, max(0, m // 2 - 1))]
        lo, hi = S[..., kl:-1].clone(), S[..., kl + 1:].clone()
        S[..., kl:-1] = torch.where(take, hi, S[..., kl:-1])
        S[..., kl + 1:] = torch.where(take, lo, S[..., kl + 1:])
    _clear_outside(S, m, kl + ku)
    return S


def _spd_lower(n, kd, g):
    """Lower band (n, kd+1), strictly dominant: element (i, j) at [j, i-j]."""
    L = _values((n, kd + 1), "normal", g)
    _clear_outside(L, n, 0)
    L[:, 0] = 0.0
    a = L.abs()
    d = a.sum(1) + 1.0
    for t in range(1, kd + 1):
        d[t:] += a[: n - t, t]
    L[:, 0] = d
    return L


def _dense(S, kl, ku, top):
    """Dense-stored matrix (.., n, n) of a band whose diagonal is row ``top``."""
    n = S.shape[-2]
    A = torch.zeros(S.shape[:-1] + (n,), dtype=F64, device=S.device)
    for d in range(-ku, kl + 1):
        src = S[..., max(0, -d):n - max(0, d), top + d]
        A.diagonal(d, dim1=-2, dim2=-1).copy_(src)
    return A


def _inputs(case, seed):
    """(matrix in band form, right-hand sides) of a case, from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind in ("spd", "chol"):
        return _spd_lower(case["n"], case["kd"], g), _values((case.get("nrhs", 1), case["n"]),
                                                             "normal", g)
    S = _band(case, g, case.get("batch"))
    if kind in ("rect", "fused"):
        return S, None
    lead = (case["batch"],) if kind == "batch" else ()
    return S, _values(lead + (case.get("nrhs", 1), case["n"]), "normal", g)


def prepare(case, seed):
    kind = case["kind"]
    S, B = _inputs(case, seed)
    st = dict(case=case, B=B)
    if kind in ("solve", "gbsv", "batch", "fused"):
        st["A"] = _dense(S, case["kl"], case["ku"], case["kl"] + case["ku"])
    elif kind == "spd":
        low = _dense(S, case["kd"], 0, 0)
        st["A"] = low + low.tril(-1).transpose(0, 1) + low.triu(1).transpose(0, 1)
    elif kind == "trans":
        st["ipiv"], st["info"] = bandlu.band_getrf(S, case["kl"], case["ku"])
        st["S"] = S
    else:
        st["S"] = S
    return st


def run(st):
    case, B = st["case"], st["B"]
    kind = case["kind"]
    if kind == "solve":
        f = policy.structure_aware_lu(st["A"])
        X = f.solve(B.clone())
        return dict(AB=f.AB, ipiv=f.ipiv, info=f.info, X=X)
    if kind == "gbsv":
        A, n = st["A"], case["n"]
        caps = policy.band_caps(n)
        kl, ku, exceeded = (int(v) for v in bandlu.band_detect(A, *caps).cpu())
        if exceeded or not policy.speedup_predicate(n, kl, ku):
            raise RuntimeError("not taken as banded")
        AB = bandlu.dense_to_band(A, kl, ku)
        X = B.clone()
        ipiv, info = bandlu.band_gbsv(AB, kl, ku, X)
        return dict(AB=AB, ipiv=ipiv, info=info, X=X)
    if kind == "batch":
        A = st["A"]
        det, dmax = bandlu.band_detect_batched(A)
        kl, ku, _ = (int(v) for v in dmax.cpu())
        AB = bandlu.dense_to_band_batched(A, kl, ku)
        ipiv, info = bandlu.band_getrf_batched(AB, kl, ku)
        X = bandlu.band_getrs_batched(AB, kl, ku, ipiv, B.clone())
        return dict(det=det, AB=AB, ipiv=ipiv, info=info, X=X)
    if kind == "spd":
        X = B.clone()
        branch = policy.structure_aware_solve(st["A"], X)
        return dict(cholesky=int(branch == "cholesky"), X=X)
    if kind == "chol":
        AB = st["S"].clone()
        X = B.clone()
        info = bandlu.band_pbtrf(AB, case["kd"])
        bandlu.band_pbtrs(AB, case["kd"], X)
        return dict(AB=AB, info=info, X=X)
    if kind == "trans":
        X = bandlu.band_getrs_t(st["S"], case["kl"], case["ku"], st["ipiv"], B.clone())
        return dict(X=X)
    if kind == "rect":
        AB = st["S"].clone()
        ipiv, info = bandlu.band_getrf_mn(AB, case["m"], case["kl"], case["ku"])
        return dict(AB=AB, ipiv=ipiv, info=info)
    if kind == "band":
        AB = st["S"].clone()
        ipiv, info = bandlu.band_getrf(AB, case["kl"], case["ku"])
        X = bandlu.band_getrs(AB, case["kl"], case["ku"], ipiv, B.clone())
        return dict(AB=AB, ipiv=ipiv, info=info, X=X)
    out, AB = bandlu.band_detect_convert(st["A"], case["kl_cap"], case["ku_cap"])
    kl, ku, _ = (int(v) for v in out.cpu())
    return dict(det=out, AB=bandlu.band_view(AB, case["kl_cap"], case["ku_cap"], kl, ku))


# -------------------------------------------------------------------- work --
def work(case):
    """Each input read once and each output written once; the operations of
    the unblocked algorithms."""
    kind, n, b = case["kind"], case["n"], case.get("batch", 1)
    r = case.get("nrhs", 1)
    if kind in ("spd", "chol"):
        kd = case["kd"]
        factor = n * kd * (kd + 2)
        solve = 4 * n * kd * r
        if kind == "spd":  # detection, the symmetry test, the band, the solution
            return dict(bytes=8 * (n * n + 2 * n * kd + n * (kd + 1) + 2 * n * r),
                        flops=factor + solve)
        return dict(bytes=8 * (2 * n * (kd + 1) + 2 * n * r), flops=factor + solve)
    kl, ku = case["kl"], case["ku"]
    ldab, inband = 2 * kl + ku + 1, n * (kl + ku + 1)
    factor = 2 * min(n, case.get("m", n)) * kl * (kl + ku + 1)
    solve = 2 * n * (2 * kl + ku) * r
    if kind == "trans":
        return dict(bytes=8 * ldab * n + 4 * n + 16 * n * r, flops=solve)
    if kind == "rect":
        return dict(bytes=8 * (inband + ldab * n) + 4 * min(n, case["m"]), flops=factor)
    if kind == "band":
        return dict(bytes=8 * (inband + ldab * n) + 4 * n + 16 * n * r, flops=factor + solve)
    if kind == "fused":
        return dict(bytes=8 * (n * n + ldab * n), flops=0)
    return dict(bytes=b * (8 * (n * n + ldab * n) + 4 * n + 16 * n * r),
                flops=b * (factor + solve))


# --------------------------------------------------------------- tolerance --
def tolerance(case):
    """Relative error of fp64 results when the sums are taken in another
    order: the column steps against blocked products, about four times the
    largest difference seen over the listed cases and fifty drawn ones (1.3e-15
    on dominant rows, 3e-12 on random entries, whose condition varies)."""
    if case["kind"] == "fused":
        return "exact"
    if case["kind"] in ("spd", "chol") or case["shift"]:
        return dict(rel=6e-15, max=3e-14)
    return dict(rel=2e-11, max=4e-11)


# ------------------------------------------------------------------- exact --
_NB = 64


def _gbtrf(S, m, kl, ku):
    """Band LU in product form, by panels of dense windows (numpy arrays)."""
    n, h = S.shape
    kv = kl + ku
    AB = S.copy()
    steps = min(m, n)
    piv = np.zeros(steps, dtype=np.int64)
    for j0 in range(0, steps, _NB):
        nb = min(_NB, steps - j0)
        rows = min(m - j0, nb + kl)
        cols = min(n - j0, nb + kv)
        jj, ii = np.meshgrid(np.arange(cols), np.arange(rows))
        r = kv + ii - jj
        ok = (r >= 0) & (r < h)
        W = np.zeros((rows, cols))
        W[ok] = AB[j0 + jj[ok], r[ok]]
        LU, p = torch.linalg.lu_factor(torch.from_numpy(W[:, :nb].copy()))
        LU, p = LU.numpy().copy(), p.numpy() - 1
        piv[j0:j0 + nb] = j0 + p[:nb] + 1
        R = W[:, nb:]
        for s in range(nb):
            if p[s] != s:
                R[[s, p[s]]] = R[[p[s], s]]
        if R.shape[1]:
            T = torch.from_numpy(LU[:nb, :nb].copy())
            U = torch.linalg.solve_triangular(T, torch.from_numpy(R[:nb].copy()), upper=False,
                                              unitriangular=True).numpy()
            R[nb:] -= LU[nb:] @ U
            R[:nb] = U
        # the multipliers as their own step left them (later interchanges undone)
        for s in range(nb - 1, 0, -1):
            if p[s] != s:
                LU[[s, p[s]], :s] = LU[[p[s], s], :s]
        W[:, :nb] = LU
        W[:, nb:] = R
        AB[j0 + jj[ok], r[ok]] = W[ok]
    return AB, piv


def _solve_columns(D, offs, B, order):
    """x_j = b_j / D[j, 0], then b_{j+offs} -= D[j, 1:] x_j, in the given order."""
    n = B.shape[0]
    lo, hi = (1, offs + 1) if offs > 0 else (offs, 0)
    for j in order:
        B[j] /= D[j, 0]
        a, b = max(0, j + lo), min(n, j + hi)
        if a < b:
            w = D[j, 1:][a - (j + lo):b - (j + lo)]
            B[a:b] -= w[:, None] * B[j]
    return B


def _gbtrs(AB, kl, ku, piv, B):
    n, kv = AB.shape[0], kl + ku
    B = B.T.copy()
    for j in range(n - 1):
        p = piv[j] - 1
        if p != j:
            B[[j, p]] = B[[p, j]]
        km = min(kl, n - 1 - j)
        B[j + 1:j + 1 + km] -= AB[j, kv + 1:kv + 1 + km, None] * B[j]
    D = np.concatenate([AB[:, kv:kv + 1], AB[:, :kv]], axis=1)
    return _solve_columns(D, -kv, B, range(n - 1, -1, -1)).T.copy()


def _gbtrs_t(AB, kl, ku, piv, B):
    n, kv = AB.shape[0], kl + ku
    B = B.T.copy()
    for j in range(n):
        a = max(0, j - kv)
        B[j] -= AB[j, kv - (j - a):kv] @ B[a:j]
        B[j] /= AB[j, kv]
    for j in range(n - 2, -1, -1):
        km = min(kl, n - 1 - j)
        B[j] -= AB[j, kv + 1:kv + 1 + km] @ B[j + 1:j + 1 + km]
        p = piv[j] - 1
        if p != j:
            B[[j, p]] = B[[p, j]]
    return B.T.copy()


def _pbtrf(S, kd):
    n = S.shape[0]
    AB = S.copy()
    for j0 in range(0, n, _NB):
        nb = min(_NB, n - j0)
        rows = min(n - j0, nb + kd)
        jj, ii = np.meshgrid(np.arange(rows), np.arange(rows))
        r = ii - jj
        ok = (r >= 0) & (r <= kd)
        W = np.zeros((rows, rows))
        W[ok] = AB[j0 + jj[ok], r[ok]]
        L = np.linalg.cholesky(np.tril(W[:nb, :nb]) + np.tril(W[:nb, :nb], -1).T)
        W[:nb, :nb] = L
        if rows > nb:
            X = torch.linalg.solve_triangular(torch.from_numpy(L), torch.from_numpy(
                W[nb:, :nb].T.copy()), upper=False).numpy().T
            W[nb:, :nb] = X
            W[nb:, nb:] -= X @ X.T
        AB[j0 + jj[ok], r[ok]] = W[ok]
    return AB


def _pbtrs(AB, kd, B):
    n = AB.shape[0]
    B = _solve_columns(AB, kd, B.T.copy(), range(n))
    for j in range(n - 1, -1, -1):
        km = min(kd, n - 1 - j)
        B[j] -= AB[j, 1:1 + km] @ B[j + 1:j + 1 + km]
        B[j] /= AB[j, 0]
    return B.T.copy()


def exact(case, seed):
    kind = case["kind"]
    S, B = _inputs(case, seed)
    S = S.cpu().numpy()
    B = None if B is None else B.cpu().numpy()
    if kind in ("spd", "chol"):
        AB = _pbtrf(S, case["kd"])
        X = _pbtrs(AB, case["kd"], B)
        return dict(cholesky=None, X=X) if kind == "spd" else dict(AB=AB, info=None, X=X)
    kl, ku = case["kl"], case["ku"]
    if kind == "fused":
        return dict(det=None, AB=S)
    if kind == "rect":
        return dict(AB=_gbtrf(S, case["m"], kl, ku)[0], ipiv=None, info=None)
    if kind == "batch":
        return _exact_batch(S, B, kl, ku)
    AB, piv = _gbtrf(S, case["n"], kl, ku)
    if kind == "trans":
        return dict(X=_gbtrs_t(AB, kl, ku, piv, B))
    return dict(AB=AB, ipiv=None, info=None, X=_gbtrs(AB, kl, ku, piv, B))


def _exact_batch(S, B, kl, ku):
    """Column steps over the whole batch at once."""
    b, n, _ = S.shape
    kv = kl + ku
    AB, X = S.copy(), B[:, 0].copy()
    k = np.arange(b)
    for j in range(n):
        km = min(kl, n - 1 - j)
        p = np.abs(AB[:, j, kv:kv + km + 1]).argmax(1)
        for c in range(min(kv, n - 1 - j) + 1):
            at = kv - c
            a = AB[k, j + c, at + p].copy()
            AB[k, j + c, at + p] = AB[:, j + c, at]
            AB[:, j + c, at] = a
        x = X[k, j + p].copy()
        X[k, j + p] = X[:, j]
        X[:, j] = x
        AB[:, j, kv + 1:kv + 1 + km] /= AB[:, j, kv, None]
        m = AB[:, j, kv + 1:kv + 1 + km]
        for c in range(1, min(kv, n - 1 - j) + 1):
            AB[:, j + c, kv - c + 1:kv - c + 1 + km] -= m * AB[:, j + c, kv - c, None]
        X[:, j + 1:j + 1 + km] -= m * X[:, j, None]
    for j in range(n - 1, -1, -1):
        X[:, j] /= AB[:, j, kv]
        a = max(0, j - kv)
        X[:, a:j] -= AB[:, j, kv - (j - a):kv] * X[:, j, None]
    return dict(det=None, AB=AB, ipiv=None, info=None, X=X[:, None])
