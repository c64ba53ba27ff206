"""GPU parity: the HIP path through the C ABI against the CPU oracle on the same
seeded inputs.  Run on an MI355X:  python -m pytest tests -m gpu -x -v"""
import math
import sys

import numpy as np
import pytest

from oracle import params as OP
from oracle import spectral_lsh as O
from workloads import make_inputs, Workload, Inputs, WORKLOADS
import parity as PR

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2607_19368_amd as P
    P.load()
    yield


def _custom(name, N, D, m, n_it, r, bits, seed=0, x="bf16", vocab=32768):
    """Zipf-embedded inputs of arbitrary shape (same recipe as the named workloads)."""
    from workloads import zipf_ids, embed, mixture
    wl = Workload(name, N, D, m, n_it, r, bits, 8.0, vocab, 0, x)
    if x == "f32":
        X, lab = mixture(seed, N, D)
        return Inputs(wl, X, lab)
    rng = np.random.default_rng(np.random.SeedSequence([seed, 0x1D5]))
    ids = zipf_ids(rng, vocab, N)
    return Inputs(wl, embed(seed, ids, D), ids)


# ------------------------------------------------------------------ feature map
# tiles used at 256 CUs: tiny, ragged, mistral7b_head -> 64 x 64; tiles64x128 ->
# 64 x 128; tiles128 -> 128 x 128; tiles256 -> 256 x 256 (all with a ragged last
# row block except tiny)
@pytest.mark.parametrize("case", ["tiny", "ragged", "mistral7b_head", "tiles64x128", "tiles128",
                                  "tiles256", "mistral7b_full", "ragged_m256"])
def test_feature_map_parity(case):
    if case == "tiny":
        inp = make_inputs("tiny")
    elif case == "ragged":
        inp = _custom("ragged", 1000, 264, 512, 16, 4, 6)
    elif case == "tiles64x128":
        inp = _custom("tiles64x128", 4090, 264, 1024, 16, 4, 6)
    elif case == "tiles128":
        inp = _custom("tiles128", 4000, 264, 2048, 16, 4, 6)
    elif case == "tiles256":
        inp = _custom("tiles256", 8000, 264, 2048, 16, 4, 6)
    elif case == "mistral7b_full":
        # the whole 4096 x 4096 x 1024 product (64 x 128 tiles, two per CU)
        inp = _custom("mistral7b_full", 4096, 4096, 1024, 16, 4, 6)
    elif case == "ragged_m256":
        # 8204 rows (the last 64-row tile partial), D = 3000 (47 K stages, the last
        # one zero-filled past D), m = 256 (64 x 64 tiles)
        inp = _custom("ragged_m256", 8204, 3000, 256, 16, 4, 6)
    else:
        inp = _custom("mistral7b_head", 1536, 4096, 1024, 16, 8, 10)
    wl = inp.workload
    _say(f"[featmap] {case} N={wl.N} D={wl.D} m={wl.m}")
    g = PR.run_gpu(inp, n_it=wl.r, want_phi=True)
    X = inp.x_float()
    Phi = O.feature_map(X, OP.projection(0, wl.D, wl.m), OP.phases(0, wl.m))
    Xh = O.bf16_round(X)
    scale = np.exp(np.sum(Xh * Xh, 1) / (2 * math.sqrt(wl.D))) * math.sqrt(2.0 / wl.m)
    err = np.abs(g.Phi - Phi) / scale[:, None]
    _say(f"   max |dPhi|/scale = {err.max():.3e}  mean = {err.mean():.3e}")
    assert err.max() <= 1e-5 and err.mean() <= 1e-6


def test_feature_map_gauss_option():
    inp = make_inputs("tiny")
    wl = inp.workload
    g = PR.run_gpu(inp, n_it=wl.r, kernel=1, want_phi=True)
    Phi = O.feature_map(inp.x_float(), OP.projection(0, wl.D, wl.m), OP.phases(0, wl.m), "gauss")
    err = np.abs(g.Phi - Phi) / math.sqrt(2.0 / wl.m)
    assert err.max() <= 1e-5


# ------------------------------------------------------------------ Lanczos .. SimHash on the oracle's Phi
# staged_m512 / staged_m256: 1024 chunks of 16 rows, more than two per CU, so
# each block of the pass streams several chunks through LDS (small m: 4 and 2
# rows per wave and chunk)
@pytest.mark.parametrize("case", ["tiny", "ragged", "staged_m512", "staged_m256"])
def test_lanczos_stage_on_oracle_phi(case):
    """Loads fp32(Phi_oracle) so both sides run Lanczos on the same operator:
    alpha/beta, Ritz values, Ritz vectors and codes must then agree closely."""
    if case == "tiny":
        inp = make_inputs("tiny")
    elif case == "ragged":
        inp = _custom("ragged", 1000, 264, 512, 40, 12, 8)
    elif case == "staged_m512":
        inp = _custom("staged_m512", 16380, 264, 512, 24, 8, 8)
    else:
        inp = _custom("staged_m256", 16380, 264, 256, 24, 8, 8)
    wl = inp.workload
    X = inp.x_float()
    Phi32 = O.feature_map(X, OP.projection(0, wl.D, wl.m), OP.phases(0, wl.m)).astype(np.float32)
    _say(f"[lanczos-stage] {case} N={wl.N} m={wl.m} n_it={wl.n_it} r={wl.r}")
    g = PR.run_gpu(inp, n_it=wl.n_it, phi_from=Phi32)
    # oracle on the very same fp32 operator
    Phi = Phi32.astype(np.float64)
    lz = O.lanczos(Phi, OP.start_vector(0, wl.N, 0), wl.n_it)
    vals, Z, _, _ = O.ritz(lz, wl.r)
    R = OP.hyperplanes(0, wl.r, wl.bits)
    gw = g.windows[0]
    assert gw.iters == lz.n_eff
    ra = np.max(np.abs(gw.alpha[:lz.n_eff] - lz.alpha) / np.abs(lz.alpha))
    rb = np.max(np.abs(gw.beta[:lz.n_eff] - lz.beta) / np.abs(lz.beta))
    rv = np.max(np.abs(gw.ritz - vals) / np.abs(vals))
    ang = PR.subspace_angle(Z, gw.Z)
    _say(f"   alpha rel {ra:.2e} beta rel {rb:.2e} ritz rel {rv:.2e} angle {ang:.2e}")
    assert ra < 1e-9 and rb < 1e-7 and rv < 1e-9 and ang < 1e-6
    # per-vector agreement (signs fixed by the first-entry rule)
    assert np.max(np.abs(gw.Z - Z)) < 1e-6
    proj = O.projections(Z, R)
    codes = O.simhash(Z, R)
    ex = np.any(np.abs(proj) < PR.EXCL, axis=1)
    assert np.array_equal(gw.codes[~ex], codes[~ex])
    assert np.max(np.abs(gw.proj - proj)) < 1e-7


# ------------------------------------------------------------------ Eigh(T) on given tridiagonals
def _tridiag_case(case):
    """(list of (alpha, beta) per window, r): beta has n entries, the last unused."""
    rng = np.random.default_rng(31)
    if case == "wilkinson21":
        n = 21
        al = np.abs(10.0 - np.arange(n))
        return [(al, np.ones(n))], 21
    if case == "toeplitz96":
        n = 96
        return [(np.full(n, 2.0), np.full(n, -1.0))], 64
    if case == "repeated_blocks":
        bd = rng.uniform(0.0, 4.0, 8)
        bo = rng.uniform(0.5, 1.5, 8)
        al = np.tile(bd, 3)
        be = np.tile(bo, 3)
        be[7] = be[15] = 0.0
        return [(al, be)], 24
    if case == "null_space":
        al = np.concatenate([np.zeros(4), rng.uniform(1.0, 3.0, 12)])
        be = np.concatenate([np.zeros(4), rng.uniform(0.2, 0.8, 12)])
        return [(al, be)], 16
    # three windows of order 21: W21+, W21- and a random T
    n = 21
    k = np.arange(n)
    return [(np.abs(10.0 - k), np.ones(n)), (10.0 - k, np.ones(n)),
            (rng.uniform(-2, 2, n), rng.uniform(0.1, 1.0, n))], 12


@pytest.mark.parametrize("case", ["wilkinson21", "toeplitz96", "repeated_blocks", "null_space",
                                  "windows"])
def test_eigensolve_stage(case):
    """Eigh(T) and the Ritz coordinates alone (slh_eigh_ritz, Algorithm 1) on
    tridiagonals loaded with slh_load, with Q = [I; 0] so that Z holds the kept
    eigenvectors S.  Wilkinson's W21+ has a top pair 1e-13 apart; the repeated
    blocks give every eigenvalue multiplicity 3; the null-space case has a
    4-fold zero eigenvalue; the Toeplitz T has the closed-form spectrum
    a + 2 b cos(k pi / (n + 1)).  Eigenvalues within 1e-12 relative of LAPACK
    (absolute 1e-13 |T| for zero ones), kept vectors orthonormal to 1e-10,
    residuals |T s - theta s| <= 1e-12 |T|, the first nonzero entry of each
    vector positive, vectors outside clusters equal to LAPACK's within their
    conditioning (1e-10 + 4 eps |T| / gap, the gap to the nearest other
    eigenvalue of T), and cluster columns spanning LAPACK's subspace.  Where
    the first nonzero entry is at rounding level (an exact zero in LAPACK's
    vector of a decoupled block) its sign is not determined, and the vector is
    compared up to sign."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    wins, r = _tridiag_case(case)
    nw, n = len(wins), len(wins[0][0])
    L = 64 if nw > 1 else max(64, n)
    ctx = P.slh_create(L * nw, 8, 256, r, 1, 0)
    if nw > 1:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
    al = np.stack([w[0] for w in wins]).astype(np.float64)
    be = np.stack([w[1] for w in wins]).astype(np.float64)
    Q = np.zeros((nw, n + 1, L))
    Q[:, np.arange(n), np.arange(n)] = 1.0
    for which, arr in ((B.SLH_OUT_ALPHA, al), (B.SLH_OUT_BETA, be), (B.SLH_OUT_Q, Q)):
        P.slh_load(ctx, which, torch.from_numpy(np.ascontiguousarray(arr)).cuda())
    ritz, iters = P.slh_eigh_ritz(ctx, n)
    Z = P.slh_copy_out(ctx, B.SLH_OUT_Z)
    assert list(iters) == [n] * nw
    for a in range(nw):
        T = O.tridiagonal(al[a], be[a][:n - 1])
        tn = np.max(np.sum(np.abs(T), axis=1))
        th_all, S_all = O.eigh_tridiagonal(al[a], be[a][:n - 1])
        th_o, S_o = th_all[n - r:], S_all[:, n - r:]
        S = Z[a][:n]
        assert np.all(Z[a][n:] == 0)
        big = np.abs(th_o) > 1e-3 * tn
        err = np.abs(ritz[a] - th_o)
        assert np.all(err[big] <= 1e-12 * np.abs(th_o[big])), (case, a, err[big].max())
        assert np.all(err[~big] <= 1e-13 * tn), (case, a, err[~big].max(initial=0))
        orth = np.abs(S.T @ S - np.eye(r)).max()
        res = np.abs(T @ S - S * ritz[a][None, :]).max()
        _say(f"[eigh] {case} window {a}: max theta err {err.max():.2e}  |S^T S - I| {orth:.2e}  "
             f"residual {res:.2e} (|T| {tn:.2f})")
        assert orth <= 1e-10 and res <= 1e-12 * tn
        for c in range(r):
            nz = np.flatnonzero(S[:, c] != 0.0)
            assert S[nz[0], c] > 0
        # clusters by the same rule as the library: gaps <= 1e-6 |T|
        gaps = np.diff(th_o) <= 1e-6 * tn
        c = 0
        while c < r:
            c1 = c
            while c1 + 1 < r and gaps[c1]:
                c1 += 1
            if c1 == c:
                kk = n - r + c
                gap = min([abs(th_all[kk] - th_all[q]) for q in (kk - 1, kk + 1) if 0 <= q < n],
                          default=tn)
                tol = 1e-10 + 4 * 2.2e-16 * tn / max(gap, 1e-300)
                first = S[np.flatnonzero(S[:, c] != 0.0)[0], c]
                d_same = np.abs(S[:, c] - S_o[:, c]).max()
                d = d_same if abs(first) > 1e-12 else min(d_same, np.abs(S[:, c] + S_o[:, c]).max())
                assert d <= tol, (case, a, c, d, tol)
            else:
                sv = np.linalg.svd(S_o[:, c:c1 + 1].T @ S[:, c:c1 + 1], compute_uv=False)
                assert sv.min() >= 1.0 - 1e-10, (case, a, c, c1, sv)
            c = c1 + 1


@pytest.mark.parametrize("n_it", [96, 160, 256])
def test_lanczos_basis_orthonormal(n_it):
    """The GPU Lanczos basis (Algorithm 2 with full re-orthogonalization: the
    three-term recurrence, then one classical Gram-Schmidt pass against the
    whole basis, beta from |z1|^2 - |h2|^2) on the oracle's Phi stays
    orthonormal: |Q^T Q - I| <= 1e-12 over the n_it vectors, and its alpha and
    beta match the oracle's (two Gram-Schmidt passes) to 1e-9."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    inp = _custom("qorth", 4000, 264, 512, n_it, 8, 8)
    wl = inp.workload
    Phi32 = O.feature_map(inp.x_float(), OP.projection(0, wl.D, wl.m),
                          OP.phases(0, wl.m)).astype(np.float32)
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    P.slh_load(ctx, B.SLH_OUT_PHI, torch.from_numpy(Phi32).cuda())
    _, iters = P.slh_lanczos(ctx, n_it)
    assert iters[0] == n_it
    Q = P.slh_copy_out(ctx, B.SLH_OUT_Q)[0][:n_it]
    orth = np.abs(Q @ Q.T - np.eye(n_it)).max()
    lz = O.lanczos(Phi32.astype(np.float64), OP.start_vector(0, wl.N, 0), n_it)
    al = P.slh_copy_out(ctx, B.SLH_OUT_ALPHA)[0]
    be = P.slh_copy_out(ctx, B.SLH_OUT_BETA)[0]
    ra = np.max(np.abs(al - lz.alpha) / np.abs(lz.alpha))
    rb = np.max(np.abs(be - lz.beta) / np.abs(lz.beta))
    _say(f"[basis] n_it={n_it}: |Q^T Q - I| = {orth:.2e}  alpha rel {ra:.2e}  beta rel {rb:.2e}")
    assert orth <= 1e-12
    assert ra <= 1e-9 and rb <= 1e-9


# ------------------------------------------------------------------ merge on the oracle's codes
@pytest.mark.parametrize("case", ["tiny", "mistral7b", "windows"])
def test_merge_stage_on_oracle_codes(case):
    """Loads oracle codes: the bucket maps and positions must be bit-exact and the
    embeddings within 1e-5 (fp32 sums)."""
    if case == "tiny":
        inp = make_inputs("tiny")
        window = 0
        codes = np.random.default_rng(1).integers(0, 64, inp.workload.N)
    elif case == "mistral7b":
        inp = make_inputs("mistral7b")
        window = 0
        # a Zipf-like code distribution: many members in a few buckets (spans chunks)
        rng = np.random.default_rng(2)
        codes = np.minimum(rng.zipf(1.3, inp.workload.N) - 1, 1023)
    else:
        inp = _custom("windows", 4096, 512, 256, 16, 4, 10)
        window = 512
        codes = np.random.default_rng(3).integers(0, 1024, inp.workload.N)
        codes[:512] = 5          # one window is a single bucket
    wl = inp.workload
    _say(f"[merge-stage] {case} N={wl.N} D={wl.D} window={window}")
    g = PR.run_gpu(inp, n_it=wl.r, window=window, codes_from=codes.astype(np.uint32))
    L = window or wl.N
    Es, Ps, t2m, base = [], [], np.zeros(wl.N, np.int64), 0
    for w in range(wl.N // L):
        mg = O.merge(inp.x_float(slice(w * L, (w + 1) * L)), codes[w * L:(w + 1) * L],
                     positions=w * L + np.arange(L))
        Es.append(mg.E)
        Ps.append(mg.P)
        t2m[w * L:(w + 1) * L] = base + mg.tok2macro
        base += len(mg.P)
    E, P = np.concatenate(Es), np.concatenate(Ps)
    assert np.array_equal(g.P, P)
    assert np.array_equal(g.t2m, t2m)
    rel = np.linalg.norm(g.E - E, axis=1) / np.maximum(np.linalg.norm(E, axis=1), 1e-30)
    _say(f"   M={len(P)} max emb rel {rel.max():.2e}")
    assert rel.max() <= 1e-5


# ------------------------------------------------------------------ end to end
E2E = {
    "tiny": dict(),
    "mistral7b": dict(),
    "qwen7b": dict(),
    # the same prompt with one pass over Phi per Lanczos step instead of the
    # resident kernel that the default takes at this size
    "qwen7b_streaming": dict(resident=0),
}


@pytest.mark.parametrize("name", list(E2E))
def test_end_to_end(name):
    inp = make_inputs(name.replace("_streaming", ""))
    wl = inp.workload
    _say(f"[e2e] {name} N={wl.N} D={wl.D} m={wl.m} n_it={wl.n_it} r={wl.r} bits={wl.bits}")
    g = PR.run_gpu(inp, n_it=wl.n_it, **E2E[name])
    o = PR.run_oracle(inp, n_it=wl.n_it)
    rep = PR.compare(o, g, wl.N)
    _say(f"   {rep}  M={len(g.P)}  rho_achieved={wl.N / len(g.P):.2f}")


# ------------------------------------------------------------------ resident Lanczos kernel
def _lanczos_on_phi(Phi32, wl, n_it, resident):
    """Lanczos + Eigh + Ritz on a loaded Phi with SLH_OPT_RESIDENT = resident
    (timing mode, so that the stage record says which path ran)."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    P.slh_set_option(ctx, B.SLH_OPT_TIMING, 1)
    P.slh_set_option(ctx, B.SLH_OPT_RESIDENT, resident)
    P.slh_load(ctx, B.SLH_OUT_PHI, torch.from_numpy(Phi32).cuda())
    ritz, iters = P.slh_lanczos(ctx, n_it)
    out = dict(ritz=ritz[0], iters=iters[0],
               Q=P.slh_copy_out(ctx, B.SLH_OUT_Q)[0][:iters[0]],
               alpha=P.slh_copy_out(ctx, B.SLH_OUT_ALPHA)[0],
               beta=P.slh_copy_out(ctx, B.SLH_OUT_BETA)[0],
               Z=P.slh_copy_out(ctx, B.SLH_OUT_Z)[0],
               used=P.slh_stage_times(ctx)["lanczos_resident"])
    return out


@pytest.mark.parametrize("case", ["m1024_ragged", "m2048"])
def test_resident_lanczos_on_oracle_phi(case):
    """The resident kernel (the whole Lanczos loop of Algorithm 2 as one
    persistent kernel, rows of Phi held in registers, blocks exchanging
    step-tagged values) on the oracle's Phi: it runs where SLH_OPT_RESIDENT
    allows it and not otherwise; its basis is orthonormal to 1e-12; alpha and
    beta match the oracle's to 1e-9; against the streaming path on the same Phi
    (the same recurrence, partial sums grouped differently) alpha, beta and the
    Ritz values agree to 1e-10 relative and the kept Ritz subspace to 1e-8 rad.
    A row count that is not a multiple of the block's 32 rows (2000) pads the
    last blocks with zero rows."""
    N, m = (2000, 1024) if case == "m1024_ragged" else (4096, 2048)
    n_it = 64
    inp = _custom("res_" + case, N, 264, m, n_it, 16, 8)
    wl = inp.workload
    Phi32 = O.feature_map(inp.x_float(), OP.projection(0, wl.D, wl.m),
                          OP.phases(0, wl.m)).astype(np.float32)
    res = _lanczos_on_phi(Phi32, wl, n_it, 1)
    stm = _lanczos_on_phi(Phi32, wl, n_it, 0)
    assert res["used"] == 1.0 and stm["used"] == 0.0
    assert res["iters"] == stm["iters"] == n_it
    Q = res["Q"]
    orth = np.abs(Q @ Q.T - np.eye(n_it)).max()
    lz = O.lanczos(Phi32.astype(np.float64), OP.start_vector(0, wl.N, 0), n_it)
    ra = np.max(np.abs(res["alpha"] - lz.alpha) / np.abs(lz.alpha))
    rb = np.max(np.abs(res["beta"] - lz.beta) / np.abs(lz.beta))
    da = np.max(np.abs(res["alpha"] - stm["alpha"]) / np.abs(stm["alpha"]))
    db = np.max(np.abs(res["beta"] - stm["beta"]) / np.abs(stm["beta"]))
    dr = np.max(np.abs(res["ritz"] - stm["ritz"]) / np.abs(stm["ritz"]))
    ang = PR.subspace_angle(stm["Z"], res["Z"])
    _say(f"[resident] {case}: |Q^T Q - I| {orth:.2e}  alpha/beta vs oracle {ra:.2e}/{rb:.2e}  "
         f"vs streaming alpha {da:.2e} beta {db:.2e} ritz {dr:.2e} angle {ang:.2e}")
    assert orth <= 1e-12
    assert ra <= 1e-9 and rb <= 1e-9
    assert da <= 1e-10 and db <= 1e-10 and dr <= 1e-10 and ang <= 1e-8


@pytest.mark.parametrize("N,m,n_it,window", [
    (100, 256, 20, 0),        # four waves a slice, four blocks, most of the last one past the end
    (8190, 256, 256, 0),      # 256 blocks, as many threads as blocks, 257 entries of h2
    (513, 512, 40, 0),        # one row in the last block that holds any
    (1000, 768, 33, 0),       # columns not a power of two
    (700, 1280, 256, 0),      # five waves
    (2500, 1536, 24, 0), (300, 1792, 24, 0),
    (4097, 2048, 24, 0),      # past 128 blocks of 32 rows
    (8193, 2048, 24, 0),      # past the registers: rows in LDS too
    (10240, 1280, 24, 0),     # ... in every slot
    (64 * 40, 512, 24, 64), (5 * 161, 1024, 24, 161), (3 * 37, 2048, 12, 37),
    (21 * 900, 1024, 24, 900)])   # two launches, of 11 and 10 windows
def test_resident_shapes_match_streaming(N, m, n_it, window):
    """Each shape of the resident kernel (column slices, rows per wave, blocks per
    window) against the streaming path on the same Phi: the same recurrence with
    partial sums grouped differently.  Basis orthonormal to 1e-12; alpha, beta to
    1e-8 relative (rounding of 1e-16 per sum amplified by |A| / beta along the
    steps, as between the streaming path and the oracle) where n_it is far below
    the rank min(N, m) (near it the extreme Ritz values have converged and the
    later entries of T are sensitive to every rounding; the Ritz values are not),
    and the Ritz values to 1e-10 of the largest."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    g = torch.Generator().manual_seed(N + m)
    Phi = torch.randn((N, m), generator=g) * torch.exp(-3.0 * torch.arange(m) / m)
    Phi = Phi.cuda()
    got = []
    for resident in (1, 0):
        ctx = P.slh_create(N, 64, m, 4, 4, 0)
        if window:
            P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, window)
        P.slh_set_option(ctx, B.SLH_OPT_TIMING, 1)
        P.slh_set_option(ctx, B.SLH_OPT_RESIDENT, resident)
        P.slh_load(ctx, B.SLH_OUT_PHI, Phi)
        ritz, iters = P.slh_lanczos(ctx, n_it)
        assert P.slh_stage_times(ctx)["lanczos_resident"] == float(resident)
        assert (iters == n_it).all()
        got.append((ritz, P.slh_copy_out(ctx, B.SLH_OUT_ALPHA), P.slh_copy_out(ctx, B.SLH_OUT_BETA),
                    P.slh_copy_out(ctx, B.SLH_OUT_Q)))
    (ritz, al, be, Q), (ritz0, al0, be0, _) = got
    worst = max(np.abs(q[:n_it] @ q[:n_it].T - np.eye(n_it)).max() for q in Q)
    da, db = np.abs(al / al0 - 1).max(), np.abs(be / be0 - 1).max()
    dr = np.abs(ritz - ritz0).max() / ritz0.max()
    _say(f"[resident shapes] {N}x{m} window {window}: |Q^T Q - I| {worst:.1e} alpha {da:.1e} beta {db:.1e} ritz {dr:.1e}")
    assert worst <= 1e-12 and dr <= 1e-10
    if 4 * n_it <= min(window or N, m):
        assert da <= 1e-8 and db <= 1e-8


@pytest.mark.timeout(120)
def test_resident_contexts_on_several_streams():
    """Contexts of two threads on streams of their own, each with a window that fills
    the chip: their resident kernels take turns (neither could finish while the
    other holds part of the chip), and every run gives the bits of a run alone."""
    import threading
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    N, m, n_it = 8192, 2048, 24
    X = 0.06 * torch.randn((N, 64), generator=torch.Generator().manual_seed(5)).cuda()
    ctx = P.slh_create(N, 64, m, 4, 4, 0)
    P.slh_feature_map(ctx, X)
    want = P.slh_lanczos(ctx, n_it)[0]
    torch.cuda.synchronize()
    got, errs = [], []

    def work():
        try:
            s = torch.cuda.Stream()
            c = P.slh_create(N, 64, m, 4, 4, 0)
            P.slh_set_stream(c, s)
            for _ in range(6):
                P.slh_feature_map(c, X)
                got.append(P.slh_lanczos(c, n_it)[0])
            s.synchronize()
        except Exception as e:  # reported by the main thread
            errs.append(e)

    ts = [threading.Thread(target=work) for _ in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errs, errs
    assert len(got) == 12 and all(np.array_equal(g, want) for g in got)


# ------------------------------------------------------------------ distinct rows
def _repeating_rows(N, D, distinct, seed):
    """N bf16 rows that hold `distinct` different ones, a few of them very often."""
    import torch
    g = torch.Generator().manual_seed(seed)
    table = (0.02 * torch.randn((distinct, D), generator=g)).bfloat16()
    ids = (distinct * torch.rand(N, generator=g) ** 3).long().clamp_(max=distinct - 1)
    ids[:distinct] = torch.randperm(distinct, generator=g)[:N]
    return table[ids[torch.randperm(N, generator=g)]].cuda()


def _spectral_run(X, m, n_it, r, bits, distinct, window=0, resident=1, normalise=0):
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    ctx = P.slh_create(X.shape[0], X.shape[1], m, r, bits, 0)
    if window:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, window)
    P.slh_set_option(ctx, B.SLH_OPT_DISTINCT, distinct)
    P.slh_set_option(ctx, B.SLH_OPT_RESIDENT, resident)
    P.slh_set_option(ctx, B.SLH_OPT_NORMALIZE, normalise)
    P.slh_feature_map(ctx, X)
    out = dict(rows=ctx.operator_rows, Phi=P.slh_copy_out(ctx, B.SLH_OUT_PHI))
    if normalise:
        out["rowsum"] = P.slh_copy_out(ctx, B.SLH_OUT_ROWSUM)
    out["ritz"], out["iters"] = P.slh_lanczos(ctx, n_it)
    out["energy"] = P.slh_spectral_energy(ctx)
    P.slh_simhash(ctx)
    for k in ("ALPHA", "Z", "PROJ", "Q", "CODES"):
        out[k] = P.slh_copy_out(ctx, getattr(B, "SLH_OUT_" + k))
    return out


@pytest.mark.parametrize("case", ["one", "one_streaming", "windows", "normalised", "ragged", "wide"])
def test_distinct_rows_match_every_row(case):
    """The operator on the distinct rows against the operator on every row
    (SLH_OPT_DISTINCT 0), the same in exact arithmetic: Phi bit for bit, the basis
    and Ritz coordinates of every token, row sums and energy.  Both sides run the
    same recurrence in fp64 with sums grouped differently, so alpha agrees to 1e-9
    (3e-11 measured, n_it far below the distinct rows), Ritz values and energy too, and
    Z and Q, whose rows are of size 1 at most, to 1e-8; a code bit may differ only
    where its projection is within 1e-7 of zero.  Normalised, the row sums differ by
    rounding, so a row's weight, and with it the fp32 rows of Phi, may differ by an ulp
    (6e-8): a thousand times wider."""
    N, D, m, distinct, window, n_it, kw = {
        "one": (4096, 512, 1024, 700, 0, 24, {}),
        "one_streaming": (4096, 512, 1024, 700, 0, 24, dict(resident=0)),
        "windows": (16 * 1111, 256, 512, 300, 1111, 24, {}),
        "normalised": (4096, 256, 1024, 900, 0, 16, dict(normalise=1)),
        "ragged": (8191, 264, 1024, 1001, 0, 24, {}),      # the last word of the bit map part full
        "wide": (2051, 2056, 2048, 1500, 0, 24, {}),      # D past one 2048-value stretch
    }[case]
    X = _repeating_rows(N, D, distinct, 3)
    if window:                                 # a different number of rows in each window
        X[:window // 2] = X[window // 2 - 1]
    a = _spectral_run(X, m, n_it, 12, 8, 1, window, **kw)
    b = _spectral_run(X, m, n_it, 12, 8, 0, window, **kw)
    L = window or N
    assert b["rows"] == L and a["rows"] <= distinct + 1 < L
    if not kw.get("normalise"):
        assert np.array_equal(a["Phi"], b["Phi"])
    else:
        assert np.abs(a["Phi"] - b["Phi"]).max() <= 2e-7 * np.abs(b["Phi"]).max()
        assert np.abs(a["rowsum"] / b["rowsum"] - 1).max() <= 1e-12
    assert np.array_equal(a["iters"], b["iters"])
    da = np.abs(a["ALPHA"] / b["ALPHA"] - 1).max()
    dr = np.abs(a["ritz"] / b["ritz"] - 1).max()
    dz, dq = np.abs(a["Z"] - b["Z"]).max(), np.abs(a["Q"][:, :n_it] - b["Q"][:, :n_it]).max()
    de = np.abs(a["energy"] / b["energy"] - 1).max()
    _say(f"[distinct rows] {case}: rows {a['rows']} of {L}, alpha {da:.1e} ritz {dr:.1e} Z {dz:.1e} Q {dq:.1e} energy {de:.1e}")
    lim = 1e-6 if kw.get("normalise") else 1e-9
    assert da <= lim and dr <= lim and dz <= 10 * lim and dq <= 10 * lim and de <= lim
    flip = (a["PROJ"] > 0) != (b["PROJ"] > 0)
    assert not flip.any() or np.abs(b["PROJ"][flip]).max() <= 100 * lim
    if not flip.any():
        assert np.array_equal(a["CODES"], b["CODES"])


@pytest.mark.parametrize("case", ["all_different", "alike_where_hashed", "fp32", "few", "other_stream"])
def test_distinct_rows_only_where_equal(case):
    """What is grouped: rows equal in every value.  Rows that agree only in the
    hashed stretches (the first 64 values and 64 from the middle), rows that all
    differ and fp32 rows are taken one by one; with fewer distinct rows than steps
    the run breaks down as it does on every row."""
    import torch
    N, D, m = 4096, 512, 1024
    X = _repeating_rows(N, D, 500, 4)
    n_it = 20
    if case == "all_different":
        X = (0.02 * torch.randn((N, D), generator=torch.Generator().manual_seed(1))).bfloat16().cuda()
    elif case == "alike_where_hashed":
        X[7, 200] += 1.0
    elif case == "fp32":
        X = X.float()
    elif case == "few":
        X = X[:3].repeat(N // 3 + 1, 1)[:N].contiguous()
    if case == "other_stream":
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            a = _spectral_run(X, m, n_it, 4, 8, 1)
        s.synchronize()
    else:
        a = _spectral_run(X, m, n_it, 4, 8, 1)
    b = _spectral_run(X, m, n_it, 4, 8, 0)
    if case in ("few", "other_stream"):
        assert a["rows"] == (4 if case == "few" else 501)
    else:
        assert a["rows"] == N
        assert all(np.array_equal(a[k], b[k]) for k in ("Phi", "Z", "CODES"))
    if case == "few":
        assert a["iters"][0] <= 6 and b["iters"][0] <= 6     # rank 3, and rounding past it
        assert abs(a["ritz"][0, -1] / b["ritz"][0, -1] - 1) <= 1e-9
    if case == "other_stream":
        assert np.abs(a["Z"] - b["Z"]).max() <= 1e-7


@pytest.mark.parametrize("N,distinct,taken", [
    (32768, 12288, True),      # the most groups: three quarters of the table's slots
    (32768, 12289, False),     # one more
    (131072, 131072, False),   # far more rows than slots
    (40000, 10000, True),
    (8192 * 4, 4 * 7167, False)])
def test_distinct_rows_up_to_the_table(N, distinct, taken):
    """The number of distinct rows alone decides whether they are grouped, the same on
    every call: up to 12288 in a window, however the table fills."""
    import torch
    import paper_2607_19368_amd as P
    D, m = 64, 256
    X = _repeating_rows(N, D, distinct, 6)
    assert len(torch.unique(X.view(torch.int16), dim=0)) == distinct
    ctx = P.slh_create(N, D, m, 4, 8, 0)
    for _ in range(4):
        P.slh_feature_map(ctx, X)
        assert ctx.operator_rows == (distinct + 1 if taken else N)
    if taken:
        a, b = (_spectral_run(X, m, 12, 4, 8, k) for k in (1, 0))
        assert np.array_equal(a["Phi"], b["Phi"])
        assert np.abs(a["ritz"] / b["ritz"] - 1).max() <= 1e-9


@pytest.mark.parametrize("N,window,distinct,taken", [(8192, 0, 7167, True), (8192, 0, 7168, False),
                                                     (64 * 1024, 64, 55, True), (64 * 1024, 64, 56, False)])
def test_distinct_rows_that_spare_an_eighth(N, window, distinct, taken):
    """Rows are grouped where groups + 1 is at most 7/8 of the window."""
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    D, m, L = 64, 1024, window or N
    X = _repeating_rows(L, D, distinct, 8).repeat(N // L, 1)
    ctx = P.slh_create(N, D, m, 4, 8, 0)
    if window:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, window)
    P.slh_feature_map(ctx, X)
    assert ctx.operator_rows == (distinct + 1 if taken else L)


@pytest.mark.parametrize("resident", [1, 0])
def test_capture_after_a_grouped_warm_up(resident):
    """Under stream capture every row is taken, also where the eager run before (which
    sized the workspaces) grouped them; every replay, on new rows in the same buffer
    and with eager runs in between, gives the bits of an eager run on every row."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    N, D, m, n_it = 4096, 512, 1024, 24
    Xs = [_repeating_rows(N, D, 700, k) for k in (11, 12, 13)]
    X = Xs[0].clone()
    codes = torch.zeros(N, dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()

    def ctx(distinct):
        c = P.slh_create(N, D, m, 12, 8, 0)
        P.slh_set_option(c, B.SLH_OPT_RESIDENT, resident)
        P.slh_set_option(c, B.SLH_OPT_DISTINCT, distinct)
        P.slh_set_stream(c, s)
        return c

    def run(c):
        P.slh_feature_map(c, X)
        P.slh_lanczos(c, n_it, want=False)
        P.slh_simhash(c, codes)

    torch.cuda.synchronize()
    a, every = ctx(1), ctx(0)
    run(a)
    assert a.operator_rows == 701
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        run(a)
    assert a.operator_rows == N
    for x in Xs + Xs[:1]:
        X.copy_(x)
        codes.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
        s.synchronize()
        got = codes.clone(), P.slh_copy_out(a, B.SLH_OUT_ALPHA), P.slh_copy_out(a, B.SLH_OUT_Z)
        run(every)
        s.synchronize()
        assert torch.equal(got[0], codes)
        assert np.array_equal(got[1], P.slh_copy_out(every, B.SLH_OUT_ALPHA))
        assert np.array_equal(got[2], P.slh_copy_out(every, B.SLH_OUT_Z))


# ------------------------------------------------------------------ merge of loaded codes
@pytest.mark.parametrize("N,bits,window,skew,compact", [
    (4096 * 5 + 1, 7, 0, 3.0, 0),          # one token in the last tile
    (16385, 16, 0, 1.0, 1),                # more codes than tokens, most buckets single
    (2 * 20001, 10, 20001, 3.0, 0),        # two long windows
    (20480, 1, 0, 1.0, 0),                 # two buckets over every tile
    (70000, 14, 0, 6.0, 0),                # a bucket of most tokens
    (3001, 6, 0, 2.0, 1), (8192, 12, 0, 3.0, 0), (512 * 6, 5, 512, 2.0, 0)])
def test_merge_bookkeeping(N, bits, window, skew, compact):
    """Macro indices, positions and sums of slh_merge on loaded codes (no feature
    map, so the norms come from the merge's own read of X) against the definition:
    one bucket per (window, code), ordered by last token; E = mean * (mean member
    norm) / |mean| in 64 bits, to 2e-6 (fp32 sums of up to 70000 rows of size 1:
    about 2^-24 sqrt(64) within a chunk and across the chunks of a bucket)."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    D = 40
    rng = np.random.default_rng(N)
    codes = np.minimum((1 << bits) * rng.random(N) ** skew, (1 << bits) - 1).astype(np.int64)
    X = (rng.standard_normal((N, D)) + 1.0).astype(np.float32)
    ctx = P.slh_create(N, D, 256, 4, bits, 0)
    if window:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, window)
    P.slh_set_option(ctx, B.SLH_OPT_POS_MODE, compact)
    P.slh_load(ctx, B.SLH_OUT_CODES, torch.from_numpy(codes.astype(np.int32)).cuda())
    E, pos, t2m, M = P.slh_merge(ctx, torch.from_numpy(X).cuda())
    key = np.arange(N) // (window or N) * (1 << 20) + codes
    _, inv = np.unique(key, return_inverse=True)
    last = np.zeros(inv.max() + 1, np.int64)
    np.maximum.at(last, inv, np.arange(N))
    order = np.argsort(last)
    rank = np.empty_like(order)
    rank[order] = np.arange(len(order))
    assert M == len(order)
    assert np.array_equal(t2m.cpu().numpy(), rank[inv])
    assert np.array_equal(pos.cpu().numpy()[:M], np.arange(M) if compact else last[order])
    S, cnt, eta = np.zeros((M, D)), np.zeros(M), np.zeros(M)
    np.add.at(S, rank[inv], X.astype(np.float64))
    np.add.at(cnt, rank[inv], 1.0)
    np.add.at(eta, rank[inv], np.linalg.norm(X.astype(np.float64), axis=1))
    ref = S * (eta / cnt / np.linalg.norm(S, axis=1))[:, None]
    err = np.linalg.norm(E.cpu().numpy()[:M] - ref, axis=1) / np.linalg.norm(ref, axis=1)
    _say(f"[merge book] N={N} bits={bits} window={window}: M={M} max rel {err.max():.1e}")
    assert err.max() <= 2e-6


@pytest.mark.parametrize("D,dtype", [(2056, "fp32"), (4104, "fp32"), (8200, "fp32"), (16392, "fp32"),
                                     (4104, "bf16"), (8200, "bf16"), (16392, "bf16")])
def test_merge_sums_of_wide_rows(D, dtype):
    """Sums of 51 rows a bucket in a window long enough for the longest chunks, at the
    widths where a thread's share of a row and the batches change: no less accurate
    than chunks of 16 rows summed one by one.  The sum of k rows of mean 1 is about k,
    so each of its roundings has a standard deviation of about 2^-24 k / sqrt(3), and a
    bucket of n rows an error of 2^-24 / (n sqrt(3)) times the root of the sum of k^2
    over its roundings: for n = 51 6.9e-8 with chunks of 16 (k = 2 .. 16 in each, then
    the chunks' sums), 6.6e-8 with sums of eight rows in a chunk of 64, but 1.1e-7 with
    sums of two and 1.4e-7 row by row."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    N, bits = 24600, 9
    g = torch.Generator(device="cuda")
    g.manual_seed(D)
    X = torch.randn((N, D), generator=g, device="cuda") + 1.0
    if dtype == "bf16":
        X = X.bfloat16()
    codes = torch.randint(0, 1 << bits, (N,), generator=g, device="cuda")
    ctx = P.slh_create(N, D, 256, 4, bits, 0)
    P.slh_load(ctx, B.SLH_OUT_CODES, codes.int())
    E, _, t2m, M = P.slh_merge(ctx, X)
    S = torch.zeros((M, D), dtype=torch.float64, device="cuda")
    eta = torch.zeros(M, dtype=torch.float64, device="cuda")
    at = t2m.long()
    for i in range(0, N, 2048):
        x = X[i:i + 2048].double()
        S.index_add_(0, at[i:i + 2048], x)
        eta.index_add_(0, at[i:i + 2048], x.norm(dim=1))
    ref = S * (eta / torch.bincount(at, minlength=M) / S.norm(dim=1))[:, None]
    err = float((E[:M].double() - ref).norm() / ref.norm())
    _say(f"[merge wide] {dtype} D={D}: {err:.2e}")
    assert err <= 6.9e-8


@pytest.mark.parametrize("N,bits,window", [(9001, 12, 0), (20001, 10, 0), (3 * 8200, 9, 8200)])
def test_merge_of_codes_past_the_tables(N, bits, window):
    """slh_load takes codes as they are given: values of 2^bits and more (here of 16
    bits, and the 0xFFFFFFFF that slh_simhash writes for tokens it does not hash) in
    windows long enough for the tiled book-keeping, whose tables hold 2^bits codes.
    They are grouped by the whole code as in a short window; of several windows, one
    holds none.  Sums as in test_merge_bookkeeping."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    D, L = 16, window or N
    rng = np.random.default_rng(N)
    values = np.concatenate([rng.permutation(0xFFFF)[:150], [0xFFFFFFFF]])
    codes = values[rng.integers(0, len(values), N)]
    assert (codes >= 1 << bits).any()
    if window:
        codes[:L] = rng.integers(0, 100, L)
    X = (rng.standard_normal((N, D)) + 1.0).astype(np.float32)
    ctx = P.slh_create(N, D, 256, 4, bits, 0)
    if window:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, window)
    P.slh_load(ctx, B.SLH_OUT_CODES, torch.from_numpy(codes.astype(np.uint32).view(np.int32)).cuda())
    E, pos, t2m, M = P.slh_merge(ctx, torch.from_numpy(X).cuda())
    _, inv = np.unique(np.arange(N) // L * (1 << 33) + codes, return_inverse=True)
    last = np.zeros(inv.max() + 1, np.int64)
    np.maximum.at(last, inv, np.arange(N))
    order = np.argsort(last)
    rank = np.empty_like(order)
    rank[order] = np.arange(len(order))
    assert M == len(order)
    assert np.array_equal(t2m.cpu().numpy(), rank[inv])
    assert np.array_equal(pos.cpu().numpy()[:M], last[order])
    S, cnt, eta = np.zeros((M, D)), np.zeros(M), np.zeros(M)
    np.add.at(S, rank[inv], X.astype(np.float64))
    np.add.at(cnt, rank[inv], 1.0)
    np.add.at(eta, rank[inv], np.linalg.norm(X.astype(np.float64), axis=1))
    ref = S * (eta / cnt / np.linalg.norm(S, axis=1))[:, None]
    err = np.linalg.norm(E.cpu().numpy()[:M] - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 2e-6


@pytest.mark.timeout(900)
def test_end_to_end_qwen14b_long():
    inp = make_inputs("qwen14b_long")
    wl = inp.workload
    _say(f"[e2e] qwen14b_long N={wl.N} D={wl.D} m={wl.m}")
    g = PR.run_gpu(inp, n_it=wl.n_it)
    o = PR.run_oracle(inp, n_it=wl.n_it)
    rep = PR.compare(o, g, wl.N)
    _say(f"   {rep}  M={len(g.P)}")


@pytest.mark.timeout(900)
def test_end_to_end_adaptive64():
    """64 windows: scores (Eq. 8), routing at the midpoint of the 32nd/33rd scores,
    chunk pooling for chunk windows, batched spectral path for the others."""
    inp = make_inputs("adaptive64")
    wl = inp.workload
    L = wl.window
    Xs = [inp.x_float(slice(w * L, (w + 1) * L)) for w in range(wl.N // L)]
    so = np.array([O.redundancy_score(x) for x in Xs])
    srt = np.sort(so)[::-1]
    tau = 0.5 * (srt[31] + srt[32])
    _say(f"[e2e] adaptive64 tau={tau:.5f} literal tau(8)={O.tau_of_rho(8):.2f}")
    g = PR.run_gpu(inp, n_it=wl.n_it, window=L, rho=wl.rho, tau=tau)
    assert np.max(np.abs(g.scores - so)) < 1e-9
    o = PR.run_oracle(inp, n_it=wl.n_it, window=L, rho=wl.rho, tau=tau)
    assert np.array_equal(g.route, o.route)
    assert int(g.route.sum()) == 32
    # small-period windows: a dense cluster of ~100 eigenvalues under one outlier
    # makes the last Ritz vectors depend on fp64 summation order (the oracle
    # disagrees with itself under token reversal); those bits are not compared
    unc = {w.w: PR.oracle_uncertainty(inp, w.w, L, wl.n_it) for w in o.windows}
    _say("   oracle self-uncertainty per window: " +
         " ".join(f"{w}:{u:.1e}" for w, u in sorted(unc.items())))
    rep = PR.compare(o, g, L, unc=unc)
    _say(f"   {rep}  M={len(g.P)}")


def test_adaptive_literal_threshold_routes_all_to_chunk():
    inp = _custom("adp_small", 8 * 256, 256, 256, 16, 8, 6)
    wl = inp.workload
    g = PR.run_gpu(inp, n_it=16, window=256, rho=8.0)
    o = PR.run_oracle(inp, n_it=16, window=256, rho=8.0)
    assert np.array_equal(g.route, o.route) and g.route.sum() == 0
    PR.compare(o, g, 256)


@pytest.mark.parametrize("case", ["bf16_fused", "f32_fused", "bf16_wide", "bf16_partial", "bf16_odd"])
def test_router_scores_both_paths(case):
    """Eq. 8 scores and routes against the oracle on both implementations: the
    fused row-norm + score kernels (D <= 4096; bf16 X streamed through LDS, fp32
    X through registers) and the separate row-norm and score kernels (D > 4096);
    scores within 1e-9, routes equal, and the compressed output compared as
    everywhere else.  bf16_partial: rows narrower than the workgroup's columns
    (D = 3584 of 4096) and windows of 300 rows (a 256-row group and a 44-row
    one); bf16_odd: D = 1032 of 2048 and windows of 131 rows (a last batch of
    one row)."""
    D = {"bf16_fused": 512, "f32_fused": 512, "bf16_wide": 4104, "bf16_partial": 3584,
         "bf16_odd": 1032}[case]
    x = "f32" if case == "f32_fused" else "bf16"
    L = {"bf16_partial": 300, "bf16_odd": 131}.get(case, 128)
    nw = 6
    inp = _custom(f"rt_{case}", nw * L, D, 256, 16, 8, 6, x=x)
    Xs = [inp.x_float(slice(w * L, (w + 1) * L)) for w in range(nw)]
    so = np.array([O.redundancy_score(xw) for xw in Xs])
    srt = np.sort(so)[::-1]
    tau = 0.5 * (srt[2] + srt[3])
    _say(f"[router] {case} D={D} scores {np.round(so, 4)} tau={tau:.5f}")
    g = PR.run_gpu(inp, n_it=16, window=L, rho=4.0, tau=tau)
    assert np.max(np.abs(g.scores - so)) < 1e-9
    o = PR.run_oracle(inp, n_it=16, window=L, rho=4.0, tau=tau)
    assert np.array_equal(g.route, o.route) and int(g.route.sum()) == 3
    PR.compare(o, g, L)


# ------------------------------------------------------------------ edge cases
@pytest.mark.parametrize("m", [256, 1024])
def test_identical_rows_break_down(m):
    """Identical rows: Phi Phi^T = |phi|^2 11^T has rank one, so Lanczos breaks
    down after two steps on both sides; the leading Ritz columns are zero.  At
    m = 1024 the run takes the resident kernel, whose blocks all leave the loop
    at the same step."""
    base = make_inputs("tiny")
    X = np.tile(base.X[:1], (256, 1))
    wl = Workload("ident", 256, 256, m, 16, 8, 6, 4.0, 0, 0, "f32")
    inp = Inputs(wl, X, np.zeros(256))
    g = PR.run_gpu(inp, n_it=16)
    o = PR.run_oracle(inp, n_it=16)
    gw, ow = g.windows[0], o.windows[0]
    _say(f"[breakdown] iters gpu={gw.iters} oracle={ow.iters}")
    assert gw.iters == ow.iters == 2
    assert np.all(gw.Z[:, :6] == 0) and np.all(gw.ritz[:6] == 0)
    # the GPU Phi differs from the oracle's by ~1e-7 relative (fp32 GEMM and epilogue)
    assert abs(gw.ritz[-1] - ow.ritz[-1]) < 1e-5 * ow.ritz[-1]
    assert abs(gw.ritz[-2]) < 1e-9 * ow.ritz[-1]
    PR.compare(o, g, 256, check_spectral=False)


@pytest.mark.parametrize("short", [1, 0])
def test_smallest_problem(short):
    wl = Workload("min", 2, 8, 256, 2, 1, 1, 2.0, 0, 0, "f32")
    X = np.array([[1, 0, 0, 0, 0, 0, 0, 0], [0, 0.5, 0, 0, 0, 0, 0, 0]], np.float32)
    inp = Inputs(wl, X, np.zeros(2))
    g = PR.run_gpu(inp, n_it=2, short_windows=short)
    o = PR.run_oracle(inp, n_it=2)
    PR.compare(o, g, 2, ritz_rel=1e-6)


@pytest.mark.parametrize("bits,r,n_it", [(16, 128, 160), (1, 1, 1)])
def test_limits(bits, r, n_it):
    inp = _custom("limits", 2048, 256, 256, n_it, r, bits)
    g = PR.run_gpu(inp, n_it=n_it)
    o = PR.run_oracle(inp, n_it=n_it)
    rep = PR.compare(o, g, 2048)
    _say(f"[limits] bits={bits} r={r} n_it={n_it}: {rep}")


def test_compact_positions_and_determinism():
    inp = make_inputs("tiny")
    wl = inp.workload
    g1 = PR.run_gpu(inp, n_it=wl.n_it, compact=True)
    g2 = PR.run_gpu(inp, n_it=wl.n_it, compact=True)
    assert np.array_equal(g1.P, np.arange(len(g1.P)))
    assert np.array_equal(g1.E, g2.E) and np.array_equal(g1.t2m, g2.t2m)
    for a, b in zip(g1.windows, g2.windows):
        assert np.array_equal(a.Z, b.Z) and np.array_equal(a.codes, b.codes)
        assert np.array_equal(a.alpha, b.alpha)



def test_timing_mode_matches_graph_mode_qwen7b():
    """The benchmark's timing mode (each Lanczos pass launched directly between
    events) and the production graph give the same bits at the full qwen7b size."""
    inp = make_inputs("qwen7b")
    wl = inp.workload
    _say("timing vs graph mode: qwen7b", wl.N, wl.D, wl.m, wl.n_it)
    g1 = PR.run_gpu(inp, n_it=wl.n_it)
    g2 = PR.run_gpu(inp, n_it=wl.n_it, timing=True)
    assert np.array_equal(g1.E, g2.E) and np.array_equal(g1.t2m, g2.t2m)
    for a, b in zip(g1.windows, g2.windows):
        assert np.array_equal(a.alpha, b.alpha) and np.array_equal(a.beta, b.beta)
        assert np.array_equal(a.Z, b.Z) and np.array_equal(a.codes, b.codes)

@pytest.mark.parametrize("routed", [False, True])
def test_two_prompts_one_context_same_buffer(routed):
    """A second prompt written into the device buffer of the first and run
    through the same context gives, bit for bit, what a fresh context and a
    fresh buffer give it: the row norms behind s(x) (Eq. 3) and the member
    norms of Eq. 7 are taken from the new prompt, not reused by address.
    Prompt B's rows are twice those of another Zipf prompt (exact in bf16), so
    every norm differs.  routed: 4 windows of 256 through slh_route first
    (whose row norms feed the feature map of the same pass)."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    from workloads import f32_to_bf16_bits
    L = 256
    ia = _custom("pa", 4 * L, 512, 256, 16, 8, 8, seed=0)
    ib = _custom("pb", 4 * L, 512, 256, 16, 8, 8, seed=1)
    xb = Inputs(ib.workload, f32_to_bf16_bits(2.0 * ib.x_float()), ib.ids)
    wl = ia.workload

    def run(ctx, Xd):
        if routed:
            P.slh_route(ctx, Xd, 8.0, 0.25)
        P.slh_feature_map(ctx, Xd)
        P.slh_lanczos(ctx, wl.n_it, want=False)
        P.slh_simhash(ctx)
        E, Pp, t2m, M = P.slh_merge(ctx, Xd)
        torch.cuda.synchronize()
        return (E.cpu().numpy().copy(), Pp.cpu().numpy().copy(), t2m.cpu().numpy().copy(),
                P.slh_copy_out(ctx, B.SLH_OUT_CODES), P.slh_copy_out(ctx, B.SLH_OUT_Z))

    def fresh(inp):
        ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
        if routed:
            P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
        return ctx

    ctx = fresh(ia)
    buf = PR.to_device_x(ia)
    out_a = run(ctx, buf)
    buf.copy_(PR.to_device_x(xb))
    out_b = run(ctx, buf)
    ref_b = run(fresh(xb), PR.to_device_x(xb))
    ref_a = run(fresh(ia), PR.to_device_x(ia))
    _say(f"[two prompts] routed={routed} M_a={len(out_a[1])} M_b={len(out_b[1])}")
    for u, v in zip(out_b, ref_b):
        assert u.shape == v.shape and np.array_equal(u, v)
    for u, v in zip(out_a, ref_a):
        assert u.shape == v.shape and np.array_equal(u, v)
    assert not np.array_equal(out_a[0][:4], out_b[0][:4])


@pytest.mark.parametrize("m", [256, 1024])
def test_merge_async_pipelined(m):
    """slh_merge_async / slh_merge_wait: two prompts through one context with the
    second prompt's steps enqueued before the first one's M is read give, bit for
    bit, the outputs and M of slh_merge on each in a context of its own.  A third
    merge (or a slh_merge) is refused while two are outstanding, a wait needs
    an outstanding merge, and outputs of the wrong place, type or shape are
    refused by the binding.  m = 1024: the resident Lanczos kernel, whose error word
    each wait checks; m = 256: the streaming path."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    ia = _custom("qa", 2048, 512, m, 16, 8, 8, seed=0)
    ib = _custom("qb", 2048, 512, m, 16, 8, 8, seed=1)
    wl = ia.workload

    def steps(ctx, X):
        P.slh_feature_map(ctx, X)
        P.slh_lanczos(ctx, wl.n_it, want=False)
        P.slh_simhash(ctx)

    def sync_run(inp):
        ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
        X = PR.to_device_x(inp)
        steps(ctx, X)
        E, Pp, t2m, M = P.slh_merge(ctx, X)
        torch.cuda.synchronize()
        return E.cpu().numpy().copy(), Pp.cpu().numpy().copy(), t2m.cpu().numpy().copy(), M

    ref = [sync_run(ia), sync_run(ib)]
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    xs = [PR.to_device_x(ia), PR.to_device_x(ib)]
    cap = P.slh_merge_capacity(ctx)
    outs = [(torch.empty((cap, wl.D), dtype=torch.float32, device="cuda"),
             torch.empty(cap, dtype=torch.int32, device="cuda"),
             torch.empty(wl.N, dtype=torch.int32, device="cuda")) for _ in range(2)]
    _say(f"[merge async] m={m} cap={cap}")
    for i, (X, o) in enumerate(zip(xs, outs)):
        steps(ctx, X)
        if i == 0:
            # outputs the library could not write through are refused before any call:
            # a host tensor, a wrong dtype, a wrong width, pos_out shorter than emb_out
            for bad in ((o[0].cpu(), o[1], o[2]), (o[0], o[1].to(torch.int64), o[2]),
                        (o[0][:, :-1], o[1], o[2]), (o[0], o[1][:-1], o[2])):
                with pytest.raises(B.SLHError):
                    P.slh_merge_async(ctx, X, *bad)
        P.slh_merge_async(ctx, X, *o)
    assert len(ctx.in_flight) == 2            # X and the outputs stay referenced
    steps(ctx, xs[0])
    with pytest.raises(B.SLHError):
        P.slh_merge_async(ctx, xs[0], *outs[0])
    with pytest.raises(B.SLHError):
        P.slh_merge(ctx, xs[0])
    Ms = [P.slh_merge_wait(ctx), P.slh_merge_wait(ctx)]
    assert len(ctx.in_flight) == 0
    with pytest.raises(B.SLHError):
        P.slh_merge_wait(ctx)
    torch.cuda.synchronize()
    for (E, Pp, t2m), M, (rE, rP, rt, rM) in zip(outs, Ms, ref):
        assert M == rM
        assert np.array_equal(E[:M].cpu().numpy(), rE)
        assert np.array_equal(Pp[:M].cpu().numpy(), rP)
        assert np.array_equal(t2m.cpu().numpy(), rt)
    assert Ms[0] != Ms[1] or not np.array_equal(ref[0][0], ref[1][0])


def test_resident_wait_timeout_reported():
    """A wait of the resident Lanczos kernel that gives up is reported, not hung:
    with SLH_OPT_WAIT_POLLS = 1 a wait for another block's value gives up after
    two polls, and the run leaves through the error path with slh_merge raising
    SLH_EHIP (timed out).  Whether some wait of a run needs more polls depends on
    the blocks' timing, so each of up to eight runs must either raise that error or, where no wait gave up,
    match a fresh context bit for bit; back at the default the same context runs
    the prompt again and matches the fresh context bit for bit."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    # the 512-thread kernel (m = 2048, 256 blocks of 32 rows), whose blocks wait
    # several microseconds for the column partials of each step
    inp = _custom("wt", 8192, 512, 2048, 16, 8, 8, seed=5)
    wl = inp.workload
    X = PR.to_device_x(inp)

    def run(ctx):
        P.slh_feature_map(ctx, X)
        P.slh_lanczos(ctx, wl.n_it, want=False)
        P.slh_simhash(ctx)
        E, Pp, t2m, M = P.slh_merge(ctx, X)
        torch.cuda.synchronize()
        return E.cpu().numpy().copy(), Pp.cpu().numpy().copy(), t2m.cpu().numpy().copy()

    def same(a, b):
        return all(u.shape == v.shape and np.array_equal(u, v) for u, v in zip(a, b))

    ref = run(P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0))
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    P.slh_set_option(ctx, B.SLH_OPT_WAIT_POLLS, 1)
    timed_out = 0
    for k in range(8):
        _say(f"[wait timeout] resident run {k} with one poll per wait")
        try:
            out = run(ctx)
        except B.SLHError as e:
            assert "timed out" in str(e)
            timed_out += 1
            break
        assert same(out, ref)
    P.slh_set_option(ctx, B.SLH_OPT_WAIT_POLLS, 0)
    assert same(run(ctx), ref)
    with pytest.raises(B.SLHError):
        P.slh_set_option(ctx, B.SLH_OPT_WAIT_POLLS, -1)
    if not timed_out:
        pytest.skip("no wait needed more than two polls in eight runs on this device")


def test_call_order_and_capacity_errors():
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    inp = make_inputs("tiny")
    wl = inp.workload
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    with pytest.raises(B.SLHError, match=r"\(-4\)"):
        P.slh_lanczos(ctx, wl.n_it)
    Xd = PR.to_device_x(inp)
    P.slh_feature_map(ctx, Xd)
    with pytest.raises(B.SLHError, match=r"\(-1\)"):
        P.slh_lanczos(ctx, wl.r - 1)
    with pytest.raises(B.SLHError, match=r"\(-4\)"):
        P.slh_merge(ctx, Xd)
    P.slh_lanczos(ctx, wl.n_it)
    P.slh_simhash(ctx)
    small = torch.empty((4, wl.D), dtype=torch.float32, device="cuda")
    with pytest.raises(B.SLHError, match=r"\(-1\)"):
        P.slh_merge(ctx, Xd, emb_out=small)
    with pytest.raises(B.SLHError, match=r"\(-1\)"):
        P.slh_feature_map(ctx, Xd[:, 1:])     # misaligned rows


def test_strided_rows():
    """X given as a view with row stride D + 24 (padded rows): same results as the
    contiguous layout, and parity with the oracle."""
    import torch
    inp = _custom("strided", 1024, 512, 256, 24, 8, 8)
    wl = inp.workload
    Xc = PR.to_device_x(inp)
    pad = torch.zeros((wl.N, wl.D + 24), dtype=Xc.dtype, device=Xc.device)
    pad[:, :wl.D] = Xc
    Xs = pad[:, :wl.D]
    assert Xs.stride(0) == wl.D + 24
    gs = PR.run_gpu(inp, n_it=wl.n_it, X=Xs)
    gc = PR.run_gpu(inp, n_it=wl.n_it, X=Xc)
    assert np.array_equal(gs.E, gc.E) and np.array_equal(gs.t2m, gc.t2m)
    o = PR.run_oracle(inp, n_it=wl.n_it)
    rep = PR.compare(o, gs, wl.N)
    _say(f"[strided] {rep}")


def test_windows_with_and_without_breakdown():
    """Four windows in one batch: windows 0 and 2 hold a single repeated row
    (rank-one operator: Lanczos stops after two steps), windows 1 and 3 are
    Zipf embeddings (no breakdown).  Each window must stop, hash and merge on
    its own, as in the oracle."""
    L = 256
    base = _custom("mixwin", 4 * L, 256, 256, 20, 6, 6)
    X = base.X.copy()
    X[0:L] = X[0]
    X[2 * L:3 * L] = X[2 * L + 5]
    inp = Inputs(base.workload, X, base.ids)
    g = PR.run_gpu(inp, n_it=20, window=L)
    o = PR.run_oracle(inp, n_it=20, window=L)
    iters_g = [w.iters for w in g.windows]
    iters_o = [w.iters for w in o.windows]
    _say(f"[mixed windows] iters gpu={iters_g} oracle={iters_o}")
    assert iters_g == iters_o and iters_g[0] == iters_g[2] == 2 and iters_g[1] == iters_g[3] == 20
    for w in (1, 3):
        gw, ow = g.windows[w], o.windows[w]
        rel = np.abs(gw.ritz - ow.ritz) / np.abs(ow.ritz)
        assert rel.max() <= PR.RITZ_REL
        assert PR.subspace_angle(ow.Z, gw.Z) < PR.ANGLE
    for w in (0, 2):
        gw, ow = g.windows[w], o.windows[w]
        assert np.all(gw.Z[:, :4] == 0) and np.all(gw.ritz[:4] == 0)
        assert abs(gw.ritz[-1] - ow.ritz[-1]) < 1e-5 * ow.ritz[-1]
    PR.compare(o, g, L, check_spectral=False)


@pytest.mark.timeout(900)
def test_end_to_end_local16():
    """Local backend at the paper's defaults: windows of 16 tokens, m = 256, a
    full 16-step Krylov space per window, on all 512 windows (and the 12 kept
    tokens) of the benchmark's prompt.  A window
    holding repeated tokens has a rank-deficient operator; with r = 16 all of its
    Ritz vectors are kept, including a basis of the null space inside the Krylov
    space, which the method leaves arbitrary when it is 2-dimensional or more.
    Such windows' SimHash bits are not determined, and the oracle's own
    reversed-order evaluation (parity.oracle_uncertainty) marks them."""
    inp = make_inputs("local16")
    wl = inp.workload
    _say(f"[e2e] local16 N={wl.N} window={wl.window} n_it={wl.n_it} r={wl.r} bits={wl.bits}")
    g = PR.run_gpu(inp, n_it=wl.n_it, window=wl.window)
    o = PR.run_oracle(inp, n_it=wl.n_it, window=wl.window)
    iters = sorted({w.iters for w in o.windows})
    unc = {w.w: PR.oracle_uncertainty(inp, w.w, wl.window, wl.n_it) for w in o.windows}
    determined = sum(u < PR.EXCL for u in unc.values())
    _say(f"   oracle steps per window: {iters}; windows with determined bits: {determined}/{len(unc)}")
    assert determined >= len(unc) // 2
    rep = PR.compare(o, g, wl.window, unc=unc)
    _say(f"   {rep}  M={len(g.P)}")
    assert rep.undecided_windows <= len(unc) // 4


@pytest.mark.parametrize("L,n_it,r,bits", [(16, 16, 16, 2), (12, 12, 8, 3), (32, 32, 16, 4),
                                           (24, 20, 8, 4)])
def test_short_windows(L, n_it, r, bits):
    """Windows of L <= 32 tokens run in one wavefront per window on the explicit
    L x L operator (SLH_OPT_SHORT_WINDOWS, on by default).  In a batch of 64
    windows, window 1 repeats one token (rank one: breakdown after two steps)
    and window 2 alternates two tokens (rank two: breakdown after three steps,
    an odd-sized tridiagonal); the rest are Zipf embeddings.  Both the short
    path and the general path must match the oracle."""
    N = 64 * L
    base = _custom("short", N, 512, 256, n_it, r, bits)
    X = base.X.copy()
    X[L:2 * L] = X[L]
    X[2 * L:3 * L:2] = X[2 * L]
    X[2 * L + 1:3 * L:2] = X[2 * L + 1]
    inp = Inputs(base.workload, X, base.ids)
    _say(f"[short windows] L={L} n_it={n_it} r={r} bits={bits} windows={N // L}")
    o = PR.run_oracle(inp, n_it=n_it, window=L)
    unc = {w.w: PR.oracle_uncertainty(inp, w.w, L, n_it) for w in o.windows}
    for short in (1, 0):
        g = PR.run_gpu(inp, n_it=n_it, window=L, short_windows=short)
        assert [w.iters for w in g.windows[1:3]] == [w.iters for w in o.windows[1:3]] == [2, 3]
        assert np.all(g.windows[1].Z[:, :r - 2] == 0) and np.all(g.windows[2].Z[:, :r - 3] == 0)
        rep = PR.compare(o, g, L, unc=unc)
        _say(f"   short={short}: {rep}  M={len(g.P)}")
        assert rep.undecided_windows <= len(unc) // 4


@pytest.mark.parametrize("case", ["tiny", "mistral7b", "local16", "windows256"])
def test_normalised_operator(case):
    """SLH_OPT_NORMALIZE: per window, the rows of Phi are scaled by s_i^-1/2 with
    s = Phi (Phi^T 1) before Lanczos (the symmetric form of the normalised
    matvec).  The estimated row sums and the whole path must match the oracle;
    the short-window kernel (local16) and the general windowed path
    (windows256) both run on the scaled rows."""
    if case == "local16":
        inp, L = make_inputs("local16", N=1036), 16
    elif case == "windows256":
        inp, L = _custom("nwin", 4 * 256, 512, 256, 24, 8, 8), 256
    else:
        inp, L = make_inputs(case), 0
    wl = inp.workload
    n_it = wl.n_it
    _say(f"[normalised] {case} N={wl.N} D={wl.D} m={wl.m} window={L} n_it={n_it}")
    g = PR.run_gpu(inp, n_it=n_it, window=L, normalise=True)
    o = PR.run_oracle(inp, n_it=n_it, window=L, normalise=True)
    rel = np.abs(g.rowsum - o.rowsum) / np.abs(o.rowsum)
    _say(f"   row sums: max rel {rel.max():.2e}")
    assert rel.max() < 1e-5
    unc = None
    if L:
        unc = {w.w: PR.oracle_uncertainty(inp, w.w, L, n_it, normalise=True) for w in o.windows}
    rep = PR.compare(o, g, L or wl.N, unc=unc)
    _say(f"   {rep}  M={len(g.P)}")
    if unc is not None:
        assert rep.undecided_windows <= len(unc) // 4


@pytest.mark.parametrize("case", ["tiny", "windows256", "local16_normalised"])
def test_spectral_energy(case):
    """slh_spectral_energy: per spectral window, sum of the kept Ritz values over
    ||Phi_w||_F^2, against the oracle's value on the same inputs (the GPU's fp32
    Phi and fp64 sums: within 1e-6 relative)."""
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    norm = False
    if case == "tiny":
        inp, L = make_inputs("tiny"), 0
    elif case == "windows256":
        inp, L = _custom("ewin", 4 * 256, 512, 256, 24, 8, 8), 256
    else:
        inp, L, norm = make_inputs("local16", N=524), 16, True
    wl = inp.workload
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    if wl.keep_last:
        P.slh_set_option(ctx, B.SLH_OPT_KEEP_LAST, wl.keep_last)
    if L:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
    if norm:
        P.slh_set_option(ctx, B.SLH_OPT_NORMALIZE, 1)
    Xd = PR.to_device_x(inp)
    P.slh_feature_map(ctx, Xd)
    ritz, iters = P.slh_lanczos(ctx, wl.n_it, want=True)
    e = P.slh_spectral_energy(ctx)
    Lw = L or wl.N
    W, psi = OP.projection(0, wl.D, wl.m), OP.phases(0, wl.m)
    eo = []
    for w in range((wl.N - wl.keep_last) // Lw):
        Phi = O.feature_map(inp.x_float(slice(w * Lw, (w + 1) * Lw)), W, psi)
        if norm:
            Phi, _ = O.normalised_features(Phi)
        vals, _, _, _ = O.ritz(O.lanczos(Phi, OP.start_vector(0, Lw, w), wl.n_it), wl.r)
        eo.append(O.spectral_energy(vals, Phi))
    eo = np.array(eo)
    rel = np.abs(e - eo) / eo
    _say(f"[energy] {case}: gpu {e[:4]} oracle {eo[:4]} max rel {rel.max():.2e}")
    assert np.all((e > 0) & (e <= 1.0 + 1e-12)) and rel.max() < 1e-6


@pytest.mark.parametrize("scheme", ["median", "mean"])
@pytest.mark.parametrize("case", ["tiny", "windows", "long"])
def test_position_schemes(scheme, case):
    """SLH_OPT_POS_SCHEME (section 3.4): the oracle's codes are loaded and the
    GPU merge must give the same members, positions and order as the oracle's
    merge under the median / mean scheme, bit for bit (embeddings 1e-5).
    windows: 8 windows of 256 tokens, half routed to chunk pooling (whose groups
    take the same scheme); long: one window of 20000 tokens (the global-memory
    book-keeping path) with a Zipf-like code distribution."""
    sid = {"median": 1, "mean": 2}[scheme]
    rho = None
    if case == "tiny":
        inp, L = make_inputs("tiny"), 0
        codes = np.random.default_rng(1).integers(0, 64, inp.workload.N)
    elif case == "windows":
        inp, L, rho = _custom("pwin", 8 * 256, 256, 256, 16, 8, 8), 256, 8.0
        codes = np.random.default_rng(2).integers(0, 256, inp.workload.N)
    else:
        inp, L = _custom("plong", 20000, 64, 256, 8, 4, 12), 0
        rng = np.random.default_rng(3)
        codes = np.minimum(rng.zipf(1.3, inp.workload.N) - 1, 4095)
    wl = inp.workload
    Lw = L or wl.N
    tau = -1.0
    route = np.ones(wl.N // Lw, bool)
    if rho is not None:
        sc = np.array([O.redundancy_score(inp.x_float(slice(w * Lw, (w + 1) * Lw)))
                       for w in range(wl.N // Lw)])
        tau = float(np.median(sc))
        route = np.array([O.route_window(Lw, v, rho, tau) for v in sc])
    _say(f"[positions] {scheme} {case} N={wl.N} window={L} spectral windows={int(route.sum())}")
    g = PR.run_gpu(inp, n_it=wl.r, window=L, rho=rho, tau=tau, codes_from=codes.astype(np.uint32),
                   scheme=sid)
    Es, Ps, t2m, base = [], [], np.zeros(wl.N, np.int64), 0
    for w in range(wl.N // Lw):
        Xw = inp.x_float(slice(w * Lw, (w + 1) * Lw))
        if route[w]:
            mg = O.merge(Xw, codes[w * Lw:(w + 1) * Lw], positions=w * Lw + np.arange(Lw),
                         scheme=scheme)
            E, P, tm = mg.E, mg.P, mg.tok2macro
        else:
            k = O.chunk_size(rho)
            E, P = O.chunk_pool(Xw, k, pos0=w * Lw, scheme=scheme)
            tm = np.arange(Lw) // k
        Es.append(E)
        Ps.append(P)
        t2m[w * Lw:(w + 1) * Lw] = base + tm
        base += len(P)
    E, P = np.concatenate(Es), np.concatenate(Ps)
    assert np.array_equal(g.P, P)
    assert np.array_equal(g.t2m, t2m)
    rel = np.linalg.norm(g.E - E, axis=1) / np.maximum(np.linalg.norm(E, axis=1), 1e-30)
    _say(f"   M={len(P)} max emb rel {rel.max():.2e}; ties in P: {int(np.sum(np.diff(P) == 0))}")
    assert rel.max() <= 1e-5


def test_position_scheme_end_to_end():
    """The whole path on the tiny mixture under the median scheme."""
    inp = make_inputs("tiny")
    wl = inp.workload
    g = PR.run_gpu(inp, n_it=wl.n_it, scheme=1)
    o = PR.run_oracle(inp, n_it=wl.n_it, scheme="median")
    rep = PR.compare(o, g, wl.N, scheme="median")
    _say(f"[positions e2e] {rep}")


@pytest.mark.parametrize("case", ["tiny", "qwen7b", "windows"])
def test_bucket_purity(case):
    """slh_bucket_purity: same-bucket token pairs with cosine > 0.7 (bit-exact
    counts against the oracle on the same codes; pairs whose fp64 cosine lies
    within 1e-12 of the threshold may differ and are counted).  qwen7b: codes
    = token id mod 4096 (identical tokens share buckets: the largest bucket
    holds ~1100 pairs of identical rows); windows: 8 windows of 256, half
    routed to chunk pooling (excluded: no LSH buckets)."""
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    rho, L = None, 0
    if case == "tiny":
        inp = make_inputs("tiny")
        codes = np.random.default_rng(1).integers(0, 16, inp.workload.N)
    elif case == "qwen7b":
        inp = make_inputs("qwen7b")
        codes = inp.ids % 4096
    else:
        inp, L, rho = _custom("purw", 8 * 256, 256, 256, 16, 8, 8), 256, 8.0
        codes = np.random.default_rng(2).integers(0, 8, inp.workload.N)
    wl = inp.workload
    Lw = L or wl.N
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    if L:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
    Xd = PR.to_device_x(inp)
    route = np.ones(wl.N // Lw, bool)
    if rho is not None:
        sc = np.array([O.redundancy_score(inp.x_float(slice(w * Lw, (w + 1) * Lw)))
                       for w in range(wl.N // Lw)])
        tau = float(np.median(sc))
        r_gpu, _ = P.slh_route(ctx, Xd, rho, tau)
        route = r_gpu.astype(bool)
    import torch
    P.slh_load(ctx, B.SLH_OUT_CODES, torch.from_numpy(codes.astype(np.int32)).cuda())
    P.slh_merge(ctx, Xd)
    sim, tot = P.slh_bucket_purity(ctx, Xd, 0.7)
    X = inp.x_float()
    osim = otot = near = 0
    for w in range(wl.N // Lw):
        if not route[w]:
            continue
        a, b = O.bucket_purity(X[w * Lw:(w + 1) * Lw], codes[w * Lw:(w + 1) * Lw])
        osim += a
        otot += b
        # pairs within 1e-12 of the threshold (their bit may differ in fp64)
        hi, _ = O.bucket_purity(X[w * Lw:(w + 1) * Lw], codes[w * Lw:(w + 1) * Lw], 0.7 + 1e-12)
        lo, _ = O.bucket_purity(X[w * Lw:(w + 1) * Lw], codes[w * Lw:(w + 1) * Lw], 0.7 - 1e-12)
        near += lo - hi
    _say(f"[purity] {case}: gpu {sim}/{tot} oracle {osim}/{otot} near-threshold {near}")
    assert tot == otot and abs(sim - osim) <= near


@pytest.mark.parametrize("case", ["tiny_keep5", "local16_keep12", "compact_keep3"])
def test_preserved_suffix(case):
    """SLH_OPT_KEEP_LAST: the last K tokens are not compressed and follow the
    compressed macro-tokens as their own rows at their own positions (reading
    R19); compression runs on the first N - K tokens (windows tile them)."""
    compact = False
    if case == "tiny_keep5":
        inp, L, K = make_inputs("tiny"), 0, 5
        inp = Inputs(Workload("tk5", 517, 256, 256, 32, 8, 6, 4.0, 0, 0, "f32"),
                     np.concatenate([inp.X, inp.X[:5] * 2.0]), np.zeros(517))
    elif case == "local16_keep12":
        inp, L, K = make_inputs("local16", N=1036), 16, 12
    else:
        inp, L, K, compact = _custom("ck3", 4 * 256 + 3, 256, 256, 16, 8, 8), 256, 3, True
    wl = inp.workload
    _say(f"[keep last] {case} N={wl.N} K={K} window={L}")
    g = PR.run_gpu(inp, n_it=wl.n_it, window=L, keep_last=K, compact=compact)
    o = PR.run_oracle(inp, n_it=wl.n_it, window=L, keep_last=K, compact=compact)
    Nc = wl.N - K
    M, Mg = len(o.P), len(g.P)
    # the suffix is the last K rows on both sides; the count of compressed rows
    # before it may differ only through codes compare() does not hold against
    # the GPU (near-zero or undetermined projections), which it checks below
    assert np.array_equal(g.P[Mg - K:], o.P[M - K:])
    assert np.array_equal(g.t2m[Nc:] - (Mg - K), np.arange(K))
    assert np.array_equal(o.t2m[Nc:] - (M - K), np.arange(K))
    assert np.array_equal(g.E[Mg - K:], o.E[M - K:].astype(np.float32))
    unc = {w.w: PR.oracle_uncertainty(inp, w.w, L, wl.n_it) for w in o.windows} if L == 16 else None
    rep = PR.compare(o, g, L or Nc, unc=unc)
    _say(f"   {rep}  M={M} gpu {Mg}")


@pytest.mark.parametrize("case,T", [("tiny", 30), ("tiny", 100), ("tiny", 1), ("tiny", 512),
                                    ("windows", 200), ("windows", 700), ("long", 300), ("long", 6000),
                                    ("keep", 90)])
def test_exact_target_length(case, T):
    """SLH_OPT_TARGET_LEN (reading R20; the paper gives no algorithm, so the
    oracle follows the same reading and parity is unpinned): with the oracle's
    codes loaded, the GPU merge must produce exactly the oracle's adjusted
    groups (positions and token maps bit-exact, embeddings 1e-5).  tiny: one
    window of 512 (merge to 30 / 1, split to 100 / 512); windows: 8 windows of
    256, half routed to chunk pooling; long: one window of 20000 tokens (more
    than one 16384-position chunk of the block scans; merged to 300, split to
    6000); keep: 512 + 12 preserved tokens."""
    import torch
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    rho, L, K = None, 0, 0
    if case == "tiny":
        inp = make_inputs("tiny")
        codes = np.random.default_rng(1).integers(0, 64, inp.workload.N)
    elif case == "windows":
        inp, L, rho = _custom("twin", 8 * 256, 256, 256, 16, 8, 8), 256, 8.0
        codes = np.random.default_rng(2).integers(0, 64, inp.workload.N)
    elif case == "long":
        inp = _custom("tlong", 20000, 64, 256, 8, 4, 12)
        codes = np.minimum(np.random.default_rng(3).zipf(1.3, 20000) - 1, 4095)
    else:
        base = make_inputs("tiny")
        inp = Inputs(Workload("tkeep", 524, 256, 256, 32, 8, 6, 4.0, 0, 0, "f32"),
                     np.concatenate([base.X, base.X[:12] * 0.5]), np.zeros(524))
        codes = np.random.default_rng(4).integers(0, 64, 524)
        K = 12
    wl = inp.workload
    Nc = wl.N - K
    Lw = L or Nc
    ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
    if K:
        P.slh_set_option(ctx, B.SLH_OPT_KEEP_LAST, K)
    if L:
        P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
    P.slh_set_option(ctx, B.SLH_OPT_TARGET_LEN, T)
    Xd = PR.to_device_x(inp)
    route = np.ones(Nc // Lw, bool)
    if rho is not None:
        sc = np.array([O.redundancy_score(inp.x_float(slice(w * Lw, (w + 1) * Lw)))
                       for w in range(Nc // Lw)])
        r_gpu, _ = P.slh_route(ctx, Xd, rho, float(np.median(sc)))
        route = r_gpu.astype(bool)
    P.slh_load(ctx, B.SLH_OUT_CODES, torch.from_numpy(codes.astype(np.int32)).cuda())
    E, Pp, t2m, M = P.slh_merge(ctx, Xd)
    torch.cuda.synchronize()
    gE, gP, gt = E[:M].cpu().numpy(), Pp[:M].cpu().numpy(), t2m.cpu().numpy()
    # oracle: budgets, adjusted groups per spectral window, chunk windows, tail
    budgets = O.target_budgets(T, route, Lw, O.chunk_size(rho) if rho else 1, K)
    X = inp.x_float()
    Es, Ps, tms = [], [], np.zeros(wl.N, np.int64)
    base = 0
    for w in range(Nc // Lw):
        sl = slice(w * Lw, (w + 1) * Lw)
        if route[w]:
            groups = O.merge(X[sl], codes[sl]).members
            groups = O.adjust_to_target(groups, budgets[w])
            Ew, Pw, tw = O.merge_groups(X[sl], groups, positions=w * Lw + np.arange(Lw))
        else:
            k = O.chunk_size(rho)
            Ew, Pw = O.chunk_pool(X[sl], k, pos0=w * Lw)
            tw = np.arange(Lw) // k
        Es.append(Ew)
        Ps.append(Pw)
        tms[sl] = base + tw
        base += len(Pw)
    oE, oP, ot = np.concatenate(Es), np.concatenate(Ps), tms[:Nc]
    if K:
        oE, oP, ot = O.preserve_suffix(oE, oP, ot, X[Nc:], Nc)
    _say(f"[target] {case} T={T}: M gpu {M} oracle {len(oP)}")
    assert M == T == len(oP)
    assert np.array_equal(gP, oP) and np.array_equal(gt, ot)
    rel = np.linalg.norm(gE - oE, axis=1) / np.maximum(np.linalg.norm(oE, axis=1), 1e-30)
    assert rel.max() <= 1e-5


@pytest.mark.parametrize("case", ["tiny", "windows256", "resident"])
def test_time_passes(case):
    """slh_time_passes replays the final step's pass over Phi as a graph:
    it returns a positive duration and leaves every result of slh_lanczos (Q,
    alpha, beta, Ritz values and vectors) and the SimHash codes bit-identical;
    it is refused before slh_lanczos and after a short-window run."""
    import paper_2607_19368_amd as P
    from paper_2607_19368_amd import slh as B
    if case == "tiny":
        inp, L = make_inputs("tiny"), 0
    elif case == "resident":                  # the resident kernel: its runs are timed
        inp, L = _custom("tpr", 2048, 264, 1024, 32, 8, 8), 0
    else:
        inp, L = _custom("tpw", 4 * 256, 512, 256, 24, 8, 8), 256
    wl = inp.workload
    Xd = PR.to_device_x(inp)

    def run(time_it):
        ctx = P.slh_create(wl.N, wl.D, wl.m, wl.r, wl.bits, 0)
        if L:
            P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, L)
        P.slh_feature_map(ctx, Xd)
        if time_it:
            with pytest.raises(B.SLHError):
                P.slh_time_passes(ctx, 4)
        P.slh_lanczos(ctx, wl.n_it)
        outs = [P.slh_copy_out(ctx, k) for k in (B.SLH_OUT_Q, B.SLH_OUT_ALPHA, B.SLH_OUT_BETA,
                                                  B.SLH_OUT_THETA, B.SLH_OUT_Z)]
        us = None
        if time_it:
            us = P.slh_time_passes(ctx, 16)
            after = [P.slh_copy_out(ctx, k) for k in (B.SLH_OUT_Q, B.SLH_OUT_ALPHA, B.SLH_OUT_BETA,
                                                       B.SLH_OUT_THETA, B.SLH_OUT_Z)]
            for a, b in zip(outs, after):
                assert np.array_equal(a, b)
        P.slh_simhash(ctx)
        return us, P.slh_copy_out(ctx, B.SLH_OUT_CODES)

    us, codes_t = run(True)
    _, codes = run(False)
    _say(f"[time passes] {case}: {us:.2f} us per pass")
    assert np.isfinite(us) and 0.0 < us < 1e5
    assert np.array_equal(codes_t, codes)
    # short windows have no passes over Phi
    inp16 = make_inputs("local16", N=524)
    w16 = inp16.workload
    ctx = P.slh_create(w16.N, w16.D, w16.m, w16.r, w16.bits, 0)
    P.slh_set_option(ctx, B.SLH_OPT_KEEP_LAST, w16.keep_last)
    P.slh_set_option(ctx, B.SLH_OPT_WINDOW_LEN, 16)
    P.slh_feature_map(ctx, PR.to_device_x(inp16))
    P.slh_lanczos(ctx, w16.n_it)
    with pytest.raises(B.SLHError):
        P.slh_time_passes(ctx, 4)

