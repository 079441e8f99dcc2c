"""GPU parity: the HIP path (called through the C ABI) against the FP64 oracle.

Sizes here span several 64-row slices and every subband; the full-size
workloads are covered in test_gpu_fullsize.py.  Float32 tolerances are stated
per test; the solver gates are those of the 64x64 parity case: relative
objective within 1e-5 and relative ||x - x_oracle|| <= 1e-4 after 200
iterations.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import synth
from oracle import blur, dwt, filters, fista, lipschitz, pipeline, precond, theta

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def W():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_1512_08401_amd import wdb
    return wdb


@pytest.fixture(scope="module")
def p64():
    """Oracle problem of the 64x64 parity workload (Haar, 3 levels, 40 nnz/px)."""
    wl = synth.WORKLOADS["parity64"]
    P = pipeline.build_problem(wl)
    P["wl"] = wl
    A = P["A"]
    P["A32"] = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    return P


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def imported(W, P):
    rp, cc, vv = theta.csr_arrays(P["A"])
    wl = P["wl"]
    return W.Theta.from_csr(wl.n, wl.wavelet, wl.levels, rp, cc, vv)


# ---------------------------------------------------------------------------
# transforms and blur
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("name,n,J", [("haar", 64, 3), ("db4", 64, 3), ("db4", 256, 4), ("db4", 16, 1),
                                      ("haar", 8, 3), ("sym6", 64, 3), ("sym6", 512, 6)])
def test_dwt_forward_inverse(W, name, n, J):
    print(f"dwt {name} n={n} J={J}", flush=True)
    u = np.random.default_rng(n + J).random((n, n)).astype(np.float32)
    x = host(W.dwt(dev(u).reshape(-1), name, J))
    xo = dwt.dwt2(u.astype(np.float64), filters.by_name(name), J)
    assert np.max(np.abs(x - xo)) <= 2e-6 * np.max(np.abs(xo))
    c = np.random.default_rng(1).standard_normal(n * n).astype(np.float32)
    v = host(W.dwt(dev(c), name, J, inverse=True))
    vo = dwt.idwt2(c.astype(np.float64), filters.by_name(name), J, n).ravel()
    assert np.max(np.abs(v - vo)) <= 2e-6 * np.max(np.abs(vo))


@pytest.mark.parametrize("name,n,J,count", [("db4", 64, 3, 11), ("sym6", 128, 4, 8), ("haar", 32, 5, 1)])
def test_dwt_batched_matches_single(W, name, n, J, count):
    """The batched transform (8 images per launch, a ragged last group when
    count = 11) against the oracle per image, and bit for bit against the
    single-image entry point, both directions."""
    print(f"dwt batched {name} n={n} J={J} count={count}", flush=True)
    u = np.random.default_rng(count).random((count, n * n)).astype(np.float32)
    x = host(W.dwt_batched(dev(u), name, J))
    for i in range(count):
        xo = dwt.dwt2(u[i].reshape(n, n).astype(np.float64), filters.by_name(name), J)
        assert np.max(np.abs(x[i] - xo)) <= 2e-6 * np.max(np.abs(xo))
        assert np.array_equal(x[i], host(W.dwt(dev(u[i]), name, J)))
    v = host(W.dwt_batched(dev(x), name, J, inverse=True))
    for i in range(count):
        assert np.array_equal(v[i], host(W.dwt(dev(x[i]), name, J, inverse=True)))
        assert np.max(np.abs(v[i] - u[i])) <= 2e-6


@pytest.mark.parametrize("name,n,J", [("haar", 2, 1), ("haar", 4, 2), ("db4", 8, 1), ("sym6", 16, 1), ("db4", 256, 1),
                                      ("db4", 256, 4), ("sym6", 256, 2), ("sym6", 512, 4), ("db4", 512, 2),
                                      ("db4", 1024, 6), ("haar", 1024, 3), ("haar", 2048, 9), ("db4", 2048, 4)])
def test_dwt_launch_plans_match_oracle(W, name, n, J):
    """Every way the transform is split: one block per image (sides up to 128),
    one to three levels per launch before it or alone, a second launch of many
    blocks (side 2048), 32 x 32 and 64 x 64 pixels per inverse block; the inverse
    also into a buffer that is only 4-byte aligned.  Bars of the tests above."""
    print(f"dwt plan {name} n={n} J={J}", flush=True)
    u = np.random.default_rng(n + J).random((n, n)).astype(np.float32)
    x = host(W.dwt(dev(u).reshape(-1), name, J))
    xo = dwt.dwt2(u.astype(np.float64), filters.by_name(name), J)
    assert np.max(np.abs(x - xo)) <= 2e-6 * np.max(np.abs(xo))
    c = np.random.default_rng(1).standard_normal(n * n).astype(np.float32)
    odd = torch.zeros(n * n + 1, device="cuda")[1:]
    v = host(W.dwt(dev(c), name, J, inverse=True, out=odd))
    vo = dwt.idwt2(c.astype(np.float64), filters.by_name(name), J, n).ravel()
    assert np.max(np.abs(v - vo)) <= 2e-6 * np.max(np.abs(vo))
    assert np.array_equal(v, host(W.dwt(dev(c), name, J, inverse=True)))


@pytest.mark.parametrize("name,n,J,count", [("sym6", 512, 6, 5), ("sym6", 1024, 6, 1), ("sym6", 2048, 8, 1),
                                            ("db4", 4096, 10, 1)])
def test_inverse_dwt_of_many_levels_matches_oracle(W, name, n, J, count):
    """Inverse transforms whose levels take more than 64 KiB of LDS (the fewest and
    the most levels of 12 taps, the fewest of 8).  Bar of the tests above."""
    print(f"idwt {name} n={n} J={J} count={count}", flush=True)
    c = np.random.default_rng(n + J).standard_normal((count, n * n)).astype(np.float32)
    v = host(W.dwt_batched(dev(c), name, J, inverse=True)).reshape(count, -1)
    for i in {0, count - 1}:
        vo = dwt.idwt2(c[i].astype(np.float64), filters.by_name(name), J, n).ravel()
        assert np.max(np.abs(v[i] - vo)) <= 2e-6 * np.max(np.abs(vo))


@pytest.mark.parametrize("name", ["haar", "db4", "sym6"])
def test_dwt_of_one_level_at_side_128(W, name):
    """A single level of side 128 goes to blocks of 16 x 16 positions, more levels to
    one block per image: both against the oracle (bar of the tests above), with
    the first level's details equal bit for bit, and a batch like one image."""
    n = 128
    u = np.random.default_rng(4).random((35, n, n)).astype(np.float32)
    one = host(W.dwt_batched(dev(u.reshape(35, -1)), name, 1)).reshape(35, -1)
    two = host(W.dwt_batched(dev(u.reshape(35, -1)), name, 2)).reshape(35, -1)
    assert np.array_equal(one[:, n * n // 4:], two[:, n * n // 4:])
    for i in (0, 34):
        xo = dwt.dwt2(u[i].astype(np.float64), filters.by_name(name), 1)
        assert np.max(np.abs(one[i] - xo)) <= 2e-6 * np.max(np.abs(xo))
        assert np.array_equal(one[i], host(W.dwt(dev(u[i]).reshape(-1), name, 1)))


def test_dwt_many_images_match_single(W):
    """More images than a launch takes, and enough blocks for the larger tile."""
    n, J, count = 64, 2, 261
    u = np.random.default_rng(7).random((count, n * n)).astype(np.float32)
    x = W.dwt_batched(dev(u), "db4", J)
    v = host(W.dwt_batched(x, "db4", J, inverse=True))
    x = host(x)
    for i in (0, 31, 32, 100, 260):
        assert np.array_equal(x[i], host(W.dwt(dev(u[i]), "db4", J)))
        assert np.array_equal(v[i], host(W.dwt(dev(x[i]), "db4", J, inverse=True)))
    assert np.max(np.abs(v - u)) <= 2e-6


@pytest.mark.parametrize("field", [synth.psf_isotropic(64, 1.0, 3.0), synth.psf_rotating(128, 4.0, 1.0),
                                   synth.psf_rotating(32, 2.5, 0.7)])
def test_blur_matches_oracle(W, field):
    print(f"blur n={field.n}", flush=True)
    u = synth.piecewise_image(field.n, 5).astype(np.float32)
    out = host(W.blur(field, dev(u)))
    ref = blur.blur(field, u.astype(np.float64))
    assert np.max(np.abs(out - ref)) <= 1e-6


# ---------------------------------------------------------------------------
# Theta_K construction
# ---------------------------------------------------------------------------
def _compare_kept(rp, cc, vv, T, K, tol_rel=1e-12):
    N = T.shape[0]
    rows = np.repeat(np.arange(N), np.diff(rp))
    got = rows.astype(np.int64) * N + cc
    r, c, v = theta.top_k(T, K)
    want = r * N + c
    amax = np.max(np.abs(T))
    thr = theta.threshold_value(T, K)
    sym = np.setxor1d(got, want)
    # kept sets may differ only where |Theta| is within rounding of the cut
    if sym.size:
        mags = np.abs(T.ravel()[sym])
        assert np.all(np.abs(mags - thr) <= tol_rel * amax), f"{sym.size} kept entries differ away from the cut"
    common, ig, iw = np.intersect1d(got, want, return_indices=True)
    assert np.max(np.abs(vv[ig] - T.ravel()[common])) <= 1e-13 * amax
    return sym.size


@pytest.mark.parametrize("case", ["parity64", "db4_32_rot", "haar_16", "db4_16_wrap", "sym6_64"])
def test_build_theta_matches_dense_oracle(W, p64, case):
    print(f"build {case}", flush=True)
    if case == "parity64":
        wl = p64["wl"]
        field, name, J, K, T = wl.psf(), wl.wavelet, wl.levels, wl.nnz, p64["T"]
    else:
        field, name, J = {"db4_32_rot": (synth.psf_rotating(32, 2.5, 1.0), "db4", 2),
                          "haar_16": (synth.psf_isotropic(16, 1.0, 2.0), "haar", 2),
                          "db4_16_wrap": (synth.psf_rotating(16, 2.0, 0.8), "db4", 1),
                          "sym6_64": (synth.psf_rotating(64, 3.0, 1.0), "sym6", 2)}[case]
        K = 20 * field.n ** 2
        T = theta.theta_dense(field, filters.by_name(name), J)
    th = W.build_theta(field, name, J, K)
    info = th.info()
    assert info["nnz"] == K
    rp, cc, vv = th.export()
    _compare_kept(rp, cc, vv, T, K)
    assert abs(info["threshold"] - theta.threshold_value(T, K)) <= 1e-12 * np.max(np.abs(T))


@pytest.mark.parametrize("rule", ["naive", "scale"])
@pytest.mark.parametrize("field,name,J", [(synth.psf_stationary(16, 1.2, 1.2), "haar", 2),
                                          (synth.psf_rotating(32, 2.0, 1.0), "haar", 3),
                                          (synth.psf_rotating(32, 2.5, 0.7), "db4", 1)])
def test_build_keeps_the_largest_entries_exactly(W, monkeypatch, field, name, J, rule):
    """The column-by-column build of a few budgets against its own full set of
    entries: the largest ranked magnitudes, equal ones by ascending linear index
    (the symmetric field has many), down to the last bit."""
    monkeypatch.setenv("WDB_BUILD_GENERAL", "1")
    n = field.n
    N = n * n
    rp, cc, vv = W.build_theta(field, name, J, N * N, rule=rule).export()
    idx = np.repeat(np.arange(N, dtype=np.int64), np.diff(rp)) * N + cc
    mag = np.abs(vv)
    if rule == "scale":
        sides = [n >> J] + [n >> lev for lev in range(J, 0, -1) for _ in range(3)]
        side = np.concatenate([np.full(t * t, t) for t in sides])
        mag = mag / side[cc]
    order = np.lexsort((idx, -mag))
    first = np.flatnonzero(np.diff(mag[order]) == 0.0)   # an entry equal to the next: a cut inside equal ones
    cuts = {1, len(vv) // 7, len(vv) - 1} | {int(first[t]) + 1 for t in (0, len(first) // 2, -1) if len(first)}
    for K in sorted(cuts):
        th = W.build_theta(field, name, J, K, rule=rule)
        r, c, v = th.export()
        keep = np.sort(order[:K])
        assert np.array_equal(np.repeat(np.arange(N, dtype=np.int64), np.diff(r)) * N + c, idx[keep]), K
        assert np.array_equal(v, vv[keep]), K
        assert th.info()["threshold"] == mag[order[K - 1]], K


@pytest.mark.parametrize("rule", ["naive", "scale"])
@pytest.mark.parametrize("field,name,J", [(synth.psf_rotating(64, 2.5, 1.0), "haar", 3),
                                          (synth.psf_rotating(32, 2.0, 0.7), "db4", 1),
                                          (synth.psf_isotropic(64, 0.5, 5.0), "sym6", 2)])
def test_build_without_the_weights_table_is_the_same(W, monkeypatch, capfd, field, name, J, rule):
    """Weights evaluated where they are used, as where their table does not fit:
    the same matrix to the last bit (the same terms in the same order)."""
    n = field.n
    monkeypatch.setenv("WDB_LOG", "1")
    got = []
    for table in ("1", "0"):
        monkeypatch.setenv("WDB_BUILD_TABLE", table)
        th = W.build_theta(field, name, J, 20 * n * n + 3, rule=rule)
        assert ("bytes kept" in capfd.readouterr().err) == (table == "1")
        got.append((*th.export(), th.info()["threshold"]))
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("case", ["haar64_iso", "db4_32_aniso", "haar16_cut"])
def test_convolution_build_matches_alg3_oracle(W, case):
    """A stationary field takes the fast path (one column per subband, circulant
    copies); the kept set and values match the oracle's Alg. 3 Theta."""
    from oracle import theta_conv
    field, name, J, K = {"haar64_iso": (synth.psf_stationary(64, 1.5, 1.5), "haar", 3, 40 * 4096),
                         "db4_32_aniso": (synth.psf_stationary(32, 2.5, 1.0, 0.6), "db4", 2, 30 * 1024),
                         "haar16_cut": (synth.psf_stationary(16, 1.2, 1.2), "haar", 2, 777)}[case]
    print(f"conv build {case}", flush=True)
    T = theta_conv.theta_convolution(field, filters.by_name(name), J)
    th = W.build_theta(field, name, J, K)
    info = th.info()
    assert info["conv_build"] == 1 and info["nnz"] == K
    rp, cc, vv = th.export()
    _compare_kept(rp, cc, vv, T, K)
    assert abs(info["threshold"] - theta.threshold_value(T, K)) <= 1e-12 * np.max(np.abs(T))


@pytest.mark.parametrize("case", ["haar64_iso", "db4_32_aniso", "haar16_cut"])
def test_circulant_storage_matches_oracle(W, case):
    """The circulant (stencil) layout of a convolution build: products and a
    200-iteration solve against the oracle's Alg. 3 Theta_K."""
    from oracle import theta_conv
    field, name, J, K0 = {"haar64_iso": (synth.psf_stationary(64, 1.5, 1.5), "haar", 3, 40 * 4096),
                          "db4_32_aniso": (synth.psf_stationary(32, 2.5, 1.0, 0.6), "db4", 2, 30 * 1024),
                          "haar16_cut": (synth.psf_stationary(16, 1.2, 1.2), "haar", 2, 777)}[case]
    print(f"circulant {case}", flush=True)
    n = field.n
    N = n * n
    T = theta_conv.theta_convolution(field, filters.by_name(name), J)
    # The kept sets of two builds agree only up to entries within rounding of the
    # cut; put the cut where the oracle's magnitudes have a clear gap, or (for the
    # partial-group case) inside a group of exactly equal circulant copies that is
    # clear of its neighbours, so both sides keep the same entries.
    mags = np.sort(np.abs(T[T != 0]).ravel())[::-1]
    amax = mags[0]
    levels, counts = np.unique(mags, return_counts=True)
    levels, counts = levels[::-1], counts[::-1]
    above = np.concatenate([[0], np.cumsum(counts)])
    gap_lo = np.concatenate([[np.inf], levels[:-1] - levels[1:]])      # to the next larger level
    gap_hi = np.concatenate([levels[:-1] - levels[1:], [np.inf]])      # to the next smaller level
    clear = (gap_lo > 1e-9 * amax) & (gap_hi > 1e-9 * amax)
    if case.endswith("cut"):
        cand = [i for i in range(len(levels)) if clear[i] and counts[i] >= 4]
        i = min(cand, key=lambda i: abs(above[i] - K0))
        K = int(above[i] + counts[i] // 2)
    else:
        cand = [i for i in range(1, len(levels)) if gap_lo[i] > 1e-9 * amax]
        i = min(cand, key=lambda i: abs(above[i] - K0))
        K = int(above[i])
    r, c, v = theta.top_k(T, K)
    A = theta.to_csr(r, c, v, N)
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    th = W.build_theta(field, name, J, K)
    assert th.info()["circulant"] >= 0
    if case.endswith("cut"):
        assert th.info()["circulant"] > 0      # the cut splits a group: explicit entries are in use
    x = np.random.default_rng(41).standard_normal(N).astype(np.float32)
    b = np.random.default_rng(42).standard_normal(N).astype(np.float32)
    th.set_kernel_layout(8, 4)
    csr = [host(th.apply(dev(x), dev(b), transpose=tr)) for tr in (False, True)]
    th.set_kernel_layout(8, 1)
    assert th.info()["group"] == 1
    for tr in (False, True):
        y = host(th.apply(dev(x), dev(b), transpose=tr))
        # same handle, padded-CSR layout: identical kept entries, float32 order only
        assert np.max(np.abs(y - csr[tr])) <= 1e-5 * np.max(np.abs(csr[tr])), tr
        if not case.endswith("cut"):
            # against the oracle's Theta_K (a cut clear of rounding-level ties); in the
            # cut case equal copies may order differently, and the kept set is pinned
            # by test_convolution_build_matches_alg3_oracle instead
            ref = (A32.T if tr else A32) @ x.astype(np.float64) - b
            assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)), tr
    start = synth.power_start(N, 9)
    th.lipschitz(start)
    u0 = (blur.blur(field, synth.piecewise_image(n, 43)) + synth.noise(n, 0.01, 44)).astype(np.float32)
    x0 = dwt.dwt2(u0.astype(np.float64), filters.by_name(name), J).astype(np.float32)
    lam = float(np.float32(2e-3))
    xg, _ = th.solve_coeffs(dev(x0), lam, 200, check_every=50)
    if case.endswith("cut"):
        th.set_kernel_layout(8, 4)
        xc, _ = th.solve_coeffs(dev(x0), lam, 200, check_every=50)
        assert np.linalg.norm(host(xg) - host(xc)) <= 1e-5 * np.linalg.norm(host(xc))
        return
    L, _ = lipschitz.lipschitz(A32, start)
    xo, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1.0 / L, 200)
    _gate(A32, x0.astype(np.float64), lam, host(xg), xo, fista.objective(A32, x0.astype(np.float64), lam, xo))


def test_convolution_build_agrees_with_general_build(W, monkeypatch):
    """At 128 x 128 (db4, 3 levels) the fast path and the column-by-column
    build give the same Theta_K up to rounding at the cut."""
    field = synth.psf_stationary(128, 2.0, 1.0, 0.3)
    K = 25 * 128 * 128
    fast = W.build_theta(field, "db4", 3, K)
    monkeypatch.setenv("WDB_BUILD_GENERAL", "1")
    slow = W.build_theta(field, "db4", 3, K)
    assert fast.info()["conv_build"] == 1 and slow.info()["conv_build"] == 0
    N = 128 * 128
    (rf, cf, vf), (rs, cs, vs) = fast.export(), slow.export()
    kf = np.repeat(np.arange(N), np.diff(rf)).astype(np.int64) * N + cf
    ks = np.repeat(np.arange(N), np.diff(rs)).astype(np.int64) * N + cs
    amax = np.max(np.abs(vs))
    thr = slow.info()["threshold"]
    diff = np.setxor1d(kf, ks)
    if diff.size:   # only entries at the cut (to rounding) may differ
        vals = np.concatenate([np.abs(vf[np.isin(kf, diff)]), np.abs(vs[np.isin(ks, diff)])])
        assert np.all(np.abs(vals - thr) <= 1e-12 * amax)
    common, i_f, i_s = np.intersect1d(kf, ks, return_indices=True)
    assert np.max(np.abs(vf[i_f] - vs[i_s])) <= 1e-13 * amax


@pytest.mark.parametrize("case", ["rot32_db4", "conv64_haar"])
def test_scale_weighted_threshold_matches_oracle(W, case):
    """Sec. 3.7 weighted rule: keep the K largest 2^-k |Theta[a, b]| (k the scale of column b),
    by the general build (spatially varying field) and by the convolution fast path."""
    field, name, J, K = {"rot32_db4": (synth.psf_rotating(32, 2.5, 1.0), "db4", 2, 20 * 1024),
                         "conv64_haar": (synth.psf_stationary(64, 1.5, 1.0, 0.7), "haar", 3, 30 * 4096)}[case]
    print(f"scale rule {case}", flush=True)
    T = theta.theta_dense(field, filters.by_name(name), J)
    n = field.n
    N = n * n
    sig = theta.column_scale_weights(n, J)
    th = W.build_theta(field, name, J, K, rule="scale")
    info = th.info()
    assert info["rule"] == 1 and info["nnz"] == K
    assert info["conv_build"] == (1 if case.startswith("conv") else 0)
    rp, cc, vv = th.export()
    got = np.repeat(np.arange(N), np.diff(rp)).astype(np.int64) * N + cc
    r, c, _ = theta.top_k_weighted(T, K, sig)
    want = r * N + c
    S = np.abs(T) * sig[None, :]
    order = np.sort(S.ravel())[::-1]
    thr = order[K - 1]
    amax = S.max()
    sym = np.setxor1d(got, want)
    if sym.size:
        assert np.all(np.abs(S.ravel()[sym] - thr) <= 1e-12 * amax), f"{sym.size} entries differ away from the cut"
    common, ig, _ = np.intersect1d(got, want, return_indices=True)
    assert np.max(np.abs(vv[ig] - T.ravel()[common])) <= 1e-13 * np.max(np.abs(T))
    assert abs(info["threshold"] - thr) <= 1e-12 * amax
    # the weighted rule keeps more coarse-column entries than the naive one
    naive = W.build_theta(field, name, J, K)
    rn, cn, _ = naive.export()
    coarse = sig[cc] >= np.median(sig)
    coarse_n = sig[cn] >= np.median(sig)
    assert coarse.sum() >= coarse_n.sum()


def test_build_theta_budget_edges(W):
    field = synth.psf_rotating(32, 2.5, 1.0)
    T = theta.theta_dense(field, filters.db4(), 2)
    # one entry: the largest magnitude
    th = W.build_theta(field, "db4", 2, 1)
    rp, cc, vv = th.export()
    a = int(np.searchsorted(rp, 1, side="left") - 1)
    assert rp[a] == 0 and rp[a + 1] == 1 and vv[0] == pytest.approx(T[a, cc[0]], rel=1e-13)
    # the field is invariant down columns, so several entries tie with the
    # maximum to rounding; the kept one must be one of them
    assert abs(vv[0]) >= np.max(np.abs(T)) * (1 - 1e-13)
    # budget beyond the non-zeros keeps every non-zero of the column windows
    th = W.build_theta(field, "db4", 2, 1024 * 1024)
    rp, cc, vv = th.export()
    N = 1024
    rows = np.repeat(np.arange(N), np.diff(rp))
    assert np.max(np.abs(vv - T[rows, cc])) <= 1e-13
    mask = np.ones_like(T, dtype=bool)
    mask[rows, cc] = False
    assert np.max(np.abs(T[mask])) <= 1e-14          # only rounding-level values are absent


# ---------------------------------------------------------------------------
# kernels on an imported oracle Theta_K
# ---------------------------------------------------------------------------
def test_apply_matches_oracle(W, p64):
    th = imported(W, p64)
    A32 = p64["A32"]
    N = A32.shape[0]
    rng = np.random.default_rng(3)
    x = rng.standard_normal(N).astype(np.float32)
    b = rng.standard_normal(N).astype(np.float32)
    y = host(th.apply(dev(x), dev(b)))
    ref = A32 @ x.astype(np.float64) - b
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref))
    yt = host(th.apply(dev(x), None, transpose=True, repeat=3))
    reft = A32.T @ x.astype(np.float64)
    assert np.max(np.abs(yt - reft)) <= 1e-5 * np.max(np.abs(reft))


def test_empty_and_ragged_operator(W):
    """Rows of very different lengths (0 .. 700) and an empty operator."""
    n, N = 32, 1024
    rng = np.random.default_rng(9)
    lens = np.zeros(N, dtype=np.int64)
    lens[rng.choice(N, 40, replace=False)] = rng.integers(1, 700, 40)
    lens[5] = N
    cols, vals = [], []
    for r in range(N):
        c = np.sort(rng.choice(N, lens[r], replace=False)).astype(np.int32)
        cols.append(c)
        vals.append(rng.standard_normal(lens[r]))
    rp = np.concatenate([[0], np.cumsum(lens)])
    cc, vv = np.concatenate(cols), np.concatenate(vals)
    th = W.Theta.from_csr(n, "haar", 2, rp, cc, vv)
    A = sp.csr_matrix((vv.astype(np.float32).astype(np.float64), cc, rp), shape=(N, N))
    x = rng.standard_normal(N).astype(np.float32)
    assert np.max(np.abs(host(th.apply(dev(x))) - A @ x)) <= 1e-4
    assert np.max(np.abs(host(th.apply(dev(x), transpose=True)) - A.T @ x)) <= 1e-4
    e = W.Theta.from_csr(n, "haar", 2, np.zeros(N + 1, dtype=np.int64), np.zeros(0, np.int32), np.zeros(0))
    b = rng.standard_normal(N).astype(np.float32)
    assert np.array_equal(host(e.apply(dev(x), dev(b))), -b.astype(np.float64))
    # the same on the tiled storage with dense and kept values (the long row's
    # far columns go to the escape lists; the empty operator has no groups)
    for op, ref, reft in ((th, A @ x, A.T @ x), (e, -b.astype(np.float64), np.zeros(N))):
        op.set_kernel_layout(8, 3)
        for kept in (0, 1):
            op.set_tile_values(kept)
            got = host(op.apply(dev(x), dev(b) if op is e else None))
            assert np.max(np.abs(got - ref)) <= 1e-4, kept
            assert np.max(np.abs(host(op.apply(dev(x), transpose=True)) - reft)) <= 1e-4, kept


def test_prox_step_matches_oracle(W, p64):
    th = imported(W, p64)
    A32 = p64["A32"]
    N = A32.shape[0]
    rng = np.random.default_rng(4)
    r, x, y = (rng.standard_normal(N).astype(np.float32) for _ in range(3))
    tau, lam, beta = 0.9, 0.05, 0.4
    xd, yd = dev(x), dev(y)
    th.prox_step(dev(r), xd, yd, tau, lam, beta)
    g = A32.T @ r.astype(np.float64)
    xn = fista.soft_threshold(y - tau * g, tau * lam)
    yn = xn + beta * (xn - x)
    assert np.max(np.abs(host(xd) - xn)) <= 1e-5 * np.max(np.abs(xn))
    assert np.max(np.abs(host(yd) - yn)) <= 1e-5 * np.max(np.abs(yn))


def test_lipschitz_matches_oracle(W, p64):
    th = imported(W, p64)
    start = synth.power_start(4096, p64["wl"].power_seed)
    L, its = th.lipschitz(start)
    Lo, itso = lipschitz.lipschitz(p64["A32"], start)
    assert abs(L - Lo) <= 1e-9 * Lo
    assert abs(its - itso) <= 1
    # independent pin: the largest singular value squared
    ev = np.linalg.norm(p64["A32"].toarray(), 2) ** 2
    assert abs(L - ev) <= 1e-8 * ev


def test_lanczos_matches_the_largest_singular_value(W, p64):
    """The restarted Lanczos estimate (the solver's default step) against the
    largest singular value squared of the same float32 operator; the stored
    L = theta + resid bounds it from above, and a solve without an explicit
    L uses it."""
    th = imported(W, p64)
    start = synth.power_start(4096, p64["wl"].power_seed)
    r = th.lipschitz_lanczos(start)
    ev = np.linalg.norm(p64["A32"].toarray(), 2) ** 2
    assert r["converged"] and r["resid"] <= 1e-12 * r["theta"]
    assert abs(r["theta"] - ev) <= 1e-11 * ev and r["L"] >= ev * (1 - 1e-13)
    th2 = imported(W, p64)
    _, info = th2.solve_coeffs(dev(p64["x0"]), p64["wl"].lam, 20, check_every=20)
    assert abs(info["lipschitz"] - ev) <= 1e-11 * ev


def test_clustered_top_eigenvalues_lanczos_vs_power_iteration(W):
    """A diagonal operator with known spectrum whose two largest eigenvalues of
    A^T A are 1e-3 apart (about the relative gap of the 1024 x 1024
    workload's operator, where the power iteration used all 20000
    iterations): the power iteration reports that it stopped at its cap with
    a lower bound, the restarted Lanczos converges to the exact top value and
    the stored L bounds it from above."""
    n, J = 64, 3
    N = n * n
    rng = np.random.default_rng(5)
    lam = rng.uniform(0.0, 0.99, N)
    lam[17], lam[2900] = 1.0, 1.0 - 1e-3
    sig = np.sqrt(lam).astype(np.float32).astype(np.float64)   # the stored float32 values
    top = float(np.max(sig) ** 2)
    rp = np.arange(N + 1, dtype=np.int64)
    th = W.Theta.from_csr(n, "haar", J, rp, np.arange(N, dtype=np.int32), sig)
    start = synth.power_start(N, 9)
    Lp, it = th.lipschitz(start, max_iters=5000, require=False)
    assert it == 5000 and Lp < top
    with pytest.raises(W.WdbError):
        th.lipschitz(start, max_iters=5000)
    r = th.lipschitz_lanczos(start)
    print(f"Lanczos: {r}; power iteration {Lp!r} after {it}", flush=True)
    assert r["converged"] and r["steps"] < 5000
    assert abs(r["theta"] - top) <= 1e-12 * top and r["L"] >= top * (1 - 1e-15)
    r = th.lipschitz_lanczos(start, max_steps=10)
    assert not r["converged"] and r["steps"] == 10 and r["theta"] <= top * (1 + 1e-15)


@pytest.mark.parametrize("n,gap,tol", [(4, 1.0, 1e-12), (4, 1.0, 0.0), (8, 1e-4, 1e-12), (16, 1e-6, 1e-12),
                                        (32, 1e-6, 0.0)])
def test_lanczos_restarts_reach_the_top_singular_value(W, n, gap, tol):
    """A basis as large as the space, several restarts towards clustered top
    values, and runs on past convergence (tol = 0: the run either meets an
    exactly invariant space or takes all its steps, in many cycles)."""
    N = n * n
    rng = np.random.default_rng(n)
    U, V = (np.linalg.qr(rng.standard_normal((N, N)))[0] for _ in range(2))
    sig = np.concatenate([1.0 - gap * np.arange(4), rng.uniform(0.0, 0.9, N - 4)]).clip(0.0)
    A = ((U * sig) @ V.T).astype(np.float32).astype(np.float64)
    th = W.Theta.from_csr(n, "haar", 1, np.arange(N + 1, dtype=np.int64) * N,
                          np.tile(np.arange(N, dtype=np.int32), N), A.ravel())
    ev = np.linalg.norm(A, 2) ** 2
    r = th.lipschitz_lanczos(synth.power_start(N, 3), tol=tol, max_steps=400)
    print(f"n={n} tol={tol}: {r}", flush=True)
    assert r["converged"] or (tol == 0.0 and r["steps"] == 400)
    assert abs(r["theta"] - ev) <= 1e-12 * ev and r["resid"] <= max(tol, 1e-12) * ev


@pytest.mark.parametrize("layout", [None, (8, 3)])
def test_objective_and_gap_match_oracle(W, p64, layout):
    """The float64 stopping test on the default layout and on the tiled one
    (its own float64 tile kernels), with uniform and scale weights."""
    th = imported(W, p64)
    if layout:
        th.set_kernel_layout(*layout)
    A32 = p64["A32"]
    x0 = p64["x0"].astype(np.float32)
    lam = p64["wl"].lam
    for seed in (0, 1):
        x = (np.random.default_rng(seed).standard_normal(4096) * 0.01).astype(np.float32)
        E, rel = th.objective(dev(x), dev(x0), lam)
        Eo, Do, gap, relo = fista.duality_gap(A32, x0.astype(np.float64), np.float64(np.float32(lam)), x.astype(np.float64))
        assert abs(E - Eo) <= 1e-12 * Eo
        assert abs(rel - relo) <= 1e-10
    th.set_l1_weights("scale")
    w = dwt.scale_index(64, 3).astype(np.float64)
    x = (np.random.default_rng(2).standard_normal(4096) * 0.01).astype(np.float32)
    E, rel = th.objective(dev(x), dev(x0), lam)
    Eo, Do, gap, relo = fista.duality_gap(A32, x0.astype(np.float64), np.float64(np.float32(lam)), x.astype(np.float64),
                                          w=w)
    assert abs(E - Eo) <= 1e-12 * Eo
    assert abs(rel - relo) <= 1e-10


def test_cached_graph_replays_and_follows_changes(W, p64):
    """A graph-replayed solve keeps its instantiated graph in the handle: a
    second solve with the same parameters replays it, other parameters or any
    change of the handle (layout, preconditioner, weights) capture a new one;
    every result equals the solve without a graph, bit for bit."""
    th = imported(W, p64)
    th.set_kernel_layout(8, 3)
    wl = p64["wl"]
    start = synth.power_start(4096, wl.power_seed)
    th.lipschitz(start)
    x0 = dev(p64["x0"].astype(np.float32))
    out = torch.empty(4096, device="cuda")

    def both(lam, **kw):
        ref, _ = th.solve_coeffs(x0, lam, 100, check_every=20, **kw)
        ref = host(ref)
        for _ in range(2):   # capture, then replay of the cached graph
            x, _ = th.solve_coeffs(x0, lam, 100, check_every=20, use_graph=True, out=out, **kw)
            assert np.array_equal(host(x), ref)
        return ref

    a = both(wl.lam)
    b = both(2 * wl.lam)
    assert not np.array_equal(a, b)
    th.set_kernel_layout(8, 4)
    both(wl.lam)
    th.set_precond("spai_scale", start=start)
    both(wl.lam, precond=True)
    th.set_l1_weights("scale")
    both(wl.lam, precond=True)
    both(wl.lam, ista=True)


def test_recorded_checks_match_synchronous_checks(W, p64):
    """Without a stopping test the checks are read once at the end; the trace
    equals the one of a solve whose stopping test never fires (synchronous
    checks), check by check."""
    th = imported(W, p64)
    th.set_kernel_layout(8, 3)
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    x0 = p64["x0"].astype(np.float32)
    xa, ia = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=20, trace_cap=20)
    xb, ib = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=20, trace_cap=20, tol=1e-300)
    assert np.array_equal(ia["trace"], ib["trace"]) and ia["objective"] == ib["objective"]
    assert np.array_equal(host(xa), host(xb))


# ---------------------------------------------------------------------------
# the solver
# ---------------------------------------------------------------------------
def _oracle_fista(P, iters, x0=None, p=None, Lp=None):
    A32 = P["A32"]
    wl = P["wl"]
    x0 = P["x0"].astype(np.float32).astype(np.float64) if x0 is None else x0
    lam = float(np.float32(wl.lam))
    if p is None:
        L, _ = lipschitz.lipschitz(A32, synth.power_start(4096, wl.power_seed))
    else:
        L = Lp
    x, _, _ = fista.fista(A32, x0, lam, 1.0 / L, iters, p=p)
    return x, fista.objective(A32, x0, lam, x)


def _gate(A32, x0, lam, x_gpu, x_o, E_o):
    E_g = fista.objective(A32, x0, lam, x_gpu)
    assert abs(E_g - E_o) <= 1e-5 * E_o, (E_g, E_o)
    assert np.linalg.norm(x_gpu - x_o) <= 1e-4 * np.linalg.norm(x_o)


def test_fista_200_iterations_parity(W, p64):
    th = imported(W, p64)
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    x0 = p64["x0"].astype(np.float32)
    x, info = th.solve_coeffs(dev(x0), wl.lam, wl.iters, check_every=20, trace_cap=20)
    assert info["iters"] == 200 and info["checks"] == 10
    x_o, E_o = _oracle_fista(p64, wl.iters)
    _gate(p64["A32"], x0.astype(np.float64), float(np.float32(wl.lam)), host(x), x_o, E_o)
    # the trace is the float64 objective of the iterates
    assert abs(info["trace"][-1, 1] - info["objective"]) == 0.0
    assert np.all(np.diff(info["trace"][:, 0]) == 20)


def test_end_to_end_parity64(W, p64):
    """GPU build + GPU transform + GPU solve against the oracle pipeline."""
    wl = p64["wl"]
    th = W.build_theta(wl.psf(), wl.wavelet, wl.levels, wl.nnz)
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    u0 = p64["u0"]
    x, info = th.solve(dev(u0).reshape(-1), wl.lam, wl.iters, check_every=50)
    x_o, E_o = _oracle_fista(p64, wl.iters)
    _gate(p64["A32"], p64["x0"], float(np.float32(wl.lam)), host(x), x_o, E_o)
    img = host(th.synthesize(x)).reshape(64, 64)
    assert np.max(np.abs(img - dwt.idwt2(host(x), filters.haar(), 3, 64))) <= 1e-5


def test_solver_is_deterministic_and_graph_matches_eager(W, p64):
    th = imported(W, p64)
    wl = p64["wl"]
    x0 = dev(p64["x0"])
    a, _ = th.solve_coeffs(x0, wl.lam, 120, check_every=20)
    b, _ = th.solve_coeffs(x0, wl.lam, 120, check_every=20)
    c, _ = th.solve_coeffs(x0, wl.lam, 120, check_every=20, use_graph=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert torch.equal(a, c)


def test_resume_matches_single_run(W, p64):
    """x^(k) only depends on (x, x_prev, k); resuming from x^(60) with k0 = 61 and
    y = x^(60) differs from one run only through the momentum term, so compare
    the resumed path with the oracle doing the same thing."""
    th = imported(W, p64)
    wl = p64["wl"]
    x0 = p64["x0"].astype(np.float32)
    x60, _ = th.solve_coeffs(dev(x0), wl.lam, 60, check_every=0)
    x, _ = th.solve_coeffs(dev(x0), wl.lam, 40, check_every=0, x_init=x60, k0=61)
    A32 = p64["A32"]
    lam = float(np.float32(wl.lam))
    L, _ = lipschitz.lipschitz(A32, synth.power_start(4096, wl.power_seed))
    xo60, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1 / L, 60)
    xo, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1 / L, 40, x_init=xo60, k0=61)
    assert np.linalg.norm(host(x) - xo) <= 1e-4 * np.linalg.norm(xo)


def test_tolerance_stop(W, p64):
    """The stopping test scores the float64 iterate (the anchor), returned in
    x64_out; x_out is its float32 rounding, with the same objective to
    rounding.  The plain float32 iterate is scored as it is."""
    th = imported(W, p64)
    wl = p64["wl"]
    A32, lam = p64["A32"], float(np.float32(wl.lam))
    x0 = p64["x0"].astype(np.float32).astype(np.float64)
    x64 = torch.empty(4096, device="cuda", dtype=torch.float64)
    x, info = th.solve_coeffs(dev(p64["x0"]), wl.lam, 5000, check_every=20, tol=1e-3, x64_out=x64)
    assert info["converged"] and info["rel_gap"] <= 1e-3 and info["iters"] % 20 == 0
    E, D, gap, rel = fista.duality_gap(A32, x0, lam, host(x64))
    assert abs(rel - info["rel_gap"]) <= 1e-9 and abs(E - info["objective"]) <= 1e-12 * E
    assert np.array_equal(host(x), host(x64).astype(np.float32).astype(np.float64))
    assert abs(fista.objective(A32, x0, lam, host(x)) - E) <= 1e-9 * E
    xp, ip = th.solve_coeffs(dev(p64["x0"]), wl.lam, 5000, check_every=20, tol=1e-3, plain_iterate=True,
                             x64_out=x64)
    assert ip["converged"]
    E, D, gap, rel = fista.duality_gap(A32, x0, lam, host(xp))
    assert abs(rel - ip["rel_gap"]) <= 1e-9 and np.array_equal(host(x64), host(xp))
    x, info = th.solve_coeffs(dev(p64["x0"]), wl.lam, 20, check_every=20, tol=1e-9)
    assert not info["converged"]


def test_graph_solve_stops_on_the_checked_iterate(W, p64):
    """With graph replay and the anchored iterate the block after a check is
    enqueued before the host reads the check.  A stop must still return the
    checked iterate: the same float32 and float64 iterates, iteration count,
    objective and gap as the eager solve, and the oracle's gap of that
    iterate."""
    th = imported(W, p64)
    wl = p64["wl"]
    A32, lam = p64["A32"], float(np.float32(wl.lam))
    outs = []
    for g in (False, True):
        x64 = torch.empty(4096, device="cuda", dtype=torch.float64)
        x, info = th.solve_coeffs(dev(p64["x0"]), wl.lam, 5000, check_every=20, tol=1e-3, use_graph=g,
                                  x64_out=x64)
        torch.cuda.synchronize()
        outs.append((host(x), host(x64), info))
    (xa, ya, ia), (xb, yb, ib) = outs
    assert ia["converged"] and ib["converged"] and 40 <= ia["iters"] < 5000
    assert ia["iters"] == ib["iters"] and ia["objective"] == ib["objective"] and ia["rel_gap"] == ib["rel_gap"]
    assert np.array_equal(xa, xb) and np.array_equal(ya, yb)
    E, D, gap, rel = fista.duality_gap(A32, p64["x0"].astype(np.float32).astype(np.float64), lam, yb)
    assert abs(rel - ib["rel_gap"]) <= 1e-9


@pytest.fixture(scope="module")
def db4_32():
    """Small db4 problem with large approximation coefficients relative to
    lambda (3 levels, lambda 5e-4): the float32 iterate's rounding sets a gap
    floor near 1e-3 here."""
    n, J, lam = 32, 3, 5e-4
    h = filters.db4()
    field = synth.psf_rotating(n, 3.0, 1.0)
    T = theta.theta_dense(field, h, J)
    r, c, v = theta.top_k(T, 20 * n * n)
    A32 = sp.csr_matrix((v.astype(np.float32).astype(np.float64), (r, c)), shape=(n * n, n * n))
    u0 = blur.observe(field, synth.piecewise_image(n, 1), synth.noise(n, 0.005, 2))
    x0 = dwt.dwt2(u0, h, J).astype(np.float32)
    return dict(n=n, J=J, lam=lam, A32=A32, x0=x0, rcv=(r, c, v))


def test_anchored_iterate_follows_the_float64_gap(W, db4_32):
    """Alg. 1 with the float64 anchor certifies the duality gap the float64
    oracle's own iterates reach (here about 1e-5 after 10000 iterations),
    while the plain float32 iterate stalls at its rounding floor.  The gap of
    the returned float64 iterate is recomputed by the oracle."""
    P = db4_32
    n, lam = P["n"], float(np.float32(P["lam"]))
    A32, x0 = P["A32"], P["x0"].astype(np.float64)
    rp, cc, vv = theta.csr_arrays(A32)
    th = W.Theta.from_csr(n, "db4", P["J"], rp, cc, vv)
    start = synth.power_start(n * n, 3)
    L, _ = th.lipschitz(start)
    iters, c = 10000, 500
    x64 = torch.empty(n * n, device="cuda", dtype=torch.float64)
    _, ia = th.solve_coeffs(dev(P["x0"]), lam, iters, check_every=c, trace_cap=iters // c, x64_out=x64)
    _, ip = th.solve_coeffs(dev(P["x0"]), lam, iters, check_every=c, trace_cap=iters // c, plain_iterate=True)
    gaps_o = []

    def cb(k, x):
        if k % c == 0:
            gaps_o.append(fista.duality_gap(A32, x0, lam, x)[3])
    Lo, _ = lipschitz.lipschitz(A32, start)
    fista.fista(A32, x0, lam, 1.0 / Lo, iters, callback=cb)
    ga, gp, go = ia["trace"][:, 2], ip["trace"][:, 2], np.array(gaps_o)
    assert go[-1] <= 3e-5                                 # the float64 iteration's own gap
    assert ga[-1] <= 1.5 * go[-1]                         # anchored: follows it
    assert np.min(gp) >= 10 * go[-1]                      # float32 iterate: stalls at its floor
    assert np.all(ga <= 1.5 * go + 1e-7)
    E, D, gap, rel = fista.duality_gap(A32, x0, lam, host(x64))
    assert abs(rel - ia["rel_gap"]) <= 1e-9


@pytest.mark.parametrize("kind", ["spai", "spai_scale", "jacobi"])
def test_preconditioner_matches_oracle(W, p64, kind):
    th = imported(W, p64)
    wl = p64["wl"]
    A32 = p64["A32"]
    start = synth.power_start(4096, wl.power_seed)
    th.set_precond(kind, eps=0.05, start=start)
    p = th.precond()
    if kind == "spai":
        po = precond.spai(A32)
    elif kind == "jacobi":
        po = precond.jacobi(A32, 0.05)
    else:
        po = precond.spai_grouped(A32, precond.scale_groups(64, 3))
    assert np.max(np.abs(p - po) / po) <= 1e-10
    Lp, _ = lipschitz.lipschitz_precond(A32, po, start)
    assert abs(th.info()["lipschitz_p"] - Lp) <= 1e-9 * Lp
    x0 = p64["x0"].astype(np.float32)
    x, info = th.solve_coeffs(dev(x0), wl.lam, 100, check_every=20, precond=True)
    x_o, E_o = _oracle_fista(p64, 100, p=po, Lp=Lp)
    _gate(A32, x0.astype(np.float64), float(np.float32(wl.lam)), host(x), x_o, E_o)


@pytest.mark.parametrize("pre", [False, True])
def test_ista_matches_oracle(W, p64, pre):
    """ISTA (no extrapolation; the un-accelerated baseline of Sec. 5) against the oracle."""
    th = imported(W, p64)
    wl = p64["wl"]
    start = synth.power_start(4096, wl.power_seed)
    th.lipschitz(start)
    A32 = p64["A32"]
    p = Lp = None
    if pre:
        th.set_precond("spai_scale", start=start)
        p = precond.spai_grouped(A32, precond.scale_groups(64, 3))
        Lp, _ = lipschitz.lipschitz_precond(A32, p, start)
    x0 = p64["x0"].astype(np.float32)
    lam = float(np.float32(wl.lam))
    xg, info = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50, precond=pre, ista=True)
    L, _ = lipschitz.lipschitz(A32, start)
    xo = fista.ista(A32, x0.astype(np.float64), lam, 1.0 / (Lp if pre else L), 200, p=p)
    _gate(A32, x0.astype(np.float64), lam, host(xg), xo, fista.objective(A32, x0.astype(np.float64), lam, xo))
    # and it is slower than Alg. 1 on the same problem: FISTA's objective after 200 is lower
    xf, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50, precond=pre)
    assert fista.objective(A32, x0.astype(np.float64), lam, host(xf)) < fista.objective(A32, x0.astype(np.float64), lam, host(xg))


# ---------------------------------------------------------------------------
# l1 weights w[i] = j(i) (the weights of the experiments of Sec. 5)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("pre", [False, True])
def test_weighted_l1_solve_matches_oracle(W, p64, pre):
    th = imported(W, p64)
    wl = p64["wl"]
    start = synth.power_start(4096, wl.power_seed)
    th.lipschitz(start)
    A32 = p64["A32"]
    w = dwt.scale_index(64, 3).astype(np.float64)
    th.set_l1_weights("scale")
    assert th.info()["l1_weights"] == 1
    p = Lp = None
    if pre:
        th.set_precond("spai_scale", start=start)
        p = precond.spai_grouped(A32, precond.scale_groups(64, 3))
        Lp, _ = lipschitz.lipschitz_precond(A32, p, start)
    x0 = p64["x0"].astype(np.float32)
    lam = float(np.float32(wl.lam))
    x64 = torch.empty(4096, device="cuda", dtype=torch.float64)
    xg, info = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50, precond=pre, x64_out=x64)
    L, _ = lipschitz.lipschitz(A32, start)
    xo, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1.0 / (Lp if pre else L), 200, p=p, w=w)
    Eo = fista.objective(A32, x0.astype(np.float64), lam, xo, w)
    Eg = fista.objective(A32, x0.astype(np.float64), lam, host(xg), w)
    assert abs(Eg - Eo) <= 1e-5 * Eo
    assert np.linalg.norm(host(xg) - xo) <= 1e-4 * np.linalg.norm(xo)
    # the float64 check is the weighted objective and gap of the float64 iterate
    E, _, _, rel = fista.duality_gap(A32, x0.astype(np.float64), lam, host(x64), w)
    assert abs(info["objective"] - E) <= 1e-10 * E and abs(info["rel_gap"] - rel) <= 1e-9
    # uniform weights again give the unweighted solve
    th.set_l1_weights("uniform")
    if pre:
        th.set_precond("none")
    xu, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50)
    x_o, E_o = _oracle_fista(p64, 200)
    _gate(A32, x0.astype(np.float64), lam, host(xu), x_o, E_o)


# ---------------------------------------------------------------------------
# mixed precision: 16-bit values, float32 accumulation
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_mixed_precision_matches_oracle_on_dequantised_theta(W, p64, fmt):
    from oracle import quant
    th = imported(W, p64)
    wl = p64["wl"]
    start = synth.power_start(4096, wl.power_seed)
    L, _ = th.lipschitz(start)
    th.set_precision(fmt)
    assert th.info()["valtype"] == {"f16": 2, "bf16": 1}[fmt]
    Q = quant.quantize(p64["A"], 64, 3, fmt)
    # one product with the 16-bit values
    x = np.random.default_rng(8).standard_normal(4096).astype(np.float32)
    b = np.random.default_rng(9).standard_normal(4096).astype(np.float32)
    y = host(th.apply(dev(x), dev(b)))
    ref = Q @ x.astype(np.float64) - b
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref))
    # 200 iterations against the oracle on the dequantised operator (same step 1/L)
    x0 = p64["x0"].astype(np.float32)
    lam = float(np.float32(wl.lam))
    xg, info = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=20)
    Lo, _ = lipschitz.lipschitz(p64["A32"], start)
    assert abs(L - Lo) <= 1e-9 * Lo
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), lam, 1.0 / Lo, 200)
    _gate(Q, x0.astype(np.float64), lam, host(xg), xo, fista.objective(Q, x0.astype(np.float64), lam, xo))
    # the float64 check scores the iterate against the unquantised operator
    Eu = fista.objective(p64["A32"], x0.astype(np.float64), lam, host(xg))
    assert abs(info["objective"] - Eu) <= 1e-10 * Eu
    # error of the 16-bit form against the float64 oracle solve, reported
    x64, E64 = _oracle_fista(p64, 200)
    print(f"{fmt}: rel objective vs FP64 oracle {abs(Eu - E64) / E64:.3e}, "
          f"rel ||x - x64|| {np.linalg.norm(host(xg) - x64) / np.linalg.norm(x64):.3e}")
    th.set_precision("f32")
    assert th.info()["valtype"] == 0


@pytest.fixture(scope="module")
def db4_64():
    """Oracle problem on 64x64 with the 8-tap filter (3 levels) and a rotating
    anisotropic field: exercises the packed column code's centring for L = 8."""
    field = synth.psf_rotating(64, 3.0, 1.0)
    h = filters.db4()
    T = theta.theta_dense(field, h, 3)
    r, c, v = theta.top_k(T, 30 * 4096)
    A = theta.to_csr(r, c, v, 4096)
    u0 = (blur.blur(field, synth.piecewise_image(64, 31)) + synth.noise(64, 0.01, 32)).astype(np.float32)
    return {"A": A, "x0": dwt.dwt2(u0.astype(np.float64), h, 3)}


def test_packed_16bit_sym6_matches_oracle(W):
    """The column code with the 12-tap filter's centring (L - 1 = 11)."""
    from oracle import quant
    field = synth.psf_rotating(64, 3.0, 1.0)
    h = filters.sym6()
    T = theta.theta_dense(field, h, 2)
    r, c, v = theta.top_k(T, 30 * 4096)
    A = theta.to_csr(r, c, v, 4096)
    rp, cc, vv = theta.csr_arrays(A)
    th = W.Theta.from_csr(64, "sym6", 2, rp, cc, vv)
    th.set_precision("f16")
    Q = quant.quantize(A, 64, 2, "f16")
    x = np.random.default_rng(28).standard_normal(4096).astype(np.float32)
    y = host(th.apply(dev(x)))
    ref = Q @ x.astype(np.float64)
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
def test_packed_16bit_db4_matches_oracle(W, db4_64, fmt):
    from oracle import quant
    A = db4_64["A"]
    rp, cc, vv = theta.csr_arrays(A)
    th = W.Theta.from_csr(64, "db4", 3, rp, cc, vv)
    start = synth.power_start(4096, 5)
    L, _ = th.lipschitz(start)
    th.set_precision(fmt)
    info = th.info()
    assert info["group16"] > 0 and info["escapes"] == 0
    Q = quant.quantize(A, 64, 3, fmt)
    x = np.random.default_rng(18).standard_normal(4096).astype(np.float32)
    b = np.random.default_rng(19).standard_normal(4096).astype(np.float32)
    ref = Q @ x.astype(np.float64) - b
    for G in (2, 4, 8, 16):   # every lane count of the packed kernels gives the same product
        th.set_packed_group(G)
        y = host(th.apply(dev(x), dev(b)))
        assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)), G
    th.set_packed_group(0)
    lam = 1e-3
    x0 = db4_64["x0"].astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), lam, 150, check_every=50)
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    Lo, _ = lipschitz.lipschitz(A32, start)
    lam32 = float(np.float32(lam))
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), lam32, 1.0 / Lo, 150)
    _gate(Q, x0.astype(np.float64), lam32, host(xg), xo, fista.objective(Q, x0.astype(np.float64), lam32, xo))


@pytest.mark.parametrize("fmt,waves,unroll", [("f16", 1, 1), ("f16", 4, 2), ("bf16", 2, 2), ("bf16", 8, 1)])
def test_tiled_16bit_db4_matches_oracle(W, db4_64, fmt, waves, unroll):
    """16-bit tiled layout (group16 3): products against the oracle's quantised
    operator, Alg. 1 and Alg. 2 (per-scale P, scale weights) solves."""
    from oracle import quant
    A = db4_64["A"]
    rp, cc, vv = theta.csr_arrays(A)
    th = W.Theta.from_csr(64, "db4", 3, rp, cc, vv)
    start = synth.power_start(4096, 5)
    th.lipschitz(start)
    th.set_precision(fmt)
    th.set_packed_group(3)
    th.set_tile_shape(waves, unroll)
    info = th.info()
    assert info["group16"] == 3 and info["tile_waves16"] == waves and info["tile_unroll16"] == unroll
    Q = quant.quantize(A, 64, 3, fmt)
    x = np.random.default_rng(18).standard_normal(4096).astype(np.float32)
    b = np.random.default_rng(19).standard_normal(4096).astype(np.float32)
    ref = Q @ x.astype(np.float64) - b
    y = host(th.apply(dev(x), dev(b)))
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref))
    lam = 1e-3
    lam32 = float(np.float32(lam))
    x0 = db4_64["x0"].astype(np.float32)
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    xg, _ = th.solve_coeffs(dev(x0), lam, 150, check_every=50)
    Lo, _ = lipschitz.lipschitz(A32, start)
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), lam32, 1.0 / Lo, 150)
    _gate(Q, x0.astype(np.float64), lam32, host(xg), xo, fista.objective(Q, x0.astype(np.float64), lam32, xo))
    th.set_precond("spai_scale", start=start)
    th.set_l1_weights("scale")
    assert th.info()["group16"] == 3
    p = precond.spai_grouped(A32, precond.scale_groups(64, 3))
    Lp, _ = lipschitz.lipschitz_precond(A32, p, start)
    w = dwt.scale_index(64, 3).astype(np.float64)
    xp, _ = th.solve_coeffs(dev(x0), lam, 150, check_every=50, precond=True)
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), lam32, 1.0 / Lp, 150, p=p, w=w)
    Eo = fista.objective(Q, x0.astype(np.float64), lam32, xo, w=w)
    Eg = fista.objective(Q, x0.astype(np.float64), lam32, host(xp), w=w)
    assert abs(Eg - Eo) <= 1e-5 * Eo
    assert np.linalg.norm(host(xp) - xo) <= 1e-4 * np.linalg.norm(xo)


def test_packed_escapes_match_oracle(W):
    """Columns far from the row's position (random, seeded) do not fit the
    16-bit code and are read from the per-row escape lists (the level-1
    subbands of a 128 x 128 image are 64 wide, beyond the code's +-22)."""
    from oracle import quant
    n, J, N = 128, 2, 16384
    rng = np.random.default_rng(23)
    rows, cols = [], []
    for r in range(N):
        near = (r + rng.integers(-3, 4, 6)) % N          # mostly same-band neighbours (some escape too)
        far = rng.integers(0, N, rng.integers(0, 4))     # arbitrary columns
        cs = np.unique(np.concatenate([near, far]))
        rows.append(np.full(cs.size, r))
        cols.append(cs)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    vals = rng.standard_normal(rows.size) * 0.1
    A = sp.csr_matrix((vals, (rows, cols)), shape=(N, N))
    A.sort_indices()
    th = W.Theta.from_csr(n, "haar", J, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data)
    th.set_precision("f16")
    assert th.info()["escapes"] > 0
    Q = quant.quantize(A, n, J, "f16")
    x = rng.standard_normal(N).astype(np.float32)
    for G in (2, 4, 8, 16):
        th.set_packed_group(G)
        y = host(th.apply(dev(x)))
        ref = Q @ x.astype(np.float64)
        assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)), G
    # the transposed packed product runs inside the solver: compare 50 iterations
    th.set_packed_group(4)
    start = synth.power_start(N, 6)
    th.lipschitz(start)
    x0 = rng.standard_normal(N).astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), 0.05, 50, check_every=0)
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    Lo, _ = lipschitz.lipschitz(A32, start)
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), float(np.float32(0.05)), 1.0 / Lo, 50)
    _gate(Q, x0.astype(np.float64), float(np.float32(0.05)), host(xg), xo,
          fista.objective(Q, x0.astype(np.float64), float(np.float32(0.05)), xo))


# ---------------------------------------------------------------------------
# batched solve (packs of 8 right-hand sides per operator, one launch per phase)
# ---------------------------------------------------------------------------
@pytest.fixture(scope="module")
def small32():
    field = synth.psf_isotropic(32, 1.0, 2.5)
    h = filters.haar()
    T = theta.theta_dense(field, h, 2)
    r, c, v = theta.top_k(T, 20 * 1024)
    A = theta.to_csr(r, c, v, 1024)
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    return {"field": field, "h": h, "A": A, "A32": A32, "H": blur.blur_matrix(field)}


@pytest.mark.parametrize("layout", ["sell", "dense", "kept"])
def test_batched_packs_equal_packs_of_one(W, layout):
    """Packs of 8, 4, 2 and 1 problems of two operators in one batch, their blocks
    dealt in turns and padded to whole turns: every problem's iterate is that of
    a batch of its own, to the last bit (the same sums in the same order)."""
    ths = []
    for n, J in ((32, 2), (64, 3)):
        th = W.build_theta(synth.psf_rotating(n, 2.5, 1.0), "haar", J, 20 * n * n + 5)
        th.lipschitz_lanczos()
        if layout == "sell":
            th.set_kernel_layout(16, 0)
        else:
            th.set_kernel_layout(8, 3)
            th.set_tile_values(layout == "kept")
        ths.append(th)
    rng = np.random.default_rng(3)
    probs = []
    for i in range(8 + 4 + 10):   # 12 of the first operator (8 + 4), 10 of the second (8 + 2)
        th = ths[0] if i < 12 else ths[1]
        probs.append((th, dev(rng.random(th.N)), 1e-3 * (1 + i % 3)))
    xs, infos = W.solve_batched(probs, 45, check_every=20)
    for i, p in enumerate(probs):
        x1, info1 = W.solve_batched([p], 45, check_every=20)
        assert np.array_equal(host(xs[i]), host(x1[0])), i
        assert abs(infos[i]["objective"] - info1[0]["objective"]) <= 1e-12 * info1[0]["objective"]


@pytest.mark.parametrize("layout", ["sell", "dense", "kept"])
@pytest.mark.parametrize("n,count,checked", [(64, 17, (0, 9, 15, 16)), (64, 26, (3, 23, 24, 25)),
                                             (256, 59, (0, 8, 55, 58)), (512, 9, (7, 8)), (512, 11, (0, 10)),
                                             (512, 26, (3, 24, 25))])
def test_batched_packs_of_every_arrangement_keep_the_iterates(W, layout, n, count, checked):
    """Packs of an operator that take turns, the last of them of one, two or four
    slots, and (9 and 11 problems of 512 x 512) a second pack by itself, with loads ahead
    and planes and (26 of 512 x 512) without: a problem's iterate is that of a batch of its own, to the last bit, and it stops at the same check."""
    th = W.build_theta(synth.psf_rotating(n, 2.5, 1.0), "haar", 3, 12 * n * n + 5)
    th.lipschitz_lanczos()
    if layout == "sell":
        th.set_kernel_layout(16, 0)
    else:
        th.set_kernel_layout(8, 3)
        th.set_tile_values(layout == "kept")
    g = torch.Generator("cuda").manual_seed(n + count)
    probs = [(th, torch.rand(th.N, device="cuda", generator=g), 1e-3 * (1 + i % 5)) for i in range(count)]
    xs, infos = W.solve_batched(probs, 30, check_every=10, tol=0.05)
    for i in checked:
        x1, info1 = W.solve_batched([probs[i]], 30, check_every=10, tol=0.05)
        assert torch.equal(xs[i], x1[0]), i
        assert infos[i]["iters"] == info1[0]["iters"], i


@pytest.mark.parametrize("layout", ["sell", "dense", "kept"])
def test_batched_with_a_large_operator_keeps_the_iterates(W, layout):
    """A batch that holds a problem of more than 512 x 512 coefficients runs the
    kernels without loads ahead and planes: the small problems' iterates stay
    those of a batch of their own, to the last bit, and the large one (the
    identity, for which Alg. 1 thresholds x0 in its first step) is exact."""
    n = 1024
    N = n * n
    one = W.Theta.from_csr(n, "haar", 1, np.arange(N + 1, dtype=np.int64), np.arange(N, dtype=np.int32), np.ones(N))
    one.lipschitz_lanczos()
    th = W.build_theta(synth.psf_rotating(64, 2.5, 1.0), "haar", 3, 20 * 4096 + 5)
    th.lipschitz_lanczos()
    for t in (one, th):
        if layout == "sell":
            t.set_kernel_layout(16, 0)
        else:
            t.set_kernel_layout(8, 3)
            t.set_tile_values(layout == "kept")
    rng = np.random.default_rng(5)
    small = [(th, dev(rng.standard_normal(4096)), 1e-3 * (1 + i)) for i in range(6)]
    big = (one, dev(rng.standard_normal(N)), 0.5)
    xs, infos = W.solve_batched(small[:3] + [big] + small[3:], 45, check_every=20, coeffs=True)
    alone, inf1 = W.solve_batched(small, 45, check_every=20, coeffs=True)
    for i, (x, info) in enumerate(zip(xs[:3] + xs[4:], infos[:3] + infos[4:])):
        assert np.array_equal(host(x), host(alone[i])), i
        assert abs(info["objective"] - inf1[i]["objective"]) <= 1e-12 * inf1[i]["objective"]
    x0 = host(big[1])
    # tau = 1 / L and L = 1 to 1e-12: float32 rounding of the step alone
    assert np.max(np.abs(host(xs[3]) - np.sign(x0) * np.maximum(np.abs(x0) - 0.5, 0.0))) <= 2e-6


@pytest.mark.parametrize("tiled", [False, True, "kept"])
def test_batched_narrowing_keeps_the_iterates(W, p64, tiled):
    """A pack narrows (8 -> 4 -> 2 -> 1 slots) as its problems stop; that must
    change only the cost: each problem's float64 iterate and stopping
    iteration equal those of the same problem solved alone (a pack of one),
    bit for bit, since every slot keeps its own sums in the same order.  The
    tiled runs use the dense and the kept-value layouts."""
    th = imported(W, p64)
    if tiled:
        th.set_kernel_layout(8, 3)
        th.set_tile_values(tiled == "kept")
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, 3))
    H = blur.blur_matrix(wl.psf())
    probs = []
    for i in range(7):
        u0 = (blur.blur(None, synth.piecewise_image(64, 300 + i), H) + synth.noise(64, 0.01, 400 + i)).astype(np.float32)
        probs.append((th, dev(u0).reshape(-1), float(np.float32(10.0 ** (-3.6 + 0.25 * i)))))
    o_all = [torch.empty(4096, device="cuda", dtype=torch.float64) for _ in probs]
    _, inf_all = W.solve_batched(probs, 4000, check_every=10, tol=1e-3, outs64=o_all)
    its = [r["iters"] for r in inf_all]
    assert len(set(its)) >= 3, its          # the pack narrows more than once
    for i, p in enumerate(probs):
        o1 = [torch.empty(4096, device="cuda", dtype=torch.float64)]
        _, inf1 = W.solve_batched([p], 4000, check_every=10, tol=1e-3, outs64=o1)
        assert inf1[0]["iters"] == its[i]
        assert torch.equal(o1[0], o_all[i]), i


@pytest.mark.parametrize("tiled64", [False, True, "kept"])
def test_batched_matches_oracle_per_problem(W, p64, small32, tiled64):
    """13 problems on two operators (chunks of 8 + 2 and 3); with tiled64 the
    64 x 64 operator's chunks run on its tiled copies (dense or kept values)
    while the 32 x 32 one stays on sliced ELL, in the same launches."""
    th64 = imported(W, p64)
    rp, cc, vv = theta.csr_arrays(small32["A"])
    th32 = W.Theta.from_csr(32, "haar", 2, rp, cc, vv)
    if tiled64:
        th64.set_kernel_layout(8, 3)
        th64.set_tile_values(tiled64 == "kept")
    wl = p64["wl"]
    start64, start32 = synth.power_start(4096, 3), synth.power_start(1024, 4)
    th64.lipschitz(start64)
    th32.lipschitz(start32)
    H64 = blur.blur_matrix(wl.psf())
    probs, oracle_inputs = [], []
    for i in range(13):
        if i < 10:
            n, th, H, A32, h, J, start = 64, th64, H64, p64["A32"], filters.haar(), 3, start64
        else:
            n, th, H, A32, h, J, start = 32, th32, small32["H"], small32["A32"], small32["h"], 2, start32
        u0 = (blur.blur(None, synth.piecewise_image(n, 100 + i), H) + synth.noise(n, 0.01, 200 + i)).astype(np.float32)
        lam = float(np.float32(10.0 ** (-3.5 + 0.15 * i)))
        probs.append((th, dev(u0).reshape(-1), lam))
        oracle_inputs.append((A32, dwt.dwt2(u0.astype(np.float64), h, J), lam, start))
    o64 = [torch.empty(p[0].N, device="cuda", dtype=torch.float64) for p in probs]
    c64 = [torch.empty(p[0].N, device="cuda", dtype=torch.float64) for p in probs]
    xs, infos = W.solve_batched(probs, 150, check_every=50, use_graph=True, outs64=o64)
    # the same problems with x0 handed over directly (the oracle's transform, in float32)
    x0s = [x0.astype(np.float32) for (_A, x0, _l, _s) in oracle_inputs]
    xc, infc = W.solve_batched([(p[0], dev(x0s[i]), p[2]) for i, p in enumerate(probs)], 150, check_every=50,
                               use_graph=True, coeffs=True, outs64=c64)
    for i, (A32, x0, lam, start) in enumerate(oracle_inputs):
        L, _ = lipschitz.lipschitz(A32, start)
        xo, _, _ = fista.fista(A32, x0, lam, 1.0 / L, 150)
        _gate(A32, x0, lam, host(xs[i]), xo, fista.objective(A32, x0, lam, xo))
        # From the image, the GPU scores against its own float32 transform of u0
        # (about 1e-6 absolute per coefficient away from the float64 one): E moves
        # by ~1e-7 relative, but the dual scaling s = lam / ||A^T r||_inf magnifies
        # the shift of the relative gap to ~2.5e-4 on these problems.
        E, _, _, rel = fista.duality_gap(A32, x0, lam, host(o64[i]))
        assert abs(infos[i]["objective"] - E) <= 1e-6 * E and abs(infos[i]["rel_gap"] - rel) <= 1e-3
        assert np.array_equal(host(xs[i]), host(o64[i]).astype(np.float32).astype(np.float64))
        # From identical float32 coefficients the float64 checks agree to rounding.
        x0f = x0s[i].astype(np.float64)
        xof, _, _ = fista.fista(A32, x0f, lam, 1.0 / L, 150)
        _gate(A32, x0f, lam, host(xc[i]), xof, fista.objective(A32, x0f, lam, xof))
        E, _, _, rel = fista.duality_gap(A32, x0f, lam, host(c64[i]))
        assert abs(infc[i]["objective"] - E) <= 1e-9 * E and abs(infc[i]["rel_gap"] - rel) <= 1e-8
    # per-problem stop flags: every problem ends below the tolerance, frozen at its own check
    xs, infos = W.solve_batched(probs, 3000, check_every=20, tol=2e-3, outs64=o64)
    assert all(r["converged"] for r in infos)
    its = [r["iters"] for r in infos]
    assert len(set(its)) > 1 and all(k % 20 == 0 for k in its)
    for i, (A32, x0, lam, start) in enumerate(oracle_inputs):
        _, _, _, rel = fista.duality_gap(A32, x0, lam, host(o64[i]))
        assert rel <= 2e-3 * (1 + 1e-6)
    # the anchored iterates certify gaps a float32 iterate cannot (its floor is
    # near 1e-4 on these problems): every problem to 1e-5, from the same float32
    # coefficients as the oracle, which recomputes each gap
    xs, infos = W.solve_batched([(p[0], dev(x0s[i]), p[2]) for i, p in enumerate(probs)], 40000,
                                check_every=100, tol=1e-5, outs64=c64, use_graph=True, coeffs=True)
    print("batched to 1e-5:", [(r["iters"], r["rel_gap"]) for r in infos], flush=True)
    assert all(r["converged"] for r in infos)
    for i, (A32, x0, lam, start) in enumerate(oracle_inputs):
        _, _, _, rel = fista.duality_gap(A32, x0s[i].astype(np.float64), lam, host(c64[i]))
        assert rel <= 1e-5 + 1e-8


# ---------------------------------------------------------------------------
# kernel layouts and the autotuner
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("slice_h,group", [(8, 0), (16, 0), (32, 0), (64, 0), (64, 4), (64, 8), (8, 16)])
def test_layouts_match_oracle(W, p64, slice_h, group):
    th = imported(W, p64)
    th.set_kernel_layout(slice_h, group)
    A32 = p64["A32"]
    rng = np.random.default_rng(slice_h + group)
    x = rng.standard_normal(4096).astype(np.float32)
    y = host(th.apply(dev(x), None))
    assert np.max(np.abs(y - A32 @ x)) <= 1e-5 * np.max(np.abs(A32 @ x))
    yt = host(th.apply(dev(x), None, transpose=True))
    assert np.max(np.abs(yt - A32.T @ x)) <= 1e-5 * np.max(np.abs(A32.T @ x))
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    x0 = p64["x0"].astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50)
    x_o, E_o = _oracle_fista(p64, 200)
    _gate(A32, x0.astype(np.float64), float(np.float32(wl.lam)), host(xg), x_o, E_o)
    # the 16-bit path and the preconditioner follow the slot layout
    th.set_precision("bf16")
    xb, _ = th.solve_coeffs(dev(x0), wl.lam, 20, check_every=0)
    assert np.all(np.isfinite(host(xb)))
    th.set_precond("spai_scale", start=synth.power_start(4096, wl.power_seed))
    po = precond.spai_grouped(A32, precond.scale_groups(64, 3))
    assert np.max(np.abs(th.precond() - po) / po) <= 1e-10


@pytest.mark.parametrize("waves,unroll,kept", [(1, 2, 0), (2, 4, 0), (4, 2, 0), (8, 4, 0),
                                               (2, 1, 1), (1, 2, 1), (4, 4, 1), (8, 1, 1)])
def test_tiled_layout_matches_oracle(W, p64, waves, unroll, kept):
    """Tiled pattern storage (layout 3), dense or kept values: products, FISTA,
    and the proximal epilogue with the preconditioner and scale weights,
    against the oracle."""
    th = imported(W, p64)
    th.set_kernel_layout(8, 3)
    th.set_tile_shape(waves, unroll)
    th.set_tile_values(kept)
    info = th.info()
    assert info["group"] == 3 and info["tile_unroll"] == unroll and info["tile_kept"] == kept
    assert info["tile_kept_values"] == 2 * p64["A32"].nnz   # every kept entry once per copy, no zeros
    A32 = p64["A32"]
    rng = np.random.default_rng(waves)
    x = rng.standard_normal(4096).astype(np.float32)
    y = host(th.apply(dev(x), None))
    assert np.max(np.abs(y - A32 @ x)) <= 1e-5 * np.max(np.abs(A32 @ x))
    yt = host(th.apply(dev(x), None, transpose=True))
    assert np.max(np.abs(yt - A32.T @ x)) <= 1e-5 * np.max(np.abs(A32.T @ x))
    wl = p64["wl"]
    start = synth.power_start(4096, wl.power_seed)
    th.lipschitz(start)
    x0 = p64["x0"].astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50)
    x_o, E_o = _oracle_fista(p64, 200)
    _gate(A32, x0.astype(np.float64), float(np.float32(wl.lam)), host(xg), x_o, E_o)
    # Alg. 2 with the per-scale preconditioner and the scale weights w[i] = j(i)
    th.set_precond("spai_scale", start=start)
    th.set_l1_weights("scale")
    p = precond.spai_grouped(A32, precond.scale_groups(64, 3))
    Lp, _ = lipschitz.lipschitz_precond(A32, p, start)
    w = dwt.scale_index(64, 3).astype(np.float64)
    lam = float(np.float32(wl.lam))
    xp, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50, precond=True)
    xo, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1.0 / Lp, 200, p=p, w=w)
    Eo = fista.objective(A32, x0.astype(np.float64), lam, xo, w=w)
    Eg = fista.objective(A32, x0.astype(np.float64), lam, host(xp), w=w)
    assert abs(Eg - Eo) <= 1e-5 * Eo
    assert np.linalg.norm(host(xp) - xo) <= 1e-4 * np.linalg.norm(xo)


def test_tiled_kept_values_match_dense_bit_for_bit(W, p64):
    """The kept-value layout adds the same products in the same order as the
    dense values (a missing entry contributes an exact 0 in both), so products,
    the float64 checks and whole solves agree bit for bit."""
    th = imported(W, p64)
    th.set_kernel_layout(8, 3)
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    x = np.random.default_rng(5).standard_normal(4096).astype(np.float32)
    x0 = p64["x0"].astype(np.float32)
    out = {}
    for kept in (0, 1):
        th.set_tile_values(kept)
        th.set_tile_shape(2, 1)
        y = host(th.apply(dev(x), dev(x0)))
        yt = host(th.apply(dev(x), transpose=True))
        xs, info = th.solve_coeffs(dev(x0), wl.lam, 120, check_every=20)
        out[kept] = (y, yt, host(xs), info["objective"], info["rel_gap"])
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(np.asarray(a), np.asarray(b))


def test_tiled_escapes_and_small_subbands_match_oracle(W):
    """A 128 x 128, 5-level operator: the coarsest subbands are 4 x 4 (one
    partial tile each); random far columns, and for some finest-level rows a
    column of the coarsest approximation (a level gap of 4, beyond the code),
    go to the escape lists."""
    n, J, N = 128, 5, 16384
    rng = np.random.default_rng(29)
    rows, cols = [], []
    for r in range(N):
        near = (r + rng.integers(-3, 4, 6)) % N
        far = rng.integers(0, N, rng.integers(0, 3))
        if r >= N // 4 and rng.random() < 0.05:   # a level-1 row: add an A_J coefficient (16 of them)
            far = np.concatenate([far, rng.integers(0, 16, 1)])
        cs = np.unique(np.concatenate([near, far]))
        rows.append(np.full(cs.size, r))
        cols.append(cs)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    vals = rng.standard_normal(rows.size) * 0.1
    A = sp.csr_matrix((vals, (rows, cols)), shape=(N, N))
    A.sort_indices()
    th = W.Theta.from_csr(n, "haar", J, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data)
    th.set_kernel_layout(8, 3)
    assert th.info()["tile_escapes"] > 0
    A32 = sp.csr_matrix((A.data.astype(np.float32).astype(np.float64), A.indices, A.indptr), shape=A.shape)
    x = rng.standard_normal(N).astype(np.float32)
    for waves, unroll, kept in ((1, 2, 0), (4, 2, 0), (1, 1, 1), (4, 2, 1)):
        th.set_tile_shape(waves, unroll)
        th.set_tile_values(kept)
        y = host(th.apply(dev(x)))
        ref = A32 @ x.astype(np.float64)
        assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref)), (waves, kept)
        yt = host(th.apply(dev(x), transpose=True))
        reft = A32.T @ x.astype(np.float64)
        assert np.max(np.abs(yt - reft)) <= 1e-5 * np.max(np.abs(reft)), (waves, kept)
    th.set_tile_shape(1, 2)
    th.set_tile_values(0)
    start = synth.power_start(N, 6)
    th.lipschitz(start)
    x0 = rng.standard_normal(N).astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), 0.05, 50, check_every=0)
    Lo, _ = lipschitz.lipschitz(A32, start)
    lam = float(np.float32(0.05))
    xo, _, _ = fista.fista(A32, x0.astype(np.float64), lam, 1.0 / Lo, 50)
    _gate(A32, x0.astype(np.float64), lam, host(xg), xo, fista.objective(A32, x0.astype(np.float64), lam, xo))
    # the 16-bit tiled layout: escapes hold the same rounded, scaled values
    from oracle import quant
    th.set_precision("f16")
    th.set_packed_group(3)
    Q = quant.quantize(A, n, J, "f16")
    y = host(th.apply(dev(x)))
    ref = Q @ x.astype(np.float64)
    assert np.max(np.abs(y - ref)) <= 1e-5 * np.max(np.abs(ref))
    xq, _ = th.solve_coeffs(dev(x0), 0.05, 50, check_every=0)
    xo, _, _ = fista.fista(Q, x0.astype(np.float64), lam, 1.0 / Lo, 50)
    _gate(Q, x0.astype(np.float64), lam, host(xq), xo, fista.objective(Q, x0.astype(np.float64), lam, xo))


def test_autotune_picks_a_layout_and_keeps_parity(W, p64, tmp_path):
    th = imported(W, p64)
    cache = str(tmp_path / "tune.txt")
    c, g, us = th.autotune(cache, reps=5)
    assert c in (8, 16, 32, 64) and g in (0, 2, 3, 4, 8, 16) and us > 0
    c2, g2, us2 = th.autotune(cache, reps=5)           # served from the cache
    assert (c2, g2, us2) == (c, g, pytest.approx(us, rel=1e-6))
    wl = p64["wl"]
    th.lipschitz(synth.power_start(4096, wl.power_seed))
    x0 = p64["x0"].astype(np.float32)
    xg, _ = th.solve_coeffs(dev(x0), wl.lam, 200, check_every=50)
    x_o, E_o = _oracle_fista(p64, 200)
    _gate(p64["A32"], x0.astype(np.float64), float(np.float32(wl.lam)), host(xg), x_o, E_o)
