"""Sizes at the edges of the kernels' blocks and of the dispatch rules."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

isdf = pytest.importorskip("paper_2208_07731_amd")

EPS = np.finfo(np.float64).eps


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


def _cc_real(phi, psi, idx):
    """C C^H as the factorisation sees it: real, or real 2 x 2 blocks."""
    a = phi[idx] @ phi[idx].conj().T
    m = a * (psi[idx] @ psi[idx].conj().T).conj()
    if psi is phi:
        return m.real
    rows = np.stack([np.stack([m.real, m.imag], 2), np.stack([-m.imag, m.real], 2)], 1)
    return rows.reshape(2 * len(idx), 2 * len(idx))


# orders around the 16-, 32- and 64-wide blocks of the diagonal kernel, the
# 256-wide outer block, the order from which the inverse is formed on its lower
# tiles (768), and ragged last blocks; complex: twice the order
@pytest.mark.parametrize("n_mu,two", [(1, 0), (15, 0), (17, 0), (63, 0), (64, 0), (65, 0), (129, 0), (255, 0), (256, 0),
                                      (257, 0), (577, 0), (767, 0), (768, 0), (833, 0), (33, 1), (129, 1), (385, 1)])
def test_cholesky_inverse_edges(n_mu, two):
    """(C C^H)^-1 against numpy's inverse.  The computed inverse of an SPD
    matrix of order n by Cholesky is within c n eps kappa of the exact one; the
    bar is 8 n eps kappa (numpy's own error included)."""
    n = (10, 11, 13)
    phi = synth.random_orthonormal(1430, 40, 3 + n_mu)
    psi = synth.random_orthonormal(1430, 44, 4 + n_mu) if two else phi
    idx = np.random.default_rng(n_mu).permutation(1430)[:n_mu]
    m = _cc_real(phi, psi, idx)
    p = dev(phi)
    theta, minv, info = isdf.fit(p, dev(psi) if two else None, dev(idx.astype(np.int32)), grid=n)
    w = minv.cpu().numpy().reshape(m.shape)
    ev = np.linalg.eigvalsh(m)
    ref = np.linalg.inv(m)
    err = np.linalg.norm(w - ref) / np.linalg.norm(ref)
    assert info["status"] == 0 and info["pivot"] == -1
    assert err <= 8 * len(m) * EPS * ev[-1] / ev[0]
    assert np.array_equal(w, w.T)
    assert ev[0] * (1 - 1e-8) <= info["pivot_min"] <= info["pivot_max"] <= ev[-1] * (1 + 1e-8)


@pytest.mark.parametrize("bad", [0, 15, 16, 63, 64, 70, 299])
def test_cholesky_names_the_failing_pivot(bad):
    """A zero orbital row makes exactly its own pivot zero."""
    phi = synth.random_orthonormal(1430, 40, 5)
    idx = np.random.default_rng(6).permutation(1430)[:300]
    phi[idx[bad]] = 0.0
    _, _, info = isdf.fit(dev(phi), None, dev(idx.astype(np.int32)), grid=(10, 11, 13), check=False)
    assert info["status"] == 1 and info["pivot"] == bad


# planes of 8 columns in 512 and 1024 threads, of 2 and of 1, just too large
# for LDS, with a factor 7 and with an axis of length 1 (both by lines); the
# third axis's column groups of 32, 16 and 8; odd column counts and pitches
@pytest.mark.parametrize("n", [(3, 16, 32), (4, 32, 32), (5, 64, 64), (2, 72, 72), (2, 9, 5), (2, 100, 90), (3, 14, 6),
                               (3, 6, 14), (1, 24, 20), (6, 1, 20), (6, 20, 1), (160, 4, 6), (72, 3, 8), (20, 27, 25)])
@pytest.mark.parametrize("n_mu,pad,cplx,single", [(37, 0, 0, 0), (18, 2, 0, 0), (35, 0, 1, 0), (70, 1, 0, 1),
                                                  (66, 0, 1, 1)])
def test_poisson_plane_edges(n, n_mu, pad, cplx, single):
    """A transform of N points has a relative error of a few eps log2 N in the
    2-norm; two of them and the multiplication stay below 16 eps log2 N (and
    half an ulp of single-precision storage)."""
    n_r = n[0] * n[1] * n[2]
    rng = np.random.default_rng(n_r + n_mu)
    x = rng.standard_normal((n_r, n_mu + pad))
    if cplx:
        x = x + 1j * rng.standard_normal(x.shape)
    if single:
        x = x.astype(np.complex64 if cplx else np.float32)
    v = isdf.poisson(dev(x)[:, :n_mu], n).cpu().numpy()
    ref = oracle.poisson(x[:, :n_mu].astype(np.complex128 if cplx else np.float64), n)
    err = np.linalg.norm(v - ref) / max(np.linalg.norm(ref), 1e-300)
    assert err <= 16 * EPS * np.log2(n_r) + (2.0 ** -24 if single else 0.0)


# 384 is the smallest order whose complex product takes the residues; 4096 and
# 4097 terms are on the two sides of the quick remainder; 16384 rows are one panel
@pytest.mark.parametrize("n_mu,rows,single,pad", [(384, 2048, 0, 0), (385, 2049, 0, 3), (601, 2305, 1, 0),
                                                  (1201, 16384 + 65, 0, 2), (2049, 2050, 0, 1), (4097, 2048, 0, 0)])
def test_complex_residue_product(n_mu, rows, single, pad):
    """Theta = G (C C^H)^-1 for complex G.  The residue form rounds operands
    scaled to 2^58: within sqrt(2 K) 2^-58 of the product of the row norms, plus
    the rounding of the result; the FP64 reference is within 2 K eps of the sum
    of moduli, itself below the product of the row norms."""
    from paper_2208_07731_amd import _lib as L

    lib = L.load()
    gen = torch.Generator(device="cuda").manual_seed(n_mu)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex128, device="cuda", generator=gen)
    d = 2.0 ** (16 * torch.rand(n_mu, dtype=torch.float64, device="cuda", generator=gen) - 8)
    w = rand(n_mu, n_mu) / n_mu ** 0.5
    w = (w + w.conj().T) / 2 + torch.diag(1 + torch.rand(n_mu, dtype=torch.float64, device="cuda", generator=gen))
    w = d[:, None] * w * d
    g = rand(rows, n_mu + pad) / torch.cat([d, torch.ones(pad, dtype=torch.float64, device="cuda")])
    # rows (re, im) and (-im, re)
    minv = torch.view_as_real(torch.stack([w, 1j * w], 1)).reshape(2 * n_mu, 2 * n_mu).contiguous()
    size = lib.isdf_apply_minv_workspace(n_mu, 0, rows)
    assert size > 0
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    dt = L.C64 if single else L.C128

    def run(m, work):
        out = torch.empty(rows, n_mu, dtype=torch.complex64 if single else torch.complex128, device="cuda")
        assert lib.isdf_apply_minv_ws(n_mu, 0, m.data_ptr(), g.data_ptr(), 2 * g.stride(0), rows, dt, out.data_ptr(),
                                      n_mu, work, size if work else 0, None) == L.OK
        return out.to(torch.complex128)

    got, fp64 = run(minv, ws.data_ptr()), run(minv, None)
    a, b = g[:, :n_mu] * d, w / d  # the balanced operands, whose norms the rounding is relative to
    bound = torch.outer(a.abs().square().sum(1).sqrt(), b.abs().square().sum(1).sqrt())
    bar = (2 * n_mu * EPS + (2 * n_mu) ** 0.5 * 2.0 ** -58 + (2.0 ** -23 if single else 0.0)) * bound
    assert torch.all((got - fp64).abs() <= bar)
    if not single:
        sample = torch.arange(0, rows, max(1, rows // 16), device="cuda")
        exact = (g[sample, :n_mu].cpu().numpy().astype(np.clongdouble) @ w.cpu().numpy().astype(np.clongdouble))
        e = lambda x: float(np.linalg.norm((x[sample].cpu().numpy() - exact).astype(np.complex128)) / np.linalg.norm(exact.astype(np.complex128)))
        assert e(got) <= e(fp64)
    # a matrix without the block form is multiplied as it is
    odd = minv.clone()
    odd[1, 0] += 0.01 * float(minv[0, 0])
    assert torch.equal(run(odd, ws.data_ptr()), run(odd, None))


# on both sides of the rule for residues (K N >= 160 (K + N)), a ragged last
# block of rows, real and complex potentials, both storage types
@pytest.mark.parametrize("n_mu,n_psi,v_complex,single,rblock", [(700, 210, 0, 0, None), (700, 200, 0, 0, None),
                                                                (701, 211, 1, 0, 2049), (701, 333, 1, 1, None),
                                                                (33, 7, 0, 0, 1000)])
def test_exchange_edges(n_mu, n_psi, v_complex, single, rblock):
    """Against complex extended-precision sums at sampled rows: FP64 products of
    n_phi and n_mu terms are within 4 (n_phi + n_mu) eps of the sum of moduli,
    residues within sqrt(2 n_mu) 2^-58 of the product of the row norms."""
    n = (15, 16, 17)
    n_r, n_phi = 15 * 16 * 17, 40
    rng = np.random.default_rng(n_mu + n_psi)
    c = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    store = np.complex64 if single else np.complex128
    env = np.exp(-3 * rng.random((n_r, 1)))
    phi, psi = (c(n_r, n_phi) * env).astype(store), (c(n_r, n_psi) * env).astype(store)
    idx = rng.permutation(n_r)[:n_mu]
    v = c(n_r, n_mu) if v_complex else rng.standard_normal((n_r, n_mu))
    v = v.astype(store if v_complex else (np.float32 if single else np.float64))
    got = isdf.exchange(dev(phi), dev(psi), dev(idx.astype(np.int32)), dev(v), rblock=rblock, grid=n).cpu().numpy()
    rows = np.r_[0:n_r:97, n_r - 1]
    x = lambda a: a.astype(np.clongdouble)
    a = x(phi[rows]) @ x(phi[idx]).conj().T
    w = x(v[rows]).conj() * a
    ref = -(w @ x(psi[idx]))
    moduli = (np.abs(v[rows]) * (np.abs(phi[rows]) @ np.abs(phi[idx]).T)) @ np.abs(psi[idx])
    norms = np.outer(np.linalg.norm(w.astype(np.complex128), axis=1), np.linalg.norm(psi[idx], axis=0))
    bar = 4 * (n_phi + n_mu) * EPS * moduli + (2 * n_mu) ** 0.5 * 2.0 ** -58 * norms
    bar = bar + (2.0 ** -23 * np.abs(ref.astype(np.complex128)) if single else 0.0)
    assert np.all(np.abs((got[rows] - ref).astype(np.complex128)) <= bar)


def test_poisson_more_columns_than_a_grid_dimension():
    """65544 tiles of 8 columns: past 65535 of them the line passes run.  Every
    column is one of 16, so the bar of test_poisson_plane_edges holds for each."""
    n, base = (1, 2, 2), np.random.default_rng(3).standard_normal((4, 16))
    m = 2 * 8 * 65544
    v = isdf.poisson(dev(np.tile(base, (1, m // 16))), n).cpu().numpy().reshape(4, m // 16, 16)
    ref = oracle.poisson(base, n)
    err = np.linalg.norm(v - ref[:, None, :], axis=(0, 2)) / np.linalg.norm(ref)
    assert err.max() <= 16 * EPS * 2


# all centroids per brick (one LDS tile, few bricks times centroids) against
# cells: a full survivor list, the last K of a tile and one more, 72^3 on the
# cells' side of the rule; an anisotropic metric
@pytest.mark.parametrize("n,k,h", [((9, 10, 11), 700, (1, 1, 1)), ((24, 25, 26), 2048, (1, 1, 1)),
                                   ((24, 25, 26), 2049, (1, 1.5, 0.7)), ((40, 41, 9), 64, (0.5, 1, 2)),
                                   ((72, 72, 72), 1800, (1, 1, 1))])
def test_kmeans_dispatch_edges(n, k, h):
    """Two Lloyd rounds and a classification against the oracle: the same
    labels wherever its two nearest distances differ by more than rounding."""
    n_r = n[0] * n[1] * n[2]
    rng = np.random.default_rng(k)
    w = rng.random(n_r) + 0.05
    c0 = oracle.grid_points(n)[rng.permutation(n_r)[:k]].astype(np.float64) + 0.25 * rng.random((k, 3))
    r = isdf.kmeans(None, None, k, c0, 2, w=dev(w), grid=n, h=h)
    ref = oracle.kmeans(n, w, c0, 2, h)
    assert np.array_equal(r.labels.cpu().numpy(), ref["labels"])
    assert np.array_equal(r.idx.cpu().numpy(), ref["idx"])
    assert abs(r.info["objective"] - ref["J"][-1]) <= 1e-12 * ref["J"][-1]


# the adjoint's products with Phi_mu on the residue side of the rule, per block
# (K N >= 160 (K + N), blocks of 2048 rows and more, the last one shorter) and
# at the interpolation rows (2048 points and more); fused and general losses,
# one set and two
@pytest.mark.parametrize("n_phi,n_psi,n_mu,fused,rblock", [(200, 0, 1001, 1, None), (200, 0, 1001, 0, 2100),
                                                           (180, 0, 2049, 1, 4000), (60, 240, 701, 0, None),
                                                           (60, 240, 701, 1, 2049)])
def test_backward_residue_edges(n_phi, n_psi, n_mu, fused, rblock):
    """Gradients against the oracle.  With a condition number kappa of C C^H the
    gradient's relative error is a few n_mu eps kappa in the worst case; the bar
    is 1e-11, that of the FP64 gradients elsewhere, and n_mu eps kappa where that
    is larger."""
    n = (16, 17, 16)
    n_r = 16 * 17 * 16
    rng = np.random.default_rng(n_mu + n_phi)
    c = lambda m: rng.standard_normal((n_r, m)) + 1j * rng.standard_normal((n_r, m))
    phi = c(n_phi)
    psi = c(n_psi) if n_psi else phi
    idx = rng.permutation(n_r)[:n_mu].astype(np.int32)
    kw = {}
    if fused:
        kw["g"] = rng.uniform(0.5, 1.5, n_r)
    else:
        kw["theta_bar"] = rng.standard_normal((n_r, n_mu)) + (1j * rng.standard_normal((n_r, n_mu)) if n_psi else 0.0)
    ref = oracle.fit_backward(phi, psi, idx, **kw)
    a, b = dev(phi), dev(psi) if n_psi else None
    _, minv, _ = isdf.fit(a, b, dev(idx), grid=n, nrows=0)
    dphi, dpsi, loss, _ = isdf.fit_backward(a, b, dev(idx), minv, grid=n, rblock=rblock,
                                            **{k: dev(v) for k, v in kw.items()})
    bar = max(1e-11, n_mu * EPS * oracle.cc_condition(phi, psi, idx))
    rel = lambda x, y: float(np.linalg.norm(x - y) / np.linalg.norm(y))
    assert rel(dphi.cpu().numpy(), ref["dphi"]) <= bar
    if n_psi:
        assert rel(dpsi.cpu().numpy(), ref["dpsi"]) <= bar
    if fused:
        assert abs(loss.item() - ref["loss"]) <= bar * ref["loss"]


# rows around the 64 of a workgroup and the 256 of the first one, columns around
# the 8 wavefronts' shares, their 16 loads in flight and the 64 staged entries;
# orbital counts around the 16 lanes of a row and the 64 loaded ahead; one pivot
@pytest.mark.parametrize("n,n_phi,n_psi,n_mu", [((1, 1, 63), 5, 0, 20), ((1, 1, 65), 17, 0, 40), ((5, 7, 9), 33, 0, 131),
                                                ((7, 8, 23), 65, 0, 700), ((7, 8, 23), 15, 70, 300), ((5, 5, 11), 3, 2, 1),
                                                ((16, 16, 3), 40, 0, 2)])
def test_qrcp_edges(n, n_phi, n_psi, n_mu):
    """Pivots against the oracle's pivoted QR up to its first near tie; squared
    diagonals within 64 k eps |R_00|^2 (each is a difference of k terms that are
    at most |R_00|^2)."""
    n_r = n[0] * n[1] * n[2]
    rng = np.random.default_rng(n_r + n_mu)
    c = lambda m: (rng.standard_normal((n_r, m)) + 1j * rng.standard_normal((n_r, m))) * np.exp(-2 * rng.random((n_r, 1)))
    phi = c(n_phi)
    psi = c(n_psi) if n_psi else phi
    n_mu = min(n_mu, n_r)
    o = oracle.qrcp(phi, psi, n_mu)
    r = isdf.qrcp(dev(phi), dev(psi) if n_psi else None, n_mu, grid=n)
    assert r.info["rank"] == o["rank"]
    rank = o["rank"]
    s = o["rdiag"][:rank] ** 2
    near = np.nonzero(o["gap"][:rank] * s <= 1e-9 * s[0])[0]
    upto = int(near[0]) if near.size else rank
    assert np.array_equal(r.idx.cpu().numpy()[:upto], o["idx"][:upto])
    assert np.max(np.abs(r.rdiag.cpu().numpy()[:upto] ** 2 - s[:upto])) <= 64 * rank * EPS * s[0]
    assert np.all(r.idx.cpu().numpy()[rank:] == -1)
