"""FP64 products by int8 residues (isdf_apply_minv_ws) against the FP64 kernel
(isdf_apply_minv) and extended-precision sums.

Tolerance: the FP64 kernel's K-term sum is within K eps (|G| |W|) of the exact
one; the residue form rounds the scaled operands, within sqrt(K) 2^-58 of the
product of the row norms, plus the rounding of the result.
"""
import numpy as np
import pytest
import torch

from paper_2208_07731_amd import _lib as L

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def _inputs(rows, n1, seed, spread):
    rng = np.random.Generator(np.random.PCG64(seed))
    d = 2.0 ** rng.uniform(-spread, spread, n1)  # density at the interpolation points
    G = np.abs(rng.standard_normal((rows, n1))) / d
    W = rng.standard_normal((n1, n1)) / np.sqrt(n1)
    W = (W + W.T) / 2 + np.diag(rng.uniform(1, 3, n1))
    return G, (d[:, None] * W) * d[None, :]


def _apply(lib, G, W, n_mu, aliased, rows, dt, ld_theta, ws):
    real = {(L.C128, 1): torch.float64, (L.C64, 1): torch.float32, (L.C128, 0): torch.complex128,
            (L.C64, 0): torch.complex64}[(dt, aliased)]
    out = torch.full((rows, ld_theta), 7.0, dtype=real, device="cuda")
    if ws is None:
        code = lib.isdf_apply_minv(n_mu, aliased, W.data_ptr(), G.data_ptr(), G.stride(0), rows, dt, out.data_ptr(),
                                   ld_theta, None)
    else:
        code = lib.isdf_apply_minv_ws(n_mu, aliased, W.data_ptr(), G.data_ptr(), G.stride(0), rows, dt, out.data_ptr(),
                                      ld_theta, ws.data_ptr(), ws.numel(), None)
    assert code == L.OK
    torch.cuda.synchronize()
    return out


# n_mu 1024 is the smallest order the residues take; odd ones leave ragged K,
# N and row tiles; 16384 rows are one panel
@pytest.mark.parametrize("n_mu,aliased,rows,dt,pad,ldpad", [
    (1024, 1, 2048, L.C128, 0, 0),
    (1025, 1, 2049, L.C128, 1, 3),
    (1290, 1, 16384 + 257, L.C64, 0, 1),
    (600, 0, 2305, L.C128, 2, 0),
    (601, 0, 2048, L.C64, 0, 5),
    (2177, 1, 2100, L.C128, 0, 0),
])
def test_residue_product(n_mu, aliased, rows, dt, pad, ldpad):
    lib = L.load()
    n1 = n_mu if aliased else 2 * n_mu
    Gh, Wh = _inputs(rows, n1, 11 * n_mu + rows, 12.0)
    G = torch.zeros(rows, n1 + pad, dtype=torch.float64, device="cuda")
    G[:, :n1] = torch.from_numpy(Gh).cuda()
    W = torch.from_numpy(np.ascontiguousarray(Wh)).cuda()
    size = lib.isdf_apply_minv_workspace(n_mu, aliased, rows)
    assert size > 0
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    got = _apply(lib, G, W, n_mu, aliased, rows, dt, n_mu + ldpad, ws)
    ref = _apply(lib, G, W, n_mu, aliased, rows, dt, n_mu + ldpad, None)
    assert torch.equal(got[:, n_mu:], ref[:, n_mu:])  # nothing written past a row
    sel = np.unique(np.concatenate([np.arange(0, rows, max(1, rows // 24)), [rows - 1]]))
    col = np.unique(np.concatenate([np.arange(0, n1, max(1, n1 // 50)), [n1 - 2, n1 - 1]]))
    exact = Gh[sel].astype(np.longdouble) @ Wh[col].astype(np.longdouble).T
    terms = np.abs(Gh[sel]) @ np.abs(Wh[col]).T
    g = got[:, :n_mu].contiguous()
    g = (torch.view_as_real(g).reshape(rows, n1) if not aliased else g).cpu().numpy()[sel][:, col]
    store = np.finfo(np.float64 if dt == L.C128 else np.float32).eps * np.abs(exact.astype(np.float64))
    bound = n1 * EPS * terms + 2 * EPS * np.abs(exact.astype(np.float64)) + store
    assert np.all(np.abs((g - exact).astype(np.float64)) <= bound)
    if dt == L.C128:  # and no further off than the FP64 kernel overall
        f = ref[:, :n_mu].contiguous()
        f = (torch.view_as_real(f).reshape(rows, n1) if not aliased else f).cpu().numpy()[sel][:, col]
        assert np.linalg.norm((g - exact).astype(np.float64)) <= np.linalg.norm((f - exact).astype(np.float64))


@pytest.mark.parametrize("what", ["nan", "inf", "huge", "tiny"])
def test_rows_out_of_range_take_the_fp64_kernel(what):
    """A row that is not finite or whose squared norm leaves the FP64 range
    sends its panel to the FP64 kernel: the results are its bits."""
    lib = L.load()
    n_mu, rows = 1100, 2304
    Gh, Wh = _inputs(rows, n_mu, 5, 3.0)
    Gh[77, 13] = {"nan": np.nan, "inf": np.inf, "huge": 1e200, "tiny": 1.0}[what]
    if what == "tiny":
        Gh[77] = 1e-200
    G, W = torch.from_numpy(Gh).cuda(), torch.from_numpy(np.ascontiguousarray(Wh)).cuda()
    ws = torch.empty(lib.isdf_apply_minv_workspace(n_mu, 1, rows), dtype=torch.uint8, device="cuda")
    got = _apply(lib, G, W, n_mu, 1, rows, L.C128, n_mu, ws)
    ref = _apply(lib, G, W, n_mu, 1, rows, L.C128, n_mu, None)
    assert torch.equal(got.view(torch.int64), ref.view(torch.int64))


def test_zero_rows_and_workspace_limits():
    lib = L.load()
    n_mu, rows = 1100, 2304
    Gh, Wh = _inputs(rows, n_mu, 6, 3.0)
    Gh[5] = 0.0
    Gh[rows - 1] = 0.0
    G, W = torch.from_numpy(Gh).cuda(), torch.from_numpy(np.ascontiguousarray(Wh)).cuda()
    size = lib.isdf_apply_minv_workspace(n_mu, 1, rows)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    got = _apply(lib, G, W, n_mu, 1, rows, L.C128, n_mu, ws)
    assert not got[5].any() and not got[rows - 1].any() and bool(torch.isfinite(got).all())
    out = torch.empty(rows, n_mu, dtype=torch.float64, device="cuda")
    assert lib.isdf_apply_minv_ws(n_mu, 1, W.data_ptr(), G.data_ptr(), n_mu, rows, L.C128, out.data_ptr(), n_mu,
                                  ws.data_ptr(), size - 1, None) == L.E_WORKSPACE
    assert lib.isdf_apply_minv_workspace(n_mu, 1, 2047) == 0  # too few rows: the FP64 kernel, no workspace


def _block_form(n_mu, seed):
    """[[re, im], [-im, re]] blocks of a Hermitian positive matrix."""
    rng = np.random.default_rng(seed)
    w = rng.standard_normal((n_mu, n_mu)) + 1j * rng.standard_normal((n_mu, n_mu))
    w = (w + w.conj().T) / (2 * np.sqrt(n_mu)) + np.diag(rng.uniform(1, 3, n_mu))
    W = np.empty((2 * n_mu, 2 * n_mu))
    W[0::2, 0::2], W[0::2, 1::2], W[1::2, 0::2], W[1::2, 1::2] = w.real, w.imag, -w.imag, w.real
    return W


# one entry of an odd row: by half a unit in the last place, by 1e-9 of the diagonal
@pytest.mark.parametrize("dt,off", [(L.C128, 0.0), (L.C128, 2.0 ** -52), (L.C128, 1e-9), (L.C64, 2.0 ** -20)])
def test_a_matrix_almost_of_block_form_is_multiplied_as_it_is(dt, off):
    """The complex product reads a matrix's even rows only, so for results in
    double it stands for a matrix of exact blocks alone, and in single for one
    within 2^-24; any other one gives the FP64 kernel's bits."""
    lib = L.load()
    n_mu, rows = 600, 2304
    Gh = np.random.default_rng(1).standard_normal((rows, 2 * n_mu))
    Wh = _block_form(n_mu, 2)
    Wh[7, 7] += off * Wh[7, 7]
    G, W = torch.from_numpy(Gh).cuda(), torch.from_numpy(Wh).cuda()
    ws = torch.empty(lib.isdf_apply_minv_workspace(n_mu, 0, rows), dtype=torch.uint8, device="cuda")
    got = _apply(lib, G, W, n_mu, 0, rows, dt, n_mu, ws)
    ref = _apply(lib, G, W, n_mu, 0, rows, dt, n_mu, None)
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(ref)) == (off != 0.0)


@pytest.mark.parametrize("prec", ["fp64", "bf16x6", "fp16x3"])
def test_the_fit_leaves_exact_blocks(prec):
    """M^-1 of two orbital sets, of the orders whose products go by residues."""
    import paper_2208_07731_amd as isdf

    rng = np.random.default_rng(4)
    c = lambda n: torch.from_numpy(rng.standard_normal((2016, n)) + 1j * rng.standard_normal((2016, n))).cuda()
    phi, psi = c(24), c(40)
    for n_mu in (449, 601):
        idx = torch.from_numpy(rng.permutation(2016)[:n_mu].astype(np.int32)).cuda()
        _, minv, _ = isdf.fit(phi, psi, idx, grid=(12, 12, 14), nrows=0, prec=prec)
        w = minv.reshape(2 * n_mu, 2 * n_mu)
        assert torch.equal(w[0::2, 0::2], w[1::2, 1::2]) and torch.equal(w[0::2, 1::2], -w[1::2, 0::2])
        assert torch.equal(w, w.T)


def test_a_flag_ends_with_its_block_of_rows():
    """A row that sends its panel to the FP64 kernel leaves the later blocks of
    rows as they are without it: the same bits by residues."""
    import paper_2208_07731_amd as isdf

    rng = np.random.default_rng(9)
    n, n_mu, n_psi, rblock = (15, 16, 34), 700, 210, 2050  # the residues take blocks of 2048 rows and more
    n_r = 15 * 16 * 34
    c = lambda m: torch.from_numpy(rng.standard_normal((n_r, m)) + 1j * rng.standard_normal((n_r, m))).cuda()
    phi, psi = c(20), c(n_psi)
    idx = torch.from_numpy(rng.permutation(n_r)[:n_mu].astype(np.int32)).cuda()
    v = torch.from_numpy(rng.standard_normal((n_r, n_mu))).cuda()
    good = isdf.exchange(phi, psi, idx, v, rblock=rblock, grid=n)
    v[1, 5] = float("nan")  # (row 1: not one that the balance of the columns samples)
    bad = isdf.exchange(phi, psi, idx, v, rblock=rblock, grid=n)
    assert bool(torch.isnan(bad[1].real).all())
    assert torch.equal(torch.view_as_real(bad[rblock:]), torch.view_as_real(good[rblock:]))
    assert not torch.equal(torch.view_as_real(bad[2:rblock]), torch.view_as_real(good[2:rblock]))


# 384: padded to 512 columns; 448: the last multiple of 64 below the line; 449,
# 512: above it.  Real: 1100 below, 1200 above
@pytest.mark.parametrize("n_mu,aliased,residues", [(384, 0, False), (448, 0, False), (449, 0, True), (512, 0, True),
                                                   (1024, 1, False), (1100, 1, False), (1200, 1, True)])
def test_the_line_between_the_kernels(n_mu, aliased, residues):
    """Where the residues would be slower the results are the FP64 kernel's bits."""
    lib = L.load()
    rows = 2304
    n1 = n_mu if aliased else 2 * n_mu
    Gh = np.random.default_rng(n_mu).standard_normal((rows, n1))
    Wh = _inputs(1, n1, n_mu, 3.0)[1] if aliased else _block_form(n_mu, n_mu)
    G, W = torch.from_numpy(Gh).cuda(), torch.from_numpy(np.ascontiguousarray(Wh)).cuda()
    ws = torch.empty(lib.isdf_apply_minv_workspace(n_mu, aliased, rows), dtype=torch.uint8, device="cuda")
    got = _apply(lib, G, W, n_mu, aliased, rows, L.C128, n_mu, ws)
    ref = _apply(lib, G, W, n_mu, aliased, rows, L.C128, n_mu, None)
    assert torch.equal(got, ref) != residues


# a raised flag in the first and in the second panel of 16384 rows, real and
# complex
@pytest.mark.parametrize("row", [77, 16384 + 77])
@pytest.mark.parametrize("n_mu,aliased", [(1200, 1), (600, 0)])
def test_a_flag_sends_its_panel_alone(n_mu, aliased, row):
    lib = L.load()
    rows, n1 = 16384 + 2304, n_mu if aliased else 2 * n_mu
    Gh = np.random.default_rng(n_mu).standard_normal((rows, n1))
    Wh = _inputs(1, n1, n_mu, 3.0)[1] if aliased else _block_form(n_mu, n_mu)
    G, W = torch.from_numpy(Gh).cuda(), torch.from_numpy(np.ascontiguousarray(Wh)).cuda()
    ws = torch.empty(lib.isdf_apply_minv_workspace(n_mu, aliased, rows), dtype=torch.uint8, device="cuda")
    apply = lambda w: _apply(lib, G, W, n_mu, aliased, rows, L.C128, n_mu, w)
    clean = apply(ws)
    G[row] = 1e-200
    got, ref = apply(ws), apply(None)
    own, other = (slice(0, 16384), slice(16384, rows))[:: 1 if row < 16384 else -1]
    assert torch.equal(got[own], ref[own])
    assert torch.equal(got[other], clean[other]) and not torch.equal(got[other], ref[other])


# blocks of more than one panel; the flagged row in the first and in the second
@pytest.mark.parametrize("n_phi,n_psi,n_mu", [(60, 0, 1201), (30, 45, 701)])
@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("row", [100, 17000])
def test_adjoint_with_a_flagged_panel(n_phi, n_psi, n_mu, fused, row):
    """One orbital row is so small that its row of G (or one row of the upstream
    gradient) is out of the residues' range: its panel goes through the FP64
    kernel, the other one by residues, each row and each loss partial once.
    Against the oracle, within 1e-11 or n_mu eps kappa."""
    import oracle
    import paper_2208_07731_amd as isdf

    n, n_r = (26, 26, 26), 26 ** 3
    rng = np.random.default_rng(n_mu + row + fused)
    c = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    phi = c(n_r, n_phi)
    psi = c(n_r, n_psi) if n_psi else phi
    idx = rng.permutation(np.setdiff1d(np.arange(n_r), [row]))[:n_mu].astype(np.int32)
    kw = {}
    if fused:
        phi[row] *= 1e-150 if n_psi else 1e-75
        kw["g"] = rng.uniform(0.5, 1.5, n_r)
    else:
        kw["theta_bar"] = c(n_r, n_mu) if n_psi else rng.standard_normal((n_r, n_mu))
        kw["theta_bar"][row] *= 1e-160
    ref = oracle.fit_backward(phi, psi, idx, **kw)
    bar = max(1e-11, n_mu * EPS * oracle.cc_condition(phi, psi, idx))
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    a, b = d(phi), d(psi) if n_psi else None
    _, minv, _ = isdf.fit(a, b, d(idx), grid=n, nrows=0)
    dphi, dpsi, loss, _ = isdf.fit_backward(a, b, d(idx), minv, grid=n, **{k: d(v) for k, v in kw.items()})
    rel = lambda x, y: float(np.linalg.norm(x.cpu().numpy() - y) / np.linalg.norm(y))
    assert rel(dphi, ref["dphi"]) <= bar
    if n_psi:
        assert rel(dpsi, ref["dpsi"]) <= bar
    if fused:
        assert abs(loss.item() - ref["loss"]) <= bar * ref["loss"]


def test_rows_at_the_points_by_residues():
    """dAbar Phi_mu at 2049 interpolation rows and Abar Phi_mu of blocks of 2100
    rows (the last one shorter, on the FP64 kernel), 256 orbitals: both products
    are on the residues' side of the rule.  Against the oracle, within 1e-11 or
    n_mu eps kappa."""
    import oracle
    import paper_2208_07731_amd as isdf

    n, n_r, n_phi, n_mu = (16, 17, 16), 16 * 17 * 16, 256, 2049
    assert L.load().isdf_residue_ops(n_mu, n_phi, n_mu, 1) == 9
    rng = np.random.default_rng(12)
    phi = rng.standard_normal((n_r, n_phi)) + 1j * rng.standard_normal((n_r, n_phi))
    idx = rng.permutation(n_r)[:n_mu].astype(np.int32)
    g = rng.uniform(0.5, 1.5, n_r)
    ref = oracle.fit_backward(phi, phi, idx, g=g)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    a = d(phi)
    _, minv, _ = isdf.fit(a, None, d(idx), grid=n, nrows=0)
    dphi, _, loss, _ = isdf.fit_backward(a, None, d(idx), minv, g=d(g), grid=n, rblock=2100)
    bar = max(1e-11, n_mu * EPS * oracle.cc_condition(phi, phi, idx))
    assert float(np.linalg.norm(dphi.cpu().numpy() - ref["dphi"]) / np.linalg.norm(ref["dphi"])) <= bar
    assert abs(loss.item() - ref["loss"]) <= bar * ref["loss"]
