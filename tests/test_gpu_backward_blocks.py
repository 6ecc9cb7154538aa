"""The adjoint streamed over row blocks of uneven length (isdf_fit_backward_rows
takes any nrows up to rblock)."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

isdf = pytest.importorskip("paper_2208_07731_amd")

EPS = np.finfo(np.float64).eps


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


# blocks that by time alone take more split-K slices than rblock and the grid's
# remainder do: 32 against 24 of Theta^T S for 9984 to 12032 rows of 168 points,
# two sets; 32 against 24 of Abar^T Phi for 12032 rows of 519 points and 64
# orbitals
@pytest.mark.parametrize("n_phi,n_psi,n_mu,fused,blocks", [
    (16, 16, 168, 0, (11008, 11008, 14848)),
    (16, 16, 168, 1, (14848, 11008, 11008)),
    (64, 0, 519, 1, (12032, 12032, 12800)),
])
def test_backward_rows_uneven_blocks(n_phi, n_psi, n_mu, fused, blocks):
    """Gradients against the oracle, within 1e-11 or n_mu eps kappa (the bar of
    the one-call gradients)."""
    from paper_2208_07731_amd import _lib as L

    lib = L.load()
    n, rblock = (24, 24, 64), 16384
    nr = 24 * 24 * 64
    assert sum(blocks) == nr and max(blocks) <= rblock
    rng = np.random.default_rng(n_mu + fused)
    c = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    phi = c(nr, n_phi)
    psi = c(nr, n_psi) if n_psi else phi
    two = n_psi > 0
    idx = rng.permutation(nr)[:n_mu].astype(np.int32)
    g = rng.uniform(0.5, 1.5, nr)
    tbar = None if fused else (c(nr, n_mu) if two else rng.standard_normal((nr, n_mu)))
    ref = oracle.fit_backward(phi, psi, idx, theta_bar=tbar, g=g if fused else None)
    bar = max(1e-11, n_mu * EPS * oracle.cc_condition(phi, psi, idx))

    tp, ts, it, gt = dev(phi), dev(psi) if two else None, dev(idx), dev(g)
    tb = None if fused else dev(tbar)
    _, minv, _ = isdf.fit(tp, ts, it, grid=n, nrows=0)
    gr, s = L.make_grid(n), torch.cuda.current_stream().cuda_stream
    q, n_q, n1 = (ts, n_psi, 2 * n_mu) if two else (tp, n_phi, n_mu)
    f64 = dict(dtype=torch.float64, device="cuda")
    u8 = dict(dtype=torch.uint8, device="cuda")
    zws = torch.empty(lib.isdf_zc_workspace(n_mu, n_phi, n_q, int(not two), 0, rblock), **u8)
    bws = torch.empty(lib.isdf_fit_backward_gram_workspace(C.byref(gr), n_mu, n_phi, n_q, int(not two), 0, rblock), **u8)
    G, A = torch.empty(rblock, n1, **f64), torch.empty(rblock, 2 * n_mu, **f64)
    B = torch.empty(rblock, 2 * n_mu, **f64) if two else None
    bp = B.data_ptr() if two else None
    dphi = torch.empty(nr, n_phi, dtype=torch.complex128, device="cuda")
    dpsi = torch.empty(nr, n_psi, dtype=torch.complex128, device="cuda") if two else dphi
    loss, info = torch.zeros((), **f64), torch.zeros(C.sizeof(L.FitInfo), **u8)
    r0 = 0
    for k, rows in enumerate(blocks):
        assert lib.isdf_zc_ab(C.byref(gr), L.C128, tp.data_ptr(), n_phi, n_phi, q.data_ptr(), n_q, n_q, it.data_ptr(),
                              n_mu, 0, r0, rows, G.data_ptr(), n1, A.data_ptr(), bp, zws.data_ptr(), zws.numel(),
                              s) == L.OK
        flags = (L.BWD_FIRST if k == 0 else 0) | (L.BWD_LAST if k == len(blocks) - 1 else 0)
        tbp = None if fused else tb.data_ptr() + r0 * n_mu * tb.element_size()
        assert lib.isdf_fit_backward_rows(C.byref(gr), L.C128, tp.data_ptr(), n_phi, n_phi, q.data_ptr(), n_q, n_q,
                                          it.data_ptr(), n_mu, 0, minv.data_ptr(), tbp, n_mu, gt.data_ptr(),
                                          dphi.data_ptr(), n_phi, dpsi.data_ptr(), n_q, loss.data_ptr(), r0, rows,
                                          rblock, G.data_ptr(), A.data_ptr(), bp, flags, info.data_ptr(),
                                          bws.data_ptr(), bws.numel(), s) == L.OK
        r0 += rows
    torch.cuda.synchronize()
    assert L.FitInfo.from_buffer_copy(bytes(info.cpu().numpy())).status == L.OK
    rel = lambda x, y: float(np.linalg.norm(x.cpu().numpy() - y) / np.linalg.norm(y))
    assert rel(dphi, ref["dphi"]) <= bar
    if two:
        assert rel(dpsi, ref["dpsi"]) <= bar
    if fused:
        assert abs(loss.item() - ref["loss"]) <= bar * ref["loss"]
