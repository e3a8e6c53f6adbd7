"""Dense CCD on the GPU (ccd_dense_solve): the pairing model of eqs.
sppairing / intpairing against the paper's table and the oracle's dense
form, and a small plane-wave basis against the oracle and against the
channel-blocked path.  The pairing Hamiltonian comes from
paper_1611_06765_amd.inputs (direct elements, then antisymmetrised), the
oracle's from its own construction."""
import numpy as np
import pytest

from conftest import golden

pytestmark = pytest.mark.gpu

ccd = pytest.importorskip("paper_1611_06765_amd.ccd")
from paper_1611_06765_amd import inputs  # noqa: E402

RTOL = 1e-12


@pytest.mark.parametrize("row", golden("pairing_table.txt"))
def test_pairing_table_on_gpu(row):
    g, eref, emp2, eccd = (float(x) for x in row)
    h, v = inputs.pairing_hamiltonian(g)
    r = ccd.dense_solve(h, v, 4, mixing=0.5 if g == -1.0 else 1.0, tol=1e-10, max_iter=400)
    assert r["status"] == ccd.CCD_OK
    assert r["e_ref"] == pytest.approx(eref, abs=1e-12)
    closed = -g * g / 4 * (1 / (4 + g) + 1 / (6 + g) + 1 / (2 + g) + 1 / (4 + g))
    assert r["e_mbpt2"] == pytest.approx(closed, abs=1e-13)
    assert r["e_mbpt2"] == pytest.approx(emp2, abs=5e-6)
    assert r["e_ccd"] == pytest.approx(eccd, abs=5e-6)


@pytest.mark.parametrize("mask", [1, 2, 4, 8, 16, 32, 64, 127])
@pytest.mark.parametrize("g", [-1.0, 0.5])
def test_pairing_terms_match_the_oracle_per_sweep(orc, g, mask):
    h, v = inputs.pairing_hamiltonian(g)
    r = ccd.dense_solve(h, v, 4, mixing=0.5, tol=0.0, max_iter=6, terms=mask)
    oh, ov = orc.pairing_model(g)
    o = orc.O1(oh, ov, 4)
    assert r["e_mbpt2"] == pytest.approx(o.emp2, rel=RTOL)
    for s in range(6):
        assert r["history"][s] == pytest.approx(o.sweep(0.5, mask), rel=RTOL, abs=1e-15), (g, mask, s)


@pytest.mark.parametrize("mask", [4, 16, 32, 64, 127])
def test_plane_waves_dense_equals_oracle_and_channel_path(orc, mask):
    """N = 2, n^2 <= 1 (14 states): dense GPU, the oracle's dense form and the
    channel-blocked GPU path agree sweep by sweep."""
    p = orc.PNM(2, 1, 0.08)
    h, v = p.kinetic(), p.dense_v()
    r = ccd.dense_solve(h, v, 2, mixing=0.7, tol=0.0, max_iter=5, terms=mask)
    o = orc.O1(h, v, 2)
    import torch
    ctx = ccd.Context([ccd.problem(2, 1, 0.08)], stream=torch.cuda.current_stream().cuda_stream).bind()
    hc = ctx.iterate(mixing=0.7, tol=0.0, max_iter=5, terms=mask, history=True)["history"][0]
    for s in range(5):
        e = o.sweep(0.7, mask)
        assert r["history"][s] == pytest.approx(e, rel=1e-12)
        assert hc[s] == pytest.approx(r["history"][s], rel=1e-10)


def test_plane_waves_dense_larger_basis(orc):
    """N = 14, n^2 <= 2 (38 states, every hole pair): three full sweeps."""
    p = orc.PNM(14, 2, 0.1)
    h, v = p.kinetic(), p.dense_v()
    r = ccd.dense_solve(h, v, 14, mixing=0.8, tol=0.0, max_iter=3)
    o = orc.O1(h, v, 14)
    assert r["e_mbpt2"] == pytest.approx(o.emp2, rel=1e-12)
    for s in range(3):
        assert r["history"][s] == pytest.approx(o.sweep(0.8), rel=1e-11)


def _random_hamiltonian(n, seed=5):
    """One-body levels one apart and weak random antisymmetrised elements, without
    any symmetry that would hide a wrong index."""
    v = np.random.default_rng(seed).normal(size=(n,) * 4) * 0.02 / n
    v = v - v.transpose(1, 0, 2, 3)
    v = v - v.transpose(0, 1, 3, 2)
    return np.arange(n, dtype=float), v + v.transpose(2, 3, 0, 1)


@pytest.mark.parametrize("n, nh", [(2, 1), (7, 3), (8, 7), (11, 5), (12, 5), (13, 12), (17, 3)])
@pytest.mark.parametrize("mask", [2, 9, 16, 32, 64, 127])
def test_sweeps_in_one_block_by_launches_and_without_intermediates(orc, n, nh, mask):
    """Model spaces on both sides of the largest that one block holds (11 states),
    with the advertised work area and with one that has no room for intermediates:
    every sweep's energy equals the oracle's and does not depend on the area."""
    import ctypes as C
    import torch
    h, v = _random_hamiltonian(n)
    o = orc.O1(h, v, nh)
    ref = [o.sweep(0.8, mask) for _ in range(5)]
    r = ccd.dense_solve(h, v, nh, mixing=0.8, tol=0.0, max_iter=5, terms=mask)
    m = (nh * (n - nh)) ** 2
    up = lambda x: -(-x // 256) * 256  # noqa: E731
    small = up(8 * n ** 4) + up(8 * n) + 2 * up(8 * m) + up(8 * -(-m // 256))
    work = torch.empty(small, dtype=torch.uint8, device="cuda")
    hist = np.zeros(5)
    opt = ccd.ccd_solver_opts()
    opt.mixing, opt.tol, opt.max_iter, opt.terms = 0.8, 0.0, 5, mask
    st = ccd._lib.ccd_dense_solve(ccd._dptr(h), ccd._dptr(v), n, nh, C.byref(opt), C.c_void_p(work.data_ptr()), small,
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream), None, None, None, None,
                                  ccd._dptr(hist))
    assert st == ccd.CCD_OK
    for s in range(5):
        assert r["history"][s] == pytest.approx(ref[s], rel=RTOL, abs=1e-15), s
        assert hist[s] == pytest.approx(ref[s], rel=RTOL, abs=1e-15), s


@pytest.mark.parametrize("n, nh, one_block", [(10, 1, True), (10, 5, True), (11, 1, True), (11, 5, True), (11, 6, True),
                                              (11, 7, False), (11, 9, False), (11, 10, False), (12, 2, False)])
def test_one_block_where_its_lds_holds_everything(orc, n, nh, one_block):
    """The elements, two sets of amplitudes and the intermediates fit 150 KiB up to
    10 states, and of 11 up to 6 holes: on both sides of that every sweep's energy is
    the oracle's, of a run past one launch's 64 sweeps too.  A whole run then waits for
    the stream once per launch of up to 64 sweeps, otherwise every four sweeps."""
    from test_gpu_batched import _kernels
    h, v = _random_hamiltonian(n, seed=n + nh)
    o = orc.O1(h, v, nh)
    ref = [o.sweep(0.8, ccd.CCD_T_ALL) for _ in range(70)]
    r = ccd.dense_solve(h, v, nh, mixing=0.8, tol=0.0, max_iter=70)
    assert r["sweeps"] == 70
    for s in range(70):
        assert r["history"][s] == pytest.approx(ref[s], rel=RTOL, abs=1e-15), s
    names = _kernels(lambda: ccd.dense_solve(h, v, nh, mixing=0.8, tol=0.0, max_iter=2), "k_dense_mbpt2")
    assert ("k_dense_one" in names, "k_dense_new" in names) == (one_block, not one_block)
