"""Parity of the HIP path (through the C ABI) with the CPU oracle.

Tolerances:
* matrix-vector product, FP64: every element within 1e-12 of max|y| (the
  FFT route and the dense sum differ only by rounding, ~1e-15 log2 M);
* FP32 matvec mode: within 2e-5 of max|y| (single-precision FFT, ~1e-7
  log2 M per pass, three passes each way);
* solutions at tolerance h: P within ~10 h of the LU solution (the true
  residual bound times a modest condition number), Q within 1e-4 relative of
  the oracle (the target this build works to).
"""
import dataclasses
import math

import numpy as np
import pytest
import torch

import workloads as w
from oracle import adjoint, dense, fftsolve, mie

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dda():
    import paper_1202_3424_amd as pkg
    assert torch.cuda.is_available()
    return pkg


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _dense_A(ijk, m, x, kh, e0, scheme):
    k = dense.kd_from_size_parameter(x, len(ijk))
    ainv = dense.site_alpha_inverse(np.asarray(m), k, kh, e0, scheme)
    return dense.assemble(ijk, ainv, k)


def _ragged():
    rng = np.random.default_rng(17)
    pts = rng.integers(0, [9, 7, 13], size=(300, 3))
    return np.unique(pts, axis=0).astype(np.int32)


MATVEC_CASES = {
    "sphere389": lambda: (w.sphere_integer(4.5), 1.33 + 0.01j),
    "ragged_9x7x13": lambda: (_ragged(), 1.5 + 0.2j),
    "line_z9": lambda: (np.array([[0, 0, i] for i in range(9)], dtype=np.int32), 2.0 + 0.5j),
    "single_site": lambda: (np.array([[3, -2, 5]], dtype=np.int32), 1.7 + 0.3j),
    "box_8x3x40": lambda: (w.brick(8, 3, 40), 1.6 + 0.1j),
    # three perpendicular lines: padded extents 192 (x, z) and 160 (y)
    "lines_96_80_96": lambda: (np.unique(np.vstack([[[i, 0, 0] for i in range(96)], [[0, j, 0] for j in range(80)],
                                                    [[0, 0, k] for k in range(96)]]), axis=0).astype(np.int32),
                               1.5 + 0.05j),
}


@pytest.mark.parametrize("name", sorted(MATVEC_CASES))
@pytest.mark.parametrize("scheme", ["LATTDR", "GKDLDR"])
def test_matvec_matches_dense(dda, name, scheme):
    ijk, mval = MATVEC_CASES[name]()
    n = len(ijk)
    m = np.full(n, mval)
    if name == "box_8x3x40":
        m = np.where(np.arange(n) % 3 == 0, mval, 1.2 + 0.0j)
    x = 1.3
    kh = np.array([[1, 0, 0], [0.36, 0.48, 0.8]])
    e0 = np.array([[0, 1, 0], np.array([0.8, -0.6, 0]) + 1j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    tgt = dda.Target(ijk, m)
    opts = dda.Options.for_size_parameter(x, polarizability=scheme)
    xv = w.random_vectors(3, (2, n, 3))
    y = dda.apply(tgt, opts, kh, e0, _cuda(xv)).cpu().numpy()
    for q in range(2):
        A = _dense_A(ijk, m, x, kh[q], e0[q], scheme)
        ref = (A @ xv[q].reshape(-1)).reshape(n, 3)
        err = np.abs(y[q] - ref).max()
        assert err <= 1e-12 * np.abs(ref).max(), (name, q, err)


def test_matvec_fp32_mode(dda):
    ijk = _ragged()
    n = len(ijk)
    m = np.full(n, 1.5 + 0.2j)
    tgt = dda.Target(ijk, m)
    opts = dda.Options.for_size_parameter(1.3, precision="fp32_matvec")
    kh, e0 = w.along_x_yz()
    xv = w.random_vectors(4, (2, n, 3))
    y = dda.apply(tgt, opts, kh, e0, _cuda(xv)).cpu().numpy()
    for q in range(2):
        ref = (_dense_A(ijk, m, 1.3, kh[q], e0[q], "LATTDR") @ xv[q].reshape(-1)).reshape(n, 3)
        assert np.abs(y[q] - ref).max() <= 2e-5 * np.abs(ref).max()


def test_matvec_full_size_ellipsoid(dda):
    """The 51,488-site ellipsoid on its 128x96x64 grid: every element of
    A x against the oracle's FFT operator (the bench's launch configuration)."""
    d = w.workload("ellipsoid51k")
    n = len(d["ijk"])
    tgt = dda.Target(d["ijk"], d["m"])
    assert tgt.grid == (128, 96, 64)
    opts = dda.Options.for_size_parameter(d["x"])
    xv = w.random_vectors(5, (1, n, 3))
    y = dda.apply(tgt, opts, d["khat"][:1], d["e0"][:1], _cuda(xv)).cpu().numpy()[0]
    k = dense.kd_from_size_parameter(d["x"], n)
    ainv = dense.site_alpha_inverse(d["m"], k, d["khat"][0], d["e0"][0])
    ref = fftsolve.FFTOperator(d["ijk"], ainv, k).apply(xv[0])
    assert np.abs(y - ref).max() <= 1e-12 * np.abs(ref).max()


# ------------------------------------------------------------------ solves

def test_solve_sphere389_vs_lu_and_mie(dda):
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8)
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    P = P.cpu().numpy()
    q_mie = mie.efficiencies(1.33 + 0.01j, 1.0)
    for q in range(2):
        lu = dense.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q])
        r = res[q]
        assert r["status"] == 0 and r["rel_residual"] < 1e-8
        assert np.abs(P[q] - lu["P"]).max() <= 1e-7 * np.abs(lu["P"]).max()
        for key in ("qext", "qabs", "qsca", "qpha"):
            assert abs(r[key] - lu[key]) <= 1e-7 * abs(lu[key]), key
            if key != "qpha":
                assert abs(r[key] / q_mie[key] - 1) < 0.03
        tr, ne = dense.residuals(lu["A"], P[q], lu["E"])
        assert abs(r["rel_residual"] - tr) <= 0.05 * tr + 1e-15
        assert abs(r["normal_eq_residual"] - ne) <= 0.05 * ne + 1e-15
        assert abs(r["kd"] - lu["k"]) < 1e-14


@pytest.mark.parametrize("scheme", ["LATTDR", "GKDLDR"])
def test_solve_two_material_vs_lu(dda, scheme):
    d = w.workload("twomat6")
    tgt = dda.Target(d["ijk"], d["m"])
    kh = np.array([[0.36, 0.48, 0.8]])
    e0 = np.array([np.array([0.8, -0.6, 0]) + 0.5j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-10, polarizability=scheme)
    P, res = dda.solve(tgt, opts, kh, e0)
    lu = dense.solve_case(d["ijk"], d["m"], d["x"], kh[0], e0[0], scheme)
    assert res[0]["status"] == 0
    assert np.abs(P.cpu().numpy()[0] - lu["P"]).max() <= 1e-8 * np.abs(lu["P"]).max()
    assert abs(res[0]["qabs"] - lu["qabs"]) <= 1e-8 * lu["qabs"]
    assert abs(res[0]["qsca"] - lu["qsca"]) <= 1e-8 * lu["qsca"]


def test_worked_example_on_gpu(dda):
    """The guide's printed 16x32x32 gold brick (GKDLDR, TOL 1e-5)."""
    import json
    import os
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "worked_example_au_brick.json")))
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(g["x"], tol=1e-5, polarizability="GKDLDR")
    _, res = dda.solve(tgt, opts, d["khat"], d["e0"], want_P=False)
    for r in res:
        assert r["status"] == 0
        for key in ("qext", "qabs", "qsca", "qpha"):
            assert abs(r[key] - g[key]) <= 1e-4 * abs(g[key]) + 5e-6, (key, r[key])
    assert abs(res[0]["qext"] - res[1]["qext"]) < 1e-4


def test_solve_full_size_ellipsoid_vs_oracle(dda):
    """The 51,488-site ellipsoid at tol 1e-5 (the benchmark workload):
    Q within 1e-4 of the oracle's FFT-BiCGSTAB, P close at sampled sites;
    the iteration count within one of the oracle's at the same tolerance,
    two products per iteration (a half-step convergence included)."""
    d = w.workload("ellipsoid51k")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5)
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    P = P.cpu().numpy()
    rng = np.random.default_rng(0)
    sample = rng.choice(len(d["ijk"]), 500, replace=False)
    for q in range(2):
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-9)
        r = res[q]
        assert r["status"] == 0 and r["rel_residual"] < 1e-5
        for key in ("qext", "qabs", "qsca"):
            assert abs(r[key] - o[key]) <= 1e-4 * abs(o[key]), (key, r[key], o[key])
        assert np.abs(P[q][sample] - o["P"][sample]).max() <= 1e-3 * np.abs(o["P"]).max()
        o5 = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-5)
        assert abs(r["iters"] - o5["iters"]) <= 1 and r["matvecs"] == 2 * r["iters"], (r, o5["iters"])


def test_batched_equals_single_bitwise(dda):
    """Each right-hand side of a batch is computed with exactly the
    arithmetic of its single solve (no cross-RHS mixing)."""
    d = w.workload("brick48")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5)
    kh, e0 = d["khat"][:6], d["e0"][:6]
    Pb, rb = dda.solve(tgt, opts, kh, e0)
    for q in (0, 3, 5):
        Ps, rs = dda.solve(tgt, opts, kh[q:q + 1], e0[q:q + 1])
        assert torch.equal(Pb[q], Ps[0])
        assert rb[q]["qext"] == rs[0]["qext"] and rb[q]["iters"] == rs[0]["iters"]


def test_deterministic(dda):
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8)
    P1, r1 = dda.solve(tgt, opts, d["khat"], d["e0"])
    P2, r2 = dda.solve(tgt, opts, d["khat"], d["e0"])
    assert torch.equal(P1, P2) and r1 == r2


def test_warm_start_at_solution(dda):
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8)
    P, _ = dda.solve(tgt, opts, d["khat"], d["e0"])
    P2, res = dda.solve(tgt, opts, d["khat"], d["e0"], P0=P)
    assert all(r["iters"] == 0 and r["status"] == 0 for r in res)
    assert torch.equal(P, P2)


def test_error_paths(dda):
    from paper_1202_3424_amd import DDAError
    ijk = w.sphere_integer(2.0)
    with pytest.raises(DDAError) as e:
        dda.Target(np.vstack([ijk, ijk[:1]]), 1.5)
    assert e.value.status == 1 and "duplicate" in str(e.value)
    with pytest.raises(DDAError):
        dda.Target(ijk, np.full(len(ijk), complex(np.nan, 0)))
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    opts = dda.Options.for_size_parameter(1.0)
    with pytest.raises(DDAError):      # e0 not transverse to khat
        dda.solve(tgt, opts, [[1, 0, 0]], [[1, 0, 0]])
    with pytest.raises(DDAError):      # khat not unit
        dda.solve(tgt, opts, [[2, 0, 0]], [[0, 1, 0]])
    with pytest.raises(DDAError):
        dda.solve(tgt, dda.Options.for_size_parameter(1.0, tol=-1.0), [[1, 0, 0]], [[0, 1, 0]])
    _, res = dda.solve(tgt, dda.Options.for_size_parameter(1.0, tol=1e-14, max_iter=1), [[1, 0, 0]], [[0, 1, 0]])
    assert res[0]["status"] == 4 and res[0]["iters"] == 1 and res[0]["qext"] > 0


def test_validity_warning(dda):
    ijk = w.brick(6, 6, 6)
    tgt = dda.Target(ijk, 2.0 + 0.5j)
    _, res = dda.solve(tgt, dda.Options.for_size_parameter(6.0, tol=1e-4), [[1, 0, 0]], [[0, 1, 0]], want_P=False)
    assert "|m|kd" in dda.last_error()


def test_fp32_matvec_solve(dda):
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5, precision="fp32_matvec")
    _, res = dda.solve(tgt, opts, d["khat"], d["e0"], want_P=False)
    for q in range(2):
        lu = dense.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], with_qsca=False)
        assert res[q]["status"] == 0 and res[q]["rel_residual"] < 2e-5
        assert abs(res[q]["qext"] - lu["qext"]) <= 1e-4 * lu["qext"]
        assert abs(res[q]["qabs"] - lu["qabs"]) <= 1e-4 * lu["qabs"]


@pytest.mark.parametrize("weights", [(1.0, 0.0), (0.0, 1.0), (0.7, -0.3)])
def test_adjoint_gradient_vs_dense(dda, weights):
    d = w.workload("twomat6")
    kh, e0 = d["khat"][0], d["e0"][0]
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-11)
    P, _ = dda.solve(tgt, opts, [kh], [e0])
    g, adj = dda.grad_eps(tgt, opts, kh, e0, P[0], *weights)
    ref, _ = adjoint.gradient_dense(d["ijk"], d["m"], d["x"], kh, e0, *weights)
    assert adj["status"] == 0
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-7 * np.abs(ref).max()


def test_autotuned_variants_bitwise_equal_default(dda):
    """Every compile-time tiling of the strided passes computes the same
    numbers: the autotuned solve equals the default-tiling solve bitwise."""
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    base = dict(tol=1e-5, polarizability="GKDLDR")
    P1, r1 = dda.solve(tgt, dda.Options.for_size_parameter(d["x"], autotune=True, **base), d["khat"], d["e0"])
    P2, r2 = dda.solve(tgt, dda.Options.for_size_parameter(d["x"], autotune=False, **base), d["khat"], d["e0"])
    assert torch.equal(P1, P2) and r1 == r2


# ------------------------------------------------------------------ mixed precision

def test_mixed_precision_matches_fp64_solve(dda):
    """FP32 FFT matvec with FP64 recurrences and FP64 residual refinement:
    the true (FP64) residual meets the tolerance and Q agrees with the FP64
    solve to 1e-4."""
    ijk = w.box_sphere(48, 24.0)
    m = np.full(len(ijk), 1.33 + 0.01j)
    tgt = dda.Target(ijk, m)
    kh, e0 = w.along_x_yz()
    o64 = dda.Options.for_size_parameter(8.0, tol=1e-5)
    o32 = dda.Options.for_size_parameter(8.0, tol=1e-5, precision="fp32_matvec")
    _, r64 = dda.solve(tgt, o64, kh, e0, want_P=False)
    _, r32 = dda.solve(tgt, o32, kh, e0, want_P=False)
    for a, b in zip(r32, r64):
        assert a["status"] == 0 and a["rel_residual"] < 1e-5, a
        for key in ("qext", "qabs", "qsca"):
            assert abs(a[key] - b[key]) <= 1e-4 * abs(b[key]), (key, a[key], b[key])


def test_sphere1m_full_size(dda):
    """The 1,099,136-site sphere on its 256^3 grid: sampled rows of A x in FP64
    and FP32 against the oracle's direct sums; the FP64 and FP32-matvec solves
    against the oracle's FP64 FFT-BiCGSTAB solution (tests/golden/
    sphere1m_oracle.json, written by make_sphere1m_oracle.py from the oracle
    alone: Q within 1e-4, P at its 64 stored sites within 1e-3 of max|P|),
    against each other (1e-4) and against Mie theory (the DDA error bound per
    quantity)."""
    d = w.workload("sphere1m")
    n = len(d["ijk"])
    tgt = dda.Target(d["ijk"], d["m"])
    assert tgt.grid == (256, 256, 256)
    k = dense.kd_from_size_parameter(d["x"], n)
    ainv = dense.site_alpha_inverse(d["m"], k, d["khat"][0], d["e0"][0])
    xv = w.random_vectors(8, (1, n, 3))
    rows = np.random.default_rng(1).choice(n, 12, replace=False)
    ref = dense.apply_rows(d["ijk"], ainv, k, xv[0], rows)
    for prec, tol in (("fp64", 1e-12), ("fp32_matvec", 2e-5)):
        o = dda.Options.for_size_parameter(d["x"], precision=prec)
        y = dda.apply(tgt, o, d["khat"][:1], d["e0"][:1], _cuda(xv)).cpu().numpy()[0]
        assert np.abs(y[rows] - ref).max() <= tol * np.abs(ref).max(), prec
    o64 = dda.Options.for_size_parameter(d["x"], tol=1e-5)
    o32 = dda.Options.for_size_parameter(d["x"], tol=1e-5, precision="fp32_matvec")
    P64, r64 = dda.solve(tgt, o64, d["khat"], d["e0"])
    P32, r32 = dda.solve(tgt, o32, d["khat"], d["e0"])
    q_mie = mie.efficiencies(1.33 + 0.01j, d["x"])
    import json
    import os
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "sphere1m_oracle.json")))
    assert g["n_sites"] == n and abs(g["kd"] - k) < 1e-14
    sample = np.array(g["sample_sites"])
    for q, ref in enumerate(g["rhs"]):
        assert ref["converged"] and ref["true_residual"] < 1e-6
        Pref = np.array(ref["P_sample_re"]) + 1j * np.array(ref["P_sample_im"])
        for r, P in ((r64[q], P64), (r32[q], P32)):
            for key in ("qext", "qabs", "qsca"):
                assert abs(r[key] - ref[key]) <= 1e-4 * abs(ref[key]), (q, key, r[key], ref[key])
            Ps = P[q].cpu().numpy()[sample]
            assert np.abs(Ps - Pref).max() <= 1e-3 * np.abs(Pref).max()
    for a, b in zip(r32, r64):
        assert a["status"] == 0 and b["status"] == 0
        assert a["rel_residual"] < 1e-5 and b["rel_residual"] < 1e-5
        for key in ("qext", "qabs", "qsca"):
            assert abs(a[key] - b[key]) <= 1e-4 * abs(b[key]), (key, a[key], b[key])
        assert abs(b["qext"] / q_mie["qext"] - 1) < 0.05
        assert abs(b["qsca"] / q_mie["qsca"] - 1) < 0.05
        assert abs(b["qabs"] / q_mie["qabs"] - 1) < 0.10


# boxes whose padded grids put every compile-time FFT length on the y and
# the z axis (x extents small and ragged: partial column tiles)
VARIANT_BOXES = [(13, 14, 32), (5, 24, 16), (5, 40, 48), (3, 64, 40), (3, 32, 128), (3, 128, 64), (3, 80, 96),
                 (3, 96, 80)]


def _box_target(dda, box, seed):
    rng = np.random.default_rng(seed)
    ijk = np.argwhere(rng.random(box) < 0.3).astype(np.int32)
    ijk = np.unique(np.vstack([ijk, [[0, 0, 0], [b - 1 for b in box]]]), axis=0).astype(np.int32)
    return dda.Target(ijk, np.full(len(ijk), 1.4 + 0.1j))


@pytest.mark.parametrize("variant", range(2, 29))
def test_every_tiling_variant_bitwise(dda, variant):
    """Each compile-time form of the strided passes (LDS tilings, the
    octant-folded z pass, the register-resident passes) gives the default
    form's product bitwise, for every compile-time length on the y and z
    axes, with ragged x tiles and two right-hand sides."""
    kh = np.array([[1, 0, 0], [0.36, 0.48, 0.8]])
    e0 = np.array([[0, 1, 0], np.array([0.8, -0.6, 0]) + 1j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    seen = set()
    for bi, box in enumerate(VARIANT_BOXES):
        tgt = _box_target(dda, box, 90 + bi)
        seen.update(tgt.grid[1:])
        xv = _cuda(w.random_vectors(6 + bi, (2, tgt.n_sites, 3)))
        for prec in ("fp64", "fp32_matvec"):
            ref = dda.apply(tgt, dda.Options.for_size_parameter(1.1, precision=prec, kernel_variant=1), kh, e0, xv)
            y = dda.apply(tgt, dda.Options.for_size_parameter(1.1, precision=prec, kernel_variant=variant), kh, e0,
                          xv)
            assert torch.equal(y, ref), (prec, variant, box, tgt.grid)
    assert {32, 48, 64, 80, 96, 128, 160, 192, 256} <= seen


def test_gather_forms_agree_bitwise(dda):
    """The gather loads its site operands before the inverse x transform in
    launches of at most 16 right-hand sides and after it in larger ones: a
    20-RHS product equals, bitwise, the same right-hand sides as two 10-RHS
    products, in FP64 and FP32, at a compile-time and a runtime length."""
    kh, e0 = w.incidences_for_orientations(41, 10)
    for bi, box in enumerate([(13, 14, 32), (9, 27, 11)]):
        tgt = _box_target(dda, box, 140 + bi)
        xv = _cuda(w.random_vectors(50 + bi, (20, tgt.n_sites, 3)))
        for prec in ("fp64", "fp32_matvec"):
            o = dda.Options.for_size_parameter(1.3, precision=prec)
            y = dda.apply(tgt, o, kh, e0, xv)
            y0 = dda.apply(tgt, o, kh[:10], e0[:10], xv[:10].contiguous())
            y1 = dda.apply(tgt, o, kh[10:], e0[10:], xv[10:].contiguous())
            assert torch.equal(y[:10], y0) and torch.equal(y[10:], y1), (prec, box, tgt.grid)


# ------------------------------------------------------------------ adjoint at full size

def _dq_difference(P, dP, E, w_sites, w_site_new, j, cq, wq):
    """Exact change of w_abs Q_abs + w_ext Q_ext when site j's 1/alpha changes
    and P -> P + dP (the algebraic difference of the oracle's formulas)."""
    w_abs, w_ext = wq
    Pn = P + dP
    d_abs = np.sum(w_sites * (2 * np.real(np.conj(P) * dP) + np.abs(dP) ** 2))
    d_abs += np.sum((w_site_new - w_sites[j]) * np.abs(Pn[j]) ** 2)
    d_ext = np.sum(np.imag(np.conj(E) * dP))
    return cq * (w_abs * d_abs + w_ext * d_ext)


def test_adjoint_gradient_40cubed_vs_finite_differences(dda):
    """The 40^3 two-material target (N = 64,000): the adjoint gradient of
    Q_abs + 0.5 Q_ext with respect to eps_j against central differences on
    the 20 seeded sites.  Each difference solves the perturbed system for the
    change dP with the localized right-hand side -dA_j P (the difference
    formulation), so the finite difference is not swamped by solver error."""
    d = w.workload("twomat40")
    ijk, m = d["ijk"], d["m"]
    kh, e0 = d["khat"][0], d["e0"][0]
    n = len(ijk)
    wq = (1.0, 0.5)
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-11)
    tgt = dda.Target(ijk, m)
    P, _ = dda.solve(tgt, opts, [kh], [e0])
    g, adj = dda.grad_eps(tgt, opts, kh, e0, P[0], *wq)
    assert adj["status"] == 0
    g = g.cpu().numpy()
    Pn = P[0].cpu().numpy()
    k = dense.kd_from_size_parameter(d["x"], n)
    cq = dense.q_prefactor(k, n)
    ainv = dense.site_alpha_inverse(m, k, kh, e0)
    w_sites = -np.imag(ainv) - (2.0 / 3.0) * k ** 3
    E = dense.incident_field(ijk, k, kh, e0)
    eps = np.asarray(m) ** 2
    for j in w.fd_sites(0):
        h = 1e-3 * abs(eps[j])
        dq = []
        for step in (h, -h, 1j * h, -1j * h):
            m_new = m.copy()
            m_new[j] = np.sqrt(eps[j] + step)
            ainv_j = dense.alpha_inverse(m_new[j], k, kh, e0)
            b = np.zeros((1, n, 3), dtype=np.complex128)
            b[0, j] = -(ainv_j - ainv[j]) * Pn[j]
            dP, r = dda.solve_rhs(dda.Target(ijk, m_new), opts, [kh], [e0], _cuda(b))
            assert r[0]["status"] == 0
            w_new = -np.imag(ainv_j) - (2.0 / 3.0) * k ** 3
            dq.append(_dq_difference(Pn, dP.cpu().numpy()[0], E, w_sites, w_new, j, cq, wq))
        fd = (dq[0] - dq[1]) / (2 * h) + 1j * (dq[2] - dq[3]) / (2 * h)
        assert abs(g[j] - fd) <= 1e-5 * np.abs(g).max() + 1e-6 * abs(fd), (j, g[j], fd)


def test_adjoint_gradient_40cubed_fp32_matvec(dda):
    """The FP32-matvec variant of the adjoint gradient against the FP64 one."""
    d = w.workload("twomat40")
    kh, e0 = d["khat"][0], d["e0"][0]
    tgt = dda.Target(d["ijk"], d["m"])
    grads = []
    for prec in ("fp64", "fp32_matvec"):
        opts = dda.Options.for_size_parameter(d["x"], tol=1e-6, precision=prec)
        P, _ = dda.solve(tgt, opts, [kh], [e0])
        g, adj = dda.grad_eps(tgt, opts, kh, e0, P[0], 1.0, 0.0)
        assert adj["status"] == 0
        grads.append(g.cpu().numpy())
    assert np.abs(grads[1] - grads[0]).max() <= 1e-4 * np.abs(grads[0]).max()


def test_qeff_autograd_function(dda):
    """QEff (torch.autograd.Function) on the 6^3 two-material target: the
    values and the gradient of Q_abs + 0.3 Q_ext against the dense oracle."""
    d = w.workload("twomat6")
    kh, e0 = d["khat"][0], d["e0"][0]
    eps = torch.tensor(np.asarray(d["m"]) ** 2, dtype=torch.complex128, device="cuda", requires_grad=True)
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-11)
    q = dda.QEff.apply(eps, d["ijk"], opts, kh, e0)
    (q[0] + 0.3 * q[1]).backward()
    ref, sol = adjoint.gradient_dense(d["ijk"], d["m"], d["x"], kh, e0, 1.0, 0.3)
    assert abs(q[0].item() - sol["qabs"]) <= 1e-8 * sol["qabs"]
    assert abs(q[1].item() - sol["qext"]) <= 1e-8 * sol["qext"]
    assert np.abs(eps.grad.cpu().numpy() - ref).max() <= 1e-7 * np.abs(ref).max()


# ------------------------------------------------------------------ batched / ragged

def test_solve_batched_matches_separate_solves(dda):
    """A ragged batch (a brick with 16 right-hand sides and six spheres of
    different grids, two each) solved concurrently in one call gives every
    right-hand side bitwise the result of solving its target alone."""
    d = w.workload("brick48")
    brick = dda.Target(d["ijk"], d["m"])
    radii = w.sphere_radii(0)[:6]
    spheres = [dda.Target(w.sphere_integer(r), 1.33 + 0.01j) for r in radii]
    kh_s, e0_s = w.along_x_yz()
    targets = [brick] + spheres
    opts = [dda.Options.for_size_parameter(d["x"], tol=1e-5)] + \
           [dda.Options.for_size_parameter(4.0, tol=1e-5) for _ in spheres]
    kh = np.vstack([d["khat"][:16]] + [kh_s] * len(spheres))
    e0 = np.vstack([d["e0"][:16]] + [e0_s] * len(spheres))
    rt = [0] * 16 + [1 + i // 2 for i in range(2 * len(spheres))]
    Ps, res = dda.solve_batched(targets, opts, rt, kh, e0)
    P0, r0 = dda.solve(brick, opts[0], d["khat"][:16], d["e0"][:16])
    for q in range(16):
        assert torch.equal(Ps[q], P0[q]) and res[q] == r0[q]
    q_mie = mie.efficiencies(1.33 + 0.01j, 4.0)
    for i, t in enumerate(spheres):
        Pi, ri = dda.solve(t, opts[1 + i], kh_s, e0_s)
        for k in range(2):
            g = 16 + 2 * i + k
            assert torch.equal(Ps[g], Pi[k]) and res[g] == ri[k]
            assert res[g]["status"] == 0
            assert abs(res[g]["qext"] / q_mie["qext"] - 1) < 0.05
            assert abs(res[g]["qsca"] / q_mie["qsca"] - 1) < 0.05


def _shared_grid_targets(dda):
    """Four targets on the 32^3 padded grid with different boxes, site
    counts, material counts and sizes: spheres of radius 5.5, 6.2 and 7.9 and
    a two-material 12 x 11 x 14 brick."""
    ts = [dda.Target(w.sphere_integer(r), m) for r, m in ((5.5, 1.33 + 0.01j), (6.2, 1.5 + 0.1j),
                                                          (7.9, 1.7 + 0.05j))]
    b = w.brick(12, 11, 14)
    mb = np.where(np.arange(len(b)) % 3 == 0, 1.4 + 0.02j, 2.0 + 0.3j)
    ts.append(dda.Target(b, mb))
    for t in ts:
        assert tuple(t.grid) == (32, 32, 32)
    return ts


@pytest.mark.parametrize("solver,precision", [("bicgstab", "fp64"), ("bicgstab", "fp32_matvec"),
                                              ("qmr", "fp64"), ("qmr", "fp32_matvec"),
                                              ("bicgstab2", "fp64"), ("bicgstab2", "fp32_matvec")])
def test_shared_launch_batch_matches_separate_solves(dda, solver, precision):
    """Targets on one padded grid share every launch of dda_solve_batched
    (each right-hand side reads its own box, sites, materials, kd and tensor
    through the per-right-hand-side table).  Every right-hand side's P and
    result equal, bitwise, those of solving its target alone, for each solver
    and precision, with per-target tolerance, size parameter and
    polarizability; with share_launches off too."""
    ts = _shared_grid_targets(dda)
    xs = (2.0, 3.1, 2.6, 1.7)
    tols = (1e-5, 1e-6, 3e-5, 1e-5)
    polz = ("LATTDR", "GKDLDR", "LATTDR", "LATTDR")
    opts = [dda.Options.for_size_parameter(x, tol=tol, polarizability=pz, solver=solver, precision=precision)
            for x, tol, pz in zip(xs, tols, polz)]
    kh_all, e0_all = w.incidences_for_orientations(11, 3)
    counts = (2, 3, 1, 2)
    rt, kh, e0 = [], [], []
    for i, c in enumerate(counts):
        rt += [i] * c
        kh.append(kh_all[:c])
        e0.append(e0_all[:c])
    # interleave the right-hand sides of different targets
    order = [0, 2, 5, 1, 3, 6, 4, 7]
    rt = np.array(rt)[order]
    kh = np.vstack(kh)[order]
    e0 = np.vstack(e0)[order]
    Ps, res = dda.solve_batched(ts, opts, rt, kh, e0)
    noshare = [dataclasses.replace(o, share_launches=False) for o in opts]
    Pn, rn = dda.solve_batched(ts, noshare, rt, kh, e0)
    for i, t in enumerate(ts):
        qs = [q for q in range(len(rt)) if rt[q] == i]
        P1, r1 = dda.solve(t, opts[i], kh[qs], e0[qs])
        for k, q in enumerate(qs):
            assert res[q]["status"] == 0, (i, res[q])
            assert torch.equal(Ps[q], P1[k]) and res[q] == r1[k], (i, q)
            assert torch.equal(Pn[q], P1[k]) and rn[q] == r1[k], (i, q)


@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
def test_shared_launch_batch_with_chained_finalize(dda, precision):
    """Spheres of radius 30 and 28 (113,081 and 91,965 sites) on one 128^3
    grid: their x passes have 3,721 and 3,249 workgroups per right-hand side,
    so the finalizes of the products run from per-thread sums formed one
    workgroup per slot, in the shared-launch batch with each right-hand
    side's own count from the batch table.  Every P and result equals,
    bitwise, that of solving its target alone."""
    ts = [dda.Target(w.sphere_integer(30.0), 1.33 + 0.01j), dda.Target(w.sphere_integer(28.0), 1.5 + 0.05j)]
    for t in ts:
        assert tuple(t.grid) == (128, 128, 128)
    opts = [dda.Options.for_size_parameter(x, precision=precision) for x in (3.0, 2.6)]
    kh, e0 = w.along_x_yz()
    rt = np.array([0, 1, 0, 1])
    khb, e0b = np.vstack([kh[:1], kh[:1], kh[1:], kh[1:]]), np.vstack([e0[:1], e0[:1], e0[1:], e0[1:]])
    Ps, res = dda.solve_batched(ts, opts, rt, khb, e0b)
    for i, t in enumerate(ts):
        qs = [q for q in range(len(rt)) if rt[q] == i]
        P1, r1 = dda.solve(t, opts[i], khb[qs], e0b[qs])
        for k, q in enumerate(qs):
            assert res[q]["status"] == 0, (i, res[q])
            assert torch.equal(Ps[q], P1[k]) and res[q] == r1[k], (i, q)


def test_batch_schedule_leaves_results_unchanged(dda):
    """Repeated calls of one batch shape run with 4, 2 and 1 jobs in flight
    while the schedule is tried, then with the fastest: every call gives the
    same P and results, bitwise."""
    ts = _shared_grid_targets(dda)[:2] + [dda.Target(w.sphere_integer(12.2), 1.4 + 0.02j),
                                          dda.Target(w.brick(20, 9, 7), 1.6 + 0.1j)]
    opts = [dda.Options.for_size_parameter(x, tol=1e-5) for x in (2.0, 2.4, 3.0, 1.5)]
    kh, e0 = w.along_x_yz()
    rt = [0, 0, 1, 1, 2, 2, 3, 3]
    kh8, e08 = np.vstack([kh] * 4), np.vstack([e0] * 4)
    P0, r0 = dda.solve_batched(ts, opts, rt, kh8, e08)
    for _ in range(5):
        P1, r1 = dda.solve_batched(ts, opts, rt, kh8, e08)
        assert r1 == r0
        assert all(torch.equal(a, b) for a, b in zip(P0, P1))


def test_shared_launch_batch_rejects_one_target_at_two_kd(dda):
    """A target listed twice must have one kd (it holds one tensor)."""
    t = _shared_grid_targets(dda)[0]
    o1 = dda.Options.for_size_parameter(2.0)
    o2 = dda.Options.for_size_parameter(2.5)
    kh, e0 = w.along_x_yz()
    with pytest.raises(RuntimeError, match="listed twice"):
        dda.solve_batched([t, t], [o1, o2], [0, 1], kh, e0)


def test_config3_batch_full(dda):
    """The whole batched workload: the 48x24x16 brick at 64 random
    orientations x 2 polarizations and 32 ragged spheres x 2, one call.
    Spheres within 5% of Mie; two brick right-hand sides against the
    oracle's FFT-BiCGSTAB to 1e-4."""
    d = w.workload("brick48")
    brick = dda.Target(d["ijk"], d["m"])
    spheres = [dda.Target(s, 1.33 + 0.01j) for s in w.sphere_batch(0)]
    kh_s, e0_s = w.along_x_yz()
    targets = [brick] + spheres
    opts = [dda.Options.for_size_parameter(d["x"], tol=1e-5)] + \
           [dda.Options.for_size_parameter(4.0, tol=1e-5) for _ in spheres]
    kh = np.vstack([d["khat"]] + [kh_s] * len(spheres))
    e0 = np.vstack([d["e0"]] + [e0_s] * len(spheres))
    rt = [0] * 128 + [1 + i // 2 for i in range(64)]
    _, res = dda.solve_batched(targets, opts, rt, kh, e0, want_P=False)
    assert all(r["status"] == 0 and r["rel_residual"] < 1e-5 for r in res)
    q_mie = mie.efficiencies(1.33 + 0.01j, 4.0)
    for r in res[128:]:
        assert abs(r["qext"] / q_mie["qext"] - 1) < 0.05
        assert abs(r["qsca"] / q_mie["qsca"] - 1) < 0.05
    for q in (0, 77):
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-9)
        for key in ("qext", "qabs", "qsca"):
            assert abs(res[q][key] - o[key]) <= 1e-4 * abs(o[key]), (q, key)


# ------------------------------------------------------------------ QMR (complex-symmetric)

def test_qmr_sphere389_vs_lu_and_oracle(dda):
    """QMR on the GPU reaches the LU solution, with the oracle's QMR
    iteration count (the smoothed-residual test decided on the device from
    its norm recurrence, on the CPU from the vector)."""
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8, solver="qmr")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    P = P.cpu().numpy()
    for q in range(2):
        lu = dense.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], with_qsca=False)
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-8, solver="qmr")
        r = res[q]
        assert r["status"] == 0 and r["rel_residual"] < 1e-8
        assert abs(r["iters"] - o["iters"]) <= 1 and r["matvecs"] == r["iters"]
        assert np.abs(P[q] - lu["P"]).max() <= 1e-7 * np.abs(lu["P"]).max()
        assert np.abs(P[q] - o["P"]).max() <= 1e-7 * np.abs(lu["P"]).max()
        for key in ("qext", "qabs", "qpha"):
            assert abs(r[key] - lu[key]) <= 1e-7 * abs(lu[key]), key


@pytest.mark.parametrize("scheme", ["LATTDR", "GKDLDR"])
def test_qmr_two_material_vs_lu(dda, scheme):
    d = w.workload("twomat6")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-10, polarizability=scheme, solver="qmr")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    lu = dense.solve_case(d["ijk"], d["m"], d["x"], d["khat"][0], d["e0"][0], scheme=scheme, with_qsca=False)
    assert res[0]["status"] == 0
    assert np.abs(P[0].cpu().numpy() - lu["P"]).max() <= 1e-8 * np.abs(lu["P"]).max()


def test_qmr_worked_example(dda):
    """The guide's printed gold brick solved with QMR (GKDLDR, TOL 1e-5)."""
    import json
    import os
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "worked_example_au_brick.json")))
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(g["x"], tol=1e-5, polarizability="GKDLDR", solver="qmr")
    _, res = dda.solve(tgt, opts, d["khat"], d["e0"], want_P=False)
    for r in res:
        assert r["status"] == 0 and r["rel_residual"] < 1e-5
        for key in ("qext", "qabs", "qsca", "qpha"):
            assert abs(r[key] - g[key]) <= 1e-4 * abs(g[key]) + 5e-6, (key, r[key])


def test_qmr_full_size_ellipsoid_vs_oracle(dda):
    """The 51,488-site ellipsoid with QMR at tol 1e-5: Q within 1e-4 of the
    oracle (tight solve), iterations within one of the oracle's QMR."""
    d = w.workload("ellipsoid51k")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="qmr")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    P = P.cpu().numpy()
    sample = np.random.default_rng(1).choice(len(d["ijk"]), 500, replace=False)
    for q in range(2):
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-9)
        oq = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-5, solver="qmr")
        r = res[q]
        assert r["status"] == 0 and r["rel_residual"] < 1e-5
        assert abs(r["iters"] - oq["iters"]) <= 1
        for key in ("qext", "qabs", "qsca"):
            assert abs(r[key] - o[key]) <= 1e-4 * abs(o[key]), (key, r[key], o[key])
        assert np.abs(P[q][sample] - o["P"][sample]).max() <= 1e-3 * np.abs(o["P"]).max()


def test_qmr_batched_deterministic_and_warm(dda):
    """QMR batches equal single solves bitwise, repeat bitwise, and a warm
    start at the solution takes no iteration."""
    d = w.workload("brick48")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="qmr")
    kh, e0 = d["khat"][:4], d["e0"][:4]
    Pb, rb = dda.solve(tgt, opts, kh, e0)
    Pb2, rb2 = dda.solve(tgt, opts, kh, e0)
    assert torch.equal(Pb, Pb2) and rb == rb2
    for q in (0, 3):
        Ps, rs = dda.solve(tgt, opts, kh[q:q + 1], e0[q:q + 1])
        assert torch.equal(Pb[q], Ps[0]) and rb[q]["iters"] == rs[0]["iters"]
    Pw, rw = dda.solve(tgt, opts, kh, e0, P0=Pb)
    assert all(r["iters"] == 0 and r["status"] == 0 for r in rw)
    assert torch.equal(Pw, Pb)


def test_qmr_fp32_matvec_matches_fp64(dda):
    """FP32-matvec QMR (with FP64 residual refinement) against FP64 QMR on
    the ellipsoid: the same residual bound and Q within 1e-4."""
    d = w.workload("ellipsoid51k")
    tgt = dda.Target(d["ijk"], d["m"])
    o64 = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="qmr")
    o32 = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="qmr", precision="fp32_matvec")
    _, r64 = dda.solve(tgt, o64, d["khat"], d["e0"], want_P=False)
    _, r32 = dda.solve(tgt, o32, d["khat"], d["e0"], want_P=False)
    for a, b in zip(r32, r64):
        assert a["status"] == 0 and a["rel_residual"] < 1e-5
        for key in ("qext", "qabs", "qsca"):
            assert abs(a[key] - b[key]) <= 1e-4 * abs(b[key]), key


def test_qmr_adjoint_gradient_vs_dense(dda):
    """The adjoint solve run with QMR gives the dense adjoint gradient."""
    d = w.workload("twomat6")
    kh, e0 = d["khat"][0], d["e0"][0]
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-11, solver="qmr")
    P, _ = dda.solve(tgt, opts, [kh], [e0])
    g, adj = dda.grad_eps(tgt, opts, kh, e0, P[0], 1.0, 0.5)
    ref, _ = adjoint.gradient_dense(d["ijk"], d["m"], d["x"], kh, e0, 1.0, 0.5)
    assert adj["status"] == 0
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-7 * np.abs(ref).max()


# ------------------------------------------------------------------ BiCGstab(2)

def test_bicgstab2_sphere389_vs_lu_and_oracle(dda):
    """BiCGstab(2) on the GPU reaches the LU solution with the oracle's
    iteration count (four products per iteration)."""
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8, solver="bicgstab2")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    P = P.cpu().numpy()
    for q in range(2):
        lu = dense.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], with_qsca=False)
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-8, solver="bicgstab2")
        r = res[q]
        assert r["status"] == 0 and r["rel_residual"] < 1e-8
        assert abs(r["iters"] - o["iters"]) <= 1 and r["matvecs"] == 4 * r["iters"]
        assert np.abs(P[q] - lu["P"]).max() <= 1e-7 * np.abs(lu["P"]).max()
        for key in ("qext", "qabs", "qpha"):
            assert abs(r[key] - lu[key]) <= 1e-7 * abs(lu[key]), key


def test_bicgstab2_worked_example(dda):
    """The guide's printed gold brick with its own solver choice (PBCGS2):
    the printed Q's, and iterations within 3 of the printed 18."""
    import json
    import os
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "worked_example_au_brick.json")))
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(g["x"], tol=1e-5, polarizability="GKDLDR", solver="bicgstab2")
    _, res = dda.solve(tgt, opts, d["khat"], d["e0"], want_P=False)
    for r, it in zip(res, g["pbcgs2_iterations"]):
        assert r["status"] == 0 and r["rel_residual"] < 1e-5
        assert abs(r["iters"] - it) <= 3
        for key in ("qext", "qabs", "qsca", "qpha"):
            assert abs(r[key] - g[key]) <= 1e-4 * abs(g[key]) + 5e-6, (key, r[key])


def test_bicgstab2_full_size_and_modes(dda):
    """The ellipsoid with BiCGstab(2): Q within 1e-4 of the oracle; batched
    equals single bitwise; FP32-matvec mode within 1e-4 of FP64; the adjoint
    solve with BiCGstab(2) gives the dense adjoint gradient."""
    d = w.workload("ellipsoid51k")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="bicgstab2")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    for q in range(2):
        o = fftsolve.solve_case(d["ijk"], d["m"], d["x"], d["khat"][q], d["e0"][q], tol=1e-9)
        assert res[q]["status"] == 0 and res[q]["rel_residual"] < 1e-5
        for key in ("qext", "qabs", "qsca"):
            assert abs(res[q][key] - o[key]) <= 1e-4 * abs(o[key]), key
    P1, r1 = dda.solve(tgt, opts, d["khat"][1:], d["e0"][1:])
    assert torch.equal(P1[0], P[1]) and r1[0]["iters"] == res[1]["iters"]
    o32 = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver="bicgstab2", precision="fp32_matvec")
    _, r32 = dda.solve(tgt, o32, d["khat"], d["e0"], want_P=False)
    for a, b in zip(r32, res):
        assert a["status"] == 0 and a["rel_residual"] < 1e-5
        assert abs(a["qext"] - b["qext"]) <= 1e-4 * abs(b["qext"])
    t = w.workload("twomat6")
    kh, e0 = t["khat"][0], t["e0"][0]
    tt = dda.Target(t["ijk"], t["m"])
    ot = dda.Options.for_size_parameter(t["x"], tol=1e-11, solver="bicgstab2")
    Pt, _ = dda.solve(tt, ot, [kh], [e0])
    g, adj = dda.grad_eps(tt, ot, kh, e0, Pt[0], 1.0, 0.5)
    ref, _ = adjoint.gradient_dense(t["ijk"], t["m"], t["x"], kh, e0, 1.0, 0.5)
    assert adj["status"] == 0
    assert np.abs(g.cpu().numpy() - ref).max() <= 1e-7 * np.abs(ref).max()


# ------------------------------------------------------------------ far field

def _random_frames(rng, n):
    v = rng.normal(size=(n, 3))
    nh = v / np.linalg.norm(v, axis=1, keepdims=True)
    u = np.cross(nh, rng.normal(size=(n, 3)))
    th = u / np.linalg.norm(u, axis=1, keepdims=True)
    return nh, th, np.cross(nh, th)


def test_far_field_amplitudes_match_oracle(dda):
    """dda_far_field against the oracle's direct sum on the same P, at
    random directions and frames, oblique elliptical incidence included."""
    from oracle import farfield
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    kh = np.array([[1, 0, 0], [0.36, 0.48, 0.8]])
    e0 = np.array([[0, 1, 0], np.array([0.8, -0.6, 0]) + 1j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-10)
    P, res = dda.solve(tgt, opts, kh, e0)
    nh, th, ph = _random_frames(np.random.default_rng(4), 50)
    f, dcs = dda.far_field(tgt, opts, P, nh, th, ph)
    Pn = P.cpu().numpy()
    for q in range(2):
        A = farfield.amplitude_vectors(d["ijk"], Pn[q], res[q]["kd"], nh)
        ref = np.stack([np.sum(th * A, axis=1), np.sum(ph * A, axis=1)], axis=1)
        assert np.abs(f[q] - ref).max() <= 1e-12 * np.abs(ref).max()
        rd = (np.abs(ref[:, 0]) ** 2 + np.abs(ref[:, 1]) ** 2) / res[q]["kd"] ** 2
        assert np.abs(dcs[q] - rd).max() <= 1e-12 * rd.max()
    with pytest.raises(dda.DDAError):
        dda.far_field(tgt, opts, P, nh, th, nh)


def test_worked_example_mueller_and_qbk_on_gpu(dda):
    """The guide's printed gold brick end to end on the GPU: solve (GKDLDR),
    far field at the 74 printed directions, Mueller elements from
    dda_mueller against the printed table and against the oracle's formulas
    on the same amplitudes, Q_bk against the printed value."""
    import json
    import os
    from oracle import farfield
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "worked_example_au_brick_mueller.json")))
    rows = np.array(g["rows"])
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8, polarizability="GKDLDR")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    nh, th, ph = w.lab_directions(rows[:, 0], rows[:, 1])
    f, _ = dda.far_field(tgt, opts, P, nh, th, ph)
    M = dda.mueller(f[0], f[1], d["e0"][0], d["e0"][1], rows[:, 1])
    s11 = rows[:, 3]
    assert np.all(np.abs(M[:, 0, 0] - s11) <= 2e-4 * s11)
    assert np.all(np.abs(M[:, 0, 1] - rows[:, 4]) <= 2e-4 * s11)
    assert np.all(np.abs(M[:, 1, 0] - rows[:, 5]) <= 1e-3 * s11)
    assert np.all(np.abs(M[:, 1, 1] - rows[:, 6]) <= 1e-3 * s11)
    assert np.all(np.abs(M[:, 2, 0]) <= 1e-4) and np.all(np.abs(M[:, 3, 0]) <= 1e-4)
    ref = farfield.mueller(farfield.amplitude_matrix(f.transpose(1, 2, 0), d["e0"][0], d["e0"][1], rows[:, 1]))
    for i in range(4):
        for j in range(4):
            assert np.abs(M[:, i, j] - ref[f"S{i + 1}{j + 1}"]).max() <= 1e-12 * s11.max(), (i, j)
    nb, tb, pb = w.lab_directions([180.0], [0.0])
    _, dcs = dda.far_field(tgt, opts, P, nb, tb, pb)
    for q in range(2):
        qbk = dcs[q, 0] / (np.pi * res[q]["aeff_d"] ** 2)
        assert abs(qbk - g["qbk"]) <= 2e-4 * g["qbk"]


def test_scattering_averages_on_gpu(dda):
    """dda_scattering_averages on the gold brick: against the oracle's
    quadrature on the same P (1e-10), Q_sca against Q_ext - Q_abs, and g,
    <cos^2> within 0.3% of the guide's printed (962-direction) values."""
    import json
    import os
    from oracle import dense as odense, farfield
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "worked_example_au_brick.json")))
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8, polarizability="GKDLDR")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    av = dda.scattering_averages(tgt, opts, d["khat"], d["e0"], P, 32, 48)
    a = odense.aeff_over_d(len(d["ijk"]))
    Pn = P.cpu().numpy()
    for q in range(2):
        qs, gg, c2 = farfield.angular_averages(d["ijk"], Pn[q], res[q]["kd"], d["khat"][q], a, 32, 48)
        assert abs(av[q]["qsca"] - qs) <= 1e-10 * qs
        assert abs(av[q]["g"] - gg) <= 1e-10 and abs(av[q]["cos2"] - c2) <= 1e-10
        assert abs(av[q]["qsca"] - res[q]["qsca"]) <= 1e-6 * res[q]["qsca"]
        assert abs(av[q]["g"] - g["g1"]) <= 3e-3 * g["g1"]
        assert abs(av[q]["cos2"] - g["cos2"]) <= 3e-3 * g["cos2"]


# ------------------------------------------------------------------ captured iteration graphs

@pytest.mark.parametrize("solver", ["bicgstab", "qmr", "bicgstab2"])
def test_graph_replays_match_eager_launches(dda, solver):
    """Batched solves replay a captured HIP graph of each chunk of Krylov
    iterations (slot 0 on the context's null stream replays on a side
    stream, the other slots capture on their own streams); every replay
    equals, bitwise, the same solves launched kernel by kernel.  Single
    solves on the null stream and on an explicit stream agree bitwise too."""
    d = w.workload("brick48")
    tgt = dda.Target(d["ijk"], d["m"])
    kh, e0 = d["khat"][:4], d["e0"][:4]
    eager = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver=solver, graphs=False)
    graph = dda.Options.for_size_parameter(d["x"], tol=1e-5, solver=solver)
    P0, r0 = dda.solve(tgt, eager, kh, e0)
    for _ in range(3):
        P1, r1 = dda.solve(tgt, graph, kh, e0)
        assert torch.equal(P1, P0) and r1 == r0
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        t2 = dda.Target(d["ijk"], d["m"])
        P2, r2 = dda.solve(t2, graph, kh, e0)
    torch.cuda.synchronize()
    assert torch.equal(P2, P0) and r2 == r0
    sph = [w.sphere_integer(r) for r in (6.5, 9.0)]
    tgts = [tgt] + [dda.Target(x, 1.33 + 0.01j) for x in sph]
    ko, eo = w.along_x_yz()
    o_e = [eager] + [dda.Options.for_size_parameter(4.0, tol=1e-5, solver=solver, graphs=False)] * 2
    o_g = [graph] + [dda.Options.for_size_parameter(4.0, tol=1e-5, solver=solver)] * 2
    rt = [0, 0, 1, 1, 2, 2]
    khs = np.vstack([kh[:2], ko, ko])
    e0s = np.vstack([e0[:2], eo, eo])
    Pe, re_ = dda.solve_batched(tgts, o_e, rt, khs, e0s)
    for _ in range(3):
        Pg, rg = dda.solve_batched(tgts, o_g, rt, khs, e0s)
        assert re_ == rg and all(torch.equal(a, b) for a, b in zip(Pe, Pg))
    # kernel timing on: sampled chunks run as direct launches, the rest
    # replay graphs; results stay bitwise equal and the launch totals match
    # the kernel-by-kernel run exactly
    counts = []
    try:
        for opts in (o_e, o_g):
            dda.set_timing(True)
            dda.set_timing_sample(3)
            Pt, rt_ = dda.solve_batched(tgts, opts, rt, khs, e0s)
            torch.cuda.synchronize()
            counts.append(dda.get_timing())
            assert rt_ == re_ and all(torch.equal(a, b) for a, b in zip(Pe, Pt))
    finally:
        dda.set_timing(False)
        dda.set_timing_sample(1)
    for name in counts[0]:
        assert counts[1][name][2] == counts[0][name][2], name
        assert counts[1][name][1] <= counts[0][name][1], name
    assert sum(v[2] for v in counts[1].values()) > 0


# ---------------------------------------------------------------- near field

NF_CASES = {
    # target, refractive index, extension fractions (ragged on purpose)
    "sphere389": (lambda: w.sphere_integer(4.5), 1.33 + 0.01j, (0.5, 0.25, 0.0, 1.0, 0.4, 0.4)),
    "ragged_9x7x13": (_ragged, 1.5 + 0.2j, (0.3, 0.3, 0.6, 0.0, 0.1, 0.2)),
    "single_site": (lambda: np.array([[3, -2, 5]], dtype=np.int32), 1.7 + 0.3j, (2.0, 3.0, 1.0, 4.0, 0.0, 2.0)),
}


@pytest.mark.parametrize("name", sorted(NF_CASES))
@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
def test_nearfield_matches_oracle_everywhere(dda, name, precision):
    """dda_nearfield on every point of a ragged extended volume against the
    oracle's direct sums on the same P (2 right-hand sides, one oblique and
    elliptical): E_sca within 1e-12 of max|E_sca| in FP64 (2e-5 in the FP32
    product), E_inc within 1e-13; the volume's origin and extents as the
    oracle's."""
    from oracle import nearfield
    mk, mval, ext = NF_CASES[name]
    ijk = mk()
    n = len(ijk)
    tgt = dda.Target(ijk, np.full(n, mval))
    kh = np.array([[1, 0, 0], [0.36, 0.48, 0.8]])
    e0 = np.array([[0, 1, 0], np.array([0.8, -0.6, 0]) + 1j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    opts = dda.Options.for_size_parameter(1.3, precision=precision)
    P = w.random_vectors(9, (2, n, 3))
    org, dims, Ei, Es = dda.nearfield(tgt, opts, ext, kh, e0, _cuda(P))
    torch.cuda.synchronize()
    k = dense.kd_from_size_parameter(1.3, n)
    o_ref, d_ref = nearfield.extended_box(ijk, ext)
    assert list(org) == list(o_ref) and list(dims) == list(d_ref)
    tol = 1e-12 if precision == "fp64" else 2e-5
    for q in range(2):
        _, _, ri, rs = nearfield.nearfield(ijk, P[q], k, kh[q], e0[q], ext)
        gi, gs = Ei[q].cpu().numpy(), Es[q].cpu().numpy()
        assert np.abs(gs - rs).max() <= tol * np.abs(rs).max(), q
        assert np.abs(gi - ri).max() <= 1e-13, q
    # the incident field is optional; E_sca is the same without it
    _, _, none, Es2 = dda.nearfield(tgt, opts, ext, kh, e0, _cuda(P), incident=False)
    assert none is None and torch.equal(Es2, Es)


# points of the volume below and above a 4-site box on x, y, z
NF_WINDOWS = {
    "plane_48": ((0, 0), (20, 0), (0, 20)),
    "strided_96": ((10, 2), (30, 14), (5, 39)),
    "strided_160": ((2, 8), (60, 1), (1, 60)),
    "runtime": ((17, 0), (0, 18), (14, 3)),
    "short": ((3, 30), (0, 6), (5, 1)),
    "y256": ((0, 61), (60, 64), (0, 0)),
    "z256": ((0, 5), (2, 12), (64, 60)),
}


@pytest.mark.parametrize("name", sorted(NF_WINDOWS))
@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
def test_nearfield_input_window(dda, name, precision):
    """The product of a volume whose sources fill only a window of it, at the
    window's corners and through every variant of the passes: all variants
    bitwise equal, and every point within the tolerances of
    test_nearfield_matches_oracle_everywhere of the oracle's direct sums."""
    from oracle import nearfield
    ends = NF_WINDOWS[name]
    ext = tuple(b / 4 for axis in ends for b in axis)
    ijk = np.array([[0, 0, 0], [3, 3, 3], [0, 3, 1], [3, 0, 2], [1, 2, 0], [2, 1, 3]], dtype=np.int32)
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    kh, e0 = np.array([[0.36, 0.48, 0.8]] * 2), np.array([[0.8, -0.6, 0]] * 2, dtype=complex)
    P = w.random_vectors(35, (2, len(ijk), 3))
    ref = None
    for variant in range(29):
        opts = dda.Options.for_size_parameter(1.3, precision=precision, kernel_variant=variant)
        org, dims, Ei, Es = dda.nearfield(tgt, opts, ext, kh, e0, _cuda(P))
        if ref is None:
            ref = Es.clone()
        assert torch.equal(Es, ref), variant
    assert list(dims) == [4 + b + a for b, a in ends]
    k = dense.kd_from_size_parameter(1.3, len(ijk))
    tol = 1e-12 if precision == "fp64" else 2e-5
    for q in range(2):
        _, _, ri, rs = nearfield.nearfield(ijk, P[q], k, kh[q], e0[q], ext)
        assert np.abs(Es[q].cpu().numpy() - rs).max() <= tol * np.abs(rs).max(), q
        assert np.abs(Ei[q].cpu().numpy() - ri).max() <= 1e-13, q


def test_nearfield_solution_satisfies_the_dda_equations(dda):
    """On a GPU solution the total field at the target's sites is the local
    field: |E_inc + E_sca - P / alpha| / |E_inc| over the sites equals the
    solve's true relative residual (to rounding), and the cached volume is
    rebuilt when another extension is asked for."""
    d = w.workload("twomat6")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-9)
    P, res = dda.solve(tgt, opts, d["khat"][:1], d["e0"][:1])
    k = res[0]["kd"]
    ainv = dense.site_alpha_inverse(np.asarray(d["m"]), k, d["khat"][0], d["e0"][0], dense.LATTDR)
    for ext in ((0.5,) * 6, (0.0, 1.0, 0.5, 0.0, 0.0, 0.34)):
        org, dims, Ei, Es = dda.nearfield(tgt, opts, ext, d["khat"][:1], d["e0"][:1], P)
        Et = (Ei + Es)[0].cpu().numpy()
        idx = d["ijk"] - np.asarray(org)
        Es_sites = Et[idx[:, 2], idx[:, 1], idx[:, 0]]
        Einc = Ei[0].cpu().numpy()[idx[:, 2], idx[:, 1], idx[:, 0]]
        r = np.linalg.norm(Es_sites - ainv * P[0].cpu().numpy()) / np.linalg.norm(Einc)
        assert r <= 1e-9 and abs(r - res[0]["rel_residual"]) <= 1e-11


def test_field_line_matches_oracle_trilinear(dda):
    """dda_field_line against the oracle's trilinear interpolation of the
    same lattice field: a line with both ends on faces of the box, a single
    point, and a box one point thick on an axis; end points outside the box
    are rejected."""
    from oracle import nearfield
    rng = np.random.default_rng(12)
    for dims, org, a, b, npt in (((7, 5, 6), (-3, 2, 0), (-3.0, 2.5, 0.2), (3.0, 6.0, 5.0), 41),
                                 ((7, 5, 6), (-3, 2, 0), (0.3, 3.7, 4.4), (0.3, 3.7, 4.4), 1),
                                 ((9, 1, 4), (0, 5, -2), (0.5, 5.0, -2.0), (8.0, 5.0, 1.0), 17)):
        nx, ny, nz = dims
        E = rng.standard_normal((2, nz, ny, nx, 3)) + 1j * rng.standard_normal((2, nz, ny, nx, 3))
        out = dda.field_line(_cuda(E), org, a, b, npt).cpu().numpy()
        for q in range(2):
            def field_at(pts, q=q):
                p = np.asarray(pts) - np.asarray(org)
                p = np.minimum(p, np.asarray(dims) - 1)     # corners beyond a one-point axis weigh 0
                return E[q][p[:, 2], p[:, 1], p[:, 0]]
            ref = nearfield.trilinear(field_at, nearfield.line_points(a, b, npt))
            assert np.abs(out[q] - ref).max() <= 1e-13 * np.abs(E).max()
    with pytest.raises(dda.DDAError):
        dda.field_line(_cuda(E), org, (0.0, 5.0, -2.5), b, 5)


def test_nearfield_error_paths(dda):
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options()
    P = _cuda(w.random_vectors(3, (1, len(d["ijk"]), 3)))
    kh, e0 = w.along_x_yz()
    for bad in ((-0.1, 0, 0, 0, 0, 0), (0, 0, 0, 0, 0, float("nan")), (20.0, 20.0, 0, 0, 0, 0)):
        with pytest.raises(dda.DDAError):
            dda.nearfield(tgt, opts, bad, kh[:1], e0[:1], P)


def test_nearfield_gold_sphere_printed_track_on_gpu(dda):
    """The guide's near-field example end to end on the GPU: GKDLDR solve of
    the N = 59728 gold pseudosphere (tol 1e-5), E on the 96^3 extended
    volume, then the readnf track along x_TF through the centre (52 points,
    trilinear) against the printed values (3e-4, as the oracle's pin), and
    sampled lattice points against the oracle's direct sums on the GPU's P
    (1e-10 of max|E_sca|)."""
    import json
    import os
    from oracle import nearfield
    g = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "nearfield_au_sphere_track.json")))
    d = w.workload("au_sphere_nf")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-5, polarizability="GKDLDR", solver="bicgstab2")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    org, dims, Ei, Es = dda.nearfield(tgt, opts, d["nf_ext"], d["khat"], d["e0"], P)
    assert list(dims) == g["header"]["dims"]
    k = res[0]["kd"]
    dl = g["header"]["aeff_um"] / res[0]["aeff_d"]
    c = 23.5
    a = np.array(g["line_um"]["a"]) / dl + c
    b = np.array(g["line_um"]["b"]) / dl + c
    rows = np.array(g["rows"])
    printed = rows[:, 3::2] + 1j * rows[:, 4::2]
    line = dda.field_line(Ei + Es, org, a, b, len(rows)).cpu().numpy()
    assert np.abs(line[0] * np.exp(-1j * k * c) - printed).max() < 3e-4
    # sampled lattice points (inside, on the surface, outside, the corners)
    rng = np.random.default_rng(21)
    pts = np.vstack([rng.integers(0, dims, size=(12, 3)), [[0, 0, 0], list(np.asarray(dims) - 1), [47, 47, 47]]])
    Pn = P.cpu().numpy()
    Esn = Es.cpu().numpy()
    for q in range(2):
        ref = nearfield.scattered_field(d["ijk"], Pn[q], k, pts + np.asarray(org))
        got = Esn[q][pts[:, 2], pts[:, 1], pts[:, 0]]
        assert np.abs(got - ref).max() <= 1e-10 * np.abs(Esn[q]).max(), q


# ---------------------------------------------------------------- edge cases

def test_degenerate_inputs_are_rejected(dda):
    """An empty target, a vacuum site, no right-hand sides, and a box whose
    padded FFT extent would exceed the supported 512 are errors, not launches."""
    with pytest.raises(dda.DDAError):
        dda.Target(np.zeros((0, 3), dtype=np.int32), 1.5)
    with pytest.raises(dda.DDAError):
        dda.Target(np.array([[0, 0, 0], [1, 0, 0]]), np.array([1.5, 1.0]))
    for axis in range(3):                    # 257 sites: padded extent 540
        ijk = np.zeros((257, 3), dtype=np.int32)
        ijk[:, axis] = np.arange(257)
        with pytest.raises(dda.DDAError, match="above the supported 512"):
            dda.Target(ijk, 1.5)
    tgt = dda.Target(w.sphere_integer(2.0), 1.5 + 0.1j)
    with pytest.raises(dda.DDAError):
        dda.solve(tgt, dda.Options.for_size_parameter(1.0), np.zeros((0, 3)), np.zeros((0, 3), complex))


@pytest.mark.parametrize("n,grid", [(135, 270), (160, 384), (256, 512)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_largest_padded_extents_match_dense(dda, axis, n, grid):
    """A line of n sites on one axis: 135 sites pad to 270 (the largest
    runtime-planned extent the padding rule produces), 160 to 384 and 256 to
    512 (the largest compile-time lengths; every extent up to 256 pads to at
    most 512).  On each axis, in FP64 and in FP32, the product equals the
    dense one (1e-12 and 2e-5 of max|y|)."""
    ijk = np.zeros((n, 3), dtype=np.int32)
    ijk[:, axis] = np.arange(n) - 40
    tgt = dda.Target(ijk, 1.4 + 0.2j)
    assert tgt.grid[axis] == grid == _library_extent(n)
    kh, e0 = [[0.0, 0.6, 0.8]], [[1.0, 0.0, 0.0]]
    xv = w.random_vectors(13, (1, n, 3))
    A = _dense_A(ijk, np.full(n, 1.4 + 0.2j), 3.0, kh[0], e0[0], "LATTDR")
    ref = (A @ xv[0].reshape(-1)).reshape(-1, 3)
    for prec, tol in (("fp64", 1e-12), ("fp32_matvec", 2e-5)):
        opts = dda.Options.for_size_parameter(3.0, precision=prec)
        y = dda.apply(tgt, opts, kh, e0, _cuda(xv)).cpu().numpy()
        assert np.abs(y[0] - ref).max() <= tol * np.abs(ref).max(), prec


@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
def test_pass3_variants_at_384_and_512_are_bitwise_equal(dda, precision):
    """Lines of 160 and 256 sites along z (padded 384 and 512 on z): every
    tiling variant of the pass-3 kernel (and of the y passes, on lines along y)
    gives bitwise the default's product."""
    for n in (160, 256):
        for axis in (1, 2):
            ijk = np.zeros((n, 3), dtype=np.int32)
            ijk[:, axis] = np.arange(n)
            ijk[: n // 2, 0] = 1            # two columns, so x tiles hold more than one
            tgt = dda.Target(ijk, 1.5 + 0.1j)
            kh, e0 = w.along_x_yz()
            xv = _cuda(w.random_vectors(21 + n, (2, n, 3)))
            base = dda.apply(tgt, dda.Options.for_size_parameter(2.0, precision=precision, autotune=False), kh,
                             e0, xv)
            for v in range(2, 29):
                o = dda.Options.for_size_parameter(2.0, precision=precision, kernel_variant=v)
                y = dda.apply(tgt, o, kh, e0, xv)
                assert torch.equal(y, base), (n, axis, v)


def test_box200_sphere_on_the_512_grid(dda):
    """A sphere of radius 100 (4,187,857 sites, box 201^3, FFT grid 512^3):
    sampled rows of A x in FP64 and FP32 against the oracle's direct sums
    (1e-12, 2e-5 of max|y|); the FP32-matvec solve at x = 8 converges, its
    sampled rows of A P equal E_inc to 1e-3 of max|E| by the oracle's sums,
    and its efficiencies lie within the DDA error of Mie theory."""
    ijk = w.sphere_integer(100.0)
    n = len(ijk)
    m = 1.33 + 0.01j
    x = 8.0
    tgt = dda.Target(ijk, m)
    assert tgt.grid == (512, 512, 512)
    k = dense.kd_from_size_parameter(x, n)
    kh, e0 = w.along_x_yz()
    ainv = dense.site_alpha_inverse(np.full(n, m), k, kh[0], e0[0])
    xv = w.random_vectors(9, (1, n, 3))
    rows = np.random.default_rng(2).choice(n, 4, replace=False)
    ref = dense.apply_rows(ijk, ainv, k, xv[0], rows)
    for prec, tol in (("fp64", 1e-12), ("fp32_matvec", 2e-5)):
        o = dda.Options.for_size_parameter(x, precision=prec)
        y = dda.apply(tgt, o, kh[:1], e0[:1], _cuda(xv)).cpu().numpy()[0]
        assert np.abs(y[rows] - ref).max() <= tol * np.abs(ref).max(), prec
    del xv, y
    o32 = dda.Options.for_size_parameter(x, tol=1e-5, precision="fp32_matvec")
    P, res = dda.solve(tgt, o32, kh, e0)
    q_mie = mie.efficiencies(m, x)
    for q, r in enumerate(res):
        assert r["status"] == 0 and r["rel_residual"] < 1e-5, r
        ainv_q = dense.site_alpha_inverse(np.full(n, m), k, kh[q], e0[q])
        Pq = P[q].cpu().numpy()
        E = dense.incident_field(ijk[rows], k, kh[q], e0[q])
        AP = dense.apply_rows(ijk, ainv_q, k, Pq, rows)
        assert np.abs(AP - E).max() <= 1e-3 * np.abs(E).max(), q
        assert abs(r["qext"] / q_mie["qext"] - 1) < 0.05
        assert abs(r["qsca"] / q_mie["qsca"] - 1) < 0.05
        assert abs(r["qabs"] / q_mie["qabs"] - 1) < 0.10


# ------------------------------------------------------------------ runtime-planned FFT lengths

def _three_lines(n):
    """Three perpendicular lines of n[0], n[1], n[2] sites from one corner:
    a sparse target whose padded grid has the extents of n on every axis."""
    pts = [[i, 0, 0] for i in range(n[0])] + [[0, j, 0] for j in range(n[1])] + [[0, 0, k] for k in range(n[2])]
    return np.unique(np.array(pts), axis=0).astype(np.int32)


def _library_extent(n):
    """The library's padded extent (include/dda.h): the smallest compile-time
    FFT length >= 2n - 1 when at most 1.4 times the 2,3,5-smooth extent, else
    the smooth extent."""
    m = fftsolve.padded_extent(n)
    for L in (32, 48, 64, 80, 96, 128, 160, 192, 256, 384, 512):
        if L >= 2 * n - 1:
            return L if 5 * L <= 7 * m else m
    return m


# box extents whose sites fill a fraction of their compile-time grids (the
# sphere batch's boxes, 13..41 sites, pad to 32..96), and extents that keep
# runtime-planned lengths (10, 18, 20 below 32; 270, 288, 300 above 256)
RT_LINES = [(14, 15, 18), (20, 23, 25), (27, 30, 36), (38, 41, 23), (9, 10, 5), (131, 140, 150)]
@pytest.mark.parametrize("n", RT_LINES, ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32_matvec", 2e-5)])
def test_matvec_runtime_lengths_match_dense(dda, n, precision, tol):
    ijk = _three_lines(n)
    tgt = dda.Target(ijk, np.where(np.arange(len(ijk)) % 2 == 0, 1.33 + 0.01j, 1.6 + 0.2j))
    assert tgt.grid == tuple(_library_extent(v) for v in n)
    m = np.where(np.arange(len(ijk)) % 2 == 0, 1.33 + 0.01j, 1.6 + 0.2j)
    kh = np.array([[1, 0, 0], [0.36, 0.48, 0.8]])
    e0 = np.array([[0, 1, 0], np.array([0.8, -0.6, 0]) + 1j * np.cross([0.36, 0.48, 0.8], [0.8, -0.6, 0])])
    opts = dda.Options.for_size_parameter(2.5, precision=precision)
    xv = w.random_vectors(40 + n[0], (2, len(ijk), 3))
    y = dda.apply(tgt, opts, kh, e0, _cuda(xv)).cpu().numpy()
    for q in range(2):
        ref = (_dense_A(ijk, m, 2.5, kh[q], e0[q], "LATTDR") @ xv[q].reshape(-1)).reshape(-1, 3)
        assert np.abs(y[q] - ref).max() <= tol * np.abs(ref).max(), (n, tgt.grid, q)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32_matvec", 2e-5)])
def test_matvec_sphere_batch_grids_match_oracle_fft(dda, precision, tol):
    """One sphere of the ragged batch per distinct padded grid (every grid
    the 32 spheres use), A x at full size against the oracle's FFT operator
    (on its own padded grid), element by element."""
    radii = w.sphere_radii(0)
    seen = {}
    for r in radii:
        ijk = w.sphere_integer(r)
        g = _library_extent(int(ijk[:, 0].max() - ijk[:, 0].min() + 1))
        seen.setdefault(g, r)
    assert sorted(seen) == [32, 48, 64, 80]
    kh, e0 = w.along_x_yz()
    for g, r in sorted(seen.items()):
        ijk = w.sphere_integer(r)
        n = len(ijk)
        tgt = dda.Target(ijk, 1.33 + 0.01j)
        assert tgt.grid == (g, g, g)
        opts = dda.Options.for_size_parameter(4.0, precision=precision)
        xv = w.random_vectors(50 + g, (1, n, 3))
        y = dda.apply(tgt, opts, kh[1:], e0[1:], _cuda(xv)).cpu().numpy()[0]
        k = dense.kd_from_size_parameter(4.0, n)
        ref = fftsolve.FFTOperator(ijk, dense.site_alpha_inverse(np.full(n, 1.33 + 0.01j), k, kh[1], e0[1]),
                                   k).apply(xv[0])
        assert np.abs(y - ref).max() <= tol * np.abs(ref).max(), (g, r)


# ------------------------------------------------------------------ non-finite inputs

def test_nonfinite_right_hand_side_or_start_is_reported(dda):
    """A NaN in b (dda_solve_rhs) or in the warm start P0 (dda_solve) ends
    that right-hand side with DDA_E_NONFINITE; the others are unaffected."""
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8)
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    b = P.clone()
    b[1, 7, 2] = complex(np.nan, 0.0)
    x, r = dda.solve_rhs(tgt, opts, d["khat"], d["e0"], b)
    assert r[0]["status"] == 0 and r[1]["status"] == 6
    P0 = P.clone()
    P0[0, 3, 1] = complex(0.0, np.inf)
    _, r = dda.solve(tgt, opts, d["khat"], d["e0"], P0=P0)
    assert r[0]["status"] == 6 and r[1]["status"] == 0


# ------------------------------------------------------------------ far field, grouped directions

def test_scattering_averages_odd_direction_sets_match_oracle(dda):
    """Direction sets of 5 x 3 = 15 per right-hand side, not a multiple of
    the four directions a workgroup takes: the averages run one direction
    per workgroup, and agree with the oracle's quadrature of the same rule on
    the same P (1e-10)."""
    from oracle import dense as odense, farfield
    d = w.workload("au_brick")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-8, polarizability="GKDLDR")
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    av = dda.scattering_averages(tgt, opts, d["khat"], d["e0"], P, 5, 3)
    a = odense.aeff_over_d(len(d["ijk"]))
    Pn = P.cpu().numpy()
    for q in range(2):
        qs, gg, c2 = farfield.angular_averages(d["ijk"], Pn[q], res[q]["kd"], d["khat"][q], a, 5, 3)
        assert abs(av[q]["qsca"] - qs) <= 1e-10 * qs
        assert abs(av[q]["g"] - gg) <= 1e-10 and abs(av[q]["cos2"] - c2) <= 1e-10


def test_far_field_four_directions_per_workgroup_match_oracle(dda):
    """2,051 directions: the far-field launch takes four directions per
    workgroup (partial last group of three) against the oracle's sums."""
    from oracle import farfield
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"], tol=1e-10)
    P, res = dda.solve(tgt, opts, d["khat"], d["e0"])
    nh, th, ph = _random_frames(np.random.default_rng(5), 2051)
    f, dcs = dda.far_field(tgt, opts, P, nh, th, ph)
    Pn = P.cpu().numpy()
    for q in range(2):
        A = farfield.amplitude_vectors(d["ijk"], Pn[q], res[q]["kd"], nh)
        ref = np.stack([np.sum(th * A, axis=1), np.sum(ph * A, axis=1)], axis=1)
        assert np.abs(f[q] - ref).max() <= 1e-12 * np.abs(ref).max()
        rd = (np.abs(ref[:, 0]) ** 2 + np.abs(ref[:, 1]) ** 2) / res[q]["kd"] ** 2
        assert np.abs(dcs[q] - rd).max() <= 1e-12 * rd.max()


def test_far_field_rhs_pairs_along_the_grid_match_oracle(dda):
    """Seven right-hand sides (three pairs, and one with an empty partner)
    over 522 directions: the launch takes the pairs along its grid's y and,
    at 131 x 4 workgroups, four directions per workgroup with a partial last
    group of two.  Every amplitude and cross section of a random P against
    the oracle's direct sum (1e-12)."""
    from oracle import dense as odense, farfield
    d = w.workload("sphere389")
    tgt = dda.Target(d["ijk"], d["m"])
    opts = dda.Options.for_size_parameter(d["x"])
    n = len(d["ijk"])
    Pn = w.random_vectors(77, (7, n, 3))
    nh, th, ph = _random_frames(np.random.default_rng(8), 522)
    f, dcs = dda.far_field(tgt, opts, _cuda(Pn), nh, th, ph)
    kd = odense.kd_from_size_parameter(d["x"], n)
    for q in range(7):
        A = farfield.amplitude_vectors(d["ijk"], Pn[q], kd, nh)
        ref = np.stack([np.sum(th * A, axis=1), np.sum(ph * A, axis=1)], axis=1)
        assert np.abs(f[q] - ref).max() <= 1e-12 * np.abs(ref).max(), q
        rd = (np.abs(ref[:, 0]) ** 2 + np.abs(ref[:, 1]) ** 2) / kd ** 2
        assert np.abs(dcs[q] - rd).max() <= 1e-12 * rd.max(), q


# ------------------------------------------------------------------ breakdown and restart

@pytest.mark.parametrize("solver", ["bicgstab", "bicgstab2"])
def test_first_step_breakdown_restarts_and_converges(dda, solver):
    """A right-hand side with b^H A b = 0 (a gain material puts 0 in A's
    numerical range; the oracle's dense A gives b) breaks BiCGSTAB and
    BiCGstab(2) down in their first step; the one restart, with the conjugate
    shadow residual, converges to the LU solution."""
    import breakdown_rhs as br
    ijk = w.brick(2, 2, 2)
    m = np.full(len(ijk), br.GAIN_M)
    kh, e0 = np.array([[1.0, 0, 0]]), np.array([[0, 1.0, 0]], dtype=complex)
    A = _dense_A(ijk, m, 1.0, kh[0], e0[0], "LATTDR")
    b = br.hermitian_zero(A).reshape(-1, 3)
    tgt = dda.Target(ijk, m)
    x, r = dda.solve_rhs(tgt, dda.Options.for_size_parameter(1.0, tol=1e-10, solver=solver), kh, e0,
                         _cuda(b[None]))
    assert r[0]["restarts"] == 1 and r[0]["status"] == 0, r[0]
    ref = np.linalg.solve(A, b.reshape(-1)).reshape(-1, 3)
    assert np.abs(x.cpu().numpy()[0] - ref).max() <= 1e-8 * np.abs(ref).max()


def test_qmr_breakdown_is_reported(dda):
    """b^T A b = 0 (exact up to rounding, from the oracle's dense A) breaks
    QMR down in its first step: the solve ends with DDA_E_BREAKDOWN and no
    restart; the same b solves normally with BiCGSTAB (b^H A b != 0)."""
    import breakdown_rhs as br
    ijk = w.brick(3, 3, 3)
    m = np.full(len(ijk), 1.5 + 0.1j)
    kh, e0 = np.array([[1.0, 0, 0]]), np.array([[0, 1.0, 0]], dtype=complex)
    A = _dense_A(ijk, m, 1.0, kh[0], e0[0], "LATTDR")
    b = br.bilinear_zero(A).reshape(-1, 3)
    tgt = dda.Target(ijk, m)
    _, r = dda.solve_rhs(tgt, dda.Options.for_size_parameter(1.0, tol=1e-10, solver="qmr"), kh, e0, _cuda(b[None]))
    assert r[0]["status"] == 5 and r[0]["restarts"] == 0, r[0]
    x, r = dda.solve_rhs(tgt, dda.Options.for_size_parameter(1.0, tol=1e-10), kh, e0, _cuda(b[None]))
    assert r[0]["status"] == 0 and r[0]["restarts"] == 0
    ref = np.linalg.solve(A, b.reshape(-1)).reshape(-1, 3)
    assert np.abs(x.cpu().numpy()[0] - ref).max() <= 1e-8 * np.abs(ref).max()


@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
@pytest.mark.parametrize("ny", [11, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 64])
def test_plane_kernel_equals_the_three_passes(dda, precision, ny):
    """Every pair of compiled (y, z) lengths at the smallest and largest box
    extents that pad to it (and x extents with a runtime-planned and a
    compile-time length): the product of the fused plane kernel is bitwise
    that of the three separate passes, which a named variant selects."""
    for nz in (11, 16, 17, 24, 25, 32, 33, 40, 41, 48, 49, 64):
        nx = 3 if (ny + nz) % 2 else 19
        rng = np.random.default_rng(1000 * ny + nz)
        keep = rng.random((nx, ny, nz)) < 0.1
        keep[0, 0, 0] = keep[-1, -1, -1] = True
        ijk = np.argwhere(keep).astype(np.int32)
        tgt = dda.Target(ijk, 1.4 + 0.1j)
        assert tgt.box == (nx, ny, nz)
        kh, e0 = w.along_x_yz()
        xv = _cuda(w.random_vectors(31, (2, len(ijk), 3)))
        y = dda.apply(tgt, dda.Options.for_size_parameter(2.0, precision=precision), kh, e0, xv)
        ref = dda.apply(tgt, dda.Options.for_size_parameter(2.0, precision=precision, kernel_variant=4), kh, e0, xv)
        assert torch.equal(y, ref), (nx, ny, nz)


@pytest.mark.parametrize("box", [(1, 1, 2), (1, 7, 13), (13, 1, 9), (2, 3, 1), (10, 5, 33), (11, 24, 3), (49, 2, 17),
                                 (3, 65, 4)])
def test_tensor_octant_over_odd_and_padded_extents(dda, box):
    """The tensor FFT at extents of one site, odd (M = 2n - 1), even and
    over-padded grid extents on each axis: the product of a scattered handful
    of sites against the dense matrix (1e-12)."""
    rng = np.random.default_rng(sum(box))
    keep = rng.random(box) < min(1.0, 60.0 / np.prod(box))
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = np.argwhere(keep).astype(np.int32)
    n = len(ijk)
    m = np.full(n, 1.5 + 0.2j)
    tgt = dda.Target(ijk, m)
    assert tgt.box == box
    kh, e0 = w.along_x_yz()
    xv = w.random_vectors(8, (2, n, 3))
    y = dda.apply(tgt, dda.Options.for_size_parameter(0.8), kh, e0, _cuda(xv)).cpu().numpy()
    for q in range(2):
        ref = (_dense_A(ijk, m, 0.8, kh[q], e0[q], "LATTDR") @ xv[q].reshape(-1)).reshape(n, 3)
        assert np.abs(y[q] - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("box,n_dir", [((21, 21, 21), 1), ((8, 48, 33), 15), ((33, 17, 16), 17), ((256, 6, 6), 70),
                                       ((255, 6, 7), 64), ((16, 48, 12), 130)])
def test_far_field_by_lines_matches_the_oracle(dda, box, n_dir):
    """Dense boxes (odd and even lines, partial tiles
    of lines, planes and directions): the amplitudes by contractions along x
    against the oracle's direct sum (1e-12)."""
    from oracle import farfield
    rng = np.random.default_rng(n_dir)
    keep = rng.random(box) < 0.93
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = (np.argwhere(keep) - [3, -2, 40]).astype(np.int32)
    n = len(ijk)
    assert n >= 8192
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    P = w.random_vectors(12, (3, n, 3))
    nh, th, ph = w.lab_directions(rng.uniform(0, 180, n_dir), rng.uniform(0, 360, n_dir))
    opts = dda.Options.for_size_parameter(4.0)
    f, dcs = dda.far_field(tgt, opts, _cuda(P), nh, th, ph)
    k = dense.kd_from_size_parameter(4.0, n)
    for q in range(3):
        A = farfield.amplitude_vectors(ijk, P[q], k, nh)
        ref = np.stack([np.sum(th * A, axis=1), np.sum(ph * A, axis=1)], axis=1)
        assert np.abs(f[q] - ref).max() <= 1e-12 * np.abs(P[q]).sum() * k ** 3 / np.sqrt(n)
        assert np.allclose(dcs[q], (np.abs(f[q]) ** 2).sum(axis=1) / k ** 2, rtol=1e-13, atol=0)


def test_far_field_by_lines_in_groups_of_right_hand_sides(dda):
    """More right-hand sides than one launch's operands hold (512 MiB): each
    one's amplitudes equal those of a call of its own, bitwise."""
    ijk = w.brick(256, 6, 6)
    n, q = len(ijk), 470
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    P = torch.randn((q, n, 3), generator=g, dtype=torch.complex128, device="cuda")
    nh, th, ph = w.lab_directions([10.0, 75.0], [0.0, 40.0])
    opts = dda.Options.for_size_parameter(4.0)
    f, _ = dda.far_field(tgt, opts, P, nh, th, ph)
    for i in (0, 1, 300, 433, q - 1):
        fi, _ = dda.far_field(tgt, opts, P[i:i + 1], nh, th, ph)
        assert np.array_equal(f[i], fi[0])


@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
@pytest.mark.parametrize("short", [1, 3, 7, 9, 10])
def test_short_plane_kernel_equals_the_three_passes(dda, precision, short):
    """Grids with a y or z extent of at most 20 (runtime-planned), the other
    short too (the short-length plane kernel) or compile-time: the product is
    bitwise that of the three separate passes, which a named variant selects."""
    for other in (1, 2, 8, 10, 11, 16, 24, 32, 40, 48, 50):
        for ny, nz in ((short, other), (other, short)):
            rng = np.random.default_rng(100 * ny + nz)
            keep = rng.random((5, ny, nz)) < 0.3
            keep[0, 0, 0] = keep[-1, -1, -1] = True
            ijk = np.argwhere(keep).astype(np.int32)
            tgt = dda.Target(ijk, 1.4 + 0.1j)
            kh, e0 = w.along_x_yz()
            xv = _cuda(w.random_vectors(32, (2, len(ijk), 3)))
            y = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision), kh, e0, xv)
            ref = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision, kernel_variant=1), kh, e0,
                            xv)
            assert torch.equal(y, ref), (ny, nz)


@pytest.mark.parametrize("nx", [1, 2, 3, 5, 8, 13, 16, 24, 25, 32, 33, 48, 50, 64, 65])
def test_plane_kernel_order_of_workgroups(dda, nx):
    """Every plane of every right-hand side is done once, whatever order the
    x extent (a whole number of mirrored runs per XCD, a contiguous part, or
    neither) and the count of right-hand sides give: bitwise the three passes."""
    rng = np.random.default_rng(nx)
    keep = rng.random((nx, 12, 16)) < 0.1
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = np.argwhere(keep).astype(np.int32)
    tgt = dda.Target(ijk, 1.4 + 0.1j)
    for q in (1, 3):
        kh, e0 = np.tile([1.0, 0, 0], (q, 1)), np.tile(np.array([0, 1, 0], complex), (q, 1))
        xv = _cuda(w.random_vectors(34, (q, len(ijk), 3)))
        for precision in ("fp64", "fp32_matvec"):
            y = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision), kh, e0, xv)
            ref = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision, kernel_variant=4), kh, e0,
                            xv)
            assert torch.equal(y, ref), (q, precision)


@pytest.mark.parametrize("radius", [4.5, 9.5])
@pytest.mark.parametrize("materials", [1, 3])
def test_incidences_as_arguments_equal_copied_ones(dda, materials, radius):
    """Up to eight incidences travel as kernel arguments, more are copied to
    the device: a nine-right-hand-side product and solve, every incidence its
    own, are bitwise the eight and the one they consist of (runtime-planned and
    compile-time x lengths)."""
    ijk = w.sphere_integer(radius)
    n = len(ijk)
    m = np.array([1.33 + 0.01j, 1.5 + 0.2j, 1.1 + 0.3j])[np.arange(n) % materials]
    tgt = dda.Target(ijk, m)
    rng = np.random.default_rng(36)
    kh = rng.normal(size=(9, 3))
    kh /= np.linalg.norm(kh, axis=1)[:, None]
    e0 = np.cross(kh, rng.normal(size=(9, 3))) + 1j * np.cross(kh, rng.normal(size=(9, 3)))
    opts = dda.Options.for_size_parameter(1.0)
    xv = _cuda(w.random_vectors(36, (9, n, 3)))
    y = dda.apply(tgt, opts, kh, e0, xv)
    P, res = dda.solve(tgt, opts, kh, e0)
    for a, b in ((0, 8), (8, 9)):
        assert torch.equal(dda.apply(tgt, opts, kh[a:b], e0[a:b], xv[a:b].contiguous()), y[a:b])
        Ps, rs = dda.solve(tgt, opts, kh[a:b], e0[a:b])
        assert torch.equal(Ps, P[a:b])
        assert [r["qext"] for r in rs] == [r["qext"] for r in res[a:b]]


def test_apply_with_overlapping_vectors(dda):
    """x and y of a product that overlap in part (one buffer, y a right-hand
    side further on): the same result as with separate buffers, the caller's
    order being taken through sorted copies then."""
    import ctypes
    from paper_1202_3424_amd import _abi, api
    ijk = w.sphere_integer(4.5)
    n = len(ijk)
    tgt = dda.Target(ijk, 1.4 + 0.1j)
    kh, e0 = w.along_x_yz()
    opts = dda.Options.for_size_parameter(1.0)
    xv = _cuda(w.random_vectors(33, (2, n, 3)))
    ref = dda.apply(tgt, opts, kh, e0, xv)
    buf = torch.zeros((3, n, 3), dtype=torch.complex128, device="cuda")
    buf[:2] = xv
    o, inc = opts.c(), api._incidences(kh, e0)
    st = _abi.load().dda_apply(tgt.ctx, tgt.handle, ctypes.byref(o), 2, inc, buf[0].data_ptr(), buf[1].data_ptr())
    assert st == 0
    torch.cuda.synchronize()
    assert torch.equal(buf[1:], ref)


# ------------------------------------------------------------------ several materials, many right-hand sides

def _three_materials(n):
    return np.array([1.33 + 0.01j, 1.6 + 0.2j, 2.0 + 0.5j])[np.arange(n) * 7 % 5 % 3]


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32_matvec", 2e-5)])
@pytest.mark.parametrize("box", [(12, 3, 4), (40, 2, 3), (3, 9, 5)])
def test_products_of_many_right_hand_sides_read_each_sites_material(dda, box, precision, tol):
    """A launch of more than 16 right-hand sides gathers its operands after
    the inverse x transform: with three materials, 24 right-hand sides equal
    the dense matrix's products (and, bitwise, launches of 8 and 16), at
    compile-time (32, 80) and runtime-planned (6) x lengths."""
    ijk = w.brick(*box)
    n = len(ijk)
    m = _three_materials(n)
    tgt = dda.Target(ijk, m)
    kh, e0 = w.incidences_for_orientations(61, 12)
    opts = dda.Options.for_size_parameter(1.1, precision=precision)
    xv = w.random_vectors(61, (24, n, 3))
    y = dda.apply(tgt, opts, kh, e0, _cuda(xv))
    for a, b in ((0, 8), (8, 24)):
        assert torch.equal(dda.apply(tgt, opts, kh[a:b], e0[a:b], _cuda(xv[a:b])), y[a:b])
    for q in (0, 9, 23):
        ref = (_dense_A(ijk, m, 1.1, kh[q], e0[q], "LATTDR") @ xv[q].reshape(-1)).reshape(n, 3)
        assert np.abs(y[q].cpu().numpy() - ref).max() <= tol * np.abs(ref).max(), q


@pytest.mark.parametrize("solver", ["bicgstab", "qmr", "bicgstab2"])
@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
@pytest.mark.parametrize("scheme", ["LATTDR", "GKDLDR"])
def test_solves_of_many_right_hand_sides_read_each_sites_material(dda, scheme, solver, precision):
    """Twenty right-hand sides on a target of three materials: every P and
    result is bitwise that of solves of ten, P agrees with the dense
    solution (the residual's tolerance over the smallest singular value), and a batch whose
    launches hold twenty right-hand sides of two such targets equals the
    separate solves."""
    ijks = []
    for seed, box in ((63, (12, 11, 13)), (64, (16, 14, 11))):   # both on the 32^3 grid: they share launches
        keep = np.random.default_rng(seed).random(box) < 0.05
        keep[0, 0, 0] = keep[-1, -1, -1] = True
        ijks.append(np.argwhere(keep).astype(np.int32))
    ms = [_three_materials(len(i)) for i in ijks]
    ts = [dda.Target(i, m) for i, m in zip(ijks, ms)]
    opts = dda.Options.for_size_parameter(1.1, tol=1e-9, solver=solver, precision=precision, polarizability=scheme)
    kh, e0 = w.incidences_for_orientations(62, 10)
    P, r = dda.solve(ts[0], opts, kh, e0)
    for a, b in ((0, 10), (10, 20)):
        Ps, rs = dda.solve(ts[0], opts, kh[a:b], e0[a:b])
        assert torch.equal(Ps, P[a:b]) and rs == r[a:b]
    k = dense.kd_from_size_parameter(1.1, len(ijks[0]))
    for q in (0, 13):
        A = _dense_A(ijks[0], ms[0], 1.1, kh[q], e0[q], scheme)
        E = dense.incident_field(ijks[0], k, kh[q], e0[q]).reshape(-1)
        ref = np.linalg.solve(A, E)
        err = np.linalg.norm(P[q].cpu().numpy().reshape(-1) - ref)
        assert r[q]["status"] == 0
        assert err <= 1.001e-9 * np.linalg.norm(E) / np.linalg.svd(A, compute_uv=False)[-1]
    rt = np.arange(20) % 2
    Pb, rb = dda.solve_batched(ts, [opts, opts], rt, kh, e0)
    for i, t in enumerate(ts):
        qs = np.flatnonzero(rt == i)
        Pi, ri = dda.solve(t, opts, kh[qs], e0[qs])
        for j, q in enumerate(qs):
            assert torch.equal(Pb[q], Pi[j]) and rb[q] == ri[j]


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32_matvec", 2e-5)])
@pytest.mark.parametrize("box", [(12, 3, 4), (40, 2, 3), (3, 9, 5)])
def test_products_of_many_right_hand_sides_read_each_components_polarizability(dda, box, precision, tol):
    """GKDLDR's 1/alpha differs from axis to axis: a 24-right-hand-side product
    of one material takes each component's own, at compile-time (32, 80) and
    runtime-planned (6) x lengths, as the dense matrix does."""
    ijk = w.brick(*box)
    n = len(ijk)
    m = np.full(n, 2.0 + 0.5j)
    tgt = dda.Target(ijk, m)
    kh, e0 = w.incidences_for_orientations(65, 12)
    opts = dda.Options.for_size_parameter(1.5, precision=precision, polarizability="GKDLDR")
    xv = w.random_vectors(65, (24, n, 3))
    y = dda.apply(tgt, opts, kh, e0, _cuda(xv))
    for a, b in ((0, 8), (8, 24)):
        assert torch.equal(dda.apply(tgt, opts, kh[a:b], e0[a:b], _cuda(xv[a:b])), y[a:b])
    for q in (0, 9, 23):
        ref = (_dense_A(ijk, m, 1.5, kh[q], e0[q], "GKDLDR") @ xv[q].reshape(-1)).reshape(n, 3)
        assert np.abs(y[q].cpu().numpy() - ref).max() <= tol * np.abs(ref).max(), q


# ------------------------------------------------------------------ plane kernel: launch shapes

@pytest.mark.parametrize("precision,ny,nz", [("fp64", 24, 16), ("fp32_matvec", 13, 33), ("fp32_matvec", 16, 40),
                                             ("fp32_matvec", 24, 38), ("fp32_matvec", 48, 16)])
@pytest.mark.parametrize("n_rhs", [4, 5])
def test_plane_kernel_with_one_and_several_workgroups_a_compute_unit(dda, precision, ny, nz, n_rhs):
    """Launches of 256 and of 320 workgroups (x extent 64), on each side of the
    line where the plane kernel's wavefront count changes, at the lengths
    where it does (FP64 48 x 32, FP32 32 x 80, 48 x 80) and at FP32 96 x 32:
    bitwise the three separate passes."""
    rng = np.random.default_rng(ny + nz)
    keep = rng.random((30, ny, nz)) < 0.1
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = np.argwhere(keep).astype(np.int32)
    tgt = dda.Target(ijk, 1.4 + 0.1j)
    assert tgt.grid[0] == 64
    kh, e0 = np.tile([1.0, 0, 0], (n_rhs, 1)), np.tile(np.array([0, 1, 0], complex), (n_rhs, 1))
    xv = _cuda(w.random_vectors(71, (n_rhs, len(ijk), 3)))
    opts = dict(precision=precision)
    y = dda.apply(tgt, dda.Options.for_size_parameter(1.0, **opts), kh, e0, xv)
    assert dda.tuned_variants(tgt, n_rhs, precision) == (0, 0, 0)
    ref = dda.apply(tgt, dda.Options.for_size_parameter(1.0, kernel_variant=4, **opts), kh, e0, xv)
    assert torch.equal(y, ref)


@pytest.mark.parametrize("precision,box,n_rhs,plane", [
    ("fp64", (2, 64, 24), 1, False), ("fp64", (16, 64, 24), 1, False), ("fp64", (24, 64, 24), 1, True),
    ("fp64", (2, 64, 24), 8, False), ("fp64", (2, 64, 24), 9, True), ("fp64", (2, 64, 16), 1, True),
    ("fp64", (2, 32, 32), 1, False), ("fp64", (2, 16, 32), 1, True), ("fp32_matvec", (2, 64, 48), 1, False),
    ("fp32_matvec", (2, 16, 48), 8, False), ("fp32_matvec", (2, 16, 48), 9, True),
    ("fp32_matvec", (2, 24, 40), 1, True), ("fp32_matvec", (2, 48, 24), 1, True)])
def test_few_workgroups_of_long_planes_take_three_passes(dda, precision, box, n_rhs, plane):
    """Grids of few workgroups (padded x extent times right-hand sides) whose
    planes are long: passes 2-4 run as three kernels in fixed variants, at
    most 32 workgroups; others take the plane kernel.  The products are
    bitwise those of a named variant."""
    rng = np.random.default_rng(sum(box))
    keep = rng.random(box) < 0.1
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = np.argwhere(keep).astype(np.int32)
    tgt = dda.Target(ijk, 1.4 + 0.1j)
    assert tgt.grid[0] == {2: 4, 16: 32, 24: 48}[box[0]]
    kh, e0 = np.tile([1.0, 0, 0], (n_rhs, 1)), np.tile(np.array([0, 1, 0], complex), (n_rhs, 1))
    xv = _cuda(w.random_vectors(72, (n_rhs, len(ijk), 3)))
    y = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision), kh, e0, xv)
    assert dda.tuned_variants(tgt, n_rhs, precision) == (0, 0 if plane else 4 if precision == "fp64" else 3, 0)
    ref = dda.apply(tgt, dda.Options.for_size_parameter(1.0, precision=precision, kernel_variant=4), kh, e0, xv)
    assert torch.equal(y, ref)


# ------------------------------------------------------------------ far field: which form

@pytest.mark.parametrize("box,drop", [((16, 16, 16), 0), ((16, 16, 16), 1), ((8, 16, 32), 0), ((30, 30, 5), 0),
                                      ((21, 21, 21), 3700), ((24, 24, 24), 5600), ((8, 8, 128), 0), ((8, 8, 128), 8),
                                      ((32, 32, 16), 10900), ((32, 32, 16), 10930)])
def test_far_field_forms_about_their_line_match_the_oracle(dda, box, drop):
    """Boxes on each side of the lines that choose between the contraction
    along x and the sum over sites (4,096 and 8,192 sites, points of the rounded
    box per site, short x), over lists and average sets on each side of the
    counts that matter: amplitudes against the oracle's direct sum (1e-12),
    averages against the oracle's quadrature (1e-10), and every direction's
    amplitude the same bits in a list of its own, every right-hand side's in a
    call of its own."""
    from oracle import farfield
    rng = np.random.default_rng(drop + box[0])
    ijk = w.brick(*box)
    inner = np.flatnonzero(~np.all((ijk == ijk.min(0)) | (ijk == ijk.max(0)), axis=1))
    ijk = np.delete(ijk, rng.choice(inner, drop, replace=False), axis=0)
    n = len(ijk)
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    assert tgt.box == box
    P = w.random_vectors(81, (2, n, 3))
    opts = dda.Options.for_size_parameter(4.0)
    k = dense.kd_from_size_parameter(4.0, n)
    nh, th, ph = w.lab_directions(rng.uniform(0, 180, 83), rng.uniform(0, 360, 83))
    f, dcs = dda.far_field(tgt, opts, _cuda(P), nh, th, ph)
    for q in range(2):
        A = farfield.amplitude_vectors(ijk, P[q], k, nh)
        ref = np.stack([np.sum(th * A, axis=1), np.sum(ph * A, axis=1)], axis=1)
        assert np.abs(f[q] - ref).max() <= 1e-12 * np.abs(P[q]).sum() * k ** 3 / np.sqrt(n)
        f1, _ = dda.far_field(tgt, opts, _cuda(P[q:q + 1]), nh[40:41], th[40:41], ph[40:41])
        assert np.array_equal(f1[0, 0], f[q, 40])
    kh, e0 = w.along_x_yz()
    a = dense.aeff_over_d(n)
    for nt, nphi in ((5, 3), (20, 60), (32, 64)):
        av = dda.scattering_averages(tgt, opts, kh, e0, _cuda(P), nt, nphi)
        one = dda.scattering_averages(tgt, opts, kh[1:], e0[1:], _cuda(P[1:]), nt, nphi)
        assert one[0] == av[1]
        qs, g, c2 = farfield.angular_averages(ijk, P[0], k, kh[0], a, nt, nphi)
        assert abs(av[0]["qsca"] - qs) <= 1e-10 * qs
        assert abs(av[0]["g"] - g) <= 1e-10 and abs(av[0]["cos2"] - c2) <= 1e-10


def test_far_field_lines_of_one_and_three_components_agree(dda):
    """A launch of few wavefronts takes one component a wavefront, a larger one
    all three: a 4,096-site target's amplitudes over 3,000 directions (three
    components) equal, bitwise, those of the same directions 500 at a time."""
    ijk = w.brick(16, 16, 16)
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    rng = np.random.default_rng(82)
    nh, th, ph = w.lab_directions(rng.uniform(0, 180, 3000), rng.uniform(0, 360, 3000))
    P = _cuda(w.random_vectors(82, (1, len(ijk), 3)))
    opts = dda.Options.for_size_parameter(3.0)
    f, dcs = dda.far_field(tgt, opts, P, nh, th, ph)
    for d in range(0, 3000, 500):
        s = slice(d, d + 500)
        fs, ds = dda.far_field(tgt, opts, P, nh[s], th[s], ph[s])
        assert np.array_equal(fs[0], f[0, s]) and np.array_equal(ds[0], dcs[0, s])


def test_far_field_work_memory_is_bounded(dda):
    """65,535 directions on 4.1 million sites: the call works through them in
    groups, so that its work memory stays within 512 MiB beside its lists
    (taken on a context of its own, whose work memory starts empty); the
    amplitudes of directions about the groups' ends are bitwise those of short
    lists."""
    import ctypes
    from paper_1202_3424_amd import _abi
    lib = _abi.load()
    ijk = w.brick(160, 160, 160)
    n, nd = len(ijk), 65535
    m = np.full(n, 1.5 + 0.1j)
    ctx, tgt = ctypes.c_void_p(), ctypes.c_void_p()
    assert lib.dda_ctx_create(0, None, ctypes.byref(ctx)) == 0
    try:
        assert lib.dda_target_create(ctx, n, ijk.ctypes.data, m.ctypes.data, ctypes.byref(tgt)) == 0
        g = torch.Generator(device="cuda")
        g.manual_seed(83)
        P = torch.randn((1, n, 3), generator=g, dtype=torch.complex128, device="cuda")
        rng = np.random.default_rng(83)
        fr = [np.ascontiguousarray(a) for a in w.lab_directions(rng.uniform(0, 180, nd), rng.uniform(0, 360, nd))]
        o = dda.Options.for_size_parameter(8.0).c()

        def far(sl):
            d = [np.ascontiguousarray(a[sl]) for a in fr]
            f = np.zeros((len(d[0]), 2), dtype=np.complex128)
            dcs = np.zeros(len(d[0]))
            assert lib.dda_far_field(ctx, tgt, ctypes.byref(o), 1, P.data_ptr(), len(d[0]), d[0].ctypes.data,
                                     d[1].ctypes.data, d[2].ctypes.data, f.ctypes.data, dcs.ctypes.data) == 0
            return f, dcs

        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        f, dcs = far(slice(0, nd))
        torch.cuda.synchronize()
        lists = nd * (9 + 4 + 1) * 8
        assert free0 - torch.cuda.mem_get_info()[0] <= (512 << 20) + lists + (8 << 20)
        for d in (0, 4090, 24570, 28668, 32760, 61436, nd - 9):
            fs, ds = far(slice(d, d + 9))
            assert np.array_equal(fs, f[d:d + 9]) and np.array_equal(ds, dcs[d:d + 9]), d
    finally:
        if tgt:
            lib.dda_target_destroy(tgt)
        lib.dda_ctx_destroy(ctx)


@pytest.mark.parametrize("precision,edge", [("fp64", 20), ("fp32_matvec", 34)])
def test_near_field_volume_is_tuned_apart_from_a_target_of_its_box(dda, precision, edge):
    """The passes of a near-field volume cover its input window: their tuned
    variants are not those of an ordinary target that fills the same box with
    the same count of right-hand sides."""
    small = dda.Target(w.brick(edge, edge, edge), 1.5 + 0.1j)
    big = dda.Target(np.array([[0, 0, 0]] + [[2 * edge - 1] * 3]), 1.5 + 0.1j)
    kh, e0 = w.incidences_for_orientations(91, 7)
    opts = dda.Options.for_size_parameter(1.3, precision=precision)
    assert dda.tuned_variants(big, 14, precision) == (-1, -1, -1)
    _, dims, _, _ = dda.nearfield(small, opts, (0.5,) * 6, kh, e0, _cuda(w.random_vectors(91, (14, edge ** 3, 3))))
    assert tuple(dims) == big.box
    assert dda.tuned_variants(big, 14, precision) == (-1, -1, -1)
    dda.apply(big, opts, kh, e0, _cuda(w.random_vectors(92, (14, 2, 3))))
    v = dda.tuned_variants(big, 14, precision)
    assert all(0 <= a < 28 for a in v) and v != (0, 0, 0)


# ------------------------------------------------------------------ grids that the plane kernel does not take

def _sparse_target(dda, box, seed, m=(1.4 + 0.1j,), p=0.02):
    """About a fiftieth of the box's points, its corners among them."""
    keep = np.random.default_rng(seed).random(box) < p
    keep[0, 0, 0] = keep[-1, -1, -1] = True
    ijk = np.argwhere(keep).astype(np.int32)
    tgt = dda.Target(ijk, np.asarray(m)[np.arange(len(ijk)) % len(m)])
    assert tgt.box == tuple(box)
    return tgt


def _launches(dda, fn):
    """fn() and the launches of each kernel category it made."""
    dda.set_timing(True)
    try:
        out = fn()
        torch.cuda.synchronize()
        return out, {k: v[2] for k, v in dda.get_timing().items()}
    finally:
        dda.set_timing(False)


# boxes whose y and z extents have compile-time lengths without a plane kernel
# (FP64 80 x 80; FP32 128 x 128)
NO_PLANE = {"fp64": ((12, 36, 34), (14, 33, 40)), "fp32_matvec": ((12, 60, 52), (14, 64, 63))}


@pytest.mark.parametrize("precision,box,n_rhs,plane", [
    ("fp64", (16, 32, 32), 4, True), ("fp64", (12, 36, 34), 4, False), ("fp64", (3, 7, 9), 2, True),
    ("fp64", (5, 9, 24), 8, False), ("fp64", (40, 48, 30), 2, True), ("fp64", (40, 30, 48), 2, False),
    ("fp32_matvec", (16, 40, 40), 4, True), ("fp32_matvec", (12, 60, 52), 4, False),
    ("fp32_matvec", (30, 60, 40), 2, True), ("fp32_matvec", (3, 70, 5), 2, False)])
def test_which_grids_take_the_plane_kernel(dda, precision, box, n_rhs, plane):
    """A product runs the forward y pass as a kernel of its own exactly where
    the plane kernel does not take its grid (and always where a variant is
    named), with bitwise the same result."""
    tgt = _sparse_target(dda, box, 101)
    kh, e0 = np.tile([1.0, 0, 0], (n_rhs, 1)), np.tile(np.array([0, 1, 0], complex), (n_rhs, 1))
    xv = _cuda(w.random_vectors(101, (n_rhs, tgt.n_sites, 3)))
    opts = dda.Options.for_size_parameter(1.0, precision=precision)
    dda.apply(tgt, opts, kh, e0, xv)   # builds the tensor, tunes
    y, launches = _launches(dda, lambda: dda.apply(tgt, opts, kh, e0, xv))
    assert (launches["fft_y_fwd"] == 0) == plane and launches["fft_z_green"] == 1
    named = dataclasses.replace(opts, kernel_variant=4)
    ref, launches = _launches(dda, lambda: dda.apply(tgt, named, kh, e0, xv))
    assert launches["fft_y_fwd"] == 1
    assert torch.equal(y, ref)


@pytest.mark.parametrize("precision", sorted(NO_PLANE))
@pytest.mark.parametrize("solver", ["bicgstab", "qmr", "bicgstab2"])
def test_tuned_separate_passes_equal_the_default_ones(dda, solver, precision):
    """A solve with the autotuned tilings of the three passes equals, bitwise,
    one with the default tilings, on a grid that runs them."""
    tgt = _sparse_target(dda, NO_PLANE[precision][0], 102)
    kh, e0 = w.along_x_yz()
    opts = dda.Options.for_size_parameter(2.0, solver=solver, precision=precision)
    (P1, r1), launches = _launches(dda, lambda: dda.solve(tgt, opts, kh, e0))
    assert launches["fft_y_fwd"] > 0
    P2, r2 = dda.solve(tgt, dataclasses.replace(opts, autotune=False), kh, e0)
    assert torch.equal(P1, P2) and r1 == r2


@pytest.mark.parametrize("precision", sorted(NO_PLANE))
@pytest.mark.parametrize("solver", ["bicgstab", "qmr", "bicgstab2"])
def test_separate_passes_in_shared_launches_and_graphs(dda, solver, precision):
    """Two targets of different boxes on one padded grid whose passes 2-4 are
    separate kernels: the batch that shares every launch (each right-hand side
    its own target's extents and tensor), replayed from graphs several times
    with other solves between, launched directly, and as separate targets
    equals, bitwise, the targets solved alone."""
    ts = [_sparse_target(dda, b, 103 + i, m=(1.4 + 0.1j, 1.7 + 0.3j)) for i, b in enumerate(NO_PLANE[precision])]
    assert ts[0].grid == ts[1].grid
    kh, e0 = w.incidences_for_orientations(103, 3)
    opts = [dda.Options.for_size_parameter(x, tol=tol, solver=solver, precision=precision)
            for x, tol in ((2.0, 1e-5), (1.6, 1e-6))]
    rt = np.array([0, 1, 1, 0, 1, 0])
    alone = []
    for i, t in enumerate(ts):
        alone.append(dda.solve(t, opts[i], kh[rt == i], e0[rt == i]))

    def check(P, r):
        for i in range(2):
            for j, q in enumerate(np.flatnonzero(rt == i)):
                assert torch.equal(P[q], alone[i][0][j]) and r[q] == alone[i][1][j], (i, q)

    for _ in range(3):
        check(*dda.solve_batched(ts, opts, rt, kh, e0))
        dda.solve(ts[0], opts[0], kh[:2], e0[:2])
        torch.cuda.synchronize()
    (P, r), launches = _launches(dda, lambda: dda.solve_batched(
        ts, [dataclasses.replace(o, graphs=False) for o in opts], rt, kh, e0))
    assert launches["fft_y_fwd"] > 0
    check(P, r)
    check(*dda.solve_batched(ts, [dataclasses.replace(o, share_launches=False) for o in opts], rt, kh, e0))


# points of the volume below and above a 4-site box on x, y, z: volumes of 7,
# 10, 24 and about 131 points (padded 15, 20, 48 and 270)
NF_RUNTIME_WINDOWS = {
    "y10_z24": ((1, 2), (2, 4), (8, 12)),
    "y24_z10": ((0, 0), (8, 12), (6, 0)),
    "x10_y10_z24": ((6, 0), (0, 6), (20, 0)),
    "y132": ((0, 3), (64, 64), (0, 3)),
    "z131": ((3, 0), (2, 1), (64, 63)),
}


@pytest.mark.parametrize("name", sorted(NF_RUNTIME_WINDOWS))
@pytest.mark.parametrize("precision", ["fp64", "fp32_matvec"])
def test_nearfield_input_window_through_runtime_planned_passes(dda, name, precision):
    """Windows of volumes with a y or z extent that has no compile-time length
    and that run separate passes: every variant of the other axis' pass gives
    the same bits, within the tolerances of
    test_nearfield_matches_oracle_everywhere of the oracle's direct sums."""
    from oracle import nearfield
    ends = NF_RUNTIME_WINDOWS[name]
    ext = tuple(b / 4 for axis in ends for b in axis)
    ijk = np.array([[0, 0, 0], [3, 3, 3], [0, 3, 1], [3, 0, 2], [1, 2, 0], [2, 1, 3]], dtype=np.int32)
    tgt = dda.Target(ijk, 1.5 + 0.1j)
    kh, e0 = np.array([[0.36, 0.48, 0.8]] * 2), np.array([[0.8, -0.6, 0]] * 2, dtype=complex)
    P = w.random_vectors(104, (2, len(ijk), 3))
    opts = dda.Options.for_size_parameter(1.3, precision=precision)
    (org, dims, Ei, Es), launches = _launches(dda, lambda: dda.nearfield(tgt, opts, ext, kh, e0, _cuda(P)))
    assert launches["fft_y_fwd"] > 0
    assert list(dims) == [4 + b + a for b, a in ends]
    for variant in range(1, 29):
        assert torch.equal(dda.nearfield(tgt, dataclasses.replace(opts, kernel_variant=variant), ext, kh, e0,
                                         _cuda(P))[3], Es), variant
    k = dense.kd_from_size_parameter(1.3, len(ijk))
    tol = 1e-12 if precision == "fp64" else 2e-5
    for q in range(2):
        _, _, ri, rs = nearfield.nearfield(ijk, P[q], k, kh[q], e0[q], ext)
        assert np.abs(Es[q].cpu().numpy() - rs).max() <= tol * np.abs(rs).max(), q
        assert np.abs(Ei[q].cpu().numpy() - ri).max() <= 1e-13, q
