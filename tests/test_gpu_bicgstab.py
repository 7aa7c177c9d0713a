"""Parity of the HIP multishift BiCGStab (multishift_bicgstab) with the oracle."""
import os

import numpy as np
import pytest

import synth
from oracle import WilsonRef, dense, krylov, rational

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0910_1048_amd as sgn  # noqa: E402
from gpu_util import dev, host, lattice  # noqa: E402

GOLD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "c1_dense.npz")


def _rel(a, b):
    a = np.asarray(a).ravel()
    b = np.asarray(b).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _solve(lat, mu, b, rf, defl=None, want_shifts=False, **kw):
    bd = dev(b)
    x = torch.empty_like(bd)
    xs = [torch.empty_like(bd) for _ in range(rf.s)] if want_shifts else None
    st = sgn.multishift_bicgstab(sgn.Problem(lat, mu, bd, x, defl, xs), rf, **kw)[0]
    if want_shifts:
        return host(x).ravel(), st, [host(t).ravel() for t in xs]
    return host(x).ravel(), st


def test_c1_bicgstab_matches_dense_rational():
    dims = (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    g = np.load(GOLD)
    rf = sgn.sgn_rational_neuberger(16, float(g["alpha"]), float(g["beta"]))
    lat = lattice(U, dims)
    x, st = _solve(lat, 0.3, b, rf, tol=1e-11)
    e = _rel(x, g["g16_b"])
    bd = dev(b)
    xb = torch.empty_like(bd)
    sb = sgn.multishift_solve(sgn.Problem(lat, 0.3, bd, xb), rf, tol=1e-11)[0]
    print(f"C1 BiCGStab: vs dense g16 {e:.2e}, {st['iterations']} iterations ({st['matvecs']} matvecs); "
          f"BiCG {sb['iterations']} iterations, BiCGStab vs BiCG {_rel(x, host(xb)):.1e}", flush=True)
    assert e < 1e-8
    assert _rel(x, host(xb)) < 1e-8


def test_8x4_bicgstab_against_oracle():
    dims = (8, 8, 8, 8)
    U = synth.gauge_field(dims, 0.4, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    W = WilsonRef(U, dims, 0.2)
    om, sg, c = rational.coefficients(16, 0.15, 2.6)
    rf = sgn.sgn_rational_neuberger(16, 0.15, 2.6)
    x, st = _solve(lattice(U, dims), 0.2, b, rf, tol=1e-11)
    xo, info = krylov.multishift_bicgstab(lambda v: W.apply(v, 0.2), b, om, sg, c, tol=1e-11, return_info=True)
    e = _rel(x, xo)
    print(f"8^4 BiCGStab: vs oracle {e:.2e}, {st['iterations']} iterations (oracle {info['iterations']}), "
          f"{st['krylov_ms']:.1f} ms", flush=True)
    assert e < 1e-8
    assert abs(st["iterations"] - info["iterations"]) <= 2


def test_bicgstab_shift_solutions_match_oracle():
    dims = (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, 2)
    b = synth.gaussian_source(dims, 2).ravel()
    W = WilsonRef(U, dims, 0.2)
    om, sg, c = rational.coefficients(10, 0.2, 2.4)
    rf = sgn.sgn_rational_neuberger(10, 0.2, 2.4)
    _, info = krylov.multishift_bicgstab(lambda v: W.apply(v, 0.25), b, om, sg, c, tol=1e-11, return_info=True)
    for form, kw in (("per-shift", dict(basis_slots=-1)), ("stored", {})):
        _, st, xs = _solve(lattice(U, dims), 0.25, b, rf, want_shifts=True, tol=1e-11, **kw)
        worst = max(_rel(xs[i], info["X"][i]) for i in range(10))
        print(f"BiCGStab {form} form, shifted solutions vs oracle: worst {worst:.1e}", flush=True)
        assert worst < 1e-8


def test_deflated_bicgstab_against_dense():
    dims = (2, 2, 2, 4)
    U = synth.gauge_field(dims, 0.5, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    H = WilsonRef(U, dims, 0.2).dense(0.3)
    lam, R = np.linalg.eig(H)
    Linv = np.linalg.inv(R)
    idx = np.argsort(np.abs(lam.real))[:8]
    Lr, Rr, lm = Linv[idx].conj(), R[:, idx].T.copy(), lam[idx]
    rest = np.delete(lam, idx)
    alpha, beta = float(np.abs(rest).min()), float(np.abs(lam).max())
    om, sg, c = rational.coefficients(12, alpha, beta)
    rf = sgn.sgn_rational_neuberger(12, alpha, beta)
    defl = sgn.Deflation(dev(Lr), dev(Rr), lm)
    x, _ = _solve(lattice(U, dims), 0.3, b, rf, defl=defl, tol=1e-12)
    target = krylov.deflation_xP(Lr.T, Rr.T, lm, b) + dense.rational_dense(H, krylov.project_out(Lr.T, Rr.T, b),
                                                                             om, sg, c)
    assert _rel(x, target) < 1e-9


def test_bicgstab_zero_source_and_errors():
    dims = (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    lat = lattice(U, dims)
    rf = sgn.sgn_rational_neuberger(8, 0.2, 2.4)
    x, st = _solve(lat, 0.3, np.zeros_like(b), rf)
    assert np.all(x == 0) and st["iterations"] == 0
    with pytest.raises(sgn.SgnError) as e:
        _solve(lat, 0.3, b, rf, tol=1e-11, maxiter=3)
    assert e.value.status == 5
    with pytest.raises(sgn.SgnError) as e:
        _solve(lat, 0.3, b, rf, basis_slots=-1, prec=sgn.F32)  # per-shift form: FP64 only
    assert e.value.status == 1
    with pytest.raises(sgn.SgnError) as e:
        _solve(lat, 0.3, b, rf, basis_slots=9)  # stored basis beyond its cap
    assert e.value.status == 3


def test_stored_basis_equals_per_shift_form():
    dims = (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    g = np.load(GOLD)
    rf = sgn.sgn_rational_neuberger(16, float(g["alpha"]), float(g["beta"]))
    lat = lattice(U, dims)
    xs, ss = _solve(lat, 0.3, b, rf, tol=1e-11)
    xe, se = _solve(lat, 0.3, b, rf, tol=1e-11, basis_slots=-1)
    print(f"BiCGStab stored vs per-shift: {_rel(xs, xe):.1e}, iterations {ss['iterations']} / {se['iterations']}",
          flush=True)
    assert _rel(xs, xe) < 1e-9
    assert _rel(xs, g["g16_b"]) < 1e-8
    # graph replays and plain launches give the same bits
    xg, _ = _solve(lat, 0.3, b, rf, tol=1e-11, graph=False)
    assert np.array_equal(xg, xs)


@pytest.mark.parametrize("prec", [sgn.F32, sgn.F32_H16])
def test_c1_mixed_bicgstab_matches_dense_rational(prec):
    dims = (4, 4, 4, 4)
    U = synth.gauge_field(dims, 0.5, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    g = np.load(GOLD)
    rf = sgn.sgn_rational_neuberger(16, float(g["alpha"]), float(g["beta"]))
    x, st = _solve(lattice(U, dims), 0.3, b, rf, tol=1e-10, prec=prec)
    e = _rel(x, g["g16_b"])
    print(f"C1 mixed BiCGStab prec={prec}: vs dense g16 {e:.2e}, {st['iterations']} iterations, "
          f"{st['reliable_updates']} reliable updates", flush=True)
    assert st["reliable_updates"] >= 1
    assert e < 1e-8


def test_8x4_mixed_bicgstab_against_oracle():
    dims = (8, 8, 8, 8)
    U = synth.gauge_field(dims, 0.4, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    W = WilsonRef(U, dims, 0.2)
    om, sg, c = rational.coefficients(16, 0.15, 2.6)
    rf = sgn.sgn_rational_neuberger(16, 0.15, 2.6)
    x, st = _solve(lattice(U, dims), 0.2, b, rf, tol=1e-10, prec=sgn.F32_H16)
    xo = krylov.multishift_bicgstab(lambda v: W.apply(v, 0.2), b, om, sg, c, tol=1e-11)
    e = _rel(x, xo)
    print(f"8^4 mixed BiCGStab: vs oracle {e:.2e}, {st['iterations']} iterations, {st['reliable_updates']} RU, "
          f"{st['total_ms']:.1f} ms", flush=True)
    assert e < 1e-8


def test_full_size_bench_configuration_residuals_with_oracle_operator():
    """24^3 x 48 in the benchmark's configuration (stored basis, FP64 -> FP32 -> FP16 links,
    tolerance 1e-9, thresholds 1e-2 / 1e-5).  Only the seed is reliable-updated, so the solve is
    repeated with verify: every shifted solution is then checked in FP64 and refined where needed.
    All 16 verified solutions satisfy their systems, checked with the oracle's operator on the
    CPU; x is their omega-weighted sum; and the benchmark's unverified result agrees with it."""
    dims = (24, 24, 24, 48)
    U = synth.gauge_field(dims, 0.4, 0)
    b = synth.gaussian_source(dims, 0).ravel()
    alpha, beta = 0.12, 2.6
    rf = sgn.sgn_rational_neuberger(16, alpha, beta)
    om, sg, c = rational.coefficients(16, alpha, beta)
    lat = lattice(U, dims)
    kw = dict(tol=1e-9, prec=sgn.F32_H16, theta32=1e-2, theta16=1e-5, delta=0.05)
    x_bench, st_b = _solve(lat, 0.2, b, rf, **kw)
    x, st, xs = _solve(lat, 0.2, b, rf, want_shifts=True, verify=True, **kw)
    print(f"24^3x48 mixed BiCGStab: iters {st['iterations']} reliable {st['reliable_updates']}, refine "
          f"iterations {st['refine_iterations']}, {st['krylov_ms']:.0f} ms", flush=True)
    W = WilsonRef(U, dims, 0.2)
    y = c * W.apply(b, 0.2).ravel()
    for i in range(rf.s):  # every shifted system
        Ax = W.apply(W.apply(xs[i], 0.2), 0.2).ravel()
        res = np.linalg.norm(y - (c * c * Ax - sg[i] * xs[i])) / np.linalg.norm(y)
        print(f"  shift {i}: oracle residual {res:.2e}, library FP64 residual {st['shift_residual'][i]:.2e}",
              flush=True)
        assert res < 1.5e-9
    assert _rel(x, om @ np.stack(xs)) < 1e-12
    e = _rel(x_bench, x)
    print(f"  unverified (benchmark) result vs verified: {e:.2e}", flush=True)
    assert e < 5e-9


@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (16, 16, 16, 17)])
@pytest.mark.parametrize("nprob", [1, 2])
def test_either_side_of_the_fused_scalar_steps(dims, nprob):
    # FP32 dotting stencils leave one partial sum per 64 sites (and one for the padding): up to 1024 of them
    # every block of the vector kernels adds them, above it is a launch of its own (65536 and 69632 sites)
    lat = lattice(synth.gauge_field(dims, 0.4, 3), dims)
    rf = sgn.sgn_rational_neuberger(16, 0.12, 2.6)
    bs = [dev(synth.gaussian_source(dims, k).ravel()) for k in range(nprob)]

    def solve(prec):
        probs = [sgn.Problem(lat, 0.1 + 0.1 * k, b, torch.empty_like(b)) for k, b in enumerate(bs)]
        sgn.multishift_bicgstab(probs, rf, tol=1e-10, prec=prec, theta32=1e-4)
        return [host(p.x) for p in probs]
    for x64, x32 in zip(solve(sgn.F64), solve(sgn.F32)):
        assert np.linalg.norm(x32 - x64) / np.linalg.norm(x64) < 1e-8
