"""Batches at the limits of their launch rules.  Launches of several right-hand sides on lattices whose shape was tuned
to the kernel without LDS staging (on small lattices the split kernel): above the 9 MiB of fields that it takes they
stay one launch, with the same bits.  Batches with a pinned shape beside an untuned one, and on either side of the
2048 vector blocks up to which the scalar steps are part of the vector kernels."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0910_1048_amd as sgn  # noqa: E402
from gpu_util import dev  # noqa: E402

CLASS = {sgn.F64: "stencil_f64", sgn.F32: "stencil_f32", sgn.F32_H16: "stencil_h16"}
CDT = {sgn.F64: np.complex128, sgn.F32: np.complex64, sgn.F32_H16: np.complex64}


def _calls(c, name, fn):
    sgn.sgn_profile_enable(c, True)
    try:
        r = fn()
        torch.cuda.synchronize()
        return sgn.sgn_profile_read(c)[name]["calls"], r
    finally:
        sgn.sgn_profile_enable(c, False)


def _split_chosen(lat):
    """as sgn_autotune leaves it where the split kernel was the fastest, for one and for several right-hand sides"""
    for p in CLASS:
        sgn.sgn_tune_set(lat, p, False, -1, 1)
        sgn.sgn_tune_set(lat, p, True, -1, 1)


# (lattices, problems on each): groups of several right-hand sides, and groups of one beside an untuned lattice;
# FP64 fields of 18.9 and 13.4 MB together, and 4.0 MB for the split kernel
@pytest.mark.parametrize("dims,nprob,tuned", [([(8, 8, 8, 8)], 24, [0]), ([(8, 8, 8, 8), (16, 16, 16, 16)], 1, [0]),
                                              ([(8, 8, 8, 8), (12, 12, 4, 4)], 2, [0, 1])])
@pytest.mark.parametrize("solver", [sgn.multishift_bicgstab, sgn.multishift_solve, sgn.multishift_qmr])
def test_solver_batches_stay_batched(dims, nprob, tuned, solver):
    c = sgn.Context(0)
    lats = [sgn.Lattice(c, dev(synth.gauge_field(d, 0.3, 3)), d, 0.15) for d in dims]
    rf = sgn.sgn_rational_neuberger(8, 0.3, 2.3)
    src = [(lat, 0.02 * k, dev(synth.gaussian_source(d, k).ravel())) for lat, d in zip(lats, dims) for k in range(nprob)]

    def solve():
        probs = [sgn.Problem(lat, mu, b, torch.empty_like(b)) for lat, mu, b in src]
        solver(probs, rf, tol=1e-8, prec=sgn.F64)
        return [p.x for p in probs]

    calls, first = _calls(c, CLASS[sgn.F64], solve)
    for k in tuned:
        _split_chosen(lats[k])
    calls2, again = _calls(c, CLASS[sgn.F64], solve)
    assert calls2 == calls
    for x, y in zip(first, again):
        assert torch.equal(x, y)


@pytest.mark.parametrize("prec", [sgn.F64, sgn.F32, sgn.F32_H16])
@pytest.mark.parametrize("nrhs", [2, 16])
def test_blocks_of_right_hand_sides_stay_one_launch(prec, nrhs):
    dims = (12, 12, 12, 12)   # 4.0 and 2.0 MB a field: two fit the split kernel, sixteen do not
    c = sgn.Context(0)
    lat = sgn.Lattice(c, dev(synth.gauge_field(dims, 0.3, 3)), dims, 0.15)
    nb = lat.spinor_bytes(prec)
    x = [torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in range(nrhs)]
    for j, t in enumerate(x):
        sgn.sgn_spinor_pack(lat, dev(synth.gaussian_source(dims, j).astype(CDT[prec])), t, prec)
    mus = [0.05 * j for j in range(nrhs)]

    def apply():
        y = [torch.empty_like(t) for t in x]
        sgn.wilson_apply_multi(lat, mus, x, y, prec)
        return y

    calls, first = _calls(c, CLASS[prec], apply)
    _split_chosen(lat)
    calls2, again = _calls(c, CLASS[prec], apply)
    assert calls == 1 and calls2 == 1
    for a, b in zip(first, again):
        assert torch.equal(a, b)


@pytest.mark.parametrize("nrhs,offered", [(1, True), (2, True), (16, False)])
def test_the_split_kernel_is_offered_for_the_fields_that_it_takes(nrhs, offered):
    dims = (12, 12, 12, 12)
    c = sgn.Context(0)
    lat = sgn.Lattice(c, dev(synth.gauge_field(dims, 0.3, 3)), dims, 0.15)
    cands = sgn.sgn_autotune(lat, sgn.F32, nrhs, reps=2)
    assert any(k["block_sites"] == 0 for k in cands) == offered


def test_a_refused_autotune_leaves_the_lattice_untuned():
    """A lattice without FP32 links cannot be tuned for FP32; the other lattices of its dimensions keep the split
    kernel, which runs the two applications of a Lanczos step in one launch."""
    dims = (8, 8, 8, 8)
    c = sgn.Context(0)
    U = dev(synth.gauge_field(dims, 0.3, 3))
    lat = sgn.Lattice(c, U, dims, 0.15)
    only64 = sgn.Lattice(c, U, dims, 0.15, prec_mask=1 << sgn.F64)
    b = dev(synth.gaussian_source(dims, 1).ravel())

    def solve():
        x = torch.empty_like(b)
        sgn.sign_lanczos_2sided(lat, 0.1, b, x, k=20, prec=sgn.F32)
        return x

    calls, first = _calls(c, CLASS[sgn.F32], solve)
    with pytest.raises(sgn.SgnError):
        sgn.sgn_autotune(only64, sgn.F32, 1, reps=2)
    calls2, again = _calls(c, CLASS[sgn.F32], solve)
    assert calls2 == calls
    assert torch.equal(first, again)


@pytest.mark.parametrize("prec", [sgn.F64, sgn.F32, sgn.F32_H16])
@pytest.mark.parametrize("solver", [sgn.multishift_bicgstab, sgn.multishift_solve, sgn.multishift_qmr])
def test_split_and_staged_groups_in_one_batch(solver, prec):
    """A lattice with a pinned staged shape beside one on the split kernel: two launches per stencil step, and the
    bits of the batch that is all on the split kernel (the pinned shape is the one whose sums that kernel leaves)."""
    c = sgn.Context(0)
    dims = [(8, 8, 8, 8), (12, 12, 4, 4)]
    lats = [sgn.Lattice(c, dev(synth.gauge_field(d, 0.3, 3)), d, 0.15) for d in dims]
    rf = sgn.sgn_rational_neuberger(8, 0.3, 2.3)
    src = [(lat, 0.02 * k, dev(synth.gaussian_source(d, k).ravel())) for k in range(2) for lat, d in zip(lats, dims)]

    def solve():
        probs = [sgn.Problem(lat, mu, b, torch.empty_like(b)) for lat, mu, b in src]
        st = solver(probs, rf, tol=1e-8, prec=prec)
        return [p.x for p in probs], [k["iterations"] for k in st]

    first, its = solve()
    for p in CLASS:
        sgn.sgn_tune_set(lats[0], p, False, 0, 1)
        sgn.sgn_tune_set(lats[0], p, True, 0, 1)
    again, its2 = solve()
    assert its == its2
    for x, y in zip(first, again):
        assert torch.equal(x, y)


# 16^4: 1024 vector blocks a problem, the most that one takes
@pytest.mark.parametrize("nprob", [2, 3])
@pytest.mark.parametrize("solver,prec", [(sgn.multishift_bicgstab, sgn.F64), (sgn.multishift_bicgstab, sgn.F32),
                                         (sgn.multishift_qmr, sgn.F64), (sgn.multishift_qmr, sgn.F32)])
def test_either_side_of_the_fused_scalar_steps_in_a_batch(solver, prec, nprob):
    c = sgn.Context(0)
    dims = (16, 16, 16, 16)
    lat = sgn.Lattice(c, dev(synth.gauge_field(dims, 0.3, 3)), dims, 0.15)
    rf = sgn.sgn_rational_neuberger(8, 0.3, 2.3)
    src = [(0.02 * k, dev(synth.gaussian_source(dims, k).ravel())) for k in range(nprob)]

    def solve(which):
        probs = [sgn.Problem(lat, mu, b, torch.empty_like(b)) for mu, b in which]
        st = solver(probs, rf, tol=1e-10, prec=prec)
        return [p.x for p in probs], [k["iterations"] for k in st]

    xs, its = solve(src)
    for k in (0, nprob - 1):
        x, it = solve(src[k:k + 1])
        if prec == sgn.F64 and solver is sgn.multishift_bicgstab:  # the same sums in the same order
            assert torch.equal(xs[k], x[0]) and it[0] == its[k]
        # else: the solvers' tolerance, times ten for its being a residual's, twice
        assert torch.linalg.norm(xs[k] - x[0]) <= 2e-9 * torch.linalg.norm(x[0])
