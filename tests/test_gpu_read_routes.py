"""The read-only passes at the edges of the rule that gives a small frame a
block of its own or three passes, and the forward rows on both sides of the
stack size from which the same rows of several frames lie side by side."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-4          # relative, as in the parity tests


def on_device(pb, pos=None, stack=0):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    to = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", t)  # noqa: E731
    args = to(pb.iobs, torch.float32), to(pb.mask, torch.uint8), pb.wl.n_modes, pb.wl.obj_shape
    plan = P.Plan(pb.offsets, *args, stack=stack) if pos is None else P.Plan.with_positions(pos, *args, stack=stack)
    return plan, to(pb.obj0, torch.complex64), to(pb.probe0, torch.complex64), to


def check(pb, plan, o, p, to, frac=None):
    host = lambda t: t.cpu().numpy()  # noqa: E731
    kw = {} if frac is None else {"frac": frac}
    assert rel_l2(host(plan.icalc(o, p)), oracle.simulate_intensity(pb.obj0, pb.probe0, pb.offsets, **kw)) < TOL
    ref, nobs = oracle.llk(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask, **kw)
    llk = host(plan.llk(o, p))
    assert abs(llk[0] - ref) < TOL * abs(ref) and llk[1] == nobs
    # along the negative gradient, the direction a line search takes
    go, gp, _ = oracle.ml_grad(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask, **kw)
    do, dp = (-go).astype(np.complex64), (-gp).astype(np.complex64)
    c = host(plan.ml_linesearch(o, p, to(do, torch.complex64), to(dp, torch.complex64)))
    r = oracle.linesearch_coefs(pb.obj0, pb.probe0, do, dp, pb.offsets, pb.iobs, pb.mask, **kw)
    assert abs(c[0] - r[0]) < TOL * abs(r[0]) and abs(c[1] - r[1]) < TOL * abs(r[1])


@pytest.mark.parametrize("n,k,j,stack", [(32, 1, 1, 0), (32, 4, 2, 0), (64, 4, 2, 0), (64, 4, 3, 0), (64, 3, 179, 0),
                                         (64, 3, 180, 0), (64, 4, 257, 0), (64, 4, 359, 0), (64, 3, 769, 0),
                                         (64, 3, 150, 40), (64, 4, 300, 255), (64, 4, 300, 256)])
def test_integer_windows(n, k, j, stack):
    print(f"[gpu-case] read routes n={n} k={k} j={j} stack={stack}", flush=True)
    shape = (2 * n + 5, 2 * n + 1)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=shape, step=0.4 * n / np.sqrt(j), mask_frac=0.03), start="ml")
    check(pb, *on_device(pb, stack=stack))


@pytest.mark.parametrize("n,k,j", [(32, 4, 128), (32, 4, 129), (64, 2, 1), (64, 2, 179), (64, 2, 180), (64, 2, 257)])
def test_sub_pixel_windows(n, k, j):
    print(f"[gpu-case] read routes, sub-pixel n={n} k={k} j={j}", flush=True)
    shape = (2 * n + 3, 2 * n + 8)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=shape, step=1.0, mask_frac=0.03), start="ml")
    pos = np.random.default_rng(n + j).uniform(-0.4 * n, 0.4 * n, (j, 2))
    pb.offsets, frac = oracle.windows_from_positions(pos, n, shape)
    pb.iobs = oracle.simulate_intensity(pb.obj_true, pb.probe_true, pb.offsets, frac=frac).astype(np.float32)
    check(pb, *on_device(pb, pos), frac=frac)


@pytest.mark.parametrize("k,j", [(1, 16), (1, 17), (4, 4), (4, 5)])
def test_forward_rows_around_the_cached_stack_size(k, j):
    print(f"[gpu-case] forward rows n=512 k={k} j={j}", flush=True)
    pb = make_problem(small("ml256", n=512, k=k, j=j, obj=(560, 571), step=5.0, mask_frac=0.03), start="ml")
    plan, o, p, _ = on_device(pb)
    got = plan.icalc(o, p).cpu().numpy()
    assert rel_l2(got, oracle.simulate_intensity(pb.obj0, pb.probe0, pb.offsets)) < TOL


def test_a_cycle_whose_line_search_takes_three_passes():
    """A plan whose projections take a frame per block keeps no row transforms: the line search forms all three."""
    import paper_2008_11511_amd as P
    n, k, j = 64, 4, 300
    print(f"[gpu-case] CG cycle n={n} k={k} j={j}", flush=True)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=(2 * n + 5, 2 * n + 1), step=0.4 * n / np.sqrt(j),
                            mask_frac=0.03), start="ml")
    plan, o, p, _ = on_device(pb)
    both = oracle.UPDATE_OBJECT | oracle.UPDATE_PROBE
    plan.ml_cycle(o, p, plan.ml_state(), 1, P.UPDATE_OBJECT | P.UPDATE_PROBE, reset=True)
    ro, rp = oracle.ml_cycle(pb.obj0, pb.probe0, oracle.CGState(), pb.offsets, pb.iobs, pb.mask, both)
    assert rel_l2(o.cpu().numpy(), ro) < TOL and rel_l2(p.cpu().numpy(), rp) < TOL
