"""The one-kernel path of small far-field frames against the oracle at the
edges of its rule: frame counts on both sides of 128 per launch, counts that
leave a part of the last block or round empty, every mode count, ragged
stacks, sub-pixel windows."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
UPD = oracle.UPDATE_OBJECT | oracle.UPDATE_PROBE
TOL = 1e-4          # relative L2 of one cycle, as in the parity tests


def on_device(pb, stack=0):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    to = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(dev, t)  # noqa: E731
    mask = to(pb.mask, torch.uint8) if pb.mask is not None else None
    plan = P.Plan(pb.offsets, to(pb.iobs, torch.float32), mask, pb.wl.n_modes, pb.wl.obj_shape, stack=stack)
    return plan, to(pb.obj0, torch.complex64), to(pb.probe0, torch.complex64)


@pytest.mark.parametrize("n,k,j,stack", [(32, 1, 3, 0), (32, 2, 129, 0), (32, 3, 131, 130), (32, 4, 257, 0),
                                         (64, 1, 1, 0), (64, 2, 127, 0), (64, 3, 128, 0), (64, 4, 259, 129),
                                         (128, 1, 130, 0), (128, 2, 129, 0), (128, 1, 127, 0)])
def test_cycles_of_small_frames(n, k, j, stack):
    print(f"[gpu-case] frames n={n} k={k} j={j} stack={stack}", flush=True)
    step = 0.4 * n / np.sqrt(j)
    wl = small("dm256", n=n, k=k, j=j, obj=(2 * n + 5, 2 * n + 1), step=step, mask_frac=0.03)
    pb = make_problem(wl, start="ml")
    plan, o, p = on_device(pb, stack)
    host = lambda t: t.cpu().numpy()  # noqa: E731
    # model intensities and the likelihood's gradient
    ic = oracle.simulate_intensity(pb.obj0, pb.probe0, pb.offsets)
    assert rel_l2(host(plan.icalc(o, p)), ic) < TOL
    go, gp, llk = plan.ml_grad(o, p)
    ro, rp, rl = oracle.ml_grad(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask)
    assert rel_l2(host(go), ro) < TOL and rel_l2(host(gp), rp) < TOL
    assert abs(host(llk)[0] - rl) < TOL * abs(rl)
    # line search along the device's own negative gradient (up to 64 points: larger frames keep the three passes)
    if n <= 64:
        c = host(plan.ml_linesearch(o, p, -go, -gp))
        rc = oracle.linesearch_coefs(pb.obj0, pb.probe0, -host(go), -host(gp), pb.offsets, pb.iobs, pb.mask)
        assert abs(c[0] - rc[0]) < TOL * abs(rc[0]) and abs(c[1] - rc[1]) < TOL * abs(rc[1])
    # one CG, one AP and one DM cycle
    om, pm = o.clone(), p.clone()
    plan.ml_cycle(om, pm, plan.ml_state(), 1, UPD, reset=True)
    mo, mp = oracle.ml_cycle(pb.obj0, pb.probe0, oracle.CGState(), pb.offsets, pb.iobs, pb.mask, UPD)
    assert rel_l2(host(om), mo) < TOL and rel_l2(host(pm), mp) < TOL
    oa, pa = o.clone(), p.clone()
    plan.ap_cycle(oa, pa, 1, UPD)
    ao, ap = oracle.ap_cycle(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask)
    assert rel_l2(host(oa), ao) < TOL and rel_l2(host(pa), ap) < TOL
    psi = plan.psi_init(o, p)
    plan.dm_cycle(o, p, psi, 1, UPD)
    do, dp, dpsi = oracle.dm_cycle(pb.obj0, pb.probe0, oracle.psi_init(pb.obj0, pb.probe0, pb.offsets), pb.offsets,
                                   pb.iobs, pb.mask)
    assert rel_l2(host(o), do) < TOL and rel_l2(host(p), dp) < TOL and rel_l2(host(psi), dpsi) < TOL


@pytest.mark.parametrize("n,k", [(32, 2), (64, 3), (128, 1), (128, 2)])
def test_small_frames_on_sub_pixel_windows(n, k):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-case] frames, sub-pixel n={n} k={k}", flush=True)
    j = 133
    rng = np.random.default_rng(n + k)
    shape = (2 * n + 3, 2 * n + 8)
    pos = rng.uniform(-0.4 * n, 0.4 * n, (j, 2))
    offs, frac = oracle.windows_from_positions(pos, n, shape)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=shape, step=1.0, mask_frac=0.03), start="ml")
    iobs = oracle.simulate_intensity(pb.obj_true, pb.probe_true, offs, frac=frac).astype(np.float32)
    dev = torch.device("cuda:0")
    plan = P.Plan.with_positions(pos, torch.from_numpy(iobs).to(dev), torch.from_numpy(pb.mask).to(dev), k, shape)
    o = torch.from_numpy(pb.obj0.astype(np.complex64)).to(dev)
    p = torch.from_numpy(pb.probe0.astype(np.complex64)).to(dev)
    assert rel_l2(plan.icalc(o, p).cpu().numpy(), oracle.simulate_intensity(pb.obj0, pb.probe0, offs, frac=frac)) < TOL
    go, gp, _ = plan.ml_grad(o, p)
    ro, rp, _ = oracle.ml_grad(pb.obj0, pb.probe0, offs, iobs, pb.mask, frac=frac)
    assert rel_l2(go.cpu().numpy(), ro) < TOL and rel_l2(gp.cpu().numpy(), rp) < TOL
    if n <= 64:
        c = plan.ml_linesearch(o, p, -go, -gp).cpu().numpy()
        rc = oracle.linesearch_coefs(pb.obj0, pb.probe0, -go.cpu().numpy(), -gp.cpu().numpy(), offs, iobs, pb.mask,
                                     frac=frac)
        assert abs(c[0] - rc[0]) < TOL * abs(rc[0]) and abs(c[1] - rc[1]) < TOL * abs(rc[1])
    psi = plan.psi_init(o, p)
    plan.dm_cycle(o, p, psi, 1, UPD)
    do, dp, dpsi = oracle.dm_cycle(pb.obj0, pb.probe0, oracle.psi_init(pb.obj0, pb.probe0, offs, frac=frac), offs,
                                   iobs, pb.mask, frac=frac)
    assert rel_l2(o.cpu().numpy(), do) < TOL and rel_l2(p.cpu().numpy(), dp) < TOL
    assert rel_l2(psi.cpu().numpy(), dpsi) < TOL
