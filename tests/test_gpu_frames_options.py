"""The options of the one-kernel path of small frames, at frame counts that
take it (128 on): a background in the intensities and the gradient, AP's
background refinement, and position updates from the projected waves and from
the gradient waves that the kernel leaves in the scratch, with the modes side
by side (32 and 64 points) and one after the other (128)."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
UPD = oracle.UPDATE_OBJECT | oracle.UPDATE_PROBE
TOL = 1e-4          # relative, as in the parity tests
SIZES = [(32, 4), (64, 3), (128, 1), (128, 2)]


def on_device(a, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", dtype)


def host(t):
    return t.cpu().numpy()


@pytest.mark.parametrize("n,k", SIZES)
def test_background(n, k):
    import paper_2008_11511_amd as P
    j = 130
    print(f"[gpu-case] frames with a background n={n} k={k} j={j}", flush=True)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=(2 * n + 5, 2 * n + 1), step=0.4 * n / np.sqrt(j),
                            mask_frac=0.03), start="ml", bg_level=5.0)
    plan = P.Plan(pb.offsets, on_device(pb.iobs, torch.float32), on_device(pb.mask, torch.uint8), k, pb.wl.obj_shape,
                  background_update=True)
    bg = on_device(pb.bg0, torch.float32)
    plan.set_background(bg)
    o, p = on_device(pb.obj0, torch.complex64), on_device(pb.probe0, torch.complex64)
    assert rel_l2(host(plan.icalc(o, p)), oracle.simulate_intensity(pb.obj0, pb.probe0, pb.offsets, bg=pb.bg0)) < TOL
    go, gp, llk = plan.ml_grad(o, p)
    ro, rp, rl = oracle.ml_grad(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask, bg=pb.bg0)
    assert rel_l2(host(go), ro) < TOL and rel_l2(host(gp), rp) < TOL and abs(host(llk)[0] - rl) < TOL * abs(rl)
    od, pd = o.clone(), p.clone()
    psi = plan.psi_init(od, pd)
    plan.dm_cycle(od, pd, psi, 1, UPD)
    ro, rp, rpsi = oracle.dm_cycle(pb.obj0, pb.probe0, oracle.psi_init(pb.obj0, pb.probe0, pb.offsets), pb.offsets,
                                   pb.iobs, pb.mask, bg=pb.bg0)
    assert rel_l2(host(od), ro) < TOL and rel_l2(host(pd), rp) < TOL and rel_l2(host(psi), rpsi) < TOL
    assert np.array_equal(host(bg), pb.bg0)             # read only so far
    plan.ap_cycle(o, p, 1, UPD | P.UPDATE_BACKGROUND)
    ro, rp, rb = oracle.ap_cycle(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask, UPD | oracle.UPDATE_BACKGROUND,
                                 bg=pb.bg0)
    assert rel_l2(host(o), ro) < TOL and rel_l2(host(p), rp) < TOL and rel_l2(host(bg), rb) < TOL


@pytest.mark.parametrize("form", ["ap", "ml"])
@pytest.mark.parametrize("n,k", SIZES)
def test_position_updates(n, k, form):
    import paper_2008_11511_amd as P
    j, shape = 133, (2 * n + 13, 2 * n + 18)
    print(f"[gpu-case] frames with position updates n={n} k={k} j={j} {form}", flush=True)
    rng = np.random.default_rng(n + k)
    pb = make_problem(small("dm256", n=n, k=k, j=j, obj=shape, step=1.0, mask_frac=0.03), start="ml")
    true = rng.uniform(-0.4 * n, 0.4 * n, (j, 2))
    offs, frac = oracle.windows_from_positions(true, n, shape)
    iobs = oracle.simulate_intensity(pb.obj_true, pb.probe_true, offs, frac=frac).astype(np.float32)
    pos0 = true + rng.choice([-0.3, 0.3], size=(j, 2))
    offs, frac = oracle.windows_from_positions(pos0, n, shape)
    plan = P.Plan.with_positions(pos0, on_device(iobs, torch.float32), on_device(pb.mask, torch.uint8), k, shape)
    o, p = on_device(pb.obj0, torch.complex64), on_device(pb.probe0, torch.complex64)
    if form == "ap":
        plan.ap_cycle(o, p, 1, UPD | P.UPDATE_POSITIONS)
        psi = oracle.fourier_project(oracle.exit_waves(pb.obj0, pb.probe0, offs, frac), iobs, pb.mask)
        ro, rp = oracle.overlap_update(pb.obj0, pb.probe0, psi, offs, UPD, frac=frac)
        sh, e = oracle.position_shifts(ro, rp, psi, offs, frac)
    else:
        plan.ml_cycle(o, p, plan.ml_state(), 1, UPD | P.UPDATE_POSITIONS, reset=True)
        sh, e = oracle.ml_position_shifts(pb.obj0, pb.probe0, offs, iobs, pb.mask, frac=frac)
        ro, rp = oracle.ml_cycle(pb.obj0, pb.probe0, oracle.CGState(), offs, iobs, pb.mask, update=UPD, frac=frac)
    pos = oracle.update_positions(pos0, pos0, sh, e)
    assert np.abs(pos - pos0).max() > 0.02                   # they move
    assert np.abs(host(plan.positions()) - pos).max() < 1e-3
    assert rel_l2(host(o), ro) < TOL and rel_l2(host(p), rp) < TOL
