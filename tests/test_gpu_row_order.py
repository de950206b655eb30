"""The row passes whose blocks take the same rows of several frames: frame
counts around the groups of four and eight, a last group of one frame, several
stacks, at the sizes that use the order and the forms of each pass."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
UPD = oracle.UPDATE_OBJECT | oracle.UPDATE_PROBE
TOL = 1e-4          # relative L2 of one cycle, as in the parity tests


@pytest.mark.parametrize("n,k,j,stack", [(256, 1, 9, 0), (256, 2, 11, 5),
                                         (512, 4, 1, 0), (512, 4, 9, 0), (512, 1, 13, 0), (512, 4, 7, 5),
                                         (1024, 1, 5, 0), (1024, 2, 3, 2)])
def test_cycles_match_the_oracle(n, k, j, stack):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    shape = (n + 45, n + 61)
    pb = make_problem(small("ml256", n=n, k=k, j=j, obj=shape, step=20.0 / np.sqrt(j), mask_frac=0.03), start="ml")
    to = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(dev, t)  # noqa: E731
    host = lambda t: t.cpu().numpy()  # noqa: E731
    plan = P.Plan(pb.offsets, to(pb.iobs, torch.float32), to(pb.mask, torch.uint8), k, shape, stack=stack)
    for form in ("ap", "dm", "ml"):
        print(f"[gpu-case] row order {form} n={n} k={k} j={j} stack={stack}", flush=True)
        o, p = to(pb.obj0, torch.complex64), to(pb.probe0, torch.complex64)
        if form == "ap":
            plan.ap_cycle(o, p, 1, UPD)
            ro, rp = oracle.ap_cycle(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask)
        elif form == "dm":
            psi = plan.psi_init(o, p)
            plan.dm_cycle(o, p, psi, 1, UPD)
            psi0 = oracle.psi_init(pb.obj0, pb.probe0, pb.offsets)
            ro, rp, rpsi = oracle.dm_cycle(pb.obj0, pb.probe0, psi0, pb.offsets, pb.iobs, pb.mask, UPD)
            assert rel_l2(host(psi), rpsi) < TOL
        else:
            plan.ml_cycle(o, p, plan.ml_state(), 1, UPD, reset=True)
            ro, rp = oracle.ml_cycle(pb.obj0, pb.probe0, oracle.CGState(), pb.offsets, pb.iobs, pb.mask, UPD)
        assert rel_l2(host(o), ro) < TOL and rel_l2(host(p), rp) < TOL
