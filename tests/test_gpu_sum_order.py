"""How the gradient's probe sums are split: the running sums in 32 bits are as
short as the probe gather's, and plans on integer windows and on positions
whose corners are integers add the same chunks in the same order."""
import numpy as np
import pytest

import oracle
from cases import make_problem, rel_l2, small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def problem(n, k, j, shape, seed, dev):
    """Object, probe, intensities of j frames around the object's centre, drawn on the host."""
    r = np.random.default_rng(seed)
    obj = (0.8 + 0.2 * r.random(shape)) * np.exp(1j * r.random(shape))
    probe = (1.0 + r.random((k, n, n))) * np.exp(1j * r.random((k, n, n)))
    iobs = torch.from_numpy((2.0 * k + r.random((j, n, n), dtype=np.float32) * 5.0)).to(dev, torch.float32)
    return (torch.from_numpy(obj.astype(np.complex64)).to(dev), torch.from_numpy(probe.astype(np.complex64)).to(dev),
            iobs)


@pytest.mark.parametrize("n,k,j,chunks", [(256, 3, 1000, 16), (512, 4, 240, 4), (128, 3, 640, 32)])
def test_probe_gradient_runs_are_no_longer_than_the_gather_s(n, k, j, chunks):
    """All frames alike: the sum's only error is that of its running sums, against j times one frame's term.  Its rms
    grows with the frames of a run (7.7 units of the last place at 62 frames, 15.4 at 125), so 1.5 times that of a run
    of j / chunks frames, emulated here, tells a run from one of twice the length."""
    import paper_2008_11511_amd as P
    dev = device()
    print(f"[gpu-case] run length n={n} k={k} j={j}", flush=True)
    shape = (n + 9, n + 14)
    obj, probe, one = problem(n, k, 1, shape, n + k, dev)
    offs = np.full((j, 2), 4, np.int32)
    term = P.Plan(offs[:1], one, None, k, shape).ml_grad(obj, probe)[1].cpu().numpy().view(np.float32)
    plan = P.Plan(offs, one.expand(j, n, n).contiguous(), None, k, shape)
    got = plan.ml_grad(obj, probe)[1].cpu().numpy().view(np.float32)
    run = np.zeros_like(term)
    length = -(-j // chunks)
    for _ in range(length):
        run = run + term
    rms = lambda s, m: float(np.sqrt(np.mean((s / (m * term.astype(np.float64)) - 1.0) ** 2)))  # noqa: E731
    assert rms(got, j) < 1.5 * rms(run, length)


@pytest.mark.parametrize("n,k,j,stack", [(128, 3, 30, 0),       # fewer frames than chunks, two frames a block
                                         (128, 1, 67, 0), (128, 2, 140, 0), (128, 3, 16, 0), (128, 3, 41, 20),
                                         (256, 1, 40, 0), (256, 3, 16, 0), (512, 1, 16, 0), (512, 4, 9, 0),
                                         (1024, 1, 26, 0),      # four groups of three chunks
                                         (1024, 2, 13, 7), (2048, 1, 7, 0)])
def test_integer_positions_give_the_integer_plan_s_gradient_bitwise(n, k, j, stack):
    """The probe's gradient and the LLK at every size; up to 16 frames, where no object tile's frames are split into
    chunks (a positions plan counts frames that may move onto a tile, so its chunks begin elsewhere), all of it."""
    import paper_2008_11511_amd as P
    dev = device()
    shape = (n + 45, n + 61)
    obj, probe, iobs = problem(n, k, j, shape, n * k + j, dev)
    offs = np.random.default_rng(j).integers(2, 40, (j, 2)).astype(np.int32)
    pos = offs + n / 2.0 - np.array(shape) / 2.0
    both = P.UPDATE_OBJECT | P.UPDATE_PROBE
    a = P.Plan(offs, iobs, None, k, shape, stack=stack)
    b = P.Plan.with_positions(pos, iobs, None, k, shape, max_shift=1.0, stack=stack)

    def outputs(plan, update):
        print(f"[gpu-case] sum order n={n} k={k} j={j} stack={stack} update={update}", flush=True)
        g_o, g_p, llk = plan.ml_grad(obj, probe)
        o, p, st = obj.clone(), probe.clone(), plan.ml_state()
        plan.ml_cycle(o, p, st, 1, update, reset=True)
        return [x.cpu().numpy() for x in ((g_p, llk, g_o, o, p) if j <= 16 else (g_p, llk))]

    ref = outputs(a, both)
    # the last call moves b's positions after its cycle, so it comes last
    for update in (both, both | P.UPDATE_POSITIONS):
        for x, y in zip(ref, outputs(b, update)):
            np.testing.assert_array_equal(x, y)


def test_gradient_of_several_hundred_frames_matches_the_oracle():
    """Chunks of 19 frames, two to a block."""
    import paper_2008_11511_amd as P
    dev = device()
    print("[gpu-case] long chunks n=256 k=3 j=304", flush=True)
    pb = make_problem(small("ml256", n=256, k=3, j=304, obj=(420, 433), step=4.0, mask_frac=0.03), start="ml")
    to = lambda a, t: torch.from_numpy(np.ascontiguousarray(a)).to(dev, t)  # noqa: E731
    plan = P.Plan(pb.offsets, to(pb.iobs, torch.float32), to(pb.mask, torch.uint8), 3, pb.wl.obj_shape)
    go, gp, llk = plan.ml_grad(to(pb.obj0, torch.complex64), to(pb.probe0, torch.complex64))
    ro, rp, rl = oracle.ml_grad(pb.obj0, pb.probe0, pb.offsets, pb.iobs, pb.mask)
    # relative L2, as in the parity tests
    assert rel_l2(go.cpu().numpy(), ro) < 1e-4 and rel_l2(gp.cpu().numpy(), rp) < 1e-4
    assert abs(llk.cpu().numpy()[0] - rl) < 1e-4 * abs(rl)
