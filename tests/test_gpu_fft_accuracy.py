"""Rounding of the 2D transform where its output is weak: an exit wave's
detector field spans many decades, and what a loss or a modulus divides by is
the weak part of it, which a norm over the whole field does not see."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# rms error over the weaker half of the field, relative to that half's rms, of
# a transform in 32 bits that multiplies each butterfly input by its twiddle
# first and then adds and subtracts (emulated on the waves below)
PRODUCT_FIRST = {64: 2.908e-06, 128: 3.131e-06, 256: 3.468e-06, 512: 3.726e-06}


def waves(n, count):
    """Exit waves: Gaussian probes of a curved phase on objects of smooth phase."""
    r = np.random.default_rng(n)
    c = np.arange(n) - n / 2.0
    y, x = np.meshgrid(c, c, indexing="ij")
    s = 20.0 * n / 64.0 / (2.0 * np.sqrt(2.0 * np.log(2.0)))
    r2 = x * x + y * y
    out = []
    for _ in range(count):
        phase = 0.5 * np.pi * r2 / (n / 2.0) ** 2
        for _ in range(12):
            f = r.uniform(-0.05, 0.05, 2)
            phase = phase + 0.2 * np.cos(2.0 * np.pi * (f[0] * y + f[1] * x) + r.uniform(0.0, 2.0 * np.pi))
        out.append(np.exp(-r2 / (2.0 * s * s)) * (0.8 + 0.2 * r.random((n, n))) * np.exp(1j * phase))
    return np.array(out).astype(np.complex64)


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("n", sorted(PRODUCT_FIRST))
def test_weak_outputs_are_rounded_at_their_own_size(n, inverse):
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-case] transform accuracy n={n} inverse={inverse}", flush=True)
    w = waves(n, max(1, min(24, 2 ** 20 // (n * n))))
    ref = (np.fft.ifft2 if inverse else np.fft.fft2)(w.astype(np.complex128), norm="ortho")
    err = np.abs(P.fft2(torch.from_numpy(w).to("cuda:0"), inverse).cpu().numpy() - ref)
    weak = np.abs(ref) < np.median(np.abs(ref))
    # differences formed as twice an input minus the sum are 1.10 to 1.18 times off
    assert np.sqrt(np.mean(err[weak] ** 2) / np.mean(np.abs(ref[weak]) ** 2)) < 1.05 * PRODUCT_FIRST[n]


def test_an_infinite_input_reaches_every_output():
    """One butterfly deep (8 points): sums and differences with an infinity are infinite, not undefined."""
    import paper_2008_11511_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[gpu-case] transform of an infinity n=8", flush=True)
    w = torch.zeros((1, 8, 8), dtype=torch.complex64)
    w[0, 0, 0] = complex(float("inf"), 0.0)
    got = P.fft2(w.to("cuda:0")).cpu().numpy()
    assert np.all(np.isposinf(got.real))
