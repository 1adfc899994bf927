"""Whitening at the sizes where the transforms change form: 128 / 256 points (LDS or registers), one or
several columns per workgroup, rows in pairs up to 2^13 points, and the largest streams."""
import math

import pytest

from tests.test_gpu_whiten import ETA, FS, U, g, run_case  # noqa: F401  (g: the fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("logl,n", [(14, 64), (15, 128), (16, 256), (17, 2048), (18, 512), (19, 8192), (21, 16384),
                                    (22, 32)])
def test_sizes(g, logl, n):  # noqa: F811
    from paper_2201_11133_amd.synth import coloured_stream
    print(f"case: whiten L=2^{logl} n={n}", flush=True)
    run_case(g, coloured_stream(400 + logl, 1 << logl), n, planar=logl % 2 == 1)


@pytest.mark.parametrize("logl", [26, 27, 28])
def test_largest(g, logl):  # noqa: F811
    """Rows and columns of 2^13 and 2^14 points, against torch's float64 transforms, within the whitening
    bound (see test_gpu_whiten)."""
    print(f"case: whiten L=2^{logl}", flush=True)
    L, n = 1 << logl, 4096
    x = torch.randn((L, 2), generator=torch.Generator(device="cuda").manual_seed(logl), device="cuda")
    psd = g.welch_psd(x, n, FS)
    raw = g.whiten(x, psd, n, FS, False)
    k = torch.arange(L // 2 + 1, device="cuda") * n
    j, fr = k // L, (k % L).double() / L
    err = bound_x = yn = amax = 0.0
    for c in range(2):
        p = psd[c]
        coef = 1 / torch.sqrt((p[j] * (1 - fr) + p[torch.clamp(j + 1, max=n // 2)] * fr) * FS / 2)
        y = torch.fft.irfft(torch.fft.rfft(x[:, c].double()) * coef, n=L)
        amax = max(amax, float(coef.max()))
        err += float((raw[:, c].double() - y).square().sum())
        yn += float(y.square().sum())
        bound_x += float(x[:, c].double().square().sum())
        del y, coef
    bound = amax * (logl + 2) * ETA * math.sqrt(bound_x) + ((logl + 2) * ETA + 4 * U) * math.sqrt(yn)
    assert math.sqrt(err) <= bound, (math.sqrt(err), bound)
