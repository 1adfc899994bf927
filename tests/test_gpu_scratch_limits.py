"""Calls whose larger scratch does not fit the device memory that is free run in the smaller one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MB = 1 << 20


@pytest.fixture
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd
    return gwd


class Ballast:
    """Leaves about `free` bytes of device memory (the amount that is reported free may lag)."""

    def __init__(self, free):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        self.t = []
        for _ in range(6):
            more = torch.cuda.mem_get_info()[0] - free
            if more > 2 * MB:
                self.t.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
        print(f"free: {torch.cuda.mem_get_info()[0] / MB:.0f} MiB of {free / MB:.0f} asked", flush=True)

    def __enter__(self):
        return self

    def __exit__(self, *a):
        del self.t
        torch.cuda.empty_cache()


def gradients(g, m, u, dz, z, saved, grad, du):
    st = g._stream_handle(None)
    B, T = u.shape[0], u.shape[1]
    g.check(g.lib.gwd_backward(m.h, 0, u.data_ptr(), B, T, saved.data_ptr(), dz.data_ptr(), grad.data_ptr(),
                               du.data_ptr(), st))
    torch.cuda.synchronize()
    return grad.clone(), du.clone()


@pytest.mark.parametrize("arch,prec,B,T,free_mb", [("tiny", "fp32", 512, 4096, 400), ("tiny", "fp64", 300, 2000, 240),
                                                   ("full", "fp32", 8, 4096, 0), ("full", "bf16", 8, 4096, 0)])
def test_backward(g, arch, prec, B, T, free_mb):
    """The small member's scratch for dL/dpre of all windows (512 windows of 4,096: 512 MiB) in parts, with the
    same gradients bit for bit; the gated member's weight-gradient partials one chunk per window (18 MiB less
    than with split windows, 9 MiB of it free), gradients within 1e-5 of their norm (FP32 sums in another
    order). A second call stays in the smaller scratch."""
    from paper_2201_11133_amd import synth
    print(f"case: {arch} {prec} B={B} T={T}", flush=True)
    dt = torch.float64 if prec == "fp64" else torch.float32
    blob = synth.tiny_weights(5) if arch == "tiny" else synth.full_weights(5)
    make = g.tiny_arch if arch == "tiny" else g.full_arch
    gen = torch.Generator(device="cuda").manual_seed(7)
    u = torch.randn((B, T, 2), generator=gen, device="cuda")
    dz = torch.randn((B, T), generator=gen, device="cuda", dtype=dt)
    z, du = torch.empty((B, T), dtype=dt, device="cuda"), torch.empty((B, T, 2), dtype=dt, device="cuda")
    res = []
    for limited in (False, True):
        m = g.Model(make(), blob, prec)
        saved = torch.empty(g.lib.gwd_saved_bytes(m.h, B, T), dtype=torch.uint8, device="cuda")
        grad = torch.empty(m.n_params, dtype=dt, device="cuda")
        g.check(g.lib.gwd_forward_train(m.h, 0, u.data_ptr(), B, T, z.data_ptr(), saved.data_ptr(), g._stream_handle(None)))
        if not limited:
            before = torch.cuda.mem_get_info()[0]
            res.append(gradients(g, m, u, dz, z, saved, grad, du))
            took = before - torch.cuda.mem_get_info()[0]
            # (partials: 72 chunks of 256 KB with one chunk per window, 144 with split ones)
            free = (free_mb * MB) if free_mb else took - 9 * MB
        else:
            with Ballast(free):
                for _ in range(2):
                    res.append(gradients(g, m, u, dz, z, saved, grad, du))
        m.close()
    (g0, d0), (g1, d1), (g2, d2) = res
    assert torch.equal(g1, g2) and torch.equal(d1, d2)
    if arch == "tiny":
        assert torch.equal(g0, g1) and torch.equal(d0, d1)
    else:
        assert torch.linalg.norm(g0 - g1) <= 1e-5 * torch.linalg.norm(g0)
        assert torch.equal(d0, d1)


@pytest.mark.parametrize("capacity", [None, 1000, 0])
def test_peak_search(g, capacity):
    """2^25 samples in 400 MiB (the list of kept peaks takes 512 MiB with the rest): the peaks and widths of a
    call with all the memory."""
    print(f"case: capacity {capacity}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.rand(1 << 25, generator=gen, device="cuda", dtype=torch.float64)
    cut = x[: 1 << 16].clone()     # (a short call in the same buffer afterwards)
    short = g.find_peaks(cut, 0.9, 2.0)
    with Ballast(400 * MB):
        if capacity is None:
            got = [g.find_peaks(x, 0.9, 2.0) for _ in range(2)]
        else:
            with pytest.raises(g.GwdError):
                g.find_peaks(x, 0.9, 2.0, capacity=capacity)
            got = []
        again = g.find_peaks(cut, 0.9, 2.0)
    want = g.find_peaks(x, 0.9, 2.0)
    assert len(want[0]) > 1000 and all(np.array_equal(a, b) for a, b in zip(short, again))
    for p, w in got:
        assert np.array_equal(p, want[0]) and np.array_equal(w, want[1])
