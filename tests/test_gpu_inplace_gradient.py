"""grad_input written over the windows, the logit gradient or the saved activations of the same call."""
import numpy as np
import pytest

from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("arch,prec", [("tiny", "fp32"), ("tiny", "fp64"), ("full", "fp32"), ("full", "bf16")])
@pytest.mark.parametrize("over", ["windows", "grad_logit", "saved"])
def test_gradient_over_its_inputs(arch, prec, over):
    """Weight and input gradients equal those of separate buffers, bit for bit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    if prec == "fp64" and over == "windows":
        pytest.skip("float32 windows do not hold a float64 gradient")
    print(f"case: {arch} {prec} over {over}", flush=True)
    B, T = (9, 1001) if arch == "tiny" else (2, 384)
    dt = torch.float64 if prec == "fp64" else torch.float32
    blob = synth.tiny_weights(5) if arch == "tiny" else synth.full_weights(5)
    m = gwd.Model(gwd.tiny_arch() if arch == "tiny" else gwd.full_arch(), blob, prec)
    u = to_dev(np.random.default_rng(1).standard_normal((B, T, 2)).astype(np.float32))
    # the logit gradient starts a buffer that also has room for the input gradient
    room = torch.empty(2 * B * T, dtype=dt, device="cuda")
    dz = torch.from_numpy(np.random.default_rng(2).standard_normal(B * T)).to(dt).cuda()
    z = torch.empty((B, T), dtype=dt, device="cuda")
    saved = torch.empty(gwd.lib.gwd_saved_bytes(m.h, B, T), dtype=torch.uint8, device="cuda")
    st = gwd._stream_handle(None)
    res = []
    for place in (None, over):
        room[: B * T] = dz
        gwd.check(gwd.lib.gwd_forward_train(m.h, 0, u.data_ptr(), B, T, z.data_ptr(), saved.data_ptr(), st))
        du = {None: torch.empty((B, T, 2), dtype=dt, device="cuda"), "windows": u, "grad_logit": room, "saved": saved}[place]
        grad = torch.empty(m.n_params, dtype=dt, device="cuda")
        gwd.check(gwd.lib.gwd_backward(m.h, 0, u.data_ptr(), B, T, saved.data_ptr(), room.data_ptr(), grad.data_ptr(),
                                       du.data_ptr(), st))
        torch.cuda.synchronize()
        res.append((grad, du.reshape(-1).view(dt)[: 2 * B * T].clone()))
    m.close()
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
