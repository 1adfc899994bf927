"""Backward products at the edges of their tiles and row chunks: the smallest window, windows that don't halve,
one and many chunks per window, dilations beyond the window, batches on both sides of the 512-block rules."""
import numpy as np
import pytest

from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("B,T,layer", [(1, 128, 29), (1, 384, 7), (3, 256, 8), (5, 640, 28), (2, 2048, 9), (65, 1024, 19),
                                       (513, 128, 3), (192, 1024, 9), (97, 2048, 28), (201, 1152, 5)])
def test_products_of_one_layer(prec, B, T, layer):
    """One layer's products in float64 from the operands its kernels read, within the forward-error bound
    of a dot product of length K, K u (|A| |B|), K the contraction length of the row products and the rows of the
    batch for the weight gradients (every order of a sum of K products meets it)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.arch import FULL, layout, unpack
    from oracle.quant import to_bf16
    from paper_2201_11133_amd import gwd, synth
    print(f"case: {prec} layer {layer}, B = {B}, T = {T}", flush=True)
    C, M, u32 = 128, B * T, 2.0 ** -24
    rng = np.random.default_rng(B + T)
    blob = synth.full_weights(4)
    p = unpack(FULL, blob.astype(np.float64))
    q = to_bf16 if prec == "bf16" else (lambda v: v)
    names = ("x_in", "pre", "dskip", "dx_in", "dg", "g", "dpre", "dx_out")
    bufs = {k: torch.empty((M, 2 * C if k in ("pre", "dpre") else C), dtype=torch.float32, device="cuda") for k in names}
    u = to_dev(rng.standard_normal((B, T, 2)).astype(np.float32))
    dz = to_dev(rng.standard_normal((B, T)).astype(np.float32))
    m = gwd.Model(gwd.full_arch(), blob, prec)
    m.capture_backward(layer, bufs)
    z = torch.empty((B, T), device="cuda")
    saved = torch.empty(gwd.lib.gwd_saved_bytes(m.h, B, T), dtype=torch.uint8, device="cuda")
    grad = torch.empty(m.n_params, device="cuda")
    st = gwd._stream_handle(None)
    gwd.check(gwd.lib.gwd_forward_train(m.h, 0, u.data_ptr(), B, T, z.data_ptr(), saved.data_ptr(), st))
    gwd.check(gwd.lib.gwd_backward(m.h, 0, u.data_ptr(), B, T, saved.data_ptr(), dz.data_ptr(), grad.data_ptr(), None, st))
    torch.cuda.synchronize()
    m.capture_backward(-1)
    m.close()
    cap = {k: v.cpu().numpy().astype(np.float64) for k, v in bufs.items()}
    gg, grads, o = grad.cpu().numpy().astype(np.float64), {}, 0
    for name, shape, _ in layout(FULL):
        n = int(np.prod(shape))
        grads[name] = gg[o:o + n].reshape(shape)
        o += n

    def check(label, got, A, Bm, K, plus=0.0):
        ref, bound = A @ Bm + plus, K * u32 * 1.01 * (np.abs(A) @ np.abs(Bm) + np.abs(plus))
        assert np.all(np.abs(got - ref) <= bound), (label, float(np.max(np.abs(got - ref) / (bound + 1e-300))))

    last = layer == FULL.n_layers - 1
    ds, dxi, x, dp, gt = cap["dskip"], cap["dx_in"], cap["x_in"], cap["dpre"], cap["g"]
    A, W = q(ds), q(p[f"skip{layer}.W"])
    if not last:
        A, W = np.hstack([A, q(dxi)]), np.vstack([W, q(p[f"res{layer}.W"])])
    check("dg", cap["dg"], A, W, W.shape[0])
    check("d skip.W", grads[f"skip{layer}.W"], q(ds).T, gt, M)
    one = np.ones((M, 1))
    check("d skip.b", grads[f"skip{layer}.b"][:, None], ds.T, one, M)
    check("d dil.b", grads[f"dil{layer}.b"][:, None], dp.T, one, M)
    if not last:
        check("d res.W", grads[f"res{layer}.W"], q(dxi).T, gt, M)
        check("d res.b", grads[f"res{layer}.b"][:, None], dxi.T, one, M)
    d = FULL.dilation(layer)
    xd, dpd = np.zeros((B, T, C)), np.zeros((B, T, 2 * C))
    if d < T:
        xd[:, d:] = x.reshape(B, T, C)[:, :-d]
        dpd[:, :-d] = dp.reshape(B, T, 2 * C)[:, d:]
    check("d dil.W tap 1", grads[f"dil{layer}.W"][:, :, 1], dp.T, x, M)
    check("d dil.W tap 0", grads[f"dil{layer}.W"][:, :, 0], dp.T, xd.reshape(M, C), M)
    W1, W0 = q(p[f"dil{layer}.W"][:, :, 1]), q(p[f"dil{layer}.W"][:, :, 0])
    check("dx", cap["dx_out"], np.hstack([dp, dpd.reshape(M, 2 * C)]), np.vstack([W1, W0]), 4 * C + 1, dxi)
    check("d h2.b", grads["h2.b"].reshape(1, 1), dz.cpu().numpy().astype(np.float64).reshape(1, M), one, M)
