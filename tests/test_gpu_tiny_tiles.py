"""The small member's one-kernel passes at the edges of their tiles (242 forward rows, 240 backward)."""
import numpy as np
import pytest

from tests.gpu_common import FP32_P_TOL, sigmoid64, to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd
    return gwd


@pytest.mark.parametrize("T,B", [(1, 3), (7, 2), (8, 1), (239, 2), (240, 1), (241, 2), (242, 1), (243, 2), (248, 1),
                                 (480, 1), (485, 900)])
def test_gradient_at_tile_edges(g, T, B):
    """FP64 gradients equal the oracle's to 1e-10 (the bound of the existing gradient test); FP32 ones to
    1e-5 in norm. 900 windows: several tiles per block."""
    from oracle.arch import TINY
    from oracle.train import bce_grad, loss_and_grad
    from paper_2201_11133_amd import synth
    from tests.test_gpu_train import backward, fwd_train
    print(f"case: B={B} T={T}", flush=True)
    blob = synth.tiny_weights(5)
    u = np.random.default_rng(T).standard_normal((B, T, 2)).astype(np.float32)
    y = (np.random.default_rng(T + 1).random((B, T)) < 0.3).astype(np.float64)
    _, g_ref, du_ref = loss_and_grad(TINY, blob.astype(np.float64), u.astype(np.float64), y)
    for prec, dt in (("fp64", torch.float64), ("fp32", torch.float32)):
        m = g.Model(g.tiny_arch(), blob, prec)
        z, saved = fwd_train(g, m, to_dev(u), B, T, dt)
        dz = torch.from_numpy(bce_grad(z.cpu().numpy().astype(np.float64), y)).to(dt).cuda()
        grad, du = backward(g, m, to_dev(u), B, T, saved, dz, dt)
        gg, dd = grad.cpu().numpy().astype(np.float64), du.cpu().numpy().astype(np.float64)
        if prec == "fp64":
            assert np.max(np.abs(gg - g_ref)) <= 1e-12 + 1e-10 * np.max(np.abs(g_ref))
            assert np.max(np.abs(dd - du_ref)) <= 1e-12 + 1e-10 * np.max(np.abs(du_ref))
        else:
            assert np.linalg.norm(gg - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
            assert np.linalg.norm(dd - du_ref) <= 1e-5 * np.linalg.norm(du_ref)
        m.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("W,S", [(256, 241), (256, 100), (512, 256), (4096, 256), (4096, 4081)])
def test_forward_tiles(g, prec, W, S):
    """Stitched scores, whose tiles start at the first owned row, equal the rows of the per-window
    logits bit for bit; in FP32 both match the oracle within its probability bound."""
    from oracle.arch import TINY, unpack
    from oracle.forward import forward_stream
    from paper_2201_11133_amd import synth
    print(f"case: {prec} W={W} S={S}", flush=True)
    blob = synth.tiny_weights(6)
    m = g.Model(g.tiny_arch(), blob, prec)
    xs = [np.random.default_rng(70 + i).standard_normal((L, 2)).astype(np.float32) for i, L in enumerate((1, 242, 256, 5003))]
    e = m.forward([to_dev(x) for x in xs], W, S, 0).cpu().numpy()
    per = m.forward([to_dev(x) for x in xs], W, S, 2).cpu().numpy().reshape(-1, W)
    at, wb = 0, 0
    for x in xs:
        L = len(x)
        nw = 1 if L <= W else -(-(L - W) // S) + 1
        a = np.arange(L)
        k = np.where(a < W - S, 0, (a - W + S) // S)
        assert np.array_equal(e[at: at + L], per[wb + k, a - k * S])
        if prec == "fp32":
            ref = forward_stream(TINY, unpack(TINY, blob.astype(np.float64)), x.astype(np.float64))
            assert np.max(np.abs(sigmoid64(e[at: at + L]) - sigmoid64(ref))) <= FP32_P_TOL
        at += L
        wb += nw
    m.close()
