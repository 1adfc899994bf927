"""The BF16/FP8 gate where its exponentials leave the range of fp32: the filter's underflows, the gate's overflows,
alone and together, in the single-layer and the fused kernels."""
import numpy as np
import pytest

from tests.gpu_common import to_dev
from tests.test_gpu_lowp import check_layer

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (filter, gate) pre-activations: e^(-2|a|) underflows from |a| = 43.7 on, e^-b overflows from b = -88.7 on
EDGES = [(60, -100), (-60, -100), (44, -89), (-44, -88.5), (43, -90), (1e4, -1e4), (20, -100), (0, -100), (0.5, -1e4),
         (60, -80), (60, 100), (-1e4, 1e4), (3e38, -3e38), (0.5, 0.25), (-2, 1), (60, -87)]


def edge_model(g, prec, per_launch):
    from oracle.arch import FULL, layout, unpack
    from paper_2201_11133_amd import synth
    blob, o = synth.full_weights(4), 0
    pairs = np.resize(np.array(EDGES, dtype=np.float32), (128, 2))
    for name, shape, _ in layout(FULL):
        if name.startswith("dil"):   # the bias alone: an exact pre-activation
            blob[o:o + int(np.prod(shape))] = np.concatenate([pairs[:, 0], pairs[:, 1]]) if name.endswith(".b") else 0
        o += int(np.prod(shape))
    m = g.Model(g.full_arch(), blob, prec)
    m.set_tiling(0, 0, 512, per_launch)
    return m, unpack(FULL, blob.astype(np.float64))


@pytest.mark.parametrize("prec", ["bf16", "fp8"])
@pytest.mark.parametrize("first,per_launch", [(0, 6), (26, 6), (10, 3), (5, 1)])
def test_gate_at_the_ends_of_its_range(prec, first, per_launch):
    """Every layer of the launch against the oracle, within the bounds of the ordinary layer test; a NaN in
    the residual stream stays one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd
    print(f"case: {prec} launch at layer {first}, {per_launch} layers per launch", flush=True)
    m, p = edge_model(gwd, prec, per_launch)
    T, C = 4096, 128
    x = np.zeros((1, T, C), dtype=np.float32)
    sk = np.random.default_rng(first).standard_normal((1, T, C)).astype(np.float32)
    nan_row = 1000
    for bad in (False, True):
        if bad:
            x[0, nan_row] = np.nan
        if per_launch == 1:
            nl, xd, skd = 1, to_dev(x), to_dev(sk.copy())
            pre, xo = torch.empty((T, 2 * C), device="cuda"), torch.zeros((T, C), device="cuda")
            m.debug_layer(0, first, xd, 1, T, pre, xo, skd)
            so = skd
        else:
            nl = m.fused_layers(first, T)
            pre, xo, so = m.debug_fused(0, first, to_dev(x), 1, T, to_dev(sk.copy()))
        torch.cuda.synchronize()
        pre = pre.cpu().numpy().astype(np.float64).reshape(nl, 1, T, 2 * C)
        xo = xo.cpu().numpy().astype(np.float64).reshape(nl, 1, T, C)
        so = so.cpu().numpy().astype(np.float64).reshape(nl, 1, T, C)
        if bad:
            stays = first + nl < 30   # (the network's last layer has no residual output)
            assert np.isnan(xo[: nl if stays else nl - 1, 0, nan_row]).all()
            if prec == "bf16":        # (the E4M3 operand of a NaN is the format's largest value)
                assert np.isnan(pre[:, 0, nan_row]).all() and np.isnan(so[:, 0, nan_row]).all()
            continue
        xb, skip_in = x.astype(np.float64), None if first == 0 else sk.astype(np.float64)
        for j in range(nl):
            assert np.isfinite(xo[j]).all() and np.isfinite(so[j]).all()
            check_layer(prec, p, first + j, xb, skip_in, pre[j], xo[j], so[j], f"layer {first + j}")
            xb, skip_in = xo[j], so[j]
    m.close()
