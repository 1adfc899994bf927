"""E4M3 operands of the residual stream beyond the format's range: both signs, around 448 and far above it, in the
fused launches (staged rows and the rows each layer hands to the next)."""
import numpy as np
import pytest

from tests.gpu_common import to_dev
from tests.test_gpu_lowp import check_layer

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("first,per_launch", [(0, 6), (10, 3), (26, 6)])
def test_residual_rows_beyond_448(first, per_launch):
    """Layer by layer against the oracle's quantiser (which saturates), within the bounds of the ordinary
    layer test: they scale with the operands' magnitudes. Conv weights of 1/32 the usual size keep the
    pre-activations in the gate's range (NaN where the filter's exponential underflows and the gate's
    overflows: |a_f| > 43 with a_g < -88)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle.arch import FULL, layout, unpack
    from oracle.quant import to_bf16
    from paper_2201_11133_amd import gwd, synth
    print(f"case: launch at layer {first}, {per_launch} layers per launch", flush=True)
    blob, o = synth.full_weights(4), 0
    for name, shape, _ in layout(FULL):
        if name.startswith("dil") and name.endswith(".W"):
            blob[o:o + int(np.prod(shape))] /= 32
        o += int(np.prod(shape))
    m = gwd.Model(gwd.full_arch(), blob, "fp8")
    T, nw, C = 4096, 1, 128
    m.set_tiling(0, 0, 512, per_launch)
    nl = m.fused_layers(first, T)
    p = unpack(FULL, blob.astype(np.float64))
    rng = np.random.default_rng(first)
    x = (rng.choice([-1.0, 1.0], (nw, T, C)) * 2.0 ** rng.uniform(-10, 13, (nw, T, C))).astype(np.float32)
    edge = np.array([446.0, 448.0, 450.0, 456.0, 464.0, 480.0, 1.0e4, 0.0], dtype=np.float32)
    x[0, 100:108, 0] = edge
    x[0, 110:118, 1] = -edge
    sk = rng.standard_normal((nw, T, C)).astype(np.float32)
    pre, xo, so = m.debug_fused(0, first, to_dev(x), nw, T, to_dev(sk.copy()))
    torch.cuda.synchronize()
    m.close()
    pre = pre.cpu().numpy().astype(np.float64).reshape(nl, nw, T, 2 * C)
    xo = xo.cpu().numpy().astype(np.float64).reshape(nl, nw, T, C)
    so = so.cpu().numpy().astype(np.float64).reshape(nl, nw, T, C)
    assert np.isfinite(pre).all() and (np.abs(x) > 448).mean() > 0.1
    xb, skip_in = to_bf16(x.astype(np.float64)), None if first == 0 else sk.astype(np.float64)
    for j in range(nl):
        check_layer("fp8", p, first + j, xb, skip_in, pre[j], xo[j], so[j], f"layer {first + j}")
        xb, skip_in = xo[j], so[j]
