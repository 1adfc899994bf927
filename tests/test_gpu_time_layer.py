"""gwd_debug_time_layer issues the launches of the last forward: its members, windows and rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

S = 4096


@pytest.mark.parametrize("prec,layer", [("bf16", 10), ("fp8", 16), ("fp32", 15)])
def test_launch_of_the_last_forward(prec, layer):
    """Windows per launch: those of the first batch times the members that one launch takes (four with sextets
    here, one in FP32). A plan in between does not change it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    print(f"case: {prec} layer {layer}", flush=True)
    blobs = np.stack([synth.full_weights(i) for i in range(4)])
    x = torch.randn((40 * S, 2), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    group = 1 if prec == "fp32" else 4
    m = gwd.Model(gwd.full_arch(), blobs, prec)
    full = [x[i * 5 * S:(i + 1) * 5 * S] for i in range(8)]
    for xs in (full, full[:1] + [f[:S] for f in full[1:]]):
        m.forward(xs, S, 256, 0)
        plan = m.plan([x[:S + 64]], S, 256, 0)
        for member in (0, 3):
            t, windows, _ = m.time_layer(member, layer, 3)
            assert windows == 8 * group and t > 0
        plan.launch()
        torch.cuda.synchronize()
        plan.close()
    one = gwd.Model(gwd.full_arch(), blobs[:1], prec)
    one.forward(full, S, 256, 0)
    assert one.time_layer(0, layer, 3)[1] == 8
    m.set_window_merging(False)
    m.forward([x], S, 256, 0)
    assert m.time_layer(0, layer, 1)[1] == 512
    m.close()
    one.close()
