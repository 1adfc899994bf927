"""Requests of one long stream and many short ones: merged windows that fill their batches, same scores."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec,lens", [("bf16", [64 * 4096] + [4096] * 600), ("fp8", [4096] * 300 + [40 * 4096 + 17] + [1, 0] * 150),
                                       ("fp32", [30 * 4096] + [777] * 200)])
def test_long_and_short_streams(prec, lens):
    """The request takes no more batches than its own windows would (a window of the longest stream's length
    would leave batches of 8 to 17 windows); the scores are those of the request's own windows, bit for bit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    print(f"case: {prec} {len(lens)} streams, longest {max(lens)}", flush=True)
    m = gwd.Model(gwd.full_arch(), synth.full_weights(3), prec)
    gen = torch.Generator(device="cuda").manual_seed(len(lens))
    xs = [torch.randn((L, 2), generator=gen, device="cuda") for L in lens]
    m.set_window_merging(False)
    ref = m.forward(xs, 4096, 256, 0).clone()
    torch.cuda.synchronize()
    own = sum(0 if L == 0 else 1 if L <= 4096 else -(-(L - 4096) // 256) + 1 for L in lens)
    m.set_window_merging(True)
    assert torch.equal(m.forward(xs, 4096, 256, 0), ref)
    _, per_launch, _ = m.time_layer(0, 16 if prec != "fp32" else 15, 1)
    plan = m.plan(xs, 4096, 256, 0)
    assert torch.equal(plan.launch(), ref)
    plan.close()
    m.close()
    # at least every stream is a window of its own
    batches = -(-sum(L > 0 for L in lens) // per_launch)
    assert batches <= -(-own // 512), (batches, per_launch)
