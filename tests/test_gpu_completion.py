"""Completion times of a plan's streams on merged windows: one per batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("batch,merging,times", [(512, True, 1), (12, True, 3), (1, True, 8), (60, False, 5)])
def test_streams_complete_with_their_batch(batch, merging, times):
    """Eight streams of 3 s: as many different times as batches with a stream's last window in them, in the order
    of the streams, the last one the total. Merged: one window per stream; three of 6,144 in batches of 8
    (2, 5 | 8, 11, 14 | 17, 20, 23 are the last ones); nine of 4,096, a batch each. Not merged: 33 windows per
    stream in batches of 60."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    print(f"case: batch {batch}, merging {merging}", flush=True)
    m = gwd.Model(gwd.full_arch(), synth.full_weights(8), "bf16")
    m.set_tiling(0, 0, batch, 0)
    m.set_window_merging(merging)
    x = torch.randn((24 * 4096, 2), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    xs = list(x.split(3 * 4096))
    plan = m.plan(xs, 4096, 256, 0)
    assert torch.equal(plan.launch(), m.forward(xs, 4096, 256, 0))
    us, total = plan.completion_us()
    plan.close()
    m.close()
    us = np.asarray(us)
    assert (us > 0).all() and (np.diff(us) >= 0).all() and us[-1] == total
    assert len(np.unique(us)) == times
