"""Stitched forwards on merged windows equal the request's own windows bit for bit."""
import numpy as np
import pytest

from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# stream lengths: one sample, the edges of tiles, of the receptive field and of a window, several
# merged windows in one stream, ragged sets with an empty stream
LENGTHS = [[1], [127, 128, 129], [3069, 3070, 3071], [4096], [4097, 0, 64], [30000], [131, 61234, 9000, 0, 4095]]


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd
    return gwd


@pytest.mark.parametrize("prec,two", [("fp32", False), ("bf16", False), ("fp8", False), ("bf16", True)])
def test_merged_windows_give_the_same_scores(g, prec, two):
    from paper_2201_11133_amd import synth
    make = synth.two_branch_weights if two else synth.full_weights
    m = g.Model(g.two_branch_arch() if two else g.full_arch(), np.stack([make(41), make(42)]), prec)
    for i, lens in enumerate(LENGTHS):
        xs = [to_dev(synth.make_stream(500 + 10 * i + j, max(L, 1) / 4096, 0)[0][:L]) if L
              else torch.zeros((0, 2), device="cuda") for j, L in enumerate(lens)]
        if i % 2:   # planar streams
            xs = [(x[:, 0].contiguous(), x[:, 1].contiguous()) for x in xs]
        for W, S in ((4096, 256), (3200, 128), (8192, 1000)):
            for batch in (1, 7, 512):   # the batch bounds the merged windows' rows
                for fuse in ((1,) if prec == "fp32" else (1, 3, 6)):
                    m.set_tiling(0, 0, batch, fuse)
                    m.set_window_merging(False)
                    ref = m.forward(xs, W, S, 1).clone()
                    m.set_window_merging(True)
                    print(f"case: {prec} {lens} W={W} S={S} batch={batch} fuse={fuse}", flush=True)
                    assert torch.equal(m.forward(xs, W, S, 1), ref)
                    if batch == 7:
                        assert torch.equal(m.forward(xs, W, S, 0), ref[: sum(lens)])
                        plan = m.plan(xs, W, S, 1)
                        assert torch.equal(plan.launch(), ref)
                        plan.close()
    assert g.lib.gwd_set_window_merging(m.h, 2) == g.ERR_ARG and g.lib.gwd_set_window_merging(None, 1) == g.ERR_ARG
    m.close()


@pytest.mark.parametrize("prec,members", [("bf16", 3), ("bf16", 4), ("bf16", 9), ("fp8", 5), ("fp8", 8)])
def test_members_of_one_launch(g, prec, members):
    """Launches over several members (all counts that divide the XCDs and some that do not, more members
    than one launch takes): each member's scores equal those of a model of its own, bit for bit, and the
    ensemble score is their minimum."""
    from paper_2201_11133_amd import synth
    print(f"case: {prec} {members} members", flush=True)
    blobs = np.stack([synth.full_weights(60 + i) for i in range(members)])
    xs = [to_dev(synth.make_stream(600 + i, L / 4096, 0)[0][:L]) for i, L in enumerate((40000, 64, 9001))]
    n = sum(len(x) for x in xs)
    m = g.Model(g.full_arch(), blobs, prec)
    e = m.forward(xs, 4096, 256, 1).clone()
    w = m.forward(xs[:1], 4096, 1024, 2).clone().reshape(members, -1)
    m.close()
    for i in range(members):
        one = g.Model(g.full_arch(), blobs[i], prec)
        assert torch.equal(e[n * (1 + i): n * (2 + i)], one.forward(xs, 4096, 256, 0))
        assert torch.equal(w[i], one.forward(xs[:1], 4096, 1024, 2))
        one.close()
    assert torch.equal(e[:n], e[n:].reshape(members, n).min(dim=0).values)


@pytest.mark.parametrize("seconds,merging", [(64, True), (400, True), (400, False)])
def test_little_free_memory(seconds, merging):
    """With 4 GiB of device memory free, a request whose windows and members would not fit together is split
    further, with the same scores."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    print(f"case: {seconds} s, merging {merging}", flush=True)
    blobs = np.stack([synth.full_weights(i) for i in range(4)])
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((seconds * 4096, 2), generator=gen, device="cuda")
    window, stride = (4096, 256) if merging else (1 << 18, (1 << 18) - 3072)
    want = gwd.Model(gwd.full_arch(), blobs, "bf16")
    want.set_window_merging(merging)
    ref = want.forward([x], window, stride).clone()
    want.close()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    m = gwd.Model(gwd.full_arch(), blobs, "bf16")
    m.set_window_merging(merging)
    free, _ = torch.cuda.mem_get_info()
    ballast = torch.empty(free - (4 << 30), dtype=torch.uint8, device="cuda")
    try:
        got = m.forward([x], window, stride)
        torch.cuda.synchronize()
        assert torch.equal(got, ref)
    finally:
        del ballast
        torch.cuda.empty_cache()
        m.close()
