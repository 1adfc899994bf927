"""A call that fails for lack of device memory leaves the next one alone."""
import pytest

from tests.test_gpu_scratch_limits import MB, Ballast

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_calls_after_a_failed_one():
    """Whitening 2^26 samples takes 1 GiB of workspace (more than other tests leave behind); with 200 MiB free it
    fails. The calls after it (peaks, the small member's forward, whitening a short stream) work and give
    what they gave before."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd, synth
    gen = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((1 << 26, 2), generator=gen, device="cuda")
    short, s = x[: 1 << 13], x[: 1 << 16, 0].double()
    m = gwd.Model(gwd.tiny_arch(), synth.tiny_weights(1), "fp32")
    psd = gwd.welch_psd(short, 1024)

    def calls():
        p, w = gwd.find_peaks(s, 1.0, 1.0)
        return (torch.from_numpy(p), torch.from_numpy(w), m.forward([short], 256, 128).clone(),
                gwd.whiten(short, psd, 1024).clone())

    want = calls()
    print("case: whitening without room for its workspace", flush=True)
    out = torch.empty_like(x)
    with Ballast(200 * MB):
        with pytest.raises(gwd.GwdError):
            gwd.whiten(x, psd, 1024, out=out)
        got = calls()
    m.close()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
