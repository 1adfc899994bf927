"""Peak walks at the edges of their blocks (64 samples, 256, 65,536) and trigger tables of many streams."""
import numpy as np
import pytest

from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_11133_amd import gwd
    return gwd


@pytest.mark.parametrize("n", [64, 255, 256, 257, 4095, 4096, 4097, 65536, 65537, 131072, 200001])
def test_walks_across_blocks(g, n):
    """Peaks next to block edges whose bases lie whole blocks away, on noise and on plateaus: indices and
    widths equal SciPy's bit for bit, at the start, end and every block edge of the signal."""
    from oracle.postproc import find_peaks
    print(f"case: n={n}", flush=True)
    rng = np.random.default_rng(n)
    at = sorted({int(v) for e in (64, 256, 4096, 65536) for k in range(0, n, e) for v in (k - 1, k, k + 1)
                 if 0 < v < n - 1} if n < 5000 else {int(v) for v in rng.integers(1, n - 1, 300)} | {n - 2, 1, 256, 65535})
    for x in (rng.standard_normal(n) * 1e-3, np.zeros(n), np.round(rng.standard_normal(n))):
        x[[a for a in at if a < n - 1]] += rng.uniform(1.0, 5.0, size=len([a for a in at if a < n - 1]))
        for height, wmin in ((0.5, 0.0), (-10.0, 100.0)):
            p, w = g.find_peaks(to_dev(x), height, wmin)
            rp, rw = find_peaks(x, height, wmin)
            assert np.array_equal(p, rp) and np.array_equal(w, rw)


@pytest.mark.parametrize("n_streams", [79, 80, 81, 700])
def test_trigger_tables(g, n_streams):
    """Stream tables that fit the kernel argument and ones that do not, with more records than the first
    copy holds."""
    from oracle.triggers import triggers
    rng = np.random.default_rng(n_streams)
    offs = np.concatenate([[0], np.cumsum(rng.integers(0, 40, n_streams))])
    e = rng.standard_normal(offs[-1]).astype(np.float32) * 4
    got = [(s, a) for s, a, _, _ in g.triggers(to_dev(e), offs, 0.9, 3)]
    assert got == [(s, a) for s, a, _, _ in triggers(e.astype(np.float64), offs, 0.9, 3)]
