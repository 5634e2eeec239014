"""Histograms at the sizes where a sample is dealt to another number of blocks,
against numpy's definition, and what a sample of 16,384 values costs."""
import numpy as np
import pytest

from oracle import stats as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0908_3889_amd import _lib
    _lib.load()
    yield


# one block and two; the last of 4096 values a block, a ragged one of 64; the
# first of 16,384; spread values and equal ones
@pytest.mark.parametrize("n", [8192, 8193, 12288, 262144, 262145, 1048576, 1048577])
def test_histogram_block_edges(n):
    from paper_0908_3889_amd import api
    x = np.random.default_rng(n).uniform(-1.05, 1.05, (2, n))
    x[1] = 0.25
    y = np.roll(x, 5, axis=1)
    xt, yt = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    for nbins in (20, 79):
        one = api.pn_histogram(xt, nbins).cpu().numpy()
        two = api.pn_histogram2d(xt, yt, nbins).cpu().numpy()
        for c in range(2):
            assert (one[c] == S.histogram(x[c], -1.0, 1.0, nbins)).all()
            assert (two[c] == S.histogram2d(x[c], y[c], -1.0, 1.0, nbins)).all()


# 16,384 values counted by one block took 3.4 times as long as 1000 (equal
# values: 2.4 times by four)
def test_time_of_a_sample_of_several_blocks():
    from paper_0908_3889_amd import api

    def us(n):
        x = torch.full((1, n), 0.25, dtype=torch.float64, device="cuda")
        api.pn_histogram2d(x, x, 79)
        best = 1e9
        for _ in range(5):
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                for _ in range(40):
                    api.pn_histogram2d(x, x, 79)
            graph.replay()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / 40)
        return best

    small, large = us(1000), us(16384)
    print(f"\n1000 values {small:.1f} us, 16384 {large:.1f} us", flush=True)
    assert large < 2.5 * small + 2.0
