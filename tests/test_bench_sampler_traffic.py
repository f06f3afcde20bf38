"""The byte model of the streaming sampler in bench.py: passes of four where all
proposals are accepted (cache read and written once) or rejected (read once), one
proposal in a pass at middle acceptances and where one row's ratios fill the LDS."""
import pytest

from bench import sampler_traffic


@pytest.mark.parametrize("acc,K,M,expect", [
    (1.0, 1, 400, ("sample_stream_kernel", 1.0, 0.25, 0.25)),
    (0.0, 1, 400, ("sample_stream_kernel", 1.0, 0.25, 0.0)),
    (0.5, 1, 400, ("sample_kernel", 1.0, 1.0, 1.0)),
    (1.0, 10, 8, ("sample_kernel", 1.0, 1.0, 1.0)),
    (0.0, 3, 24, ("sample_kernel", 1.0, 1.0, 1.0))])
def test_limits(acc, K, M, expect):
    got = sampler_traffic(acc, 800 * K * 8, 800 * K * M * 8)
    assert got[0] == expect[0]
    # the first passes, before the chain's acceptance is known, differ a little
    assert got[1:] == pytest.approx(expect[1:], abs=2e-3)


@pytest.mark.parametrize("acc", [0.97, 0.9, 0.82, 0.2, 0.1, 0.05])
def test_between(acc):
    kernel, rows, reads, writes = sampler_traffic(acc, 6400, 6400 * 400)
    assert kernel == "sample_stream_kernel"
    assert rows > 1.0 and 0.25 < reads < 1.0 and 0.0 < writes <= reads
