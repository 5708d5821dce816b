"""The runtime model's order statistics at every register size of the kernel:
each worker count at and around the sizes it is built for, against a sort of the
same SplitMix64 words on the host.  Past 64 workers the kernel orders 25-bit
keys and ranks the few draws where neighbours share them exactly; 2^19 draws of
128 workers hold several of those.  A result is one fp64 logarithm, one or two
divisions and a sum: 4 units in the last place."""
import numpy as np
import pytest

from tests.gpu_helpers import torch_mod

pytestmark = pytest.mark.gpu
GAMMA, M1, M2 = np.uint64(0x9E3779B97F4A7C15), np.uint64(0xBF58476D1CE4E5B9), np.uint64(0x94D049BB133111EB)


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def _words(n, seed, first, draws):
    with np.errstate(over="ignore"):
        d = np.arange(first, first + draws, dtype=np.uint64)[:, None]
        c = (np.uint64(4 << 56) | (d << np.uint64(16)) | np.arange(n, dtype=np.uint64)[None, :]) + np.uint64(1)
        z = np.uint64(seed) + c * GAMMA
        z = (z ^ (z >> np.uint64(30))) * M1
        z = (z ^ (z >> np.uint64(27))) * M2
        return (z ^ (z >> np.uint64(31))) >> np.uint64(11)


def _check(lib, torch, n, k, draws, shift=1.0, rate=1.0, seed=11, first=77, rep=None):
    rep = n % k == 0 if rep is None else rep
    new = lambda: torch.full((draws,), -1.0, dtype=torch.float64, device="cuda")  # noqa: E731
    tu, tr, tm = new(), (new() if rep else None), new()
    lib.coded_simulate_runtimes(n, k, seed, first, tu, tr, tm, shift=shift, rate=rate)
    torch.cuda.synchronize()
    top = _words(n, seed, first, draws)
    t0 = lambda w: shift - np.log((w.astype(np.float64) + 0.5) * 2.0 ** -53) / rate  # noqa: E731
    want = [(tu, t0(top.min(axis=1)) / n), (tm, t0(np.sort(top, axis=1)[:, n - k]) / k)]
    if rep:
        want.append((tr, t0(top.reshape(draws, k, n // k).max(axis=2).min(axis=1)) / k))
    for got, ref in want:
        g = got.cpu().numpy()
        assert np.max(np.abs(g - ref) / np.abs(ref)) <= 4 * 2.0 ** -52, (n, k)


@pytest.mark.parametrize("n", list(range(1, 26)) + [28, 29, 32, 33, 36, 37, 40, 41, 48, 49, 56, 57, 63, 64, 65, 72, 73, 84, 85,
                                                    96, 97, 112, 113, 127, 128])
def test_every_size(lib, torch, n):
    for k in sorted({1, 2 if n > 1 else 1, (n + 1) // 2, max(1, n // 2), max(1, n - 1), n}):
        _check(lib, torch, n, k, 1000)


@pytest.mark.parametrize("k", [1, 64, 100, 128])
def test_shared_keys(lib, torch, k):
    _check(lib, torch, 128, k, 1 << 19, rep=False)


@pytest.mark.parametrize("shift,rate", [(0.0, 1.0), (1.0, 3.7), (-2.5, 0.013), (1.0, 1e-120), (1.0, 1e120), (1e-3, 7e99)])
def test_shift_and_rate(lib, torch, shift, rate):
    _check(lib, torch, 12, 4, 2000, shift, rate)


def test_single_outputs(lib, torch):
    """Each scheme alone gives what it gives beside the others."""
    n, k, draws = 20, 10, 3000
    new = lambda: torch.zeros(draws, dtype=torch.float64, device="cuda")  # noqa: E731
    both = [new(), new(), new()]
    lib.coded_simulate_runtimes(n, k, 5, 0, *both)
    for i in range(3):
        one = [None, None, None]
        one[i] = new()
        lib.coded_simulate_runtimes(n, k, 5, 0, *one)
        torch.cuda.synchronize()
        assert torch.equal(one[i], both[i])


def test_more_draws_than_one_grid_takes(lib, torch):
    """2^32 + 5 draws: windows around the ends of the launches, and no draw left out."""
    n, k, count = 2, 1, 2 ** 32 + 5
    tm = torch.full((count,), -1.0, dtype=torch.float64, device="cuda")
    lib.coded_simulate_runtimes(n, k, 3, 0, None, None, tm)
    assert float(tm.min()) >= 1.0
    for first, size in ((0, 1000), (2 ** 31 - 300, 600), (2 ** 32 - 300, 305)):
        part = torch.empty(size, dtype=torch.float64, device="cuda")
        lib.coded_simulate_runtimes(n, k, 3, first, None, None, part)
        assert torch.equal(part, tm[first:first + size])
