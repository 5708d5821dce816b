"""Encodes with more than eight parity rows: groups of parity rows over the same
block rows, with row counts that are no multiple of the eight they are dealt in.

Integer inputs keep every sum exact, so the planes equal the oracle's."""
import numpy as np
import pytest

import synth
from oracle import coded as oc
from tests.gpu_helpers import device_tensor, make_inputs, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# two groups (one partial) and more; one, seven, eight, nine and seventeen block rows; several rows per
# workgroup, one, and several column chunks
@pytest.mark.parametrize("n,k,q,r", [(12, 3, 3, 40), (19, 10, 70, 1024), (64, 48, 48 * 8, 2050), (30, 7, 7 * 9 - 2, 3000),
                                     (128, 64, 64 * 17 - 5, 33), (40, 4, 4 * 131, 9), (20, 2, 34, 3),
                                     # planes past the sizes that take one column a thread (96 Ki elements times
                                     # groups in fp32, 256 Ki in bf16), and either side of them
                                     (12, 3, 3 * 4000, 40), (64, 48, 48 * 70, 2050), (30, 7, 7 * 40 - 3, 3000),
                                     (128, 64, 64 * 1100 - 5, 33), (40, 4, 4 * 6100, 9), (4, 3, 3 * 1024, 96),
                                     (4, 3, 3 * 1025, 96), (4, 3, 3 * 1024, 256), (4, 3, 3 * 1025, 256),
                                     (5, 3, 3 * 300 - 1, 1021)])
def test_encode_groups(lib, torch, dtype, n, k, q, r):
    P, A, _ = make_inputs(n, k, q, r, 1, 17, dtype, integer=True)
    code = lib.Code.systematic(P, 2)
    dA = device_tensor(A, dtype)
    par = lib.alloc_parity(code, q, r, dA.dtype)
    par.fill_(-3.0)
    lib.coded_encode(code, dA, par)
    torch.cuda.synchronize()
    ref = oc.encode(oc.systematic_generator(P), oc.pad_and_split(A, k))[k:]
    got = par.float().cpu().numpy().astype(np.float64)
    if dtype == "f32":
        assert np.array_equal(got[0], ref) and np.all(got[1] == 0)
    else:
        assert np.array_equal(got[0] + got[1], ref)     # whole numbers below 2^16: 8 + 8 bits hold them


def test_groups_of_the_longest_rows(lib, torch):
    # 16 groups of parity rows, 4102 column chunks each: more than 65535 together, which a launch takes
    n, r = 128, 4_200_000
    P = np.arange(1, n, dtype=np.float32).reshape(n - 1, 1)
    code = lib.Code.systematic(P, 1)
    A = (torch.arange(r, device="cuda", dtype=torch.int64) % 1021 - 510).to(torch.float32).reshape(1, r)
    par = lib.alloc_parity(code, 1, r, A.dtype)
    lib.coded_encode(code, A, par)
    torch.cuda.synchronize()
    got = par.reshape(n - 1, r)
    for p in range(n - 1):
        assert bool((got[p] == A[0] * float(p + 1)).all())      # whole numbers below 2^24
