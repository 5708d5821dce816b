"""fp32 single-vector worker products (Sec. III-A) for rows of any length, stride
and alignment, through the C ABI against the oracle.

Integer-valued inputs make every sum exact, so Y must equal the oracle's bit
for bit.  Row lengths sit at the edges of the kernels' ranges (64, 128, 256,
512, 1024, 2048, 4096, 6144, 8192) and their remainders modulo 4; row counts
give one, two and four rows per group; everything beside the operands holds
NaN, so a read that strays into a sum shows."""
import numpy as np
import pytest

from oracle import coded as oc
from tests.gpu_helpers import device_tensor, make_inputs, torch_mod

pytestmark = pytest.mark.gpu

R = [1, 2, 3, 4, 5, 63, 64, 65, 127, 129, 256, 259, 511, 513, 1023, 1025, 2047, 2050, 4095, 4097, 6143, 6145, 8191, 8193,
     8200]


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def _check(lib, torch, n, k, q, r, planes, apad=0, lead=0, mask=None):
    P, A, X = make_inputs(n, k, q, r, 1, 3 + r, integer=True)
    code = lib.Code.systematic(P, planes)
    buf = torch.full((lead + q * (r + apad) + 16,), float("nan"), device="cuda")
    dA = buf[lead:lead + q * (r + apad)].view(q, r + apad)[:, :r]
    dA.copy_(device_tensor(A))
    xb = torch.full((lead + r + 16,), float("nan"), device="cuda")
    dX = xb[lead:lead + r]
    dX.copy_(device_tensor(X[:, 0]))
    par = lib.alloc_parity(code, q, r, torch.float32)
    lib.coded_encode(code, dA, par)
    Y = lib.alloc_y(code, q, 1, torch.float64)
    Y.fill_(-7.0)
    lib.coded_worker_mm(code, dA, par, dX, Y, worker_mask=mask)
    torch.cuda.synchronize()
    ref = oc.worker_products(oc.encode(oc.systematic_generator(P), oc.pad_and_split(A, k)), X)
    if mask is not None:
        ref[mask == 0] = -7.0
    assert np.array_equal(Y.cpu().numpy().reshape(ref.shape), ref), (n, k, q, r, planes, apad, lead)


@pytest.mark.parametrize("r", R)
@pytest.mark.parametrize("planes", [1, 2, 3])
def test_row_lengths(lib, torch, r, planes):
    _check(lib, torch, 5, 3, 50, r, planes)


@pytest.mark.parametrize("r", [61, 100, 200, 403, 900])
@pytest.mark.parametrize("qb", [1, 31, 700, 3000, 11000])
def test_rows_per_group(lib, torch, r, qb):
    _check(lib, torch, 5, 3, 3 * qb - 1 if qb > 1 else 2, r, 2)


@pytest.mark.parametrize("apad,lead", [(1, 0), (0, 1), (3, 2), (5, 3)])
@pytest.mark.parametrize("r", [64, 400, 1000, 1200, 5000, 9000])
def test_strides_and_alignment(lib, torch, apad, lead, r):
    _check(lib, torch, 6, 4, 40, r, 2, apad, lead)


def test_mask_and_streamed_size(lib, torch):
    mask = np.zeros(16, dtype=np.uint8)
    mask[[0, 11, 12, 15]] = 1
    for r in (90, 777, 1301):
        _check(lib, torch, 16, 12, 500, r, 2, mask=mask)
    for r in (901, 8001):                      # past 256 MB: non-temporal loads
        _check(lib, torch, 3, 2, 50000000 // r, r, 2)
