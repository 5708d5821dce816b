"""Multi-column fp32 worker products (Sec. III-A) for rows of any length, stride
and alignment, through the C ABI against the oracle.

Integer-valued inputs make every sum exact in fp64, so Y must equal the
oracle's bit for bit.  Row lengths sit at the edges of the K chunks (64 and
128) and their remainders modulo 4, column counts at each tile width;
everything beside the operands holds NaN, so a read that strays into a sum
shows.  The merged hi + lo rows are compared on Gaussian inputs too."""
import numpy as np
import pytest

from oracle import coded as oc
from tests.gpu_helpers import device_tensor, make_inputs, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def _view(torch, M, pad, lead):
    rows, cols = M.shape
    buf = torch.full((lead + rows * (cols + pad) + 16,), float("nan"), device="cuda")
    v = buf[lead:lead + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    v.copy_(device_tensor(M))
    return v


def _run(lib, torch, n, k, q, r, s, planes, apad=0, xpad=0, lead=0, integer=True):
    P, A, X = make_inputs(n, k, q, r, s, 3 + r + s, integer=integer)
    code = lib.Code.systematic(P, planes)
    dA, dX = _view(torch, A, apad, lead), _view(torch, X, xpad, lead)
    par = lib.alloc_parity(code, q, r, torch.float32)
    lib.coded_encode(code, dA, par)
    Y = lib.alloc_y(code, q, s, torch.float64)
    Y.fill_(float("nan"))
    lib.coded_worker_mm(code, dA, par, dX, Y)
    torch.cuda.synchronize()
    ref = oc.worker_products(oc.encode(oc.systematic_generator(P), oc.pad_and_split(A, k)), X)
    return Y.cpu().numpy().reshape(ref.shape), ref


@pytest.mark.parametrize("r", [1, 3, 4, 5, 7, 62, 63, 65, 66, 67, 127, 129, 130, 191, 193, 255, 257, 514])
@pytest.mark.parametrize("s", [2, 5, 12, 40])
def test_row_lengths(lib, torch, r, s):
    for planes in (1, 2):
        got, ref = _run(lib, torch, 5, 3, 70, r, s, planes)
        assert np.array_equal(got, ref), (r, s, planes)


@pytest.mark.parametrize("apad,xpad,lead", [(1, 0, 1), (0, 3, 2), (3, 1, 3), (4, 4, 0)])
@pytest.mark.parametrize("r,s", [(132, 3), (257, 7), (130, 16), (321, 33)])
def test_strides_and_alignment(lib, torch, apad, xpad, lead, r, s):
    got, ref = _run(lib, torch, 6, 4, 45, r, s, 2, apad, xpad, lead)
    assert np.array_equal(got, ref)


# several tiles with a ragged last one; blocks of padding only; no parity; one row per block
@pytest.mark.parametrize("n,k,q,r,s", [(20, 16, 1999, 131, 20), (64, 48, 49, 70, 9), (4, 4, 33, 131, 7), (5, 3, 1, 90, 3),
                                       (64, 48, 700, 257, 32),
                                       # both sides of the tile rules: 16 x 4 tiles up to 256 workgroups (4 columns)
                                       # and up to 192 and 384 (8), 16 x 16 tiles, 32 x 32 in one launch with a last
                                       # tile of 1 and of 17 columns, and launches of 32 columns
                                       (20, 16, 2300, 70, 4), (20, 16, 2800, 70, 4), (20, 16, 1000, 70, 8), (20, 16, 1500, 70, 8),
                                       (20, 16, 2900, 70, 8), (20, 16, 2000, 66, 96), (20, 16, 3000, 66, 65),
                                       (20, 16, 3000, 66, 49), (20, 16, 9000, 65, 49), (4, 2, 2666, 65, 20)])
def test_tiles(lib, torch, n, k, q, r, s):
    got, ref = _run(lib, torch, n, k, q, r, s, 2)
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("s", [8, 9, 33])
def test_gaussian_parity(lib, torch, s):
    """fp64 sums of r products of hi + lo: r times 2^-53 of the sum of magnitudes, and the plane's 2^-48."""
    n, k, q, r = 20, 16, 500, 1001
    got, ref = _run(lib, torch, n, k, q, r, s, 2, integer=False)
    P, A, X = make_inputs(n, k, q, r, s, 3 + r + s)
    mag = oc.worker_products(oc.encode(np.abs(oc.systematic_generator(P)), oc.pad_and_split(np.abs(A), k)), np.abs(X))
    assert np.all(np.abs(got - ref) <= (2 * r * 2.0 ** -53 + 2.0 ** -47) * mag)
