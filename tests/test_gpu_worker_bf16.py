"""bf16 worker products on the matrix cores (Sec. III-A: every worker multiplies
its coded block by the multicast input) for rows of any length, stride and
alignment, through the C ABI against the oracle.

Integer-valued inputs make every product and partial sum exact in fp32, so Y
must equal the oracle's bit for bit in whatever order it is summed.  The
shapes sit at the edges of the tiles and chunks (64, 128, 256, 512 elements of
K; 8, 16, 32, 64 columns; 16 to 128 row slots) and of the rules that choose
between them.  Everything beside the operands (row padding of A, of X, and the
elements around them) holds NaN, so a read that strays into a result shows."""
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


def _padded(torch, M, pad, lead):
    """M (bf16 values) as a view of row stride cols + pad that starts `lead` elements into a NaN-filled buffer."""
    rows, cols = M.shape
    buf = torch.full((lead + rows * (cols + pad) + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    view = buf[lead:lead + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]
    view.copy_(device_tensor(M, "bf16"))
    return view


def _check(lib, torch, n, k, q, r, s, planes, apad=0, xpad=0, lead=0, mask=None):
    P, A, X = make_inputs(n, k, q, r, s, 7 + r + s, "bf16", integer=True)
    code = lib.Code.systematic(P, planes)
    dA = _padded(torch, A, apad, lead)
    dX = _padded(torch, X, xpad, lead)
    if s == 1 and not xpad:
        dX = dX.view(-1) if dX.is_contiguous() else dX
    par = lib.alloc_parity(code, q, r, torch.bfloat16)
    lib.coded_encode(code, dA, par)
    Y = lib.alloc_y(code, q, s, torch.float32)
    Y.fill_(-7.0)
    lib.coded_worker_mm(code, dA, par, dX, Y, worker_mask=mask)
    torch.cuda.synchronize()
    ref = oc.worker_products(oc.encode(oc.systematic_generator(P), oc.pad_and_split(A, k)), X)
    if mask is not None:
        ref[mask == 0] = -7.0
    got = Y.cpu().numpy().astype(np.float64)
    assert np.array_equal(got.reshape(ref.shape), ref), (n, k, q, r, s, planes, apad, xpad, lead)


# K at the edges of the pieces and chunks, one column count per tile width
@pytest.mark.parametrize("r", [1, 7, 8, 9, 15, 63, 64, 65, 127, 129, 255, 257, 511, 513, 1024, 1025, 1031])
@pytest.mark.parametrize("s", [1, 3, 17, 40])
def test_row_lengths(lib, torch, r, s):
    _check(lib, torch, 5, 3, 100, r, s, 2)


@pytest.mark.parametrize("s", [2, 7, 8, 9, 15, 16, 24, 31, 32, 33, 63, 64, 65, 96, 100])
@pytest.mark.parametrize("planes", [1, 2])
def test_column_counts(lib, torch, s, planes):
    _check(lib, torch, 6, 4, 150, 331, s, planes)


# tile choices: many workgroups (128-, 64-, 32-row tiles), few, short rows, one row per block, last block all padding
@pytest.mark.parametrize("n,k,q,r,s", [(16, 12, 13000, 70, 40), (16, 12, 13001, 530, 20), (16, 12, 13001, 1030, 5),
                                       (16, 12, 9000, 300, 12), (4, 4, 33, 1301, 9), (3, 1, 40, 1033, 12),
                                       (64, 48, 60, 1100, 8), (64, 48, 49, 90, 33), (5, 3, 1, 1040, 2)])
def test_tiles(lib, torch, n, k, q, r, s):
    _check(lib, torch, n, k, q, r, s, 2)


@pytest.mark.parametrize("apad,xpad,lead", [(1, 0, 1), (3, 5, 2), (5, 1, 4), (6, 9, 7), (8, 8, 0)])
@pytest.mark.parametrize("r,s", [(1032, 4), (200, 1), (264, 24), (1027, 64)])
def test_strides_and_alignment(lib, torch, apad, xpad, lead, r, s):
    _check(lib, torch, 5, 3, 70, r, s, 2, apad, xpad, lead)


# Rows shorter than one 16-byte piece: the vector kernel.
@pytest.mark.parametrize("r", [2, 3, 5, 6, 7])
@pytest.mark.parametrize("s,planes,apad,xpad", [(1, 2, 0, 0), (1, 1, 3, 0), (4, 2, 1, 2), (5, 1, 0, 3), (18, 2, 2, 1)])
def test_tiny_rows(lib, torch, r, s, planes, apad, xpad):
    _check(lib, torch, 6, 4, 101, r, s, planes, apad=apad, xpad=xpad, lead=1)


def test_tiny_rows_mask(lib, torch):
    mask = np.zeros(6, dtype=np.uint8)
    mask[[1, 4]] = 1
    _check(lib, torch, 6, 4, 101, 6, 3, 2, mask=mask)


# Rows of whole 16-byte pieces that take one step of K (up to 224 elements; 256
# with up to 32 columns, 384 with up to 16), either side of the steps of 64, one
# and two column tiles traded between rows, column remainders of 1 to 3, blocks
# of less than a 16-row tile and of more than a workgroup's 256 slots, padding
# rows, odd strides of X.
@pytest.mark.parametrize("r", [8, 56, 64, 72, 128, 136, 192, 200, 224, 232, 256, 264, 320, 328, 384, 392])
@pytest.mark.parametrize("s", [1, 2, 15, 17, 31, 33, 47, 48, 62, 64, 67])
def test_short_rows(lib, torch, r, s):
    _check(lib, torch, 6, 4, 1131, r, s, 2, xpad=s % 3)


@pytest.mark.parametrize("n,k,q,planes", [(5, 3, 2, 2), (4, 4, 45, 2), (64, 48, 47, 2), (6, 4, 2049, 1), (3, 1, 300, 2)])
@pytest.mark.parametrize("r,s", [(64, 5), (160, 64), (256, 20), (384, 16)])
def test_short_row_blocks(lib, torch, n, k, q, planes, r, s):
    _check(lib, torch, n, k, q, r, s, planes, apad=8)


def test_short_row_mask(lib, torch):
    mask = np.zeros(16, dtype=np.uint8)
    mask[[1, 11, 13, 15]] = 1
    for r, s in ((72, 40), (264, 3)):
        _check(lib, torch, 16, 12, 700, r, s, 2, mask=mask)


# Enough rows for the tiles of 64 and 128 rows (512 and 1024 workgroups of 128),
# rows past the short ones and, from 256 MB on, streamed ones.  Checked on the
# GPU in fp64, exact for the integers.
@pytest.mark.parametrize("q,r,s", [(50000, 270, 33), (50000, 264, 20), (110000, 330, 64), (110000, 264, 20), (110000, 400, 130),
                                   (230000, 400, 1), (230000, 648, 3), (190000, 776, 17), (120000, 1100, 33),
                                   (70000, 2048, 48), (45000, 2056, 48)])
def test_many_rows(lib, torch, q, r, s):
    n, k = 20, 16
    gen = torch.Generator(device="cuda").manual_seed(q + r + s)
    A = torch.randint(-3, 4, (q, r), device="cuda", generator=gen).bfloat16()
    X = torch.randint(-3, 4, (r, s), device="cuda", generator=gen).bfloat16()
    P = torch.randint(-2, 3, (n - k, k), device="cuda", generator=gen).double()
    code = lib.Code.systematic(P.cpu().numpy(), 2)
    par = lib.alloc_parity(code, q, r, torch.bfloat16)
    lib.coded_encode(code, A, par)
    qb = code.qb(q)
    B = torch.zeros((k * qb, s), dtype=torch.float64, device="cuda")
    for i in range(0, q, 20000):
        B[i:min(q, i + 20000)] = A[i:i + 20000].double() @ X.double()
    B = B.view(k, qb * s)
    ref = torch.cat([B, P @ B]).view(n, qb, s)
    Y = lib.alloc_y(code, q, s, torch.float32)
    Y.fill_(float("nan"))
    lib.coded_worker_mm(code, A, par, X if s > 1 else X.view(-1), Y)
    assert torch.equal(Y.view(n, qb, s).double(), ref)


def test_mask(lib, torch):
    mask = np.zeros(16, dtype=np.uint8)
    mask[[0, 11, 12, 15]] = 1
    _check(lib, torch, 16, 12, 500, 1100, 10, 2, mask=mask)


def test_streamed_sizes(lib, torch):
    """Past the size from which A is read with non-temporal loads."""
    for s in (3, 20):
        _check(lib, torch, 4, 3, 34000, 2050, s, 2)
