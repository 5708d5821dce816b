"""Decodes of codes past the register elimination: one to 54 missing blocks, row
and column tiles with remainders, both Y types, strided and unaligned outputs, a
singular system.

As in the chunk tests the block products are integers from 1 to 7 and the solve
runs in fp64, so a result off by the condition number (under 1e6 here) times a
few 2^-53 rounds to the integer in fp32.  With fp32 Y the parity results are
rounded, 2^-24 of up to 7 k 4 in size, times the condition number: those
compare within that."""
import numpy as np
import pytest

import synth
from tests.gpu_helpers import torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = torch_mod()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def _sets(n, k, m, P, batch, seed):
    """Survivor sets with m missing blocks, the best conditioned of a few draws, in any order."""
    g = np.random.default_rng(seed)
    found = []
    for _ in range(4 * batch):
        miss = np.sort(g.choice(k, m, replace=False))
        par = np.sort(g.choice(n - k, m, replace=False))
        S = np.concatenate([np.setdiff1d(np.arange(k), miss), k + par]).astype(np.int32)
        cond = np.linalg.cond(P[par][:, miss].astype(np.float64)) if m else 1.0
        g.shuffle(S)
        found.append((cond, len(found), S))
    found.sort()
    return np.stack([S for _, _, S in found[:batch]]), found[batch - 1][0]


def _results(P, k, q, s, seed):
    g = np.random.default_rng(seed)
    qb = -(-q // k)
    B = np.zeros((k * qb, s))
    B[:q] = g.integers(1, 8, (q, s))
    Bb = B.reshape(k, qb * s)
    return B[:q], np.concatenate([Bb, P.astype(np.float64) @ Bb]).reshape(-1, qb, s)


# (n, k, m): row tiles of 16, 32 and 64 with and without remainders, an empty
# second half of the rows, the widest accepted system, more than 64 survivors,
# codes without parity workers (k = 128 takes the whole survivor mask)
CODES = [(128, 128, 0), (65, 65, 0), (127, 127, 0), (128, 127, 1), (66, 50, 16), (66, 50, 0), (34, 17, 17),
         (96, 64, 31), (128, 96, 32), (66, 33, 33), (100, 50, 48), (128, 74, 54),
         # systems of up to 64 columns (half the threads), up to 20 survivors, and exactly 64 columns
         (36, 18, 9), (100, 20, 20), (100, 20, 3), (60, 40, 20), (110, 32, 32)]


@pytest.mark.parametrize("n,k,m", CODES)
@pytest.mark.parametrize("rows,s,pad", [(1, 1, 0), (16, 2, 1), (33, 1, 0), (11, 4, 4), (300, 4, 0)])
@pytest.mark.parametrize("batch", [1, 5])
def test_decode_wide(lib, torch, n, k, m, rows, s, pad, batch):
    P = synth.parity_matrix(n, k, 6)
    sets, cond = _sets(n, k, m, P, batch, n + m)
    assert cond < 1e6
    q = max(1, k * rows - (rows > 1) * 3)
    B, Y = _results(P, k, q, s, rows)
    code = lib.Code.systematic(P, 2)
    ref = torch.from_numpy(B.astype(np.float32)).cuda()
    for dt in (torch.float64, torch.float32):
        dY = torch.from_numpy(Y).cuda().to(dt)
        out = torch.full((batch, q, s + pad), -1.0, device="cuda")
        info = torch.full((batch,), 9, dtype=torch.int32, device="cuda")
        lib.coded_decode_batched(code, torch.from_numpy(sets).cuda(), dY, q, out[:, :, :s], info)
        one = torch.full((q, s + pad), -1.0, device="cuda")
        oinfo = torch.full((1,), 9, dtype=torch.int32, device="cuda")
        lib.coded_decode(code, sets[-1], dY, q, one[:, :s], oinfo)
        torch.cuda.synchronize()
        assert torch.all(info == 0) and int(oinfo) == 0
        assert torch.equal(one, out[-1])              # alone as in a batch
        assert torch.all(out[:, :, s:] == -1.0)
        got = out[:, :, :s]
        if dt == torch.float64:
            assert torch.equal(got, ref.expand(batch, q, s))
        else:
            # every rounded result is off by at most 2^-24 of 28 k; the solve
            # multiplies the 2-norm of k of them by the condition number over
            # the smallest column norm, at least 1/2 here
            assert float((got - ref).abs().max()) <= 2.0 ** -24 * 28 * k * 2 * cond * np.sqrt(k)


@pytest.mark.parametrize("n", [65, 128])
@pytest.mark.parametrize("s", [1, 3])
def test_product_without_parity_workers(lib, torch, n, s):
    """coded_matmul with k = n > 64: every worker survives, and the blocks are copied."""
    q, r = 2 * n + 1, 24
    A = torch.from_numpy(synth.integers((q, r), 3, synth.STREAM_A).astype(np.float32)).cuda()
    X = torch.from_numpy(synth.integers((r, s), 3, synth.STREAM_X).astype(np.float32)).cuda()
    ref = A.double() @ X.double()
    X = X.view(-1) if s == 1 else X
    code = lib.Code.systematic(np.zeros((0, n)), 2)
    parity = lib.alloc_parity(code, q, r, torch.float32)
    out = torch.full((q, s) if s > 1 else (q,), -1.0, device="cuda")
    info = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    lib.coded_matmul(code, A, parity, X, out, lib.matmul_workspace(code, A, X), info, 2, 0)
    torch.cuda.synchronize()
    assert int(info) == 0 and torch.equal(out.view(q, s).double(), ref)


@pytest.mark.parametrize("n,k,batch", [(34, 17, 2 ** 23 + 3), (16, 12, 2 ** 24 + 3)])
def test_more_sets_than_one_grid_takes(lib, torch, n, k, batch):
    """One set per workgroup of 512 threads (a wide code) or of 256: more than 2^32 threads."""
    P = synth.integer_parity_matrix(n, k, 3)
    B, Y = _results(P, k, k, 1, 5)
    sets = torch.arange(k, dtype=torch.int32, device="cuda").repeat(batch, 1)
    for b in (0, 2 ** 22 - 1, 2 ** 22, batch - 3, batch - 1):
        sets[b, b % k] = k + int(np.flatnonzero(P[:, b % k])[0])
    sets[batch - 2, 3] = n
    out = torch.full((batch, k), -1.0, device="cuda")
    info = torch.full((batch,), 9, dtype=torch.int32, device="cuda")
    lib.coded_decode_batched(lib.Code.systematic(P, 2), sets, torch.from_numpy(Y).cuda(), k, out, info)
    torch.cuda.synchronize()
    assert int(info[batch - 2]) == -1 and torch.all(out[batch - 2] == -1.0)
    info[batch - 2] = 0
    out[batch - 2] = out[0]
    assert torch.all(info == 0)
    assert torch.equal(out, torch.from_numpy(B[:, 0].astype(np.float32)).cuda().expand(batch, k))


# Blocks of 2^31 - 1 elements (the longest accepted): a copied block and a
# recovered one, single elements and groups of four.
@pytest.mark.parametrize("n,q,s", [(1, 2 ** 31 - 1, 1), (1, 2 ** 29 - 1, 4), (2, 2 ** 31 - 1, 1), (2, 2 ** 29 - 1, 4)])
def test_decode_of_the_longest_blocks(lib, torch, n, q, s):
    code = lib.Code.systematic(np.ones((n - 1, 1)), 2)
    Y = torch.empty((n, q, s), dtype=torch.float32, device="cuda")
    period = (1 << 20) + 7                               # values 0 .. 2^20 + 6, no two chunks alike
    pattern = torch.arange(period, device="cuda", dtype=torch.float32)
    flat = Y[n - 1].view(-1)
    for i in range(0, q * s, period):
        part = flat[i:i + period]
        part.copy_(pattern[:part.numel()])
    if n == 2:
        Y[0].fill_(-2.0)
    out = torch.full((q, s), -1.0, device="cuda")
    info = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    lib.coded_decode(code, [n - 1], Y, q, out, info)
    torch.cuda.synchronize()
    assert int(info) == 0
    assert torch.equal(out, Y[n - 1])


@pytest.mark.parametrize("n,k,m", [(96, 64, 20), (128, 96, 32)])
def test_singular_wide_set(lib, torch, n, k, m):
    """Two equal parity rows: a zero pivot, reported, and nothing written; its neighbours in the batch decode."""
    P = synth.integer_parity_matrix(n, k, 3).astype(np.float64)
    P[4] = P[3]
    g = np.random.default_rng(1)
    miss = np.sort(g.choice(k, m, replace=False))
    bad = np.concatenate([np.setdiff1d(np.arange(k), miss), k + np.arange(m)]).astype(np.int32)
    good = np.concatenate([np.setdiff1d(np.arange(k), miss[:1]), [k]]).astype(np.int32)
    P[0, miss[0]] = 2.0
    q, s = 7 * k, 2
    B, Y = _results(P, k, q, s, 2)
    out = torch.full((3, q, s), -1.0, device="cuda")
    info = torch.zeros(3, dtype=torch.int32, device="cuda")
    sets = torch.from_numpy(np.stack([good, bad, good])).cuda()
    lib.coded_decode_batched(lib.Code.systematic(P, 2), sets, torch.from_numpy(Y).cuda(), q, out, info)
    torch.cuda.synchronize()
    assert info[0] == 0 and info[2] == 0 and k - m < int(info[1]) <= k
    ref = torch.from_numpy(B.astype(np.float32)).cuda()
    assert torch.equal(out[0], ref) and torch.equal(out[2], ref)
    assert torch.all(out[1] == -1.0)
