"""Decodes at the edges of the copying of systematic survivors (chunks of up to
128 four-element items in one sequence, longer ones block by block), with worker
masks past 64 bits, strided outputs and invalid sets in a batch.

The block products are integers from 1 to 7 and the solve runs in fp64, so its
result, off by the system's condition number (under 1e6 here) times a few 2^-53,
rounds to exactly the integer in fp32."""
import math

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


def _case(lib, torch, n, k, q, s, batch, pad):
    P = synth.parity_matrix(n, k, 4)
    g = np.random.default_rng(q + s)
    qb = -(-q // k)
    B = np.zeros((k * qb, s))
    B[:q] = g.integers(1, 8, (q, s))
    Bb = B.reshape(k, qb * s)
    Y = np.concatenate([Bb, P.astype(np.float64) @ Bb]).reshape(n, qb, s)
    sets, _ = lib.coded_draw_survivor_sets(n, k, 9, min(3 * batch, math.comb(n, k)))
    cond = []
    for S in sets:
        par = [w - k for w in S if w >= k]
        miss = sorted(set(range(k)) - set(S.tolist()))
        cond.append(np.linalg.cond(P[par][:, miss].astype(np.float64)) if miss else 1.0)
    sets = sets[np.resize(np.argsort(cond, kind="stable")[:batch], batch)].copy()
    for S in sets:
        g.shuffle(S)
    return lib.Code.systematic(P, 2), B[:q], sets, torch.from_numpy(Y).cuda(), torch.full((batch, q, s + pad), -1.0, device="cuda")


# (n, k, q, s): one row per block; 16, 127, 128 and 129 items of four elements per chunk; several chunks; wide masks
SHAPES = [(5, 3, 3, 4), (25, 23, 23 * 16 - 5, 4), (32, 24, 24 * 64 - 1, 8), (16, 12, 12 * 127, 4), (16, 12, 12 * 128, 4),
          (16, 12, 12 * 129 - 7, 4), (64, 48, 48 * 300 - 11, 8), (96, 64, 64 * 20 - 3, 4), (128, 96, 96 * 9, 4),
          (70, 60, 60 * 200 - 1, 8), (10, 8, 1001, 3)]


@pytest.mark.parametrize("n,k,q,s", SHAPES)
@pytest.mark.parametrize("batch,pad", [(1, 0), (7, 4), (1100, 0)])
def test_decode_chunks(lib, torch, n, k, q, s, batch, pad):
    if batch > 1000 and q * s * batch > 3e7:
        pytest.skip("batch too large for this shape")
    code, B, sets, Y, out = _case(lib, torch, n, k, q, s, batch, pad)
    info = torch.full((batch,), 9, dtype=torch.int32, device="cuda")
    view = out[:, :, :s]
    lib.coded_decode_batched(code, torch.from_numpy(sets).cuda(), Y, q, view, info)
    torch.cuda.synchronize()
    assert torch.all(info == 0)
    ref = torch.from_numpy(B.astype(np.float32)).cuda()
    assert torch.equal(view, ref.expand(batch, q, s))
    assert torch.all(out[:, :, s:] == -1.0)
    if batch == 7:
        one = torch.zeros((q, s), device="cuda")
        lib.coded_decode(code, sets[3], Y, q, one, info[:1])
        torch.cuda.synchronize()
        assert torch.equal(one, ref)


@pytest.mark.parametrize("n,k", [(16, 12), (64, 48), (128, 96)])
def test_invalid_sets_in_a_batch(lib, torch, n, k):
    q, s = 5 * k, 4
    code, B, sets, Y, out = _case(lib, torch, n, k, q, s, 6, 0)
    sets[1, 0] = n
    sets[2, 3] = -1
    sets[4, 1] = sets[4, 2]
    info = torch.zeros(6, dtype=torch.int32, device="cuda")
    lib.coded_decode_batched(code, torch.from_numpy(sets).cuda(), Y, q, out, info)
    torch.cuda.synchronize()
    assert info.tolist() == [0, -1, -1, 0, -1, 0]
    ref = torch.from_numpy(B.astype(np.float32)).cuda()
    for b in range(6):
        assert torch.equal(out[b], ref if b in (0, 3, 5) else torch.full_like(ref, -1.0))


# Outputs whose rows lie one after another, taken four at a time at any
# alignment: blocks of 1 to 3 elements past a group, odd totals (whose last pair
# would start inside Y and end past it), several chunks, a last block with no
# and with few rows in A.
@pytest.mark.parametrize("n,k,q,s", [(16, 12, 12 * 5, 1), (16, 12, 12 * 7 - 1, 1), (25, 23, 23 * 65 - 22, 1),
                                     (64, 48, 48 * 131, 1), (64, 48, 48 * 43 - 5, 3), (20, 16, 16 * 1027 - 3, 1),
                                     (32, 24, 24 * 37 - 23, 5), (10, 8, 9, 6), (44, 33, 33 * 9 - 1, 7)])
@pytest.mark.parametrize("batch,shift,f32", [(2, 0, False), (2, 1, True), (7, 3, False), (1100, 2, False)])
def test_decode_flat(lib, torch, n, k, q, s, batch, shift, f32):
    if batch > 1000 and q * s * batch > 3e7:
        pytest.skip("batch too large for this shape")
    code, B, sets, Y, _ = _case(lib, torch, n, k, q, s, batch, 0)
    if f32:
        # integer parity rows keep the results whole numbers below 2^24
        P = synth.integer_parity_matrix(n, k, 5)
        keep = [np.sort(S) for S in sets]
        sets = np.stack([S if np.linalg.matrix_rank(np.vstack([np.eye(k), P])[S]) == k else
                         np.arange(k, dtype=np.int32) for S in keep])
        code = lib.Code.systematic(P, 2)
        Bb = np.zeros((k * -(-q // k), s))
        Bb[:q] = B
        Bb = Bb.reshape(k, -1)
        Y = torch.from_numpy(np.concatenate([Bb, np.asarray(P, np.float64) @ Bb]).reshape(n, -1, s)).cuda().float()
    whole = torch.full((batch * q * s + shift + 8,), -1.0, device="cuda")
    view = whole[shift:shift + batch * q * s].view(batch, q, s)
    info = torch.full((batch,), 9, dtype=torch.int32, device="cuda")
    lib.coded_decode_batched(code, torch.from_numpy(sets).cuda(), Y, q, view, info)
    torch.cuda.synchronize()
    assert torch.all(info == 0)
    ref = torch.from_numpy(B.astype(np.float32)).cuda()
    assert torch.equal(view, ref.expand(batch, q, s))
    assert torch.all(whole[:shift] == -1.0) and torch.all(whole[shift + batch * q * s:] == -1.0)
