"""The passes of the FP64 split where their work distribution changes: operands
with fewer and with more work items than the launches have blocks, rows read
one by one and as one run of memory, and exponent chains that are wrong from a
chosen level on (replayed for one operand only, or for both at different
levels).  Slices, chains, status and products bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import seeded_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_04663_amd as E
    E.lib()
    return E


def chain_operand(shape, right, gap, seed):
    """Entries m 2^-e, 7-bit m, e from classes: the first `right` levels follow
    the speculated 9 bits per level, every later one lies `gap` bits below."""
    rng = np.random.default_rng(seed)
    off = np.cumsum([0] + [9] * (right - 1) + [gap] * (6 - right))
    cls = rng.integers(0, 6, shape)
    # (a class of mantissas with 8 significant bits leaves no residual, so each
    # class is a level of its own)
    x = (1.0 + rng.integers(0, 128, shape) / 128.0) * np.exp2(-off[cls].astype(np.float64))
    return np.where(rng.integers(0, 2, shape) == 1, -x, x)


# 64 x 32 items: 1 and 6 (one block each), 1155 (more than the 1024 blocks of
# the pass and the 512 units of a replay)
SHAPES = [(1, 1), (70, 65), (2100, 1101)]


@pytest.mark.parametrize("contiguous", [True, False])
@pytest.mark.parametrize("as_b", [0, 1])
@pytest.mark.parametrize("right,gap", [(6, 9), (1, 22), (3, 14), (5, 30)])
@pytest.mark.parametrize("shape", SHAPES)
def test_split_bit_exact(emu, shape, right, gap, as_b, contiguous):
    X = chain_operand(shape, right, gap, 31 * right + gap)
    if right == 6:
        X = S.make("wide", 77, shape, np.float64)
    big = torch.zeros((shape[0], shape[1] + (0 if contiguous else 3)), dtype=torch.float64)
    big[:, :shape[1]] = torch.from_numpy(X)
    d = big.cuda()[:, :shape[1]]
    emu.domain_status()
    ref, v, _, st = O.split_f64(X)
    s, vg = emu.split_f64(d, as_b=bool(as_b))
    assert np.array_equal(vg.cpu().numpy(), v)
    assert np.array_equal(s.cpu().numpy().view(np.uint16), ref)
    assert emu.domain_status() == st


@pytest.mark.parametrize("nprod", [3, 15, 21])
@pytest.mark.parametrize("ra,rb", [(1, 6), (6, 2), (4, 2)])
@pytest.mark.parametrize("M,N,K", [(40, 50, 60), (700, 130, 1500)])
def test_dgemm_with_replays_bit_exact(emu, M, N, K, ra, rb, nprod):
    A = chain_operand((M, K), ra, 13, 5) if ra < 6 else S.make("normal", 5, (M, K), np.float64)
    B = chain_operand((K, N), rb, 14, 6) if rb < 6 else S.make("normal", 6, (K, N), np.float64)
    rng = np.random.default_rng(M + nprod)
    r = np.concatenate([[0, M - 1], rng.integers(0, M, 60)]).astype(np.int64)
    c = np.concatenate([[0, N - 1], rng.integers(0, N, 60)]).astype(np.int64)
    ref, st = O.emu_dgemm_entries(A, B, r, c, nprod)
    emu.domain_status()
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    for _ in range(2):      # the second call finds the first one's state and planes
        C = emu.dgemm(dA, dB, nprod).cpu().numpy()
        got = np.ascontiguousarray(C[r, c])
        assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
    assert emu.domain_status() == st


def test_subnormal_slices_exceed_the_chain(emu):
    """Near the lower end of the domain the slices are subnormal and rounded
    coarser than the projection, so a residual can be larger than the chain
    speculated.  One k-block's work item shows such a residual (2^-134 at level
    2), others have exactly the speculated maximum of one level each."""
    X = np.zeros((64, 192))
    X[:2, 0] = [2.0 ** -121 + 2.0 ** -138, 2.0 ** -120]
    X[0, 32] = 2.0 ** -121 + 1.5 * 2.0 ** -130
    X[0, 64] = 2.0 ** -121 + 2.0 ** -134
    X[0, 96] = 2.0 ** -121 + 2.0 ** -147
    X[0, 128] = 2.0 ** -121 + 2.0 ** -156
    X[0, 160] = 2.0 ** -121 + 2.0 ** -165
    ref, v, _, st = O.split_f64(X)
    assert list(v[:3]) == [-120, -129, -134] and st == O.ST_SUBNORMAL
    for as_b in (0, 1):
        emu.domain_status()
        s, vg = emu.split_f64(torch.from_numpy(X.T.copy() if as_b else X).cuda(), as_b=bool(as_b))
        s = s.cpu().numpy().view(np.uint16)
        assert np.array_equal(vg.cpu().numpy(), v)
        assert np.array_equal(s.transpose(0, 2, 1) if as_b else s, ref)
        assert emu.domain_status() == st


@pytest.mark.parametrize("zero_from", [1, 2, 4])
def test_identically_zero_levels(emu, zero_from):
    """Integers of 8 zero_from bits leave nothing for the levels after those."""
    n = 8 * zero_from
    rng = np.random.default_rng(n)
    X = rng.integers(-2 ** n, 2 ** n, (130, 1101)).astype(np.float64)
    X[5, 7] = 2.0 ** n
    ref, v, _, st = O.split_f64(X)
    s, vg = emu.split_f64(torch.from_numpy(X).cuda())
    zero = np.iinfo(np.int32).min
    assert v[zero_from - 1] > zero and (v[zero_from:] == zero).all()
    assert np.array_equal(vg.cpu().numpy(), v)
    assert np.array_equal(s.cpu().numpy().view(np.uint16), ref)
