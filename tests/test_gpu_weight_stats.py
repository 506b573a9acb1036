"""Weights, range check and class lists made from one reading of the operands:
rows whose entries underflow when scaled (to an exact zero, which is in the
domain, or to a subnormal, which is not), extents around the passes' slices, and
reductions around the list kernel's runs; against the oracle's scaled and
K-binned forms, bit for bit."""
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
    yield E
    E.set_split_scope(E.SCOPE_OPERAND)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bits(a):
    return np.ascontiguousarray(a).view(np.uint64)


ROWS = {
    "plain": [1.0, 0.5, 2.0 ** -100],
    "zero_only": [2.0 ** 1000, 2.0 ** -100, 1.5 * 2.0 ** 999],         # underflows to 0
    "zero_and_subnormal": [2.0 ** 1000, 2.0 ** -100, 2.0 ** -60],       # 2^-1060: out of range
    "zero_and_small": [2.0 ** 1000, 2.0 ** -100, 2.0 ** 800],           # 2^-200: out of range
    "small": [2.0 ** 300, 2.0 ** 170, 1.0],                             # 2^-130 and 2^-300
    "edge": [2.0 ** 126, 1.0, 2.0 ** 50],                               # exactly 2^-126
    "empty": [0.0, 0.0, 0.0],
}


@pytest.mark.parametrize("as_b", [0, 1])
@pytest.mark.parametrize("kind", list(ROWS))
def test_scaled_split_status(emu, kind, as_b):
    X = S.make("uniform", 9, (70, 130), np.float64)
    X[7, :] = 0.0
    X[7, [3, 64, 129]] = ROWS[kind]
    s = O.scale_exponents(X)
    ref, v, _, st = O.split_f64(np.ldexp(X, -s[:, None]))
    emu.set_split_scope(emu.SCOPE_ROWCOL)
    try:
        emu.domain_status()
        got, vg = emu.split_f64(dev(X.T if as_b else X), as_b=bool(as_b))
        status = emu.domain_status()
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    g = got.cpu().numpy().view(np.uint16)
    assert status == st
    assert np.array_equal(vg.cpu().numpy(), v)
    assert np.array_equal(g.transpose(0, 2, 1) if as_b else g, ref)


@pytest.mark.parametrize("ta,tb", [("N", "N"), ("T", "T")])
@pytest.mark.parametrize("K", [1, 63, 65, 257, 1024, 1025, 4500])
def test_kbin_lists(emu, K, ta, tb):
    """Classes mixed along the reduction, some indices left out."""
    M, N = 70, 66
    rng = np.random.default_rng(K)
    A, B = S.make("normal", K, (M, K), np.float64), S.make("normal", K + 1, (K, N), np.float64)
    B *= np.exp2(rng.integers(0, 8, K) * -9.0)[:, None]
    A[:, rng.integers(0, K, 1 + K // 50)] = 0.0
    if K == 1:
        A[:] = 1.0
    r, c = rng.integers(0, M, 60), rng.integers(0, N, 60)
    ref, _ = O.emu_dgemm_entries(A, B, r, c, 10, scope=O.SCOPE_KBIN)
    emu.set_split_scope(emu.SCOPE_KBIN)
    try:
        C = emu.dgemm_ex(dev(A.T if ta == "T" else A), dev(B.T if tb == "T" else B), 10,
                         transa=ta, transb=tb).cpu().numpy()
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    assert np.array_equal(bits(C[r, c]), bits(ref))


# 64-row slices and 256-thread rows of the statistics, weights of more than 256 x 256 rows
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (65, 64, 63), (3, 1030, 1025), (66000, 3, 5), (4, 66000, 70)])
def test_rowcol_extents(emu, M, N, K):
    A, B = S.make("wide", 3, (M, K), np.float64), S.make("wide", 4, (K, N), np.float64)
    rng = np.random.default_rng(M)
    r = np.concatenate([[0, M - 1], rng.integers(0, M, 60)])
    c = np.concatenate([[0, N - 1], rng.integers(0, N, 60)])
    ref, st = O.emu_dgemm_entries(A, B, r, c, 15, scope=O.SCOPE_ROWCOL)
    emu.set_split_scope(emu.SCOPE_ROWCOL)
    try:
        emu.domain_status()
        C = emu.dgemm(dev(A), dev(B), 15).cpu().numpy()
        assert emu.domain_status() == st
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    assert np.array_equal(bits(C[r, c]), bits(ref))


@pytest.mark.parametrize("as_b", [0, 1])
@pytest.mark.parametrize("low", [2.0 ** -60, 2.0 ** 800, None])
def test_underflowing_rows_far_apart(emu, low, as_b):
    """A row that underflows in one block's share, the entry below the domain in
    another's: the whole operand is looked through, in one pass."""
    X = S.make("uniform", 10, (600, 2100), np.float64)
    X[[7, 597]] = 0.0
    X[7, [0, 9]] = [2.0 ** 1000, 2.0 ** -100]
    X[597, [3, 64, 2099]] = [2.0 ** 1000, 2.0 ** -100, low or 2.0 ** 990]
    ref, v, _, st = O.split_f64(np.ldexp(X, -O.scale_exponents(X)[:, None]))
    assert bool(st & O.ST_RANGE) == (low is not None)
    emu.set_split_scope(emu.SCOPE_ROWCOL)
    try:
        emu.domain_status()
        got, vg = emu.split_f64(dev(X.T if as_b else X), as_b=bool(as_b))
        assert emu.domain_status() == st
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    g = got.cpu().numpy().view(np.uint16)
    assert np.array_equal(vg.cpu().numpy(), v)
    assert np.array_equal(g.transpose(0, 2, 1) if as_b else g, ref)


@pytest.mark.parametrize("which", ["A", "B"])
def test_underflowing_row_costs_no_walk(emu, which):
    """One subnormal entry among ordinary ones: the call takes about as long as
    without it (twice is far above what the timer varies by; one thread walking
    the row of 16384 entries took ten times as long)."""
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn((256, 16384), generator=g, device="cuda", dtype=torch.float64)
    B = torch.randn((16384, 256), generator=g, device="cuda", dtype=torch.float64)

    def ms():
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        t = []
        for _ in range(9):
            ev[0].record()
            emu.dgemm(A, B, 6)
            ev[1].record()
            ev[1].synchronize()
            t.append(ev[0].elapsed_time(ev[1]))
        return sorted(t)[4]
    emu.set_split_scope(emu.SCOPE_ROWCOL)
    try:
        plain = ms()
        X = A if which == "A" else B
        X[37, 101] = 5e-324
        X[37 if which == "A" else 3, 102 if which == "A" else 101] = 5.0
        walked = ms()
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    assert walked < 2.0 * plain, (plain, walked)
