"""The panel kernel's persistent workgroups (reductions up to K = 2048, and d = 3
at any length) and the three store paths of the product kernels: whole tiles,
tiles at the edge, and the general one (old C, weights).  More tiles than CUs,
so that workgroups walk several; reductions at both ends of the rules (one
panel, a padded last panel, the last persistent length and the first longer
one); sampled entries, corners included, bit-exact against the oracle."""
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def sample(M, N, seed, n=150):
    rng = np.random.default_rng(seed)
    r = np.concatenate([[0, M - 1, 0, M - 1], rng.integers(0, M, n)]).astype(np.int64)
    c = np.concatenate([[0, 0, N - 1, N - 1], rng.integers(0, N, n)]).astype(np.int64)
    return r, c


def same_bits(a, b):
    return np.array_equal(np.ascontiguousarray(a).view(np.uint64),
                          np.ascontiguousarray(b).view(np.uint64))


# 306 tiles of 128 x 64 (d = 3, 4) or 594 of 64 x 64 (d = 5, 6), ragged in both
@pytest.mark.parametrize("K", [225, 256, 480, 512, 1024, 2048, 2049])
@pytest.mark.parametrize("nprod", [6, 10, 15, 21])
def test_walked_tiles_bit_exact(emu, nprod, K):
    M, N = 2100, 1090
    A = S.make("wide", K + nprod, (M, K), np.float64)
    B = S.make("uniform", K + nprod + 1, (K, N), np.float64)
    r, c = sample(M, N, K)
    ref, st = O.emu_dgemm_entries(A, B, r, c, nprod)
    C = torch.full((M, N + 2), float("nan"), dtype=torch.float64, device="cuda")
    got = emu.dgemm(dev(A), dev(B), nprod, C[:, :N]).cpu().numpy()
    assert st == 0 and same_bits(got[r, c], ref)
    assert torch.isnan(C[:, N:]).all() and not np.isnan(got).any()


# 450 tiles of 128 x 64, 900 of 64 x 64: the panel kernel at every depth, d = 4 too
# (above, its short reductions take fewer rounds on the other kernel); K = 480
# pads to 512
PANELS = (2300, 1540)


@pytest.mark.parametrize("K", [256, 480, 512, 1024])
@pytest.mark.parametrize("nprod", [10, 21])
def test_walked_tiles_by_rounds(emu, nprod, K):
    M, N = PANELS
    A = S.make("wide", K + nprod, (M, K), np.float64)
    B = S.make("uniform", K + nprod + 1, (K, N), np.float64)
    r, c = sample(M, N, K)
    ref, st = O.emu_dgemm_entries(A, B, r, c, nprod)
    got = emu.dgemm(dev(A), dev(B), nprod).cpu().numpy()
    assert st == 0 and same_bits(got[r, c], ref)


# one product count per kernel: 1, 3 (128- and 64-row tiles), 6 .. 21, 26 and up
@pytest.mark.parametrize("M,N,K", [(1024, 1152, 256), (1000, 1100, 300), (300, 70, 300),
                                   (*PANELS, 256)])
@pytest.mark.parametrize("nprod", [1, 3, 6, 10, 15, 21, 36])
def test_store_paths_bit_exact(emu, nprod, M, N, K):
    A = S.make("normal", 3 * nprod, (M, K), np.float64)
    B = S.make("normal", 3 * nprod + 1, (K, N), np.float64)
    C0 = S.make("uniform", 3 * nprod + 2, (M, N), np.float64)
    r, c = sample(M, N, nprod)
    dA, dB = dev(A), dev(B)
    ref, _ = O.emu_dgemm_entries(A, B, r, c, nprod)
    assert same_bits(emu.dgemm(dA, dB, nprod).cpu().numpy()[r, c], ref)
    upd = emu.dgemm_ex(dA, dB, nprod, dev(C0), alpha=-1.5, beta=0.75).cpu().numpy()
    want = (-1.5 * ref) + (0.75 * C0[r, c])
    assert same_bits(upd[r, c], want)
    emu.set_split_scope(emu.SCOPE_ROWCOL)
    try:
        got = emu.dgemm(dA, dB, nprod).cpu().numpy()[r, c]
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
    ref, _ = O.emu_dgemm_entries(A, B, r, c, nprod, scope=O.SCOPE_ROWCOL)
    assert same_bits(got, ref)


@pytest.mark.parametrize("M,N,K", [(384, 256, 300), (385, 257, 300), (100, 90, 2100), (640, 640, 64)])
def test_sgemm_store_paths(emu, M, N, K):
    """The update is applied to the plain call's own product, element by element."""
    A, B = S.make("normal", 1, (M, K), np.float32), S.make("normal", 2, (K, N), np.float32)
    C0 = S.make("uniform", 3, (M, N), np.float32)
    P = emu.sgemm(dev(A), dev(B)).cpu().numpy()
    ref = A.astype(np.float64) @ B.astype(np.float64)
    # entrywise: the FP32 rounding bound of a K-term sum of six products
    bound = 2.0 ** -22 * (np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))) + 1e-30
    assert (np.abs(P - ref) <= bound).all()
    C = torch.full((M, N + 1), float("nan"), dtype=torch.float32, device="cuda")
    C[:, :N] = dev(C0)
    got = emu.sgemm_ex(dev(A), dev(B), C[:, :N], alpha=-1.5, beta=0.75).cpu().numpy()
    assert np.array_equal(got, np.float32(-1.5) * P + np.float32(0.75) * C0)
    assert torch.isnan(C[:, N:]).all()
