"""The SGEMM's 64 x 64 tile: sizes around its edges, odd k-block counts, split
and unsplit reductions with whole and partial groups of panels, against an FP64
reference (the bound of the emulated SGEMM) and, where both cut the reduction
into the same parts, bit for bit against the streamed split."""
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


# 1 .. 9 k-blocks (odd and even, both sides of a panel), 4 panels (a group of
# three and one more), 12; 64 parts of a long reduction
SHAPES = [(1, 1, 1), (64, 64, 32), (63, 65, 33), (65, 64, 96), (128, 1, 256), (130, 100, 257),
          (257, 259, 300), (1100, 700, 1000), (1024, 1024, 2048), (1000, 1010, 3001),
          (40, 100, 16640), (200, 3000, 1000)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_error_bound(emu, M, N, K):
    A, B = S.make("normal", M + K, (M, K), np.float32), S.make("normal", N + K, (K, N), np.float32)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    C = torch.full((M, N + 1), float("nan"), dtype=torch.float32, device="cuda")
    got = emu.sgemm(dA, dB, C[:, :N]).cpu().numpy().astype(np.float64)
    ref = (dA.double() @ dB.double()).cpu().numpy()
    ab = (dA.double().abs() @ dB.double().abs()).cpu().numpy()
    # omitted products 2^-22, and the FP32 roundings of a panel's six products
    # and of the panel sums, each relative to |A||B|
    cap = 2.0 ** -22 + (6 * 256 + -(-K // 256)) * 2.0 ** -24
    assert np.max(np.abs(got - ref) / np.maximum(ab, 1e-30)) <= cap
    # normwise: the measured 0.5 .. 1.3e-7 with room for the sample (one entry
    # may be off by the rounding of the split and of the sum, 2 x 2^-24 |A||B|)
    assert O.e_F(got, ref) <= (3e-7 if M * N > 100 else cap * ab.max() / np.abs(ref).max())
    assert torch.isnan(C[:, N:]).all()


@pytest.mark.parametrize("M,N,K", [(63, 65, 33), (130, 100, 257), (1500, 1408, 700)])
def test_same_bits_as_streamed(emu, M, N, K):
    A, B = S.make("normal", 5, (M, K), np.float32), S.make("uniform", 6, (K, N), np.float32)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    a = emu.sgemm(dA, dB)
    emu.set_sgemm_split(emu.SGEMM_SPLIT_STREAMED)
    try:
        b = emu.sgemm(dA, dB)
    finally:
        emu.set_sgemm_split(emu.SGEMM_SPLIT_PASS)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("M,N,K", [(119, 69, 14422), (65, 169, 31153), (128, 179, 20992)])
def test_many_splits_keep_the_accuracy(emu, M, N, K):
    """More than 16 parts of the reduction: the error stays at that of 16 (1.25e-7
    .. 1.29e-7 measured there on these sizes, 1.49e-7 .. 1.64e-7 with the parts
    added in one chain, 2^-24 sqrt(parts / 3) being the chain's share)."""
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((M, K), generator=g, device="cuda")
    B = torch.randn((K, N), generator=g, device="cuda")
    ref = A.double() @ B.double()
    e = ((emu.sgemm(A, B).double() - ref).norm() / ref.norm()).item()
    assert e <= 1.38e-7
