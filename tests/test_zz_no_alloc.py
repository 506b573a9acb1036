"""The allocation-free entry point emu_dgemm_noalloc against emu_dgemm.

Called through the C ABI (ctypes) with torch-owned device buffers: the result
must be bit-identical to emu_dgemm's on the same inputs, on consecutive calls
that share the fixed scratch (the second one smaller, so stale planes of the
first call sit beyond what it reads), without the library's workspace ever
being allocated; sizes beyond the scratch are refused before any launch, and
the status word of the scratch reaches emu_domain_status.
"""
import ctypes

import numpy as np
import pytest
import torch

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


def noalloc(emu, A, B, C, nprod):
    """emu_dgemm_noalloc through the C ABI on the current stream."""
    L = emu.lib()
    M, K = A.shape
    N = B.shape[1]
    L.emu_set_stream(ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    return L.emu_dgemm_noalloc(M, N, K, A.data_ptr(), A.stride(0), B.data_ptr(), B.stride(0),
                               C.data_ptr(), C.stride(0), nprod)


@pytest.mark.parametrize("nprod", [6, 21])
def test_noalloc_matches_dgemm_on_consecutive_calls(emu, nprod):
    emu.release_workspace()
    shapes = [(700, 650, 900), (130, 70, 300)]          # the second call is smaller
    outs = []
    for i, (M, N, K) in enumerate(shapes):
        A = dev(S.make("wide", 901 + 2 * i, (M, K), np.float64))
        B = dev(S.make("uniform", 902 + 2 * i, (K, N), np.float64))
        C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
        assert noalloc(emu, A, B, C, nprod) == emu.EMU_OK, emu.lib().emu_last_error()
        torch.cuda.synchronize()
        assert emu.workspace_bytes() == 0                # nothing was allocated
        outs.append((A, B, C.cpu().numpy()))
    assert emu.domain_status() == 0
    for A, B, got in outs:
        ref = emu.dgemm(A, B, nprod).cpu().numpy()
        assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))


def test_noalloc_padded_leading_dimensions(emu):
    M, N, K = 257, 129, 513
    A = dev(np.pad(S.make("wide", 911, (M, K), np.float64), ((0, 0), (0, 7))))[:, :K]
    B = dev(np.pad(S.make("wide", 912, (K, N), np.float64), ((0, 0), (0, 3))))[:, :N]
    C = torch.zeros((M, N + 5), dtype=torch.float64, device="cuda")
    assert noalloc(emu, A, B, C[:, :N], 15) == emu.EMU_OK
    ref = emu.dgemm(A, B, 15).cpu().numpy()
    assert np.array_equal(C[:, :N].cpu().numpy(), ref)
    assert not C[:, N:].cpu().numpy().any()              # nothing written past N


def test_noalloc_refuses_sizes_beyond_the_scratch(emu):
    L = emu.lib()
    P = ctypes.c_void_p(0x1000)                          # never dereferenced
    assert L.emu_dgemm_noalloc(4096, 4096, 4096, P, 4096, P, 4096, P, 4096, 21) == emu.EMU_ENOMEM
    assert b"scratch" in L.emu_last_error()
    assert L.emu_dgemm_noalloc(4, 4, 4, P, 4, P, 4, P, 4, 7) == emu.EMU_EINVAL


# fit the scratch in the packing of the other kernels, not in the panel kernel's
# whole panels (10, 25 and 32 k-blocks) or taller tiles
@pytest.mark.parametrize("M,N,K,nprod", [(6408, 6408, 320, 15), (3144, 3144, 800, 15),
                                         (3848, 3848, 1000, 10)])
def test_noalloc_short_reductions_near_the_scratch(emu, M, N, K, nprod):
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((M, K), generator=g, device="cuda", dtype=torch.float64)
    B = torch.randn((K, N), generator=g, device="cuda", dtype=torch.float64)
    C = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    assert noalloc(emu, A, B, C, nprod) == emu.EMU_OK, emu.lib().emu_last_error()
    ref = emu.dgemm(A, B, nprod)              # the panel kernel, on the workspace
    assert torch.equal(C.view(torch.int64), ref.view(torch.int64))
    emu.release_workspace()


@pytest.mark.parametrize("scope", ["SCOPE_OPERAND", "SCOPE_KBIN"])
def test_workspace_limit_leaves_the_panel_kernel(emu, monkeypatch, scope):
    """A short reduction whose panel packing exceeds EMU_WORKSPACE_LIMIT runs on
    the other kernels, with the same bits; a longer one is refused."""
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randn((1600, 300), generator=g, device="cuda", dtype=torch.float64)
    B = torch.randn((300, 1600), generator=g, device="cuda", dtype=torch.float64)
    L = torch.randn((1600, 1100), generator=g, device="cuda", dtype=torch.float64)
    emu.set_split_scope(getattr(emu, scope))
    try:
        emu.release_workspace()
        ref = emu.dgemm(A, B, 15)
        panels = emu.workspace_bytes()
        emu.release_workspace()
        monkeypatch.setenv("EMU_WORKSPACE_LIMIT", str(panels - 1))
        got = emu.dgemm(A, B, 15)
        plain = emu.workspace_bytes()
        assert 0 < plain < panels
        assert torch.equal(got.view(torch.int64), ref.view(torch.int64))
        emu.release_workspace()
        monkeypatch.setenv("EMU_WORKSPACE_LIMIT", str(plain - 1))
        with pytest.raises(emu.EmuError):
            emu.dgemm(A, B, 15)
        monkeypatch.delenv("EMU_WORKSPACE_LIMIT")
        emu.dgemm(L, L.T.contiguous(), 15)
        long = emu.workspace_bytes()
        emu.release_workspace()
        monkeypatch.setenv("EMU_WORKSPACE_LIMIT", str(long - 1))
        with pytest.raises(emu.EmuError):
            emu.dgemm(L, L.T.contiguous(), 15)
    finally:
        emu.set_split_scope(emu.SCOPE_OPERAND)
        emu.release_workspace()


def test_noalloc_reports_status(emu):
    A = dev(np.ldexp(S.make("uniform", 921, (60, 300), np.float64), -45))
    B = dev(np.ldexp(S.make("uniform", 922, (300, 40), np.float64), -45))
    C = torch.empty((60, 40), dtype=torch.float64, device="cuda")
    emu.domain_status()
    assert noalloc(emu, A, B, C, 21) == emu.EMU_OK
    assert emu.domain_status() == emu.STATUS_INEXACT
    assert noalloc(emu, A, B, C, 6) == emu.EMU_OK
    assert emu.domain_status() == 0
