"""Packing and row sums of weights, bit for bit, where the 16-byte loads meet ragged rows: every remainder of K by 16 around the
32-value granule, the 128-value tile and the four tiles a thread packs, odd row counts, and a base address of any alignment."""
import numpy as np
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

from gpu_util import layout_from_canonical

pytestmark = pytest.mark.gpu


def canonical(w):
    rows, K = w.shape
    padded = np.zeros((rows, K + K % 2), np.int8)
    padded[:, :K] = w
    u = padded.view(np.uint8) & 15
    return u[:, 0::2] | (u[:, 1::2] << 4)


@pytest.mark.parametrize("N,K", [(1, 1), (3, 15), (65, 16), (64, 17), (63, 31), (17, 33), (5, 127), (130, 128), (66, 129), (7, 500), (64, 511), (65, 512),
                                 (2, 513), (70, 1040), (9, 4095), (12, 4112), (4, 5001)])
@pytest.mark.parametrize("offset", [0, 1, 7])
def test_pack_and_row_sums(N, K, offset):
    rng = np.random.default_rng(N * 7 + K)
    w = rng.integers(-8, 8, size=(N, K), dtype=np.int8)
    base = torch.full((N * K + offset + 64,), 127, dtype=torch.int8, device="cuda")       # what lies around the matrix must not show
    wd = base[offset:offset + N * K].view(N, K)
    wd.copy_(torch.from_numpy(w))
    got = fptq.fptq_pack_weights(wd).cpu().numpy()
    assert np.array_equal(got, layout_from_canonical(canonical(w), N, K))
    assert np.array_equal(fptq.fptq_weight_row_sums(wd).cpu().numpy(), w.sum(axis=1, dtype=np.int32))


@pytest.mark.parametrize("N,K", [(28673, 4100), (43700, 4111)])
def test_large_matrices(N, K):
    """Sizes at which the workgroups go along K, and at which the packed weights are streamed."""
    torch.manual_seed(N)
    w = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda")
    kt = (K + 127) // 128
    codes = torch.zeros((N, kt * 128), dtype=torch.uint8, device="cuda")
    codes[:, :K] = w.view(torch.uint8) & 15
    want = (codes[:, 0::2] | (codes[:, 1::2] << 4)).view(N, kt, 64).transpose(0, 1).contiguous().view(-1)
    assert torch.equal(fptq.fptq_pack_weights(w), want)
    assert torch.equal(fptq.fptq_weight_row_sums(w), w.sum(dim=1, dtype=torch.int32))


def test_row_sums_of_full_bytes():
    """Row sums take the int8 as it is, not its low nibble."""
    w = torch.arange(-128, 128, dtype=torch.int16).to(torch.int8).repeat(3, 5)[:, :1237].contiguous().cuda()
    assert torch.equal(fptq.fptq_weight_row_sums(w).cpu(), w.cpu().sum(dim=1, dtype=torch.int32))
