"""Packing and row sums of weights, bit for bit, where the 16-byte loads meet ragged rows: every remainder of K by 16 around the
32-value granule, the 128-value tile and the four tiles a thread packs, odd row counts, and a base address of any alignment."""
import numpy as np
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

from gpu_util import launched, layout_from_canonical

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


@pytest.mark.parametrize("N,K", [(28673, 4100), (43700, 4111), (28673, 4096), (49250, 4111), (24701, 8192)])
def test_large_matrices(N, K):
    """Sizes around those at which the workgroups go along K, and at which the packed weights are streamed."""
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


def test_order_and_stores_by_size_and_width():
    """Along K only where rows are 4, 8, 12 or 16 KB and the matrix is large (other widths were up to 13 % slower that way), streamed only where little of
    the integers would stay in the last-level cache (matrices of 171 to 192 MB were up to 27 % slower streamed)."""
    def kernel(N, K):
        w = torch.zeros((N, K), dtype=torch.int8, device="cuda")
        out = torch.empty(fptq.fptq_packed_bytes(N, K), dtype=torch.uint8, device="cuda")
        return launched(lambda: fptq.fptq_pack_weights(w, out=out))[0]
    plain, along, streamed = kernel(512, 512), kernel(28672, 4096), kernel(39400, 5120)
    assert len({plain, along, streamed, kernel(49200, 4096)}) == 4
    for N, K in ((28672, 4000), (28672, 4352), (18944, 7168), (29312, 6144), (4096, 28672), (6272, 28672), (39200, 5120)):
        assert kernel(N, K) == plain, (N, K)
    for N, K in ((14336, 8192), (9600, 12288), (7200, 16384), (49100, 4096)):
        assert kernel(N, K) == along, (N, K)
