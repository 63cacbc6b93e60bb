"""The INT8 tiles' unrolled K loops at every remainder: each tile shape, and the split over workgroups, against the simple kernel; and both sides of the
lines between the few-token kernel and the tiles."""
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

pytestmark = pytest.mark.gpu


def operands(M, N, K):
    torch.manual_seed(K)
    x, w = (torch.randint(-8, 8, (n, K), dtype=torch.int8, device="cuda") for n in (M, N))
    return fptq.fptq_pack_weights(x), fptq.fptq_pack_weights(w), torch.rand(N, device="cuda") * 0.015 + 0.005


# up to four K groups, each unrolled by up to four K tiles: 1 to 33 K tiles reach every remainder of every group after no, one and two whole turns
@pytest.mark.parametrize("tile", range(1, 9))
@pytest.mark.parametrize("first", [1, 9, 17, 25])
def test_every_remainder_of_every_tile(tile, first):
    M, N = 70, 200
    for tiles in range(first, first + 8 + (first == 25)):
        K = tiles * 128 - (tiles % 3) * 37
        xq, wq, s_w = operands(M, N, K)
        y_ref, a_ref = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 0.37, s_w, want_acc=True)
        fptq.fptq_set_gemm_tile(tile)
        try:
            y, a = fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.37, s_w, want_acc=True)
        finally:
            fptq.fptq_set_gemm_tile(0)
        assert torch.equal(a, a_ref) and torch.equal(y.view(torch.int16), y_ref.view(torch.int16)), (tile, K)


@pytest.mark.parametrize("tiles", range(48, 66, 2))
def test_split_over_workgroups(tiles):
    M, N, K = 70, 200, tiles * 128 - 5
    xq, wq, s_w = operands(M, N, K)
    nbytes = fptq.fptq_linear_workspace_bytes(M, N, K)
    assert nbytes > 0
    y_ref, a_ref = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 0.37, s_w, want_acc=True)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        y, a = fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, 0.37, s_w, ws, want_acc=True)
        assert torch.equal(a, a_ref) and torch.equal(y.view(torch.int16), y_ref.view(torch.int16))


@pytest.mark.parametrize("M,N,K", [(33, 8192, 300), (33, 8193, 300), (64, 8200, 2100), (47, 10239, 1000), (16, 12296, 640), (17, 12288, 640), (17, 12289, 640),
                                   (32, 12400, 1920), (32, 12400, 1921), (25, 33001, 100)])
def test_both_sides_of_the_few_token_lines(M, N, K):
    xq, wq, s_w = operands(M, N, K)
    d = torch.rand(M, device="cuda") + 0.5
    y_ref, a_ref = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 0.37, s_w, d, want_acc=True)
    y, a = fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.37, s_w, d, want_acc=True)
    assert torch.equal(a, a_ref) and torch.equal(y.view(torch.int16), y_ref.view(torch.int16))
    assert torch.equal(fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.37, s_w, d).view(torch.int16), y_ref.view(torch.int16))
    wsum = torch.randint(-500, 500, (N,), dtype=torch.int32, device="cuda")
    y, a = fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.37, s_w, 3, wsum, d, want_acc=True)
    want = ((a_ref - 3 * wsum).float() * (s_w * 0.37) * d[:, None]).to(torch.bfloat16)        # the epilogue's products in their order, each rounded
    assert torch.equal(a, a_ref) and torch.equal(y, want)
