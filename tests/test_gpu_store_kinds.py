"""What a call without accumulators stores: such calls run other instances of the matrix kernels than calls that ask for the accumulators, one per way of
storing the rows (whole 64-byte pieces streamed, other multiples of eight channels cached, any width).  Every tile of both kernels, forced, with and
without a zero point, into NaNs, at the address of the allocation and 16 bytes past it, against the same layer in PyTorch: integers in fp64 (exact),
the fp32 epilogue operation by operation."""
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

pytestmark = pytest.mark.gpu

# two tiles and a part in each direction, the last channels in the middle of every tile's run of a wave
WIDTHS = [(300, 544), (300, 552), (300, 547), (140, 32), (130, 8), (129, 1)]
# INT8 tiles by number, the split over K, six-bit tiles by tokens
TILES = [1, 2, 3, 4, 5, 6, 7, 8, "split", 128, 192, 256]
_operands = {}


def layer(M, N, K):
    """Operands of a layer, its integers, and y(zero_point, d) in fp32 as the library defines it."""
    if (M, N, K) not in _operands:
        torch.manual_seed(M * 7 + N)
        x, w = (torch.randint(-8, 8, (rows, K), dtype=torch.int8, device="cuda") for rows in (M, N))
        s_w, d = torch.rand(N, device="cuda") * 0.015 + 0.005, torch.rand(M, device="cuda") + 0.5
        _operands[M, N, K] = (fptq.fptq_pack_weights(x), fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w), s_w, d,
                              (x.double() @ w.double().t().contiguous()).to(torch.int32))
    return _operands[M, N, K]


def expected(acc, wsum, s_a, s_w, zp, d):
    y = (acc - zp * wsum).float() * (torch.tensor(s_a, device="cuda") * s_w)
    return (y if d is None else y * d[:, None]).to(torch.bfloat16)


@pytest.fixture(scope="module", autouse=True)
def operands_given_back():
    yield
    _operands.clear()


@pytest.fixture
def unforced():
    yield
    fptq.fptq_set_gemm_tile(0)
    fptq.fptq_set_linear_prefill(0)


def call(tile, M, N, K, operands, s_a, zp, d, out):
    xq, wq, wsum, s_w, _, _ = operands
    if tile == "split":
        ws = torch.zeros(fptq.fptq_linear_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
        assert ws.numel()
        return fptq.fptq_w4a4_linear_ws(xq, wq, M, N, K, s_a, s_w, ws, d, out=out)
    if tile < 128:
        fptq.fptq_set_gemm_tile(tile)
        if zp is None:
            return fptq.fptq_w4a4_linear(xq, wq, M, N, K, s_a, s_w, d, out=out)
        return fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, s_a, s_w, zp, wsum, d, out=out)
    fptq.fptq_set_linear_prefill(tile)
    assert fptq.fptq_linear_launch_plan(M, N, K, with_scratch=True)[0] == "linear_prefill_kernel"
    scratch = torch.full((fptq.fptq_linear_scratch_bytes(M, N, K),), 0xFF, dtype=torch.uint8, device="cuda")
    return fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, s_a, s_w, scratch, *((0, None) if zp is None else (zp, wsum)), d, out=out)


@pytest.mark.parametrize("M,N", WIDTHS)
@pytest.mark.parametrize("tile", TILES)
def test_every_tile_and_store(unforced, tile, M, N):
    K = 6300 if tile == "split" else 700
    operands = layer(M, N, K)
    _, _, wsum, s_w, d, acc = operands
    for zp in (None,) if tile == "split" else (None, -8, 3):
        for dd in (None, d):
            want = expected(acc, wsum, 0.37, s_w, zp or 0, dd)
            for offset in (0, 8):
                buf = torch.full((offset + M * N + 64 * N + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
                out = buf[offset:offset + M * N].view(M, N)
                y = call(tile, M, N, K, operands, 0.37, zp, dd, out)
                assert y.data_ptr() == out.data_ptr()
                where = f"zero point {zp}, token scales {dd is not None}, offset {offset}"
                assert torch.equal(out.view(torch.int16), want.view(torch.int16)), where
                assert bool(buf[:offset].isnan().all()) and bool(buf[offset + M * N:].isnan().all()), where


@pytest.mark.parametrize("tile", [t for t in TILES if t != "split"])
def test_streamed_rows_of_partial_lines(unforced, tile):
    """A width that is no multiple of 32 and an output above 256 MB: streaming stores whose last channels are cut off."""
    M, N, K = 8200, 16392, 130
    operands = layer(M, N, K)
    _, _, wsum, s_w, d, acc = operands
    for zp, dd in ((None, None), (5, d)):
        want = expected(acc, wsum, 0.37, s_w, zp or 0, dd)
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        call(tile, M, N, K, operands, 0.37, zp, dd, out)
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), zp
