"""Calls of very many values: HIP refuses a launch of 2^32 threads or more, so they go to a kernel that spreads a row over fewer waves."""
import pytest
import torch

from paper_2506_04985_amd import binding as fptq
import fptq_workloads as synth

from gpu_util import captured

pytestmark = pytest.mark.gpu


def launches(M, K, call):
    """The launch of a call that names M x K values, captured and never run: its buffers hold next to nothing."""
    small = [torch.zeros(64, dtype=torch.uint8, device="cuda").data_ptr() for _ in range(5)]
    _, grid, block = captured(lambda: call(fptq.lib(), M, K, *small, fptq.fptq_packed_bytes(M, K), torch.cuda.current_stream().cuda_stream))
    return grid, block


def ok(rc):
    assert rc == 0, fptq.lib().fptq_last_error()


def hadamard(B, mode):
    return lambda L, M, K, x, r, out, r_out, _, n, stream: ok(L.fptq_quantize_act_hadamard(x, M, K, B, mode, 1e-5, r, 0.5, out, n, r_out, stream))


def static(mode):
    return lambda L, M, K, x, r, out, r_out, _, n, stream: ok(L.fptq_quantize_act(x, M, K, mode, 1e-5, r, 0.5, out, n, r_out, stream))


def dynamic(L, M, K, x, r, out, r_out, _, n, stream):
    ok(L.fptq_quantize_act_dynamic(x, M, K, out, n, r_out, stream))


def residual(L, M, K, x, r, out, r_out, y, n, stream):
    ok(L.fptq_residual_norm_quantize(x, y, M, K, r, 1e-5, 0.5, x, r_out, out, n, stream))


@pytest.mark.parametrize("mode", [synth.MODE_NONE, synth.MODE_GIVEN])
@pytest.mark.parametrize("M,K,B", [((1 << 16) + 1, 1 << 20, 256), ((1 << 25) + 1, 2048, 256), ((1 << 26) - 4, 1536, 512), ((1 << 16) + 1, 1 << 20, 1024), (1 << 17, 1 << 20, 2048),
                                   ((1 << 18) + 1, 1 << 20, 4096), (1, 1 << 38, 512), (3, 1 << 38, 4096)])
def test_hadamard(M, K, B, mode):
    grid, block = launches(M, K, hadamard(B, mode))
    assert block == 256 and grid * block < 1 << 32
    assert grid * 4 >= min(M * (K // max(B, 1024)), (1 << 26) - 4) // 2        # and no more rows to a wave than it takes


@pytest.mark.parametrize("mode", [synth.MODE_NONE, synth.MODE_GIVEN])
@pytest.mark.parametrize("M,K", [((1 << 25) + 1, 2056), ((1 << 26) - 4, 4096), ((1 << 24) - 1, 10000), (1 << 20, 1 << 20)])
def test_static(M, K, mode):
    grid, block = launches(M, K, static(mode))
    assert grid * block < 1 << 32


@pytest.mark.parametrize("call", [dynamic, residual])
@pytest.mark.parametrize("M,K", [(1 << 24, 3080), ((1 << 26) - 4, 4096), ((1 << 24) - 1, 4096), (1 << 24, 3072)])
def test_whole_rows(M, K, call):
    grid, block = launches(M, K, call)
    assert grid * block < 1 << 32


def test_a_wave_walks_its_spans():
    """What such calls run, on 137 GB: rows at both ends and in the middle, and the scale of every row."""
    M, K, B = (1 << 16) + 3, 1 << 20, 256
    if torch.cuda.mem_get_info()[0] < 230 << 30:
        pytest.skip("needs 172 GB of device memory")
    x = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    rows = [0, 1, 2, M // 2, M - 2, M - 1]
    torch.manual_seed(4)
    x[rows] = torch.randn((len(rows), K), device="cuda").to(torch.bfloat16)
    r = torch.rand(M, device="cuda") + 0.5
    xq, r_out = fptq.fptq_quantize_act_hadamard(x, 0.4, B, synth.MODE_GIVEN, 0.0, r)
    assert torch.equal(r, r_out)
    few, _ = fptq.fptq_quantize_act_hadamard(x[rows], 0.4, B, synth.MODE_GIVEN, 0.0, r[rows])
    assert torch.equal(xq.view(K // 128, M, 64)[:, rows], few.view(K // 128, len(rows), 64))
    others = xq.view(K // 128, M, 64)[:, 3:M // 2:997]
    assert int(others.count_nonzero()) == 0
    del x, xq
    torch.cuda.empty_cache()
