"""Quantizers on rows whose length is no multiple of eight or whose address is only 2-byte aligned: chunks loaded where they lie, at the edges
of the rows, of the width classes and of the register path, against the oracle; nothing outside the matrix is used or written."""
import numpy as np
import pytest
import torch

from paper_2506_04985_amd import binding as fptq
import fptq_workloads as synth

from gpu_util import dev, host_bits, launched

pytestmark = pytest.mark.gpu

SHAPES = [(3, 1, 1), (5, 7, 0), (4, 9, 1), (3, 16, 3), (2, 127, 0), (6, 1001, 1), (3, 2047, 0), (2, 2048, 1), (3, 2049, 0), (2, 4097, 5), (2, 8191, 0), (2, 8195, 1),
          (1, 16385, 0), (2, 32767, 1), (1, 32768, 1), (1, 32769, 0), (900, 333, 1), (900, 4094, 0)]


# many short rows, which a wave takes each: rows below a chunk, the ends of the five width classes
MANY = [(769, 1, 1), (770, 7, 0), (771, 8, 1), (1030, 9, 1), (769, 63, 0), (901, 511, 1), (769, 512, 1), (770, 513, 0), (769, 1024, 1),
        (3073, 1025, 0), (3074, 2047, 0), (3073, 2049, 0), (3073, 3072, 1), (3073, 3073, 0)]


def place(bits, offset):
    """The matrix at an odd place in a larger buffer of NaNs."""
    M, K = bits.shape
    base = torch.full((M * K + offset + 40,), float("nan"), dtype=torch.bfloat16, device="cuda")
    x = base[offset:offset + M * K].view(M, K)
    x.view(torch.int16).copy_(torch.from_numpy(bits.view(np.int16)))
    return x, base


def draw(M, K, seed=0):
    rng = np.random.default_rng(M * 7 + K + seed)
    return synth.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32) * np.exp(rng.standard_normal((M, 1))).astype(np.float32)), rng


def padding_is_zero(xq, M, K):
    full = fptq.fptq_unpack(xq, M, (K + 127) // 128 * 128).cpu().numpy()
    return not full[:, K:].any()


@pytest.mark.parametrize("M,K,offset", [*SHAPES, *MANY])
def test_static_and_dynamic(oracle, M, K, offset):
    xb, rng = draw(M, K)
    x, _ = place(xb, offset)
    given = rng.uniform(0.3, 2, M).astype(np.float32)
    s_a = np.float32(0.4)
    for mode in (synth.MODE_NONE, synth.MODE_RMS, synth.MODE_GIVEN):
        r_ref = oracle.row_scale(xb, mode, 1e-5, given)
        xq, r = fptq.fptq_quantize_act(x, float(s_a), mode, 1e-5, dev(given))
        assert np.array_equal(r.cpu().numpy().view(np.uint32), r_ref.view(np.uint32))
        assert np.array_equal(fptq.fptq_unpack(xq, M, K).cpu().numpy(), oracle.quantize(xb, s_a, None if mode == synth.MODE_NONE else r_ref))
        assert padding_is_zero(xq, M, K)
    xq, _ = fptq.fptq_quantize_act_asym(x, float(s_a), 3, synth.MODE_GIVEN, row_scale_in=dev(given))
    assert np.array_equal(fptq.fptq_unpack(xq, M, K).cpu().numpy(), oracle.quantize_zp(xb, s_a, 3, given)) and padding_is_zero(xq, M, K)
    xq, s = fptq.fptq_quantize_act_dynamic(x)
    q_ref, s_ref = oracle.quantize_dynamic(xb)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(fptq.fptq_unpack(xq, M, K).cpu().numpy(), q_ref) and padding_is_zero(xq, M, K)


@pytest.mark.parametrize("alias", [None, "x", "y"])
@pytest.mark.parametrize("M,K,offset", [*SHAPES, *MANY, (2, 16392, 0), (3, 28672, 0), (1, 32760, 0)])
def test_residual_step(oracle, M, K, offset, alias):
    xb, rng = draw(M, K)
    yb, _ = draw(M, K, 1)
    x, x_base = place(xb, offset)
    y, y_base = place(yb, offset)
    o, o_base = place(np.zeros_like(xb), offset)
    s_prev = rng.uniform(0.2, 3, M).astype(np.float32)
    target, base = {None: (o, o_base), "x": (x, x_base), "y": (y, y_base)}[alias]
    x_next, s_next, xq = fptq.fptq_residual_norm_quantize(x, y, 0.45, dev(s_prev), 1e-5, x_next=target)
    ref = oracle.residual_norm_quantize(xb, yb, np.float32(0.45), s_prev, 1e-5)
    assert x_next.data_ptr() == target.data_ptr() and np.array_equal(host_bits(target), ref["x_next"])
    assert np.array_equal(s_next.cpu().numpy().view(np.uint32), ref["s_next"].view(np.uint32))
    assert np.array_equal(fptq.fptq_unpack(xq, M, K).cpu().numpy(), ref["q"]) and padding_is_zero(xq, M, K)
    assert bool(base[:offset].isnan().all()) and bool(base[offset + M * K:].isnan().all())


@pytest.mark.parametrize("M,K", [(769, 63), (2048, 333), (8192, 1001), (3073, 4095)])
def test_many_short_rows_share_workgroups(M, K):
    """A workgroup per row was up to four times as slow there as four rows to a workgroup, a wave each."""
    x, y = (torch.randn((M, K), device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.empty(fptq.fptq_packed_bytes(M, K), dtype=torch.uint8, device="cuda")
    s, o = torch.empty(M, device="cuda"), torch.empty_like(x)
    for call in (lambda: fptq.fptq_quantize_act(x, 0.4, synth.MODE_RMS, 1e-5, None, out=q, row_scale_out=s),
                 lambda: fptq.fptq_quantize_act_dynamic(x, out=q, token_scale_out=s),
                 lambda: fptq.fptq_residual_norm_quantize(x, y, 0.45, None, 1e-5, x_next=o, s_next=s, out=q)):
        assert launched(call)[1] == (M + 3) // 4
