"""The quantizers that cut a row into pieces of a wave each (scale given or none, and the Hadamard quantizers): edges of the pieces, the classes of
the dispatch, and inputs whose products are no numbers."""
import numpy as np
import pytest
import torch

from paper_2506_04985_amd import binding as fptq
import fptq_workloads as synth

from gpu_util import dev, dev_bf16, launched

pytestmark = pytest.mark.gpu
MODES = [synth.MODE_NONE, synth.MODE_GIVEN]


def draw(M, K, mode, seed):
    return synth.draw(synth.LinearCase("p", f"m{M}k{K}", M, 8, K, "normal", 0.0, 3, 20.0, mode, seed), with_weights=False)


def with_specials(bits, every):
    """NaNs, infinities, values near the largest and the smallest, zeros of both signs, all over."""
    v = torch.tensor([float("nan"), float("inf"), -float("inf"), 3e38, -3e38, 1e-40, -0.0, 1e30]).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    b = bits.copy().reshape(-1)
    at = np.arange(every // 2, b.size, every)
    b[at] = v[np.arange(at.size) % 8]
    return b.reshape(bits.shape)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("M,K", [(1, 8), (3, 504), (3, 512), (5, 520), (2, 2040), (2, 2048), (3, 2056), (700, 72), (257, 1024),
                                 (1024, 8192), (1030, 8200), (2047, 9992),          # 16 to 40 MB: four chunks a lane, and above
                                 (2, 32768), (3, 40000)])
def test_static_quantizer_in_pieces(oracle, mode, M, K):
    inp = draw(M, K, mode, seed=M + K)
    for bits in (inp.x_bits, with_specials(inp.x_bits, 97)):
        xq, r = fptq.fptq_quantize_act(dev_bf16(bits), 0.4, mode, 0.0, dev(inp.row_scale_in))
        rows = np.unique(np.r_[0, M - 1, np.linspace(0, M - 1, 40).astype(int)])
        r_ref = oracle.row_scale(bits, mode, 0.0, inp.row_scale_in)
        assert np.array_equal(r.cpu().numpy().view(np.uint32), r_ref.view(np.uint32))
        q = fptq.fptq_unpack(xq, M, K).cpu().numpy()
        assert np.array_equal(q[rows], oracle.quantize(bits[rows], np.float32(0.4), r_ref[rows]))


@pytest.mark.parametrize("M,K,pieces", [(2048, 4088, 8), (2056, 4096, 2), (40000, 256, 1), (20000, 512, 1), (14000, 1024, 1), (13297, 1104, 1), (7140, 2056, 1), (85481, 1104, 1),
                                        (45900, 2056, 1), (4000, 3080, 2), (1790, 8200, 17), (1700, 11008, 22), (1000, 13824, 7), (4096, 14336, 28), (8000, 3200, 2),
                                        (10000, 4104, 2), (524288, 512, 1), (35000, 4096, 1), (33000, 4400, 3)])
def test_pieces_of_a_row(M, K, pieces):
    """Short rows are not cut, and no piece is mostly padding; codes as those of ten rows, which are cut by 512 values."""
    torch.manual_seed(M)
    x, r = torch.randn((M, K), device="cuda").to(torch.bfloat16), torch.rand(M, device="cuda") + 0.5
    out, r_out = torch.full((fptq.fptq_packed_bytes(M, K),), 0xEE, dtype=torch.uint8, device="cuda"), torch.empty_like(r)
    assert launched(lambda: fptq.fptq_quantize_act(x, 0.4, synth.MODE_GIVEN, 0.0, r, out=out, row_scale_out=r_out))[1] == (M * pieces + 3) // 4
    assert torch.equal(r, r_out)
    for i in (0, M // 2 + 1, M - 10):
        part, _ = fptq.fptq_quantize_act(x[i:i + 10], 0.4, synth.MODE_GIVEN, 0.0, r[i:i + 10].clone())
        assert torch.equal(out.view(-1, M, 64)[:, i:i + 10], part.view(-1, 10, 64))


def test_one_chunk_for_the_shortest_rows():
    """Chunks that lie past a row's end are loaded and computed all the same."""
    def kernel(M, K):
        x, out = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda"), torch.empty(fptq.fptq_packed_bytes(M, K), dtype=torch.uint8, device="cuda")
        return launched(lambda: fptq.fptq_quantize_act(x, 0.4, synth.MODE_NONE, 0.0, None, out=out, want_row_scale=False))[0]
    assert kernel(40000, 256) == kernel(20000, 512) == kernel(100, 512) != kernel(14000, 1024)


@pytest.mark.parametrize("mode", MODES)
def test_static_quantizer_beyond_the_last_level_cache(mode):
    """More than 256 MB: streamed.  Codes of the whole call and of its parts."""
    M, K = 8200, 16392
    torch.manual_seed(3)
    x = torch.randn((M, K), device="cuda").to(torch.bfloat16)
    r = torch.rand(M, device="cuda") + 0.5 if mode == synth.MODE_GIVEN else None
    q = fptq.fptq_unpack(fptq.fptq_quantize_act(x, 0.4, mode, 0.0, r)[0], M, K)
    for i in (0, 4096, M - 100):
        part = slice(i, i + 100)
        p = fptq.fptq_unpack(fptq.fptq_quantize_act(x[part], 0.4, mode, 0.0, None if r is None else r[part].clone())[0], 100, K)
        assert torch.equal(p, q[part])


# the last three: with RMS scale a wave walks a row, several spans of one and of two, four and eight chunks a lane; without, the many rows are a wave per block
@pytest.mark.parametrize("mode,M,K,B", [(mode, *shape) for shape in ((3, 256, 256), (5, 768, 256), (6, 1280, 256), (2, 512, 512), (5, 1536, 512), (7, 3072, 1024), (300, 2560, 512))
                                        for mode in (synth.MODE_NONE, synth.MODE_RMS, synth.MODE_GIVEN)]
                         + [(mode, *shape) for shape in ((4100, 16384, 2048), (4100, 32768, 4096)) for mode in MODES]
                         + [(synth.MODE_RMS, *shape) for shape in ((300, 3072, 1024), (300, 6144, 2048), (300, 12288, 4096))])
def test_hadamard_special_values(oracle, mode, M, K, B):
    """What the transform spreads over a block is the same tree of additions, so NaNs and infinities come out where the definition has them."""
    inp = draw(min(M, 400), K, mode, seed=M + K + B)
    bits = with_specials(inp.x_bits, 5 * B + 3)
    rep = -(-M // bits.shape[0])
    full = np.tile(bits, (rep, 1))[:M]
    scale = None if inp.row_scale_in is None else np.tile(inp.row_scale_in, rep)[:M]
    xq, r = fptq.fptq_quantize_act_hadamard(dev_bf16(full), 0.5, B, mode, 1e-5, dev(scale))
    q = fptq.fptq_unpack(xq, M, K)
    rows = np.arange(0, bits.shape[0], max(1, bits.shape[0] // 40))
    r_ref = oracle.row_scale(bits[rows], mode, 1e-5, None if scale is None else scale[rows])
    ref = oracle.quantize_hadamard(bits[rows], np.float32(0.5), B, None if mode == synth.MODE_NONE else r_ref)
    assert np.array_equal(q[torch.from_numpy(rows).cuda()].cpu().numpy(), ref)
    if M > bits.shape[0]:
        assert torch.equal(q[:bits.shape[0]], q[bits.shape[0]:2 * bits.shape[0]])


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("M,K,B", [(12400, 11008, 256), (9800, 13824, 512), (11000, 12288, 512), (12000, 11264, 1024), (9400, 14336, 2048), (4700, 28672, 4096)])
def test_hadamard_beyond_the_last_level_cache(mode, M, K, B):
    """More than 256 MB: streamed.  Codes of the whole call and of its parts, which are not."""
    assert M * K * 2 > 256 << 20
    torch.manual_seed(B)
    x = torch.randn((M, K), device="cuda").to(torch.bfloat16)
    r = torch.rand(M, device="cuda") + 0.5 if mode == synth.MODE_GIVEN else None
    xq, s = fptq.fptq_quantize_act_hadamard(x, 0.4, B, mode, 1e-5, r)
    for i in range(0, M, M // 4):
        n = min(M // 4, M - i)
        part, ps = fptq.fptq_quantize_act_hadamard(x[i:i + n], 0.4, B, mode, 1e-5, None if r is None else r[i:i + n].clone())
        assert torch.equal(xq.view(-1, M, 64)[:, i:i + n], part.view(-1, n, 64)) and torch.equal(s[i:i + n], ps)
