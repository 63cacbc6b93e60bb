"""The six-bit kernel of large problems, forced on shapes at the edges of its tiles: bit for bit the oracle's result, or that of
the library's other kernels where the oracle would take too long."""
import pytest
import torch

from paper_2506_04985_amd import binding as fptq
import fptq_workloads as synth

from gpu_util import dev, dev_bf16, host_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[256, 192, 128])
def forced(request):
    fptq.fptq_set_linear_prefill(request.param)         # tokens per tile
    yield request.param
    fptq.fptq_set_linear_prefill(0)


def scratch_for(M, N, K):
    n = fptq.fptq_linear_scratch_bytes(M, N, K)
    assert n > 0
    return torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")        # nothing in it may matter


# one to thirteen K tiles (the loop is unrolled by six and keeps five in flight), tokens and channels around the tiles,
# widths the 16-byte stores do not divide, K that no tile divides
@pytest.mark.parametrize("M,N,K", [(65, 1, 1), (100, 8, 128), (128, 260, 256), (385, 40, 700), (255, 255, 129), (256, 256, 384),
                                   (257, 257, 500), (129, 300, 640), (66, 70, 768), (300, 520, 896), (513, 64, 1030), (90, 776, 1537)])
def test_matches_oracle(forced, oracle, M, N, K):
    case = synth.LinearCase("p6", f"m{M}", M, N, K, "normal", 0.0, 1, 4.0, synth.MODE_RMS, M + N + K)
    inp = synth.draw(case)
    ref = oracle.w4a4_linear(inp.x_bits, inp.w_int, inp.s_a, inp.s_w, synth.MODE_RMS, case.eps)
    xq, _ = fptq.fptq_quantize_act(dev_bf16(inp.x_bits), float(inp.s_a), synth.MODE_RMS, case.eps)
    wq = fptq.fptq_pack_weights(dev(inp.w_int))
    y, acc = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, float(inp.s_a), dev(inp.s_w), scratch_for(M, N, K), want_acc=True)
    assert (acc.cpu().numpy() == ref["acc"]).all()
    assert (host_bits(y) == ref["y"]).all()
    y = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, float(inp.s_a), dev(inp.s_w), scratch_for(M, N, K))
    assert (host_bits(y) == ref["y"]).all()


@pytest.mark.parametrize("M,N,K,zp", [(300, 520, 2504, 0), (1000, 1032, 1280, 0), (333, 771, 4096, -8), (260, 264, 904, 7)])
def test_equals_the_int8_kernel(forced, M, N, K, zp):
    torch.manual_seed(M + K)
    xq = fptq.fptq_pack_weights(torch.randint(-8, 8, (M, K), dtype=torch.int8, device="cuda"))
    w = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda")
    wq, ws = fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w)
    s_w, d = torch.rand(N, device="cuda") * 0.015 + 0.005, torch.rand(M, device="cuda") + 0.5
    got = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.37, s_w, scratch_for(M, N, K), zp, ws, d, want_acc=True)
    fptq.fptq_set_linear_prefill(2)
    want = fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.37, s_w, zp, ws, d, want_acc=True)
    assert torch.equal(got[1], want[1]) and torch.equal(got[0].view(torch.int16), want[0].view(torch.int16))


@pytest.mark.parametrize("tiles", range(30, 41))
def test_k_tiles_around_the_line_of_the_loops(forced, tiles):
    """Up to 32 K tiles run the loop unrolled by two (256 and 192 tokens), more of them the one unrolled by six, at each of its remainders."""
    M, N, K = 203, 264 + tiles % 3, tiles * 128 - tiles % 4 * 41
    torch.manual_seed(K)
    xq = fptq.fptq_pack_weights(torch.randint(-8, 8, (M, K), dtype=torch.int8, device="cuda"))
    wq = fptq.fptq_pack_weights(torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda"))
    s_w, d = torch.rand(N, device="cuda") * 0.015 + 0.005, torch.rand(M, device="cuda") + 0.5
    want, acc = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 0.37, s_w, d, want_acc=True)
    got = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.37, s_w, scratch_for(M, N, K), row_out_scale=d, want_acc=True)
    assert torch.equal(got[1], acc) and torch.equal(got[0].view(torch.int16), want.view(torch.int16))
    got = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.37, s_w, scratch_for(M, N, K), row_out_scale=d)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("M,N,zp,with_d", [(289, 264, None, False), (65, 257, None, False), (289, 264, None, True), (255, 72, 3, False), (130, 515, -8, True)])
def test_epilogue_of_any_scale(forced, M, N, zp, with_d):
    """Channel scales from subnormal to infinite and NaN (the kernel folds a factor of 64 into ordinary ones), with and without token
    scales and a zero point; nothing is written past the last row."""
    K = 300
    torch.manual_seed(M)
    xq = fptq.fptq_pack_weights(torch.randint(-8, 8, (M, K), dtype=torch.int8, device="cuda"))
    w = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda")
    w[::5] = 0
    wq, ws = fptq.fptq_pack_weights(w), fptq.fptq_weight_row_sums(w)
    d = torch.rand(M, device="cuda") + 0.5 if with_d else None
    for odd in ([], [1e-42, 2.0 ** -126], [2.0 ** 122, 3e38], [float("inf")], [float("nan")]):
        s_w = torch.rand(N, device="cuda") * 0.015 + 0.005
        s_w[torch.arange(len(odd)) * 35] = torch.tensor(odd, device="cuda")
        buf = torch.full(((M + 300) * N,), 77.0, dtype=torch.bfloat16, device="cuda")
        scratch = scratch_for(M, N, K)
        args = (0, None) if zp is None else (zp, ws)
        fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 1.0, s_w, scratch, *args, d, out=buf[:M * N].view(M, N))
        want = fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 1.0, s_w, d) if zp is None else None
        if zp is not None:
            fptq.fptq_set_linear_prefill(2)
            want = fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 1.0, s_w, zp, ws, d)
            fptq.fptq_set_linear_prefill(forced)
        got = buf[:M * N].view(M, N)
        assert torch.equal(got.isnan(), want.isnan())
        assert torch.equal(got.nan_to_num(nan=0.0).view(torch.int16), want.nan_to_num(nan=0.0).view(torch.int16))
        assert bool((buf[M * N:] == 77.0).all())


def test_streamed_rows_of_partial_lines(forced):
    """A width that is no multiple of 32 and an output above 256 MB: streaming stores whose last channels are cut off."""
    M, N, K = 8200, 16392, 130
    torch.manual_seed(1)
    xq = fptq.fptq_pack_weights(torch.randint(-8, 8, (M, K), dtype=torch.int8, device="cuda"))
    wq = fptq.fptq_pack_weights(torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda"))
    s_w = torch.rand(N, device="cuda") * 0.015 + 0.005
    got, noalloc = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.37, s_w, scratch_for(M, N, K), out=got)
    fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.37, s_w, out=noalloc)
    want = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 0.37, s_w)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16)) and torch.equal(noalloc.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("K", [131071, 131070])
@pytest.mark.parametrize("x,w", [(-8, -8), (7, -8), (-8, 7), (7, 7)])
def test_longest_sums_of_the_largest_products(forced, K, x, w):
    """|64 K| is just below 2^23 and the running sums stay below 2^24, where fp32 still counts by ones; a few products of
    one in an otherwise constant row must show."""
    M, N = 70, 40
    xi = torch.full((M, K), x, dtype=torch.int8, device="cuda")
    wi = torch.full((N, K), w, dtype=torch.int8, device="cuda")
    xi[torch.arange(M), torch.arange(M) * 1801] = 1
    wi[torch.arange(N), K - 1 - torch.arange(N) * 3203] = -1
    xq, wq = fptq.fptq_pack_weights(xi), fptq.fptq_pack_weights(wi)
    s_w = torch.ones(N, device="cuda")
    _, acc = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 1.0, s_w, scratch_for(M, N, K), want_acc=True)
    _, ref = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 1.0, s_w, want_acc=True)
    assert torch.equal(acc, ref)


@pytest.mark.parametrize("zp", [-8, 7])
@pytest.mark.parametrize("x,w", [(-8, -8), (7, -8), (-8, 7), (7, 7)])
def test_zero_point_of_the_longest_sums(forced, x, w, zp):
    """acc - z sum_k w reaches 120 K, 15 / 16 of 2^24 at the largest K: still an exact integer in fp32, where the INT8 kernel's limit is
    half the K.  Against the epilogue's definition on host integers, and the simple kernel."""
    M, N, K = 70, 40, 131071
    xi = torch.full((M, K), x, dtype=torch.int8, device="cuda")
    wi = torch.full((N, K), w, dtype=torch.int8, device="cuda")
    xi[torch.arange(M), torch.arange(M) * 1801] = 1
    wi[torch.arange(N), K - 1 - torch.arange(N) * 3203] = -1
    xq, wq, sums = fptq.fptq_pack_weights(xi), fptq.fptq_pack_weights(wi), fptq.fptq_weight_row_sums(wi)
    s_w, d = torch.rand(N, device="cuda") * 0.015 + 0.005, torch.rand(M, device="cuda") + 0.5
    y, acc = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.37, s_w, scratch_for(M, N, K), zp, sums, d, want_acc=True)
    fptq.fptq_set_linear_prefill(2)
    y_ref, acc_ref = fptq.fptq_w4a4_linear_zp(xq, wq, M, N, K, 0.37, s_w, zp, sums, d, want_acc=True)
    assert torch.equal(acc, acc_ref) and torch.equal(y.view(torch.int16), y_ref.view(torch.int16))
    exact = acc_ref.cpu().long() - zp * wi.cpu().long().sum(1)
    assert int(exact.abs().max()) < 1 << 24
    cw = torch.tensor(0.37, dtype=torch.float32) * s_w.cpu()
    assert torch.equal(y.cpu(), (exact.float() * cw * d.cpu()[:, None]).to(torch.bfloat16))


def test_random_rows_of_the_longest_sums(forced):
    M, N, K = 66, 264, 131071
    torch.manual_seed(4)
    for lo, hi in ((-8, 8), (-8, -4), (4, 8), (-1, 2)):
        xq = fptq.fptq_pack_weights(torch.randint(lo, hi, (M, K), dtype=torch.int8, device="cuda"))
        wq = fptq.fptq_pack_weights(torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda").sort(dim=1).values)
        s_w = torch.ones(N, device="cuda")
        _, acc = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 1.0, s_w, scratch_for(M, N, K), want_acc=True)
        _, ref = fptq.fptq_w4a4_linear_ref(xq, wq, M, N, K, 1.0, s_w, want_acc=True)
        assert torch.equal(acc, ref)


@pytest.mark.parametrize("M,N,K,workgroups", [(4096, 8192, 4096, 16 * 32), (2048, 4096, 11008, 16 * 16), (512, 8192, 8192, 0)])
def test_tile_per_problem(M, N, K, workgroups):
    """Large tiles, small ones where the large ones would leave compute units idle, neither where the small ones would."""
    plan = fptq.fptq_linear_launch_plan(M, N, K, with_scratch=True)
    assert plan[:2] == ("linear_prefill_kernel", workgroups) if workgroups else plan[0].startswith("GemmCfg")
    assert (fptq.fptq_linear_scratch_bytes(M, N, K) > 0) == (workgroups > 0)


def test_too_little_scratch_or_none_gives_the_plain_layer():
    M, N, K = 4096, 8192, 4096
    need = fptq.fptq_linear_scratch_bytes(M, N, K)
    assert need > 0 and fptq.fptq_linear_launch_plan(M, N, K, with_scratch=True)[0] == "linear_prefill_kernel"
    assert fptq.fptq_linear_scratch_bytes(8, N, K) == 0
    torch.manual_seed(2)
    xq = torch.randint(0, 256, (fptq.fptq_packed_bytes(M, K),), dtype=torch.uint8, device="cuda")
    wq = torch.randint(0, 256, (fptq.fptq_packed_bytes(N, K),), dtype=torch.uint8, device="cuda")
    s_w = torch.rand(N, device="cuda") * 0.015 + 0.005
    want = fptq.fptq_w4a4_linear_noalloc(xq, wq, M, N, K, 0.5, s_w)
    small = torch.zeros(need - 256, dtype=torch.uint8, device="cuda")
    for scratch in (None, small, torch.empty(need, dtype=torch.uint8, device="cuda")):
        got = fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.5, s_w, scratch)
        assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert int(small.max()) == 0
    got = fptq.fptq_w4a4_linear(xq, wq, M, N, K, 0.5, s_w)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    with pytest.raises(fptq.FptqError):
        fptq.fptq_w4a4_linear_scratch(xq, wq, M, N, K, 0.5, s_w, torch.empty(need + 64, dtype=torch.uint8, device="cuda")[64:])
