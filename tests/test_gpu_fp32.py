"""GPU parity, fp32: config 1 (B1, 16x16 grid, 6 heads x 64) and ragged/edge shapes, all three
mixers, element by element against the CPU oracle; window/padding maps bit-exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_26636_amd import binding, synth
from parity import check, FP32_TOL, err_fp32, to_device, to_host

pytestmark = pytest.mark.gpu


def _run_all(q, k, v, H, W, window, eps=1e-6):
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    out = {}
    o = torch.empty_like(dq); binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W), eps); out["linear"] = to_host(o)
    o = torch.empty_like(dq); binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window); out["window"] = to_host(o)
    o = torch.empty_like(dq); binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W)); out["full"] = to_host(o)
    torch.cuda.synchronize()
    return out


def test_config1_all_three_mixers():
    c = synth.CONFIGS[1]
    q, k, v = synth.config_qkv(1)
    got = _run_all(q, k, v, c["H"], c["W"], c["window"])
    check(err_fp32(got["linear"], oracle.linear_attn_quadratic(q, k, v, 1e-6)), FP32_TOL)
    check(err_fp32(got["window"], oracle.window_attn(q, k, v, c["H"], c["W"], *c["window"])), FP32_TOL)
    check(err_fp32(got["full"], oracle.full_attn(q, k, v)), FP32_TOL)


@pytest.mark.parametrize("B,heads,H,W,window", [
    (2, 3, 7, 9, (4, 4)),      # ragged grid, padded windows, N = 63 (not a multiple of any tile)
    (1, 2, 37, 37, (8, 8)),    # the 518 px / patch 14 geometry
    (1, 1, 1, 1, (1, 1)),      # a single token
    (1, 2, 5, 67, (5, 67)),    # window = grid, N = 335 spans several key tiles with a tail
    (3, 1, 16, 24, (16, 3)),   # rectangular windows
    (1, 1, 20, 20, (32, 32)),  # window larger than the grid
])
def test_ragged_and_edge_shapes(B, heads, H, W, window):
    N = H * W
    q, k, v = synth.qkv(7, B, heads, N, 64, 1.0, False)
    got = _run_all(q, k, v, H, W, window)
    check(err_fp32(got["linear"], oracle.linear_attn_quadratic(q, k, v, 1e-6)), FP32_TOL)
    check(err_fp32(got["window"], oracle.window_attn(q, k, v, H, W, *window)), FP32_TOL)
    check(err_fp32(got["full"], oracle.full_attn(q, k, v)), FP32_TOL)


@pytest.mark.parametrize("B,heads,H,W,window", [
    (1, 1, 1, 33, (1, 32)),    # one key past a tile of 32; a window of one token
    (1, 2, 8, 16, (8, 8)),     # four full tiles, one per key group; windows of two tiles
    (1, 1, 3, 43, (3, 43)),    # 129 keys: the second step of the four key groups has one tile of one key
    (2, 12, 21, 21, (7, 7)),   # 49-slot windows: a tile and a half, queries and keys
    (2, 16, 33, 65, (8, 8)),   # enough windows for two and for one key group per query block
])
def test_attention_tile_edges(B, heads, H, W, window):
    N = H * W
    q, k, v = synth.qkv(17, B, heads, N, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.empty_like(dq)
    binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window)
    check(err_fp32(to_host(o), oracle.window_attn(q, k, v, H, W, *window)), FP32_TOL)
    if N < 1000:
        binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W))
        check(err_fp32(to_host(o), oracle.full_attn(q, k, v)), FP32_TOL)


@pytest.mark.parametrize("H,W,window,P", [
    (1, 65, None, 0), (1, 96, None, 0), (1, 97, None, 0), (1, 128, None, 0), (1, 129, None, 0),  # 3 to 5 tiles on 4 wavefronts (4: staged)
    (20, 30, (10, 10), 0), (14, 32, (4, 32), 3),                                                 # 4 tiles: not whole rows, whole rows
    (1, 383, None, 1), (20, 21, None, 5),    # prefix tokens: key counts 384, 425
    (20, 30, (9, 11), 0), (20, 30, (12, 30), 2), (11, 13, (11, 8), 64),  # windows: ragged, of whole rows, with prefix queries
])
def test_keys_split_over_wavefronts(H, W, window, P):
    """Launches of few queries (the keys split over the wavefronts of a workgroup), with logits that
    climb along the sequence so that the softmax reference goes up in late tiles too."""
    N = P + H * W
    q, k, v = synth.qkv(44, 1, 2, N, 64, 1.0, False)
    k = (k * np.linspace(0.2, 6.0, N, dtype=np.float32)[None, None, :, None]).astype(np.float32)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), device="cuda")
    if window is None:
        binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W))
        ref = oracle.full_attn(q, k, v)
    else:
        binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window)
        ref = oracle.window_attn_prefix(q, k, v, P, H, W, *window)
    check(err_fp32(to_host(o), ref), FP32_TOL)


@pytest.mark.parametrize("row", [2949840, 2949844, 1 << 22])
def test_slices_of_four_gigabytes(row):
    """300 tokens whose K and V rows lie `row` elements apart: the last stride at which a slice's byte offsets fit 32
    bits, the first at which they do not, and offsets beyond 2^32 (the tiles are staged through LDS then)."""
    q, k, v = synth.qkv(46, 1, 1, 300, 64, 1.0, False)
    dq = to_device(q, False)
    wide = [torch.empty(299 * row + 64, device="cuda").as_strided(dq.shape, (300 * row, 300 * row, row, 1)) for _ in range(2)]
    for t, x in zip(wide, (k, v)):
        t.copy_(to_device(x, False))
    o = torch.full(dq.shape, float("nan"), device="cuda")
    binding.jv_full_attn_fwd(dq, *wide, o, (1, 300))
    check(err_fp32(to_host(o), oracle.full_attn(q, k, v)), FP32_TOL)


@pytest.mark.parametrize("N", [160, 256, 1030])
def test_values_near_the_largest_floats(N):
    """Weights of at most 1, also where a late key is some binary orders above the early ones: values of 1e37
    pass through the sums without overflow (the oracle's maximum-subtracted softmax in 64 bits)."""
    g = np.random.default_rng(45)
    q, k, v = np.zeros((1, 2, N, 64), np.float32), np.zeros((1, 2, N, 64), np.float32), None
    q[..., 0] = 8.0  # logits are k[..., 0]
    k[..., 0] = 0.1 * g.standard_normal((1, 2, N))
    k[:, :, 128 + 5::32, 0] = np.linspace(4.5, 5.4, k[:, :, 128 + 5::32].shape[2])  # one key of every later tile: 2^6.5 .. 2^7.8
    v = (1e37 * g.uniform(0.5, 1.0, (1, 2, N, 64))).astype(np.float32)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), device="cuda")
    binding.jv_full_attn_fwd(dq, dk, dv, o, (1, N))
    check(err_fp32(to_host(o), oracle.full_attn(q, k, v)), FP32_TOL)


# (heads, tokens) of the two kernels whose operands are sums of three bf16 numbers
SPLIT_KERNELS = {"kF32Few": [(2, 70), (3, 161), (2, 385), (6, 1030)], "kF32Many": [(300, 70), (200, 161), (64, 385), (50, 1030)]}
SPLIT_SIZES = [c for sizes in SPLIT_KERNELS.values() for c in sizes]


def _full64(q, k, v):
    s = (q.double() @ k.double().transpose(-1, -2).contiguous()) * 0.125
    return torch.softmax(s, -1) @ v.double()


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
@pytest.mark.parametrize("what", ["plain", "tiny", "large", "climb", "fall", "outlier"])
def test_split_operands(heads, N, what):
    """Magnitudes from 1e-30 to 1e30 (products of order one), and K and V that grow or shrink by 2^24 along the sequence."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    q, k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(3))
    ramp = torch.exp2(torch.linspace(-12, 12, N, device="cuda"))[:, None]
    if what == "tiny":
        q, k, v = q * 1e-20, k * 1e20, v * 1e-30
    elif what == "large":
        q, k, v = q * 1e20, k * 1e-20, v * 1e30
    elif what == "climb":
        k, v = k * torch.exp2(torch.linspace(-24, 0, N, device="cuda"))[:, None], v * ramp
    elif what == "fall":
        k, v = k * torch.exp2(torch.linspace(0, -24, N, device="cuda"))[:, None], v * ramp.flip(0)
    elif what == "outlier":  # one row of each tile 2^10 above the others
        v[:, :, 5::32] *= 1024.0
    o = torch.full_like(q, float("nan"))
    binding.jv_full_attn_fwd(q, k, v, o, (1, N))
    ref = _full64(q, k, v)
    # sums of up to 1 030 fp32 products and logits of up to 40: 3e-7 measured with the fp32 matrix instructions at these lengths
    check(float((o.double() - ref).norm() / ref.norm()), 5e-7)


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
@pytest.mark.parametrize("most", [8, 24, 60])
def test_channels_of_different_magnitude(heads, N, most):
    """Channel by channel a power of two on V, and one on K whose inverse is on Q: every number keeps its 24 bits whatever the others
    are, so that the result has the same bits times V's powers."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + 3)
    q, k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(3))
    qk, on_v = (torch.exp2(torch.randint(-most, most + 1, (1, heads, 1, 64), generator=g, device="cuda").float()) for _ in range(2))
    plain, o = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    binding.jv_full_attn_fwd(q, k, v, plain, (1, N))
    binding.jv_full_attn_fwd(q * qk, k / qk, v * on_v, o, (1, N))
    ref = _full64(q, k, v)
    # a channel, and a query, by its own norm: 3e-7 of the whole measured with the fp32 matrix instructions, a row of 64 numbers up to three times that
    channel, row = ((plain.double() - ref).norm(dim=d) / ref.norm(dim=d) for d in (2, 3))
    check(float(channel.max()), 1e-6)
    check(float(row.max()), 1e-6)
    assert torch.equal(o, plain * on_v)


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
def test_rows_of_different_magnitude(heads, N):
    """Every query attends almost to its own key, and values grow by 2^24 along the sequence: a row of small values next to large ones of
    weights near 1e-8, by its own norm."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + 4)
    k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(2))
    k = 12.0 * k / k.norm(dim=-1, keepdim=True)
    v = v * torch.exp2(torch.linspace(-12, 12, N, device="cuda"))[:, None]
    o = torch.full_like(k, float("nan"))
    binding.jv_full_attn_fwd(k, k, v, o, (1, N))
    ref = _full64(k, k, v)
    # exponents of up to 26 binary orders, each rounded to 2^-20, from scores of up to 144, rounded to 2^-17: 2^-17 of a weight
    check(float(((o.double() - ref).norm(dim=-1) / ref.norm(dim=-1)).max()), 2.0 ** -17)


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
def test_many_small_weights(heads, N):
    """One key of weight 1 and a value of 2^-32, all others of weights near 2^-32 and values near 1: half of the result comes from weights that far
    below the largest."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + 5)
    q, k = torch.zeros(1, heads, N, 64, device="cuda"), torch.zeros(1, heads, N, 64, device="cuda")
    v = torch.rand(1, heads, N, 64, generator=g, device="cuda") + 0.5
    q[..., 9] = 8.0
    k[:, :, N // 2, 9] = 22.0
    v[:, :, N // 2] *= 2.0 ** -32 * N
    o = torch.full_like(q, float("nan"))
    binding.jv_full_attn_fwd(q, k, v, o, (1, N))
    ref = _full64(q, k, v)
    # an exponent of 32 binary orders rounded to 2^-19, and sums of up to 1 030 numbers of one sign
    check(float(((o.double() - ref).norm(dim=-1) / ref.norm(dim=-1)).max()), 2.0 ** -18)


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
def test_logits_far_below_zero(heads, N):
    """Finite logits near -1e36: the weights are relative to the largest of them, however low that is."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + 2)
    v = torch.randn(1, heads, N, 64, generator=g, device="cuda")
    q, k = torch.zeros_like(v), torch.zeros_like(v)
    q[..., 5] = 2.0 ** 60
    k[..., 5] = -(2.0 ** 60)
    k[:, :, N // 3, 5] = -(2.0 ** 59)  # one key far above the others ...
    k[:, 1::2, N - 1, 5] = -(2.0 ** 59)  # ... and two of them alike in every other head
    o = torch.full_like(q, float("nan"))
    binding.jv_full_attn_fwd(q, k, v, o, (1, N))
    ref = v[:, :, N // 3].clone()
    ref[:, 1::2] = 0.5 * (v[:, 1::2, N // 3].double() + v[:, 1::2, N - 1].double()).float()
    # weights of 0 and 1 (or 1/2) alone: the rounding of a quotient
    assert torch.allclose(o, ref[:, :, None].expand_as(o), rtol=3e-7, atol=3e-7)


@pytest.mark.parametrize("heads,N", SPLIT_SIZES)
def test_infinities_and_nan(heads, N):
    """What is not finite ends where the formula puts it: a key's value in its channel of every query, a query's
    in its own row, a key's score of -inf nowhere."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + 1)
    q, k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(3))
    v[0, 0, N - 1, 7] = float("inf")
    v[0, 0, 3, 40] = float("-inf")
    v[0, 1, 33, 9] = float("nan")
    q[0, 1, 5, 0] = float("nan")
    q[..., 63] = q[..., 63].abs() + 0.1
    k[0, 1, 40, 63] = float("-inf")  # a score of -inf: no weight
    o = torch.full_like(q, 123.0)
    binding.jv_full_attn_fwd(q, k, v, o, (1, N))
    ref = _full64(q, k, v)
    assert torch.equal(torch.isnan(o), torch.isnan(ref))
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(o), inf) and torch.equal(o[inf].double(), ref[inf])
    real = torch.isfinite(ref)
    check(float((o.double()[real] - ref[real]).norm() / ref[real].norm()), 5e-7)  # (as above)


@pytest.mark.parametrize("H,W,window,P", [
    (5, 7, (1, 1), 0),         # every token alone: the result is its value row
    (5, 7, (1, 2), 0), (7, 5, (3, 1), 3), (9, 11, (2, 2), 5), (6, 6, (2, 4), 0), (3, 5, (4, 2), 0),
    (9, 11, (3, 3), 0),        # one slot more: the tiles
    (2, 4, (2, 4), 0),         # one window that spans the grid
])
def test_windows_of_a_few_slots(H, W, window, P):
    N = P + H * W
    q, k, v = synth.qkv(22, 2, 3, N, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.full_like(dq, float("nan"))
    binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window)
    grid = to_host(o)[:, :, P:]
    check(err_fp32(grid, oracle.window_attn(q[:, :, P:], k[:, :, P:], v[:, :, P:], H, W, *window)), FP32_TOL)
    assert torch.isfinite(o).all()
    if window == (1, 1):
        assert torch.equal(o, dv)
    # a score of -inf takes no part, and a value no window holds stays out of it
    if window == (2, 2):
        dk[..., P, :] = -3e38
        dv[..., P, :] = 5.0
        dv[..., P + 2, 7] = float("inf")
        binding.jv_window_attn_fwd(dq.abs() + 1, dk, dv, o, (H, W), window)
        c = torch.arange(H * W, device="cuda")
        assert torch.equal(torch.isinf(o[0, 0, P:, 7]), (c // W < 2) & (c % W // 2 == 1))
        assert not torch.isnan(o[:, :, P:]).any()


@pytest.mark.parametrize("H,W,window,P", [
    (8, 8, (64, 64), 0), (5, 9, (6, 10), 2), (1, 70, (40, 16), 0), (70, 1, (16, 40), 0), (9, 11, (4, 200), 3), (3, 5, (128, 128), 0),
])
def test_windows_beyond_the_grid_are_those_that_end_with_it(H, W, window, P):
    N = P + H * W
    q, k, v = synth.qkv(23, 2, 3, N, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o, inside = torch.full_like(dq, float("nan")), torch.full_like(dq, float("nan"))
    binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window)
    binding.jv_window_attn_fwd(dq, dk, dv, inside, (H, W), (min(window[0], H), min(window[1], W)))
    assert torch.equal(o, inside)    # the same launch
    check(err_fp32(to_host(o)[:, :, P:], oracle.window_attn(q[:, :, P:], k[:, :, P:], v[:, :, P:], H, W, *window)), FP32_TOL)


@pytest.mark.parametrize("N", [15, 16, 17, 63, 64, 65, 129, 513, 1100])
def test_linear_chunk_edges(N):
    # chunks of 64 tokens, groups of 16 in the state pass, tiles of 32 in the apply pass
    q, k, v = synth.qkv(18, 1, 3, N, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.empty_like(dq)
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (1, N), 1e-6)
    check(err_fp32(to_host(o), oracle.linear_attn_quadratic(q, k, v, 1e-6)), FP32_TOL)


# (B, heads, tokens, fused projection): one launch's tiles of 16 tokens, groups of 32 and rounds of 256; parts of the queries
# (8, 5, 2, 1, ragged last ones); either side of each limit of linear_f32_in_one
ONE_LAUNCH = [(1, 1, 1, False), (1, 1, 15, False), (1, 3, 17, True), (2, 3, 33, False), (1, 8, 255, False), (1, 6, 256, False), (1, 6, 257, True),
              (1, 8, 900, False), (1, 8, 901, False), (3, 4, 300, True), (2, 12, 700, False), (2, 12, 701, False), (1, 32, 777, True),
              (4, 16, 600, False), (4, 14, 1400, False), (4, 16, 2400, False), (5, 13, 100, False)]


@pytest.mark.parametrize("B,heads,N,fused", ONE_LAUNCH)
def test_linear_attention_in_one_launch(B, heads, N, fused):
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    if fused:
        qkv = torch.randn(B, N, 3, heads, 64, generator=g, device="cuda")
        q, k, v = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        o = torch.full((B, N, heads, 64), float("nan"), device="cuda").permute(0, 2, 1, 3)
    else:
        q, k, v = (torch.randn(B, heads, N, 64, generator=g, device="cuda") for _ in range(3))
        o = torch.full_like(q, float("nan"))
    binding.jv_linear_attn_fwd(q, k, v, o, (1, N), 1e-6)
    q64, k64 = q.double().clamp_min(0), k.double().clamp_min(0)
    ref = q64 @ (k64.transpose(-1, -2).contiguous() @ v.double()) / ((q64 * k64.sum(2, keepdim=True)).sum(-1, keepdim=True) + 1e-6)
    # 1.15e-7 is the two launches' error at these lengths (7 to 10 e-8 measured); few tokens add the rounding of a single quotient
    check(float((o.double() - ref).norm() / ref.norm()), 1.2e-7)


@pytest.mark.parametrize("heads,N", [(1, 4096), (1, 4097), (16, 4160), (17, 4160), (3, 10001), (1, 65536)])
def test_linear_attention_of_long_sequences(heads, N):
    """Above 4 096 tokens of at most 16 heads the states are summed in a pass of their own."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    q, k, v = (torch.randn(1, heads, N, 64, generator=g, device="cuda") for _ in range(3))
    o = torch.full_like(q, float("nan"))
    binding.jv_linear_attn_fwd(q, k, v, o, (1, N), 1e-6)
    q64, k64 = q.double().clamp_min(0), k.double().clamp_min(0)
    ref = q64 @ (k64.transpose(-1, -2) @ v.double()) / ((q64 * k64.sum(2, keepdim=True)).sum(-1, keepdim=True) + 1e-6)
    # sums in chunks of at most 1 024 tokens: plain fp32 sums of that length and of their 64 results
    # measured 2.11e-7 on 65 536 tokens, sums of 8 192 tokens 2.49e-7
    check(float((o.double() - ref).norm() / ref.norm()), 2.2e-7)
    focused = torch.full_like(q, float("nan"))
    ws = binding.jv_linear_block_focused_fwd(q, k, v, focused, (1, N), 3)
    f64 = [x ** 3 * (x.norm(dim=-1, keepdim=True) / (x ** 3).norm(dim=-1, keepdim=True).clamp_min(1e-300)) for x in (q64, k64)]
    ref = f64[0] @ (f64[1].transpose(-1, -2) @ v.double()) / ((f64[0] * f64[1].sum(2, keepdim=True)).sum(-1, keepdim=True) + 1e-6)
    check(float((focused.double() - ref).norm() / ref.norm()), 1e-6)
    assert ws.numel() <= 32 << 20    # (the allocation-free entry point takes what it took)
    static = torch.full_like(q, float("nan"))
    binding.jv_linear_attn_fwd_static(q, k, v, static, (1, N), 1e-6)
    assert torch.equal(static, o)


def test_long_sequence_split_reduction_fp32():
    # N large enough that the state reduction is split over several workgroups per head
    B, heads, H, W = 1, 2, 48, 50
    q, k, v = synth.qkv(8, B, heads, H * W, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.empty_like(dq)
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W), 1e-6)
    ref, _, _ = oracle.linear_attn_state(q, k, v, 1e-6)
    check(err_fp32(to_host(o), ref), FP32_TOL)


def test_strided_views_of_a_fused_qkv_buffer():
    # [B, N, 3, heads, d] as a QKV projection writes it; the mixers read it in place
    B, heads, H, W = 2, 3, 6, 10
    N = H * W
    q, k, v = synth.qkv(9, B, heads, N, 64, 1.0, False)
    fused = torch.empty(B, N, 3, heads, 64, device="cuda")
    for i, x in enumerate((q, k, v)):
        fused[:, :, i] = torch.from_numpy(x).cuda().permute(0, 2, 1, 3)
    dq, dk, dv = (fused[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    obuf = torch.empty(B, N, heads, 64, device="cuda")
    o = obuf.permute(0, 2, 1, 3)
    binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W))
    check(err_fp32(to_host(o), oracle.full_attn(q, k, v)), FP32_TOL)
    binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), (4, 4))
    check(err_fp32(to_host(o), oracle.window_attn(q, k, v, H, W, 4, 4)), FP32_TOL)
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W))
    check(err_fp32(to_host(o), oracle.linear_attn_quadratic(q, k, v, 1e-6)), FP32_TOL)


def test_non_default_scale_and_eps():
    B, heads, H, W = 1, 2, 8, 8
    q, k, v = synth.qkv(10, B, heads, H * W, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (q, k, v))
    o = torch.empty_like(dq)
    binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W), scale=0.05)
    check(err_fp32(to_host(o), oracle.full_attn(q, k, v, scale=0.05)), FP32_TOL)
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W), eps=3.0)
    check(err_fp32(to_host(o), oracle.linear_attn_quadratic(q, k, v, 3.0)), FP32_TOL)


def test_all_negative_queries_give_exact_zero():
    B, heads, H, W = 1, 1, 4, 4
    q, k, v = synth.qkv(11, B, heads, H * W, 64, 1.0, False)
    dq, dk, dv = (to_device(x, False) for x in (-np.abs(q), k, v))
    o = torch.full_like(dq, 7.0)
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W))
    assert torch.count_nonzero(o).item() == 0


def test_device_maps_are_bit_exact():
    for H, W, wh, ww in [(3, 3, 2, 2), (37, 37, 8, 8), (64, 64, 16, 16), (16, 16, 8, 8),
                         (5, 9, 4, 2), (256, 256, 16, 16), (7, 7, 9, 3)]:
        ti, pm, wt = binding.jv_window_maps_device(H, W, wh, ww)
        want = oracle.window_maps(H, W, wh, ww)
        for g, w in zip((ti, pm, wt), want):
            g = g.cpu().numpy()
            assert g.dtype == w.dtype and g.shape == w.shape and g.tobytes() == w.tobytes()


def test_padding_never_reaches_the_output():
    # window attention on a ragged grid: poison everything around the tensors with NaN
    B, heads, H, W = 1, 2, 5, 7
    N = H * W
    q, k, v = synth.qkv(12, B, heads, N, 64, 1.0, False)
    big = torch.full((3, B, heads, N + 8, 64), float("nan"), device="cuda")
    views = []
    for i, x in enumerate((q, k, v)):
        big[i, :, :, 4:4 + N] = torch.from_numpy(x).cuda()
        views.append(big[i, :, :, 4:4 + N])
    o = torch.empty(B, heads, N, 64, device="cuda")
    binding.jv_window_attn_fwd(*views, o, (H, W), (4, 4))
    check(err_fp32(to_host(o), oracle.window_attn(q, k, v, H, W, 4, 4)), FP32_TOL)

def test_padding_takes_no_part_where_values_are_infinite():
    # padded keys stand in for the window's first token, absent partial states for the last one:
    # an infinity there stays what the sums make of it (0 x inf would turn it into NaN)
    H = W = 6
    q, k, v = (torch.rand(1, 1, H * W, 64, device="cuda") + 0.1 for _ in range(3))
    v[..., 0, 5] = v[..., 4, 7] = float("inf")       # first tokens of the windows at (0, 0) and (0, 4)
    o = torch.empty_like(q)
    binding.jv_window_attn_fwd(q, k, v, o, (H, W), (4, 4))
    first = torch.zeros(H, W, dtype=torch.bool, device="cuda")
    second = first.clone()
    first[:4, :4] = True
    second[:4, 4:] = True
    assert torch.equal(torch.isinf(o[0, 0, :, 5]), first.flatten())
    assert torch.equal(torch.isinf(o[0, 0, :, 7]), second.flatten())
    assert not torch.isnan(o).any()
    N = 190                                            # three partial states, summed four at a time
    q, k, v = (torch.rand(1, 1, N, 64, device="cuda") + 0.1 for _ in range(3))
    v[..., N - 1, 5] = float("inf")
    o = torch.empty_like(q)
    binding.jv_linear_attn_fwd(q, k, v, o, (1, N))
    assert torch.isinf(o[..., 5]).all() and not torch.isnan(o).any()
    assert torch.isfinite(o[..., 6:]).all()


def test_linear_denominators_without_a_finite_reciprocal():
    # eps = 0 and a denominator of 64 * 2^-67 * 2^-67 = 2^-128, whose reciprocal is 2^128 = inf in
    # fp32; the result is the one live value row, up to the roundings of its sum over 64 equal
    # channels (63 additions, each within 2^-24 of the sum so far)
    N = 5
    q = torch.full((1, 2, N, 64), 2.0 ** -67, device="cuda")
    k = torch.full_like(q, -1.0)
    k[:, :, 0] = 2.0 ** -67
    v = torch.from_numpy(synth.normal((1, 2, N, 64), 19)).cuda() * 2.0 ** 40
    o = torch.empty_like(q)
    binding.jv_linear_attn_fwd(q, k, v, o, (1, N), 0.0)
    check(err_fp32(to_host(o), to_host(v[:, :, :1].expand_as(o))), 64 * 2.0 ** -24)


class _LikeATensor:
    """Has what the binding asks of a tensor, without being one."""
    def __init__(self, t):
        self.t = t

    def __getattr__(self, name):
        return getattr(self.t, name)


def test_calls_take_every_form_of_their_arguments():
    # the compiled marshalling takes tensors and pairs in tuples or lists; the rest goes through ctypes
    H, W, N = 8, 6, 48
    dq, dk, dv = (to_device(x, False) for x in synth.qkv(20, 1, 2, N, 64, 1.0, False))
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    sq = tuple(torch.from_numpy(a).cuda() for a in synth.squeeze_weights(128, 16, 3, 21))

    def result(call, *args, **kwargs):
        o = torch.full_like(dq, float("nan"))
        call(dq, dk, dv, o, *args, **kwargs)
        assert torch.isfinite(o).all()
        return o
    want = result(binding.jv_window_attn_fwd, (H, W), (4, 4))
    for window in ([4, 4], (4, 4, 1), torch.tensor([4, 4]), np.array([4, 4]), {0: 4, 1: 4}):
        assert torch.equal(result(binding.jv_window_attn_fwd, (H, W), window), want)
    for grid in ([H, W], torch.Size((H, W)), np.array([H, W]), (n for n in (H, W))):
        assert torch.equal(result(binding.jv_window_attn_fwd, grid, (4, 4)), want)
    o = torch.full_like(dq, float("nan"))
    binding.jv_window_attn_fwd(*(_LikeATensor(t) for t in (dq, dk, dv, o)), (H, W), (4, 4))
    assert torch.equal(o, want)
    for call, kwargs in ((binding.jv_linear_attn_fwd, {}), (binding.jv_linear_block_fwd, {"squeeze": sq}),
                         (binding.jv_linear_block_focused_fwd, {"focus_p": 3, "squeeze": sq})):
        want = result(call, (H, W), workspace=ws, **kwargs)
        assert torch.equal(result(call, (H, W), workspace=_LikeATensor(ws), **kwargs), want)
        if kwargs:
            kwargs["squeeze"] = [_LikeATensor(t) for t in sq]
            assert torch.equal(result(call, (H, W), workspace=ws, **kwargs), want)
    for focus_p in (0, 17, np.int64(0)):
        with pytest.raises(binding.JvError):
            result(binding.jv_linear_block_focused_fwd, (H, W), focus_p, workspace=ws)
    for call in (binding.jv_full_attn_fwd, binding.jv_linear_attn_fwd, binding.jv_linear_block_fwd):
        assert torch.equal(result(call, (n for n in (H, W)), stream=torch.cuda.current_stream()), result(call, (H, W)))
