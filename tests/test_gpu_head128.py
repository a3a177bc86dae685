"""GPU parity at head_dim 128 (the wide heads of the paper's largest backbones, Tab. 3/4): full
and window attention (Eq. 1, Sec. 3.2.2) and linear attention (Eq. 2) on bf16 tensors against
the CPU oracle, which is written for any head width.

Tolerance as for 64 channels: max |g - r| / RMS(r) <= 2e-2 on the fp32-output run; the
bf16-output run is its nearest-even rounding, bit for bit (parity.check_bf16_pair)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_26636_amd import binding, synth
from parity import BF16_TOL, check, check_bf16_pair, err_bf16, rows_of, to_device, to_host

pytestmark = pytest.mark.gpu

D = 128


def _full(q, k, v, H, W, out_dtype=torch.bfloat16, scale=0.0):
    dq, dk, dv = (to_device(x, True) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), dtype=out_dtype, device="cuda")
    binding.jv_full_attn_fwd(dq, dk, dv, o, (H, W), scale)
    torch.cuda.synchronize()
    return o


def _window(q, k, v, H, W, window, out_dtype=torch.bfloat16, scale=0.0):
    dq, dk, dv = (to_device(x, True) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), dtype=out_dtype, device="cuda")
    binding.jv_window_attn_fwd(dq, dk, dv, o, (H, W), window, scale)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("B,heads,H,W,vscale", [
    (2, 3, 16, 16, 1.0),    # N = 256: two query blocks of 128, eight key stages; peaked softmax
    (1, 2, 37, 37, 0.125),  # N = 1369: ragged query block and ragged key stage
    (1, 2, 5, 7, 1.0),      # N = 35: one stage and three keys
    (1, 1, 1, 1, 1.0),      # a single token
    (2, 2, 24, 40, 0.5),    # N = 960 = 30 stages
    (1, 2, 33, 33, 1.0),    # N = 1089: a one-key tail
    (1, 1, 1, 31, 1.0),     # less than one stage
    (1, 2, 8, 8, 1.0),      # exactly two stages
    (1, 1, 8, 12, 0.5),     # exactly three: once round the ring
    (2, 1, 8, 16, 1.0),     # four
    (1, 1, 10, 16, 1.0),    # five
    (1, 1, 3, 43, 1.0),     # N = 129: four stages and one key
])
def test_full_attention_small_shapes(B, heads, H, W, vscale):
    q, k, v = synth.qkv(60, B, heads, H * W, D, vscale, True)
    ref = oracle.full_attn(q, k, v)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32), _full(q, k, v, H, W), ref)


@pytest.mark.parametrize("B,heads,H,W,window,vscale", [
    (2, 2, 16, 16, (8, 8), 1.0),      # 64-slot windows
    (1, 2, 37, 37, (8, 8), 0.125),    # padded 40 x 40, windows of 64 / 40 / 25 real tokens
    (1, 2, 32, 48, (16, 16), 0.5),    # 256-slot windows
    (2, 1, 7, 9, (4, 4), 1.0),        # tiny ragged windows: less than one stage
    (1, 2, 20, 20, (32, 32), 1.0),    # window larger than the grid: whole stages of padding
    (1, 2, 18, 30, (6, 30), 1.0),     # windows spanning whole rows
    (1, 1, 40, 24, (24, 16), 0.5),    # 384-slot rectangular windows, ragged at the bottom
    (1, 1, 17, 40, (16, 16), 0.5),    # bottom windows hold one real row: seven stages of padding
    (1, 2, 16, 64, (8, 32), 0.5),     # windows as wide as a key stage (one window row per stage)
    (1, 1, 8, 8, (8, 2), 1.0),        # narrow windows: sixteen window rows per stage
    (2, 1, 6, 5, (3, 1), 1.0),        # one-column windows of three tokens: less than a stage
    (1, 1, 48, 4, (24, 4), 0.5),      # 96-slot windows: three stages exactly
    (1, 1, 10, 8, (5, 8), 1.0),       # whole-row windows of 40 tokens: a stage and a quarter
])
def test_window_attention_small_shapes(B, heads, H, W, window, vscale):
    q, k, v = synth.qkv(61, B, heads, H * W, D, vscale, True)
    ref = oracle.window_attn(q, k, v, H, W, *window)
    check_bf16_pair(_window(q, k, v, H, W, window, torch.float32), _window(q, k, v, H, W, window), ref)


def test_default_scale_is_one_over_sqrt_128_and_explicit_scale():
    B, heads, H, W = 1, 2, 10, 10
    q, k, v = synth.qkv(62, B, heads, H * W, D, 1.0, True)
    ref = oracle.full_attn(q, k, v)                       # the oracle's default: 1/sqrt(d)
    check(err_bf16(to_host(_full(q, k, v, H, W, torch.float32)), ref), BF16_TOL)
    ref = oracle.full_attn(q, k, v, scale=0.3)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32, 0.3), _full(q, k, v, H, W, scale=0.3), ref)


def test_large_logits_need_the_running_maximum():
    B, heads, H, W = 1, 1, 16, 32
    q, k, v = synth.qkv(63, B, heads, H * W, D, 1.0, True)
    ramp = np.linspace(0.2, 6.0, H * W, dtype=np.float32).reshape(1, 1, -1, 1)
    k = synth.round_to_bf16(k * ramp)
    ref = oracle.full_attn(q, k, v)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32), _full(q, k, v, H, W), ref)


def test_prefix_tokens():
    """Prefix tokens in front of the grid: window rule of the library (grid tokens attend inside
    their window, prefix tokens to everything) and full attention over all tokens."""
    B, heads, H, W, P = 2, 2, 12, 9, 5
    q, k, v = synth.qkv(64, B, heads, P + H * W, D, 0.5, True)
    ref = oracle.window_attn_prefix(q, k, v, P, H, W, 4, 4)
    check_bf16_pair(_window(q, k, v, H, W, (4, 4), torch.float32), _window(q, k, v, H, W, (4, 4)), ref)
    ref = oracle.full_attn(q, k, v)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32), _full(q, k, v, H, W), ref)


def test_prefix_tokens_with_unpadded_windows():
    """The same rule where the grid part runs on the ring kernel (windows that tile the grid, their
    width a divisor of the 32-key stage) and the prefix queries on the query-slot limit."""
    B, heads, P = 2, 2, 5
    for H, W, window in [(8, 8, (4, 4)), (16, 32, (16, 16)), (6, 16, (3, 8))]:
        q, k, v = synth.qkv(67, B, heads, P + H * W, D, 0.5, True)
        ref = oracle.window_attn_prefix(q, k, v, P, H, W, *window)
        check_bf16_pair(_window(q, k, v, H, W, window, torch.float32), _window(q, k, v, H, W, window), ref)


def test_fused_projection_layout_and_rerun_bits():
    """Q, K, V as strided views of one [B, N, 3, heads, 128] buffer (the layout a fused QKV
    projection leaves), O as [B, N, heads, 128]; several launches give the same bits."""
    B, heads, H, W = 2, 3, 20, 12
    N = H * W
    q, k, v = synth.qkv(65, B, heads, N, D, 0.5, True)
    fused = torch.empty(B, N, 3, heads, D, device="cuda", dtype=torch.bfloat16)
    for i, x in enumerate((q, k, v)):
        fused[:, :, i] = to_device(x, True).permute(0, 2, 1, 3)
    views = [fused[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    out = torch.empty(B, N, heads, D, device="cuda", dtype=torch.bfloat16)
    o = out.permute(0, 2, 1, 3)
    binding.jv_window_attn_fwd(*views, o, (H, W), (8, 8))
    assert torch.equal(o, _window(q, k, v, H, W, (8, 8)))
    first = o.clone()
    for _ in range(4):
        binding.jv_window_attn_fwd(*views, o, (H, W), (8, 8))
        assert torch.equal(o, first)
    binding.jv_full_attn_fwd(*views, o, (H, W))
    assert torch.equal(o, _full(q, k, v, H, W))
    binding.jv_window_attn_fwd(*views, o, (H, W), (4, 4))   # windows that tile the grid: the ring kernel
    assert torch.equal(o, _window(q, k, v, H, W, (4, 4)))
    first = o.clone()
    for _ in range(4):
        binding.jv_window_attn_fwd(*views, o, (H, W), (4, 4))
        assert torch.equal(o, first)


def test_prefix_in_views_with_wide_token_strides():
    """Tokens 3 072 elements apart, as in the fused projection of eight heads, and so many of them that 64 times the sequence
    (the sequence is one row of its geometry) spans more bytes than 32 bits count: the bits of separate tensors, and the
    oracle's rows.  P = 5 takes the chains, 1 369 tokens the same rule on its other side."""
    heads, P = 2, 5
    for H, W in [(64, 85), (37, 37)]:
        N = P + H * W
        q, k, v = synth.qkv(71, 1, heads, N, D, 0.125, True)
        fused = torch.empty(1, N, 3, 8, D, device="cuda", dtype=torch.bfloat16)
        for i, x in enumerate((q, k, v)):
            fused[:, :, i, :heads] = to_device(x, True).permute(0, 2, 1, 3)
        views = [fused[:, :, i, :heads].permute(0, 2, 1, 3) for i in range(3)]
        o = torch.empty(1, N, heads, D, device="cuda", dtype=torch.bfloat16).permute(0, 2, 1, 3)
        binding.jv_window_attn_fwd(*views, o, (H, W), (16, 16))
        assert torch.equal(o, _window(q, k, v, H, W, (16, 16)))
        binding.jv_full_attn_fwd(*views, o, (H, W))
        assert torch.equal(o, _full(q, k, v, H, W))
        rows = synth.sample_rows(1, heads, N, 64, seed=7)
        check_bf16_pair(_full(q, k, v, H, W, torch.float32), o, oracle.full_attn_rows(q, k, v, rows), rows)


def test_vit_layer_size_elementwise():
    """A layer of the benchmark's size with wide heads (batch 8, 64 x 64 grid, 8 heads x 128):
    every element of window and full attention against the oracle."""
    B, heads, H, W = 8, 8, 64, 64
    q, k, v = synth.qkv(66, B, heads, H * W, D, 0.125, True)
    ref = oracle.window_attn(q, k, v, H, W, 16, 16)
    check_bf16_pair(_window(q, k, v, H, W, (16, 16), torch.float32), _window(q, k, v, H, W, (16, 16)), ref)
    ref = oracle.full_attn(q, k, v)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32), _full(q, k, v, H, W), ref)


def test_long_sequences_sampled_rows():
    """One image of 256 x 256 tokens (65 536): the state pass splits the tokens over many chunks,
    window attention walks 256 windows per head through the ring; and full attention on 16 384
    tokens (512 key stages).  Sampled rows against the oracle."""
    B, heads, H, W = 1, 2, 256, 256
    q, k, v = synth.qkv(68, B, heads, H * W, D, 0.125, True)
    rows = synth.sample_rows(B, heads, H * W, 96, seed=5)
    ref = oracle.linear_attn_rows(q, k, v, rows, 1e-6)
    check_bf16_pair(_linear(q, k, v, H, W, torch.float32), _linear(q, k, v, H, W), ref, rows)
    ref = oracle.window_attn_rows(q, k, v, H, W, 16, 16, rows)
    check_bf16_pair(_window(q, k, v, H, W, (16, 16), torch.float32), _window(q, k, v, H, W, (16, 16)), ref, rows)
    H = W = 128
    q, k, v = synth.qkv(69, B, heads, H * W, D, 0.125, True)
    rows = synth.sample_rows(B, heads, H * W, 96, seed=6)
    ref = oracle.full_attn_rows(q, k, v, rows)
    check_bf16_pair(_full(q, k, v, H, W, torch.float32), _full(q, k, v, H, W), ref, rows)


def test_fp32_tensors_are_refused():
    q = torch.zeros(1, 1, 16, D, device="cuda")
    with pytest.raises(binding.JvError) as e:
        binding.jv_full_attn_fwd(q, q.clone(), q.clone(), torch.empty_like(q), (4, 4))
    assert e.value.status == binding.JV_ERR_UNSUPPORTED


def _linear(q, k, v, H, W, out_dtype=torch.bfloat16, eps=1e-6):
    dq, dk, dv = (to_device(x, True) for x in (q, k, v))
    o = torch.full(dq.shape, float("nan"), dtype=out_dtype, device="cuda")
    binding.jv_linear_attn_fwd(dq, dk, dv, o, (H, W), eps)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("B,heads,H,W,vscale", [
    (2, 3, 16, 16, 1.0),     # one chunk per head
    (1, 2, 37, 37, 0.125),   # ragged last tile
    (1, 2, 5, 7, 1.0),       # less than one tile
    (1, 1, 1, 1, 1.0),       # a single token
    (1, 1, 64, 80, 0.5),     # 5 120 tokens: several chunks per head, partial states combined
    (2, 2, 33, 31, 0.5),     # 1 023 tokens
])
def test_linear_attention_small_shapes(B, heads, H, W, vscale):
    q, k, v = synth.qkv(67, B, heads, H * W, D, vscale, True)
    ref = oracle.linear_attn_quadratic(q, k, v, 1e-6)
    check_bf16_pair(_linear(q, k, v, H, W, torch.float32), _linear(q, k, v, H, W), ref)


def test_linear_attention_vit_layer_size_elementwise_and_rerun_bits():
    B, heads, H, W = 8, 8, 64, 64
    q, k, v = synth.qkv(68, B, heads, H * W, D, 0.125, True)
    ref = oracle.linear_attn_state(q, k, v, 1e-6)[0]
    o = _linear(q, k, v, H, W)
    check_bf16_pair(_linear(q, k, v, H, W, torch.float32), o, ref)
    for _ in range(3):
        assert torch.equal(_linear(q, k, v, H, W), o)


def test_linear_attention_prefix_and_fused_layout():
    """Prefix tokens are ordinary tokens of linear attention; Q, K, V as views of a fused
    [B, N, 3, heads, 128] buffer give the same bits as contiguous tensors."""
    B, heads, H, W, P = 2, 3, 20, 12, 4
    N = P + H * W
    q, k, v = synth.qkv(69, B, heads, N, D, 0.5, True)
    ref = oracle.linear_attn_quadratic(q, k, v, 1e-6)
    o = _linear(q, k, v, H, W)
    check_bf16_pair(_linear(q, k, v, H, W, torch.float32), o, ref)
    fused = torch.empty(B, N, 3, heads, D, device="cuda", dtype=torch.bfloat16)
    for i, x in enumerate((q, k, v)):
        fused[:, :, i] = to_device(x, True).permute(0, 2, 1, 3)
    views = [fused[:, :, i].permute(0, 2, 1, 3) for i in range(3)]
    out = torch.empty(B, N, heads, D, device="cuda", dtype=torch.bfloat16).permute(0, 2, 1, 3)
    binding.jv_linear_attn_fwd(*views, out, (H, W))
    assert torch.equal(out, o)


@pytest.mark.parametrize("ksize", [3, 5])
@pytest.mark.parametrize("B,heads,H,W,P", [(2, 2, 13, 11, 0), (1, 3, 37, 37, 0), (1, 1, 1, 1, 0), (2, 2, 12, 9, 5)])
def test_linear_block_static_and_squeeze_dynamic(B, heads, H, W, P, ksize):
    """The paper's linear-attention block (Eq. 4) on 128-channel heads: static filters and the
    squeeze-dynamic generator, against the oracle; prefix tokens get no convolution term."""
    C, hidden = heads * D, 8
    q, k, v = synth.qkv(70, B, heads, P + H * W, D, 0.5, True)
    kern = synth.dwc_static_kernel(C, ksize, 7400 + ksize)
    sq = synth.squeeze_weights(C, hidden, ksize, 7500 + ksize)
    dev = lambda *a: tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in a)

    def block(out_dtype, **kw):
        dq, dk, dv = (to_device(x, True) for x in (q, k, v))
        o = torch.full(dq.shape, float("nan"), dtype=out_dtype, device="cuda")
        binding.jv_linear_block_fwd(dq, dk, dv, o, (H, W), 1e-6, ksize=ksize, **kw)
        torch.cuda.synchronize()
        return o

    ref = oracle.linear_block(q, k, v, H, W, 1e-6, static_kernel=kern, ksize=ksize)
    check_bf16_pair(block(torch.float32, static_kernel=dev(kern)[0]), block(torch.bfloat16, static_kernel=dev(kern)[0]), ref)
    ref = oracle.linear_block(q, k, v, H, W, 1e-6, squeeze=sq, ksize=ksize)
    check_bf16_pair(block(torch.float32, squeeze=dev(*sq)), block(torch.bfloat16, squeeze=dev(*sq)), ref)


# (B, heads, tokens): one chunk of one team of wavefronts (1 to 256 tokens); one chunk of two teams, 5 and 6 tiles of 64, the last one with 1 and
# 10 tokens; chunks of two teams, the last one with 1, 64, 65 and 76 tokens; as many chunks of one team; apply ranges of 1 to 8 tiles
CHUNKS = [(1, 2, 1), (1, 2, 63), (1, 3, 65), (2, 2, 256), (64, 4, 257), (64, 4, 330), (64, 4, 512), (8, 8, 1025), (8, 8, 1088), (8, 8, 1089), (8, 8, 1100),
          (1, 2, 300), (1, 3, 1000), (4, 8, 4096)]


@pytest.mark.parametrize("B,heads,N", CHUNKS)
@pytest.mark.parametrize("fused", [False, True])
def test_linear_attention_chunks_of_wide_heads(B, heads, N, fused):
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    if fused:
        qkv = torch.randn(B, N, 3, heads, 128, generator=g, device="cuda").to(torch.bfloat16)
        q, k, v = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
    else:
        q, k, v = (torch.randn(B, heads, N, 128, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    o = torch.full((B, heads, N, 128), float("nan"), device="cuda")
    binding.jv_linear_attn_fwd(q, k, v, o, (1, N), 1e-6)
    q64, k64 = q.double().clamp_min(0), k.double().clamp_min(0)
    ref = q64 @ (k64.transpose(-1, -2).contiguous() @ v.double()) / ((q64 * k64.sum(2, keepdim=True)).sum(-1, keepdim=True) + 1e-6)
    # state and normaliser as two bf16 numbers: 2^-17 of a number, at random in sums of 128
    check(float((o.double() - ref).norm() / ref.norm()), 2.0 ** -17)
    o16 = torch.empty_like(o, dtype=torch.bfloat16)
    binding.jv_linear_attn_fwd(q, k, v, o16, (1, N), 1e-6)
    assert torch.equal(o16, o.to(torch.bfloat16))


def test_linear_block_variants_refused_for_wide_heads():
    """The focused map and token-wise filters are built for 64-channel heads."""
    B, heads, H, W = 1, 1, 4, 4
    q = torch.zeros(B, heads, H * W, D, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(binding.JvError) as e:
        binding.jv_linear_block_focused_fwd(q, q.clone(), q.clone(), torch.empty_like(q), (H, W), 3)
    assert e.value.status == binding.JV_ERR_UNSUPPORTED
    tok = tuple(torch.from_numpy(a).cuda() for a in synth.squeeze_weights(heads * D, 64, 3, 7600))
    with pytest.raises(binding.JvError) as e:
        binding.jv_linear_block_fwd(q, q.clone(), q.clone(), torch.empty_like(q), (H, W), token=tok)
    assert e.value.status in (binding.JV_ERR_UNSUPPORTED, binding.JV_ERR_WORKSPACE_TOO_SMALL)


def _device_blocks(blocks):
    return [{k: (torch.from_numpy(v).cuda().to(torch.bfloat16) if k.startswith("w_") else torch.from_numpy(v).cuda())
             for k, v in b.items()} for b in blocks]


@pytest.mark.parametrize("fold", [False, True], ids=["layernorm passes", "layernorm folded"])
def test_encoder_with_wide_heads(fold):
    """A small hybrid encoder whose width is heads x 128 (the head width follows from width and
    heads): every mixer type, a mixed pattern, prefix tokens, against the oracle's encoder."""
    B, H, W, heads, hidden = 2, 8, 8, 2, 512
    C = heads * D
    blocks = [synth.block_weights(C, hidden, 7100 + i) for i in range(3)]
    for b in blocks:
        for key in ("b_qkv", "b_o", "b_fc1", "b_fc2", "ln1_b", "ln2_b"):
            b[key] = synth.normal(b[key].shape, 7200 + len(key)) * 0.1
    dev = _device_blocks(blocks)
    for pattern, P in (([0, 0, 0], 0), ([1, 1, 1], 0), ([2, 2, 2], 0), ([0, 1, 2], 0), ([1, 0, 2], 3)):
        x = synth.normal((B, P + H * W, C), 7000 + P)
        dx = torch.from_numpy(x).cuda()
        enc = binding.Encoder(dev, pattern, heads, hidden, window=(4, 4), n_prefix=P, fold_layernorm=fold)
        y = torch.empty_like(dx)
        enc.forward(dx, y, (H, W))
        ref = oracle.encoder_forward(x, blocks, pattern, H, W, heads, window=(4, 4), n_prefix=P)
        check(err_bf16(to_host(y), ref), BF16_TOL)
        enc.close()


def test_encoder_wide_heads_block_variants():
    """Linear-attention blocks of a wide-head encoder carry the convolution branch (squeeze-dynamic
    and static filters) like 64-channel ones; the focused map is refused."""
    B, H, W, heads, hidden = 2, 12, 10, 2, 256
    C = heads * D
    x = synth.normal((B, H * W, C), 7700)
    blocks = [synth.block_weights(C, hidden, 7710 + i) for i in range(3)]
    blocks[0]["dwc"] = {"squeeze": synth.squeeze_weights(C, 8, 3, 7720), "ksize": 3}
    blocks[2]["dwc"] = {"static_kernel": synth.dwc_static_kernel(C, 5, 7721), "ksize": 5}
    dev = _device_blocks([{k: v for k, v in b.items() if k != "dwc"} for b in blocks])
    dev[0]["dwc"] = {"squeeze": tuple(torch.from_numpy(a).cuda() for a in blocks[0]["dwc"]["squeeze"]), "ksize": 3}
    dev[2]["dwc"] = {"static_kernel": torch.from_numpy(blocks[2]["dwc"]["static_kernel"]).cuda(), "ksize": 5}
    pattern = [0, 1, 0]
    enc = binding.Encoder(dev, pattern, heads, hidden, window=(4, 5))
    dx = torch.from_numpy(x).cuda()
    y = torch.empty_like(dx)
    enc.forward(dx, y, (H, W))
    ref = oracle.encoder_forward(x, blocks, pattern, H, W, heads, window=(4, 5))
    check(err_bf16(to_host(y), ref), BF16_TOL)
    enc.close()
    with pytest.raises(binding.JvError) as e:
        binding.Encoder(_device_blocks([synth.block_weights(C, hidden, 7730)]), [0], heads, hidden, window=(4, 4), la_focus_p=3)
    assert e.value.status == binding.JV_ERR_UNSUPPORTED
