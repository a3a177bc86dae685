"""The rules that choose kernels by sizes (csrc/jv_plan.h), on the host: a small program compiled
against the header answers what the launchers would choose."""
import os
import shutil
import subprocess

import pytest

import test_gpu_bf16_attn
import test_gpu_bf16_linear
import test_gpu_fp32
import test_gpu_linear_block
import test_gpu_prefix

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_26636_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule(expressions): the values of C++ integer expressions over namespace jv."""
    def ask(expressions):
        d = tmp_path_factory.mktemp("rules")
        lines = "".join(f'    std::printf("%lld\\n", (long long)({e}));\n' for e in expressions)
        (d / "main.cpp").write_text('#include <cstdio>\n#include "jv_plan.h"\nusing namespace jv;\nint main() {\n' + lines + "}\n")
        exe = str(d / "rules")
        # (signed overflow in a rule ends the program)
        cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-static-libubsan",
               "-Wall", "-I", CSRC, str(d / "main.cpp"), "-o", exe]
        built = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert built.returncode == 0, built.stdout
        ran = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
        assert ran.returncode == 0, ran.stdout
        return [int(x) for x in ran.stdout.split()]
    return ask


def test_ring_of_v_rows_at_every_width(rule):
    """The ring's bytes are counted without wrapping, so grids of up to 2^24 columns never pass for small ones."""
    sizes = [(k, w) for k in (3, 5) for w in (1, 3, 64, 85, 86, 128, 172, 173, 1 << 10, 1 << 20, 1 << 22, 1 << 23, (1 << 24) - 1, 1 << 24)]
    got = rule([f"conv_ring_lds({k}, {w})" for k, w in sizes])
    for (k, w), lds in zip(sizes, got):
        rows = 128 + 2 * (k // 2) * (w + 1) + 32
        assert lds == 65 * 64 * 4 + 512 + rows * 128
    most, = rule(["kRingMostLds"])
    assert {(k, w) for (k, w), lds in zip(sizes, got) if lds <= most} == {
        (k, w) for k, w in sizes if w <= (172 if k == 3 else 85)}


def test_ring_or_direct_loads_of_v(rule):
    """(ksize, generated filters, W, N, workgroups) on either side of every line of the rule, and the launches that
    the GPU tests of the ring count on."""
    direct = [(3, 0, 14, 196, 12), (3, 0, 85, 3400, 168), (3, 0, 64, 4096, 256), (5, 0, 37, 1369, 96), (3, 1, 37, 1369, 96), (3, 1, 16, 257, 256),
              (3, 0, 173, 4096, 4096), (5, 0, 86, 4096, 4096), (3, 0, 1 << 24, 1 << 24, 8192), (5, 0, 1 << 23, 1 << 23, 4096)]
    ring = [(3, 0, 10, 100, 12), (3, 0, 16, 128, 4), (3, 1, 16, 256, 4), (3, 0, 64, 4096, 257), (5, 1, 37, 1369, 96), (3, 1, 128, 8192, 512), (3, 0, 172, 4096, 4096), (5, 0, 85, 4096, 4096)]
    got = rule([f"conv_takes_ring({k}, {g}, {w}, {n}, {wg})" for k, g, w, n, wg in direct + ring])
    assert got == [0] * len(direct) + [1] * len(ring)

    shapes = [(k, w, p + h * w) for k, h, w, p in test_gpu_linear_block.WINDOW_OF_V]
    rounds = rule([f"apply_rounds(512, {n})" for _, _, n in shapes])
    many = rule([f"conv_takes_ring({k}, 0, {w}, {n}, 512 * (({n} + 256 * {r} - 1) / (256 * {r})))" for (k, w, n), r in zip(shapes, rounds)])
    alone = rule([f"conv_takes_ring({k}, 0, {w}, {n}, 2 * (({n} + 255) / 256))" for k, w, n in shapes])
    steps = [(min(n, 256 * r) + 127) // 128 for (_, _, n), r in zip(shapes, rounds)]
    assert many == [w <= (172 if k == 3 else 85) for k, w, _ in shapes] and not any(alone)
    assert min(steps) == 3 and max(steps) == 16 and sum(s >= 8 for s in steps) >= 12

    for k, h, w, p in test_gpu_linear_block.RING_OR_DIRECT:
        n = p + h * w
        assert rule([f"conv_takes_ring({k}, 0, {w}, {n}, {wg} * (({n} + 256 * apply_rounds({wg}, {n}) - 1) / (256 * apply_rounds({wg}, {n}))))"
                     for wg in (256, 258)]) == [0, 1]


def test_query_blocks_of_full_attention(rule):
    """(queries, lanes) on either side of the rule, as measured, and the sizes that the GPU test of equal bits counts on."""
    one, two = [(1374, 16), (1374, 32), (1374, 48), (5184, 16), (100, 512), (200, 1)], [(8192, 16), (4096, 64), (4096, 128), (256, 400)]
    either, same = test_gpu_bf16_attn.EITHER_SIZE, [c for c in test_gpu_bf16_attn.ONE_SIZE if c[0] > 64]
    ask = one + two + either + [(n, 1) for n, _ in either] + same + [(n, 1) for n, _ in same]
    got = rule([f"ring_query_blocks({n}, {lanes})" for n, lanes in ask])
    assert got == [1] * len(one) + [2] * (len(two) + len(either)) + [1] * (len(either) + 2 * len(same))


def test_key_groups_of_full_attention(rule):
    """(queries, keys, lanes) on either side of the rule, and the sizes that the GPU test of key groups counts on."""
    one, two = [(671, 671, 1), (641, 641, 1), (1374, 1374, 35), (4096, 4096, 13), (64, 672, 769), (1 << 24, 1 << 24, 65535)], [
        (672, 672, 1), (1374, 1374, 34), (4096, 4096, 12), (64, 672, 768), (49152, 49152, 1)]
    two += [(n, n, lanes) for n, lanes in test_gpu_bf16_attn.KEY_GROUPS]
    got = rule([f"ring_key_groups({q}, {k}, {lanes})" for q, k, lanes in one + two])
    assert got == [1] * len(one) + [2] * len(two)


def test_staged_or_direct_keys_of_fp32_attention(rule):
    """(tiles, whole rows, blocks of 32 queries, bytes of a slice of K and V)"""
    staged = [(4, 1, 24, 1 << 15), (4, 1, 512, 1 << 15), (4, 1, 1024, 1 << 15), (4, 1, 1280, 1 << 15), (4, 1, 2040, 1 << 15),
              (10, 1, 10, (300 + 64) * 2949844 * 4), (10, 0, 10, 1 << 40)]
    direct = [(3, 1, 24, 1 << 15), (5, 1, 24, 1 << 15), (4, 0, 24, 1 << 15), (4, 1, 513, 1 << 15), (4, 1, 768, 1 << 15), (4, 1, 1536, 1 << 15),
              (43, 1, 516, 1 << 19), (10, 1, 10, (300 + 64) * 2949840 * 4)]
    got = rule([f"f32_keys_staged({t}, {r}, {w}, {b}ll)" for t, r, w, b in staged + direct])
    assert got == [1] * len(staged) + [0] * len(direct)


def test_kernels_of_fp32_attention(rule):
    """(tiles, whole rows, queries of a window, windows times (batch, head)s, bytes of a slice) on either side of every line of the rule."""
    want = {"kF32Short1": [(1, 1, 32, 1, 0), (1, 0, 9, 1 << 20, 1 << 40)], "kF32Short2": [(2, 1, 64, 1, 0), (2, 0, 49, 320, 1 << 40)],
            "kF32Short4": [(4, 1, 128, 1, 0), (4, 1, 128, 128, 0), (10, 1, 320, 1, 1 << 32), (57, 0, 1824, 22, 1 << 40)],
            "kF32Few": [(3, 1, 96, 170, 0), (4, 0, 128, 128, 0), (4, 0, 5, 600, 0), (5, 1, 160, 102, 0), (7, 0, 224, 109, 0), (7, 1, 224, 146, 0), (8, 1, 256, 160, 0), (16, 0, 512, 48, 0),
                        (17, 1, 544, 60, 0), (43, 1, 1369, 12, (1 << 32) - 1), (43, 1, 1369, 35, 0), (72, 1, 2304, 21, 0), (43, 1, 5, 4096, 0), (25, 1, 800, 74, 0), (25, 1, 800, 81, 0)],
            "kF32Many": [(2, 1, 64, 321, 0), (3, 1, 96, 171, 0), (4, 1, 128, 129, 0), (4, 0, 128, 225, 0), (5, 1, 160, 103, 0), (7, 0, 224, 110, 0), (7, 1, 224, 147, 0), (8, 1, 256, 161, 0),
                         (16, 0, 512, 49, 0), (18, 1, 576, 86, 0), (43, 1, 1369, 36, 0), (72, 1, 2304, 22, 0), (25, 1, 800, 73, 0), (25, 1, 800, 82, 0), (43, 1, 1369, 72, 1 << 40), (72, 1, 1 << 24, 1 << 32, 0)]}
    for kernel, calls in want.items():
        assert rule([f"f32_kernel({t}, {r}, {q}, {n}ll, {kv}ll) == {kernel}" for t, r, q, n, kv in calls]) == [1] * len(calls)
    for kernel, sizes in test_gpu_fp32.SPLIT_KERNELS.items():  # (batch x heads, tokens)
        assert rule([f"f32_kernel(({n} + 31) / 32, 1, {n}, {bh}, 1 << 20) == {kernel}" for bh, n in sizes]) == [1] * len(sizes)


def test_prefix_chains_of_64_channel_heads(rule):
    """(prefix tokens, grid tokens, batch x heads) on either side of every line of the rule, as measured."""
    one = [(5, 576, 12), (1, 784, 16), (5, 784, 64), (5, 1369, 144), (16, 1369, 192), (5, 2304, 160), (5, 4096, 256), (33, 1000, 64),
           (33, 1369, 96), (33, 1369, 144), (64, 2304, 128), (64, 4096, 144), (64, 1500, 4), (5, 100, 4)]
    chains = [(1, 896, 4), (5, 1000, 64), (5, 1369, 12), (5, 1369, 128), (16, 1369, 96), (5, 4096, 192), (1, 16384, 128),
              (33, 1369, 64), (33, 2304, 96), (64, 4096, 128), (64, 1536, 4)]
    got = rule([f"prefix_in_chains({p + n}, {p}, {bh})" for p, n, bh in one + chains])
    assert got == [0] * len(one) + [1] * len(chains)


def test_number_of_prefix_chains(rule):
    """At least as many stages as chains, rows for all their sums, the GPU test's counts (four (batch, head)s) and both sides of every line."""
    sizes = [(p + h * w, p, 4) for p, h, w, _ in test_gpu_prefix.CHAIN_COUNTS]
    sizes += [(1374, 5, 16), (1374, 5, 17), (1088, 1, 4), (1985, 1, 48), (1985, 1, 49), (3969, 1, 32), (3969, 1, 33), (3968, 1, 32), (9208, 1, 512)]
    want = [c for _, _, _, c in test_gpu_prefix.CHAIN_COUNTS] + [16, 8, 8, 16, 8, 32, 16, 16, 8]
    assert rule([f"prefix_chain_count({k}, {q}, {bh})" for k, q, bh in sizes]) == want
    for (keys, queries, _), chains in zip(sizes, want):
        assert (keys + 63) // 64 >= chains and 3 * chains * queries <= keys - queries


def test_prefix_chains_of_128_channel_heads(rule):
    ring = [(5, 500, 4), (5, 576, 128), (5, 784, 160), (16, 784, 128), (5, 1369, 192), (5, 2304, 384), (5, 4096, 384), (16, 1024, 144),
            (32, 2304, 256), (33, 2304, 128), (33, 4096, 128), (64, 4096, 112), (64, 4096, 512), (32, 1519, 4), (64, 1369, 4)]
    chains = [(1, 512, 4), (5, 576, 64), (5, 1000, 144), (16, 1024, 112), (5, 1369, 160), (5, 4096, 256), (32, 2304, 160), (33, 4096, 96),
              (64, 4096, 80), (32, 1536, 4), (64, 3100, 4)]
    got = rule([f"prefix_in_chains_wide({p + n}, {p}, {bh})" for p, n, bh in ring + chains])
    assert got == [0] * len(ring) + [1] * len(chains)


def test_32_bit_offsets_of_wide_heads(rule):
    """Every key of a slice, and the two stages of 32 tokens (32 grid rows where stages are strided) counted past it, within 2^31 bytes; a whole
    sequence as one row (W = tokens) counts tokens, not rows; no overflow at the largest arguments."""
    fits = lambda whole, n, w, sn: (n + 64 * (1 if whole else w)) * sn * 2 + 512 < 1 << 31
    cases = [(1, 5457, 5457, 3072), (1, 349461, 349461, 3072), (1, 349462, 349462, 3072), (0, 5456, 88, 3072), (0, 300000, 700, 3072),
             (0, 300000, 800, 3072), (1, 1 << 24, 1 << 24, 63), (1, 1 << 24, 1 << 24, 64), (0, 1 << 24, 1 << 24, 1 << 24)]
    got = rule([f"wide_offsets_fit({w}, {n}, {W}, {sn})" for w, n, W, sn in cases])
    assert got == [int(fits(*c)) for c in cases] and got[:3] == [1, 1, 0]


def test_linear_attention_in_one_launch(rule):
    """One launch up to the stated token counts, its workgroups (four a part, (batch, head)s in eights) at most one a unit, and the
    GPU test on both sides."""
    limits = {1: 900, 8: 900, 9: 800, 16: 800, 17: 700, 24: 700, 25: 1400, 56: 1400, 57: 2400, 64: 2400}
    assert rule([f"linear_f32_in_one({bh}, {n}) + 2 * linear_f32_in_one({bh}, {n} + 1)" for bh, n in limits.items()]) == [1] * len(limits)
    assert rule([f"linear_f32_in_one({bh}, 1)" for bh in (65, 1 << 16)]) == [0, 0]
    parts = rule([f"linear_f32_parts({bh})" for bh in range(1, 65)])
    assert all(1 <= p <= 8 and 4 * p * ((bh + 7) // 8) <= 32 for bh, p in enumerate(parts, 1))  # units of an XCD
    one = rule([f"linear_f32_in_one({b * h}, {n})" for b, h, n, _ in test_gpu_fp32.ONE_LAUNCH])
    assert one == [0 if (b * h, n) in ((8, 901), (24, 701), (65, 100)) else 1 for b, h, n, _ in test_gpu_fp32.ONE_LAUNCH]


def test_bf16_linear_attention_in_one_launch(rule):
    """As above for bf16: limits, parts, and the GPU test on both sides."""
    limits = {1: 1700, 39: 1700, 40: 2400, 47: 2400, 48: 3100, 79: 3100, 80: 4300, 95: 4300, 96: 4600, 256: 4600, 318: 1000, 368: 1000, 369: 1400, 512: 1400, 552: 1000, 553: 1400, 768: 1400}
    assert rule([f"linear_bf16_in_one({bh}, {n}) + 2 * linear_bf16_in_one({bh}, {n} + 1)" for bh, n in limits.items()]) == [1] * len(limits)
    assert rule([f"linear_bf16_in_one({bh}, {n})" for bh, n in ((257, 577), (317, 577), (318, 299), (318, 577), (520, 577), (769, 577), (65535, 400), (256, 1 << 24))]) == [0, 0, 0, 1, 1, 0, 0, 0]
    parts = rule([f"linear_bf16_parts({bh})" for bh in (*range(1, 257), 257, 65535)])
    assert all(p == (256 // bh if bh <= 256 else 1) for bh, p in zip((*range(1, 257), 257, 65535), parts))
    one = rule([f"linear_bf16_in_one({b * h}, {n})" for b, h, n, _ in test_gpu_bf16_linear.ONE_LAUNCH])
    two = ((39, 1701), (40, 2401), (48, 3101), (80, 4301), (128, 4601), (272, 577), (320, 299), (320, 1001), (384, 1401))
    assert one == [0 if (b * h, n) in two else 1 for b, h, n, _ in test_gpu_bf16_linear.ONE_LAUNCH]
