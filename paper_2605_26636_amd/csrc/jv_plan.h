// Rules that choose kernels by sizes, as plain C++ without HIP: the launchers use them, and a host
// program can ask them what a call takes.
#pragma once

namespace jv {

// Ring of V rows of the linear-attention apply pass with convolution (la_apply_conv_bf16): rows of
// 128 bytes for a step's tokens and the grid rows its taps reach, and behind them a repeat of the first.
// Grids have up to 2^24 columns: bytes are counted in 64 bits.
constexpr int kRingStep = 128, kRingRepeat = 32;
constexpr int kRingFixedLds = (64 * 64 + 64) * 4 + 4 * 32 * 4;  // the state, afterwards four query tiles; 1 / denominators
constexpr int kRingMostLds = 80 * 1024;                         // two workgroups share a compute unit
constexpr long long conv_ring_lds(int ksize, long long W) {
    return kRingFixedLds + (kRingStep + 2 * (ksize / 2) * (W + 1) + kRingRepeat) * 128;
}
// The ring, or V loaded tap by tap (la_apply_bf16; the same bits).  Grids for which two rings do not share a compute
// unit (above 172 columns for 3 x 3, 85 for 5 x 5) load V directly; at the widest below, 64 x 128 in chunks of 256 tokens, the ring fetches
// every row twice and still takes 18 us instead of 19.6.  A workgroup fills its ring before the first step, which a launch of one
// workgroup a unit waits out: up to 256 of them, of more than a step, load V directly too, unless the state pass has
// left V in the caches (the filters come from its token sum) and there are two steps or 25 taps.  Direct / ring, us, the block with
// static filters: 14 x 14 x 12 heads 15.4 / 16.0, 40 x 85 x 12 (168 workgroups) 20.5 / 21.6, 64 x 64 x 16 (256) 20.4 / 21.2, but
// 10 x 10 x 12 (one step) 15.2 / 12.1, 2 of 64 x 64 x 16 (512) 30.1 / 28.4; with generated ones 3 x 3 40 x 85 x 12 27.2 / 28.0,
// 11 x 12 x 12 22.3 / 21.8, 5 x 5 14 x 14 x 12 30.1 / 28.9.
constexpr bool conv_takes_ring(int ksize, bool generated, int W, int N, int n_wg) {
    return conv_ring_lds(ksize, W) <= kRingMostLds && (n_wg > 256 || N <= kRingStep || (generated && (ksize == 5 || N <= 2 * kRingStep)));
}

// Rounds of 256 tokens (64 per wavefront), 1 to kApplyRounds, that a workgroup of the apply pass of linear attention on bf16 tensors
// takes.  Its time is its rounds and about one and a half more for summing the states and splitting them into
// operands; 512 workgroups run at a time.  Against 1 024 tokens halved until there are 512
// workgroups, us: 32 images of 37 x 37 with 16 heads 77.0 -> 74.2 (one chunk instead of 1 024 + 345), with
// 8 heads of 128 and the 3 x 3 convolution 174 -> 145, 11 of 50 x 60 with 12 heads 55.5 -> 53.0.
constexpr int kApplyRounds = 8;
constexpr int apply_rounds(long long bh, int N) {
    const int rounds = (N + 255) / 256;
    long long best = -1;
    int chosen = 1;
    for (int per = kApplyRounds; per > 0; --per) {
        const long long cost = ((bh * ((rounds + per - 1) / per) + 511) / 512) * (2 * per + 3);
        if (best < 0 || cost < best) {
            best = cost;
            chosen = per;
        }
    }
    return chosen;
}

// fp32 linear attention, both passes in one launch (la_fused_f32): its workgroups, four for each of `parts` parts of a (batch, head)'s
// queries, form the state again and again, which pays while they fit the chip's 256 units once and the tokens
// are few.  Two launches / one, us, on three tensors in turn (and on ones read for the first time, of which several workgroups read the same
// bytes): 6 (batch, head)s of 256 tokens 9.9 / 5.5 (11.4 / 6.6), 8 of 900 14.0 / 12.3 (14.1 / 14.0), 6 of 1 024 13.5 / 12.6 (14.0 / 14.3);
// 16 of 576 13.5 / 9.8 (14.2 / 11.6), 12 of 800 13.4 / 12.8 (14.4 / 14.3); 17 of 700 13.7 / 13.2 (15.2 / 15.0), 20 of 800 14.6 / 14.5 (15.6 / 16.2); 25 of 1 400
// 21.7 / 21.4 (23.3 / 23.4), 48 of 1 369 34.4 / 27.7 (37.2 / 31.2), of 2 304 47.6 / 46.3; 64 of 256 12.9 / 8.7 (14.1 / 10.1), of 2 400 56.6 / 50.8 (61.1 / 57.6); 80 of 576 25.2 / 25.6.
// A (batch, head) runs on one XCD: the parts are as many as its 32 units take for the XCD with the most (batch, head)s (12 of 595 tokens, two launches / 5 parts,
// 40 workgroups on some XCDs / 4: 13.2 / 16.9 / 10.2 us; 9 of 400 11.6 / 13.0 / 8.2, 20 of 576 13.6 / 18.6 / 11.5, 18 of 784 14.1 / 23.7 / 14.4).
constexpr int linear_f32_parts(int bh) { return bh > 32 ? 1 : 8 / ((bh + 7) / 8); }
constexpr bool linear_f32_in_one(int bh, int N) {
    return N <= (bh <= 8 ? 900 : bh <= 16 ? 800 : bh <= 24 ? 700 : bh <= 56 ? 1400 : bh <= 64 ? 2400 : 0);
}

// bf16 linear attention of 64-channel heads, both passes in one launch (la_fused_bf16, one workgroup a unit): its workgroups, one for each
// of linear_bf16_parts parts of a (batch, head)'s queries, form the state again, which pays while they fit the chip once and what a unit takes in
// stands behind two or three launches' round trips; the more (batch, head)s, the fewer parts and the longer it does.  Beyond 256 of them, where
// the last round of workgroups is well filled and the others neither all start nor all memory.  Two or three launches / one, us (in brackets tensors
// read for the first time, as above): 6 (batch, head)s of 196 tokens 10.1 / 6.9 (12.2 / 7.7), 12 of 1 374 14.5 / 11.9 (15.5 / 13.8), of 1 700 15.1 / 12.9 (15.7 / 14.9), 24 of
// 1 900 15.2 / 15.8 (17.1 / 17.7); 40 of 2 304 21.1 / 18.2 (22.5 / 20.9), of 2 900 22.6 / 22.4 (23.9 / 25.2); 48 of 3 100 27.8 / 24.6 (29.8 / 28.0), 64 of 784 14.0 / 12.6 (15.4 / 14.7), of 3 100
// 30.1 / 26.8 (32.4 / 30.9), of 3 500 31.0 / 29.9 (33.5 / 34.2), 72 of 4 300 41.3 / 36.6 (43.9 / 45.0); 80 of 4 300 43.8 / 40.1 (45.3 / 45.0), of 4 600 44.2 / 42.1 (47.2 / 49.9);
// 128 of 400 13.6 / 11.2 (15.4 / 12.1), of 4 600 62.5 / 59.8 (66.2 / 63.6), of 5 200 70 / 72 (74 / 75), 256 of 784 30.2 / 22.7 (31.3 / 25.4), of 4 300 109 / 102 (113 / 107), of
// 4 600 113 / 113 (118 / 118), of 4 800 118 / 122 (125 / 126); 300 of 196 16.2 / 19.1, 320 of 784 39.5 / 34.2 (40.6 / 38.4), of 1 400 55.4 / 56.4 (58.9 / 59.8), 384 of
// 1 374 62 / 59 (66 / 63), 512 of 300 25.6 / 24.3 (26.6 / 27.1), 640 of 1 374 96 / 92 (101 / 97), 1 024 of 400 52 / 56.
constexpr int linear_bf16_parts(int bh) { return bh > 256 ? 1 : 256 / bh; }
constexpr bool linear_bf16_in_one(int bh, int N) {
    if (bh > 256) {
        const int rounds = (bh + 255) / 256;
        return bh <= 768 && 100 * bh > 62 * 256 * rounds && N >= 300 && N <= (100 * bh > 72 * 256 * rounds ? 1400 : 1000);
    }
    return N <= (bh < 40 ? 1700 : bh < 48 ? 2400 : bh < 80 ? 3100 : bh < 96 ? 4300 : 4600);
}

// bf16 attention over whole grid rows (attn_ring_bf16): blocks of 32 queries per wavefront, two or (the same bits) one, for
// `queries` query slots in each of `lanes` windows times (batch, head)s.  Two workgroups of 256 queries on a compute unit
// do the most per second, but three of 128 come close, and the smaller blocks leave fewer units with less than
// their share.  Time of a launch's last round by the workgroups a unit has in it, and of a full round, as measured at
// 1 374 keys, us: 256 queries 32.6 (one), 45.4 (two); 128 queries 21.6, 28.4, 38.5 (three).  Two blocks / one, us: 1 374 tokens
// x 16 heads 20.2 / 14.3, x 32 32.6 / 28.4, x 48 45.2 / 36.2, 5 184 x 16 151 / 130, 8 192 x 16 257 / 291, 4 096 x 64 260 / 281, x 128 515 / 550.
constexpr float last_round(long long rest, float one, float two, float three) {
    return rest == 0 ? 0.f : rest <= 256 ? one : rest <= 512 ? two : three;
}
constexpr int ring_query_blocks(int queries, long long lanes) {
    const long long blocks2 = (queries + 255) / 256 * lanes, blocks1 = (queries + 127) / 128 * lanes;
    const float t2 = (float)(blocks2 / 512) * 45.4f + last_round(blocks2 % 512, 32.6f, 45.4f, 0.f);
    const float t1 = (float)(blocks1 / 768) * 38.5f + last_round(blocks1 % 768, 21.6f, 28.4f, 38.5f);
    return 1.08f * t1 < t2 ? 1 : 2;  // (rounds overlap, to the large blocks' advantage)
}

// ... and the key groups of a workgroup: two (attn_ring_bf16<.., 1, 2>, 64 queries a workgroup) while their workgroups, twice as
// many, fit the chip at once, three to a unit.  One group / two, us: 700 tokens x 20 heads 12.7 / 9.7, x 64 (704 workgroups) 17.5 / 16.2, 1 374 x 12 21.5 / 18.9,
// x 32 (704) 28.6 / 26.0, x 40 (880) 29.5 / 34.1, 4 096 x 12 (768) 75 / 67, x 16 (1 024) 82 / 90, 8 192 x 6 (768) 144 / 129.  The order of summation differs,
// so that a long sequence's last bits depend on how many there are; below 21 tiles of keys there is one group, and they do not.
constexpr int ring_key_groups(int queries, int keys, long long lanes) {
    return keys >= 21 * 32 && (long long)((queries + 63) / 64) * lanes <= 768 ? 2 : 1;
}

// fp32 attention of few queries, the keys cut over the four wavefronts of a workgroup (`waves` blocks of 32 queries in all, windows of
// `tiles` tiles of 32 keys): attn_few_f32, or attn_short_f32<4> where that is faster or K and V span more bytes than 32-bit offsets
// count.  With a tile per wavefront attn_few_f32 has nothing to fetch ahead and its splits stand alone, and only its third
// workgroup on a unit tells: rounds of 768 against 512.  Windows of whole grid rows of 4 tiles, staged / few, us: 100 keys x 64 (batch, head)s 7.3 / 7.8,
// 128 x 64 7.3 / 7.8; 7 tiles x 37 16.3 / 13.4.
constexpr bool f32_keys_staged(int tiles, bool whole_rows, long long waves, long long kv_bytes) {
    return kv_bytes >= (1ll << 32) || (tiles == 4 && whole_rows && (waves - 1) % 768 < 512);
}
// fp32 attention: `queries` query slots in each of `lanes` windows times (batch, head)s, windows of `tiles` tiles of 32 keys, K and V slices of up to kv_bytes.
// attn_f32 does the most per second, but its workgroups take 128 queries, and a unit with one of them waits out its barriers; attn_few_f32's take 32, with
// four wavefronts each.  Every unit takes workgroups in rounds: of attn_few_f32 each as long as the one before, of attn_f32 three of them at
// once, the first as long as `round` of attn_few_f32's, two `extra` and three twice `round`.  Few / many, us: 1 369 tokens (43 tiles) of
// 516 blocks of 32 queries (3 rounds / 1) 62 / 91, 903 (4 / 1) 84 / 92, 1 419 (6 / 2) 123 / 128, 1 591 (7 / 2) 140 / 128; 25 tiles 900 (4 / 1) 54 / 56, 1 275 (5 / 2)
// 66 / 77, 1 600 (7 / 2) 87 / 78, 1 900 (8 / 3) 100 / 105; 13 tiles 767 (3 / 1) 26 / 32, 1 274 (5 / 2) 41 / 44, 1 404 (6 / 2) 47 / 44; 8 tiles 768 (3 / 1) 19 / 22, 896 (4 / 1) 24 / 22,
// 1 280 (5 / 2) 29 / 30; 7 tiles 637 (3 / 1) 19.0 / 19.7, 903 (4 / 2) 23 / 26, 1 281 (6 / 2) 31 / 28; 5 tiles 400 (2 / 1) 13.1 / 15.3, 640 (3 / 1) 16.4 / 15.8; 4 tiles 516 (3 / 1) 13.8 / 13.0;
// windows of 22 x 22 (16 tiles) 768 (3 / 1) 32 / 40, 1 024 (4 / 1) 43 / 41.
constexpr bool f32_few(int tiles, int queries, long long lanes) {
    const long long few = ((queries + 31) / 32 * lanes + 255) / 256, many = ((queries + 127) / 128 * lanes + 255) / 256;
    const int round = tiles <= 5 ? 2 : tiles <= 16 ? 3 : 4, extra = round + (tiles < 8 ? 1 : 2);
    return few <= many / 3 * 2 * round + (many % 3 == 0 ? 0 : many % 3 == 1 ? round : extra);
}
// Windows of one or two tiles leave nothing to share keys for: attn_short_f32 where its start is the shorter one.  Short / many, us: 1 tile
// always (windows of 5 x 5, 3 072 blocks 53 / 59); 2 tiles of 256 blocks 7.1 / 8.0, of 640 11.2 / 11.9; from there to 1 024 it would be 3 to 6 % shorter still, but
// is further from 64 bits (2.0e-7 / 1.4e-7).  The same of 257 to 512 blocks of four tiles, two key groups of attn_short_f32 against attn_few_f32: 4 to 10 %, and
// 2.7e-7 / 1.9e-7.
enum F32Kernel { kF32Many, kF32Few, kF32Short1, kF32Short2, kF32Short4 };
constexpr F32Kernel f32_kernel(int tiles, bool whole_rows, int queries, long long lanes, long long kv_bytes) {
    const long long blocks = (queries + 31) / 32 * lanes;  // of 32 queries
    if (tiles == 1) return kF32Short1;
    if (tiles == 2) return blocks <= 640 ? kF32Short2 : kF32Many;
    if (!f32_few(tiles, queries, lanes)) return kF32Many;
    return f32_keys_staged(tiles, whole_rows, blocks, kv_bytes) ? kF32Short4 : kF32Few;
}

constexpr int kStage = 64, kStageWide = 32;  // keys of a stage, heads of 64 and of 128 channels

// Wide heads: do 32-bit byte offsets inside a slice of `tokens` tokens, `sn` elements apart, reach every key of the ring kernel
// (attn_ring_wide_bf16) and of the prefix chains?  Counted two stages past the end: 32 tokens each where windows span whole grid rows, the
// whole sequence as one row among them; up to 32 rows of the grid of `W` columns where a stage takes a few columns of each.  Views of a
// fused projection with prefix tokens (the sequence as one row), general kernel / here, us: window attention of 3 x 5 457 tokens
// x 8 heads 217 / 68, 16 389 x 8 530 / 73; full attention of 5 476 x 8 231 / 135, 2 x 9 549 x 8 1 052 / 722.
constexpr bool wide_offsets_fit(bool whole_rows, long long tokens, long long W, long long sn) {
    return (tokens + 2ll * kStageWide * (whole_rows ? 1 : W)) * sn * 2 + 512 < (1ll << 31);
}

// Prefix tokens: `queries` <= 64 queries against the `keys` tokens of a whole sequence, per (batch, head) (jv_attn_bf16.hip).
// Keys come in stages; chains of stages run as workgroups of their own whose sums wait in the rows of O
// behind the queries, kPrefixRows of them for a query of a chain.
constexpr int kPrefixChains = 8, kPrefixChainsWide = 16, kPrefixRows = 3;
constexpr bool prefix_rows_fit(int keys, int queries, int chains) { return kPrefixRows * chains * queries <= keys - queries; }

// Heads of 64 channels: chains as workgroups, or (the bits of eight) as the wavefronts of one workgroup.  The
// chains' loads and sums of a stage overlap, for a second launch and the way of the sums through memory: they pay from two
// stages a chain on, as long as the launch's eight times as many workgroups fit the chip at once, and with two
// blocks of queries, which write twice the sums, for fewer (batch, head)s.  One workgroup / chains, window attention included, us,
// 5 tokens in front of 576 tokens x 12 13.6 / 14.9, 1 000 x 64 22.5 / 20.4, 1 369 x 128 39.7 / 39.0, x 192 49.2 / 51.5,
// 4 096 x 192 119.2 / 116.6, x 256 146.2 / 147.8; 33 in front of 1 369 x 96 38.3 / 37.9, x 144 43.0 / 50.5;
// 64 in front of 2 304 x 96 51.8 / 51.5, x 128 57.4 / 62.0, 4 096 x 128 90.6 / 88.7, x 144 95.7 / 106.4.
constexpr bool prefix_in_chains(int keys, int queries, int bh) {
    const int stages = (keys + kStage - 1) / kStage;
    const int most = queries > 32 ? (stages < 43 ? 3 * stages : 128) : stages < 64 ? 128 : 192;
    return stages >= 2 * kPrefixChains - 1 && bh <= most && prefix_rows_fit(keys, queries, kPrefixChains);
}
// How many chains: 8; 16 or 32 where that many workgroups a (batch, head) still leave few to a unit, from about two stages a chain on, since
// a chain is bound by the round trips of its stages, one after the other, and 4 096 tokens are eight of them for each of 8 chains.  8 chains / as
// chosen, window attention included, us: 1 token in front of 1 156 tokens x 12 16.4 / 15.6, 5 in front of 1 369 x 12 17.0 / 16.2 (x 32 with 16 chains 18.0),
// 2 025 x 16 19.3 / 17.3, x 32 23.4 / 22.4 (x 64 30.3 / 32.0), 4 096 x 48 39.8 / 38.4 (x 64 46.4 / 48.6); with 32 4 096 x 16 26.3 / 21.5, x 32 32.4 / 31.2
// (1 in front of 4 096 x 64 45.8 / 49.8), 1 in front of 9 207 x 12 42.4 / 27.9, 5 of 16 384 x 16 75.8 / 48.0, 64 of 16 384 x 16 99.8 / 56.5.
constexpr int prefix_chain_count(int keys, int queries, int bh) {
    const int stages = (keys + kStage - 1) / kStage;
    if (stages >= 63 && bh <= 32 && prefix_rows_fit(keys, queries, 32)) return 32;
    return stages >= 18 && bh <= (stages < 31 ? 16 : 48) && prefix_rows_fit(keys, queries, 16) ? 16 : kPrefixChains;
}
// Heads of 128 channels: chains, or one workgroup of the ring kernel that walks all keys.  A (batch, head) has a
// wavefront per chain and block of 32 queries, which fetches the keys once more and writes the sums of its queries: the more
// of both there are for a stage, the sooner the chip is full without chains.  The line is fitted to 313 launches of 512 to 4 096
// tokens (0.1 % off the better of the two on average, 4 % at worst).  Ring kernel / chains, window attention included, us,
// 5 tokens in front of 576 tokens x 64 29.8 / 25.8, x 128 37.0 / 38.8, 1 369 x 160 85.7 / 82.1, x 256 124.5 / 127.7,
// 4 096 x 256 356 / 348, x 384 505 / 514; 32 in front of 2 304 x 160 138.5 / 137.7, x 256 201 / 224;
// 64 in front of 4 096 x 64 140 / 117, x 80 165 / 145, x 128 219 / 251, x 512 672 / 1 069.
constexpr bool prefix_in_chains_wide(int keys, int queries, int bh) {
    const int stages = (keys + kStageWide - 1) / kStageWide, line = stages < 87 ? 3 * stages + 60 : 320;
    const long long blocks = (long long)bh * ((queries + 31) / 32);
    return stages > kPrefixChainsWide && blocks * (96 + queries) <= 96 * line && prefix_rows_fit(keys, queries, kPrefixChainsWide);
}

}  // namespace jv
