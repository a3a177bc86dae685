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

// Prefix tokens: `queries` <= 64 queries against the `keys` tokens of a whole sequence, per (batch, head) (jv_attn_bf16.hip).
// Keys come in stages; chains of stages run as workgroups of their own whose sums wait in the rows of O
// behind the queries, kPrefixRows of them for a query of a chain.
constexpr int kStage = 64;
constexpr int kPrefixChains = 8, kPrefixRows = 3;
constexpr bool prefix_rows_fit(int keys, int queries, int chains) { return kPrefixRows * chains * queries <= keys - queries; }

// Heads of 64 channels: chains as workgroups, or (the same bits) as the wavefronts of one workgroup.  The
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

}  // namespace jv
