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

}  // namespace jv
