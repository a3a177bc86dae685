// bf16 matrix product with fused epilogue on tiles smaller than 256 x 256, for the token counts
// at which 256 x 256 tiles leave compute units without work.
#include <type_traits>

#include "jv_gemm.h"

namespace jv {

// ---------------------------------------------------------------------------------------
// y = epilogue(a w^T + bias):  a [M, K], w [N, K], bf16 with K contiguous.  A workgroup of
// WM x WN wavefronts owns a tile of 32 MT WM tokens x 64 WN features, a wavefront 32 MT tokens x
// 64 features of it (MT x 2 blocks of 32 x 32).  K is walked in blocks of 64; the rows of a and w
// go straight into LDS through a ring of STAGES blocks (row layout and rotation of the 256 x 256
// kernel).  A block is four steps of 16 in K, and a step's operands are read two steps ahead.  So the barrier
// of a block sits before its last two steps, when every operand of the block has been read: behind it
// the first operands of the next block are read and the block STAGES ahead is fetched into the
// slot just left, under the matrix instructions of those two steps, so that neither starts with an
// LDS round trip and STAGES - 1 blocks are in flight.
// The launch deals contiguous ranges of tiles to the XCDs.  Which of the two tile indices runs
// fastest decides what an XCD's L2 holds: with `tokens_fast` a range is a band of features over
// all tokens (each row of w is fetched by one XCD, a by all eight), else a band of tokens.
// PARTS: K is summed in `parts` parts that are then added in order, which is what a K split of
// that many gives, without the parts' way through memory (and the idle units of an unsplit launch).
// grid (8 * ceil(tiles * k_split / 8)), 64 WM WN threads.
// ---------------------------------------------------------------------------------------
constexpr int kBlockK = 64;

template <int WM, int WN, int MT, int STAGES, int EPI>
struct TileShape {
    static constexpr int kWaves = WM * WN, kThreads = 64 * kWaves;
    static constexpr int kBM = 32 * MT * WM, kBN = 64 * WN;
    static constexpr int kRow = 2 * kBlockK, kRowsPerLoad = 1024 / kRow;  // bytes of a row in LDS; rows of a 1 KB load instruction
    static constexpr int kPartA = kBM * kRow, kPartW = kBN * kRow, kStage = kPartA + kPartW;
    static constexpr int kLoadsA = kBM / kRowsPerLoad / kWaves, kLoadsW = kBN / kRowsPerLoad / kWaves;  // per wavefront
    static constexpr int kTable = EPI == JV_EPI_GELU ? kPhiSteps * 8 : 0;
    static constexpr int kRing = STAGES * kStage > kWaves * 8192 ? STAGES * kStage : kWaves * 8192;
    static constexpr int kLds = kRing + kTable;
    static_assert(kBM % (kRowsPerLoad * kWaves) == 0 && kBN % (kRowsPerLoad * kWaves) == 0, "whole load instructions per wavefront");
    // Rotation of a row's 16-byte chunks: 16 consecutive rows spread over all 64 banks.
    static __device__ int rotation(int row) { return (row >> 1) & 7; }
    static __device__ unsigned offset(int row, int chunk) { return (unsigned)(row * kRow + ((chunk ^ rotation(row)) << 4)); }
};

template <int N>
__device__ inline void wait_vm_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The activation of an epilogue on four outputs (GELU: phi_table as the kernels build it).
template <int EPI>
__device__ inline void tile_activation(f32x4 &val, const float *phi_table) {
    if (EPI == JV_EPI_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e] = gelu_from_table(val[e], phi_table);
    }
    if (EPI == JV_EPI_SILU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e] = val[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-val[e]));
    }
}

template <int WM, int WN, int MT, int STAGES, int EPI, bool OUT_BF16, bool PARTS>
__global__ void __launch_bounds__(64 * WM * WN)
gemm_tile_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ W, const float *__restrict__ bias,
                 const void *residual, void *Y, int M, int N, int K, int lda, int tiles_m, int tiles_n,
                 int tokens_fast, int k_split, long long y_split, int parts) {
#ifdef __HIP_DEVICE_COMPILE__  // (the host pass does not know the buffer-resource builtins)
    using S = TileShape<WM, WN, MT, STAGES, EPI>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int wm = wave / WN, wn = wave % WN;
    const int n_tiles = tiles_m * tiles_n, n_work = n_tiles * k_split;
    const int per_xcd = (n_work + 7) / 8;
    int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || item >= n_work) return;  // whole workgroup
    // the tiles of one part of K follow one another: neighbouring tiles share rows of a or w, the parts of a tile nothing
    const int k_part = item / n_tiles;
    item -= k_part * n_tiles;
    const int tm = tokens_fast ? item % tiles_m : item / tiles_n;
    const int tn = tokens_fast ? item / tiles_m : item % tiles_n;
    const int m0 = tm * S::kBM, n0 = tn * S::kBN;
    const int all_b = K / kBlockK, b0 = all_b * k_part / k_split, n_b = all_b * (k_part + 1) / k_split - b0;

    // Global -> LDS: lane = 8 * (row in group of 8) + LDS chunk slot, and it fetches the global
    // chunk that belongs in that slot under the row rotation.  Buffer loads: the tile's first row
    // is the base, the offset inside the tile a vector register that never changes, the position
    // in K the scalar offset, so that a load costs no vector arithmetic.  Rows past the end of
    // the matrix re-read its last row (the launcher bounds lda and K: offsets fit 32 bits).
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(A + (size_t)m0 * lda), 0, 0x7fffffff, 0x00027000);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(W + (size_t)n0 * K), 0, 0x7fffffff, 0x00027000);
    unsigned a_off[S::kLoadsA], w_off[S::kLoadsW];
    const int lrow = lane / (S::kRow / 16), lchunk = lane % (S::kRow / 16);
#pragma unroll
    for (int j = 0; j < S::kLoadsA; ++j) {
        const int r = (wave * S::kLoadsA + j) * S::kRowsPerLoad + lrow;
        a_off[j] = 2u * ((unsigned)min(r, M - 1 - m0) * (unsigned)lda + 8 * (lchunk ^ S::rotation(r)));
    }
#pragma unroll
    for (int j = 0; j < S::kLoadsW; ++j) {
        const int r = (wave * S::kLoadsW + j) * S::kRowsPerLoad + lrow;
        w_off[j] = 2u * ((unsigned)min(r, N - 1 - n0) * (unsigned)K + 8 * (lchunk ^ S::rotation(r)));
    }
    constexpr int kLoads = S::kLoadsA + S::kLoadsW;
    // load j of block `blk` (counted from b0) into `slot`
    auto issue = [&](int blk, int slot, int j) __attribute__((always_inline)) {
        const unsigned kbytes = (unsigned)(b0 + blk) * (unsigned)S::kRow;
        unsigned char *base = smem + slot * S::kStage;
        if (j < S::kLoadsA) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)(base + (wave * S::kLoadsA + j) * 1024), 16, a_off[j < S::kLoadsA ? j : 0], kbytes, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(base + S::kPartA + (wave * S::kLoadsW + j - S::kLoadsA) * 1024), 16, w_off[j < S::kLoadsA ? 0 : j - S::kLoadsA], kbytes, 0, 0);
    };
    // Everything but the youngest `blocks` blocks this wavefront has issued has landed; barrier.
    auto landed = [&](int blocks) __attribute__((always_inline)) {
        if (STAGES > 4 && blocks >= 4) wait_vm_and_barrier<4 * kLoads>();
        else if (STAGES > 3 && blocks >= 3) wait_vm_and_barrier<3 * kLoads>();
        else if (STAGES > 2 && blocks >= 2) wait_vm_and_barrier<2 * kLoads>();
        else if (STAGES > 1 && blocks >= 1) wait_vm_and_barrier<kLoads>();
        else wait_vm_and_barrier<0>();
    };

    f32x16 acc[2][MT];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nt][mt][v] = 0.f;
    f32x16 total[2][PARTS ? MT : 1];  // the sums of the parts of K before this one
    int part = 1, part_end = PARTS ? n_b / parts : 0;
    if (PARTS)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) total[nt][PARTS ? mt : 0] = acc[nt][mt];
    // Operands of a step (16 in K), each read two steps before it is used.  The reads are in
    // assembly with counted waits: left to itself the compiler waits for all of them.
    constexpr int kSteps = kBlockK / 16, kSets = kSteps, kReads = MT + 2;
    static_assert(MT <= 2, "operand reads are written out for one or two token blocks");
    u32x4 aop[kSets][MT], wop[kSets][2];
    unsigned a_addr[kSteps], w_addr[kSteps];  // LDS byte address of this lane's row in slot 0, per step
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        a_addr[s] = lds_address(smem) + S::offset(wm * 32 * MT + li, 2 * s + g);
        w_addr[s] = lds_address(smem) + S::kPartA + S::offset(wn * 64 + li, 2 * s + g);
    }
    auto read_op = [&](int set, int i, unsigned aa, unsigned wa) __attribute__((always_inline)) {
        if (i == 0) wop[set][0] = lds_read_b128_at<0>(wa);
        if (i == 1) aop[set][0] = lds_read_b128_at<0>(aa);
        if (i == 2) wop[set][1] = lds_read_b128_at<32 * S::kRow>(wa);
        if (i == 3) aop[set][MT - 1] = lds_read_b128_at<32 * S::kRow>(aa);
    };
    // Wait until at most `pending` steps' reads are outstanding, the operands of `set` tied to it.
    auto wait_ops = [&](int set, auto pending_tag) __attribute__((always_inline)) {
        constexpr int pending = decltype(pending_tag)::value * kReads;
        u32x4(&w)[2] = wop[set], (&a)[MT] = aop[set];
        if (MT > 1) asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(w[0]), "+v"(w[1]), "+v"(a[0]), "+v"(a[MT - 1]) : "n"(pending));
        else asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(w[0]), "+v"(w[1]), "+v"(a[0]) : "n"(pending));
    };
    using N0 = std::integral_constant<int, 0>; using N1 = std::integral_constant<int, 1>;

#pragma unroll
    for (int s = 0; s < STAGES; ++s)
        if (s < n_b)
#pragma unroll
            for (int j = 0; j < kLoads; ++j) issue(s, s, j);
    // GELU's table behind the ring, built while the first blocks are in flight
    float *phi_table = (float *)(smem + S::kRing);
    if (EPI == JV_EPI_GELU)
        phi_table_fill(phi_table, tid, S::kThreads);
    landed(min(STAGES, n_b) - 1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < kReads; ++i) read_op(s, i, a_addr[s], w_addr[s]);
    // One block in `slot`.  Its steps issue, among their matrix instructions, the operand reads
    // of the step two ahead and the refill loads.  `next`: there is a block p + 1; from step
    // kBarStep on the reads are of that block, so the wait for it and the barrier sit in front
    // of that step; behind it this block's slot is free and takes block p + STAGES (`refill`).
    // With more than two stages the loads are spread over kSteps steps, the last of them in the
    // block after (`tail`: block p - 1 + STAGES is being loaded).
    constexpr int kBarStep = kSteps - 2;
    constexpr int kSpread = STAGES > 2 ? kSteps : 2, kPerStep = (kLoads + kSpread - 1) / kSpread;
    int slot = 0;
    auto block = [&](int p, auto tail_tag, auto refill_tag, auto next_tag) __attribute__((always_inline)) {
        constexpr bool tail = decltype(tail_tag)::value, refill = decltype(refill_tag)::value, next = decltype(next_tag)::value;
        if (PARTS && p == part_end) {
            ++part;
            part_end = n_b * part / parts;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    total[nt][PARTS ? mt : 0] += acc[nt][mt];
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[nt][mt][v] = 0.f;
                }
        }
        const int nslot = slot + 1 == STAGES ? 0 : slot + 1, pslot = slot == 0 ? STAGES - 1 : slot - 1;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int set = s, rset = (s + 2) % kSets;
            if (s == kBarStep && next) {
                if (refill) wait_vm_and_barrier<(STAGES - 2) * kLoads>();
                else landed(min(STAGES - 2, n_b - 2 - p));
            }
            const bool ahead = s >= kBarStep;  // reads of the next block
            const bool reads = !ahead || next;
            const unsigned soff = (unsigned)((ahead ? nslot : slot) * S::kStage);
            const unsigned aa = a_addr[(s + 2) % kSteps] + soff, wa = w_addr[(s + 2) % kSteps] + soff;
            if (next || s + 1 < kSteps) wait_ops(set, N1());
            else wait_ops(set, N0());
            const int load0 = s >= kBarStep ? (s - kBarStep) * kPerStep : (s + 2) * kPerStep;
            const bool loads = s >= kBarStep ? refill : (tail && kSpread == kSteps);
#pragma unroll
            for (int m = 0; m < 2 * MT; ++m) {
                acc[m & 1][m >> 1] = mfma32(as_bf16x8(wop[set][m & 1]), as_bf16x8(aop[set][m >> 1]), acc[m & 1][m >> 1]);
#pragma unroll
                for (int r = 0; r < kReads; ++r)  // reads spread over the first instructions
                    if (reads && r * 2 * MT / kReads == m) read_op(rset, r, aa, wa);
#pragma unroll
                for (int l = 0; l < kPerStep; ++l)
                    if (loads && l * 2 * MT / kPerStep == m && load0 + l < kLoads)
                        issue(s >= kBarStep ? p + STAGES : p - 1 + STAGES, s >= kBarStep ? slot : pslot, load0 + l);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        slot = nslot;
    };
    using T = std::true_type; using F = std::false_type;
    int p = 0;
    if (n_b > STAGES) {
        block(0, F(), T(), T());
        for (p = 1; p + STAGES < n_b; ++p) block(p, T(), T(), T());
        block(p++, T(), F(), T());
    }
    for (; p + 1 < n_b; ++p) block(p, F(), F(), T());
    block(p, F(), F(), F());

    if (PARTS)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = total[nt][PARTS ? mt : 0] + acc[nt][mt];
    // Epilogue: accumulator register v of block (nt, mt) is feature n0 + 64 wn + 32 nt + 8 (v/4) +
    // 4 g + v%4 of token m0 + 32 (MT wm + mt) + li.  Each wavefront turns its 32 x 64 blocks into
    // token rows in 8 KB of LDS of its own and stores whole rows; the residual is read in the
    // same row layout.
    f32x4 bias_reg[2][4];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int col = n0 + wn * 64 + nt * 32 + 8 * q4 + 4 * g;
            f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            bias_reg[nt][q4] = (bias && col < N) ? *(const f32x4 *)(bias + col) : zero;
        }
    constexpr bool kResidual = EPI == JV_EPI_RESIDUAL;
    constexpr bool kStageF32 = !OUT_BF16 || kResidual;
    const int frow = lane >> 4, fchunk = lane & 15, fcol = n0 + wn * 64 + 4 * fchunk;
    const int row_base = m0 + wm * 32 * MT;
    f32x4 res_reg[MT][8];
    u32x2 res16_reg[MT][8];
    if (kResidual) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int row = row_base + mt * 32 + 4 * r + frow;
                const bool inside = row < M && fcol < N;
                u32x2 zero2 = {0u, 0u};
                f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
                if (OUT_BF16) res16_reg[mt][r] = inside ? *(const u32x2 *)((const __bf16 *)residual + (size_t)row * N + fcol) : zero2;
                else res_reg[mt][r] = inside ? *(const f32x4 *)((const float *)residual + (size_t)row * N + fcol) : zero4;
            }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // nobody reads the ring any more
    unsigned char *stage = smem + wave * 8192;
    char *y_part = (char *)Y + (size_t)k_part * (size_t)y_split * (OUT_BF16 ? 2 : 4);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 val = {acc[nt][mt][4 * q4], acc[nt][mt][4 * q4 + 1], acc[nt][mt][4 * q4 + 2], acc[nt][mt][4 * q4 + 3]};
                val += bias_reg[nt][q4];
                tile_activation<EPI>(val, phi_table);
                if (kStageF32) {
                    *(f32x4 *)(stage + li * 256 + (((8 * nt + 2 * q4 + g) ^ (li & 15)) << 4)) = val;
                } else {
                    u32x2 pk = {pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
                    *(u32x2 *)(stage + tile_off_row(li, 4 * nt + q4) + 8 * g) = pk;
                }
            }
        if (!kStageF32) {  // 8 lanes per token row (128 bytes), 8 rows per instruction
            const int col = n0 + wn * 64 + 8 * (lane & 7);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int orow = 8 * r + (lane >> 3), row = row_base + mt * 32 + orow;
                const u32x4 out = *(const u32x4 *)(stage + tile_off_row(orow, lane & 7));
                if (row < M && col < N) *(u32x4 *)((__bf16 *)y_part + (size_t)row * N + col) = out;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int orow = 4 * r + frow, row = row_base + mt * 32 + orow;
                f32x4 out = *(const f32x4 *)(stage + orow * 256 + ((fchunk ^ (orow & 15)) << 4));
                if (OUT_BF16) {
                    if (kResidual) {
                        const u32x2 rr = res16_reg[mt][r];
                        out[0] += bf16_lo(rr[0]); out[1] += bf16_hi(rr[0]);
                        out[2] += bf16_lo(rr[1]); out[3] += bf16_hi(rr[1]);
                    }
                    u32x2 pk = {pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
                    if (row < M && fcol < N) *(u32x2 *)((__bf16 *)y_part + (size_t)row * N + fcol) = pk;
                } else {
                    if (kResidual) out += res_reg[mt][r];
                    if (row < M && fcol < N) *(f32x4 *)((float *)y_part + (size_t)row * N + fcol) = out;
                }
            }
        }
    }
#endif
}

// ---------------------------------------------------------------------------------------
// Tiles of 256 tokens x 192 features: three quarters of a 256 x 256 tile, for launches of which a
// round of the larger tiles would be half empty.  8 wavefronts of 64 tokens x 96 features (2 x 3 blocks:
// five operand reads per six matrix instructions).  A block of 64 in K is 32 KB of a and 24 KB of w, of which
// LDS holds three and two: the a part of block p + 2 goes out during the first half of block p, into the slot
// block p - 1 has left, the w part behind the barrier, into block p's own.  The rest, the order of
// summation included, as gemm_tile_kernel.
// grid (8 * ceil(tiles / 8)), 512 threads, kTile192Lds bytes of dynamic LDS.
// ---------------------------------------------------------------------------------------
constexpr int kT192N = 192, kT192PartA = 256 * 128, kT192PartW = kT192N * 128, kT192Ring = 3 * kT192PartA + 2 * kT192PartW;
constexpr int kTile192Lds = kT192Ring + kPhiSteps * 8;

template <int EPI, bool OUT_BF16>
__global__ void __launch_bounds__(512)
gemm_tile192_kernel(const __bf16 *__restrict__ A, const __bf16 *__restrict__ W, const float *__restrict__ bias,
                    const void *residual, void *Y, int M, int N, int K, int lda, int tiles_m, int tiles_n, int tokens_fast) {
#ifdef __HIP_DEVICE_COMPILE__  // (the host pass does not know the buffer-resource builtins)
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *wring = smem + 3 * kT192PartA;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int wm = wave >> 1, wn = wave & 1;
    const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) / 8;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || item >= n_tiles) return;  // whole workgroup
    const int tm = tokens_fast ? item % tiles_m : item / tiles_n, tn = tokens_fast ? item / tiles_m : item % tiles_n;
    const int m0 = tm * 256, n0 = tn * kT192N, n_b = K / kBlockK;

    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(A + (size_t)m0 * lda), 0, 0x7fffffff, 0x00027000);
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(W + (size_t)n0 * K), 0, 0x7fffffff, 0x00027000);
    constexpr int kLoadsA = 4, kLoadsW = 3;  // per wavefront and block, 8 rows each
    unsigned a_off[kLoadsA], w_off[kLoadsW];
    const int lrow = lane >> 3, lchunk = lane & 7;
    auto rotation = [](int row) { return (row >> 1) & 7; };
#pragma unroll
    for (int j = 0; j < kLoadsA; ++j) {
        const int r = (wave * kLoadsA + j) * 8 + lrow;
        a_off[j] = 2u * ((unsigned)min(r, M - 1 - m0) * (unsigned)lda + 8 * (lchunk ^ rotation(r)));
    }
#pragma unroll
    for (int j = 0; j < kLoadsW; ++j) {
        const int r = (wave * kLoadsW + j) * 8 + lrow;
        w_off[j] = 2u * ((unsigned)min(r, N - 1 - n0) * (unsigned)K + 8 * (lchunk ^ rotation(r)));
    }
    auto issue_a = [&](int blk, int slot, int j) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_void *)(smem + slot * kT192PartA + (wave * kLoadsA + j) * 1024), 16, a_off[j], (unsigned)blk * 128u, 0, 0);
    };
    auto issue_w = [&](int blk, int slot, int j) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, (lds_void *)(wring + slot * kT192PartW + (wave * kLoadsW + j) * 1024), 16, w_off[j], (unsigned)blk * 128u, 0, 0);
    };

    f32x16 acc[3][2];  // [feature block][token block]
#pragma unroll
    for (int nt = 0; nt < 3; ++nt)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nt][mt][v] = 0.f;
    // Operands of a step, each read two steps before it is used (assembly and counted waits, as in gemm_tile_kernel).
    u32x4 aop[4][2], wop[4][3];
    unsigned a_addr[4], w_addr[4];  // LDS byte address of this lane's row in slot 0, per step
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int ar = wm * 64 + li, wr = wn * 96 + li;
        a_addr[s] = lds_address(smem) + (unsigned)(ar * 128 + (((2 * s + g) ^ rotation(ar)) << 4));
        w_addr[s] = lds_address(wring) + (unsigned)(wr * 128 + (((2 * s + g) ^ rotation(wr)) << 4));
    }
    auto read_op = [&](int set, int i, unsigned aa, unsigned wa) __attribute__((always_inline)) {
        if (i == 0) wop[set][0] = lds_read_b128_at<0>(wa);
        if (i == 1) aop[set][0] = lds_read_b128_at<0>(aa);
        if (i == 2) wop[set][1] = lds_read_b128_at<32 * 128>(wa);
        if (i == 3) wop[set][2] = lds_read_b128_at<64 * 128>(wa);
        if (i == 4) aop[set][1] = lds_read_b128_at<32 * 128>(aa);
    };
    auto wait_ops = [&](int set, auto pending_tag) __attribute__((always_inline)) {
        constexpr int pending = decltype(pending_tag)::value * 5;
        u32x4(&w)[3] = wop[set], (&a)[2] = aop[set];
        asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(a[0]), "+v"(a[1]) : "n"(pending));
    };
    using N0 = std::integral_constant<int, 0>; using N1 = std::integral_constant<int, 1>;
    using T = std::true_type; using F = std::false_type;

#pragma unroll
    for (int b = 0; b < 2; ++b)
        if (b < n_b) {
#pragma unroll
            for (int j = 0; j < kLoadsA; ++j) issue_a(b, b, j);
#pragma unroll
            for (int j = 0; j < kLoadsW; ++j) issue_w(b, b, j);
        }
    // GELU's table behind the ring, built while the first blocks are in flight
    float *phi_table = (float *)(smem + kT192Ring);
    if (EPI == JV_EPI_GELU)
        phi_table_fill(phi_table, tid, 512);
    if (n_b > 1) wait_vm_and_barrier<kLoadsA + kLoadsW>();
    else wait_vm_and_barrier<0>();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 5; ++i) read_op(s, i, a_addr[s], w_addr[s]);
    // One block.  `refill`: there is a block p + 2; `next`: there is a block p + 1, whose operands are read from
    // step 2 on: it has landed at the barrier in front of that step, where only the a part of p + 2 may be in flight.
    int a_slot = 0, w_slot = 0;
    auto block = [&](int p, auto refill_tag, auto next_tag) __attribute__((always_inline)) {
        constexpr bool refill = decltype(refill_tag)::value, next = decltype(next_tag)::value;
        const int a_next = a_slot == 2 ? 0 : a_slot + 1, a_free = a_slot == 0 ? 2 : a_slot - 1, w_next = w_slot ^ 1;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int rset = (s + 2) % 4;
            if (s == 2 && next) {
                if (refill) wait_vm_and_barrier<kLoadsA>();
                else wait_vm_and_barrier<0>();
            }
            const bool ahead = s >= 2, reads = !ahead || next;
            const unsigned aa = a_addr[(s + 2) % 4] + (unsigned)((ahead ? a_next : a_slot) * kT192PartA);
            const unsigned wa = w_addr[(s + 2) % 4] + (unsigned)((ahead ? w_next : w_slot) * kT192PartW);
            if (next || s + 1 < 4) wait_ops(s, N1());
            else wait_ops(s, N0());
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                acc[m % 3][m / 3] = mfma32(as_bf16x8(wop[s][m % 3]), as_bf16x8(aop[s][m / 3]), acc[m % 3][m / 3]);
                if (reads && m < 5) read_op(rset, m, aa, wa);
                if (refill && s < 2 && (m == 1 || m == 4)) issue_a(p + 2, a_free, 2 * s + (m == 4));
                if (refill && s == 2 && (m == 1 || m == 4)) issue_w(p + 2, w_slot, m == 4);
                if (refill && s == 3 && m == 1) issue_w(p + 2, w_slot, 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        a_slot = a_next;
        w_slot = w_next;
    };
    int p = 0;
    for (; p + 2 < n_b; ++p) block(p, T(), T());
    for (; p + 1 < n_b; ++p) block(p, F(), T());
    block(p, F(), F());

    // Epilogue: register v of block (nt, mt) is feature n0 + 96 wn + 32 nt + 8 (v / 4) + 4 g + v % 4 of token
    // m0 + 64 wm + 32 mt + li.  Two wavefronts that share their tokens turn 32 x 192 blocks into token rows in
    // LDS and store sixteen rows each, 384 (fp32: 768) bytes at a time, whole lines; the residual is read in
    // the same layout.
    constexpr bool kResidual = EPI == JV_EPI_RESIDUAL, kStageF32 = !OUT_BF16 || kResidual;
    constexpr int kPitch = kStageF32 ? 784 : 400, kPieces = kStageF32 ? 48 : 24, kPasses = kPieces / 4;  // 16-byte pieces of a row
    f32x4 bias_reg[3][4];
#pragma unroll
    for (int nt = 0; nt < 3; ++nt)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int col = n0 + wn * 96 + nt * 32 + 8 * q4 + 4 * g;
            bias_reg[nt][q4] = (bias && col < N) ? *(const f32x4 *)(bias + col) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    unsigned char *stage = smem + wm * 32 * kPitch;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int row0 = m0 + wm * 64 + mt * 32 + 16 * wn;  // first of the rows this wavefront stores
        f32x4 res[kPasses];
        u32x2 res16[kPasses];
        if (kResidual)
#pragma unroll
            for (int r = 0; r < kPasses; ++r) {
                const int piece = lane + 64 * r, row = row0 + piece / kPieces, col = n0 + 4 * (piece % kPieces);
                const bool inside = row < M && col < N;
                if (OUT_BF16) res16[r] = inside ? *(const u32x2 *)((const __bf16 *)residual + (size_t)row * N + col) : u32x2{0u, 0u};
                else res[r] = inside ? *(const f32x4 *)((const float *)residual + (size_t)row * N + col) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        lds_barrier();  // nobody reads the ring, or the rows before, any more
#pragma unroll
        for (int nt = 0; nt < 3; ++nt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                f32x4 val = {acc[nt][mt][4 * q4], acc[nt][mt][4 * q4 + 1], acc[nt][mt][4 * q4 + 2], acc[nt][mt][4 * q4 + 3]};
                val += bias_reg[nt][q4];
                tile_activation<EPI>(val, phi_table);
                if (kStageF32) *(f32x4 *)(stage + li * kPitch + 384 * wn + 128 * nt + 32 * q4 + 16 * g) = val;
                else *(u32x2 *)(stage + li * kPitch + 192 * wn + 64 * nt + 16 * q4 + 8 * g) = u32x2{pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3])};
            }
        lds_barrier();
#pragma unroll
        for (int r = 0; r < kPasses; ++r) {
            const int piece = lane + 64 * r, srow = piece / kPieces, sp = piece % kPieces, row = row0 + srow;
            const int col = n0 + (kStageF32 ? 4 : 8) * sp;
            const bool inside = row < M && col < N;  // (N % 8 == 0: a piece is in or out whole)
            const u32x4 raw = *(const u32x4 *)(stage + (16 * wn + srow) * kPitch + 16 * sp);
            if (!kStageF32) {
                if (inside) *(u32x4 *)((__bf16 *)Y + (size_t)row * N + col) = raw;
            } else {
                f32x4 out = __builtin_bit_cast(f32x4, raw);
                if (OUT_BF16) {
                    out[0] += bf16_lo(res16[r][0]); out[1] += bf16_hi(res16[r][0]);
                    out[2] += bf16_lo(res16[r][1]); out[3] += bf16_hi(res16[r][1]);
                    if (inside) *(u32x2 *)((__bf16 *)Y + (size_t)row * N + col) = u32x2{pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3])};
                } else {
                    if (kResidual) out += res[r];
                    if (inside) *(f32x4 *)((float *)Y + (size_t)row * N + col) = out;
                }
            }
        }
    }
#endif
}

template <int EPI, bool OUT_BF16>
static jv_status launch_tile192(const void *a, const void *w, const float *bias, const void *residual, void *y, int M, int N, int K,
                                int lda, hipStream_t stream) {
    static LdsLimit lds_limit;
    jv_status st = ensure_lds_limit(lds_limit, (const void *)gemm_tile192_kernel<EPI, OUT_BF16>, kTile192Lds);
    if (st != JV_OK) return st;
    const int tiles_m = (M + 255) / 256, tiles_n = (N + kT192N - 1) / kT192N;
    hipLaunchKernelGGL((gemm_tile192_kernel<EPI, OUT_BF16>), dim3(8 * ((tiles_m * tiles_n + 7) / 8)), dim3(512), kTile192Lds, stream,
                       (const __bf16 *)a, (const __bf16 *)w, bias, residual, y, M, N, K, lda, tiles_m, tiles_n, M < N ? 1 : 0);
    return launch_status("gemm_tile192_kernel");
}
static jv_status tile192_epilogue(int epi, bool out_bf16, const void *a, const void *w, const float *bias, const void *residual, void *y,
                                  int M, int N, int K, int lda, hipStream_t stream) {
    switch (epi) {
        case JV_EPI_NONE: return out_bf16 ? launch_tile192<JV_EPI_NONE, true>(a, w, bias, residual, y, M, N, K, lda, stream) : launch_tile192<JV_EPI_NONE, false>(a, w, bias, residual, y, M, N, K, lda, stream);
        case JV_EPI_GELU: return out_bf16 ? launch_tile192<JV_EPI_GELU, true>(a, w, bias, residual, y, M, N, K, lda, stream) : launch_tile192<JV_EPI_GELU, false>(a, w, bias, residual, y, M, N, K, lda, stream);
        case JV_EPI_RESIDUAL: return out_bf16 ? launch_tile192<JV_EPI_RESIDUAL, true>(a, w, bias, residual, y, M, N, K, lda, stream) : launch_tile192<JV_EPI_RESIDUAL, false>(a, w, bias, residual, y, M, N, K, lda, stream);
        case JV_EPI_SILU: return out_bf16 ? launch_tile192<JV_EPI_SILU, true>(a, w, bias, residual, y, M, N, K, lda, stream) : launch_tile192<JV_EPI_SILU, false>(a, w, bias, residual, y, M, N, K, lda, stream);
    }
    return fail(JV_ERR_INVALID_ARG, "unknown epilogue");
}

template <int WM, int WN, int MT, int STAGES, int EPI, bool OUT_BF16, bool PARTS = false>
static jv_status launch_tiles(int k_split, long long y_split, const void *a, const void *w, const float *bias,
                              const void *residual, void *y, int M, int N, int K, int lda, hipStream_t stream, int parts = 1) {
    using S = TileShape<WM, WN, MT, STAGES, EPI>;
    auto kernel = gemm_tile_kernel<WM, WN, MT, STAGES, EPI, OUT_BF16, PARTS>;
    static LdsLimit lds_limit;
    jv_status st = ensure_lds_limit(lds_limit, (const void *)kernel, S::kLds);
    if (st != JV_OK) return st;
    const int tiles_m = (M + S::kBM - 1) / S::kBM, tiles_n = (N + S::kBN - 1) / S::kBN;
    const dim3 grid(8 * ((tiles_m * tiles_n * k_split + 7) / 8));
    hipLaunchKernelGGL(kernel, grid, dim3(S::kThreads), S::kLds, stream, (const __bf16 *)a, (const __bf16 *)w, bias, residual, y,
                       M, N, K, lda, tiles_m, tiles_n, M < N ? 1 : 0, k_split, y_split, parts);
    return launch_status("gemm_tile_kernel");
}

template <int WM, int WN, int MT, int STAGES, typename... Args>
static jv_status launch_epilogue(int epi, bool out_bf16, Args... args) {
    switch (epi) {
        case JV_EPI_NONE: return out_bf16 ? launch_tiles<WM, WN, MT, STAGES, JV_EPI_NONE, true>(args...) : launch_tiles<WM, WN, MT, STAGES, JV_EPI_NONE, false>(args...);
        case JV_EPI_GELU: return out_bf16 ? launch_tiles<WM, WN, MT, STAGES, JV_EPI_GELU, true>(args...) : launch_tiles<WM, WN, MT, STAGES, JV_EPI_GELU, false>(args...);
        case JV_EPI_RESIDUAL: return out_bf16 ? launch_tiles<WM, WN, MT, STAGES, JV_EPI_RESIDUAL, true>(args...) : launch_tiles<WM, WN, MT, STAGES, JV_EPI_RESIDUAL, false>(args...);
        case JV_EPI_SILU: return out_bf16 ? launch_tiles<WM, WN, MT, STAGES, JV_EPI_SILU, true>(args...) : launch_tiles<WM, WN, MT, STAGES, JV_EPI_SILU, false>(args...);
    }
    return fail(JV_ERR_INVALID_ARG, "unknown epilogue");
}

jv_status gemm_tiles_forward(GemmTile tile, int k_split, long long y_split, const void *a, const void *w,
                             const float *bias, const void *residual, void *y, int M, int N, int K, int lda,
                             int epi, bool out_bf16, hipStream_t stream) {
    switch (tile) {
        case kTile256x192: return tile192_epilogue(epi, out_bf16, a, w, bias, residual, y, M, N, K, lda, stream);
        case kTile256x128: return launch_epilogue<4, 2, 2, 3>(epi, out_bf16, k_split, y_split, a, w, bias, residual, y, M, N, K, lda, stream);
        case kTile128x128Deep: return launch_epilogue<2, 2, 2, 4>(epi, out_bf16, k_split, y_split, a, w, bias, residual, y, M, N, K, lda, stream);
        case kTile128x128: return launch_epilogue<2, 2, 2, 2>(epi, out_bf16, k_split, y_split, a, w, bias, residual, y, M, N, K, lda, stream);
        case kTile64x128: return launch_epilogue<2, 2, 1, 3>(epi, out_bf16, k_split, y_split, a, w, bias, residual, y, M, N, K, lda, stream);
        case kTile64x64: return launch_epilogue<2, 1, 1, 4>(epi, out_bf16, k_split, y_split, a, w, bias, residual, y, M, N, K, lda, stream);
        default: return fail(JV_ERR_INVALID_ARG, "no kernel for this tile shape");
    }
}

template <int WM, int WN, int MT, int STAGES, typename... Args>
static jv_status launch_parts(bool out_bf16, Args... args) {
    return out_bf16 ? launch_tiles<WM, WN, MT, STAGES, JV_EPI_RESIDUAL, true, true>(args...) : launch_tiles<WM, WN, MT, STAGES, JV_EPI_RESIDUAL, false, true>(args...);
}
jv_status gemm_residual_parts(GemmTile tile, int parts, const void *a, const void *w, const float *bias, const void *residual, void *y,
                              int M, int N, int K, bool out_bf16, hipStream_t stream) {
    switch (tile) {
        case kTile256x128: return launch_parts<4, 2, 2, 3>(out_bf16, 1, 0, a, w, bias, residual, y, M, N, K, K, stream, parts);
        case kTile128x128Deep: return launch_parts<2, 2, 2, 4>(out_bf16, 1, 0, a, w, bias, residual, y, M, N, K, K, stream, parts);
        case kTile64x128: return launch_parts<2, 2, 1, 3>(out_bf16, 1, 0, a, w, bias, residual, y, M, N, K, K, stream, parts);
        default: return fail(JV_ERR_INVALID_ARG, "no kernel for this tile shape");
    }
}

}  // namespace jv
