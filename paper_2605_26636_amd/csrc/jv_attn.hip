// Softmax attention over windows of the token grid (Sec. 3.2.2 of the paper) and over the whole
// grid (Eq. 1).  Full attention is the one-window case of the same kernels: a window that
// spans the grid.  Queries and keys are addressed by (window, slot); slot -> token is the
// row-major position inside the window, and slots that fall outside the H x W grid are
// padding: excluded as keys, skipped as queries.
#include <math.h>

#include "jv_common.h"
#include "jv_mfma.h"
#include "jv_plan.h"

namespace jv {

// slot of window (wy, wx) -> token index, or -1 for padding / past the window.
__device__ inline int slot_token(const WindowGeom &g, int wy, int wx, int slot) {
    if (slot >= g.slots) return -1;
    int r = wy * g.wh + slot / g.ww, c = wx * g.ww + slot % g.ww;
    return (r < g.H && c < g.W) ? r * g.W + c : -1;
}

// ---------------------------------------------------------------------------------------
// fp32 path: tiles of 32 keys x 32 queries on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32: fp32 operands and accumulation, 64 cycles per instruction).
// Bound by those instructions: 128 of them per tile against 16 exponentials per lane.  Scores
// are formed transposed, S^T = K Q^T, so that a lane owns one query column: the maximum and the
// sum are in-lane plus one exchange with lane ^ 32, and accumulator register v of the score tile
// is, as it stands, the B operand of step v of O^T += V^T P^T (k-slot g of step v is the key that
// lane half g holds in register v).
// A workgroup is four wavefronts, QW = 4 / KW blocks of 32 queries times KW groups of keys: per
// step it stages KW tiles of K and V in LDS (fetched into registers under the arithmetic of the
// step before) and wavefront (qw, kw) takes tile kw.  With KW > 1 the KW running softmaxes of a
// query block are merged through LDS at the end.  KW = 2 and 4 cut a problem of few queries into two
// and four times as many wavefronts (attn_direct_f32 takes most launches that KW = 4 could: f32_keys_staged);
// KW = 1 stages a quarter of the bytes per flop.
// Measured: 2 304 tokens x 64 heads 798 us = 109 TFLOP/s (a loop of these instructions alone reaches 138, at
// the 2.1 GHz the chip holds under them).
// Only the first q_slots query slots of every window are computed.
// grid (ceil(q_slots / (32 QW)), n_win, B*heads), 256 threads.
// ---------------------------------------------------------------------------------------
constexpr int kF32Tile = 2 * 32 * kHeadDim * 4;  // K rows, then V rows, of 32 keys: 16 KB

// Workgroup -> (query block, window, batch * head) with a contiguous range of the launch per XCD
// (the hardware deals workgroups to the eight XCDs in turn): the query blocks that read one
// head's keys share an L2.
__device__ inline void f32_item(int &qblock, int &win, int &bh) {
    const long long nx = gridDim.x, ny = gridDim.y, total = nx * ny * gridDim.z;
    const long long lin = blockIdx.x + nx * (blockIdx.y + ny * blockIdx.z);
    const long long share = total >> 3, extra = total & 7, xcd = lin & 7;
    const long long item = xcd * share + (xcd < extra ? xcd : extra) + (lin >> 3);
    qblock = (int)(item % nx);
    win = (int)((item / nx) % ny);
    bh = (int)(item / (nx * ny));
}

// Tail of the fp32 kernels.  A wavefront without partners stores its rows ...
__device__ inline void f32_store_row(const f32x16 (&acc)[2], float inv, float *row) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            f32x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = acc[cb][4 * v4 + e] * inv;
            *(f32x4 *)(row + 32 * cb + 8 * v4) = out;
        }
}
// ... and one with partners leaves its sums as [query][channel] rows of 256 bytes (chunks rotated by the row) for
__device__ inline void f32_park(const f32x16 (&acc)[2], unsigned char *mine, int li, int half) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const f32x4 part = {acc[cb][4 * v4], acc[cb][4 * v4 + 1], acc[cb][4 * v4 + 2], acc[cb][4 * v4 + 3]};
            *(f32x4 *)(mine + li * 256 + (((8 * cb + 2 * v4 + half) ^ (li & 15)) << 4)) = part;
        }
}
// the merge of the KW softmaxes of each query block: O = sum_k 2^(m_k - M) acc_k / sum_k 2^(m_k - M) l_k.
template <int KW, class Token>
__device__ inline void f32_merge(const unsigned char *parts, const float (&ms)[4][32], const float (&ls)[4][32], int qblock, int q_slots,
                                 Token token, float *op, long long sn, int tid) {
    constexpr int QW = 4 / KW;
    const int chunk = tid & 15, srow = tid >> 4;
#pragma unroll
    for (int i = 0; i < 2 * QW; ++i) {
        const int query = srow + 16 * i, w0 = (query >> 5) * KW, ql = query & 31;
        const int slot = qblock * (32 * QW) + query;
        const int tok = slot < q_slots ? token(slot) : -1;
        if (tok < 0) continue;
        float top = ms[w0][ql];
#pragma unroll
        for (int k = 1; k < KW; ++k) top = fmaxf(top, ms[w0 + k][ql]);
        f32x4 out = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const float w = __builtin_amdgcn_exp2f(ms[w0 + k][ql] - top);
            out += w * *(const f32x4 *)(parts + (w0 + k) * (32 * 256) + ql * 256 + ((chunk ^ (ql & 15)) << 4));
            den = fmaf(w, ls[w0 + k][ql], den);
        }
        *(f32x4 *)(op + (long long)tok * sn + 4 * chunk) = out * (1.0f / den);
    }
}

template <int KW>
__global__ void __launch_bounds__(256, 2)
attn_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads,
         float scale_log2, int q_slots) {
    constexpr int QW = 4 / KW;
    __shared__ __align__(16) unsigned char tiles[KW * kF32Tile];
    __shared__ __align__(16) float bias[KW * 32];  // 0 for a real key, -inf for padding
    __shared__ float ms[4][32], ls[4][32];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    const int kw = wave % KW, qw = wave / KW;
    int qblock, win, bh;
    f32_item(qblock, win, bh);
    const int b = bh / heads, h = bh % heads, wy = win / g.wins_x, wx = win % g.wins_x;
    const float *qp = (const float *)qt.ptr + b * qt.sb + h * qt.sh;
    const float *kp = (const float *)kt.ptr + b * kt.sb + h * kt.sh;
    const float *vp = (const float *)vt.ptr + b * vt.sb + h * vt.sh;
    float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh;
    const int first = wy * g.wh * g.W + wx * g.ww;  // the window's first token: always real
    const bool padded = (wy + 1) * g.wh > g.H || (wx + 1) * g.ww > g.W;
    const bool rows = g.ww == g.W;                  // windows of whole grid rows: slots are consecutive tokens
    auto token = [&](int slot) {
        if (!rows) return slot_token(g, wy, wx, slot);
        return slot < g.slots && first + slot < g.H * g.W ? first + slot : -1;
    };

    // Queries: lane (half, li) holds channels 32 half .. +31 of query li.
    const int q0 = qblock * (32 * QW) + qw * 32;
    const bool live = q0 < q_slots;  // the same in the whole wavefront
    f32x4 q[8];
    int qtok = q0 + li < q_slots ? token(q0 + li) : -1;
    {
        const float *row = qp + (long long)(qtok < 0 ? first : qtok) * qt.sn + 32 * half;
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = *(const f32x4 *)(row + 4 * i);
    }
    f32x16 acc[2];  // channels 32 cb + 8 (v / 4) + 4 half + v % 4 of query li
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
    float m = -INFINITY, l = 0.f;

    // Staging: this thread moves 16-byte chunk `chunk` of rows srow + 16 i of a step's KW tiles.
    // K rows are read a row per lane (chunk rotated by the row), V rows 32 channels at a time by
    // the two lane halves, four rows apart (row halves exchanged in every other group of four
    // rows): both without bank conflicts.
    const int chunk = tid & 15, srow = tid >> 4;
    f32x4 kreg[2 * KW], vreg[2 * KW];
    float breg[2 * KW];
    auto fetch = [&](int step) {
#pragma unroll
        for (int i = 0; i < 2 * KW; ++i) {
            int tok = token(step * (32 * KW) + srow + 16 * i);
            breg[i] = tok < 0 ? -INFINITY : 0.f;
            if (tok < 0) tok = first;
            kreg[i] = *(const f32x4 *)(kp + (long long)tok * kt.sn + 4 * chunk);
            vreg[i] = *(const f32x4 *)(vp + (long long)tok * vt.sn + 4 * chunk);
        }
    };
    auto stage = [&]() {
#pragma unroll
        for (int i = 0; i < 2 * KW; ++i) {
            const int r = (srow + 16 * i) & 31;
            unsigned char *tile = tiles + (i >> 1) * kF32Tile + r * 256;
            if (breg[i] != 0.f) kreg[i] = vreg[i] = f32x4{0.f, 0.f, 0.f, 0.f};  // 0 x inf of a padded key's row would be NaN
            *(f32x4 *)(tile + ((chunk ^ (r & 15)) << 4)) = kreg[i];
            *(f32x4 *)(tile + kF32Tile / 2 + ((chunk ^ ((r & 4) << 1)) << 4)) = vreg[i];
            if (chunk == 0) bias[srow + 16 * i] = breg[i];
        }
    };
    const unsigned char *ktile = tiles + kw * kF32Tile, *vtile = ktile + kF32Tile / 2;
    const int n_step = (g.slots + 32 * KW - 1) / (32 * KW);
    fetch(0);
    for (int step = 0; step < n_step; ++step) {
        if (step > 0) __syncthreads();  // the tiles before have been read
        stage();
        __syncthreads();
        if (step + 1 < n_step) fetch(step + 1);
        if (!live || (step * KW + kw) * 32 >= g.slots) continue;
        f32x16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const f32x4 kk = *(const f32x4 *)(ktile + li * 256 + (((8 * half + i) ^ (li & 15)) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[e], q[i][e], s, 0, 0, 0);
        }
        float top = -INFINITY;
        if (padded || (step * KW + kw + 1) * 32 > g.slots) {  // (uniform) only here can a key be padding
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const f32x4 bb = *(const f32x4 *)(bias + 32 * kw + 8 * v4 + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[4 * v4 + e] += bb[e];
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) top = fmaxf(top, s[v]);
        float lo, hi;
        pair_values(top, &lo, &hi);
        const float m_new = fmaxf(m, fmaxf(lo, hi) * scale_log2);
        const float ref = m_new == -INFINITY ? 0.f : m_new;  // padding only so far
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        m = m_new;
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], scale_log2, -ref));
            sum += s[v];
        }
        l = fmaf(l, alpha, sum);
        if (__any(alpha != 1.0f)) {  // some query's maximum went up: rare after the first tiles
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[0][v] *= alpha;
                acc[1][v] *= alpha;
            }
        }
        const unsigned char *vrow = vtile + half * 4 * 256 + ((li * 4) ^ (half * 128));
        const unsigned char *vrow1 = vtile + half * 4 * 256 + ((li * 4) ^ (half * 128) ^ 128);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int off = (8 * (v / 4) + v % 4) * 256;
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(*(const float *)(vrow + off), s[v], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(*(const float *)(vrow1 + off), s[v], acc[1], 0, 0, 0);
        }
    }
    {
        float lo, hi;
        pair_values(l, &lo, &hi);
        l = lo + hi;
    }
    if (KW == 1) {
        if (qtok >= 0) f32_store_row(acc, 1.0f / l, op + (long long)qtok * ot.sn + 4 * half);
        return;
    }
    __syncthreads();
    f32_park(acc, tiles + wave * (32 * 256), li, half);
    if (half == 0) {
        ms[wave][li] = m;
        ls[wave][li] = l;
    }
    __syncthreads();
    f32_merge<KW>(tiles, ms, ls, qblock, q_slots, token, op, ot.sn, tid);
}

// attn_f32<4> with K and V fetched straight into operand registers: its wavefronts share queries and
// no keys, so nothing is staged and the key loop has no barrier.  A contraction step takes channels
// 8 i + 4 half + e (i = 0 .. 7, e = 0 .. 3): a lane's K and Q operands are 16-byte pieces of one row and an
// instruction reads 32 bytes of every row; a V operand is one dword of a row, an instruction
// two runs of 128 bytes.  Half tiles of K and V rotate through three sets of sixteen registers, each
// fetched while the matrix instructions of two others run (1 024 cycles each); with no LDS but the merge's
// and 168 registers three workgroups fit a compute unit.  Against attn_f32<4>, us: 1 369 tokens x 12 heads
// 104.6 -> 87.2 (516 workgroups: four units have three and the others two; x 11 68.7 -> 60.0), 256 x 6 10.6 -> 9.7,
// 1 025 + 5 x 36 139 -> 112, windows of 14 x 14 on 40 x 40 x 24 49.4 -> 39.7.  The matrix instructions are 44 us of the 61.
// (Two chains of score products instead of one: the same; two workgroups per unit and more registers: the same.)
// grid (ceil(q_slots / 32), n_win, B*heads), 256 threads.  Byte offsets inside a (batch, head) slice of K
// and V below 2^32.
__global__ void __launch_bounds__(256, 3)
attn_direct_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads,
                float scale_log2, int q_slots) {
    constexpr int KW = 4;
    __shared__ __align__(16) unsigned char parts[4 * 32 * 256];
    __shared__ float ms[4][32], ls[4][32];
    const int tid = threadIdx.x, kw = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    int qblock, win, bh;
    f32_item(qblock, win, bh);
    const int b = bh / heads, h = bh % heads, wy = win / g.wins_x, wx = win % g.wins_x;
    const float *qp = (const float *)qt.ptr + b * qt.sb + h * qt.sh;
    const char *kp = (const char *)((const float *)kt.ptr + b * kt.sb + h * kt.sh);  // (uniform)
    const char *vp = (const char *)((const float *)vt.ptr + b * vt.sb + h * vt.sh);
    const unsigned ksn = 4u * (unsigned)kt.sn, vsn = 4u * (unsigned)vt.sn;
    const unsigned vlane = 4u * half * vsn + 4u * li;
    const int first = wy * g.wh * g.W + wx * g.ww;  // the window's first token: always real
    const bool rows = g.ww == g.W;                  // windows of whole grid rows: slots are consecutive tokens
    auto token = [&](int slot) {
        if (!rows) return slot_token(g, wy, wx, slot);
        return slot < g.slots && first + slot < g.H * g.W ? first + slot : -1;
    };
    f32x4 q[8];
    {
        const int slot = qblock * 32 + li, qtok = slot < q_slots ? token(slot) : -1;
        const float *row = qp + (long long)(qtok < 0 ? first : qtok) * qt.sn + 4 * half;
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = *(const f32x4 *)(row + 8 * i);
    }
    f32x16 acc[2];  // channels 32 cb + 8 (v / 4) + 4 half + v % 4 of query li
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
    float m = -1.0e30f, l = 0.f;  // (finite stand-in for "no maximum yet")
    const int n_tile = (g.slots + 31) / 32;
    float set[3][16];
    // K operands of steps 4 hf .. + 3 of the tile whose key li is token `tok` (negative: padding)
    auto fetch_k = [&](float (&r)[16], int tok, int hf) __attribute__((always_inline)) {
        const unsigned at = (unsigned)(tok < 0 ? first : tok) * ksn + 16u * half;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 x = *(const f32x4 *)(kp + at + 32 * (4 * hf + i));
#pragma unroll
            for (int e = 0; e < 4; ++e) r[4 * i + e] = x[e];
        }
    };
    // r[2 j + cb]: channel 32 cb + li of key 16 hf + 8 (j / 4) + 4 half + j % 4
    auto fetch_v = [&](float (&r)[16], int tok, unsigned pad, int hf) __attribute__((always_inline)) {
        if (rows && pad == 0u) {
            const char *row = vp + (unsigned)(__builtin_amdgcn_readfirstlane(tok) + 16 * hf) * (size_t)vsn;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                r[2 * j] = *(const float *)(row + vlane);
                r[2 * j + 1] = *(const float *)(row + vlane + 128);
                row += (j == 3 ? 5 : 1) * (size_t)vsn;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int t = __shfl(tok, 16 * hf + 8 * (j / 4) + 4 * half + j % 4, 64);
                const unsigned at = (unsigned)(t < 0 ? first : t) * vsn + 4u * li;
                r[2 * j] = *(const float *)(vp + at);
                r[2 * j + 1] = *(const float *)(vp + at + 128);
            }
            // (keeps the two branches' loads apart: merged into one set they would take every address
            // in a vector register of its own)
            asm volatile("");
        }
    };
    auto real_token = [&](int tile, int &tok, unsigned &pad) __attribute__((always_inline)) {
        tok = token(32 * tile + li);
        pad = (unsigned)__builtin_amdgcn_ballot_w64(tok < 0);  // bit j: key j of the tile is padding
    };
    int tok = 0;
    unsigned pad = 0u;
    // A tile whose K operands are in (or on their way to) ka and kb; leaves those of tile + KW in kb and vc.
    auto run_tile = [&](int tile, float (&ka)[16], float (&kb)[16], float (&vc)[16]) __attribute__((always_inline)) {
        const int cur = tok;
        const unsigned cur_pad = pad, pads = half ? pad >> 4 : pad;
        const bool more = tile + KW < n_tile;
        fetch_v(vc, cur, cur_pad, 0);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[i], q[i / 4][i % 4], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_v(ka, cur, cur_pad, 1);
        if (more) real_token(tile + KW, tok, pad);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kb[i], q[4 + i / 4][i % 4], s, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_k(kb, tok, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (cur_pad != 0u) {  // (uniform) padded keys have no weight ...
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j] = (pads >> (8 * (j / 4) + j % 4)) & 1u ? -INFINITY : s[j];
        }
        // The reference stays while no logit is more than 8 binary orders above it (numerator and
        // denominator share it, so the result is the same), and goes up to the maximum otherwise.  The weights
        // take a factor of 2^-8, exactly: none is above 1, and values up to the largest floats pass through the
        // sums as under the maximum itself.  (The sixteen products: 1.5 % of a launch that leaves units with one
        // workgroup.  A reference 8 orders up instead costs none, but rounds the exponents of the largest weights
        // more coarsely: 4.7e-7 against 4.5e-7 from 64 bits at 1 369 tokens.)
        float top = s[0];
#pragma unroll
        for (int j = 1; j < 16; ++j) top = fmaxf(top, s[j]);
        if (__any(top * scale_log2 > m + 8.0f)) {
            float lo, hi;
            pair_values(top, &lo, &hi);
            const float m_new = fmaxf(m, fmaxf(lo, hi) * scale_log2), alpha = __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                acc[0][j] *= alpha;
                acc[1][j] *= alpha;
            }
        }
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            s[j] = __builtin_amdgcn_exp2f(fmaf(s[j], scale_log2, -m)) * 0x1p-8f;
            sum += s[j];
        }
        l += sum;
        auto product = [&](float (&r)[16], int hf) __attribute__((always_inline)) {
            if (cur_pad != 0u) {  // ... and zeros for the values they meet (0 x inf would be NaN)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool p = (pads >> (16 * hf + 8 * (j / 4) + j % 4)) & 1u;
                    r[2 * j] = p ? 0.f : r[2 * j];
                    r[2 * j + 1] = p ? 0.f : r[2 * j + 1];
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(r[2 * j], s[8 * hf + j], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(r[2 * j + 1], s[8 * hf + j], acc[1], 0, 0, 0);
            }
        };
        product(vc, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_k(vc, tok, 1);
        __builtin_amdgcn_sched_barrier(0);
        product(ka, 1);
    };
    if (kw < n_tile) {
        real_token(kw, tok, pad);
        fetch_k(set[0], tok, 0);
        fetch_k(set[1], tok, 1);
        for (int tile = kw;;) {
            run_tile(tile, set[0], set[1], set[2]);
            if ((tile += KW) >= n_tile) break;
            run_tile(tile, set[1], set[2], set[0]);
            if ((tile += KW) >= n_tile) break;
            run_tile(tile, set[2], set[0], set[1]);
            if ((tile += KW) >= n_tile) break;
        }
    }
    {
        float lo, hi;
        pair_values(l, &lo, &hi);
        l = lo + hi;
    }
    f32_park(acc, parts + kw * (32 * 256), li, half);
    if (half == 0) {
        ms[kw][li] = m;
        ls[kw][li] = l;
    }
    __syncthreads();
    float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh;
    f32_merge<KW>(parts, ms, ls, qblock, q_slots, token, op, ot.sn, tid);
}

// Windows of a few slots, of which a 32 x 32 tile would be padding but for a corner: sixteen lanes per
// query (four channels each) walk over the real tokens of its window.  Bound by the tensors' way
// through memory and, with more keys, by the exchange that ends each dot product.
// grid (ceil(tokens / 16), B*heads), 256 threads.
__global__ void __launch_bounds__(256)
attn_small_window_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads, float scale) {
    const int tok = blockIdx.x * 16 + (threadIdx.x >> 4), c4 = 4 * (threadIdx.x & 15);
    if (tok >= g.H * g.W) return;  // all sixteen lanes
    const int bh = blockIdx.y, b = bh / heads, h = bh % heads;
    const float *kp = (const float *)kt.ptr + b * kt.sb + h * kt.sh + c4;
    const float *vp = (const float *)vt.ptr + b * vt.sb + h * vt.sh + c4;
    const f32x4 q = *(const f32x4 *)((const float *)qt.ptr + b * qt.sb + h * qt.sh + (long long)tok * qt.sn + c4);
    const int row = tok / g.W, col = tok % g.W, r0 = row - row % g.wh, c0 = col - col % g.ww;
    const int r1 = min(r0 + g.wh, g.H), c1 = min(c0 + g.ww, g.W);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (int r = r0; r < r1; ++r)
        for (int c = c0; c < c1; ++c) {
            const f32x4 k = *(const f32x4 *)(kp + (long long)(r * g.W + c) * kt.sn);
            const f32x4 v = *(const f32x4 *)(vp + (long long)(r * g.W + c) * vt.sn);
            float s = fmaf(q[0], k[0], q[1] * k[1]) + fmaf(q[2], k[2], q[3] * k[3]);
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            s *= scale;
            const float m_new = fmaxf(m, s), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = expf(m - ref), p = expf(s - ref);
            m = m_new;
            l = fmaf(l, alpha, p);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(acc[e], alpha, p * v[e]);
        }
    *(f32x4 *)((float *)ot.ptr + b * ot.sb + h * ot.sh + (long long)tok * ot.sn + c4) = acc * (1.0f / l);
}

// q_slots: number of leading query slots of each window to compute (all keys always take part).  With
// fewer than all of them the rows of O behind them are scratch.
jv_status attn_bf16_check(const Problem &pr, const WindowGeom &g, int q_slots);
jv_status attn_bf16(const Problem &pr, const WindowGeom &g, float scale, int q_slots, hipStream_t stream);

template <int KW>
static jv_status launch_attn_f32(const Problem &pr, const WindowGeom &g, float scale, int q_slots, hipStream_t stream) {
    constexpr int kQueries = 32 * (4 / KW);
    const dim3 grid((unsigned)((q_slots + kQueries - 1) / kQueries), g.n_win, pr.B * pr.heads);
    hipLaunchKernelGGL(attn_f32<KW>, grid, dim3(256), 0, stream, pr.q, pr.k, pr.v, pr.o, g, pr.heads,
                       scale * 1.4426950408889634f, q_slots);
    return launch_status("attn_f32");
}

static jv_status attn_dispatch(const Problem &pr, const WindowGeom &g, float scale, int q_slots,
                               hipStream_t stream) {
    if (pr.bf16) return attn_bf16(pr, g, scale, q_slots, stream);
    if (g.n_win > 65535) return fail(JV_ERR_UNSUPPORTED, "more than 65535 windows");
    if (q_slots > g.slots) q_slots = g.slots;
    // Tiles / lanes per query, us: 64 x 64 tokens x 6 heads in windows of 1 slot 161 / 6.5, of 4 44 / 8.8, of 8
    // 24 / 11, of 16 15 / 16; 16 x 16 tokens x 6 heads of 8 slots 5.8 / 5.6, of 9 5.8 / 6.0, of 12 5.8 / 7.0.
    if (g.slots <= 8 && q_slots == g.slots) {
        hipLaunchKernelGGL(attn_small_window_f32, dim3((g.H * g.W + 15) / 16, pr.B * pr.heads), dim3(256), 0, stream,
                           pr.q, pr.k, pr.v, pr.o, g, pr.heads, scale);
        return launch_status("attn_small_window_f32");
    }
    // Key groups per query block: as long as the launch has fewer than four wavefronts per SIMD
    // (1 024 SIMDs) with every wavefront on queries of its own, the keys of a window are cut
    // over two or four wavefronts, if it has tiles for them.
    const long long waves = (long long)((q_slots + 31) / 32) * g.n_win * pr.B * pr.heads;
    const int tiles = (g.slots + 31) / 32;
    if (waves < 2048 && tiles > 2) {
        const long long max_sn = pr.k.sn > pr.v.sn ? pr.k.sn : pr.v.sn;
        if (f32_keys_staged(tiles, g.ww == g.W, waves, ((long long)g.H * g.W + 64) * max_sn * 4))
            return launch_attn_f32<4>(pr, g, scale, q_slots, stream);
        hipLaunchKernelGGL(attn_direct_f32, dim3((unsigned)((q_slots + 31) / 32), g.n_win, pr.B * pr.heads), dim3(256), 0, stream,
                           pr.q, pr.k, pr.v, pr.o, g, pr.heads, scale * 1.4426950408889634f, q_slots);
        return launch_status("attn_direct_f32");
    }
    if (waves < 4096 && tiles > 1) return launch_attn_f32<2>(pr, g, scale, q_slots, stream);
    return launch_attn_f32<1>(pr, g, scale, q_slots, stream);
}

// All tokens of the sequence as one window of 1 x N slots (token = slot).
static WindowGeom sequence_geom(int N) {
    WindowGeom g;
    g.H = 1; g.W = N; g.wh = 1; g.ww = N;
    g.Hp = 1; g.Wp = N; g.wins_x = 1; g.wins_y = 1; g.n_win = 1; g.slots = N;
    return g;
}

// The same tensors from token `first` on.
static TensorArg from_token(const TensorArg &t, int first, bool bf16) {
    TensorArg r = t;
    r.ptr = (const char *)t.ptr + (long long)first * t.sn * (bf16 ? 2 : 4);
    return r;
}

jv_status window_check(const Problem &pr, int wh, int ww) {
    WindowGeom g;
    jv_status st = make_window_geom(pr.H, pr.W, wh, ww, &g);
    if (st != JV_OK) return st;
    if (g.n_win > 65535) return fail(JV_ERR_UNSUPPORTED, "more than 65535 windows");
    return JV_OK;
}

jv_status window_forward(const Problem &pr, int wh, int ww, float scale, hipStream_t stream) {
    WindowGeom g;
    jv_status st = window_check(pr, wh, ww);
    if (st != JV_OK) return st;
    // fp32: a window side beyond the grid's ends with the grid, which has the same windows without the tiles of
    // padding (8 x 8 tokens x 6 heads in windows of 64 x 64: 332 us with them, 8 without).
    if (pr.bf16) make_window_geom(pr.H, pr.W, wh, ww, &g);
    else make_window_geom(pr.H, pr.W, wh < pr.H ? wh : pr.H, ww < pr.W ? ww : pr.W, &g);
    if (pr.P == 0) return attn_dispatch(pr, g, resolve_scale(scale, pr.D), g.slots, stream);
    // Prefix tokens: the grid tokens run window attention among themselves; the prefix
    // tokens (the first P query slots of the whole sequence) attend to every token.
    Problem grid = pr;
    grid.P = 0;
    grid.N = pr.H * pr.W;
    grid.q = from_token(pr.q, pr.P, pr.bf16);
    grid.k = from_token(pr.k, pr.P, pr.bf16);
    grid.v = from_token(pr.v, pr.P, pr.bf16);
    grid.o = from_token(pr.o, pr.P, pr.o_bf16);
    // The prefix tokens go first: their partial sums lie in the grid rows of O until the windows
    // overwrite them.  Nothing is launched for a grid that the window kernels refuse.
    if (pr.bf16 && (st = attn_bf16_check(grid, g, g.slots)) != JV_OK) return st;
    if ((st = attn_dispatch(pr, sequence_geom(pr.N), resolve_scale(scale, pr.D), pr.P, stream)) != JV_OK) return st;
    return attn_dispatch(grid, g, resolve_scale(scale, pr.D), g.slots, stream);
}

jv_status full_forward(const Problem &pr, float scale, hipStream_t stream) {
    if (pr.P > 0) return attn_dispatch(pr, sequence_geom(pr.N), resolve_scale(scale, pr.D), pr.N, stream);
    // One window that spans the grid; the token order inside it is the raster order.
    WindowGeom g;
    g.H = pr.H; g.W = pr.W; g.wh = pr.H; g.ww = pr.W;
    g.Hp = pr.H; g.Wp = pr.W; g.wins_x = 1; g.wins_y = 1; g.n_win = 1; g.slots = pr.N;
    return attn_dispatch(pr, g, resolve_scale(scale, pr.D), g.slots, stream);
}

}  // namespace jv

extern "C" {

jv_status jv_window_attn_fwd(const jv_attn_desc *desc, const void *q, const void *k,
                             const void *v, void *o, int32_t win_h, int32_t win_w, float scale,
                             void *hip_stream) {
    jv::clear_error();
    jv::Problem pr;
    jv_status st = jv::make_problem(desc, q, k, v, o, &pr);
    if (st != JV_OK) return st;
    return jv::window_forward(pr, win_h, win_w, scale, (hipStream_t)hip_stream);
}

jv_status jv_full_attn_fwd(const jv_attn_desc *desc, const void *q, const void *k,
                           const void *v, void *o, float scale, void *hip_stream) {
    jv::clear_error();
    jv::Problem pr;
    jv_status st = jv::make_problem(desc, q, k, v, o, &pr);
    if (st != JV_OK) return st;
    return jv::full_forward(pr, scale, (hipStream_t)hip_stream);
}

}  // extern "C"
