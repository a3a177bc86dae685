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
// fp32 path: tiles of 32 keys x 32 queries on the bf16 matrix instructions
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation; sixteen times the rate of the fp32 ones).  Every operand is the sum of
// three bf16 numbers, each the rounding of what the ones before leave: all 24 bits of a number, whatever the others are, down to 2^-110 in magnitude (below it
// to 2^-133, the smallest bf16 number).  Six of the nine products are formed; what is left out is below 2^-24 of the product of two numbers (2^-28 of it
// on average).  Errors against 64 bits are those of the rounding of the sums: the small products are added up first, and the
// sums of a tile (attn_f32) or of half a tile (attn_few_f32) on their own before they join the others.  attn_f32: 64 heads of 1 369 tokens 2.0e-7, of
// 2 304 2.3e-7 (fp32 matrix instructions 5.6e-7 and 9.2e-7); attn_few_f32: 12 heads of 1 369 2.4e-7, 8 of 4 096 2.9e-7 (4.5e-7 and 6.5e-7).
// (Two fp16 numbers an operand, scaled by the largest magnitude of K, of V and of a query, and three products: 20 to 30 % faster, but what is 2^14
// times smaller than the largest loses bits, a small channel of V beside a large one for instance.)
// Infinities and NaN turn into NaN on the way (inf - inf), and so does what overflows: a wavefront whose sums are not finite
// goes over its keys once more with the fp32 matrix instructions (f32_again).
// Scores are formed transposed, S^T = K Q^T, so that a lane owns one query column: the maximum and the
// sum are in-lane plus one exchange with lane ^ 32, and accumulator registers 8 f .. + 7 of the score tile
// are, as they stand, the B operand of step f of O^T += V^T P^T (k-slot (g, 4 r + e) of it is key 16 f + 8 r + 4 g + e).
// Only the first q_slots query slots of every window are computed.
// ---------------------------------------------------------------------------------------

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

// A window of one (batch, head) as the kernels address it.
struct F32Window {
    WindowGeom g;
    int wy, wx, first;  // first: the window's first token, always real
    bool rows;          // windows of whole grid rows: slots are consecutive tokens
    const float *q, *k, *v;
    float *o;
    long long qsn, ksn, vsn, osn;
    __device__ int token(int slot) const {  // -1: padding, or past the window
        if (!rows) return slot_token(g, wy, wx, slot);
        return slot < g.slots && first + slot < g.H * g.W ? first + slot : -1;
    }
};
__device__ inline F32Window f32_window(const TensorArg &q, const TensorArg &k, const TensorArg &v, const TensorArg &o, const WindowGeom &g,
                                       int heads, int win, int bh) {
    F32Window w;
    const int b = bh / heads, h = bh % heads;
    w.g = g;
    w.wy = win / g.wins_x;
    w.wx = win % g.wins_x;
    w.first = w.wy * g.wh * g.W + w.wx * g.ww;
    w.rows = g.ww == g.W;
    w.q = (const float *)q.ptr + b * q.sb + h * q.sh;
    w.k = (const float *)k.ptr + b * k.sb + h * k.sh;
    w.v = (const float *)v.ptr + b * v.sb + h * v.sh;
    w.o = (float *)o.ptr + b * o.sb + h * o.sh;
    w.qsn = q.sn;
    w.ksn = k.sn;
    w.vsn = v.sn;
    w.osn = o.sn;
    return w;
}

// A number as the sum of three bf16 numbers, each the rounding of what the ones before leave: 8 + 8 + 8 bits.
struct Split {
    bf16x8 part[3];
};
// What the rounding of x to half `HALF` of r leaves (exact).  One instruction: the dot product of r with (-1, 0) or (0, -1) on top of x.  (The
// constants are hidden from the compiler, which would encode them as the inline -1.0 of 32 bits: another pair of bf16 numbers.)
template <int HALF>
__device__ inline float split_rest(unsigned r, float x) {
    unsigned k = HALF ? 0xbf800000u : 0x0000bf80u;
    asm("" : "+s"(k));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, r), __builtin_bit_cast(bf16x2, k), x, false);
}
// Seven instructions for two numbers.  (The first part of what lies within 2^-9 of the largest float is infinite, see f32_again.)
__device__ inline void split_pair(float x0, float x1, unsigned (&r)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        r[i] = pack_bf16x2(x0, x1);
        if (i == 2) break;
        x0 = split_rest<0>(r[i], x0);
        x1 = split_rest<1>(r[i], x1);
    }
}
__device__ inline Split split8(const float *x) {
    u32x4 part[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned r[3];
        split_pair(x[2 * i], x[2 * i + 1], r);
#pragma unroll
        for (int j = 0; j < 3; ++j) part[j][i] = r[j];
    }
    return {as_bf16x8(part[0]), as_bf16x8(part[1]), as_bf16x8(part[2])};
}
// Four channels of a row into its rows of 128 bytes of the three parts' tiles, one behind the other.
constexpr int kPartTile = 32 * kHeadDim * 2;
__device__ inline void split_store(unsigned char *at, f32x4 x) {
    unsigned a[3], b[3];
    split_pair(x[0], x[1], a);
    split_pair(x[2], x[3], b);
#pragma unroll
    for (int j = 0; j < 3; ++j) *(u32x2 *)(at + j * kPartTile) = u32x2{a[j], b[j]};
}
__device__ inline Split split_load(const unsigned char *at, int stride) {
    Split x;
#pragma unroll
    for (int j = 0; j < 3; ++j) x.part[j] = as_bf16x8(*(const u32x4 *)(at + j * stride));
    return x;
}
// a b + c but for the product of the first parts, smallest first.
__device__ inline f32x16 mfma_small(const Split &a, const Split &b, f32x16 c) {
    c = mfma32(a.part[0], b.part[2], c);
    c = mfma32(a.part[2], b.part[0], c);
    c = mfma32(a.part[1], b.part[1], c);
    c = mfma32(a.part[0], b.part[1], c);
    return mfma32(a.part[1], b.part[0], c);
}

// Queries: lane (half, i) has channels 16 t + 8 half .. + 7 of query i (t = 0 .. 3), x[8 t ..].
__device__ inline void f32_queries(const F32Window &w, int qtok, int half, float (&x)[32]) {
    const float *row = w.q + (long long)(qtok < 0 ? w.first : qtok) * w.qsn + 8 * half;
#pragma unroll
    for (int c = 0; c < 8; ++c) *(f32x4 *)(x + 4 * c) = *(const f32x4 *)(row + 16 * (c / 2) + 4 * (c % 2));
}
// Many queries: of a wavefront's 32 two parts are in registers and the third in LDS, 1 KB a step of 16 channels.
struct F32Queries {
    bf16x8 first[4], second[4];
    const unsigned char *third;  // this lane's
    __device__ void split(const float (&x)[32], unsigned char *rest) {
        third = rest;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const Split q = split8(x + 8 * t);
            first[t] = q.part[0];
            second[t] = q.part[1];
            *(u32x4 *)(rest + 1024 * t) = as_u32x4(q.part[2]);
        }
    }
    __device__ Split operator[](int t) const { return {first[t], second[t], as_bf16x8(*(const u32x4 *)(third + 1024 * t))}; }
};

// 32 queries of a wavefront: acc[cb][v] is channel 32 cb + 8 (v / 4) + 4 half + v % 4 of query lane % 32.
struct F32State {
    f32x16 acc[2];
    float m, ref, l;  // m: -inf until a key has a finite score; ref: what the weights are relative to, m or 0
    // (Sets of 16 registers stay sets: where the compiler sees single numbers put into them it carries 32 numbers round the key loop and copies
    // or spills them.)
    __device__ void whole() { asm("" : "+v"(acc[0]), "+v"(acc[1])); }
    __device__ void clear() {
        m = -INFINITY;
        ref = l = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
        whole();
    }
    __device__ void times(float x) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[0][v] *= x;
            acc[1][v] *= x;
        }
        whole();
    }
    // Scores -> weights relative to the reference, at most 2^8, summed into l.  The reference stays while no
    // logit is more than 8 binary orders above it (numerator and denominator share it, so the result is the
    // same), and goes up to the maximum otherwise.
    __device__ void weights(f32x16 &s, float factor) {
        float top = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) top = fmaxf(top, s[v]);
        if (__any(top * factor > m + 8.0f)) {
            float lo, hi;
            pair_values(top, &lo, &hi);
            const float m_new = fmaxf(m, fmaxf(lo, hi) * factor);
            ref = m_new == -INFINITY ? 0.f : m_new;  // padding only so far
            const float alpha = __builtin_amdgcn_exp2f(m - ref);
            m = m_new;
            l *= alpha;
            times(alpha);
        }
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], factor, -ref));
            sum += s[v];
        }
        l += sum;
    }
    // False where something is not finite.
    __device__ bool finite() const {
        float x[4] = {l, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v % 4] = fmaf(acc[0][v], 0.f, fmaf(acc[1][v], 0.f, x[v % 4]));
        return fabsf((x[0] + x[1]) + (x[2] + x[3])) < INFINITY;
    }
};

// Scores of a tile whose K rows (tile_off_row) start at `ktile`.
__device__ inline f32x16 f32_scores(const unsigned char *ktile, int li, int half, const F32Queries &q) {
    Split k[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) k[t] = split_load(ktile + tile_off_row(li, 2 * t + half), kPartTile);
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) s = mfma_small(k[t], q[t], s);
#pragma unroll
    for (int t = 0; t < 4; ++t) s = mfma32(k[t].part[0], q.first[t], s);
    return s;
}
// Byte offset of a lane's transposing reads in a tile of V (tile_off_tr), channel block cb.
__device__ inline unsigned f32_value_offset(int lane, int cb) {
    const int b = lane >> 4, j = lane & 15;
    return tile_off_tr(4 * (lane >> 5) + (j >> 2), cb * 4 + (b & 1) * 2 + ((j & 3) >> 1)) + (j & 1) * 8;
}
// acc += V^T P^T for the weights p of a tile.
__device__ inline void f32_values(F32State &st, const unsigned char *vtile, const unsigned (&voff)[2], const f32x16 &p) {
    Split w[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = p[8 * f + j];
        w[f] = split8(x);
    }
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        Split v[2];
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const unsigned char *at = vtile + voff[cb] + 16 * 128 * f + j * kPartTile;
                const u32x2 r0 = lds_read_tr16(at), r1 = lds_read_tr16(at + 1024);
                v[f].part[j] = as_bf16x8(u32x4{r0[0], r0[1], r1[0], r1[1]});
            }
        f32x16 sum;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[i] = 0.f;
        sum = mfma_small(v[1], w[1], mfma_small(v[0], w[0], sum));
        st.acc[cb] += mfma32(v[1].part[0], w[1].part[0], mfma32(v[0].part[0], w[0].part[0], sum));
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A wavefront's keys (tiles tile0, tile0 + step, ...) on the fp32 matrix instructions, straight from memory: half of the loads of a tile are in
// flight at a time.  With an infinity in V of every head (of one head) 1 369 tokens x 12 heads take 108 (91) us instead of 69, x 64 542 (307) instead of 205; the fp32
// instructions alone took 95 and 326.
__device__ inline void f32_again(F32State &st, const F32Window &w, int qtok, float scale_log2, int tile0, int step, int li, int half) {
    st.clear();
    float x[32];
    f32_queries(w, qtok, half, x);
#pragma clang loop unroll(disable)
    for (int k0 = 32 * tile0; k0 < w.g.slots; k0 += 32 * step) {
        const int ktok = w.token(k0 + li);
        const float *krow = w.k + (long long)(ktok < 0 ? w.first : ktok) * w.ksn + 8 * half;
        f32x4 k[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) k[c] = *(const f32x4 *)(krow + 16 * (c / 2) + 4 * (c % 2));
        float v[2][8];
        auto fetch_v = [&](int from) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int tok = __shfl(ktok, 8 * ((from + j) / 4) + 4 * half + j % 4, 64);
                const float *row = w.v + (long long)(tok < 0 ? w.first : tok) * w.vsn + li;
                v[0][j] = tok < 0 ? 0.f : row[0];  // (0 x inf would be NaN)
                v[1][j] = tok < 0 ? 0.f : row[32];
            }
        };
        fetch_v(0);
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(k[i / 4][i % 4], x[i], s, 0, 0, 0);
        const unsigned pad = (unsigned)__builtin_amdgcn_ballot_w64(ktok < 0) >> (4 * half);
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = (pad >> (8 * (i / 4) + i % 4)) & 1u ? -INFINITY : s[i];
        st.weights(s, scale_log2);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i == 8) {
                __builtin_amdgcn_sched_barrier(0);
                fetch_v(8);
            }
            const float p = s[i] * 0x1p-8f;  // none above 1: values up to the largest floats pass through the sums
            st.acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[0][i % 8], p, st.acc[0], 0, 0, 0);
            st.acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[1][i % 8], p, st.acc[1], 0, 0, 0);
        }
    }
    st.l *= 0x1p-8f;  // all of it relative to a reference 8 orders up
    st.m += 8.0f;
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
template <int KW>
__device__ inline void f32_merge(const F32Window &w, const unsigned char *parts, const float (&ms)[4][32], const float (&ls)[4][32],
                                 int qblock, int q_slots, int tid) {
    constexpr int QW = 4 / KW;
    const int chunk = tid & 15;
#pragma unroll
    for (int i = 0; i < 2 * QW; ++i) {
        const int query = (tid >> 4) + 16 * i, w0 = (query >> 5) * KW, ql = query & 31;
        const int slot = qblock * (32 * QW) + query;
        const int to = slot < q_slots ? w.token(slot) : -1;
        if (to < 0) continue;
        float top = ms[w0][ql];
#pragma unroll
        for (int k = 1; k < KW; ++k) top = fmaxf(top, ms[w0 + k][ql]);
        f32x4 out = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const float x = __builtin_amdgcn_exp2f(ms[w0 + k][ql] - top) * (1.0f / KW);  // (values up to the largest floats pass through the sum)
            out += x * *(const f32x4 *)(parts + (w0 + k) * (32 * 256) + ql * 256 + ((chunk ^ (ql & 15)) << 4));
            den = fmaf(x, ls[w0 + k][ql], den);
        }
        *(f32x4 *)(w.o + (long long)to * w.osn + 4 * chunk) = out * (1.0f / den);
    }
}

// Few tiles of keys: the same tiles on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32), whose operands are
// staged in LDS as they are.  With a tile or two to a wavefront the splits of the other kernels stand alone at its start.
// A workgroup of four wavefronts takes QW = 4 / KW blocks of 32 queries times KW groups of keys: per
// step it stages KW tiles of K and V in LDS (fetched into registers under the arithmetic of the
// step before) and wavefront (qw, kw) takes tile kw.  With KW > 1 the KW running softmaxes of a
// query block are merged through LDS at the end.
// grid (ceil(q_slots / (32 QW)), n_win, B*heads), 256 threads.
template <int KW>
__global__ void __launch_bounds__(256, 2)
attn_short_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads,
         float scale_log2, int q_slots) {
    constexpr int QW = 4 / KW, kF32Tile = 2 * 32 * kHeadDim * 4;  // K rows, then V rows, of 32 keys: 16 KB
    __shared__ __align__(16) unsigned char tiles[KW * kF32Tile];
    __shared__ __align__(16) float bias[KW * 32];  // 0 for a real key, -inf for padding
    __shared__ float ms[4][32], ls[4][32];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    const int kw = wave % KW, qw = wave / KW;
    int qblock, win, bh;
    f32_item(qblock, win, bh);
    const F32Window w = f32_window(qt, kt, vt, ot, g, heads, win, bh);
    const bool padded = (w.wy + 1) * g.wh > g.H || (w.wx + 1) * g.ww > g.W;

    // Queries: lane (half, li) holds channels 32 half .. +31 of query li.
    const int q0 = qblock * (32 * QW) + qw * 32;
    const bool live = q0 < q_slots;  // the same in the whole wavefront
    f32x4 q[8];
    int qtok = q0 + li < q_slots ? w.token(q0 + li) : -1;
    {
        const float *row = w.q + (long long)(qtok < 0 ? w.first : qtok) * w.qsn + 32 * half;
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
            int tok = w.token(step * (32 * KW) + srow + 16 * i);
            breg[i] = tok < 0 ? -INFINITY : 0.f;
            if (tok < 0) tok = w.first;
            kreg[i] = *(const f32x4 *)(w.k + (long long)tok * w.ksn + 4 * chunk);
            vreg[i] = *(const f32x4 *)(w.v + (long long)tok * w.vsn + 4 * chunk);
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
        if (qtok >= 0) f32_store_row(acc, 1.0f / l, w.o + (long long)qtok * w.osn + 4 * half);
        return;
    }
    __syncthreads();
    f32_park(acc, tiles + wave * (32 * 256), li, half);
    if (half == 0) {
        ms[wave][li] = m;
        ls[wave][li] = l;
    }
    __syncthreads();
    f32_merge<KW>(w, tiles, ms, ls, qblock, q_slots, tid);
}

// Many queries: a workgroup of four wavefronts takes 128 queries of a window.  Per step it splits a tile of K and V
// (fetched under the arithmetic of the step before) into LDS, where every wavefront reads it.  Bound by the issue of matrix (48 a tile,
// 1 536 cycles) and vector instructions (about 250), which overlap in part.  Measured: 2 304 tokens x 64
// heads 791 -> 512 us (fp32 matrix instructions / here), 1 369 x 64 328 -> 188, 784 x 64 118 -> 78, windows of 16 x 16 on 48 x 48 x 64
// 103 -> 73.  (All three parts of the queries in registers, which spill: 200 us for 1 369 x 64; two workgroups a unit, whose registers do not: 207.)
// grid (ceil(q_slots / 128), n_win, B*heads), 256 threads.
__global__ void __launch_bounds__(256, 3)
attn_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads, float scale_log2, int q_slots) {
    __shared__ __align__(16) unsigned char tile[6 * kPartTile];  // the three parts of K, then of V
    __shared__ __align__(16) unsigned char qrest[4][4 * 1024];   // the third parts of the queries
    __shared__ __align__(16) float bias[32];                     // 0 for a real key, -inf for padding
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    int qblock, win, bh;
    f32_item(qblock, win, bh);
    const F32Window w = f32_window(qt, kt, vt, ot, g, heads, win, bh);
    const bool padded = (w.wy + 1) * g.wh > g.H || (w.wx + 1) * g.ww > g.W;

    // Staging: this thread moves 16-byte chunk `chunk` of rows srow and srow + 16 of a tile.
    const int chunk = tid & 15, srow = tid >> 4;
    f32x4 kreg[2], vreg[2];
    float breg[2];
    auto fetch = [&](int step) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            int tok = w.token(32 * step + srow + 16 * i);
            breg[i] = tok < 0 ? -INFINITY : 0.f;
            if (tok < 0) tok = w.first;
            kreg[i] = *(const f32x4 *)(w.k + (long long)tok * w.ksn + 4 * chunk);
            vreg[i] = *(const f32x4 *)(w.v + (long long)tok * w.vsn + 4 * chunk);
        }
    };
    fetch(0);
    const int q0 = qblock * 128 + wave * 32;
    const bool live = q0 < q_slots;  // the same in the whole wavefront
    const int qtok = q0 + li < q_slots ? w.token(q0 + li) : -1;
    F32Queries q;
    {
        float x[32];
        f32_queries(w, qtok, half, x);
        q.split(x, qrest[wave] + 16 * lane);
    }
    F32State st;
    st.clear();
    const unsigned voff[2] = {f32_value_offset(lane, 0), f32_value_offset(lane, 1)};
    const int n_step = (g.slots + 31) / 32;
    for (int step = 0; step < n_step; ++step) {
        __syncthreads();  // the tile before has been read
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = srow + 16 * i;
            if (breg[i] != 0.f) kreg[i] = vreg[i] = f32x4{0.f, 0.f, 0.f, 0.f};  // 0 x inf of a padded key's row would be NaN
            split_store(tile + tile_off_row(r, chunk >> 1) + 8 * (chunk & 1), kreg[i]);
            split_store(tile + 3 * kPartTile + tile_off_tr(r, chunk >> 1) + 8 * (chunk & 1), vreg[i]);
            if (chunk == 0) bias[r] = breg[i];
        }
        __syncthreads();
        if (step + 1 < n_step) fetch(step + 1);
        if (!live) continue;
        f32x16 s = f32_scores(tile, li, half, q);
        if (padded || 32 * (step + 1) > g.slots) {  // (uniform) only here can a key be padding
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const f32x4 b = *(const f32x4 *)(bias + 8 * v4 + 4 * half);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[4 * v4 + e] += b[e];
            }
        }
        st.weights(s, scale_log2);
        f32_values(st, tile + 3 * kPartTile, voff, s);
    }
    if (!live) return;
    if (__any(!st.finite())) f32_again(st, w, qtok, scale_log2, 0, 1, li, half);
    if (qtok < 0) return;
    float lo, hi;
    pair_values(st.l, &lo, &hi);
    f32_store_row(st.acc, 1.0f / (lo + hi), w.o + (long long)qtok * w.osn + 4 * half);
}

// Few queries: a workgroup takes 32 of them and its four wavefronts every fourth tile of keys each, whose softmaxes are merged
// at the end.  They share queries and no keys, so K and V go straight into operand registers and the key loop has no barrier:
// a lane's K operands are 16-byte pieces of one row, a V operand eight dwords of a channel (an instruction reads two runs of 128
// bytes).  Half tiles of K and V rotate through three sets of sixteen registers, each
// fetched while the matrix instructions of two others run; three workgroups fit a compute unit.  Bound by its loads (32 cache lines for an
// instruction's K operands), the splits (280 vector instructions a tile) and the matrix instructions together.  Against the fp32 matrix
// instructions, us: 1 369 tokens x 12 heads 88.1 -> 62.9 (516 workgroups: four units have three and the others two; x 11 60.4 -> 45.8),
// 1 030 x 35 112 -> 82, windows of 14 x 14 on 40 x 40 x 12 22.4 -> 21.1.
// (Products added straight to the sums of the tiles before: 59.6 us for 1 369 x 12, but 3.5e-7 from 64 bits, and 5.4e-7 at 4 096 tokens.)
// grid (ceil(q_slots / 32), n_win, B*heads), 256 threads.  Byte offsets inside a (batch, head) slice of K and V below 2^32.
__global__ void __launch_bounds__(256, 3)
attn_few_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, WindowGeom g, int heads, float scale_log2, int q_slots) {
    __shared__ __align__(16) unsigned char parts[4][32 * 256];
    __shared__ __align__(16) unsigned char qs[3 * 4 * 1024];  // [part][step of 16 channels][lane]
    __shared__ float ms[4][32], ls[4][32];
    const int tid = threadIdx.x, kw = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    int qblock, win, bh;
    f32_item(qblock, win, bh);
    const F32Window w = f32_window(qt, kt, vt, ot, g, heads, win, bh);
    const char *kp = (const char *)w.k, *vp = (const char *)w.v;  // (uniform)
    const unsigned ksn = 4u * (unsigned)kt.sn, vsn = 4u * (unsigned)vt.sn;
    const unsigned vlane = 4u * half * vsn + 4u * li;
    const int qslot = qblock * 32 + li, qtok = qslot < q_slots ? w.token(qslot) : -1;
    {
        float x[32];
        f32_queries(w, qtok, half, x);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t != kw) continue;  // (uniform; constant indices of x)
            const Split q = split8(x + 8 * t);
#pragma unroll
            for (int j = 0; j < 3; ++j) *(u32x4 *)(qs + (4 * j + t) * 1024 + lane * 16) = as_u32x4(q.part[j]);
        }
    }
    F32State st;
    st.clear();
    const int n_tile = (g.slots + 31) / 32;
    f32x4 set[3][4];
    // K operands of steps 2 hf, 2 hf + 1 of the tile whose key li is token `tok` (negative: padding)
    auto fetch_k = [&](f32x4 (&r)[4], int tok, int hf) __attribute__((always_inline)) {
        const unsigned at = (unsigned)(tok < 0 ? w.first : tok) * ksn + 32u * half;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = *(const f32x4 *)(kp + at + 128 * hf + 64 * (i / 2) + 16 * (i % 2));
    };
    // element 8 cb + j: channel 32 cb + li of key 16 hf + 8 (j / 4) + 4 half + j % 4
    auto fetch_v = [&](f32x4 (&r)[4], int tok, unsigned pad, int hf) __attribute__((always_inline)) {
        if (w.rows && pad == 0u) {
            const char *row = vp + (unsigned)(__builtin_amdgcn_readfirstlane(tok) + 16 * hf) * (size_t)vsn;
            unsigned at = vlane;
            asm volatile("" : "+v"(at));  // (a 32-bit offset to a scalar base: widened ahead of the loop it would be added in vector registers)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                r[j / 4][j % 4] = *(const float *)(row + at);
                r[2 + j / 4][j % 4] = *(const float *)(row + at + 128);
                row += (j == 3 ? 5 : 1) * (size_t)vsn;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int t = __shfl(tok, 16 * hf + 8 * (j / 4) + 4 * half + j % 4, 64);
                const unsigned at = (unsigned)(t < 0 ? w.first : t) * vsn + 4u * li;
                r[j / 4][j % 4] = *(const float *)(vp + at);
                r[2 + j / 4][j % 4] = *(const float *)(vp + at + 128);
            }
            // (keeps the two branches' loads apart: merged into one set they would take every address
            // in a vector register of its own)
            asm volatile("");
        }
    };
    auto real_token = [&](int tile, int &tok, unsigned &pad) __attribute__((always_inline)) {
        tok = w.token(32 * tile + li);
        pad = (unsigned)__builtin_amdgcn_ballot_w64(tok < 0);  // bit j: key j of the tile is padding
    };
    int tok = 0;
    unsigned pad = 0u;
    // A tile whose K operands are in (or on their way to) ka and kb; leaves those of the next in kb and vc.
    auto run_tile = [&](int tile, f32x4 (&ka)[4], f32x4 (&kb)[4], f32x4 (&vc)[4]) __attribute__((always_inline)) {
        const int cur = tok;
        const unsigned cur_pad = pad, pads = half ? pad >> 4 : pad;
        f32x16 s;
        auto scores = [&](f32x4 (&r)[4], int hf) __attribute__((always_inline)) {
            bf16x8 q0[2], k0[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const Split q = split_load(qs + (2 * hf + t) * 1024 + lane * 16, 4096), k = split8((const float *)&r[2 * t]);
                s = mfma_small(k, q, s);
                q0[t] = q.part[0];
                k0[t] = k.part[0];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) s = mfma32(k0[t], q0[t], s);
        };
        fetch_v(vc, cur, cur_pad, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
        scores(ka, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_v(ka, cur, cur_pad, 1);
        if (tile + 4 < n_tile) real_token(tile + 4, tok, pad);
        __builtin_amdgcn_sched_barrier(0);
        scores(kb, 1);
        __builtin_amdgcn_sched_barrier(0);
        fetch_k(kb, tok, 0);  // (behind the last tile its own keys again: loads behind a branch would be waited for all at once)
        __builtin_amdgcn_sched_barrier(0);
        if (cur_pad != 0u) {  // (uniform) padded keys have no weight ...
#pragma unroll
            for (int j = 0; j < 16; ++j) s[j] = (pads >> (8 * (j / 4) + j % 4)) & 1u ? -INFINITY : s[j];
        }
        st.weights(s, scale_log2);
        auto product = [&](f32x4 (&r)[4], int hf) __attribute__((always_inline)) {
            if (cur_pad != 0u) {  // ... and zeros for the values they meet (0 x inf would be NaN)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool x = (pads >> (16 * hf + 8 * (j / 4) + j % 4)) & 1u;
                    r[j / 4][j % 4] = x ? 0.f : r[j / 4][j % 4];
                    r[2 + j / 4][j % 4] = x ? 0.f : r[2 + j / 4][j % 4];
                }
            }
            float p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = s[8 * hf + j];
            const Split x = split8(p);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const Split v = split8((const float *)&r[2 * cb]);
                f32x16 sum;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[i] = 0.f;
                st.acc[cb] += mfma32(v.part[0], x.part[0], mfma_small(v, x, sum));
            }
        };
        product(vc, 0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_k(vc, tok, 1);
        __builtin_amdgcn_sched_barrier(0);
        product(ka, 1);
    };
    __syncthreads();  // the queries
    if (kw < n_tile) {
        real_token(kw, tok, pad);
        fetch_k(set[0], tok, 0);
        fetch_k(set[1], tok, 1);
        for (int tile = kw;;) {
            run_tile(tile, set[0], set[1], set[2]);
            if ((tile += 4) >= n_tile) break;
            run_tile(tile, set[1], set[2], set[0]);
            if ((tile += 4) >= n_tile) break;
            run_tile(tile, set[2], set[0], set[1]);
            if ((tile += 4) >= n_tile) break;
        }
    }
    if (__any(!st.finite())) f32_again(st, w, qtok, scale_log2, kw, 4, li, half);
    f32_park(st.acc, parts[kw], li, half);
    {
        float lo, hi;
        pair_values(st.l, &lo, &hi);
        if (half == 0) {
            ms[kw][li] = st.m;
            ls[kw][li] = lo + hi;
        }
    }
    __syncthreads();
    f32_merge<4>(w, &parts[0][0], ms, ls, qblock, q_slots, tid);
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
    const int tiles = (g.slots + 31) / 32;
    const long long lanes = (long long)g.n_win * pr.B * pr.heads, max_sn = pr.k.sn > pr.v.sn ? pr.k.sn : pr.v.sn;
    const F32Kernel kernel = f32_kernel(tiles, g.ww == g.W, q_slots, lanes, ((long long)g.H * g.W + 64) * max_sn * 4);
    const int queries = kernel == kF32Many || kernel == kF32Short1 ? 128 : kernel == kF32Short2 ? 64 : 32;
    const auto f = kernel == kF32Many ? attn_f32 : kernel == kF32Few ? attn_few_f32 : kernel == kF32Short1 ? attn_short_f32<1> :
                   kernel == kF32Short2 ? attn_short_f32<2> : attn_short_f32<4>;
    hipLaunchKernelGGL(f, dim3((unsigned)((q_slots + queries - 1) / queries), g.n_win, pr.B * pr.heads), dim3(256), 0, stream,
                       pr.q, pr.k, pr.v, pr.o, g, pr.heads, scale * 1.4426950408889634f, q_slots);
    return launch_status("fp32 attention");
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
