// Linear attention (Eq. 2 of the paper, key-sum normaliser; phi = ReLU unless the focused map
// of Eq. 3 is asked for):
//   pass 1  la_state_*  : S_p = sum_j relu(k_j)^T v_j, z_p = sum_j relu(k_j) over one token chunk
//   pass 2  la_apply_*  : S = sum_p S_p, z = sum_p z_p;  o_i = relu(q_i) S / (relu(q_i).z + eps)
//
// Workspace layout (fp32): partial p of (batch b, head h) starts at
//   ((p * B*heads) + b*heads + h) * kStateFloats
// and holds S transposed, St[c2][c1] (c2 = value channel, c1 = key channel), then z[c1].
#include "jv_linear.h"
#include "jv_mfma.h"
#include "jv_plan.h"

namespace jv {

LinearPlan plan_linear(int B, int heads, int N, bool bf16) {
    LinearPlan p;
    const long long bh = (long long)B * heads;
    if (!bf16) {
        // Chunks of at least 64 tokens (16 per wavefront, one round of loads in the state pass), down
        // to which a problem is cut until it has two workgroups per compute unit.  Up to eight
        // partial states are summed by every workgroup of the apply pass for itself, up to 64 in a
        // pass of their own: that pays where eight chunks of up to 16 heads leave half of the chip idle for
        // long.  Eight states / up to 64, us: 6 heads of 4 096 tokens 22.7 / 24.5, of 6 144 32.5 / 28.7, of
        // 16 384 66 / 46, of 262 144 783 / 388; 16 heads of 8 192 48.3 / 46.9, 24 of 8 192 62 / 70.
        long long want = (512 + bh - 1) / bh, most = (N + 63) / 64;
        want = want > most ? most : want;
        want = want > 64 ? 64 : want;
        if (want > 8 && (N <= 4096 || bh > 16)) want = 8;
        p.chunk = (int)((((N + want - 1) / want + 63) / 64) * 64);
        p.n_split = (N + p.chunk - 1) / p.chunk;
        p.apply_tokens = 1024;
        while (p.apply_tokens > 128 && bh * ((N + p.apply_tokens - 1) / p.apply_tokens) < 512) p.apply_tokens /= 2;
        p.combine = p.n_split > 8;
        return p;
    }
    // Aim for about two workgroups per compute unit, chunks of at least 256 tokens.
    long long want = (512 + bh - 1) / bh;
    long long max_split = (N + 255) / 256;
    if (want > max_split) want = max_split;
    if (want < 1) want = 1;
    if (want > 64) want = 64;
    long long chunk = (N + want - 1) / want;
    chunk = ((chunk + 255) / 256) * 256;
    p.chunk = (int)chunk;
    p.n_split = (int)((N + chunk - 1) / chunk);
    p.apply_tokens = 256 * apply_rounds(bh, N);
    p.combine = p.n_split > 4;
    return p;
}

size_t linear_workspace_floats(const LinearPlan &p, int B, int heads) {
    return (size_t)(p.n_split + (p.combine ? 1 : 0)) * B * heads * kStateFloats;
}

// ---------------------------------------------------------------------------------------
// fp32 path: both passes on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32: operand lane
// (half, i) holds row or column i at contraction index `half`; fp32 throughout), whose rate
// would stream the tensors at 9.8 TB/s, so problems that fill the chip are bound by memory and small ones,
// where both passes are one launch, by latency.
// ---------------------------------------------------------------------------------------

// Focused feature map (Eq. 3; see focus_bf16x8 in the bf16 path) of a rectified row given the
// largest entry `top` of the row: x <- x^p as a fraction of top; the caller scales the row by
// top * sqrt(sum (x / top)^2 / sum (x / top)^2p).
__device__ inline float focus_power(float x, int p, float &ss, float &sy) {
    float y = x;
    for (int i = 1; i < p; ++i) y *= x;
    ss = fmaf(x, x, ss);
    sy = fmaf(y, y, sy);
    return y;
}

// State pass.  Wavefront w of a workgroup takes every fourth group of 16 tokens of the chunk.
// The contraction runs over tokens and both operands are channels of one token, so a lane's
// operand is one element of a K or V row straight from global memory (two rows of 128
// contiguous bytes per load instruction): no staging.  St = V^T relu(K) in four 32 x 32 blocks.
// Measured: 256 tokens x 6 heads 4.5 us (plain FMAs, one workgroup per head: 30 us).
// grid (n_split, B*heads), 256 threads.
__global__ void __launch_bounds__(256, 2)
la_state_f32(TensorArg kt, TensorArg vt, float *__restrict__ ws, int heads, int N, int chunk,
             int focus_p) {
    __shared__ __align__(16) float part[4][kHeadDim * kHeadDim];
    __shared__ float zpart[4][kHeadDim];
    const int bh = blockIdx.y, b = bh / heads, h = bh % heads, p = blockIdx.x;
    const int BH = gridDim.y;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    const float *kp = (const float *)kt.ptr + b * kt.sb + h * kt.sh + li;
    const float *vp = (const float *)vt.ptr + b * vt.sb + h * vt.sh + li;
    f32x16 acc[2][2];  // [value block][key block]
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][0][v] = acc[0][1][v] = acc[1][0][v] = acc[1][1][v] = 0.f;
    float z[2] = {0.f, 0.f};
    const int n0 = p * chunk, n1 = min(N, n0 + chunk);
    float k[8][2], v[8][2], knext[8][2], vnext[8][2];
    // Rows are walked with a running pointer per lane: a 64-bit multiplication per row costs more
    // than the products.
    auto fetch = [&](int base) {
        const float *kr = kp + (long long)(base + half) * kt.sn, *vr = vp + (long long)(base + half) * vt.sn;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            knext[u][0] = kr[0]; knext[u][1] = kr[32];
            vnext[u][0] = vr[0]; vnext[u][1] = vr[32];
            kr += 2 * kt.sn;
            vr += 2 * vt.sn;
        }
    };
    auto reduce = [&]() {
        if (focus_p > 1) {  // uniform; a token's row lies in the 32 lanes of one half
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float top = fmaxf(k[u][0], k[u][1]);
#pragma unroll
                for (int off = 16; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off, 64));
                const float inv_top = top > 0.f ? 1.0f / top : 0.f;
                float ss = 0.f, sy = 0.f;
#pragma unroll
                for (int c = 0; c < 2; ++c) k[u][c] = focus_power(k[u][c] * inv_top, focus_p, ss, sy);
#pragma unroll
                for (int off = 16; off > 0; off >>= 1) {
                    ss += __shfl_xor(ss, off, 64);
                    sy += __shfl_xor(sy, off, 64);
                }
                const float scale = top > 0.f ? top * sqrtf(ss / sy) : 0.f;
#pragma unroll
                for (int c = 0; c < 2; ++c) k[u][c] *= scale;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            z[0] += k[u][0];
            z[1] += k[u][1];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[u][i], k[u][j], acc[i][j], 0, 0, 0);
        }
    };
    int base = n0 + 16 * wave;
    bool whole = base + 16 <= n1;
    if (whole) fetch(base);
    while (whole) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                k[u][c] = fmaxf(knext[u][c], 0.f);
                v[u][c] = vnext[u][c];
            }
        base += 64;
        whole = base + 16 <= n1;
        if (whole) fetch(base);  // the next group's rows, in flight under this group's products
        reduce();
    }
    if (base < n1) {  // the last group of the chunk, with fewer than 16 tokens
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int n = base + 2 * u + half;
            k[u][0] = k[u][1] = v[u][0] = v[u][1] = 0.f;
            if (n < n1) {
                const float *kr = kp + (long long)n * kt.sn, *vr = vp + (long long)n * vt.sn;
                k[u][0] = fmaxf(kr[0], 0.f); k[u][1] = fmaxf(kr[32], 0.f);
                v[u][0] = vr[0]; v[u][1] = vr[32];
            }
        }
        reduce();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                part[wave][(32 * i + 8 * (v / 4) + 4 * half + v % 4) * kHeadDim + 32 * j + li] = acc[i][j][v];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        z[j] += __shfl_xor(z[j], 32, 64);
        if (half == 0) zpart[wave][32 * j + li] = z[j];
    }
    __syncthreads();
    float *out = ws + ((size_t)p * BH + bh) * kStateFloats;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = 4 * (tid + 256 * i);
        *(f32x4 *)(out + e) = (*(const f32x4 *)&part[0][e] + *(const f32x4 *)&part[1][e]) +
                              (*(const f32x4 *)&part[2][e] + *(const f32x4 *)&part[3][e]);
    }
    if (tid < kHeadDim)
        out[kHeadDim * kHeadDim + tid] = (zpart[0][tid] + zpart[1][tid]) + (zpart[2][tid] + zpart[3][tid]);
}

// Apply pass.  The workgroup sums the partial states into LDS; every wavefront keeps all of St
// (and z) as operands in registers and walks over tiles of 32 tokens: O^T = St relu(Q)^T with
// lane (half, i) holding channels 32 half .. +31 of token i, so the denominator is 32 FMAs per
// lane and one exchange.  Query and output rows pass through LDS: global memory sees whole rows.
// Measured: 256 tokens x 6 heads 6.6 us (plain FMAs, one workgroup per head: 58 us).
// grid (ceil(N / tokens), B*heads), 256 threads; tokens is a multiple of 128.
__global__ void __launch_bounds__(256, 2)
la_apply_f32(TensorArg qt, TensorArg ot, const float *__restrict__ ws, int heads, int N,
             int n_split, int tokens, float eps, int focus_p) {
    // 16-byte chunks of a row are rotated by the row: row-per-lane accesses without bank conflicts
    __shared__ __align__(16) unsigned char St[kHeadDim * 256];
    __shared__ __align__(16) float z[kHeadDim];
    __shared__ __align__(16) unsigned char stage[4][32 * 256];
    const int bh = blockIdx.y, b = bh / heads, h = bh % heads;
    const int BH = gridDim.y;
    const float *qp = (const float *)qt.ptr + b * qt.sb + h * qt.sh;
    float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, li = lane & 31;
    const int n1 = min(N, (int)(blockIdx.x + 1) * tokens);
    const int srow = lane >> 4, chunk = lane & 15;  // row layout of a tile: 4 rows per instruction
    f32x4 q[8], next[8];
    auto fetch = [&](int base) {
        if (base + 32 <= n1) {
            const float *row = qp + (long long)(base + srow) * qt.sn + 4 * chunk;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                next[r] = *(const f32x4 *)row;
                row += 4 * qt.sn;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                next[r] = *(const f32x4 *)(qp + (long long)min(base + 4 * r + srow, n1 - 1) * qt.sn + 4 * chunk);
        }
    };
    int base = blockIdx.x * tokens + 32 * wave;
    fetch(base);
    // St and z as 1040 16-byte pieces, five per thread (the fifth for the first 16 threads); the
    // partials of four pieces and four chunks at a time, so that the sum is not a chain of round trips
    {
        const float *src = ws + (size_t)bh * kStateFloats;
        f32x4 s[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) s[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int p0 = 0; p0 < n_split; p0 += 4) {
#pragma unroll
            for (int dp = 0; dp < 4; ++dp) {
                const float *part = src + (size_t)min(p0 + dp, n_split - 1) * BH * kStateFloats;
                const bool live = p0 + dp < n_split;
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const f32x4 x = *(const f32x4 *)(part + 4 * min(tid + 256 * i, kStateFloats / 4 - 1));
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[i][e] += live ? x[e] : 0.f;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const int e = tid + 256 * i, row = e >> 4, c = e & 15;
            if (row < kHeadDim) *(f32x4 *)(St + row * 256 + ((c ^ (row & 15)) << 4)) = s[i];
            else if (row == kHeadDim) *(f32x4 *)(z + 4 * c) = s[i];
        }
    }
    __syncthreads();
    f32x4 sreg[2][8], zreg[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
            sreg[cb][i] = *(const f32x4 *)(St + (32 * cb + li) * 256 + (((8 * half + i) ^ (li & 15)) << 4));
        zreg[i] = *(const f32x4 *)(z + 32 * half + 4 * i);
    }
    unsigned char *mine = stage[wave];
    for (; base < n1; base += 128) {
        // query rows -> LDS -> 32 channels of one token per lane (the buffer is this wavefront's own)
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int row = 4 * r + srow;
            *(f32x4 *)(mine + row * 256 + ((chunk ^ (row & 15)) << 4)) = next[r];
        }
        if (base + 128 < n1) fetch(base + 128);
        f32x4 top4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            q[i] = *(const f32x4 *)(mine + li * 256 + (((8 * half + i) ^ (li & 15)) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[i][e] = fmaxf(q[i][e], 0.f);
                top4[e] = fmaxf(top4[e], q[i][e]);
            }
        }
        float lo, hi;
        if (focus_p > 1) {  // uniform; a token's row lies in lanes li and li + 32
            pair_values(fmaxf(fmaxf(top4[0], top4[1]), fmaxf(top4[2], top4[3])), &lo, &hi);
            const float top = fmaxf(lo, hi), inv_top = top > 0.f ? 1.0f / top : 0.f;
            float ss = 0.f, sy = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) q[i][e] = focus_power(q[i][e] * inv_top, focus_p, ss, sy);
            pair_values(ss, &lo, &hi);
            ss = lo + hi;
            pair_values(sy, &lo, &hi);
            sy = lo + hi;
            const float scale = top > 0.f ? top * sqrtf(ss / sy) : 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] *= scale;
        }
        f32x4 den4 = {0.f, 0.f, 0.f, 0.f};
        f32x16 acc[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                den4[e] = fmaf(q[i][e], zreg[i][e], den4[e]);
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                    acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(sreg[cb][i][e], q[i][e], acc[cb], 0, 0, 0);
            }
        pair_values((den4[0] + den4[1]) + (den4[2] + den4[3]), &lo, &hi);
        // Below 2^-128 (eps 0, small queries and keys) 1 / den overflows where the quotient need not:
        // small denominators and their numerators first take a factor 2^60.  (32 divisions instead,
        // 256 tokens x 6 heads: 10.8 against 10.2 us a call.)
        float den = (lo + hi) + eps;
        if (__any(den < 0x1p-100f)) {
            const float up = den < 0x1p-100f ? 0x1p60f : 1.0f;
            den *= up;
            acc[0] *= up;
            acc[1] *= up;
        }
        const float inv = 1.0f / den;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                f32x4 out;
#pragma unroll
                for (int e = 0; e < 4; ++e) out[e] = acc[cb][4 * v4 + e] * inv;
                *(f32x4 *)(mine + li * 256 + (((8 * cb + 2 * v4 + half) ^ (li & 15)) << 4)) = out;
            }
        float *orow = op + (long long)(base + srow) * ot.sn + 4 * chunk;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int row = 4 * r + srow;
            const f32x4 out = *(const f32x4 *)(mine + row * 256 + ((chunk ^ (row & 15)) << 4));
            if (base + row < n1) *(f32x4 *)orow = out;
            orow += 4 * ot.sn;
        }
    }
}

// Both passes in one launch, for few tokens: a workgroup forms sixteen value channels of a (batch, head)'s
// state from all of its tokens, and applies them to a part of its queries, so that no workgroup waits for another's
// sums.  Bound by round trips to memory and by the matrix instructions of one unit (0.9 us per pass and 256 tokens): two launches
// make two round trips more, and here K, V and the first queries of eight wavefronts are all in flight at once.  K and V
// are read by four workgroups for every part of the queries, which run on one XCD and share its L2.  Tiles of 16 x 16 x 4
// (v_mfma_f32_16x16x4_f32: lane (g, i) holds row or column i at contraction index g), in two chains of sums: 256 tokens
// x 6 heads 9.9 -> 5.5 us in two launches / here, 8.5e-8 from 64 bits (1.08e-7 before).  One part of the queries
// instead of eight 7.1 us, sixteen wavefronts a workgroup 9.6 (registers spill).
// grid (32 ceil(B*heads / 8), ceil(tiles of 16 tokens / apply_tiles)), 512 threads.
constexpr int kFusedWaves = 8;
__global__ void __launch_bounds__(64 * kFusedWaves)
la_fused_f32(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, int heads, int BH, int N, int apply_tiles, float eps) {
    __shared__ __align__(16) float part[kFusedWaves][16 * kHeadDim + kHeadDim];  // 16 rows of St, then z
    // 16-byte chunks of a row are rotated by the row: row-per-lane reads without bank conflicts
    __shared__ __align__(16) unsigned char St[16 * 256];
    __shared__ __align__(16) float z[kHeadDim];
    const int bh = (int)(blockIdx.x >> 5) * 8 + (int)(blockIdx.x & 7), c0 = 16 * (int)((blockIdx.x >> 3) & 3);
    if (bh >= BH) return;  // (the whole workgroup)
    const int b = bh / heads, h = bh % heads;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 4, li = lane & 15;
    const float *kp = (const float *)kt.ptr + b * kt.sb + h * kt.sh + 4 * li;
    const float *vp = (const float *)vt.ptr + b * vt.sb + h * vt.sh + c0 + li;
    const float *qp = (const float *)qt.ptr + b * qt.sb + h * qt.sh + 4 * g;
    float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh + c0 + 4 * g;

    // State: wavefront w takes every eighth group of 32 tokens.  Lane (g, i) has tokens 4 u + g: channels 4 i .. + 3 of K
    // (column i of key block e is channel 4 i + e) and channel c0 + i of V.
    f32x4 k[8];
    float v[8];
    auto fetch_kv = [&](int base) __attribute__((always_inline)) {
        const float *kr = kp + (long long)(base + g) * kt.sn, *vr = vp + (long long)(base + g) * vt.sn;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool real = base + 4 * u + g < N;
            k[u] = *(const f32x4 *)(real ? kr : kp);
            v[u] = *(real ? vr : vp);
            kr += 4 * kt.sn;
            vr += 4 * vt.sn;
        }
    };
    // Queries: tiles of 16 tokens, lane (g, i) has channels 16 u + 4 g .. + 3 of token i
    f32x4 q[2][4];
    auto fetch_q = [&](f32x4 (&r)[4], int tile) __attribute__((always_inline)) {
        const float *row = qp + (long long)min(16 * tile + li, N - 1) * qt.sn;
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = *(const f32x4 *)(row + 16 * u);
    };
    const int tile0 = (int)blockIdx.y * apply_tiles, n_tile = min((N + 15) / 16, tile0 + apply_tiles);
    int base = 32 * wave;
    if (base < N) fetch_kv(base);
    if (tile0 + wave < n_tile) fetch_q(q[0], tile0 + wave);
    if (tile0 + wave + kFusedWaves < n_tile) fetch_q(q[1], tile0 + wave + kFusedWaves);
    f32x4 acc[2][4], zsum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[0][e] = acc[1][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    while (base < N) {
        f32x4 kr[8];
        float vr[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool real = base + 4 * u + g < N;
            vr[u] = real ? v[u] : 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) kr[u][e] = real ? fmaxf(k[u][e], 0.f) : 0.f;
        }
        base += 32 * kFusedWaves;
        if (base < N) fetch_kv(base);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            zsum += kr[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[u & 1][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[u], kr[u][e], acc[u & 1][e], 0, 0, 0);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[0][e] += acc[1][e];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *(f32x4 *)(part[wave] + (4 * g + r) * kHeadDim + 4 * li) = f32x4{acc[0][0][r], acc[0][1][r], acc[0][2][r], acc[0][3][r]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        zsum[e] += __shfl_xor(zsum[e], 16, 64);
        zsum[e] += __shfl_xor(zsum[e], 32, 64);
    }
    if (g == 0) *(f32x4 *)(part[wave] + 16 * kHeadDim + 4 * li) = zsum;
    __syncthreads();
    if (tid < 17 * 16) {
        f32x4 s[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) s[w] = *(const f32x4 *)(part[w] + 4 * tid) + *(const f32x4 *)(part[w + 4] + 4 * tid);
        const f32x4 sum = (s[0] + s[1]) + (s[2] + s[3]);
        const int row = tid >> 4, c = tid & 15;
        if (row < 16) *(f32x4 *)(St + row * 256 + ((c ^ row) << 4)) = sum;
        else *(f32x4 *)(z + 4 * c) = sum;
    }
    __syncthreads();
    f32x4 sreg[4], zreg[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        sreg[u] = *(const f32x4 *)(St + li * 256 + (((4 * u + g) ^ li) << 4));
        zreg[u] = *(const f32x4 *)(z + 16 * u + 4 * g);
    }
    auto apply = [&](f32x4 (&r)[4], int tile) __attribute__((always_inline)) {
        f32x4 out[2], den4 = {0.f, 0.f, 0.f, 0.f};
        out[0] = out[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = fmaxf(r[u][e], 0.f);
                den4[e] = fmaf(x, zreg[u][e], den4[e]);
                out[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(sreg[u][e], x, out[e & 1], 0, 0, 0);
            }
        if (tile + 2 * kFusedWaves < n_tile) fetch_q(r, tile + 2 * kFusedWaves);
        float den = (den4[0] + den4[1]) + (den4[2] + den4[3]);
        den += __shfl_xor(den, 16, 64);
        den += __shfl_xor(den, 32, 64);
        den += eps;
        const float up = den < 0x1p-100f ? 0x1p60f : 1.0f;  // (as in la_apply_f32)
        const float inv = 1.0f / (den * up);
        const int n = 16 * tile + li;
        if (n < N) *(f32x4 *)(op + (long long)n * ot.sn) = ((out[0] + out[1]) * up) * inv;
    };
    for (int tile = tile0 + wave; tile < n_tile; tile += 2 * kFusedWaves) {
        apply(q[0], tile);
        if (tile + kFusedWaves < n_tile) apply(q[1], tile + kFusedWaves);
    }
}

size_t linear_workspace_bytes(int B, int heads, int N, bool bf16) {
    return linear_workspace_floats(plan_linear(B, heads, N, bf16), B, heads) * sizeof(float);
}

static jv_status linear_f32(const Problem &pr, const LinearPlan &plan, float eps, float *ws, int focus_p, hipStream_t stream) {
    const int BH = pr.B * pr.heads;
    if (focus_p == 1 && linear_f32_in_one(BH, pr.N)) {
        const int tiles = (pr.N + 15) / 16, parts = linear_f32_parts(BH), apply_tiles = (tiles + parts - 1) / parts;
        hipLaunchKernelGGL(la_fused_f32, dim3(32 * ((BH + 7) / 8), (tiles + apply_tiles - 1) / apply_tiles), dim3(64 * kFusedWaves), 0, stream,
                           pr.q, pr.k, pr.v, pr.o, pr.heads, BH, pr.N, apply_tiles, eps);
        return launch_status("la_fused_f32");
    }
    hipLaunchKernelGGL(la_state_f32, dim3(plan.n_split, BH), dim3(256), 0, stream, pr.k, pr.v, ws,
                       pr.heads, pr.N, plan.chunk, focus_p);
    jv_status st = launch_status("la_state_f32");
    if (st != JV_OK) return st;
    const float *states = ws;
    if (plan.combine) {
        float *sum = ws + (size_t)plan.n_split * BH * kStateFloats;
        if ((st = combine_states(ws, sum, nullptr, plan.n_split, BH, stream)) != JV_OK) return st;
        states = sum;
    }
    hipLaunchKernelGGL(la_apply_f32, dim3((pr.N + plan.apply_tokens - 1) / plan.apply_tokens, BH), dim3(256), 0, stream,
                       pr.q, pr.o, states, pr.heads, pr.N, plan.combine ? 1 : plan.n_split, plan.apply_tokens, eps, focus_p);
    return launch_status("la_apply_f32");
}

// The block of Eq. 4.  Order of launches: state pass (which also sums V over the tokens when
// the filters are generated from it), optional combine, filter generator, apply pass (bf16:
// the convolution is fused into it; fp32: a pass of its own adds it).
jv_status linear_block_forward(const Problem &pr, float eps, const jv_dwc_params *dwc,
                               void *workspace, size_t workspace_bytes, hipStream_t stream,
                               int focus_p) {
    if (focus_p < 1 || focus_p > 16) return fail(JV_ERR_INVALID_ARG, "focusing power must be 1 .. 16");
    if (pr.D == kHeadDimWide) {
        if (focus_p != 1) return fail(JV_ERR_UNSUPPORTED, "head_dim 128: the focused map is built for 64-channel heads");
        DwcPlan cv;
        jv_status st = plan_dwc_wide(dwc, linear_wide_workspace_floats(pr.B, pr.heads, pr.N), pr.B, pr.heads, pr.N, &cv);
        if (st != JV_OK) return st;
        const size_t need = cv.total_floats * sizeof(float);
        if (workspace_bytes < need)
            return fail(JV_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes, need);
        float *ws = (float *)workspace;
        if (cv.mode == JV_DWC_NONE) return linear_wide_bf16(pr, eps, ws, stream);
        float *vsum = cv.mode == JV_DWC_SQUEEZE_DYNAMIC ? ws + cv.vsum_off : nullptr;
        if ((st = linear_wide_state(pr, ws, vsum, stream)) != JV_OK) return st;
        DwcArg arg;
        if ((st = dwc_wide_filters(pr, cv, ws, stream, &arg)) != JV_OK) return st;
        return linear_wide_apply(pr, eps, ws, stream, cv.ksize, &arg);
    }
    const LinearPlan plan = plan_linear(pr.B, pr.heads, pr.N, pr.bf16);
    DwcPlan cv;
    jv_status st = plan_dwc(dwc, plan, pr.B, pr.heads, pr.N, &cv);
    if (st != JV_OK) return st;
    if (workspace_bytes < cv.total_floats * sizeof(float))
        return fail(JV_ERR_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, %zu needed", workspace_bytes,
                    cv.total_floats * sizeof(float));
    float *ws = (float *)workspace;
    if (cv.mode == JV_DWC_TOKEN_DYNAMIC) {
        // Plain linear attention into an fp32 tensor (O itself when it is fp32), then one pass
        // that adds every token's own convolution term and rounds once.
        if (!pr.bf16) {  // fp32 tensors: the two passes, then the convolution added in place
            if ((st = linear_f32(pr, plan, eps, ws, focus_p, stream)) != JV_OK) return st;
            return token_dwc_forward_f32(pr, cv, ws, stream);
        }
        Problem la = pr;
        if (pr.o_bf16) {
            const long long C = (long long)pr.heads * kHeadDim;
            la.o = {ws + cv.la_off, (long long)pr.N * C, kHeadDim, C};
            la.o_bf16 = false;
        }
        DwcPlan none = cv;
        none.mode = JV_DWC_NONE;
        if ((st = linear_bf16(la, plan, eps, ws, none, focus_p, stream)) != JV_OK) return st;
        return token_dwc_forward(pr, la.o, cv, ws, stream);
    }
    if (pr.bf16) return linear_bf16(pr, plan, eps, ws, cv, focus_p, stream);
    if ((st = linear_f32(pr, plan, eps, ws, focus_p, stream)) != JV_OK) return st;
    if (cv.mode == JV_DWC_NONE) return JV_OK;
    DwcArg arg = {cv.static_kernel, 0, pr.H, pr.W, pr.P};
    if (cv.mode == JV_DWC_SQUEEZE_DYNAMIC) {
        if ((st = vsum_f32_launch(pr, plan, ws + cv.vsum_off, stream)) != JV_OK) return st;
        if ((st = squeeze_generate(cv, ws, plan.n_split, pr.B, pr.heads, pr.N, stream)) != JV_OK) return st;
        arg.kappa = ws + cv.kappa_off;
        arg.kappa_sb = (long long)pr.heads * kHeadDim * cv.ksize * cv.ksize;
    }
    return dwc_add_f32_launch(pr, arg, cv.ksize, stream);
}

}  // namespace jv

// ---------------------------------------------------------------------------------------
// Scratch of the allocation-free entry point (jv_linear_attn_fwd_static): the partial and
// combined linear-attention states live in a fixed array in device memory that belongs to the
// library's code object -- one copy per GPU, at its own address on each, held until the
// process ends.  In host code the array's name is only a handle for the symbol lookup below;
// what the kernels get is the device address that lookup returns.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char jv_static_scratch[JV_STATIC_SCRATCH_BYTES];

namespace jv {
// Device address of jv_static_scratch on the current device, looked up once per device.
static jv_status static_scratch_address(void **out) {
    constexpr int kMaxDevices = 64;
    static std::atomic<void *> address[kMaxDevices];  // zero-initialised
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(JV_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(JV_ERR_UNSUPPORTED, "device ordinal %d above %d", dev, kMaxDevices - 1);
    void *p = address[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(jv_static_scratch));
        if (e != hipSuccess || !p)
            return fail(JV_ERR_HIP, "hipGetSymbolAddress(static scratch): %s", hipGetErrorString(e));
        address[dev].store(p, std::memory_order_release);  // (two threads may both look it up: same value)
    }
    *out = p;
    return JV_OK;
}
}  // namespace jv

static jv_status check_linear_args(float eps, const void *workspace) {
    if (!(eps >= 0.0f)) return jv::fail(JV_ERR_INVALID_ARG, "eps must be >= 0");
    if (!workspace) return jv::fail(JV_ERR_INVALID_ARG, "workspace is null");
    if ((uintptr_t)workspace & 255)
        return jv::fail(JV_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    return JV_OK;
}

extern "C" {

size_t jv_linear_attn_workspace_bytes(const jv_attn_desc *desc) {
    return jv_linear_block_workspace_bytes(desc, nullptr);
}

size_t jv_linear_block_workspace_bytes(const jv_attn_desc *desc, const jv_dwc_params *dwc) {
    jv::clear_error();
    if (jv::check_desc(desc) != JV_OK) return 0;
    jv::DwcPlan cv;
    const int N = desc->n_prefix + desc->grid_h * desc->grid_w;
    if (desc->head_dim == jv::kHeadDimWide) {
        if (jv::plan_dwc_wide(dwc, jv::linear_wide_workspace_floats(desc->batch, desc->heads, N), desc->batch,
                              desc->heads, N, &cv) != JV_OK)
            return 0;
        return cv.total_floats * sizeof(float);
    }
    const jv::LinearPlan plan = jv::plan_linear(desc->batch, desc->heads, N, desc->dtype == JV_BF16);
    if (jv::plan_dwc(dwc, plan, desc->batch, desc->heads, N, &cv) != JV_OK) return 0;
    return cv.total_floats * sizeof(float);
}

jv_status jv_linear_attn_fwd(const jv_attn_desc *desc, const void *q, const void *k,
                             const void *v, void *o, float eps, void *workspace,
                             size_t workspace_bytes, void *hip_stream) {
    return jv_linear_block_fwd(desc, q, k, v, o, eps, nullptr, workspace, workspace_bytes, hip_stream);
}

jv_status jv_linear_block_fwd(const jv_attn_desc *desc, const void *q, const void *k,
                              const void *v, void *o, float eps, const jv_dwc_params *dwc,
                              void *workspace, size_t workspace_bytes, void *hip_stream) {
    jv::clear_error();
    jv::Problem pr;
    jv_status st = jv::make_problem(desc, q, k, v, o, &pr);
    if (st != JV_OK) return st;
    if ((st = check_linear_args(eps, workspace)) != JV_OK) return st;
    return jv::linear_block_forward(pr, eps, dwc, workspace, workspace_bytes, (hipStream_t)hip_stream);
}

jv_status jv_linear_attn_fwd_static(const jv_attn_desc *desc, const void *q, const void *k,
                                    const void *v, void *o, float eps, void *hip_stream) {
    jv::clear_error();
    jv::Problem pr;
    jv_status st = jv::make_problem(desc, q, k, v, o, &pr);
    if (st != JV_OK) return st;
    if (!(eps >= 0.0f)) return jv::fail(JV_ERR_INVALID_ARG, "eps must be >= 0");
    jv::DwcPlan plain;
    if ((st = jv::plan_dwc(nullptr, jv::plan_linear(pr.B, pr.heads, pr.N, pr.bf16), pr.B, pr.heads, pr.N, &plain)) != JV_OK)
        return st;
    // what jv_linear_attn_workspace_bytes answers
    const size_t need = (pr.D == jv::kHeadDimWide ? jv::linear_wide_workspace_floats(pr.B, pr.heads, pr.N)
                                                  : plain.total_floats) * sizeof(float);
    if (need > (size_t)JV_STATIC_SCRATCH_BYTES)
        return jv::fail(JV_ERR_UNSUPPORTED, "this problem needs %zu bytes of scratch, the static scratch holds %zu",
                        need, (size_t)JV_STATIC_SCRATCH_BYTES);
    void *scratch = nullptr;
    if ((st = jv::static_scratch_address(&scratch)) != JV_OK) return st;
    // Nothing in the scratch has to start at zero: the state pass writes every partial state it
    // later reads in full.
    return jv::linear_block_forward(pr, eps, nullptr, scratch, need, (hipStream_t)hip_stream);
}

jv_status jv_linear_block_focused_fwd(const jv_attn_desc *desc, const void *q, const void *k,
                                      const void *v, void *o, float eps, int32_t focus_p,
                                      const jv_dwc_params *dwc, void *workspace,
                                      size_t workspace_bytes, void *hip_stream) {
    jv::clear_error();
    jv::Problem pr;
    jv_status st = jv::make_problem(desc, q, k, v, o, &pr);
    if (st != JV_OK) return st;
    if ((st = check_linear_args(eps, workspace)) != JV_OK) return st;
    return jv::linear_block_forward(pr, eps, dwc, workspace, workspace_bytes, (hipStream_t)hip_stream, focus_p);
}

}  // extern "C"
