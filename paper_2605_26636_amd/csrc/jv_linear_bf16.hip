// Linear attention (Eq. 2 of the paper, key-sum normaliser; phi = ReLU, or the focused map of
// Eq. 3 for the ablation variant) for bf16 tensors on the matrix cores, fp32 accumulation.
//
//   la_state_bf16   streams K and V once: every wavefront owns a 64 x 64 fp32 state in
//                   accumulators and adds relu(K_tile)^T V_tile per 64-token tile; the token
//                   axis is the contraction axis of both operands, so tiles go through LDS
//                   and come back with transposing reads.  z falls out of the same operands.
//   la_combine      sums the partial states when there are many chunks.
//   la_apply_bf16   sums the (few) partials, splits S and z into bf16 high and low parts held
//                   in registers, and streams Q -> O:  O^T = S^T relu(Q)^T on the matrix
//                   cores, the denominator relu(q).z as one more row block, fp32 divide.
//   la_state_wide_bf16, la_apply_wide_bf16   the same two passes for heads of 128 channels: the
//                   128 x 128 state as four 64 x 64 quadrants, one per wavefront of a workgroup.
#include <type_traits>

#include "jv_linear.h"
#include "jv_mfma.h"
#include "jv_plan.h"

namespace jv {

// Focused feature map (Eq. 3 of the paper, one of the block variants its Table 1 measures):
//   phi_p(x) = |r| / |r^p| * r^p,   r = relu(x), powers element-wise, norms over the 64 channels
// of the token's head; p is an integer >= 2 here (p = 1 is ReLU itself).  A token row is spread
// over the 8 consecutive lanes lane/8*8 .. +7, 8 channels each.  The row is divided by its
// largest entry before the power so that nothing overflows; fp32 arithmetic, result rounded to
// bf16 (the operand type of the matrix instructions).
__device__ inline float row8_combine(float x, bool take_max) {
    // lanes ^1 and ^2 through quad permutes, then the other quad of the 8-lane group through
    // the half-row mirror
    auto with = [&](float a, float b) { return take_max ? fmaxf(a, b) : a + b; };
    auto dpp = [](float v, auto ctrl_tag) {
        constexpr int ctrl = decltype(ctrl_tag)::value;
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true));
    };
    x = with(x, dpp(x, std::integral_constant<int, 0xB1>()));   // quad_perm [1, 0, 3, 2]
    x = with(x, dpp(x, std::integral_constant<int, 0x4E>()));   // quad_perm [2, 3, 0, 1]
    x = with(x, dpp(x, std::integral_constant<int, 0x141>()));  // row_half_mirror
    return x;
}

__device__ inline u32x4 focus_bf16x8(u32x4 x, int p) {
    float r[8] = {bf16_lo(x[0]), bf16_hi(x[0]), bf16_lo(x[1]), bf16_hi(x[1]),
                  bf16_lo(x[2]), bf16_hi(x[2]), bf16_lo(x[3]), bf16_hi(x[3])};
    float top = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        r[e] = fmaxf(r[e], 0.f);
        top = fmaxf(top, r[e]);
    }
    top = row8_combine(top, true);
    const float inv_top = top > 0.f ? __builtin_amdgcn_rcpf(top) : 0.f;
    float y[8], ss = 0.f, sy = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        r[e] *= inv_top;
        y[e] = r[e];
    }
    for (int i = 1; i < p; ++i) {  // uniform trip count
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] *= r[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        ss = fmaf(r[e], r[e], ss);
        sy = fmaf(y[e], y[e], sy);
    }
    ss = row8_combine(ss, false);
    sy = row8_combine(sy, false);
    // |r| = top * sqrt(ss); sy >= 1 whenever top > 0 (the largest entry contributes 1)
    const float scale = top > 0.f ? top * __builtin_amdgcn_sqrtf(ss) * __builtin_amdgcn_rsqf(sy) : 0.f;
    u32x4 out = {pack_bf16x2(y[0] * scale, y[1] * scale), pack_bf16x2(y[2] * scale, y[3] * scale),
                 pack_bf16x2(y[4] * scale, y[5] * scale), pack_bf16x2(y[6] * scale, y[7] * scale)};
    return out;
}
__device__ inline u32x4 feature_map_bf16x8(u32x4 x, int focus_p) {
    return focus_p > 1 ? focus_bf16x8(x, focus_p) : relu_bf16x8(x);  // uniform
}

constexpr int kWaveLds = 64 * 68 * 4;  // per-wave LDS: K and V tiles (16 KB) or a padded state
constexpr int kStateLds = 4 * kWaveLds + 2 * 8 * kHeadDim * 4;

// grid (8 * ceil(n_split * B*heads / 8)), 256 threads, kStateLds bytes of dynamic LDS.
// VSUM: also write the chunk's token sum of V (the input of the dynamic-filter generator of
// the block's convolution branch) to vsum[part][bh][64]; it falls out of the V operands.
// KEEP_V: the apply pass reads V again (convolution branch), so V is loaded with the default
// cache policy; K, and V otherwise, are read once and loaded as a stream.
template <bool VSUM, bool KEEP_V>
__global__ void __launch_bounds__(256, 2)
la_state_bf16(TensorArg kt, TensorArg vt, float *__restrict__ ws, float *__restrict__ vsum,
              int heads, int N, int chunk, int focus_p, int n_split, int BH) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5;
    // Items are the (batch * head, chunk) pairs, chunk fastest.  The hardware deals consecutive
    // workgroups to the eight XCDs in turn; workgroup w takes item (w % 8) * ceil(items / 8) + w / 8,
    // so that an XCD walks a contiguous range of heads -- the same heads whose partial states
    // la_combine sums on that XCD and whose token chunks the apply pass gives it: the states stay
    // in one L2 from pass to pass (8 x 4096 tokens x 16 heads: 58.2 -> 56.1 us for the layer; 2 x
    // 16 384 tokens: 61 -> 59 us).
    const int items = n_split * BH, per_xcd = (items + 7) >> 3;
    const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (item >= items) return;  // whole workgroup
    const int bh = item / n_split, b = bh / heads, h = bh % heads, part = item % n_split;
    const __bf16 *kp = (const __bf16 *)kt.ptr + b * kt.sb + h * kt.sh;
    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh;
    unsigned char *ktile = smem + wave * kWaveLds;
    unsigned char *vtile = ktile + 8192;
    const int n0 = part * chunk, n1 = min(N, n0 + chunk);
    const int lrow = lane >> 3, lchunk = lane & 7;

    f32x16 acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    float zacc[2] = {0.f, 0.f}, vacc[2] = {0.f, 0.f};

    u32x4 kreg[8], vreg[8];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = t0 + r * 8 + lrow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            kreg[r] = zero;
            vreg[r] = zero;
            if (n < n1) {
                kreg[r] = ld_stream((const u32x4 *)(kp + (long long)n * kt.sn + lchunk * 8));
                const u32x4 *vsrc = (const u32x4 *)(vp + (long long)n * vt.sn + lchunk * 8);
                vreg[r] = KEEP_V ? *vsrc : ld_stream(vsrc);
            }
        }
    };

    int t = n0 + wave * 64;
    if (t < n1) fetch(t);
    for (; t < n1; t += 256) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const unsigned off = tile_off_tr(r * 8 + lrow, lchunk);
            *(u32x4 *)(ktile + off) = feature_map_bf16x8(kreg[r], focus_p);
            *(u32x4 *)(vtile + off) = vreg[r];
        }
        if (t + 256 < n1) fetch(t + 256);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 a[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = load_tr_operand(ktile, 16 * ks, i, lane);
                bv[i] = load_tr_operand(vtile, 16 * ks, i, lane);
            }
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                u32x4 au = as_u32x4(a[mi]);
#pragma unroll
                for (int w = 0; w < 4; ++w) zacc[mi] = add_bf16x2(au[w], zacc[mi]);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = mfma32(a[mi], bv[ni], acc[mi][ni]);
            }
            if (VSUM) {
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    u32x4 bu = as_u32x4(bv[ni]);
#pragma unroll
                    for (int w = 0; w < 4; ++w) vacc[ni] = add_bf16x2(bu[w], vacc[ni]);
                }
            }
        }
    }

    // Cross-wave sum through LDS, in a fixed order.
    __syncthreads();
    float *mine = (float *)(smem + wave * kWaveLds);
    float *zbuf = (float *)(smem + 4 * kWaveLds);
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int c2 = 32 * ni + (lane & 31), c1 = 32 * mi + 8 * q4 + 4 * g;
                f32x4 val = {acc[mi][ni][4 * q4], acc[mi][ni][4 * q4 + 1], acc[mi][ni][4 * q4 + 2],
                             acc[mi][ni][4 * q4 + 3]};
                *(f32x4 *)(mine + c2 * 68 + c1) = val;
            }
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
        zbuf[(wave * 2 + g) * kHeadDim + 32 * mi + (lane & 31)] = zacc[mi];
        if (VSUM) zbuf[(8 + wave * 2 + g) * kHeadDim + 32 * mi + (lane & 31)] = vacc[mi];
    }
    __syncthreads();
    float *out = ws + ((size_t)part * BH + bh) * kStateFloats;
#pragma unroll
    for (int i = 0; i < kHeadDim * kHeadDim / 4 / 256; ++i) {  // 16-byte pieces, 4 per thread
        const int e4 = tid + 256 * i, at = (e4 >> 4) * 68 + (e4 & 15) * 4;
        f32x4 s = *(const f32x4 *)((const float *)smem + at);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *(const f32x4 *)((const float *)(smem + w * kWaveLds) + at);
        *(f32x4 *)(out + 4 * e4) = s;
    }
    if (tid < kHeadDim) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) s += zbuf[w * kHeadDim + tid];
        out[kHeadDim * kHeadDim + tid] = s;
    } else if (VSUM && tid < 2 * kHeadDim) {
        float s = 0.f;
#pragma unroll
        for (int w = 8; w < 16; ++w) s += zbuf[w * kHeadDim + tid - kHeadDim];
        vsum[((size_t)part * BH + bh) * kHeadDim + tid - kHeadDim] = s;
    }
}

// grid (8 * ceil(B*heads / 8), ceil((kStateFloats + 64) / 1024)), 256
// threads: dst[bh] = sum_p ws[p][bh], one
// 16-byte piece per thread, the loads of sixteen partials in flight at a time, and states in contiguous ranges per XCD, as
// la_state_bf16 and la_apply_bf16 take them.  With vsum (the
// partial token sums of V, [n_split][B*heads][64]) the sixteen threads after the state's last
// piece sum those too, into partial 0 (each element is read and written by one thread).
__global__ void __launch_bounds__(256)
la_combine(const float *__restrict__ ws, float *__restrict__ dst, float *vsum, int n_split, int BH) {
    const int bh = (blockIdx.x & 7) * ((BH + 7) >> 3) + (blockIdx.x >> 3);
    if (bh >= BH) return;  // whole workgroup
    const int e4 = blockIdx.y * 256 + threadIdx.x;
    constexpr int kStateVec = kStateFloats / 4, kSumVec = kHeadDim / 4;
    if (e4 >= kStateVec + kSumVec || (e4 >= kStateVec && !vsum)) return;
    const bool state = e4 < kStateVec;
    const f32x4 *src = state ? (const f32x4 *)ws + (size_t)bh * kStateVec + e4
                             : (const f32x4 *)vsum + (size_t)bh * kSumVec + (e4 - kStateVec);
    const size_t stride4 = (size_t)BH * (state ? kStateVec : kSumVec);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < n_split; p0 += 16) {
        f32x4 part[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            part[i] = p0 + i < n_split ? src[(size_t)(p0 + i) * stride4] : zero;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += part[i];
    }
    if (state) ((f32x4 *)dst)[(size_t)bh * kStateVec + e4] = sum;
    else ((f32x4 *)vsum)[(size_t)bh * kSumVec + (e4 - kStateVec)] = sum;
}

jv_status combine_states(const float *ws, float *dst, float *vsum, int n_split, int BH, hipStream_t stream) {
    hipLaunchKernelGGL(la_combine, dim3(8 * ((BH + 7) / 8), ((kStateFloats + kHeadDim) / 4 + 255) / 256), dim3(256), 0,
                       stream, ws, dst, vsum, n_split, BH);
    return launch_status("la_combine");
}

// The partial states of one (batch, head) summed into LDS by 256 threads: St[c2][c1] with the
// 8-float group index rotated by the row, then z.  16-byte loads, all of them issued before the first use.
__device__ inline void sum_states(const float *states, int n_part, long long part_stride, float *St, float *zs, int tid) {
    const f32x4 *src = (const f32x4 *)states;
    const long long stride4 = part_stride / 4;
    constexpr int kVec = kStateFloats / 4, kIter = (kVec + 255) / 256;
    f32x4 part[kIter][4];
#pragma unroll
    for (int it = 0; it < kIter; ++it)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int e4 = it * 256 + tid;
            f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            part[it][p] = (e4 < kVec && p < n_part) ? src[p * stride4 + e4] : zero;
        }
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
        const int e4 = it * 256 + tid;
        if (e4 >= kVec) break;
        f32x4 sum = part[it][0];
        for (int p = 4; p < n_part; ++p) sum += src[p * stride4 + e4];  // more than 4: rare
#pragma unroll
        for (int p = 1; p < 4; ++p) sum += part[it][p];
        const int e = 4 * e4;
        if (e < kHeadDim * kHeadDim) {
            const int c2 = e >> 6, c1 = e & 63;  // 4 consecutive c1 stay inside one group
            *(f32x4 *)(St + c2 * 64 + ((((c1 >> 3) ^ (c2 & 7)) << 3) | (c1 & 7))) = sum;
        } else {
            *(f32x4 *)(zs + e - kHeadDim * kHeadDim) = sum;
        }
    }
}

// What the kernels that apply a state share.  A operands: S^T rows c2 = 32 mi + li, k-slots c1 = 16 ks + 8 g + (0..7), as bf16 high + low
// parts; the denominator block: row 0 = z high part, row 1 = z low part, other rows zero.
struct ApplyOperands {
    bf16x8 s_hi[2][4], s_lo[2][4], z_op[4];
};
__device__ inline void apply_operands(ApplyOperands &o, const float *St, const float *zs, int li, int g) {
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c2 = 32 * mi + li, grp = 2 * ks + g;
            const float *row = St + c2 * 64 + ((grp ^ (c2 & 7)) << 3);
            const f32x4 x0 = *(const f32x4 *)row, x1 = *(const f32x4 *)(row + 4);
            const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const __bf16 hi = (__bf16)x[e];
                o.s_hi[mi][ks][e] = hi;
                o.s_lo[mi][ks][e] = (__bf16)(x[e] - (float)hi);
            }
        }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float zv = zs[16 * ks + 8 * g + e];
            const __bf16 hi = (__bf16)zv;
            const __bf16 lo = (__bf16)(zv - (float)hi);
            o.z_op[ks][e] = li == 0 ? hi : (li == 1 ? lo : (__bf16)0.f);
        }
}
// acc = S^T relu(q)^T for the query in row `row` of qtile (tile_off_row); returns 1 / (denominator + eps).
__device__ inline float apply_products(const ApplyOperands &o, const unsigned char *qtile, int row, int g, float eps, f32x16 (&acc)[2]) {
    f32x16 accz;
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[0][v] = 0.f; acc[1][v] = 0.f; accz[v] = 0.f; }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 qb = as_bf16x8(*(const u32x4 *)(qtile + tile_off_row(row, 2 * ks + g)));
        accz = mfma32(o.z_op[ks], qb, accz);
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            acc[mi] = mfma32(o.s_lo[mi][ks], qb, acc[mi]);
            acc[mi] = mfma32(o.s_hi[mi][ks], qb, acc[mi]);
        }
    }
    // den lives in rows 0 and 1 of the denominator block: registers 0, 1 of lanes g = 0.
    float den_lo, den_hi;
    pair_values(accz[0] + accz[1], &den_lo, &den_hi);
    return __builtin_amdgcn_rcpf(den_lo + eps);
}
// 32 tokens from n0 on, those below n1, through 4 KB of LDS of the wavefront's own: whole rows.
__device__ inline void apply_store_bf16(const f32x16 (&acc)[2], float inv, unsigned char *otile, __bf16 *op, long long sn, int n0, int n1, int lane) {
    const int g = lane >> 5, li = lane & 31, lrow = lane >> 3, lchunk = lane & 7;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const u32x2 pk = {pack_bf16x2(acc[mi][4 * q4] * inv, acc[mi][4 * q4 + 1] * inv),
                              pack_bf16x2(acc[mi][4 * q4 + 2] * inv, acc[mi][4 * q4 + 3] * inv)};
            *(u32x2 *)(otile + tile_off_row(li, 4 * mi + q4) + 8 * g) = pk;
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int orow = r * 8 + lrow, on = n0 + orow;
        const u32x4 val = *(const u32x4 *)(otile + tile_off_row(orow, lchunk));
        if (on < n1) st_stream((u32x4 *)(op + (long long)on * sn + lchunk * 8), val);
    }
}
__device__ inline void apply_store_f32(const f32x16 (&acc)[2], float inv, float *op, long long sn, int n, int n1, int g) {
    if (n >= n1) return;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const f32x4 val = {acc[mi][4 * q4] * inv, acc[mi][4 * q4 + 1] * inv, acc[mi][4 * q4 + 2] * inv, acc[mi][4 * q4 + 3] * inv};
            *(f32x4 *)(op + (long long)n * sn + 32 * mi + 8 * q4 + 4 * g) = val;
        }
}

// grid (8 * ceil(n_chunks * B*heads / 8)), 256 threads.  Workgroups are dealt to the eight XCDs
// in turn; the index is remapped so that the workgroups one XCD receives walk (batch, head)
// pairs chunk by chunk: the token chunks of a pair then share that XCD's L2 copy of the state.
// `states` holds n_part partial states per (batch, head), part_stride floats apart.
// KS = 0: linear attention alone.  KS = 3 or 5: the block's convolution branch is added before
// the store: the normalised tile is staged in LDS as fp32, and the lane that stores 8 channels
// of 4 consecutive tokens first adds sum_taps kappa[c][tap] * V[token + tap][c] for them (V rows
// of the neighbouring tokens come from the caches: every V row is used by KS*KS tokens).
template <bool O_BF16, int KS>
__global__ void __launch_bounds__(256, 2)
la_apply_bf16(TensorArg qt, TensorArg ot, const float *__restrict__ states, int n_part,
              long long part_stride, int heads, int N, int tokens_per_wg, int n_chunks, int n_wg,
              float eps, TensorArg vt, DwcArg cv, int focus_p) {
    // St[c2][c1] fp32 with the 8-float group index rotated by the row, then z; afterwards the
    // same bytes stage output tiles (4 KB of bf16 per wave, or 8 KB of fp32 with the
    // convolution).  Then one 8 KB query tile per wave, then the filters as [tap][channel].
    constexpr int kStageBytes = KS ? 4 * 8192 : kStateFloats * 4;
    __shared__ __align__(16) unsigned char smem[kStageBytes + 4 * 8192 + KS * KS * kHeadDim * 4];
    float *St = (float *)smem;
    float *zs = St + kHeadDim * kHeadDim;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int per_xcd = (n_wg + 7) / 8;
    const int wg = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (wg >= n_wg) return;  // whole workgroup
    const int bh = wg / n_chunks, b = bh / heads, h = bh % heads;
    const __bf16 *qp = (const __bf16 *)qt.ptr + b * qt.sb + h * qt.sh;
    const int n0 = (wg % n_chunks) * tokens_per_wg, n1 = min(N, n0 + tokens_per_wg);
    const int lrow = lane >> 3, lchunk = lane & 7;

    // Query tiles are fetched one step ahead; start the first fetch before the state prologue.
    u32x4 qreg[8];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = t0 + r * 8 + lrow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            qreg[r] = zero;
            if (n < n1) qreg[r] = ld_stream((const u32x4 *)(qp + (long long)n * qt.sn + lchunk * 8));
        }
    };
    int t = n0 + wave * 64;
    if (t < n1) fetch(t);

    float *kap = (float *)(smem + kStageBytes + 4 * 8192);
    if (KS) {
        const float *kbase = cv.kappa + b * cv.kappa_sb + (size_t)h * kHeadDim * KS * KS;
        for (int e = tid; e < kHeadDim * KS * KS; e += 256) kap[(e % (KS * KS)) * kHeadDim + e / (KS * KS)] = kbase[e];
    }

    sum_states(states + (size_t)bh * kStateFloats, n_part, part_stride, St, zs, tid);
    __syncthreads();

    ApplyOperands ops;
    apply_operands(ops, St, zs, li, g);
    __syncthreads();  // the state bytes are reused as output staging from here on

    unsigned char *qtile = smem + kStageBytes + wave * 8192;
    unsigned char *otile = smem + wave * (KS ? 8192 : 4096);
    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh;
    for (; t < n1; t += 256) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
            *(u32x4 *)(qtile + tile_off_row(r * 8 + lrow, lchunk)) = feature_map_bf16x8(qreg[r], focus_p);
        if (t + 256 < n1) fetch(t + 256);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            if (t + 32 * nt >= n1) break;  // wave-uniform
            const int row = 32 * nt + li;
            f32x16 acc[2];
            const float inv = apply_products(ops, qtile, row, g, eps, acc);
            if (KS) {
                // fp32 staging: 256-byte token rows, 16-byte chunk index rotated by the row
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        f32x4 val = {acc[mi][4 * q4] * inv, acc[mi][4 * q4 + 1] * inv,
                                     acc[mi][4 * q4 + 2] * inv, acc[mi][4 * q4 + 3] * inv};
                        *(f32x4 *)(otile + li * 256 + (((8 * mi + 2 * q4 + g) ^ (li & 15)) << 4)) = val;
                    }
                // A lane finishes 4 consecutive tokens x 8 channels: the taps of neighbouring
                // tokens overlap, so one tap row needs 4 + KS - 1 loads instead of 4 * KS.
                // Out-of-grid taps (and slots past the end of the range) read a valid row with
                // weight zero, so the loads of a tap row are all in flight at once.
                constexpr int kPad = KS / 2, kSpan = 4 + KS - 1;
                const int tok0 = t + 32 * nt + 4 * lrow;            // first of this lane's tokens
                const int last = n1 - 1;
                float sum[4][8];
                int gr[4], gc[4];
                bool on_grid[4];  // prefix tokens (grid index below zero) get no convolution term
                {
                    const int g0 = min(tok0, last) - cv.P;  // grid index of the lane's first token
                    const int base = max(g0, 0);
                    int r0 = base / cv.W, c0 = base - r0 * cv.W;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int orow = 4 * lrow + r;
                        const f32x4 o0 = *(const f32x4 *)(otile + orow * 256 + (((2 * lchunk) ^ (orow & 15)) << 4));
                        const f32x4 o1 = *(const f32x4 *)(otile + orow * 256 + (((2 * lchunk + 1) ^ (orow & 15)) << 4));
                        sum[r][0] = o0[0]; sum[r][1] = o0[1]; sum[r][2] = o0[2]; sum[r][3] = o0[3];
                        sum[r][4] = o1[0]; sum[r][5] = o1[1]; sum[r][6] = o1[2]; sum[r][7] = o1[3];
                        gr[r] = r0;
                        gc[r] = c0;
                        on_grid[r] = g0 + r >= 0;
                        if (on_grid[r] && ++c0 == cv.W) { c0 = 0; ++r0; }
                    }
                }
#pragma unroll 1
                for (int di = -kPad; di <= kPad; ++di) {
                    u32x4 vv[kSpan];
#pragma unroll
                    for (int j = 0; j < kSpan; ++j) {
                        const int src = tok0 + j - kPad + di * cv.W;  // token of column j in this tap row
                        const int safe = min(max(src, 0), N - 1);
                        vv[j] = *(const u32x4 *)(vp + (long long)safe * vt.sn + lchunk * 8);
                    }
                    const float *krow = kap + (di + kPad) * KS * kHeadDim + 8 * lchunk;
#pragma unroll
                    for (int dj = -kPad; dj <= kPad; ++dj) {
                        const f32x4 k0 = *(const f32x4 *)(krow + (dj + kPad) * kHeadDim);
                        const f32x4 k1 = *(const f32x4 *)(krow + (dj + kPad) * kHeadDim + 4);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const bool ok = tok0 + r <= last && on_grid[r] && (unsigned)(gr[r] + di) < (unsigned)cv.H &&
                                            (unsigned)(gc[r] + dj) < (unsigned)cv.W;
                            const float m = ok ? 1.0f : 0.0f;
                            const u32x4 x = vv[r + dj + kPad];
                            sum[r][0] = fmaf(k0[0] * m, bf16_lo(x[0]), sum[r][0]);
                            sum[r][1] = fmaf(k0[1] * m, bf16_hi(x[0]), sum[r][1]);
                            sum[r][2] = fmaf(k0[2] * m, bf16_lo(x[1]), sum[r][2]);
                            sum[r][3] = fmaf(k0[3] * m, bf16_hi(x[1]), sum[r][3]);
                            sum[r][4] = fmaf(k1[0] * m, bf16_lo(x[2]), sum[r][4]);
                            sum[r][5] = fmaf(k1[1] * m, bf16_hi(x[2]), sum[r][5]);
                            sum[r][6] = fmaf(k1[2] * m, bf16_lo(x[3]), sum[r][6]);
                            sum[r][7] = fmaf(k1[3] * m, bf16_hi(x[3]), sum[r][7]);
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int on = tok0 + r;
                    if (on <= last) {
                        if (O_BF16) {
                            __bf16 *op = (__bf16 *)ot.ptr + b * ot.sb + h * ot.sh;
                            u32x4 pk = {pack_bf16x2(sum[r][0], sum[r][1]), pack_bf16x2(sum[r][2], sum[r][3]),
                                        pack_bf16x2(sum[r][4], sum[r][5]), pack_bf16x2(sum[r][6], sum[r][7])};
                            st_stream((u32x4 *)(op + (long long)on * ot.sn + lchunk * 8), pk);
                        } else {
                            float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh + (long long)on * ot.sn + lchunk * 8;
                            f32x4 s0 = {sum[r][0], sum[r][1], sum[r][2], sum[r][3]};
                            f32x4 s1 = {sum[r][4], sum[r][5], sum[r][6], sum[r][7]};
                            *(f32x4 *)op = s0;
                            *(f32x4 *)(op + 4) = s1;
                        }
                    }
                }
            } else if (O_BF16) {
                apply_store_bf16(acc, inv, otile, (__bf16 *)ot.ptr + b * ot.sb + h * ot.sh, ot.sn, t + 32 * nt, n1, lane);
            } else {
                apply_store_f32(acc, inv, (float *)ot.ptr + b * ot.sb + h * ot.sh, ot.sn, t + row, n1, g);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Both passes in one launch, for launches whose state pass would leave the chip idle: a workgroup forms the whole state of a (batch, head), as
// la_state_bf16 does, and applies it to a part of its queries, as la_apply_bf16 does, so that no workgroup waits for
// another's sums.  Bound by round trips to memory (one and a half instead of the three or four of two or three launches) and by
// what one unit takes in: K and V of a (batch, head), once for every part of its queries, whose workgroups run on one XCD and share its L2.
// Eight wavefronts take tiles of 64 tokens in turn for the state, then units of 32 queries.
// grid (8 * ceil(n_wg / 8)), n_wg = parts * B*heads, part fastest; 512 threads, kFusedLds bytes of dynamic LDS.
// ---------------------------------------------------------------------------------------
constexpr int kFusedWaves = 8;
constexpr int kFusedZ = kFusedWaves * kWaveLds, kFusedSt = kFusedZ + 2 * kFusedWaves * kHeadDim * 4, kFusedLds = kFusedSt + kStateFloats * 4;

template <bool O_BF16>
__global__ void __launch_bounds__(64 * kFusedWaves, 1)
la_fused_bf16(TensorArg qt, TensorArg kt, TensorArg vt, TensorArg ot, int heads, int N, int units_per_wg, int n_parts, int n_wg, float eps) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int per_xcd = (n_wg + 7) / 8, wg = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (wg >= n_wg) return;  // whole workgroup
    const int bh = wg / n_parts, b = bh / heads, h = bh % heads;
    const __bf16 *qp = (const __bf16 *)qt.ptr + b * qt.sb + h * qt.sh;
    const __bf16 *kp = (const __bf16 *)kt.ptr + b * kt.sb + h * kt.sh;
    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh;
    const int lrow = lane >> 3, lchunk = lane & 7;
    unsigned char *ktile = smem + wave * kWaveLds, *vtile = ktile + 8192;

    u32x4 kreg[8], vreg[8], qreg[4];
    auto fetch = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = t0 + r * 8 + lrow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            kreg[r] = vreg[r] = zero;
            if (n < N) {
                kreg[r] = *(const u32x4 *)(kp + (long long)n * kt.sn + lchunk * 8);
                vreg[r] = *(const u32x4 *)(vp + (long long)n * vt.sn + lchunk * 8);
            }
        }
    };
    auto fetch_q = [&](int unit) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = 32 * unit + r * 8 + lrow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            qreg[r] = zero;
            if (n < N) qreg[r] = ld_stream((const u32x4 *)(qp + (long long)n * qt.sn + lchunk * 8));
        }
    };
    const int unit0 = (wg % n_parts) * units_per_wg, unit1 = min((N + 31) / 32, unit0 + units_per_wg);
    int t = wave * 64, unit = unit0 + wave;
    if (t < N) fetch(t);
    if (unit < unit1) fetch_q(unit);

    f32x16 acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    float zacc[2] = {0.f, 0.f};
    for (; t < N; t += 64 * kFusedWaves) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const unsigned off = tile_off_tr(r * 8 + lrow, lchunk);
            *(u32x4 *)(ktile + off) = relu_bf16x8(kreg[r]);
            *(u32x4 *)(vtile + off) = vreg[r];
        }
        if (t + 64 * kFusedWaves < N) fetch(t + 64 * kFusedWaves);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 a[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = load_tr_operand(ktile, 16 * ks, i, lane);
                bv[i] = load_tr_operand(vtile, 16 * ks, i, lane);
            }
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                const u32x4 au = as_u32x4(a[mi]);
#pragma unroll
                for (int w = 0; w < 4; ++w) zacc[mi] = add_bf16x2(au[w], zacc[mi]);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = mfma32(a[mi], bv[ni], acc[mi][ni]);
            }
        }
    }

    // Cross-wave sum through LDS, in a fixed order, into St[c2][c1] with the 8-float group index rotated by the row, then z.
    __syncthreads();
    float *mine = (float *)(smem + wave * kWaveLds), *zbuf = (float *)(smem + kFusedZ), *St = (float *)(smem + kFusedSt), *zs = St + kHeadDim * kHeadDim;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int c2 = 32 * ni + li, c1 = 32 * mi + 8 * q4 + 4 * g;
                const f32x4 val = {acc[mi][ni][4 * q4], acc[mi][ni][4 * q4 + 1], acc[mi][ni][4 * q4 + 2], acc[mi][ni][4 * q4 + 3]};
                *(f32x4 *)(mine + c2 * 68 + c1) = val;
            }
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) zbuf[(wave * 2 + g) * kHeadDim + 32 * mi + li] = zacc[mi];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e4 = tid + 512 * i, c2 = e4 >> 4, c1 = (e4 & 15) * 4;
        f32x4 s[4];
#pragma unroll
        for (int w = 0; w < 4; ++w)
            s[w] = *(const f32x4 *)((const float *)(smem + w * kWaveLds) + c2 * 68 + c1) + *(const f32x4 *)((const float *)(smem + (w + 4) * kWaveLds) + c2 * 68 + c1);
        *(f32x4 *)(St + c2 * 64 + ((((c1 >> 3) ^ (c2 & 7)) << 3) | (c1 & 7))) = (s[0] + s[1]) + (s[2] + s[3]);
    }
    if (tid < kHeadDim) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < 2 * kFusedWaves; ++w) s += zbuf[w * kHeadDim + tid];
        zs[tid] = s;
    }
    __syncthreads();
    if (unit >= unit1) return;

    ApplyOperands ops;
    apply_operands(ops, St, zs, li, g);
    unsigned char *qtile = smem + wave * kWaveLds, *otile = qtile + 4096;  // (the sums there have been read)
    for (; unit < unit1; unit += kFusedWaves) {
#pragma unroll
        for (int r = 0; r < 4; ++r) *(u32x4 *)(qtile + tile_off_row(r * 8 + lrow, lchunk)) = relu_bf16x8(qreg[r]);
        if (unit + kFusedWaves < unit1) fetch_q(unit + kFusedWaves);
        f32x16 out[2];
        const float inv = apply_products(ops, qtile, li, g, eps, out);
        const int n0 = 32 * unit;
        if (O_BF16) apply_store_bf16(out, inv, otile, (__bf16 *)ot.ptr + b * ot.sb + h * ot.sh, ot.sn, n0, N, lane);
        else apply_store_f32(out, inv, (float *)ot.ptr + b * ot.sb + h * ot.sh, ot.sn, n0 + li, N, g);
    }
}

// ---------------------------------------------------------------------------------------
// The apply pass with the convolution branch on a window of V that moves through LDS.  What bounds
// la_apply_bf16<., KS> is its V loads (every V row comes through the vector memory path 4.5 times
// for KS = 3: 30 of 85 us at 32 images of 37 x 37, 16 heads) and the vector instructions of the taps
// and their masks; here every row is fetched once per workgroup.  That shape: 97 -> 63 us for 270 MB
// (4.3 TB/s), vector instructions now 45 % of the time; 8 images of 64 x 64 44 -> 36 us.
// The workgroup walks its chunk in steps of 128 tokens, 32 per wavefront.  Its ring in LDS holds the
// grid cells whose taps a step needs, 128 + 2 pad (W + 1) rows (pad = KS / 2, cells outside the grid as
// zeros), and the 128 cells the next step adds are in flight in registers meanwhile.  The 32
// rows behind the ring's end repeat its first, so that a wavefront's sources in a tap row are consecutive.
// The product is formed as relu(Q) S with the columns of S dealt so that lane (g, li) holds channels
// 2 li and 2 li + 1 of the tokens 8 q4 + 4 g .. + 3 (q4 = 0 .. 3): the filters of two channels
// stay in registers for the whole pass, a V row is one dword per lane, nothing is staged, and
// an output row leaves as 128 contiguous bytes.  Taps outside the grid's width are skipped under the execution mask.
// Grid and XCD mapping as la_apply_bf16, 256 threads, conv_ring_lds bytes of dynamic LDS.
// ---------------------------------------------------------------------------------------
static_assert(kRingFixedLds == kStateFloats * 4 + 4 * 32 * 4, "the ring follows the state");

// The 3 x 3 taps of one token and two channels, row by row (the order in which la_apply_bf16 adds them):
// s0 += k[di][dj][0] x[di][dj][0], s1 likewise, column dj in the lanes of use[dj] only.  For wavefronts whose lanes are all active.
__device__ inline void masked_taps3(const unsigned long long (&use)[3], const float (&k)[9][2], const float (*x0)[2], const float (*x1)[2],
                                    const float (*x2)[2], float &s0, float &s1) {
    unsigned long long saved;
    asm("s_mov_b64 %2, exec\n\t"
        "s_mov_b64 exec, %3\n\tv_fmac_f32 %0, %6, %24\n\tv_fmac_f32 %1, %7, %25\n\t"
        "s_mov_b64 exec, %4\n\tv_fmac_f32 %0, %8, %26\n\tv_fmac_f32 %1, %9, %27\n\t"
        "s_mov_b64 exec, %5\n\tv_fmac_f32 %0, %10, %28\n\tv_fmac_f32 %1, %11, %29\n\t"
        "s_mov_b64 exec, %3\n\tv_fmac_f32 %0, %12, %30\n\tv_fmac_f32 %1, %13, %31\n\t"
        "s_mov_b64 exec, %4\n\tv_fmac_f32 %0, %14, %32\n\tv_fmac_f32 %1, %15, %33\n\t"
        "s_mov_b64 exec, %5\n\tv_fmac_f32 %0, %16, %34\n\tv_fmac_f32 %1, %17, %35\n\t"
        "s_mov_b64 exec, %3\n\tv_fmac_f32 %0, %18, %36\n\tv_fmac_f32 %1, %19, %37\n\t"
        "s_mov_b64 exec, %4\n\tv_fmac_f32 %0, %20, %38\n\tv_fmac_f32 %1, %21, %39\n\t"
        "s_mov_b64 exec, %5\n\tv_fmac_f32 %0, %22, %40\n\tv_fmac_f32 %1, %23, %41\n\t"
        "s_mov_b64 exec, %2"
        : "+v"(s0), "+v"(s1), "=&s"(saved)
        : "s"(use[0]), "s"(use[1]), "s"(use[2]), "v"(k[0][0]), "v"(k[0][1]), "v"(k[1][0]), "v"(k[1][1]), "v"(k[2][0]), "v"(k[2][1]),
          "v"(k[3][0]), "v"(k[3][1]), "v"(k[4][0]), "v"(k[4][1]), "v"(k[5][0]), "v"(k[5][1]), "v"(k[6][0]), "v"(k[6][1]),
          "v"(k[7][0]), "v"(k[7][1]), "v"(k[8][0]), "v"(k[8][1]), "v"(x0[0][0]), "v"(x0[0][1]), "v"(x0[1][0]), "v"(x0[1][1]),
          "v"(x0[2][0]), "v"(x0[2][1]), "v"(x1[0][0]), "v"(x1[0][1]), "v"(x1[1][0]), "v"(x1[1][1]), "v"(x1[2][0]), "v"(x1[2][1]),
          "v"(x2[0][0]), "v"(x2[0][1]), "v"(x2[1][0]), "v"(x2[1][1]), "v"(x2[2][0]), "v"(x2[2][1]));
}
// s0 += k0 x0, s1 += k1 x1 in the lanes of `mask`.
__device__ inline void masked_fma2(unsigned long long mask, float k0, float k1, float x0, float x1, float &s0, float &s1) {
    unsigned long long saved;
    asm("s_and_saveexec_b64 %2, %3\n\t"
        "v_fmac_f32 %0, %4, %6\n\tv_fmac_f32 %1, %5, %7\n\t"
        "s_mov_b64 exec, %2"
        : "+v"(s0), "+v"(s1), "=&s"(saved)
        : "s"(mask), "v"(k0), "v"(k1), "v"(x0), "v"(x1)
        : "scc");
}

template <bool O_BF16, int KS>
__global__ void __launch_bounds__(256, 2)
la_apply_conv_bf16(TensorArg qt, TensorArg ot, const float *__restrict__ states, int n_part, long long part_stride,
                   int heads, int N, int tokens_per_wg, int n_chunks, int n_wg, float eps, TensorArg vt, DwcArg cv,
                   int focus_p) {
    constexpr int kPad = KS / 2, kSpan = 4 + KS - 1, kTaps = KS * KS;
    extern __shared__ __align__(16) unsigned char smem[];
    float *St = (float *)smem, *zs = St + kHeadDim * kHeadDim;
    unsigned char *ring = smem + kRingFixedLds;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int per_xcd = (n_wg + 7) / 8;
    const int wg = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (wg >= n_wg) return;  // whole workgroup
    const int bh = wg / n_chunks, b = bh / heads, h = bh % heads;
    const int n0 = (wg % n_chunks) * tokens_per_wg, n1 = min(N, n0 + tokens_per_wg);
    const int lrow = lane >> 3, lchunk = lane & 7;
    const __bf16 *qp = (const __bf16 *)qt.ptr + b * qt.sb + h * qt.sh + 8 * lchunk;

    u32x4 qreg[4];
    auto fetch_q = [&](int t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = t + 8 * r + lrow;
            qreg[r] = u32x4{0u, 0u, 0u, 0u};
            if (n < n1) qreg[r] = ld_stream((const u32x4 *)(qp + (long long)n * qt.sn));
        }
    };
    fetch_q(n0 + 32 * wave);

    // Ring: the cell `c` cells behind the chunk's first needed one sits in row c mod rows.
    const int W = cv.W, cells = cv.H * W, rows = kRingStep + 2 * kPad * (W + 1);
    const int first = n0 - cv.P - kPad * (W + 1);
    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh + (long long)cv.P * vt.sn + 8 * lchunk;
    const int vrow = tid >> 3;  // this thread's 16 bytes (chunk lchunk) of every 32nd row
    auto load_v = [&](int c) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if ((unsigned)(first + c) < (unsigned)cells) v = *(const u32x4 *)(vp + (long long)(first + c) * vt.sn);
        return v;
    };
    auto put_v = [&](int slot, u32x4 v) {
        *(u32x4 *)(ring + slot * 128 + 16 * lchunk) = v;
        if (slot < kRingRepeat) *(u32x4 *)(ring + (rows + slot) * 128 + 16 * lchunk) = v;
    };
    for (int c0 = 0; c0 < rows; c0 += 256) {
        u32x4 v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = c0 + 32 * r + vrow < rows ? load_v(c0 + 32 * r + vrow) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (c0 + 32 * r + vrow < rows) put_v(c0 + 32 * r + vrow, v[r]);
    }
    float kap[kTaps][2];  // filters of channels 2 li, 2 li + 1
    {
        const float *kbase = cv.kappa + b * cv.kappa_sb + (size_t)(h * kHeadDim + 2 * li) * kTaps;
#pragma unroll
        for (int tap = 0; tap < kTaps; ++tap) {
            kap[tap][0] = kbase[tap];
            kap[tap][1] = kbase[kTaps + tap];
        }
    }
    sum_states(states + (size_t)bh * kStateFloats, n_part, part_stride, St, zs, tid);
    __syncthreads();
    // B operands: column li of block ni is channel c2 = 2 li + ni, k-slots c1 = 16 ks + 8 g + (0..7), as
    // bf16 hi + lo; A operand of the denominator: row 0 = z high part, row 1 = z low part, other rows zero.
    bf16x8 s_hi[2][4], s_lo[2][4], z_op[4];
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int c2 = 2 * li + ni, grp = 2 * ks + g;
            const float *row = St + c2 * 64 + ((grp ^ (c2 & 7)) << 3);
            const f32x4 x0 = *(const f32x4 *)row, x1 = *(const f32x4 *)(row + 4);
            const float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const __bf16 hi = (__bf16)x[e];
                s_hi[ni][ks][e] = hi;
                s_lo[ni][ks][e] = (__bf16)(x[e] - (float)hi);
            }
        }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float zv = zs[16 * ks + 8 * g + e];
            const __bf16 hi = (__bf16)zv;
            const __bf16 lo = (__bf16)(zv - (float)hi);
            z_op[ks][e] = li == 0 ? hi : (li == 1 ? lo : (__bf16)0.f);
        }
    lds_barrier();  // the state's bytes hold query tiles from here on, and the ring is filled

    unsigned char *qtile = smem + wave * 4096;
    float *inv_row = (float *)(smem + kStateFloats * 4) + 32 * wave;
    const int own0 = 32 * wave + 4 * g;  // this lane's tokens in a step: own0 + 8 q4 + r
    const int col_group = 8 % W, col_step = kRingStep % W;
    int col0 = ((n0 - cv.P + own0) % W + W) % W;  // grid column of the first of them
    int base = 0;                          // ring row of the step's first needed cell
    for (int t = n0; t < n1; t += kRingStep) {
        // the first cell that only the next step needs, counted from `first`
        const int fresh = t - n0 + rows;
        const bool more = t + kRingStep < n1;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *(u32x4 *)(qtile + tile_off_row(8 * r + lrow, lchunk)) = feature_map_bf16x8(qreg[r], focus_p);
        u32x4 vreg[4];
        if (more) {
#pragma unroll
            for (int r = 0; r < 4; ++r) vreg[r] = load_v(fresh + 32 * r + vrow);
            fetch_q(t + kRingStep + 32 * wave);
        }
        if (t + 32 * wave < n1) {  // wave-uniform
            f32x16 acc[2], accz;
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[0][v] = 0.f; acc[1][v] = 0.f; accz[v] = 0.f; }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 qb = as_bf16x8(*(const u32x4 *)(qtile + tile_off_row(li, 2 * ks + g)));
                accz = mfma32(z_op[ks], qb, accz);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    acc[ni] = mfma32(qb, s_lo[ni][ks], acc[ni]);
                    acc[ni] = mfma32(qb, s_hi[ni][ks], acc[ni]);
                }
            }
            // den lives in rows 0 and 1 of the denominator block: registers 0, 1 of lanes g = 0.
            float den_lo, den_hi;
            pair_values(accz[0] + accz[1], &den_lo, &den_hi);
            if (g == 0) inv_row[li] = __builtin_amdgcn_rcpf(den_lo + eps);
            const unsigned char *tap_base[KS];  // this lane's dword of the first source of every tap row
#pragma unroll
            for (int di = 0; di < KS; ++di) {
                unsigned slot = (unsigned)(base + own0 + di * W);
                slot = min(slot, slot - (unsigned)rows);
                tap_base[di] = ring + slot * 128 + 4 * li;
            }
            int col = col0;
            const bool prefix = t < cv.P, whole = t + 32 * wave + 32 <= n1;
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 inv = *(const f32x4 *)(inv_row + 8 * q4 + 4 * g);
                float sum[4][2];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sum[r][0] = acc[0][4 * q4 + r] * inv[r];
                    sum[r][1] = acc[1][4 * q4 + r] * inv[r];
                }
                // Lanes whose tap column dj is inside the grid's width: token r's left neighbour is unless
                // (col + r) % W = 0, and so on.
                unsigned long long use[4][KS];
                if (KS == 3 && W >= 4) {
                    unsigned long long inner[5];  // token r and its left neighbour are in one grid row
                    inner[0] = __builtin_amdgcn_ballot_w64(col != 0);
#pragma unroll
                    for (int r = 1; r < 5; ++r) inner[r] = __builtin_amdgcn_ballot_w64(col != W - r);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        use[r][0] = inner[r];
                        use[r][1] = ~0ull;
                        use[r][2] = inner[r + 1];
                    }
                } else {
                    int c = col;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
#pragma unroll
                        for (int dj = 0; dj < KS; ++dj) use[r][dj] = __builtin_amdgcn_ballot_w64((unsigned)(c + dj - kPad) < (unsigned)W);
                        if (++c >= W) c = 0;
                    }
                }
                if (prefix) {  // uniform: prefix tokens take no taps
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const unsigned long long live = __builtin_amdgcn_ballot_w64(t + own0 + 8 * q4 + r >= cv.P);
#pragma unroll
                        for (int dj = 0; dj < KS; ++dj) use[r][dj] &= live;
                    }
                }
                auto tap_row = [&](int di, float (&x)[kSpan][2]) __attribute__((always_inline)) {
                    const unsigned *src = (const unsigned *)(tap_base[di] + 1024 * q4);
#pragma unroll
                    for (int j = 0; j < kSpan; ++j) {
                        const unsigned u = src[32 * j];
                        x[j][0] = bf16_lo(u);
                        x[j][1] = bf16_hi(u);
                    }
                };
                if constexpr (KS == 3) {
                    float x[3][kSpan][2];
#pragma unroll
                    for (int di = 0; di < 3; ++di) tap_row(di, x[di]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) masked_taps3(use[r], kap, &x[0][r], &x[1][r], &x[2][r], sum[r][0], sum[r][1]);
                } else {  // (five rows of sources do not fit beside the filters)
#pragma unroll
                    for (int di = 0; di < KS; ++di) {
                        float x[kSpan][2];
                        tap_row(di, x);
#pragma unroll
                        for (int dj = 0; dj < KS; ++dj)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                masked_fma2(use[r][dj], kap[di * KS + dj][0], kap[di * KS + dj][1], x[r + dj][0], x[r + dj][1], sum[r][0], sum[r][1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                const int n = t + own0 + 8 * q4;
                char *out = (char *)ot.ptr + (b * ot.sb + h * ot.sh + (long long)n * ot.sn + 2 * li) * (O_BF16 ? 2 : 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (whole || n + r < n1) {
                        if (O_BF16) __builtin_nontemporal_store(pack_bf16x2(sum[r][0], sum[r][1]), (unsigned *)out);
                        else *(float2 *)out = float2{sum[r][0], sum[r][1]};
                    }
                    out += ot.sn * (O_BF16 ? 2 : 4);
                }
                col += col_group;
                if (col >= W) col -= W;
            }
        }
        if (more) {
            lds_barrier();  // nobody reads the oldest 128 rows any more
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                unsigned slot = (unsigned)(base + 32 * r + vrow);
                put_v((int)min(slot, slot - (unsigned)rows), vreg[r]);
            }
            lds_barrier();
        }
        base += kRingStep;
        if (base >= rows) base -= rows;
        col0 += col_step;
        if (col0 >= W) col0 -= W;
    }
}

template <bool O_BF16, int KS>
static jv_status launch_apply(hipStream_t stream, const Problem &pr, const float *states, int n_part,
                         long long part_stride, int apply_tokens, float eps, const DwcArg &cv,
                         int focus_p) {
    const int n_chunks = (pr.N + apply_tokens - 1) / apply_tokens, n_wg = n_chunks * pr.B * pr.heads;
    if constexpr (KS != 0) {
        if (conv_takes_ring(KS, cv.kappa_sb != 0, pr.W, pr.N, n_wg)) {
            static LdsLimit lds_limit;
            jv_status st = ensure_lds_limit(lds_limit, (const void *)la_apply_conv_bf16<O_BF16, KS>, kRingMostLds);
            if (st != JV_OK) return st;
            hipLaunchKernelGGL((la_apply_conv_bf16<O_BF16, KS>), dim3(8 * ((n_wg + 7) / 8)), dim3(256), (unsigned)conv_ring_lds(KS, pr.W), stream,
                               pr.q, pr.o, states, n_part, part_stride, pr.heads, pr.N, apply_tokens, n_chunks,
                               n_wg, eps, pr.v, cv, focus_p);
            return launch_status("la_apply_conv_bf16");
        }
    }
    hipLaunchKernelGGL((la_apply_bf16<O_BF16, KS>), dim3(8 * ((n_wg + 7) / 8)), dim3(256), 0, stream,
                       pr.q, pr.o, states, n_part, part_stride, pr.heads, pr.N, apply_tokens, n_chunks,
                       n_wg, eps, pr.v, cv, focus_p);
    return launch_status("la_apply_bf16");
}

jv_status linear_bf16(const Problem &pr, const LinearPlan &plan, float eps, float *ws,
                      const DwcPlan &dwc, int focus_p, hipStream_t stream) {
    static LdsLimit lds_limit[3];
    jv_status st = ensure_lds_limit(lds_limit[0], (const void *)la_state_bf16<false, false>, kStateLds);
    if (st == JV_OK) st = ensure_lds_limit(lds_limit[1], (const void *)la_state_bf16<false, true>, kStateLds);
    if (st == JV_OK) st = ensure_lds_limit(lds_limit[2], (const void *)la_state_bf16<true, true>, kStateLds);
    if (st != JV_OK) return st;
    const int BH = pr.B * pr.heads;
    if (dwc.mode == JV_DWC_NONE && focus_p == 1 && linear_bf16_in_one(BH, pr.N)) {
        static LdsLimit one_limit[2];
        st = ensure_lds_limit(one_limit[pr.o_bf16], pr.o_bf16 ? (const void *)la_fused_bf16<true> : (const void *)la_fused_bf16<false>, kFusedLds);
        if (st != JV_OK) return st;
        const int units = (pr.N + 31) / 32, most = linear_bf16_parts(BH), per = (units + most - 1) / most, parts = (units + per - 1) / per;
        const auto kernel = pr.o_bf16 ? la_fused_bf16<true> : la_fused_bf16<false>;
        hipLaunchKernelGGL(kernel, dim3(8 * ((parts * BH + 7) / 8)), dim3(64 * kFusedWaves), kFusedLds, stream, pr.q, pr.k, pr.v, pr.o, pr.heads,
                           pr.N, per, parts, parts * BH, eps);
        return launch_status("la_fused_bf16");
    }
    const bool dynamic = dwc.mode == JV_DWC_SQUEEZE_DYNAMIC;
    if (dynamic)
        hipLaunchKernelGGL((la_state_bf16<true, true>), dim3(8 * ((plan.n_split * BH + 7) / 8)), dim3(256), kStateLds, stream,
                           pr.k, pr.v, ws, ws + dwc.vsum_off, pr.heads, pr.N, plan.chunk, focus_p, plan.n_split, BH);
    else if (dwc.mode != JV_DWC_NONE)
        hipLaunchKernelGGL((la_state_bf16<false, true>), dim3(8 * ((plan.n_split * BH + 7) / 8)), dim3(256), kStateLds, stream,
                           pr.k, pr.v, ws, (float *)nullptr, pr.heads, pr.N, plan.chunk, focus_p, plan.n_split, BH);
    else
        hipLaunchKernelGGL((la_state_bf16<false, false>), dim3(8 * ((plan.n_split * BH + 7) / 8)), dim3(256), kStateLds, stream,
                           pr.k, pr.v, ws, (float *)nullptr, pr.heads, pr.N, plan.chunk, focus_p, plan.n_split, BH);
    if ((st = launch_status("la_state_bf16")) != JV_OK) return st;
    const float *states = ws;
    int n_part = plan.n_split;
    long long part_stride = (long long)BH * kStateFloats;
    if (plan.combine) {
        float *dst = ws + (size_t)plan.n_split * BH * kStateFloats;
        if ((st = combine_states(ws, dst, dynamic ? ws + dwc.vsum_off : (float *)nullptr, plan.n_split, BH, stream)) != JV_OK) return st;
        states = dst;
        n_part = 1;
    }
    DwcArg cv = {dwc.static_kernel, 0, pr.H, pr.W, pr.P};
    if (dynamic) {
        if ((st = squeeze_generate(dwc, ws, n_part, pr.B, pr.heads, pr.N, stream)) != JV_OK) return st;
        cv.kappa = ws + dwc.kappa_off;
        cv.kappa_sb = (long long)pr.heads * kHeadDim * dwc.ksize * dwc.ksize;
    }
    const int ks = dwc.mode == JV_DWC_NONE ? 0 : dwc.ksize;
    if (pr.o_bf16) {
        if (ks == 0) return launch_apply<true, 0>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
        else if (ks == 3) return launch_apply<true, 3>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
        else return launch_apply<true, 5>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
    } else {
        if (ks == 0) return launch_apply<false, 0>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
        else if (ks == 3) return launch_apply<false, 3>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
        else return launch_apply<false, 5>(stream, pr, states, n_part, part_stride, plan.apply_tokens, eps, cv, focus_p);
    }
}

// ---------------------------------------------------------------------------------------
// The apply pass folded into the output projection that follows a linear-attention block
// (Sec. 3.2.3: the block keeps the projection W_O it inherits).  With o_h = relu(q_h) S_h / den_h,
// den_h = relu(q_h) . z_h + eps, the projected output of a token is
//     sum_h o_h W_O[:, h]^T = sum_h (relu(q_h) / den_h) (W_O[:, h] S_h^T)^T,
// i.e. one product of the scaled queries A'[t, 64 h + i] = relu(q_h[t, i]) / den_h[t] with a
// weight matrix of the image, W'_b[n, 64 h + i] = sum_c W_O[n, 64 h + c] St_bh[c][i]  (St is the
// state as la_state_bf16 stores it, St[c][i] = sum_t relu(k[t, i]) v[t, c]).  Both operands are
// rounded to bf16 once; the product runs on the GEMM with one weight matrix per image.
// ---------------------------------------------------------------------------------------

// grid (C / 64, B*heads), 256 threads: 64 output features n x the 64 columns of head h of W'_b;
// a thread forms a 4 x 4 block of them (two 16-byte LDS reads per 16 multiply-adds), in fp32.
__global__ void __launch_bounds__(256)
la_fold_projection(const float *__restrict__ states, const __bf16 *__restrict__ w_o,
                   __bf16 *__restrict__ w_fold, int heads, int C) {
    __shared__ __align__(16) float St[kHeadDim][kHeadDim + 4];   // [c][i]
    __shared__ __align__(16) float Wt[kHeadDim][kHeadDim + 4];   // [c][n - n0]
    const int tid = threadIdx.x, bh = blockIdx.y, b = bh / heads, h = bh % heads, n0 = blockIdx.x * 64;
    const float *sp = states + (size_t)bh * kStateFloats;
    for (int e = tid; e < kHeadDim * kHeadDim; e += 256) St[e >> 6][e & 63] = sp[e];
    for (int e = tid; e < kHeadDim * kHeadDim; e += 256)
        Wt[e & 63][e >> 6] = (float)w_o[(size_t)(n0 + (e >> 6)) * C + h * kHeadDim + (e & 63)];
    __syncthreads();
    const int nb = (tid >> 4) * 4, ib = (tid & 15) * 4;
    float acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[a][i] = 0.f;
#pragma unroll 8
    for (int c = 0; c < kHeadDim; ++c) {
        const f32x4 w4 = *(const f32x4 *)&Wt[c][nb], s4 = *(const f32x4 *)&St[c][ib];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[a][i] = fmaf(w4[a], s4[i], acc[a][i]);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        u32x2 pk = {pack_bf16x2(acc[a][0], acc[a][1]), pack_bf16x2(acc[a][2], acc[a][3])};
        *(u32x2 *)(w_fold + ((size_t)b * C + n0 + nb + a) * C + h * kHeadDim + ib) = pk;
    }
}

// grid (ceil(B * N * heads / 32)), 256 threads: 8 lanes per (token, head) row of 64 channels, rows in
// the order (batch, token, head), so that a workgroup writes 4 KB of consecutive bytes of a_out.
__global__ void __launch_bounds__(256)
la_scale_queries(TensorArg qt, const float *__restrict__ states, __bf16 *__restrict__ a_out, int heads,
                 int N, long long rows, float eps) {
    const long long row = (long long)blockIdx.x * 32 + (threadIdx.x >> 3);
    if (row >= rows) return;  // all eight lanes of a row together
    const int l8 = threadIdx.x & 7;
    const int h = (int)(row % heads);
    const long long tn = row / heads;
    const int n = (int)(tn % N), b = (int)(tn / N);
    const u32x4 q = relu_bf16x8(ld_stream((const u32x4 *)((const __bf16 *)qt.ptr + b * qt.sb + h * qt.sh + (long long)n * qt.sn + l8 * 8)));
    const float *zp = states + ((size_t)b * heads + h) * kStateFloats + kHeadDim * kHeadDim + l8 * 8;
    const f32x4 z0 = *(const f32x4 *)zp, z1 = *(const f32x4 *)(zp + 4);
    float r[8] = {bf16_lo(q[0]), bf16_hi(q[0]), bf16_lo(q[1]), bf16_hi(q[1]),
                  bf16_lo(q[2]), bf16_hi(q[2]), bf16_lo(q[3]), bf16_hi(q[3])};
    float den = r[0] * z0[0] + r[1] * z0[1] + r[2] * z0[2] + r[3] * z0[3] +
                r[4] * z1[0] + r[5] * z1[1] + r[6] * z1[2] + r[7] * z1[3];
    den += __shfl_xor(den, 1, 64);
    den += __shfl_xor(den, 2, 64);
    den += __shfl_xor(den, 4, 64);
    const float inv = 1.0f / (den + eps);
    u32x4 out = {pack_bf16x2(r[0] * inv, r[1] * inv), pack_bf16x2(r[2] * inv, r[3] * inv),
                 pack_bf16x2(r[4] * inv, r[5] * inv), pack_bf16x2(r[6] * inv, r[7] * inv)};
    st_stream((u32x4 *)(a_out + ((size_t)tn * heads + h) * kHeadDim + l8 * 8), out);
}

// State pass, sum of the partial states into `states` ([B*heads][kStateFloats], one per head),
// then the two operands of the fused projection: w_fold [B][C][C] and a_out [B*N][C], C = 64 heads.
// ws: the linear-attention workspace (the partial states).  64-channel heads, ReLU map, no
// convolution branch (the caller checks).
jv_status linear_fused_projection_operands(const Problem &pr, float eps, float *ws, float *states,
                                           const void *w_o, void *w_fold, void *a_out, hipStream_t stream) {
    static LdsLimit lds_limit;
    jv_status st = ensure_lds_limit(lds_limit, (const void *)la_state_bf16<false, false>, kStateLds);
    if (st != JV_OK) return st;
    const LinearPlan plan = plan_linear(pr.B, pr.heads, pr.N);
    const int BH = pr.B * pr.heads, C = pr.heads * kHeadDim;
    hipLaunchKernelGGL((la_state_bf16<false, false>), dim3(8 * ((plan.n_split * BH + 7) / 8)), dim3(256), kStateLds, stream,
                       pr.k, pr.v, ws, (float *)nullptr, pr.heads, pr.N, plan.chunk, 1, plan.n_split, BH);
    if ((st = launch_status("la_state_bf16")) != JV_OK) return st;
    if ((st = combine_states(ws, states, nullptr, plan.n_split, BH, stream)) != JV_OK) return st;
    hipLaunchKernelGGL(la_fold_projection, dim3(C / 64, BH), dim3(256), 0, stream, states, (const __bf16 *)w_o,
                       (__bf16 *)w_fold, pr.heads, C);
    if ((st = launch_status("la_fold_projection")) != JV_OK) return st;
    const long long rows = (long long)pr.B * pr.N * pr.heads;
    hipLaunchKernelGGL(la_scale_queries, dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, stream, pr.q, states,
                       (__bf16 *)a_out, pr.heads, pr.N, rows, eps);
    return launch_status("la_scale_queries");
}

// ---------------------------------------------------------------------------------------
// head_dim 128.  la_state_wide_bf16 (below) leaves four 64 x 64 quadrant states per head,
// la_combine_wide sums the partial ones, and the one that has the whole sum leaves it as operands of the apply pass: every number as a bf16
// high part and the bf16 rest, per quadrant kStateFloats * 4 bytes: St hi, St lo, z hi [64], z lo [64].  St[c2][c1] lies where that pass's
// operands take it, whose loads and the stores here then cover whole lines: eight c1 of a lane, lanes, k-steps of 16 c1, blocks
// of 32 c2 (wide_state_at).  (As rows of c1 every instruction touched 32 of them: 64 x 196 tokens x 8 heads 43.7 us.)  The apply pass:
//   o[c2] = sum_i relu(q_i) S_ij[:, c2] / (sum_i relu(q_i) . z_i + eps),   j = c2 / 64,
// q_i the two 64-channel halves of a query row.  A workgroup streams one token chunk of one
// (batch, head); its four wavefronts own the four 32-channel quarters of the output, each with
// the matching rows of S_0j^T and S_1j^T as bf16 high + low operands in registers (what a
// wavefront of the 64-channel kernel holds for its 64 output channels), and all four run over
// the same 64-token query tile in LDS; the denominator is one more row block, as there.
// KS = 3 or 5: the block's convolution branch is added before the store, as in la_apply_bf16:
// the normalised tile is staged as fp32 (512-byte token rows, the 16-byte chunk index rotated
// by the row), and the thread that stores 8 channels of 4 consecutive tokens first adds
// sum_taps kappa[c][tap] * V[token + tap][c] for them; the sum is rounded once.
// grid (n_chunks * B*heads), 256 threads.
// ---------------------------------------------------------------------------------------
// Position of St[32 block + li][16 ks + 8 g + e] in a state.
__device__ inline int wide_state_at(int block, int ks, int g, int li, int e) { return ((block * 4 + ks) * 64 + g * 32 + li) * 8 + e; }
__device__ inline void store_pairs(unsigned char *hi, unsigned char *lo, f32x4 x) {
    const u32x2 h = {pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])};
    *(u32x2 *)hi = h;
    *(u32x2 *)lo = u32x2{pack_bf16x2(x[0] - bf16_lo(h[0]), x[1] - bf16_hi(h[0])), pack_bf16x2(x[2] - bf16_lo(h[1]), x[3] - bf16_hi(h[1]))};
}

template <bool O_BF16, int KS>
__global__ void __launch_bounds__(256, 2)
la_apply_wide_bf16(TensorArg qt, TensorArg ot, const float *__restrict__ states, int heads, int N,
                   int tokens_per_wg, int n_chunks, float eps, TensorArg vt, DwcArg cv) {
    // ring of query tiles [64 tokens][256 B], one with the convolution; output tile (bf16 rows of 256 B, or fp32 rows of 512 B with
    // the convolution); the filters as [tap][channel]
    constexpr int kOutBytes = KS ? 32768 : 16384, kSlots = KS ? 1 : 4, kTile = 16384;
    __shared__ __align__(16) unsigned char smem[kSlots * kTile + kOutBytes + KS * KS * kHeadDimWide * 4];
    unsigned char *otile = smem + kSlots * kTile;
    float *kap = (float *)(smem + kSlots * kTile + kOutBytes);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = lane >> 5, li = lane & 31;
    const int bh = blockIdx.x / n_chunks, b = bh / heads, h = bh % heads;
    const __bf16 *qp = (const __bf16 *)qt.ptr + b * qt.sb + h * qt.sh;
    const int n0 = (blockIdx.x % n_chunks) * tokens_per_wg, n1 = min(N, n0 + tokens_per_wg);
    const int frow = tid >> 4, fchunk = tid & 15;  // this thread's 16 bytes of rows frow + 16 r of a tile
    const int n_tile = (n1 - n0 + 63) / 64;

    // The next query tile.  Without the convolution tiles go from global memory straight into LDS, the first four before anything
    // else is waited for, so that memory works under the start (8 x 4 096 tokens x 8 heads 70.1 -> 67.6 us for both passes).  A wavefront moves rows 16 r + 4 wave +
    // lane / 16 (r < 4); the lane fetches the chunk that belongs in its slot of the row (wide_off_row).  Rows past the range
    // are its last one again, so that all wavefronts issue the same loads.  With the convolution, whose waits for V would wait for them too (and
    // whose output tile leaves no room), one tile passes through registers.
    auto issue = [&](int tile) {
        unsigned char *to = smem + (tile % kSlots) * kTile;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row0 = 16 * r + 4 * wave, row = row0 + (lane >> 4), n = min(n0 + 64 * tile + row, n1 - 1);
            const __bf16 *from = qp + (long long)n * qt.sn + ((lane & 15) ^ (row & 15)) * 8;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                             (__attribute__((address_space(3))) void *)(to + row0 * 256), 16, 0, kDmaStreamAux);
        }
    };
    u32x4 qreg[4];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = t0 + 16 * r + frow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            qreg[r] = zero;
            if (n < n1) qreg[r] = ld_stream((const u32x4 *)(qp + (long long)n * qt.sn + fchunk * 8));
        }
    };
    if (KS) fetch(n0);
    if (KS) {  // (read after the first barrier of the token loop)
        const float *kbase = cv.kappa + b * cv.kappa_sb + (size_t)h * kHeadDimWide * KS * KS;
        for (int e = tid; e < kHeadDimWide * KS * KS; e += 256) kap[(e % (KS * KS)) * kHeadDimWide + e / (KS * KS)] = kbase[e];
    }

    // A operands: rows c2 of S_ij^T (this wavefront's quarter), k-slots c1 = 16 ks + 8 g + (0..7).
    const int j = wave >> 1;
    bf16x8 s_hi[2][4], s_lo[2][4], z_op[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const unsigned char *st = (const unsigned char *)(states + ((size_t)bh * 4 + 2 * i + j) * kStateFloats);
        constexpr int kZ = kHeadDim * kHeadDim;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const unsigned char *row = st + 2 * wide_state_at(wave & 1, ks, g, li, 0);
            s_hi[i][ks] = as_bf16x8(*(const u32x4 *)row);
            s_lo[i][ks] = as_bf16x8(*(const u32x4 *)(row + 2 * kZ));
            z_op[i][ks] = as_bf16x8(*(const u32x4 *)(st + 4 * kZ + 2 * kHeadDim * (li & 1) + 2 * (16 * ks + 8 * g)));
        }
    }
    // (behind the loads of the states, and of a number known to the compiler, so that it can wait for the states alone: tiles past
    // the range are its last row again)
    if (!KS) {
#pragma unroll
        for (int tile = 0; tile < kSlots; ++tile) issue(tile);
    }
    // denominator block: row 0 = z high part, row 1 = z low part, other rows zero
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            if (li >= 2) z_op[i][ks] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});

    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh;
    unsigned qaddr[8];  // this lane's operands of a tile's first 32 tokens in slot 0
#pragma unroll
    for (int c = 0; c < 8; ++c) qaddr[c] = lds_address(smem) + wide_off_row(li, 2 * c + g);
    for (int tile = 0; tile < n_tile; ++tile) {
        const int t = n0 + 64 * tile;
        if (KS) {
            __syncthreads();  // the previous tile has been read, and its output rows stored
#pragma unroll
            for (int r = 0; r < 4; ++r) *(u32x4 *)(smem + wide_off_row(16 * r + frow, fchunk)) = relu_bf16x8(qreg[r]);
            if (t + 64 < n1) fetch(t + 64);
            __syncthreads();
        } else {
            // This tile has landed; at most the three issued behind it may be on their way (stores in between count too: the
            // wait is then a little stricter).
            const int behind = min(kSlots - 1, max(kSlots, n_tile) - 1 - tile);
            if (behind == 3) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
            else if (behind == 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
            else if (behind == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();  // ... for every wavefront, and the output rows before have been read
        }
        const unsigned slot = (unsigned)(tile % kSlots) * kTile;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            if (t + 32 * nt >= n1) break;  // the same for every wavefront of the workgroup
            f32x16 acc, accz;
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[v] = 0.f; accz[v] = 0.f; }
            u32x4 qb[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) qb[c] = nt ? lds_read_b128_at<32 * 256>(qaddr[c] + slot) : lds_read_b128_at<0>(qaddr[c] + slot);
            lds_reads_landed(qb[0], qb[1], qb[2], qb[3]);
            lds_reads_landed(qb[4], qb[5], qb[6], qb[7]);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const bf16x8 q = as_bf16x8(KS ? qb[4 * i + ks] : relu_bf16x8(qb[4 * i + ks]));
                    accz = mfma32(z_op[i][ks], q, accz);
                    acc = mfma32(s_lo[i][ks], q, acc);
                    acc = mfma32(s_hi[i][ks], q, acc);
                }
            // den lives in rows 0 and 1 of the denominator block: registers 0, 1 of lanes g = 0.
            float den_lo, den_hi;
            pair_values(accz[0] + accz[1], &den_lo, &den_hi);
            const float inv = __builtin_amdgcn_rcpf(den_lo + eps);
            if (KS) {
                const int row = 32 * nt + li;
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x4 val = {acc[4 * q4] * inv, acc[4 * q4 + 1] * inv, acc[4 * q4 + 2] * inv, acc[4 * q4 + 3] * inv};
                    *(f32x4 *)(otile + row * 512 + (((8 * wave + 2 * q4 + g) ^ (row & 15)) << 4)) = val;
                }
            } else if (O_BF16) {
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    u32x2 pk = {pack_bf16x2(acc[4 * q4] * inv, acc[4 * q4 + 1] * inv),
                                pack_bf16x2(acc[4 * q4 + 2] * inv, acc[4 * q4 + 3] * inv)};
                    *(u32x2 *)(otile + wide_off_row(32 * nt + li, 4 * wave + q4) + 8 * g) = pk;
                }
            } else {
                const int n = t + 32 * nt + li;
                float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh;
                if (n < n1) {
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        f32x4 val = {acc[4 * q4] * inv, acc[4 * q4 + 1] * inv, acc[4 * q4 + 2] * inv, acc[4 * q4 + 3] * inv};
                        *(f32x4 *)(op + (long long)n * ot.sn + 32 * wave + 8 * q4 + 4 * g) = val;
                    }
                }
            }
        }
        if (KS) {
            __syncthreads();  // the four quarters of every row are in the output tile, and the query tile has been read
            // This thread finishes channels 8 fchunk .. + 7 of tokens tok0 .. tok0 + 3: the taps of
            // neighbouring tokens overlap, so one tap row needs 4 + KS - 1 loads instead of 4 * KS.
            // Out-of-grid taps (and tokens past the end of the range) read a valid row with
            // weight zero, so the loads of a tap row are all in flight at once.
            constexpr int kPad = KS / 2, kSpan = 4 + KS - 1;
            const int tok0 = t + 4 * frow, last = n1 - 1;
            float sum[4][8];
            int gr[4], gc[4];
            bool on_grid[4];  // prefix tokens (grid index below zero) get no convolution term
            {
                const int g0 = min(tok0, last) - cv.P;  // grid index of the thread's first token
                const int base = max(g0, 0);
                int r0 = base / cv.W, c0 = base - r0 * cv.W;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int orow = 4 * frow + r;
                    const f32x4 o0 = *(const f32x4 *)(otile + orow * 512 + (((2 * fchunk) ^ (orow & 15)) << 4));
                    const f32x4 o1 = *(const f32x4 *)(otile + orow * 512 + (((2 * fchunk + 1) ^ (orow & 15)) << 4));
                    sum[r][0] = o0[0]; sum[r][1] = o0[1]; sum[r][2] = o0[2]; sum[r][3] = o0[3];
                    sum[r][4] = o1[0]; sum[r][5] = o1[1]; sum[r][6] = o1[2]; sum[r][7] = o1[3];
                    gr[r] = r0;
                    gc[r] = c0;
                    on_grid[r] = g0 + r >= 0;
                    if (on_grid[r] && ++c0 == cv.W) { c0 = 0; ++r0; }
                }
            }
#pragma unroll 1
            for (int di = -kPad; di <= kPad; ++di) {
                u32x4 vv[kSpan];
#pragma unroll
                for (int jj = 0; jj < kSpan; ++jj) {
                    const int src = tok0 + jj - kPad + di * cv.W;  // token of column jj in this tap row
                    const int safe = min(max(src, 0), N - 1);
                    vv[jj] = *(const u32x4 *)(vp + (long long)safe * vt.sn + fchunk * 8);
                }
                const float *krow = kap + (di + kPad) * KS * kHeadDimWide + 8 * fchunk;
#pragma unroll
                for (int dj = -kPad; dj <= kPad; ++dj) {
                    const f32x4 k0 = *(const f32x4 *)(krow + (dj + kPad) * kHeadDimWide);
                    const f32x4 k1 = *(const f32x4 *)(krow + (dj + kPad) * kHeadDimWide + 4);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool ok = tok0 + r <= last && on_grid[r] && (unsigned)(gr[r] + di) < (unsigned)cv.H &&
                                        (unsigned)(gc[r] + dj) < (unsigned)cv.W;
                        const float m = ok ? 1.0f : 0.0f;
                        const u32x4 x = vv[r + dj + kPad];
                        sum[r][0] = fmaf(k0[0] * m, bf16_lo(x[0]), sum[r][0]);
                        sum[r][1] = fmaf(k0[1] * m, bf16_hi(x[0]), sum[r][1]);
                        sum[r][2] = fmaf(k0[2] * m, bf16_lo(x[1]), sum[r][2]);
                        sum[r][3] = fmaf(k0[3] * m, bf16_hi(x[1]), sum[r][3]);
                        sum[r][4] = fmaf(k1[0] * m, bf16_lo(x[2]), sum[r][4]);
                        sum[r][5] = fmaf(k1[1] * m, bf16_hi(x[2]), sum[r][5]);
                        sum[r][6] = fmaf(k1[2] * m, bf16_lo(x[3]), sum[r][6]);
                        sum[r][7] = fmaf(k1[3] * m, bf16_hi(x[3]), sum[r][7]);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int on = tok0 + r;
                if (on <= last) {
                    if (O_BF16) {
                        __bf16 *op = (__bf16 *)ot.ptr + b * ot.sb + h * ot.sh;
                        u32x4 pk = {pack_bf16x2(sum[r][0], sum[r][1]), pack_bf16x2(sum[r][2], sum[r][3]),
                                    pack_bf16x2(sum[r][4], sum[r][5]), pack_bf16x2(sum[r][6], sum[r][7])};
                        st_stream((u32x4 *)(op + (long long)on * ot.sn + fchunk * 8), pk);
                    } else {
                        float *op = (float *)ot.ptr + b * ot.sb + h * ot.sh + (long long)on * ot.sn + fchunk * 8;
                        f32x4 s0 = {sum[r][0], sum[r][1], sum[r][2], sum[r][3]};
                        f32x4 s1 = {sum[r][4], sum[r][5], sum[r][6], sum[r][7]};
                        *(f32x4 *)op = s0;
                        *(f32x4 *)(op + 4) = s1;
                    }
                }
            }
        } else {
            lds_barrier();  // the four quarters of every row are in the output tile, and the query tile has been read
            if (O_BF16) {
                __bf16 *op = (__bf16 *)ot.ptr + b * ot.sb + h * ot.sh;
                u32x4 val[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) val[r] = lds_read_b128_ordered(lds_address(otile) + wide_off_row(16 * r + frow, fchunk));
                lds_reads_landed(val[0], val[1], val[2], val[3]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int n = t + 16 * r + frow;
                    if (n < n1) st_stream((u32x4 *)(op + (long long)n * ot.sn + fchunk * 8), val[r]);
                }
            }
        }
        if (!KS && tile + kSlots < n_tile) issue(tile + kSlots);
    }
    if (!KS && n_tile < kSlots) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (nothing may land in the LDS of the next workgroup)
}

// State pass for heads of 128 channels: S = relu(K)^T V (128 x 128) and z = sum relu(K) of one
// token chunk, K and V read once.  TEAMS (1, 2) teams of four wavefronts take tiles of 64 tokens in turn, which each
// shares in LDS of its own -- K (rectified) and V, each as two half tiles of 64 channels in the tile_off_tr layout --
// and wavefront 2i + j of a team accumulates the quadrant S_ij = relu(K_i)^T V_j (channels 64i .. 64i+63
// of K against 64j .. 64j+63 of V) exactly as la_state_bf16 accumulates its one state, and z_i.
// Two tile buffers: the next tile is fetched into registers while this one is reduced, and
// stored after it; one barrier per tile.  At the end two teams' sums meet in LDS, each team adding up and storing
// the half for one block of 32 K channels.  The quadrants are written as four states of
// kStateFloats floats, quadrant 2i + j of (batch, head) bh at index 4 bh + 2i + j of `part`.
// Bound by memory, the states among it (66 KB a workgroup, written here and read by the sum): with one team there are twice as
// many, 34 MB beside 67 MB of K and V for 16 384 tokens x 8 heads (both passes, with the sum's and the states' present form, 46.9 -> 41.6 us, with the convolution 84 -> 68; 32 x 1 369 x 8 heads 94 -> 81).
// Where two teams would leave as many states, two workgroups of one team overlap each other's start and end: 64 x 196
// tokens x 8 heads 37.7 with one team, 42.0 with two (states as rows).
// VSUM: also write the chunk's token sum of V (the input of the dynamic-filter generator of the
// block's convolution branch) to vsum[part][bh][128]; it falls out of the V operands of the
// wavefronts with i = 0.
// grid (n_split, B*heads), 256 TEAMS threads, TEAMS * kStateWideTeamLds bytes of dynamic LDS.
constexpr int kStateWideTeamLds = 2 * 4 * 8192;

template <bool VSUM, int TEAMS>
__global__ void __launch_bounds__(256 * TEAMS, 2)
la_state_wide_bf16(TensorArg kt, TensorArg vt, float *__restrict__ ws, float *__restrict__ vsum, int heads, int N,
                   int chunk) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), tid = threadIdx.x & 255, wave = tid >> 6, lane = tid & 63;
    unsigned char *smem = lds + team * kStateWideTeamLds;
    const int bh = blockIdx.y, b = bh / heads, h = bh % heads, part = blockIdx.x;
    const int BH = gridDim.y;
    const __bf16 *kp = (const __bf16 *)kt.ptr + b * kt.sb + h * kt.sh;
    const __bf16 *vp = (const __bf16 *)vt.ptr + b * vt.sb + h * vt.sh;
    const int n0 = part * chunk, n1 = min(N, n0 + chunk);
    // loads: 16 threads per token row (one 16-byte chunk each), 16 rows per pass, 4 passes per tile
    const int lrow = tid >> 4, lchunk = tid & 15;
    const int qi = wave >> 1, qj = wave & 1;

    f32x16 acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;
    float zacc[2] = {0.f, 0.f}, vacc[2] = {0.f, 0.f};

    u32x4 kreg[4], vreg[4];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = t0 + r * 16 + lrow;
            u32x4 zero = {0u, 0u, 0u, 0u};
            kreg[r] = zero;
            vreg[r] = zero;
            if (n < n1) {
                kreg[r] = ld_stream((const u32x4 *)(kp + (long long)n * kt.sn + lchunk * 8));
                vreg[r] = ld_stream((const u32x4 *)(vp + (long long)n * vt.sn + lchunk * 8));
            }
        }
    };
    auto stash = [&](int buf) {
        unsigned char *kt0 = smem + buf * 32768 + (lchunk >> 3) * 8192, *vt0 = kt0 + 16384;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const unsigned off = tile_off_tr(r * 16 + lrow, lchunk & 7);
            *(u32x4 *)(kt0 + off) = relu_bf16x8(kreg[r]);
            *(u32x4 *)(vt0 + off) = vreg[r];
        }
    };

    int buf = 0;
    int t = n0 + 64 * team;
    if (t < n1) fetch(t);
    for (int t0 = n0; t0 < n1; t0 += 64 * TEAMS, t += 64 * TEAMS) {
        if (t < n1) stash(buf);
        __syncthreads();
        if (t >= n1) break;  // (the second team, behind its last tile: the loop's last round)
        if (t + 64 * TEAMS < n1) fetch(t + 64 * TEAMS);
        const unsigned char *ktile = smem + buf * 32768 + qi * 8192;
        const unsigned char *vtile = smem + buf * 32768 + 16384 + qj * 8192;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 a[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = load_tr_operand(ktile, 16 * ks, i, lane);
                bv[i] = load_tr_operand(vtile, 16 * ks, i, lane);
            }
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                u32x4 au = as_u32x4(a[mi]);
#pragma unroll
                for (int w = 0; w < 4; ++w) zacc[mi] = add_bf16x2(au[w], zacc[mi]);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) acc[mi][ni] = mfma32(a[mi], bv[ni], acc[mi][ni]);
            }
            if (VSUM && qi == 0) {  // wave-uniform
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) {
                    u32x4 bu = as_u32x4(bv[ni]);
#pragma unroll
                    for (int w = 0; w < 4; ++w) vacc[ni] = add_bf16x2(bu[w], vacc[ni]);
                }
            }
        }
        buf ^= 1;
    }

    // St[c2][c1] (c2: channel of V_j, c1: channel of K_i), then z_i[c1]: straight from the registers
    // (8 KB per wavefront and block of 32 K channels, once per chunk); as pairs where there is one chunk.
    auto store = [&](auto block_tag) __attribute__((always_inline)) {
        constexpr int mi = decltype(block_tag)::value;
        float *out = ws + ((size_t)part * BH * 4 + (size_t)bh * 4 + wave) * kStateFloats;
        const int g = lane >> 5, li = lane & 31;
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int at = wide_state_at(ni, 2 * mi + q4 / 2, q4 % 2, li, 4 * g);  // c1 = 32 mi + 8 q4 + 4 g .. + 3
                f32x4 val = {acc[mi][ni][4 * q4], acc[mi][ni][4 * q4 + 1], acc[mi][ni][4 * q4 + 2],
                             acc[mi][ni][4 * q4 + 3]};
                unsigned char *to = (unsigned char *)out + 2 * at;
                if (gridDim.x == 1) store_pairs(to, to + 2 * kHeadDim * kHeadDim, val);
                else *(f32x4 *)(out + at) = val;
            }
        float lo, hi;
        pair_values(zacc[mi], &lo, &hi);  // the two halves of the tokens
        const float z = lo + hi;
        if (g == 0 && gridDim.x == 1) {
            __bf16 *to = (__bf16 *)(out + kHeadDim * kHeadDim) + 32 * mi + li;
            to[0] = (__bf16)z;
            to[kHeadDim] = (__bf16)(z - (float)(__bf16)z);
        } else if (g == 0) {
            out[kHeadDim * kHeadDim + 32 * mi + li] = z;
        }
        if (VSUM && qi == 0) {
            pair_values(vacc[mi], &lo, &hi);
            if (g == 0) vsum[((size_t)part * BH + bh) * kHeadDimWide + kHeadDim * qj + 32 * mi + li] = lo + hi;
        }
    };
    if constexpr (TEAMS == 1) {
        store(std::integral_constant<int, 0>());
        store(std::integral_constant<int, 1>());
    } else {
        // The other team's sums: this team keeps block `team` of K channels and hands over the other.
        constexpr int kHandOver = (32 + 1 + 1) * 64 * 4;  // a wavefront's: acc[.][0 .. 1], z, token sums of V
        static_assert(4 * kHandOver <= kStateWideTeamLds, "");
        __syncthreads();  // both teams have read their last tiles
        float *out_sums = (float *)(lds + (team ^ 1) * kStateWideTeamLds + wave * kHandOver) + lane;
        const float *in_sums = (const float *)(smem + wave * kHandOver) + lane;
        auto keep = [&](auto mine_tag) __attribute__((always_inline)) {
            constexpr int mine = decltype(mine_tag)::value, other = 1 - mine;
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) out_sums[64 * (16 * ni + v)] = acc[other][ni][v];
            out_sums[64 * 32] = zacc[other];
            out_sums[64 * 33] = vacc[other];
            __syncthreads();
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mine][ni][v] += in_sums[64 * (16 * ni + v)];
            zacc[mine] += in_sums[64 * 32];
            vacc[mine] += in_sums[64 * 33];
            store(mine_tag);
        };
        if (team == 0) keep(std::integral_constant<int, 0>());
        else keep(std::integral_constant<int, 1>());
    }
}

// Sum of the partial states of wide heads, as pairs.  Sixteen partials in flight: the sum of 32 is two round trips (7.7 -> 4.7 us for
// half as many of 8 heads as with eight in flight).  grid (quadrants, ceil(kStateFloats / 256)), 64 threads.
__global__ void __launch_bounds__(64)
la_combine_wide(const float *__restrict__ ws, unsigned char *__restrict__ dst, int n_split, int quadrants) {
    const int e4 = blockIdx.y * 64 + threadIdx.x;  // 16-byte piece of a state
    constexpr int kVec = kStateFloats / 4, kZ = kHeadDim * kHeadDim;
    if (e4 >= kVec) return;
    const f32x4 *src = (const f32x4 *)ws + (size_t)blockIdx.x * kVec + e4;
    const size_t stride4 = (size_t)quadrants * kVec;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < n_split; p0 += 16) {
        f32x4 part[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            part[i] = p0 + i < n_split ? src[(size_t)(p0 + i) * stride4] : zero;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += part[i];
    }
    const int e = 4 * e4;
    unsigned char *to = dst + (size_t)blockIdx.x * (kStateFloats * 4) + (e < kZ ? 2 * e : 4 * kZ + 2 * (e - kZ));
    store_pairs(to, to + (e < kZ ? 2 * kZ : 2 * kHeadDim), sum);
}

LinearPlan plan_linear_wide(int B, int heads, int N) {
    LinearPlan p = plan_linear(B, heads, N);
    // Several chunks: workgroups of two teams, one per compute unit, at least 256 tokens each, where those are fewer than
    // plan_linear has, whose states size the workspace.
    if (p.n_split > 1) {
        const long long bh = (long long)B * heads;
        long long want = (256 + bh - 1) / bh, most = (N + 255) / 256;
        want = want < most ? want : most;
        want = want < 64 ? want : 64;
        p.chunk = (int)(((N + want - 1) / want + 255) / 256 * 256);
        p.n_split = (N + p.chunk - 1) / p.chunk;
    }
    p.combine = p.n_split > 1;  // the apply pass reads one state per quadrant
    // (the token chunks of the apply pass follow from B * heads as in plan_linear; every workgroup
    // loads its head's state once, 64 KB)
    return p;
}
size_t linear_wide_workspace_floats(int B, int heads, int N) {
    LinearPlan p = plan_linear(B, heads, N);
    p.combine = p.n_split > 1;
    return linear_workspace_floats(p, B, 4 * heads);
}
jv_status linear_wide_state(const Problem &pr, float *ws, float *vsum, hipStream_t stream) {
    if (4ll * pr.B * pr.heads > 65535) return fail(JV_ERR_UNSUPPORTED, "head_dim 128: batch * heads above 16383");
    const LinearPlan plan = plan_linear_wide(pr.B, pr.heads, pr.N);
    auto launch = [&](auto vsum_tag, auto teams_tag) {
        constexpr bool VSUM = decltype(vsum_tag)::value;
        constexpr int TEAMS = decltype(teams_tag)::value;
        static LdsLimit lds_limit;
        const jv_status st = ensure_lds_limit(lds_limit, (const void *)la_state_wide_bf16<VSUM, TEAMS>, TEAMS * kStateWideTeamLds);
        if (st != JV_OK) return st;
        hipLaunchKernelGGL((la_state_wide_bf16<VSUM, TEAMS>), dim3(plan.n_split, (unsigned)(pr.B * pr.heads)), dim3(256 * TEAMS),
                           TEAMS * kStateWideTeamLds, stream, pr.k, pr.v, ws, vsum, pr.heads, pr.N, plan.chunk);
        return launch_status("la_state_wide_bf16");
    };
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    const bool teams = plan_linear(pr.B, pr.heads, pr.N).n_split > plan.n_split;  // (where they leave fewer states)
    if (vsum) return teams ? launch(std::true_type(), two) : launch(std::true_type(), one);
    return teams ? launch(std::false_type(), two) : launch(std::false_type(), one);
}

jv_status linear_wide_apply(const Problem &pr, float eps, float *ws, hipStream_t stream, int ksize, const DwcArg *cv) {
    jv_status st;
    const LinearPlan plan = plan_linear_wide(pr.B, pr.heads, pr.N);
    const long long BHv = 4ll * pr.B * pr.heads;  // quadrant states
    const float *states = ws;
    if (plan.combine) {
        float *dst = ws + (size_t)plan.n_split * BHv * kStateFloats;
        hipLaunchKernelGGL(la_combine_wide, dim3((unsigned)BHv, (kStateFloats + 255) / 256), dim3(64), 0, stream, ws, (unsigned char *)dst,
                           plan.n_split, (int)BHv);
        if ((st = launch_status("la_combine_wide")) != JV_OK) return st;
        states = dst;
    }
    const int n_chunks = (pr.N + plan.apply_tokens - 1) / plan.apply_tokens;
    const long long n_wg = (long long)n_chunks * pr.B * pr.heads;
    if (n_wg >= (1ll << 31)) return fail(JV_ERR_UNSUPPORTED, "head_dim 128: too many token chunks");
    const DwcArg none = {nullptr, 0, pr.H, pr.W, pr.P};
    auto launch = [&](auto bf_tag, auto ks_tag) {
        constexpr bool O_BF16 = decltype(bf_tag)::value;
        constexpr int KS = decltype(ks_tag)::value;
        hipLaunchKernelGGL((la_apply_wide_bf16<O_BF16, KS>), dim3((unsigned)n_wg), dim3(256), 0, stream, pr.q, pr.o, states,
                           pr.heads, pr.N, plan.apply_tokens, n_chunks, eps, pr.v, KS ? *cv : none);
    };
    const int ks = cv ? ksize : 0;
    if (pr.o_bf16) {
        if (ks == 0) launch(std::true_type(), std::integral_constant<int, 0>());
        else if (ks == 3) launch(std::true_type(), std::integral_constant<int, 3>());
        else launch(std::true_type(), std::integral_constant<int, 5>());
    } else {
        if (ks == 0) launch(std::false_type(), std::integral_constant<int, 0>());
        else if (ks == 3) launch(std::false_type(), std::integral_constant<int, 3>());
        else launch(std::false_type(), std::integral_constant<int, 5>());
    }
    return launch_status("la_apply_wide_bf16");
}

jv_status linear_wide_bf16(const Problem &pr, float eps, float *ws, hipStream_t stream) {
    jv_status st = linear_wide_state(pr, ws, nullptr, stream);
    return st == JV_OK ? linear_wide_apply(pr, eps, ws, stream, 0, nullptr) : st;
}

}  // namespace jv
