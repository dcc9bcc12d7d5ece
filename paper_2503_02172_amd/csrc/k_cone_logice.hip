// Operator kernels of the two cone / fuzzy-logic models the paper benchmarks
// beside BetaE (Experiments, Baselines; Table 1: ConE and LogicE). Their
// projections share BetaE's plan (per-hop MLP passes on the MFMA GEMM, with
// the first hop's first layer from precomputed tables); what differs, and
// lives here, is each model's state, negation, intersection and packing for
// the scorer.
//
// ConE   state [theta; psi]: per dimension a sector cone with axis theta in
//        [-pi, pi) and half-aperture psi in [0, pi]; an entity is a cone of
//        aperture 0.
//          projection  x = [theta + theta_r; psi + psi_r] -> 3 dense layers ->
//                      theta = pi tanh(y), psi = pi/2 (tanh(2 y') + 1)
//                      (the output maps run in the last layer's epilogue)
//          negation    the complementary cone: theta - pi (theta >= 0) or
//                      theta + pi, and pi - psi
//          intersection u_j = [theta_j - psi_j; theta_j + psi_j]; attention
//                      logits W2 ReLU(W1 u_j + b1) + b2 (2d -> d -> d),
//                      softmax across branches per dimension, axis = angle
//                      of sum_j w_j (cos theta_j, sin theta_j); psi =
//                      min_j psi_j * sigmoid(W4 mean_j ReLU(W3 u_j + b3) + b4).
//                      Both first layers read u_j: they run as one GEMM with
//                      the two weight matrices stacked ([W1; W3], 2d -> 2d).
// LogicE state [l; u]: lower and upper truth bounds in [0, 1], l <= u.
//          projection  x = [l; u; Rel[r]] (width 3d) -> 3 dense layers ->
//                      l = sigmoid(y_l), u = l + sigmoid(y_u) (1 - l)
//                      (sigmoid in the GEMM epilogue, the bound map after it)
//          negation    [l; u] -> [1 - u; 1 - l]
//          intersection a t-norm over the branches, coordinate-wise on the
//                      lower and on the upper bounds (product, minimum or
//                      Lukasiewicz max(0, a + b - 1)), folded from the first
//                      branch on.
// Negation is never a kernel of its own: the plan marks the edges that read
// a negated value (an intersection input, a projection source, a scored
// row), and the reading kernel applies it.
#include <algorithm>

#include "kgq_internal.hpp"
#include "mfma_tile.hpp"

namespace kgq {

constexpr float kPi = 3.14159265358979323846f;

// ConE complement of one dimension's cone.
__device__ __forceinline__ void cone_negate(float& theta, float& psi)
{
    theta = theta >= 0.f ? theta - kPi : theta + kPi;
    psi = kPi - psi;
}

__device__ __forceinline__ int32_t checked_id_cl(int32_t id, int64_t n, int* flag)
{
    if (id < 0 || (int64_t)id >= n) {
        atomicOr(flag, kErrRange);
        return 0;
    }
    return id;
}

// ---------------------------------------------------------------------------
// Load time
// ---------------------------------------------------------------------------

// ConE entity tables: the anchor state [theta; 0] row-major [N x 2d], and the
// scorer's blocked table [block][k][sin(theta/2) (256) | cos(theta/2) (256)]
// (zero past N). The half-angle sines and cosines are computed once here in
// double precision.
__global__ __launch_bounds__(256) void k_cone_entity_prep(const float* src, int64_t N, int d, int64_t n_pad,
                                                          float* ent_rm, float* blocked)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_pad) return;
    const int64_t blk = e / kEntBlock;
    const int lo = (int)(e % kEntBlock);
    float* dst = blocked + blk * (int64_t)d * 2 * kEntBlock + lo;
    for (int k = 0; k < d; ++k) {
        float s = 0.f, c = 0.f;
        if (e < N) {
            const float th = src[e * d + k];
            ent_rm[e * 2 * d + k] = th;
            ent_rm[e * 2 * d + d + k] = 0.f;
            s = (float)sin(0.5 * (double)th);
            c = (float)cos(0.5 * (double)th);
        }
        dst[(int64_t)k * 2 * kEntBlock] = s;
        dst[(int64_t)k * 2 * kEntBlock + kEntBlock] = c;
    }
}

void launch_cone_entity_prep(const float* src, int64_t N, int d, int64_t n_blocks, float* ent_rm, float* blocked,
                             hipStream_t s)
{
    const int64_t n_pad = n_blocks * kEntBlock;
    hipLaunchKernelGGL(k_cone_entity_prep, dim3((unsigned)((n_pad + 255) / 256)), dim3(256), 0, s, src, N, d, n_pad,
                       ent_rm, blocked);
}

// ---------------------------------------------------------------------------
// Projection inputs (hops whose source is not an anchor, or is negated)
// ---------------------------------------------------------------------------

// x row m: ConE (width 2d) the source state (complemented where neg[m]) plus
// Rel[r]; LogicE (width 3d) [source (complemented where neg[m]); Rel[r]].
template <int MODEL>
__global__ __launch_bounds__(1024) void k_mlp_proj_prep(const int32_t* src_row, const int32_t* anchor_ref,
                                                       const int32_t* rel_ref, const int32_t* neg,
                                                       const int32_t* anchors, const int32_t* rels,
                                                       const float* states, const float* ent_rm, const float* rel,
                                                       int64_t n_ent, int n_rel, int d, float* x, int* flag)
{
    const int m = blockIdx.x;
    const int W = 2 * d;
    const int32_t sr = src_row[m];
    const float* base;
    if (sr >= 0) {
        base = states + (int64_t)sr * W;
    } else {
        const int64_t a = checked_id_cl(anchors[anchor_ref[m]], n_ent, flag);
        base = ent_rm + a * W;
    }
    const bool inv = neg && neg[m];
    const int64_t r = checked_id_cl(rels[rel_ref[m]], n_rel, flag);
    if (MODEL == KGQ_CONE) {
        const float* rr = rel + r * W;
        float* dst = x + (int64_t)m * W;
        for (int k = threadIdx.x; k < d; k += blockDim.x) {
            float th = base[k], ps = base[d + k];
            if (inv) cone_negate(th, ps);
            dst[k] = th + rr[k];
            dst[d + k] = ps + rr[d + k];
        }
    } else {
        const float* rr = rel + r * d;
        float* dst = x + (int64_t)m * 3 * d;
        for (int k = threadIdx.x; k < d; k += blockDim.x) {
            const float l = base[k], u = base[d + k];
            dst[k] = inv ? 1.0f - u : l;
            dst[d + k] = inv ? 1.0f - l : u;
            dst[2 * d + k] = rr[k];
        }
    }
}

// The same in split form: a wavefront per row.
template <int MODEL>
__global__ __launch_bounds__(256) void k_mlp_proj_prep_split(const int32_t* src_row, const int32_t* anchor_ref,
                                                             const int32_t* rel_ref, const int32_t* neg,
                                                             const int32_t* anchors, const int32_t* rels,
                                                             const float* states, const float* ent_rm,
                                                             const float* rel, int64_t n_ent, int n_rel, int d, int M,
                                                             SplitRows x, int* flag)
{
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M) return;
    const int W = 2 * d;
    const int32_t sr = src_row[m];
    const float* base = sr >= 0 ? states + (int64_t)sr * W
                                : ent_rm + (int64_t)checked_id_cl(anchors[anchor_ref[m]], n_ent, flag) * W;
    const bool inv = neg && neg[m];
    const int64_t r = checked_id_cl(rels[rel_ref[m]], n_rel, flag);
    const int width = MODEL == KGQ_CONE ? W : 3 * d, n8 = (int)(plane_ld(width) / 8);
    // four columns at a time: none straddles two fields (d is a multiple of 4)
    auto four = [&](int k) {
        if (k >= width) return make_float4(0.f, 0.f, 0.f, 0.f);
        auto at = [](const float* p) { return *reinterpret_cast<const float4*>(p); };
        float4 v;
        if (MODEL == KGQ_CONE) {
            v = at(base + k);
            const float4 q = at(rel + r * W + k);
            if (inv) {
                float z = 0.f;
                if (k < d) {
                    cone_negate(v.x, z);
                    cone_negate(v.y, z);
                    cone_negate(v.z, z);
                    cone_negate(v.w, z);
                } else {
                    cone_negate(z, v.x);
                    cone_negate(z, v.y);
                    cone_negate(z, v.z);
                    cone_negate(z, v.w);
                }
            }
            return make_float4(v.x + q.x, v.y + q.y, v.z + q.z, v.w + q.w);
        }
        if (k >= W) return at(rel + r * d + k - W);
        if (!inv) return at(base + k);
        v = at(base + (k < d ? k + d : k - d));
        return make_float4(1.0f - v.x, 1.0f - v.y, 1.0f - v.z, 1.0f - v.w);
    };
    split_row_wave([&](int c, float (&v)[8]) {
#pragma unroll
                       for (int h = 0; h < 2; ++h) {
                           const float4 q = four(8 * c + 4 * h);
                           v[4 * h] = q.x;
                           v[4 * h + 1] = q.y;
                           v[4 * h + 2] = q.z;
                           v[4 * h + 3] = q.w;
                       }
                   },
                   n8, x.rows + (int64_t)m * n8 * 8, x.scale + m, lane);
}

void launch_mlp_proj_prep(int model, const int32_t* src_row, const int32_t* anchor_ref, const int32_t* rel_ref,
                          const int32_t* neg, int M, const int32_t* anchors, const int32_t* rels,
                          const float* states, const float* ent_rm, const float* rel, int64_t n_ent, int n_rel,
                          int d, float* x, SplitRows split, int* flag, hipStream_t s)
{
    if (M <= 0) return;
    if (split.rows && model == KGQ_CONE)
        hipLaunchKernelGGL(k_mlp_proj_prep_split<KGQ_CONE>, dim3((M + 3) / 4), dim3(256), 0, s, src_row, anchor_ref,
                           rel_ref, neg, anchors, rels, states, ent_rm, rel, n_ent, n_rel, d, M, split, flag);
    else if (split.rows)
        hipLaunchKernelGGL(k_mlp_proj_prep_split<KGQ_LOGICE>, dim3((M + 3) / 4), dim3(256), 0, s, src_row, anchor_ref,
                           rel_ref, neg, anchors, rels, states, ent_rm, rel, n_ent, n_rel, d, M, split, flag);
    else if (model == KGQ_CONE)
        hipLaunchKernelGGL(k_mlp_proj_prep<KGQ_CONE>, dim3(M), dim3(row_threads(d)), 0, s, src_row, anchor_ref, rel_ref, neg,
                           anchors, rels, states, ent_rm, rel, n_ent, n_rel, d, x, flag);
    else
        hipLaunchKernelGGL(k_mlp_proj_prep<KGQ_LOGICE>, dim3(M), dim3(row_threads(d)), 0, s, src_row, anchor_ref, rel_ref, neg,
                           anchors, rels, states, ent_rm, rel, n_ent, n_rel, d, x, flag);
}

// LogicE projection output: the last layer wrote sigmoid(y) into both halves
// of each destination row; turn the upper half into u = l + s (1 - l).
__global__ __launch_bounds__(256) void k_logic_bounds(const int32_t* rowmap, int d, float* states)
{
    float* row = states + (int64_t)rowmap[blockIdx.x] * 2 * d;
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        const float l = row[k];
        row[d + k] = l + row[d + k] * (1.0f - l);
    }
}

void launch_logic_bounds(const int32_t* rowmap, int M, int d, float* states, hipStream_t s)
{
    if (M <= 0) return;
    hipLaunchKernelGGL(k_logic_bounds, dim3(M), dim3(256), 0, s, rowmap, d, states);
}

// ---------------------------------------------------------------------------
// Intersections (vertical fusion: all branches of a group in one pass)
// ---------------------------------------------------------------------------

// ConE: u_j = [theta_j - psi_j; theta_j + psi_j] of every input row of the
// stage (complemented first where the branch is negated), the input of the
// stacked first layers.
__global__ __launch_bounds__(256) void k_cone_int_prep(GroupArgs g, const float* states, int d, float* x_int)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int neg = g.neg_mask[gi];
    for (int j = 0; j < n; ++j) {
        const bool inv = (neg >> j) & 1;
        const float* src = states + (int64_t)(i0 + j) * 2 * d;
        float* dst = x_int + (int64_t)(i0 + j) * 2 * d;
        for (int k = threadIdx.x; k < d; k += blockDim.x) {
            float th = src[k], ps = src[d + k];
            if (inv) cone_negate(th, ps);
            dst[k] = th - ps;
            dst[d + k] = th + ps;
        }
    }
}

// The same in split form: a wavefront per input row.
__global__ __launch_bounds__(256) void k_cone_int_prep_split(GroupArgs g, const float* states, int d, SplitRows x)
{
    const int gi = blockIdx.x, lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    if (j >= g.n_in[gi]) return;
    const int64_t row = g.in_start[gi] + j;
    const bool inv = (g.neg_mask[gi] >> j) & 1;
    const float* src = states + row * 2 * d;
    const int n8 = (int)(plane_ld(2 * d) / 8);
    split_row_wave([&](int c, float (&v)[8]) {
                       // (d is a multiple of 4: four values lie on one side of it)
#pragma unroll
                       for (int h = 0; h < 2; ++h) {
                           const int k = 8 * c + 4 * h, i = k < d ? k : k - d;
                           float th[4] = {}, ps[4] = {};
                           if (k < 2 * d) {
                               *reinterpret_cast<float4*>(th) = *reinterpret_cast<const float4*>(src + i);
                               *reinterpret_cast<float4*>(ps) = *reinterpret_cast<const float4*>(src + d + i);
                           }
#pragma unroll
                           for (int t = 0; t < 4; ++t) {
                               if (inv && k < 2 * d) cone_negate(th[t], ps[t]);
                               v[4 * h + t] = k < d ? th[t] - ps[t] : th[t] + ps[t];
                           }
                       }
                   },
                   n8, x.rows + row * n8 * 8, x.scale + row, lane);
}

void launch_cone_int_prep(const GroupArgs& g, const float* states, int d, float* x_int, SplitRows split, hipStream_t s)
{
    if (g.n_groups <= 0) return;
    if (split.rows)
        hipLaunchKernelGGL(k_cone_int_prep_split, dim3(g.n_groups), dim3(64 * kGroupInputs), 0, s, g, states, d, split);
    else
        hipLaunchKernelGGL(k_cone_int_prep, dim3(g.n_groups), dim3(256), 0, s, g, states, d, x_int);
}

// Value k of a row in split form.
__device__ __forceinline__ float split_value(const float* row, float scale, int k)
{
    const _Float16* p = reinterpret_cast<const _Float16*>(row + (k & ~7)) + (k & 7);
    return fmaf((float)p[8], kSplitLow, (float)p[0]) * scale;
}

// ConE axis: attention-weighted mean of the branch axes' unit vectors; and
// the mean over branches of the aperture set function's hidden features
// (columns d .. 2d-1 of the stacked first layer's output).
template <bool SPLIT>
__global__ __launch_bounds__(1024) void k_cone_combine_axis(GroupArgs g, const float* states, const float* logits,
                                                           const float* hid, const float* hid_scale, int d, float* zmean,
                                                           SplitRows zsplit, float* out_states)
{
    extern __shared__ __align__(16) float zrow[];      // SPLIT: the mean, d floats padded to whole stages
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int neg = g.neg_mask[gi];
    const int64_t orow = g.out_row[gi];
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float mx = logits[(int64_t)i0 * d + k];
        for (int j = 1; j < n; ++j) mx = fmaxf(mx, logits[(int64_t)(i0 + j) * d + k]);
        float z = 0.f, cx = 0.f, sy = 0.f, zm = 0.f;
        for (int j = 0; j < n; ++j) {
            const float w = expf(logits[(int64_t)(i0 + j) * d + k] - mx);
            float th = states[(int64_t)(i0 + j) * 2 * d + k], ps = states[(int64_t)(i0 + j) * 2 * d + d + k];
            if ((neg >> j) & 1) cone_negate(th, ps);
            float sn, cs;
            sincosf(th, &sn, &cs);
            z += w;
            cx += w * cs;
            sy += w * sn;
            if (SPLIT) zm += split_value(hid + (i0 + j) * plane_ld(2 * d), hid_scale[i0 + j], d + k);
            else zm += hid[(int64_t)(i0 + j) * 2 * d + d + k];
        }
        // the weights' common factor 1/z does not change the angle
        out_states[orow * 2 * d + k] = atan2f(sy / z, cx / z);
        if (SPLIT) zrow[k] = zm / (float)n;
        else zmean[(int64_t)gi * d + k] = zm / (float)n;
    }
    if constexpr (SPLIT) {
        const int ld = (int)plane_ld(d);
        for (int k = d + threadIdx.x; k < ld; k += blockDim.x) zrow[k] = 0.f;
        __syncthreads();
        if (threadIdx.x < 64)
            split_row_wave([&](int c, float (&v)[8]) {
#pragma unroll
                               for (int t = 0; t < 8; ++t) v[t] = zrow[c * 8 + t];
                           },
                           ld / 8, zsplit.rows + (int64_t)gi * ld, zsplit.scale + gi, threadIdx.x);
    }
}

void launch_cone_combine_axis(const GroupArgs& g, const float* states, const float* logits, const float* hid,
                              const float* hid_scale, int d, float* zmean, SplitRows zsplit, float* out_states,
                              hipStream_t s)
{
    if (g.n_groups <= 0) return;
    if (hid_scale)
        hipLaunchKernelGGL(k_cone_combine_axis<true>, dim3(g.n_groups), dim3(row_threads(d)), plane_ld(d) * 4, s, g, states,
                           logits, hid, hid_scale, d, zmean, zsplit, out_states);
    else
        hipLaunchKernelGGL(k_cone_combine_axis<false>, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, logits, hid,
                           nullptr, d, zmean, zsplit, out_states);
}

// ConE half-aperture: min over branches (complemented where negated) times
// the sigmoid gate.
__global__ __launch_bounds__(1024) void k_cone_combine_arg(GroupArgs g, const float* states, const float* gate, int d,
                                                          float* out_states)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int neg = g.neg_mask[gi];
    const int64_t orow = g.out_row[gi];
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float m = 0.f;
        for (int j = 0; j < n; ++j) {
            float ps = states[(int64_t)(i0 + j) * 2 * d + d + k];
            if ((neg >> j) & 1) ps = kPi - ps;
            m = j == 0 ? ps : fminf(m, ps);
        }
        out_states[orow * 2 * d + d + k] = m * (1.0f / (1.0f + expf(-gate[(int64_t)gi * d + k])));
    }
}

void launch_cone_combine_arg(const GroupArgs& g, const float* states, const float* gate, int d, float* out_states,
                             hipStream_t s)
{
    if (g.n_groups <= 0) return;
    hipLaunchKernelGGL(k_cone_combine_arg, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, gate, d, out_states);
}

// LogicE: the t-norm over the branches of each group, coordinate-wise.
template <int TNORM>
__global__ __launch_bounds__(1024) void k_logic_combine(GroupArgs g, const float* states, int d, float* out_states)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int neg = g.neg_mask[gi];
    const int64_t orow = g.out_row[gi];
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float lo = 0.f, hi = 0.f;
        for (int j = 0; j < n; ++j) {
            const float* src = states + (int64_t)(i0 + j) * 2 * d;
            float l = src[k], u = src[d + k];
            if ((neg >> j) & 1) {
                const float t = 1.0f - u;
                u = 1.0f - l;
                l = t;
            }
            if (j == 0) {
                lo = l;
                hi = u;
            } else if (TNORM == KGQ_TNORM_MIN) {
                lo = fminf(lo, l);
                hi = fminf(hi, u);
            } else if (TNORM == KGQ_TNORM_LUKASIEWICZ) {
                lo = fmaxf(lo + l - 1.0f, 0.f);
                hi = fmaxf(hi + u - 1.0f, 0.f);
            } else {
                lo *= l;
                hi *= u;
            }
        }
        out_states[orow * 2 * d + k] = lo;
        out_states[orow * 2 * d + d + k] = hi;
    }
}

void launch_logic_combine(int tnorm, const GroupArgs& g, const float* states, int d, float* out_states,
                          hipStream_t s)
{
    if (g.n_groups <= 0) return;
    if (tnorm == KGQ_TNORM_MIN)
        hipLaunchKernelGGL(k_logic_combine<KGQ_TNORM_MIN>, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, d,
                           out_states);
    else if (tnorm == KGQ_TNORM_LUKASIEWICZ)
        hipLaunchKernelGGL(k_logic_combine<KGQ_TNORM_LUKASIEWICZ>, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, d,
                           out_states);
    else
        hipLaunchKernelGGL(k_logic_combine<KGQ_TNORM_PRODUCT>, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, d,
                           out_states);
}

// ---------------------------------------------------------------------------
// ConE query packing for the VALU scorer: [row_block][k][field][TQ] with the
// five fields of each (complemented where the scored row is negated) query
// cone that the scorer's max form reads (k_score.hip): tan(theta/2),
// cos(psi/2) / r, sin(psi/2) / |cos(theta/2)|, sin(psi/2) / r and
// r |cos(theta/2)|, r = center_reg. |cos(theta/2)| is at least 1e-18 and r at
// least 2^-30, so every field and the scorer's products of them stay finite;
// what the floors change is below the rounding of the sums. One workgroup per
// block of TQ rows; padding rows are zero.
// ---------------------------------------------------------------------------

template <int TQ>
__global__ __launch_bounds__(256) void k_pack_cone(const int32_t* src_row, const int32_t* neg, int n_rows,
                                                   const float* states, int d, float r, float* qpack)
{
    const int qb = blockIdx.x;
    float* out = qpack + (int64_t)qb * d * 5 * TQ;
    for (int o = threadIdx.x; o < d * TQ; o += blockDim.x) {
        const int i = o % TQ, k = o / TQ;
        const int j = qb * TQ + i;
        float f[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        if (j < n_rows) {
            const float* st = states + (int64_t)src_row[j] * 2 * d;
            float th = st[k], ps = st[d + k];
            if (neg && neg[j]) cone_negate(th, ps);
            float ca, sa, cb, sb;
            sincosf(0.5f * th, &sa, &ca);
            sincosf(0.5f * ps, &sb, &cb);
            if (fabsf(ca) < 1e-18f) ca = 1e-18f;
            f[0] = sa / ca;
            f[1] = cb / r;
            f[2] = sb / fabsf(ca);
            f[3] = sb / r;
            f[4] = r * fabsf(ca);
        }
        float* dst = out + (int64_t)k * 5 * TQ + i;
#pragma unroll
        for (int t = 0; t < 5; ++t) dst[t * TQ] = f[t];
    }
}

void launch_pack_cone(const int32_t* src_row, const int32_t* neg, int n_rows, int n_rows_pad, const float* states,
                      int d, float center_reg, float* qpack, hipStream_t s)
{
    if (n_rows_pad <= 0) return;
    const int tq = score_tq(KGQ_CONE, n_rows);
    const dim3 grid(n_rows_pad / tq);
    const float r = std::max(center_reg, 0x1p-30f);
    if (score_small(n_rows))
        hipLaunchKernelGGL(k_pack_cone<kTqConeSmall>, grid, dim3(256), 0, s, src_row, neg, n_rows, states, d, r, qpack);
    else
        hipLaunchKernelGGL(k_pack_cone<kTqCone>, grid, dim3(256), 0, s, src_row, neg, n_rows, states, d, r, qpack);
}

}  // namespace kgq
