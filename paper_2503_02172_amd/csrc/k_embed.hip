// Query-plan operator kernels other than the dense layers and the scorer:
// parameter re-layout at load time, anchor gathers, translation chains,
// intersection / negation combines, query packing and id validation.
//
// Operators (the paper's Eq. 2 maps a query's relations, conjunctions and
// negations to projection, intersection and negation functions):
//   GQE   projection q + Rel[r]; intersection sum_j softmax_j(s_j) q_j with
//         s_j = W2 ReLU(W1 q_j + b1) + b2 (softmax across branches, per dim).
//   Q2B   projection (c + C[r], o + softplus(O[r])); intersection: attention
//         as above on the centers; offset min_j(o_j) * sigmoid(W4 mean_j
//         ReLU(W3 o_j + b3) + b4).
//   BetaE negation (alpha, beta) -> (1/alpha, 1/beta); intersection:
//         attention weights from [alpha; beta] (W1: 2d -> 2d, W2: 2d -> d),
//         applied to alpha and beta; projection MLP (Eq. 4) runs on the MFMA
//         GEMM, with x = [alpha; beta] + Rel[r] built here.
// Ids read from device memory are range-checked in every kernel that reads
// them: an out-of-range id raises a flag bit and is replaced by 0, so no
// access ever leaves a table.
#include <algorithm>
#include <cmath>

#include "kgq_internal.hpp"
#include "mfma_tile.hpp"

namespace kgq {

__device__ __forceinline__ float bf16_to_f32(uint16_t h)
{
    return __uint_as_float(((uint32_t)h) << 16);
}

__device__ __forceinline__ float load_param(const void* src, int bf16, int64_t i)
{
    return bf16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(src)[i])
                : reinterpret_cast<const float*>(src)[i];
}

// ---------------------------------------------------------------------------
// Load-time kernels
// ---------------------------------------------------------------------------

// 64 entities x 64 coordinates per workgroup, transposed through LDS: rows are
// read (and copied row-major in float32) along the coordinates, the blocked
// dimension-major layout is written along the entities.
__global__ __launch_bounds__(256) void k_relayout_points(const void* src, int bf16, int64_t N, int d,
                                                         float* rowmajor, float* blocked)
{
    __shared__ float tile[64][65];
    const int t = threadIdx.x;
    const int64_t e0 = (int64_t)blockIdx.x * 64;
    const int k0 = blockIdx.y * 64, c = k0 + (t & 15) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = (t >> 4) + 16 * i;
        const int64_t at = (e0 + r) * d + c;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e0 + r < N && c < d) {      // (d is a multiple of 4)
            if (bf16) {
                const ushort4 h = *reinterpret_cast<const ushort4*>(reinterpret_cast<const uint16_t*>(src) + at);
                v = make_float4(bf16_to_f32(h.x), bf16_to_f32(h.y), bf16_to_f32(h.z), bf16_to_f32(h.w));
            } else {
                v = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(src) + at);
            }
            *reinterpret_cast<float4*>(rowmajor + at) = v;
        }
        float (*col)[65] = tile + (t & 15) * 4;
        col[0][r] = v.x;
        col[1][r] = v.y;
        col[2][r] = v.z;
        col[3][r] = v.w;
    }
    __syncthreads();
    float* dst = blocked + (e0 / kEntBlock) * (int64_t)d * kEntBlock + e0 % kEntBlock + (t & 63);
    for (int k = t >> 6; k < 64 && k0 + k < d; k += 4) dst[(int64_t)(k0 + k) * kEntBlock] = tile[k][t & 63];
}

void launch_relayout_points(const void* src, int src_bf16, int64_t N, int d, int64_t n_blocks,
                            float* rowmajor, float* blocked, hipStream_t s)
{
    hipLaunchKernelGGL(k_relayout_points, dim3((unsigned)(n_blocks * (kEntBlock / 64)), (d + 63) / 64), dim3(256), 0, s,
                       src, src_bf16, N, d, rowmajor, blocked);
}

// Sum of one value per thread over a workgroup of 256, the same in each.
__device__ __forceinline__ double block_sum(double v)
{
    __shared__ double sh[4];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__global__ __launch_bounds__(256) void k_table_range(const float4* __restrict__ x, int64_t n4, double* __restrict__ part)
{
    __shared__ float sh_lo[4], sh_hi[4];
    float lo = __builtin_inff(), hi = -__builtin_inff();
    double sum = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)kStatBlocks * 256) {
        const float4 v = x[i];
        lo = fminf(fminf(fminf(lo, v.x), fminf(v.y, v.z)), v.w);
        hi = fmaxf(fmaxf(fmaxf(hi, v.x), fmaxf(v.y, v.z)), v.w);
        sum += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off, 64));
        hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        sh_lo[threadIdx.x >> 6] = lo;
        sh_hi[threadIdx.x >> 6] = hi;
    }
    sum = block_sum(sum);
    if (threadIdx.x == 0) {
        double* o = part + 3 * blockIdx.x;
        o[0] = fminf(fminf(sh_lo[0], sh_lo[1]), fminf(sh_lo[2], sh_lo[3]));
        o[1] = fmaxf(fmaxf(sh_hi[0], sh_hi[1]), fmaxf(sh_hi[2], sh_hi[3]));
        o[2] = sum;
    }
}

__global__ __launch_bounds__(256) void k_table_spread(const float4* __restrict__ x, int64_t n4, double* __restrict__ part)
{
    float most = 0.f;
    double logs = 0.0, count = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)kStatBlocks * 256) {
        const float4 q = x[i];
        const float v[4] = {fabsf(q.x), fabsf(q.y), fabsf(q.z), fabsf(q.w)};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            most = fmaxf(most, v[t]);
            if (v[t] != 0.f) {
                logs += (double)log2f(v[t]);       // (NaN and infinities pass through)
                count += 1.0;
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) most = fmaxf(most, __shfl_xor(most, off, 64));
    __shared__ float sh_most[4];
    if ((threadIdx.x & 63) == 0) sh_most[threadIdx.x >> 6] = most;
    logs = block_sum(logs);
    count = block_sum(count);
    if (threadIdx.x == 0) {
        double* o = part + 3 * blockIdx.x;
        o[0] = fmaxf(fmaxf(sh_most[0], sh_most[1]), fmaxf(sh_most[2], sh_most[3]));
        o[1] = logs;
        o[2] = count;
    }
}

void launch_table_spread(const float* x, int64_t n, double* part, hipStream_t s)
{
    hipLaunchKernelGGL(k_table_spread, dim3(kStatBlocks), dim3(256), 0, s, reinterpret_cast<const float4*>(x), n / 4, part);
}

float table_spread(const double* part)
{
    double most = 0.0, logs = 0.0, count = 0.0;
    for (int b = 0; b < kStatBlocks; ++b) {
        most = std::max(most, part[3 * b]);
        logs += part[3 * b + 1];
        count += part[3 * b + 2];
    }
    if (!(logs - logs == 0.0) || !(most < HUGE_VAL)) return HUGE_VALF;
    return count > 0.0 ? (float)(most / std::exp2(logs / count)) : 1.f;
}

void launch_table_stats(const float* x, int64_t n, double* part, hipStream_t s)
{
    const float4* x4 = reinterpret_cast<const float4*>(x);
    hipLaunchKernelGGL(k_table_range, dim3(kStatBlocks), dim3(256), 0, s, x4, n / 4, part);
}

// A score is gamma - scale * distance in float32. The quantisation error of a
// distance, each of its 2 x width values off by at most half a quantum and 0.29
// of one at the root mean square, is 0.41 sqrt(width) quanta at every distance.
// A score near gamma, of an entity that all but coincides with the query, is
// rounded by 0.29 ulp, at least 0.29 x 2^-24 gamma, and further away the float
// sum's own error, 0.25 sqrt(width) 2^-24 of the distance, soon exceeds that.
// So the table takes the fixed-point form where the quantisation error is at
// most a quarter of the rounding at gamma: however near the entities are to
// each other or to the query, the score's error then grows by 3% at most, and
// from a distance of about gamma / 50 on it is below the float form's.
// Uniform tables of half width gamma / width take it up to a width of 500
// (GQE; LogicE at gamma = 1 up to 2,000); a wider range, or one stretched by
// outliers or by columns of different centres, doesn't. Measured error against
// 64 bits on uniform tables: 1.1e-6 in floats, 1.2e-7 here (63,361 x 400);
// 1.9e-7 and 3.0e-8 (LogicE, 14,505 x 800).
L1Fixed choose_l1_fixed(double lo, double hi, double sum, int width, double gamma, double scale)
{
    L1Fixed f;
    const double range = hi - lo;
    if (!(sum - sum == 0.0) || !(range > 0.0) || !(range < 1e30) || !(range > 1e-30)) return f;   // NaN, inf, no range
    const double u_max = std::floor(4294967295.0 / width);
    const float q = std::nextafter((float)(range / u_max), 1e38f);     // range / q <= u_max
    const double error = 0.41 * std::sqrt((double)width) * (double)q * scale;
    if (!(error <= 0.25 * 0.29 * 0x1p-24 * std::fabs(gamma))) return f;
    f.on = true;
    f.lo = (float)lo;
    f.hi = (float)hi;
    f.quantum = q;
    return f;
}

__global__ __launch_bounds__(256) void k_l1_quantise(float4* __restrict__ blk, int64_t n4, L1Fixed f, double inv_quantum)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const float4 v = blk[i];
    double ex = 0.0;
    blk[i] = make_float4(__uint_as_float(l1_fixed_word(v.x, f, inv_quantum, ex)),
                         __uint_as_float(l1_fixed_word(v.y, f, inv_quantum, ex)),
                         __uint_as_float(l1_fixed_word(v.z, f, inv_quantum, ex)),
                         __uint_as_float(l1_fixed_word(v.w, f, inv_quantum, ex)));
}

void launch_l1_quantise(float* blk, int64_t n, const L1Fixed& f, hipStream_t s)
{
    const int64_t n4 = n / 4;
    hipLaunchKernelGGL(k_l1_quantise, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<float4*>(blk), n4, f, 1.0 / (double)f.quantum);
}

// Digamma for x > 0 in double precision: shift the argument up with
// psi(x) = psi(x + 1) - 1/x until x >= 8, then the asymptotic series
// psi(x) = ln x - 1/(2x) - sum_{n>=1} B_2n / (2n x^2n), kept through B_12
// (Abramowitz & Stegun 6.3.18); the first dropped term is below 2e-14 at x = 8.
__device__ double digamma_d(double x)
{
    double shift = 0.0;
    while (x < 8.0) {
        shift -= 1.0 / x;
        x += 1.0;
    }
    const double f = 1.0 / (x * x);
    const double tail = f * (-1.0 / 12.0 + f * (1.0 / 120.0 + f * (-1.0 / 252.0 + f * (1.0 / 240.0
                      + f * (-1.0 / 132.0 + f * (691.0 / 32760.0))))));
    return shift + log(x) - 0.5 / x + tail;
}

// ln Gamma(x) for x >= 8 by Stirling's series (Abramowitz & Stegun 6.1.41),
// kept through the z^-11 term; the first dropped term is below 2e-14 at x = 8.
__device__ __forceinline__ double lngamma_stirling(double x)
{
    const double r = 1.0 / x, f = r * r;
    const double tail = r * (1.0 / 12.0 + f * (-1.0 / 360.0 + f * (1.0 / 1260.0 + f * (-1.0 / 1680.0
                      + f * (1.0 / 1188.0 + f * (-691.0 / 360360.0))))));
    return (x - 0.5) * log(x) - x + 0.91893853320467274178 + tail;   // + ln sqrt(2 pi)
}

// ln B(a, b) = ln Gamma(a) + ln Gamma(b) - ln Gamma(a + b) in double
// precision for a, b > 0. Each argument below 8 is shifted up with
// ln Gamma(x) = ln Gamma(x + 1) - ln x, and the three products of the shifted
// factors share one logarithm (at most 8 factors each, all in (0, 8), so the
// products of fp32-sourced arguments stay within double range). Other
// arguments give NaN: the Beta distribution needs positive shape parameters.
__device__ __forceinline__ double lnbeta_pos(double a, double b)
{
    if (!(a > 0.0 && b > 0.0)) return __builtin_nan("");
    double c = a + b, pa = 1.0, pb = 1.0, pc = 1.0;
    while (a < 8.0) { pa *= a; a += 1.0; }
    while (b < 8.0) { pb *= b; b += 1.0; }
    while (c < 8.0) { pc *= c; c += 1.0; }
    return lngamma_stirling(a) + lngamma_stirling(b) - lngamma_stirling(c) - log((pa / pc) * pb);
}

// The same for any arguments: those that are not positive take the library
// lgamma (for the entity table as loaded; the scored query states are
// regulariser outputs or their reciprocals, always positive).
__device__ __forceinline__ double lnbeta_d(double a, double b)
{
    if (!(a > 0.0 && b > 0.0)) return lgamma(a) + lgamma(b) - lgamma(a + b);
    return lnbeta_pos(a, b);
}

// BetaE entity tables: alpha|beta decoded to fp32 (row-major, for anchor
// gathers), U|V row-major for the matrix-core scorer (zero rows past N), and
// E_e, all from the stored values.
__global__ __launch_bounds__(128) void k_betae_entity_prep(const void* src, int bf16, int64_t N, int d, int64_t n_pad,
                                    float* ab_rowmajor, float* uv_rowmajor, double* e_const)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_pad) return;
    float* dst = uv_rowmajor + e * 2 * d;
    double acc = 0.0;
    for (int k = 0; k < d; ++k) {
        float u = 0.f, v = 0.f;
        if (e < N) {
            const float af = load_param(src, bf16, e * 2 * d + k);
            const float bf = load_param(src, bf16, e * 2 * d + d + k);
            ab_rowmajor[e * 2 * d + k] = af;
            ab_rowmajor[e * 2 * d + d + k] = bf;
            const double a = af, b = bf;
            const double pa = digamma_d(a), pb = digamma_d(b), pab = digamma_d(a + b);
            u = (float)(pab - pa);
            v = (float)(pab - pb);
            const double lnb = lnbeta_d(a, b);
            acc += -lnb + a * pa + b * pb - (a + b) * pab;
        }
        dst[k] = u;
        dst[d + k] = v;
    }
    e_const[e] = acc;
}

void launch_betae_entity_prep(const void* src, int src_bf16, int64_t N, int d, int64_t n_blocks,
                              float* ab_rowmajor, float* uv_rowmajor, double* e_const, hipStream_t s)
{
    const int64_t n_pad = n_blocks * kEntBlock;
    hipLaunchKernelGGL(k_betae_entity_prep, dim3((unsigned)((n_pad + 127) / 128)), dim3(128), 0, s,
                       src, src_bf16, N, d, n_pad, ab_rowmajor, uv_rowmajor, e_const);
}

__global__ void k_softplus(const float* src, float* dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x = src[i];
    dst[i] = (float)((x > 0.0 ? x : 0.0) + log1p(exp(-fabs(x))));
}

void launch_softplus(const float* src, float* dst, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_softplus, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
}

// ---------------------------------------------------------------------------
// Validation
// ---------------------------------------------------------------------------

__global__ void k_clear_flag(int* flag) { *flag = 0; }

void launch_clear_flag(int* flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, flag);
}

// Plan upload: 16-byte words read from pinned host memory (over the bus)
// and written to the device slot, by a kernel in the caller's stream order.
__global__ __launch_bounds__(256) void k_fetch_words(const int4* __restrict__ src, int4* __restrict__ dst,
                                                     int64_t n4)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (int64_t)gridDim.x * 256)
        dst[i] = src[i];
}

void launch_fetch_words(const int32_t* host_src, int32_t* dst, int64_t n_words, hipStream_t s)
{
    const int64_t n4 = (n_words + 3) / 4;
    if (n4 <= 0) return;
    const int grid = (int)std::min<int64_t>(64, (n4 + 255) / 256);
    hipLaunchKernelGGL(k_fetch_words, dim3(grid), dim3(256), 0, s, reinterpret_cast<const int4*>(host_src),
                       reinterpret_cast<int4*>(dst), n4);
}

__device__ __forceinline__ int32_t checked_id(int32_t id, int64_t n, int* flag)
{
    if (id < 0 || (int64_t)id >= n) {
        atomicOr(flag, kErrRange);
        return 0;
    }
    return id;
}

// arity: one thread per query. For a mixed batch na_q / nr_q hold the
// per-query arity (from the plan) and unused slots must be -1.
__global__ void k_validate(const int32_t* anchors, const int32_t* rels, const int32_t* arity_q,
                           int B, int sa, int sr, int fixed_na, int fixed_nr,
                           int64_t n_ent, int n_rel, int* flag)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= B) return;
    const int na = arity_q ? arity_q[2 * q] : fixed_na;
    const int nr = arity_q ? arity_q[2 * q + 1] : fixed_nr;
    int bits = 0;
    for (int s = 0; s < sa; ++s) {
        const int32_t v = anchors[(int64_t)q * sa + s];
        if (s < na) { if (v < 0 || (int64_t)v >= n_ent) bits |= kErrRange; }
        else if (v != -1) bits |= kErrPadding;
    }
    for (int s = 0; s < sr; ++s) {
        const int32_t v = rels[(int64_t)q * sr + s];
        if (s < nr) { if (v < 0 || v >= n_rel) bits |= kErrRange; }
        else if (v != -1) bits |= kErrPadding;
    }
    if (bits) atomicOr(flag, bits);
}

void launch_validate(const int32_t* anchors, const int32_t* rels, const int32_t* arity_q,
                     int B, int sa, int sr, int fixed_na, int fixed_nr,
                     int64_t n_ent, int n_rel, int* flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_validate, dim3((B + 255) / 256), dim3(256), 0, s, anchors, rels, arity_q,
                       B, sa, sr, fixed_na, fixed_nr, n_ent, n_rel, flag);
}

// ---------------------------------------------------------------------------
// GQE / Query2Box translation chains (horizontal fusion of consecutive
// projections: the whole chain is one pass over the row)
// ---------------------------------------------------------------------------

__global__ void k_chain(int model, const int32_t* anchor_ref, const int32_t* rel_off, const int32_t* rel_ref,
                        const int32_t* dst_row, const int32_t* anchors, const int32_t* rels, const float* ent_rm,
                        const float* rel_c, const float* rel_o, int64_t n_ent, int n_rel, int d, float* states,
                        int* flag)
{
    const int c = blockIdx.x;
    const int64_t a = checked_id(anchors[anchor_ref[c]], n_ent, flag);
    const int h0 = rel_off[c], h1 = rel_off[c + 1];
    const int W = model == 0 ? d : 2 * d;
    float* out = states + (int64_t)dst_row[c] * W;
    // d is a multiple of 4: 128-bit accesses, one float4 per thread per step
    for (int k = threadIdx.x * 4; k < d; k += blockDim.x * 4) {
        float4 x = *reinterpret_cast<const float4*>(ent_rm + a * d + k);
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int h = h0; h < h1; ++h) {
            const int64_t r = checked_id(rels[rel_ref[h]], n_rel, flag);
            const float4 v = *reinterpret_cast<const float4*>(rel_c + r * d + k);
            x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
            if (model == 1) {
                const float4 u = *reinterpret_cast<const float4*>(rel_o + r * d + k);
                o.x += u.x; o.y += u.y; o.z += u.z; o.w += u.w;
            }
        }
        *reinterpret_cast<float4*>(out + k) = x;
        if (model == 1) *reinterpret_cast<float4*>(out + d + k) = o;
    }
}

void launch_chain(int model, const int32_t* anchor_ref, const int32_t* rel_off, const int32_t* rel_ref,
                  const int32_t* dst_row, int n_chain, const int32_t* anchors, const int32_t* rels,
                  const float* ent_rm, const float* rel_c, const float* rel_o, int64_t n_ent, int n_rel, int d,
                  float* states, int* flag, hipStream_t s)
{
    if (n_chain <= 0) return;
    hipLaunchKernelGGL(k_chain, dim3(n_chain), dim3(128), 0, s, model, anchor_ref, rel_off, rel_ref, dst_row,
                       anchors, rels, ent_rm, rel_c, rel_o, n_ent, n_rel, d, states, flag);
}

// ---------------------------------------------------------------------------
// Intersections (vertical fusion: all branches of a group in one pass)
// ---------------------------------------------------------------------------

// Attention weights across the n (2 .. kGroupInputs) branches of one
// dimension. Unrolled over the maximum with a guard, so that w stays in
// registers.
__device__ __forceinline__ void softmax_branches(const float* logits, int64_t ld, int n, int k,
                                                 float (&w)[kGroupInputs])
{
    float mx = logits[k];
#pragma unroll
    for (int j = 1; j < kGroupInputs; ++j)
        if (j < n) mx = fmaxf(mx, logits[j * ld + k]);
    float z = 0.f;
#pragma unroll
    for (int j = 0; j < kGroupInputs; ++j) {
        w[j] = j < n ? expf(logits[j * ld + k] - mx) : 0.f;
        z += w[j];
    }
    const float inv = 1.0f / z;
#pragma unroll
    for (int j = 0; j < kGroupInputs; ++j) w[j] *= inv;
}

__global__ void k_combine_center(int model, GroupArgs g, const float* states, int W,
                                 const float* logits, const float* zfeat, float* zmean,
                                 const int32_t* rels, const float* rel_c, int n_rel, int d,
                                 float* out_states, int* flag)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int64_t orow = g.out_row[gi];
    const int p0 = g.post_off[gi], p1 = g.post_off[gi + 1];
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float w[kGroupInputs];
        softmax_branches(logits + (int64_t)i0 * d, d, n, k, w);
        float c = 0.f;
        for (int j = 0; j < n; ++j) c += w[j] * states[(int64_t)(i0 + j) * W + k];
        // folded post-chain: the translations of the projections that follow
        for (int h = p0; h < p1; ++h) c += rel_c[(int64_t)checked_id(rels[g.post_ref[h]], n_rel, flag) * d + k];
        out_states[orow * W + k] = c;
        if (model == 1) {
            float z = 0.f;
            for (int j = 0; j < n; ++j) z += zfeat[(int64_t)(i0 + j) * d + k];
            zmean[(int64_t)gi * d + k] = z / (float)n;
        }
    }
}

void launch_combine_center(int model, const GroupArgs& g, const float* states, int W,
                           const float* logits, const float* zfeat, float* zmean,
                           const int32_t* rels, const float* rel_c, int n_rel, int d,
                           float* out_states, int* flag, hipStream_t s)
{
    if (g.n_groups <= 0) return;
    hipLaunchKernelGGL(k_combine_center, dim3(g.n_groups), dim3(row_threads(d)), 0, s, model, g, states, W, logits,
                       zfeat, zmean, rels, rel_c, n_rel, d, out_states, flag);
}

__global__ void k_combine_offset(GroupArgs g, const float* states, int W, const float* gate,
                                 const int32_t* rels, const float* rel_o, int n_rel, int d,
                                 float* out_states, int* flag)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int64_t orow = g.out_row[gi];
    const int p0 = g.post_off[gi], p1 = g.post_off[gi + 1];
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float m = states[(int64_t)i0 * W + d + k];
        for (int j = 1; j < n; ++j) m = fminf(m, states[(int64_t)(i0 + j) * W + d + k]);
        const float gv = gate[(int64_t)gi * d + k];
        float o = m * (1.0f / (1.0f + expf(-gv)));
        for (int h = p0; h < p1; ++h) o += rel_o[(int64_t)checked_id(rels[g.post_ref[h]], n_rel, flag) * d + k];
        out_states[orow * W + d + k] = o;
    }
}

void launch_combine_offset(const GroupArgs& g, const float* states, int W, const float* gate,
                           const int32_t* rels, const float* rel_o, int n_rel, int d,
                           float* out_states, int* flag, hipStream_t s)
{
    if (g.n_groups <= 0) return;
    hipLaunchKernelGGL(k_combine_offset, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, states, W, gate, rels,
                       rel_o, n_rel, d, out_states, flag);
}

// Eight values k .. k + 7 of a row of `width` (a multiple of 4), zeros past it.
__device__ __forceinline__ void load8(const float* row, int k, int width, float (&v)[8])
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float4 q = k + 4 * h < width ? *reinterpret_cast<const float4*>(row + k + 4 * h) : make_float4(0.f, 0.f, 0.f, 0.f);
        v[4 * h] = q.x;
        v[4 * h + 1] = q.y;
        v[4 * h + 2] = q.z;
        v[4 * h + 3] = q.w;
    }
}

// BetaE: copy each intersection input row, inverting both shape parameters
// of negated branches (negation), into the attention MLP input buffer.
__global__ void k_betae_int_prep(GroupArgs g, const float* states, int d, float* x_int)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int neg = g.neg_mask[gi];
    const int W = 2 * d;
    // every input's value read before any is stored: a load issued after a
    // store waits (vmcnt) for that store too
    for (int k = threadIdx.x; k < W; k += blockDim.x) {
        float v[kGroupInputs];
#pragma unroll
        for (int j = 0; j < kGroupInputs; ++j)
            if (j < n) {
                const float x = states[(int64_t)(i0 + j) * W + k];
                v[j] = ((neg >> j) & 1) ? 1.0f / x : x;
            }
#pragma unroll
        for (int j = 0; j < kGroupInputs; ++j)
            if (j < n) x_int[(int64_t)(i0 + j) * W + k] = v[j];
    }
}

// The same in split form: a wavefront per input row.
__global__ __launch_bounds__(256) void k_betae_int_prep_split(GroupArgs g, const float* states, int d, SplitRows x)
{
    const int gi = blockIdx.x, lane = threadIdx.x & 63, j = threadIdx.x >> 6;
    if (j >= g.n_in[gi]) return;
    const int64_t row = g.in_start[gi] + j;
    const bool inv = (g.neg_mask[gi] >> j) & 1;
    const int W = 2 * d, n8 = (int)(plane_ld(W) / 8);
    const float* src = states + row * W;
    split_row_wave([&](int c, float (&v)[8]) { load8(src, c * 8, W, v);
                       if (inv)
#pragma unroll
                           for (int t = 0; t < 8; ++t) v[t] = c * 8 + t < W ? 1.0f / v[t] : 0.f; },
                   n8, x.rows + row * n8 * 8, x.scale + row, lane);
}

void launch_betae_int_prep(const GroupArgs& g, const float* states, int d, float* x_int, SplitRows split, hipStream_t s)
{
    if (g.n_groups <= 0) return;
    if (split.rows)
        hipLaunchKernelGGL(k_betae_int_prep_split, dim3(g.n_groups), dim3(64 * kGroupInputs), 0, s, g, states, d, split);
    else
        hipLaunchKernelGGL(k_betae_int_prep, dim3(g.n_groups), dim3(row_threads(2 * d)), 0, s, g, states, d, x_int);
}

__global__ void k_betae_combine(GroupArgs g, const float* sin, const float* logits, int d, float* states)
{
    const int gi = blockIdx.x;
    const int i0 = g.in_start[gi];
    const int n = g.n_in[gi];
    const int64_t orow = g.out_row[gi];
    const int neg = g.neg_mask[gi];
    const int W = 2 * d;
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float w[kGroupInputs];
        softmax_branches(logits + (int64_t)i0 * d, d, n, k, w);
        float al = 0.f, be = 0.f;
        for (int j = 0; j < n; ++j) {
            float a = sin[(int64_t)(i0 + j) * W + k], b = sin[(int64_t)(i0 + j) * W + d + k];
            if ((neg >> j) & 1) {
                a = 1.0f / a;
                b = 1.0f / b;
            }
            al += w[j] * a;
            be += w[j] * b;
        }
        states[orow * W + k] = al;
        states[orow * W + d + k] = be;
    }
}

void launch_betae_combine(const GroupArgs& g, const float* sin, const float* logits, int d,
                          float* states, hipStream_t s)
{
    if (g.n_groups <= 0) return;
    hipLaunchKernelGGL(k_betae_combine, dim3(g.n_groups), dim3(row_threads(d)), 0, s, g, sin, logits, d, states);
}

__global__ void k_betae_proj_prep(const int32_t* src_row, const int32_t* anchor_ref, const int32_t* rel_ref,
                                  const int32_t* neg, const int32_t* anchors, const int32_t* rels,
                                  const float* states, const float* ent_ab, const float* rel, int64_t n_ent,
                                  int n_rel, int d, float* x, int* flag)
{
    const int m = blockIdx.x;
    const int W = 2 * d;
    const int32_t sr = src_row[m];
    const float* base;
    if (sr >= 0) {
        base = states + (int64_t)sr * W;
    } else {
        const int64_t a = checked_id(anchors[anchor_ref[m]], n_ent, flag);
        base = ent_ab + a * W;
    }
    const bool inv = neg && neg[m];   // negated source: reciprocal of both shape parameters
    const int64_t r = checked_id(rels[rel_ref[m]], n_rel, flag);
    const float* rr = rel + r * W;
    float* dst = x + (int64_t)m * W;
    for (int k = threadIdx.x; k < W; k += blockDim.x) {
        const float v = base[k];
        dst[k] = (inv ? 1.0f / v : v) + rr[k];
    }
}

// The same in split form: a wavefront per row.
__global__ __launch_bounds__(256) void k_betae_proj_prep_split(const int32_t* src_row, const int32_t* anchor_ref,
                                                               const int32_t* rel_ref, const int32_t* neg,
                                                               const int32_t* anchors, const int32_t* rels,
                                                               const float* states, const float* ent_ab,
                                                               const float* rel, int64_t n_ent, int n_rel, int d, int M,
                                                               SplitRows x, int* flag)
{
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M) return;
    const int W = 2 * d, n8 = (int)(plane_ld(W) / 8);
    const int32_t sr = src_row[m];
    const float* base = sr >= 0 ? states + (int64_t)sr * W
                                : ent_ab + (int64_t)checked_id(anchors[anchor_ref[m]], n_ent, flag) * W;
    const bool inv = neg && neg[m];
    const float* rr = rel + (int64_t)checked_id(rels[rel_ref[m]], n_rel, flag) * W;
    split_row_wave([&](int c, float (&v)[8]) {
                       float r[8];
                       load8(base, c * 8, W, v);
                       load8(rr, c * 8, W, r);
#pragma unroll
                       for (int t = 0; t < 8; ++t)
                           v[t] = c * 8 + t < W ? (inv ? 1.0f / v[t] : v[t]) + r[t] : 0.f;
                   },
                   n8, x.rows + (int64_t)m * n8 * 8, x.scale + m, lane);
}

void launch_betae_proj_prep(const int32_t* src_row, const int32_t* anchor_ref, const int32_t* rel_ref,
                            const int32_t* neg, int M, const int32_t* anchors, const int32_t* rels,
                            const float* states, const float* ent_ab, const float* rel,
                            int64_t n_ent, int n_rel, int d, float* x, SplitRows split, int* flag, hipStream_t s)
{
    if (M <= 0) return;
    if (split.rows)
        hipLaunchKernelGGL(k_betae_proj_prep_split, dim3((M + 3) / 4), dim3(256), 0, s, src_row, anchor_ref, rel_ref, neg,
                           anchors, rels, states, ent_ab, rel, n_ent, n_rel, d, M, split, flag);
    else
        hipLaunchKernelGGL(k_betae_proj_prep, dim3(M), dim3(row_threads(2 * d)), 0, s, src_row, anchor_ref, rel_ref, neg,
                           anchors, rels, states, ent_ab, rel, n_ent, n_rel, d, x, flag);
}

// BetaE first-hop projection, first layer, from the precomputed tables: the
// layer is linear in its input [alpha; beta] + Rel[r], so
// W1 (E[a] + Rel[r]) + b1 = (E W1^T)[a] + (Rel W1^T + b1)[r].
__global__ __launch_bounds__(256) void k_betae_proj1(const int32_t* anchor_ref, const int32_t* rel_ref,
                                                     const int32_t* anchors, const int32_t* rels, const float* pe,
                                                     const float* pr, int64_t n_ent, int n_rel, int w, float* h1,
                                                     int* flag)
{
    const int m = blockIdx.x;
    const int64_t a = checked_id(anchors[anchor_ref[m]], n_ent, flag);
    const int64_t r = checked_id(rels[rel_ref[m]], n_rel, flag);
    const float* x = pe + a * w;
    const float* y = pr + r * w;
    float* dst = h1 + (int64_t)m * w;
    for (int k = 4 * threadIdx.x; k < w; k += 4 * 256) {      // w = 4d is a multiple of 16
        const float4 u = *reinterpret_cast<const float4*>(x + k);
        const float4 v = *reinterpret_cast<const float4*>(y + k);
        float4 o;
        o.x = fmaxf(u.x + v.x, 0.f);
        o.y = fmaxf(u.y + v.y, 0.f);
        o.z = fmaxf(u.z + v.z, 0.f);
        o.w = fmaxf(u.w + v.w, 0.f);
        *reinterpret_cast<float4*>(dst + k) = o;
    }
}

// The same in split form: a wavefront per row.
__global__ __launch_bounds__(256) void k_betae_proj1_split(const int32_t* anchor_ref, const int32_t* rel_ref,
                                                           const int32_t* anchors, const int32_t* rels,
                                                           const float* pe, const float* pr, int64_t n_ent, int n_rel,
                                                           int w, int M, SplitRows h1, int* flag)
{
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (m >= M) return;
    const float* x = pe + (int64_t)checked_id(anchors[anchor_ref[m]], n_ent, flag) * w;
    const float* y = pr + (int64_t)checked_id(rels[rel_ref[m]], n_rel, flag) * w;
    const int n8 = (int)(plane_ld(w) / 8);
    split_row_wave([&](int c, float (&v)[8]) {
                       float r[8];
                       load8(x, c * 8, w, v);
                       load8(y, c * 8, w, r);
#pragma unroll
                       for (int t = 0; t < 8; ++t) v[t] = fmaxf(v[t] + r[t], 0.f);
                   },
                   n8, h1.rows + (int64_t)m * n8 * 8, h1.scale + m, lane);
}

void launch_betae_proj1(const int32_t* anchor_ref, const int32_t* rel_ref, int M, const int32_t* anchors,
                        const int32_t* rels, const float* pe, const float* pr, int64_t n_ent, int n_rel, int w,
                        float* h1, SplitRows split, int* flag, hipStream_t s)
{
    if (M <= 0) return;
    if (split.rows)
        hipLaunchKernelGGL(k_betae_proj1_split, dim3((M + 3) / 4), dim3(256), 0, s, anchor_ref, rel_ref, anchors, rels, pe,
                           pr, n_ent, n_rel, w, M, split, flag);
    else
        hipLaunchKernelGGL(k_betae_proj1, dim3(M), dim3(256), 0, s, anchor_ref, rel_ref, anchors, rels, pe, pr, n_ent,
                           n_rel, w, h1, flag);
}

// ---------------------------------------------------------------------------
// Query packing for the VALU scorers (GQE, Query2Box, LogicE): [row_block][k][field][TQ].
// One workgroup per block of TQ rows transposes through LDS, KC dimensions at
// a time (as many as a 32 KiB tile holds, so that all loads of a chunk are in
// flight together): the state rows are read along k and the packed block is
// written in its own order, both contiguous.
// ---------------------------------------------------------------------------

// NEGL (LogicE): a row with neg[j] != 0 is packed complemented, [1 - u; 1 - l]
// of its state [l; u] (d = 2 * half coordinates): coordinate c reads the
// state's coordinate (c + half) mod d and packs 1 minus it.
template <int TQ, int F, bool NEGL>
__global__ __launch_bounds__(256) void k_pack(const int32_t* src_row, const int32_t* neg, int half, int n_rows,
                                              const float* states, int W, int d, float* qpack)
{
    // dimensions per chunk: up to a 32 KiB tile (d = 400: one or two
    // chunks), a multiple of 4 so that no float4 straddles two fields
    constexpr int KC = 8192 / (TQ * F) / 4 * 4;
    constexpr int RS = F * KC + 1;            // padded LDS row: the transposed reads hit distinct banks
    __shared__ float tile[TQ * RS];
    __shared__ int srcs[TQ];
    __shared__ int negs[TQ];
    const int qb = blockIdx.x;
    const int t = threadIdx.x;
    if (t < TQ) {
        const int j = qb * TQ + t;
        srcs[t] = j < n_rows ? src_row[j] : -1;
        negs[t] = (NEGL && j < n_rows && neg) ? neg[j] : 0;
    }
    __syncthreads();
    float* out = qpack + (int64_t)qb * d * F * TQ;
    for (int k0 = 0; k0 < d; k0 += KC) {
        const int kc = min(KC, d - k0);           // a multiple of 4
        const int n4 = TQ * F * kc / 4;            // float4 elements of this chunk
        constexpr int PER4 = (TQ * F * KC / 4 + 255) / 256;   // float4 loads per thread (the last may be idle)
        // All loads of the chunk are issued before any is used: each reads a
        // valid address (row 0 for padding rows or past the chunk's end) and
        // the empty asm keeps the compiler from moving a load into the
        // validity branch, where the loads would wait for each other.
        float4 v[PER4];
#pragma unroll
        for (int u = 0; u < PER4; ++u) {
            const int e = 4 * (t + 256 * u);
            const int i = min(e / (F * kc), TQ - 1), rem = e - i * (F * kc);
            const int f = rem / kc, kk = rem - f * kc;
            const int src = srcs[i];
            const bool ok = t + 256 * u < n4 && src >= 0;
            int col = f * d + k0 + kk;
            if (NEGL && negs[i]) col = col >= half ? col - half : col + half;
            const int64_t off = ok ? (int64_t)src * W + col : 0;
            v[u] = *reinterpret_cast<const float4*>(states + off);
        }
#pragma unroll
        for (int u = 0; u < PER4; ++u) asm volatile("" : "+v"(v[u].x), "+v"(v[u].y), "+v"(v[u].z), "+v"(v[u].w));
#pragma unroll
        for (int u = 0; u < PER4; ++u) {
            if (t + 256 * u >= n4) break;
            const int e = 4 * (t + 256 * u);
            const int i = e / (F * kc), rem = e - i * (F * kc);
            const int f = rem / kc, kk = rem - f * kc;
            const bool ok = srcs[i] >= 0;
            float* dst = tile + i * RS + f * KC + kk;
            float4 x = v[u];
            if (NEGL && negs[i]) x = make_float4(1.0f - x.x, 1.0f - x.y, 1.0f - x.z, 1.0f - x.w);
            dst[0] = ok ? x.x : 0.f;
            dst[1] = ok ? x.y : 0.f;
            dst[2] = ok ? x.z : 0.f;
            dst[3] = ok ? x.w : 0.f;
        }
        __syncthreads();
        for (int o = t; o < kc * F * TQ; o += 256) {
            const int i = o % TQ, f = (o / TQ) % F, kk = o / (TQ * F);
            out[(int64_t)k0 * F * TQ + o] = tile[i * RS + f * KC + kk];
        }
        __syncthreads();
    }
}

// The same layout in fixed point (L1Fixed; one field), for the L1 scorer's
// integer form, and each row's base. A wavefront takes whole rows (every
// fourth of the block's), so that a row's clamped amount is one wave sum in a
// fixed order.
template <int TQ, bool NEGL>
__global__ __launch_bounds__(256) void k_pack_l1(const int32_t* src_row, const int32_t* neg, int n_rows,
                                                 const float* states, int W, int d, L1Fixed f, double inv_quantum,
                                                 float gamma, float dist_scale, uint32_t* qpack, double* base)
{
    constexpr int KC = 8192 / TQ / 4 * 4;     // coordinates per chunk (a 32 KiB tile)
    constexpr int RS = KC + 1;
    constexpr int RW = TQ / 4;                // rows per wavefront
    constexpr int PER = (KC + 255) / 256;     // float4 loads per lane, row and chunk
    __shared__ uint32_t tile[TQ * RS];
    const int qb = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int half = d / 2;
    int src[RW];
    bool ng[RW];
    double ex[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int j = qb * TQ + wave + 4 * r;
        src[r] = j < n_rows ? src_row[j] : -1;
        ng[r] = NEGL && j < n_rows && neg && neg[j];
        ex[r] = 0.0;
    }
    uint32_t* out = qpack + (int64_t)qb * d * TQ;
    for (int k0 = 0; k0 < d; k0 += KC) {
        const int kc = min(KC, d - k0);
        // every load of the chunk first (clamped into the row: no branch)
        float4 v[RW][PER];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                int col = k0 + min(4 * (lane + 64 * p), kc - 4);
                if (NEGL && ng[r]) col = col >= half ? col - half : col + half;
                v[r][p] = *reinterpret_cast<const float4*>(states + (int64_t)max(src[r], 0) * W + col);
            }
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int p = 0; p < PER; ++p) {
                const int k = 4 * (lane + 64 * p);
                if (k >= kc) continue;
                float x[4] = {v[r][p].x, v[r][p].y, v[r][p].z, v[r][p].w};
                uint32_t* dst = tile + (wave + 4 * r) * RS + k;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (NEGL && ng[r]) x[c] = 1.0f - x[c];
                    dst[c] = l1_fixed_word(src[r] >= 0 ? x[c] : f.lo, f, inv_quantum, ex[r]);
                }
            }
        __syncthreads();
        for (int o = t; o < kc * TQ; o += 256) out[(int64_t)k0 * TQ + o] = tile[(o % TQ) * RS + o / TQ];
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        double e = ex[r];
        for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
        if (lane == 0) base[qb * TQ + wave + 4 * r] = (double)gamma - (double)dist_scale * e;
    }
}

void launch_pack_l1(int model, const int32_t* src_row, const int32_t* neg, int n_rows, int n_rows_pad,
                    const float* states, int W, int d, const L1Fixed& f, float gamma, float dist_scale, float* qpack,
                    double* base, hipStream_t s)
{
    if (n_rows_pad <= 0) return;
    const dim3 grid(n_rows_pad / score_tq(model, n_rows));
    uint32_t* q = reinterpret_cast<uint32_t*>(qpack);
    const double inv = 1.0 / (double)f.quantum;
    const bool small = score_small(n_rows);
    if (model == KGQ_LOGICE) {
        if (small) hipLaunchKernelGGL((k_pack_l1<kTqGqeSmall, true>), grid, dim3(256), 0, s, src_row, neg, n_rows, states, W, d, f, inv, gamma, dist_scale, q, base);
        else hipLaunchKernelGGL((k_pack_l1<kTqGqe, true>), grid, dim3(256), 0, s, src_row, neg, n_rows, states, W, d, f, inv, gamma, dist_scale, q, base);
    } else {
        if (small) hipLaunchKernelGGL((k_pack_l1<kTqGqeSmall, false>), grid, dim3(256), 0, s, src_row, nullptr, n_rows, states, W, d, f, inv, gamma, dist_scale, q, base);
        else hipLaunchKernelGGL((k_pack_l1<kTqGqe, false>), grid, dim3(256), 0, s, src_row, nullptr, n_rows, states, W, d, f, inv, gamma, dist_scale, q, base);
    }
}

// BetaE: the query rows row-major, [row][alpha (d) | beta (d)], the A operand
// of the matrix-core scorer, and C_q = sum_i lnB(alpha_i, beta_i) per row in
// double precision (rows are regulariser outputs or their reciprocals, so
// positive; lnbeta_pos keeps the kernel at 45 VGPRs where the library lgamma
// fallback took 176). A negated answer row (neg[j] != 0) is packed as the
// reciprocals of its shape parameters. One workgroup per row. SPLIT: the row
// in the split form of the f16 matrix-core tile, with its scale.
template <bool SPLIT>
__global__ __launch_bounds__(256) void k_pack_rows(const int32_t* src_row, const int32_t* neg, const float* states,
                                                   int d, float* qrows, double* cq, float* q_scale)
{
    __shared__ double part[4];
    __shared__ float big[4];
    const int j = blockIdx.x;
    const int t = threadIdx.x;
    const bool inv = neg && neg[j];
    const float* st = states + (int64_t)src_row[j] * 2 * d;
    if constexpr (SPLIT) {
        // the row's largest magnitude, then chunks of 8 (32 bytes each)
        const int n8 = (int)(plane_ld(2 * d) / 8);
        float* dst = qrows + (int64_t)j * n8 * 8;
        auto load8 = [&](int c, float (&x)[8]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = 8 * c + 4 * h;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k < 2 * d) {
                    v = *reinterpret_cast<const float4*>(st + k);
                    if (inv) v = make_float4(1.0f / v.x, 1.0f / v.y, 1.0f / v.z, 1.0f / v.w);
                }
                x[4 * h] = v.x;
                x[4 * h + 1] = v.y;
                x[4 * h + 2] = v.z;
                x[4 * h + 3] = v.w;
            }
        };
        float x[8], m = 0.f;
        for (int c = t; c < n8; c += 256) {
            load8(c, x);
#pragma unroll
            for (int u = 0; u < 8; ++u) m = fmaxf(m, fabsf(x[u]));
        }
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        if ((t & 63) == 0) big[t >> 6] = m;
        __syncthreads();
        const float sc = split_scale(fmaxf(fmaxf(big[0], big[1]), fmaxf(big[2], big[3])));
        for (int c = t; c < n8; c += 256) {
            if (n8 > 256) load8(c, x);
            store_split8(dst + 8 * c, x, split_inverse(sc));
        }
        if (t == 0) q_scale[j] = sc;
    } else {
        float* dst = qrows + (int64_t)j * 2 * d;
        for (int k = 4 * t; k < 2 * d; k += 4 * 256) {
            float4 v = *reinterpret_cast<const float4*>(st + k);
            if (inv) v = make_float4(1.0f / v.x, 1.0f / v.y, 1.0f / v.z, 1.0f / v.w);
            *reinterpret_cast<float4*>(dst + k) = v;
        }
    }
    double lnb = 0.0;
    for (int k = t; k < d; k += 256) {
        float af = st[k], bf = st[d + k];
        if (inv) {
            af = 1.0f / af;
            bf = 1.0f / bf;
        }
        const double a = af, b = bf;
        lnb += lnbeta_pos(a, b);
    }
    for (int off = 32; off > 0; off >>= 1) lnb += __shfl_xor(lnb, off, 64);
    if ((t & 63) == 0) part[t >> 6] = lnb;
    __syncthreads();
    if (t == 0) cq[j] = (part[0] + part[1]) + (part[2] + part[3]);
}

void launch_pack(int model, const int32_t* src_row, const int32_t* neg, int n_rows, int n_rows_pad,
                 const float* states, int W, int d, float center_reg, float* qpack, double* cq, float* q_scale,
                 hipStream_t s)
{
    if (n_rows_pad <= 0) return;
    if (model == KGQ_BETAE) {
        if (q_scale)
            hipLaunchKernelGGL(k_pack_rows<true>, dim3(n_rows), dim3(256), 0, s, src_row, neg, states, d, qpack, cq, q_scale);
        else
            hipLaunchKernelGGL(k_pack_rows<false>, dim3(n_rows), dim3(256), 0, s, src_row, neg, states, d, qpack, cq, nullptr);
        return;
    }
    if (model == KGQ_CONE) {
        launch_pack_cone(src_row, neg, n_rows, n_rows_pad, states, d, center_reg, qpack, s);
        return;
    }
    const int tq = score_tq(model, n_rows);
    const bool small = score_small(n_rows);
    const dim3 grid(n_rows_pad / tq);          // n_rows_pad is a multiple of score_row_pad, hence of tq
    if (model == KGQ_GQE) {
        if (small) hipLaunchKernelGGL((k_pack<kTqGqeSmall, 1, false>), grid, dim3(256), 0, s, src_row, nullptr, 0, n_rows, states, W, d, qpack);
        else hipLaunchKernelGGL((k_pack<kTqGqe, 1, false>), grid, dim3(256), 0, s, src_row, nullptr, 0, n_rows, states, W, d, qpack);
    } else if (model == KGQ_LOGICE) {
        // the 2d bound coordinates as one field (d here is the width 2d)
        if (small) hipLaunchKernelGGL((k_pack<kTqGqeSmall, 1, true>), grid, dim3(256), 0, s, src_row, neg, d / 2, n_rows, states, W, d, qpack);
        else hipLaunchKernelGGL((k_pack<kTqGqe, 1, true>), grid, dim3(256), 0, s, src_row, neg, d / 2, n_rows, states, W, d, qpack);
    } else {
        if (small) hipLaunchKernelGGL((k_pack<kTqQ2bSmall, 2, false>), grid, dim3(256), 0, s, src_row, nullptr, 0, n_rows, states, W, d, qpack);
        else hipLaunchKernelGGL((k_pack<kTqQ2b, 2, false>), grid, dim3(256), 0, s, src_row, nullptr, 0, n_rows, states, W, d, qpack);
    }
}

}  // namespace kgq
