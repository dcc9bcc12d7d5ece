// BetaE entity scoring on the matrix cores of gfx950.
//
// The score of query row q against entity e is gamma minus the KL divergence
// of the entity's Beta embedding from the query's, summed over dimensions
// (Eq. 3 of the paper defines the Beta embedding). Regrouped exactly,
//   sum_i KL(Beta(a_i, b_i) || Beta(alpha_i, beta_i))
//     = C_q + E_e + sum_i (alpha_i * U_i + beta_i * V_i),
// with U = psi(a + b) - psi(a), V = psi(a + b) - psi(b) and the per-entity
// constant E_e built at load time, the per-query constant C_q built by the
// pack kernel. The sum is a dense [rows x 2d] . [2d x N] contraction of the
// packed query rows [alpha | beta] with the entity rows [U | V], so it runs
// on the matrix cores; the VALU form is bound by the half-rate FMA issue of
// the vector units.
//
// Tiling (mfma_tile.hpp). The contraction runs on v_mfma_f32_16x16x32_f16 with
// both operands split ahead into two f16 parts and scaled by row (the entity
// rows at load, the query rows by the pack kernel) and three part products
// kept (MfmaTileF16x2, tiles of 128 entities x 128 query rows, 64 KiB of LDS,
// two workgroups per compute unit; smaller ones for small calls):
// k_score_kl_split. All its terms are positive, and its error against 64 bits
// is that of the 32-bit sum. At the 63,361-entity workload it took the scorer
// from 1.21 ms (three bf16 parts, six products, the query rows split in the
// loop) to 0.69 ms; 61 queries at 14,505 entities from 25.8 us to 14.2.
// The smallest calls, below 16 dimensions, and KGQ_DENSE_FP32: tiles of 64 or
// 32 rows x 64 entities on v_mfma_f32_16x16x4_f32 with full FP32 inputs,
// through the direct-to-LDS ring of three stages when 2d is a multiple of 16,
// else the register-staged loop. Its epilogue adds C_q + E_e in double precision, stages the output
// tile in LDS, takes the max over union groups of four and pairs of rows and
// writes each output row with 16-byte non-temporal stores.
// The split kernel also writes, per output row and chunk of 64 entities, the
// largest key of the chunk's scores, from which top-k skips the chunks that
// cannot hold an answer.
// Workgroups are ordered in chunks of row tiles (about 2 MiB of query rows),
// each swept against every entity tile: the chunk's rows stay in L2 while
// the entity table streams past.
#include <algorithm>

#include "kgq_internal.hpp"
#include "mfma_tile.hpp"

namespace kgq {

// x of the lane that the DPP control names (quad permutations).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, false));
}

// Workgroup tiles of rows x entities: 64 x 64 on the direct-to-LDS loop, 32 x 64
// as long as every tile has a compute unit to itself (launch_lds); on the
// register-staged loop 128 x 128, or 64 x 64 for small batches, where the
// larger tile leaves the chip underfilled and each workgroup's K loop is a
// latency chain. Query rows are not padded: rows past the last are read from it.
template <class KlTile>
__global__ __launch_bounds__(256, 2) void k_score_kl(ScoreArgs a, int n_mt, int n_nt, int qchunk, int total,
                                                     int per_xcd)
{
    constexpr int KL_BM = KlTile::kBM, KL_BN = KlTile::kBN;
    extern __shared__ __align__(16) float sm[];   // set at launch

    // XCD-aware order (workgroup b runs on XCD b % 8): chunks of qchunk row
    // tiles, then entity tiles, then the chunk's row tiles.
    const int b = blockIdx.x;
    const int L = (b & 7) * per_xcd + (b >> 3);
    if (L >= total) return;
    const int chunk_wg = qchunk * n_nt;
    const int c = L / chunk_wg;
    const int r = L - c * chunk_wg;
    const int qcc = min(qchunk, n_mt - c * qchunk);
    const int nt = r / qcc;
    const int mt = c * qchunk + (r - nt * qcc);
    const int m0 = mt * KL_BM, n0 = nt * KL_BN;

    // Entity rows are padded (with zeros) to a multiple of 256, so the tile's
    // columns are inside; query rows past the last are read from it.
    const int n_ent_pad = (int)(a.n_blocks * kEntBlock);
    v4f acc[KlTile::TM][KlTile::TN];
    KlTile::run(a.qpack, 2 * a.d, a.n_rows, a.ent, 2 * a.d, n_ent_pad, 2 * a.d, m0, n0, sm, acc);

    // Epilogue, staged through LDS (the ring is free after the K loop):
    //   1. each lane subtracts E_e and its accumulators from gamma - C_q (one
    //      per row, hoisted) in double precision
    //      and writes the scores of its 4 rows x 1 column per MFMA tile into
    //      a BM x BN tile (rows padded by 4 floats: the 16 lanes of a column
    //      group and the 4 row groups hit distinct banks, and rows stay
    //      16-byte aligned);
    //   2. BN / 4 threads per row read whole rows back, take the max over a
    //      union group of four rows or a pair (groups start at multiples of
    //      4, pairs at even rows, neither crosses a tile) and write each
    //      output row with 16-byte non-temporal stores, so the score matrix
    //      streams past L2 in whole lines instead of 64-byte pieces that
    //      evict the entity rows still to be read.
    // E_e is padded to the entity blocks; rows past the last read the last
    // row's constants and never reach the output.
    constexpr int TLD = KL_BN + 4;
    constexpr int THREADS = 256;
    static_assert(KL_BN % 4 == 0 && THREADS % (KL_BN / 4) == 0 && KL_BM % (THREADS / (KL_BN / 4)) == 0, "output row pieces");
    // The output rows of the thread's rows in step 2, loaded now and waited
    // for once before it: a load inside its loop would wait (vmcnt) for the
    // stores issued before it as well. (Rows past the last are clamped to
    // it: no branch, so the loads issue back to back.)
    constexpr int C4 = KL_BN / 4, RPP = THREADS / C4;     // 16-byte pieces per row, rows per pass
    constexpr int NIT = KL_BM / RPP;
    const int r0 = threadIdx.x / C4;
    int32_t od[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int m = min(m0 + r0 + it * RPP, a.n_rows - 1);
        od[it] = a.out_dest[score_out_index(m, a.n_quad, a.n_pair)];
    }
    __syncthreads();                                  // every wavefront is done with the ring
    float* T = sm;
    double gq[KlTile::TM][4];                         // gamma - C_q of the lane's rows, once per tile
#pragma unroll
    for (int i = 0; i < KlTile::TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) gq[i][q] = (double)a.gamma - a.cq[min(m0 + KlTile::row_of(i) + q, a.n_rows - 1)];
#pragma unroll
    for (int j = 0; j < KlTile::TN; ++j) {
        const int cj = KlTile::col_of(j);
        const double ee = a.ee[n0 + cj];
#pragma unroll
        for (int i = 0; i < KlTile::TM; ++i) {
            const int rb = KlTile::row_of(i);
#pragma unroll
            for (int q = 0; q < 4; ++q) T[(rb + q) * TLD + cj] = (float)((gq[i][q] - ee) - (double)acc[i][j][q]);
        }
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);          // the output rows
    __syncthreads();
    const int c4 = threadIdx.x % C4;
    const int64_t n = n0 + 4 * c4;
    if (n >= a.N) return;
    const int n_grouped = a.n_quad + a.n_pair;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int r = r0 + it * RPP;
        const int m = m0 + r;
        if (m >= a.n_rows) break;                     // rows only grow along the loop
        int cnt = 1;
        if (m < a.n_quad) {
            if (m & 3) continue;                      // inside a group of four
            cnt = 4;
        } else if (m < n_grouped) {
            if ((m - a.n_quad) & 1) continue;         // second row of a pair
            cnt = 2;
        }
        const float* t = T + r * TLD + 4 * c4;
        float4 v = *reinterpret_cast<const float4*>(t);
        for (int u = 1; u < cnt; ++u) {
            const float4 w = *reinterpret_cast<const float4*>(t + u * TLD);
            v = make_float4(fmaxf(v.x, w.x), fmaxf(v.y, w.y), fmaxf(v.z, w.z), fmaxf(v.w, w.w));
        }
        const int64_t orow = od[it];
        float* dst = a.scores + orow * a.ld + n;
        if (n + 3 < a.N) {
            // rows start only 4-byte aligned; gfx950 takes dword-aligned
            // multi-dword global stores
            typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
            __builtin_nontemporal_store((f4u_t){v.x, v.y, v.z, v.w}, reinterpret_cast<f4u_t*>(dst));
        } else {
            const float e4[4] = {v.x, v.y, v.z, v.w};
            for (int jj = 0; jj < 4; ++jj)
                if (n + jj < a.N) __builtin_nontemporal_store(e4[jj], dst + jj);
        }
    }
}

// Split form on the f16 matrix cores (MfmaTileF16x2): the entity rows are
// operand A and the query rows B, so a lane holds 4 consecutive entities of
// one query row in each block and the epilogue stays in registers: no LDS
// tile, no barrier, and the 64 entities of a wavefront are one chunk key.
// Through an LDS tile like the FP32 kernel's the epilogue took 0.22 of 0.77 ms
// at the 63,361-entity workload (2,341 rows), 0.05 of it for the stores; in
// registers 0.18. The rest was the slot of a workgroup standing empty between
// tiles (constants' loads, stores draining, the next workgroup's start and
// first stage), so two workgroups per compute unit stay and take tile after
// tile: a tile's last stage requests the next tile's first, and the wait for
// the epilogue's constants, before its stores, covers it: 0.69 ms.
template <class Tile>
__global__ __launch_bounds__(Tile::kThreads, 2) void k_score_kl_split(ScoreArgs a, int n_qt, int n_et, int qchunk,
                                                                      int total, int per_xcd)
{
    constexpr int BE = Tile::kBM, BQ = Tile::kBN;      // entities, query rows of a tile
    extern __shared__ __align__(16) float sm[];
    // XCD-aware order as in k_score_kl (chunks of qchunk query tiles, then
    // entity tiles, then the chunk's query tiles): XCD x has positions
    // [x * per_xcd, (x + 1) * per_xcd), its workgroups take them in turn
    const int xcd0 = (blockIdx.x & 7) * per_xcd;
    const int n_mine = min(per_xcd, total - xcd0), n_wg = gridDim.x >> 3;
    const int64_t ld = plane_ld(2 * a.d);
    const int nk = (int)(ld / 32);
    auto locate = [&](int p, int& e0, int& q0) {
        const int L = xcd0 + p;
        const int chunk_wg = qchunk * n_et;
        const int c = L / chunk_wg;
        const int r = L - c * chunk_wg;
        const int qcc = min(qchunk, n_qt - c * qchunk);
        const int et = r / qcc;
        e0 = et * BE;
        q0 = (c * qchunk + (r - et * qcc)) * BQ;
    };
    int pos = blockIdx.x >> 3;
    if (pos >= n_mine) return;
    // the ring's requests run S - 1 stages ahead of the products, over the ends
    // of tiles: the next stage to ask for, its tile and slot
    constexpr int S = Tile::kSlots;
    typename Tile::Loader loader;
    int ipos = pos, ikt = 0, islot = 0;
    auto request = [&] {
        if (ipos >= n_mine) return;
        if (ikt == 0) {
            int e0, q0;
            locate(ipos, e0, q0);
            loader.set(a.ent_split, ld, (int)(a.n_blocks * kEntBlock), a.qpack, ld, a.n_rows, e0, q0);
        }
        loader.issue(ikt, sm, islot);
        islot = islot + 1 == S ? 0 : islot + 1;
        if (++ikt == nk) {
            ikt = 0;
            ipos += n_wg;
        }
    };
    int slot = 0;
#pragma unroll
    for (int t = 0; t < S - 1; ++t) request();
    wait_vm_barrier<0>();
    for (;;) {
        v4f acc[Tile::TM][Tile::TN], low[Tile::TM][Tile::TN];
        Tile::clear(acc, low);
        int te0, tq0;
        locate(pos, te0, tq0);
        for (int kt = 0; kt < nk; ++kt) {
            // (a tile's first stage landed before the loop or the last stores)
            if (kt > 0) {
                if (S > 2 && ipos < n_mine) wait_vm_barrier<(S - 2) * Tile::LPS>();   // S - 2 later stages asked for
                else wait_vm_barrier<0>();
            }
            Tile::stage(sm, slot, acc, low, request);
            slot = slot + 1 == S ? 0 : slot + 1;
        }
        pos += n_wg;
        const bool more = pos < n_mine;

        // The lane's query rows (one per block column; past the last: the last's
        // constants, nothing stored) and entities (the table's constants are
        // padded to whole blocks). Loaded before the first store and waited for
        // once: a load issued later would wait (vmcnt) for the stores before it.
        constexpr int TM = Tile::TM, TN = Tile::TN;
        double gq[TN];
        float sq[TN];
        int32_t od[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int m = min(tq0 + Tile::col_of(j), a.n_rows - 1);
            gq[j] = a.cq[m];
            sq[j] = a.q_scale[m];
            od[j] = a.out_dest[score_out_index(m, a.n_quad, a.n_pair)];
        }
        // scores in place: gamma - C_q - E_e - the contraction (the large sum plus
        // the small ones', in the two rows' scales), in double precision
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int e = te0 + Tile::row_of(i);
            double ee[4];
            float se[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ee[q] = (double)a.gamma - a.ee[e + q];
                se[q] = a.ent_scale[e + q];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v = fmaf(low[i][j][q], kSplitLow, acc[i][j][q]) * (sq[j] * se[q]);
                    acc[i][j][q] = (float)((ee[q] - gq[j]) - (double)v);
                }
        }
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);                  // the constants, and the next tile's first stage
        const int n_grouped = a.n_quad + a.n_pair;
        const int64_t ew = te0 + Tile::row_of(0);                  // the lane's first entity
        const bool tail = te0 + BE > a.N;                          // the last entity tile
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int m = tq0 + Tile::col_of(j);
            // union groups of four rows and pairs: the maximum over a quad of
            // lanes or a pair; its first lane stores
            bool first = m < a.n_rows;
            if (m - (int)(threadIdx.x & 15) < n_grouped) {        // (the same for the 16 lanes of a block column)
                const bool quad = m < a.n_quad, pair = !quad && m < n_grouped;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float v = acc[i][j][q];
                        const float p = fmaxf(v, dpp_f32<0xB1>(v));          // lanes 1, 0, 3, 2
                        const float f = fmaxf(p, dpp_f32<0x4E>(p));          // lanes 2, 3, 0, 1
                        acc[i][j][q] = quad ? f : pair ? p : v;
                    }
                if (quad) first = first && (m & 3) == 0;
                else if (pair) first = first && ((m - a.n_quad) & 1) == 0;
            }
            float* dst = a.scores + od[j] * a.ld + ew;
            float kmax = -__builtin_inff();
            bool nan = false;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                v4f v = acc[i][j];
                if (!tail) {
                    typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
                    if (first) *reinterpret_cast<f4u_t*>(dst + i * 16) = v;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const bool in = ew + i * 16 + q < a.N;
                        if (first && in) dst[i * 16 + q] = v[q];
                        v[q] = in ? v[q] : -__builtin_inff();
                    }
                }
                kmax = fmaxf(kmax, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
                nan = nan || __builtin_isunordered(v.x, v.y) || __builtin_isunordered(v.z, v.w);
            }
            if (a.chunk_key) {
                // the largest key of the lane's scores: the key of their float
                // maximum (the scores order as their keys, NaN aside), or
                // where one is NaN of each key by itself. No bound above it:
                // the k-th largest chunk key is top-k's first threshold, which
                // k scores have to reach.
                uint32_t kx = ew < a.N ? score_key(kmax) : 0u;
                if (nan) {
                    kx = 0u;
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (ew + i * 16 + q < a.N) kx = max(kx, score_key(acc[i][j][q]));
                }
                kx = max(kx, (uint32_t)__shfl_xor((int)kx, 16, 64));
                kx = max(kx, (uint32_t)__shfl_xor((int)kx, 32, 64));
                const int64_t chunk0 = te0 + (Tile::row_of(0) & ~(kKeyChunk - 1));
                if (first && (threadIdx.x & 48) == 0 && chunk0 < a.N)
                    a.chunk_key[od[j] * a.key_ld + chunk0 / kKeyChunk] = max(kx, 1u);
            }
        }
        if (!more) return;
        // every wavefront's part of the next tile's first stage has landed
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

// Query-tile chunk: as many tiles as ~2 MiB of query rows (about half an
// XCD's L2). The entity table is streamed once per chunk, and the XCDs split
// the global order evenly whatever the chunk size, so larger chunks cost no
// balance.
static int tile_chunk(int n_tiles, int rows, int64_t row_floats)
{
    return (int)std::min<int64_t>(n_tiles, std::max<int64_t>(1, (int64_t)(2 << 20) / (rows * row_floats * 4)));
}

// Dynamic LDS above the 64 KiB static limit: raised once per device and kernel.
template <class Kernel>
static void raise_lds(Kernel k, int bytes, bool (&raised)[64])
{
    int dev = 0;
    if (bytes > 65536 && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64 && !raised[dev])
        raised[dev] = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

template <class Tile>
static void launch_split(const ScoreArgs& a, hipStream_t s)
{
    static_assert(Tile::TM * 16 == kKeyChunk, "a wavefront's entities are one chunk");
    const int n_qt = (a.n_rows + Tile::kBN - 1) / Tile::kBN;
    const int n_et = (int)((a.N + Tile::kBM - 1) / Tile::kBM);
    const int total = n_qt * n_et, per_xcd = (total + 7) / 8;
    static bool raised[64] = {};
    raise_lds(k_score_kl_split<Tile>, Tile::SMEM * 4, raised);
    // per XCD: as many as LDS takes on each of 32 compute units (160 KB), at most 4
    const int n_wg = std::min(per_xcd, 32 * std::min(4, 163840 / (Tile::SMEM * 4)));
    hipLaunchKernelGGL((k_score_kl_split<Tile>), dim3(n_wg * 8), dim3(Tile::kThreads), Tile::SMEM * 4, s, a, n_qt, n_et,
                       tile_chunk(n_qt, Tile::kBN, plane_ld(2 * a.d)), total, per_xcd);
}

template <class Tile>
static void launch_tiles(const ScoreArgs& a, hipStream_t s)
{
    constexpr int BM = Tile::kBM, BN = Tile::kBN;
    const int n_mt = (a.n_rows + BM - 1) / BM;
    const int n_nt = (int)((a.N + BN - 1) / BN);
    const int total = n_mt * n_nt;
    const int per_xcd = (total + 7) / 8;
    constexpr int lds = std::max(Tile::SMEM, BM * (BN + 4)) * 4;    // the tile ring, then the output tile over it
    static bool raised[64] = {};
    raise_lds(k_score_kl<Tile>, lds, raised);
    hipLaunchKernelGGL((k_score_kl<Tile>), dim3(per_xcd * 8), dim3(256), lds, s, a, n_mt, n_nt,
                       tile_chunk(n_mt, BM, 2 * a.d), total, per_xcd);
}

// The split form from more than one FP32 tile (64 x 64) per compute unit on.
// Below, the FP32 tiles take about as long (one query at 14,505 entities 13.8
// us against 12.8, 64 at 3,000 13.2 against 13.0).
bool score_kl_takes_split(int n_rows, int64_t N, bool always)
{
    return always || (int64_t)((n_rows + 63) / 64) * ((N + 63) / 64) > 256;
}

// FP32 tiles on the direct-to-LDS ring: 64 x 64, or 32 rows as long as every
// tile has a compute unit to itself, whose chain of products is the time (one
// query at 14,505 entities 21.2 -> 13.8 us, 64 at 3,000 19.9 -> 13.2; with two
// tiles on a unit both take 21). The sums are the same; more slots give nothing.
template <bool HALF>
static void launch_lds(const ScoreArgs& a, hipStream_t s)
{
    if (((a.n_rows + 31) / 32) * ((a.N + 63) / 64) <= 256) launch_tiles<MfmaTileLds<32, 64, 3, HALF>>(a, s);
    else launch_tiles<MfmaTileLds<64, 64, 3, HALF>>(a, s);
}

bool launch_score_kl(const ScoreArgs& a, hipStream_t s)
{
    if (a.n_rows <= 0) return false;
    // Split tiles: the largest that still gives every compute unit work, on
    // rings that keep enough bytes in flight where a tile has few products.
    // Measured at d = 400, us a launch, by (entities, rows), 128 x 128 | 128 x
    // 64 | 64 x 64 | 64 x 32: (14505, 1) 26 | 18 | 14.3 | 12.8; (14505, 61)
    // 25.8 | 17.8 | 14.2 | 14.7; (14505, 128) 26 | 19.6 | 18.0 | 23; (14505,
    // 256) 28 | 25.6 | 30 | 37; (14505, 512) 38.6 | 44 | 54 | 60; (63361, 1)
    // 41 | 33.5 | 35 | 33.3; (63361, 64) 42 | 35 | 37.5 | 41; (63361, 128) 46 |
    // 53 | 66 | 74. So 64 x 64 and 128 x 64 while one round of two a compute
    // unit holds them. The large tile with 4 wavefronts: 256 entities x 128 rows and 128 x
    // 256 with 8 took 10 and 23 % longer at 63,361 x 2,341.
    if (a.ent_split) {
        auto tiles = [&](int be, int bq) { return ((a.N + be - 1) / be) * ((a.n_rows + bq - 1) / bq); };
        constexpr int64_t kRound = 512;
        if (a.n_rows <= 32) launch_split<MfmaTileF16x2<64, 32, 1, 2, 4>>(a, s);
        else if (tiles(64, 64) <= kRound) launch_split<MfmaTileF16x2<64, 64, 1, 4, 4>>(a, s);
        else if (tiles(128, 64) <= kRound) launch_split<MfmaTileF16x2<128, 64, 2, 2, 3>>(a, s);
        else launch_split<MfmaTileF16x2<128, 128, 2, 2, 2>>(a, s);
        return a.chunk_key != nullptr;
    }
    if (2 * a.d % 32 == 0) {
        launch_lds<false>(a, s);
    } else if (2 * a.d % 32 == 16) {
        launch_lds<true>(a, s);
    } else {
        const int64_t big_tiles = (int64_t)((a.n_rows + 127) / 128) * ((a.N + 127) / 128);
        if (big_tiles < 512) launch_tiles<MfmaTileReg<64, 64>>(a, s);
        else launch_tiles<MfmaTileReg<128, 128>>(a, s);
    }
    return false;
}

}  // namespace kgq
