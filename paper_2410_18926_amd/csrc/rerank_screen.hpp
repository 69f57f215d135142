// Exact re-rank with screened candidates (Sec. 2.2 last step; Sec. 4.1: the original d-dimensional query).
//
// The re-rank reads m rows per query from HBM to return k of them.  Here all m rows are read once at HALF the width - from
// a binary16 copy of the corpus, on the matrix cores - and only the few that can still be among the k best are read in full:
//   k_screen_union   per group of up to 16 queries the union of their candidate rows (LDS hash table), and the group's queries
//                    as binary16 columns;
//   k_screen_gather  every distinct row of a group once, contracted against all queries of the group with
//                    v_mfma_f32_16x16x32_f16 (rows of the product: 16 corpus rows, columns: 16 queries); the approximate
//                    dissimilarities of the (query, candidate) entries are written in the order of the group's list;
//   k_screen_finish  per query: the k-th smallest approximate value, the candidates within twice the error bound of it, their
//                    exact dissimilarities - same arithmetic, same order as in the kernels that evaluate every candidate - and
//                    the k smallest (distance, id).
// The result is the plain re-rank's, bit for bit: a candidate is dropped only if the bound PROVES that k others are nearer.
//
// Error bound.  q^ = binary16(s q) / s with s the power of two that brings max|s q| into [512, 1024) (elements below
// binary16's normal range are set to 0), x^ = the stored binary16 row, dq = q - q^, dx = x - x^:
//   <q^, x^> - <q, x> = -<dq, x> - <q^, dx>,   so   |.| <= |dq| |x| + |q^| |dx|            (an identity and Cauchy-Schwarz)
// |dq|, |q^| are the query's actual norms; |x| and |dx| enter through their maxima over the corpus (inner product, cosine) or
// through |x| of the row and the largest |dx| / |x| (Euclidean, where norms may be heavy-tailed and |x|^2 is read anyway),
// measured when the copy is made.  An element of x^ in binary16's subnormal range counts as lost altogether, so nothing
// rests on how the matrix core treats such inputs.  The products are exact in float; the K additions of the matrix core add
// at most K 2^-23 |q^| |x^| even if it truncates.  The exact value is itself a float sum: d/64 + 10 roundings in a chain add
// (d/64 + 16) 2^-24 |q| |x|.  All norms are rounded up by 1e-3 relative.
// With E the bound, A_k the k-th smallest approximate value: k candidates have an exact value <= A_k + E, so everything among
// the k best (ties included) has an approximate value <= A_k + 2 E.  Values that are not numbers are never dropped.
// Where a float sum of the exact evaluation may overflow (|q| |x| beyond 1e38, or the |q| a cosine is divided by), values that are far
// apart tie at an infinity or at one, and the lowest ids win: every candidate of such a query is kept.  (Euclidean: a query of that
// length has c0 beyond every 2 |q| |x|, the rows of the copy being at most 65504 sqrt(d) long.)
#pragma once
#include "common.hpp"
#include "rerank.hpp"
#include "rerank_group.hpp"
#include "score_mfma.hpp"

namespace lorann {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

constexpr int kScreenGroup = 16;          // queries per group: the columns of one matrix-core tile
constexpr int kScreenEntries = 3276;      // (query, candidate) entries of a group: 0.8 of a 4096-slot table (32 KiB of LDS; four blocks of eight wavefronts fill a CU)
constexpr int kScreenSlots = 4096;
constexpr int kScreenUnionThreads = 512;
constexpr int kScreenPerThread = (kScreenEntries + kScreenUnionThreads - 1) / kScreenUnionThreads;
constexpr float kHalfMin = 6.103515625e-5f;       // smallest normal binary16

// Row stride of the binary16 copy in elements: whole k-steps of the matrix-core instruction (32), zero padded.
inline int half_stride(int d) { return (d + 31) & ~31; }

// Queries per group for m candidates each.
inline int screen_group_size(int m) { return m >= kScreenEntries / 2 ? 1 : (kScreenEntries / m < kScreenGroup ? kScreenEntries / m : kScreenGroup); }

// Measured, one MI355X, microseconds per launch: 1M x 768, batch 10 000, m = 200: union 32 -> 36, gather 556 -> 283, finish / top-k
// 18 -> 79 (11 rows per query in full); 1M x 1024, m = 300: 66 + 1572 + 28 -> 61 + 783 + 118.  The gather reads its rows at 5.0 TB/s
// (5.9 TB/s at 2 KB rows); reading them as streaming data costs a third of that (283 -> 379): a row's 128-byte lines are
// requested in two halves, and the second half must still find the line in the cache.

// What the copy lost, as maxima over the rows (non-negative floats, rounded up): the ingredients of the error bound.
struct HalfStats {
    float abs_max;      // |x|_inf (a NaN compares above everything as bits)
    float norm;         // |x|
    float err;          // |dx|: rounding error, elements in the subnormal range lost altogether
    float lost;         // |x^| over the elements in the subnormal range alone (what the matrix core may lose of the stored row)
    float rel_err;      // |dx| / |x|
    float rel_round;    // |x - x^| / |x|
    float rel_lost;     // lost / |x^|
};

// dst[row][0 .. ld) = binary16(src[row][0 .. d)), zero padded; *st = the maxima above (float bits, cleared before).
// One wavefront per row, grid-stride, block = 256; one set of atomics per block (per wavefront they took longer than the copy).
__global__ __launch_bounds__(256) void k_corpus_to_half_rows(const float* __restrict__ src, _Float16* __restrict__ dst, int64_t n, int d, int ld,
                                                             uint32_t* __restrict__ st) {
    const int lane = threadIdx.x & 63;
    __shared__ uint32_t s_mx[7];
    if (threadIdx.x < 7) s_mx[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t mx[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
    for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < n; row += (int64_t)gridDim.x * 4) {
        const float* p = src + (size_t)row * d;
        _Float16* o = dst + (size_t)row * ld;
        uint32_t am = 0u;
        double nn = 0.0, er = 0.0, rd = 0.0, ls = 0.0, nh = 0.0;
        for (int i = lane; i < ld; i += 64) {
            const float x = i < d ? p[i] : 0.0f;
            am = max(am, __float_as_uint(x) & 0x7fffffffu);
            const _Float16 h = (_Float16)x;
            o[i] = h;
            const double xd = (double)x, hd = (double)(float)h, e = xd - hd;
            const bool sub = fabsf((float)h) < kHalfMin;
            nn += xd * xd; rd += e * e; nh += hd * hd;
            er += sub ? fmax(xd * xd, e * e) : e * e;
            ls += sub ? hd * hd : 0.0;
        }
        nn = wave_sum_f64(nn); er = wave_sum_f64(er); rd = wave_sum_f64(rd); ls = wave_sum_f64(ls); nh = wave_sum_f64(nh);
        auto up = [](double v) { return __float_as_uint((float)(sqrt(v) * (1.0 + 1e-6))); };
        mx[0] = max(mx[0], am);
        mx[1] = max(mx[1], up(nn)); mx[2] = max(mx[2], up(er)); mx[3] = max(mx[3], up(ls));
        if (nn > 0.0) { mx[4] = max(mx[4], up(er / nn)); mx[5] = max(mx[5], up(rd / nn)); }
        if (nh > 0.0) mx[6] = max(mx[6], up(ls / nh));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx[0] = max(mx[0], (uint32_t)__shfl_xor((int)mx[0], o, 64));
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 7; ++i) atomicMax(&s_mx[i], mx[i]);
    }
    __syncthreads();
    if (threadIdx.x < 7) atomicMax(&st[threadIdx.x], s_mx[threadIdx.x]);
}

// Rows of the corpus as queries, evenly spaced: dst[i] = row (2 i + 1) n / (2 count).  grid = count, block = 256.
__global__ __launch_bounds__(256) void k_sample_rows(const float* __restrict__ corpus, float* __restrict__ dst, int64_t n, int d, int count) {
    const size_t row = (size_t)((2 * (int64_t)blockIdx.x + 1) * n / (2 * (int64_t)count));
    for (int i = threadIdx.x; i < d; i += 256) dst[(size_t)blockIdx.x * d + i] = corpus[row * d + i];
}

struct ScreenRerankArgs {
    const float* Q;              // [nq][d]
    const void* corpus;          // rows the exact dissimilarities are taken from: float [n][d] or binary16 [n][ld]
    const _Float16* half;        // [n][ld]  the binary16 copy
    const float* sqnorm;         // [n] |x|^2 of the float rows (Euclidean) or NULL
    const int64_t* ids;          // [n] or NULL
    const int32_t* cand;         // [nq][m] candidate rows, valid ones first, -1 padded
    const int32_t* qorder;       // [nq] visiting order
    _Float16* qhalf;             // [ngroups][gq][ld] the groups' queries, scaled
    float4* qstat;               // [nq] x: E (inner product, cosine) or c1 (Euclidean), y: c2, z: c0, w: 1 / s
    int32_t* u_row;              // [ngroups][gstride] distinct rows of each group
    uint32_t* u_meta;            // [ngroups][gstride] low half: bit g = query g wants the row; high half: its first entry
                                 //                    (one entry per query that wants the row, queries ascending)
    uint16_t* entry;             // [nq][m] number of each candidate's entry in its group's list
    int32_t* qgroup;             // [nq] group of each query
    int32_t* u_count;            // [ngroups] number of distinct rows
    float* approx;               // [ngroups][gstride] approximate dissimilarity of each entry; Euclidean: [..][2] lower and upper
                                 //                    bound of the exact one
    int64_t* out_ids;            // [nq][k]
    float* out_dists;            // [nq][k]
    int32_t* kept;               // [nq] candidates that were read in full, or NULL
    int nq, d, ld, m, k, gq, slices;
    int gstride;                 // entries of a group's lists: gq * m rounded up to whole tiles of 16
    int metric;                  // 0 inner product, 1 squared Euclidean, 2 cosine
    // the bound's ingredients: norm >= |x|, err >= |dx| (inner product, cosine); rel_err >= |dx| / |x|,
    // rel_norm >= | |x^|^2 - |x|^2 | / |x|^2 (Euclidean: the norms of the float rows are what is stored)
    // nscale >= |row the distance is taken from| / |float row|
    float norm, err, rel_err, rel_norm, nscale;
};

// grid = ngroups, block = kScreenUnionThreads, dynamic LDS = 8 * kScreenSlots (gq > 1).
// Bound by latency (a chain of LDS atomics and a few round trips to L2), so all of a thread's candidates are requested at once
// and their table slots stay in registers.
__global__ __launch_bounds__(kScreenUnionThreads) void k_screen_union(ScreenRerankArgs a) {
    constexpr int NT = kScreenUnionThreads;
    extern __shared__ __align__(16) unsigned char smem[];
    int32_t* tkey = reinterpret_cast<int32_t*>(smem);                        // [kScreenSlots]
    uint32_t* tmeta = reinterpret_cast<uint32_t*>(tkey + kScreenSlots);      // [kScreenSlots] mask, then mask | offset << 16
    __shared__ int s_q[kScreenGroup];
    __shared__ int s_rows, s_entries;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int grp = blockIdx.x, g0 = grp * a.gq, ng = min(a.gq, a.nq - g0);
    const int m = a.m, total = ng * m;
    const size_t gbase = (size_t)grp * a.gstride;
    if (tid < kScreenGroup) {
        const int q = a.qorder[g0 + min(tid, ng - 1)];
        s_q[tid] = q;
        if (tid < ng) a.qgroup[q] = grp;
    }
    if (tid == 0) { s_rows = 0; s_entries = 0; }
    if (a.gq > 1)
        for (int s = tid; s < kScreenSlots; s += NT) { tkey[s] = -1; tmeta[s] = 0u; }
    __syncthreads();
    int rows[kScreenPerThread], slot[kScreenPerThread];
    if (a.gq > 1) {
#pragma unroll
        for (int u = 0; u < kScreenPerThread; ++u) {
            const int t = min(u * NT + tid, total - 1), g = t / m;
            rows[u] = a.cand[(size_t)s_q[g] * m + (t - g * m)];
        }
    }
    // the group's queries as binary16 columns, their scales and error bounds: one wavefront per query
    for (int g = wv; g < ng; g += NT / 64) {
        const int q = s_q[g];
        const float* qr = a.Q + (size_t)q * a.d;
        float am = 0.0f;
        for (int i = lane; i < a.d; i += 64) am = fmaxf(am, fabsf(qr[i]));
        am = wave_max_f32(am);
        int e = 0;
        (void)frexpf(am, &e);                                  // am = f * 2^e, f in [0.5, 1)
        e = am > 0.0f && am < INFINITY ? max(-118, min(127, 10 - e)) : 0;
        const float s = ldexpf(1.0f, e), inv = ldexpf(1.0f, -e);
        float nn = 0.0f, ne = 0.0f, nh = 0.0f;                 // of s q: |.|^2, |rounding error|^2, |rounded|^2
        _Float16* o = a.qhalf + ((size_t)grp * a.gq + g) * a.ld;
        for (int i = lane; i < a.ld; i += 64) {
            const float x = i < a.d ? qr[i] * s : 0.0f;
            _Float16 h = (_Float16)x;
            if (fabsf((float)h) < kHalfMin) h = (_Float16)0.0f;
            o[i] = h;
            const float hf = (float)h, er = x - hf;
            nn = fmaf(x, x, nn); ne = fmaf(er, er, ne); nh = fmaf(hf, hf, nh);
        }
        nn = wave_sum_f32(nn); ne = wave_sum_f32(ne); nh = wave_sum_f32(nh);
        if (lane == 0) {
            const float qn = sqrtf(nn) * 1.001f, qe = sqrtf(ne) * 1.001f, qh = sqrtf(nh) * 1.001f;
            const float acc = (float)a.ld * 1.1920929e-7f, gam = (float)(a.d / 64 + 20) * 6.6e-8f;
            float4 st;
            if (a.metric == 1) {
                // |q|, ... in the query's own scale; bound = c1 |x| + c2 |x|^2 + c0
                const float n1 = qn * inv, e1 = qe * inv, h1 = qh * inv;
                st.x = 1.002f * (2.0f * (e1 + h1 * a.rel_err + acc * h1 * (1.0f + a.rel_err)) + 2.0f * gam * n1 + 9.6e-7f * n1);
                st.y = 1.002f * (gam * a.nscale * a.nscale + 4.8e-7f + a.rel_norm);
                st.z = 1.002f * gam * n1 * n1 + 1e-37f;
            } else {
                // in the scaled query's units; cosine: 1 - v / |q| rounds, so values that differ by a few 2^-24 |q| may tie
                st.x = 1.001f * (qe * a.norm + qh * a.err + acc * qh * (a.norm + a.err) + gam * qn * a.norm +
                                 (a.metric == 2 ? 4.8e-7f * qn * (1.0f + a.norm) : 0.0f)) + s * 1.4e-45f * (float)(a.d + 64) + 1e-30f;
                if (!(qn * inv * (a.norm + a.err) < 1e38f)) st.x = INFINITY;         // a partial sum of the exact value may overflow
                st.y = 0.0f; st.z = 0.0f;
            }
            st.w = inv;
            a.qstat[q] = st;
        }
    }
    if (a.gq == 1) {          // one query per group: its candidates are distinct rows
        int n = 0;
        for (int t0 = 0; t0 < m; t0 += NT) {                   // uniform
            const int t = t0 + tid;
            const int row = t < m ? a.cand[(size_t)s_q[0] * m + t] : -1;
            if (row >= 0) { a.u_row[gbase + t] = row; a.u_meta[gbase + t] = 1u | ((uint32_t)t << 16); a.entry[(size_t)s_q[0] * m + t] = (uint16_t)t; }
            n += row >= 0 ? 1 : 0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
        if (lane == 0 && n) atomicAdd(&s_rows, n);
        __syncthreads();
        if (tid == 0) a.u_count[grp] = s_rows;
        return;
    }
    // open addressing, key = row
#pragma unroll
    for (int u = 0; u < kScreenPerThread; ++u) {
        slot[u] = -1;
        const int t = u * NT + tid;
        if (t < total && rows[u] >= 0) {
            const int g = t / m;
            uint32_t h = ((uint32_t)rows[u] * 2654435761u) >> 7;
            for (;;) {
                h &= (uint32_t)(kScreenSlots - 1);
                const int old = atomicCAS(&tkey[h], -1, rows[u]);
                if (old == -1 || old == rows[u]) { atomicOr(&tmeta[h], 1u << g); slot[u] = (int)h; break; }
                ++h;
            }
        }
    }
    __syncthreads();
    for (int s0 = 0; s0 < kScreenSlots; s0 += NT) {            // number the rows and their entries, a wavefront at a time
        const int s = s0 + tid;
        const int row = tkey[s];
        const uint32_t mask = tmeta[s];
        const int mine = __popc(mask);
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (lane >= o) incl += t; }
        const unsigned long long used = __ballot(row >= 0);
        int base_r = 0, base_e = 0;
        if (lane == 63) { base_r = atomicAdd(&s_rows, __popcll(used)); base_e = atomicAdd(&s_entries, incl); }
        base_r = __builtin_amdgcn_readlane(base_r, 63); base_e = __builtin_amdgcn_readlane(base_e, 63);
        if (row >= 0) {
            const int at = base_r + __popcll(used & ((1ull << lane) - 1ull));
            const uint32_t meta = mask | ((uint32_t)(base_e + incl - mine) << 16);
            a.u_row[gbase + at] = row;
            a.u_meta[gbase + at] = meta;
            tmeta[s] = meta;
        }
    }
    __syncthreads();
    if (tid == 0) a.u_count[grp] = s_rows;
#pragma unroll
    for (int u = 0; u < kScreenPerThread; ++u) {
        if (slot[u] >= 0) {
            const int t = u * NT + tid, g = t / m;
            const uint32_t meta = tmeta[slot[u]];
            a.entry[(size_t)s_q[g] * m + (t - g * m)] = (uint16_t)((meta >> 16) + __popc(meta & ((1u << g) - 1u)));
        }
    }
}

// grid = ngroups * slices, block = 256 (4 independent wavefronts), dynamic LDS = gq * (2 * ld + 16) bytes: the group's queries,
// rows padded by 16 bytes against bank conflicts.
// A wavefront takes tiles of 16 rows.  Operand layout of v_mfma_f32_16x16x32_f16 (measured on gfx950 with its int8 sibling): lane l
// holds eight consecutive k (k-group l / 16) of row / column l % 16; result register v of lane l is D[4 * (l / 16) + v][l % 16].
// So a lane loads 16 bytes of one row per k-step, the four lanes of a row 64 consecutive bytes, and rows go straight from memory
// into the registers that feed the matrix core.  Chunks of KC k-steps, two requested ahead across tile borders.
// Bound by HBM: per 16-row tile of 1.5 KB rows 24 KB are read for 24 matrix-core instructions.
template <bool L2>
__global__ __launch_bounds__(256) void k_screen_gather(ScreenRerankArgs a) {
    constexpr int KC = 4;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int grp = blockIdx.x / a.slices, sl = blockIdx.x - grp * a.slices;
    const int g0 = grp * a.gq, ng = min(a.gq, a.nq - g0);
    const int nuniq = a.u_count[grp];
    const int ntiles = (nuniq + 15) >> 4;
    const int per = (ntiles + a.slices - 1) / a.slices;
    const int t_beg = sl * per, t_end = min(ntiles, t_beg + per);
    if (t_beg >= t_end) return;                                 // uniform over the block
    const int ld = a.ld;
    const int qstride = 2 * ld + 16;
    {
        const int pieces = ld >> 3;                             // 16-byte pieces of a query
        const uint4* src = reinterpret_cast<const uint4*>(a.qhalf + (size_t)grp * a.gq * ld);
#pragma unroll 4
        for (int t = tid; t < ng * pieces; t += 256) {
            const int g = t / pieces, i = t - g * pieces;
            *reinterpret_cast<uint4*>(smem + g * qstride + 16 * i) = src[t];
        }
    }
    __syncthreads();
    const int i16 = lane & 15, kg = lane >> 4;
    const unsigned char* qb = smem + min(i16, ng - 1) * qstride + 16 * kg;
    const int q = a.qorder[g0 + min(i16, ng - 1)];              // this lane's column
    const float4 qs = a.qstat[q];
    const size_t gbase = (size_t)grp * a.gstride;
    float* out = a.approx + gbase * (L2 ? 2 : 1);
    const int nk = ld >> 5, nchunks = (nk + KC - 1) / KC;
    const uint32_t below = (1u << i16) - 1u;
    int tile = t_beg + wv, chunk = 0;
    if (tile >= t_end) return;                                  // no block barrier below
    const int n_steps = ((t_end - tile + 3) >> 2) * nchunks;

    // Loads return in order, so what a step waits for must have been requested before the rows that are still to come: row
    // numbers run two tiles ahead of the rows, (mask, entry) words two tiles ahead of their use, norms one.
    auto row_of = [&](int t) { return a.u_row[gbase + min(16 * min(t, t_end - 1) + i16, nuniq - 1)]; };      // clamped: unconditional loads
    auto words_of = [&](const void* p, int t) { return *reinterpret_cast<const i32x4*>(static_cast<const int32_t*>(p) + gbase + 16 * min(t, t_end - 1) + 4 * kg); };
    f16x8 st[3][KC];
    int p_tile = tile, p_chunk = 0;                             // next chunk to request
    int p_next = row_of(p_tile + 4), p_next2 = row_of(p_tile + 8);
    const _Float16* p_row = a.half + (size_t)row_of(p_tile) * ld + 8 * kg;
    auto request = [&](f16x8 (&dst)[KC]) {
#pragma unroll
        for (int u = 0; u < KC; ++u) dst[u] = *reinterpret_cast<const f16x8*>(p_row + 32 * min(p_chunk * KC + u, nk - 1));
        if (++p_chunk == nchunks) {                             // uniform
            p_chunk = 0;
            p_tile += 4;
            p_row = a.half + (size_t)p_next * ld + 8 * kg;
            p_next = p_next2;
            p_next2 = row_of(p_tile + 8);
        }
    };
    i32x4 meta = words_of(a.u_meta, tile), meta1 = words_of(a.u_meta, tile + 4), rows1 = {0, 0, 0, 0};      // of this tile, of the next
    float nrm[4] = {0.0f, 0.0f, 0.0f, 0.0f}, nrm1[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto norms = [&](const i32x4& rw, int t, float (&n4)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) n4[v] = a.sqnorm[16 * min(t, t_end - 1) + 4 * kg + v < nuniq ? rw[v] : 0];
    };
    if (L2) { norms(words_of(a.u_row, tile), tile, nrm); rows1 = words_of(a.u_row, tile + 4); }
    f32x4v acc = {0.0f, 0.0f, 0.0f, 0.0f};
    request(st[0]);
    request(st[1]);
    i32x4 meta2;
    for (int s0 = 0; s0 < n_steps; s0 += 3) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if (s0 + b < n_steps) {                             // uniform
                if (chunk == 0) {
                    meta2 = words_of(a.u_meta, tile + 8);
                    if (L2) { norms(rows1, tile + 4, nrm1); rows1 = words_of(a.u_row, tile + 8); }
                }
                request(st[(b + 2) % 3]);
#pragma unroll
                for (int u = 0; u < KC; ++u) {
                    if (chunk * KC + u < nk) {                  // uniform
                        const f16x8 bq = *reinterpret_cast<const f16x8*>(qb + 64 * (chunk * KC + u));
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(st[b][u], bq, acc, 0, 0, 0);
                    }
                }
                if (++chunk == nchunks) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const uint32_t mk = (uint32_t)meta[v];
                        if (((mk >> i16) & 1u) && 16 * tile + 4 * kg + v < nuniq) {
                            const uint32_t at = (mk >> 16) + __popc(mk & below);
                            if (L2) {
                                const float n2 = nrm[v], n1 = sqrtf(n2) * a.nscale;
                                const float val = fmaf(-2.0f * qs.w, acc[v], n2);
                                const float e = fmaf(qs.x, n1, fmaf(qs.y, n2, qs.z));
                                *reinterpret_cast<float2*>(out + 2 * at) = make_float2(val - e, val + e);
                            } else {
                                out[at] = -acc[v];
                            }
                        }
                        nrm[v] = nrm1[v];
                    }
                    meta = meta1;
                    meta1 = meta2;
                    acc = (f32x4v){0.0f, 0.0f, 0.0f, 0.0f};
                    chunk = 0;
                    tile += 4;
                }
            }
        }
    }
}

// SW wavefronts per query choose the survivors (EPL candidates per lane, m <= 64 * SW * EPL), RW of them read their rows:
//   SW = RW = 1   four queries per block
//   SW = 1, RW = 4   one query per block: the survivors' rows - about k - are in flight together
//   SW = RW = 4   one query per block, many candidates
// grid = ceil(nq / (4 / RW)), block = 256, dynamic LDS = (4 / RW) * 64 * SW * EPL * 12 bytes.
// NV, T as in k_group_gather (NV = 0: any d); VEC: d % 4 == 0, a lane owns elements 4 (lane + 64 v) .. + 3, else elements lane + 64 j.
template <bool L2, int NV, bool VEC, typename T, int SW, int RW, int EPL>
__global__ __launch_bounds__(256) void k_screen_finish(ScreenRerankArgs a) {
    const bool cosine = a.metric == 2;
    constexpr int QPB = 4 / RW, CAP = 64 * SW * EPL;
    constexpr int RB = NV == 0 ? 1 : RW == 4 || sizeof(T) == 2 || NV <= 2 ? 4 : 2;     // rows in flight per wavefront
    using V = typename Row4<T>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_cnt[4], s_part[2][4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int sub = RW == 1 ? wv : 0, w0 = RW == 1 ? 0 : wv;             // query of the block, wavefront of the query
    const int64_t q = (int64_t)blockIdx.x * QPB + sub;
    if (q >= a.nq) return;                                               // RW = 4: never; RW = 1: wavefronts are independent
    int64_t* s_id = reinterpret_cast<int64_t*>(smem) + (size_t)sub * CAP;                                   // row, then id of each survivor
    uint32_t* s_key = reinterpret_cast<uint32_t*>(smem + (size_t)QPB * CAP * 8) + (size_t)sub * CAP;        // order-preserving key of its distance
    auto meet = [&]() { if (RW == 1) wave_lds_sync(); else __syncthreads(); };
    auto meet_sel = [&]() { if (SW == 1) wave_lds_sync(); else __syncthreads(); };
    const int m = a.m, d = a.d;
    const int32_t* crow = a.cand + (size_t)q * m;
    const uint16_t* erow = a.entry + (size_t)q * m;
    const size_t gbase = (size_t)a.qgroup[q] * a.gstride;
    const int ldr = sizeof(T) == 2 ? a.ld : d;
    const T* corpus = static_cast<const T*>(a.corpus);
    const float* qrow = a.Q + (size_t)q * d;
    const int d4 = d % 4 == 0 ? d >> 2 : 0;
    float4 y[NV > 0 ? NV : 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (VEC) y[v] = reinterpret_cast<const float4*>(qrow)[min(lane + 64 * v, d4 - 1)];
        else y[v] = make_float4(qrow[min(lane + 256 * v, d - 1)], qrow[min(lane + 256 * v + 64, d - 1)], qrow[min(lane + 256 * v + 128, d - 1)], qrow[min(lane + 256 * v + 192, d - 1)]);
    }
    float qn = 0.0f;
    if (cosine) {
        float acc = 0.0f;
        for (int i = lane; i < d; i += 64) acc = fmaf(qrow[i], qrow[i], acc);
        qn = sqrtf(wave_sum_f32(acc));
    }
    if (SW == RW || w0 == 0) {                                            // uniform over the wavefront
    const float4 qs = a.qstat[q];
    int row[EPL], at[EPL];
    float lo[EPL];
    uint32_t key[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {                                       // clamped addresses: the loads go out together
        const int t = (e * SW + w0) * 64 + lane, tc = min(t, m - 1);
        row[e] = crow[tc];
        at[e] = erow[tc];
        if (t >= m) row[e] = -1;
    }
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const size_t ec = gbase + (row[e] >= 0 ? at[e] : 0);
        if (L2) { const float2 b = reinterpret_cast<const float2*>(a.approx)[ec]; lo[e] = b.x; key[e] = float_key_asc(b.y); }
        else { lo[e] = a.approx[ec]; key[e] = float_key_asc(lo[e]); }
    }
    int par = 0;
    auto count = [&](auto f) {                                            // over all candidates of the query (uniform result)
        int c = 0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) c += __popcll(__ballot(row[e] >= 0 && f(e)));
        if (SW > 1) {
            if (lane == 0) s_part[par][wv] = c;
            __syncthreads();
            c = s_part[par][0] + s_part[par][1] + s_part[par][2] + s_part[par][3];
            par ^= 1;             // (two sets of counters: one barrier per count keeps readers and the next writers apart)
        }
        return c;
    };
    const int cnt = count([&](int) { return true; });
    const int kk = min(a.k, cnt);
    // the kk-th smallest upper bound, its last 8 bits rounded up (a slightly larger threshold is as safe)
    uint32_t kth = 0u;
    if (kk > 0) {
        for (int b = 31; b >= 8; --b) {
            const uint32_t probe = kth | (1u << b);
            if (count([&](int e) { return key[e] < probe; }) < kk) kth = probe;
        }
    }
    float thr = key_to_float(kth | 255u);
    if (!L2) thr += 2.0f * qs.x;
    thr += 1e-6f * fabsf(thr);
    if (cosine && !(qn > 1e-15f && qn < INFINITY)) thr = NAN;      // (a query of length zero or infinity ties with everything: nothing is dropped)
    if (lane == 0 && w0 == 0) s_cnt[sub] = 0;
    meet_sel();
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const bool in = row[e] >= 0 && !(lo[e] > thr);
        const unsigned long long mk = __ballot(in);
        int base = 0;
        if (lane == 0 && mk) base = atomicAdd(&s_cnt[sub], __popcll(mk));
        base = __builtin_amdgcn_readfirstlane(base);
        if (in) s_id[base + __popcll(mk & ((1ull << lane) - 1ull))] = row[e];
    }
    }
    meet();
    const int c = s_cnt[sub];
    if (a.kept && lane == 0 && w0 == 0) a.kept[q] = c;
    auto finish = [&](int i, float acc) {       // lane 63 records the distance of survivor i
        float dist;
        if (L2) dist = acc;
        else if (!cosine) dist = -acc;
        else dist = qn > 0.0f ? 1.0f - acc / qn : 1.0f;
        s_key[i] = min(float_key_asc(dist), float_key_asc(INFINITY));
    };
    for (int i0 = w0 * RB; i0 < c; i0 += RW * RB) {
        if constexpr (NV > 0) {
            float4 x[RB][NV];
            if constexpr (VEC) {
                V xs[RB][NV];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int rw = __builtin_amdgcn_readfirstlane((int)s_id[min(i0 + r, c - 1)]);
                    const V* p4 = reinterpret_cast<const V*>(corpus + (size_t)rw * ldr);
#pragma unroll
                    for (int v = 0; v < NV; ++v) xs[r][v] = row_load(p4 + min(lane + 64 * v, d4 - 1));
                }
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int v = 0; v < NV; ++v) x[r][v] = widen4(xs[r][v]);
            } else {
                T xs[RB][4 * NV];
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int rw = __builtin_amdgcn_readfirstlane((int)s_id[min(i0 + r, c - 1)]);
                    const T* p = corpus + (size_t)rw * ldr;
#pragma unroll
                    for (int j = 0; j < 4 * NV; ++j) xs[r][j] = p[min(lane + 64 * j, d - 1)];
                }
#pragma unroll
                for (int r = 0; r < RB; ++r)
#pragma unroll
                    for (int v = 0; v < NV; ++v) x[r][v] = make_float4(widen1(xs[r][4 * v]), widen1(xs[r][4 * v + 1]), widen1(xs[r][4 * v + 2]), widen1(xs[r][4 * v + 3]));
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                if (i0 + r >= c) break;                                   // uniform
                float acc = 0.0f;
                auto add = [&](float qv, float xv) {
                    if (L2) { const float t = qv - xv; acc = fmaf(t, t, acc); }
                    else acc = fmaf(xv, qv, acc);
                };
#pragma unroll
                for (int v = 0; v < NV; ++v) {                            // only the last slice can be partial
                    const float4 yy = y[v], xv = x[r][v];
                    if (VEC) {
                        if (v + 1 < NV || lane + 64 * v < d4) { add(yy.x, xv.x); add(yy.y, xv.y); add(yy.z, xv.z); add(yy.w, xv.w); }
                    } else {
                        if (v + 1 < NV || lane + 256 * v < d) add(yy.x, xv.x);
                        if (v + 1 < NV || lane + 256 * v + 64 < d) add(yy.y, xv.y);
                        if (v + 1 < NV || lane + 256 * v + 128 < d) add(yy.z, xv.z);
                        if (v + 1 < NV || lane + 256 * v + 192 < d) add(yy.w, xv.w);
                    }
                }
                acc = wave_sum_f32_lane63(acc);
                if (lane == 63) finish(i0 + r, acc);
            }
        } else {
            const int rw = __builtin_amdgcn_readfirstlane((int)s_id[i0]);
            const T* p = corpus + (size_t)rw * ldr;
            float acc = 0.0f;
            if (d4) {
                const V* p4 = reinterpret_cast<const V*>(p);
                const float4* q4 = reinterpret_cast<const float4*>(qrow);
                for (int i = lane; i < d4; i += 64) {
                    const float4 xv = widen4(row_load(p4 + i)), yy = q4[i];
                    if (L2) {
                        const float a0 = yy.x - xv.x, a1 = yy.y - xv.y, a2 = yy.z - xv.z, a3 = yy.w - xv.w;
                        acc = fmaf(a0, a0, acc); acc = fmaf(a1, a1, acc); acc = fmaf(a2, a2, acc); acc = fmaf(a3, a3, acc);
                    } else {
                        acc = fmaf(xv.x, yy.x, acc); acc = fmaf(xv.y, yy.y, acc); acc = fmaf(xv.z, yy.z, acc); acc = fmaf(xv.w, yy.w, acc);
                    }
                }
            } else {
                for (int i = lane; i < d; i += 64) {
                    const float xv = widen1(p[i]);
                    if (L2) { const float t = qrow[i] - xv; acc = fmaf(t, t, acc); }
                    else acc = fmaf(xv, qrow[i], acc);
                }
            }
            acc = wave_sum_f32_lane63(acc);
            if (lane == 63) finish(i0, acc);
        }
    }
    meet();
    // rows -> ids, each by the thread that ranks the survivor
    const int first = w0 * 64 + lane, step = 64 * RW;
    for (int i = first; i < c; i += step) { const int64_t rw = s_id[i]; s_id[i] = a.ids ? a.ids[rw] : rw; }
    meet();
    for (int i = first; i < c; i += step) {
        const uint32_t mk = s_key[i];
        const int64_t mi = s_id[i];
        int rank = 0;
        for (int j = 0; j < c; ++j) {
            const uint32_t kj = s_key[j];
            const int64_t ij = s_id[j];
            rank += kj < mk || (kj == mk && (ij < mi || (ij == mi && j < i))) ? 1 : 0;
        }
        if (rank < a.k) { a.out_ids[q * a.k + rank] = mi; a.out_dists[q * a.k + rank] = key_to_float(mk); }
    }
    for (int i = c + first; i < a.k; i += step) { a.out_ids[q * a.k + i] = -1; a.out_dists[q * a.k + i] = INFINITY; }
}

}  // namespace lorann
