// Per-query candidate selection of the batched scoring path (the candidate-selection step of Sec. 2.2; the
// paper's candidate count t is called m here).
//
// k_pair_max has already computed, for every (query, cluster) pair, the best score of the cluster.  One block
// per query now walks the query's pairs in descending order of that best score and keeps a running threshold T,
// at most the m-th best score seen so far: a cluster whose best score is below T cannot contribute a candidate, and
// because the pairs are sorted the walk stops at the first such cluster.  A query's best candidates sit in very
// few of its w clusters, so typically one or two clusters are scored here (point-parallel, 4-way int8 dot
// products); all the others were dismissed by their maxima alone.  The scores that reach T are held in LDS and counted
// in bins, off which T is read whenever new ones have arrived; the exact top-m (score descending, row ascending) is
// selected once, at the end.  Only if more scores tie with T than LDS can hold does the query go to the exact
// per-query kernel.
#pragma once
#include "common.hpp"
#include "select_exact.hpp"

namespace lorann {

// m-th largest among the keys f(i), i in [0, n), for which f returns true (at least m of them, m >= 1).
// f(i, key&) -> bool.  Returns the key; need_ties = how many of the keys equal to it belong to the top m.
// hist: 256 ints of LDS; sh: 2 words of LDS.  Block = 256 threads; contains barriers, so every thread must
// call it with the same arguments.
template <typename F>
__device__ __forceinline__ uint32_t block_mth_largest(int n, int m, int* hist, uint32_t* sh, int& need_ties, F f) {
    const int tid = threadIdx.x;
    if (tid == 0) { sh[0] = 0u; sh[1] = (uint32_t)m; }
    uint32_t mask = 0u;
    for (int shift = 24; shift >= 0; shift -= 8) {
        hist[tid] = 0;
        __syncthreads();
        const uint32_t prefix = sh[0];
        for (int i = tid; i < n; i += 256) {
            uint32_t key;
            if (f(i, key) && (key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
        }
        __syncthreads();
        if (tid < 64) {     // descending digit walk: the digit where the count from the top reaches need
            const int need = (int)sh[1];
            const int h0 = hist[255 - 4 * tid], h1 = hist[254 - 4 * tid], h2 = hist[253 - 4 * tid], h3 = hist[252 - 4 * tid];
            const int mine = h0 + h1 + h2 + h3;
            int incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (tid >= o) incl += t; }
            const int excl = incl - mine;
            if (excl < need && incl >= need) {
                int cum = excl, dgt = 255 - 4 * tid;
                if (cum + h0 >= need) { }
                else { cum += h0; if (cum + h1 >= need) { dgt -= 1; } else { cum += h1; if (cum + h2 >= need) { dgt -= 2; } else { cum += h2; dgt -= 3; } } }
                sh[0] = prefix | ((uint32_t)dgt << shift);
                sh[1] = (uint32_t)(need - cum);
            }
        }
        mask |= 255u << shift;
        __syncthreads();
    }
    need_ties = (int)sh[1];
    const uint32_t T = sh[0];
    __syncthreads();
    return T;
}


// (score, row) entries a query holds in LDS: 2048 (16 KiB, more blocks per CU) or 6144 for m > 1024.
inline int select_query_cap(int m) { return m <= 1024 ? 2048 : 6144; }

// Block-wide minimum of `v` written to *dst (scratch: one int of LDS, clobbered).  Contains barriers.
__device__ __forceinline__ void block_min_to(int32_t* dst, int v, int* scratch) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    if (threadIdx.x == 0) *scratch = 0x7fffffff;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicMin(scratch, v);
    __syncthreads();
    if (threadIdx.x == 0) *dst = *scratch;
}

// Scores are counted in bins of their distance from the query's best one (known from the pair maxima), in the order-preserving
// key space: distances below 64 have a bin each, beyond that 64 bins per power of two, so the m-th best score is known to
// 1/64 of its distance from the best at any time, whatever the scores' scale.  (Sixteen per power of two left several hundred entries
// in the last bin at m = 300 and above, and ranking those took longer than the walk's last clusters.)
constexpr int kSelectBins = 1792;      // 28 * 64 >= 64 + 26 * 64
__device__ __forceinline__ int select_bin(uint32_t dist) {
    const int e = 31 - __clz((int)(dist | 1u));
    return e < 6 ? (int)dist : (e - 5) * 64 + (int)((dist >> (e - 6)) & 63u);
}
__device__ __forceinline__ uint32_t select_bin_first(int bin) { return bin < 64 ? (uint32_t)bin : (uint32_t)(64 + (bin & 63)) << ((bin >> 6) - 1); }
__device__ __forceinline__ uint32_t select_bin_last(int bin) { return select_bin_first(bin + 1) - 1u; }       // (wraps to 2^32 - 1 in the last bin)

struct QuerySelectArgs {
    const int32_t* sel;          // [nq][w] clusters of each query
    const int32_t* pos_of_slot;  // [nq*w]
    const uint32_t* pmax;        // [npairs] key of each pair's best score (0: the cluster is empty), bucket order
    const int8_t* Z;             // [npairs][r_pad] bucket order
    const float* sigma;          // [npairs] bucket order
    const int8_t* Bp;            // [n][r_pad]
    const int64_t* off;          // [L+1]
    const float* sqnorm;         // [n] (Euclidean) or NULL
    const float* pt_scale;       // [n] step size of each point's code (column-wise quantization) or NULL
    const float* pt_first;       // [n] unquantized first row of B_c (mixed-precision decomposition) or NULL
    const float* rho0;           // [npairs] bucket order: unquantized first component of each pair's r, or NULL
    int32_t* cand;               // out [nq][m]: candidate rows, unordered, -1 padded
    float* tau;                  // out [nq]: score of the m-th candidate (-inf if fewer than m points were scored)
    int32_t* n_kept;             // out [nq]: scores held in LDS when the walk ended (-1: handed to the exact kernel)
    int32_t* qkey;               // out [nq]: smallest candidate row (locality hint for the order of the re-rank)
    int32_t* fb_list;            // out: queries that need the exact per-query kernel
    int32_t* fb_count;           //      and their number (0 on entry)
    const int32_t* qorder;       // [nq] queries grouped by nearest cluster (visiting order)
    int nq, w, m;
    int cap;                     // select_query_cap(m)
    int run_shift;               // log2 of the queries per run (see the kernel)
    // large clusters (quarters.hpp), one-wavefront kernel only: best scores of the quarters of their work items, or NULL
    const uint32_t* sub;         // [places][64][4]
    const int32_t* bucket_off;   // [L+1]
    const int32_t* sub_first;    // [L]
    int sub_chunks, sub_groups;
};

// Dynamic LDS of k_select_query: the list and what is known of each pair.
inline size_t select_query_lds(int cap, int w) { return (size_t)cap * 8 + (size_t)w * 28; }

// grid = 512 * ceil(nq / 512), block = 256, dynamic LDS = select_query_lds bytes.  RB = r_pad / 16; EXT: column-wise step sizes
// (and, if pt_first is given, the mixed-precision decomposition).
// Queries are visited grouped by nearest cluster (workgroups are dealt round-robin over the 8 XCDs): queries that
// score the same cluster run together and share its codes in L2.
// INLINE_FB (small batches): a query whose survivor list overflows is finished right here by the exact per-query
// routine instead of being handed to a later launch.
//
// Bound by latency: a typical query scores one or two clusters of a thousand points.  So everything about the w pairs is fetched in
// one round trip, the four wavefronts walk a cluster on their own - pieces of 64 PT points, two pieces requested ahead, scores that
// reach T appended under one atomic per wavefront - and meet only at its end (or when the list is nearly full), where one wavefront
// reads the new T off the bins.  The exact selection happens once, over the few entries of the m-th score's bin.
template <int RB, bool L2, bool EXT, bool INLINE_FB>
__global__ __launch_bounds__(256) void k_select_query(QuerySelectArgs a) {
    constexpr int ZW = RB * 4, PT = RB == 2 ? 2 : 1, PIECE = 64 * PT;
    extern __shared__ __align__(16) unsigned char qs_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = a.w, m = a.m, cap = a.cap;
    uint32_t* keys = reinterpret_cast<uint32_t*>(qs_smem);               // [cap]
    int32_t* rows = reinterpret_cast<int32_t*>(keys + cap);              // [cap]
    uint32_t* pk = reinterpret_cast<uint32_t*>(rows + cap);              // [w] key of the pair's best score
    int* ppos = reinterpret_cast<int*>(pk + w);                          // [w] position of the pair, first row, points, scale, first component of r
    int* prow = ppos + w;
    int* pcnt = prow + w;
    float* psig = reinterpret_cast<float*>(pcnt + w);
    float* prho = psig + w;
    int* order = reinterpret_cast<int*>(prho + w);
    __shared__ __align__(16) int bins[kSelectBins];                                    // later: (key, row) entries of one bin
    __shared__ int hist[256];
    __shared__ int wsum[4];
    __shared__ uint32_t sh[2], s_T;
    __shared__ int s_count, s_more[2], s_bin, s_out, s_ties;
    // position in the visiting order: runs of 64 consecutive queries go to one XCD (they share clusters and hence
    // codes in that XCD's L2), successive runs to successive XCDs - a popular, large cluster (many queries, each
    // with much to score) is spread over all of them instead of making one XCD the last to finish
    const int slot = (int)(blockIdx.x >> 3);
    const int rs = a.run_shift;
    const int si = ((((slot >> rs) << 3) + (int)(blockIdx.x & 7)) << rs) + (slot & ((1 << rs) - 1));
    if (si >= a.nq) return;
    const int q = __builtin_amdgcn_readfirstlane(a.qorder[si]);     // uniform over the block: scalar loads below
    const bool mixed = EXT && a.pt_first != nullptr;
    if (tid == 0) { s_count = 0; s_more[0] = 0; s_more[1] = 0; s_T = 0u; }
    if (tid < w) {
        const int pos = a.pos_of_slot[(size_t)q * w + tid], c = a.sel[(size_t)q * w + tid];
        const int64_t r0 = a.off[c], r1 = a.off[c + 1];
        const float s = a.sigma[pos];
        pk[tid] = a.pmax[pos];
        ppos[tid] = pos;
        prow[tid] = (int)r0; pcnt[tid] = (int)(r1 - r0);
        psig[tid] = L2 ? 2.0f * s : s;
        const float rf = mixed ? a.rho0[pos] : 0.0f;
        prho[tid] = L2 ? 2.0f * rf : rf;
    }
    for (int i = tid; i < kSelectBins; i += 256) bins[i] = 0;
    __syncthreads();
    if (tid < w) {      // order the pairs by best score, descending (ties: lower rank first)
        const uint32_t k = pk[tid];
        int rank = 0;
        for (int u = 0; u < w; ++u) rank += (pk[u] > k || (pk[u] == k && u < tid)) ? 1 : 0;
        order[rank] = tid;
    }
    __syncthreads();

    const uint32_t kmax = pk[order[0]];      // key of the best score of all
    uint32_t T = 0u;          // running threshold key, at most the m-th best score seen so far (0: none yet)
    float Tf = -INFINITY;     // the same as a score
    bool overflow = false;
    int par = 0;
    const int limit = cap - 4 * PIECE;       // a wavefront adds at most one piece after it has seen the count at or below this

    // Keep the list's entries >= T only (stable, in place); returns how many.
    auto filter = [&](int n) {
        int kept = 0;
        for (int base = 0; base < n; base += 256) {
            const int i = base + tid;
            uint32_t k = 0u;
            int32_t r = 0;
            if (i < n) { k = keys[i]; r = rows[i]; }
            const bool keep = i < n && k >= T;
            int tot;
            const int rank = block_flag_scan<4>(keep, wsum, tot);     // barriers: the chunk is in registers before any write
            if (keep) { keys[kept + rank] = k; rows[kept + rank] = r; }
            kept += tot;
        }
        __syncthreads();
        if (tid == 0) s_count = kept;
        return kept;
    };
    // T from the bins: the far edge of the bin that holds the m-th best score seen (all four wavefronts meet around it).
    auto read_bins = [&]() {
        if (wv == 0) {
            constexpr int PL = kSelectBins / 64;         // 28 consecutive bins per lane
            int mine = 0;
            const i32x4* b4 = reinterpret_cast<const i32x4*>(bins) + lane * (PL / 4);
#pragma unroll
            for (int j = 0; j < PL / 4; ++j) { const i32x4 h = b4[j]; mine += (h[0] + h[1]) + (h[2] + h[3]); }
            int incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) { const int t = __shfl_up(incl, o, 64); if (lane >= o) incl += t; }
            // the lane whose run holds the m-th best; its bins are then looked through one per lane
            const int src = __ffsll((unsigned long long)__ballot(incl >= m)) - 1;
            const int cum = __builtin_amdgcn_readlane(incl - mine, src);
            int x = lane < PL ? bins[src * PL + lane] : 0;
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) { const int t = __shfl_up(x, o, 64); if (lane >= o) x += t; }
            const int j = __ffsll((unsigned long long)__ballot(cum + x >= m)) - 1;
            if (lane == 0) {
                const uint32_t last = select_bin_last(src * PL + j);
                s_bin = src * PL + j;
                s_T = kmax > last ? kmax - last : 0u;
            }
        }
    };

    for (int o = 0; o < w && !overflow; ++o) {
        const int jp = __builtin_amdgcn_readfirstlane(order[o]);
        const uint32_t best = pk[jp];
        if (best == 0u || best < T) break;               // sorted: no later cluster can reach T either (uniform)
        const int m_c = __builtin_amdgcn_readfirstlane(pcnt[jp]), r0 = __builtin_amdgcn_readfirstlane(prow[jp]);
        const float sp = psig[jp], r0p = prho[jp];
        const i32x4* zp = reinterpret_cast<const i32x4*>(a.Z) + (size_t)__builtin_amdgcn_readfirstlane(ppos[jp]) * RB;
        i32x4 zv[RB];                                    // (in flight with the first codes)
#pragma unroll
        for (int u = 0; u < RB; ++u) zv[u] = zp[u];
        i32x4 code[3][PT][RB];
        float bias[3][PT], psc[3][PT], pf[3][PT];
        // clamped addresses instead of branches, so that the loads overlap (m_c > 0: the pair has a best score)
        auto request = [&](int b, int piece) {
#pragma unroll
            for (int e = 0; e < PT; ++e) {
                const size_t row = (size_t)r0 + min(piece * PIECE + e * 64 + lane, m_c - 1);
                const i32x4* bp = reinterpret_cast<const i32x4*>(a.Bp) + row * RB;
#pragma unroll
                for (int u = 0; u < RB; ++u) code[b][e][u] = bp[u];
                if (L2) bias[b][e] = a.sqnorm[row];
                if (EXT) { psc[b][e] = a.pt_scale[row]; pf[b][e] = mixed ? a.pt_first[row] : 0.0f; }
            }
        };
        const int pieces = (m_c + PIECE - 1) / PIECE;
        int piece = wv;
        int z[ZW];                                       // uniform: scalar registers
        for (;;) {
            if (piece < pieces) {
                request(0, piece);
                request(1, piece + 4);
#pragma unroll
                for (int u = 0; u < ZW; ++u) z[u] = __builtin_amdgcn_readfirstlane(zv[u >> 2][u & 3]);
                bool full = false;
                while (piece < pieces && !full) {        // uniform over the wavefront
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        if (piece < pieces && !full) {
                            full = __builtin_amdgcn_readfirstlane(*(volatile int*)&s_count) > limit;
                            if (!full) {
                                request((b + 2) % 3, piece + 8);
#pragma unroll
                                for (int e = 0; e < PT; ++e) {
                                    const int t = piece * PIECE + e * 64 + lane;
                                    int y = 0;
#pragma unroll
                                    for (int u = 0; u < RB; ++u)
#pragma unroll
                                        for (int x = 0; x < 4; ++x) y = dot4_i8(code[b][e][u][x], z[4 * u + x], y);
                                    float sc = __fmaf_rn((float)y, EXT ? __fmul_rn(sp, psc[b][e]) : sp, L2 ? -bias[b][e] : -0.0f);
                                    if (EXT && mixed) sc = __fmaf_rn(r0p, pf[b][e], sc);
                                    const bool in = t < m_c && !(sc < Tf);
                                    const unsigned long long mk = __ballot(in);
                                    if (mk) {
                                        int base = 0;
                                        if (lane == 0) base = atomicAdd(&s_count, __popcll(mk));
                                        base = __builtin_amdgcn_readfirstlane(base);
                                        if (in) {
                                            const uint32_t key = float_key_asc(sc);
                                            const int at = base + __popcll(mk & ((1ull << lane) - 1ull));
                                            keys[at] = key;
                                            rows[at] = r0 + t;
                                            atomicAdd(&bins[select_bin(key < kmax ? kmax - key : 0u)], 1);
                                        }
                                    }
                                }
                                piece += 4;
                            }
                        }
                    }
                }
            }
            if (piece < pieces && lane == 0) s_more[par] = 1;
            __syncthreads();
            const int n = s_count;                       // (nothing is added before the next barrier)
            const bool more = s_more[par] != 0;
            if (tid == 0) s_more[par ^ 1] = 0;
            if (n >= m) read_bins();                     // uniform
            __syncthreads();
            par ^= 1;
            if (s_T > T) T = s_T;
            if (n > limit) {                             // uniform
                int left = filter(n);
                if (left > limit) {                      // one bin holds too many: select exactly
                    __syncthreads();
                    int ties;
                    T = block_mth_largest(left, m, hist, sh, ties, [&](int i, uint32_t& key) { key = keys[i]; return true; });
                    left = filter(left);
                }
                __syncthreads();
                if (left > limit) { overflow = true; break; }     // too many scores tie with the threshold
            }
            Tf = T > 0x007fffffu ? key_to_float(T) : -INFINITY;
            if (!more) break;
        }
    }

    int32_t* out = a.cand + (size_t)q * m;
    if (overflow && INLINE_FB) {       // uniform
        if (tid == 0) { a.n_kept[q] = -1; a.tau[q] = key_to_float(T); a.qkey[q] = 0; }
        SelectArgs sa;
        sa.qlist = nullptr; sa.qcount = nullptr; sa.sel = a.sel; sa.pos_of_slot = a.pos_of_slot; sa.Z = a.Z; sa.sigma = a.sigma;
        sa.Bp = a.Bp; sa.off = a.off; sa.sqnorm = a.sqnorm; sa.pt_scale = a.pt_scale; sa.pt_first = a.pt_first; sa.rho0 = a.rho0;
        sa.cand = a.cand; sa.fb_total = nullptr; sa.w = w; sa.m = m;
        __syncthreads();
        select_exact_query<RB>(sa, q);
        return;
    }
    if (overflow) {
        if (tid == 0) {
            a.fb_list[atomicAdd(a.fb_count, 1)] = q; a.n_kept[q] = -1; a.tau[q] = key_to_float(T);
            a.qkey[q] = prow[order[0]];                  // first row of its most promising cluster
        }
        return;
    }
    const int count = s_count;
    int mn = 0x7fffffff;
    if (count < m) {        // every scored point is a candidate
        if (tid == 0) { a.n_kept[q] = count; a.tau[q] = -INFINITY; }
        for (int i = tid; i < m; i += 256) { const int r = i < count ? rows[i] : -1; out[i] = r; if (r >= 0) mn = min(mn, r); }
        block_min_to(a.qkey + q, mn, hist);
        return;
    }
    // The m-th best score lies in bin s_bin: entries of nearer bins are candidates, the bin's own are ranked (score descending,
    // row ascending).  Entries below T - an exact selection may have raised it into the bin - are none.
    const int bin = s_bin;
    const uint32_t dist0 = select_bin_first(bin), near = bin == 0 ? 0xffffffffu : kmax - dist0;       // keys of the bin: T .. near
    __syncthreads();
    if (tid == 0) { s_out = 0; s_ties = 0; a.n_kept[q] = count; }
    __syncthreads();
    uint32_t* bkey = reinterpret_cast<uint32_t*>(bins);
    int32_t* brow = reinterpret_cast<int32_t*>(bins) + 256;
    for (int i0 = 0; i0 < count; i0 += 256) {            // uniform
        const int i = i0 + tid;
        const uint32_t k = i < count ? keys[i] : 0u;
        const int32_t r = i < count ? rows[i] : 0;
        const bool above = k > near, member = k >= T && k <= near && k != 0u;
        const unsigned long long ma = __ballot(above), mb = __ballot(member);
        int ba = 0, bb = 0;
        if (lane == 0) { if (ma) ba = atomicAdd(&s_out, __popcll(ma)); if (mb) bb = atomicAdd(&s_ties, __popcll(mb)); }
        ba = __builtin_amdgcn_readfirstlane(ba); bb = __builtin_amdgcn_readfirstlane(bb);
        const unsigned long long below = (1ull << lane) - 1ull;
        if (above) { out[ba + __popcll(ma & below)] = r; mn = min(mn, r); }
        if (member) { const int at = bb + __popcll(mb & below); if (at < 256) { bkey[at] = k; brow[at] = r; } }
    }
    __syncthreads();
    const int n_above = s_out, nb = s_ties, need = m - n_above;
    if (nb <= 256) {                                     // uniform
        if (tid < nb) {
            const uint32_t k = bkey[tid];
            const int32_t r = brow[tid];
            int rank = 0;
            for (int u = 0; u < nb; ++u) rank += (bkey[u] > k || (bkey[u] == k && brow[u] < r)) ? 1 : 0;
            if (rank < need) { out[n_above + rank] = r; mn = min(mn, r); }
            if (rank == need - 1) a.tau[q] = key_to_float(k);
        }
    } else {
        // a long run of (nearly) equal scores: radix selection of the need-th best key of the bin, ties to the lower rows
        int ties, dummy;
        const uint32_t KT = block_mth_largest(count, need, hist, sh, ties, [&](int i, uint32_t& key) { key = keys[i]; return keys[i] >= T && keys[i] <= near; });
        const uint32_t RT = block_mth_largest(count, ties, hist, sh, dummy, [&](int i, uint32_t& key) { key = ~(uint32_t)rows[i]; return keys[i] == KT; });
        if (tid == 0) { s_out = n_above; a.tau[q] = key_to_float(KT); }
        __syncthreads();
        for (int i = tid; i < count; i += 256) {
            const uint32_t k = keys[i];
            if (k > near || k < KT || (k == KT && (~(uint32_t)rows[i]) < RT)) continue;
            out[atomicAdd(&s_out, 1)] = rows[i];
            mn = min(mn, rows[i]);
        }
    }
    block_min_to(a.qkey + q, mn, hist);
}

}  // namespace lorann
