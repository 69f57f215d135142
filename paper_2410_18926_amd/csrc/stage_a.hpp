// First 8-bit product and re-quantization (Sec. 3.3): for every (query, cluster) pair,
// R = q'_i8^T A_c in int32, z = round(127 R / max|R|) as int8, and the pair's combined scale
// sigma = max|R|/127 * Delta_x * DeltaA_c * DeltaB_c.  With one scalar DeltaA per cluster the
// de-quantize / re-quantize pair of Sec. 3.3 reduces to this integer expression.
//
// Pairs are grouped by cluster (counting sort), so one wavefront handles 16 pairs of the same cluster as an
// int8 matrix-core product  [16 pairs x d'] . [d' x r]  with v_mfma_i32_16x16x64_i8.
// Register layout of that instruction (measured on gfx950): both operands give lane l sixteen consecutive
// k-bytes of row/column l%16 (k-group l/16); result register v of lane l holds D[4*(l/16) + v][l%16].
#pragma once
#include "common.hpp"

namespace lorann {

__device__ __forceinline__ i32x4 load16(const int8_t* p) { return *reinterpret_cast<const i32x4*>(p); }

// Maximum over each row of 16 lanes, in every lane of the row (rotations inside the row, no LDS traffic).
__device__ __forceinline__ uint32_t row16_max_u32(uint32_t v) {
    auto turned = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, true); };
    v = max(v, turned(v, std::integral_constant<int, 0x128>{}));     // row_ror:8, 4, 2, 1
    v = max(v, turned(v, std::integral_constant<int, 0x124>{}));
    v = max(v, turned(v, std::integral_constant<int, 0x122>{}));
    v = max(v, turned(v, std::integral_constant<int, 0x121>{}));
    return v;
}

// slot / w by a multiplication: magic = ceil(2^32 / w).  Exact while slot * (magic * w - 2^32) < 2^32; the second factor is below w <= 256,
// and a launch has at most 2^15 * 256 slots.
inline uint32_t slot_division_magic(int w) { return (uint32_t)(((uint64_t(1) << 32) + (uint64_t)w - 1) / (uint64_t)w); }
__device__ __forceinline__ int query_of_slot(int slot, int w, uint32_t magic) { return w == 1 ? slot : (int)__umulhi((uint32_t)slot, magic); }

// Find c with off[c] <= t < off[c+1] (off non-decreasing, off[0] = 0, t < off[L]).
__device__ __forceinline__ int find_bucket(const int32_t* __restrict__ off, int L, int t) {
    int lo = 0, hi = L;   // invariant: off[lo] <= t < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// The same search done by a whole wavefront for one (uniform) t: every round the 64 lanes probe 64 evenly
// spaced entries of the current range, so the range shrinks 64-fold per dependent load instead of 2-fold.
__device__ __forceinline__ int find_bucket_wave(const int32_t* __restrict__ off, int L, int t) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = L;   // invariant: off[lo] <= t < off[hi]
    while (hi - lo > 1) {
        const int span = hi - lo;
        const int step = (span + 63) >> 6;                 // >= 1
        const int probe = lo + (lane + 1) * step;          // lo < probe; lanes beyond hi do not count
        const bool le = probe < hi && off[probe] <= t;
        const int n = __popcll(__ballot(le));              // off is non-decreasing: the first n probes are <= t
        const int nlo = lo + n * step;
        const int nhi = min(hi, nlo + step);
        lo = nlo; hi = nhi;
    }
    return lo;
}

// The same search started from a guess: if t lies within the 63 buckets from c_guess - 31 on, ONE round of probes
// finds it (buckets of similar size make an interpolated guess land that close); otherwise the full search runs.
__device__ __forceinline__ int find_bucket_near(const int32_t* __restrict__ off, int L, int t, int c_guess) {
    const int lane = threadIdx.x & 63;
    const int lo = max(0, min(c_guess - 31, L - 63));
    const int probe = min(lo + lane, L);
    const int n = __popcll(__ballot(off[probe] <= t));     // off is non-decreasing: the first n probes are <= t
    if (n >= 1 && n <= 63 && lo + n <= L) return lo + n - 1;     // off[lo + n - 1] <= t < off[lo + n]
    return find_bucket_wave(off, L, t);
}

// grid = ceil((npairs / 16 + L) / (4 * tpw)) blocks of 256: the 16-pair tiles of all clusters form one list
// (tile_off: tiles before each cluster) and every wavefront takes tpw consecutive tiles of it, so the work per
// wavefront is the same however unevenly the pairs are spread over the clusters; a wavefront whose tiles span
// several clusters serves them one after the other.  A_c stays in registers across the tiles of one cluster when
// d' <= 256.
// RT = r_pad / 16 result tiles (2 or 4); RES: d' <= 256, A_c resident.  A is [L][r][dp]; Z is [npairs][r_pad] in
// bucket order.
// COLS: column-wise quantization (Sec. 3.3 as printed) - sA is [L][r], one step size per column of A_c; the float
// approximation rho_j = R_j * (Delta_x * DeltaA_cj) is re-quantized like a query: z = rint(rho * 127 / |rho|_inf),
// sigma = |rho|_inf / 127 (every operation a single IEEE float operation); sB is not used.
// COLS with A_first != NULL (Sec. 4.2 mixed-precision decomposition; the queries' codes then have 0 in component
// 0): rho_j = fma(x_0, A_first[c][j], R_j * (Delta_x * DeltaA_cj)) with x_0 = qproj[query][0]; rho_0 goes to
// rho0[pair] as it is, z_0 = 0, and the maximum and the codes come from rho_1.. alone.
// Bound by latency: a tile is one chain (gather of the query codes, product, maximum of each row, codes, store), so the epilogue's
// inputs are requested in front of the product, the row maxima are register rotations, and the quotients need no division.
// Batch 10 000 on one MI355X, microseconds, before and after: L = 1024, d' = 256, r = 32 37 -> 28; L = 2048, r = 48 82 -> 53;
// d' = 128, r = 24, w = 64 58 -> 46; 1000 queries over L = 64 21 -> 14.
template <int RT, bool RES, bool COLS = false>
__global__ __launch_bounds__(256) void k_stage_a(const int8_t* __restrict__ q8, const float* __restrict__ dx,
                                                  const int8_t* __restrict__ A, const float* __restrict__ sA,
                                                  const float* __restrict__ sB, const int32_t* __restrict__ bucket_off,
                                                  const int32_t* __restrict__ tile_off, int tpw, int tiles_guess,
                                                  const int32_t* __restrict__ slot_of_pos,
                                                  int L, int dp, int r, int w, uint32_t w_magic, int8_t* __restrict__ Z, float* __restrict__ sigma,
                                                  const float* __restrict__ qproj = nullptr, const float* __restrict__ A_first = nullptr,
                                                  float* __restrict__ rho0 = nullptr) {
    const int lane = threadIdx.x & 63;
    const int i = lane & 15, g = lane >> 4;
    // this wavefront's tiles [g0, g1) of the list of all tiles; wavefronts are independent: no block barrier below
    const int gw = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int g0 = gw * tpw;
    const int g1 = min(g0 + tpw, tile_off[L]);
    if (g0 >= g1) return;
    // (tiles_guess: about how many tiles there are, for the first guess of the cluster that holds tile g0)
    int c = __builtin_amdgcn_readfirstlane(find_bucket_near(tile_off, L, g0, (int)((long long)g0 * L / max(1, tiles_guess))));
    for (; g0 < g1; ++c) {                                // clusters this wavefront's tiles belong to
    const int t_beg = tile_off[c], t_end = c + 1 < L ? tile_off[c + 1] : tile_off[L];
    if (t_end <= g0) continue;                            // (a cluster without pairs)
    const int first = g0 - t_beg, last = min(g1, t_end) - t_beg;      // its tiles [first, last) are ours
    g0 = t_beg + last;
    const int pbeg = bucket_off[c], end = bucket_off[c + 1];
    const int8_t* Ac = A + (size_t)c * r * dp;
    constexpr int SB = 4;                                // k-steps whose operands are requested together
    const int steps = (dp + 63) >> 6;                    // uniform trip count: the MFMA runs with all lanes on
    constexpr bool a_resident = RES;                     // requires steps <= SB
    const i32x4 zero4 = (i32x4){0, 0, 0, 0};

    // Operands are requested with clamped addresses instead of branches around the loads (so that they overlap)
    // and what lies outside the matrices is zeroed in registers afterwards.
    auto fetch_a = [&](int s0, i32x4 (&bv)[SB][RT]) {
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const int kc = min(64 * (s0 + u) + 16 * g, dp - 16);
#pragma unroll
            for (int t = 0; t < RT; ++t) bv[u][t] = load16(Ac + (size_t)min(t * 16 + i, r - 1) * dp + kc);
        }
#pragma unroll
        for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int t = 0; t < RT; ++t)
                if (!(t * 16 + i < r)) bv[u][t] = zero4;
    };
    i32x4 bres[RES ? SB : 1][RT];
    if constexpr (RES) fetch_a(0, bres);

    int slot_next = slot_of_pos[min(pbeg + first * 16 + i, end - 1)];
    for (int tile = first; tile < last; ++tile) {
    const int base = pbeg + tile * 16;
    const bool row_ok = base + i < end;
    const int8_t* qrow = q8 + (size_t)query_of_slot(slot_next, w, w_magic) * dp;
    // what the epilogue needs of the pairs is requested here, not where it is used: two dependent round trips per row otherwise
    // (lane i < 4 of row group g: pair 4 g + i)
    int eslot[COLS ? 4 : 1];
#pragma unroll
    for (int v = 0; v < (COLS ? 4 : 1); ++v) eslot[v] = slot_of_pos[min(base + 4 * g + (COLS ? v : (i & 3)), end - 1)];
    // the next tile's pair numbers are requested now, its query rows when this tile is done
    slot_next = slot_of_pos[min(base + 16 + i, end - 1)];

    i32x4 acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = zero4;
    float edx[COLS ? 4 : 1], ex0[COLS ? 4 : 1];
#pragma unroll
    for (int v = 0; v < (COLS ? 4 : 1); ++v) {
        const int qv = query_of_slot(eslot[v], w, w_magic);
        edx[v] = dx[qv];
        ex0[v] = COLS && A_first != nullptr ? qproj[(size_t)qv * dp] : 0.0f;
    }

    for (int s0 = 0; s0 < steps; s0 += SB) {
        i32x4 av[SB], bload[RES ? 1 : SB][RT];
#pragma unroll
        for (int u = 0; u < SB; ++u) av[u] = load16(qrow + min(64 * (s0 + u) + 16 * g, dp - 16));
        if constexpr (!RES) fetch_a(s0, bload);
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            if (s0 + u < steps) {                        // uniform
                // d' is a multiple of 16: a 16-byte group is all in or all out
                const bool a_ok = row_ok && 64 * (s0 + u) + 16 * g < dp;
                const i32x4 a = a_ok ? av[u] : zero4;
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, RES ? bres[RES ? u : 0][t] : bload[RES ? 0 : u][t], acc[t], 0, 0, 0);
            }
        }
    }

    // acc[t][v] = R[pair 4g+v][column 16t+i].  Row maximum over the r columns: over t here, over i by shuffles.
    if constexpr (COLS) {
        const bool mixed = A_first != nullptr;           // uniform
        float dA[RT], a0[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            dA[t] = sA[(size_t)c * r + min(t * 16 + i, r - 1)];
            a0[t] = mixed ? A_first[(size_t)c * r + min(t * 16 + i, r - 1)] : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int pos = base + 4 * g + v;
            const float dxq = edx[v], x0 = ex0[v];
            float rho[RT], mx = 0.0f;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                rho[t] = t * 16 + i < r ? __fmul_rn((float)acc[t][v], __fmul_rn(dxq, dA[t])) : 0.0f;
                if (mixed) {
                    if (t * 16 + i < r) rho[t] = __fmaf_rn(x0, a0[t], rho[t]);
                    if (t == 0 && i == 0) {                  // the unquantized first component of r
                        if (pos < end) rho0[pos] = rho[0];
                        rho[0] = 0.0f;                       // out of the maximum; its code is rint(0) = 0
                    }
                }
                mx = fmaxf(mx, fabsf(rho[t]));
            }
            mx = __uint_as_float(row16_max_u32(__float_as_uint(mx)));      // (non-negative: ordered like its bits; a NaN counts as the largest)
            if (pos < end) {
                const bool any = mx > 0.0f;
                const float cx = any ? (float)(127.0 / (double)mx) : 0.0f;
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    int zc = (int)rintf(__fmul_rn(rho[t], cx));
                    zc = max(-127, min(127, zc));
                    Z[(size_t)pos * (RT * 16) + t * 16 + i] = (int8_t)(any ? zc : 0);
                }
                if (i == 0) sigma[pos] = any ? (float)((double)mx / 127.0) : 0.0f;
            }
        }
        continue;
    }
    uint32_t mxs = 0u;                                   // lane i < 4: the maximum of row 4 g + i
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        uint32_t mx = 0;
#pragma unroll
        for (int t = 0; t < RT; ++t) mx = max(mx, (uint32_t)abs(acc[t][v]));
        mx = row16_max_u32(mx);
        mxs = i == v ? mx : mxs;
        // (254 a + mx) / (2 mx): the quotient (at most 127) from a float product, off by one at most, corrected by its remainder
        const uint32_t den = max(2u * mx, 1u);
        const float inv = __builtin_amdgcn_rcpf((float)den);
        const int pos = base + 4 * g + v;
        if (pos < end) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const int R = acc[t][v];
                const uint32_t num = 254u * (uint32_t)abs(R) + mx;        // < 2^32 because d' <= 1024
                uint32_t q = (uint32_t)((float)num * inv);
                const int32_t rem = (int32_t)(num - q * den);             // -den <= rem < 2 den < 2^27 (the exact quotient has 0 <= rem < den)
                q = rem < 0 ? q - 1u : rem >= (int32_t)den ? q + 1u : q;
                Z[(size_t)pos * (RT * 16) + t * 16 + i] = (int8_t)(R < 0 ? -(int)q : (int)q);
            }
        }
    }
    {
        const int pos = base + 4 * g + i;
        if (i < 4 && pos < end)
            sigma[pos] = mxs != 0u ? (float)((double)mxs / 127.0 * (double)edx[0] * (double)sA[c] * (double)sB[c]) : 0.0f;
    }
    }   // tiles of this cluster
    }   // clusters of this wavefront
}

}  // namespace lorann
