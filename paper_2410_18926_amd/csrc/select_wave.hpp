// Per-query candidate selection by ONE WAVEFRONT per query: the walk of select_query.hpp for batches that fill the machine.
//
// Same method - the query's pairs in descending order of their best score, a running threshold T read off bins of the
// scores' distances from the query's best one, the exact top-m selected once at the end - but nothing is shared between
// wavefronts: the number of held scores is a scalar, there are no barriers, and the memory latency of one query's short
// clusters is covered by the other queries of the SIMD instead of by its own four wavefronts waiting for each other.
// The list is shorter (512 or 1024 entries: LDS decides how many queries a CU holds) and is thinned out whenever it fills - down to
// the m best exactly if need be, ties to the lower rows, so that no number of equal scores overflows it.
// In a large cluster only the quarters of work items whose best score (kept by the scoring kernel) reaches T are looked at; those
// best scores, each of another point, first raise T themselves.
//
// Measured on one MI355X, microseconds per launch, against the block kernel as it was before its bins / with them: 1M x 768, batch
// 10 000, m = 200: 129 / 104 / 74; 1M x 1024 (rank 48, ten clusters per query): 600 / 612 / 495, bound by the 3.2 GB of codes that
// miss the L2s; 1M x 128 with heavy-tailed norms (a cluster of 144 000 points): 640 / 675 / 494, m = 10 there 317 / 234 / 201; both
// end on the few queries that look at a thousand pieces.  A piece costs some 40 vector instructions, twice that when scores arrive.
#pragma once
#include "score_mfma.hpp"
#include "select_query.hpp"
#include "walk_offsets.hpp"

namespace lorann {

constexpr int kWaveBins = 512;             // distances below 16 have a bin each, beyond that 16 bins per power of two (464 used)
__device__ __forceinline__ int wave_bin(uint32_t dist) {
    const int e = 31 - __clz((int)(dist | 1u));
    return e < 4 ? (int)dist : (e - 3) * 16 + (int)((dist >> (e - 4)) & 15u);
}
__device__ __forceinline__ uint32_t wave_bin_first(int bin) { return bin < 16 ? (uint32_t)bin : (uint32_t)(16 + (bin & 15)) << ((bin >> 4) - 1); }

// Inclusive prefix sum over the 64 lanes with data-parallel-primitive moves (row shifts, then the rows' totals).
__device__ __forceinline__ int wave_prefix_i32(int v) {
    auto moved = [](int x, auto ctrl, auto row_mask, auto bound) { return __builtin_amdgcn_update_dpp(0, x, decltype(ctrl)::value, decltype(row_mask)::value, 0xf, decltype(bound)::value); };
    using std::integral_constant;
    v += moved(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{}, integral_constant<bool, true>{});
    v += moved(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{}, integral_constant<bool, true>{});
    v += moved(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{}, integral_constant<bool, true>{});
    v += moved(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{}, integral_constant<bool, true>{});
    v += moved(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}, integral_constant<bool, false>{});
    v += moved(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{}, integral_constant<bool, false>{});
    return v;
}

// List entries of a query: EPL * 64, at least 160 more than m (64 arrive at a time, and thinning out should not follow at once).
constexpr int kSelectWaveMaxM = 864;
inline int select_wave_epl(int m) { return m <= 352 ? 8 : 16; }
inline size_t select_wave_lds(int epl, int w) { return 4 * ((size_t)epl * 64 * 8 + kWaveBins * 4 + (size_t)((w + 3) & ~3) * 20); }

// grid = 8 * ceil(ceil(nq / 4) / 8) rounded up to whole runs (see select_query.hpp for the order of the queries), block = 256: four
// independent wavefronts, dynamic LDS = select_wave_lds bytes.  RB = r_pad / 16; EXT: column-wise step sizes (and, if pt_first is
// given, the mixed-precision decomposition).  m <= 64 * EPL - 160.
template <int RB, bool L2, bool EXT, int EPL>
__global__ __launch_bounds__(256) void k_select_wave(QuerySelectArgs a) {
    constexpr int ZW = RB * 4, CAP = 64 * EPL, LIMIT = CAP - 64;
    extern __shared__ __align__(16) unsigned char sw_smem[];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int w = a.w, m = a.m;
    const int w4 = (w + 3) & ~3;
    unsigned char* mine = sw_smem + (size_t)wv * ((size_t)CAP * 8 + kWaveBins * 4 + (size_t)w4 * 20);
    uint32_t* keys = reinterpret_cast<uint32_t*>(mine);                  // [CAP] keys; entries that have just arrived: what `convert` makes keys of
    int32_t* rows = reinterpret_cast<int32_t*>(keys + CAP);              // [CAP]
    int* bins = reinterpret_cast<int*>(rows + CAP);                      // [kWaveBins]
    int* ppos = bins + kWaveBins;                                        // [w] position of the pair, first row, points, scale, first component of r
    int* prow = ppos + w4;
    int* pcnt = prow + w4;
    float* psig = reinterpret_cast<float*>(pcnt + w4);
    float* prho = psig + w4;
    // runs of consecutive queries go to one XCD, successive runs to successive XCDs (four queries per block)
    const int slot = (int)(blockIdx.x >> 3);
    const int rs = a.run_shift - 2;
    const int si = __builtin_amdgcn_readfirstlane((((((slot >> rs) << 3) + (int)(blockIdx.x & 7)) << rs) + (slot & ((1 << rs) - 1))) * 4 + wv);
    if (si >= a.nq) return;                                              // wavefronts are independent: no block barrier below
    const int q = __builtin_amdgcn_readfirstlane(a.qorder[si]);
    const bool mixed = EXT && a.pt_first != nullptr;
    auto lds_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint32_t pk[4] = {0u, 0u, 0u, 0u};          // keys of the best scores of the pairs not visited yet: pair 64 i + lane (w <= 256)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = 64 * i + lane;
        if (64 * i < w && j < w) {
            const int pos = a.pos_of_slot[(size_t)q * w + j], c = a.sel[(size_t)q * w + j];
            const int64_t r0 = a.off[c], r1 = a.off[c + 1];
            const float s = a.sigma[pos];
            const float rf = mixed ? a.rho0[pos] : 0.0f;
            pk[i] = a.pmax[pos];
            ppos[j] = pos; prow[j] = (int)r0; pcnt[j] = (int)(r1 - r0);
            psig[j] = L2 ? 2.0f * s : s;
            prho[j] = L2 ? 2.0f * rf : rf;
        }
    }
#pragma unroll
    for (int i = 0; i < kWaveBins / 64; ++i) bins[64 * i + lane] = 0;
    lds_sync();
    // the pair of the best score that is left (ties: lower rank first), which is then taken out; key 0: none
    auto next_pair = [&](uint32_t& best) {
        best = ~wave_min_u32(~max(max(pk[0], pk[1]), max(pk[2], pk[3])));
        int j = 0;
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            const unsigned long long holders = __ballot(pk[i] == best);
            if (holders) j = 64 * i + __ffsll(holders) - 1;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) if (64 * i + lane == j) pk[i] = 0u;
        return j;
    };
    uint32_t kmax;                              // key of the best score of all
    int jp = next_pair(kmax);
    uint32_t best = kmax;
    uint32_t T = 0u;          // running threshold key, at most the m-th best score seen so far (0: none yet)
    float Tf = -INFINITY;     // the same as a score
    int n = 0, n_keys = 0;    // entries in the list, those of them that are keys (uniform)
    uint32_t T_tie = 0u, R_tie = 0u;      // m of the entries seen beat every later one of key T_tie in a row beyond R_tie
    bool strict = false;      // so no later point of this cluster can win a tie with T: scores have to exceed it
    const unsigned long long below = (1ull << lane) - 1ull;

    auto read_bins = [&]() {                    // T := far edge of the bin that holds the m-th best score seen (n >= m)
        lds_sync();
        int h[8], sum = 0;
        const i32x4* b4 = reinterpret_cast<const i32x4*>(bins) + 2 * lane;
        const i32x4 x0 = b4[0], x1 = b4[1];
#pragma unroll
        for (int j = 0; j < 4; ++j) { h[j] = x0[j]; h[4 + j] = x1[j]; }
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += h[j];
        const int incl = wave_prefix_i32(sum);
        const unsigned long long reached = __ballot(incl >= m);
        if (reached == 0ull) return 0;          // fewer than m scores (a large cluster's quarters may be empty)
        const int src = __ffsll(reached) - 1;
        int cum = incl - sum, j = 0;
#pragma unroll
        for (int u = 0; u < 7; ++u) { const bool next = j == u && cum + h[u] < m; cum += next ? h[u] : 0; j += next ? 1 : 0; }
        const int bin = 8 * src + __builtin_amdgcn_readlane(j, src);
        const uint32_t last = wave_bin_first(bin + 1) - 1u;
        const uint32_t t = kmax > last ? kmax - last : 0u;
        if (t > T) T = t;
        return bin;
    };
    auto set_threshold = [&]() { Tf = T > 0x007fffffu ? key_to_float(strict ? T + 1u : T) : -INFINITY; };
    auto thin_out = [&]() {                     // keep the entries >= T, of those equal to T the ones that can still count (stable, in place)
        lds_sync();
        const uint32_t R = T == T_tie ? R_tie : 0x7fffffffu;
        int kept = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            const uint32_t k = i < n ? keys[i] : 0u;
            const int32_t r = i < n ? rows[i] : 0;
            const bool in = i < n && (k > T || (k == T && (uint32_t)r <= R));
            const unsigned long long mk = __ballot(in);
            if (in) { const int at = kept + __popcll(mk & below); keys[at] = k; rows[at] = r; }
            kept += __popcll(mk);
            lds_sync();
        }
        n = kept;
    };
    // Largest key K in [lo, hi) with at least m entries >= K, given that lo has; stops early at a K that exactly m entries reach
    // (exact := true).  ek: the list's keys, EPL per lane, 0 beyond its end.
    auto mth_largest = [&](const uint32_t (&ek)[EPL], uint32_t lo, uint32_t hi, bool& exact) {
        auto reach = [&](uint32_t v) { int c = 0;
#pragma unroll
            for (int e = 0; e < EPL; ++e) c += __popcll(__ballot(ek[e] >= v));
            return c; };
        int at_lo = reach(lo);
        while (at_lo != m && hi - lo > 1u) {     // uniform
            const uint32_t mid = lo + ((hi - lo) >> 1);
            const int c = reach(mid);
            if (c >= m) { lo = mid; at_lo = c; } else hi = mid;
        }
        exact = at_lo == m;
        return lo;
    };
    auto load_keys = [&](uint32_t (&ek)[EPL]) {
        lds_sync();
#pragma unroll
        for (int e = 0; e < EPL; ++e) ek[e] = 64 * e + lane < n ? keys[64 * e + lane] : 0u;
    };
    // Smallest row in [lo, hi] up to which at least `need` entries count; entries(mid): how many do up to row `mid`.
    auto row_of_ties = [&](int need, uint32_t lo, uint32_t hi, auto entries) {
        while (lo < hi) {                        // uniform
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (entries(mid) >= need) hi = mid; else lo = mid + 1u;
        }
        return lo;
    };

    constexpr bool INT = !L2 && !EXT;           // one scale per pair, no bias: integer scores are compared, and converted once accepted
    int n_read = 0, bin = 0;                    // entries when the bins were last read
    for (; best != 0u && best >= T; jp = next_pair(best)) {       // in falling order: no later cluster can reach T either
        const int m_c = __builtin_amdgcn_readfirstlane(pcnt[jp]), r0 = __builtin_amdgcn_readfirstlane(prow[jp]);
        const float sp = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(psig[jp]))), r0p = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(prho[jp])));
        const i32x4* zp = reinterpret_cast<const i32x4*>(a.Z) + (size_t)__builtin_amdgcn_readfirstlane(ppos[jp]) * RB;
        // the cluster's codes, norms, ... as buffers: lanes beyond its end read zeros (walk_offsets.hpp), and no lane computes an address
        const auto codes = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(a.Bp) + (size_t)r0 * (RB * 16), 0, m_c * (RB * 16), 0x00027000);
        const auto norms = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(L2 ? a.sqnorm + r0 : reinterpret_cast<const float*>(a.Bp)), 0, L2 ? m_c * 4 : 0, 0x00027000);
        const auto steps = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(EXT ? a.pt_scale + r0 : reinterpret_cast<const float*>(a.Bp)), 0, EXT ? m_c * 4 : 0, 0x00027000);
        const auto firsts = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(mixed ? a.pt_first + r0 : reinterpret_cast<const float*>(a.Bp)), 0, mixed ? m_c * 4 : 0, 0x00027000);
        i32x4 zv[RB];                                    // (in flight with the first codes)
#pragma unroll
        for (int u = 0; u < RB; ++u) zv[u] = zp[u];
        struct Piece { i32x4 code[RB]; float bias, scale, first; };
        auto request = [&](Piece& pc, int own, int base) {       // point base + own: base uniform, own of the lane
            constexpr int CB = RB * 16;
            const PieceOffset at = piece_offset(own, base, CB), at4 = piece_offset(own, base, 4);
#pragma unroll
            for (int u = 0; u < RB; ++u) pc.code[u] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(codes, at.vector + 16 * u, at.scalar, 0));
            if (L2) pc.bias = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(norms, at4.vector, at4.scalar, 0));
            if (EXT) {
                pc.scale = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(steps, at4.vector, at4.scalar, 0));
                pc.first = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(firsts, at4.vector, at4.scalar, 0));
            }
        };
        // entries that arrived as scores (or integer scores) of this cluster become keys and are counted in the bins
        auto convert = [&]() {
            lds_sync();
            for (int i0 = n_keys; i0 < n; i0 += 64) {
                const int i = i0 + lane;
                if (i < n) {
                    const float sc = INT ? __fmaf_rn((float)(int)keys[i], sp, -0.0f) : __uint_as_float(keys[i]);
                    const uint32_t key = min(float_key_asc(sc), 0xfffffffeu);      // (a NaN of all ones: mth_largest needs a key above all)
                    keys[i] = key;
                    atomicAdd(&bins[wave_bin(key < kmax ? kmax - key : 0u)], 1);
                }
            }
            n_keys = n;
        };
        int yT = (int)0x80000000;                        // INT: no integer score below it can reach T
        auto int_threshold = [&]() {
            if (!INT || Tf == -INFINITY) return;
            if (!(sp > 0.0f)) { yT = 0.0f >= Tf ? (int)0x80000000 : 0x7fffffff; return; }
            const float t = Tf / sp;
            yT = (int)fminf(fmaxf(floorf(t - 1e-6f * fabsf(t)) - 1.0f, -1.0e9f), 1.0e9f);
            if (strict) for (int i = 0; i < 3 && __fmaf_rn((float)yT, sp, -0.0f) < Tf; ++i) ++yT;      // the tied score itself
        };
        if (strict) { strict = false; set_threshold(); }
        int_threshold();
        auto make_room = [&](int row0) {                 // the list is nearly full; no later point of the cluster has a row below row0
            convert();
            bin = read_bins();
            thin_out();
            if (n > LIMIT) {                             // one bin holds too many: the m best exactly (m <= LIMIT - 96)
                uint32_t ek[EPL];
                load_keys(ek);
                bool exact;
                T = mth_largest(ek, max(T, 1u), max(bin == 0 ? 0xffffffffu : kmax - wave_bin_first(bin) + 1u, T + 1u), exact);      // (as in the final selection)
                thin_out();
            }
            if (n > LIMIT) {                             // too many tie with the m-th: those in the lowest rows (over the list in LDS: rare)
                auto entries = [&](auto f) {
                    int c = 0;
                    for (int i0 = 0; i0 < n; i0 += 64) c += __popcll(__ballot(i0 + lane < n && f(i0 + lane)));
                    return c;
                };
                uint32_t first = 0x7fffffffu, last = 0u;
                for (int i = lane; i < n; i += 64) if (keys[i] == T) { first = min(first, (uint32_t)rows[i]); last = max(last, (uint32_t)rows[i]); }
                const int above = entries([&](int i) { return keys[i] > T; });
                R_tie = row_of_ties(m - above, wave_min_u32(first), ~wave_min_u32(~last), [&](uint32_t mid) { return entries([&](int i) { return keys[i] == T && (uint32_t)rows[i] <= mid; }); });
                T_tie = T;
                thin_out();
            }
            strict = T == T_tie && R_tie < (uint32_t)row0;
            n_keys = n;
            set_threshold();
            int_threshold();
            n_read = n;
        };
        const bool large = a.sub && m_c > kSubMinPoints;  // uniform: looked into by quarters if it has them
        // one piece of up to 64 points: this lane's is point base + own
        int z[ZW];                                       // uniform: scalar registers
        auto score = [&](const Piece& pc, int own, int base) {
            if (n > LIMIT) make_room(r0 + (large ? base & ~(kChunkPoints - 1) : base));      // (quarters: rows ascend from chunk to chunk)
            int y = 0;
#pragma unroll
            for (int u = 0; u < RB; ++u)
#pragma unroll
                for (int x = 0; x < 4; ++x) y = dot4_i8(pc.code[u][x], z[4 * u + x], y);
            bool in;
            uint32_t raw;
            if (INT) { in = y >= yT; raw = (uint32_t)y; }
            else {
                float sc = __fmaf_rn((float)y, EXT ? __fmul_rn(sp, pc.scale) : sp, L2 ? -pc.bias : -0.0f);
                if (EXT && mixed) sc = __fmaf_rn(r0p, pc.first, sc);
                in = !(sc < Tf);
                raw = __float_as_uint(sc);
            }
            in = in && base + own < m_c;
            const unsigned long long mk = __ballot(in);
            if (mk) {
                if (in) {
                    const int at = n + __popcll(mk & below);
                    keys[at] = raw;
                    rows[at] = r0 + base + own;
                }
                n += __popcll(mk);
            }
        };
        int nq4 = 0;                                     // quarters of a large cluster
        const uint32_t* subp = nullptr;
        size_t sub_step = 0;
        if (large) {
            const int c = __builtin_amdgcn_readfirstlane(a.sel[(size_t)q * w + jp]), pos = __builtin_amdgcn_readfirstlane(ppos[jp]);
            const int at = pos - a.bucket_off[c], first = a.sub_first[c], chunks = (m_c + kChunkPoints - 1) / kChunkPoints;
            if (first + chunks <= a.sub_chunks) {
                nq4 = 4 * chunks;
                subp = a.sub + ((size_t)first * a.sub_groups + (at >> 6)) * 256 + (at & 63) * 4;
                sub_step = (size_t)a.sub_groups * 256;
            }
        }
        if (nq4 == 0) {
            Piece ring[4];
#pragma unroll
            for (int b = 0; b < kWalkAhead; ++b) request(ring[b], lane, 64 * b);
#pragma unroll
            for (int u = 0; u < ZW; ++u) z[u] = __builtin_amdgcn_readfirstlane(zv[u >> 2][u & 3]);
            // (no branch around the requests: the compiler would copy the pieces at the join and wait for them; pieces beyond the end
            // read zeros and add nothing)
            for (int p0 = 0; p0 < m_c; p0 += 256) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    request(ring[(b + kWalkAhead) & 3], lane, p0 + 64 * (b + kWalkAhead));
                    score(ring[b], lane, p0 + 64 * b);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < ZW; ++u) z[u] = __builtin_amdgcn_readfirstlane(zv[u >> 2][u & 3]);
            auto sub_key = [&](int i) { return i < nq4 ? subp[(size_t)(i >> 2) * sub_step + (i & 3)] : 0u; };
            if (n + nq4 >= m) {     // the quarters' best scores are scores of distinct points: counted among the seen ones they may raise T
                for (int i0 = 0; i0 < nq4; i0 += 64) { const uint32_t k = sub_key(i0 + lane); if (k) atomicAdd(&bins[wave_bin(k < kmax ? kmax - k : 0u)], 1); }
                (void)read_bins();      // (the bin itself is read again before the final selection: n_read)
                n_read = -1;
                for (int i0 = 0; i0 < nq4; i0 += 64) { const uint32_t k = sub_key(i0 + lane); if (k) atomicAdd(&bins[wave_bin(k < kmax ? kmax - k : 0u)], -1); }
                set_threshold();
                int_threshold();
            }
            // a quarter is two pieces of eight runs of eight points; two quarters are on their way at any time
            for (int i0 = 0; i0 < nq4; i0 += 64) {
                const uint32_t k = sub_key(i0 + lane);
                unsigned long long todo = __ballot(k != 0u && k >= T);
                const int own = quarter_point(lane);
                auto next = [&]() {                      // first point of the next quarter; none left: beyond the cluster's end (uniform)
                    if (todo == 0ull) return m_c;
                    const int i = i0 + __ffsll(todo) - 1;
                    todo &= todo - 1ull;
                    return (i >> 2) * 512 + (i & 3) * 8;
                };
                Piece ring[4];
                int t0 = next(), t1 = next();
                request(ring[0], own, t0);
                request(ring[1], own, t0 + kQuarterHalf);
                request(ring[2], own, t1);
                request(ring[3], own, t1 + kQuarterHalf);
                while (t0 < m_c) {                       // uniform
                    score(ring[0], own, t0);
                    score(ring[1], own, t0 + kQuarterHalf);
                    t0 = next();
                    request(ring[0], own, t0);
                    request(ring[1], own, t0 + kQuarterHalf);
                    score(ring[2], own, t1);
                    score(ring[3], own, t1 + kQuarterHalf);
                    t1 = next();
                    request(ring[2], own, t1);
                    request(ring[3], own, t1 + kQuarterHalf);
                }
            }
        }
        convert();
        if (n >= m && n != n_read) { bin = read_bins(); set_threshold(); n_read = n; }
    }

    int32_t* out = a.cand + (size_t)q * m;
    uint32_t ek[EPL];
    load_keys(ek);
    uint32_t K = 0u, lowest = 0xffffffffu;
    bool exact = true;
    if (n > m) {
        // the m-th best lies between T and the near edge of its bin (scores that are no numbers sit beyond the best one)
        const uint32_t dist0 = wave_bin_first(bin), hi = bin == 0 ? 0xffffffffu : kmax - dist0 + 1u;
        K = mth_largest(ek, max(T, 1u), max(hi, T + 1u), exact);
    }
    // entries above K, and of those equal to it the ones in the lowest rows
    uint32_t R = 0xffffffffu;
    int32_t er[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) er[e] = 64 * e + lane < n ? rows[64 * e + lane] : 0x7fffffff;
    if (!exact) {
        int above = 0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) above += __popcll(__ballot(ek[e] > K));
        // 1 <= m - above < the entries equal to K.  (Rows in registers: one query in a hundred gets here, bisecting over LDS took it 13 us,
        // and the kernel lasts as long as its slowest query: 10 000 queries of the 768-d workload 68 us against 53.)
        R = row_of_ties(m - above, 0u, 0x7fffffffu, [&](uint32_t mid) {
            int c = 0;
#pragma unroll
            for (int e = 0; e < EPL; ++e) c += __popcll(__ballot(ek[e] == K && (uint32_t)er[e] <= mid));
            return c;
        });
    }
    int at0 = 0, mn = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const bool in = 64 * e + lane < n && (ek[e] > K || (ek[e] == K && (uint32_t)er[e] <= R));
        const unsigned long long mk = __ballot(in);
        if (in) { out[at0 + __popcll(mk & below)] = er[e]; mn = min(mn, er[e]); lowest = min(lowest, ek[e]); }
        at0 += __popcll(mk);
    }
    for (int i = at0 + lane; i < m; i += 64) out[i] = -1;
    const uint32_t mnw = wave_min_u32((uint32_t)mn), low = wave_min_u32(lowest);
    if (lane == 0) { a.qkey[q] = (int32_t)mnw; a.n_kept[q] = n; a.tau[q] = n >= m ? key_to_float(low) : -INFINITY; }
}

}  // namespace lorann
