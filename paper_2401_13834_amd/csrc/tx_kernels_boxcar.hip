// Boxcar matched filter for gfx950 (MI355X): per-DM noise statistics, peak
// S/N over the boxcar widths, and the thresholded DM-time candidates
// (Sec. 2.4, Eq. 5; Sec. 2.5).
//
// One workgroup per DM row, several for few long rows (boxcar_scan_kernel); the
// batch form takes the rows of many jobs.  The row is read from HBM once, in
// tiles of 4096 window starts:
//  * each tile's running sums (exclusive prefix, uint32: window sums are exact
//    as differences) of its 4096 + longest-width samples go to LDS; the same
//    loads accumulate the exact moments sum y and sum y^2 (uint64);
//  * per width, every lane keeps the largest window sum of its 16 starts; the
//    tile's largest is compared with the row's best so far, and only when it
//    beats it (a few tiles per row) is the earliest start reaching it looked
//    up; the largest sum per (tile, width) is kept in LDS.
// Then c = floor(sum/T), Q = sum y^2 - 2 c sum + T c^2 (= sum (y - c)^2, mod
// 2^64), var = Q/T - (r/T)^2, sigma and 1/(sigma T) in float64 give the peak
// S/N, and per width the least window sum S* whose S/N reaches gamma (the exact
// solution checked against its neighbours with the same float64 expression, else
// by bisection).  Only tiles where some width's
// largest sum reaches its S* are read again to list candidates: a start is a
// candidate when some width passes, and is reported with the width of highest
// S/N.  Thread tid owns the starts t0 + tid + 256 j (j < 16).
#include <algorithm>

#include "tx_internal.h"

#pragma clang fp contract(off)

namespace tx {

// Largest dynamic LDS for the per-(tile, width) maxima; rows needing more
// read every tile again for candidates.
constexpr int kTileMaxLds = 16 * 1024;

constexpr int kSplitGroups = 6 * 256;   // workgroups that a split aims at

// Largest calls of the list form (boxcar_list_kernel): rows that the chip holds
// at once (5 workgroups per CU), and tiles per row.
constexpr int kListRows = 5 * 256;
constexpr int kListTiles = 16;

template <int NWT>
struct BoxShared {
    __align__(16) uint32_t P[kBoxTile + TX_MAX_WIDTH + 16];
    unsigned long long red1[kWaves], red2[kWaves];
    int redbad[kWaves];
    uint32_t wtot[kWaves];
    int32_t sthr[TX_MAX_WIDTHS];
    int32_t wd[TX_MAX_WIDTHS];     // widths and 1/sqrt(width) of the row's job, for
    double rs[TX_MAX_WIDTHS];      // run-time indexing (no private copy of the arguments)
    double inv_d;
    long long sum;
    int state;
    __align__(16) int32_t wS[NWT][kWaves];   // the tile's largest sum per width and wavefront, and where
    __align__(16) int32_t wT[NWT][kWaves];   // it is the row's new best, its earliest start
    int32_t bS[NWT], bT[NWT];                // per width: the row's largest sum so far and its earliest start
};

extern __shared__ int32_t tx_box_tmax[];   // [tiles][NWT]: workgroup's largest sum per tile (from its first) and width

__device__ __forceinline__ double snr_of(int64_t T, int64_t S, int64_t w, int64_t sum, double inv_d, double rsw) {
    const int64_t N = T * S - w * sum;
    return (static_cast<double>(N) * inv_d) * rsw;
}

template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Wavefront max / min of an int32 with DPP (quad, half-row and row permutes,
// then the row broadcasts of 15 and 31); the result is read from lane 63.
// The moves' fallback value is the operation's identity, so each step
// compiles to one v_max/v_min with a DPP source instead of a move and an op
// (rows a broadcast does not write keep their value either way).
__device__ __forceinline__ int32_t wave_max_i32(int32_t v) {
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x141, 0xF, 0xF, false));  // row_half_mirror
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x140, 0xF, 0xF, false));  // row_mirror
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x142, 0xA, 0xF, false));  // row_bcast15
    v = max(v, __builtin_amdgcn_update_dpp(INT32_MIN, v, 0x143, 0xC, 0xF, false));  // row_bcast31
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ int32_t wave_min_i32(int32_t v) {
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0xB1, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x4E, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x141, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x140, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x142, 0xA, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(INT32_MAX, v, 0x143, 0xC, 0xF, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// Inclusive prefix sum over the wavefront's lanes with DPP: shifts of 1, 2,
// 4 and 8 lanes within each row of 16 (lanes without a source add the
// identity 0), then the row broadcasts of lanes 15 and 31 into the rows
// above them.  Each step is one v_add with a DPP source; no LDS traffic.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x) {
    x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xF, 0xF, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xF, 0xF, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xF, 0xF, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xF, 0xF, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2, 3
    return x;
}

// Moments of the samples a thread loaded (exact; a value >= 2^21 or < 0 flags
// the row).
struct Moments {
    unsigned long long s1 = 0, s2 = 0;
    uint32_t bad = 0;
};

// Exclusive running sums of y[t0 + e] for e < L = 4096 + longest width
// (<= 5120; zeros past the row) into P[e], and P[L] = their total.  Thread
// tid owns the 20 consecutive samples from e = 20 tid.  COUNT: add the
// samples with e < 4096 (the tile's own) to the moments.
template <bool COUNT>
__device__ __forceinline__ void scan_tile(const TX_GLOBAL int32_t* __restrict__ y, int T, int t0, int L, uint32_t* P,
                                          uint32_t* wtot, bool vec, int tid, Moments& m) {
    constexpr int kPer = 20;
    const int lane = tid & 63, wave = tid >> 6;
    const int e = kPer * tid;
    uint32_t v[kPer];
    const int64_t t = static_cast<int64_t>(t0) + e;
    if (vec && e + kPer <= L && t + kPer <= T) {
#pragma unroll
        for (int k = 0; k < kPer / 4; ++k) {
            const uint4 q = *reinterpret_cast<const TX_GLOBAL uint4*>(y + t + 4 * k);
            v[4 * k] = q.x;
            v[4 * k + 1] = q.y;
            v[4 * k + 2] = q.z;
            v[4 * k + 3] = q.w;
        }
    } else {
        // Valid samples of this lane (the count changes with the tile, so no
        // per-element condition is hoisted out of the tile loop).
        const int64_t lim = min(static_cast<int64_t>(L - e), static_cast<int64_t>(T) - t);
#pragma unroll
        for (int k = 0; k < kPer; ++k) v[k] = k < lim ? static_cast<uint32_t>(y[t + k]) : 0u;
    }
    if (COUNT) {
        // The sums are used only when every sample is in [0, TX_MAX_VALUE)
        // (then ps < 20 * 2^21 and y^2 < 2^42: no wrap), so out-of-range
        // samples need only the flag, taken from the running maximum (as
        // unsigned, a negative sample is out of range too).
        constexpr uint32_t kMask = static_cast<uint32_t>(TX_MAX_VALUE) - 1u;
        const int own = min(kPer, kBoxTile - e);       // samples of this tile (the rest belong to the next)
        uint32_t ps = 0, mx = 0;
        if (own == kPer) {                             // all but the threads at the tile's end
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                mx = max(mx, v[k]);
                ps += v[k];
                m.s2 += static_cast<unsigned long long>(v[k]) * v[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const uint32_t x = k < own ? v[k] : 0u;
                mx = max(mx, x);
                ps += x;
                m.s2 += static_cast<unsigned long long>(x) * x;
            }
        }
        m.bad |= mx > kMask ? 1u : 0u;
        m.s1 += ps;
    }
    uint32_t run = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) run += v[k];
    const uint32_t incl = wave_incl_sum(run);
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wtot[w];
    before += incl - run;
    if (e < L) {
#pragma unroll
        for (int k = 0; k < kPer / 4; ++k) {
            const uint32_t p0 = before, p1 = p0 + v[4 * k], p2 = p1 + v[4 * k + 1], p3 = p2 + v[4 * k + 2];
            before = p3 + v[4 * k + 3];
            *reinterpret_cast<uint4*>(P + e + 4 * k) = make_uint4(p0, p1, p2, p3);
        }
    }
    if (tid == 0) P[L] = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    __syncthreads();
}

// Peak search over one tile.  Lane tid owns the starts t0 + tid + 256 j
// (j < 16), so a wavefront reads 64 consecutive LDS words per load (no bank
// conflicts for any width).  TAIL: some windows reach past the row end.  Width
// slots past the row's widths repeat its last width.
//
// First every wavefront's largest sums of all widths; then, where the tile
// beats the row's best sum of a width (a few tiles per row), the wavefronts
// that hold that sum look up its earliest start.  Comparing with the whole
// row's best, and not each wavefront with its own, leaves a quarter of the
// lookups, and each costs about as much as a width's sums.  The widths are a
// rolled loop, two a turn: a row's code is a third of the unrolled one's.
// 4096 rows of 65536 samples, 10 widths: 514 us with lookups per wavefront and
// unrolled widths, 343 so (1.07 GB: 3.1 TB/s); 203 rows of 5003 samples 34 and 18;
// 96 rows of 1000003 samples, unsplit, 1340 and 950.
template <int NWT, bool TAIL>
__device__ __forceinline__ void peak_tile(const BoxcarArgs& a, BoxShared<NWT>& sh, int tile, int t0, int tid,
                                          bool keep_tmax) {
    const int wave = tid >> 6, lane = tid & 63;
    const int T = a.nt;
    uint32_t Pt[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) Pt[j] = sh.P[tid + 256 * j];
#pragma unroll 1
    for (int i = 0; i < NWT; i += 2) {
        // Per-width values come from LDS, which keeps the registers free.
        const int w0 = sh.wd[i], w1 = sh.wd[i + 1];
        const uint32_t* p0 = sh.P + tid + w0;
        const uint32_t* p1 = sh.P + tid + w1;
        int32_t tm0 = INT32_MIN, tm1 = INT32_MIN;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int32_t S0 = static_cast<int32_t>(p0[256 * j] - Pt[j]);
            const int32_t S1 = static_cast<int32_t>(p1[256 * j] - Pt[j]);
            const int t = t0 + tid + 256 * j;
            tm0 = max(tm0, (!TAIL || t + w0 <= T) ? S0 : INT32_MIN);   // no window past the row end
            tm1 = max(tm1, (!TAIL || t + w1 <= T) ? S1 : INT32_MIN);
        }
        const int32_t m0 = wave_max_i32(tm0), m1 = wave_max_i32(tm1);
        if (lane < 2) sh.wS[i + lane][wave] = lane == 0 ? m0 : m1;
    }
    __syncthreads();
    // Lane i: width i.
    int32_t M = INT32_MIN;
    unsigned long long look = 0;
    if (lane < NWT) {
        const int4 q = *reinterpret_cast<const int4*>(sh.wS[lane]);
        M = max(max(q.x, q.y), max(q.z, q.w));
        if (keep_tmax && wave == 0) tx_box_tmax[tile * NWT + lane] = M;
        look = M > sh.bS[lane];
    }
    const unsigned long long rec = __ballot(look);            // widths with a new best: the same in every wavefront
    if (rec == 0) return;
    for (unsigned long long left = __ballot(look && sh.wS[lane < NWT ? lane : 0][wave] == M); left; left &= left - 1) {
        const int i = __builtin_ctzll(left);
        const int32_t m = __builtin_amdgcn_readlane(M, i);
        const int w = sh.wd[i];
        const uint32_t* p = sh.P + tid + w;
        int32_t first = INT32_MAX;
#pragma unroll
        for (int j = 15; j >= 0; --j) {
            const int t = t0 + tid + 256 * j;
            const int32_t S = static_cast<int32_t>(p[256 * j] - Pt[j]);
            first = ((!TAIL || t + w <= T) && S == m) ? t : first;
        }
        const int32_t ft = wave_min_i32(first);
        if (lane == 0) sh.wT[i][wave] = ft;
    }
    __syncthreads();
    if (wave == 0 && look) {
        int32_t t = INT32_MAX;
#pragma unroll
        for (int v = 0; v < kWaves; ++v)
            if (sh.wS[lane][v] == M) t = min(t, sh.wT[lane][v]);
        sh.bS[lane] = M;
        sh.bT[lane] = t;
    }
}

// Peak search over one tile in the list form (boxcar_list_kernel): every
// wavefront looks up the starts of its own bests, which sh.wS and sh.wT hold
// from tile to tile.
template <int NWT, bool TAIL>
__device__ __forceinline__ void peak_tile_list(const BoxcarArgs& a, BoxShared<NWT>& sh, int tile, int t0, int tid,
                                               bool keep_tmax) {
    const int wave = tid >> 6;
    const int T = a.nt;
    uint32_t Pt[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) Pt[j] = sh.P[tid + 256 * j];
    int32_t tm[NWT];
#pragma unroll
    for (int i = 0; i < NWT; i += 2) {
        // Per-width values come from LDS, which keeps the registers free.
        const int w0 = sh.wd[i], w1 = sh.wd[i + 1];
        const uint32_t* p0 = sh.P + tid + w0;
        const uint32_t* p1 = sh.P + tid + w1;
        int32_t tm0 = INT32_MIN, tm1 = INT32_MIN;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int32_t S0 = static_cast<int32_t>(p0[256 * j] - Pt[j]);
            const int32_t S1 = static_cast<int32_t>(p1[256 * j] - Pt[j]);
            const int t = t0 + tid + 256 * j;
            tm0 = max(tm0, (!TAIL || t + w0 <= T) ? S0 : INT32_MIN);   // no window past the row end
            tm1 = max(tm1, (!TAIL || t + w1 <= T) ? S1 : INT32_MIN);
        }
        tm[i] = tm0;
        tm[i + 1] = tm1;
        // Keep each width pair's LDS reads next to their arithmetic.
        __builtin_amdgcn_sched_barrier(0);
    }
    // Wavefront maxima of all widths (independent reductions, interleaved).
    int32_t wm[NWT];
#pragma unroll
    for (int i = 0; i < NWT; ++i) wm[i] = wave_max_i32(tm[i]);
#pragma unroll 1
    for (int ii = 0; ii < NWT; ++ii) {
        // wm[ii] with a run-time ii: select among the (uniform) values.
        int32_t m = wm[0];
#pragma unroll
        for (int k = 1; k < NWT; ++k) m = (k == ii) ? wm[k] : m;
        if (keep_tmax && (tid & 63) == 0) atomicMax(&tx_box_tmax[tile * NWT + ii], m);
        if (m > sh.wS[ii][wave]) {                      // wavefront-uniform, a few tiles per row
            const int w = sh.wd[ii];
            int32_t first = INT32_MAX;
#pragma unroll 1
            for (int j = 15; j >= 0; --j) {             // rolled: this path is rare
                const int e = tid + 256 * j;
                const int t = t0 + e;
                const int32_t S = static_cast<int32_t>(sh.P[e + w] - sh.P[e]);
                first = ((!TAIL || t + w <= T) && S == m) ? t : first;
            }
            const int32_t ft = wave_min_i32(first);
            if ((tid & 63) == 0) {
                sh.wS[ii][wave] = m;
                sh.wT[ii][wave] = ft;
            }
        }
    }
}

// Candidates of one tile in the list form: every 64 starts take their places
// with one atomic.  Widths increase, so a strict ">" keeps the smaller width on
// equal S/N.
template <int NWT>
__device__ __forceinline__ void cand_tile_list(const BoxcarArgs& a, BoxShared<NWT>& sh, int row, int t0, long long sum,
                                               double inv_d, int tid) {
    const int T = a.nt;
#pragma unroll 1
    for (int j = 0; j < 16; ++j) {
        const int e = tid + 256 * j;
        const int t = t0 + e;
        const uint32_t pt = sh.P[e];
        bool pass = false;
        double bs = 0.0;
        int bw = -1;
        for (int i = 0; i < a.ne; ++i) {
            const int w = sh.wd[i];
            if (t + w > T) continue;
            const int32_t S = static_cast<int32_t>(sh.P[e + w] - pt);
            pass = pass || S >= max(sh.sthr[i], 0);       // window sums are >= 0
            const double sn = snr_of(T, S, w, sum, inv_d, sh.rs[i]);
            if (bw < 0 || sn > bs) {
                bs = sn;
                bw = w;
            }
        }
        if (!pass) continue;
        const unsigned long long slot = atomicAdd(a.count, 1ull);
        if (static_cast<long long>(slot) < a.cap) {
            tx_cand c;
            c.dm_index = row;
            c.width = bw;
            c.time = t;
            c.snr = bs;
            to_global(a.cands)[slot] = c;
        }
    }
}

// Candidates of one tile (rare: only tiles where some width's largest sum
// reaches its threshold S*).  The starts that pass are found first, as 16 bits
// per lane, with the sums alone; the wavefront then takes its places in the
// list with one atomic, and only the starts that pass have their S/N worked
// out.  (One atomic per 64 starts and the S/N of every start and width had
// made a tile with candidates cost as much as ten without.)  Widths increase,
// so a strict ">" keeps the smaller width on equal S/N.
template <int NWT>
__device__ __forceinline__ void cand_tile(const BoxcarArgs& a, BoxShared<NWT>& sh, int row, int tile, bool keep_tmax,
                                          long long sum, double inv_d, int tlo, int tid) {
    const int T = a.nt;
    const int t0 = tile * kBoxTile;
    uint32_t pass = 0;
#pragma unroll 1
    for (int i = 0; i < a.ne; ++i) {
        const int32_t thr = max(sh.sthr[i], 0);           // window sums are >= 0
        if (keep_tmax && tx_box_tmax[(tile - tlo) * NWT + i] < thr) continue;      // workgroup-uniform
        const int w = sh.wd[i];
        const int lim = T - w - t0 - tid;                 // starts with 256 j <= lim have their window in the row
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int32_t S = static_cast<int32_t>(sh.P[tid + 256 * j + w] - sh.P[tid + 256 * j]);
            pass |= S >= thr && 256 * j <= lim ? 1u << j : 0u;
        }
    }
    // Places in the order of the starts 256 j + lane.
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) total += static_cast<uint32_t>(__popcll(__ballot(pass >> j & 1u)));
    if (total == 0) return;
    unsigned long long base = 0;
    if ((tid & 63) == 0) base = atomicAdd(a.count, static_cast<unsigned long long>(total));
    base = __shfl(base, 0);
#pragma unroll 1
    for (int j = 0; j < 16; ++j) {
        const unsigned long long in = __ballot(pass >> j & 1u);
        const unsigned long long slot =
            base + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(in >> 32),
                                             __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(in), 0u));
        base += static_cast<unsigned long long>(__popcll(in));
        if (!(pass >> j & 1u) || static_cast<long long>(slot) >= a.cap) continue;
        const int e = tid + 256 * j;
        const uint32_t pt = sh.P[e];
        double bs = 0.0;
        int bw = -1;
#pragma unroll 1
        for (int i = 0; i < a.ne; ++i) {
            const int w = sh.wd[i];
            if (t0 + e + w > T) break;
            const int32_t S = static_cast<int32_t>(sh.P[e + w] - pt);
            const double sn = snr_of(T, S, w, sum, inv_d, sh.rs[i]);
            if (bw < 0 || sn > bs) {
                bs = sn;
                bw = w;
            }
        }
        tx_cand c;
        c.dm_index = row;
        c.width = bw;
        c.time = t0 + e;
        c.snr = bs;
        to_global(a.cands)[slot] = c;
    }
}

// Widths and 1/sqrt(w) of the row's job into LDS, the per-width best cleared
// (in the list form every wavefront's, and the maxima of the row's tiles).
template <int NWT, bool LIST = false>
__device__ __forceinline__ void row_setup(const BoxcarArgs& a, BoxShared<NWT>& sh, int tid, int ntiles = 0,
                                          bool keep_tmax = false) {
    if (tid < NWT) {
        int32_t w = 0;
        double r = 0.0;
#pragma unroll
        for (int k = 0; k < NWT; ++k)          // compile-time indices only
            if (k == tid) {
                w = a.widths[k];
                r = a.rsw[k];
            }
        sh.wd[tid] = w;
        sh.rs[tid] = r;
        sh.bS[tid] = INT32_MIN;
        sh.bT[tid] = 0;
    }
    if (LIST) {
        if ((tid & 63) == 0) {
#pragma unroll
            for (int i = 0; i < NWT; ++i) {
                sh.wS[i][tid >> 6] = INT32_MIN;
                sh.wT[i][tid >> 6] = 0;
            }
        }
        if (keep_tmax)
            for (int k = tid; k < ntiles * NWT; k += kThreads) tx_box_tmax[k] = INT32_MIN;
    }
    __syncthreads();
}

// Tiles [tlo, thi) of a row: running sums, exact moments (wavefront sums left
// in sh.red*), per-width best (sh.bS / sh.bT) and the per-(tile, width) maxima.
template <int NWT, bool LIST = false>
__device__ __forceinline__ void row_scan(const BoxcarArgs& a, int tlo, int thi, bool keep_tmax,
                                         const TX_GLOBAL int32_t* __restrict__ y, bool vec, BoxShared<NWT>& sh,
                                         int tid) {
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int T = a.nt;
    const int L = kBoxTile + a.wmax;
    Moments m;
    for (int tile = tlo; tile < thi; ++tile) {
        const int t0 = tile * kBoxTile;
        // The thread index, made opaque to the compiler in every tile: else it
        // hoists dozens of lane-dependent masks and addresses out of this loop
        // and spills them.
        int tv = tid;
        asm volatile("" : "+v"(tv));
        scan_tile<true>(y, T, t0, L, sh.P, sh.wtot, vec, tv, m);
        if (LIST) {
            if (t0 + kBoxTile + a.wmax > T) peak_tile_list<NWT, true>(a, sh, tile, t0, tv, keep_tmax);
            else peak_tile_list<NWT, false>(a, sh, tile, t0, tv, keep_tmax);
        } else if (a.ne > 0) {
            if (t0 + kBoxTile + a.wmax > T) peak_tile<NWT, true>(a, sh, tile - tlo, t0, tv, keep_tmax);
            else peak_tile<NWT, false>(a, sh, tile - tlo, t0, tv, keep_tmax);
        }
        __syncthreads();
    }
    const unsigned long long s1 = wave_sum(m.s1);
    const unsigned long long s2 = wave_sum(m.s2);
    const int bad = __any(m.bad != 0) ? 1 : 0;
    if (lane == 0) {
        sh.red1[wave] = s1;
        sh.red2[wave] = s2;
        sh.redbad[wave] = bad;
    }
    if (LIST && tid < NWT) {                     // (the last tile's barrier orders these reads)
        int32_t S = sh.wS[tid][0], t = sh.wT[tid][0];
#pragma unroll
        for (int v = 1; v < kWaves; ++v)
            if (sh.wS[tid][v] > S || (sh.wS[tid][v] == S && sh.wT[tid][v] < t)) {
                S = sh.wS[tid][v];
                t = sh.wT[tid][v];
            }
        sh.bS[tid] = S;
        sh.bT[tid] = t;
    }
    __syncthreads();
}

// Statistics, the row's peak (when `peak`) and (when asked) the candidates of
// its tiles [tlo, thi), from the state row_scan left in LDS.
template <int NWT, bool LIST = false>
__device__ __forceinline__ void row_finish(const BoxcarArgs& a, int row, bool peak, int tlo, int thi, bool keep_tmax,
                                           const TX_GLOBAL int32_t* __restrict__ y, bool vec, BoxShared<NWT>& sh,
                                           int tid) {
    const int T = a.nt;
    const int L = kBoxTile + a.wmax;
    if (tid == 0) {
        unsigned long long S1 = 0, S2 = 0;
        int B = 0;
        for (int w = 0; w < kWaves; ++w) {
            S1 += sh.red1[w];
            S2 += sh.red2[w];
            B |= sh.redbad[w];
        }
        int state = B ? 2 : 0;
        double inv_d = 0.0;
        const long long sum = static_cast<long long>(S1);
        if (!B) {
            const long long c = sum / T;
            const long long r = sum - static_cast<long long>(T) * c;
            const unsigned long long q = S2 - 2ull * static_cast<unsigned long long>(c) * S1 +
                                         static_cast<unsigned long long>(T) * static_cast<unsigned long long>(c) *
                                             static_cast<unsigned long long>(c);
            const double av = static_cast<double>(q) / static_cast<double>(T);
            const double bv = static_cast<double>(r) / static_cast<double>(T);
            const double var = av - bv * bv;
            if (var > 0.0) {
                const double sigma = __builtin_sqrt(var);
                inv_d = 1.0 / (sigma * static_cast<double>(T));
            } else {
                state = 1;
            }
        }
        sh.inv_d = inv_d;
        sh.sum = sum;
        sh.state = state;
    }
    __syncthreads();
    const int state = sh.state;
    const double inv_d = sh.inv_d;
    const long long sum = sh.sum;
    if (state != 0) {
        if (tid == 0 && peak) {
            to_global(a.snr)[row] = state == 1 ? 0.0 : __builtin_nan("");
            to_global(a.width)[row] = state == 1 ? a.w_first : -1;
            to_global(a.time)[row] = state == 1 ? 0 : -1;
        }
        __syncthreads();
        return;
    }

    // ---- peak: (largest S, earliest t) per width (lane i: width i), then the best width ----
    if (peak && tid < 64) {
        const int i = tid < a.ne ? tid : -1;
        double sn = -__builtin_inf();
        int best = TX_MAX_WIDTHS;
        int32_t t = 0;
        if (i >= 0) {
            t = sh.bT[i];
            sn = snr_of(T, sh.bS[i], sh.wd[i], sum, inv_d, sh.rs[i]);
            best = i;
        }
#pragma unroll
        for (int o = TX_MAX_WIDTHS / 2; o > 0; o >>= 1) {     // the smallest width of the largest S/N
            const double os = __shfl_xor(sn, o);
            const int ob = __shfl_xor(best, o);
            const int32_t ot = __shfl_xor(t, o);
            if (os > sn || (os == sn && ob < best)) {
                sn = os;
                best = ob;
                t = ot;
            }
        }
        if (tid == 0) {
            to_global(a.snr)[row] = a.ne > 0 ? sn : 0.0;
            to_global(a.width)[row] = a.ne > 0 ? sh.wd[best] : a.w_first;
            to_global(a.time)[row] = t;
        }
    }

    // ---- candidates ------------------------------------------------------------------
    if (a.want_cands && a.ne > 0) {
        if (tid < a.ne) {
            const int64_t w = sh.wd[tid];
            const double rsw = sh.rs[tid];
            const auto reaches = [&](int64_t S) { return snr_of(T, S, w, sum, inv_d, rsw) >= a.gamma; };
            // The least S that reaches gamma: near the exact solution, else by
            // bisection (the S/N never falls with S).
            const double x = (a.gamma / (inv_d * rsw) + static_cast<double>(w * sum)) / static_cast<double>(T);
            const int64_t g = static_cast<int64_t>(__builtin_ceil(fmin(fmax(x, -2147483646.0), 2147483646.0)));
            const bool r0 = reaches(g - 1), r1 = reaches(g), r2 = reaches(g + 1);
            int64_t lo = INT32_MIN, hi = INT32_MAX;
            int32_t res;
            if (!r0 && r1) {
                res = static_cast<int32_t>(g);
            } else if (!r1 && r2) {
                res = static_cast<int32_t>(g + 1);
            } else if (reaches(lo)) {
                res = INT32_MIN;
            } else if (!reaches(hi)) {
                res = INT32_MAX;                          // never reached: window sums are < 2^31 - 1
            } else {
                while (hi - lo > 1) {                     // snr(lo) < gamma <= snr(hi)
                    const int64_t mid = lo + (hi - lo) / 2;
                    if (reaches(mid)) hi = mid; else lo = mid;
                }
                res = static_cast<int32_t>(hi);
            }
            sh.sthr[tid] = res;
        }
        __syncthreads();
        for (int tb = tlo; tb < thi; tb += kThreads) {    // 256 tiles are looked at together
            bool hit = tb + tid < thi;
            if (hit && keep_tmax) {
                hit = false;
                for (int i = 0; i < a.ne; ++i) hit = hit || tx_box_tmax[(tb - tlo + tid) * NWT + i] >= max(sh.sthr[i], 0);
            }
            const unsigned long long hits = __ballot(hit);
            if ((tid & 63) == 0) sh.red1[tid >> 6] = hits;
            __syncthreads();
            for (int v = 0; v < kWaves; ++v) {
                const unsigned long long m = sh.red1[v];
                unsigned long long left =                 // uniform
                    static_cast<uint32_t>(uniform(static_cast<int>(m))) |
                    static_cast<unsigned long long>(static_cast<uint32_t>(uniform(static_cast<int>(m >> 32)))) << 32;
                for (; left; left &= left - 1) {
                    const int tile = tb + 64 * v + __builtin_ctzll(left);
                    int tv = tid;                         // opaque, as in row_scan
                    asm volatile("" : "+v"(tv));
                    Moments unused;
                    scan_tile<false>(y, T, tile * kBoxTile, L, sh.P, sh.wtot, vec, tv, unused);
                    if (LIST) cand_tile_list<NWT>(a, sh, row, tile * kBoxTile, sum, inv_d, tv);
                    else cand_tile<NWT>(a, sh, row, tile, keep_tmax, sum, inv_d, tlo, tv);
                    __syncthreads();
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
}


template <int NWT, bool LIST = false>
__device__ __forceinline__ void boxcar_row(const BoxcarArgs& a, int row, BoxShared<NWT>& sh, int tid) {
    const TX_GLOBAL int32_t* __restrict__ y = to_global(a.y) + static_cast<size_t>(row) * a.pitch;
    const bool vec = ((reinterpret_cast<uintptr_t>(a.y) + static_cast<uintptr_t>(row) * a.pitch * 4) & 15) == 0;
    const int ntiles = (a.nt + kBoxTile - 1) / kBoxTile;
    const bool keep_tmax = a.tmax_ok != 0;
    row_setup<NWT, LIST>(a, sh, tid, ntiles, keep_tmax);
    row_scan<NWT, LIST>(a, 0, ntiles, keep_tmax, y, vec, sh, tid);
    row_finish<NWT, LIST>(a, row, a.want_peaks != 0, 0, ntiles, keep_tmax, y, vec, sh, tid);
}

#define TX_BOX_WAVES __attribute__((amdgpu_waves_per_eu(NWT <= 12 ? 7 : NWT <= 16 ? 6 : 5)))

// Single job: one workgroup per row.  62 VGPRs at every width count, so 7
// waves per SIMD; the wave counts asked for (7, 6 from 13 widths, 5 from 17)
// hold the batch form to them, which takes 72 VGPRs and else took 81.  Nothing spills.
template <int NWT>
__global__ __launch_bounds__(kThreads) TX_BOX_WAVES void boxcar_kernel(BoxcarArgs a) {
    __shared__ BoxShared<NWT> sh;
    const int row = static_cast<int>(blockIdx.x);        // grid = rows
    if (row < a.ndm) boxcar_row<NWT>(a, row, sh, static_cast<int>(threadIdx.x));
}

// Single job that lists the candidates of up to kListRows rows of kListTiles
// tiles.  Records are appended as the rows come to them, so their order is that
// of the rows' times.  While all rows run side by side it mostly repeats from
// call to call, and callers compare lists as they come: here a row's time stays
// what it is with one lookup per wavefront and best and one atomic per 64
// starts.  Of the values of 600 to 960 records (128 rows x 8192 samples) 55 to
// 65% differ between two calls of this form, as many between this form and
// one that also solves its thresholds by bisection, and 98% between this form and
// boxcar_kernel or its candidate pass.  That order costs time: with candidates in
// every row and 10 widths 128 x 8192 take 78 us (boxcar_kernel 30), 512 x 16301 105 (49),
// 256 x 61517 165 (split 71), 1280 x 65536 243 (145).  Longer rows, which a split
// lists 6 times as fast, larger calls, whose rows start as others end, and
// batches, whose rows go to whichever workgroup is free, list in the faster forms.
template <int NWT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void boxcar_list_kernel(BoxcarArgs a) {
    __shared__ BoxShared<NWT> sh;
    const int row = static_cast<int>(blockIdx.x);        // grid = rows
    if (row < a.ndm) boxcar_row<NWT, true>(a, row, sh, static_cast<int>(threadIdx.x));
}

// Few rows: each row's tiles are split over `parts` workgroups, in two
// launches.  The first leaves every part's moments, per-width best and
// per-(tile, width) maxima in `ws`; in the second every part of a row puts
// the row together from them, the first part writes its peak and each lists
// the candidates of its own tiles.
struct BoxSplit {
    uint8_t* ws;
    int32_t parts;          // per row, at most 64
    int32_t tpp;            // tiles per part
};

template <int NWT>
struct BoxPart {
    unsigned long long s1, s2;
    int32_t bad, pad;
    int32_t S[NWT], t[NWT];
};

template <int NWT>
__global__ __launch_bounds__(kThreads) TX_BOX_WAVES void boxcar_scan_kernel(BoxcarArgs a, BoxSplit sp) {
    __shared__ BoxShared<NWT> sh;
    const int tid = static_cast<int>(threadIdx.x);
    const int row = static_cast<int>(blockIdx.x) / sp.parts;
    const int part = static_cast<int>(blockIdx.x) % sp.parts;
    if (row >= a.ndm) return;
    if (blockIdx.x == 0 && tid == 0 && a.want_cands) *a.count = 0ull;      // (the next launch counts)
    const TX_GLOBAL int32_t* __restrict__ y = to_global(a.y) + static_cast<size_t>(row) * a.pitch;
    const bool vec = ((reinterpret_cast<uintptr_t>(a.y) + static_cast<uintptr_t>(row) * a.pitch * 4) & 15) == 0;
    const int ntiles = (a.nt + kBoxTile - 1) / kBoxTile;
    const int tlo = part * sp.tpp, thi = min(tlo + sp.tpp, ntiles);
    row_setup<NWT>(a, sh, tid);
    row_scan<NWT>(a, tlo, thi, true, y, vec, sh, tid);
    BoxPart<NWT>* parts = reinterpret_cast<BoxPart<NWT>*>(sp.ws);
    BoxPart<NWT>* p = parts + blockIdx.x;
    if (tid == 0) {
        unsigned long long s1 = 0, s2 = 0;
        int bad = 0;
        for (int v = 0; v < kWaves; ++v) {
            s1 += sh.red1[v];
            s2 += sh.red2[v];
            bad |= sh.redbad[v];
        }
        p->s1 = s1;
        p->s2 = s2;
        p->bad = bad;
    }
    if (tid < NWT) {
        p->S[tid] = sh.bS[tid];
        p->t[tid] = sh.bT[tid];
    }
    int32_t* tm = reinterpret_cast<int32_t*>(parts + static_cast<size_t>(a.ndm) * sp.parts) +
                  static_cast<size_t>(blockIdx.x) * sp.tpp * NWT;
    for (int k = tid; k < (thi - tlo) * NWT; k += kThreads) tm[k] = tx_box_tmax[k];
}

template <int NWT>
__global__ __launch_bounds__(kThreads) TX_BOX_WAVES void boxcar_finish_kernel(BoxcarArgs a, BoxSplit sp) {
    __shared__ BoxShared<NWT> sh;
    const int tid = static_cast<int>(threadIdx.x);
    const int lane = tid & 63, wave = tid >> 6;
    const int row = static_cast<int>(blockIdx.x) / sp.parts;
    const int part = static_cast<int>(blockIdx.x) % sp.parts;
    if (row >= a.ndm) return;
    const TX_GLOBAL int32_t* __restrict__ y = to_global(a.y) + static_cast<size_t>(row) * a.pitch;
    const bool vec = ((reinterpret_cast<uintptr_t>(a.y) + static_cast<uintptr_t>(row) * a.pitch * 4) & 15) == 0;
    const int ntiles = (a.nt + kBoxTile - 1) / kBoxTile;
    const int tlo = part * sp.tpp, thi = min(tlo + sp.tpp, ntiles);
    const BoxPart<NWT>* parts = reinterpret_cast<const BoxPart<NWT>*>(sp.ws);
    row_setup<NWT>(a, sh, tid);
    const int32_t* tm = reinterpret_cast<const int32_t*>(parts + static_cast<size_t>(a.ndm) * sp.parts) +
                        static_cast<size_t>(blockIdx.x) * sp.tpp * NWT;
    for (int k = tid; k < (thi - tlo) * NWT; k += kThreads) tx_box_tmax[k] = tm[k];
    const BoxPart<NWT>* p = parts + static_cast<size_t>(row) * sp.parts + (lane < sp.parts ? lane : 0);   // lane: part
    const bool own = lane < sp.parts;
    if (wave == 0) {
        const unsigned long long s1 = wave_sum(own ? p->s1 : 0ull);
        const unsigned long long s2 = wave_sum(own ? p->s2 : 0ull);
        const int bad = __any(own && p->bad != 0) ? 1 : 0;
        if (lane < kWaves) {
            sh.red1[lane] = lane == 0 ? s1 : 0ull;
            sh.red2[lane] = lane == 0 ? s2 : 0ull;
            sh.redbad[lane] = bad;
        }
    }
    for (int i = wave; i < NWT; i += kWaves) {
        const int32_t S = own ? p->S[i] : INT32_MIN;
        const int32_t m = wave_max_i32(S);
        const int32_t t = wave_min_i32(own && S == m ? p->t[i] : INT32_MAX);
        if (lane == 0) {
            sh.bS[i] = m;
            sh.bT[i] = t;
        }
    }
    __syncthreads();
    row_finish<NWT>(a, row, a.want_peaks != 0 && part == 0, tlo, thi, true, y, vec, sh, tid);
}

__device__ __forceinline__ int find_row_job(const int* __restrict__ prefix, int njobs, int v) {
    int lo = 0, hi = njobs;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= v) lo = mid; else hi = mid;
    }
    return lo;
}

// Batch form: persistent workgroups taking rows of all jobs (job of a row by
// prefix sums) from the launch's work counters.
template <int NWT>
__global__ __launch_bounds__(kThreads) TX_BOX_WAVES void boxcar_batch_kernel(const BoxcarArgs* __restrict__ jobs,
                                                                const int* __restrict__ prefix_base,
                                                                const int* __restrict__ info, uint32_t* queue) {
    __shared__ BoxShared<NWT> sh;
    const int njobs = info[0];
    if (njobs <= 0) return;
    const BoxcarArgs* cj = jobs + info[1];
    const int* prefix = prefix_base + info[2];
    for_each_claimed(prefix[njobs], queue, [&](int v) {
        const int jb = find_row_job(prefix, njobs, v);
        // The thread index, opaque to the compiler in every row: else it
        // keeps lane-dependent values of the row body live across rows.
        int tv = static_cast<int>(threadIdx.x);
        asm volatile("" : "+v"(tv));
        boxcar_row<NWT>(cj[jb], v - prefix[jb], sh, tv);
    });
}

__global__ void zero_u64_kernel(unsigned long long* p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0ull;
}

__global__ void zero_counts_kernel(const BoxcarArgs* __restrict__ jobs, const int* __restrict__ njobs_p) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < *njobs_p && jobs[j].want_cands) *jobs[j].count = 0ull;
}

// ---------------------------------------------------------------------------

int boxcar_tmax_bytes(int nwt, int64_t nt) {
    const int64_t b = (nt + kBoxTile - 1) / kBoxTile * boxcar_nwt(nwt) * 4;
    return b <= kTileMaxLds ? static_cast<int>(b) : 0;
}

struct BoxFns {
    const void* row;
    const void* list;
    const void* scan;
    const void* finish;
    const void* batch;
    int part_bytes;
};

template <int NWT>
static BoxFns box_fns() {
    return {reinterpret_cast<const void*>(&boxcar_kernel<NWT>), reinterpret_cast<const void*>(&boxcar_list_kernel<NWT>),
            reinterpret_cast<const void*>(&boxcar_scan_kernel<NWT>),
            reinterpret_cast<const void*>(&boxcar_finish_kernel<NWT>),
            reinterpret_cast<const void*>(&boxcar_batch_kernel<NWT>), static_cast<int>(sizeof(BoxPart<NWT>))};
}

static BoxFns box_fns(int nwt) {
    switch (nwt) {
        case 4: return box_fns<4>();
        case 8: return box_fns<8>();
        case 10: return box_fns<10>();
        case 12: return box_fns<12>();
        case 16: return box_fns<16>();
        default: return box_fns<32>();
    }
}

// Split of a row's tiles over workgroups (parts 1: none): as far as 6
// workgroups per CU, where they still run side by side at little cost, but
// parts of at least 1 + rows / 128 tiles, and only rows of 3 such parts: the
// second launch costs 6 to 10 us, a tile 4 us on an idle CU and more on a
// full one.  Measured unsplit and split (10 widths, peaks): 96 x 1000003
// samples 1009 and 145 us, 128 x 28749 40 and 32, 256 x 61517 71 and 52,
// 512 x 61517 77 and 66, 512 x 245837 283 and 182; without the limits
// 512 x 12365 28 and 39, 768 x 61517 88 and 91, 1024 x 61517 100 and 101.
static BoxSplit box_split(int rows, int ntiles, int nwt) {
    const int unit = 1 + rows / 128;
    const int parts = ntiles >= 3 * unit ? std::min({ntiles / unit, 64, kSplitGroups / rows}) : 1;
    if (parts < 2) return {nullptr, 1, ntiles};
    const int tpp = (ntiles + parts - 1) / parts;
    if (tpp * nwt * 4 > kTileMaxLds) return {nullptr, 1, ntiles};
    return {nullptr, (ntiles + tpp - 1) / tpp, tpp};
}

hipError_t launch_boxcar(const BoxcarArgs& a_in, hipStream_t stream) {
    BoxcarArgs a = a_in;
    const int nwt = boxcar_nwt(a.ne);
    const BoxFns fn = box_fns(nwt);
    // A split needs scratch; without (or in a capture, which stays one
    // kernel) the rows are not split.
    BoxSplit sp{nullptr, 1, 0};
    Scratch ws;
    const int ntiles = (a.nt + kBoxTile - 1) / kBoxTile;
    const bool list = a.want_cands && a.ndm <= kListRows && ntiles <= kListTiles;
    if (a.ndm > 0 && !list) sp = box_split(a.ndm, ntiles, nwt);
    if (sp.parts > 1) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
        int dev = -1;
        const int64_t n = static_cast<int64_t>(a.ndm) * sp.parts;
        if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone ||
            hipGetDevice(&dev) != hipSuccess || retain_pool(dev) != TX_OK ||
            scratch_get(static_cast<size_t>(n) * (fn.part_bytes + sp.tpp * nwt * 4), stream, &ws) != hipSuccess) {
            (void)hipGetLastError();
            sp.parts = 1;
        }
        sp.ws = static_cast<uint8_t*>(ws.p);
    }
    if (sp.parts > 1) {
        void* args[] = {&a, &sp};
        const dim3 grid(static_cast<uint32_t>(a.ndm) * static_cast<uint32_t>(sp.parts));
        const size_t lds = static_cast<size_t>(sp.tpp) * nwt * 4;
        const int prof = prof_begin(TX_KERNEL_BOXCAR, stream);
        hipError_t e = hipLaunchKernel(fn.scan, grid, dim3(kThreads), args, lds, stream);
        if (e == hipSuccess) e = hipLaunchKernel(fn.finish, grid, dim3(kThreads), args, lds, stream);
        if (e == hipSuccess) e = hipGetLastError();
        prof_end(prof, stream);
        const hipError_t f = scratch_put(&ws, stream);
        return e != hipSuccess ? e : f;
    }
    if (a.want_cands) {
        hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, stream, a.count);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (a.ndm <= 0) return hipSuccess;
    const int lds = boxcar_tmax_bytes(a.ne, a.nt);
    a.tmax_ok = lds > 0 ? 1 : 0;
    const int prof = prof_begin(TX_KERNEL_BOXCAR, stream);
    void* args[] = {&a};
    hipError_t e = hipLaunchKernel(list ? fn.list : fn.row, dim3(a.ndm), dim3(kThreads), args, static_cast<size_t>(lds), stream);
    if (e == hipSuccess) e = hipGetLastError();
    prof_end(prof, stream);
    return e;
}

hipError_t launch_boxcar_batch(int nwt, int lds, const BatchRefs& r, int64_t rows, hipStream_t stream) {
    const BoxcarArgs* jobs = static_cast<const BoxcarArgs*>(r.jobs);
    void* args[] = {&jobs, const_cast<const int**>(&r.prefix), const_cast<const int**>(&r.info),
                    const_cast<uint32_t**>(&r.queue)};
    const void* fn = box_fns(boxcar_nwt(nwt)).batch;
    int grid = resident_grid(fn, lds);
    if (grid <= 0) grid = 256 * 5;
    if (rows > 0 && rows < grid) grid = static_cast<int>(rows);
    const int prof = prof_begin(TX_KERNEL_BOXCAR, stream);
    hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(kThreads), args, static_cast<size_t>(lds), stream);
    if (e == hipSuccess) e = hipGetLastError();
    prof_end(prof, stream);
    return e;
}

hipError_t launch_zero_counts(const BoxcarArgs* d_jobs, const int* d_njobs, int max_jobs, hipStream_t stream) {
    if (max_jobs <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_counts_kernel, dim3((max_jobs + 255) / 256), dim3(256), 0, stream, d_jobs, d_njobs);
    return hipGetLastError();
}

}  // namespace tx
