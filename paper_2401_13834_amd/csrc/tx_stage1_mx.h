// First stage of the sub-band dedispersion on the matrix cores (gfx950); see
// stage1_mx_tiles.  Included by tx_kernels_dedisp.hip only.
#pragma once

#include <type_traits>

#include "tx_internal.h"

namespace tx {

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

template <int CTRL>
__device__ __forceinline__ int dpp_move(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}

// ---------------------------------------------------------------------------
// B[j][s][e] = sum over ch in s of x[ch][e - (D_j & 15) + D(c_j, f_ch)],
// D_j = D(c_j, f_s): the first stage's series, each row starting D_j & 15
// elements early (the second stage's table holds the same offset).
//
// The sum over channels is a product of a 0/1 matrix and the samples: with
// time v = u + D_j (aligned at the sub-band's reference channel) a channel's
// samples are shifted by d = D(c_j, f_ch) - D_j only, and neighbouring trials
// by nearly the same d.  One 16x16x64 integer MFMA takes 4 channels (one per
// 16 lanes): its B operand holds, per lane, 16 consecutive bytes of a channel
// from the smallest shift of 4 trials; its A operand has 16 rows = 4 trials x
// 4 consecutive outputs, each row a single 1 at its trial's shift beyond that
// smallest one plus its output's place; so it adds 4 channels to 4 trials x 64
// outputs exactly (int8 x int8 into int32).  A lane's bytes start at 4 QN n
// (n = lane & 15), so its operands of consecutive outputs are consecutive
// registers: a second A, moved by 4 bytes, serves the next 4 outputs from the
// same registers, and every other 4 outputs take the window 8 bytes on.
// Trials spread over more than the 16 bytes allow are covered by further
// windows 16 bytes on (nwin; 1.24 on average on the 4096-channel block with
// DM steps of 0.5, bases being rounded down to 4 bytes: the spreads alone, which
// the plan's estimate takes, need 1.18).  Samples are made signed (x - 128); the accumulators
// start at 128 m.
//
// Workgroup = (sub-band, 16 coarse trials, a run of tiles of TT = 64 QN
// outputs), wave w owns trials j0 + 4w .. +3.  Tiles are cut at multiples
// of TT of v for all trials, so that the workgroups of a sub-band read the
// same samples at about the same time.  Rows are staged as in the
// general form (16-byte pieces straight to LDS, range-checked,
// double-buffered, here also from one tile to the next) but from the smallest
// d of the workgroup's trials: TT plus the spread of d, where the general
// form's rows span the trials' full delays.
//
// A lane reads 4 (1 + 2 / QN) bytes of LDS per 4 trials x 4 outputs (the
// general form: 16 (1 + 1 / Q)), and its VALU work is one xor per such dword.
// Bound by the SIMDs' issue: on the 4096-channel, 4096-trial block (8.5e10
// additions) the matrix cores are busy 0.80 of 1.7 ms (43% of the clocks, counted; 2.05 GHz),
// and beside every MFMA of 16 clocks go 3.2 other VALU, 0.9 LDS and 3.0 scalar
// instructions; the general form takes 2.4 ms.  Measured choices: QN = 18 (114 registers, 4
// workgroups per CU) 1.71, 10 1.88, 26 1.94, 34 1.95 ms; exact 1-byte bases
// (v_alignbyte on every operand dword, 8% fewer windows) 2.05; making samples
// signed in LDS 1.95; the next window's samples read ahead 2.0 (128 registers
// with spills, or 3 workgroups per CU); 32 trials per workgroup 1.64, but 3%
// slower on 8192 channels and up to 15% on a few dozen coarse trials.
// ---------------------------------------------------------------------------
// LDS bytes of the tables per channel (padded to a multiple of 4).
constexpr int kMxTabBytes = 17 * kWaves + 4;
constexpr int kMxOneHot = 26 * 16;            // LDS bytes of the table of 16-byte one-hot vectors
constexpr int kMxPad = 320;                   // bytes past the tables (entries are read one channel quad ahead)

// s_waitcnt operand for "vector memory count n", other counters untouched.
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// One stage of a transpose of 4 vectors among 4 neighbouring lanes: lanes
// with `up` clear keep a and take the neighbour's a as b, the others keep b
// and take the neighbour's b as a.
template <int CTRL>
__device__ __forceinline__ void swap_step(v4i& a, v4i& b, bool up) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int na = __builtin_amdgcn_update_dpp(0, a[k], CTRL, 0xF, 0xF, true);
        const int nb = __builtin_amdgcn_update_dpp(0, b[k], CTRL, 0xF, 0xF, true);
        const int x = up ? nb : a[k];
        b[k] = up ? b[k] : na;
        a[k] = x;
    }
}

template <int QN>
__device__ __forceinline__ void stage1_mx_tiles(const Stage1Args& a, int item, uint8_t* lds, int* red, int tid) {
    constexpr int J = 4 * kWaves;            // trials per workgroup: a row of 16 lanes of the table pass
    static_assert(J == 16, "one DPP row per channel");
    constexpr int TS = 4 * QN;               // outputs (bytes) per lane and trial
    constexpr int TT = 16 * TS;
    constexpr int NR = QN + 2;               // operand dwords of a window
    static_assert(QN % 8 == 2, "pieces of 8 outputs, 4 at a time and one left");
    const int jc = item % a.n_jchunks;
    const int rest = item / a.n_jchunks;
    const int tr = rest % a.n_ttiles;        // run of tiles
    const int s = rest / a.n_ttiles;
    const int j0 = jc * J;
    const int jl = min(j0 + J, a.ngroups) - 1;
    const int lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int ch0 = s * a.m;
    const int xo = a.x_off;
    const TX_GLOBAL int32_t* __restrict__ dT = to_global(a.dT);
    const size_t gp = static_cast<size_t>(a.gpad);
    const TX_GLOBAL int32_t* __restrict__ cT = to_global(a.cT) + static_cast<size_t>(s) * gp;
    // The run's tiles within the workgroup's range of v.
    const int vend = (uniform(cT[jl]) & ~15) + a.len;
    int v0 = ((uniform(cT[j0]) & ~15) / TT + tr * a.tiles_per_run) * TT;   // the tile's first v
    const int v_stop = min(vend, v0 + a.tiles_per_run * TT);
    if (v0 >= v_stop) return;

    // Tables at the top of LDS.  Per channel (padded to a multiple of 4) and
    // trial: the smallest shift of its 4 trials from the staged row's start,
    // rounded down to 4 bytes (high half), and its own beyond that (low half);
    // per 4 channels and 4 trials the windows; per channel the byte
    // of its row that the staged row starts at for v = 0 (a dropped channel:
    // past the row); and A operands by the place of
    // their 1, place p - 5 at row p (none outside 0..15).
    const int mp = (a.m + 3) & ~3;
    const int fix_off = (a.lds_bytes - kMxOneHot - kMxPad - mp * kMxTabBytes) & ~15;
    v4u* onehot = reinterpret_cast<v4u*>(lds + fix_off);
    uint32_t* tab = reinterpret_cast<uint32_t*>(lds + fix_off + kMxOneHot);   // [mp][J]
    uint32_t* rst = tab + mp * J;                                             // [mp]
    int32_t* tab_n = reinterpret_cast<int32_t*>(rst + mp);                    // [mp / 4][kWaves]
    if (tid < 26) {
        const int q = (tid - 5) >> 2;
        const uint32_t one = 1u << (((tid - 5) & 3) * 8);
        onehot[tid] = v4u{q == 0 ? one : 0u, q == 1 ? one : 0u, q == 2 ? one : 0u, q == 3 ? one : 0u};
    }
    int span = 0;
    for (int t = tid; t < mp * J; t += kThreads) {
        const int c = t >> 4, k = t & 15;
        const int ch = ch0 + min(c, a.m - 1);
        const int j = min(j0 + k, jl);
        const int d = xo + dT[static_cast<size_t>(ch) * gp + j] - cT[j];
        int lo = min(d, dpp_move<0xB1>(d)), hi = max(d, dpp_move<0xB1>(d));   // quad_perm [1,0,3,2]
        lo = min(lo, dpp_move<0x4E>(lo));                                       // quad_perm [2,3,0,1]
        hi = max(hi, dpp_move<0x4E>(hi));
        int rlo = min(lo, dpp_move<0x124>(lo));                                 // row_ror:4, row_ror:8
        rlo = min(rlo, dpp_move<0x128>(rlo));
        int rhi = max(hi, dpp_move<0x124>(hi));
        rhi = max(rhi, dpp_move<0x128>(rhi));
        const int st = rlo & ~15;
        // (a padding channel adds nothing)
        const int l4 = (lo - st) & ~3;
        tab[t] = (static_cast<uint32_t>(l4) << 16) | (c < a.m ? static_cast<uint32_t>(d - st - l4) : 0xC000u);
        if (k == 0) {
            const bool keep = !a.mask || to_global(a.mask)[ch] != 0;
            rst[c] = keep ? static_cast<uint32_t>(st) : 0x80000000u;
        }
        span = max(span, rhi - st);
    }
    span = uniform(block_max(span, red));
    const int rowbytes = (span + TT + 35) & ~15;      // last byte read: span + 7 + TT + 12
    const int nbuf = 8 * rowbytes <= fix_off ? 2 : 1;   // two staging buffers where each holds 4 rows
    const int nch = max(4, min(mp, (fix_off / nbuf / rowbytes) & ~3));
    const int buf_bytes = nch * rowbytes;
    for (int t = tid; t < mp / 4 * kWaves; t += kThreads) {     // (4 channels, 4 trials)
        const uint32_t* e = tab + t / kWaves * 4 * J + t % kWaves * 4;
        uint32_t r = 0;
        for (int c = 0; c < min(4, a.m - t / kWaves * 4); ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) r = max(r, e[c * J + k] & 0xFFFFu);
        tab_n[t] = 1 + ((r + 7) >> 4);
    }

    // Row c of the round of channels [cb, cb + nch) of the tile at v into
    // `dat`: whole 16-byte pieces straight to LDS through a buffer resource of
    // the row (zeros past its end, and everywhere for a dropped channel).
    // Samples past a row's valid bytes enter only elements that no output
    // uses, so a row ends with the piece that straddles them; the input's
    // last row must not be read past them, and that piece of it goes through
    // registers.
    const uint32_t valid = static_cast<uint32_t>(a.x_len + xo);      // from the row's base
    const uint8_t* xs = a.x + static_cast<size_t>(ch0) * a.x_pitch;
    const int last_row = a.nchan - 1 - ch0;
    const int pieces = rowbytes >> 4, kfull = pieces >> 6;
    const bool tail = lane < (pieces & 63);
    auto stage_row = [&](int v, int cb, int c, uint32_t st, uint8_t* dat) {
        const uint8_t* row = xs + static_cast<size_t>(cb + c) * a.x_pitch;
        const uint32_t whole = (cb + c == last_row ? valid : valid + 15u) & ~15u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(row), static_cast<short>(0), static_cast<int>(whole), kRawBufferWord3);
        const uint32_t o0 = st + static_cast<uint32_t>(v);
        uint32_t off = o0 + 16u * lane;
        uint8_t* dst = dat + c * rowbytes;
        uint8_t* d16 = dst;
        for (int k = 0; k < kfull; ++k, off += 1024u, d16 += 1024)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, to_lds(d16), 16, off, 0, 0, 0);
        if (tail) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, to_lds(d16), 16, off, 0, 0, 0);
        if (cb + c == last_row && whole - o0 < static_cast<uint32_t>(rowbytes)) {
            __builtin_amdgcn_s_waitcnt(kWaitVm0);            // (the loads have written zeros there)
            if (static_cast<uint32_t>(lane) < valid - whole) dst[whole - o0 + lane] = to_global(row)[whole + lane];
        }
    };
    auto stage = [&](int v, int cb, uint8_t* dat) {
        const int nc = min(nch, a.m - cb);
        for (int c = wave; c < nc; c += kWaves)
            stage_row(v, cb, c, static_cast<uint32_t>(uniform(static_cast<int>(rst[cb + c]))), dat);
    };

    // v of element 0 of the rows of the wave's trials (uniform).
    int e0[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) e0[p] = uniform(cT[min(j0 + 4 * wave + p, jl)]) & ~15;
    const int kg = lane >> 4;
    const uint32_t* lane_t = tab + kg * J + 4 * wave + ((lane >> 2) & 3);   // the lane's entry of channel quad 0
    const int lane_b = kg * rowbytes + TS * (lane & 15);
    const uint8_t* lane_a = reinterpret_cast<const uint8_t*>(onehot + 5);
    const int z = 128 * a.m;
    v4i acc[QN];
#pragma unroll
    for (int q = 0; q < QN; ++q) acc[q] = v4i{z, z, z, z};

    __syncthreads();
    stage(v0, 0, lds);
    int buf = 0;
    bool stores = false;                      // (uniform) the wave's stores of the last tile follow its rows' loads
    for (; v0 < v_stop; v0 += TT) {
        const bool active = j0 + 4 * wave <= jl && v0 < e0[3] + a.len && v0 + TT > e0[0];   // some trial of the wave needs the tile
        for (int cb = 0; cb < a.m; cb += nch) {
            const int nc = min(nch, a.m - cb);
            const bool last = cb + nch >= a.m;
            uint8_t* dat = lds + buf * buf_bytes;
            buf ^= nbuf - 1;
            // This wave's rows of the round have landed; after the barrier
            // every wave's have, and nobody still reads the other buffer.
            // Stores of the last tile, issued after those rows' loads, may
            // still be on their way.
            if (stores) __builtin_amdgcn_s_waitcnt(wait_vm(QN / 2));
            else __builtin_amdgcn_s_waitcnt(kWaitVm0);
            stores = false;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int nv = last ? v0 + TT : v0, ncb = last ? 0 : cb + nch;   // the next round
            // The next round's rows are loaded one by one between the passes:
            // a row's loads take longer to issue than to arrive when a wave
            // issues all of its rows at once.
            const int nnc = nbuf == 2 && nv < v_stop ? min(nch, a.m - ncb) : 0;
            uint8_t* ndat = lds + buf * buf_bytes;
            int nr = wave;
            if (active) {
                int dl = static_cast<int>(dat - lds) + lane_b;
                // The tables' entries of a channel quad are read one quad
                // ahead (past the end of the table after the last).
                const uint32_t* tp = lane_t + cb * J;
                const int32_t* np = tab_n + cb / 4 * kWaves + wave;
                uint32_t nt = *tp;
                int nn = *np;
                uint32_t nst = rst[nnc > nr ? ncb + nr : 0];
                for (int c = 0; c < nc; c += 4) {
                    int pos = static_cast<int16_t>(nt) + (lane & 3);       // the place of the row's 1
                    // The window's samples in LDS.  Windows that only the
                    // quad's other channels need (no 1 of this channel is in
                    // them) stay within the row.
                    int wo = dl + static_cast<int>(nt >> 16);
                    const int wlast = dl + rowbytes - TT - 8;
                    int nwin = uniform(nn);
                    tp += 4 * J;
                    np += kWaves;
                    nt = *tp;
                    nn = *np;
                    dl += 4 * rowbytes;
                    if (nr < nnc) {
                        const uint32_t st = static_cast<uint32_t>(uniform(static_cast<int>(nst)));
                        stage_row(nv, ncb, nr, st, ndat);
                        nr += kWaves;
                        nst = rst[nnc > nr ? ncb + nr : 0];
                    }
                    __builtin_amdgcn_s_setprio(1);        // (1 to 2% on the 4096-channel block)
                    do {
                        asm volatile("" : "+v"(wo));      // (each window's samples are read anew)
                        const uint32_t* w = reinterpret_cast<const uint32_t*>(lds + wo);
                        uint32_t x[NR];
#pragma unroll
                        for (int q = 0; q < NR; ++q) x[q] = w[q];
                        const uint8_t* ap = lane_a + 16 * min(max(pos, -5), 16);
                        const v4i ae = *reinterpret_cast<const v4i*>(ap);
                        const v4i ao = *reinterpret_cast<const v4i*>(ap + 64);
                        // Samples are made signed while the matrix core works
                        // on the last ones.
                        uint32_t b[NR];
#pragma unroll
                        for (int q = 0; q < 4; ++q) b[q] = x[q] ^ 0x80808080u;
#pragma unroll
                        for (int q = 0; q < QN; q += 2) {
                            const v4i bv = {static_cast<int>(b[q]), static_cast<int>(b[q + 1]),
                                            static_cast<int>(b[q + 2]), static_cast<int>(b[q + 3])};
                            acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ae, bv, acc[q], 0, 0, 0);
                            acc[q + 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ao, bv, acc[q + 1], 0, 0, 0);
                            if (q + 2 < QN) {
                                b[q + 4] = x[q + 4] ^ 0x80808080u;
                                b[q + 5] = x[q + 5] ^ 0x80808080u;
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        wo = min(wo + 16, wlast);
                        pos -= 16;
                    } while (--nwin > 0);
                    __builtin_amdgcn_s_setprio(0);
                }
            }
            for (; nr < nnc; nr += kWaves) 
                stage_row(nv, ncb, nr, static_cast<uint32_t>(uniform(static_cast<int>(rst[ncb + nr]))), ndat);
            if (last && active) {
                // Outputs: lane (p, n) holds outputs TS n .. TS n + TS - 1 of
                // trial p, as QN / 2 pieces of 8 uint16 (16 bytes).  Lanes n
                // are transposed in fours, 4 pieces at a time, so that 4 lanes
                // store 64 contiguous bytes; the last piece leaves by itself.
                // Stores are range-checked buffer stores, all issued, so that
                // the next round can wait for its rows and not for them.
                int lv = lane;                            // opaque: nothing of this pass is kept across tiles
                asm volatile("" : "+v"(lv));
                const int g4 = lv >> 4, b4 = lv & 3;
                const uint32_t len = static_cast<uint32_t>(a.len);
                const int eg = v0 - (g4 == 0 ? e0[0] : g4 == 1 ? e0[1] : g4 == 2 ? e0[2] : e0[3]);
                const bool real = j0 + 4 * wave + g4 <= jl;
                const uint32_t jb = static_cast<uint32_t>(a.nsub) * static_cast<uint32_t>(a.B_pitch) * 2u;
                uint16_t* rows = a.B + (static_cast<size_t>(j0 + 4 * wave) * a.nsub + s) * a.B_pitch;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    rows, static_cast<short>(0), static_cast<int>(3u * jb + 2u * len), kRawBufferWord3);
                auto put = [&](int e, const v4i& v) {
                    const uint32_t off = real && static_cast<uint32_t>(e) < len
                                             ? g4 * jb + 2u * static_cast<uint32_t>(e) : 0x80000000u;
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rs, off, 0, 0);
                };
                auto piece = [&](int i) {
                    const v4i f = acc[2 * i], g = acc[2 * i + 1];
                    return v4i{f[0] | (f[1] << 16), f[2] | (f[3] << 16), g[0] | (g[1] << 16), g[2] | (g[3] << 16)};
                };
                const int e4 = eg + TS * (lv & 12) + 8 * b4;
#pragma unroll
                for (int h = 0; h < QN / 8; ++h) {
                    v4i w[4] = {piece(4 * h), piece(4 * h + 1), piece(4 * h + 2), piece(4 * h + 3)};
                    swap_step<0xB1>(w[0], w[1], b4 & 1);
                    swap_step<0xB1>(w[2], w[3], b4 & 1);
                    swap_step<0x4E>(w[0], w[2], b4 & 2);
                    swap_step<0x4E>(w[1], w[3], b4 & 2);
#pragma unroll
                    for (int k = 0; k < 4; ++k) put(e4 + TS * k + 32 * h, w[k]);
                }
                put(eg + TS * (lv & 15) + TS - 8, piece(QN / 2 - 1));
                stores = true;
#pragma unroll
                for (int q = 0; q < QN; ++q) acc[q] = v4i{z, z, z, z};
            }
            if (nbuf == 1 && nv < v_stop) {
                __syncthreads();                          // `dat` has been read
                stage(nv, ncb, lds);
                stores = false;                           // (the rows come after the stores)
            }
        }
    }
}

}  // namespace tx
