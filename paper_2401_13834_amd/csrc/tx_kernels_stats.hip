// Per-channel power sums of uint8 channel rows for gfx950, the statistics the
// paper's narrow-band RFI filter works on (Sec. 2.2: channels that are
// outliers in skewness and kurtosis across the band are removed).
//
// sums[c] = (sum x, sum x^2, sum x^3, sum x^4) over x = in[c][0 .. nt), exact
// in uint64.  A workgroup reduces one chunk of one row: lanes read 16-byte
// pieces (coalesced along the row) and sum the powers of y = x - 128, whose
// squares fit 16 bits: y and y^2 4 bytes at a time (v_dot4_i32_i8), y^3 and
// y^4 as dot products of 16-bit pairs (v_dot2_i32_i16, v_dot2_u32_u16).  The
// sums of x follow from those of y exactly (integers, mod 2^64), and go
// to the row with 64-bit atomic adds.  Bound: HBM for reads; 3.5 VALU
// operations per byte.  Powers of x byte by byte, with a 64-bit multiply-add
// for each x^4, were bound by VALU: 116 us on 4096 x 122300 samples, now 92
// (5.4 TB/s).
#include <algorithm>

#include "tx_internal.h"

namespace tx {

namespace {

constexpr int kStep = 16384;    // samples a workgroup takes at a time
// Steps per workgroup: up to 8, while 8192 workgroups (4 rounds of 8 per CU)
// remain; a workgroup's reduction and atomics cost about as much as a step
// (4096 x 122300 samples: 111 us with one step each, 92 with up to 7).
constexpr int kMaxSteps = 8;
constexpr int kMinGroups = 8192;

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(256) void power_sums_kernel(const uint8_t* __restrict__ in, int64_t in_pitch,
                                                         int64_t nt, int32_t nchunks, int64_t chunk,
                                                         unsigned long long* __restrict__ sums) {
    __shared__ unsigned long long red[4][4];
    const int c = blockIdx.x / nchunks;
    const int k = blockIdx.x - c * nchunks;
    const int64_t t0 = static_cast<int64_t>(k) * chunk;
    const int64_t t1 = min<int64_t>(nt, t0 + chunk);
    const uint8_t* row = in + static_cast<int64_t>(c) * in_pitch;
    // Sums of y, y^2, y^3 (signed, as two's complement) and y^4.
    unsigned long long s1 = 0, s2 = 0, s3 = 0, s4 = 0;
    const auto add = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        int32_t a1 = 0, a2 = 0, a3 = 0;      // per 16 bytes: |.| <= 2^11, 2^18, 2^25
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t a4 = 0;                 // per 8 bytes: <= 2^31
#pragma unroll
            for (int j = 2 * h; j < 2 * h + 2; ++j) {
                const int32_t y = static_cast<int32_t>(w[j] ^ 0x80808080u);
                a1 = __builtin_amdgcn_sdot4(y, 0x01010101, a1, false);
                a2 = __builtin_amdgcn_sdot4(y, y, a2, false);
                const s16x2 p = __builtin_bit_cast(s16x2, y);
                const s16x2 odd = p >> 8, even = (p << 8) >> 8;
                const s16x2 odd2 = odd * odd, even2 = even * even;       // <= 2^14
                a3 = __builtin_amdgcn_sdot2(odd, odd2, a3, false);
                a3 = __builtin_amdgcn_sdot2(even, even2, a3, false);
                a4 = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, odd2), __builtin_bit_cast(u16x2, odd2), a4, false);
                a4 = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, even2), __builtin_bit_cast(u16x2, even2), a4,
                                            false);
            }
            s4 += a4;
        }
        s1 += static_cast<long long>(a1);
        s2 += static_cast<uint32_t>(a2);
        s3 += static_cast<long long>(a3);
    };
    const uint8_t* p = row + 16 * static_cast<int64_t>(threadIdx.x);
    int64_t ts = t0;
    for (; ts + kStep <= t1; ts += kStep) {  // all of a thread's pieces in flight
        uint4 v[kStep / 4096];
#pragma unroll
        for (int i = 0; i < kStep / 4096; ++i) v[i] = *reinterpret_cast<const uint4*>(p + ts + 4096 * i);
#pragma unroll
        for (int i = 0; i < kStep / 4096; ++i) add(v[i]);
    }
    for (int64_t t = ts + 16 * static_cast<int64_t>(threadIdx.x); t < t1; t += 16 * 256) {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (t + 16 <= t1) {
            add(*reinterpret_cast<const uint4*>(row + t));
        } else {
            for (int j = 0; t + j < t1; ++j) w[j >> 2] |= static_cast<uint32_t>(row[t + j]) << (8 * (j & 3));
            add(make_uint4(w[0], w[1], w[2], w[3]));
        }
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    s3 = wave_sum(s3);
    s4 = wave_sum(s4);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        red[wave][0] = s1;
        red[wave][1] = s2;
        red[wave][2] = s3;
        red[wave][3] = s4;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        unsigned long long m[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = red[0][i] + red[1][i] + red[2][i] + red[3][i];
        // x = y + 128; the zeros that fill up the last piece add nothing.
        const unsigned long long n = static_cast<unsigned long long>((t1 - t0 + 15) / 16 * 16);
        const unsigned long long v =
            threadIdx.x == 0   ? m[0] + (n << 7)
            : threadIdx.x == 1 ? m[1] + (m[0] << 8) + (n << 14)
            : threadIdx.x == 2 ? m[2] + 384 * m[1] + 49152 * m[0] + (n << 21)
                               : m[3] + (m[2] << 9) + 98304 * m[1] + (m[0] << 23) + (n << 28);
        atomicAdd(&sums[4 * c + threadIdx.x], v);
    }
}

__global__ void zero_sums_kernel(unsigned long long* __restrict__ sums, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) sums[i] = 0ull;
}

}  // namespace

hipError_t launch_power_sums(const uint8_t* d_in, int64_t in_pitch, int32_t nchan, int64_t nt, uint64_t* d_sums,
                             hipStream_t stream) {
    if (nchan < 1) return hipSuccess;
    unsigned long long* sums = reinterpret_cast<unsigned long long*>(d_sums);
    const int64_t n4 = 4 * static_cast<int64_t>(nchan);
    hipLaunchKernelGGL(zero_sums_kernel, dim3(static_cast<unsigned>((n4 + 255) / 256)), dim3(256), 0, stream, sums, n4);
    if (nt > 0) {
        const int64_t steps = (nt + kStep - 1) / kStep * nchan;
        const int64_t chunk = std::max<int64_t>(1, std::min<int64_t>(steps / kMinGroups, kMaxSteps)) * kStep;
        const int64_t nchunks = (nt + chunk - 1) / chunk;
        const int64_t grid = nchunks * nchan;
        if (grid > INT32_MAX) return hipErrorInvalidValue;
        hipLaunchKernelGGL(power_sums_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0, stream, d_in, in_pitch,
                           nt, static_cast<int32_t>(nchunks), chunk, sums);
    }
    return hipGetLastError();
}

}  // namespace tx
