// Rotary embedding on [heads, n, 128] bf16, in place (Appendix, "RoPE Matrix Representation").
//
// A thread owns four planes of one position: the angles position * base^(-2p/128) and their sines / cosines are evaluated once in
// fp64 (positions reach 2^20, far beyond what fp32 angles resolve) and used for every head; 16 threads hold a row, 16 bytes each.
// The rotated pair is the fp64 result rounded once to bf16, nearest even.  That result is found in fp32 wherever fp32
// decides it: the fp32 value is within 2^-21 (|a| + |b|) of the exact one, and where both ends of that interval round to the
// same bf16 number, so does the exact value.  The few pairs near a rounding boundary (about one in 2^11) and values outside the
// range in which the bound holds are evaluated in fp64.
// Bound by the memory (every element read and written once).  With fp64 arithmetic throughout, 2-byte accesses and one
// head's load in flight the kernel took 164 us for 32 heads x 32768 positions (3.3 TB/s); now 101 us (5.3 TB/s),
// what a large copy reaches.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "vs_common.h"
#include "vs_wave.h"

namespace {

__device__ __forceinline__ double bf16_to_f64(uint16_t b) { return static_cast<double>(__uint_as_float(static_cast<uint32_t>(b) << 16)); }

// fp64 -> bf16 with a single rounding: truncate to fp32, fold the lost bits into a sticky bit
// (round to odd), then round the fp32 to nearest-even bf16.
__device__ __forceinline__ uint16_t f64_to_bf16(double x) {
    float f = __double2float_rz(x);
    uint32_t u = __float_as_uint(f);
    if (static_cast<double>(f) != x) u |= 1u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

constexpr int kThreads = 256;
constexpr int kPositions = kThreads / 16;      // per workgroup
constexpr int kSmallPositions = kThreads / 64; // the same, one plane per thread
constexpr int kBatch = 4;                      // heads whose loads are in flight together

// (a, b) -> (a c - b s, a s + b c); a, b and the results are bf16 bit patterns in the low halves
__device__ __forceinline__ void rotate(uint32_t& a, uint32_t& b, double c, double s, float cf, float sf) {
    const float xa = __uint_as_float(a << 16), xb = __uint_as_float(b << 16);
    const float ra = fmaf(xa, cf, -(xb * sf)), rb = fmaf(xa, sf, xb * cf);
    // rounding of c, s (2^-25 each), of the product and of the sum: below 2^-22 (|a| + |b|) while nothing over- or underflows
    const float size = fabsf(xa) + fabsf(xb);
    const float err = size * 4.76837158203125e-07f;          // 2^-21
    const uint32_t pa = pack_bf16(ra - err, ra + err), pb = pack_bf16(rb - err, rb + err);
    // size in [2^-60, 2^120): also false for NaN and infinity
    const bool in_range = __float_as_uint(size) - 0x21800000u < 0x5a000000u;
    if (in_range && (pa & 0xffffu) == (pa >> 16) && (pb & 0xffffu) == (pb >> 16)) {
        a = pa & 0xffffu;
        b = pb & 0xffffu;
    } else {
        const double da = bf16_to_f64(static_cast<uint16_t>(a)), db = bf16_to_f64(static_cast<uint16_t>(b));
        a = f64_to_bf16(da * c - db * s);
        b = f64_to_bf16(da * s + db * c);
    }
}

// PAIRING 0: planes 4 q .. 4 q + 3 of thread q are the elements 8 q .. 8 q + 7;  1: elements 4 q .. + 3 with 64 + 4 q .. + 3
template <int PAIRING>
__global__ __launch_bounds__(kThreads) void rope_kernel(uint16_t* x, int heads, int heads_per_group, long long n, long long pos0,
                                                        double theta_base) {
    __shared__ double theta[64];
    if (threadIdx.x < 64) theta[threadIdx.x] = pow(theta_base, -2.0 * static_cast<int>(threadIdx.x) / 128.0);
    __syncthreads();
    const int q = threadIdx.x & 15;
    const long long t = static_cast<long long>(blockIdx.x) * kPositions + (threadIdx.x >> 4);
    if (t >= n) return;
    double c[4], s[4];
    float cf[4], sf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        sincos(static_cast<double>(pos0 + t) * theta[4 * q + i], &s[i], &c[i]);
        cf[i] = static_cast<float>(c[i]);
        sf[i] = static_cast<float>(s[i]);
    }
    const int h0 = blockIdx.y * heads_per_group, h1 = min(h0 + heads_per_group, heads);
    for (int h = h0; h < h1; h += kBatch) {
        uint2 u[kBatch][2];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const uint16_t* row = x + (static_cast<long long>(min(h + j, h1 - 1)) * n + t) * 128;
            if (PAIRING == 0) {
                const uint4 w = *reinterpret_cast<const uint4*>(row + 8 * q);
                u[j][0] = make_uint2(w.x, w.y);
                u[j][1] = make_uint2(w.z, w.w);
            } else {
                u[j][0] = *reinterpret_cast<const uint2*>(row + 4 * q);
                u[j][1] = *reinterpret_cast<const uint2*>(row + 64 + 4 * q);
            }
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (h + j >= h1) break;
            uint32_t w[4] = {u[j][0].x, u[j][0].y, u[j][1].x, u[j][1].y};
            if (PAIRING == 0) {                              // word i is plane i
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t a = w[i] & 0xffffu, b = w[i] >> 16;
                    rotate(a, b, c[i], s[i], cf[i], sf[i]);
                    w[i] = a | (b << 16);
                }
            } else {                                         // words 0, 1: first elements of planes 0 .. 3; words 2, 3: second elements
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    uint32_t a0 = w[i] & 0xffffu, a1 = w[i] >> 16, b0 = w[2 + i] & 0xffffu, b1 = w[2 + i] >> 16;
                    rotate(a0, b0, c[2 * i], s[2 * i], cf[2 * i], sf[2 * i]);
                    rotate(a1, b1, c[2 * i + 1], s[2 * i + 1], cf[2 * i + 1], sf[2 * i + 1]);
                    w[i] = a0 | (a1 << 16);
                    w[2 + i] = b0 | (b1 << 16);
                }
            }
            uint16_t* row = x + (static_cast<long long>(h + j) * n + t) * 128;
            if (PAIRING == 0) {
                *reinterpret_cast<uint4*>(row + 8 * q) = make_uint4(w[0], w[1], w[2], w[3]);
            } else {
                *reinterpret_cast<uint2*>(row + 4 * q) = make_uint2(w[0], w[1]);
                *reinterpret_cast<uint2*>(row + 64 + 4 * q) = make_uint2(w[2], w[3]);
            }
        }
    }
}

// The same with one plane per thread, 64 threads a row: a quarter of the angles in a thread's way, which is what the time of a
// small call consists of.  The first heads are requested before the angle is evaluated.
template <int PAIRING>
__global__ __launch_bounds__(kThreads) void rope_small_kernel(uint16_t* x, int heads, int heads_per_group, long long n, long long pos0,
                                                              double theta_base) {
    const int plane = threadIdx.x & 63;
    const long long t = static_cast<long long>(blockIdx.x) * kSmallPositions + (threadIdx.x >> 6);
    if (t >= n) return;
    const int h0 = blockIdx.y * heads_per_group, h1 = min(h0 + heads_per_group, heads);
    uint32_t a[kBatch], b[kBatch];
    auto load = [&](int h) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (h + j >= h1) break;
            const uint16_t* row = x + (static_cast<long long>(h + j) * n + t) * 128;
            if (PAIRING == 0) {
                const uint32_t w = *reinterpret_cast<const uint32_t*>(row + 2 * plane);
                a[j] = w & 0xffffu;
                b[j] = w >> 16;
            } else {
                a[j] = row[plane];
                b[j] = row[plane + 64];
            }
        }
    };
    load(h0);
    double c, s;
    sincos(static_cast<double>(pos0 + t) * pow(theta_base, -2.0 * plane / 128.0), &s, &c);
    const float cf = static_cast<float>(c), sf = static_cast<float>(s);
    for (int h = h0; h < h1; h += kBatch) {
        if (h > h0) load(h);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (h + j >= h1) break;
            rotate(a[j], b[j], c, s, cf, sf);
            uint16_t* row = x + (static_cast<long long>(h + j) * n + t) * 128;
            if (PAIRING == 0) {
                *reinterpret_cast<uint32_t*>(row + 2 * plane) = a[j] | (b[j] << 16);
            } else {
                row[plane] = static_cast<uint16_t>(a[j]);
                row[plane + 64] = static_cast<uint16_t>(b[j]);
            }
        }
    }
}

}  // namespace

extern "C" int vs_rope_apply(void* x_bf16, int heads, int64_t n, int64_t pos0, double theta_base, int pairing,
                             void* stream) {
    if (!x_bf16 || !vs::aligned16(x_bf16) || heads <= 0 || n <= 0 || pos0 < 0) return VS_ERR_INVALID_ARG;
    if (!(theta_base > 1.0) || !isfinite(theta_base)) return VS_ERR_INVALID_ARG;
    if (pairing != 0 && pairing != 1) return VS_ERR_INVALID_ARG;
    if (n > VS_MAX_SEQ) return VS_ERR_UNSUPPORTED;
    // Few angles: one plane per thread.  1 head x 1000 positions 4.3 us with four planes, 3.1 with one, 8 x 1000 6.5 and 4.6, 8 x 2000
    // 6.8 and 5.9, 16 x 1500 7.8 and 7.2; on the other side 1 x 4096 4.5 and 4.7, 4 x 6000 7.9 and 8.0, 8 x 3500 8.1 and 8.2,
    // 32 x 2000 11.7 and 12.4 (wider accesses, a quarter of the requests).
    // Short sequences: the heads are shared out over up to four workgroups per compute unit (three with one plane); every group
    // evaluates the angles again, whole batches of heads stay together.
    const int batches = (heads + kBatch - 1) / kBatch;
    const bool small = n <= (heads == 1 ? 3072 : 4096) && n * batches <= 6144;
    const int positions = small ? kSmallPositions : kPositions;
    const unsigned blocks = static_cast<unsigned>((n + positions - 1) / positions);
    int groups = small ? static_cast<int>(768 / blocks) : blocks < 1024 ? static_cast<int>((1024 + blocks - 1) / blocks) : 1;
    if (groups < 1) groups = 1;
    if (groups > batches) groups = batches;
    const int per_group = (batches + groups - 1) / groups * kBatch;
    groups = (heads + per_group - 1) / per_group;
    const dim3 grid(blocks, static_cast<unsigned>(groups));
    auto* const kernel = small ? (pairing == 0 ? rope_small_kernel<0> : rope_small_kernel<1>) : (pairing == 0 ? rope_kernel<0> : rope_kernel<1>);
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, static_cast<hipStream_t>(stream), static_cast<uint16_t*>(x_bf16), heads, per_group,
                       static_cast<long long>(n), static_cast<long long>(pos0), theta_base);
    VS_LAUNCH_CHECK();
    return VS_OK;
}
