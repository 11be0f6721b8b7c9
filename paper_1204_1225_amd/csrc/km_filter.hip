// Trace pre-filter: a finite impulse response applied to every trace before
// migration (the rho filter that makes the summation of Eq. (1) return a
// zero-phase wavelet), and its transpose after demigration.
//
//   forward  y[n] = sum_k h[k] x[n + c - k]
//   adjoint  x[m] = sum_k h[k] y[m - c + k]
// (zero outside [0, N)).  Both are correlations out[n] = sum_k w[k] in[n + off + k]:
// forward with the reversed taps and off = c - (K - 1), adjoint with the taps
// and off = -c.
//
// Each trace is staged in LDS between zeros by one wavefront (a workgroup
// filters kFirWaves traces at a time), or by the whole workgroup where the
// traces are few or long; it is fully staged before any of its output is written, so
// the output may be the input.  A lane produces kOut consecutive outputs from a
// window of input values in registers: 4 taps cost one 16-byte read of the
// trace and one broadcast 16-byte read of the taps for 4 kOut FMAs, each output
// summed in tap order.  Bounds for the 3D survey (200 000 x 1500 samples, 65
// taps): 0.50 ms of FP32 issue, 0.51 ms for the traces at the rate of a large
// copy.  With 4 outputs per lane and single reads the LDS held it at 1.55 ms.
#include <algorithm>

#include "km_kernels.h"

namespace km {

constexpr int kFirThreads = 256;
constexpr int kFirWaves = kFirThreads / kLanes;
constexpr int kOut = 8;

// Four floats at any float address (rows may have any stride).
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));

// LDS floats of one staged trace: `lead` zeros (lead >= K, lead + off a
// multiple of 4 for either direction's off), the record, zeros to the last
// read of a lane that starts inside the record.  TIGHT (records that leave no
// room for that): K zeros on each side, single reads clamped to the row; what a
// clamped read returns is used only by outputs past the record, which are dropped.
__host__ __device__ inline int fir_row(int n, int K) { return ((n + kOut - 1) / kOut * kOut + 2 * K + 3 + kOut + 3) & ~3; }

template <bool TIGHT>
__global__ __launch_bounds__(kFirThreads) void fir_kernel(const float* in, int64_t in_stride, float* out,
                                                         int64_t out_stride, int64_t n_traces, int n, int K,
                                                         const float* __restrict__ taps, int c, int adjoint,
                                                         int per) {
    extern __shared__ __align__(16) float fir_lds[];
    float* sW = fir_lds;  // [K rounded up to 4] correlation weights
    const int off = adjoint ? -c : c - (K - 1);  // -(K - 1) .. 0
    const int lead = TIGHT ? K : K + ((-(off + K)) & 3);
    const int row = TIGHT ? n + 2 * K : fir_row(n, K);
    // `per` traces at a time: thread `lane` of `width` on trace `sub`
    const int width = kFirThreads / per;
    const int sub = threadIdx.x / width, lane = threadIdx.x % width;
    float* sIn = fir_lds + ((K + 3) & ~3) + sub * row;  // sIn[lead + p] = in[p]
    for (int k = threadIdx.x; k < K; k += kFirThreads) sW[k] = adjoint ? taps[k] : taps[K - 1 - k];
    for (int p = lane; p < lead; p += width) sIn[p] = 0.0f;
    for (int p = lead + n + lane; p < row; p += width) sIn[p] = 0.0f;
    for (int64_t j0 = static_cast<int64_t>(blockIdx.x) * per; j0 < n_traces; j0 += static_cast<int64_t>(gridDim.x) * per) {
        const int64_t j = j0 + sub;
        __syncthreads();  // the previous trace's readers are done
        if (j < n_traces) {
            const float* src = in + j * in_stride;
            constexpr int kAhead = 4;  // loads in flight
            for (int p0 = 4 * lane; p0 < n; p0 += 4 * width * kAhead) {
                float4_any v[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int p = p0 + 4 * width * u;
                    if (p + 4 <= n) v[u] = *reinterpret_cast<const float4_any*>(src + p);
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int p = p0 + 4 * width * u;
                    if (p + 4 <= n) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) sIn[lead + p + r] = v[u][r];
                    }
                }
            }
            for (int p = (n & ~3) + lane; p < n; p += width) sIn[lead + p] = src[p];
        }
        __syncthreads();
        if (j >= n_traces) continue;
        float* dst = out + j * out_stride;
        for (int n0 = lane * kOut; n0 < n; n0 += width * kOut) {
            const int x0 = n0 + lead + off;  // sIn[x0 + k + r] = in[n0 + r + off + k]
            auto read4 = [&](int i) {
                if (!TIGHT) return *reinterpret_cast<const float4*>(sIn + i);
                return make_float4(sIn[min(i, row - 1)], sIn[min(i + 1, row - 1)], sIn[min(i + 2, row - 1)],
                                   sIn[min(i + 3, row - 1)]);
            };
            float acc[kOut], w[kOut + 4];
#pragma unroll
            for (int r = 0; r < kOut; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int m = 0; m < kOut; m += 4) {
                const float4 v = read4(x0 + m);
                w[m] = v.x, w[m + 1] = v.y, w[m + 2] = v.z, w[m + 3] = v.w;
            }
            int k = 0;
            for (; k + 4 <= K; k += 4) {
                const float4 v = read4(x0 + k + kOut);
                const float4 h = *reinterpret_cast<const float4*>(sW + k);
                w[kOut] = v.x, w[kOut + 1] = v.y, w[kOut + 2] = v.z, w[kOut + 3] = v.w;
                const float hk[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int r = 0; r < kOut; ++r) acc[r] = fmaf(hk[u], w[u + r], acc[r]);
#pragma unroll
                for (int m = 0; m < kOut; ++m) w[m] = w[m + 4];
            }
            for (; k < K; ++k) {
                const float hk = sW[k];
#pragma unroll
                for (int r = 0; r < kOut; ++r) acc[r] = fmaf(hk, w[r], acc[r]);
#pragma unroll
                for (int m = 0; m < kOut - 1; ++m) w[m] = w[m + 1];
                w[kOut - 1] = sIn[min(x0 + k + kOut, row - 1)];
            }
            if (n0 + kOut <= n) {
#pragma unroll
                for (int r = 0; r < kOut; r += 4)
                    *reinterpret_cast<float4_any*>(dst + n0 + r) =
                        float4_any{acc[r], acc[r + 1], acc[r + 2], acc[r + 3]};
            } else {
#pragma unroll
                for (int r = 0; r < kOut; ++r)
                    if (n0 + r < n) dst[n0 + r] = acc[r];
            }
        }
    }
}

static size_t fir_bytes(int n, int K, int per) {
    return sizeof(float) * (static_cast<size_t>((K + 3) & ~3) + static_cast<size_t>(per) * fir_row(n, K));
}

// The least LDS a call needs (the tight layout).
size_t fir_lds_bytes(int n, int K) {
    return sizeof(float) * (static_cast<size_t>((K + 3) & ~3) + n + 2 * static_cast<size_t>(K));
}

hipError_t launch_fir(const float* in, int64_t in_stride, float* out, int64_t out_stride, int64_t n_traces, int n,
                      const float* taps, int K, int c, int adjoint, hipStream_t s) {
    // A wavefront per trace where there are traces enough to fill the chip so, and as long as
    // four workgroups share a CU's LDS; else a workgroup per trace.  us, the one / the other:
    // 256 x 1500 samples, 65 taps 9.5 / 8.2; 256 x 600, 129 taps 10.5 / 8.2; 2000 x 600 11.1 /
    // 11.3; 6000 x 1500 25.5 / 24.3; 20 000 x 1500 70 / 74; 256 and 20 000 x 3000, 129 taps
    // 26.9 / 11.2 and 263 / 231.
    const int per = n_traces >= 4096 && fir_bytes(n, K, kFirWaves) <= 40 * 1024 ? kFirWaves : 1;
    const int64_t blocks = std::min<int64_t>((n_traces + per - 1) / per, 256 * 16);
    const bool tight = fir_bytes(n, K, per) > 160 * 1024;
    return launch_with_lds(tight ? fir_kernel<true> : fir_kernel<false>, dim3(static_cast<unsigned>(blocks)),
                           dim3(kFirThreads), tight ? fir_lds_bytes(n, K) : fir_bytes(n, K, per), s, in, in_stride, out,
                           out_stride, n_traces, n, K, taps, c, adjoint, per);
}

}  // namespace km
