// Offset stack and the moveout measure of the offset images (the redundant
// images of the Introduction: their disagreement in reflector depth measures
// the velocity error; once they agree they are summed).
//
// stack_kernel   stack[p] = sum_b image[b][p]: one pass over the image, float4
//                when aligned; HBM-bound.
// cig_kernel     one workgroup per image column: the column's n_bins depth
//                vectors are staged in LDS (zero-padded on both sides), the stack
//                is formed in float64, every (bin, lag) correlation over the depth
//                window is a float64 dot product of LDS rows, then 16 lanes per
//                bin pick the best lag (ties to the smaller |lag|, then the
//                negative one) and refine it by the parabola through its
//                neighbours; one wavefront fits the shift against offset^2.
#include <algorithm>
#include <climits>

#include "km_kernels.h"

namespace km {

constexpr int kCigThreads = 256;

__global__ __launch_bounds__(256) void stack_kernel(const float* __restrict__ img, int n_bins, int64_t n_points,
                                                    int vec, float* __restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (vec) {
        const int64_t n4 = n_points >> 2;
        const float4* in4 = reinterpret_cast<const float4*>(img);
        float4* out4 = reinterpret_cast<float4*>(out);
        for (int64_t i = t0; i < n4; i += stride) {
            float4 s = in4[i];
            for (int b = 1; b < n_bins; ++b) {
                const float4 v = in4[static_cast<int64_t>(b) * n4 + i];
                s.x += v.x;
                s.y += v.y;
                s.z += v.z;
                s.w += v.w;
            }
            out4[i] = s;
        }
    } else {
        for (int64_t i = t0; i < n_points; i += stride) {
            float s = img[i];
            for (int b = 1; b < n_bins; ++b) s += img[static_cast<int64_t>(b) * n_points + i];
            out[i] = s;
        }
    }
}

// One workgroup per image column at a time.  LDS: the rows [n_bins][rl] float,
// zero for `lead` >= L floats before the column and behind it; the stack [nz]
// double; the correlations C [n_bins][2 L + 1] double; shifts and peaks
// [n_bins] double each.  The partial sums of the depth parts, [zs][n_bins][2 L
// + 1] double, take the rows' place once the correlations are formed.
//
// Correlation: thread item = (bin, block of LB lags, depth part).  A rotating
// window of LB row values in registers makes a depth step cost one row read,
// one stack read (the same for the lanes of a part) and LB float64 FMAs.  The
// work is n_bins (2 L + 1) window FMAs per column, 0.28 ms of float64 issue for
// the 3D survey (65536 columns, 16 bins, 400 depths, 25 lags) beside 0.38 ms
// for reading the image at the rate of a large copy; with blocks of 5 lags the
// LDS reads held it at 2.36 ms.
struct CigShape {
    int lb, nblk, zs, lead, rl;
    int region;  // bytes of the rows, a multiple of 16
};

// Row length: lead and tail zeros, a multiple of 4 floats (16-byte row stores);
// 4 times an odd number unless `tight`, so that the bins of a wavefront read
// different banks.
__host__ __device__ inline CigShape cig_shape(int n_bins, int nz, int L, int lb, bool tight) {
    CigShape s;
    const int nl = 2 * L + 1;
    s.lb = lb;
    s.nblk = (nl + lb - 1) / lb;
    s.lead = (L + 3) & ~3;
    s.rl = (s.lead + nz + (s.nblk * lb - L) + lb - 2 + 3) & ~3;
    if (!tight && (s.rl & 4) == 0) s.rl += 4;
    const int items = n_bins * s.nblk;
    s.zs = items >= kCigThreads ? 1 : kCigThreads / items;
    // the partial sums fit in the rows' place
    const int fit = static_cast<int>(static_cast<int64_t>(s.rl) / (2 * nl));
    if (s.zs > fit) s.zs = fit > 1 ? fit : 1;
    s.region = static_cast<int>((static_cast<int64_t>(n_bins) * s.rl * 4 + 15) & ~int64_t{15});
    return s;
}

inline size_t cig_shape_bytes(const CigShape& s, int n_bins, int nz, int L) {
    const size_t nl = 2 * static_cast<size_t>(L) + 1, nb = n_bins;
    return (nb * s.rl * sizeof(float) + 15) / 16 * 16 + sizeof(double) * (nz + nb * nl + 2 * nb);
}

// The lag block that wastes least: FMAs of the padded lags plus the reads and
// conversions of a step (about 4 FMAs' time), among the blocks that fit in LDS.
constexpr int kCigMaxLds = 160 * 1024;
inline CigShape cig_choose(int n_bins, int nz, int L) {
    CigShape best = cig_shape(n_bins, nz, L, 5, true);
    double cost = 1.0e300;
    for (const int lb : {13, 11, 9, 7, 5}) {
        const CigShape s = cig_shape(n_bins, nz, L, lb, false);
        const double c = s.nblk * (lb + 4.0);
        if (c < cost && cig_shape_bytes(s, n_bins, nz, L) <= static_cast<size_t>(kCigMaxLds)) {
            cost = c;
            best = s;
        }
    }
    return best;
}

// Partial C_b(l) over depths [za, zb) for l = lag0 .. lag0 + LB - 1: slot
// (u + j) % LB of the window holds row[z + u + lag0 + j].  Steps past zb use a
// zero stack value; where that meets an infinity or a NaN below the depth window
// the sums are formed again without them (a guard around those steps instead:
// 1.20 -> 1.23 ms on the 3D survey).
template <int LB>
__device__ __forceinline__ void lag_block(const double* sS, const float* row, int lag0, int za, int zb, double* c) {
    double w[LB];
#pragma unroll
    for (int j = 0; j < LB; ++j) c[j] = 0.0;
    if (za >= zb) return;
#pragma unroll
    for (int m = 0; m < LB - 1; ++m) w[m] = static_cast<double>(row[za + lag0 + m]);
    for (int z = za; z < zb; z += LB) {
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            // the row's tail is long enough that every read stays in it
            w[(u + LB - 1) % LB] = static_cast<double>(row[z + u + lag0 + LB - 1]);
            const double sv = (z + u < zb) ? sS[z + u] : 0.0;
#pragma unroll
            for (int j = 0; j < LB; ++j) c[j] = fma(sv, w[(u + j) % LB], c[j]);
        }
    }
    bool nan = false;
#pragma unroll
    for (int j = 0; j < LB; ++j) nan = nan || c[j] != c[j];
    if (nan) {
#pragma unroll
        for (int j = 0; j < LB; ++j) c[j] = 0.0;
#pragma unroll 1
        for (int z = za; z < zb; ++z) {
#pragma unroll
            for (int j = 0; j < LB; ++j) c[j] = fma(sS[z], static_cast<double>(row[z + lag0 + j]), c[j]);
        }
    }
}

// Sum over the wavefront, every lane gets it (fixed order).
__device__ __forceinline__ double wave_sum_d(double v) { return last_lane_d(wave_scan_d(v)); }

// One step of a 16-lane group's best lag: against the lane ROR places away (lane
// moves, as in wave_sum_d; through LDS permutes they held the kernel at 1.23 ms,
// now 1.20 ms).
template <int ROR>
__device__ __forceinline__ void better_lag(double& top, int& rank) {
    const double v = dpp_d<0x120 + ROR, 0xf>(top);
    const int r = __builtin_amdgcn_update_dpp(0, rank, 0x120 + ROR, 0xf, 0xf, true);
    if (v > top || (v == top && r < rank)) {
        top = v;
        rank = r;
    }
}

template <int LB>
__global__ __launch_bounds__(kCigThreads) void cig_kernel(const float* __restrict__ img, int n_bins, int ny, int nx,
                                                         int nz, int L, int z_lo, int z_hi, CigShape shape, int vec,
                                                         const float* __restrict__ offsets, float* stack,
                                                         float* shift, float* peak, float* curvature) {
    extern __shared__ __align__(16) unsigned char cig_lds[];
    const int nl = 2 * L + 1;
    const int rl = shape.rl, lead = shape.lead, nblk = shape.nblk, zs = shape.zs;
    const int items = n_bins * nblk * zs;
    const int zlen = (z_hi - z_lo + zs - 1) / zs;
    float* sRow = reinterpret_cast<float*>(cig_lds);                // [n_bins][rl]
    double* sP = reinterpret_cast<double*>(cig_lds);                // [zs][n_bins][nl], in the rows' place
    double* sS = reinterpret_cast<double*>(cig_lds + shape.region);  // [nz]
    double* sC = sS + nz;                                           // [n_bins][nl]
    double* sShift = sC + static_cast<int64_t>(n_bins) * nl;        // [n_bins]
    double* sPeak = sShift + n_bins;                                // [n_bins]
    const int64_t ncol = static_cast<int64_t>(ny) * nx;
    const int64_t bin_stride = ncol * nz;
    const int tid = threadIdx.x;

    for (int64_t col = blockIdx.x; col < ncol; col += gridDim.x) {
        __syncthreads();  // the previous column's readers are done
        const float* src = img + col * nz;
        if (vec) {  // nz a multiple of 4, image 16-byte aligned
            const int n4 = nz >> 2, total = n_bins * n4;
            constexpr int kAhead = 4;
            for (int e0 = tid; e0 < total; e0 += kAhead * kCigThreads) {
                float4 v[kAhead];
                int at[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int e = e0 + u * kCigThreads;
                    const int b = e / n4, k = e - b * n4;
                    at[u] = e < total ? b * rl + lead + 4 * k : -1;
                    if (e < total) v[u] = *reinterpret_cast<const float4*>(src + b * bin_stride + 4 * k);
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (at[u] >= 0) *reinterpret_cast<float4*>(sRow + at[u]) = v[u];
            }
        } else {
            for (int e = tid; e < n_bins * nz; e += kCigThreads) {
                const int b = e / nz, k = e - b * nz;
                sRow[b * rl + lead + k] = src[b * bin_stride + k];
            }
        }
        const int pad = rl - nz;  // the zeros around the column
        for (int e = tid; e < n_bins * pad; e += kCigThreads) {
            const int b = e / pad, k = e - b * pad;
            sRow[b * rl + (k < lead ? k : nz + k)] = 0.0f;
        }
        __syncthreads();
        for (int z = tid; z < nz; z += kCigThreads) {
            double s = 0.0;
            for (int b = 0; b < n_bins; ++b) s += static_cast<double>(sRow[b * rl + lead + z]);
            sS[z] = s;
            if (stack) stack[col * nz + z] = static_cast<float>(s);
        }
        __syncthreads();
        // (items beyond the workgroup's threads only where zs = 1: their sums go to sC)
        for (int it0 = 0; it0 < items; it0 += kCigThreads) {
            const int it = it0 + tid;
            const bool has = it < items;
            // bins vary fastest over the lanes: different rows, one stack value per part
            const int b = it % n_bins, rest = it / n_bins;
            const int blk = rest % nblk, part = rest / nblk;
            const int lag0 = -L + blk * LB;
            double cc[LB];
            if (has) {
                const int za = z_lo + part * zlen, zb = min(z_hi, za + zlen);
                lag_block<LB>(sS, sRow + b * rl + lead, lag0, za, zb, cc);
            }
            if (zs > 1) __syncthreads();  // every row has been read
            if (has) {
                double* out = (zs > 1 ? sP + static_cast<int64_t>(part) * n_bins * nl : sC) + b * nl + lag0 + L;
#pragma unroll
                for (int j = 0; j < LB; ++j)
                    if (lag0 + j <= L) out[j] = cc[j];
            }
        }
        __syncthreads();
        if (zs > 1) {
            for (int w = tid; w < n_bins * nl; w += kCigThreads) {
                double c = 0.0;
                for (int part = 0; part < zs; ++part) c += sP[static_cast<int64_t>(part) * n_bins * nl + w];
                sC[w] = c;
            }
            __syncthreads();
        }
        // best lag per bin, 16 lanes each: the largest C, ties to the smaller |lag|,
        // then the negative one (rank 0, 1, 2, ... = lag 0, -1, 1, -2, 2, ...)
        for (int b0 = 0; b0 < n_bins; b0 += kCigThreads / kGroup) {
            const int b = b0 + tid / kGroup;
            const double* c = sC + static_cast<int64_t>(min(b, n_bins - 1)) * nl + L;  // c[lag]
            auto lag_of = [](int r) { return (r & 1) ? -((r + 1) >> 1) : (r >> 1); };
            int rank = INT_MAX;
            double top = -__builtin_inf();
            for (int r = tid % kGroup; r < nl; r += kGroup) {
                const double v = c[lag_of(r)];
                if (v > top || (v == top && r < rank)) {
                    top = v;
                    rank = r;
                }
            }
            better_lag<8>(top, rank);
            better_lag<4>(top, rank);
            better_lag<2>(top, rank);
            better_lag<1>(top, rank);
            if (!(c[0] == c[0]) || rank == INT_MAX) {  // nothing compares with a NaN at lag 0
                top = c[0];
                rank = 0;
            }
            if (b < n_bins && tid % kGroup == 0) {
                const int best = lag_of(rank);
                double sh = best;
                if (best > -L && best < L) {
                    const double cm = c[best - 1], c0 = c[best], cp = c[best + 1];
                    const double den = cm - 2.0 * c0 + cp;
                    if (den < 0.0) sh = best + 0.5 * (cm - cp) / den;
                }
                sShift[b] = sh;
                sPeak[b] = top;
                shift[b * ncol + col] = static_cast<float>(sh);
                if (peak) peak[b * ncol + col] = static_cast<float>(top);
            }
        }
        __syncthreads();
        if (curvature && tid < kLanes) {  // one wavefront, lanes over the bins
            double n = 0.0, mq = 0.0, ms = 0.0;
            for (int b = tid; b < n_bins; b += kLanes) {
                if (sPeak[b] > 0.0) {
                    const double h = offsets[b];
                    mq += h * h;
                    ms += sShift[b];
                    n += 1.0;
                }
            }
            n = wave_sum_d(n);
            mq = wave_sum_d(mq);
            ms = wave_sum_d(ms);
            double g = 0.0;
            if (n >= 2.0) {
                mq /= n;
                ms /= n;
                double num = 0.0, den = 0.0;
                for (int b = tid; b < n_bins; b += kLanes) {
                    if (sPeak[b] > 0.0) {
                        const double h = offsets[b];
                        const double dq = h * h - mq;
                        num += dq * (sShift[b] - ms);
                        den += dq * dq;
                    }
                }
                num = wave_sum_d(num);
                den = wave_sum_d(den);
                if (den > 0.0) g = num / den;
            }
            if (tid == 0) curvature[col] = static_cast<float>(g);
        }
    }
}

size_t cig_lds_bytes(int n_bins, int nz, int max_lag) {
    return cig_shape_bytes(cig_choose(n_bins, nz, max_lag), n_bins, nz, max_lag);
}

hipError_t launch_stack(const float* img, int n_bins, int64_t n_points, float* out, hipStream_t s) {
    const int vec = (n_points % 4 == 0) && (reinterpret_cast<uintptr_t>(img) % 16 == 0) &&
                    (reinterpret_cast<uintptr_t>(out) % 16 == 0);
    const int64_t work = vec ? n_points / 4 : n_points;
    const int64_t blocks = std::min<int64_t>((work + 255) / 256, 256 * 64);
    hipLaunchKernelGGL(stack_kernel, dim3(static_cast<unsigned>(std::max<int64_t>(blocks, 1))), dim3(256), 0, s,
                       img, n_bins, n_points, vec, out);
    return hipGetLastError();
}

hipError_t launch_cig(const float* img, int n_bins, int ny, int nx, int nz, int max_lag, int z_lo, int z_hi,
                      const float* offsets, float* stack, float* shift, float* peak, float* curvature,
                      hipStream_t s) {
    const int64_t ncol = static_cast<int64_t>(ny) * nx;
    const int64_t blocks = std::min<int64_t>(ncol, 1 << 20);
    const CigShape c = cig_choose(n_bins, nz, max_lag);
    const int vec = nz % 4 == 0 && reinterpret_cast<uintptr_t>(img) % 16 == 0;
    auto kernel = c.lb == 13 ? cig_kernel<13>
                  : c.lb == 11 ? cig_kernel<11>
                  : c.lb == 9  ? cig_kernel<9>
                  : c.lb == 7  ? cig_kernel<7>
                               : cig_kernel<5>;
    return launch_with_lds(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kCigThreads),
                           cig_shape_bytes(c, n_bins, nz, max_lag), s, img, n_bins, ny, nx, nz, max_lag, z_lo, z_hi,
                           c, vec, offsets, stack, shift, peak, curvature);
}

}  // namespace km
