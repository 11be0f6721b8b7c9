// Migration kernel: Eq. (1) as an image-stationary gather.
//
// Workgroup = (offset bin b, column tile, depth chunk).  Each wavefront keeps
// CWQ groups of 4 image columns x (16 * KS) depths of float32 accumulators
// in registers; the traces of bin b stream through LDS in blocks.  The traces
// near the tile are listed first, a thread per trace; a listed trace enters a
// block only if it can have a pair inside the aperture of the tile and chunk,
// and only the time window its pairs can read is staged (the double-square-root
// time grows with the squared leg lengths, so the window follows from the
// tile's bounding box and the chunk's tables).  For every column group the
// wavefront computes the two squared leg lengths of 16 traces at once (lane =
// (column, trace)), hands them to the depth lanes through the LDS crossbar,
// derives from ballots which 16-depth slots can hold a pair inside the aperture
// and which are wholly inside, and evaluates those slots two at a time.  The
// source leg's share of a pair is kept from trace to trace while the source
// stays the same (SrcLeg), unless the traces seldom share it (own_legs); the
// receiver's costs one square root, the weight one reciprocal, then the sample
// index and fraction, one 8-byte LDS read of the staged (sample, difference)
// pair, the interpolation and, at the aperture's edge, the lane's mask.  Table times and the anti-alias filter use the same
// blocks with their own staged forms (plain samples; float64 double running
// sums, one slot at a time).  With 16-bit traces the S16 kernels keep the
// samples' 16-bit storage in LDS instead (packed pairs; single samples for table
// times) and widen them on read.
//
// What bounds it: VALU issue (200 000 traces over 16 x 256 x 256 x 400 points:
// 19.4 lane-slots per pair inside the aperture, 2.6 of them transcendentals of 2.3
// issue slots each, together 89 % of the slots; waits for LDS 0.5 % of the
// wavefronts' cycles).  394 -> 318 ms over 16 x 128 x 128 x 400 points from keeping source legs, testing the aperture
// only at its edge (13 instead of 15 VALU instructions per pair and lane),
// reading a trace's row and clamp bounds by one broadcast, and staging 4
// samples per lane; evaluating single slots where only one of a pair is inside
// ran 396 ms (fewer instructions, less overlap).  On small images the wavefronts
// are too few: see the tiles at the end of the file.
#include <utility>

#include "km_kernels.h"

namespace km {

// Sample k of trace j: zero outside [0, nt), times the per-trace scale for
// 16-bit storage.
__device__ __forceinline__ float trace_sample(const Params& P, int64_t j, int k, float sc) {
    if (k < 0 || k >= P.nt) return 0.0f;
    if (P.dtype == F32) return static_cast<const float*>(P.data)[j * P.stride + k];
    return widen16(static_cast<const uint16_t*>(P.data)[j * P.stride + k], P.dtype) * sc;
}

// Stage the window of samples lo .. lo + len - 1 of trace j as len floats
// (the whole-record windows of table traveltimes).  One wavefront.
__device__ __forceinline__ void stage_window_f(const Params& P, int64_t j, int lo, int len, float* dst, int lane) {
    const float sc = (P.dtype != F32 && P.scale) ? P.scale[j] : 1.0f;
    for (int e0 = 0; e0 < len; e0 += 4 * kLanes) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kLanes + lane;
            v[u] = e < len ? trace_sample(P, j, lo + e, sc) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kLanes + lane;
            if (e < len) dst[e] = v[u];
        }
    }
}

// 16-bit storage bits of sample k of trace row src (zero bits, +0, outside the record).
__device__ __forceinline__ uint32_t sample_bits16(const Params& P, const uint16_t* src, int k) {
    return (k >= 0 && k < P.nt) ? static_cast<uint32_t>(src[k]) : 0u;
}

// Stage the window of samples lo .. lo + len - 1 of trace j as len - 1 packed
// pairs dst[e] = bits(D[lo + e]) | bits(D[lo + e + 1]) << 16 of the 16-bit
// storage (half the LDS of float (sample, difference) pairs); the reads widen
// them and apply the trace's scale.  One wavefront.
__device__ __forceinline__ void stage_window_16p(const Params& P, int64_t j, int lo, int len, uint32_t* dst, int lane) {
    const uint16_t* src = static_cast<const uint16_t*>(P.data) + j * P.stride;
    for (int e0 = 0; e0 < len - 1; e0 += 2 * kLanes) {
        uint32_t a[2], b[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = e0 + u * kLanes + lane;
            a[u] = 0u;
            b[u] = 0u;
            if (e < len - 1) {
                a[u] = sample_bits16(P, src, lo + e);
                b[u] = sample_bits16(P, src, lo + e + 1);
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = e0 + u * kLanes + lane;
            if (e < len - 1) dst[e] = a[u] | (b[u] << 16);
        }
    }
}

// Stage the window of samples lo .. lo + len - 1 of trace j as len 16-bit
// storage values (half the LDS of float samples: the whole-record windows of
// table traveltimes).  One wavefront.
__device__ __forceinline__ void stage_window_16(const Params& P, int64_t j, int lo, int len, uint16_t* dst, int lane) {
    const uint16_t* src = static_cast<const uint16_t*>(P.data) + j * P.stride;
    for (int e0 = 0; e0 < len; e0 += 4 * kLanes) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kLanes + lane;
            v[u] = e < len ? sample_bits16(P, src, lo + e) : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kLanes + lane;
            if (e < len) dst[e] = static_cast<uint16_t>(v[u]);
        }
    }
}

// The two samples of a packed pair (low half: the first), widened.
template <int DT>
__device__ __forceinline__ void widen_pair(uint32_t w, float& a, float& b) {
    if (DT == BF16) {
        a = __uint_as_float(w << 16);
        b = __uint_as_float(w & 0xffff0000u);
    } else {
        a = widen16(w & 0xffffu, DT);
        b = widen16(w >> 16, DT);
    }
}

// Samples k and k + 1 of a window staged by stage_window_16, k counted in
// 16-bit values from s: the two aligned words that hold them, funnel-shifted
// (for even k the second word is not used; it is still inside the
// workgroup's LDS, as the trace block's slot records follow the windows).
__device__ __forceinline__ uint32_t read_pair16(const uint32_t* s, int k) {
    const uint32_t w0 = s[k >> 1], w1 = s[(k >> 1) + 1];
    return __builtin_amdgcn_alignbit(w1, w0, static_cast<uint32_t>(k & 1) << 4);
}

// Four consecutive samples of a row that may start at any sample.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t ushort4_any __attribute__((ext_vector_type(4), aligned(2)));

// The value of the next lane (lane 63: 0).
__device__ __forceinline__ float next_lane(float v) { return dpp_f<0x130>(v); }

// Samples e .. e + 3 of a window of len samples from sample lo of trace j, the
// lane's share of a staging step (zero past the record's ends).
__device__ __forceinline__ void load_quad(const Params& P, int64_t j, int lo, int len, int e, float* v) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = 0.0f;
    if (e >= len) return;
    const float sc = (P.dtype != F32 && P.scale) ? P.scale[j] : 1.0f;
    if (lo < 0 || lo + ((len - 1) & ~3) + 4 > P.nt) {  // some lane's 4 samples leave the record: checked loads
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = trace_sample(P, j, lo + e + u, sc);
    } else if (P.dtype == F32) {
        const float4_any w =
            *reinterpret_cast<const float4_any*>(static_cast<const float*>(P.data) + j * P.stride + lo + e);
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = w[u];
    } else {
        const ushort4_any w =
            *reinterpret_cast<const ushort4_any*>(static_cast<const uint16_t*>(P.data) + j * P.stride + lo + e);
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = widen16(w[u], P.dtype) * sc;
    }
}

// Write the pairs e .. e + 3 of a window (lane 63 only hands its first sample down).
__device__ __forceinline__ void store_quad(const float* v, int len, int e, float2* dst, int lane) {
    const float nx = next_lane(v[0]);
    if (e < len - 1 && lane < kLanes - 1) {
        float4* o = reinterpret_cast<float4*>(dst + e);
        o[0] = make_float4(v[0], v[1] - v[0], v[1], v[2] - v[1]);
        o[1] = make_float4(v[2], v[3] - v[2], v[3], nx - v[3]);
    }
}

// Stage, for positions lo .. lo + len - 1 of trace j, the double running sum
// I2[n] = sum_{m <= n} sum_{k <= m} D[k] (float64, from position lo; D zero
// outside [0, nt)): the anti-alias triangles are second differences of it.
// One wavefront, 4 positions per lane: with s the lane's samples' sum and P the
// sum before the lane, I1 runs P + v0, P + v0 + v1, ... and adds 4 P + 4 v0 + 3
// v1 + 2 v2 + v3 to I2, so two scans over the lanes serve 256 positions.  Bound
// by the scans' chain of additions: with one position per lane, two scans for 64,
// an anti-aliased 50 x 48 x 256 x 8 image of 10 000 traces ran 25.0 ms, now 14.1
// ms.  dst is 16-byte aligned with room for len rounded up to 4.
__device__ __forceinline__ void stage_window_i2(const Params& P, int64_t j, int lo, int len, double* dst, int lane) {
    double c1 = 0.0, c2 = 0.0;  // I1 and I2 at the position before the step
    for (int e0 = 0; e0 < len; e0 += 4 * kLanes) {
        const int e = e0 + 4 * lane;
        float v[4];
        load_quad(P, j, lo, len, e, v);
        const double d0 = v[0], d1 = v[1], d2 = v[2], d3 = v[3];
        const double t1 = d0 + d1, t2 = t1 + d2, t3 = t2 + d3;  // running sums within the lane
        const double s1 = wave_scan_d(t3);
        const double p1 = c1 + prev_lane_d(s1);  // I1 before the lane
        const double u1 = t1 + d0, u2 = u1 + t2, u3 = u2 + t3;  // their running sums
        const double s2 = wave_scan_d(fma(4.0, p1, u3));
        const double p2 = c2 + prev_lane_d(s2);  // I2 before the lane
        if (e < len) {
            double2* o = reinterpret_cast<double2*>(dst + e);
            o[0] = make_double2(p2 + (p1 + d0), p2 + fma(2.0, p1, u1));
            o[1] = make_double2(p2 + fma(3.0, p1, u2), p2 + fma(4.0, p1, u3));
        }
        c1 += last_lane_d(s1);
        c2 += last_lane_d(s2);
    }
}

// Stage the windows of the block's slots first, first + step, ... as pairs
// dst[e] = (D[lo + e], D[lo + e + 1] - D[lo + e]): the interpolation then reads
// one pair and needs one FMA.  One wavefront; a window is 16-byte aligned and
// has room for its pair count rounded up to a multiple of 4.  A lane takes 4
// consecutive samples (one load, two stores), and the loads of four traces are
// in flight together.  With one sample per lane, checked and addressed one by
// one, staging was a tenth of the VALU work of the survey's migration.
__device__ __forceinline__ void stage_pairs(const Params& P, int64_t lo, const int4* sMeta, float* sTr, int nb,
                                            int first, int step, int lane) {
    constexpr int kAhead = 4;
    for (int t0 = first; t0 < nb; t0 += kAhead * step) {
        float v[kAhead][4];
        int4 mt[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int t = t0 + u * step;
            mt[u] = sMeta[min(t, nb - 1)];
            // past the last slot: an empty window
            if (t >= nb) mt[u].z = mt[u].y - 1;
            load_quad(P, lo + mt[u].w, mt[u].y, mt[u].z - mt[u].y + 1, 4 * lane, v[u]);
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int len = mt[u].z - mt[u].y + 1;
            float2* dst = reinterpret_cast<float2*>(sTr + mt[u].x);
            store_quad(v[u], len, 4 * lane, dst, lane);
            for (int e0 = 4 * (kLanes - 1); e0 < len - 1; e0 += 4 * (kLanes - 1)) {  // windows of more than 252 pairs
                float w[4];
                load_quad(P, lo + mt[u].w, mt[u].y, len, e0 + 4 * lane, w);
                store_quad(w, len, e0 + 4 * lane, dst, lane);
            }
        }
    }
}

// What a pair needs of its source leg, per depth slot of one column group.
// The traces of a bin come in shot order (the order every generator and most
// acquisitions give), so consecutive traces of a block often share their
// source: the source leg's share of a pair is evaluated when the source
// changes and kept in registers until it changes again.  Each value is formed
// by the operations the pair evaluation would use, so a pair has the same bits
// whether its source leg was kept or not.
//   square root        a = A + B h^2 and sqrt(a)
//   anti-alias         sqrt(a) and its reciprocal
//   extended           the leg time (float64) and the reciprocal square root seed
//   tables             base and increment of the leg time, amplitude
//   tables, extended   the leg time (float64), amplitude
template <int KS, int TT, bool PX>
struct SrcLeg {
    float a[KS], s[KS];
};
template <int KS>
struct SrcLeg<KS, TT_DSR, true> {
    double t[KS];
    float q[KS];
};
template <int KS>
struct SrcLeg<KS, TT_TABLE, false> {
    float base[KS], inc[KS], amp[KS];
};
template <int KS>
struct SrcLeg<KS, TT_LTABLE, false> : SrcLeg<KS, TT_TABLE, false> {};
template <int KS>
struct SrcLeg<KS, TT_TABLE, true> {
    double t[KS];
    float amp[KS];
};
template <int KS>
struct SrcLeg<KS, TT_LTABLE, true> : SrcLeg<KS, TT_TABLE, true> {};

// Two slots of one (column group, trace) pairing with square-root times.
// (sa, ss): the source leg of each slot; hr2: the receiver leg.
template <bool TF, int WK>
__device__ __forceinline__ void mig_pair(float A0, float B0, float A1, float B1, float sa0, float ss0, float sa1,
                                         float ss1, float hr2, const float2* row, float tfo, float wlo, float whi,
                                         float& v0, float& v1, float& r0, float& r1) {
    const float ar0 = fmaf(B0, hr2, A0), ar1 = fmaf(B1, hr2, A1);
    float w0 = ss0 + __builtin_amdgcn_sqrtf(ar0);
    float w1 = ss1 + __builtin_amdgcn_sqrtf(ar1);
    if (TF) {
        w0 = w0 + tfo;
        w1 = w1 + tfo;
    }
    w0 = __builtin_amdgcn_fmed3f(w0, wlo, whi);
    w1 = __builtin_amdgcn_fmed3f(w1, wlo, whi);
    const float2 e0 = row[static_cast<int32_t>(w0)];
    const float2 e1 = row[static_cast<int32_t>(w1)];
    r0 = (WK == W_COSCOS) ? __builtin_amdgcn_rcpf(sa0 * ar0) : 1.0f;
    r1 = (WK == W_COSCOS) ? __builtin_amdgcn_rcpf(sa1 * ar1) : 1.0f;
    v0 = fmaf(__builtin_amdgcn_fractf(w0), e0.y, e0.x);
    v1 = fmaf(__builtin_amdgcn_fractf(w1), e1.y, e1.x);
}

// mig_pair on a window staged as packed 16-bit pairs (stage_window_16p): the
// pair is widened and interpolated, and the trace's scale joins the weight.
template <bool TF, int WK, int DT>
__device__ __forceinline__ void mig_pair16(float A0, float B0, float A1, float B1, float sa0, float ss0, float sa1,
                                           float ss1, float hr2, const uint32_t* row, float scl, float tfo, float wlo,
                                           float whi, float& v0, float& v1, float& r0, float& r1) {
    const float ar0 = fmaf(B0, hr2, A0), ar1 = fmaf(B1, hr2, A1);
    float w0 = ss0 + __builtin_amdgcn_sqrtf(ar0);
    float w1 = ss1 + __builtin_amdgcn_sqrtf(ar1);
    if (TF) {
        w0 = w0 + tfo;
        w1 = w1 + tfo;
    }
    w0 = __builtin_amdgcn_fmed3f(w0, wlo, whi);
    w1 = __builtin_amdgcn_fmed3f(w1, wlo, whi);
    float a0, b0, a1, b1;
    widen_pair<DT>(row[static_cast<int32_t>(w0)], a0, b0);
    widen_pair<DT>(row[static_cast<int32_t>(w1)], a1, b1);
    r0 = (WK == W_COSCOS) ? __builtin_amdgcn_rcpf(sa0 * ar0) * scl : scl;
    r1 = (WK == W_COSCOS) ? __builtin_amdgcn_rcpf(sa1 * ar1) * scl : scl;
    v0 = fmaf(__builtin_amdgcn_fractf(w0), b0 - a0, a0);
    v1 = fmaf(__builtin_amdgcn_fractf(w1), b1 - a1, a1);
}

// Accumulate the values of slots k and k + 1.  Only where the slots are not
// wholly inside the aperture (full: wavefront-uniform) is a lane's value
// tested against its aperture (hm <= R) and dropped outside it.  Invalid lanes
// of a full slot add a finite value that is never stored.
template <int WK, int KS, bool RREG>
__device__ __forceinline__ void mask_add2(const ChunkTables<KS>& T, const float* sR, uint32_t full, int k, int d,
                                          float hm, float v0, float v1, float r0, float r1, float& acc0,
                                          float& acc1) {
    if (((full >> k) & 3u) != 3u) {
        // a branch, not two selects per slot; the weights are formed before it
        asm volatile("" : "+v"(r0), "+v"(r1));
        const float R0 = RREG ? T.R[k] : sR[k * kGroup + d];
        const float R1 = RREG ? T.R[k + 1] : sR[(k + 1) * kGroup + d];
        v0 = (hm <= R0) ? v0 : 0.0f;
        v1 = (hm <= R1) ? v1 : 0.0f;
    }
    acc0 = (WK == W_COSCOS) ? fmaf(v0, r0, acc0) : acc0 + v0;
    acc1 = (WK == W_COSCOS) ? fmaf(v1, r1, acc1) : acc1 + v1;
}

// One slot with the extended-precision time: (ts, qs) the source leg's time
// and seed, Hr the receiver's squared length, the clamp as integer bounds [ilo, ihi] (or float64 [wlo, whi] with
// t_first).  One slot at a time: the float64 temporaries of two slots in
// flight would cost more registers than the latency they hide.
template <bool TF, int WK>
__device__ __forceinline__ void mig_slot_ext(float A, float B, double ts, float qs, double Hr, float hm,
                                             const float2* row, double inv_dt, double tfo, int ilo, int ihi,
                                             double wlo, double whi, float R, float& acc) {
    // keep the tables' float64 conversions inside the loop (hoisted, they
    // would hold two more registers per slot)
    asm volatile("" : "+v"(A), "+v"(B));
    const LegTimeX r = leg_time_ext(A, B, Hr);
    double w = (ts + r.t) * inv_dt;
    int i;
    if (TF) {
        w = fmin(fmax(w + tfo, wlo), whi);
        i = static_cast<int32_t>(w);
    } else {
        i = min(max(static_cast<int32_t>(w), ilo), ihi);
    }
    const float2 e = row[i];
    float v = fmaf(static_cast<float>(__builtin_amdgcn_fract(w)), e.y, e.x);
    v = (hm <= R) ? v : 0.0f;
    const float g = qs * r.q;
    acc = (WK == W_COSCOS) ? fmaf(v, g * g, acc) : acc + v;
}

// The smoothed value of a pair with the anti-alias triangle filter.  row[n] = I2 at window
// position n (staged by stage_window_i2): the smoothed sample at c is
// alpha T_L(c) + beta T_{L+1}(c), T_L(c) = I2[c+L-1] - 2 I2[c-1] + I2[c-L-1],
// read as five (n, n + 1) pairs for c = i and c = i + 1.
template <bool TF, int WK>
__device__ __forceinline__ float aa_value(const PairAA& p, const double* row) {
    const int i = p.i, L = p.L;
    const double a1 = row[i + L - 1], b1 = row[i + L];
    const double a2 = row[i - 1], b2 = row[i];
    const double a3 = row[i - L - 1], b3 = row[i - L];
    const double b4 = row[i + L + 1];
    const double a5 = row[i - L - 2];
    // a4 = b1, b5 = a3
    const double tl0 = fma(-2.0, a2, a1 + a3), tl1 = fma(-2.0, b2, b1 + b3);   // T_L(i), T_L(i + 1)
    const double tm0 = fma(-2.0, a2, b1 + a5), tm1 = fma(-2.0, b2, b4 + a3);   // T_{L+1}(i), T_{L+1}(i + 1)
    const double al = p.alpha, be = p.beta;
    const double v0 = fma(be, tm0, al * tl0), v1 = fma(be, tm1, al * tl1);
    return static_cast<float>(fma(static_cast<double>(p.f), v1 - v0, v0));
}

// One slot at a time (two in flight need more registers than the eight
// float64 reads leave).  (ss, is): square root of the source leg and its
// reciprocal.
template <bool TF, int WK>
__device__ __forceinline__ void mig_slot_aa(float A, float B, float ss, float is, float hr2, float hm,
                                            const double* row, float tfo, float wlo, float whi, float R, float dxs,
                                            float dys, float dxr, float dyr, float adx, float ady, float lmax,
                                            const float* invsq, float& acc) {
    const PairAA p = pair_aa<TF, WK>(A, B, ss, is, hr2, tfo, wlo, whi, dxs, dys, dxr, dyr, adx, ady, lmax, invsq);
    float v = aa_value<TF, WK>(p, row);
    v = (hm <= R) ? v : 0.0f;
    acc = (WK == W_COSCOS) ? fmaf(v, p.r, acc) : acc + v;
}

// The source legs of every slot from the leg's squared length (float32 and,
// for the extended kernels, float64).  vd, vl: byte offset of the lane's depth in
// slot 0 of a table row, and how far it is to the row's last depth.  Table slot pairs
// that no lane of the wavefront can use are not read (a pair is evaluated whole, so
// both its slots are filled).
template <int KS, int WK, int TT, bool PX>
__device__ __forceinline__ void source_leg(const Params& P, const ChunkTables<KS>& T, float hs2, double Hs, LCol C,
                                           int vd, int vl, SrcLeg<KS, TT, PX>& S) {
    if constexpr (is_table(TT)) {
        constexpr bool LAT = TT == TT_LTABLE;
        const float hmin = uniform_f(rows_min(hs2));
        const uint64_t any = __builtin_amdgcn_ballot_w64(hmin <= T.rhi);
        if constexpr (PX) {
            const TLegX L = table_leg_ext(P, Hs);
            const int vb = 4 * ((LAT ? C.off : 0) + L.off) + vd;
#pragma unroll
            for (int k = 0; k < KS; ++k)
                if ((any >> (k & ~1)) & 3ull) {
                    S.t[k] = LAT ? ltable_time_ext_at(P, L.f, C, vb + min(64 * k, vl)) : table_time_ext_at(P, L.f, vb + min(64 * k, vl));
                    if (P.tamp) S.amp[k] = table_amp_at<LAT>(P, static_cast<float>(L.f), C, vb + min(64 * k, vl));
                }
        } else {
            const TLeg L = table_leg(P, hs2);
            const int vb = 4 * ((LAT ? C.off : 0) + L.off) + vd;
#pragma unroll
            for (int k = 0; k < KS; ++k)
                if ((any >> (k & ~1)) & 3ull) {
                    const TTime t = LAT ? ltable_time_at(P, L.f, C, vb + min(64 * k, vl)) : table_time_at(P, L.f, vb + min(64 * k, vl));
                    S.base[k] = t.base;
                    S.inc[k] = t.inc;
                    if (P.tamp) S.amp[k] = table_amp_at<LAT>(P, L.f, C, vb + min(64 * k, vl));
                }
        }
    } else if constexpr (PX) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const LegTimeX l = leg_time_ext(T.A[k], T.B[k], Hs);
            S.t[k] = l.t;
            S.q[k] = l.q;
        }
    } else {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const float a = fmaf(T.B[k], hs2, T.A[k]);
            const float r = __builtin_amdgcn_sqrtf(a);
            S.a[k] = TT == TT_AA ? r : a;
            S.s[k] = TT == TT_AA ? __builtin_amdgcn_rcpf(r) : r;
        }
    }
}

// A pair with table times, the source leg's share kept: time and (with
// amplitude tables) weight at the table byte offset vb of the receiver leg.
template <bool TF, bool LAT>
__device__ __forceinline__ Pair pair_table(const Params& P, TTime ts, float as, float fr, int vb, float wlo, float whi,
                                           LCol C) {
    double w = pair_time(P, ts, LAT ? ltable_time_at(P, fr, C, vb) : table_time_at(P, fr, vb));
    if (TF) w = w + P.tf_off_d;
    w = fmin(fmax(w, static_cast<double>(wlo)), static_cast<double>(whi));
    Pair p;
    p.i = static_cast<int32_t>(w);
    p.f = static_cast<float>(w - static_cast<double>(p.i));
    p.r = 1.0f;
    if (P.tamp) p.r = as * table_amp_at<LAT>(P, fr, C, vb);
    return p;
}

template <bool TF, bool LAT>
__device__ __forceinline__ Pair pair_table_ext(const Params& P, double ts, float as, double fr, int vb, float wlo,
                                               float whi, LCol C) {
    double w = (ts + (LAT ? ltable_time_ext_at(P, fr, C, vb) : table_time_ext_at(P, fr, vb))) * P.inv_dt;
    if (TF) w = w + P.tf_off_d;
    w = fmin(fmax(w, static_cast<double>(wlo)), static_cast<double>(whi));
    Pair p;
    p.i = static_cast<int32_t>(w);
    p.f = static_cast<float>(w - static_cast<double>(p.i));
    p.r = 1.0f;
    if (P.tamp) p.r = as * table_amp_at<LAT>(P, static_cast<float>(fr), C, vb);
    return p;
}

// Kernels that have a second form, for traces whose sources do not repeat (OWN): there
// a kept leg costs more than it saves, as it is formed for every slot, its reads are
// waited for before the receiver's are asked for, and it holds registers.  ms, random
// trace order, kept / own legs / before legs were kept (square-root times, extended
// ones, tables): 10 000 traces -> 16 x 103 x 97 x 107 1.84 / 1.62 / 1.78, 2.89 / 2.28
// / 2.47, 3.74 / 3.07 / 3.05; 36 864 -> 10 x 90 x 80 x 300 25.9 / 22.4 / 28.3, 46.9 /
// 40.4 / 48.7, 52.7 / 43.3 / 50.6.  Not for the extended tables and the anti-alias
// filter, nor for shapes with trace parts, which gain little (59 against 57 us on
// 1536 traces) and whose short calls would wait for the sample (58.1 -> 59.8 us).
constexpr bool own_legs(int tt, bool px, int ts) { return ts == 1 && (tt == TT_DSR || (is_table(tt) && !px)); }

// Whether at least half of the traces have the source of the trace before them, from
// 64 places among them (one wavefront; the same answer in all): the reads, made ahead
// of the bin's, and the answer.
struct SourceSample {
    float x0, y0, x1, y1;
    bool has;
};
__device__ __forceinline__ SourceSample sample_sources(const Params& P) {
    const int64_t j = P.n_traces * (threadIdx.x & (kLanes - 1)) / kLanes;
    SourceSample s{0.0f, 0.0f, 0.0f, 0.0f, j + 1 < P.n_traces};
    if (s.has) {
        s.x0 = P.src[2 * j];
        s.y0 = P.src[2 * j + 1];
        s.x1 = P.src[2 * j + 2];
        s.y1 = P.src[2 * j + 3];
    }
    return s;
}
__device__ __forceinline__ bool sources_repeat(const SourceSample& s) {
    const uint64_t same = __builtin_amdgcn_ballot_w64(s.has && s.x0 == s.x1 && s.y0 == s.y1);
    return 2 * __builtin_popcountll(same) >= __builtin_popcountll(__builtin_amdgcn_ballot_w64(s.has));
}

// RREG: the masked slots take the lanes' aperture values from registers
// (else from the LDS copy, which costs fewer registers).
// TT: traveltime kind (TT_TABLE: one-way time table, W = 1; TT_LTABLE: one
// table per node of a lateral grid, W = 1).
// PX: extended-precision times (eval_pair_ext, table_leg_ext); the squared
// leg lengths then also reach the depth lanes in float64.
//
// LDS (lds_bytes): window storage [P.cap floats; a window of n samples takes
// n - 1 pairs, rounded up to whole quads], per block slot the trace geometry (float4) and (float offset,
// first sample, last sample, trace - bin start) (int4) and (row offset, clamp
// bounds, scale) (float4) [P.tb each], the aperture values [KS * 16], the tile box
// [4 per wavefront], the candidates of two passes [2 x NW * 4], the
// per-wavefront counts [2 x 16] and the list of near traces [P.list_cap].
// [lo, hi): the traces of bin b.  OWN: no source leg is kept, every pair forms both.
template <int NW, int CWQ, int KS, int TS, bool TF, int WK, bool RREG, int TT = TT_DSR, bool PX = false, int S16 = 0,
          bool OWN = false>
__device__ __forceinline__ void migrate_tile(const Params& P, int64_t lo, int64_t hi, int b, int tile, int zc,
                                             float* lds) {
    static_assert(!OWN || own_legs(TT, PX, TS), "no such form");
    static_assert(!(PX && TT == TT_AA), "no extended-precision anti-alias kernels");
    // S16: the 16-bit storage type (BF16 or F16) staged as it is, 0 for float staging
    static_assert(!(S16 && (PX || TT == TT_AA)), "16-bit staging: float32 time, no anti-alias filter");
    static_assert(KS % 2 == 0, "slots are evaluated in pairs");
    constexpr int NG = NW * kGroupsPerWave;  // candidate traces per pass: one per 16-lane group
    static_assert(NG <= kLanes && NW <= kBoxFloats / 4, "at most 16 wavefronts");
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    // column wavefront and trace part of this wavefront
    constexpr int NC = NW / TS;
    const int cw = wave % NC, part = wave / NC;
    const int g = lane / kGroup, d = lane % kGroup;
    const int ncol = P.nx * P.ny;
    const int z0 = zc * P.zspan;
    const int z1 = min(z0 + P.zspan, P.nz);  // end of the chunk's depths
    const int nt = P.nt;
    // staged-row index of sample k is k + koff (the time includes kLead with t_first)
    const int koff = TF ? kLead : 0;
    // staged form: (sample, difference) pairs for the square-root times (windows
    // of a few hundred samples), plain samples for the whole-record windows of
    // table times (half the LDS per trace), float64 double running sums with
    // the anti-alias filter
    constexpr bool PAIRS = TT == TT_DSR && !S16;
    constexpr bool AA = TT == TT_AA;
    constexpr bool P16 = TT == TT_DSR && S16;  // packed 16-bit pairs
    constexpr bool T16 = is_table(TT) && S16;  // 16-bit samples
    // anti-aliasing: largest half-width, and the reach of a pair's reads around
    // its sample (L + 2 below, L + 2 above counting the pair's second sample)
    const int lmax = AA ? P.aa_max : 0;

    float* sTr = lds;                                                    // [cap]
    float4* sGeo = reinterpret_cast<float4*>(lds + P.cap);               // [tb]
    int4* sMeta = reinterpret_cast<int4*>(lds + P.cap + 4 * P.tb);       // [tb]
    float4* sBnd = reinterpret_cast<float4*>(lds + P.cap + 8 * P.tb);    // [tb]
    float* sR = lds + P.cap + 12 * P.tb;                                 // [KS * 16]
    float* sBox = sR + KS * kGroup;                                      // [kBoxFloats]
    uint32_t* sCand = reinterpret_cast<uint32_t*>(sBox + kBoxFloats);    // [2][kCandMax]
    float* sInvSq = sBox + kBoxFloats + 2 * kCandMax;                    // [kAAMaxHalf + 2]: 1 / n^2
    int* sCnt = reinterpret_cast<int*>(sInvSq + kInvSqFloats);           // [2][16]
    int* sList = sCnt + 32;                                              // [list_cap]
    if (AA)
        for (int t = threadIdx.x; t < kAAMaxHalf + 2; t += blockDim.x)
            sInvSq[t] = t > 0 ? 1.0f / static_cast<float>(t * t) : 0.0f;

    ChunkTables<KS> T;
    load_chunk_tables<KS, 1, TT, PX>(P, z0, z1, d, WK == W_COSCOS, T, sR);

    constexpr bool LAT = TT == TT_LTABLE;
    // bytes from the lane's depth in slot 0 to the row's last: a lane past it reads that one.
    // The clamp costs two operations per read (2.64 s for 200 000 traces -> 16 x 256 x 256 x
    // 400 points, 2.54 s without); a second body for the chunks that need none ran 2.59 s
    // there, but 5.34 against 5.12 ms on 25 600 traces -> 8 x 80 x 80 x 152.
    const int vl = 4 * (P.nz - 1 - z0 - d);
    // first column of the wavefront's groups; group q's lane column is col0 + 4 q + g
    const int col0 = (tile * NC + cw) * CWQ * kGroupsPerWave;

    float acc[CWQ][KS];
#pragma unroll
    for (int q = 0; q < CWQ; ++q)
#pragma unroll
        for (int k = 0; k < KS; ++k) acc[q][k] = 0.0f;

    const float tfo = P.tf_off;
    const double tfod = P.tf_off_d;

    // Bounding box of the tile's columns.  A leg longer than sqrt(r2)(1 + 2^-22)
    // from every column cannot pass the float32 aperture test, so a trace whose
    // source or receiver lies farther than that from the box (with a 1e-5
    // margin on the squared radius) has no pair in this tile and depth chunk.
    {
        float bx0 = __builtin_inff(), bx1 = -__builtin_inff(), by0 = __builtin_inff(), by1 = -__builtin_inff();
#pragma unroll
        for (int q = 0; q < CWQ; ++q) {
            const int col = col0 + kGroupsPerWave * q + g;
            if (col < ncol) {
                const float x = P.x[col % P.nx], y = P.y[col / P.nx];
                bx0 = fminf(bx0, x);
                bx1 = fmaxf(bx1, x);
                by0 = fminf(by0, y);
                by1 = fmaxf(by1, y);
            }
        }
        bx0 = wave_min(bx0);
        bx1 = wave_max(bx1);
        by0 = wave_min(by0);
        by1 = wave_max(by1);
        if (lane == 0) {
            sBox[4 * wave] = bx0;
            sBox[4 * wave + 1] = bx1;
            sBox[4 * wave + 2] = by0;
            sBox[4 * wave + 3] = by1;
        }
    }
    __syncthreads();
    float bx0 = sBox[0], bx1 = sBox[1], by0 = sBox[2], by1 = sBox[3];
    for (int w = 1; w < NW; ++w) {
        bx0 = fminf(bx0, sBox[4 * w]);
        bx1 = fmaxf(bx1, sBox[4 * w + 1]);
        by0 = fminf(by0, sBox[4 * w + 2]);
        by1 = fmaxf(by1, sBox[4 * w + 3]);
    }
    // wavefront-uniform: kept in scalar registers
    bx0 = uniform_f(bx0);
    bx1 = uniform_f(bx1);
    by0 = uniform_f(by0);
    by1 = uniform_f(by1);
    const float reach = uniform_f(T.rmax * 1.00001f);

    // Windows need a time that does not decrease with the squared leg length:
    // B >= 0 on every depth that can be inside the aperture (else, and for
    // table times, the whole record is staged).
    bool mono_lane = true;
#pragma unroll
    for (int k = 0; k < KS; ++k) mono_lane = mono_lane && (!(T.R[k] >= 0.0f) || T.B[k] >= 0.0f);
    const bool windows = TT == TT_DSR && __builtin_amdgcn_ballot_w64(!mono_lane) == 0;
    const int first_lo = TF ? -1 : 0;  // lowest staged sample (t_first = 0 gives u >= 0)

    // Table times: the pairs of slots k and k + 1, of the trace whose row offset, bounds and scale are bd.
    auto add_table_pairs = [&](const Pair& p0, const Pair& p1, const float4& bd, uint32_t full, int k, float hm, int q) {
        const int rb = __float_as_int(bd.x);
        const float* row = sTr + rb;
        const uint32_t* sw = reinterpret_cast<const uint32_t*>(sTr);
        float a0, b0, a1, b1;
        if (S16) {
            widen_pair<S16>(read_pair16(sw, rb + p0.i), a0, b0);
            widen_pair<S16>(read_pair16(sw, rb + p1.i), a1, b1);
        } else {
            a0 = row[p0.i], b0 = row[p0.i + 1];
            a1 = row[p1.i], b1 = row[p1.i + 1];
        }
        mask_add2<W_COSCOS, KS, RREG>(T, sR, full, k, d, hm, fmaf(p0.f, b0 - a0, a0), fmaf(p1.f, b1 - a1, a1),
                                      S16 ? p0.r * bd.w : p0.r, S16 ? p1.r * bd.w : p1.r, acc[q][k], acc[q][k + 1]);
    };

    // Square-root times: slots k and k + 1, (a, s) their source legs and roots.
    auto add_root_pairs = [&](float a0, float s0, float a1, float s1, float hr2, const float4& bd, uint32_t full,
                              int k, float hm, int q) {
        const int rb = __float_as_int(bd.x);
        float v0, v1, r0, r1;
        if (S16) {
            mig_pair16<TF, WK, S16>(T.A[k], T.B[k], T.A[k + 1], T.B[k + 1], a0, s0, a1, s1, hr2,
                                    reinterpret_cast<const uint32_t*>(sTr) + rb, bd.w, tfo, bd.y, bd.z, v0, v1, r0, r1);
        } else {
            mig_pair<TF, WK>(T.A[k], T.B[k], T.A[k + 1], T.B[k + 1], a0, s0, a1, s1, hr2,
                             reinterpret_cast<const float2*>(sTr) + rb, tfo, bd.y, bd.z, v0, v1, r0, r1);
        }
        mask_add2<S16 ? W_COSCOS : WK, KS, RREG>(T, sR, full, k, d, hm, v0, v1, r0, r1, acc[q][k], acc[q][k + 1]);
    };
    // Extended square-root times: slot k, (t, s) its source leg's time and seed.
    auto add_ext_slot = [&](double t, float s, double Hr, const float4& bd, int k, float hm, int q) {
        const float R = RREG ? T.R[k] : sR[k * kGroup + d];
        mig_slot_ext<TF, WK>(T.A[k], T.B[k], t, s, Hr, hm, reinterpret_cast<const float2*>(sTr) + __float_as_int(bd.x),
                             P.inv_dt, tfod, static_cast<int>(bd.y), static_cast<int>(bd.z), bd.y, bd.z, R, acc[q][k]);
    };

    // The near traces (source and receiver within reach of the box) of the bin
    // are listed first, one thread per trace, and only those are examined
    // further: list entries lp .. nl - 1 are waiting, traces from jn on are
    // not listed yet.  Every wavefront holds the same lp, nl, jn.
    int64_t jn = (T.rmax >= 0.0f) ? lo : hi;
    int nl = 0, lp = 0, cpar = 0, cpass = 0;
    const int nf = min(list_threads(NW), P.list_cap);  // threads that list, one trace each per pass
    for (;;) {
        // ---- Build a block: passes of NG candidates (list entries lp ...), each
        // evaluated by the 16 lanes of one group.  Its window [wl, wl + len) of
        // samples covers, with a 2-sample margin, every time of a pair inside the
        // aperture: over the chunk's depths that can hold such a pair, the time at
        // the box's nearest distances bounds it from below, the time at the
        // farthest distances (capped at the depth's aperture) from above.
        int nb = 0, used = 0;
        for (;;) {
            if (lp == nl) {
                // list more near traces, in trace order, as long as a pass of nf fits; the
                // old entries' readers are behind the first barrier
                lp = 0;
                nl = 0;
                while (nl + nf <= P.list_cap && jn < hi) {
                    const int tid = fresh_v(threadIdx.x);
                    const int64_t j = jn + tid;
                    bool near = false;
                    if (j < hi && tid < nf) {
                        const float ls = box_dist2(P.src[2 * j], P.src[2 * j + 1], bx0, bx1, by0, by1);
                        const float lr = box_dist2(P.rec[2 * j], P.rec[2 * j + 1], bx0, bx1, by0, by1);
                        near = fmaxf(ls, lr) <= reach;
                    }
                    const uint64_t m = __builtin_amdgcn_ballot_w64(near);
                    int* cnt = sCnt + 16 * cpar;  // the two halves alternate: one barrier per pass
                    cpar ^= 1;
                    if (lane == 0) cnt[wave] = __builtin_popcountll(m);
                    __syncthreads();
                    int before = 0, total = 0;
                    for (int w = 0; w < NW; ++w) {
                        const int c = cnt[w];
                        before += w < wave ? c : 0;
                        total += c;
                    }
                    if (near)
                        sList[nl + before + __builtin_popcountll(m & ((1ull << lane) - 1ull))] =
                            static_cast<int>(j - lo);
                    nl += __builtin_amdgcn_readfirstlane(total);
                    jn += nf;
                }
                if (nl == 0) break;
                __syncthreads();  // the list
            }
            const int gi = wave * kGroupsPerWave + g;
            const int nc = min(NG, nl - lp);  // candidates of this pass
            int wl = 0, len = 0;
            float4 sr = make_float4(kFar, kFar, kFar, kFar);
            if (gi < nc) {
                const int64_t j = lo + sList[lp + gi];
                sr = make_float4(P.src[2 * j], P.src[2 * j + 1], P.rec[2 * j], P.rec[2 * j + 1]);
                wl = first_lo;
                len = nt + 2 - first_lo;  // samples first_lo .. nt + 1
                if (AA) {
                    // positions -(2 lmax + 4) .. nt + 2 lmax + 4: every clamped sample's reads
                    wl = -(2 * lmax + 4);
                    len = nt + 4 * lmax + 9;
                }
                if (windows) {
                    const float ls = box_dist2(sr.x, sr.y, bx0, bx1, by0, by1);
                    const float lr = box_dist2(sr.z, sr.w, bx0, bx1, by0, by1);
                    const float m = fmaxf(ls, lr);
                    const float ms = box_far2(sr.x, sr.y, bx0, bx1, by0, by1);
                    const float mr = box_far2(sr.z, sr.w, bx0, bx1, by0, by1);
                    float umin = __builtin_inff(), umax = -__builtin_inff();
                    bool any = false, bad = false;
#pragma unroll
                    for (int k = 0; k < KS; ++k) {
                        const float R = RREG ? T.R[k] : sR[k * kGroup + d];
                        if (m <= R) {
                            const float a = __builtin_amdgcn_sqrtf(fmaf(T.B[k], ls, T.A[k])) +
                                            __builtin_amdgcn_sqrtf(fmaf(T.B[k], lr, T.A[k]));
                            const float c = __builtin_amdgcn_sqrtf(fmaf(T.B[k], fminf(ms, R), T.A[k])) +
                                            __builtin_amdgcn_sqrtf(fmaf(T.B[k], fminf(mr, R), T.A[k]));
                            any = true;
                            bad = bad || !(a == a && c == c);
                            umin = fminf(umin, a);
                            umax = fmaxf(umax, c);
                        }
                    }
                    umin = group_min(umin);
                    umax = group_max(umax);
                    if (PX) {  // physical tables: seconds -> samples (a monotone rounding)
                        const float sc = static_cast<float>(P.inv_dt);
                        umin = umin * sc;
                        umax = umax * sc;
                    }
                    const uint32_t gany = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(any) >> (kGroup * g)) & 0xFFFFu;
                    const uint32_t gbad = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(bad) >> (kGroup * g)) & 0xFFFFu;
                    if (!gany) {
                        len = 0;  // no depth of the chunk can hold a pair
                    } else if (!gbad) {
                        if (TF) {
                            umin = umin + tfo;
                            umax = umax + tfo;
                        }
                        // sample indices, clamped before conversion
                        const float clo = -static_cast<float>(2 * lmax + 16);
                        const float chi = static_cast<float>(nt + 2 * lmax + 16);
                        const int fmin = static_cast<int>(floorf(fminf(fmaxf(umin, clo), chi))) - koff;
                        const int fmax = static_cast<int>(floorf(fminf(fmaxf(umax, clo), chi))) - koff;
                        if (AA) {
                            // reads reach lmax + 2 around the sample; the clamp range
                            // [wl + lmax + 2, wh - lmax - 2] must hold the pairs' samples
                            const int a0 = max(fmin - lmax - 4, -(2 * lmax + 4));
                            const int a1 = min(fmax + lmax + 4, nt + 2 * lmax + 4);
                            if (a0 + lmax + 2 > a1 - lmax - 2) {
                                len = 0;  // every triangle lies outside the record
                            } else {
                                wl = a0;
                                len = a1 - a0 + 1;
                            }
                        } else if (fmin - 2 > nt - 1 || fmax + 3 < 0) {
                            len = 0;  // every such time reads zeros: nothing to add
                        } else {
                            wl = max(fmin - 2, first_lo);
                            len = max(min(fmax + 3, nt + 1) - wl + 1, 2);
                        }
                    }
                }
            }
            // window start and length, 16 bits each (records of at most 20000 samples); the
            // two halves alternate, so that one barrier per pass is enough (it also
            // stands between the last block's readers and the next writes of its slots)
            uint32_t* cand = sCand + kCandMax * cpass;
            cpass ^= 1;
            if (d == 0) cand[gi] = static_cast<uint32_t>(wl + kWindowBias) | (static_cast<uint32_t>(len) << 16);
            __syncthreads();
            // Every wavefront takes the same decision: candidates 0 .. k - 1 join the
            // block (the others do not fit and open the next one).
            int clen = 0, cwl = 0, cn = 0;  // LDS floats of the candidate's window, its first and number of samples
            if (lane < nc) {
                const uint32_t c = cand[lane];
                cwl = static_cast<int>(c & 0xFFFFu) - kWindowBias;
                cn = static_cast<int>(c >> 16);
                clen = cn > 0 ? (AA      ? 2 * ((cn + 3) & ~3)  // whole quads of positions: stage_window_i2
                                 : T16   ? (cn + 1) / 2
                                 : P16   ? cn - 1
                                 : PAIRS ? 2 * ((cn + 2) & ~3)  // whole quads of pairs: stage_pairs
                                         : cn)
                              : 0;
            }
            const int plen = wave_scan(clen), pcnt = wave_scan(clen > 0 ? 1 : 0);  // inclusive prefix sums
            const bool fits = used + plen <= P.cap && nb + pcnt <= P.tb;
            const uint64_t nofit = __builtin_amdgcn_ballot_w64(lane < nc && !fits);
            const int k = nofit ? static_cast<int>(__builtin_ctzll(nofit)) : nc;
            if (wave == 0 && lane < k && clen > 0) {
                const int slot = nb + pcnt - 1;
                const int jl = sList[lp + lane];
                const int64_t j = lo + jl;
                sGeo[slot] = make_float4(P.src[2 * j], P.src[2 * j + 1], P.rec[2 * j], P.rec[2 * j + 1]);
                const int off = used + plen - clen, cwh = cwl + cn - 1;  // window samples cwl .. cwh
                sMeta[slot] = make_int4(off, cwl, cwh, jl);
                // the row's offset (position of sample 0 plus koff), the clamp bounds and,
                // with 16-bit staging, the trace's scale (applied per pair with the weight)
                sBnd[slot] = make_float4(
                    __int_as_float((PAIRS || AA ? off / 2 : T16 ? 2 * off : off) - cwl - koff),
                    static_cast<float>(cwl + koff + (AA ? lmax + 2 : 0)),
                    static_cast<float>(cwh - 1 + koff - (AA ? lmax + 1 : 0)), (S16 && P.scale) ? P.scale[j] : 1.0f);
            }
            if (k > 0) {
                nb += __builtin_amdgcn_readlane(pcnt, k - 1);
                used += __builtin_amdgcn_readlane(plen, k - 1);
            }
            lp += k;
            if (k < nc) break;
        }
        if (nb == 0) break;  // the bin is exhausted (a block that breaks off full holds a trace)
        __syncthreads();     // the block's slots
        const int sl = fresh_v(lane);
        if (PAIRS) stage_pairs(P, lo, sMeta, sTr, nb, wave, NW, sl);
        for (int t = PAIRS ? nb : wave; t < nb; t += NW) {
            const int4 mt = sMeta[t];
            if (AA) stage_window_i2(P, lo + mt.w, mt.y, mt.z - mt.y + 1, reinterpret_cast<double*>(sTr + mt.x), sl);
            else if (T16) stage_window_16(P, lo + mt.w, mt.y, mt.z - mt.y + 1, reinterpret_cast<uint16_t*>(sTr + mt.x), sl);
            else if (P16) stage_window_16p(P, lo + mt.w, mt.y, mt.z - mt.y + 1, reinterpret_cast<uint32_t*>(sTr + mt.x), sl);
            else stage_window_f(P, lo + mt.w, mt.y, mt.z - mt.y + 1, sTr + mt.x, sl);
        }
        __syncthreads();

        // Column group by column group over the block, so that one group's source
        // legs (SrcLeg) live in registers from trace to trace.
#pragma unroll
        for (int q = 0; q < CWQ; ++q) {
            // the lane's column of this group (looked up again for every block: the
            // registers it would take are worth more than the few reads)
            const int col = col0 + kGroupsPerWave * q + fresh_v(g);
            const bool has = col < ncol;
            const float px = has ? P.x[col % P.nx] : kFar, py = has ? P.y[col / P.nx] : kFar;
            const LCol lc = LAT ? lateral_col(P, px, py) : LCol{0, 0.0f, 0.0f};
            SrcLeg<KS, TT, PX> S;
            float hs2 = 0.0f, dxs = 0.0f, dys = 0.0f;  // the kept source leg: squared length, components
            // position of the source whose leg is kept (none yet: equal to nothing)
            float curx = __builtin_nanf(""), cury = __builtin_nanf("");
            for (int t0 = 0; t0 < nb; t0 += kGroup) {
                const int nbt = min(kGroup, nb - t0);
                // lane (g, d): legs of column group member g and trace t0 + d
                const float4 sr = sGeo[min(t0 + d, nb - 1)];
                const Legs Lp = legs(px, py, sr);
                LegsX Lx{0.0, 0.0};
                if (PX) Lx = legs_ext(px, py, sr);
                // traces that some column of the group can reach at some depth of the chunk
                uint32_t live = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(rows_min(Lp.hmax) <= T.rmax)) &
                                ((1u << nbt) - 1u);
                // this wavefront's share of the traces (by the trace's place in the bin, so that the
                // sums do not depend on where a block ends)
                if (TS > 1)
                    live &= static_cast<uint32_t>(
                        __builtin_amdgcn_ballot_w64(sMeta[min(t0 + d, nb - 1)].w % TS == part));
                if (!live) continue;
                // bit t: trace t0 + t has another source than the trace before it (t = 0: than the kept one)
                const float ux = dpp_f<0x111>(sr.x), uy = dpp_f<0x111>(sr.y);
                uint32_t fresh = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(
                                     d == 0 ? !(sr.x == curx && sr.y == cury) : !(sr.x == ux && sr.y == uy))) & 0xFFFFu;
                // The receiver leg of trace t reaches the depth lanes through the LDS
                // crossbar; the next live trace's is requested before trace t is evaluated.
                const int row4 = 4 * (lane & ~(kGroup - 1));  // crossbar address of the lane's row
                if constexpr (OWN) {
                    // both legs of every pair; the next live trace's lengths are requested before
                    // trace tc is evaluated
                    int t = __builtin_ctz(live);
                    float hs2n = bperm_f(row4 | 4 * t, Lp.hs2), hr2n = bperm_f(row4 | 4 * t, Lp.hr2);
                    double Hsn = 0.0, Hrn = 0.0;
                    if (PX) {
                        Hsn = bperm_d(row4 | 4 * t, Lx.hs2);
                        Hrn = bperm_d(row4 | 4 * t, Lx.hr2);
                    }
                    for (;;) {
                        const int tc = t;
                        const float hs2 = hs2n, hr2 = hr2n;
                        const double Hs = Hsn, Hr = Hrn;
                        const float4 bd = sBnd[t0 + tc];
                        live ^= 1u << tc;
                        const bool more = live != 0;
                        if (more) {
                            t = __builtin_ctz(live);
                            hs2n = bperm_f(row4 | 4 * t, Lp.hs2);
                            hr2n = bperm_f(row4 | 4 * t, Lp.hr2);
                            if (PX) {
                                Hsn = bperm_d(row4 | 4 * t, Lx.hs2);
                                Hrn = bperm_d(row4 | 4 * t, Lx.hr2);
                            }
                        }
                        float hm;
                        asm("v_max_f32 %0, %1, %2" : "=v"(hm) : "v"(hs2), "v"(hr2));
                        uint32_t any, full;
                        slot_masks<KS>(T, hm, any, full);
                        if (!any) {
                            if (!more) break;
                            continue;
                        }
                        if constexpr (is_table(TT)) {
                            const TLeg Ls = table_leg(P, hs2), Lr = table_leg(P, hr2);
                            const int vs = 4 * ((LAT ? lc.off : 0) + Ls.off + z0 + d);
                            const int vr = 4 * ((LAT ? lc.off : 0) + Lr.off + z0 + d);
#pragma unroll
                            for (int k = 0; k < KS; k += 2) {
                                if (!((any >> k) & 3u)) continue;
                                const int o0 = min(64 * k, vl), o1 = min(64 * k + 64, vl);
                                float s0 = 1.0f, s1 = 1.0f;
                                if (P.tamp) {
                                    s0 = table_amp_at<LAT>(P, Ls.f, lc, vs + o0);
                                    s1 = table_amp_at<LAT>(P, Ls.f, lc, vs + o1);
                                }
                                const TTime ts0 = LAT ? ltable_time_at(P, Ls.f, lc, vs + o0) : table_time_at(P, Ls.f, vs + o0);
                                const TTime ts1 = LAT ? ltable_time_at(P, Ls.f, lc, vs + o1) : table_time_at(P, Ls.f, vs + o1);
                                const Pair p0 = pair_table<TF, LAT>(P, ts0, s0, Lr.f, vr + o0, bd.y, bd.z, lc);
                                const Pair p1 = pair_table<TF, LAT>(P, ts1, s1, Lr.f, vr + o1, bd.y, bd.z, lc);
                                add_table_pairs(p0, p1, bd, full, k, hm, q);
                            }
                        } else if constexpr (PX) {
#pragma unroll
                            for (int k = 0; k < KS; ++k) {
                                if (!((any >> k) & 1u)) continue;
                                float A = T.A[k], B = T.B[k];
                                asm volatile("" : "+v"(A), "+v"(B));  // as in mig_slot_ext
                                const LegTimeX l = leg_time_ext(A, B, Hs);
                                add_ext_slot(l.t, l.q, Hr, bd, k, hm, q);
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < KS; k += 2) {
                                if (!((any >> k) & 3u)) continue;
                                const float a0 = fmaf(T.B[k], hs2, T.A[k]), a1 = fmaf(T.B[k + 1], hs2, T.A[k + 1]);
                                add_root_pairs(a0, __builtin_amdgcn_sqrtf(a0), a1, __builtin_amdgcn_sqrtf(a1), hr2, bd,
                                               full, k, hm, q);
                            }
                        }
                        if (!more) break;
                    }
                    continue;
                }
                int t = __builtin_ctz(live);
                float hr2n = bperm_f(row4 | 4 * t, Lp.hr2);
                double Hrn = 0.0;
                if (PX) Hrn = bperm_d(row4 | 4 * t, Lx.hr2);
                for (;;) {
                    const int tc = t;
                    const float hr2 = hr2n;
                    const double Hr = Hrn;
                    // row offset, clamp bounds and scale of the trace, the same for every lane
                    // (vector registers: a clamp with two scalar bounds costs a move per pair)
                    const float4 bd = sBnd[t0 + tc];
                    live ^= 1u << tc;
                    const bool more = live != 0;
                    if (more) {
                        t = __builtin_ctz(live);
                        hr2n = bperm_f(row4 | 4 * t, Lp.hr2);
                        if (PX) Hrn = bperm_d(row4 | 4 * t, Lx.hr2);
                    }
                    const uint32_t upto = (2u << tc) - 1u;
                    if (fresh & upto) {
                        fresh &= ~upto;
                        curx = uniform_read(sr.x, tc);
                        cury = uniform_read(sr.y, tc);
                        hs2 = bperm_f(row4 | 4 * tc, Lp.hs2);
                        if constexpr (AA) {
                            dxs = px - curx;
                            dys = py - cury;
                        }
                        double Hs = 0.0;
                        if (PX) Hs = bperm_d(row4 | 4 * tc, Lx.hs2);
                        source_leg<KS, WK, TT, PX>(P, T, hs2, Hs, lc, 4 * (z0 + d), vl, S);
                    }
                    // max(hs2, hr2): one v_max (fmaxf would first quiet both inputs)
                    float hm;
                    asm("v_max_f32 %0, %1, %2" : "=v"(hm) : "v"(hs2), "v"(hr2));
                    uint32_t any, full;
                    slot_masks<KS>(T, hm, any, full);
                    if (!any) {
                        if (!more) break;
                        continue;
                    }
                    // in pairs / doubles / 16-bit samples / floats or packed 16-bit pairs
                    const int rb = __float_as_int(bd.x);
                    const float wlo = bd.y, whi = bd.z, scl = bd.w;
                    if constexpr (is_table(TT) && PX) {
                        const TLegX Lr = table_leg_ext(P, Hr);
                        const int vr = 4 * ((LAT ? lc.off : 0) + Lr.off + z0 + d);
                        const float* row = sTr + rb;
#pragma unroll
                        for (int k = 0; k < KS; k += 2) {
                            if ((any >> k) & 3u) {
                                const Pair p0 = pair_table_ext<TF, LAT>(P, S.t[k], S.amp[k], Lr.f, vr + min(64 * k, vl), wlo, whi, lc);
                                const Pair p1 = pair_table_ext<TF, LAT>(P, S.t[k + 1], S.amp[k + 1], Lr.f, vr + min(64 * k + 64, vl), wlo, whi, lc);
                                const float a0 = row[p0.i], b0 = row[p0.i + 1];
                                const float a1 = row[p1.i], b1 = row[p1.i + 1];
                                mask_add2<W_COSCOS, KS, RREG>(T, sR, full, k, d, hm, fmaf(p0.f, b0 - a0, a0),
                                                              fmaf(p1.f, b1 - a1, a1), p0.r, p1.r, acc[q][k], acc[q][k + 1]);
                            }
                        }
                    } else if constexpr (is_table(TT)) {
                        const TLeg Lr = table_leg(P, hr2);
                        const int vr = 4 * ((LAT ? lc.off : 0) + Lr.off + z0 + d);
#pragma unroll
                        for (int k = 0; k < KS; k += 2) {
                            if ((any >> k) & 3u) {
                                const Pair p0 = pair_table<TF, LAT>(P, TTime{S.base[k], S.inc[k]}, S.amp[k], Lr.f, vr + min(64 * k, vl), wlo, whi, lc);
                                const Pair p1 = pair_table<TF, LAT>(P, TTime{S.base[k + 1], S.inc[k + 1]}, S.amp[k + 1], Lr.f, vr + min(64 * k + 64, vl), wlo, whi, lc);
                                add_table_pairs(p0, p1, bd, full, k, hm, q);
                            }
                        }
                    } else if constexpr (AA) {
                        // column minus receiver of trace tc, for the operator dip
                        const float dxr = px - uniform_read(sr.z, tc), dyr = py - uniform_read(sr.w, tc);
                        const double* rowd = reinterpret_cast<const double*>(sTr) + rb;
#pragma unroll
                        for (int k = 0; k < KS; ++k) {
                            if ((any >> k) & 1u) {
                                const float R = RREG ? T.R[k] : sR[k * kGroup + d];
                                mig_slot_aa<TF, WK>(T.A[k], T.B[k], S.a[k], S.s[k], hr2, hm, rowd, tfo, wlo, whi, R,
                                                    dxs, dys, dxr, dyr, P.aa_dx, P.aa_dy, static_cast<float>(lmax),
                                                    sInvSq, acc[q][k]);
                            }
                        }
                    } else if constexpr (PX) {
#pragma unroll
                        for (int k = 0; k < KS; ++k)
                            if ((any >> k) & 1u) add_ext_slot(S.t[k], S.q[k], Hr, bd, k, hm, q);
                    } else {
#pragma unroll
                        for (int k = 0; k < KS; k += 2)
                            if ((any >> k) & 3u)
                                add_root_pairs(S.a[k], S.s[k], S.a[k + 1], S.s[k + 1], hr2, bd, full, k, hm, q);
                    }
                    if (!more) break;
                }
            }
        }
    }

    if (TS > 1) {
        // the parts' sums through LDS (the window storage is free), added in part order
        __syncthreads();
        constexpr int kPart = NC * CWQ * KS * kLanes;
        float* mine = sTr + cw * (CWQ * KS * kLanes) + lane;
        if (part > 0)
#pragma unroll
            for (int e = 0; e < CWQ * KS; ++e) mine[(part - 1) * kPart + e * kLanes] = acc[e / KS][e % KS];
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int e = 0; e < CWQ * KS; ++e)
#pragma unroll
            for (int o = 0; o < TS - 1; ++o) acc[e / KS][e % KS] += mine[o * kPart + e * kLanes];
    }

    float* img = P.image + static_cast<int64_t>(b) * ncol * P.nz;
#pragma unroll
    for (int q = 0; q < CWQ; ++q) {
        const int col = col0 + kGroupsPerWave * q + fresh_v(g);
        if (col >= ncol) continue;
        float* colp = img + static_cast<int64_t>(col) * P.nz;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int iz = z0 + k * kGroup + d;
            if (iz < z1) {
                const float fac = depth_factor<PX>(P, iz);
                const float val = fac != 0.0f ? acc[q][k] * fac : 0.0f;
                colp[iz] = P.accumulate ? colp[iz] + val : val;
            }
        }
    }
}

// Bin b, column tile, depth chunk of a problem: the form its order of traces asks for.
template <int NW, int CWQ, int KS, int TS, bool TF, int WK, bool RREG, int TT = TT_DSR, bool PX = false, int S16 = 0>
__device__ __forceinline__ void migrate_item(const Params& P, int b, int tile, int zc, float* lds) {
    int64_t lo, hi;
    if constexpr (own_legs(TT, PX, TS)) {
        const SourceSample sample = sample_sources(P);
        bin_range(P.bin, P.n_traces, b, lo, hi);
        if (!sources_repeat(sample)) {
            migrate_tile<NW, CWQ, KS, TS, TF, WK, RREG, TT, PX, S16, true>(P, lo, hi, b, tile, zc, lds);
            return;
        }
    } else {
        bin_range(P.bin, P.n_traces, b, lo, hi);
    }
    migrate_tile<NW, CWQ, KS, TS, TF, WK, RREG, TT, PX, S16>(P, lo, hi, b, tile, zc, lds);
}

// Store zeros into a tile whose (column, trace) pairs are all outside the
// aperture (known from the counting kernel): its image values are exactly 0.
template <int NW, int CWQ, int KS, int TS>
__device__ __forceinline__ void zero_tile(const Params& P, int b, int tile, int zc) {
    if (P.accumulate) return;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = threadIdx.x / kLanes;
    if (wave >= NW / TS) return;  // the column wavefronts
    const int g = lane / kGroup, d = lane % kGroup;
    const int ncol = P.nx * P.ny;
    const int z0 = zc * P.zspan;
    const int z1 = min(z0 + P.zspan, P.nz);  // end of the chunk's depths
    float* img = P.image + static_cast<int64_t>(b) * ncol * P.nz;
#pragma unroll
    for (int q = 0; q < CWQ; ++q) {
        const int col = ((tile * (NW / TS) + wave) * CWQ + q) * kGroupsPerWave + g;
        if (col >= ncol) continue;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int iz = z0 + k * kGroup + d;
            if (iz < z1) img[static_cast<int64_t>(col) * P.nz + iz] = 0.0f;
        }
    }
}

// Held to 4 wavefronts per SIMD (128 VGPRs; the 4-group shapes spill about 20,
// outside the pair loops) so that two 8-wavefront workgroups share a CU: 331
// ms against 592 ms at the 173 registers the compiler takes by itself (8 waves x
// 4 groups, the survey of the file comment).
template <int NW, int CWQ, int KS, int TS, bool TF, int WK, int TT = TT_DSR, bool PX = false, int S16 = 0>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(KS <= 8 ? 4 : 1)))
void migrate_kernel(Params P) {
    extern __shared__ __align__(16) float lds[];
    constexpr bool RREG = true;
    migrate_item<NW, CWQ, KS, TS, TF, WK, RREG, TT, PX, S16>(P, blockIdx.z, blockIdx.x, blockIdx.y, lds);
}

// Batched persistent form: work items (problem, bin, column tile, depth
// chunk) are taken from a queue in list order (longest first).  A negative
// tile field -1 - tile marks an item with no pair in aperture: zero store.
// At least 4 wavefronts per SIMD (<= 128 VGPRs) for the 8-slot shapes, so
// that two 8-wavefront workgroups share a CU as they do in single launches.
template <int NW, int CWQ, int KS, int TS, bool TF, int WK, bool PX = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(KS <= 8 ? 4 : 2)))
void migrate_batch_kernel(const Params* __restrict__ probs,
                                                                const int4* __restrict__ items,
                                                                int64_t n_items, unsigned int* counter) {
    extern __shared__ __align__(16) float lds[];
    __shared__ int64_t s_item;
    for (;;) {
        __syncthreads();  // also: the last item's LDS is free
        if (threadIdx.x == 0) s_item = static_cast<int64_t>(atomicAdd(counter, 1u));
        __syncthreads();
        const int64_t it = s_item;
        if (it >= n_items) break;
        const int4 w = items[it];  // (problem, bin, tile, zchunk)
        const Params P = probs[w.x];
        if (w.z < 0) zero_tile<NW, CWQ, KS, TS>(P, w.y, -1 - w.z, w.w);
        else migrate_item<NW, CWQ, KS, TS, TF, WK, false, TT_DSR, PX>(P, w.y, w.z, w.w, lds);
    }
}

// ---------------------------------------------------------------------------
// Launch tables
// ---------------------------------------------------------------------------

// The plain kernels of one time precision (PX) for the weight and t_first cases.
template <int NW, int CWQ, int KS, int TS, bool PX>
static hipError_t launch_migrate_dsr(const Params& P, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    if (P.has_tf) {
        if (P.weight == W_COSCOS)
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_COSCOS, TT_DSR, PX>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_DSR, PX>, grid, block, lds, s, P);
    }
    if (P.weight == W_COSCOS)
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_COSCOS, TT_DSR, PX>, grid, block, lds, s, P);
    return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_DSR, PX>, grid, block, lds, s, P);
}

// The 16-bit staging kernels (float32 time), per storage type: square-root
// times per weight and t_first case, the two table kinds per t_first case.
template <int NW, int CWQ, int KS, int TS, int DT>
static hipError_t launch_migrate_s16_dt(const Params& P, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    if (P.ttab) {
        if (P.n_gx > 0) {
            if (P.has_tf)
                return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_LTABLE, false, DT>, grid, block, lds, s, P);
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_LTABLE, false, DT>, grid, block, lds, s, P);
        }
        if (P.has_tf)
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_TABLE, false, DT>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_TABLE, false, DT>, grid, block, lds, s, P);
    }
    if (P.has_tf) {
        if (P.weight == W_COSCOS)
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_COSCOS, TT_DSR, false, DT>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_DSR, false, DT>, grid, block, lds, s, P);
    }
    if (P.weight == W_COSCOS)
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_COSCOS, TT_DSR, false, DT>, grid, block, lds, s, P);
    return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_DSR, false, DT>, grid, block, lds, s, P);
}

template <int NW, int CWQ, int KS, int TS>
static hipError_t launch_migrate_s16(const Params& P, dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    if (P.dtype == BF16) return launch_migrate_s16_dt<NW, CWQ, KS, TS, BF16>(P, grid, block, lds, s);
    return launch_migrate_s16_dt<NW, CWQ, KS, TS, F16>(P, grid, block, lds, s);
}

template <int NW, int CWQ, int KS, int TS>
static hipError_t launch_migrate_shape(const Params& P, hipStream_t s) {
    dim3 grid(P.n_coltiles, P.n_zchunks, P.n_bins), block(NW * 64);
    const size_t lds = lds_bytes(P, KS);
    if (P.s16) return launch_migrate_s16<NW, CWQ, KS, TS>(P, grid, block, lds, s);  // the host checked the kind
    if (P.ttab && P.n_gx > 0) {  // laterally varying tables: W = 1
        if (P.prec) {
            if (P.has_tf)
                return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_LTABLE, true>, grid, block, lds, s, P);
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_LTABLE, true>, grid, block, lds, s, P);
        }
        if (P.has_tf) return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_LTABLE>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_LTABLE>, grid, block, lds, s, P);
    }
    if (P.ttab) {  // table traveltimes: W = 1 (the host rejects other weights)
        if (P.prec) {
            if (P.has_tf)
                return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_TABLE, true>, grid, block, lds, s, P);
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_TABLE, true>, grid, block, lds, s, P);
        }
        if (P.has_tf) return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_TABLE>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_TABLE>, grid, block, lds, s, P);
    }
    if (P.aa_max > 0) {  // anti-alias triangle filter
        if (P.has_tf) {
            if (P.weight == W_COSCOS)
                return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_COSCOS, TT_AA>, grid, block, lds, s, P);
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, true, W_UNIT, TT_AA>, grid, block, lds, s, P);
        }
        if (P.weight == W_COSCOS)
            return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_COSCOS, TT_AA>, grid, block, lds, s, P);
        return launch_with_lds(migrate_kernel<NW, CWQ, KS, TS, false, W_UNIT, TT_AA>, grid, block, lds, s, P);
    }
    if (P.prec) return launch_migrate_dsr<NW, CWQ, KS, TS, true>(P, grid, block, lds, s);
    return launch_migrate_dsr<NW, CWQ, KS, TS, false>(P, grid, block, lds, s);
}

// The batch kernel of (shape, t_first, weight, precision).
template <int NW, int CWQ, int KS, int TS>
static const void* batch_kernel_of(int has_tf, int weight, int prec) {
    if (prec) {
        if (has_tf) return weight == W_COSCOS ? (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, true, W_COSCOS, true>
                                              : (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, true, W_UNIT, true>;
        return weight == W_COSCOS ? (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, false, W_COSCOS, true>
                                  : (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, false, W_UNIT, true>;
    }
    if (has_tf) return weight == W_COSCOS ? (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, true, W_COSCOS>
                                          : (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, true, W_UNIT>;
    return weight == W_COSCOS ? (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, false, W_COSCOS>
                              : (const void*)migrate_batch_kernel<NW, CWQ, KS, TS, false, W_UNIT>;
}

template <int NW, int CWQ, int KS, int TS>
static hipError_t launch_migrate_batch_shape(const Params* probs, const int4* items, int64_t n_items,
                                             unsigned int* counter, int has_tf, int weight, int prec, int n_wg,
                                             size_t lds, hipStream_t s) {
    dim3 grid(n_wg), block(NW * 64);
    using K = void (*)(const Params*, const int4*, int64_t, unsigned int*);
    const K kern = reinterpret_cast<K>(const_cast<void*>(batch_kernel_of<NW, CWQ, KS, TS>(has_tf, weight, prec)));
    return launch_with_lds(kern, grid, block, lds, s, probs, items, n_items, counter);
}

// Waves, column groups per wave, depth slots, LDS budget for the trace block,
// trace parts.  The small tiles (ms, square-root times, before: 8 waves x 4 groups):
//   1536 traces -> 8 x 128 x 200 points    0.521 -> 0.058  (16 waves, 4 parts, 4 slots)
//   6144 traces -> 8 x 256 x 256           1.91  -> 0.289  (16 waves, 4 parts, 8 slots)
//   16384 traces -> 16 x 512 x 400         2.57  -> 1.89   (4 waves, 1 group)
//   20736 traces -> 10 x 80 x 80 x 300     17.9  -> 14.6   (8 waves, 2 groups)
// build.py compiles this file once per shape (KM_PART = its index: a shape has
// about 50 kernels) and once without KM_PART for the dispatch.
constexpr TileShape kMigrateShapes[] = {
    {4, 4, 8, 32768, 0, 1},
    {16, 4, 8, 155648, 0, 1},
    {8, 4, 8, 77824, 0, 1},
    {4, 3, 16, 49152, 0, 1},
    {4, 2, 16, 49152, 0, 1},
    {8, 2, 8, 77824, 0, 1},
    {4, 1, 8, 40960, 0, 1},
    {16, 1, 8, 77824, 0, 4},
    {16, 1, 4, 77824, 0, 4},
};
constexpr int kMigrateShapeCount = static_cast<int>(sizeof(kMigrateShapes) / sizeof(kMigrateShapes[0]));

using MigrateLaunch = hipError_t (*)(const Params& P, hipStream_t s);
using MigrateBatchLaunch = hipError_t (*)(const Params* probs, const int4* items, int64_t n_items,
                                          unsigned int* counter, int has_tf, int weight, int prec, int n_wg,
                                          size_t lds, hipStream_t s);
using MigrateBatchKernel = const void* (*)(int has_tf, int weight, int prec);
struct MigratePart {
    MigrateLaunch launch;
    MigrateBatchLaunch launch_batch;
    MigrateBatchKernel batch_kernel;
};
template <int SHAPE>
MigratePart migrate_part();

#ifdef KM_PART

template <>
MigratePart migrate_part<KM_PART>() {
    constexpr TileShape S = kMigrateShapes[KM_PART];
    return {launch_migrate_shape<S.waves, S.column_groups, S.depth_slots, S.trace_parts>,
            launch_migrate_batch_shape<S.waves, S.column_groups, S.depth_slots, S.trace_parts>,
            batch_kernel_of<S.waves, S.column_groups, S.depth_slots, S.trace_parts>};
}

#else

template <int... I>
static MigratePart part_of(int shape, std::integer_sequence<int, I...>) {
    MigratePart p{nullptr, nullptr, nullptr};
    ((shape == I ? (void)(p = migrate_part<I>()) : (void)0), ...);
    return p;
}

static MigratePart part_of(int shape) {
    return part_of(shape, std::make_integer_sequence<int, kMigrateShapeCount>());
}

int migrate_shape_count() { return kMigrateShapeCount; }
const TileShape& migrate_shape(int i) { return kMigrateShapes[i]; }

hipError_t launch_migrate(int shape, const Params& P, hipStream_t s) {
    const MigratePart p = part_of(shape);
    return p.launch ? p.launch(P, s) : hipErrorInvalidValue;
}

hipError_t launch_migrate_batch(int shape, const Params* probs, const int4* items, int64_t n_items,
                                unsigned int* counter, int has_tf, int weight, int prec, int n_wg, size_t lds,
                                hipStream_t s) {
    const MigratePart p = part_of(shape);
    return p.launch_batch ? p.launch_batch(probs, items, n_items, counter, has_tf, weight, prec, n_wg, lds, s)
                          : hipErrorInvalidValue;
}

const void* migrate_batch_kernel_ptr(int shape, int has_tf, int weight, int prec) {
    const MigratePart p = part_of(shape);
    return p.batch_kernel ? p.batch_kernel(has_tf, weight, prec) : nullptr;
}

#endif

}  // namespace km
