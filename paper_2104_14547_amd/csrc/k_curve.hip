// Rational B-spline curves in the plane and in space on gfx950.
//
//   C(u) = sum_i N_i^p(u) w_i P_i / sum_i N_i^p(u) w_i
//
// is eq. NURBS with one parametric direction: NURBS-Diff (Sec. 3) gets its
// curve layer from the surface formulas by dropping a direction.  Per sample
// the forward takes the span, the p+1 non-zero basis functions (Sec. 3.1.2
// steps 1-2), the homogeneous sum and the rational divide (step 3), and on
// request dC/du = (A_u - C W_u) / W (Appendix A, eq. NURBSuDerivative1).  The
// backward is Sec. 3.2 without v: with g = dL/dC at a sample,
//   dL/dP_i += N_i w_i g / W                    (eq. NURBSuDerivative4)
//   dL/dw_i += N_i (P_i - C) . g / W            (eq. NURBSvDerivative5)
//   dL/dN_i  = w_i (P_i - C) . g / W            (eq. NURBSvDerivative6)
// and dL/dU_k from dL/dN_i through the knot adjoint of the recursion
// (Sec. 3.2.1).  dL/dw is taken directly from P_i - C (not as P . dL/dPw +
// dL/dPw_w), so no difference of two large sums is formed.
//
// Work decomposition.  A workgroup (4 waves, 1 to 4 in the backward) owns one
// chunk of up to kCurveChunk consecutive samples of one curve and stages that
// curve's knots and control polygon in LDS.  Forward: one sample per lane.
// Backward: the chunk's samples are put in span order (sorted parameters, the
// usual case, are in it already; others go through a stable counting sort in
// LDS) and the samples of a span are cut into items, one item per lane at a
// time; sorted samples with few to a span go one to a lane as they are.  Lanes
// of one span form runs; a DPP segmented scan (the surface backward's, one
// v_fmac_f32_dpp per value and step) sums each run, whose last
// lane adds the sums into the wave's LDS accumulators, without atomics.  At
// the end of the chunk the waves' accumulators are added in wave order.
// A curve with one chunk writes its gradients directly; longer curves write
// one partial per chunk to the workspace and a finalize kernel adds the
// partials in chunk order.  Every sum has a fixed order, so results are
// bitwise reproducible.
#include <algorithm>

#include "kernels.hpp"
#include "launch.hpp"
#include "../../include/nurbsdiff.h"

namespace nd {
namespace {

__device__ __forceinline__ void curve_post_error(int* err, int code) {
    if (err) atomicCAS(err, 0, code);
}

// Data checks (NURBS_VALIDATE): knots and weights by the curve's first
// chunk, parameters by every chunk.
__device__ void curve_validate(const CurveArgs& a, int p, int c, int chunk, int s0, int s1, const float* U,
                               const float* w, const float* us) {
    const int t = threadIdx.x;
    const int nU = a.nc + p + 1;
    bool bad_k = false, bad_w = false, bad_d = false;
    if (chunk == 0) {
        for (int i = t; i + 1 < nU; i += blockDim.x) bad_k |= !(U[i] <= U[i + 1]);
        if (t == 0) bad_k |= !(U[p] < U[p + 1]) || !(U[a.nc - 1] < U[a.nc]);
        for (int i = t; i < a.nc; i += blockDim.x) bad_w |= !(w[i] > 0.f);
    }
    const float lo = U[p], hi = U[a.nc];
    for (int s = s0 + t; s < s1; s += blockDim.x) bad_d |= !(us[s] >= lo && us[s] <= hi);
    if (bad_k) curve_post_error(a.err, NURBS_EKNOTS);
    if (bad_w) curve_post_error(a.err, NURBS_EWEIGHTS);
    if (bad_d) curve_post_error(a.err, NURBS_EDOMAIN);
}

// (curve, chunk) of this workgroup, and the chunk's sample range
struct CurveBlock {
    int c, chunk, s0, s1;
};
__device__ __forceinline__ CurveBlock curve_block(const CurveArgs& a) {
    CurveBlock b;
    const int blk = (int)blockIdx.x;
    b.c = blk / a.nchunks;
    b.chunk = blk - b.c * a.nchunks;
    b.s0 = b.chunk * kCurveChunk;
    b.s1 = min(a.ns, b.s0 + kCurveChunk);
    return b;
}

// Stage the curve's knots and control points (xyz or xy, times the weight if
// HOM, and the weight) in LDS.
template <int DIM, bool HOM = false>
__device__ __forceinline__ void stage_curve(const CurveArgs& a, int p, int c, float* U, float4* Pw) {
    const int nU = a.nc + p + 1;
    const float* kn = a.knots + (size_t)c * nU;
    const float* cp = a.ctrl + (size_t)c * a.nc * DIM;
    const float* w = a.w + (size_t)c * a.nc;
    for (int i = threadIdx.x; i < nU; i += blockDim.x) U[i] = kn[i];
    for (int i = threadIdx.x; i < a.nc; i += blockDim.x) {
        const float wt = w[i], f = HOM ? wt : 1.f;
        Pw[i] = make_float4(cp[i * DIM] * f, cp[i * DIM + 1] * f, DIM == 3 ? cp[i * DIM + 2] * f : 0.f, wt);
    }
}

// --------------------------------------------------------------------------
// forward
// --------------------------------------------------------------------------
// What bounds it: VALU issue.  So what samples share is formed once per
// workgroup: the homogeneous control points and, where a workgroup has samples
// enough to repay it, the reciprocals of every span's knot intervals (not
// beyond degree kCurveTabDeg, where the table would hold a workgroup's LDS to
// fewer residents).  16384 cubic space curves x 1024 samples: 53.5 us, 3.8 TB/s
// of points written; with both formed per sample 62 us, 3.9e7 wave instructions
// (63 us of issue).  With and without the table, 16384 curves of 16 control
// points: degree 1, 16 samples 13.4 and 12.7 us; 3, 256 25.5 and 25.6; 3, 1024
// 57 and 59; 4, 256 27.5 and 30.8; 4, 64 17.3 and 14.9.
constexpr int kCurveTabDeg = 4;
inline bool curve_tab(int p, int ns) { return p >= 2 && ns >= (p >= 4 ? 256 : 512); }

template <int P, int DIM, bool DU, bool kTab>
__global__ void __launch_bounds__(kWG) k_curve_fwd(CurveArgs a, float* __restrict__ pts, float* __restrict__ du) {
    constexpr int kInv = P * (P + 1) / 2;
    __shared__ float U[kWG];
    __shared__ float4 Pw[kWG];
    __shared__ float tab[kTab ? kWG * kInv : 1];
    const CurveBlock b = curve_block(a);
    stage_curve<DIM, true>(a, P, b.c, U, Pw);
    __syncthreads();
    if constexpr (kTab) {
        for (int i = threadIdx.x; i < a.nc - P; i += kWG) {
            float K[2 * P], inv[kInv];
#pragma unroll
            for (int t = 0; t < 2 * P; ++t) K[t] = U[i + 1 + t];
            span_inv<P>(K, inv);
#pragma unroll
            for (int t = 0; t < kInv; ++t) tab[i * kInv + t] = inv[t];
        }
        __syncthreads();
    }
    const float* us = a.us + (a.u_shared ? 0 : (size_t)b.c * a.ns);
    if (a.err) curve_validate(a, P, b.c, b.chunk, b.s0, b.s1, U, a.w + (size_t)b.c * a.nc, us);
    const size_t base = (size_t)b.c * a.ns;
    for (int s = b.s0 + (int)threadIdx.x; s < b.s1; s += kWG) {
        const float x = clamp_param(U, P, a.nc - 1, us[s]);
        const int k = find_span(U, P, a.nc - 1, x);
        float N[P + 1], dN[P + 1];
        if constexpr (kTab) {
            float K[2 * P], inv[kInv], st[kInv];
#pragma unroll
            for (int t = 0; t < 2 * P; ++t) K[t] = U[k - P + 1 + t];
#pragma unroll
            for (int t = 0; t < kInv; ++t) inv[t] = tab[(k - P) * kInv + t];
            span_basis<P>(K, inv, x, N, st);
        } else if constexpr (DU) {
            basis_d1_f32<P>(U, k, x, N, dN);
        } else {
            basis_f32<P>(U, k, x, N);
        }
        float4 A = make_float4(0.f, 0.f, 0.f, 0.f), Au = A;
#pragma unroll
        for (int r = 0; r <= P; ++r) {
            const float4 hq = Pw[k - P + r];
            A = fma4(N[r], hq, A);
            if constexpr (DU) Au = fma4(dN[r], hq, Au);
        }
        const float inv = recip_fast(A.w);
        const float cx = A.x * inv, cy = A.y * inv, cz = A.z * inv;
        float* o = pts + (base + s) * DIM;
        if constexpr (DIM == 3) store3(o, cx, cy, cz);
        else *reinterpret_cast<float2*>(o) = make_float2(cx, cy);
        if constexpr (DU) {
            float* d = du + (base + s) * DIM;
            const float ex = (Au.x - cx * Au.w) * inv, ey = (Au.y - cy * Au.w) * inv;
            if constexpr (DIM == 3) store3(d, ex, ey, (Au.z - cz * Au.w) * inv);
            else *reinterpret_cast<float2*>(d) = make_float2(ex, ey);
        }
    }
}

// --------------------------------------------------------------------------
// backward
// --------------------------------------------------------------------------

// Sorted samples of a chunk that has few to a span are taken as they come, one
// to a lane, as items would hold one or two of them: no span order, no items.
// 16384 cubic curves of 64 control points x 64 samples 34 us (42 in items, 62
// with the kernel before items), 2048 of 240 x 512 31 (37; 27).
__host__ __device__ inline bool curve_direct(int chunk, int spans) { return chunk <= 4 * spans; }

// Waves of a backward workgroup, by the samples of its chunk and the spans (the
// batch must not decide: the waves fix the order of the sums).  Samples taken
// as they come: a pass or two over them.  Items: enough waves that a lane's
// item holds several samples, few enough that a pass over the items fills
// every one, and with one wave the workgroup's barriers cost nothing (16384
// cubic curves of 32 control points x 384 samples: 62 us with one wave, 89 with
// two, 146 with four; x 1024: 123 with two, 179 with four; 64 curves x 256: 12,
// 11, 10.5).  Long polygons fill four with fewer samples (2048 of 240 x 1024: 42
// us, 57 with two).
inline int curve_waves(int chunk, int spans) {
    if (curve_direct(chunk, spans)) return chunk <= kWave ? 1 : chunk <= 2 * kWave ? 2 : 4;
    if (spans >= 128 && chunk <= 8 * spans) return 4;
    return chunk <= 384 ? 1 : chunk <= 1024 ? 2 : 4;
}

// The workgroup's LDS (dynamic, sized by the curve's control points).
struct CurveLds {
    float4 *pw;       // [nc] control points (xyz, w)
    float4 *acc;      // [waves][nc]: (dL/dP xyz, dL/dw)
    float *U, *acck;  // [nU], [waves][nU]
    float *us;        // [chunk] parameters, clamped into the domain
    int *first;       // [spans + 1]: first sample (in span order) of each span
    int *item;        // [spans + 1]: first item of each span
    int *hist;        // [waves][spans]: unsorted parameters only
    int *wsum;        // [waves]
    unsigned short *perm;  // [chunk]: unsorted parameters only
};
__host__ __device__ inline size_t curve_lds_bytes(int waves, int nc, int p, int chunk) {
    const size_t nU = nc + p + 1, ns = nc - p;
    return 16 * (size_t)nc * (1 + waves) + 4 * nU * (1 + waves) + 4 * (2 * (ns + 1) + waves * (ns + 1)) +
           6 * (size_t)chunk;
}
template <int W>
__device__ __forceinline__ CurveLds curve_lds(char* base, int nc, int p, int chunk) {
    const int nU = nc + p + 1, ns = nc - p;
    CurveLds l;
    l.pw = reinterpret_cast<float4*>(base);
    l.acc = l.pw + nc;
    l.U = reinterpret_cast<float*>(l.acc + W * nc);
    l.acck = l.U + nU;
    l.us = l.acck + W * nU;
    l.first = reinterpret_cast<int*>(l.us + chunk);
    l.item = l.first + ns + 1;
    l.hist = l.item + ns + 1;
    l.wsum = l.hist + W * ns;
    l.perm = reinterpret_cast<unsigned short*>(l.wsum + W);
    return l;
}

// Exclusive prefix over the spans' counts n(0), n(1), ..., n(spans - 1) into
// out[0 .. spans], out[spans] the total.
template <int W, class N>
__device__ __forceinline__ int span_prefix(const CurveLds& l, int spans, int* out, const N& n) {
    const int t = threadIdx.x;
    int all = 0;
    for (int c0 = 0; c0 < spans; c0 += W * kWave) {
        const int v = c0 + t < spans ? n(c0 + t) : 0;
        int x = v;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int y = __shfl_up(x, d);
            if (lane_id() >= d) x += y;
        }
        int sum = 0;
        if constexpr (W == 1) {
            sum = bcast_lane(x, kWave - 1);
        } else {
            __syncthreads();
            if (lane_id() == kWave - 1) l.wsum[t / kWave] = x;
            __syncthreads();
            int before = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                if (w < t / kWave) before += l.wsum[w];
                sum += l.wsum[w];
            }
            x += before;
        }
        if (c0 + t < spans) out[c0 + t] = all + x - v;
        all += sum;
    }
    if (t == 0) out[spans] = all;
    __syncthreads();
    return all;
}

// Whether the chunk's n parameters (l.us) are sorted.
template <int W>
__device__ __forceinline__ bool curve_sorted(const CurveLds& l, int p, int nc, int n) {
    constexpr int kT = W * kWave;
    const int t = threadIdx.x, spans = nc - p;
    bool bad = false;
    for (int s = t + 1; s < n; s += kT) bad |= !(l.us[s - 1] <= l.us[s]);
    // knots out of order (only flagged, under NURBS_VALIDATE) go by find_span,
    // which stays in range whatever they are
    for (int c = t; c < spans; c += kT) bad |= !(l.U[p + c] <= l.U[p + c + 1]);
    if (t == 0) bad |= !(l.U[nc - 1] < l.U[nc]);
    return !__syncthreads_or(bad);
}

// Put the chunk's n samples (l.us) in span order: l.first, and l.perm when the
// parameters are not sorted.  The order within a span is the input's.
template <int W>
__device__ __forceinline__ void curve_order(const CurveLds& l, int p, int nc, int n, bool sorted) {
    constexpr int kT = W * kWave;
    const int t = threadIdx.x, spans = nc - p, wv = t / kWave, lane = lane_id();
    if (sorted) {
        // sorted: a span starts at the first sample not below its knot, one
        // search per knot instead of one per sample; an empty span starts
        // where the next one does
        for (int c = t; c <= spans; c += kT) {
            const float x = l.U[p + c];
            int lo = c == spans ? n : 0, hi = n;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (l.us[mid] < x) lo = mid + 1; else hi = mid;
            }
            l.first[c] = lo;
        }
        __syncthreads();
        return;
    }
    // stable counting sort: each wave takes its part of the samples
    auto span_of = [&](int s) { return find_span(l.U, p, nc - 1, l.us[s]) - p; };
    for (int i = t; i < W * spans; i += kT) l.hist[i] = 0;
    __syncthreads();
    const int per = (n + kT - 1) / kT * kWave;
    const int q0 = min(n, wv * per), q1 = min(n, q0 + per);
    int* h = l.hist + wv * spans;
    for (int s = q0 + lane; s < q1; s += kWave) atomicAdd(h + span_of(s), 1);
    __syncthreads();
    span_prefix<W>(l, spans, l.first, [&](int c) {
        int x = 0;
        for (int w = 0; w < W; ++w) x += l.hist[w * spans + c];
        return x;
    });
    for (int c = t; c < spans; c += kT) {
        int at = l.first[c];
        for (int w = 0; w < W; ++w) {
            const int x = l.hist[w * spans + c];
            l.hist[w * spans + c] = at;
            at += x;
        }
    }
    __syncthreads();
    int bits = 0;
    while ((1 << bits) < spans) ++bits;
    for (int s = q0; s < q1; s += kWave) {
        const bool act = s + lane < q1;
        const int k = act ? span_of(s + lane) : 0;
        // lanes of the same span
        unsigned long long m = __ballot(act);
        for (int i = 0; i < bits; ++i) {
            const bool bit = (k >> i) & 1;
            const unsigned long long v = __ballot(bit);
            m &= bit ? v : ~v;
        }
        const int rank = __popcll(m & ((1ull << lane) - 1ull));
        const int base = h[k];
        wave_lds_sync();
        if (act && rank == 0) h[k] = base + __popcll(m);
        wave_lds_sync();
        if (act) l.perm[base + rank] = (unsigned short)(s + lane);
    }
    __syncthreads();
}

// Cut the spans into items of samples, l.item; returns their number.
// A lane's samples share their span, so the span's knots, reciprocals and
// control points are read once for all of them and the sums over them stay in
// registers; the scan over the wave and the LDS adds come once per 64 items.
// The length is the least that fills the waves once (a multiple of that for
// curves of many spans): an item more than the lanes would cost a whole pass.
// The room is more than twice the spans used, so that the second length is
// about a span's average and not all of its samples.
template <int W>
__device__ __forceinline__ int curve_items(const CurveLds& l, int spans, int n) {
    constexpr int kT = W * kWave;
    int used = 0;
    for (int c0 = 0; c0 < spans; c0 += kT) {
        const int c = c0 + (int)threadIdx.x;
        used += __syncthreads_count(c < spans && l.first[c + 1] > l.first[c]);
    }
    const int room = kT * ((2 * used + kT) / kT);  // more than twice the spans used
    // half an item lost per span, none with one sample to an item
    int len = n <= room ? 1 : (2 * n + 2 * room - used - 1) / (2 * room - used);
    auto count = [&](int c) { return (l.first[c + 1] - l.first[c] + len - 1) / len; };
    int nitems = span_prefix<W>(l, spans, l.item, count);
    if (nitems > room) {
        len = (n + room - used - 1) / (room - used);  // a whole one: fits
        nitems = span_prefix<W>(l, spans, l.item, count);
    }
    return nitems;
}

// One sample's parameter (from LDS) and dL/dC.
template <int DIM>
struct CurveSample {
    float u, g[3];
    __device__ __forceinline__ void load(const float* us, const float* gpts, int s) {
        u = us[s];
        const float* p = gpts + (size_t)s * DIM;
        if constexpr (DIM == 3) {
            const float3u v = *reinterpret_cast<const float3u*>(p);
            g[0] = v.x;
            g[1] = v.y;
            g[2] = v.z;
        } else {
            g[0] = p[0];
            g[1] = p[1];
            g[2] = 0.f;
        }
    }
};

// The scan over the wave multiplies what comes from another run by 0, which a
// NaN or an infinity survives: then the wave takes a scan that selects, so such
// a value reaches its own span's sums and no others.
template <int P1, int K>
__device__ __forceinline__ bool wave_finite(const float4 (&c)[P1], const float (&g)[K]) {
    float z = 0.f;
#pragma unroll
    for (int r = 0; r < P1; ++r)
        z = __builtin_fmaf(c[r].x, 0.f, __builtin_fmaf(c[r].y, 0.f,
            __builtin_fmaf(c[r].z, 0.f, __builtin_fmaf(c[r].w, 0.f, z))));
#pragma unroll
    for (int t = 0; t < K; ++t) z = __builtin_fmaf(g[t], 0.f, z);
    return __ballot(z != 0.f) == 0ull;
}

template <int P1, int K>
__device__ __forceinline__ void seg_scan_select(float4 (&c)[P1], float (&g)[K], const Runs& rn) {
    const int lane = lane_id();
    // first lane of the run: the one after the last run end below this lane
    const unsigned long long ends = __ballot(rn.head) & ((1ull << lane) - 1ull);
    const int first = ends ? kWave - __builtin_clzll(ends) : 0;
#pragma unroll 1
    for (int d = 1; d < kWave; d <<= 1) {
        const bool in = lane - d >= first;
        auto step = [&](float& x) {
            const float y = __shfl_up(x, d);
            if (in) x += y;
        };
#pragma unroll
        for (int r = 0; r < P1; ++r) {
            step(c[r].x);
            step(c[r].y);
            step(c[r].z);
            step(c[r].w);
        }
#pragma unroll
        for (int t = 0; t < K; ++t) step(g[t]);
    }
}

// What bounds it: VALU issue of the per-sample work (basis, curve point,
// adjoint): about 150 instructions a step, 7.2e7 wave instructions (117 us of
// issue) for 16384 cubic space curves of 32 control points x 1024 samples,
// 152 us in all.  One sample per lane with a wave-wide scan and LDS adds for
// every 64 samples, a search per sample and the adjoint's reciprocals taken
// twice took 270-300 us.  Items of a lane's own consecutive samples, so that
// its reads lie hundreds of bytes from its neighbours': 155 us (at degree 1,
// 64 control points, 4096 x 4096 samples 285 us a pass against 160); dL/dC
// staged in LDS: 189 us (fewer workgroups resident).  A loop that ends by a
// vote of the lanes instead of the wave's longest item, counted before it: 240
// us a pass against 204.  Parameters in random order (4096 quartic curves x
// 1000 samples): 847 -> 112 us a pass.
// Degree 5 is held to three waves per SIMD (168 registers, no spills; 181 and two
// waves otherwise): 16384 curves of 32 control points x 1024 samples 262 -> 218 us.
template <int P, int DIM, int W>
__global__ void __launch_bounds__(W* kWave, P == 5 ? 3 : 1) k_curve_bwd(CurveArgs a, const float* __restrict__ gpts,
                                                        float* __restrict__ gctrl, float* __restrict__ gw,
                                                        float* __restrict__ gk, float* __restrict__ part,
                                                        unsigned mask) {
    extern __shared__ float4 curve_dyn[];
    constexpr int kT = W * kWave;
    const CurveBlock b = curve_block(a);
    const int nU = a.nc + P + 1, spans = a.nc - P, n = b.s1 - b.s0;
    const CurveLds l = curve_lds<W>(reinterpret_cast<char*>(curve_dyn), a.nc, P, min(a.ns, kCurveChunk));
    const float* us = a.us + (a.u_shared ? 0 : (size_t)b.c * a.ns);
    stage_curve<DIM>(a, P, b.c, l.U, l.pw);
    const float* kn = a.knots + (size_t)b.c * nU;
    const float ulo = kn[P], uhi = kn[a.nc];
    for (int i = threadIdx.x; i < n; i += kT) l.us[i] = fminf(fmaxf(us[b.s0 + i], ulo), uhi);
    const float* g0 = gpts + ((size_t)b.c * a.ns + b.s0) * DIM;
    for (int i = threadIdx.x; i < W * a.nc; i += kT) l.acc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = threadIdx.x; i < W * nU; i += kT) l.acck[i] = 0.f;
    __syncthreads();
    if (a.err) curve_validate(a, P, b.c, b.chunk, b.s0, b.s1, l.U, a.w + (size_t)b.c * a.nc, us);
    const bool in_order = curve_sorted<W>(l, P, a.nc, n);
    const bool direct = in_order && curve_direct(min(a.ns, kCurveChunk), spans);
    int nitems = n;
    if (!direct) {
        curve_order<W>(l, P, a.nc, n, in_order);
        nitems = curve_items<W>(l, spans, n);
    }
    const bool want_k = (mask & NURBS_GRAD_KU) != 0;
    const int wv = threadIdx.x / kWave;
    const int lane = lane_id();
    float4* acc = l.acc + wv * a.nc;
    float* acck = l.acck + wv * nU;
    constexpr int kSentinel = 1 << 20;  // span of lanes past the last item
    for (int base = wv * kWave; base < nitems; base += kT) {
        const bool act = base + lane < nitems;
        const int it = min(base + lane, nitems - 1);
        // the item's span (the last one that starts at or before it), its m
        // items and the end j1 of its samples.  The items of a span take its
        // samples in turn, so that their lanes read neighbouring samples at
        // each step.
        int lo = 0, m = 1, i = it, j1 = it + 1;
        if (direct) {
            lo = find_span(l.U, P, a.nc - 1, l.us[it]) - P;
        } else {
            int hi = spans;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (l.item[mid] <= it) lo = mid; else hi = mid;
            }
            m = l.item[lo + 1] - l.item[lo];
            i = l.first[lo] + it - l.item[lo];
            j1 = l.first[lo + 1];
        }
        const int k = lo + P;
        float K[2 * P], inv[P * (P + 1) / 2];
#pragma unroll
        for (int t = 0; t < 2 * P; ++t) K[t] = l.U[k - P + 1 + t];
        span_inv<P>(K, inv);
        float4 q[P + 1];
#pragma unroll
        for (int r = 0; r <= P; ++r) q[r] = l.pw[k - P + r];
        // per control point r of the span: (dL/dP xyz, dL/dw); per knot of its window
        float4 c4[P + 1];
        float gU[2 * P];
#pragma unroll
        for (int r = 0; r <= P; ++r) c4[r] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int t = 0; t < 2 * P; ++t) gU[t] = 0.f;
        // steps of the wave's longest item
        int steps = act ? (j1 - i + m - 1) / m : 0;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) steps = max(steps, __shfl_xor(steps, d));
        steps = uniform(steps);
        // one sample ahead: the loads of the next overlap the current one's work
        CurveSample<DIM> nx;
        nx.load(l.us, g0, in_order ? i : (int)l.perm[i]);
#pragma unroll 1
        for (int j = 0; j < steps; ++j, i += m) {
            const CurveSample<DIM> x = nx;
            const int ni = min(i + m, j1 - 1);
            nx.load(l.us, g0, in_order ? ni : (int)l.perm[ni]);
            if (i >= j1 || !act) continue;  // no sample for this lane
            const float u = x.u;
            float N[P + 1], st[P * (P + 1) / 2];
            span_basis<P>(K, inv, u, N, st);
            float Wsum = 0.f, C[3] = {0.f, 0.f, 0.f}, Nw[P + 1];
#pragma unroll
            for (int r = 0; r <= P; ++r) {
                Nw[r] = N[r] * q[r].w;
                Wsum += Nw[r];
                C[0] = __builtin_fmaf(Nw[r], q[r].x, C[0]);
                C[1] = __builtin_fmaf(Nw[r], q[r].y, C[1]);
                if constexpr (DIM == 3) C[2] = __builtin_fmaf(Nw[r], q[r].z, C[2]);
            }
            const float ic = recip(Wsum);
            const float h[3] = {x.g[0] * ic, x.g[1] * ic, x.g[2] * ic};
#pragma unroll
            for (int d = 0; d < DIM; ++d) C[d] *= ic;
            float e[P + 1];
#pragma unroll
            for (int r = 0; r <= P; ++r) {
                float pg = (q[r].x - C[0]) * h[0];
                pg = __builtin_fmaf(q[r].y - C[1], h[1], pg);
                if constexpr (DIM == 3) pg = __builtin_fmaf(q[r].z - C[2], h[2], pg);
                c4[r].x = __builtin_fmaf(Nw[r], h[0], c4[r].x);
                c4[r].y = __builtin_fmaf(Nw[r], h[1], c4[r].y);
                if constexpr (DIM == 3) c4[r].z = __builtin_fmaf(Nw[r], h[2], c4[r].z);
                c4[r].w = __builtin_fmaf(N[r], pg, c4[r].w);
                e[r] = q[r].w * pg;
            }
            if (want_k) {
                span_adjoint<P>(K, inv, u, st, e, gU);
            }
        }
        // runs of lanes on one span: DPP segmented scans, then the last lane
        // of each run adds the run's sums; for a fixed r the run ends touch
        // distinct control points
        const Runs rn = wave_runs(act ? k : kSentinel);
        if (wave_finite(c4, gU)) {
#pragma unroll
            for (int r = 0; r <= P; ++r) seg_scan4(c4[r], rn);
            if (want_k) {
#pragma unroll
                for (int t = 0; t < 2 * P; t += 2) seg_scan2(gU[t], gU[t + 1], rn);
            }
        } else {
            seg_scan_select(c4, gU, rn);
        }
        const bool wr = rn.head && act;
#pragma unroll
        for (int r = 0; r <= P; ++r) {
            if (wr) {
                float4 v = acc[k - P + r];
                v.x += c4[r].x;
                v.y += c4[r].y;
                if constexpr (DIM == 3) v.z += c4[r].z;
                v.w += c4[r].w;
                acc[k - P + r] = v;
            }
            wave_lds_sync();
        }
        if (want_k) {
#pragma unroll
            for (int t = 0; t < 2 * P; ++t) {
                if (wr) acck[k - P + 1 + t] += gU[t];
                wave_lds_sync();
            }
        }
    }
    __syncthreads();
    // the chunk's totals, waves added in order
    const bool one = a.nchunks == 1;
    float* pc = one ? nullptr : part + ((size_t)b.c * a.nchunks + b.chunk) * a.part_floats;
    for (int i = threadIdx.x; i < a.nc; i += kT) {
        float4 v = l.acc[i];
#pragma unroll
        for (int w2 = 1; w2 < W; ++w2) {
            const float4 o = l.acc[w2 * a.nc + i];
            v.x += o.x;
            v.y += o.y;
            v.z += o.z;
            v.w += o.w;
        }
        if (one) {
            const size_t ci = (size_t)b.c * a.nc + i;
            if (mask & NURBS_GRAD_CTRL) {
                gctrl[ci * DIM] = v.x;
                gctrl[ci * DIM + 1] = v.y;
                if constexpr (DIM == 3) gctrl[ci * DIM + 2] = v.z;
            }
            if (mask & NURBS_GRAD_W) gw[ci] = v.w;
        } else {
            reinterpret_cast<float4*>(pc)[i] = v;
        }
    }
    if (want_k) {
        for (int t = threadIdx.x; t < nU; t += kT) {
            float v = l.acck[t];
#pragma unroll
            for (int w2 = 1; w2 < W; ++w2) v += l.acck[w2 * nU + t];
            if (one) gk[(size_t)b.c * nU + t] = v;
            else pc[4 * a.nc + t] = v;
        }
    }
}

// Multi-chunk curves: gradient entry e of curve c is the sum of its chunk
// partials in chunk order.  One thread per (curve, entry).
template <int DIM>
__global__ void __launch_bounds__(kWG) k_curve_fin(CurveArgs a, int p, const float* __restrict__ part,
                                                   float* __restrict__ gctrl, float* __restrict__ gw,
                                                   float* __restrict__ gk, unsigned mask) {
    const int nU = a.nc + p + 1;
    const int per = a.nc + nU;
    const long long id = (long long)blockIdx.x * kWG + threadIdx.x;
    if (id >= (long long)a.B * per) return;
    const int c = (int)(id / per), e = (int)(id - (long long)c * per);
    const float* pc = part + (size_t)c * a.nchunks * a.part_floats;
    if (e < a.nc) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int ch = 0; ch < a.nchunks; ++ch) {
            const float4 o = reinterpret_cast<const float4*>(pc + (size_t)ch * a.part_floats)[e];
            v.x += o.x;
            v.y += o.y;
            v.z += o.z;
            v.w += o.w;
        }
        const size_t ci = (size_t)c * a.nc + e;
        if (mask & NURBS_GRAD_CTRL) {
            gctrl[ci * DIM] = v.x;
            gctrl[ci * DIM + 1] = v.y;
            if constexpr (DIM == 3) gctrl[ci * DIM + 2] = v.z;
        }
        if (mask & NURBS_GRAD_W) gw[ci] = v.w;
    } else if (mask & NURBS_GRAD_KU) {
        const int t = e - a.nc;
        float v = 0.f;
        for (int ch = 0; ch < a.nchunks; ++ch) v += pc[(size_t)ch * a.part_floats + 4 * a.nc + t];
        gk[(size_t)c * nU + t] = v;
    }
}

template <int P, int DIM>
hipError_t curve_fwd_launch(const CurveArgs& a, hipStream_t st, float* pts, float* du) {
    const dim3 grid((unsigned)((long long)a.B * a.nchunks));
    constexpr bool kMayTab = P <= kCurveTabDeg;
    if (du) hipLaunchKernelGGL((k_curve_fwd<P, DIM, true, false>), grid, dim3(kWG), 0, st, a, pts, du);
    else if (kMayTab && curve_tab(P, a.ns))
        hipLaunchKernelGGL((k_curve_fwd<P, DIM, false, kMayTab>), grid, dim3(kWG), 0, st, a, pts, du);
    else hipLaunchKernelGGL((k_curve_fwd<P, DIM, false, false>), grid, dim3(kWG), 0, st, a, pts, du);
    return hipGetLastError();
}

template <int P, int DIM, int W>
void curve_bwd_kernel(const CurveArgs& a, hipStream_t st, const float* gpts, float* gctrl, float* gw, float* gk,
                      float* part, unsigned mask) {
    const dim3 grid((unsigned)((long long)a.B * a.nchunks));
    const size_t lds = curve_lds_bytes(W, a.nc, P, std::min(a.ns, kCurveChunk));
    hipLaunchKernelGGL((k_curve_bwd<P, DIM, W>), grid, dim3(W * kWave), lds, st, a, gpts, gctrl, gw, gk, part, mask);
}

template <int P, int DIM>
hipError_t curve_bwd_launch(const CurveArgs& a, hipStream_t st, const float* gpts, float* gctrl, float* gw,
                            float* gk, float* part, unsigned mask) {
    const int w = curve_waves(std::min(a.ns, kCurveChunk), a.nc - P);
    if (w == 1) curve_bwd_kernel<P, DIM, 1>(a, st, gpts, gctrl, gw, gk, part, mask);
    else if (w == 2) curve_bwd_kernel<P, DIM, 2>(a, st, gpts, gctrl, gw, gk, part, mask);
    else curve_bwd_kernel<P, DIM, 4>(a, st, gpts, gctrl, gw, gk, part, mask);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.nchunks == 1) return e;
    const long long items = (long long)a.B * (2 * a.nc + P + 1);
    hipLaunchKernelGGL((k_curve_fin<DIM>), dim3((unsigned)((items + kWG - 1) / kWG)), dim3(kWG), 0, st, a, P, part,
                       gctrl, gw, gk, mask);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_curve_fwd(int p, int dim, hipStream_t st, const CurveArgs& a, float* pts, float* du) {
    switch (p * 4 + dim) {
#define C(P)                                                     \
    case P * 4 + 2: return curve_fwd_launch<P, 2>(a, st, pts, du); \
    case P * 4 + 3: return curve_fwd_launch<P, 3>(a, st, pts, du);
        C(1) C(2) C(3) C(4) C(5) C(6) C(7)
#undef C
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_curve_bwd(int p, int dim, hipStream_t st, const CurveArgs& a, const float* gpts, float* gctrl,
                            float* gw, float* gk, float* part, unsigned mask) {
    switch (p * 4 + dim) {
#define C(P)                                                                               \
    case P * 4 + 2: return curve_bwd_launch<P, 2>(a, st, gpts, gctrl, gw, gk, part, mask); \
    case P * 4 + 3: return curve_bwd_launch<P, 3>(a, st, gpts, gctrl, gw, gk, part, mask);
        C(1) C(2) C(3) C(4) C(5) C(6) C(7)
#undef C
        default: return hipErrorInvalidValue;
    }
}

}  // namespace nd
