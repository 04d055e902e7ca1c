// Backward of surfaces at scattered parameter pairs, over pairs ordered by
// cell.  A cell is a pair of knot spans: its pairs touch the same
// (p+1)(q+1) control points and the same 2p + 2q knots, so their terms are
// summed in registers, and a control point's gradient is the sum over the
// (p+1)(q+1) cells that touch it.  With h = g / W (h_w = -(S - c).g / W, c a
// control point of the cell) a cell needs only
//   M_rh = sum_k Nu_r(k) Nv_h(k) h(k)   (4 values per control point)
//   dP = w M_xyz,   dw = (P - c) . M_xyz + M_w  (eqs. NURBSuDerivative4, 5)
// and the knot adjoints of its pairs (eq. NURBSvDerivative6, Sec. 3.2.1).
// The frame c keeps the two parts of dw as small as the cell.
//
//   k_uv_hist   each pair's cell; pairs per (chunk, cell)
//   k_uv_scan   prefix over chunks, then over cells; cells cut into items of
//               at most `seg` pairs
//   k_uv_order  stable order by cell: pair indices, one wave per chunk
//   k_uv_cell   one wave per item: sums of its pairs, in FP64
//   k_uv_sum    sums over items in a fixed order, in FP64
//
// The order within a cell is the input's, so every sum has a fixed order and
// results are bitwise reproducible, with no atomics on results and no pass to
// find a fixed-point scale.  What bounds it: k_uv_cell's per-pair VALU work
// (span basis, the two contractions of the patch, the knot adjoints); the sums
// M are on the matrix cores in FP64 (v_mfma_f64_4x4x4, 16 to a wave's 64
// bicubic pairs), where the atomic path has 80 64-bit LDS atomics a pair, as
// many conversions and a second evaluation of every term.  Measured, forward
// and backward: 64 bicubic 16 x 16 surfaces x 65536 pairs 238 us (atomic path
// 585 us), of them k_uv_cell 125, k_uv_order 33, k_uv_hist 16, k_uv_sum 13,
// k_uv_scan 9, the forward 48; one surface of degree (4, 5), 48 x 41 net, 50001
// pairs 122 to 140 us, most of it the host (1.81 ms, its accumulators did not
// fit in LDS).  With M summed on the VALU (one output per lane) k_uv_cell took
// 138 us, without the next pairs' loads in flight 144; k_uv_sum 37 us with one
// thread to a control point's value, 19 with one item's load in flight;
// k_uv_hist and k_uv_scan 18 and 13 us with 128 chunks to a surface instead of
// 64.  Largest relative error (2-norm) of a gradient against 64 bits, on the
// same inputs: 1.9e-7 and 1.7e-7 (atomic path 5.9e-7 and 5.7e-7).
#include "device.hpp"
#include "launch.hpp"
#include "../../include/nurbsdiff.h"

#include <algorithm>

namespace nd {
namespace {

// The (tables of the) group's surfaces: index b within the group.
struct SortPtrs {
    unsigned* hist;        // [group][nchunk][cells]: pairs, then their prefix over chunks
    int* cell_start;       // [group][cells + 1]
    int* item_start;       // [group][cells + 1]
    int* item_cell;        // [group][items]
    unsigned* order;       // [group][npts]
    unsigned short* cell;  // [group][npts]
    double* slots;         // [group][items][slot]
};

// --------------------------------------------------------------------------
// ordering
// --------------------------------------------------------------------------
__global__ void __launch_bounds__(kWG) k_uv_hist(UvArgs a, UvSort s, SortPtrs t, int b0) {
    extern __shared__ unsigned hist[];
    __shared__ float lku[kWG], lkv[kWG];
    const int g = blockIdx.y, b = b0 + g, tid = threadIdx.x;
    const int nU = a.nu_c + a.p + 1, nV = a.nv_c + a.q + 1;
    const float* gku = a.ku + (size_t)b * nU;
    const float* gkv = a.kv + (size_t)b * nV;
    for (int i = tid; i < nU; i += kWG) lku[i] = gku[i];
    for (int i = tid; i < nV; i += kWG) lkv[i] = gkv[i];
    for (int i = tid; i < s.cells; i += kWG) hist[i] = 0u;
    __syncthreads();
    const float* uv = a.uv + (a.uv_shared ? 0 : (size_t)b * a.npts * 2);
    const int k0 = blockIdx.x * s.chunk, k1 = min(a.npts, k0 + s.chunk);
    if (a.err) {
        bool bad_k = false, bad_w = false, bad_d = false;
        if (blockIdx.x == 0) {
            for (int i = tid; i + 1 < nU; i += kWG) bad_k |= !(lku[i] <= lku[i + 1]);
            for (int i = tid; i + 1 < nV; i += kWG) bad_k |= !(lkv[i] <= lkv[i + 1]);
            if (tid == 0)
                bad_k |= !(lku[a.p] < lku[a.p + 1]) || !(lku[a.nu_c - 1] < lku[a.nu_c]) ||
                         !(lkv[a.q] < lkv[a.q + 1]) || !(lkv[a.nv_c - 1] < lkv[a.nv_c]);
            const float* w = a.w + (size_t)b * a.nu_c * a.nv_c;
            for (int i = tid; i < a.nu_c * a.nv_c; i += kWG) bad_w |= !(w[i] > 0.f);
        }
        for (int k = k0 + tid; k < k1; k += kWG) {
            const float u = uv[2 * (size_t)k], v = uv[2 * (size_t)k + 1];
            bad_d |= !(u >= lku[a.p] && u <= lku[a.nu_c] && v >= lkv[a.q] && v <= lkv[a.nv_c]);
        }
        if (bad_k) atomicCAS(a.err, 0, NURBS_EKNOTS);
        if (bad_w) atomicCAS(a.err, 0, NURBS_EWEIGHTS);
        if (bad_d) atomicCAS(a.err, 0, NURBS_EDOMAIN);
    }
    for (int k = k0 + tid; k < k1; k += kWG) {
        const float2 x = *reinterpret_cast<const float2*>(uv + 2 * (size_t)k);
        const int ku = find_span(lku, a.p, a.nu_c - 1, clamp_param(lku, a.p, a.nu_c - 1, x.x));
        const int kv = find_span(lkv, a.q, a.nv_c - 1, clamp_param(lkv, a.q, a.nv_c - 1, x.y));
        const int c = (ku - a.p) * s.ncv + (kv - a.q);
        t.cell[(size_t)g * a.npts + k] = (unsigned short)c;
        atomicAdd(hist + c, 1u);
    }
    __syncthreads();
    unsigned* o = t.hist + ((size_t)g * s.nchunk + blockIdx.x) * s.cells;
    for (int i = tid; i < s.cells; i += kWG) o[i] = hist[i];
}

// One workgroup per surface, of four waves up to 1024 cells (2000 surfaces of 9
// cells: 59 us with sixteen), sixteen beyond.  cells <= 4 WG <= kUvCellsMax.
constexpr int kScanPer = 4;
template <int WG>
__global__ void __launch_bounds__(WG) k_uv_scan(UvSort s, SortPtrs t) {
    constexpr int kCells = kScanPer * WG;
    __shared__ int tot[kCells];
    __shared__ int2 wsum[WG / kWave];
    const int g = blockIdx.x, tid = threadIdx.x;
    unsigned* h = t.hist + (size_t)g * s.nchunk * s.cells;
    for (int c = tid; c < kCells; c += WG) {
        unsigned run = 0;
        if (c < s.cells) {
            constexpr int kU = 32;  // chunks in flight
            for (int j0 = 0; j0 < s.nchunk; j0 += kU) {
                unsigned v[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) v[u] = j0 + u < s.nchunk ? h[(size_t)(j0 + u) * s.cells + c] : 0u;
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if (j0 + u < s.nchunk) {
                        h[(size_t)(j0 + u) * s.cells + c] = run;
                        run += v[u];
                    }
            }
        }
        tot[c] = (int)run;
    }
    __syncthreads();
    // exclusive prefix of (pairs, items) over the cells, four per thread
    int n[kScanPer], sum = 0, isum = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        n[i] = tot[tid * kScanPer + i];
        sum += n[i];
        isum += (n[i] + s.seg - 1) / s.seg;
    }
    int x = sum, y = isum;
    for (int d = 1; d < kWave; d <<= 1) {
        const int xo = __shfl_up(x, d), yo = __shfl_up(y, d);
        if (lane_id() >= d) {
            x += xo;
            y += yo;
        }
    }
    if (lane_id() == kWave - 1) wsum[tid / kWave] = make_int2(x, y);
    __syncthreads();
    int at = x - sum, it = y - isum;
    for (int w = 0; w < tid / kWave; ++w) {
        at += wsum[w].x;
        it += wsum[w].y;
    }
    int* cs = t.cell_start + (size_t)g * (s.cells + 1);
    int* is = t.item_start + (size_t)g * (s.cells + 1);
    int* ic = t.item_cell + (size_t)g * s.items;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        const int c = tid * kScanPer + i;
        if (c <= s.cells) {
            cs[c] = at;
            is[c] = it;
        }
        const int ni = (n[i] + s.seg - 1) / s.seg;
        for (int j = 0; j < ni; ++j) ic[it + j] = c;
        at += n[i];
        it += ni;
    }
    if (tid == WG - 1 && s.cells == kCells) {
        cs[s.cells] = at;
        is[s.cells] = it;
    }
}

// One wave per chunk: its pairs in input order, 64 at a time.  The lanes of
// one cell find each other by ballots over the bits of the cell index, the
// cell's counter in LDS gives the first position.
__global__ void __launch_bounds__(kWave) k_uv_order(UvArgs a, UvSort s, SortPtrs t, int bits) {
    extern __shared__ unsigned next[];
    const int g = blockIdx.y, lane = lane_id();
    const unsigned* h = t.hist + ((size_t)g * s.nchunk + blockIdx.x) * s.cells;
    const int* cs = t.cell_start + (size_t)g * (s.cells + 1);
    for (int c = lane; c < s.cells; c += kWave) next[c] = h[c] + (unsigned)cs[c];
    wave_lds_sync();
    const unsigned short* cell = t.cell + (size_t)g * a.npts;
    unsigned* order = t.order + (size_t)g * a.npts;
    const int k0 = blockIdx.x * s.chunk, k1 = min(a.npts, k0 + s.chunk);
    // eight rows of 64 pairs fetched together
    constexpr int kU = 8;
    for (int kk = k0; kk < k1; kk += kU * kWave) {
        int cs8[kU];
#pragma unroll
        for (int i = 0; i < kU; ++i) cs8[i] = (int)cell[min(kk + i * kWave + lane, k1 - 1)];
#pragma unroll
        for (int row = 0; row < kU; ++row) {
            const int k = kk + row * kWave;
            if (k >= k1) break;
            const bool act = k + lane < k1;
            const int c = act ? cs8[row] : 0;
            unsigned long long m = __ballot(act);
            for (int i = 0; i < bits; ++i) {
                const bool bit = (c >> i) & 1;
                const unsigned long long v = __ballot(bit);
                m &= bit ? v : ~v;
            }
            const int rank = __popcll(m & ((1ull << lane) - 1ull));
            const unsigned base = next[c];
            wave_lds_sync();
            if (act && rank == 0) next[c] = base + (unsigned)__popcll(m);
            wave_lds_sync();
            if (act) order[base + rank] = (unsigned)(k + lane);
        }
    }
}

// --------------------------------------------------------------------------
// the pairs of an item
// --------------------------------------------------------------------------
template <int DM>
struct SpanTab {
    float K[2 * DM];                 // the span's knot window
    float inv[DM * (DM + 1) / 2];    // its reciprocals
};

#define ND_BY_DEGREE(d, BODY)                                                             \
    switch (d) {                                                                          \
        case 1: if constexpr (1 <= DM) { constexpr int D = 1; BODY } break;               \
        case 2: if constexpr (2 <= DM) { constexpr int D = 2; BODY } break;               \
        case 3: if constexpr (3 <= DM) { constexpr int D = 3; BODY } break;               \
        case 4: if constexpr (4 <= DM) { constexpr int D = 4; BODY } break;               \
        case 5: if constexpr (5 <= DM) { constexpr int D = 5; BODY } break;               \
        case 6: if constexpr (6 <= DM) { constexpr int D = 6; BODY } break;               \
        case 7: if constexpr (7 <= DM) { constexpr int D = 7; BODY } break;               \
        default: break;                                                                   \
    }

template <int DM>
__device__ __forceinline__ void span_load(const float* __restrict__ U, int k, int d, SpanTab<DM>& t) {
#pragma unroll
    for (int i = 0; i < 2 * DM; ++i) t.K[i] = i < 2 * d ? uniform_f(U[k - d + 1 + i]) : 0.f;
    ND_BY_DEGREE(d, span_inv<D>(t.K, t.inv);)
#pragma unroll
    for (int i = 0; i < DM * (DM + 1) / 2; ++i) t.inv[i] = i < d * (d + 1) / 2 ? uniform_f(t.inv[i]) : 0.f;
}

template <int DM>
__device__ __forceinline__ void span_basis_rt(const SpanTab<DM>& t, int d, float x, float N[DM + 1],
                                              float s[DM * (DM + 1) / 2]) {
#pragma unroll
    for (int r = 0; r <= DM; ++r) N[r] = 0.f;
    ND_BY_DEGREE(d, span_basis<D>(t.K, t.inv, x, N, s);)
}

template <int DM>
__device__ __forceinline__ void span_adjoint_rt(const SpanTab<DM>& t, int d, float x,
                                                const float s[DM * (DM + 1) / 2], const float e[DM + 1],
                                                float g[2 * DM]) {
#pragma unroll
    for (int i = 0; i < 2 * DM; ++i) g[i] = 0.f;
    ND_BY_DEGREE(d, span_adjoint<D>(t.K, t.inv, x, s, e, g);)
}

// Row pitch of the 64 pairs' values in LDS: 16-byte rows, 4 banks apart, so
// the 16 rows that a b128 read touches lie in different banks.
constexpr int kPitch = kWave + 4;

template <int PM, int QM>
struct CellLds {
    float4 patch[(PM + 1) * (QM + 1)];  // ((P - c) w, w) of the cell's control points
    float nu[PM + 1][kPitch];
    float tv[4 * (QM + 1)][kPitch];     // Nv_h h_c
};

// Sum of v over the wave's lanes for each of n <= 16 values per lane, in a
// fixed order; lane 4t returns value t's sum.  buf: n rows of kRed doubles.
constexpr int kRed = kWave + 2;
template <int N>
__device__ __forceinline__ double wave_sums(double* buf, const double (&v)[N], int n) {
    static_assert(N <= kWave / 4, "four lanes to a value");
    const int lane = lane_id();
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i < n) buf[i * kRed + lane] = v[i];
    wave_lds_sync();
    double x = 0.0;
    const int row = min(lane >> 2, n - 1);
#pragma unroll
    for (int j = 0; j < kWave / 4; ++j) x += buf[row * kRed + (lane & 3) * (kWave / 4) + j];
    x += __shfl_xor(x, 1);
    x += __shfl_xor(x, 2);
    wave_lds_sync();
    return x;
}

template <int PM, int QM>
__global__ void __launch_bounds__(kWG) k_uv_cell(UvArgs a, UvSort s, SortPtrs t, int b0,
                                                const float* __restrict__ gpts, unsigned mask) {
    __shared__ CellLds<PM, QM> lds_all[kWavesPerWG];
    static_assert(sizeof(CellLds<PM, QM>) - sizeof(float4) * (PM + 1) * (QM + 1) >=
                      sizeof(double) * kRed * 2 * (PM > QM ? PM : QM),
                  "the knot sums reuse the pairs' rows");
    CellLds<PM, QM>& L = lds_all[threadIdx.x / kWave];
    const int g = blockIdx.y, b = b0 + g, lane = lane_id();
    const int item = uniform((int)(blockIdx.x * kWavesPerWG + threadIdx.x / kWave));
    const int* cs = t.cell_start + (size_t)g * (s.cells + 1);
    const int* is = t.item_start + (size_t)g * (s.cells + 1);
    if (item >= is[s.cells]) return;
    const int p = a.p, q = a.q;
    const int cell = uniform(t.item_cell[(size_t)g * s.items + item]);
    const int cu = cell / s.ncv, cv = cell - cu * s.ncv;
    const int s0 = uniform(cs[cell]) + (item - uniform(is[cell])) * s.seg;
    const int s1 = min(s0 + s.seg, uniform(cs[cell + 1]));

    SpanTab<PM> tu;
    SpanTab<QM> tv;
    const int nU = a.nu_c + p + 1, nV = a.nv_c + q + 1;
    span_load<PM>(a.ku + (size_t)b * nU, cu + p, p, tu);
    span_load<QM>(a.kv + (size_t)b * nV, cv + q, q, tv);
    // domain ends, for the clamp
    const float ulo = uniform_f(a.ku[(size_t)b * nU + p]), uhi = uniform_f(a.ku[(size_t)b * nU + a.nu_c]);
    const float vlo = uniform_f(a.kv[(size_t)b * nV + q]), vhi = uniform_f(a.kv[(size_t)b * nV + a.nv_c]);

    // the cell's control points in its frame; lane i < (p+1)(q+1) holds point i
    const int npatch = (p + 1) * (q + 1);
    const size_t cp0 = (size_t)b * a.nu_c * a.nv_c;
    float4 pc;  // (P - c, w) of control point min(lane, npatch - 1)
    {
        const int mid = (cu + (p >> 1)) * a.nv_c + cv + (q >> 1);
        const float* c = a.ctrl + 3 * (cp0 + mid);
        const int i = min(lane, npatch - 1), r = i / (q + 1), h = i - r * (q + 1);
        const size_t ij = cp0 + (size_t)(cu + r) * a.nv_c + cv + h;
        const float* P = a.ctrl + 3 * ij;
        pc = make_float4(P[0] - c[0], P[1] - c[1], P[2] - c[2], a.w[ij]);
        if (lane < npatch) L.patch[lane] = make_float4(pc.x * pc.w, pc.y * pc.w, pc.z * pc.w, pc.w);
    }
    wave_lds_sync();

    const bool want_pw = (mask & (NURBS_GRAD_CTRL | NURBS_GRAD_W)) != 0;
    const bool want_ku = (mask & NURBS_GRAD_KU) != 0, want_kv = (mask & NURBS_GRAD_KV) != 0;
    const float* uvb = a.uv + (a.uv_shared ? 0 : (size_t)b * a.npts * 2);
    const float* gb = gpts + (size_t)b * a.npts * 3;
    const unsigned* order = t.order + (size_t)g * a.npts;

    // M_rh of value c on the matrix cores (v_mfma_f64_4x4x4: four blocks, one per
    // h, of 4 rows r x 4 values c, over 4 pairs): lane l holds row r = l / 16 and
    // column (h, c) = l % 16 of the result, and hands in pair quarter l / 16 of
    // row r = l % 4 and of column l % 16.  Degrees above 3 take more tiles.
    constexpr int kRT = (PM + 4) / 4, kHT = (QM + 4) / 4;
    double acc[kRT][kHT];
#pragma unroll
    for (int i = 0; i < kRT; ++i)
#pragma unroll
        for (int j = 0; j < kHT; ++j) acc[i][j] = 0.0;
    double sku[2 * PM], skv[2 * QM];
#pragma unroll
    for (int i = 0; i < 2 * PM; ++i) sku[i] = 0.0;
#pragma unroll
    for (int i = 0; i < 2 * QM; ++i) skv[i] = 0.0;

    // the next 64 pairs' values and the index of the 64 after them are on the
    // way while the current ones are worked on
    size_t id = order[min(s0 + lane, s1 - 1)];
    float2 nx = *reinterpret_cast<const float2*>(uvb + 2 * id);
    float3u ng = *reinterpret_cast<const float3u*>(gb + 3 * id);
    id = order[min(s0 + kWave + lane, s1 - 1)];
    for (int k = s0; k < s1; k += kWave) {
        const bool act = k + lane < s1;
        const float2 x = nx;
        const float3u gv = ng;
        if (k + kWave < s1) {
            nx = *reinterpret_cast<const float2*>(uvb + 2 * id);
            ng = *reinterpret_cast<const float3u*>(gb + 3 * id);
            id = order[min(k + 2 * kWave + lane, s1 - 1)];
        }
        const float u = fminf(fmaxf(x.x, ulo), uhi), v = fminf(fmaxf(x.y, vlo), vhi);
        const float g0 = act ? gv.x : 0.f, g1 = act ? gv.y : 0.f, g2 = act ? gv.z : 0.f;
        float Nu[PM + 1], Nv[QM + 1], su[PM * (PM + 1) / 2], sv[QM * (QM + 1) / 2];
        span_basis_rt<PM>(tu, p, u, Nu, su);
        span_basis_rt<QM>(tv, q, v, Nv, sv);
        // R_r = sum_h Nv_h Pw_rh, Q_h = sum_r Nu_r Pw_rh
        float4 R[PM + 1], Q[QM + 1], A = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int h = 0; h <= QM; ++h) Q[h] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int r = 0; r <= PM; ++r) {
            R[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r > p) continue;
#pragma unroll
            for (int h = 0; h <= QM; ++h) {
                if (h > q) continue;
                const float4 c = L.patch[r * (q + 1) + h];
                R[r] = fma4(Nv[h], c, R[r]);
                Q[h] = fma4(Nu[r], c, Q[h]);
            }
            A = fma4(Nu[r], R[r], A);
        }
        const float iw = recip(A.w);
        const float h0 = iw * g0, h1 = iw * g1, h2 = iw * g2;
        const float sg = iw * __builtin_fmaf(A.z, h2, __builtin_fmaf(A.y, h1, A.x * h0));  // (S - c).g / W
        if (want_pw) {
            wave_lds_sync();
#pragma unroll
            for (int r = 0; r <= PM; ++r)
                if (r <= p) L.nu[r][lane] = Nu[r];
#pragma unroll
            for (int h = 0; h <= QM; ++h)
                if (h <= q) {
                    L.tv[4 * h][lane] = Nv[h] * h0;
                    L.tv[4 * h + 1][lane] = Nv[h] * h1;
                    L.tv[4 * h + 2][lane] = Nv[h] * h2;
                    L.tv[4 * h + 3][lane] = -(Nv[h] * sg);
                }
            wave_lds_sync();
        }
        if (want_ku) {
            float e[PM + 1], gk[2 * PM];
#pragma unroll
            for (int r = 0; r <= PM; ++r)
                e[r] = __builtin_fmaf(R[r].x, h0, __builtin_fmaf(R[r].y, h1, __builtin_fmaf(R[r].z, h2, -R[r].w * sg)));
            span_adjoint_rt<PM>(tu, p, u, su, e, gk);
#pragma unroll
            for (int i = 0; i < 2 * PM; ++i) sku[i] += (double)gk[i];
        }
        if (want_kv) {
            float f[QM + 1], gk[2 * QM];
#pragma unroll
            for (int h = 0; h <= QM; ++h)
                f[h] = __builtin_fmaf(Q[h].x, h0, __builtin_fmaf(Q[h].y, h1, __builtin_fmaf(Q[h].z, h2, -Q[h].w * sg)));
            span_adjoint_rt<QM>(tv, q, v, sv, f, gk);
#pragma unroll
            for (int i = 0; i < 2 * QM; ++i) skv[i] += (double)gk[i];
        }
        if (want_pw) {
            // pairs past the item's end hold h = 0; rows past the degree hold 0
            // too, or reach only values that are not kept
            const int quarter = lane >> 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float4 x4[kRT], y4[kHT];
#pragma unroll
                for (int i = 0; i < kRT; ++i)
                    x4[i] = *reinterpret_cast<const float4*>(&L.nu[min(4 * i + (lane & 3), PM)][16 * quarter + 4 * j]);
#pragma unroll
                for (int i = 0; i < kHT; ++i)
                    y4[i] = *reinterpret_cast<const float4*>(
                        &L.tv[min(16 * i + (lane & 15), 4 * QM + 3)][16 * quarter + 4 * j]);
#pragma unroll
                for (int i = 0; i < kRT; ++i)
#pragma unroll
                    for (int h = 0; h < kHT; ++h) {
                        if (4 * i > p || 4 * h > q) continue;
                        acc[i][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(x4[i].x, y4[h].x, acc[i][h], 0, 0, 0);
                        acc[i][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(x4[i].y, y4[h].y, acc[i][h], 0, 0, 0);
                        acc[i][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(x4[i].z, y4[h].z, acc[i][h], 0, 0, 0);
                        acc[i][h] = __builtin_amdgcn_mfma_f64_4x4x4f64(x4[i].w, y4[h].w, acc[i][h], 0, 0, 0);
                    }
            }
        }
    }

    double* out = t.slots + ((size_t)g * s.items + item) * s.slot;
    if (want_pw) {
#pragma unroll
        for (int i = 0; i < kRT; ++i)
#pragma unroll
            for (int j = 0; j < kHT; ++j) {
                // M_x, M_y, M_z, M_w of one control point sit in four neighbouring lanes
                const double M = acc[i][j];
                const int l0 = lane & ~3, r = 4 * i + (lane >> 4), h = 4 * j + ((lane >> 2) & 3);
                const double mx = __shfl(M, l0), my = __shfl(M, l0 + 1), mz = __shfl(M, l0 + 2);
                const bool kept = r <= p && h <= q;
                const int src = kept ? r * (q + 1) + h : 0;
                const float px = __shfl(pc.x, src), py = __shfl(pc.y, src), pz = __shfl(pc.z, src),
                            w = __shfl(pc.w, src);
                const double dw = (double)px * mx + (double)py * my + (double)pz * mz + M;
                if (kept) out[4 * src + (lane & 3)] = (lane & 3) == 3 ? dw : (double)w * M;
            }
    }
    double* buf = reinterpret_cast<double*>(&L.nu[0][0]);
    if (want_ku) {
        const double x = wave_sums<2 * PM>(buf, sku, 2 * p);
        if ((lane & 3) == 0 && (lane >> 2) < 2 * p) out[4 * npatch + (lane >> 2)] = x;
    }
    if (want_kv) {
        const double x = wave_sums<2 * QM>(buf, skv, 2 * q);
        if ((lane & 3) == 0 && (lane >> 2) < 2 * q) out[4 * npatch + 2 * p + (lane >> 2)] = x;
    }
}

// --------------------------------------------------------------------------
// sums over items
// --------------------------------------------------------------------------
// Entry o of every item of cell c, in order.
__device__ __forceinline__ double cell_sum(const int* __restrict__ is, const double* __restrict__ slots, int slot,
                                           int c, int o) {
    double x = 0.0;
    const int end = is[c + 1];
#pragma unroll 8
    for (int i = is[c]; i < end; ++i) x += slots[(size_t)i * slot + o];
    return x;
}

// Grid (blocks, surfaces).  The first cblk workgroups: 4 values x 2^rbits
// (>= p + 1) rows of cells to a control point; the others: one wave per knot, its lanes over the cells.
__global__ void __launch_bounds__(kWG) k_uv_sum(UvArgs a, UvSort s, SortPtrs t, int b0, int cblk, int rbits,
                                               unsigned mask, float* __restrict__ gc, float* __restrict__ gw,
                                               float* __restrict__ gku, float* __restrict__ gkv) {
    const int g = blockIdx.y, b = b0 + g, p = a.p, q = a.q;
    const int ncu = a.nu_c - p, ncv = s.ncv;
    const int* is = t.item_start + (size_t)g * (s.cells + 1);
    const double* slots = t.slots + (size_t)g * s.items * s.slot;
    if ((int)blockIdx.x < cblk) {
        // lanes: value c (4), then row r of the control point's cells (a power
        // of two of them); rows are added in a fixed tree
        const int lanes = 4 << rbits;
        const int e = (int)blockIdx.x * (kWG / lanes) + (int)threadIdx.x / lanes;
        const int c = threadIdx.x & 3, r = (threadIdx.x >> 2) & ((1 << rbits) - 1);
        const int ncp = a.nu_c * a.nv_c, ij = min(e, ncp - 1);
        const int i = ij / a.nv_c, j = ij - i * a.nv_c, cu = i - r;
        double x = 0.0;
        if (r <= p && cu >= 0 && cu < ncu) {
            const int v0 = max(0, j - q), v1 = min(j, ncv - 1), o = 4 * (r * (q + 1) + j) + c;
            int at = is[cu * ncv + v0];
            for (int cv = v0; cv <= v1; ++cv) {
                const int end = is[cu * ncv + cv + 1];
#pragma unroll 8
                for (; at < end; ++at) x += slots[(size_t)at * s.slot + o - 4 * cv];
            }
        }
        for (int d = 4; d < lanes; d <<= 1) x += __shfl_xor(x, d);
        if (e >= ncp || r != 0 || !(mask & (c == 3 ? NURBS_GRAD_W : NURBS_GRAD_CTRL))) return;
        if (c < 3) gc[3 * ((size_t)b * ncp + ij) + c] = (float)x;
        else gw[(size_t)b * ncp + ij] = (float)x;
        return;
    }
    const int nU = a.nu_c + p + 1, nV = a.nv_c + q + 1, lane = lane_id();
    int e = ((int)blockIdx.x - cblk) * kWavesPerWG + (int)threadIdx.x / kWave;
    if (e >= nU + nV) return;
    const bool in_v = e >= nU;
    if (!(mask & (in_v ? NURBS_GRAD_KV : NURBS_GRAD_KU))) return;
    if (in_v) e -= nU;
    // knot e is entry e - 1 - c of the window of span cell c of its direction
    const int d = in_v ? q : p, nc = in_v ? ncv : ncu, other = in_v ? ncu : ncv;
    const int lo = max(0, e - 2 * d), hi = min(nc - 1, e - 1);
    const int base = 4 * (p + 1) * (q + 1) + (in_v ? 2 * p : 0);
    double x = 0.0;
    const int span = hi - lo + 1;
    for (int m = lane; m < span * other; m += kWave) {
        const int c = lo + m / other, o = m % other;
        x += cell_sum(is, slots, s.slot, in_v ? o * ncv + c : c * ncv + o, base + e - 1 - c);
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) x += __shfl_xor(x, m);
    if (lane == 0) (in_v ? gkv + (size_t)b * nV : gku + (size_t)b * nU)[e] = (float)x;
}

template <int PM, int QM>
void launch_cell(dim3 grid, hipStream_t st, const UvArgs& a, const UvSort& s, const SortPtrs& t, int b0,
                 const float* gpts, unsigned mask) {
    hipLaunchKernelGGL((k_uv_cell<PM, QM>), grid, dim3(kWG), 0, st, a, s, t, b0, gpts, mask);
}

}  // namespace

namespace {
constexpr int kLongItems = 32768;  // pairs from which items are longer

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
int sort_slot(int p, int q) { return 4 * (p + 1) * (q + 1) + 2 * p + 2 * q; }

// Tables and slots of one surface; those of G take at most G times as much.
size_t sort_bytes(size_t cells, size_t chunks, size_t items, size_t slot, size_t npts) {
    return al256(4 * chunks * cells) + 2 * al256(4 * (cells + 1)) + al256(4 * items) + al256(4 * npts) +
           al256(2 * npts) + al256(8 * items * slot);
}
}  // namespace

bool uv_sort_plan(int B, int p, int q, int nu_c, int nv_c, int npts, size_t head, UvSort* out) {
    UvSort s{};
    s.ncv = nv_c - q;
    const long long cells = (long long)(nu_c - p) * s.ncv;
    // Where the line lies.  An item costs a wave's pass however few pairs it
    // has, so a full chip wants cells of many pairs; against accumulators in LDS
    // (kUvLdsAccMax) the atomic path is the better one below about 32 to a
    // cell, and at low degrees, where a pair has few atomics, below more.  64
    // surfaces of degree (4, 1), 42 x 13 net: 4095 pairs (9 to a cell) 129 us
    // here, 71 there; (4, 5), 36 x 30, 6618 pairs (8): 244, 150; (2, 4), 19 x 35,
    // 13058 (25): 200, 163; 256 of (3, 3), 16 x 16, 64 to a cell: 238, 411; 256 of
    // (1, 1), 16 x 16, 64 and 256 to a cell: 202, 173 and 408, 581 (a single
    // surface gains from about one pair to a cell on, but what decides must
    // not depend on the batch).  Accumulators in global memory: one pair to a
    // cell is enough (8 surfaces of (3, 3), 60 x 60: 83 us, 184), at degree
    // (1, 1) two (one surface: 58 us, 64; with one pair to a cell 56, 45).
    // Above kUvCellsMax cells the counters of a chunk outgrow their LDS.
    const long long terms = (p + 1) * (q + 1), nacc = 4ll * nu_c * nv_c + nu_c + nv_c + p + q + 2;
    const long long least = nacc <= kUvLdsAccMax ? std::max(32ll, 384 / terms) : std::max(1ll, 8 / terms);
    if (npts < 1 || cells > kUvCellsMax || npts < least * cells) return false;
    s.cells = (int)cells;
    // nothing that fixes the order of a sum depends on B, so that a surface's
    // result does not depend on the batch it is in
    // 64 chunks of 256 to 2048 pairs, more chunks beyond
    const long long c = ((long long)npts + 63) / 64;
    s.chunk = (int)std::min<long long>(2048, std::max<long long>(256, (c + kWave - 1) / kWave * kWave));
    s.nchunk = (npts + s.chunk - 1) / s.chunk;
    s.seg = npts >= kLongItems ? 512 : 128;
    s.items = (int)(std::min<long long>(cells, npts) + npts / s.seg);
    s.slot = sort_slot(p, q);
    const size_t one = sort_bytes(s.cells, s.nchunk, s.items, s.slot, npts);
    s.total = head + group_ws(B, one);
    s.group = (int)std::min<size_t>(B, (s.total - head) / one);
    const size_t G = (size_t)s.group;
    s.hist = head;
    s.cell_start = s.hist + al256(4 * G * s.nchunk * s.cells);
    s.item_start = s.cell_start + al256(4 * G * (s.cells + 1));
    s.item_cell = s.item_start + al256(4 * G * (s.cells + 1));
    s.order = s.item_cell + al256(4 * G * s.items);
    s.cell_of = s.order + al256(4 * G * npts);
    s.slots = s.cell_of + al256(2 * G * npts);
    *out = s;
    return true;
}

size_t uv_sort_asked(int B, int p, int q, int nu_c, int nv_c, int npts, size_t head) {
    if (npts < 1) return 0;
    // a lower degree on the same net has more cells, fewer pairs may take more
    // and shorter items and more chunks
    const size_t cells = std::min<size_t>(kUvCellsMax, (size_t)(nu_c - 1) * (nv_c - 1)), n = (size_t)npts;
    const size_t chunks = std::max(std::min<size_t>(64, (n + 255) / 256), (n + 2047) / 2048);
    const size_t items = std::min(cells, n) +
                         (npts < kLongItems ? n / 128 : std::max<size_t>(n / 512, (kLongItems - 1) / 128));
    return head + group_ws(B, sort_bytes(cells, chunks, items, sort_slot(p, q), n));
}

hipError_t launch_uv_bwd_sorted(const UvArgs& a, const UvSort& s, char* ws, hipStream_t st, const float* gpts,
                                unsigned mask, float* gc, float* gw, float* gku, float* gkv) {
    SortPtrs t;
    t.hist = reinterpret_cast<unsigned*>(ws + s.hist);
    t.cell_start = reinterpret_cast<int*>(ws + s.cell_start);
    t.item_start = reinterpret_cast<int*>(ws + s.item_start);
    t.item_cell = reinterpret_cast<int*>(ws + s.item_cell);
    t.order = reinterpret_cast<unsigned*>(ws + s.order);
    t.cell = reinterpret_cast<unsigned short*>(ws + s.cell_of);
    t.slots = reinterpret_cast<double*>(ws + s.slots);
    int bits = 0;
    while ((1 << bits) < s.cells) ++bits;
    const size_t lds = sizeof(unsigned) * (size_t)s.cells;
    int rbits = 0;
    while ((1 << rbits) < a.p + 1) ++rbits;
    const int cblk = ((4 << rbits) * a.nu_c * a.nv_c + kWG - 1) / kWG;
    const int kblk = (a.nu_c + a.p + 1 + a.nv_c + a.q + 1 + kWavesPerWG - 1) / kWavesPerWG;
    for (int b0 = 0; b0 < a.B; b0 += s.group) {
        const unsigned nb = (unsigned)std::min(s.group, a.B - b0);
        hipLaunchKernelGGL(k_uv_hist, dim3((unsigned)s.nchunk, nb), dim3(kWG), lds, st, a, s, t, b0);
        if (s.cells <= kScanPer * kWG) hipLaunchKernelGGL(k_uv_scan<kWG>, dim3(nb), dim3(kWG), 0, st, s, t);
        else hipLaunchKernelGGL(k_uv_scan<kUvCellsMax / kScanPer>, dim3(nb), dim3(kUvCellsMax / kScanPer), 0, st, s, t);
        hipLaunchKernelGGL(k_uv_order, dim3((unsigned)s.nchunk, nb), dim3(kWave), lds, st, a, s, t, bits);
        const dim3 gi((unsigned)((s.items + kWavesPerWG - 1) / kWavesPerWG), nb);
        const int m = std::max(a.p, a.q);
        if (m <= 3) launch_cell<3, 3>(gi, st, a, s, t, b0, gpts, mask);
        else if (m <= 5) launch_cell<5, 5>(gi, st, a, s, t, b0, gpts, mask);
        else launch_cell<7, 7>(gi, st, a, s, t, b0, gpts, mask);
        hipLaunchKernelGGL(k_uv_sum, dim3((unsigned)(cblk + kblk), nb), dim3(kWG), 0, st, a, s, t, b0, cblk, rbits, mask,
                           gc, gw, gku, gkv);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace nd
