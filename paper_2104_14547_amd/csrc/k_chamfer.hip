// Chamfer and Hausdorff distances between point sets on gfx950 (the losses
// of NURBS-Diff Sec. 4, eqs. ChamferDistance and HausdorffDistance):
//
//   CD = sum_i min_j |P_i - Q_j| + sum_j min_i |P_i - Q_j|
//   HD = max_i min_j |P_i - Q_j| + max_j min_i |P_i - Q_j|
//
// Which point is nearest (and which distance is largest) is an integer
// decision.  It is taken in float32 on the float32 inputs with the squared
// distance formed as  d2 = fma(dz, dz, fma(dy, dy, dx * dx))  (dz = 0 in the
// plane), a strictly smaller d2 winning, so the first index wins ties; the
// largest d2 with the first index wins for the Hausdorff terms.  Distances,
// sums and gradients are then taken from the chosen pairs: distances in
// FP64, gradients as FP32 unit vectors.
//
// Nearest neighbours: brute force over all pairs.  k_nn: a workgroup takes QL
// x 256 query points (QL per lane, in registers) and one contiguous range of
// the target set, staged through LDS 256 points at a time; every target read
// is shared by the lane's QL queries.  It keeps the least d2 and the group of
// kNnGroup consecutive targets it came from, not the index: a running minimum
// (v_min3_f32, two distances to an instruction) instead of a compare and two
// selects per pair.  k_nn_pick, one thread per query, takes the range with the
// strictly smallest d2 (ranges and groups in index order, so ties go to the
// smaller index) and finds the first target of its group with that d2: the
// distances of one group again, from the same formula, so the same bits.  Both
// directions of a Chamfer distance run in one launch.  What bounds it: VALU
// issue, 3 subtractions, 1 multiply, 2 FMAs and half a minimum per pair (9
// instructions when every pair carried its index).  16384 x 16384 points in
// space, both directions: 84 us (two launches of 56 us before), the whole loss
// with its gradients 88 us (132); 8 pairs of 1000 and 1531 points in the
// plane 27 us (77: nine launches, and ranges too long to fill the chip).
//
// Gradient with respect to P (k_nn_pick, k_cd_grad):
//   dCD/dP_i = (P_i - Q_a(i))/|.| + sum_{j : b(j) = i} (P_i - Q_j)/|.|
//   dHD/dP_i = [i = i*] (P_i - Q_a(i*))/|.| + [i = b(j*)] (P_i - Q_j*)/|.|
// (a: nearest target of each point, b: nearest point of each target,
// i*, j* the farthest ones).  The sum over the targets that chose a point
// is accumulated in 2^-40 fixed point with 64-bit integer atomics: exact
// and order-independent, so bitwise reproducible (no float atomics).
#include "device.hpp"
#include "launch.hpp"
#include "../../include/nurbsdiff.h"

#include <algorithm>
#include <type_traits>

namespace nd {
namespace {

constexpr int kNnTile = kWG;   // targets per LDS stage
constexpr int kNnGroup = 16;   // targets whose least d2 is kept as one

__device__ __forceinline__ float nn_d2(float px, float py, float pz, float4 q) {
    const float dx = px - q.x, dy = py - q.y, dz = pz - q.z;
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __fmul_rn(dx, dx)));
}

template <int DIM>
__device__ __forceinline__ float4 load_pt(const float* __restrict__ X, long long i) {
    const float* p = X + i * DIM;
    return make_float4(p[0], p[1], DIM == 3 ? p[2] : 0.f, 0.f);
}

// One direction of a search: each query point of X against all of Y.
struct NnDir {
    const float *X, *Y;
    int n, m, ql, qblocks, range, nranges;
    float* pd2;    // [B][nranges][n] least d2 of each range
    int* pgrp;     // [B][nranges][n] the group it came from
    int* idx;      // [B][n]
    float* d2;     // [B][n]
};

// k_nn of one direction's workgroup (qb, r) of cloud pair b.
template <int DIM, int QL>
__device__ __forceinline__ void nn_range(const NnDir& s, int b, int qb, int r, float4* tile) {
    const int i0 = qb * QL * kWG, j0 = r * s.range, j1 = min(s.m, j0 + s.range);
    const float* Xb = s.X + (long long)b * s.n * DIM;
    const float* Yb = s.Y + (long long)b * s.m * DIM;
    float px[QL], py[QL], pz[QL], best[QL];
    int bg[QL];
#pragma unroll
    for (int q = 0; q < QL; ++q) {
        const float4 p = load_pt<DIM>(Xb, min(i0 + q * kWG + (int)threadIdx.x, s.n - 1));
        px[q] = p.x;
        py[q] = p.y;
        pz[q] = p.z;
        best[q] = __builtin_inff();
        bg[q] = -1;
    }
    for (int t0 = j0; t0 < j1; t0 += kNnTile) {
        const int cnt = min(kNnTile, j1 - t0);
        __syncthreads();
        // past the end: the last target again, whose distance changes no minimum
        if ((int)threadIdx.x < (cnt + kNnGroup - 1) / kNnGroup * kNnGroup)
            tile[threadIdx.x] = load_pt<DIM>(Yb, t0 + min((int)threadIdx.x, cnt - 1));
        __syncthreads();
        for (int g = 0; g * kNnGroup < cnt; ++g) {
            float run[QL];
#pragma unroll
            for (int q = 0; q < QL; ++q) run[q] = __builtin_inff();
#pragma unroll
            for (int j = 0; j < kNnGroup; j += 2) {
                const float4 y0 = tile[g * kNnGroup + j], y1 = tile[g * kNnGroup + j + 1];
#pragma unroll
                for (int q = 0; q < QL; ++q)
                    run[q] = fminf(fminf(run[q], nn_d2(px[q], py[q], pz[q], y0)), nn_d2(px[q], py[q], pz[q], y1));
            }
#pragma unroll
            for (int q = 0; q < QL; ++q)
                if (run[q] < best[q]) {
                    best[q] = run[q];
                    bg[q] = t0 / kNnGroup + g;
                }
        }
    }
    const long long o = ((long long)b * s.nranges + r) * s.n;
#pragma unroll
    for (int q = 0; q < QL; ++q) {
        const int i = i0 + q * kWG + (int)threadIdx.x;
        if (i < s.n) {
            s.pd2[o + i] = best[q];
            s.pgrp[o + i] = bg[q];
        }
    }
}

// Grid: (workgroups of both directions, B).  zero: nzero 64-bit words cleared
// on the way (the gradient's accumulators, used by the next kernel).
template <int DIM>
__global__ void __launch_bounds__(kWG) k_nn(NnDir s0, NnDir s1, unsigned long long* __restrict__ zero,
                                           long long nzero) {
    __shared__ float4 tile[kNnTile];
    for (long long i = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * kWG + threadIdx.x; i < nzero;
         i += (long long)gridDim.x * gridDim.y * kWG)
        zero[i] = 0ull;
    const int first = s0.qblocks * s0.nranges;
    const bool second = (int)blockIdx.x >= first;
    const NnDir& s = second ? s1 : s0;
    const int w = (int)blockIdx.x - (second ? first : 0);
    const int qb = w / s.nranges, r = w - qb * s.nranges;
    if (s.ql == 4) nn_range<DIM, 4>(s, blockIdx.y, qb, r, tile);
    else if (s.ql == 2) nn_range<DIM, 2>(s, blockIdx.y, qb, r, tile);
    else nn_range<DIM, 1>(s, blockIdx.y, qb, r, tile);
}

// The nearest target of query i: index and d2 (see the top of the file).
template <int DIM>
__device__ __forceinline__ int nn_pick(const NnDir& s, int b, int i, float* d2) {
    const long long o = (long long)b * s.nranges * s.n + i;
    float best = __builtin_inff();
    int br = -1;
    // ranges' minima loaded together, then compared in range order: sixteen
    // while they last, then eight.  A few queries among 10^5 targets have
    // hundreds of ranges and a thread to a query, so the loads' latency is the
    // time (one query: 53 us with eight, 46 with sixteen, 43 with 32, whose
    // registers cost 5000 pairs of 16 points 10 %).
    int r0 = 0;
    auto take = [&](auto n) {
        constexpr int kU = decltype(n)::value;
        float d[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u)
            d[u] = kU == 16 || r0 + u < s.nranges ? s.pd2[o + (long long)(r0 + u) * s.n] : __builtin_inff();
#pragma unroll
        for (int u = 0; u < kU; ++u)
            if (d[u] < best) {
                best = d[u];
                br = r0 + u;
            }
        r0 += kU;
    };
    while (r0 + 16 <= s.nranges) take(std::integral_constant<int, 16>{});
    while (r0 < s.nranges) take(std::integral_constant<int, 8>{});
    const float* Yb = s.Y + (long long)b * s.m * DIM;
    const float4 p = load_pt<DIM>(s.X + (long long)b * s.n * DIM, i);
    int bi = 0;
    if (br < 0) {
        // no distance below +inf (or only NaN): the first target, as an
        // ordered scan that starts from it would keep
        best = nn_d2(p.x, p.y, p.z, load_pt<DIM>(Yb, 0));
    } else {
        const int j0 = s.pgrp[o + (long long)br * s.n] * kNnGroup;
#pragma unroll
        for (int j = kNnGroup - 1; j >= 0; --j) {
            const int k = min(j0 + j, s.m - 1);
            if (nn_d2(p.x, p.y, p.z, load_pt<DIM>(Yb, k)) == best) bi = k;
        }
    }
    *d2 = best;
    return bi;
}

// nurbs_nearest: one thread per query.
template <int DIM>
__global__ void __launch_bounds__(kWG) k_nn_pick(NnDir s) {
    const int b = blockIdx.y, i = blockIdx.x * kWG + threadIdx.x;
    if (i >= s.n) return;
    float d2;
    const int bi = nn_pick<DIM>(s, b, i, &d2);
    s.idx[(long long)b * s.n + i] = bi;
    s.d2[(long long)b * s.n + i] = d2;
}

// FP64 distance of a chosen pair and the FP32 unit vector from Y to X.
template <int DIM>
__device__ __forceinline__ double pair_dist(const float* X, long long i, const float* Y, long long j, float dir[3]) {
    double s = 0.0, d[3];
#pragma unroll
    for (int x = 0; x < DIM; ++x) {
        d[x] = (double)X[i * DIM + x] - (double)Y[j * DIM + x];
        s += d[x] * d[x];
    }
    const double r = sqrt(s);
#pragma unroll
    for (int x = 0; x < 3; ++x) dir[x] = (x < DIM && r > 0.0) ? (float)(d[x] / r) : 0.f;
    return r;
}

// Per cloud pair: the Chamfer sum (FP64) and the Hausdorff arg-maxes.
// k_cd_pick: a workgroup finds the nearest points of 256 points of P or of Q
// and reduces them (a tree over the workgroup); k_cd_final reduces the
// workgroups' partials, a thread's share in order and then a tree.  The
// arg-maxes take the largest float32 d2 with the smallest index.  Fixed order
// throughout.
struct ChState {
    double cd;
    int istar, jstar;
};
struct ChPart {
    double cd;
    float v;
    int i;
};

__device__ __forceinline__ void argmax_merge(float& v, int& i, float v2, int i2) {
    if (v2 > v || (v2 == v && i2 < i)) {
        v = v2;
        i = i2;
    }
}

// Tree over the workgroup of (sum, arg-max); thread 0 ends with the result.
__device__ __forceinline__ void cd_tree(double& cd, float& v, int& i, double* sd, float* sv, int* si) {
    const int t = threadIdx.x;
    sd[t] = cd;
    sv[t] = v;
    si[t] = i;
    __syncthreads();
    for (int h = kWG / 2; h > 0; h >>= 1) {
        if (t < h) {
            sd[t] += sd[t + h];
            argmax_merge(sv[t], si[t], sv[t + h], si[t + h]);
        }
        __syncthreads();
    }
    cd = sd[0];
    v = sv[0];
    i = si[0];
    __syncthreads();
}

// Fixed-point accumulation of the targets' pulls: each unit vector
// component (|u| <= 1) is rounded to a multiple of 2^-40 and added as a
// 64-bit integer.  Integer addition is exact and associative, so the sums
// do not depend on the order the atomics land in (bitwise reproducible);
// with at most 2^22 targets they stay below 2^62.
constexpr double kFixScale = 1099511627776.0;  // 2^40

// Grid (blocks of P, then blocks of Q; B).  part: [B][gridDim.x].
template <int DIM>
__global__ void __launch_bounds__(kWG) k_cd_pick(NnDir s0, NnDir s1, int blocks0, ChPart* __restrict__ part,
                                                unsigned long long* __restrict__ acc) {
    __shared__ double sd[kWG];
    __shared__ float sv[kWG];
    __shared__ int si[kWG];
    const int b = blockIdx.y;
    const bool second = (int)blockIdx.x >= blocks0;
    const NnDir& s = second ? s1 : s0;
    const int i = ((int)blockIdx.x - (second ? blocks0 : 0)) * kWG + (int)threadIdx.x;
    double r = 0.0;
    float v = -1.f;
    int at = s.n;
    if (i < s.n) {
        const int j = nn_pick<DIM>(s, b, i, &v);
        s.idx[(long long)b * s.n + i] = j;
        at = i;
        const float* Xb = s.X + (long long)b * s.n * DIM;
        const float* Yb = s.Y + (long long)b * s.m * DIM;
        double d[3], ss = 0.0;
#pragma unroll
        for (int x = 0; x < DIM; ++x) {
            d[x] = (double)Xb[(long long)i * DIM + x] - (double)Yb[(long long)j * DIM + x];
            ss += d[x] * d[x];
        }
        r = sqrt(ss);
        if (second && acc && r != 0.0) {
            // Q's point pulls its nearest point of P: the unit vector from Q to P
            unsigned long long* o = acc + ((long long)b * s.m + j) * 3;
#pragma unroll
            for (int x = 0; x < DIM; ++x)
                atomicAdd(o + x, (unsigned long long)__double2ll_rn(-d[x] / r * kFixScale));
        }
        if (!(v > -1.f)) {  // NaN: no candidate
            v = -1.f;
            at = s.n;
        }
    }
    cd_tree(r, v, at, sd, sv, si);
    if (threadIdx.x == 0) part[(long long)b * gridDim.x + blockIdx.x] = ChPart{r, v, at};
}

// One workgroup per cloud pair.
template <int DIM>
__global__ void __launch_bounds__(kWG) k_cd_final(const float* __restrict__ P, int n, const float* __restrict__ Q,
                                                 int m, const int* __restrict__ a, const int* __restrict__ bq,
                                                 const ChPart* __restrict__ part, int blocks0, int blocks1,
                                                 float* __restrict__ out, ChState* __restrict__ st) {
    __shared__ double sd[kWG];
    __shared__ float sv[kWG];
    __shared__ int si[kWG];
    const int b = blockIdx.x, t = threadIdx.x;
    const ChPart* pb = part + (long long)b * (blocks0 + blocks1);
    double cd = 0.0;
    float vi = -1.f, vj = -1.f;
    int ii = n, jj = m;
    for (int k = t; k < blocks0 + blocks1; k += kWG) {
        cd += pb[k].cd;
        if (k < blocks0) argmax_merge(vi, ii, pb[k].v, pb[k].i);
        else argmax_merge(vj, jj, pb[k].v, pb[k].i);
    }
    double none = 0.0;
    cd_tree(cd, vi, ii, sd, sv, si);
    cd_tree(none, vj, jj, sd, sv, si);
    if (t != 0) return;
    ii = min(ii, n - 1);  // only NaN distances: the last point stands for none
    jj = min(jj, m - 1);
    const float* Pb = P + (long long)b * n * DIM;
    const float* Qb = Q + (long long)b * m * DIM;
    float dir[3];
    const double hd = pair_dist<DIM>(Pb, ii, Qb, a[(long long)b * n + ii], dir) +
                      pair_dist<DIM>(Pb, bq[(long long)b * m + jj], Qb, jj, dir);
    out[2 * b] = (float)cd;
    out[2 * b + 1] = (float)hd;
    st[b].cd = cd;
    st[b].istar = ii;
    st[b].jstar = jj;
}

// dCD/dP and dHD/dP, one thread per point of P.
template <int DIM>
__global__ void __launch_bounds__(kWG) k_cd_grad(const float* __restrict__ P, int n, const float* __restrict__ Q,
                                                int m, const int* __restrict__ a, const int* __restrict__ bq,
                                                const ChState* __restrict__ st,
                                                const unsigned long long* __restrict__ acc, float* __restrict__ gcd,
                                                float* __restrict__ ghd) {
    const int b = blockIdx.y;
    const int i = blockIdx.x * kWG + threadIdx.x;
    if (i >= n) return;
    const float* Pb = P + (long long)b * n * DIM;
    const float* Qb = Q + (long long)b * m * DIM;
    const int ai = a[(long long)b * n + i];
    double d[3] = {0.0, 0.0, 0.0}, s = 0.0;
#pragma unroll
    for (int x = 0; x < DIM; ++x) {
        d[x] = (double)Pb[(long long)i * DIM + x] - (double)Qb[(long long)ai * DIM + x];
        s += d[x] * d[x];
    }
    const double r = sqrt(s);
    double u[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) u[x] = r > 0.0 ? d[x] / r : 0.0;
    const long long o = ((long long)b * n + i) * DIM;
    if (gcd) {
        const unsigned long long* ac = acc + ((long long)b * n + i) * 3;
#pragma unroll
        for (int x = 0; x < DIM; ++x) gcd[o + x] = (float)(u[x] + (double)(long long)ac[x] / kFixScale);
    }
    if (ghd) {
        const ChState cs = st[b];
        double h[3] = {0.0, 0.0, 0.0};
        if (i == cs.istar) {
#pragma unroll
            for (int x = 0; x < 3; ++x) h[x] += u[x];
        }
        if (i == bq[(long long)b * m + cs.jstar]) {
            double e[3], s2 = 0.0;
#pragma unroll
            for (int x = 0; x < DIM; ++x) {
                e[x] = (double)Pb[(long long)i * DIM + x] - (double)Qb[(long long)cs.jstar * DIM + x];
                s2 += e[x] * e[x];
            }
            const double r2 = sqrt(s2);
#pragma unroll
            for (int x = 0; x < DIM; ++x) h[x] += r2 > 0.0 ? e[x] / r2 : 0.0;
        }
#pragma unroll
        for (int x = 0; x < DIM; ++x) ghd[o + x] = (float)h[x];
    }
}

NnDir nn_dir(const NnSplit& sp, const float* X, int n, const float* Y, int m, int* idx, float* d2, float* pd2,
             int* pgrp) {
    NnDir s;
    s.X = X; s.Y = Y; s.n = n; s.m = m;
    s.ql = sp.ql; s.qblocks = sp.qblocks; s.range = sp.range; s.nranges = sp.nranges;
    s.pd2 = pd2; s.pgrp = pgrp; s.idx = idx; s.d2 = d2;
    return s;
}

int blocks_of(int n) { return (n + kWG - 1) / kWG; }

}  // namespace

// Queries per lane and target ranges of a search of n points among m: about
// four workgroups per CU over the launch (`dirs` searches of B pairs).  Four
// queries to a lane share each target read, so as many as leave ranges of 128
// targets and more; small sets take one query per lane and ranges of 64.
NnSplit nn_split(int B, int n, int m, int dirs, int num_cus) {
    NnSplit s;
    const long long want = std::max(1ll, 4ll * std::max(num_cus, 1) / dirs);
    for (s.ql = 4;; s.ql /= 2) {
        s.qblocks = (n + s.ql * kWG - 1) / (s.ql * kWG);
        const long long r = (want + (long long)B * s.qblocks - 1) / ((long long)B * s.qblocks);
        long long range = ((m + r - 1) / r + 63) / 64 * 64;
        if (range > kNnTile) range = (range + kNnTile - 1) / kNnTile * kNnTile;
        s.range = (int)range;
        s.nranges = (int)((m + range - 1) / range);
        if (s.ql == 1 || range >= 128) return s;
    }
}

hipError_t launch_nn(int dim, hipStream_t st, int B, const float* X, int n, const float* Y, int m,
                     const NnSplit& sp, int* idx, float* d2, int* pgrp, float* pd2) {
    const NnDir s = nn_dir(sp, X, n, Y, m, idx, d2, pd2, pgrp);
    const dim3 grid((unsigned)(s.qblocks * s.nranges), (unsigned)B), pick((unsigned)blocks_of(n), (unsigned)B);
#define ND_NN(D)                                                                                        \
    hipLaunchKernelGGL((k_nn<D>), grid, dim3(kWG), 0, st, s, s, (unsigned long long*)nullptr, 0ll);     \
    hipLaunchKernelGGL((k_nn_pick<D>), pick, dim3(kWG), 0, st, s);
    if (dim == 3) { ND_NN(3) }
    else if (dim == 2) { ND_NN(2) }
    else return hipErrorInvalidValue;
#undef ND_NN
    return hipGetLastError();
}

hipError_t launch_cd(int dim, hipStream_t st, int B, const float* P, int n, const float* Q, int m, const NnSplit& sp,
                     const NnSplit& sq, int* a, int* bq, int* pgrp_p, float* pd2_p, int* pgrp_q, float* pd2_q,
                     float* out, void* state, void* part, void* acc, float* gcd, float* ghd) {
    ChState* cs = reinterpret_cast<ChState*>(state);
    ChPart* cp = reinterpret_cast<ChPart*>(part);
    unsigned long long* ac = gcd ? reinterpret_cast<unsigned long long*>(acc) : nullptr;
    const NnDir s0 = nn_dir(sp, P, n, Q, m, a, nullptr, pd2_p, pgrp_p);
    const NnDir s1 = nn_dir(sq, Q, m, P, n, bq, nullptr, pd2_q, pgrp_q);
    const dim3 gs((unsigned)(s0.qblocks * s0.nranges + s1.qblocks * s1.nranges), (unsigned)B);
    const int b0 = blocks_of(n), b1 = blocks_of(m);
    const dim3 gp((unsigned)(b0 + b1), (unsigned)B), gn((unsigned)b0, (unsigned)B);
#define ND_CD(D)                                                                                                   \
    hipLaunchKernelGGL((k_nn<D>), gs, dim3(kWG), 0, st, s0, s1, ac, ac ? (long long)B * n * 3 : 0ll);               \
    hipLaunchKernelGGL((k_cd_pick<D>), gp, dim3(kWG), 0, st, s0, s1, b0, cp, ac);                                   \
    hipLaunchKernelGGL((k_cd_final<D>), dim3((unsigned)B), dim3(kWG), 0, st, P, n, Q, m, a, bq, cp, b0, b1, out, cs); \
    if (gcd || ghd) hipLaunchKernelGGL((k_cd_grad<D>), gn, dim3(kWG), 0, st, P, n, Q, m, a, bq, cs, ac, gcd, ghd);
    if (dim == 3) { ND_CD(3) }
    else if (dim == 2) { ND_CD(2) }
    else return hipErrorInvalidValue;
#undef ND_CD
    return hipGetLastError();
}

size_t cd_part_bytes(int n, int m) { return sizeof(ChPart) * (size_t)(blocks_of(n) + blocks_of(m)); }

size_t cd_state_bytes() { return sizeof(ChState); }

}  // namespace nd
