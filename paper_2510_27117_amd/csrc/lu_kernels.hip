// Kernels of the factorised TU reformulation (Theorem and Remark of Sec. 2.4.1)
// for gfx950.  The reformulated matrix is never stored: its rows are the
// original rows on the lifted vector z = (xbar, t) with t = S xbar, and
//     t        = M^{-1} (-B_JIbar xbar)          (lift)
//     S^T v    = -B_JIbar^T (M^{-T} v)           (projection of the pivot part)
// where M = L U is the pivot block in elimination order (entries of L and U in
// {-1, 0, 1}, unit diagonal of L, +-1 diagonal of U).
//
// Triangular solves run in place on one FP64 vector, level by level (a row reads
// only rows of earlier levels).  Runs of narrow levels go to one workgroup
// that keeps the vector in LDS and separates the levels with barriers; a wide
// level is one launch over its rows.  The candidates' exact lift solves the
// same systems in int32 for 64 candidates per wavefront (one lane per
// candidate: the systems of different candidates never interact).
#include "gfors_internal.h"

namespace gfors {

namespace {

// Sums of a step's rows, its updates and its solves run in FP64 and are rounded
// once, to the FP32 state: the launches take some microseconds and wait on loads,
// so the wider adds are free, and the order of the lanes no longer shows.  Error of
// the duals after 300 steps against FP64 (2-norm, medians of eight seeds; FP32
// throughout -> now): quadratic assignments of 100 variables 0.84e-6 -> 0.35e-6,
// 1,600 1.9e-6 -> 0.42e-6, 6,400 1.7e-6 -> 0.38e-6, 28,900 4.2e-6 -> 0.50e-6.  What
// is left is the rounding of the state itself, which decides on the smallest (36
// variables: 0.17 - 5.7e-6 -> 0.50 - 6.6e-6, medians 0.79e-6 and 0.75e-6).
__device__ __forceinline__ double dmad(int a, float x, double s) {
    return fma(static_cast<double>(a), static_cast<double>(x), s);
}

__device__ __forceinline__ double lu_block_sum256(double v, double *sh) {
    v = lane_group_sum(v, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) t = ((sh[0] + sh[1]) + sh[2]) + sh[3];
    __syncthreads();
    return t;
}

// One row of an in-place solve: x_k = d_k (x_k - sum_e a_e x_{c_e}), a_e and d_k = +-1.
__device__ __forceinline__ void trsv_row(int p, const int *__restrict__ row, const int *__restrict__ ptr,
                                         const int *__restrict__ ent, double *x) {
    const int rk = row[p];
    const int k = rk >> 1;
    double acc = x[k];
    const int e1 = ptr[p + 1];
    for (int e = ptr[p]; e < e1; ++e) {
        const int c = ent[e];
        const double v = x[c >> 1];
        acc = (c & 1) ? acc + v : acc - v;
    }
    x[k] = (rk & 1) ? -acc : acc;
}

}  // namespace

// What the last run of an FP32 iterate's lift writes: x32 = x rounded once, and
// with xold given xbar = 2 x32 - xold (the lifted part of xbar).
struct LuOut {
    float *x32 = nullptr;
    const float *xold = nullptr;
    float *xbar = nullptr;
};
__device__ __forceinline__ void lu_put(const LuOut &o, int k, double t) {
    if (!o.x32) return;
    const float v = static_cast<float>(t);
    const float old = o.xold ? o.xold[k] : 0.f;
    o.x32[k] = v;
    if (o.xbar) o.xbar[k] = 2.f * v - old;
}

// Levels [l0, l1) of a solve in one workgroup.  LDSX: the whole vector (r
// entries) and the run's rows and entries are staged in LDS first (their
// loads are independent of each other), so that each level costs LDS reads
// and a barrier only; the vector is written back at the end.
template <bool LDSX>
__global__ void __launch_bounds__(256)
k_lu_trsv_seg(const int *__restrict__ row, const int *__restrict__ ptr, const int *__restrict__ ent,
              const int *__restrict__ lvl, int l0, int l1, double *__restrict__ x, int r, LuOut out) {
    extern __shared__ __align__(16) unsigned char lu_lds[];
    if (!LDSX) {
        for (int l = l0; l < l1; ++l) {
            const int p1 = lvl[l + 1];
            for (int p = lvl[l] + static_cast<int>(threadIdx.x); p < p1; p += 256) trsv_row(p, row, ptr, ent, x);
            __syncthreads();
        }
        for (int i = threadIdx.x; i < r; i += 256) lu_put(out, i, x[i]);
        return;
    }
    const int pb = lvl[l0], pe = lvl[l1];
    const int np = pe - pb, eb = ptr[pb], ne = ptr[pe] - eb;
    double *xs = reinterpret_cast<double *>(lu_lds);
    int *srow = reinterpret_cast<int *>(xs + r);
    int *sptr = srow + np;          // np + 1 entries, relative to eb
    int *sent = sptr + np + 1;
    for (int i = threadIdx.x; i < r; i += 256) xs[i] = x[i];
    for (int i = threadIdx.x; i < np; i += 256) srow[i] = row[pb + i];
    for (int i = threadIdx.x; i <= np; i += 256) sptr[i] = ptr[pb + i] - eb;
    for (int i = threadIdx.x; i < ne; i += 256) sent[i] = ent[eb + i];
    __syncthreads();
    for (int l = l0; l < l1; ++l) {
        const int p1 = lvl[l + 1] - pb;
        for (int p = lvl[l] - pb + static_cast<int>(threadIdx.x); p < p1; p += 256) trsv_row(p, srow, sptr, sent, xs);
        __syncthreads();
    }
    for (int i = threadIdx.x; i < r; i += 256) {
        x[i] = xs[i];
        lu_put(out, i, xs[i]);
    }
}

// One wide level: rows [p0, p1) of the level order, one thread each.
__global__ void __launch_bounds__(256)
k_lu_trsv_level(const int *__restrict__ row, const int *__restrict__ ptr, const int *__restrict__ ent,
                int p0, int p1, double *__restrict__ x) {
    const int p = p0 + static_cast<int>(blockIdx.x * 256 + threadIdx.x);
    if (p < p1) trsv_row(p, row, ptr, ent, x);
}

// The output of a lift whose last run is a wide level or the identity.
__global__ void k_lu_put(int r, const double *__restrict__ x, LuOut out) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < r) lu_put(out, k, x[k]);
}

// LDS bytes of a staged run (vector, rows, pointers, entries).
size_t lu_seg_lds_bytes(const LuSolve &sv, const LuSeg &sg) {
    const int np = sv.hlvl[sg.b] - sv.hlvl[sg.a];
    const int ne = sv.hptr_at_lvl[sg.b] - sv.hptr_at_lvl[sg.a];
    return static_cast<size_t>(sv.r) * sizeof(double) + 4u * static_cast<size_t>(2 * np + 1 + ne);
}

void launch_lu_trsv(hipStream_t s, const LuSolve &sv, double *x, float *x32, const float *xold, float *xbar) {
    const int r = sv.r;
    LuOut out;
    out.x32 = x32;
    out.xold = xold;
    out.xbar = xbar;
    bool put = x32 == nullptr;
    for (int g = 0; g < sv.nseg; ++g) {
        const LuSeg &sg = sv.seg[g];
        if (sg.wide) {
            const int p0 = sg.a, p1 = sg.b;
            k_lu_trsv_level<<<(p1 - p0 + 255) / 256, 256, 0, s>>>(sv.row, sv.ptr, sv.ent, p0, p1, x);
            continue;
        }
        const size_t lds = lu_seg_lds_bytes(sv, sg);
        const LuOut o = g == sv.nseg - 1 ? out : LuOut();
        put = put || g == sv.nseg - 1;
        if (sv.use_lds && lds <= kLuLdsBytes)
            k_lu_trsv_seg<true><<<1, 256, lds, s>>>(sv.row, sv.ptr, sv.ent, sv.lvl, sg.a, sg.b, x, r, o);
        else
            k_lu_trsv_seg<false><<<1, 256, 0, s>>>(sv.row, sv.ptr, sv.ent, sv.lvl, sg.a, sg.b, x, r, o);
    }
    if (!put && r > 0) k_lu_put<<<(r + 255) / 256, 256, 0, s>>>(r, x, out);
}

// y[i] (+)= sgn * sum_e val_e x[col_e] over rows [0, nrows), LPR lanes per row.
template <int LPR, typename TI, bool ACC>
__global__ void __launch_bounds__(256)
k_lu_mv(int nrows, const int *__restrict__ rp, const int *__restrict__ ci, const int *__restrict__ val,
        const TI *__restrict__ x, double *__restrict__ y, double sgn) {
    const int tid = blockIdx.x * 256 + threadIdx.x;
    const int i = tid / LPR, sub = tid & (LPR - 1);
    double acc = 0.0;
    if (i < nrows) {
        const int e1 = rp[i + 1];
#pragma unroll 8
        for (int e = rp[i] + sub; e < e1; e += LPR) acc = fma(static_cast<double>(val[e]), static_cast<double>(x[ci[e]]), acc);
    }
    if (LPR > 1) acc = lane_group_sum(acc, LPR);
    if (i < nrows && sub == 0) y[i] = ACC ? y[i] + sgn * acc : sgn * acc;
}

template <typename TI, bool ACC>
static void mv_lpr(hipStream_t s, int lpr, int nrows, const int *rp, const int *ci, const int *val,
                   const TI *x, double *y, double sgn) {
    if (nrows <= 0) return;
    const int blocks = static_cast<int>((static_cast<int64_t>(nrows) * lpr + 255) / 256);
    switch (lpr) {
        case 1: k_lu_mv<1, TI, ACC><<<blocks, 256, 0, s>>>(nrows, rp, ci, val, x, y, sgn); break;
        case 4: k_lu_mv<4, TI, ACC><<<blocks, 256, 0, s>>>(nrows, rp, ci, val, x, y, sgn); break;
        case 16: k_lu_mv<16, TI, ACC><<<blocks, 256, 0, s>>>(nrows, rp, ci, val, x, y, sgn); break;
        default: k_lu_mv<64, TI, ACC><<<blocks, 256, 0, s>>>(nrows, rp, ci, val, x, y, sgn); break;
    }
}
void launch_lu_mv_f32(hipStream_t s, int lpr, int nrows, const int *rp, const int *ci, const int *val,
                      const float *x, double *y, double sgn) {
    mv_lpr<float, false>(s, lpr, nrows, rp, ci, val, x, y, sgn);
}
void launch_lu_mv_f64(hipStream_t s, int lpr, int nrows, const int *rp, const int *ci, const int *val,
                      const double *x, double *y, double sgn, bool accumulate) {
    if (accumulate) mv_lpr<double, true>(s, lpr, nrows, rp, ci, val, x, y, sgn);
    else mv_lpr<double, false>(s, lpr, nrows, rp, ci, val, x, y, sgn);
}

// The dual update with its sum in FP64, rounded once.
__device__ __forceinline__ float lu_dual_update(double s, float om, float rt, float tau2, float y_in, bool ineq) {
    const double y = y_in + static_cast<double>(tau2) * (rt - om * s);
    return static_cast<float>(ineq ? fmax(y, 0.0) : y);
}
// -s1 + (2/s_o) s2
__device__ __forceinline__ double lu_grad(bool hasq, const float *two_so, double s1, double s2) {
    return hasq ? fma(static_cast<double>(two_so[0]), s2, -s1) : -s1;
}
// Pivot part of the primal gradient, position k:
//   v_k = -sum_{j} a_{j, nk+k} wy_j + (2/s_o) sum_i Q_{nk+k, i} x_i
// (column nk + k of the lifted rows, row nk + k of the lifted Q; x lifted).
template <int LPR, bool HASQ>
__global__ void __launch_bounds__(256)
k_lu_tail_grad(int r, int nk, const int *__restrict__ rpT, const int *__restrict__ ciT,
               const int *__restrict__ valT, const float *__restrict__ wy, const int *__restrict__ rpQ,
               const int *__restrict__ ciQ, const int *__restrict__ valQ, const float *__restrict__ x,
               const float *__restrict__ two_so, double *__restrict__ v) {
    const int tid = blockIdx.x * 256 + threadIdx.x;
    const int k = tid / LPR, sub = tid & (LPR - 1);
    double s1 = 0.0, s2 = 0.0;
    if (k < r) {
        const int i = nk + k;
        for (int e = rpT[i] + sub; e < rpT[i + 1]; e += LPR) s1 = dmad(valT[e], wy[ciT[e]], s1);
        if (HASQ)
            for (int e = rpQ[i] + sub; e < rpQ[i + 1]; e += LPR) s2 = dmad(valQ[e], x[ciQ[e]], s2);
    }
    s1 = lane_group_sum(s1, LPR);
    if (HASQ) s2 = lane_group_sum(s2, LPR);
    if (k < r && sub == 0) v[k] = lu_grad(HASQ, two_so, s1, s2);
}

// Primal step of the kept variables (Algorithm 2) with the pivot part of the
// gradient: g_i = c~_i + rho - sum_j a_ji wy_j + (2/s_o) (Q z)_i
//               - sum_k (B_JIbar)_{k i} u_k - 2 rho x_i,   u = M^{-T} v.
template <int LPR, bool HASQ>
__global__ void __launch_bounds__(256)
k_lu_primal(int nk, const int *__restrict__ rpT, const int *__restrict__ ciT, const int *__restrict__ valT,
            const float *__restrict__ wy, const int *__restrict__ rpQ, const int *__restrict__ ciQ,
            const int *__restrict__ valQ, const int *__restrict__ rpB, const int *__restrict__ ciB,
            const int *__restrict__ valB, const double *__restrict__ u, const float *__restrict__ x_in,
            float *__restrict__ x_out, float *__restrict__ xbar, const float *__restrict__ ct,
            const float *__restrict__ tau1, const float *__restrict__ two_so,
            const double *__restrict__ rho, DevCounters *__restrict__ ctr) {
    const int tid = blockIdx.x * 256 + threadIdx.x;
    const int i = tid / LPR, sub = tid & (LPR - 1);
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (i < nk) {
        // the first entries of the three lists together (a chain of bounds,
        // index and operand each; U of Q's), then what is left of each list
        constexpr int U = 4;
        int e1 = rpT[i] + sub, eq = HASQ ? rpQ[i] + sub : 0, e3 = rpB[i] + sub;
        const int z1 = rpT[i + 1], zq = HASQ ? rpQ[i + 1] : 0, z3 = rpB[i + 1];
        const int c1 = e1 < z1 ? ciT[e1] : -1, c3 = e3 < z3 ? ciB[e3] : -1;
        const int a1 = e1 < z1 ? valT[e1] : 0, a3 = e3 < z3 ? valB[e3] : 0;
        int cq[U], aq[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool in = HASQ && eq + k * LPR < zq;
            cq[k] = in ? ciQ[eq + k * LPR] : -1;
            aq[k] = in ? valQ[eq + k * LPR] : 0;
        }
        const float w1 = c1 >= 0 ? wy[c1] : 0.f;
        const double u3 = c3 >= 0 ? u[c3] : 0.0;
        float xq[U];
#pragma unroll
        for (int k = 0; k < U; ++k) xq[k] = cq[k] >= 0 ? x_in[cq[k]] : 0.f;
        s1 = dmad(a1, w1, s1);
        s3 = fma(static_cast<double>(a3), u3, s3);
#pragma unroll
        for (int k = 0; k < U; ++k) s2 = dmad(aq[k], xq[k], s2);
        for (int e = e1 + LPR; e < z1; e += LPR) s1 = dmad(valT[e], wy[ciT[e]], s1);
        if (HASQ)
            for (int e = eq + U * LPR; e < zq; e += LPR) s2 = dmad(valQ[e], x_in[ciQ[e]], s2);
        for (int e = e3 + LPR; e < z3; e += LPR) s3 = fma(static_cast<double>(valB[e]), u[ciB[e]], s3);
    }
    s1 = lane_group_sum(s1, LPR);
    if (HASQ) s2 = lane_group_sum(s2, LPR);
    s3 = lane_group_sum(s3, LPR);
    if (i < nk && sub == 0) {
        const float xi = x_in[i];
        double g = (ct[i] + rho[0]) - s1;
        if (HASQ) g = fma(static_cast<double>(two_so[0]), s2, g);
        g -= s3;
        g -= 2.0 * rho[0] * xi;
        const float xn = static_cast<float>(fmin(fmax(xi - tau1[0] * g, 0.0), 1.0));
        x_out[i] = xn;
        xbar[i] = 2.f * xn - xi;
    }
    if (tid == 0) ctr->k += 1;
}

// Dual step of the lifted rows.  Long rows (kHeavyLen+ entries) are cut into
// chunks spread over the device: the first nchunk workgroups sum a_e xbar_{c_e}
// of one chunk each; lu_heavy_row adds a row's chunk sums in order and applies
//   y_j = Pi(y_j + tau2 (rt_j - omega_j s_j)),  wy_j = omega_j y_j.
// The other workgroups update the remaining rows, LPR lanes each (as k_dual).
template <int LPR>
__global__ void __launch_bounds__(256)
k_lu_dual(LuDualArgs A) {
    __shared__ double ws[4];
    if (static_cast<int>(blockIdx.x) < A.nchunk) {
        const int c = blockIdx.x;
        const int j = A.ch_row[c], e0 = A.ch_e0[c], e1 = A.ch_e1[c];
        const int c0 = A.rowc0[j], b0 = A.rp[j];
        double s = 0.0;
#pragma unroll 8
        for (int e = e0 + static_cast<int>(threadIdx.x); e < e1; e += 256) {
            const int col = c0 >= 0 ? c0 + (e - b0) : A.ci[e];
            s = dmad(A.val[e], A.xbar[col], s);
        }
        s = lane_group_sum(s, 64);
        if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) A.part[c] = ((ws[0] + ws[1]) + ws[2]) + ws[3];
        return;
    }
    const int tid = (blockIdx.x - A.nchunk) * 256 + threadIdx.x;
    const int row = tid / LPR, sub = tid & (LPR - 1);
    double s = 0.0;
    bool own = row < A.m;
    if (own) {
        const int e0 = A.rp[row], e1 = A.rp[row + 1];
        if (A.skip_len > 0 && e1 - e0 >= A.skip_len) own = false;
#pragma unroll 4
        for (int e = e0 + sub; own && e < e1; e += LPR)
            s = dmad(A.val[e], A.xbar[A.ci[e]], s);
    }
    s = lane_group_sum(s, LPR);
    if (own && sub == 0) {
        const float om = A.omega[row];
        const float y = lu_dual_update(s, om, A.rt[row], A.tau2, A.y_in[row], row < A.m1);
        A.y_out[row] = y;
        A.wy[row] = om * y;
    }
}

__device__ __forceinline__ void lu_heavy_row(int h, const LuHeavyArgs &A) {
    const int j = A.order[h];
    double sum = 0.0;
#pragma unroll 8
    for (int c = A.first[h]; c < A.first[h + 1]; ++c) sum += A.part[c];
    const float om = A.omega[j];
    const float y = lu_dual_update(sum, om, A.rt[j], A.tau2, A.y_in[j], j < A.m1);
    A.y_out[j] = y;
    A.wy[j] = om * y;
}
__global__ void k_lu_heavy_combine(LuHeavyArgs A) {
    const int h = blockIdx.x * 64 + threadIdx.x;
    if (h < A.nheavy) lu_heavy_row(h, A);
}

void launch_lu_dual(hipStream_t s, int lpr, const LuDualArgs &A) {
    const int blocks = A.nchunk + (A.rows ? static_cast<int>((static_cast<int64_t>(A.m) * lpr + 255) / 256) : 0);
    if (blocks <= 0) return;
    switch (lpr) {
#define GF_CASE(L) case L: k_lu_dual<L><<<blocks, 256, 0, s>>>(A); break;
        GF_CASE(1) GF_CASE(2) GF_CASE(4) GF_CASE(8) GF_CASE(16) GF_CASE(32) GF_CASE(64)
#undef GF_CASE
        default: break;
    }
}
void launch_lu_dual_heavy(hipStream_t s, const LuHeavyArgs &A) {
    if (A.nheavy > 0) k_lu_heavy_combine<<<(A.nheavy + 63) / 64, 64, 0, s>>>(A);
}

// ---------------------------------------------------------------------------
// The narrow parts of a step in one workgroup each (a solve is a chain of
// levels, bound by latency wherever it runs; what can go are the launches
// around it and the loads inside it).  A thread owns one position of a solve's
// level order, its row, level and first four entries in registers, all loaded
// before anything waits; the vector sits in LDS, so a level costs an LDS read
// or two, the adds and a barrier.
// 90,000-variable quadratic assignment (599 pivots, 14 levels), us a step:
// combine 4.5 + gradient 9.5 + transposed solve 8.3 -> 14.0; lift solve 9.8 -> 7.5.
// ---------------------------------------------------------------------------
struct LuRun {
    const int *row = nullptr, *ptr = nullptr, *ent = nullptr, *lvl = nullptr;
    int l0 = 0, l1 = 0;   // levels; none: the identity
    int p0 = 0, p1 = 0;   // their positions
};
struct LuLane {
    int k = 0, lev = -1, sign = 0, e0 = 0, e1 = 0, c[4] = {0, 0, 0, 0};
};
// ends[i]: end position of the run's i-th level, relative to its first position
__device__ __forceinline__ void lu_stage_levels(const LuRun &S, int *ends) {
    for (int i = threadIdx.x; i < S.l1 - S.l0; i += blockDim.x) ends[i] = S.lvl[S.l0 + i + 1] - S.p0;
}
// Without branches around the loads (positions and entries are clamped), so that
// they go out together with the caller's.
__device__ __forceinline__ void lu_load_lane(const LuRun &S, LuLane &t) {
    if (S.p1 <= S.p0) return;   // uniform
    const int p = S.p0 + static_cast<int>(threadIdx.x);
    const bool own = p < S.p1;
    const int q = min(p, S.p1 - 1);
    const int rk = S.row[q];
    t.e0 = S.ptr[q];
    t.e1 = S.ptr[q + 1];
    t.k = rk >> 1;
    t.sign = rk & 1;
    const int last = max(t.e1 - 1, 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) t.c[u] = S.ent[min(t.e0 + u, last)];   // unused past the row's end
    t.lev = own ? 0 : -1;   // the level itself from the staged level ends
}
__device__ __forceinline__ void lu_run(const LuRun &S, LuLane &t, const int *ends, double *xs) {
    const int nl = S.l1 - S.l0;
    if (nl <= 0) return;
    if (t.lev >= 0) {
        int lo = 0, hi = nl - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ends[mid] > static_cast<int>(threadIdx.x)) hi = mid;
            else lo = mid + 1;
        }
        t.lev = lo;
    }
    for (int l = 0; l < nl; ++l) {
        if (t.lev == l) {
            double acc = xs[t.k];
            double v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = t.e0 + u < t.e1 ? xs[t.c[u] >> 1] : 0.0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (t.e0 + u < t.e1) acc = (t.c[u] & 1) ? acc + v[u] : acc - v[u];
            for (int e = t.e0 + 4; e < t.e1; ++e) {
                const int c = S.ent[e];
                const double w = xs[c >> 1];
                acc = (c & 1) ? acc + w : acc - w;
            }
            xs[t.k] = t.sign ? -acc : acc;
        }
        __syncthreads();
    }
}

template <bool HASQ>
__global__ void __launch_bounds__(kLuOneMax)
k_lu_mid(LuHeavyArgs H, int lpr, int r, int nk, const int *__restrict__ rpT, const int *__restrict__ ciT,
         const int *__restrict__ valT, const float *wy, const int *__restrict__ rpQ, const int *__restrict__ ciQ,
         const int *__restrict__ valQ, const float *__restrict__ x, const float *__restrict__ two_so, LuRun S1, LuRun S2,
         double *__restrict__ v) {
    __shared__ double xs[kLuOneMax];
    __shared__ int ends1[kLuOneMax], ends2[kLuOneMax];
    LuLane t1, t2;
    const int sub = threadIdx.x & (lpr - 1), grp = threadIdx.x / lpr, ngrp = blockDim.x / lpr;
    // the first pass's entries of K^T and Q, fetched with the solves' lanes (one
    // chain of latencies for all), before the heavy rows are known
    constexpr int U = 4, UQ = 12;
    const int i0 = nk + min(grp, r - 1);
    int f0 = rpT[i0] + sub, f1 = rpT[i0 + 1], g0 = HASQ ? rpQ[i0] + sub : 0, g1 = HASQ ? rpQ[i0 + 1] : 0;
    lu_load_lane(S1, t1);
    lu_load_lane(S2, t2);
    int cf[U], af[U], cg[UQ], ag[UQ];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool in = f0 + u * lpr < f1;
        cf[u] = in ? ciT[f0 + u * lpr] : -1;
        af[u] = in ? valT[f0 + u * lpr] : 0;
    }
#pragma unroll
    for (int u = 0; u < UQ; ++u) {
        const bool in = HASQ && g0 + u * lpr < g1;
        cg[u] = in ? ciQ[g0 + u * lpr] : -1;
        ag[u] = in ? valQ[g0 + u * lpr] : 0;
    }
    lu_stage_levels(S1, ends1);
    lu_stage_levels(S2, ends2);
    // the last threads update the heavy rows while the others take the gradient's Q part
    for (int h = blockDim.x - 1 - threadIdx.x; h < H.nheavy; h += blockDim.x) lu_heavy_row(h, H);
    if (HASQ)
        for (int b = 0; b < r; b += ngrp) {
            const int k = b + grp;
            double s2 = 0.0;
            if (b == 0) {
                float w[UQ];
#pragma unroll
                for (int u = 0; u < UQ; ++u) w[u] = cg[u] >= 0 ? x[cg[u]] : 0.f;
#pragma unroll
                for (int u = 0; u < UQ; ++u) s2 = dmad(ag[u], w[u], s2);
                for (int e = g0 + UQ * lpr; e < g1; e += lpr) s2 = dmad(valQ[e], x[ciQ[e]], s2);
            } else if (k < r) {
                const int zq = rpQ[nk + k + 1];
#pragma unroll 8
                for (int e = rpQ[nk + k] + sub; e < zq; e += lpr) s2 = dmad(valQ[e], x[ciQ[e]], s2);
            }
            s2 = lane_group_sum(s2, lpr);
            if (k < r && sub == 0) xs[k] = s2;
        }
    __syncthreads();   // the heavy rows' wy
    for (int b = 0; b < r; b += ngrp) {
        const int k = b + grp;
        double s1 = 0.0;
        if (b == 0) {
            float w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = cf[u] >= 0 ? wy[cf[u]] : 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) s1 = dmad(af[u], w[u], s1);
            for (int e = f0 + U * lpr; e < f1; e += lpr) s1 = dmad(valT[e], wy[ciT[e]], s1);
        } else if (k < r) {
            const int z1 = rpT[nk + k + 1];
#pragma unroll 4
            for (int e = rpT[nk + k] + sub; e < z1; e += lpr) s1 = dmad(valT[e], wy[ciT[e]], s1);
        }
        s1 = lane_group_sum(s1, lpr);
        if (k < r && sub == 0) xs[k] = lu_grad(HASQ, two_so, s1, xs[k]);
    }
    __syncthreads();
    lu_run(S1, t1, ends1, xs);
    lu_run(S2, t2, ends2, xs);
    for (int k = threadIdx.x; k < r; k += blockDim.x) v[k] = xs[k];
}

// Both solves of a lift of t, the result to out.
__global__ void __launch_bounds__(kLuOneMax)
k_lu_lift(int r, LuRun S1, LuRun S2, const double *__restrict__ t, LuOut out) {
    __shared__ double xs[kLuOneMax];
    __shared__ int ends1[kLuOneMax], ends2[kLuOneMax];
    LuLane t1, t2;
    const int k = threadIdx.x;
    lu_stage_levels(S1, ends1);
    lu_stage_levels(S2, ends2);
    lu_load_lane(S1, t1);
    lu_load_lane(S2, t2);
    if (k < r) xs[k] = t[k];
    const float old = k < r ? out.xold[k] : 0.f;
    __syncthreads();
    lu_run(S1, t1, ends1, xs);
    lu_run(S2, t2, ends2, xs);
    if (k < r) {
        const float v = static_cast<float>(xs[k]);
        out.x32[k] = v;
        out.xbar[k] = 2.f * v - old;
    }
}

bool lu_fits(const LuSolve &a, const LuSolve &b) {
    auto one = [](const LuSolve &s) { return s.nseg == 0 || (s.nseg == 1 && !s.seg[0].wide && s.use_lds); };
    auto deep = [](const LuSolve &s) { return s.nseg > 0 && s.seg[0].b - s.seg[0].a > 1; };
    return a.r > 0 && a.r <= kLuOneMax && one(a) && one(b) && a.use_lds && b.use_lds && (deep(a) || deep(b));
}
static LuRun lu_run_of(const LuSolve &s) {
    LuRun S;
    if (s.nseg == 1) {
        S.row = s.row;
        S.ptr = s.ptr;
        S.ent = s.ent;
        S.lvl = s.lvl;
        S.l0 = s.seg[0].a;
        S.l1 = s.seg[0].b;
        S.p0 = s.hlvl[S.l0];
        S.p1 = s.hlvl[S.l1];
    }
    return S;
}
int lu_threads(int r) { return r <= 256 ? 256 : (r <= 512 ? 512 : kLuOneMax); }

void launch_lu_mid(hipStream_t s, const LuHeavyArgs &H, int lpr, bool hasq, int r, int nk, const int *rpT,
                   const int *ciT, const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                   const float *x, const float *two_so, const LuSolve &a, const LuSolve &b, double *v) {
    const LuRun A = lu_run_of(a), B = lu_run_of(b);
    if (hasq)
        k_lu_mid<true><<<1, lu_threads(r), 0, s>>>(H, lpr, r, nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, x, two_so, A, B, v);
    else
        k_lu_mid<false><<<1, lu_threads(r), 0, s>>>(H, lpr, r, nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, x, two_so, A, B, v);
}
void launch_lu_lift(hipStream_t s, int r, const LuSolve &a, const LuSolve &b, const double *t, float *x32,
                    const float *xold, float *xbar) {
    LuOut out;
    out.x32 = x32;
    out.xold = xold;
    out.xbar = xbar;
    k_lu_lift<<<1, lu_threads(r), 0, s>>>(r, lu_run_of(a), lu_run_of(b), t, out);
}

// xbar's lifted part: t(xbar_k) = 2 t(x_k) - t(x_{k-1}) (the lift is linear).
__global__ void k_lu_xbar_tail(int r, int nk, const float *__restrict__ x_new, const float *__restrict__ x_old,
                               float *__restrict__ xbar) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < r) xbar[nk + k] = 2.f * x_new[nk + k] - x_old[nk + k];
}

void launch_lu_tail_grad(hipStream_t s, int lpr, bool hasq, int r, int nk, const int *rpT, const int *ciT,
                         const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                         const float *x, const float *two_so, double *v) {
    if (r <= 0) return;
    const int blocks = static_cast<int>((static_cast<int64_t>(r) * lpr + 255) / 256);
#define GF_TG(L) \
    do { if (hasq) k_lu_tail_grad<L, true><<<blocks, 256, 0, s>>>(r, nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, x, two_so, v); \
         else k_lu_tail_grad<L, false><<<blocks, 256, 0, s>>>(r, nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, x, two_so, v); } while (0)
    switch (lpr) {
        case 1: GF_TG(1); break;
        case 4: GF_TG(4); break;
        case 16: GF_TG(16); break;
        default: GF_TG(64); break;
    }
#undef GF_TG
}

void launch_lu_primal(hipStream_t s, int lpr, bool hasq, int nk, const int *rpT, const int *ciT,
                      const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                      const int *rpB, const int *ciB, const int *valB, const double *u, const float *x_in,
                      float *x_out, float *xbar, const float *ct, const float *tau1, const float *two_so,
                      const double *rho, DevCounters *ctr) {
    const int blocks = static_cast<int>((static_cast<int64_t>(nk) * lpr + 255) / 256);
#define GF_PR(L) \
    do { if (hasq) k_lu_primal<L, true><<<blocks, 256, 0, s>>>(nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, rpB, ciB, valB, u, x_in, x_out, xbar, ct, tau1, two_so, rho, ctr); \
         else k_lu_primal<L, false><<<blocks, 256, 0, s>>>(nk, rpT, ciT, valT, wy, rpQ, ciQ, valQ, rpB, ciB, valB, u, x_in, x_out, xbar, ct, tau1, two_so, rho, ctr); } while (0)
    switch (lpr) {
        case 1: GF_PR(1); break;
        case 4: GF_PR(4); break;
        case 16: GF_PR(16); break;
        default: GF_PR(64); break;
    }
#undef GF_PR
}

void launch_lu_xbar_tail(hipStream_t s, int r, int nk, const float *x_new, const float *x_old, float *xbar) {
    if (r > 0) k_lu_xbar_tail<<<(r + 255) / 256, 256, 0, s>>>(r, nk, x_new, x_old, xbar);
}

// d[i] = a[i] - b[i] in FP64 (FP32 operands), i < n.
__global__ void k_lu_diff64(int n, const float *__restrict__ a, const float *__restrict__ b, double *__restrict__ d) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) d[i] = b ? static_cast<double>(a[i]) - static_cast<double>(b[i]) : static_cast<double>(a[i]);
}
void launch_lu_diff64(hipStream_t s, int n, const float *a, const float *b, double *d) {
    if (n > 0) k_lu_diff64<<<(n + 255) / 256, 256, 0, s>>>(n, a, b, d);
}

// FP64 residual rows on lifted FP64 vectors (Theorem 2, CheckHalt of Sec. 3):
//   s^y_j = (y_{k-1} - y_k)_j / tau2 - omega_j (row_j . d1),  d1 = lift(xbar_{k-1} - x_k)
//   gap_j = omega_j (r_j - row_j . d2), positive part on inequality rows, d2 = lift(x_k)
__global__ void __launch_bounds__(256)
k_lu_res_rows(const int *__restrict__ tb0, const int *__restrict__ tb1, int m1, const int *__restrict__ rp,
              const int *__restrict__ ci, const int *__restrict__ val, const double *__restrict__ omega64,
              const int64_t *__restrict__ rhs, const double *__restrict__ d1, const double *__restrict__ d2,
              const float *__restrict__ y_prev, const float *__restrict__ y, const double *__restrict__ tau2d,
              double *__restrict__ part) {
    __shared__ double sh[4];
    const int t = blockIdx.x;
    const double tau2 = tau2d[0];
    const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;
    double a1 = 0.0, a2 = 0.0;
    for (int j0 = tb0[t]; j0 < tb1[t]; j0 += 16) {
        const int j = j0 + grp;
        double s1 = 0.0, s2 = 0.0;
        if (j < tb1[t])
            for (int e = rp[j] + sub; e < rp[j + 1]; e += 16) {
                const double a = static_cast<double>(val[e]);
                s1 += a * d1[ci[e]];
                s2 += a * d2[ci[e]];
            }
        s1 = lane_group_sum(s1, 16);
        s2 = lane_group_sum(s2, 16);
        if (j < tb1[t] && sub == 0) {
            const double om = omega64[j];
            const double sy = (static_cast<double>(y_prev[j]) - static_cast<double>(y[j])) / tau2 - om * s1;
            double g = om * (static_cast<double>(rhs[j]) - s2);
            if (j < m1 && g < 0.0) g = 0.0;
            a1 += sy * sy;
            a2 += g * g;
        }
    }
    a1 = lu_block_sum256(a1, sh);
    a2 = lu_block_sum256(a2, sh);
    if (threadIdx.x == 0) { part[2 * t] = a1; part[2 * t + 1] = a2; }
}
void launch_lu_res_rows(hipStream_t s, const Tiles &rt, int m1, const int *rp, const int *ci, const int *val,
                        const double *omega64, const int64_t *rhs, const double *d1, const double *d2,
                        const float *y_prev, const float *y, const double *tau2d, double *part) {
    if (rt.count)
        k_lu_res_rows<<<rt.count, 256, 0, s>>>(rt.b0, rt.b1, m1, rp, ci, val, omega64, rhs, d1, d2, y_prev, y,
                                                tau2d, part);
}

// FP64 residual of the kept variables:  s^x_i = -dx_i/tau1 - 2 rho dx_i + (2/s_o) (Q' dx)_i
// with (Q' dx) given (null without Q); binary gap x_i (1 - x_i).
__global__ void __launch_bounds__(256)
k_lu_res_vars(const int *__restrict__ tb0, const int *__restrict__ tb1, const double *__restrict__ qd,
              const float *__restrict__ x, const float *__restrict__ xp, const double *__restrict__ rho,
              const double *__restrict__ tau1d, const double *__restrict__ two_sod, double *__restrict__ part) {
    __shared__ double sh[4];
    const int t = blockIdx.x;
    const double r = rho[0], tau1 = tau1d[0], tso = two_sod[0];
    double a1 = 0.0, a2 = 0.0;
    for (int i = tb0[t] + threadIdx.x; i < tb1[t]; i += 256) {
        const double xi = x[i];
        const double dx = xi - static_cast<double>(xp[i]);
        double sx = -dx / tau1 - 2.0 * r * dx;
        if (qd) sx += tso * qd[i];
        a1 += sx * sx;
        a2 += xi * (1.0 - xi);
    }
    a1 = lu_block_sum256(a1, sh);
    a2 = lu_block_sum256(a2, sh);
    if (threadIdx.x == 0) { part[2 * t] = a1; part[2 * t + 1] = a2; }
}
void launch_lu_res_vars(hipStream_t s, const Tiles &vt, const double *qd, const float *x, const float *xp,
                        const double *rho, const double *tau1d, const double *two_sod, double *part) {
    if (vt.count) k_lu_res_vars<<<vt.count, 256, 0, s>>>(vt.b0, vt.b1, qd, x, xp, rho, tau1d, two_sod, part);
}

// ---------------------------------------------------------------------------
// Exact lift of the candidates (EvalBest on the reformulated model).
// XI[k][l] (int32, candidate-minor with stride K) first receives
//   d_{J_{a_k}} - (B_JIbar x_l)_k,
// then the in-place solves L forward, U backward turn it into x_{I_{b_k}} of
// candidate l (its value s + S x_l, any integer).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_lu_eval_rhs(int r, int W, int K, const int *__restrict__ rp, const int *__restrict__ ci,
              const int *__restrict__ val, const int64_t *__restrict__ dJ, const uint64_t *__restrict__ X,
              int *__restrict__ XI) {
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= r * W) return;
    const int k = g / W, w = g - k * W;
    int acc = static_cast<int>(dJ[k]);
    // 64 entries at a time: lane j loads entry j's column, coefficient and
    // candidate word (one gather for all 64), then every lane walks them in
    // entry order through lane reads (integer sums: the order is free anyway)
    const int e0 = rp[k], e1 = rp[k + 1];
    for (int eb = e0; eb < e1; eb += 64) {
        const int e = eb + lane;
        const bool in = e < e1;
        const int vl = in ? val[e] : 0;
        const uint64_t wl = in ? X[static_cast<int64_t>(ci[e]) * W + w] : 0ull;
        const uint32_t wlo = static_cast<uint32_t>(wl), whi = static_cast<uint32_t>(wl >> 32);
        const int cnt = min(64, e1 - eb);
        for (int j = 0; j < cnt; ++j) {
            const int vj = __builtin_amdgcn_readlane(vl, j);
            const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wlo), j));
            const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(whi), j));
            const uint32_t half = lane < 32 ? lo : hi;
            if ((half >> (lane & 31)) & 1u) acc -= vj;
        }
    }
    XI[static_cast<int64_t>(k) * K + 64 * w + lane] = acc;
}

__device__ __forceinline__ void trsm_row(int p, const int *__restrict__ row, const int *__restrict__ ptr,
                                         const int *__restrict__ ent, int *__restrict__ XI, int K, int l) {
    const int rk = row[p];
    const int k = rk >> 1;
    int acc = XI[static_cast<int64_t>(k) * K + l];
    for (int e = ptr[p]; e < ptr[p + 1]; ++e) {
        const int c = ent[e];
        const int v = XI[static_cast<int64_t>(c >> 1) * K + l];
        acc = (c & 1) ? acc + v : acc - v;
    }
    XI[static_cast<int64_t>(k) * K + l] = (rk & 1) ? -acc : acc;
}

// Narrow levels [l0, l1): workgroup w owns candidates 64w .. 64w+63; its four
// wavefronts split the rows of a level.
__global__ void __launch_bounds__(256)
k_lu_trsm_seg(const int *__restrict__ row, const int *__restrict__ ptr, const int *__restrict__ ent,
              const int *__restrict__ lvl, int l0, int l1, int *__restrict__ XI, int K) {
    const int l = 64 * blockIdx.x + (threadIdx.x & 63);
    const int wv = threadIdx.x >> 6;
    for (int lv = l0; lv < l1; ++lv) {
        const int p1 = lvl[lv + 1];
        for (int p = lvl[lv] + wv; p < p1; p += 4) trsm_row(p, row, ptr, ent, XI, K, l);
        __syncthreads();
    }
}
// A wide level: rows [p0, p1), four per workgroup, 64 candidates per wavefront.
__global__ void __launch_bounds__(256)
k_lu_trsm_level(const int *__restrict__ row, const int *__restrict__ ptr, const int *__restrict__ ent,
                int p0, int p1, int *__restrict__ XI, int K) {
    const int p = p0 + 4 * static_cast<int>(blockIdx.x) + (threadIdx.x >> 6);
    const int l = 64 * blockIdx.y + (threadIdx.x & 63);
    if (p < p1) trsm_row(p, row, ptr, ent, XI, K, l);
}

void launch_lu_trsm(hipStream_t s, const LuSolve &sv, int *XI, int K) {
    const int W = K / 64;
    for (int g = 0; g < sv.nseg; ++g) {
        const LuSeg &sg = sv.seg[g];
        if (sg.wide) {
            dim3 grid((sg.b - sg.a + 3) / 4, W);
            k_lu_trsm_level<<<grid, 256, 0, s>>>(sv.row, sv.ptr, sv.ent, sg.a, sg.b, XI, K);
        } else {
            k_lu_trsm_seg<<<W, 256, 0, s>>>(sv.row, sv.ptr, sv.ent, sv.lvl, sg.a, sg.b, XI, K);
        }
    }
}

void launch_lu_eval_rhs(hipStream_t s, int r, int K, const int *rp, const int *ci, const int *val,
                        const int64_t *dJ, const uint64_t *X, int *XI) {
    const int W = K / 64;
    const int64_t waves = static_cast<int64_t>(r) * W;
    if (waves > 0) k_lu_eval_rhs<<<static_cast<int>((waves + 3) / 4), 256, 0, s>>>(r, W, K, rp, ci, val, dJ, X, XI);
}

// Value of lifted column c for candidate l (lane) of word w: a kept variable's
// bit, or the lifted integer of position c - nk.
__device__ __forceinline__ int64_t lifted_val(int c, int nk, const uint64_t *__restrict__ X, int W, int w,
                                              int lane, const int *__restrict__ XI, int K) {
    if (c < nk) return static_cast<int64_t>((X[static_cast<int64_t>(c) * W + w] >> lane) & 1ull);
    return static_cast<int64_t>(XI[static_cast<int64_t>(c - nk) * K + 64 * w + lane]);
}

// Rows of the reformulated model on the lifted integer point, one wavefront
// per (row chunk, candidate word).  A row in one chunk is decided at once
// (violation: lhs < rhs on an inequality row, lhs != rhs on an equality row:
// one count for its candidate); a row in several chunks adds its partial sums
// into rsum[slot] and is decided by k_lu_eval_multi.
__global__ void __launch_bounds__(256)
k_lu_eval_rows(int nch, int W, int K, int nk, int m1, const int *__restrict__ ch_row,
               const int *__restrict__ ch_e0, const int *__restrict__ ch_e1, const int *__restrict__ ch_slot,
               const int *__restrict__ ci, const int *__restrict__ val, const int64_t *__restrict__ rhs,
               const uint64_t *__restrict__ X, const int *__restrict__ XI, int *__restrict__ vcnt,
               unsigned long long *__restrict__ rsum) {
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= nch * W) return;
    const int c = g / W, w = g - c * W;
    const int j = ch_row[c];
    int64_t acc = 0;
    // 64 entries at a time: lane q loads entry q's column and coefficient and,
    // for a kept variable, its candidate word (one gather for all 64); every
    // lane then walks them in entry order through lane reads, loading only the
    // lifted integers (one coalesced load per lifted entry)
    const int e0 = ch_e0[c], e1 = ch_e1[c];
    for (int eb = e0; eb < e1; eb += 64) {
        const int e = eb + lane;
        const bool in = e < e1;
        const int cl = in ? ci[e] : 0;
        const int vl = in ? val[e] : 0;
        const uint64_t wl = (in && cl < nk) ? X[static_cast<int64_t>(cl) * W + w] : 0ull;
        const uint32_t wlo = static_cast<uint32_t>(wl), whi = static_cast<uint32_t>(wl >> 32);
        const int cnt = min(64, e1 - eb);
        for (int q = 0; q < cnt; ++q) {
            const int cq = __builtin_amdgcn_readlane(cl, q);
            const int vq = __builtin_amdgcn_readlane(vl, q);
            int64_t xv;
            if (cq < nk) {   // uniform over the wavefront
                const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wlo), q));
                const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(whi), q));
                xv = static_cast<int64_t>(((lane < 32 ? lo : hi) >> (lane & 31)) & 1u);
            } else {
                xv = static_cast<int64_t>(XI[static_cast<int64_t>(cq - nk) * K + 64 * w + lane]);
            }
            acc += static_cast<int64_t>(vq) * xv;
        }
    }
    const int slot = ch_slot[c];
    const int l = 64 * w + lane;
    if (slot < 0) {
        const bool bad = j < m1 ? acc < rhs[j] : acc != rhs[j];
        if (bad) atomicAdd(&vcnt[l], 1);
    } else {
        atomicAdd(&rsum[static_cast<int64_t>(slot) * K + l], static_cast<unsigned long long>(acc));
    }
}
__global__ void __launch_bounds__(256)
k_lu_eval_multi(int nslot, int K, int m1, const int *__restrict__ slot_row, const int64_t *__restrict__ rhs,
                const unsigned long long *__restrict__ rsum, int *__restrict__ vcnt) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= static_cast<int64_t>(nslot) * K) return;
    const int sl = static_cast<int>(t / K), l = static_cast<int>(t - static_cast<int64_t>(sl) * K);
    const int j = slot_row[sl];
    const int64_t acc = static_cast<int64_t>(rsum[t]);
    const bool bad = j < m1 ? acc < rhs[j] : acc != rhs[j];
    if (bad) atomicAdd(&vcnt[l], 1);
}

// Objective beyond the sampler's sum over kept variables: per candidate
//   zx_l = -c'_0 + sum_k c_{I_{b_k}} x_{I_{b_k}}   (k_lu_eval_lin, also the initialiser)
//        + <z_l, Q z_l>                               (k_lu_eval_quad, Q rows in chunks)
// on the lifted integer point z_l, so that the total is the reformulated
// objective <x', Q' x'> + <c', x'> = f(x) - c'_0.
__global__ void __launch_bounds__(512)
k_lu_eval_lin(int r, int K, const int64_t *__restrict__ c_tail, int64_t c0, const int *__restrict__ XI,
              int64_t *__restrict__ zx) {
    // workgroup = 64 candidates; its 8 wavefronts split the positions k
    __shared__ int64_t part[8][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int l = 64 * blockIdx.x + lane;
    int64_t acc = 0;
#pragma unroll 4
    for (int k = wv; k < r; k += 8) acc += c_tail[k] * static_cast<int64_t>(XI[static_cast<int64_t>(k) * K + l]);
    part[wv][lane] = acc;
    __syncthreads();
    if (wv == 0) {
        int64_t t = -c0;
        for (int j = 0; j < 8; ++j) t += part[j][lane];
        zx[l] = t;
    }
}
__global__ void __launch_bounds__(256)
k_lu_eval_quad(int nch, int W, int K, int nk, const int *__restrict__ ch_row, const int *__restrict__ ch_e0,
               const int *__restrict__ ch_e1, const int *__restrict__ ciQ, const int *__restrict__ valQ,
               const uint64_t *__restrict__ X, const int *__restrict__ XI, unsigned long long *__restrict__ zx) {
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= nch * W) return;
    const int c = g / W, w = g - c * W;
    const int a = ch_row[c];
    const int64_t va = lifted_val(a, nk, X, W, w, lane, XI, K);
    if (__ballot(va != 0) == 0) return;   // no candidate of the word has x_a != 0 (uniform)
    int64_t acc = 0;
    // 64 entries at a time, as in k_lu_eval_rows (every lane of the wavefront
    // takes part in the lane reads; lanes with x_a = 0 add nothing at the end)
    const int e0 = ch_e0[c], e1 = ch_e1[c];
    for (int eb = e0; eb < e1; eb += 64) {
        const int e = eb + lane;
        const bool in = e < e1;
        const int cl = in ? ciQ[e] : 0;
        const int vl = in ? valQ[e] : 0;
        const uint64_t wl = (in && cl < nk) ? X[static_cast<int64_t>(cl) * W + w] : 0ull;
        const uint32_t wlo = static_cast<uint32_t>(wl), whi = static_cast<uint32_t>(wl >> 32);
        const int cnt = min(64, e1 - eb);
        for (int q = 0; q < cnt; ++q) {
            const int cq = __builtin_amdgcn_readlane(cl, q);
            const int vq = __builtin_amdgcn_readlane(vl, q);
            int64_t xv;
            if (cq < nk) {   // uniform over the wavefront
                const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(wlo), q));
                const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(whi), q));
                xv = static_cast<int64_t>(((lane < 32 ? lo : hi) >> (lane & 31)) & 1u);
            } else {
                xv = static_cast<int64_t>(XI[static_cast<int64_t>(cq - nk) * K + 64 * w + lane]);
            }
            acc += static_cast<int64_t>(vq) * xv;
        }
    }
    if (va != 0 && acc) atomicAdd(&zx[64 * w + lane], static_cast<unsigned long long>(acc * va));
}

void launch_lu_eval_rows(hipStream_t s, int nch, int K, int nk, int m1, const int *ch_row, const int *ch_e0,
                         const int *ch_e1, const int *ch_slot, const int *ci, const int *val, const int64_t *rhs,
                         const uint64_t *X, const int *XI, int *vcnt, int64_t *rsum) {
    const int W = K / 64;
    const int64_t waves = static_cast<int64_t>(nch) * W;
    if (waves > 0)
        k_lu_eval_rows<<<static_cast<int>((waves + 3) / 4), 256, 0, s>>>(
            nch, W, K, nk, m1, ch_row, ch_e0, ch_e1, ch_slot, ci, val, rhs, X, XI, vcnt,
            reinterpret_cast<unsigned long long *>(rsum));
}
void launch_lu_eval_multi(hipStream_t s, int nslot, int K, int m1, const int *slot_row, const int64_t *rhs,
                          const int64_t *rsum, int *vcnt) {
    const int64_t t = static_cast<int64_t>(nslot) * K;
    if (t > 0)
        k_lu_eval_multi<<<static_cast<int>((t + 255) / 256), 256, 0, s>>>(
            nslot, K, m1, slot_row, rhs, reinterpret_cast<const unsigned long long *>(rsum), vcnt);
}
void launch_lu_eval_obj(hipStream_t s, int r, int K, const int64_t *c_tail, int64_t c0, const int *XI,
                        int nqch, int nk, const int *qch_row, const int *qch_e0, const int *qch_e1,
                        const int *ciQ, const int *valQ, const uint64_t *X, int64_t *zx) {
    k_lu_eval_lin<<<K / 64, 512, 0, s>>>(r, K, c_tail, c0, XI, zx);
    const int W = K / 64;
    const int64_t waves = static_cast<int64_t>(nqch) * W;
    if (waves > 0)
        k_lu_eval_quad<<<static_cast<int>((waves + 3) / 4), 256, 0, s>>>(
            nqch, W, K, nk, qch_row, qch_e0, qch_e1, ciQ, valQ, X, XI, reinterpret_cast<unsigned long long *>(zx));
}

// Fill of int32 / int64 arrays (no memset nodes in captured graphs).
__global__ void k_lu_fill_i64(int64_t *__restrict__ p, int64_t v, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_lu_fill_i64(hipStream_t s, int64_t *p, int64_t v, int64_t n) {
    if (n > 0) k_lu_fill_i64<<<static_cast<int>((n + 255) / 256), 256, 0, s>>>(p, v, n);
}
__global__ void k_lu_fill_i32(int *__restrict__ p, int v, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_lu_fill_i32(hipStream_t s, int *p, int v, int64_t n) {
    if (n > 0) k_lu_fill_i32<<<static_cast<int>((n + 255) / 256), 256, 0, s>>>(p, v, n);
}

}  // namespace gfors
