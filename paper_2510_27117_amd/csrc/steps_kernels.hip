// Whole runs of PDHG iterations (Algorithm 2) in one launch, for gfx950: a
// workgroup owns one instance, keeps its vectors in registers and LDS, and
// iterates there with two workgroup barriers per iteration.
//
// What it replaces is two launches per iteration, whose cost on small problems
// is the dispatch (about 2.7 us each in a replayed graph) and not the work.
// Three forms, by where the coefficients live:
//   k_steps_regs     sparse, each lane's entries in registers (E per lane and
//                    row / variable): LDS holds only the two gathered vectors
//   k_steps_lds      any coefficients, both orders of the matrix in LDS
//   k_steps_dense16  rows dense over the instance, int16: one copy in LDS
// Each adds its terms over the same lanes in the same order as the
// launch-per-step kernels of the same shape (k_dual<L> / k_primal<L>; the
// dense-block kernels for the last), so a run equals theirs bit for bit.
//
// The bound is latency: an LDS gather, the adds, a cross-lane sum, the update
// and a barrier, twice per iteration; no bandwidth is near its limit.  100
// iterations, launches per step against this: set cover 200 x 100, 530 us
// against 48 (k_steps_regs; 166 with the entries in LDS and shuffles through
// it); 60 knapsacks of 300 to 3,000 variables and 3 to 9 rows, 2,470 us against
// 149 (k_steps_dense16 in registers; 245 with the matrix in LDS and a second
// barrier).
#include "gfors_internal.h"

#include <algorithm>

namespace gfors {

namespace {

template <int VB>
struct Coef {
    using type = int;
};
template <>
struct Coef<2> {
    using type = int16_t;
};

// The rows and variables of instance t; local row j: its inequality rows,
// then its equality rows.
struct Inst {
    int v0, nv, r0, nr1, e0, nr;
    __device__ Inst(const ResidentArgs &A, int t)
        : v0(static_cast<int>(A.inst_var0[t])), nv(static_cast<int>(A.inst_nvar[t])), r0(0), nr1(A.m1), e0(A.m1), nr(A.m) {
        if (A.inst_rows) {
            r0 = A.inst_rows[2 * t];
            nr1 = A.inst_rows[2 * t + 2] - r0;
            e0 = A.m1 + A.inst_rows[2 * t + 1];
            nr = nr1 + A.inst_rows[2 * t + 3] - A.inst_rows[2 * t + 1];
        }
    }
    __device__ int row(int j) const { return j < nr1 ? r0 + j : e0 + (j - nr1); }
    __device__ int local(int g, int m1) const { return g < m1 ? g - r0 : nr1 + (g - e0); }
};

__device__ __forceinline__ void store_row(const ResidentArgs &A, int g, float y_prev, float y, float wy) {
    A.y_prev[g] = y_prev;
    A.y_out[g] = y;
    A.wy[g] = wy;
}
__device__ __forceinline__ void store_var(const ResidentArgs &A, int i, float xbar_before, float x_prev, float x) {
    if (A.xbar_save) A.xbar_save[i] = xbar_before;
    A.x_prev[i] = x_prev;
    A.x_out[i] = x;
    A.xbar[i] = 2.f * x - x_prev;
}

}  // namespace

// Sparse rows with the entries in registers.  A group of lpr_d lanes serves P
// rows (j = group, group + groups), a group of lpr_p lanes P variables; a lane
// holds up to E entries of each as LDS offsets (with the int16 coefficient in
// the upper half where VB = 2).  Slots past a row's end read a zero operand.
template <int VB, int E, int P>
__global__ void __launch_bounds__(kResidentThreads)
k_steps_regs(ResidentArgs A, int nsteps, int lpr_d, int lpr_p) {
    extern __shared__ __align__(16) unsigned char lds[];
    const Inst I(A, blockIdx.x);
    const int nt = blockDim.x, tid = threadIdx.x, t = blockIdx.x;
    float *xbar = reinterpret_cast<float *>(lds), *wy = xbar + (I.nv + 1);
    const int sub_d = tid & (lpr_d - 1), sub_p = tid & (lpr_p - 1);
    uint32_t ed[P][E], ep[P][E];
    float om[P], rt[P], y[P], x[P], ct[P], xb[P];
    int jr[P], iv[P];
    bool own_r[P], own_v[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int j = tid / lpr_d + p * (nt / lpr_d), i = tid / lpr_p + p * (nt / lpr_p);
        const int g = j < I.nr ? I.row(j) : 0;
        jr[p] = j;
        iv[p] = i;
        own_r[p] = j < I.nr && sub_d == 0;
        own_v[p] = i < I.nv && sub_p == 0;
        const int f = j < I.nr ? A.rp[g] : 0, len = j < I.nr ? A.rp[g + 1] - f : 0;
        const int fT = i < I.nv ? A.rpT[I.v0 + i] : 0, lenT = i < I.nv ? A.rpT[I.v0 + i + 1] - fT : 0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int e = sub_d + u * lpr_d, eT = sub_p + u * lpr_p;
            uint32_t a = 4u * static_cast<uint32_t>(e < len ? A.ci[f + e] - I.v0 : I.nv);
            uint32_t b = 4u * static_cast<uint32_t>(eT < lenT ? I.local(A.ciT[fT + eT], A.m1) : I.nr);
            if (VB == 2) {
                a |= static_cast<uint32_t>(e < len ? A.val[f + e] : 0) << 16;
                b |= static_cast<uint32_t>(eT < lenT ? A.valT[fT + eT] : 0) << 16;
            }
            ed[p][u] = a;
            ep[p][u] = b;
        }
        om[p] = j < I.nr ? A.omega[g] : 0.f;
        rt[p] = j < I.nr ? A.rt[g] : 0.f;
        y[p] = j < I.nr ? A.y_in[g] : 0.f;
        x[p] = i < I.nv ? A.x_in[I.v0 + i] : 0.f;
        ct[p] = i < I.nv ? A.ct[I.v0 + i] : 0.f;
        xb[p] = i < I.nv ? A.xbar_in[I.v0 + i] : 0.f;
        if (own_v[p]) xbar[i] = xb[p];
    }
    if (tid == 0) {
        xbar[I.nv] = 0.f;
        wy[I.nr] = 0.f;
    }
    auto at = [](const float *base, uint32_t e) {
        return *reinterpret_cast<const float *>(reinterpret_cast<const unsigned char *>(base) + (VB == 2 ? e & 0xffffu : e));
    };
    auto add = [](float s, uint32_t e, float v) {
        if (VB == 2) return fmaf(static_cast<float>(static_cast<int>(e) >> 16), v, s);
        return s + v;
    };
    const float rh = static_cast<float>(A.rho[t]);
    const float tau1 = A.tau1[t], tau2 = A.tau2[t];
    __syncthreads();
    for (int it = 0; it < nsteps; ++it) {
        const bool last = it == nsteps - 1;
        float s[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float v[E];
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = at(xbar, ed[p][u]);
            s[p] = 0.f;
#pragma unroll
            for (int u = 0; u < E; ++u) s[p] = add(s[p], ed[p][u], v[u]);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            s[p] = lane_group_sum(s[p], lpr_d);
            const float yn = dual_update(s[p], om[p], rt[p], tau2, y[p], jr[p] < I.nr1);
            if (own_r[p]) {
                wy[jr[p]] = om[p] * yn;
                if (last) store_row(A, I.row(jr[p]), y[p], yn, om[p] * yn);
            }
            y[p] = yn;
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float v[E];
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = at(wy, ep[p][u]);
            s[p] = 0.f;
#pragma unroll
            for (int u = 0; u < E; ++u) s[p] = add(s[p], ep[p][u], v[u]);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            s[p] = lane_group_sum(s[p], lpr_p);
            const float xi = x[p], xn = primal_update(s[p], ct[p], rh, tau1, xi);
            const float xo = 2.f * xn - xi;
            if (own_v[p]) {
                xbar[iv[p]] = xo;
                if (last) store_var(A, I.v0 + iv[p], xb[p], xi, xn);
            }
            x[p] = xn;
            xb[p] = xo;
        }
        __syncthreads();
    }
    if (t == 0 && tid == 0) A.ctr->k += nsteps;
}

// VB: bytes of a stored coefficient (0: all are 1).  DENSE: every row spans all
// variables of its instance, so one copy by rows serves both products and no
// index is stored.
template <int VB, bool DENSE>
__global__ void __launch_bounds__(kResidentThreads)
k_steps_lds(ResidentArgs A, int nsteps, int lpr_d, int lpr_p) {
    extern __shared__ __align__(16) unsigned char lds[];
    using VT = typename Coef<VB>::type;
    const Inst I(A, blockIdx.x);
    const int t = blockIdx.x, nt = blockDim.x, tid = threadIdx.x, nv = I.nv, nr = I.nr;
    float *xbar = reinterpret_cast<float *>(lds);
    float *x = xbar + nv, *ct = x + nv;
    float *wy = ct + nv, *y = wy + nr, *rt = y + nr, *om = rt + nr;
    int *rp = reinterpret_cast<int *>(om + nr);
    int *cp = rp + (nr + 1);
    unsigned char *tail = reinterpret_cast<unsigned char *>(DENSE ? rp : cp + (nv + 1));
    for (int i = tid; i < nv; i += nt) {
        xbar[i] = A.xbar_in[I.v0 + i];
        x[i] = A.x_in[I.v0 + i];
        ct[i] = A.ct[I.v0 + i];
    }
    for (int j = tid; j < nr; j += nt) {
        const int g = I.row(j);
        y[j] = A.y_in[g];
        rt[j] = A.rt[g];
        om[j] = A.omega[g];
    }
    VT *val = reinterpret_cast<VT *>(tail), *valT = nullptr;
    uint16_t *ix = nullptr, *ixT = nullptr;
    if (DENSE) {
        for (int j = 0; VB && j < nr; ++j) {
            const int g0 = A.rp[I.row(j)];
            for (int i = tid; i < nv; i += nt) val[j * nv + i] = static_cast<VT>(A.val[g0 + i]);
        }
    } else {
        const int b1 = A.rp[I.r0], n1 = A.rp[I.r0 + I.nr1] - b1, b2 = A.rp[I.e0];
        const int nz = n1 + A.rp[I.e0 + (nr - I.nr1)] - b2;
        const int bT = A.rpT[I.v0];
        for (int j = tid; j <= nr; j += nt)
            rp[j] = j <= I.nr1 ? A.rp[I.r0 + j] - b1 : n1 + A.rp[I.e0 + (j - I.nr1)] - b2;
        for (int i = tid; i <= nv; i += nt) cp[i] = A.rpT[I.v0 + i] - bT;
        valT = val + (VB ? nz : 0);
        ix = reinterpret_cast<uint16_t *>(valT + (VB ? nz : 0));
        ixT = ix + nz;
        for (int e = tid; e < nz; e += nt) {
            const int g = e < n1 ? b1 + e : b2 + (e - n1);
            ix[e] = static_cast<uint16_t>(A.ci[g] - I.v0);
            ixT[e] = static_cast<uint16_t>(I.local(A.ciT[bT + e], A.m1));
            if (VB) {
                val[e] = static_cast<VT>(A.val[g]);
                valT[e] = static_cast<VT>(A.valT[bT + e]);
            }
        }
    }
    const float rh = static_cast<float>(A.rho[t]);
    const float tau1 = A.tau1[t], tau2 = A.tau2[t];
    const int sub_d = tid & (lpr_d - 1), grp_d = tid / lpr_d, ngrp_d = nt / lpr_d;
    const int sub_p = tid & (lpr_p - 1), grp_p = tid / lpr_p, ngrp_p = nt / lpr_p;
    __syncthreads();
    for (int it = 0; it < nsteps; ++it) {
        const bool last = it == nsteps - 1;
        for (int b = 0; b < nr; b += ngrp_d) {
            const int j = b + grp_d;
            float s = 0.f;
            if (j < nr) {
                const int f = DENSE ? j * nv : rp[j], len = DENSE ? nv : rp[j + 1] - f;
#pragma unroll 4
                for (int e = sub_d; e < len; e += lpr_d) {
                    const float xv = xbar[DENSE ? e : ix[f + e]];
                    if (VB) s = fmaf(static_cast<float>(val[f + e]), xv, s);
                    else s += xv;
                }
            }
            s = lane_group_sum(s, lpr_d);
            if (j < nr && sub_d == 0) {
                const float o = om[j], yp = y[j], yn = dual_update(s, o, rt[j], tau2, yp, j < I.nr1);
                y[j] = yn;
                wy[j] = o * yn;
                if (last) store_row(A, I.row(j), yp, yn, o * yn);
            }
        }
        __syncthreads();
        for (int b = 0; b < nv; b += ngrp_p) {
            const int i = b + grp_p;
            float s = 0.f;
            if (i < nv) {
                const int f = DENSE ? i : cp[i], len = DENSE ? nr : cp[i + 1] - f;
#pragma unroll 4
                for (int e = sub_p; e < len; e += lpr_p) {
                    const float w = wy[DENSE ? e : ixT[f + e]];
                    if (VB) s = fmaf(static_cast<float>(DENSE ? val[e * nv + i] : valT[f + e]), w, s);
                    else s += w;
                }
            }
            s = lane_group_sum(s, lpr_p);
            if (i < nv && sub_p == 0) {
                const float xi = x[i], xn = primal_update(s, ct[i], rh, tau1, xi);
                if (last) store_var(A, I.v0 + i, xbar[i], xi, xn);
                x[i] = xn;
                xbar[i] = 2.f * xn - xi;
            }
        }
        __syncthreads();
    }
    if (t == 0 && tid == 0) A.ctr->k += nsteps;
}

// Dense int16 rows: thread k of tile q (2,048 columns, 256 threads) owns the
// eight consecutive columns 2048 q + 8 k with their x, xbar and costs in
// registers.  Coefficients: R > 0 keeps up to R rows of them in registers,
// converted; R = 0 keeps the int16 matrix in LDS and
// reads a row's eight with one 16-byte load.  Row sums: lanes, then the tile's
// four wavefronts, then the tiles in order, as k_dual_block16 and its combine
// add them.  Every wavefront then updates every row for itself (row = lane)
// and hands omega y to its lanes by lane reads, so an iteration has one barrier.
template <int R, int NT>
__global__ void __launch_bounds__(NT)
k_steps_dense16(ResidentArgs A, int nsteps) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int RM = R ? R : 64, SLOTS = NT / 64;
    __shared__ float red[2][RM][SLOTS + 1];   // + 1: rows on different banks
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int v0 = static_cast<int>(A.inst_var0[t]), nv = static_cast<int>(A.inst_nvar[t]);
    const int nr = A.blk_nrow[t], r0 = A.blk_row0[t];
    const int s8 = (nv + 7) / 8, ntile = (nv + kBlockCols - 1) / kBlockCols;
    int4 *mat = reinterpret_cast<int4 *>(lds);
    if constexpr (R == 0)
        for (int r = 0; r < nr; ++r) {
            const int4 *src = reinterpret_cast<const int4 *>(A.pval + A.pbase[r0 + r]);
            for (int q = tid; q < s8; q += static_cast<int>(blockDim.x)) mat[r * s8 + q] = src[q];
        }
    float x[8], xb[8], ct[8], a[RM][R ? 8 : 1];
    const int col = (tid >> 8) * kBlockCols + 8 * (tid & 255);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const bool in = col + k < nv;
        const int i = v0 + (in ? col + k : 0);
        x[k] = in ? A.x_in[i] : 0.f;
        xb[k] = in ? A.xbar_in[i] : 0.f;
        ct[k] = in ? A.ct[i] : 0.f;
    }
    if constexpr (R > 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int4 q = make_int4(0, 0, 0, 0);
            if (r < nr && col < nv) q = reinterpret_cast<const int4 *>(A.pval + A.pbase[r0 + r])[col / 8];
            unpack8(q, a[r]);
        }
    }
    int grow = 0;
    float om = 0.f, rt = 0.f, y = 0.f;
    if (lane < nr) {
        grow = A.blk_rows[r0 + lane];
        om = A.omega[grow];
        rt = A.rt[grow];
        y = A.y_in[grow];
    }
    const float rh = static_cast<float>(A.rho[t]);
    const float tau1 = A.tau1[t], tau2 = A.tau2[t];
    const int of = wave_sum4_of(lane);
    __syncthreads();
    for (int it = 0; it < nsteps; ++it) {
        const bool last = it == nsteps - 1;
        float(*rd)[SLOTS + 1] = red[it & 1];   // the other half is still read by slower wavefronts
        auto four = [&](int r) {
            float s[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                s[u] = 0.f;
                float b[8];
                if constexpr (R == 0) {
                    if (r + u >= nr || col >= nv) continue;
                    unpack8(mat[(r + u) * s8 + col / 8], b);
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) s[u] = fmaf(R ? a[r + u][R ? k : 0] : b[k], xb[k], s[u]);
            }
            const float v = wave_sum4(s[0], s[1], s[2], s[3]);
            if ((lane & 15) == 0 && r + of < nr) rd[r + of][tid >> 6] = v;
        };
        if constexpr (R > 0) {
#pragma unroll
            for (int r = 0; r < R; r += 4)
                if (r < nr) four(r);
        } else {
            for (int r = 0; r < nr; r += 4) four(r);
        }
        __syncthreads();
        float w = 0.f;
        if (lane < nr) {
            float s = 0.f;
            for (int q = 0; q < ntile; ++q) {
                const float *f = rd[lane] + 4 * q;
                s += ((f[0] + f[1]) + f[2]) + f[3];
            }
            const float yn = dual_update(s, om, rt, tau2, y, grow < A.m1);
            w = om * yn;
            if (last && tid < 64) store_row(A, grow, y, yn, w);
            y = yn;
        }
        auto w_of = [&](int r) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), r)); };
        float g[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) g[k] = 0.f;
        if constexpr (R > 0) {
#pragma unroll
            for (int r = 0; r < R; r += 4) {
                if (r >= nr) break;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float wr = w_of(r + u);   // 0 past the last row
#pragma unroll
                    for (int k = 0; k < 8; ++k) g[k] = fmaf(a[r + u][R ? k : 0], wr, g[k]);
                }
            }
        } else {
#pragma unroll 2
            for (int r = 0; r < nr; ++r) {
                const float wr = w_of(r);
                float b[8];
                unpack8(mat[r * s8 + min(col / 8, s8 - 1)], b);
#pragma unroll
                for (int k = 0; k < 8; ++k) g[k] = fmaf(b[k], wr, g[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float xi = x[k], xn = primal_update(g[k], ct[k], rh, tau1, xi);
            if (last && col + k < nv) store_var(A, v0 + col + k, xb[k], xi, xn);
            x[k] = xn;
            xb[k] = col + k < nv ? 2.f * xn - xi : 0.f;
        }
    }
    if (t == 0 && tid == 0) A.ctr->k += nsteps;
}

void launch_steps_resident(hipStream_t s, const ResidentArgs &A, int T, const ResidentShape &sh, int nsteps, int lpr_d,
                           int lpr_p) {
    if (sh.dense16) {
        // the coefficients in registers (8 per row and thread) while the
        // workgroup's share of the register file holds them, else in LDS
        const int tiles = (sh.nv + kBlockCols - 1) / kBlockCols;
        if (tiles == 1 && sh.nr <= 8) k_steps_dense16<8, 256><<<T, 256, 0, s>>>(A, nsteps);
        else if (tiles == 1 && sh.nr <= 16) k_steps_dense16<16, 256><<<T, 256, 0, s>>>(A, nsteps);
        else if (tiles == 1 && sh.nr <= 24) k_steps_dense16<24, 256><<<T, 256, 0, s>>>(A, nsteps);
        else if (tiles == 2 && sh.nr <= 16) k_steps_dense16<16, 512><<<T, 512, 0, s>>>(A, nsteps);
        else if (tiles <= 4 && sh.nr <= 8) k_steps_dense16<8, 1024><<<T, 256 * tiles, 0, s>>>(A, nsteps);
        else k_steps_dense16<0, 1024><<<T, 256 * tiles, sh.lds, s>>>(A, nsteps);
        return;
    }
    const int64_t lanes = std::max(static_cast<int64_t>(sh.nr) * lpr_d, static_cast<int64_t>(sh.nv) * lpr_p);
    int threads = 64;
    while (threads < kResidentThreads && threads < lanes) threads *= 2;
    // registers: at most two rows / variables per lane group and the entries
    // per lane that 128 registers hold (fewer with coefficients, which the
    // compiler unpacks ahead of the loop), local offsets below 64 KiB
    const int E = std::max((sh.len_r + lpr_d - 1) / lpr_d, (sh.len_c + lpr_p - 1) / lpr_p);
    const int P = static_cast<int>((lanes + threads - 1) / threads);
    if (!sh.dense && sh.vb != 4 && P <= 2 && E <= (sh.vb == 0 ? 16 / P : 8 / P) && std::max(sh.nv, sh.nr) < 16383) {
        const size_t lds = 4 * (static_cast<size_t>(sh.nv) + sh.nr + 2);
#define GF_REG(VB, EE, PP) k_steps_regs<VB, EE, PP><<<T, threads, lds, s>>>(A, nsteps, lpr_d, lpr_p)
        if (sh.vb == 0) {
            if (P == 2) { if (E <= 4) GF_REG(0, 4, 2); else GF_REG(0, 8, 2); }
            else if (E <= 2) GF_REG(0, 2, 1);
            else if (E <= 4) GF_REG(0, 4, 1);
            else if (E <= 8) GF_REG(0, 8, 1);
            else GF_REG(0, 16, 1);
        } else {
            if (P == 2) GF_REG(2, 4, 2);
            else if (E <= 2) GF_REG(2, 2, 1);
            else if (E <= 4) GF_REG(2, 4, 1);
            else GF_REG(2, 8, 1);
        }
#undef GF_REG
        return;
    }
#define GF_LDS(VB, D) k_steps_lds<VB, D><<<T, threads, sh.lds, s>>>(A, nsteps, lpr_d, lpr_p)
    if (sh.dense) {
        if (sh.vb == 0) GF_LDS(0, true); else if (sh.vb == 2) GF_LDS(2, true); else GF_LDS(4, true);
    } else {
        if (sh.vb == 0) GF_LDS(0, false); else if (sh.vb == 2) GF_LDS(2, false); else GF_LDS(4, false);
    }
#undef GF_LDS
}

}  // namespace gfors
