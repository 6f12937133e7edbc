// Internal declarations shared by the gfors host code and its HIP kernels.
// Device data layout (all carved from the caller's workspace):
//   constraint rows  : CSR of the ORIGINAL integer coefficients of [A; B]
//                      (inequality rows first), int32 row_ptr / col / val
//                      (val absent when every coefficient is 1); its
//                      transpose (one row per variable) for K^T y without
//                      atomics; Q in full symmetric CSR.
//   PDHG vectors     : x double-buffered (x_{k-1}, x_k), xbar, y double-
//                      buffered, wy = omega o y, FP32; omega_j = 1/(||a_j|| s_K)
//                      and rt_j = r_j omega_j per row; ct = c / s_o per variable.
//   candidates       : bit-packed, variable-major uint64 [n][K/64].
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace gfors {

// Philox4x32-10 constants (Salmon et al., SC'11).
constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

// Per-problem scalars that kernels read from device memory (so that captured
// graphs stay valid as the loop advances).
struct DevCounters {
    int64_t k;       // PDHG iterations done
    int64_t round;   // Philox sampling rounds done
    int64_t pad[6];
};

// Per-instance device arrays.
struct DevInst {
    double *rho;          // current penalty rho_n
    int64_t *ntrig;       // triggers so far (n of UpdatePenalty)
    int64_t *zbest;       // incumbent objective (INT64_MAX = none)
    int64_t *inc_k, *inc_round, *inc_l;
    int32_t *improved;    // set by the last incumbent update
    int32_t *inc_W;       // words-per-variable of the round that produced the incumbent
    double *rho_min, *rho_max, *rho_T, *rho_p, *rho_delta;
    float *tau1, *tau2, *two_so;   // per-instance FP32 scalars (batched kernels)
    double *tau1d, *tau2d, *two_sod;
    int64_t *hist;        // [T][hist_cap] incumbent after each round
    int32_t hist_cap;
};

// Tile tables.  A tile is a piece of work that never crosses an instance.
struct Tiles {
    int32_t count = 0;
    int32_t *inst = nullptr;   // instance of each tile
    int32_t *b0 = nullptr;     // begin (quad / list position / row / var)
    int32_t *b1 = nullptr;     // end
    int32_t *first = nullptr;  // [T+1] first tile of each instance (tiles sorted by instance)
};

// Launch shapes picked per problem (heuristic or timed by the autotuner).
// slices: 1 = fused CSR kernel; > 1 = XCD-sliced partial SpMV + combine.
struct LaunchCfg {
    int lpr_dual = 16;     // lanes per row for the dual SpMV
    int lpr_primal = 4;    // lanes per row for the transposed SpMV (+Q)
    int slices_dual = 1;
    int slices_primal = 1;
    int sell_dual = 0;     // 1: SELL-64 layout (lane = row) instead of CSR
    int sell_primal = 0;
    int bits_dual = 0;     // 1: skip zero operands through an LDS bitmap
    int bits_primal = 0;
};

constexpr int64_t kMaxLdsBitmapBytes = 64 * 1024;

// A SELL-64 matrix (possibly cut into P column slices, each with nchunk chunks).
struct SellView {
    int nrows = 0, P = 1, nchunk = 0, ns = 0;   // ns: columns per slice (multiple of 64)
    const int *ptr = nullptr, *ci = nullptr, *val = nullptr, *row_of = nullptr;
    // per slot: first column of a row whose entries in the slice are one
    // contiguous range (else -1) and the row's entry count in the slice
    const int *c0 = nullptr, *len = nullptr;
    const int16_t *val16 = nullptr;   // the coefficients as int16 when all fit (else null)
};

constexpr int kXcdSlices = 8;   // XCDs per MI355X
// Evaluation kinds of rows whose violation is a bitwise function of the
// candidate words (per-row byte: kind << 4 | truth table of pair rows).
constexpr int kEvalCover = 0;        // inequality, coefficients 1, rhs 1:  violated iff none set
constexpr int kEvalAtMostOne = 1;    // inequality, coefficients -1, rhs -1: violated iff >= 2 set
constexpr int kEvalExactlyOne = 2;   // equality, coefficients +-1, rhs +-1: violated iff != 1 set
constexpr int kEvalPair = 3;         // one or two entries: truth table over (x_p, x_q)
constexpr int kLprBlock = 256;  // launch shape "a workgroup of 256 lanes per row"; 256 + L:
                                // rows of kHeavyLen+ entries a workgroup each, others L lanes
constexpr int kHeavyLen = 256;
constexpr int kLightHole = 0x7fffffff;   // signed-index slot of a heavy item inside the light range
constexpr int kHgChunk = 512;   // entries per workgroup of the heavy shift-group primal
constexpr int kHgWidth = 16;    // variables per shift group (32 measured slower: fewer entries in flight)

// ------------------------------------------------- sums over a wavefront's lanes
// v[l] + v[l ^ D] in every lane, on the vector ALU (row permutations and the
// half / quarter swaps of gfx950; a shuffle through LDS takes about ten times
// as long).  The addends are those of v + __shfl_xor(v, D), so are the bits.
template <int CTRL, int BANKS = 0xf>
__device__ __forceinline__ float dpp_move(float old, float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xf, BANKS, false));
}
template <int D>
__device__ __forceinline__ float xor_sum(float v) {
    if constexpr (D == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else if constexpr (D == 8) {
        return v + dpp_move<0x128>(v, v);                       // row_ror:8
    } else if constexpr (D == 4) {
        float t = dpp_move<0x104, 0x5>(v, v);                   // row_shl:4 into banks 0, 2
        t = dpp_move<0x114, 0xa>(t, v);                         // row_shr:4 into banks 1, 3
        return v + t;
    } else if constexpr (D == 2) {
        return v + dpp_move<0x4e>(v, v);                        // quad_perm 2 3 0 1
    } else {
        return v + dpp_move<0xb1>(v, v);                        // quad_perm 1 0 3 2
    }
}
// Sums of a, b, c, d over the wavefront (the same tree as xor_sum<32> .. <1>
// each) for the price of one and a half: lane 0 holds a's, 16 c's, 32 b's, 48 d's.
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d) {
    const auto ab = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    const auto cd = __builtin_amdgcn_permlane32_swap(__float_as_uint(c), __float_as_uint(d), false, false);
    const float p = __uint_as_float(ab[0]) + __uint_as_float(ab[1]), q = __uint_as_float(cd[0]) + __uint_as_float(cd[1]);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v = xor_sum<8>(v);
    v = v + dpp_move<0x124>(v, v);                              // row_ror:4 (the row repeats every 8 lanes)
    v = xor_sum<2>(v);
    return xor_sum<1>(v);
}
// The same of a double, its two halves moved as above.
template <int D>
__device__ __forceinline__ double xor_sum(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    if constexpr (D >= 16) {
        auto swap = [](int w) {
            if constexpr (D == 32) return __builtin_amdgcn_permlane32_swap(w, w, false, false);
            else return __builtin_amdgcn_permlane16_swap(w, w, false, false);
        };
        const auto l = swap(lo), h = swap(hi);
        return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    } else {
        auto partner = [](int w) {
            const float f = __int_as_float(w);
            if constexpr (D == 8) return __float_as_int(dpp_move<0x128>(f, f));
            else if constexpr (D == 4) return __float_as_int(dpp_move<0x114, 0xa>(dpp_move<0x104, 0x5>(f, f), f));
            else if constexpr (D == 2) return __float_as_int(dpp_move<0x4e>(f, f));
            else return __float_as_int(dpp_move<0xb1>(f, f));
        };
        return v + __hiloint2double(partner(hi), partner(lo));
    }
}
// Sum over groups of L lanes (a power of two <= 64), widest distance first.
template <typename T>
__device__ __forceinline__ T lane_group_sum(T v, int L) {
    if (L >= 64) v = xor_sum<32>(v);
    if (L >= 32) v = xor_sum<16>(v);
    if (L >= 16) v = xor_sum<8>(v);
    if (L >= 8) v = xor_sum<4>(v);
    if (L >= 4) v = xor_sum<2>(v);
    if (L >= 2) v = xor_sum<1>(v);
    return v;
}
// Which of wave_sum4's operands (0..3) a lane's quarter holds.
__device__ __forceinline__ int wave_sum4_of(int lane) {
    const int q = lane >> 4;
    return ((q & 1) << 1) | (q >> 1);
}

// Eight int16 values of a 16-byte load as floats.
__device__ __forceinline__ void unpack8(const int4 q, float *a) {
    const uint32_t w[4] = {static_cast<uint32_t>(q.x), static_cast<uint32_t>(q.y), static_cast<uint32_t>(q.z),
                           static_cast<uint32_t>(q.w)};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        a[2 * h] = static_cast<float>(static_cast<int16_t>(w[h] & 0xffffu));
        a[2 * h + 1] = static_cast<float>(static_cast<int16_t>(w[h] >> 16));
    }
}

// ------------------------------------------------------------------ PDHG
// The updates that end a row's / a variable's sum (Algorithm 2, Q = 0).
__device__ __forceinline__ float dual_update(float s, float om, float rt, float tau2, float y_in, bool ineq) {
    const float t = rt - om * s;
    float y = y_in + tau2 * t;
    if (ineq) y = fmaxf(y, 0.f);
    return y;
}
__device__ __forceinline__ float primal_update(float s, float ct, float rh, float tau1, float xi) {
    float g = ct + rh;
    g -= s;
    g -= 2.f * rh * xi;
    return fminf(fmaxf(xi - tau1 * g, 0.f), 1.f);
}

// Runs of PDHG steps with each instance in one workgroup (k_steps_*).
constexpr int kResidentThreads = 1024;   // largest workgroup
struct ResidentArgs {
    int m1 = 0, m = 0;
    const int64_t *inst_var0 = nullptr, *inst_nvar = nullptr;
    const int *inst_rows = nullptr;   // [T+1][2] first inequality / equality row; null: one instance
    const int *rp = nullptr, *ci = nullptr, *val = nullptr, *rpT = nullptr, *ciT = nullptr, *valT = nullptr;
    const float *omega = nullptr, *rt = nullptr, *ct = nullptr, *tau1 = nullptr, *tau2 = nullptr;
    const double *rho = nullptr;
    // dense rows in int16 (k_steps_dense16): the padded copy of the dense-block kernels
    const int *blk_row0 = nullptr, *blk_nrow = nullptr, *blk_rows = nullptr;
    const int64_t *pbase = nullptr;
    const int16_t *pval = nullptr;
    // state before; after (x_k, x_{k-1}, y_k, y_{k-1}, xbar, wy); xbar before the last step if wanted
    const float *x_in = nullptr, *y_in = nullptr, *xbar_in = nullptr;
    float *x_out = nullptr, *x_prev = nullptr, *y_out = nullptr, *y_prev = nullptr, *xbar = nullptr, *wy = nullptr;
    float *xbar_save = nullptr;
    DevCounters *ctr = nullptr;
};
// What the launch needs to know of the problem: bytes of a stored coefficient
// (0 when all are 1, 2 or 4), dense rows, the largest instance and its longest
// row / variable, the LDS that the form with the matrix in LDS takes, and the
// lanes per row / variable that its rule gives.
struct ResidentShape {
    int vb = 0, nv = 0, nr = 0, len_r = 0, len_c = 0, lpr_d = 1, lpr_p = 1;
    bool dense = false, dense16 = false;
    size_t lds = 0;
};
// Dense int16 rows: whether the coefficients stay in registers (eight columns of
// up to 24, 16 or 8 rows a thread of one, two or four tiles), else in LDS.
inline bool resident16_regs(const ResidentShape &sh) {
    const int tiles = (sh.nv + 2047) / 2048;
    return tiles == 1 ? sh.nr <= 24 : tiles == 2 ? sh.nr <= 16 : tiles <= 4 && sh.nr <= 8;
}
void launch_steps_resident(hipStream_t s, const ResidentArgs &A, int T, const ResidentShape &sh, int nsteps, int lpr_d,
                           int lpr_p);

// val16: the coefficients as int16 when every |a| <= 32767 (else null)
void launch_dual(hipStream_t s, int lpr, bool unit, bool batched, int m, int m1,
                 const int *rp, const int *ci, const int *val, const int16_t *val16, const float *omega,
                 const float *rt, const float *xbar, const float *y_in, float *y_out,
                 float *wy, float tau2, const float *tau2_inst, const int *row_inst,
                 int skip_len);

// The update of a variable without rows, s2 = (Q x)_i.
__device__ __forceinline__ float primal_update_q(float s2, float ct, float rh, float two_so, float tau1, float xi) {
    float g = ct + rh;
    g = fmaf(two_so, s2, g);
    g -= 2.f * rh * xi;
    return fminf(fmaxf(xi - tau1 * g, 0.f), 1.f);
}
// The step over codes (two bits per variable) of x, up to kCodesLanes lanes per
// row.  A table that fits in LDS bounds n above; below, its latency does (us a step,
// this kernel against k_primal, ten entries a row: 5.8 : 4.3 at 50,000 variables,
// 6.3 : 6.6 at 100,000, 7.7 : 11.3 at 200,000, 17.6 : 25.5 at 500,000).  Longer rows
// narrow the lead (40 entries: 28 : 36) and leave less to gain from 4 lanes; a single
// long row is walked by its 4 lanes alone while k_primal's tuned lanes go up to 64
// (200,000 variables of ten entries and one row of 64, 128, 256, 1,024 entries:
// 11.3 : 15.0, 14.4 : 15.0, 20.0 : 16.9, 56 : 25; 90,000 entries: 3,712 : 482).
constexpr int64_t kMinCodes = 1 << 17, kMaxCodes = 128 * 1024 * 4, kCodesPerRow = 64, kCodesLongest = 128;
constexpr int kCodesLanes = 4;
// LDS of a workgroup: the codes of every block of 64 variables, and a block of zeros
constexpr size_t primal_codes_lds(int64_t n) { return static_cast<size_t>((n + 63) / 64 + 1) * 16; }
void launch_q_codes(hipStream_t s, int n, const float *x, uint4 *codes);
void launch_primal_codes(hipStream_t s, int lpr, int n, const int *rpQ, const int *packQ, const float *x_in,
                         const uint4 *codes_in, uint4 *codes_out, float *x_out, float *xbar, const float *ct, float tau1,
                         float two_so, const double *rho, DevCounters *ctr);
// How k_primal reads Q: not at all, an index and an int32 value per entry, or both
// in a word (24 + 8 bits, ciQ points at the words).
constexpr int kQInt32 = 1, kQPacked = 2;
void launch_primal(hipStream_t s, int lpr, int kmode, int qmode, bool batched, int n,
                   const int *rpT, const int *colT0, const int *ciT, const int *valT, const float *wy,
                   const int *rpQ, const int *ciQ, const int *valQ, const float *x_in,
                   float *x_out, float *xbar, const float *ct, float tau1, float two_so,
                   const float *tau1_inst, const float *two_so_inst, const double *rho,
                   const int *var_inst, DevCounters *ctr, int skip_len);
// Heavy rows / variables, a workgroup each, taken in `order` (longest first).
// rowc0: first column of a dense row, else -1; val16: the coefficients as int16
// when all fit (else null); rowunit: rows whose coefficients are all 1 (or null).
struct DualLongArgs {
    int count = 0, m1 = 0;
    const int *order = nullptr, *rp = nullptr, *rowc0 = nullptr, *ci = nullptr, *val = nullptr;
    const int16_t *val16 = nullptr;
    const uint8_t *rowunit = nullptr;
    const float *omega = nullptr, *rt = nullptr, *xbar = nullptr, *y_in = nullptr;
    float *y_out = nullptr, *wy = nullptr;
};
struct PrimalLongArgs {
    int count = 0;
    const int *order = nullptr, *rpT = nullptr, *ciT = nullptr, *valT = nullptr;
    const float *wy = nullptr, *x_in = nullptr;
    float *x_out = nullptr, *xbar = nullptr;
    const float *ct = nullptr;
    const double *rho = nullptr;
};
// Heavy variables in shift groups (k_primal_light): launch slots, chunks, groups.
struct HgroupArgs {
    int nslot = 0, ngroup = 0;
    const int *ord = nullptr, *ch_g = nullptr, *ch_b = nullptr, *ch_e = nullptr;
    const int *var0 = nullptr, *w = nullptr, *e0 = nullptr, *c0 = nullptr, *ciT = nullptr, *valT = nullptr;
    const float *wy = nullptr;
    float *part = nullptr;
};
void launch_primal_long(hipStream_t s, bool unit, bool batched, const PrimalLongArgs &A, float tau1,
                        const float *tau1_inst, const int *var_inst);

void launch_spmv_part(hipStream_t s, int lpr, bool unit, int nrows, int P, const int *rpP,
                      const int *ci, const int *val, const float *v, float *part);
void launch_dual_combine(hipStream_t s, bool batched, int m, int m1, int P, const float *part,
                         const float *omega, const float *rt, const float *y_in, float *y_out,
                         float *wy, float tau2, const float *tau2_inst, const int *row_inst,
                         uint64_t *wybits);
void launch_primal_combine(hipStream_t s, bool batched, int n, int P, const float *part,
                           const float *x_in, float *x_out, float *xbar, const float *ct,
                           float tau1, const float *tau1_inst, const double *rho,
                           const int *var_inst, DevCounters *ctr, uint64_t *xbits);

void launch_sell(hipStream_t s, const SellView &sv, int mode, bool unit, bool batched,
                 const float *v, float *part, int m1, const float *omega, const float *rt,
                 const float *y_in, float *y_out, float *wy, float tau2, const float *tau2_inst,
                 const int *row_inst, const float *x_in, float *x_out, float *xbar,
                 const float *ct, float tau1, const float *tau1_inst, const double *rho,
                 const int *var_inst, DevCounters *ctr);

void launch_nzbits(hipStream_t s, const float *v, int64_t n, int64_t nwords64, uint64_t *bits);
void launch_dual_long(hipStream_t s, bool unit, bool batched, const DualLongArgs &A, float tau2,
                      const float *tau2_inst, const int *row_inst);
void launch_sell_bits(hipStream_t s, const SellView &sv, int mode, bool unit, bool batched,
                      int ncols, const float *v, const uint32_t *bits, float *part, int m1,
                      const float *omega, const float *rt, const float *y_in, float *y_out,
                      float *wy, float tau2, const float *tau2_inst, const int *row_inst,
                      const float *x_in, float *x_out, float *xbar, const float *ct, float tau1,
                      const float *tau1_inst, const double *rho, const int *var_inst,
                      DevCounters *ctr, int nc);
int sell_bits_blocks(const SellView &sv, int nc);
void launch_sell_part_bits(hipStream_t s, const SellView &sv, int ns, int ncols, bool unit,
                           const float *v, const uint32_t *bits, float *part);
void launch_primal_bits(hipStream_t s, int lpr, bool unit, bool batched, int n, int m,
                        const int *rpT, const int *ciT, const int *valT, const float *wy,
                        const uint32_t *bits, const float *x_in, float *x_out, float *xbar,
                        const float *ct, float tau1, const float *tau1_inst, const double *rho,
                        const int *var_inst, DevCounters *ctr, uint64_t *xbits, int deg);

// Dense-block SpMVs of batched instances whose rows are dense over their
// instance's variables (at most 64 rows per instance, no Q).
struct BlockView {
    int ntile = 0;
    const int *tile_inst = nullptr, *tile_c0 = nullptr;   // per tile: instance, first column
    const int *row0 = nullptr, *nrow = nullptr;            // per instance: its rows in `rows`
    const int *rows = nullptr;                             // rows of each instance, in order
    const int *row_rank = nullptr;                         // per row: index within its instance
    const int *inst_tile0 = nullptr, *inst_ntile = nullptr;   // per instance: its tiles
    float *pp = nullptr;                                   // per tile: 64 row sums
    // padded int16 copy (each row of an instance at a multiple of 8 entries,
    // zero past its end; null when absent) and the first entry of every row
    // of `rows` in it
    const int16_t *pval = nullptr;
    const int64_t *pbase = nullptr;
};
// A step of the padded int16 form in one launch: rows from the tile sums pp_in
// (launch_dual_block_sums before the first step), the primal step, and the tile
// sums of the next step into pp_out (null: the last step of a run).
void launch_dual_block_sums(hipStream_t s, const BlockView &b, const int64_t *inst_var0, const int64_t *inst_nvar,
                            const float *xbar, float *pp);
void launch_step_block(hipStream_t s, const BlockView &b, int m1, const int64_t *inst_var0, const int64_t *inst_nvar,
                       const float *pp_in, float *pp_out, const float *omega, const float *rt,
                       const float *tau2_inst, const float *y_in, float *y_out, float *wy, const float *x_in,
                       float *x_out, float *xbar, const float *ct, const float *tau1_inst, const double *rho,
                       DevCounters *ctr);
constexpr int kBlockCols = 2048;   // columns per tile of the dense-block SpMVs (256 threads x 8)
void launch_dual_block(hipStream_t s, const BlockView &b, int m, int m1, const int *rp, const int *val,
                       const int16_t *val16, const int64_t *inst_var0, const int64_t *inst_nvar,
                       const float *xbar, const float *omega, const float *rt, const float *tau2_inst,
                       const int *row_inst, const float *y_in, float *y_out, float *wy);
void launch_primal_block(hipStream_t s, const BlockView &b, const int *rp, const int *val, const int16_t *val16,
                         const int64_t *inst_var0, const int64_t *inst_nvar, const float *wy,
                         const float *x_in, float *x_out, float *xbar, const float *ct, const float *tau1_inst,
                         const double *rho, DevCounters *ctr);

// Primal step with wy staged in LDS slices of SL rows (unit coefficients,
// every variable in deg <= 8 rows, one instance, no Q); ell[u n + i] = the
// u-th row of variable i (ascending).  Returns false for an unsupported deg.
int primal_lds_slice(size_t lds_limit, int64_t m);
// Light rows / variables [i0, i0 + L) of D <= 8 entries each, indices entry-major
// with the coefficient's sign (|a| = 1) in bit 31; one instance, no Q.  xbits:
// nonzero bitmap of xbar (only when the range is every variable), or null.
// The heavy items of A (or of the shift groups G) ride in the same launch.
void launch_dual_light(hipStream_t s, bool unit, int D, const DualLongArgs &A, int i0, int L, const int *sidx,
                       float tau2);
void launch_primal_light(hipStream_t s, bool unit, int D, const PrimalLongArgs &A, const HgroupArgs *G, int i0, int L,
                         const int *sidx, float tau1, DevCounters *ctr, uint64_t *xbits);
bool launch_primal_lds(hipStream_t s, int n, int m, int deg, int SL, const int *ell, const float *wy,
                       const float *x_in, float *x_out, float *xbar, const float *ct, float tau1,
                       const double *rho, DevCounters *ctr, uint64_t *xbits);

void launch_copy_f32(hipStream_t s, float *dst, const float *src, int64_t n);
void launch_set_xbar(hipStream_t s, int64_t n, const float *x, const float *xp, float *xbar);
void launch_fill_f32(hipStream_t s, float *dst, float v, int64_t n);
// dst[i] = v for a pseudorandom `percent` of the entries, else 0 (stand-in iterates)
void launch_fill_share(hipStream_t s, float *dst, float v, int percent, int64_t n);

// ------------------------------------------------- FP64 (Preprocess, residuals)
void launch_spmv64(hipStream_t s, int nrows, const int *rp, const int *ci, const int *val,
                   const double *rowscale, const double *v, double *w);
void launch_scale64(hipStream_t s, int64_t n, double *x, const double *a, double sign);
void launch_fill64(hipStream_t s, double *x, double v, int64_t n);
void launch_tile_sumsq(hipStream_t s, const Tiles &t, const double *x, double *part);
void launch_inst_sum(hipStream_t s, int T, const Tiles &t, const double *part, int stride,
                     int comp, double *out, int out_stride, bool take_sqrt);
void launch_tile_scale_inv(hipStream_t s, const Tiles &t, double *x, const double *nrm);

void launch_res_rows(hipStream_t s, const Tiles &rt, int m1, const int *rp, const int *ci,
                     const int *val, const double *omega64, const int64_t *rhs,
                     const float *xsave, const float *x, const float *y_prev,
                     const float *y, const double *tau2d, double *part);
void launch_res_vars(hipStream_t s, const Tiles &vt, const int *rpQ, const int *ciQ,
                     const int *valQ, const float *x, const float *xp, const double *rho,
                     const double *tau1d, const double *two_sod, double *part);

// --------------------------------------------------------- sampling / eval
void launch_philox_peak(hipStream_t s, int blocks, int iters, uint32_t *sink);
void launch_read_peak(hipStream_t s, int blocks, const void *p, int64_t n16, uint32_t *sink);
// Monotone relaxation repair (Sec. 2.4) of the sampled candidates: in each of
// the nrows relaxed set-partitioning rows (variables var[rp[r]..rp[r+1]) in
// (cost, index) order) only the first set variable of every candidate stays
// set; cleared costs are taken off the candidates' objectives in zpart[0..K).
void launch_mono_repair(hipStream_t s, int nrows, int W, int K, const int *rp, const int *var,
                        const int64_t *cost, uint64_t *X, uint8_t *xkind, int64_t *zpart);
// Customized 3D-assignment sampler (Algorithm 4): candidates of an n x n x n
// assignment from p into X (cleared first, with zpart[0, nzpart) and xkind),
// objectives into zpart[0 .. K); part: int[2 n] scratch.
constexpr int kA3MaxN = 1024;     // largest n
constexpr int kA3MaxTop = 4096;   // largest gamma n
void launch_a3(hipStream_t s, const float *p, int n, int m, int K, int L, uint32_t key0,
               uint32_t key1, const DevCounters *ctr, const int64_t *cost, int *part, uint64_t *X,
               int W, int64_t *zpart, int64_t nzpart, uint8_t *xkind);
void launch_sample(hipStream_t s, int W, bool obj64, const float *p, const int64_t *cost,
                   uint64_t *X, const Tiles &st, const int64_t *inst_var0,
                   const int64_t *inst_nvar, int64_t *zpart, int K, uint32_t key0,
                   uint32_t key1, const DevCounters *ctr, int threshold_mode, uint8_t *xkind);

void launch_eval_cover(hipStream_t s, int ntiles, const int *tile_ids, const Tiles &et,
                       const int *rows, const uint8_t *rkind, const int *rp, const int *ci,
                       const uint64_t *X, const uint8_t *xkind, int W, int *vpart, int K,
                       bool pair_rows);   // most rows of two entries: four rows in flight per group
void launch_eval_general(hipStream_t s, int ntiles, const int *tile_ids, const Tiles &et,
                         bool acc64, const int *rows, const int *rp, const int *ci,
                         const int *val, const int64_t *rhs, int m1, const uint64_t *X,
                         const uint8_t *xkind, int W, int *vpart, int K, bool long_rows,
                         bool coef24);
// Tiles of <= 32 general rows densified as int8 digit planes (npl in 1..3);
// acc64: some row's sum of |a| reaches 2^31.
void launch_eval_mfma(hipStream_t s, int ntiles, const int *tile_ids, const Tiles &et, int npl, bool acc64,
                      const int *rows, const int64_t *mf_off, const int *mf_c0, const int *mf_span,
                      const int8_t *dig, const int64_t *rhs, int m1, const uint64_t *X, int W,
                      int *vpart, int K);
// Entries of one magnitude; at most kQuadBitsMax of them in a tile (16-bit counts).
constexpr int64_t kQuadBitsMax = 65535;
void launch_eval_quad_bits(hipStream_t s, const Tiles &qt, const int *rpQ, const int *rowQ, const int *ciQ,
                           const int *valQ, const uint64_t *X, const uint8_t *xkind, int W, int mag, int64_t *zqpart,
                           int K);
void launch_eval_quad(hipStream_t s, const Tiles &qt, const int *rpQ, const int *rowQ,
                      const int *ciQ, const int *valQ, const uint64_t *X, int W, int64_t *zqpart,
                      int K, bool q24);
void launch_reduce_cand(hipStream_t s, int T, int K, int S, const Tiles &et, const int *vpart,
                        const Tiles &st, const int64_t *zpart, const Tiles &qt,
                        const int64_t *zqpart, int has_q, int32_t *rv, int64_t *rz,
                        int32_t *viol, int64_t *z);
// S: the slices of launch_reduce_cand; with S = 1 that launch is left out and the
// per-tile partials are added here.
void launch_argmin_update(hipStream_t s, int T, int K, int W, int S, const Tiles &et, const int *vpart,
                          const Tiles &st, const int64_t *zpart, const Tiles &qt, const int64_t *zqpart, int has_q,
                          int32_t *viol, int64_t *z, DevInst di, DevCounters *ctr, int advance);
void launch_extract_best(hipStream_t s, int64_t n, int T, const int *var_inst, const uint64_t *X,
                         DevInst di, uint8_t *xbest, DevCounters *ctr, int advance);

// ---------------------------------------------------------------------------
// Factorised TU reformulation (lu_kernels.hip)
// ---------------------------------------------------------------------------
// A run of a level-scheduled in-place triangular solve: levels [a, b) in one
// workgroup (wide = 0), or positions [a, b) of one wide level (wide = 1).
struct LuSeg {
    int wide, a, b;
};
// Device arrays of one solve (positions in level order) and its launch plan
// (host array).
struct LuSolve {
    int r = 0, nseg = 0;
    int use_lds = 1;   // stage the vector and the run in LDS for one-workgroup runs when they fit
    const int *row = nullptr, *ptr = nullptr, *ent = nullptr, *lvl = nullptr;
    const LuSeg *seg = nullptr;
    // host copies: first position of each level, first entry of each level's first position
    const int *hlvl = nullptr, *hptr_at_lvl = nullptr;
};
// LDS that a one-workgroup run may stage the solved vector in (of the 160 KB).
constexpr size_t kLuLdsBytes = 128 * 1024;

// In-place solve; with x32 given also x32 = x rounded, and with xbar given
// xbar[k] = 2 x32[k] - xold[k].
void launch_lu_trsv(hipStream_t s, const LuSolve &sv, double *x, float *x32 = nullptr, const float *xold = nullptr,
                    float *xbar = nullptr);
void launch_lu_mv_f32(hipStream_t s, int lpr, int nrows, const int *rp, const int *ci, const int *val,
                      const float *x, double *y, double sgn);
void launch_lu_mv_f64(hipStream_t s, int lpr, int nrows, const int *rp, const int *ci, const int *val,
                      const double *x, double *y, double sgn, bool accumulate);
void launch_lu_tail_grad(hipStream_t s, int lpr, bool hasq, int r, int nk, const int *rpT, const int *ciT,
                         const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                         const float *x, const float *two_so, double *v);
void launch_lu_primal(hipStream_t s, int lpr, bool hasq, int nk, const int *rpT, const int *ciT,
                      const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                      const int *rpB, const int *ciB, const int *valB, const double *u, const float *x_in,
                      float *x_out, float *xbar, const float *ct, const float *tau1, const float *two_so,
                      const double *rho, DevCounters *ctr);
// The dual step's row sums: chunks of the heavy rows into part, the other rows
// (lpr lanes each) updated; launch_lu_dual_heavy then ends the heavy rows.
struct LuDualArgs {
    int m = 0, m1 = 0, nchunk = 0, skip_len = 0;
    bool rows = true;                    // some row is not heavy
    const int *ch_row = nullptr, *ch_e0 = nullptr, *ch_e1 = nullptr, *rowc0 = nullptr, *rp = nullptr, *ci = nullptr,
              *val = nullptr;
    const float *xbar = nullptr, *omega = nullptr, *rt = nullptr, *y_in = nullptr;
    double *part = nullptr;
    float *y_out = nullptr, *wy = nullptr;
    float tau2 = 0.f;
};
struct LuHeavyArgs {
    int nheavy = 0, m1 = 0;
    const int *first = nullptr, *order = nullptr;
    const double *part = nullptr;
    const float *omega = nullptr, *rt = nullptr, *y_in = nullptr;
    float *y_out = nullptr, *wy = nullptr;
    float tau2 = 0.f;
};
void launch_lu_dual(hipStream_t s, int lpr, const LuDualArgs &A);
void launch_lu_dual_heavy(hipStream_t s, const LuHeavyArgs &A);
// One workgroup for what lies between the row sums and the primal step: the
// heavy rows' updates, the pivot gradient and both transposed solves; and for
// the lift's two solves.  lu_fits: whether a pair of solves qualifies (not
// without levels: there is nothing to save then).  lu_threads: its workgroup.
constexpr int kLuOneMax = 1024;   // pivots of the one-workgroup form (a thread each)
bool lu_fits(const LuSolve &a, const LuSolve &b);
int lu_threads(int r);
void launch_lu_mid(hipStream_t s, const LuHeavyArgs &H, int lpr, bool hasq, int r, int nk, const int *rpT,
                   const int *ciT, const int *valT, const float *wy, const int *rpQ, const int *ciQ, const int *valQ,
                   const float *x, const float *two_so, const LuSolve &a, const LuSolve &b, double *v);
void launch_lu_lift(hipStream_t s, int r, const LuSolve &a, const LuSolve &b, const double *t, float *x32,
                    const float *xold, float *xbar);
void launch_lu_xbar_tail(hipStream_t s, int r, int nk, const float *x_new, const float *x_old, float *xbar);
void launch_lu_diff64(hipStream_t s, int n, const float *a, const float *b, double *d);
void launch_lu_res_rows(hipStream_t s, const Tiles &rt, int m1, const int *rp, const int *ci, const int *val,
                        const double *omega64, const int64_t *rhs, const double *d1, const double *d2,
                        const float *y_prev, const float *y, const double *tau2d, double *part);
void launch_lu_res_vars(hipStream_t s, const Tiles &vt, const double *qd, const float *x, const float *xp,
                        const double *rho, const double *tau1d, const double *two_sod, double *part);
void launch_lu_trsm(hipStream_t s, const LuSolve &sv, int *XI, int K);
void launch_lu_eval_rhs(hipStream_t s, int r, int K, const int *rp, const int *ci, const int *val,
                        const int64_t *dJ, const uint64_t *X, int *XI);
void launch_lu_eval_rows(hipStream_t s, int nch, int K, int nk, int m1, const int *ch_row, const int *ch_e0,
                         const int *ch_e1, const int *ch_slot, const int *ci, const int *val, const int64_t *rhs,
                         const uint64_t *X, const int *XI, int *vcnt, int64_t *rsum);
void launch_lu_eval_multi(hipStream_t s, int nslot, int K, int m1, const int *slot_row, const int64_t *rhs,
                          const int64_t *rsum, int *vcnt);
void launch_lu_eval_obj(hipStream_t s, int r, int K, const int64_t *c_tail, int64_t c0, const int *XI,
                        int nqch, int nk, const int *qch_row, const int *qch_e0, const int *qch_e1,
                        const int *ciQ, const int *valQ, const uint64_t *X, int64_t *zx);
void launch_lu_fill_i64(hipStream_t s, int64_t *p, int64_t v, int64_t n);
void launch_lu_fill_i32(hipStream_t s, int *p, int v, int64_t n);

}  // namespace gfors
