// Column sweep of the layer-wise quantizer (Sec. 4.3 of the paper: quantize one column, propagate its
// residual to the columns not yet quantized) on the per-group asymmetric min-max grid (Eq. (1), (2), (4)).
//
// Per output row, for sweep positions j = 0 .. d_in-1:
//   group start:  s = (max - min) / (2^b - 1) of the current values of the group (1 if max == min),
//                 z = clamp(rne(-min / s), 0, 2^b - 1)
//   q = clamp(rne(w_j / s) + z, 0, 2^b - 1),  w^ = s (q - z),  e = (w_j - w^) / U_jj
//   (w_j / s and the division by U_jj are multiplications by correctly rounded fp64 reciprocals),
//   w_k -= e U_jk for k > j.
//
// Precision.  A code is rne(w_j / s); one wrong rounding at a near-tie changes the rest of its row, so the value
// that is rounded has to agree with exact arithmetic to about 1e-7 of a grid step over thousands of columns.  The
// library therefore never stores the compensated weight w_j itself in fp32.  It keeps the ORIGINAL weight (exact)
// and, apart from it, the feedback sum  c_j = -sum_{i<j} e_i U_ij  (a fraction of a grid step, so its fp32 rounding
// is ~1e-8 of a step): the working copy in memory holds c, every MFMA accumulation starts from zero and is added
// to c once, and inside a 32-column inner block the values w = w0 + c, the scale, the decision and the feedback
// run in fp64 registers.
//
// gfx950 schedule (lazy batch of B = 128 columns inside super-blocks of up to 512 columns):
//   panel kernel    64 rows per workgroup carried through the blocks of a super-block: the feedback between the
//                   super-block's blocks is applied inside the kernel (split-fp16 MFMAs on operands stored in
//                   fragment order), the sequential part runs four lanes per row with DPP broadcasts, the rest of
//                   a block is updated with fp32 MFMAs on tiles in LDS.  See panel_body.
//   far update      W[:, cols] += D Un[rows, cols] for the columns beyond a super-block, once per super-block
//                   (K = its width), as a split-fp16 MFMA GEMM (three v_mfma_f32_32x32x16_f16 products per term,
//                   fp32 accuracy), 128 x 256 tile per workgroup, the W tile loaded straight into the accumulators;
//                   the part beyond the next super-block shares a launch with the next panel.  See trailing_tile.
//   Groups wider than a block are runs of whole super-blocks (width 512, 384, 256 or 128, whichever divides the
//   group; one group per row: 512): their scale and zero-point are fixed by group_params_kernel when the sweep
//   reaches them, after the far update has brought every later column up to date.
//   The loss is the sum of e^2 (equal to tr((W-W^) Hd (W-W^)^T) because U Hd U^T = I), kept per row and
//   reduced in a fixed order.
#include "common.hpp"
#include "planner.hpp"
#include <type_traits>

#pragma clang fp contract(off)

namespace onecomp {
namespace {

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

constexpr int SB = 128;        // lazy-batch block
constexpr int SBIG = 512;      // super-block: columns beyond it are updated once per 512 columns
constexpr int ROWS = plan::PANEL_ROWS;   // rows per workgroup of the panel kernel
constexpr int SP = SB + 1;     // LDS pitch (floats) of row tiles: lane l reading column c hits bank (l + c) % 32

// ------------------------------------------------------------------------------------------
// working copy: Wf[r][p] = float(W[r][perm[p]])
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ inline float to_f32(T v);
template <>
__device__ inline float to_f32<float>(float v) { return v; }
template <>
__device__ inline float to_f32<uint16_t>(uint16_t v) { return __uint_as_float(uint32_t(v) << 16); }

// the sweep's scalars live in a 256-byte slot: the Scalars of its split products, then (offset 64) the flag that
// a residual was saturated
__device__ __host__ inline uint32_t* sat_flag(Scalars* sc) { return reinterpret_cast<uint32_t*>(sc) + 16; }

// maximum over the workgroup's four waves, in every thread
__device__ __forceinline__ float block_max(float v, float* part) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    return fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
}

// Before a sweep, in one launch: rows of U (workgroups 0 .. n_u - 1) and of W (the others).  A workgroup leaves the maximum of
// its rows in max_u or max_w, which operands_kernel reduces: no scalar has to be cleared before.  Both parts are bound by memory and
// narrow layers by the launches: with clearing, the two maxima, the scalars, the operands and the panel's fragments in
// launches of their own and the sums cleared, whole calls, us: 256 x 512 193, 1999 x 2048 798, 14336 x 4096 2937; now 174, 761, 2782.
constexpr int PREP_WGS = 1024;   // at most, of either part
__device__ __forceinline__ float row_ratio_max(const float* __restrict__ U, int n, int first, int step, float* part) {
    // max_k |U_jk / U_jj| = max_k |U_jk| / |U_jj| exactly: rounding a quotient is monotone in the numerator
    float mm = 0.f;
    for (int j = first; j < n; j += step) {
        const float* row = U + int64_t(j) * n;
        float m = 0.f;
        for (int k4 = ((j + 1) & ~3) + 4 * threadIdx.x; k4 < n; k4 += 1024) {
            const float4v v = *reinterpret_cast<const float4v*>(row + k4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k4 + e > j) m = fmaxf(m, fabsf(v[e]));
        }
        m = m / fabsf(row[j]);
        if (!(m < 3.0e38f)) m = 3.0e38f;   // NaN / inf from a failed factorization: keep the scalars finite
        mm = fmaxf(mm, m);
    }
    return block_max(mm, part);
}

template <typename T>
__global__ __launch_bounds__(256) void prepare_kernel(const float* __restrict__ U, int n, int n_u, float* __restrict__ max_u,
                                                     const T* __restrict__ W, int64_t d_out, const int32_t* __restrict__ perm,
                                                     float* __restrict__ rowloss, float* __restrict__ max_w,
                                                     float* __restrict__ W0p) {
    __shared__ float part[4];
    if (int(blockIdx.x) < n_u) {
        const float m = row_ratio_max(U, n, blockIdx.x, n_u, part);
        if (threadIdx.x == 0) max_u[blockIdx.x] = m;
        return;
    }
    // max |W|, and under a column order the gathered copy W0p from which the sweep reads the weights
    const int64_t d_in = n, wg = blockIdx.x - n_u, n_w = gridDim.x - n_u;
    float m = 0.f;
    for (int64_t r = wg; r < d_out; r += n_w) {
        if (threadIdx.x == 0) rowloss[r] = 0.f;
        if (perm) {
            for (int p = threadIdx.x; p < d_in; p += 256) {
                const float v = to_f32<T>(W[r * d_in + perm[p]]);
                W0p[r * d_in + p] = v;
                m = fmaxf(m, fabsf(v));
            }
        } else {   // rows are 16-byte aligned: d_in is a multiple of 128
            constexpr int V = 16 / sizeof(T);
            for (int p = threadIdx.x * V; p < d_in; p += 256 * V) {
                const uint4v raw = *reinterpret_cast<const uint4v*>(W + r * d_in + p);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (sizeof(T) == 2) {
                        m = fmaxf(m, fabsf(__uint_as_float(raw[e] << 16)));
                        m = fmaxf(m, fabsf(__uint_as_float(raw[e] & 0xFFFF0000u)));
                    } else {
                        m = fmaxf(m, fabsf(__uint_as_float(raw[e])));
                    }
                }
            }
        }
    }
    m = block_max(m, part);
    if (threadIdx.x == 0) max_w[wg] = m;
}

constexpr int IB = 32;          // columns swept in registers at a time

// ------------------------------------------------------------------------------------------
// panel kernel: one launch sweeps a whole super-block of up to four
// 128-column blocks for 64 rows per workgroup.  Rows never interact, so the workgroup carries its rows through
// the blocks without any grid-wide step in between:
//   near update   (left-looking) before block b is swept, its columns receive the feedback of blocks 0 .. b-1 of
//                 the super-block: W_b += D_b' Un[b', b] as split-fp16 MFMAs (see the trailing kernel) whose
//                 operands are loaded from global memory already in MFMA fragment order, 16 bytes per lane:
//                 the residual fragments were written by this workgroup after block b', the fragments of the
//                 normalized U blocks by operands_kernel.  Wave w owns the block's column tile w (64 x 32).
//   sequential    four lanes per row (a quad), each holding 8 of the 32 columns of the inner block; the current
//                 column is broadcast inside the quad by DPP, the grid arithmetic is replicated, the feedback is
//                 8 FMAs per lane.  All four waves work (16 rows each).  127 cycles a column: one wave per SIMD issues
//                 21 fp64 operations and the four waves read 16 KB of U from LDS, each as long.
//   inner update  the inner block's 32 errors reach the remaining columns of the block through fp32 MFMAs
//                 (v_mfma_f32_16x16x4_f32) on the tile in LDS.
// A block took 57 thousand cycles with the errors, codes and residuals of every column written as the columns went by, eight
// conversions per lane and column, barriers around the inner updates and the residuals split twice behind the block; now 41.
// ------------------------------------------------------------------------------------------
struct PanelArgs {
    const float* Wf;            // [d_out x d_in] accumulated feedback c of the earlier super-blocks (block form: the
                                // sums c_k = sum_i (w_i - w^_i) R_ik / R_kk); of the first one (s0 == 0) not read
    const void* W0;             // the layer's weights in sweep order (the caller's matrix, or the gathered fp32 copy
                                // under a column order)
    int w0_bf16;
    const double* s64;          // [d_out] wide groups: the current group's scale in fp64 (group_params_kernel)
    uint32_t* sat;              // set to 1 if a residual had to be saturated when it was split into fp16 halves
    const float* U;
    uint8_t* Q;                 // sweep order (the caller's array, or the staging copy under a column order)
    float* scales;
    float* zeros;
    float* W_hat;               // sweep order, or nullptr
    uint16_t *Dh, *Dl;          // [SBIG x ldD] transposed residual panels for the far update
    uint16_t *Fh, *Fl;          // [workgroup][3][8 k-steps][2 row tiles][64 lanes][8] residual fragments (own use)
    const uint16_t *Bh, *Bl;    // [6 block pairs][8 k-steps][4 column tiles][64 lanes][8] of this super-block
    const Scalars* sc;
    float* rowloss;
    int d_out, d_in, s0, nb, lgG, n_g, ldD;
    int wide_g;             // >= 0: the whole super-block lies in group wide_g, whose scale and zero-point are already
                            // in scales / zeros (groups of whole super-blocks, or one group per row); lgG is then 7
    float qmax;             // highest code of the grid
    float qs;               // 0: min-max grid of Eq. (2); > 0: symmetric grid of Eq. (3) with zero-point qs
    int mse;                // scale search: the group's range is shrunk by 1 - i / 100, i < 80; least squared error wins
};

// Scale and zero-point of a group from the smallest and largest of its current values, in fp64, operation by
// operation as the definition reads: Eq. (2), or Eq. (3) when qs > 0 (symmetric grid, zero-point qs); cand > 0: from
// the range shrunk by 1 - cand / 100 (scale search).
__device__ __forceinline__ void grid_params(double mn, double mx, const int cand, const double qmax, const double qs,
                                            double& s, double& z) {
    if (cand > 0) {
        const double p = 1.0 - double(cand) * 0.01;
        mn *= p; mx *= p;
    }
    if (qs > 0.0) {
        s = fmax(fabs(mn), fabs(mx)) / qs;
        if (s == 0.0) s = 1.0;
        z = qs;
    } else {
        s = (mx - mn) / qmax;
        if (s == 0.0) s = 1.0;
        z = fmin(fmax(rint(-mn / s), 0.0), qmax);
    }
}

// Scale search of one group ("mse" option of Sec. 4.3).  partial(z, 1 / s) returns the sum of ((w - w^) / s)^2 over
// this lane's values of the group on the grid (s, z) (mse_term per value); reduce(x) sums x over the lanes that share
// the group.  Candidate i takes (s, z) by the grid's rule from the range shrunk by p_i = 1 - i / 100 (grid_params,
// fp64: a zero-point at an exact rounding tie, e.g. a group with min = -max, then falls the same way for every
// candidate and for the final parameters); the errors are summed and compared in fp32; the first smallest error
// wins, candidate 0 is the plain rule.  All lanes of the group return the same index.
constexpr int MSE_CANDIDATES = 80;
// one value's squared error in units of the scale: t = v / s + z, ((t - clamp(rne(t), 0, qmax)))^2; the caller
// multiplies the sum by s^2.  (rne(v / s) + z and rne(v / s + z) agree except at exact ties, where both choices give
// the same error.)
__device__ __forceinline__ float mse_term(float v, float zi, float rsi, float qmax) {
    const float t = fmaf(v, rsi, zi);
    const float d = t - __builtin_amdgcn_fmed3f(rintf(t), 0.f, qmax);
    return d * d;
}
template <typename P, typename R>
__device__ __forceinline__ int mse_search(const double mn, const double mx, const double qmax, const double qs,
                                          P&& partial, R&& reduce) {
    float best = 3.0e38f;
    int ibest = 0;
#pragma unroll 1
    for (int i = 0; i < MSE_CANDIDATES; ++i) {
        double sd, zd;
        grid_params(mn, mx, i, qmax, qs, sd, zd);
        const float si = float(sd);
        const float err = si * si * reduce(partial(float(zd), 1.0f / si));
        if (err < best) { best = err; ibest = i; }
    }
    return ibest;
}

// LDS of a panel workgroup.  Inverse form: 79 KB, so that a tile of the far update or a second panel workgroup fits on the CU
// beside it (matrix pipes under one, vector units under the other).  Block form: 95 KB, so a workgroup, of far tiles too,
// has its CU to itself.
//   sU    the block's U off its 32 x 32 diagonal sub-blocks: six sub-blocks, row by row
//   sUd   the diagonal sub-blocks in fp64, rows divided by their diagonal entries, zeros on and below the diagonal: rows
//         8 g .. 8 g + 7 hold the slices (8 columns) g .. 3, and behind them zeros for the lanes of finished slices
//   sRd   reciprocals of the diagonal
//   sC    the row tile, see panel_body
//   sUg   (block form) the diagonal sub-blocks in fp32
constexpr int UB = IB * IB, UD_SLICES = 8 * (4 + 3 + 2 + 1), UD_ZERO = 3 * 8 * 8;   // doubles: slices of a sub-block, zeros
__host__ __device__ constexpr int u_off(int I, int J) { return (3 * I - I * (I - 1) / 2 + J - I - 1) * UB; }
__host__ __device__ constexpr int ud_first(int g) { return 8 * (4 * g - g * (g - 1) / 2) * 8; }   // slice (8 g, g)
constexpr int LDS_UD = 6 * UB * 4, LDS_RD = LDS_UD + (4 * UD_SLICES * 8 + UD_ZERO) * 8, LDS_C = LDS_RD + SB * 8;
constexpr int LDS_UG = LDS_C + ROWS * SP * 4;
constexpr int panel_lds(bool direct) { return LDS_UG + (direct ? 4 * UB * 4 : 0); }
static_assert(panel_lds(false) <= 80 * 1024, "a second workgroup fits beside a panel's");
static_assert(panel_lds(true) <= 160 * 1024, "a CU's LDS");

template <int CTRL>
__device__ __forceinline__ float dpp_quad(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_quad(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u)), CTRL, 0xF, 0xF, true));
    const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), CTRL, 0xF, 0xF, true));
    return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}
// what this wave has written to LDS is visible to all its lanes (LDS operations of a wave are executed in order; this keeps
// the compiler from moving them past each other)
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
constexpr int quad_bcast(int o) { return o | (o << 2) | (o << 4) | (o << 6); }
constexpr int QUAD_SWAP1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);   // lanes 0<->1, 2<->3
constexpr int QUAD_SWAP2 = 2 | (3 << 2) | (0 << 4) | (1 << 6);   // lanes 0<->2, 1<->3

// What a block of 128 columns starts from.  The feedback of all earlier columns is kept apart from the weights:
//   sC   (LDS, fp32)  c = -sum_i e_i U_i,col over the finished columns i: the part from earlier super-blocks comes
//                     from the working copy (a.Wf), the part from the earlier blocks of this super-block from the
//                     near update (split-fp16 MFMAs accumulated from zero), the part from the earlier inner blocks
//                     of this block from fp32 MFMAs accumulated from zero; each part is added once in fp32.  A finished
//                     column holds its error e until the inner update has taken it, then its residual as an fp16 pair;
//   w0v  (registers)  the ORIGINAL weights of this lane's 4 x 8 columns (exact: the input is bf16 or fp32).
// The value that is quantized is w0 + c formed in fp64.
//
// From the sequential part to the end of a block a wave touches its own 16 rows only, and no barrier stands between.
//
// DIRECT (block form of the factor): a.U holds U only on its 128 x 128 diagonal blocks and -U_jj R_jk / R_kk
// elsewhere (R = U^-1).  The working copy then accumulates c_k = sum_i (w_i - w^_i) R_ik / R_kk over the finished
// columns i of earlier blocks, where w are the ORIGINAL weights; a block starts from
//   w_b + c Un_bb ,   Un_bb = rows of U_bb divided by their diagonal entries,
// which is the state the sweep with the full U has on entering the block (e = (w - w^) R and
// U_AB = -U_AA R_AB U_BB for finished columns A, remaining columns B).  Inside the block nothing changes; what the
// block passes on is w - w^ measured from the original weights instead of the compensated ones.
template <int GB, bool DIRECT>  // GB: group width seen inside an inner block: 16 (G == 16) or 32 (G = 32, 64, 128)
__device__ __forceinline__ void panel_body(const PanelArgs& a, const int wg, char* psm) {
    float* const sU = reinterpret_cast<float*>(psm);
    double* const sUd = reinterpret_cast<double*>(psm + LDS_UD);
    double* const sRd = reinterpret_cast<double*>(psm + LDS_RD);
    float* const sC = reinterpret_cast<float*>(psm + LDS_C);
    // the diagonal sub-blocks as they come in; the inverse form is done with them before sC is written
    constexpr int LDS_DIAG = DIRECT ? LDS_UG : LDS_C;
    const float* const sUg = reinterpret_cast<const float*>(psm + LDS_DIAG);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = wg * ROWS;
    const int64_t d_in = a.d_in;
    const int G = 1 << a.lgG;
    // sequential part: quad = row, lane in quad = slice of 8 columns
    const int qrow = tid >> 2, sl = tid & 3;
    const int grow = min(r0 + qrow, a.d_out - 1);
    const bool row_ok = (r0 + qrow) < a.d_out;
    // MFMA accumulator layout: register r of lane l = row (r/4)*8 + (l/32)*4 + r%4, column l%32
    const int lr = (lane >> 5) * 4, lc = lane & 31;
    const double qmax = double(a.qmax), qsd = double(a.qs);
    const float f_d = a.sc->f_d, f_inv = a.sc->f_inv;
    const uint32_t lds0 = uint32_t(uintptr_t((ONECOMP_LDS char*)psm));
    double s = 1.0, rs = 1.0, z = 0.0;
    double lossacc = 0.0;   // of this lane's columns
    bool saturated = false;
    if (a.wide_g >= 0) {
        s = a.s64[grow];
        z = double(a.zeros[int64_t(grow) * a.n_g + a.wide_g]);
        rs = 1.0 / s;
    }
    if (tid < UD_ZERO) sUd[4 * UD_SLICES * 8 + tid] = 0.0;

#pragma unroll 1
    for (int b = 0; b < a.nb; ++b) {
        const int j0 = a.s0 + b * SB;
        __syncthreads();   // everybody is done with the previous block's tiles
        // opaque copies: what is computed from them is not hoisted out of the loop, to be spilled there
        int bw = wave, blane = lane;
        asm volatile("" : "+s"(bw));
        asm volatile("" : "+v"(blane));
        // ---- U's diagonal block -> LDS, eight rows of a sub-block (1 KB) per wave load, no registers involved
        {
            const float* ub = a.U + int64_t(j0) * d_in + j0;
            __amdgpu_buffer_rsrc_t rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(ub), 0, int((int64_t(SB - 1) * d_in + SB) * 4), 0x00020000);
#pragma unroll
            for (int q = 0; q < 10; ++q) {
                // four loads per sub-block; sub-blocks 0 .. 5: those off the diagonal, then (wave, wave)
                const int t = q < 6 ? 6 * bw + q : 4 * bw + q - 6, blk = t >> 2;
                const int I = q < 6 ? (blk >= 3) + (blk >= 5) : bw, J = q < 6 ? (blk < 3 ? blk + 1 : blk < 5 ? blk - 1 : 3) : bw;
                const int row = 32 * I + 8 * (t & 3) + (blane >> 3);
                lds_load16(lds0 + (q < 6 ? 0 : LDS_DIAG) + t * 1024, uint32_t((row * int(d_in) + 32 * J + (blane & 7) * 4) * 4),
                           rsrc);
            }
        }
        float w0v[32];
        // ---- feedback sums of this block's columns, wave = column tile: what earlier super-blocks left in the
        // working copy plus the near update from the earlier blocks of this super-block, accumulated from zero
        {
            float16v cf[2], acc[2];
            {
                // Whole workgroups: one lane offset and a scalar one per row (32 addresses in registers would be kept for
                // the whole sweep).  In a short one rows past d_out read the last row: see panel_feedback_offset.
                const int rows = min(ROWS, a.d_out - r0), col = j0 + 32 * bw + (blane & 31);
                const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float*>(a.Wf + int64_t(r0) * d_in), 0, a.s0 > 0 ? int(rows * d_in * 4) : 0, 0x00020000);
                auto load = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const plan::FeedbackOffset o =
                                plan::panel_feedback_offset<decltype(whole)::value>(rows, int(d_in), blane, mt, r, col);
                            cf[mt][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o.lane, o.scalar, 0));
                            acc[mt][r] = 0.f;
                        }
                };
                if (rows == ROWS) load(std::true_type{});
                else load(std::false_type{});
            }
            if (b > 0)
            {
                // rolling window of WIN k-steps of operand fragments (a source block has 8 k-steps)
                constexpr int WIN = 4;
                uint4v win[WIN][6];
                // descriptors, one lane offset and scalar offsets: no addresses in vector registers
                constexpr int F_BYTES = 3 * 8 * 2 * 64 * 16, B_BYTES = 6 * 8 * 4 * 64 * 16, DESC = 0x00020000;
                const int64_t fo0 = int64_t(wg) * (F_BYTES / 2);
                const __amdgpu_buffer_rsrc_t rfh = __builtin_amdgcn_make_buffer_rsrc(a.Fh + fo0, 0, F_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rfl = __builtin_amdgcn_make_buffer_rsrc(a.Fl + fo0, 0, F_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rbh = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.Bh), 0, B_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rbl = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.Bl), 0, B_BYTES, DESC);
                const int b0 = ((b * (b - 1) / 2) * 8 * 4 + bw) * 1024;
                auto issue = [&](int bp, int ks, uint4v(&d)[6]) __attribute__((always_inline)) {
                    const int fo = (bp * 8 + ks) * 2 * 1024, bo = b0 + (bp * 8 + ks) * 4 * 1024;
                    const int vo = blane * 16;
                    d[0] = __builtin_amdgcn_raw_buffer_load_b128(rfl, vo, fo, 0);
                    d[1] = __builtin_amdgcn_raw_buffer_load_b128(rfh, vo, fo, 0);
                    d[2] = __builtin_amdgcn_raw_buffer_load_b128(rfl, vo + 1024, fo, 0);
                    d[3] = __builtin_amdgcn_raw_buffer_load_b128(rfh, vo + 1024, fo, 0);
                    d[4] = __builtin_amdgcn_raw_buffer_load_b128(rbh, vo, bo, 0);
                    d[5] = __builtin_amdgcn_raw_buffer_load_b128(rbl, vo, bo, 0);
                };
#pragma unroll
                for (int ks = 0; ks < WIN; ++ks) issue(0, ks, win[ks]);
#pragma unroll 1
                for (int bp = 0; bp < b; ++bp) {
                    const bool more = bp + 1 < b;
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        uint4v(&cur)[6] = win[ks % WIN];
                        const half8v al0 = __builtin_bit_cast(half8v, cur[0]), ah0 = __builtin_bit_cast(half8v, cur[1]);
                        const half8v al1 = __builtin_bit_cast(half8v, cur[2]), ah1 = __builtin_bit_cast(half8v, cur[3]);
                        const half8v bhv = __builtin_bit_cast(half8v, cur[4]), blv = __builtin_bit_cast(half8v, cur[5]);
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al0, bhv, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al1, bhv, acc[1], 0, 0, 0);
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah0, blv, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah1, blv, acc[1], 0, 0, 0);
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah0, bhv, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah1, bhv, acc[1], 0, 0, 0);
                        // refill the slot just consumed: k-step ks + WIN of this source block or of the next
                        if (ks + WIN < 8) issue(bp, ks + WIN, cur);
                        else if (more) issue(bp + 1, ks + WIN - 8, cur);
                    }
                }
            }
            // c = (near update) / (f_d f_u) + (earlier super-blocks): one fp32 rounding
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mt][r] = __builtin_fmaf(acc[mt][r], f_inv, cf[mt][r]);
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));   // the direct loads have landed
            __syncthreads();
            // the original weights of this lane's row: columns 32 q + 8 sl + i of the block in w0v[8 q + i]
            // (requested here, so that they arrive behind the conversions and take no registers in the near update)
            if (a.w0_bf16) {
                const uint16_t* wp = static_cast<const uint16_t*>(a.W0) + int64_t(grow) * d_in + j0 + 8 * sl;
                uint4v raw[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) raw[q] = *reinterpret_cast<const uint4v*>(wp + 32 * q);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        w0v[8 * q + 2 * i] = __uint_as_float(raw[q][i] << 16);
                        w0v[8 * q + 2 * i + 1] = __uint_as_float(raw[q][i] & 0xFFFF0000u);
                    }
            } else {
                const float* wp = static_cast<const float*>(a.W0) + int64_t(grow) * d_in + j0 + 8 * sl;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float4v v = *reinterpret_cast<const float4v*>(wp + 32 * q + 4 * h);
#pragma unroll
                        for (int i = 0; i < 4; ++i) w0v[8 * q + 4 * h + i] = v[i];
                    }
            }
            // sub-block (wave, wave) for the sequential part, four columns at a time (converting there: eight operations per
            // lane and column)
            {
                const float* ug = sUg + wave * UB;
                if (lane < IB) sRd[32 * wave + lane] = 1.0 / double(ug[lane * (IB + 1)]);
                wave_fence();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int id = q * 64 + lane, j = id >> 3, g = j >> 3, k0 = (id & 7) * 4;
                    const float4v v = *reinterpret_cast<const float4v*>(ug + 4 * id);
                    const double rd = sRd[32 * wave + j];
                    double2 lo, hi;
                    lo.x = k0 > j ? double(v[0]) * rd : 0.0;
                    lo.y = k0 + 1 > j ? double(v[1]) * rd : 0.0;
                    hi.x = k0 + 2 > j ? double(v[2]) * rd : 0.0;
                    hi.y = k0 + 3 > j ? double(v[3]) * rd : 0.0;
                    if ((k0 >> 3) >= g) {
                        double2* const dst = reinterpret_cast<double2*>(
                            sUd + wave * UD_SLICES * 8 + (4 * g - g * (g - 1) / 2) * 64 + (j & 7) * (4 - g) * 8 + k0 - 8 * g);
                        dst[0] = lo;
                        dst[1] = hi;
                    }
                }
            }
            __syncthreads();
            if constexpr (!DIRECT) {
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sC[(mt * 32 + (r / 4) * 8 + (blane >> 5) * 4 + (r % 4)) * SP + 32 * bw + (blane & 31)] = acc[mt][r];
            } else {
                // eight 32 x 32 tiles of (c / diag) U_bb, accumulated from zero; column tile nt needs k < 32 (nt + 1)
                // (U_bb is upper triangular), so wave w takes (row tile 0, column tile w) and (1, 3 - w): five chunks
                // of 32 k, 16 MFMAs each.  A chunk's 32 operand values are read before its first MFMA, and the two
                // tiles' chunks alternate so that one tile's LDS reads fall behind the other's MFMAs.
                float16v c0, c1;
#pragma unroll
                for (int r = 0; r < 16; ++r) { c0[r] = 0.f; c1[r] = 0.f; }
                if (j0 > 0) {
                    const float rd = float(sRd[32 * wave + lc]);   // c_k / U_kk as the A operand
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            sC[(mt * 32 + (r / 4) * 8 + lr + (r % 4)) * SP + 32 * wave + lc] = acc[mt][r] * rd;
                    __syncthreads();
                    const int nt0 = wave, nt1 = 3 - wave;
                    const float* ap0 = sC + lc * SP + (lane >> 5);
                    const float* ap1 = sC + (32 + lc) * SP + (lane >> 5);
                    auto chunk = [&](float16v& c, const float* ap, const int nt, const int ch) __attribute__((always_inline)) {
                        const float* bp = (ch == nt ? sUg + ch * UB : sU + u_off(ch, nt)) + (lane >> 5) * IB + lc;
                        float av[16], bv[16];
#pragma unroll
                        for (int kk = 0; kk < 16; ++kk) {
                            av[kk] = ap[32 * ch + 2 * kk];
                            bv[kk] = bp[2 * kk * IB];
                        }
#pragma unroll
                        for (int kk = 0; kk < 16; ++kk) c = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk], bv[kk], c, 0, 0, 0);
                    };
#pragma unroll 1
                    for (int ch = 0; ch < 4; ++ch) {
                        if (ch <= nt0) chunk(c0, ap0, nt0, ch);
                        if (ch <= nt1) chunk(c1, ap1, nt1, ch);
                    }
                    __syncthreads();   // every wave is done reading sC as an operand
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sC[((r / 4) * 8 + lr + (r % 4)) * SP + wave * 32 + lc] = c0[r];
                    sC[(32 + (r / 4) * 8 + lr + (r % 4)) * SP + (3 - wave) * 32 + lc] = c1[r];
                }
            }
            __syncthreads();
        }

#pragma unroll 1
        for (int jb = 0; jb < SB; jb += IB) {
            double w[8];
            float* const crow = sC + qrow * SP + jb + 8 * sl;
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = double(w0v[i]) + double(crow[i]);
            double s_first = s, z_first = z;   // GB == 16: the grid of the inner block's first group
            auto fix_grid = [&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                const int col = j0 + jb + j;
                bool fresh;
                double mn, mx;
                // this lane's values of the group: eight per inner block that the group spans
                auto value = [&](int k) __attribute__((always_inline)) {
                    return double(w0v[k]) + double(crow[(k >> 3) * IB + (k & 7)]);
                };
                if constexpr (GB == 16) {
                    // group = the 16 columns held by lanes 2 (j / 16) and 2 (j / 16) + 1 of the quad
                    fresh = true;
                    mn = w[0]; mx = w[0];
#pragma unroll
                    for (int i = 1; i < 8; ++i) { mn = fmin(mn, w[i]); mx = fmax(mx, w[i]); }
                    mn = fmin(mn, dpp_quad<QUAD_SWAP1>(mn));
                    mx = fmax(mx, dpp_quad<QUAD_SWAP1>(mx));
                    mn = dpp_quad<quad_bcast(j / 8)>(mn);
                    mx = dpp_quad<quad_bcast(j / 8)>(mx);
                } else {
                    fresh = a.wide_g < 0 && (col & (G - 1)) == 0;
                    if (fresh) {   // uniform: the group's G <= 128 columns are unfinished
                        mn = w[0]; mx = w[0];
#pragma unroll
                        for (int i = 1; i < 8; ++i) { mn = fmin(mn, w[i]); mx = fmax(mx, w[i]); }
#pragma unroll
                        for (int k = 8; k < 32; ++k) {
                            if (k % 8 == 0 && 4 * k >= G) break;
                            const double v = value(k);
                            mn = fmin(mn, v); mx = fmax(mx, v);
                        }
                        mn = fmin(mn, dpp_quad<QUAD_SWAP1>(mn));
                        mx = fmax(mx, dpp_quad<QUAD_SWAP1>(mx));
                        mn = fmin(mn, dpp_quad<QUAD_SWAP2>(mn));
                        mx = fmax(mx, dpp_quad<QUAD_SWAP2>(mx));
                    }
                }
                if (!fresh) return;
                int cand = 0;
                if constexpr (GB != 16) {
                    if (a.mse) {   // uniform; this lane's quarter of the group, held in registers
                        float gv[32];
#pragma unroll
                        for (int k = 0; k < 32; ++k) gv[k] = k < 8 ? float(w[k & 7]) : 4 * (k & 24) < G ? float(value(k)) : 0.f;
                        const int n8 = G >> 5;   // batches of 8 values: 1, 2 or 4
                        const float qmf = a.qmax;
                        cand = mse_search(mn, mx, qmax, qsd,
                                   [&](float zi, float rsi) __attribute__((always_inline)) {
                                       float e0 = 0.f, e1 = 0.f;
#pragma unroll
                                       for (int k = 0; k < 8; k += 2) {
                                           e0 += mse_term(gv[k], zi, rsi, qmf);
                                           e1 += mse_term(gv[k + 1], zi, rsi, qmf);
                                       }
                                       if (n8 > 1) {
#pragma unroll
                                           for (int k = 8; k < 16; k += 2) {
                                               e0 += mse_term(gv[k], zi, rsi, qmf);
                                               e1 += mse_term(gv[k + 1], zi, rsi, qmf);
                                           }
                                       }
                                       if (n8 > 2) {
#pragma unroll
                                           for (int k = 16; k < 32; k += 2) {
                                               e0 += mse_term(gv[k], zi, rsi, qmf);
                                               e1 += mse_term(gv[k + 1], zi, rsi, qmf);
                                           }
                                       }
                                       return e0 + e1;
                                   },
                                   [&](float x) __attribute__((always_inline)) {
                                       x += dpp_quad<QUAD_SWAP1>(x);
                                       return x + dpp_quad<QUAD_SWAP2>(x);
                                   });
                    }
                } else {
                    if (a.mse) {   // uniform; the group's 16 values sit in two lanes of the quad
                        float gv[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k) gv[k] = float(w[k]);
                        const float qmf = a.qmax;
                        cand = mse_search(mn, mx, qmax, qsd,
                                   [&](float zi, float rsi) __attribute__((always_inline)) {
                                       float e0 = 0.f, e1 = 0.f;
#pragma unroll
                                       for (int k = 0; k < 8; k += 2) {
                                           e0 += mse_term(gv[k], zi, rsi, qmf);
                                           e1 += mse_term(gv[k + 1], zi, rsi, qmf);
                                       }
                                       return e0 + e1;
                                   },
                                   [&](float x) __attribute__((always_inline)) {
                                       x += dpp_quad<QUAD_SWAP1>(x);
                                       return dpp_quad<quad_bcast(j / 8)>(x);
                                   });
                    }
                }
                grid_params(mn, mx, cand, qmax, qsd, s, z);
                rs = 1.0 / s;
                if constexpr (GB == 16 && j == 0) { s_first = s; z_first = z; }
                if (sl == 0 && row_ok) {
                    a.scales[int64_t(grow) * a.n_g + (col >> a.lgG)] = float(s);
                    a.zeros[int64_t(grow) * a.n_g + (col >> a.lgG)] = float(z);
                }
            };
            // (w - s (q - z), q - z) of a value on the current grid.  w / s correctly rounded, as the definition's division
            // gives it (an exact tie, possible in a row's first group where weights and scale are short binary numbers,
            // then falls the same way): t0 = w * fl(1 / s), residual by FMA, one correction step; no division, no branch.
            // q - z = clamp(rint(t) + z, 0, qmax) - z = clamp(rint(t), -z, qmax - z): whole numbers, nothing is rounded.
            auto quantize = [&](double v, double sq, double rsq, double zq, double& d) __attribute__((always_inline)) {
                const double t0 = v * rsq;
                const double t = __builtin_fma(__builtin_fma(-t0, sq, v), rsq, t0);
                d = fmin(fmax(rint(t), -zq), qmax - zq);
                return __builtin_fma(-sq, d, v);
            };
            auto pin = [](double& v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); };   // here, in this order
            // The sequential part.  Row j of the inner block's U triangle (this lane's 8 columns, divided by U_jj) is read two
            // steps ahead; it is zero up to column j, so a finished register keeps the value that was quantized (but see below).
            // One wave per SIMD has nothing else to cover the chain of a step (broadcast, nine dependent fp64 operations,
            // the update of the next column's register), so the other seven updates of the step before are issued between its
            // operations, in this order: left alone, the compiler puts them in a block behind the chain (169 cycles a
            // column), or each at its register's next use.
            const double* const ud = sUd + (jb >> 5) * UD_SLICES * 8;
            {
                double2 u[3][4];
                auto read_row = [&](auto jc, double2(&dst)[4]) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value, g = j / 8;
                    const double* p = (g == 0 || sl >= g ? ud + ud_first(g) + (sl - g) * 8 : sUd + 4 * UD_SLICES * 8) + (j % 8) * (4 - g) * 8;
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[i] = *reinterpret_cast<const double2*>(p + 2 * i);
                };
                read_row(std::integral_constant<int, 0>{}, u[0]);
                read_row(std::integral_constant<int, 1>{}, u[1]);
                double res = 0.0;   // of the step before
                static_for<0, IB>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    // update k of the step before: column j + k (mod 8); the first one, k = 0, has been made
                    auto late = [&](auto kc) __attribute__((always_inline)) {
                        constexpr int k = decltype(kc)::value, i = (j + k) % 8, pj = j - 1;
                        if constexpr (j > 0 && (pj < 24 || i > pj % 8)) {
                            const double2& up = u[(j + 2) % 3][i / 2];
                            w[i] = __builtin_fma(-res, i % 2 ? up.y : up.x, w[i]);
                            pin(w[i]);
                        }
                    };
                    constexpr bool fix = j % GB == 0;   // the group's grid needs all values up to date
                    if constexpr (fix) {
                        static_for<1, 8>(late);
                        fix_grid(jc);
                    }
                    auto between = [&](auto kc) __attribute__((always_inline)) {
                        if constexpr (!fix) late(kc);
                    };
                    double wj = dpp_quad<quad_bcast(j / 8)>(w[j % 8]);
                    pin(wj);
                    between(std::integral_constant<int, 1>{});
                    double t0 = wj * rs;
                    pin(t0);
                    between(std::integral_constant<int, 2>{});
                    double r1 = __builtin_fma(-t0, s, wj);
                    pin(r1);
                    between(std::integral_constant<int, 3>{});
                    double t = __builtin_fma(r1, rs, t0);
                    pin(t);
                    between(std::integral_constant<int, 4>{});
                    between(std::integral_constant<int, 5>{});
                    t = fmin(fmax(rint(t), -z), qmax - z);   // pinned, the compiler would quiet NaNs before each of these
                    between(std::integral_constant<int, 6>{});
                    between(std::integral_constant<int, 7>{});
                    if constexpr (j + 2 < IB) read_row(std::integral_constant<int, j + 2>{}, u[(j + 2) % 3]);
                    res = __builtin_fma(-s, t, wj);
                    pin(res);
                    if constexpr (j + 1 < IB) {
                        constexpr int i = (j + 1) % 8;
                        const double2& un = u[j % 3][i / 2];
                        w[i] = __builtin_fma(-res, i % 2 ? un.y : un.x, w[i]);
                        pin(w[i]);
                    }
                });
            }
            // What the inner block leaves, from the values that were quantized: this lane's eight columns.  The errors go to
            // sC's finished columns for the inner update, codes, W^ = s (q - z) and the residual fragments to memory.
            // The residual is w - w^ (block form: against the original weights), negated, scaled by a power of two and split
            // into fp16 hi + lo (hi = rne(x), lo = rne(x - hi): 22 significant bits); saturated far above anything a
            // sweep of a sane layer produces, and the saturation is reported (the loss then comes back as +infinity).
            uint32_t pair[8];   // the residuals, hi in the lower half
            {
                const bool first = GB == 16 && sl < 2;
                const double sq = first ? s_first : s, zq = first ? z_first : z;
                const double rsq = GB == 16 ? 1.0 / sq : rs;
                float err[8];
                uint32_t codes[2];
                double loss;
                bool big;
                auto settle = [&]() __attribute__((always_inline)) {
                    codes[0] = codes[1] = 0;
                    loss = lossacc;
                    big = false;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        double d;
                        const double r = quantize(w[i], sq, rsq, zq, d);
                        const double e = r * sRd[jb + 8 * sl + i];
                        loss = __builtin_fma(e, e, loss);
                        err[i] = float(e);
                        codes[i / 4] |= uint32_t(int(d + zq)) << (8 * (i % 4));
                        float x = -float(DIRECT ? __builtin_fma(-sq, d, double(w0v[i])) : r) * f_d;
                        big |= !(fabsf(x) <= 60000.f);
                        x = fminf(fmaxf(x, -60000.f), 60000.f);
                        const _Float16 h = (_Float16)x;
                        const _Float16 l = (_Float16)(x - (float)h);
                        pair[i] = uint32_t(__builtin_bit_cast(uint16_t, h)) | (uint32_t(__builtin_bit_cast(uint16_t, l)) << 16);
                    }
                };
                settle();
                // A residual that is not finite (an infinite weight or a NaN) times U's zero has also reached the columns in
                // front of it, whose codes are decided: the wave then takes its rows through the inner block again, column by
                // column from where they began, and spares finished columns.
                if (__builtin_expect(__any(!(loss < __builtin_inf())), 0)) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) w[i] = double(w0v[i]) + double(crow[i]);
#pragma unroll 1
                    for (int j = 0; j < IB; ++j) {   // w turns: column j is in w[0] of slice g
                        const int g = j >> 3, jr = j & 7;
                        const double sg = GB == 16 && g < 2 ? s_first : s, zg = GB == 16 && g < 2 ? z_first : z;
                        const double rsg = GB == 16 ? 1.0 / sg : rs;
                        double d;
                        const double r = quantize(__shfl(w[0], (lane & ~3) + g, 64), sg, rsg, zg, d);
                        const double* const p = ud + ud_first(g) + (sl - g) * 8 + jr * (4 - g) * 8;
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (sl > g || (sl == g && i > 0 && jr + i < 8)) w[i] = __builtin_fma(-r, p[(jr + i) & 7], w[i]);
                        const double w0 = w[0];
#pragma unroll
                        for (int i = 0; i < 7; ++i) w[i] = w[i + 1];
                        w[7] = w0;
                    }
                    settle();
                }
                lossacc = loss;
                saturated |= row_ok && big;
#pragma unroll
                for (int i = 0; i < 8; ++i) crow[i] = err[i];
                if (row_ok) {
                    uint32_t* const qp = reinterpret_cast<uint32_t*>(a.Q + int64_t(grow) * d_in + j0 + jb + 8 * sl);
                    qp[0] = codes[0];
                    qp[1] = codes[1];
                    if (a.W_hat) {
                        float* const hp = a.W_hat + int64_t(grow) * d_in + j0 + jb + 8 * sl;
                        const float sf = float(sq), zf = float(zq);
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            float4v hat;
#pragma unroll
                            for (int e = 0; e < 4; ++e) hat[e] = sf * (float((codes[h] >> (8 * e)) & 255u) - zf);
                            *reinterpret_cast<float4v*>(hp + 4 * h) = hat;
                        }
                    }
                }
                short8v fh, fl;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    fh[i] = short(uint16_t(pair[i]));
                    fl[i] = short(uint16_t(pair[i] >> 16));
                }
                // MFMA A-operand fragments for this workgroup's own near updates: lane L of k-step ks, row tile mt holds
                // row mt*32 + L%32, columns ks*16 + 8 (L/32) + 0..7; rows past d_out hold copies of the last row
                if (b + 1 < a.nb) {
                    const int ks = (jb >> 4) + (sl >> 1), it = (ks * 2 + (qrow >> 5)) * 64 + (qrow & 31) + 32 * (sl & 1);
                    const int64_t off = ((int64_t(wg) * 3 + b) * (8 * 2 * 64) + it) * 8;
                    *reinterpret_cast<short8v*>(a.Fh + off) = fh;
                    *reinterpret_cast<short8v*>(a.Fl + off) = fl;
                }
            }
            // Remaining columns of the block: c_col -= sum_i e_i U[jb+i][col], accumulated from zero and then added to the
            // tile in LDS.  A wave updates the 16 rows it sweeps, so the waves run through the block without a barrier, and
            // 16 x 16 tiles share its rows evenly: 6, 4 and 2 tiles of 32 x 32 on four waves behind barriers took 8.3
            // thousand cycles a block.
            if (jb + IB < SB) {
                wave_fence();   // the other lanes' errors
                const int l16 = lane & 15, lk = lane >> 4, I = jb >> 5;
                float av[8];
#pragma unroll
                for (int kk = 0; kk < 8; ++kk) av[kk] = -sC[(16 * wave + l16) * SP + jb + 4 * kk + lk];
                // a pair of tiles takes the even and the odd columns of 32: one LDS access brings both tiles' values, without
                // bank conflicts; the operands and the old values of a pair are read a pair ahead
                const float* const bp = sU + u_off(I, I + 1) + lk * IB + 2 * l16;
                float* const cp = sC + (16 * wave + 4 * lk) * SP + jb + IB + 2 * l16;
                float2 bv[2][8], old[2][4];
                auto load = [&](int J, float2(&bd)[8], float2(&od)[4]) __attribute__((always_inline)) {
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) bd[kk] = *reinterpret_cast<const float2*>(bp + J * UB + 4 * kk * IB);
#pragma unroll
                    for (int r = 0; r < 4; ++r) od[r] = make_float2(cp[J * IB + r * SP], cp[J * IB + r * SP + 1]);
                };
                auto update = [&](int J, const float2(&bd)[8], const float2(&od)[4]) __attribute__((always_inline)) {
                    float4v c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kk], bd[kk].x, c0, 0, 0, 0);
                        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kk], bd[kk].y, c1, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        cp[J * IB + r * SP] = od[r].x + c0[r];
                        cp[J * IB + r * SP + 1] = od[r].y + c1[r];
                    }
                };
                const int n_J = 3 - I;
                load(0, bv[0], old[0]);
                if (n_J > 1) load(1, bv[1], old[1]);
                update(0, bv[0], old[0]);
                if (n_J > 2) load(2, bv[0], old[0]);
                if (n_J > 1) update(1, bv[1], old[1]);
                if (n_J > 2) update(2, bv[0], old[0]);
                wave_fence();
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) crow[i] = __uint_as_float(pair[i]);
#pragma unroll
            for (int i = 0; i < 24; ++i) w0v[i] = w0v[i + 8];   // the next inner block's first
        }

        // ---- block done: the residuals again, transposed (k-major) for the far update, 8 rows x 4 columns per lane
        wave_fence();
        {
            const int r8 = 16 * wave + 8 * (lane & 1), c4 = 4 * (lane >> 1);
            uint32_t v[4][8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c][e] = __float_as_uint(sC[(r8 + e) * SP + c4 + c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t off = int64_t(b * SB + c4 + c) * a.ldD + r0 + r8;
                uint4v dh, dl;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    dh[e] = __builtin_amdgcn_perm(v[c][2 * e + 1], v[c][2 * e], 0x05040100u);
                    dl[e] = __builtin_amdgcn_perm(v[c][2 * e + 1], v[c][2 * e], 0x07060302u);
                }
                *reinterpret_cast<uint4v*>(a.Dh + off) = dh;
                *reinterpret_cast<uint4v*>(a.Dl + off) = dl;
            }
        }
        // the fragments written above are read back by other waves of this workgroup (same CU, same L1): a
        // workgroup-scope release, completed by the barrier at the top of the loop
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }
    lossacc += dpp_quad<QUAD_SWAP1>(lossacc);
    lossacc += dpp_quad<QUAD_SWAP2>(lossacc);
    if (sl == 0 && row_ok) a.rowloss[grow] += float(lossacc);
    if (saturated) *a.sat = 1u;
}

// ------------------------------------------------------------------------------------------
// The panel with 16 rows per workgroup and 16 lanes per row, two of an inner block's 32 columns each, for layers whose
// workgroups of 64 rows would leave most CUs idle.  The steps of a row, and what reaches an entry of it in which order, are
// panel_body's, so the results are bit-equal; what a wave does besides the chain of steps (codes, errors, residuals, grids,
// feedback sums) is a quarter: a block of 128 columns takes 13 us instead of 20.
//   near update   one 32-row tile whose rows 16 .. 31 repeat rows 0 .. 15 (its results are not taken)
//   sequential    the current column reaches the row's lanes as one DPP move (row_newbcast) of 64 bits
//   inner update  all 16 rows in one tile, the waves take 32 columns each, between two barriers
// LDS: sU, sRd, sC as there; sUd the diagonal sub-blocks in fp64, zeros up to the diagonal, rows 0 .. 15 whole, of rows 16 ..
// 31 the last 16 columns, and zeros for the lanes of the other ones.  The diagonal sub-blocks come in where sC will be (inverse
// form), or behind it (block form).  Two workgroups fit on a CU in either.
// No scale search (its sums would be added in another order): groups whose search runs in the panel take panel_body.
// ------------------------------------------------------------------------------------------
constexpr int ROWS16 = 16, F16_BYTES = 3 * 8 * 2 * ROWS16 * 8 * 2;   // .. of residual fragments, hi or lo, per workgroup
constexpr int UD16 = 16 * IB + 16 * 16, UD16_ZERO = 16 * 16;   // doubles of a diagonal sub-block, and of the zeros behind the four
constexpr int L16_RD = LDS_UD + (4 * UD16 + UD16_ZERO) * 8, L16_C = L16_RD + SB * 8, L16_C_BYTES = ROWS16 * SP * 4;
constexpr int panel16_lds(bool direct) { return L16_C + (direct ? L16_C_BYTES + 4 * UB * 4 : 4 * UB * 4); }
static_assert(L16_C_BYTES <= 4 * UB * 4 && L16_C_BYTES % 16 == 0, "the diagonal sub-blocks as they come in cover sC");
static_assert(panel16_lds(true) <= 80 * 1024, "a second workgroup fits beside a panel's");

// value of lane J of every 16 lanes, in all of them.  A DPP operand must not come from the two instructions before, which the
// compiler does not see into the statement: it keeps that distance itself.
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
    double o;
    asm volatile("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(o) : "v"(v), "n"(J));
    return o;
}
constexpr int ROW_ROR = 0x120, ROW_HALF_MIRROR = 0x141;   // DPP: rotation in 16 lanes (+ distance), mirror in 8

template <int GB, bool DIRECT>
__device__ __forceinline__ void panel_body16(const PanelArgs& a, const int wg, char* psm) {
    float* const sU = reinterpret_cast<float*>(psm);
    double* const sUd = reinterpret_cast<double*>(psm + LDS_UD);
    double* const sRd = reinterpret_cast<double*>(psm + L16_RD);
    float* const sC = reinterpret_cast<float*>(psm + L16_C);
    constexpr int LDS_DIAG = DIRECT ? L16_C + L16_C_BYTES : L16_C;
    const float* const sUg = reinterpret_cast<const float*>(psm + LDS_DIAG);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r0 = wg * ROWS16;
    const int64_t d_in = a.d_in;
    const int G = 1 << a.lgG;
    const int srow = tid >> 4, sl = tid & 15;   // sequential part: row, slice of two columns
    const int grow = min(r0 + srow, a.d_out - 1);
    const bool row_ok = (r0 + srow) < a.d_out;
    const int lr = (lane >> 5) * 4, lc = lane & 31;   // 32 x 32 accumulators: register r = row (r/4)*8 + lr + r%4, column lc
    const double qmax = double(a.qmax), qsd = double(a.qs);
    const float f_d = a.sc->f_d, f_inv = a.sc->f_inv;
    const uint32_t lds0 = uint32_t(uintptr_t((ONECOMP_LDS char*)psm));
    uint16_t* const Fh = a.Fh + int64_t(wg) * (F16_BYTES / 2);
    uint16_t* const Fl = a.Fl + int64_t(wg) * (F16_BYTES / 2);
    double s = 1.0, rs = 1.0, z = 0.0;
    double lossacc = 0.0;   // of this lane's columns
    bool saturated = false;
    if (a.wide_g >= 0) {
        s = a.s64[grow];
        z = double(a.zeros[int64_t(grow) * a.n_g + a.wide_g]);
        rs = 1.0 / s;
    }
    static_assert(UD16_ZERO == 256, "a zero per thread");
    sUd[4 * UD16 + tid] = 0.0;

#pragma unroll 1
    for (int b = 0; b < a.nb; ++b) {
        const int j0 = a.s0 + b * SB;
        __syncthreads();   // everybody is done with the previous block's tiles
        {   // U's diagonal block -> LDS as in panel_body
            const float* ub = a.U + int64_t(j0) * d_in + j0;
            const __amdgpu_buffer_rsrc_t rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(ub), 0, int((int64_t(SB - 1) * d_in + SB) * 4), 0x00020000);
#pragma unroll
            for (int q = 0; q < 10; ++q) {
                const int t = q < 6 ? 6 * wave + q : 4 * wave + q - 6, blk = t >> 2;
                const int I = q < 6 ? (blk >= 3) + (blk >= 5) : wave, J = q < 6 ? (blk < 3 ? blk + 1 : blk < 5 ? blk - 1 : 3) : wave;
                const int row = 32 * I + 8 * (t & 3) + (lane >> 3);
                lds_load16(lds0 + (q < 6 ? 0 : LDS_DIAG) + t * 1024, uint32_t((row * int(d_in) + 32 * J + (lane & 7) * 4) * 4), rsrc);
            }
        }
        float w0v[8];   // original weights: columns 32 q + 2 sl + i of the block in w0v[2 q + i]
        {
            float cf[8];
            float16v acc;
            const int rows = min(ROWS16, a.d_out - r0), col = j0 + 32 * wave + lc;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.Wf + int64_t(r0) * d_in), 0,
                                                                                  a.s0 > 0 ? int(rows * d_in * 4) : 0, 0x00020000);
#pragma unroll
            for (int r = 0; r < 8; ++r) {   // rows past d_out read the last one
                const plan::FeedbackOffset o = plan::panel_feedback_offset<false>(rows, int(d_in), lane, 0, r, col);
                cf[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o.lane, o.scalar, 0));
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            if (a.w0_bf16) {
                const uint16_t* wp = static_cast<const uint16_t*>(a.W0) + int64_t(grow) * d_in + j0 + 2 * sl;
#pragma unroll
                for (int q = 0; q < 4; ++q) w0v[2 * q] = __uint_as_float(*reinterpret_cast<const uint32_t*>(wp + 32 * q));
            } else {
                const float* wp = static_cast<const float*>(a.W0) + int64_t(grow) * d_in + j0 + 2 * sl;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float2 v = *reinterpret_cast<const float2*>(wp + 32 * q);
                    w0v[2 * q] = v.x;
                    w0v[2 * q + 1] = v.y;
                }
            }
            if (b > 0) {
                constexpr int WIN = 4, B_BYTES = 6 * 8 * 4 * 64 * 16, DESC = 0x00020000;
                uint4v win[WIN][4];
                const __amdgpu_buffer_rsrc_t rfh = __builtin_amdgcn_make_buffer_rsrc(Fh, 0, F16_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rfl = __builtin_amdgcn_make_buffer_rsrc(Fl, 0, F16_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rbh = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.Bh), 0, B_BYTES, DESC);
                const __amdgpu_buffer_rsrc_t rbl = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.Bl), 0, B_BYTES, DESC);
                const int b0 = ((b * (b - 1) / 2) * 8 * 4 + wave) * 1024;
                const int va = (lane >> 5) * 256 + (lane & 15) * 16, vb = lane * 16;
                auto issue = [&](int bp, int ks, uint4v(&d)[4]) __attribute__((always_inline)) {
                    const int fo = (bp * 8 + ks) * 512, bo = b0 + (bp * 8 + ks) * 4 * 1024;
                    d[0] = __builtin_amdgcn_raw_buffer_load_b128(rfl, va, fo, 0);
                    d[1] = __builtin_amdgcn_raw_buffer_load_b128(rfh, va, fo, 0);
                    d[2] = __builtin_amdgcn_raw_buffer_load_b128(rbh, vb, bo, 0);
                    d[3] = __builtin_amdgcn_raw_buffer_load_b128(rbl, vb, bo, 0);
                };
#pragma unroll
                for (int ks = 0; ks < WIN; ++ks) issue(0, ks, win[ks]);
#pragma unroll 1
                for (int bp = 0; bp < b; ++bp) {
                    const bool more = bp + 1 < b;
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        uint4v(&cur)[4] = win[ks % WIN];
                        const half8v al = __builtin_bit_cast(half8v, cur[0]), ah = __builtin_bit_cast(half8v, cur[1]);
                        const half8v bh = __builtin_bit_cast(half8v, cur[2]), bl = __builtin_bit_cast(half8v, cur[3]);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, acc, 0, 0, 0);
                        if (ks + WIN < 8) issue(bp, ks + WIN, cur);
                        else if (more) issue(bp + 1, ks + WIN - 8, cur);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) cf[r] = __builtin_fmaf(acc[r], f_inv, cf[r]);
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));   // the direct loads have landed
            __syncthreads();
            {   // sub-block (wave, wave) for the sequential part
                const float* ug = sUg + wave * UB;
                if (lane < IB) sRd[32 * wave + lane] = 1.0 / double(ug[lane * (IB + 1)]);
                wave_fence();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int id = q * 64 + lane, j = id >> 3, k0 = (id & 7) * 4;
                    const float4v v = *reinterpret_cast<const float4v*>(ug + 4 * id);
                    const double rd = sRd[32 * wave + j];
                    double2 lo, hi;
                    lo.x = k0 > j ? double(v[0]) * rd : 0.0;
                    lo.y = k0 + 1 > j ? double(v[1]) * rd : 0.0;
                    hi.x = k0 + 2 > j ? double(v[2]) * rd : 0.0;
                    hi.y = k0 + 3 > j ? double(v[3]) * rd : 0.0;
                    if (j < 16 || k0 >= 16) {
                        double2* const dst = reinterpret_cast<double2*>(sUd + wave * UD16 + (j < 16 ? j * IB + k0 : 16 * j + 256 + k0 - 16));
                        dst[0] = lo;
                        dst[1] = hi;
                    }
                }
            }
            if (a.w0_bf16)
#pragma unroll
                for (int q = 3; q >= 0; --q) {
                    const uint32_t v = __float_as_uint(w0v[2 * q]);
                    w0v[2 * q] = __uint_as_float(v << 16);
                    w0v[2 * q + 1] = __uint_as_float(v & 0xFFFF0000u);
                }
            __syncthreads();
            auto to_lds = [&](auto&& v) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 8; ++r) sC[((r / 4) * 8 + lr + (r % 4)) * SP + 32 * wave + lc] = v(r);
            };
            if constexpr (!DIRECT) {
                to_lds([&](int r) __attribute__((always_inline)) { return cf[r]; });
            } else {
                // (c / diag) U_bb as in panel_body, a column tile per wave
                float16v c0;
#pragma unroll
                for (int r = 0; r < 16; ++r) c0[r] = 0.f;
                if (j0 > 0) {
                    const float rd = float(sRd[32 * wave + lc]);
                    to_lds([&](int r) __attribute__((always_inline)) { return cf[r] * rd; });
                    __syncthreads();
                    const float* ap = sC + (lc & 15) * SP + (lane >> 5);
#pragma unroll 1
                    for (int ch = 0; ch <= wave; ++ch) {
                        const float* bp = (ch == wave ? sUg + ch * UB : sU + u_off(ch, wave)) + (lane >> 5) * IB + lc;
                        float av[16], bv[16];
#pragma unroll
                        for (int kk = 0; kk < 16; ++kk) {
                            av[kk] = ap[32 * ch + 2 * kk];
                            bv[kk] = bp[2 * kk * IB];
                        }
#pragma unroll
                        for (int kk = 0; kk < 16; ++kk) c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk], bv[kk], c0, 0, 0, 0);
                    }
                    __syncthreads();   // every wave is done reading sC as an operand
                }
                to_lds([&](int r) __attribute__((always_inline)) { return c0[r]; });
            }
            __syncthreads();
        }

#pragma unroll 1
        for (int jb = 0; jb < SB; jb += IB) {
            float* const crow = sC + srow * SP + jb + 2 * sl;
            double w[2] = {double(w0v[0]) + double(crow[0]), double(w0v[1]) + double(crow[1])};
            double s_first = s, z_first = z;   // GB == 16: the grid of the inner block's first group
            auto fix_grid = [&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                const int col = j0 + jb + j;
                double mn, mx;
                if constexpr (GB == 16) {   // the 16 columns of lanes 8 (j / 16) .. + 7
                    mn = fmin(w[0], w[1]);
                    mx = fmax(w[0], w[1]);
                    mn = fmin(mn, dpp_quad<QUAD_SWAP1>(mn));
                    mx = fmax(mx, dpp_quad<QUAD_SWAP1>(mx));
                    mn = fmin(mn, dpp_quad<QUAD_SWAP2>(mn));
                    mx = fmax(mx, dpp_quad<QUAD_SWAP2>(mx));
                    mn = fmin(mn, dpp_quad<ROW_HALF_MIRROR>(mn));
                    mx = fmax(mx, dpp_quad<ROW_HALF_MIRROR>(mx));
                    mn = row_bcast<j / 2>(mn);
                    mx = row_bcast<j / 2>(mx);
                } else {
                    if (a.wide_g >= 0 || (col & (G - 1)) != 0) return;   // uniform: the group's G <= 128 columns are unfinished
                    mn = fmin(w[0], w[1]);
                    mx = fmax(w[0], w[1]);
#pragma unroll
                    for (int k = 2; k < 8; ++k) {   // two values per inner block that the group spans
                        if (k % 2 == 0 && 16 * k >= G) break;
                        const double v = double(w0v[k]) + double(crow[(k >> 1) * IB + (k & 1)]);
                        mn = fmin(mn, v);
                        mx = fmax(mx, v);
                    }
                    mn = fmin(mn, dpp_quad<ROW_ROR + 8>(mn));
                    mx = fmax(mx, dpp_quad<ROW_ROR + 8>(mx));
                    mn = fmin(mn, dpp_quad<ROW_ROR + 4>(mn));
                    mx = fmax(mx, dpp_quad<ROW_ROR + 4>(mx));
                    mn = fmin(mn, dpp_quad<ROW_ROR + 2>(mn));
                    mx = fmax(mx, dpp_quad<ROW_ROR + 2>(mx));
                    mn = fmin(mn, dpp_quad<ROW_ROR + 1>(mn));
                    mx = fmax(mx, dpp_quad<ROW_ROR + 1>(mx));
                }
                grid_params(mn, mx, 0, qmax, qsd, s, z);
                rs = 1.0 / s;
                if constexpr (GB == 16 && j == 0) { s_first = s; z_first = z; }
                if (sl == 0 && row_ok) {
                    a.scales[int64_t(grow) * a.n_g + (col >> a.lgG)] = float(s);
                    a.zeros[int64_t(grow) * a.n_g + (col >> a.lgG)] = float(z);
                }
            };
            // (w - s (q - z), q - z) of a value on the current grid, see panel_body
            auto quantize = [&](double v, double sq, double rsq, double zq, double& d) __attribute__((always_inline)) {
                const double t0 = v * rsq;
                const double t = __builtin_fma(__builtin_fma(-t0, sq, v), rsq, t0);
                d = fmin(fmax(rint(t), -zq), qmax - zq);
                return __builtin_fma(-sq, d, v);
            };
            auto pin = [](double& v) __attribute__((always_inline)) { asm volatile("" : "+v"(v)); };   // here, in this order
            // this lane's columns of U's rows 0 .. 15 and 16 .. 31, zero up to the diagonal
            const double* const ud = sUd + (jb >> 5) * UD16 + 2 * sl;
            const double* const ud_hi = sUd + (sl >= 8 ? (jb >> 5) * UD16 + 16 * IB + 2 * (sl - 8) : 4 * UD16 + 2 * sl);
            auto u_row = [&](int j) __attribute__((always_inline)) { return j < 16 ? ud + j * IB : ud_hi + (j - 16) * 16; };
            {
                double2 u[3];
                u[0] = *reinterpret_cast<const double2*>(u_row(0));
                u[1] = *reinterpret_cast<const double2*>(u_row(1));
                double res = 0.0;   // of the step before
                static_for<0, IB>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    auto late = [&]() __attribute__((always_inline)) {   // the other column's update of the step before
                        if constexpr (j > 0) {
                            const double2& up = u[(j + 2) % 3];
                            w[(j + 1) % 2] = __builtin_fma(-res, (j + 1) % 2 ? up.y : up.x, w[(j + 1) % 2]);
                            pin(w[(j + 1) % 2]);
                        }
                    };
                    constexpr bool fix = j % GB == 0;   // the group's grid needs all values up to date
                    if constexpr (fix) {
                        late();
                        fix_grid(jc);
                    }
                    double wj = row_bcast<j / 2>(w[j % 2]);
                    if constexpr (!fix) late();
                    double t0 = wj * rs;
                    pin(t0);
                    if constexpr (j + 2 < IB) u[(j + 2) % 3] = *reinterpret_cast<const double2*>(u_row(j + 2));
                    double r1 = __builtin_fma(-t0, s, wj);
                    pin(r1);
                    double t = __builtin_fma(r1, rs, t0);
                    pin(t);
                    t = fmin(fmax(rint(t), -z), qmax - z);   // pinned, the compiler would quiet NaNs before each of these
                    res = __builtin_fma(-s, t, wj);
                    pin(res);
                    if constexpr (j + 1 < IB) {
                        const double2& un = u[j % 3];
                        w[(j + 1) % 2] = __builtin_fma(-res, (j + 1) % 2 ? un.y : un.x, w[(j + 1) % 2]);
                        pin(w[(j + 1) % 2]);
                    }
                });
            }
            uint32_t pair[2];   // the residuals, hi in the lower half
            {
                const bool first = GB == 16 && sl < 8;
                const double sq = first ? s_first : s, zq = first ? z_first : z;
                const double rsq = GB == 16 ? 1.0 / sq : rs;
                float err[2];
                uint32_t codes;
                double loss;
                bool big;
                auto settle = [&]() __attribute__((always_inline)) {
                    codes = 0;
                    loss = lossacc;
                    big = false;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        double d;
                        const double r = quantize(w[i], sq, rsq, zq, d);
                        const double e = r * sRd[jb + 2 * sl + i];
                        loss = __builtin_fma(e, e, loss);
                        err[i] = float(e);
                        codes |= uint32_t(int(d + zq)) << (8 * i);
                        float x = -float(DIRECT ? __builtin_fma(-sq, d, double(w0v[i])) : r) * f_d;
                        big |= !(fabsf(x) <= 60000.f);
                        x = fminf(fmaxf(x, -60000.f), 60000.f);
                        const _Float16 h = (_Float16)x;
                        const _Float16 l = (_Float16)(x - (float)h);
                        pair[i] = uint32_t(__builtin_bit_cast(uint16_t, h)) | (uint32_t(__builtin_bit_cast(uint16_t, l)) << 16);
                    }
                };
                settle();
                if (__builtin_expect(__any(!(loss < __builtin_inf())), 0)) {   // see panel_body
                    w[0] = double(w0v[0]) + double(crow[0]);
                    w[1] = double(w0v[1]) + double(crow[1]);
#pragma unroll 1
                    for (int j = 0; j < IB; ++j) {
                        const double sg = GB == 16 && j < 16 ? s_first : s, zg = GB == 16 && j < 16 ? z_first : z;
                        const double rsg = GB == 16 ? 1.0 / sg : rs;
                        double d;
                        const double r = quantize(__shfl((j & 1) ? w[1] : w[0], (lane & ~15) + (j >> 1), 64), sg, rsg, zg, d);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if (2 * sl + i > j) w[i] = __builtin_fma(-r, u_row(j)[i], w[i]);
                    }
                    settle();
                }
                lossacc = loss;
                saturated |= row_ok && big;
                crow[0] = err[0];
                crow[1] = err[1];
                if (row_ok) {
                    *reinterpret_cast<uint16_t*>(a.Q + int64_t(grow) * d_in + j0 + jb + 2 * sl) = uint16_t(codes);
                    if (a.W_hat) {
                        const float sf = float(sq), zf = float(zq);
                        *reinterpret_cast<float2*>(a.W_hat + int64_t(grow) * d_in + j0 + jb + 2 * sl) =
                            make_float2(sf * (float(codes & 255u) - zf), sf * (float(codes >> 8) - zf));
                    }
                }
                // A-operand fragments for the near updates: k-step, half of its columns, row, column of the half
                if (b + 1 < a.nb) {
                    const int off = ((b * 8 + (jb >> 4) + (sl >> 3)) * 2 + ((sl >> 2) & 1)) * (ROWS16 * 8) + srow * 8 + 2 * (sl & 3);
                    *reinterpret_cast<uint32_t*>(Fh + off) = __builtin_amdgcn_perm(pair[1], pair[0], 0x05040100u);
                    *reinterpret_cast<uint32_t*>(Fl + off) = __builtin_amdgcn_perm(pair[1], pair[0], 0x07060302u);
                }
            }
            // Remaining columns of the block, see panel_body: 32 columns per wave
            if (jb + IB < SB) {
                __syncthreads();   // the other waves' errors
                const int I = jb >> 5;
                if (wave < 3 - I) {
                    const int l16 = lane & 15, lk = lane >> 4;
                    const float* const bp = sU + u_off(I, I + 1 + wave) + lk * IB + 2 * l16;
                    float* const cp = sC + 4 * lk * SP + jb + IB * (1 + wave) + 2 * l16;
                    float av[8];
                    float2 bv[8], old[4];
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        av[kk] = -sC[l16 * SP + jb + 4 * kk + lk];
                        bv[kk] = *reinterpret_cast<const float2*>(bp + 4 * kk * IB);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) old[r] = make_float2(cp[r * SP], cp[r * SP + 1]);
                    float4v c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kk], bv[kk].x, c0, 0, 0, 0);
                        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kk], bv[kk].y, c1, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        cp[r * SP] = old[r].x + c0[r];
                        cp[r * SP + 1] = old[r].y + c1[r];
                    }
                }
                __syncthreads();
            }
            crow[0] = __uint_as_float(pair[0]);
            crow[1] = __uint_as_float(pair[1]);
#pragma unroll
            for (int i = 0; i < 6; ++i) w0v[i] = w0v[i + 2];   // the next inner block's first
        }

        // ---- block done: the residuals transposed (k-major) for the far update, 8 rows of a column per lane
        __syncthreads();
        {
            const int r8 = 8 * (tid & 1), c = tid >> 1;
            uint32_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __float_as_uint(sC[(r8 + e) * SP + c]);
            const int64_t off = int64_t(b * SB + c) * a.ldD + r0 + r8;
            uint4v dh, dl;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                dh[e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x05040100u);
                dl[e] = __builtin_amdgcn_perm(v[2 * e + 1], v[2 * e], 0x07060302u);
            }
            *reinterpret_cast<uint4v*>(a.Dh + off) = dh;
            *reinterpret_cast<uint4v*>(a.Dl + off) = dl;
        }
        // the fragments written above are read back by other waves of this workgroup: see panel_body
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }
#pragma unroll
    for (int o = 1; o < 16; o *= 2) lossacc += __shfl_xor(lossacc, o, 16);
    if (sl == 0 && row_ok) a.rowloss[grow] += float(lossacc);
    if (saturated) *a.sat = 1u;
}

// ------------------------------------------------------------------------------------------
// Operands of the trailing GEMMs and of the panel's near updates (once per layer).  The feedback e_j U_jk is computed as
// (w_j - w^_j) * (U_jk / U_jj): the residual is bounded by the weights and the normalized row by the
// regression coefficients between input channels, so both fit fp16 after a power-of-two scaling taken
// from their maxima, whereas e and U themselves span the scale of 1 / sqrt(H_jj).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ Scalars make_scales(float mw, float mu) {
    // largest magnitudes land at 2^13 (residuals, x8 headroom before saturation) and 2^14 (rows of U)
    int ew = 0, eu = 0;
    if (mw > 0.f) (void)frexpf(mw, &ew);   // mw = m * 2^ew, 0.5 <= m < 1
    if (mu > 0.f) (void)frexpf(mu, &eu);
    const int sd = max(-60, min(60, 13 - ew)), su = max(-60, min(60, 14 - eu));
    Scalars s;
    s.max_w_bits = __float_as_uint(mw);
    s.max_u_bits = __float_as_uint(mu);
    s.f_d = ldexpf(1.f, sd);
    s.f_u = ldexpf(1.f, su);
    s.f_all = ldexpf(1.f, sd + su);
    s.f_inv = ldexpf(1.f, -(sd + su));
    return s;
}
// u / dj * f_u as fp16 hi + lo
__device__ __forceinline__ void split_ratio(float u, float dj, float f_u, short& hi, short& lo) {
    float x = u / dj * f_u;
    x = fminf(fmaxf(x, -60000.f), 60000.f);
    const _Float16 h = (_Float16)x;
    hi = __builtin_bit_cast(short, h);
    lo = __builtin_bit_cast(short, (_Float16)(x - (float)h));
}

// Every workgroup forms the scales from the maxima that prepare_kernel left (8 KB out of L2; a launch for it: 4.7 us), the first
// one leaves them in sc and clears the saturation flag.
// Workgroups 0 .. n_near - 1, NEAR_PARTS per block pair, the fragments of the normalized U blocks that the panel kernel's near
// updates multiply with: for super-block S (sbw columns wide, n_pairs block pairs), block pair p = b (b - 1) / 2 + b' (b' < b),
// k-step ks, column tile nt, lane L:
//   Un[sbw S + 128 b' + 16 ks + 8 (L/32) + e][sbw S + 128 b + 32 nt + L%32] * f_u,  e = 0 .. 7,  fp16 hi and lo.
// The others, rows of the trailing updates' operand, which is read beyond row j's 128-column block only; the rest of Uh / Ul
// stays unwritten.
constexpr int NEAR_PARTS = 4;
__global__ __launch_bounds__(256) void operands_kernel(const float* __restrict__ U, int n, const float* __restrict__ max_u, int n_u,
                                                      const float* __restrict__ max_w, int n_w, Scalars* __restrict__ sc,
                                                      uint16_t* __restrict__ Bh, uint16_t* __restrict__ Bl, int sbw, int n_pairs,
                                                      int n_near, uint16_t* __restrict__ Uh, uint16_t* __restrict__ Ul) {
    __shared__ float part[4];
    float mu = 0.f, mw = 0.f;
#pragma unroll
    for (int q = 0; q < PREP_WGS / 256; ++q) {
        const int i = threadIdx.x + 256 * q;
        if (i < n_u) mu = fmaxf(mu, max_u[i]);
        if (i < n_w) mw = fmaxf(mw, max_w[i]);
    }
    mu = block_max(mu, part);
    mw = block_max(mw, part);
    const Scalars s = make_scales(mw, mu);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *sc = s;
        *sat_flag(sc) = 0u;
    }
    const float f_u = s.f_u;
    if (int(blockIdx.x) < n_near) {
        const int pair = blockIdx.x / NEAR_PARTS, S = pair / n_pairs, p = pair % n_pairs;
        const int b = (p >= 3) ? 3 : (p >= 1 ? 2 : 1), bp = p - b * (b - 1) / 2;
        const int k00 = S * sbw + bp * SB, n00 = S * sbw + b * SB;
        if (n00 >= n) return;
        constexpr int each = 8 * 4 * 64 / NEAR_PARTS;
        for (int it = blockIdx.x % NEAR_PARTS * each + threadIdx.x, i = 0; i < each / 256; ++i, it += 256) {
            const int L = it & 63, nt = (it >> 6) & 3, ks = it >> 8;
            const int col = n00 + nt * 32 + (L & 31), k0 = k00 + ks * 16 + 8 * (L >> 5);
            short8v h8, l8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                short h, l;
                split_ratio(U[int64_t(k0 + e) * n + col], U[int64_t(k0 + e) * n + k0 + e], f_u, h, l);
                h8[e] = h;
                l8[e] = l;
            }
            const int64_t off = (int64_t(pair) * (8 * 4 * 64) + it) * 8;
            *reinterpret_cast<short8v*>(Bh + off) = h8;
            *reinterpret_cast<short8v*>(Bl + off) = l8;
        }
        return;
    }
    for (int j = blockIdx.x - n_near; j < n; j += gridDim.x - n_near) {
        const int64_t row = int64_t(j) * n;
        const float dj = U[row + j];
        for (int k4 = (j / SB + 1) * SB + 4 * threadIdx.x; k4 < n; k4 += 1024) {
            const float4v v = *reinterpret_cast<const float4v*>(U + row + k4);
            short4v h4, l4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                short h, l;
                split_ratio(v[e], dj, f_u, h, l);
                h4[e] = h;
                l4[e] = l;
            }
            *reinterpret_cast<short4v*>(Uh + row + k4) = h4;
            *reinterpret_cast<short4v*>(Ul + row + k4) = l4;
        }
    }
}

// ------------------------------------------------------------------------------------------
// trailing update:  Wf[:, c0 .. c1) += f_inv * D[:, ek .. ek+K) * Un[u0 .. u0+K, c0 .. c1)
// with D = -(w - w^) f_d (stored transposed, Dt[k][row], by the panel kernel) and Un = U_jk / U_jj f_u
// (operands_kernel).
//
// fp32 accuracy from fp16 MFMAs: both operands are split x = hi + lo (fp16 each, |lo| <= 2^-11 |hi|) and
// three products are accumulated in fp32, hi*hi + hi*lo + lo*hi; the dropped lo*lo term and the rounding
// of lo are ~2^-22 relative to each product, i.e. the level of fp32 rounding itself.
//
// 128 x 256 tile per workgroup, 4 waves in 2 x 2 (64 x 128 each: 2 x 4 tiles of v_mfma_f32_32x32x16_f16, three
// products each), two workgroups per CU so that one workgroup's read and write of its W tile (the update is
// close to the HBM / MFMA ridge: 384 flop per byte of W at K = 512) overlaps the other's inner loop.
// Both operands are k-major, their fragments come from LDS transpose reads.  Operand tiles go global -> LDS
// directly (lds_load16) in steps of 16 k: four panels (Dt hi, Dt lo, Un hi, Un lo) of 16 rows, 24 KB, in a
// ring of three slots.  16-byte chunk c of panel row r sits at chunk position c ^ ((r & 3) << 2), which spreads
// the four rows of a transpose read over four 64-byte bank groups.
// Half-iteration h:  24 MFMAs on the fragments of k-step h (registers);  LDS -> fragments of k-step h+1;
// loads of k-step h+3 into the slot k-step h was read from;  wait for k-step h+2 + barrier.
// Tiles are ranked so that each XCD (blockIdx % 8) owns a contiguous run, m fastest inside bands of 8 row tiles:
// the workgroups resident on one XCD share their Dt and Un panels through its L2.
// ------------------------------------------------------------------------------------------
// The same with a 64 x 128 tile (32 x 64 per wave, 12 KB a step, six slots) for launches of few tiles, see launch_trailing.
// An entry's products are added in the same order.  Rows of 64 left-operand entries are 128 bytes, eight chunks: their
// position is c ^ ((r & 2) << 1).
template <int MT_, int NT_, int NBUF_>   // 32 x 32 tiles of a wave, slots of the LDS ring
struct TrailShape {
    static constexpr int MT = MT_, NT = NT_, NBUF = NBUF_, TM = 64 * MT, TN = 64 * NT, KT = 16;
    static constexpr int A_ROWB = TM * 2, B_ROWB = TN * 2;                     // bytes per panel row
    static constexpr int A_PANELB = KT * A_ROWB, B_PANELB = KT * B_ROWB;       // 4 KB, 8 KB
    static constexpr int OFF_AH = 0, OFF_AL = A_PANELB, OFF_BH = 2 * A_PANELB, OFF_BL = 2 * A_PANELB + B_PANELB;
    static constexpr int STAGEB = 2 * A_PANELB + 2 * B_PANELB;                 // 24 KB
    static constexpr size_t LDS_BYTES = size_t(NBUF) * STAGEB;                 // 72 KB: two workgroups per CU
    static constexpr int LPW = STAGEB / 4096;                                  // loads per wave and step
    static constexpr int A_LPW = MT;                                           // .. of the left operand
    static_assert(MT <= 2 && NT % 2 == 0 && A_LPW + NT == LPW, "a wave loads MT and NT KB");
};
using TrailBig = TrailShape<2, 4, 3>;
using TrailSmall = TrailShape<1, 2, 6>;

struct TrailArgs {
    float* Wf;
    const uint16_t *Dh, *Dl;   // [SBIG x ldD] fp16 bits
    const uint16_t *Uh, *Ul;   // [d_in x d_in] fp16 bits
    const Scalars* sc;
    int d_out, ldD, d_in;
    int ek, K, u0, c0, c1;     // K % 32 == 0, c0 % 8 == 0, c1 % 8 == 0
    int n_mt, n_nt, chunk;
    int n_nt0, h0, h1;         // not INCREMENT: the first n_nt0 column tiles cover [c0, h0), the others [h1, c1)
    int first;                 // INCREMENT: nothing has been added to these columns, they are written without being read
    int tri, fold;             // PRODUCT: Triangle (h0 == c1, c0 == 0) and triangular_tile's argument
    uint32_t* max_bits;        // PRODUCT: max |C| joins this (nullptr: not wanted)
};

// INCREMENT: the accumulators start at zero and the product is added to the tile of C once, at the end, with one
// fp32 rounding (the sweep: every rounding inside the MFMA chain then happens at the size of the increment, not of
// the sum it joins).  SUM: the tile of C is loaded, scaled, into the accumulators before the loop.  PRODUCT: C is written without
// being read, see split_product.
enum TrailMode : int { SUM, INCREMENT, PRODUCT };
template <typename S, TrailMode MODE>
__device__ __forceinline__ void trailing_tile(const TrailArgs& a, const int bid, char* tl) {
    constexpr bool FROM_ZERO = MODE == INCREMENT;
    constexpr int MT = S::MT, NT = S::NT, NBUF = S::NBUF, TM = S::TM, TN = S::TN, KT = S::KT, LPW = S::LPW;
    constexpr int A_ROWB = S::A_ROWB, B_ROWB = S::B_ROWB, A_PANELB = S::A_PANELB, B_PANELB = S::B_PANELB, STAGEB = S::STAGEB;
    constexpr int OFF_AH = S::OFF_AH, OFF_AL = S::OFF_AL, OFF_BH = S::OFF_BH, OFF_BL = S::OFF_BL;
    int mt_, nt_;
    const bool triangle = MODE == PRODUCT && a.tri != TRI_NONE;
    if (!(triangle ? plan::triangular_tile(bid, a.n_mt, a.n_nt, a.tri == TRI_LOWER, a.fold, mt_, nt_)
                   : plan::trail_tile(bid, a.chunk, a.n_mt, a.n_nt, mt_, nt_)))
        return;
    const int m0 = mt_ * TM;
    const bool beyond = !FROM_ZERO && nt_ >= a.n_nt0;
    const int n0 = beyond ? a.h1 + (nt_ - a.n_nt0) * TN : a.c0 + nt_ * TN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int d_out = a.d_out, c1 = FROM_ZERO || beyond ? a.c1 : a.h0;
    const int64_t d_in = a.d_in;
    const uint32_t lds0 = uint32_t(uintptr_t((ONECOMP_LDS char*)tl));

    // this wave's 1 KB loads per k-step.  128 x 256: rows 4 wave .. 4 wave + 3 of both Dt panels (one load each), the same
    // rows of the Un panels (two loads of two rows each); 64 x 128: eight rows of one Dt panel (waves 0, 1: hi, 2, 3: lo),
    // four rows of each Un panel
    uint32_t voff_a, voff_b[NT / 2];
    {
        constexpr int CPR = A_ROWB / 16;   // chunks per row
        const int row = (MT == 2 ? 4 * wave : 8 * (wave & 1)) + lane / CPR;
        const int c = (lane % CPR) ^ (MT == 2 ? (row & 3) << 2 : (row & 2) << 1);
        voff_a = (m0 + c * 8 < a.ldD) ? uint32_t((row * a.ldD + m0 + c * 8) * 2) : LDS_DMA_OOB;
    }
#pragma unroll
    for (int q = 0; q < NT / 2; ++q) {
        constexpr int CPR = B_ROWB / 16;
        const int row = 4 * wave + (NT == 4 ? 2 * q : 0) + lane / CPR;
        const int c = (lane % CPR) ^ ((row & 3) << 2);
        voff_b[q] = (n0 + c * 8 < c1) ? uint32_t((int64_t(row) * d_in + n0 + c * 8) * 2) : LDS_DMA_OOB;
    }
    const int k_lo = triangle && a.tri == TRI_LOWER ? n0 : 0, k_hi = triangle && a.tri == TRI_UPPER ? min(a.K, n0 + TN) : a.K;
    const int n_kb = (k_hi - k_lo) / KT;
    struct Desc {
        __amdgpu_buffer_rsrc_t ah, al, bh, bl;
    };
    // descriptors of the next k-step, empty ones behind the last.  The bases advance by additions: formed by products in
    // every step, they held back a 64 x 128 tile (14.2 against 13.9 us, 512 columns at d_out 4096).
    const uint16_t *pah = a.Dh + int64_t(a.ek + k_lo) * a.ldD, *pal = a.Dl + int64_t(a.ek + k_lo) * a.ldD;
    const uint16_t *pbh = a.Uh + int64_t(a.u0 + k_lo) * d_in, *pbl = a.Ul + int64_t(a.u0 + k_lo) * d_in;
    const int step_a = KT * a.ldD, step_b = KT * a.d_in;
    int ahead = n_kb;
    auto next_desc = [&]() __attribute__((always_inline)) {
        Desc d;
        const int ra = ahead > 0 ? step_a * 2 : 0, rb = ahead > 0 ? step_b * 2 : 0;
        --ahead;
        d.ah = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pah), 0, ra, 0x00020000);
        d.al = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pal), 0, ra, 0x00020000);
        d.bh = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pbh), 0, rb, 0x00020000);
        d.bl = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(pbl), 0, rb, 0x00020000);
        pah += step_a;
        pal += step_a;
        pbh += step_b;
        pbl += step_b;
        return d;
    };
    // load number i of a k-step into the slot at LDS byte address dst
    auto gload1 = [&](const Desc& d, uint32_t dst, int i) __attribute__((always_inline)) {
        if (i < S::A_LPW) {
            if (MT == 2) lds_load16(dst + (i == 0 ? OFF_AH : OFF_AL) + wave * 1024, voff_a, i == 0 ? d.ah : d.al);
            else if (wave < 2) lds_load16(dst + OFF_AH + wave * 1024, voff_a, d.ah);
            else lds_load16(dst + OFF_AL + (wave - 2) * 1024, voff_a, d.al);
        } else {
            const int q = (i - S::A_LPW) % (NT / 2);
            const bool hi = i - S::A_LPW < NT / 2;
            lds_load16(dst + (hi ? OFF_BH : OFF_BL) + (wave * (NT / 2) + q) * 1024, voff_b[q], hi ? d.bh : d.bl);
        }
    };

    // transpose-read addressing: within 16 lanes, lane 4 k + c reads 8 bytes of panel row k at byte 8 c of a
    // 32-byte column group; two reads (rows +0 and +4) make one MFMA operand (k = 8 (lane / 32) + 0..7)
    const int i16 = lane & 15, g16 = (lane >> 4) & 1, kb8 = lane >> 5;
    const int kq = i16 >> 2;
    const int lo = (2 * g16 + ((i16 & 3) >> 1)) * 16 + (i16 & 1) * 8;
    int fa[MT], fb[NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
        fa[m] = OFF_AH + (kb8 * 8 + kq) * A_ROWB + (((wr * MT + m) ^ (MT == 2 ? kq : kq >> 1)) << 6) + lo;
#pragma unroll
    for (int n = 0; n < NT; ++n) fb[n] = OFF_BH + (kb8 * 8 + kq) * B_ROWB + (((wc * NT + n) ^ kq) << 6) + lo;

    struct Frags {
        half8v ah[MT], al[MT], bh[NT], bl[NT];
    };
    auto rd2 = [&](const char* p, int rowb) __attribute__((always_inline)) {
        short4v x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ONECOMP_LDS short4v*)(p));
        short4v x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ONECOMP_LDS short4v*)(p + 4 * rowb));
        return __builtin_bit_cast(half8v, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    constexpr int N_FRAGS = 2 * (MT + NT), N_MMA = 3 * MT * NT;
    // fragment r of the slot at tl + sb, in the order the MFMAs use them
    auto rd = [&](Frags& f, int r, int sb) __attribute__((always_inline)) {
        const char* s = tl + sb;
        if (r == 0) f.al[0] = rd2(s + fa[0] + A_PANELB, A_ROWB);
        else if (r <= NT) f.bh[r - 1] = rd2(s + fb[r - 1], B_ROWB);
        else if (r == NT + 1) f.ah[0] = rd2(s + fa[0], A_ROWB);
        else if (r <= 2 * NT + 1) f.bl[r - NT - 2] = rd2(s + fb[r - NT - 2] + B_PANELB, B_ROWB);
        else if (r == 2 * NT + 2) f.al[MT - 1] = rd2(s + fa[MT - 1] + A_PANELB, A_ROWB);
        else f.ah[MT - 1] = rd2(s + fa[MT - 1], A_ROWB);
    };

    // prologue: the ring's k-steps in flight, then the W tile (scaled by the exact power of two f_d f_u) straight into
    // the accumulators; register r of lane l is row (r/4)*8 + (l/32)*4 + r%4, column l%32 of a 32 x 32 tile
    for (int kb = 0; kb < NBUF; ++kb)
        if (kb < n_kb) {
            const Desc d = next_desc();
#pragma unroll
            for (int i = 0; i < LPW; ++i) gload1(d, lds0 + kb * STAGEB, i);
        }
    const float f_all = a.sc->f_all, f_inv = a.sc->f_inv;
    float16v acc[MT][NT];
    const int lr = (lane >> 5) * 4, lc = lane & 31;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if constexpr (MODE != SUM) {
                    acc[m][n][r] = 0.f;
                } else {
                    const int rr = min(m0 + wr * (32 * MT) + m * 32 + (r / 4) * 8 + lr + (r % 4), d_out - 1);
                    const int cc = min(n0 + wc * (32 * NT) + n * 32 + lc, c1 - 1);
                    acc[m][n][r] = a.Wf[int64_t(rr) * d_in + cc] * f_all;
                }
            }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
    __syncthreads();
    Frags Fc, FH;
#pragma unroll
    for (int r = 0; r < N_FRAGS; ++r) rd(Fc, r, 0);
    __syncthreads();   // slot 0 is overwritten by the loads of the first half-iteration

    // the MFMAs of one k-step: per row tile m the products lo*hi, hi*lo, hi*hi against the column tiles, consecutive MFMAs on
    // different accumulators; `between(i)` is placed behind MFMA i
    auto mma = [&](const Frags& f, auto&& between) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < N_MMA; ++i) {
            const int m = i / (3 * NT), p = i % (3 * NT) / NT, n = i % NT;
            if (p == 0) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.al[m], f.bh[n], acc[m][n], 0, 0, 0);
            else if (p == 1) acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.ah[m], f.bl[n], acc[m][n], 0, 0, 0);
            else acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.ah[m], f.bh[n], acc[m][n], 0, 0, 0);
            between(i);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // what goes behind MFMA i of a k-step: a fragment of the next one or a load
    auto beside = [&](Frags& f, int i, int sb, const Desc& d, uint32_t dst) __attribute__((always_inline)) {
        if constexpr (N_MMA >= 2 * N_FRAGS) {
            if ((i & 1) == 0) rd(f, i / 2, sb);
            else if (i / 2 < LPW) gload1(d, dst, i / 2);
        } else {
            rd(f, i, sb);
            if (i < LPW) gload1(d, dst, i);
        }
    };
    static_assert(N_MMA >= N_FRAGS && N_FRAGS >= LPW, "every fragment and every load has its place");

    int s0 = 0;   // slot of k-step kb
#pragma unroll 1
    for (int kb = 0; kb < n_kb; kb += 2) {
        const int s1 = (s0 == NBUF - 1) ? 0 : s0 + 1, s2 = (s1 == NBUF - 1) ? 0 : s1 + 1;
        // Loads and fragment reads past the last k-step are not branched around: the loads get an empty
        // descriptor (they deposit zeros into a slot nobody reads again), the reads fetch stale data nobody uses.
        {   // k-step kb from Fc; fragments of kb+1 -> FH; loads of kb+NBUF -> slot s0
            const Desc d = next_desc();
            const uint32_t dst = lds0 + s0 * STAGEB;
            const int sb = s1 * STAGEB;
            mma(Fc, [&](int i) __attribute__((always_inline)) {
                beside(FH, i, sb, d, dst);
            });
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(LPW * (NBUF - 2)));   // k-step kb+2 has landed
            __syncthreads();
        }
        {   // k-step kb+1 from FH; fragments of kb+2 -> Fc; loads of kb+1+NBUF -> slot s1
            const Desc d = next_desc();
            const uint32_t dst = lds0 + s1 * STAGEB;
            const int sb = s2 * STAGEB;
            mma(FH, [&](int i) __attribute__((always_inline)) {
                beside(Fc, i, sb, d, dst);
            });
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(LPW * (NBUF - 2)));   // k-step kb+3 has landed
            __syncthreads();
        }
        s0 = s2;
    }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));   // no LDS write may be in flight when the workgroup ends
    if (MODE == PRODUCT && a.max_bits) {
        float mx = 0.f;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool in = m0 + wr * (32 * MT) + m * 32 + (r / 4) * 8 + lr + (r % 4) < d_out && n0 + wc * (32 * NT) + n * 32 + lc < c1;
                    mx = fmaxf(mx, in ? fabsf(acc[m][n][r] * f_inv) : 0.f);
                }
        mx = wave_max(mx);
        if (lane == 0 && __float_as_uint(mx) > __hip_atomic_load(a.max_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(a.max_bits, __float_as_uint(mx));
    }
    // uniform branch: interior tiles store without per-element masks
    if ((m0 + TM <= d_out) && (n0 + TN <= c1)) {
        float* wp = a.Wf + int64_t(m0 + wr * (32 * MT) + lr) * d_in + n0 + wc * (32 * NT) + lc;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if constexpr (FROM_ZERO) {
                // the tile's current values: 32 independent loads at a time (the operand registers are free now)
#pragma unroll
                for (int n2 = 0; n2 < NT; n2 += 2) {
                    float16v old[2] = {};
                    if (!a.first) {
#pragma unroll
                        for (int n = 0; n < 2; ++n)
#pragma unroll
                            for (int r = 0; r < 16; ++r)
                                old[n][r] = wp[int64_t(m * 32 + (r / 4) * 8 + (r % 4)) * d_in + (n2 + n) * 32];
                    }
#pragma unroll
                    for (int n = 0; n < 2; ++n)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            wp[int64_t(m * 32 + (r / 4) * 8 + (r % 4)) * d_in + (n2 + n) * 32] =
                                __builtin_fmaf(acc[m][n2 + n][r], f_inv, old[n][r]);
                }
            } else {
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        wp[int64_t(m * 32 + (r / 4) * 8 + (r % 4)) * d_in + n * 32] = acc[m][n][r] * f_inv;
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rr = m0 + wr * (32 * MT) + m * 32 + (r / 4) * 8 + lr + (r % 4);
                    const int cc = n0 + wc * (32 * NT) + n * 32 + lc;
                    if (rr < d_out && cc < c1) {
                        float* q = a.Wf + int64_t(rr) * d_in + cc;
                        if constexpr (FROM_ZERO) *q = __builtin_fmaf(acc[m][n][r], f_inv, a.first ? 0.f : *q);
                        else *q = acc[m][n][r] * f_inv;
                    }
                }
    }
}

template <typename S, TrailMode MODE>
__global__ __launch_bounds__(256, 2) void trailing_kernel(TrailArgs a) {
    extern __shared__ __attribute__((aligned(1024))) char dyn_lds[];
    trailing_tile<S, MODE>(a, blockIdx.x, dyn_lds);
}

// One launch = the panel sweep of a super-block next to the far update of the previous super-block on the
// columns beyond the panel's.  The panel needs only 64 rows' worth of workgroups, far fewer than there are CUs, and
// its workgroups are the first of the grid, so they are resident from the start; the update's tiles fill the other
// CUs, and all of them once the panel is done.  The two parts touch disjoint columns of the working copy, and the
// panel writes the residual panels of its own super-block into the buffer the update does not read.
template <int GB, bool DIRECT, int ROWS_WG>
__global__ __launch_bounds__(256, 2) void panel_far_kernel(PanelArgs pa, TrailArgs ta, int n_panel) {
    extern __shared__ __attribute__((aligned(1024))) char dyn_lds[];
    if (int(blockIdx.x) < n_panel) {
        if constexpr (ROWS_WG == ROWS) panel_body<GB, DIRECT>(pa, blockIdx.x, dyn_lds);
        else panel_body16<GB, DIRECT>(pa, blockIdx.x, dyn_lds);
    }
    else trailing_tile<TrailBig, INCREMENT>(ta, blockIdx.x - n_panel, dyn_lds);
}

// Scale and zero-point of one wide group (columns g0 .. g0 + G - 1 of every row, G a multiple of 128) from its current
// values w0 + c in fp64: W0 the weights in sweep order, C the working copy (accumulated feedback; nullptr = none, the
// first group of a row or one group per row), which the caller guarantees to be complete for these columns: the far
// updates of all earlier super-blocks have run.  One workgroup per row; the fp64 scale goes to s64[row].
//
// The scale search is bound by its VALU operations, five per value and candidate.  A thread owns a candidate and a
// quarter of the values, which every lane reads from LDS at the same address, so that a candidate's grid (fp64
// divisions) is formed once per thread and nothing is reduced before the end; with the values spread over the threads
// every one of the 80 candidates had its divisions in all threads and a workgroup sum.  The sums are kept short (32
// values, four accumulators; 4096 values; the row).  1999 rows of 2048: 260 -> 49 us.
// Without the search (MSE false) the row's range is all there is: no values kept and four waves, so that eight workgroups
// share a CU.  14336 x 4096 bf16 in groups of 256, whole sweep: 2.79 ms when the search's workgroup of five waves with its
// values' LDS did this as well, 2.60 like this.
constexpr int GP_SLICES = 4, GP_THREADS = GP_SLICES * MSE_CANDIDATES, GP_CHUNK = 4096;
constexpr int gp_threads(bool mse) { return mse ? GP_THREADS : 256; }
template <typename T, bool MSE>
__global__ __launch_bounds__(gp_threads(MSE), 8) void group_params_kernel(   // 8: waves per SIMD
    const T* __restrict__ W0, const float* __restrict__ C, int d_out, int d_in, int g0, int G, float qmax, float qs, int n_g,
    int g_idx, float* __restrict__ scales, float* __restrict__ zeros, double* __restrict__ s64) {
    constexpr int THREADS = gp_threads(MSE), WAVES = THREADS / 64;
    __shared__ double smn[WAVES], smx[WAVES];
    __shared__ float part[MSE ? GP_SLICES : 1][MSE ? MSE_CANDIDATES : 1];
    __shared__ __attribute__((aligned(16))) float val[MSE ? GP_CHUNK : 4];
    const int tid = threadIdx.x;
    for (int64_t r = blockIdx.x; r < d_out; r += gridDim.x) {
        const T* row = W0 + r * d_in + g0;
        const float* crow = C ? C + r * d_in + g0 : nullptr;
        auto value = [&](int c) __attribute__((always_inline)) {
            return double(to_f32<T>(row[c])) + (crow ? double(crow[c]) : 0.0);
        };
        double mn = value(0), mx = mn;
        const bool keep = MSE && G <= GP_CHUNK;
        for (int c = tid; c < G; c += THREADS) {
            const double v = value(c);
            mn = fmin(mn, v); mx = fmax(mx, v);
            if (keep) val[c] = float(v);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            mn = fmin(mn, __shfl_xor(mn, off, 64));
            mx = fmax(mx, __shfl_xor(mx, off, 64));
        }
        if ((tid & 63) == 0) { smn[tid >> 6] = mn; smx[tid >> 6] = mx; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { mn = fmin(mn, smn[w]); mx = fmax(mx, smx[w]); }
        int cand = 0;
        if constexpr (MSE) {
            const int slice = tid / MSE_CANDIDATES, i = tid % MSE_CANDIDATES;
            double sd, zd;
            grid_params(mn, mx, i, double(qmax), double(qs), sd, zd);
            const float si = float(sd), zi = float(zd), rsi = 1.0f / si;
            float err = 0.f;
            for (int b = 0; b < G; b += GP_CHUNK) {
                const int cols = min(GP_CHUNK, G - b);
                if (!keep) {
                    __syncthreads();
                    for (int c = tid; c < cols; c += GP_THREADS) val[c] = float(value(b + c));
                    __syncthreads();
                }
                const float4v* src = reinterpret_cast<const float4v*>(val) + slice * (cols / (4 * GP_SLICES));
                float e_chunk = 0.f;
                for (int c = 0; c < cols / (4 * GP_SLICES); c += 8) {
                    float4v e4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float4v x = src[c + j];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float t = fmaf(x[e], rsi, zi);
                            const float d = t - __builtin_amdgcn_fmed3f(rintf(t), 0.f, qmax);   // see mse_term
                            e4[e] = fmaf(d, d, e4[e]);
                        }
                    }
                    e_chunk += (e4[0] + e4[1]) + (e4[2] + e4[3]);
                }
                err += e_chunk;
            }
            part[slice][i] = err;
            __syncthreads();
            if (tid < 64) {   // the first smallest error, as mse_search takes it
                auto total = [&](int k) __attribute__((always_inline)) {
                    return (part[0][k] + part[1][k]) + (part[2][k] + part[3][k]);
                };
                float best = 3.0e38f;
                auto offer = [&](float x, int k) __attribute__((always_inline)) {
                    if (x < best || (x == best && k < cand)) { best = x; cand = k; }
                };
                offer(si * si * total(tid), tid);
                if (tid < MSE_CANDIDATES - 64) {
                    const int k = tid + 64;
                    double s2, z2;
                    grid_params(mn, mx, k, double(qmax), double(qs), s2, z2);
                    offer(float(s2) * float(s2) * total(k), k);
                }
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) offer(__shfl_xor(best, off, 64), __shfl_xor(cand, off, 64));
            }
        }
        double s, z;
        if (tid == 0) {
            grid_params(mn, mx, cand, double(qmax), double(qs), s, z);
            scales[r * n_g + g_idx] = float(s);
            zeros[r * n_g + g_idx] = float(z);
            s64[r] = s;
        }
        __syncthreads();   // the next row's values and partial results go to the same LDS
    }
}

// Column order (activation ordering): the sweep stages its codes in sweep order (coalesced rows); the caller's
// arrays are then written in ORIGINAL column order, coalesced, gathering from the staged row (a row is a few KB and
// stays in cache).  W^ is recomputed as s (q - z), the same fp32 operations the sweep used.
__global__ __launch_bounds__(256) void inv_perm_kernel(const int32_t* __restrict__ perm, int n, int32_t* __restrict__ inv) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < n) inv[perm[p]] = p;
}

__global__ __launch_bounds__(256) void unpermute_kernel(const uint8_t* __restrict__ Qs, const float* __restrict__ scales,
                                                       const float* __restrict__ zeros, const int32_t* __restrict__ inv,
                                                       int d_out, int d_in, int G, int n_g, uint8_t* __restrict__ Q,
                                                       float* __restrict__ W_hat) {
    for (int64_t r = blockIdx.y; r < d_out; r += gridDim.y) {
        const int oc = (blockIdx.x * 256 + threadIdx.x) * 4;   // d_in % 128 == 0: whole groups of 4 columns
        if (oc >= d_in) continue;
        const int4 pv = *reinterpret_cast<const int4*>(inv + oc);
        const int ps[4] = {pv.x, pv.y, pv.z, pv.w};
        uint32_t pk = 0;
        float4v h;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t q = Qs[r * d_in + ps[e]];
            const int g = ps[e] / G;
            h[e] = scales[r * n_g + g] * (float(q) - zeros[r * n_g + g]);
            pk |= q << (8 * e);
        }
        *reinterpret_cast<uint32_t*>(Q + r * d_in + oc) = pk;
        if (W_hat) *reinterpret_cast<float4v*>(W_hat + r * d_in + oc) = h;
    }
}

// loss = sum of the per-row sums, fixed order; +infinity if a residual was saturated on its way into the fp16
// operands of the feedback products (the codes of later columns are then not those of the sweep).  One workgroup.
__global__ __launch_bounds__(1024) void loss_kernel(const float* __restrict__ rowloss, int d_out,
                                                   const uint32_t* __restrict__ sat, float* __restrict__ loss) {
    __shared__ double part[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < d_out; i += 1024) s += double(rowloss[i]);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = *sat ? __builtin_inff() : float(part[0]);
}

struct SweepWs {
    float* Wf;        // [d_out x d_in] working copy, sweep order
    uint16_t* Dh;     // 2 x [SBIG x ldD] scaled negated residuals of a super-block, transposed, fp16 hi; two buffers:
    uint16_t* Dl;     // one is read by the far update while the next super-block fills the other       fp16 lo
    uint16_t* Uh;     // [d_in x d_in] scaled rows U_jk / U_jj, fp16 hi
    uint16_t* Ul;     //                                        fp16 lo
    float* rowloss;   // [d_out]
    uint16_t *Fh, *Fl;   // panel kernel: residual fragments, [workgroups][3 x 8 x 2 x 64 x 8]
    uint16_t *Bh, *Bl;   // panel kernel: fragments of the normalized U blocks, [super-blocks][6 x 8 x 4 x 64 x 8]
    Scalars* sc;
    uint8_t* Qs;         // [d_out x d_in] codes in sweep order (used under a column order)
    int32_t* inv;        // [d_in] inverse of the column order
    float* W0p;          // [d_out x d_in] the weights gathered into sweep order (used under a column order)
    double* s64;         // [d_out] fp64 scale of the wide group being swept
};

constexpr size_t F_PER_WG = size_t(3) * 8 * 2 * 64 * 8 * 2;    // bytes of Fh (or Fl) per workgroup of the panel kernel
constexpr size_t B_PER_SB = size_t(6) * 8 * 4 * 64 * 8 * 2;    // bytes of Bh (or Bl) per super-block

// leading dimension of the transposed residual panels: whole 64-row workgroups of the panel kernel
inline int64_t ld_d(int64_t d_out) { return ceil_div(d_out, ROWS) * ROWS; }

SweepWs carve(void* ws, int64_t d_out, int64_t d_in) {
    char* p = static_cast<char*>(ws);
    SweepWs w;
    w.Wf = reinterpret_cast<float*>(p); p += align_up(size_t(d_out) * d_in * sizeof(float), 256);   // feedback sums c
    w.Dh = reinterpret_cast<uint16_t*>(p); p += 2 * size_t(SBIG) * ld_d(d_out) * 2;
    w.Dl = reinterpret_cast<uint16_t*>(p); p += 2 * size_t(SBIG) * ld_d(d_out) * 2;
    w.Uh = reinterpret_cast<uint16_t*>(p); p += align_up(size_t(d_in) * d_in * 2, 256);
    w.Ul = reinterpret_cast<uint16_t*>(p); p += align_up(size_t(d_in) * d_in * 2, 256);
    w.rowloss = reinterpret_cast<float*>(p); p += align_up(size_t(d_out) * sizeof(float), 256);
    const size_t fb = size_t(ceil_div(d_out, ROWS)) * F_PER_WG, bb = size_t(ceil_div(d_in, SBIG)) * B_PER_SB;
    w.Fh = reinterpret_cast<uint16_t*>(p); p += fb;
    w.Fl = reinterpret_cast<uint16_t*>(p); p += fb;
    w.Bh = reinterpret_cast<uint16_t*>(p); p += bb;
    w.Bl = reinterpret_cast<uint16_t*>(p); p += bb;
    w.sc = reinterpret_cast<Scalars*>(p); p += 256;
    w.Qs = reinterpret_cast<uint8_t*>(p); p += align_up(size_t(d_out) * d_in, 256);
    w.inv = reinterpret_cast<int32_t*>(p); p += align_up(size_t(d_in) * sizeof(int32_t), 256);
    w.W0p = reinterpret_cast<float*>(p); p += align_up(size_t(d_out) * d_in * sizeof(float), 256);
    w.s64 = reinterpret_cast<double*>(p);
    return w;
}

// fills in t's work map; returns the number of workgroups
template <typename S, TrailMode MODE>
int trail_grid(TrailArgs& t) {
    t.n_mt = int(ceil_div(t.d_out, S::TM));
    if (MODE == INCREMENT) {
        t.n_nt = int(ceil_div(t.c1 - t.c0, S::TN));
    } else {
        t.n_nt0 = t.h0 > t.c0 ? int(ceil_div(t.h0 - t.c0, S::TN)) : 0;
        t.n_nt = t.n_nt0 + (t.c1 > t.h1 ? int(ceil_div(t.c1 - t.h1, S::TN)) : 0);
    }
    t.chunk = int(ceil_div(int64_t(t.n_mt) * t.n_nt, 8));
    return t.chunk * 8;
}
template <typename S, TrailMode MODE>
onecomp_status launch_trailing_shape(TrailArgs t, hipStream_t stream) {
    static std::atomic<uint64_t> lds_ok{0};
    if (allow_dynamic_lds(reinterpret_cast<const void*>(&trailing_kernel<S, MODE>), int(S::LDS_BYTES), lds_ok) != ONECOMP_OK)
        return ONECOMP_ERR_HIP;
    const int wgs = trail_grid<S, MODE>(t);
    // Triangular products whose tiles are all resident at once, two on a CU: the shortest join the longest (4096 x 4096, us of the
    // corrected target, 512 tiles, longest first all the way : folded 1072 : 1023; with more tiles 4096 x 8192 3417 : 3437, 14336 x
    // 4096 2982 : 3019).
    const int total = t.n_mt * t.n_nt, cus = device_cus();
    t.fold = total > cus && total <= 2 * cus ? cus : total;
    hipLaunchKernelGGL((trailing_kernel<S, MODE>), dim3(unsigned(wgs)), dim3(256), S::LDS_BYTES, stream, t);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}
// The 128 x 256 tiles move half the operand bytes per flop, but a launch of few of them is as long as one tile on a CU of its
// own.  us of a launch, 128 x 256 : 64 x 128 tiles, d_out 4096 (64 of the former), 512 columns: K 512 22.6 : 13.9, K 128 13 :
// 7.5; d_out 8192 (128 tiles), 512 columns, K 512 32.0 : 26.6.  Whole sweep, 4096 columns, d_out 10240 (160 tiles) 1193 : 1193,
// 14336 (224) 1441 : 1457.
template <TrailMode MODE>
onecomp_status launch_trailing(TrailArgs t, hipStream_t stream) {
    return 2 * trail_grid<TrailBig, MODE>(t) <= device_cus() ? launch_trailing_shape<TrailSmall, MODE>(t, stream)
                                                             : launch_trailing_shape<TrailBig, MODE>(t, stream);
}

template <int GB, bool DIRECT, int ROWS_WG>
onecomp_status launch_panel_rows(const PanelArgs& pa, const TrailArgs& ta, int far_wgs, hipStream_t stream) {
    static std::atomic<uint64_t> lds_ok{0};
    // (both bodies share the launch with tiles of the far update)
    constexpr int own = ROWS_WG == ROWS ? panel_lds(DIRECT) : panel16_lds(DIRECT);
    constexpr int lds = own > int(TrailBig::LDS_BYTES) ? own : int(TrailBig::LDS_BYTES);
    if (allow_dynamic_lds(reinterpret_cast<const void*>(&panel_far_kernel<GB, DIRECT, ROWS_WG>), lds, lds_ok) != ONECOMP_OK)
        return ONECOMP_ERR_HIP;
    const int n_panel = int(ceil_div(pa.d_out, ROWS_WG));
    hipLaunchKernelGGL((panel_far_kernel<GB, DIRECT, ROWS_WG>), dim3(unsigned(n_panel + far_wgs)), dim3(256), lds, stream, pa, ta,
                       n_panel);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}
// 16 rows per workgroup where they all fit on the CUs at once, two on each, and the launch's far tiles add little behind them:
// more rows per workgroup are less work in all, and a launch of many tiles is as long as its work.  us of a whole sweep, 64 : 16
// rows, 4096 columns, group 128: d_out 256 (512 columns) 99 : 74, 1024 732 : 523, 4096 825 : 677, 5120 879 : 779, 7168 986 : 945,
// 8192 1068 : 1051 (up to 256 far tiles; all launches 1106), 9600 1154 : 1209 (panels three deep), 14336 1373 : 1719.  4096 x
// 14336, inverse form, 64 rows 4335; 16 rows up to 256, 512, 768, 1024 and any number of far tiles 4180, 4086, 4074, 4132, 4338.
template <int GB, bool DIRECT>
onecomp_status launch_panel(const PanelArgs& pa, const TrailArgs& ta, int far_wgs, hipStream_t stream) {
    const int64_t n16 = ceil_div(pa.d_out, ROWS16), cus = device_cus();
    const bool searched = pa.mse && pa.wide_g < 0;
    return !searched && n16 <= 2 * cus && 2 * n16 + far_wgs <= 5 * cus
               ? launch_panel_rows<GB, DIRECT, ROWS16>(pa, ta, far_wgs, stream)
               : launch_panel_rows<GB, DIRECT, ROWS>(pa, ta, far_wgs, stream);
}

}  // namespace

size_t sweep_workspace_bytes(int64_t d_out, int64_t d_in, int block) {
    (void)block;
    return align_up(size_t(d_out) * d_in * sizeof(float), 256) + 4 * size_t(SBIG) * ld_d(d_out) * 2 +
           2 * align_up(size_t(d_in) * d_in * 2, 256) + align_up(size_t(d_out) * sizeof(float), 256) +
           2 * size_t(ceil_div(d_out, ROWS)) * F_PER_WG + 2 * size_t(ceil_div(d_in, SBIG)) * B_PER_SB + 256 +
           align_up(size_t(d_out) * d_in, 256) + align_up(size_t(d_in) * sizeof(int32_t), 256) +
           align_up(size_t(d_out) * d_in * sizeof(float), 256) + align_up(size_t(d_out) * sizeof(double), 256);
}

// C[:, c0 .. c1) += f_inv * (D[ek .. ek + K, :])^T * B[u0 .. u0 + K, c0 .. c1): the split-fp16 product of the sweep's
// trailing update, for other callers (see the declaration).
onecomp_status split_update(float* C, int64_t d_out, int64_t d_in, const uint16_t* Dh, const uint16_t* Dl, int64_t ldD,
                            const uint16_t* Bh, const uint16_t* Bl, const Scalars* sc, int ek, int K, int u0, int c0,
                            int c1, hipStream_t stream) {
    return split_update_around(C, d_out, d_in, Dh, Dl, ldD, Bh, Bl, sc, ek, K, u0, c0, c1, c1, c1, stream);
}

onecomp_status split_update_around(float* C, int64_t d_out, int64_t d_in, const uint16_t* Dh, const uint16_t* Dl,
                                   int64_t ldD, const uint16_t* Bh, const uint16_t* Bl, const Scalars* sc, int ek, int K,
                                   int u0, int c0, int h0, int h1, int c1, hipStream_t stream) {
    if ((h0 <= c0 && c1 <= h1) || K <= 0) return ONECOMP_OK;
    TrailArgs t;
    t.Wf = C; t.Dh = Dh; t.Dl = Dl; t.Uh = Bh; t.Ul = Bl; t.sc = sc;
    t.d_out = int(d_out); t.ldD = int(ldD); t.d_in = int(d_in);
    t.ek = ek; t.K = K; t.u0 = u0; t.c0 = c0; t.c1 = c1;
    t.h0 = h0; t.h1 = h1; t.first = 0; t.tri = TRI_NONE; t.max_bits = nullptr;
    return launch_trailing<SUM>(t, stream);
}

onecomp_status split_product(float* C, int64_t d_out, int64_t d_in, const uint16_t* Dh, const uint16_t* Dl, int64_t ldD,
                             const uint16_t* Bh, const uint16_t* Bl, const Scalars* sc, int K, Triangle tri, uint32_t* max_bits,
                             hipStream_t stream) {
    TrailArgs t;
    t.Wf = C; t.Dh = Dh; t.Dl = Dl; t.Uh = Bh; t.Ul = Bl; t.sc = sc;
    t.d_out = int(d_out); t.ldD = int(ldD); t.d_in = int(d_in);
    t.ek = 0; t.K = K; t.u0 = 0; t.c0 = 0; t.c1 = int(d_in);
    t.h0 = t.h1 = t.c1; t.first = 1; t.tri = tri; t.fold = 0; t.max_bits = max_bits;
    // Tiles of different lengths even out better the smaller they are: up to one 128 x 256 tile per CU 64 x 128 ones are the faster.
    // us of the corrected target, 128 x 256 : 64 x 128 tiles (number of the former): 2048 x 2048 (128) 298 : 253, 1500 x 4096 (192)
    // 569 : 520, 2048 x 4096 (256) 650 : 635, 2500 x 4096 (320) 790 : 792, 3072 x 4096 (384) 824 : 855, 14336 x 4096 2982 : 3334.
    if (tri != TRI_NONE && trail_grid<TrailBig, PRODUCT>(t) <= device_cus()) return launch_trailing_shape<TrailSmall, PRODUCT>(t, stream);
    return launch_trailing<PRODUCT>(t, stream);
}

int64_t split_update_ld(int64_t d_out) { return ld_d(d_out); }

onecomp_status sweep_run(const void* W, onecomp_dtype w_dtype, int64_t d_out, int64_t d_in, const float* U,
                         int form, const int32_t* perm, int bits, int group_size, int block, int grid, uint8_t* Q,
                         float* scales, float* zeros, float* W_hat, float* loss, void* workspace, hipStream_t stream) {
    (void)block;
    const bool direct = form == ONECOMP_FACTOR_BLOCK;   // block form of the factor: see panel_body
    // Wide groups whose parameters can be fixed before the sweep enters them: one group per row (its values are the
    // original weights), or groups made of whole super-blocks (all earlier feedback has reached the working copy
    // once the previous super-block's far update is complete).  These run through the panel kernel.
    const bool wide_static = group_size > SB;
    // super-block width: 512 columns, or for wide groups the largest of 512 / 384 / 256 / 128 that divides the group,
    // so that a group is a run of whole super-blocks
    const int sbw = plan::sweep_superblock_width(group_size, d_in);
    const int sb_pairs = (sbw / SB) * (sbw / SB - 1) / 2;   // block pairs (b' < b) inside a super-block
    if (direct && group_size > SB && group_size != d_in) return ONECOMP_ERR_UNSUPPORTED;
    SweepWs w = carve(workspace, d_out, d_in);
    const int n_u = int(d_in < PREP_WGS ? d_in : PREP_WGS), n_w = int(d_out < PREP_WGS ? d_out : PREP_WGS);
    float *const max_u = reinterpret_cast<float*>(w.Dh), *const max_w = max_u + PREP_WGS;   // the panels write Dh later
    auto prepare = [&](auto* W_) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(W_)>>;
        hipLaunchKernelGGL(prepare_kernel<T>, dim3(unsigned(n_u + n_w)), dim3(256), 0, stream, U, int(d_in), n_u, max_u, W_, d_out,
                           perm, w.rowloss, max_w, w.W0p);
    };
    if (w_dtype == ONECOMP_BF16) prepare(static_cast<const uint16_t*>(W));
    else prepare(static_cast<const float*>(W));
    ONECOMP_CHECK_LAUNCH();
    const int n_near = NEAR_PARTS * sb_pairs * int(ceil_div(d_in, sbw));
    hipLaunchKernelGGL(operands_kernel, dim3(unsigned(n_near + (d_in < 2048 ? d_in : 2048))), dim3(256), 0, stream, U, int(d_in), max_u,
                       n_u, max_w, n_w, w.sc, w.Bh, w.Bl, sbw, sb_pairs, n_near, w.Uh, w.Ul);
    ONECOMP_CHECK_LAUNCH();

    TrailArgs t;
    t.Wf = w.Wf; t.Dh = w.Dh; t.Dl = w.Dl; t.Uh = w.Uh; t.Ul = w.Ul; t.sc = w.sc;
    t.ek = 0; t.K = 0; t.u0 = 0; t.c0 = 0; t.c1 = 0; t.n_nt = 0; t.chunk = 0;
    t.d_out = int(d_out); t.ldD = int(ld_d(d_out)); t.d_in = int(d_in);
    t.n_nt0 = 0; t.h0 = 0; t.h1 = 0; t.first = 0; t.tri = TRI_NONE; t.fold = 0; t.max_bits = nullptr;
    // fills t for Wf[:, c0 .. c1) += residual columns ek .. ek+K of buffer `buf` times rows u0 .. u0+K of Un;
    // returns the number of workgroups (0: nothing to do)
    const size_t d_buf = size_t(SBIG) * ld_d(d_out);
    auto set_trailing = [&](int buf, int ek, int K, int u0, int c0, int c1) -> int {
        if (c1 <= c0) return 0;
        t.Dh = w.Dh + buf * d_buf; t.Dl = w.Dl + buf * d_buf;
        t.ek = ek; t.K = K; t.u0 = u0; t.c0 = c0; t.c1 = c1;
        t.first = u0 == 0;   // the first super-block's feedback is the first there is
        return trail_grid<TrailBig, INCREMENT>(t);
    };
    auto trailing = [&](int buf, int ek, int K, int u0, int c0, int c1) -> onecomp_status {
        return set_trailing(buf, ek, K, u0, c0, c1) == 0 ? ONECOMP_OK : launch_trailing<INCREMENT>(t, stream);
    };

    onecomp_status st;
    {
        // Groups no wider than a block: one launch sweeps a super-block of 512 columns (the feedback between its
        // blocks is applied inside the panel kernel).  The columns beyond a super-block receive its feedback once,
        // with K = its width: first those of the next super-block, then, in the same launch as the next panel,
        // the rest.
        PanelArgs pa;
        pa.Wf = w.Wf; pa.U = U;
        // where the panel finds the original weights in sweep order: under a column order, the gathered fp32 copy
        pa.W0 = perm ? static_cast<const void*>(w.W0p) : W;
        pa.w0_bf16 = !perm && w_dtype == ONECOMP_BF16;
        pa.s64 = w.s64; pa.sat = sat_flag(w.sc);
        pa.Q = perm ? w.Qs : Q; pa.scales = scales; pa.zeros = zeros; pa.W_hat = perm ? nullptr : W_hat;
        pa.Fh = w.Fh; pa.Fl = w.Fl; pa.sc = w.sc; pa.rowloss = w.rowloss;
        pa.d_out = int(d_out); pa.d_in = int(d_in); pa.n_g = int(d_in / group_size); pa.ldD = int(ld_d(d_out));
        pa.lgG = 0;
        while ((1 << pa.lgG) < group_size) ++pa.lgG;
        if (wide_static) pa.lgG = 7;
        pa.wide_g = -1;
        const bool symmetric = grid == ONECOMP_GRID_SYMMETRIC || grid == ONECOMP_GRID_SYMMETRIC_MSE;
        pa.mse = grid == ONECOMP_GRID_MINMAX_MSE || grid == ONECOMP_GRID_SYMMETRIC_MSE;
        pa.qs = symmetric ? float((1 << (bits - 1)) - 1) : 0.f;
        pa.qmax = symmetric ? 2.f * pa.qs : float((1 << bits) - 1);
        int buf = 0, p0 = 0, p1 = 0;   // previous super-block: residual buffer and column range
        for (int s0 = 0; s0 < d_in; s0 += sbw) {
            const int s1 = int(d_in < int64_t(s0) + sbw ? d_in : int64_t(s0) + sbw);
            int far_wgs = 0;
            const bool group_start = wide_static && s0 % group_size == 0;
            if (s0 > 0 && group_start) {   // every later column must be current before the group's range is taken
                if ((st = trailing(buf ^ 1, 0, p1 - p0, p0, s0, int(d_in))) != ONECOMP_OK) return st;
            } else if (s0 > 0) {
                if ((st = trailing(buf ^ 1, 0, p1 - p0, p0, s0, s1)) != ONECOMP_OK) return st;
                far_wgs = set_trailing(buf ^ 1, 0, p1 - p0, p0, s1, int(d_in));
            }
            if (group_start) {
                const dim3 pgrid{unsigned(d_out < 2048 ? d_out : 2048)};
                const int g_idx = s0 / group_size;
                // the feedback of the earlier columns (none before the first group; the block form only takes one
                // group per row, whose grid comes from the original weights)
                const float* cur = (direct || s0 == 0) ? nullptr : w.Wf;
                auto params = [&](auto kernel, auto* W0) {
                    hipLaunchKernelGGL(kernel, pgrid, dim3(gp_threads(pa.mse)), 0, stream, W0, cur, int(d_out), int(d_in), s0,
                                       group_size, pa.qmax, pa.qs, pa.n_g, g_idx, scales, zeros, w.s64);
                };
                if (pa.w0_bf16) {
                    const uint16_t* W0 = static_cast<const uint16_t*>(pa.W0);
                    if (pa.mse) params(group_params_kernel<uint16_t, true>, W0);
                    else params(group_params_kernel<uint16_t, false>, W0);
                } else {
                    const float* W0 = static_cast<const float*>(pa.W0);
                    if (pa.mse) params(group_params_kernel<float, true>, W0);
                    else params(group_params_kernel<float, false>, W0);
                }
                ONECOMP_CHECK_LAUNCH();
            }
            if (wide_static) pa.wide_g = s0 / group_size;
            pa.s0 = s0; pa.nb = (s1 - s0) / SB;
            pa.Dh = w.Dh + buf * d_buf; pa.Dl = w.Dl + buf * d_buf;
            pa.Bh = w.Bh + size_t(s0 / sbw) * sb_pairs * (8 * 4 * 64 * 8);
            pa.Bl = w.Bl + size_t(s0 / sbw) * sb_pairs * (8 * 4 * 64 * 8);
            if (group_size == 16 && direct) st = launch_panel<16, true>(pa, t, far_wgs, stream);
            else if (group_size == 16) st = launch_panel<16, false>(pa, t, far_wgs, stream);
            else if (direct) st = launch_panel<32, true>(pa, t, far_wgs, stream);
            else st = launch_panel<32, false>(pa, t, far_wgs, stream);
            if (st != ONECOMP_OK) return st;
            buf ^= 1; p0 = s0; p1 = s1;
        }
    }
    if (perm) {
        hipLaunchKernelGGL(inv_perm_kernel, dim3(unsigned(ceil_div(d_in, 256))), dim3(256), 0, stream, perm, int(d_in),
                           w.inv);
        ONECOMP_CHECK_LAUNCH();
        hipLaunchKernelGGL(unpermute_kernel, dim3(unsigned(ceil_div(d_in, 1024)), unsigned(d_out < 4096 ? d_out : 4096)),
                           dim3(256), 0, stream, w.Qs, scales, zeros, w.inv, int(d_out), int(d_in), group_size,
                           int(d_in / group_size), Q, W_hat);
        ONECOMP_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(loss_kernel, dim3(1), dim3(1024), 0, stream, w.rowloss, int(d_out), sat_flag(w.sc), loss);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

}  // namespace onecomp
