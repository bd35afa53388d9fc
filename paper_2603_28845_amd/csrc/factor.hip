// Damping, activation ordering and the Cholesky-based inverse factor (Sec. 4.3.1 of the paper:
// lambda = eta * mean(diag H), Cholesky of H + lambda I; Sec. 4.3: optional "actorder").
//
// Wanted: upper-triangular U, positive diagonal, U^T U = Hd^-1 for the damped (permuted) matrix Hd.
// Route: let R be Hd with both index orders reversed, R = L L^T its lower Cholesky factor and
// V = L^-1.  Reversing a lower-triangular matrix gives an upper-triangular one, so
// Hd = M M^T with M = rev(L) upper, and U = M^-1 = rev(V):  U[i][k] = V[n-1-i][n-1-k].
// One Cholesky plus one triangular inverse (2 n^3 / 3 flops), all in fp64; U is rounded once to fp32.
//
// gfx950 design
//   * blocked right-looking Cholesky, block 128: diagonal block factored (and its halves inverted) inside one
//     workgroup's LDS; panel solve and trailing update are fp64 MFMA GEMMs (v_mfma_f64_16x16x4_f64),
//     128 x 128 or 128 x 64 tile per workgroup, operands streamed global -> LDS directly through a ring of slots; a launch
//     has one workgroup per tile that has work, the longest tiles first.
//   * triangular inverse of narrow factors: row by row beside the trailing updates;
//     of wider ones by recursive doubling over aligned block pairs: for block size s = 128 * 2^l,
//     V[C,A] = -V[C,C] (L[C,A] V[A,A]); every level is two batched GEMMs, so the whole inverse is
//     ~2 log2(n/128) large launches instead of n/128 skinny ones.
//   * wide factors (factor_slabs): left-looking over slabs of columns, whose updates, and the inverse's long products, are
//     taken from 8-bit residues on the integer matrix cores (residue.hip), rounded against the norms of rows and columns as
//     little as in fp64 (an entry's own size does not count: residue.hip).
//   * ordering by rank counting (stable, deterministic), no floating-point atomics anywhere.
#include "common.hpp"
#include "planner.hpp"
#include "residue.hpp"
#include <type_traits>

namespace onecomp {
namespace {

constexpr int NB = 128;  // block size of the factorization (= GEMM tile side)

// ------------------------------------------------------------------------------------------
// small preparation kernels
// ------------------------------------------------------------------------------------------
// diag -> keys (original diagonal), dfix (dead channels -> 1), lambda = damp * mean(dfix); natural: the identity into perm_out.  One
// workgroup: every entry is a line and a page of its own, so a thread has eight of them on the way.
__global__ __launch_bounds__(1024) void prep_diag_kernel(const float* __restrict__ H, int n, double damp,
                                                        float* __restrict__ keys, double* __restrict__ dfix,
                                                        double* __restrict__ lam, int32_t* __restrict__ info,
                                                        int natural, int32_t* __restrict__ perm_out) {
    __shared__ double part[1024];
    double s = 0.0;
    for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 1024) {
        float h[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) h[q] = i0 + 1024 * q < n ? H[int64_t(i0 + 1024 * q) * (n + 1)] : 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = i0 + 1024 * q;
            if (i >= n) break;
            keys[i] = h[q] == h[q] ? h[q] : -__builtin_inff();   // a NaN goes last: every position of the order is taken once
            const double d = (h[q] == 0.0f) ? 1.0 : double(h[q]);
            dfix[i] = d;
            s += d;  // fixed order per thread
            if (natural && perm_out) perm_out[i] = i;
        }
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w >= 64; w >>= 1) {
        if (threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 64) {
        s = part[threadIdx.x];
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) s += __shfl_down(s, w, 64);
        if (threadIdx.x == 0) {
            *lam = damp * (s / double(n));
            *info = 0;
        }
    }
}

// perm: stable descending order of keys.  rank by counting: n^2 comparisons, two operations each.
// A lane owns a key and the 16 waves of a workgroup share out the keys it is compared with, which arrive as scalar
// loads; a thread per key that walked through all of them left the chip to 56 workgroups at d_in 14336 and waited for
// one load after the other: 805 -> 26 us.
constexpr int ORDER_KEYS = 64, ORDER_WAVES = 16;
__global__ __launch_bounds__(64 * ORDER_WAVES) void order_kernel(const float* __restrict__ keys, int n,
                                                                int32_t* __restrict__ perm,
                                                                int32_t* __restrict__ perm_out) {
    __shared__ int part[ORDER_WAVES][ORDER_KEYS];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i0 = blockIdx.x * ORDER_KEYS, i = i0 + lane;
    const float ki = keys[min(i, n - 1)];
    const int each = (n + ORDER_WAVES - 1) / ORDER_WAVES;
    const int k0 = min(wave * each, n), k1 = min(k0 + each, n);
    const int b0 = max(k0, min(k1, i0)), b1 = max(k0, min(k1, i0 + ORDER_KEYS));   // this workgroup's own keys
    int rank = 0;
#pragma unroll 16
    for (int k = k0; k < b0; ++k) rank += keys[k] >= ki;
    for (int k = b0; k < b1; ++k) rank += (keys[k] > ki) || (keys[k] == ki && k < i);
#pragma unroll 16
    for (int k = b1; k < k1; ++k) rank += keys[k] > ki;
    part[wave][lane] = rank;
    __syncthreads();
    if (wave != 0 || i >= n) return;
    int pos = 0;
    for (int w = 0; w < ORDER_WAVES; ++w) pos += part[w][lane];
    perm[pos] = i;
    if (perm_out) perm_out[pos] = i;
}

// A[r][c] = Hd[p[n-1-r]][p[n-1-c]] in fp64 (reversed, permuted, damped); upper triangle of H is read.  Only the
// 128 x 128 blocks on and below the diagonal are written: the factorization never reads the others, and in natural
// order (this kernel) those are the ones whose source rows are read along the row.  Also: V's zeros above the diagonal
// of its diagonal blocks, and the copy of block (1, 0) that the first panel solve takes (panel_kernel).
__global__ __launch_bounds__(256) void build_kernel(const float* __restrict__ H, int n,
                                                   const double* __restrict__ dfix, const double* __restrict__ lam,
                                                   double* __restrict__ A, double* __restrict__ V,
                                                   double* __restrict__ Pn) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int r = blockIdx.y;
    if (c >= n || c / NB > r / NB) return;
    const int i = n - 1 - r, k = n - 1 - c;
    double v;
    if (i == k) v = dfix[i] + *lam;
    else v = double(H[int64_t(min(i, k)) * n + max(i, k)]);
    A[int64_t(r) * n + c] = v;
    if (c > r) V[int64_t(r) * n + c] = 0.0;
    if (c < NB && r / NB == 1) Pn[(r - NB) * NB + c] = v;
}

// The same under a column order.  H's upper triangle then comes in at scattered places, half of them along columns: 64
// bytes fetched for 4.  So the triangle is mirrored into a full matrix S first, 64 x 64 tiles at a time, and every row
// of A takes its values from one row of S, read along the row into LDS and gathered there.  d_in 14336: 1362 us in one
// pass of gathers -> 257 + 405 us in the two.
__global__ __launch_bounds__(256) void mirror_kernel(const float* __restrict__ H, int n, float* __restrict__ S) {
    __shared__ float tile[64][65];
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    if (c0 < r0) return;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = r0 + ty + 4 * q, c = c0 + tx;
        float v = 0.f;
        if (r < n && c < n && r <= c) v = H[int64_t(r) * n + c];
        tile[ty + 4 * q][tx] = v;
        if (r < n && c < n && r <= c) S[int64_t(r) * n + c] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = c0 + ty + 4 * q, c = r0 + tx;   // below the diagonal
        if (r < n && c < r) S[int64_t(r) * n + c] = tile[tx][ty + 4 * q];
    }
}

constexpr int GATHER_COLS = 16384;   // columns of S in LDS at a time: two workgroups per CU
__global__ __launch_bounds__(512) void build_order_kernel(const float* __restrict__ S, int n,
                                                         const int32_t* __restrict__ perm,
                                                         const double* __restrict__ dfix,
                                                         const double* __restrict__ lam, double* __restrict__ A,
                                                         double* __restrict__ V, double* __restrict__ Pn) {
    extern __shared__ float srow[];
    const int r = n - 1 - int(blockIdx.x);   // the longest rows first
    const int i = perm[n - 1 - r];
    const int c_end = min(n, (r / NB + 1) * NB);
    for (int b = 0; b < n; b += GATHER_COLS) {
        const int cols = min(GATHER_COLS, n - b);
        const float* src = S + int64_t(i) * n + b;
        if (b > 0) __syncthreads();
        if (n % 4 == 0) {
            for (int c = threadIdx.x * 4; c < cols; c += 512 * 4)
                *reinterpret_cast<float4v*>(srow + c) = *reinterpret_cast<const float4v*>(src + c);
        } else {
            for (int c = threadIdx.x; c < cols; c += 512) srow[c] = src[c];
        }
        __syncthreads();
        for (int c = threadIdx.x; c < c_end; c += 512) {
            const int k = perm[n - 1 - c];
            if (unsigned(k - b) >= unsigned(cols)) continue;
            const double v = k == i ? dfix[i] + *lam : double(srow[k - b]);
            A[int64_t(r) * n + c] = v;
            if (c > r) V[int64_t(r) * n + c] = 0.0;
            if (c < NB && r / NB == 1) Pn[(r - NB) * NB + c] = v;
        }
    }
}

// U[i][k] = float(V[n-1-i][n-1-k]) for k >= i, 0 below the diagonal.
__global__ __launch_bounds__(256) void output_kernel(const double* __restrict__ V, int n, float* __restrict__ U) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int i = blockIdx.y;
    if (k >= n) return;
    float u = 0.f;
    if (k >= i) u = float(V[int64_t(n - 1 - i) * n + (n - 1 - k)]);
    U[int64_t(i) * n + k] = u;
}

// Block form (no triangular inverse of the whole factor).  With R = U^-1, i.e. R[i][k] = L[n-1-i][n-1-k] and
// Hd = R R^T:  F = U on the NB x NB diagonal blocks (the index-reversed inverses of the diagonal blocks of L, which
// the factorization leaves in V);  F[i][k] = -U_ii R_ik / R_kk where i and k lie in different blocks.
// rdiag[r] = 1 / L[r][r] = V[r][r].
__global__ __launch_bounds__(256) void rdiag_kernel(const double* __restrict__ V, int n, double* __restrict__ rdiag) {
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < n) rdiag[r] = V[int64_t(r) * n + r];
}

__global__ __launch_bounds__(256) void output_block_kernel(const double* __restrict__ L, const double* __restrict__ V,
                                                          const double* __restrict__ rdiag, int n,
                                                          float* __restrict__ F) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int i = blockIdx.y;
    if (k >= n) return;
    float f = 0.f;
    if (k >= i) {
        const int ri = n - 1 - i, rk = n - 1 - k;   // ri >= rk
        if (ri / NB == rk / NB) f = float(V[int64_t(ri) * n + rk]);
        else f = float(-(rdiag[ri] * rdiag[rk]) * L[int64_t(ri) * n + rk]);
    }
    F[int64_t(i) * n + k] = f;
}

// ------------------------------------------------------------------------------------------
// diagonal block: Cholesky and the inverses of its two 64 x 64 diagonal halves.  One workgroup of 512 threads (8 waves).
// A block (bs x bs, bs <= 128) at A + off*(n+1).  The inverses of the halves of L_kk and the quarter of L_kk between them go
// to Pk, sub-block by sub-block in the order in which the panel solve's MFMAs take them; nothing else leaves the
// workgroup.  A non-positive pivot sets *info (first one wins) and is replaced by 1.
//
// The block is 36 sub-blocks of 16 x 16 (on and below the diagonal); finished ones live in LDS (row pitch 17 doubles,
// 76.5 KB: small enough for two workgroups per CU, so the factorization can share a launch with GEMM tiles), those that
// still take updates in the accumulators of the wave that owns their row.  Everything but the 16 x 16 leaves runs on
// v_mfma_f64_16x16x4_f64 with sub-blocks as operands.  The whole is a chain of latencies on one CU, exposed in every step
// with a short trailing update (d_in 4096: all of them), so what counts is what stands between two pivots:
//   wave 0: the leaf of (J,J) in registers, which leaves T = L_JJ^-1; from T, still in the registers in operand layout,
//     L_J+1,J = A_J+1,J T^T and A_J+1,J+1 -= L L^T (computed transposed, so that one product's result is the next one's
//     operand), then the next leaf.
//   waves 1-3 and 5-7 (SIMDs 1-3, two waves each to cover each other's waits): L_IJ = A_IJ T^T for I > J + 1 while wave 0
//     does its two products, then, beside the next leaf, A_IK -= L_IJ L_KJ^T for the next two columns, and on three of them a
//     column each of the halves' inverses, X_J = -T_J P_J, P_J+1 = sum_K L_J+1,K X_K.
//   wave 4 (SIMD 0, next to the leaves): sends what is finished to memory.
// Before: the inverse of the whole 128-wide block here, all products on four waves and through LDS, the trailing update of
// the block in front of it in the same workgroup: 37 us a launch, now 14.
// MFMA operand layouts (lane l): A[i][k]: i = l % 16, k = l / 16;  B[k][j]: k = l / 16, j = l % 16;
// C/D register r: row 4 r + l / 16, column l % 16.
// ------------------------------------------------------------------------------------------
constexpr int SBW = 16;      // sub-block width
constexpr int SBP = SBW + 1;
constexpr int SBS = SBW * SBP;
constexpr int NSB = NB / SBW;
constexpr int HALF = NB / 2;   // the block's diagonal is inverted in halves
constexpr int POTRF_THREADS = 512;
constexpr int POTRF_LDS_DOUBLES = NSB * (NSB + 1) / 2 * SBS;   // the lower sub-blocks
__device__ __forceinline__ int sub(int I, int J) { return ((I * (I + 1)) / 2 + J) * SBS; }   // J <= I

// 1 / sqrt(p): v_rsq_f64 is good to 5e-8 relative (measured over 120 binades), the first Newton step brings it to 4e-15,
// the second to rounding.
__device__ inline double rsqrt_refined(double p) {
    double y = __builtin_amdgcn_rsq(p);
    const double h = 0.5 * p;
    y = y * __builtin_fma(-h * y, y, 1.5);
    y = y * __builtin_fma(-h * y, y, 1.5);
    return y;
}

// DPP row_newbcast:J (lane J of every 16-lane row) is the one DPP form of 64-bit instructions; hipcc's builtin offers it
// for 32 bits only, which costs two moves per broadcast instead of none.  A DPP operand must not have been written by
// the two instructions before: the compiler does not look into these statements, so the broadcast keeps that distance
// itself (s_nop 1), and they are volatile, that is, stay in order.  The update relies on its operand being older and on
// the compiler placing no copy of it right in front, which tests/test_factor_isa.py checks in the generated code.
// c += (lane J of b) * m; b does not come from the two instructions before
template <int J>
__device__ __forceinline__ void fma_bcast16(double& c, double b, double m) {
    asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(c) : "v"(b), "v"(m), "n"(J));
}
// value of lane J of every 16-lane row, in all lanes of the row
template <int J>
__device__ __forceinline__ double bcast16(double v) {
    double o;
    asm volatile("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf"
                 : "=v"(o) : "v"(v), "n"(J));
    return o;
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// where the operand fragments of sub-block (I, J) begin in Pk
__device__ __forceinline__ int packed(int I, int J) { return (I * (I + 1) / 2 + J) * (SBW * SBW); }

// The leaf of potrf_body again, on the sub-block D in LDS, where a pivot was not positive: every such pivot is replaced by 1
// and the first one of the factorization left in *info.  Returns D_i, and Z = Lh^-1 in x.  Columns are scaled by the refined
// reciprocal as there, not divided: an infinite pivot leaves NaN, and so a pivot that is reported, by either.
__device__ __forceinline__ double leaf_with_bad_pivots(double* D, int i, int lk, double (&x)[4], int32_t* info, int row0) {
    double my_d = 1.0;
    int bad_at = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = (4 * k + lk == i) ? 1.0 : 0.0;
#pragma unroll 1
    for (int j = 0; j < SBW; ++j) {
        double p = D[j * SBP + j];
        if (!(p > 0.0)) {
            if (bad_at < 0) bad_at = j;
            p = 1.0;
        }
        if (i == j) my_d = p;
        const double y = __builtin_amdgcn_rcp(p), t = -(D[i * SBP + j] * y);
        const double nm = i > j ? __builtin_fma(t, __builtin_fma(-p, y, 1.0), t) : 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = 4 * k + lk;
            if (c > j) D[i * SBP + c] = __builtin_fma(D[c * SBP + j], nm, D[i * SBP + c]);
            x[k] = __builtin_fma(__shfl(x[k], j, SBW), nm, x[k]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the other lanes' entries
    }
    if (bad_at >= 0 && i == 0 && lk == 0 && *info == 0) *info = row0 + bad_at + 1;
    return my_d;
}

// S: POTRF_LDS_DOUBLES doubles of LDS
__device__ __forceinline__ void potrf_body(const double* __restrict__ A, double* __restrict__ Pk, int n, int off, int bs,
                                           int32_t* __restrict__ info, double* S) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lk = lane >> 4;
    const double* __restrict__ const Ab = A + int64_t(off) * (n + 1);
    // operand fragments of a sub-block M (pointer to its first element), k-step q = 0..3
    auto frag_rowk = [&](const double* M, int q) __attribute__((always_inline)) {   // M[l%16][4q + l/16]
        return M[l16 * SBP + 4 * q + lk];
    };
    // M[4 r + l/16][l%16], r = 0..3: the accumulator layout and, register r for k-step r, also that of a B operand
    auto load_c = [&](const double* M) __attribute__((always_inline)) {
        double4v c;
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = M[(4 * r + lk) * SBP + l16];
        return c;
    };
    auto store_c = [&](double* M, const double4v& c) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) M[(4 * r + lk) * SBP + l16] = c[r];
    };
    // c + sign A B, A by its row fragments, B in accumulator layout
    auto mul_add = [&](const double* MA, const double4v& b, double4v c, double sign) __attribute__((always_inline)) {
        double a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = sign * frag_rowk(MA, q);
#pragma unroll
        for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], c, 0, 0, 0);
        return c;
    };
    // c + the products lo .. hi, whose operands `load` gives; they are read a product ahead
    auto chain = [&](int lo, int hi, double4v c, auto&& load) __attribute__((always_inline)) {
        double a0[4], b0[4], a1[4], b1[4];
        auto multiply = [&](const double (&a)[4], const double (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], c, 0, 0, 0);
        };
        load(lo, a0, b0);
        int k = lo;
        for (; k + 2 <= hi; k += 2) {
            load(k + 1, a1, b1);
            multiply(a0, b0);
            load(k + 2, a0, b0);
            multiply(a1, b1);
        }
        if (k < hi) {
            load(hi, a1, b1);
            multiply(a0, b0);
            multiply(a1, b1);
        } else {
            multiply(a0, b0);
        }
        return c;
    };
    // c + sum over J = lo .. hi of L_IJ L_KJ^T
    auto mul_add_t = [&](int I, int K, int lo, int hi, double4v c) __attribute__((always_inline)) {
        const double* const MA = S + sub(I, 0);
        const double* const MB = S + sub(K, 0);
        return chain(lo, hi, c, [&](int J, double (&a)[4], double (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] = frag_rowk(MA + J * SBS, q);
                b[q] = frag_rowk(MB + J * SBS, q);
            }
        });
    };
    const double4v zero4 = {0.0, 0.0, 0.0, 0.0};
    // sub-block (I, J) of the matrix, its row fragments: loads without a branch, and the identity padding of a short last
    // block where the values are first used, so that nobody waits for them earlier
    auto fetch = [&](int I, int J) __attribute__((always_inline)) {
        double4v c;
        const double* p = Ab + int64_t(I * SBW + l16) * n + J * SBW + lk;
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = *(I * SBW + l16 < bs && J * SBW + 4 * q + lk < bs ? p + 4 * q : Ab);
        return c;
    };
    auto padded = [&](int I, int J, double4v c) __attribute__((always_inline)) {
        if (bs < NB)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = I * SBW + l16, col = J * SBW + 4 * q + lk;
                if (row >= bs || col >= bs) c[q] = row == col ? 1.0 : 0.0;
            }
        return c;
    };
    auto store_rowk = [&](double* M, const double4v& f) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) M[l16 * SBP + 4 * q + lk] = f[q];
    };
    // finished sub-block (I, J), in LDS, to the panel solve's operands: its row fragments, a lane's four side by side
    auto pack = [&](int I, int J) __attribute__((always_inline)) {
        if (I * SBW >= bs) return;
        double4v f;
#pragma unroll
        for (int q = 0; q < 4; ++q) f[q] = frag_rowk(S + sub(I, J), q);
        *reinterpret_cast<double4v*>(Pk + packed(I, J) + 4 * lane) = f;
    };

    // Leaf of block column J: wave 0 factors the diagonal sub-block in registers (lane i (mod 16) = row i; lanes
    // 16..63 shadow lanes 0..15) as Lh D Lh^T and leaves its inverse factor T = D^-1/2 Lh^-1 in the sub-block's place: the
    // panel solves below and the inverses of the halves need that, nothing reads L_JJ itself.
    // From one pivot to the next: one update, its broadcast, v_rcp_f64, its error and the column scaled by it, the column
    // corrected (the raw column is broadcast, not the scaled one, so nothing else waits for the reciprocal).  What does not
    // lie on that chain is issued behind its instructions: the updates of the other columns and the rows of
    // Z = Lh^-1, which follow without divisions, z_m = e_m - sum_{k<m} Lh[m][k] z_k: row m is final once rows 0 .. m-1 have
    // been eliminated from it and is then broadcast inside each 16-lane row to the lanes below.  Row q of lanes computes
    // the columns c = 4 k + q of Z: lane (q, i) has Z[i][4 k + q] in x[k].
    // Before, with Z behind the last pivot and the reciprocal corrected in front of the column: 2920 cycles a leaf, now 2080;
    // of these, 400 were what a pivot replaced by 1 cost every pivot.
    // The reciprocal is good to 4.6e-8 relative, a column corrected by its error to 2.2e-15, and that is an update's relative
    // error; columns scaled by reciprocal square roots with one step each had 8e-15.
    double x[4];   // wave 0: T of the last leaf, k-step q of its row fragments in x[q]
    auto leaf = [&](int J) __attribute__((always_inline)) {
        double* DJ = S + sub(J, J);
        const int i = l16;
        // Entries above the diagonal (c > i) are carried along: they never reach a valid entry (a broadcast of column j
        // takes lane c >= j).  The 16 steps form one straight-line block; whether a pivot was bad is asked once, behind it.
        double r[SBW];
        double my_d = 1.0;
#pragma unroll
        for (int c = 0; c < SBW; ++c) r[c] = DJ[i * SBP + c];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (4 * k + lk == i) ? 1.0 : 0.0;
        double p = bcast16<0>(r[0]);           // pivot, the same in every lane
        double y = __builtin_amdgcn_rcp(p);
        double e = __builtin_fma(-p, y, 1.0), t = -(r[0] * y);
        static_for<0, SBW>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j + 1 < SBW) {
                const double nm = __builtin_fma(t, e, t);
                fma_bcast16<j + 1>(r[j + 1], r[j], nm);   // r[j] was last written before p was broadcast
                const double pj = p;
                p = bcast16<j + 1>(r[j + 1]);
                y = __builtin_amdgcn_rcp(p);
                __builtin_amdgcn_sched_barrier(0);
                const double nlh = (i > j) ? nm : 0.0;
                my_d = (i == j) ? pj : my_d;
                // columns beyond j are still zero in row j of Z
                constexpr int rest = SBW - 2 - j, half = rest < 3 ? rest : 3, zs = j / 4 + 1;
                auto updates = [&](auto lo, auto hi, auto zhi) __attribute__((always_inline)) {
                    static_for<decltype(lo)::value, decltype(hi)::value>([&](auto cc) {
                        constexpr int c = decltype(cc)::value;
                        fma_bcast16<c>(r[c], r[j], nm);
                    });
                    static_for<0, decltype(zhi)::value>([&](auto kc) {
                        constexpr int k = decltype(kc)::value;
                        fma_bcast16<j>(x[k], x[k], nlh);   // x[k] was last written a pivot ago
                    });
                    __builtin_amdgcn_sched_barrier(0);
                };
                updates(std::integral_constant<int, j + 2>{}, std::integral_constant<int, j + 2 + half>{},
                        std::integral_constant<int, 0>{});
                e = __builtin_fma(-p, y, 1.0);
                t = -(r[j + 1] * y);
                updates(std::integral_constant<int, j + 2 + half>{}, std::integral_constant<int, SBW>{},
                        std::integral_constant<int, zs>{});
            } else {
                my_d = (i == j) ? p : my_d;
            }
        });
        if (__builtin_expect(__any(!(my_d > 0.0)), 0)) my_d = leaf_with_bad_pivots(DJ, i, lk, x, info, off + J * SBW);
        // every lane has read its row before any lane overwrites the sub-block (one wave: program order); zeros above
        // the diagonal
        const double rdi = rsqrt_refined(my_d);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] *= rdi;
            DJ[i * SBP + 4 * k + lk] = x[k];
        }
    };
    // The three roles pass the same barriers, two per column: behind its leaf and behind its solve.
    if (wave == 0) {
        store_rowk(S, padded(0, 0, fetch(0, 0)));
        leaf(0);
#pragma unroll 1
        for (int J = 0; J < NSB - 1; ++J) {
            __syncthreads();
            // L_J+1,J, transposed: register r of the result is L_J+1,J[l%16][4 r + l/16], a row fragment
            double4v lt = zero4;
            double* const D = S + sub(J + 1, J + 1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                lt = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q], frag_rowk(S + sub(J + 1, J), q), lt, 0, 0, 0);
            double4v c = load_c(D);
            store_rowk(S + sub(J + 1, J), lt);
#pragma unroll
            for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f64_16x16x4f64(-lt[q], lt[q], c, 0, 0, 0);
            store_c(D, c);
            __syncthreads();
            leaf(J + 1);
        }
        __syncthreads();
    } else {
        // Column inv_c of the halves' inverses, beside leaf J + 1, in the waves whose rows are complete first (not in
        // wave 4: its products slow the leaf beside them, 2900 -> 3700 cycles)
        const int inv_c = wave > 4 ? 7 - wave : NSB / 2;
        double4v pc = zero4;   // the column's next P
        auto inverse_step = [&](int J) __attribute__((always_inline)) {
            const int C = (J & (NSB / 2)) + inv_c;
            if (inv_c >= NSB / 2 - 1 || C > J) return;
            double4v xj = load_c(S + sub(J, J));
            if (C < J) {
                xj = mul_add(S + sub(J, J), pc, zero4, -1.0);
                store_c(S + sub(J, C), xj);   // in place of L_JC, which only this column's earlier products needed
            }
            if ((J + 1) % (NSB / 2) != 0) {
                pc = mul_add(S + sub(J + 1, J), xj, zero4, 1.0);
                if (C < J)
                    pc = chain(C, J - 1, pc, [&](int K, double (&a)[4], double (&b)[4]) __attribute__((always_inline)) {
                        const double4v x = load_c(S + sub(K, C));
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            a[q] = frag_rowk(S + sub(J + 1, K), q);
                            b[q] = x[q];
                        }
                    });
            }
            if (C < J) pack(J, C);
        };
        if (wave == 4) {
            const double4v a10 = fetch(1, 0), a11 = fetch(1, 1);
            store_rowk(S + sub(1, 0), padded(1, 0, a10));
            store_rowk(S + sub(1, 1), padded(1, 1, a11));
#pragma unroll 1
            for (int J = 0; J < NSB; ++J) {
                __syncthreads();
                if (J + 1 < NSB) __syncthreads();
                pack(J, J);
                if (J < NSB / 2)
                    for (int I = NSB / 2; I < NSB; ++I) pack(I, J);
            }
            return;
        }
        // A row of sub-blocks per wave, the longest ones on different SIMDs.  Its sub-blocks are held transposed: the
        // accumulators of (I, K) are then the B operand of its solve, whose result is L_IK's row fragments.  Column J + 1
        // takes its last update beside leaf J + 1 and column J + 2 all that there are before, so that 6 to 8 products are
        // due on a wave then at most; updating all columns would be 27 products in all beside the first leaf and 1 beside
        // the last.  Sums are held with the sign reversed, so that the products need no negated operand.
        const int I = wave < 4 ? NSB - wave : NSB + 1 - wave;
        double4v cur = fetch(I, 0), nxt = fetch(I, 1), pre = fetch(I, 2);   // (I, J); (I, J + 1); (I, J + 2) as it was
        cur = padded(I, 0, cur);
        nxt = -padded(I, 1, nxt);
#pragma unroll 1
        for (int J = 0; J < NSB; ++J) {
            const bool active = J + 2 <= I;
            __syncthreads();
            if (J + 1 < NSB) {
                if (active) {   // L_IJ = A_IJ T^T
                    double4v lt = zero4;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        lt = __builtin_amdgcn_mfma_f64_16x16x4f64(frag_rowk(S + sub(J, J), q), cur[q], lt, 0, 0, 0);
                    store_rowk(S + sub(I, J), lt);
                }
                __syncthreads();
                if (active) {
                    cur = -mul_add_t(J + 1, I, J, J, nxt);
                    nxt = -padded(I, J + 2, pre);
                    if (J + 3 <= I) pre = fetch(I, J + 3);
                    if (J + 2 == I) store_rowk(S + sub(I, J + 1), cur);   // wave 0 solves it
                    nxt = mul_add_t(J + 2, I, 0, J, nxt);
                    if (J + 2 == I) store_rowk(S + sub(I, I), -nxt);      // wave 0 takes over its last update
                }
            }
            inverse_step(J);
        }
    }
}

// ------------------------------------------------------------------------------------------
// fp64 MFMA GEMM:  C = alpha * A * op(B) + beta * C   (batched, optional triangular structure)
// ------------------------------------------------------------------------------------------
constexpr int GT = 128;  // tile side

enum : int { G_BTRANS = 1, G_ALOWER = 2, G_BLOWER = 4 };

struct GemmArgs {
    const double* A; int64_t lda, sa;
    const double* B; int64_t ldb, sb;
    double* C; int64_t ldc, sc;
    int m, n, k;   // sizes of every batch entry but the last
    int m_last;    // rows of the last batch entry (<= m)
    int k_last;    // inner size of the last batch entry (<= k)
    int batch;
    double alpha, beta;
    int flags;
    double* copy;      // where block (1, 0) also goes, rows of NB (nullptr: nowhere)
};

constexpr int RK = 8, RNS = 4;                      // inner steps per ring slot, ring slots of the GEMM tile
constexpr int R_PART_BYTES = GT * RK * 8;           // 8 KB: the A part or the B part of a stage
constexpr int R_STAGE_BYTES = 2 * R_PART_BYTES;
constexpr int GEMM_LDS_DOUBLES = RNS * R_STAGE_BYTES / 8;
constexpr int LDS_DOUBLES = GEMM_LDS_DOUBLES > POTRF_LDS_DOUBLES ? GEMM_LDS_DOUBLES : POTRF_LDS_DOUBLES;

// The workgroup's LDS: one static array per kernel, shared by the GEMM tile code and the factorization code.
__device__ __forceinline__ double* wg_lds() {
    __shared__ double lds[LDS_DOUBLES];
    return lds;
}

// ------------------------------------------------------------------------------------------
// One TM x TN tile (tm, tn) of batch entry z with WR x WC waves; K > 0: an inner range of that length.
// 128 x 128: 2 x 4 waves of 64 x 32, so that with two workgroups per CU four waves share a SIMD and cover each other's
// waits.  64 x 64 (2 x 2 waves of 32 x 32) and 128 x 64 (4 x 2 of 32 x 32): for launches whose 128-wide tiles would
// leave CUs idle.
// The operands are streamed global -> LDS directly (buffer_load ... lds) through a ring of NS slots
// of SUB parts of RK inner steps each, NS - 1 stages ahead of the MFMAs: no staging registers, no LDS stores, no
// multiplication by alpha on the way (alpha = +-1 is folded into the accumulators: they start as (beta / alpha) C and the
// result is alpha acc, both exact), one barrier per stage.  A direct load deposits lane l at slot + 16 l, so rows cannot be
// padded; the 16-byte chunks (two doubles) are permuted instead, which costs nothing on the global side because
// every lane supplies its own address:
//   A-form part (rows x RK k, a row is 64 B = 4 chunks): chunk c of row r sits at position c ^ ((r >> 2) & 3);
//     the 16 rows x 2 k that one half-wave reads for an MFMA operand then fall into 64 different banks.
//   NN B part (RK k-rows x TN columns, a k-row is TN / 2 chunks): chunk c of k-row kr sits at c ^ ((kr & 1) << 3).
// ------------------------------------------------------------------------------------------

template <bool bt, int WR, int WC, int TM, int TN, int SUB, int NS, int K = 0>
__device__ __forceinline__ void dgemm_tile_ring(const GemmArgs& g, const int tn, const int tm, const int z, double* lds) {
    constexpr int NW = WR * WC;
    constexpr int NI = TM / (16 * WR), NJ = TN / (16 * WC);       // 16 x 16 MFMA tiles per wave
    constexpr int A_LOADS = TM / 16, B_LOADS = TN / 16;           // 1 KB loads of a part
    constexpr int LA = SUB * A_LOADS / NW, LPW = LA + SUB * B_LOADS / NW;   // loads per wave and stage: A's come first
    constexpr int A_BYTES = TM * RK * 8, PART_BYTES = A_BYTES + TN * RK * 8, STAGE_BYTES = SUB * PART_BYTES;
    constexpr int KROW = TN * 8;        // bytes of a k-row of a row-major B part
    static_assert(SUB * A_LOADS % NW == 0 && SUB * B_LOADS % NW == 0, "a load belongs to one operand in every wave");
    const bool last = (z == g.batch - 1);
    const int m = last ? g.m_last : g.m;
    const int kdim = last ? g.k_last : g.k;
    if (tm * TM >= m) return;
    const double* __restrict__ A = g.A + z * g.sa;
    const double* __restrict__ B = g.B + z * g.sb;
    double* __restrict__ C = g.C + z * g.sc;
    int k_lo = 0, k_hi = kdim;
    if (g.flags & G_BLOWER) k_lo = tn * TN;
    if (g.flags & G_ALOWER) k_hi = min(kdim, (tm + 1) * TM);
    const int n_st = K > 0 ? K / (SUB * RK) : k_hi > k_lo ? (k_hi - k_lo) / (SUB * RK) : 0;   // inner ranges are multiples of 16

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / WC, wc = wave % WC;
    const int m0 = tm * TM, n0 = tn * TN;
    const int rw = wr * (NI * 16);
    const int cw = wc * (NJ * 16);
    const int l16 = lane & 15, lk = lane >> 4;
    const uint32_t lds0 = uint32_t(uintptr_t((ONECOMP_LDS char*)lds));

    // descriptor bases: the tile's first operand row / column at the start of the inner range; a stage's descriptor
    // starts SUB * RK inner steps further on (64-bit scalar arithmetic), so that the 32-bit offsets of the lanes stay
    // below 128 rows x ld
    const double* const abase = A + int64_t(m0) * g.lda + k_lo;
    const double* const bbase = bt ? B + int64_t(n0) * g.ldb + k_lo : B + int64_t(k_lo) * g.ldb + n0;
    const int64_t step_b = bt ? int64_t(SUB * RK) : int64_t(SUB * RK) * g.ldb;   // doubles along k per stage
    uint32_t voff[LPW], ldst[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        const bool is_a = q < LA;
        const int j = wave + NW * (is_a ? q : q - LA);
        const int sp = j / (is_a ? A_LOADS : B_LOADS), jj = j % (is_a ? A_LOADS : B_LOADS);   // part, load of the part
        if (is_a || bt) {
            const int row = 16 * jj + (lane >> 2);
            const int c = (lane & 3) ^ ((row >> 2) & 3);
            const bool ok = is_a ? (m0 + row < m) : (n0 + row < g.n);
            voff[q] = ok ? uint32_t((int64_t(row) * (is_a ? g.lda : g.ldb) + sp * RK + 2 * c) * 8) : LDS_DMA_OOB;
        } else {
            const int e = jj * 64 + lane;       // 16-byte chunk of the part
            const int kr = e / (KROW / 16), c = (e % (KROW / 16)) ^ ((kr & 1) << 3);
            voff[q] = (n0 + 2 * c < g.n) ? uint32_t((int64_t(sp * RK + kr) * g.ldb + 2 * c) * 8) : LDS_DMA_OOB;
        }
        ldst[q] = sp * PART_BYTES + (is_a ? 0 : A_BYTES) + jj * 1024;
    }
    // loads of the next stage into a slot; past the end: an empty range, which deposits zeros
    const double* pa = abase;
    const double* pb = bbase;
    int ahead = n_st;   // stages that have not been requested
    auto issue = [&](int slot_no) __attribute__((always_inline)) {
        const uint32_t slot = lds0 + uint32_t(slot_no) * STAGE_BYTES;
        const uint32_t range = ahead > 0 ? 0x7FFFFFFFu : 0u;
        --ahead;
        const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(pa), 0, range, 0x00020000);
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(pb), 0, range, 0x00020000);
        pa += SUB * RK;
        pb += step_b;
#pragma unroll
        for (int q = 0; q < LPW; ++q) lds_load16(slot + ldst[q], voff[q], q < LA ? ra : rb);
    };
    for (int st = 0; st < NS - 1; ++st) issue(st);

    // accumulators start as (beta / alpha) C (alpha = +-1: exact); register r of lane l: row 4 r + l / 16,
    // column l % 16 of its 16 x 16 tile
    const double binit = g.beta * g.alpha;   // beta / alpha for alpha = +-1
    double4v acc[NI][NJ];
    const bool full = (m0 + TM <= m) && (n0 + TN <= g.n);
    double* __restrict__ ct = C + int64_t(m0 + rw + lk) * g.ldc + n0 + cw + l16;
    if (g.beta == 0.0) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0;
    } else if (full) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = binit * ct[int64_t(i * 16 + 4 * r) * g.ldc + j * 16];
    } else {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = m0 + rw + i * 16 + 4 * r + lk;
                    const int col = n0 + cw + j * 16 + l16;
                    double c = 0.0;
                    if (row < m && col < g.n) c = binit * C[int64_t(row) * g.ldc + col];
                    acc[i][j][r] = c;
                }
    }

    // fragment addresses inside a stage (bytes), inner steps 0 .. 3; steps 4 .. 7: A-form ^ 32, NN + 4 KB
    int fa[NI], fb[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int row = rw + i * 16 + l16;
        fa[i] = row * 64 + (((lk >> 1) ^ ((row >> 2) & 3)) << 4) + (lk & 1) * 8;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int col = cw + j * 16 + l16;
        if (bt) fb[j] = A_BYTES + col * 64 + (((lk >> 1) ^ ((col >> 2) & 3)) << 4) + (lk & 1) * 8;
        else fb[j] = A_BYTES + lk * KROW + (((col >> 1) ^ ((lk & 1) << 3)) << 4) + (col & 1) * 8;
    }
    const char* ldsc = reinterpret_cast<const char*>(lds);

    auto stage = [&](auto slot_c) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value;
        // the loads of the NS - 2 stages behind this one may still be in flight: wait for its own, publish them,
        // and refill the slot every wave has finished reading (that of the stage before)
        __builtin_amdgcn_s_waitcnt(wait_vmcnt(LPW * (NS - 2)));
        __syncthreads();
        issue((slot + NS - 1) % NS);
        const char* sp = ldsc + slot * STAGE_BYTES;
#pragma unroll
        for (int e = 0; e < 2 * SUB; ++e) {   // four inner steps each
            const char* pp = sp + (e >> 1) * PART_BYTES;
            const int h = e & 1;
            double a[NI], b[NJ];
#pragma unroll
            for (int i = 0; i < NI; ++i) a[i] = *reinterpret_cast<const double*>(pp + (h ? fa[i] ^ 32 : fa[i]));
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                b[j] = *reinterpret_cast<const double*>(pp + (bt ? (h ? fb[j] ^ 32 : fb[j]) : fb[j] + h * 4 * KROW));
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    // The slots are constants: all stages unrolled where their number is known, else one round of the ring per iteration.
    // With slots and descriptors computed in every stage the scalar work behind its barrier held the MFMAs back: factor of
    // d_in 8192 8446 -> 7654 us, 14336 36.0 -> 33.6 ms.
    if constexpr (K > 0) {
        static_for<0, K / (SUB * RK)>([&](auto st) __attribute__((always_inline)) {
            stage(std::integral_constant<int, decltype(st)::value % NS>{});
        });
    } else {
        for (int st = 0; st < n_st; st += NS)
            static_for<0, NS>([&](auto slot_c) __attribute__((always_inline)) {
                if (st + decltype(slot_c)::value < n_st) stage(slot_c);
            });
    }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));   // no LDS write may be in flight when the slots are reused or the workgroup ends

    const double aout = g.alpha;
    if (bt && g.copy && m0 == NB && n0 < NB) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = rw + i * 16 + 4 * r + lk;
                    if (m0 + row < m) g.copy[row * NB + n0 + cw + j * 16 + l16] = aout * acc[i][j][r];
                }
    }
    if (full) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) ct[int64_t(i * 16 + 4 * r) * g.ldc + j * 16] = aout * acc[i][j][r];
    } else {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = m0 + rw + i * 16 + 4 * r + lk;
                    const int col = n0 + cw + j * 16 + l16;
                    if (row < m && col < g.n) C[int64_t(row) * g.ldc + col] = aout * acc[i][j][r];
                }
    }
}

// Work map of a GEMM launch: one workgroup per tile that has work, in a one-dimensional grid (workgroups that return
// at once are not free: each still waits for its turn at a CU, and a quarter of such workgroups in a launch cost a
// quarter of its time).  Workgroups are dispatched in rank order; with a triangular operand the tiles differ in
// length (B lower: the inner range starts at the tile's column, so tile columns get shorter to the right; A lower: it
// ends at the tile's row, so tile rows get longer downwards) and the longest tiles come first, so that no long tile
// starts when the rest of the launch is nearly done.  Order: the last batch entry (the only one that can be
// shorter), then the other entries interleaved tile by tile.
struct GemmGrid {
    int tn_cnt, tm_full, tm_last, per_full, per_last, total;
};
template <int T>
__host__ __device__ inline GemmGrid gemm_grid(const GemmArgs& g) {
    GemmGrid q;
    q.tn_cnt = (g.n + T - 1) / T;
    q.tm_full = (g.m + T - 1) / T;
    q.tm_last = (g.m_last + T - 1) / T;
    q.per_full = q.tm_full * q.tn_cnt;
    q.per_last = q.tm_last * q.tn_cnt;
    q.total = q.per_last + (g.batch - 1) * q.per_full;
    return q;
}
template <int T>
__device__ __forceinline__ void gemm_tile_from_rank(const GemmArgs& g, int v, int& tm, int& tn, int& z) {
    const GemmGrid q = gemm_grid<T>(g);
    int rem, tm_cnt;
    if (v < q.per_last) {
        z = g.batch - 1;
        rem = v;
        tm_cnt = q.tm_last;
    } else {
        v -= q.per_last;
        z = v % (g.batch - 1);
        rem = v / (g.batch - 1);
        tm_cnt = q.tm_full;
    }
    if (g.flags & G_BLOWER) {   // tile columns left to right, rows fastest
        tn = rem / tm_cnt;
        tm = rem % tm_cnt;
    } else if (g.flags & G_ALOWER) {   // tile rows from the bottom
        tm = tm_cnt - 1 - rem / q.tn_cnt;
        tn = rem % q.tn_cnt;
    } else {
        tm = rem / q.tn_cnt;
        tn = rem % q.tn_cnt;
    }
}

// The launches of the inverse.  128-wide tiles run eight waves per workgroup (64 x 32 per wave, under 128 registers):
// four waves share a SIMD and cover each other's waits (64 -> 66 TFLOP/s on large products against four waves).
template <int T>
struct GemmShape;
template <>
struct GemmShape<128> {
    static constexpr int WR = 2, WC = 4, WAVES = WR * WC, SLOTS = RNS;
};
template <>
struct GemmShape<64> {
    static constexpr int WR = 2, WC = 2, WAVES = WR * WC, SLOTS = 6;
};
template <int T>
__global__ __launch_bounds__(64 * GemmShape<T>::WAVES, 2) void dgemm_kernel(GemmArgs g) {
    using S = GemmShape<T>;
    __shared__ double lds[S::SLOTS * 2 * T * RK];
    int tm, tn, z;
    gemm_tile_from_rank<T>(g, blockIdx.x, tm, tn, z);
    tm = __builtin_amdgcn_readfirstlane(tm);   // the divisions leave them in vector registers
    tn = __builtin_amdgcn_readfirstlane(tn);
    z = __builtin_amdgcn_readfirstlane(z);
    dgemm_tile_ring<false, S::WR, S::WC, T, T, 1, S::SLOTS>(g, tn, tm, z, lds);
}

// Trailing update of one step of the blocked Cholesky together with the factorization of the next diagonal block:
// workgroup 0, the first of the grid and therefore resident from the start, factors the block (the panel solve's launch
// has brought it up to date) while the other workgroups update the columns that are due.  Takes the
// single-workgroup factorization off the critical path of every step whose update is longer.
// A: the whole matrix; the trailing matrix begins at block row and column step + 1 and has `rest` rows.  Step -1, a launch
// of one workgroup: the first diagonal block.  NARROW: few columns, see plan::syrk_lag; slab_cols > 0: the first slab_cols
// block columns only.
template <bool NARROW>
__global__ __launch_bounds__(POTRF_THREADS, 4) void syrk_potrf_kernel(double* __restrict__ A, double* __restrict__ V,
                                                                     double* __restrict__ Pn, double* __restrict__ Pk,
                                                                     int n, int step, int rest,
                                                                     int stride, int lag, int base, int inv_cols,
                                                                     int slab_cols, int32_t* __restrict__ info) {
    const int off = (step + 1) * NB, n_t = (rest + GT - 1) / GT;
    if (blockIdx.x == 0) {
        potrf_body(A, Pk, n, off, min(NB, rest), info, wg_lds());
        return;
    }
    int tm, tn;   // NARROW: tn counts columns of 64
    bool inverse = false;
    if (!(!NARROW         ? plan::syrk_tile(blockIdx.x, plan::syrk_grid(n_t, stride), tm, tn)
          : slab_cols > 0 ? plan::syrk_slab_tile(blockIdx.x, n_t, slab_cols, tm, tn)
                          : plan::syrk_narrow_tile(blockIdx.x, n_t, inv_cols, tm, tn, inverse)))
        return;
    tm = __builtin_amdgcn_readfirstlane(tm);   // the divisions leave them in vector registers
    tn = __builtin_amdgcn_readfirstlane(tn);
    const int k0 = NARROW || tn == 0 ? step : __builtin_amdgcn_readfirstlane(plan::syrk_first_panel(tn, step, lag, base));
    GemmArgs g{};   // C -= P P^T with P the panels k0 .. step below the diagonal block
    g.A = A + int64_t(off) * n + k0 * NB; g.lda = n;
    g.B = g.A; g.ldb = n;
    g.C = A + int64_t(off) * n + off; g.ldc = n;
    g.m = g.m_last = g.n = rest;
    g.k = g.k_last = (step + 1 - k0) * NB;
    g.batch = 1;
    g.alpha = -1.0; g.beta = 1.0; g.flags = G_BTRANS;
    g.copy = Pn;   // the next step's block below the diagonal, unsolved
    if (NARROW && __builtin_amdgcn_readfirstlane(int(inverse))) {   // V[i, :] += L[i, step] V[step, :], the rows below
        g.B = V + int64_t(step) * NB * n;
        g.C = V + int64_t(off) * n;
        g.n = (step + 1) * NB;
        g.alpha = 1.0; g.beta = tn < 2 * step ? 1.0 : 0.0; g.flags = 0;
        dgemm_tile_ring<false, 4, 2, GT, 64, 2, 3, NB>(g, tn, tm, 0, wg_lds());
        return;
    }
    if constexpr (NARROW) dgemm_tile_ring<true, 4, 2, GT, 64, 2, 3, NB>(g, tn, tm, 0, wg_lds());
    else dgemm_tile_ring<true, 2, 4, GT, GT, 1, RNS>(g, tn, tm, 0, wg_lds());
}

// ------------------------------------------------------------------------------------------
// Panel solve of the blocked Cholesky, P <- P L_kk^-T for the panel of `rest` rows below diagonal block `step`, and the
// update of the next diagonal block, A -= P P^T, which the chain of diagonal blocks waits for.
// With V1, V2 the inverses of the halves of L_kk and L21 the quarter between them, columns 0 .. 63 and 64 .. 127 are
//     X1 = P1 V1^T,   X2 = (P2 - X1 L21^T) V2^T :
// 36 products of 16 x 16 sub-blocks per 16 rows, as many as with the inverse of the whole block, which would lengthen
// the chain by 64 products and their waits.  A 128 x 128 GEMM tile per workgroup would occupy only rest / 128 of the
// CUs for about 23 us; here a workgroup takes two groups of 16 rows, and its four waves share out each group's column
// tiles (c and 3 - c: equal lengths of the triangular inner range).  Rows and results go through LDS; the operands, shared
// by all workgroups and resident in L2, come from Pk in MFMA operand order, 32 bytes a lane, and are requested before
// the rows have arrived (gathered from the rows of V and A, 8 bytes a lane: 2 us more a launch).
// Workgroups 0 .. n_pairs - 1: a sub-block (I, J) of the next diagonal block each.  They solve the row groups I and J of the
// next block row (from Pn, the copy of its unsolved values: its place in A is being overwritten by the workgroups
// that solve it) and multiply them: 36 short products side by side.  One workgroup for the whole 128 x 128 x 128 update
// took 12 us of every step; here the launch takes 9 us, with the update and with its operands packed.
// The next four: V's diagonal block, whose columns are the solutions of the same system for the unit vectors (transposed
// rows), 32 columns each.  The next 4 inv_blocks: row block `step` of the inverse, where that
// goes along with the factorization (factor_run), V[step, :] = -L_kk^-1 V[step, :], again the same system for transposed rows.
// Layouts as in potrf_body: A[i][k]: i = l % 16, k = l / 16; B[k][j]: k = l / 16, j = l % 16;
// D register r: row 4 r + l / 16, column l % 16.
// ------------------------------------------------------------------------------------------
constexpr int TR = 32;          // rows per workgroup
constexpr int TRP = NB + 2;     // LDS pitch in doubles: the 16 rows x 2 k of a half-wave fall into 64 different banks
constexpr int PANEL_PAIRS = NSB * (NSB + 1) / 2;
constexpr int PANEL_UNITS = NB / TR;

template <int H>   // waves of column tiles H and 3 - H of each half
__device__ __forceinline__ void panel_body(const double* __restrict__ Pk, int bs, int rt, double* sP, double* sX) {
    constexpr int C[2] = {H, 3 - H};
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    double4v b1[2][4], b2[2][4], b3[2][4];   // operands of the three products
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        // sub-block rows behind a short last block: the first sub-block instead, for results that nobody takes
        const bool top = C[u] * SBW < bs, low = HALF + C[u] * SBW < bs;
#pragma unroll
        for (int k = 0; k <= C[u]; ++k) b1[u][k] = *reinterpret_cast<const double4v*>(Pk + (top ? packed(C[u], k) : 0) + 4 * lane);
#pragma unroll
        for (int k = 0; k < 4; ++k) b2[u][k] = *reinterpret_cast<const double4v*>(Pk + (low ? packed(4 + C[u], k) : 0) + 4 * lane);
#pragma unroll
        for (int k = 0; k <= C[u]; ++k)
            b3[u][k] = *reinterpret_cast<const double4v*>(Pk + (low ? packed(4 + C[u], 4 + k) : 0) + 4 * lane);
    }
    double* const p = sP + (rt * 16 + li) * TRP + lk;    // row fragments of the row group
    double* const x = sX + (rt * 16 + li) * TRP + lk;
    double* const pc = sP + (rt * 16 + lk) * TRP + li;   // its accumulator layout
    double* const xc = sX + (rt * 16 + lk) * TRP + li;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4 * (C[u] + 1); ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(p[4 * ks], b1[u][ks >> 2][ks & 3], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) xc[4 * r * TRP + C[u] * 16] = acc[r];
    }
    __syncthreads();
    {
        double4v acc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[u][r] = -pc[4 * r * TRP + HALF + C[u] * 16];
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) {
            const double a = x[4 * ks];
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b2[u][ks >> 2][ks & 3], acc[u], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) pc[4 * r * TRP + HALF + C[u] * 16] = -acc[u][r];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4 * (C[u] + 1); ++ks)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(p[HALF + 4 * ks], b3[u][ks >> 2][ks & 3], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) xc[4 * r * TRP + HALF + C[u] * 16] = acc[r];
    }
    __syncthreads();
}

// n_pairs: PANEL_PAIRS, or 0 where the next diagonal block is brought up to date otherwise.  Vd: V's diagonal block, rows
// of ldd; V and inv_blocks > 0 only with ldd == n.
__global__ __launch_bounds__(256) void panel_kernel(double* __restrict__ A, double* __restrict__ V, double* __restrict__ Vd,
                                                   int ldd, const double* __restrict__ Pn, const double* __restrict__ Pk,
                                                   int n, int step, int rest, int n_pairs, int inv_blocks) {
    __shared__ __align__(16) double sP[TR * TRP];
    __shared__ __align__(16) double sX[TR * TRP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t off = int64_t(step) * NB;
    const int bs = min(NB, n - int(off));
    double* __restrict__ const P = A + (off + NB) * n + off;
    const int n_inv = PANEL_UNITS + NB / TR * inv_blocks;
    const bool pair = int(blockIdx.x) < n_pairs;
    const int inv = int(blockIdx.x) - n_pairs;   // 0 .. n_inv - 1: columns of V
    const bool is_inv = !pair && inv < n_inv;
    int I = 0, J = 0, m0 = 0;
    if (pair) {
        const int b = blockIdx.x;
        I = (b >= 1) + (b >= 3) + (b >= 6) + (b >= 10) + (b >= 15) + (b >= 21) + (b >= 28);
        J = int(blockIdx.x) - I * (I + 1) / 2;
        if (I * SBW >= rest) return;
    } else if (!is_inv) {
        m0 = (inv - n_inv) * TR;
    }
    // thread t: 16-byte pieces t % 8, t % 8 + 8, .. of row t / 8
    const int r = tid >> 3, c0 = (tid & 7) * 2;
    const int row = pair ? (r < SBW ? I : J) * SBW + (r & (SBW - 1)) : m0 + r;   // of the panel
    // transposed: rows t / 32, t / 32 + 8, .. of the block, its column t % 32
    const int vr = tid >> 5, vc = tid & 31;
    double* const vcol = (inv < PANEL_UNITS ? Vd + inv * TR : V + off * n + (inv - PANEL_UNITS) * TR) + vc;
    if (is_inv) {
        double v[16];
        if (inv < PANEL_UNITS) {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = vr + 8 * e == inv * TR + vc ? -1.0 : 0.0;
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = vr + 8 * e < bs ? vcol[int64_t(vr + 8 * e) * ldd] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) sP[vc * TRP + vr + 8 * e] = v[e];
    } else {
        const double* const src = pair ? Pn + row * NB + c0 : P + int64_t(row) * n + c0;
        double2 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = row < rest ? *reinterpret_cast<const double2*>(src + 16 * e) : make_double2(0.0, 0.0);
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<double2*>(sP + r * TRP + c0 + 16 * e) = v[e];
    }
    // the element of the next diagonal block this thread will update
    const int er = I * SBW + (tid >> 4), ec = J * SBW + (tid & 15);
    double* const D = A + (off + NB + er) * n + off + NB + ec;
    const bool inside = pair && er < rest && ec < rest;
    double d = inside ? *D : 0.0;
    if (wave < 2) panel_body<0>(Pk, bs, wave & 1, sP, sX);
    else panel_body<1>(Pk, bs, wave & 1, sP, sX);
    if (is_inv) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int vrow = vr + 8 * e;
            if (vrow < bs && (inv >= PANEL_UNITS || (vrow >= inv * TR + vc && inv * TR + vc < bs))) vcol[int64_t(vrow) * ldd] = -sX[vc * TRP + vrow];
        }
        return;
    }
    if (!pair) {
        if (row < rest) {
            double* const dst = P + int64_t(row) * n + c0;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                *reinterpret_cast<double2*>(dst + 16 * e) = *reinterpret_cast<const double2*>(sX + r * TRP + c0 + 16 * e);
        }
        return;
    }
    // a quarter of the inner range per wave, the four partial products added in order
    const int li = lane & 15, lk = lane >> 4;
    double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const int k = wave * 32 + 4 * ks + lk;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sX[li * TRP + k], sX[(SBW + li) * TRP + k], acc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) sP[wave * (SBW * SBW) + (4 * q + lk) * SBW + li] = acc[q];   // P has been read
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) d -= sP[w * (SBW * SBW) + tid];
    if (inside) *D = d;
}

onecomp_status dgemm(const GemmArgs& g, hipStream_t stream) {
    if (g.m <= 0 || g.n <= 0 || g.batch <= 0 || g.m_last <= 0) return ONECOMP_OK;
    // 128-wide tiles move half the operand bytes per flop of 64-wide ones, but a launch of few of them leaves CUs idle
    // and ends with its longest tile (the triangular operand makes the inner ranges differ).  Whole factor, us, with
    // 64-wide tiles in no launch / in launches of up to 256 / 1024 128-wide tiles: d_in 512: 336 / 262 / 262;
    // 2048: 1423 / 1071 / 1070; 4096: 3103 / 2570 / 2555; 8192: 10234 / 9953 / 9602; 14336: 38.2 ms each way.
    const int t128 = gemm_grid<128>(g).total;
    if (t128 > 4 * device_cus()) {
        hipLaunchKernelGGL(dgemm_kernel<128>, dim3(unsigned(t128)), dim3(64 * GemmShape<128>::WAVES), 0, stream, g);
    } else {
        hipLaunchKernelGGL(dgemm_kernel<64>, dim3(unsigned(gemm_grid<64>(g).total)), dim3(64 * GemmShape<64>::WAVES), 0, stream, g);
    }
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

struct Workspace {
    double* A;      // n x n: reversed damped matrix, then L in its lower triangle
    double* V;      // n x n: L^-1 (lower)
    double* T;      // n x n: temporaries of the inverse
    double* Pk;     // in T's first half: operands of a panel solve, see potrf_body
    double* Pn;     // up to 128 x 128, in T's second half: the block below a diagonal block before its panel is solved
    double* dfix;   // n
    double* lam;    // 1
    float* keys;    // n
    int32_t* perm;  // n
};

Workspace carve(void* ws, int64_t n) {
    char* p = static_cast<char*>(ws);
    const size_t mat = align_up(size_t(n) * n * sizeof(double), 256);
    Workspace w;
    w.A = reinterpret_cast<double*>(p); p += mat;
    w.V = reinterpret_cast<double*>(p); p += mat;
    w.T = reinterpret_cast<double*>(p); p += mat;
    w.Pk = w.T;   // n / 16 <= 8 block rows: at most n n doubles; 36 sub-blocks: not more than the half before Pn
    w.Pn = w.T + align_up(size_t(n) * n / 2, 32);   // min(128, n - 128) rows of 128 fit behind it for every n > 128
    w.dfix = reinterpret_cast<double*>(p); p += align_up(size_t(n) * sizeof(double), 256);
    w.lam = reinterpret_cast<double*>(p); p += 256;
    w.keys = reinterpret_cast<float*>(p); p += align_up(size_t(n) * sizeof(float), 256);
    w.perm = reinterpret_cast<int32_t*>(p);
    return w;
}

// V's diagonal blocks from where factor_slabs keeps them, zeros above their diagonals
__global__ __launch_bounds__(256) void place_diagonal_kernel(const double* __restrict__ Vd, int n, double* __restrict__ V) {
    const int b = blockIdx.x, c = threadIdx.x & (NB - 1);
    for (int r = threadIdx.x / NB; r < NB; r += 256 / NB) {
        const int row = b * NB + r, col = b * NB + c;
        if (row < n && col < n) V[int64_t(row) * n + col] = c <= r ? Vd[(int64_t(b) * NB + r) * NB + c] : 0.0;
    }
}

// ---- left-looking Cholesky of wide matrices -----------------------------------------------------------------------------
// A slab of block columns is brought up to date by everything left of it in one product of 8-bit residues, then factored
// block by block as the narrow matrices are, the trailing updates ending at the slab's edge, and its own residues are
// taken.  Left-looking, so that every entry is put together from residues once, over the longest inner range there is.
// Whole factor, right-looking in fp64 : by residues, us, inverse and block form: d_in 5120 2603 : 2859, 1656 : 1793; 6528 4340 :
// 4433, 2787 : 2769; 6656 4549 : 4524, 2917 : 2792; 7168 5407 : 5163, 3521 : 3168; 8192 7708 : 6431, 4949 : 3901; 14336 33.9 :
// 22.4 ms, 19.9 : 12.0; 28672 233 : 129, 130 : 66.9.  Wider than RESIDUE_MAX the sums' bounds have not been worked out.
constexpr int RESIDUE_MIN = 6656, RESIDUE_MAX = residue::MAX_K;
bool by_residues(int n) { return n >= RESIDUE_MIN && n <= RESIDUE_MAX; }
// Columns of a slab: longer inner ranges and whole patches of tiles against the updates inside the slab.  512 : 768 : 1024, us,
// inverse form: d_in 7168 5068 : 5041 : -; 8192 6592 : 6491 : 6428; 14336 23.0 ms : - : 22.3; 28672 129.3 : - : 127.8.
int slab_width(int n) { return n >= 8192 ? 1024 : 512; }
// The inverse's products of block pairs of at least this size go by residues.  From 2048 on: d_in 8192 6592 -> 6769 us, 28672
// 127.8 -> 128.9 ms.  Blocks of 4096 with a last one of so many rows below, whole factor by residues : in fp64, us: 2432 4542 :
// 4433, 2560 4623 : 4524, 2816 4883 : 5006, 3072 5163 : 5309, 3584 5957 : 6200.
constexpr int64_t RESIDUE_INVERSE_MIN = 4096, RESIDUE_INVERSE_MIN_ROWS = 2816;

onecomp_status factor_slabs(const Workspace& w, int n, char* product, int32_t* info, hipStream_t stream) {
    const int slab_cols = slab_width(n), slab = slab_cols / NB, nblk = int(ceil_div(n, NB));
    // residues of L, V's diagonal blocks, operands of the panel solve and the block below the diagonal: in place of V and T
    char* p = reinterpret_cast<char*>(w.V);
    const residue::Operand R(p, n, n);
    p += align_up(residue::operand_bytes(n, n), 256);
    double* const Vd = reinterpret_cast<double*>(p);
    p += size_t(nblk) * NB * NB * sizeof(double);
    double* const Pk = reinterpret_cast<double*>(p);
    p += size_t(PANEL_PAIRS) * SBW * SBW * sizeof(double);
    double* const Pn1 = reinterpret_cast<double*>(p);
    p += size_t(NB) * NB * sizeof(double);
    if (p > reinterpret_cast<char*>(w.dfix) || residue::product_bytes(n, slab_cols) > size_t(n) * n * sizeof(float)) return ONECOMP_ERR_UNSUPPORTED;
    int32_t* const shift = reinterpret_cast<int32_t*>(w.keys);
    double* const left = w.dfix;
    onecomp_status st = residue::row_bounds(w.A, n, shift, left, stream);
    if (st != ONECOMP_OK) return st;
    for (int s0 = 0; s0 < nblk; s0 += slab) {
        const int s1 = min(s0 + slab, nblk), c0 = s0 * NB, width = min(slab_cols, n - c0);
        double* const Pn = s0 > 0 ? Pn1 : w.Pn;   // the first one has been written beside the matrix
        if (s0 > 0) {
            st = residue::update_columns(w.A, n, c0, width, shift, R, Pn, product, stream);
            if (st != ONECOMP_OK) return st;
        }
        hipLaunchKernelGGL(syrk_potrf_kernel<true>, dim3(1), dim3(POTRF_THREADS), 0, stream, w.A, w.V, Pn, Pk, n, s0 - 1, n - c0, 1,
                           1, 0, 0, 0, info);
        ONECOMP_CHECK_LAUNCH();
        for (int s = s0; s < s1; ++s) {
            const int rest = max(0, n - (s + 1) * NB), pairs = s + 1 < s1 ? PANEL_PAIRS : 0;
            hipLaunchKernelGGL(panel_kernel, dim3(pairs + PANEL_UNITS + unsigned(ceil_div(rest, TR))), dim3(256), 0, stream, w.A, w.V,
                               Vd + int64_t(s) * NB * NB, NB, Pn, Pk, n, s, rest, pairs, 0);
            ONECOMP_CHECK_LAUNCH();
            if (s + 1 == s1) break;
            const int cols = s1 - 1 - s;   // block columns of the slab behind this one
            hipLaunchKernelGGL(syrk_potrf_kernel<true>, dim3(unsigned(plan::syrk_slab_grid(nblk - 1 - s, cols))),
                               dim3(POTRF_THREADS), 0, stream, w.A, w.V, Pn, Pk, n, s, rest, 1, 1, s, 0, cols, info);
            ONECOMP_CHECK_LAUNCH();
        }
        if (s1 < nblk) {
            st = residue::convert_columns(w.A, n, s1 * NB, c0, width, shift, left, R, stream);
            if (st != ONECOMP_OK) return st;
        }
    }
    hipLaunchKernelGGL(place_diagonal_kernel, dim3(unsigned(nblk)), dim3(256), 0, stream, Vd, n, w.V);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

}  // namespace

size_t factor_workspace_bytes(int64_t n) {
    return 3 * align_up(size_t(n) * n * sizeof(double), 256) + align_up(size_t(n) * sizeof(double), 256) + 256 +
           2 * align_up(size_t(n) * sizeof(float), 256);
}

onecomp_status factor_run(const float* H, int64_t d_in, float damp, int act_order, int form, int32_t* perm_out,
                          float* U, int32_t* info, void* workspace, hipStream_t stream) {
    const int n = int(d_in);
    Workspace w = carve(workspace, n);
    onecomp_status st;

    hipLaunchKernelGGL(prep_diag_kernel, dim3(1), dim3(1024), 0, stream, H, n, double(damp), w.keys, w.dfix, w.lam, info,
                       int(!act_order), perm_out);
    ONECOMP_CHECK_LAUNCH();
    if (act_order) {   // w.T is free until the triangular inverse
        hipLaunchKernelGGL(order_kernel, dim3(unsigned(ceil_div(n, ORDER_KEYS))), dim3(64 * ORDER_WAVES), 0, stream, w.keys, n, w.perm,
                           perm_out);
        ONECOMP_CHECK_LAUNCH();
        float* S = reinterpret_cast<float*>(w.T);
        const unsigned tiles = unsigned(ceil_div(n, 64));
        hipLaunchKernelGGL(mirror_kernel, dim3(tiles, tiles), dim3(256), 0, stream, H, n, S);
        ONECOMP_CHECK_LAUNCH();
        hipLaunchKernelGGL(build_order_kernel, dim3(unsigned(n)), dim3(512), min(n, GATHER_COLS) * sizeof(float), stream,
                           S, n, w.perm, w.dfix, w.lam, w.A, w.V, w.Pn);
    } else {
        hipLaunchKernelGGL(build_kernel, dim3(unsigned(ceil_div(n, 256)), unsigned(n)), dim3(256), 0, stream, H, n,
                           w.dfix, w.lam, w.A, w.V, w.Pn);
    }
    ONECOMP_CHECK_LAUNCH();

    const int nblk = int(ceil_div(n, NB));
    const bool wide = by_residues(n);
    if (wide && (st = factor_slabs(w, n, reinterpret_cast<char*>(U), info, stream)) != ONECOMP_OK) return st;

    // ---- blocked right-looking Cholesky of A (lower) ----
    // diagonal block 0 on its own; every later one inside the launch that updates the trailing matrix before it
    if (!wide) {
        hipLaunchKernelGGL(syrk_potrf_kernel<true>, dim3(1), dim3(POTRF_THREADS), 0, stream, w.A, w.V, w.Pn, w.Pk, n, -1, n, 1, 1,
                           0, 0, 0, info);
        ONECOMP_CHECK_LAUNCH();
    }
    // One step: panel solve below diagonal block s, then a trailing update fused with the factorization of diagonal
    // block s + 1.  The next step needs block column s + 1 only, so that one is updated at once and the others every
    // `lag` steps, by all panels solved since, in turn: a launch updates every lag-th column with k = 128 lag.  A rank-128
    // update of everything is bound by reading and writing the trailing matrix; the lag divides these bytes while
    // every launch keeps the same work to hide the next diagonal block behind.  The additions to a tile happen in
    // the same order whatever the lag, so the factor is bit-equal.
    // Narrow factors take the inverse along: once V[s, :] is known (the panel solve's launch), V[i, :] += L[i, s] V[s, :]
    // for the rows below, beside the trailing update, which leaves room in every launch the chain of diagonal blocks
    // bounds; V's blocks below the diagonal hold these sums until their row's turn.
    const bool along = !wide && form == ONECOMP_FACTOR_INVERSE && nblk <= plan::INVERSE_ALONG_MAX;
    int base = 0, lag = plan::syrk_lag(nblk);
    for (int s = 0; s < nblk && !wide; ++s) {
        const int rest = max(0, n - (s + 1) * NB), inv = along ? s : 0;
        hipLaunchKernelGGL(panel_kernel, dim3(PANEL_PAIRS + PANEL_UNITS + NB / TR * inv + unsigned(ceil_div(rest, TR))), dim3(256),
                           0, stream, w.A, w.V, w.V + int64_t(s) * NB * (n + 1), n, w.Pn, w.Pk, n, s, rest, PANEL_PAIRS, inv);
        ONECOMP_CHECK_LAUNCH();
        if (rest == 0) break;
        const int next_lag = plan::syrk_lag(nblk - 2 - s);
        const int stride = next_lag == lag ? lag : 1;   // where the lag changes every column is brought up to date
        if (lag == 1) {
            const int inv_cols = along ? 2 * (s + 1) : 0;
            hipLaunchKernelGGL(syrk_potrf_kernel<true>, dim3(unsigned(plan::syrk_narrow_grid(nblk - 1 - s, inv_cols))),
                               dim3(POTRF_THREADS), 0, stream, w.A, w.V, w.Pn, w.Pk, n, s, rest, 1, 1, s, inv_cols, 0, info);
        } else {
            hipLaunchKernelGGL(syrk_potrf_kernel<false>, dim3(unsigned(plan::syrk_grid(nblk - 1 - s, stride).total)),
                               dim3(POTRF_THREADS), 0, stream, w.A, w.V, w.Pn, w.Pk, n, s, rest, stride, lag, base, 0, 0, info);
        }
        ONECOMP_CHECK_LAUNCH();
        if (stride != lag) base = s + 1;
        lag = next_lag;
    }

    // ---- V = L^-1 by recursive doubling over aligned block pairs, from the diagonal blocks ----
    const size_t mat = align_up(size_t(n) * n * sizeof(double), 256);
    for (int64_t s = NB; s < n && form == ONECOMP_FACTOR_INVERSE && !along; s *= 2) {
        const int64_t pairs = ceil_div(n, 2 * s);
        // last pair may have a short or empty C range
        int64_t m_last = n - ((pairs - 1) * 2 * s + s);
        int64_t batch = pairs;
        if (m_last <= 0) { batch = pairs - 1; m_last = s; }
        if (batch <= 0) continue;
        if (m_last > s) m_last = s;
        const int64_t stride = 2 * s * (int64_t(n) + 1);
        // Row c of L carries channel c's scale and column c of V its inverse: the first product's terms are free of them, the
        // second one's operands are balanced.
        int32_t* const inner = reinterpret_cast<int32_t*>(w.dfix);
        int64_t first = 0;   // pairs that go by residues
        if (wide && s >= RESIDUE_INVERSE_MIN) {
            first = m_last >= RESIDUE_INVERSE_MIN_ROWS ? batch : batch - 1;
            if (first > 0 && (st = residue::inner_exponents(w.V, n, inner, stream)) != ONECOMP_OK) return st;
        }
        for (int64_t p = 0; p < first; ++p) {
            const int64_t o = 2 * s * p, m = p == batch - 1 ? m_last : s;
            double* const ca = w.V + (o + s) * n + o;
            // V[C,A] = L[C,A] V[A,A], then V[C,A] = -V[C,C] V[C,A]; U is free until the factor is written
            st = residue::triangular_product(w.A + (o + s) * n + o, n, w.V + o * (int64_t(n) + 1), n, ca, n, int(m), int(s), int(s), true,
                                             1.0, w.T, mat, U, size_t(n) * n * sizeof(float), nullptr,
                                             reinterpret_cast<int32_t*>(w.keys), w.perm, stream);
            if (st != ONECOMP_OK) return st;
            st = residue::triangular_product(w.V + (o + s) * (int64_t(n) + 1), n, ca, n, ca, n, int(m), int(s), int(m), false, -1.0, w.T,
                                             mat, U, size_t(n) * n * sizeof(float), inner + o + s,
                                             reinterpret_cast<int32_t*>(w.keys), w.perm, stream);
            if (st != ONECOMP_OK) return st;
        }
        if (first == batch) continue;
        const int64_t skip = first * stride;
        // T[C,A] = L[C,A] * V[A,A]        (V[A,A] lower triangular)
        GemmArgs a{};
        a.A = w.A + s * n + skip; a.lda = n; a.sa = stride;
        a.B = w.V + skip; a.ldb = n; a.sb = stride;
        a.C = w.T + s * n + skip; a.ldc = n; a.sc = stride;
        a.m = int(s); a.m_last = int(m_last); a.n = int(s); a.k = int(s); a.k_last = int(s); a.batch = int(batch - first);
        a.alpha = 1.0; a.beta = 0.0; a.flags = G_BLOWER;
        if ((st = dgemm(a, stream)) != ONECOMP_OK) return st;
        // V[C,A] = -V[C,C] * T[C,A]       (V[C,C] lower triangular)
        GemmArgs b{};
        b.A = w.V + s * (int64_t(n) + 1) + skip; b.lda = n; b.sa = stride;
        b.B = w.T + s * n + skip; b.ldb = n; b.sb = stride;
        b.C = w.V + s * n + skip; b.ldc = n; b.sc = stride;
        b.m = int(s); b.m_last = int(m_last); b.n = int(s); b.k = int(s); b.k_last = int(m_last); b.batch = int(batch - first);
        b.alpha = -1.0; b.beta = 0.0; b.flags = G_ALOWER;
        if ((st = dgemm(b, stream)) != ONECOMP_OK) return st;
    }

    if (form == ONECOMP_FACTOR_BLOCK) {   // V's diagonal blocks, the rest comes from L itself
        hipLaunchKernelGGL(rdiag_kernel, dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, stream, w.V, n, w.dfix);
        ONECOMP_CHECK_LAUNCH();
        hipLaunchKernelGGL(output_block_kernel, dim3(unsigned(ceil_div(n, 256)), unsigned(n)), dim3(256), 0, stream, w.A,
                           w.V, w.dfix, n, U);
        ONECOMP_CHECK_LAUNCH();
        return ONECOMP_OK;
    }

    hipLaunchKernelGGL(output_kernel, dim3(unsigned(ceil_div(n, 256)), unsigned(n)), dim3(256), 0, stream, w.V, n, U);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

}  // namespace onecomp
