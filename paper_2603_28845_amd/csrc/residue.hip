// fp64 products on the 8-bit integer matrix cores, by residues.
//
// The entries of an fp64 row are scaled by a power of two and rounded to integers, multiples of 2^-54.4 of the row's norm (the
// largest entries keep 53 bits and more, those a thousandth of the norm 44, with none below 2^-55).  The product of two such
// rows is an integer below M / 2, M the product of MODULI pairwise coprime moduli of 8 bits, so it is known from its
// residues (Chinese remainder theorem), and these are products of 8-bit residues: one v_mfma_i32_32x32x32_i8 product per
// modulus, exact in 32 bits.  (The route of K. Ozaki, Y. Uchino and T. Imamura, "Ozaki scheme II", 2025.)  What is rounded:
// each entry once, by at most half a unit, and the result once.  With a and b the rows' norms the sum is off by 0.4 2^-54 a b
// in the root mean square whatever the length, less than a chain of fp64 additions leaves (measured against 80-bit sums:
// 0.23 to 0.67 of its error at lengths of 1024 to 8192).  That is an error against the norms: a sum far below them, whose terms are
// too, keeps fewer of its own digits than in fp64.  Gram matrices are no such case: entries of U that are not the rounded exact
// ones, in fp64 : so, activations with outlier channels, damping 1e-2, d_in 8192 1.9e-6 : 1.2e-6, 14336 2.4e-6 : 1.4e-6, 28672
// 3.3e-6 : 1.9e-6 (block form 1.3e-6 : 0.8e-6); 8192, half rank, damping 1e-2 1.6e-5 : 0.9e-5, 1e-4 9.4e-4 : 5.3e-4, 2e-5
// 3.9e-3 : 2.3e-3; full rank, channels of log-normal scales 3.9e-7 : 4.8e-7.  Factors that decay away from the diagonal are: H = 0.9^|i - j| has as many digits in every
// entry above 1e-6 of its row's norm, wrong ones further down (all entries: 4.6 % : 7.5 % not the rounded ones).
//
// Why: the fp64 matrix rate is 77 TFLOP/s; 14 products at the 8-bit rate (3.6 POP/s in registers, 2.3 in a product out of
// L2) are 165 at inner ranges of 8192, 120 to 135 at 2048 and in products of few tiles.  To this the conversions add about
// 8 + 14 bytes per operand entry and 2 x 14 + 16 per result, so the inner range has to be long.
//
// Scales: row a gets the largest s with |a|^2 4^s <= 2^BOUND_LOG2 (BOUND below M / 2 by a tenth, for what rounding adds).
#include "residue.hpp"
#include <type_traits>

namespace onecomp {
namespace residue {
namespace {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef int int16v __attribute__((ext_vector_type(16)));

struct DeviceTables {
    int m[MODULI];
    float inv[MODULI];
};
constexpr DeviceTables device_tables() {
    DeviceTables t{};
    for (int i = 0; i < MODULI; ++i) {
        t.m[i] = MOD[i];
        t.inv[i] = TAB.inv[i];
    }
    return t;
}
__constant__ DeviceTables d_tab = device_tables();   // where the modulus is known at run time only

// 16 entries of one row, scaled by 2^s -> 16 bytes per modulus at dst, dst + plane, ...
// Conversions of fp64 to integers and back instead, and the compiler's choice of products: 120 vector instructions an entry,
// 30 of them fp64 at a quarter of the rate; now 100.
__device__ __forceinline__ void convert_piece(const double (&x)[16], char* __restrict__ dst, int64_t plane) {
    int n0[16], n1[16], n2[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) split_entry(x[e], n0[e], n1[e], n2[e]);
#pragma unroll
    for (int i = 0; i < MODULI; ++i) {
        uint4v w;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = entry_residue(n0[4 * q + e], n1[4 * q + e], n2[4 * q + e], i);
            // the low bytes of the four
            const uint32_t lo = __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), hi = __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu);
            w[q] = lo | hi;
        }
        *reinterpret_cast<uint4v*>(dst + i * plane) = w;
    }
}
// 2^e for the exponents that scales have
__device__ __forceinline__ double power(int e) { return __builtin_ldexp(1.0, e); }
// where entries [k, k + 16) of row `row` go inside a plane
__device__ __forceinline__ int64_t piece_offset(int row, int k, int64_t block) {
    return int64_t(row >> 5) * block + (k >> 5) * 1024 + ((k >> 4) & 1) * 512 + (row & 31) * 16;
}

__global__ __launch_bounds__(256) void row_bounds_kernel(const double* __restrict__ A, int n, int32_t* __restrict__ shift,
                                                        double* __restrict__ left) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double d = A[int64_t(i) * (n + 1)];
    left[i] = d;
    shift[i] = d > 0.0 ? shift_of(d) : NO_SHIFT;
}

// A workgroup takes 32 rows; 128 columns at a time come in along the rows and go through LDS, from which a lane takes 16
// entries of a row (32 lanes x 16 bytes of pitch 1040: 64 different banks).  Straight from memory, 128 bytes a lane, the
// lines a wave touches do not stay in the first-level cache: 16 ps an entry against 8.
constexpr int CV_COLS = 128, CV_PITCH = CV_COLS + 2;
__device__ __forceinline__ void stage_rows(const double* __restrict__ src, int64_t ld, int rows_ok, int cols_ok, double* tile,
                                           const int32_t* __restrict__ inner = nullptr) {
    const int r = threadIdx.x >> 6, c = (threadIdx.x & 63) * 2;
    const double p0 = power(inner && c < cols_ok ? inner[c] : 0), p1 = power(inner && c < cols_ok ? inner[c + 1] : 0);
    double2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        v[q] = make_double2(0.0, 0.0);
        if (r + 4 * q < rows_ok && c < cols_ok) v[q] = *reinterpret_cast<const double2*>(src + int64_t(r + 4 * q) * ld + c);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (inner) v[q] = make_double2(v[q].x * p0, v[q].y * p1);
        *reinterpret_cast<double2*>(tile + (r + 4 * q) * CV_PITCH + c) = v[q];
    }
}
__device__ __forceinline__ void take_piece(const double* tile, double (&x)[16]) {
    const double* p = tile + (threadIdx.x & 31) * CV_PITCH + (threadIdx.x >> 5) * 16;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const double2 v = *reinterpret_cast<const double2*>(p + 2 * q);
        x[2 * q] = v.x;
        x[2 * q + 1] = v.y;
    }
}
// sum over the eight threads of a row, the same in each of them
__device__ __forceinline__ double row_sum(double s, double* part) {
    const int r = threadIdx.x & 31, seg = threadIdx.x >> 5;
    __syncthreads();
    part[seg * 32 + r] = s;
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s += part[q * 32 + r];
    return s;
}

__global__ __launch_bounds__(256) void convert_columns_kernel(const double* __restrict__ L, int n, int r0, int c0, int width,
                                                             int32_t* __restrict__ shift, double* __restrict__ left,
                                                             Operand R) {
    __shared__ __align__(16) double tile[32 * CV_PITCH];
    __shared__ double part[256];
    const int row0 = r0 + blockIdx.x * 32, row = row0 + (threadIdx.x & 31), seg = threadIdx.x >> 5;
    const double* const src = L + int64_t(row0) * n + c0;
    double x[16], s = 0.0;
    for (int c = 0; c < width; c += CV_COLS) {
        __syncthreads();
        stage_rows(src + c, n, n - row0, width - c, tile);
        __syncthreads();
        take_piece(tile, x);
#pragma unroll
        for (int e = 0; e < 16; ++e) s = __builtin_fma(x[e], x[e], s);
    }
    int32_t sh = row < n ? shift[row] : NO_SHIFT;
    s = row_sum(s, part);
    const double rest = row < n ? left[row] - s : 0.0;
    // beyond the diagonal entry by more than rounding: the row's own pivot will not be positive, nothing is bounded
    if (sh != NO_SHIFT && !(__builtin_ldexp(rest, 2 * sh) > -0x1p98)) sh = NO_SHIFT;
    __syncthreads();   // every thread of the row has read both
    if (seg == 0 && row < n) {
        left[row] = rest;
        shift[row] = sh;
    }
    const double scale = power(sh == NO_SHIFT ? 0 : sh);
    for (int c = 0; c < width; c += CV_COLS) {
        __syncthreads();
        stage_rows(src + c, n, n - row0, width - c, tile);
        __syncthreads();
        take_piece(tile, x);
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = sh == NO_SHIFT ? 0.0 : x[e] * scale;
        const int k = c0 + c + seg * 16;
        if (c + seg * 16 < width) convert_piece(x, R.data + piece_offset(row, k, R.block), R.plane);
    }
}

// Rows of a matrix whose norms are known, a workgroup per 32 rows and 512 columns.  lower: entries right of the diagonal
// count as zero whatever they hold (up to the end of the rows' 256-wide tile they are read all the same); columns that no
// product tile of these rows takes are not written.  inner, here and below:
// column k of the left operand counts 2^inner[k] times, row k of the right one 2^-inner[k] times (nullptr: 1).
constexpr int CV_CHUNK = 512;
__global__ __launch_bounds__(256) void convert_rows_kernel(const double* __restrict__ src, int64_t ld, int rows, int k_len,
                                                          int lower, const int32_t* __restrict__ inner,
                                                          const int32_t* __restrict__ shift, Operand R) {
    __shared__ __align__(16) double tile[32 * CV_PITCH];
    const int row0 = blockIdx.x * 32, row = row0 + (threadIdx.x & 31), seg = threadIdx.x >> 5;
    const int k_end = min(min(int(R.block >> 5), int(blockIdx.y + 1) * CV_CHUNK), lower ? (row0 / TILE + 1) * TILE : INT32_MAX);
    const int32_t sh = row < rows ? shift[row] : NO_SHIFT;
    const double scale = power(sh == NO_SHIFT ? 0 : sh);
    double x[16];
    for (int k0 = blockIdx.y * CV_CHUNK; k0 < k_end; k0 += CV_COLS) {
        __syncthreads();
        stage_rows(src + int64_t(row0) * ld + k0, ld, rows - row0, k_len - k0, tile, inner ? inner + k0 : nullptr);
        __syncthreads();
        take_piece(tile, x);
        const int k = k0 + seg * 16;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            x[e] = sh == NO_SHIFT || (lower && k + e > row) ? 0.0 : x[e] * scale;
        if (k < k_end) convert_piece(x, R.data + piece_offset(row, k, R.block), R.plane);
    }
}
// Columns [c0, c0 + cols) of a matrix of k_len rows and n columns, as rows of R; partial: column_norm_kernel's.  lower: the
// matrix is lower triangular.
__global__ __launch_bounds__(256) void convert_transposed_kernel(const double* __restrict__ src, int64_t ld, int c0, int cols,
                                                                int k_len, int lower, const int32_t* __restrict__ inner,
                                                                const double* __restrict__ partial, int n,
                                                                int32_t* __restrict__ shift, Operand R) {
    const int r = blockIdx.x * 32 + (threadIdx.x & 31), seg = threadIdx.x >> 5, col = c0 + r;
    const int k_end = min(int(R.block >> 5), int(blockIdx.y + 1) * CV_CHUNK);
    const int k_begin = lower ? (c0 + int(blockIdx.x) * 32) / TILE * TILE : 0;
    int32_t sh = NO_SHIFT;
    if (r < cols) {
        double norm = 0.0;
        for (int y = 0; y * CV_CHUNK < k_len; ++y) norm += partial[int64_t(y) * n + col];
        sh = shift_of(norm);
        if (blockIdx.y == 0 && seg == 0) shift[col] = sh;
    }
    const int s = sh == NO_SHIFT ? 0 : sh;
    for (int k = blockIdx.y * CV_CHUNK + seg * 16; k < k_end; k += 128) {
        if (k < k_begin) continue;
        double x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            x[e] = 0.0;
            if (sh != NO_SHIFT && k + e < k_len && !(lower && k + e < col)) x[e] = src[int64_t(k + e) * ld + col];
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = x[e] * (inner && k + e < k_len ? power(s - inner[k + e]) : power(s));
        convert_piece(x, R.data + piece_offset(r, k, R.block), R.plane);
    }
}

// scales of the rows of a matrix, a wave per row; lower as above
__global__ __launch_bounds__(256) void row_shift_kernel(const double* __restrict__ src, int64_t ld, int rows, int k_len, int lower,
                                                       const int32_t* __restrict__ inner, int32_t* __restrict__ shift) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= rows) return;
    const int end = lower ? min(k_len, row + 1) : k_len;
    double s = 0.0;
#pragma unroll 8
    for (int k = lane; k < end; k += 64) {
        const double v = src[int64_t(row) * ld + k] * (inner ? power(inner[k]) : 1.0);
        s = __builtin_fma(v, v, s);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) shift[row] = shift_of(s);
}
// partial[y][col]: squares of column `col` in rows [512 y, 512 y + 512); lower as above
__global__ __launch_bounds__(256) void column_norm_kernel(const double* __restrict__ src, int64_t ld, int cols, int k_len, int lower,
                                                         const int32_t* __restrict__ inner, double* __restrict__ partial) {
    __shared__ double part[4][64];
    const int l = threadIdx.x & 63, seg = threadIdx.x >> 6, col = blockIdx.x * 64 + l;
    const int k1 = min(k_len, int(blockIdx.y + 1) * CV_CHUNK);
    double s = 0.0;
    if (col < cols) {
#pragma unroll 8
        for (int k = max(int(blockIdx.y) * CV_CHUNK, lower ? int(blockIdx.x) * 64 : 0) + seg; k < k1; k += 4) {
            const double v = lower && k < col ? 0.0 : src[int64_t(k) * ld + col] * (inner ? power(-inner[k]) : 1.0);
            s = __builtin_fma(v, v, s);
        }
    }
    part[seg][l] = s;
    __syncthreads();
    if (seg == 0 && col < cols) partial[int64_t(blockIdx.y) * cols + col] = (part[0][l] + part[1][l]) + (part[2][l] + part[3][l]);
}

__global__ __launch_bounds__(256) void inner_exponents_kernel(const double* __restrict__ V, int n, int32_t* __restrict__ inner) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double d = V[int64_t(i) * (n + 1)];
    int e = 0;
    if (d > 0.0 && d < __builtin_inf()) __builtin_frexp(d, &e);
    inner[i] = -e;
}

// Columns of B taken at a time: few enough that their residues and those of the product stay in the 256 MB cache behind the
// L2s for the most part, enough tiles to fill the chip.
constexpr int64_t PIECE_COLS = 2048;

// ---- the products -----------------------------------------------------------------------------------------------------
// out = A B^T mod m for every modulus m, A and B by their residues: 256 x 256 tile per workgroup, four waves of 128 x 128, one
// per SIMD (256 accumulators in AGPRs); both operands are in operand order, so a load is 1 KB of memory -> 1 KB of LDS and a
// fragment is one conflict-free 16-byte read.  Steps of 64 through a ring of four slots of 32 KB; the operands of a step's first
// half are read before the barrier that publishes the next step's, and reads and loads stand one by one behind MFMAs, so that
// with a single wave per SIMD no MFMA waits for them.  In long launches the chip's power is the bound (4.3 ms at d_in 28672: MFMAs busy
// 82 % of the cycles at 1.48 GHz, 2.54 POP/s; 0.3 ms: 43 to 60 % at 2.0 to 1.85 GHz, 1.9 to 2.35 POP/s, which start and end of a tile
// take), so what counts is bytes out of LDS per product: these waves read two thirds of what eight of 128 x 64 did.
// A factor's products, us, eight waves : four: d_in 28672 91.7 : 87.4 ms (inner ranges of 8192 2171 : 2010, 2048 963 : 950, 1024
// 494 : 508), 14336 in block form 5785 : 5643.
// Accumulators start at 2^22 m, so they stay positive and below 2^31 (margins_hold).
// Workgroup -> tile: patches of 32 tiles, each with one modulus, go round the XCDs (workgroup b runs on XCD b % 8), so that
// the 32 tiles an XCD works on share their operands in its L2; with a triangular operand the longest patches come first.
enum : int { FULL = 0, SYRK = 1, LOWER_B = 2, LOWER_A = 3 };
struct ProductArgs {
    const char *A, *B;
    char* out;                       // [modulus][row / 4][column][row % 4]
    int64_t a_plane, b_plane, out_plane, a_block, b_block;
    int m_t, n_t, stages, shape, out_cols, patch_cols;
    int k0;                          // LOWER_B: first stage of tile column 0
};
constexpr int STAGE_BYTES = 2 * TILE * K_STEP, SLOTS = 4;

__global__ __launch_bounds__(256, 1) void product_kernel(ProductArgs g) {
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave >> 1, wc = wave & 1;
    const int patch_rows = 32 / g.patch_cols;
    const int unit = int(blockIdx.x >> 8) * 8 + int(blockIdx.x & 7), w = (blockIdx.x >> 3) & 31;
    const int patch = unit / MODULI, mod = unit % MODULI;
    const int p_r = (g.m_t + patch_rows - 1) / patch_rows, p_c = (g.n_t + g.patch_cols - 1) / g.patch_cols;
    if (patch >= p_r * p_c) return;
    const int pr = g.shape == LOWER_A ? p_r - 1 - patch / p_c : patch % p_r;
    const int pc = g.shape == LOWER_A ? patch % p_c : patch / p_r;
    const int tm = __builtin_amdgcn_readfirstlane(pr * patch_rows + w % patch_rows);
    const int tn = __builtin_amdgcn_readfirstlane(pc * g.patch_cols + w / patch_rows);
    if (tm >= g.m_t || tn >= g.n_t || (g.shape == SYRK && tn > tm)) return;
    const int begin = g.shape == LOWER_B ? g.k0 + tn * (TILE / K_STEP) : 0;
    const int end = g.shape == LOWER_A ? min(g.stages, (tm + 1) * (TILE / K_STEP)) : g.stages;
    const int n_st = end - begin;

    const uint32_t lds0 = uint32_t(uintptr_t((ONECOMP_LDS char*)lds)), lane16 = lane * 16;
    // a wave requests two row blocks of either operand, 2 KB each per step
    const char* pa = g.A + mod * g.a_plane + (tm * 8 + wave * 2) * g.a_block + int64_t(begin) * 2048;
    const char* pb = g.B + mod * g.b_plane + (tn * 8 + wave * 2) * g.b_block + int64_t(begin) * 2048;
    int ahead = n_st;   // steps not requested yet; past the end: an empty range, which deposits zeros
    struct Desc {
        __amdgpu_buffer_rsrc_t a[2], b[2];
        uint32_t lds;
    };
    auto next_desc = [&](int slot) __attribute__((always_inline)) {
        const uint32_t range = ahead > 0 ? 0x7FFFFFFFu : 0u;
        --ahead;
        Desc d;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            d.a[q] = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(pa + q * g.a_block), 0, range, 0x00020000);
            d.b[q] = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(pb + q * g.b_block), 0, range, 0x00020000);
        }
        d.lds = lds0 + slot * STAGE_BYTES + wave * 4096;
        pa += 2048;
        pb += 2048;
        return d;
    };
    auto load = [&](const Desc& d, int i) __attribute__((always_inline)) {   // number i of a step's eight
        const int q = i >> 2, half = i & 1;
        if (i & 2) lds_load16(d.lds + STAGE_BYTES / 2 + q * 2048 + half * 1024, lane16 + half * 1024, d.b[q]);
        else lds_load16(d.lds + q * 2048 + half * 1024, lane16 + half * 1024, d.a[q]);
    };
    auto issue = [&](int slot) __attribute__((always_inline)) {
        const Desc d = next_desc(slot);
#pragma unroll
        for (int i = 0; i < 8; ++i) load(d, i);
    };
    for (int st = 0; st < SLOTS - 1; ++st) issue(st);
    const int m = d_tab.m[mod];
    int16v acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = m << 22;
    struct Frags {
        int4v a[4], b[4];
    };
    Frags F0, F1;
    const char* const fa = lds + wr * 4 * 2048 + lane16;
    const char* const fb = lds + STAGE_BYTES / 2 + wc * 4 * 2048 + lane16;
    auto read = [&](Frags& f, int r, int off) __attribute__((always_inline)) {   // fragment r of eight, as the products take them
        if (r & 1) f.b[r >> 1] = *reinterpret_cast<const int4v*>(fb + off + (r >> 1) * 2048);
        else f.a[r >> 1] = *reinterpret_cast<const int4v*>(fa + off + (r >> 1) * 2048);
    };
    // sixteen MFMAs; `between(i)` goes behind number i
    auto multiply = [&](const Frags& f, auto&& between) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            const int i = n >> 2, j = i & 1 ? 3 - (n & 3) : n & 3;   // one operand stays from one MFMA to the next
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
            between(n);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(8 * (SLOTS - 2)));
    __syncthreads();
    issue(SLOTS - 1);
#pragma unroll
    for (int r = 0; r < 8; ++r) read(F0, r, 0);
    auto stage = [&](auto slot_c) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value, next = (slot + 1) % SLOTS;
        multiply(F0, [&](int n) __attribute__((always_inline)) {
            if (n < 8) read(F1, n, slot * STAGE_BYTES + 1024);
        });
        // the next step has landed; every wave has read this one
        __builtin_amdgcn_s_waitcnt(wait_vmcnt(8 * (SLOTS - 2)));
        __syncthreads();
        const Desc d = next_desc(slot);
        multiply(F1, [&](int n) __attribute__((always_inline)) {
            if (n & 1) load(d, n >> 1);
            else read(F0, n >> 1, next * STAGE_BYTES);
        });
    };
    int st = 0;
#pragma unroll 1
    for (; st + SLOTS <= n_st; st += SLOTS) {
        stage(std::integral_constant<int, 0>{});
        stage(std::integral_constant<int, 1>{});
        stage(std::integral_constant<int, 2>{});
        stage(std::integral_constant<int, 3>{});
    }
    if (st < n_st) stage(std::integral_constant<int, 0>{});
    if (st + 1 < n_st) stage(std::integral_constant<int, 1>{});
    if (st + 2 < n_st) stage(std::integral_constant<int, 2>{});
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));   // no LDS write may be in flight when the workgroup ends

    const float inv = d_tab.inv[mod];
    const int l32 = lane & 31, lh = lane >> 5;
    uint32_t* const o = reinterpret_cast<uint32_t*>(g.out + mod * g.out_plane) + int64_t(tm * (TILE / 4) + wr * 32 + lh) * g.out_cols +
                        tn * TILE + wc * 128 + l32;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t r[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) r[e] = sum_residue(acc[i][j][4 * q + e], m, inv);
                o[int64_t(i * 8 + 2 * q) * g.out_cols + j * 32] = r[0] | r[1] << 8 | r[2] << 16 | r[3] << 24;
            }
}

// C = beta C + alpha x from x's residues; a thread has four rows of a column.  copy: see update_columns.
__global__ __launch_bounds__(256) void reconstruct_kernel(const char* __restrict__ res, int64_t plane, int res_cols, int rows,
                                                         int cols, const int32_t* __restrict__ sa,
                                                         const int32_t* __restrict__ sb, double* __restrict__ C, int64_t ldc,
                                                         double scale, int syrk, double* __restrict__ copy) {
    const int col = blockIdx.x * 256 + threadIdx.x, row0 = blockIdx.y * 4;
    if (col >= cols || (syrk && int(blockIdx.x) > row0 / TILE)) return;
    const char* const p = res + (int64_t(blockIdx.y) * res_cols + col) * 4;
    uint32_t w[MODULI];
#pragma unroll
    for (int i = 0; i < MODULI; ++i) w[i] = *reinterpret_cast<const uint32_t*>(p + i * plane);
    double c[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) c[e] = syrk && row0 + e < rows ? C[int64_t(row0 + e) * ldc + col] : 0.0;
    const int32_t eb = sb[col];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = row0 + e;
        if (row >= rows) break;
        Fraction f;
#pragma unroll
        for (int i = 0; i < MODULI; ++i) f.add((w[i] >> (8 * e)) & 255u, i);
        double v = unscaled(f.value() * scale, sa[row], eb);
        v += c[e];
        C[int64_t(row) * ldc + col] = v;
        if (copy && row >= 128 && row < 256 && col < 128) copy[(row - 128) * 128 + col] = v;
    }
}

onecomp_status product(const Operand& A, const Operand& B, int m, int n, int k, int shape, int k0, char* out, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    onecomp_status st = allow_dynamic_lds(reinterpret_cast<const void*>(product_kernel), SLOTS * STAGE_BYTES, lds_set);
    if (st != ONECOMP_OK) return st;
    ProductArgs g{};
    g.A = A.data; g.B = B.data; g.out = out;
    g.a_plane = A.plane; g.b_plane = B.plane; g.out_plane = pad_rows(m) * pad_rows(n);
    g.a_block = A.block; g.b_block = B.block;
    g.m_t = int(pad_rows(m) / TILE); g.n_t = int(pad_rows(n) / TILE);
    g.stages = int(pad_k(k) / K_STEP); g.shape = shape; g.out_cols = int(pad_rows(n)); g.k0 = k0;
    g.patch_cols = g.n_t >= 8 ? 8 : g.n_t >= 4 ? 4 : g.n_t >= 2 ? 2 : 1;
    const int64_t units = ceil_div(g.m_t, 32 / g.patch_cols) * ceil_div(g.n_t, g.patch_cols) * MODULI;
    hipLaunchKernelGGL(product_kernel, dim3(unsigned(ceil_div(units, 8) * 256)), dim3(256), SLOTS * STAGE_BYTES, stream, g);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}
onecomp_status reconstruct(const char* res, int m, int n, const int32_t* sa, const int32_t* sb, double* C, int64_t ldc, double alpha,
                           int syrk, double* copy, hipStream_t stream) {
    hipLaunchKernelGGL(reconstruct_kernel, dim3(unsigned(ceil_div(n, 256)), unsigned(ceil_div(m, 4))), dim3(256), 0, stream, res,
                       pad_rows(m) * pad_rows(n), int(pad_rows(n)), m, n, sa, sb, C, ldc, alpha * TAB.M, syrk, copy);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

}  // namespace

onecomp_status row_bounds(const double* A, int n, int32_t* shift, double* left, hipStream_t stream) {
    hipLaunchKernelGGL(row_bounds_kernel, dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, stream, A, n, shift, left);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

onecomp_status inner_exponents(const double* V, int n, int32_t* inner, hipStream_t stream) {
    hipLaunchKernelGGL(inner_exponents_kernel, dim3(unsigned(ceil_div(n, 256))), dim3(256), 0, stream, V, n, inner);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

onecomp_status convert_columns(const double* L, int n, int r0, int c0, int width, int32_t* shift, double* left, const Operand& R,
                               hipStream_t stream) {
    hipLaunchKernelGGL(convert_columns_kernel, dim3(unsigned(ceil_div(n - r0, 32))), dim3(256), 0, stream, L, n, r0, c0, width,
                       shift, left, R);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

onecomp_status update_columns(double* A, int n, int c0, int width, const int32_t* shift, const Operand& R, double* copy,
                              void* scratch, hipStream_t stream) {
    char* const out = static_cast<char*>(scratch);
    const Operand P = R.from(c0);
    const onecomp_status st = product(P, P, n - c0, width, c0, SYRK, 0, out, stream);
    if (st != ONECOMP_OK) return st;
    return reconstruct(out, n - c0, width, shift + c0, shift + c0, A + int64_t(c0) * (n + 1), n, -1.0, 1, copy, stream);
}

onecomp_status triangular_product(const double* A, int64_t lda, const double* B, int64_t ldb, double* C, int64_t ldc, int m, int n,
                                  int k, bool lower_b, double alpha, void* operands, size_t operand_len, void* product_mem,
                                  size_t product_len, const int32_t* inner, int32_t* shift_a, int32_t* shift_b, hipStream_t stream) {
    // scratch: the columns' partial norms, the residues of A, those of as many columns of B as there is room for
    const unsigned chunks = unsigned(ceil_div(pad_k(k), CV_CHUNK));
    double* const partial = static_cast<double*>(operands);
    const size_t len_p = align_up(size_t(chunks) * n * sizeof(double), 256), len_a = align_up(operand_bytes(m, k), 256);
    int64_t piece = n < PIECE_COLS ? pad_rows(n) : PIECE_COLS;
    auto fits = [&]() {
        return len_p + len_a + operand_bytes(piece, k) <= operand_len && product_bytes(m, piece) <= product_len;
    };
    while (piece > TILE && !fits()) piece -= TILE;
    if (!fits() || k > MAX_K) return ONECOMP_ERR_UNSUPPORTED;
    const Operand RA(static_cast<char*>(operands) + len_p, m, k);
    hipLaunchKernelGGL(row_shift_kernel, dim3(unsigned(ceil_div(m, 4))), dim3(256), 0, stream, A, lda, m, k, int(!lower_b), inner,
                       shift_a);
    ONECOMP_CHECK_LAUNCH();
    hipLaunchKernelGGL(convert_rows_kernel, dim3(unsigned(ceil_div(m, 32)), chunks), dim3(256), 0, stream, A, lda, m, k,
                       int(!lower_b), inner, shift_a, RA);
    ONECOMP_CHECK_LAUNCH();
    hipLaunchKernelGGL(column_norm_kernel, dim3(unsigned(ceil_div(n, 64)), unsigned(ceil_div(k, CV_CHUNK))), dim3(256), 0, stream, B, ldb,
                       n, k, int(lower_b), inner, partial);
    ONECOMP_CHECK_LAUNCH();
    char* const out = static_cast<char*>(product_mem);
    for (int64_t c0 = 0; c0 < n; c0 += piece) {
        const int cols = int(n - c0 < piece ? n - c0 : piece);
        const Operand RB(static_cast<char*>(operands) + len_p + len_a, cols, k);
        hipLaunchKernelGGL(convert_transposed_kernel, dim3(unsigned(ceil_div(cols, 32)), chunks), dim3(256), 0, stream, B, ldb,
                           int(c0), cols, k, int(lower_b), inner, partial, n, shift_b, RB);
        ONECOMP_CHECK_LAUNCH();
        onecomp_status st = product(RA, RB, m, cols, k, lower_b ? LOWER_B : LOWER_A, int(c0 / K_STEP), out, stream);
        if (st != ONECOMP_OK) return st;
        st = reconstruct(out, m, cols, shift_a, shift_b + c0, C + c0, ldc, alpha, 0, nullptr, stream);
        if (st != ONECOMP_OK) return st;
    }
    return ONECOMP_OK;
}

}  // namespace residue
}  // namespace onecomp
