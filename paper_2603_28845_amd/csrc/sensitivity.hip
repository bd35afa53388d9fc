// Activation-aware sensitivity of one layer under a candidate quantization configuration (Sec. 4.1 of the
// paper, "AutoBit"): the weight perturbation dW = W^ - W of a fast round-to-nearest (RTN) proxy, weighted by the
// diagonals of the Kronecker-factored curvature,
//     err = 1/2 tr(B dW A dW^T)  ->  1/2 sum_r sum_c b_r a_c dW_rc^2      (A, B diagonal, as the paper uses them)
// in this library's d_out x d_in storage (a over input channels, b over output rows).  The RTN proxy rounds
// every group of G consecutive input channels of a row to its own grid (Eq. (1), (2) or (3), (4)), no feedback.
//
// gfx950: W is read once from HBM.  A team of TS <= 64 lanes of one wave owns a group at a time, 16 bytes per lane and
// load.  Per-workgroup partial sums are combined in a fixed order: bit-wise reproducible.
// Once W comes in at full width the kernel is bound by its VALU operations: with eight weights of a group per lane 24 per
// weight at 4096 x 4096 bf16 in groups of 64 and 128 (counted by SQ_INSTS_VALU), nine of them the weight's own (unpacking,
// range, rounding, sum), the rest what a group costs every lane of its team: the reduction of the range, two divisions and a
// reciprocal, addresses.  So a lane takes 16 weights of a group where there are as many (sensitivity_run), and that rest is
// kept small: a group of up to two (fp32: four) loads per lane stays in registers between the pass for min / max
// and the one that rounds (wider groups read it again, from cache), the lanes of a row of 16 meet through DPP operands,
// the position in the matrix advances by additions (a 64-bit division per group cost more than the group's arithmetic),
// and the grid is a multiple of the groups of a row where it can be, so that a team keeps its slice of `a`.
// 4096 x 4096 bf16, G 64 / 128, us of a call with eight and with 16 weights per lane: 14.0 -> 12.3.
#include "common.hpp"

namespace onecomp {
namespace {

// V consecutive elements (16 bytes) as floats
template <typename T>
struct Vec;
template <>
struct Vec<float> {
    static constexpr int V = 4;
    static __device__ inline void load(const float* p, float (&v)[4]) {
        const float4v x = *reinterpret_cast<const float4v*>(p);
        v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
    }
};
template <>
struct Vec<uint16_t> {
    static constexpr int V = 8;
    static __device__ inline void load(const uint16_t* p, float (&v)[8]) {
        const uint4v x = *reinterpret_cast<const uint4v*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __uint_as_float(x[e] << 16);
            v[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
        }
    }
};

struct SensArgs {
    const void* W;
    const float* a;      // [d_in]
    const float* b;      // [d_out] or nullptr (ones)
    float* partial;      // [gridDim.x]
    int64_t n_groups;    // d_out * d_in / G
    int d_in, G, n_g, ts;
    float qmax, qs;      // highest code; qs > 0: symmetric grid with zero-point qs
};

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}

// minimum and maximum over a team of ts lanes (a power of two, teams aligned), left in every lane
__device__ __forceinline__ void team_range(float& mn, float& mx, int ts) {
    auto step = [&](float a, float b) __attribute__((always_inline)) { mn = fminf(mn, a); mx = fmaxf(mx, b); };
    step(dpp_f<0xB1>(mn), dpp_f<0xB1>(mx));                     // lane ^ 1
    if (ts >= 4) step(dpp_f<0x4E>(mn), dpp_f<0x4E>(mx));        // lane ^ 2
    if (ts >= 8) step(dpp_f<0x141>(mn), dpp_f<0x141>(mx));      // mirrored in 8 lanes: the other quad
    if (ts >= 16) step(dpp_f<0x140>(mn), dpp_f<0x140>(mx));     // mirrored in 16 lanes: the other half
    for (int off = 16; off < ts; off *= 2) step(__shfl_xor(mn, off, 64), __shfl_xor(mx, off, 64));
}

__device__ __forceinline__ void load_a(const float* p, float4v (&a)[1]) { a[0] = *reinterpret_cast<const float4v*>(p); }
__device__ __forceinline__ void load_a(const float* p, float4v (&a)[2]) {
    a[0] = *reinterpret_cast<const float4v*>(p);
    a[1] = *reinterpret_cast<const float4v*>(p + 4);
}

// K: loads per lane that hold a whole group (G <= K ts V); 0: any group, read twice
template <typename T, int K>
__global__ __launch_bounds__(256) void sens_kernel(SensArgs g) {
    constexpr int V = Vec<T>::V, KR = K > 0 ? K : 1;
    __shared__ float team_sum[128];
    const T* W = static_cast<const T*>(g.W);
    const int tid = threadIdx.x;
    const int ts = g.ts;                         // lanes per team, a power of two in 2 .. 64; a lane takes V elements
    const int team = tid / ts, tl = tid % ts, teams = 256 / ts;
    const int total = int(gridDim.x) * teams;    // at most 2048 x 128
    int64_t gi = int64_t(blockIdx.x) * teams + team;
    int64_t row = unsigned(gi) / unsigned(g.n_g);
    int gc = int(unsigned(gi) % unsigned(g.n_g));    // the group's place in its row
    const int row_step = total / g.n_g, gc_step = total % g.n_g;
    float acc = 0.f;
    float v[KR][V];
    float4v av[KR][V / 4];
    auto fetch = [&](const T* wp, float (&x)[KR][V]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tl * V + k * ts * V < g.G) Vec<T>::load(wp + tl * V + k * ts * V, x[k]);
    };
    auto fetch_a = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tl * V + k * ts * V < g.G) load_a(g.a + c0 + tl * V + k * ts * V, av[k]);
    };
    if (gi < g.n_groups) {
        fetch(W + row * g.d_in + gc * g.G, v);
        fetch_a(gc * g.G);
    }
    while (gi < g.n_groups) {
        const int c0 = gc * g.G;
        const T* wp = W + row * g.d_in + c0;
        const float br = g.b ? g.b[row] : 1.0f;
        gi += total; row += row_step; gc += gc_step;
        if (gc >= g.n_g) { gc -= g.n_g; ++row; }
        float nv[KR][V];
        if (gi < g.n_groups) fetch(W + row * g.d_in + gc * g.G, nv);   // the next group is on its way meanwhile
        float mn = 3.0e38f, mx = -3.0e38f;
        auto range = [&](const float (&x)[V]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < V; ++e) { mn = fminf(mn, x[e]); mx = fmaxf(mx, x[e]); }
        };
        if constexpr (K > 0) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (tl * V + k * ts * V < g.G) range(v[k]);
        } else {
            for (int c = tl * V; c < g.G; c += ts * V) {
                float x[V];
                Vec<T>::load(wp + c, x);
                range(x);
            }
        }
        team_range(mn, mx, ts);
        float s, z;
        if (g.qs > 0.f) {
            s = fmaxf(fabsf(mn), fabsf(mx)) / g.qs;
            if (s == 0.f) s = 1.f;
            z = g.qs;
        } else {
            s = (mx - mn) / g.qmax;
            if (s == 0.f) s = 1.f;
            z = fminf(fmaxf(rintf(-mn / s), 0.f), g.qmax);
        }
        const float rs = 1.0f / s;
        const float top = g.qmax - z;            // code minus zero-point lies in [-z, top] (whole numbers: exact)
        float part = 0.f;
        auto add = [&](const float (&x)[V], const float4v (&a)[V / 4]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float u = __builtin_amdgcn_fmed3f(rintf(x[e] * rs), -z, top);
                const float d = x[e] - s * u;
                part = __builtin_fmaf(a[e / 4][e % 4] * d, d, part);
            }
        };
        if constexpr (K > 0) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (tl * V + k * ts * V < g.G) add(v[k], av[k]);
            if (gc_step != 0 && gi < g.n_groups) fetch_a(gc * g.G);
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) v[k][e] = nv[k][e];
        } else {
            for (int c = tl * V; c < g.G; c += ts * V) {     // the group is in cache
                float x[V];
                float4v a[V / 4];
                Vec<T>::load(wp + c, x);
                load_a(g.a + c0 + c, a);
                add(x, a);
            }
        }
        acc = __builtin_fmaf(br, part, acc);
    }
    // team sum (fixed butterfly), then teams and workgroups in index order
    for (int off = ts >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (tl == 0) team_sum[team] = acc;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
        for (int i = 0; i < teams; ++i) t += team_sum[i];
        g.partial[blockIdx.x] = t;
    }
}

constexpr int SENS_WGS = 2048;
// one load latency, then the waves' butterflies and one exchange (a tree over LDS: 1 us more)
__global__ __launch_bounds__(1024) void sens_final_kernel(const float* __restrict__ partial, int n, float* __restrict__ err) {
    __shared__ double part[16];
    const int tid = threadIdx.x;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < SENS_WGS / 1024; ++k)
        if (tid + 1024 * k < n) s += double(partial[tid + 1024 * k]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((tid & 63) == 0) part[tid >> 6] = s;
    __syncthreads();
    if (tid < 16) {
        s = part[tid];
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) s += __shfl_xor(s, off, 16);
        if (tid == 0) *err = float(0.5 * s);
    }
}

// Scratch of the entry point that takes no workspace: the per-workgroup partial sums, SENS_WGS floats (8 KB), in
// device memory that belongs to the loaded code object (one copy per GPU, held until the process ends).  In host
// code the array's name is only a handle: the device address is looked up once per device and used from then on.
static __device__ __align__(256) float scratch[SENS_WGS];

// device address of `scratch` on the current device (nullptr on failure); looked up on the first call per device
float* scratch_address() {
    static std::atomic<float*> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    const bool cached = dev >= 0 && dev < 64;
    float* p = cached ? cache[dev].load(std::memory_order_acquire) : nullptr;
    if (p) return p;
    if (hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    if (cached) cache[dev].store(p, std::memory_order_release);
    return p;
}

}  // namespace

size_t sensitivity_workspace_bytes() { return size_t(SENS_WGS) * sizeof(float); }

onecomp_status sensitivity_run_static(const void* W, onecomp_dtype w_dtype, int64_t d_out, int64_t d_in,
                                      const float* a_diag, const float* b_diag, int bits, int group_size, int grid,
                                      float* err, hipStream_t stream) {
    float* ws = scratch_address();
    if (!ws) return ONECOMP_ERR_HIP;
    return sensitivity_run(W, w_dtype, d_out, d_in, a_diag, b_diag, bits, group_size, grid, err, ws, stream);
}

onecomp_status sensitivity_run(const void* W, onecomp_dtype w_dtype, int64_t d_out, int64_t d_in, const float* a_diag,
                               const float* b_diag, int bits, int group_size, int grid, float* err, void* workspace,
                               hipStream_t stream) {
    SensArgs g;
    g.W = W; g.a = a_diag; g.b = b_diag; g.partial = static_cast<float*>(workspace);
    g.d_in = int(d_in); g.G = group_size; g.n_g = int(d_in / group_size);
    g.n_groups = d_out * int64_t(g.n_g);
    const int vec = w_dtype == ONECOMP_BF16 ? 8 : 4;          // elements per 16-byte lane load
    int ts = 2;
    while (ts < 64 && ts * 2 * vec <= group_size) ts *= 2;    // one pass over the group if it fits 64 lanes
    // Up to 16 weights per lane, in two or four loads: what a group costs every lane of its team is then shared by twice or
    // four times as many.  us of a candidate, one load : 16 : 32 weights, 14336 x 4096: bf16, groups of 64 35.2 : 28.3 : 31.9,
    // of 128 35.8 : 28.6 : 28.4; fp32 (4 : 8 : 16), groups of 64 55.9 : 41.9 : 40.3.
    const int loads = w_dtype == ONECOMP_BF16 ? 2 : 4;
    while (ts > 2 && ceil_div(group_size, ts / 2 * vec) <= loads) ts /= 2;
    g.ts = ts;
    g.qs = grid == ONECOMP_GRID_SYMMETRIC ? float((1 << (bits - 1)) - 1) : 0.f;
    g.qmax = grid == ONECOMP_GRID_SYMMETRIC ? 2.f * g.qs : float((1 << bits) - 1);
    const int64_t teams = 256 / ts;
    // a whole number of rows per step of the grid, where one fits, keeps every team on the same slice of `a`
    int64_t cd = teams, rest = g.n_g;                         // greatest common divisor of teams and n_g
    while (rest != 0) { const int64_t r = cd % rest; cd = rest; rest = r; }
    const int64_t unit = g.n_g / cd;
    const int64_t most = unit <= SENS_WGS ? SENS_WGS / unit * unit : SENS_WGS;
    const int64_t need = ceil_div(g.n_groups, teams);
    const int wgs = int(need < most ? need : most);
    const int k = int(ceil_div(group_size, ts * vec));        // loads per lane and group
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(wgs), dim3(256), 0, stream, g); };
    if (w_dtype == ONECOMP_BF16) launch(k == 1 ? sens_kernel<uint16_t, 1> : k == 2 ? sens_kernel<uint16_t, 2> : sens_kernel<uint16_t, 0>);
    else launch(k <= 2 ? sens_kernel<float, 2> : k <= 4 ? sens_kernel<float, 4> : sens_kernel<float, 0>);
    ONECOMP_CHECK_LAUNCH();
    hipLaunchKernelGGL(sens_final_kernel, dim3(1), dim3(1024), 0, stream, g.partial, wgs, err);
    ONECOMP_CHECK_LAUNCH();
    return ONECOMP_OK;
}

}  // namespace onecomp
