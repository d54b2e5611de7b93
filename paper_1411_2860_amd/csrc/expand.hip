// expand.hip -- synthesis of contraction-index gradients from projected ones
// (the adjoint of the projection in the pack step).  For R = A Q_{r,K} B
// computed as R = (A C_N)(D_N B) truncated to the first r projections, the
// gradient with respect to A is dA = (dR (D_N B)^T) C_N^T restricted to those
// projections, i.e. every projected gradient value is spread back over the L
// indices of its group with the coefficients of C (B side: of D^T):
//
//   out(p, jL + t) = sum_{l<r} in(p, l*Gp + j) * coef[t, l]
//
// One thread per (p, group j) writes the L outputs of its group, 16 at a time:
// for each projection l it loads in(p, l*Gp + j) once and adds it, times the
// 16 coefficients coef[t0 .. t0 + 15, l], to 16 accumulators; the loads of
// kExpandAhead projections are in flight together (one at a time, whole backward:
// 4096 x 4096 x 4096, L = r = 64, BF16 573 us, 478 us; L = 64, r = 32 313 and 266 us), and
// the workgroup stages the coefficients transposed in LDS, so they arrive as
// 16-byte broadcast reads.  The thread index runs along p when the output is stored
// with p contiguous (each output is then one coalesced store per wave) and
// along (p, j), j fastest, otherwise (the workgroup then parks its groups'
// runs in LDS and 16 consecutive lanes write each run).
#include "common.h"

#include <type_traits>

namespace pj {

namespace {

constexpr int kExpandChunk = 16;          // outputs of a group per pass
constexpr int kExpandMaxR = 256;
constexpr int kExpandAhead = 8;           // projections whose loads are in flight together

// in(p, kk) of RC projections l = 0 .. RC - 1 (zero from r up), the partials
// added last first; all loads of a partial in flight together.
template <typename T, int RC>
__device__ __forceinline__ void load_projected(const T* __restrict__ src, int64_t step, int r, int nparts,
                                               int64_t part, T (&v)[RC])
{
#pragma unroll
    for (int l = 0; l < RC; ++l) v[l] = src[(nparts - 1) * part + (l < r ? l : 0) * step];
    for (int q = nparts - 2; q >= 0; --q) {
        T u[RC];
#pragma unroll
        for (int l = 0; l < RC; ++l) u[l] = src[q * part + (l < r ? l : 0) * step];
#pragma unroll
        for (int l = 0; l < RC; ++l) v[l] += u[l];
    }
#pragma unroll
    for (int l = 0; l < RC; ++l) v[l] = l < r ? v[l] : T(0);
}

// acc[e] += in(p, kk) * c[l][e] of N projections.
template <int N, typename T>
__device__ __forceinline__ void add_projections(const T* __restrict__ src, int64_t step, int nparts, int64_t part,
                                                const T* c, T (&acc)[kExpandChunk])
{
    T v[N];
    load_projected<T, N>(src, step, N, nparts, part, v);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int e = 0; e < kExpandChunk; ++e) acc[e] += v[i] * c[i * kExpandChunk + e];
}

template <typename T, bool OUT_T>
__global__ __launch_bounds__(256) void expand_kernel(const T* __restrict__ in, int64_t ldi, int in_trans,
                                                     T* __restrict__ out, int64_t ldo, int64_t P, int64_t K, int L,
                                                     int r, int64_t Gp, const T* __restrict__ coef, int64_t slow0,
                                                     int nparts, int64_t part)
{
    __shared__ __align__(16) T cs[kExpandMaxR * kExpandChunk];      // [l][e] = coef[t0 + e, l]
    __shared__ T st[OUT_T ? 1 : 256 * (kExpandChunk + 1)];          // row-major output: runs re-dealt to lanes
    const int64_t fast = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t slow = slow0 + blockIdx.y;
    const int64_t G = (K + L - 1) / L;
    int64_t p, j;
    if (OUT_T) {               // (p fast, one group j per grid row)
        p = fast;
        j = slow;
    } else {                   // (p, j) flattened, j fastest
        p = fast / G;
        j = fast - p * G;
    }
    const bool live = p < P && j < G;
    const int tlim = live ? (int)((K - j * L) < L ? (K - j * L) : L) : 0;   // the last group may be partial
    const int64_t step = in_trans ? Gp * ldi : Gp;                          // from one projection to the next
    const T* src = in + (in_trans ? j * ldi + p : p * ldi + j);
    // the chunk loop runs over [0, L) for every thread (it holds barriers)
    for (int t0 = 0; t0 < L; t0 += kExpandChunk) {
        __syncthreads();
        for (int x = threadIdx.x; x < r * kExpandChunk; x += 256) {
            const int l = x / kExpandChunk, e = x - l * kExpandChunk;
            cs[x] = t0 + e < L ? coef[(int64_t)(t0 + e) * L + l] : T(0);
        }
        __syncthreads();
        T acc[kExpandChunk];
#pragma unroll
        for (int e = 0; e < kExpandChunk; ++e) acc[e] = T(0);
        if (t0 < tlim) {
            int l = 0;
            auto add = [&](auto n) {
                add_projections<n.value>(src + l * step, step, nparts, part, cs + l * kExpandChunk, acc);
                l += n.value;
            };
            while (l + kExpandAhead <= r) add(std::integral_constant<int, kExpandAhead>());
            // the rest in powers of two: a full chunk for r = 1 took 49 us where one load takes 36
            // (64 x 1728 over 3328, L = 4)
            if (l + 4 <= r) add(std::integral_constant<int, 4>());
            if (l + 2 <= r) add(std::integral_constant<int, 2>());
            if (l < r) add(std::integral_constant<int, 1>());
        }
        if (OUT_T) {
            const int64_t k0 = j * L + t0;
#pragma unroll
            for (int e = 0; e < kExpandChunk; ++e)
                if (t0 + e < tlim) out[(k0 + e) * ldo + p] = acc[e];
        } else {
            // the workgroup's 256 groups (consecutive j, one row p) each hold a
            // run of up to 16 outputs: park them in LDS, then 16 consecutive
            // lanes write each run
#pragma unroll
            for (int e = 0; e < kExpandChunk; ++e) st[threadIdx.x * (kExpandChunk + 1) + e] = acc[e];
            __syncthreads();
            const int64_t fb = (int64_t)blockIdx.x * 256;
            for (int q = threadIdx.x; q < 256 * kExpandChunk; q += 256) {
                const int g = q / kExpandChunk, e = q - g * kExpandChunk;
                const int64_t pg = (fb + g) / G, jg = (fb + g) - pg * G;
                if (pg < P) {
                    const int64_t kq = jg * L + t0 + e;
                    if (t0 + e < L && kq < K) out[pg * ldo + kq] = st[g * (kExpandChunk + 1) + e];
                }
            }
        }
    }
}

// Few projections, FP32.  Row-major output and input, L a multiple of 4: a
// thread owns 4 consecutive indices t of a group (the same in every group it
// visits, so its 4 x RC coefficients stay in registers), L / 4 threads a group,
// and a wave stores 1 KB of one row.  The workgroup stages the projected values
// of kExRows rows and kExGroups groups in LDS, [row][l][group].  Bound by HBM
// (the output): 4096 x 4096, L = 64, r = 8 (67 MB written): 33.6 us with 64-byte
// runs through LDS, 28 us from four partials of the projected gradient (33 us with its
// loads one after another).  Rows that are not 16-byte aligned are stored value by
// value (whole backward, 512 x 4093, L = 64, r = 16: 169 us in the general kernel, 77).
constexpr int kExRows = 4, kExGroups = 64;

template <int RC>
__global__ __launch_bounds__(256) void expand_rows_kernel(const float* __restrict__ in, int64_t ldi,
                                                          float* __restrict__ out, int64_t ldo, int64_t P, int64_t K,
                                                          int L, int r, int64_t Gp, const float* __restrict__ coef,
                                                          int nparts, int64_t part, int vec)
{
    static_assert(kExRows * kExGroups == 256, "one thread a row and group");
    __shared__ float xs[kExRows][RC][kExGroups];
    const int64_t G = (K + L - 1) / L;
    const int64_t p0 = (int64_t)blockIdx.x * kExRows, j0 = (int64_t)blockIdx.y * kExGroups;
    const int ng = (int)(G - j0 < kExGroups ? G - j0 : kExGroups);
    const int tpg = L / 4, gpp = 256 / tpg;              // threads a group, groups a pass
    const int t = 4 * (threadIdx.x % tpg), gt = threadIdx.x / tpg;
    {
        const int j = threadIdx.x % kExGroups, row = threadIdx.x / kExGroups;
        float v[RC];
        const int64_t p = p0 + row < P ? p0 + row : P - 1;
        load_projected<float, RC>(in + p * ldi + j0 + (j < ng ? j : 0), Gp, r, nparts, part, v);
#pragma unroll
        for (int l = 0; l < RC; ++l) xs[row][l][j] = v[l];
    }
    float c[RC][4];
#pragma unroll
    for (int l = 0; l < RC; ++l)
#pragma unroll
        for (int e = 0; e < 4; ++e) c[l][e] = coef[(t + e) * L + (l < r ? l : 0)];
    __syncthreads();
    if (gt >= gpp) return;                               // 256 is not a multiple of L / 4
    for (int row = 0; row < kExRows && p0 + row < P; ++row)
        for (int g = gt; g < ng; g += gpp) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int l = 0; l < RC; ++l) {
                const float x = xs[row][l][g];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += x * c[l][e];
            }
            const int64_t k = (j0 + g) * L + t;
            float* dst = out + (p0 + row) * ldo + k;
            if (vec && k + 3 < K) {
                *reinterpret_cast<f32x4*>(dst) = acc;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < K) dst[e] = acc[e];
            }
        }
}

// Transposed output and input (p contiguous in both): one thread per (p, group
// j) keeps the group's RC values in registers for all L outputs; coefficients
// from LDS.  4096 x 4096, L = 64, r = 8: 22 us reading them again for every 16
// outputs (41 us from four partials), 18 us from four partials.
template <int RC>
__global__ __launch_bounds__(256) void expand_cols_kernel(const float* __restrict__ in, int64_t ldi,
                                                          float* __restrict__ out, int64_t ldo, int64_t P, int64_t K,
                                                          int L, int r, int64_t Gp, const float* __restrict__ coef,
                                                          int nparts, int64_t part)
{
    __shared__ __align__(16) float cs[256 * RC];         // [t][l]
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j = blockIdx.y;
    float v[RC];
    load_projected<float, RC>(in + j * ldi + (p < P ? p : P - 1), Gp * ldi, r, nparts, part, v);
    for (int x = threadIdx.x; x < L * RC; x += 256) cs[x] = coef[(x / RC) * L + (x % RC < r ? x % RC : 0)];
    __syncthreads();
    if (p >= P) return;
    const int n = (int)(K - j * L < L ? K - j * L : L);  // the last group may be partial
    float* dst = out + j * L * ldo + p;
#pragma unroll 4
    for (int t = 0; t < n; ++t) {
        float acc = 0.0f;
#pragma unroll
        for (int l = 0; l < RC; ++l) acc += v[l] * cs[t * RC + l];
        dst[t * ldo] = acc;
    }
}

// Whether the kernels above apply (FP32).
bool expand_few(int L, int r, int in_trans, int out_trans)
{
    return r <= 16 && L <= 256 && in_trans == out_trans && (out_trans || L % 4 == 0);
}

// Runs them where they do: 1 launched, 0 not applicable, -1 failed.
int launch_few(const ExpandArgs& a, hipStream_t s)
{
    if (!expand_few(a.L, a.r, a.in_trans, a.out_trans)) return 0;
    const int64_t G = cdiv(a.K, a.L);
#define PJ_EXF(KERN_, RC_, GX_, GY_, ...)                                                                        \
    hipLaunchKernelGGL(KERN_<RC_>, dim3((unsigned)(GX_), (unsigned)(GY_)), dim3(256), 0, s, (const float*)a.in, a.ldi, \
                       (float*)a.out, a.ldo, a.P, a.K, a.L, a.r, a.Gp, (const float*)a.coef, a.nparts, a.part __VA_ARGS__)
    if (a.out_trans) {
        const int64_t gx = cdiv(a.P, 256);
        if (gx > 0x7fffffff || G > 65535) return 0;
        if (a.r <= 4) PJ_EXF(expand_cols_kernel, 4, gx, G);
        else if (a.r <= 8) PJ_EXF(expand_cols_kernel, 8, gx, G);
        else PJ_EXF(expand_cols_kernel, 16, gx, G);
    } else {
        const int vec = a.ldo % 4 == 0 && (uintptr_t)a.out % 16 == 0;
        const int64_t gx = cdiv(a.P, kExRows), gy = cdiv(G, kExGroups);
        if (gx > 0x7fffffff || gy > 65535) return 0;
        if (a.r <= 4) PJ_EXF(expand_rows_kernel, 4, gx, gy, , vec);
        else if (a.r <= 8) PJ_EXF(expand_rows_kernel, 8, gx, gy, , vec);
        else PJ_EXF(expand_rows_kernel, 16, gx, gy, , vec);
    }
#undef PJ_EXF
    return hipGetLastError() == hipSuccess ? 1 : -1;
}

template <typename T>
int launch_t(const ExpandArgs& a, hipStream_t s)
{
    if (a.r < 1 || a.r > kExpandMaxR || a.L < 1) return -2;
    if constexpr (sizeof(T) == 4) {
        const int e = launch_few(a, s);
        if (e != 0) return e < 0 ? e : 0;
    }
    const int64_t G = cdiv(a.K, a.L);
    const int64_t fast = a.out_trans ? a.P : a.P * G;
    const int64_t slow = a.out_trans ? G : 1;
    if (cdiv(fast, 256) > 0x7fffffff) return -2;
    // the grid's y dimension is limited: launch in slices
    for (int64_t y0 = 0; y0 < slow; y0 += 65535) {
        const int64_t ny = (slow - y0 < 65535) ? slow - y0 : 65535;
        if (a.out_trans)
            hipLaunchKernelGGL((expand_kernel<T, true>), dim3((unsigned)cdiv(fast, 256), (unsigned)ny), dim3(256), 0,
                               s, (const T*)a.in, a.ldi, a.in_trans, (T*)a.out, a.ldo, a.P, a.K, a.L, a.r, a.Gp,
                               (const T*)a.coef, y0, a.nparts, a.part);
        else
            hipLaunchKernelGGL((expand_kernel<T, false>), dim3((unsigned)cdiv(fast, 256), (unsigned)ny), dim3(256), 0,
                               s, (const T*)a.in, a.ldi, a.in_trans, (T*)a.out, a.ldo, a.P, a.K, a.L, a.r, a.Gp,
                               (const T*)a.coef, y0, a.nparts, a.part);
        if (hipGetLastError() != hipSuccess) return -1;
    }
    return 0;
}

}  // namespace

// Whether the synthesis reads every partial of its input once: the kernels for few
// projections, and the general one where a group is a single pass.
bool expand_once(int is_double, int L, int r, int in_trans, int out_trans)
{
    return !is_double && (L <= kExpandChunk || expand_few(L, r, in_trans, out_trans));
}

int launch_expand(int is_double, const ExpandArgs& a, hipStream_t s)
{
    return is_double ? launch_t<double>(a, s) : launch_t<float>(a, s);
}

}  // namespace pj
