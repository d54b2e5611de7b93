// fft.hip -- the reduced cross-correlation in the frequency domain (paper
// Sec. III-A: the correlation of the projected signal with the projected
// kernel may be carried out with FFTs; Sec. III-C, eq. (19) and (21): the
// cost model of that realisation).  Same result as the implicit GEMM of
// conv.hip (reading R9, full rate):
//     y[aL + b] = sum_{l<r} sum_{c<T} sc_l[a + c] h_{l,b}[c],   h_{l,b}[c] = kd_l[cL - b],
// i.e. for every output phase b a sum over l of stride-1 correlations of the
// projected signal row sc_l with T taps.  Overlap-save: segment s covers rows
// a in [sP, sP + P) with P = F - T + 1; in the F-point DFT domain
//     Y_{b,s} = sum_{l<r} conj(FFT(h_{l,b})) * FFT(sc_l[sP .. sP + F))
// and the first P samples of IFFT(Y_{b,s}) are the rows of the segment
// (circular correlation without wrap-around there).
//
// Kernels: (0) the projections of the signal blocks and of the kernel at every
// lag; (1) the taps of every (l, b) and (2) every (l, s) signal segment
// transformed; (3) the bin-wise
// contraction over l; (4) the inverse transform of every (b, s) with the
// rows written to y.  All sequences are real, so an F-point transform is a
// complex one of H = F / 2 points on x[2n] + i x[2n + 1] plus a split of the
// result into even and odd parts, and a spectrum is H complex values: bins
// 1 .. H - 1, and the two real bins 0 and H together in entry 0.
#include "conv.h"

namespace pj {

namespace {

constexpr int kFftThreads = 256;
constexpr int kFftMax = 4096;            // largest transform F

struct cf {
    float x, y;
};

// Roots of unity w[q] = exp(-2 pi i q / kFftMax), a constant table evaluated
// in FP64 by the compiler and rounded once (Taylor series on one octant,
// |angle| <= pi / 4, the other octants by symmetry).  An F-point transform
// reads every (kFftMax / F)-th entry.
struct RootTable {
    cf w[kFftMax];
};
constexpr double root_series(double x, int first)    // first = 0: cos x, 1: sin x
{
    double term = first ? x : 1.0, sum = term;
    for (int n = first + 1; n < 24; n += 2) {
        term *= -x * x / ((double)n * (n + 1));
        sum += term;
    }
    return sum;
}
constexpr RootTable make_roots()
{
    RootTable t{};
    constexpr double two_pi = 6.283185307179586476925286766559;
    constexpr int o = kFftMax / 8;
    for (int q = 0; q < kFftMax; ++q) {
        const int quad = q / (2 * o), m = q % (2 * o);          // angle = quad pi / 2 + m 2 pi / kFftMax
        const int d = m <= o ? m : 2 * o - m;                   // reflected into the first octant
        const double x = two_pi * d / kFftMax;
        const double c0 = root_series(x, 0), s0 = root_series(x, 1);
        const double c = m <= o ? c0 : s0, s = m <= o ? s0 : c0;
        const double cc = quad == 0 ? c : quad == 1 ? -s : quad == 2 ? -c : s;
        const double ss = quad == 0 ? s : quad == 1 ? c : quad == 2 ? -s : -c;
        t.w[q] = cf{(float)cc, (float)-ss};
    }
    return t;
}
__device__ constexpr RootTable kRoots = make_roots();

__device__ __forceinline__ cf operator+(cf a, cf b) { return cf{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cf operator-(cf a, cf b) { return cf{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cf operator*(cf a, cf b)
{
    return cf{fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ cf conj(cf a) { return cf{a.x, -a.y}; }
__device__ __forceinline__ cf mul_neg_i(cf a) { return cf{a.y, -a.x}; }

__device__ __forceinline__ void dft2(cf& a, cf& b)
{
    const cf t = a - b;
    a = a + b;
    b = t;
}

__device__ __forceinline__ void dft4(cf& a, cf& b, cf& c, cf& d)
{
    dft2(a, c);
    dft2(b, d);
    d = mul_neg_i(d);
    dft2(a, b);
    dft2(c, d);
    const cf t = b;      // natural order: a, c, b, d -> frequencies 0, 1, 2, 3
    b = c;
    c = t;
}

__device__ __forceinline__ void dft8(cf (&v)[8])
{
    constexpr float h = 0.70710678118654752440f;
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    v[3] = cf{h * (v[3].x + v[3].y), h * (v[3].y - v[3].x)};       // exp(-i pi / 4)
    v[5] = mul_neg_i(v[5]);
    v[7] = cf{h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y)};      // exp(-3 i pi / 4)
    dft2(v[0], v[1]);
    dft2(v[2], v[3]);
    dft2(v[4], v[5]);
    dft2(v[6], v[7]);
    const cf t1 = v[1], t3 = v[3], t4 = v[4], t6 = v[6];
    // sums are frequencies 0..3 (v0, v2, v4, v6), differences 4..7 (v1, v3, v5, v7)
    v[1] = v[2];
    v[2] = t4;
    v[3] = t6;
    v[4] = t1;
    v[6] = v[5];
    v[5] = t3;
}

// LDS slot of element i: one pad slot of 8 bytes every 8 elements, so that the
// stride-8 stores of the first pass fall on all 64 banks.
__device__ __forceinline__ constexpr int fft_slot(int i) { return i + (i >> 3); }
template <int H> __host__ __device__ constexpr int fft_lds_slots() { return H + H / 8; }

// The twiddles of a thread, all read from the table (rounded once: products of
// table entries measured 1.8x the error of the whole correlation) and asked
// for before the data, so that no pass waits for them: exp(-2 pi i k m / (Ns R))
// of every pass after the first, and of the real split, exp(-2 pi i k / F).
template <int H>
struct Twiddles {
    static constexpr int kPass8 = H == 256 ? 2 : 3;                                     // passes of radix 8
    static constexpr int RL = H == 256 || H == 2048 ? 4 : H == 1024 ? 2 : 1;            // radix of the last pass (1: none)
    cf w8[kPass8 - 1][8], wl[8], ws[8];
    __device__ __forceinline__ explicit Twiddles(int t)
    {
        int Ns = 8;
#pragma unroll
        for (int s = 0; s + 1 < kPass8; ++s, Ns *= 8)
#pragma unroll
            for (int m = 1; m < 8; ++m) w8[s][m] = kRoots.w[(t & (Ns - 1)) * m * (kFftMax / (Ns * 8))];
        if constexpr (RL > 1) {
#pragma unroll
            for (int i = 0; i < 8 / RL; ++i)
#pragma unroll
                for (int m = 1; m < RL; ++m) wl[m * (8 / RL) + i] = kRoots.w[(t + i * (H / 8)) * m * (kFftMax / H)];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) ws[i] = kRoots.w[(t + i * (H / 8)) * (kFftMax / (2 * H))];
    }
};

// Forward complex transform of H points held as 8 registers by each of H / 8
// threads, PB independent transforms per thread: v[p][i] is element
// t + i H / 8 before and after (natural order).  Stockham passes of radix 8
// with one pass of radix 2 or 4 last where H is not a power of 8; element j of
// a pass of radix R reads j + m H / R and goes to (j / Ns) Ns R + j % Ns + m Ns.
// LDS carries the data between passes (lds[p] of fft_lds_slots<H>() slots).
template <int H, int PB>
__device__ __forceinline__ void fft_exchange(cf (&v)[PB][8], cf* lds, int t, const int (&dst)[8])
{
    __syncthreads();                                  // the slots' last readers are done
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) lds[p * fft_lds_slots<H>() + fft_slot(dst[i])] = v[p][i];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[p][i] = lds[p * fft_lds_slots<H>() + fft_slot(t + i * (H / 8))];
}

template <int H, int PB>
__device__ __forceinline__ void fft_forward(cf (&v)[PB][8], cf* lds, int t, const Twiddles<H>& tw)
{
    constexpr int kPass8 = Twiddles<H>::kPass8, RL = Twiddles<H>::RL;
    int Ns = 1;
#pragma unroll
    for (int s = 0; s < kPass8; ++s) {
        const int k = t & (Ns - 1);
        if (s > 0) {
#pragma unroll
            for (int p = 0; p < PB; ++p)
#pragma unroll
                for (int m = 1; m < 8; ++m) v[p][m] = v[p][m] * tw.w8[s - 1][m];
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) dft8(v[p]);
        if (s + 1 < kPass8 || RL > 1) {
            int dst[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) dst[m] = (t - k) * 8 + k + m * Ns;
            fft_exchange<H, PB>(v, lds, t, dst);
        }
        Ns *= 8;
    }
    // last pass, Ns = H / RL: element j = t + i H / 8 stays in place
    if constexpr (RL > 1) {
        constexpr int NI = 8 / RL;
#pragma unroll
        for (int p = 0; p < PB; ++p) {
#pragma unroll
            for (int i = NI; i < 8; ++i) v[p][i] = v[p][i] * tw.wl[i];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if constexpr (RL == 4)
                    dft4(v[p][i], v[p][NI + i], v[p][2 * NI + i], v[p][3 * NI + i]);
                else
                    dft2(v[p][i], v[p][NI + i]);
            }
        }
    }
}

// Spectra of PB real sequences from the transforms Z of x[2n] + i x[2n + 1]
// (v as left by fft_forward), sequence p written to dst + p H if p < nlive:
// with E, O the transforms of the even and odd samples,
// X[k] = E[k] + exp(-2 pi i k / F) O[k], E[k] = (Z[k] + conj Z[H - k]) / 2,
// O[k] = (Z[k] - conj Z[H - k]) / 2i.
template <int H, int PB>
__device__ __forceinline__ void real_spectrum(cf (&v)[PB][8], cf* lds, int t, const Twiddles<H>& tw, int nlive,
                                              cf* __restrict__ dst)
{
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) lds[p * fft_lds_slots<H>() + fft_slot(t + i * (H / 8))] = v[p][i];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        if (p >= nlive) continue;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = t + i * (H / 8);
            const cf z = v[p][i];
            const cf zc = conj(lds[p * fft_lds_slots<H>() + fft_slot(k == 0 ? 0 : H - k)]);
            const cf e = z + zc, o = mul_neg_i(z - zc);
            const cf x = e + tw.ws[i] * o;
            dst[(int64_t)p * H + k] = k == 0 ? cf{z.x + z.y, z.x - z.y} : cf{0.5f * x.x, 0.5f * x.y};
        }
    }
}

// (1) and (2), one launch: the workgroups below `ntapwg` transform the taps,
// Hf[(l L + b) H + f] = spectrum of h_{l,b}, h_{l,b}[c] = kd_l[cL - b] for c < T
// (zero-padded to F); the others the signal segments,
// Sf[(l nseg + s) H + f] = spectrum of sc_l[sP .. sP + F) (zero past nbp).
// Neither side alone fills the chip, and neither needs the other.  A thread
// carries kFwdPB transforms through one set of twiddles, 256 / (H / 8) thread
// groups a workgroup.  Bound by the latency of its passes (radix 8, data in
// registers, three exchanges through LDS for 2048 points): 20 us for 256 taps
// and 1376 segments of 4096 points against 106 us for a radix-2 transform in
// LDS of each (twelve barriers, full-length complex data).
constexpr int kFwdPB = 2;
template <int H>
__global__ __launch_bounds__(kFftThreads) void fft_forward_kernel(
    const float* __restrict__ kd, int r, int L, int T, int64_t ntapwg, const float* __restrict__ sc, int64_t nbp, int64_t nseg, int P, cf* __restrict__ Hf,
    cf* __restrict__ Sf)
{
    constexpr int TH = H / 8, NB = kFftThreads / TH, PB = kFwdPB;
    constexpr int SLOTS = NB * PB * fft_lds_slots<H>();
    __shared__ cf lds[SLOTS];
    const int t = threadIdx.x % TH, sub = threadIdx.x / TH;
    const Twiddles<H> tw(t);
    cf v[PB][8];
    const bool taps = (int64_t)blockIdx.x < ntapwg;
    const int64_t ntr = taps ? (int64_t)r * L : (int64_t)r * nseg;
    const int64_t q0 = ((taps ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - ntapwg) * NB + sub) * PB;
    if (taps) {
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int64_t q = q0 + p < ntr ? q0 + p : 0;
            const int64_t l = q / L, b = q - l * L;
            const float* lag = kd + l * T * L + L - 1 - b;       // kd_l[cL - b] at lag[cL]
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = 2 * (t + i * TH);
                v[p][i] = cf{c < T ? lag[(int64_t)c * L] : 0.0f, c + 1 < T ? lag[(int64_t)(c + 1) * L] : 0.0f};
            }
        }
    } else {
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int64_t q = q0 + p < ntr ? q0 + p : 0;
            const int64_t l = q / nseg, s = q - l * nseg;
            const float* row = sc + l * nbp;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int64_t n = s * P + 2 * (t + i * TH);
                v[p][i] = cf{n < nbp ? row[n] : 0.0f, n + 1 < nbp ? row[n + 1] : 0.0f};
            }
        }
    }
    cf* my = lds + sub * PB * fft_lds_slots<H>();
    fft_forward<H, PB>(v, my, t, tw);
    const int64_t left = ntr - q0;
    real_spectrum<H, PB>(v, my, t, tw, left < 0 ? 0 : left < PB ? (int)left : PB, (taps ? Hf : Sf) + q0 * H);
}

// (3) Yf[(b nseg + s) H + f] = sum_{l<r} conj(Hf[(l L + b) H + f]) Sf[(l nseg + s) H + f],
// highest l first (entry 0: the two real bins, multiplied separately).  A
// thread owns one bin f of kSegs segments and kPhases phases, so each spectrum
// value it loads serves several products; bound by the loads from L2 (2 x 8:
// 28 us, 4 x 4: 21, 8 x 4 and 8 x 8: 19 at 2^22 samples, L = r = 16, F = 4096).
// Waves are workgroups of their own: bins are independent, and F / 128 of them
// along x put the same bins of every segment on one XCD.
constexpr int kSegs = 8, kPhases = 4;
__global__ __launch_bounds__(64) void fft_contract_kernel(const cf* __restrict__ Hf, const cf* __restrict__ Sf,
                                                           int r, int L, int64_t nseg, int H, cf* __restrict__ Yf)
{
    const int f = blockIdx.x * 64 + threadIdx.x;      // H is a multiple of 64
    const int64_t s0 = (int64_t)blockIdx.z * kSegs;
    const int b0 = blockIdx.y * kPhases;
    cf acc[kSegs][kPhases];
#pragma unroll
    for (int i = 0; i < kSegs; ++i)
#pragma unroll
        for (int j = 0; j < kPhases; ++j) acc[i][j] = cf{0.0f, 0.0f};
    const cf *sp[kSegs], *hp[kPhases];
#pragma unroll
    for (int i = 0; i < kSegs; ++i) sp[i] = Sf + (s0 + i < nseg ? s0 + i : s0) * H + f;
#pragma unroll
    for (int j = 0; j < kPhases; ++j) hp[j] = Hf + (int64_t)(b0 + j < L ? b0 + j : b0) * H + f;
    cf sv[2][kSegs], hv[2][kPhases];                  // the spectra of projection l - 1 load during the products of l
    auto load = [&](int l, cf (&sd)[kSegs], cf (&hd)[kPhases]) {
#pragma unroll
        for (int i = 0; i < kSegs; ++i) sd[i] = sp[i][(int64_t)l * nseg * H];
#pragma unroll
        for (int j = 0; j < kPhases; ++j) hd[j] = hp[j][(int64_t)l * L * H];
    };
    auto products = [&](const cf (&sd)[kSegs], const cf (&hd)[kPhases]) {
#pragma unroll
        for (int j = 0; j < kPhases; ++j) {
            const float p = f == 0 ? 0.0f : hd[j].y, q = f == 0 ? hd[j].y : hd[j].x;
#pragma unroll
            for (int i = 0; i < kSegs; ++i) {         // conj(h) s
                acc[i][j].x = fmaf(hd[j].x, sd[i].x, fmaf(p, sd[i].y, acc[i][j].x));
                acc[i][j].y = fmaf(q, sd[i].y, fmaf(-p, sd[i].x, acc[i][j].y));
            }
        }
    };
    load(r - 1, sv[0], hv[0]);
    int l = r - 1;
    for (; l >= 1; l -= 2) {
        load(l - 1, sv[1], hv[1]);
        products(sv[0], hv[0]);
        load(l >= 2 ? l - 2 : 0, sv[0], hv[0]);
        products(sv[1], hv[1]);
    }
    if (l == 0) products(sv[0], hv[0]);
#pragma unroll
    for (int i = 0; i < kSegs; ++i)
#pragma unroll
        for (int j = 0; j < kPhases; ++j)
            if (s0 + i < nseg && b0 + j < L) Yf[((int64_t)(b0 + j) * nseg + s0 + i) * H + f] = acc[i][j];
}

// (4) rows a of segment s, phases b0 .. b0 + PB - 1: y[(sP + a) L + b] =
// (inverse transform of Yf[b, s])[a] for a < P (and inside the output).  A
// thread carries the same elements of PB phases, which are neighbours in y,
// through one set of twiddles.  Z[k] = E[k] + i O[k] with E[k] =
// (Y[k] + conj Y[H - k]) / 2, O[k] = exp(2 pi i k / F) (Y[k] - conj Y[H - k]) / 2;
// the inverse transform is the forward one with real and imaginary parts
// exchanged before and after.  Four phases a thread make 16-byte stores of y
// (`vec`): 24 us for 1376 transforms of 4096 points and 16.8 MB of outputs, 38 us
// with two phases, 106 us for radix-2 transforms storing single samples L apart.
template <int H, int PB>
__global__ __launch_bounds__(kFftThreads) void fft_out_kernel(const cf* __restrict__ Yf, int L, int64_t nseg,
                                                              int64_t ntr, int P, int64_t nout, int vec,
                                                              float* __restrict__ y)
{
    constexpr int TH = H / 8, NB = kFftThreads / TH;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cf* lds = reinterpret_cast<cf*>(smem_raw);
    const int t = threadIdx.x % TH, sub = threadIdx.x / TH;
    const int64_t q = (int64_t)blockIdx.x * NB + sub;     // q = (phase group) of a segment, group fastest
    const bool live = q < ntr;
    const int ng = (L + PB - 1) / PB;
    const int64_t s = live ? q / ng : 0;
    const int b0 = live ? (int)(q - s * ng) * PB : 0;
    const float scale = 0.5f / (float)H;
    const Twiddles<H> tw(t);
    cf v[PB][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = t + i * TH;
        const cf w = conj(tw.ws[i]);
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const cf* src = Yf + ((int64_t)(b0 + p < L ? b0 + p : b0) * nseg + s) * H;
            const cf a = src[k], m = conj(src[k == 0 ? 0 : H - k]);
            cf e, o;
            if (k == 0) {
                e = cf{a.x + a.y, 0.0f};
                o = cf{a.x - a.y, 0.0f};
            } else {
                e = a + m;
                o = w * (a - m);
            }
            v[p][i] = cf{(e.y + o.x) * scale, (e.x - o.y) * scale};     // e + i o, parts exchanged
        }
    }
    fft_forward<H, PB>(v, lds + sub * PB * fft_lds_slots<H>(), t, tw);
    if (!live) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int a = 2 * (t + i * TH);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t m = (s * P + a + h) * L + b0;
            if (a + h >= P) continue;
            if constexpr (PB == 4) {
                if (vec && m + 3 < nout) {
                    *reinterpret_cast<f32x4*>(y + m) =
                        h ? f32x4{v[0][i].x, v[1][i].x, v[2][i].x, v[3][i].x}
                          : f32x4{v[0][i].y, v[1][i].y, v[2][i].y, v[3][i].y};
                    continue;
                }
            }
#pragma unroll
            for (int p = 0; p < PB; ++p)
                if (b0 + p < L && m + p < nout) y[m + p] = h ? v[p][i].x : v[p][i].y;
        }
    }
}

// Projection of the signal and of the kernel, one launch.  Workgroups below
// `nsig` project 256 blocks of the signal, one block per thread held in
// registers (L <= LMAX; `vec`: its samples as 16-byte loads), all r
// projections with wave-uniform coefficients: sc_l[i] = sum_t s[iL + t] C[t, l],
// zero past the signal.  The others project the kernel at 256 consecutive lags
// for 8 projections: kd_l[q] = sum_u D[l, u] k'(q + u), q = e - (L - 1),
// e < T L, neighbouring lags on neighbouring lanes (taps formed inside the
// transform read the kernel at a stride of 2 L: 17 us for that alone).  Bound
// by HBM: 15 us at 2^22 samples, L = r = 16 (34 MB).
constexpr int kProjL = 32, kLagProj = 8;
template <int LMAX>
__global__ __launch_bounds__(256) void fft_project_kernel(
    const float* __restrict__ s, int64_t W, int L, int r, int vec, const float* __restrict__ CT,
    float* __restrict__ sc, int64_t nbp, int64_t nsig, const float* __restrict__ k, int64_t N, int reverse, int64_t T,
    const float* __restrict__ DT, float* __restrict__ kd)
{
    if ((int64_t)blockIdx.x < nsig) {
        if constexpr (LMAX > 0) {
            const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
            const int64_t n0 = i * L;
            float x[LMAX];
#pragma unroll
            for (int t = 0; t < LMAX; t += 4) {
                if (vec && t < L && n0 + t + 3 < W) {
                    const f32x4 c = *reinterpret_cast<const f32x4*>(s + n0 + t);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[t + e] = c[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[t + e] = t + e < L && n0 + t + e < W ? s[n0 + t + e] : 0.0f;
                }
            }
            if (i >= nbp) return;
            for (int l = 0; l < r; l += 4) {               // four rows of coefficients in flight
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float* c = CT + (l + j < r ? l + j : 0) * L;
                    v[j] = 0.0f;
#pragma unroll
                    for (int t = 0; t < LMAX; ++t) v[j] = fmaf(c[t < L ? t : 0], x[t], v[j]);   // x is zero past L
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (l + j < r) sc[(l + j) * nbp + i] = v[j];
            }
        }
        return;
    }
    const int64_t ne = cdiv(T * L, 256), w = (int64_t)blockIdx.x - nsig;
    const int l0 = (int)(w / ne) * kLagProj;
    const int64_t e = (w % ne) * 256 + threadIdx.x;
    float acc[kLagProj];
#pragma unroll
    for (int j = 0; j < kLagProj; ++j) acc[j] = 0.0f;
#pragma unroll 4
    for (int u = 0; u < L; ++u) {
        const int64_t n = e - (L - 1) + u;
        const bool in = n >= 0 && n < N;
        const float x0 = k[in ? (reverse ? N - 1 - n : n) : 0];
        const float x = in ? x0 : 0.0f;
#pragma unroll
        for (int j = 0; j < kLagProj; ++j) acc[j] = fmaf(DT[u * L + (l0 + j < r ? l0 + j : 0)], x, acc[j]);
    }
    if (e >= T * L) return;
#pragma unroll
    for (int j = 0; j < kLagProj; ++j)
        if (l0 + j < r) kd[(l0 + j) * T * L + e] = acc[j];
}

int launch_project(const ConvArgs& a, const ConvFftGeom& g, float* sc, float* kd, hipStream_t st)
{
    const bool own = a.L <= kProjL && a.r <= kProjL;
    const int64_t nsig = own ? cdiv(g.nbp, 256) : 0;
    const int64_t nlag = cdiv(g.T * a.L, 256) * cdiv(a.r, kLagProj);
    if (nsig + nlag > 0x7fffffff) return -2;
    if (!own && launch_conv_signal_rows(a, sc, g.nbp, st) != 0) return -1;
    const int vec = a.L % 4 == 0 && (uintptr_t)a.s % 16 == 0;
#define PJ_PROJ(LM_)                                                                                             \
    hipLaunchKernelGGL(fft_project_kernel<LM_>, dim3((unsigned)(nsig + nlag)), dim3(256), 0, st, a.s, a.W, a.L, a.r, \
                       vec, a.CT, sc, g.nbp, nsig, a.k, a.N, a.reverse, g.T, a.DT, kd)
    if (!own) PJ_PROJ(0);
    else if (a.L <= 8) PJ_PROJ(8);
    else if (a.L <= 16) PJ_PROJ(16);
    else PJ_PROJ(32);
#undef PJ_PROJ
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int H, int PB>
int launch_out(const cf* Yf, int L, const ConvFftGeom& g, float* y, hipStream_t st)
{
    constexpr int NB = kFftThreads / (H / 8);
    constexpr size_t lds = (size_t)NB * PB * fft_lds_slots<H>() * sizeof(cf);
    if (lds > 65536 && hipFuncSetAttribute((const void*)fft_out_kernel<H, PB>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return -1;
    const int64_t ntr = g.nseg * cdiv(L, PB);
    hipLaunchKernelGGL((fft_out_kernel<H, PB>), dim3((unsigned)cdiv(ntr, NB)), dim3(kFftThreads), lds, st, Yf, L,
                       g.nseg, ntr, (int)g.P, g.nout, PB == 4 && L % 4 == 0 && (uintptr_t)y % 16 == 0, y);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int H>
int launch_transforms(const ConvArgs& a, const ConvFftGeom& g, const float* sc, const float* kd, cf* Hf, cf* Sf,
                      cf* Yf, hipStream_t st)
{
    constexpr int NB = kFftThreads / (H / 8) * kFwdPB;
    const int64_t ntapwg = cdiv((int64_t)a.r * a.L, NB), nsigwg = cdiv((int64_t)a.r * g.nseg, NB);
    hipLaunchKernelGGL(fft_forward_kernel<H>, dim3((unsigned)(ntapwg + nsigwg)), dim3(kFftThreads), 0, st, kd,
                       a.r, a.L, (int)g.T, ntapwg, sc, g.nbp, g.nseg, (int)g.P, Hf, Sf);
    if (hipGetLastError() != hipSuccess) return -1;
    dim3 cgrid((unsigned)(H / 64), (unsigned)cdiv(a.L, kPhases), (unsigned)cdiv(g.nseg, kSegs));
    hipLaunchKernelGGL(fft_contract_kernel, cgrid, dim3(64), 0, st, Hf, Sf, a.r, a.L, g.nseg, H, Yf);
    if (hipGetLastError() != hipSuccess) return -1;
    if (a.L == 1) return launch_out<H, 1>(Yf, a.L, g, a.y, st);
    if (a.L == 2) return launch_out<H, 2>(Yf, a.L, g, a.y, st);
    return launch_out<H, 4>(Yf, a.L, g, a.y, st);
}

}  // namespace

// Transform size: the smallest power of two, at least 512, with at least
// three quarters of it left for outputs (P = F - T + 1 >= 3F / 4), at most
// kFftMax (there a quarter is accepted; longer kernels use the direct path).
ConvFftGeom conv_fft_geom(int64_t W, int64_t N, int L, int r)
{
    ConvFftGeom g;
    g.nout = W - N + 1;
    g.T = (N + L - 2) / L + 1;
    g.rows = cdiv(g.nout, L);
    int F = 512;
    while (F < kFftMax && 4 * (F - g.T + 1) < 3 * F) F *= 2;
    g.F = F;
    g.P = F - g.T + 1;
    g.ok = 4 * g.P >= F;                               // at least a quarter of each transform is output
    g.nseg = g.ok ? cdiv(g.rows, g.P) : 0;
    g.nbp = rup(g.nseg * g.P + F, 128);              // projected rows, zero past the signal
    g.sc_bytes = rup((int64_t)r * g.nbp * 4, 256);
    g.kd_bytes = rup((int64_t)r * g.T * L * 4, 256);
    g.hf_bytes = rup((int64_t)r * L * F * 4, 256);       // F / 2 complex values per spectrum
    g.sf_bytes = rup((int64_t)r * g.nseg * F * 4, 256);
    g.yf_bytes = rup((int64_t)L * g.nseg * F * 4, 256);
    g.total = g.sc_bytes + g.kd_bytes + g.hf_bytes + g.sf_bytes + g.yf_bytes;
    return g;
}

// Which realisation proj_conv1d uses: estimated times (fitted to measurements
// on MI355X) of the direct path -- the one-launch vector-ALU kernel for L <= 8
// (W r T products at about 2e13 per second), otherwise the matrix-core
// implicit GEMM over a phase tile of 32, 64, 128 or 256 (the power of two
// covering L, at least 32) after two small launches -- and of the FFT path (30 us,
// about 0.12 ms + 0.004 ms per signal row and phase, r + L, per 2^22 samples,
// scaled by the share of each transform that is output); the FFT path is taken
// when it is estimated at least 20 % faster.  The estimate is of earlier
// transforms and two to three times too long now, so calls near the line run the direct
// path although the FFT path is up to 4.5 times as fast (2^22 samples, L = 16, N = 16384,
// r = 1: 223 against 49 us; L = 16, N = 1024, r = 16: 247 and 68; L = 32, N = 16384, r = 4: 267
// and 53; L = 64, N = 16384, r = 8: 264 and 70).  On a stationary signal its error is
// also the lower one (rms 1.9e-7 against 5.8e-7 for the first).  The line has not
// been moved because a transform rounds a whole segment by its loudest part, which a
// caller of the direct path may not expect: where four template lengths of the
// same signal are 1e-4 times as loud, their outputs' rms error is 8e-4 to 1.2e-3 of
// them by FFT, 2e-7 to 6e-7 direct.
bool conv_prefers_fft(int64_t W, int64_t N, int L, int r)
{
    const ConvFftGeom f = conv_fft_geom(W, N, L, r);
    if (!f.ok || f.T < 16) return false;
    const double scale = (double)W / 4194304.0;
    const double t_fft = 30e-6 + scale * (0.12e-3 + 0.004e-3 * (r + L)) * (3.0 * f.F / (4.0 * f.P));
    double t_direct;
    if (L <= 8) {
        t_direct = 8e-6 + (double)W * r * f.T / 2.0e13;
    } else {
        const double bn = L > 128 ? 256.0 : L > 64 ? 128.0 : L > 32 ? 64.0 : 32.0;   // phase tile
        t_direct = 25e-6 + 2.0 * ((double)W / L) * bn * r * f.T / 1.0e14;
    }
    return t_fft < 0.8 * t_direct;
}

int launch_conv_fft(const ConvArgs& a, hipStream_t st)
{
    const ConvFftGeom g = conv_fft_geom(a.W, a.N, a.L, a.r);
    if (!g.ok) return -2;
    char* w = (char*)a.ws;
    float* sc = (float*)w;
    float* kd = (float*)(w + g.sc_bytes);
    cf* Hf = (cf*)(w + g.sc_bytes + g.kd_bytes);
    cf* Sf = (cf*)((char*)Hf + g.hf_bytes);
    cf* Yf = (cf*)((char*)Sf + g.sf_bytes);
    if (launch_project(a, g, sc, kd, st) != 0) return -1;
    switch (g.F) {
    case 512:  return launch_transforms<256>(a, g, sc, kd, Hf, Sf, Yf, st);
    case 1024: return launch_transforms<512>(a, g, sc, kd, Hf, Sf, Yf, st);
    case 2048: return launch_transforms<1024>(a, g, sc, kd, Hf, Sf, Yf, st);
    case 4096: return launch_transforms<2048>(a, g, sc, kd, Hf, Sf, Yf, st);
    default:   return -2;
    }
}

}  // namespace pj
