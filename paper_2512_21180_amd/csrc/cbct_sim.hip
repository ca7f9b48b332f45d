// Projection-data simulator kernels (see cbct_sim.h): Philox4x32-10 counter
// based random numbers, Poisson counts of the attenuated beam and the
// negative-log normalisation (monochromatic, or polychromatic over energy
// bins with the water-bone decomposition), or additive Gaussian noise.  One
// thread per element, but for the Poisson counts, which a wave decides together
// (WavePoisson); the Poisson rejection loop is bounded (64 trials).
#include <hip/hip_runtime.h>

#include "cbct_internal.h"
#include "cbct_sim.h"

namespace cbct {
namespace {

constexpr int kT = 256;

struct Words {
    uint32_t w[4];
};

// Philox4x32-10: ten rounds of (two 32x32 multiplications, xor with the other
// counter words and the key), key advanced by the Weyl increments in between.
__device__ inline Words philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                               uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one v_mad_u64_u32 each
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Words{{c0, c1, c2, c3}};
}

__device__ inline Words draw(uint64_t seed, uint32_t sid, uint64_t i, uint32_t j)
{
    return philox((uint32_t)i, (uint32_t)(i >> 32), j, sid, (uint32_t)seed, (uint32_t)(seed >> 32));
}

__device__ inline double unif53(uint32_t a, uint32_t b)
{
    return ((double)(a >> 5) * 67108864.0 + (double)(b >> 6)) * (1.0 / 9007199254740992.0);
}

// ln k! of a whole k >= 0: Stirling's series from 16 up (its first left-out
// term is below 1e-16 there), the logarithm of the exact product below.
__device__ inline double ln_factorial(double k)
{
    if (k < 16.0) {
        double f = 1.0;
        for (double j = 2.0; j <= k; j += 1.0)
            f *= j;
        return log(f);
    }
    const double r = 1.0 / k, r2 = r * r;
    double s = fma(r2, -691.0 / 360360.0, 1.0 / 1188.0);
    s = fma(r2, s, -1.0 / 1680.0);
    s = fma(r2, s, 1.0 / 1260.0);
    s = fma(r2, s, -1.0 / 360.0);
    s = fma(r2, s, 1.0 / 12.0);
    return fma(k + 0.5, log(k), -k) + (0.9189385332046727 + r * s);
}

// Poisson(lam): CDF inversion below 10, Hormann's PTRS from 10 up.  Trial j
// of the variate uses counter word 2 = trial0 + j.
__device__ __forceinline__ int64_t poisson(double lam, uint64_t seed, uint32_t sid, uint64_t i,
                                           uint32_t trial0)
{
    if (!(lam > 0.0))
        return 0;
    if (lam < 10.0) {
        const Words d = draw(seed, sid, i, trial0);
        const double u = unif53(d.w[0], d.w[1]);
        double p = exp(-lam), F = p;
        int64_t k = 0;
        while (u > F && k < 1000) {
            ++k;
            p *= lam / (double)k;
            F += p;
        }
        return k;
    }
    const double sl = sqrt(lam), ll = log(lam);
    const double b = 0.931 + 2.53 * sl;
    const double a = -0.059 + 0.02483 * b;
    const double log_inv_alpha = log(1.1239 + 1.1328 / (b - 3.4));
    const double v_r = 0.9277 - 3.6224 / (b - 2.0);
    for (uint32_t j = 0; j < 64; ++j) {
        const Words d = draw(seed, sid, i, trial0 + j);
        const double U = unif53(d.w[0], d.w[1]) - 0.5;
        const double V = unif53(d.w[2], d.w[3]);
        const double us = 0.5 - fabs(U);
        const double kf = floor((2.0 * a / us + b) * U + lam + 0.43);
        if (us >= 0.07 && V <= v_r)
            return (int64_t)kf;
        if (kf < 0.0 || (us < 0.013 && V > us))
            continue;
        if (log(V) + log_inv_alpha - log(a / (us * us) + b) <= -lam + kf * ll - ln_factorial(kf))
            return (int64_t)kf;
    }
    return (int64_t)floor(lam + 0.5);
}

__global__ void __launch_bounds__(kT) k_philox(size_t n, uint64_t seed, uint32_t sid, uint32_t *out)
{
    const size_t i = (size_t)blockIdx.x * kT + threadIdx.x;
    if (i >= n)
        return;
    const Words d = philox((uint32_t)i, (uint32_t)((uint64_t)i >> 32), 0, sid, (uint32_t)seed,
                           (uint32_t)(seed >> 32));
    uint4 v = make_uint4(d.w[0], d.w[1], d.w[2], d.w[3]);
    reinterpret_cast<uint4 *>(out)[i] = v;
}

// ---- Poisson counts of a wave's elements --------------------------------------
//
// `poisson` alone, one thread per element, is bound by FP64 issue: a wave
// follows its slowest lane through logarithms, lgamma and further trials,
// about 3000 vector instructions per variate.  `WavePoisson` decides the same
// tests from cheaper values with bounds on their errors:
//   * lam from a 64-entry table and a degree-5 polynomial (relative error
//     below 1e-15, taken as 1e-12 and more wherever it enters);
//   * from a mean of 10 up the first trial's immediate acceptance in FP32
//     (four in five variates); below 10 the inversion with tabulated 1 / k;
//   * what is left goes to a queue of the wave in LDS and is tested 64 at a
//     time, every lane with an item of its own: the count in FP64, the
//     acceptance test as k (log1p(x) - x) with x = (lam - k) / k in FP32,
//     Stirling's series for the rest; a rejected item returns to the queue
//     with its next trial.
// A decision closer to its threshold than the error bound is taken by
// `poisson` itself, so the counts are `poisson`'s own.  Clinical scan, ten
// bins (9.4e8 variates): see k_sim_poly.
constexpr int kQueue = 128;        // at most 63 left by a drain plus 64 pushed
constexpr uint32_t kExact = 255;   // trial field of an item `poisson` decides
constexpr double kLamMax = 1e7;    // above it `poisson` decides

struct PoissonLds {
    double exp2_64[64];            // 2^(j / 64)
    double inv[64];                // 1 / k
};

__device__ inline void poisson_tables(PoissonLds &T)
{
    if (threadIdx.x < 64) {
        T.exp2_64[threadIdx.x] = exp2((double)threadIdx.x * (1.0 / 64.0));
        T.inv[threadIdx.x] = 1.0 / (double)threadIdx.x;
    }
    __syncthreads();
}

// exp(x) for |x| <= 700: 2^(n/64) times the polynomial of |r| <= ln2 / 128
__device__ inline double exp_table(const PoissonLds &T, double x)
{
    const double nf = rint(x * 92.33248261689366);            // 64 / ln 2
    // ln 2 / 64 in two parts, the first of 25 bits
    double r = fma(nf, -0x1.62e42fp-7, x);
    r = fma(nf, -0x1.df473de6af279p-32, r);
    const int n = (int)nf;
    double q = fma(r, 1.0 / 120.0, 1.0 / 24.0);
    q = fma(r, q, 1.0 / 6.0);
    q = fma(r, q, 0.5);
    q = fma(r, q, 1.0);
    const double t = T.exp2_64[n & 63];
    return ldexp(fma(t * r, q, t), n >> 6);
}

__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One wave's counts: lane l holds element base + l, `lam_of(lane, bin)` gives
// an element's exact mean, count[bin * 64 + lane] receives the counts.
template <class LamOf>
struct WavePoisson {
    const PoissonLds &T;
    double *qlam;                  // [kQueue]
    uint32_t *qid;                 // [kQueue] lane | bin << 8 | trial << 16
    int64_t *count;
    uint64_t seed;
    uint32_t sid;
    uint64_t base;
    const LamOf &lam_of;
    int queued = 0;                // wave uniform

    __device__ void push(bool p, double lam, uint32_t id)
    {
        const uint64_t m = __ballot(p);
        const int at = queued + (int)__builtin_amdgcn_mbcnt_hi(
                                    (uint32_t)(m >> 32),
                                    __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (p) {
            qlam[at] = lam;
            qid[at] = id;
        }
        queued += (int)__popcll(m);
        wave_lds_fence();
    }

    // bin e of the lane's element: mean i0 exp(-att)
    __device__ void first(int e, bool live, int lane, double i0, double att)
    {
        int64_t c = 0;
        bool todo = false;
        uint32_t trial = 0;
        double lam = 0.0;
        // exp(-att) underflows to zero from 746 on
        if (live && i0 > 0.0 && !(att > 760.0 && i0 < 1e38)) {
            if (!(fabs(att) <= 700.0 && i0 < 1e30)) {
                todo = true;
                trial = kExact;
            } else {
                lam = i0 * exp_table(T, -att);
                const Words d = draw(seed, sid, base + lane, 256u * (uint32_t)e);
                if (lam < 10.0 - 1e-9) {
                    const double u = unif53(d.w[0], d.w[1]);
                    // left = u - F after each term: the count is the number of
                    // terms it stays above zero (four terms a turn, no branch
                    // in them: one a turn spent its time in the loop's masks).
                    // Its error is below 1e-14: sixty terms of three roundings.
                    double p = exp_table(T, -lam), left = u - p;
                    double least = fabs(left);
                    int k = left > 0.0;
#pragma unroll 1
                    for (int t = 1; t < 61 && __any(left > 0.0); t += 4) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            p *= lam * T.inv[t + q];
                            left -= p;
                            least = fmin(least, fabs(left));
                            k += left > 0.0;
                        }
                    }
                    c = k;
                    todo = least < 1e-13 || left > 0.0;
                    trial = kExact;
                } else if (!(lam > 10.0 + 1e-9 && lam < kLamMax)) {
                    todo = true;
                    trial = kExact;
                } else {
                    // FP32 values of the first trial: |U|, us and V err by at
                    // most 2^-23 of themselves plus 2^-27 (unif53 leaves out the
                    // first word's last five bits), the slope by a few
                    // 2^-23 of itself
                    const float sl = __builtin_amdgcn_sqrtf((float)lam);
                    const float b = fmaf(2.53f, sl, 0.931f);
                    const float a = fmaf(0.02483f, b, -0.059f);
                    const float vr = fmaf(-3.6224f, __builtin_amdgcn_rcpf(b - 2.0f), 0.9277f);
                    const float U = (float)(int)(d.w[0] ^ 0x80000000u) * 0x1p-32f;
                    const float V = (float)d.w[2] * 0x1p-32f;
                    const float us = 0.5f - fabsf(U);
                    const float slope = fmaf(2.0f * a, __builtin_amdgcn_rcpf(us), b);
                    const double t = (lam + 0.43) + (double)(slope * U);
                    const double kf = floor(t);
                    const float fr = (float)(t - kf), mar = 1e-6f * slope;
                    c = (int64_t)(int)kf;
                    todo = !(us >= 0.070001f && V <= vr - 4e-6f && fr > mar && fr < 1.0f - mar);
                }
            }
        }
        if (live)
            count[e * 64 + lane] = c;
        push(todo, lam, (uint32_t)lane | (uint32_t)e << 8 | trial << 16);
    }

    // the last min(64, queued) items: one trial each
    __device__ void drain(int lane)
    {
        const int nb = queued < 64 ? queued : 64;
        queued -= nb;
        const bool on = lane < nb;
        const int at = queued + (on ? lane : 0);
        const double lam = qlam[at];
        const uint32_t id = qid[at];
        wave_lds_fence();
        const uint32_t el = id & 63u, e = (id >> 8) & 255u, j = id >> 16;
        bool exact = on && j >= 64u, again = false;
        int64_t c = 0;
        if (on && !exact) {
            const Words d = draw(seed, sid, base + el, 256u * e + j);
            const double U = unif53(d.w[0], d.w[1]) - 0.5, V = unif53(d.w[2], d.w[3]);
            const double us = 0.5 - fabs(U);
            const double b = 0.931 + 2.53 * sqrt(lam);
            const double a = -0.059 + 0.02483 * b;
            const double vr = 0.9277 - 3.6224 / (b - 2.0);
            const double arg = (2.0 * a / us + b) * U + lam + 0.43;
            const double kf = floor(arg), m = 1e-12 * (fabs(arg) + lam);
            exact = !(arg - kf > m && arg - kf < 1.0 - m) || fabs(V - vr) < 1e-11;
            c = (int64_t)kf;
            if (!(us >= 0.07 && V <= vr)) {
                if (kf < 0.0 || (us < 0.013 && V > us)) {
                    again = true;
                } else if (kf < 2.0 || kf > 2.0 * kLamMax) {
                    exact = true;
                } else {
                    const float bf = (float)b, af = (float)a, uf = (float)us, kk = (float)kf;
                    // log(V / alpha / (a / us^2 + b))
                    const float ia = fmaf(1.1328f, __builtin_amdgcn_rcpf(bf - 3.4f), 1.1239f);
                    const float lhs = __logf((float)V * ia) -
                                      __logf(fmaf(af, __builtin_amdgcn_rcpf(uf * uf), bf));
                    // -lam + k log(lam) - log(k!) by Stirling's series
                    const float ik = 1.0f / kk, x = (float)(lam - kf) * ik;
                    const float t = x / (2.0f + x), t2 = t * t;
                    float g;
                    if (fabsf(t) < 0.2f) {
                        // log1p(x) - x = 2 atanh(t) - x = 2 t^3 (1/3 + t^2/5 + ..) - x t
                        g = fmaf(t2, fmaf(t2, fmaf(t2, 1.0f / 11.0f, 1.0f / 9.0f), 1.0f / 7.0f),
                                 0.2f);
                        g = fmaf(2.0f * t * t2, fmaf(t2, g, 1.0f / 3.0f), -x * t);
                    } else {
                        g = __logf(1.0f + x) - x;
                    }
                    const float i2 = ik * ik;
                    const float st = ik * fmaf(i2, fmaf(i2, 1.0f / 1260.0f, -1.0f / 360.0f),
                                               1.0f / 12.0f);
                    const float rhs = fmaf(kk, g, -0.5f * __logf(6.28318531f * kk)) - st;
                    const float diff = lhs - rhs;
                    // errors: lhs 2e-6 of its size (up to 60) plus 1e-6, rhs a
                    // few 1e-7 of its size, and 5e-6 from the series at k = 2
                    const float mar = 2e-4f + 4e-6f * fabsf(rhs);
                    exact = exact || !(fabsf(diff) > mar);
                    again = diff > 0.0f;
                }
            }
            again = again && !exact;
        }
        if (exact) {
            c = poisson(lam_of((int)el, (int)e), seed, sid, base + el, 256u * e);
        }
        if (on && !again)
            count[e * 64 + el] = c;
        push(again, lam, id + 0x10000u);
    }

    // every bin's first trials, the queue drained whenever it holds a wave
    template <class Bin>
    __device__ void run(int bins, bool live, int lane, Bin &&beam)
    {
#pragma unroll 1
        for (int e = 0; e <= bins; ++e) {
            if (e < bins) {
                double i0 = 0.0, att = 0.0;
                if (live)
                    beam(e, i0, att);
                first(e, live, lane, i0, att);
            }
#pragma unroll 1
            while (queued >= (e < bins ? 64 : 1))
                drain(lane);
        }
        wave_lds_fence();
    }
};

// Threads of a workgroup and its dynamic LDS: above 16 bins two waves, which
// keeps the counts of 32 bins under 64 KB.
int poisson_threads(int bins) { return bins > 16 ? 128 : kT; }

size_t poisson_lds_bytes(int bins)
{
    return (size_t)(poisson_threads(bins) / 64) * (kQueue * 12 + (size_t)bins * 64 * 8);
}

template <class LamOf>
__device__ inline WavePoisson<LamOf> wave_poisson(const PoissonLds &T, char *lds, int wave,
                                                  int bins, uint64_t seed, uint32_t sid,
                                                  uint64_t base, const LamOf &f)
{
    char *w = lds + (size_t)wave * (kQueue * 12 + (size_t)bins * 64 * 8);
    double *ql = reinterpret_cast<double *>(w);
    int64_t *cnt = reinterpret_cast<int64_t *>(w + kQueue * 8);
    uint32_t *qi = reinterpret_cast<uint32_t *>(w + kQueue * 8 + (size_t)bins * 64 * 8);
    return WavePoisson<LamOf>{T, ql, qi, cnt, seed, sid, base, f};
}

__global__ void __launch_bounds__(kT, 4) k_poisson_log(size_t n, const float *p, float *y, int64_t *cnt,
                                                    double I0, uint64_t seed, uint32_t sid)
{
    extern __shared__ __align__(16) char lds[];
    __shared__ PoissonLds T;
    poisson_tables(T);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const size_t base = (size_t)blockIdx.x * blockDim.x + 64 * wave, i = base + lane;
    const bool live = i < n;
    auto lam_of = [&](int l, int) { return I0 * exp(-(double)p[base + l]); };
    auto W = wave_poisson(T, lds, wave, 1, seed, sid, base, lam_of);
    W.run(1, live, lane, [&](int, double &i0, double &att) {
        i0 = I0;
        att = (double)p[i];
    });
    if (!live)
        return;
    const int64_t c = W.count[lane];
    if (cnt)
        cnt[i] = c;
    const double r = (double)(c < 1 ? 1 : c) / I0;
    y[i] = (float)(-log(r < 1.0 ? r : 1.0));
}

// Water-bone decomposition constants (Sec. 2.2); tau_0 = 0 makes rho_w
// continuous at tau_0.
constexpr float kTau0 = 0.0f, kTau1 = 1.2f, kTau2 = 1.6f, kKappaB = 0.409f;

__global__ void __launch_bounds__(kT) k_water_bone(size_t n, const float *hu, float *rw,
                                                   float *rb)
{
    const size_t i = (size_t)blockIdx.x * kT + threadIdx.x;
    if (i >= n)
        return;
    const float r = fmaf(0.001f, hu[i], 1.0f);   // modified CT number
    float w = 0.0f, b = 0.0f;
    if (r >= kTau2) {
        b = kKappaB * r;
    } else if (r >= kTau1) {
        const float inv = 1.0f / (kTau2 - kTau1);
        w = kTau1 * (kTau2 - r) * inv;
        b = kKappaB * kTau2 * (r - kTau1) * inv;
    } else if (r >= kTau0) {
        w = r;
    }
    rw[i] = w;
    rb[i] = b;
}

constexpr int kMaxBins = 32;

struct PolyArgs {
    size_t n, npix;
    int nbins;
    double r_min;                  // smallest positive response (zero-signal floor)
    double mu_w[kMaxBins], mu_b[kMaxBins], resp[kMaxBins];
};

// Per element: one Poisson variate per energy bin of the attenuated beam
// (bin e's trials counted from 256 e), the response-weighted signal, and its
// negative log over the noise-free air signal, clamped at one.  The means and
// sums are FP64 in bin order and the counts WavePoisson's, so
// the counts equal those of an FP64 evaluation of the same model.  Bound by
// VALU issue (86 % of the slots, 500 instructions per variate).  360 x 512 x
// 512 elements, ten bins: 74.2 ms one element per thread through `poisson`,
// 17.2 ms with the queue, 16.7 with a multiply-add per Philox product, 14.3 with
// the inversion's terms free of branches.
__global__ void __launch_bounds__(kT, 4) k_sim_poly(PolyArgs A, const float *pw, const float *pb,
                                                 const float *I0, uint64_t seed, uint32_t sid,
                                                 float *y, float *signal, int64_t *counts)
{
    extern __shared__ __align__(16) char lds[];
    __shared__ PoissonLds T;
    poisson_tables(T);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const size_t base = (size_t)blockIdx.x * blockDim.x + 64 * wave, i = base + lane;
    const bool live = i < A.n;
    const size_t pix = live ? i % A.npix : 0;
    const double w = live ? (double)pw[i] : 0.0, b = live ? (double)pb[i] : 0.0;
    // the two products rounded, then summed
    auto att_of = [&](int e, double w, double b) {
#pragma clang fp contract(off)
        return A.mu_w[e] * w + A.mu_b[e] * b;
    };
    auto lam_of = [&](int l, int e) {
        const size_t k = base + l;
        return (double)I0[(size_t)e * A.npix + k % A.npix] *
               exp(-att_of(e, (double)pw[k], (double)pb[k]));
    };
    auto W = wave_poisson(T, lds, wave, A.nbins, seed, sid, base, lam_of);
    W.run(A.nbins, live, lane, [&](int e, double &i0, double &att) {
        i0 = (double)I0[(size_t)e * A.npix + pix];
        att = att_of(e, w, b);
    });
    if (!live)
        return;
    double sig = 0.0, air = 0.0;
    for (int e = 0; e < A.nbins; ++e) {
        const int64_t c = W.count[e * 64 + lane];
        if (counts)
            counts[(size_t)e * A.n + i] = c;
        sig += A.resp[e] * (double)c;
        air += A.resp[e] * (double)I0[(size_t)e * A.npix + pix];
    }
    if (signal)
        signal[i] = (float)sig;
    if (!(air > 0.0)) {
        y[i] = 0.0f;
        return;
    }
    const double r = (sig < A.r_min ? A.r_min : sig) / air;
    y[i] = (float)(-log(r < 1.0 ? r : 1.0));
}

__global__ void __launch_bounds__(kT) k_gaussian(size_t n, const float *clean, float *out,
                                                 double sigma, uint64_t seed, uint32_t sid)
{
    const size_t i = (size_t)blockIdx.x * kT + threadIdx.x;
    if (i >= n)
        return;
    const Words d = draw(seed, sid, i, 0);
    const double u1 = 1.0 - unif53(d.w[0], d.w[1]);
    const double u2 = unif53(d.w[2], d.w[3]);
    const double z = sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925286766559 * u2);
    out[i] = (float)((double)clean[i] + sigma * z);
}

cbct_status sim_done(hipError_t e)
{
    if (e == hipSuccess)
        return CBCT_OK;
    set_hip_error(e);
    return CBCT_E_HIP;
}

dim3 grid_for(size_t n) { return dim3((unsigned)((n + kT - 1) / kT)); }

}  // namespace
}  // namespace cbct

using namespace cbct;

extern "C" cbct_status cbct_philox_blocks(size_t n_blocks, uint64_t seed, uint32_t stream_id,
                                          uint32_t *out, void *stream)
{
    if (!out)
        return CBCT_E_NULL;
    if (n_blocks == 0)
        return CBCT_OK;
    if (n_blocks / kT >= 0x7fffffffu)
        return CBCT_E_SHAPE;
    hipLaunchKernelGGL(k_philox, grid_for(n_blocks), dim3(kT), 0, (hipStream_t)stream, n_blocks,
                       seed, stream_id, out);
    return sim_done(hipGetLastError());
}

extern "C" cbct_status cbct_sim_poisson_log(size_t n, const float *p, float *y, int64_t *counts,
                                            double I0, uint64_t seed, uint32_t stream_id,
                                            void *stream)
{
    if (!p || !y)
        return CBCT_E_NULL;
    if (!(I0 > 0.0))
        return CBCT_E_ARG;
    if (n == 0)
        return CBCT_OK;
    if (n / kT >= 0x7fffffffu)
        return CBCT_E_SHAPE;
    hipLaunchKernelGGL(k_poisson_log, grid_for(n), dim3(kT), poisson_lds_bytes(1), (hipStream_t)stream, n, p, y,
                       counts, I0, seed, stream_id);
    return sim_done(hipGetLastError());
}

extern "C" cbct_status cbct_water_bone(size_t n, const float *hu, float *rho_w, float *rho_b,
                                       void *stream)
{
    if (!hu || !rho_w || !rho_b)
        return CBCT_E_NULL;
    if (n == 0)
        return CBCT_OK;
    if (n / kT >= 0x7fffffffu)
        return CBCT_E_SHAPE;
    hipLaunchKernelGGL(k_water_bone, grid_for(n), dim3(kT), 0, (hipStream_t)stream, n, hu, rho_w,
                       rho_b);
    return sim_done(hipGetLastError());
}

extern "C" cbct_status cbct_poly_bins(int cap, double *centres_kev, double *resp, int *n_bins)
{
    if (!n_bins)
        return CBCT_E_NULL;
    *n_bins = 10;
    if (cap < 10)
        return centres_kev || resp ? CBCT_E_SHAPE : CBCT_OK;
    for (int k = 0; k < 10; ++k) {
        // bins [10 i, 10 (i + 1)) keV for i = 2..11, centred
        const double e = 10.0 * (k + 2) + 5.0;
        // piecewise linear through (20, 5), (60, 20), (120, 10) keV
        double r;
        if (e <= 20.0)
            r = 5.0;
        else if (e <= 60.0)
            r = 5.0 + (e - 20.0) * (15.0 / 40.0);
        else if (e < 120.0)
            r = 20.0 - (e - 60.0) * (10.0 / 60.0);
        else
            r = 10.0;
        if (centres_kev)
            centres_kev[k] = e;
        if (resp)
            resp[k] = r;
    }
    return CBCT_OK;
}

extern "C" cbct_status cbct_sim_poly(size_t n, size_t npix, const float *pw, const float *pb,
                                     int n_bins, const double *mu_w, const double *mu_b,
                                     const double *resp, const float *I0, uint64_t seed,
                                     uint32_t stream_id, float *y, float *signal,
                                     int64_t *counts, void *stream)
{
    if (!pw || !pb || !mu_w || !mu_b || !resp || !I0 || !y)
        return CBCT_E_NULL;
    if (n_bins < 1 || n_bins > kMaxBins || npix == 0 || n % npix != 0)
        return CBCT_E_SHAPE;
    if (n == 0)
        return CBCT_OK;
    if (n / kT >= 0x7fffffffu)
        return CBCT_E_SHAPE;
    PolyArgs A{};
    A.n = n;
    A.npix = npix;
    A.nbins = n_bins;
    for (int e = 0; e < n_bins; ++e) {
        if (!(resp[e] >= 0.0) || !(mu_w[e] == mu_w[e]) || !(mu_b[e] == mu_b[e]))
            return CBCT_E_ARG;
        A.mu_w[e] = mu_w[e];
        A.mu_b[e] = mu_b[e];
        A.resp[e] = resp[e];
        if (resp[e] > 0.0 && (A.r_min == 0.0 || resp[e] < A.r_min))
            A.r_min = resp[e];
    }
    const unsigned bt = (unsigned)poisson_threads(n_bins);
    hipLaunchKernelGGL(k_sim_poly, dim3((unsigned)((n + bt - 1) / bt)), dim3(bt),
                       poisson_lds_bytes(n_bins), (hipStream_t)stream, A, pw, pb, I0,
                       seed, stream_id, y, signal, counts);
    return sim_done(hipGetLastError());
}

extern "C" cbct_status cbct_sim_gaussian(size_t n, const float *clean, float *out, double sigma,
                                         uint64_t seed, uint32_t stream_id, void *stream)
{
    if (!clean || !out)
        return CBCT_E_NULL;
    if (n == 0)
        return CBCT_OK;
    if (n / kT >= 0x7fffffffu)
        return CBCT_E_SHAPE;
    hipLaunchKernelGGL(k_gaussian, grid_for(n), dim3(kT), 0, (hipStream_t)stream, n, clean, out,
                       sigma, seed, stream_id);
    return sim_done(hipGetLastError());
}
