// FDK reconstruction with offset-detector redundancy weights: the
// initialisation x <- FDK_w(y) of arXiv 2512.21180, Alg. 1 (and the classic
// baseline it is compared with).  Feldkamp-Davis-Kress for a circular orbit
// and a flat panel, in coordinates scaled to the isocentre (R = sid,
// D = sdd, u_i = u R / D, v_i = v R / D):
//   filter:       q = du_i * (p w(u) R / sqrt(R^2 + u_i^2 + v_i^2)) (*) h,
//                 h the Ram-Lak kernel at pitch du_i
//   backproject:  f(r) = (2 pi / n) sum_a R^2 / U^2 q(a, u(r), v(r)),
//                 U = R - (x cos + y sin), bilinear between pixel centres,
//                 zero off the panel.
// Redundancy weight: 1/2 for a centred panel; for a panel offset by off_u,
// sin^2(pi/4 (1 + s u / Delta)) over the overlap |u| <= Delta = W/2 - |off_u|
// (s = sign(off_u)) and 1 beyond it, so conjugate rays' weights add to one
// (Wang, Med. Phys. 2002).
//
// Optional Hann apodisation of the ramp (gain |omega| (1/2 + 1/2 cos(2 pi
// omega du_i)), the spatial kernel h/2 + (h(. - 1) + h(. + 1))/4).
//
// Filter up to 512 columns (`k_fdk_filter_mm`): the rows' product with the
// ramp's Toeplitz matrix on FP32 matrix instructions; the Hann window is in
// the matrix.  Wider panels (`k_fdk_filter`): one workgroup per panel row of
// one projection; the weighted row is staged in LDS between two zero pads of
// nu + 1 words, so every output sums all odd offsets in one fixed order
// without bounds tests; the ramp output is formed at columns -1 .. nu and the
// Hann window applied to it.
// Backprojection (`k_fdk_brick`): bricks of 16 x 16 voxel columns over panel
// windows staged in LDS, angles in order, the sums in registers; where bricks
// are too few or a window too large for LDS, `k_fdk_backproject`: one thread
// per voxel.
#include <hip/hip_runtime.h>

#include <cmath>

#include "cbct_internal.h"
#include "cbct_lds.h"
#include "cbct_nn.h"

namespace cbct {
namespace {

constexpr int kT = 256;
constexpr int kMaxNu = 4096;

struct FdkArgs {
    DevGeom g;
    float R, D, dui, delta, sgn;   // sgn = 0: centred panel (w = 1/2)
    float dbeta;
    int hann;                      // 1: Hann-apodised ramp
};

__device__ inline float red_weight(const FdkArgs &A, float u)
{
    if (A.sgn == 0.0f)
        return 0.5f;
    const float t = A.sgn * u;
    if (t > A.delta)
        return 1.0f;
    const float sw = sinf(0.7853981633974483f * (1.0f + fmaxf(t / A.delta, -1.0f)));
    return sw * sw;
}

__global__ void __launch_bounds__(kT) k_fdk_filter(FdkArgs A, const float *p, float *q)
{
    extern __shared__ float lds[];
    const DevGeom &g = A.g;
    const int nu = g.nu;
    const int P = nu + 1;              // zero pads of nu + 1 words on each side
    float *row = lds + P;
    float *coef = lds + 2 * P + nu;    // coef[m] = 1 / (pi^2 (2m+1)^2)
    float *qr = coef + (nu + 1) / 2;   // ramp output at columns -1 .. nu
    const int a = blockIdx.x / g.nv, iv = blockIdx.x % g.nv;
    const size_t base = ((size_t)a * g.nv + iv) * nu;
    const float vi = (g.off_v + ((float)iv - g.cv) * g.dv) * (A.R / A.D);
    for (int k = threadIdx.x; k < nu; k += kT) {
        const float u = g.off_u + ((float)k - g.cu) * g.du;
        const float ui = u * (A.R / A.D);
        const float cw = A.R * rsqrtf(fmaf(A.R, A.R, fmaf(ui, ui, vi * vi)));
        row[k] = p[base + k] * red_weight(A, u) * cw;
    }
    for (int k = threadIdx.x; k < P; k += kT) {
        lds[k] = 0.0f;
        lds[P + nu + k] = 0.0f;
    }
    for (int m = threadIdx.x; m < (nu + 1) / 2; m += kT) {
        const float n = (float)(2 * m + 1);
        coef[m] = 1.0f / (9.869604401089358f * n * n);
    }
    __syncthreads();
    const float scale = 1.0f / A.dui;  // du_i * h, h ~ 1 / du_i^2
    // Ram-Lak output at columns -1 .. nu (the zero-padded row's convolution)
    for (int j = threadIdx.x - 1; j <= nu; j += kT) {
        float acc = 0.0f;
        for (int m = 0; m < (nu + 1) / 2; ++m) {
            const int n = 2 * m + 1;
            acc = fmaf(coef[m], row[j - n] + row[j + n], acc);
        }
        qr[j + 1] = scale * fmaf(0.25f, row[j], -acc);
    }
    __syncthreads();
    // Hann window: the kernel h/2 + (h(. - 1) + h(. + 1))/4
    for (int j = threadIdx.x; j < nu; j += kT)
        q[base + j] = A.hann ? fmaf(0.5f, qr[j + 1], 0.25f * (qr[j] + qr[j + 2])) : qr[j + 1];
}

// The filter as a matrix product: out[r][j] = sum_k in[r][k] h[k - j] over the
// weighted rows, on v_mfma_f32_16x16x4_f32 (FP32 operands and sums).  A
// workgroup holds 16 WM whole rows in LDS (37 KB with the table: four per CU);
// a wave forms 16 rows x 128 columns in eight accumulators, so each row
// operand serves eight products, and reads the Toeplitz operand as 64
// consecutive words of the kernel's table.  Whole rows are read before any
// is written, as the one-row kernel does, so `q` may be `p`.  A row with an
// infinite or undefined value is summed directly instead: in the product the
// ramp's zeros would spread it over the even offsets.  Bound by the
// matrix cores: 2 nu operations per output, half of them on the ramp's zeros
// (splitting columns by parity would save those, but not under the Hann
// window).  184320 rows of 512: 4.33 ms by direct sums from LDS (two reads
// per operation), 0.86 here.
constexpr int kMmNu = 512;
constexpr int kMmN = 128;            // columns per wave
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Row stride in LDS: 4 mod 64 words, so the 16 x 4 operand of a step (rows on
// lanes mod 16, k on lanes / 16) falls on 64 different banks.
__host__ __device__ inline int mm_stride(int nu) { return (nu + 63) / 64 * 64 + 4; }

// The ramp output at column j of a weighted row, as `k_fdk_filter` sums it:
// odd offsets only, nothing read off the row.
__device__ inline float ramp_direct(const float *row, int nu, int j)
{
    float acc = 0.0f;
    for (int n = 1; n <= nu; n += 2) {
        const float l = j - n >= 0 ? row[j - n] : 0.0f, r = j + n < nu ? row[j + n] : 0.0f;
        acc = fmaf(1.0f / (9.869604401089358f * (float)n * (float)n), l + r, acc);
    }
    return fmaf(0.25f, j >= 0 && j < nu ? row[j] : 0.0f, -acc);
}

template <int WM>
__global__ void __launch_bounds__(kT) k_fdk_filter_mm(FdkArgs A, int rows, const float *p, float *q)
{
    constexpr int WN = 4 / WM;
    constexpr int kN = kMmN * WN, kCols = kN / 64;   // columns formed, per lane when staging
    extern __shared__ float lds[];
    __shared__ uint32_t unbounded[4];   // per wave: its rows with an infinite or undefined value
    const DevGeom &g = A.g;
    const int nu = g.nu, S = mm_stride(nu), K = (nu + 3) & ~3;
    float *h = lds + 16 * WM * S;    // h[d + kN], d = k - j
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = blockIdx.x * (16 * WM);
    // kernel values at offsets -kN .. K - 1 (unit 1 / du_i^2)
    auto ramp = [](int n) {
        if (n == 0)
            return 0.25f;
        return n & 1 ? -1.0f / (9.869604401089358f * (float)n * (float)n) : 0.0f;
    };
    for (int i = threadIdx.x; i < kN + K; i += kT) {
        const int n = i - kN;
        h[i] = A.hann ? fmaf(0.5f, ramp(n), 0.25f * (ramp(n - 1) + ramp(n + 1))) : ramp(n);
    }
    {
        float ui[kCols], rw[kCols];
#pragma unroll
        for (int m = 0; m < kCols; ++m) {
            const float u = g.off_u + ((float)(lane + 64 * m) - g.cu) * g.du;
            ui[m] = u * (A.R / A.D);
            rw[m] = red_weight(A, u);
        }
        uint32_t bad = 0u;
#pragma unroll
        for (int k = 0; k < 4 * WM; ++k) {
            const int row = w + 4 * k, rr = r0 + row;   // uniform
            const int iv = rr % g.nv;
            const float vi = (g.off_v + ((float)iv - g.cv) * g.dv) * (A.R / A.D);
            const float *src = p + (size_t)rr * nu;
            float x[kCols];
#pragma unroll
            for (int m = 0; m < kCols; ++m)
                x[m] = rr < rows && lane + 64 * m < nu ? src[lane + 64 * m] : 0.0f;
#pragma unroll
            for (int m = 0; m < kCols; ++m) {
                const float cw = A.R * rsqrtf(fmaf(A.R, A.R, fmaf(ui[m], ui[m], vi * vi)));
                x[m] = lane + 64 * m < nu ? x[m] * rw[m] * cw : 0.0f;
                if (lane + 64 * m < S)
                    lds[row * S + lane + 64 * m] = x[m];
            }
            bool finite = true;
#pragma unroll
            for (int m = 0; m < kCols; ++m)
                finite = finite && fabsf(x[m]) < INFINITY;
            bad |= __any(!finite) ? 1u << k : 0u;
        }
        if (lane == 0)
            unbounded[w] = bad;
    }
    __syncthreads();
    const float scale = 1.0f / A.dui;  // du_i * h, h ~ 1 / du_i^2
    uint32_t skip[4], some = 0u;   // row r is bit r / 4 of skip[r % 4]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        skip[i] = __builtin_amdgcn_readfirstlane(unbounded[i]);
        some |= skip[i];
    }
    if (some)
        for (int row = 0; row < 16 * WM; ++row)
            if (unbounded[row & 3] >> (row >> 2) & 1u)
                for (int j = threadIdx.x; j < nu; j += kT) {
                    const float *x = lds + row * S;
                    float v = ramp_direct(x, nu, j);
                    if (A.hann)
                        v = fmaf(0.5f, v,
                                 0.25f * (ramp_direct(x, nu, j - 1) + ramp_direct(x, nu, j + 1)));
                    q[(size_t)(r0 + row) * nu + j] = scale * v;
                }
    const int wm = w / WN, j0 = (w % WN) * kMmN;
    if (j0 >= nu)
        return;
    const float *a = lds + (16 * wm + (lane & 15)) * S + (lane >> 4);
    const float *b = h + kN + (lane >> 4) - j0 - (lane & 15);
    f32x4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t)
        acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int k = 0; k < K; k += 4) {
        const float av = a[k];
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b[k - 16 * t], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int j = j0 + 16 * t + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * wm + 4 * (lane >> 4) + r, rr = r0 + row;
            if (j < nu && rr < rows && !(skip[r] >> (row >> 2) & 1u))
                q[(size_t)rr * nu + j] = scale * acc[t][r];
        }
    }
}

// ---- backprojection from staged panel windows ---------------------------------

constexpr int kBrick = 16;          // voxel columns per brick edge, one per thread
constexpr int kWinChunk = kT;       // angles whose windows are tabulated at a time

// The panel window of a brick at one angle: columns [U0, U1] and rows [V0, V1]
// that the bilinear reads of its voxels may touch, clipped to the panel with
// one zero column and two zero rows around it.  Extremes of the projections
// lie at the corners (U is linear and the column a ratio of linear functions
// of x, y).  U0 is a multiple of 4 where rows are loaded in fours.
struct FdkWin {
    int U0, V0, cols, rows;   // cols = 0: nothing on the panel
};

__device__ inline FdkWin fdk_window(const FdkArgs &A, int a, float xa, float xb, float ya,
                                    float yb, float za, float zb, bool vec)
{
    const DevGeom &g = A.g;
    const AngRec ar = g.angs[a];
    const float inv_du = 1.0f / g.du, inv_dv = 1.0f / g.dv;
    float ul = INFINITY, uh = -INFINITY, ml = INFINITY, mh = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float x = k & 1 ? xb : xa, y = k & 2 ? yb : ya;
        const float m = A.D / (A.R - fmaf(x, ar.c, y * ar.s));
        const float u = fmaf(fmaf(m, fmaf(y, ar.c, -x * ar.s), -g.off_u), inv_du, g.cu);
        ul = fminf(ul, u);
        uh = fmaxf(uh, u);
        ml = fminf(ml, m);
        mh = fmaxf(mh, m);
    }
    const float vl = fmaf(fminf(ml * za, mh * za) - g.off_v, inv_dv, g.cv);
    const float vh = fmaf(fmaxf(ml * zb, mh * zb) - g.off_v, inv_dv, g.cv);
    FdkWin w{0, 0, 0, 0};
    // one pixel of margin for rounding
    if (!(uh > -2.0f && ul < (float)g.nu + 1.0f && vh > -2.0f && vl < (float)g.nv + 1.0f))
        return w;
    int u0 = max((int)floorf(ul) - 1, -1);
    if (vec)
        u0 &= ~3;
    const int u1 = min((int)floorf(fminf(uh, (float)g.nu)) + 2, g.nu);
    w.U0 = u0;
    w.cols = u1 - u0 + 1;
    w.V0 = max((int)floorf(fmaxf(vl, -2.0f)) - 1, -2);
    w.rows = min((int)floorf(fminf(vh, (float)g.nv)) + 2, g.nv + 1) - w.V0 + 1;
    return w;
}

// One voxel's value at one angle, read from the projection itself: column
// u0f with fraction au, row position fv.
__device__ inline float fdk_sample(const DevGeom &g, const float *qa, int u0, float au, float fv)
{
    const float v0f = floorf(fv), av = fv - v0f;
    const int v0 = (int)v0f;
    if (v0 < -1 || v0 >= g.nv)
        return 0.0f;
    const bool uin0 = u0 >= 0, uin1 = u0 + 1 < g.nu;
    const bool vin0 = v0 >= 0, vin1 = v0 + 1 < g.nv;
    const float q00 = (uin0 && vin0) ? qa[(size_t)v0 * g.nu + u0] : 0.0f;
    const float q01 = (uin1 && vin0) ? qa[(size_t)v0 * g.nu + u0 + 1] : 0.0f;
    const float q10 = (uin0 && vin1) ? qa[(size_t)(v0 + 1) * g.nu + u0] : 0.0f;
    const float q11 = (uin1 && vin1) ? qa[(size_t)(v0 + 1) * g.nu + u0 + 1] : 0.0f;
    const float r0 = fmaf(au, q01 - q00, q00);
    const float r1 = fmaf(au, q11 - q10, q10);
    return fmaf(av, r1 - r0, r0);
}

// A workgroup owns 16 x 16 voxel columns x KZ layers, a thread one column: the
// source distance, the panel column and its fraction are one computation for
// KZ voxels, and a voxel costs a row position, its fraction and floor, two
// LDS reads and three interpolations.  Each angle's panel window is staged in
// LDS through a buffer resource over the projection, whose range check
// supplies the zero rows; windows of the next 256 angles are tabulated one
// angle per thread.  A window above `cap` words is read from memory instead.
// Voxels off the panel sideways contribute nothing (their lanes are off);
// rows off the panel read the window's zero rows.
// 256^3 x 360 x 512^2: 9.66 ms with one thread per voxel (four strided global
// reads each, 40 VALU instructions), 2.5 here (2.9 with eight layers; 2.8 with sixteen and three
// workgroups per CU instead of four).
template <int KZ, bool VEC>
__global__ void __launch_bounds__(kT) k_fdk_brick(FdkArgs A, int cap, const float *q, float *f)
{
    extern __shared__ float lds[];
    __shared__ FdkWin wins[kWinChunk];
    const DevGeom &g = A.g;
    const int nbx = (g.nx + kBrick - 1) / kBrick, nby = (g.ny + kBrick - 1) / kBrick;
    const int bx = blockIdx.x % nbx, by = blockIdx.x / nbx % nby, bz = blockIdx.x / (nbx * nby);
    const int tid = threadIdx.x;
    const int ix = bx * kBrick + (tid & 15), iy = by * kBrick + (tid >> 4), k0 = bz * KZ;
    auto cx = [&](int i) { return g.ox + ((float)i - 0.5f * (float)(g.nx - 1)) * g.vx; };
    auto cy = [&](int i) { return g.oy + ((float)i - 0.5f * (float)(g.ny - 1)) * g.vy; };
    auto cz = [&](int i) { return g.oz + ((float)i - 0.5f * (float)(g.nz - 1)) * g.vz; };
    const bool live = ix < g.nx && iy < g.ny;
    const float x = cx(ix), y = cy(iy);
    const float inv_du = 1.0f / g.du, inv_dv = 1.0f / g.dv;
    const uint32_t pbytes = 4u * (uint32_t)g.nu * (uint32_t)g.nv;
    float acc[KZ];
#pragma unroll
    for (int k = 0; k < KZ; ++k)
        acc[k] = 0.0f;
    for (int a = 0; a < g.n_angles; ++a) {
        if (a % kWinChunk == 0) {
            __syncthreads();   // every reader of the previous windows is done
            if (a + tid < g.n_angles)
                wins[tid] = fdk_window(A, a + tid, cx(bx * kBrick),
                                       cx(min(bx * kBrick + kBrick, g.nx) - 1), cy(by * kBrick),
                                       cy(min(by * kBrick + kBrick, g.ny) - 1), cz(k0),
                                       cz(min(k0 + KZ, g.nz) - 1), VEC);
            __syncthreads();
        }
        const FdkWin &W = wins[a % kWinChunk];
        const int cols = __builtin_amdgcn_readfirstlane(W.cols);
        if (cols == 0)
            continue;
        const int U0 = __builtin_amdgcn_readfirstlane(W.U0);
        const int V0 = __builtin_amdgcn_readfirstlane(W.V0);
        const int rows = __builtin_amdgcn_readfirstlane(W.rows);
        const int S = (cols + 3) & ~3;   // window row stride
        const bool staged = S * rows <= cap;
        const float *qa = q + (size_t)a * g.nv * g.nu;
        if (staged) {
            const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
                (void *)qa, (short)0, (int)pbytes, kBufferWord3);
            __syncthreads();   // the previous angle's readers are done
            // element i of the window: row i / n, with n elements a row; the
            // reciprocal is exact for i n < 2^32 (at most 2^14 x 2^12)
            constexpr int kE = VEC ? 4 : 1, kB = VEC ? 4 : 8;
            const uint32_t n = (uint32_t)S / kE, count = n * (uint32_t)rows;
            const uint32_t magic = 0xffffffffu / n + 1u;
            for (uint32_t i0 = tid; i0 < count; i0 += kB * kT) {
                float v[kB][kE];
#pragma unroll
                for (int b = 0; b < kB; ++b) {
                    const uint32_t i = i0 + b * kT;
                    const uint32_t r = n == 1 ? i : __umulhi(i, magic);
                    const int u = U0 + (int)((i - r * n) * kE), vr = V0 + (int)r;
                    const bool in = i < count && (unsigned)u < (unsigned)g.nu &&
                                    (unsigned)vr < (unsigned)g.nv;
                    const uint32_t off = in ? 4u * (uint32_t)(vr * g.nu + u) : pbytes;
                    if constexpr (VEC) {
                        const auto d = __builtin_amdgcn_raw_buffer_load_b128(res, (int)off, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            v[b][e] = __uint_as_float(d[e]);
                    } else {
                        v[b][0] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(res, (int)off, 0, 0));
                    }
                }
#pragma unroll
                for (int b = 0; b < kB; ++b) {
                    const uint32_t i = i0 + b * kT;
                    if (i < count) {
                        if constexpr (VEC)
                            *(float4 *)(lds + 4 * i) =
                                make_float4(v[b][0], v[b][1], v[b][2], v[b][3]);
                        else
                            lds[i] = v[b][0];
                    }
                }
            }
            __syncthreads();
        }
        const AngRec ar = g.angs[a];
        const float U = A.R - fmaf(x, ar.c, y * ar.s);
        const float rU = 1.0f / U;
        const float fu = fmaf(fmaf(A.D * rU, fmaf(y, ar.c, -x * ar.s), -g.off_u), inv_du, g.cu);
        const float u0f = floorf(fu), au = fu - u0f, wr = A.R * rU, w2 = wr * wr;
        const bool on = live && u0f >= -1.0f && u0f < (float)g.nu;
        const int u0 = (int)u0f;
        const float m = A.D * rU;
        if (on && staged) {
            // byte address of row 0 of the panel in this column
            const int col = (int)lds_addr(lds) + 4 * (min(max(u0 - U0, 0), cols - 2) - V0 * S);
#pragma unroll
            for (int k = 0; k < KZ; ++k) {
                const float fv = fmaf(fmaf(m, cz(k0 + k), -g.off_v), inv_dv, g.cv);
                const float av = __builtin_amdgcn_fractf(fv);
                const int v0 = min(max(floor_i32(fv), V0), V0 + rows - 2);
                const lds_float *r = lds_ptr((uint32_t)mad_i24(v0, 4 * S, col));
                const float q00 = r[0], q01 = r[1], q10 = r[S], q11 = r[S + 1];
                const float r0 = fmaf(au, q01 - q00, q00);
                const float r1 = fmaf(au, q11 - q10, q10);
                acc[k] = fmaf(w2, fmaf(av, r1 - r0, r0), acc[k]);
            }
        } else if (on) {
#pragma unroll 1
            for (int k = 0; k < KZ; ++k) {
                const float fv = fmaf(fmaf(m, cz(k0 + k), -g.off_v), inv_dv, g.cv);
                const float val = fdk_sample(g, qa, u0, au, fv);
#pragma unroll
                for (int j = 0; j < KZ; ++j)   // a register index has to be constant
                    acc[j] = j == k ? fmaf(w2, val, acc[j]) : acc[j];
            }
        }
    }
    if (!live)
        return;
#pragma unroll
    for (int k = 0; k < KZ; ++k)
        if (k0 + k < g.nz)
            f[((size_t)(k0 + k) * g.ny + iy) * g.nx + ix] = A.dbeta * acc[k];
}

__global__ void __launch_bounds__(kT) k_fdk_backproject(FdkArgs A, const float *q, float *f)
{
    const DevGeom &g = A.g;
    const size_t nvox = (size_t)g.nx * g.ny * g.nz;
    const size_t s = (size_t)blockIdx.x * kT + threadIdx.x;
    if (s >= nvox)
        return;
    const int ix = (int)(s % g.nx), iy = (int)((s / g.nx) % g.ny);
    const int iz = (int)(s / ((size_t)g.nx * g.ny));
    const float x = g.ox + ((float)ix - 0.5f * (float)(g.nx - 1)) * g.vx;
    const float y = g.oy + ((float)iy - 0.5f * (float)(g.ny - 1)) * g.vy;
    const float z = g.oz + ((float)iz - 0.5f * (float)(g.nz - 1)) * g.vz;
    const float inv_du = 1.0f / g.du, inv_dv = 1.0f / g.dv;
    float acc = 0.0f;
    for (int a = 0; a < g.n_angles; ++a) {
        const AngRec ar = g.angs[a];
        const float U = A.R - fmaf(x, ar.c, y * ar.s);
        const float rU = 1.0f / U;
        const float fu = fmaf(fmaf(A.D * rU, fmaf(y, ar.c, -x * ar.s), -g.off_u), inv_du, g.cu);
        const float fv = fmaf(fmaf(A.D * rU, z, -g.off_v), inv_dv, g.cv);
        const float u0f = floorf(fu);
        const int u0 = (int)u0f;
        if (u0 < -1 || u0 >= g.nu)
            continue;
        const float val = fdk_sample(g, q + (size_t)a * g.nv * g.nu, u0, fu - u0f, fv);
        const float wr = A.R * rU;
        acc = fmaf(wr * wr, val, acc);
    }
    f[s] = A.dbeta * acc;
}

}  // namespace
}  // namespace cbct

using namespace cbct;

extern "C" cbct_status cbct_fdk(const cbct_geom *g, const float *sino, int window, float *work,
                                float *vol, void *stream)
{
    if (!g || !sino || !work || !vol)
        return CBCT_E_NULL;
    if (window != 0 && window != 1)
        return CBCT_E_ARG;
    if (!g->dev_block)
        return CBCT_E_ARG;
    const cbct_geom_desc &d = g->desc;
    if (d.nu > kMaxNu)
        return CBCT_E_SHAPE;
    // a full orbit of equally spaced angles
    const int n = d.n_angles;
    for (int a = 0; a < n; ++a) {
        const double want = g->angles[0] + 2.0 * M_PI * a / n;
        if (std::fabs(g->angles[a] - want) > 1e-9)
            return CBCT_E_ARG;
    }
    FdkArgs A{};
    A.g = g->dev;
    A.R = (float)d.sid_mm;
    A.D = (float)d.sdd_mm;
    A.dui = (float)(d.du_mm * d.sid_mm / d.sdd_mm);
    A.delta = (float)(0.5 * d.nu * d.du_mm - std::fabs(d.off_u_mm));
    A.sgn = d.off_u_mm > 0 ? 1.0f : (d.off_u_mm < 0 ? -1.0f : 0.0f);
    if (A.sgn != 0.0f && !(A.delta > 0))
        return CBCT_E_GEOM;   // no overlap: no redundancy weighting possible
    A.dbeta = (float)(2.0 * M_PI / n);
    A.hann = window;
    hipStream_t s = (hipStream_t)stream;
    const size_t rows = (size_t)n * d.nv;
    // enough waves along the columns for whole rows, the others on more rows;
    // a few hundred rows make too few such workgroups (8 projections of 40 x 50:
    // five, 21 us for the call against 17 us with one workgroup per row)
    const int wm = d.nu <= kMmN ? 4 : d.nu <= 2 * kMmN ? 2 : 1;
    if (d.nu <= kMmNu && rows >= (size_t)64 * 16 * wm) {
        const size_t lds =
            ((size_t)16 * wm * mm_stride(d.nu) + kMmN * (4 / wm) + ((d.nu + 3) & ~3)) *
            sizeof(float);
        const dim3 grid((unsigned)((rows + 16 * wm - 1) / (16 * wm)));
        if (wm == 4)
            hipLaunchKernelGGL(k_fdk_filter_mm<4>, grid, dim3(kT), lds, s, A, (int)rows, sino, work);
        else if (wm == 2)
            hipLaunchKernelGGL(k_fdk_filter_mm<2>, grid, dim3(kT), lds, s, A, (int)rows, sino, work);
        else
            hipLaunchKernelGGL(k_fdk_filter_mm<1>, grid, dim3(kT), lds, s, A, (int)rows, sino, work);
    } else {
        const size_t lds =
            (2 * ((size_t)d.nu + 1) + d.nu + (d.nu + 1) / 2 + d.nu + 2) * sizeof(float);
        hipLaunchKernelGGL(k_fdk_filter, dim3((unsigned)rows), dim3(kT), lds, s, A, sino, work);
    }
    const size_t nvox = (size_t)d.nx * d.ny * d.nz;
    // Bricks where two per CU are there (of eight layers if not of sixteen) and
    // a window at the isocentre, a brick's diagonal wide, takes at most 25 (20) KB:
    // windows nearer the source are up to twice that, the buffer holds 36 KB
    // (four workgroups per CU).
    const double mu = d.sdd_mm / (d.sid_mm * d.du_mm), mv = d.sdd_mm / (d.sid_mm * d.dv_mm);
    auto words = [&](int kz) {
        return (kBrick * std::hypot(d.vx_mm, d.vy_mm) * mu + 6.0) * (kz * d.vz_mm * mv + 6.0);
    };
    auto bricks = [&](int kz) {
        return (size_t)((d.nx + kBrick - 1) / kBrick) * ((d.ny + kBrick - 1) / kBrick) *
               ((d.nz + kz - 1) / kz);
    };
    constexpr int kCap = 9216;   // window words
    constexpr size_t kEnough = 512;
    const int kz = bricks(16) >= kEnough && words(16) <= 6400.0 ? 16
                   : bricks(8) >= kEnough && words(8) <= 5120.0 ? 8 : 0;
    const bool vec = d.nu % 4 == 0 && ((uintptr_t)work & 15) == 0;
    const float *filtered = work;
    if (kz && (size_t)d.nv * d.nu < ((size_t)1 << 28)) {
        const dim3 grid((unsigned)bricks(kz));
        const size_t lds = kCap * sizeof(float);
        if (kz == 16 && vec)
            hipLaunchKernelGGL((k_fdk_brick<16, true>), grid, dim3(kT), lds, s, A, kCap, filtered, vol);
        else if (kz == 16)
            hipLaunchKernelGGL((k_fdk_brick<16, false>), grid, dim3(kT), lds, s, A, kCap, filtered, vol);
        else if (vec)
            hipLaunchKernelGGL((k_fdk_brick<8, true>), grid, dim3(kT), lds, s, A, kCap, filtered, vol);
        else
            hipLaunchKernelGGL((k_fdk_brick<8, false>), grid, dim3(kT), lds, s, A, kCap, filtered, vol);
    } else {
        hipLaunchKernelGGL(k_fdk_backproject, dim3((unsigned)((nvox + kT - 1) / kT)), dim3(kT), 0,
                           s, A, filtered, vol);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_hip_error(e);
        return CBCT_E_HIP;
    }
    return CBCT_OK;
}
