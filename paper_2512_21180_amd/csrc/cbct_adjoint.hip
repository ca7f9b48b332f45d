// Adjoint A^T for gfx950: atomic-free gather over LDS-staged panel windows.
//
// Operator: the transpose of the plane-sampled cone-beam projector
// (arXiv 2512.21180, Sec. 2.2, backprojection P* as the adjoint of P).  The
// weight of voxel (i,j,k) in ray (a,u,v) is
//   ds(u,v) * hat(q_u(p) - q_vox) * hat(k(u,v,p) - k),   hat(s) = max(0, 1-|s|),
// where p is the voxel's index along the ray's sampling axis and q_vox its
// in-plane index; these are the weights the forward kernel applies.
//
// A workgroup owns a brick of 8 x 7 x 4 KV output voxels (KV = 4, 2 or 1,
// chosen by the plan so that the window fits in LDS); wave w owns the KV
// voxel layers k0 + KV w .. k0 + KV w + KV - 1.  The in-plane weight of a
// sample is shared by two voxels: a ray crossing the plane p at in-plane
// index q lies in the segment [s, s + 1), s = floor(q), and weighs 1 - f on
// voxel s and f on voxel s + 1 (f = q - s) with the same z weights.  So the
// lanes own (plane, segment) pairs rather than voxels: on x planes lane l
// takes plane i0 + l % 8 and segment j0 - 1 + l / 8 (eight segments feed
// the seven output rows), on y planes lane l < 63 takes plane j0 + l / 9
// and segment i0 - 1 + l % 9 (nine segments, eight output columns).  Each
// column whose ray crosses the lane's plane in its segment (the test is the
// forward's floor, so every column falls in exactly one segment) gets its
// z run computed once and added with weight 1 - f and f to two register
// sums; after the last angle the four shares of every output voxel (own and
// lower segment, both axes) are added in a fixed order through LDS and
// written once -- no atomics, and the order does not depend on timing.
// Against one voxel per lane this halves the z runs per voxel.
// For each angle the brick's panel window is staged in LDS, pre-multiplied
// by the ray length per plane ds, together with the column constants; the
// window's columns, the source-panel scales that give its rows and the row
// taps NT come from a table the host computes in FP64 per angle and brick
// column.  Per voxel and column, the rows with non-zero weight lie above
// the row v_c where the ray crosses z = k - 1 and span less than 2 / beta
// rows (beta: rows to z index, at least that of the brick's nearest point
// to the source); the run of NT = floor(2 / beta) + 1 rows that starts at
// floor(v_c) + 1, the first row above v_c, holds them all.  The start is
// taken as floor(v_c + 1 - delta), delta a few times the FP32 rounding of v_c
// (adj_start_delta): it is the first row above v_c, or one row lower when
// v_c lies within 2 delta above an integer -- a row of zero weight, and then
// the run still reaches the last non-zero row unless 2 / beta also lies
// within 2 delta below an integer (a row of weight below 2 delta beta is
// then left out, about once in 10^6 runs).
// The taps use the clamped hat, so rows outside the support add exact
// zeros (a run that would leave the window starts lower instead).  The
// window is stored column-major, so a run is consecutive LDS words read two
// at a time with immediate offsets in a fully unrolled sequence.
//
// Angles: one wave lists the next angles at which the window meets the panel
// (32 tested at once, one per lane); of every four listed angles each wave
// finds one's column ranges, which all waves use; and where four windows fit
// in a workgroup's share of the LDS they are staged together, one round trip to memory
// and two barriers for four angles.  When every wave found every
// angle's ranges and each angle was tested, staged and gathered by itself the
// clinical adjoint took 13.98 ms (now 12.70), the 64^3 one 220 us (150), four
// channels of 128^3 x 180 x 256^2 6.0 ms (4.7).  Bound by the taps where windows
// are tall (clinical case: LDS pipe busy 62 % of the cycles, a third of all with
// second passes; the 6.5e9 VALU instructions take half of them at two cycles
// each), by the per-column set-up where runs are short.
// SOLO kernels do take every angle by itself (see take_solo); the bits are the same.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "cbct_internal.h"
#include "cbct_lds.h"
#include "cbct_storage.h"

namespace cbct {
namespace {

constexpr int kThreads = 256;
// Window rows per wave and staging batch (loads in flight per lane).
constexpr int kStageRows = 24;
// Columns of at least 4 kStageRows rows take the staging whose batches stay
// inside the column (bricks of KV = 4, the clinical windows).
constexpr bool adj_tall(int KV, int HS) { return KV == 4 && HS >= 4 * kStageRows; }

struct BrickArgs {
    DevGeom g;
    const BrickWin *wins;  // [n_angles][nby][nbx] panel windows
    int W, H, HS;          // window columns (even) and rows, LDS column stride
    int nbx, nby, nbz;
    int KV;                // voxels per lane along z (bricks 8 x 7 x 4 KV)
    int gw;                // panel windows staged at a time: 4, 2 or 1
    int area;              // LDS words of the windows
    int split, per;        // ranges of angles gathered apart, angles in each
    float rbias;           // 1 - adj_start_delta(nv)
    int plan_bk;           // layers of the plan's bricks (four channels take shorter ones)
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float sat(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }

// A run's LDS address is a plain 32-bit number (lds_addr, lds_ptr): it comes
// out of one float-to-integer conversion with no base to add.

// Fractional panel column of the ray through (x, y, .) and its source-panel
// scale lambda (a point at height z lands at V = lambda z).  Used only for a
// voxel's column range, which is widened to whole columns and trimmed by the
// exact weights, so approximate reciprocals are enough.
__device__ inline void project_xy(const DevGeom &g, float inv_du, float c, float s, float x,
                                  float y, float &u, float &lam)
{
    const float den = fmaf(c, x, fmaf(s, y, -g.sid));
    lam = -g.sdd * __builtin_amdgcn_rcpf(den);
    u = fmaf(fmaf(lam, fmaf(-s, x, c * y), -g.off_u), inv_du, g.cu);
}

// One angle of a brick's work list: the angles at which the brick's window
// meets the panel, in order.
struct AngleEnt {
    int a;
    uint32_t u01;       // window columns U0 | U1 << 16
    int V0;             // first window row
    uint32_t hn;        // window rows | row taps << 16
    int x_lo, x_hi;     // columns sampled on x planes
    float lmin, lmax;   // extreme source-panel scales of the brick's support
};
static_assert(sizeof(AngleEnt) == 32, "AngleEnt layout");
constexpr int kListAngles = kAdjListAngles, kGroup = kAdjGroup;

__device__ inline AngleEnt uniform_ent(const AngleEnt &e)
{
    AngleEnt r;
    r.a = __builtin_amdgcn_readfirstlane(e.a);
    r.u01 = __builtin_amdgcn_readfirstlane(e.u01);
    r.V0 = __builtin_amdgcn_readfirstlane(e.V0);
    r.hn = __builtin_amdgcn_readfirstlane(e.hn);
    r.x_lo = __builtin_amdgcn_readfirstlane(e.x_lo);
    r.x_hi = __builtin_amdgcn_readfirstlane(e.x_hi);
    r.lmin = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(e.lmin)));
    r.lmax = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(e.lmax)));
    return r;
}

// Inputs of one angle's gather for one lane.
struct GatherIn {
    const DevGeom &g;
    int x_lo, x_hi;
    const float *yt;
    const float4 *cr;
    int HS, U0, V0;
    int VS1;   // largest run start: max(V1 - NT + 1, V0), so a run ends in the window
    int k0;
    int pl[2], sg[2];   // per sampling axis (0: x planes, 1: y planes): this lane's
                        // plane and in-plane segment; pl < 0: no work on that axis
    uint2 range;        // per axis the lane's columns, from U0: first | last << 16
    float inv_rvs;
    float rbias;        // 1 - delta: run start floor(v_c + 1 - delta)
    int eights;         // runs above 32 taps: their eights
};

__device__ inline float centre_x(const DevGeom &g, float i)
{
    return g.ox + (i - 0.5f * (float)(g.nx - 1)) * g.vx;
}

__device__ inline float centre_y(const DevGeom &g, float j)
{
    return g.oy + (j - 0.5f * (float)(g.ny - 1)) * g.vy;
}

// Accumulate one angle's contributions of the columns whose rays cross this
// lane's plane inside its segment [s, s + 1) of the in-plane index (the
// forward's floor(q) = s): such a sample weighs 1 - f on in-plane voxel s and
// f on voxel s + 1 (f = q - s), and the same z weights on both, so each
// column's z run is computed once for the two voxels: lo[ax][n] collects the
// 1 - f share (voxel s), hi[ax][n] the f share (voxel s + 1) for the KV
// voxels k0 + n.  NT taps per voxel and column (rows past the non-zero run
// have zero weight).  Forced inline: a call would impose the calling
// convention's register budget and stack on the kernel.
// C channels share a run's columns, rows and weights; their values lie side by
// side in the window.
// LONG: runs of in.eights times NT taps.
template <int NT, int KV, int C, bool LONG = false>
__device__ __forceinline__ void gather_angle(const GatherIn &in, float (&lo)[C][2][KV],
                                             float (&hi)[C][2][KV])
{
    const DevGeom &g = in.g;
    const int HS = in.HS, U0 = in.U0, V0 = in.V0, VS1 = in.VS1;
    const int k0 = in.k0;
    const float inv_rvs = in.inv_rvs;
    const float *yt = in.yt;
    const float4 *cr = in.cr;
    // Per voxel n: the row v_c where a ray with parameter t crosses z index
    // k0 + n - 1 is Bk / t + A0 - (1 - delta); the hat argument at row r is
    // t ((r - cv) rvs + rv0) + Kb - k.
    float Bk[KV], KbK[KV];
#pragma unroll
    for (int n = 0; n < KV; ++n) {
        const float kk = (float)(k0 + n);
        Bk[n] = (kk - 1.0f - g.Kb) * inv_rvs;
        KbK[n] = g.Kb - kk;
    }
    const float A0 = fmaf(-g.rv0, inv_rvs, g.cv + in.rbias);

    const float V0f = (float)V0, VS1f = (float)VS1;
#pragma unroll
    for (int cls = 0; cls < 2; ++cls) {
        const uint32_t range = cls == 0 ? in.range.x : in.range.y;
        const float fp = (float)in.pl[cls], sf = (float)in.sg[cls];
        const int uh = U0 + (int)(range >> 16);
        for (int u = U0 + (int)(range & 0xffffu); u <= uh; ++u) {
            if (cls == 1 && u >= in.x_lo && u < in.x_hi)
                continue;   // those columns are sampled on x planes
            const float4 cq = cr[u - U0];
            const float f = fmaf(fp, cq.y, cq.x) - sf;
            if (!(f >= 0.0f && f < 1.0f))
                continue;   // the ray crosses this plane in another segment
            const float wl = 1.0f - f;
            const float t = fmaf(fp, cq.w, cq.z);
            const float beta = t * g.rvs;
            const float rt = __builtin_amdgcn_rcpf(t);
            // LDS byte address of row 0 of this column in the window, signed
            // (row 0 lies below the window when V0 > 0; every row read,
            // vsf >= V0, has a non-negative address); exact in FP32: LDS
            // addresses are far below 2^24
            const float colb = (float)((int)lds_addr(yt) + 4 * C * ((u - U0) * HS - V0));
#pragma unroll
            for (int n = 0; n < KV; ++n) {
                // run start: the first row above v_c (floor(v_c) + 1), or one
                // row lower, of zero weight (see the file comment); clamped
                // into [V0, VS1] (a start moved down to VS1 only adds rows
                // below the run, of zero weight)
                const float vsf =
                    __builtin_amdgcn_fmed3f(floorf(fmaf(rt, Bk[n], A0)), V0f, VS1f);
                // hat argument at the run start; (vsf - cv) is exact, which keeps
                // the rounding of this difference of two large z indices small
                float s = fmaf(t, fmaf(vsf - g.cv, g.rvs, g.rv0), KbK[n]);
                const lds_float *py = lds_ptr((uint32_t)fmaf(vsf, 4.0f * C, colb));
                float csum[C];
#pragma unroll
                for (int c = 0; c < C; ++c)
                    csum[c] = 0.0f;
                const int turns = LONG ? in.eights : 1;
#pragma unroll 1
                for (int e = 0; e < turns; ++e) {
                    float yv[NT][C];
#pragma unroll
                    for (int m = 0; m < NT; ++m) {
                        if constexpr (C == 4) {
                            const f32x4 q =
                                *(__attribute__((address_space(3))) const f32x4 *)(py + 4 * m);
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                yv[m][c] = q[c];
                        } else {
#pragma unroll
                            for (int c = 0; c < C; ++c)
                                yv[m][c] = py[C * m + c];
                        }
                    }
#pragma unroll
                    for (int m = 0; m < NT; ++m) {
                        const float hat = sat(1.0f - fabsf(s));
#pragma unroll
                        for (int c = 0; c < C; ++c)
                            csum[c] = fmaf(hat, yv[m][c], csum[c]);
                        s += beta;
                    }
                    py += NT * C;
                }
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    lo[c][cls][n] = fmaf(wl, csum[c], lo[c][cls][n]);
                    hi[c][cls][n] = fmaf(f, csum[c], hi[c][cls][n]);
                }
            }
        }
    }
}

// The columns whose rays cross this lane's planes inside its segments at one
// angle, per sampling axis as first | last << 16 counted from U0 (none: last
// below first), from the window's column records cr.  All four waves of a brick
// need the same ranges, so each finds them for one angle of a group.
__device__ inline uint2 column_ranges(const DevGeom &g, const AngleEnt &e, const int (&pl)[2],
                                      const int (&sg)[2], float inv_du, const float4 *cr)
{
    const AngRec ar = g.angs[e.a];
    const int U0 = (int)(e.u01 & 0xffffu), U1 = (int)(e.u01 >> 16);
    uint32_t out[2];
#pragma unroll
    for (int cls = 0; cls < 2; ++cls) {
        out[cls] = 1u;
        // this axis has columns at this angle (uniform) and this lane a segment
        if (cls == 0 ? e.x_lo >= e.x_hi : (e.x_lo == 0 && e.x_hi == g.nu))
            continue;
        if (pl[cls] < 0)
            continue;
        const float fp = (float)pl[cls], sf = (float)sg[cls];
        int c_lo, c_hi;   // this axis' columns
        float u1, u2, lam;
        if (cls == 0) {   // x planes: plane i, segment [s, s + 1) in y
            c_lo = e.x_lo;
            c_hi = e.x_hi - 1;
            const float xp = centre_x(g, fp), ya = centre_y(g, sf);
            project_xy(g, inv_du, ar.c, ar.s, xp, ya, u1, lam);
            project_xy(g, inv_du, ar.c, ar.s, xp, ya + g.vy, u2, lam);
        } else {          // y planes: plane j, segment [s, s + 1) in x
            c_lo = 0;
            c_hi = g.nu - 1;
            const float yp = centre_y(g, fp), xa = centre_x(g, sf);
            project_xy(g, inv_du, ar.c, ar.s, xa, yp, u1, lam);
            project_xy(g, inv_du, ar.c, ar.s, xa + g.vx, yp, u2, lam);
        }
        // The segment's columns lie between the projections of its two
        // edges (within rounding, far below a column): trim the candidate
        // range's ends to columns that are members by the exact test (the
        // membership test in the gather keeps the partition exact in any case).
        int ul = max(max((int)floorf(fminf(u1, u2)), c_lo), U0);
        int uh = min(min((int)ceilf(fmaxf(u1, u2)), c_hi), U1);
        auto member = [&](int u) {
            if (cls == 1 && u >= e.x_lo && u < e.x_hi)
                return false;
            const float4 cq = cr[u - U0];
            const float f = fmaf(fp, cq.y, cq.x) - sf;
            return f >= 0.0f && f < 1.0f;
        };
        while (ul <= uh && !member(ul))
            ++ul;
        while (uh > ul && !member(uh))
            --uh;
        if (ul <= uh)
            out[cls] = (uint32_t)(ul - U0) | (uint32_t)(uh - U0) << 16;
    }
    return make_uint2(out[0], out[1]);
}

// The column records of one angle's window, by one wave.
__device__ inline void stage_columns(const DevGeom &g, const AngleEnt &e, int lane, float4 *cr)
{
    const int U0 = (int)(e.u01 & 0xffffu), U1 = (int)(e.u01 >> 16);
    for (int u = U0 + lane; u <= U1; u += 64) {   // lane: first column, from U0
        const ColRec col = g.cols[(size_t)e.a * g.nu + u];
        cr[u - U0] = make_float4(col.pb, col.ps, col.t0, col.tau);
    }
}

// Stage one angle's panel window into short columns: SB rows of loads in
// flight per lane.  Windows of up to 32 columns (HALF) put two rows on a
// wave's lanes.  Rows past Hs (zeros) that would leave the column go to row
// HS - 1, a spare row no tap reads (HS > H >= Hs).
template <int SB, bool HALF, int C>
__device__ __forceinline__ void stage_short(const DevGeom &g, __amdgpu_buffer_rsrc_t rows, int U0,
                                            int Wc, int Hs, int HS, int w, int lane, float *yt)
{
    constexpr int kRows = HALF ? 8 : 4;   // rows of one load of the four waves
    const int row_bytes = 4 * C * g.nu;
    const int r0 = HALF ? 2 * w + (lane >> 5) : w;
    for (int uu = HALF ? lane & 31 : lane; uu < Wc; uu += 64) {
        float *dst = yt + (size_t)uu * HS * C;
        for (int v = 0; v < Hs; v += kRows * SB) {
            int off = 4 * C * (U0 + uu) + (v + r0) * row_bytes;
            asm volatile("" : "+v"(off));   // one register (see gather_brick)
            float val[SB][C];
#pragma unroll
            for (int jj = 0; jj < SB; ++jj) {
                const int o = off + kRows * jj * row_bytes;
                if constexpr (C == 4) {
                    const auto d = __builtin_amdgcn_raw_buffer_load_b128(rows, o, 0, 0);
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        val[jj][c] = __uint_as_float(d[c]);
                } else if constexpr (C == 2) {
                    const auto d = __builtin_amdgcn_raw_buffer_load_b64(rows, o, 0, 0);
                    val[jj][0] = __uint_as_float(d[0]);
                    val[jj][1] = __uint_as_float(d[1]);
                } else {
                    val[jj][0] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(rows, o, 0, 0));
                }
            }
#pragma unroll
            for (int jj = 0; jj < SB; ++jj) {
                float *d = dst + (size_t)C * min(v + r0 + kRows * jj, HS - 1);
                if constexpr (C == 4) {
                    *(float4 *)d = make_float4(val[jj][0], val[jj][1], val[jj][2], val[jj][3]);
                } else if constexpr (C == 2) {
                    *(float2 *)d = make_float2(val[jj][0], val[jj][1]);
                } else {
                    *d = val[jj][0];
                }
            }
        }
    }
}

// Stage one angle's panel window into a tall column layout (HS >= 4 SB):
// Wc columns (from U0) x Hs rows of the ds-weighted projection, whose rows
// V0 .. V1 the buffer resource `rows` holds, into yt, column-major with
// stride HS, and the columns' records into cr.  Columns on lanes, rows on
// waves (stride 4), SB rows per wave and batch.  A batch that would run past
// the column starts lower instead, at the last row of the wave's residue
// class that keeps it inside (it then stores some rows of the wave's
// previous batch again, with the same values), so its stores take immediate
// offsets from one address.
template <int SB>
__device__ __forceinline__ void stage_tall(const DevGeom &g, __amdgpu_buffer_rsrc_t rows, int U0,
                                           int Wc, int Hs, int HS, int w, int lane, float *yt)
{
    const int row_bytes = 4 * g.nu;
    const int top = HS - 1 - 4 * (SB - 1);   // >= 3 in tall columns
    const int vtop = top - ((top - w) & 3);  // largest start = w mod 4
    for (int uu = lane; uu < Wc; uu += 64) {
        const int cb = 4 * (U0 + uu);   // byte offset of the column in a row
        float *dst = yt + (size_t)uu * HS;
        for (int vv0 = w; vv0 < Hs; vv0 += 4 * SB) {
            const int vb = min(vv0, vtop);
            int off = cb + vb * row_bytes;   // kept in one register (see gather_brick)
            asm volatile("" : "+v"(off));
            float val[SB];
#pragma unroll
            for (int jj = 0; jj < SB; ++jj)
                val[jj] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rows, off + 4 * jj * row_bytes, 0, 0));
            float *d = dst + vb;
#pragma unroll
            for (int jj = 0; jj < SB; ++jj)
                d[4 * jj] = val[jj];
        }
    }
}

// Brick coordinates.
struct BrickAt {
    int bx, by, bz;
};

// Gather one brick: bricks hold kAdjBI x kAdjBJ x 4 KV output
// voxels.  Lane roles (wave w owns the KV voxel layers from 4 KV (brick z) +
// KV w up): on x planes lane l takes plane i0 + l % 8 and in-plane segment
// j0 - 1 + l / 8 (eight segments serve the seven output rows j0 .. j0 + 6);
// on y planes lane l < 63 takes plane j0 + l / 9 and segment i0 - 1 + l % 9
// (nine segments serve the eight output columns).  After the last angle the
// four shares each output voxel receives (lo of its own segment and hi of
// the one below, on each axis) are added in a fixed order through LDS.
// Only the given range of the angles is gathered; where there are several,
// `part` receives its sums in FP32.
// `lds` holds the column table and the panel window, column-major ([W][HS],
// HS = 2 mod 4, which suits the gather's reads); then the exchange.
template <class VS, int KV, bool TALL, int C = 1, bool SOLO = false>
__device__ __forceinline__ void gather_brick(const BrickArgs &A, BrickAt at, int range,
                                             const float *ws, typename VS::T *const (&vol)[C],
                                             float *part, float *lds)
{
    constexpr int kBK = 4 * KV;
    constexpr int kSB = kStageRows;
    const DevGeom &g = A.g;
    const int HS = A.HS, recs = 4 * A.W;                // words of the column records before a window
    const int win = recs + A.W * HS * C;                // words of a window with them
    uint2 *ranges = (uint2 *)(lds + A.area);            // [kGroup][64]
    AngleEnt *list = (AngleEnt *)(ranges + kGroup * 64);
    int *listed = (int *)(list + kListAngles);

    // this range of the angles
    const int a_lo = range * A.per, a_hi = min(a_lo + A.per, g.n_angles);
    const int bx = at.bx, by = at.by, bz = at.bz;

    // the wave index is uniform (scalar registers for its row and layer indices)
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = bx * kAdjBI, j0 = by * kAdjBJ;
    const int k0 = bz * kBK + w * KV;
    int pl[2] = {i0 + (lane & 7), j0 + lane / 9};
    const int sg[2] = {j0 - 1 + (lane >> 3), i0 - 1 + lane % 9};
    if (pl[0] >= g.nx || sg[0] >= g.ny)
        pl[0] = -1;
    if (lane >= 63 || pl[1] >= g.ny || sg[1] >= g.nx)
        pl[1] = -1;

    // z extent of the brick's support (voxel centres +- one pitch), uniform
    const int kz0 = bz * kBK, kz1 = min(kz0 + kBK, g.nz) - 1;
    auto support_z = [&](int k, int side) {
        const float c = g.oz + ((float)k - 0.5f * (float)(g.nz - 1)) * g.vz;
        return side < 0 ? c - g.vz : c + g.vz;
    };
    const float zs0 = support_z(kz0, -1), zs1 = support_z(kz1, 1);
    // the brick column's panel windows, one per angle (host FP64)
    const BrickWin *wcol = A.wins + (size_t)by * A.nbx + bx;
    const size_t wstep = (size_t)A.nbx * A.nby;

    const float inv_du = 1.0f / g.du, inv_dv = 1.0f / g.dv;
    // z of this wave's first voxel layer (wave-uniform)
    const float zc_w0 = g.oz + ((float)k0 - 0.5f * (float)(g.nz - 1)) * g.vz;
    const float inv_rvs = 1.0f / g.rvs;
    float lo[C][2][KV], hi[C][2][KV];
#pragma unroll
    for (int c = 0; c < 2 * C; ++c)
#pragma unroll
        for (int n = 0; n < KV; ++n) {
            lo[c >> 1][c & 1][n] = 0.0f;
            hi[c >> 1][c & 1][n] = 0.0f;
        }

    // One angle's window: rows V0 .. V1 of the ds-weighted projection through a
    // buffer resource holding exactly those rows: the range check returns
    // zero for every row past V1 (the window's zero rows and a batch's rows
    // past Hs) without touching memory, so no load needs a test of its own.
    // Byte offsets within the rows are 32-bit (nv nu < 2^24).  The loads of a batch
    // of rows are issued before any of them is used, so their latencies
    // overlap instead of adding up row after row, and every store is
    // unconditional, so no load can be moved behind the wait for the others.
    // The batch's first row offset for a lane is kept in one
    // register (the empty asm stops the compiler from hoisting a lane
    // offset per row out of the loop, which costs a register per row);
    // each load adds a wave-uniform row offset.
    auto stage_window = [&](const AngleEnt &e, float *yt) {
        const int U0 = (int)(e.u01 & 0xffffu), Wc = (int)(e.u01 >> 16) - U0 + 1;
        const int nrows = (int)(e.hn & 0xffffu), NT = (int)(e.hn >> 16);
        // staged rows; rows past V1 (only when the window is shorter than a
        // run) are zero
        const int Hs = max(nrows, NT);
        const float *proj = ws + ((size_t)e.a * g.nv + e.V0) * g.nu * C;   // row V0, ds-weighted
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
            (void *)proj, (short)0, nrows * g.nu * 4 * C, kBufferWord3);
        if constexpr (TALL) {
            // Batches no longer than the window needs: SB rows per wave
            // cover 4 SB rows, SB = 16 up to 64 rows, 20 up to 80, else 24
            // (and more batches past 96 rows), so fewer rows past the window
            // are loaded and stored.  (Seven lengths from 8 to 24 saved a
            // further tenth of the staged rows but cost registers and were
            // slower.)
            if (Hs <= 64)
                stage_tall<16>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else if (Hs <= 80)
                stage_tall<20>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else
                stage_tall<kSB>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
        } else if constexpr (C > 1) {   // 16 registers of loads in flight
            if (Wc <= 32)
                stage_short<16 / C, true, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else
                stage_short<16 / C, false, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
        } else if (Wc <= 32) {
            if (Hs <= 32)
                stage_short<4, true, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else if (Hs <= 64)
                stage_short<8, true, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else
                stage_short<12, true, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
        } else {
            if (Hs <= 32)
                stage_short<8, false, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else if (Hs <= 64)
                stage_short<16, false, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
            else
                stage_short<kSB, false, C>(g, rows, U0, Wc, Hs, HS, w, lane, yt);
        }
    };

    // One angle's gather from its staged window; `columns` gives the lane's ranges.
    auto gather = [&](const AngleEnt &e, auto columns, const float *yt) {
        const int U0 = (int)(e.u01 & 0xffffu), V0 = e.V0;
        const int V1 = V0 + (int)(e.hn & 0xffffu) - 1, NT = (int)(e.hn >> 16);
        const int VS1 = max(V1 - NT + 1, V0);
        // this wave's KV voxel layers (z of the voxel centres +- one
        // pitch) land on rows [wv0, wv1] for every ray through the brick's
        // box (lambda is extreme at the box corners); a wave whose rows miss
        // the staged rows entirely has only zero weights and skips the angle
        // (wave-uniform branch; one row of margin for rounding).
        const float zl = zc_w0 - g.vz, zh = zc_w0 + (float)(KV - 1) * g.vz + g.vz;
        const float wv0 = fmaf(fminf(e.lmin * zl, e.lmax * zl) - g.off_v, inv_dv, g.cv);
        const float wv1 = fmaf(fmaxf(e.lmin * zh, e.lmax * zh) - g.off_v, inv_dv, g.cv);
        if (wv1 < (float)V0 - 1.0f || wv0 > (float)V1 + 1.0f)
            return;
        // compile-time tap count (NT rounded up to a supported count; extra
        // taps read zero weight)
        const GatherIn in{g, e.x_lo, e.x_hi, yt, (const float4 *)(yt - recs), HS, U0, V0, VS1,
                          k0, {pl[0], pl[1]}, {sg[0], sg[1]}, columns(), inv_rvs, A.rbias, NT >> 3};
        if constexpr (C > 1) {   // at most 8 (see kMaxTapsMc)
            switch (NT) {
            case 4: gather_angle<4, KV, C>(in, lo, hi); break;
            case 5: gather_angle<5, KV, C>(in, lo, hi); break;
            case 6: gather_angle<6, KV, C>(in, lo, hi); break;
            case 7: gather_angle<7, KV, C>(in, lo, hi); break;
            default: gather_angle<8, KV, C>(in, lo, hi); break;
            }
        } else {
            switch (NT) {
            case 4: gather_angle<4, KV, C>(in, lo, hi); break;
            case 5: gather_angle<5, KV, C>(in, lo, hi); break;
            case 6: gather_angle<6, KV, C>(in, lo, hi); break;
            case 7: gather_angle<7, KV, C>(in, lo, hi); break;
            case 8: gather_angle<8, KV, C>(in, lo, hi); break;
            case 9: gather_angle<9, KV, C>(in, lo, hi); break;
            case 10: gather_angle<10, KV, C>(in, lo, hi); break;
            case 11: gather_angle<11, KV, C>(in, lo, hi); break;
            case 12: gather_angle<12, KV, C>(in, lo, hi); break;
            case 13: gather_angle<13, KV, C>(in, lo, hi); break;
            case 14: gather_angle<14, KV, C>(in, lo, hi); break;
            case 15: gather_angle<15, KV, C>(in, lo, hi); break;
            case 16: gather_angle<16, KV, C>(in, lo, hi); break;
            case 18: gather_angle<18, KV, C>(in, lo, hi); break;
            case 20: gather_angle<20, KV, C>(in, lo, hi); break;
            case 24: gather_angle<24, KV, C>(in, lo, hi); break;
            case 28: gather_angle<28, KV, C>(in, lo, hi); break;
            case 32: gather_angle<32, KV, C>(in, lo, hi); break;
            default: gather_angle<8, KV, C, true>(in, lo, hi); break;
            }
        }
    };

    // One angle's entry: columns and row taps from the table, rows from the
    // extreme source-panel scales (positive) at the support's lowest and highest
    // z; false where the window misses the panel.
    auto entry = [&](int a, AngleEnt &e) {
        const BrickWin bw = wcol[(size_t)a * wstep];
        const AngRec ar = g.angs[a];
        const int U0 = (int)(bw.u01 & 0xffffu);
        const int U1 = min((int)(bw.u01 >> 16), U0 + A.W - 1);
        auto window_rows = [&](float za, float zb, int &v0, int &v1) {
            const float vmin =
                fmaf(fminf(bw.lmin * za, bw.lmax * za) - g.off_v, inv_dv, g.cv);
            const float vmax =
                fmaf(fmaxf(bw.lmin * zb, bw.lmax * zb) - g.off_v, inv_dv, g.cv);
            v0 = max((int)floorf(vmin) - 2, 0);
            v1 = min(min((int)ceilf(vmax) + 2, g.nv - 1), v0 + A.H - 1);
        };
        int V0, V1;
        window_rows(zs0, zs1, V0, V1);
        const bool seen = U0 <= U1 && V0 <= V1;
        if constexpr (C == 4) {
            // A run starts at most NT - 1 rows below its window's last
            // row, and from another start its weights round
            // differently: for the bits of a single call the starts are
            // bounded by the window P0 .. P1 of the plan's brick that
            // holds this one.  So this window keeps the rows of P0 .. P1
            // that a run may take from its own start (at most one row
            // above the highest crossing of z index k - 1) or from the
            // bounded one.
            const int p0 = kz0 / A.plan_bk * A.plan_bk;
            const int p1 = min(p0 + A.plan_bk, g.nz) - 1;
            int P0, P1;
            window_rows(support_z(p0, -1), support_z(p1, 1), P0, P1);
            const float zc = zs1 - 2.0f * g.vz;
            const float vc =
                fmaf(fmaxf(bw.lmin * zc, bw.lmax * zc) - g.off_v, inv_dv, g.cv);
            V0 = min(V0, max(P1 - bw.nt + 1, P0));
            V1 = min(P1, max(V1, (int)floorf(vc) + 1 + bw.nt));
        }
        e = AngleEnt{a, (uint32_t)U0 | (uint32_t)U1 << 16, V0,
                     (uint32_t)(V1 - V0 + 1) | (uint32_t)bw.nt << 16, ar.x_lo, ar.x_hi, bw.lmin,
                     bw.lmax};
        return seen;
    };

    if constexpr (SOLO) {
        // ---- one angle after another, each wave finding its column ranges: the
        // window and its records alone in LDS
        __syncthreads();   // the previous work item's readers are done
        for (int a = a_lo; a < a_hi; ++a) {
            AngleEnt e;
            if (!__builtin_amdgcn_readfirstlane((int)entry(a, e)))
                continue;
            e = uniform_ent(e);
            __syncthreads();   // the previous angle's readers are done
            // wave 0's column records are loaded with its rows, stored after them
            const int U0 = (int)(e.u01 & 0xffffu), Wc = (int)(e.u01 >> 16) - U0 + 1;
            float4 *cr = (float4 *)lds;
            ColRec col;
            if (w == 0)
                col = g.cols[(size_t)e.a * g.nu + U0 + min(lane, Wc - 1)];
            stage_window(e, lds + recs);
            if (w == 0) {
                cr[min(lane, Wc - 1)] = make_float4(col.pb, col.ps, col.t0, col.tau);
                stage_columns(g, e, lane + 64, cr);
            }
            __syncthreads();
            gather(e, [&] { return column_ranges(g, e, pl, sg, inv_du, cr); }, lds + recs);
        }
    }
    for (int base = SOLO ? a_hi : a_lo; base < a_hi; base += kListAngles) {
        __syncthreads();   // the readers of the previous list (or work item) are done
        // ---- the next 32 angles at which the window meets the panel
        if (w == 0) {
            AngleEnt e{};
            const int a = base + lane;
            const bool seen = lane < kListAngles && a < a_hi && entry(a, e);
            const uint64_t m = __ballot(seen);
            if (seen)
                list[__builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)] = e;
            if (lane == 0)
                *listed = (int)__popcll(m);
        }
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane(*listed);
        // ---- groups of four angles: wave w finds the column ranges of angle w
        // of the group (all waves use them), from the records in that angle's
        // window, or, where fewer than four windows fit, from a copy in the
        // window's place before it is staged
        for (int first = 0; first < n; first += kGroup) {
            const int m = min(kGroup, n - first);
            const bool all = A.gw == kGroup;
            if (first > 0)
                __syncthreads();   // the previous group's readers are done
            if (w < m) {
                const AngleEnt e = uniform_ent(list[first + w]);
                float4 *cr = (float4 *)(lds + w * (all ? win : recs));
                stage_columns(g, e, lane, cr);
                if (!all) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    ranges[w * 64 + lane] = column_ranges(g, e, pl, sg, inv_du, cr);
                }
            }
            if (all) {
                for (int i = 0; i < m; ++i)
                    stage_window(uniform_ent(list[first + i]), lds + i * win + recs);
                if (w < m) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    ranges[w * 64 + lane] =
                        column_ranges(g, uniform_ent(list[first + w]), pl, sg, inv_du,
                                      (const float4 *)(lds + w * win));
                }
            }
            for (int i = 0; i < m; i += A.gw) {
                const int mi = min(A.gw, m - i);
                if (!all) {
                    __syncthreads();   // the windows' readers, or the ranges', are done
                    for (int j = 0; j < mi; ++j) {
                        const AngleEnt e = uniform_ent(list[first + i + j]);
                        float *yt = lds + j * win + recs;
                        stage_window(e, yt);
                        if (w == j)
                            stage_columns(g, e, lane, (float4 *)(yt - recs));
                    }
                }
                __syncthreads();
                for (int j = 0; j < mi; ++j)
                    gather(uniform_ent(list[first + i + j]), [&] { return ranges[(i + j) * 64 + lane]; },
                           lds + j * win + recs);
            }
        }
    }

    // ---- each output voxel's four shares, added in a fixed order: x planes
    // (lo of its own segment, hi of the segment below), then y planes (same)
    float *xch = lds + (size_t)w * (4 * 64 * KV);
    const int io = lane & 7, jo = lane >> 3;
    const int i = i0 + io, j = j0 + jo;
    const int xl = ((jo + 1) << 3) | io, xh = (jo << 3) | io;   // x-plane lanes
    const int yl = jo * 9 + io + 1, yh = jo * 9 + io;           // y-plane lanes
#pragma unroll
    for (int c = 0; c < C; ++c) {
        __syncthreads();   // every wave is done with the window, or the last channel
#pragma unroll
        for (int n = 0; n < KV; ++n) {
            xch[(0 * KV + n) * 64 + lane] = lo[c][0][n];
            xch[(1 * KV + n) * 64 + lane] = hi[c][0][n];
            xch[(2 * KV + n) * 64 + lane] = lo[c][1][n];
            xch[(3 * KV + n) * 64 + lane] = hi[c][1][n];
        }
        __syncthreads();
        if (jo < kAdjBJ && i < g.nx && j < g.ny) {
#pragma unroll
            for (int n = 0; n < KV; ++n) {
                const int k = k0 + n;
                if (k < g.nz) {
                    float v = xch[(0 * KV + n) * 64 + xl] + xch[(1 * KV + n) * 64 + xh];
                    v += xch[(2 * KV + n) * 64 + yl];
                    v += xch[(3 * KV + n) * 64 + yh];
                    const size_t at = ((size_t)k * g.ny + j) * g.nx + i;
                    if (C == 1 && part)
                        part[at] = v;
                    else
                        VS::st(vol[c], at, v);
                }
            }
        }
    }
}

// Workgroups are dealt to the 8 XCDs round robin (XCD = id % 8).  XCD xc
// takes the brick rows by = xc, xc + 8, ... (every z layer of them, so each
// XCD holds an even share of cheap and costly bricks), in the order bx, bz,
// row: workgroups resident together on one XCD are neighbouring bricks whose
// panel windows overlap in its L2 (adjoint 33 -> 27 ms for the clinical
// case at the time; a contiguous brick range per XCD unbalances the XCDs, 71 ms).
// Rows past the last multiple of eight are dealt out by brick columns, so no
// XCD has a row more than another: with whole rows 10 rows (64^3) gave two XCDs
// twice the others' work, 19 rows (128^3) three XCDs half as much again.
// The brick of slot li of XCD xc; bx = -1 for the padding slots.
__device__ inline BrickAt brick_of_slot(const BrickArgs &A, int xc, int li)
{
    const int plane = A.nbx * A.nbz, whole = plane * (A.nby / 8);
    if (li < whole) {
        const int row = li / plane, rest = li - row * plane, bz = rest / A.nbx;
        return {rest - bz * A.nbx, xc + 8 * row, bz};
    }
    const int columns = (A.nby & 7) * A.nbx, each = (columns + 7) / 8;
    li -= whole;
    const int bz = li / each, c = xc + 8 * (li - bz * each), row = c / A.nbx;
    return {c < columns ? c - row * A.nbx : -1, (A.nby & ~7) + row, bz};
}

// Slots per XCD of one case (padded so that every XCD has the same count).
__host__ __device__ inline int slots_per_xcd(const BrickArgs &A)
{
    return A.nbz * (A.nbx * (A.nby / 8) + ((A.nby % 8) * A.nbx + 7) / 8);
}

template <class VS, int KV, bool TALL, bool SOLO>
__global__ void __launch_bounds__(kThreads, 4)
adjoint_brick(BrickArgs A, const float *__restrict__ ws, typename VS::T *__restrict__ vol,
              float *__restrict__ part)
{
    extern __shared__ float lds[];
    const BrickAt b = brick_of_slot(A, blockIdx.x & 7, blockIdx.x >> 3);
    if (b.bx < 0)
        return;
    const int ch = blockIdx.y;
    const size_t nvox = (size_t)A.g.nx * A.g.ny * A.g.nz;
    const size_t nsino = (size_t)A.g.n_angles * A.g.nv * A.g.nu;
    typename VS::T *const out[1] = {vol + ch * nvox};
    const size_t at = ((size_t)blockIdx.z * gridDim.y + ch) * nvox;
    gather_brick<VS, KV, TALL, 1, SOLO>(A, b, blockIdx.z, ws + ch * nsino, out,
                                        part ? part + at : nullptr, lds);
}

// The ranges' volumes added in order.
template <class VS>
__global__ void __launch_bounds__(kThreads)
add_ranges(size_t n, int split, const float *__restrict__ part, typename VS::T *__restrict__ vol)
{
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n)
        return;
    float v = part[i];
    for (int r = 1; r < split; ++r)
        v += part[r * n + i];
    VS::st(vol, i, v);
}

// ---- C channels of one geometry in one gather --------------------------------

// A run's rows, their weights and the columns' set-up are the same for every
// channel: per run of NT taps C channels take 8 + NT (2 + C) + 2 C vector
// instructions instead of C (10 + 3 NT), and a brick's ranges and lists are made once.
// For windows that hold C channels in a workgroup's share of the LDS and runs
// of at most 8 taps.  Four channels take bricks of at most eight layers, whose
// sums and taps fit the 168 registers of three waves per SIMD.  Four channels of
// 128^3 x 180 x 256^2, projection and gradient together: 6.50 ms channel by channel, 5.30 so;
// 5.78 as two pairs, 5.89 with sixteen layers (65 registers spilled).
constexpr int kMaxTapsMc = 8;

template <int C>
struct McAdjArgs {
    BrickArgs A;
    const float *ws;       // [n_angles][nv][nu][C], ds-weighted
    float *vol[C];
};

template <int KV, int C>
__global__ void __launch_bounds__(kThreads, 3)
adjoint_mc(McAdjArgs<C> B)
{
    extern __shared__ float lds[];
    const BrickAt b = brick_of_slot(B.A, blockIdx.x & 7, blockIdx.x >> 3);
    if (b.bx < 0)
        return;
    gather_brick<F32, KV, false, C>(B.A, b, 0, B.ws, B.vol, nullptr, lds);
}

struct McSinos {
    const float *y[4];
};

// ds_weight for C channels, packed.
template <int C>
__global__ void __launch_bounds__(kThreads)
ds_weight_mc(DevGeom g, McSinos y, float *__restrict__ out)
{
    const int row = blockIdx.x;   // a * nv + v
    const int a = row / g.nv, v = row - a * g.nv;
    const size_t base = (size_t)row * g.nu;
    const float v2 = g.rows[v].y;
    const ColRec *cols = g.cols + (size_t)a * g.nu;
    for (int u = threadIdx.x; u < g.nu; u += kThreads) {
        const ColRec c = cols[u];
        const float ds = ray_ds(c.dsf, c.n2, v2);
        if constexpr (C == 4)
            *(float4 *)(out + 4 * (base + u)) =
                make_float4(y.y[0][base + u] * ds, y.y[1][base + u] * ds, y.y[2][base + u] * ds,
                            y.y[3][base + u] * ds);
        else
            *(float2 *)(out + 2 * (base + u)) =
                make_float2(y.y[0][base + u] * ds, y.y[1][base + u] * ds);
    }
}

// The ds-weighted copy of a sinogram that the bricks stage from:
// out = y ds(a, u, v) in FP32 (ds by ray_ds, the forward's ray length per
// plane), so that the ray length is computed once per element instead of
// once per brick that stages it.  One workgroup per panel row of one angle
// and channel.
template <class SS>
__global__ void __launch_bounds__(kThreads)
ds_weight(DevGeom g, const typename SS::T *__restrict__ y, float *__restrict__ out)
{
    const int row = blockIdx.x;   // a * nv + v
    const int a = row / g.nv, v = row - a * g.nv;
    const size_t base = ((size_t)blockIdx.y * g.n_angles * g.nv + row) * g.nu;
    const float v2 = g.rows[v].y;
    const ColRec *cols = g.cols + (size_t)a * g.nu;
    for (int u = threadIdx.x; u < g.nu; u += kThreads) {
        const ColRec c = cols[u];
        out[base + u] = SS::wide(SS::raw(y, base + u)) * ray_ds(c.dsf, c.n2, v2);
    }
}

// ---- batched adjoint: one launch over all (case, brick) items ---------------

struct AdjCase {
    BrickArgs A;
    const float *ws;   // the case's ds-weighted sinogram
    void *vol;
    float *part;       // partial volumes of the ranges of angles, if several
};

struct BatchAdjArgs {
    int n_cases, n_items;
    int first[kMaxBatch + 1];   // first slot (per XCD) of each case, its ranges in turn
    AdjCase c[kMaxBatch];
};

template <class VS, bool SOLO>
__global__ void __launch_bounds__(kThreads, 4)
adjoint_batch(BatchAdjArgs B)
{
    extern __shared__ float lds[];
    // one item per workgroup; per XCD the slots of case 0, then case 1, ...,
    // each case's slots mapped to bricks as in adjoint_brick
    const int xc = blockIdx.x & 7, li = blockIdx.x >> 3;
    int cs = 0;
    while (cs + 1 < B.n_cases && li >= B.first[cs + 1])
        ++cs;
    const AdjCase &C = B.c[cs];
    const int slots = slots_per_xcd(C.A), range = (li - B.first[cs]) / slots;
    const BrickAt b = brick_of_slot(C.A, xc, li - B.first[cs] - range * slots);
    if (b.bx < 0)
        return;
    const size_t nvox = (size_t)C.A.g.nx * C.A.g.ny * C.A.g.nz;
    float *part = C.part ? C.part + range * nvox : nullptr;
    typename VS::T *const vs[1] = {(typename VS::T *)C.vol};
    switch (C.A.KV) {   // uniform over the workgroup
    case 4: gather_brick<VS, 4, false, 1, SOLO>(C.A, b, range, C.ws, vs, part, lds); break;
    case 2: gather_brick<VS, 2, false, 1, SOLO>(C.A, b, range, C.ws, vs, part, lds); break;
    default: gather_brick<VS, 1, false, 1, SOLO>(C.A, b, range, C.ws, vs, part, lds); break;
    }
}

}  // namespace

// Window columns, rounded up to even (adj_window_words).
static int even_width(const AdjPlan &p) { return p.W + (p.W & 1); }

// Words of one panel window of C channels with its column records.
static size_t window_words(const AdjPlan &p, int C)
{
    return adj_window_words(p.W, p.WS, C);
}

// With as many windows at a time as a workgroup's share of the LDS holds, a
// group of angles takes two barriers and one round trip to memory instead of
// eight and four.
constexpr size_t kShareWords = kAdjShareWords;

static int windows_at_a_time(const AdjPlan &p, int C)
{
    const size_t w = window_words(p, C);
    return 4 * w <= kShareWords ? 4 : 2 * w <= kShareWords ? 2 : 1;
}

// Words the windows take; a group's column records use them too before fewer
// than four windows are staged.
static size_t window_area(const AdjPlan &p, int C)
{
    const size_t n = windows_at_a_time(p, C), records = (size_t)kGroup * even_width(p) * 4;
    return std::max(n * window_words(p, C), records);
}

static BrickArgs brick_args(const DevGeom &g, const AdjPlan &p, int C = 1, bool solo = false)
{
    const int bk = 4 * p.KV;
    return BrickArgs{g, p.wins, solo ? p.W : even_width(p), p.H, p.WS, (g.nx + kAdjBI - 1) / kAdjBI,
                     (g.ny + kAdjBJ - 1) / kAdjBJ, (g.nz + bk - 1) / bk, p.KV,   // WS: column stride
                     windows_at_a_time(p, C), (int)window_area(p, C), p.split,
                     (g.n_angles + p.split - 1) / p.split, 1.0f - adj_start_delta(g.nv),
                     bk};
}

// The windows, the column ranges and the list of angles, or the final exchange
// (four shares per lane and voxel layer, four waves) if that is larger.
static size_t brick_lds(const AdjPlan &p, int C = 1, bool solo = false)
{
    static_assert(sizeof(AngleEnt) == 8 * sizeof(float), "kAdjSideWords counts eight words");
    const size_t gather =
        solo ? (size_t)p.W * (p.WS + 4) : window_area(p, C) + kAdjSideWords;
    const size_t exchange = (size_t)4 * 4 * 64 * p.KV;
    return std::max(gather, exchange) * sizeof(float);
}

// Workgroups of so much LDS that a CU holds (160 KB, given out in 1280 bytes).
static size_t per_cu(size_t bytes) { return 128 / ((bytes + 1279) / 1280); }

// One angle after another, without the list and the ranges in LDS: where their
// 3 KB would cost a CU one of its (at most four) workgroups, and for fewer
// angles than a group.  Windows of 38 to 40 KB: 182 x 156 x 113 x 180 angles of
// 410 x 330, 3.00 ms with three workgroups and groups of angles, 2.82 with four
// and one by one; shorter bricks with four and groups 3.23.  One angle of
// 512 x 512 into 256^3: 105 us in a group, 95 alone; four angles 209 and 213.
static bool take_solo(const AdjPlan &p, int n_angles)
{
    const size_t grouped = std::min<size_t>(per_cu(brick_lds(p)), 4);
    const size_t solo = std::min<size_t>(per_cu(brick_lds(p, 1, true)), 4);
    return solo > grouped || n_angles < kGroup;
}

// Words of the ranges' volumes of n voxels.
static size_t part_words(const AdjPlan &p, size_t n) { return p.split > 1 ? n * p.split : 0; }

template <class VS>
static void launch_add_ranges(size_t n, int split, const float *part, typename VS::T *vol,
                              hipStream_t s)
{
    hipLaunchKernelGGL(add_ranges<VS>, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, n, split, part, vol);
}

static hipError_t launch_ds_weight(const DevGeom &g, const void *sino, cbct_dtype st, float *ws,
                                   int channels, hipStream_t s)
{
    dim3 grid((unsigned)(g.n_angles * g.nv), channels), block(kThreads);
    // the volume type plays no part here: dispatch on (F32, st)
    return dispatch_storage(CBCT_F32, st, [&](auto, auto ss) -> hipError_t {
        using SS = decltype(ss);
        hipLaunchKernelGGL((ds_weight<SS>), grid, block, 0, s, g, (const typename SS::T *)sino, ws);
        return hipGetLastError();
    });
}

// Bricks from which channels are gathered together: four workgroups per CU are
// left (with fewer, the channels' bricks side by side fill the chip better).
constexpr long kMcBricks = 1024;

int adjoint_mc_channels(const cbct_geom *g, int left)
{
    const AdjPlan &p = g->adj;
    // adjoint_mc gathers all angles in one range
    if (!p.ok || p.split > 1 || p.NTmax > kMaxTapsMc)
        return 1;
    const BrickArgs A = brick_args(g->dev, p);
    if ((long)A.nbx * A.nby * A.nbz < kMcBricks)
        return 1;
    for (int c : {4, 2})
        if (left >= c && window_words(p, c) <= kShareWords)
            return c;
    return 1;
}

template <int C>
static hipError_t launch_mc(const cbct_geom *g, const float *const *sinos, float *const *vols,
                            float *ws, hipStream_t s)
{
    const DevGeom &d = g->dev;
    AdjPlan p = g->adj;
    if (C == 4)
        p.KV = std::min(p.KV, 2);   // the plan's window holds the shorter bricks' too
    McAdjArgs<C> B{brick_args(d, p, C), ws, {}};
    B.A.plan_bk = 4 * g->adj.KV;
    McSinos y{};
    for (int c = 0; c < C; ++c) {
        B.vol[c] = vols[c];
        y.y[c] = sinos[c];
    }
    const size_t lds = brick_lds(p, C);
    const dim3 grid(8 * slots_per_xcd(B.A)), block(kThreads);
    hipLaunchKernelGGL(ds_weight_mc<C>, dim3((unsigned)(d.n_angles * d.nv)), block, 0, s, d, y, ws);
    if constexpr (C == 2) {
        if (p.KV == 4) {
            hipLaunchKernelGGL((adjoint_mc<4, 2>), grid, block, lds, s, B);
            return hipGetLastError();
        }
    }
    if (p.KV == 2)
        hipLaunchKernelGGL((adjoint_mc<2, C>), grid, block, lds, s, B);
    else
        hipLaunchKernelGGL((adjoint_mc<1, C>), grid, block, lds, s, B);
    return hipGetLastError();
}

hipError_t launch_adjoint_mc(const cbct_geom *g, int C, const float *const *sinos,
                             float *const *vols, hipStream_t s)
{
    const size_t nsino = (size_t)g->dev.n_angles * g->dev.nv * g->dev.nu;
    ScratchLease lease;
    hipError_t e = scratch_acquire(nsino * C * sizeof(float), s, lease);
    if (e == hipSuccess)
        e = C == 4 ? launch_mc<4>(g, sinos, vols, (float *)lease.ptr, s)
                   : launch_mc<2>(g, sinos, vols, (float *)lease.ptr, s);
    const hipError_t r = scratch_release(s, lease);
    return e != hipSuccess ? e : r;
}

static hipError_t gather_channels(const DevGeom &g, const AdjPlan &p, const void *sino,
                                  cbct_dtype st, void *vol, cbct_dtype vt, int channels,
                                  hipStream_t s)
{
    const bool solo = take_solo(p, g.n_angles);
    BrickArgs A = brick_args(g, p, 1, solo);
    dim3 grid(8 * slots_per_xcd(A), channels, p.split), block(kThreads);
    const size_t nsino = (size_t)g.n_angles * g.nv * g.nu * channels;
    const size_t nvox = (size_t)g.nx * g.ny * g.nz * channels;
    ScratchLease lease;
    hipError_t e = scratch_acquire((nsino + part_words(p, nvox)) * sizeof(float), s, lease);
    if (e == hipSuccess)
        e = launch_ds_weight(g, sino, st, (float *)lease.ptr, channels, s);
    if (e == hipSuccess)
        e = dispatch_storage(vt, st, [&](auto vs, auto) -> hipError_t {
            using VS = decltype(vs);
            const size_t lds = brick_lds(p, 1, solo);
            const float *w = (const float *)lease.ptr;
            float *part = p.split > 1 ? (float *)lease.ptr + nsino : nullptr;
            auto *x = (typename VS::T *)vol;
            auto launch = [&](auto one, auto grouped) {
                hipLaunchKernelGGL(solo ? one : grouped, grid, block, lds, s, A, w, x, part);
            };
            if (adj_tall(p.KV, p.WS))
                launch(adjoint_brick<VS, 4, true, true>, adjoint_brick<VS, 4, true, false>);
            else if (p.KV == 4)
                launch(adjoint_brick<VS, 4, false, true>, adjoint_brick<VS, 4, false, false>);
            else if (p.KV == 2)
                launch(adjoint_brick<VS, 2, false, true>, adjoint_brick<VS, 2, false, false>);
            else
                launch(adjoint_brick<VS, 1, false, true>, adjoint_brick<VS, 1, false, false>);
            if (part)
                launch_add_ranges<VS>(nvox, p.split, part, x, s);
            return hipGetLastError();
        });
    const hipError_t r = scratch_release(s, lease);
    return e != hipSuccess ? e : r;
}

// Staged projections and partial volumes held at a time: stacks that take more
// run in several launches.
constexpr size_t kStageBytes = (size_t)4 << 30;

hipError_t launch_adjoint_brick(const DevGeom &g, const AdjPlan &p, const void *sino,
                                cbct_dtype st, void *vol, cbct_dtype vt, int channels,
                                hipStream_t s)
{
    const size_t nvox = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.n_angles * g.nv * g.nu;
    const size_t one = (nsino + part_words(p, nvox)) * sizeof(float);
    const int most = (int)std::max<size_t>(1, std::min<size_t>(channels, kStageBytes / one));
    for (int c0 = 0; c0 < channels; c0 += most) {
        const hipError_t e =
            gather_channels(g, p, (const char *)sino + c0 * nsino * storage_bytes(st), st,
                            (char *)vol + c0 * nvox * storage_bytes(vt), vt,
                            std::min(most, channels - c0), s);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_adjoint_batch(int n, const cbct_geom *const *gs, const void *const *sinos,
                                void *const *vols, cbct_dtype st, cbct_dtype vt, hipStream_t s)
{
    BatchAdjArgs B{};
    B.n_cases = n;
    size_t lds = 0, total = 0;
    int items = 0;
    size_t off[kMaxBatch], parts[kMaxBatch];
    bool solo = false;
    for (int i = 0; i < n; ++i)
        solo = solo || take_solo(gs[i]->adj, gs[i]->dev.n_angles);
    for (int i = 0; i < n; ++i) {
        const cbct_geom *g = gs[i];
        B.first[i] = items;
        B.c[i] = AdjCase{brick_args(g->dev, g->adj, 1, solo), nullptr, vols[i], nullptr};
        items += slots_per_xcd(B.c[i].A) * g->adj.split;
        lds = std::max(lds, brick_lds(g->adj, 1, solo));
        off[i] = total;
        total += (size_t)g->dev.n_angles * g->dev.nv * g->dev.nu;
        parts[i] = total;
        total += part_words(g->adj, (size_t)g->dev.nx * g->dev.ny * g->dev.nz);
    }
    B.first[n] = items;
    B.n_items = items;
    const int grid = 8 * items;
    ScratchLease lease;
    hipError_t e = scratch_acquire(total * sizeof(float), s, lease);
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        B.c[i].ws = (const float *)lease.ptr + off[i];
        if (gs[i]->adj.split > 1)
            B.c[i].part = (float *)lease.ptr + parts[i];
        e = launch_ds_weight(gs[i]->dev, sinos[i], st, (float *)lease.ptr + off[i], 1, s);
    }
    if (e == hipSuccess)
        e = dispatch_storage(vt, st, [&](auto vs, auto) -> hipError_t {
            using VS = decltype(vs);
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), lds, s, B);
            };
            solo ? launch(adjoint_batch<VS, true>) : launch(adjoint_batch<VS, false>);
            for (int i = 0; i < n; ++i)
                if (B.c[i].part)
                    launch_add_ranges<VS>((size_t)B.c[i].A.g.nx * B.c[i].A.g.ny * B.c[i].A.g.nz,
                                          B.c[i].A.split, B.c[i].part, (typename VS::T *)vols[i], s);
            return hipGetLastError();
        });
    const hipError_t r = scratch_release(s, lease);
    return e != hipSuccess ? e : r;
}

}  // namespace cbct
