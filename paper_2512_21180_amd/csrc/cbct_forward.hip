// Forward projector A for gfx950: plane sweep over LDS-staged boxes.
//
// Operator: the plane-sampled cone-beam line integral (arXiv 2512.21180,
// Sec. 2.2, projection operator P).  A workgroup owns one tile of up to 64
// columns x 4R rows of one angle, all sampled along the same axis; wave w
// holds rows [w R, w R + R) and lane l column u0 + l, so each thread carries
// R rays of one column and shares their in-plane interpolation index.  Where
// 64 columns of rays spread over more than 64 voxels (pixels coarser than
// voxels), tiles are 32 columns x 8R rows: lane l then holds column l % 32
// and the rows of row group 2w + l / 32.
//
// The tile sweeps the voxel-centre planes of its axis.  On plane p every ray
// of the tile lands inside a box of at most 64 (in-plane) x 32 (z) voxels
// spanned by the corner rays (the boxes of all planes are tabulated in LDS
// at the tile's start); the box is staged in LDS (zero outside the volume)
// one plane ahead of its use, double-buffered, one barrier per plane.
// Each sample is the bilinear interpolant read from LDS; each ray keeps its
// own running sum in a register, so the summation order is the plane order
// whatever the launch shape, and the result is written once, coalesced along
// the detector row.  Tiles are assigned XCD-contiguously so that the
// workgroups sharing an L2 work on neighbouring tiles of the same angle.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cbct_internal.h"
#include "cbct_lds.h"
#include "cbct_transpose.h"
#include "cbct_storage.h"

namespace cbct {
namespace {

constexpr int kThreads = 256;
// Planes whose boxes are loaded ahead (two: 7.83 ms against 7.82, 11 registers more).
constexpr int kPlanes = 1;
// Rays whose LDS reads run ahead of the arithmetic.  With all eight rays' reads
// first (as the compiler orders them when nothing holds it) a wave's reads
// leave in a burst that keeps the others' waiting, and take 100 registers:
// clinical forward 9.6 ms; 8.11 one ray ahead, 8.13 two, 8.21 three, 8.35 four
// (at five waves per SIMD).
constexpr int kAhead = 1;
// Volume copies made at a time: stacks and batches whose copies take more run in
// several launches (each of half a billion voxels), as do those whose copies
// find no memory; a single volume's copies that find none are not made, and
// its rays summed one per thread instead.
constexpr size_t kCopyBytes = (size_t)4 << 30;

constexpr int kQS = 68;        // LDS row stride (floats): box rows are <= 64 wide
constexpr int kMaxRows = 32;   // box rows (z) per plane
constexpr int kBoxChunk = 256; // planes whose boxes are tabulated at a time
static_assert(kBoxChunk == kThreads, "the box table is filled one plane per thread");
// LDS: two staging boxes, then the box table (one int4 per plane of a chunk)
constexpr size_t kFwdLds = 2 * (size_t)kMaxRows * kQS * sizeof(float) + kBoxChunk * 16;

// Sweep one tile.  R (rays per thread) is a property of the plan; the per
// ray arithmetic does not depend on it, so any launch shape gives the same
// bits.  `lds` holds two boxes of kMaxRows x kQS floats and the box table.
//
// On plane p the box spans in-plane indices [qlo, qlo + qw) and z indices
// [klo, klo + kw), from the corner rays' crossings widened by one voxel for
// rounding; a wave stages four rows per load, a quad of voxels per lane.
// tub: log2 of the tile width (6 or 5).  R: rays per thread, fixed at compile
// time: the plans take 8, 4, 2 or 1, and a kernel with arrays of eight rays
// for any of them spills 22 of its 72 registers, some reloads per plane.
// v: the volume in FP32, vt: the same with x and y swapped ([nz][nx][ny]).  Tiles that
// sweep x planes read their boxes from it, so a box row (fixed z, in-plane
// index y) is contiguous; in the volume itself its voxels lie nx apart, a
// cache line each (the clinical forward, an earlier build: 12.2 ms reading
// them strided, 8.8 ms from the transposed copy).
template <class SS, int R>
__device__ __forceinline__ void sweep_tile(const DevGeom &g, const TileRec &T, int tub,
                           const float *__restrict__ v, const float *__restrict__ vt,
                           typename SS::T *__restrict__ sino, float *lds)
{
    const int tid = threadIdx.x;
    // the wave index is uniform: the staging's slot tests below are scalar
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int uc = lane & ((1 << tub) - 1);                   // tile column
    const int row0 = ((w << (6 - tub)) + (lane >> tub)) * R;  // first tile row
    const int ul = min(uc, T.nu_t - 1);
    const ColRec c = g.cols[(size_t)T.a * g.nu + T.u0 + ul];

    float kb[R], ks[R], acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int vr = T.v0 + min(row0 + r, T.nv_t - 1);
        const float vz = g.rows[vr].x;
        kb[r] = fmaf(c.t0, vz, g.Kb);
        ks[r] = c.tau * vz;
        acc[r] = 0.0f;
    }

    // corner rays (uniform): columns u0 and u0 + nu_t - 1, rows v0 and v0 + nv_t - 1
    const ColRec cA = g.cols[(size_t)T.a * g.nu + T.u0];
    const ColRec cB = g.cols[(size_t)T.a * g.nu + T.u0 + T.nu_t - 1];
    const float zA = g.rows[T.v0].x, zB = g.rows[T.v0 + T.nv_t - 1].x;
    const float kbA0 = fmaf(cA.t0, zA, g.Kb), ksA0 = cA.tau * zA;
    const float kbA1 = fmaf(cA.t0, zB, g.Kb), ksA1 = cA.tau * zB;
    const float kbB0 = fmaf(cB.t0, zA, g.Kb), ksB0 = cB.tau * zA;
    const float kbB1 = fmaf(cB.t0, zB, g.Kb), ksB1 = cB.tau * zB;

    const bool xp = T.cls == 0;
    const int nq = xp ? g.ny : g.nx;
    const float *src = xp ? vt : v;    // rows of nq voxels between zero pads
    const int sp = sweep_pitch(nq);    // plane stride
    const int sk = sp * (xp ? g.nx : g.ny);   // z stride
    struct Box {
        int qlo, klo, qw, kw;
    };
    // The box of every plane is computed once per tile, one plane per
    // thread, into an LDS table of kBoxChunk planes (refilled when the sweep
    // passes a chunk); the sweep reads it back as wave-uniform values.
    int4 *boxes = (int4 *)(lds + 2 * kMaxRows * kQS);
    auto fill_boxes = [&](int base) {
        const int p = base + tid;
        if (p <= T.p_hi) {
            const float fp = (float)p;
            const float qa = fmaf(fp, cA.ps, cA.pb), qb = fmaf(fp, cB.ps, cB.pb);
            const float k0 = fmaf(fp, ksA0, kbA0), k1 = fmaf(fp, ksA1, kbA1);
            const float k2 = fmaf(fp, ksB0, kbB0), k3 = fmaf(fp, ksB1, kbB1);
            const int qlo = (int)floorf(fminf(qa, qb)) - 1;
            const int klo = (int)floorf(fminf(fminf(k0, k1), fminf(k2, k3))) - 1;
            const int qw = min((int)floorf(fmaxf(qa, qb)) + 3 - qlo, 64);
            const int kw = min((int)floorf(fmaxf(fmaxf(k0, k1), fmaxf(k2, k3))) + 3 - klo, kMaxRows);
            boxes[tid] = make_int4(qlo, klo, qw, kw);
        }
    };
    auto box_of = [&](int p, int base) {
        const int4 v = boxes[p - base];
        Box b;
        b.qlo = __builtin_amdgcn_readfirstlane(v.x);
        b.klo = __builtin_amdgcn_readfirstlane(v.y);
        b.qw = __builtin_amdgcn_readfirstlane(v.z);
        b.kw = __builtin_amdgcn_readfirstlane(v.w);
        return b;
    };
    // A wave's load takes four box rows of up to 16 quads of voxels (row
    // 4 s + lane / 16, quad lane % 16 for slot s; wave w has slots w and w + 4),
    // so a plane's box takes five loads and five LDS stores of 16 bytes a lane
    // in all, where a load per row took four times as many.  A quad that
    // straddles the volume's edge reads the row's zero pad; lanes
    // outside the volume or the box get an offset past the end, for which the
    // buffer resource returns zero.  The values stay in registers until the
    // LDS store, so the loads of the next plane stay in flight while this
    // plane is summed.
    const uint32_t vbytes = (uint32_t)sk * (uint32_t)g.nz * (uint32_t)sizeof(float);
    const __amdgpu_buffer_rsrc_t vres =
        __builtin_amdgcn_make_buffer_rsrc((void *)src, (short)0, (int)vbytes, kBufferWord3);
    const int quad = 4 * (lane & 15), srow = 4 * w + (lane >> 4);
    const uint32_t lane_off = 4u * ((uint32_t)srow * (uint32_t)sk + (uint32_t)quad + kSweepPad);
    auto fetch = [&](int p, const Box &b, float4 (&st)[2]) {
        const bool qin = quad < b.qw && (unsigned)(b.qlo + quad + 3) < (unsigned)(nq + 3);
        // modular: exact for quads inside the volume
        const uint32_t off0 = lane_off + 4u * ((uint32_t)b.qlo + (uint32_t)p * (uint32_t)sp +
                                               (uint32_t)b.klo * (uint32_t)sk);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (i == 0 || b.kw > 4 * w + 16) {
                const bool in = qin && (unsigned)(b.klo + srow + 16 * i) < (unsigned)g.nz;
                // the offset stays alive past its load (the empty asm), so it
                // cannot be formed in the load's own registers: those may
                // still await an earlier load, and the wave would then wait
                // for all loads in flight here
                const uint32_t off = in ? off0 + (uint32_t)i * 64u * (uint32_t)sk : vbytes;
                const auto d = __builtin_amdgcn_raw_buffer_load_b128(vres, (int)off, 0, 0);
                st[i] = make_float4(__uint_as_float(d[0]), __uint_as_float(d[1]),
                                    __uint_as_float(d[2]), __uint_as_float(d[3]));
                asm volatile("" ::"v"(off));
            }
    };

    __syncthreads();   // the previous work item's readers of lds are done
    int p = T.p_lo, base = T.p_lo;
    fill_boxes(base);
    __syncthreads();
    // One plane: store its box (in registers since kPlanes planes ago), start
    // the loads of the plane kPlanes later into the same registers, sum the rays.
    auto plane = [&](int p, Box &bx, float4 (&stage)[2]) {
        float *buf = lds + (p & 1) * (kMaxRows * kQS);
        const Box cb = bx;
        float *dst = buf + srow * kQS + quad;
        *(float4 *)dst = stage[0];
        if (cb.kw > 4 * w + 16)
            *(float4 *)(dst + 16 * kQS) = stage[1];
        __syncthreads();
        if (p + kPlanes <= T.p_hi) {
            if (p + kPlanes - base == kBoxChunk) {   // uniform: next chunk of boxes
                base += kBoxChunk;
                fill_boxes(base);   // every reader of the old chunk is past the barrier
                __syncthreads();
            }
            bx = box_of(p + kPlanes, base);
            fetch(p + kPlanes, bx, stage);
        }
        const float fp = (float)p;
        const float q = fmaf(fp, c.ps, c.pb);
        const float qf = floorf(q);
        const float wq = q - qf;
        // byte address this column would have in z row 0 (the box's first
        // row, klo, lies at its position in box row 0)
        const int colz =
            (int)(lds_addr(buf) + 4u * (uint32_t)((int)qf - cb.qlo)) - cb.klo * (4 * kQS);
        // ray r's arithmetic runs while the reads of the next kAhead rays are
        // in flight; the scheduling barriers keep that order
        float wk[R], v00[R], v10[R], v01[R], v11[R];
        auto read = [&](int r) {
            // z index k of the ray on this plane: its weight is the
            // exact fraction of k, its row address one floor conversion
            // and one multiply-add (every ray's floor(k) lies in the box
            // rows [klo, klo + kw - 1), so the address is inside the box)
            const float k = fmaf(fp, ks[r], kb[r]);
            wk[r] = __builtin_amdgcn_fractf(k);
            const lds_float *row = lds_ptr((uint32_t)mad_i24(floor_i32(k), 4 * kQS, colz));
            v00[r] = row[0];
            v10[r] = row[1];
            v01[r] = row[kQS];
            v11[r] = row[kQS + 1];
        };
#pragma unroll
        for (int r = 0; r < kAhead; ++r)
            read(r);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            __builtin_amdgcn_sched_barrier(0);
            if (r + kAhead < R)
                read(r + kAhead);
            __builtin_amdgcn_sched_barrier(0);
            const float lo = fmaf(wq, v10[r] - v00[r], v00[r]);
            const float hi = fmaf(wq, v11[r] - v01[r], v01[r]);
            acc[r] += fmaf(wk[r], hi - lo, lo);
        }
    };
    Box nb[kPlanes];
    float4 stage[kPlanes][2];
#pragma unroll
    for (int i = 0; i < kPlanes; ++i)
        if (p + i <= T.p_hi) {
            nb[i] = box_of(p + i, base);
            fetch(p + i, nb[i], stage[i]);
        }
    while (p <= T.p_hi) {
#pragma unroll
        for (int i = 0; i < kPlanes; ++i) {
            if (p > T.p_hi)
                break;
            plane(p, nb[i], stage[i]);
            ++p;
        }
    }

    if (uc < T.nu_t) {
        // every ray's length factor first, its row record loaded with the
        // others' (the empty asm keeps the compiler from moving each load
        // behind its ray's store test, where the loads would wait one by one)
        // (the row index passes through an empty asm here, so that the
        // loads are not hoisted above the sweep, where they would hold
        // eight registers throughout)
        int rb = row0;
        asm volatile("" : "+v"(rb));
        float ds[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            ds[r] = g.rows[T.v0 + min(rb + r, T.nv_t - 1)].y;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ds[r] = ray_ds(c.dsf, c.n2, ds[r]);
            asm volatile("" : "+v"(ds[r]));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int vr = row0 + r;
            if (vr < T.nv_t)
                SS::st(sino, ((size_t)T.a * g.nv + T.v0 + vr) * g.nu + T.u0 + uc, acc[r] * ds[r]);
        }
    }
}

struct SweepArgs {
    DevGeom g;
    const TileRec *tiles;
    int tub;   // log2 of the tile width
};

// Seven waves per SIMD (72 registers; the LDS of seven workgroups fits a CU).
// The sweep is bound by the LDS pipe: its reads of two words and its 16-byte
// stores keep it busy for all of the 1.65e7 cycles (clinical case), the 5.2e9
// VALU instructions (two cycles for an add or FMA, four for a fraction, a
// conversion or a 24-bit multiply-add) for three quarters; more waves fill the
// gaps between dependent reads: 8.06 ms at five, 7.84 at six, 7.71 at seven.
template <class SS, int R>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7, 7)))
forward_sweep(SweepArgs A, const float *__restrict__ vol, const float *__restrict__ volt,
              typename SS::T *__restrict__ sino)
{
    extern __shared__ float lds[];
    // XCD-contiguous tile order: workgroups are dealt to the 8 XCDs round
    // robin, so XCD x receives ids x, x+8, ...; give it tiles
    // [x * n/8, (x+1) * n/8).
    const int nb = gridDim.x;
    const int t = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
    const TileRec T = A.tiles[t];
    if (T.nu_t == 0)
        return;
    const int ch = blockIdx.y;
    const size_t nsino = (size_t)A.g.n_angles * A.g.nv * A.g.nu;
    const size_t nv = (size_t)A.g.nz * A.g.ny * sweep_pitch(A.g.nx);
    const size_t nt = (size_t)A.g.nz * A.g.nx * sweep_pitch(A.g.ny);
    sweep_tile<SS, R>(A.g, T, A.tub, vol + ch * nv, volt + ch * nt, sino + ch * nsino, lds);
}

// ---- batched forward: one launch over all (case, tile) items ----------------

struct FwdCase {
    DevGeom g;
    const TileRec *tiles;
    int R, tub, n_tiles;
    const float *vol, *volt;   // the volume, and with x and y swapped
    void *sino;
};

struct BatchFwdArgs {
    int n_cases, n_items;
    int first[kMaxBatch + 1];   // first item of each case
    FwdCase c[kMaxBatch];
};

template <class SS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(7, 7)))
forward_batch(BatchFwdArgs B)
{
    extern __shared__ float lds[];
    // one item per workgroup, XCD-contiguous as in forward_sweep; the
    // hardware dispatcher balances the uneven items
    const int per = gridDim.x >> 3;
    const int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (item >= B.n_items)
        return;
    int cs = 0;
    while (cs + 1 < B.n_cases && item >= B.first[cs + 1])
        ++cs;
    const FwdCase &C = B.c[cs];
    const TileRec T = C.tiles[item - B.first[cs]];
    if (T.nu_t == 0)
        return;
    auto *sino = (typename SS::T *)C.sino;
    switch (C.R) {   // uniform over the workgroup; the bits do not depend on it
    case 8: sweep_tile<SS, 8>(C.g, T, C.tub, C.vol, C.volt, sino, lds); break;
    case 4: sweep_tile<SS, 4>(C.g, T, C.tub, C.vol, C.volt, sino, lds); break;
    case 2: sweep_tile<SS, 2>(C.g, T, C.tub, C.vol, C.volt, sino, lds); break;
    default: sweep_tile<SS, 1>(C.g, T, C.tub, C.vol, C.volt, sino, lds); break;
    }
}

}  // namespace

// The sweep of `channels` channels, staged from copies in the library's device
// buffer (in FP32, with x and y swapped for the tiles that sweep x planes).
static hipError_t sweep_channels(const DevGeom &g, const FwdPlan &p, const void *vol, cbct_dtype vt,
                                 void *sino, cbct_dtype st, int channels, hipStream_t s)
{
    SweepArgs A{g, p.tiles, p.TU == 32 ? 5 : 6};
    const size_t lds = kFwdLds;
    dim3 grid(p.n_tiles, channels), block(kThreads);
    ScratchLease lease;
    hipError_t e = scratch_acquire(
        sweep_words(g.nx, g.ny, (size_t)g.nz * channels, p.axes) * sizeof(float), s, lease);
    if (e == hipSuccess) {
        const SweepVolumes v =
            make_sweep_volumes(vol, vt, (float *)lease.ptr, g.nx, g.ny, g.nz * channels, p.axes, s);
        e = dispatch_storage(vt, st, [&](auto, auto ss) -> hipError_t {
            using SS = decltype(ss);
            auto *y = (typename SS::T *)sino;
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, grid, block, lds, s, A, v.vol, v.volt, y);
            };
            switch (p.R) {
            case 8: launch(forward_sweep<SS, 8>); break;
            case 4: launch(forward_sweep<SS, 4>); break;
            case 2: launch(forward_sweep<SS, 2>); break;
            default: launch(forward_sweep<SS, 1>); break;
            }
            return hipGetLastError();
        });
    }
    const hipError_t r = scratch_release(s, lease);
    return e != hipSuccess ? e : r;
}

hipError_t launch_forward_tiled(const DevGeom &g, const FwdPlan &p, const void *vol,
                                cbct_dtype vt, void *sino, cbct_dtype st, int channels,
                                hipStream_t s)
{
    const size_t nvox = (size_t)g.nx * g.ny * g.nz, nsino = (size_t)g.n_angles * g.nv * g.nu;
    const size_t one = sweep_words(g.nx, g.ny, g.nz, p.axes) * sizeof(float);
    int most = (int)std::max<size_t>(1, std::min<size_t>(channels, kCopyBytes / std::max<size_t>(one, 1)));
    for (int c0 = 0; c0 < channels;) {
        const int c = std::min(most, channels - c0);
        const char *x = (const char *)vol + c0 * nvox * storage_bytes(vt);
        char *y = (char *)sino + c0 * nsino * storage_bytes(st);
        hipError_t e = sweep_channels(g, p, x, vt, y, st, c, s);
        if (e == hipErrorOutOfMemory) {   // before any work was enqueued
            (void)hipGetLastError();
            if (c > 1) {
                most = c / 2;
                continue;
            }
            e = launch_forward_simple(g, x, vt, y, st, 1, s);
        }
        if (e != hipSuccess)
            return e;
        c0 += c;
    }
    return hipSuccess;
}

hipError_t launch_forward_batch(int n, const cbct_geom *const *gs, const void *const *vols,
                                void *const *sinos, cbct_dtype vt, cbct_dtype st, hipStream_t s)
{
    BatchFwdArgs B{};
    B.n_cases = n;
    int items = 0;
    size_t off[kMaxBatch], total = 0;   // words of the cases' copies in the library's buffer
    for (int i = 0; i < n; ++i) {
        const cbct_geom *g = gs[i];
        B.first[i] = items;
        B.c[i] = FwdCase{g->dev, g->fwd.tiles, g->fwd.R, g->fwd.TU == 32 ? 5 : 6,
                         g->fwd.n_tiles, nullptr, nullptr, sinos[i]};
        items += g->fwd.n_tiles;
        off[i] = total;
        total += (sweep_words(g->dev.nx, g->dev.ny, g->dev.nz, g->fwd.axes) + 63) & ~(size_t)63;
    }
    B.first[n] = items;
    B.n_items = items;
    const int grid = (items + 7) / 8 * 8;
    // fewer cases at a time, down to one
    auto in_parts = [&]() -> hipError_t {
        if (n == 1)
            return launch_forward_tiled(gs[0]->dev, gs[0]->fwd, vols[0], vt, sinos[0], st, 1, s);
        const int h = n / 2;
        const hipError_t e = launch_forward_batch(h, gs, vols, sinos, vt, st, s);
        return e != hipSuccess ? e
                               : launch_forward_batch(n - h, gs + h, vols + h, sinos + h, vt, st, s);
    };
    if (total * sizeof(float) > kCopyBytes)
        return in_parts();
    ScratchLease lease;
    hipError_t e = scratch_acquire(total * sizeof(float), s, lease);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        (void)scratch_release(s, lease);
        return in_parts();
    }
    if (e == hipSuccess) {
        for (int i = 0; i < n; ++i) {
            const DevGeom &d = gs[i]->dev;
            const SweepVolumes v = make_sweep_volumes(vols[i], vt, (float *)lease.ptr + off[i],
                                                      d.nx, d.ny, d.nz, gs[i]->fwd.axes, s);
            B.c[i].vol = v.vol;
            B.c[i].volt = v.volt;
        }
        e = dispatch_storage(vt, st, [&](auto, auto ss) -> hipError_t {
            hipLaunchKernelGGL((forward_batch<decltype(ss)>), dim3(grid), dim3(kThreads), kFwdLds, s, B);
            return hipGetLastError();
        });
    }
    const hipError_t r = scratch_release(s, lease);
    return e != hipSuccess ? e : r;
}

}  // namespace cbct
