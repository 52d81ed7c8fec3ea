// apply_impl.hpp -- the hot path: r = c u + D[u] - S[q] as the zero-padded
// FFT convolution of eq. (16), in four kernels.
//
//   k_fwd_xy   per occupied z-plane and chunk of kx: scatter of the boundary
//              fields (Fig. 4) fused with their x-transform, done as a direct
//              DFT over the few nodes of each grid row (the field is zero
//              elsewhere), then the y-FFT in LDS.   -> Y[f][kx][z][ky]
//   k_zpass    per (kx, tile of ky): forward z-FFT of every field (input zero
//              outside the occupied planes), products with the compact kernel
//              spectra summed into each output (eqs. 15-16), inverse z-FFT,
//              keep the occupied planes (zsched.hpp).  -> Z[o][kx][z][ky]
//   k_inv_y    per occupied z-plane and chunk of kx: inverse y-FFT in
//              registers/LDS, rows y < ny stored with kx contiguous
//                                                      -> W[o][z][y][kx] (in Y)
//   k_gather   eight lanes per node: the inverse x-transform of its row
//              evaluated only at its own x (Sec. 4: only the boundary
//              values are needed), plus c u and the self-term
//              correction                              -> r
//              (nodes of long rows read their row's inverse FFT, made by
//              k_rows_inv, instead)
//
// 2D plans: k_mid2d takes the place of the first three (one kx per block, no Y
// and Z), with the fields folded in for few nodes; k_gather_wide or
// k_rows_gather that of the last where the plan's kFlat bits say so.
//
// Layout: complex intermediates are interleaved (re, im) in the working
// precision R.  Y is tiled for the z pass, [f][kx][ky / KT][z][KT] (the 16-bit
// form: [f][kx][z][ky]); Z is [o][kx][z][ky].  Kernel spectra
// are reals over one octant in the order of spec_index (16-bit form:
// [c][kx][ky][kz]).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fft_device.hpp"
#include "internal.hpp"
#include "kinds.hpp"
#include "zsched.hpp"

namespace bemfft {

struct ApplyArgs {
    int nx, ny, nz;
    int px, py, pz;
    int hx, hy, hz;
    int hzs;          // stored kz row length of the spectra (hz, or padded)
    int z0, nzo;
    int m;
    int zsched;       // radix schedule of the z pass (0, 1, or 2 for Navier)
    int64_t off;      // batched apply: offset of this member's q, u, r
    int gid;          // batched apply: member index in the whole batch
    const int *gx, *gy, *gz, *rowptr, *perm;
    const double *w, *nrm, *C, *SC;
    const double *q, *u;
    double *r;
    const void *spec, *twx, *twy, *twz;
    void *vf;  // [F][m] boundary fields in sorted order, working precision
    void *Xd;  // [nd][F][hx] transforms of the long rows
    const int *row_dense;   // [nzo * ny]: index into dense_rows, or -1
    const int *dense_rows;  // [nd]: row index (zz * ny + y) of each long row
    int nd;
    int flat;               // 2D: the kernels of the plan, kFlat bits
    int row_inv;            // 1: the long rows' inverse x transform is an FFT (k_rows_inv)
    int fwd_xg;             // kx per thread in the forward direct DFT (1 or 2)
    void *Y, *Z;
};

// Consecutive members of a group with one z length and schedule.
struct ZRange {
    int first, nmem, pz, zsched;
};

// Launch extents of one group of batch members (same family, precision and padded
// x and y sizes): the largest per-member extents.  Members whose bodies occupy
// different numbers of planes differ in their z length; only the z pass is
// launched by length, so that many small bodies still fill the chip.
struct GroupDims {
    int nmem;
    int max_m, max_nd, max_nzo;
    int hx, px, py;
    int row_inv;  // some member takes the row FFT for its long rows
    int flat;     // 2D: kFlat bits of every member
    const ZRange *z;  // 3D: host array of nz ranges
    int nz;
};

// The 2D kernels that a plan takes (flat_rule in api.hip; a batch's members take
// their own plan's): k_mid2d with the fields folded in, k_gather_wide, k_rows_gather.
constexpr int kFlatFold = 1, kFlatWide = 2, kFlatRows = 4;
constexpr int kWaveRow = 8;  // longer rows are summed by a wavefront in the folded form

// Base pointers of a batched apply (device memory, so that a captured graph
// of the launches serves any call) and the members still iterating.
struct BatchIO {
    const double *q, *u;
    double *r;
    const int *active;  // null: all members
};

__host__ __device__ constexpr int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }
__host__ __device__ constexpr int mini(int a, int b) { return a < b ? a : b; }
constexpr int kMaxPx = 1024;         // largest padded length along x (2D plans; 3D stop at 512)

// Complex value stored in 16 bits per part (the intermediates Y and Z of the
// 16-bit form); arithmetic stays FP32.
struct alignas(4) cbf16 {
    __bf16 x, y;
};
// Storage conversions: identity for cx<R>, FP32 <-> BF16 (round to nearest
// even) for cbf16.
template <typename S, typename R>
__device__ __forceinline__ S to_store(cx<R> v) {
    if constexpr (std::is_same<S, cbf16>::value) return cbf16{(__bf16)(float)v.x, (__bf16)(float)v.y};
    else return v;
}
template <typename R, typename S>
__device__ __forceinline__ cx<R> from_store(S v) {
    if constexpr (std::is_same<S, cbf16>::value) return cx<R>{(R)(float)v.x, (R)(float)v.y};
    else return v;
}

// (k x) mod p for 0 <= k x < 2^24, with a float estimate of the quotient.
__device__ __forceinline__ int mod_small(int kx, int x, int p, float inv_p) {
    const int prod = kx * x;
    int r = prod - (int)((float)prod * inv_p) * p;
    if (r < 0) r += p;
    if (r >= p) r -= p;
    return r;
}

// Schedules of the 2D plans' transforms.  Few pencils are in flight and each
// waits for its own instructions, so more lanes with fewer points each are
// faster than the bulk schedules (256 points in FP64: 1.8 us at 16 points per
// lane, 0.9 at 4; 512 in FP32: 1.8 at 16, 1.1 at 8), as far as a pencil stays in one wavefront.
template <int P> struct FlatShape : PencilShape<P> {};
template <> struct FlatShape<32> : FFTShape<32, 8, 4, 4, 2> {};
template <> struct FlatShape<64> : FFTShape<64, 16, 4, 4, 4> {};
template <> struct FlatShape<128> : FFTShape<128, 32, 4, 4, 4, 2> {};
template <> struct FlatShape<256> : FFTShape<256, 64, 4, 4, 4, 4> {};
template <> struct FlatShape<384> : FFTShape<384, 32, 12, 4, 4, 2> {};
template <> struct FlatShape<512> : FFTShape<512, 64, 8, 8, 8> {};
template <int P, int KIND>
using LineShape = std::conditional_t<KIND == 0 || KIND == 3, FlatShape<P>, PencilShape<P>>;

// ------------------------------------------------------------------ k_fields
// Boundary fields of every node in sorted order (the zero-extended data of
// Fig. 4 before it is placed on the grid): Laplace q w and u n_i w;
// Navier t_j w and the symmetrised u (x) n w; half-space sigma_b w.
template <typename R, int KIND>
__device__ __forceinline__ void fields_body(const ApplyArgs &a, const int bx, const int by, const int bz) {
    const int s = bx * 256 + threadIdx.x;
    if (s >= a.m) return;
    R *vf = static_cast<R *>(a.vf);
    const int j = a.perm[s];
    const double wt = a.w[s];
    const double n[3] = {a.nrm[s], a.nrm[a.m + s], a.nrm[2 * a.m + s]};
    if constexpr (KIND == 3) {
#pragma unroll
        for (int c = 0; c < 3; ++c) vf[c * a.m + s] = (R)(a.q[c * a.m + j] * wt);
    } else if constexpr (KIND == 0 || KIND == 1) {
        const double uw = a.u[j] * wt;
        vf[s] = (R)(a.q[j] * wt);
#pragma unroll
        for (int i = 0; i < (KIND == 0 ? 2 : 3); ++i) vf[(1 + i) * a.m + s] = (R)(uw * n[i]);
    } else {
        double uu[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            vf[c * a.m + s] = (R)(a.q[c * a.m + j] * wt);
            uu[c] = a.u[c * a.m + j];
        }
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            const int i = pair_i(p), k = pair_j(p);
            const double v = (i == k ? uu[i] * n[i] : uu[i] * n[k] + uu[k] * n[i]) * wt;
            vf[(3 + p) * a.m + s] = (R)v;
        }
    }
}

template <typename R, int KIND>
__global__ __launch_bounds__(256) void k_fields(ApplyArgs a) {
    fields_body<R, KIND>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Batched form: blockIdx.z = member * zdiv + the kernel's own z index.
template <typename R, int KIND>
__global__ __launch_bounds__(256) void kb_fields(const ApplyArgs *members, const BatchIO *io, int zdiv) {
    ApplyArgs a = members[blockIdx.z / zdiv];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    a.r = io->r + a.off;
    fields_body<R, KIND>(a, blockIdx.x, blockIdx.y, blockIdx.z % zdiv);
}

// All F field values of sorted node s at once (one set of loads), computed
// from q and u exactly as fields_body stores them (same operations, same
// rounding), for the long-row transforms, which do not wait for k_fields.
template <typename R, int KIND>
__device__ __forceinline__ void node_fields(const ApplyArgs &a, const int s, R *v) {
    constexpr int F = Terms<KIND>::F;
    const int j = a.perm[s];
    const double wt = a.w[s];
    if constexpr (KIND == 3) {  // half-space: the three traction components
#pragma unroll
        for (int c = 0; c < 3; ++c) v[c] = (R)(a.q[c * a.m + j] * wt);
    } else if constexpr (KIND == 0 || KIND == 1) {
        v[0] = (R)(a.q[j] * wt);
        const double uw = a.u[j] * wt;
#pragma unroll
        for (int f = 1; f < F; ++f) v[f] = (R)(uw * a.nrm[(f - 1) * a.m + s]);
    } else {
        static_assert(F == 9, "Navier: three tractions and six symmetrised u n products");
        double uu[3], nn[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] = (R)(a.q[c * a.m + j] * wt);
            uu[c] = a.u[c * a.m + j];
            nn[c] = a.nrm[c * a.m + s];
        }
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            const int i = pair_i(p), k = pair_j(p);
            v[3 + p] = (R)((i == k ? uu[i] * nn[i] : uu[i] * nn[k] + uu[k] * nn[i]) * wt);
        }
    }
}

// ------------------------------------------------------------------ long rows
// Long grid rows (e.g. rows of a box face lying in a grid plane) are
// x-transformed with an FFT instead of the direct sum: the row's nodes are
// placed on a zero pencil (nodes sharing a cell are summed in order) and
// transformed; kx < Hx is kept.                          -> Xd[d][f][kx]
template <typename R, int PX, int KIND>
struct RowCfg {
    using SH = LineShape<PX, KIND>;
    static constexpr int TPP = SH::TPP;
    static constexpr int PPB = 256 / TPP;  // pencils per block
};

template <typename R, int PX, int KIND>
__device__ __forceinline__ void rows_fft_body(const ApplyArgs &a, const int bx, const int by, const int bz) {
    // one block per long row: every thread places whole cells (all fields of
    // a node at once, one round of gathers), then each wavefront transforms
    // its pencils; fields beyond one block's pencils take further passes
    using Cfg = RowCfg<R, PX, KIND>;
    constexpr int TPP = Cfg::TPP, NPEN = Cfg::PPB, E = PX / TPP, PS = pstride<PX>();
    constexpr int F = Terms<KIND>::F;
    const int d = bx;
    if (d >= a.nd) return;  // block-uniform: batched members with fewer long rows
    __shared__ cx<R> buf[NPEN * PS];
    __shared__ cx<R> tw[PX];
    const int tid = threadIdx.x;
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    for (int i = tid; i < PX; i += 256) tw[i] = gtwx[i];
    const int row = a.dense_rows[d];
    const int s0 = a.rowptr[row], s1 = a.rowptr[row + 1];
    const int pen = tid / TPP, t = tid % TPP;
    cx<R> *pb = buf + pen * PS;
    cx<R> *Xd = static_cast<cx<R> *>(a.Xd);
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += NPEN) {
#pragma unroll
        for (int e = 0; e < E; ++e) pb[pslot(t + e * TPP)] = {R(0), R(0)};
        __syncthreads();
        for (int s = s0 + tid; s < s1; s += 256) {
            const int x = a.gx[s];
            if (s > s0 && a.gx[s - 1] == x) continue;  // summed by the first node of the cell
            R v[F];
            node_fields<R, KIND>(a, s, v);  // all fields of the node from one set of loads
            for (int s2 = s + 1; s2 < s1 && a.gx[s2] == x; ++s2) {
                R v2[F];
                node_fields<R, KIND>(a, s2, v2);
#pragma unroll
                for (int f = 0; f < F; ++f) v[f] += v2[f];
            }
#pragma unroll
            for (int fl = 0; fl < NPEN; ++fl)
                if (f0 + fl < F) buf[fl * PS + pslot(x)] = {v[f0 + fl], R(0)};
        }
        __syncthreads();
        const int f = f0 + pen;
        cx<R> xr[E];
#pragma unroll
        for (int e = 0; e < E; ++e) xr[e] = pb[pslot(t + e * TPP)];
        fft_regs_s<R, typename Cfg::SH, -1>(xr, pb, tw, t);
        if (f < F) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int kx = t + e * TPP;
                if (kx < a.hx) Xd[((size_t)d * F + f) * a.hx + kx] = xr[e];
            }
        }
        __syncthreads();  // the next pass rewrites the pencils
    }
}

// Field scatter and long-row transforms in one launch (they do not depend on each
// other): the first nfb blocks scatter the fields, the rest transform rows.
template <typename R, int PX, int KIND>
__global__ __launch_bounds__(256) void k_fields_rows(ApplyArgs a, int nfb) {
    if ((int)blockIdx.x < nfb) fields_body<R, KIND>(a, blockIdx.x, 0, 0);
    else rows_fft_body<R, PX, KIND>(a, blockIdx.x - nfb, 0, 0);
}

// Batched form: blockIdx.z = member * zdiv + the kernel's own z index.
template <typename R, int PX, int KIND>
__global__ __launch_bounds__(256) void kb_rows_fft(const ApplyArgs *members, const BatchIO *io, int zdiv) {
    ApplyArgs a = members[blockIdx.z / zdiv];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    a.r = io->r + a.off;
    rows_fft_body<R, PX, KIND>(a, blockIdx.x, blockIdx.y, blockIdx.z % zdiv);
}

// Blocks go to the 8 XCDs round-robin, so block b runs on XCD b % 8; item(b)
// gives each XCD one contiguous run of the total work items (-1: none), so
// that neighbouring items share its L2.  Grid: 8 * ceil(total / 8) blocks.
__device__ __forceinline__ int xcd_item(int b, int total) {
    const int per = (total + 7) / 8;
    const int lam = (b % 8) * per + b / 8;
    return b / 8 < per && lam < total ? lam : -1;
}

// ------------------------------------------------------------------ k_fwd_xy
template <typename R, int PY, int KIND>
struct FwdCfg {
    static constexpr int F = Terms<KIND>::F;
    static constexpr int TPP = PencilShape<PY>::TPP;
    static constexpr int CB = (int)sizeof(cx<R>);
    static constexpr int PS = pstride<PY>();
    static constexpr int FIXED = PY * CB;
    // kx per block: 4 in FP32; 2 in FP64, where more, smaller blocks hide the
    // node loads of the direct DFT better (the 128^3 cube: 82 -> 72 us)
    static constexpr int KXC = clampi(mini(256 / (F * TPP), (64 * 1024 - FIXED) / (F * PS * CB)), 1, CB == 16 ? 2 : 4);
    static constexpr int NT = F * KXC * TPP;
};

// XG: kx per thread in the direct DFT (1, or 2 on plans whose short rows
// hold few nodes, where one node load then serves two kx).
template <typename R, int PY, int KIND, int XG_, typename YS = cx<R>>
__device__ __forceinline__ void fwd_xy_body(const ApplyArgs &a, const int bx, const int zz) {
    using Cfg = FwdCfg<R, PY, KIND>;
    constexpr int F = Cfg::F, KXC = Cfg::KXC, NT = Cfg::NT, TPP = Cfg::TPP, PS = Cfg::PS, E = PY / TPP;
    __shared__ cx<R> buf[F * KXC * PS];
    __shared__ cx<R> tw[PY];
    const int tid = threadIdx.x;
    const int kx0 = bx * KXC;
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    const cx<R> *gtwy = static_cast<const cx<R> *>(a.twy);
    const R *vf = static_cast<const R *>(a.vf);
    const cx<R> *Xd = static_cast<const cx<R> *>(a.Xd);
    for (int i = tid; i < PY; i += NT) tw[i] = gtwy[i];
    __syncthreads();
    const float inv_px = 1.0f / (float)a.px;
    // x-transform of the zero-extended fields for rows y < ny: a direct DFT
    // over the row's few nodes, or the row FFT of a long row.  A thread takes
    // one row and XG consecutive kx: each node's data is loaded once for the
    // XG kx and its twiddles are stepped from (kx x) mod px.
    constexpr int XG = clampi(XG_, 1, KXC);
    constexpr int NG = (KXC + XG - 1) / XG;
    for (int it = tid; it < NG * a.ny; it += NT) {
        const int gk = it % NG, y = it / NG;
        const int kxa = kx0 + gk * XG;
        const int row = zz * a.ny + y;
        const int dense = a.row_dense[row];
        const int r0 = a.rowptr[row], r1 = a.rowptr[row + 1];
        cx<R> acc[XG][F];
        if (dense >= 0) {
#pragma unroll
            for (int k = 0; k < XG; ++k)
#pragma unroll
                for (int f = 0; f < F; ++f)
                    acc[k][f] = (kxa + k < a.hx) ? Xd[((size_t)dense * F + f) * a.hx + kxa + k] : cx<R>{R(0), R(0)};
        } else {
#pragma unroll
            for (int k = 0; k < XG; ++k)
#pragma unroll
                for (int f = 0; f < F; ++f) acc[k][f] = {R(0), R(0)};
            // the x twiddles come from the block's LDS table when Px = Py
            // (the same table), else through the caches
            auto row_sum = [&](const cx<R> *twt) {
#pragma unroll 4
                for (int s = r0; s < r1; ++s) {
                    const int xg = a.gx[s];
                    R vv[F];
#pragma unroll
                    for (int f = 0; f < F; ++f) vv[f] = vf[f * a.m + s];
                    int idx = mod_small(kxa, xg, a.px, inv_px);
#pragma unroll
                    for (int k = 0; k < XG; ++k) {
                        const cx<R> w = twt[idx];
#pragma unroll
                        for (int f = 0; f < F; ++f) {
                            acc[k][f].x += vv[f] * w.x;
                            acc[k][f].y += vv[f] * w.y;
                        }
                        idx += xg;
                        if (idx >= a.px) idx -= a.px;
                    }
                }
            };
            if (a.px == PY) row_sum(tw);
            else row_sum(gtwx);
        }
#pragma unroll
        for (int k = 0; k < XG; ++k)
            if (gk * XG + k < KXC)
#pragma unroll
                for (int f = 0; f < F; ++f) buf[(f * KXC + gk * XG + k) * PS + pslot(y)] = acc[k][f];
    }
    __syncthreads();
    // y-FFT in registers (rows y >= ny are zero), stored straight from them
    const int pen = tid / TPP, t = tid % TPP;
    const int f = pen / KXC, kx = kx0 + pen % KXC;
    cx<R> *pb = buf + pen * PS;
    cx<R> x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        // rows y >= P/2 lie beyond the grid (ny <= P/2): zero at compile time
        const int y = t + e * TPP;
        x[e] = (e < E / 2 && y < a.ny) ? pb[pslot(y)] : cx<R>{R(0), R(0)};
    }
    fft_regs<R, PY, -1>(x, pb, tw, t);
    if (kx < a.hx) {
        YS *Y = static_cast<YS *>(a.Y) + (size_t)(f * a.hx + kx) * a.nzo * PY;
        if constexpr (std::is_same<YS, cbf16>::value) {
            Y += (size_t)zz * PY;
#pragma unroll
            for (int e = 0; e < E; ++e) Y[t + e * TPP] = to_store<YS>(x[e]);
        } else {
            const int l = z_tile_log2(KIND, sizeof(R) == 8, a.pz, a.zsched);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int ky = t + e * TPP;
                Y[((((ky >> l) * a.nzo) + zz) << l) + (ky & ((1 << l) - 1))] = x[e];
            }
        }
    }
}

// Items (kx group, plane), planes fastest: the blocks in flight on one XCD
// write neighbouring planes of the same tiles of Y, so its L2 joins their
// parts of a cache line.  The 16-bit form writes whole lines and takes its
// blocks as they come (grid: planes, kx groups; with kx groups fastest the
// 190^3 cube's pass took 122 us instead of 114, Navier's 283 instead of 254).
template <typename R, int PY, int KIND, int XG, typename YS>
__device__ __forceinline__ void fwd_xy_item(const ApplyArgs &a, const int b) {
    constexpr int KXC = FwdCfg<R, PY, KIND>::KXC;
    if constexpr (std::is_same<YS, cbf16>::value) {
        fwd_xy_body<R, PY, KIND, XG, YS>(a, blockIdx.y, blockIdx.x);
    } else {
        const int lam = xcd_item(b, (a.hx + KXC - 1) / KXC * a.nzo);
        if (lam >= 0) fwd_xy_body<R, PY, KIND, XG, YS>(a, lam / a.nzo, lam % a.nzo);
    }
}

template <typename R, int PY, int KIND, int XG, typename YS = cx<R>>
__global__ __launch_bounds__((FwdCfg<R, PY, KIND>::NT)) void k_fwd_xy(ApplyArgs a) {
    fwd_xy_item<R, PY, KIND, XG, YS>(a, blockIdx.x);
}

// Batched form: blockIdx.z = member.
template <typename R, int PY, int KIND>
__global__ __launch_bounds__((FwdCfg<R, PY, KIND>::NT)) void kb_fwd_xy(const ApplyArgs *members, const BatchIO *io) {
    const ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    fwd_xy_item<R, PY, KIND, 1, cx<R>>(a, blockIdx.x);
}

// ------------------------------------------------------------------ k_zpass
// A wavefront owns PPW = 64/TPP pencils (consecutive ky at one kx) from load
// to store; with D = 2 (Navier) two wavefronts share them, one with the even
// frequencies and one with the odd ones, and add their halves at the end,
// each storing half of the planes.  Lane t of a pencil loads the rows its
// first FFT stage needs straight into registers (the next field's while the
// current one is transformed), multiplies the transformed values in registers
// and stores the inverse transform's rows from registers.  LDS carries the
// exchanges between FFT stages and, in FP32, the spectrum rows: read straight
// from memory they would be 4-byte loads over many rows per instruction, each
// value four times (the two reflections); so a field's rows come in as one
// run of 16-byte direct-to-LDS loads, in flight during the transform.
template <typename R, typename SH, int KIND>
struct ZCfg {
    static constexpr int D = SH::D, L = SH::L, PZ = D * L;
    static_assert(D == z_split(KIND, sizeof(R) == 8, PZ), "the stored spectra's split");
    static constexpr int TPP = SH::TPP;
    static constexpr int PPW = 64 / TPP;
    static constexpr int KT = 1 << z_tile_log2(KIND, sizeof(R) == 8, PZ, SH::SCHED);
    static constexpr int CB = (int)sizeof(cx<R>);
    static constexpr int PS = SH::PS;
    static constexpr int WAVES = TPP == 4 ? 2 : 4;  // a block's ky divide every Py (a multiple of 32)
    static constexpr int SETS = WAVES / D;  // groups of PPW pencils per block
    static constexpr int TY = PPW * SETS;
    static constexpr int NT = 64 * WAVES;
    static constexpr int E = SH::E;
    static constexpr int EI = D == 1 ? E / 2 : E;  // elements that hold planes (n < P/2)
    static constexpr bool STAGE = sizeof(R) == 4;  // spectrum rows through LDS
    // The next field's planes are loaded during the current field's transform
    // while they, the field and the sums take at most 160 registers: beyond,
    // the overlap costs more occupancy than it hides (FP64 Laplace: 256 points
    // 84 -> 79 us with it, 384 points 389 -> 532; FP64 Navier: 256 points 342
    // -> 326, 192 points 150 -> 335; FP32 Navier, 384 points: 619 -> 567).
    static constexpr bool PREFETCH = ((Terms<KIND>::O + 1) * E + EI) * (CB / 4) <= 160;
    static constexpr int NC = max_field_ncomp<KIND>();
    static constexpr int CHUNK = (PPW * spec_len(D, 0, PZ / 2 + 1) * (int)sizeof(R) + 1023) / 1024 * 1024;
    static_assert(PPW <= KT, "a wavefront's ky share a tile");
    static_assert(E % 2 == 0, "lower and reflected frequencies are told apart by e");
};

// Buffer descriptor of a uniform byte range: loads past its end return zero,
// stores past its end are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_range(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
typedef unsigned uvec2 __attribute__((ext_vector_type(2)));
typedef unsigned uvec4 __attribute__((ext_vector_type(4)));
template <typename R>
__device__ __forceinline__ cx<R> buf_load(__amdgpu_buffer_rsrc_t r, int off) {
    if constexpr (sizeof(R) == 4) return __builtin_bit_cast(cx<R>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    else return __builtin_bit_cast(cx<R>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
template <typename R>
__device__ __forceinline__ R buf_load_real(__amdgpu_buffer_rsrc_t r, int off) {
    if constexpr (sizeof(R) == 4) return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    else return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <typename R>
__device__ __forceinline__ void buf_store(cx<R> v, __amdgpu_buffer_rsrc_t r, int off) {
    if constexpr (sizeof(R) == 4) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uvec2, v), r, off, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uvec4, v), r, off, 0, 0);
}

template <typename R>
__device__ __forceinline__ void mac(cx<R> &acc, cx<R> v, R s, bool imag) {
    if (imag) {  // (i s) v
        acc.x -= s * v.y;
        acc.y += s * v.x;
    } else {
        acc.x += s * v.x;
        acc.y += s * v.y;
    }
}

template <typename R, typename SH, int KIND>
__device__ __forceinline__ void zpass_body(const ApplyArgs &a, const int kx, const int by) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass cannot type-check the buffer builtins
    using Cfg = ZCfg<R, SH, KIND>;
    using T = Terms<KIND>;
    constexpr int D = Cfg::D, L = Cfg::L, PZ = Cfg::PZ, PPW = Cfg::PPW, TY = Cfg::TY, NT = Cfg::NT, TPP = Cfg::TPP;
    constexpr int E = Cfg::E, EI = Cfg::EI, PS = Cfg::PS, KT = Cfg::KT, CB = Cfg::CB, RB = (int)sizeof(R);
    constexpr int F = T::F, O = T::O, NC = Cfg::NC, CHUNK = Cfg::CHUNK;
    constexpr bool STAGE = Cfg::STAGE;
    constexpr bool kPrefetch = Cfg::PREFETCH;
    __shared__ cx<R> buf[Cfg::WAVES * PPW * PS];
    __shared__ cx<R> tab[zt_size<SH>()];
    __shared__ __attribute__((aligned(16))) char sspec[STAGE ? Cfg::WAVES * NC * CHUNK : 16];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
    const int r = D == 2 ? wave & 1 : 0;  // frequencies D k + r
    const int b = lane / TPP, t = lane % TPP;
    const int ky0 = by * TY + wave / D * PPW;  // the wavefront's first ky
    const int ky = ky0 + b;
    cx<R> *pb = buf + (wave * PPW + b) * PS;
    zt_fill<R, SH>(tab, static_cast<const cx<R> *>(a.twz), tid, NT);
    __syncthreads();
    cx<R> acc[O][E];
#pragma unroll
    for (int o = 0; o < O; ++o)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[o][e] = {R(0), R(0)};

    // Lane t holds plane n = t + e TPP of the occupied planes, n < P/2 (a shift
    // of all planes does not change a convolution, so the first occupied one
    // is n = 0); planes past the last one lie past the tile's end and read as
    // zero.
    const size_t fstride = (size_t)a.hx * a.nzo * a.py;
    const cx<R> *Yt = static_cast<const cx<R> *>(a.Y) + ((size_t)kx * a.py + ky0 / KT * KT) * a.nzo;
    const int yoff = (t * KT + ky0 % KT + b) * CB;
    const int ybytes = a.nzo * KT * CB;
    auto load_field = [&](int f, cx<R> *x) {
        const auto rs = buf_range(Yt + f * fstride, ybytes);
#pragma unroll
        for (int e = 0; e < EI; ++e) x[e] = buf_load<R>(rs, yoff + e * (TPP * KT * CB));
    };
    // Spectrum rows of the wavefront: those of ky, or reflected to Py - ky from
    // Py/2 on (Py/2 itself has both names, and its spectra odd in y are zero,
    // so its sign is immaterial) -- one run of rows either way, in reverse
    // order when reflected.  Frequency D k + r of element k = t + e TPP sits
    // at k for e < E/2 and, reflected to P - kz, at L - r - k above (P/2
    // itself, k = L/2 of part 0, is read there too: its spectra odd in z are
    // zero).
    constexpr int HZ = PZ / 2 + 1, L0 = spec_len(D, 0, HZ), L1 = spec_len(D, 1, HZ);
    const bool fy = 2 * ky0 >= a.py;
    const int row0 = fy ? a.py - ky0 - (PPW - 1) : ky0, brow = fy ? PPW - 1 - b : b;
    const int len = r ? L1 : L0;
    const int lo = brow * len + t, hi = brow * len + (L - r - t) - (E - 1) * TPP;
    auto spec_rows = [&](int c) {
        const R *p = static_cast<const R *>(a.spec) + (size_t)(c * a.hx + kx) * a.hy * spec_row(D, HZ) +
                     (r ? (size_t)a.hy * L0 : 0) + (size_t)row0 * len;
        return buf_range(p, PPW * len * RB);
    };
    char *sw = sspec + (STAGE ? wave * NC * CHUNK : 0);
    auto stage_spec = [&](auto fc) {  // the spectrum rows of field f into LDS
        constexpr int f = decltype(fc)::value;
        static_for<0, field_ncomp<KIND>(f)>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const auto rs = spec_rows(field_comp<KIND>(f, i));
#pragma unroll
            for (int k = 0; k < CHUNK / 1024; ++k)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rs, (__attribute__((address_space(3))) void *)(sw + i * CHUNK + k * 1024), 16, lane * 16 + k * 1024,
                    0, 0, 0);
        });
    };

    [[maybe_unused]] cx<R> xn[kPrefetch ? EI : 1];
    if constexpr (kPrefetch) load_field(0, xn);
    static_for<0, F>([&](auto fc) {
        constexpr int f = decltype(fc)::value;
        // one field per scheduling region: without the barrier the scheduler
        // starts every field's loads at once and runs out of registers
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (STAGE) {
            stage_spec(fc);  // the previous field's rows have been used
            __builtin_amdgcn_sched_barrier(0);  // and before the loads below, for the count of the wait
        }
        cx<R> x[E];
        if constexpr (kPrefetch) {
#pragma unroll
            for (int e = 0; e < EI; ++e) x[e] = xn[e];
            if constexpr (f + 1 < F) load_field(f + 1, xn);  // in flight during this field's transform
        } else {
            load_field(f, x);
        }
#pragma unroll
        for (int e = EI; e < E; ++e) x[e] = {R(0), R(0)};
        if (D == 2 && r) {
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = cmul(x[e], tab[t + e * TPP]);
        }
        z_fft<R, SH, -1>(x, pb, tab, t);
        if constexpr (STAGE) {
            // the staged rows have arrived: only the loads issued after them
            // (the next field's) may be outstanding
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPrefetch && f + 1 < F ? EI : 0) : "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<0, T::N>([&](auto tc) {
            constexpr int term = decltype(tc)::value;
            if constexpr (T::f(term) == f) {
                constexpr int c = T::c(term), slot = term_slot<KIND>(term);
                constexpr int mask = comp_oddmask(KIND, c);
                const R *sp = reinterpret_cast<const R *>(sw + slot * CHUNK);
                const auto rs = spec_rows(c);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int k = e < E / 2 ? lo + e * TPP : hi + (E - 1 - e) * TPP;
                    const R sv = STAGE ? sp[k] : buf_load_real<R>(rs, k * RB);
                    const bool flip = (fy && (mask & 2)) != ((e >= E / 2) && (mask & 4));
                    mac<R>(acc[T::o(term)][e], x[e], flip ? -sv : sv, comp_imag(KIND, c));
                }
            }
        });
        // the sums are formed here, not sunk past the next field's branch
        // (which would keep every field's values live)
#pragma unroll
        for (int o = 0; o < O; ++o)
#pragma unroll
            for (int e = 0; e < E; ++e) asm volatile("" : "+v"(acc[o][e].x), "+v"(acc[o][e].y));
    });

    __builtin_amdgcn_sched_barrier(0);
    const size_t slab = (size_t)a.nzo * a.py;
    const int zbytes = (int)(slab * CB);
    const int zoff = (t * a.py + ky) * CB, zstep = TPP * a.py * CB;
    auto slot = [](int i) { return i + (i >> SH::SHIFT); };
#pragma unroll
    for (int o = 0; o < O; ++o) {
        if (D == 2 && o > 0) __syncthreads();  // the other wavefront has read this one's half
        z_fft<R, SH, 1>(acc[o], pb, tab, t);
        const auto rs = buf_range(static_cast<const cx<R> *>(a.Z) + (size_t)(o * a.hx + kx) * slab, zbytes);
        if constexpr (D == 1) {
#pragma unroll
            for (int e = 0; e < E / 2; ++e) buf_store<R>(acc[o][e], rs, zoff + e * zstep);
        } else {
            // the even wavefront stores e < E/2, the odd one the rest
            const cx<R> *pother = buf + ((wave ^ 1) * PPW + b) * PS;
            if (r) {
#pragma unroll
                for (int e = 0; e < E; ++e) acc[o][e] = cmulc(acc[o][e], tab[t + e * TPP]);
            }
            wave_lds_sync();
            if (r) {
#pragma unroll
                for (int e = 0; e < E / 2; ++e) pb[slot(t + e * TPP)] = acc[o][e];
            } else {
#pragma unroll
                for (int e = E / 2; e < E; ++e) pb[slot(t + e * TPP)] = acc[o][e];
            }
            __syncthreads();
            if (r) {
#pragma unroll
                for (int e = E / 2; e < E; ++e)
                    buf_store<R>(cadd(pother[slot(t + e * TPP)], acc[o][e]), rs, zoff + e * zstep);
            } else {
#pragma unroll
                for (int e = 0; e < E / 2; ++e)
                    buf_store<R>(cadd(acc[o][e], pother[slot(t + e * TPP)]), rs, zoff + e * zstep);
            }
        }
    }
#endif
}

// (kx, ky-block) items, ordered so that the blocks of one kx and their
// mirrored ky blocks (which read the same octant rows of the spectra) follow
// each other on the same L2.
template <typename R, typename SH, int KIND>
__device__ __forceinline__ void zpass_item(const ApplyArgs &a, const int b, const int nby) {
    const int lam = xcd_item(b, a.hx * nby);
    if (lam < 0) return;
    const int kx = lam / nby, j = lam % nby;
    const int by = (j & 1) ? nby - 1 - (j >> 1) : (j >> 1);
    zpass_body<R, SH, KIND>(a, kx, by);
}

// At least two wavefronts per SIMD: FP64 Navier would take a few registers
// more than the 256 that allow them.
template <typename R, typename SH, int KIND>
__global__ __launch_bounds__((ZCfg<R, SH, KIND>::NT), 2) void k_zpass(ApplyArgs a, int nby) {
    zpass_item<R, SH, KIND>(a, blockIdx.x, nby);
}

// Batched form: blockIdx.z = member.  The member's arguments are copied first: read
// through the pointer they are fetched again after every scheduling barrier (two
// Navier bodies of 64^3 in FP64 at 64 points: 119 -> 50 us).
template <typename R, typename SH, int KIND>
__global__ __launch_bounds__((ZCfg<R, SH, KIND>::NT), 2) void kb_zpass(const ApplyArgs *members, const BatchIO *io,
                                                                     int nby) {
    const ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    zpass_item<R, SH, KIND>(a, blockIdx.x, nby);
}

// ------------------------------------------------------------------ k_mid2d
// 2D plans: everything between the fields and W for one kx, in one block.  The
// F fields' columns at a kx fit in LDS together, so the y FFT, the spectral
// product and the inverse y FFT follow each other there (x[e] of lane t is
// ky = t + e TPP throughout) and only W is written: the forward pass, the
// product and the inverse y pass as kernels of their own took 18.8 + 8.6 +
// 12.1 us for the 500-point square in FP64 and 7.8 + 3.6 + 7.7 us for a 256^2
// half-space surface in FP32, against 21.7 and 8.7 us.  All of them are bound by
// latency (a few loads that wait for each other, barriers), so the block has
// more threads than the pencils need -- every row of the direct DFT gets its own
// as far as possible --, the rows' extents and the spectra are loaded before
// anything waits, and a row's nodes are fetched four at a time.
//
// FOLD: the node data come from q and u directly and rows of more than kWaveRow
// nodes are summed by their wavefront (one round of loads instead of a chain of
// them; long rows always, others unless a wavefront has many), which saves the launch before (fields and long-row
// transforms, 7.9 us on the square).  Each block then reads every node's data,
// so this is for few nodes and few long rows.
//
// LEAN, for batches: the fields come from k_fields' buffer and fewer nodes are
// fetched at a time (the sums keep their order, so a member has its plan's bits).  Many
// members fill the chip, and then wavefronts count, not latency: 63 registers
// against 224 for the folded form at 256 points in FP32.  32 circles on 128^2, us:
// folded from q and u 72 (FP32) and 87 (FP64), lean 37 and 56; 32 discs of 0.15 on
// 256^2 FP64, not folded, 183 and 141.
template <typename R, int PY, int KIND>
struct Mid2dCfg {
    static constexpr int F = Terms<KIND>::F, O = Terms<KIND>::O;
    using SH = FlatShape<PY>;
    static constexpr int TPP = SH::TPP, E = SH::E, PS = pstride<PY>();
    // threads: one per grid row up to 256, at least one per pencil lane
    static constexpr int NT = clampi((PY / 2 + 63) / 64 * 64, (F * TPP + 63) / 64 * 64, 256);
    // 1024 points in FP64: without a twiddle table in LDS three blocks fit on a
    // CU, and all 513 of them on the chip at once (with it, two: 512)
    static constexpr bool TWL = PY * sizeof(cx<R>) < 16384;
    static constexpr int WPE = KIND == 0 && PY == 1024 ? 3 : 1;  // wavefronts per SIMD that the registers must allow
    static_assert(F * TPP <= NT && O <= F, "a thread for every pencil lane");
};

// Component of the term (output o, field f): O = 1 has one per field.
template <int KIND>
__device__ __forceinline__ int term_comp2d(int o, int f) {
    if constexpr (Terms<KIND>::O == 1) return f;
    else {
        static_assert(KIND != 3 || (Terms<3>::c(0) == 0 && Terms<3>::c(1) == 2 && Terms<3>::c(2) == 4 && Terms<3>::c(3) == 2 &&
                                    Terms<3>::c(4) == 1 && Terms<3>::c(5) == 5 && Terms<3>::c(6) == 6 && Terms<3>::c(7) == 7 &&
                                    Terms<3>::c(8) == 3));
        return (int)((0x376512420ull >> (4 * (3 * o + f))) & 15);  // the table, four bits each
    }
}

template <typename R, int PY, int KIND, bool FOLD, bool LEAN = false>
__device__ __forceinline__ void mid2d_body(const ApplyArgs &a, const int kx, const int all_rows) {
    using Cfg = Mid2dCfg<R, PY, KIND>;
    constexpr int F = Cfg::F, O = Cfg::O, TPP = Cfg::TPP, E = Cfg::E, PS = Cfg::PS, NT = Cfg::NT;
    using SH = typename Cfg::SH;
    constexpr int NS = O == 1 ? 1 : F;              // spectra per thread
    constexpr int NR = (PY / 2 + NT - 1) / NT;      // grid rows per thread
    constexpr int CH = LEAN || NR > 1 ? 2 : 8;      // nodes of a row fetched together
    constexpr int WS = LEAN || NR > 1 ? 1 : 2, WC = 2;  // and rows of the wavefront's, nodes per lane
    __shared__ cx<R> buf[F * PS];
    __shared__ cx<R> twl[Cfg::TWL ? PY : 1];
    __shared__ unsigned char keep[PY / 2];
    const int tid = threadIdx.x, pen = tid / TPP, t = tid % TPP;
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    const cx<R> *gtwy = static_cast<const cx<R> *>(a.twy);
    const R *vf = static_cast<const R *>(a.vf);
    const cx<R> *Xd = static_cast<const cx<R> *>(a.Xd);
    const R *spec = static_cast<const R *>(a.spec);
    if constexpr (Cfg::TWL)
        for (int i = tid; i < PY; i += NT) twl[i] = gtwy[i];
    // the rows' extents and this lane's spectra
    int dn[NR], r0[NR], r1[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int y = tid + k * NT;
        const bool in = y < a.ny;
        dn[k] = in ? a.row_dense[y] : -1;
        r0[k] = in ? a.rowptr[y] : 0;
        r1[k] = in ? a.rowptr[y + 1] : 0;
    }
    R sp[NS][E];
    bool im[NS];
    if (pen < F) {
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            const int c = O == 1 ? pen : term_comp2d<KIND>(pen, n);  // O > 1: O = F, pencil = output
            const int odd = comp_oddmask(KIND, c);
            im[n] = comp_imag(KIND, c);
            const R *sc = spec + ((size_t)c * a.hx + kx) * a.hy;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int ky = t + e * TPP;
                const R v = sc[ky < a.hy ? ky : PY - ky];
                sp[n][e] = ky >= a.hy && (odd & 2) ? -v : v;
            }
        }
    }
    if constexpr (Cfg::TWL) __syncthreads();
    // x transform at kx of every row's nodes
    const float inv_px = 1.0f / (float)a.px;
    // C nodes s, s + stride, ... below s1, with their twiddles, fetched together
    auto fetch = [&](auto cc, const cx<R> *twt, int s, int stride, int s1, cx<R> *w, R (*v)[F]) {
        constexpr int C = decltype(cc)::value;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const bool in = s + k * stride < s1;
            const int sk = in ? s + k * stride : 0;
            w[k] = twt[mod_small(kx, a.gx[sk], a.px, inv_px)];
            if constexpr (FOLD && !LEAN) {
                node_fields<R, KIND>(a, sk, v[k]);
            } else {
#pragma unroll
                for (int f = 0; f < F; ++f) v[k][f] = vf[f * a.m + sk];
            }
#pragma unroll
            for (int f = 0; f < F; ++f) v[k][f] = in ? v[k][f] : R(0);
        }
    };
    auto add = [&](auto cc, const cx<R> *w, const R (*v)[F], cx<R> *acc) {
        constexpr int C = decltype(cc)::value;
#pragma unroll
        for (int k = 0; k < C; ++k)
#pragma unroll
            for (int f = 0; f < F; ++f) {
                acc[f].x += v[k][f] * w[k].x;
                acc[f].y += v[k][f] * w[k].y;
            }
    };
    constexpr std::integral_constant<int, CH> ch;
    constexpr std::integral_constant<int, WC> wc;
    auto x_rows = [&](const cx<R> *twt) {
        // the first CH nodes, or the long row's transform, of all of the thread's
        // rows together, and the first nodes of the rows that the wavefront sums
        cx<R> w[NR][CH];
        R v[NR][CH][F];
        cx<R> acc[NR][F];
        bool wide[NR];
        const int lane = tid & 63;
        int wsrc[WS], wk[WS], ws0[WS], ws1[WS];
        cx<R> wx[WS][WC];
        R wv[WS][WC][F];
        unsigned long long todo[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const bool dense = !FOLD && dn[k] >= 0;
            if (!FOLD && __any(dense)) {
#pragma unroll
                for (int f = 0; f < F; ++f) acc[k][f] = dense ? Xd[((size_t)dn[k] * F + f) * a.hx + kx] : cx<R>{R(0), R(0)};
                if (dense) r1[k] = r0[k];  // nothing left to sum
            } else {
#pragma unroll
                for (int f = 0; f < F; ++f) acc[k][f] = {R(0), R(0)};
            }
            if (FOLD || __any(r1[k] > r0[k])) fetch(ch, twt, r0[k], 1, r1[k], w[k], v[k]);
            if constexpr (FOLD) {
                wide[k] = r1[k] - r0[k] > kWaveRow;
                if (__popcll(__ballot(wide[k])) > 4) wide[k] = dn[k] >= 0;
                todo[k] = __ballot(wide[k]);
            }
        }
        auto next = [&](int &k, int &src, int &s0, int &s1) {  // next row of the wavefront's: false if none
            k = 0;
            if constexpr (NR > 1) k = todo[0] ? 0 : 1;
            if (!todo[k]) return false;
            src = __ffsll((long long)todo[k]) - 1;
            todo[k] &= todo[k] - 1;
            s0 = __shfl(r0[k], src, 64);
            s1 = __shfl(r1[k], src, 64);
            return true;
        };
        auto finish = [&](const cx<R> (&part)[F], int k, int src) {
            cx<R> sum[F];
#pragma unroll
            for (int f = 0; f < F; ++f) sum[f] = part[f];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1)
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    sum[f].x += __shfl_xor(sum[f].x, off, 64);
                    sum[f].y += __shfl_xor(sum[f].y, off, 64);
                }
            if (lane == src)
#pragma unroll
                for (int f = 0; f < F; ++f) buf[f * PS + pslot(tid + k * NT)] = sum[f];
        };
        auto rest = [&](int s, int s1, cx<R> (&part)[F]) {
            cx<R> lx[WC];
            R lv[WC][F];
            for (; s - lane < s1; s += WC * 64) {
                fetch(wc, twt, s, 64, s1, lx, lv);
                add(wc, lx, lv, part);
            }
        };
        if constexpr (FOLD) {
            bool on[WS];
#pragma unroll
            for (int i = 0; i < WS; ++i) {
                on[i] = next(wk[i], wsrc[i], ws0[i], ws1[i]);
                if (on[i]) fetch(wc, twt, ws0[i] + lane, 64, ws1[i], wx[i], wv[i]);
            }
#pragma unroll
            for (int i = 0; i < WS; ++i)
                if (on[i]) {
                    cx<R> part[F];
#pragma unroll
                    for (int f = 0; f < F; ++f) part[f] = {R(0), R(0)};
                    add(wc, wx[i], wv[i], part);
                    rest(ws0[i] + lane + WC * 64, ws1[i], part);
                    finish(part, wk[i], wsrc[i]);
                }
            int k, src, s0, s1;
            while (next(k, src, s0, s1)) {
                cx<R> part[F];
#pragma unroll
                for (int f = 0; f < F; ++f) part[f] = {R(0), R(0)};
                rest(s0 + lane, s1, part);
                finish(part, k, src);
            }
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int y = tid + k * NT, n = r1[k] - r0[k];
            if (y >= a.ny) continue;
            keep[y] = all_rows || n > 0 || dn[k] >= 0;
            if (FOLD && wide[k]) continue;
            if (n > 0) {
                add(ch, w[k], v[k], acc[k]);
                for (int s = r0[k] + CH; s < r1[k]; s += CH) {
                    fetch(ch, twt, s, 1, r1[k], w[k], v[k]);
                    add(ch, w[k], v[k], acc[k]);
                }
            }
#pragma unroll
            for (int f = 0; f < F; ++f) buf[f * PS + pslot(y)] = acc[k][f];
        }
    };
    if constexpr (Cfg::TWL) {
        if (a.px == PY) x_rows(twl);  // the same table
        else x_rows(gtwx);
    } else {
        x_rows(gtwx);
    }
    __syncthreads();
    cx<R> *pb = buf + pen * PS;
    const cx<R> *tw;
    if constexpr (Cfg::TWL) tw = twl;
    else tw = gtwy;
    cx<R> x[E];
    if (pen < F) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int y = t + e * TPP;  // rows y >= PY / 2 lie beyond the grid
            x[e] = (e < E / 2 && y < a.ny) ? pb[pslot(y)] : cx<R>{R(0), R(0)};
        }
        fft_regs_s<R, SH, -1>(x, pb, tw, t);
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (O == 1) x[e] = im[0] ? cx<R>{-sp[0][e] * x[e].y, sp[0][e] * x[e].x} : cx<R>{sp[0][e] * x[e].x, sp[0][e] * x[e].y};
            pb[pslot(t + e * TPP)] = x[e];
        }
    }
    __syncthreads();
    if (pen < O) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            cx<R> acc = {R(0), R(0)};
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const cx<R> v = buf[f * PS + pslot(t + e * TPP)];
                if constexpr (O == 1) acc = {acc.x + v.x, acc.y + v.y};
                else mac<R>(acc, v, sp[f % NS][e], im[f % NS]);
            }
            x[e] = acc;
        }
    }
    if constexpr (O > 1) __syncthreads();  // every pencil's readers
    if (pen < O) {
        fft_regs_s<R, SH, 1>(x, pb, tw, t);
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < E / 2; ++e) {
            const int y = t + e * TPP;
            if (y < a.ny) pb[pslot(y)] = x[e];
        }
    }
    __syncthreads();
    cx<R> *W = static_cast<cx<R> *>(a.Y);
#pragma unroll
    for (int o = 0; o < O; ++o)
        for (int y = tid; y < a.ny; y += NT)
            if (keep[y]) W[((size_t)o * a.ny + y) * a.hx + kx] = buf[o * PS + pslot(y)];
}

// kx in runs per XCD: its L2 joins the columns' 8- or 16-byte parts of W's lines.
template <typename R, int PY, int KIND, bool FOLD>
__global__ __launch_bounds__((Mid2dCfg<R, PY, KIND>::NT), (Mid2dCfg<R, PY, KIND>::WPE)) void k_mid2d(ApplyArgs a, int all_rows) {
    const int kx = xcd_item(blockIdx.x, a.hx);
    if (kx >= 0) mid2d_body<R, PY, KIND, FOLD>(a, kx, all_rows);
}

template <typename R, int PY, int KIND, bool FOLD, bool LEAN>
__global__ __launch_bounds__((Mid2dCfg<R, PY, KIND>::NT), (Mid2dCfg<R, PY, KIND>::WPE)) void kb_mid2d(const ApplyArgs *members, const BatchIO *io) {
    ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    const int kx = xcd_item(blockIdx.x, a.hx);
    if (kx >= 0) mid2d_body<R, PY, KIND, FOLD, LEAN>(a, kx, 0);
}

// ------------------------------------------------------------------ k_inv_y
template <typename R, int PY, int KIND>
struct InvYCfg {
    static constexpr int O = Terms<KIND>::O;
    static constexpr int TPP = PencilShape<PY>::TPP;
    static constexpr int CB = (int)sizeof(cx<R>);
    static constexpr int PS = pstride<PY>();
    static constexpr int KXC = clampi(mini(256 / (O * TPP), (64 * 1024 - PY * CB) / (O * PS * CB)), 1, 16);
    static constexpr int NT = O * KXC * TPP;
};

// all_rows = 0 (the apply): only rows that hold nodes are stored, the
// gather reads nothing else; all_rows = 1 (the grid evaluation): every row.
template <typename R, int PY, int KIND, typename ZS = cx<R>>
__device__ __forceinline__ void inv_y_body(const ApplyArgs &a, const int bx, const int by, const int all_rows) {
    if (by >= a.nzo) return;  // batched: a member with fewer occupied planes
    using Cfg = InvYCfg<R, PY, KIND>;
    constexpr int O = Cfg::O, KXC = Cfg::KXC, NT = Cfg::NT, TPP = Cfg::TPP, PS = Cfg::PS, E = PY / TPP;
    __shared__ cx<R> buf[O * KXC * PS];
    __shared__ cx<R> tw[PY];
    __shared__ unsigned char keep[PY / 2];
    const int tid = threadIdx.x;
    const int kx0 = bx * KXC;
    const int zz = by;
    const cx<R> *gtwy = static_cast<const cx<R> *>(a.twy);
    for (int i = tid; i < PY; i += NT) tw[i] = gtwy[i];
    for (int y = tid; y < a.ny; y += NT)
        keep[y] = all_rows || a.rowptr[zz * a.ny + y + 1] > a.rowptr[zz * a.ny + y];
    const int pen = tid / TPP, t = tid % TPP;
    const int o = pen / KXC, kx = kx0 + pen % KXC;
    cx<R> x[E];
    if (kx < a.hx) {
        const ZS *Zr = static_cast<const ZS *>(a.Z) + ((size_t)(o * a.hx + kx) * a.nzo + zz) * PY;
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = from_store<R>(Zr[t + e * TPP]);
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = {R(0), R(0)};
    }
    __syncthreads();  // twiddle table, row flags
    cx<R> *pb = buf + pen * PS;
    fft_regs<R, PY, 1>(x, pb, tw, t);
    wave_lds_sync();
#pragma unroll
    for (int e = 0; e < E / 2; ++e) {  // ny <= Py/2: rows y >= Py/2 hold no node
        const int y = t + e * TPP;
        if (y < a.ny) pb[pslot(y)] = x[e];
    }
    __syncthreads();  // the transposed store reads every pencil
    const int nk = min(KXC, a.hx - kx0);
    cx<R> *W = static_cast<cx<R> *>(a.Y);
    for (int i = tid; i < O * a.ny * KXC; i += NT) {
        const int kl = i % KXC, rest = i / KXC;
        const int y = rest % a.ny, oo = rest / a.ny;
        if (kl < nk && keep[y])
            W[((size_t)(oo * a.nzo + zz) * a.ny + y) * a.hx + kx0 + kl] = buf[(oo * KXC + kl) * PS + pslot(y)];
    }
}

template <typename R, int PY, int KIND, typename ZS = cx<R>>
__global__ __launch_bounds__((InvYCfg<R, PY, KIND>::NT)) void k_inv_y(ApplyArgs a, int all_rows) {
    inv_y_body<R, PY, KIND, ZS>(a, blockIdx.x, blockIdx.y, all_rows);
}

// Batched form: blockIdx.z = member * zdiv + the kernel's own z index.
template <typename R, int PY, int KIND>
__global__ __launch_bounds__((InvYCfg<R, PY, KIND>::NT)) void kb_inv_y(const ApplyArgs *members, const BatchIO *io, int zdiv) {
    const ApplyArgs a = members[blockIdx.z / zdiv];
    if (io->active && !io->active[a.gid]) return;
    inv_y_body<R, PY, KIND>(a, blockIdx.x, blockIdx.y, 0);
}

// ------------------------------------------------------------------ whole rows, inverse x
template <typename R, int PX>
struct RowInvCfg {
    static constexpr int TPP = PencilShape<PX>::TPP;
    static constexpr int CB = (int)sizeof(cx<R>);
    static constexpr int PS = pstride<PX>();
    static constexpr int PPB = clampi(mini(256 / TPP, (64 * 1024 - PX * CB) / (PS * CB)), 1, 64);
    static constexpr int NT = PPB * TPP;
};

// Inverse x transform of two real rows from their half spectra Wa, Wb (Hx =
// PX/2 + 1 coefficients; a missing row is zero): the spectra are extended to
// Hermitian sequences A, B (imaginary parts at kx = 0 and PX/2 dropped, as
// the node gather does) and packed as A + iB, so one complex inverse FFT of
// length PX holds row a in its real and row b in its imaginary part.  Lane t
// of the pencil ends with x[e] = value at t + e TPP.  tw: the LDS twiddle
// table, already synchronised.
template <typename R, typename SH>
__device__ __forceinline__ void inv_x_load(const cx<R> *Wa, const cx<R> *Wb, bool va, bool vb, int t,
                                           cx<R> (&x)[SH::E]) {
    constexpr int PX = SH::P, TPP = SH::TPP, E = SH::E;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = t + e * TPP;
        const bool lo = 2 * k <= PX;
        const int kk = lo ? k : PX - k;  // kk < Hx
        cx<R> A = va ? Wa[kk] : cx<R>{R(0), R(0)};
        cx<R> B = vb ? Wb[kk] : cx<R>{R(0), R(0)};
        if (kk == 0 || 2 * kk == PX) {
            A.y = R(0);
            B.y = R(0);
        }
        if (!lo) {  // Hermitian extension: conj of the mirrored coefficient
            A.y = -A.y;
            B.y = -B.y;
        }
        x[e] = {A.x - B.y, A.y + B.x};  // A + iB
    }
}
template <typename R, int PX>
__device__ __forceinline__ void inv_x_pair(const cx<R> *Wa, const cx<R> *Wb, bool va, bool vb, cx<R> *pen,
                                           const cx<R> *tw, int t, cx<R> (&x)[PX / PencilShape<PX>::TPP]) {
    inv_x_load<R, PencilShape<PX>>(Wa, Wb, va, vb, t, x);
    fft_regs<R, PX, 1>(x, pen, tw, t);
}

// Long rows (those whose forward x transform was an FFT) get their inverse x
// transform by FFT too: row (d, o) of W -> Xr[d][o][x], x < nx, in the
// buffer of the forward row transforms (free after the forward pass).  The
// gather then reads their nodes' values instead of summing the row's
// spectrum once per node.
template <typename R, int PX, int KIND>
__device__ __forceinline__ void rows_inv_body(const ApplyArgs &a, const int bx) {
    using Cfg = RowInvCfg<R, PX>;
    constexpr int O = Terms<KIND>::O, TPP = Cfg::TPP, PS = Cfg::PS, PPB = Cfg::PPB, NT = Cfg::NT, E = PX / TPP;
    __shared__ cx<R> buf[PPB * PS];
    __shared__ cx<R> tw[PX];
    const int nrows = a.row_inv ? a.nd * O : 0;
    if (bx * PPB * 2 >= nrows) return;  // block-uniform: batched members with fewer long rows
    const int tid = threadIdx.x;
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    for (int i = tid; i < PX; i += NT) tw[i] = gtwx[i];
    __syncthreads();
    const int pen = tid / TPP, t = tid % TPP;
    const int ra = (bx * PPB + pen) * 2, rb = ra + 1;
    const bool va = ra < nrows, vb = rb < nrows;
    const cx<R> *W = static_cast<const cx<R> *>(a.Y);
    const size_t ostride = (size_t)a.nzo * a.ny;  // rows of W per output
    const cx<R> *Wa = W + ((size_t)(ra % O) * ostride + (va ? a.dense_rows[ra / O] : 0)) * a.hx;
    const cx<R> *Wb = W + ((size_t)(rb % O) * ostride + (vb ? a.dense_rows[rb / O] : 0)) * a.hx;
    cx<R> x[E];
    inv_x_pair<R, PX>(Wa, Wb, va, vb, buf + pen * PS, tw, t, x);
    R *Xr = static_cast<R *>(a.Xd);
#pragma unroll
    for (int e = 0; e < E / 2; ++e) {  // nx <= Px/2
        const int xg = t + e * TPP;
        if (xg < a.nx) {
            if (va) Xr[(size_t)ra * a.nx + xg] = x[e].x;
            if (vb) Xr[(size_t)rb * a.nx + xg] = x[e].y;
        }
    }
}

template <typename R, int PX, int KIND>
__global__ __launch_bounds__((RowInvCfg<R, PX>::NT)) void k_rows_inv(ApplyArgs a) {
    rows_inv_body<R, PX, KIND>(a, blockIdx.x);
}

// Batched form: blockIdx.z = member.
template <typename R, int PX, int KIND>
__global__ __launch_bounds__((RowInvCfg<R, PX>::NT)) void kb_rows_inv(const ApplyArgs *members, const BatchIO *io) {
    const ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    rows_inv_body<R, PX, KIND>(a, blockIdx.x);
}

// ------------------------------------------------------------------ k_gather
// Eight lanes per node: the inverse x transform of the node's row in W,
//   sum_kx cf Re(W[kx] exp(+2 pi i kx x / Px)),  cf = 1 at kx = 0 and Px/2,
//   2 between (the real field from its half spectrum),
// evaluated at the node's x only.  Lane l of a node takes kx = 1 + l, 9 + l,
// ... (the eight lanes read consecutive coefficients), accumulates in FP64,
// and a fixed shuffle tree sums the lanes (reproducible); the first lane
// adds kx = 0, Px/2 and r = c u - (exact - grid) self term q.
constexpr int kGatherLanes = 8;

template <typename R, int KIND>
__device__ __forceinline__ void gather_body(const ApplyArgs &a, const int bx) {
    constexpr int O = Terms<KIND>::O, L = kGatherLanes;
    __shared__ cx<R> twx[(KIND == 0 || KIND == 3) ? kMaxPx : kMaxPx / 2];  // 3D: px <= 512
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    for (int i = threadIdx.x; i < a.px; i += 256) twx[i] = gtwx[i];
    __syncthreads();
    const int sub = threadIdx.x % L;
    const int s = bx * (256 / L) + threadIdx.x / L;
    if (s >= a.m) return;  // the node's eight lanes leave together
    const int zz = a.gz[s] - a.z0, y = a.gy[s], xg = a.gx[s];
    const int dr = a.row_inv ? a.row_dense[zz * a.ny + y] : -1;
    if (dr >= 0) {  // a long row: its values come from the row FFT
        if (sub != 0) return;
        const R *Xr = static_cast<const R *>(a.Xd);
        const int j = a.perm[s];
#pragma unroll
        for (int o = 0; o < O; ++o) {
            double v = (double)Xr[((size_t)dr * O + o) * a.nx + xg];
#pragma unroll
            for (int l = 0; l < O; ++l) {
                v += a.C[((size_t)s * O + o) * O + l] * a.u[l * a.m + j];
                v -= a.SC[((size_t)s * O + o) * O + l] * a.q[l * a.m + j];
            }
            a.r[o * a.m + j] = v;
        }
        return;
    }
    const int hx = a.hx, px = a.px;
    const size_t rstride = (size_t)a.nzo * a.ny * hx;  // between outputs
    const cx<R> *row = static_cast<const cx<R> *>(a.Y) + ((size_t)zz * a.ny + y) * hx;
    double acc[O];
#pragma unroll
    for (int o = 0; o < O; ++o) acc[o] = 0.0;
    // with one output the ends of the row and the free term are loaded before the
    // sum (a 128^3 body in FP32: 6.5 -> 6.0 us; with three outputs the registers
    // cost more: 13.1 -> 13.6 us for Navier in FP64 at 93^3)
    constexpr bool EARLY = O == 1;
    int j = 0;
    cx<R> v0{}, vn{};
    double fc = 0.0, fs = 0.0, fu = 0.0, fq = 0.0;
    if constexpr (EARLY) {
        j = a.perm[s];
        v0 = row[0];
        vn = row[hx - 1];
        fc = a.C[s];
        fs = a.SC[s];
        fu = a.u[j];
        fq = a.q[j];
    }
    const int step = (L * xg) % px;
    int idx = ((1 + sub) * xg) % px;  // (kx x) mod px
    int kx = 1 + sub;
    // eight coefficients per output in flight before they are used.  Past
    // the row's end a lane loads kx = 1 (in bounds: the loop runs only when
    // hx >= 3) and weighs it by zero -- a product, so the load stays
    // unconditional and the chunk's loads are waited for together.
    for (; kx < hx - 1; kx += 8 * L) {
        cx<R> v[8][O];
        R mk[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool in = kx + k * L < hx - 1;
            const int kc = in ? kx + k * L : 1;
            mk[k] = in ? R(1) : R(0);
#pragma unroll
            for (int o = 0; o < O; ++o) v[k][o] = row[o * rstride + kc];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const cx<R> w = twx[idx];
#pragma unroll
            for (int o = 0; o < O; ++o) acc[o] += (double)((v[k][o].x * w.x + v[k][o].y * w.y) * mk[k]);
            idx += step;
            if (idx >= px) idx -= px;
        }
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1)
#pragma unroll
        for (int o = 0; o < O; ++o) acc[o] += __shfl_xor(acc[o], off, 64);
    if (sub != 0) return;
    const R wn = (xg & 1) ? R(-1) : R(1);  // exp(i pi x)
    if constexpr (EARLY) {
        double v = (double)v0.x + (double)(vn.x * wn) + 2.0 * acc[0];
        v += fc * fu;
        v -= fs * fq;
        a.r[j] = v;
        return;
    }
    j = a.perm[s];
#pragma unroll
    for (int o = 0; o < O; ++o) {
        v0 = row[o * rstride];
        vn = row[o * rstride + hx - 1];
        double v = (double)v0.x + (double)(vn.x * wn) + 2.0 * acc[o];
#pragma unroll
        for (int l = 0; l < O; ++l) {
            v += a.C[((size_t)s * O + o) * O + l] * a.u[l * a.m + j];
            v -= a.SC[((size_t)s * O + o) * O + l] * a.q[l * a.m + j];
        }
        a.r[o * a.m + j] = v;
    }
}

template <typename R, int KIND>
__global__ __launch_bounds__(256) void k_gather(ApplyArgs a) {
    gather_body<R, KIND>(a, blockIdx.x);
}

// Free term of sorted node s: c u - (exact - grid) self term q, per output.
template <int O>
__device__ __forceinline__ void free_term(const ApplyArgs &a, const int s, const int j, double *b) {
    double u[O], q[O];
#pragma unroll
    for (int l = 0; l < O; ++l) {
        u[l] = a.u[l * a.m + j];
        q[l] = a.q[l * a.m + j];
    }
#pragma unroll
    for (int o = 0; o < O; ++o) {
        b[o] = 0.0;
#pragma unroll
        for (int l = 0; l < O; ++l) {
            b[o] += a.C[((size_t)s * O + o) * O + l] * u[l];
            b[o] -= a.SC[((size_t)s * O + o) * O + l] * q[l];
        }
    }
}

// As k_gather for 2D plans of few nodes, where eight lanes per node leave most
// of the chip idle and a lane with a long chain: L lanes per node, so that one
// round of eight coefficients per lane covers the row, the twiddles straight
// from the table (no staging, no barrier) and the free term's loads ahead of the
// sum.  2000 nodes of a 500 x 500 square in FP64: 9.2 -> 4.7 us.
template <typename R, int KIND, int L>
__device__ __forceinline__ void gather_wide_body(const ApplyArgs &a, const int bx) {
    constexpr int O = Terms<KIND>::O;
    const int sub = threadIdx.x % L;
    const int s = bx * (256 / L) + threadIdx.x / L;
    if (s >= a.m) return;  // the node's lanes leave together
    const int y = a.gy[s], xg = a.gx[s], j = a.perm[s];
    const int dr = a.row_inv ? a.row_dense[y] : -1;
    double b[O];
    free_term<O>(a, s, j, b);
    if (dr >= 0) {  // a long row: its values come from the row FFT
        const R *Xr = static_cast<const R *>(a.Xd);
        if (sub == 0)
#pragma unroll
            for (int o = 0; o < O; ++o) a.r[o * a.m + j] = (double)Xr[((size_t)dr * O + o) * a.nx + xg] + b[o];
        return;
    }
    const int hx = a.hx, px = a.px;
    const float inv_px = 1.0f / (float)px;
    const size_t rstride = (size_t)a.ny * hx;  // between outputs
    const cx<R> *row = static_cast<const cx<R> *>(a.Y) + (size_t)y * hx;
    const cx<R> *twx = static_cast<const cx<R> *>(a.twx);
    cx<R> v0[O], vn[O];
    double acc[O];
#pragma unroll
    for (int o = 0; o < O; ++o) {
        v0[o] = row[o * rstride];
        vn[o] = row[o * rstride + hx - 1];
        acc[o] = 0.0;
    }
    for (int kx = 1 + sub; kx < hx - 1; kx += 8 * L) {
        cx<R> v[8][O], w[8];
        R mk[8];  // zero past the row's end, where coefficient 1 stands in
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool in = kx + k * L < hx - 1;
            const int kc = in ? kx + k * L : 1;
            mk[k] = in ? R(1) : R(0);
            w[k] = twx[mod_small(kc, xg, px, inv_px)];
#pragma unroll
            for (int o = 0; o < O; ++o) v[k][o] = row[o * rstride + kc];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int o = 0; o < O; ++o) acc[o] += (double)((v[k][o].x * w[k].x + v[k][o].y * w[k].y) * mk[k]);
    }
#pragma unroll
    for (int off = L / 2; off > 0; off >>= 1)
#pragma unroll
        for (int o = 0; o < O; ++o) acc[o] += __shfl_xor(acc[o], off, 64);
    if (sub != 0) return;
    const R wn = (xg & 1) ? R(-1) : R(1);  // exp(i pi x)
#pragma unroll
    for (int o = 0; o < O; ++o) a.r[o * a.m + j] = ((double)v0[o].x + (double)(vn[o].x * wn) + 2.0 * acc[o]) + b[o];
}

template <typename R, int KIND, int L>
__global__ __launch_bounds__(256) void k_gather_wide(ApplyArgs a) {
    gather_wide_body<R, KIND, L>(a, blockIdx.x);
}

template <typename R, int KIND, int L>
__global__ __launch_bounds__(256) void kb_gather_wide(const ApplyArgs *members, const BatchIO *io) {
    ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    a.r = io->r + a.off;
    gather_wide_body<R, KIND, L>(a, blockIdx.x);
}

// 2D plans whose nodes all lie in long rows (a whole loaded surface): inverse x
// transform of one row's outputs and its nodes' results in one block, without
// the row's values going through memory.  256^2 half-space
// surface in FP32: k_rows_inv 6.6 + k_gather 12.6 us -> 10.1 us.
template <typename R, int PX, int KIND>
__device__ __forceinline__ void rows_gather_body(const ApplyArgs &a, const int d) {
    using SH = LineShape<PX, KIND>;
    constexpr int O = Terms<KIND>::O, TPP = SH::TPP, PS = pstride<PX>(), E = SH::E;
    constexpr int NP = (O + 1) / 2;  // two outputs per pencil
    static_assert(NP * TPP <= 256, "a thread for every pencil lane");
    __shared__ cx<R> buf[NP * PS];
    __shared__ cx<R> tw[PX];
    const int tid = threadIdx.x;
    if (d >= a.nd) return;  // block-uniform: batched members with fewer rows
    const cx<R> *gtwx = static_cast<const cx<R> *>(a.twx);
    for (int i = tid; i < PX; i += 256) tw[i] = gtwx[i];
    const int y = a.dense_rows[d];
    const int s0 = a.rowptr[y], s1 = a.rowptr[y + 1];
    const int pen = tid / TPP, t = tid % TPP;
    cx<R> x[E];
    if (pen < NP) {
        const cx<R> *W = static_cast<const cx<R> *>(a.Y) + (size_t)y * a.hx;
        const size_t ostride = (size_t)a.ny * a.hx;
        const bool vb = 2 * pen + 1 < O;
        inv_x_load<R, SH>(W + 2 * pen * ostride, W + (2 * pen + (vb ? 1 : 0)) * ostride, true, vb, t, x);
    }
    // items (node, output), outputs fastest: neighbouring lanes read neighbouring
    // parts of the 72 bytes of a node's blocks.  The first O items of a thread
    // (all of a row of 256 nodes): their loads run beside the transform's.
    const int i0 = s0 * O + tid, i1 = s1 * O;
    double b[O];
    int j[O], xg[O];
    auto item = [&](int i, double &bi, int &ji, int &xi) {
        const int s = i / O, o = i % O;
        ji = a.perm[s];
        xi = a.gx[s];
        bi = 0.0;
#pragma unroll
        for (int l = 0; l < O; ++l) {
            bi += a.C[(size_t)i * O + l] * a.u[l * a.m + ji];
            bi -= a.SC[(size_t)i * O + l] * a.q[l * a.m + ji];
        }
        ji += o * a.m;
    };
#pragma unroll
    for (int k = 0; k < O; ++k)
        if (i0 + 256 * k < i1) item(i0 + 256 * k, b[k], j[k], xg[k]);
    __syncthreads();
    if (pen < NP) {
        fft_regs_s<R, SH, 1>(x, buf + pen * PS, tw, t);
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < E / 2; ++e) buf[pen * PS + pslot(t + e * TPP)] = x[e];
    }
    __syncthreads();
    auto value = [&](int i, int xi) {
        const cx<R> v = buf[i % O / 2 * PS + pslot(xi)];
        return (double)(i % O % 2 ? v.y : v.x);
    };
#pragma unroll
    for (int k = 0; k < O; ++k)
        if (i0 + 256 * k < i1) a.r[j[k]] = value(i0 + 256 * k, xg[k]) + b[k];
    for (int i = i0 + 256 * O; i < i1; i += 256) {
        item(i, b[0], j[0], xg[0]);
        a.r[j[0]] = value(i, xg[0]) + b[0];
    }
}

template <typename R, int PX, int KIND>
__global__ __launch_bounds__(256) void k_rows_gather(ApplyArgs a) {
    rows_gather_body<R, PX, KIND>(a, blockIdx.x);
}

template <typename R, int PX, int KIND>
__global__ __launch_bounds__(256) void kb_rows_gather(const ApplyArgs *members, const BatchIO *io) {
    ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    a.r = io->r + a.off;
    rows_gather_body<R, PX, KIND>(a, blockIdx.x);
}

template <typename R, int KIND>
__global__ __launch_bounds__(256) void kb_gather(const ApplyArgs *members, const BatchIO *io) {
    ApplyArgs a = members[blockIdx.z];
    if (io->active && !io->active[a.gid]) return;
    a.q = io->q + a.off;
    a.u = io->u + a.off;
    a.r = io->r + a.off;
    gather_body<R, KIND>(a, blockIdx.x);
}

// ------------------------------------------------------------------ launchers
template <typename R, int PY, int KIND, typename YS = cx<R>>
int launch_fwd(const ApplyArgs &a, hipStream_t st) {
    using Cfg = FwdCfg<R, PY, KIND>;
    const int nkx = (a.hx + Cfg::KXC - 1) / Cfg::KXC;
    const dim3 grid = std::is_same<YS, cbf16>::value ? dim3(a.nzo, nkx) : dim3(8 * ((nkx * a.nzo + 7) / 8));  // xcd_item
    if (a.fwd_xg == 2) hipLaunchKernelGGL((k_fwd_xy<R, PY, KIND, 2, YS>), grid, dim3(Cfg::NT), 0, st, a);
    else hipLaunchKernelGGL((k_fwd_xy<R, PY, KIND, 1, YS>), grid, dim3(Cfg::NT), 0, st, a);
    BF_HIP(hipGetLastError());
    return 0;
}
template <typename R, int PY, int KIND, typename ZS = cx<R>>
int launch_inv_y(const ApplyArgs &a, int all_rows, hipStream_t st) {
    using Cfg = InvYCfg<R, PY, KIND>;
    dim3 grid((a.hx + Cfg::KXC - 1) / Cfg::KXC, a.nzo);
    hipLaunchKernelGGL((k_inv_y<R, PY, KIND, ZS>), grid, dim3(Cfg::NT), 0, st, a, all_rows);
    BF_HIP(hipGetLastError());
    return 0;
}
template <typename R, int PZ, int KIND, int SCHED>
int launch_z(const ApplyArgs &a, hipStream_t st) {
    using SH = ZSched<R, KIND, PZ, SCHED>;
    using Cfg = ZCfg<R, SH, KIND>;
    static_assert(Cfg::KT == 1 << z_tile_log2(KIND, sizeof(R) == 8, PZ, SCHED), "the forward pass's tiles");
    if (a.py % Cfg::TY != 0 || 2 * a.nzo > PZ + 1) {
        set_error("z pass: y length or planes do not fit the schedule");
        return BEMFFT_EUNSUPPORTED;
    }
    const int nby = a.py / Cfg::TY;
    const int per = (a.hx * nby + 7) / 8;  // xcd_item
    hipLaunchKernelGGL((k_zpass<R, SH, KIND>), dim3(8 * per), dim3(Cfg::NT), 0, st, a, nby);
    BF_HIP(hipGetLastError());
    return 0;
}

#define BF_SIZE_SWITCH(len, FN, ...)                        \
    switch (len) {                                          \
        case 32: return FN<32>(__VA_ARGS__);                \
        case 64: return FN<64>(__VA_ARGS__);                \
        case 96: return FN<96>(__VA_ARGS__);                \
        case 128: return FN<128>(__VA_ARGS__);              \
        case 192: return FN<192>(__VA_ARGS__);              \
        case 256: return FN<256>(__VA_ARGS__);              \
        case 320: return FN<320>(__VA_ARGS__);              \
        case 384: return FN<384>(__VA_ARGS__);              \
        case 512: return FN<512>(__VA_ARGS__);              \
        default: break;                                     \
    }

// As BF_SIZE_SWITCH, plus length 1024 for the 2D families (grids of up to
// 512 points per axis); 3D plans never reach it and do not compile it.
#define BF_SIZE_SWITCH_K(KIND_, len, FN, ...)                              \
    if constexpr (KIND_ == 0 || KIND_ == 3) {                              \
        if ((len) == 1024) return FN<1024>(__VA_ARGS__);                   \
    }                                                                      \
    BF_SIZE_SWITCH(len, FN, __VA_ARGS__)

template <typename R, int KIND>
struct Launch {
    static constexpr bool FLAT = KIND == 0 || KIND == 3;  // 2D plans
    template <int P> static int fwd(const ApplyArgs &a, hipStream_t st) { return launch_fwd<R, P, KIND>(a, st); }
    template <int P> static int rows(const ApplyArgs &a, hipStream_t st) {
        using Cfg = RowCfg<R, P, KIND>;
        const int nfb = a.flat & kFlatRows ? 0 : (a.m + 255) / 256;  // long rows take q and u themselves
        const int nrb = a.nd;  // one block per long row
        hipLaunchKernelGGL((k_fields_rows<R, P, KIND>), dim3(nfb + nrb), dim3(256), 0, st, a, nfb);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P> static int rows_inv(const ApplyArgs &a, hipStream_t st) {
        using Cfg = RowInvCfg<R, P>;
        const int nb = (a.nd * Terms<KIND>::O + 2 * Cfg::PPB - 1) / (2 * Cfg::PPB);
        hipLaunchKernelGGL((k_rows_inv<R, P, KIND>), dim3(nb), dim3(Cfg::NT), 0, st, a);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P> static int brows_inv(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        using Cfg = RowInvCfg<R, P>;
        const int nb = (g.max_nd * Terms<KIND>::O + 2 * Cfg::PPB - 1) / (2 * Cfg::PPB);
        hipLaunchKernelGGL((kb_rows_inv<R, P, KIND>), dim3(nb, 1, g.nmem), dim3(Cfg::NT), 0, st, dm, io);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int dispatch_rows_inv(const ApplyArgs &a, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, a.px, rows_inv, a, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    template <int P> static int inv_y(const ApplyArgs &a, int all_rows, hipStream_t st) {
        return launch_inv_y<R, P, KIND>(a, all_rows, st);
    }
    template <int P> static int z(const ApplyArgs &a, hipStream_t st) {
        if constexpr (KIND == 2) {
            if (a.zsched == 2) return launch_z<R, P, KIND, 2>(a, st);
        }
        return a.zsched == 1 ? launch_z<R, P, KIND, 1>(a, st) : launch_z<R, P, KIND, 0>(a, st);
    }

    // Everything up to W.  all_rows: W of every row y < ny (the grid
    // evaluation), not only of those that hold nodes (the apply).  ev (optional):
    // events 0-3 recorded around the three stages; 2D plans have one between
    // the fields and W, counted as the second.
    static int front(const ApplyArgs &a, int all_rows, hipStream_t st, hipEvent_t *ev = nullptr) {
        if (ev) BF_HIP(hipEventRecord(ev[0], st));
        if constexpr (FLAT) {
            const bool fold = a.flat & kFlatFold;
            if (!fold) BF_CHECK(a.nd > 0 ? dispatch_rows(a, st) : fields(a, st));
            if (ev) BF_HIP(hipEventRecord(ev[1], st));
            BF_CHECK(dispatch_mid(a, fold, all_rows, st));
            if (ev) BF_HIP(hipEventRecord(ev[2], st));
        } else {
            if (a.nd > 0) {
                BF_CHECK(dispatch_rows(a, st));  // fields and long-row transforms, one launch
            } else {
                BF_CHECK(fields(a, st));
            }
            BF_CHECK(dispatch_fwd(a, st));
            if (ev) BF_HIP(hipEventRecord(ev[1], st));
            BF_CHECK(dispatch_z(a, st));
            if (ev) BF_HIP(hipEventRecord(ev[2], st));
            BF_CHECK(dispatch_inv_y(a, all_rows, st));
        }
        if (ev) BF_HIP(hipEventRecord(ev[3], st));
        return 0;
    }

    // ev (optional): five events recorded around the four stages.
    static int run(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev = nullptr) {
        BF_CHECK(front(a, 0, st, ev));
        BF_CHECK(back(a, st));
        if (ev) BF_HIP(hipEventRecord(ev[4], st));
        return 0;
    }
    // W -> r
    static int back(const ApplyArgs &a, hipStream_t st) {
        if constexpr (FLAT) {
            if (a.flat & kFlatRows) return dispatch_rows_gather(a, st);
        }
        if (a.nd > 0 && a.row_inv) BF_CHECK(dispatch_rows_inv(a, st));
        if constexpr (FLAT) {
            if (a.flat & kFlatWide)
                return a.px >= 1024 ? gather_wide<64>(a, st) : a.px >= 512 ? gather_wide<32>(a, st) : gather_wide<16>(a, st);
        }
        return gather(a, st);
    }
    template <int L> static int gather_wide(const ApplyArgs &a, hipStream_t st) {
        constexpr int NPB = 256 / L;  // nodes per block
        hipLaunchKernelGGL((k_gather_wide<R, KIND, L>), dim3((a.m + NPB - 1) / NPB), dim3(256), 0, st, a);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P> static int rows_gather(const ApplyArgs &a, hipStream_t st) {
        hipLaunchKernelGGL((k_rows_gather<R, P, KIND>), dim3(a.nd), dim3(256), 0, st, a);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int dispatch_rows_gather(const ApplyArgs &a, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, a.px, rows_gather, a, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    template <int L>
    static int bgather_wide(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        constexpr int NPB = 256 / L;
        hipLaunchKernelGGL((kb_gather_wide<R, KIND, L>), dim3((g.max_m + NPB - 1) / NPB, 1, g.nmem), dim3(256), 0, st, dm,
                           io);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P>
    static int brows_gather(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        hipLaunchKernelGGL((kb_rows_gather<R, P, KIND>), dim3(g.max_nd, 1, g.nmem), dim3(256), 0, st, dm, io);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int dispatch_brows_gather(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, g.px, brows_gather, dm, io, g, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    template <int P> static int mid(const ApplyArgs &a, bool fold, int all_rows, hipStream_t st) {
        const dim3 grid(8 * ((a.hx + 7) / 8)), block(Mid2dCfg<R, P, KIND>::NT);
        if (fold) hipLaunchKernelGGL((k_mid2d<R, P, KIND, true>), grid, block, 0, st, a, all_rows);
        else hipLaunchKernelGGL((k_mid2d<R, P, KIND, false>), grid, block, 0, st, a, all_rows);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int dispatch_mid(const ApplyArgs &a, bool fold, int all_rows, hipStream_t st) {
        if (a.pz != 1) {
            set_error("2D plans need pz == 1");
            return BEMFFT_EUNSUPPORTED;
        }
        BF_SIZE_SWITCH_K(KIND, a.py, mid, a, fold, all_rows, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    template <int P>
    static int bmid(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, bool fold, bool lean, hipStream_t st) {
        const dim3 grid(8 * ((g.hx + 7) / 8), 1, g.nmem), block(Mid2dCfg<R, P, KIND>::NT);
        if (fold && lean) hipLaunchKernelGGL((kb_mid2d<R, P, KIND, true, true>), grid, block, 0, st, dm, io);
        else if (fold) hipLaunchKernelGGL((kb_mid2d<R, P, KIND, true, false>), grid, block, 0, st, dm, io);
        else hipLaunchKernelGGL((kb_mid2d<R, P, KIND, false, true>), grid, block, 0, st, dm, io);
        BF_HIP(hipGetLastError());
        return 0;
    }
    // Blocks of the folded form that stay resident, at its two wavefronts per SIMD:
    // beyond, the lean form is faster although it takes the fields in a launch of
    // their own (circles on 128^2 FP32, 387, 516 and 1032 blocks of 512: 15.4, 20.7 and
    // 28.0 us, lean 16.3, 16.9 and 18.7).
    template <int P> static int fold_resident() { return 256 * (8 / (Mid2dCfg<R, P, KIND>::NT / 64)); }
    static int dispatch_fold_resident(int py) {
        BF_SIZE_SWITCH_K(KIND, py, fold_resident);
        return 0;
    }
    static int dispatch_bmid(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, bool fold, bool lean,
                             hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, g.py, bmid, dm, io, g, fold, lean, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int fields(const ApplyArgs &a, hipStream_t st) {
        hipLaunchKernelGGL((k_fields<R, KIND>), dim3((a.m + 255) / 256), dim3(256), 0, st, a);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int gather(const ApplyArgs &a, hipStream_t st) {
        constexpr int NPB = 256 / kGatherLanes;  // nodes per block
        hipLaunchKernelGGL((k_gather<R, KIND>), dim3((a.m + NPB - 1) / NPB), dim3(256), 0, st, a);
        BF_HIP(hipGetLastError());
        return 0;
    }
    static int dispatch_fwd(const ApplyArgs &a, hipStream_t st) {
        BF_SIZE_SWITCH(a.py, fwd, a, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    // ---- batched: one launch per stage for all members of a group
    template <int P> static int bfwd(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        using Cfg = FwdCfg<R, P, KIND>;
        dim3 grid(8 * (((g.hx + Cfg::KXC - 1) / Cfg::KXC * g.max_nzo + 7) / 8), 1, g.nmem);
        hipLaunchKernelGGL((kb_fwd_xy<R, P, KIND>), grid, dim3(Cfg::NT), 0, st, dm, io);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P> static int brows(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        using Cfg = RowCfg<R, P, KIND>;
        dim3 grid(g.max_nd, 1, g.nmem);  // one block per long row
        hipLaunchKernelGGL((kb_rows_fft<R, P, KIND>), grid, dim3(256), 0, st, dm, io, 1);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P> static int binv(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        using Cfg = InvYCfg<R, P, KIND>;
        dim3 grid((g.hx + Cfg::KXC - 1) / Cfg::KXC, g.max_nzo, g.nmem);
        hipLaunchKernelGGL((kb_inv_y<R, P, KIND>), grid, dim3(Cfg::NT), 0, st, dm, io, 1);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int PZ, int SCHED>
    static int bz_s(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, const ZRange &r, hipStream_t st) {
        using SH = ZSched<R, KIND, PZ, SCHED>;
        using Cfg = ZCfg<R, SH, KIND>;
        const int nby = g.py / Cfg::TY;
        dim3 grid(8 * ((g.hx * nby + 7) / 8), 1, r.nmem);
        hipLaunchKernelGGL((kb_zpass<R, SH, KIND>), grid, dim3(Cfg::NT), 0, st, dm + r.first, io, nby);
        BF_HIP(hipGetLastError());
        return 0;
    }
    template <int P>
    static int bz(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, const ZRange &r, hipStream_t st) {
        if constexpr (KIND == 2) {
            if (r.zsched == 2) return bz_s<P, 2>(dm, io, g, r, st);
        }
        return r.zsched == 1 ? bz_s<P, 1>(dm, io, g, r, st) : bz_s<P, 0>(dm, io, g, r, st);
    }
    static int dispatch_brows(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, g.px, brows, dm, io, g, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_bfwd(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        BF_SIZE_SWITCH(g.py, bfwd, dm, io, g, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_bz(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, const ZRange &r, hipStream_t st) {
        BF_SIZE_SWITCH(r.pz, bz, dm, io, g, r, st);
        set_error("unsupported z length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_binv(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        BF_SIZE_SWITCH(g.py, binv, dm, io, g, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_brows_inv(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, g.px, brows_inv, dm, io, g, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int run_batch(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st) {
        bool fold = false, lean = true;
        if constexpr (FLAT) {
            fold = g.flat & kFlatFold;
            lean = !fold || g.nmem * g.hx > dispatch_fold_resident(g.py);
        }
        if (lean && (fold || !(g.flat & kFlatRows))) {  // all in long rows: those take q and u themselves
            hipLaunchKernelGGL((kb_fields<R, KIND>), dim3((g.max_m + 255) / 256, 1, g.nmem), dim3(256), 0, st, dm, io, 1);
            BF_HIP(hipGetLastError());
        }
        if (!fold && g.max_nd > 0) BF_CHECK(dispatch_brows(dm, io, g, st));
        if constexpr (FLAT) {
            BF_CHECK(dispatch_bmid(dm, io, g, fold, lean, st));
        } else {
            BF_CHECK(dispatch_bfwd(dm, io, g, st));
            for (int i = 0; i < g.nz; ++i) BF_CHECK(dispatch_bz(dm, io, g, g.z[i], st));
            BF_CHECK(dispatch_binv(dm, io, g, st));
        }
        if constexpr (FLAT) {
            if (g.flat & kFlatRows) return dispatch_brows_gather(dm, io, g, st);
        }
        if (g.max_nd > 0 && g.row_inv) BF_CHECK(dispatch_brows_inv(dm, io, g, st));
        if constexpr (FLAT) {
            if (g.flat & kFlatWide)
                return g.px >= 1024  ? bgather_wide<64>(dm, io, g, st)
                       : g.px >= 512 ? bgather_wide<32>(dm, io, g, st)
                                     : bgather_wide<16>(dm, io, g, st);
        }
        constexpr int NPB = 256 / kGatherLanes;  // nodes per block
        hipLaunchKernelGGL((kb_gather<R, KIND>), dim3((g.max_m + NPB - 1) / NPB, 1, g.nmem), dim3(256), 0, st, dm, io);
        BF_HIP(hipGetLastError());
        return 0;
    }

    static int dispatch_rows(const ApplyArgs &a, hipStream_t st) {
        BF_SIZE_SWITCH_K(KIND, a.px, rows, a, st);
        set_error("unsupported x length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_inv_y(const ApplyArgs &a, int all_rows, hipStream_t st) {
        BF_SIZE_SWITCH(a.py, inv_y, a, all_rows, st);
        set_error("unsupported y length");
        return BEMFFT_EUNSUPPORTED;
    }
    static int dispatch_z(const ApplyArgs &a, hipStream_t st) {
        BF_SIZE_SWITCH(a.pz, z, a, st);
        set_error("unsupported z length");
        return BEMFFT_EUNSUPPORTED;
    }
};

// Per-family entry points, instantiated in one source file per family.
template <int KIND>
int apply_kind(int precision, const ApplyArgs &a, hipStream_t st, hipEvent_t *ev);
template <int KIND>
int apply_batch_kind(int precision, const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st);

// The same for one precision, each in a source file of its own.
template <int KIND, int PREC>
int apply_prec(const ApplyArgs &a, hipStream_t st, hipEvent_t *ev);
template <int KIND, int PREC>
int apply_batch_prec(const ApplyArgs *dm, const BatchIO *io, const GroupDims &g, hipStream_t st);
template <int KIND, int PREC>
int volume_prec(const ApplyArgs &a, double *out, hipStream_t st, hipEvent_t *ev);

// Apply arguments of plan p with the spectra/tables of 'shared' and the
// intermediate buffers of 'ws' (q, u, r left null).
void fill_apply_args(const bemfft_plan *p, const Engine &shared, const Engine &ws, ApplyArgs *a);
// Intermediate buffers of one apply of plan p (Y, Z, fields, long rows),
// without spectra or tables.
int alloc_intermediates(const bemfft_plan *p, int precision, Engine *e);

}  // namespace bemfft
