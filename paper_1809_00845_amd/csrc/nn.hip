// nn.hip -- a small convolutional network that proposes the initial guess
// of the iterative solve (the unknown flux q of a Dirichlet problem, Sec. 4),
// with its own forward, backward and optimiser kernels.
//
// Input: voxel channels on the plan's grid, nonzero only at boundary nodes:
// a = w/h^2, a n_x, a n_y, a n_z, a s u and a s b, with s = 1/rms(u) over
// the Dirichlet nodes and b the right-hand side of the solve (minus the
// operator applied to the known values, one application of eq. 16).
// Layers: 3x3x3 convolutions with dilations d_l (zero padding), ReLU between
// layers, one output channel read back at the node voxels as s h q.
// Training (FP32 storage and arithmetic, the convolutions on the matrix
// cores) minimises the weighted squared error sum_j wt_j (y(v_j) - s h q_j)^2
// against solved problems, with Adam.
// Inference (the guess) runs in FP16 on the matrix cores with FP32
// accumulation.  The solve keeps the guess only when its residual is smaller
// than ||b|| (plain GMRES from zero otherwise).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <type_traits>
#include <vector>

#include "internal.hpp"

struct bemfft_net {
    int G = 0, cin = 0, width = 0, nl = 0;
    int64_t V = 0;  // G^3
    std::vector<int> dil, ci, co;
    std::vector<int64_t> woff, boff;
    int64_t nparam = 0;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // params, grads, Adam moments
    float *xcl = nullptr;                   // training input, channel-last [V][8]
    float *post = nullptr;                  // activations per layer [V][co] (after the ReLU of hidden layers)
    float *ga = nullptr, *gb = nullptr;     // gradient ping-pong [V][width]
    float *part = nullptr;                  // weight-gradient partial sums
    float *red = nullptr;                   // loss partial sums
    float *y = nullptr;                     // output of the last forward [V]
    int64_t t = 0;                          // Adam step
    double *dq = nullptr, *du = nullptr, *db = nullptr;  // right-hand side scratch [cap]
    int64_t cap = 0;
    // inference in FP16: channel-last activations [V][16] (ping-pong), packed
    // weights [layer][27][16][16], biases [layer][16], scale s on the device
    _Float16 *ha = nullptr, *hb = nullptr, *wp = nullptr;
    float *bp = nullptr;
    double *sdev = nullptr;
    int64_t *d_woff = nullptr, *d_boff = nullptr;
    int *d_ci = nullptr, *d_co = nullptr;
};

namespace bemfft {
namespace {

constexpr int kWgBlocks = 512;  // most weight-gradient blocks (partial sums) of a layer
constexpr int64_t kMaxTargets = 65536LL * 256;  // loss partial sums: one per 256 targets

__device__ __forceinline__ void vox_xyz(int64_t v, int G, int &x, int &y, int &z) {
    x = (int)(v % G);
    y = (int)((v / G) % G);
    z = (int)(v / ((int64_t)G * G));
}

__global__ void k_fill(float *a, int64_t n, float v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = v;
}

// known values into their slots: u where bc = 0 (or bc absent), q where bc = 1
__global__ void k_nn_split(const uint8_t *bc, const double *known, double *q, double *u, int64_t m) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= m) return;
    const bool qk = bc != nullptr && bc[j] != 0;
    q[j] = qk ? known[j] : 0.0;
    u[j] = qk ? 0.0 : known[j];
}

// input channels at the node voxels (the buffer was cleared before); r is
// the operator applied to the known values (b = -r).  Nodes that share a
// voxel add up; atomics keep that correct whatever the node order.
__global__ void k_nn_input(const int *gx, const int *gy, const int *gz, const int *perm, const double *w,
                           const double *nrm, const double *known, const double *r, const uint8_t *bc, int64_t m,
                           int G, double inv_h2, double s_host, const double *s_dev, float *x, int64_t V) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= m) return;
    const double s = s_dev ? *s_dev : s_host;
    const int j = perm[k];
    const int64_t v = ((int64_t)gz[k] * G + gy[k]) * G + gx[k];
    const double ww = w[k] * inv_h2;
    const double u = (bc == nullptr || bc[j] == 0) ? known[j] : 0.0;
    atomicAdd(&x[v], (float)ww);
    atomicAdd(&x[V + v], (float)(ww * nrm[k]));
    atomicAdd(&x[2 * V + v], (float)(ww * nrm[m + k]));
    atomicAdd(&x[3 * V + v], (float)(ww * nrm[2 * m + k]));
    atomicAdd(&x[4 * V + v], (float)(ww * s * u));
    atomicAdd(&x[5 * V + v], (float)(-ww * s * r[j]));
}

// gW[c][ci][t] = sum over the chunks of part; gb[c] likewise.  A block
// takes 32 outputs; eight groups of 32 threads sum eight contiguous slices
// of the chunks, added in a fixed order: deterministic.
__global__ __launch_bounds__(256) void k_conv_w_reduce(const float *part, int nchunk, int cin, int cout, float *gW,
                                                       float *gb) {
    __shared__ float sm[8][32];
    const int o = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const int i = blockIdx.x * 32 + o;
    const int nw = cout * cin * 27;
    int off = -1;
    if (i < nw) {
        const int c = i / (cin * 27), r = i % (cin * 27), k = r / 27, t = r % 27;
        off = (c * cin + k) * 28 + t;
    } else if (i < nw + cout) {
        off = ((i - nw) * cin + 0) * 28 + 27;
    }
    const int per = (nchunk + 7) / 8, c0 = sl * per, c1 = c0 + per < nchunk ? c0 + per : nchunk;
    const int64_t stride = (int64_t)cout * cin * 28;
    float s = 0.f;
    if (off >= 0) {
        int ch = c0;
        for (; ch + 16 <= c1; ch += 16) {  // sixteen loads in flight, added in order
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = part[(ch + i) * stride + off];
#pragma unroll
            for (int i = 0; i < 16; ++i) s += v[i];
        }
        for (; ch < c1; ++ch) s += part[ch * stride + off];
    }
    sm[sl][o] = s;
    __syncthreads();
    if (sl == 0 && off >= 0) {
        const float tot = ((sm[0][o] + sm[1][o]) + (sm[2][o] + sm[3][o])) + ((sm[4][o] + sm[5][o]) + (sm[6][o] + sm[7][o]));
        if (i < nw) gW[i] = tot;
        else gb[i - nw] = tot;
    }
}

// weighted squared error at the node voxels; dL/dy scattered into gy
// (targets whose voxel lies outside [0, V) are skipped: no access is made)
__global__ void k_nn_loss(const float *y, const int *vox, const float *tgt, const float *wt, int64_t nt, int64_t V,
                          float *gy, float *red) {
    __shared__ float sm[4];
    const int64_t i = blockIdx.x * 256 + threadIdx.x;
    float l = 0.f;
    if (i < nt) {
        const int v = vox[i];
        if (v >= 0 && v < V) {
            const float e = y[v] - tgt[i];
            l = wt[i] * e * e;
            atomicAdd(&gy[v], 2.f * wt[i] * e);
        }
    }
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
    if (threadIdx.x % 64 == 0) sm[threadIdx.x / 64] = l;
    __syncthreads();
    if (threadIdx.x == 0) red[blockIdx.x] = (sm[0] + sm[1]) + (sm[2] + sm[3]);
}

__global__ void k_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float c1, float c2, float eps) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// x0 at the Dirichlet slots: y(v_j) / (s h)
__global__ void k_nn_gather(const float *y, const int *gx, const int *gy, const int *gz, const int *perm,
                            const uint8_t *bc, int64_t m, int G, const double *s_dev, double h, double *x0) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= m) return;
    const int j = perm[k];
    const int64_t v = ((int64_t)gz[k] * G + gy[k]) * G + gx[k];
    x0[j] = (bc == nullptr || bc[j] == 0) ? (double)y[v] / (*s_dev * h) : 0.0;
}

// s = 1/rms(u) over the Dirichlet slots (1 if there are none or u = 0):
// one block, fixed-order reduction; eight values per thread in flight (one at
// a time the loop waited for each load: 20k nodes 24 -> 5 us).
__global__ __launch_bounds__(1024) void k_nn_scale(const double *known, const uint8_t *bc, int64_t m, double *s_out) {
    __shared__ double ss[16], sc[16];
    double a = 0.0, c = 0.0;
    for (int64_t j0 = threadIdx.x; j0 < m; j0 += 8 * 1024) {
        double k[8];
        bool on[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t j = j0 + i * 1024;
            on[i] = j < m;
            const int64_t jc = on[i] ? j : 0;
            k[i] = known[jc];
            if (bc != nullptr) on[i] = on[i] && bc[jc] == 0;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            a += on[i] ? k[i] * k[i] : 0.0;
            c += on[i] ? 1.0 : 0.0;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        c += __shfl_xor(c, o, 64);
    }
    if (threadIdx.x % 64 == 0) {
        ss[threadIdx.x / 64] = a;
        sc[threadIdx.x / 64] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = c = 0.0;
        for (int w = 0; w < 16; ++w) {
            a += ss[w];
            c += sc[w];
        }
        *s_out = (a > 0.0 && c > 0.0) ? 1.0 / sqrt(a / c) : 1.0;
    }
}

__device__ __forceinline__ int xcd_rank(int b, int nb) { return nb % 8 == 0 ? (b % 8) * (nb / 8) + b / 8 : b; }

// ---------------------------------------------------------------- FP16 inference
// Implicit-GEMM convolution on the matrix cores: for each tap t, the 16 x 16
// weight block W[c][ci][t] (rows c) times the 16 x 16 block of activations
// act[v_j + d o_t][ci] of 16 consecutive voxels (columns j), accumulated in
// FP32 over the 27 taps.  Activations are FP16, channel-last [V][16], so one
// lane's four B values are one 8-byte load.  Operand layout of the 16x16x16
// MFMA (wave of 64): A[i][k] at lane i + 16 (k / 4), element k % 4; B[k][j] at
// lane j + 16 (k / 4), element k % 4; D[i][j] at lane j + 16 (i / 4),
// element i % 4.
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// planar FP32 [cin][V] -> channel-last FP16 [V][16], channels >= cin zero
__global__ void k_to_cl16(const float *x, int cin, int64_t V, _Float16 *o) {
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= V) return;
    h4 w[4];
#pragma unroll
    for (int c = 0; c < 16; ++c) w[c / 4][c % 4] = (_Float16)(c < cin ? x[(int64_t)c * V + v] : 0.f);
    h4 *dst = reinterpret_cast<h4 *>(o + v * 16);
#pragma unroll
    for (int q = 0; q < 4; ++q) dst[q] = w[q];
}

// FP32 parameters W[co][ci][27], b[co] of every layer -> FP16 Wp[l][27][16][16]
// (zero-padded to 16 x 16) and FP32 bp[l][16]
__global__ void k_pack16(const float *p, const int64_t *woff, const int64_t *boff, const int *ci, const int *co,
                         _Float16 *wp, float *bp) {
    const int l = blockIdx.y;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // t*256 + c*16 + k
    if (i >= 27 * 256) return;
    const int t = i / 256, c = (i / 16) % 16, k = i % 16;
    const float w = (c < co[l] && k < ci[l]) ? p[woff[l] + ((int64_t)c * ci[l] + k) * 27 + t] : 0.f;
    wp[(int64_t)l * 27 * 256 + i] = (_Float16)w;
    if (i < 16) bp[l * 16 + i] = i < co[l] ? p[boff[l] + i] : 0.f;
}

// Tiles of 16 consecutive voxels; each wave keeps its weight operands in
// registers and walks many tiles.  gfx950's 16x16x32 FP16 product takes two
// taps per instruction (K = 2 x 16 input channels): for each (dy, dz) row the
// dx = -1 and 0 taps share one product and dx = +1 takes one with a zero
// second half, so a tile needs 18 products instead of 27.  Lane (j, kq) holds
// voxel j's channels 8 (kq % 2) .. + 7 of the first tap (kq < 2) or of the
// second (kq >= 2), loaded as one 16-byte word; neighbours outside the grid
// are zero padding.  Blocks are mapped so that the 8 XCDs (blocks go round-
// robin to them) each sweep one contiguous range of tiles: the dilated taps
// then re-read planes that the same XCD's L2 just fetched.  Three
// accumulators (one per dz) keep three independent MFMA chains.
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

template <bool LAST>
__global__ __launch_bounds__(256) void k_conv16(const _Float16 *__restrict__ in, const _Float16 *__restrict__ Wp,
                                                const float *__restrict__ bias, _Float16 *__restrict__ out,
                                                float *__restrict__ y, int G, int d, int64_t ntiles) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int half = 8 * (kq & 1);  // this lane's eight channels of its tap
    const bool first = kq < 2;      // first tap of the pair (else the second)
    const h8 zero8 = {};
    // A operands: per (dz, dy) row, the pair (dx = -1, dx = 0) and (dx = +1, none)
    h8 A[9][2];
#pragma unroll
    for (int rq = 0; rq < 9; ++rq) {
        const int t0 = rq * 3;  // tap index q * 9 + r * 3 + (dx + 1), rq = q * 3 + r
        const int ta = first ? t0 : t0 + 1;
        A[rq][0] = *reinterpret_cast<const h8 *>(Wp + (ta * 16 + j) * 16 + half);
        A[rq][1] = first ? *reinterpret_cast<const h8 *>(Wp + ((t0 + 2) * 16 + j) * 16 + half) : zero8;
    }
    float br[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) br[r] = bias[4 * kq + r];
    const int64_t V = (int64_t)G * G * G;
    const int xcd = blockIdx.x % 8, lb = blockIdx.x / 8, nlb = gridDim.x / 8;
    const int64_t per = (ntiles + 7) / 8;
    const int64_t t_lo = xcd * per, t_hi = (t_lo + per < ntiles) ? t_lo + per : ntiles;
    for (int64_t tile = t_lo + (int64_t)lb * 4 + wave; tile < t_hi; tile += (int64_t)nlb * 4) {
        const int64_t v = tile * 16 + j;
        const bool valid = v < V;
        int x, yy, z;
        vox_xyz(valid ? v : 0, G, x, yy, z);
        f4 acc[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};
        // pair 0: x - d (first) and x (second); pair 1: x + d (first), zero
        const int xa = first ? x - d : x;
        const int xb = x + d;
#pragma unroll
        for (int q = 0; q < 3; ++q) {  // dz = q - 1
            const int zz = z + d * (q - 1);
#pragma unroll
            for (int r = 0; r < 3; ++r) {  // dy = r - 1
                const int y2 = yy + d * (r - 1);
                const bool row_ok = valid && y2 >= 0 && y2 < G && zz >= 0 && zz < G;
                const _Float16 *rowp = in + (((int64_t)zz * G + y2) * G) * 16 + half;
                h8 b0 = zero8, b1 = zero8;
                if (row_ok && xa >= 0) b0 = *reinterpret_cast<const h8 *>(rowp + (int64_t)xa * 16);
                if (row_ok && first && xb < G) b1 = *reinterpret_cast<const h8 *>(rowp + (int64_t)xb * 16);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[q * 3 + r][0], b0, acc[q], 0, 0, 0);
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[q * 3 + r][1], b1, acc[q], 0, 0, 0);
            }
        }
        if (valid) {
            const f4 s = (acc[0] + acc[1]) + acc[2];
            if (!LAST) {
                h4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (_Float16)fmaxf(s[r] + br[r], 0.f);
                *reinterpret_cast<h4 *>(out + v * 16 + 4 * kq) = o;
            } else if (kq == 0) {
                y[v] = s[0] + br[0];
            }
        }
    }
}

// Positions (consecutive voxels) that a block of the kernels that share rows takes at
// once, and the largest dilation they take.
constexpr int kQPos = 256;
constexpr int kQMaxD = 16;

// Voxel coordinates by multiplication: q = v / G for v < G^3, G <= 256, with
// magic = floor(2^32 / G) + 1.
__device__ __forceinline__ void vox_fast(int v, int G, unsigned magic, int &x, int &y, int &z) {
    const int r = (int)__umulhi((unsigned)v, magic);
    x = v - r * G;
    z = (int)__umulhi((unsigned)r, magic);
    y = r - z * G;
}

typedef unsigned u4 __attribute__((ext_vector_type(4)));
// Descriptor of an array of 'bytes' bytes: loads past it return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t nn_range(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
constexpr int kOutside = (int)0x80000000u;  // a byte offset past every array

// As k_conv16 for dilations up to kQMaxD, with a third of the loads: the three
// dx taps of a (dz, dy) row read the same input shifted along x, so the tile's
// unshifted input u is loaded once per row and multiplied by the three taps
// into three accumulators, Q_dx[u] = sum_(dy,dz) W_(dx,dy,dz) in[u + rows], and
//     out[v] = Q_-1[v - d] + Q_0[v] + Q_1[v + d]
// is put together through LDS.  k_conv16 is bound by its 18 16-byte loads per
// tile (1.0 GB through the L1 caches per 96^3 layer, 54 us); here five loads
// per tile (two rows per 16x16x32 product) serve 15 products.  A block takes
// kQPos positions, of which the outer d on each side only feed their
// neighbours.  96^3, 16 channels: 54 -> 27 us per layer (25 for the
// one-channel last one).
template <bool LAST>
__global__ __launch_bounds__(256) void k_conv16q(const _Float16 *__restrict__ in, const _Float16 *__restrict__ Wp,
                                                 const float *__restrict__ bias, _Float16 *__restrict__ out,
                                                 float *__restrict__ y, int G, unsigned magic, int d, int nrange) {
    constexpr int T = kQPos / 64;  // tiles of 16 per wavefront
    typedef typename std::conditional<LAST, float, f4>::type QT;
    constexpr int QW = LAST ? 1 : 4;  // values per position
    __shared__ QT qm[kQPos * QW], qp[kQPos * QW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int half = 8 * (kq & 1);  // this lane's eight channels of its row
    const bool first = kq < 2;      // first row of the pair (else the second)
    h8 A[3][5];
    int delta[5];  // byte offset of the lane's row of pair i
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int row = first ? 2 * i : 2 * i + 1;  // (dz + 1) * 3 + dy + 1; row 9 is empty
        const int rc = row < 9 ? row : 0;
        delta[i] = (((rc / 3 - 1) * G + rc % 3 - 1) * G * d) * 32;
#pragma unroll
        for (int x3 = 0; x3 < 3; ++x3) {
            A[x3][i] = h8{};
            if (row < 9) A[x3][i] = *reinterpret_cast<const h8 *>(Wp + ((row * 3 + x3) * 16 + j) * 16 + half);
        }
    }
    float br[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) br[r] = bias[4 * kq + r];
    const int V = G * G * G, own = kQPos - 2 * d;
    const auto rs = nn_range(in, V * 32);
    const int nb = gridDim.x, per = (nrange + nb - 1) / nb;
    const int r_lo = xcd_rank(blockIdx.x, nb) * per;
    const int r_hi = r_lo + per < nrange ? r_lo + per : nrange;
    for (int rg = r_lo; rg < r_hi; ++rg) {
        f4 q0[T];
        int xs[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int pos = (wave * T + i) * 16 + j, v = rg * own - d + pos;
            const bool valid = v >= 0 && v < V;
            int x, yy, z;
            vox_fast(valid ? v : 0, G, magic, x, yy, z);
            xs[i] = x;
            const bool vy[3] = {yy >= d, true, yy + d < G}, vz[3] = {valid && z >= d, valid, valid && z + d < G};
            h8 B[5];
#pragma unroll
            for (int p = 0; p < 5; ++p) {
                const int ra = 2 * p, rb = 2 * p + 1;  // constants
                const bool oka = vz[ra / 3] && vy[ra % 3], okb = rb < 9 && vz[rb / 3 % 3] && vy[rb % 3];
                const bool ok = first ? oka : okb;
                B[p] = __builtin_bit_cast(
                    h8, __builtin_amdgcn_raw_buffer_load_b128(rs, ok ? v * 32 + 2 * half + delta[p] : kOutside, 0, 0));
            }
            f4 acc[3];
#pragma unroll
            for (int x3 = 0; x3 < 3; ++x3) acc[x3] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < 5; ++p)
#pragma unroll
                for (int x3 = 0; x3 < 3; ++x3)
                    acc[x3] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[x3][p], B[p], acc[x3], 0, 0, 0);
            if constexpr (LAST) {
                if (kq == 0) {
                    qm[pos] = acc[0][0];
                    qp[pos] = acc[2][0];
                }
            } else {
                qm[pos * 4 + kq] = acc[0];
                qp[pos * 4 + kq] = acc[2];
            }
            q0[i] = acc[1];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int pos = (wave * T + i) * 16 + j, v = rg * own - d + pos;
            if (pos < d || pos >= kQPos - d || v >= V) continue;
            const bool lo = xs[i] >= d, hi = xs[i] + d < G;
            if constexpr (LAST) {
                if (kq == 0) y[v] = ((q0[i][0] + (lo ? qm[pos - d] : 0.f)) + (hi ? qp[pos + d] : 0.f)) + br[0];
            } else {
                const f4 m = qm[(pos - d) * 4 + kq], p = qp[(pos + d) * 4 + kq];
                h4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float sm = (q0[i][r] + (lo ? m[r] : 0.f)) + (hi ? p[r] : 0.f);
                    o[r] = (_Float16)fmaxf(sm + br[r], 0.f);
                }
                *reinterpret_cast<h4 *>(out + (int64_t)v * 16 + 4 * kq) = o;
            }
        }
        __syncthreads();  // the next range rewrites qm and qp
    }
}

// ---------------------------------------------------------------- FP32 training on the matrix cores
// Every layer trains as an implicit GEMM on gfx950's FP32 16x16x4 matrix
// product: FP32 operands, FP32 accumulation.  Activations and their
// gradients are channel-last: [V][16] for the hidden layers, [V][8] for the
// input (channels 6 and 7 zero), [V] for the one-channel output; so a lane
// fetches the channels of its products with one 8- or 16-byte load.
// Operand layout (wave of 64): A[i][k] at lane i + 16 k, B[k][j] at lane
// j + 16 k, D[i][j] at lane j + 16 (i / 4), element i % 4.  The K index of a
// product is a summation index, so lane group k may hold any channel: with
// CP stored channels, lane (j, k) of step s (NS = CP / 4 steps) takes
// channel NS k + s.  Output rows beyond a layer's channels are zero.  Work
// is split in contiguous ranges, ranked so that each of the 8 XCDs (blocks
// go round-robin to them) sweeps one contiguous eighth of the grid: the
// dilated taps then re-read planes its own L2 fetched.
typedef float f2 __attribute__((ext_vector_type(2)));
template <int N>
using fvec = typename std::conditional<N == 4, f4, typename std::conditional<N == 2, f2, float>::type>::type;

__device__ __forceinline__ float lane_elem(float v, int) { return v; }
template <typename T>
__device__ __forceinline__ float lane_elem(T v, int s) { return v[s]; }

// Planar input [6][V] -> channel-last [V][8], channels 6 and 7 zero.
__global__ void k_to_cl8(const float *x, int64_t V, float *o) {
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= V) return;
    f4 a, b;
#pragma unroll
    for (int c = 0; c < 4; ++c) a[c] = x[c * V + v];
    b[0] = x[4 * V + v];
    b[1] = x[5 * V + v];
    b[2] = 0.f;
    b[3] = 0.f;
    reinterpret_cast<f4 *>(o + v * 8)[0] = a;
    reinterpret_cast<f4 *>(o + v * 8)[1] = b;
}

// Weight operands of one layer in LDS: sA[t][lane] holds lane (j, k)'s NS
// values of tap t, W[j][NS k + s][t] (forward) or W[NS k + s][j][t] (data
// gradient, transposed); zero beyond the layer's channels.
template <int NS, bool TRANSPOSED>
__device__ __forceinline__ void stage_weights(const float *__restrict__ W, int cin, int cout, fvec<NS> (*sA)[64]) {
    for (int i = threadIdx.x; i < 27 * 64; i += blockDim.x) {
        const int t = i / 64, ln = i % 64, jj = ln & 15, k = ln >> 4;
        fvec<NS> a = {};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = NS * k + s;  // the K channel of this lane group and step
            float w = 0.f;
            if (!TRANSPOSED && jj < cout && c < cin) w = W[(jj * cin + c) * 27 + t];
            if (TRANSPOSED && c < cout && jj < cin) w = W[(c * cin + jj) * 27 + t];
            if constexpr (NS == 1) a = w;
            else a[s] = w;
        }
        sA[t][ln] = a;
    }
}

// One z plane (dz = q - 1, times SIGN) of a tile's taps: B[r * 3 + s3] holds
// lane (j, k)'s NS channels of voxel (x + SIGN d dx, y + SIGN d dy, z + SIGN
// d dz) of the channel-last array src (CP channels per voxel), zero outside
// the grid or for lane groups beyond KMAX channels.
template <int CP, int NS, int SIGN>
__device__ __forceinline__ void load_plane(const float *__restrict__ src, int x, int y, int z, bool valid, int q, int G,
                                           int d, int kq, fvec<NS> *B) {
    const int zz = z + SIGN * d * (q - 1);
    const bool zok = valid && NS * kq < CP && zz >= 0 && zz < G;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int y2 = y + SIGN * d * (r - 1);
        const bool rok = zok && y2 >= 0 && y2 < G;
        const int row = (zz * G + y2) * G;
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const int xx = x + SIGN * d * (s3 - 1);
            const bool ok = rok && xx >= 0 && xx < G;
            // branch-free: an in-bounds load, then zero where the tap leaves the grid
            // (keeps the loads in one block, so waits count only the loads needed)
            const fvec<NS> val = *reinterpret_cast<const fvec<NS> *>(src + (ok ? (int64_t)(row + xx) * CP + NS * kq : 0));
            B[r * 3 + s3] = ok ? val : fvec<NS>{};
        }
    }
}

// Forward of one layer, out[v][c] = b[c] + sum_{ci, t} W[c][ci][t] in[v + d o_t][ci]:
// per tap t, D (16 output channels x 16 consecutive voxels) += W_t (16 x CP)
// in(. + d o_t) (CP x 16), NS products of four channels.
template <int CIN, int CP, int COUT>
__global__ __launch_bounds__(256) void k_conv_fwd_mx(const float *__restrict__ in, const float *__restrict__ W,
                                                     const float *__restrict__ bias, float *__restrict__ post, int G,
                                                     int d, int relu, int ntiles) {
    constexpr int NS = CP / 4;
    typedef fvec<NS> VT;
    __shared__ VT sA[27][64];
    stage_weights<NS, false>(W, CIN, COUT, sA);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    f4 br;
#pragma unroll
    for (int r = 0; r < 4; ++r) br[r] = 4 * kq + r < COUT ? bias[4 * kq + r] : 0.f;
    const int V = G * G * G;
    const int nb = gridDim.x, per = (ntiles + nb - 1) / nb;
    const int t_lo = xcd_rank(blockIdx.x, nb) * per;
    const int t_hi = t_lo + per < ntiles ? t_lo + per : ntiles;
    int tile = t_lo + wave;
    VT Bc[9], Bn[9];
    int x = 0, y = 0, z = 0, v = 0;
    bool valid = false;
    auto coords = [&](int tl, int &cx, int &cy, int &cz, int &cv, bool &cval) {
        cv = tl * 16 + j;
        cval = cv < V;
        const int vv = cval ? cv : 0;
        cx = vv % G;
        cy = (vv / G) % G;
        cz = vv / (G * G);
    };
    if (tile < t_hi) {
        coords(tile, x, y, z, v, valid);
        load_plane<CP, NS, 1>(in, x, y, z, valid, 0, G, d, kq, Bc);
    }
    for (; tile < t_hi; tile += 4) {
        int xn = 0, yn = 0, zn = 0, vn = 0;
        bool validn = false;
        const bool more = tile + 4 < t_hi;
        if (more) coords(tile + 4, xn, yn, zn, vn, validn);
        f4 acc[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) acc[r] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            __builtin_amdgcn_sched_barrier(0);  // one plane's weight words live at a time
            if (q < 2) load_plane<CP, NS, 1>(in, x, y, z, valid, q + 1, G, d, kq, Bn);
            else if (more) load_plane<CP, NS, 1>(in, xn, yn, zn, validn, 0, G, d, kq, Bn);
#pragma unroll
            for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const VT a = sA[q * 9 + r * 3 + s3][lane];
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(lane_elem(a, s), lane_elem(Bc[r * 3 + s3], s),
                                                                      acc[r], 0, 0, 0);
                }
#pragma unroll
            for (int e = 0; e < 9; ++e) Bc[e] = Bn[e];
        }
        if (valid) {
            const f4 o = ((acc[0] + acc[1]) + acc[2]) + br;
            if constexpr (COUT == 16) {
                f4 p;
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] = relu ? fmaxf(o[r], 0.f) : o[r];
                *reinterpret_cast<f4 *>(post + (int64_t)v * 16 + 4 * kq) = p;
            } else if (kq == 0) {
                post[v] = relu ? fmaxf(o[0], 0.f) : o[0];
            }
        }
        x = xn;
        y = yn;
        z = zn;
        v = vn;
        valid = validn;
    }
}

// Data gradient between 16-channel layers, gin[v][ci] = (prev[v][ci] > 0)
// sum_{c, t} W[c][ci][t] g[v - d o_t][c], prev the activations of that layer
// (positive where its ReLU passes): per tap t, D (16 input channels x 16
// voxels) += W_t^T (16 x 16) g(. - d o_t) (16 x 16); the same plane pipeline
// as the forward.
__global__ __launch_bounds__(256) void k_conv_bwd_data_mx(const float *__restrict__ g, const float *__restrict__ W,
                                                          const float *__restrict__ prev, float *__restrict__ gin,
                                                          int G, int d, int ntiles) {
    constexpr int COUT = 16, NS = 4;
    typedef fvec<NS> VT;
    __shared__ VT sA[27][64];
    stage_weights<NS, true>(W, 16, COUT, sA);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int V = G * G * G;
    const int nb = gridDim.x, per = (ntiles + nb - 1) / nb;
    const int t_lo = xcd_rank(blockIdx.x, nb) * per;
    const int t_hi = t_lo + per < ntiles ? t_lo + per : ntiles;
    int tile = t_lo + wave;
    VT Bc[9], Bn[9];
    int x = 0, y = 0, z = 0, v = 0;
    bool valid = false;
    auto coords = [&](int tl, int &cx, int &cy, int &cz, int &cv, bool &cval) {
        cv = tl * 16 + j;
        cval = cv < V;
        const int vv = cval ? cv : 0;
        cx = vv % G;
        cy = (vv / G) % G;
        cz = vv / (G * G);
    };
    if (tile < t_hi) {
        coords(tile, x, y, z, v, valid);
        load_plane<COUT, NS, -1>(g, x, y, z, valid, 0, G, d, kq, Bc);
    }
    for (; tile < t_hi; tile += 4) {
        int xn = 0, yn = 0, zn = 0, vn = 0;
        bool validn = false;
        const bool more = tile + 4 < t_hi;
        if (more) coords(tile + 4, xn, yn, zn, vn, validn);
        f4 acc[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) acc[r] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            __builtin_amdgcn_sched_barrier(0);  // one plane's weight words live at a time
            if (q < 2) load_plane<COUT, NS, -1>(g, x, y, z, valid, q + 1, G, d, kq, Bn);
            else if (more) load_plane<COUT, NS, -1>(g, xn, yn, zn, validn, 0, G, d, kq, Bn);
#pragma unroll
            for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const VT a = sA[q * 9 + r * 3 + s3][lane];
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        acc[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(lane_elem(a, s), lane_elem(Bc[r * 3 + s3], s),
                                                                      acc[r], 0, 0, 0);
                }
#pragma unroll
            for (int e = 0; e < 9; ++e) Bc[e] = Bn[e];
        }
        if (valid) {
            const f4 o = (acc[0] + acc[1]) + acc[2];
            const f4 pp = *reinterpret_cast<const f4 *>(prev + (int64_t)v * 16 + 4 * kq);
            f4 w;
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = pp[r] > 0.f ? o[r] : 0.f;
            *reinterpret_cast<f4 *>(gin + (int64_t)v * 16 + 4 * kq) = w;
        }
        x = xn;
        y = yn;
        z = zn;
        v = vn;
        valid = validn;
    }
}

// Data gradient between 16-channel layers for dilations up to kQMaxD, with a
// third of the loads of the kernel above: as in k_conv16q the gradient of a
// (dz, dy) row is loaded once per tile and multiplied by the row's three dx taps
// into three accumulators,
//     Q_dx[u] = sum_(dy,dz) W_(dx,dy,dz)^T g[u - rows],
//     gin[v] = Q_-1[v + d] + Q_0[v] + Q_1[v - d],
// summed through LDS.  Two tiles share each weight word read from LDS (at one
// tile per word those reads alone take as long as the products).  A wavefront
// takes two pairs of tiles; the next plane's loads are in flight during a
// plane's products.  gin is zero where prev (the layer's activations) is not
// positive.
// Bound: the FP32 matrix cores, 12.2 GFLOP at 96^3 = 78 us at 157 TFLOP/s plus
// the d positions computed twice per side; 164 -> 121 us, of which an eighth is
// blocks with fewer ranges than others.
// (The forward pass of the hidden layers gains as much in this form, 168 -> 120
// and 94 -> 68 us, but it adds in another order, and a value that rounding alone
// puts on either side of its ReLU's zero then moves the gradient by 1e-6 and
// more; the forward kernel keeps its order.)
__global__ __launch_bounds__(256) void k_conv_bwd_data_q(const float *__restrict__ g, const float *__restrict__ W,
                                                         const float *__restrict__ prev, float *__restrict__ gin, int G,
                                                         unsigned magic, int d, int nrange) {
    constexpr int NS = 4;
    typedef fvec<NS> VT;
    __shared__ VT sA[27][64];
    __shared__ f4 qm[kQPos * 4], qp[kQPos * 4];
    stage_weights<NS, true>(W, 16, 16, sA);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int V = G * G * G, own = kQPos - 2 * d;
    const auto rs = nn_range(g, V * 64);
    const int nb = gridDim.x, per = (nrange + nb - 1) / nb;
    const int r_lo = xcd_rank(blockIdx.x, nb) * per;
    const int r_hi = r_lo + per < nrange ? r_lo + per : nrange;
    struct Pos {
        int v, x, y, z;
        bool valid;
    };
    auto position = [&](int rg, int i) {  // tile i of the wavefront's four
        Pos p;
        p.v = rg * own - d + (wave * 4 + i) * 16 + j;
        p.valid = p.v >= 0 && p.v < V;
        vox_fast(p.valid ? p.v : 0, G, magic, p.x, p.y, p.z);
        return p;
    };
    // the rows of plane dz = q - 1 of tile position p
    auto load = [&](const Pos &p, int q, VT *B) {
        const int dz = (1 - q) * d;
        const bool zok = p.valid && p.z + dz >= 0 && p.z + dz < G;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int dy = (1 - r) * d;
            const bool ok = zok && p.y + dy >= 0 && p.y + dy < G;
            const int off = ok ? (p.v + (dz * G + dy) * G) * 64 + kq * 16 : kOutside;
            B[r] = __builtin_bit_cast(VT, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        }
    };
    VT Bc[2][3], Bn[2][3];
    Pos pc[2];
    if (r_lo < r_hi) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pc[i] = position(r_lo, i);
            load(pc[i], 0, Bc[i]);
        }
    }
    for (int rg = r_lo; rg < r_hi; ++rg) {
        f4 q0[4];
        int xs[4];
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            Pos pn[2];
            f4 acc[2][3];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int x3 = 0; x3 < 3; ++x3) acc[i][x3] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                __builtin_amdgcn_sched_barrier(0);  // one plane's weight words live at a time
                if (q < 2) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) load(pc[i], q + 1, Bn[i]);
                } else if (pr == 0 || rg + 1 < r_hi) {  // the next pair, or the next range's first
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        pn[i] = position(pr == 0 ? rg : rg + 1, pr == 0 ? 2 + i : i);
                        load(pn[i], 0, Bn[i]);
                    }
                }
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int x3 = 0; x3 < 3; ++x3) {
                        const VT a = sA[q * 9 + r * 3 + x3][lane];
#pragma unroll
                        for (int s = 0; s < NS; ++s)  // alternating accumulators
#pragma unroll
                            for (int i = 0; i < 2; ++i)
                                acc[i][x3] = __builtin_amdgcn_mfma_f32_16x16x4f32(lane_elem(a, s), lane_elem(Bc[i][r], s),
                                                                                  acc[i][x3], 0, 0, 0);
                    }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int r = 0; r < 3; ++r) Bc[i][r] = Bn[i][r];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int pos = (wave * 4 + 2 * pr + i) * 16 + j;
                qm[pos * 4 + kq] = acc[i][0];
                qp[pos * 4 + kq] = acc[i][2];
                q0[2 * pr + i] = acc[i][1];
                xs[2 * pr + i] = pc[i].x;
                pc[i] = pn[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int pos = (wave * 4 + i) * 16 + j, v = rg * own - d + pos;
            if (pos < d || pos >= kQPos - d || v >= V) continue;
            // the term of tap dx is in range if x - dx d is
            const bool okm = xs[i] + d < G, okp = xs[i] >= d;
            const f4 m = qm[(pos + d) * 4 + kq], p = qp[(pos - d) * 4 + kq];
            const f4 pp = *reinterpret_cast<const f4 *>(prev + (int64_t)v * 16 + 4 * kq);
            f4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float sum = (q0[i][r] + (okm ? m[r] : 0.f)) + (okp ? p[r] : 0.f);
                o[r] = pp[r] > 0.f ? sum : 0.f;
            }
            *reinterpret_cast<f4 *>(gin + (int64_t)v * 16 + 4 * kq) = o;
        }
        __syncthreads();  // the next range rewrites qm and qp
    }
}

// Forward of the one-channel output layer (no ReLU), dilations up to kQMaxD:
// rows of the product are the three dx taps (three of sixteen) instead of the
// output channels (one of sixteen), so a tile takes 36 products and 9 loads
// instead of 108 and 27.  96^3: 146 -> 57 us.
__global__ __launch_bounds__(256) void k_conv_fwd_q1(const float *__restrict__ in, const float *__restrict__ W,
                                                     const float *__restrict__ bias, float *__restrict__ y, int G,
                                                     unsigned magic, int d, int nrange) {
    constexpr int T = kQPos / 64;
    __shared__ float qm[kQPos], qp[kQPos];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    f4 A[9];  // lane (dx = j, kq): W[4 kq + s][tap]
#pragma unroll
    for (int r = 0; r < 9; ++r)
#pragma unroll
        for (int s = 0; s < 4; ++s) A[r][s] = j < 3 ? W[(4 * kq + s) * 27 + r * 3 + j] : 0.f;
    const float b0 = bias[0];
    const int V = G * G * G, own = kQPos - 2 * d;
    const auto rs = nn_range(in, V * 64);
    const int nb = gridDim.x, per = (nrange + nb - 1) / nb;
    const int r_lo = xcd_rank(blockIdx.x, nb) * per;
    const int r_hi = r_lo + per < nrange ? r_lo + per : nrange;
    for (int rg = r_lo; rg < r_hi; ++rg) {
        float q0[T];
        int xs[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int pos = (wave * T + i) * 16 + j, v = rg * own - d + pos;
            const bool valid = v >= 0 && v < V;
            int x, yy, z;
            vox_fast(valid ? v : 0, G, magic, x, yy, z);
            xs[i] = x;
            const bool vy[3] = {yy >= d, true, yy + d < G}, vz[3] = {valid && z >= d, valid, valid && z + d < G};
            f4 acc[3], B[9];  // one sum per dz, alternating
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                const bool ok = vz[r / 3] && vy[r % 3];
                const int off = ok ? (v + ((r / 3 - 1) * G + r % 3 - 1) * G * d) * 64 + kq * 16 : kOutside;
                B[r] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[3 * q + r][s], B[3 * q + r][s], acc[q], 0, 0, 0);
            const f4 sm = (acc[0] + acc[1]) + acc[2];
            if (kq == 0) {
                qm[pos] = sm[0];
                qp[pos] = sm[2];
            }
            q0[i] = sm[1];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int pos = (wave * T + i) * 16 + j, v = rg * own - d + pos;
            if (kq != 0 || pos < d || pos >= kQPos - d || v >= V) continue;
            y[v] = ((q0[i] + (xs[i] >= d ? qm[pos - d] : 0.f)) + (xs[i] + d < G ? qp[pos + d] : 0.f)) + b0;
        }
        __syncthreads();
    }
}

// Data gradient of the one-channel output layer, gin[v][ci] = (prev[v][ci] > 0)
// sum_t W[ci][t] g[v - d o_t]: the contraction runs over the 27 taps (seven
// products of four taps per tile instead of 27 with one used channel each).
// Bound by the 16-channel array read and written.  96^3: 81 -> 26 us.
__global__ __launch_bounds__(256) void k_conv_bwd_data1(const float *__restrict__ g, const float *__restrict__ W,
                                                        const float *__restrict__ prev, float *__restrict__ gin, int G,
                                                        unsigned magic, int d, int ntiles) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kq = lane >> 4;
    float A[7];
    int tx[7], ty[7], tz[7];  // d o_t of the lane's tap 4 s + kq
#pragma unroll
    for (int s = 0; s < 7; ++s) {
        const int t = 4 * s + kq;
        A[s] = t < 27 ? W[j * 27 + t] : 0.f;
        tx[s] = d * (t % 3 - 1);
        ty[s] = d * (t / 3 % 3 - 1);
        tz[s] = t < 27 ? d * (t / 9 - 1) : 2 * G;  // tap 27 does not exist
    }
    const int V = G * G * G;
    const auto rs = nn_range(g, V * 4);
    const int nb = gridDim.x, per = (ntiles + nb - 1) / nb;
    const int t_lo = xcd_rank(blockIdx.x, nb) * per;
    const int t_hi = t_lo + per < ntiles ? t_lo + per : ntiles;
    for (int tile = t_lo + wave; tile < t_hi; tile += 4) {
        const int v = tile * 16 + j;
        const bool valid = v < V;
        int x, y, z;
        vox_fast(valid ? v : 0, G, magic, x, y, z);
        float B[7];
#pragma unroll
        for (int s = 0; s < 7; ++s) {
            const int xx = x - tx[s], yy = y - ty[s], zz = z - tz[s];
            const bool ok = valid && xx >= 0 && xx < G && yy >= 0 && yy < G && zz >= 0 && zz < G;
            B[s] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, ok ? ((zz * G + yy) * G + xx) * 4 : kOutside, 0, 0));
        }
        f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < 7; ++s) acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[s], B[s], acc[s & 1], 0, 0, 0);
        if (valid) {
            const f4 o = acc[0] + acc[1];
            const f4 pp = *reinterpret_cast<const f4 *>(prev + (int64_t)v * 16 + 4 * kq);
            f4 w;
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = pp[r] > 0.f ? o[r] : 0.f;
            *reinterpret_cast<f4 *>(gin + (int64_t)v * 16 + 4 * kq) = w;
        }
    }
}

// Weight and bias gradients of one 16-channel-output layer, gW[c][ci][t] =
// sum_v g[v][c] in[v + d o_t][ci].  With u = v + d dx (the tap's x offset moved
// to the gradient),
//     gW[c][ci][dz, dy, dx] = sum_u g[u - d dx][c] in[u + d (dz, dy)][ci],
// so a (dz, dy) row of the input serves its three dx taps: D (16 output
// channels x 16 input channels) += g (16 x 4 voxels) in^T (4 x 16), four voxels
// per product, one accumulator for each of the 27 taps.  A block walks slabs of
// kSlab voxels u; lane (j, k) of wave w keeps the three shifted g of voxels
// 64 k + 16 w + i (i < 16, the K index of product i) in registers for the slab.
// Row by row the slab's input (zero where the row leaves the grid) is fetched
// with coalesced 16-byte loads, one row ahead, and stored transposed in LDS,
// [ci][u] with padded rows, so that one 16-byte LDS read feeds twelve products.
// With the 8-channel input layer two rows share the sixteen columns of a
// product.  The four wavefronts' sums are added through LDS in a fixed order
// into the partial part[blockIdx.x][c][ci][28] (taps 0..26, bias in slot 27 of
// ci 0), which k_conv_w_reduce adds up in a fixed order: deterministic.
// Bound: the FP32 matrix cores (78 us at 96^3 and 16 channels).  Staging every
// tap 190 us; nine taps per block, three blocks sharing a slab, 142 us (g
// loaded three times as often, each time waited for); now
// 128 (six channels 185 -> 76); the address and LDS work issues in between the
// products, not beside them.
constexpr int kSlab = 256;

template <int CIN, int CP>
__global__ __launch_bounds__(256) void k_conv_bwd_w(const float *__restrict__ g, const float *__restrict__ in,
                                                    float *__restrict__ part, int G, unsigned magic, int d,
                                                    int nslabs) {
    constexpr int QV = CP / 4;                // 16-byte words per voxel of the input
    constexpr int NF = kSlab * QV / 256;      // of them per thread and row
    constexpr int RP = 16 / CP;               // rows sharing the columns of a product
    constexpr int NG = (9 + RP - 1) / RP;     // groups of the nine (dz, dy) rows
    constexpr int LD = kSlab + 4;             // padded row of the transposed slab
    __shared__ __align__(16) float sT[2][16 * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int V = G * G * G;
    const int ubase = 64 * kq + 16 * wave;  // this lane's product voxels: ubase + i
    const auto rg = nn_range(g, V * 64), ri = nn_range(in, V * CP * 4);
    f4 acc[NG][3];
#pragma unroll
    for (int a = 0; a < NG; ++a)
#pragma unroll
        for (int x3 = 0; x3 < 3; ++x3) acc[a][x3] = f4{0.f, 0.f, 0.f, 0.f};
    float accb = 0.f;  // bias of channel j from this lane's voxels
    const int nb = gridDim.x, per = (nslabs + nb - 1) / nb;
    const int s_lo = xcd_rank(blockIdx.x, nb) * per;
    const int s_hi = s_lo + per < nslabs ? s_lo + per : nslabs;
    for (int slab = s_lo; slab < s_hi; ++slab) {
        const int v0 = slab * kSlab;
        // staged words: f = tid + 256 i is voxel f / QV, channels 4 (f % QV) .. + 3
        int uy[NF], uz[NF];
        bool uval[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int vs = v0 + (tid + 256 * i) / QV;
            int x;
            uval[i] = vs < V;
            vox_fast(uval[i] ? vs : 0, G, magic, x, uy[i], uz[i]);
        }
        auto fetch = [&](int a, f4 (*R)[NF]) {  // the rows of group a
#pragma unroll
            for (int h = 0; h < RP; ++h) {
                const int row = a * RP + h, dz = d * (row / 3 - 1), dy = d * (row % 3 - 1);
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int yy = uy[i] + dy, zz = uz[i] + dz;
                    const bool ok = row < 9 && uval[i] && yy >= 0 && yy < G && zz >= 0 && zz < G;
                    const int off = ok ? (v0 + (dz * G + dy) * G) * (CP * 4) + 16 * (tid + 256 * i) : kOutside;
                    R[h][i] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(ri, off, 0, 0));
                }
            }
        };
        f4 R[RP][NF];
        fetch(0, R);
        float ga[3][16];
        int gx, gy, gz;  // coordinates of the lane's first product voxel
        vox_fast(v0 + ubase < V ? v0 + ubase : 0, G, magic, gx, gy, gz);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int u = v0 + ubase + i;
            int ux = gx + i;
            while (ux >= G) ux -= G;
#pragma unroll
            for (int x3 = 0; x3 < 3; ++x3) {
                const int xv = ux - d * (x3 - 1);  // x of v = u - d dx
                const bool ok = u < V && xv >= 0 && xv < G;
                ga[x3][i] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rg, ok ? (u - d * (x3 - 1)) * 64 + j * 4 : kOutside, 0, 0));
            }
            accb += ga[1][i];
        }
        __syncthreads();  // the previous slab's products have read both buffers
#pragma unroll
        for (int a = 0; a < NG; ++a) {
            float *T = sT[a & 1];
#pragma unroll
            for (int h = 0; h < RP; ++h)
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    const int f = tid + 256 * i, u = f / QV, c0 = h * CP + 4 * (f % QV);
#pragma unroll
                    for (int e = 0; e < 4; ++e) T[(c0 + e) * LD + u] = R[h][i][e];
                }
            __syncthreads();
            if (a + 1 < NG) fetch(a + 1, R);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const f4 b = *reinterpret_cast<const f4 *>(T + j * LD + ubase + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int x3 = 0; x3 < 3; ++x3)
                        acc[a][x3] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(ga[x3][4 * h + e], b[e], acc[a][x3], 0, 0, 0);
            }
        }
    }
    // block sums in a fixed order, eight accumulators at a time
    float *pb = part + (int64_t)blockIdx.x * 16 * CIN * 28;
    float *sR = &sT[0][0];  // [8][4][256]
    static_assert(2 * 16 * LD >= 8 * 4 * 256, "the sums fit the slab's buffers");
#pragma unroll
    for (int b0 = 0; b0 < NG * 3; b0 += 8) {
        __syncthreads();
#pragma unroll
        for (int b = b0; b < b0 + 8 && b < NG * 3; ++b)
            *reinterpret_cast<f4 *>(sR + ((b - b0) * 4 + wave) * 256 + lane * 4) = acc[b / 3][b % 3];
        __syncthreads();
#pragma unroll
        for (int b = b0; b < b0 + 8 && b < NG * 3; ++b) {
            const float *q = sR + (b - b0) * 1024 + tid;
            const int ln = tid >> 2, c = 4 * (ln >> 4) + (tid & 3), col = ln & 15;
            const int row = b / 3 * RP + col / CP, ci = col % CP;
            if (row < 9 && ci < CIN) pb[(c * CIN + ci) * 28 + 3 * row + b % 3] = (q[0] + q[256]) + (q[512] + q[768]);
        }
    }
    accb += __shfl_xor(accb, 16, 64);
    accb += __shfl_xor(accb, 32, 64);
    __syncthreads();
    if (kq == 0) sR[wave * 16 + j] = accb;
    __syncthreads();
    if (tid < 16) pb[(tid * CIN + 0) * 28 + 27] = (sR[tid] + sR[16 + tid]) + (sR[32 + tid] + sR[48 + tid]);
}

// Weight and bias gradients of the one-channel output layer, gW[ci][t] =
// sum_u g[u - d o_t] in[u][ci]: the rows of a product are taps (27 of two
// sixteens) instead of output channels (one of sixteen), so the 16-channel
// array is read once and not once per tap.  Sixteen voxels per step; lane (j,
// k) takes taps j and 16 + j, channel j, voxels 4 k + s.  Partials and
// reduction as above.  96^3: 146 -> 38 us.
__global__ __launch_bounds__(256) void k_conv_bwd_w1(const float *__restrict__ g, const float *__restrict__ in,
                                                     float *__restrict__ part, int G, unsigned magic, int d,
                                                     int ntiles) {
    __shared__ float sR[4][512];
    __shared__ float sB[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kq = lane >> 4;
    const int V = G * G * G;
    const auto rg = nn_range(g, V * 4), ri = nn_range(in, V * 64);
    int tx[2], ty[2], tz[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int t = 16 * h + j;
        tx[h] = d * (t % 3 - 1);
        ty[h] = d * (t / 3 % 3 - 1);
        tz[h] = t < 27 ? d * (t / 9 - 1) : 2 * G;  // no such tap
    }
    f4 acc[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    float accb = 0.f;
    const int nb = gridDim.x, per = (ntiles + nb - 1) / nb;
    const int t_lo = xcd_rank(blockIdx.x, nb) * per;
    const int t_hi = t_lo + per < ntiles ? t_lo + per : ntiles;
    for (int tile = t_lo + wave; tile < t_hi; tile += 4) {
        const int u0 = tile * 16 + 4 * kq;
        int x0, y0, z0;
        vox_fast(u0 < V ? u0 : 0, G, magic, x0, y0, z0);
        float A[2][4], B[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int u = u0 + s;
            int x = x0 + s, y = y0, z = z0;
            if (x >= G) {  // at most one row further: G >= 4
                x -= G;
                if (++y == G) {
                    y = 0;
                    ++z;
                }
            }
            const bool uok = u < V;
            B[s] = __builtin_bit_cast(float,
                                      __builtin_amdgcn_raw_buffer_load_b32(ri, uok ? u * 64 + j * 4 : kOutside, 0, 0));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int xx = x - tx[h], yy = y - ty[h], zz = z - tz[h];
                const bool ok = uok && xx >= 0 && xx < G && yy >= 0 && yy < G && zz >= 0 && zz < G;
                A[h][s] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(rg, ok ? ((zz * G + yy) * G + xx) * 4 : kOutside, 0, 0));
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[h][s], B[s], acc[h], 0, 0, 0);
            if (j == 13) accb += A[0][s];  // tap 13 is the centre: g itself
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) sR[wave][h * 256 + lane * 4 + r] = acc[h][r];
    accb += __shfl_xor(accb, 16, 64);
    accb += __shfl_xor(accb, 32, 64);
    if (lane == 13) sB[wave] = accb;
    __syncthreads();
    float *pb = part + (int64_t)blockIdx.x * 16 * 28;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int i = h * 256 + tid, ln = tid >> 2, t = 16 * h + 4 * (ln >> 4) + (tid & 3), ci = ln & 15;
        const float s = (sR[0][i] + sR[1][i]) + (sR[2][i] + sR[3][i]);
        if (t < 27) pb[ci * 28 + t] = s;
    }
    if (tid == 0) pb[27] = (sB[0] + sB[1]) + (sB[2] + sB[3]);
}

int grid1(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 65535); }

// Blocks for a sweep of n work items, about 'each' per block; above 8, a
// multiple of 8 (one equal share per XCD).  cap is a multiple of 8.
int mx_blocks(int64_t n, int64_t each, int cap) {
    int64_t b = std::max<int64_t>(1, std::min<int64_t>((n + each - 1) / each, cap));
    if (b > 8) b = (b + 7) / 8 * 8;
    return (int)b;
}

// The factor of vox_fast.
unsigned vox_magic(int G) { return (unsigned)((1ull << 32) / (unsigned)G + 1); }

// Ranges and blocks of the kernels that share rows: as many blocks as stay resident
// (two per CU for the FP32 ones; with one exchange array and three per CU
// k_conv_bwd_data_q took 126 instead of 120 us), one share of ranges each.
int q_ranges(int64_t V, int d) {
    const int own = kQPos - 2 * d;
    return (int)((V + own - 1) / own);
}

template <int CIN, int CP, int COUT>
int conv_fwd(const float *in, const float *W, const float *b, float *post, int G, int d, int relu, hipStream_t st) {
    const int64_t V = (int64_t)G * G * G;
    if (COUT == 1 && d <= kQMaxD) {
        const int nr = q_ranges(V, d);
        hipLaunchKernelGGL(k_conv_fwd_q1, dim3(mx_blocks(nr, 1, 1024)), dim3(256), 0, st, in, W, b, post, G, vox_magic(G),
                           d, nr);
    } else {  // (one output, d > kQMaxD: the halo would be too large a part of a range)
        const int ntiles = (int)((V + 15) / 16);
        hipLaunchKernelGGL((k_conv_fwd_mx<CIN, CP, COUT>), dim3(mx_blocks(ntiles, 32, 2048)), dim3(256), 0, st, in, W, b,
                           post, G, d, relu, ntiles);
    }
    BF_HIP(hipGetLastError());
    return 0;
}

int layer_fwd(bemfft_net *n, int l, const float *in, hipStream_t st) {
    const float *W = n->p + n->woff[l], *b = n->p + n->boff[l];
    float *post = n->post + (int64_t)l * n->width * n->V;
    const int relu = l < n->nl - 1;
    const int ci = n->ci[l], co = n->co[l];
    if (ci == 6 && co == 16) return conv_fwd<6, 8, 16>(in, W, b, post, n->G, n->dil[l], relu, st);
    if (ci == 16 && co == 16) return conv_fwd<16, 16, 16>(in, W, b, post, n->G, n->dil[l], relu, st);
    if (ci == 16 && co == 1) return conv_fwd<16, 16, 1>(in, W, b, post, n->G, n->dil[l], relu, st);
    set_error("network: unsupported layer shape");
    return BEMFFT_EUNSUPPORTED;
}

// x: planar [6][V]; converted to the channel-last n->xcl first
int forward(bemfft_net *n, const float *x, hipStream_t st) {
    hipLaunchKernelGGL(k_to_cl8, dim3((unsigned)((n->V + 255) / 256)), dim3(256), 0, st, x, n->V, n->xcl);
    const float *in = n->xcl;
    for (int l = 0; l < n->nl; ++l) {
        BF_CHECK(layer_fwd(n, l, in, st));
        in = n->post + (int64_t)l * n->width * n->V;
    }
    n->y = n->post + (int64_t)(n->nl - 1) * n->width * n->V;
    return 0;
}

int bwd_w(const float *g, const float *in, float *part, int cin, int cout, int G, int d, float *gW, float *gb,
          hipStream_t st) {
    const int64_t V = (int64_t)G * G * G;
    const int nslabs = (int)((V + kSlab - 1) / kSlab), ntiles = (int)((V + 15) / 16);
    const int nch = cout == 1 ? mx_blocks(ntiles, 32, kWgBlocks) : mx_blocks(nslabs, 1, kWgBlocks);
    if (cout == 1)
        hipLaunchKernelGGL(k_conv_bwd_w1, dim3(nch), dim3(256), 0, st, g, in, part, G, vox_magic(G), d, ntiles);
    else if (cin == 6)
        hipLaunchKernelGGL((k_conv_bwd_w<6, 8>), dim3(nch), dim3(256), 0, st, g, in, part, G, vox_magic(G), d, nslabs);
    else
        hipLaunchKernelGGL((k_conv_bwd_w<16, 16>), dim3(nch), dim3(256), 0, st, g, in, part, G, vox_magic(G), d,
                           nslabs);
    const int tot = cout * cin * 27 + cout;
    hipLaunchKernelGGL(k_conv_w_reduce, dim3((tot + 31) / 32), dim3(256), 0, st, part, nch, cin, cout, gW, gb);
    BF_HIP(hipGetLastError());
    return 0;
}

int bwd_d(const float *g, const float *W, const float *prev, float *gin, int cout, int G, int d, hipStream_t st) {
    const int64_t V = (int64_t)G * G * G;
    const int ntiles = (int)((V + 15) / 16), nr = d <= kQMaxD ? q_ranges(V, d) : 0;
    if (cout == 1)
        hipLaunchKernelGGL(k_conv_bwd_data1, dim3(mx_blocks(ntiles, 16, 2048)), dim3(256), 0, st, g, W, prev, gin, G,
                           vox_magic(G), d, ntiles);
    else if (d <= kQMaxD)
        hipLaunchKernelGGL(k_conv_bwd_data_q, dim3(mx_blocks(nr, 1, 512)), dim3(256), 0, st, g, W, prev, gin, G,
                           vox_magic(G), d, nr);
    else
        hipLaunchKernelGGL(k_conv_bwd_data_mx, dim3(mx_blocks(ntiles, 32, 2048)), dim3(256), 0, st, g, W, prev, gin, G,
                           d, ntiles);
    BF_HIP(hipGetLastError());
    return 0;
}

// gradients of all parameters for the loss at the given node voxels
int gradients(bemfft_net *n, const float *x, int64_t nt, const int *vox, const float *tgt, const float *wt,
              double *loss, hipStream_t st) {
    BF_CHECK(forward(n, x, st));
    float *gcur = n->ga, *gnext = n->gb;
    hipLaunchKernelGGL(k_fill, dim3(grid1(n->V)), dim3(256), 0, st, gcur, n->V, 0.f);
    const int nb = (int)((nt + 255) / 256);
    hipLaunchKernelGGL(k_nn_loss, dim3(nb), dim3(256), 0, st, n->y, vox, tgt, wt, nt, n->V, gcur, n->red);
    BF_HIP(hipGetLastError());
    std::vector<float> hred(nb);
    BF_HIP(hipMemcpyAsync(hred.data(), n->red, nb * sizeof(float), hipMemcpyDeviceToHost, st));
    for (int l = n->nl - 1; l >= 0; --l) {
        const float *in = l == 0 ? n->xcl : n->post + (int64_t)(l - 1) * n->width * n->V;
        float *gW = n->g + n->woff[l], *gb = n->g + n->boff[l];
        const int ci = n->ci[l], co = n->co[l], d = n->dil[l];
        BF_CHECK(bwd_w(gcur, in, n->part, ci, co, n->G, d, gW, gb, st));
        if (l > 0) {
            BF_CHECK(bwd_d(gcur, n->p + n->woff[l], in, gnext, co, n->G, d, st));
            std::swap(gcur, gnext);
        }
    }
    BF_HIP(hipStreamSynchronize(st));
    double L = 0.0;
    for (float v : hred) L += v;
    if (loss) *loss = L;
    return 0;
}

int input_impl(bemfft_net *n, bemfft_plan *p, const uint8_t *bc, const double *known, double s_host,
               const double *s_dev, float *x, hipStream_t st) {
    if (p->dim != 3 || p->kernel != BEMFFT_LAPLACE3D || p->n[0] != n->G || p->n[1] != n->G || p->n[2] != n->G) {
        set_error("net_input: needs a Laplace 3D plan on the network's grid");
        return BEMFFT_EINVAL;
    }
    if (p->m > n->cap) {
        BF_HIP(hipStreamSynchronize(st));
        for (double **q : {&n->dq, &n->du, &n->db}) {
            if (*q) (void)hipFree(*q);
            *q = nullptr;
        }
        n->cap = 0;
        if (hipMalloc(&n->dq, p->m * 8) != hipSuccess || hipMalloc(&n->du, p->m * 8) != hipSuccess ||
            hipMalloc(&n->db, p->m * 8) != hipSuccess) {
            set_error("net_input: allocation failed");
            return BEMFFT_ENOMEM;
        }
        n->cap = p->m;
    }
    const unsigned gm = (unsigned)((p->m + 255) / 256);
    hipLaunchKernelGGL(k_nn_split, dim3(gm), dim3(256), 0, st, bc, known, n->dq, n->du, p->m);
    BF_HIP(hipGetLastError());
    BF_CHECK(launch_apply(p, p->eng, n->dq, n->du, n->db, st));
    hipLaunchKernelGGL(k_fill, dim3(grid1(n->cin * n->V)), dim3(256), 0, st, x, n->cin * n->V, 0.f);
    hipLaunchKernelGGL(k_nn_input, dim3(gm), dim3(256), 0, st, p->d_gx, p->d_gy, p->d_gz, p->d_perm, p->d_w, p->d_nrm,
                       known, n->db, bc, p->m, n->G, 1.0 / (p->h * p->h), s_host, s_dev, x, n->V);
    BF_HIP(hipGetLastError());
    return 0;
}

// FP16 inference: x planar FP32 [6][V] -> n->y (FP32 [V])
int infer(bemfft_net *n, const float *x, hipStream_t st) {
    const int64_t V = n->V;
    hipLaunchKernelGGL(k_to_cl16, dim3((unsigned)((V + 255) / 256)), dim3(256), 0, st, x, n->cin, V, n->ha);
    hipLaunchKernelGGL(k_pack16, dim3(27, n->nl), dim3(256), 0, st, n->p, n->d_woff, n->d_boff, n->d_ci, n->d_co,
                       n->wp, n->bp);
    BF_HIP(hipGetLastError());
    const int64_t ntiles = (V + 15) / 16;
    // a multiple of 8 blocks (one share per XCD), at most 8 per CU
    const int64_t per_xcd = ((ntiles + 7) / 8 + 3) / 4;
    const unsigned blocks = 8u * (unsigned)std::max<int64_t>(1, std::min<int64_t>(per_xcd, 256));
    float *y = n->post + (int64_t)(n->nl - 1) * n->width * V;
    _Float16 *in = n->ha, *out = n->hb;
    for (int l = 0; l < n->nl; ++l) {
        const _Float16 *W = n->wp + (int64_t)l * 27 * 256;
        const float *b = n->bp + l * 16;
        const int d = n->dil[l];
        const bool last = l == n->nl - 1;
        if (d <= kQMaxD) {
            const int own = kQPos - 2 * d, nrange = (int)((V + own - 1) / own);
            // as many blocks as stay resident (3 or 4 per CU), one share of ranges each
            const dim3 grid(mx_blocks(nrange, 1, last ? 1024 : 768));
            if (last)
                hipLaunchKernelGGL(k_conv16q<true>, grid, dim3(256), 0, st, in, W, b, out, y, n->G, vox_magic(n->G), d,
                                   nrange);
            else
                hipLaunchKernelGGL(k_conv16q<false>, grid, dim3(256), 0, st, in, W, b, out, y, n->G, vox_magic(n->G), d,
                                   nrange);
        } else if (last) {
            hipLaunchKernelGGL(k_conv16<true>, dim3(blocks), dim3(256), 0, st, in, W, b, out, y, n->G, d, ntiles);
        } else {
            hipLaunchKernelGGL(k_conv16<false>, dim3(blocks), dim3(256), 0, st, in, W, b, out, y, n->G, d, ntiles);
        }
        BF_HIP(hipGetLastError());
        std::swap(in, out);
    }
    n->y = y;
    return 0;
}

}  // namespace
}  // namespace bemfft

using namespace bemfft;

extern "C" {

int bemfft_net_create(bemfft_net **out, int grid, int width, int nlayers, const int *dilations, uint64_t seed,
                      void *stream) {
    (void)stream;
    if (!out || grid < 4 || grid > 256 || width != 16 || nlayers < 2 || nlayers > 8 || !dilations) {
        set_error("net_create: grid in [4, 256], width 16, 2..8 layers, dilations required");
        return BEMFFT_EINVAL;
    }
    *out = nullptr;
    bemfft_net *n = new (std::nothrow) bemfft_net();
    if (!n) return BEMFFT_ENOMEM;
    n->G = grid;
    n->cin = 6;
    n->width = width;
    n->nl = nlayers;
    n->V = (int64_t)grid * grid * grid;
    for (int l = 0; l < nlayers; ++l) {
        if (dilations[l] < 1 || dilations[l] > grid) {
            delete n;
            set_error("net_create: bad dilation");
            return BEMFFT_EINVAL;
        }
        n->dil.push_back(dilations[l]);
        n->ci.push_back(l == 0 ? n->cin : width);
        n->co.push_back(l == nlayers - 1 ? 1 : width);
    }
    std::vector<float> hp;
    std::mt19937_64 rng(seed);
    std::normal_distribution<double> nd(0.0, 1.0);
    for (int l = 0; l < nlayers; ++l) {
        n->woff.push_back((int64_t)hp.size());
        const int fan = n->ci[l] * 27;
        const double sd = std::sqrt(2.0 / fan) * (l == nlayers - 1 ? 0.1 : 1.0);
        for (int i = 0; i < n->co[l] * fan; ++i) hp.push_back((float)(sd * nd(rng)));
        n->boff.push_back((int64_t)hp.size());
        for (int i = 0; i < n->co[l]; ++i) hp.push_back(0.f);
    }
    n->nparam = (int64_t)hp.size();
    const int nch = kWgBlocks;
    const size_t act = (size_t)nlayers * width * n->V * sizeof(float);
    if (hipMalloc(&n->p, n->nparam * 4) != hipSuccess || hipMalloc(&n->g, n->nparam * 4) != hipSuccess ||
        hipMalloc(&n->m, n->nparam * 4) != hipSuccess || hipMalloc(&n->v, n->nparam * 4) != hipSuccess ||
        hipMalloc(&n->post, act) != hipSuccess ||
        hipMalloc(&n->xcl, (size_t)8 * n->V * 4) != hipSuccess ||
        hipMalloc(&n->ga, (size_t)width * n->V * 4) != hipSuccess ||
        hipMalloc(&n->gb, (size_t)width * n->V * 4) != hipSuccess ||
        hipMalloc(&n->part, (size_t)nch * width * width * 28 * 4) != hipSuccess ||
        hipMalloc(&n->red, (size_t)65536 * 4) != hipSuccess ||
        hipMalloc(&n->ha, (size_t)n->V * 16 * 2) != hipSuccess || hipMalloc(&n->hb, (size_t)n->V * 16 * 2) != hipSuccess ||
        hipMalloc(&n->wp, (size_t)nlayers * 27 * 256 * 2) != hipSuccess ||
        hipMalloc(&n->bp, (size_t)nlayers * 16 * 4) != hipSuccess || hipMalloc(&n->sdev, 8) != hipSuccess ||
        hipMalloc(&n->d_woff, nlayers * 8) != hipSuccess || hipMalloc(&n->d_boff, nlayers * 8) != hipSuccess ||
        hipMalloc(&n->d_ci, nlayers * 4) != hipSuccess || hipMalloc(&n->d_co, nlayers * 4) != hipSuccess ||
        hipMemcpy(n->d_woff, n->woff.data(), nlayers * 8, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(n->d_boff, n->boff.data(), nlayers * 8, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(n->d_ci, n->ci.data(), nlayers * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(n->d_co, n->co.data(), nlayers * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(n->p, hp.data(), n->nparam * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(n->m, 0, n->nparam * 4) != hipSuccess || hipMemset(n->v, 0, n->nparam * 4) != hipSuccess) {
        bemfft_net_destroy(n);
        set_error("net_create: allocation failed");
        return BEMFFT_ENOMEM;
    }
    *out = n;
    return 0;
}

int bemfft_net_destroy(bemfft_net *n) {
    if (!n) return 0;
    for (float *q : {n->p, n->g, n->m, n->v, n->xcl, n->post, n->ga, n->gb, n->part, n->red})
        if (q) (void)hipFree(q);
    for (double *q : {n->dq, n->du, n->db, n->sdev})
        if (q) (void)hipFree(q);
    for (void *q : {(void *)n->ha, (void *)n->hb, (void *)n->wp, (void *)n->bp, (void *)n->d_woff, (void *)n->d_boff,
                    (void *)n->d_ci, (void *)n->d_co})
        if (q) (void)hipFree(q);
    delete n;
    return 0;
}

int64_t bemfft_net_num_params(const bemfft_net *n) { return n ? n->nparam : 0; }

int bemfft_net_get_params(const bemfft_net *n, float *host) {
    if (!n || !host) return BEMFFT_EINVAL;
    BF_HIP(hipMemcpy(host, n->p, n->nparam * 4, hipMemcpyDeviceToHost));
    return 0;
}

int bemfft_net_set_params(bemfft_net *n, const float *host) {
    if (!n || !host) return BEMFFT_EINVAL;
    BF_HIP(hipMemcpy(n->p, host, n->nparam * 4, hipMemcpyHostToDevice));
    return 0;
}

int bemfft_net_input(bemfft_net *n, bemfft_plan *p, const uint8_t *bc, const double *known, double scale, float *x,
                     void *stream) {
    if (!n || !p || !known || !x) {
        set_error("net_input: null argument");
        return BEMFFT_EINVAL;
    }
    return input_impl(n, p, bc, known, scale, nullptr, x, (hipStream_t)stream);
}

int bemfft_net_forward(bemfft_net *n, const float *x, float *y, void *stream) {
    if (!n || !x || !y) return BEMFFT_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    BF_CHECK(forward(n, x, st));
    BF_HIP(hipMemcpyAsync(y, n->y, n->V * 4, hipMemcpyDeviceToDevice, st));
    return 0;
}

int bemfft_net_infer(bemfft_net *n, const float *x, float *y, void *stream) {
    if (!n || !x || !y) return BEMFFT_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    BF_CHECK(infer(n, x, st));
    BF_HIP(hipMemcpyAsync(y, n->y, n->V * 4, hipMemcpyDeviceToDevice, st));
    return 0;
}

int bemfft_net_gradients(bemfft_net *n, const float *x, int64_t nt, const int *vox, const float *tgt, const float *wt,
                         double *loss, float *grad_host, void *stream) {
    if (!n || !x || nt < 1 || nt > kMaxTargets || !vox || !tgt || !wt) {
        set_error("net_gradients: null argument or target count outside [1, 2^24]");
        return BEMFFT_EINVAL;
    }
    BF_CHECK(gradients(n, x, nt, vox, tgt, wt, loss, (hipStream_t)stream));
    if (grad_host) BF_HIP(hipMemcpy(grad_host, n->g, n->nparam * 4, hipMemcpyDeviceToHost));
    return 0;
}

int bemfft_net_train_step(bemfft_net *n, const float *x, int64_t nt, const int *vox, const float *tgt, const float *wt,
                          float lr, double *loss, void *stream) {
    if (!n || !x || nt < 1 || nt > kMaxTargets || !vox || !tgt || !wt || !(lr > 0.f)) {
        set_error("net_train_step: null argument, target count outside [1, 2^24] or lr <= 0");
        return BEMFFT_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    BF_CHECK(gradients(n, x, nt, vox, tgt, wt, loss, st));
    n->t += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - (float)std::pow(b1, (double)n->t), c2 = 1.f - (float)std::pow(b2, (double)n->t);
    hipLaunchKernelGGL(k_adam, dim3(grid1(n->nparam)), dim3(256), 0, st, n->p, n->g, n->m, n->v, n->nparam, lr, b1, b2,
                       c1, c2, 1e-8f);
    BF_HIP(hipGetLastError());
    return 0;
}

int bemfft_net_guess(bemfft_net *n, bemfft_plan *p, const uint8_t *bc, const double *known, float *xbuf,
                     double *x0, void *stream) {
    if (!n || !p || !known || !xbuf || !x0) return BEMFFT_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(k_nn_scale, dim3(1), dim3(1024), 0, st, known, bc, p->m, n->sdev);
    BF_HIP(hipGetLastError());
    BF_CHECK(input_impl(n, p, bc, known, 1.0, n->sdev, xbuf, st));
    BF_CHECK(infer(n, xbuf, st));
    hipLaunchKernelGGL(k_nn_gather, dim3((unsigned)((p->m + 255) / 256)), dim3(256), 0, st, n->y, p->d_gx, p->d_gy,
                       p->d_gz, p->d_perm, bc, p->m, n->G, n->sdev, p->h, x0);
    BF_HIP(hipGetLastError());
    return 0;
}

// Node voxel index and weight of each node in the caller's order (for the
// training targets).
int bemfft_plan_node_voxels(const bemfft_plan *p, int *vox_host, double *w_host) {
    if (!p) return BEMFFT_EINVAL;
    const int64_t m = p->m;
    std::vector<int> gx(m), gy(m), gz(m), perm(m);
    std::vector<double> w(m);
    BF_HIP(hipMemcpy(gx.data(), p->d_gx, m * 4, hipMemcpyDeviceToHost));
    BF_HIP(hipMemcpy(gy.data(), p->d_gy, m * 4, hipMemcpyDeviceToHost));
    BF_HIP(hipMemcpy(gz.data(), p->d_gz, m * 4, hipMemcpyDeviceToHost));
    BF_HIP(hipMemcpy(perm.data(), p->d_perm, m * 4, hipMemcpyDeviceToHost));
    BF_HIP(hipMemcpy(w.data(), p->d_w, m * 8, hipMemcpyDeviceToHost));
    for (int64_t k = 0; k < m; ++k) {
        const int j = perm[k];
        if (vox_host) vox_host[j] = (int)(((int64_t)gz[k] * p->n[1] + gy[k]) * p->n[0] + gx[k]);
        if (w_host) w_host[j] = w[k];
    }
    return 0;
}

}  // extern "C"
