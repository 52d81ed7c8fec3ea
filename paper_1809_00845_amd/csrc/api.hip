// api.hip -- plan creation, the apply entry point and error reporting.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "volume_impl.hpp"
#include "fft_device.hpp"
#include "internal.hpp"
#include "kinds.hpp"

namespace bemfft {

namespace {
thread_local std::string g_last_error;
constexpr double kPi = 3.141592653589793238462643383279502884;
const int64_t kSizes[] = {32, 64, 96, 128, 192, 256, 320, 384, 512, 1024};  // 1024: 2D only
// A grid row holding this many nodes is x-transformed by FFT.
constexpr int kDenseRow = 24;
// 2D plans whose fields are not folded (fold_rule) transform shorter rows so: the
// sums of k_mid2d take each row in one thread and grow with the busiest, the row FFTs
// of k_fields_rows do not.  512^2 grids with 10, 16 and 23 nodes in each row, us an
// apply with the limit at 24 and 8: Laplace FP64 53, 92, 126 and 41, FP32 33, 53, 87
// and 28, half-space FP32 45, 67, 102 and 35; 256^2, 10 and 23 nodes, 22, 36 and 18 in
// FP64.  Rows of 6 are faster summed: 34.3 and, with the limit at 6, 40.8.
constexpr int kDenseRow2d = 8;
// Where eight lanes per node leave a 2D plan's chip idle, k_gather_wide sums a row
// in one round (one output up to this many nodes, three up to twice as many): rows of
// 0 to 23 nodes, us with it and without, Laplace 2997 nodes 20.1 and 20.3, 3967
// 35.9 and 35.8, 6008 49.1 and 47.0; half-space 3967 55.7 and 63.7, 6008 74.8 and 83.0.
constexpr int kWideNodes = 4096;
// When no other row holds more than this many nodes, the forward direct DFT
// takes two kx per thread (each node load serves both; measured on the
// 128^3 cube: 42 -> 38 us).  Plans with busier short rows keep one kx per
// thread, whose work per thread is then balanced better (the sphere).  3D plans;
// a 2D plan's block has one kx.
constexpr int kFewNodesRow = 4;
// The long rows' inverse x transform goes through a row FFT (one more launch,
// a few microseconds) when the per-node sums it replaces exceed this many
// complex products: the nodes of long rows x Hx x outputs.  Measured: the
// 128^3 cube (3e6) is faster without it, the 256^2 half-space surface (5e7)
// was 1.4x faster with it (2D plans whose nodes all lie in long rows now always
// take a row FFT, k_rows_gather).
constexpr double kRowInvWork = 8.0e6;

template <typename T>
int dev_upload(T **dst, const std::vector<T> &src) {
    *dst = nullptr;
    if (src.empty()) return 0;
    if (hipMalloc(dst, src.size() * sizeof(T)) != hipSuccess) {
        set_error("hipMalloc failed");
        return BEMFFT_ENOMEM;
    }
    BF_HIP(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
    return 0;
}

void dev_free(void *p) {
    if (p) (void)hipFree(p);
}

// Flat-panel self integrals of the single-layer kernel over a node's own
// measure w (straight segment in 2D, square in 3D), and the grid value at
// offset 0 (the same integral for the reference measure h^(d-1), per unit
// measure; Navier: orientation averaged).  O x O blocks, row-major.
void self_blocks(int kernel, double w, const double n[3], double h, double nu, double mu, double *self,
                 double *k0w) {
    const double l = std::log(1.0 + std::sqrt(2.0));
    if (kernel == BEMFFT_LAPLACE2D) {
        self[0] = w * (1.0 - std::log(0.5 * w)) / (2.0 * kPi);
        k0w[0] = w * (1.0 - std::log(0.5 * h)) / (2.0 * kPi);
        return;
    }
    if (kernel == BEMFFT_LAPLACE3D) {
        self[0] = std::sqrt(w) * l / kPi;
        k0w[0] = w * l / (kPi * h);
        return;
    }
    if (kernel == BEMFFT_HALFSPACE) {
        // the apply is r = K[sigma] - u, i.e. "S" = -K: blocks of -K over the
        // node's own square of area w (int 1/r = 4 s ln(1 + sqrt 2) for side s,
        // int x^2/r^3 = half of it) and over the reference cell h x h
        const double g = 1.0 / (2.0 * kPi * mu);
        const double a = 4.0 * std::sqrt(w) * l * g, aref = 4.0 * l / h * w * g;
        const double dg[3] = {1.0 - 0.5 * nu, 1.0 - 0.5 * nu, 1.0 - nu};
        for (int i = 0; i < 9; ++i) self[i] = k0w[i] = 0.0;
        for (int k = 0; k < 3; ++k) {
            self[4 * k] = -a * dg[k];
            k0w[4 * k] = -aref * dg[k];
        }
        return;
    }
    const double pre = 1.0 / (16.0 * kPi * mu * (1.0 - nu));
    const double i1 = 4.0 * std::sqrt(w) * l;
    const double i1ref = 4.0 * l / h;  // per unit measure
    for (int k = 0; k < 3; ++k)
        for (int j = 0; j < 3; ++j) {
            const double d = (k == j) ? 1.0 : 0.0;
            self[3 * k + j] = pre * i1 * ((3.0 - 4.0 * nu) * d + 0.5 * (d - n[k] * n[j]));
            k0w[3 * k + j] = pre * i1ref * w * ((3.0 - 4.0 * nu) + 1.0 / 3.0) * d;
        }
}

template <typename R>
std::vector<cx<R>> twiddle_table(int64_t p) {
    std::vector<cx<R>> t(p);
    for (int64_t i = 0; i < p; ++i) {
        ctrig::CS w = ctrig::cs2pi(i, p);
        t[i] = {(R)w.c, (R)(-w.s)};
    }
    return t;
}

// Smallest supported length of at least len.
int64_t auto_pad_len(int64_t len) {
    for (int64_t s : kSizes)
        if (s >= len) return s;
    return -1;
}
int64_t auto_pad(int64_t n) { return auto_pad_len(2 * n); }

}  // namespace

void set_error(const std::string &msg) { g_last_error = msg; }

void free_engine(Engine *e) {
    dev_free(e->spec);
    dev_free(e->twx);
    dev_free(e->twy);
    dev_free(e->twz);
    dev_free(e->Y);
    dev_free(e->Z);
    dev_free(e->vf);
    dev_free(e->Xd);
    *e = Engine{};
}

template <typename R>
static int upload_tw(Engine *e, const bemfft_plan *p) {
    cx<R> *d = nullptr;
    BF_CHECK(dev_upload(&d, twiddle_table<R>(p->P[0])));
    e->twx = d;
    BF_CHECK(dev_upload(&d, twiddle_table<R>(p->P[1])));
    e->twy = d;
    BF_CHECK(dev_upload(&d, twiddle_table<R>(p->P[2])));
    e->twz = d;
    return 0;
}

int upload_twiddles(Engine *e, const bemfft_plan *p) {
    return e->precision == BEMFFT_FP64 ? upload_tw<double>(e, p) : upload_tw<float>(e, p);
}

// Schedule of the z pass without autotuning: the fastest at each padded length
// pz, from z-pass times measured on MI355X (us, every plane of the half pencil
// occupied; hx x py pencils 129 x 256 unless given; schedules 0, 1, 2).
//   Laplace FP32: 0 -- 96: 26, 28; 128: 26, 29; 192: 38, 43; 256: 43, 49;
//     320: 78, 86; 384: 96, 100; 512: 128, 127.
//   Laplace FP64: 1 at 128, 384 and 512 -- 96: 40, 42; 128: 47, 43; 192: 76, 91;
//     256: 115, 115; 320: 197, 204; 384: 371, 192; 512: 252, 246.
//   Navier FP32: 0 below 320 -- 96: 67, 74; 128: 74, 82; 192: 136, 148; 256: 188,
//     193, 195 -- and 1 from there (129 x 128) -- 320: 218, 166; 384: 166, 159,
//     158; 512: 237, 201, 201.  Schedule 0 of 128 and 256 points puts eight pencils
//     in a wavefront, 1 four: with few pencils the chip needs the wavefronts (256
//     points, 33 x 64: 31, 27; 129 x 64: 62, 52; 129 x 128: 98, 98.  128 points, 33
//     x 64: 25, 18; 129 x 128: 49, 46).
//   Navier FP64 -- 96: 177, 190; 128: 651, 180; 192: 327, 302; 256: schedule 1
//     (narrower tiles, z_tile_log2) unless the pencils are many and long rows lie
//     beside short ones;
//     384 (129 x 128): 353, 354, 383, but 1467, 1484, 1459 for the 180-plane cube
//     of 192^3 (193 x 384); 512: 1351, 1348, 402.
// 64 points, Navier at 32 and Navier FP64 at 320 have one schedule; Laplace at 32
// has its own for large planes (zsched.hpp).
static int default_zsched(const bemfft_plan *p, bool fp64) {
    const int kernel = p->kernel;
    const int64_t pz = p->P[2], hx = p->H[0], py = p->P[1];
    if (kernel != BEMFFT_NAVIER3D) return fp64 && (pz == 128 || pz == 384 || pz == 512) ? 1 : 0;
    const bool few = hx * py <= 129 * 128;
    if (!fp64) return pz >= 320 || ((pz == 128 || pz == 256) && few) ? 1 : 0;
    if (pz == 512 || (pz == 384 && !few)) return 2;
    return pz == 128 || pz == 192 || (pz == 256 && (few || !p->mixed_rows)) ? 1 : 0;
}

int alloc_workspace(bemfft_plan *p, Engine *e) {
    BF_CHECK(alloc_intermediates(p, e->precision, e));
    e->zsched = default_zsched(p, e->precision == BEMFFT_FP64);
    // 16-bit spectra: kz rows padded to a multiple of 8 values (16-byte runs)
    e->hzs = e->precision == BEMFFT_BF16_MFMA ? (p->H[2] + 7) / 8 * 8 : spec_row(z_split(p->kernel, e->precision == BEMFFT_FP64, p->P[2]), (int)p->H[2]);
    const size_t spec = (size_t)p->K * p->H[0] * p->H[1] * e->hzs * e->sreal;
    if (hipMalloc(&e->spec, spec) != hipSuccess) {
        set_error("hipMalloc of the spectra failed");
        return BEMFFT_ENOMEM;
    }
    e->bytes += spec;
    return 0;
}

void fill_apply_args(const bemfft_plan *p, const Engine &e, const Engine &ws, ApplyArgs *out) {
    ApplyArgs a{};
    a.nx = (int)p->n[0];
    a.ny = (int)p->n[1];
    a.nz = (int)p->n[2];
    a.px = (int)p->P[0];
    a.py = (int)p->P[1];
    a.pz = (int)p->P[2];
    a.hx = (int)p->H[0];
    a.hy = (int)p->H[1];
    a.hz = (int)p->H[2];
    a.hzs = (int)e.hzs;
    a.z0 = (int)p->z0;
    a.nzo = (int)p->nzo;
    a.m = (int)p->m;
    a.gx = p->d_gx;
    a.gy = p->d_gy;
    a.gz = p->d_gz;
    a.rowptr = p->d_rowptr;
    a.perm = p->d_perm;
    a.w = p->d_w;
    a.nrm = p->d_nrm;
    a.C = p->d_C;
    a.SC = p->d_SC;
    a.spec = e.spec;
    a.twx = e.twx;
    a.twy = e.twy;
    a.twz = e.twz;
    a.Y = ws.Y;
    a.Z = ws.Z;
    a.vf = ws.vf;
    a.Xd = ws.Xd;
    a.row_dense = p->d_row_dense;
    a.dense_rows = p->d_dense_rows;
    a.nd = (int)p->nd;
    a.row_inv = p->row_inv;
    a.flat = p->flat;
    a.fwd_xg = p->fwd_xg;
    a.zsched = e.zsched;
    a.off = 0;
    a.gid = 0;
    *out = a;
}

int alloc_intermediates(const bemfft_plan *p, int precision, Engine *e) {
    e->precision = precision;
    e->creal = precision == BEMFFT_FP64 ? 8 : 4;
    e->sreal = precision == BEMFFT_FP64 ? 8 : (precision == BEMFFT_FP32 ? 4 : 2);
    const size_t cb = 2 * e->creal, sb = 2 * e->sreal;
    const size_t rows = (size_t)p->H[0] * p->nzo * p->P[1];
    // Y also holds the inverse y pass's rows in the arithmetic precision:
    // O nzo ny Hx complex values, never more than F Hx nzo Py stored ones
    // (2D plans keep what comes before those in LDS)
    const bool flat = p->dim == 2;
    const size_t ysz = std::max(flat ? 0 : (size_t)p->F * rows * sb, (size_t)p->O * p->nzo * p->n[1] * p->H[0] * cb);
    const size_t zsz = flat ? 0 : (size_t)p->O * rows * sb;
    const size_t vsz = (size_t)p->F * p->m * e->creal;
    const size_t xsz = std::max<size_t>(1, (size_t)p->nd * p->F * p->H[0] * cb);
    if (hipMalloc(&e->Y, ysz) != hipSuccess || (zsz > 0 && hipMalloc(&e->Z, zsz) != hipSuccess) ||
        hipMalloc(&e->vf, vsz) != hipSuccess || hipMalloc(&e->Xd, xsz) != hipSuccess) {
        set_error("hipMalloc of the intermediates failed");
        return BEMFFT_ENOMEM;
    }
    e->bytes = ysz + zsz + vsz + xsz;
    return 0;
}

int launch_apply(bemfft_plan *p, const Engine &e, const double *q, const double *u, double *r, hipStream_t st,
                 hipEvent_t *ev) {
    ApplyArgs a;
    fill_apply_args(p, e, e, &a);
    a.q = q;
    a.u = u;
    a.r = r;
    if (p->kernel == 0) return apply_kind<0>(e.precision, a, st, ev);
    if (p->kernel == 1) return apply_kind<1>(e.precision, a, st, ev);
    if (p->kernel == 3) return apply_kind<3>(e.precision, a, st, ev);
    return apply_kind<2>(e.precision, a, st, ev);
}

}  // namespace bemfft

using namespace bemfft;

namespace {

void destroy_plan_state(bemfft_plan *p) {
    free_engine(&p->eng);
    free_engine(&p->eng64);
    dev_free(p->d_gx);
    dev_free(p->d_gy);
    dev_free(p->d_gz);
    dev_free(p->d_perm);
    dev_free(p->d_rowptr);
    dev_free(p->d_w);
    dev_free(p->d_nrm);
    dev_free(p->d_C);
    dev_free(p->d_SC);
    dev_free(p->d_row_dense);
    dev_free(p->d_dense_rows);
    dev_free(p->s_V);
    dev_free(p->s_vec);
    dev_free(p->s_red);
    dev_free(p->s_hbuf);
    if (p->h_pinned) (void)hipHostFree(p->h_pinned);
}

// Implicit free term: c_j = -D[1]_j (Laplace), C_j = -[D e_1, D e_2, D e_3]_j
// (Navier), from the FP64 operator with c = 0 and q = 0.
int implicit_free_term(bemfft_plan *p, const Engine &e64, hipStream_t st, std::vector<double> &Cs) {
    const int64_t m = p->m;
    const int nc = p->ncomp;
    double *q = nullptr, *u = nullptr, *r = nullptr;
    const size_t bytes = (size_t)nc * m * sizeof(double);
    if (hipMalloc(&q, bytes) != hipSuccess || hipMalloc(&u, bytes) != hipSuccess || hipMalloc(&r, bytes) != hipSuccess) {
        dev_free(q);
        dev_free(u);
        dev_free(r);
        set_error("hipMalloc failed");
        return BEMFFT_ENOMEM;
    }
    std::vector<int> perm(m);
    int status = 0;
    std::vector<double> hu((size_t)nc * m), hr((size_t)nc * m);
    Cs.assign((size_t)m * nc * nc, 0.0);
    if (hipMemcpy(perm.data(), p->d_perm, m * sizeof(int), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemsetAsync(q, 0, bytes, st) != hipSuccess)
        status = BEMFFT_EDEVICE;
    for (int l = 0; l < nc && status == 0; ++l) {
        std::fill(hu.begin(), hu.end(), 0.0);
        std::fill(hu.begin() + (size_t)l * m, hu.begin() + (size_t)(l + 1) * m, 1.0);
        if (hipMemcpyAsync(u, hu.data(), bytes, hipMemcpyHostToDevice, st) != hipSuccess) { status = BEMFFT_EDEVICE; break; }
        status = launch_apply(p, e64, q, u, r, st);
        if (status) break;
        if (hipMemcpyAsync(hr.data(), r, bytes, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) { status = BEMFFT_EDEVICE; break; }
        for (int64_t s = 0; s < m; ++s)
            for (int k = 0; k < nc; ++k) Cs[((size_t)s * nc + k) * nc + l] = -hr[(size_t)k * m + perm[s]];
    }
    dev_free(q);
    dev_free(u);
    dev_free(r);
    if (status == BEMFFT_EDEVICE) set_error("implicit free term: HIP failure");
    return status;
}

int autotune_zsched(bemfft_plan *p, hipStream_t st);
int num_zsched(const bemfft_plan *p);

// 2D: the fields are folded into k_mid2d (which saves the launch before it, 3 us,
// but has every block fetch every node from q and u) where that is faster: few long
// rows, which a wavefront sums one after the other, and either a short transform, whose
// blocks leave CUs idle, or few nodes, in rows that are fetched in one round.
// Measured (us an apply, folded and not): long rows beside two nodes per row on 128^2,
// 1, 3, 5, 8 of them: 11.5, 13.0, 14.8, 17.3 and 14.3; on 512^2 23.8, 26.0, 28.0, 31.4
// and 27.0.  128^2, 13 and 16 nodes in each row (1,728, 2,112 nodes): 13.5, 15.6 and
// 14.3, 14.0.  190^2, 6 and 8 per row 15.9, 17.7 and 17.0, 20.5.  256^2, 4 and 6 per row: 15.4, 17.3 and 15.6, 16.6; 512^2, 2 and 2 to 3
// per row: 21.8, 26.3 and 22.0, 24.7, the square's sides (1,020 nodes beside two long
// rows) 24.7 and 27.2.  A circle, whose top and bottom rows hold 8 to 40 nodes:
// 128^2 12.3 and 14.2, 256^2 20.4 and 17.7, 512^2 32.6 and 29.0.
constexpr int kFoldRows = 3, kFoldNodes = 1792, kFoldLight = 1152, kFoldAll = 4096;

bool fold_rule(const bemfft_plan *p, const std::vector<int> &rowptr) {
    int64_t long_rows = 0, heavy = 0, light = 0, busiest = 0;  // light: nodes of the rows that are not heavy
    for (size_t r = 0; r + 1 < rowptr.size(); ++r) {
        const int64_t c = rowptr[r + 1] - rowptr[r];
        long_rows += c >= kDenseRow;
        if (c >= kDenseRow2d) {
            ++heavy;
        } else {
            light += c;
            busiest = std::max(busiest, c);
        }
    }
    if (long_rows > kFoldRows || p->m > kFoldAll) return false;
    if (p->H[0] < 256 && p->m <= kFoldNodes) return true;
    // with 1024 points along y a thread has two rows and fetches two nodes of each at once
    return heavy <= kFoldRows && light <= kFoldLight && busiest <= (p->P[1] > 512 ? 2 : kDenseRow2d - 1);
}

int plan_create_impl(bemfft_plan *p, const bemfft_grid *grid, int64_t m, const double *nodes,
                     const double *normals, const double *weights, int kernel, double nu, double mu,
                     const bemfft_plan_opts *opts) {
    auto t0 = std::chrono::steady_clock::now();
    if (kernel < 0 || kernel > 3) { set_error("unknown kernel"); return BEMFFT_EINVAL; }
    const bool halfspace = kernel == BEMFFT_HALFSPACE;
    KindInfo ki = kind_info(kernel);
    if (grid->dim != ki.dim) { set_error("grid dimension does not match the kernel"); return BEMFFT_EINVAL; }
    // kernels index the [F][m] field and [O][m] node arrays with 32-bit products
    // (f * m + s, with F up to 9), and the plan sorts with 32-bit node indices
    const int64_t m_max = (int64_t)INT32_MAX / std::max(ki.F, 3);
    if (m < 1 || m > m_max) {
        set_error("node count out of range [1, " + std::to_string(m_max) + "]");
        return BEMFFT_EINVAL;
    }
    if (!nodes || (!normals && !halfspace)) { set_error("nodes and normals are required"); return BEMFFT_EINVAL; }
    if (!(grid->h > 0.0) || !std::isfinite(grid->h)) { set_error("grid spacing must be positive"); return BEMFFT_EINVAL; }
    if ((kernel == BEMFFT_NAVIER3D || halfspace) && (!(nu > -1.0 && nu < 0.5) || !(mu > 0.0))) {
        set_error("elasticity needs nu in (-1, 1/2) and mu > 0");
        return BEMFFT_EINVAL;
    }
    const int prec = opts ? (int)opts->precision : BEMFFT_FP64;
    const int cmode = opts ? (int)opts->c_mode : BEMFFT_C_IMPLICIT;
    if (prec != BEMFFT_FP64 && prec != BEMFFT_FP32 && prec != BEMFFT_BF16_MFMA) {
        set_error("unknown precision");
        return BEMFFT_EINVAL;
    }
    if (prec == BEMFFT_BF16_MFMA && ki.dim != 3) {
        set_error("the 16-bit form runs the z transforms on the matrix cores: 3D plans only");
        return BEMFFT_EINVAL;
    }
    if (cmode < 0 || cmode > 2) { set_error("unknown c_mode"); return BEMFFT_EINVAL; }
    if (cmode == BEMFFT_C_USER && !(opts && opts->c_user)) { set_error("C_USER needs c_user"); return BEMFFT_EINVAL; }
    if (opts && (opts->autotune < 0 || opts->autotune > 4)) { set_error("autotune must be in [0, 4]"); return BEMFFT_EINVAL; }
    const int cell_quad = opts ? opts->cell_quad : 0;
    if (cell_quad < 0 || cell_quad > 8) { set_error("cell_quad must be in [0, 8]"); return BEMFFT_EINVAL; }
    hipStream_t st = opts ? (hipStream_t)opts->stream : nullptr;
    const int d = ki.dim;
    p->dim = d;
    p->kernel = kernel;
    p->cmode = cmode;
    p->ncomp = ki.ncomp;
    p->F = ki.F;
    p->K = ki.K;
    p->O = ki.O;
    p->m = m;
    p->h = grid->h;
    p->nu = nu;
    p->mu = mu;
    p->cell_quad = cell_quad;
    for (int a = 0; a < 3; ++a) {
        p->origin[a] = a < d ? grid->origin[a] : 0.0;
        p->n[a] = a < d ? grid->n[a] : 1;
        const int64_t nmax = d == 2 ? 512 : 256;  // padded lengths up to 1024 (2D) / 512 (3D)
        if (p->n[a] < 1 || p->n[a] > nmax) {
            set_error("grid size per axis must be in [1, " + std::to_string(nmax) + "]");
            return BEMFFT_EINVAL;
        }
        if (a < d) {
            int64_t pad = grid->pad[a] ? grid->pad[a] : auto_pad(p->n[a]);
            if (pad < 2 * p->n[a] - 1 || !fft_size_supported(pad) || pad == 1 || (d == 3 && pad > 512)) {
                set_error("padded length " + std::to_string(pad) + " on axis " + std::to_string(a) +
                          " is unsupported or shorter than 2n-1");
                return BEMFFT_EUNSUPPORTED;
            }
            p->pad[a] = p->P[a] = pad;
            p->H[a] = pad / 2 + 1;
        } else {
            p->pad[a] = p->P[a] = 1;
            p->H[a] = 1;
        }
    }
    // snap, validate
    std::vector<int> g((size_t)m * 3, 0);
    std::vector<double> w(m), nr((size_t)m * 3, 0.0);
    for (int64_t j = 0; j < m; ++j) {
        for (int a = 0; a < d; ++a) {
            const double x = nodes[j * d + a];
            const double nv = normals ? normals[j * d + a] : 0.0;
            if (!std::isfinite(x) || !std::isfinite(nv)) { set_error("non-finite node or normal"); return BEMFFT_EINVAL; }
            const double gi = std::floor((x - p->origin[a]) / p->h + 0.5);
            if (gi < 0.0 || gi >= (double)p->n[a]) {
                set_error("node " + std::to_string(j) + " lies outside the grid");
                return BEMFFT_EINVAL;
            }
            g[j * 3 + a] = (int)gi;
            nr[j * 3 + a] = nv;
        }
        // default measure: the grid's line or surface element (the half-space
        // grid is the surface itself: h^2)
        w[j] = weights ? weights[j] : (halfspace ? p->h * p->h : std::pow(p->h, d - 1));
        if (!(w[j] > 0.0) || !std::isfinite(w[j])) { set_error("weights must be positive and finite"); return BEMFFT_EINVAL; }
    }
    // sort by (z, y, x): rows of the grid become contiguous runs
    std::vector<int> perm(m);
    std::iota(perm.begin(), perm.end(), 0);
    std::stable_sort(perm.begin(), perm.end(), [&](int a, int b) {
        if (g[a * 3 + 2] != g[b * 3 + 2]) return g[a * 3 + 2] < g[b * 3 + 2];
        if (g[a * 3 + 1] != g[b * 3 + 1]) return g[a * 3 + 1] < g[b * 3 + 1];
        return g[a * 3] < g[b * 3];
    });
    const int zlo = g[perm[0] * 3 + 2], zhi = g[perm[m - 1] * 3 + 2];
    p->z0 = zlo;
    p->nzo = zhi - zlo + 1;
    if (d == 3 && grid->pad[2] == 0 && prec != BEMFFT_BF16_MFMA) {
        // Only offsets between occupied planes occur along z, in the apply and
        // in the grid evaluation alike, so a padded length of 2 nzo - 1 carries
        // the same sums; a body that does not fill its box then takes a shorter
        // transform (a length that the caller asked for is kept, and the 16-bit
        // form, bound by other loads, keeps the grid's: 33 us, 35 at the shorter one).
        // Navier takes 384 rather than 320, which is slower with every schedule (z
        // pass of a 160^3 cube with 150 planes, 320 and 384: FP32 470 and 419 us,
        // FP64 1472 and 1015).
        int64_t pz = auto_pad_len(2 * p->nzo - 1);
        if (pz == 320 && kernel == BEMFFT_NAVIER3D) pz = 384;
        if (pz < p->P[2]) {
            p->P[2] = pz;
            p->H[2] = pz / 2 + 1;
        }
    }
    const int64_t ny = p->n[1];
    std::vector<int> rowptr((size_t)p->nzo * ny + 1, 0);
    std::vector<int> sgx(m), sgy(m), sgz(m);
    std::vector<double> sw(m), snr((size_t)3 * m);
    for (int64_t s = 0; s < m; ++s) {
        const int j = perm[s];
        sgx[s] = g[j * 3];
        sgy[s] = g[j * 3 + 1];
        sgz[s] = g[j * 3 + 2];
        sw[s] = w[j];
        for (int a = 0; a < 3; ++a) snr[a * m + s] = nr[j * 3 + a];
        rowptr[(size_t)(sgz[s] - zlo) * ny + sgy[s] + 1] += 1;
    }
    for (size_t i = 1; i < rowptr.size(); ++i) rowptr[i] += rowptr[i - 1];
    // long rows get their x-transform from a row FFT
    const bool fold = p->dim == 2 && fold_rule(p, rowptr);
    const int dense = p->dim == 2 && !fold ? kDenseRow2d : kDenseRow;
    std::vector<int> row_dense((size_t)p->nzo * ny, -1), dense_rows;
    for (int64_t z = 0; z < p->nzo; ++z) {
        for (int64_t y = 0; y < ny; ++y) {
            const int64_t row = z * ny + y;
            if (rowptr[row + 1] - rowptr[row] >= dense) {
                row_dense[row] = (int)dense_rows.size();
                dense_rows.push_back((int)row);
            }
        }
    }
    p->nd = (int64_t)dense_rows.size();
    {
        int64_t busiest = 0;  // nodes of the busiest row that is not a long row
        for (size_t row = 0; row + 1 < rowptr.size(); ++row) {
            const int64_t c = rowptr[row + 1] - rowptr[row];
            if (c < dense) busiest = std::max(busiest, c);
        }
        p->fwd_xg = busiest <= kFewNodesRow ? 2 : 1;
    }
    {
        int64_t long_nodes = 0;
        for (int r : dense_rows) long_nodes += rowptr[r + 1] - rowptr[r];
        if (p->dim == 2)
            p->flat = (fold ? kFlatFold : 0) |
                      (long_nodes == m ? kFlatRows : m <= (p->O == 1 ? kWideNodes : 2 * kWideNodes) ? kFlatWide : 0);
        p->mixed_rows = p->nd > 0 && long_nodes < m;
        p->row_inv = (double)long_nodes * (double)p->H[0] * p->O > kRowInvWork ? 1 : 0;
    }
    // per-node free term and self correction blocks (sorted order)
    const int O = p->O;
    std::vector<double> C((size_t)m * O * O, 0.0), SC((size_t)m * O * O, 0.0);
    p->h_diag_dir.assign((size_t)O * m, 0.0);
    p->h_self.assign((size_t)O * O * m, 0.0);
    for (int64_t s = 0; s < m; ++s) {
        double self[9], k0w[9], n3[3] = {snr[s], snr[m + s], snr[2 * m + s]};
        self_blocks(kernel, sw[s], n3, p->h, nu, mu, self, k0w);
        for (int i = 0; i < O * O; ++i) SC[(size_t)s * O * O + i] = self[i] - k0w[i];
        for (int i = 0; i < O * O; ++i) p->h_self[(size_t)perm[s] * O * O + i] = self[i];
        for (int k = 0; k < O; ++k) p->h_diag_dir[(size_t)k * m + perm[s]] = -self[k * O + k];
    }
    int st_ = 0;
    st_ = dev_upload(&p->d_gx, sgx);
    if (!st_) st_ = dev_upload(&p->d_gy, sgy);
    if (!st_) st_ = dev_upload(&p->d_gz, sgz);
    if (!st_) st_ = dev_upload(&p->d_perm, perm);
    if (!st_) st_ = dev_upload(&p->d_rowptr, rowptr);
    if (!st_) st_ = dev_upload(&p->d_w, sw);
    if (!st_) st_ = dev_upload(&p->d_nrm, snr);
    if (!st_) st_ = dev_upload(&p->d_SC, SC);
    if (!st_) st_ = dev_upload(&p->d_C, C);  // zero until set below
    if (!st_) st_ = dev_upload(&p->d_row_dense, row_dense);
    if (!st_ && !dense_rows.empty()) st_ = dev_upload(&p->d_dense_rows, dense_rows);
    BF_CHECK(st_);
    // spectra in FP64, and the working-precision engine
    Engine e64;
    e64.precision = BEMFFT_FP64;
    e64.creal = 8;
    e64.sreal = 8;
    int status = alloc_workspace(p, &e64);
    if (!status) status = upload_twiddles(&e64, p);
    if (!status) status = build_spectra(p, &e64, st);
    if (status) { free_engine(&e64); return status; }
    // free term
    std::vector<double> Cs;
    if (halfspace) {  // r = K[sigma] - u for every mode
        Cs.assign((size_t)m * O * O, 0.0);
        for (int64_t s = 0; s < m; ++s)
            for (int k = 0; k < O; ++k) Cs[((size_t)s * O + k) * O + k] = -1.0;
    } else if (cmode == BEMFFT_C_IMPLICIT) {
        status = implicit_free_term(p, e64, st, Cs);
        if (status) { free_engine(&e64); return status; }
    } else {
        Cs.assign((size_t)m * O * O, 0.0);
        for (int64_t s = 0; s < m; ++s)
            for (int k = 0; k < O; ++k)
                for (int l = 0; l < O; ++l) {
                    double v;
                    if (cmode == BEMFFT_C_HALF) v = (k == l) ? 0.5 : 0.0;
                    else v = opts->c_user[(size_t)perm[s] * O * O + k * O + l];
                    if (!std::isfinite(v)) { free_engine(&e64); set_error("non-finite c_user"); return BEMFFT_EINVAL; }
                    Cs[((size_t)s * O + k) * O + l] = v;
                }
    }
    if (hipMemcpy(p->d_C, Cs.data(), Cs.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        free_engine(&e64);
        set_error("upload of c failed");
        return BEMFFT_EDEVICE;
    }
    p->h_c.assign((size_t)m * O * O, 0.0);
    p->h_diag_neu.assign((size_t)O * m, 0.0);
    for (int64_t s = 0; s < m; ++s) {
        for (int i = 0; i < O * O; ++i) p->h_c[(size_t)perm[s] * O * O + i] = Cs[(size_t)s * O * O + i];
        for (int k = 0; k < O; ++k) p->h_diag_neu[(size_t)k * m + perm[s]] = Cs[((size_t)s * O + k) * O + k];
    }
    if (prec == BEMFFT_FP64) {
        p->eng = e64;
        p->has64 = true;
    } else {
        Engine e32;  // FP32 or 16-bit working engine
        e32.precision = prec;
        status = alloc_workspace(p, &e32);  // sets the element sizes
        if (!status) status = upload_twiddles(&e32, p);
        if (!status) {
            // the FP64 spectra rounded once to the stored precision, on the device
            status = convert_spectra(p, e64, &e32, st);
            if (!status && hipStreamSynchronize(st) != hipSuccess) {
                set_error("spectrum conversion failed");
                status = BEMFFT_EDEVICE;
            }
        }
        if (status == 0 && opts && opts->keep_fp64) {
            p->eng64 = e64;  // the refinement's FP64 operator
            p->has64 = true;
        } else {
            free_engine(&e64);
        }
        if (status) { free_engine(&e32); free_engine(&p->eng64); p->has64 = false; return status; }
        p->eng = e32;
    }
    if (hipStreamSynchronize(st) != hipSuccess) { set_error("plan: stream sync failed"); return BEMFFT_EDEVICE; }
    const int tune = opts ? opts->autotune : 0;
    // the 16-bit z pass has one schedule (its transforms are matrix products)
    if (p->dim == 3 && prec != BEMFFT_BF16_MFMA) {
        p->zsched = p->eng.zsched;
        if (tune >= 2 && tune - 2 < num_zsched(p)) p->eng.zsched = p->zsched = tune - 2;
        else if (tune == 1) BF_CHECK(autotune_zsched(p, st));
    }
    p->plan_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return 0;
}

// Cache entries hold zsched + 4 (fwd_xg - 1); the "4:" prefix keeps entries
// written for other sets of schedules from being read.
std::string tune_key(const bemfft_plan *p) {
    return "4:" + std::to_string(p->kernel) + ":" + std::to_string(p->eng.precision) + ":" + std::to_string(p->P[0]) +
           "x" + std::to_string(p->P[1]) + "x" + std::to_string(p->P[2]) + "/" + std::to_string(num_zsched(p));
}

// Compiled z schedules of a plan: the default and the alternative one, and a
// third for the Navier family where the padded z length is 256, 384 or 512.
int num_zsched(const bemfft_plan *p) {
    const int64_t pad = p->pad[2];
    return (p->kernel == BEMFFT_NAVIER3D && (pad == 256 || pad == 384 || pad == 512)) ? 3 : 2;
}

// First schedule that is the same as s at the plan's z length: some lengths have
// fewer different ones than numbers.
template <bool N, bool F, int P>
int z_first_of(int s) {
    if constexpr (N) {
        if (s == 2) return z_first<N, F, P, 2>();
    }
    return s == 1 ? z_first<N, F, P, 1>() : 0;
}
template <bool N, bool F>
int z_first_at(int64_t pz, int s) {
    switch (pz) {
        case 32: return z_first_of<N, F, 32>(s);
        case 64: return z_first_of<N, F, 64>(s);
        case 96: return z_first_of<N, F, 96>(s);
        case 128: return z_first_of<N, F, 128>(s);
        case 192: return z_first_of<N, F, 192>(s);
        case 256: return z_first_of<N, F, 256>(s);
        case 320: return z_first_of<N, F, 320>(s);
        case 384: return z_first_of<N, F, 384>(s);
        case 512: return z_first_of<N, F, 512>(s);
        default: return s;
    }
}
int first_zsched(const bemfft_plan *p, int s) {
    const bool fp64 = p->eng.precision == BEMFFT_FP64;
    if (p->kernel == BEMFFT_NAVIER3D) return fp64 ? z_first_at<true, true>(p->P[2], s) : z_first_at<true, false>(p->P[2], s);
    return fp64 ? z_first_at<false, true>(p->P[2], s) : z_first_at<false, false>(p->P[2], s);
}

int tune_cache_lookup(const std::string &key) {
    const char *path = std::getenv("BEMFFT_TUNE_CACHE");
    if (!path || !*path) return -1;
    FILE *f = std::fopen(path, "r");
    if (!f) return -1;
    char k[128];
    int v = -1, found = -1;
    while (std::fscanf(f, "%127s %d", k, &v) == 2)
        if (key == k) found = v;
    std::fclose(f);
    return found;  // checked against the plan's schedules by the caller
}

void tune_cache_store(const std::string &key, int v) {
    const char *path = std::getenv("BEMFFT_TUNE_CACHE");
    if (!path || !*path) return;
    FILE *f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "%s %d\n", key.c_str(), v);
    std::fclose(f);
}

// Time the working-precision apply with each different z schedule (numbers of the
// same one get its time) and keep the fastest, then, with that schedule, the other number of kx per thread
// in the forward direct DFT (1 or 2) and keep the faster.
int autotune_zsched(bemfft_plan *p, hipStream_t st) {
    const std::string key = tune_key(p);
    const int nsched = num_zsched(p);
    const int cached = tune_cache_lookup(key);
    if (cached >= 0 && cached % 4 < nsched && cached / 4 < 2) {
        p->eng.zsched = p->zsched = cached % 4;
        p->fwd_xg = cached / 4 + 1;
        return 0;
    }
    const size_t bytes = (size_t)p->ncomp * p->m * sizeof(double);
    double *q = nullptr, *u = nullptr, *r = nullptr;
    hipEvent_t e0, e1;
    if (hipMalloc(&q, bytes) != hipSuccess || hipMalloc(&u, bytes) != hipSuccess || hipMalloc(&r, bytes) != hipSuccess) {
        dev_free(q);
        dev_free(u);
        dev_free(r);
        set_error("autotune: allocation failed");
        return BEMFFT_ENOMEM;
    }
    std::vector<double> ones((size_t)p->ncomp * p->m, 1.0);
    int status = 0;
    if (hipMemcpy(q, ones.data(), bytes, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(u, ones.data(), bytes, hipMemcpyHostToDevice) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
        hipEventCreate(&e1) != hipSuccess)
        status = BEMFFT_EDEVICE;
    const int reps = 20;
    // mean apply time in us with the plan's current settings
    auto time_apply = [&](double *us) {
        for (int i = 0; i < 3 && status == 0; ++i) status = launch_apply(p, p->eng, q, u, r, st);
        if (status) return;
        if (hipEventRecord(e0, st) != hipSuccess) { status = BEMFFT_EDEVICE; return; }
        for (int i = 0; i < reps && status == 0; ++i) status = launch_apply(p, p->eng, q, u, r, st);
        float ms = 0.f;
        if (status == 0 && (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                            hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
            status = BEMFFT_EDEVICE;
        *us = 1e3 * ms / reps;
    };
    for (int sched = 0; sched < nsched && status == 0; ++sched) {
        const int first = first_zsched(p, sched);
        p->eng.zsched = sched;
        if (first < sched) p->tune_us[sched] = p->tune_us[first];
        else time_apply(&p->tune_us[sched]);
    }
    if (status == 0) {
        p->zsched = 0;
        for (int sched = 1; sched < nsched; ++sched)
            if (p->tune_us[sched] < p->tune_us[p->zsched]) p->zsched = sched;
        p->eng.zsched = p->zsched;
    }
    // the width in use was timed with every schedule above; only the other one
    // needs applies of its own
    if (status == 0) {
        const int xg0 = p->fwd_xg, xg1 = 3 - xg0;
        p->fwd_tune_us[xg0 - 1] = p->tune_us[p->zsched];
        p->fwd_xg = xg1;
        time_apply(&p->fwd_tune_us[xg1 - 1]);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    dev_free(q);
    dev_free(u);
    dev_free(r);
    if (status) {
        if (status == BEMFFT_EDEVICE) set_error("autotune: HIP failure");
        return status;
    }
    p->fwd_xg = p->fwd_tune_us[1] < p->fwd_tune_us[0] ? 2 : 1;
    tune_cache_store(key, p->zsched + 4 * (p->fwd_xg - 1));
    return 0;
}

}  // namespace

extern "C" {

int bemfft_plan_create(bemfft_plan **out, const bemfft_grid *grid, int64_t m, const double *nodes,
                       const double *normals, const double *weights, int kernel, double nu, double mu,
                       const bemfft_plan_opts *opts) {
    if (!out || !grid) {
        set_error("out and grid must be non-null");
        return BEMFFT_EINVAL;
    }
    *out = nullptr;
    bemfft_plan *p = new (std::nothrow) bemfft_plan();
    if (!p) {
        set_error("host allocation failed");
        return BEMFFT_ENOMEM;
    }
    int st = plan_create_impl(p, grid, m, nodes, normals, weights, kernel, nu, mu, opts);
    if (st) {
        destroy_plan_state(p);
        delete p;
        return st;
    }
    *out = p;
    return 0;
}

int bemfft_apply(bemfft_plan *p, const double *q, const double *u, double *r, void *stream) {
    if (!p || !q || !u || !r) {
        set_error("apply: null argument");
        return BEMFFT_EINVAL;
    }
    return launch_apply(p, p->eng, q, u, r, (hipStream_t)stream);
}

int bemfft_apply_profile(bemfft_plan *p, const double *q, const double *u, double *r, int reps,
                         double *stage_ms, void *stream) {
    if (!p || !q || !u || !r || !stage_ms || reps < 1) {
        set_error("apply_profile: bad argument");
        return BEMFFT_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t ev[5];
    for (int i = 0; i < 5; ++i)
        if (hipEventCreate(&ev[i]) != hipSuccess) {
            for (int k = 0; k < i; ++k) (void)hipEventDestroy(ev[k]);
            set_error("hipEventCreate failed");
            return BEMFFT_EDEVICE;
        }
    double acc[4] = {0, 0, 0, 0};
    int status = 0;
    for (int it = 0; it < reps && status == 0; ++it) {
        status = launch_apply(p, p->eng, q, u, r, st, ev);
        if (status) break;
        if (hipEventSynchronize(ev[4]) != hipSuccess) { status = BEMFFT_EDEVICE; break; }
        for (int k = 0; k < 4; ++k) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev[k], ev[k + 1]) != hipSuccess) { status = BEMFFT_EDEVICE; break; }
            acc[k] += ms;
        }
    }
    for (int i = 0; i < 5; ++i) (void)hipEventDestroy(ev[i]);
    if (status == BEMFFT_EDEVICE) set_error("apply_profile: HIP failure");
    for (int k = 0; k < 4; ++k) stage_ms[k] = acc[k] / reps;
    return status;
}

int bemfft_eval_grid(bemfft_plan *p, const double *q, const double *u, double *out, void *stream) {
    if (!p || !q || !u || !out) {
        set_error("eval_grid: null argument");
        return BEMFFT_EINVAL;
    }
    ApplyArgs a;
    fill_apply_args(p, p->eng, p->eng, &a);
    a.q = q;
    a.u = u;
    hipStream_t st = (hipStream_t)stream;
    if (p->kernel == 0) return volume_kind<0>(p->eng.precision, a, out, st, nullptr);
    if (p->kernel == 1) return volume_kind<1>(p->eng.precision, a, out, st, nullptr);
    if (p->kernel == 3) return volume_kind<3>(p->eng.precision, a, out, st, nullptr);
    return volume_kind<2>(p->eng.precision, a, out, st, nullptr);
}

int bemfft_plan_get_info(const bemfft_plan *p, bemfft_plan_info *info) {
    if (!p || !info) {
        set_error("null argument");
        return BEMFFT_EINVAL;
    }
    std::memset(info, 0, sizeof(*info));
    info->dim = p->dim;
    info->kernel = p->kernel;
    info->precision = p->eng.precision;
    info->c_mode = p->cmode;
    info->m = p->m;
    info->ncomp = p->ncomp;
    for (int a = 0; a < 3; ++a) {
        info->n[a] = p->n[a];
        info->pad[a] = p->pad[a];
    }
    info->z_lo = p->z0;
    info->z_count = p->nzo;
    info->nfields = p->F;
    info->nspectra = p->K;
    info->noutputs = p->O;
    info->workspace_bytes = (int64_t)(p->eng.bytes + p->eng64.bytes);
    info->spectra_bytes = (int64_t)p->K * p->H[0] * p->H[1] * p->eng.hzs * (int64_t)p->eng.sreal;
    info->spectrum_parity_residual = p->parity_resid;
    info->plan_seconds = p->plan_seconds;
    info->zsched = p->zsched;
    for (int i = 0; i < 3; ++i) info->tune_us[i] = p->tune_us[i];
    info->fwd_xg = p->fwd_xg;
    for (int i = 0; i < 2; ++i) info->fwd_tune_us[i] = p->fwd_tune_us[i];
    return 0;
}

int bemfft_plan_get_lengths(const bemfft_plan *p, int64_t lengths[3]) {
    if (!p || !lengths) {
        set_error("null argument");
        return BEMFFT_EINVAL;
    }
    for (int a = 0; a < 3; ++a) lengths[a] = p->P[a];
    return 0;
}

int bemfft_plan_get_c(const bemfft_plan *p, double *c_host) {
    if (!p || !c_host) {
        set_error("null argument");
        return BEMFFT_EINVAL;
    }
    std::memcpy(c_host, p->h_c.data(), p->h_c.size() * sizeof(double));
    return 0;
}

int bemfft_plan_destroy(bemfft_plan *p) {
    if (!p) return 0;
    destroy_plan_state(p);
    delete p;
    return 0;
}

int bemfft_fft3d_c2c_f64(double *data, int64_t px, int64_t py, int64_t pz, int direction, void *stream) {
    if (!data || (direction != 1 && direction != -1)) {
        set_error("fft3d: bad argument");
        return BEMFFT_EINVAL;
    }
    return fft3d_c2c_f64(data, px, py, pz, direction, (hipStream_t)stream);
}

const char *bemfft_strerror(int status) {
    switch (status) {
        case BEMFFT_OK: return "ok";
        case BEMFFT_EINVAL: return "invalid argument";
        case BEMFFT_ENOMEM: return "out of memory";
        case BEMFFT_EDEVICE: return "HIP runtime error";
        case BEMFFT_EUNSUPPORTED: return "unsupported size";
        case BEMFFT_EBREAKDOWN: return "breakdown (non-finite values)";
        case BEMFFT_ENOCONV: return "not converged within maxit";
        default: return "unknown status";
    }
}

const char *bemfft_last_error(void) { return g_last_error.c_str(); }

int bemfft_supported_sizes(int64_t *sizes, int cap) {
    int n = (int)(sizeof(kSizes) / sizeof(kSizes[0]));
    for (int i = 0; i < n && i < cap; ++i) sizes[i] = kSizes[i];
    return n;
}

}  // extern "C"
