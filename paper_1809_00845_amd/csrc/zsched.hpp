// zsched.hpp -- transforms of the z pass and their radix schedules.
//
// The pass transforms pencils of at most P/2 occupied planes, zero-padded to
// P, and needs only the first P/2 planes of the result.  A pencil is
// transformed at length P in one wavefront (D = 1), or, where Navier's three
// output transforms and the field's do not fit the registers at length P, its
// frequencies are split by parity over two wavefronts (D = 2, radix-2
// decimation in frequency): with w = exp(-2 pi i / P),
//     X[2 k + r] = sum_(n < P/2) x[n] w^(r n) W_(P/2)^(n k),   r = 0, 1,
// and back y[n] = y_0[n] + w^-n y_1[n], each a plain transform of length P/2
// without padding.  (A split by residue mod 4 was measured too, 5 waves per
// SIMD for the 128^3 Laplace cube against 3: 71 us against 41, because Y is
// then read four times.)
#pragma once

#include "fft_device.hpp"

namespace bemfft {

// L points per pencil, TPP lanes per pencil, radices Rs.  Element i of a
// pencil sits at LDS slot i + (i >> SHIFT) of its PS slots: the shift and the
// stride with the fewest bank conflicts over the schedule's exchanges (none
// where there is one exchange), by enumeration.
template <int D_, int L_, int TPP_, int SHIFT_, int PS_, int... Rs>
struct ZShape {
    static constexpr int D = D_, L = L_, TPP = TPP_, SHIFT = SHIFT_, PS = PS_;
    static constexpr int E = L_ / TPP_;
    static constexpr int SCHED = 0;  // what z_tile_log2 asks for: not 0 where a schedule has its own tiles
    using rad = Radices<Rs...>;
    static_assert(PS >= L - 1 + ((L - 1) >> SHIFT) + 1, "pencil slots");
};

// Laplace at 32 points: a pencil is so short that a block is mostly latency, so
// four lanes per pencil, half the wavefronts of eight, keep a large plane's blocks
// resident at once (one plane of 184^2 points on a 192^2 grid, 193 x 384 pencils,
// FP32 18.0 -> 13.4 us, FP64 23.6 -> 16.8; 8 planes of 120^2: 12.4 -> 10.4).
//
// ZSel<NAV, F64, P, S>: schedule S of padded length P (NAV: Navier, else
// Laplace; F64: FP64).  S = 0 and 1 exist for every family, S = 2 for Navier.
// D depends on (NAV, F64, P) only, as the stored spectra do.
template <bool NAV, bool F64, int P, int S> struct ZSel;
template <bool N, bool F, int S> struct ZSel<N, F, 32, S> { using type = ZShape<1, 32, 8, 3, 40, 4, 4, 2>; };
template <bool F> struct ZSel<false, F, 32, 0> { using type = ZShape<1, 32, 4, 3, 36, 8, 4>; };
template <bool N, bool F, int S> struct ZSel<N, F, 64, S> { using type = ZShape<1, 64, 8, 3, 72, 8, 8>; };
template <bool N, bool F, int S> struct ZSel<N, F, 96, S> { using type = ZShape<1, 96, 8, 3, 120, 4, 4, 6>; };
template <bool N, bool F> struct ZSel<N, F, 96, 1> { using type = ZShape<1, 96, 8, 4, 104, 6, 4, 4>; };
template <bool N, bool F, int S> struct ZSel<N, F, 128, S> { using type = ZShape<1, 128, 16, 4, 135, 8, 4, 4>; };
template <bool N, bool F> struct ZSel<N, F, 128, 0> { using type = ZShape<1, 128, 8, 4, 136, 16, 8>; };
template <bool N, bool F, int S> struct ZSel<N, F, 192, S> { using type = ZShape<1, 192, 16, 5, 197, 12, 4, 4>; };
template <bool N> struct ZSel<N, false, 192, 0> { using type = ZShape<1, 192, 16, 2, 239, 4, 4, 12>; };
template <> struct ZSel<false, true, 192, 0> { using type = ZShape<1, 192, 16, 2, 239, 4, 4, 12>; };
template <> struct ZSel<true, true, 192, 1> { using type = ZShape<1, 192, 16, 2, 239, 4, 4, 12>; };
template <bool F> struct ZSel<false, F, 256, 0> { using type = ZShape<1, 256, 16, 4, 271, 16, 16>; };
template <bool F> struct ZSel<false, F, 256, 1> { using type = ZShape<1, 256, 32, 4, 271, 8, 8, 4>; };
template <bool F> struct ZSel<false, F, 320, 0> { using type = ZShape<1, 320, 16, 2, 399, 4, 4, 20>; };
template <bool F> struct ZSel<false, F, 320, 1> { using type = ZShape<1, 320, 16, 5, 329, 20, 4, 4>; };
template <bool F> struct ZSel<false, F, 384, 0> { using type = ZShape<1, 384, 16, 4, 407, 8, 6, 8>; };
template <bool F> struct ZSel<false, F, 384, 1> { using type = ZShape<1, 384, 32, 4, 407, 4, 4, 4, 6>; };
template <bool F> struct ZSel<false, F, 512, 0> { using type = ZShape<1, 512, 32, 4, 543, 8, 8, 8>; };
template <bool F> struct ZSel<false, F, 512, 1> { using type = ZShape<1, 512, 32, 4, 543, 16, 16, 2>; };
template <bool F, int S> struct ZSel<true, F, 256, S> { using type = ZShape<2, 128, 16, 4, 135, 8, 8, 2>; };
template <> struct ZSel<true, false, 256, 0> { using type = ZShape<2, 128, 8, 4, 136, 16, 8>; };
template <bool F> struct ZSel<true, F, 256, 1> { using type = ZShape<2, 128, 16, 4, 135, 8, 4, 4>; };
struct ZShapeNav256Few : ZShape<2, 128, 16, 4, 135, 8, 4, 4> {
    static constexpr int SCHED = 1;
};
template <> struct ZSel<true, true, 256, 1> { using type = ZShapeNav256Few; };
template <bool F, int S> struct ZSel<true, F, 320, S> { using type = ZShape<2, 160, 16, 9, 160, 10, 2, 2, 2, 2>; };
template <> struct ZSel<true, false, 320, 0> { using type = ZShape<2, 160, 8, 3, 184, 4, 4, 10>; };
template <int S> struct ZSel<true, false, 384, S> { using type = ZShape<2, 192, 16, 2, 239, 4, 4, 12>; };
template <> struct ZSel<true, false, 384, 0> { using type = ZShape<2, 192, 16, 5, 197, 12, 4, 4>; };
template <int S> struct ZSel<true, true, 384, S> { using type = ZShape<1, 384, 64, 9, 384, 6, 2, 2, 2, 2, 2, 2>; };
template <> struct ZSel<true, true, 384, 2> { using type = ZShape<1, 384, 32, 4, 407, 4, 4, 4, 6>; };
template <int S> struct ZSel<true, false, 512, S> { using type = ZShape<2, 256, 16, 4, 271, 16, 16>; };
template <> struct ZSel<true, false, 512, 0> { using type = ZShape<2, 256, 32, 4, 271, 8, 8, 4>; };
template <int S> struct ZSel<true, true, 512, S> { using type = ZShape<1, 512, 32, 4, 543, 8, 8, 8>; };
template <> struct ZSel<true, true, 512, 2> { using type = ZShape<1, 512, 64, 4, 543, 8, 8, 8>; };
template <typename R, int KIND, int P, int S>
using ZSched = typename ZSel<KIND == 2, sizeof(R) == 8, P, S>::type;

// First schedule that is the same as schedule S of a length (S itself if none is).
template <bool N, bool F, int P, int S, int T = 0>
constexpr int z_first() {
    if constexpr (T >= S) return S;
    else return std::is_same<typename ZSel<N, F, P, T>::type, typename ZSel<N, F, P, S>::type>::value ? T : z_first<N, F, P, S, T + 1>();
}

// Parts D of the frequencies in the z pass and the stored spectra of a family,
// precision and length.
__host__ __device__ constexpr int z_split(int kernel, bool f64, int64_t p) {
    return kernel != 2 ? 1 : (f64 ? (p == 256 || p == 320 ? 2 : 1) : (p >= 256 ? 2 : 1));
}

// log2 of Y's tile width along ky: Y is stored [f][kx][ky / KT][z][KT], with
// rows of 64 bytes (8 ky in FP32, 4 in FP64), or 128 where an FP64 wavefront
// takes 8 ky or two wavefronts share a pencil.  A z-pass wavefront then reads a
// few long runs of one compact tile.  Forward / z pass, 128^3 Laplace cube, us,
// with rows of 32, 64 and 128 bytes: FP32 44 / 42, 37 / 43, 37 / 47; FP64
// (64, 128) 60 / 78, 58 / 87.  Narrower rows cost the forward pass partial
// lines, wider ones the z pass.  Laplace at 32 points takes 16 ky, the pencils of
// a wavefront with four lanes each.  Navier FP64 at 256 points: rows of 64 bytes
// in schedule 1, 128 in the others (z pass with 128 and 64 bytes: 33 x 64 pencils
// 44.0, 38.3 us; 129 x 128 202, 189; two far plates, 129 x 256, 369, 354; but the
// forward pass of a body with long and short rows pays: the 100-point cube on
// 128^3 347, 336 and 148, 164).
__host__ __device__ constexpr int z_tile_log2(int kernel, bool f64, int pz, int sched) {
    if (kernel != 2 && pz == 32) return 4;
    if (kernel == 2 && f64 && pz == 256 && sched == 1) return 2;
    return f64 && pz > 128 && z_split(kernel, f64, pz) == 1 ? 2 : 3;
}

// Stored spectra of 3D plans at FP32 and FP64: [c][kx][part r][ky][k], k the
// frequency kz = D k + r <= P/2; rows of part 0 are padded to whole 16-byte
// runs, so that the rows of consecutive ky are one aligned run.
__host__ __device__ constexpr int spec_len(int d, int r, int hz) {
    return r == 0 ? ((hz - 1) / d + 1 + 3) / 4 * 4 : (hz - 1) / d;
}
// Values per (c, kx, ky) row, all parts; 2D plans (hz = 1) store one.
__host__ __device__ constexpr int spec_row(int d, int hz) {
    return hz == 1 ? 1 : spec_len(d, 0, hz) + (d == 2 ? spec_len(d, 1, hz) : 0);
}
// Position of (kx, ky, kz) of component c.
__host__ __device__ constexpr int64_t spec_index(int d, int c, int hx, int hy, int hz, int kx, int ky, int kz) {
    const int64_t base = ((int64_t)c * hx + kx) * hy * spec_row(d, hz);
    if (hz == 1) return base + ky;
    const int r = kz % d, l0 = spec_len(d, 0, hz);
    return base + (r == 0 ? (int64_t)ky * l0 : (int64_t)hy * l0 + (int64_t)ky * spec_len(d, 1, hz)) + kz / d;
}

// Twiddle table of a schedule in LDS: for D = 2 w^n, n < L; then per stage
// after the first exp(-2 pi i s k / (NS RAD)) at (s - 1) NS + k, so that
// neighbouring lanes read neighbouring values.
template <typename SH>
constexpr int zt_stage0() { return SH::D == 2 ? SH::L : 0; }
template <typename SH>
constexpr int zt_size() { return zt_stage0<SH>() + SH::L; }
template <typename R, int L, int PSTEP>
__device__ __forceinline__ void zt_fill_stages(cx<R> *, const cx<R> *, int, int, int, int, Radices<>) {}
template <typename R, int L, int PSTEP, int RAD, int... REST>
__device__ __forceinline__ void zt_fill_stages(cx<R> *tab, const cx<R> *tw, int ns, int off, int tid, int nt,
                                               Radices<RAD, REST...>) {
    if (ns > 1) {
        for (int i = tid; i < (RAD - 1) * ns; i += nt)
            tab[off + i] = tw[(i / ns + 1) * (i % ns) * (PSTEP * L / (ns * RAD))];
        off += (RAD - 1) * ns;
    }
    zt_fill_stages<R, L, PSTEP>(tab, tw, ns * RAD, off, tid, nt, Radices<REST...>{});
}
template <typename R, typename SH>
__device__ __forceinline__ void zt_fill(cx<R> *tab, const cx<R> *tw, int tid, int nt) {
    for (int i = tid; i < zt_stage0<SH>(); i += nt) tab[i] = tw[i];
    zt_fill_stages<R, SH::L, SH::D>(tab, tw, 1, zt_stage0<SH>(), tid, nt, typename SH::rad{});
}

// Stage of radix RAD with NS points done (the Stockham rule of
// fft_device.hpp); OFF: its twiddles in the table.
template <typename R, typename SH, int RAD, int NS, int OFF, int DIR>
__device__ __forceinline__ void z_stage(cx<R> (&x)[SH::E], cx<R> *pen, const cx<R> *tab, int t) {
    constexpr int E = SH::E, TPP = SH::TPP, L = SH::L, NB = E / RAD, STRIDE = L / RAD, SHIFT = SH::SHIFT;
    constexpr bool FIRST = NS == 1, LAST = NS * RAD == L;
    static_assert(E % RAD == 0, "radix must divide the points per lane");
    auto slot = [](int i) { return i + (i >> SHIFT); };
    cx<R> v[NB][RAD];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int s = 0; s < RAD; ++s) {
            if constexpr (FIRST) v[b][s] = x[b + s * NB];
            else v[b][s] = pen[slot(t + b * TPP + s * STRIDE)];
        }
    if constexpr (!FIRST) wave_lds_sync();  // all reads of this stage precede its writes
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int j = t + b * TPP;
        const int k = j % NS;
        if constexpr (!FIRST) {
#pragma unroll
            for (int s = 1; s < RAD; ++s) {
                const cx<R> w = tab[OFF + (s - 1) * NS + k];
                v[b][s] = (DIR < 0) ? cmul(v[b][s], w) : cmulc(v[b][s], w);
            }
        }
        DFT<RAD, DIR, R>::run(v[b]);
        if constexpr (LAST) {
#pragma unroll
            for (int s = 0; s < RAD; ++s) x[b + s * NB] = v[b][s];
        } else {
            const int base = (j / NS) * NS * RAD + k;
#pragma unroll
            for (int s = 0; s < RAD; ++s) pen[slot(base + s * NS)] = v[b][s];
        }
    }
    if constexpr (!LAST) wave_lds_sync();  // writes visible to the next stage
}
template <typename R, typename SH, int NS, int OFF, int DIR>
__device__ __forceinline__ void z_stages(cx<R> (&)[SH::E], cx<R> *, const cx<R> *, int, Radices<>) {}
template <typename R, typename SH, int NS, int OFF, int DIR, int RAD, int... REST>
__device__ __forceinline__ void z_stages(cx<R> (&x)[SH::E], cx<R> *pen, const cx<R> *tab, int t,
                                         Radices<RAD, REST...>) {
    z_stage<R, SH, RAD, NS, OFF, DIR>(x, pen, tab, t);
    z_stages<R, SH, NS * RAD, OFF + (NS > 1 ? (RAD - 1) * NS : 0), DIR>(x, pen, tab, t, Radices<REST...>{});
}

// Transform of length L of one pencil, in registers: lane t holds x[t + e TPP]
// before and after (unscaled; DIR = -1 forward, +1 inverse).  pen: the
// pencil's PS slots; tab: the table of zt_fill.
template <typename R, typename SH, int DIR>
__device__ __forceinline__ void z_fft(cx<R> (&x)[SH::E], cx<R> *pen, const cx<R> *tab, int t) {
    static_assert(64 % SH::TPP == 0, "a pencil must not straddle wavefronts");
    wave_lds_sync();  // earlier users of the pencil's slots are done
    z_stages<R, SH, 1, zt_stage0<SH>(), DIR>(x, pen, tab, t, typename SH::rad{});
}

}  // namespace bemfft
