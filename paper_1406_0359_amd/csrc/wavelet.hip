// SARA dictionary Psi / Psi^dagger (Section 2.2): Dirac basis plus Daubechies Db1..Db8
// wavelet bases, each scaled by 1/sqrt(q) so that Psi Psi^dagger = I (tight frame, as
// used in Section 3).
//
// Each wavelet basis is an L-level periodised orthonormal 2D DWT in Mallat layout.  One level
// on an axis of even length Ls:  a[i] = sum_k h[k] x[(2i+k) mod Ls],  d[i] = sum_k g[k] x[...]
// with g[k] = (-1)^k h[2N-1-k]; a level filters axis 1 then axis 0 of the top-left Ls x Ls
// block and the next level recurses on its LL quarter.  Synthesis is the exact transpose.
//
// All wavelet bases run in the same launch; a level is one launch of 2D tiles (both axes
// through LDS).  The finest synthesis level sums every basis (and the Dirac block) per
// output tile and writes the image once.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "lds_limit.h"
#include "partials.h"

namespace purify {

namespace {

struct WavArgs {
    int n, q, nwav;
    int block[MAX_WAV];   // alpha block of each wavelet basis
    int flen[MAX_WAV];    // filter length 2N
    int dirac_block;      // -1 if no Dirac basis
};

// Every level is one launch of 2D tiles, both axes through LDS.  The filters' lengths are
// template arguments of the two filtering steps and a workgroup's taps sit in scalar registers,
// so a step is a straight run of multiply-adds; each thread filters P adjacent positions, whose
// inputs overlap: 2P + F - 2 values read from LDS give 2P outputs of F taps.  (With a runtime
// filter length and one position a thread, three LDS reads fed four multiply-adds.)
//
// Tile geometry: TP0 x TP1 positions (2 TP0 x 2 TP1 image samples).  The first step filters
// axis 1, a thread per P1 positions of a window row; the second axis 0, a thread per P0
// positions of a column, its lanes along the row so that loads and stores are contiguous.
template <int TP0_, int TP1_, int P1_, int P0_, int NT_>
struct Geo {
    static constexpr int TP0 = TP0_, TP1 = TP1_, P1 = P1_, P0 = P0_, NT = NT_;
    static constexpr int HALO = MAX_TAPS - 2;
    static constexpr int W0 = 2 * TP0 + HALO;       // window rows (at most)
    static constexpr int W1 = 2 * TP1 + HALO;       // window columns (at most)
    static constexpr int C0 = TP0 + HALO / 2;       // synthesis: window positions per subband
    static constexpr int C1 = TP1 + HALO / 2;
    static constexpr int SEG = TP1 / P1;            // first step: threads per window row
    static constexpr int LW = W1 > 32 ? 64 : 32;    // lanes that load one window row
    static constexpr int LR = NT / LW;              // rows loaded at a time
    static constexpr int RB = (W0 + LR - 1) / LR;   // loads a thread
    static constexpr int RH = (C0 + LR - 1) / LR;   // synthesis: loads of the low, of the high rows
    // LDS strides.  Analysis windows keep pad elements after every 8 (a thread's P1 = 4
    // positions start 8 apart); synthesis windows hold the low and the high half of a row C1
    // apart, at an odd stride.
    template <typename T> static constexpr int pad() { return sizeof(T) == 4 ? 2 : 1; }
    template <typename T> static constexpr int is() {
        constexpr int w = W1 + pad<T>() * (W1 / 8);
        constexpr int m = sizeof(T) == 4 ? 16 : 8, want = sizeof(T) == 4 ? 8 : 4;
        return w + (want - w % m + m) % m;
    }
    static constexpr int WS = 2 * C1 + 1;
    static constexpr int MS = 2 * TP1 + 2;
    static_assert(W0 * SEG <= NT && 2 * TP1 * (TP0 / P0) <= NT, "one task a thread");
    static_assert(W1 <= 64 && NT % 64 == 0, "one lane a window column");
};
// 32 x 32 samples.  (64 x 32 samples with 320 threads have less halo but fewer workgroups a CU to
// hide the windows' loads behind: 4096^2 analysis 500 -> 678 us, synthesis 732 -> 991 us.)
using GeoWav = Geo<16, 16, 4, 2, 256>;

// Taps of one basis: lowpass h; highpass g[k] = (-1)^k h[F - 1 - k].
template <typename T, int F>
struct Taps {
    T h[F];
    __device__ __forceinline__ explicit Taps(const T* __restrict__ f) {
#pragma unroll
        for (int k = 0; k < F; ++k) h[k] = f[k];
    }
    __device__ __forceinline__ T lo(int k) const { return h[k]; }
    __device__ __forceinline__ T hi(int k) const { return (k & 1) ? -h[F - 1 - k] : h[F - 1 - k]; }
};

__device__ __forceinline__ float fma_(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return fma(a, b, c); }

// f(std::integral_constant<int, F>) for a filter length F = 2, 4, ..., 16 (uniform)
template <typename Fn>
__device__ __forceinline__ void with_flen(int F, Fn f) {
    switch (F) {
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 8: f(std::integral_constant<int, 8>{}); break;
        case 10: f(std::integral_constant<int, 10>{}); break;
        case 12: f(std::integral_constant<int, 12>{}); break;
        case 14: f(std::integral_constant<int, 14>{}); break;
        default: f(std::integral_constant<int, 16>{}); break;
    }
}

// P adjacent positions of one axis: lo[p] = sum_k h[k] v[2p + k], hi[p] = sum_k g[k] v[2p + k]
template <typename T, int F, int P>
__device__ __forceinline__ void analyse(const cpx<T>* v, const Taps<T, F>& t, cpx<T>* lo, cpx<T>* hi) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
        T lx = 0, ly = 0, hx = 0, hy = 0;
#pragma unroll
        for (int k = 0; k < F; ++k) {
            const cpx<T> a = v[2 * p + k];
            lx = fma_(t.lo(k), a.x, lx);
            ly = fma_(t.lo(k), a.y, ly);
            hx = fma_(t.hi(k), a.x, hx);
            hy = fma_(t.hi(k), a.y, hy);
        }
        lo[p] = mk<T>(lx, ly);
        hi[p] = mk<T>(hx, hy);
    }
}

// The transpose: sample pairs 2j, 2j + 1 from the coefficients j - t, t < F/2; lo and hi hold
// P + F/2 - 1 coefficients from j_0 - (F/2 - 1) on.  Adds to even[p] and odd[p].
template <typename T, int F, int P>
__device__ __forceinline__ void synthesise(const cpx<T>* lo, const cpx<T>* hi, const Taps<T, F>& tp, cpx<T>* even,
                                           cpx<T>* odd) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int t = 0; t < F / 2; ++t) {
            const cpx<T> l = lo[p + F / 2 - 1 - t], h = hi[p + F / 2 - 1 - t];
            even[p].x = fma_(tp.lo(2 * t), l.x, even[p].x);
            even[p].y = fma_(tp.lo(2 * t), l.y, even[p].y);
            even[p].x = fma_(tp.hi(2 * t), h.x, even[p].x);
            even[p].y = fma_(tp.hi(2 * t), h.y, even[p].y);
            odd[p].x = fma_(tp.lo(2 * t + 1), l.x, odd[p].x);
            odd[p].y = fma_(tp.lo(2 * t + 1), l.y, odd[p].y);
            odd[p].x = fma_(tp.hi(2 * t + 1), h.x, odd[p].x);
            odd[p].y = fma_(tp.hi(2 * t + 1), h.y, odd[p].y);
        }
    }
}

// One analysis level on a tile.  src: the image (finest level, shared by all bases, times
// `scale`; src_bstride = 0) or the previous level's LL blocks (compact slots).  Detail subbands
// go to the alpha block; the LL subband to `llout` (compact slots of (n/2)^2 per basis, row
// stride Ls/2), or into the alpha block at the coarsest level (llout == null), so no launch
// reads what it writes.  Where Ls/2 is smaller than a tile the window repeats periodically and
// the surplus positions are not written.
// One basis a workgroup (blockIdx.y), the Dirac block a workgroup of its own (blockIdx.y ==
// nwav), or with ALL every basis and the Dirac block in turn: a thread's inputs of a window row
// then stay in registers for all bases, and `mid` is double-buffered in the window's LDS, so a
// basis costs one barrier.
// XHAT (finest level only): the image is x + a p with a the CG step length from xa's partial
// sums, formed as the window is read.
// Bound: large images by the write of the coefficients (4096^2, nine bases and five levels: 1.34
// GB in and out, 275 us at the copy rate of 4.9 TB/s) beside about as much arithmetic; small ones
// by the latency of a launch's window, taps and two steps.  With register-blocked steps of fixed
// filter length 4096^2 FP32 takes 503 us (644 before), 1024^2 43 (63), 256^2 FP64 19 (32).
template <typename T, typename G, bool ALL, bool XHAT>
__global__ void __launch_bounds__(G::NT)
k_wav_fwd(const cpx<T>* __restrict__ src, size_t src_bstride, cpx<T>* __restrict__ alpha,
          cpx<T>* __restrict__ llout, const T* __restrict__ filt, WavArgs A, int Ls, T scale, XhatArgs<T> xa) {
    constexpr int IS = G::template is<T>(), PADE = G::template pad<T>(), MS = G::MS, P1 = G::P1, P0 = G::P0;
    constexpr int IN = G::W0 * IS, MID = G::W0 * MS;
    static_assert(2 * P1 == 8, "window pads follow the segments");
    __shared__ __attribute__((aligned(16))) cpx<T> sm[ALL ? (IN > 2 * MID ? IN : 2 * MID) : IN + MID];
    const int n = A.n;
    const size_t N = (size_t)n * n;
    const int half = Ls >> 1;
    const int tiles1 = half > G::TP1 ? half / G::TP1 : 1;
    const int ti0 = blockIdx.x / tiles1, ti1 = blockIdx.x % tiles1;
    const int r0 = 2 * G::TP0 * ti0, c0 = 2 * G::TP1 * ti1;
    const int z0 = ALL ? 0 : (int)blockIdx.y;
    const bool dirac = ALL ? A.dirac_block >= 0 : z0 == A.nwav;
    // the window's extent: the basis' filter (ALL: the longest, the last basis'), or the tile
    // itself for the Dirac block
    const int F0 = ALL ? A.flen[A.nwav - 1] : (dirac ? 2 : A.flen[z0]);
    const int R0 = 2 * G::TP0 + F0 - 2, R1 = 2 * G::TP1 + F0 - 2;
    {   // lane = column, all of a thread's rows in flight before any is stored
        const cpx<T>* s = src + (ALL || dirac ? 0 : (size_t)z0 * src_bstride);
        const int b = threadIdx.x % G::LW, a0 = threadIdx.x / G::LW;
        const uint32_t co = (c0 + b) & (Ls - 1), lgs = __builtin_ctz(Ls);   // sides are powers of two
        T xs = 0;
        if constexpr (XHAT) xs = cg_alpha<T>(xa.rho_part, xa.rho_count, xa.pq_part, xa.pq_count);
        (void)xs;
        if (b < R1) {
            cpx<T> v[G::RB], pv[XHAT ? G::RB : 1];
#pragma unroll
            for (int k = 0; k < G::RB; ++k) {
                // beyond the window: its last row again (a condition here would make the
                // compiler wait for each load in a block of its own)
                const int a = min(a0 + k * G::LR, R0 - 1);
                const uint32_t o = ((uint32_t)((r0 + a) & (Ls - 1)) << lgs) + co;
                v[k] = s[o];
                if constexpr (XHAT) pv[k] = xa.p[o];
            }
            (void)pv;
#pragma unroll
            for (int k = 0; k < G::RB; ++k) {
                const int a = min(a0 + k * G::LR, R0 - 1);
                if constexpr (XHAT) v[k] = v[k] + xs * pv[k];
                sm[a * IS + b + PADE * (b >> 3)] = v[k];
            }
        }
    }
    __syncthreads();
    if (dirac) {   // the tile's own samples
        for (int i = threadIdx.x; i < 4 * G::TP0 * G::TP1; i += G::NT) {
            const int a = i / (2 * G::TP1), b = i % (2 * G::TP1);
            if (r0 + a < n && c0 + b < n)
                alpha[(size_t)A.dirac_block * N + (size_t)(r0 + a) * n + c0 + b] = scale * sm[a * IS + b + PADE * (b >> 3)];
        }
        if constexpr (!ALL) return;
    }
    // first step's task: window row, P1 positions from seg P1
    const int row = threadIdx.x / G::SEG, seg = threadIdx.x % G::SEG;
    const cpx<T>* wrow = sm + row * IS + seg * (2 * P1 + PADE);
    constexpr int NV = 2 * P1 + G::HALO;
    cpx<T> v[NV];
    if constexpr (ALL) {
        if (row < R0) {
#pragma unroll
            for (int j = 0; j < NV; ++j) v[j] = wrow[j + PADE * (j >> 3)];   // beyond R1: not used
        }
        __syncthreads();   // the window is in registers: its LDS becomes `mid`
    }
    // second step's task: column (low | high along axis 1), P0 positions from g0 P0
    const int col = threadIdx.x % (2 * G::TP1), g0 = threadIdx.x / (2 * G::TP1);
    const int i1 = G::TP1 * ti1 + (col >= G::TP1 ? col - G::TP1 : col);
    const bool two = g0 < G::TP0 / P0 && i1 < half;
    const int z1 = ALL ? A.nwav : z0 + 1;
    for (int z = z0; z < z1; ++z) {
        cpx<T>* mid = ALL ? sm + (z & 1) * MID : sm + IN;
        const int F = A.flen[z];
        const T* h = filt + z * 2 * MAX_TAPS;
        if (row < 2 * G::TP0 + F - 2) {
            with_flen(F, [&](auto f) {
                constexpr int FL = decltype(f)::value;
                const Taps<T, FL> t(h);
                if constexpr (!ALL) {
#pragma unroll
                    for (int j = 0; j < 2 * P1 + FL - 2; ++j) v[j] = wrow[j + PADE * (j >> 3)];
                }
                cpx<T> lo[P1], hi[P1];
                analyse<T, FL, P1>(v, t, lo, hi);
#pragma unroll
                for (int p = 0; p < P1; ++p) {
                    mid[row * MS + seg * P1 + p] = lo[p];
                    mid[row * MS + G::TP1 + seg * P1 + p] = hi[p];
                }
            });
        }
        __syncthreads();
        if (two) {
            const size_t blk = (size_t)A.block[z] * N;
            const int i0 = G::TP0 * ti0 + P0 * g0;
            const int cl = col >= G::TP1 ? half + i1 : i1;
            cpx<T>* al = alpha + blk + (size_t)i0 * n + cl;
            cpx<T>* ah = al + (size_t)half * n;
            const bool toll = col < G::TP1 && llout;
            cpx<T>* ll = toll ? llout + (size_t)z * (N / 4) + (size_t)i0 * half + cl : al;
            const size_t lld = toll ? half : n;
            with_flen(F, [&](auto f) {
                constexpr int FL = decltype(f)::value;
                const Taps<T, FL> t(h);
                cpx<T> u[2 * P0 + FL - 2], lo[P0], hi[P0];
#pragma unroll
                for (int j = 0; j < 2 * P0 + FL - 2; ++j) u[j] = mid[(2 * P0 * g0 + j) * MS + col];
                analyse<T, FL, P0>(u, t, lo, hi);
#pragma unroll
                for (int p = 0; p < P0; ++p) {
                    if (i0 + p < half) {
                        ll[p * lld] = scale * lo[p];
                        ah[(size_t)p * n] = scale * hi[p];
                    }
                }
            });
        }
    }
}

// Synthesis of one level on a tile of 2 TP0 x 2 TP1 samples of one basis: the window of the four
// subbands the tile reaches (TP + F/2 - 1 positions per axis per subband, periodic) goes into
// `in` (rows [0, C0) low and [C0, 2 C0) high along axis 0 for the filter's own C0 = TP0 + F/2 - 1;
// columns low at 0 and high at G::C1), axis 1 is undone into `mid` (high rows at G::C0), then
// axis 0.
template <typename T, typename G>
struct SynthWin {
    T x[2 * G::RH], y[2 * G::RH];
};

// A thread's window elements (lane = window column) into registers: the low rows (the LL block
// or the axis-1 detail), then the high rows (the two other details); rows past the filter's own
// are clamped to the last one as in k_wav_fwd, and lanes past its columns to the last column (left
// to run on they read up to thirty more columns a row: 4096^2 FP32 Psi, Db2 alone 111 -> 102 us,
// all bases 617 -> 607).  SKIP leaves out loads wholly past the rows (only where a barrier parts
// the loads from the stores, or the compiler joins the two blocks), and takes two rows a wave where
// a row is at most 32 columns (Psi 1024^2 FP32 57.7 -> 56.3 us, 4096^2 629 -> 617, 4096^2 with Db1
// and Db2 alone 161 -> 150).  Sides are powers of two, so a row's offset is a shift (64-bit products
// took as many cycles here as a filter step).
template <typename T, typename G, bool SKIP>
__device__ __forceinline__ void synth_load(SynthWin<T, G>& w, const cpx<T>* __restrict__ ab,
                                           const cpx<T>* __restrict__ lls, int lld, int n, int half, int m0, int m1,
                                           int F, int tid) {
    const int C0 = G::TP0 + F / 2 - 1, C1 = G::TP1 + F / 2 - 1;
    const int s0 = m0 / 2 - F / 2 + 1, s1 = m1 / 2 - F / 2 + 1;   // first window index
    // windows of at most half a wave's lanes: two rows a wave
    const bool narrow = SKIP && G::LW == 64 && 2 * C1 <= 32;
    const int b = min(narrow ? tid & 31 : tid % G::LW, 2 * C1 - 1), a0 = narrow ? tid >> 5 : tid / G::LW;
    const int LR = narrow ? 2 * G::LR : G::LR;
    const bool h1 = b >= C1;
    const int i1 = (s1 + (h1 ? b - C1 : b)) & (half - 1);
    const cpx<T>* lowp = h1 ? ab + half + i1 : lls + i1;
    const int lowsh = h1 ? __builtin_ctz(n) : __builtin_ctz(lld);
    const cpx<T>* highp = ab + (size_t)half * n + (h1 ? half + i1 : i1);
    const int highsh = __builtin_ctz(n);
#pragma unroll
    for (int k = 0; k < G::RH; ++k) {
        if (SKIP && k * LR >= C0) break;
        const uint32_t r = (s0 + min(a0 + k * LR, C0 - 1)) & (half - 1);
        const cpx<T> l = lowp[r << lowsh], h = highp[r << highsh];
        w.x[k] = l.x;
        w.y[k] = l.y;
        w.x[G::RH + k] = h.x;
        w.y[G::RH + k] = h.y;
    }
}

template <typename T, typename G, bool SKIP>
__device__ __forceinline__ void synth_store(const SynthWin<T, G>& w, int F, cpx<T>* in, int tid) {
    const int C0 = G::TP0 + F / 2 - 1, C1 = G::TP1 + F / 2 - 1;
    // windows of at most half a wave's lanes: two rows a wave
    const bool narrow = SKIP && G::LW == 64 && 2 * C1 <= 32;
    const int b = narrow ? tid & 31 : tid % G::LW, a0 = narrow ? tid >> 5 : tid / G::LW;
    const int LR = narrow ? 2 * G::LR : G::LR;
    const int c = b >= C1 ? G::C1 + b - C1 : b;
    if (b >= 2 * C1) return;
#pragma unroll
    for (int k = 0; k < G::RH; ++k) {
        if (SKIP && k * LR >= C0) break;
        cpx<T>* row = in + min(a0 + k * LR, C0 - 1) * G::WS + c;
        row[0] = mk<T>(w.x[k], w.y[k]);
        row[C0 * G::WS] = mk<T>(w.x[G::RH + k], w.y[G::RH + k]);
    }
}

// undo axis 1: a thread per P1 sample pairs of a window row.  INPLACE: `mid` reuses `in`'s LDS
// (a barrier of the whole workgroup between the reads and the writes).
template <typename T, typename G, bool INPLACE>
__device__ __forceinline__ void synth_axis1(int F, const T* __restrict__ h, const cpx<T>* in, cpx<T>* mid, int tid,
                                            bool active) {
    constexpr int P1 = G::P1;
    const int u = tid / G::SEG, seg = tid % G::SEG;
    const int C0 = G::TP0 + F / 2 - 1;
    const bool on = active && u < 2 * C0;
    constexpr int NV = P1 + MAX_TAPS / 2 - 1;
    cpx<T> lo[NV], hi[NV];
    if (on) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if (j < P1 + F / 2 - 1) {
                lo[j] = in[u * G::WS + seg * P1 + j];
                hi[j] = in[u * G::WS + G::C1 + seg * P1 + j];
            }
        }
    }
    if constexpr (INPLACE) __syncthreads();
    if (on) {
        with_flen(F, [&](auto f) {
            const Taps<T, decltype(f)::value> t(h);
            cpx<T> e[P1], o[P1];
#pragma unroll
            for (int p = 0; p < P1; ++p) e[p] = o[p] = mk<T>(0, 0);
            synthesise<T, decltype(f)::value, P1>(lo, hi, t, e, o);
            cpx<T>* m = mid + (u < C0 ? u : G::C0 + u - C0) * G::MS + 2 * seg * P1;
#pragma unroll
            for (int p = 0; p < P1; ++p) {
                m[2 * p] = e[p];
                m[2 * p + 1] = o[p];
            }
        });
    }
}

// undo axis 0: a thread per P0 sample pairs of a column (task col, g0), added to even and odd
template <typename T, typename G>
__device__ __forceinline__ void synth_axis0(int F, const T* __restrict__ h, const cpx<T>* mid, int col, int g0,
                                            cpx<T>* even, cpx<T>* odd) {
    with_flen(F, [&](auto f) {
        constexpr int FL = decltype(f)::value, NV = G::P0 + FL / 2 - 1;
        const Taps<T, FL> t(h);
        cpx<T> lo[NV], hi[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            lo[j] = mid[(g0 * G::P0 + j) * G::MS + col];
            hi[j] = mid[(G::C0 + g0 * G::P0 + j) * G::MS + col];
        }
        synthesise<T, FL, G::P0>(lo, hi, t, even, odd);
    });
}

// One synthesis level (output side Ls, level >= 1) for every basis (blockIdx.y): the
// coarser LL comes from `llin` (compact slots of (n/2)^2 per basis) or, at the coarsest
// level, from the alpha block; the result goes to `out` (compact slots, row stride Ls).
template <typename T, typename G>
__global__ void __launch_bounds__(G::NT)
k_wav_inv_level(const cpx<T>* __restrict__ alpha, const cpx<T>* __restrict__ llin, int ll_from_alpha,
                cpx<T>* __restrict__ out, const T* __restrict__ filt, WavArgs A, int Ls) {
    __shared__ __attribute__((aligned(16))) cpx<T> in[G::W0 * G::WS];
    __shared__ __attribute__((aligned(16))) cpx<T> mid[2 * G::C0 * G::MS];
    const int n = A.n;
    const size_t N = (size_t)n * n;
    const int half = Ls >> 1;
    const int tiles1 = Ls > 2 * G::TP1 ? Ls / (2 * G::TP1) : 1;
    const int m0 = 2 * G::TP0 * (blockIdx.x / tiles1), m1 = 2 * G::TP1 * (blockIdx.x % tiles1);
    const int z = blockIdx.y, F = A.flen[z];
    const T* h = filt + z * 2 * MAX_TAPS;
    const cpx<T>* ab = alpha + (size_t)A.block[z] * N;
    const int tid = threadIdx.x;
    {
        SynthWin<T, G> w;
        synth_load<T, G, false>(w, ab, ll_from_alpha ? ab : llin + (size_t)z * (N / 4), ll_from_alpha ? n : half, n, half, m0,
                         m1, F, tid);
        synth_store<T, G, false>(w, F, in, tid);
    }
    __syncthreads();
    synth_axis1<T, G, false>(F, h, in, mid, tid, true);
    __syncthreads();
    const int col = tid % (2 * G::TP1), g0 = tid / (2 * G::TP1);
    if (g0 >= G::TP0 / G::P0 || m1 + col >= Ls) return;
    cpx<T> e[G::P0], o[G::P0];
#pragma unroll
    for (int p = 0; p < G::P0; ++p) e[p] = o[p] = mk<T>(0, 0);
    synth_axis0<T, G>(F, h, mid, col, g0, e, o);
    const int r = m0 + 2 * G::P0 * g0;
    cpx<T>* d = out + (size_t)z * (N / 4) + (size_t)r * Ls + m1 + col;
#pragma unroll
    for (int p = 0; p < G::P0; ++p) {
        if (r + 2 * p < Ls) {
            d[(size_t)(2 * p) * Ls] = e[p];
            d[(size_t)(2 * p + 1) * Ls] = o[p];
        }
    }
}

// Finest synthesis level of small images: a 16 x 16 tile, one group of 128 threads a basis, all
// bases at once (a 256^2 image has one such tile a CU, so a basis after another would wait out
// each window's latency in turn).  The groups' partial sums are added in basis order, with the
// Dirac block, times `scale`.
using GeoFinal = Geo<8, 8, 2, 2, 128>;

template <typename T>
__global__ void __launch_bounds__(128 * MAX_WAV)
k_wav_inv_final(const cpx<T>* __restrict__ alpha, const cpx<T>* __restrict__ llin, int ll_from_alpha,
                cpx<T>* __restrict__ x, const T* __restrict__ filt, WavArgs A, T scale) {
    using G = GeoFinal;
    constexpr int FP = 2 * G::TP0;
    constexpr int IN = G::W0 * G::WS, MID = 2 * G::C0 * G::MS, SZ = IN > MID ? IN : MID;
    static_assert(FP * FP <= SZ, "a partial tile fits in the basis' window");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int n = A.n;
    const size_t N = (size_t)n * n;
    const int half = n >> 1;
    const int tiles = n / FP;
    const int m0 = FP * (blockIdx.x / tiles), m1 = FP * (blockIdx.x % tiles);
    const int z = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7), tid = threadIdx.x & 127;
    cpx<T>* in = reinterpret_cast<cpx<T>*>(smem_raw) + z * SZ;
    const int F = A.flen[z];
    const T* h = filt + z * 2 * MAX_TAPS;
    const cpx<T>* ab = alpha + (size_t)A.block[z] * N;
    {
        SynthWin<T, G> w;
        synth_load<T, G, false>(w, ab, ll_from_alpha ? ab : llin + (size_t)z * (N / 4), ll_from_alpha ? n : half, n, half, m0,
                         m1, F, tid);
        synth_store<T, G, false>(w, F, in, tid);
    }
    // the tile's Dirac samples are read before the barriers
    const int pix = threadIdx.x;
    const size_t po = (size_t)(m0 + (pix / FP) % FP) * n + m1 + pix % FP;
    cpx<T> dv = mk<T>(0, 0);
    if (pix < FP * FP && A.dirac_block >= 0) dv = alpha[(size_t)A.dirac_block * N + po];
    __syncthreads();
    synth_axis1<T, G, true>(F, h, in, in, tid, true);
    __syncthreads();
    const int col = tid % FP, g0 = tid / FP;
    cpx<T> e[G::P0], o[G::P0];
#pragma unroll
    for (int p = 0; p < G::P0; ++p) e[p] = o[p] = mk<T>(0, 0);
    const bool on = g0 < G::TP0 / G::P0;
    if (on) synth_axis0<T, G>(F, h, in, col, g0, e, o);
    __syncthreads();
    if (on) {
#pragma unroll
        for (int p = 0; p < G::P0; ++p) {
            in[(2 * (g0 * G::P0 + p)) * FP + col] = e[p];
            in[(2 * (g0 * G::P0 + p) + 1) * FP + col] = o[p];
        }
    }
    __syncthreads();
    const cpx<T>* all = reinterpret_cast<const cpx<T>*>(smem_raw);
    for (int i = pix; i < FP * FP; i += blockDim.x) {
        cpx<T> s = dv;
        size_t oi = po;
        if (i != pix) {   // fewer than two bases: a thread has a second pixel
            oi = (size_t)(m0 + i / FP) * n + m1 + i % FP;
            s = A.dirac_block >= 0 ? alpha[(size_t)A.dirac_block * N + oi] : mk<T>(0, 0);
        }
        for (int b = 0; b < A.nwav; ++b) s = s + all[b * SZ + i];
        x[oi] = scale * s;
    }
}

// Finest synthesis level of large images, one basis at a time per workgroup, with the next
// basis' window loaded into registers while the current one is filtered and stored to `in` after
// its second step, so the loads have both steps to arrive.  The sums over the bases stay in
// registers.
// Bound by the windows' loads (1.5 times the coefficients, the halos from L2): 1024^2 FP32 whole
// synthesis 75 -> 56 us, 4096^2 789 -> 607 us, 1024^2 FP64 195 -> 91 us.
template <typename T, typename G>
__global__ void __launch_bounds__(G::NT)
k_wav_inv_final_pipe(const cpx<T>* __restrict__ alpha, const cpx<T>* __restrict__ llin, int ll_from_alpha,
                     cpx<T>* __restrict__ x, const T* __restrict__ filt, WavArgs A, int raster, T scale) {
    __shared__ __attribute__((aligned(16))) cpx<T> in[G::W0 * G::WS];
    __shared__ __attribute__((aligned(16))) cpx<T> mid[2 * G::C0 * G::MS];
    const int n = A.n;
    const size_t N = (size_t)n * n;
    const int half = n >> 1;
    const int tiles1 = n / (2 * G::TP1);
    // unless raster, each XCD takes a contiguous range of tiles, so that the windows' halos meet in one L2
    // (1024^2 FP32 64 -> 58 us, FP64 98 -> 91 us; the analysis, which writes, lost 4% so)
    const int bx = raster || gridDim.x % 8 ? blockIdx.x : (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const int m0 = 2 * G::TP0 * (bx / tiles1), m1 = 2 * G::TP1 * (bx % tiles1);
    const int tid = threadIdx.x;
    const int lld = ll_from_alpha ? n : half;
    const int col = tid % (2 * G::TP1), g0 = tid / (2 * G::TP1);
    const bool on = g0 < G::TP0 / G::P0;
    const size_t off = (size_t)(m0 + 2 * G::P0 * g0) * n + m1 + col;
    // the sums start from the Dirac block, whose loads then run beside the first window's (loaded
    // after the bases: 4096^2 FP32 Psi 619 -> 612 us, Dirac + Db8 157 -> 140, Dirac + Db1 106 -> 99,
    // 1024^2 57 -> 56)
    cpx<T> e[G::P0], o[G::P0];
#pragma unroll
    for (int p = 0; p < G::P0; ++p) {
        e[p] = o[p] = mk<T>(0, 0);
        if (A.dirac_block >= 0 && on) {
            const cpx<T>* d = alpha + (size_t)A.dirac_block * N + off + (size_t)(2 * p) * n;
            e[p] = d[0];
            o[p] = d[n];
        }
    }
    SynthWin<T, G> w;
    auto load = [&](int z) {
        const cpx<T>* ab = alpha + (size_t)A.block[z] * N;
        synth_load<T, G, true>(w, ab, ll_from_alpha ? ab : llin + (size_t)z * (N / 4), lld, n, half, m0, m1, A.flen[z], tid);
    };
    load(0);
    synth_store<T, G, true>(w, A.flen[0], in, tid);
    __syncthreads();
    for (int z = 0; z < A.nwav; ++z) {
        const int F = A.flen[z];
        const T* h = filt + z * 2 * MAX_TAPS;
        const bool more = z + 1 < A.nwav;
        if (more) load(z + 1);
        synth_axis1<T, G, false>(F, h, in, mid, tid, true);
        __syncthreads();
        if (on) {
            cpx<T> be[G::P0], bo[G::P0];   // this basis' sums, added once formed
#pragma unroll
            for (int p = 0; p < G::P0; ++p) be[p] = bo[p] = mk<T>(0, 0);
            synth_axis0<T, G>(F, h, mid, col, g0, be, bo);
#pragma unroll
            for (int p = 0; p < G::P0; ++p) {
                e[p] = e[p] + be[p];
                o[p] = o[p] + bo[p];
            }
        }
        if (more) synth_store<T, G, true>(w, A.flen[z + 1], in, tid);
        __syncthreads();
    }
    if (!on) return;
#pragma unroll
    for (int p = 0; p < G::P0; ++p) {
        const size_t a = off + (size_t)(2 * p) * n;
        x[a] = scale * e[p];
        x[a + n] = scale * o[p];
    }
}

template <typename T>
__global__ void __launch_bounds__(256)
k_scale_copy_c(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst, T scale, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) dst[i] = scale * src[i];
}

WavArgs wav_args(const Plan& P) {
    WavArgs A{};
    A.n = P.n;
    A.q = P.q;
    A.nwav = P.nwav;
    for (int i = 0; i < P.nwav; ++i) {
        A.block[i] = P.wav_block[i];
        A.flen[i] = 2 * P.wav_N[i];
    }
    A.dirac_block = P.has_dirac ? 0 : -1;
    return A;
}

}  // namespace

// The finest analysis level can form x + alpha p on small images, whose CG update it then
// overlaps; on large ones reading p beside x would cost more than the update kernel's pass.
bool psi_adj_takes_xhat(const Plan& P) { return P.nwav > 0 && P.n < 1024; }

template <typename T, typename G, bool ALL, bool XHAT>
void fwd_level(const Plan& P, const WavArgs& A, int groups, int Ls, const cpx<T>* src, size_t bstride, cpx<T>* alpha,
               cpx<T>* llout, T scale, const XhatArgs<T>& xa, hipStream_t s) {
    const int half = Ls / 2;
    const dim3 g(std::max(1, half / G::TP0) * std::max(1, half / G::TP1), groups);
    hipLaunchKernelGGL((k_wav_fwd<T, G, ALL, XHAT>), g, dim3(G::NT), 0, s, src, bstride, alpha, llout,
                       (const T*)P.filters, A, Ls, scale, xa);
}

template <typename T>
void launch_psi_adj(const Plan& P, const cpx<T>* x, cpx<T>* alpha, hipStream_t s, const XhatArgs<T>* xa,
                    hipEvent_t first_done) {
    if (xa && !psi_adj_takes_xhat(P)) return;   // callers check psi_adj_takes_xhat first
    const WavArgs A = wav_args(P);
    const T scale = (T)(1.0 / std::sqrt((double)P.q));
    const int64_t N = P.N;
    if (P.nwav == 0) {
        hipLaunchKernelGGL(k_scale_copy_c<T>, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, x,
                           alpha, scale, N);
        return;
    }
    const XhatArgs<T> none{};
    // LL ping-pong buffers, one (n/2)^2 slot per basis each
    cpx<T>* llb[2] = {(cpx<T>*)P.ws2, (cpx<T>*)P.ws2 + (size_t)P.nwav * (N / 4)};
    for (int lev = 0; lev < P.levels; ++lev) {
        const int Ls = P.n >> lev;
        cpx<T>* llout = lev + 1 < P.levels ? llb[lev & 1] : nullptr;
        if (lev > 0) {
            fwd_level<T, GeoWav, false, false>(P, A, P.nwav, Ls, llb[(lev - 1) & 1], (size_t)(N / 4), alpha, llout,
                                               (T)1, none, s);
            continue;
        }
        // large images: one pass over the image for all bases (small ones need the bases'
        // separate workgroups to fill the device)
        const int ztot = P.nwav + (P.has_dirac ? 1 : 0);
        if (P.n >= 1024) fwd_level<T, GeoWav, true, false>(P, A, 1, Ls, x, 0, alpha, llout, scale, none, s);
        else if (xa) fwd_level<T, GeoWav, false, true>(P, A, ztot, Ls, x, 0, alpha, llout, scale, *xa, s);
        else fwd_level<T, GeoWav, false, false>(P, A, ztot, Ls, x, 0, alpha, llout, scale, none, s);
        if (first_done) (void)hipEventRecord(first_done, s);
    }
}

template <typename T, typename G>
void inv_level(const Plan& P, const WavArgs& A, const cpx<T>* alpha, const cpx<T>* in, int from_alpha, cpx<T>* out,
               int Ls, hipStream_t s) {
    const dim3 g(std::max(1, Ls / (2 * G::TP0)) * std::max(1, Ls / (2 * G::TP1)), P.nwav);
    hipLaunchKernelGGL((k_wav_inv_level<T, G>), g, dim3(G::NT), 0, s, alpha, in, from_alpha, out,
                       (const T*)P.filters, A, Ls);
}
template <typename T, typename G>
void inv_final_pipe(const Plan& P, const WavArgs& A, const cpx<T>* alpha, const cpx<T>* in, int from_alpha, cpx<T>* x,
                    T scale, hipStream_t s) {
    // Filters of at most four taps have hardly a halo to share in an L2; where the image and the
    // coefficients (Dirac's among them) reach the 256 MB of the last-level cache their tiles go in
    // raster order, all XCDs on one stretch of memory.  XCD ranges and raster, us: 4096^2 FP32 Db1
    // 94 and 88, Db2 108 and 102, both 153 and 144, Dirac with Db1 109 and 103, with Db2 119 and 112,
    // with both 166 and 154; FP64 165 and 158, 195 and 184, 277 and 265; 2048^2 FP64 Dirac with both 92
    // and 85.  2048^2 FP32 Db2 32.4 and 33.4, and with all nine bases 4096^2 617 and 643, so neither
    // of those.
    int fmax = 0;
    for (int z = 0; z < A.nwav; ++z) fmax = std::max(fmax, A.flen[z]);
    const int raster = fmax <= 4 && (size_t)(P.q + 1) * P.N * sizeof(cpx<T>) >= (size_t)256 << 20;
    hipLaunchKernelGGL((k_wav_inv_final_pipe<T, G>), dim3(P.N / (4 * G::TP0 * G::TP1)), dim3(G::NT), 0, s, alpha, in,
                       from_alpha, x, (const T*)P.filters, A, raster, scale);
}

template <typename T>
void launch_psi(const Plan& P, const cpx<T>* alpha, cpx<T>* x, hipStream_t s) {
    const WavArgs A = wav_args(P);
    const T scale = (T)(1.0 / std::sqrt((double)P.q));
    const int64_t N = P.N;
    if (P.nwav == 0) {
        hipLaunchKernelGGL(k_scale_copy_c<T>, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s,
                           alpha, x, scale, N);
        return;
    }
    // LL ping-pong buffers, one (n/2)^2 slot per basis each
    cpx<T>* llb[2] = {(cpx<T>*)P.ws2, (cpx<T>*)P.ws2 + (size_t)P.nwav * (N / 4)};
    int cur = -1;   // buffer holding the current LL, -1: the alpha block (coarsest level)
    for (int lev = P.levels - 1; lev >= 1; --lev) {
        const int Ls = P.n >> lev;
        const int dst = cur == 0 ? 1 : 0;
        const cpx<T>* in = cur < 0 ? alpha : llb[cur];
        inv_level<T, GeoWav>(P, A, alpha, in, cur < 0 ? 1 : 0, llb[dst], Ls, s);
        cur = dst;
    }
    const cpx<T>* in = cur < 0 ? alpha : llb[cur];
    // from 512^2 on there are at least as many 32 x 32 tiles as CUs and one basis after another
    // has the next one's window in flight (512^2 FP64 60 -> 39 us, FP32 52 -> 32 us)
    if (P.n >= 512) {
        inv_final_pipe<T, GeoWav>(P, A, alpha, in, cur < 0 ? 1 : 0, x, scale, s);
        return;
    }
    constexpr int SZ = std::max(GeoFinal::W0 * GeoFinal::WS, 2 * GeoFinal::C0 * GeoFinal::MS);
    const size_t lds = (size_t)P.nwav * SZ * sizeof(cpx<T>);
    auto f = k_wav_inv_final<T>;
    set_lds_limit(f, lds);
    const int tiles = P.n / 16;
    hipLaunchKernelGGL(f, dim3(tiles * tiles), dim3(128 * P.nwav), lds, s, alpha, in, cur < 0 ? 1 : 0, x,
                       (const T*)P.filters, A, scale);
}

template void launch_psi_adj<float>(const Plan&, const cpx<float>*, cpx<float>*, hipStream_t,
                                    const XhatArgs<float>*, hipEvent_t);
template void launch_psi_adj<double>(const Plan&, const cpx<double>*, cpx<double>*, hipStream_t,
                                     const XhatArgs<double>*, hipEvent_t);
template void launch_psi<float>(const Plan&, const cpx<float>*, cpx<float>*, hipStream_t);
template void launch_psi<double>(const Plan&, const cpx<double>*, cpx<double>*, hipStream_t);

}  // namespace purify
