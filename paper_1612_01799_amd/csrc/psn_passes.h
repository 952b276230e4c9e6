// The five pruned passes of one solve (paper section 2: the size-8N transform
// pair of I_1 with the G-tensor multiply; section 3: its cost).
//
// Layout (C order, last index contiguous), M = 2n:
//   rho, u : [i0][i1][i2]            n^3 reals
//   W1     : [i0][k2/BL][i1][k2%BL]  n^3 complex, k2 = 0..n-1, tiled over k2
//            (BL = the axis-1 column tile) so that an axis-1 workgroup's
//            column block is one contiguous run
//   W2     : n * M * n complex, blocked over k1 and tiled over k2 (W2Index)
//            so that both the axis-1 passes (fixed i0, all k1) and the axis-0
//            pass (fixed k1, all i0) read and write long contiguous runs
//   K      : [k1~][k2/KT][k0~][k2%KT] (n+1)^2 * n reals, folded k~ = min(k, M-k)
//   Kb     : [k1~][k0~]              (n+1)^2 reals
// The real-to-complex transform along axis 2 gives n+1 frequencies; the two
// real ones (k2 = 0 and k2 = n) travel packed as one complex value in column
// 0 (real part: k2 = 0, imaginary part: k2 = n).  The middle pass separates
// them with the conjugate-symmetric partner (-k0, -k1) and applies their own
// kernel values: Z' = a Z(k) + b conj(Z(-k)), a = (K0+Kn)/2, b = (K0-Kn)/2.
//
// Zero padding is never formed.  A length-M transform of a line whose second
// half is zero splits into two length-n transforms: even outputs are DFT_n(x),
// odd outputs DFT_n(x * w^j) with w = exp(-2 pi i / M).  Likewise a length-M
// inverse keeping only the first n outputs is IDFT_n(even) + w^-j IDFT_n(odd).
//
//   P1  axis 2, real -> complex   rho -> W1   (two reals per complex lane)
//   P2  axis 1, forward           W1  -> W2   (n inputs, M outputs)
//   P3  axis 0, forward, x K, inverse, in place on W2 (n in, n out)
//   P4  axis 1, inverse           W2  -> W1   (M inputs, n outputs)
//   P5  axis 2, complex -> real   W1  -> u
// The 1/M^3 of the inverse transform is folded into K.
#pragma once

#include "psn_device.h"
#include "psn_internal.h"

#include <type_traits>

namespace psn {

constexpr int kMaxLdsP3 = 163840;  // gfx950: 160 KB of LDS per workgroup

constexpr int pick_cols_p3(int N, int bmax, int cxbytes, int T) {
    for (int b = bmax; b >= 1; --b)
        if (N % b == 0 && (2 * b * N + ((2 * N + 15) & ~15)) * cxbytes <= kMaxLdsP3 && b * T <= 1024) return b;
    return 1;
}

// largest P3 tile width <= bmax that fits and divides the W2 layout tile
constexpr int pick_cols_p3_div(int N, int bmax, int cxbytes, int T, int layout_tile) {
    for (int b = bmax; b >= 1; --b)
        if (N % b == 0 && layout_tile % b == 0 && (2 * b * N + ((2 * N + 15) & ~15)) * cxbytes <= kMaxLdsP3 &&
            b * T <= 1024)
            return b;
    return 1;
}

// LDS row pitch of the contiguous passes (in elements): room for the skew of
// one slot per 16, rounded to 8 mod 32 so that the rows one wave touches at
// once (8-byte elements: 4 rows per 256-byte bank sweep; 16-byte: 2 rows)
// start in different banks
constexpr int rows_padded(int N) {
    int np = N + (N >> 4) + 1;
    while (np % 32 != 8) ++np;
    return np;
}

// lines per workgroup of the contiguous passes (up to `threads` threads);
// their LDS, at most `lds` bytes, holds the lines and the 2N-entry twiddle table
constexpr int pick_lines(int N, int T, int cxbytes, int threads, int lds) {
    int l = 1;
    for (int p = 2; p * T <= threads; p *= 2)
        if (N % p == 0 && (p * rows_padded(N) + ((2 * N + 15) & ~15)) * cxbytes <= lds) l = p;
    if (l * T < 64) {
        // a power of two leaves less than a wave: any divisor of N that fits
        for (int d = threads / T; d > l; --d)
            if (N % d == 0 && (d * rows_padded(N) + ((2 * N + 15) & ~15)) * cxbytes <= lds) return d;
    }
    return l;
}
// P1 and P5: up to 512 threads and 80 KB, so that two workgroups share a CU
// (at n = 512 FP32, 16 lines instead of 8: both passes about 5 % faster)
constexpr int kMaxLdsRows = 81920;

// W2 layout, tile-major: element (i0, k1, k2) lives at
//   slot / KB * blk + (i0 * (N / BL) + k2 / BL) * (KB * BL) + (slot % KB) * BL + k2 % BL
// with slot(k1) putting rows k1 and M-k1 next to each other (rows 0 and n
// form pair 0) and blk = N * N * KB plus a small pad, so that the k1 blocks of
// one tile, otherwise a power of two apart, do not share cache sets.  So the axis-1 passes (one i0, one tile of BL columns, all k1)
// write and read runs of KB * BL contiguous elements, and the two workgroups
// of the axis-0 pass that share a kernel row (k1 and M-k1) read the two halves
// of the same 128-byte lines.  BL is the column tile of the axis-1 passes.
//
// Paired form (PAIR): two consecutive i0 of a column sit next to each other,
//   slot / KB * blk + (i0 / 2 * (N / BL) + k2 / BL) * (2 KB BL) + (slot % KB) * 2 BL + (k2 % BL) * 2 + i0 % 2,
// so a slot row of a tile holds BL columns x 2 i0 (128 bytes in FP32), the
// axis-0 pass reads one 16-byte pair per lane and whole rows per eight lanes,
// and the axis-1 passes, each workgroup handling an i0 pair, move runs of
// 2 KB BL elements.
template <int N, int BL, bool PAIR = false>
struct W2Index {
    static constexpr int KB = psn_host::w2_k1_block(N);
    static constexpr size_t blk = size_t(N) * N * KB + psn_host::kW2BlockPad;  // stride of k1 blocks
    static_assert(N % BL == 0 && (2 * N) % KB == 0, "");
    static __device__ __forceinline__ int slot(int k1) {
        if (k1 == 0) return 0;
        if (k1 == N) return 1;
        return k1 < N ? 2 * k1 : 2 * (2 * N - k1) + 1;
    }
    static __device__ __forceinline__ size_t at(int i0, int k1, int k2) {
        const int sl = slot(k1);
        if constexpr (PAIR) {
            return size_t(sl / KB) * blk + (size_t(i0 >> 1) * (N / BL) + k2 / BL) * size_t(2 * KB * BL) +
                   size_t(sl % KB) * (2 * BL) + (k2 % BL) * 2 + (i0 & 1);
        } else {
            return size_t(sl / KB) * blk + (size_t(i0) * (N / BL) + k2 / BL) * size_t(KB * BL) +
                   size_t(sl % KB) * BL + k2 % BL;
        }
    }
    // stride between consecutive i0 (PAIR: consecutive i0 pairs) at fixed (k1, k2)
    static constexpr size_t s0 = size_t(N) * KB * (PAIR ? 2 : 1);
};

// Sizes whose W2 is stored in the paired form, so that the axis-0 pass moves
// whole 128-byte lines and not halves of them (a bare read, scale and write of
// W2 in its order is 17-19 % faster so at n = 512).
// FP32, n = 128 and n >= 256 (PairW2): the axis-0 pass splits
// each line by decimation in time into its even and odd samples, giving four
// half-length chains per line and one 16-byte access per lane; the axis-1
// passes take an i0 pair per thread.  (n = 384: 1.47 -> 1.37 ms a solve; 96 to
// 192 measured 5 to 15 % slower so and keep the plain form.)
template <int N, int DT>
struct PairW2 {
    static constexpr bool value = DT == DT_F32 && (N >= 256 || N == 128);
};
// FP64 arithmetic, n >= 96 (LaneW2): neighbouring lanes take the two i0 of a
// pair in every strided pass, on tiles of 4 columns (4 columns x 2 i0 x 16
// bytes).  n = 512: P2 + P3 + P4 4.93 -> 4.80 ms, n = 256: 0.64 -> 0.60 ms.  SPLIT's W1
// then moves in pieces of 48 bytes: P1 + P5 of 32 of n = 192 0.83 + 0.81 -> 0.85 + 0.85 ms.
template <int N, int DT>
struct LaneW2 {
    static constexpr bool value = DT != DT_F32 && N >= 96;
};

// W1 layout, tiled over k2: element (i0, i1, k2) lives at
//   ((i0 * (N / BL) + k2 / BL) * N + i1) * BL + k2 % BL,
// so the axis-1 passes (one i0, one tile of BL columns, all i1) move one
// contiguous block and the axis-2 passes (a few lines i1 of one i0) move
// runs of lines * BL elements.
template <int N, int BL>
struct W1Index {
    static_assert(N % BL == 0, "");
    static __device__ __forceinline__ size_t at(int i0, int i1, int k2) {
        return ((size_t(i0) * (N / BL) + k2 / BL) * N + i1) * BL + k2 % BL;
    }
};

// Cubes whose axes 1 and 0 run plane by plane in one launch (plane_conv), up to
// n = 64: three launches a solve instead of five.  Three against five launches, the same
// box, us a solve for one density and a batch of 13 and of 32:
//   n = 32  FP32 15.2 / 22.3                      FP64 15.1 / 19.3
//   n = 48  FP32 18.5 / 21.8                      FP64 20.8 / 25.8, 71 / 83, 136 / 158
//   n = 64  FP32 22.1 / 25.3,  80 / 85, 153 / 166   FP64 28.5 / 32.5, 134 / 139, 323 / 384
//                                              SPLIT 28.2 / 32.5, 132 / 132, 315 / 354
// At n = 96 FP32 a CU holds one workgroup of a plane only: one density 52 us against
// 46 in five launches, 13 of them 384 against 269.
template <int N, int DT>
struct PlaneCfg {
    using Real = typename Prec<DT>::Real;
    static constexpr int CX = sizeof(cx<Real>);
    // 8 elements per thread, or 12 with a factor 3 (two stages for 48 points and
    // not three: plane_conv 18.4 -> 12.6 us in FP64)
    static constexpr int T = N / (odd_part(N) > 1 ? 4 * odd_part(N) : elems8(N));
    static constexpr int threads = N * T;
    static constexpr int pitch() {
        int p = LdsLine<Real>::slots(N);
        while (p % 16 != 8) ++p;
        return p;
    }
    static constexpr size_t lds = size_t(N * pitch() + TwLds<Real>::slots(N)) * CX;
    static constexpr bool value = N <= psn_host::kPlaneMax;
    static_assert(!value || (threads <= 1024 && lds <= size_t(kMaxLdsP3)), "a plane fits a workgroup");
};

template <int N, int DT>
struct Cfg {
    using P = Prec<DT>;
    using Real = typename P::Real;
    using Io = typename P::Io;
    using Kt = typename P::Kt;
    static constexpr int E = elems_per_thread(N, sizeof(Real));
    static constexpr int T = N / E;
    static constexpr int CX = sizeof(cx<Real>);
    static constexpr int T24 = strided_team(N);                                // P2, P4 team (two chains)
    static constexpr int IP = LaneW2<N, DT>::value ? 2 : 1;                    // i0 per P2, P4 workgroup, in neighbouring lanes
    static constexpr int BS = PlaneCfg<N, DT>::value ? 1 : pick_cols_p3(N, IP == 2 && CX == 16 ? 4 : 8, CX, T24);  // P2, P4 columns
    static constexpr int T3 = strided_team(N);                                 // P3 team (two chains)
    static constexpr int BP3 = pick_cols_p3_div(N, DT == DT_F32 ? 8 : 4, CX, T3, BS);  // P3 columns (divide BS)
    static_assert(BS % BP3 == 0, "P3 tile must lie inside the W2 layout tile");
    static constexpr int LC = pick_lines(N, T, CX, 512, kMaxLdsRows);          // P1, P5 lines
    static constexpr int NP = rows_padded(N);
};

// One launch serves up to kMaxBatch problems of the same size.  The table
// travels by value in the kernel arguments (no device copy, capturable in a
// graph); workgroup units are numbered problem-major.
constexpr int kMaxBatch = kMaxBatchHost;

// Storage of the axis-1 output W2: split precision keeps it in FP64.  The
// middle pass reads and writes W2 in narrow column tiles at large strides,
// where 12-byte elements straddle the memory's 64-byte sectors; W1, moved in
// whole tile runs by the axis passes, keeps the 12-byte form.
template <int DT>
constexpr int w2_dt() {
    return DT == DT_SPLIT ? DT_F64 : DT;
}

template <int DT>
struct Prob {
    const typename Prec<DT>::Io* rho;
    typename Prec<DT>::Io* u;
    Work<DT> w1;
    Work<w2_dt<DT>()> w2;
    const typename Prec<DT>::Kt* K;
    const typename Prec<DT>::Kt* Kb;
    const cx<typename Prec<DT>::Real>* tw;
};

template <int DT>
struct Batch {
    int count;
    Prob<DT> p[kMaxBatch];
};

// Workgroup ids are dealt to the XCDs round robin; give each XCD a contiguous
// run of units so neighbouring tiles (which may share 128-byte lines) meet in
// the same L2.
// `first` blocks (a multiple of 8) before the units do other work.
__device__ __forceinline__ int xcd_unit(int first = 0) {
    const int g = int(blockIdx.x) - first;
    return (g % 8) * ((int(gridDim.x) - first) / 8) + g / 8;
}

// Grid size for `units` units dealt by xcd_unit().
inline int xcd_grid(long units) { return int(8 * ((units + 7) / 8)); }

// The LC * N W1 elements of an axis-2 workgroup in tile-contiguous order:
// element j = tid + LC * T * q is line lj = j / BL % LC and column
// k = j / (BL * LC) * BL + j % BL, so consecutive threads touch consecutive W1
// addresses.  When BL divides T, k = k0 + T * q with lj and k0 fixed per thread.
template <int N, int LC, int T, int BL>
struct TileOrder {
    static constexpr bool split = T % BL == 0;
    static __device__ __forceinline__ void at(int tid, int q, int& lj, int& k0, int& off) {
        if constexpr (split) {
            lj = (tid / BL) % LC;
            k0 = (tid / (BL * LC)) * BL + tid % BL;
            off = T * q;
        } else {
            const int j = tid + LC * T * q;
            lj = (j / BL) % LC;
            k0 = (j / (BL * LC)) * BL + j % BL;
            off = 0;
        }
    }
};

// ------------------------------------------------------------------ P1
template <int N, int DT>
__global__ void __launch_bounds__((Cfg<N, DT>::LC * Cfg<N, DT>::T))
p1_r2c(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using F = TeamFFT<N, C::T, Real, -1, false>;
    constexpr int units = N * N / C::LC;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    const cx<Real>* __restrict__ tw = P.tw;
    const int t = threadIdx.x % C::T, ln = threadIdx.x / C::T;
    const int line0 = (ug % units) * C::LC;  // first line of the workgroup; all share i0
    const int i0 = line0 / N, i1b = line0 % N;
    const typename C::Io* x = P.rho + (size_t(line0) + ln) * N;

    // z[j] = x[2j] + i x[2j+1]; zero for j >= n/2 (the padding)
    cx<Real> d[F::EM];
    static_assert(F::EI == F::E && F::EO == F::E, "every lane holds E elements");
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int pos = F::in_pos(t, e);
        if (pos < N / 2) d[e] = {Real(x[2 * pos]), Real(x[2 * pos + 1])};
        else d[e] = {Real(0), Real(0)};
    }
    TwLds<Real> tl{sb + C::LC * C::NP};
    tl.fill(tw, N, threadIdx.x, C::LC * C::T);
    LdsRows<Real> lds{sb + ln * C::NP};
    F::run1(d, t, tl, lds);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < F::E; ++e) lds.put2(t, F::out_pos(0, e), d[e]);  // out_pos(t, e) = t + out_pos(0, e)
    __syncthreads();
    // X[k] = E[k] + w^k O[k], E = (Z[k] + conj Z[n-k])/2, O = (Z[k] - conj Z[n-k])/(2i).
    // Element j of the workgroup's LC * N outputs is (line j / BS % LC,
    // k = j / (BS * LC) * BS + j % BS): consecutive threads write consecutive
    // W1 addresses.
    constexpr int BL = C::BS;
    using W1I = W1Index<N, BL>;
    using TO = TileOrder<N, C::LC, C::T, BL>;
#pragma unroll
    for (int q = 0; q < F::E; ++q) {
        int lj, k0, off;
        TO::at(int(threadIdx.x), q, lj, k0, off);
        const int k = k0 + off;
        const LdsRows<Real> row{sb + lj * C::NP};
        const cx<Real> Z = row.get2(k0, off);
        cx<Real> X;
        if (k == 0) {
            X = {Z.x + Z.y, Z.x - Z.y};  // (X[0], X[n]) packed
        } else {
            const cx<Real> Zr = conj(row.get2(N - k0, -off));
            const cx<Real> Ev = scale(Z + Zr, Real(0.5));
            const cx<Real> Od = rot<-1>(scale(Z - Zr, Real(0.5)));
            X = Ev + Od * tl(k);
        }
        w1.st(W1I::at(i0, i1b + lj, k), X);
    }
}

// ------------------------------------------------------------------ P2
// Unit = (i0, tile of B columns k2).  Both outputs of a line (DFT_n of x and
// of x w^j) are computed in lockstep from the same loads.
// LDS view of the strided passes: both chains side by side, or one at a time
template <class Real, bool SEQ>
using ChainLds = std::conditional_t<SEQ, LdsColsSeq<Real>, LdsCols2<Real>>;

// Minimum waves per SIMD asked of the compiler for P2 and P4 with em slots per
// chain and thread (TeamFFT::EM).
constexpr int p24_waves(int em, bool f32) { return f32 ? 1 : em <= 9 ? 4 : em <= 12 ? 3 : 1; }

template <int N, int DT, int B, int TT, bool SEQ>
__global__ void __launch_bounds__((Cfg<N, DT>::IP * B * TT),
                                  (p24_waves(TeamFFT<N, TT, typename Prec<DT>::Real, -1, false>::EM, DT == DT_F32)))
p2_fwd(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using F = TeamFFT<N, TT, Real, -1, false>;
    constexpr int IP = C::IP, BI = B * IP;  // i0 and lines per workgroup
    using WI = W2Index<N, C::BS, IP == 2>;
    static_assert(B == C::BS, "the axis-1 tile is the W2 layout tile");
    constexpr int tiles = N / B;
    constexpr int units = N / IP * tiles;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + (SEQ ? 1 : 2) * BI * N;
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    const auto& w2 = P.w2;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    const int i0b = u / tiles * IP, tile = u % tiles;
    const int l = threadIdx.x % BI, t = threadIdx.x / BI;
    const int i0 = i0b + l % IP, k2 = tile * B + l / IP;
    using W1I = W1Index<N, B>;

    cx<Real> d[2][F::EM];
    F::each_in(t, [&](int e) {
        const int pos = F::in_pos(t, e);
        d[0][e] = w1.ld(W1I::at(i0, pos, k2));
        d[1][e] = tw[pos];
    });
    TwLds<Real> tl{stw};
    tl.fill(tw, N, threadIdx.x, BI * TT);  // visible after the first exchange
    F::each_in(t, [&](int e) { d[1][e] = d[0][e] * d[1][e]; });
    ChainLds<Real, SEQ> lds{sb, BI, l};
    F::template run<2>(d, t, tl, lds);
    {
        // Stage the workgroup's output in LDS in W2 order (slot-major, BI
        // elements per slot), then store whole runs of KB * BI elements, two
        // consecutive elements per lane.  The two-chain exchange area holds all
        // 2N slots; the one-chain area holds N, so that variant stages in two
        // rounds.
        constexpr int KB = WI::KB, RUN = KB * BI;
        constexpr int HALF = SEQ ? N : 2 * N;  // slots per round
        const size_t tile0 = WI::at(i0b, 0, tile * B);  // (slot 0, column tile*B): start of block 0's run
#pragma unroll
        for (int h = 0; h < 2 * N / HALF; ++h) {
            __syncthreads();  // the last exchange's (or round's) reads are done
            const int th = here(t);
            F::each_out(th, [&](int e) {
                const int m = F::out_pos(th, e);
#pragma unroll
                for (int ch = 0; ch < 2; ++ch) {
                    const int sl = WI::slot(2 * m + ch) - h * HALF;
                    if (sl >= 0 && sl < HALF) sb[sl * BI + l] = d[ch][e];
                }
            });
            __syncthreads();
            for (int g = 2 * int(threadIdx.x); g < HALF * BI; g += 2 * BI * TT) {
                const int gg = h * HALF * BI + g;
                w2.st2(tile0 + size_t(gg / RUN) * WI::blk + gg % RUN, sb[g], sb[g + 1]);
            }
        }
    }
}

// ------------------------------------------------------------------ P3
// One workgroup = SL rows of W2 and B adjacent columns k2.  With SL = 2 the
// rows are k1 and M-k1, which share a kernel row and sit next to each other in
// the W2 layout, so each i0 is one run of 2 * B elements; with SL = 1 the two
// rows go to consecutive units instead.  The two parity chains (even and odd
// k0) of each line advance in lockstep, stored side by side in LDS, so one pair
// of barriers and one 16-byte access per element serve both.  Workgroup ids
// are dealt to the XCDs round robin; each XCD gets a contiguous run of units,
// so tiles sharing 128-byte lines and rows sharing a kernel row meet in the
// same L2.  The data and the pre-twiddles of the odd chain are loaded before any
// arithmetic, the kernel values after the forward transform (but for EARLY, below);
// the stage twiddles come from a copy of the table in LDS.  Column 0 (the packed k2 = 0 / k2 = n pair)
// is col0_conv's, on workgroups of the same launch.
template <int N>
struct P3Rows {
    static constexpr bool value = N >= 512;
};

// LDS of P3: the exchange area plus the stage twiddles
template <int N, int DT, int B, int TT, int SL, bool SEQ>
constexpr size_t lds_p3() {
    using Real = typename Cfg<N, DT>::Real;
    using Ff = TeamFFT<N, TT, Real, -1, false>;
    using Fi = TeamFFT<N, TT, Real, +1, true>;
    const size_t rows = P3Rows<N>::value ? Ff::rows_size() + (Ff::template same_rows<Fi>() ? 0 : Fi::rows_size())
                                         : TwLds<Real>::slots(N);
    return (size_t(SEQ ? 1 : 2) * B * SL * N + rows) * Cfg<N, DT>::CX;
}

// Per-stage twiddle rows for the half-length transforms of the paired middle
// pass (n >= 512, where the saved index arithmetic outweighs the fill).
template <int N>
struct P3PRows {
    static constexpr bool value = N >= 512;
};
template <int N, int DT, int TT>
constexpr size_t p3p_tw_entries() {
    using Real = typename Cfg<N, DT>::Real;
    using Ff = TeamFFT<N / 2, TT, Real, -1, false>;
    using Fi = TeamFFT<N / 2, TT, Real, +1, true>;
    if constexpr (P3PRows<N>::value) return Ff::rows_size() + (Ff::template same_rows<Fi>() ? 0 : Fi::rows_size());
    else return TwLds<Real>::slots(N);
}

template <int N, int DT, int B, int TT, int SL, int G>
constexpr size_t lds_p3p() {
    return (size_t(G) * (N / 2) * B * SL + p3p_tw_entries<N, DT, TT>()) * Cfg<N, DT>::CX;
}

// Column 0 of W2 carries Z = A + iB with A, B the spectra of the real k2 = 0
// and k2 = n planes.  With the partner row -k the product is
// Z' = a Z(k) + b conj(Z(-k)), a = (K0+Kn)/2 (stored in K's column 0) and
// b = (K0-Kn)/2 (stored in Kb).  A row pair is rows q and M-q (row 0 pairs
// with itself, as does row n).  It is a short dependent chain over few
// workgroups and 128-byte lines of 8 used bytes, so it runs as the first
// workgroups of P3's own launch (of NT threads and LDS bytes, G row pairs each) beside the
// other columns, and not as a launch of its own.  One density: n = 96 FP32 55 ->
// 49 us, n = 128 67 -> 62, n = 96 FP64 73 -> 68, n = 128 112 -> 106, n = 162 248 ->
// 233; the axis-0 pass and column 0 at n = 256 FP32 160 -> 154, n = 512 1160 -> 1145.
// The other columns' workgroups neither read nor write column 0.
template <int N, int DT, int NT, size_t LDS>
struct Col0 {
    // a row pair has four teams, one for each row and parity of k0 (one team that
    // took both parities needed 30 registers more than P3 has in FP64)
    static constexpr int T = 4 * Cfg<N, DT>::T3 <= NT ? Cfg<N, DT>::T3 : mid_plan(N) ? N / elems8(N) : NT / 4;
    // row pairs that the threads and that the LDS hold; threads past the last
    // pair only join the barriers, on one more region of LDS
    static constexpr int gt = NT / (4 * T), gl = int(LDS / (size_t(4) * N * Cfg<N, DT>::CX));
    static constexpr int G = gt * 4 * T == NT && gt <= gl ? gt : gt < gl - 1 ? gt : gl - 1;
    static_assert(G >= 1, "a workgroup holds a row pair");
    static constexpr int groups = (N + G - 1) / G;  // workgroups per problem
    static __host__ __device__ __forceinline__ int blocks(int count) { return (count * groups + 7) / 8 * 8; }
};

template <int N, int DT, int NT, size_t LDS>
__device__ __forceinline__ void col0_conv(const Batch<DT>& bt, int blk, void* smem) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using Kt = typename C::Kt;
    using G0 = Col0<N, DT, NT, LDS>;
    using Ff = TeamFFT<N, G0::T, Real, -1, false>;
    using Fi = TeamFFT<N, G0::T, Real, +1, true>;
    using WI = W2Index<N, C::BS, PairW2<N, DT>::value || LaneW2<N, DT>::value>;
    static_assert(Ff::EM == Fi::EM, "same plan, reversed");
    if (blk >= bt.count * G0::groups) return;  // whole workgroup
    const Prob<DT>& P = bt.p[blk / G0::groups];
    const auto& w2 = P.w2;
    const cx<Real>* __restrict__ tw = P.tw;
    const int g = threadIdx.x / (4 * G0::T);  // row pair within the workgroup
    const int set = threadIdx.x & 1, p = (threadIdx.x >> 1) & 1;
    const int t = (threadIdx.x >> 2) % G0::T;
    const int qg = (blk % G0::groups) * G0::G + g;
    const bool live = g < G0::G && qg < N;  // the last workgroup may hold pairs past the end
    const int q = live ? qg : N - 1;
    cx<Real>* sb = static_cast<cx<Real>*>(smem) + size_t(g < G0::G ? g : G0::G) * 4 * N;
    const int k1 = set == 0 ? q : (q == 0 ? N : 2 * N - q);
    const int kt1 = (q == 0) ? (set ? N : 0) : q;
    const int partner = (q == 0) ? set : 1 - set;
    const uint32_t kr = uint32_t(psn_host::k_index(N, kt1, 0, 0)), kb = uint32_t(kt1) * (N + 1);  // plane kt1, column 0

    cx<Real> d[Ff::EM];
    Ff::each_in(t, [&](int e) { d[e] = w2.ld(WI::at(Ff::in_pos(t, e), k1, 0)); });
    if (p) Ff::each_in(t, [&](int e) { d[e] = d[e] * gld(tw + Ff::in_pos(t, e)); });
    LdsCols<Real> lds{sb + set + 2 * p, 4, 0};
    Ff::run(d, t, tw, lds);
    __syncthreads();
    Ff::each_out(t, [&](int e) { sb[(set + 2 * p) * N + Ff::out_pos(t, e)] = d[e]; });
    __syncthreads();
    Ff::each_out(t, [&](int e) {
        const int m = Ff::out_pos(t, e);
        const int k0 = 2 * m + p;
        const int kt0 = k0 <= N ? k0 : 2 * N - k0;
        const int mp = p == 0 ? (m == 0 ? 0 : N - m) : N - 1 - m;
        const cx<Real> zp = conj(sb[(partner + 2 * p) * N + mp]);
        const Real a = Real(gld(byte_off(P.K, (kr + uint32_t(kt0 * psn_host::k_tile(N))) * uint32_t(sizeof(Kt)))));
        const Real b = Real(gld(byte_off(P.Kb, (kb + uint32_t(kt0)) * uint32_t(sizeof(Kt)))));
        d[e] = scale(d[e], a) + scale(zp, b);
    });
    Fi::run(d, here(t), tw, lds);
    const int to = here(t);
    __syncthreads();
    if (p) {
        Fi::each_out(to, [&](int e) {
            const int i = Fi::out_pos(to, e);
            sb[set * N + i] = mul_conj(d[e], gld(tw + i));
        });
    }
    __syncthreads();
    if (live && p == 0) {
        Fi::each_out(to, [&](int e) {
            const int i = Fi::out_pos(to, e);
            w2.st(WI::at(i, k1, 0), d[e] + sb[set * N + i]);
        });
    }
}

// Minimum waves per SIMD asked of the compiler for P3 with em slots per chain
// and thread (TeamFFT::EM): what fits without spills in every default tile.  (Two
// FP64 candidates spill: 12 threads a line at n = 96, 44 bytes; P4 with 8 at n = 96
// and 32 at n = 384, 20 and 28.)
constexpr int p3_waves(int em, bool f32) {
    if (f32) return em <= 9 ? 6 : em <= 10 ? 5 : em <= 12 ? 4 : em <= 20 ? 3 : 1;
    return em <= 9 ? 4 : em <= 12 ? 3 : 1;
}

// EARLY (row pairs on teams of 12 elements per thread): the twiddles w stay in
// registers and, in FP64, the kernel values are loaded with the data.  Fewer
// waves fit, and many densities in one launch still run faster so: 32 of
// n = 192, the 12-element teams late and early, FP32 2.07 and 1.96 ms; n = 96 FP32 288
// and 238 us; the fastest late tile and this one, n = 192 FP64 3.90 and 3.73 ms,
// n = 96 FP64 501 and 438 us.  20 elements early: 1.60 ms against 1.30 late (32 of 160, FP32).
template <int N, int DT, int B, int TT, int SL, bool SEQ, bool EARLY>
__global__ void __launch_bounds__((B * TT * SL),
                                  (EARLY ? DT == DT_F32 ? 3 : 1
                                         : p3_waves(TeamFFT<N, TT, typename Prec<DT>::Real, -1, false>::EM, DT == DT_F32)))
p3_conv(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using Ff = TeamFFT<N, TT, Real, -1, false>;
    using Fi = TeamFFT<N, TT, Real, +1, true>;
    static_assert(SL == 1 || SL == 2, "one row or a row pair per workgroup");
    constexpr int tiles = N / B;
    constexpr int units = (2 / SL) * N * tiles;  // per problem
    constexpr int IP = C::IP;                    // consecutive i0 in neighbouring lanes
    using WI = W2Index<N, C::BS, IP == 2>;
    static_assert(C::BS % B == 0, "the axis-0 tile lies inside a W2 layout tile");
    static_assert(TT % IP == 0 && (N / Ff::R0) % IP == 0, "an i0 pair is two neighbouring threads of a line");
    constexpr size_t s0 = WI::s0;  // stride of i0 (of i0 pairs) in W2
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + (SEQ ? 1 : 2) * B * SL * N;

    constexpr size_t lds_bytes = lds_p3<N, DT, B, TT, SL, SEQ>();
    const int first = Col0<N, DT, B * TT * SL, lds_bytes>::blocks(bt.count);
    if (int(blockIdx.x) < first) return col0_conv<N, DT, B * TT * SL, lds_bytes>(bt, int(blockIdx.x), smem);
    const int ug = xcd_unit(first);
    if (ug >= bt.count * units) return;  // whole workgroup
    const Prob<DT>& P = bt.p[ug / units];
    const auto& w2 = P.w2;
    const typename C::Kt* __restrict__ K = P.K;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    int q, tile, set;
    if constexpr (SL == 1) {
        const int item = u >> 1;
        set = u & 1;
        q = item / tiles;
        tile = item % tiles;
    } else {
        q = u / tiles;
        tile = u % tiles;
        set = (threadIdx.x / (B * IP)) & 1;
    }
    // lanes run over i0 % IP, the columns, the rows and the rest of i0
    const int par = threadIdx.x % IP, c = (threadIdx.x / IP) % B;
    const int tp = threadIdx.x / (IP * B * SL), t = IP * tp + par;
    const int k2 = tile * B + c;
    // Addresses: a base uniform over the workgroup (row q, column tile * B)
    // plus a 32-bit lane offset.  Row M-q sits IP * BS elements after row q in
    // the W2 layout; its kernel row is q as well, except for the pair (0, n).
    static_assert(WI::s0 * N * sizeof(cx<double>) < (size_t(1) << 32) &&
                      size_t(N + 1) * (N + 1) * N * sizeof(double) < (size_t(1) << 32),
                  "lane byte offsets fit 32 bits");
    const size_t ub = WI::at(0, q, tile * B);
    // element e sits at the uniform base xb(e) plus the lane offset xl (the lanes
    // of column 0, which col0_conv has, take column 1's and store nothing)
    const uint32_t xl = uint32_t(IP * (k2 == 0 ? 1 : c) + par) + uint32_t(set * IP) * C::BS + uint32_t(tp) * uint32_t(s0);
    auto xb = [&](int e) { return ub + size_t(Ff::in_pos(0, e) / IP) * s0; };
    // Kernel values of the even and odd outputs a = 2m, b = 2m + 1 of
    // m = out_pos(t, e) = t + m0(e), at the folded index min(a, 2N - a) of
    // this lane's kernel row (plane q, or n for the set-1 row of pair 0) in the
    // tiled K layout, where the folded k0 steps by the K tile width KT.  When a
    // whole element lies on one side of n, the folded index is a constant plus
    // 2t or minus 2t: a uniform base plus one of two lane offsets.
    constexpr int KT = psn_host::k_tile(N);
    const uint32_t kl = uint32_t(psn_host::k_index(N, (set != 0 && q == 0) ? N : q, 0, k2));
    const uint32_t kup = (kl + uint32_t(2 * t * KT)) * uint32_t(sizeof(typename C::Kt));
    const uint32_t kdn = (kl + uint32_t(2 * (TT - 1 - t) * KT)) * uint32_t(sizeof(typename C::Kt));
    auto kval = [&](int e, int odd) -> Real {
        const int m0 = Ff::out_pos(0, e);
        if (2 * (m0 + Ff::out_last(e)) + 1 <= N) return Real(gld(byte_off(sbase(K + (2 * m0 + odd) * KT), kup)));
        if (2 * m0 >= N) return Real(gld(byte_off(sbase(K + (2 * N - 2 * m0 - odd - 2 * (TT - 1)) * KT), kdn)));
        const int a = 2 * (m0 + t) + odd;
        return Real(gld(K + kl + uint32_t(a <= N ? a : 2 * N - a) * KT));
    };
    // w^i0 of slot e's input position, which is its output position too
    auto pre = [&](int e) {
        return gld(byte_off(sbase_here(tw + Ff::in_pos(0, e)), uint32_t(t) * uint32_t(C::CX)));
    };

    static_assert(Ff::EM == Fi::EM, "same plan, reversed");
    cx<Real> d[2][Ff::EM];
    cx<Real> w[EARLY ? Ff::EI : 1];
    Real kk[2][Ff::EO];
    auto load_k = [&]() {
        Ff::each_out(t, [&](int e) {
            kk[0][e] = kval(e, 0);
            kk[1][e] = kval(e, 1);
        });
    };
    Ff::each_in(t, [&](int e) {
        d[0][e] = w2.ld(xb(e), xl);
        if constexpr (EARLY) d[1][e] = w[e] = gld(tw + Ff::in_pos(t, e));
        else d[1][e] = pre(e);
    });
    if constexpr (EARLY && DT != DT_F32) load_k();
    // Stage twiddles: per-stage rows of both transforms (shared when their
    // radices match) for n >= 512, where the saved index arithmetic outweighs
    // the scattered reads that fill them; else the swizzled 2N-entry table.
    constexpr bool kRows = P3Rows<N>::value;
    cx<Real>* rows_i = stw + (Ff::template same_rows<Fi>() ? 0 : Ff::rows_size());
    using Tw = std::conditional_t<kRows, TwRows<Real>, TwLds<Real>>;
    if constexpr (kRows) {
        Ff::fill_rows(stw, tw, threadIdx.x, B * TT * SL);  // visible after the first exchange
        if constexpr (!Ff::template same_rows<Fi>()) Fi::fill_rows(rows_i, tw, threadIdx.x, B * TT * SL);
    } else {
        TwLds<Real>{stw}.fill(tw, N, threadIdx.x, B * TT * SL);
    }
    Ff::each_in(t, [&](int e) { d[1][e] = d[0][e] * d[1][e]; });
    ChainLds<Real, SEQ> lds{sb, B * SL, c + B * set * (SL - 1)};
    // But for EARLY, few values stay live across the transforms, so that more
    // waves fit: the kernel values are loaded after the forward one, the twiddles
    // w again at the end, and the addresses of the exchanges are formed anew for
    // the inverse (here) instead of being kept.  n = 512 FP64: 166 -> 124 VGPRs,
    // four waves per SIMD instead of three, 2.55 -> 2.39 ms; n = 320 FP64, with the
    // three-stage teams: 212 -> 112, four instead of two.
    Ff::template run<2>(d, t, Tw{stw}, lds);
    if constexpr (!EARLY) __builtin_amdgcn_sched_barrier(0);
    if constexpr (!EARLY || DT == DT_F32) load_k();
    // the multiply by K is folded into the first stage of the inverse
    Fi::template run_scaled<2>(d, EARLY ? t : here(t), Tw{kRows ? rows_i : stw}, lds, kk);
    if constexpr (!EARLY) __builtin_amdgcn_sched_barrier(0);
    if (k2 != 0) {
        Ff::each_in(t, [&](int e) {
            if constexpr (EARLY) w2.st(xb(e), xl, twfma<+1>(d[1][e], w[e], d[0][e]));
            else w2.st(xb(e), xl, twfma<+1>(d[1][e], pre(e), d[0][e]));
        });
    }
}

// ------------------------------------------------------------------ P4
// Unit = (i0, tile of B columns k2).  The even and odd rows of a line are
// inverted in lockstep and combined as y = y_even + w^-j y_odd.
template <int N, int DT, int B, int TT, bool SEQ>
__global__ void __launch_bounds__((Cfg<N, DT>::IP * B * TT),
                                  (p24_waves(TeamFFT<N, TT, typename Prec<DT>::Real, +1, false>::EM, DT == DT_F32)))
p4_inv(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using F = TeamFFT<N, TT, Real, +1, false>;
    constexpr int IP = C::IP, BI = B * IP;  // i0 and lines per workgroup
    using WI = W2Index<N, C::BS, IP == 2>;
    static_assert(B == C::BS, "the axis-1 tile is the W2 layout tile");
    constexpr int tiles = N / B;
    constexpr int units = N / IP * tiles;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + (SEQ ? 1 : 2) * BI * N;
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    const auto& w2 = P.w2;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    const int l = threadIdx.x % BI, t = threadIdx.x / BI;
    const int i0 = u / tiles * IP + l % IP, k2 = u % tiles * B + l / IP;
    using W1I = W1Index<N, B>;

    cx<Real> d[2][F::EM];
    F::each_in(t, [&](int e) {
        const int pos = F::in_pos(t, e);
        d[0][e] = w2.ld(WI::at(i0, 2 * pos, k2));
        d[1][e] = w2.ld(WI::at(i0, 2 * pos + 1, k2));
    });
    TwLds<Real> tl{stw};
    tl.fill(tw, N, threadIdx.x, BI * TT);  // visible after the first exchange
    ChainLds<Real, SEQ> lds{sb, BI, l};
    F::template run<2>(d, t, tl, lds);
    const int to = here(t);
    F::each_out(to, [&](int e) { w1.st(W1I::at(i0, F::out_pos(to, e), k2),
                  twfma<+1>(d[1][e], gld(byte_off(sbase(tw + F::out_pos(0, e)), uint32_t(to) * uint32_t(C::CX))), d[0][e])); });
}

// ------------------------------------------------------------------ paired W2
// Axis-1 forward over an i0 pair: unit = (i0 pair, tile of B columns k2).
// The two lines of each column (i0 = 2p and 2p + 1) are transformed one after
// the other through the same LDS exchange area; the first one's outputs wait
// in registers.  The outputs are then staged in LDS in the paired W2 order and
// stored as whole runs of 2 KB B elements, one 16-byte (FP32) pair per lane.
// Minimum waves per SIMD asked of the compiler for the paired axis-1 passes:
// with up to 8 points per thread, two 512-thread workgroups per CU (the LDS
// allows two) need at most 128 VGPRs.
constexpr int p24p_waves(int e, bool seq) { return e > 8 ? 1 : (seq ? 3 : 4); }

template <int N, int DT, int B, int TT, bool SEQ>
__global__ void __launch_bounds__((B * TT), p24p_waves(N / TT, SEQ))
p2p_fwd(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using F = TeamFFT<N, TT, Real, -1, false>;
    using WI = W2Index<N, C::BS, true>;
    static_assert(B == C::BS, "the axis-1 tile is the W2 layout tile");
    constexpr int tiles = N / B;
    constexpr int units = (N / 2) * tiles;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + (SEQ ? 1 : 2) * B * N;
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    const auto& w2 = P.w2;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    const int pr = u / tiles, tile = u % tiles;
    const int c = threadIdx.x % B, t = threadIdx.x / B;
    const int k2 = tile * B + c;
    using W1I = W1Index<N, B>;

    cx<Real> xa[F::EI], xb[F::EI], w[F::EI];
    F::each_in(t, [&](int e) {
        const int pos = F::in_pos(t, e);
        xa[e] = w1.ld(W1I::at(2 * pr, pos, k2));
        xb[e] = w1.ld(W1I::at(2 * pr + 1, pos, k2));
        w[e] = tw[pos];
    });
    TwLds<Real> tl{stw};
    tl.fill(tw, N, threadIdx.x, B * TT);  // visible after the first exchange
    ChainLds<Real, SEQ> lds{sb, B, c};
    cx<Real> ra[2][F::EM], d[2][F::EM];
    F::each_in(t, [&](int e) {
        ra[0][e] = xa[e];
        ra[1][e] = xa[e] * w[e];
    });
    F::template run<2>(ra, t, tl, lds);
    F::each_in(t, [&](int e) {
        d[0][e] = xb[e];
        d[1][e] = xb[e] * w[e];
    });
    F::template run<2>(d, t, tl, lds);
    {
        // Stage in rounds of HALF slots: element (slot, column, i0 parity) at
        // ((slot - h HALF) B + c) 2 + parity, the order of the W2 runs.
        constexpr int KB = WI::KB, RUN = 2 * KB * B;
        constexpr int HALF = SEQ ? N / 2 : N;  // slots per round
        const size_t tile0 = WI::at(2 * pr, 0, tile * B);  // start of block 0's run
#pragma unroll
        for (int h = 0; h < 2 * N / HALF; ++h) {
            __syncthreads();  // the last exchange's (or round's) reads are done
            F::each_out(t, [&](int e) {
                const int m = F::out_pos(t, e);
#pragma unroll
                for (int ch = 0; ch < 2; ++ch) {
                    const int sl = WI::slot(2 * m + ch) - h * HALF;
                    if (sl >= 0 && sl < HALF) {
                        sb[(sl * B + c) * 2] = ra[ch][e];
                        sb[(sl * B + c) * 2 + 1] = d[ch][e];
                    }
                }
            });
            __syncthreads();
            for (int g = 2 * int(threadIdx.x); g < 2 * HALF * B; g += 2 * B * TT) {
                const int gg = h * 2 * HALF * B + g;
                w2.st2(tile0 + size_t(gg / RUN) * WI::blk + gg % RUN, sb[g], sb[g + 1]);
            }
        }
    }
}

// Axis-0 pass on the paired layout.  One workgroup = SL rows of W2 (k1 and
// M-k1 when SL = 2) and B adjacent columns.  A line x (n samples along i0)
// is split by decimation in time: with w = exp(-2 pi i / 2n) and H = n/2,
//   A = DFT_H(x[2i]),  B = DFT_H(x[2i+1]),
//   C = DFT_H(x[2i] w^2i),  D = DFT_H(x[2i+1] w^(2i+1)),
// and the padded forward transform is X[2m] = A[m] + w^2m B[m],
// X[2m + 2H] = A[m] - w^2m B[m] (likewise X[2m+1], X[2m+1+2H] from C and D).
// After the multiply by K, the inverse that keeps the first n samples splits
// by decimation in frequency into four half-length inverses whose inputs are
// P = ks A + kd w^2m B and Q = ks B + kd w^-2m A (ks, kd = sum and difference
// of the kernel values of the two outputs) for the even outputs (likewise R,
// S for the odd ones); then u[2i] = P[i] + w^-2i R[i] and
// u[2i+1] = Q[i] + w^-(2i+1) S[i].  Each lane loads and stores the pair
// (x[2i], x[2i+1]) of its column as one access; all four chains advance in
// lockstep, G of them per LDS exchange round.  Column 0 is col0_conv's.
template <int N, int DT, int B, int TT, int SL, int G>
__global__ void __launch_bounds__((B * TT * SL), (TeamFFT<N / 2, TT, typename Prec<DT>::Real, -1, false>::EM <= 8 ? 4 : 2))
p3p_conv(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    constexpr int H = N / 2;
    using Ff = TeamFFT<H, TT, Real, -1, false>;
    using Fi = TeamFFT<H, TT, Real, +1, true>;
    static_assert(SL == 1 || SL == 2, "one row or a row pair per workgroup");
    static_assert(G == 4 || G == 2, "four chains exchanged all at once or two at a time");
    constexpr int tiles = N / B;
    constexpr int units = (2 / SL) * N * tiles;  // per problem
    using WI = W2Index<N, C::BS, true>;
    static_assert(C::BS % B == 0, "the axis-0 tile lies inside a W2 layout tile");
    constexpr size_t sp = WI::s0;  // stride of i0 pairs in W2
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + size_t(G) * H * B * SL;

    constexpr size_t lds_bytes = lds_p3p<N, DT, B, TT, SL, G>();
    const int first = Col0<N, DT, B * TT * SL, lds_bytes>::blocks(bt.count);
    if (int(blockIdx.x) < first) return col0_conv<N, DT, B * TT * SL, lds_bytes>(bt, int(blockIdx.x), smem);
    const int ug = xcd_unit(first);
    if (ug >= bt.count * units) return;  // whole workgroup
    const Prob<DT>& P = bt.p[ug / units];
    const auto& w2 = P.w2;
    const typename C::Kt* __restrict__ K = P.K;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    int q, tile, set;
    if constexpr (SL == 1) {
        const int item = u >> 1;
        set = u & 1;
        q = item / tiles;
        tile = item % tiles;
    } else {
        q = u / tiles;
        tile = u % tiles;
        set = (threadIdx.x / B) & 1;
    }
    const int c = threadIdx.x % B, t = threadIdx.x / (B * SL);
    const int k2 = tile * B + c;
    static_assert(WI::s0 * H * sizeof(cx<double>) < (size_t(1) << 32) &&
                      size_t(N + 1) * (N + 1) * N * sizeof(double) < (size_t(1) << 32),
                  "lane byte offsets fit 32 bits");
    // pair i = in_pos(t, e) of row q (set 0) or M-q (set 1, 2 BS elements on)
    const size_t ub = WI::at(0, q, tile * B);
    // (the lanes of column 0, which col0_conv has, take column 1's and store nothing)
    const uint32_t xl = uint32_t(2 * (k2 == 0 ? 1 : c)) + uint32_t(set) * (2 * C::BS) + uint32_t(t) * uint32_t(sp);
    auto xb = [&](int e) { return ub + size_t(Ff::in_pos(0, e)) * sp; };

    static_assert(Ff::EM == Fi::EM, "same plan, reversed");
    cx<Real> d[4][Ff::EM];
    Ff::each_in(t, [&](int e) { w2.ld_pair(xb(e), xl, d[0][e], d[1][e]); });
    // kernel values of outputs 2m, 2m+1 (m = out_pos(t, e) = t + m0) and of
    // their partners n - 2m, n - 2m - 1: a uniform base plus one of two lane
    // offsets in the tiled K row (plane q, or n for the set-1 row of pair 0)
    constexpr int KT = psn_host::k_tile(N);
    using Kt = typename C::Kt;
    const uint32_t kl = uint32_t(psn_host::k_index(N, (set != 0 && q == 0) ? N : q, 0, k2));
    const uint32_t kup = (kl + uint32_t(2 * t * KT)) * uint32_t(sizeof(Kt));
    const uint32_t kdn = (kl + uint32_t(2 * (TT - 1 - t) * KT)) * uint32_t(sizeof(Kt));
    auto kv = [&](int e, int odd, int mirror) -> Real {
        const int m0 = Ff::out_pos(0, e);
        if (!mirror) return Real(gld(byte_off(sbase(K + (2 * m0 + odd) * KT), kup)));
        return Real(gld(byte_off(sbase(K + (N - 2 * m0 - odd - 2 * (TT - 1)) * KT), kdn)));
    };
    // Stage twiddles of the half-length transforms: per-stage rows for
    // n >= 512 (filled from every other entry of the 2n table), else the
    // swizzled 2n table read at even entries.
    constexpr bool kRows = P3PRows<N>::value;
    TwLds<Real> tl{stw};
    cx<Real>* rows_i = stw + (Ff::template same_rows<Fi>() ? 0 : Ff::rows_size());
    if constexpr (kRows) {
        Ff::template fill_rows<1, 2>(stw, tw, threadIdx.x, B * TT * SL);  // visible after the first exchange
        if constexpr (!Ff::template same_rows<Fi>()) Fi::template fill_rows<1, 2>(rows_i, tw, threadIdx.x, B * TT * SL);
    } else {
        tl.fill(tw, N, threadIdx.x, B * TT * SL);   // visible after the first exchange
        if constexpr (Ff::S == 1) __syncthreads();  // no exchange: the combine reads the table
    }
    // pre-twiddles w^2i, w^(2i+1) of the pair this lane holds
    Ff::each_in(t, [&](int e) {
        const int i = Ff::in_pos(t, e);
        d[2][e] = d[0][e] * gld(tw + 2 * i);
        d[3][e] = d[1][e] * gld(tw + 2 * i + 1);
    });
    using Lds = std::conditional_t<G == 4, LdsColsN<Real, 4>, LdsColsSeq<Real, 2>>;
    Lds lds{sb, B * SL, int(threadIdx.x % (B * SL))};
    if constexpr (G == 4) lds.plane = 2 * H * B * SL;
    TwHalf<Real> th{tl};
    if constexpr (kRows) Ff::template run<4>(d, t, TwRows<Real>{stw}, lds);
    else Ff::template run<4>(d, t, th, lds);
    Ff::each_out(t, [&](int e) {
        const int m = Ff::out_pos(t, e);
        // w^2m = exp(-2 pi i m / n)
        const cx<Real> W = kRows ? gld(byte_off(sbase(tw + 2 * Ff::out_pos(0, e)), uint32_t(2 * t * C::CX)))
                                 : tl(2 * m);
#pragma unroll
        for (int odd = 0; odd < 2; ++odd) {
            const Real k0 = kv(e, odd, 0), k1 = kv(e, odd, 1);
            const Real ks = k0 + k1, kd = k0 - k1;
            const cx<Real> a = d[2 * odd][e], b = d[2 * odd + 1][e];
            // P = ks a + (kd W) b,  Q = ks b + conj(kd W) a
            const cx<Real> kw = scale(W, kd);
            d[2 * odd][e] = {fmad(ks, a.x, fmad(kw.x, b.x, -kw.y * b.y)), fmad(ks, a.y, fmad(kw.x, b.y, kw.y * b.x))};
            d[2 * odd + 1][e] = {fmad(ks, b.x, fmad(kw.x, a.x, kw.y * a.y)), fmad(ks, b.y, fmad(kw.x, a.y, -kw.y * a.x))};
        }
    });
    if constexpr (kRows) Fi::template run<4>(d, t, TwRows<Real>{rows_i}, lds);
    else Fi::template run<4>(d, t, th, lds);
    if (k2 != 0) {
        Fi::each_out(t, [&](int e) {
            const int i = Fi::out_pos(t, e);
            const cx<Real> u0 = twfma<+1>(d[2][e], gld(tw + 2 * i), d[0][e]);
            const cx<Real> u1 = twfma<+1>(d[3][e], gld(tw + 2 * i + 1), d[1][e]);
            w2.st_pair(xb(e), xl, u0, u1);
        });
    }
}

// Axis-1 inverse over an i0 pair: unit = (i0 pair, tile of B columns k2).
// Each lane loads rows 2j and 2j+1 of its column as (i0 = 2p, 2p + 1) pairs;
// the two lines are inverted one after the other and combined as
// y = y_even + w^-j y_odd.
template <int N, int DT, int B, int TT, bool SEQ>
__global__ void __launch_bounds__((B * TT), p24p_waves(N / TT, SEQ))
p4p_inv(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using F = TeamFFT<N, TT, Real, +1, false>;
    using WI = W2Index<N, C::BS, true>;
    static_assert(B == C::BS, "the axis-1 tile is the W2 layout tile");
    constexpr int tiles = N / B;
    constexpr int units = (N / 2) * tiles;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    cx<Real>* stw = sb + (SEQ ? 1 : 2) * B * N;
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    const auto& w2 = P.w2;
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units;
    const int pr = u / tiles, tile = u % tiles;
    const int c = threadIdx.x % B, t = threadIdx.x / B;
    const int k2 = tile * B + c;
    using W1I = W1Index<N, B>;

    cx<Real> a[2][F::EM], b[2][F::EM];
    F::each_in(t, [&](int e) {
        const int pos = F::in_pos(t, e);
        w2.ld_pair(WI::at(2 * pr, 2 * pos, k2), a[0][e], b[0][e]);
        w2.ld_pair(WI::at(2 * pr, 2 * pos + 1, k2), a[1][e], b[1][e]);
    });
    TwLds<Real> tl{stw};
    tl.fill(tw, N, threadIdx.x, B * TT);  // visible after the first exchange
    if constexpr (F::S == 1) __syncthreads();  // no exchange: the combine reads the table
    ChainLds<Real, SEQ> lds{sb, B, c};
    // the combine twiddles w^-j come from the LDS table (fewer live registers)
    F::template run<2>(a, t, tl, lds);
    F::each_out(t, [&](int e) {
        const int j = F::out_pos(t, e);
        w1.st(W1I::at(2 * pr, j, k2), twfma<+1>(a[1][e], tl(j), a[0][e]));
    });
    const int tb = here(t);  // the addresses of the second line are formed anew: no spills at 128 VGPRs
    F::template run<2>(b, tb, tl, lds);
    F::each_out(tb, [&](int e) {
        const int j = F::out_pos(tb, e);
        w1.st(W1I::at(2 * pr + 1, j, k2), twfma<+1>(b[1][e], tl(j), b[0][e]));
    });
}

// ------------------------------------------------------------------ small cubes
// Axes 1 and 0 of one k2 plane in one launch, for small n (PlaneCfg): a workgroup
// holds the n x n plane of one k2 and the outputs k1 = 2m + p of one parity p in
// LDS, rows m; what the five passes do in P2, P3, column 0 and P4.  The two
// parities' inverses along axis 1 go to the two halves of W2 as [p][i0][k2][i1]
// and P5 adds them, so that 2n workgroups share a plane's work (n would leave
// most CUs idle) and none waits for another.  Latency bound: few waves, a chain
// of 8 to 10 exchanges; the kernel values are loaded first of all.
//   1  line i0 along i1: DFT_n(x w^(p i1)), written to row m, column i0
//   2  row m along i0: both parities of k0, x K, inverse, back to row m
//      (k2 = 0, the packed column: Z' = a Z(k) + b conj(Z(-k)), the partner row
//      and position read from LDS, as in col0_conv)
//   3  line i0 along m: inverse, times w^-(p i1)
// A row's own LDS is the exchange area of the team that has it; the row pitch
// of 8 mod 16 spreads a column's accesses over the banks.
template <int N, int DT>
__global__ void __launch_bounds__((PlaneCfg<N, DT>::threads)) plane_conv(const Batch<DT> bt) {
    using PC = PlaneCfg<N, DT>;
    using Real = typename PC::Real;
    using Kt = typename Prec<DT>::Kt;
    constexpr int T = PC::T, LP = PC::pitch();
    using Ff = TeamFFT<N, T, Real, -1, false>;
    using Fr = TeamFFT<N, T, Real, +1, true>;   // starts from Ff's output layout
    using Fi = TeamFFT<N, T, Real, +1, false>;
    constexpr int KT = psn_host::k_tile(N);
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    const int ug = xcd_unit();
    constexpr int units = 2 * N;  // per problem
    if (ug >= bt.count * units) return;  // whole workgroup
    const Prob<DT>& P = bt.p[ug / units];
    const cx<Real>* __restrict__ tw = P.tw;
    const int u = ug % units, k2 = u >> 1, p = u & 1;
    const int t = threadIdx.x % T, ln = threadIdx.x / T;  // ln: i0 in steps 1 and 3, m in step 2
    const size_t line = (size_t(ln) * N + k2) * N;        // of W1 and of W2's halves

    cx<Real> a[1][Ff::EM];
    Ff::each_in(t, [&](int e) { a[0][e] = P.w1.ld(line + Ff::in_pos(t, e)); });
    TwLds<Real> tl{sb + N * LP};
    tl.fill(tw, N, threadIdx.x, PC::threads);  // visible after the first barrier
    static_assert(LdsLine<Real>::slots(N) <= LP, "a padded line fits its row");
    LdsLine<Real> row{sb + ln * LP};
    if (p) Ff::each_in(t, [&](int e) { a[0][e] = a[0][e] * gld(tw + Ff::in_pos(t, e)); });
    Ff::template run<1>(a, t, tl, row);
    __syncthreads();  // the last exchange's reads are done
    Ff::each_out(t, [&](int e) { sb[Ff::out_pos(t, e) * LP + ln] = a[0][e]; });
    __syncthreads();

    const int k1 = 2 * ln + p, k1f = k1 <= N ? k1 : 2 * N - k1;
    const Kt* const Krow = P.K + psn_host::k_index(N, k1f, 0, k2);
    auto fold = [](int k) { return k <= N ? k : 2 * N - k; };
    Real kk[2][Ff::EO];
    Ff::each_out(t, [&](int e) {
        const int m = Ff::out_pos(t, e);
        kk[0][e] = Real(gld(Krow + fold(2 * m) * KT));
        kk[1][e] = Real(gld(Krow + fold(2 * m + 1) * KT));
    });
    cx<Real> d[2][Ff::EM];
    Ff::each_in(t, [&](int e) {
        const int i = Ff::in_pos(t, e);
        d[0][e] = sb[ln * LP + i];
        d[1][e] = d[0][e] * tl(i);
    });
    Ff::template run<2>(d, here(t), tl, row);
    if (k2 == 0) {  // whole workgroup
        const Kt* const Kbr = P.Kb + size_t(k1f) * (N + 1);
        const int pm = p ? N - 1 - ln : (N - ln) % N;  // row of -k1
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            __syncthreads();
            Ff::each_out(t, [&](int e) { sb[ln * LP + Ff::out_pos(t, e)] = d[q][e]; });
            __syncthreads();
            Ff::each_out(t, [&](int e) {
                const int m = Ff::out_pos(t, e);
                const cx<Real> z = conj(sb[pm * LP + (q ? N - 1 - m : (N - m) % N)]);
                d[q][e] = scale(d[q][e], kk[q][e]) + scale(z, Real(gld(Kbr + fold(2 * m + q))));
                kk[q][e] = Real(1);
            });
        }
    }
    Fr::template run_scaled<2>(d, here(t), tl, row, kk);
    __syncthreads();  // the last exchange's reads are done
    Ff::each_in(t, [&](int e) {
        const int i = Ff::in_pos(t, e);
        sb[ln * LP + i] = twfma<+1>(d[1][e], tl(i), d[0][e]);
    });
    __syncthreads();

    Fi::each_in(t, [&](int e) { a[0][e] = sb[Fi::in_pos(t, e) * LP + ln]; });
    Fi::template run<1>(a, here(t), tl, row);  // its first exchange waits for every line's loads
    const size_t out = size_t(p) * N * N * N + line;
    Fi::each_out(t, [&](int e) {
        const int i = Fi::out_pos(t, e);
        P.w2.st(out + i, p ? mul_conj(a[0][e], tl(i)) : a[0][e]);
    });
}

// ------------------------------------------------------------------ P5
template <int N, int DT>
__global__ void __launch_bounds__((Cfg<N, DT>::LC * Cfg<N, DT>::T))
p5_c2r(const Batch<DT> bt) {
    using C = Cfg<N, DT>;
    using Real = typename C::Real;
    using Io = typename C::Io;
    using F = TeamFFT<N, C::T, Real, +1, false>;
    constexpr int units = N * N / C::LC;  // per problem
    extern __shared__ __align__(16) unsigned char smem[];
    cx<Real>* sb = reinterpret_cast<cx<Real>*>(smem);
    const int ug = xcd_unit();
    if (ug >= bt.count * units) return;
    const Prob<DT>& P = bt.p[ug / units];
    const Work<DT>& w1 = P.w1;
    Io* __restrict__ u = P.u;
    const cx<Real>* __restrict__ tw = P.tw;
    const int t = threadIdx.x % C::T, ln = threadIdx.x / C::T;
    const int line0 = (ug % units) * C::LC;  // first line of the workgroup; all share i0
    const int i0 = line0 / N, i1b = line0 % N;
    const size_t base = (size_t(line0) + ln) * N;  // of this thread's line in u

    // Y[k] = (V[k] + conj V[n-k]) + i (V[k] - conj V[n-k]) w^-k; V[0], V[n] real and packed.
    // The workgroup's LC lines of W1 are read with consecutive threads on
    // consecutive addresses (element j is line j / BS % LC, k = j / (BS * LC) * BS
    // + j % BS) into the LDS rows; each line's team then takes V[k] and its
    // partner V[n-k] from there (the first exchange of the transform waits
    // before reusing the rows).
    constexpr int BL = C::BS;
    using W1I = W1Index<N, BL>;
    TwLds<Real> tl{sb + C::LC * C::NP};
    tl.fill(tw, N, threadIdx.x, C::LC * C::T);
    using TO = TileOrder<N, C::LC, C::T, BL>;
    cx<Real> d[F::EM];
    static_assert(F::EI == F::E && F::EO == F::E, "every lane holds E elements");
#pragma unroll
    for (int q = 0; q < F::E; ++q) {
        int lj, k0, off;
        TO::at(int(threadIdx.x), q, lj, k0, off);
        const size_t i = W1I::at(i0, i1b + lj, k0 + off);
        if constexpr (PlaneCfg<N, DT>::value) d[q] = P.w2.ld(i) + P.w2.ld(size_t(N) * N * N + i);
        else d[q] = w1.ld(i);
    }
#pragma unroll
    for (int q = 0; q < F::E; ++q) {
        int lj, k0, off;
        TO::at(int(threadIdx.x), q, lj, k0, off);
        LdsRows<Real>{sb + lj * C::NP}.put2(k0, off, d[q]);
    }
    __syncthreads();
    LdsRows<Real> lds{sb + ln * C::NP};
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int pos = F::in_pos(t, e);
        const int pc = pos - t;  // compile-time part of the position
        const cx<Real> a = lds.get2(t, pc);
        if (pos == 0) {
            d[e] = {a.x + a.y, a.x - a.y};
        } else {
            const cx<Real> b = conj(lds.get2(N - t, -pc));
            d[e] = (a + b) + rot<+1>(mul_conj(a - b, tl(pos)));
        }
    }
    F::run1(d, t, tl, lds);
    // z[j] = u[2j] + i u[2j+1]; only j < n/2 lies inside the box
#pragma unroll
    for (int e = 0; e < F::E; ++e) {
        const int pos = F::out_pos(t, e);
        if (pos < N / 2) {
            u[base + 2 * pos] = Io(d[e].x);
            u[base + 2 * pos + 1] = Io(d[e].y);
        }
    }
}

// ------------------------------------------------------------------ launcher
// Kernels needing more than 64 KB of dynamic LDS must say so once.
inline bool allow_lds(const void* fn, size_t bytes) {
    if (bytes <= 65536) return true;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) == hipSuccess;
}

// ------------------------------------------------------------------ schedules
// Tile shapes of the strided passes: B adjacent columns per workgroup, TT
// threads per line.  Each pass has four candidates; the autotuner times them once
// per (n, precision) and keeps the fastest.  A candidate that does not fit (LDS,
// threads, radix plan) or is not there for a size is candidate 0 again: the axis-0
// pass has three of its own at FP64 n = 128, 256 and 512, two at FP64 and one at FP32
// n = 162, P2/P4 two at n = 162.
//   P2/P4 (they keep the W2 layout tile, B = BS), n a power of two: the two chains
//     together in FP32, one after the other in FP64 (LaneW2); twice the elements
//     per thread; the other way of the two; four elements.  With an odd factor, the
//     chains one after the other but for the third: 8 elements on a power-of-two
//     team, on N / 8 threads, together, and all odd factors in every thread (12 or
//     20 elements).
//   P3: one row with the chains one after the other; the row pair k1, M-k1; the
//     chains together, or with an odd factor (in FP64 only 3) the row pair on 12
//     or 20 elements, the fastest for many densities per launch (13 of 160^3 FP32
//     0.51 against 0.54 ms, while one density takes 67 against 51 us; n = 96 and 192:
//     p3_conv); with an odd factor, 8 elements on N / 8 threads.
// The one-chain exchange stages the W2 runs of P2 in two rounds of n slots.
struct TileV {
    int B, TT;
    int SL = 1;        // rows per workgroup (the axis-0 pass only)
    bool SEQ = false;  // exchange the two chains one at a time (half the LDS)
    bool EARLY = false;  // the axis-0 pass holds w and, in FP64, K from its start (p3_conv)
};

// ip: i0 per workgroup of the axis-1 passes; the axis-0 pass has SL rows per
// workgroup instead and its teams split into i0 pairs (ip = 2)
constexpr bool tile_ok(int N, TileV v, int cxbytes, int ip, bool axis0) {
    const int lines = v.B * (axis0 ? v.SL : ip);
    return v.B >= 1 && v.TT >= 1 && (v.SL == 1 || v.SL == 2) && N % v.B == 0 && v.TT <= N && (mid_plan(N) || N % v.TT == 0) &&
           lines * v.TT <= 1024 && ((v.SEQ ? 1 : 2) * lines * N + ((2 * N + 15) & ~15)) * cxbytes <= kMaxLdsP3 &&
           (!axis0 || v.TT % ip == 0) && team_plan(N, N / v.TT).n > 0 && N / v.TT <= 20;
}

template <int N, int DT>
struct Sched {
    using C = Cfg<N, DT>;
    static constexpr TileV d24{C::BS, C::T24, 1, mid_plan(N) || C::IP == 2}, d3{C::BP3, C::T3, N % 4 ? 2 : 1, true};  // 162: the row pair, whose 108 threads hold column 0's teams
    static constexpr int odd = odd_part(N), eo = 4 * odd;
    static constexpr bool mid = mid_plan(N);
    static constexpr int tm = N / elems8(N);
    static constexpr TileV pick24(TileV v) { return tile_ok(N, v, C::CX, C::IP, false) ? v : d24; }
    static constexpr TileV pick3(TileV v) { return tile_ok(N, v, C::CX, C::IP, true) && C::BS % v.B == 0 ? v : d3; }
    static constexpr TileV v24[psn_host::kScheduleCandidates] = {
        d24, pick24(mid ? TileV{C::BS, tm, 1, true} : TileV{C::BS, N / 16}),
        pick24(TileV{C::BS, C::T24, 1, !d24.SEQ}),
        pick24(mid ? TileV{C::BS, N / eo, 1, true} : TileV{C::BS, N / 4})};
    static constexpr TileV v3[psn_host::kScheduleCandidates] = {
        d3, pick3(TileV{C::BP3, C::T3, 2, true}), pick3(mid && (DT == DT_F32 || odd == 3) ? TileV{C::BP3, N / eo, 2, true, odd == 3} : TileV{C::BP3, C::T3, d3.SL}),
        mid && N % 4 == 0 ? pick3(TileV{C::BP3, tm, 1, true}) : d3};
    static_assert(tile_ok(N, d24, C::CX, C::IP, false) && tile_ok(N, d3, C::CX, C::IP, true), "default tiles must fit");
};

// Axis-0 tiles on the paired layout: B columns, TT threads per half line
// (n/2 points), SL rows per workgroup, G chains per LDS exchange round.
struct TileP {
    int B, TT;
    int SL = 1;
    int G = 4;
};

constexpr bool tilep_ok(int N, TileP v, int cxbytes) {
    return v.B >= 1 && v.TT >= 1 && (v.SL == 1 || v.SL == 2) && (v.G == 2 || v.G == 4) && N % v.B == 0 &&
           (mid_plan(N / 2) || (N / 2) % v.TT == 0) && v.B * v.TT * v.SL <= 1024 &&
           (size_t(v.G) * (N / 2) * v.B * v.SL + ((2 * N + 15) & ~15)) * cxbytes <= size_t(kMaxLdsP3) &&
           team_plan(N / 2, N / 2 / v.TT).n > 0 && N / 2 / v.TT <= 16;
}
constexpr TileP pick_tilep(int N, TileP v, TileP dflt, int cxbytes, int layout_tile) {
    return (tilep_ok(N, v, cxbytes) && layout_tile % v.B == 0) ? v : dflt;
}

template <int N, int DT>
struct SchedP {
    using C = Cfg<N, DT>;
    static constexpr int H = N / 2;
    static constexpr int T = strided_team(H);
    static constexpr int e4 = H >= 4 ? 4 : H, e16 = H >= 16 ? 16 : H;
    // eight points per chain and thread, two chains per exchange round (all
    // four at once halves the workgroups per CU and measured 45 % slower at
    // n = 512); the row pair k1, M-k1 per workgroup; four points per chain
    // (twice the threads, one more exchange; with an odd factor: no idle
    // threads in the outer stages instead); sixteen points per chain (one
    // exchange fewer, half the threads; with an odd factor: the same, and the
    // row pair)
    static constexpr TileP d3{C::BP3, T, 1, 2};
    static constexpr TileP v3[psn_host::kScheduleCandidates] = {
        d3, pick_tilep(N, TileP{C::BP3, T, 2, 2}, d3, C::CX, C::BS),
        pick_tilep(N, TileP{C::BP3, mid_plan(H) ? H / elems8(H) : H / e4, 1, 2}, d3, C::CX, C::BS),
        pick_tilep(N, mid_plan(H) ? TileP{C::BP3, H / elems8(H), 2, 2} : TileP{C::BP3, H / e16, 1, 2}, d3,
                   C::CX, C::BS)};
};

// What the candidate indices of this size and precision name, in 32 bits (FNV-1a
// over the tiles), for records that outlive the library: an index recorded by a
// build with another table would name another tile.  0: one form, no candidates.
template <int N, int DT>
constexpr uint32_t sched_tag() {
    if constexpr (PlaneCfg<N, DT>::value) {
        return 0;
    } else {
        uint32_t h = 2166136261u;
        auto add = [&](int v) { h = (h ^ uint32_t(v)) * 16777619u; };
        auto tile = [&](const TileV& v) { add(v.B), add(v.TT), add(v.SL), add(v.SEQ), add(v.EARLY); };
        add(Cfg<N, DT>::IP);
        for (const TileV& v : Sched<N, DT>::v24) tile(v);
        if constexpr (PairW2<N, DT>::value)
            for (const TileP& v : SchedP<N, DT>::v3) add(v.B), add(v.TT), add(v.SL), add(v.G);
        else
            for (const TileV& v : Sched<N, DT>::v3) tile(v);
        return h ? h : 1;
    }
}
template <int DT>
uint32_t sched_tag_of(int n) {
    switch (n) {
#define PSN_CASE(NN) \
    case NN: return sched_tag<NN, DT>();
        PSN_FOR_EACH_SIZE(PSN_CASE)
#undef PSN_CASE
        default: return 0;
    }
}

// LDS of the strided passes: the exchange area plus the stage twiddle rows
template <int N, int DT, int B, int TT, bool SEQ>
constexpr size_t lds_p24() {
    return (size_t(SEQ ? 1 : 2) * Cfg<N, DT>::IP * B * N + TwLds<typename Cfg<N, DT>::Real>::slots(N)) * Cfg<N, DT>::CX;
}

template <int N, int DT, int I>
hipError_t launch_p2(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileV v = Sched<N, DT>::v24[I];
    const size_t lds = lds_p24<N, DT, v.B, v.TT, v.SEQ>();
    static const bool ok = allow_lds(reinterpret_cast<const void*>(&p2_fwd<N, DT, v.B, v.TT, v.SEQ>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p2_fwd<N, DT, v.B, v.TT, v.SEQ>), dim3(xcd_grid(long(bt.count) * (N / Cfg<N, DT>::IP) * (N / v.B))),
                       dim3(Cfg<N, DT>::IP * v.B * v.TT), lds, s, bt);
    return hipSuccess;
}

template <int N, int DT, int I>
hipError_t launch_p4(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileV v = Sched<N, DT>::v24[I];
    const size_t lds = lds_p24<N, DT, v.B, v.TT, v.SEQ>();
    static const bool ok = allow_lds(reinterpret_cast<const void*>(&p4_inv<N, DT, v.B, v.TT, v.SEQ>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p4_inv<N, DT, v.B, v.TT, v.SEQ>), dim3(xcd_grid(long(bt.count) * (N / Cfg<N, DT>::IP) * (N / v.B))),
                       dim3(Cfg<N, DT>::IP * v.B * v.TT), lds, s, bt);
    return hipSuccess;
}

template <int N, int DT, int I>
hipError_t launch_p3(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileV v = Sched<N, DT>::v3[I];
    constexpr size_t lds = lds_p3<N, DT, v.B, v.TT, v.SL, v.SEQ>();
    using G0 = Col0<N, DT, v.B * v.TT * v.SL, lds>;
    static const bool ok = allow_lds(reinterpret_cast<const void*>(&p3_conv<N, DT, v.B, v.TT, v.SL, v.SEQ, v.EARLY>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p3_conv<N, DT, v.B, v.TT, v.SL, v.SEQ, v.EARLY>),
                       dim3(G0::blocks(bt.count) + xcd_grid(long(bt.count) * (2 / v.SL) * N * (N / v.B))),
                       dim3(v.B * v.TT * v.SL), lds, s, bt);
    return hipSuccess;
}

// the axis-1 passes on the paired layout: the same tiles, one i0 pair per workgroup
template <int N, int DT, int I>
hipError_t launch_p2p(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileV v = Sched<N, DT>::v24[I];
    const size_t lds = lds_p24<N, DT, v.B, v.TT, v.SEQ>();
    static const bool ok = allow_lds(reinterpret_cast<const void*>(&p2p_fwd<N, DT, v.B, v.TT, v.SEQ>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p2p_fwd<N, DT, v.B, v.TT, v.SEQ>), dim3(xcd_grid(long(bt.count) * (N / 2) * (N / v.B))),
                       dim3(v.B * v.TT), lds, s, bt);
    return hipSuccess;
}

template <int N, int DT, int I>
hipError_t launch_p4p(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileV v = Sched<N, DT>::v24[I];
    const size_t lds = lds_p24<N, DT, v.B, v.TT, v.SEQ>();
    static const bool ok = allow_lds(reinterpret_cast<const void*>(&p4p_inv<N, DT, v.B, v.TT, v.SEQ>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p4p_inv<N, DT, v.B, v.TT, v.SEQ>), dim3(xcd_grid(long(bt.count) * (N / 2) * (N / v.B))),
                       dim3(v.B * v.TT), lds, s, bt);
    return hipSuccess;
}

template <int N, int DT, int I>
hipError_t launch_p3p(const Batch<DT>& bt, hipStream_t s) {
    constexpr TileP v = SchedP<N, DT>::v3[I];
    static_assert(tilep_ok(N, v, Cfg<N, DT>::CX), "paired axis-0 tile must fit");
    constexpr size_t lds = lds_p3p<N, DT, v.B, v.TT, v.SL, v.G>();
    using G0 = Col0<N, DT, v.B * v.TT * v.SL, lds>;
    static const bool ok =
        allow_lds(reinterpret_cast<const void*>(&p3p_conv<N, DT, v.B, v.TT, v.SL, v.G>), lds);
    if (!ok) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((p3p_conv<N, DT, v.B, v.TT, v.SL, v.G>),
                       dim3(G0::blocks(bt.count) + xcd_grid(long(bt.count) * (2 / v.SL) * N * (N / v.B))),
                       dim3(v.B * v.TT * v.SL), lds, s, bt);
    return hipSuccess;
}

template <int N, int DT>
hipError_t launch_p24(const Batch<DT>& bt, hipStream_t s, int v, bool forward) {
    if constexpr (PairW2<N, DT>::value) {
        switch (v) {
            case 1: return forward ? launch_p2p<N, DT, 1>(bt, s) : launch_p4p<N, DT, 1>(bt, s);
            case 2: return forward ? launch_p2p<N, DT, 2>(bt, s) : launch_p4p<N, DT, 2>(bt, s);
            case 3: return forward ? launch_p2p<N, DT, 3>(bt, s) : launch_p4p<N, DT, 3>(bt, s);
            default: return forward ? launch_p2p<N, DT, 0>(bt, s) : launch_p4p<N, DT, 0>(bt, s);
        }
    } else {
        switch (v) {
            case 1: return forward ? launch_p2<N, DT, 1>(bt, s) : launch_p4<N, DT, 1>(bt, s);
            case 2: return forward ? launch_p2<N, DT, 2>(bt, s) : launch_p4<N, DT, 2>(bt, s);
            case 3: return forward ? launch_p2<N, DT, 3>(bt, s) : launch_p4<N, DT, 3>(bt, s);
            default: return forward ? launch_p2<N, DT, 0>(bt, s) : launch_p4<N, DT, 0>(bt, s);
        }
    }
}

template <int N, int DT>
hipError_t launch_p3v(const Batch<DT>& bt, hipStream_t s, int v) {
    if constexpr (PairW2<N, DT>::value) {
        switch (v) {
            case 1: return launch_p3p<N, DT, 1>(bt, s);
            case 2: return launch_p3p<N, DT, 2>(bt, s);
            case 3: return launch_p3p<N, DT, 3>(bt, s);
            default: return launch_p3p<N, DT, 0>(bt, s);
        }
    } else {
        switch (v) {
            case 1: return launch_p3<N, DT, 1>(bt, s);
            case 2: return launch_p3<N, DT, 2>(bt, s);
            case 3: return launch_p3<N, DT, 3>(bt, s);
            default: return launch_p3<N, DT, 0>(bt, s);
        }
    }
}

// Enqueue the kernels of one solve (five; three for PlaneCfg sizes) for bt.count
// problems of size N with schedule (v24 for P2/P4, v3 for P3).
template <int N, int DT>
hipError_t solve_n(const Batch<DT>& bt, hipStream_t s, hipEvent_t* ev, int v24, int v3) {
    using C = Cfg<N, DT>;
    constexpr size_t tws = TwLds<typename C::Real>::slots(N);
    const size_t lds_rows = (size_t(C::LC) * C::NP + tws) * C::CX;
    const long cnt = bt.count;
    auto mark = [&](int i) {
        if (ev) (void)hipEventRecord(ev[i], s);
    };
    static const bool lds_ok = allow_lds(reinterpret_cast<const void*>(&p1_r2c<N, DT>), lds_rows) &&
                               allow_lds(reinterpret_cast<const void*>(&p5_c2r<N, DT>), lds_rows);
    if (!lds_ok) return hipErrorInvalidValue;
    [[maybe_unused]] hipError_t e;
    mark(0);
    hipLaunchKernelGGL((p1_r2c<N, DT>), dim3(xcd_grid(cnt * N * N / C::LC)), dim3(C::LC * C::T), lds_rows, s, bt);
    mark(1);
    if constexpr (PlaneCfg<N, DT>::value) {
        using PC = PlaneCfg<N, DT>;
        static const bool ok = allow_lds(reinterpret_cast<const void*>(&plane_conv<N, DT>), PC::lds);
        if (!ok) return hipErrorInvalidConfiguration;
        mark(2);
        hipLaunchKernelGGL((plane_conv<N, DT>), dim3(xcd_grid(cnt * 2 * N)), dim3(PC::threads), PC::lds, s, bt);
        mark(3);
        mark(4);
    } else {
        if ((e = launch_p24<N, DT>(bt, s, v24, true)) != hipSuccess) return e;
        mark(2);
        if ((e = launch_p3v<N, DT>(bt, s, v3)) != hipSuccess) return e;
        mark(3);
        if ((e = launch_p24<N, DT>(bt, s, v24, false)) != hipSuccess) return e;
        mark(4);
    }
    hipLaunchKernelGGL((p5_c2r<N, DT>), dim3(xcd_grid(cnt * N * N / C::LC)), dim3(C::LC * C::T), lds_rows, s, bt);
    mark(5);
    return hipGetLastError();
}

// Time the candidates of the strided passes on one problem's workspace and return
// the fastest indices.  Its contents are what earlier work left: the ranking comes
// out as on a density, though the times may not (the axis-0 pass of 32 of n = 192
// FP64 took 3.31 ms on stale values and 3.65 on white noise, at a lower clock).
template <int N, int DT>
hipError_t tune_n(const Batch<DT>& bt, hipStream_t s, int* best24, int* best3) {
    *best24 = *best3 = 0;
    if constexpr (PlaneCfg<N, DT>::value) {
        return hipSuccess;  // one schedule
    } else {
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t e = hipEventCreate(&a);
    if (e == hipSuccess) e = hipEventCreate(&b);
    // one timed launch sequence
    auto timed = [&](auto&& launch, float* ms) -> hipError_t {
        hipError_t le = hipEventRecord(a, s);
        if (le == hipSuccess) le = launch();
        if (le == hipSuccess) le = hipEventRecord(b, s);
        if (le == hipSuccess) le = hipEventSynchronize(b);
        if (le == hipSuccess) le = hipEventElapsedTime(ms, a, b);
        return le;
    };
    // Candidates are timed in interleaved rounds (so clock changes hit all of
    // them alike); each keeps its best time; round 0 only warms up.
    constexpr int NC = psn_host::kScheduleCandidates;
    float t24[NC], t3[NC];
    for (int v = 0; v < NC; ++v) t24[v] = t3[v] = 1e30f;
    for (int round = 0; round < 7 && e == hipSuccess; ++round) {
        for (int v = 0; v < NC && e == hipSuccess; ++v) {
            float x = 0.f, y = 0.f;
            e = timed([&] {
                    hipError_t r = launch_p24<N, DT>(bt, s, v, true);
                    return r == hipSuccess ? launch_p24<N, DT>(bt, s, v, false) : r;
                }, &x);
            if (e == hipSuccess) e = timed([&] { return launch_p3v<N, DT>(bt, s, v); }, &y);
            if (e == hipSuccess && round > 0) {
                t24[v] = x < t24[v] ? x : t24[v];
                t3[v] = y < t3[v] ? y : t3[v];
            }
        }
    }
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    if (e != hipSuccess) return e;
    for (int v = 1; v < NC; ++v) {
        if (t24[v] < 0.97f * t24[*best24]) *best24 = v;
        if (t3[v] < 0.97f * t3[*best3]) *best3 = v;
    }
    return hipSuccess;
    }
}

template <int DT>
Prob<DT> prob_of(const psn_host::Slot& sl) {
    using Real = typename Prec<DT>::Real;
    using Io = typename Prec<DT>::Io;
    using Kt = typename Prec<DT>::Kt;
    Prob<DT> pr{};
    pr.rho = static_cast<const Io*>(sl.rho);
    pr.u = static_cast<Io*>(sl.u);
    if constexpr (DT == DT_SPLIT) {
        pr.w1 = {static_cast<uint32_t*>(sl.W1)};
        pr.w2 = {static_cast<cx<double>*>(sl.W2)};
    } else {
        pr.w1 = {static_cast<cx<Real>*>(sl.W1)};
        pr.w2 = {static_cast<cx<Real>*>(sl.W2)};
    }
    pr.K = static_cast<const Kt*>(sl.plan->K);
    pr.Kb = static_cast<const Kt*>(sl.plan->Kb);
    pr.tw = static_cast<const cx<Real>*>(sl.plan->tw);
    return pr;
}

// Slots [0, count) share n, precision and schedule (the caller groups them
// so); v24/v3 >= 0 override the plans' schedule.
template <int DT>
hipError_t solve_group(const psn_host::Slot* slots, int count, hipStream_t s, hipEvent_t* ev, int v24o = -1,
                       int v3o = -1) {
    const int v24 = v24o >= 0 ? v24o : slots[0].plan->sched24, v3 = v3o >= 0 ? v3o : slots[0].plan->sched3;
    for (int base = 0; base < count; base += kMaxBatch) {
        Batch<DT> bt{};
        bt.count = count - base < kMaxBatch ? count - base : kMaxBatch;
        for (int i = 0; i < bt.count; ++i) bt.p[i] = prob_of<DT>(slots[base + i]);
        hipError_t e = hipErrorInvalidValue;
        switch (slots[0].plan->n) {
#define PSN_CASE(NN) \
    case NN: e = solve_n<NN, DT>(bt, s, ev, v24, v3); break;
            PSN_FOR_EACH_SIZE(PSN_CASE)
#undef PSN_CASE
            default: break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Time the candidates on a batch group's own entries (their workspaces in
// the batch arena, with stale contents): the first kMaxBatch of them in one
// launch, as the batch runs them.
template <int DT>
hipError_t tune_slots(const psn_host::Slot* slots, int count, hipStream_t s, int* best24, int* best3) {
    Batch<DT> bt{};
    bt.count = count < kMaxBatch ? count : kMaxBatch;
    for (int i = 0; i < bt.count; ++i) bt.p[i] = prob_of<DT>(slots[i]);
    switch (slots[0].plan->n) {
#define PSN_CASE(NN) \
    case NN: return tune_n<NN, DT>(bt, s, best24, best3);
        PSN_FOR_EACH_SIZE(PSN_CASE)
#undef PSN_CASE
        default: return hipErrorInvalidValue;
    }
}

template <int DT>
hipError_t tune_plan(const psn_plan* p, hipStream_t s, int* best24, int* best3) {
    Batch<DT> bt{};
    bt.count = 1;
    bt.p[0] = prob_of<DT>(psn_host::Slot{p, nullptr, nullptr, p->W1, p->W2});
    switch (p->n) {
#define PSN_CASE(NN) \
    case NN: return tune_n<NN, DT>(bt, s, best24, best3);
        PSN_FOR_EACH_SIZE(PSN_CASE)
#undef PSN_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace psn

// Defines the per-precision entry points of one compilation unit.
#define PSN_DEFINE_PRECISION(DTV, SUFFIX)                                                                       \
    namespace psn_host {                                                                                        \
    hipError_t launch_group_##SUFFIX(const Slot* slots, int count, hipStream_t stream, hipEvent_t* ev, int v24, \
                                     int v3) {                                                                  \
        return psn::solve_group<DTV>(slots, count, stream, ev, v24, v3);                                        \
    }                                                                                                           \
    hipError_t tune_slots_##SUFFIX(const Slot* slots, int count, hipStream_t stream, int* best24, int* best3) { \
        return psn::tune_slots<DTV>(slots, count, stream, best24, best3);                                       \
    }                                                                                                           \
    hipError_t tune_##SUFFIX(const psn_plan* p, hipStream_t stream, int* best24, int* best3) {                \
        return psn::tune_plan<DTV>(p, stream, best24, best3);                                                   \
    }                                                                                                           \
    uint32_t sched_tag_##SUFFIX(int n) { return psn::sched_tag_of<DTV>(n); }                                    \
    }
