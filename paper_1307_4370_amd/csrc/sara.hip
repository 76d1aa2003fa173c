// SARA dictionary Psi = (1/sqrt q) [Dirac, Db1, ..., Db8] (Sec. 3.3) and its
// adjoint, as periodised orthonormal 2-D DWTs in the Mallat layout.
//
// Analysis, one launch per level for all selected Daubechies bases at once
// (the bases are independent and computed in parallel, as in Sec. 5): a
// workgroup owns a TO x TO tile of each of the four sub-bands, stages the
// (2 TO + Lf - 2)^2 input region (periodic) in LDS, filters rows then columns
// and writes LL to the next level's input (or the coefficient plane at the
// last level) and LH / HL / HH to their Mallat positions.
//
// The final coefficients can go through an epilogue instead of a plain store:
// the SDMM update of the l1 term (Algorithm 1 steps 7-9 for i = 1,
// soft threshold of eq. prox1), which also accumulates f1 = sum w |alpha|.
//
// Synthesis is the exact transpose, columns then rows; its last level sums all
// bases and the Dirac plane for one output tile, so Psi alpha is written once.
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace riop {

constexpr int kMaxTaps = 16;
constexpr int kTO = 16;  // output tile side per sub-band (analysis) / half the output tile (synthesis)

// Tiles of TO cover a band of `half`; the last of a row or column may be partial:
// its region wraps as any other and its outputs past the band are dropped.
// WHOLE kernels serve bands that the tiles divide: the tests for a partial tile
// cost 3 % of the analysis and 1 % of the synthesis.
__host__ __device__ constexpr int tiles_of(int half, int TO) { return (int)((unsigned)(half + TO - 1) / TO); }

template <typename R> struct AnaArgs {
    const C<R> *in;     // level input: x (level 1, shared) or per-basis LL slot
    long in_bstride;    // complex elements between bases' inputs (0 when shared)
    C<R> *ll_out;       // next-level LL slot (per basis) or nullptr at the last level
    long ll_bstride;
    C<R> *alpha;        // coefficient planes (q x n x n)
    const R *filt;      // [9][2][kMaxTaps] low / high pass
    int basis[8];       // Daubechies order of each launched basis
    int plane[8];       // plane index of each launched basis
    int n, s, TO, last;  // image side, level side, tile side, whether this is the last level
    int nbases;         // Daubechies bases launched
    int dirac_plane;    // level 1: plane of the Dirac basis, done by blockIdx.y = nbases (-1: none)
    int dirac_blocks;   // its blocks (the rest of that row of blocks is idle)
    R scale;            // 1/sqrt(q) applied to final coefficients
    int *flag;          // level 1: set to 1 where the input holds a NaN or Inf (nullptr: not checked)
    int prox;
    Prox1<R> px;
};

// Block sum of f1 into this block's own partial slot (no atomics; the
// consumer adds the slots in a fixed order).
__device__ inline void block_add_f1(double f1, double *part) {
    __shared__ double red[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) f1 += __shfl_xor(f1, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = f1;
    __syncthreads();
    if (threadIdx.x == 0) part[(long)blockIdx.y * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// A final coefficient c (unscaled): stored, or the prox epilogue with its
// operands z = z1[j] and w (the weight) already loaded.
template <typename R>
__device__ inline void emit_coef(const AnaArgs<R> &a, long j, C<R> c, C<R> z, R w, double &f1) {
    c = cscale<R>(c, a.scale);
    if (!a.prox) {
        a.alpha[j] = c;
        return;
    }
    const R lam = (R)(*a.px.gamma) * w;
    const C<R> v = cadd<R>(c, z);
    const R mag = sqrt(v.x * v.x + v.y * v.y);
    const R sc = mag > lam ? R(1) - lam / mag : R(0);
    const C<R> r = cscale<R>(v, sc);
    const C<R> zn = csub<R>(v, r);
    a.px.z1[j] = zn;
    a.px.w1[j] = csub<R>(r, zn);
    f1 += (double)w * sqrt((double)c.x * c.x + (double)c.y * c.y);
}

// One level of the analysis for one basis (blockIdx.y) and one TO x TO tile
// of each sub-band (blockIdx.x), 256 threads; at level 1 blockIdx.y = nbases
// copies the Dirac plane.
// Bound by LDS traffic and latency at level 1 (the output is written once, the
// 8 bases read one input through the caches).  The filter length is a template
// parameter of the tile, so that every tap loop unrolls and its LDS reads are
// issued together; a thread filters 4 neighbouring outputs of a row from one
// window of 2 * 4 + Lf - 2 inputs (16-byte reads, free of bank conflicts at the
// even row stride) and 2 of a column from Lf + 2.  Only the low-pass taps are
// loaded: g[m] = (-1)^m h[Lf - 1 - m].
// 1024^2, 4 levels, 9 bases, FP32: level 1 42 -> 28 us, all levels and the
// Dirac plane 77 -> 48 us (a run-time tap count put a branch before every
// read, one output and one read per tap).
template <int TO> constexpr int ana_stride() { return TO == 16 ? 20 : TO; }  // row-filtered planes: spreads 4 rows over the banks
template <int TO> constexpr int ana_region() { return 2 * TO + kMaxTaps - 2; }

// Element i >= 0 of a periodic line of s elements; i < 2 s unless `tiny` (a
// wave-uniform flag: the division stays off the path of all but tiny levels).
__device__ inline int wrap(int i, int s, bool tiny) {
    if (tiny) return i % s;
    return i - (i >= s ? s : 0);
}

template <typename R, int TO, bool WHOLE, int NB>
__device__ inline void ana_tile(const AnaArgs<R> &a, int bi, C<R> *smem) {
    constexpr int Lf = 2 * NB, IR = 2 * TO + Lf - 2, IRM = ana_region<TO>(), RS = ana_stride<TO>();
    constexpr int VL = TO < 4 ? TO : 4;  // outputs per thread along a row
    constexpr int VK = TO < 2 ? TO : 2;  // and along a column
    const int s = a.s, half = s >> 1, n = a.n;
    const int tiles = tiles_of(half, TO);
    const int k0 = (blockIdx.x / tiles) * TO, l0 = (blockIdx.x % tiles) * TO;
    C<R> *reg = smem;                            // [IRM][IRM]
    C<R> *rows = reg + IRM * IRM;                // [low, high][IRM][RS]
    const C<R> *in = a.in + bi * a.in_bstride;
    const R *ht = a.filt + NB * 2 * kMaxTaps;
    R h[Lf];
#pragma unroll
    for (int m = 0; m < Lf; ++m) h[m] = ht[m];
    auto g = [&](int m) { return (m & 1) ? -h[Lf - 1 - m] : h[Lf - 1 - m]; };

    // This thread's column outputs: VK rows of column l of the low or high
    // plane, low (t = 0) and high (t = 1) filtered.  Their prox operands are
    // loaded before the filtering.
    constexpr int kItems = 2 * (TO / VK) * TO;
    const int p = threadIdx.x / (kItems / 2), kq = threadIdx.x % (kItems / 2);
    const int k = (kq / TO) * VK, l = kq % TO;
    const bool mine = threadIdx.x < kItems && (WHOLE || (l0 + l < half && k0 + k < half));
    // Rows past the first are inside with it unless the band's side is odd.
    const bool odd = half & 1;
    auto inside = [&](int v) { return WHOLE || v == 0 || !odd || k0 + k + v < half; };
    const long base = (long)a.plane[bi] * n * n + (long)(k0 + k) * n + p * half + l0 + l;
    auto place = [&](int v, int t) { return base + (long)(v + t * half) * n; };
    C<R> zq[VK][2];
    R wq[VK][2];
#pragma unroll
    for (int v = 0; v < VK; ++v)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            zq[v][t] = mk<R>(0, 0);
            wq[v][t] = R(1);
            if (a.prox && mine && inside(v) && (p || t || a.last)) {  // the low-low band goes to the next level
                zq[v][t] = a.px.z1[place(v, t)];
                if (a.px.weights) wq[v][t] = a.px.weights[place(v, t)];
            }
        }

    // The region (at most 46 wide): thread (ty, tx) stages column tx of rows
    // ty, ty + 4, ..., all loads issued before any is stored.
    {
        const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
        constexpr int RPT = (IR + 3) / 4;
        const bool tiny = WHOLE ? IR > s : 2 * (tiles - 1) * TO + IR > 2 * s;
        const unsigned gc = wrap(2 * l0 + min(tx, IR - 1), s, tiny);
        C<R> st[RPT];
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            st[i] = in[(unsigned)wrap(2 * k0 + min(ty + 4 * i, IR - 1), s, tiny) * s + gc];
        if (a.flag && bi == 0) {
            FiniteCheck<R> fc;
#pragma unroll
            for (int i = 0; i < RPT; ++i) fc.add(st[i]);
            fc.report(a.flag);
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = ty + 4 * i;
            if (tx < IR && r < IR) reg[r * IRM + tx] = st[i];
        }
    }
    __syncthreads();
    // Rows (axis 1): low[r][l] = sum_m h[m] in[r][2 l + m], high with g.
    for (int idx = threadIdx.x; idx < IR * (TO / VL); idx += 256) {
        const int r = idx / (TO / VL), q = (idx % (TO / VL)) * VL;
        constexpr int NI = 2 * VL + Lf - 2;
        C<R> v[NI];
        const C<R> *row = reg + r * IRM + 2 * q;
        if constexpr (sizeof(R) == 4) {
#pragma unroll
            for (int m = 0; m < NI; m += 2) {
                const float4 t = *reinterpret_cast<const float4 *>(row + m);
                v[m] = mk<R>(t.x, t.y);
                v[m + 1] = mk<R>(t.z, t.w);
            }
        } else {
#pragma unroll
            for (int m = 0; m < NI; ++m) v[m] = row[m];
        }
#pragma unroll
        for (int o = 0; o < VL; ++o) {
            R lr = 0, li = 0, hr = 0, hi = 0;
#pragma unroll
            for (int m = 0; m < Lf; ++m) {
                lr += h[m] * v[2 * o + m].x;
                li += h[m] * v[2 * o + m].y;
                hr += g(m) * v[2 * o + m].x;
                hi += g(m) * v[2 * o + m].y;
            }
            rows[r * RS + q + o] = mk<R>(lr, li);
            rows[(IRM + r) * RS + q + o] = mk<R>(hr, hi);
        }
    }
    __syncthreads();
    // Columns (axis 0).
    double f1 = 0.0;
    if (mine) {
        constexpr int NI = 2 * VK + Lf - 2;
        C<R> v[NI];
        const C<R> *col = rows + (p * IRM + 2 * k) * RS + l;
#pragma unroll
        for (int m = 0; m < NI; ++m) v[m] = col[m * RS];
#pragma unroll
        for (int o = 0; o < VK; ++o) {
            if (!inside(o)) break;
            R lr = 0, li = 0, hr = 0, hi = 0;
#pragma unroll
            for (int m = 0; m < Lf; ++m) {
                lr += h[m] * v[2 * o + m].x;
                li += h[m] * v[2 * o + m].y;
                hr += g(m) * v[2 * o + m].x;
                hi += g(m) * v[2 * o + m].y;
            }
            if (p == 0 && !a.last) a.ll_out[bi * a.ll_bstride + (long)(k0 + k + o) * half + l0 + l] = mk<R>(lr, li);
            else emit_coef<R>(a, place(o, 0), mk<R>(lr, li), zq[o][0], wq[o][0], f1);
            emit_coef<R>(a, place(o, 1), mk<R>(hr, hi), zq[o][1], wq[o][1], f1);
        }
    }
    if (a.prox) block_add_f1(f1, a.px.f1_part);
}

// Dirac coefficient j = base + i of pixel value x.
template <typename R>
__device__ inline void dirac_coef(const AnaArgs<R> &a, long i, C<R> x, double &f1) {
    const long j = (long)a.dirac_plane * a.n * a.n + i;
    const C<R> z = a.prox ? a.px.z1[j] : mk<R>(0, 0);
    const R w = a.prox && a.px.weights ? a.px.weights[j] : R(1);
    emit_coef<R>(a, j, x, z, w, f1);
}

template <typename R, int TO, bool WHOLE> __global__ void __launch_bounds__(256) dwt_analysis(AnaArgs<R> a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C<R> *smem = reinterpret_cast<C<R> *>(smem_raw);
    const int bi = blockIdx.y;
    if (bi == a.nbases) {  // level 1: the Dirac plane, alpha_0 = x / sqrt(q)
        if ((int)blockIdx.x >= a.dirac_blocks) return;
        const int n = a.n, tiles = tiles_of(n >> 1, TO);
        const long N = (long)n * n;
        double f1 = 0.0;
        // A block per whole tile copies its tile, whose input the other bases read.
        if (WHOLE && a.dirac_blocks == (int)gridDim.x) {
            const int i0 = (blockIdx.x / tiles) * 2 * TO, j0 = (blockIdx.x % tiles) * 2 * TO;
#pragma unroll
            for (int u = 0; u < (4 * TO * TO + 255) / 256; ++u) {
                const int e = threadIdx.x + 256 * u;
                if (e >= 4 * TO * TO) break;
                const long i = (long)(i0 + e / (2 * TO)) * n + j0 + e % (2 * TO);
                dirac_coef<R>(a, i, a.in[i], f1);
            }
            if (a.prox) block_add_f1(f1, a.px.f1_part);
            return;
        }
        const long step = a.dirac_blocks * 256L;
        for (long i0 = (long)blockIdx.x * 256 + threadIdx.x; i0 < N; i0 += 4 * step) {
            C<R> x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = i0 + u * step < N ? a.in[i0 + u * step] : mk<R>(0, 0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * step < N) dirac_coef<R>(a, i0 + u * step, x[u], f1);
        }
        if (a.prox) block_add_f1(f1, a.px.f1_part);
        return;
    }
    switch (a.basis[bi]) {
        case 1: ana_tile<R, TO, WHOLE, 1>(a, bi, smem); break;
        case 2: ana_tile<R, TO, WHOLE, 2>(a, bi, smem); break;
        case 3: ana_tile<R, TO, WHOLE, 3>(a, bi, smem); break;
        case 4: ana_tile<R, TO, WHOLE, 4>(a, bi, smem); break;
        case 5: ana_tile<R, TO, WHOLE, 5>(a, bi, smem); break;
        case 6: ana_tile<R, TO, WHOLE, 6>(a, bi, smem); break;
        case 7: ana_tile<R, TO, WHOLE, 7>(a, bi, smem); break;
        default: ana_tile<R, TO, WHOLE, 8>(a, bi, smem); break;
    }
}

// A dictionary of the Dirac basis alone.
template <typename R> __global__ void __launch_bounds__(256) dirac_analysis(AnaArgs<R> a) {
    const long N = (long)a.n * a.n;
    double f1 = 0.0;
    FiniteCheck<R> fc;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x) {
        const C<R> x = a.in[i];
        fc.add(x);
        dirac_coef<R>(a, i, x, f1);
    }
    if (a.flag) fc.report(a.flag);
    if (a.prox) block_add_f1(f1, a.px.f1_part);
}

template <typename R> struct SynArgs {
    const C<R> *alpha;  // coefficient planes (q x n x n)
    const C<R> *ll_in;  // per-basis LL slot for this level (nullptr at the coarsest level)
    long ll_in_bstride;
    C<R> *ll_out;       // per-basis output slot (levels > 1)
    long ll_out_bstride;
    C<R> *x;            // final image (level 1)
    const R *filt;
    int basis[8];
    int plane[8];
    int nbases;
    int dirac_plane;    // -1 if the Dirac basis is not selected
    int n, s, TO, coarsest;
    R scale;
    int *flag;          // set to 1 where alpha holds a NaN or Inf (nullptr: not checked)
};

// Synthesis of one (2 TO)^2 output tile of basis DbN by 256 threads (a group;
// thread t), from the four KR^2 sub-band regions, KR = TO + N - 1, staged in LDS:
// columns (axis 0), then rows.  As in the analysis, N is a template parameter of
// the filter steps, so their loops unroll and issue their LDS reads together.
// Output rows (and columns) 2 r and 2 r + 1 read the same N inputs with the even
// and the odd taps; a thread forms two such pairs from N + 1 inputs.
// Bound by LDS reads and, where there are few tiles, by latency: the last level
// sums all bases for a tile, so NG groups per block each take every NG-th basis
// (their sums are added in a fixed order at the end).
// 512^2, 4 levels, 9 bases, FP64: last level 36 -> 25 us, all 63 -> 48;
// 1024^2, FP32: last level 44 -> 38 us, all 74 -> 64.
template <int TO> constexpr int syn_kr() { return TO + kMaxTaps / 2 - 1; }  // the widest region
template <int TO> constexpr int syn_cells() { return 4 * syn_kr<TO>() * syn_kr<TO>() + 4 * TO * syn_kr<TO>(); }
template <int TO> constexpr int syn_pairs() { return TO < 2 ? 1 : 2; }

// The regions' loads: thread (t / 32, t % 32) takes column t % 32 of rows t / 32,
// t / 32 + 8 and t / 32 + 16 (KR <= 23) of each band.
template <typename R> struct SynRegion {
    C<R> ll[3], lh[3], hl[3], hh[3];
};

template <typename R, bool WHOLE>
__device__ inline void syn_load(const SynArgs<R> &a, int bi, int t, int i0, int j0, SynRegion<R> &v) {
    const int N = a.basis[bi], n = a.n, half = a.s >> 1, TO = a.TO, KR = TO + N - 1;
    const int c = t & 31, r0 = t >> 5;
    if (c >= KR) return;
    // The region starts at -7 at least and ends at half + TO - 2 at most: one period
    // either way is enough, but for tiny levels.
    const bool tiny = half < (WHOLE ? kMaxTaps / 2 : kTO), last = !WHOLE && max(i0, j0) / 2 + TO > half;
    auto wrap_band = [&](int k) {
        if (tiny) return (k % half + half) % half;
        if (last) k -= k >= half ? half : 0;
        return k + (k < 0 ? half : 0);
    };
    const int kst = i0 / 2 - N + 1;
    const unsigned l = wrap_band(j0 / 2 - N + 1 + c);
    // Band origins, uniform; offsets inside a plane are 32-bit.
    const C<R> *plane = a.alpha + (long)a.plane[bi] * n * n;
    const C<R> *lh = plane + half, *hl = plane + (long)half * n, *hh = hl + half;
    const C<R> *ll = a.coarsest ? plane : a.ll_in + bi * a.ll_in_bstride;
    const unsigned ls = a.coarsest ? n : half;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int r = r0 + 8 * q;
        if (r < KR) {
            const unsigned k = wrap_band(kst + r), o = k * (unsigned)n + l;
            v.ll[q] = ll[k * ls + l];
            v.lh[q] = lh[o];
            v.hl[q] = hl[o];
            v.hh[q] = hh[o];
        }
    }
    if (a.flag) {
        FiniteCheck<R> fc;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (r0 + 8 * q < KR) {
                if (a.coarsest) fc.add(v.ll[q]);
                fc.add(v.lh[q]);
                fc.add(v.hl[q]);
                fc.add(v.hh[q]);
            }
        fc.report(a.flag);
    }
}

// LDS of a group: the regions LL, HL, LH, HH (KR^2 each), then the
// column-filtered low and high planes (2 TO x KR each).
template <typename R>
__device__ inline void syn_stage(const SynArgs<R> &a, int bi, int t, const SynRegion<R> &v, C<R> *smem) {
    const int KR = a.TO + a.basis[bi] - 1, c = t & 31, r0 = t >> 5, KR2 = KR * KR;
    if (c >= KR) return;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int r = r0 + 8 * q;
        if (r < KR) {
            smem[r * KR + c] = v.ll[q];
            smem[KR2 + r * KR + c] = v.hl[q];
            smem[2 * KR2 + r * KR + c] = v.lh[q];
            smem[3 * KR2 + r * KR + c] = v.hh[q];
        }
    }
}

// NP output pairs (even: 2 i, odd: 2 i + 1, i = i0 .. i0 + NP - 1) of the 1-D
// synthesis from low lo[i0 ..] and high hi[i0 ..] inputs `stride` apart, the
// first of which is entry i0 of a region that starts N - 1 entries early.
template <typename R, int N, int NP>
__device__ inline void syn_pairs_1d(const R (&h)[2 * N], const C<R> *lo, const C<R> *hi, int stride,
                                    C<R> (&out)[2 * NP]) {
    auto g = [&](int m) { return (m & 1) ? -h[2 * N - 1 - m] : h[2 * N - 1 - m]; };
    C<R> l[N + NP - 1], u[N + NP - 1];
#pragma unroll
    for (int i = 0; i < N + NP - 1; ++i) {
        l[i] = lo[i * stride];
        u[i] = hi[i * stride];
    }
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int par = 0; par < 2; ++par) {
            R re = 0, im = 0;
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const int m = 2 * t + par, r = q + N - 1 - t;
                re += h[m] * l[r].x + g(m) * u[r].x;
                im += h[m] * l[r].y + g(m) * u[r].y;
            }
            out[2 * q + par] = mk<R>(re, im);
        }
}

template <typename R, int TO, int N> __device__ inline void syn_cols(const R *filt, int t, C<R> *smem) {
    constexpr int KR = TO + N - 1, KR2 = KR * KR, NP = syn_pairs<TO>(), per = (TO / NP) * KR;
    R h[2 * N];
#pragma unroll
    for (int m = 0; m < 2 * N; ++m) h[m] = filt[N * 2 * kMaxTaps + m];
    C<R> *mid = smem + 4 * KR2;
    for (int w = t; w < 2 * per; w += 256) {  // low plane from (LL, HL), high plane from (LH, HH)
        const int p = w / per, q = w - p * per, rp = (q / KR) * NP, c = q % KR;
        const C<R> *lo = smem + 2 * p * KR2 + rp * KR + c;
        C<R> out[2 * NP];
        syn_pairs_1d<R, N, NP>(h, lo, lo + KR2, KR, out);
#pragma unroll
        for (int i = 0; i < 2 * NP; ++i) mid[(p * 2 * TO + 2 * rp + i) * KR + c] = out[i];
    }
}

// Output columns of thread t: row ii, columns jj .. jj + 2 NP - 1 (false: none; those
// past the level are dropped by the caller).
template <int TO> __device__ inline bool syn_place(int t, int &ii, int &jj) {
    constexpr int NP = syn_pairs<TO>(), per = TO / NP;
    ii = t / per;
    jj = 2 * NP * (t - ii * per);
    return t < 2 * TO * per;
}

template <typename R, int TO, int N>
__device__ inline void syn_rows(const R *filt, int t, const C<R> *smem, C<R> (&acc)[2 * syn_pairs<TO>()]) {
    constexpr int KR = TO + N - 1, NP = syn_pairs<TO>();
    R h[2 * N];
#pragma unroll
    for (int m = 0; m < 2 * N; ++m) h[m] = filt[N * 2 * kMaxTaps + m];
    int ii, jj;
    if (!syn_place<TO>(t, ii, jj)) return;
    const C<R> *lo = smem + 4 * KR * KR + ii * KR + jj / 2;
    C<R> out[2 * NP];
    syn_pairs_1d<R, N, NP>(h, lo, lo + 2 * TO * KR, 1, out);
#pragma unroll
    for (int i = 0; i < 2 * NP; ++i) acc[i] = cadd<R>(acc[i], out[i]);
}

#define SYN_BASES(FN, N, ...)                          \
    switch (N) {                                       \
        case 1: FN<R, TO, 1>(__VA_ARGS__); break;      \
        case 2: FN<R, TO, 2>(__VA_ARGS__); break;      \
        case 3: FN<R, TO, 3>(__VA_ARGS__); break;      \
        case 4: FN<R, TO, 4>(__VA_ARGS__); break;      \
        case 5: FN<R, TO, 5>(__VA_ARGS__); break;      \
        case 6: FN<R, TO, 6>(__VA_ARGS__); break;      \
        case 7: FN<R, TO, 7>(__VA_ARGS__); break;      \
        default: FN<R, TO, 8>(__VA_ARGS__); break;     \
    }

// Levels > 1: one basis per blockIdx.y, writes the finer LL slot.
template <typename R, int TO, bool WHOLE> __global__ void __launch_bounds__(256) dwt_synthesis(SynArgs<R> a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C<R> *smem = reinterpret_cast<C<R> *>(smem_raw);
    constexpr int TS = 2 * TO, NA = 2 * syn_pairs<TO>();
    const int bi = blockIdx.y, t = threadIdx.x, tiles = tiles_of(a.s, TS);
    const int i0 = (blockIdx.x / tiles) * TS, j0 = (blockIdx.x % tiles) * TS;
    SynRegion<R> v;
    syn_load<R, WHOLE>(a, bi, t, i0, j0, v);
    syn_stage<R>(a, bi, t, v, smem);
    __syncthreads();
    SYN_BASES(syn_cols, a.basis[bi], a.filt, t, smem)
    __syncthreads();
    C<R> acc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = mk<R>(0, 0);
    SYN_BASES(syn_rows, a.basis[bi], a.filt, t, smem, acc)
    int ii, jj;
    if (syn_place<TO>(t, ii, jj) && (WHOLE || (i0 + ii < a.s && j0 + jj < a.s))) {
        C<R> *out = a.ll_out + bi * a.ll_out_bstride + (long)(i0 + ii) * a.s + j0 + jj;
        const bool odd = !WHOLE && (a.s & 2);  // else the NA columns are inside together
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if (i < 2 || !odd || j0 + jj + i < a.s) out[i] = acc[i];
    }
}

// Level 1: sum of all bases (and the Dirac plane) for one output tile.  Group g
// takes bases g, 2 NG - 1 - g, 2 NG + g, ... (long and short filters in turn); the
// next basis's regions load while the current one is filtered.
template <typename R, int TO, bool WHOLE, int NG>
__global__ void __launch_bounds__(256 * NG, sizeof(R) == 4 ? 4 : 2) dwt_synthesis_final(SynArgs<R> a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int TS = 2 * TO, NA = 2 * syn_pairs<TO>();
    const int g = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;
    C<R> *all = reinterpret_cast<C<R> *>(smem_raw), *smem = all + g * syn_cells<TO>();
    const int n = a.n, tiles = tiles_of(n, TS);
    const int i0 = (blockIdx.x / tiles) * TS, j0 = (blockIdx.x % tiles) * TS;
    auto basis = [&](int step) { return step * NG + ((step & 1) ? NG - 1 - g : g); };
    int ii, jj;
    const bool mine = syn_place<TO>(t, ii, jj) && (WHOLE || (i0 + ii < n && j0 + jj < n));
    const long o = (long)(i0 + ii) * n + j0 + jj;
    const bool odd = !WHOLE && (n & 2);  // else the NA columns are inside together
    auto inside = [&](int i) { return i < 2 || !odd || j0 + jj + i < n; };
    C<R> acc[NA], dirac[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = dirac[i] = mk<R>(0, 0);
    if (a.dirac_plane >= 0 && g == 0 && mine) {
        FiniteCheck<R> fc;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            if (inside(i)) dirac[i] = a.alpha[(long)a.dirac_plane * n * n + o + i];
            fc.add(dirac[i]);
        }
        if (a.flag) fc.report(a.flag);
    }
    SynRegion<R> v;
    if (basis(0) < a.nbases) syn_load<R, WHOLE>(a, basis(0), t, i0, j0, v);
    const int steps = (a.nbases + NG - 1) / NG;
    for (int step = 0; step < steps; ++step) {
        const int bi = basis(step), bn = basis(step + 1);
        const bool on = bi < a.nbases;
        __syncthreads();  // the previous basis's readers are done
        if (on) syn_stage<R>(a, bi, t, v, smem);
        if (bn < a.nbases) syn_load<R, WHOLE>(a, bn, t, i0, j0, v);
        __syncthreads();
        if (on) SYN_BASES(syn_cols, a.basis[bi], a.filt, t, smem)
        __syncthreads();
        if (on) SYN_BASES(syn_rows, a.basis[bi], a.filt, t, smem, acc)
    }
    if constexpr (NG > 1) {  // [group - 1][output][thread]
        __syncthreads();
        if (g > 0) {
#pragma unroll
            for (int i = 0; i < NA; ++i) all[((g - 1) * NA + i) * 256 + t] = acc[i];
        }
        __syncthreads();
        if (g > 0) return;
        for (int k = 0; k < NG - 1; ++k)
#pragma unroll
            for (int i = 0; i < NA; ++i) acc[i] = cadd<R>(acc[i], all[(k * NA + i) * 256 + t]);
    }
    if (!mine) return;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        C<R> z = acc[i];
        if (a.dirac_plane >= 0) z = cadd<R>(z, dirac[i]);
        if (inside(i)) a.x[o + i] = cscale<R>(z, a.scale);
    }
}
#undef SYN_BASES

template <typename R> __global__ void dirac_only_synthesis(SynArgs<R> a, long N) {
    FiniteCheck<R> fc;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x) {
        const C<R> z = a.alpha[(long)a.dirac_plane * N + i];
        fc.add(z);
        a.x[i] = cscale<R>(z, a.scale);
    }
    if (a.flag) fc.report(a.flag);
}

// ---------------------------------------------------------------------------
// Host side.

// Tile side: the smallest power of two whose tiles over `rows` bases are at most
// `blocks`, up to kTO and the one that covers the band.  Small tiles have the
// shorter chain while their blocks are all in flight, large ones the least overlap
// and the fewest idle threads; tiles that divide the band (the rule before) have
// neither where its side has few factors of 2: 9 bases, one level, FP32 / FP64, 972^2
// (band 486, tiles of 2 -> 16) analysis 719 -> 33 us / 1300 -> 64, synthesis
// 960 -> 48 / 1900 -> 78; 216^2 (108, tiles of 4 -> 16) 16 -> 9 / 24 -> 9 and 24 -> 15 / 37 -> 21.
static int tile_side(int half, int rows, int blocks) {
    int TO = 1;
    while (TO < kTO && TO < half && (long)tiles_of(half, TO) * tiles_of(half, TO) * rows > blocks) TO *= 2;
    return TO;
}

// Two blocks per CU.  Analysis, 8 bases, tiles of 8 / 16, FP32 and FP64: bands of 36 (200 blocks of
// 8) 6.3 / 6.9 us and 6.5 / 7.2, of 64 (512) 6.4 / 6.6 and 6.8 / 7.1, of 96 (1152)
// 7.4 / 7.1 and 9.6 / 8.0; one basis, tiles of 4 / 16: 48 (144) 6.3 / 6.8 and 6.4 / 7.2.
static int level_tile(int half, int nb) { return tile_side(half, nb, 512); }

// The analysis of many bases keeps the side of its first level where that divides
// the band: every side is another kernel, whose code (a path per basis) is cold where
// the levels above run other tiles (512^2, 4 levels, 8 bases, FP64, tiles of 8 and 4 on
// the last two levels 42.2 -> 46.4 us, 1024^2 of 8 on the last one 98.9 -> 101).  With
// one basis the smaller tiles are still faster (576^2, 6 levels 45.4 -> 42.5).
// With the l1 prox every block has a partial of f1 in the solver's workspace, so
// there the tiles are no smaller than the largest that divides the band: a plan
// needs no more memory than with those (5 KB of 1.8 MB at 64^2).
static int analysis_tile(int n, int half, int nb, bool prox) {
    const int first = level_tile(n >> 1, nb), TO = nb > 3 && half % first == 0 ? first : level_tile(half, nb);
    return prox ? std::max(TO, std::min(kTO, half & -half)) : TO;
}

// The last synthesis level sums all bases in a block, so blocks are fewer and longer.
// FP64, 8 bases, tiles of 1 / 2 / 4 / 8 / 16: bands of 12 15.1 / 19.3 / 19.1 / 22.0 / 20.7
// us, of 32 27.9 / 17.8 / 18.9 / 20.1 / 19.8, of 128 (256 tiles of 8) - / - / 36.5 / 19.5 /
// 20.3, of 144 (324) - / - / 54.8 / 24.6 / 21.8.  In FP32 tiles of kTO share the bases among
// four groups, which pays from two bases on: 48 13.8 us, 17.2 with tiles of 4 (one
// basis 8.0, 6.6).
template <typename R> static int final_tile(int half, int nb) {
    const bool groups = sizeof(R) == 4 && nb > 1 && 2 * half > kTO;
    return groups ? kTO : tile_side(half, 1, 256);
}

static size_t ll_offset(int n, int level) {
    // Slot of the LL produced by level `level` (1-based): sum of sizes of the earlier slots.
    size_t off = 0;
    for (int j = 1; j < level; ++j) {
        const size_t s = (size_t)(n >> j);
        off += s * s;
    }
    return off;
}

static int dirac_blocks(int n) { return (int)std::min<long>(((long)n * n + 255) / 256, 4096); }

// Blocks of level 1 that copy the Dirac plane: one per tile, but where the tiles
// are small no more than have 256 pixels each (every block has a partial of f1).
static int dirac_row_blocks(int n, int nb, bool prox) {
    const int tiles = tiles_of(n >> 1, analysis_tile(n, n >> 1, nb, prox));
    return std::min(tiles * tiles, dirac_blocks(n));
}

int psi_adj_blocks(const riop_plan *p) {
    const int n = p->n, dirac = p->mask & 1, nb = p->q - dirac;
    if (nb == 0) return dirac_blocks(n);
    int total = dirac ? dirac_row_blocks(n, nb, true) : 0;
    for (int lev = 1; lev <= p->L; ++lev) {
        const int half = (n >> (lev - 1)) >> 1, tiles = tiles_of(half, analysis_tile(n, half, nb, true));
        total += tiles * tiles * nb;
    }
    return total;
}

template <typename R, int TO> static size_t ana_lds() {
    return sizeof(C<R>) * (size_t)(ana_region<TO>() * (ana_region<TO>() + 2 * ana_stride<TO>()));
}
// Groups per block of the last synthesis level: with fewer tiles than fill the
// GPU (4 blocks of 256 threads per CU in single, 2 in double precision) the
// bases of a tile run side by side.
template <typename R> static int syn_groups(int tiles) {
    if (sizeof(R) == 8) return tiles >= 512 ? 1 : 2;
    return tiles >= 1024 ? 1 : tiles >= 512 ? 2 : 4;
}

template <typename R, int TO, bool WHOLE>
static void launch_synthesis(const SynArgs<R> &a, int nb, bool final_level, hipStream_t st) {
    const int tiles = tiles_of(a.s >> 1, TO), blocks = tiles * tiles;
    const size_t lds = sizeof(C<R>) * (size_t)syn_cells<TO>();
    if (!final_level) {
        hipLaunchKernelGGL((dwt_synthesis<R, TO, WHOLE>), dim3(blocks, nb), dim3(256), lds, st, a);
        return;
    }
#define FINAL(NG) \
    hipLaunchKernelGGL((dwt_synthesis_final<R, TO, WHOLE, NG>), dim3(blocks), dim3(256 * NG), NG * lds, st, a)
    switch (TO < 16 ? 1 : syn_groups<R>(blocks)) {
        case 1: FINAL(1); break;
        case 2:
            if constexpr (TO == 16) FINAL(2);
            break;
        default:
            if constexpr (TO == 16 && sizeof(R) == 4) FINAL(4);
    }
#undef FINAL
}

template <typename R>
static void psi_adj_impl(riop_plan *p, const void *x, void *alpha, const Prox1<R> *px, int *flag, hipStream_t st) {
    const int n = p->n, L = p->L;
    AnaArgs<R> a{};
    a.alpha = static_cast<C<R> *>(alpha);
    a.filt = p->filters.as<R>();
    a.n = n;
    a.scale = (R)p->scale_q;
    a.prox = px != nullptr;
    if (px) a.px = *px;
    a.in = static_cast<const C<R> *>(x);
    a.flag = flag;
    a.dirac_plane = -1;
    for (int i = 0; i < p->q; ++i) {
        if (p->bases[i] == 0) {
            a.dirac_plane = i;
        } else {
            a.basis[a.nbases] = p->bases[i];
            a.plane[a.nbases] = i;
            ++a.nbases;
        }
    }
    const int nb = a.nbases;
    if (nb == 0) {
        TimedScope ts(p, KK_PSI_ADJ, st);
        hipLaunchKernelGGL(dirac_analysis<R>, dim3(dirac_blocks(n)), dim3(256), 0, st, a);
        RIOP_HIP(hipGetLastError());
        return;
    }
    C<R> *ll = p->ll.as<C<R>>();
    for (int lev = 1; lev <= L; ++lev) {
        const int s = n >> (lev - 1), half = s >> 1;
        a.s = s;
        a.TO = analysis_tile(n, half, nb, a.prox);
        a.last = lev == L;
        if (lev > 1) {
            a.in = ll + ll_offset(n, lev - 1);
            a.in_bstride = (long)p->ll_stride;
            a.flag = nullptr;
        }
        a.ll_out = a.last ? nullptr : ll + ll_offset(n, lev);
        a.ll_bstride = (long)p->ll_stride;
        const int tiles = tiles_of(half, a.TO);
        TimedScope ts(p, KK_PSI_ADJ, st);
        a.dirac_blocks = lev == 1 && a.dirac_plane >= 0 ? dirac_row_blocks(n, nb, a.prox) : 0;
        const dim3 grid(tiles * tiles, nb + (a.dirac_blocks > 0 ? 1 : 0));
        switch (a.TO) {
#define ANA(T, WHOLE) hipLaunchKernelGGL((dwt_analysis<R, T, WHOLE>), grid, dim3(256), (ana_lds<R, T>()), st, a)
#define ANA_TILE(T)                      \
    case T:                              \
        if (half % T == 0) ANA(T, true); \
        else ANA(T, false);              \
        break;
            ANA_TILE(16) ANA_TILE(8) ANA_TILE(4) ANA_TILE(2)
            default: ANA(1, true);
#undef ANA_TILE
#undef ANA
        }
        RIOP_HIP(hipGetLastError());
        a.px.f1_part += a.prox ? (long)tiles * tiles * nb + a.dirac_blocks : 0;
    }
}

template <typename R> void launch_psi_adj(riop_plan *p, const void *x, void *alpha, hipStream_t st, int *flag) {
    psi_adj_impl<R>(p, x, alpha, nullptr, flag, st);
}

template <typename R>
void launch_psi_adj_prox(riop_plan *p, const void *x, const Prox1<R> &px, hipStream_t st) {
    psi_adj_impl<R>(p, x, p->sd.w1.ptr /* unused for prox stores */, &px, nullptr, st);
}

template <typename R> void launch_psi(riop_plan *p, const void *alpha, void *x, hipStream_t st, int *flag) {
    const int n = p->n, L = p->L;
    SynArgs<R> a{};
    a.alpha = static_cast<const C<R> *>(alpha);
    a.filt = p->filters.as<R>();
    a.n = n;
    a.scale = (R)p->scale_q;
    a.x = static_cast<C<R> *>(x);
    a.flag = flag;
    a.dirac_plane = -1;
    int nb = 0;
    for (int i = 0; i < p->q; ++i) {
        if (p->bases[i] == 0) {
            a.dirac_plane = i;
        } else {
            a.basis[nb] = p->bases[i];
            a.plane[nb] = i;
            ++nb;
        }
    }
    a.nbases = nb;
    if (nb == 0) {
        const long N = (long)n * n;
        const int blocks = (int)std::min<long>((N + 255) / 256, 4096);
        TimedScope ts(p, KK_PSI, st);
        hipLaunchKernelGGL(dirac_only_synthesis<R>, dim3(blocks), dim3(256), 0, st, a, N);
        RIOP_HIP(hipGetLastError());
        return;
    }
    C<R> *ll = p->ll.as<C<R>>();
    for (int lev = L; lev >= 1; --lev) {
        const int s = n >> (lev - 1), half = s >> 1;
        a.s = s;
        a.TO = lev == 1 ? final_tile<R>(half, nb) : level_tile(half, nb);
        a.coarsest = lev == L;
        a.ll_in = a.coarsest ? nullptr : ll + ll_offset(n, lev);
        a.ll_in_bstride = (long)p->ll_stride;
        TimedScope ts(p, KK_PSI, st);
        if (lev > 1) {
            a.ll_out = ll + ll_offset(n, lev - 1);
            a.ll_out_bstride = (long)p->ll_stride;
        }
        switch (a.TO) {
#define SYN_TILE(T)                                                       \
    case T:                                                               \
        if (half % T == 0) launch_synthesis<R, T, true>(a, nb, lev == 1, st); \
        else launch_synthesis<R, T, false>(a, nb, lev == 1, st);          \
        break;
            SYN_TILE(16) SYN_TILE(8) SYN_TILE(4) SYN_TILE(2)
            default: launch_synthesis<R, 1, true>(a, nb, lev == 1, st);
#undef SYN_TILE
        }
        RIOP_HIP(hipGetLastError());
    }
}

template void launch_psi_adj<float>(riop_plan *, const void *, void *, hipStream_t, int *);
template void launch_psi_adj<double>(riop_plan *, const void *, void *, hipStream_t, int *);
template void launch_psi<float>(riop_plan *, const void *, void *, hipStream_t, int *);
template void launch_psi<double>(riop_plan *, const void *, void *, hipStream_t, int *);
template void launch_psi_adj_prox<float>(riop_plan *, const void *, const Prox1<float> &, hipStream_t);
template void launch_psi_adj_prox<double>(riop_plan *, const void *, const Prox1<double> &, hipStream_t);

}  // namespace riop
