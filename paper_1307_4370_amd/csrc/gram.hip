// Precomputed Gram operator H = G^T G of the interpolation matrix, the
// acceleration of the CG x-update the paper proposes (Sec. 4.5 and Sec. 7:
// store G^T G so that CG no longer forms the M-length vector G F D Z p at
// every iteration).
//
// H is real, symmetric and banded: H[c, c + d] is nonzero only for offsets
// d = (da, db) with |da|, |db| < J (grid indices periodic mod K).  The plan
// stores one K x K plane per offset of the half set (laid out in row chunks, see gram_round)
//     da = 0, 0 <= db < J   and   1 <= da < J, -J < db < J
// (J + (J - 1)(2J - 1) planes: 113 for J = 8), H_d[c] = H[c, c + d]; the other
// half follows from symmetry, H[c, c - d] = H_d[c - d].
//
// Build: H_d[c] = sum_m w_m(c) w_m(c + d), w_m the separable Kaiser-Bessel
// window weights of visibility m (the plan's own polynomials, so H is the Gram
// of exactly the G that degridding and gridding apply).  One wavefront per
// visibility stages its J x J window weights in LDS and walks the list of
// (cell, partner, offset) triples with both cells inside the window, adding
// products with double-precision atomics into double planes (summed in no
// fixed order); the planes are then rounded to the plan's type.
//
// Apply: out[c] = sum_{d in half} H_d[c] in[c + d] + sum_{d in half, d != 0}
// H_d[c - d] in[c - d], a tile of cells per workgroup (see gram_apply).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.hpp"

namespace riop {

int gram_planes(int J) { return J + (J - 1) * (2 * J - 1); }

// Offset (da, db) of plane k.
static void gram_offset(int J, int k, int *da, int *db) {
    if (k < J) {
        *da = 0;
        *db = k;
    } else {
        const int r = k - J;
        *da = 1 + r / (2 * J - 1);
        *db = r % (2 * J - 1) - (J - 1);
    }
}

constexpr int kGramWaves = 4;  // wavefronts per build block

template <typename R>
__global__ void __launch_bounds__(64 * kGramWaves)
    gram_build(const uint32_t *__restrict__ cell, const R *__restrict__ frac, const R *__restrict__ kc, long M, int K,
               int J, int nks, const int3 *__restrict__ triples, int ntriples, double *__restrict__ H) {
    __shared__ double wsh[kGramWaves][16 * 16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double *wv = wsh[wave];
    const long K2 = (long)K * K;
    const long nwaves = (long)gridDim.x * kGramWaves;
    for (long v = (long)blockIdx.x * kGramWaves + wave; v < M; v += nwaves) {
        const uint32_t cv = cell[v];
        const int a0 = (int)(cv & 0xffffu), b0 = (int)(cv >> 16);
        // 1-D weights of tap t: phi(rho + J/2 - 1 - t) from the pair polynomials
        // (tap t and J - 1 - t share the even part E and odd part O in s = 2 rho - 1).
        double wu = 0.0, wvv = 0.0;
        if (lane < 2 * J) {
            const int axis = lane / J, t = lane % J;
            const R rho = frac[2 * v + axis];
            const R s = R(2) * rho - R(1), u = s * s;
            const int jp = t < J / 2 ? t : J - 1 - t;
            const R *ce = kc + (jp * 2 + 0) * nks;
            const R *co = kc + (jp * 2 + 1) * nks;
            R e = ce[nks - 1], o = co[nks - 1];
            for (int k = nks - 2; k >= 0; --k) {
                e = e * u + ce[k];
                o = o * u + co[k];
            }
            const R wt = t < J / 2 ? e + s * o : e - s * o;
            if (axis == 0) wu = (double)wt;
            else wvv = (double)wt;
        }
        // Window weights w(i, j) = wu_i wv_j into LDS (every lane takes part
        // in each shuffle, so the sources are always active).
        for (int base = 0; base < J * J; base += 64) {
            const int c = base + lane;
            const bool in = c < J * J;
            const int i = in ? c / J : 0, j = in ? c - (c / J) * J : 0;
            const double a = __shfl(wu, i), b = __shfl(wvv, J + j);
            if (in) wv[c] = a * b;
        }
        __builtin_amdgcn_wave_barrier();
        for (int t = lane; t < ntriples; t += 64) {
            const int3 tr = triples[t];  // (cell, partner, plane), cells as i * J + j
            const int i = tr.x / J, j = tr.x - (tr.x / J) * J;
            int ga = a0 + i, gb = b0 + j;
            if (ga >= K) ga -= K;
            if (gb >= K) gb -= K;
            atomicAdd(&H[(long)tr.z * K2 + (long)ga * K + gb], wv[tr.x] * wv[tr.y]);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Stored layout: rows cut into chunks of CW cells, the planes innermost but for
// the chunk's cells: H[k1][chunk][plane][cell].  CW is the largest power of two
// up to kGramCols that divides K, so the planes take K^2 values each and no
// padding.  All planes of a chunk lie within some tens of KB, a chunk's planes a
// constant 256 or 512 B apart (less for narrower chunks); whole planes one after
// the other, a power of two apart, fell into the same cache sets.
constexpr int kGramRows = 4, kGramCols = 64;
static int gram_chunk(int K) { return std::min(K & -K, kGramCols); }

template <typename R>
__global__ void gram_round(const double *__restrict__ Hd, R *__restrict__ H, int K, int CW, int nplanes) {
    const long K2 = (long)K * K, row_len = (long)K * nplanes, n = K * row_len;
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const long k1 = i / row_len;
        const int r = (int)(i - k1 * row_len), j = r % CW, d = (r / CW) % nplanes, k2 = r / (CW * nplanes) * CW + j;
        H[i] = (R)Hd[d * K2 + k1 * K + k2];
    }
}

__global__ void fill_zero_f64(double *p, long n) {
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = 0.0;
}

// Four consecutive plane values (16-byte loads; K and so every address is a
// multiple of 4 values).
template <typename R> struct Quad {
    R v[4];
};
template <typename R> __device__ inline Quad<R> load_quad(const R *p) {
    Quad<R> q;
    if constexpr (sizeof(R) == 4) {
        const float4 a = *reinterpret_cast<const float4 *>(p);
        q.v[0] = a.x, q.v[1] = a.y, q.v[2] = a.z, q.v[3] = a.w;
    } else {
        const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
        q.v[0] = a.x, q.v[1] = a.y, q.v[2] = b.x, q.v[3] = b.y;
    }
    return q;
}

// One workgroup per kGramRows x kGramCols tile of output cells; a wavefront
// covers the tile, four cells of a row per lane, and the four wavefronts share
// the row offsets da (da mod 4), their double sums added in a fixed order at
// the end.  The input tile with its J - 1 border is staged in LDS (periodic), so
// a lane reads each input value of a row once for all its (cell, db) pairs.
// The planes are what bounds it: both terms of offset d read plane d, at the
// cell and at the cell less d.  The second is read as the two aligned quads
// that hold it (their position in the quads, -db mod 4, is known at compile
// time; a quad never crosses the periodic edge, since 4 divides K).  Blocks are
// dealt round-robin to the 8 XCDs, so each XCD gets a contiguous range of tiles:
// its L2 then holds the plane rows that its second reads ask for again.
// K = 512, J = 8, FP32 (118 MB of planes, cold): 78 us with one thread
// per cell over whole planes -> 41 us (64 us over whole planes with this kernel).
// CW: the chunk width if known at compile time (plane offsets are then
// immediates), 0 to take `cw`.
template <typename R, int J, int CW>
__global__ void __launch_bounds__(256) gram_apply(const R *__restrict__ H, const C<R> *__restrict__ in,
                                                  C<R> *__restrict__ out, int K, int cw) {
    constexpr int W = J - 1, XW = kGramCols + 2 * W, XH = kGramRows + 2 * W, P = 2 * J - 1, NP = J + W * P;
    constexpr int kX = XH * XW * (int)sizeof(C<R>), kSum = 3 * 64 * 8 * (int)sizeof(double);
    __shared__ __align__(16) unsigned char smem[kX > kSum ? kX : kSum];
    C<R> *xs = reinterpret_cast<C<R> *>(smem);
    const int nb = gridDim.x, xcd = blockIdx.x & 7, per = nb >> 3, rem = nb & 7;
    const int blk = xcd * per + min(xcd, rem) + (blockIdx.x >> 3);
    const int tiles = (K + kGramCols - 1) / kGramCols, width = CW ? CW : cw;
    const int r0 = (blk / tiles) * kGramRows, c0 = (blk % tiles) * kGramCols;
    for (int e = threadIdx.x; e < XH * XW; e += 256) {
        const int i = e / XW, j = e - i * XW;
        // r0 - W and c0 - W are at least -K (K >= 2 J).
        xs[e] = in[(long)((r0 - W + i + K) % K) * K + (c0 - W + j + K) % K];
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row = lane >> 4, col = (lane & 15) * 4;
    const bool active = c0 + col < K;
    const int k1 = r0 + row, k2 = active ? c0 + col : 0;
    // Quads of a row that hold the cells k2 - W .. k2 + 3 + W: k2 + 4 (q - Q).
    constexpr int Q = (W + 3) / 4, NQ = 2 * Q + 1;
    size_t quad[NQ];  // their places in a row's chunks
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        int c = k2 + 4 * (q - Q);
        c += c < 0 ? K : 0;
        c -= c >= K ? K : 0;
        quad[q] = (size_t)(c / width) * (NP * width) + c % width;
    }
    double ar[4] = {}, ai[4] = {};
    auto add = [&](R h, C<R> x, int i) {
        ar[i] += (double)h * x.x;
        ai[i] += (double)h * x.y;
    };
    // Both terms of offsets (da, db), db = LO .. W (LO = 0 for da = 0, whose
    // own cell has no second term).
    auto offsets = [&](auto lo, int da) {
        constexpr int LO = decltype(lo)::value;
        const R *Hd = H + (da == 0 ? 0 : J + (da - 1) * P) * width;
        const size_t row_len = (size_t)K * NP;
        const R *Hf = Hd + k1 * row_len + quad[Q];
        const R *Hb = Hd + (k1 - da + (k1 < da ? K : 0)) * row_len;
        const C<R> *xf = xs + (row + W + da) * XW + col + W, *xb = xs + (row + W - da) * XW + col + W;
#pragma unroll
        for (int db = LO; db <= W; ++db) {
            const int plane = (db - LO) * width;
            const Quad<R> f = load_quad(Hf + plane);
#pragma unroll
            for (int i = 0; i < 4; ++i) add(f.v[i], xf[i + db], i);
            if (LO == 0 && db == 0) continue;
            const int q = (4 * Q - db) / 4, off = (4 * Q - db) & 3;  // cell k2 - db: quad q, place off
            const Quad<R> a = load_quad(Hb + quad[q] + plane), b = off ? load_quad(Hb + quad[q + 1] + plane) : a;
#pragma unroll
            for (int i = 0; i < 4; ++i) add(i + off < 4 ? a.v[(i + off) & 3] : b.v[(i + off) & 3], xb[i - db], i);
        }
    };
    for (int da = wave; da < J; da += 4) {
        if (da == 0) offsets(std::integral_constant<int, 0>{}, da);
        else offsets(std::integral_constant<int, -W>{}, da);
    }
    __syncthreads();  // the input tile is no longer read
    double *sum = reinterpret_cast<double *>(smem);  // [wave - 1][value][lane]
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sum[((wave - 1) * 8 + 2 * i) * 64 + lane] = ar[i];
            sum[((wave - 1) * 8 + 2 * i + 1) * 64 + lane] = ai[i];
        }
    }
    __syncthreads();
    if (wave == 0 && active) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            for (int w = 0; w < 3; ++w) {
                ar[i] += sum[(w * 8 + 2 * i) * 64 + lane];
                ai[i] += sum[(w * 8 + 2 * i + 1) * 64 + lane];
            }
            out[(size_t)k1 * K + k2 + i] = mk<R>((R)ar[i], (R)ai[i]);
        }
    }
}

template <typename R> static void gram_build_t(riop_plan *p, hipStream_t st) {
    const int J = p->J, K = p->K, np_ = gram_planes(J);
    const long K2 = (long)K * K;
    RIOP_REQUIRE(J <= 16, RIOP_ENOTSUP, "Gram build supports J <= 16");
    // (cell, partner, plane) triples with both cells inside the J x J window.
    std::vector<int3> tri;
    for (int k = 0; k < np_; ++k) {
        int da, db;
        gram_offset(J, k, &da, &db);
        for (int i = 0; i + da < J; ++i)
            for (int j = std::max(0, -db); j < J && j + db < J; ++j)
                tri.push_back(make_int3(i * J + j, (i + da) * J + (j + db), k));
    }
    DevBuf tri_d, Hd;
    tri_d.alloc(sizeof(int3) * tri.size());
    RIOP_HIP(hipMemcpyAsync(tri_d.ptr, tri.data(), sizeof(int3) * tri.size(), hipMemcpyHostToDevice, st));
    Hd.alloc(sizeof(double) * np_ * K2);
    hipLaunchKernelGGL(fill_zero_f64, dim3(4096), dim3(256), 0, st, Hd.as<double>(), (long)np_ * K2);
    if (p->M > 0) {
        const long blocks = std::min<long>((p->M + kGramWaves - 1) / kGramWaves, 16384);
        hipLaunchKernelGGL((gram_build<R>), dim3((unsigned)blocks), dim3(64 * kGramWaves), 0, st,
                           (const uint32_t *)p->cell.as<uint32_t>(), (const R *)p->frac.as<R>(),
                           (const R *)p->kcoef_compact.as<R>(), (long)p->M, K, J, p->n_even,
                           (const int3 *)tri_d.as<int3>(), (int)tri.size(), Hd.as<double>());
    }
    p->gram.alloc(sizeof(R) * np_ * K2);
    hipLaunchKernelGGL((gram_round<R>), dim3(4096), dim3(256), 0, st, (const double *)Hd.as<double>(), p->gram.as<R>(),
                       K, gram_chunk(K), np_);
    RIOP_HIP(hipGetLastError());
    RIOP_HIP(hipStreamSynchronize(st));  // the temporaries go out of scope
}

void gram_build_plan(riop_plan *p, hipStream_t st) {
    RIOP_REQUIRE(p->n_even == p->n_odd || p->n_even == p->n_odd + 1, RIOP_EDEVICE, "kernel polynomial layout");
    if (p->prec == RIOP_F64)
        gram_build_t<double>(p, st);
    else
        gram_build_t<float>(p, st);
}

template <typename R> void launch_gram_apply(riop_plan *p, const void *in_grid, void *out_grid, hipStream_t st) {
    const int K = p->K, cw = gram_chunk(K);
    RIOP_REQUIRE(cw >= 4, RIOP_EDEVICE, "grid side must be a multiple of 4");
    const dim3 g((unsigned)((K + kGramCols - 1) / kGramCols * (K / kGramRows))), t(256);
    TimedScope ts(p, KK_GRAM, st);
    switch (p->J) {
#define GA_LAUNCH(JJ, CW)                                                                                    \
    hipLaunchKernelGGL((gram_apply<R, JJ, CW>), g, t, 0, st, (const R *)p->gram.as<R>(),                     \
                       static_cast<const C<R> *>(in_grid), static_cast<C<R> *>(out_grid), K, cw)
#define GA(JJ)                                      \
    case JJ:                                        \
        if (cw == kGramCols) GA_LAUNCH(JJ, kGramCols); \
        else GA_LAUNCH(JJ, 0);                      \
        break;
        GA(2) GA(4) GA(6) GA(8) GA(10) GA(12) GA(14) GA(16)
#undef GA
#undef GA_LAUNCH
        default: throw Error{RIOP_ENOTSUP, "unsupported kernel width"};
    }
    RIOP_HIP(hipGetLastError());
}

template void launch_gram_apply<float>(riop_plan *, const void *, void *, hipStream_t);
template void launch_gram_apply<double>(riop_plan *, const void *, void *, hipStream_t);

}  // namespace riop
