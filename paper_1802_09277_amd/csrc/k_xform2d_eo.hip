// gfx950 kernels of the space-time slab solver: both FP64 spatial eigenbasis
// transforms of a 2-D image in one pass (eq. equ:ST:generalDecompA with fast
// diagonalisation of K_x + lambda M_x), for n <= 96.
//
// The eigenvectors are even or odd (first the h1 = ceil(n/2) even ones), so
// with the image folded along both axes the transform falls into four
// products of half the size, one for each pair (row parity p, column parity
// q), n^3 multiply-adds instead of 2 n^3:
//   forward  Y_pq = U_p^T X_pq U_q,   X_pq[i][k] = x[i][k] +- its mirror images,
//   inverse  Z_pq = U_p Y_pq U_q^T,   x = sum of the Z_pq, the mirrored elements
//            with the signs of the odd parts.
// One wave per pair, four waves per image: a wave takes 16 rows at a time
// through the first product (MFMA A = data, from global memory, B = U_q), and
// the accumulators of that product are the B operand of the second as they
// are (A = U_p): rows go to lines of the first product in the order that the
// second one's k steps take them.  Data thus pass through registers only, one
// LDS copy of U_even and U_odd serves both products, and waves run without
// barriers; the inverse exchanges its four parts tile by tile through LDS.
// The four waves of an image read it again, from L1 and L2 (forward).  Bound
// by latency at two to four waves per SIMD (registers) and, for many images,
// by the MFMAs (65^2: 90 a wave and image, 24 to 30 % busy).  Against the image and
// U in LDS, eight waves to an image, two barriers to a product: a slab inverse
// (a transform each way and the temporal solve) of 256 x 5 images of 65^2 142
// -> 86 us (forward 62 -> 41, inverse 67 -> 35), 192 x 5 of 61^2 83 -> 56,
// 160 x 3 of 79^2 86 -> 58, 100 x 4 of 90^2 119 -> 66, 400 x 4 of 20^2 41 ->
// 22, 24 x 4 of 40^2 19.2 -> 17.4, 16 x 4 of 16^2 14.5 (both).  Per axis
// (k_xform_eo) 65^2 took 120 us.
#include <algorithm>
#include <atomic>

#include "kernels_common.hpp"

namespace sth {

struct Eo2dArgs {
    const double* in;
    double* out;
    const double* T;                            // packed panels (xform_eo_pack)
    const int* guard;
    double alpha;
    long nimg, ldi, ldo;
    int n, k4;                                  // k4: packed rows (xform_eo_rows)
};

typedef double d2v __attribute__((ext_vector_type(2), aligned(8)));

// Column tiles NJ of a half; REM: a half of 16 NJ + 1 (n = 33, 34, 65, 66: the
// meshes of 2^k elements with degree 3 and 4), whose last output row and
// column are vector multiply-adds on the registers of the products instead of
// another tile each way.
//
// LDS row of U: even half, odd half, their remainder columns, pad (lane groups
// four rows apart fall into distinct banks)
template <int NJ> constexpr int eo2d_row() { return 32 * NJ + 4; }
template <int NJ, bool REM> constexpr int eo2d_rows() { return 16 * NJ + (REM ? 4 : 0); }
template <int NJ, bool REM, bool INV> constexpr size_t eo2d_lds() {
    return sizeof(double) * ((size_t)eo2d_rows<NJ, REM>() * eo2d_row<NJ>() + (INV ? 2 * 4 * 256 : 0));
}
// waves per SIMD that the registers leave room for
template <int NJ, bool INV> constexpr int eo2d_waves() { return NJ == 1 ? 4 : (NJ == 2 && INV ? 3 : 2); }

template <int NJ, bool REM, bool INV, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(eo2d_waves<NJ, INV>())))
void k_xform2d_eo(Eo2dArgs a) {
    if (guard_off(a.guard)) return;
    constexpr int W = 16 * NJ, R = eo2d_row<NJ>(), ROWS = eo2d_rows<NJ, REM>();
    extern __shared__ double sm[];
    double* xch = sm + ROWS * R;                // [parity of the round][pq][r][lane]
    const int n = a.n, h1 = (n + 1) / 2, h0 = n / 2;
    const int nfull = h0 / 16;                  // chunks and row tiles with all 16 k in both halves
    const int ntail = (h1 - 16 * nfull + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int p = wave >> 1, q = wave & 1;      // row and column parity
    const int hp = p ? h0 : h1, hq = q ? h0 : h1;
    const double sp = p ? -1.0 : 1.0, sq = q ? -1.0 : 1.0;
    // A row of the image for this lane in row tile t: full tiles in the order
    // of the second product's k steps (its accumulator row lg + 4 r is row
    // 4 lg + r), the last tile as it is.  Forward: the mirrored row as well,
    // which the middle row does not have.
    struct Row {
        const double *x, *m;
        double f;
    };
    auto row_of = [&](long img, int t) {
        const double* src = a.in + img * a.ldi;
        const int i = 16 * t + (t < nfull ? 4 * (lr & 3) + (lr >> 2) : lr);
        Row w;
        if (INV) {
            w.x = src + (long)((p && h0 ? h1 : 0) + min(i, hp > 0 ? hp - 1 : 0)) * n + (q ? h1 : 0);
            w.m = nullptr;
            w.f = 0.0;
        } else {
            const int ic = min(i, h1 - 1);
            w.x = src + (long)ic * n;
            w.m = src + (long)(n - 1 - ic) * n;
            w.f = ic < h0 ? sp : 0.0;
        }
        return w;
    };
    // full chunk ch: k = 16 ch + 4 lg + s (and its mirror images)
    constexpr int ND = INV ? 1 : 4;
    struct Raw {
        d2v v[ND][2];
    };
    auto load = [&](const Row& w, int ch) {
        Raw o;
        const int k = 16 * ch + 4 * lg;
        o.v[0][0] = *reinterpret_cast<const d2v*>(w.x + k);
        o.v[0][1] = *reinterpret_cast<const d2v*>(w.x + k + 2);
        if constexpr (!INV) {
            const int m = n - 4 - k;            // elements m + 3 .. m mirror k .. k + 3
            o.v[1][0] = *reinterpret_cast<const d2v*>(w.x + m + 2);
            o.v[1][1] = *reinterpret_cast<const d2v*>(w.x + m);
            o.v[2][0] = *reinterpret_cast<const d2v*>(w.m + k);
            o.v[2][1] = *reinterpret_cast<const d2v*>(w.m + k + 2);
            o.v[3][0] = *reinterpret_cast<const d2v*>(w.m + m + 2);
            o.v[3][1] = *reinterpret_cast<const d2v*>(w.m + m);
        }
        return o;
    };
    auto fold = [&](const Raw& o, double f, int s) {
        const int h = s / 2, e = s % 2;
        if constexpr (INV) return o.v[0][h][e];
        else return (o.v[0][h][e] + sq * o.v[1][h][1 - e]) + f * (o.v[2][h][e] + sq * o.v[3][h][1 - e]);
    };
    long img = blockIdx.x;
    Row rn = row_of(img, 0);                    // (a block has an image)
    constexpr int NT = REM ? 1 : 4;
    constexpr bool AHEAD = NJ > 1;              // a chunk ahead, as registers allow
    Raw nx;
    if (AHEAD && nfull > 0) nx = load(rn, 0);
    // U, packed as [tile][k][16 even, 16 odd] and [k][2 remainder columns]: the
    // 16-byte copies of a thread in flight together
    const int nt = min(NJ, (h1 + 15) / 16), m = nt * a.k4 * 16;
    {
        constexpr int U = (NJ * ROWS * 16 + 255) / 256;
        double2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = reinterpret_cast<const double2*>(a.T)[min(tid + 256 * u, m - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tid + 256 * u, c = i & 15, g = i >> 4, t = NJ == 1 ? 0 : g / a.k4, k = g - t * a.k4;
            if (i < m) *reinterpret_cast<double2*>(sm + k * R + (c < 8 ? 0 : W - 16) + 16 * t + 2 * c) = v[u];
        }
    }
    for (int i = tid; i < a.k4 * (W - 16 * nt); i += 256) {     // tiles past the half
        const int k = i / (W - 16 * nt), c = 16 * nt + i % (W - 16 * nt);
        sm[k * R + c] = sm[k * R + W + c] = 0.0;
    }
    for (int i = tid; i < (ROWS - a.k4) * 2 * W; i += 256) sm[(a.k4 + i / (2 * W)) * R + i % (2 * W)] = 0.0;
    if (REM)
        for (int i = tid; i < 2 * a.k4; i += 256) sm[(i >> 1) * R + 2 * W + (i & 1)] = a.T[(long)NJ * a.k4 * 32 + i];
    __syncthreads();
    const double* ucol = sm + q * W + lr;       // first product: column lr of tile jt at + 16 jt
    const double* urow = sm + p * W + lr;       // second product: output row lr of tile mt at + 16 mt
    const int nrt = nfull + (ntail > 0);
    for (; img < a.nimg; img += gridDim.x) {
        const long inext = img + gridDim.x < a.nimg ? img + gridDim.x : img;
        d4 z[NJ][NJ];
        double zr[NJ], zc[NJ], zz = 0.0;        // remainder row, column and corner, summed over the lane groups at the end
#pragma unroll
        for (int mt = 0; mt < NJ; ++mt) {
            zr[mt] = zc[mt] = 0.0;
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) z[mt][jt] = d4{0, 0, 0, 0};
        }
#pragma unroll 1
        for (int t = 0; t < nrt; ++t) {
            const bool full = t < nfull;
            const Row rc = rn;
            rn = row_of(t + 1 < nrt ? img : inext, t + 1 < nrt ? t + 1 : 0);
            // the last chunk's data, used after the full ones: k = 16 nfull +
            // 4 s + lg (rows of U past the half are zero)
            double tv[NT];
#pragma unroll
            for (int s = 0; s < NT; ++s) {
                const int k = 16 * nfull + 4 * s + lg;
                tv[s] = 0.0;
                if (s < ntail) {
                    if constexpr (INV) {
                        tv[s] = k < hq ? rc.x[k] : 0.0;
                    } else {
                        const int kc = min(k, h1 - 1);
                        const double cm = kc < h0 ? sq : 0.0;   // (the middle element once)
                        tv[s] = (rc.x[kc] + cm * rc.x[n - 1 - kc]) + rc.f * (rc.m[kc] + cm * rc.m[n - 1 - kc]);
                    }
                }
            }
            d4 c[NJ];
            double tc = 0.0;                    // remainder column of the first product
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) c[jt] = d4{0, 0, 0, 0};
#pragma unroll 1
            for (int ch = 0; ch < nfull; ++ch) {
                const Raw cx = AHEAD ? nx : load(rc, ch);
                if (AHEAD) nx = load(ch + 1 < nfull ? rc : rn, ch + 1 < nfull ? ch + 1 : 0);
                const double* u = ucol + (16 * ch + 4 * lg) * R;
                const double* ur = sm + (16 * ch + 4 * lg) * R + 2 * W + q;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double v = fold(cx, rc.f, s);
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) c[jt] = Mfma16<double>::op(v, u[s * R + 16 * jt], c[jt]);
                    if (REM) tc += v * ur[s * R];
                }
            }
            {
                const double* u = ucol + (16 * nfull + lg) * R;
                const double* ur = sm + (16 * nfull + lg) * R + 2 * W + q;
#pragma unroll
                for (int s = 0; s < NT; ++s) {
                    if (s >= ntail) break;
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) c[jt] = Mfma16<double>::op(tv[s], u[4 * s * R + 16 * jt], c[jt]);
                    if (REM) tc += tv[s] * ur[4 * s * R];
                }
            }
            if (REM) {
                tc += __shfl_xor(tc, 16);
                tc += __shfl_xor(tc, 32);
            }
            // second product: k step r of this tile
            const double* u = urow + (16 * t + (full ? 4 * lg : lg)) * R;
            const double* ur = sm + (16 * t + (full ? 4 * lg : lg)) * R + 2 * W + p;
            const int us = full ? R : 4 * R;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!full && r >= ntail) break;
                double tr = 0.0, wr = 0.0;
                if (REM) {
                    tr = __shfl(tc, lg + 4 * r);
                    wr = ur[r * us];
                    zz += wr * tr;
                }
#pragma unroll
                for (int mt = 0; mt < NJ; ++mt) {
                    const double w = u[r * us + 16 * mt];
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) z[mt][jt] = Mfma16<double>::op(w, c[jt][r], z[mt][jt]);
                    if (REM) {
                        zc[mt] += w * tr;
                        zr[mt] += wr * c[mt][r];
                    }
                }
            }
        }
        if (REM) {
            auto sum = [](double& v) {
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
            };
            sum(zz);
#pragma unroll
            for (int mt = 0; mt < NJ; ++mt) {
                sum(zr[mt]);
                sum(zc[mt]);
            }
        }
        double* dst = a.out + img * a.ldo;
        if constexpr (!INV) {
            dst += (long)(p ? h1 : 0) * n + (q ? h1 : 0);
#pragma unroll
            for (int mt = 0; mt < NJ; ++mt)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * mt + lg + 4 * r, j = 16 * jt + lr;
                        if (i < hp && j < hq) dst[(long)i * n + j] = z[mt][jt][r];
                    }
            if (REM && lg == 0) {
#pragma unroll
                for (int mt = 0; mt < NJ; ++mt) {
                    if (W < hp) dst[(long)W * n + 16 * mt + lr] = zr[mt];
                    if (W < hq) dst[(long)(16 * mt + lr) * n + W] = zc[mt];
                }
                if (lr == 0 && W < hp && W < hq) dst[(long)W * n + W] = zz;
            }
        } else {
            // the four parts of a tile, from one LDS buffer while the other fills;
            // wave (p, q) forms the elements mirrored along rows (p), columns (q)
            auto put = [&](int i, int j, double v) {
                double* o = dst + (long)(p ? n - 1 - i : i) * n + (q ? n - 1 - j : j);
                if (EPI == 0) *o = v;
                else if (EPI == 1) *o += a.alpha * v;
                else *o = a.alpha * v;
            };
            auto all = [&](const double* e) { return (e[0] + sq * e[256]) + sp * (e[512] + sq * e[768]); };
#pragma unroll
            for (int mt = 0; mt < NJ; ++mt)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) {
                    double* e = xch + ((mt * NJ + jt) % 2) * 1024 + lane;
#pragma unroll
                    for (int r = 0; r < 4; ++r) e[(2 * p + q) * 256 + 64 * r] = z[mt][jt][r];
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * mt + lg + 4 * r, j = 16 * jt + lr;
                        const double v = all(e + 64 * r);
                        if (i < hp && j < hq) put(i, j, v);
                    }
                }
            if (REM) {
                // remainder row (lane group 0), column (1) and corner (2)
                double* e = xch + ((NJ * NJ) % 2) * 1024 + lane;
#pragma unroll
                for (int mt = 0; mt < NJ; ++mt) e[(2 * p + q) * 256 + 64 * mt] = lg == 0 ? zr[mt] : (lg == 1 ? zc[mt] : zz);
                __syncthreads();
#pragma unroll
                for (int mt = 0; mt < NJ; ++mt) {
                    const int i = lg == 1 ? 16 * mt + lr : W, j = lg == 0 ? 16 * mt + lr : W;
                    const double v = all(e + 64 * mt);
                    if ((lg < 2 || (lane == 32 && mt == 0)) && i < hp && j < hq) put(i, j, v);
                }
            }
            if ((NJ * NJ + REM) % 2) __syncthreads();   // (the next image starts on the first buffer again)
        }
    }
}

bool xform2d_eo_supported(int n) { return n >= 1 && n <= 96; }

template <int NJ, bool REM, bool INV, int EPI>
static hipError_t eo2d_go(const Eo2dArgs& a, hipStream_t st) {
    static std::atomic<bool> attr_set{false};       // set once; the attribute call is idempotent
    constexpr size_t shm = eo2d_lds<NJ, REM, INV>();
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_xform2d_eo<NJ, REM, INV, EPI>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    // persistent blocks: as many as fit at once, all with the same number of
    // images up to one
    const long fit = 256 * std::max<long>(1, std::min<long>(160 * 1024 / shm, eo2d_waves<NJ, INV>()));
    const long rounds = (a.nimg + fit - 1) / fit;
    hipLaunchKernelGGL((k_xform2d_eo<NJ, REM, INV, EPI>), dim3((unsigned)((a.nimg + rounds - 1) / rounds)), dim3(256),
                       shm, st, a);
    return hipGetLastError();
}

template <bool INV, int EPI>
static hipError_t eo2d_launch(const Eo2dArgs& a, hipStream_t st) {
    const int h1 = (a.n + 1) / 2;
    if (h1 <= 16) return eo2d_go<1, false, INV, EPI>(a, st);
    if (h1 == 17) return eo2d_go<1, true, INV, EPI>(a, st);
    if (h1 <= 32) return eo2d_go<2, false, INV, EPI>(a, st);
    if (h1 == 33) return eo2d_go<2, true, INV, EPI>(a, st);
    return eo2d_go<3, false, INV, EPI>(a, st);
}

hipError_t launch_xform2d_eo(bool inv, int epi, const double* in, double* out, const double* T, int n, long nimg,
                             double alpha, hipStream_t st, const int* guard, long ldi, long ldo) {
    if (nimg <= 0) return hipSuccess;
    if (!xform2d_eo_supported(n)) return hipErrorInvalidValue;
    const long nn = (long)n * n;
    const Eo2dArgs a{in, out, T, guard, alpha, nimg, ldi ? ldi : nn, ldo ? ldo : nn, n, xform_eo_rows(n)};
    if (!inv) return epi == 0 ? eo2d_launch<false, 0>(a, st) : hipErrorInvalidValue;
    if (epi == 0) return eo2d_launch<true, 0>(a, st);
    if (epi == 1) return eo2d_launch<true, 1>(a, st);
    if (epi == 2) return eo2d_launch<true, 2>(a, st);
    return hipErrorInvalidValue;
}

}  // namespace sth
