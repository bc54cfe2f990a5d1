// gfx950 kernels of the space-time slab solver: the FP64 spatial eigenbasis
// transforms one axis at a time (eq. equ:ST:generalDecompA with fast
// diagonalisation of K_x + lambda M_x), for every n <= kEoMaxN.
//
// The eigenvectors of the uniform mesh are even or odd under the reflection
// i -> n-1-i and ordered [even | odd] (h1 = ceil(n/2) even ones, h0 = n/2 odd
// ones), so an axis takes two products of half the size:
//   forward: y_j = sum_{k<h1} U[k][j] (x_k + x_{n-1-k}), j even (the middle
//            x of an odd n once), y_j = sum_{k<h0} U[k][j] (x_k - x_{n-1-k}), j odd;
//   inverse: p_i = sum_{j even} U[i][j] y_j, q_i = sum_{j odd} U[i][j] y_j,
//            x_i = p_i + q_i, x_{n-1-i} = p_i - q_i, i < h1.
// FP64 matrix and vector rate are the same on this card (77.6 and 70 TFLOP/s
// measured in registers), so halving the multiply-adds is what counts.  Large
// n is bound by the MFMAs (n = 256, 3072 images: 0.92 to 1.01 ms per axis, 51 to
// 56 TFLOP/s at 72 to 78 % MFMA busy, the clock 2.1 to 2.2 GHz under this load,
// 2.4 without; 384 images 127 to 144 us at 59 to 66 %),
// small n by HBM and latency.  A slab inverse (two transforms of each axis
// and the temporal solve), against panels of the full matrix for padded
// widths that are a multiple of 32 and tiles staged per block otherwise:
// 64 x 6 images of 258^2 2750 -> 709 us, 40 x 3 of 100^2 131 -> 55 us,
// 20 x 4 cubes of 32^3 142 -> 74 us, 3072 images of 256^2 (both split) 4.82
// -> 4.23 ms.
//
// A block holds a panel of 16 NJ output columns of both half matrices in LDS
// (rows padded by four words: the k of two lane groups fall into distinct
// banks); each wave walks over tiles of 16 lines with no
// further barrier, both halves of a tile from the same loads.  Data goes
// through registers in stages of two chunks of 16 k (and the 16 mirrored
// elements, or the odd coefficients), the next stage's loads in flight during
// the MFMAs.  A last chunk of fewer than 16 k takes ceil(r / 4) MFMA steps
// instead of four.  A half of 16 m + 1 columns (n = 2^k + 1, 2^k + 2: the
// meshes of 2^k elements with degree 3 and 4) computes its last column by
// vector multiply-adds from the same registers, 4 cycles a step, instead of
// a tile of 16 columns, 64 cycles.
//  x axis (contiguous): lines of n elements; MFMA A = data, B = panel.
//  strided axis: line c = (batch c / inner, column c % inner), element stride
//    inner; tiles run over batch ends, so that no column is padding.
//    MFMA A = panel^T, B = data: stores of 16 consecutive columns.
// Blocks are persistent; the panels of one tile stream sit on one XCD (ids
// b, b + 8, ...) and share its data in L2.
#include <algorithm>
#include <atomic>

#include "kernels_common.hpp"

namespace sth {

constexpr int kEoMaxJ = 5;                      // 16-column tiles of a panel, per half
constexpr long kEoFill = 2048;                  // (line tile, panel) pairs that fill the card: two per SIMD

struct EoArgs {
    const double* in;
    double* out;
    const double* T;                            // packed panels (xform_eo_pack)
    const int* guard;
    double alpha;
    long nlines, ntiles;
    int n, inner, tiles, npanel, k4;            // tiles: column tiles per half; k4: LDS rows
};

typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// waves per SIMD that the registers of a panel width leave room for
template <int NJ> constexpr int eo_waves() { return NJ <= 2 ? 4 : 2; }

template <bool XAXIS, bool INV, int EPI, int NJ, bool REM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(eo_waves<NJ>()))) void k_xform_eo(EoArgs a) {
    if (guard_off(a.guard)) return;
    constexpr int W = 16 * NJ, R = 2 * W + 4;   // LDS row: even half, odd half, the two columns past them, pad
    extern __shared__ double sm[];
    const int n = a.n, h1 = (n + 1) / 2, h0 = n / 2, k4 = a.k4;
    const int nfull = h0 / 16;                  // chunks with all 16 k in both halves
    const int ntail = (h1 - 16 * nfull + 3) / 4;   // MFMA steps of the last chunk
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int b = blockIdx.x, xcd = b & 7, q = b >> 3;
    const int panel = q % a.npanel;
    const long stream = (long)(q / a.npanel) * 8 + xcd;
    const long nstream = (long)gridDim.x / a.npanel;
    const int j0 = panel * W;                   // first column of the panel within its half
    const bool rem = REM && panel == a.npanel - 1;
    // stage the panel's column tiles (packed as [tile][k][16 even, 16 odd]):
    // 16-byte copies, eight in flight per thread; tiles past the last are not read
    const int jt_n = min(NJ, a.tiles - panel * NJ);
    for (int jt = 0; jt < jt_n; ++jt) {
        const double2* src = reinterpret_cast<const double2*>(a.T) + (long)(panel * NJ + jt) * k4 * 16;
        const int m = k4 * 16, nt = blockDim.x;
        for (int i0 = tid; i0 < m; i0 += 8 * nt) {
            double2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[min(i0 + u * nt, m - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = min(i0 + u * nt, m - 1), c = i & 15;      // (repeats store the same value)
                *reinterpret_cast<double2*>(sm + (i >> 4) * R + (c < 8 ? 0 : W - 16) + 16 * jt + 2 * c) = v[u];
            }
        }
    }
    for (int i = tid; i < k4 * (W - 16 * jt_n); i += blockDim.x) {  // (a last panel of fewer tiles)
        const int k = i / (W - 16 * jt_n), c = 16 * jt_n + i % (W - 16 * jt_n);
        sm[k * R + c] = sm[k * R + W + c] = 0.0;
    }
    if (REM)
        for (int i = tid; i < 2 * k4; i += blockDim.x)
            sm[(i >> 1) * R + 2 * W + (i & 1)] = a.T[(long)a.tiles * k4 * 32 + i];
    __syncthreads();
    // A tile of 16 lines: wave-uniform offsets of its first line plus 32-bit
    // lane offsets (the launcher checks that they fit), so that the addresses
    // of the loads of a stage stay in scalar registers.  Lanes past the last
    // line read it again and store nothing.
    const unsigned ks = XAXIS ? 1u : (unsigned)a.inner;         // element stride of a line
    struct Tile {
        long u;
        unsigned d;
        bool ok;
    };
    auto tile_of = [&](long t) {
        Tile l;
        const long left = a.nlines - t * 16;
        const unsigned m = min((long)lr, left - 1);
        l.ok = lr < left;
        if (XAXIS) {
            l.u = t * 16 * (long)n;
            l.d = m * (unsigned)n;
        } else {
            const long bt = t * 16 / a.inner;   // a tile may run over batch ends
            const unsigned c0 = (unsigned)(t * 16 - bt * a.inner), c = c0 + m;
            const unsigned db = c / (unsigned)a.inner, col = c - db * (unsigned)a.inner;
            l.u = bt * n * a.inner;
            l.d = db * (unsigned)(n * a.inner) + col;
        }
        return l;
    };
    // full chunk c, step s of lane group lg: k = 16 c + 4 lg + s; last chunk:
    // k = 16 nfull + 4 s + lg.  x: element k (inverse: even coefficient k),
    // y: element n-1-k (odd coefficient h1 + k).  The loads of a stage are
    // unconditional (a chunk past the end repeats the last one) and their
    // values are first touched when the stage runs.
    constexpr int G = NJ <= 2 ? 1 : 2;          // chunks per stage
    double nx[G][4], ny[G][4];
    auto load = [&](long ui, unsigned di, int c0) {
        const unsigned da = di + 4 * lg * ks, db = INV ? da : di + (12 - 4 * lg) * ks;
#pragma unroll
        for (int cc = 0; cc < G; ++cc) {
            const int c = G > 1 ? min(c0 + cc, nfull - 1) : c0;
            if constexpr (XAXIS) {
                const double* pa = a.in + ui + 16 * c;
                const double* pb = a.in + ui + (INV ? h1 + 16 * c : n - 16 - 16 * c);
                const d2u a0 = *reinterpret_cast<const d2u*>(pa + da), a1 = *reinterpret_cast<const d2u*>(pa + 2 + da);
                const d2u b0 = *reinterpret_cast<const d2u*>(pb + db), b1 = *reinterpret_cast<const d2u*>(pb + 2 + db);
                nx[cc][0] = a0[0];
                nx[cc][1] = a0[1];
                nx[cc][2] = a1[0];
                nx[cc][3] = a1[1];
                ny[cc][0] = INV ? b0[0] : b1[1];
                ny[cc][1] = INV ? b0[1] : b1[0];
                ny[cc][2] = INV ? b1[0] : b0[1];
                ny[cc][3] = INV ? b1[1] : b0[0];
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double* pa = a.in + ui + (long)(16 * c + s) * ks;
                    const double* pb = a.in + ui + (long)(INV ? h1 + 16 * c + s : n - 13 - 16 * c - s) * ks;
                    nx[cc][s] = pa[da];
                    ny[cc][s] = pb[db];
                }
            }
        }
    };
    // tiles go round over the streams first, then over the waves, so that a
    // few tiles spread over all blocks
    const long tstep = nw * nstream;
    long tile = wave * nstream + stream;
    if (tile >= a.ntiles) return;               // (no barrier below)
    Tile tn = tile_of(tile);
    if (nfull > 0) load(tn.u, tn.d, 0);
    for (; tile < a.ntiles; tile += tstep) {
        const Tile tc = tn;
        tn = tile_of(min(tile + tstep, a.ntiles - 1));
        // opaque copies: addresses are formed per tile instead of being kept
        // in registers for every step and output
        int lgo = lg, lro = lr;
        asm volatile("" : "+v"(lgo), "+v"(lro));
        // the last chunk's data, used at the end of the tile
        double tx[4], ty[4];
        if (ntail > 0) {
            const double* p = a.in + tc.u;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 16 * nfull + 4 * s + lgo;
                tx[s] = p[tc.d + (k < h1 ? (unsigned)k * ks : 0u)];
                ty[s] = p[tc.d + (k < h0 ? (unsigned)(INV ? h1 + k : n - 1 - k) * ks : 0u)];
            }
        }
        d4 ae[NJ], ao[NJ];
        double se = 0.0, so = 0.0;
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) ae[jt] = ao[jt] = d4{0, 0, 0, 0};
        struct Ops {
            double e[NJ], o[NJ], re, ro;
        };
        auto fetch = [&](const double* row, Ops& w) {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {
                w.e[jt] = row[lro + 16 * jt];
                w.o[jt] = row[lro + W + 16 * jt];
            }
            if (REM) {
                w.re = row[2 * W];
                w.ro = row[2 * W + 1];
            }
        };
        auto mma = [&](const Ops& w, double x, double y) {
            // (the middle element of an odd n has y = 0; the odd half's row of it is zero)
            const double e = INV ? x : x + y, o = INV ? y : x - y;
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) {
                ae[jt] = XAXIS ? Mfma16<double>::op(e, w.e[jt], ae[jt]) : Mfma16<double>::op(w.e[jt], e, ae[jt]);
                ao[jt] = XAXIS ? Mfma16<double>::op(o, w.o[jt], ao[jt]) : Mfma16<double>::op(w.o[jt], o, ao[jt]);
            }
            if (REM) {
                se += e * w.re;
                so += o * w.ro;
            }
        };
        const double* lrow = sm + 4 * lgo * R;
#pragma unroll 1
        for (int c0 = 0; c0 < nfull; c0 += G) {
            double cx[G][4], cy[G][4];
#pragma unroll
            for (int cc = 0; cc < G; ++cc)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    cx[cc][s] = nx[cc][s];
                    cy[cc][s] = ny[cc][s];
                }
            const bool here = c0 + G < nfull;   // the next stage belongs to this tile
            load(here ? tc.u : tn.u, here ? tc.d : tn.d, here ? c0 + G : 0);
            // the operands of step s + 1 are read before the MFMAs of step s
            Ops w[2];
            fetch(lrow + 16 * c0 * R, w[0]);
#pragma unroll
            for (int cc = 0; cc < G; ++cc) {
                if (G > 1 && c0 + cc >= nfull) break;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int q = 4 * cc + s;
                    if (q + 1 < 4 * G) fetch(lrow + (16 * (c0 + (q + 1) / 4) + (q + 1) % 4) * R, w[(q + 1) & 1]);
                    mma(w[q & 1], cx[cc][s], cy[cc][s]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (ntail > 0) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s >= ntail) break;
                const int k = 16 * nfull + 4 * s + lgo;
                Ops w;
                fetch(sm + k * R, w);
                mma(w, k < h1 ? tx[s] : 0.0, k < h0 ? ty[s] : 0.0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // Outputs of column j = j0 + 16 jt + jl: the even and the odd mode, or
        // element j and its mirror image (once in the middle), for the lane's
        // line (strided axis) or line lgo + 4 r (x axis).  The update reads the
        // old values first, all of them, so that their loads overlap.
        const long left = a.nlines - tile * 16;
        auto put = [&](double* p, double v, double old) {
            if (EPI == 0) *p = v;
            else if (EPI == 1) *p = old + a.alpha * v;
            else *p = a.alpha * v;
        };
        auto first = [&](int jt, int r) -> double* {
            if (XAXIS) return a.out + tc.u + j0 + 16 * jt + (unsigned)((lgo + 4 * r) * n + lro);
            return a.out + tc.u + (long)(j0 + 16 * jt + 4 * r) * ks + (tc.d + lgo * ks);
        };
        auto second = [&](int jt, int r) -> double* {
            if (XAXIS && !INV) return a.out + tc.u + h1 + j0 + 16 * jt + (unsigned)((lgo + 4 * r) * n + lro);
            if (XAXIS) return a.out + tc.u + (n - 16 - j0 - 16 * jt) + ((lgo + 4 * r) * n + 15 - lro);
            if (!INV) return a.out + tc.u + (long)(h1 + j0 + 16 * jt + 4 * r) * ks + (tc.d + lgo * ks);
            return a.out + tc.u + (long)(n - 4 - j0 - 16 * jt - 4 * r) * ks + (tc.d + (3 - lgo) * ks);
        };
        auto col = [&](int jt, int r) { return j0 + 16 * jt + (XAXIS ? lro : lgo + 4 * r); };
        auto row_ok = [&](int r) { return XAXIS ? lgo + 4 * r < left : tc.ok; };
        double oe[EPI == 1 ? NJ : 1][4], oo[EPI == 1 ? NJ : 1][4];
        if constexpr (EPI == 1) {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    oe[jt][r] = oo[jt][r] = 0.0;
                    if (row_ok(r) && col(jt, r) < h1) oe[jt][r] = *first(jt, r);
                    if (row_ok(r) && col(jt, r) < h0) oo[jt][r] = *second(jt, r);
                }
        }
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double v = INV ? ae[jt][r] + ao[jt][r] : ae[jt][r];
                const double w = INV ? ae[jt][r] - ao[jt][r] : ao[jt][r];
                if (row_ok(r) && col(jt, r) < h1) put(first(jt, r), v, oe[EPI == 1 ? jt : 0][r]);
                if (row_ok(r) && col(jt, r) < h0) put(second(jt, r), w, oo[EPI == 1 ? jt : 0][r]);
            }
        if (rem) {
            se += __shfl_xor(se, 16);
            so += __shfl_xor(so, 16);
            se += __shfl_xor(se, 32);
            so += __shfl_xor(so, 32);
            // lane group 0 stores the first output of its line, group 1 the second
            const int j = 16 * a.tiles;
            if (tc.ok && (lg == 0 ? j < h1 : lg == 1 && j < h0)) {
                const unsigned k = lg == 0 ? j : (INV ? n - 1 - j : h1 + j);
                double* p = a.out + tc.u + (tc.d + k * ks);
                const double v = INV ? (lg == 0 ? se + so : se - so) : (lg == 0 ? se : so);
                put(p, v, EPI == 1 ? *p : 0.0);
            }
        }
    }
}

// Column tiles of a half of an axis of n, and whether a remainder column follows.
static int eo_tiles(int n, bool* rem) {
    const int h1 = (n + 1) / 2;
    *rem = h1 > 16 && h1 % 16 == 1;
    return *rem ? h1 / 16 : (h1 + 15) / 16;
}
static int eo_rows(int n) {
    const int h1 = (n + 1) / 2, nfull = n / 2 / 16;
    return 16 * nfull + 4 * ((h1 - 16 * nfull + 3) / 4);
}
static size_t eo_lds(int n, int nj) { return sizeof(double) * (size_t)eo_rows(n) * (32 * nj + 4); }

// Column tiles of a panel: as many as LDS and the register budget allow (each
// panel reads the data again, from L2), fewer where the line tiles alone
// leave waves idle: then narrower panels shorten both a block's staging and
// a wave's chain of MFMAs (a slab inverse of 9 images of 300^2: 61 us, against
// 84 us with the widest panels that fit; from 1024 to 2048 pairs 24 images of
// 256^2 93 -> 81, 36 of 200^2 83 -> 70, at 4096 the same).
static int eo_panel_tiles(int n, long ntiles) {
    bool rem;
    const int tiles = eo_tiles(n, &rem);
    auto panels = [&](int nj) { return (tiles + nj - 1) / nj; };
    int nj = std::min(tiles, kEoMaxJ);
    while (nj > 1 && (eo_lds(n, nj) > 160 * 1024 || panels(nj) == panels(nj - 1))) --nj;
    while (nj > 1 && ntiles * panels(nj) < kEoFill) {
        --nj;
        while (nj > 1 && panels(nj) == panels(nj - 1)) --nj;
    }
    return nj;
}

bool xform_eo_supported(int n) {
    return n >= 1 && n <= kEoMaxN && eo_lds(n, 1) <= 160 * 1024;
}

// lane offsets of the strided axis (bytes in 32 bits): 16 lines over
// 16 / inner + 2 batches, one line deep
bool xform_eo_s_supported(int n, long inner) {
    return xform_eo_supported(n) && inner >= 1 && (16 / inner + 3) * n * inner < (1L << 29);
}

template <bool XAXIS, bool INV, int EPI, int NJ, bool REM>
static hipError_t eo_go(EoArgs a, hipStream_t st) {
    static std::atomic<bool> attr_set{false};       // set once; the attribute call is idempotent
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_xform_eo<XAXIS, INV, EPI, NJ, REM>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    a.npanel = (a.tiles + NJ - 1) / NJ;
    a.k4 = eo_rows(a.n);
    const size_t shm = eo_lds(a.n, NJ);
    // Persistent blocks of eight waves: as many as fit at once, a multiple of
    // 8 npanel, no more than the tiles need.
    const int nw = 8;
    const long per_cu = std::max<long>(1, std::min<long>((long)(160 * 1024 / shm), 4L * eo_waves<NJ>() / nw));
    const long unit = 8L * a.npanel;
    const long need = (a.ntiles + 7) / 8 * unit;
    const long fit = std::max(unit, 256 * per_cu / unit * unit);
    hipLaunchKernelGGL((k_xform_eo<XAXIS, INV, EPI, NJ, REM>), dim3((unsigned)std::min(need, fit)), dim3(64 * nw),
                       shm, st, a);
    return hipGetLastError();
}

template <bool XAXIS, bool INV, int EPI>
static hipError_t eo_launch(EoArgs a, hipStream_t st) {
    if (a.nlines <= 0) return hipSuccess;
    if (!xform_eo_supported(a.n)) return hipErrorInvalidValue;
    bool rem;
    a.tiles = eo_tiles(a.n, &rem);
    a.ntiles = (a.nlines + 15) / 16;
#define STH_EO_CASE(J) \
    case J: return rem ? eo_go<XAXIS, INV, EPI, J, true>(a, st) : eo_go<XAXIS, INV, EPI, J, false>(a, st);
    switch (eo_panel_tiles(a.n, a.ntiles)) {
        STH_EO_CASE(1) STH_EO_CASE(2) STH_EO_CASE(3) STH_EO_CASE(4) STH_EO_CASE(5)
        default: return hipErrorInvalidValue;
    }
#undef STH_EO_CASE
}

int xform_eo_rows(int n) { return eo_rows(n); }

size_t xform_eo_pack_len(int n) {
    bool rem;
    return xform_eo_supported(n) ? (size_t)eo_rows(n) * (32 * eo_tiles(n, &rem) + 2) : 0;
}

void xform_eo_pack(bool inv, const double* A, int n, int lda, double* out) {
    bool rem;
    const int h1 = (n + 1) / 2, h0 = n / 2, tiles = eo_tiles(n, &rem), k4 = eo_rows(n);
    // entry k of column j of a half: row k of A forward, row j (column k of the half) inverse
    auto entry = [&](int half, int k, int j) {
        const int kn = inv && half ? h0 : h1, jn = !inv && half ? h0 : h1;
        if (k >= kn || j >= jn) return 0.0;
        return inv ? A[(size_t)j * lda + (half ? h1 + k : k)] : A[(size_t)k * lda + (half ? h1 + j : j)];
    };
    for (int jt = 0; jt < tiles; ++jt)
        for (int k = 0; k < k4; ++k)
            for (int c = 0; c < 32; ++c) *out++ = entry(c / 16, k, 16 * jt + c % 16);
    for (int k = 0; k < k4; ++k)
        for (int half = 0; half < 2; ++half) *out++ = rem ? entry(half, k, 16 * tiles) : 0.0;
}

hipError_t launch_xform_eo_x(bool inv, int epi, const double* in, double* out, const double* T, int n,
                             long lines, double alpha, hipStream_t st, const int* guard) {
    const EoArgs a{in, out, T, guard, alpha, lines, 0, n, 1, 0, 0, 0};
    if (!inv) return epi == 0 ? eo_launch<true, false, 0>(a, st) : hipErrorInvalidValue;
    if (epi == 0) return eo_launch<true, true, 0>(a, st);
    if (epi == 1) return eo_launch<true, true, 1>(a, st);
    if (epi == 2) return eo_launch<true, true, 2>(a, st);
    return hipErrorInvalidValue;
}

hipError_t launch_xform_eo_s(bool inv, const double* in, double* out, const double* T, int n, long nbatch,
                             long inner, hipStream_t st, const int* guard) {
    if (!xform_eo_s_supported(n, inner)) return hipErrorInvalidValue;
    const EoArgs a{in, out, T, guard, 1.0, nbatch * inner, 0, n, (int)inner, 0, 0, 0};
    return inv ? eo_launch<false, true, 0>(a, st) : eo_launch<false, false, 0>(a, st);
}

}  // namespace sth
