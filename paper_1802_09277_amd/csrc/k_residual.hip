// gfx950 kernels of the space-time slab solver: the residual
//   r_n = f_n - A_n u_n + B_n u_{n-1} (eq. equ_linear_system, A_n = K_t (x) M_x
//   + M_t (x) K_x, B_n = N_t (x) M_x with N_t = e_1 e_{N_t}^T, eq. structureAn)
// by sum factorisation: banded 1-D passes of M_1/K_1, then the dense
// N_t x N_t contraction in registers.
#include <atomic>
#include <type_traits>

#include "kernels_common.hpp"

namespace sth {

// ---------------------------------------------------------------------------
// residual
// ---------------------------------------------------------------------------
template <int DIM> struct ResTile;
template <> struct ResTile<2> { static constexpr int TX = 32, TY = 8, TZ = 1; };
template <> struct ResTile<3> { static constexpr int TX = 8, TY = 8, TZ = 4; };

constexpr int kMaxP = 4;
constexpr int kBand = 2 * kMaxP + 1;

template <int DIM, int NT>
__global__ __launch_bounds__(256) void k_residual(int p, int n, const double* __restrict__ M1b,
                                                  const double* __restrict__ K1b, TimeOp op,
                                                  const double* __restrict__ f,
                                                  const double* __restrict__ u, double* __restrict__ r,
                                                  long s0, double sign, int tiles_x, int tiles_y) {
    using Tl = ResTile<DIM>;
    constexpr int TX = Tl::TX, TY = Tl::TY, TZ = Tl::TZ;
    constexpr int HXM = TX + 2 * kMaxP, HYM = TY + 2 * kMaxP, HZM = (DIM == 3) ? TZ + 2 * kMaxP : 1;
    __shared__ double Us[HZM * HYM * HXM];
    __shared__ double As[HZM * HYM * TX];
    __shared__ double Bs[HZM * HYM * TX];
    __shared__ double Cs[(DIM == 3) ? HZM * TY * TX : 1];
    __shared__ double Ds[(DIM == 3) ? HZM * TY * TX : 1];
    __shared__ double bxM[TX * kBand], bxK[TX * kBand], byM[TY * kBand], byK[TY * kBand];
    __shared__ double bzM[TZ * kBand], bzK[TZ * kBand];

    const int tid = threadIdx.x;
    const int B = 2 * p + 1;
    const int HX = TX + 2 * p, HY = TY + 2 * p, HZ = (DIM == 3) ? TZ + 2 * p : 1;
    int tile = blockIdx.x;
    const int tx = tile % tiles_x;
    tile /= tiles_x;
    const int ty = tile % tiles_y;
    const int tz = tile / tiles_y;
    const int gx0 = tx * TX, gy0 = ty * TY, gz0 = tz * TZ;
    const long s = s0 + blockIdx.y;
    long Nx = (long)n * n;
    if (DIM == 3) Nx *= n;
    const long slab_len = NT * Nx;

    // band rows of the tile
    for (int i = tid; i < TX * B; i += 256) {
        int lx = i / B, k = i % B, gx = gx0 + lx;
        bxM[lx * kBand + k] = (gx < n) ? M1b[(long)gx * B + k] : 0.0;
        bxK[lx * kBand + k] = (gx < n) ? K1b[(long)gx * B + k] : 0.0;
    }
    for (int i = tid; i < TY * B; i += 256) {
        int ly = i / B, k = i % B, gy = gy0 + ly;
        byM[ly * kBand + k] = (gy < n) ? M1b[(long)gy * B + k] : 0.0;
        byK[ly * kBand + k] = (gy < n) ? K1b[(long)gy * B + k] : 0.0;
    }
    if (DIM == 3) {
        for (int i = tid; i < TZ * B; i += 256) {
            int lz = i / B, k = i % B, gz = gz0 + lz;
            bzM[lz * kBand + k] = (gz < n) ? M1b[(long)gz * B + k] : 0.0;
            bzK[lz * kBand + k] = (gz < n) ? K1b[(long)gz * B + k] : 0.0;
        }
    }

    const int lx = tid % TX, ly = (tid / TX) % TY, lz = tid / (TX * TY);
    const int gx = gx0 + lx, gy = gy0 + ly, gz = gz0 + lz;
    const bool own = gx < n && gy < n && (DIM == 2 || gz < n);

    double acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = 0.0;

#pragma unroll
    for (int tr = 0; tr <= NT; ++tr) {
        const double* src;
        if (tr < NT) {
            src = u + s * slab_len + (long)tr * Nx;
        } else {
            if (s == 0) break;
            src = u + (s - 1) * slab_len + (long)(NT - 1) * Nx;   // end trace of slab n-1
        }
        __syncthreads();
        for (int i = tid; i < HZ * HY * HX; i += 256) {
            int hx = i % HX, hy = (i / HX) % HY, hz = i / (HX * HY);
            int x = gx0 - p + hx, y = gy0 - p + hy, z = gz0 - p + hz;
            double v = 0.0;
            if (x >= 0 && x < n && y >= 0 && y < n && (DIM == 2 || (z >= 0 && z < n))) {
                long off = (DIM == 3) ? ((long)z * n + y) * n + x : (long)y * n + x;
                v = src[off];
            }
            Us[(hz * HYM + hy) * HXM + hx] = v;
        }
        __syncthreads();
        // x pass: A = M1 u, B = K1 u along x
        for (int i = tid; i < HZ * HY * TX; i += 256) {
            int ix = i % TX, hy = (i / TX) % HY, hz = i / (TX * HY);
            const double* row = &Us[(hz * HYM + hy) * HXM + ix];
            double a = 0.0, b = 0.0;
            for (int k = 0; k < B; ++k) {
                a += bxM[ix * kBand + k] * row[k];
                b += bxK[ix * kBand + k] * row[k];
            }
            As[(hz * HYM + hy) * TX + ix] = a;
            Bs[(hz * HYM + hy) * TX + ix] = b;
        }
        __syncthreads();
        double Mu = 0.0, Ku = 0.0;
        if (DIM == 2) {
            for (int k = 0; k < B; ++k) {
                double a = As[(ly + k) * TX + lx], b = Bs[(ly + k) * TX + lx];
                Mu += byM[ly * kBand + k] * a;
                Ku += byK[ly * kBand + k] * a + byM[ly * kBand + k] * b;
            }
        } else {
            // y pass: C = M1y A, D = K1y A + M1y B
            for (int i = tid; i < HZ * TY * TX; i += 256) {
                int ix = i % TX, iy = (i / TX) % TY, hz = i / (TX * TY);
                double c = 0.0, d = 0.0;
                for (int k = 0; k < B; ++k) {
                    double a = As[(hz * HYM + iy + k) * TX + ix], b = Bs[(hz * HYM + iy + k) * TX + ix];
                    c += byM[iy * kBand + k] * a;
                    d += byK[iy * kBand + k] * a + byM[iy * kBand + k] * b;
                }
                Cs[(hz * TY + iy) * TX + ix] = c;
                Ds[(hz * TY + iy) * TX + ix] = d;
            }
            __syncthreads();
            for (int k = 0; k < B; ++k) {
                double c = Cs[((lz + k) * TY + ly) * TX + lx], d = Ds[((lz + k) * TY + ly) * TX + lx];
                Mu += bzM[lz * kBand + k] * c;
                Ku += bzK[lz * kBand + k] * c + bzM[lz * kBand + k] * d;
            }
        }
        if (tr < NT) {
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] -= op.Kt[t * kNt + tr] * Mu + op.Mt[t * kNt + tr] * Ku;
        } else {
            acc[0] += Mu;
        }
    }
    if (!own) return;
    long pt = (DIM == 3) ? ((long)gz * n + gy) * n + gx : (long)gy * n + gx;
    double* rs = r + s * slab_len + pt;
    const double* fs = f ? f + s * slab_len + pt : nullptr;
#pragma unroll
    for (int t = 0; t < NT; ++t) rs[(long)t * Nx] = (fs ? fs[(long)t * Nx] : 0.0) + sign * acc[t];
}

template <int DIM>
static hipError_t residual_dim(int Nt, int p, int n, const double* M1b, const double* K1b,
                               const TimeOp& op, const double* f, const double* u, double* r,
                               long s0, long ns, double sign, hipStream_t st) {
    using Tl = ResTile<DIM>;
    int tiles_x = (n + Tl::TX - 1) / Tl::TX, tiles_y = (n + Tl::TY - 1) / Tl::TY;
    int tiles_z = (DIM == 3) ? (n + Tl::TZ - 1) / Tl::TZ : 1;
    dim3 grid(tiles_x * tiles_y * tiles_z, (unsigned)ns);
#define STH_RES_CASE(NTV)                                                                          \
    case NTV:                                                                                      \
        if constexpr (DIM == 2 || NTV == 8) {                                                      \
            hipLaunchKernelGGL((k_residual<DIM, NTV>), grid, dim3(256), 0, st, p, n, M1b, K1b, op, \
                               f, u, r, s0, sign, tiles_x, tiles_y);                               \
            break;                                                                                 \
        }                                                                                          \
        return hipErrorInvalidValue;
    switch (Nt) {
        STH_RES_CASE(2) STH_RES_CASE(3) STH_RES_CASE(4) STH_RES_CASE(5)
        STH_RES_CASE(6) STH_RES_CASE(7) STH_RES_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef STH_RES_CASE
    return hipGetLastError();
}

// 2D residual with whole rows per block: thread column x (one per thread,
// TXT >= n threads across a row), RT thread rows, RY output rows per thread.
// Per time row of u: the (TY + 2P) x n strip is staged in LDS (x halo zero),
// the x pass (M_1, K_1 along x) goes to LDS, the y pass and the temporal
// contraction stay in registers.
constexpr int kRY = 4;

// MAXR: rows of the (TY + 2P)-row strip that one thread stages (RT = 1:
// kRY + 2P; RT >= 2: at most kRY + P)
template <int NT, int P, int MAXR>
__global__ __launch_bounds__(512) void k_residual2d(int n, int TXT, int RT, const double* __restrict__ M1b,
                                                     const double* __restrict__ K1b, const double* __restrict__ ktmt,
                                                     const double* __restrict__ f,
                                                     const double* __restrict__ u, double* __restrict__ r,
                                                     long s0, double sign) {
    constexpr int B = 2 * P + 1;
    extern __shared__ double sm[];
    const int TY = RT * kRY, HY = TY + 2 * P, W = n + 2 * P;
    double* Us = sm;
    double* As = Us + HY * W;
    double* Bs = As + HY * n;
    double* byM = Bs + HY * n;
    double* byK = byM + TY * B;
    const int nthreads = TXT * RT;
    const int tid = threadIdx.x;
    const int xr = tid % TXT, yr = tid / TXT;
    const int y0 = blockIdx.x * TY;
    const long s = s0 + blockIdx.y;
    const long Nx = (long)n * n, slab = NT * Nx;
    for (int i = tid; i < HY * 2 * P; i += nthreads) {
        int rr = i / (2 * P), c = i % (2 * P);
        Us[rr * W + (c < P ? c : n + c)] = 0.0;
    }
    for (int i = tid; i < TY * B; i += nthreads) {
        int gy = y0 + i / B;
        byM[i] = gy < n ? M1b[(long)gy * B + i % B] : 0.0;
        byK[i] = gy < n ? K1b[(long)gy * B + i % B] : 0.0;
    }
    const bool xin = xr < n;
    double bxM[B], bxK[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
        bxM[k] = xin ? M1b[(long)xr * B + k] : 0.0;
        bxK[k] = xin ? K1b[(long)xr * B + k] : 0.0;
    }
    double acc[kRY][NT];
#pragma unroll
    for (int i = 0; i < kRY; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[i][t] = 0.0;

    // rows of u needed per time row: staged through registers one time row
    // ahead, so the global loads of row tr+1 overlap the LDS passes of row tr
    const int NR = (s > 0) ? NT + 1 : NT;
    double pre[MAXR];
    auto load_rows = [&](int tr) {
        const double* src = (tr < NT) ? u + s * slab + (long)tr * Nx
                                       : u + (s - 1) * slab + (long)(NT - 1) * Nx;   // end trace of slab n-1
#pragma unroll
        for (int k = 0; k < MAXR; ++k) {
            const int rr = yr + RT * k, gy = y0 - P + rr;
            pre[k] = (xin && rr < HY && gy >= 0 && gy < n) ? src[(long)gy * n + xr] : 0.0;
        }
    };
    load_rows(0);
#pragma unroll 1
    for (int tr = 0; tr < NR; ++tr) {
        // column tr of K_t and M_t: uniform loads from the device copy
        double kc[NT], mc[NT];
        const int trc = tr < NT ? tr : 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            kc[t] = ktmt[t * kNt + trc];
            mc[t] = ktmt[kNt * kNt + t * kNt + trc];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < MAXR; ++k) {
            const int rr = yr + RT * k;
            if (xin && rr < HY) Us[rr * W + P + xr] = pre[k];
        }
        if (tr + 1 < NR) load_rows(tr + 1);
        __syncthreads();
        if (xin) {
            for (int rr = yr; rr < HY; rr += RT) {
                const double* row = Us + rr * W + xr;
                double a = 0.0, b = 0.0;
#pragma unroll
                for (int k = 0; k < B; ++k) {
                    a += bxM[k] * row[k];
                    b += bxK[k] * row[k];
                }
                As[rr * n + xr] = a;
                Bs[rr * n + xr] = b;
            }
        }
        __syncthreads();
        if (xin) {
#pragma unroll
            for (int i = 0; i < kRY; ++i) {
                const int ly = yr + RT * i;
                double Mu = 0.0, Ku = 0.0;
#pragma unroll
                for (int k = 0; k < B; ++k) {
                    double a = As[(ly + k) * n + xr], b = Bs[(ly + k) * n + xr];
                    double m = byM[ly * B + k];
                    Mu += m * a;
                    Ku += byK[ly * B + k] * a + m * b;
                }
                if (tr < NT) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[i][t] -= kc[t] * Mu + mc[t] * Ku;
                } else {
                    acc[i][0] += Mu;
                }
            }
        }
    }
    if (!xin) return;
#pragma unroll
    for (int i = 0; i < kRY; ++i) {
        const int gy = y0 + yr + RT * i;
        if (gy >= n) continue;
        const long off = s * slab + (long)gy * n + xr;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            double fv = f ? f[off + (long)t * Nx] : 0.0;
            r[off + (long)t * Nx] = fv + sign * acc[i][t];
        }
    }
}

template <int NT, int P, int MAXR>
static hipError_t residual2d_go(int n, const double* M1b, const double* K1b, const double* ktmt, const double* f,
                                const double* u, double* r, long s0, long ns, double sign, hipStream_t st) {
    int TXT = (n + 7) / 8 * 8;
    int RT = TXT >= 256 ? 1 : 256 / TXT;
    int TY = RT * kRY, HY = TY + 2 * P;
    size_t shm = sizeof(double) * ((size_t)HY * (n + 2 * P) + 2 * (size_t)HY * n + 2 * (size_t)TY * (2 * P + 1));
    const void* k = (const void*)k_residual2d<NT, P, MAXR>;
    static std::atomic<bool> attr_set{false};       // set once; the attribute call is idempotent
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const dim3 grid((unsigned)((n + TY - 1) / TY), (unsigned)ns);
    hipLaunchKernelGGL((k_residual2d<NT, P, MAXR>), grid, dim3(TXT * RT), shm, st, n, TXT, RT, M1b, K1b, ktmt, f,
                       u, r, s0, sign);
    return hipGetLastError();
}

template <int NT, int P>
static hipError_t residual2d_launch(int n, const double* M1b, const double* K1b, const double* ktmt,
                                    const double* f, const double* u, double* r, long s0, long ns, double sign,
                                    hipStream_t st) {
    if ((n + 7) / 8 * 8 > 128)                      // one thread row
        return residual2d_go<NT, P, kRY + 2 * P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
    return residual2d_go<NT, P, kRY + P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
}

template <int P>
static hipError_t residual2d_nt(int Nt, int n, const double* M1b, const double* K1b, const double* ktmt,
                                const double* f, const double* u, double* r, long s0, long ns, double sign,
                                hipStream_t st) {
    switch (Nt) {
        case 2: if (P + 1 <= 2) return residual2d_launch<2, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st); break;
        case 3: if (P + 1 <= 3) return residual2d_launch<3, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st); break;
        case 4: if (P + 1 <= 4) return residual2d_launch<4, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st); break;
        case 5: return residual2d_launch<5, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
        case 6: return residual2d_launch<6, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
        case 7: return residual2d_launch<7, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
        case 8: return residual2d_launch<8, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
        default: break;
    }
    return hipErrorInvalidValue;
}

// 2-D residual for large images: one wave per (slab, range of columns of x,
// range of YR rows of y), with no LDS and no barrier.  A wave's 64 lanes
// hold 64 consecutive columns; the P lanes at either end only supply the
// neighbours of the others (chunks of 64 - 2P output columns overlap by 2P).
// The wave marches along y: for each input row and time row it applies M_1
// and K_1 along x (neighbours by cross-lane reads), keeps the last 2P+1
// results per time row in registers, and completes each output row with the
// y pass and the temporal contraction (256^2 x 3 on 256 slabs 288 us, 128^2 x
// 4 on 256 113 us: 4.2 and 3.6 TB/s; LDS shuffles for the neighbours 292 and
// 120 us).  The next input row is loaded while
// the current one is processed.  With `partial` the block's sum of squares
// of r goes to partial[blockIdx.x] (fixed order).
// waves per SIMD the marching kernel asks for: 4 (at most 128 VGPRs) where
// its windows and time rows are small enough to fit them without spilling
// more than a few registers, else what the compiler picks
template <int NT, int P>
constexpr int march_waves() { return NT <= 4 && (NT + 1) * (2 * P + 1) <= 20 ? 4 : 1; }

template <int NT, int P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(march_waves<NT, P>())))
void k_residual2d_march(int n, int nxc, int nyr, int YR, long nwaves,
                                                          const double* __restrict__ M1b,
                                                          const double* __restrict__ K1b,
                                                          const double* __restrict__ ktmt,
                                                          const double* __restrict__ f,
                                                          const double* __restrict__ u, double* __restrict__ r,
                                                          long s0, double sign, double* __restrict__ partial) {
    constexpr int B = 2 * P + 1, NR = NT + 1;   // band width; time rows with the coupling row
    constexpr int XS = 64 - 2 * P;              // output columns per wave
    const int lane = threadIdx.x & 63;
    const long w = (long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double ssq = 0.0;
    if (w < nwaves) {
        const long per_slab = (long)nxc * nyr;
        const long s = s0 + w / per_slab;
        const int rem = (int)(w % per_slab);
        const int x = (rem % nxc) * XS - P + lane;
        const bool xin = x >= 0 && x < n;
        const bool xout = xin && lane >= P && lane < 64 - P;
        const int yb = (rem / nxc) * YR, ye = min(n, yb + YR);
        const long Nx = (long)n * n, slab = NT * Nx;
        const bool has_prev = s > 0;
        double bm[B], bk[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            bm[k] = xin ? M1b[(long)x * B + k] : 0.0;
            bk[k] = xin ? K1b[(long)x * B + k] : 0.0;
        }
        // input row y of time row tr (tr = NT: the last time row of slab s - 1)
        double v[NR];
        auto load = [&](int y) {
            const bool yin = y >= 0 && y < n;
#pragma unroll
            for (int tr = 0; tr < NR; ++tr) {
                const bool ok = yin && xin && (tr < NT || has_prev);
                const long base = tr < NT ? s * slab + (long)tr * Nx : (s - 1) * slab + (long)(NT - 1) * Nx;
                v[tr] = ok ? u[base + (long)y * n + x] : 0.0;
            }
        };
        double wa[NR][B], wb[NR][B];
#pragma unroll
        for (int tr = 0; tr < NR; ++tr)
#pragma unroll
            for (int k = 0; k < B; ++k) wa[tr][k] = wb[tr][k] = 0.0;
        // f of output row yo, loaded one input row ahead of its use
        double fv[NT];
        auto load_f = [&](int yo) {
            const bool ok = f && xout && yo >= yb && yo < ye;
            const long off = s * slab + (long)yo * n + x;
#pragma unroll
            for (int t = 0; t < NT; ++t) fv[t] = ok ? f[off + (long)t * Nx] : 0.0;
        };
        load(yb - P);
        load_f(yb - 2 * P);
#pragma unroll 1
        for (int y = yb - P; y < ye + P; ++y) {
            double cv[NR], fc[NT];
#pragma unroll
            for (int tr = 0; tr < NR; ++tr) cv[tr] = v[tr];
#pragma unroll
            for (int t = 0; t < NT; ++t) fc[t] = fv[t];
            if (y + 1 < ye + P) {
                load(y + 1);
                load_f(y + 1 - P);
            }
            // x pass of input row y for every time row, into the windows
            // (lanes whose neighbours fall outside the wave are not output)
#pragma unroll
            for (int tr = 0; tr < NR; ++tr) {
                double a = bm[P] * cv[tr], b = bk[P] * cv[tr];
                double up = cv[tr], dn = cv[tr];
#pragma unroll
                for (int d = 1; d <= P; ++d) {
                    up = wave_dpp<kDppWaveShl1, 0xf>(up);        // column x + d
                    dn = wave_dpp<kDppWaveShr1, 0xf>(dn);        // column x - d
                    a += bm[P + d] * up + bm[P - d] * dn;
                    b += bk[P + d] * up + bk[P - d] * dn;
                }
#pragma unroll
                for (int k = 0; k + 1 < B; ++k) {
                    wa[tr][k] = wa[tr][k + 1];
                    wb[tr][k] = wb[tr][k + 1];
                }
                wa[tr][B - 1] = a;
                wb[tr][B - 1] = b;
            }
            // output row y - P: y pass and temporal contraction
            const int yo = y - P;
            if (yo >= yb) {
                double cm[B], ck[B];
#pragma unroll
                for (int k = 0; k < B; ++k) {
                    cm[k] = M1b[(long)yo * B + k];
                    ck[k] = K1b[(long)yo * B + k];
                }
                double acc[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = 0.0;
#pragma unroll
                for (int tr = 0; tr < NT; ++tr) {
                    double Mu = 0.0, Ku = 0.0;
#pragma unroll
                    for (int k = 0; k < B; ++k) {
                        Mu += cm[k] * wa[tr][k];
                        Ku += ck[k] * wa[tr][k] + cm[k] * wb[tr][k];
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[t] -= ktmt[t * kNt + tr] * Mu + ktmt[kNt * kNt + t * kNt + tr] * Ku;
                }
                double Mc = 0.0;                         // B_n u_{n-1}: M_x on the coupling row
#pragma unroll
                for (int k = 0; k < B; ++k) Mc += cm[k] * wa[NT][k];
                acc[0] += Mc;
                if (xout) {
                    const long off = s * slab + (long)yo * n + x;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const double val = fc[t] + sign * acc[t];
                        r[off + (long)t * Nx] = val;
                        ssq += val * val;
                    }
                }
            }
        }
    }
    if (partial) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ssq += __shfl_xor(ssq, off);
        __shared__ double red[4];
        if (lane == 0) red[threadIdx.x >> 6] = ssq;
        __syncthreads();
        if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

// ---------------------------------------------------------------------------
// 3-D residual, marching along z.  A thread stands on one (x, y) column of
// its block's tile and walks down z with the last 2P+1 planes of every time
// row (and of the coupling row, the last time row of slab s - 1) in
// registers.  Per output plane the z pass and the temporal contraction come
// first, in registers:
//   al_t = sum_tr K_t[t][tr] M_z u_tr + M_t[t][tr] K_z u_tr - [t = 0] M_z u_{s-1},
//   be_t = sum_tr M_t[t][tr] M_z u_tr,
// so that r_t = f_t - M_y (M_x al_t + K_x be_t) - K_y M_x be_t leaves five
// banded sums in the plane: the two x ones read al, be from LDS, the y ones
// read their results from LDS (two barriers per plane).
// Tiles are hx x hy columns; an axis that the tile covers whole needs no
// halo (hpx, hpy = 0), otherwise the outer P columns only feed the others.
// About 7 (2P+1) + 3 N_t FP64 multiply-adds and 4 (2P+1) LDS reads per
// unknown, times the halo (1.4 at n = 33): issue and LDS bound it, ahead of
// the 24 B per unknown.  100 slabs of 33^3 x 4 unknowns (P = 2): 150 us,
// 2.3 TB/s algorithmic, against 1212 us of a kernel with a tile in LDS per
// time row and eight times the LDS passes; 50 slabs of 22^3 x 4 (P = 3): 43
// against 238 us.
// ---------------------------------------------------------------------------
constexpr int kRes3Threads = 512;

// Registers: the window takes 2 (N_t + 1)(2P + 1) VGPRs.  Small ones leave
// room for two blocks per compute unit (128 VGPRs) with the in-plane sums one
// band entry at a time; in the middle one block with these sums unrolled,
// their LDS loads in flight together, is faster (N_t = 4, P = 2: 150 us
// against 178 us at 128 VGPRs; N_t = 3, P = 2: 89 against 65 us); large ones
// spill when unrolled.
template <int NT, int P> constexpr int res3_waves() { return (NT + 1) * (2 * P + 1) <= 20 && P > 1 ? 4 : 2; }
template <int NT, int P> constexpr int res3_unroll() {
    constexpr bool spills = (NT + 1) * (2 * P + 1) > 35 || NT > 7 - P;
    return spills || res3_waves<NT, P>() == 4 ? 1 : 2 * P + 1;
}

template <int NT, int P>
__global__ __launch_bounds__(kRes3Threads) __attribute__((amdgpu_waves_per_eu(res3_waves<NT, P>())))
void k_residual3d(int n, int hx_n, int hy_n, int hpx, int hpy, int tiles_x,
                                                             int tiles_y, int zc, int nzc, long nblocks,
                                                             const double* __restrict__ M1b,
                                                             const double* __restrict__ K1b,
                                                             const double* __restrict__ ktmt,
                                                             const double* __restrict__ f,
                                                             const double* __restrict__ u, double* __restrict__ r,
                                                             long s0, double sign) {
    constexpr int B = 2 * P + 1, NR = NT + 1;
    extern __shared__ double sm[];
    const int lx_n = hx_n + 2 * P, ly_n = hy_n + 2 * P;
    const int apl = hy_n * lx_n, xpl = ly_n * hx_n;
    double* al = sm;                            // [2 NT][hy_n][lx_n]: al_t, be_t, zero columns at either end
    double* xs = al + 2 * NT * apl;             // [2 NT][ly_n][hx_n]: M_x al + K_x be, M_x be; zero rows
    double* bx = xs + 2 * NT * xpl;             // [2 B][hx_n] bands of the tile's columns, k-major
    double* by = bx + 2 * B * hx_n;             // [2 B][hy_n]
    const int tid = threadIdx.x;
    const int hx = tid % hx_n, hy = tid / hx_n;
    // consecutive blocks (neighbours in a slab, which share halo columns) on one XCD
    const long q8 = nblocks / 8, r8 = nblocks % 8;
    const long xcd = blockIdx.x % 8, at = blockIdx.x / 8;
    long blk = xcd * q8 + (xcd < r8 ? xcd : r8) + at;
    const int tx = (int)(blk % tiles_x);
    blk /= tiles_x;
    const int ty = (int)(blk % tiles_y);
    blk /= tiles_y;
    const int zi0 = (int)(blk % nzc) * zc;
    const long s = s0 + blk / nzc;
    const int ze = min(n, zi0 + zc);
    const int gx = tx * (hx_n - 2 * hpx) - hpx + hx, gy = ty * (hy_n - 2 * hpy) - hpy + hy;
    const bool pos = hy < hy_n;
    const bool in = pos && gx >= 0 && gx < n && gy >= 0 && gy < n;
    const bool outx = in && hx >= hpx && hx < hx_n - hpx;
    const bool out = outx && hy >= hpy && hy < hy_n - hpy;
    const long Np = (long)n * n, Nx = Np * n, slab = NT * Nx;
    for (int i = tid; i < 2 * NT * apl; i += blockDim.x) al[i] = 0.0;
    for (int i = tid; i < 2 * NT * xpl; i += blockDim.x) xs[i] = 0.0;
    for (int i = tid; i < B * hx_n; i += blockDim.x) {
        const int k = i / hx_n, g = tx * (hx_n - 2 * hpx) - hpx + i % hx_n;
        bx[i] = g >= 0 && g < n ? M1b[(long)g * B + k] : 0.0;
        bx[B * hx_n + i] = g >= 0 && g < n ? K1b[(long)g * B + k] : 0.0;
    }
    for (int i = tid; i < B * hy_n; i += blockDim.x) {
        const int k = i / hy_n, g = ty * (hy_n - 2 * hpy) - hpy + i % hy_n;
        by[i] = g >= 0 && g < n ? M1b[(long)g * B + k] : 0.0;
        by[B * hy_n + i] = g >= 0 && g < n ? K1b[(long)g * B + k] : 0.0;
    }
    __syncthreads();
    const long col = (long)gy * n + gx;
    const bool has_prev = in && s > 0;
    double w[B][NR], v[NR];
    auto load = [&](int z) {
        const bool zin = z >= 0 && z < n;
#pragma unroll
        for (int tr = 0; tr < NR; ++tr) {
            const bool ok = zin && (tr < NT ? in : has_prev);
            const long base = tr < NT ? s * slab + (long)tr * Nx : (s - 1) * slab + (long)(NT - 1) * Nx;
            v[tr] = ok ? u[base + z * Np + col] : 0.0;
        }
    };
    // input plane zi into window slot PH, and output plane zi - P from it
    auto plane = [&](auto ph, int zi) {
        constexpr int PH = decltype(ph)::value;
#pragma unroll
        for (int tr = 0; tr < NR; ++tr) w[PH][tr] = v[tr];
        if (zi + 1 < ze + P) load(zi + 1);
        const int z = zi - P;
        if (z < zi0) return;
        double fv[NT];
        const long off = s * slab + z * Np + col;
#pragma unroll
        for (int t = 0; t < NT; ++t) fv[t] = (f && out) ? f[off + (long)t * Nx] : 0.0;
        double mu[NR], ku[NT];
#pragma unroll
        for (int tr = 0; tr < NR; ++tr) mu[tr] = 0.0;
#pragma unroll
        for (int tr = 0; tr < NT; ++tr) ku[tr] = 0.0;
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const double m = M1b[(long)z * B + k], kk = K1b[(long)z * B + k];
#pragma unroll
            for (int tr = 0; tr < NR; ++tr) {
                mu[tr] += m * w[(PH + 1 + k) % B][tr];
                if (tr < NT) ku[tr] += kk * w[(PH + 1 + k) % B][tr];
            }
        }
        if (pos) {
            double* ap = al + hy * lx_n + P + hx;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                double a = t == 0 ? -mu[NT] : 0.0, b = 0.0;
#pragma unroll
                for (int tr = 0; tr < NT; ++tr) {
                    const double kt = ktmt[t * kNt + tr], mt = ktmt[kNt * kNt + t * kNt + tr];
                    a += kt * mu[tr] + mt * ku[tr];
                    b += mt * mu[tr];
                }
                ap[t * apl] = a;
                ap[(NT + t) * apl] = b;
            }
        }
        __syncthreads();
        if (outx) {
            const double* ap = al + hy * lx_n + hx;
            double e[NT], b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) e[t] = b[t] = 0.0;
#pragma unroll res3_unroll<NT, P>()
            for (int k = 0; k < B; ++k) {
                const double m = bx[k * hx_n + hx], kk = bx[(B + k) * hx_n + hx];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const double at = ap[t * apl + k], bt = ap[(NT + t) * apl + k];
                    e[t] += m * at + kk * bt;
                    b[t] += m * bt;
                }
            }
            double* xp = xs + (hy + P) * hx_n + hx;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                xp[t * xpl] = e[t];
                xp[(NT + t) * xpl] = b[t];
            }
        }
        __syncthreads();
        if (out) {
            const double* xp = xs + hy * hx_n + hx;
            double acc[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = 0.0;
#pragma unroll res3_unroll<NT, P>()
            for (int k = 0; k < B; ++k) {
                const double m = by[k * hy_n + hy], kk = by[(B + k) * hy_n + hy];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] += m * xp[t * xpl + k * hx_n] + kk * xp[(NT + t) * xpl + k * hx_n];
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) r[off + (long)t * Nx] = fv[t] - sign * acc[t];
        }
    };
    load(zi0 - P);
    // the window slot of a plane is a compile-time index: B planes per trip
    // (zi is uniform over the block, so the barriers are reached by all)
#pragma unroll 1
    for (int zi = zi0 - P; zi < ze + P; zi += B) {
        plane(std::integral_constant<int, 0>{}, zi);
        if (zi + 1 < ze + P) plane(std::integral_constant<int, 1>{}, zi + 1);
        if (zi + 2 < ze + P) plane(std::integral_constant<int, 2>{}, zi + 2);
        if constexpr (B > 3) {
            if (zi + 3 < ze + P) plane(std::integral_constant<int, 3>{}, zi + 3);
            if (zi + 4 < ze + P) plane(std::integral_constant<int, 4>{}, zi + 4);
        }
        if constexpr (B > 5) {
            if (zi + 5 < ze + P) plane(std::integral_constant<int, 5>{}, zi + 5);
            if (zi + 6 < ze + P) plane(std::integral_constant<int, 6>{}, zi + 6);
        }
        if constexpr (B > 7) {
            if (zi + 7 < ze + P) plane(std::integral_constant<int, 7>{}, zi + 7);
            if (zi + 8 < ze + P) plane(std::integral_constant<int, 8>{}, zi + 8);
        }
    }
}

// Tile of the 3-D residual: the hx x hy columns (at most 512 threads, LDS for
// two blocks per compute unit if some tile allows it, else for one) with the
// fewest threads over the whole image, halo and overhang included.  (The search
// takes 2 to 5 us of host time: once, at set-up.)
bool residual3d_tile(int Nt, int p, int n, Res3Tile* best) {
    const int B = 2 * p + 1;
    for (size_t cap : {size_t(80) * 1024, size_t(160) * 1024}) {
        long cost = -1;
        for (int hx = 1; hx <= n && hx <= kRes3Threads; ++hx) {
            const int hpx = hx == n ? 0 : p;
            if (hx - 2 * hpx < 1) continue;
            for (int hy = 1; hy <= n && hx * hy <= kRes3Threads; ++hy) {
                const int hpy = hy == n ? 0 : p;
                if (hy - 2 * hpy < 1) continue;
                const size_t shm = sizeof(double) * (2 * (size_t)Nt * (hy * (hx + 2 * p) + (hy + 2 * p) * hx) +
                                                     2 * (size_t)B * (hx + hy));
                if (shm > cap) continue;
                const int tx = (n + hx - 2 * hpx - 1) / (hx - 2 * hpx), ty = (n + hy - 2 * hpy - 1) / (hy - 2 * hpy);
                const long c = (long)tx * ty * ((hx * hy + 63) / 64);
                if (cost < 0 || c < cost || (c == cost && hx > best->hx)) {
                    cost = c;
                    *best = Res3Tile{hx, hy, hpx, hpy, tx, ty, shm};
                }
            }
        }
        if (cost >= 0) return true;
    }
    return false;
}

// output planes per block: all of them, or fewer where the slabs and tiles
// alone leave compute units idle; a chunk of zc planes walks zc + 2p input
// planes, of which the 2p halo ones cost about a third of an output plane
// (loads, no passes)
static int residual3d_planes(int n, int p, long tiles) {
    int best = n;
    double cost = -1.0;
    for (int c = 1; c <= n;) {          // (each chunk length once, with its fewest chunks)
        const int zc = (n + c - 1) / c;
        c = zc > 1 ? (n + zc - 2) / (zc - 1) : n + 1;
        const long blocks = tiles * ((n + zc - 1) / zc);
        const double t = (double)((blocks + 511) / 512) * (zc + 2 * p / 3.0);
        if (cost < 0 || t < cost) {
            cost = t;
            best = zc;
        }
    }
    return best;
}

template <int NT, int P>
static hipError_t residual3d_launch(int n, const double* M1b, const double* K1b, const double* ktmt, const double* f,
                                    const double* u, double* r, long s0, long ns, double sign, const Res3Tile& t,
                                    hipStream_t st) {
    if (!t.hx) return hipErrorInvalidValue;
    static std::atomic<bool> attr_set{false};       // set once; the attribute call is idempotent
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_residual3d<NT, P>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set.store(true, std::memory_order_release);
    }
    const long tiles = ns * t.tiles_x * t.tiles_y;
    const int zc = residual3d_planes(n, P, tiles), nzc = (n + zc - 1) / zc;
    const long blocks = tiles * nzc;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_residual3d<NT, P>), dim3((unsigned)blocks), dim3((t.hx * t.hy + 63) / 64 * 64), t.shm, st, n,
                       t.hx, t.hy, t.hpx, t.hpy, t.tiles_x, t.tiles_y, zc, nzc, blocks, M1b, K1b, ktmt, f, u, r, s0,
                       sign);
    return hipGetLastError();
}

template <int P>
static hipError_t residual3d_nt(int Nt, int n, const double* M1b, const double* K1b, const double* ktmt,
                                const double* f, const double* u, double* r, long s0, long ns, double sign,
                                const Res3Tile& t, hipStream_t st) {
#define STH_R3_CASE(NTV)                                                                                      \
    case NTV:                                                                                                  \
        if constexpr (NTV > P && !(P == 4 && NTV == 8))                                                        \
            return residual3d_launch<NTV, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, t, st);                 \
        return hipErrorInvalidValue;
    switch (Nt) {
        STH_R3_CASE(2) STH_R3_CASE(3) STH_R3_CASE(4) STH_R3_CASE(5) STH_R3_CASE(6) STH_R3_CASE(7) STH_R3_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef STH_R3_CASE
}

// rows of y per wave of the marching kernel: the longest range that still
// gives at least 8192 waves (halo rows: 2P per range)
static int march_rows(int n, int p, long ns) {
    const long nxc = (n + 63 - 2 * p) / (64 - 2 * p);
    for (int yr : {128, 64, 32})
        if (ns * nxc * ((n + yr - 1) / yr) >= 8192) return yr;
    return 16;
}

template <int NT, int P>
static hipError_t residual2d_march_launch(int n, const double* M1b, const double* K1b, const double* ktmt,
                                          const double* f, const double* u, double* r, long s0, long ns, double sign,
                                          double* partial, long* nblocks, hipStream_t st) {
    const int nxc = (n + 63 - 2 * P) / (64 - 2 * P), YR = march_rows(n, P, ns), nyr = (n + YR - 1) / YR;
    const long nwaves = ns * nxc * nyr, blocks = (nwaves + 3) / 4;
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    if (nblocks) *nblocks = blocks;
    hipLaunchKernelGGL((k_residual2d_march<NT, P>), dim3((unsigned)blocks), dim3(256), 0, st, n, nxc, nyr, YR, nwaves,
                       M1b, K1b, ktmt, f, u, r, s0, sign, partial);
    return hipGetLastError();
}

template <int P>
static hipError_t residual2d_march_nt(int Nt, int n, const double* M1b, const double* K1b, const double* ktmt,
                                      const double* f, const double* u, double* r, long s0, long ns, double sign,
                                      double* partial, long* nblocks, hipStream_t st) {
#define STH_RM_CASE(NTV)                                                                                    \
    case NTV:                                                                                                \
        if constexpr (2 * (NTV + 1) * (2 * P + 1) <= 64)                                                     \
            return residual2d_march_launch<NTV, P>(n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, partial, nblocks, st); \
        return hipErrorInvalidValue;
    switch (Nt) {
        STH_RM_CASE(2) STH_RM_CASE(3) STH_RM_CASE(4) STH_RM_CASE(5) STH_RM_CASE(6) STH_RM_CASE(7) STH_RM_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef STH_RM_CASE
}

// the marching kernel serves 2-D images of 128 or more columns where its
// windows (2 (N_t + 1)(2p + 1) doubles per lane) fit the registers
static bool residual_marches(int dim, int n, int p, int Nt) {
    return dim == 2 && n >= 128 && p >= 1 && p <= kMaxP && 2 * (Nt + 1) * (2 * p + 1) <= 64;
}

// ... and narrower ones where its waves' columns are used to 60 % and fill 900
// waves of 16 rows (its chain over the rows is long): 101^2 x 3 on 300 slabs
// 78 -> 59 us, on 20 slabs 13 against 19; 79^2 x 4 on 160 40 -> 33; 60^2 x 3 on
// 400 38 -> 28, but 62^2 (two ranges of 60 columns) 38 against 40; 70^2 x 3 on
// 120 18 against 27.
static bool residual_marches_narrow(int n, int p, int Nt, long ns) {
    const long xs = 64 - 2 * p, nxc = (n + xs - 1) / xs;
    return p >= 1 && 2 * (Nt + 1) * (2 * p + 1) <= 64 && 10 * n >= 6 * nxc * xs && ns * n * n >= 900 * 16 * xs;
}

hipError_t launch_residual_norm(int dim, int Nt, int p, int n, const double* M1b, const double* K1b,
                                const double* ktmt, const double* f, const double* u, double* r, long ns,
                                double* partial, long max_partial, double* out, double* out_host, hipStream_t st) {
    if (ns <= 0) return hipSuccess;
    if (!residual_marches(dim, n, p, Nt)) return hipErrorInvalidValue;
    const int nxc = (n + 63 - 2 * p) / (64 - 2 * p), YR = march_rows(n, p, ns), nyr = (n + YR - 1) / YR;
    if ((ns * nxc * nyr + 3) / 4 > max_partial) return hipErrorInvalidValue;
    long blocks = 0;
    hipError_t e;
    switch (p) {
        case 1: e = residual2d_march_nt<1>(Nt, n, M1b, K1b, ktmt, f, u, r, 0, ns, 1.0, partial, &blocks, st); break;
        case 2: e = residual2d_march_nt<2>(Nt, n, M1b, K1b, ktmt, f, u, r, 0, ns, 1.0, partial, &blocks, st); break;
        case 3: e = residual2d_march_nt<3>(Nt, n, M1b, K1b, ktmt, f, u, r, 0, ns, 1.0, partial, &blocks, st); break;
        default: e = residual2d_march_nt<4>(Nt, n, M1b, K1b, ktmt, f, u, r, 0, ns, 1.0, partial, &blocks, st); break;
    }
    if (e != hipSuccess) return e;
    return launch_sum_partials(partial, (int)blocks, out, out_host, 1, nullptr, CycleFlag{}, st);
}

bool residual_norm_fused(int dim, int n, int p, int Nt) { return residual_marches(dim, n, p, Nt); }

hipError_t launch_residual(int dim, int Nt, int p, int n, const double* M1b, const double* K1b,
                           const TimeOp& op, const double* ktmt, const double* f, const double* u, double* r,
                           long s0, long ns, double sign, const Res3Tile& tile, hipStream_t st) {
    if (ns <= 0) return hipSuccess;
    if (p < 1 || p > kMaxP) return hipErrorInvalidValue;
    if (residual_marches(dim, n, p, Nt) || (dim == 2 && residual_marches_narrow(n, p, Nt, ns))) {
        switch (p) {
            case 1: return residual2d_march_nt<1>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, nullptr, nullptr, st);
            case 2: return residual2d_march_nt<2>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, nullptr, nullptr, st);
            case 3: return residual2d_march_nt<3>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, nullptr, nullptr, st);
            case 4: return residual2d_march_nt<4>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, nullptr, nullptr, st);
        }
    }
    if (dim == 2) {
        int TXT = (n + 7) / 8 * 8, RT = TXT >= 256 ? 1 : 256 / TXT;
        int TY = RT * kRY, HY = TY + 2 * p;
        size_t shm = sizeof(double) * ((size_t)HY * (n + 2 * p) + 2 * (size_t)HY * n + 2 * (size_t)TY * (2 * p + 1));
        if (shm > 150 * 1024 || TXT * RT > 512) return residual_dim<2>(Nt, p, n, M1b, K1b, op, f, u, r, s0, ns, sign, st);
        switch (p) {
            case 1: return residual2d_nt<1>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
            case 2: return residual2d_nt<2>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
            case 3: return residual2d_nt<3>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
            case 4: return residual2d_nt<4>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, st);
        }
    }
    if (dim == 3) {
        // degree 4 with 8 time rows: the window of the marching kernel spills
        // (1090 us against 933 us of the per-tile kernel on 40 slabs of 32^3 x 8;
        // with 7 rows it is ahead, 763 against 828 us)
        if (p == 4 && Nt == 8) return residual_dim<3>(Nt, p, n, M1b, K1b, op, f, u, r, s0, ns, sign, st);
        switch (p) {
            case 1: return residual3d_nt<1>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, tile, st);
            case 2: return residual3d_nt<2>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, tile, st);
            case 3: return residual3d_nt<3>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, tile, st);
            case 4: return residual3d_nt<4>(Nt, n, M1b, K1b, ktmt, f, u, r, s0, ns, sign, tile, st);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace sth
