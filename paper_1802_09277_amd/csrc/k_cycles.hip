// gfx950 kernels of the space-time slab solver: whole V(1,1) cycles of the
// time-parallel multigrid (Section 3.1) in the spatial eigenbasis, on chip.
//
// In the eigenbasis a cycle couples nothing across spatial modes, and the
// time line of one mode (up to 1024 slabs on every level) fits the registers
// of one wave: lane g keeps LA consecutive finest-level slabs, and LA/2,
// LA/4, LA/8 slabs of the levels below.  The wave reads the residual
// r^ = f^ - L u^ once, takes m cycles and writes r^ once: the cycles are taken
// on the residual alone,
//   smoothing step  u += omega A^{-1} r :  r <- (1 - omega) r + e_1 delta,
//     delta = omega (last row of A^{-1}) r of the previous slab;
//   correction      u += P e            :  r <- r - (A P) e + e_1 (P e)[last, previous slab],
// (D = diag(A) is the smoother's block, so A A^{-1} r = r), and on the coarse
// levels, which start from zero, u = omega A^{-1} f on the way down and the
// closed form u' = (2 - omega) u + (1 - omega) P e + omega q A^{-1} e_1 on the
// way up (q the coupling row of the previous slab of u + P e).  The iterate
// that belongs to a residual is formed once, at the end:
//   u^ = L^{-1}(f^ - r^), the exact solve parallel in time.
// Residual norms of every cycle come out with it, so the host decides on
// convergence after a batch of cycles.
//
// One mode per wave makes the N_t x N_t matrices of the mode (A_l^{-1} per
// level, A P_h; a table formed at setup) wave-uniform: they are scalar loads
// and scalar operands of the multiply-adds, whose vector registers are left to
// the time line (modes across the lanes kept them in vector registers or LDS:
// 3.9 ms per batch against 2.2 ms on 65536 modes x 1024 slabs x 3).  Rows
// between lanes and the recurrence x_s = a_s + gamma x_{s-1} of the exact
// solve go by data-parallel primitives (through LDS shuffles 9 to 14 % slower);
// no barrier inside a cycle.  A block takes eight modes, pieces of 64 bytes of
// each row (float: 32), transposed through LDS on the way in and out.  (Blocks
// of 16, whole lines, are 4 to 15 % slower in whole solves of 8 thousand to 262
// thousand modes, in float as well: one block per compute unit, whose transfers
// nothing overlaps.)
//
// A cycle takes about 5 N_t + 10 multiply-adds per unknown and no memory
// traffic, against 40 B per unknown of passes over the vectors level by
// level; a batch moves 16 B per unknown, 24 with the iterate.  On 65536 modes
// x 1024 slabs x 3 (1.6 GB vectors) a cycle takes 0.13 ms; a batch of 8 takes
// 1.23 ms, one of 2 1.13 ms and 2.04 ms with the iterate: there the transfers
// bound it (2.4 to 2.9 TB/s by rows of modes, 3.7 by time lines; one block per
// compute unit at 250 registers, so little of them overlaps the cycles).
// Solves, from passes level by level: the 12 cycles there 24.2 -> 8.6 ms,
// 4489 modes x 256 slabs x 5 1082 -> 262 us, 1024 x 16 x 4 114 -> 36 us (with
// the transforms and launches that changed besides).
#include <algorithm>

#include "kernels_common.hpp"

namespace sth {

struct CycArgs {
    int L, m;
    int steps;                  // damped block-Jacobi steps instead of cycles (ONE, m = 0)
    int rin_lines, rout_lines;  // residual by time lines: [mode][row of a lane][lane]
    long S, Nx;
    double omega;
    // per mode: A_l^{-1} (l < L), A P_0, A P_1 (one level: A), the two norm
    // weights; behind the last mode P (2 N_t x N_t)
    const double* tab;
    const void* rin;
    const void* fh;
    void* rout;
    void* uout;
    double* partial;            // [cycle 0..m][3][gridDim], or null
};

static int tab_len(int Nt, int L) { return (L + (L > 1 ? 2 : 1)) * Nt * Nt + 2; }

// Column c of A^{-1} of one level for the mode shift mu, with one step of
// iterative refinement against A = K_t + mu M_t: the solve through the
// temporal eigenvectors is accurate to their condition number (up to 1e6)
// times the rounding, which the residual form would leave in the result.
template <int NT>
__device__ __forceinline__ void inverse_column(const TimeMix& tm, const double* ktmt, double mu, int c, double* z) {
    double e[NT], d[NT];
    auto solve = [&](const double* b, double* x) {
        if (tm.schur) shifted_solve<NT, true>(tm, mu, b, x);
        else shifted_solve<NT, false>(tm, mu, b, x);
    };
#pragma unroll
    for (int t = 0; t < NT; ++t) e[t] = t == c ? 1.0 : 0.0;
    solve(e, z);
    eig_residual_point<NT>(ktmt, mu, z, 0.0, e);
    solve(e, d);
#pragma unroll
    for (int t = 0; t < NT; ++t) z[t] += d[t];
}

// the table of CycArgs::tab, one thread per mode and matrix column
template <int NT>
__global__ __launch_bounds__(256) void k_mode_table(int dim, int n, int L, long Nx, const TimeMix* __restrict__ tm,
                                                    const double* __restrict__ ktmt, const double* __restrict__ mu1,
                                                    const double* __restrict__ vw, Transfer tr,
                                                    double* __restrict__ tab, int len) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const int cols = (L + (L > 1 ? 2 : 1)) * NT;
    const long m = idx / cols;
    const int q = (int)(idx % cols), l = q / NT, c = q % NT;
    if (m >= Nx) return;
    const double mu = mode_shift(dim, mu1, n, m);
    double z[NT];
    if (l < L) {
        inverse_column<NT>(tm[l], ktmt + (long)l * 2 * kNt * kNt, mu, c, z);
    } else {
        // column c of A P_h, or of A
        for (int t = 0; t < NT; ++t) {
            double v = 0.0;
            for (int k = 0; k < NT; ++k) {
                const double p = L > 1 ? tr.P[((l - L) * NT + k) * kNt + c] : (k == c ? 1.0 : 0.0);
                v += (ktmt[t * kNt + k] + mu * ktmt[kNt * kNt + t * kNt + k]) * p;
            }
            z[t] = v;
        }
    }
    double* o = tab + m * len + l * NT * NT + c;
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t * NT] = z[t];
    if (m == 0 && q < NT)                       // P, behind the last mode
        for (int i = 0; i < 2 * NT; ++i) tab[Nx * len + i * NT + c] = tr.P[i * kNt + c];
    if (q == 0) {
        const ModeWeights w = vw ? mode_weights(dim, vw, n, m) : ModeWeights{0.0, 0.0};
        tab[m * len + len - 2] = w.lo;
        tab[m * len + len - 1] = w.up;
    }
}

// wave-uniform tables: scalar loads
typedef const __attribute__((address_space(4))) double* uptr;

// ONE: a single level.  A cycle is the exact solve e = L^{-1} r, whose result
// goes to uout, and r becomes its residual r - L e (m = 1).
// Waves per SIMD to leave registers for: two blocks of 8 per compute unit up
// to 24 values per lane, so that one block's transfers overlap the other's
// cycles (a first batch of 8 on 65536 modes x 512 slabs x 3: 722 against 1094
// us; 10404 modes x 150 slabs x 6: 128 against 170 us a batch; a handful of
// spilled registers costs less), else one block.
constexpr int MB = 8;                           // modes (waves) per block
template <int NT, int LA> constexpr int cycles_waves() { return LA * NT <= 24 ? 4 : 2; }
template <int NT, int LA, typename VT, bool ONE>
__global__ __launch_bounds__(64 * MB) __attribute__((amdgpu_waves_per_eu(cycles_waves<NT, LA>()))) void k_cycles(CycArgs a, int len) {
    constexpr int NM = NT * NT, E = LA * NT;
    constexpr int KB = E < 12 ? E : 12;         // rows per transposition
    constexpr int PITCH = 72;                   // 64 lanes, padded against bank conflicts of the eight modes
    __shared__ double tile[KB][MB][PITCH];
    __shared__ double red[MB][kMaxBatch + 1][3];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The blocks of one XCD take a contiguous range of modes, so that the lines
    // that neighbours share stay in its L2 (against eight modes' neighbours only:
    // 66564 modes x 64 slabs x 6, whose rows do not start on a line, 270 -> 236
    // us, 65536 x 1024 x 3 1.32 -> 1.21 ms).
    const long m0 = ((long)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8) * MB;
    const long mode = m0 + wave < a.Nx ? m0 + wave : a.Nx - 1;
    const double* tab0 = a.tab + mode * len;
    const double* ptab0 = a.tab + a.Nx * len;
    // Uniform matrices, as opaque pointers formed for each phase: their entries
    // are loaded (scalar cache) where they are used instead of being kept, and
    // spilled, across the phases of a cycle.
    auto mat = [&](int l) {                     // A_l^{-1}; L, L + 1: A P_h; L + 2: weights
        const double* p = tab0 + l * NM;
        asm volatile("" : "+s"(p));
        return (uptr)(unsigned long long)p;
    };
    auto transfer = [&] {
        const double* p = ptab0;
        asm volatile("" : "+s"(p));
        return (uptr)(unsigned long long)p;
    };
    const double om = a.omega;
    const int nv = (int)max(0L, min((long)LA, a.S - (long)lane * LA));      // slabs of this lane inside the line
    double r[LA][NT];

    // rows of MB modes <-> time lines: element e = (slab i, row t) of
    // lane g is row g E + e
    const int cw = tid % MB, cg = tid / MB;       // the thread's mode and lane on the row side
    const long cm = m0 + cw;
    const int ce = cm < a.Nx ? NT * (int)max(0L, min((long)LA, a.S - (long)cg * LA)) : 0;    // its valid rows
    const long c0 = (long)cg * E * a.Nx + cm;
    // (the loads of two transpositions ahead are in flight)
    auto read = [&](const void* src, auto&& use) {
        const VT* p = static_cast<const VT*>(src) + c0;
        constexpr int NC = (E + KB - 1) / KB;
        VT v[2][KB];
        auto load = [&](int c, VT* q) {
#pragma unroll
            for (int k = 0; k < KB; ++k) q[k] = c * KB + k < ce ? p[(c * KB + k) * a.Nx] : (VT)0;
        };
        load(0, v[0]);
        if (NC > 1) load(1, v[1]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KB; ++k) tile[k][cw][cg] = (double)v[c % 2][k];
            __syncthreads();
            if (c + 2 < NC) load(c + 2, v[c % 2]);
#pragma unroll
            for (int k = 0; k < KB; ++k)
                if (c * KB + k < E) use(c * KB + k, tile[k][wave][lane]);
        }
    };
    auto write = [&](void* dst, auto&& get) {
        VT* p = static_cast<VT*>(dst) + c0;
#pragma unroll
        for (int e0 = 0; e0 < E; e0 += KB) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KB; ++k)
                if (e0 + k < E) tile[k][wave][lane] = get(e0 + k);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < KB; ++k)
                if (e0 + k < ce) p[(e0 + k) * a.Nx] = (VT)tile[k][cw][cg];
        }
    };
    // a residual between two batches stays by time lines: whole lanes in
    // order, no transposition (S is a multiple of LA there)
    const int lanes = (int)(a.S / LA);
    if (a.rin_lines) {
        const VT* p = static_cast<const VT*>(a.rin) + mode * E * lanes + min(lane, lanes - 1);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double v = (double)p[e * lanes];
            r[e / NT][e % NT] = lane < lanes ? v : 0.0;
        }
    } else {
        read(a.rin, [&](int e, double v) { r[e / NT][e % NT] = v; });
    }

    // value of the previous lane (0 for the first)
    auto prev = [&](double v) { return wave_dpp<kDppWaveShr1, 0xf>(v); };
    // exact solve of a level over NS slabs per lane, in place: u_s = a_s +
    // x_{s-1} A^{-1} e_1 with a_s = A^{-1} f_s, the scalars x over the lanes by
    // a prefix sum with the constant factor gamma^NS
    auto exact = [&](auto& f, int l) {
        constexpr int NS = sizeof(f) / sizeof(f[0]);
        const uptr inv = mat(l);
        double z[NS][NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < NT; ++k) {
                const double c = inv[t * NT + k];
#pragma unroll
                for (int j = 0; j < NS; ++j) z[j][t] = k ? z[j][t] + c * f[j][k] : c * f[j][k];
            }
        const double gamma = inv[(NT - 1) * NT];
        double y = 0.0, G = 1.0;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            y = z[j][NT - 1] + gamma * y;
            G *= gamma;
        }
        // within rows of 16 lanes, then row 0 into 1 and 2 into 3, then the
        // first half into the second, with the power of the factor between
        double w = G;
        y += G * wave_dpp<kDppRowShr + 1, 0xf>(y);
        w *= lane & 1 ? G : 1.0;
        G *= G;
        y += G * wave_dpp<kDppRowShr + 2, 0xf>(y);
        w *= lane & 2 ? G : 1.0;
        G *= G;
        y += G * wave_dpp<kDppRowShr + 4, 0xf>(y);
        w *= lane & 4 ? G : 1.0;
        G *= G;
        y += G * wave_dpp<kDppRowShr + 8, 0xf>(y);
        w *= lane & 8 ? G : 1.0;
        G *= G;
        y += w * wave_dpp<kDppRowBcast15, 0xa>(y);
        w *= lane & 16 ? G : 1.0;
        y += w * wave_dpp<kDppRowBcast31, 0xc>(y);
        double x = prev(y);
#pragma unroll
        for (int j = 0; j < NS; ++j) {
#pragma unroll
            for (int t = 0; t < NT; ++t) f[j][t] = z[j][t] + x * inv[t * NT];
            x = f[j][NT - 1];
        }
    };
    // fc = restriction of the slab rows g
    auto restrict_to = [&](auto& fc, const auto& g) {
        constexpr int NC = sizeof(fc) / sizeof(fc[0]);
        const uptr P = transfer();
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NT; ++c) {
                    const double p = P[(h * NT + t) * NT + c];
#pragma unroll
                    for (int j = 0; j < NC; ++j)
                        fc[j][c] = h + t ? fc[j][c] + p * g[2 * j + h][t] : p * g[2 * j][0];
                }
    };
    // a coarse level on the way down: f becomes u = omega A^{-1} f, fc the
    // restricted residual (1 - omega) f + e_1 u[last, previous slab]
    auto down = [&](auto& f, auto& fc, int l) {
        constexpr int NS = sizeof(f) / sizeof(f[0]);
        const uptr inv = mat(l), P = transfer();
        double q = 0.0;
#pragma unroll
        for (int k = 0; k < NT; ++k) q += inv[(NT - 1) * NT + k] * f[NS - 1][k];
        q = prev(om * q);
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            double z[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) z[t] = 0.0;
#pragma unroll
            for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int t = 0; t < NT; ++t) z[t] += inv[t * NT + k] * f[j][k];
#pragma unroll
            for (int t = 0; t < NT; ++t) f[j][t] *= 1.0 - om;
            f[j][0] += q;
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NT; ++c)
                    fc[j / 2][c] = (j % 2 || t ? fc[j / 2][c] : 0.0) + P[(j % 2 * NT + t) * NT + c] * f[j][t];
#pragma unroll
            for (int t = 0; t < NT; ++t) f[j][t] = om * z[t];
            q = f[j][NT - 1];
        }
    };
    // ... and up: u <- (2 - omega) u + (1 - omega) P e + omega q A^{-1} e_1 (e is used up)
    auto up = [&](auto& u, auto& e, int l) {
        constexpr int NS = sizeof(u) / sizeof(u[0]);
        const uptr inv = mat(l), P = transfer();
        double v[NS];                           // coupling rows of u + P e
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            v[j] = u[j][NT - 1];
#pragma unroll
            for (int k = 0; k < NT; ++k) v[j] += P[(j % 2 * NT + NT - 1) * NT + k] * e[j / 2][k];
        }
        double q = prev(v[NS - 1]);
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const double s = om * q;
#pragma unroll
            for (int t = 0; t < NT; ++t) u[j][t] = (2.0 - om) * u[j][t] + s * inv[t * NT];
            q = v[j];
        }
#pragma unroll
        for (int j = 0; j < NS / 2; ++j)
#pragma unroll
            for (int t = 0; t < NT; ++t) e[j][t] *= 1.0 - om;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                    const double p = P[(h * NT + t) * NT + k];
#pragma unroll
                    for (int j = 0; j < NS / 2; ++j) u[2 * j + h][t] += p * e[j][k];
                }
    };
    // damped block Jacobi on the finest level's residual
    auto smooth = [&] {
        const uptr inv0 = mat(0);
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < NT; ++k) d += inv0[(NT - 1) * NT + k] * r[LA - 1][k];
        d = prev(om * d);
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            double dn = 0.0;
#pragma unroll
            for (int k = 0; k < NT; ++k) dn += inv0[(NT - 1) * NT + k] * r[i][k];
#pragma unroll
            for (int t = 0; t < NT; ++t) r[i][t] *= 1.0 - om;
            r[i][0] += d;
            d = om * dn;
        }
    };
    // ||r||^2 of the mode after cycle c, and its two weighted forms
    auto sums = [&](int c) {
        if (!a.partial) return;
        double s2 = 0.0;
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            double q = 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) q += r[i][t] * r[i][t];
            s2 += i < nv ? q : 0.0;
        }
        s2 += wave_dpp<kDppRowShr + 1, 0xf>(s2);
        s2 += wave_dpp<kDppRowShr + 2, 0xf>(s2);
        s2 += wave_dpp<kDppRowShr + 4, 0xf>(s2);
        s2 += wave_dpp<kDppRowShr + 8, 0xf>(s2);
        s2 += wave_dpp<kDppRowBcast15, 0xa>(s2);
        s2 += wave_dpp<kDppRowBcast31, 0xc>(s2);          // the total in the last lane
        if (m0 + wave >= a.Nx) s2 = 0.0;
        if (lane == 63) {
            red[wave][c][0] = s2;
            const uptr w = mat(a.L + (ONE ? 1 : 2));
            red[wave][c][1] = w[0] * s2;
            red[wave][c][2] = w[1] * s2;
        }
    };

    sums(0);
    if constexpr (ONE) {
        if (a.steps) {
            // what the steps add to the iterate, omega A^{-1} (r_0 + .. of each
            // step): local to a slab and those that its steps reach, so that
            // infinities and NaN go no further than step by step
            double z[LA][NT];
#pragma unroll
            for (int i = 0; i < LA; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) z[i][t] = r[i][t];
#pragma unroll 1
            for (int i = 1; i < a.steps; ++i) {
                smooth();
#pragma unroll
                for (int j = 0; j < LA; ++j)
#pragma unroll
                    for (int t = 0; t < NT; ++t) z[j][t] += r[j][t];
            }
            const uptr inv0 = mat(0);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                    const double c = om * inv0[t * NT + k];
#pragma unroll
                    for (int i = 0; i < LA; ++i) r[i][t] = k ? r[i][t] + c * z[i][k] : c * z[i][0];
                }
            write(a.uout, [&](int k) { return r[k / NT][k % NT]; });
        }
        if (a.m > 0) {
            double e[LA][NT];
#pragma unroll
            for (int i = 0; i < LA; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) e[i][t] = r[i][t];
            exact(e, 0);
            const uptr ap = mat(1);
            double q = prev(e[LA - 1][NT - 1]);
#pragma unroll
            for (int i = 0; i < LA; ++i) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int k = 0; k < NT; ++k) r[i][t] -= ap[t * NT + k] * e[i][k];
                r[i][0] += q;
                q = e[i][NT - 1];
            }
            sums(1);
            if (a.uout) write(a.uout, [&](int k) { return e[k / NT][k % NT]; });
        }
    } else {
        const int L = a.L;
#pragma unroll 1
        for (int cyc = 0; cyc < a.m; ++cyc) {
            double u1[LA / 2][NT];
            // finest level: pre-smoothing, its residual restricted
            smooth();
            restrict_to(u1, r);
            // levels below: the coarsest one exactly
            if (LA < 4 || L == 2) {
                exact(u1, 1);
            } else if constexpr (LA >= 4) {
                double u2[LA / 4][NT];
                down(u1, u2, 1);
                if (LA < 8 || L == 3) {
                    exact(u2, 2);
                } else if constexpr (LA >= 8) {
                    double u3[LA / 8][NT];
                    down(u2, u3, 2);
                    exact(u3, 3);
                    up(u2, u3, 2);
                }
                up(u1, u2, 1);
            }
            // finest level: the correction, then the post-smoothing step
            {
                const uptr P = transfer();
                auto last = [&](int i) {        // (P e)[last] of slab i
                    double v = 0.0;
#pragma unroll
                    for (int k = 0; k < NT; ++k) v += P[(i % 2 * NT + NT - 1) * NT + k] * u1[i / 2][k];
                    return v;
                };
                double q = prev(last(LA - 1));
#pragma unroll
                for (int i = 0; i < LA; ++i) {
                    r[i][0] += q;
                    q = last(i);
                }
            }
            const uptr ap = mat(L);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int k = 0; k < NT; ++k) {
                        const double c = ap[h * NM + t * NT + k];
#pragma unroll
                        for (int j = 0; j < LA / 2; ++j) r[2 * j + h][t] -= c * u1[j][k];
                    }
            smooth();
            if (sizeof(VT) < sizeof(double)) {
                // FP32 storage: rounded in every cycle, so that the result
                // does not depend on where a batch ends
#pragma unroll
                for (int i = 0; i < LA; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t) r[i][t] = (double)(VT)r[i][t];
            }
            sums(cyc + 1);
        }
    }
    if (a.rout && a.rout_lines) {
        VT* p = static_cast<VT*>(a.rout) + mode * E * lanes + lane;
        if (lane < lanes && m0 + wave < a.Nx)
#pragma unroll
            for (int e = 0; e < E; ++e) p[e * lanes] = (VT)r[e / NT][e % NT];
    } else if (a.rout) {
        write(a.rout, [&](int k) { return r[k / NT][k % NT]; });
    }
    if (a.uout && (!ONE || (a.m == 0 && !a.steps))) {
        // the iterate of this residual: u^ = L^{-1}(f^ - r^)
        read(a.fh, [&](int e, double v) { r[e / NT][e % NT] = v - r[e / NT][e % NT]; });
        exact(r, 0);
        write(a.uout, [&](int k) { return r[k / NT][k % NT]; });
    }
    if (a.partial) {
        __syncthreads();
        if (tid < 3 * (a.m + 1)) {
            double v = 0.0;
            for (int w = 0; w < MB; ++w) v += red[w][tid / 3][tid % 3];
            a.partial[(long)tid * gridDim.x + blockIdx.x] = v;
        }
    }
}

// Slabs per lane: the fewest that hold the line and divide into its levels;
// 16 (N_t <= 3: 96 registers of residual and 84 of coarse levels) at most.
int cycles_lane_slabs(int Nt, int L, long S) {
    if (Nt < 2 || Nt > 6 || L < 1 || L > 4 || S < 1) return 0;
    int LA = 1;
    while (LA < (1 << (L - 1)) || 64L * LA < S) LA *= 2;
    return LA <= (Nt <= 3 ? 16 : 8) ? LA : 0;
}

bool cycles_supported(int Nt, int L, long S) { return cycles_lane_slabs(Nt, L, S) > 0; }

static long cycles_blocks(long Nx) { return ((Nx + MB - 1) / MB + 7) / 8 * 8; }

long cycles_partials(long Nx) { return 3L * (kMaxBatch + 1) * cycles_blocks(Nx); }

size_t cycles_table_len(int Nt, int L, long Nx) { return (size_t)Nx * tab_len(Nt, L) + 2 * Nt * Nt; }

hipError_t launch_cycles_table(int dim, int Nt, int L, const TimeMix* tm, const double* ktmt, const double* mu1, int n,
                               long Nx, const Transfer& tr, const double* vw, double* tab, hipStream_t st) {
    const dim3 grid((unsigned)((Nx * (L + 2) * Nt + 255) / 256));
#define STH_TAB_NT(NTV)                                                                                          \
    case NTV:                                                                                                    \
        hipLaunchKernelGGL((k_mode_table<NTV>), grid, dim3(256), 0, st, dim, n, L, Nx, tm, ktmt, mu1, vw, tr, tab, \
                           tab_len(Nt, L));                                                                      \
        return hipGetLastError();
    switch (Nt) {
        STH_TAB_NT(2) STH_TAB_NT(3) STH_TAB_NT(4) STH_TAB_NT(5) STH_TAB_NT(6)
        default: return hipErrorInvalidValue;
    }
#undef STH_TAB_NT
}

// sum j of the batch by block j (fixed order) to the host
__global__ __launch_bounds__(256) void k_cycle_sums(const double* __restrict__ partial, long count,
                                                    double* out_host, SolveStart start, int nsums) {
    __shared__ double red[4];
    const bool fin = (int)blockIdx.x == nsums;              // the solve's prologue
    const double* p = fin ? start.partial : partial + (long)blockIdx.x * count;
    int nz = 0;
    if (fin) {
        count = kNormBlocks;
        for (int i = threadIdx.x; i < kNormBlocks; i += 256) nz |= p[kNormBlocks + i] != 0.0;
        nz = __syncthreads_or(nz);
    }
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    long i = threadIdx.x;
    for (; i + 768 < count; i += 1024) {
        s0 += p[i];
        s1 += p[i + 256];
        s2 += p[i + 512];
        s3 += p[i + 768];
    }
    for (; i < count; i += 256) s0 += p[i];
    double v = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        v = (red[0] + red[1]) + (red[2] + red[3]);
        if (fin) {
            *start.out = *start.out_host = v;
            start.flags[0] = *start.flag_host = nz ? 1 : 0;
            start.flags[1] = nz ? 0 : 1;
        } else {
            out_host[blockIdx.x] = v;
        }
    }
}

template <int NT, int LA, typename VT>
static hipError_t cycles_go(const CycArgs& a, long* blocks, hipStream_t st) {
    const int len = tab_len(NT, a.L);
    *blocks = cycles_blocks(a.Nx);
    const dim3 grid((unsigned)*blocks), block(64 * MB);
    if constexpr (LA > 1)
        if (a.L > 1 && !a.steps) {
            hipLaunchKernelGGL((k_cycles<NT, LA, VT, false>), grid, block, 0, st, a, len);
            return hipGetLastError();
        }
    if constexpr (sizeof(VT) == 8) {
        hipLaunchKernelGGL((k_cycles<NT, LA, VT, true>), grid, block, 0, st, a, len);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;        // (float vectors: several levels only)
}

template <int NT, typename VT>
static hipError_t cycles_launch(const CycArgs& a, int LA, long* blocks, hipStream_t st) {
#define STH_CYC(LAV) \
    if (LA == LAV) return cycles_go<NT, LAV, VT>(a, blocks, st);
    STH_CYC(1) STH_CYC(2) STH_CYC(4) STH_CYC(8)
    if constexpr (NT <= 3) { STH_CYC(16) }
#undef STH_CYC
    return hipErrorInvalidValue;
}

hipError_t launch_smoothing(int Nt, int L, const double* tab, long Nx, double omega, long S, int steps,
                            const double* r, double* uout, hipStream_t st) {
    const int LA = cycles_lane_slabs(Nt, 1, S);      // (no levels: as many lanes as there are slabs)
    if (!LA || steps < 1 || r == uout) return hipErrorInvalidValue;
    const CycArgs a{L, 0, steps, 0, 0, S, Nx, omega, tab, r, r, nullptr, uout, nullptr};
    long blocks = 0;
    switch (Nt) {
        case 2: return cycles_launch<2, double>(a, LA, &blocks, st);
        case 3: return cycles_launch<3, double>(a, LA, &blocks, st);
        case 4: return cycles_launch<4, double>(a, LA, &blocks, st);
        case 5: return cycles_launch<5, double>(a, LA, &blocks, st);
        case 6: return cycles_launch<6, double>(a, LA, &blocks, st);
        default: return hipErrorInvalidValue;
    }
}

bool cycles_lines(int Nt, int L, long S) {
    const int LA = cycles_lane_slabs(Nt, L, S);
    return LA && L > 1 && S % LA == 0;
}

hipError_t launch_cycles(int Nt, int L, const double* tab, long Nx, double omega, long S, int m,
                         const double* rin, const double* fh, double* rout, double* uout, double* partial,
                         long max_partial, double* out_host, hipStream_t st, int vt, bool rin_lines, bool rout_lines,
                         const SolveStart* start) {
    const int LA = cycles_lane_slabs(Nt, L, S);
    if (!LA || m < 0 || m > kMaxBatch || (L == 1 && m > 1)) return hipErrorInvalidValue;
    if (partial && 3L * (m + 1) * cycles_blocks(Nx) > max_partial) return hipErrorInvalidValue;
    if ((rout && rout == rin) || (uout && (uout == rin || uout == rout || uout == fh))) return hipErrorInvalidValue;
    if ((rin_lines || rout_lines) && !cycles_lines(Nt, L, S)) return hipErrorInvalidValue;
    const CycArgs a{L, m, 0, rin_lines, rout_lines, S, Nx, omega, tab, rin, fh, rout, uout, partial};
    hipError_t e = hipErrorInvalidValue;
    long blocks = 0;
#define STH_CYC_NT(NTV)                                                                            \
    case NTV:                                                                                      \
        e = vt ? cycles_launch<NTV, float>(a, LA, &blocks, st)                                     \
               : cycles_launch<NTV, double>(a, LA, &blocks, st);                                   \
        break;
    switch (Nt) {
        STH_CYC_NT(2) STH_CYC_NT(3) STH_CYC_NT(4) STH_CYC_NT(5) STH_CYC_NT(6)
        default: break;
    }
#undef STH_CYC_NT
    if (e != hipSuccess || !partial) return e;
    hipLaunchKernelGGL(k_cycle_sums, dim3(3 * (m + 1) + (start ? 1 : 0)), dim3(256), 0, st, partial, blocks, out_host,
                       start ? *start : SolveStart{}, 3 * (m + 1));
    return hipGetLastError();
}

}  // namespace sth
