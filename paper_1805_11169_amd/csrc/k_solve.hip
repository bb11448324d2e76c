// Assembly of S and K = W - W1 - W2 (Eqs. 8-9), the Tikhonov-regularised
// Cholesky factorisation of S + eps I, and RK4 for i S dC/dt = K C.
//
// Assembly.  With W = V_1(r) + V_2(R) + W_c(r, R), the one-coordinate parts of
// Eq. 9b cancel against Eqs. 9c-9d except at the ket's own trajectory:
//     K[b][a] = Wc[b][a] - E1[b][a] S2[b][a] - S1[b][a] E2[b][a]
//               - (V_1(r^a) + V_2(R^a)) S[b][a],     S = S1 o S2,
// where Wc, E1, E2 are the Eq. 9b-9d integrals with W_c alone (with a bilinear
// W_c, from the matrices of r and R).  Per step the
// kernel forms S_k+1, K^- = K(psi_k+1, x_k) (end of the step just taken),
// K_k+1 = K(psi_k+1, x_k+1) (start of the next), the midpoint averages, and
// the regularised matrices handed to the factorisation.
//
// Cholesky (lower, in place, two matrices per launch): right-looking with
// 64-wide panels.  k_chol_panel factors the diagonal block (every work-group
// for itself), inverts it and solves for the rows below.
// k_chol_update subtracts L21 L21^H from the trailing lower triangle on FP64
// matrix cores.  A pivot that is not positive raises the solve flag.
//
// RK4 (classical, S and K linear in time between the step ends, so the
// midpoint is their average).  Each stage is two launches over the 64-row
// blocks of the factor.  k_rk_fwd: a work-group takes its rows of K v, solves
// L y = K v for its block after the blocks above it are done (it subtracts
// their contributions as they arrive), then applies the inverse of its
// diagonal block (from k_chol_panel).
// k_rk_bwd: the same for L^H x = y from the bottom up, then the stage update
// k = -i x of its rows.  Work-groups take blocks in ticket order, so a
// work-group only ever waits on work-groups that are already running, and
// every wait is bounded.
#include "icwf_plan.hpp"

namespace icwf {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ inline dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------ assembly
__global__ void k_assemble(const double2 *__restrict__ S1, const double2 *__restrict__ S2,
                           const double2 *__restrict__ E1a, const double2 *__restrict__ E1b,
                           const double2 *__restrict__ E2a, const double2 *__restrict__ E2b,
                           double2 *__restrict__ Wc, int bilinear, const double2 *__restrict__ Scur,
                           const double2 *__restrict__ Kcur, const double *__restrict__ r,
                           const double *__restrict__ R, const double *__restrict__ r_new,
                           const double *__restrict__ R_new, ModelParams mp, int N, int Np, double eps,
                           int part, double2 *__restrict__ Snext, double2 *__restrict__ Kminus,
                           double2 *__restrict__ Knext, double2 *__restrict__ Amid, double2 *__restrict__ Anext,
                           double2 *__restrict__ Kmid, const int32_t *__restrict__ flags, const long long *__restrict__ zoff, const ModelParams *__restrict__ mpd) {
    const long long zo_ = batch_offset(zoff);
    S1 = zshift(S1, zo_);
    S2 = zshift(S2, zo_);
    E1a = zshift(E1a, zo_);
    E1b = zshift(E1b, zo_);
    E2a = zshift(E2a, zo_);
    E2b = zshift(E2b, zo_);
    Wc = zshift(Wc, zo_);
    Scur = zshift(Scur, zo_);
    Kcur = zshift(Kcur, zo_);
    r = zshift(r, zo_);
    R = zshift(R, zo_);
    r_new = zshift(r_new, zo_);
    R_new = zshift(R_new, zo_);
    Snext = zshift(Snext, zo_);
    Kminus = zshift(Kminus, zo_);
    Knext = zshift(Knext, zo_);
    Amid = zshift(Amid, zo_);
    Anext = zshift(Anext, zo_);
    Kmid = zshift(Kmid, zo_);
    flags = zshift(flags, zo_);
    if (zoff) mp = *zshift(mpd, zo_);

    if (flags[kFlagHalt]) return;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)Np * Np) return;
    const int b = (int)(idx / Np), a = (int)(idx - (size_t)b * Np);
    const double2 s1 = S1[idx], s2 = S2[idx];
    const double2 S = cmul(s1, s2);
    const double reg = (a == b) ? eps : 0.0;
    if (part & kAssembleS) {
        Snext[idx] = S;
        Anext[idx] = make_double2(S.x + reg, S.y);
        if (part == kAssembleS) {
            const double2 sc = Scur[idx];
            Amid[idx] = make_double2(0.5 * (sc.x + S.x) + reg, 0.5 * (sc.y + S.y));
        }
    }
    if (!(part & kAssembleK)) return;
    double2 w, e1, e2;
    if (bilinear) {
        // W_c = lam r R: e1, e2 = <b|r|a>, <b|R|a>; the matrices of Eqs. 9b-9d
        // are lam times their product and lam R^a e1, lam r^a e2
        e1 = E1a[idx];
        e2 = E2a[idx];
        w = cscale(cmul(e1, e2), mp.p[3]);
        if (part != kAssembleKnext) Wc[idx] = w;
    } else {
        w = (b <= a) ? Wc[idx] : cconj(Wc[(size_t)a * Np + b]);
    }
    auto coupling = [&](const double2 *e1_at, const double2 *e2_at, double ra, double Ra, double c) {
        const double2 x1 = bilinear ? cscale(e1, mp.p[3] * Ra) : e1_at[idx];
        const double2 x2 = bilinear ? cscale(e2, mp.p[3] * ra) : e2_at[idx];
        return csub(csub(csub(w, cmul(x1, s2)), cmul(s1, x2)), cscale(S, c));
    };
    double ca = 0.0, cn = 0.0;
    if (a < N) {
        ca = model_v1(mp, r[a]) + model_v2(mp, R[a]);
        cn = model_v1(mp, r_new[a]) + model_v2(mp, R_new[a]);
    }
    if (part != kAssembleKnext) {
        const double2 km = coupling(E1a, E2a, r[a], R[a], ca);
        if (part == kAssembleInitial) {
            // start of the run: K_0 = K(psi_0, x_0) -> the slot of parity 0
            Knext[idx] = km;
            return;
        }
        Kminus[idx] = km;
        const double2 kc = Kcur[idx];
        Kmid[idx] = make_double2(0.5 * (kc.x + km.x), 0.5 * (kc.y + km.y));
    }
    if (part != kAssembleKminus) Knext[idx] = coupling(E1b, E2b, r_new[a], R_new[a], cn);
}

// ------------------------------------------------------------------ Cholesky
constexpr int NB = kCholNb;   // 64

__device__ inline void raise_solve(int32_t *flags) {
    atomicOr(&flags[kFlagSolve], 1);
    atomicOr(&flags[kFlagHalt], 1);
}

// Broadcast lane `src` (wave-uniform) of a double to the whole wave.
__device__ inline double bcast(double v, int src) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), src);
    return __hiloint2double(hi, lo);
}

// The panel at column kb: the 64 x 64 diagonal block L11 L11^H = A11, its
// inverse, and the rows below, L21 = A21 L11^-H.  One work-group of four waves
// per 64 rows below, and one more for the diagonal block's own results; each
// factors the diagonal block itself, so the panel needs no communication
// between work-groups.
//
// The block is held in LDS as 16 x 16 tiles.  A block column of 16 is
// eliminated by one wave without a barrier, lane = row (the 16 pivot rows and
// up to 48 below them), its 16 columns in registers: the pivot and the pivot
// rows' entries come by readlane, so a column costs a short chain (readlane,
// reciprocal root, scaling) and the update of the columns after it.  The other
// waves then update the tiles to the right on matrix cores, one wave inverting
// the 16 x 16 triangle meanwhile.  The rows below are solved transposed,
// L11 Z = A21^H, 16 rows per wave: the accumulator layout of a matrix product
// is the layout of its right operand, so Z_J = L_JJ^-1 (A_J^H - sum_I L_JI Z_I)
// runs from register to register.  Products are summed by themselves and then
// subtracted: accumulated onto the entry, each product rounded it twice (re
// and im of the factors), and the solves' error was a quarter larger (N = 250,
// mean of 8 ensembles against long double, relative to LAPACK's: 1.76, 1.37
// so).  What bounds it is the chain of 64 columns
// (a panel 30-36 us alone, 65-71 us on a compute unit that also runs the
// contraction, whose matrix products hold the FP64 pipe 64 cycles at a time):
// two matrices at N = 64, all kernels of the factorisation, 105 -> 37 us
// against one barrier and one LDS round trip per column, with the inverses and
// the last copy in kernels of their own; N = 500, 658 -> 326 us; N = 1024
// beside the contraction, 1.68 -> 1.42 ms.
constexpr int kTiles = 10;       // 16 x 16 tiles (I, K), K <= I, of the block
typedef double2 Tile[16][17];
__device__ constexpr int tile_of(int I, int K) { return I * (I + 1) / 2 + K; }

struct PanelShared {
    Tile L[kTiles];              // the block's lower tiles
    Tile inv[4];                 // inverses of its diagonal tiles
    Tile x[4];                   // off-diagonal tiles of the block's inverse
    double dinv[NB];
};

// acc += X Y^H for 16 x 16 tiles in LDS
__device__ __forceinline__ void tile_mul_h(dbl4 &re, dbl4 &im, const Tile &X, const Tile &Y) {
    const int lane = threadIdx.x & 63, row = lane & 15, quarter = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double2 x = X[row][4 * q + quarter], y = Y[row][4 * q + quarter];
        re = mfma(x.x, y.x, re);
        re = mfma(x.y, y.y, re);
        im = mfma(x.y, y.x, im);
        im = mfma(-x.x, y.y, im);
    }
}
// acc += s X Z, Z in accumulator layout
__device__ __forceinline__ void tile_mul(dbl4 &re, dbl4 &im, const Tile &X, dbl4 zre, dbl4 zim, double s) {
    const int lane = threadIdx.x & 63, row = lane & 15, quarter = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double2 x = cscale(X[row][4 * q + quarter], s);
        re = mfma(x.x, zre[q], re);
        re = mfma(-x.y, zim[q], re);
        im = mfma(x.x, zim[q], im);
        im = mfma(x.y, zre[q], im);
    }
}
// a tile in accumulator layout
__device__ __forceinline__ void tile_load(dbl4 &re, dbl4 &im, const Tile &X) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double2 x = X[mfma_row_f64(lane, v)][lane & 15];
        re[v] = x.x;
        im[v] = x.y;
    }
}
__device__ __forceinline__ void tile_store(Tile &X, dbl4 re, dbl4 im) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < 4; ++v) X[mfma_row_f64(lane, v)][lane & 15] = make_double2(re[v], im[v]);
}

// Columns 16 J .. 16 J + 15 of the block, by one wave; false if a pivot is not
// positive.
__device__ __forceinline__ bool eliminate_block(PanelShared &sh, int J) {
    const int lane = threadIdx.x & 63, r = lane & 15, I = J + (lane >> 4);
    const bool mine = I < 4;
    Tile &T = sh.L[tile_of(mine ? I : J, J)];
    double2 a[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) a[c] = T[r][c];
    bool ok = true;
    double diag = 0.0;                               // L_rr
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        double piv = bcast(a[j].x, j);
        ok = ok && piv > 0.0;
        piv = piv > 0.0 ? piv : 1.0;
        // 1/sqrt(piv) from the hardware estimate and two Newton steps
        // y <- y (3 - piv y^2) / 2 (each squares the relative error)
        double dinv = __builtin_amdgcn_rsq(piv);
        dinv = dinv * fma(-0.5 * piv * dinv, dinv, 1.5);
        dinv = dinv * fma(-0.5 * piv * dinv, dinv, 1.5);
        // the updates take a_rj conj(a_cj) / piv, so that they do not wait for
        // (nor carry the rounding of) the scaled column
        const double2 u = cscale(a[j], dinv * dinv);
#pragma unroll
        for (int c = j + 1; c < 16; ++c) {
            const double lx = bcast(a[j].x, c), ly = bcast(a[j].y, c);
            a[c].x = fma(-u.y, ly, fma(-u.x, lx, a[c].x));
            a[c].y = fma(u.x, ly, fma(-u.y, lx, a[c].y));
        }
        // L_jj = piv y, and the reciprocal of that very number, which the
        // inverses use as well
        const double d = piv * dinv;
        dinv = fma(dinv, fma(-d, dinv, 1.0), dinv);
        a[j] = cscale(a[j], dinv);
        sh.dinv[16 * J + j] = dinv;
        diag = r == j ? d : diag;
    }
    // the diagonal tile: zero above the diagonal, the diagonal real
    const int top = I == J ? r : 16;
    if (mine)
#pragma unroll
        for (int c = 0; c < 16; ++c)
            T[r][c] = make_double2(c > top ? 0.0 : c == top ? diag : a[c].x, c >= top ? 0.0 : a[c].y);
    return ok;
}

// Inverse of the diagonal tile J by one wave, lane = row: with
// y_r = e_r - sum_{k<r} L_rk x_k, row r of the inverse is x_r = y_r / L_rr; step
// j takes row j's y by readlane and subtracts L_rj x_j from the rows below it.
__device__ __forceinline__ void invert_tile(PanelShared &sh, int J) {
    const int lane = threadIdx.x & 63, r = lane & 15;
    const Tile &T = sh.L[tile_of(J, J)];
    double2 y[16], l[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        const double2 x = T[r][c];                   // zero above the diagonal
        l[c] = make_double2(c == r ? 0.0 : x.x, x.y);
        y[c] = make_double2(c == r ? 1.0 : 0.0, 0.0);
    }
#pragma unroll
    for (int j = 0; j < 15; ++j) {
        const double d = sh.dinv[16 * J + j];
#pragma unroll
        for (int c = 0; c <= j; ++c) {
            const double px = bcast(y[c].x, j) * d, py = bcast(y[c].y, j) * d;
            y[c].x = fma(l[j].y, py, fma(-l[j].x, px, y[c].x));
            y[c].y = fma(-l[j].y, px, fma(-l[j].x, py, y[c].y));
        }
    }
    const double d = sh.dinv[16 * J + r];
    if (lane < 16)
#pragma unroll
        for (int c = 0; c < 16; ++c) sh.inv[J][r][c] = cscale(y[c], d);
}

__global__ void __launch_bounds__(256, 2) k_chol_panel(double2 *A0, double2 *A1, int Np, int kb,
                                                       double2 *__restrict__ diag, double2 *__restrict__ X0,
                                                       double2 *__restrict__ X1, double2 *__restrict__ F0,
                                                       double2 *__restrict__ F1, int32_t *__restrict__ flags,
                                                       const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    A0 = zshift(A0, zo_);
    A1 = zshift(A1, zo_);
    diag = zshift(diag, zo_);
    X0 = zshift(X0, zo_);
    X1 = zshift(X1, zo_);
    F0 = zshift(F0, zo_);
    F1 = zshift(F1, zo_);
    flags = zshift(flags, zo_);

    if (flags[kFlagHalt]) return;
    // the panel is a latency chain that shares compute units with the
    // contraction on the other stream: its waves take the issue slots first
    __builtin_amdgcn_s_setprio(3);
    __shared__ PanelShared sh;
    double2 *A = blockIdx.y ? A1 : A0;
    const int t = threadIdx.x, lane = t & 63, row = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool own = blockIdx.x == gridDim.x - 1;    // this work-group keeps the diagonal block's results
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int K = 0; K <= I; ++K)
            sh.L[tile_of(I, K)][t >> 4][t & 15] = A[(size_t)(kb + 16 * I + (t >> 4)) * Np + kb + 16 * K + (t & 15)];
    // the rows below, conjugate transposed, in accumulator layout: this lane
    // has the row `row` of its wave's 16 and the columns 16 J + quarter + 4 v
    double2 *arow = A + (size_t)(kb + NB + 64 * blockIdx.x + 16 * wave + row) * Np + kb + quarter;
    dbl4 zre[4], zim[4];
    auto load_rows = [&]() __attribute__((always_inline)) {
        if (own) return;
#pragma unroll
        for (int J = 0; J < 4; ++J)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double2 x = arow[16 * J + 4 * v];
                zre[J][v] = x.x;
                zim[J][v] = -x.y;
            }
    };
    __syncthreads();
    auto eliminate = [&](int J) {
        if (!eliminate_block(sh, J) && own && lane == 0) raise_solve(flags);
    };
    for (int J = 0; J < 3; ++J) {
        if (wave == 0) eliminate(J);
        if (wave == 1 && J > 0) invert_tile(sh, J - 1);
        __syncthreads();
        // tiles (I, K), J < K <= I, over the waves
        int n = 0;
        for (int K = J + 1; K < 4; ++K)
            for (int I = K; I < 4; ++I, ++n) {
                if ((n & 3) != wave) continue;
                dbl4 re, im, pre = {0, 0, 0, 0}, pim = {0, 0, 0, 0};
                tile_load(re, im, sh.L[tile_of(I, K)]);
                tile_mul_h(pre, pim, sh.L[tile_of(I, J)], sh.L[tile_of(K, J)]);
                tile_store(sh.L[tile_of(I, K)], re - pre, im - pim);
            }
        __syncthreads();
    }
    if (wave == 0) eliminate(3);
    if (wave == 1) invert_tile(sh, 2);
    if (wave > 1) load_rows();                       // in flight over the last block column
    __syncthreads();
    if (wave == 1) invert_tile(sh, 3);
    if (wave < 2) load_rows();
    __syncthreads();
    if (!own) {
#pragma unroll
        for (int J = 0; J < 4; ++J) {
            dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0}, sre = {0, 0, 0, 0}, sim = {0, 0, 0, 0};
#pragma unroll
            for (int I = 0; I < J; ++I) tile_mul(sre, sim, sh.L[tile_of(J, I)], zre[I], zim[I], 1.0);
            tile_mul(re, im, sh.inv[J], zre[J] - sre, zim[J] - sim, 1.0);
            zre[J] = re;
            zim[J] = im;
#pragma unroll
            for (int v = 0; v < 4; ++v) arow[16 * J + 4 * v] = make_double2(re[v], -im[v]);
        }
        return;
    }
    // the diagonal block's results.  The factored block goes to a scratch
    // tile while other work-groups of the launch may still be reading the
    // unfactored one; this work-group of the next launch copies it into place.
    double2 *D = diag + (size_t)blockIdx.y * NB * NB;
    const bool last = kb + NB == Np;
    if (kb > 0) {
        const int pb = kb - NB;
        for (int e = t; e < NB * NB; e += 256) {
            const int rr = e / NB, cc = e % NB;
            if (cc <= rr) A[(size_t)(pb + rr) * Np + pb + cc] = D[e];
        }
        __syncthreads();                             // D is read before it is written again
    }
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int K = 0; K <= I; ++K) {
            const int rr = 16 * I + (t >> 4), cc = 16 * K + (t & 15);
            const double2 x = sh.L[tile_of(I, K)][t >> 4][t & 15];
            if (last) {
                if (cc <= rr) A[(size_t)(kb + rr) * Np + kb + cc] = x;
            } else {
                D[rr * NB + cc] = x;
            }
        }
    __syncthreads();
    // its inverse, by distance from the diagonal:
    // X_IK = -X_II sum_{K<=M<I} L_IM X_MK
    auto product = [&](int I, int K, auto tile, Tile &out) {
        dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0}, ore = {0, 0, 0, 0}, oim = {0, 0, 0, 0};
        for (int M = K; M < I; ++M) {
            dbl4 xr, xi;
            tile_load(xr, xi, tile(M, K));
            tile_mul(re, im, sh.L[tile_of(I, M)], xr, xi, 1.0);
        }
        tile_mul(ore, oim, sh.inv[I], re, im, -1.0);
        tile_store(out, ore, oim);
    };
    auto inverse = [&](int M, int K) -> Tile & {
        if (M == K) return sh.inv[M];
        if (M == K + 1) return sh.x[K];
        return M == 2 ? sh.L[tile_of(2, 0)] : M - K == 2 ? sh.x[3] : sh.L[tile_of(3, 0)];
    };
    if (wave < 3) product(wave + 1, wave, inverse, sh.x[wave]);
    __syncthreads();
    if (wave == 0) product(2, 0, inverse, sh.L[tile_of(2, 0)]);
    if (wave == 1) product(3, 1, inverse, sh.x[3]);
    __syncthreads();
    if (wave == 0) product(3, 0, inverse, sh.L[tile_of(3, 0)]);
    __syncthreads();
    double2 *X = blockIdx.y ? X1 : X0;
    double2 *F = blockIdx.y ? F1 : F0;               // the same block in a full Np x Np inverse, or null
#pragma unroll
    for (int I = 0; I < 4; ++I)
#pragma unroll
        for (int K = 0; K < 4; ++K) {
            const int rr = 16 * I + (t >> 4), cc = 16 * K + (t & 15);
            const double2 x = K <= I ? inverse(I, K)[t >> 4][t & 15] : make_double2(0.0, 0.0);
            X[(size_t)(kb + rr) * NB + cc] = x;
            if (F) F[(size_t)(kb + rr) * Np + kb + cc] = x;
        }
}

// Trailing update A[i][k] -= sum_j L[i][j] conj(L[k][j]) over the lower
// triangle i >= k of rows/cols kb+NB .. Np-1, j over the panel; one
// work-group per 32 x 32 tile, wave w on its 16 x 16 fragment (w / 2, w % 2),
// so a tile's 64-deep reduction runs on four matrix-core streams at once.  A
// lane takes two neighbouring columns j of its row per load pair (whole
// 128-byte lines over its row's four lanes), all of them requested before the
// first product: the launch is a few microseconds of latency and its products
// (N = 1024: 40 -> 12 us beside the contraction, against 16-byte accesses 256
// bytes apart, one product ahead).
__global__ void __launch_bounds__(256, 2) k_chol_update(double2 *A0, double2 *A1, int Np, int kb,
                                                        const int32_t *__restrict__ flags,
                                                        const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    A0 = zshift(A0, zo_);
    A1 = zshift(A1, zo_);
    flags = zshift(flags, zo_);

    if (flags[kFlagHalt]) return;
    double2 *A = blockIdx.y ? A1 : A0;
    const int t = blockIdx.x;
    int ti = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    while (ti * (ti + 1) / 2 > t) --ti;
    const int tk = t - ti * (ti + 1) / 2;
    const int base = kb + NB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int f = wave >> 1, g = wave & 1;
    const int i0 = base + 32 * ti + 16 * f, k0 = base + 32 * tk + 16 * g;
    const int row = lane & 15, quarter = lane >> 4;
    const double2 *xp = A + (size_t)(i0 + row) * Np + kb + 2 * quarter;
    const double2 *yp = A + (size_t)(k0 + row) * Np + kb + 2 * quarter;
    double2 x[NB / 4], y[NB / 4], o[4];
#pragma unroll
    for (int s = 0; s < NB / 8; ++s)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            x[2 * s + e] = xp[8 * s + e];
            y[2 * s + e] = yp[8 * s + e];
        }
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = A[(size_t)(i0 + mfma_row_f64(lane, v)) * Np + k0 + row];
    dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < NB / 4; ++s) {
        // x conj(y) = (xr yr + xi yi) + i (xi yr - xr yi)
        re = mfma(x[s].x, y[s].x, re);
        im = mfma(x[s].y, y[s].x, im);
        re = mfma(x[s].y, y[s].y, re);
        im = mfma(-x[s].x, y[s].y, im);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
        A[(size_t)(i0 + mfma_row_f64(lane, v)) * Np + k0 + row] = make_double2(o[v].x - re[v], o[v].y - im[v]);
}

// ------------------------------------------------------------------ explicit inverse of L
// Batched complex GEMM on 64 x 64 output tiles, O = alpha A B; 4 waves per
// tile, each on a 32 x 32 quarter as 2 x 2 MFMA fragments (rows i, columns j,
// reduction k), 16-wide k chunks of A and B staged through double-buffered
// LDS.  Batch entry z: factor f = z / npairs, pair p = z % npairs, operands
// at base[f] + p stride.
struct GemmBatch {
    const double2 *A[2], *B[2];
    double2 *O[2];
    long long stride;      // element offset between consecutive pairs (A, B and O alike)
    int lda, ldb, ldo;
    int M, N, K;           // output rows and columns, reduction length (multiples of 64)
    int npairs;
    double alpha;
    int lower_a, lower_b;  // A / B lower triangular: the reduction skips the chunks that are zero
};

constexpr int kGT = 64, kGKC = 16, kGLD = kGKC + 1;

__global__ void __launch_bounds__(256, 2) k_cgemm(GemmBatch g, const int32_t *__restrict__ flags) {
    if (flags[kFlagHalt]) return;
    __shared__ double2 sA[2][kGT][kGLD];   // [i][k] of A
    __shared__ double2 sB[2][kGT][kGLD];   // [j][k] of B
    const int z = blockIdx.z, f = z / g.npairs, p = z - f * g.npairs;
    const size_t off = (size_t)p * g.stride;
    const double2 *__restrict__ A = (f ? g.A[1] : g.A[0]) + off;
    const double2 *__restrict__ B = (f ? g.B[1] : g.B[0]) + off;
    double2 *__restrict__ O = (f ? g.O[1] : g.O[0]) + off;
    const int nt = g.N / kGT;
    const int ti = blockIdx.x / nt, tj = blockIdx.x - ti * nt;
    const int i0 = ti * kGT, j0 = tj * kGT;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int row = lane & 15, quarter = lane >> 4;
    const int wi = 32 * (wave >> 1), wj = 32 * (wave & 1);
    dbl4 re[2][2], im[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            re[a][c] = dbl4{0, 0, 0, 0};
            im[a][c] = dbl4{0, 0, 0, 0};
        }
    // B lower triangular: B[k][j] = 0 for k < j, so the tile's columns
    // j >= j0 need k >= j0; A lower triangular: rows i < i0 + 64 need
    // k < i0 + 64.  Only exact zeros are skipped.
    const int kbeg = g.lower_b ? j0 : 0;
    const int kend = g.lower_a ? min(g.K, i0 + kGT) : g.K;
    const int nch = kend > kbeg ? (kend - kbeg) / kGKC : 0;
    // staging: element e = t + 256 m (m < 4); A as [i][k] (64 x 16), B as
    // [k][j] (16 x 64); held as plain doubles (an array of double2 would be
    // placed in scratch memory)
    double rax[4], ray[4], rbx[4], rby[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int e = t + 256 * m;
            const double2 va = A[(size_t)(i0 + (e >> 4)) * g.lda + k0 + (e & 15)];
            const double2 vb = B[(size_t)(k0 + (e >> 6)) * g.ldb + j0 + (e & 63)];
            rax[m] = va.x;
            ray[m] = va.y;
            rbx[m] = vb.x;
            rby[m] = vb.y;
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int e = t + 256 * m;
            sA[buf][e >> 4][e & 15] = make_double2(rax[m], ray[m]);
            sB[buf][e & 63][e >> 6] = make_double2(rbx[m], rby[m]);
        }
    };
    if (nch > 0) {
        fetch(kbeg);
        stash(0);
    }
    __syncthreads();
    for (int ch = 0; ch < nch; ++ch) {
        const int buf = ch & 1;
        const bool more = ch + 1 < nch;
        if (more) fetch(kbeg + (ch + 1) * kGKC);
#pragma unroll
        for (int s4 = 0; s4 < kGKC / 4; ++s4) {
            const int kk = 4 * s4 + quarter;
            double2 xv[2], yv[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                xv[a] = sA[buf][wi + 16 * a + row][kk];
                yv[a] = sB[buf][wj + 16 * a + row][kk];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    // x y = (xr yr - xi yi) + i (xr yi + xi yr)
                    re[a][c] = mfma(xv[a].x, yv[c].x, re[a][c]);
                    re[a][c] = mfma(-xv[a].y, yv[c].y, re[a][c]);
                    im[a][c] = mfma(xv[a].x, yv[c].y, im[a][c]);
                    im[a][c] = mfma(xv[a].y, yv[c].x, im[a][c]);
                }
        }
        if (more) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + wi + 16 * a + mfma_row_f64(lane, v);
                const int j = j0 + wj + 16 * c + row;
                const double2 o = make_double2(g.alpha * re[a][c][v], g.alpha * im[a][c][v]);
                O[(size_t)i * g.ldo + j] = o;
            }
}

// ------------------------------------------------------------------ RK4 stage solves
// Blocks hand their part of y (forward) and x (backward) on through memory
// itself: every entry holds kPending until its block writes it, and whoever
// needs it reads it until it holds something else, so a hand-off is one store
// and one load (with a flag beside the data: a store, a fence, a flag, and a
// load of each; the step's four stages, N = 250: 172 -> 99 us, N = 500: 326 ->
// 183 us, N = 1500: 1.09 -> 0.60 ms, K v taken into the forward kernel).  k_rk_bwd puts kPending back into the y it has read,
// k_rk_fwd into the x of the stage before; the words start so at create.
// solve_sync: the two tickets, each kernel clearing the other's.
constexpr unsigned long long kPending = 0x7ff8dead00c0ffeeull;   // a NaN no arithmetic produces
constexpr int kSyncTicketF = 0, kSyncTicketB = 1;

// The work-group's ticket, and whether it finds the simulation halted (slot[2]
// in LDS: every wave of it goes the same way).
__device__ inline int take_ticket(int32_t *ctr, const int32_t *flags, int (&slot)[2], bool *halt) {
    if (threadIdx.x == 0) {
        const bool h = halted(flags);                // (both on their way together)
        slot[0] = atomicAdd(ctr, 1);
        slot[1] = h;
    }
    __syncthreads();
    *halt = slot[1] != 0;
    return slot[0];
}

__device__ inline unsigned long long peek(const double *p) {
    return __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void post(double *p, unsigned long long v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void post(double2 *p, double2 v) {
    post(&p->x, (unsigned long long)__double_as_longlong(v.x));
    post(&p->y, (unsigned long long)__double_as_longlong(v.y));
}
__device__ inline void post_pending(double2 *p) {
    post(&p->x, kPending);
    post(&p->y, kPending);
}
// The value at p once it is there (`seen`: what a first look gave).  Bounded:
// after ~2^20 looks it raises the flags and returns 0.
__device__ inline double await(const double *p, unsigned long long seen, int32_t *status) {
    for (int it = 0; seen == kPending && it < (1 << 20); ++it) {
        __builtin_amdgcn_s_sleep(1);
        seen = peek(p);
    }
    if (seen == kPending) {
        atomicOr(&status[kFlagHang], 1);
        atomicOr(&status[kFlagHalt], 1);
        return 0.0;
    }
    return __longlong_as_double((long long)seen);
}

// Parts of a matrix a matrix-vector product reads: all of it, the lower
// triangle with the diagonal, or the upper triangle with the diagonal.
enum MatPart : int { kPartAll = 0, kPartLower = 1, kPartUpper = 2 };

// Row-times-vector sums of the stage solves: one row per 256-thread
// work-group, wave w taking the 64-column chunks w, w + 4, ... (so that a
// triangular part spreads evenly), the four wave sums added in wave order
// (a fixed summation order).  Every thread returns the row's sum.
template <typename Term>
__device__ inline double2 row_sum_wg(int rowi, int Np, int part, Term term) {
    __shared__ double2 wsum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lo = part == kPartUpper ? (rowi & ~63) : 0, hi = part == kPartLower ? rowi + 1 : Np;
    double2 acc = make_double2(0, 0);
    for (int c = lo + 64 * wave + lane; c < hi; c += 256)
        if (part != kPartUpper || c >= rowi) acc = cadd(acc, term(c));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        acc.x += __shfl_xor(acc.x, off);
        acc.y += __shfl_xor(acc.y, off);
    }
    if (lane == 0) wsum[wave] = acc;
    __syncthreads();
    return cadd(cadd(wsum[0], wsum[1]), cadd(wsum[2], wsum[3]));
}

// y = M v over the part of M (one row per work-group)
__global__ void __launch_bounds__(256) k_matvec(const double2 *__restrict__ M, const double2 *__restrict__ v,
                                                double2 *__restrict__ y, int Np, int part,
                                                const int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    M = zshift(M, zo_);
    v = zshift(v, zo_);
    y = zshift(y, zo_);
    flags = zshift(flags, zo_);

    if (flags[kFlagHalt]) return;
    const int rowi = blockIdx.x;
    const double2 *m = M + (size_t)rowi * Np;
    const double2 acc = row_sum_wg(rowi, Np, part, [&](int c) { return cmul(m[c], v[c]); });
    if (threadIdx.x == 0) y[rowi] = acc;
}

// Forward stage kernel: y_B = L_BB^-1 (rhs_B - sum_{C<B} L_BC y_C), with
// L_BB^-1 from k_chol_panel and rhs = K v (K == nullptr: rhs as given).  256
// threads; thread t: row i = t / 4 of the block, columns 4 c + q, q = t % 4.
// Everything that does not depend on the blocks above (rhs_B, the block's
// slices of L and of L_BB^-1) is loaded before the waits.
//
// Eq. 8 amplifies the rounding of K v by up to 1 / (2 sqrt(eps)), so its sum
// is a shallow one: a thread adds each 16 of its terms as a tree, the trees to
// four running sums in turn, and these and the row's four threads pairwise (at
// Np = 1536 a chain of 6 and 8 levels above it, as a 256-lane sum has; one
// chain of 384 terms a thread left 2.1 to 4.2 times its error at N = 400 to
// 1984, rms against long double).
__global__ void __launch_bounds__(256) k_rk_fwd(const double2 *__restrict__ K, const double2 *__restrict__ v,
                                                const double2 *__restrict__ rhs, const double2 *__restrict__ L,
                                                const double2 *__restrict__ Linv, double2 *__restrict__ ybuf,
                                                double2 *__restrict__ xbuf, int Np, int32_t *__restrict__ sync,
                                                int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    K = zshift(K, zo_);
    v = zshift(v, zo_);
    rhs = zshift(rhs, zo_);
    L = zshift(L, zo_);
    Linv = zshift(Linv, zo_);
    ybuf = zshift(ybuf, zo_);
    xbuf = zshift(xbuf, zo_);
    sync = zshift(sync, zo_);
    flags = zshift(flags, zo_);

    __shared__ double2 yc[2][NB], uvec[NB], vc[4 * NB];
    __shared__ int slot[2];
    bool halt;
    const int B = take_ticket(&sync[kSyncTicketF], flags, slot, &halt);
    if (B == 0 && threadIdx.x == 0) sync[kSyncTicketB] = 0;
    const int t = threadIdx.x, i = t >> 2, q = t & 3;
    const int r0 = B * NB;
    if (t < NB) post_pending(&xbuf[r0 + t]);
    if (halt) {                                      // nobody waits for ever
        if (t < NB) post(&ybuf[r0 + t], make_double2(0, 0));
        return;
    }
    // row i of K v, 128 columns of K in flight at a time and v through LDS
    double2 kv[4] = {};
    if (K) {
        const double2 *krow = K + (size_t)(r0 + i) * Np + q;
        for (int g = 0; g < Np; g += 4 * NB) {
            if (g > 0) __syncthreads();              // the previous columns' v is read
            vc[t] = g + t < Np ? v[g + t] : make_double2(0, 0);
            double2 x[2][16];
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (g + (h + u) * NB < Np)
#pragma unroll
                        for (int c = 0; c < 16; ++c) x[u][c] = krow[g + (h + u) * NB + 4 * c];
                if (h == 0) __syncthreads();
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (g + (h + u) * NB >= Np) break;
#pragma unroll
                    for (int c = 0; c < 16; ++c) x[u][c] = cmul(x[u][c], vc[(h + u) * NB + 4 * c + q]);
#pragma unroll
                    for (int w = 8; w > 0; w >>= 1)
#pragma unroll
                        for (int c = 0; c < w; ++c) x[u][c] = cadd(x[u][c], x[u][c + w]);
                    kv[h + u] = cadd(kv[h + u], x[u][0]);
                }
            }
        }
        kv[0] = cadd(cadd(kv[0], kv[1]), cadd(kv[2], kv[3]));
        kv[0].x += __shfl_xor(kv[0].x, 1);
        kv[0].y += __shfl_xor(kv[0].y, 1);
        kv[0].x += __shfl_xor(kv[0].x, 2);
        kv[0].y += __shfl_xor(kv[0].y, 2);
    }
    double2 iv[16];   // row i of L_BB^-1
#pragma unroll
    for (int c = 0; c < 16; ++c) iv[c] = Linv[(size_t)(r0 + i) * NB + 4 * c + q];
    double2 part = make_double2(0, 0);
    // contributions of the blocks above, as they complete: the words of block
    // C are awaited by the first 128 threads
    const double *words = reinterpret_cast<const double *>(ybuf);
    unsigned long long seen = t < 2 * NB && B > 0 ? peek(words + t) : 0;
    for (int C = 0; C < B; ++C) {
        double2 lv[16];
        const double2 *lrow = L + (size_t)(r0 + i) * Np + C * NB + q;
#pragma unroll
        for (int c = 0; c < 16; ++c) lv[c] = lrow[4 * c];
        if (t < 2 * NB) {
            const double x = await(words + (size_t)C * 2 * NB + t, seen, flags);
            reinterpret_cast<double *>(yc[C & 1])[t] = x;
            if (C + 1 < B) seen = peek(words + (size_t)(C + 1) * 2 * NB + t);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 16; ++c) part = cadd(part, cmul(lv[c], yc[C & 1][4 * c + q]));
    }
    part.x += __shfl_xor(part.x, 1);
    part.y += __shfl_xor(part.y, 1);
    part.x += __shfl_xor(part.x, 2);
    part.y += __shfl_xor(part.y, 2);
    if (q == 0) uvec[i] = csub(K ? kv[0] : rhs[r0 + i], part);
    __syncthreads();
    double2 y = make_double2(0, 0);
#pragma unroll
    for (int c = 0; c < 16; ++c) y = cadd(y, cmul(iv[c], uvec[4 * c + q]));
    y.x += __shfl_xor(y.x, 1);
    y.y += __shfl_xor(y.y, 1);
    y.x += __shfl_xor(y.x, 2);
    y.y += __shfl_xor(y.y, 2);
    if (q == 0) post(&ybuf[r0 + i], y);
}

// The RK4 stage update of row ii from its solve x = (S + eps I)^-1 K v:
// k = -i x; stage 0 stores the initial coefficients C = x.
__device__ inline void stage_update(int ii, double2 u, int stage, double dt, int N, double2 *__restrict__ C,
                                    double2 *__restrict__ Cacc, double2 *__restrict__ Cstage,
                                    double *__restrict__ r, double *__restrict__ R,
                                    const double *__restrict__ r_new, const double *__restrict__ R_new,
                                    int32_t *__restrict__ flags) {
    bool bad = false;
    if (stage == 0) {
        C[ii] = (ii < N) ? u : make_double2(0, 0);
        bad = !(isfinite(u.x) && isfinite(u.y));
    } else {
        const double2 k = make_double2(u.y, -u.x);   // -i x
        const double2 c = C[ii];
        if (stage == 1) {
            Cacc[ii] = k;
            Cstage[ii] = cadd(c, cscale(k, 0.5 * dt));
        } else if (stage == 2) {
            Cacc[ii] = cadd(Cacc[ii], cscale(k, 2.0));
            Cstage[ii] = cadd(c, cscale(k, 0.5 * dt));
        } else if (stage == 3) {
            Cacc[ii] = cadd(Cacc[ii], cscale(k, 2.0));
            Cstage[ii] = cadd(c, cscale(k, dt));
        } else {
            const double2 cn = cadd(c, cscale(cadd(Cacc[ii], k), dt / 6.0));
            C[ii] = cn;
            bad = !(isfinite(cn.x) && isfinite(cn.y));
            if (ii < N && r) {   // r == nullptr: Heun trajectories, positions set by the corrector
                r[ii] = r_new[ii];
                R[ii] = R_new[ii];
            }
        }
    }
    if (bad) {
        atomicOr(&flags[kFlagNonfinite], 1);
        atomicOr(&flags[kFlagHalt], 1);
    }
}

// Backward stage kernel: x_B = L_BB^-H (y_B - sum_{C>B} L_CB^H x_C), blocks
// from the bottom up; then the RK4 stage update of the block's rows.
// stage: 1..4; 0 = initial coefficients (C = x).
__global__ void __launch_bounds__(256) k_rk_bwd(const double2 *__restrict__ L, const double2 *__restrict__ Linv,
                                                double2 *__restrict__ ybuf, double2 *__restrict__ xbuf, int Np,
                                                int nblk, int stage, double dt, int N, double2 *__restrict__ C,
                                                double2 *__restrict__ Cacc, double2 *__restrict__ Cstage,
                                                double *__restrict__ r, double *__restrict__ R,
                                                const double *__restrict__ r_new, const double *__restrict__ R_new,
                                                int32_t *__restrict__ sync, int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    L = zshift(L, zo_);
    Linv = zshift(Linv, zo_);
    ybuf = zshift(ybuf, zo_);
    xbuf = zshift(xbuf, zo_);
    C = zshift(C, zo_);
    Cacc = zshift(Cacc, zo_);
    Cstage = zshift(Cstage, zo_);
    r = zshift(r, zo_);
    R = zshift(R, zo_);
    r_new = zshift(r_new, zo_);
    R_new = zshift(R_new, zo_);
    sync = zshift(sync, zo_);
    flags = zshift(flags, zo_);

    __shared__ double2 xc[2][NB], uvec[NB];
    __shared__ int slot[2];
    bool halt;
    const int ticket = take_ticket(&sync[kSyncTicketB], flags, slot, &halt);
    const int B = nblk - 1 - ticket;
    if (ticket == 0 && threadIdx.x == 0) sync[kSyncTicketF] = 0;
    const int t = threadIdx.x, i = t >> 2, q = t & 3;
    const int r0 = B * NB;
    double2 yb = make_double2(0, 0);
    if (q == 0) {
        yb = ybuf[r0 + i];
        post_pending(&ybuf[r0 + i]);
    }
    if (halt) {                                      // nobody waits for ever
        if (q == 0) post(&xbuf[r0 + i], make_double2(0, 0));
        return;
    }
    double2 iv[16];   // column i of L_BB^-1
#pragma unroll
    for (int c = 0; c < 16; ++c) iv[c] = Linv[(size_t)(r0 + 4 * c + q) * NB + i];
    // contributions of the blocks below (already solved): sum_k conj(L[C64+k][B64+i]) x[C64+k]
    double2 part = make_double2(0, 0);
    const double *words = reinterpret_cast<const double *>(xbuf);
    unsigned long long seen = t < 2 * NB && B < nblk - 1 ? peek(words + (size_t)(nblk - 1) * 2 * NB + t) : 0;
    for (int Cb = nblk - 1; Cb > B; --Cb) {
        double2 lv[16];
        const double2 *lcol = L + (size_t)(Cb * NB + q) * Np + r0 + i;
#pragma unroll
        for (int c = 0; c < 16; ++c) lv[c] = lcol[(size_t)(4 * c) * Np];
        if (t < 2 * NB) {
            const double x = await(words + (size_t)Cb * 2 * NB + t, seen, flags);
            reinterpret_cast<double *>(xc[Cb & 1])[t] = x;
            if (Cb - 1 > B) seen = peek(words + (size_t)(Cb - 1) * 2 * NB + t);
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 16; ++c) part = cadd(part, cmulc(lv[c], xc[Cb & 1][4 * c + q]));
    }
    part.x += __shfl_xor(part.x, 1);
    part.y += __shfl_xor(part.y, 1);
    part.x += __shfl_xor(part.x, 2);
    part.y += __shfl_xor(part.y, 2);
    if (q == 0) uvec[i] = csub(yb, part);
    __syncthreads();
    double2 u = make_double2(0, 0);
#pragma unroll
    for (int c = 0; c < 16; ++c) u = cadd(u, cmulc(iv[c], uvec[4 * c + q]));
    u.x += __shfl_xor(u.x, 1);
    u.y += __shfl_xor(u.y, 1);
    u.x += __shfl_xor(u.x, 2);
    u.y += __shfl_xor(u.y, 2);
    if (q == 0) {
        post(&xbuf[r0 + i], u);
        stage_update(r0 + i, u, stage, dt, N, C, Cacc, Cstage, r, R, r_new, R_new, flags);
    }
}

// The four stages of one block (N <= 64) in one work-group of 16 waves: no
// launch between them.  Thread t has row t / 16 of K, L^-1 and L^-H, columns
// t % 16 + 16 m, so a product is four terms per thread and a sum over the 16
// lanes of a DPP row; L^-H comes from L^-1 through LDS.  The next stage's
// matrices are requested before this stage's sums.  Latency-bound: 14 us for
// the step's four stages against 53 in twelve launches (41 with rows summed
// over 64 lanes by shuffles, which fill the LDS pipe).
constexpr int kSoloWaves = 16;

struct SoloArgs {
    const double2 *K[4], *X[4];
    double2 *C;
    double *r, *R;
    const double *r_new, *R_new;
    int32_t *flags;
    double dt;
    int N;
};

__global__ void __launch_bounds__(64 * kSoloWaves) k_rk4_solo(SoloArgs g, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    int32_t *flags = zshift(g.flags, zo_);
    if (flags[kFlagHalt]) return;
    __shared__ double2 tr[NB][NB + 1];               // L^-1 on its way to L^-H
    __shared__ double2 v[NB], w[NB], y[NB], sol[NB]; // the stage's vector, K v, L^-1 K v, the solution
    const int t = threadIdx.x, row = t >> 4, c = t & 15;
    double2 *C = zshift(g.C, zo_);
    double2 k[2][4], x[2][4], h[4];
    auto load = [&](int s) __attribute__((always_inline)) {
        const double2 *K = zshift(g.K[s], zo_) + row * NB + c, *X = zshift(g.X[s], zo_) + row * NB + c;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            k[s & 1][m] = K[16 * m];
            x[s & 1][m] = X[16 * m];
        }
    };
    // row `row` of M u, on the 16 lanes of the row
    auto times = [&](const double2 (&a)[4], const double2 *u) __attribute__((always_inline)) {
        double2 p = cmul(a[0], u[c]);
#pragma unroll
        for (int m = 1; m < 4; ++m) p = cadd(p, cmul(a[m], u[c + 16 * m]));
        return make_double2(row16_sum(p.x), row16_sum(p.y));
    };
    load(0);
    double2 c0 = make_double2(0, 0), acc = c0;
    if (t < NB) {
        c0 = C[t];
        v[t] = c0;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (s < 3) load(s + 1);
#pragma unroll
        for (int m = 0; m < 4; ++m) tr[row][c + 16 * m] = x[s & 1][m];
        __syncthreads();
        double2 p = times(k[s & 1], v);
        if (c == 0) w[row] = p;
#pragma unroll
        for (int m = 0; m < 4; ++m) h[m] = cconj(tr[c + 16 * m][row]);
        __syncthreads();
        p = times(x[s & 1], w);
        if (c == 0) y[row] = p;
        __syncthreads();
        p = times(h, y);
        if (c == 0) sol[row] = p;
        __syncthreads();
        if (t < NB) {
            // k = -i x and the stage update, as stage_update
            const double2 u = sol[t], kk = make_double2(u.y, -u.x);
            if (s < 3) {
                acc = s == 0 ? kk : cadd(acc, cscale(kk, 2.0));
                v[t] = cadd(c0, cscale(kk, s < 2 ? 0.5 * g.dt : g.dt));
            } else {
                const double2 cn = cadd(c0, cscale(cadd(acc, kk), g.dt / 6.0));
                C[t] = cn;
                if (!(isfinite(cn.x) && isfinite(cn.y))) {
                    atomicOr(&flags[kFlagNonfinite], 1);
                    atomicOr(&flags[kFlagHalt], 1);
                }
                if (t < g.N && g.r) {                // r == nullptr: Heun trajectories, positions set by the corrector
                    zshift(g.r, zo_)[t] = zshift(g.r_new, zo_)[t];
                    zshift(g.R, zo_)[t] = zshift(g.R_new, zo_)[t];
                }
            }
        }
    }
}

// Stages through the explicit inverse of the factor, A^-1 = L^-H L^-1, with
// one step of iterative refinement: x0 = L^-H (L^-1 rhs) (two triangular
// k_matvec), res = rhs - A x0 (k_rk_resid, A formed from S as in the
// assembly), x = x0 + L^-H (L^-1 res) (k_matvec, then k_rk_apply with the
// stage update of the row).  The refinement brings the explicit inverse's
// error, of the order of cond(A) times its rounding, back to that of a
// solve with the factor.  One row per work-group.
__global__ void __launch_bounds__(256) k_rk_resid(const double2 *__restrict__ Sa, const double2 *__restrict__ Sb,
                                                  double eps, const double2 *__restrict__ x,
                                                  const double2 *__restrict__ rhs, double2 *__restrict__ res, int Np,
                                                  const int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    Sa = zshift(Sa, zo_);
    Sb = zshift(Sb, zo_);
    x = zshift(x, zo_);
    rhs = zshift(rhs, zo_);
    res = zshift(res, zo_);
    flags = zshift(flags, zo_);

    if (flags[kFlagHalt]) return;
    const int rowi = blockIdx.x;
    const double2 *ma = Sa + (size_t)rowi * Np;
    const double2 *mb = Sb ? Sb + (size_t)rowi * Np : nullptr;
    const double2 acc = row_sum_wg(rowi, Np, kPartAll, [&](int c) {
        const double reg = (c == rowi) ? eps : 0.0;
        const double2 sa = ma[c];
        double2 a;
        if (mb) {                                    // midpoint: (S_a + S_b) / 2 + eps I
            const double2 sb = mb[c];
            a = make_double2(0.5 * (sa.x + sb.x) + reg, 0.5 * (sa.y + sb.y));
        } else {                                     // endpoint: S_a + eps I
            a = make_double2(sa.x + reg, sa.y);
        }
        return cmul(a, x[c]);
    });
    if (threadIdx.x == 0) res[rowi] = csub(rhs[rowi], acc);
}

__global__ void __launch_bounds__(256) k_rk_apply(const double2 *__restrict__ H, const double2 *__restrict__ z,
                                                  const double2 *__restrict__ x0, int Np, int stage, double dt, int N,
                                                  double2 *__restrict__ C, double2 *__restrict__ Cacc,
                                                  double2 *__restrict__ Cstage, double *__restrict__ r,
                                                  double *__restrict__ R, const double *__restrict__ r_new,
                                                  const double *__restrict__ R_new, int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    H = zshift(H, zo_);
    z = zshift(z, zo_);
    x0 = zshift(x0, zo_);
    C = zshift(C, zo_);
    Cacc = zshift(Cacc, zo_);
    Cstage = zshift(Cstage, zo_);
    r = zshift(r, zo_);
    R = zshift(R, zo_);
    r_new = zshift(r_new, zo_);
    R_new = zshift(R_new, zo_);
    flags = zshift(flags, zo_);

    if (flags[kFlagHalt]) return;
    const int rowi = blockIdx.x;
    const double2 *m = H + (size_t)rowi * Np;
    const double2 acc = row_sum_wg(rowi, Np, kPartUpper, [&](int c) { return cmul(m[c], z[c]); });   // (L^-H z)_rowi
    if (threadIdx.x == 0)
        stage_update(rowi, cadd(x0[rowi], acc), stage, dt, N, C, Cacc, Cstage, r, R, r_new, R_new, flags);
}

// H = F^H over the lower part of F (F = L^-1): 32 x 32 tiles through LDS,
// tile (bi, bj) of F with bi >= bj to tile (bj, bi) of H (the parts of F
// above and of H below the diagonal are neither read nor written).
__global__ void __launch_bounds__(256) k_conj_transpose(const double2 *__restrict__ F0, const double2 *__restrict__ F1,
                                                        double2 *__restrict__ H0, double2 *__restrict__ H1, int Np,
                                                        const int32_t *__restrict__ flags) {
    if (flags[kFlagHalt]) return;
    const int bi = blockIdx.x, bj = blockIdx.y;
    if (bi < bj) return;
    const double2 *F = blockIdx.z ? F1 : F0;
    double2 *H = blockIdx.z ? H1 : H0;
    __shared__ double2 tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 8 rows per pass
#pragma unroll
    for (int r = ty; r < 32; r += 8) tile[r][tx] = F[(size_t)(32 * bi + r) * Np + 32 * bj + tx];
    __syncthreads();
#pragma unroll
    for (int r = ty; r < 32; r += 8) H[(size_t)(32 * bj + r) * Np + 32 * bi + tx] = cconj(tile[tx][r]);
}

__global__ void k_set_table(long long *__restrict__ tab, BatchTable t, int n) {
    if ((int)threadIdx.x < n) tab[threadIdx.x] = t.off[threadIdx.x];
}

__global__ void k_fill_u64(unsigned long long *p, int n, unsigned long long v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_i32(int32_t *p, int n, int32_t v, const long long *__restrict__ zoff) {
    const long long zo_ = batch_offset(zoff);
    p = zshift(p, zo_);

    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

void launch_assemble(const Dims &d, const Bufs &b, int parity, AssemblePart part, hipStream_t s) {
    const int Np = padded(d.N);
    const size_t tot = (size_t)Np * Np;
    const bool initial = part == kAssembleInitial;
    const int cur = parity, nxt = initial ? parity : 1 - parity;
    hipLaunchKernelGGL(k_assemble, dim3((unsigned)((tot + 255) / 256), 1, d.batch), dim3(256), 0, s, b.S1, b.S2,
                       b.E1a, b.E1b, b.E2a, b.E2b, b.Wc, d.bilinear, b.Smat[cur], b.Kmat[cur], b.r, b.R, b.r_new, b.R_new, d.mp,
                       d.N, Np, d.eps, (int)part, b.Smat[nxt], b.Kminus, b.Kmat[nxt], b.Lmid, b.L[nxt], b.Kmid, b.flags,
                       d.zoff, d.mpd);
}

void launch_cholesky(const Dims &d, const Bufs &b, double2 *A0, double2 *A1, double2 *X0, double2 *X1, int count,
                     hipStream_t s, double2 *F0, double2 *F1, double2 *H0, double2 *H1, bool inverses) {
    const int Np = padded(d.N);
    for (int kb = 0; kb < Np; kb += NB) {
        const int below = Np - kb - NB;
        hipLaunchKernelGGL(k_chol_panel, dim3(below / 64 + 1, count, d.batch), dim3(256), 0, s, A0, A1, Np, kb,
                           b.chol_diag, X0, X1, F0, F1, b.flags, d.zoff);
        if (below > 0) {
            const int mt = below / 32;
            hipLaunchKernelGGL(k_chol_update, dim3(mt * (mt + 1) / 2, count, d.batch), dim3(256), 0, s, A0, A1, Np, kb,
                               b.flags, d.zoff);
        }
    }
    if (F0 && inverses) launch_factor_inverses(d, b, A0, A1, count, s, F0, F1, H0, H1);
}

void launch_factor_inverses(const Dims &d, const Bufs &b, const double2 *A0, const double2 *A1, int count,
                            hipStream_t s, double2 *F0, double2 *F1, double2 *H0, double2 *H1) {
    const int Np = padded(d.N);
    double2 *Fs[2] = {F0, F1 ? F1 : F0};
    // X = L^-1 by block recursion, [[A, 0], [C, D]]^-1 = [[A', 0], [-D' C A', D']],
    // from the 64 x 64 diagonal inverses up: at block size h, the Np / (2 h) pairs
    // of every factor take T = C A' and then -D' T (X's upper triangle stays zero)
    const double2 *L2[2] = {A0, A1};
    for (int h = NB; h < Np; h *= 2) {
        GemmBatch g{};
        g.lda = g.ldb = g.ldo = Np;
        g.M = g.N = g.K = h;
        g.npairs = Np / (2 * h);
        g.stride = 2LL * h * (Np + 1);
        const dim3 grid((h / kGT) * (h / kGT), 1, count * g.npairs);
        for (int f = 0; f < 2; ++f) {                      // T = C A'
            g.A[f] = L2[f] + (size_t)h * Np;
            g.B[f] = Fs[f];
            g.O[f] = b.Tinv[f] + (size_t)h * Np;
        }
        g.alpha = 1.0;
        g.lower_a = 0;
        g.lower_b = 1;                                     // A' lower triangular
        hipLaunchKernelGGL(k_cgemm, grid, dim3(256), 0, s, g, b.flags);
        for (int f = 0; f < 2; ++f) {                      // X_DA = -D' T
            g.A[f] = Fs[f] + (size_t)h * Np + h;
            g.B[f] = b.Tinv[f] + (size_t)h * Np;
            g.O[f] = Fs[f] + (size_t)h * Np;
        }
        g.alpha = -1.0;
        g.lower_a = 1;                                     // D' lower triangular
        g.lower_b = 0;
        hipLaunchKernelGGL(k_cgemm, grid, dim3(256), 0, s, g, b.flags);
    }
    // L^-H for the stage solves
    hipLaunchKernelGGL(k_conj_transpose, dim3(Np / 32, Np / 32, count), dim3(256), 0, s, F0, F1 ? F1 : F0, H0,
                       H1 ? H1 : H0, Np, b.flags);
}

void launch_rk4(const Dims &d, const Bufs &b, int parity, hipStream_t s) {
    const int Np = padded(d.N), nblk = Np / NB;
    const int cur = parity, nxt = 1 - parity;
    const double2 *Ks[4] = {b.Kmat[cur], b.Kmid, b.Kmid, b.Kminus};
    const double2 *Ls[4] = {b.L[cur], b.Lmid, b.Lmid, b.L[nxt]};
    const double2 *Xs[4] = {b.Linv[cur], b.Linvmid, b.Linvmid, b.Linv[nxt]};
    const double2 *Fs[4] = {b.Finv[cur], b.Finvmid, b.Finvmid, b.Finv[nxt]};
    const double2 *Hs[4] = {b.Hinv[cur], b.Hinvmid, b.Hinvmid, b.Hinv[nxt]};
    // with Heun trajectories the last stage leaves x_k in place for the corrector
    double *cr = d.traj == 1 ? nullptr : b.r, *cR = d.traj == 1 ? nullptr : b.R;
    if (!d.sinv && nblk == 1) {
        SoloArgs g{};
        for (int st = 0; st < 4; ++st) {
            g.K[st] = Ks[st];
            g.X[st] = Xs[st];
        }
        g.C = b.C;
        g.r = cr;
        g.R = cR;
        g.r_new = b.r_new;
        g.R_new = b.R_new;
        g.flags = b.flags;
        g.dt = d.dt;
        g.N = d.N;
        hipLaunchKernelGGL(k_rk4_solo, dim3(1, 1, d.batch), dim3(64 * kSoloWaves), 0, s, g, d.zoff);
        return;
    }
    for (int st = 1; st <= 4; ++st) {
        const double2 *v = (st == 1) ? b.C : b.Cstage;
        if (d.sinv) {
            hipLaunchKernelGGL(k_matvec, dim3(Np, 1, d.batch), dim3(256), 0, s, Ks[st - 1], v, b.rhs, Np,
                               (int)kPartAll, b.flags, d.zoff);
            // A of the stage: S_k + eps I, the midpoint average + eps I (stages 2, 3), S_k+1 + eps I
            const double2 *Sa = st == 4 ? b.Smat[nxt] : b.Smat[cur];
            const double2 *Sb = (st == 2 || st == 3) ? b.Smat[nxt] : nullptr;
            hipLaunchKernelGGL(k_matvec, dim3(Np, 1, d.batch), dim3(256), 0, s, Fs[st - 1], b.rhs, b.zvec, Np,
                               (int)kPartLower, b.flags, d.zoff);
            hipLaunchKernelGGL(k_matvec, dim3(Np, 1, d.batch), dim3(256), 0, s, Hs[st - 1], b.zvec, b.y, Np,
                               (int)kPartUpper, b.flags, d.zoff);
            hipLaunchKernelGGL(k_rk_resid, dim3(Np, 1, d.batch), dim3(256), 0, s, Sa, Sb, d.eps, b.y, b.rhs, b.res,
                               Np, b.flags, d.zoff);
            hipLaunchKernelGGL(k_matvec, dim3(Np, 1, d.batch), dim3(256), 0, s, Fs[st - 1], b.res, b.zvec, Np,
                               (int)kPartLower, b.flags, d.zoff);
            hipLaunchKernelGGL(k_rk_apply, dim3(Np, 1, d.batch), dim3(256), 0, s, Hs[st - 1], b.zvec, b.y, Np, st,
                               d.dt, d.N, b.C, b.Cacc, b.Cstage, cr, cR, b.r_new, b.R_new, b.flags, d.zoff);
            continue;
        }
        hipLaunchKernelGGL(k_rk_fwd, dim3(nblk, 1, d.batch), dim3(256), 0, s, Ks[st - 1], v, nullptr, Ls[st - 1],
                           Xs[st - 1], b.ysol, b.xsol, Np, b.solve_sync, b.flags, d.zoff);
        hipLaunchKernelGGL(k_rk_bwd, dim3(nblk, 1, d.batch), dim3(256), 0, s, Ls[st - 1], Xs[st - 1], b.ysol, b.xsol,
                           Np, nblk, st, d.dt, d.N, b.C, b.Cacc, b.Cstage, cr, cR, b.r_new, b.R_new, b.solve_sync, b.flags,
                           d.zoff);
    }
}

void launch_solve_initial(const Dims &d, const Bufs &b, int parity, double2 *rhs, hipStream_t s) {
    const int Np = padded(d.N), nblk = Np / NB;
    hipLaunchKernelGGL(k_rk_fwd, dim3(nblk), dim3(256), 0, s, nullptr, nullptr, rhs, b.L[parity], b.Linv[parity],
                       b.ysol, b.xsol, Np, b.solve_sync, b.flags, nullptr);
    hipLaunchKernelGGL(k_rk_bwd, dim3(nblk), dim3(256), 0, s, b.L[parity], b.Linv[parity], b.ysol, b.xsol, Np, nblk, 0,
                       d.dt, d.N, b.C, b.Cacc, b.Cstage, b.r, b.R, b.r_new, b.R_new, b.solve_sync, b.flags, nullptr);
}

void launch_solve_reset(const Dims &d, const Bufs &b, hipStream_t s) {
    const int Np = padded(d.N);
    hipLaunchKernelGGL(k_fill_u64, dim3((2 * Np + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(b.ysol), 2 * Np, kPending);
    hipLaunchKernelGGL(k_fill_u64, dim3((2 * Np + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(b.xsol), 2 * Np, kPending);
}

void launch_set_table(long long *tab, const BatchTable &t, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_set_table, dim3(1), dim3(kMaxBatch), 0, s, tab, t, n);
}

void launch_fill_i32(int32_t *p, int n, int32_t v, hipStream_t s, int batch, const long long *zoff) {
    hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256, 1, batch), dim3(256), 0, s, p, n, v, zoff);
}

}  // namespace icwf
