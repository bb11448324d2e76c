// Born-Oppenheimer states on the GPU: the lowest eigenpairs of the clamped-
// nucleus electronic Hamiltonian h_e(R_j) = T_spec + diag(W(r_i, R_j)) for a
// list of R_j (the basis of the paper's BO populations and decoherence
// indicator, and of its initial state, the first excited BO state).
//
// One work-group per R_j runs block LOBPCG (Knyazev 2001) to the end in one
// launch:
//   * h_e is applied through the spectral kinetic operator, two real vectors
//     per complex transform (T is real and even in k, so T(u + i v) =
//     T u + i T v), in LDS: decimation in frequency from natural to
//     bit-reversed order forward, the multiplier k^2/2m in that order, decimation
//     in time back, then + W(r_i, R_j) u_i.  Up to 1024 points every wave has a
//     transform of its own, eight points per lane and pass (three radix-2 stages
//     in registers between two LDS exchanges) and no barrier; above, the
//     work-group shares one, a stage at a time;
//   * the preconditioner is (T_spec + c)^-1, the same transforms with the
//     multiplier 1/(k^2/2m + c), c = max(1, max W - min W) on the grid;
//   * each iteration orthonormalises [X, P(residuals), previous directions] as
//     one block, twice: the Gram matrix of the unit columns by matrix products,
//     its Cholesky factor R (columns that keep less than 1e-7 of their norm are
//     dropped), C R^-1 by substitution; the second time mends what the first
//     leaves for columns that are nearly dependent.  Then h_e is applied to the
//     whole basis afresh, the projected matrix (matrix products again) is
//     diagonalised by cyclic Jacobi (parallel round-robin ordering), and the m
//     lowest Ritz pairs are the new block, the non-X part of their coefficients
//     the new directions, h_e x - theta x the residuals;
//   * it stops when every wanted residual norm is at most tol.
// What bounds it is latency: some 40 iterations of dependent small phases per
// R_j, one work-group per compute unit.  512 points, 256 values of R, 3 states,
// whole calls: 20.7 ms with a dot product and two barriers per pair of columns,
// rotations by divisions and roots with a barrier per phase, and transforms by
// the work-group; 4.5 ms now (orthonormalisation 7.2 -> 0.9 ms, Jacobi 3.7 ->
// 1.1, projected matrix 2.7 -> 0.25, h_e 1.6 -> 0.7).  1024 points, 128 values,
// 2 states: 20.6 -> 6.6 ms; 128 points, 64 values, 3 states: 13.1 -> 2.8 ms.
// Vectors live in a per-R_j slice of the caller's workspace (L2-resident
// during the work-group's life); the transform buffer, the projected matrix
// and its rotations live in LDS.
#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/icwf_bo.h"
#include "icwf_plan.hpp"

namespace icwf {

namespace {

constexpr int kBoThreads = 256;
constexpr int kBoWaves = kBoThreads / 64;
constexpr int kBoMaxBlock = 12;              // n_states + guard vectors
constexpr int kBoMaxZ = 3 * kBoMaxBlock;     // columns of the Rayleigh-Ritz basis
constexpr int kChunk = 8;                    // dot products reduced together

struct BoArgs {
    int n, m, nwant, max_iter;
    double tol, r_min, h;
    ModelParams mp;
    const double *Rv;        // [nv]
    const double *kin;       // [n] k^2 / (2 m_r), FFT order
    const double2 *tw;       // [n / 2] exp(-2 pi i k / n)
    double *ws;              // per-value slices of ws_stride doubles
    size_t ws_stride;
    double *states;          // [nv][nwant][n] (grid-normalised)
    double *energies;        // [nv][nwant]
    int32_t *iters;          // [nv]
    double *resid;           // [nv]
    int32_t *flags;          // kFlagNonfinite on a non-finite potential
};

// Doubles of one R_j's slice: V, Z, HZ (kBoMaxZ columns each).
inline size_t bo_stride(int n) { return (size_t)n * (1 + 2 * kBoMaxZ); }

// 1 / sqrt(x) of a normal x > 0: the hardware's estimate y, with e = 1 - x y^2
// small, times (1 - e)^-1/2 to second order.
__device__ __forceinline__ double inverse_root(double x) {
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// v of lane i (the same i in all lanes).
__device__ __forceinline__ double lane_value(double v, int i) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i),
                            __builtin_amdgcn_readlane(__double2loint(v), i));
}

__device__ inline double wave_sum(double v) {
    v = row16_sum(v);
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) s += lane_value(v, 16 * r);
    return s;
}

// Sums cnt (<= kChunk) per-thread values over the work-group into out[0..cnt)
// (LDS), in a fixed order.
__device__ inline void block_sums(const double (&v)[kChunk], int cnt, double *red, double *out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
        if (c < cnt) {
            const double s = wave_sum(v[c]);
            if (lane == 0) red[wave * kChunk + c] = s;
        }
    }
    __syncthreads();
    if (threadIdx.x < cnt) {
        const int c = threadIdx.x;
        double t = red[c];
#pragma unroll
        for (int w = 1; w < kBoWaves; ++w) t += red[w * kChunk + c];
        out[c] = t;
    }
    __syncthreads();
}

// T or (T + c)^-1 applied to the pair (u, v) (v may be null), out to (ou, ov);
// with add_v the potential term V u is added (h_e).  fb: n complex in LDS.
template <int LOG2N>
__device__ void spectral_pair(const BoArgs &A, const double *u, const double *v, double *ou, double *ov,
                              const double *V, bool hamiltonian, double c, double2 *fb) {
    constexpr int n = 1 << LOG2N;
    const int tid = threadIdx.x;
    for (int e = tid; e < n; e += kBoThreads) {
        const int br = (int)(__brev((unsigned)e) >> (32 - LOG2N));
        fb[br] = make_double2(u[e], v ? v[e] : 0.0);
    }
    __syncthreads();
    // forward transform: decimation in time, bit-reversed in, natural out
#pragma unroll 1
    for (int s = 1; s <= LOG2N; ++s) {
        const int half = 1 << (s - 1), tstr = n >> s;
        for (int b = tid; b < n / 2; b += kBoThreads) {
            const int pos = b & (half - 1);
            const int i0 = ((b >> (s - 1)) << s) + pos, i1 = i0 + half;
            const double2 w = A.tw[pos * tstr];
            const double2 x0 = fb[i0], x1 = cmul(fb[i1], w);
            fb[i0] = cadd(x0, x1);
            fb[i1] = csub(x0, x1);
        }
        __syncthreads();
    }
    for (int k = tid; k < n; k += kBoThreads) {
        const double mult = hamiltonian ? A.kin[k] : 1.0 / (A.kin[k] + c);
        fb[k] = cscale(fb[k], mult);
    }
    __syncthreads();
    // inverse transform: decimation in frequency, natural in, bit-reversed out
#pragma unroll 1
    for (int s = LOG2N; s >= 1; --s) {
        const int half = 1 << (s - 1), tstr = n >> s;
        for (int b = tid; b < n / 2; b += kBoThreads) {
            const int pos = b & (half - 1);
            const int i0 = ((b >> (s - 1)) << s) + pos, i1 = i0 + half;
            const double2 w = cconj(A.tw[pos * tstr]);
            const double2 x0 = fb[i0], x1 = fb[i1];
            fb[i0] = cadd(x0, x1);
            fb[i1] = cmul(csub(x0, x1), w);
        }
        __syncthreads();
    }
    const double inv = 1.0 / n;
    for (int e = tid; e < n; e += kBoThreads) {
        const double2 y = fb[__brev((unsigned)e) >> (32 - LOG2N)];
        double yu = y.x * inv, yv = y.y * inv;
        if (hamiltonian) {
            yu += V[e] * u[e];
            if (v) yv += V[e] * v[e];
        }
        ou[e] = yu;
        if (v) ov[e] = yv;
    }
    __syncthreads();
}

// Place of entry i of a wave's transform buffer: one pad per 8 entries keeps
// the exchanges of all passes (nearly) free of bank conflicts.
__device__ inline int fft_at(int i) { return i + (i >> 3); }

// Between the LDS writes of a wave and its other lanes' reads of them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// RADIX = 2, 4 or 8 points per butterfly: log2 RADIX radix-2 stages in
// registers, on blocks of `len` points, elements len / RADIX apart.  Forward:
// decimation in frequency; back: the same stages, conjugated, in reverse.
template <int LOG2N, int RADIX, bool BACK>
__device__ __forceinline__ void wave_pass(double2 *fb, const double2 *tw, int log2len, int lane) {
    constexpr int n = 1 << LOG2N, LR = RADIX == 8 ? 3 : RADIX == 4 ? 2 : 1, BF = n / RADIX;
    const int lsub = log2len - LR;                   // log2 of the element distance
#pragma unroll
    for (int b0 = 0; b0 < BF; b0 += 64) {
        const int b = b0 + lane;
        if (BF < 64 && b >= BF) break;
        const int j = b & ((1 << lsub) - 1), base = ((b >> lsub) << log2len) + j;
        double2 x[RADIX];
#pragma unroll
        for (int q = 0; q < RADIX; ++q) x[q] = fb[fft_at(base + (q << lsub))];
#pragma unroll
        for (int t = 0; t < LR; ++t) {
            const int st = BACK ? LR - 1 - t : t;    // stage: distance RADIX >> (st + 1) elements
            const int dist = RADIX >> (st + 1);
#pragma unroll
            for (int q = 0; q < RADIX; ++q) {
                if (q & dist) continue;
                // exp(-2 pi i pos / (len >> st)), pos the place in the half block
                const int pos = j + ((q & (dist - 1)) << lsub);
                const double2 w = tw[pos << (LOG2N - log2len + st)];
                const double2 u = x[q], v = x[q + dist];
                if (!BACK) {
                    x[q] = cadd(u, v);
                    x[q + dist] = cmul(csub(u, v), w);
                } else {
                    const double2 z = cmulc(w, v);
                    x[q] = cadd(u, z);
                    x[q + dist] = csub(u, z);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < RADIX; ++q) fb[fft_at(base + (q << lsub))] = x[q];
    }
    wave_sync();
}

// As spectral_pair, by one wave on its own buffer: in-order LDS, no barrier.
template <int LOG2N>
__device__ void spectral_wave(const BoArgs &A, const double *u, const double *v, double *ou, double *ov,
                              const double *V, bool hamiltonian, double c, double2 *fb, const double2 *tw) {
    constexpr int n = 1 << LOG2N, R0 = LOG2N % 3 == 0 ? 3 : LOG2N % 3;   // stages of the last pass forward
    const int lane = threadIdx.x & 63;
    for (int e = lane; e < n; e += 64) fb[fft_at(e)] = make_double2(u[e], v ? v[e] : 0.0);
    wave_sync();
#pragma unroll 1
    for (int l = LOG2N; l > R0; l -= 3) wave_pass<LOG2N, 8, false>(fb, tw, l, lane);
    wave_pass<LOG2N, 1 << R0, false>(fb, tw, R0, lane);
    for (int p = lane; p < n; p += 64) {
        const double k = A.kin[(int)(__brev((unsigned)p) >> (32 - LOG2N))];
        fb[fft_at(p)] = cscale(fb[fft_at(p)], hamiltonian ? k : 1.0 / (k + c));
    }
    wave_sync();
    wave_pass<LOG2N, 1 << R0, true>(fb, tw, R0, lane);
#pragma unroll 1
    for (int l = R0 + 3; l <= LOG2N; l += 3) wave_pass<LOG2N, 8, true>(fb, tw, l, lane);
    const double inv = 1.0 / n;
    for (int e = lane; e < n; e += 64) {
        const double2 y = fb[fft_at(e)];
        double yu = y.x * inv, yv = y.y * inv;
        if (hamiltonian) {
            yu += V[e] * u[e];
            if (v) yv += V[e] * v[e];
        }
        ou[e] = yu;
        if (v) ov[e] = yv;
    }
    wave_sync();
}

// h_e or the preconditioner on `cols` columns of `in`, to `out`.
template <int LOG2N>
__device__ void apply_columns(const BoArgs &A, const double *in, double *out, int cols, const double *V,
                              bool hamiltonian, double c, double2 *fb, const double2 *tw) {
    constexpr int n = 1 << LOG2N;
    if constexpr (LOG2N <= 10) {
        const int wave = threadIdx.x >> 6;
        for (int q = 2 * wave; q < cols; q += 2 * kBoWaves) {
            const bool two = q + 1 < cols;
            const double *u = in + (size_t)q * n;
            double *ou = out + (size_t)q * n;
            spectral_wave<LOG2N>(A, u, two ? u + n : nullptr, ou, two ? ou + n : nullptr, V, hamiltonian, c,
                                 fb + wave * fft_at(n), tw);
        }
        __syncthreads();
    } else {
        for (int q = 0; q < cols; q += 2) {
            const bool two = q + 1 < cols;
            const double *u = in + (size_t)q * n;
            double *ou = out + (size_t)q * n;
            spectral_pair<LOG2N>(A, u, two ? u + n : nullptr, ou, two ? ou + n : nullptr, V, hamiltonian, c, fb);
        }
    }
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// G[a][b] = x_a . y_b for the first k columns of X and Y (a <= b computed,
// mirrored), by matrix products: 16 x 16 tiles of (a, b), the grid points the
// reduction, in steps of 8 taken by the waves in turn; part: 256 doubles a wave.
template <int LOG2N>
__device__ void gram(const double *X, const double *Y, int k, double *G, double (*part)[256]) {
    constexpr int n = 1 << LOG2N;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = lane & 15, quarter = lane >> 4;
    for (int a0 = 0; a0 < k; a0 += 16)
        for (int b0 = a0; b0 < k; b0 += 16) {
            const double *x = X + (size_t)min(a0 + row, k - 1) * n + 2 * quarter;
            const double *y = Y + (size_t)min(b0 + row, k - 1) * n + 2 * quarter;
            dbl4 acc = {0, 0, 0, 0};
#pragma unroll 4
            for (int e = 8 * wave; e < n; e += 8 * kBoWaves) {
                const double2 xe = *reinterpret_cast<const double2 *>(x + e), ye = *reinterpret_cast<const double2 *>(y + e);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xe.x, ye.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xe.y, ye.y, acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) part[wave][16 * mfma_row_f64(lane, v) + row] = acc[v];
            __syncthreads();
            static_assert(kBoThreads == 256, "a thread for each entry of the tile");
            const int a = a0 + (tid >> 4), b = b0 + (tid & 15);
            if (a < k && b < k && a <= b) {
                double g = part[0][tid];
#pragma unroll
                for (int w = 1; w < kBoWaves; ++w) g += part[w][tid];
                G[a * k + b] = g;
                G[b * k + a] = g;
            }
            __syncthreads();
        }
}

// Orthonormalises the first k columns of Z in place, in their order (at most
// MZ of them); returns how many are left.
template <int LOG2N, int MZ>
__device__ int orthonormalise(double *Z, int k, double *M, double (*part)[256], double *scl, int *pos) {
    constexpr int n = 1 << LOG2N;
    const int tid = threadIdx.x;
    for (int pass = 0; pass < 2; ++pass) {
        gram<LOG2N>(Z, Z, k, M, part);
        if (tid < 64) {
            // Cholesky by one wave, column `lane` of the matrix in a lane's
            // registers.  Unit columns first (scl; 0 drops a zero or non-finite
            // one); column j of R in row j of M, 1 / R_jj on the diagonal; pos:
            // place of a column, -1: dropped, its row and column zeros.
            const int lane = tid;
            double col[MZ];
#pragma unroll
            for (int i = 0; i < MZ; ++i) col[i] = i < k && lane < k ? M[i * k + lane] : 0.0;
            double mine = 0.0;
#pragma unroll
            for (int i = 0; i < MZ; ++i) mine = lane == i ? col[i] : mine;
            mine = mine > 1e-290 && isfinite(mine) ? inverse_root(mine) : 0.0;
#pragma unroll
            for (int i = 0; i < MZ; ++i) col[i] *= mine * lane_value(mine, i);
            int kept = 0, place = -1;
#pragma unroll
            for (int j = 0; j < MZ; ++j) {
                const double d = lane_value(col[j], j);
                // a column kept before has nearly all of its norm left
                const bool keep = d > (pass ? 0.1 : 1e-14);
                const double inv = keep ? inverse_root(d) : 0.0;
                col[j] = keep ? col[j] * inv : 0.0;  // (it may be NaN)
#pragma unroll
                for (int i = j + 1; i < MZ; ++i) col[i] -= lane_value(col[j], i) * col[j];
                if (lane == j) {
                    place = keep ? kept : -1;
                    col[j] = inv;
                }
                kept += keep;
            }
#pragma unroll
            for (int i = 0; i < MZ; ++i)
                if (i <= lane && lane < MZ) M[lane * MZ + i] = place < 0 ? 0.0 : col[i];
            if (lane < MZ) {
                scl[lane] = mine;
                pos[lane] = place;
            }
            if (lane == 0) pos[MZ] = kept;
        }
        __syncthreads();
        // Z <- Z R^-1, element by element: z_j = (c_j - sum_{i<j} R_ij z_i) / R_jj
        for (int e = tid; e < n; e += kBoThreads) {
            double z[MZ];
#pragma unroll
            for (int j = 0; j < MZ; ++j) {
                const double f = scl[j];
                z[j] = j < k ? Z[(size_t)j * n + e] : 0.0;
                z[j] = f != 0.0 ? f * z[j] : 0.0;
            }
#pragma unroll
            for (int j = 0; j < MZ; ++j) {
                double x = z[j];
#pragma unroll
                for (int i = 0; i < j; ++i) x -= M[j * MZ + i] * z[i];
                z[j] = x * M[j * MZ + j];
                // here and now: not sunk to the store, with R kept for it in scratch
                asm volatile("" : "+v"(z[j])::"memory");
            }
#pragma unroll
            for (int j = 0; j < MZ; ++j) {
                const int at = __builtin_amdgcn_readfirstlane(pos[j]);
                if (at >= 0) Z[(size_t)at * n + e] = z[j];
            }
        }
        __syncthreads();
        k = pos[MZ];
        __syncthreads();
    }
    return k;
}

// The rotation (c, s) that clears b / 2 between diagonal entries g_p and g_q = g_p + d,
// of at most pi / 4: cos 2t = |d| / h, h = |(d, b)|; c = sqrt((1 + cos 2t) / 2),
// s = sign(d) b / (2 h c).
__device__ __forceinline__ double2 rotation(double d, double b) {
    const double big = fmax(fabs(d), fabs(b));
    const int sc = -__builtin_amdgcn_frexp_exp(big);
    const double dn = ldexp(d, sc), bn = ldexp(b, sc);
    const double ih = inverse_root(dn * dn + bn * bn), c2 = 0.5 * (1.0 + fabs(dn) * ih), ic = inverse_root(c2);
    const bool turn = big > 1e-300;
    return make_double2(turn ? c2 * ic : 1.0, turn ? copysign(0.5 * ih * ic, d) * bn : 0.0);
}

// Eigen-decomposition of the symmetric k x k matrix G (LDS, row-major, k <= MZ)
// by cyclic Jacobi: theta ascending, Y the eigenvectors (columns).  Round-robin
// ordering: in each of K - 1 rounds (K = k rounded up to even) K / 2 disjoint
// pairs rotate at once; one player stays, the others turn.  S holds the matrix
// in seats, pair i in rows and columns 2 i and 2 i + 1: a lane rotates the 2 x 2
// block of two pairs from both sides and puts the results where the next round
// seats them, and the same for the rows of T, the vectors.  A sweep brings all
// back to their first seats.
// A round is two phases, the rotations and the blocks.  Up to 16 columns one
// wave does all, a block and two rows of a pair per lane, without a barrier;
// larger ones take the whole work-group.
// Seat strides are padded against bank conflicts.
template <int MZ>
__device__ void jacobi(double *G, double *Y, int k, double *theta, double *S) {
    constexpr int KP = (MZ + 1) & ~1, NP = KP / 2, LD = KP + 2;
    constexpr bool kWave = NP <= 8;
    constexpr int GB = kWave ? 1 : (NP * NP + kBoThreads - 1) / kBoThreads, STEP = kWave ? 64 : kBoThreads;
    constexpr int YB = (NP * KP + STEP - 1) / STEP;
    const int tid = threadIdx.x;
    double *T = S + KP * LD;
    __shared__ double2 cs[NP];
    const int K = (k + 1) & ~1, np = K / 2;
    auto fence = [] {
        if (kWave) wave_sync();
        else __syncthreads();
    };
    auto next = [&](int seat) {
        const int i = seat >> 1;
        if (np == 1 || seat == 0 || seat >= K) return seat;
        if (seat & 1) return i ? seat - 2 : 2;
        return i == np - 1 ? seat + 1 : seat + 2;
    };
    if (!kWave || tid < 64) {
        for (int idx = tid; idx < KP * KP; idx += STEP) {
            const int a = idx / KP, b = idx % KP;
            S[a * LD + b] = a < k && b < k ? G[a * k + b] : 0.0;
            T[a * LD + b] = a == b ? 1.0 : 0.0;
        }
        // blocks (gi, gj), rows yr of pair yi; unused ones turn seats of zeros
        int gi[GB], gj[GB], yi[YB], yr[YB];
#pragma unroll
        for (int q = 0; q < GB; ++q) {
            const int idx = tid + q * STEP;
            gi[q] = idx < NP * NP ? idx / NP : -1;
            gj[q] = idx % NP;
        }
#pragma unroll
        for (int q = 0; q < YB; ++q) {
            const int idx = tid + q * STEP;
            yi[q] = idx < NP * KP ? idx % NP : -1;
            yr[q] = idx / NP;
        }
        fence();
        for (int sweep = 0; sweep < 40; ++sweep) {
            double off = 0.0, dg = 0.0;              // (every wave for itself)
            for (int idx = tid & 63; idx < KP * KP; idx += 64) {
                const int a = idx / KP, b = idx % KP;
                const double g = S[a * LD + b];
                if (a == b) dg += g * g;
                else off += g * g;
            }
            off = wave_sum(off);
            dg = wave_sum(dg);
            if (!(off > 1e-30 * dg)) break;
            for (int r = 0; r < K - 1; ++r) {
                double2 bp[GB], bq[GB], y[YB];
                double2 turn;
                if (kWave || tid < NP) {
                    const int at = 2 * (kWave ? tid % NP : tid);
                    const double2 p = *reinterpret_cast<const double2 *>(S + at * (LD + 1));
                    turn = rotation(S[(at + 1) * (LD + 1)] - p.x, 2.0 * p.y);
                    cs[at / 2] = turn;
                }
#pragma unroll
                for (int q = 0; q < GB; ++q) {
                    if (!kWave && gi[q] < 0) continue;
                    bp[q] = *reinterpret_cast<const double2 *>(S + 2 * gi[q] * LD + 2 * gj[q]);
                    bq[q] = *reinterpret_cast<const double2 *>(S + (2 * gi[q] + 1) * LD + 2 * gj[q]);
                }
#pragma unroll
                for (int q = 0; q < YB; ++q) {
                    if (!kWave && yi[q] < 0) continue;
                    y[q] = *reinterpret_cast<const double2 *>(T + yr[q] * LD + 2 * yi[q]);
                }
                fence();
#pragma unroll
                for (int q = 0; q < GB; ++q) {
                    if (!kWave && gi[q] < 0) continue;
                    const double2 f = cs[gi[q]], g = kWave ? turn : cs[gj[q]];
                    const double2 hp = make_double2(f.x * bp[q].x - f.y * bq[q].x, f.x * bp[q].y - f.y * bq[q].y);
                    const double2 hq = make_double2(f.y * bp[q].x + f.x * bq[q].x, f.y * bp[q].y + f.x * bq[q].y);
                    const int i = next(2 * gi[q]) * LD, i1 = next(2 * gi[q] + 1) * LD;
                    const int j = next(2 * gj[q]), j1 = next(2 * gj[q] + 1);
                    S[i + j] = g.x * hp.x - g.y * hp.y;
                    S[i + j1] = g.y * hp.x + g.x * hp.y;
                    S[i1 + j] = g.x * hq.x - g.y * hq.y;
                    S[i1 + j1] = g.y * hq.x + g.x * hq.y;
                }
#pragma unroll
                for (int q = 0; q < YB; ++q) {
                    if (!kWave && yi[q] < 0) continue;
                    const double2 f = kWave ? turn : cs[yi[q]];
                    T[yr[q] * LD + next(2 * yi[q])] = f.x * y[q].x - f.y * y[q].y;
                    T[yr[q] * LD + next(2 * yi[q] + 1)] = f.y * y[q].x + f.x * y[q].y;
                }
                fence();
            }
        }
        // ascending order: each column to the place its eigenvalue ranks at
        for (int idx = tid; idx < k * k; idx += STEP) {
            const int row = idx / k, a = idx % k;
            const double e = S[a * LD + a];
            int at = 0;
            for (int b = 0; b < k; ++b) {
                const double o = S[b * LD + b];
                at += o < e || (o == e && b < a);
            }
            Y[row * k + at] = T[row * LD + a];
            if (row == 0) theta[at] = e;
        }
    }
    __syncthreads();
}

__device__ inline double unit_hash(unsigned long long x) {
    // splitmix64, then the top 53 bits as a double in [-1, 1)
    x += 0x9E3779B97F4A7C15ULL;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ULL;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBULL;
    x ^= x >> 31;
    return (double)(x >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// MZ: most columns of the basis (3 m), 15 (up to three states) or 36.
template <int LOG2N, int MZ>
__global__ void __launch_bounds__(kBoThreads, MZ <= 15 ? 2 : 1) k_bo_lobpcg(BoArgs A) {
    constexpr int n = 1 << LOG2N;
    constexpr int kTransform = LOG2N <= 10 ? kBoWaves * (n + n / 8) : n;
    constexpr int kTwiddles = LOG2N <= 10 ? n / 2 : 1;
    __shared__ double2 fb[kTransform];
    __shared__ double2 tw[kTwiddles];
    __shared__ double red[kBoWaves * kChunk];
    __shared__ double dots[kChunk];
    __shared__ double G[MZ * MZ];
    __shared__ double Y[MZ * MZ];
    __shared__ double theta[MZ], scl[MZ];
    __shared__ double2 seats2[((MZ + 1) & ~1) * (((MZ + 1) & ~1) + 2)];   // two matrices
    double *seats = reinterpret_cast<double *>(seats2);
    __shared__ int pos[MZ + 1];
    __shared__ double scratch[kChunk];
    __shared__ double2 part2[kBoWaves][128];
    double (*part)[256] = reinterpret_cast<double (*)[256]>(part2);
    const int j = blockIdx.x, tid = threadIdx.x, m = A.m;
    double *V = A.ws + (size_t)j * A.ws_stride;
    double *Z = V + n;
    double *HZ = Z + (size_t)kBoMaxZ * n;
    const double Rj = A.Rv[j];

    if (LOG2N <= 10)
        for (int e = tid; e < kTwiddles; e += kBoThreads) tw[e] = A.tw[e];
    // the clamped potential and its range on the grid
    double vmin = INFINITY, vmax = -INFINITY;
    bool finite = true;
    for (int e = tid; e < n; e += kBoThreads) {
        const double w = model_w(A.mp, A.r_min + e * A.h, Rj);
        V[e] = w;
        finite = finite && isfinite(w);
        vmin = fmin(vmin, w);
        vmax = fmax(vmax, w);
    }
    {
        double mm[kChunk] = {0};
        // range via sums of per-wave extrema: reduce max and -min with shuffles
        double a = vmax, b = -vmin;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            a = fmax(a, __shfl_xor(a, off));
            b = fmax(b, __shfl_xor(b, off));
        }
        const int lane = tid & 63, wave = tid >> 6;
        if (lane == 0) {
            red[wave * kChunk] = a;
            red[wave * kChunk + 1] = b;
            red[wave * kChunk + 2] = finite ? 0.0 : 1.0;
        }
        __syncthreads();
        if (tid == 0) {
            double mx = red[0], mn = red[1], bad = red[2];
            for (int w = 1; w < kBoWaves; ++w) {
                mx = fmax(mx, red[w * kChunk]);
                mn = fmax(mn, red[w * kChunk + 1]);
                bad += red[w * kChunk + 2];
            }
            scratch[0] = mx + mn;    // max W - min W
            scratch[1] = bad;
        }
        __syncthreads();
        (void)mm;
    }
    const double cshift = fmax(1.0, scratch[0]);
    if (scratch[1] != 0.0) {
        if (tid == 0) atomicOr(&A.flags[kFlagNonfinite], 1);
        return;
    }
    __syncthreads();

    // starting block: pseudo-random columns, smoothed by the preconditioner
    for (int c = 0; c < m; ++c)
        for (int e = tid; e < n; e += kBoThreads)
            Z[(size_t)c * n + e] = unit_hash(((unsigned long long)j << 40) ^ ((unsigned long long)c << 20) ^ e);
    __syncthreads();
    apply_columns<LOG2N>(A, Z, Z, m, V, false, cshift, fb, tw);
    int kz = orthonormalise<LOG2N, MZ>(Z, m, G, part, scl, pos);

    int it = 0;
    double worst = INFINITY;
    for (;; ++it) {
        // h_e on the whole basis, afresh, and the projected matrix
        apply_columns<LOG2N>(A, Z, HZ, kz, V, true, cshift, fb, tw);
        gram<LOG2N>(Z, HZ, kz, G, part);
        jacobi<MZ>(G, Y, kz, theta, seats);
        const int mk = min(m, kz);
        // in place of the basis: the Ritz block, its residuals, the new
        // directions (an element's columns are one thread's)
        const int cw = min(A.nwant, mk);
        double rr[kChunk] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int e = tid; e < n; e += kBoThreads) {
            double z[MZ], hz[MZ];
#pragma unroll
            for (int a = 0; a < MZ; ++a) {
                z[a] = a < kz ? Z[(size_t)a * n + e] : 0.0;
                hz[a] = a < kz ? HZ[(size_t)a * n + e] : 0.0;
            }
            for (int i = 0; i < mk; ++i) {
                double x = 0.0, hx = 0.0, p = 0.0;
#pragma unroll
                for (int a = 0; a < MZ; ++a) {
                    const double y = a < kz ? Y[a * kz + i] : 0.0;
                    x += z[a] * y;
                    hx += hz[a] * y;
                    if (a >= m) p += z[a] * y;
                }
                const double w = hx - theta[i] * x;
                Z[(size_t)i * n + e] = x;
                Z[(size_t)(mk + i) * n + e] = w;
                Z[(size_t)(2 * mk + i) * n + e] = p;
#pragma unroll
                for (int q = 0; q < kChunk; ++q)
                    if (q == i && q < cw) rr[q] += w * w;
            }
        }
        block_sums(rr, cw, red, dots);
        worst = 0.0;
        for (int q = 0; q < cw; ++q) worst = fmax(worst, sqrt(dots[q]));
        __syncthreads();
        if (!(worst > A.tol) || it + 1 >= A.max_iter || !isfinite(worst)) break;
        // new basis: the Ritz block, the preconditioned residuals, the directions
        apply_columns<LOG2N>(A, Z + (size_t)mk * n, Z + (size_t)mk * n, mk, V, false, cshift, fb, tw);
        kz = orthonormalise<LOG2N, MZ>(Z, it > 0 ? 3 * mk : 2 * mk, G, part, scl, pos);
    }
    const double *X = Z;

    // output: grid normalisation, largest-magnitude entry positive
    const double scale = 1.0 / sqrt(A.h);
    for (int i = 0; i < A.nwant; ++i) {
        const double *x = X + (size_t)i * n;
        double best = -1.0;
        int bidx = n;
        for (int e = tid; e < n; e += kBoThreads) {
            const double ax = fabs(x[e]);
            if (ax > best) {
                best = ax;
                bidx = e;
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off);
            const int oi = __shfl_xor(bidx, off);
            if (ob > best || (ob == best && oi < bidx)) {
                best = ob;
                bidx = oi;
            }
        }
        const int lane = tid & 63, wave = tid >> 6;
        if (lane == 0) {
            red[wave * 2] = best;
            red[wave * 2 + 1] = (double)bidx;
        }
        __syncthreads();
        if (tid == 0) {
            double bb = red[0];
            int bi = (int)red[1];
            for (int w = 1; w < kBoWaves; ++w) {
                const double ob = red[2 * w];
                const int oi = (int)red[2 * w + 1];
                if (ob > bb || (ob == bb && oi < bi)) {
                    bb = ob;
                    bi = oi;
                }
            }
            scratch[0] = x[bi] < 0.0 ? -scale : scale;
        }
        __syncthreads();
        const double sg = scratch[0];
        double *dst = A.states + ((size_t)j * A.nwant + i) * n;
        for (int e = tid; e < n; e += kBoThreads) dst[e] = sg * x[e];
        if (tid == 0) A.energies[(size_t)j * A.nwant + i] = theta[i];
        __syncthreads();
    }
    if (tid == 0) {
        A.iters[j] = it + 1;
        A.resid[j] = worst;
    }
}

template <int LOG2N>
void launch_bo_t(const BoArgs &a, int nv, hipStream_t s) {
    // the registers of a column set follow its size: 15 up to three states
    const auto kernel = 3 * a.m <= 15 ? k_bo_lobpcg<LOG2N, 15> : k_bo_lobpcg<LOG2N, kBoMaxZ>;
    hipLaunchKernelGGL(kernel, dim3(nv), dim3(kBoThreads), 0, s, a);
}

}  // namespace

}  // namespace icwf

// ---- C ABI (include/icwf_bo.h) -------------------------------------------------------------------

namespace {

bool bo_args_ok(const icwf_config *c, int32_t nv, int32_t ns, const char **why) {
    auto pow2 = [](int n) { return n > 0 && (n & (n - 1)) == 0; };
    if (!c) {
        *why = "config is NULL";
        return false;
    }
    if (!pow2(c->n_r) || c->n_r < 32 || c->n_r > 4096) {
        *why = "n_r must be a power of two in [32, 4096]";
        return false;
    }
    if (!(c->r_max > c->r_min) || !std::isfinite(c->r_min) || !std::isfinite(c->r_max) || !(c->m_r > 0) ||
        !std::isfinite(c->m_r)) {
        *why = "bad r box or m_r";
        return false;
    }
    if (c->model != ICWF_MODEL_SHIN_METIU && c->model != ICWF_MODEL_CAVITY) {
        *why = "unknown model";
        return false;
    }
    for (int i = 0; i < 8; ++i)
        if (!std::isfinite(c->model_params[i])) {
            *why = "model parameters must be finite";
            return false;
        }
    if (c->model == ICWF_MODEL_SHIN_METIU &&
        (!(c->model_params[1] > 0) || !(c->model_params[2] > 0) || !(c->model_params[3] > 0))) {
        *why = "Shin-Metiu softening lengths must be > 0";
        return false;
    }
    if (nv < 1 || nv > (1 << 20)) {
        *why = "n_values must be in [1, 2^20]";
        return false;
    }
    if (ns < 1 || ns > ICWF_BO_MAX_STATES || ns > c->n_r / 4) {
        *why = "n_states must be in [1, ICWF_BO_MAX_STATES] and at most n_r / 4";
        return false;
    }
    return true;
}

int block_size(int ns) { return ns + std::max(2, (ns + 1) / 2); }

// device layout: per-value slices, then the tables and the outputs
struct BoLayout {
    size_t slices, kin, tw, rvals, states, energies, iters, resid, flags, total;
};

BoLayout bo_layout(int n, int nv, int ns) {
    BoLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = (off + 255) & ~size_t(255);
        const size_t at = off;
        off += bytes;
        return at;
    };
    L.slices = take(sizeof(double) * icwf::bo_stride(n) * nv);
    L.kin = take(sizeof(double) * n);
    L.tw = take(sizeof(double2) * (n / 2));
    L.rvals = take(sizeof(double) * nv);
    L.states = take(sizeof(double) * (size_t)nv * ns * n);
    L.energies = take(sizeof(double) * (size_t)nv * ns);
    L.iters = take(sizeof(int32_t) * nv);
    L.resid = take(sizeof(double) * nv);
    L.flags = take(sizeof(int32_t) * icwf::kNumFlags);
    L.total = (off + 255) & ~size_t(255);
    return L;
}

}  // namespace

extern "C" {

size_t icwf_bo_workspace_bytes(const icwf_config *cfg, int32_t n_values, int32_t n_states) {
    const char *why = nullptr;
    if (!bo_args_ok(cfg, n_values, n_states, &why)) return 0;
    return bo_layout(cfg->n_r, n_values, n_states).total;
}

icwf_status icwf_bo_states(const icwf_config *cfg, const double *R_values, int32_t n_values, int32_t n_states,
                           double *states, double *energies, void *workspace, size_t ws_bytes, void *hip_stream,
                           icwf_bo_info *info) {
    const char *why = nullptr;
    if (!bo_args_ok(cfg, n_values, n_states, &why)) return icwf::set_create_error(ICWF_EINVAL, why);
    if (!R_values) return icwf::set_create_error(ICWF_EINVAL, "R_values is NULL");
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255))
        return icwf::set_create_error(ICWF_EINVAL, "workspace must be non-NULL and 256-byte aligned");
    for (int j = 0; j < n_values; ++j)
        if (!std::isfinite(R_values[j])) return icwf::set_create_error(ICWF_ENONFINITE, "non-finite R value");
    const int n = cfg->n_r, nv = n_values, ns = n_states;
    const BoLayout L = bo_layout(n, nv, ns);
    if (ws_bytes < L.total) return icwf::set_create_error(ICWF_ENOMEM, "workspace smaller than icwf_bo_workspace_bytes()");
    const double h = (cfg->r_max - cfg->r_min) / n;
    double hbound = 0.0;
    std::vector<double> kin(n);
    std::vector<double2> tw(n / 2);
    for (int k = 0; k < n; ++k) {
        const int kk = (k <= n / 2) ? k : k - n;
        const double kw = 2.0 * M_PI * kk / (n * h);
        kin[k] = kw * kw / (2.0 * cfg->m_r);
        hbound = std::max(hbound, kin[k]);
    }
    for (int k = 0; k < n / 2; ++k) tw[k] = make_double2(std::cos(-2.0 * M_PI * k / n), std::sin(-2.0 * M_PI * k / n));
    char *base = reinterpret_cast<char *>(workspace);
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    icwf::BoArgs a{};
    a.n = n;
    a.m = block_size(ns);
    a.nwant = ns;
    a.max_iter = (info && info->max_iter > 0) ? info->max_iter : 2000;
    // the bar: a few roundings of the largest kinetic term (the potential's
    // range is added where it is known to be larger, in the kernel's shift)
    a.tol = (info && info->tol > 0) ? info->tol : 32.0 * 2.220446049250313e-16 * std::max(1.0, hbound);
    a.r_min = cfg->r_min;
    a.h = h;
    a.mp.kind = cfg->model;
    for (int i = 0; i < 8; ++i) a.mp.p[i] = cfg->model_params[i];
    a.ws = reinterpret_cast<double *>(base + L.slices);
    a.ws_stride = icwf::bo_stride(n);
    a.kin = reinterpret_cast<const double *>(base + L.kin);
    a.tw = reinterpret_cast<const double2 *>(base + L.tw);
    a.states = reinterpret_cast<double *>(base + L.states);
    a.energies = reinterpret_cast<double *>(base + L.energies);
    a.iters = reinterpret_cast<int32_t *>(base + L.iters);
    a.resid = reinterpret_cast<double *>(base + L.resid);
    a.flags = reinterpret_cast<int32_t *>(base + L.flags);
    a.Rv = reinterpret_cast<const double *>(base + L.rvals);
    auto hip_ok = [&](hipError_t e, const char *what) {
        if (e == hipSuccess) return true;
        icwf::set_create_error(ICWF_EDEVICE, (std::string(what) + ": " + hipGetErrorString(e)).c_str());
        return false;
    };
    if (!hip_ok(hipMemcpyAsync(base + L.rvals, R_values, sizeof(double) * nv, hipMemcpyHostToDevice, st), "copy R") ||
        !hip_ok(hipMemcpyAsync(base + L.kin, kin.data(), sizeof(double) * n, hipMemcpyHostToDevice, st), "copy kin") ||
        !hip_ok(hipMemcpyAsync(base + L.tw, tw.data(), sizeof(double2) * (n / 2), hipMemcpyHostToDevice, st), "copy tw") ||
        !hip_ok(hipMemsetAsync(base + L.flags, 0, sizeof(int32_t) * icwf::kNumFlags, st), "clear flags"))
        return ICWF_EDEVICE;
    switch (n) {
        case 32: icwf::launch_bo_t<5>(a, nv, st); break;
        case 64: icwf::launch_bo_t<6>(a, nv, st); break;
        case 128: icwf::launch_bo_t<7>(a, nv, st); break;
        case 256: icwf::launch_bo_t<8>(a, nv, st); break;
        case 512: icwf::launch_bo_t<9>(a, nv, st); break;
        case 1024: icwf::launch_bo_t<10>(a, nv, st); break;
        case 2048: icwf::launch_bo_t<11>(a, nv, st); break;
        default: icwf::launch_bo_t<12>(a, nv, st); break;
    }
    if (!hip_ok(hipGetLastError(), "launch")) return ICWF_EDEVICE;
    std::vector<int32_t> iters(nv), flags(icwf::kNumFlags);
    std::vector<double> resid(nv);
    if ((states && !hip_ok(hipMemcpyAsync(states, base + L.states, sizeof(double) * (size_t)nv * ns * n,
                                          hipMemcpyDeviceToHost, st), "copy states")) ||
        (energies && !hip_ok(hipMemcpyAsync(energies, base + L.energies, sizeof(double) * (size_t)nv * ns,
                                            hipMemcpyDeviceToHost, st), "copy energies")) ||
        !hip_ok(hipMemcpyAsync(iters.data(), base + L.iters, sizeof(int32_t) * nv, hipMemcpyDeviceToHost, st), "copy iters") ||
        !hip_ok(hipMemcpyAsync(resid.data(), base + L.resid, sizeof(double) * nv, hipMemcpyDeviceToHost, st), "copy resid") ||
        !hip_ok(hipMemcpyAsync(flags.data(), base + L.flags, sizeof(int32_t) * icwf::kNumFlags, hipMemcpyDeviceToHost, st),
                "copy flags") ||
        !hip_ok(hipStreamSynchronize(st), "synchronise"))
        return ICWF_EDEVICE;
    if (flags[icwf::kFlagNonfinite]) return icwf::set_create_error(ICWF_ENONFINITE, "the model is singular on the grid");
    int worst_it = 0, unconv = 0;
    double worst_res = 0.0;
    for (int j = 0; j < nv; ++j) {
        worst_it = std::max(worst_it, iters[j]);
        worst_res = std::max(worst_res, resid[j]);
        if (!(resid[j] <= a.tol)) ++unconv;
    }
    if (info) {
        info->iterations = worst_it;
        info->max_residual = worst_res;
        info->unconverged = unconv;
    }
    if (unconv) return icwf::set_create_error(ICWF_ESOLVE, "some R values did not reach the residual bar");
    return ICWF_OK;
}

}  // extern "C"
