// The single-species matrices of Eq. 9 (9a, and the conditioned factors of
// 9c-9d) and the two-body contraction of Eq. 9b.
//
// Single species (k_zgemm, k_zgemm_split): out[b][a] = h sum_k conj(X[b][k]) Y[a][k] for the
// pairs (X, Y) = (psi1, psi1) -> S1, (psi1, G1) -> E1, (psi2, psi2) -> S2,
// (psi2, G2) -> E2, where G is the ket weighted by the coupling potential at
// the ket's own trajectory: G1^a_i = W_c(r_i, R^a) psi1^a_i, G2^a_j =
// W_c(r^a, R_j) psi2^a_j.  Complex = four real FP64 MFMA products.
//
// Two-body (k_wc_sep): where W_c is, to its rounding, a short sum of products
// u_k(r) v_k(R), Wc[b][a] = hr hR sum_k (sum_i conj(psi1^b_i) psi1^a_i u_k(r_i))
// (sum_j conj(psi2^b_j) psi2^a_j v_k(R_j)).
//
// Two-body without such a sum (k_wc): Wc[b][a] = hr hR sum_j conj(psi2^b_j) psi2^a_j
//                             sum_i conj(psi1^b_i) psi1^a_i W_c(r_i, R_j)
// for b <= a (the matrix is Hermitian).  The inner i-sum is a real GEMM whose
// A operand, the pair product P1 = conj(psi1^b) psi1^a, is generated in
// registers (never stored) and whose B operand is the W_c table; the j-sum
// with the pair product P2 is fused into the epilogue of every 32-wide j
// tile.  FP64: v_mfma_f64_16x16x4 throughout.  Mixed: P1 and the table in
// FP32 on v_mfma_f32_16x16x4 with FP32 accumulation over i inside a j tile,
// the epilogue and the sum over j tiles in FP64.
#include <algorithm>

#include "icwf_plan.hpp"

namespace icwf {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));

__device__ inline dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline flt4 mfma(float a, float b, flt4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- conditioned kets
// Both species in one launch: the first `blocks1` work-groups species 1.
struct CondSpecies {
    const double2 *psi;
    const double *cond_a, *cond_b;
    double2 *Ga, *Gb;
    int n;
    double x_min, h;
};

__global__ void k_cond_kets(CondSpecies s1, CondSpecies s2, unsigned blocks1, ModelParams mp, int Np,
                            const int32_t *__restrict__ flags, const long long *__restrict__ zoff,
                            const ModelParams *__restrict__ mpd) {
    const long long zo_ = batch_offset(zoff);
    flags = zshift(flags, zo_);
    if (zoff) mp = *zshift(mpd, zo_);

    if (flags[kFlagHalt]) return;
    const bool first = blockIdx.x < blocks1;
    const CondSpecies &c = first ? s1 : s2;
    const size_t idx = (size_t)(first ? blockIdx.x : blockIdx.x - blocks1) * blockDim.x + threadIdx.x;
    if (idx >= (size_t)Np * c.n) return;
    const int a = (int)(idx / c.n);
    const int i = (int)(idx - (size_t)a * c.n);
    const double x = c.x_min + i * c.h;
    const double2 p = zshift(c.psi, zo_)[idx];
    const double xa = zshift(c.cond_a, zo_)[a], xb = zshift(c.cond_b, zo_)[a];
    const double wa = first ? model_wc(mp, x, xa) : model_wc(mp, xa, x);
    zshift(c.Ga, zo_)[idx] = cscale(p, wa);
    if (c.Gb) {
        const double wb = first ? model_wc(mp, x, xb) : model_wc(mp, xb, x);
        zshift(c.Gb, zo_)[idx] = cscale(p, wb);
    }
}

// ---------------------------------------------------------------- batched conj-NT complex GEMM
struct ZBatch {
    const double2 *X[6];
    const double2 *Y[6];
    double2 *out[6];
    int K[6];
    double scale[6];
    double w0[6], w1[6];     // weight w0 + w1 k of the reduction's point k (weighted == 0: none)
    int weighted[6];
};

// Work-group of 4 waves per 64 x 64 output tile, wave w on the 32 x 32
// quarter (rows 32 (w / 2), columns 32 (w % 2)) as 2 x 2 MFMA fragments with
// rows = b, columns = a, k the reduction index; lane l supplies
// A = X[b][k] and B = Y[a][k] with b, a = l % 16 of the fragment and
// k = l / 16 of the k step.  The 64 rows of X and of Y of a 16-wide k chunk are
// staged in LDS (two buffers: the coalesced global loads of chunk c + 1 are in
// flight while the matrix cores work on chunk c).  Hermitian outputs compute
// the upper tiles and write the lower ones as their conjugates.
constexpr int kZT = 64, kZKC = 16, kZLD = kZKC + 1;

// Entry z (wave-uniform) of a kernel-argument array, by selects: an indexed
// access would copy the whole argument struct to scratch.
template <typename T>
__device__ inline T zpick(const T (&a)[6], int z) {
    T r = a[0];
    r = z == 1 ? a[1] : r;
    r = z == 2 ? a[2] : r;
    r = z == 3 ? a[3] : r;
    r = z == 4 ? a[4] : r;
    r = z == 5 ? a[5] : r;
    return r;
}

__device__ inline void triangle_tile(int t, int *tb, int *ta) {
    int a = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((a + 1) * (a + 2) / 2 <= t) ++a;
    while (a * (a + 1) / 2 > t) --a;
    *ta = a;
    *tb = t - a * (a + 1) / 2;
}

// Output tile (bt, at) of a launch over nt x nt tiles: by rows, or of a
// Hermitian output its upper tiles one after the other (a run of work-groups
// goes round the XCDs: by rows, the XCDs of the last columns had a fifth more
// than their share).  False: none left.
__device__ inline bool zgemm_tile(int t, int nt, bool herm, int *bt, int *at) {
    if (!herm) {
        *bt = t / nt;
        *at = t - *bt * nt;
        return true;
    }
    if (t >= nt * (nt + 1) / 2) return false;
    triangle_tile(t, bt, at);
    return true;
}

template <bool BATCHED>
__global__ void __launch_bounds__(256, 2) k_zgemm(ZBatch zb, int Np, const int32_t *__restrict__ flags, int zcnt,
                                                  const long long *__restrict__ zoff) {
    // grid z: zcnt products of each simulation of the launch
    const int sim = BATCHED ? blockIdx.z / zcnt : 0, z = blockIdx.z - sim * zcnt;
    const long long zo_ = BATCHED ? batch_offset(zoff, sim) : 0;
    flags = zshift(flags, zo_);
    if (flags[kFlagHalt]) return;
    const double2 *__restrict__ X = zshift(zpick(zb.X, z), zo_);
    const double2 *__restrict__ Y = zshift(zpick(zb.Y, z), zo_);
    const bool herm = X == Y;   // the output is Hermitian: upper tiles only
    int bt, at;
    if (!zgemm_tile(blockIdx.x, Np / kZT, herm, &bt, &at)) return;
    __shared__ double2 sX[2][kZT][kZLD];
    __shared__ double2 sY[2][kZT][kZLD];
    const int K = zpick(zb.K, z);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int row = lane & 15, quarter = lane >> 4;
    const int b0 = bt * kZT, a0 = at * kZT;
    const int wb = 32 * (wave >> 1), wa = 32 * (wave & 1);
    dbl4 re[2][2], im[2][2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            re[f][g] = dbl4{0, 0, 0, 0};
            im[f][g] = dbl4{0, 0, 0, 0};
        }
    // staging: element e = t + 256 m of a chunk is row e / 16, k e % 16
    const int srow = t >> 4, sk = t & 15;
    const double2 *xs = X + (size_t)(b0 + srow) * K + sk;   // rows srow + 16 m
    const double2 *ys = Y + (size_t)(a0 + srow) * K + sk;
    const size_t rstep = (size_t)16 * K;
    const bool weighted = zpick(zb.weighted, z) != 0;
    const double w0 = zpick(zb.w0, z), w1 = zpick(zb.w1, z);
    double2 rx0 = xs[0], rx1 = xs[rstep], rx2 = xs[2 * rstep], rx3 = xs[3 * rstep];
    double2 ry0 = ys[0], ry1 = ys[rstep], ry2 = ys[2 * rstep], ry3 = ys[3 * rstep];
    auto weigh = [&](int k0) __attribute__((always_inline)) {
        if (!weighted) return;
        const double w = w0 + w1 * (k0 + sk);
        ry0 = cscale(ry0, w);
        ry1 = cscale(ry1, w);
        ry2 = cscale(ry2, w);
        ry3 = cscale(ry3, w);
    };
    weigh(0);
    sX[0][srow][sk] = rx0;
    sX[0][srow + 16][sk] = rx1;
    sX[0][srow + 32][sk] = rx2;
    sX[0][srow + 48][sk] = rx3;
    sY[0][srow][sk] = ry0;
    sY[0][srow + 16][sk] = ry1;
    sY[0][srow + 32][sk] = ry2;
    sY[0][srow + 48][sk] = ry3;
    __syncthreads();
    const int nch = K / kZKC;
    for (int ch = 0; ch < nch; ++ch) {
        const int buf = ch & 1;
        const bool more = ch + 1 < nch;
        if (more) {
            const int k0 = (ch + 1) * kZKC;
            rx0 = xs[k0];
            rx1 = xs[rstep + k0];
            rx2 = xs[2 * rstep + k0];
            rx3 = xs[3 * rstep + k0];
            ry0 = ys[k0];
            ry1 = ys[rstep + k0];
            ry2 = ys[2 * rstep + k0];
            ry3 = ys[3 * rstep + k0];
        }
#pragma unroll
        for (int s4 = 0; s4 < kZKC / 4; ++s4) {
            const int kk = 4 * s4 + quarter;
            double2 xv[2], yv[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                xv[f] = sX[buf][wb + 16 * f + row][kk];
                yv[f] = sY[buf][wa + 16 * f + row][kk];
            }
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    // conj(x) y = (xr yr + xi yi) + i (xr yi - xi yr)
                    re[f][g] = mfma(xv[f].x, yv[g].x, re[f][g]);
                    re[f][g] = mfma(xv[f].y, yv[g].y, re[f][g]);
                    im[f][g] = mfma(xv[f].x, yv[g].y, im[f][g]);
                    im[f][g] = mfma(-xv[f].y, yv[g].x, im[f][g]);
                }
        }
        if (more) {
            const int nb = buf ^ 1;
            weigh((ch + 1) * kZKC);
            sX[nb][srow][sk] = rx0;
            sX[nb][srow + 16][sk] = rx1;
            sX[nb][srow + 32][sk] = rx2;
            sX[nb][srow + 48][sk] = rx3;
            sY[nb][srow][sk] = ry0;
            sY[nb][srow + 16][sk] = ry1;
            sY[nb][srow + 32][sk] = ry2;
            sY[nb][srow + 48][sk] = ry3;
        }
        __syncthreads();
    }
    const double sc = zpick(zb.scale, z);
    double2 *out = zshift(zpick(zb.out, z), zo_);
    const bool mirror = herm && bt < at;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = b0 + wb + 16 * f + mfma_row_f64(lane, v);
                const int a = a0 + wa + 16 * g + row;
                const double2 o = make_double2(sc * re[f][g][v], sc * im[f][g][v]);
                out[(size_t)b * Np + a] = o;
                if (mirror) out[(size_t)a * Np + b] = cconj(o);
            }
}

// The same products where 64 x 64 tiles are too few for the device: a
// work-group per 16 F x 16 F tile, its four waves taking the steps of the
// reduction (16 points each) in turn, operands straight from global memory one
// step ahead, four consecutive points per lane; the four partial tiles meet in
// LDS.  The sums do not depend on F.
template <int F, bool BATCHED>
__global__ void __launch_bounds__(256, 2) k_zgemm_split(ZBatch zb, int Np, const int32_t *__restrict__ flags, int zcnt,
                                                        const long long *__restrict__ zoff) {
    const int sim = BATCHED ? blockIdx.z / zcnt : 0, z = blockIdx.z - sim * zcnt;
    const long long zo_ = BATCHED ? batch_offset(zoff, sim) : 0;
    flags = zshift(flags, zo_);
    if (flags[kFlagHalt]) return;
    const double2 *X = zshift(zpick(zb.X, z), zo_);
    const double2 *Y = zshift(zpick(zb.Y, z), zo_);
    const bool herm = X == Y;   // the output is Hermitian: upper tiles only
    constexpr int W = 4, T = 16 * F, EP = 4, ITEMS = 4 * F * F;
    int bt, at;
    if (!zgemm_tile(blockIdx.x, Np / T, herm, &bt, &at)) return;
    bt = __builtin_amdgcn_readfirstlane(bt);
    at = __builtin_amdgcn_readfirstlane(at);
    __shared__ double2 red[W][ITEMS][64];
    const int K = zpick(zb.K, z);
    const int t = threadIdx.x, lane = t & 63, row = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int b0 = bt * T, a0 = at * T;
    dbl4 re[F][F], im[F][F];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int g = 0; g < F; ++g) {
            re[f][g] = dbl4{0, 0, 0, 0};
            im[f][g] = dbl4{0, 0, 0, 0};
        }
    const int count = (K / (4 * EP) - wave + W - 1) / W;     // steps of this wave
    if (count > 0) {
        constexpr uint32_t kStep = 64u * EP;                 // bytes of a row per step
        const gchar *xat = opaque(X + (size_t)b0 * K) + (size_t)wave * kStep;
        const gchar *yat = opaque(Y + (size_t)a0 * K) + (size_t)wave * kStep;
        const uint32_t off = (uint32_t)row * K * 16u + quarter * 16u * EP, frow = 256u * K;
        dbl2 x[F][EP], y[F][EP];
        auto load = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    x[f][e] = *reinterpret_cast<const gdouble2 *>(xat + (size_t)f * frow + off + 16u * e);
                    y[f][e] = *reinterpret_cast<const gdouble2 *>(yat + (size_t)f * frow + off + 16u * e);
                }
            pin_loads();
        };
        load();
        const bool weighted = zpick(zb.weighted, z) != 0;
        const double w0 = zpick(zb.w0, z), w1 = zpick(zb.w1, z);
        int k = 4 * EP * wave + EP * quarter;
        for (int s = 0; s < count; ++s) {
            dbl2 xc[F][EP], yc[F][EP];
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    xc[f][e] = x[f][e];
                    yc[f][e] = y[f][e];
                }
            if (weighted) {
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    const double w = w0 + w1 * (k + e);
#pragma unroll
                    for (int f = 0; f < F; ++f) yc[f][e] *= w;
                }
                k += 4 * EP * W;
            }
            const size_t st = s + 1 < count ? W * kStep : 0;  // the last step loads its own operands again (never used)
            xat += st;
            yat += st;
            load();
#pragma unroll
            for (int e = 0; e < EP; ++e)
#pragma unroll
                for (int f = 0; f < F; ++f)
#pragma unroll
                    for (int g = 0; g < F; ++g) {
                        // conj(x) y = (xr yr + xi yi) + i (xr yi - xi yr)
                        re[f][g] = mfma(xc[f][e].x, yc[g][e].x, re[f][g]);
                        im[f][g] = mfma(xc[f][e].x, yc[g][e].y, im[f][g]);
                        re[f][g] = mfma(xc[f][e].y, yc[g][e].y, re[f][g]);
                        im[f][g] = mfma(-xc[f][e].y, yc[g][e].x, im[f][g]);
                    }
        }
    }
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int g = 0; g < F; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][(f * F + g) * 4 + v][lane] = make_double2(re[f][g][v], im[f][g][v]);
    __syncthreads();
    const double sc = zpick(zb.scale, z);
    double2 *out = zshift(zpick(zb.out, z), zo_);
#pragma unroll
    for (int q = 0; q < ITEMS / W; ++q) {
        const int it = q * W + wave, v = it & 3, g = (it >> 2) % F, f = (it >> 2) / F;
        // Hermitian: by fragments of 16, so that the entries below the
        // diagonal are the conjugates of those above it whatever F is
        if (herm && bt * F + f > at * F + g) continue;
        const bool mirror = herm && bt * F + f < at * F + g;
        const double2 o = cscale(cadd(cadd(red[0][it][lane], red[1][it][lane]), cadd(red[2][it][lane], red[3][it][lane])), sc);
        const int b = b0 + 16 * f + mfma_row_f64(lane, v), a = a0 + 16 * g + row;
        out[(size_t)b * Np + a] = o;
        if (mirror) out[(size_t)a * Np + b] = cconj(o);
    }
}

// Up to 768 padded trajectories (alone or in a batch, which has to give the
// same sums) the split kernel, on tiles of 16 while those of 32 leave compute
// units idle.  Six products of one simulation at 512 x 256, tiles of 16, 32
// and the 64 of k_zgemm: N = 64, 21, 30 and 83 us; N = 250, 51, 48 and 86;
// N = 500, 164, 102 and 142; N = 1024, 287, 179 and 176.
static void launch_zgemm(const Dims &d, const ZBatch &zb, int c, const int32_t *flags, hipStream_t s) {
    const int Np = padded(d.N);
    auto go = [&](auto kernel, int T) {
        hipLaunchKernelGGL(kernel, dim3((Np / T) * (Np / T), 1, c * d.batch), dim3(256), 0, s, zb, Np, flags, c,
                           d.zoff);
    };
    if (Np > 768) go(d.zoff ? k_zgemm<true> : k_zgemm<false>, kZT);
    else if ((long long)c * d.batch * (Np / 32) * (Np / 32) <= 256)
        go(d.zoff ? k_zgemm_split<1, true> : k_zgemm_split<1, false>, 16);
    else go(d.zoff ? k_zgemm_split<2, true> : k_zgemm_split<2, false>, 32);
}

// ---------------------------------------------------------------- two-body contraction
template <typename T>
struct WcTraits;
template <>
struct WcTraits<double> {
    typedef dbl4 acc4;
    typedef double2 cplx;   // psi1 operand
};
template <>
struct WcTraits<float> {
    typedef flt4 acc4;
    typedef float2 cplx;    // FP32 copy of psi1 (written by the propagation)
};

// Block = 4 waves on a 16 (b) x 16 (a) tile of the upper triangle (tile
// index tb <= ta); wave w owns b = b_tile + 4w .. 4w + 3 against all 16 a.
// MFMA rows are a, columns are j, k is i; lane l supplies A = P1(b, a0 + l%16,
// i) and B = W_c(i, j0 + l%16) with i in the quarter l/16 of the current i
// chunk.  Each (j tile, i chunk) step stages the 32 psi1 rows of the tile and
// the W_c chunk in LDS (two buffers): the loads of step s + 1 are in flight
// while the matrix cores work on step s.  The j-sums of the epilogue go to
// LDS once per j tile.
//
// The staging goes straight from global memory into LDS (16 bytes per lane
// and load; no staging registers, four times fewer load instructions than
// 4-byte loads).  A load fills 64 consecutive 16-byte slots of a padded
// buffer: psi1 rows of 32 slots plus a pad slot (528 bytes), W_c rows of
// 16 slots plus one (FP64) or plus four (FP32), so that the operand reads
// stay free of bank conflicts; a lane whose slot is padding, or past the tile,
// loads an in-bounds entry that is never read.  FP32 takes the i of a chunk
// interleaved over the four lane quarters (i = 4 s + quarter at quad s), FP64
// in four consecutive runs (i = QS quarter + s).  FP32 accumulators take half
// the registers of FP64 ones, so its j tiles are 64 wide (each pair product
// feeds eight matrix products instead of four).
template <typename T>
struct WcChunk {
    static constexpr int KC = sizeof(T) == 8 ? 32 : 64;   // i per chunk (LDS budget: 2 blocks / CU)
    static constexpr int JT = sizeof(T) == 8 ? 32 : 64;   // j per tile
    static constexpr int JF = JT / 16;                    // 16-wide j fragments
    static constexpr int CPLX = 2 * sizeof(T);            // bytes of a psi1 entry
    static constexpr int LDA = 528 / CPLX;                 // padded psi1 row (entries): 33 slots
    static constexpr int LDW = sizeof(T) == 8 ? 34 : 80;   // padded W_c chunk row (entries)
    static constexpr bool INTERLEAVE = sizeof(T) == 4;
    static constexpr int ALOADS = (32 * 33 + 63) / 64;                 // loads per psi1 buffer
    static constexpr int AROWS = (64 * 16 * ALOADS + 527) / 528;       // rows the buffer holds
    static constexpr int WSLOTS = LDW * sizeof(T) / 16;                // slots per W_c row
    static constexpr int WDATA = JT * sizeof(T) / 16;                  // of which data
    static constexpr int WLOADS = (KC * WSLOTS + 63) / 64;
    static constexpr int WROWS = (64 * 16 * WLOADS + LDW * (int)sizeof(T) - 1) / (LDW * (int)sizeof(T));
};

typedef __attribute__((address_space(3))) void lds_void;

template <typename T, bool BATCHED>
__global__ void __launch_bounds__(256, 2) k_wc(const typename WcTraits<T>::cplx *__restrict__ psi1,
                                               const double2 *__restrict__ psi2,
                                               const T *__restrict__ wtab, int nr, int nR, double scale,
                                               double2 *__restrict__ Wc, int Np, int accumulate,
                                               int ntiles, int spq, int nparts, int32_t *__restrict__ queue,
                                               const int32_t *__restrict__ order, double2 *__restrict__ part,
                                               const int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = BATCHED ? batch_offset(zoff) : 0;
    psi1 = zshift(psi1, zo_);
    psi2 = zshift(psi2, zo_);
    wtab = zshift(wtab, zo_);
    Wc = zshift(Wc, zo_);
    queue = zshift(queue, zo_);
    order = zshift(order, zo_);
    part = zshift(part, zo_);
    flags = zshift(flags, zo_);

    typedef typename WcTraits<T>::acc4 acc4;
    typedef typename WcTraits<T>::cplx C2;
    typedef WcChunk<T> CK;
    constexpr int KC = CK::KC, LDA = CK::LDA, LDW = CK::LDW, QS = KC / 4, JT = CK::JT, JF = CK::JF;
    constexpr int AROWS = CK::AROWS, WROWS = CK::WROWS;
    // two staging buffers as separate arrays: the compiler can then tell the
    // reads of one from the direct loads into the other
    __shared__ __align__(16) C2 sA0[AROWS][LDA], sA1[AROWS][LDA];   // rows 0..15: a rows, 16..31: b rows
    __shared__ __align__(16) T sW0[WROWS][LDW], sW1[WROWS][LDW];
    __shared__ double2 wl[4][4][16];   // [wave][b][a] block partial of Wc
    __shared__ int s_unit, s_queue, s_done;
    // persistent: the work-group takes upper-triangle tiles from queues until
    // none is left (fewer work-groups than CU slots leaves room for work on
    // another stream).  Queue q hands out the q-th eighth of the tile order
    // (blocks of neighbouring tiles); a work-group takes from the queue of
    // its own XCD first, then from the others.  The last spq tiles of each
    // queue come as nparts units each, one per nparts-th of the j tiles, so
    // that the final round ends with small pieces of work: each unit leaves
    // its partial sum in `part`, and the unit that completes last adds them
    // in part order (whatever the order of completion) and writes the tile.
    auto queue_range = [&](int q, int *lo, int *nfull, int *nsp) {
        *lo = (int)((long long)q * ntiles / kWcQueues);
        const int n = (int)((long long)(q + 1) * ntiles / kWcQueues) - *lo;
        *nsp = n < spq ? n : spq;
        *nfull = n - *nsp;
    };
    // the XCD this work-group runs on (its queue; any value is correct)
    const int xcd = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & (kWcQueues - 1);   // HW_REG_XCC_ID
    for (;;) {
        if (threadIdx.x == 0) {
            // a halt ends the work-group as a whole, here and nowhere else: the
            // factorisation beside this launch may raise it at any time, and
            // waves that each read it for themselves would part company
            // (read with the queue, not ahead of it)
            const bool halt = halted(flags);
            int got = -1, gq = 0;
            for (int o = 0; o < kWcQueues && got < 0; ++o) {
                const int q = (xcd + o) & (kWcQueues - 1);
                int lo, nf, ns;
                queue_range(q, &lo, &nf, &ns);
                const int units = nf + ns * nparts;
                if (__hip_atomic_load(&queue[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= units) continue;
                const int k = atomicAdd(&queue[q], 1);
                if (k < units) {
                    got = k;
                    gq = q;
                }
            }
            s_unit = halt ? -1 : got;
            s_queue = gq;
        }
        __syncthreads();
        const int unit = s_unit, q = s_queue;
        __syncthreads();
        if (unit < 0) break;
        int lo, nfull, nsp;
        queue_range(q, &lo, &nfull, &nsp);
        int pos = lo + unit, half = -1, slot = 0;   // half: this unit's part of a split tile
        if (unit >= nfull) {
            const int j = unit - nfull;
            pos = lo + nfull + j / nparts;
            half = j - (j / nparts) * nparts;
            slot = q * spq + j / nparts;
        }
        int tb, ta;
        triangle_tile(order[pos], &tb, &ta);

        const int t = threadIdx.x;
        const int lane = t & 63, wave = t >> 6;
        const int row = lane & 15, quarter = lane >> 4;
        const int a_base = ta * 16;
        const int b_tile = tb * 16;
        const int b_base = b_tile + 4 * wave;

        for (int e = lane; e < 64; e += 64) wl[wave][e >> 4][e & 15] = make_double2(0, 0);

        const int nchunk = nr / KC, ntj = half < 0 ? nR / JT : nR / JT / nparts, nsteps = nchunk * ntj;
        const int jt0 = half > 0 ? half * ntj : 0;   // first j tile of this unit
        typedef C2 ATile[AROWS][LDA];
        typedef T WTile[WROWS][LDW];
        // tile row rr of the staging buffers: a rows first, then b rows
        auto tile_row = [&](int rr) { return rr < 16 ? a_base + rr : b_tile + rr - 16; };
        // one step's operands into (A, W): 64 slots per load, load m of
        // the buffer by wave m mod 4; slot -> (row, slot in the row)
        auto fetch = [&](int step, ATile &A, WTile &W) __attribute__((always_inline)) {
            const int jl = step / nchunk, ch = step - jl * nchunk, jt = jt0 + jl;
            const int i0 = ch * KC, j0 = jt * JT;
            const float4 *src_a = reinterpret_cast<const float4 *>(psi1);
            const float4 *src_w = reinterpret_cast<const float4 *>(wtab);
    #pragma unroll
            for (int m = 0; m < (CK::ALOADS + 3) / 4; ++m) {
                const int blk = 4 * m + wave;
                if (blk < CK::ALOADS) {
                    const int slot = 64 * blk + lane;
                    int rr = slot / 33, c = slot - 33 * rr;
                    if (rr >= 32) rr = 31;
                    if (c >= 32) c = 0;
                    // 16-byte units: a psi1 row is nr entries of CPLX bytes
                    const uint32_t off = (uint32_t)(((size_t)tile_row(rr) * nr + i0) * CK::CPLX / 16 + c);
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const float *>(src_a + off),
                                                     (lds_void *)(reinterpret_cast<char *>(&A[0][0]) + 1024 * blk), 16,
                                                     0, 0);
                }
            }
    #pragma unroll
            for (int m = 0; m < (CK::WLOADS + 3) / 4; ++m) {
                const int blk = 4 * m + wave;
                if (blk < CK::WLOADS) {
                    const int slot = 64 * blk + lane;
                    int ii = slot / CK::WSLOTS, c = slot - CK::WSLOTS * ii;
                    if (ii >= KC) ii = KC - 1;
                    if (c >= CK::WDATA) c = 0;
                    const uint32_t off = (uint32_t)(((size_t)(i0 + ii) * nR + j0) * sizeof(T) / 16 + c);
                    __builtin_amdgcn_global_load_lds(reinterpret_cast<const float *>(src_w + off),
                                                     (lds_void *)(reinterpret_cast<char *>(&W[0][0]) + 1024 * blk), 16,
                                                     0, 0);
                }
            }
        };
        // the loads have landed (vmcnt(0))
        auto stash = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0x0f70); };

        acc4 acc[4][2][JF];   // [b][re/im][j fragment]
        // one (j tile, i chunk) step on the buffers (A, W); the next step's
        // operands are staged into (An, Wn) meanwhile
        auto body = [&](int step, ATile &A, WTile &W, ATile &An, WTile &Wn) __attribute__((always_inline)) {
            const int jl = step / nchunk, ch = step - jl * nchunk, jt = jt0 + jl;
            if (ch == 0) {
    #pragma unroll
                for (int bb = 0; bb < 4; ++bb)
    #pragma unroll
                    for (int c = 0; c < 2; ++c)
    #pragma unroll
                        for (int jf = 0; jf < JF; ++jf) acc[bb][c][jf] = acc4{0, 0, 0, 0};
            }
            if (step + 1 < nsteps) fetch(step + 1, An, Wn);
            // operands of i-quad s + 1 are read from LDS while the matrix
            // cores work on quad s
            C2 xa, xb[4];
            T w[JF];
            auto operands = [&](int s, C2 &oa, C2 (&ob)[4], T (&ow)[JF]) __attribute__((always_inline)) {
                const int col = CK::INTERLEAVE ? 4 * s + quarter : quarter * QS + s;
                oa = A[row][col];
    #pragma unroll
                for (int jf = 0; jf < JF; ++jf) ow[jf] = W[col][16 * jf + row];
    #pragma unroll
                for (int bb = 0; bb < 4; ++bb) ob[bb] = A[16 + 4 * wave + bb][col];
            };
            operands(0, xa, xb, w);
    #pragma unroll
            for (int s = 0; s < QS; ++s) {
                C2 na, nb[4];
                T nw[JF];
                if (s + 1 < QS) operands(s + 1, na, nb, nw);
    #pragma unroll
                for (int bb = 0; bb < 4; ++bb) {
                    const C2 p = cmulc(xb[bb], xa);   // conj(psi1^b_i) psi1^a_i
                    const T pr = (T)p.x, pi = (T)p.y;
    #pragma unroll
                    for (int jf = 0; jf < JF; ++jf) {
                        acc[bb][0][jf] = mfma(pr, w[jf], acc[bb][0][jf]);
                        acc[bb][1][jf] = mfma(pi, w[jf], acc[bb][1][jf]);
                    }
                }
                if (s + 1 < QS) {
                    xa = na;
    #pragma unroll
                    for (int jf = 0; jf < JF; ++jf) w[jf] = nw[jf];
    #pragma unroll
                    for (int bb = 0; bb < 4; ++bb) xb[bb] = nb[bb];
                }
            }
            // keep the wait for the next step's operands after the matrix
            // products
            __builtin_amdgcn_sched_barrier(0);
            if (step + 1 < nsteps) stash();
            if (ch == nchunk - 1) {
                // epilogue: lane holds T(b, a = a_base + mfma_row(T, lane, v), j = j0 + 16 jf + row);
                // multiply by P2 = conj(psi2^b_j) psi2^a_j and sum over the 16 j of the fragment
                const int j0 = jt * JT;
                auto p2 = [&](int rr, int jj) { return psi2[(size_t)tile_row(rr) * nR + j0 + jj]; };
                // the a-row entries are loaded once for all b (two j
                // fragments), or again for each b (four: their registers are
                // needed for the accumulators)
                constexpr bool HOIST = JF <= 2;
                double2 p2a[HOIST ? JF : 1][4];
                if constexpr (HOIST) {
    #pragma unroll
                    for (int jf = 0; jf < JF; ++jf)
    #pragma unroll
                        for (int v = 0; v < 4; ++v) p2a[jf][v] = p2(mfma_row(T(0), lane, v), 16 * jf + row);
                }
                // one b at a time keeps the live registers low
    #pragma unroll
                for (int bb = 0; bb < 4; ++bb) {
                    double2 ws[4];
    #pragma unroll
                    for (int v = 0; v < 4; ++v) ws[v] = make_double2(0, 0);
    #pragma unroll
                    for (int jf = 0; jf < JF; ++jf) {
                        const double2 p2b = p2(16 + 4 * wave + bb, 16 * jf + row);
    #pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const double2 pa = HOIST ? p2a[HOIST ? jf : 0][v] : p2(mfma_row(T(0), lane, v), 16 * jf + row);
                            const double2 P2 = cmulc(p2b, pa);
                            const double2 Tv = make_double2((double)acc[bb][0][jf][v], (double)acc[bb][1][jf][v]);
                            ws[v] = cadd(ws[v], cmul(P2, Tv));
                        }
                    }
    #pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double2 x = make_double2(row16_sum(ws[v].x), row16_sum(ws[v].y));
                        if (row == 0) {
                            double2 &dst = wl[wave][bb][mfma_row(T(0), lane, v)];
                            dst = cadd(dst, x);
                        }
                    }
                }
            }
            __syncthreads();
        };
        fetch(0, sA0, sW0);
        stash();
        __syncthreads();
        // the buffers by name in each half of the loop (the reads of one need
        // not wait for the direct loads into the other)
        for (int step = 0; step < nsteps; step += 2) {
            body(step, sA0, sW0, sA1, sW1);
            if (step + 1 < nsteps) body(step + 1, sA1, sW1, sA0, sW0);
        }
        // write the 4 x 16 partials of this wave
        const int bb = lane >> 4, a = lane & 15;
        double2 *dst = Wc + (size_t)(b_base + bb) * Np + a_base + a;
        if (half < 0) {
            const double2 x = cscale(wl[wave][bb][a], scale);
            *dst = accumulate ? cadd(*dst, x) : x;
        } else {
            double2 *pp = part + (size_t)slot * nparts * 256 + wave * 64 + lane;
            pp[256 * half] = wl[wave][bb][a];
            __threadfence();
            __syncthreads();
            if (threadIdx.x == 0) s_done = atomicAdd(&queue[kWcQueues + slot], 1);
            __syncthreads();
            if (s_done == nparts - 1) {
                __threadfence();
                double2 acc = pp[0];
                for (int h = 1; h < nparts; ++h) acc = cadd(acc, pp[256 * h]);
                const double2 x = cscale(acc, scale);
                *dst = accumulate ? cadd(*dst, x) : x;
            }
        }
    }
}

// FP64 rank-K part of the two-body contraction:
//     Wc[b][a] (+)= hr hR sum_k alpha_k(b, a) beta_k(b, a),
//     alpha_k(b, a) = sum_i conj(psi1^b_i) psi1^a_i u_k(r_i),
//     beta_k(b, a)  = sum_j conj(psi2^b_j) psi2^a_j v_k(R_j),
// for W_c ~ sum_k u_k(r) v_k(R).  MFMA rows = a, columns = 16 ranks k,
// reduction over the grid points; the A operand, the pair product, is formed
// in registers and feeds RB column blocks of ranks.  Ranks above K have zero
// factors.
//
// A unit is 16 a x B b.  The four waves of its work-group take the 8-point
// steps of the grid in turn: each sums a quarter of every stretch of it, so
// the four partial sums are of one size and their chains of roundings a
// quarter as long (Wc against 80-bit sums, rms over pairs relative to max |Wc|:
// 1.8e-16 at 512 x 256, K = 28, where the dense table's sum has 1.9e-16; 2.1e-16
// and 3.3e-16 at 1024 x 512; 0.9e-16 and 1.2e-16 for the cavity's K = 1).
// They read their operands straight from global memory, two consecutive
// points per lane: no staging through LDS and no barrier inside a pass, so a
// wave only waits for its own loads, which are issued one step ahead.  Only
// the partial sums meet in LDS, 32 KB at a time.  Matrix cores bound it (16
// products per 16 pair-product operations): 0.57 of the FP64 peak on 32 ranks
// at N = 512, 512 x 256, 0.73 at 4096 x 256, where a unit's sums are longer
// against its two reductions.
constexpr int kSepWaves = 4;

// Operand loads of one wave's steps of one species: uniform bases plus lane
// offsets in bytes; step s takes the points 8 s + 2 quarter and
// 8 s + 2 quarter + 1.
template <int B, int RB>
struct SepOperands {
    const gchar *xa_at, *xb_at, *f_at;
    uint32_t xoff, boff, foff, brow, frb;
    dbl2 xa[2], xb[B][2], f[RB];

    __device__ __forceinline__ static dbl2 ld(const gchar *base, uint32_t off) {
        return *reinterpret_cast<const gdouble2 *>(base + off);
    }
    __device__ __forceinline__ void load(dbl2 (&of)[RB]) {
        xa[0] = ld(xa_at, xoff);
        xa[1] = ld(xa_at, xoff + 16u);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) of[rb] = ld(f_at + (size_t)rb * frb, foff);
#pragma unroll
        for (int bb = 0; bb < B; ++bb) {
            xb[bb][0] = ld(xb_at + (size_t)bb * brow, boff);
            xb[bb][1] = ld(xb_at + (size_t)bb * brow, boff + 16u);
        }
        pin_loads();
    }
    // the loads of step lo (n >= 32: every wave has a step)
    __device__ __forceinline__ void begin(const double2 *X, const double *F, int n, int k0, int a_base, int b_base,
                                          int lo) {
        const int lane = threadIdx.x & 63, row = lane & 15, quarter = lane >> 4;
        xa_at = opaque(X + (size_t)a_base * n + (size_t)lo * 8);
        xb_at = opaque(X + (size_t)b_base * n + (size_t)lo * 8);
        f_at = opaque(F + (size_t)k0 * n + (size_t)lo * 128);
        xoff = (uint32_t)row * n * 16u + quarter * 32u;
        boff = quarter * 32u;
        foff = (uint32_t)lane * 16u;
        brow = 16u * n;
        frb = 128u * n;
        load(f);
    }
    // `count` steps, every kSepWaves-th from the first
    __device__ __forceinline__ void accumulate(dbl4 (&acc)[B][2][RB], int count) {
#pragma unroll
        for (int bb = 0; bb < B; ++bb)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) acc[bb][c][rb] = dbl4{0, 0, 0, 0};
        // a step: the pair products of its two points, then its loads'
        // registers take the next step's operands while the matrix cores work
        auto step = [&](dbl2 (&fc)[RB], dbl2 (&fn)[RB], bool last) __attribute__((always_inline)) {
            double pr[B][2], pi[B][2];
#pragma unroll
            for (int bb = 0; bb < B; ++bb)
#pragma unroll
                for (int e = 0; e < 2; ++e) {        // conj(X^b) X^a
                    pr[bb][e] = fma(xb[bb][e].y, xa[e].y, xb[bb][e].x * xa[e].x);
                    pi[bb][e] = fma(-xb[bb][e].y, xa[e].x, xb[bb][e].x * xa[e].y);
                }
            const size_t st = last ? 0 : 128 * kSepWaves;   // the last step loads its own operands again (never used)
            xa_at += st;
            xb_at += st;
            f_at += 8 * st;
            load(fn);
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int bb = 0; bb < B; ++bb)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        acc[bb][0][rb] = mfma(pr[bb][e], fc[rb][e], acc[bb][0][rb]);
                        acc[bb][1][rb] = mfma(pi[bb][e], fc[rb][e], acc[bb][1][rb]);
                    }
        };
        dbl2 g[RB];
        int s = 0;
        for (; s + 1 < count; s += 2) {
            step(f, g, false);
            step(g, f, s + 2 >= count);
        }
        if (s < count) step(f, g, true);
    }
};

// LDS of a work-group: the partial sums of one round, the alphas of the pass,
// and the running sums over the ranks of each column block.
template <int B>
struct SepShared {
    static constexpr int W = kSepWaves, ROUND = 32 / W;   // items per round
    double2 red[W][ROUND][64];
    double2 alpha[8 * B][64];
    double2 wl[2][B][16];
};

// One pass over RB blocks of 16 ranks from k0.  Items (bb, rb, v): one
// accumulator register pair (re, im) of every lane; item j is summed over the
// waves by wave j mod W.
template <int B, int RB>
__device__ __forceinline__ void sep_pass(SepShared<B> &sh, const double2 *__restrict__ psi1,
                                         const double2 *__restrict__ psi2, const double *__restrict__ U,
                                         const double *__restrict__ V, int nr, int nR, int k0, int a_base,
                                         int b_base) {
    const int lane = threadIdx.x & 63, row = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int W = kSepWaves, T = 4 * B * RB, IPR = SepShared<B>::ROUND < T ? SepShared<B>::ROUND : T;
    dbl4 acc[B][2][RB];
    SepOperands<B, RB> op;
    const int steps1 = nr >> 3, steps2 = nR >> 3;
    op.begin(psi1, U, nr, k0, a_base, b_base, wave);
#pragma unroll
    for (int sp = 0; sp < 2; ++sp) {
        const int steps = sp ? steps2 : steps1;
        op.accumulate(acc, steps / W);
        // the second species' first loads are in flight over the reduction
        if (sp == 0) op.begin(psi2, V, nR, k0, a_base, b_base, wave);
#pragma unroll
        for (int r = 0; r < T / IPR; ++r) {
            __syncthreads();                         // the previous round's sums are read
#pragma unroll
            for (int j = 0; j < IPR; ++j) {
                const int it = r * IPR + j, bb = it / (4 * RB), rb = (it / 4) % RB, v = it & 3;
                sh.red[wave][j][lane] = make_double2(acc[bb][0][rb][v], acc[bb][1][rb][v]);
            }
            __syncthreads();
            for (int j = wave; j < IPR; j += W) {
                const int it = r * IPR + j;
                const double2 x = cadd(cadd(sh.red[0][j][lane], sh.red[1][j][lane]),
                                       cadd(sh.red[2][j][lane], sh.red[3][j][lane]));
                if (sp == 0) {
                    sh.alpha[it][lane] = x;          // read back by this wave only
                } else {
                    const int bb = it / (4 * RB), rb = (it / 4) % RB, v = it & 3;
                    const double2 al = sh.alpha[it][lane];
                    const double2 p = make_double2(fma(-al.y, x.y, al.x * x.x), fma(al.y, x.x, al.x * x.y));
                    const double2 y = make_double2(row16_sum(p.x), row16_sum(p.y));
                    if (row == 0) {
                        double2 &dst = sh.wl[rb][bb][mfma_row_f64(lane, v)];
                        dst = cadd(dst, y);
                    }
                }
            }
        }
    }
}

template <int B, bool BATCHED>
__global__ void __launch_bounds__(64 * kSepWaves, 2) k_wc_sep(const double2 *__restrict__ psi1, const double2 *__restrict__ psi2,
                                                   const double *__restrict__ U, const double *__restrict__ V,
                                                   const int32_t *__restrict__ kpad_at, int nr, int nR, double scale,
                                                   double2 *__restrict__ Wc, int Np, int accumulate, int ntiles,
                                                   int32_t *__restrict__ queue, const int32_t *__restrict__ order,
                                                   const int32_t *__restrict__ flags, const long long *__restrict__ zoff) {
    const long long zo_ = BATCHED ? batch_offset(zoff) : 0;
    psi1 = zshift(psi1, zo_);
    psi2 = zshift(psi2, zo_);
    U = zshift(U, zo_);
    V = zshift(V, zo_);
    kpad_at = zshift(kpad_at, zo_);
    Wc = zshift(Wc, zo_);
    queue = zshift(queue, zo_);
    order = zshift(order, zo_);
    flags = zshift(flags, zo_);

    __shared__ SepShared<B> sh;
    __shared__ int s_unit;
    const int kpad = __builtin_amdgcn_readfirstlane(*kpad_at);
    constexpr int G = 16 / B;                        // units per tile
    const int units = ntiles * G;
    const bool queued = (int)gridDim.x < units;      // else one unit per work-group
    // units from the per-XCD queues over the blocked tile order, as k_wc
    const int xcd = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & (kWcQueues - 1);   // HW_REG_XCC_ID
    // (a halt ends the work-group as a whole, through the unit one thread
    // takes, as in k_wc)
    auto take = [&] {
        const bool halt = halted(flags);
        int got = queued ? -1 : (int)blockIdx.x;
        for (int o = 0; o < kWcQueues && got < 0; ++o) {
            const int q = (xcd + o) & (kWcQueues - 1);
            const int lo = (int)((long long)q * units / kWcQueues);
            const int n = (int)((long long)(q + 1) * units / kWcQueues) - lo;
            if (__hip_atomic_load(&queue[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= n) continue;
            const int k = atomicAdd(&queue[q], 1);
            if (k < n) got = lo + k;
        }
        return halt ? -1 : got;
    };
    if (threadIdx.x == 0) s_unit = take();
    __syncthreads();
    int unit = s_unit;
    for (;;) {
        unit = __builtin_amdgcn_readfirstlane(unit);
        if (unit < 0 || unit >= units) break;
        __syncthreads();                             // s_unit is read
        if (queued && threadIdx.x == 64 * (kSepWaves - 1)) s_unit = take();   // the next unit, while this one is worked on
        int tb, ta;
        triangle_tile(order[unit / G], &tb, &ta);
        const int a_base = __builtin_amdgcn_readfirstlane(ta * 16);
        const int b_base = __builtin_amdgcn_readfirstlane(tb * 16 + (unit % G) * B);
        const int t = threadIdx.x;
        if (t < 2 * B * 16) (&sh.wl[0][0][0])[t] = make_double2(0, 0);
        int k0 = 0;
        for (; k0 + 32 <= kpad; k0 += 32) sep_pass<B, 2>(sh, psi1, psi2, U, V, nr, nR, k0, a_base, b_base);
        if (k0 < kpad) sep_pass<B, 1>(sh, psi1, psi2, U, V, nr, nR, k0, a_base, b_base);
        __syncthreads();
        if (t < B * 16) {
            const int bb = t >> 4, a = t & 15;
            const double2 x = cscale(cadd(sh.wl[0][bb][a], sh.wl[1][bb][a]), scale);
            double2 *dst = Wc + (size_t)(b_base + bb) * Np + a_base + a;
            *dst = accumulate ? cadd(*dst, x) : x;
        }
        if (!queued) break;
        __syncthreads();                             // wl is read
        unit = s_unit;
    }
}

}  // namespace

std::vector<int32_t> wc_tile_order(int Np) {
    const int T = Np / 16, S = 8, nS = (T + S - 1) / S;
    std::vector<int32_t> ord;
    ord.reserve((size_t)T * (T + 1) / 2);
    for (int sb = 0; sb < nS; ++sb)
        for (int sa = sb; sa < nS; ++sa)
            for (int tb = sb * S; tb < std::min(T, sb * S + S); ++tb)
                for (int ta = std::max(tb, sa * S); ta < std::min(T, sa * S + S); ++ta)
                    ord.push_back(ta * (ta + 1) / 2 + tb);
    return ord;
}

static void launch_kets(const Dims &d, const Bufs &b, const CondSpecies &s1, const CondSpecies &s2, hipStream_t s) {
    if (d.bilinear) return;
    const int Np = padded(d.N);
    const unsigned blocks1 = (unsigned)(((size_t)Np * d.nr + 255) / 256), blocks2 = (unsigned)(((size_t)Np * d.nR + 255) / 256);
    hipLaunchKernelGGL(k_cond_kets, dim3(blocks1 + blocks2, 1, d.batch), dim3(256), 0, s, s1, s2, blocks1, d.mp, Np,
                       b.flags, d.zoff, d.mpd);
}

void launch_cond_kets(const Dims &d, const Bufs &b, hipStream_t s, bool next) {
    launch_kets(d, b, {b.psi1, b.R, b.R_new, b.G1a, next ? b.G1b : nullptr, d.nr, d.r_min, d.hr},
                {b.psi2, b.r, b.r_new, b.G2a, next ? b.G2b : nullptr, d.nR, d.R_min, d.hR}, s);
}

void launch_cond_kets_next(const Dims &d, const Bufs &b, hipStream_t s) {
    launch_kets(d, b, {b.psi1, b.R_new, b.R_new, b.G1b, nullptr, d.nr, d.r_min, d.hr},
                {b.psi2, b.r_new, b.r_new, b.G2b, nullptr, d.nR, d.R_min, d.hR}, s);
}

void launch_single_species(const Dims &d, const Bufs &b, bool both, hipStream_t s, int parts) {
    ZBatch zb{};
    int c = 0;
    auto add = [&](const double2 *X, const double2 *Y, double2 *o, int K, double sc) {
        zb.X[c] = X;
        zb.Y[c] = Y;
        zb.out[c] = o;
        zb.K[c] = K;
        zb.scale[c] = sc;
        ++c;
    };
    if (parts & kSingleOverlaps) {
        add(b.psi1, b.psi1, b.S1, d.nr, d.hr);
        if (d.bilinear) {
            add(b.psi1, b.psi1, b.E1a, d.nr, d.hr);
            zb.weighted[1] = 1;
            zb.w0[1] = d.r_min;
            zb.w1[1] = d.hr;
        }
        add(b.psi2, b.psi2, b.S2, d.nR, d.hR);
        if (d.bilinear) {
            add(b.psi2, b.psi2, b.E2a, d.nR, d.hR);
            zb.weighted[3] = 1;
            zb.w0[3] = d.R_min;
            zb.w1[3] = d.hR;
        }
    }
    if ((parts & kSingleCouplings) && !d.bilinear) {
        add(b.psi1, b.G1a, b.E1a, d.nr, d.hr);
        if (both) add(b.psi1, b.G1b, b.E1b, d.nr, d.hr);
        add(b.psi2, b.G2a, b.E2a, d.nR, d.hR);
        if (both) add(b.psi2, b.G2b, b.E2b, d.nR, d.hR);
    }
    if (c == 0) return;
    launch_zgemm(d, zb, c, b.flags, s);
}

void launch_single_species_next(const Dims &d, const Bufs &b, hipStream_t s) {
    if (d.bilinear) return;
    ZBatch zb{};
    zb.X[0] = b.psi1;
    zb.Y[0] = b.G1b;
    zb.out[0] = b.E1b;
    zb.K[0] = d.nr;
    zb.scale[0] = d.hr;
    zb.X[1] = b.psi2;
    zb.Y[1] = b.G2b;
    zb.out[1] = b.E2b;
    zb.K[1] = d.nR;
    zb.scale[1] = d.hR;
    launch_zgemm(d, zb, 2, b.flags, s);
}

// The sum-of-products contraction.  Fewer b per unit where the launch would
// otherwise leave compute units without work; the sums of a pair do not depend
// on it (512 x 256, K = 28: N = 64, 16 us with 1, 22 with 2, 36 with 4; N = 250,
// 159, 107 and 117 us; N = 500, 550, 340 and 305 us).
static void launch_wc_sep(const Dims &d, const Bufs &b, int accumulate, hipStream_t s) {
    const int Np = padded(d.N), T16 = Np / 16, tiles = T16 * (T16 + 1) / 2;
    auto go = [&](auto kernel, int B) {
        const int units = tiles * (16 / B), grid = std::min(units, d.wc_grid);
        if (grid < units) launch_fill_i32(b.wc_queue, kWcQueues, 0, s, d.batch, d.zoff);
        hipLaunchKernelGGL(kernel, dim3(grid, 1, d.batch), dim3(64 * kSepWaves), 0, s, b.psi1, b.psi2, b.lr_u, b.lr_v,
                           b.lr_pad, d.nr, d.nR, d.hr * d.hR, b.Wc, Np, accumulate, tiles, b.wc_queue, b.wc_order,
                           b.flags, d.zoff);
    };
    const long long all = (long long)tiles * d.batch;
    if (all * 16 <= 512) go(d.zoff ? k_wc_sep<1, true> : k_wc_sep<1, false>, 1);
    else if (all * 4 <= 768) go(d.zoff ? k_wc_sep<2, true> : k_wc_sep<2, false>, 2);
    else go(d.zoff ? k_wc_sep<4, true> : k_wc_sep<4, false>, 4);
}

int contraction_route(const Dims &d) {
    if (d.bilinear) return ICWF_CONTRACTION_BILINEAR;
    if (d.products) return ICWF_CONTRACTION_PRODUCTS;
    // the FP32 pass tiles the grid in chunks of 64 x 64 points: smaller grids
    // take the dense FP64 contraction of the whole table instead
    const bool fp32_fits = d.nr >= WcChunk<float>::KC && d.nR >= WcChunk<float>::JT;
    return d.prec == 1 && fp32_fits ? ICWF_CONTRACTION_FP32 : ICWF_CONTRACTION_TABLE;
}

void launch_wc(const Dims &d, const Bufs &b, hipStream_t s) {
    const int route = contraction_route(d);
    if (route == ICWF_CONTRACTION_BILINEAR) return;  // the assembly multiplies <b|r|a> by <b|R|a>
    const int Np = padded(d.N);
    const int T16 = Np / 16;
    const int blocks = T16 * (T16 + 1) / 2;
    const double scale = d.hr * d.hR;
    // the last round of tiles split in kWcParts (fewer where R has fewer j
    // tiles)
    const int grid = std::min(blocks, d.wc_grid);
    auto split = [&](int jt, int *nparts, int *spq) {
        *nparts = std::min(kWcParts, d.nR / jt);
        const int nsplit = *nparts >= 2 ? std::min(grid, wc_split_tiles(Np)) : 0;
        *spq = wc_split_per_queue(nsplit);   // split tiles per queue
    };
    int nparts, spq;
    if (route == ICWF_CONTRACTION_PRODUCTS) {
        launch_wc_sep(d, b, 0, s);
    } else if (route == ICWF_CONTRACTION_FP32) {
        // mixed: FP32 matrix cores on the residual of the rank-K split, FP64 rank-K part added
        split(WcChunk<float>::JT, &nparts, &spq);
        launch_fill_i32(b.wc_queue, kWcQueues + kWcQueues * spq, 0, s, d.batch, d.zoff);
        hipLaunchKernelGGL((d.zoff ? k_wc<float, true> : k_wc<float, false>), dim3(grid, 1, d.batch), dim3(256), 0, s,
                           b.psi1_f32, b.psi2, b.wc32, d.nr, d.nR, scale, b.Wc, Np, 0, blocks, spq, nparts,
                           b.wc_queue, b.wc_order, b.wc_part, b.flags, d.zoff);
        if (d.lr_rank > 0) launch_wc_sep(d, b, 1, s);
    } else {
        split(WcChunk<double>::JT, &nparts, &spq);
        launch_fill_i32(b.wc_queue, kWcQueues + kWcQueues * spq, 0, s, d.batch, d.zoff);
        hipLaunchKernelGGL((d.zoff ? k_wc<double, true> : k_wc<double, false>), dim3(grid, 1, d.batch), dim3(256), 0, s, b.psi1, b.psi2, b.wc64, d.nr, d.nR,
                           scale, b.Wc, Np, 0, blocks, spq, nparts, b.wc_queue, b.wc_order, b.wc_part, b.flags,
                           d.zoff);
    }
}

}  // namespace icwf
