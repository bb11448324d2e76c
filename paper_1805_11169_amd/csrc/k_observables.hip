// Observables of the ansatz (text around the Shin-Metiu figure), all from the
// wavefunction on the grid, Eq. 7 evaluated at the grid points:
//     Psi(r_i, R_j) = sum_a C_a psi1^a_i psi2^a_j          (one complex GEMM)
//     rho(r_i) = hR sum_j |Psi_ij|^2,   rho(R_j) = hr sum_i |Psi_ij|^2,
//     norm = hr sum_i rho(r_i)  (= C^H S C),
//     chi^(n)(R_j) = hr sum_i phi_n(r_i; R_j) Psi_ij  (BO projections, real phi_n),
//     P_n = hR sum_j |chi^(n)_j|^2,  D_nm = hR sum_j |chi^(n)_j|^2 |chi^(m)_j|^2.
// The GEMM costs N n_r n_R complex products, against N^2 (n_r + n_R) for the
// same densities written with the single-species overlaps.  Computed on
// demand, not every step; every sum runs in a fixed order (bitwise
// repeatable).  Output layout: [norm, rho_r[nr], rho_R[nR], pop[n_bo], D[n_bo][n_bo]].
#include "icwf_plan.hpp"

namespace icwf {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

__device__ inline dbl4 mfma(double a, double b, dbl4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Psi = U^T V, U[a][i] = C_a psi1[a][i], V[a][j] = psi2[a][j], a < Np.  A
// work-group per 16 F x 16 F tile of Psi, F x F fragments of v_mfma_f64_16x16x4
// with rows = i, columns = j and the trajectory a as the reduction index; its
// four waves take the steps of the reduction (16 trajectories each) in turn,
// operands straight from global memory (the 16 grid points of a fragment are
// consecutive) one step ahead; the partial tiles meet in LDS and are added in
// the order of the waves.  Bound by the reads of psi from L2 where the tiles
// fill the device, by latency on small grids.  Against 64 x 64 tiles through
// LDS, a wave to a quarter of the tile (32 work-groups on 512 x 256), whole
// call: N = 1024 on 512 x 256, 276 -> 82 us; N = 2048 on 1024 x 256, 496 -> 138;
// N = 1500 on 1024 x 512, 362 -> 180; N = 4096 on 4096 x 512, 1.44 -> 1.20 ms.
template <int F>
__global__ void __launch_bounds__(256) k_obs_psi(const double2 *__restrict__ psi1,
                                                       const double2 *__restrict__ psi2,
                                                       const double2 *__restrict__ C, int nr, int nR, int Np,
                                                       double2 *__restrict__ Psi) {
    constexpr int T = 16 * F;
    __shared__ double2 part[4][T * T];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int row = lane & 15, quarter = lane >> 4;
    const int i0 = blockIdx.y * T, j0 = blockIdx.x * T;
    dbl4 re[F][F], im[F][F];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int g = 0; g < F; ++g) {
            re[f][g] = dbl4{0, 0, 0, 0};
            im[f][g] = dbl4{0, 0, 0, 0};
        }
    const double2 *pu = psi1 + i0 + row, *pv = psi2 + j0 + row;
    double2 c[4], u[4][F], v[4][F];
    auto load = [&](int a0) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int a = a0 + 4 * s + quarter;
            c[s] = C[a];
#pragma unroll
            for (int f = 0; f < F; ++f) {
                u[s][f] = pu[(size_t)a * nr + 16 * f];
                v[s][f] = pv[(size_t)a * nR + 16 * f];
            }
        }
    };
    load(16 * wave);
    for (int a0 = 16 * wave; a0 < Np; a0 += 64) {
        double2 uc[4][F], vc[4][F];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int f = 0; f < F; ++f) {
                uc[s][f] = cmul(c[s], u[s][f]);
                vc[s][f] = v[s][f];
            }
        if (a0 + 64 < Np) load(a0 + 64);
        pin_loads();
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int f = 0; f < F; ++f)
#pragma unroll
                for (int g = 0; g < F; ++g) {
                    re[f][g] = mfma(uc[s][f].x, vc[s][g].x, re[f][g]);
                    re[f][g] = mfma(-uc[s][f].y, vc[s][g].y, re[f][g]);
                    im[f][g] = mfma(uc[s][f].x, vc[s][g].y, im[f][g]);
                    im[f][g] = mfma(uc[s][f].y, vc[s][g].x, im[f][g]);
                }
    }
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int g = 0; g < F; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                part[wave][(16 * f + mfma_row_f64(lane, q)) * T + 16 * g + row] = make_double2(re[f][g][q], im[f][g][q]);
    __syncthreads();
    for (int e = t; e < T * T; e += 256)
        Psi[(size_t)(i0 + e / T) * nR + j0 + e % T] =
            cadd(cadd(part[0][e], part[1][e]), cadd(part[2][e], part[3][e]));
}

__device__ inline double block_sum(double v, double *red) {
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    const double s = red[0];
    __syncthreads();
    return s;
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// rho_r[i] = hR sum_j |Psi_ij|^2: one wave per row, four rows per block.
__global__ void k_obs_rho_r(const double2 *__restrict__ Psi, int nr, int nR, double hR, double *__restrict__ rho) {
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= nr) return;
    double acc = 0.0;
    for (int j = lane; j < nR; j += 64) {
        const double2 p = Psi[(size_t)i * nR + j];
        acc += p.x * p.x + p.y * p.y;
    }
    acc = wave_sum(acc);
    if (lane == 0) rho[i] = hR * acc;
}

// rho_R[j] = hr sum_i |Psi_ij|^2 in two passes, so that tall grids fill the
// device: block (x, y) sums rows y nr/S ... (y + 1) nr/S - 1 of 64 columns
// (four row slices reduced in LDS in a fixed order) into part[y][j]; then
// the S partial sums of each column are added in order.
__global__ void k_obs_rho_R_part(const double2 *__restrict__ Psi, int nr, int nR, double *__restrict__ part) {
    __shared__ double red[4][64];
    const int c = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + c;
    const int rows = nr / kRhoSlices, i0 = blockIdx.y * rows;
    double acc = 0.0;
    if (j < nR)
        for (int i = i0 + sl; i < i0 + rows; i += 4) {
            const double2 p = Psi[(size_t)i * nR + j];
            acc += p.x * p.x + p.y * p.y;
        }
    red[sl][c] = acc;
    __syncthreads();
    if (sl == 0 && j < nR) part[(size_t)blockIdx.y * nR + j] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

__global__ void k_obs_rho_R_sum(const double *__restrict__ part, int nR, double hr, double *__restrict__ rho) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nR) return;
    double acc = 0.0;
    for (int s = 0; s < kRhoSlices; ++s) acc += part[(size_t)s * nR + j];
    rho[j] = hr * acc;
}

// out[0] = hr sum_i rho_r[i]; one block.
__global__ void k_obs_norm(const double *__restrict__ rho_r, int nr, double hr, double *__restrict__ out) {
    __shared__ double part[4];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nr; i += blockDim.x) acc += rho_r[i];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = hr * (((part[0] + part[1]) + part[2]) + part[3]);
}

// chi[nb][j] = hr sum_i bo[j][nb][i] Psi_ij: one wave per (j, nb).
__global__ void k_obs_chi(const double *__restrict__ bo, const double2 *__restrict__ Psi, int nr, int nR,
                          int n_bo, double hr, double2 *__restrict__ chi) {
    const int j = blockIdx.x, nb = blockIdx.y, lane = threadIdx.x;
    const double *phi = bo + ((size_t)j * n_bo + nb) * nr;
    double sr = 0.0, si = 0.0;
    for (int i = lane; i < nr; i += 64) {
        const double2 p = Psi[(size_t)i * nR + j];
        sr += phi[i] * p.x;
        si += phi[i] * p.y;
    }
    sr = wave_sum(sr);
    si = wave_sum(si);
    if (lane == 0) chi[(size_t)nb * nR + j] = make_double2(hr * sr, hr * si);
}

// pop[n] and D[n][m]; one block.
__global__ void k_obs_pop(const double2 *__restrict__ chi, int nR, int n_bo, double hR, double *__restrict__ pop,
                          double *__restrict__ D) {
    __shared__ double red[256];
    for (int n = 0; n < n_bo; ++n) {
        for (int m = 0; m <= n; ++m) {
            double acc = 0.0;
            for (int j = threadIdx.x; j < nR; j += blockDim.x) {
                const double2 cn = chi[(size_t)n * nR + j], cm = chi[(size_t)m * nR + j];
                const double dn = cn.x * cn.x + cn.y * cn.y, dm = cm.x * cm.x + cm.y * cm.y;
                acc += (n == m) ? dn : dn * dm;
            }
            // P_n from the m == n pass, D_nn from a separate sum of dn^2
            const double s = block_sum(acc, red);
            if (n == m) {
                double acc2 = 0.0;
                for (int j = threadIdx.x; j < nR; j += blockDim.x) {
                    const double2 cn = chi[(size_t)n * nR + j];
                    const double dn = cn.x * cn.x + cn.y * cn.y;
                    acc2 += dn * dn;
                }
                const double s2 = block_sum(acc2, red);
                if (threadIdx.x == 0) {
                    pop[n] = hR * s;
                    D[n * n_bo + n] = hR * s2;
                }
            } else if (threadIdx.x == 0) {
                D[n * n_bo + m] = hR * s;
                D[m * n_bo + n] = hR * s;
            }
        }
    }
}

// What an observables call returns beside the observables, behind them in one
// array, so that it all comes back in one copy: r[N], R[N], C[N], the scalars
// and the flags.
__global__ void k_obs_tail(const double *__restrict__ r, const double *__restrict__ R, const double2 *__restrict__ C,
                           const double *__restrict__ scal, const int32_t *__restrict__ flags, int N,
                           double *__restrict__ tail) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) {
        tail[i] = r[i];
        tail[N + i] = R[i];
        const double2 c = C[i];
        tail[2 * N + 2 * i] = c.x;
        tail[2 * N + 2 * i + 1] = c.y;
    }
    if (blockIdx.x == 0 && threadIdx.x < kObsScalars) tail[4 * N + threadIdx.x] = scal[threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x < kNumFlags)
        reinterpret_cast<int32_t *>(tail + 4 * N + kObsScalars)[threadIdx.x] = flags[threadIdx.x];
}

}  // namespace

void launch_grid_observables(const double2 *Psi, int nr, int nR, double hr, double hR, int n_bo, const double *bo,
                             double2 *chi, double *part, double *out, hipStream_t s) {
    double *rho_r = out + 1, *rho_R = out + 1 + nr;
    hipLaunchKernelGGL(k_obs_rho_r, dim3((nr + 3) / 4), dim3(256), 0, s, Psi, nr, nR, hR, rho_r);
    hipLaunchKernelGGL(k_obs_rho_R_part, dim3((nR + 63) / 64, kRhoSlices), dim3(256), 0, s, Psi, nr, nR, part);
    hipLaunchKernelGGL(k_obs_rho_R_sum, dim3((nR + 255) / 256), dim3(256), 0, s, part, nR, hr, rho_R);
    hipLaunchKernelGGL(k_obs_norm, dim3(1), dim3(256), 0, s, rho_r, nr, hr, out);
    if (n_bo > 0) {
        hipLaunchKernelGGL(k_obs_chi, dim3(nR, n_bo), dim3(64), 0, s, bo, Psi, nr, nR, n_bo, hr, chi);
        double *pop = out + 1 + nr + nR;
        hipLaunchKernelGGL(k_obs_pop, dim3(1), dim3(256), 0, s, chi, nR, n_bo, hR, pop, pop + n_bo);
    }
}

void launch_observables(const Dims &d, const Bufs &b, hipStream_t s) {
    const int Np = padded(d.N);
    auto go = [&](auto kernel, int tile) {               // (the grids are powers of two >= 32)
        hipLaunchKernelGGL(kernel, dim3(d.nR / tile, d.nr / tile), dim3(256), 0, s, b.psi1, b.psi2, b.C, d.nr, d.nR, Np,
                           b.obs_psi);
    };
    // 32 x 32 tiles where there is one for a CU (whole call with tiles of 32 and
    // 16: N = 2048 on 1024 x 256, 138 and 164 us; N = 1024 on 512 x 256, 90 and 82)
    if ((size_t)d.nr * d.nR >= (size_t)256 * 32 * 32) go(k_obs_psi<2>, 32);
    else go(k_obs_psi<1>, 16);
    launch_grid_observables(b.obs_psi, d.nr, d.nR, d.hr, d.hR, d.n_bo, b.bo, b.obs_chi, b.obs_part, b.obs_out, s);
    double *tail = b.obs_out + obs_len(d.nr, d.nR, d.n_bo);
    hipLaunchKernelGGL(k_obs_tail, dim3((d.N + 255) / 256), dim3(256), 0, s, b.r, b.R, b.C, b.scal, b.flags, d.N, tail);
}

}  // namespace icwf
