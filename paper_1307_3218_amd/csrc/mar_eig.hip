// Subspace eigensolve and Fermi-weighted assembly.
//
// For seed j with m = nu_eff vectors, A = K^T H K (m x m, FP64) is
// diagonalized, and the same rotations are applied to the rows of the
// m x (1 + |P(j)|) matrix R = [e_1 | K[P(j), :]^T]. No m x m eigenvector
// matrix is formed. At the end the levels eps_alpha are known and row alpha of
// R holds
//     R[alpha][0]     = y_1alpha            (first component of y_alpha)
//     R[alpha][1 + t] = e_i . v_alpha,  i = P(j)[t],  v_alpha = K y_alpha
// which is all the Green's-function assembly needs (Sec. 2):
//     rho_ij = 2 sum_alpha f_alpha (e_i.v_alpha)(e_j.v_alpha),
//     w_alpha = (e_j^T S v_alpha)(v_alpha^T e_j) = sqrt(S_jj) y_1alpha (e_j.v_alpha)
// (K^T S e_j = sqrt(S_jj) e_1 because u_1 = e_j / sqrt(S_jj) and K^T S K = I),
//     E_j = sum_{i in P(j)} rho_ij H_ij,   N_j = sum_{i in P(j)} rho_ij S_ij.
//
// Two methods: Householder reduction to tridiagonal form and implicit QL
// (k_tri, k_tri_big, k_ql; the ordinary passes), and the parallel cyclic
// Jacobi method (k_eig; all eigenvectors of the reference seed of an eigen
// state, solves with a cap on Jacobi sweeps, rows too long for a wavefront):
// each step rotates m / 2 disjoint index pairs at once (a round-robin
// tournament, so that every pair meets once per sweep of m - 1 steps or m
// steps for odd m), A <- J^T A J; sweeps repeat until one rotates nothing.
#include <algorithm>
#include <cfloat>
#include <cstdint>

#include <type_traits>

#include "mar_device.h"
#include "mar_internal.h"

namespace mar {

__device__ __forceinline__ double fermi_occ(double eps, double mu, double kT) {
    if (kT == 0.0) return eps < mu ? 1.0 : (eps > mu ? 0.0 : 0.5);
    const double x = (eps - mu) / kT;
    const double t = exp(-fabs(x));
    return x >= 0.0 ? t / (1.0 + t) : 1.0 / (1.0 + t);
}

// Logistic step F(x) = 1/(1+e^-x), and the window of a smoothed delta of width
// sigma over [a, b] (sigma = 0: sharp, 1/2 at an endpoint) for Eq. 3.
__device__ __forceinline__ double logistic_step(double x) {
    const double t = exp(-fabs(x));
    return x >= 0.0 ? 1.0 / (1.0 + t) : t / (1.0 + t);
}
__device__ __forceinline__ double smooth_step(double x, double sigma) {
    if (sigma == 0.0) return x > 0.0 ? 1.0 : (x < 0.0 ? 0.0 : 0.5);
    return logistic_step(x / sigma);
}
__device__ __forceinline__ double level_window(double eps, double a, double b, double sigma) {
    return smooth_step(b - eps, sigma) - smooth_step(a - eps, sigma);
}

// Threads of the eigensolver's workgroup: four waves per SIMD, so that the
// LDS latencies of the Jacobi steps of one seed hide behind each other.
constexpr int EIG_WG = 1024;
constexpr int EIG_WAVES = EIG_WG / 64;
// Per-thread work lists of a Jacobi step when they are short (at most JB blocks
// and JR entries of R per thread, fixed for the whole iteration).
constexpr int JB = 3, JR = 4;

// Parallel cyclic Jacobi on the symmetric m x m matrix A (in LDS or global
// memory, upper triangle only: a_ij, i <= j, at A[i * ld + j]; an odd ld spreads
// the column accesses over the LDS banks), each rotation also applied to the
// rows of the m x nr matrix R (R <- J^T R). Run by the whole workgroup.
// Step s of a sweep pairs the indices of a round-robin tournament of n = m
// rounded up to even players (player n - 1 = m is a bye for odd m): position k
// holds players idx(k) and idx(n - 1 - k), idx(0) = 0, idx(i) = 1 + (i - 1 + s)
// mod (n - 1). A pair (p, q) rotates when |a_pq| > eps sqrt(|a_pp a_qq|), with
// the symmetric Schur rotation that zeroes a_pq (tau = (a_qq - a_pp) / (2 a_pq),
// t = sign(tau) / (|tau| + sqrt(1 + tau^2)), c = 1 / sqrt(1 + t^2), s = t c):
// a_pp -= t a_pq, a_qq += t a_pq, a_pq = 0. Every other element belongs to one
// 2 x 2 block of two pairs, J_1^T B J_2, updated in place by one thread (blocks
// k1 <= k2 of pair positions). When the blocks and R's entries make at most JB
// and JR per thread, each thread keeps its list for the whole iteration and
// issues all loads of a step at once; otherwise wave w takes the block rows
// k1 = w, w + 16, ..., its lanes the block columns. Sweeps repeat until one
// rotates nothing, at most max_sweeps. Scratch: cs, sn, tt (n / 2 doubles
// each), cnt (one int). Returns 0 when converged, 1 otherwise. The levels are
// A's diagonal.
__device__ __forceinline__ int jacobi_eig(double* A, int ld, int m, double* R, int nr, double* cs, double* sn,
                                          double* tt, int* cnt, int max_sweeps) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = m + (m & 1), np = n / 2, n1 = n - 1;
    auto off = [&](int i, int j) { return i <= j ? i * ld + j : j * ld + i; };   // a_ij in the upper triangle
    // the pair at position k of step st, p < q (q == m: the bye)
    auto pair = [&](int k, int st, int& p, int& q) {
        int a = k - 1 + st, bb = n - 2 - k + st;
        a = k == 0 ? 0 : 1 + (a >= n1 ? a - n1 : a);
        bb = 1 + (bb >= n1 ? bb - n1 : bb);
        p = a < bb ? a : bb;
        q = a < bb ? bb : a;
    };
    // J_1^T B J_2 on the block of positions k1 < k2 (pairs (p1, q1), (p2, q2)); a bye's row or column is
    // absent (its loads read a_p1p2 again and are dropped)
    auto block = [&](int p1, int q1, double c1, double s1, int p2, int q2, double c2, double s2) {
        const bool hq1 = q1 < m, hq2 = q2 < m, hw = hq1 && hq2;
        const int ox = off(p1, p2);
        const int oy = hq2 ? off(p1, q2) : ox, oz = hq1 ? off(q1, p2) : ox, ow = hw ? off(q1, q2) : ox;
        const double x = A[ox];
        const double y = hq2 ? A[oy] : 0.0, z = hq1 ? A[oz] : 0.0, w = hw ? A[ow] : 0.0;
        const double xr = c1 * x - s1 * z, yr = c1 * y - s1 * w;   // rows: J_1^T B
        const double zr = s1 * x + c1 * z, wr = s1 * y + c1 * w;
        A[ox] = c2 * xr - s2 * yr;                                  // columns: (J_1^T B) J_2
        if (hq2) A[oy] = s2 * xr + c2 * yr;
        if (hq1) A[oz] = c2 * zr - s2 * wr;
        if (hw) A[ow] = s2 * zr + c2 * wr;
    };
    // fixed per-thread lists when short: blocks (k1, k2), k1 <= k2, numbered row by row, and R entries (k, col)
    const int nblk = np * (np + 1) / 2;
    const bool lists = nblk <= JB * EIG_WG && np * nr <= JR * EIG_WG;
    int bk1[JB], bk2[JB], rk[JR], rc[JR];
#pragma unroll
    for (int i = 0; i < JB; ++i) {
        int lin = tid + i * EIG_WG, k1 = 0;
        bk1[i] = -1;
        bk2[i] = 0;
        if (lists && lin < nblk) {
            while (lin >= np - k1) {
                lin -= np - k1;
                ++k1;
            }
            bk1[i] = k1;
            bk2[i] = k1 + lin;
        }
    }
#pragma unroll
    for (int i = 0; i < JR; ++i) {
        const int lin = tid + i * EIG_WG;
        rk[i] = lists && lin < np * nr ? lin / nr : -1;
        rc[i] = lists && lin < np * nr ? lin - (lin / nr) * nr : 0;
    }
    if (tid == 0) *cnt = 0;
    __syncthreads();
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        for (int st = 0; st < n1; ++st) {
            // the rotations of this step, one pair per thread
            for (int k = tid; k < np; k += EIG_WG) {
                int p, q;
                pair(k, st, p, q);
                double c = 1.0, sv = 0.0, t = 0.0;
                if (q < m) {
                    const double apq = A[p * ld + q], app = A[p * ld + p], aqq = A[q * ld + q];   // p < q
                    if (apq != 0.0 && apq * apq > (DBL_EPSILON * DBL_EPSILON) * fabs(app * aqq)) {
                        const double tau = (aqq - app) * recip(2.0 * apq);
                        if (fabs(tau) > 1e150) {
                            t = 0.5 * recip(tau);
                        } else {
                            const double r = 1.0 + tau * tau;
                            t = copysign(recip(fabs(tau) + r * rsqrt_nr(r)), tau);
                        }
                        c = rsqrt_nr(1.0 + t * t);
                        sv = t * c;
                        atomicAdd(cnt, 1);
                    }
                }
                cs[k] = c;
                sn[k] = sv;
                tt[k] = t;
            }
            __syncthreads();
            if (lists) {
#pragma unroll
                for (int i = 0; i < JB; ++i) {
                    const int k1 = bk1[i], k2 = bk2[i];
                    if (k1 < 0) continue;
                    int p1, q1;
                    pair(k1, st, p1, q1);
                    const double c1 = cs[k1], s1 = sn[k1];
                    if (k1 == k2) {
                        if (s1 != 0.0) {
                            const double apq = A[p1 * ld + q1], t = tt[k1];
                            A[p1 * ld + p1] -= t * apq;
                            A[q1 * ld + q1] += t * apq;
                            A[p1 * ld + q1] = 0.0;
                        }
                        continue;
                    }
                    const double c2 = cs[k2], s2 = sn[k2];
                    if (s1 == 0.0 && s2 == 0.0) continue;
                    int p2, q2;
                    pair(k2, st, p2, q2);
                    block(p1, q1, c1, s1, p2, q2, c2, s2);
                }
#pragma unroll
                for (int i = 0; i < JR; ++i) {
                    const int k = rk[i], col = rc[i];
                    if (k < 0) continue;
                    const double sv = sn[k];
                    if (sv == 0.0) continue;
                    int p, q;
                    pair(k, st, p, q);
                    const double c = cs[k], rp = R[p * nr + col], rq = R[q * nr + col];
                    R[p * nr + col] = c * rp - sv * rq;
                    R[q * nr + col] = sv * rp + c * rq;
                }
            } else {
                for (int k1 = wave; k1 < np; k1 += EIG_WAVES) {
                    int p1, q1;
                    pair(k1, st, p1, q1);
                    const double c1 = cs[k1], s1 = sn[k1];
                    for (int k2 = k1 + lane; k2 < np; k2 += 64) {
                        if (k2 == k1) {
                            if (s1 != 0.0) {
                                const double apq = A[p1 * ld + q1], t = tt[k1];
                                A[p1 * ld + p1] -= t * apq;
                                A[q1 * ld + q1] += t * apq;
                                A[p1 * ld + q1] = 0.0;
                            }
                            continue;
                        }
                        const double c2 = cs[k2], s2 = sn[k2];
                        if (s1 == 0.0 && s2 == 0.0) continue;
                        int p2, q2;
                        pair(k2, st, p2, q2);
                        block(p1, q1, c1, s1, p2, q2, c2, s2);
                    }
                }
                for (int k = wave; k < np; k += EIG_WAVES) {
                    const double sv = sn[k];
                    if (sv == 0.0) continue;
                    int p, q;
                    pair(k, st, p, q);
                    const double c = cs[k];
                    for (int col = lane; col < nr; col += 64) {
                        const double rp = R[p * nr + col], rq = R[q * nr + col];
                        R[p * nr + col] = c * rp - sv * rq;
                        R[q * nr + col] = sv * rp + c * rq;
                    }
                }
            }
            __syncthreads();
        }
        const int rotated = *cnt;
        __syncthreads();
        if (tid == 0) *cnt = 0;
        __syncthreads();
        if (rotated == 0) return 0;
    }
    return 1;
}

size_t eig_lds_bytes(int nu, int max_row, bool a_in_lds) {
    size_t n = (a_in_lds ? (size_t)nu * (nu + 1) : 0) + (size_t)nu * (max_row + 1) + 4 * (size_t)nu + 8 + 72 + 64 + 2;
    return n * sizeof(double);
}

bool eig_a_fits_lds(int nu, int max_row) { return eig_lds_bytes(nu, max_row, true) <= 160 * 1024; }

// Rows K[P(j), :] of each seed, gathered from the seed-interleaved basis into
// Kp[(b * nu + k) * max_row + t] (FP64), with the seed's nu_eff copied beside
// them, so that the eigensolve can run while the basis is reused.
template <typename T>
__global__ __launch_bounds__(WG) void k_gather_rows(int nseeds, const int32_t* __restrict__ seeds, int B, int nu,
                                                    const int32_t* __restrict__ nu_eff_blk, const T* __restrict__ K,
                                                    int64_t stride, const int32_t* __restrict__ Hrp,
                                                    const int32_t* __restrict__ Hcol, int max_row,
                                                    double* __restrict__ Kp, int32_t* __restrict__ nu_copy) {
    const int b = blockIdx.x;
    if (b >= nseeds) return;
    const int m = nu_eff_blk[b];
    if (threadIdx.x == 0) nu_copy[b] = m;
    if (m <= 0) return;
    const int j = seeds[b];
    const int rlo = Hrp[j], nP = Hrp[j + 1] - rlo;
    for (int idx = threadIdx.x; idx < m * nP; idx += WG) {
        const int k = idx / nP, t = idx - k * nP;
        Kp[((int64_t)b * nu + k) * max_row + t] = (double)K[(int64_t)k * stride + (int64_t)Hcol[rlo + t] * B + b];
    }
}

// Orders LDS among the lanes of one wavefront, and among NT threads that share a seed (64: one wavefront).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <int NT>
__device__ __forceinline__ void group_sync() {
    if constexpr (NT == 64) wave_sync();
    else __syncthreads();
}

// What a seed's eigenpairs give, run by NT threads (a workgroup of them, or NT = 64: one of its
// wavefronts): R's rows hold y_1alpha, then e_i.v_alpha
// (i in P(j)), then (mode 2) v_ref.v_alpha; d the levels. The Eq. 3 component (mode 2), or the kept rows for an
// assembly at a Fermi level found later (zc; k_assemble takes the same sums in the same order), or the Fermi-weighted
// assembly. fz: m doubles, rhoL: 64 doubles of LDS.
template <int NT>
__device__ __forceinline__ void eig_results(const EigExtra& ex, int b, int m, int nu, const double* R, int NR,
                                            const double* d, double* fz, double* rhoL, int tj, int rlo, int nP, double sq,
                                            int max_row, double mu, double kT, const double* __restrict__ Hval,
                                            const double* __restrict__ SvalH, double* __restrict__ rho,
                                            double* __restrict__ e_seed, double* __restrict__ n_seed,
                                            int32_t* __restrict__ nu_eff_out, double* eps_b, double* w_b, double* zc) {
    const int tid = threadIdx.x % NT;
    if (ex.mode == 2) {   // Eq. 3 with the inner-product signs: sum_alpha s_alpha (e_j.v_alpha) window_alpha
        const double lo = ex.win[1], hi = ex.win[2];
        for (int a = tid; a < m; a += NT) {
            const double c = R[a * NR + 1 + tj] * level_window(d[a], lo, hi, ex.sigma);
            fz[a] = R[a * NR + NR - 1] >= 0.0 ? c : -c;
        }
        group_sync<NT>();
        if (tid == 0) {
            double phi = 0.0;
            for (int a = 0; a < m; ++a) phi += fz[a];
            ex.phi[b] = phi;
            nu_eff_out[b] = m;
        }
        return;
    }
    if (zc != nullptr) {
        double* zb = zc + (int64_t)b * nu * max_row;
        for (int idx = tid; idx < m * nP; idx += NT) {
            const int a = idx / nP, t = idx - a * nP;
            zb[a * max_row + t] = R[a * NR + 1 + t];
        }
        for (int a = tid; a < m; a += NT) {
            eps_b[a] = d[a];
            w_b[a] = sq * R[a * NR] * R[a * NR + 1 + tj];
        }
        for (int a = m + tid; a < nu; a += NT) {
            eps_b[a] = 0.0;
            w_b[a] = 0.0;
        }
        if (tid == 0) nu_eff_out[b] = m;
        return;
    }
    for (int a = tid; a < m; a += NT) {
        const double ea = d[a];
        const double zj = R[a * NR + 1 + tj];
        fz[a] = fermi_occ(ea, mu, kT) * zj;
        if (eps_b) eps_b[a] = ea;
        if (w_b) w_b[a] = sq * R[a * NR] * zj;
    }
    for (int a = m + tid; a < nu; a += NT) {
        if (eps_b) eps_b[a] = 0.0;
        if (w_b) w_b[a] = 0.0;
    }
    group_sync<NT>();
    for (int cb = 0; cb < nP; cb += NT / 8) {
        const int t = cb + (tid >> 3), pi = tid & 7;
        double s = 0.0;
        if (t < nP)
            for (int a = pi; a < m; a += 8) s += fz[a] * R[a * NR + 1 + t];
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        if (t < nP && pi == 0) {
            const double r = 2.0 * s;
            rho[rlo + t] = r;
            rhoL[t] = r;
        }
    }
    group_sync<NT>();
    if (tid < 64) {   // nP <= 63
        const bool in = tid < nP;
        const double r = in ? rhoL[tid] : 0.0;
        const double E = wave_sum(r * (in ? Hval[rlo + tid] : 0.0)), N = wave_sum(r * (in ? SvalH[rlo + tid] : 0.0));
        if (tid == 0) {
            e_seed[b] = E;
            n_seed[b] = N;
            nu_eff_out[b] = m;
        }
    }
}

// The outputs of a seed whose eigensolve did not converge: NU_NOCONV, and NaN in every output.
template <int NT>
__device__ __forceinline__ void eig_failed(const EigExtra& ex, int b, int m, int nu, int rlo, int nP, double* __restrict__ rho,
                                           double* __restrict__ e_seed, double* __restrict__ n_seed,
                                           int32_t* __restrict__ nu_eff_out, double* eps_b, double* w_b, const double* zc) {
    const int tid = threadIdx.x % NT;
    const double nan = __builtin_nan("");
    if (ex.mode == 1) {
        for (int idx = tid; idx < m * m; idx += NT) {
            const int a = idx / m, c = idx - a * m;
            ex.Y[((int64_t)b * nu + a) * nu + c] = nan;
        }
    } else if (ex.mode == 2) {
        if (tid == 0) ex.phi[b] = nan;
    } else if (zc == nullptr) {
        for (int t = tid; t < nP; t += NT) rho[rlo + t] = nan;
        if (tid == 0) {
            e_seed[b] = nan;
            n_seed[b] = nan;
        }
    }
    for (int a = tid; a < nu; a += NT) {
        if (eps_b) eps_b[a] = nan;
        if (w_b) w_b[a] = nan;
    }
    if (tid == 0) nu_eff_out[b] = NU_NOCONV;
}

// A seed without a subspace (outside the matrix, S not positive definite, padding).
template <int NT>
__device__ __forceinline__ void eig_empty(int b, int m, int nu, double* __restrict__ e_seed, double* __restrict__ n_seed,
                                          int32_t* __restrict__ nu_eff_out, double* eps_b, double* w_b) {
    if (threadIdx.x % NT == 0) {
        nu_eff_out[b] = m;
        e_seed[b] = 0.0;
        n_seed[b] = 0.0;
    }
    for (int a = threadIdx.x % NT; a < nu; a += NT) {
        if (eps_b) eps_b[a] = 0.0;
        if (w_b) w_b[a] = 0.0;
    }
}

template <bool LDS_A>
__global__ __launch_bounds__(EIG_WG) void k_eig(EigExtra ex, int nseeds, const int32_t* __restrict__ seeds, int nu,
                                            double* __restrict__ h, const int32_t* __restrict__ nu_eff_blk,
                                            const double* __restrict__ Kp, const int32_t* __restrict__ Hrp,
                                            const int32_t* __restrict__ Hcol, const double* __restrict__ Hval,
                                            const double* __restrict__ SvalH, const double* __restrict__ diagS,
                                            int max_row, double mu, double kT, double* __restrict__ rho,
                                            double* __restrict__ e_seed, double* __restrict__ n_seed,
                                            int32_t* __restrict__ nu_eff_out, double* __restrict__ eps_out,
                                            double* __restrict__ w_out, double* __restrict__ zc) {
    extern __shared__ double smem[];
    const int b = blockIdx.x;
    if (b >= nseeds) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = nu_eff_blk[b];
    double* eps_b = eps_out ? eps_out + (int64_t)b * nu : nullptr;
    double* w_b = w_out ? w_out + (int64_t)b * nu : nullptr;
    if (m <= 0) {
        eig_empty<EIG_WG>(b, m, nu, e_seed, n_seed, nu_eff_out, eps_b, w_b);
        return;
    }
    const int j = seeds[b];
    const int rlo = Hrp[j];
    const int nP = Hrp[j + 1] - rlo;
    // columns of R: [e_1 | K[P(j),:]^T] (+ [K^T v_ref] in mode 2), or [e_1 | I_m] in mode 1
    const int NR = ex.mode == 1 ? m + 1 : (ex.mode == 2 ? nP + 2 : nP + 1);

    double* A;
    int ld;
    double* p = smem;
    if constexpr (LDS_A) {
        A = p;
        ld = m | 1;   // odd: the Jacobi steps' column accesses spread over the banks
        p += (size_t)nu * (nu + 1);
    } else {
        A = h + (int64_t)b * nu * nu;
        ld = nu;
    }
    double* Rl = p;
    double* R = ex.mode == 1 ? ex.Rg + (int64_t)b * nu * (nu + 1) : Rl;
    p += (size_t)nu * (max_row + (ex.mode == 2 ? 2 : 1));
    double* d = p;
    p += nu;
    double* e = p;
    p += nu;
    double* v = p;
    p += nu;
    double* q = p;
    p += nu;
    double* red = p;
    p += 8;
    p += 72;
    double* rhoL = p;
    p += 64;
    int* tjp = reinterpret_cast<int*>(p);

    // A = K^T H K from its computed upper triangle (h[b][k][n], k <= n), which is all the Jacobi
    // iteration keeps (in place in h when A does not fit in LDS).
    const double* hb = h + (int64_t)b * nu * nu;
    if constexpr (LDS_A) {
        for (int r = wave; r < m; r += EIG_WAVES)
            for (int c = r + lane; c < m; c += 64) A[r * ld + c] = hb[(int64_t)r * nu + c];
    }
    for (int idx = tid; idx < m * NR; idx += EIG_WG) {
        const int k = idx / NR, c = idx - k * NR;
        double r0;
        if (c == 0) r0 = k == 0 ? 1.0 : 0.0;
        else if (ex.mode == 1) r0 = k == c - 1 ? 1.0 : 0.0;
        else if (c <= nP) r0 = Kp[((int64_t)b * nu + k) * max_row + (c - 1)];
        else r0 = ex.pref[(int64_t)k * ex.pB + b];
        R[idx] = r0;
    }
    if (tid < nP && Hcol[rlo + tid] == j) *tjp = tid;
    __syncthreads();

    // Jacobi: A's diagonal becomes the levels, R's rows the vectors' components (cs, sn, tt in v, q, e)
    int* failp = tjp + 1;
    {
        // a separate call for R in global memory (mode 1), so that the LDS case compiles to LDS instructions
        const int f = ex.mode == 1 ? jacobi_eig(A, ld, m, R, NR, v, q, e, tjp + 2, ex.eig_max_sweeps)
                                   : jacobi_eig(A, ld, m, Rl, NR, v, q, e, tjp + 2, ex.eig_max_sweeps);
        __syncthreads();
        for (int a = tid; a < m; a += EIG_WG) d[a] = A[a * ld + a];
        if (tid == 0) *failp = f;
    }
    __syncthreads();
    if (*failp != 0) {
        eig_failed<EIG_WG>(ex, b, m, nu, rlo, nP, rho, e_seed, n_seed, nu_eff_out, eps_b, w_b, zc);
        return;
    }

    const double sq = sqrt(diagS[j]);
    if (ex.mode == 1) {   // the full subspace eigenvectors y_alpha and levels
        for (int idx = tid; idx < m * m; idx += EIG_WG) {
            const int a = idx / m, c = idx - a * m;
            ex.Y[((int64_t)b * nu + a) * nu + c] = R[a * NR + 1 + c];
        }
        for (int a = tid; a < nu; a += EIG_WG) eps_b[a] = a < m ? d[a] : 0.0;
        if (tid == 0) nu_eff_out[b] = m;
        return;
    }
    eig_results<EIG_WG>(ex, b, m, nu, R, NR, d, q, rhoL, *tjp, rlo, nP, sq, max_row, mu, kT, Hval, SvalH, rho, e_seed, n_seed,
                        nu_eff_out, eps_b, w_b, zc);
}

// ---------------------------------------------------------------------------
// The eigensolve of the ordinary passes: Householder reduction of A to tridiagonal form (k_tri, k_tri_big), then the
// implicit QL iteration (k_ql). Every reflector and rotation is applied to R's columns K[P(j), :]^T (and K^T v_ref) as
// well; the reflectors leave the first basis vector alone, so R's column e_1 enters at the QL iteration. The Jacobi
// iteration above takes about ten sweeps of m - 1 steps over all of A; this takes one reduction over A and about
// 0.85 m^2 rotations of two rows of R.
//
// k_tri: A's rows and, below them, R's columns as further rows, in the registers of 512 threads (m <= 16 CJ, at most
// 32 RI rows in all): thread (tr, tc) holds rows tr + 32 i and columns tc + 16 j. With v = 0 and w = tau p on the
// further rows, p = A v and A -= v w^T + w v^T are one formula for all rows. The column of a step and the products p
// go through LDS, twice buffered, two barriers a step. The reflector 1 - tau v v^T keeps v unscaled (v is the column
// but for its first element, tau = 1 / (|beta| (|beta| + |alpha|))), so that the products need not wait for a
// reciprocal. d and e leave in the first two rows of the seed's h, R's columns where they were. What bounds it: the
// latency of a step (two sums over a wavefront, one over 16 lanes, a reciprocal square root, two barriers); 512
// threads instead of 256 with twice the elements each halve it and leave room for two workgroups on a compute unit
// (nu = 100, 1024 seeds: 1.30 -> 0.64 ms).
constexpr int TRI_TH = 512;
template <int CJ, int RI>
__global__ __launch_bounds__(TRI_TH, RI <= 4 ? 4 : 2) void k_tri(EigExtra ex, const int32_t* __restrict__ seeds, int nu,
                                                double* __restrict__ h, const int32_t* __restrict__ nu_eff_blk,
                                                double* __restrict__ Kp, const int32_t* __restrict__ Hrp, int max_row,
                                                double* __restrict__ pref) {
    constexpr int NX = 16 * CJ;               // elements of a column (zero past m)
    __shared__ double xs[2][NX], ps[2][32 * RI], dd[NX], ee[NX], amx[TRI_TH / 64];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tr = tid >> 4, tc = tid & 15;
    const int m = nu_eff_blk[b];
    if (m <= 0) return;
    const int j0 = seeds[b], nP = Hrp[j0 + 1] - Hrp[j0], nR = nP + (ex.mode == 2 ? 1 : 0);
    double* hb = h + (int64_t)b * nu * nu;
    double* kb = Kp + (int64_t)b * nu * max_row;
    double A[RI][CJ];
    double mx = 0.0;
#pragma unroll
    for (int ii = 0; ii < RI; ++ii)
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj) {
            const int i = tr + 32 * ii, c = tc + 16 * jj;
            double v = 0.0;
            if (c < m) {
                if (i < m) v = hb[(int64_t)min(i, c) * nu + max(i, c)];
                else if (i - m < nP) v = kb[(int64_t)c * max_row + (i - m)];
                else if (i - m < nR) v = pref[(int64_t)c * ex.pB + b];
                if (i < m) mx = fmax(mx, fabs(v));
            }
            A[ii][jj] = v;
        }
    // A scaled to a largest entry in [1/2, 1), so that the squares of a step stay in range
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (lane == 0) amx[wave] = mx;
    __syncthreads();
    mx = 0.0;
#pragma unroll
    for (int i = 0; i < TRI_TH / 64; ++i) mx = fmax(mx, amx[i]);
    const int sc = mx > 0.0 && mx < INFINITY ? -ilogb(mx) - 1 : 0;
#pragma unroll
    for (int ii = 0; ii < RI; ++ii)
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj)
            if (tr + 32 * ii < m) A[ii][jj] = ldexp(A[ii][jj], sc);
    for (int k = 0; k + 2 < m; ++k) {
        double* x = xs[k & 1];
        double* p = ps[k & 1];
        // column k below the diagonal, zeros elsewhere
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj)
            if (jj == (k >> 4) && tc == (k & 15)) {
#pragma unroll
                for (int ii = 0; ii < RI; ++ii) {
                    const int i = tr + 32 * ii;
                    if (i == k) dd[k] = A[ii][jj];
                    if (i < NX) x[i] = i > k && i < m ? A[ii][jj] : 0.0;
                }
            }
        __syncthreads();
        double sg = 0.0;                       // the entries below the subdiagonal; every wavefront the same
        for (int i = lane; i < NX; i += 64) {
            const double xi = i == k + 1 ? 0.0 : x[i];
            sg = fma(xi, xi, sg);
        }
        sg = wave_sum(sg);
        const double al = x[k + 1];
        double beta = al, tau = 0.0, v1 = 0.0;
        // else the column is in form (to 1e-145 of A's scale). Not by comparing n2 with al^2: entries up to 1e-8 |al|,
        // which a small overlap leaves in every column, are below n2's last place and would be dropped
        const bool refl = sg > 1e-290;
        if (refl) {
            const double n2 = fma(al, al, sg), r = n2 * rsqrt_nr(n2);
            beta = -copysign(r, al);
            v1 = al - beta;
            tau = recip(fma(r, fabs(al), n2));
        }
        if (tid == 0) ee[k] = beta;
        auto vat = [&](int i) { return refl ? (i == k + 1 ? v1 : x[i]) : 0.0; };
        double vj[CJ], sr[RI];
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj) vj[jj] = vat(tc + 16 * jj);
        // p = A v: over the thread's columns, then over the 16 threads of a row
#pragma unroll
        for (int ii = 0; ii < RI; ++ii) {
            sr[ii] = 0.0;
            if (32 * ii + 31 <= k) continue;   // rows done with (uniform)
#pragma unroll
            for (int jj = 0; jj < CJ; ++jj) sr[ii] = fma(A[ii][jj], vj[jj], sr[ii]);
        }
#pragma unroll
        for (int ii = 0; ii < RI; ++ii) {
            if (32 * ii + 31 <= k) continue;
            sr[ii] += dpp_move<0xb1>(sr[ii]);
            sr[ii] += dpp_move<0x4e>(sr[ii]);
            sr[ii] += dpp_move<0x141>(sr[ii]);
            sr[ii] += dpp_move<0x140>(sr[ii]);
            if (tc == 0) p[tr + 32 * ii] = sr[ii];
        }
        __syncthreads();
        double pv = 0.0, wj[CJ];
        for (int i = lane; i < NX; i += 64) pv += i > k ? p[i] * vat(i) : 0.0;
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj) wj[jj] = p[tc + 16 * jj];
        pv = wave_sum(pv);
        const double kk = 0.5 * tau * tau * pv;   // w = tau p - kk v
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj) wj[jj] = fma(tau, wj[jj], -kk * vj[jj]);
#pragma unroll
        for (int ii = 0; ii < RI; ++ii) {
            if (32 * ii + 31 <= k) continue;
            const int i = tr + 32 * ii;
            const double vi = i < m ? vat(i < NX ? i : 0) : 0.0, wi = fma(tau, sr[ii], -kk * vi);
#pragma unroll
            for (int jj = 0; jj < CJ; ++jj) A[ii][jj] = fma(-vi, wj[jj], fma(-wi, vj[jj], A[ii][jj]));
        }
    }
    __syncthreads();
#pragma unroll
    for (int ii = 0; ii < RI; ++ii)
#pragma unroll
        for (int jj = 0; jj < CJ; ++jj) {
            const int i = tr + 32 * ii, c = tc + 16 * jj;
            if (i < m && i == c && i + 2 >= m) dd[i] = A[ii][jj];
            if (i < m && m >= 2 && i == m - 1 && c == m - 2) ee[c] = A[ii][jj];
            if (c < m && i >= m) {
                if (i - m < nP) kb[(int64_t)c * max_row + (i - m)] = A[ii][jj];
                else if (i - m < nR) pref[(int64_t)c * ex.pB + b] = A[ii][jj];
            }
        }
    __syncthreads();
    for (int i = tid; i < m; i += TRI_TH) hb[i] = ldexp(dd[i], -sc);
    for (int i = tid; i + 1 < m; i += TRI_TH) hb[nu + i] = ldexp(ee[i], -sc);
}

// The same reduction for larger m, with A (both triangles, scaled) in global memory in place of h and R's columns as
// rows in LDS: a pass per step that applies the step before's update to the remaining rows and multiplies them by the
// new reflector's vector, one wavefront per row. The next column is formed from the updated row before the pass, so
// that each element of A crosses the L2 once each way per step. Three barriers a step.
constexpr int TRI_WG = 1024;
inline size_t tri_big_lds(int nu, int nr) { return ((size_t)nr * nu + 5 * (size_t)nu + nr + 16 + 2) * 8; }
__global__ __launch_bounds__(TRI_WG) void k_tri_big(EigExtra ex, const int32_t* __restrict__ seeds, int nu, double* h,
                                                    const int32_t* __restrict__ nu_eff_blk, double* Kp,
                                                    const int32_t* __restrict__ Hrp, int max_row, double* pref) {
    extern __shared__ double smem[];
    constexpr int NW = TRI_WG / 64;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = nu_eff_blk[b];
    if (m <= 0) return;
    const int j0 = seeds[b], nP = Hrp[j0 + 1] - Hrp[j0], nR = nP + (ex.mode == 2 ? 1 : 0);
    double* A = h + (int64_t)b * nu * nu;
    double* kb = Kp + (int64_t)b * nu * max_row;
    double* Rt = smem;                       // [nR][m]
    double* v2 = Rt + (size_t)nR * nu;       // two reflector vectors
    double* w = v2 + 2 * nu;
    double* x = w + nu;
    double* p = x + nu;                      // [m + nR]
    double* amx = p + nu + nR;
    double mx = 0.0;
    for (int i = wave; i < m; i += NW)
        for (int c = i + lane; c < m; c += 64) mx = fmax(mx, fabs(A[(int64_t)i * nu + c]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (lane == 0) amx[wave] = mx;
    __syncthreads();
    mx = 0.0;
    for (int i = 0; i < NW; ++i) mx = fmax(mx, amx[i]);
    const int sc = mx > 0.0 && mx < INFINITY ? -ilogb(mx) - 1 : 0;
    for (int i = wave; i < m; i += NW)
        for (int c = i + lane; c < m; c += 64) {
            const double v = ldexp(A[(int64_t)i * nu + c], sc);
            A[(int64_t)i * nu + c] = v;
            A[(int64_t)c * nu + i] = v;
            if (i == 0) x[c] = v;
        }
    for (int idx = tid; idx < nR * m; idx += TRI_WG) {
        const int k = idx / nR, t = idx - k * nR;
        Rt[(int64_t)t * m + k] = t < nP ? kb[(int64_t)k * max_row + t] : pref[(int64_t)k * ex.pB + b];
    }
    double dkeep = 0.0, ekeep = 0.0;   // thread k keeps d_k and e_k (m <= TRI_WG: the launcher)
    __syncthreads();
    double ptau = 0.0;
    for (int k = 0; k + 2 < m; ++k) {
        double* v = v2 + (k & 1) * nu;
        const double* vp = v2 + ((k + 1) & 1) * nu;
        double sg = 0.0;
        for (int i = k + 2 + lane; i < m; i += 64) sg += x[i] * x[i];
        sg = wave_sum(sg);
        const double al = x[k + 1];
        double beta = al, tau = 0.0, scal = 0.0;
        if (sg > 0.0) {
            const double n2 = fma(al, al, sg);
            beta = -copysign(n2 * rsqrt_nr(n2), al);
            tau = (beta - al) * recip(beta);
            scal = recip(al - beta);
        }
        if (tid == k) {
            dkeep = x[k];
            ekeep = beta;
        }
        for (int i = k + 1 + tid; i < m; i += TRI_WG) v[i] = i == k + 1 ? 1.0 : x[i] * scal;
        __syncthreads();
        // rows k + 1 .. m - 1 of A, then R's columns: the step before's update, and the product with v
        for (int r = k + 1 + wave; r < m + nR; r += NW) {
            double* a = r < m ? A + (int64_t)r * nu : nullptr;
            double* l = Rt + (int64_t)(r - m) * m;
            const double vr = k > 0 && r < m ? vp[r] : 0.0, wr = k > 0 ? (r < m ? w[r] : ptau * p[r]) : 0.0;
            double s = 0.0;
            if (r < m) {
#pragma unroll 4
                for (int c = k + 1 + lane; c < m; c += 64) {
                    double t = a[c];
                    if (k > 0) {
                        t = fma(-vr, w[c], fma(-wr, vp[c], t));
                        a[c] = t;
                    }
                    s = fma(t, v[c], s);
                }
            } else {
                // (column k of R, which the step before's update touches too, takes no further ones)
                if (k > 0 && lane == 0) l[k] = fma(-wr, vp[k], l[k]);
                for (int c = k + 1 + lane; c < m; c += 64) {
                    double t = l[c];
                    if (k > 0) {
                        t = fma(-wr, vp[c], t);
                        l[c] = t;
                    }
                    s = fma(t, v[c], s);
                }
            }
            s = wave_sum(s);
            if (lane == 0) p[r] = s;
        }
        __syncthreads();
        double pv = 0.0;
        for (int i = k + 1 + lane; i < m; i += 64) pv += p[i] * v[i];
        pv = wave_sum(pv);
        const double kk = 0.5 * tau * tau * pv, w1 = tau * p[k + 1] - kk;   // v_{k+1} = 1
        for (int c = k + 1 + tid; c < m; c += TRI_WG) {
            const double wc = tau * p[c] - kk * v[c];
            w[c] = wc;
            x[c] = A[(int64_t)(k + 1) * nu + c] - wc - w1 * v[c];
        }
        ptau = tau;
        __syncthreads();
    }
    // the last two rows and R's columns with the last update
    const double* vp = v2 + ((m + 1) & 1) * nu;   // of step m - 3
    if (m >= 3)
        for (int idx = tid; idx < nR * 2; idx += TRI_WG) {
            const int t = idx / 2, c = m - 2 + idx % 2;
            Rt[(int64_t)t * m + c] = fma(-ptau * p[m + t], vp[c], Rt[(int64_t)t * m + c]);
        }
    __syncthreads();
    double dl = 0.0;
    if (tid == 0) {
        dl = A[(int64_t)(m - 1) * nu + m - 1];
        if (m >= 3) dl -= 2.0 * vp[m - 1] * w[m - 1];
    }
    const double dm2 = m >= 2 ? x[m - 2] : 0.0, em2 = m >= 2 ? x[m - 1] : 0.0;
    __syncthreads();
    if (tid + 2 < m) {
        A[tid] = ldexp(dkeep, -sc);
        A[nu + tid] = ldexp(ekeep, -sc);
    }
    if (tid == 0) {
        A[m - 1] = ldexp(dl, -sc);
        if (m >= 2) {
            A[m - 2] = ldexp(dm2, -sc);
            A[nu + m - 2] = ldexp(em2, -sc);
        }
    }
    for (int idx = tid; idx < nR * m; idx += TRI_WG) {
        const int k = idx / nR, t = idx - k * nR;
        if (t < nP) kb[(int64_t)k * max_row + t] = Rt[(int64_t)t * m + k];
        else pref[(int64_t)k * ex.pB + b] = Rt[(int64_t)t * m + k];
    }
}

// Implicit QL iteration on the tridiagonal (d, e) of a seed with Wilkinson shifts, one wavefront per seed: every lane
// carries the recurrence of the rotations, lane c applies them to column c of R (rows i + 1 and i of R; row i stays in
// a register for the next rotation, which takes rows i and i - 1). The next d, e and row of R are requested one
// rotation ahead. What bounds it: about 1.1 m^2 rotations in sequence, each 24 FP64 operations and a dozen others that one
// wavefront issues one after the other (an FP64 operation every seven cycles: 269 cycles a rotation at nu = 100; the
// recurrence's dependent chain is shorter), so the seeds of a launch share the chip: four to a workgroup, one on each
// SIMD. All control is kept in scalar registers (the dimension, the block's ends and addresses are the same in every
// lane) and the underflow check out of the loop: with masks, per-lane address products and selects a rotation took 350
// cycles (nu = 30, 256 seeds: 193 us, now 151; nu = 100, 1024 seeds: 1.61 ms, now 1.19; nu = 300, 64 seeds: 12.5, now
// 8.5).
constexpr int QL_MAX_ITER = 60;   // iterations allowed per level (about two are needed)
inline size_t ql_lds_bytes(int nu, int nr) { return (((size_t)nu * nr + 3 * (size_t)nu + 66) * 8 + 15) & ~(size_t)15; }
__global__ __launch_bounds__(256) void k_ql(EigExtra ex, int nseeds, const int32_t* __restrict__ seeds, int nu,
                                           const double* __restrict__ h, const int32_t* __restrict__ nu_eff_blk,
                                           const double* __restrict__ Kp, const int32_t* __restrict__ Hrp,
                                           const int32_t* __restrict__ Hcol, const double* __restrict__ Hval,
                                           const double* __restrict__ SvalH, const double* __restrict__ diagS,
                                           int max_row, double mu, double kT, double* __restrict__ rho,
                                           double* __restrict__ e_seed, double* __restrict__ n_seed,
                                           int32_t* __restrict__ nu_eff_out, double* __restrict__ eps_out,
                                           double* __restrict__ w_out, double* __restrict__ zc,
                                           int seed_doubles) {
    extern __shared__ double smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.x * (blockDim.x >> 6) + wave;
    if (b >= nseeds) return;
    const int m = nu_eff_blk[b];
    double* eps_b = eps_out ? eps_out + (int64_t)b * nu : nullptr;
    double* w_b = w_out ? w_out + (int64_t)b * nu : nullptr;
    if (m <= 0) {
        eig_empty<64>(b, m, nu, e_seed, n_seed, nu_eff_out, eps_b, w_b);
        return;
    }
    const int j = seeds[b], rlo = Hrp[j], nP = Hrp[j + 1] - rlo;
    const int NR = nP + 1 + (ex.mode == 2 ? 1 : 0);
    // {d_i, e_i}; the entry in front of the first is read ahead of the last rotation and not used
    double2* de = reinterpret_cast<double2*>(smem + (size_t)wave * seed_doubles) + 1;
    double* fz = reinterpret_cast<double*>(de + nu);
    double* rhoL = fz + nu;
    double* R = rhoL + 64;
    const double* hb = h + (int64_t)b * nu * nu;
    int tj = 0;
    {
        const unsigned long long at = __ballot(lane < nP && Hcol[rlo + (lane < nP ? lane : 0)] == j);
        if (at) tj = __ffsll(at) - 1;
    }
    const double* Rl = R + (lane < NR ? lane : 0);
    double* Rw = R + (lane < NR ? lane : 0);   // lanes past the columns repeat column 0
    bool fail = false;
    int sc = 0;
    unsigned xmin = ~0u;   // high word of the smallest f^2 + g^2 met
    // SAFE, the second time, only when some f^2 + g^2 underflowed: with the check on every rotation
    auto iterate = [&](auto safe_form) {
        constexpr bool SAFE = decltype(safe_form)::value;
        double mx = 0.0;
        for (int i = lane; i < m; i += 64) {
            const double di = hb[i], ei = i + 1 < m ? hb[nu + i] : 0.0;
            mx = fmax(mx, fmax(fabs(di), fabs(ei)));
            de[i] = make_double2(di, ei);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        sc = mx > 0.0 && mx < INFINITY ? -ilogb(mx) - 1 : 0;
        for (int i = lane; i < m; i += 64) de[i] = make_double2(ldexp(de[i].x, sc), ldexp(de[i].y, sc));
        // lane = column: e_1, the gathered rows, and v_ref's products; eight rows in flight
        const double* col = lane >= 1 && lane <= nP ? Kp + (int64_t)b * nu * max_row + (lane - 1) : ex.pref + b;
        const int64_t cst = lane <= nP ? max_row : ex.pB;
        const bool mem = lane >= 1 && lane < NR;
        for (int k0 = 0; k0 < m; k0 += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k0 + u == 0 ? 1.0 : 0.0;
            if (mem) {
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = col[min(k0 + u, m - 1) * cst];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (lane < NR && k0 + u < m) R[(k0 + u) * NR + lane] = v[u];
        }
        wave_sync();
        fail = false;
        for (int l = 0; l + 1 < m && !fail; ++l) {
            for (int iter = 0;; ++iter) {
                // the first negligible e_i, i >= l: the block l .. mm is unreduced
                int mm = m - 1;
                for (int base = l; base < m - 1; base += 64) {
                    const int i = base + lane;
                    bool small = false;
                    if (i < m - 1) small = fabs(de[i].y) <= DBL_EPSILON * (fabs(de[i].x) + fabs(de[i + 1].x)) + 1e-32;
                    const unsigned long long bal = __ballot(small);
                    if (bal) {
                        mm = base + __ffsll(bal) - 1;
                        break;
                    }
                }
                if (mm == l) break;
                if (iter == QL_MAX_ITER) {
                    fail = true;
                    break;
                }
                const double2 del = de[l];
                double2 dei = de[mm - 1];
                double di1 = de[mm].x;
                double hr = Rl[mm * NR], ri = Rl[(mm - 1) * NR];
                // shift: e_l / (g + sign(g) sqrt(1 + g^2)), g = (d_{l+1} - d_l) / (2 e_l); e_l / (2 g) for a huge g
                double g = (de[l + 1].x - del.x) * recip(2.0 * del.y);
                const double ag = fabs(g), q1 = fma(g, g, 1.0);
                const double den = ag > 1e150 ? 2.0 * ag : ag + q1 * rsqrt_nr(q1);
                g = di1 - del.x + copysign(del.y * recip(den), ag == 0.0 ? del.y : del.y * (g < 0.0 ? -1.0 : 1.0));
                double s = 1.0, c = 1.0, p = 0.0;
                double2* dp = de + mm;
                double* rp = Rw + mm * NR;
#pragma unroll 4
                for (int i = mm - l; i > 0; --i) {
                    const double2 den2 = dp[-2];
                    const double rn = rp[-2 * NR];
                    const double f = s * dei.y, bb = c * dei.y, x = fma(g, g, fma(f, f, 1e-300));
                    const double y = __builtin_amdgcn_rsq(x), xy = x * y, u = fma(-xy, y, 1.0);
                    // third-order step: 23 bits to full precision
                    const double cr = fma(u, fma(0.375, u, 0.5), 1.0), yc = y * cr;
                    double r = xy * cr;
                    s = f * yc;
                    c = g * yc;
                    xmin = min(xmin, (unsigned)(__builtin_bit_cast(uint64_t, x) >> 32));
                    if (SAFE && x < 1e-290) {   // the identity: the matrix splits here
                        r = s = 0.0;
                        c = 1.0;
                    }
                    g = di1 - p;
                    const double rr = fma(c, bb + bb, (dei.x - g) * s);
                    p = s * rr;
                    *dp = make_double2(g + p, r);
                    g = fma(c, rr, -bb);
                    *rp = fma(s, ri, c * hr);
                    hr = fma(c, ri, -(s * hr));
                    di1 = dei.x;
                    dei = den2;
                    ri = rn;
                    --dp;
                    rp -= NR;
                }
                de[l] = make_double2(di1 - p, g);
                de[mm].y = 0.0;
                Rw[l * NR] = hr;
                wave_sync();
            }
        }
    };
    iterate(std::false_type{});
    if (xmin <= 0x03b8f2b0u) iterate(std::true_type{});   // 1e-290
    if (fail) {
        eig_failed<64>(ex, b, m, nu, rlo, nP, rho, e_seed, n_seed, nu_eff_out, eps_b, w_b, zc);
        return;
    }
    // the levels side by side (d_i moves to or behind a place that is read already)
    double* d = reinterpret_cast<double*>(de);
    for (int base = 0; base < m; base += 64) {
        const double v = ldexp(de[min(base + lane, m - 1)].x, -sc);
        wave_sync();
        if (base + lane < m) d[base + lane] = v;
        wave_sync();
    }
    eig_results<64>(ex, b, m, nu, R, NR, d, fz, rhoL, tj, rlo, nP, sqrt(diagS[j]), max_row, mu, kT, Hval, SvalH, rho, e_seed,
                    n_seed, nu_eff_out, eps_b, w_b, zc);
}

LaunchInfo launch_eig(int nseeds, const int32_t* seeds, int nu, double* h, const int32_t* nu_eff_blk,
                      double* Kp, const int32_t* Hrp, const int32_t* Hcol, const double* Hval,
                      const double* SvalH, const double* diagS, int max_row, double mu, double kT, double* rho,
                      double* e_seed, double* n_seed, int32_t* nu_eff_out, double* eps_out, double* w_out,
                      double* zc, const EigExtra& ex, hipStream_t s) {
    const int rcols = max_row + (ex.mode == 2 ? 1 : 0);   // R's LDS share (mode 1 keeps R in global memory)
    LaunchInfo li;
    li.wgs = nseeds;
    const double nv = (double)nu;
    li.bytes = (double)nseeds * (nv * nv * 8.0 + nv * max_row * 8.0 + (max_row + 3) * 8.0 * 3);
    li.flops = (double)nseeds * ((4.0 / 3.0) * nv * nv * nv + 4.0 * nv * nv * (max_row + 1));
    // Reduction and QL iteration, except where all eigenvectors are wanted (mode 1: one seed), a cap on Jacobi sweeps
    // was asked for, or a row of R outgrows a wavefront or the reduction's LDS.
    // Measured (ms, Jacobi / this): nu = 30, 256 seeds 0.29 / 0.19; nu = 47, 777 seeds 2.02 / 0.50; nu = 100, 256 seeds
    // 1.71 / 1.39, 1024 seeds 6.6 / 1.9; nu = 300, 64 seeds 112 / 14. The reduction and iteration are the more accurate
    // of the two (rho against LAPACK at nu = 100: 2e-15 against 1.5e-14).
    const size_t big = tri_big_lds(nu, rcols), ql = ql_lds_bytes(nu, rcols + 1);
    if (!ex.jacobi && ex.mode != 1 && rcols + 1 <= 64 && ql <= 160 * 1024 &&
        (nu <= 128 || (nu <= TRI_WG && big <= 160 * 1024))) {
        double* pref = const_cast<double*>(ex.pref);
#define MAR_TRI(CJ, RI)                                                                                          \
    hipLaunchKernelGGL((k_tri<CJ, RI>), dim3(nseeds), dim3(TRI_TH), 0, s, ex, seeds, nu, h, nu_eff_blk, Kp, Hrp, \
                       max_row, pref)
        const int ri = (nu + rcols + 31) / 32;   // rows of 32 threads (rcols <= 63)
        if (nu <= 32) { if (ri <= 2) MAR_TRI(2, 2); else MAR_TRI(2, 3); }
        else if (nu <= 64) { if (ri <= 3) MAR_TRI(4, 3); else MAR_TRI(4, 4); }
        else if (nu <= 96) { if (ri <= 4) MAR_TRI(6, 4); else MAR_TRI(6, 5); }
        else if (nu <= 128) { if (ri <= 4) MAR_TRI(8, 4); else if (ri <= 5) MAR_TRI(8, 5); else MAR_TRI(8, 6); }
        else {
            static std::atomic<uint64_t> done{0};
            allow_full_lds((const void*)k_tri_big, done);
            hipLaunchKernelGGL(k_tri_big, dim3(nseeds), dim3(TRI_WG), big, s, ex, seeds, nu, h, nu_eff_blk, Kp, Hrp, max_row, pref);
        }
#undef MAR_TRI
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void*)k_ql, done);
        // four seeds to a workgroup, one on each SIMD, as far as LDS allows: workgroups of one wavefront shared one
        // SIMD (nu = 100, 1024 seeds: 2.58 -> 1.79 ms)
        int wv = 4;
        while (wv > 1 && wv * ql > 160 * 1024) wv /= 2;
        hipLaunchKernelGGL(k_ql, dim3((nseeds + wv - 1) / wv), dim3(64 * wv), wv * ql, s, ex, nseeds, seeds, nu, h, nu_eff_blk, Kp, Hrp, Hcol, Hval, SvalH,
                           diagS, max_row, mu, kT, rho, e_seed, n_seed, nu_eff_out, eps_out, w_out, zc, (int)(ql / 8));
        return li;
    }
    const bool lds_a = eig_a_fits_lds(nu, rcols);
    const size_t lds = eig_lds_bytes(nu, rcols, lds_a);
    if (lds_a) {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void*)k_eig<true>, done);
        hipLaunchKernelGGL((k_eig<true>), dim3(nseeds), dim3(EIG_WG), lds, s, ex, nseeds, seeds, nu, h, nu_eff_blk, Kp, Hrp,
                           Hcol, Hval, SvalH, diagS, max_row, mu, kT, rho, e_seed, n_seed, nu_eff_out, eps_out, w_out,
                           zc);
    } else {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void*)k_eig<false>, done);
        hipLaunchKernelGGL((k_eig<false>), dim3(nseeds), dim3(EIG_WG), lds, s, ex, nseeds, seeds, nu, h, nu_eff_blk, Kp,
                           Hrp, Hcol, Hval, SvalH, diagS, max_row, mu, kT, rho, e_seed, n_seed, nu_eff_out, eps_out,
                           w_out, zc);
    }
    return li;
}

// ---------------------------------------------------------------------------
// Assembly at a Fermi level held on the device (after k_eig with zc != nullptr):
// the same sums, in the same order, as the fused epilogue of k_eig.
__global__ __launch_bounds__(WG) void k_assemble(int nseeds, const int32_t* __restrict__ seeds, int nu,
                                                 const int32_t* __restrict__ nu_eff, const double* __restrict__ eps,
                                                 const double* __restrict__ zc, int max_row,
                                                 const int32_t* __restrict__ Hrp, const int32_t* __restrict__ Hcol,
                                                 const double* __restrict__ Hval, const double* __restrict__ SvalH,
                                                 const double* __restrict__ mu_p, double kT, double* __restrict__ rho,
                                                 double* __restrict__ e_seed, double* __restrict__ n_seed) {
    __shared__ double fz[MAX_NU_ASSEMBLE];
    __shared__ double rhoL[64];
    __shared__ int tjs;
    const int b = blockIdx.x, tid = threadIdx.x;
    if (b >= nseeds) return;
    const int m = nu_eff[b];
    if (m <= 0) {
        // a seed whose subspace eigensolve did not converge gets NaN outputs, as in k_eig
        const double fill = m == NU_NOCONV ? __builtin_nan("") : 0.0;
        if (m == NU_NOCONV)
            for (int t = Hrp[seeds[b]] + tid; t < Hrp[seeds[b] + 1]; t += WG) rho[t] = fill;
        if (tid == 0) {
            e_seed[b] = fill;
            n_seed[b] = fill;
        }
        return;
    }
    const int j = seeds[b];
    const int rlo = Hrp[j], nP = Hrp[j + 1] - rlo;
    if (tid < nP && Hcol[rlo + tid] == j) tjs = tid;
    __syncthreads();
    const int tj = tjs;
    const double mu = *mu_p;
    const double* zb = zc + (int64_t)b * nu * max_row;
    for (int a = tid; a < m; a += WG) fz[a] = fermi_occ(eps[(int64_t)b * nu + a], mu, kT) * zb[a * max_row + tj];
    __syncthreads();
    for (int cb = 0; cb < nP; cb += WG / 8) {
        const int t = cb + (tid >> 3), pi = tid & 7;
        double s = 0.0;
        if (t < nP)
            for (int a = pi; a < m; a += 8) s += fz[a] * zb[a * max_row + t];
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        s += __shfl_xor(s, 4);
        if (t < nP && pi == 0) {
            const double r = 2.0 * s;
            rho[rlo + t] = r;
            rhoL[t] = r;
        }
    }
    __syncthreads();
    if (tid < 64) {   // nP <= 63
        const bool in = tid < nP;
        const double r = in ? rhoL[tid] : 0.0;
        const double E = wave_sum(r * (in ? Hval[rlo + tid] : 0.0)), N = wave_sum(r * (in ? SvalH[rlo + tid] : 0.0));
        if (tid == 0) {
            e_seed[b] = E;
            n_seed[b] = N;
        }
    }
}

LaunchInfo launch_assemble(int nseeds, const int32_t* seeds, int nu, const int32_t* nu_eff, const double* eps,
                           const double* zc, int max_row, const int32_t* Hrp, const int32_t* Hcol,
                           const double* Hval, const double* SvalH, const double* mu, double kT, double* rho,
                           double* e_seed, double* n_seed, hipStream_t s) {
    LaunchInfo li;
    if (nu > MAX_NU_ASSEMBLE || max_row > 64) {
        li.wgs = -1;
        return li;
    }
    if (nseeds > 0)
        hipLaunchKernelGGL(k_assemble, dim3(nseeds), dim3(WG), 0, s, nseeds, seeds, nu, nu_eff, eps, zc, max_row, Hrp,
                           Hcol, Hval, SvalH, mu, kT, rho, e_seed, n_seed);
    li.wgs = nseeds;
    li.bytes = (double)nseeds * ((double)nu * (max_row + 1) * 8.0 + 3.0 * max_row * 8.0);
    li.flops = (double)nseeds * 2.0 * nu * (max_row + 1);
    return li;
}

// ---------------------------------------------------------------------------
// Fermi level on the device: mu with N(mu) = sum_j 2 sum_alpha f((eps_alpha^(j)
// - mu)/kT) w_alpha^(j) equal to n_target, by bisection on [min eps - 40 kT,
// max eps + 40 kT] over the listed seeds' subspace levels (alpha < nu_eff).
// Every sum runs in a fixed order.
constexpr int MU_WGS = 512;   // workgroups of the level bounds

__device__ __forceinline__ void wg_minmax(double& lo, double& hi, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off));
        hi = fmax(hi, __shfl_xor(hi, off));
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) {
        red[wave] = lo;
        red[4 + wave] = hi;
    }
    __syncthreads();
    lo = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
    hi = fmax(fmax(red[4], red[5]), fmax(red[6], red[7]));
}

__global__ __launch_bounds__(WG) void k_mu_bounds(int64_t nseeds, int nu, const int32_t* __restrict__ nu_eff,
                                                  const double* __restrict__ eps, double* __restrict__ part) {
    __shared__ double red[8];
    double lo = INFINITY, hi = -INFINITY;
    const int64_t npair = nseeds * nu;
    for (int64_t p = (int64_t)blockIdx.x * WG + threadIdx.x; p < npair; p += (int64_t)gridDim.x * WG) {
        const int64_t b = p / nu;
        const int a = (int)(p - b * nu);
        if (a < nu_eff[b]) {
            lo = fmin(lo, eps[p]);
            hi = fmax(hi, eps[p]);
        }
    }
    wg_minmax(lo, hi, red);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = lo;
        part[2 * blockIdx.x + 1] = hi;
    }
}

// Bisection of counts over the levels, LEVEL_D halvings per launch: the midpoints that the next LEVEL_D halvings can
// meet form a binary tree of LEVEL_P points (heap order, left: the lower half). A launch first sums the partial counts
// of the launch before, in a fixed order and in every workgroup alike, and walks that tree to the new interval; then
// it counts at the points of the next tree over its share of the levels. So each halving takes the decision that one
// at a time would, and a search is LEVEL_PASSES launches instead of two per halving (a counting launch of 3-5 us and a
// one-thread sum of up to 512 partials, 10 us; 42 us for three counts). An interval that a launch leaves unchanged has
// collapsed to neighbouring doubles and stays (about 60 halvings); the last kernel finishes the ones that have not.
// Count t (blockIdx.y): the Fermi level's N(mu) or, DOS, n(eta) for k - 1, k - 1/2 and k.
// st[t][pass & 1] = {lo, hi, collapsed}.
constexpr int LEVEL_D = 4, LEVEL_P = (1 << LEVEL_D) - 1, LEVEL_PASSES = 22, LEVEL_WGS = 256, LEVEL_BITS = 200;

struct LevelArgs {
    int64_t nseeds;
    int nu;
    const int32_t* nu_eff;
    const double *eps, *w;
    double width;           // kT, or sigma
    double target[3];
    int nwg;                // workgroups that count (per target)
    const double* bounds;   // [nb][2] partial level bounds
    int nb;
    double* part;           // [2][target][nwg][LEVEL_P]
    double* st;             // [target][2][4]
};

// The LEVEL_P midpoints of [lo, hi] into mid, by the first threads.
__device__ __forceinline__ void level_points(double lo, double hi, double* mid) {
    const int q = threadIdx.x;
    if (q < LEVEL_P) {
        int d = 0;
        while ((2 << d) - 1 <= q) ++d;   // depth of heap node q; its path from the root in the low d bits of q + 1
        for (int i = d - 1; i >= 0; --i) {
            const double m = 0.5 * (lo + hi);
            if (((q + 1) >> i) & 1) lo = m;
            else hi = m;
        }
        mid[q] = 0.5 * (lo + hi);
    }
}

// Counts at the points mid over the levels first, first + step, ... into cnt (a sum per point over the workgroup).
template <bool DOS, int NT>
__device__ __forceinline__ void level_count(const LevelArgs& a, const double* mid, int64_t first, int64_t step, double* red,
                                            double* cnt) {
    double s[LEVEL_P];
#pragma unroll
    for (int q = 0; q < LEVEL_P; ++q) s[q] = 0.0;
    const int64_t npair = a.nseeds * a.nu;
    for (int64_t p = first; p < npair; p += step) {
        const int64_t b = p / a.nu;
        if ((int)(p - b * a.nu) >= a.nu_eff[b]) continue;
        const double e = a.eps[p], w = a.w[p];
#pragma unroll
        for (int q = 0; q < LEVEL_P; ++q)
            s[q] += DOS ? w * smooth_step(mid[q] - e, a.width) : 2.0 * fermi_occ(e, mid[q], a.width) * w;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < LEVEL_P; ++q) {
        const double v = wave_sum(s[q]);
        if (lane == 0) red[wave * LEVEL_P + q] = v;
    }
    __syncthreads();
    if (threadIdx.x < LEVEL_P) {
        double t = 0.0;
        for (int i = 0; i < NT / 64; ++i) t += red[i * LEVEL_P + threadIdx.x];
        cnt[threadIdx.x] = t;
    }
    __syncthreads();
}

// LEVEL_D halvings by the counts at mid's points; run by one thread.
__device__ __forceinline__ void level_walk(const double* mid, const double* cnt, double target, double& lo, double& hi) {
    int q = 0;
    for (int d = 0; d < LEVEL_D; ++d) {
        if (cnt[q] < target) {
            lo = mid[q];
            q = 2 * q + 2;
        } else {
            hi = mid[q];
            q = 2 * q + 1;
        }
    }
}

// The interval at the start of launch `pass` into sh = {lo, hi, collapsed}: from the level bounds (pass 0) or from the
// interval and the partial counts of the launch before.
template <bool DOS, int NT>
__device__ __forceinline__ void level_state(const LevelArgs& a, int pass, int t, double* sh, double* mid, double* red,
                                            double* cnt) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (pass == 0) {
        double lo = INFINITY, hi = -INFINITY;
        for (int g = tid; g < a.nb; g += NT) {
            lo = fmin(lo, a.bounds[2 * g]);
            hi = fmax(hi, a.bounds[2 * g + 1]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o));
            hi = fmax(hi, __shfl_xor(hi, o));
        }
        if (lane == 0) {
            red[2 * wave] = lo;
            red[2 * wave + 1] = hi;
        }
        __syncthreads();
        if (tid == 0) {
            for (int i = 1; i < NT / 64; ++i) {
                lo = fmin(lo, red[2 * i]);
                hi = fmax(hi, red[2 * i + 1]);
            }
            if (!(lo <= hi)) lo = hi = 0.0;   // no levels at all
            sh[0] = DOS ? lo - 1.0 : lo - 40.0 * a.width;
            sh[1] = DOS ? hi + 1.0 : hi + 40.0 * a.width;
            sh[2] = 0.0;
        }
        __syncthreads();
        return;
    }
    const double* prev = a.st + (t * 2 + ((pass - 1) & 1)) * 4;
    if (tid < 3) sh[tid] = prev[tid];
    __syncthreads();
    if (sh[2] != 0.0) return;
    level_points(sh[0], sh[1], mid);
    const double* pt = a.part + ((int64_t)((pass - 1) & 1) * gridDim.y + t) * a.nwg * LEVEL_P;
    // sixteen lanes of workgroups per point, each in order, then the lanes in order
    const int q = tid % 16, r = tid / 16;
    double s = 0.0;
    if (tid < 256 && q < LEVEL_P)
        for (int g = r; g < a.nwg; g += 16) s += pt[(int64_t)g * LEVEL_P + q];
    if (tid < 256) red[tid] = s;
    __syncthreads();
    if (tid < LEVEL_P) {
        double n = 0.0;
        for (int i = 0; i < 16; ++i) n += red[i * 16 + tid];
        cnt[tid] = n;
    }
    __syncthreads();
    if (tid == 0) {
        const double lo = sh[0], hi = sh[1];
        level_walk(mid, cnt, a.target[t], sh[0], sh[1]);
        sh[2] = sh[0] == lo && sh[1] == hi ? 1.0 : 0.0;
    }
    __syncthreads();
}

template <bool DOS>
__global__ __launch_bounds__(WG) void k_level_pass(LevelArgs a, int pass) {
    __shared__ double sh[3], mid[LEVEL_P + 1], cnt[LEVEL_P + 1], red[WG];
    const int t = blockIdx.y;
    level_state<DOS, WG>(a, pass, t, sh, mid, red, cnt);
    if (blockIdx.x == 0 && threadIdx.x < 3) a.st[(t * 2 + (pass & 1)) * 4 + threadIdx.x] = sh[threadIdx.x];
    if (sh[2] != 0.0) return;
    level_points(sh[0], sh[1], mid);
    __syncthreads();
    level_count<DOS, WG>(a, mid, (int64_t)blockIdx.x * WG + threadIdx.x, (int64_t)a.nwg * WG, red, cnt);
    if (threadIdx.x < LEVEL_P)
        a.part[(((int64_t)(pass & 1) * gridDim.y + t) * a.nwg + blockIdx.x) * LEVEL_P + threadIdx.x] = cnt[threadIdx.x];
}

// The rest of the LEVEL_BITS halvings for an interval that has not collapsed (one workgroup per count), and the
// result, the interval's middle, into out[DOS: {eps_k, eta(k - 1), eta(k)}] and out2 (or null).
constexpr int LEVEL_FIN = 1024;
template <bool DOS>
__global__ __launch_bounds__(LEVEL_FIN) void k_level_finish(LevelArgs a, double* out, double* out2) {
    __shared__ double sh[3], mid[LEVEL_P + 1], cnt[LEVEL_P + 1], red[LEVEL_FIN];
    const int t = blockIdx.y;
    level_state<DOS, LEVEL_FIN>(a, LEVEL_PASSES, t, sh, mid, red, cnt);
    for (int done = LEVEL_PASSES * LEVEL_D; done < LEVEL_BITS && sh[2] == 0.0; done += LEVEL_D) {
        __syncthreads();
        level_points(sh[0], sh[1], mid);
        __syncthreads();
        level_count<DOS, LEVEL_FIN>(a, mid, threadIdx.x, LEVEL_FIN, red, cnt);
        if (threadIdx.x == 0) {
            const double lo = sh[0], hi = sh[1];
            level_walk(mid, cnt, a.target[t], sh[0], sh[1]);
            sh[2] = sh[0] == lo && sh[1] == hi ? 1.0 : 0.0;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = 0.5 * (sh[0] + sh[1]);
        out[DOS ? (t == 1 ? 0 : (t == 0 ? 1 : 2)) : 0] = m;
        if (out2) *out2 = m;
    }
}

template <bool DOS>
static LaunchInfo level_search(int64_t nseeds, int nu, const int32_t* nu_eff, const double* eps, const double* w,
                               double width, const double* target, int nt, double* work, double* out, double* out2,
                               hipStream_t s) {
    static_assert(LEVEL_BITS % LEVEL_D == 0 && LEVEL_PASSES * LEVEL_D < LEVEL_BITS && LEVEL_P <= 16, "tree depth");
    const int64_t npair = nseeds * nu;
    const int nb = (int)std::min<int64_t>(MU_WGS, std::max<int64_t>(1, (npair + WG - 1) / WG));
    LevelArgs a{};
    a.nseeds = nseeds;
    a.nu = nu;
    a.nu_eff = nu_eff;
    a.eps = eps;
    a.w = w;
    a.width = width;
    for (int t = 0; t < nt; ++t) a.target[t] = target[t];
    a.nwg = (int)std::min<int64_t>(LEVEL_WGS, nb);
    a.bounds = work;
    a.nb = nb;
    a.st = work + 2 * MU_WGS;
    a.part = a.st + 3 * 2 * 4;
    hipLaunchKernelGGL(k_mu_bounds, dim3(nb), dim3(WG), 0, s, nseeds, nu, nu_eff, eps, work);
    for (int pass = 0; pass < LEVEL_PASSES; ++pass)
        hipLaunchKernelGGL((k_level_pass<DOS>), dim3(a.nwg, nt), dim3(WG), 0, s, a, pass);
    hipLaunchKernelGGL((k_level_finish<DOS>), dim3(1, nt), dim3(LEVEL_FIN), 0, s, a, out, out2);
    LaunchInfo li;
    li.wgs = nb;
    li.bytes = (double)(LEVEL_PASSES + 1) * npair * 20.0;
    li.flops = (double)LEVEL_PASSES * LEVEL_P * nt * npair * 30.0;
    return li;
}

size_t level_search_doubles(int nt) { return 2 * MU_WGS + 3 * 2 * 4 + (size_t)2 * nt * LEVEL_WGS * LEVEL_P; }

LaunchInfo launch_fermi_search(int64_t nseeds, int nu, const int32_t* nu_eff, const double* eps, const double* w,
                               double n_target, double kT, double* work, double* mu, double* mu_out, hipStream_t s) {
    return level_search<false>(nseeds, nu, nu_eff, eps, w, kT, &n_target, 1, work, mu, mu_out, s);
}

// Eigen states (Sec. 3, Eq. 3; Appendix): integrated density of states
//   n(eta) = sum_j sum_alpha w_alpha^(j) F((eta - eps_alpha^(j)) / sigma)
// (F the logistic step; sigma = 0: the unit step, 1/2 at 0), bisected for the
// three counts k - 1, k - 1/2 and k on [min eps - 1, max eps + 1];
// lv = {eta(k - 1/2), eta(k - 1), eta(k)}.
LaunchInfo launch_dos_search(int64_t nseeds, int nu, const int32_t* nu_eff, const double* eps, const double* w,
                             double sigma, int k, double* work, double* lv, hipStream_t s) {
    const double target[3] = {k - 1.0, k - 0.5, (double)k};
    return level_search<true>(nseeds, nu, nu_eff, eps, w, sigma, target, 3, work, lv, nullptr, s);
}

// Contributions c_alpha^(j) = (e_j . v_alpha^(j)) window_alpha of every seed
// (kept rows zc, levels eps) and the reference: the largest |c| (first seed,
// then first alpha, on ties). ref = {position b, alpha, seed j}; refseed[0] = j.
__device__ __forceinline__ void first_largest(double& v, int& at) {   // over a wavefront, the smaller index on ties
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(v, o);
        const int oa = __shfl_xor(at, o);
        if (ov > v || (ov == v && oa < at)) {
            v = ov;
            at = oa;
        }
    }
}

__global__ __launch_bounds__(64) void k_es_contrib(int nseeds, const int32_t* __restrict__ seeds, int nu,
                                                   const int32_t* __restrict__ nu_eff, const double* __restrict__ eps,
                                                   const double* __restrict__ zc, int max_row,
                                                   const int32_t* __restrict__ Hrp, const int32_t* __restrict__ Hcol,
                                                   const double* __restrict__ lv, double sigma,
                                                   double* __restrict__ cmax, int32_t* __restrict__ amax) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int m = nu_eff[b];
    double best = -1.0;
    int ba = 0;
    if (m > 0) {
        const int j = seeds[b];
        const int rlo = Hrp[j], nP = Hrp[j + 1] - rlo;
        const unsigned long long at = __ballot(lane < nP && Hcol[rlo + (lane < nP ? lane : 0)] == j);
        const int tj = at ? __ffsll(at) - 1 : 0;
        const double* zb = zc + (int64_t)b * nu * max_row;
        for (int a = lane; a < m; a += 64) {
            const double c = fabs(zb[a * max_row + tj] * level_window(eps[(int64_t)b * nu + a], lv[1], lv[2], sigma));
            if (c > best) {
                best = c;
                ba = a;
            }
        }
        if (best < 0.0) ba = m;   // a lane without an alpha
        first_largest(best, ba);
    }
    if (lane == 0) {
        cmax[b] = best;
        amax[b] = best < 0.0 ? 0 : ba;
    }
}

__global__ __launch_bounds__(1024) void k_es_argmax(int nseeds, const int32_t* __restrict__ seeds,
                                                    const double* __restrict__ cmax, const int32_t* __restrict__ amax,
                                                    int32_t* __restrict__ ref, int32_t* __restrict__ refseed) {
    __shared__ double vs[16];
    __shared__ int as[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double best = -1.0;
    int bb = nseeds;
    for (int b = tid; b < nseeds; b += 1024)
        if (cmax[b] > best) {
            best = cmax[b];
            bb = b;
        }
    first_largest(best, bb);
    if (lane == 0) {
        vs[wave] = best;
        as[wave] = bb;
    }
    __syncthreads();
    if (tid != 0) return;
    for (int i = 1; i < 16; ++i)
        if (vs[i] > best || (vs[i] == best && as[i] < bb)) {
            best = vs[i];
            bb = as[i];
        }
    if (!(best > -1.0)) bb = 0;   // no contribution at all
    ref[0] = bb;
    ref[1] = nseeds > 0 ? amax[bb] : 0;
    ref[2] = nseeds > 0 ? seeds[bb] : 0;
    refseed[0] = ref[2];
}

LaunchInfo launch_es_reference(int nseeds, const int32_t* seeds, int nu, const int32_t* nu_eff, const double* eps,
                               const double* zc, int max_row, const int32_t* Hrp, const int32_t* Hcol,
                               const double* lv, double sigma, double* cmax, int32_t* amax, int32_t* ref,
                               int32_t* refseed, hipStream_t s) {
    if (nseeds > 0)
        hipLaunchKernelGGL(k_es_contrib, dim3(nseeds), dim3(64), 0, s, nseeds, seeds, nu, nu_eff, eps, zc, max_row, Hrp,
                           Hcol, lv, sigma, cmax, amax);
    hipLaunchKernelGGL(k_es_argmax, dim3(1), dim3(1024), 0, s, nseeds, seeds, cmax, amax, ref, refseed);
    LaunchInfo li;
    li.wgs = nseeds;
    li.bytes = (double)nseeds * nu * 16.0;
    return li;
}

// Reference seed (solved alone, B = 1): pick among its subspace eigenvectors
// the one with the largest |(e_j . v_alpha) window_alpha| (v_alpha = K y_alpha),
// and form v_ref = K y_ref over all rows.
template <typename T>
__global__ __launch_bounds__(WG) void k_es_pick(const T* __restrict__ K, int64_t stride, const int32_t* __restrict__ seed,
                                                int nu, const int32_t* __restrict__ nu_eff,
                                                const double* __restrict__ Y, const double* __restrict__ eps,
                                                const double* __restrict__ lv, double sigma,
                                                double* __restrict__ yref) {
    __shared__ double cs[WG];
    __shared__ int as[WG];
    const int m = nu_eff[0];
    const int j = seed[0];
    double best = -1.0;
    int ba = 0;
    for (int a = threadIdx.x; a < m; a += WG) {
        double z = 0.0;
        for (int k = 0; k < m; ++k) z += (double)K[(int64_t)k * stride + j] * Y[(int64_t)a * nu + k];
        const double c = fabs(z * level_window(eps[a], lv[1], lv[2], sigma));
        if (c > best) {
            best = c;
            ba = a;
        }
    }
    cs[threadIdx.x] = best;
    as[threadIdx.x] = ba;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int t = 1; t < WG; ++t)
        if (cs[t] > best || (cs[t] == best && as[t] < ba)) {
            best = cs[t];
            ba = as[t];
        }
    for (int k = 0; k < nu; ++k) yref[k] = k < m ? Y[(int64_t)ba * nu + k] : 0.0;
}

template <typename T>
__global__ __launch_bounds__(WG) void k_es_vref(const T* __restrict__ K, int64_t stride, int64_t M, int nu,
                                                const int32_t* __restrict__ nu_eff, const double* __restrict__ yref,
                                                double* __restrict__ vref) {
    const int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (i >= M) return;
    const int m = nu_eff[0];
    double v = 0.0;
    for (int k = 0; k < m; ++k) v += (double)K[(int64_t)k * stride + i] * yref[k];
    vref[i] = v;
}

template <typename T>
LaunchInfo launch_es_refvec(const T* K, int64_t stride, int64_t M, const int32_t* seed, int nu,
                            const int32_t* nu_eff, const double* Y, const double* eps, const double* lv, double sigma,
                            double* yref, double* vref, hipStream_t s) {
    hipLaunchKernelGGL((k_es_pick<T>), dim3(1), dim3(WG), 0, s, K, stride, seed, nu, nu_eff, Y, eps, lv, sigma, yref);
    const int64_t wgs = (M + WG - 1) / WG;
    hipLaunchKernelGGL((k_es_vref<T>), dim3((unsigned)wgs), dim3(WG), 0, s, K, stride, M, nu, nu_eff, yref, vref);
    LaunchInfo li;
    li.wgs = wgs;
    li.bytes = (double)nu * M * (sizeof(T) + 8.0 / nu);
    return li;
}
template LaunchInfo launch_es_refvec<float>(const float*, int64_t, int64_t, const int32_t*, int, const int32_t*,
                                            const double*, const double*, const double*, double, double*, double*,
                                            hipStream_t);
template LaunchInfo launch_es_refvec<double>(const double*, int64_t, int64_t, const int32_t*, int, const int32_t*,
                                             const double*, const double*, const double*, double, double*, double*,
                                             hipStream_t);

template <typename T>
static LaunchInfo launch_gather_t(int B, int nseeds, const int32_t* seeds, int nu, const int32_t* nu_eff_blk,
                                  const T* K, int64_t stride, const int32_t* Hrp, const int32_t* Hcol, int max_row,
                                  double* Kp, int32_t* nu_copy, hipStream_t s) {
    hipLaunchKernelGGL((k_gather_rows<T>), dim3(nseeds), dim3(WG), 0, s, nseeds, seeds, B, nu, nu_eff_blk, K, stride, Hrp,
                       Hcol, max_row, Kp, nu_copy);
    LaunchInfo li;
    li.wgs = nseeds;
    li.bytes = (double)nseeds * nu * max_row * (sizeof(T) + 8.0);
    return li;
}

template <>
LaunchInfo launch_gather<float>(int B, int nseeds, const int32_t* seeds, int nu, const int32_t* nu_eff_blk,
                                const float* K, int64_t stride, const int32_t* Hrp, const int32_t* Hcol, int max_row,
                                double* Kp, int32_t* nu_copy, hipStream_t s) {
    return launch_gather_t<float>(B, nseeds, seeds, nu, nu_eff_blk, K, stride, Hrp, Hcol, max_row, Kp, nu_copy, s);
}

template <>
LaunchInfo launch_gather<double>(int B, int nseeds, const int32_t* seeds, int nu, const int32_t* nu_eff_blk,
                                 const double* K, int64_t stride, const int32_t* Hrp, const int32_t* Hcol, int max_row,
                                 double* Kp, int32_t* nu_copy, hipStream_t s) {
    return launch_gather_t<double>(B, nseeds, seeds, nu, nu_eff_blk, K, stride, Hrp, Hcol, max_row, Kp, nu_copy, s);
}

}  // namespace mar
