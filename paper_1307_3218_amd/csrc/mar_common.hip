// Type-independent FP64 kernels: fixed-order reduction of partial sums, the
// norm / breakdown decision of one Gram-Schmidt step, and the energy sum.
#include <algorithm>

#include "mar_device.h"
#include "mar_internal.h"

namespace mar {

// out[o] = sum_c part[c * L + o] for o < L, summed in a fixed order (chunk
// lanes strided by CL, then the CL lane sums in order). When h != nullptr the
// first nk*B outputs are also the subspace-matrix column n: o = k * B + b is
// written to h[b][k][n].
template <int OPW>
__global__ __launch_bounds__(WG) void k_reduce(const double* __restrict__ part, int64_t nchunks, int64_t L,
                                               double* __restrict__ out, double* __restrict__ h, int B, int nu,
                                               int n, int64_t hL) {
    constexpr int CL = WG / OPW;  // chunk lanes
    const int oi = threadIdx.x % OPW, cl = threadIdx.x / OPW;
    const int64_t o = (int64_t)blockIdx.x * OPW + oi;
    double s0 = 0.0, s1 = 0.0;
    if (o < L) {
        int64_t c = cl;
        for (; c + CL < nchunks; c += 2 * CL) {
            s0 += part[c * L + o];
            s1 += part[(c + CL) * L + o];
        }
        if (c < nchunks) s0 += part[c * L + o];
    }
    __shared__ double lds[WG];
    lds[threadIdx.x] = s0 + s1;
    __syncthreads();
    if (cl == 0 && o < L) {
        double t = 0.0;
        for (int k = 0; k < CL; ++k) t += lds[k * OPW + oi];
        out[o] = t;
        if (h != nullptr && o < hL) {
            const int64_t k = o / B, b = o % B;
            h[(b * nu + k) * (int64_t)nu + n] = t;
        }
    }
}

LaunchInfo launch_reduce(const double* part, int64_t nchunks, int64_t L, double* out, double* h, int B, int nu,
                         int n, hipStream_t s) {
    const int64_t hL = h ? (int64_t)(n + 1) * B : 0;
    LaunchInfo li;
    if (L <= 2048) {
        const int64_t wgs = (L + 3) / 4;
        hipLaunchKernelGGL((k_reduce<4>), dim3(wgs), dim3(WG), 0, s, part, nchunks, L, out, h, B, nu, n, hL);
        li.wgs = wgs;
    } else {
        const int64_t wgs = (L + 15) / 16;
        hipLaunchKernelGGL((k_reduce<16>), dim3(wgs), dim3(WG), 0, s, part, nchunks, L, out, h, B, nu, n, hL);
        li.wgs = wgs;
    }
    li.bytes = (double)(nchunks + 1) * L * 8.0;
    li.flops = (double)nchunks * L;
    return li;
}

// The reductions of one step of the delayed schedule in one launch.
//
// Workgroups below w1 sum the projection's partials, OPW outputs each: out[o] = sum over its partials in a fixed order
// (lanes strided by CL = WG / OPW, each lane's in order, then the CL lane sums in order). Without a plan the partials
// are part[c * L + o], c < nchunks. With the plan of a support-restricted sweep, o = (r * nk + k) * B + b sums over the
// groups g that read slab k (ksmin[g] <= ks = k / kg; ksmin does not fall with g) the partial of workgroup
// off[g] + ks - ksmin[g].
// The workgroups behind them take the first stage of the S-norm sums, whose partials np.part[c][L2] one product kernel
// left, a row per workgroup: np.tmp[y][L2] sums the rows of range y, four lanes of 64 outputs per workgroup; the
// coefficient kernel adds the ranges.
//
// What bounds it is latency, not the partials (18 MB at nu = 30, 256 seeds on 16384 rows): the plan is copied to LDS
// once per workgroup and eight partials are in flight per lane. Measured there: 6.3 us per step; 14.1 us with a plan
// entry and a partial at a time, and 8.9 us more in two launches for the norms.
constexpr int64_t PLAN_LDS = 4096;   // groups of a plan copied to LDS (more: a caller's own grid, read in place)
struct NormPart {
    const double* part;   // nullptr: none
    double* tmp;
    int64_t rows, rows_per;
    int L, nx;            // outputs, workgroups per range
};

template <int OPW, bool SP>
__global__ __launch_bounds__(WG) void k_reduce_step(const double* __restrict__ part, const int32_t* __restrict__ plan,
                                                    int64_t grid, int64_t nchunks, int kg, int nk, int B, int64_t L,
                                                    double* __restrict__ out, int64_t w1, NormPart np) {
    constexpr int CL = WG / OPW, U = 8;
    extern __shared__ int2 pl[];   // SP: off - ksmin and ksmin of every group
    __shared__ double lds[WG];
    if ((int64_t)blockIdx.x >= w1) {
        const int j = (int)((int64_t)blockIdx.x - w1), x = j % np.nx;
        const int oi = threadIdx.x % 64, cl = threadIdx.x / 64;
        const int o = x * 64 + oi;
        const int64_t y = j / np.nx, c0 = y * np.rows_per, c1 = c0 + np.rows_per < np.rows ? c0 + np.rows_per : np.rows;
        double t[U] = {};
        if (o < np.L) {
            int64_t c = c0 + cl;
            for (; c + 4 * (U - 1) < c1; c += 4 * U)
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] += np.part[(c + 4 * u) * np.L + o];
            for (; c < c1; c += 4) t[0] += np.part[c * np.L + o];
        }
        lds[threadIdx.x] = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        __syncthreads();
        if (cl == 0 && o < np.L) np.tmp[y * np.L + o] = ((lds[oi] + lds[64 + oi]) + lds[128 + oi]) + lds[192 + oi];
        return;
    }
    const int oi = threadIdx.x % OPW, cl = threadIdx.x / OPW;
    const int64_t o = (int64_t)blockIdx.x * OPW + oi, oc = o < L ? o : L - 1;
    double s0 = 0.0;
    if constexpr (SP) {
        const int ng = plan[0];
        const int32_t* off = plan + 8;
        const int32_t* ksm = off + grid;
        const bool staged = grid <= PLAN_LDS;
        auto entry = [&](int g) { return make_int2(off[g] - ksm[g], ksm[g]); };
        if (staged)
            for (int g = threadIdx.x; g < ng; g += WG) pl[g] = entry(g);
        __syncthreads();
        const int64_t b = oc % B, k = (oc / B) % nk, r = oc / ((int64_t)nk * B);
        const int ks = (int)(k / kg);
        const double* at = part + (r * kg + k % kg) * B + b;
        const int64_t wstep = (int64_t)3 * kg * B;
        for (int g = cl; g < ng; g += CL * U) {
            if ((staged ? pl[g] : entry(g)).y > ks) break;
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int gu = g + u * CL;
                const int gc = gu < ng ? gu : g;
                const int2 e = staged ? pl[gc] : entry(gc);
                const bool in = gu < ng && e.y <= ks;
                v[u] = at[(in ? e.x + ks : 0) * wstep];
                if (!in) v[u] = 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) s0 += v[u];
        }
    } else {
        for (int64_t c = cl; c < nchunks; c += CL * U) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t cu = c + u * CL;
                v[u] = part[(cu < nchunks ? cu : c) * L + oc];
                if (cu >= nchunks) v[u] = 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) s0 += v[u];
        }
    }
    lds[threadIdx.x] = s0;
    __syncthreads();
    if (cl == 0 && o < L) {
        double t = 0.0;
        for (int c = 0; c < CL; ++c) t += lds[c * OPW + oi];
        out[o] = t;
    }
}

// Rows per range of the norm sums: at most NORM_RANGES ranges, which one wavefront of the coefficient kernel adds, and
// at least 64 rows each (two rounds of loads).
static int64_t norm_rows_per(int64_t rows) {
    const int64_t r = (rows + NORM_RANGES - 1) / NORM_RANGES;
    return r < 64 ? 64 : r;
}
int norm_ranges(int64_t rows) { return rows > 0 ? (int)((rows + norm_rows_per(rows) - 1) / norm_rows_per(rows)) : 0; }

LaunchInfo launch_reduce_step(const double* part, int64_t nchunks, const int32_t* plan, int64_t grid, int kg, int nk,
                              int B, double* out, const double* npart, int64_t nrows, double* ntmp, hipStream_t s) {
    const int64_t L = (int64_t)3 * nk * B;
    const int opw = L <= 2048 ? 4 : 16;
    const int64_t w1 = (L + opw - 1) / opw;
    NormPart np{npart, ntmp, nrows, norm_rows_per(nrows), 2 * B, (2 * B + 63) / 64};
    const int64_t w2 = npart ? (int64_t)np.nx * norm_ranges(nrows) : 0;
    const dim3 g((unsigned)(w1 + w2));
    const size_t lds = plan && grid <= PLAN_LDS ? (size_t)grid * sizeof(int2) : 0;
    if (plan && opw == 4)
        hipLaunchKernelGGL((k_reduce_step<4, true>), g, dim3(WG), lds, s, part, plan, grid, nchunks, kg, nk, B, L, out, w1, np);
    else if (plan)
        hipLaunchKernelGGL((k_reduce_step<16, true>), g, dim3(WG), lds, s, part, plan, grid, nchunks, kg, nk, B, L, out, w1, np);
    else if (opw == 4)
        hipLaunchKernelGGL((k_reduce_step<4, false>), g, dim3(WG), 0, s, part, plan, grid, nchunks, kg, nk, B, L, out, w1, np);
    else
        hipLaunchKernelGGL((k_reduce_step<16, false>), g, dim3(WG), 0, s, part, plan, grid, nchunks, kg, nk, B, L, out, w1, np);
    LaunchInfo li;
    li.wgs = w1 + w2;
    li.bytes = plan ? (double)L * 8.0 : (double)(nchunks + 1) * L * 8.0;
    li.flops = plan ? 0.0 : (double)nchunks * L;
    if (npart) {
        li.bytes += (double)(nrows + norm_ranges(nrows)) * 2 * B * 8.0;
        li.flops += (double)nrows * 2 * B;
    }
    return li;
}

// Norm and breakdown of the new residual of each seed (all in FP64):
//   beta = sqrt(w^T S w), eta^2 = |c1|^2 + |c2|^2 + beta^2,
//   breakdown if beta <= tau * eta -> nu_eff = n + 1 and the seed stops;
//   w^T S w < 0 (or not finite) -> nu_eff = -1 (S not positive definite).
__global__ __launch_bounds__(WG) void k_norm(int B, int nk, const double* __restrict__ beta2,
                                             const double* __restrict__ c1, const double* __restrict__ c2,
                                             double tau, int32_t* __restrict__ active, int32_t* __restrict__ nu_eff,
                                             double* __restrict__ beta, int n) {
    // thread (part, b): partial sums of |c1|^2 + |c2|^2 over k = part, part + np, ...
    __shared__ double lds[WG];
    const int np = WG / B;
    const int b = threadIdx.x % B, part = threadIdx.x / B;
    double s = 0.0;
    if (part < np)
        for (int k = part; k < nk; k += np) {
            const double a1 = c1[(int64_t)k * B + b], a2 = c2[(int64_t)k * B + b];
            s += a1 * a1 + a2 * a2;
        }
    lds[threadIdx.x] = s;
    __syncthreads();
    if ((int)threadIdx.x >= B) return;
    double cc = 0.0;
    for (int q = 0; q < np; ++q) cc += lds[q * B + b];
    if (!active[b]) {
        beta[b] = 0.0;
        return;
    }
    const double bb = beta2[b];
    if (!(bb >= 0.0) || !(bb < INFINITY)) {
        nu_eff[b] = -1;
        active[b] = 0;
        beta[b] = 0.0;
        return;
    }
    const double bt = sqrt(bb);
    const double eta = sqrt(cc + bb);
    if (bt <= tau * eta) {
        nu_eff[b] = n + 1;
        active[b] = 0;
        beta[b] = 0.0;
    } else {
        beta[b] = bt;
    }
}

LaunchInfo launch_norm(int B, int nk, const double* beta2, const double* c1, const double* c2, double tau,
                       int32_t* active, int32_t* nu_eff, double* beta, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_norm, dim3(1), dim3(WG), 0, s, B, nk, beta2, c1, c2, tau, active, nu_eff, beta, n);
    LaunchInfo li;
    li.wgs = 1;
    li.bytes = (2.0 * nk + 3.0) * B * 8.0;
    return li;
}

// out = sum of x[0..n) in a fixed order (strided lane sums, then a tree).
__global__ __launch_bounds__(WG) void k_sum(const double* __restrict__ x, int64_t n, double* __restrict__ out) {
    __shared__ double lds[WG];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += WG) s += x[i];
    lds[threadIdx.x] = s;
    __syncthreads();
    for (int w = WG / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) lds[threadIdx.x] += lds[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = lds[0];
}

LaunchInfo launch_sum(const double* x, int64_t n, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(WG), 0, s, x, n, out);
    LaunchInfo li;
    li.wgs = 1;
    li.bytes = (double)(n + 1) * 8.0;
    return li;
}

// Zero n16 16-byte words (the padded rows of the work vectors, and the basis
// of a seed block under support tracking; a kernel rather than a memset so the
// sequence stays capturable). A grid-stride loop over a bounded grid: a launch
// must stay below 2^32 work-items, and the basis of the largest instance is
// 80 GB (5e9 words).
constexpr int64_t ZERO_MAX_WGS = 16384;
__global__ __launch_bounds__(WG) void k_zero(double2* __restrict__ p, int64_t n16) {
    const int64_t step = (int64_t)gridDim.x * WG;
    for (int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x; i < n16; i += step) p[i] = make_double2(0.0, 0.0);
}

LaunchInfo launch_zero(void* p, int64_t bytes, hipStream_t s) {
    const int64_t n16 = bytes / 16;
    const int64_t need = (n16 + WG - 1) / WG;
    const int64_t wgs = need < ZERO_MAX_WGS ? need : ZERO_MAX_WGS;
    LaunchInfo li;
    if (wgs > 0) hipLaunchKernelGGL(k_zero, dim3((unsigned)wgs), dim3(WG), 0, s, (double2*)p, n16);
    li.wgs = wgs;
    li.bytes = (double)bytes;
    return li;
}

// A wavefront's own LDS writes become visible to its other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// ---------------------------------------------------------------------------
// Delayed-reorthogonalization schedule: small FP64 per-seed algebra of step n.
//
// Entering step n, u_0..u_{n-1} are final (K^T S K = I) and u~ (slab n) has
// had one Gram-Schmidt pass and unit S-norm; y = H u~. The projection sweep
// gave, per seed, c2 = K^T S u~ (second-pass coefficients of u~), g = K^T S y,
// e = K^T y, and the self products u~.S y, u~.y. With
//   gamma = sqrt(1 - |c2|^2),  u_n = (u~ - K c2) / gamma,
// and the relation H K = K R collected from earlier steps (R upper Hessenberg
// of the Gram-Schmidt coefficients, column n-1 completed here), this kernel
// produces
//   column n of A = K^T H K:  A[:n+1, n] = (E - G q) / gamma,  q = R c2,
//     E = [e ; (u~.y - c2.e) / gamma],  G the Euclidean Gram matrix K^T K;
//   column n of G from t = K^T u~ = (A[:n, n-1] - G c1_prev) / beta~_prev;
//   the first-pass coefficients of H u_n against the S-basis,
//     c1 = (F - q) / gamma,  F = [g ; (u~.S y - c2.g) / gamma];
//   and the update coefficients (c2, g, gamma, F_n) for k_upd2.
// The final norm of the vector appended at step n-1 is beta~_prev * gamma; it
// is tested here against tau * eta (eta^2 = |c1_prev|^2 + beta~_prev^2 (|c2|^2 +
// gamma^2)), the same test the two-pass schedule applies, one step later.
// Slab n holds u~ unnormalized, s u~ with s = beta~_prev (1 at n = 0), and so
// do the sweep's right-hand sides; the products are rescaled here, and the
// update coefficients go out multiplied by s (k_upd2 divides by s gamma).
// A stopped seed gets gamma = inf, so that its slabs become zero.
// A is h[b][k][n]; G is [nu][nu]; R is column-major [nu][nu+1] (R_{p,k} at
// k*(nu+1) + p).
//
// One workgroup of W wavefronts per seed. What bounds it is latency: a few KB to a few hundred KB per seed, passed
// through a chain of sums. Lane = row p of R and G (64 rows at a time), wavefront w takes the columns k = w mod W, so that
// rows are read whole; the W partial sums meet in LDS. The scalar sums are formed by every wavefront for itself, from the
// vectors in LDS, without a barrier. KU > 0 (nu <= 64, nu <= KU W): the two matrices and the vectors are requested at the
// start, before anything is known of the step, and kept in registers: one trip to memory and three barriers. KU = 0: the
// columns are read eight at a time, 64 rows after another with one barrier each (the partial sums alternate between two
// buffers). Measured (us per step, 256 seeds): 7.4 at nu = 30 and (FP64, 128 seeds) 8.1 at nu = 50, where a workgroup of
// 256 threads with four columns in flight and a barrier for every scalar sum took 11.9 and 13.1; 26 at nu = 300 (64
// seeds), 48 before.
template <int W, int KU>
__global__ __launch_bounds__(W * 64) void k_coef(int B, int nu, int n, const double* __restrict__ red,
                                                 double* __restrict__ Ah, double* __restrict__ Gm,
                                                 double* __restrict__ Rm, double* __restrict__ C1,
                                                 double* __restrict__ BT, double* __restrict__ UU,
                                                 double* __restrict__ cA, double* __restrict__ cB,
                                                 float* __restrict__ cAf, float* __restrict__ cBf,
                                                 double* __restrict__ gam, double* __restrict__ Fn,
                                                 int32_t* __restrict__ active, int32_t* __restrict__ nu_eff, double tau,
                                                 const double* __restrict__ redb, int nrange) {
    constexpr int NT = W * 64;
    constexpr bool PRE = KU > 0;
    extern __shared__ double sm[];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = n + 1;
    double* c2 = sm;
    double* g = c2 + (nu + 1);
    double* e = g + (nu + 1);
    double* c1p = e + (nu + 1);
    double* q = c1p + (nu + 1);
    double* v = q + (nu + 1);        // column n of G
    double* gq = v + (nu + 1);
    double* ps = gq + (nu + 1);      // partial sums: PRE [4][W][64], else [2][3][W][64]
    double* A = Ah + (int64_t)b * nu * nu;
    double* G = Gm + (int64_t)b * nu * nu;
    double* Rc = Rm + (int64_t)b * nu * (nu + 1);

    double rr[PRE ? KU : 1], gg[PRE ? KU : 1], ap = 0.0;
    if constexpr (PRE) {
        // columns and rows past the step's read column and row 0: finite, and taken with a zero or not used
        const int pr = lane <= nu ? lane : 0, pg = lane < n ? lane : 0;
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int k = wv + i * W;
            rr[i] = Rc[(int64_t)(k < n - 1 ? k : 0) * (nu + 1) + pr];
            gg[i] = G[(int64_t)(k < n ? k : 0) * nu + pg];
        }
        ap = A[lane < n ? (int64_t)lane * nu + (n - 1) : 0];
    }
    auto stop = [&](int nu_new) {
        for (int k = tid; k < n; k += NT) {
            cA[(int64_t)k * B + b] = 0.0;
            cB[(int64_t)k * B + b] = 0.0;
            if (cAf) {
                cAf[(int64_t)k * B + b] = 0.0f;
                cBf[(int64_t)k * B + b] = 0.0f;
            }
        }
        if (tid == 0) {
            gam[b] = INFINITY;
            Fn[b] = 0.0;
            if (nu_new >= 0) {
                nu_eff[b] = nu_new;
                active[b] = 0;
            }
        }
    };
    // Step n >= 1 (nrange > 0): the breakdown test of slab n, the unnormalized residual of step n - 1, from the range
    // sums redb[nrange][2 B] of {u~.S u~ [B], u~.u~ [B]}: beta~ = sqrt(u~.S u~) <= tau sqrt(|c1_prev|^2 + beta~^2)
    // stops the seed at nu_eff = n; a negative or non-finite u~.S u~ flags S as not positive definite
    // (nu_eff = -1). Otherwise beta~ and u~.u~ / beta~^2 become BT and UU.
    const bool was_active = active[b] != 0;
    double btp = BT[b], uu = UU[b], bb = 0.0, ww = 0.0;
    if (nrange > 0) {
        const int64_t row = (int64_t)min(lane, nrange - 1) * 2 * B + b;
        const double rb = redb[row], rw = redb[row + B];
        bb = wave_sum(lane < nrange ? rb : 0.0);
        ww = wave_sum(lane < nrange ? rw : 0.0);
        if (was_active) {
            btp = sqrt(bb);
            uu = ww / bb;
        }
    }
    const double sc = n >= 1 ? btp : 1.0;   // scale of slab n
    for (int k = tid; k < n; k += NT) {
        c2[k] = red[((int64_t)0 * nk + k) * B + b] / sc;
        g[k] = red[((int64_t)1 * nk + k) * B + b] / sc;
        e[k] = red[((int64_t)2 * nk + k) * B + b] / sc;
        c1p[k] = C1[(int64_t)b * nu + k];
    }
    const double utsy = red[((int64_t)1 * nk + n) * B + b] / sc / sc;
    const double uty = red[((int64_t)2 * nk + n) * B + b] / sc / sc;
    __syncthreads();
    double p0 = 0.0, p1 = 0.0, p2 = 0.0, p3 = 0.0;
    for (int k = lane; k < n; k += 64) {
        p0 += c2[k] * c2[k];
        p1 += c1p[k] * c1p[k];
        p2 += c2[k] * e[k];
        p3 += c2[k] * g[k];
    }
    const double s_cc = wave_sum(p0), s_c1p = wave_sum(p1), s_ce = wave_sum(p2), s_cg = wave_sum(p3);
    if (nrange > 0 && was_active) {
        const bool bad = !(bb >= 0.0) || !(bb < INFINITY);
        if (bad || btp <= tau * sqrt(s_c1p + bb)) {
            if (tid == 0) {
                nu_eff[b] = bad ? -1 : n;
                active[b] = 0;
                BT[b] = 0.0;
            }
            stop(-1);
            return;
        }
        if (tid == 0) {
            BT[b] = btp;
            UU[b] = uu;
        }
    }
    if (!was_active) {
        stop(-1);
        return;
    }
    const double gam2 = 1.0 - s_cc;
    if (!(gam2 > 0.0)) {  // u~ lies in span(K): the Krylov space is exhausted
        stop(n);
        return;
    }
    const double gm = sqrt(gam2);
    if (n >= 1) {
        const double bf = btp * gm;
        const double eta = sqrt(s_c1p + btp * btp * (s_cc + gam2));
        if (bf <= tau * eta) {
            stop(n);
            return;
        }
        // column n - 1 of R, its zeros included
        for (int p = tid; p <= nu; p += NT)
            Rc[(int64_t)(n - 1) * (nu + 1) + p] = p < n ? c1p[p] + btp * c2[p] : p == n ? btp * gm : 0.0;
    }
    // From the sums over all k: q = R[:n+1, :n] c2 (its column n - 1 formed here), then with G c1_prev and G c2 the
    // column n of G, its products with c2 and q on the way. Every wavefront does all rows.
    double p4 = 0.0, p5 = 0.0, p6 = 0.0;
    auto row_q = [&](int p, double sum) {
        if (n >= 1 && p <= n) sum += (p < n ? c1p[p] + btp * c2[p] : btp * gm) * c2[n - 1];
        if (p <= n) q[p] = sum;
    };
    auto row_v = [&](int p, double gc1, double gc2, double a) {
        if (p < n) {
            const double t = (a - gc1) / btp, x = (t - gc2) / gm;
            v[p] = x;
            p4 += c2[p] * t;
            p5 += c2[p] * gc2;
            p6 += x * q[p];
        }
    };
    auto total = [&](const double* s) {   // the W partial sums of the lane's row, in order
        double t = 0.0;
#pragma unroll
        for (int u = 0; u < W; ++u) t += s[u * 64 + lane];
        return t;
    };
    if constexpr (PRE) {
        double sq = 0.0, s1 = 0.0, s2 = 0.0, sw = 0.0;
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int k = wv + i * W, kc = k < n ? k : 0;
            const double x2 = k < n ? c2[kc] : 0.0, x1 = k < n ? c1p[kc] : 0.0;
            if (n >= 2) sq += rr[i] * (k < n - 1 ? x2 : 0.0);
            s1 += gg[i] * x1;
            s2 += gg[i] * x2;
        }
        ps[tid] = sq;
        ps[NT + tid] = s1;
        ps[2 * NT + tid] = s2;
        __syncthreads();
        row_q(lane, total(ps));
        row_v(lane, total(ps + NT), total(ps + 2 * NT), ap);
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < KU; ++i) {
            const int k = wv + i * W, kc = k < n ? k : 0;
            sw += gg[i] * (k < n ? q[kc] : 0.0);
        }
        ps[3 * NT + tid] = sw;   // a place of its own: other wavefronts may still read the first sums
        __syncthreads();
        if (tid < n) gq[tid] = total(ps + 3 * NT);
    } else {
        constexpr int U = 8;
        int buf = 0;
        for (int c = 0; c * 64 <= n; ++c, buf ^= 1) {
            const int p = c * 64 + lane;
            double s[U] = {};
            // the chunk's rows begin at column c * 64 - 1
            int k0 = c * 64 - 1 - (W - 1);
            k0 = k0 > 0 ? k0 / W * W : 0;
            for (int k = k0 + wv; k < n - 1; k += W * U)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ku = k + u * W;
                    const bool in = ku < n - 1;
                    const double r = Rc[(int64_t)(in ? ku : k) * (nu + 1) + (p <= nu ? p : 0)];
                    s[u] += r * (in ? c2[in ? ku : k] : 0.0);
                }
            double* pb = ps + buf * 3 * NT;
            pb[tid] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
            __syncthreads();
            row_q(p, total(pb));
        }
        wave_lds_sync();
        for (int c = 0; c * 64 < n; ++c, buf ^= 1) {
            const int p = c * 64 + lane, pc = p < n ? p : 0;
            const double a = A[(int64_t)pc * nu + (n - 1)];
            double s1[4] = {}, s2[4] = {}, sw[4] = {};
            for (int k = wv; k < n; k += W * U) {
                double x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ku = k + u * W;
                    x[u] = G[(int64_t)(ku < n ? ku : 0) * nu + pc];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ku = k + u * W, kc = ku < n ? ku : 0;
                    const double y = ku < n ? x[u] : 0.0;
                    s1[u & 3] += y * c1p[kc];
                    s2[u & 3] += y * c2[kc];
                    sw[u & 3] += y * q[kc];
                }
            }
            double* pb = ps + buf * 3 * NT;
            pb[tid] = (s1[0] + s1[1]) + (s1[2] + s1[3]);
            pb[NT + tid] = (s2[0] + s2[1]) + (s2[2] + s2[3]);
            pb[2 * NT + tid] = (sw[0] + sw[1]) + (sw[2] + sw[3]);
            __syncthreads();
            row_v(p, total(pb), total(pb + NT), a);
            if (p < n) gq[p] = total(pb + 2 * NT);
        }
        __syncthreads();
    }
    wave_lds_sync();
    const double s_ct = wave_sum(p4), s_cgc = wave_sum(p5), s_vq = wave_sum(p6);
    const double gnn = (uu - 2.0 * s_ct + s_cgc) / gam2;
    const double En = (uty - s_ce) / gm;
    const double Fnn = (utsy - s_cg) / gm;
    const double qn = q[n];
    for (int p = tid; p <= n; p += NT) {
        // (G q)_p over k <= n: the old columns, then column n
        const double sgq = p < n ? gq[p] + v[p] * qn : s_vq + gnn * qn;
        const double Ep = p < n ? e[p] : En;
        A[(int64_t)p * nu + n] = (Ep - sgq) / gm;
        const double Fp = p < n ? g[p] : Fnn;
        C1[(int64_t)b * nu + p] = (Fp - q[p]) / gm;
        const double gp = p < n ? v[p] : gnn;
        G[(int64_t)p * nu + n] = gp;
        G[(int64_t)n * nu + p] = gp;
        if (p < n) {
            cA[(int64_t)p * B + b] = sc * c2[p];
            cB[(int64_t)p * B + b] = sc * g[p];
            if (cAf) {  // the same coefficients rounded once to the basis precision
                cAf[(int64_t)p * B + b] = (float)(sc * c2[p]);
                cBf[(int64_t)p * B + b] = (float)(sc * g[p]);
            }
        }
    }
    if (tid == 0) {
        gam[b] = sc * gm;
        Fn[b] = sc * Fnn;
    }
}

// Dynamic LDS of k_coef: seven vectors, and the partial sums of W wavefronts.
constexpr size_t coef_lds(int nu, int W, bool pre) { return (size_t)(7 * (nu + 1) + (pre ? 4 : 6) * W * 64) * sizeof(double); }

template <int W, int KU>
static void coef(int B, int nu, int n, const double* red, double* A, double* G, double* R, double* C1, double* BT,
                 double* UU, double* cA, double* cB, float* cAf, float* cBf, double* gam, double* Fn, int32_t* active,
                 int32_t* nu_eff, double tau, const double* redb, int nrange, hipStream_t s) {
    const size_t lds = coef_lds(nu, W, KU > 0);
    static std::atomic<uint64_t> done{0};
    if (lds > 64 * 1024) allow_full_lds((const void*)k_coef<W, KU>, done);
    hipLaunchKernelGGL((k_coef<W, KU>), dim3(B), dim3(W * 64), lds, s, B, nu, n, red, A, G, R, C1, BT, UU, cA, cB, cAf,
                       cBf, gam, Fn, active, nu_eff, tau, redb, nrange);
}

LaunchInfo launch_coef(int B, int nu, int n, const double* red, double* A, double* G, double* R, double* C1,
                       double* BT, double* UU, double* cA, double* cB, float* cAf, float* cBf,
                       double* gam, double* Fn, int32_t* active, int32_t* nu_eff, double tau, const double* redb,
                       int nrange, hipStream_t s) {
    // 4 wavefronts hold the matrices up to nu = 32, 8 up to nu = 64 (7.4 us per step at nu = 30 against 7.5 for 8; 8.1 at
    // nu = 50 against 9.1 for 4); at nu = 100 the columns read as they are used take 17.3 us, kept in registers 17.8
    // past nu = 2047 the vectors leave LDS for eight wavefronts' sums (nu <= 2485), then for two
    LaunchInfo li;
    constexpr size_t max_lds = 160 * 1024;
    auto f = nu <= 32 ? coef<4, 8> : nu <= 64 ? coef<8, 8> : coef_lds(nu, 16, false) <= max_lds ? coef<16, 0>
             : coef_lds(nu, 8, false) <= max_lds ? coef<8, 0> : coef<2, 0>;
    if (coef_lds(nu, 2, false) > max_lds) {
        li.wgs = -1;
        return li;
    }
    f(B, nu, n, red, A, G, R, C1, BT, UU, cA, cB, cAf, cBf, gam, Fn, active, nu_eff, tau, redb, nrange, s);
    li.wgs = B;
    const double nn = (double)n + 1.0;
    li.bytes = (double)B * (3.0 * nn * nn + 8.0 * nn) * 8.0;
    li.flops = (double)B * 8.0 * nn * nn;
    return li;
}

}  // namespace mar
