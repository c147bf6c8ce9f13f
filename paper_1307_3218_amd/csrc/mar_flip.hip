// Local flipping refinement of an eigenvector (Appendix).
//
// The components a_l of phi (level eps) change sign one at a time when that
// lowers R = |r|^2 (+ c p^2), r = (H - eps S) phi, p = phi_ref^T S phi. A flip
// of a_l changes r by -2 a_l (H - eps S) e_l on the rows of P(l) only (H and S
// are symmetric) and p by -2 a_l s_l, s = S phi_ref, so no product with the
// matrix is needed after the first residual. The rows are visited by colour of
// a distance-2 colouring of H's pattern, and in index order within a colour.
// Rows of one colour have disjoint column supports, so the |r|^2 part of each
// row's single-flip change does not depend on the colour's other flips: it is
// computed for all rows of the colour at once. Without the penalty the rows
// then decide at once. The penalty couples every row through p, so with it one
// wave walks the colour's rows in index order, each deciding on the p left by
// the flips before it: a sequential descent, every accepted flip lowering R.
// Sweeps repeat until one flips nothing or max_sweeps have run.
//
// k_flip_setup (a thread per row) lays the rows out in colour order: H - eps S and the columns, phi and s = S phi_ref
// beside them, and the first residual. k_flip is one workgroup: the colours follow one another, and a colour's rows, one
// to a thread, are few (21 to 622 at M = 16384). What bounds it is the chain of one colour's instructions on a few
// wavefronts: r is kept in LDS while it fits, the next colour's rows are on their way while this one decides, a row
// applies its flip at once, since no other row of the colour reads the entries it changes (one barrier per colour), and
// rows are padded (weight 0 at r[M] = 0) instead of branching on their length. Every sum runs in a fixed order, with
// products and sums rounded separately (no fused multiply-add), so that every decision is reproducible. Measured at
// M = 16384, 40 colours, the whole call: 1.12 ms (k_flip 0.9, k_flip_setup 0.02); 7.9 ms with r, H and S read through the
// caches in row order and three barriers per colour. An address for every entry took k_flip a fifth longer; rows requested
// two or three colours ahead, or 256 threads, 5 to 10 %.
#include "mar_device.h"
#include "mar_internal.h"

namespace mar {

constexpr int FLIP_CH = 20;   // entries of a row held in registers

// Entries of 64 consecutive rows of the colour order lie together, V entries (16 bytes) of a row at a time: entry q of
// row e is at flip_at(e) + flip_entry(q), and a wavefront's load reads 1 KB.
__device__ __forceinline__ int64_t flip_at(int64_t e, int width, int V) { return (e >> 6) * 64 * width + (e & 63) * V; }
__device__ __forceinline__ int flip_entry(int q, int V) { return q / V * 64 * V + q % V; }

__global__ __launch_bounds__(WG) void k_flip_setup(int64_t M, const int32_t* __restrict__ rp,
                                                   const int32_t* __restrict__ col, const double* __restrict__ hv,
                                                   const double* __restrict__ sv, double eps,
                                                   const double* __restrict__ phi, const double* __restrict__ phi_ref,
                                                   int width, int scale, const int32_t* __restrict__ crow,
                                                   double* __restrict__ av, int32_t* __restrict__ ac,
                                                   double* __restrict__ r, double* __restrict__ srow,
                                                   double* __restrict__ pe, double* __restrict__ se) {
#pragma clang fp contract(off)
    const int64_t e = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (e >= M) return;
    const int l = crow[e], lo = rp[l], n = rp[l + 1] - lo;
    double* ae = av + flip_at(e, width, 2);
    int32_t* ce = ac + flip_at(e, width, 4);
    double t = 0.0, u = 0.0;   // the row's products in column order
    for (int q = 0; q < n; ++q) {
        const int c = col[lo + q];
        const double s = sv[lo + q], a = hv[lo + q] - eps * s;
        ae[flip_entry(q, 2)] = a;
        ce[flip_entry(q, 4)] = c * scale;
        t = t + a * phi[c];
        if (phi_ref) u = u + s * phi_ref[c];
    }
    for (int q = n; q < width; ++q) {   // padding: weight 0 at r[M] = 0
        ae[flip_entry(q, 2)] = 0.0;
        ce[flip_entry(q, 4)] = (int32_t)M * scale;
    }
    if (e == 0) r[M] = 0.0;
    r[l] = t;
    pe[e] = phi[l];
    if (phi_ref) srow[l] = se[e] = u;
}

template <bool LDSR>
__global__ __launch_bounds__(FLIP_WG) void k_flip(int64_t M, double* __restrict__ phi, bool pen, double cpen, int nround,
                                                  const int32_t* __restrict__ round, const int32_t* __restrict__ crow,
                                                  int max_sweeps, int width, const double* __restrict__ av,
                                                  const int32_t* __restrict__ ac, double* rg,
                                                  const double* __restrict__ srow, double* pe,
                                                  const double* __restrict__ se, double* __restrict__ Rout,
                                                  int32_t* __restrict__ info) {
#pragma clang fp contract(off)
    extern __shared__ double rl[];
    __shared__ double red[FLIP_WG];
    __shared__ double dl[FLIP_WG], xl[FLIP_WG], yl[FLIP_WG], zl[FLIP_WG];   // penalty: a round's rows
    __shared__ uint8_t fl[FLIP_WG];
    __shared__ double p_sh;
    __shared__ int nflip;
    const int tid = threadIdx.x;
    double* r = LDSR ? rl : rg;
    auto wg_sum = [&](double v) {
        red[tid] = v;
        __syncthreads();
        for (int w = FLIP_WG / 2; w > 0; w >>= 1) {
            if (tid < w) red[tid] = red[tid] + red[tid + w];
            __syncthreads();
        }
        const double t = red[0];
        __syncthreads();
        return t;
    };
    auto norm2 = [&]() {
        double s = 0.0;
        for (int64_t i = tid; i < M; i += FLIP_WG) s = s + r[i] * r[i];
        return wg_sum(s);
    };
    if constexpr (LDSR)
        for (int64_t i = tid; i <= M; i += FLIP_WG) rl[i] = rg[i];
    if (tid == 0) {
        p_sh = 0.0;
        nflip = 0;
    }
    __syncthreads();
    if (pen) {
        // p = sum over the rows in index order: products a round at a time into LDS, then added by one thread
        double p = 0.0;
        for (int64_t b = 0; b < M; b += FLIP_WG) {
            if (b + tid < M) dl[tid] = srow[b + tid] * phi[b + tid];
            __syncthreads();
            if (tid == 0) {
                const int n = (int)(M - b < FLIP_WG ? M - b : FLIP_WG);
                for (int i = 0; i < n; ++i) p = p + dl[i];
            }
            __syncthreads();
        }
        if (tid == 0) p_sh = p;
        __syncthreads();
    }
    double R = norm2();
    if (tid == 0 && Rout) Rout[0] = R + (pen ? cpen * p_sh * p_sh : 0.0);
    auto barrier = [&]() {   // between rounds: r in LDS is all that threads exchange, and requests stay in flight
        if constexpr (LDSR)
            lds_barrier();
        else
            __syncthreads();
    };
    // A row per thread and round, requested FLIP_AHEAD rounds ahead into one of FLIP_AHEAD + 1 sets of registers that the
    // steps of the unrolled loop take in turn (handing the values from set to set would wait for them).
    struct Row {
        double a, s, w[FLIP_CH];
        int c[FLIP_CH];
    } set[FLIP_AHEAD + 1];
    auto request = [&](Row& n, int t) __attribute__((always_inline)) {
        if (t >= nround) t -= nround;
        const int b = round[2 * t], e = b + tid < round[2 * t + 1] ? b + tid : 0;   // threads without a row read row 0
        n.a = pe[e];
        if (pen) n.s = se[e];
        const double2* ae = (const double2*)(av + flip_at(e, width, 2));
        const int4* ce = (const int4*)(ac + flip_at(e, width, 4));
#pragma unroll
        for (int q = 0; q < FLIP_CH; q += 4) {
            const double2 x = ae[q / 2 * 64], y = ae[q / 2 * 64 + 64];
            const int4 z = ce[q / 4 * 64];
            n.w[q] = x.x, n.w[q + 1] = x.y, n.w[q + 2] = y.x, n.w[q + 3] = y.y;
            n.c[q] = z.x, n.c[q + 1] = z.y, n.c[q + 2] = z.z, n.c[q + 3] = z.w;
        }
    };
    auto res = [&](int c) __attribute__((always_inline)) -> double& {   // columns are byte offsets where r is in LDS
        return LDSR ? *(double*)((char*)rl + c) : rg[c];
    };
    int sweeps = 0, mine = 0;
    int64_t flips = 0;
    auto step = [&](const Row& g, int t) __attribute__((always_inline)) {
        const int b = round[2 * t], e = b + tid, e1 = round[2 * t + 1];
        const bool in = e < e1;
        const double a = g.a;
        // the |r|^2 part of the row's single-flip change, summed in the row's column order
        double d = 0.0, rv[FLIP_CH];
#pragma unroll
        for (int q = 0; q < FLIP_CH; ++q) rv[q] = res(g.c[q]);
#pragma unroll
        for (int q = 0; q < FLIP_CH; ++q) d = d + g.w[q] * ((4.0 * a) * a * g.w[q] - (4.0 * a) * rv[q]);
        for (int q = FLIP_CH; q < width && in; ++q) {
            const double wq = av[flip_at(e, width, 2) + flip_entry(q, 2)];
            d = d + wq * ((4.0 * a) * a * wq - (4.0 * a) * res(ac[flip_at(e, width, 4) + flip_entry(q, 4)]));
        }
        bool f = in && d < 0.0;
        if (pen) {
            dl[tid] = d;
            xl[tid] = (4.0 * a) * a * g.s * g.s;
            yl[tid] = (4.0 * a) * g.s;
            zl[tid] = (2.0 * a) * g.s;
            barrier();
            if (tid < 64) {
                // One wavefront decides the round's rows in index order on the p left by the flips before: 64 rows at
                // once on the current p; those up to the first that flips keep their decision, the ones behind it
                // decide again on the new p.
                double p = p_sh;
                const int n = e1 - b;
                for (int base = 0; base < n; base += 64) {
                    const int i = base + tid;
                    const bool has = i < n;
                    const double di = dl[has ? i : 0], xi = xl[has ? i : 0], yi = yl[has ? i : 0], zi = zl[has ? i : 0];
                    int from = 0;
                    bool flip = false;
                    while (from < 64) {
                        const unsigned long long bal = __ballot(has && tid >= from && di + cpen * (xi - yi * p) < 0.0);
                        if (bal == 0) break;
                        const int first = __ffsll(bal) - 1;
                        if (tid == first) flip = true;
                        p = p - read_lane(zi, first);
                        from = first + 1;
                    }
                    if (has) fl[i] = flip ? 1 : 0;
                }
                if (tid == 0) p_sh = p;
            }
            barrier();
            f = in && fl[tid] != 0;
        }
        if (f) {
#pragma unroll
            for (int q = 0; q < FLIP_CH; ++q) res(g.c[q]) = rv[q] - (2.0 * a) * g.w[q];   // column l: row l (symmetric)
            for (int q = FLIP_CH; q < width; ++q) {
                double& rq = res(ac[flip_at(e, width, 4) + flip_entry(q, 4)]);
                rq = rq - (2.0 * a) * av[flip_at(e, width, 2) + flip_entry(q, 2)];
            }
            pe[e] = -a;
            ++mine;
        }
        barrier();
    };
#pragma unroll
    for (int u = 0; u < FLIP_AHEAD; ++u) request(set[u], u);
    for (int sw = 0; sw < max_sweeps; ++sw) {
        mine = 0;
        for (int t = 0; t < nround; t += FLIP_AHEAD + 1) {
#pragma unroll
            for (int u = 0; u <= FLIP_AHEAD; ++u) {
                request(set[(u + FLIP_AHEAD) % (FLIP_AHEAD + 1)], t + u + FLIP_AHEAD);
                step(set[u], t + u);
            }
        }
        if (mine) atomicAdd(&nflip, mine);
        R = norm2();   // its barriers order the count too
        const int nf = nflip;
        sweeps = sw + 1;
        flips += nf;
        if (tid == 0 && Rout) Rout[sw + 1] = R + (pen ? cpen * p_sh * p_sh : 0.0);
        __syncthreads();
        if (tid == 0) nflip = 0;
        __syncthreads();
        if (nf == 0) break;
    }
    for (int64_t e = tid; e < M; e += FLIP_WG) phi[crow[e]] = pe[e];
    if (tid == 0 && info) {
        info[0] = sweeps;
        info[1] = (int32_t)(flips < 0x7fffffff ? flips : 0x7fffffff);
    }
}

static int flip_width(int max_row) { return max_row > FLIP_CH ? (max_row + 3) / 4 * 4 : FLIP_CH; }

size_t flip_workspace(int64_t M, int max_row) {
    return (size_t)(M + 63) / 64 * 64 * ((size_t)flip_width(max_row) * 12) + ((size_t)M * 4 + 1) * 8;
}

LaunchInfo launch_flip(int64_t M, const int32_t* rp, const int32_t* col, const double* hv, const double* sv, int max_row,
                       double eps, double* phi, const double* phi_ref, double cpen, int nround, const int32_t* round,
                       const int32_t* crow, int max_sweeps, void* work, double* Rout, int32_t* info, hipStream_t st) {
    const bool pen = phi_ref != nullptr && cpen != 0.0;
    const int width = flip_width(max_row);
    const size_t nel = (size_t)(M + 63) / 64 * 64 * width;
    double* av = (double*)work;
    int32_t* ac = (int32_t*)(av + nel);
    double* r = (double*)(ac + nel);
    double* srow = r + M + 1;   // s in row order
    double* pe = srow + M;      // phi and s in colour order
    double* se = pe + M;
    // r in LDS beside 21 KB of fixed arrays
    constexpr int lds_max = 138 * 1024;
    const size_t lds = (size_t)(M + 1) * 8;
    const bool fits = lds <= lds_max;
    const unsigned wgs = (unsigned)((M + WG - 1) / WG);
    hipLaunchKernelGGL(k_flip_setup, dim3(wgs), dim3(WG), 0, st, M, rp, col, hv, sv, eps, phi, pen ? phi_ref : nullptr,
                       width, fits ? 8 : 1, crow, av, ac, r, srow, pe, se);
    static std::atomic<uint64_t> done{0};
    if (fits) allow_lds((const void*)k_flip<true>, done, lds_max);
    hipLaunchKernelGGL((fits ? k_flip<true> : k_flip<false>), dim3(1), dim3(FLIP_WG), fits ? lds : 0, st, M, phi, pen, cpen,
                       nround, round, crow, max_sweeps, width, av, ac, r, srow, pe, se, Rout, info);
    LaunchInfo li;
    li.wgs = 1;
    return li;
}

}  // namespace mar
