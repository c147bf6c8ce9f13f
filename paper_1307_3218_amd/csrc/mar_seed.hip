// The Krylov phase of one seed in one workgroup, for small row sets: a local
// region (the rows within `hops` block hops of the seed) or a small cell.
//
// The seed-interleaved kernels run one launch per phase and step over a block
// of seeds; on a few hundred rows each launch is a few microseconds of latency,
// and with local regions every seed of a block streams the union of the
// block's regions. Here a workgroup keeps one seed's rows to itself and runs
// the whole recurrence (Sec. 2: u_1 = e_j / sqrt(S_jj), w = H u_n, two
// classical Gram-Schmidt passes in the S-inner product, A[:, n] = K^T w)
// between workgroup barriers. The work vectors and the first nl basis vectors
// live in LDS (vector k is read in every step n >= k, so the first ones are
// read most), the others in a scratch slab of the workgroup, which stays in
// the L2 / last-level cache. Per step: one product with H, two with S, and
// four sweeps over the basis (K^T w with K^T S w, w -= K c1, K^T S w,
// w -= K c2).
//
// What bounds it: on a few hundred rows the latency of the phases between
// barriers (seven per step: 4.6 us per step at 256 rows, FP32, nu = 30, of
// which the bytes are a tenth); with part of the basis outside LDS the L2 and
// last-level-cache reads of that part. Measured, whole Krylov phase: 0.14 ms
// for 256 seeds of the 256-row cell (FP32, nu = 30; the blocks' launches took
// 1.3 ms), 5.5 ms for 1024 seeds in regions of 6 hops (564 to 908 rows, FP32,
// nu = 100: 48 of 100 basis vectors in LDS; the blocks 78 ms), 8.3 ms for
// 2048 seeds of a 2048-row cell (FP64, nu = 30: 6 of 30 vectors in LDS; 9.5 ms
// with 4 in LDS and the wavefronts of a projection split over groups of
// vectors only, half of them idle).
// Two wavefronts per SIMD with 256 registers each: four with 128 spilled and
// ran 2.5 times slower. Between most phases only LDS is ordered (lds_barrier):
// a full barrier waits for the stores and the requested matrix values as well
// and cost 1000 cycles a phase.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "mar_device.h"
#include "mar_internal.h"

namespace mar {

constexpr int SEED_WG = 512;    // threads per compute unit: two wavefronts per SIMD, 256 registers each (at 128 the phases spill)
constexpr int SEED_G = 4;       // basis vectors a wavefront projects together
constexpr int SEED_NF = 4;      // 16-byte vectors of a lane kept in registers during a projection
constexpr int SEED_KP = 4;      // ranges of basis vectors in an update: 16 lanes of a wavefront each
constexpr int SEED_UN = 16;     // basis vectors of one range in flight

template <typename T>
struct SeedArgs {
    SeedGeom g;
    int64_t M;
    const int32_t *brp, *bcol;
    const T *hv, *sv;
    const double* diagS;
    const int32_t* seeds;
    int ns, nu, hops;
    double tau;
    T* scratch;             // g.sstride elements per workgroup
    const int32_t* Hrp;
    int max_row;
    double* h;              // [seed][nu][nu]
    double* Kp;             // [seed][nu][max_row]
    int32_t* nu_out;        // [seed]
    const double* vref;     // or null: also pref[k * pB + seed] = u_k . vref
    double* pref;
    int64_t pB;
    T* keep;                // or null: every basis vector also to keep[seed][nu][rows] (whole cells)
};

// Sums of V (4 or 8) values per lane over a wavefront: afterwards lane holds in v[0] the sum of value lane / (64 / V).
// Each of the first log2(V) exchanges keeps one half of the values; the exchanges are register moves between lanes
// (row swaps and DPP), not LDS permutes, whose latency the phases of a step would wait for.
template <int V>
__device__ __forceinline__ void wave_sum_multi(double (&v)[V], int lane) {
    static_assert(V == 4 || V == 8, "two or three halving exchanges");
#pragma unroll
    for (int i = 0; i < V / 2; ++i) v[i] = swap_add32(v[i], v[i + V / 2]);
#pragma unroll
    for (int i = 0; i < V / 4; ++i) v[i] = swap_add16(v[i], v[i + V / 4]);
    if constexpr (V == 8) {
        const bool up = (lane & 8) != 0;
        const double keep = up ? v[1] : v[0], send = up ? v[0] : v[1];
        v[0] = keep + dpp_move<0x128>(send);   // row_ror:8
    }
    v[0] += dpp_move<0xb1>(v[0]);    // lane ^ 1
    v[0] += dpp_move<0x4e>(v[0]);    // lane ^ 2
    v[0] += dpp_move<0x141>(v[0]);   // row_half_mirror: the other quad of eight lanes
    if constexpr (V == 4) v[0] += dpp_move<0x140>(v[0]);   // row_mirror: the other half of the row
}

// The row set of seed block I0: list[0 .. n) ascending block rows within hops of it (every block row when
// hops < 0), gptr their first block, lptr / lcol the local column of each of their blocks (n: outside).
// The breadth-first search keeps a hash table (key, slot value) in the memory of the basis, which is not in use
// yet. Entries are found in any order and then ranked, so the result does not depend on timing.
__device__ __forceinline__ int region_rows(int64_t nbrow, const int32_t* __restrict__ brp,
                                           const int32_t* __restrict__ bcol, int I0, int hops, int cap, int hs,
                                           int* list, int* gptr, int* lptr, uint16_t* lcol, int* hkey, int* hval,
                                           int* raw, int* misc) {
    const int tid = threadIdx.x, nt = blockDim.x;
    int n;
    if (hops < 0) {
        n = (int)nbrow;
        for (int i = tid; i <= n; i += nt) lptr[i] = brp[i];
        for (int i = tid; i < n; i += nt) {
            list[i] = i;
            gptr[i] = brp[i];
        }
        const int ne = brp[n];
        for (int p = tid; p < ne; p += nt) lcol[p] = (uint16_t)bcol[p];
        __syncthreads();
        return n;
    }
    for (int i = tid; i < hs; i += nt) hkey[i] = -1;
    __syncthreads();
    auto slot0 = [&](int I) { return (int)(((unsigned)I * 2654435761u) >> 7) & (hs - 1); };
    if (tid == 0) {
        const int s = slot0(I0);
        hkey[s] = I0;
        raw[0] = I0;
        misc[0] = 1;
    }
    __syncthreads();
    int f0 = 0, f1 = 1;
    for (int h = 0; h < hops && f0 < f1; ++h) {
        for (int e = f0 + tid; e < f1; e += nt) {
            const int I = raw[e];
            for (int p = brp[I]; p < brp[I + 1]; ++p) {
                const int J = bcol[p];
                int s = slot0(J);
                // at most cap keys enter a table of hs >= 2 cap slots: the probe always ends
                for (;;) {
                    const int old = atomicCAS(&hkey[s], -1, J);
                    if (old == -1) {
                        const int at = atomicAdd(&misc[0], 1);
                        if (at < cap) raw[at] = J;
                        break;
                    }
                    if (old == J) break;
                    s = (s + 1) & (hs - 1);
                }
            }
        }
        __syncthreads();
        f0 = f1;
        f1 = min(misc[0], cap);
        __syncthreads();
    }
    n = f1;
    // rank: position of each block row among the ascending ones
    for (int e = tid; e < n; e += nt) {
        const int I = raw[e];
        int r = 0;
        for (int k = 0; k < n; ++k) r += raw[k] < I ? 1 : 0;
        list[r] = I;
        int s = slot0(I);
        while (hkey[s] != I) s = (s + 1) & (hs - 1);
        hval[s] = r;
    }
    __syncthreads();
    for (int e = tid; e < n; e += nt) {
        gptr[e] = brp[list[e]];
        lptr[e + 1] = brp[list[e] + 1] - brp[list[e]];
    }
    __syncthreads();
    if (tid == 0) {
        int s = 0;
        lptr[0] = 0;
        for (int e = 0; e < n; ++e) {
            s += lptr[e + 1];
            lptr[e + 1] = s;
        }
    }
    __syncthreads();
    for (int e = tid; e < n; e += nt) {
        const int base = gptr[e], l = lptr[e + 1] - lptr[e];
        for (int t = 0; t < l; ++t) {
            const int J = bcol[base + t];
            int s = slot0(J), v = n;
            while (hkey[s] != -1) {
                if (hkey[s] == J) {
                    v = hval[s];
                    break;
                }
                s = (s + 1) & (hs - 1);
            }
            lcol[lptr[e] + t] = (uint16_t)v;
        }
    }
    __syncthreads();
    return n;
}

template <typename T, bool ACC64>
__global__ __launch_bounds__(SEED_WG) void k_seed(SeedArgs<T> a) {
    constexpr int VEC = Vec16<T>::n;
    using VT = typename Vec16<T>::type;
    using AT = typename std::conditional<ACC64, double, T>::type;
    extern __shared__ __align__(16) char sm[];
    const SeedGeom g = a.g;
    T* Kl = reinterpret_cast<T*>(sm);                       // nl basis vectors (first the region search's tables)
    T* u = reinterpret_cast<T*>(sm + g.oU);                 // work vectors, four zeros behind the rows
    T* y = u + 4 * g.nbcap + 4;
    T* z = y + 4 * g.nbcap + 4;
    double* d0 = reinterpret_cast<double*>(sm + g.oD);      // K^T w, then c2
    double* d1 = d0 + a.nu + 1;                             // c1
    double* cp = reinterpret_cast<double*>(sm + g.oP);      // sums of the chunks of rows (more than one)
    T* cT = reinterpret_cast<T*>(sm + g.oC);                // update coefficients in the basis precision
    int* list = reinterpret_cast<int*>(sm + g.oList);
    int* gptr = list + g.nbcap;
    int* lptr = gptr + g.nbcap;
    int* misc = lptr + g.nbcap + 1;
    uint16_t* lcol = reinterpret_cast<uint16_t*>(sm + g.oCol);
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, nw = nt >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nu = a.nu;
    for (int b = blockIdx.x; b < a.ns; b += gridDim.x) {
        const int j = a.seeds[b];
        __syncthreads();
        if (j < 0 || j >= a.M) {
            if (tid == 0) a.nu_out[b] = -2;
            continue;
        }
        int* tab = reinterpret_cast<int*>(sm);
        const int nb = region_rows(g.nbrow, a.brp, a.bcol, j / 4, a.hops, g.nbcap, g.hs, list, gptr, lptr, lcol, tab,
                                   tab + g.hs, tab + 2 * g.hs, misc);
        // basis vectors of this seed's nr rows: the first nl in LDS, vector k >= nl at Kg + k nr
        const int nr = 4 * nb, nvec = nr / VEC;
        int nl = (int)(g.kbytes / ((size_t)nr * sizeof(T)));
        nl = min(nl, nu);
        T* kept = a.keep != nullptr ? a.keep + (int64_t)b * nu * nr : nullptr;
        T* Kg = kept ? kept : a.scratch + (int64_t)blockIdx.x * g.sstride - (int64_t)nl * nr;
        if (tid == 0) {   // local block row of the seed: the list is ascending
            int lo = 0, hi = nb - 1;
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (list[mid] < j / 4) lo = mid + 1;
                else hi = mid;
            }
            misc[1] = lo;
        }
        __syncthreads();
        const int jl = 4 * misc[1] + j % 4;
        const T u1 = (T)(1.0 / sqrt(a.diagS[j]));
        T* K0 = nl > 0 ? Kl : Kg;
        for (int i = tid; i < nr; i += nt) {
            const T v = i == jl ? u1 : (T)0;
            u[i] = v;
            K0[i] = v;
            if (kept && nl > 0) kept[i] = v;
        }
        if (tid < 4) u[nr + tid] = y[nr + tid] = z[nr + tid] = (T)0;

        // Row i of a product: its first CH blocks' values and local columns (the zeros behind the rows for a block
        // outside the set or past the row's end). A thread's first row keeps its columns for the whole solve.
        constexpr int CH = 5;
        T wv[CH][4];
        int jc[CH], voff, rlen;
        auto row_columns = [&](int i, int t0, int (&J)[CH], int& vo, int& l) {
            const int I = i >> 2, lo = lptr[I];
            l = lptr[I + 1] - lo;
            vo = gptr[I] * 16 + (i & 3) * 4;
#pragma unroll
            for (int t = 0; t < CH; ++t) J[t] = t0 + t < l ? lcol[lo + t0 + t] : nb;
        };
        auto row_values = [&](const T* __restrict__ val, int vo, int l, int t0) {
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int tt = max(0, min(t0 + t, l - 1));
                const VT* vp = reinterpret_cast<const VT*>(val + (int64_t)vo + tt * 16);
#pragma unroll
                for (int q = 0; q < 4 / VEC; ++q) {
                    T o[VEC];
                    unpack(vp[q], o);
#pragma unroll
                    for (int c = 0; c < VEC; ++c) wv[t][q * VEC + c] = o[c];
                }
            }
        };
        __syncthreads();
        row_columns(min(tid, nr - 1), 0, jc, voff, rlen);
        // out[i] = sum over the row's blocks of val x. The first row's values were requested before the barrier
        // ahead of this (prefetch), so that their latency overlaps the phase before.
        auto prefetch = [&](const T* __restrict__ val) { row_values(val, voff, rlen, 0); };
        auto product = [&](const T* __restrict__ val, const T* x, T* out) {
            auto blocks = [&](const int (&J)[CH], T s) {
                T xv[CH][4];
#pragma unroll
                for (int t = 0; t < CH; ++t)
#pragma unroll
                    for (int q = 0; q < 4 / VEC; ++q) {
                        T o[VEC];
                        unpack(reinterpret_cast<const VT*>(x + 4 * J[t])[q], o);
#pragma unroll
                        for (int c = 0; c < VEC; ++c) xv[t][q * VEC + c] = o[c];
                    }
#pragma unroll
                for (int t = 0; t < CH; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) s = fma(wv[t][c], xv[t][c], s);
                return s;
            };
            for (int i = tid; i < nr; i += nt) {
                int J[CH], vo = voff, l = rlen;
#pragma unroll
                for (int t = 0; t < CH; ++t) J[t] = jc[t];
                if (i != tid) {
                    row_columns(i, 0, J, vo, l);
                    row_values(val, vo, l, 0);
                }
                T s = blocks(J, (T)0);
                for (int t0 = CH; t0 < l; t0 += CH) {
                    row_columns(i, t0, J, vo, l);
                    row_values(val, vo, l, t0);
                    s = blocks(J, s);
                }
                out[i] = s;
            }
        };
        // o0[k] = u_k . x0 (and o1[k] = u_k . x1) for k < nk: wavefronts over pairs of a group of basis vectors (in LDS,
        // then in memory) and a chunk of the rows, lanes over the rows with their x in registers; sums of a lane in T,
        // across lanes in FP64. Sums of several chunks meet in cp, one barrier later. (Wavefronts over the groups alone
        // left half of them idle at 2048 rows and nu = 30, where the chunks are four.) The last sums, rounded, are the
        // update coefficients cT.
        const int nlv = (nvec + 63) / 64, nch = (nlv + SEED_NF - 1) / SEED_NF, cf = (nlv + nch - 1) / nch;   // equal chunks
        auto groups = [&](int nk) {
            return (min(nk, nl) + SEED_G - 1) / SEED_G + (nk > nl ? (nk - nl + SEED_G - 1) / SEED_G : 0);
        };
        auto dots = [&](auto two, const T* x0, const T* x1, int nk, double* o0, double* o1) {
            constexpr int NR = decltype(two)::value ? 2 : 1;
            constexpr int V = SEED_G * NR;
            const int kl = min(nk, nl), gl = (kl + SEED_G - 1) / SEED_G, ng = groups(nk);
            for (int ch = 0; ch < nch; ++ch) {
                const int c0 = ch * 64 * cf, first = (wave - ch * ng) & (nw - 1);
                if (first >= ng) continue;
                T f0[SEED_NF][VEC], f1[SEED_NF][VEC];
                int vs[SEED_NF];
                const int nf = min(cf, nlv - ch * cf);
#pragma unroll
                for (int f = 0; f < SEED_NF; ++f) {
                    const int v = c0 + f * 64 + lane;
                    const bool in = v < nvec;
                    vs[f] = in ? v : 0;
                    unpack(reinterpret_cast<const VT*>(x0)[vs[f]], f0[f]);
                    if constexpr (NR == 2) unpack(reinterpret_cast<const VT*>(x1)[vs[f]], f1[f]);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) {
                        f0[f][i] = in ? f0[f][i] : (T)0;
                        if constexpr (NR == 2) f1[f][i] = in ? f1[f][i] : (T)0;
                    }
                }
                auto group = [&](const T* base, int kb, int kz) {
                    AT acc[V];
#pragma unroll
                    for (int i = 0; i < V; ++i) acc[i] = (AT)0;
                    T k4[SEED_G][VEC];
#pragma unroll
                    for (int f = 0; f < SEED_NF; ++f) {
                        if (f >= nf) break;
#pragma unroll
                        for (int q = 0; q < SEED_G; ++q) {
                            const int k = kb + q < kz ? kb + q : kz - 1;
                            unpack(reinterpret_cast<const VT*>(base + (int64_t)k * nr)[vs[f]], k4[q]);
                        }
#pragma unroll
                        for (int q = 0; q < SEED_G; ++q)
#pragma unroll
                            for (int i = 0; i < VEC; ++i) {
                                acc[q * NR] = fma((AT)k4[q][i], (AT)f0[f][i], acc[q * NR]);
                                if constexpr (NR == 2) acc[q * NR + 1] =
                                    fma((AT)k4[q][i], (AT)f1[f][i], acc[q * NR + 1]);
                            }
                    }
                    double s[V];
#pragma unroll
                    for (int i = 0; i < V; ++i) s[i] = (double)acc[i];
                    wave_sum_multi<V>(s, lane);
                    constexpr int LPV = 64 / V;
                    const int idx = lane / LPV, k = kb + idx / NR;
                    if (lane % LPV == 0 && k < kz) {
                        const bool second = NR == 2 && idx % NR == 1;
                        if (nch > 1) {
                            cp[(2 * ch + (second ? 1 : 0)) * nu + k] = s[0];
                        } else {
                            (second ? o1 : o0)[k] = s[0];
                            if (idx % NR == NR - 1) cT[k] = (T)s[0];
                        }
                    }
                };
                int g = first;
                for (; g < gl; g += nw) group(Kl, g * SEED_G, kl);
                for (; g < ng; g += nw) group(Kg, nl + (g - gl) * SEED_G, nk);
            }
            if (nch > 1) {
                lds_barrier();
                for (int k = tid; k < nk; k += nt) {
                    double t0 = 0.0, t1 = 0.0;
                    for (int ch = 0; ch < nch; ++ch) {
                        t0 += cp[2 * ch * nu + k];
                        if constexpr (NR == 2) t1 += cp[(2 * ch + 1) * nu + k];
                    }
                    o0[k] = t0;
                    if constexpr (NR == 2) o1[k] = t1;
                    cT[k] = (T)(NR == 2 ? t1 : t0);
                }
            }
        };
        // rb (y - K cT) into o0 and o1. A wavefront takes 16 vectors of 16 bytes; its four rows of 16 lanes take the
        // basis vectors k = 0, 1, 2, 3 modulo 4, and their sums meet through lane exchanges.
        auto update = [&](int nk, double rb, T* o0, T* o1) {
            const int part = lane >> 4;
            for (int v0 = wave * 16; v0 < nvec; v0 += nw * 16) {
                const int v = v0 + (lane & 15), vs = v < nvec ? v : 0;
                AT acc[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = (AT)0;
                auto range = [&](const T* base, int ka, int kz) {
                    for (int kb = ka; kb < kz; kb += SEED_KP * SEED_UN) {
                        T e[SEED_UN][VEC], c[SEED_UN];
#pragma unroll
                        for (int q = 0; q < SEED_UN; ++q) {
                            if (kb + SEED_KP * q >= kz) break;
                            const int k = kb + SEED_KP * q + part, ks = min(k, kz - 1);
                            unpack(reinterpret_cast<const VT*>(base + (int64_t)ks * nr)[vs], e[q]);
                            c[q] = k < kz ? cT[ks] : (T)0;
                        }
#pragma unroll
                        for (int q = 0; q < SEED_UN; ++q) {
                            if (kb + SEED_KP * q >= kz) break;
#pragma unroll
                            for (int i = 0; i < VEC; ++i) acc[i] = fma((AT)e[q][i], (AT)c[q], acc[i]);
                        }
                    }
                };
                range(Kl, 0, min(nk, nl));
                range(Kg, nl, nk);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = swap_add16(acc[i], acc[i]);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = swap_add32(acc[i], acc[i]);
                if (part == 0 && v < nvec) {
                    T yv[VEC];
                    unpack(reinterpret_cast<const VT*>(y)[v], yv);
#pragma unroll
                    for (int i = 0; i < VEC; ++i) yv[i] = (T)((double)(T)((AT)yv[i] - acc[i]) * rb);
                    reinterpret_cast<VT*>(o0)[v] = pack(yv);
                    reinterpret_cast<VT*>(o1)[v] = pack(yv);
                }
            }
        };
        // y . z in FP64, by one wavefront
        auto self_dot = [&]() {
            double s = 0.0;
            for (int v = lane; v < nvec; v += 64) {
                T p[VEC], q[VEC];
                unpack(reinterpret_cast<const VT*>(y)[v], p);
                unpack(reinterpret_cast<const VT*>(z)[v], q);
#pragma unroll
                for (int i = 0; i < VEC; ++i) s += (double)p[i] * (double)q[i];
            }
            return wave_sum(s);
        };

        double* hb = a.h + (int64_t)b * nu * nu;
        int m = nu;
        // The step's order keeps no requested values alive across the loop's back edge, where the compiler would wait
        // for them: S w, the two passes, then H u_{n+1}.
        prefetch(a.hv);
        product(a.hv, u, y);
        for (int nk = 1;; ++nk) {   // basis vectors so far; y = H u_nk
            const int n = nk - 1;
            if (nk == nu) {
                __syncthreads();
                dots(std::false_type{}, y, y, nk, d0, d0);
                lds_barrier();
                for (int k = tid; k < nk; k += nt) hb[(int64_t)k * nu + n] = d0[k];
                break;
            }
            prefetch(a.sv);
            lds_barrier();
            product(a.sv, y, z);
            __syncthreads();   // also the newest basis vector's store to global memory, two phases ago
            dots(std::true_type{}, y, z, nk, d0, d1);   // K^T w and c1 = K^T S w
            lds_barrier();
            for (int k = tid; k < nk; k += nt) hb[(int64_t)k * nu + n] = d0[k];
            prefetch(a.sv);
            update(nk, 1.0, y, y);                      // first pass
            lds_barrier();
            product(a.sv, y, z);
            lds_barrier();
            if (wave == (groups(nk) * nch & (nw - 1))) {   // the next wavefront after the groups'
                const double s = self_dot();
                if (lane == 0) d1[nu] = s;
            }
            dots(std::false_type{}, z, z, nk, d0, d0);   // c2
            prefetch(a.hv);
            lds_barrier();
            double s1 = 0.0, s2 = 0.0;                  // |c1|^2, |c2|^2 in every wavefront: the same sums
            for (int k = lane; k < nk; k += 64) {
                s1 += d1[k] * d1[k];
                s2 += d0[k] * d0[k];
            }
            s1 = wave_sum(s1);
            s2 = wave_sum(s2);
            const double ww = d1[nu];                   // w^T S w after the first pass
            if (!(ww >= 0.0) || !(ww < INFINITY)) {
                m = -1;
                break;
            }
            T* Kn = (nk < nl ? Kl : Kg) + (int64_t)nk * nr;
            // beta^2 = w^T S w - |c2|^2 after the second pass (K^T S K = I), unless c2 is a visible part of w (near
            // a breakdown), where it is formed from the vector itself
            if (s2 <= 1e-4 * ww) {
                const double bb = ww - s2;
                if (bb <= a.tau * a.tau * (s1 + s2 + bb)) {
                    m = nk;
                    break;
                }
                update(nk, rsqrt_nr(bb), u, Kn);
                lds_barrier();
            } else {
                update(nk, 1.0, y, y);
                lds_barrier();
                row_values(a.sv, voff, rlen, 0);
                product(a.sv, y, z);
                lds_barrier();
                const double bb = self_dot();           // every wavefront: the same value
                if (!(bb >= 0.0) || !(bb < INFINITY)) m = -1;
                else if (bb <= a.tau * a.tau * (s1 + s2 + bb)) m = nk;
                if (m != nu) break;
                const double rb = rsqrt_nr(bb);
                for (int i = tid; i < nr; i += nt) u[i] = Kn[i] = (T)((double)y[i] * rb);
                row_values(a.hv, voff, rlen, 0);
                lds_barrier();
            }
            if (kept && nk < nl)
                for (int i = tid; i < nr; i += nt) kept[(int64_t)nk * nr + i] = u[i];
            product(a.hv, u, y);
        }
        __syncthreads();
        if (tid == 0) a.nu_out[b] = m;
        if (m <= 0) continue;
        // rows K[P(j), :] of the seed: the blocks of its block row, zero outside the region
        const int I = misc[1], nP = a.Hrp[j + 1] - a.Hrp[j];
        for (int idx = tid; idx < m * nP; idx += nt) {
            const int k = idx / nP, t = idx - k * nP;
            const int J = lcol[lptr[I] + t / 4];
            double v = 0.0;
            if (J < nb) v = k < nl ? (double)Kl[(int64_t)k * nr + 4 * J + t % 4] : (double)Kg[(int64_t)k * nr + 4 * J + t % 4];
            a.Kp[((int64_t)b * nu + k) * a.max_row + t] = v;
        }
        if (a.vref != nullptr) {   // whole cells only: local rows are global rows
            for (int k = wave; k < nu; k += nw) {
                double s = 0.0;
                if (k < m) {
                    if (k < nl)
                        for (int i = lane; i < nr; i += 64) s += (double)Kl[(int64_t)k * nr + i] * a.vref[i];
                    else
                        for (int i = lane; i < nr; i += 64) s += (double)Kg[(int64_t)k * nr + i] * a.vref[i];
                }
                s = wave_sum(s);
                if (lane == 0) a.pref[(int64_t)k * a.pB + b] = s;
            }
        }
    }
}

SeedGeom seed_geometry(int64_t nbrow, int64_t nnzb, int blocks_per_row, int hops, int64_t nbcap, int nu, size_t elem,
                       int64_t ns, int n_cu) {
    SeedGeom g;
    g.ok = false;
    g.nbrow = nbrow;
    if (nbcap < 1 || nbcap > SEED_MAX_BLOCKS) return g;
    g.nbcap = (int)nbcap;
    const int64_t nr = 4 * nbcap;
    const int64_t ecap = hops < 0 ? nnzb : nbcap * blocks_per_row;
    g.hs = 1;
    while (hops >= 0 && g.hs < 2 * (int)nbcap) g.hs *= 2;
    const size_t tables = hops < 0 ? 0 : (size_t)(2 * g.hs + (int)nbcap) * 4;
    auto up = [](size_t x) { return (x + 15) & ~(size_t)15; };
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off += up(b);
        return (int)o;
    };
    const int oU = take((size_t)3 * (nr + 4) * elem);
    const int64_t nch = (nr * (int64_t)elem / 16 + 64 * SEED_NF - 1) / (64 * SEED_NF);
    const int oP = take(nch > 1 ? (size_t)nch * 2 * nu * 8 : 0);
    const int oD = take((size_t)2 * (nu + 1) * 8), oC = take((size_t)nu * elem);
    const int oL = take((size_t)(3 * nbcap + 1 + 8) * 4), oCol = take((size_t)ecap * 2);
    const size_t fixed = off, slab = (size_t)nr * elem;
    // As many workgroups per compute unit (4, 2 or 1, sharing SEED_WG threads) as there are seeds for and as keep
    // every basis vector in LDS; a basis that does not fit gets the whole LDS of a compute unit.
    for (int wgs = ns > 2 * n_cu ? 4 : (ns > n_cu ? 2 : 1); wgs >= 1; wgs /= 2) {
        const size_t total = (size_t)160 * 1024 / wgs;
        const size_t kb = std::max(up(tables), up((size_t)nu * slab));
        if (fixed + kb > total && (wgs > 1 || fixed + up(tables) > total)) continue;
        g.threads = SEED_WG / wgs;
        g.kbytes = std::min(kb, (total - fixed) & ~(size_t)15);
        g.oU = (int)g.kbytes + oU;
        g.oP = (int)g.kbytes + oP;
        g.oD = (int)g.kbytes + oD;
        g.oC = (int)g.kbytes + oC;
        g.oList = (int)g.kbytes + oL;
        g.oCol = (int)g.kbytes + oCol;
        g.lds = g.kbytes + fixed;
        g.grid = (int)std::min<int64_t>(ns, (int64_t)n_cu * wgs);
        // the kernel keeps as many vectors of its seed's own row count in LDS; the largest set leaves the most out
        // (a smaller one at most as many elements)
        const int64_t nl = std::min<int64_t>(nu, (int64_t)(g.kbytes / slab));
        g.sstride = ((int64_t)nu - nl) * nr;
        g.ok = true;
        return g;
    }
    return g;
}

template <typename T>
static LaunchInfo launch_seed_t(const SeedGeom& g, const DevMat& H, const DevMat& SH, int64_t M, const double* diagS,
                                const int32_t* seeds, int ns, int nu, int hops, double tau, T* scratch,
                                const int32_t* Hrp, int max_row, double* h, double* Kp, int32_t* nu_out,
                                const double* vref, double* pref, int64_t pB, T* keep, bool acc64, hipStream_t s) {
    LaunchInfo li;
    if (!g.ok || !H.bsr || SH.nnz != H.nnz || H.n != g.nbrow) {
        li.wgs = -1;
        return li;
    }
    constexpr bool F32 = std::is_same<T, float>::value;
    SeedArgs<T> a{g, M, H.ptr, H.idx, F32 ? (const T*)H.v32 : (const T*)H.v64, F32 ? (const T*)SH.v32 : (const T*)SH.v64,
                  diagS, seeds, ns, nu, hops, tau, scratch, Hrp, max_row, h, Kp, nu_out, vref, pref, pB, keep};
    if (F32 && acc64) {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void*)k_seed<T, F32>, done);
        hipLaunchKernelGGL((k_seed<T, F32>), dim3(g.grid), dim3(g.threads), g.lds, s, a);
    } else {
        static std::atomic<uint64_t> done{0};
        allow_full_lds((const void*)k_seed<T, false>, done);
        hipLaunchKernelGGL((k_seed<T, false>), dim3(g.grid), dim3(g.threads), g.lds, s, a);
    }
    li.wgs = g.grid;
    // operands and results once: both matrices on the rows that the seeds can reach, the subspace matrices, the gathered
    // rows, a kept basis (the basis itself stays in LDS and the caches: its sweeps there are not counted)
    const double rows = 4.0 * g.nbcap, el = sizeof(T);
    const double part = std::min(1.0, (double)ns * g.nbcap / (double)H.n);
    li.bytes = part * ((double)H.nnz * (32.0 * el + 4.0) + (double)H.n * 4.0) +
               (double)ns * nu * (0.5 * (nu + 1.0) + max_row) * 8.0 + (keep ? (double)ns * nu * rows * el : 0.0);
    li.flops = (double)ns * rows * (5.0 * nu * (nu + 1.0) + 6.0 * nu * 4.0 * ((double)H.nnz / (double)H.n));
    return li;
}

template <>
LaunchInfo launch_seed<float>(const SeedGeom& g, const DevMat& H, const DevMat& SH, int64_t M, const double* diagS,
                              const int32_t* seeds, int ns, int nu, int hops, double tau, float* scratch,
                              const int32_t* Hrp, int max_row, double* h, double* Kp, int32_t* nu_out,
                              const double* vref, double* pref, int64_t pB, float* keep, bool acc64,
                              hipStream_t s) {
    return launch_seed_t<float>(g, H, SH, M, diagS, seeds, ns, nu, hops, tau, scratch, Hrp, max_row, h, Kp, nu_out, vref,
                                pref, pB, keep, acc64, s);
}
template <>
LaunchInfo launch_seed<double>(const SeedGeom& g, const DevMat& H, const DevMat& SH, int64_t M, const double* diagS,
                               const int32_t* seeds, int ns, int nu, int hops, double tau, double* scratch,
                               const int32_t* Hrp, int max_row, double* h, double* Kp, int32_t* nu_out,
                               const double* vref, double* pref, int64_t pB, double* keep, bool acc64,
                               hipStream_t s) {
    return launch_seed_t<double>(g, H, SH, M, diagS, seeds, ns, nu, hops, tau, scratch, Hrp, max_row, h, Kp, nu_out, vref,
                                 pref, pB, keep, acc64, s);
}

// ---------------------------------------------------------------------------
// Eigen states on the basis kept by a first pass, [seed][nu][nr]. k_es_dots: pref[k * ns + seed] = u_k . v_ref, a
// workgroup per seed, a wavefront per vector; bound by the reads of the basis (1 GB for 2048 seeds at nu = 30, FP64: 0.17 ms, 5.8 TB/s).
template <typename T>
__global__ __launch_bounds__(WG) void k_es_dots(const T* __restrict__ keep, int64_t nr, int nu,
                                                const int32_t* __restrict__ nu_eff, const double* __restrict__ vref,
                                                double* __restrict__ pref) {
    typedef typename Vec16<T>::type VT;
    constexpr int VEC = Vec16<T>::n;
    const int b = blockIdx.x, lane = threadIdx.x & 63, ns = gridDim.x, m = nu_eff[b];
    for (int k = threadIdx.x >> 6; k < nu; k += WG / 64) {
        double s = 0.0;
        if (k < m) {
            const VT* u = reinterpret_cast<const VT*>(keep + ((int64_t)b * nu + k) * nr);
            for (int v = lane; v < nr / VEC; v += 64) {
                T e[VEC];
                unpack(u[v], e);
#pragma unroll
                for (int i = 0; i < VEC; ++i) s += (double)e[i] * vref[v * VEC + i];
            }
            s = wave_sum(s);
        }
        if (lane == 0) pref[(int64_t)k * ns + b] = s;
    }
}

// The kept basis, subspace matrix, gathered rows and dimension of the reference seed (ref[0]: its place) on their own.
template <typename T>
__global__ __launch_bounds__(WG) void k_es_take(const int32_t* __restrict__ ref, const T* __restrict__ keep, int64_t nK,
                                                const double* __restrict__ h, int64_t nh, const double* __restrict__ Kp,
                                                int64_t nKp, const int32_t* __restrict__ nu_eff, T* __restrict__ keep1,
                                                double* __restrict__ h1, double* __restrict__ Kp1,
                                                int32_t* __restrict__ nu1) {
    const int64_t b = ref[0], i0 = (int64_t)blockIdx.x * WG + threadIdx.x, st = (int64_t)gridDim.x * WG;
    for (int64_t i = i0; i < nK; i += st) keep1[i] = keep[b * nK + i];
    for (int64_t i = i0; i < nh; i += st) h1[i] = h[b * nh + i];
    for (int64_t i = i0; i < nKp; i += st) Kp1[i] = Kp[b * nKp + i];
    if (i0 == 0) nu1[0] = nu_eff[b];
}

template <typename T>
LaunchInfo launch_es_dots(const T* keep, int64_t nr, int nu, int ns, const int32_t* nu_eff, const double* vref,
                          double* pref, hipStream_t s) {
    hipLaunchKernelGGL((k_es_dots<T>), dim3(ns), dim3(WG), 0, s, keep, nr, nu, nu_eff, vref, pref);
    LaunchInfo li;
    li.wgs = ns;
    li.bytes = (double)ns * nu * nr * sizeof(T);
    li.flops = 2.0 * ns * nu * nr;
    return li;
}
template <typename T>
LaunchInfo launch_es_take(const int32_t* ref, const T* keep, int64_t nr, int nu, int max_row, const double* h,
                          const double* Kp, const int32_t* nu_eff, T* keep1, double* h1, double* Kp1, int32_t* nu1,
                          hipStream_t s) {
    hipLaunchKernelGGL((k_es_take<T>), dim3(128), dim3(WG), 0, s, ref, keep, nr * nu, h, (int64_t)nu * nu, Kp,
                       (int64_t)nu * max_row, nu_eff, keep1, h1, Kp1, nu1);
    LaunchInfo li;
    li.wgs = 128;
    li.bytes = 2.0 * ((double)nr * nu * sizeof(T) + (double)nu * (nu + max_row) * 8.0);
    return li;
}
#define MAR_ES(T)                                                                                                     \
    template LaunchInfo launch_es_dots<T>(const T*, int64_t, int, int, const int32_t*, const double*, double*, hipStream_t); \
    template LaunchInfo launch_es_take<T>(const int32_t*, const T*, int64_t, int, int, const double*, const double*,  \
                                          const int32_t*, T*, double*, double*, int32_t*, hipStream_t);
MAR_ES(float)
MAR_ES(double)
#undef MAR_ES

// ---------------------------------------------------------------------------
// Largest number of block rows within h hops of any block row, h = 0 .. depth, or cap + 1 where some set is larger than
// cap: a workgroup per block row, its set in a hash table in LDS, every level of one search.
__global__ __launch_bounds__(WG) void k_region_sizes(int64_t nbrow, const int32_t* __restrict__ brp,
                                                     const int32_t* __restrict__ bcol, int depth, int cap, int hs,
                                                     int32_t* __restrict__ out) {
    extern __shared__ int shm[];
    int* key = shm;
    int* raw = key + hs;
    int* best = raw + cap;
    __shared__ int cnt;
    const int tid = threadIdx.x;
    for (int k = tid; k <= depth; k += WG) best[k] = 0;
    for (int64_t I0 = blockIdx.x; I0 < nbrow; I0 += gridDim.x) {
        for (int i = tid; i < hs; i += WG) key[i] = -1;
        __syncthreads();
        auto slot0 = [&](int I) { return (int)(((unsigned)I * 2654435761u) >> 7) & (hs - 1); };
        if (tid == 0) {
            key[slot0((int)I0)] = (int)I0;
            raw[0] = (int)I0;
            cnt = 1;
        }
        __syncthreads();
        int f0 = 0, f1 = 1, h = 0;
        for (;;) {
            if (tid == 0) best[h] = max(best[h], f1);
            // no further level: the set is complete or too large, or an earlier one was too large from there on
            if (h == depth || f0 == f1 || f1 > cap || best[h + 1] > cap) break;
            for (int e = f0 + tid; e < f1; e += WG) {
                const int I = raw[e];
                for (int p = brp[I]; p < brp[I + 1] && atomicAdd(&cnt, 0) <= cap; ++p) {
                    const int J = bcol[p];
                    int s = slot0(J);
                    // WG lanes stop adding once cap + 1 keys are in: at most cap + WG + 1 of hs >= 2 (cap + WG) slots fill
                    for (;;) {
                        const int old = atomicCAS(&key[s], -1, J);
                        if (old == -1) {
                            const int at = atomicAdd(&cnt, 1);
                            if (at < cap) raw[at] = J;
                            break;
                        }
                        if (old == J) break;
                        s = (s + 1) & (hs - 1);
                    }
                }
            }
            __syncthreads();
            f0 = f1;
            f1 = min(cnt, cap + 1);
            ++h;
            __syncthreads();
        }
        for (int k = h + 1 + tid; k <= depth; k += WG) best[k] = max(best[k], f1);
        __syncthreads();
    }
    for (int k = tid; k <= depth; k += WG) atomicMax(&out[k], best[k]);
}

__global__ void k_region_init(int32_t* out, int n) {
    for (int i = threadIdx.x; i < n; i += WG) out[i] = 0;
}

LaunchInfo launch_region_sizes(int64_t nbrow, const int32_t* brp, const int32_t* bcol, int depth, int cap, int32_t* out,
                               hipStream_t s) {
    int hs = 1;
    while (hs < 2 * (cap + WG)) hs *= 2;
    hipLaunchKernelGGL(k_region_init, dim3(1), dim3(WG), 0, s, out, depth + 1);
    const unsigned wgs = (unsigned)std::min<int64_t>(nbrow, 2048);
    hipLaunchKernelGGL(k_region_sizes, dim3(wgs), dim3(WG), (size_t)(hs + cap + depth + 1) * 4, s, nbrow, brp, bcol, depth,
                       cap, hs, out);
    LaunchInfo li;
    li.wgs = wgs;
    return li;
}

}  // namespace mar
