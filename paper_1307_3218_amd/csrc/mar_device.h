// Device helpers shared by the streaming kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace mar {

// 16-byte vector of T: one global_load/store_dwordx4 per lane.
template <typename T> struct Vec16;
template <> struct Vec16<float> { typedef float4 type; static constexpr int n = 4; };
template <> struct Vec16<double> { typedef double2 type; static constexpr int n = 2; };

__device__ __forceinline__ void unpack(const float4& v, float (&a)[4]) { a[0] = v.x; a[1] = v.y; a[2] = v.z; a[3] = v.w; }
__device__ __forceinline__ void unpack(const double2& v, double (&a)[2]) { a[0] = v.x; a[1] = v.y; }
__device__ __forceinline__ float4 pack(const float (&a)[4]) { return make_float4(a[0], a[1], a[2], a[3]); }
__device__ __forceinline__ double2 pack(const double (&a)[2]) { return make_double2(a[0], a[1]); }

// Non-temporal 16-byte loads (streamed data that should not displace reused lines in L2).
typedef float nf4 __attribute__((ext_vector_type(4)));
typedef double nd2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void unpack_nt(const float4* p, float (&a)[4]) {
    const nf4 v = __builtin_nontemporal_load(reinterpret_cast<const nf4*>(p));
    a[0] = v.x; a[1] = v.y; a[2] = v.z; a[3] = v.w;
}
__device__ __forceinline__ void unpack_nt(const double2* p, double (&a)[2]) {
    const nd2 v = __builtin_nontemporal_load(reinterpret_cast<const nd2*>(p));
    a[0] = v.x; a[1] = v.y;
}

// Non-temporal 16-byte stores: results that only later kernels read, kept from displacing the lines
// that the storing kernel still reuses from L2.
__device__ __forceinline__ void store_nt(float4* p, const float (&a)[4]) {
    const nf4 v = {a[0], a[1], a[2], a[3]};
    __builtin_nontemporal_store(v, reinterpret_cast<nf4*>(p));
}
__device__ __forceinline__ void store_nt(double2* p, const double (&a)[2]) {
    const nd2 v = {a[0], a[1]};
    __builtin_nontemporal_store(v, reinterpret_cast<nd2*>(p));
}

// Seed-interleaved vectors: element e of an [M][B] array belongs to row e / B
// and seed e % B. A lane owns one 16-byte vector of VEC elements:
//   B >= VEC: the vector covers seeds (lane_vector_index % P) * VEC + [0, VEC),
//             P = B / VEC lanes share a row;
//   B <  VEC: the vector covers VEC / B rows of all B seeds; element i is seed i % B.
template <typename T, int B>
struct SeedMap {
    static constexpr int VEC = Vec16<T>::n;
    static constexpr int SW = B < VEC ? B : VEC;   // seeds per lane after folding
    static constexpr int P = B < VEC ? 1 : B / VEC; // lanes per row (distinct seed groups)
    static_assert(P <= 64, "B too large for one wavefront per row group");
};

// Map a hardware workgroup id to a logical one so that consecutive logical ids
// run on the same XCD (the dispatcher deals workgroups round-robin over 8 XCDs,
// each with its own L2). Bijective on [0, n).
__device__ __forceinline__ int64_t xcd_remap(int64_t bid, int64_t n) {
    constexpr int NX = 8;
    const int64_t per = n / NX, rem = n % NX;
    const int64_t x = bid % NX, local = bid / NX;
    return x * per + (x < rem ? x : rem) + local;
}

// Chunk-interleaved order: the dispatcher deals workgroup ids round-robin over the 8 XCDs, and XCD x takes
// the x-th chunk of each run of 8 chunks of `chunk` consecutive tiles, in order. When a run of 8 chunks
// spans the distance to a row's far neighbours (the next plane of cells of a lattice), those neighbours
// were read by the same XCD one chunk earlier instead of a whole contiguous range away. Bijective on
// [0, 8 * chunk * k); ids past the real tiles are skipped by the caller.
__device__ __forceinline__ int64_t xcd_chunk(int64_t bid, int64_t chunk) {
    constexpr int NX = 8;
    const int64_t x = bid % NX, l = bid / NX;
    return ((l / chunk) * NX + x) * chunk + l % chunk;
}

// 1/x and 1/sqrt(x) (x > 0, normal) from the hardware estimates and two Newton steps each (full FP64
// precision: the estimates carry about 23 bits and each step doubles them).
__device__ __forceinline__ double recip(double x) {
    double y = __builtin_amdgcn_rcp(x);
    double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
    e = fma(-x, y, 1.0);
    return fma(y, e, y);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

// Moves between lanes without LDS. dpp_move<CTRL>(v): v of the lane that the DPP control names (0xb1: lane ^ 1, 0x4e:
// lane ^ 2, 0x141: 7 - lane within eight lanes, 0x140: 15 - lane within a row of 16, 0x128: lane ^ 8).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// v of lane k (k the same in every lane).
__device__ __forceinline__ double read_lane(double v, int k) {
    const uint64_t x = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, k);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), k);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Lanes 0..31: a + a of lane + 32; lanes 32..63: b + b of lane - 32.
__device__ __forceinline__ double swap_add32(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
// Lanes with bit 4 clear: a + a of lane + 16; the others: b + b of lane - 16.
__device__ __forceinline__ double swap_add16(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ float swap_add32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned x = r[0], y = r[1];   // (a bit cast of the vector's element itself reads element 0)
    return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
}
__device__ __forceinline__ float swap_add16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned x = r[0], y = r[1];   // (a bit cast of the vector's element itself reads element 0)
    return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
}
// Sum over a wavefront, the same bits in every lane (each exchange adds the same two operands in both lanes).
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0xb1>(v);
    v += dpp_move<0x4e>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    v = swap_add16(v, v);
    return swap_add32(v, v);
}

// Barrier that orders LDS only: loads and stores of global memory stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Workgroup reduction of per-seed partial sums (fixed order, deterministic).
// Thread t holds vals[v][i] for seed (t % P) * SW + i. For every v and every
// seed b in [0, P*SW) the sum over the workgroup's 256 threads is passed to
// emit(v, b, sum) by exactly one thread (always the same thread for a given
// (v, b)). Values cross waves through LDS in chunks of SeedReduce::NVC values,
// so the exchange buffer holds SeedReduce::LDS elements whatever NV is.
template <int P, int SW, int NV>
struct SeedReduce {
    static constexpr int NVC_RAW = 768 / (P * SW);
    static constexpr int NVC = NVC_RAW < 1 ? 1 : (NVC_RAW > NV ? NV : NVC_RAW);
    static constexpr int LDS = 4 * NVC * P * SW;
};

template <int P, int SW, int NV, typename A, typename F>
__device__ __forceinline__ void wg_seed_reduce(A (&vals)[NV][SW], A* lds, F&& emit) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if constexpr (P < 64) {
#pragma unroll
        for (int off = P; off < 64; off <<= 1) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int i = 0; i < SW; ++i) vals[v][i] += __shfl_xor(vals[v][i], off);
        }
    }
    constexpr int NVC = SeedReduce<P, SW, NV>::NVC;
    constexpr int TOT = NVC * P * SW;
#pragma unroll
    for (int c0 = 0; c0 < NV; c0 += NVC) {
        if (lane < P) {
#pragma unroll
            for (int v = 0; v < NVC; ++v)
                if (c0 + v < NV) {
#pragma unroll
                    for (int i = 0; i < SW; ++i) lds[wave * TOT + (v * P + lane) * SW + i] = vals[c0 + v][i];
                }
        }
        __syncthreads();
        for (int o = threadIdx.x; o < TOT; o += 256) {
            const int v = c0 + o / (P * SW);
            if (v < NV) {
                A s = lds[o];
                s += lds[TOT + o];
                s += lds[2 * TOT + o];
                s += lds[3 * TOT + o];
                emit(v, o % (P * SW), s);
            }
        }
        __syncthreads();
    }
}

// Lets kernel f use up to `bytes` of dynamic LDS (160 KB less its static LDS at most). The attribute belongs to the
// current device, so it is set once per device (bit d of done for device d; concurrent first calls both set it, which is
// harmless).
inline void allow_lds(const void* f, std::atomic<uint64_t>& done, int bytes) {
    int dev = 0;
    const bool known = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64;
    const uint64_t bit = known ? 1ull << dev : 0;
    if (known && (done.load(std::memory_order_acquire) & bit)) return;
    (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (known) done.fetch_or(bit, std::memory_order_acq_rel);
}

inline void allow_full_lds(const void* f, std::atomic<uint64_t>& done) { allow_lds(f, done, 160 * 1024); }

}  // namespace mar
