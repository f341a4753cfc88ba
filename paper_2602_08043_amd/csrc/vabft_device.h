// Device-side helpers shared by the HIP kernels of the V-ABFT path (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "vabft.h"

namespace vabft {

constexpr int WAVE = 64;

// ---------------------------------------------------------------------------
// element types
// ---------------------------------------------------------------------------
struct bf16_t { uint16_t bits; };
struct f16_t { _Float16 v; };
struct f8_t { uint8_t bits; };   // OCP FP8 E4M3
struct bf8_t { uint8_t bits; };  // OCP FP8 E5M2

template <typename T> struct Elem;

template <> struct Elem<bf16_t> {
    using acc_t = float;
    static constexpr int bytes = 2;
    static constexpr int vec = 8;  // elements per 16-byte chunk
    static __device__ __forceinline__ float to_acc(uint16_t raw) { return __uint_as_float(((uint32_t)raw) << 16); }
    // float -> bf16 bit pattern, round to nearest even; NaN stays NaN
    static __device__ __forceinline__ uint16_t from_acc(float x) {
        uint32_t u = __float_as_uint(x);
        if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);
        u += 0x7fffu + ((u >> 16) & 1u);
        return (uint16_t)(u >> 16);
    }
};

template <> struct Elem<f16_t> {
    using acc_t = float;
    static constexpr int bytes = 2;
    static constexpr int vec = 8;
    static __device__ __forceinline__ float to_acc(uint16_t raw) {
        _Float16 h;
        __builtin_memcpy(&h, &raw, 2);
        return (float)h;
    }
    static __device__ __forceinline__ uint16_t from_acc(float x) {
        _Float16 h = (_Float16)x;  // v_cvt_f16_f32, round to nearest even
        uint16_t r;
        __builtin_memcpy(&r, &h, 2);
        return r;
    }
};

template <> struct Elem<f8_t> {
    using acc_t = float;
    static constexpr int bytes = 1;
    static constexpr int vec = 16;  // elements per 16-byte chunk
    static __device__ __forceinline__ float to_acc(uint8_t raw) { return __builtin_amdgcn_cvt_f32_fp8((int)raw, 0); }
};

template <> struct Elem<bf8_t> {
    using acc_t = float;
    static constexpr int bytes = 1;
    static constexpr int vec = 16;
    static __device__ __forceinline__ float to_acc(uint8_t raw) { return __builtin_amdgcn_cvt_f32_bf8((int)raw, 0); }
};

template <> struct Elem<float> {
    using acc_t = float;
    static constexpr int bytes = 4;
    static constexpr int vec = 4;
};

template <> struct Elem<double> {
    using acc_t = double;
    static constexpr int bytes = 8;
    static constexpr int vec = 2;
};

// ---------------------------------------------------------------------------
// wave-level reductions (all lanes of the group end with the result)
// ---------------------------------------------------------------------------
// The partner exchanges of a butterfly (lane ^ 32, 16, 8, 4, 2, 1) as register moves: a lane swap for the halves and
// the odd and even rows of 16, a rotation inside a row for 8 and 4, a quad permutation for 2 and 1.  Through LDS
// (ds_bpermute) each of the six steps was a round trip of about 100 cycles, a large part of what a short kernel does
// after its last load.  TOP is the size of the group, steps run downwards from TOP / 2: after the step at 8 lane i and
// lane i ^ 8 agree, so rotating by 4 is as good as lane ^ 4; in a group of 8 the first step pairs lane i with lane i ^ 7
// (a mirror), after which the steps at 2 and 1 complete the group as well.  Every lane must be active.
template <int OFF, int TOP> __device__ __forceinline__ void lane_exchange(uint32_t v, uint32_t& a, uint32_t& b) {
    if constexpr (OFF == 32 || OFF == 16) {
        const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap(v, v, false, false)
                                 : __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0];  // the lower lane's value in both lanes of a pair
        b = r[1];  // the upper lane's
    } else {
        constexpr int CTRL = OFF == 8 ? 0x128 : OFF == 4 ? (TOP == 8 ? 0x141 : 0x124) : OFF == 2 ? 0x4E : 0xB1;
        a = v;
        b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
    }
}
template <int OFF, int TOP> __device__ __forceinline__ void lane_exchange(float v, float& a, float& b) {
    uint32_t x, y;
    lane_exchange<OFF, TOP>(__float_as_uint(v), x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int OFF, int TOP> __device__ __forceinline__ void lane_exchange(int v, int& a, int& b) {
    uint32_t x, y;
    lane_exchange<OFF, TOP>((uint32_t)v, x, y);
    a = (int)x;
    b = (int)y;
}
template <int OFF, int TOP> __device__ __forceinline__ void lane_exchange(double v, double& a, double& b) {
    uint32_t xl, yl, xh, yh;
    lane_exchange<OFF, TOP>((uint32_t)__double2loint(v), xl, yl);
    lane_exchange<OFF, TOP>((uint32_t)__double2hiint(v), xh, yh);
    a = __hiloint2double((int)xh, (int)xl);
    b = __hiloint2double((int)yh, (int)yl);
}
// sum over aligned groups of W lanes (a power of two)
template <int W, int TOP = W, typename T> __device__ __forceinline__ T group_sum(T v) {
    if constexpr (W > 1) {
        T a, b;
        lane_exchange<W / 2, TOP>(v, a, b);
        return group_sum<W / 2, TOP>((T)(a + b));
    } else {
        return v;
    }
}
template <int W, int TOP = W, typename T> __device__ __forceinline__ T group_max(T v) {
    if constexpr (W > 1) {
        T a, b;
        lane_exchange<W / 2, TOP>(v, a, b);
        return group_max<W / 2, TOP>(a > b ? a : b);
    } else {
        return v;
    }
}
template <int W, int TOP = W, typename T> __device__ __forceinline__ T group_min(T v) {
    if constexpr (W > 1) {
        T a, b;
        lane_exchange<W / 2, TOP>(v, a, b);
        return group_min<W / 2, TOP>(a < b ? a : b);
    } else {
        return v;
    }
}
template <typename T> __device__ __forceinline__ T wave_sum(T v) { return group_sum<WAVE>(v); }
template <typename T> __device__ __forceinline__ T wave_max(T v) { return group_max<WAVE>(v); }
template <typename T> __device__ __forceinline__ T wave_min(T v) { return group_min<WAVE>(v); }

// Partials exchanged between workgroups (which may sit on different XCDs with private L2s) go
// through device-scope relaxed atomic stores and loads: they are performed at the device's
// coherence point, so no cache write-back / invalidate fence is needed around the ticket.
// The order relied on is the hardware's, not the language's (a release fence at agent scope writes back the
// whole L2 on this chip and cost 27 us per launch):
//   1. an agent-scope atomic store is a write-through store: the issuing XCD's L2 keeps no dirty copy, the
//      value goes to the memory-side coherence point that all XCDs share;
//   2. s_waitcnt vmcnt(0) returns only when that point has acknowledged every outstanding store of the wavefront;
//   3. the workgroup barrier that follows puts all wavefronts' waits in front of the one thread's ticket
//      atomicAdd, itself executed at the same coherence point, so a workgroup that sees ticket == tiles_n - 1
//      comes after every other workgroup's partials there;
//   4. the last arriver reads the partials with agent-scope atomic loads, which are not served from its
//      XCD's L2 or the compute unit's vector cache.
// The s_waitcnt builtin and the barrier are also compiler barriers for these atomics (volatile-like side effects),
// so the compiler keeps the same order.  A back-to-back soak test on rotating inputs watches this protocol.
template <typename acc_t> struct AgentWord;
template <> struct AgentWord<float> { using u = uint32_t; };
template <> struct AgentWord<double> { using u = uint64_t; };
template <typename acc_t> __device__ __forceinline__ acc_t ld_agent(const acc_t* p) {
    using u = typename AgentWord<acc_t>::u;
    return __builtin_bit_cast(acc_t, __hip_atomic_load(reinterpret_cast<const u*>(p), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT));
}
template <typename acc_t> __device__ __forceinline__ void st_agent(acc_t* p, acc_t v) {
    using u = typename AgentWord<acc_t>::u;
    __hip_atomic_store(reinterpret_cast<u*>(p), __builtin_bit_cast(u, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Fold of the per-workgroup partials [count][3] of (S1, S2, S3) (Algorithm 1, k-loop) by the first 256
// threads of a workgroup, in the order the encode kernels use when they fold them themselves:
// thread t adds partials t, t + 256, ... in increasing order, a butterfly inside each of the four
// wavefronts, and (after a workgroup barrier) the four wavefront results in order.
// s_red: 12 doubles of LDS, [3][4].
__device__ __forceinline__ void fold_s_partials_to_lds(const double* __restrict__ partial, int count, int t,
                                                       double* s_red) {
    if (t < 256) {
        double a1 = 0, a2 = 0, a3 = 0;
        // four partials per round: their twelve loads are in flight together (one trip to memory per round, not per
        // partial), the additions stay in increasing order of b
        for (int b0 = t; b0 < count; b0 += 4 * 256) {
            double q[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int b = b0 + u * 256;
                const double* src = partial + 3 * (int64_t)(b < count ? b : t);
                q[u][0] = src[0];
                q[u][1] = src[1];
                q[u][2] = src[2];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = b0 + u * 256 < count;
                a1 = ok ? a1 + q[u][0] : a1;
                a2 = ok ? a2 + q[u][1] : a2;
                a3 = ok ? a3 + q[u][2] : a3;
            }
        }
        a1 = wave_sum(a1);
        a2 = wave_sum(a2);
        a3 = wave_sum(a3);
        if ((t & 63) == 0) {
            s_red[0 * 4 + (t >> 6)] = a1;
            s_red[1 * 4 + (t >> 6)] = a2;
            s_red[2 * 4 + (t >> 6)] = a3;
        }
    }
}
__device__ __forceinline__ double folded_s(const double* s_red, int q) {
    double v = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += s_red[q * 4 + w];
    return v;
}

// one stored element of C (FP16 for an FP8 problem), read and written in the accumulator type; _agent: past the caches
template <typename STORE, typename T> struct CElemOf {
    using store_t = STORE;
    using acc_t = typename Elem<T>::acc_t;
    static __device__ __forceinline__ acc_t from(store_t x) {
        if constexpr (std::is_same<STORE, acc_t>::value)
            return x;
        else
            return Elem<T>::to_acc(x);
    }
    static __device__ __forceinline__ store_t to(acc_t v) {
        if constexpr (std::is_same<STORE, acc_t>::value)
            return v;
        else
            return Elem<T>::from_acc(v);
    }
    static __device__ __forceinline__ acc_t get(const store_t* p) { return from(*p); }
    static __device__ __forceinline__ void put(store_t* p, acc_t v) { *p = to(v); }
    static __device__ __forceinline__ acc_t get_agent(const store_t* p) {
        if constexpr (sizeof(store_t) == 2)
            return from(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        else
            return ld_agent(p);
    }
    static __device__ __forceinline__ void put_agent(store_t* p, acc_t v) {
        if constexpr (sizeof(store_t) == 2)
            __hip_atomic_store(p, to(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else
            st_agent(p, v);
    }
};
template <typename T> struct CElem;
template <> struct CElem<bf16_t> : CElemOf<uint16_t, bf16_t> {};
template <> struct CElem<f16_t> : CElemOf<uint16_t, f16_t> {};
template <> struct CElem<f8_t> : CElemOf<uint16_t, f16_t> {};
template <> struct CElem<bf8_t> : CElemOf<uint16_t, f16_t> {};
template <> struct CElem<float> : CElemOf<float, float> {};
template <> struct CElem<double> : CElemOf<double, double> {};

// The column of a flagged row's error under the single-error-per-row model (section 2.2): D1 = C^{r1'} - C^{r1}, D2 = C^{r2'} -
// C^{r2}, column D2 / D1 - 1 for the linear weights w(k) = k + 1; -2 where that is not finite, further than 0.25 from an integer or
// outside 0..N-1 (more than one error, or an error too close to the rounding noise of the weighted sums).  by: D1.
template <typename acc_t>
__device__ __forceinline__ int locate_row(acc_t expected, acc_t expected2, acc_t rowsum, acc_t rowsum2, int N, acc_t& by) {
    const double d1 = (double)rowsum - (double)expected, d2 = (double)rowsum2 - (double)expected2;
    by = (acc_t)d1;
    if (d1 != 0.0 && isfinite(d1) && isfinite(d2)) {
        const double q = d2 / d1 - 1.0, j = rint(q);
        if (isfinite(q) && fabs(q - j) <= 0.25 && j >= 0.0 && j <= (double)(N - 1)) return (int)j;
    }
    return -2;
}

template <typename T> __device__ __forceinline__ T type_max();
template <> __device__ __forceinline__ float type_max<float>() { return 3.402823466e+38f; }
template <> __device__ __forceinline__ double type_max<double>() { return 1.7976931348623157e+308; }

// 16-byte global load of raw bits
struct alignas(16) raw16 { uint32_t w[4]; };

__device__ __forceinline__ raw16 ld16(const void* p) { return *reinterpret_cast<const raw16*>(p); }

// splitmix64 output for counter `index` of the stream seeded with `seed`
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t index) {
    uint64_t z = seed + (index + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

}  // namespace vabft
