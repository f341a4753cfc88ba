// Verified GEMM for every type, shape and alignment that the whole-tile kernels do not take or would leave most of the
// chip idle on.  A workgroup owns one small tile of C; its K range is dealt in steps of 128 bytes per row to its
// wavefronts, each of which multiplies the whole tile over its own steps, so that the loop has no barrier.
//
// What bounds it.  Problems with few 256 x 256 tiles are a chain of memory latencies on a few compute units: here a
// 64 x 64 (or smaller) tile with K split over four or eight wavefronts gives many of them, each with one or two steps
// of loads outstanding.  A 64 x 64 step of 16-bit operands takes 16 KiB through the vector L1 (64 B / clk per compute
// unit) and through LDS (128 B / clk, once in and once out) per 32 MFMAs of 16 cycles on each of four SIMDs: large
// 16-bit problems are bound at about half the matrix rate and belong to the LDS-tiled kernels; FP32 and FP64, with four
// and eight times the matrix time per byte, are matrix-bound here at any size (FP32 4096^3: 138 of 157 TFLOP/s, FP64
// 4096^3: 65 of 79).
//
// Where there are tiles enough to fill the chip without it, K is not split: each wavefront multiplies a 64 x 64 (or 32 x
// 64) tile of its own over all of K, four side by side in a workgroup that meets once, to add up the row sums (Shape::OWN).
// With a short K a split tile is all epilogue -- two of four wavefronts without a step, a tree of exchanges in LDS, an
// arrival per 64 columns -- at two workgroups per compute unit.  Checked calls with the A-side pass: FP32 4096 x 4096 x 64
// 83 us, now 40; FP8 8192 x 8192 x 128 190, now 88; FP64 8192 x 8192 x 256 777, now 679.  The wavefront sums K in four
// chains, as four wavefronts do: with one chain (1 - 4 % faster) the error of C against more precision doubled (FP32
// 8192 x 1024 x 1024 5.7e-7, now 2.9e-7).
//
// Where there are few tiles and a long K, several workgroups share the K of a tile (SPLIT): the last to arrive adds their tiles
// up and goes on as if it had computed the sum alone.  FP32 93 x 345 x 5527 51 us, now 15.6 (fused call inside a HIP graph).
//
// Operands pass from global memory through registers into LDS rows of the wavefront's own and back as MFMA fragments.
// Loading fragments straight into registers needs no LDS, but puts 16 rows side by side in a quarter of a wavefront,
// one tag look-up per lane: measured 14 B / clk of L1, 2048^3 BF16 (N x K) 75 us against 42.  With eight lanes per row of
// 128 bytes every load takes whole lines.  The XOR swizzle of the 16-byte chunks keeps the fragment reads free of bank
// conflicts; the chunk a lane fetches is chosen for it, so the LDS writes are linear.
//
// Fragments.  v_mfma_*_16x16xK with the operands swapped (D' = B^T A^T): lane l of a result tile owns C row l % 16.
// A lane's chunk is VK consecutive k of one row (16 bytes; 8 for FP8, widened to FP16: exact), the four 16-lane groups
// hold consecutive chunks; FP32 and FP64 take one MFMA per element of the chunk, so the k that one instruction sees are
// VK apart, which the contraction does not mind as A and B agree on it.  Columns are dealt to the fragments with stride
// NF (column of fragment ni, index i = i * NF + ni): with B stored K x N a lane reads NF = 4 consecutive columns of VK
// LDS rows and has VK k-values of four fragments after a transpose in registers (none for FP32 / FP64), and a lane's
// results are consecutive columns of C.
//
// Loads need no alignment beyond the element's (the hardware takes unaligned global accesses).  Rows and columns past
// the end are clamped and their results dropped; k past the end is zero in both operands.  FP16 1021 x 1531 x 2047,
// nothing aligned: 30 us, against 530 with element-wise guarded loads into 256 x 256 tiles.
//
// Check: the wavefronts' partial tiles are added in LDS as a fixed tree, the injector edits the sum, row sums (and
// weighted and column sums) are taken from it before it is rounded to the output type, and the last workgroup of a
// tile-row to arrive folds the tile-columns' partials and compares (section 2.2, Eq. abft-check).  With the A-side
// pass fused, the first (or last) workgroups of the launch run it (row_threshold.h), a wavefront or a part of one per row, and count as
// arrivals of their tile-row: one launch instead of three (pass over A, GEMM, compare).
#pragma once
#include "gemm_common.h"
#include "row_threshold.h"

namespace vabft {
namespace gd {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) __fp16 fp16x2_t;

// ES: bytes of an element; VK: k-values of a lane's chunk; CB: bytes of that chunk in memory; KU: chunks per step
// (a row's share of a step is 128 contiguous bytes); NJ: matrix instructions per chunk
template <typename T> struct Traits;
template <> struct Traits<bf16_t> {
    static constexpr int ES = 2, VK = 8, CB = 16, KU = 2, NJ = 1;
    using accv_t = f32x4_t;
    using out_t = uint16_t;
};
template <> struct Traits<f16_t> {
    static constexpr int ES = 2, VK = 8, CB = 16, KU = 2, NJ = 1;
    using accv_t = f32x4_t;
    using out_t = uint16_t;
};
template <> struct Traits<f8_t> {
    static constexpr int ES = 1, VK = 8, CB = 8, KU = 4, NJ = 1;
    using accv_t = f32x4_t;
    using out_t = uint16_t;
};
template <> struct Traits<bf8_t> {
    static constexpr int ES = 1, VK = 8, CB = 8, KU = 4, NJ = 1;
    using accv_t = f32x4_t;
    using out_t = uint16_t;
};
template <> struct Traits<float> {
    static constexpr int ES = 4, VK = 4, CB = 16, KU = 2, NJ = 4;
    using accv_t = f32x4_t;
    using out_t = float;
};
template <> struct Traits<double> {
    static constexpr int ES = 8, VK = 2, CB = 16, KU = 2, NJ = 2;
    using accv_t = f64x4_t;
    using out_t = double;
};

// 16 bytes at an address in global memory, aligned to the element
typedef const __attribute__((address_space(1))) char* gptr_t;
template <int ES> __device__ __forceinline__ u32x4_t load16g(gptr_t p) {
    typedef uint32_t e_t __attribute__((ext_vector_type(4), aligned(1)));
    typedef uint32_t h_t __attribute__((ext_vector_type(4), aligned(2)));
    typedef uint32_t w_t __attribute__((ext_vector_type(4), aligned(4)));
    if constexpr (ES == 1)
        return *reinterpret_cast<const __attribute__((address_space(1))) e_t*>(p);
    else if constexpr (ES == 2)
        return *reinterpret_cast<const __attribute__((address_space(1))) h_t*>(p);
    else
        return *reinterpret_cast<const __attribute__((address_space(1))) w_t*>(p);
}
// elements 0 .. n-1 of 16 bytes, the rest zero
template <int ES> __device__ u32x4_t load_elems(gptr_t p, int n) {
    u32x4_t o = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 16 / ES; ++e)
        if (e < n) {
            if constexpr (ES == 1)
                o[e / 4] |= (uint32_t) reinterpret_cast<const __attribute__((address_space(1))) uint8_t*>(p)[e] << (8 * (e & 3));
            else if constexpr (ES == 2)
                o[e / 2] |= (uint32_t) reinterpret_cast<const __attribute__((address_space(1))) uint16_t*>(p)[e] << (16 * (e & 1));
            else
#pragma unroll
                for (int q = 0; q < ES / 4; ++q)
                    o[e * (ES / 4) + q] = reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(p)[e * (ES / 4) + q];
        }
    return o;
}

// 16 bytes shifted down by s elements, zero behind
template <int ES> __device__ __forceinline__ u32x4_t shift_elems(u32x4_t v, int s) {
    const int ds = s * ES >> 2;
    uint32_t y[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        uint32_t x = 0u;
#pragma unroll
        for (int f = i; f < 4; ++f) x = ds == f - i ? v[f] : x;
        y[i] = x;
    }
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = ES >= 4 ? y[i] : __builtin_amdgcn_alignbit(y[i + 1], y[i], (uint32_t)(s * ES & 3) * 8);
    return o;
}

// chunk as loaded (CB bytes) -> MFMA fragment (16 bytes)
template <typename T> __device__ __forceinline__ raw16 to_frag(const uint32_t* w) {
    if constexpr (Traits<T>::ES == 1)
        return raw16{{widen2<T>(w[0], false), widen2<T>(w[0], true), widen2<T>(w[1], false), widen2<T>(w[1], true)}};
    else
        return raw16{{w[0], w[1], w[2], w[3]}};
}
// VK rows of four columns, CD dwords each -> fragment of column ni
template <typename T, int CD> __device__ __forceinline__ raw16 to_frag_t(const uint32_t (*w)[CD], int ni) {
    raw16 o;
    if constexpr (Traits<T>::ES == 8) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            o.w[2 * j] = w[j][2 * ni];
            o.w[2 * j + 1] = w[j][2 * ni + 1];
        }
    } else if constexpr (Traits<T>::ES == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) o.w[j] = w[j][ni];
    } else if constexpr (Traits<T>::ES == 2) {
        const uint32_t sel = (ni & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
        for (int d = 0; d < 4; ++d) o.w[d] = __builtin_amdgcn_perm(w[2 * d + 1][ni >> 1], w[2 * d][ni >> 1], sel);
    } else {
        uint32_t c[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            // byte ni of rows 4d .. 4d+3
            const uint32_t sel = 0x0c0c0000u | (uint32_t)(4 + ni) << 8 | (uint32_t)ni;
            const uint32_t lo = __builtin_amdgcn_perm(w[4 * d + 1][0], w[4 * d][0], sel);
            const uint32_t hi = __builtin_amdgcn_perm(w[4 * d + 3][0], w[4 * d + 2][0], sel);
            c[d] = lo | (hi << 16);
        }
        o = to_frag<T>(c);
    }
    return o;
}

// instruction j of the NJ that multiply a chunk
template <typename T>
__device__ __forceinline__ typename Traits<T>::accv_t mfma(const raw16& b, const raw16& a, int j,
                                                           typename Traits<T>::accv_t c) {
    if constexpr (std::is_same<T, bf16_t>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b), __builtin_bit_cast(bf16x8_t, a),
                                                       c, 0, 0, 0);
    else if constexpr (Traits<T>::ES <= 2)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, b), __builtin_bit_cast(f16x8_t, a), c,
                                                      0, 0, 0);
    else if constexpr (std::is_same<T, float>::value)
        return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(b.w[j]), __uint_as_float(a.w[j]), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f64_16x16x4f64(__hiloint2double((int)b.w[2 * j + 1], (int)b.w[2 * j]),
                                                    __hiloint2double((int)a.w[2 * j + 1], (int)a.w[2 * j]), c, 0, 0, 0);
}

// four consecutive accumulator values -> stored elements at p (aligned to the element only); STREAM: past the caches
template <bool STREAM, typename V> __device__ __forceinline__ void put(V* p, V x) {
    if constexpr (STREAM)
        __builtin_nontemporal_store(x, p);
    else
        *p = x;
}
template <typename T, bool STREAM, typename acc_t> __device__ __forceinline__ void store4(void* p, const acc_t* v) {
    if constexpr (std::is_same<T, double>::value || std::is_same<T, float>::value) {
        typedef acc_t v_t __attribute__((ext_vector_type(16 / sizeof(acc_t)), aligned(sizeof(acc_t))));
#pragma unroll
        for (int q = 0; q < (int)sizeof(acc_t) / 4; ++q) {
            v_t x;
#pragma unroll
            for (int e = 0; e < 16 / (int)sizeof(acc_t); ++e) x[e] = v[q * (16 / (int)sizeof(acc_t)) + e];
            put<STREAM>(reinterpret_cast<v_t*>(p) + q, x);
        }
    } else {
        using h2 = typename std::conditional<std::is_same<T, bf16_t>::value, bf16x2_t, f16x2_t>::type;
        typedef uint32_t v_t __attribute__((ext_vector_type(2), aligned(2)));
        v_t x;
        x[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{v[0], v[1]}), h2));
        x[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{v[2], v[3]}), h2));
        put<STREAM>(reinterpret_cast<v_t*>(p), x);
    }
}
// 8 bytes of stored elements from as many accumulator values
template <typename T, typename acc_t> __device__ __forceinline__ uint64_t word8(const acc_t* v) {
    uint64_t w;
    if constexpr (std::is_same<T, double>::value || std::is_same<T, float>::value) {
        __builtin_memcpy(&w, v, 8);
    } else {
        using h2 = typename std::conditional<std::is_same<T, bf16_t>::value, bf16x2_t, f16x2_t>::type;
        const h2 x[2] = {__builtin_convertvector((f32x2_t{v[0], v[1]}), h2), __builtin_convertvector((f32x2_t{v[2], v[3]}), h2)};
        __builtin_memcpy(&w, x, 8);
    }
    return w;
}
template <typename T, typename acc_t> __device__ __forceinline__ typename Traits<T>::out_t to_out(acc_t v) {
    if constexpr (std::is_same<T, double>::value || std::is_same<T, float>::value)
        return v;
    else if constexpr (std::is_same<T, bf16_t>::value)
        return Elem<bf16_t>::from_acc(v);
    else
        return Elem<f16_t>::from_acc(v);
}

// B bytes from an LDS address aligned to them (to 16 at most)
template <int B> __device__ __forceinline__ void copy_bytes(uint32_t* to, const unsigned char* from) {
    __builtin_memcpy(to, __builtin_assume_aligned(from, B < 16 ? B : 16), B);
}
// N consecutive values between LDS and registers, at a place aligned to all of them or to 16 bytes
template <int N, typename acc_t> __device__ __forceinline__ void copy_aligned(acc_t* to, const acc_t* from) {
    constexpr int B = N * (int)sizeof(acc_t), AL = B < 16 ? B : 16;
    __builtin_memcpy(__builtin_assume_aligned(to, AL), __builtin_assume_aligned(from, AL), B);
}

// WVK wavefronts share the K of one tile, or (WVK = 1) WN wavefronts side by side have a tile each
template <typename T, int TRANSB, int MF, int NF, int WVK, int WN> struct Shape {
    using acc_t = typename Elem<T>::acc_t;
    static constexpr int NW = WVK * WN, NT = 64 * NW;
    static constexpr bool OWN = WN > 1;  // a tile per wavefront
    static_assert(WVK == 1 || WN == 1, "one or the other");
    static constexpr int BM = 16 * MF, BNW = 16 * NF, BN = BNW * WN;  // of a wavefront's tile, of the workgroup
    static constexpr int PITCH = BNW + 16 / (int)sizeof(acc_t);  // 16-byte aligned rows, four banks of skew
    static constexpr int SLOTS = WVK > 1 ? 2 : 1;                // partial tiles left after the tree's register rounds
    static constexpr int TILE_BYTES = SLOTS * BM * PITCH * (int)sizeof(acc_t);
    static constexpr int ROUND_BYTES = WVK > 2 ? (WVK / 2) * MF * NF * 64 * 4 * (int)sizeof(acc_t) : 0;
    static constexpr int WAVE_BYTES = (BM + BNW) * 128;  // operand rows of one step of one wavefront
    static constexpr int cmax(int a, int b) { return a > b ? a : b; }
    static constexpr int AREA = cmax(WAVE_BYTES, OWN ? TILE_BYTES : 0);  // LDS of a wavefront
    static constexpr int SUMS = OWN ? NW * AREA : 0;                     // OWN: the wavefronts' row sums, [2][WN][BM]
    static constexpr int LDS =
        (OWN ? SUMS + 2 * WN * BM * (int)sizeof(acc_t) : cmax(cmax(TILE_BYTES, ROUND_BYTES), NW * AREA)) + 128;
    // epilogue: consecutive columns of a thread (a wavefront with a tile of its own stores whole pieces of rows, in
    // passes), threads per row, rows per pass
    static constexpr int ET = OWN ? 64 : NT;
    static constexpr int EPT = OWN ? 4 : BM * BN / NT < 16 ? BM * BN / NT : 16;
    static constexpr int TPR = BNW / EPT, RPP = ET / TPR, PASSES = BM / RPP;
    static_assert(TPR <= 64 && BM % RPP == 0 && BM % NW == 0 && (OWN || PASSES == 1), "epilogue mapping");
};

// K shared by d.split workgroups: each leaves its tile (the sum of the wavefronts') in the workspace, and the last one to
// arrive at the tile's counter adds them up in a fixed order, four sums side by side, puts the result back into LDS and goes
// on with the tile; the others are done (false).
template <typename S> __device__ bool join_split(const DirectArgs& d, int at, int z, typename S::acc_t* tile, int* s_last) {
    using acc_t = typename S::acc_t;
    constexpr int E = S::EPT * (int)sizeof(acc_t) >= 8 ? 8 / (int)sizeof(acc_t) : 1, Q = S::EPT / E;  // of a store; stores
    using word_t = typename std::conditional<E * sizeof(acc_t) == 8, uint64_t, uint32_t>::type;
    const int tid = threadIdx.x;
    acc_t* const mine = tile + tid / S::TPR * S::PITCH + tid % S::TPR * S::EPT;
    word_t* const first = reinterpret_cast<word_t*>(d.g.apart) + (int64_t)at * d.split * Q * S::NT + tid;
    alignas(16) acc_t v[S::EPT];
    copy_aligned<S::EPT>(v, mine);
    if constexpr (S::SLOTS == 2) {
        alignas(16) acc_t u[S::EPT];
        copy_aligned<S::EPT>(u, mine + S::BM * S::PITCH);
#pragma unroll
        for (int e = 0; e < S::EPT; ++e) v[e] += u[e];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        word_t w;
        __builtin_memcpy(&w, v + q * E, sizeof(w));
        __hip_atomic_store(first + (int64_t)(z * Q + q) * S::NT, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's part is performed
    __syncthreads();
    int32_t* const ticket = d.g.tickets + (d.g.tiles_m + 1 + at) * d.g.ticket_stride;  // behind the tile-rows'
    if (tid == 0) *s_last = atomicAdd(ticket, 1) == d.split - 1;
    __syncthreads();
    if (!*s_last) return false;
    if (tid == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    acc_t sum[4][S::EPT] = {};
    for (int z0 = 0; z0 < d.split; z0 += 4) {
        word_t w[4][Q];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < Q; ++q)
                w[j][q] = z0 + j < d.split ? __hip_atomic_load(first + (int64_t)((z0 + j) * Q + q) * S::NT, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)
                                           : (word_t)0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                acc_t x[E];
                __builtin_memcpy(x, &w[j][q], sizeof(x));
#pragma unroll
                for (int e = 0; e < E; ++e) sum[j][q * E + e] += x[e];
            }
    }
#pragma unroll
    for (int e = 0; e < S::EPT; ++e) v[e] = (sum[0][e] + sum[1][e]) + (sum[2][e] + sum[3][e]);
    copy_aligned<S::EPT>(mine, v);
    if constexpr (S::SLOTS == 2) {
        alignas(16) const acc_t zero[S::EPT] = {};
        copy_aligned<S::EPT>(mine + S::BM * S::PITCH, zero);
    }
    __syncthreads();
    return true;
}

// Workgroups of a launch, at most: a launch holds fewer than 2^32 threads in one dimension, and tiles of 32 rows of a tall
// and narrow product may be more.  They go on in a second launch: a second dimension costs every workgroup of every launch
// (BF16 1 x 4096 x 4096 7.0 us, 7.3; with the row's width out of the launch's record 7.6).
constexpr int LAUNCH_MOST = 1 << 22;

}  // namespace gd

// Folds the partial row sums of `rows` rows from row0 on and compares; SUB groups of R neighbouring threads share the
// tile-columns of R rows, so that a wavefront reads whole pieces of lines: loads for other workgroups' partials pass the
// caches by, one request per piece.  Against SUB neighbouring threads per row: 16 x 4096 x 4096 14.4 -> 11.7 us, 1024^3
// 12.6 -> 12.0.  This code runs once, at the end, in one workgroup: every instruction of it is time of the launch (1.3 ns, a taken
// branch more), so it has no branch per load, a batch of loads of about the size that there are partials for, all in flight at
// once, and one barrier for the fold.  With 16 guarded loads to a batch and a barrier per halving (fused calls in a graph):
// FP32 256^3 8.3 -> 7.8 us, BF16 1024^3 10.9 -> 10.0, 7 x 1792 x 512 7.2 -> 6.3, 24 x 11008 x 4096 (172 partials to a row)
// 20.3 -> 18.7.  Returns the number of flagged rows to the first wavefront.
// W: weighted sums too; with d.wsum == 2 flagged rows are localised and corrected here (locate_row), and corrected receives how
// many.
template <typename T, bool W, int R, int SUB>
__device__ __forceinline__ int direct_compare(const DirectArgs& d, int row0, int rows, unsigned char* smem, int& corrected) {
    using acc_t = typename Elem<T>::acc_t;
    const GemmArgs& g = d.g;
    const int r = threadIdx.x % R, sub = threadIdx.x / R;
    const bool act = r < rows;
    const int gi = row0 + (act ? r : 0);
    // (with the partials in flight, not a round trip behind their fold)
    const acc_t want = ld_agent(reinterpret_cast<const acc_t*>(g.expected) + gi);
    const acc_t t = ld_agent(reinterpret_cast<const acc_t*>(g.T) + gi);
    const int64_t step = (int64_t)SUB * g.M;
    int64_t at = (int64_t)sub * g.M;  // of this thread's next partial, from its row's first
    acc_t s4[4] = {0, 0, 0, 0}, w4[4] = {0, 0, 0, 0};
    const auto batch = [&](auto u_c, int t0) __attribute__((always_inline)) {
        constexpr int U = decltype(u_c)::value;
        int left = g.tiles_n - t0 - sub;  // (opaque, so that no other batch's conditions are worked out in front of this one)
        asm volatile("" : "+v"(left));
        const auto load = [&](const void* partials, acc_t* v) __attribute__((always_inline)) {
            const acc_t* const row = reinterpret_cast<const acc_t*>(partials) + gi;
            int64_t a = at;
#pragma unroll
            for (int j = 0; j < U; ++j, a += step) v[j] = ld_agent(row + (j * SUB < left ? a : 0));
        };
        acc_t v[U], v2[U];
        load(g.rowpart, v);
        if constexpr (W) {
            load(g.rowpart2, v2);
#pragma unroll
            for (int j = 0; j < U; ++j) w4[j & 3] += j * SUB < left ? v2[j] : (acc_t)0;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) s4[j & 3] += j * SUB < left ? v[j] : (acc_t)0;
        at += U * step;
    };
    // (as many as leave the kernel the registers that the product takes, and with them its wavefronts per SIMD: FP64 2048^3 with
    // 24 281 us, with 8 272)
    constexpr int MOST = sizeof(acc_t) == 8 || R * SUB > 256 ? 8 : R == 32 ? 24 : 16;
    if (g.tiles_n <= 2 * SUB)
        batch(std::integral_constant<int, 2>(), 0);
    else if (MOST > 8 && g.tiles_n <= 8 * SUB)
        batch(std::integral_constant<int, 8>(), 0);
    else
        for (int t0 = 0; t0 < g.tiles_n; t0 += MOST * SUB) batch(std::integral_constant<int, MOST>(), t0);
    acc_t s = (s4[0] + s4[1]) + (s4[2] + s4[3]), s2 = (w4[0] + w4[1]) + (w4[2] + w4[3]);
    if constexpr (SUB > 1) {
        // the groups of a wavefront, then the wavefronts (a power of two of them)
        constexpr int NW = R * SUB / 64;
        static_assert(R <= 64 && R >= 16, "");
        const auto in_wave = [](acc_t q) {
            acc_t a, b;
            if constexpr (R <= 32) {
                lane_exchange<32, WAVE>(q, a, b);
                q = a + b;
            }
            if constexpr (R <= 16) {
                lane_exchange<16, WAVE>(q, a, b);
                q = a + b;
            }
            return q;
        };
        acc_t* const red = reinterpret_cast<acc_t*>(smem);  // [2][NW][R]
        const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
        s = in_wave(s);
        if constexpr (W) s2 = in_wave(s2);
        if (wave > 0 && lane < R) {
            red[wave * R + lane] = s;
            if constexpr (W) red[(NW + wave) * R + lane] = s2;
        }
        __syncthreads();
        if (wave == 0) {
            const auto over_waves = [&](acc_t q, const acc_t* from) {
                acc_t x[NW];
                x[0] = q;
#pragma unroll
                for (int w = 1; w < NW; ++w) x[w] = from[w * R + r];
#pragma unroll
                for (int h = 1; h < NW; h *= 2)
#pragma unroll
                    for (int w = 0; w + h < NW; w += 2 * h) x[w] += x[w + h];
                return x[0];
            };
            s = over_waves(s, red);
            if constexpr (W) s2 = over_waves(s2, red + NW * R);
        }
    }
    int f = 0, fixed = 0;
    if (act && sub == 0) {
        const acc_t e = want - s;
        f = !(fabs(e) <= t);
        reinterpret_cast<acc_t*>(g.rowsum)[gi] = s;
        if constexpr (W) reinterpret_cast<acc_t*>(g.rowsum2)[gi] = s2;
        reinterpret_cast<acc_t*>(g.E)[gi] = e;
        g.flags[gi] = f;
        if constexpr (W) {
            if (d.wsum == 2) {
                int column = -1;
                acc_t by = 0;
                if (f) {
                    const acc_t want2 = ld_agent(reinterpret_cast<const acc_t*>(g.w.expected2) + gi);
                    column = locate_row<acc_t>(want, want2, s, s2, g.N, by);
                    if (g.w.correct && column >= 0) {
                        // (all of the row is in memory: its tiles were stored past the caches, before they arrived)
                        using C = CElem<T>;
                        auto* const c = reinterpret_cast<typename C::store_t*>(g.C) + (int64_t)gi * g.ldc + column;
                        C::put_agent(c, C::get_agent(c) - by);
                        fixed = 1;
                    }
                }
                g.w.loc[gi] = column;
                reinterpret_cast<acc_t*>(g.w.delta)[gi] = by;
            }
        }
    }
    if constexpr (W) corrected = SUB > 1 ? (int)__popcll(__ballot(fixed)) : __syncthreads_count(fixed);
    return SUB > 1 ? (int)__popcll(__ballot(f)) : __syncthreads_count(f);
}

// The last workgroup of tile-row bm to arrive (GEMM tiles and, with the A-side pass fused, its workgroups) compares the
// tile-row.  Where there are few tile-columns, tile-rows share a counter and a compare, as many as have the rows that a
// workgroup has threads: finished compares add to one word for the whole launch, 11 ns each (FP32 8192 x 64 x 64 10.1 -> 7.2
// us, 100000 x 64 x 64 49 -> 32).  If one counter serves all rows, who completes it knows nflag, one round trip to memory less.
// Every thread of every workgroup calls this after its partials are written.  store_c
// comes behind the arrival (in front of it, the wait for the partials would be one for the stores of C as well) and, in the
// workgroup that compares, behind that.
template <typename T, typename S, bool W, typename F>
__device__ __forceinline__ void direct_tile_row_check(const DirectArgs& d, int bm, int* s_last, unsigned char* smem, F store_c) {
    const GemmArgs& g = d.g;
    constexpr int SHARE = S::NT / S::BM;  // tile-rows of a shared counter
    const bool shared = g.tiles_n <= 4 || (g.tiles_m * g.tiles_n <= 64 && g.M <= S::NT);
    static_assert((SHARE & (SHARE - 1)) == 0, "");
    const int tile_rows = shared ? SHARE : 1, at = shared ? bm / SHARE : bm, row0 = at * tile_rows * S::BM;
    const int counters = shared ? (g.tiles_m + SHARE - 1) / SHARE : g.tiles_m, rows = min(tile_rows * S::BM, g.M - row0);
    // (a workgroup of the A-side pass has a power of two of rows)
    const int arrivals = (rows + S::BM - 1) / S::BM * g.tiles_n +
                         (d.stat_blocks ? (rows + d.stat_rows - 1) >> __builtin_ctz((unsigned)d.stat_rows) : 0);
    __builtin_amdgcn_s_waitcnt(0);  // this wavefront's partials are performed
    __syncthreads();
    int before = 0;
    if (threadIdx.x == 0 && arrivals > 1) before = atomicAdd(&g.tickets[at * g.ticket_stride], 1);
    // (workgroups that come by the thousand store C while the arrival is on its way; where there are few, the compare is
    // what the launch ends with and does not wait for the stores)
    const bool stored = W && d.wsum == 2;  // C is in memory already
    if constexpr (S::OWN) store_c();
    if (threadIdx.x == 0) *s_last = before == arrivals - 1;
    __syncthreads();
    if (!*s_last) {
        if constexpr (!S::OWN)
            if (!stored) store_c();
        return;
    }
    int fixed = 0;
    const int cnt = rows > S::BM ? direct_compare<T, W, S::NT, 1>(d, row0, rows, smem, fixed)
                                 : direct_compare<T, W, S::BM, SHARE>(d, row0, rows, smem, fixed);
    if (threadIdx.x == 0) {
        if (arrivals > 1) __hip_atomic_store(&g.tickets[at * g.ticket_stride], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (counters == 1) {
            *g.d_nflag = cnt;
            if (stored) *g.w.ncorrected = fixed;
        } else if (stored) {
            // finished compares, corrected rows and flagged rows in one word (of 2^20 rows at most)
            unsigned long long* done = done_counter(g);
            const unsigned long long old = atomicAdd(done, (1ull << 42) | (unsigned long long)fixed << 21 | (unsigned long long)cnt);
            if ((int)(old >> 42) == counters - 1) {
                *g.d_nflag = (int)(old & 0x1fffff) + cnt;
                *g.w.ncorrected = (int)(old >> 21 & 0x1fffff) + fixed;
                __hip_atomic_store(done, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            // one 64-bit atomic counts the finished compares (high word) and the flagged rows (low word); whoever
            // completes the count publishes nflag and leaves the counter zero
            unsigned long long* done = done_counter(g);
            const unsigned long long old = atomicAdd(done, (1ull << 32) | (unsigned long long)(unsigned)cnt);
            if ((int)(old >> 32) == counters - 1) {
                *g.d_nflag = (int)(unsigned)(old & 0xffffffffull) + cnt;
                __hip_atomic_store(done, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if constexpr (!S::OWN)
        if (!stored) store_c();
}

// The A-side pass inside the GEMM launch: d.stat_rows rows per workgroup, a wavefront or (short rows) 32 or 16 lanes of one
// per row
template <typename T, typename S, bool W, int LW, int NL>
__device__ __forceinline__ void direct_stats_rows(const DirectArgs& d, int block, double S1, double S2, double S3) {
    using acc_t = typename Elem<T>::acc_t;
    const GemmArgs& g = d.g;
    const int lane = threadIdx.x % LW, m = block * d.stat_rows + threadIdx.x / LW;
    // (lanes behind the last row read it again: the exchanges need every lane)
    const char* row = reinterpret_cast<const char*>(g.A) + (int64_t)min(m, g.M - 1) * g.lda * Elem<T>::bytes;
    const RowSums<acc_t> r = row_sums<T, W, NL, LW>(row, g.K, lane, reinterpret_cast<const acc_t*>(g.Be),
                                                    W ? reinterpret_cast<const acc_t*>(g.w.Be2) : nullptr);
    if (lane == 0 && m < g.M) {
        double mu;
        const acc_t t = (acc_t)row_threshold(r, g.K, g.N, S1, S2, S3, g.e_max, g.c_sigma, mu);
        acc_t* astat = reinterpret_cast<acc_t*>(g.astat) + 3 * (int64_t)m;
        astat[0] = r.mx;
        astat[1] = r.mn;
        astat[2] = (acc_t)mu;
        st_agent(reinterpret_cast<acc_t*>(const_cast<void*>(g.expected)) + m, r.dot);
        st_agent(reinterpret_cast<acc_t*>(const_cast<void*>(g.T)) + m, t);
        if constexpr (W) st_agent(reinterpret_cast<acc_t*>(g.w.expected2) + m, r.dot2);
    }
}
template <typename T, typename S, bool W>
__device__ __forceinline__ void direct_stats(const DirectArgs& d, int block, double* s_red, int* s_last, unsigned char* smem) {
    const GemmArgs& g = d.g;
    const bool fold = g.s_nparts != 0;
    if (fold) {
        fold_s_partials_to_lds(g.s_partial, g.s_nparts, threadIdx.x, s_red);
        __syncthreads();
        if (block == 0 && threadIdx.x < 3 && g.S) g.S[threadIdx.x] = folded_s(s_red, threadIdx.x);
    }
    // (ahead of the row: not one more round trip behind it)
    const double S1 = fold ? folded_s(s_red, 0) : g.S[0], S2 = fold ? folded_s(s_red, 1) : g.S[1],
                 S3 = fold ? folded_s(s_red, 2) : g.S[2];
    if (d.stat_rows == S::NW)
        direct_stats_rows<T, S, W, 64, 4>(d, block, S1, S2, S3);
    else if (d.stat_rows == 2 * S::NW)
        direct_stats_rows<T, S, W, 32, 1>(d, block, S1, S2, S3);
    else
        direct_stats_rows<T, S, W, 16, 1>(d, block, S1, S2, S3);
    direct_tile_row_check<T, S, W>(d, block * d.stat_rows / S::BM, s_last, smem, [] {});
}

// ANY: for rows so far apart that 32 bits do not hold a tile's byte offsets, and for rows of under 16 bytes.
// D: steps in flight from global memory.
// SPLIT: d.split workgroups share the K of a tile (kernels of their own: the code in the others, skipped, cost short calls 3 %).
// W: position-weighted row sums too (d.wsum; kernels of their own for the same reason).
// Wavefronts to a SIMD that the compiler has to leave registers for: a few registers more would be a workgroup less on the compute
// unit.
template <typename T, int TRANSB, int MF, int WVK, bool ANY, bool SPLIT> constexpr int direct_min_waves() {
    if (WVK == 8 && TRANSB && MF == 1) return 4;  // (B stored K x N: LDS for one workgroup)
    if (WVK == 4 && MF == 2 && !ANY) return 3;  // (BF16 1024 x 1024 x 512 with two 10.0 us, with three 7.8)
    return 2;
}
template <typename T, int TRANSB, int MF, int NF, int WVK, int WN, int D, bool ANY, bool SPLIT, bool W>
__global__ __launch_bounds__(64 * WVK * WN, (direct_min_waves<T, TRANSB, MF, WVK, ANY, SPLIT>())) void gemm_direct_kernel(const DirectArgs d) {
    using S = gd::Shape<T, TRANSB, MF, NF, WVK, WN>;
    using OFF = typename std::conditional<ANY, uint64_t, uint32_t>::type;
    using Tr = gd::Traits<T>;
    using acc_t = typename Elem<T>::acc_t;
    using accv_t = typename Tr::accv_t;
    constexpr int ES = Tr::ES, VK = Tr::VK, CB = Tr::CB, KU = Tr::KU;
    constexpr int KC = 4 * VK, KSTEP = KC * KU;  // k of one chunk over the four lane groups, k of one step
    constexpr int CD = 4 * ES / 4;               // dwords of four columns (B stored K x N)
    constexpr int LA = 2 * MF, LB = 2 * NF;  // 1 KiB loads of a step
    constexpr int RB = S::BNW * ES, V = 16 / ES;    // K x N B: bytes of a row of the tile; elements of a lane's 16 bytes
    static_assert(KSTEP * ES == 128, "a row's share of a step is 128 bytes");
    static_assert(TRANSB || NF == 4, "a lane reads four columns of B stored K x N");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int* const s_last = reinterpret_cast<int*>(smem + S::LDS - 128);
    double* const s_red = reinterpret_cast<double*>(smem + S::LDS - 112);
    const GemmArgs& g = d.g;
    const bool verify = d.verify != 0;
    const int tid = threadIdx.x;
    const int block = d.first_block + ((int)blockIdx.x ^ d.mirror);  // the A-side pass's, then the tiles'
    if (verify && block == 0 && tid == 0) {
        if (g.block_mode) {  // a compare kernel that follows counts into these
            *g.d_nflag = 0;
            *g.d_nblockflag = 0;
        }
        if (g.d_ncolflag) *g.d_ncolflag = 0;
    }
    static_assert(!SPLIT || (!S::OWN && !ANY), "");
    if (block < d.stat_blocks) {
        direct_stats<T, S, W>(d, block, s_red, s_last, smem);
        return;
    }
    const int nth = block - d.stat_blocks;
    const int lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wk = S::OWN ? 0 : wave, wn = S::OWN ? wave : 0;
    // Workgroup z of the d.split that share the K of a tile, and the whole steps [s0, s0 + full) it takes of all of them
    const int tiles = g.tiles_m * g.tiles_n, split = SPLIT ? d.split : 1, z = SPLIT ? nth / tiles : 0;
    int bm, bn;
    tile_of_block(nth - z * tiles, g.tiles_m, g.tiles_n, bm, bn);
    const int steps = g.K / KSTEP, s0 = SPLIT ? (int)((int64_t)steps * z / split) : 0;
    const int full = (SPLIT ? (int)((int64_t)steps * (z + 1) / split) : steps) - s0;
    const int rest = z == split - 1 ? g.K - steps * KSTEP : 0;  // k behind the last whole step
    const int row0 = bm * S::BM, col0 = bn * S::BN + wn * S::BNW;

    // Rows of under 16 bytes (ANY) are read element by element, already finished (load_part)
    const bool tiny = ANY && (g.K < V || (!TRANSB && g.N < V));
    // Steps are dealt to the wavefronts in turn.  The k behind the last whole step are the end of a step that ends where K
    // does: read like any other (all of it is inside the rows), first of its wavefront's, and the k before them cleared in both
    // operands (clear_front).  With loads of its own for it, clamped and shifted, and the step's code a second time, its 500
    // instructions ran with nothing in flight but the next step (fused calls, so / now): FP16 500 x 999 x 777 10.4 / 9.3 us,
    // BF16 530 x 3584 x 283 (N x K) 16.2 / 14.0, FP32 1000 x 1200 x 1500 45.5 / 42.8, FP64 1777 x 1061 x 331 (N x K) 43.9 / 38.6;
    // whole steps only, 256^3 in FP32 7.55 / 7.68, of 336 problems 4 more than 3 % slower; plain products 0.09 us (1.3 %) slower with
    // 32 x 64 tiles, up to 4 % with a FP64 B stored N x K, whose products the compiler puts in another order.
    const int whole = !tiny && full > wk ? (full - wk + WVK - 1) / WVK : 0;  // steps of this wavefront
    const bool ends_here = rest > 0 && full % WVK == wk && g.K >= KSTEP;
    // (64 rows: as a value that the compiler does not see through, or it keeps addresses for both cases and spills them)
    const int tail = MF >= 4 ? __builtin_amdgcn_readfirstlane((int)ends_here) : (int)ends_here;
    // k that the loads count from, this wavefront's first whole step.  Where it has none, its only step, which is read again behind
    // itself: known late, so that the first loads do not wait for it, but with 64 rows, where a second base would be spilled.
    const int kfirst = MF >= 4 && whole == 0 && g.K >= KSTEP ? g.K - KSTEP : (s0 + wk) * KSTEP;

    // ---- global memory -> registers ---------------------------------------------------------------------------
    // Row loads: load t covers LDS rows 8 t .. 8 t + 7, eight lanes each; the lane at position lane % 8 of row r
    // fetches chunk (lane % 8) ^ ((r >> 1) & 7), so that the 16 rows of a fragment read hit 16 distinct slots.
    const int lrow = lane >> 3;
    const char* abase = reinterpret_cast<const char*>(g.A) + ((int64_t)row0 * g.lda + kfirst) * ES;
    OFF aoff[LA];
#pragma unroll
    for (int t = 0; t < LA; ++t) {
        const int r = min(row0 + 8 * t + lrow, g.M - 1) - row0;
        aoff[t] = (OFF)r * (OFF)(g.lda * ES) + (OFF)(((lane & 7) ^ ((4 * t + (lane >> 4)) & 7)) << 4);
    }
    const char* bbase;
    OFF boff[LB];
    if constexpr (TRANSB != 0) {
        bbase = reinterpret_cast<const char*>(g.B) + ((int64_t)col0 * g.ldb + kfirst) * ES;
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            // LDS row ni * 16 + i holds column i * NF + ni of the tile
            const int q = 8 * t + lrow, r = min(col0 + (q & 15) * NF + (q >> 4), g.N - 1) - col0;
            boff[t] = (OFF)r * (OFF)(g.ldb * ES) + (OFF)(((lane & 7) ^ ((4 * t + (lane >> 4)) & 7)) << 4);
        }
    } else {
        // LDS row k of RB bytes: the tile's columns of row k of the step, in groups of V; a group that would cross the
        // row's end starts at N - V instead (see column_of)
        const int c = max(0, min(col0 + lane * 16 % RB / ES, g.N - V));
        bbase = reinterpret_cast<const char*>(g.B) + ((int64_t)kfirst * g.ldb) * ES;
#pragma unroll
        for (int t = 0; t < LB; ++t) boff[t] = (OFF)((t * 1024 + lane * 16) / RB) * (OFF)(g.ldb * ES) + (OFF)c * ES;
    }
    const int64_t bstep = TRANSB ? ES : g.ldb * ES;    // bytes of one k
    struct Stage {
        gd::u32x4_t a[LA], b[LB];
    };
    // k0: of the step, from kfirst
    auto load_at = [&](int64_t k0, Stage& st) __attribute__((always_inline)) {
        // (base and offsets opaque, so that each load is scalar base + 32-bit lane offset and no sum of the two, nor
        // the offset widened to 64 bits, is kept across the loop)
        gd::gptr_t pa = (gd::gptr_t)(abase + k0 * ES);
        gd::gptr_t pb = (gd::gptr_t)(bbase + k0 * bstep);
        asm volatile("" : "+s"(pa), "+s"(pb));
#pragma unroll
        for (int t = 0; t < LA; ++t) asm volatile("" : "+v"(aoff[t]));
#pragma unroll
        for (int t = 0; t < LB; ++t) asm volatile("" : "+v"(boff[t]));
#pragma unroll
        for (int t = 0; t < LA; ++t) st.a[t] = gd::load16g<ES>(pa + aoff[t]);
#pragma unroll
        for (int t = 0; t < LB; ++t) st.b[t] = gd::load16g<ES>(pb + boff[t]);
    };
    // i: this wavefront's step number
    auto load_step = [&](int i, Stage& st) __attribute__((always_inline)) { load_at((int64_t)i * (WVK * KSTEP), st); };
    auto clear_front = [&](Stage& st) __attribute__((always_inline)) {
        const int before = KSTEP - rest;
        uint32_t keep[2][4];  // (of a lane's chunks in even and odd loads)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int bytes = (before - (((lane & 7) ^ ((4 * t + (lane >> 4)) & 7)) << 4) / ES) * ES;  // of the chunk to clear
#pragma unroll
            for (int q = 0; q < 4; ++q) keep[t][q] = bytes >= 4 * q + 4 ? 0u : ~0u << (8 * max(0, bytes - 4 * q) & 31);
        }
#pragma unroll
        for (int t = 0; t < LA; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) st.a[t][q] &= keep[t & 1][q];
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            const uint32_t row = (t * 1024 + lane * 16) / RB < before ? 0u : ~0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) st.b[t][q] &= TRANSB ? keep[t & 1][q] : row;
        }
    };
    // Step i where only the first len < KSTEP k are inside K (of a K of less than a step): rows along k are read where they still
    // have 16 bytes and shifted by finish_part, rows along n past K are replaced by the last one and cleared by finish_part.
    auto beyond = [&](int t, int len) { return (((lane & 7) ^ ((4 * t + (lane >> 4)) & 7)) << 4) / ES + V - len; };
    auto load_part = [&](int i, int len, Stage& st) __attribute__((always_inline)) {
        const int64_t k0 = (int64_t)i * (WVK * KSTEP);
        const gd::gptr_t pa = (gd::gptr_t)(abase + k0 * ES), pb = (gd::gptr_t)(bbase + k0 * bstep);
        if (!tiny) {
#pragma unroll
            for (int t = 0; t < LA; ++t) st.a[t] = gd::load16g<ES>(pa + aoff[t] - (int64_t)max(0, beyond(t, len)) * ES);
#pragma unroll
            for (int t = 0; t < LB; ++t) {
                const int64_t back = TRANSB ? (int64_t)max(0, beyond(t, len)) * ES
                                            : (int64_t)max(0, (t * 1024 + lane * 16) / RB - (len - 1)) * bstep;
                st.b[t] = gd::load16g<ES>(pb + boff[t] - back);
            }
        } else if constexpr (ANY) {
            for (int t = 0; t < LA; ++t) st.a[t] = gd::load_elems<ES>(pa + aoff[t], V - beyond(t, len));
            for (int t = 0; t < LB; ++t) {
                const int k = (t * 1024 + lane * 16) / RB;
                // (K x N: counted from where the load starts, which for a group that would cross the row's end is N - V)
                const int n = TRANSB ? V - beyond(t, len) : k < len ? g.N - max(0, min(col0 + lane * 16 % RB / ES, g.N - V)) : 0;
                st.b[t] = gd::load_elems<ES>(pb + boff[t], n);
            }
        }
    };
    auto finish_part = [&](int len, Stage& st) __attribute__((always_inline)) {
        if (tiny) return;
#pragma unroll
        for (int t = 0; t < LA; ++t) st.a[t] = gd::shift_elems<ES>(st.a[t], min(V, max(0, beyond(t, len))));
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            if constexpr (TRANSB != 0)
                st.b[t] = gd::shift_elems<ES>(st.b[t], min(V, max(0, beyond(t, len))));
            else if ((t * 1024 + lane * 16) / RB >= len)
                st.b[t] = gd::u32x4_t{0u, 0u, 0u, 0u};
        }
    };

    accv_t acc[MF][NF];
    const auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MF; ++mi)
#pragma unroll
            for (int ni = 0; ni < NF; ++ni)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0;
    };
    // ---- registers -> the wavefront's own LDS rows -> fragments -> MFMA ----------------------------------------
    // No other wavefront reads these rows and LDS operations of one wavefront complete in order, so one buffer and
    // no barrier will do.
    unsigned char* const stage = smem + wave * S::AREA;
    const unsigned char* const frag0 = stage + l16 * 128;
    const int swz = (l16 >> 1) & 7;
    // multiplies the step in st; reload() runs as soon as its registers are free
    auto compute = [&](Stage& st, auto reload) __attribute__((always_inline)) {
        // (FP64, a tile per wavefront: the step begins 4 bytes behind a multiple of 8, whatever the code in front of it.  The same
        // instructions 4 bytes further on took 768 x 5519 x 67 36.8 us plain, here 29.2, 4000 x 4000 x 64 62 / 55, 1987 x 8097 x 139
        // 121 / 116 checked; in the other types and forms it is within 1 % either way)
        if constexpr (S::OWN && sizeof(acc_t) == 8) asm volatile(".p2align 3\n\ts_nop 0");
#pragma unroll
        for (int t = 0; t < LA; ++t) *reinterpret_cast<gd::u32x4_t*>(stage + t * 1024 + lane * 16) = st.a[t];
#pragma unroll
        for (int t = 0; t < LB; ++t) *reinterpret_cast<gd::u32x4_t*>(stage + (LA + t) * 1024 + lane * 16) = st.b[t];
        __builtin_amdgcn_sched_barrier(0);
        reload();
        __builtin_amdgcn_sched_barrier(0);
        // 16-bit, B stored K x N, K shared by the wavefronts: the second chunk's fragments are on their way while the first's are
        // multiplied.  (Left to the compiler it comes out so or not: if not, BF16 and FP16 4 x 768 x 5376 9.8 us, not 8.5.)
        constexpr bool AHEAD = TRANSB == 0 && ES == 2 && !S::OWN;
        constexpr int HELD = AHEAD ? KU : 1;
        raw16 af[HELD][MF], bf[NF];
        uint32_t w[HELD][VK][CD];
        const auto frag = [&](int f, int u) __attribute__((always_inline)) {
            // the lane's chunk: 16-byte slot and, for 8-byte chunks, its half
            const int at = CB == 16 ? ((4 * u + lq) ^ swz) << 4 : (((2 * u + (lq >> 1)) ^ swz) << 4) + 8 * (lq & 1);
            uint32_t c[Tr::CB / 4];
            gd::copy_bytes<Tr::CB>(c, frag0 + f * 2048 + at);
            return gd::to_frag<T>(c);
        };
        const auto fetch_b = [&](int u) __attribute__((always_inline)) {
            if constexpr (TRANSB != 0) {
#pragma unroll
                for (int ni = 0; ni < NF; ++ni) bf[ni] = frag(MF + ni, u);
            } else {
#pragma unroll
                for (int e = 0; e < VK; ++e)
                    gd::copy_bytes<4 * CD>(w[u % HELD][e], stage + LA * 1024 + (u * KC + lq * VK + e) * RB + l16 * NF * ES);
            }
        };
        const auto fetch_a = [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int mi = 0; mi < MF; ++mi) af[u % HELD][mi] = frag(mi, u);
        };
        const auto transpose = [&](int u) __attribute__((always_inline)) {
            if constexpr (TRANSB == 0) {
#pragma unroll
                for (int ni = 0; ni < NF; ++ni) bf[ni] = gd::to_frag_t<T, CD>(w[u % HELD], ni);
            }
        };
        const auto multiply = [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < Tr::NJ; ++j)
#pragma unroll
                for (int mi = 0; mi < MF; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NF; ++ni) acc[mi][ni] = gd::mfma<T>(bf[ni], af[u % HELD][mi], j, acc[mi][ni]);
        };
        if constexpr (AHEAD) {
            fetch_b(0);
            fetch_a(0);
            transpose(0);
            __builtin_amdgcn_sched_barrier(0);
            fetch_b(1);
            fetch_a(1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(0);
            transpose(1);
            multiply(1);
        } else {
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                fetch_b(u);
                transpose(u);
                fetch_a(u);
                multiply(u);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const bool columns = !S::OWN || col0 < g.N;  // (of the last wavefronts of a tile-row some may have none)
    const int cnt = columns && !tiny ? whole + tail : 0;
    Stage sg[D];
    // (as little as may be in front of the first loads: 1.3 ns an instruction)
    if (cnt > 0) {
        const int first = tail ? g.K - KSTEP - kfirst : 0;
        load_at(first, sg[0]);
        if (MF < 4 && whole == 0) {
            abase += (int64_t)first * ES;
            bbase += first * bstep;
        }
        const int last = __builtin_amdgcn_readfirstlane(whole > 0 ? whole - 1 : 0);
        static_for<1, D>([&](auto q_c) { load_step(min(decltype(q_c)::value - tail, last), sg[decltype(q_c)::value]); });
        __builtin_amdgcn_sched_barrier(0);
        if (tail) clear_front(sg[0]);
        clear_acc();
        // OWN: K in four chains behind each other, as many as where wavefronts share it, for the same rounding error.
        // (A loop per chain: with the change of chains inside one loop the accumulators went through scratch memory.)
        accv_t done[S::OWN ? MF : 1][S::OWN ? NF : 1] = {};
        const int chain = S::OWN ? (cnt + 3) / 4 : cnt;
        for (int i = -tail, end = chain - tail;; end = min(end + chain, whole)) {  // (step -1: the one that K ends in)
            for (;;) {  // (past the last step the last one is read again, and dropped)
                compute(sg[0], [&] { load_step(min(i + D, last), sg[0]); });
                if (++i == end) break;
                if constexpr (D == 2) {
                    compute(sg[1], [&] { load_step(min(i + D, last), sg[1]); });
                    if (++i == end) break;
                }
            }
            if constexpr (!S::OWN) break;
#pragma unroll
            for (int f = 0; f < (S::OWN ? MF * NF : 0); ++f)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const acc_t sum = done[f / NF][f % NF][r] + acc[f / NF][f % NF][r];
                    done[f / NF][f % NF][r] = sum;
                    acc[f / NF][f % NF][r] = i == whole ? sum : (acc_t)0;
                }
            if (i == whole) break;
        }
    } else {
        clear_acc();
        if (g.K < KSTEP && wk == 0 && !tiny && columns) {
            load_part(0, rest, sg[0]);
            finish_part(rest, sg[0]);
            compute(sg[0], [] {});
        }
    }
    if constexpr (ANY) {
        if (tiny)
            for (int q = wk; q * KSTEP < g.K; q += WVK) {
                load_part(q / WVK, min(KSTEP, g.K - q * KSTEP), sg[0]);
                compute(sg[0], [] {});
            }
    }

    // ---- partial tiles of the WVK wavefronts -> LDS, as a tree ---------------------------------------------------
    if constexpr (!S::OWN) __syncthreads();  // the operand rows are no longer read
    if constexpr (WVK > 2) {
        accv_t* const buf = reinterpret_cast<accv_t*>(smem);
        constexpr int F = MF * NF * 64;  // vectors of one wavefront
#pragma unroll
        for (int active = WVK; active > 2; active /= 2) {
            const int half = active / 2;
            if (wk >= half && wk < active) {
#pragma unroll
                for (int f = 0; f < MF * NF; ++f)
                    buf[(wk - half) * F + f * 64 + lane] = acc[f / NF][f % NF];
            }
            __syncthreads();
            if (wk < half) {
#pragma unroll
                for (int f = 0; f < MF * NF; ++f)
                    acc[f / NF][f % NF] += buf[wk * F + f * 64 + lane];
            }
            __syncthreads();
        }
    }
    acc_t* const tile = reinterpret_cast<acc_t*>(smem + (S::OWN ? wave * S::AREA : 0));  // [SLOTS][BM][PITCH]
    // The column of C that column j of the tile holds, or -1.  With B stored K x N, a group of V columns that would
    // cross the end of the row was read from N - V on: its first columns repeat those of the group before.
    const bool nedge = col0 + S::BNW > g.N;  // wavefront-uniform
    auto edge_column = [&](int j) {  // (where nedge)
        if (TRANSB) return col0 + j < g.N ? col0 + j : -1;
        const int c = col0 + j / V * V, back = c - max(0, min(c, g.N - V));
        return j % V >= back && c - back + j % V < g.N ? c - back + j % V : -1;
    };
    auto column_of = [&](int j) { return nedge ? edge_column(j) : col0 + j; };
    // first of the NF columns of a lane's results r (FP64 results sit at index lq + 4 r of the fragment, the others at
    // 4 lq + r)
    const auto frag_col = [&](int r) { return (sizeof(acc_t) == 8 ? lq + 4 * r : 4 * lq + r) * NF; };
    const auto to_tile = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MF; ++mi)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc_t* p = tile + (wk * S::BM + mi * 16 + l16) * S::PITCH + frag_col(r);
                alignas(16) acc_t x[NF];
#pragma unroll
                for (int ni = 0; ni < NF; ++ni) x[ni] = acc[mi][ni][r];
                gd::copy_aligned<NF>(p, x);
            }
    };
    const bool inject = g.inj.mode != 0;
    if (wk < S::SLOTS && (!S::OWN || inject)) to_tile();  // (OWN: row sums first, see the epilogue)
    if constexpr (!S::OWN) __syncthreads();
    if constexpr (SPLIT) {
        if (!gd::join_split<S>(d, bm * g.tiles_n + bn, z, tile, s_last)) return;
    }

    // ---- fault injector (section 6.1 "Error injection"): the sum of the partial tiles, edited in place --------------
    if (inject) {
        const InjectArgs& inj = g.inj;
        for (int e = S::OWN ? lane : tid; e < S::BM * S::BNW; e += S::ET) {
            const int r = e / S::BNW, c = e % S::BNW, gi = row0 + r, gj = column_of(c);
            acc_t* p = tile + r * S::PITCH + c;
            acc_t x = *p;
            if (S::SLOTS == 2) x += p[(S::SLOTS - 1) * S::BM * S::PITCH];
            if (gi < g.M && gj >= 0) {
                const auto flip = [&](int bit) {
                    const acc_t before = x;
                    x = flip_bit(before, bit);
                    log_fault(inj, gi, gj, bit, (double)before, (double)x);
                };
                if (inj.mode == 1) {
                    for (int q = 0; q < inj.n_list; ++q) {
                        const int fb = inj.d_list[3 * q + 2];
                        if (inj.d_list[3 * q] == gi && inj.d_list[3 * q + 1] == gj && fb >= 0 && fb < acc_bits<acc_t>()) flip(fb);
                    }
                } else {
                    const int bit = bernoulli_bit(inj, gi, gj, g.N);
                    if (bit >= 0) flip(bit);
                }
            }
            *p = x;
        }
        if constexpr (!S::OWN) __syncthreads();
    }

    // ---- epilogue: a thread owns EPT consecutive columns of a row -----------------------------------------------
    constexpr bool wsum = W;
    const bool csum = d.csum != 0;
    using out_t = typename Tr::out_t;
    constexpr int EPT = S::EPT, PASSES = S::PASSES;
    static_assert(EPT * sizeof(acc_t) < 16 || EPT * sizeof(acc_t) % 16 == 0, "LDS vectors");
    const int tr = (S::OWN ? lane : tid) / S::TPR, tc = tid % S::TPR * EPT;
    const auto store_row = [&](int gi, const acc_t* v) __attribute__((always_inline)) {
        if (gi >= g.M) return;
        out_t* c = reinterpret_cast<out_t*>(g.C) + (int64_t)gi * g.ldc;
        if (EPT >= 4 && !nedge) {
#pragma unroll
            for (int e = 0; e + 3 < EPT; e += 4) gd::store4<T, S::OWN>(c + col0 + tc + e, v + e);
        } else {
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int gj = column_of(tc + e);
                if (gj >= 0) c[gj] = gd::to_out<T, acc_t>(v[e]);
            }
        }
    };
    // sums of row row0 + srow over the columns of partial number part, which the thread stores if has_sum
    acc_t rs = 0, rs2 = 0;
    int srow = tr, part = bn;
    bool has_sum = tid % S::TPR == 0;
    alignas(16) acc_t v[PASSES][EPT];
    if constexpr (S::OWN) {
        // Row sums straight from the accumulators: 15 additions and two exchanges per 16 rows, and the tile's way through
        // LDS to whole pieces of rows covers the partials' way to memory.  From the tile in LDS, 16 passes of three
        // additions and four exchanges, they took longer than the product of a short K.
        if (inject) {
#pragma unroll
            for (int mi = 0; mi < MF; ++mi)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    alignas(16) acc_t x[NF];
                    gd::copy_aligned<NF>(x, tile + (mi * 16 + l16) * S::PITCH + frag_col(r));
#pragma unroll
                    for (int ni = 0; ni < NF; ++ni) acc[mi][ni][r] = x[ni];
                }
        }
        if (verify) {
            const int first = frag_col(0);
#pragma unroll
            for (int mi = 0; mi < MF; ++mi) {
                acc_t x[4 * NF];
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int ni = 0; ni < NF; ++ni)
                        x[r * NF + ni] = !nedge || column_of(frag_col(r) + ni) >= 0 ? acc[mi][ni][r] : (acc_t)0;
                acc_t s2 = 0;
                if (wsum) {
                    // weights from the lane's first column on; that column's own weight goes with the plain sum below
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int ni = 0; ni < NF; ++ni) {
                            const int j = frag_col(r) + ni;
                            s2 = fma((acc_t)(nedge ? max(0, column_of(j)) - (col0 + first) : j - first), x[r * NF + ni], s2);
                        }
                }
#pragma unroll
                for (int w = 1; w < 4 * NF; w *= 2)
#pragma unroll
                    for (int e = 0; e + w < 4 * NF; e += 2 * w) x[e] += x[e + w];
                acc_t s = x[0];
                if (wsum) s2 = fma((acc_t)(col0 + first + 1), s, s2);
                const auto over_groups = [](acc_t q) {  // the four lanes of a row
                    acc_t a, b;
                    lane_exchange<32, WAVE>(q, a, b);
                    lane_exchange<16, WAVE>((acc_t)(a + b), a, b);
                    return (acc_t)(a + b);
                };
                s = over_groups(s);
                if (wsum) s2 = over_groups(s2);
                rs = lq == mi ? s : rs;  // row 16 lq + l16 = lane
                rs2 = lq == mi ? s2 : rs2;
            }
            if (g.block_mode && Tr::ES > 2) {  // compared per block of 64 columns: one partial per wavefront
                srow = lane;
                part = bn * WN + wn;
                has_sum = lane < S::BM && col0 < g.N;
            } else {
                acc_t* const sums = reinterpret_cast<acc_t*>(smem + S::SUMS);
                if (lane < S::BM) {
                    sums[wn * S::BM + lane] = rs;
                    sums[(WN + wn) * S::BM + lane] = rs2;
                }
                __syncthreads();
                srow = tid;
                has_sum = tid < S::BM;
                if (has_sum) {
                    static_assert(WN == 4, "");
                    rs = (sums[tid] + sums[S::BM + tid]) + (sums[2 * S::BM + tid] + sums[3 * S::BM + tid]);
                    rs2 = (sums[4 * S::BM + tid] + sums[5 * S::BM + tid]) + (sums[6 * S::BM + tid] + sums[7 * S::BM + tid]);
                }
            }
        }
    } else {
        const int gi = row0 + tr;
        acc_t* const src = tile + tr * S::PITCH + tc;
        gd::copy_aligned<EPT>(v[0], src);
        if (S::SLOTS == 2 && !inject) {
            alignas(16) acc_t u[EPT];
            gd::copy_aligned<EPT>(u, src + (S::SLOTS - 1) * S::BM * S::PITCH);
#pragma unroll
            for (int e = 0; e < EPT; ++e) v[0][e] += u[e];
        }
        if (verify) {
            acc_t x[EPT];
#pragma unroll
            for (int e = 0; e < EPT; ++e) x[e] = v[0][e];
            if (nedge) {
#pragma unroll
                for (int e = 0; e < EPT; ++e) x[e] = edge_column(tc + e) >= 0 ? x[e] : (acc_t)0;
            }
            if (csum) {
#pragma unroll
                for (int e = 0; e < EPT; ++e) src[e] = gi < g.M ? x[e] : (acc_t)0;
            }
            acc_t s2 = 0;
            if (wsum) {
                // weights from the thread's first column on; that column's own weight goes with the plain sum below
#pragma unroll
                for (int e = 0; e < EPT; ++e)
                    s2 = fma((acc_t)(nedge ? max(0, edge_column(tc + e)) - (col0 + tc) : e), x[e], s2);
            }
#pragma unroll
            for (int w = 1; w < EPT; w *= 2)
#pragma unroll
                for (int e = 0; e + w < EPT; e += 2 * w) x[e] += x[e + w];
            acc_t s = x[0];
            if (wsum) s2 = fma((acc_t)(col0 + tc + 1), s, s2);
            rs = group_sum<S::TPR>(s);
            if (wsum) rs2 = group_sum<S::TPR>(s2);
        }
    }
    if (verify && has_sum && row0 + srow < g.M) {
        st_agent(reinterpret_cast<acc_t*>(g.rowpart) + (int64_t)part * g.M + row0 + srow, rs);
        if constexpr (W) st_agent(reinterpret_cast<acc_t*>(g.rowpart2) + (int64_t)part * g.M + row0 + srow, rs2);
    }
    if constexpr (S::OWN) {
        if (!inject) to_tile();
#pragma unroll
        for (int p = 0; p < PASSES; ++p) gd::copy_aligned<EPT>(v[p], tile + (p * S::RPP + tr) * S::PITCH + tc);
    }
    const auto store_c = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) store_row(row0 + p * S::RPP + tr, v[p]);
    };
    if constexpr (W && !S::OWN) {
        // Flagged rows are corrected by the workgroup that compares them: C has to be in memory by then, not in this XCD's cache.
        // (rows of C are aligned to 8 bytes; whole groups of them, and what the edge leaves by elements)
        if (d.wsum == 2 && row0 + tr < g.M) {
            out_t* const c = reinterpret_cast<out_t*>(g.C) + (int64_t)(row0 + tr) * g.ldc;
            constexpr int G = 8 / (int)sizeof(out_t);
#pragma unroll
            for (int e = 0; e < EPT; e += G) {
                if constexpr (EPT % G == 0) {
                    if (!nedge) {
                        __hip_atomic_store(reinterpret_cast<uint64_t*>(c + col0 + tc + e), gd::word8<T>(v[0] + e), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        continue;
                    }
                }
#pragma unroll
                for (int q = 0; q < G && e + q < EPT; ++q) {
                    const int gj = column_of(tc + e + q);
                    if (gj >= 0) CElem<T>::put_agent(reinterpret_cast<typename CElem<T>::store_t*>(c) + gj, v[0][e + q]);
                }
            }
        }
    }
    const bool check = verify && !g.block_mode;
    if (!check) store_c();
    if (!verify) return;
    if (csum) {
        if constexpr (!S::OWN) __syncthreads();
        for (int c = S::OWN ? lane : tid; c < S::BNW; c += S::ET) {
            acc_t q[4] = {0, 0, 0, 0};
            for (int r = 0; r < S::BM; r += 4)
#pragma unroll
                for (int k = 0; k < 4; ++k) q[k] += !S::OWN || row0 + r + k < g.M ? tile[(r + k) * S::PITCH + c] : (acc_t)0;
            const int gj = column_of(c);
            if (gj >= 0)  // compared by a kernel of their own
                reinterpret_cast<acc_t*>(g.colpart)[(int64_t)bm * g.N + gj] = (q[0] + q[1]) + (q[2] + q[3]);
        }
    }
    if (check) direct_tile_row_check<T, S, W>(d, bm, s_last, smem, store_c);
}

template <bool W, typename T, int TRANSB, int MF, int NF, int WVK, int D, bool ANY = false, int WN = 1, bool SPLIT = false>
static int gemm_direct_launch_shape(const DirectArgs& d, hipStream_t st) {
    using S = gd::Shape<T, TRANSB, MF, NF, WVK, WN>;
    if constexpr (!SPLIT && WVK > 1 && !ANY)
        if (d.split > 1) return gemm_direct_launch_shape<W, T, TRANSB, MF, NF, WVK, D, ANY, WN, true>(d, st);
    auto kern = gemm_direct_kernel<T, TRANSB, MF, NF, WVK, WN, D, ANY, SPLIT, W>;
    if constexpr (S::LDS > 65536) {
        static bool attr_set = false;
        if (!attr_set) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    S::LDS) != hipSuccess)
                return VABFT_EDEVICE;
            attr_set = true;
        }
    }
    const int blocks = d.stat_blocks + d.tile_blocks;
    DirectArgs part = d;
    for (int64_t at = 0; at < blocks; at += gd::LAUNCH_MOST) {
        part.first_block = (int32_t)(d.mirror ? blocks - at : at);
        kern<<<dim3((unsigned)std::min<int64_t>(blocks - at, gd::LAUNCH_MOST)), dim3(S::NT), S::LDS, st>>>(part);
    }
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

// shape: see DirectShape.  Two steps are in flight from global memory where the registers allow it.
template <bool W, typename T, int TRANSB> static int gemm_direct_launch_tb(const DirectArgs& d, int shape, hipStream_t st) {
    constexpr int NS = TRANSB ? 2 : 4;  // a lane reads four columns of a K x N B
    switch (shape) {
        case DIRECT_16: return gemm_direct_launch_shape<W, T, TRANSB, 1, NS, 8, TRANSB ? 2 : 1>(d, st);
        case DIRECT_32: return gemm_direct_launch_shape<W, T, TRANSB, 2, NS, 8, TRANSB ? 2 : 1>(d, st);
        case DIRECT_32W: return gemm_direct_launch_shape<W, T, TRANSB, 2, 4, 4, 1>(d, st);
        case DIRECT_ANY: return gemm_direct_launch_shape<W, T, TRANSB, 2, 4, 4, 1, true>(d, st);
        case DIRECT_64:
            if constexpr (!std::is_same<T, double>::value)
                return gemm_direct_launch_shape<W, T, TRANSB, 4, 4, 4, std::is_same<T, float>::value || !TRANSB ? 1 : 2>(d, st);
            break;
        case DIRECT_OWN32: return gemm_direct_launch_shape<W, T, TRANSB, 2, 4, 1, 1, false, 4>(d, st);
        case DIRECT_OWN64:
            if constexpr (!std::is_same<T, double>::value)
                return gemm_direct_launch_shape<W, T, TRANSB, 4, 4, 1, 1, false, 4>(d, st);
    }
    return VABFT_EINVAL;
}
template <bool W, typename T> static int gemm_direct_launch_t(const DirectArgs& d, int shape, int transB, hipStream_t st) {
    return transB ? gemm_direct_launch_tb<W, T, 1>(d, shape, st) : gemm_direct_launch_tb<W, T, 0>(d, shape, st);
}

}  // namespace vabft
