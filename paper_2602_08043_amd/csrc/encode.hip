// Checksum encode B*r1 with per-row (max, min, mean) statistics and the three B aggregates
// of Algorithm 1 (paper section 2.2 Eq. r1 / encoded matrices; section 3.5; Algorithm 1 k-loop),
// and the A-side pass: row statistics, expected checksum A*(B r1) and the threshold T_m
// (section 3.4 boxed formula).  Both are single streaming passes bound by HBM bandwidth.
#include <algorithm>
#include <type_traits>

#include "row_threshold.h"
#include "unpack.h"
#include "vabft_device.h"
#include "vabft_host.h"

namespace vabft {

// ---------------------------------------------------------------------------
// S1, S2, S3 without a launch of their own: every block publishes the three sums over its own
// rows k (Algorithm 1: S1 += |mu_Bk|, S2 += sigma_Bk^2, S3 += mu_Bk^2) and takes an arrival ticket;
// the last block folds all partials in block order.  Partials and ticket go through device-scope
// relaxed atomics (the blocks sit on XCDs with private L2s); the ticket is left at zero.
// s1..s3 need to be valid in thread 0 only.  Every thread of the block must call this.
// ---------------------------------------------------------------------------
// (leaves, entry: which threads of the first wavefront leave an entry, and which; of count)
__device__ __forceinline__ void publish_entry_and_fold_S(bool leaves, int entry, int count, double s1, double s2, double s3,
                                                         double* __restrict__ partial, int32_t* __restrict__ ticket,
                                                         double* __restrict__ S) {
    __shared__ int s_last;
    __shared__ double s_red[3][4];
    const int t = threadIdx.x;
    double* const mine = partial + 3 * (int64_t)entry;
    if (S == nullptr) {
        // deferred fold: the partials stay where they are (plain stores: the consumer is a later kernel
        // on the stream, which folds them in this same order)
        if (leaves) {
            mine[0] = s1;
            mine[1] = s2;
            mine[2] = s3;
        }
        return;
    }
    if (leaves) {
        st_agent(mine, s1);
        st_agent(mine + 1, s2);
        st_agent(mine + 2, s3);
    }
    if (t < 64) __builtin_amdgcn_s_waitcnt(0);  // the partials are performed before the ticket is taken
    if (t == 0) s_last = atomicAdd(ticket, 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    if (t < 256) {
        // thread t folds entries t, t + 256, ... in increasing order; butterfly inside each of the
        // four wavefronts; the four results in order
        double a1 = 0, a2 = 0, a3 = 0;
        for (int b = t; b < count; b += 256) {
            const double* q = partial + 3 * (int64_t)b;
            a1 += ld_agent(q);
            a2 += ld_agent(q + 1);
            a3 += ld_agent(q + 2);
        }
        a1 = wave_sum(a1);
        a2 = wave_sum(a2);
        a3 = wave_sum(a3);
        if ((t & 63) == 0) {
            s_red[0][t >> 6] = a1;
            s_red[1][t >> 6] = a2;
            s_red[2][t >> 6] = a3;
        }
    }
    __syncthreads();
    if (t < 3) {
        const int nw = blockDim.x < 256 ? (blockDim.x + 63) / 64 : 4;
        double v = 0;
        for (int w = 0; w < nw; ++w) v += s_red[t][w];
        S[t] = v;
    }
    if (t == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_and_fold_S(double s1, double s2, double s3, double* __restrict__ partial,
                                                   int32_t* __restrict__ ticket, double* __restrict__ S) {
    publish_entry_and_fold_S(threadIdx.x == 0, blockIdx.x, gridDim.x, s1, s2, s3, partial, ticket, S);
}

// the three per-row terms of S1, S2, S3 from (row sum, max, min) of a row of N elements
template <typename acc_t>
__device__ __forceinline__ void row_terms(acc_t sum, acc_t mx, acc_t mn, int N, double& t1, double& t2, double& t3) {
    const double mu = (double)sum / (double)N;
    double var = ((double)mx - mu) * (mu - (double)mn);  // section 3.5: sigma^2 <= (max - mu)(mu - min)
    var = var > 0 ? var : 0;
    t1 = fabs(mu);
    t2 = var;
    t3 = mu * mu;
}

// ---------------------------------------------------------------------------
// B stored K x N: WAVES wavefronts per block reduce RPB rows k, WAVES / RPB wavefronts per row (each a
// contiguous segment of the row, combined in segment order).  RPB is WAVES when that gives enough
// blocks to fill the chip, else half of it, and so on down to 1.
// WAVES is 16 when the kernel folds S1..S3 itself (the fold's tail is one atomic per block on one address,
// about 11 ns each, so fewer and larger blocks are faster: 11.7 against 13.9 us at 4096 x 4096 BF16) and 8 when
// the fold is deferred (smaller blocks retire and refill sooner: 25.3 against 28.3 us at 8192 x 8192 FP16).
// ---------------------------------------------------------------------------

// W: also the position-weighted checksum B*r2, r2 = [1..N] (section 2.2): Be2[k] = sum_n (n+1) B[k,n].
template <typename T, bool W, int RPB, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void encode_rows_kernel(const void* __restrict__ B, int K, int N, int64_t ldb,
                                                           typename Elem<T>::acc_t* __restrict__ Be,
                                                           typename Elem<T>::acc_t* __restrict__ Be2,
                                                           typename Elem<T>::acc_t* __restrict__ bstat,
                                                           double* __restrict__ s_partial,
                                                           int32_t* __restrict__ ticket, double* __restrict__ S) {
    using acc_t = typename Elem<T>::acc_t;
    constexpr int V = Elem<T>::vec;
    constexpr int WPR = WAVES / RPB;  // wavefronts per row
    __shared__ double terms[RPB][3];
    __shared__ acc_t seg[WAVES][4];  // (sum, weighted sum, max, min) of each wavefront's segment
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * RPB + wave / WPR, part = wave % WPR;
    acc_t sum = 0, sum2 = 0, mx = -type_max<acc_t>(), mn = type_max<acc_t>();
    if (k < K) {
        const char* row = reinterpret_cast<const char*>(B) + (int64_t)k * ldb * Elem<T>::bytes;
        int done = 0;
        {
            const int nchunks = N / V;
            // segment of this wavefront: a multiple of 64 chunks, the last one takes what is left
            const int per = ((nchunks + WPR - 1) / WPR + 63) / 64 * 64;
            const int c_end = part == WPR - 1 ? nchunks : min(nchunks, (part + 1) * per);
            int c = part * per + lane;
            for (; c + 192 < c_end; c += 256) {
                raw16 r0 = ld16u<T>(row + (int64_t)c * 16);
                raw16 r1 = ld16u<T>(row + (int64_t)(c + 64) * 16);
                raw16 r2 = ld16u<T>(row + (int64_t)(c + 128) * 16);
                raw16 r3 = ld16u<T>(row + (int64_t)(c + 192) * 16);
                acc_t v[4][V];
                Unpack<T>::run(r0, v[0]);
                Unpack<T>::run(r1, v[1]);
                Unpack<T>::run(r2, v[2]);
                Unpack<T>::run(r3, v[3]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        sum += v[u][e];
                        if constexpr (W) sum2 = fma((acc_t)((c + 64 * u) * V + e + 1), v[u][e], sum2);
                        mx = fmax(mx, v[u][e]);
                        mn = fmin(mn, v[u][e]);
                    }
            }
            for (; c < c_end; c += 64) {
                raw16 r0 = ld16u<T>(row + (int64_t)c * 16);
                acc_t v[V];
                Unpack<T>::run(r0, v);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    sum += v[e];
                    if constexpr (W) sum2 = fma((acc_t)(c * V + e + 1), v[e], sum2);
                    mx = fmax(mx, v[e]);
                    mn = fmin(mn, v[e]);
                }
            }
            done = nchunks * V;
        }
        // what the 16-byte pieces do not cover (everything, for unaligned rows): the last segment's wavefront
        if (part == WPR - 1) {
            for (int n = done + lane; n < N; n += 64) {
                acc_t x = Unpack<T>::one(row, n);
                sum += x;
                if constexpr (W) sum2 = fma((acc_t)(n + 1), x, sum2);
                mx = fmax(mx, x);
                mn = fmin(mn, x);
            }
        }
        sum = wave_sum(sum);
        mx = wave_max(mx);
        mn = wave_min(mn);
        if constexpr (W) sum2 = wave_sum(sum2);
    }
    if constexpr (WPR > 1) {
        if (lane == 0) {
            seg[wave][0] = sum;
            seg[wave][1] = sum2;
            seg[wave][2] = mx;
            seg[wave][3] = mn;
        }
        __syncthreads();
        if (part == 0 && lane == 0) {
            sum = seg[wave][0];
            sum2 = seg[wave][1];
            mx = seg[wave][2];
            mn = seg[wave][3];
#pragma unroll
            for (int q = 1; q < WPR; ++q) {  // segments in order
                sum += seg[wave + q][0];
                sum2 += seg[wave + q][1];
                mx = fmax(mx, seg[wave + q][2]);
                mn = fmin(mn, seg[wave + q][3]);
            }
        }
    }
    double t1 = 0, t2 = 0, t3 = 0;
    if (k < K && part == 0 && lane == 0) {
        if constexpr (W) Be2[k] = sum2;
        Be[k] = sum;
        bstat[3 * (int64_t)k + 0] = mx;
        bstat[3 * (int64_t)k + 1] = mn;
        bstat[3 * (int64_t)k + 2] = (acc_t)((double)sum / (double)N);
        row_terms(sum, mx, mn, N, t1, t2, t3);
    }
    if (part == 0 && lane == 0) {
        terms[wave / WPR][0] = t1;
        terms[wave / WPR][1] = t2;
        terms[wave / WPR][2] = t3;
    }
    __syncthreads();
    double s1 = 0, s2 = 0, s3 = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < RPB; ++w) {  // rows of the block in order
            s1 += terms[w][0];
            s2 += terms[w][1];
            s3 += terms[w][2];
        }
    }
    publish_and_fold_S(s1, s2, s3, s_partial, ticket, S);
}

// ---------------------------------------------------------------------------
// B stored N x K (weight layout): column reduction in two steps.
// Step 1: block (kx, ny) reduces rows [ny*rows_per_block, ...) of 64*V columns.
// part layout: [nsplit][4][K] (sum, max, min, weighted sum; the last only when W).
// The weight of row n is n + 1 (the vector r2), or wvec[n] when a weight vector is given (then the
// weighted sum is the dot product of every column with that vector).
// ---------------------------------------------------------------------------
template <typename T, bool W, int COLS_NL>
__global__ __launch_bounds__(256) void encode_cols_kernel(const void* __restrict__ Bt, int K, int N, int64_t ldb,
                                                          int rows_per_block,
                                                          typename Elem<T>::acc_t* __restrict__ part,
                                                          const typename Elem<T>::acc_t* __restrict__ wvec) {
    using acc_t = typename Elem<T>::acc_t;
    constexpr int V = Elem<T>::vec;
    __shared__ acc_t red[3][W ? 4 : 3][65 * V];  // waves 1..3 park their partials here, [e][lane] with pitch 65
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // A lane whose columns would cross the end of the row takes the last V instead, lanes behind it the same: the wavefront
    // has one loop.  (With a loop of its own for what is left over, element by element, the last workgroups took twice
    // as long: FP8 2047 rows and columns 30 against 27 us, BF16 5000 x 5000, where nothing is left over, 17.3 against 16.1.)
    const int k0 = min((blockIdx.x * 64 + lane) * V, max(0, K - V));
    const int n_begin = blockIdx.y * rows_per_block;
    const int n_end = min(N, n_begin + rows_per_block);
    acc_t sum[V], sum2[V], mx[V], mn[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        sum[e] = 0;
        sum2[e] = 0;
        mx[e] = -type_max<acc_t>();
        mn[e] = type_max<acc_t>();
    }
    if (K >= V) {
        int n = n_begin + wave;
        // COLS_NL rows in flight per wavefront (a wavefront reads 1 KiB of every fourth row of the slab)
        for (; n + 4 * (COLS_NL - 1) < n_end; n += 4 * COLS_NL) {
            raw16 r[COLS_NL];
#pragma unroll
            for (int u = 0; u < COLS_NL; ++u)
                r[u] = ld16u<T>(reinterpret_cast<const char*>(Bt) + ((int64_t)(n + 4 * u) * ldb + k0) * Elem<T>::bytes);
#pragma unroll
            for (int u = 0; u < COLS_NL; ++u) {
                acc_t v[V];
                Unpack<T>::run(r[u], v);
                const acc_t w = !W ? (acc_t)0 : (wvec ? wvec[n + 4 * u] : (acc_t)(n + 4 * u + 1));
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    sum[e] += v[e];
                    if constexpr (W) sum2[e] = fma(w, v[e], sum2[e]);
                    mx[e] = fmax(mx[e], v[e]);
                    mn[e] = fmin(mn[e], v[e]);
                }
            }
        }
        for (; n < n_end; n += 4) {
            raw16 r0 = ld16u<T>(reinterpret_cast<const char*>(Bt) + ((int64_t)n * ldb + k0) * Elem<T>::bytes);
            acc_t v[V];
            Unpack<T>::run(r0, v);
            const acc_t w = !W ? (acc_t)0 : (wvec ? wvec[n] : (acc_t)(n + 1));
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sum[e] += v[e];
                if constexpr (W) sum2[e] = fma(w, v[e], sum2[e]);
                mx[e] = fmax(mx[e], v[e]);
                mn[e] = fmin(mn[e], v[e]);
            }
        }
    } else {
        for (int n = n_begin + wave; n < n_end; n += 4) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                if (k0 + e < K) {
                    acc_t x = Unpack<T>::one(Bt, (int64_t)n * ldb + k0 + e);
                    sum[e] += x;
                    if constexpr (W) sum2[e] = fma(wvec ? wvec[n] : (acc_t)(n + 1), x, sum2[e]);
                    mx[e] = fmax(mx[e], x);
                    mn[e] = fmin(mn[e], x);
                }
            }
        }
    }
    // LDS layout [e][lane] with a pitch of 65: conflict free both for a wavefront writing one e at a time and for
    // consecutive threads reading consecutive columns (lane * V + e) afterwards
    constexpr int PITCH = 65;
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            red[wave - 1][0][e * PITCH + lane] = sum[e];
            red[wave - 1][1][e * PITCH + lane] = mx[e];
            red[wave - 1][2][e * PITCH + lane] = mn[e];
            if constexpr (W) red[wave - 1][3][e * PITCH + lane] = sum2[e];
        }
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sum[e] += red[w][0][e * PITCH + lane];
                acc_t a = red[w][1][e * PITCH + lane], b = red[w][2][e * PITCH + lane];
                mx[e] = fmax(mx[e], a);
                mn[e] = fmin(mn[e], b);
                if constexpr (W) sum2[e] += red[w][3][e * PITCH + lane];
            }
        // the block's results go back through the first area so that the global stores are contiguous
        // (LDS operations of one wavefront complete in order: the reads above are done)
#pragma unroll
        for (int e = 0; e < V; ++e) {
            red[0][0][e * PITCH + lane] = sum[e];
            red[0][1][e * PITCH + lane] = mx[e];
            red[0][2][e * PITCH + lane] = mn[e];
            if constexpr (W) red[0][3][e * PITCH + lane] = sum2[e];
        }
    }
    __syncthreads();
    {
        acc_t* p = part + (int64_t)blockIdx.y * 4 * K;
        const int kbase = blockIdx.x * 64 * V;
#pragma unroll
        for (int j = 0; j < (64 * V + 255) / 256; ++j) {
            const int idx = threadIdx.x + 256 * j;  // column kbase + idx = lane idx / V, element idx % V
            if (idx < 64 * V && kbase + idx < K) {
                const int behind = max(0, kbase + idx / V * V - max(0, K - V));  // columns that the lane was moved back by
                const int at = (idx % V + behind) * PITCH + idx / V;
                p[kbase + idx] = red[0][0][at];
                p[(int64_t)K + kbase + idx] = red[0][1][at];
                p[2 * (int64_t)K + kbase + idx] = red[0][2][at];
                if constexpr (W) p[3 * (int64_t)K + kbase + idx] = red[0][3][at];
            }
        }
    }
}

// Step 2: combine the nsplit partials of column k in a fixed order: 16 columns per block,
// 16 groups of threads per column; group g folds splits g, g+16, ... in increasing order and
// the 16 group results are folded in group order.
template <typename acc_t, bool W>
__global__ __launch_bounds__(256) void encode_cols_combine_kernel(const acc_t* __restrict__ part, int nsplit, int K,
                                                                  int N, acc_t* __restrict__ Be,
                                                                  acc_t* __restrict__ Be2,
                                                                  acc_t* __restrict__ bstat,
                                                                  double* __restrict__ s_partial,
                                                                  int32_t* __restrict__ ticket,
                                                                  double* __restrict__ S) {
    __shared__ acc_t red[W ? 4 : 3][16][16];
    __shared__ double terms[16][3];
    const int kl = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int k = blockIdx.x * 16 + kl;
    acc_t sum = 0, sum2 = 0, mx = -type_max<acc_t>(), mn = type_max<acc_t>();
    if (k < K) {
        for (int s = grp; s < nsplit; s += 16) {
            const acc_t* p = part + (int64_t)s * 4 * K;
            sum += p[k];
            if constexpr (W) sum2 += p[3 * (int64_t)K + k];
            const acc_t a = p[(int64_t)K + k], b = p[2 * (int64_t)K + k];
            mx = fmax(mx, a);
            mn = fmin(mn, b);
        }
    }
    red[0][grp][kl] = sum;
    red[1][grp][kl] = mx;
    red[2][grp][kl] = mn;
    if constexpr (W) red[3][grp][kl] = sum2;
    __syncthreads();
    if (grp == 0 && k < K) {
        sum = red[0][0][kl];
        mx = red[1][0][kl];
        mn = red[2][0][kl];
        if constexpr (W) sum2 = red[3][0][kl];
#pragma unroll
        for (int g = 1; g < 16; ++g) {
            sum += red[0][g][kl];
            if constexpr (W) sum2 += red[3][g][kl];
            const acc_t a = red[1][g][kl], b = red[2][g][kl];
            mx = fmax(mx, a);
            mn = fmin(mn, b);
        }
        Be[k] = sum;
        if constexpr (W) Be2[k] = sum2;
        bstat[3 * (int64_t)k + 0] = mx;
        bstat[3 * (int64_t)k + 1] = mn;
        bstat[3 * (int64_t)k + 2] = (acc_t)((double)sum / (double)N);
    }
    // S1, S2, S3: the block's 16 columns in order, then across blocks
    if (grp == 0) {
        double t1 = 0, t2 = 0, t3 = 0;
        if (k < K) row_terms(sum, mx, mn, N, t1, t2, t3);
        terms[kl][0] = t1;
        terms[kl][1] = t2;
        terms[kl][2] = t3;
    }
    __syncthreads();
    double s1 = 0, s2 = 0, s3 = 0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            s1 += terms[c][0];
            s2 += terms[c][1];
            s3 += terms[c][2];
        }
    }
    publish_and_fold_S(s1, s2, s3, s_partial, ticket, S);
}

// ---------------------------------------------------------------------------
// The same column reduction in one launch, for matrices of few enough rows: a workgroup of 16 wavefronts takes all rows of
// LPR * V columns, LPR lanes to a row, and finishes them (panel_pays: where that is the faster form).  The two steps above
// cost a second launch and the partials' way through memory; here the rows' loads are what it takes, 8 KiB in flight per
// wavefront, and FP8's and 16-bit types' arithmetic.  Over the rows of a wavefront two values share a lane swap (one value to
// a swap, BF16 96 x 64 7.4 us against 5.4, FP8 10.1 / 5.9).
// The panels whose columns share a cache line run on one XCD, one after the other.
// ---------------------------------------------------------------------------
constexpr int PANEL_WAVES = 16;

template <typename T, int LPR_> struct Panel {
    static constexpr int V = Elem<T>::vec;
    static constexpr int LPR = LPR_, COLS = LPR * V, GROUPS = 64 / LPR;  // (a multiple of 16 columns: of a term of S1..S3)
    static constexpr int NL = V == 16 || V == 2 ? 4 : 8;                 // rows in flight per lane
    static_assert(COLS % 16 == 0 && (LPR == 1 || LPR == 2 || LPR == 4 || LPR == 8), "");
};

// Lanes of the lower half (of even rows of 16): x of this lane combined with x of its partner OFF lanes on; the others: y.
template <int OFF> __device__ __forceinline__ void swap_lanes(uint32_t& x, uint32_t& y) {
    const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                             : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}
template <int OFF, typename F> __device__ __forceinline__ float pair_over_rows(float x, float y, F f) {
    uint32_t a = __float_as_uint(x), b = __float_as_uint(y);
    swap_lanes<OFF>(a, b);
    return f(__uint_as_float(a), __uint_as_float(b));
}
template <int OFF, typename F> __device__ __forceinline__ double pair_over_rows(double x, double y, F f) {
    uint32_t al = (uint32_t)__double2loint(x), bl = (uint32_t)__double2loint(y);
    uint32_t ah = (uint32_t)__double2hiint(x), bh = (uint32_t)__double2hiint(y);
    swap_lanes<OFF>(al, bl);
    swap_lanes<OFF>(ah, bh);
    return f(__hiloint2double((int)ah, (int)al), __hiloint2double((int)bh, (int)bl));
}
// Over the rows of a wavefront: v[e] of all lanes with the same lane % LPR, two values to a lane swap while there are two.
// Leaves v[0 .. V / 4) (V = 2: v[0]): element first + i, with first of the lane (panel_first), in the first LPR lanes
// of every 16.
template <int V, int LPR, typename A, typename F> __device__ __forceinline__ void over_rows(A* v, F f) {
#pragma unroll
    for (int e = 0; e < V / 2; ++e) v[e] = pair_over_rows<32>(v[e], v[e + V / 2], f);
    constexpr int H = V / 4;
    if constexpr (H > 0) {
#pragma unroll
        for (int e = 0; e < H; ++e) v[e] = pair_over_rows<16>(v[e], v[e + H], f);
    } else {
        v[0] = pair_over_rows<16>(v[0], v[0], f);
    }
#pragma unroll
    for (int e = 0; e < (H > 0 ? H : 1); ++e) {
        A a, b;
        lane_exchange<8, 64>(v[e], a, b);
        v[e] = f(a, b);
        if constexpr (LPR <= 4) {
            lane_exchange<4, 64>(v[e], a, b);
            v[e] = f(a, b);
        }
        if constexpr (LPR <= 2) {
            lane_exchange<2, 64>(v[e], a, b);
            v[e] = f(a, b);
        }
        if constexpr (LPR == 1) {
            lane_exchange<1, 64>(v[e], a, b);
            v[e] = f(a, b);
        }
    }
}
template <int V> __device__ __forceinline__ int panel_first(int lane) {
    return (lane >> 5) * (V / 2) + (V >= 4 ? (lane >> 4 & 1) * (V / 4) : 0);
}

// What becomes of a column's (sum, max, min, weighted sum).  Encode: B r1 and statistics, terms of S1..S3 (Be2: weighted).
template <typename acc_t> struct PanelEncode {
    acc_t* Be;
    acc_t* Be2;
    acc_t* bstat;
    double* s_partial;
    int32_t* ticket;
    double* S;
    static constexpr bool AGGREGATES = true;
    __device__ const acc_t* weights() const { return nullptr; }
    __device__ void column(int k, int rows, acc_t sum, acc_t mx, acc_t mn, acc_t sum2) const {
        if (Be2) Be2[k] = sum2;
        Be[k] = sum;
        bstat[3 * (int64_t)k + 0] = mx;
        bstat[3 * (int64_t)k + 1] = mn;
        bstat[3 * (int64_t)k + 2] = (acc_t)((double)sum / (double)rows);
    }
};

template <typename T, bool W, int LPR, typename Out>
__global__ __launch_bounds__(64 * PANEL_WAVES) void panel_kernel(const void* __restrict__ Bt, int K, int N, int64_t ldb,
                                                                 const Out out) {
    using acc_t = typename Elem<T>::acc_t;
    using P = Panel<T, LPR>;
    constexpr int V = P::V, COLS = P::COLS, Q = W ? 4 : 3, STEP = PANEL_WAVES * P::GROUPS;
    __shared__ acc_t red[PANEL_WAVES][Q][COLS];
    __shared__ double terms[COLS][3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cl = lane % P::LPR;
    // G panels to a line of 128 bytes: of every 8 G consecutive workgroups those G that run on one XCD take a line's
    constexpr int G = 128 / (16 * P::LPR);
    const int chunk = blockIdx.x / (8 * G), r = blockIdx.x % (8 * G);
    const int panel = (chunk + 1) * 8 * G <= (int)gridDim.x ? chunk * 8 * G + r % 8 * G + r / 8 : (int)blockIdx.x;
    // (a lane whose columns would cross the end of the row takes the last V instead, lanes behind it the same)
    const int nominal = panel * COLS + cl * V, k0 = min(nominal, K - V);
    acc_t sum[V], sum2[W ? V : 1], mx[V], mn[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        sum[e] = 0;
        if constexpr (W) sum2[e] = 0;
        mx[e] = -type_max<acc_t>();
        mn[e] = type_max<acc_t>();
    }
    // (a panel's columns from its first on: a lane moved back leaves them at other threads' places)
    if (Out::AGGREGATES && tid < COLS) terms[tid][0] = terms[tid][1] = terms[tid][2] = 0;
    const acc_t* const wvec = out.weights();
    const char* const base = reinterpret_cast<const char*>(Bt) + (int64_t)k0 * Elem<T>::bytes;
    const int rows = panel * COLS < K ? N : 0;  // (a launch of whole chunks ends with workgroups that have no columns)
    for (int n = wave * P::GROUPS + lane / P::LPR; n < rows; n += STEP * P::NL) {
        raw16 x[P::NL];
        acc_t w[P::NL];
#pragma unroll
        for (int u = 0; u < P::NL; ++u) {  // (rows behind the last one: loaded again, not counted)
            const int row = min(n + u * STEP, N - 1);
            x[u] = ld16u<T>(base + (int64_t)row * ldb * Elem<T>::bytes);
            if constexpr (W) w[u] = wvec ? wvec[row] : (acc_t)(row + 1);
        }
#pragma unroll
        for (int u = 0; u < P::NL; ++u) {
            if (n + u * STEP >= N) break;
            acc_t v[V];
            Unpack<T>::run(x[u], v);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sum[e] += v[e];
                if constexpr (W) sum2[e] = fma(w[u], v[e], sum2[e]);
                mx[e] = fmax(mx[e], v[e]);
                mn[e] = fmin(mn[e], v[e]);
            }
        }
    }
    const auto add = [](acc_t a, acc_t b) { return a + b; };
    over_rows<V, P::LPR>(sum, add);
    over_rows<V, P::LPR>(mx, [](acc_t a, acc_t b) { return fmax(a, b); });
    over_rows<V, P::LPR>(mn, [](acc_t a, acc_t b) { return fmin(a, b); });
    if constexpr (W) over_rows<V, P::LPR>(sum2, add);
    if (lane % 16 < P::LPR) {
        const int at = cl * V + panel_first<V>(lane);
#pragma unroll
        for (int e = 0; e < (V + 3) / 4; ++e) {
            red[wave][0][at + e] = sum[e];
            red[wave][1][at + e] = mx[e];
            red[wave][2][at + e] = mn[e];
            if constexpr (W) red[wave][3][at + e] = sum2[e];
        }
    }
    __syncthreads();
    if (tid < COLS) {  // (within the first wavefront) the wavefronts', sums in pairs and those in pairs: one after the other,
                       // rounding errors of 2500 rows of FP16 were 1.06 2^-24 sqrt(rows); in two launches, by slabs, 0.84
        const int at = tid / V * V, first = panel * COLS + at, k = min(first, K - V) + tid % V;
        acc_t v[4] = {0, -type_max<acc_t>(), type_max<acc_t>(), 0};
#pragma unroll
        for (int q = 0; q < PANEL_WAVES; q += 4) {
            const auto four = [&](int i) { return (red[q][i][tid] + red[q + 1][i][tid]) + (red[q + 2][i][tid] + red[q + 3][i][tid]); };
            v[0] += four(0);
            if constexpr (W) v[3] += four(3);
#pragma unroll
            for (int j = q; j < q + 4; ++j) {
                v[1] = fmax(v[1], red[j][1][tid]);
                v[2] = fmin(v[2], red[j][2][tid]);
            }
        }
        const bool own = k >= first && k < K;  // (not the columns that a lane moved back shares with the one before it)
        if (own) out.column(k, N, v[0], v[1], v[2], v[3]);
        if constexpr (Out::AGGREGATES) {
            double t1, t2, t3;
            row_terms(v[0], v[1], v[2], N, t1, t2, t3);
            if (own) {
                terms[k - panel * COLS][0] = t1;
                terms[k - panel * COLS][1] = t2;
                terms[k - panel * COLS][2] = t3;
            }
        }
    }
    if constexpr (Out::AGGREGATES) {
        __syncthreads();
        // S1..S3: 16 columns in order, as the combining step above leaves them
        double s[3] = {0, 0, 0};
        const int entry = panel * (COLS / 16) + tid;
        const bool leaves = tid < COLS / 16 && entry * 16 < K;
        if (leaves)
#pragma unroll
            for (int c = 0; c < 16; ++c)
#pragma unroll
                for (int q = 0; q < 3; ++q) s[q] += terms[tid * 16 + c][q];
        publish_entry_and_fold_S(leaves, entry, (K + 15) / 16, s[0], s[1], s[2], out.s_partial, out.ticket, out.S);
    }
}

// ---------------------------------------------------------------------------
// A side: one wavefront per row m: (max, min, mean), dot with Be, threshold
// ---------------------------------------------------------------------------
// W: also the expected weighted checksum C^{r2} = A (B r2) (section 2.2).
// THR_NL: 16-byte pieces of the row in flight per lane.  Rows of 1024 pieces or more run 4 (30.0 against 31.8 us
// at 8192 x 8192 FP16), shorter ones 2 (8.8 against 9.5 us at 4096 x 4096 BF16).
template <typename T, bool W, int THR_NL>
__global__ __launch_bounds__(256) void threshold_rows_kernel(const void* __restrict__ A, int M, int K, int N,
                                                             int64_t lda,
                                                             const typename Elem<T>::acc_t* __restrict__ Be,
                                                             const typename Elem<T>::acc_t* __restrict__ Be2,
                                                             const double* __restrict__ S, double e_max,
                                                             double c_sigma,
                                                             typename Elem<T>::acc_t* __restrict__ astat,
                                                             typename Elem<T>::acc_t* __restrict__ expected,
                                                             typename Elem<T>::acc_t* __restrict__ expected2,
                                                             typename Elem<T>::acc_t* __restrict__ Tout) {
    using acc_t = typename Elem<T>::acc_t;
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= M) return;
    const char* row = reinterpret_cast<const char*>(A) + (int64_t)m * lda * Elem<T>::bytes;
    const double S1 = S[0], S2 = S[1], S3 = S[2];  // (ahead of the row: not one more round trip behind it)
    const RowSums<acc_t> r = row_sums<T, W, THR_NL>(row, K, lane, Be, Be2);
    if (lane == 0) {
        double mu;
        const double t = row_threshold(r, K, N, S1, S2, S3, e_max, c_sigma, mu);
        if constexpr (W) expected2[m] = r.dot2;
        astat[3 * (int64_t)m + 0] = r.mx;
        astat[3 * (int64_t)m + 1] = r.mn;
        astat[3 * (int64_t)m + 2] = (acc_t)mu;
        expected[m] = r.dot;
        Tout[m] = (acc_t)t;
    }
}

// ---------------------------------------------------------------------------
// Offline check (section 3.6 "Offline ABFT"): row sums of the product as it sits in memory after
// quantisation to the output type, compared with the expected checksum.  One wavefront per row.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void check_offline_kernel(const void* __restrict__ C, int M, int N, int64_t ldc,
                                                            const typename Elem<T>::acc_t* __restrict__ expected,
                                                            const typename Elem<T>::acc_t* __restrict__ Tthr,
                                                            typename Elem<T>::acc_t* __restrict__ rowsum,
                                                            typename Elem<T>::acc_t* __restrict__ E,
                                                            int32_t* __restrict__ flags, int32_t* __restrict__ nflag) {
    using acc_t = typename Elem<T>::acc_t;
    constexpr int V = Elem<T>::vec;
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= M) return;
    const char* row = reinterpret_cast<const char*>(C) + (int64_t)m * ldc * Elem<T>::bytes;
    acc_t part[4] = {0, 0, 0, 0};
    int done = 0;
    {
        const int nchunks = N / V;
        int c = lane;
        for (; c + 192 < nchunks; c += 256) {
            raw16 r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = ld16u<T>(row + (int64_t)(c + 64 * u) * 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc_t v[V];
                Unpack<T>::run(r[u], v);
                acc_t cs = 0;
#pragma unroll
                for (int e = 0; e < V; ++e) cs += v[e];
                part[u] += cs;
            }
        }
        for (; c < nchunks; c += 64) {
            acc_t v[V];
            Unpack<T>::run(ld16u<T>(row + (int64_t)c * 16), v);
#pragma unroll
            for (int e = 0; e < V; ++e) part[0] += v[e];
        }
        done = nchunks * V;
    }
    for (int n = done + lane; n < N; n += 64) part[1] += Unpack<T>::one(row, n);
    const acc_t s = wave_sum((part[0] + part[1]) + (part[2] + part[3]));
    if (lane == 0) {
        const acc_t e = expected[m] - s;
        const int f = !(fabs(e) <= Tthr[m]);
        rowsum[m] = s;
        E[m] = e;
        flags[m] = f;
        if (f) atomicAdd(nflag, 1);
    }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------

// Rows per block of the column reduction over a (rows x cols) row-major matrix: 128 or 64.  Smaller slabs put more
// loads in flight, and every halving doubles the slab partials the finishing kernel folds.  Measured (two launches,
// N x K layouts): 8192 x 8192 FP16 42.2 us with 128-row slabs, 33.3 with 64-row slabs and eight rows in flight per
// wavefront; 4096 x 4096 FP32 23.3 -> 17.2; 11008 x 4096 BF16 (172 slabs of 64 rows) 23.0 -> 28.2, hence the
// limit on the row count; below 64 rows the fold costs more than the slabs bring.
static int col_rows_per_block(int dtype, int64_t rows, int64_t cols) {
    const int64_t v = dtype == VABFT_F64 ? 2 : dtype == VABFT_F32 ? 4 : (dtype == VABFT_F8E4M3 || dtype == VABFT_F8E5M2) ? 16 : 8;
    const int64_t xblocks = (cols + 64 * v - 1) / (64 * v);
    const int64_t blocks128 = xblocks * ((rows + 127) / 128);
    return (blocks128 < 512 || (blocks128 < 2048 && rows <= 8192)) ? 64 : 128;
}

// Rows k per block of the finishing kernel: 16, or fewer (K x N layout) where 16 would leave most of the
// chip's 256 compute units without a block and a wavefront with more than 4 KiB of a row.  (Rows of up to 4 KiB are
// one batch of loads for one wavefront: splitting them only adds arrivals, 11 ns each on one address, to the fold.)
static int encode_rows_per_block(const vabft_problem* p, int waves) {
    if (p->transB) return 16;
    const int64_t eb = p->dtype == VABFT_F64 ? 8 : p->dtype == VABFT_F32 ? 4 : (p->dtype == VABFT_F8E4M3 || p->dtype == VABFT_F8E5M2) ? 1 : 2;
    int rpb = waves;
    while (rpb > 1 && (p->K + rpb - 1) / rpb < 256 && p->N * eb * rpb > 4096 * waves) rpb >>= 1;
    // (4 KiB of FP8 are twice the arithmetic: half of that, where the arrivals stay few.  512 x 8000 deferred 5.7 against 3.8
    // us, weighted 10.2 / 7.2; with more blocks, 2000 x 4096, 7.4 against 8.3)
    if (eb == 1)
        while (rpb > 1 && (p->K + rpb / 2 - 1) / (rpb / 2) <= 128 && p->N * eb * rpb > 2048 * waves) rpb >>= 1;
    return rpb;
}
constexpr int ENC_WAVES_OWN_FOLD = 16, ENC_WAVES_DEFERRED = 8;
// Wavefronts per workgroup of the row walk.  The smaller workgroup is only used for many rows, where both sizes give
// one wavefront per row: with several wavefronts per row the split of a row into segments (and with it
// the rounding of Be) would depend on the workgroup size, and both routes must produce the same bits.
static int encode_rows_waves(const vabft_problem* p, bool deferred) {
    if (deferred && p->K > 255 * ENC_WAVES_OWN_FOLD) return ENC_WAVES_DEFERRED;
    return ENC_WAVES_OWN_FOLD;
}
// Per-block partials of (S1, S2, S3), [blocks][3] doubles: the number an encode with the fold deferred leaves
// (what the fused GEMM folds, and what the workspace reserves; an encode that folds them itself leaves no more)
int s_partial_count(const vabft_problem* p) {
    const int rpb = encode_rows_per_block(p, encode_rows_waves(p, true));
    return (p->K + rpb - 1) / rpb;
}

size_t encode_workspace_bytes(const vabft_problem* p) {
    size_t bytes = 0;
    if (p->transB) {
        const size_t acc_bytes = p->dtype == VABFT_F64 ? 8 : 4;
        const size_t rpb = col_rows_per_block(p->dtype, p->N, p->K);
        const size_t nsplit = ((size_t)p->N + rpb - 1) / rpb;
        bytes += nsplit * 4 * (size_t)p->K * acc_bytes;  // (sum, max, min, weighted sum) per slab
    }
    return bytes;
}

// Column reductions of rows x cols: in one launch (panel_kernel) or two.  A workgroup's time grows with the rows, the launch's
// with both; workgroups behind the first 256, on few of the compute units, take a second one's time.  Two launches / one (us,
// columns x rows): BF16 96 x 64 8.1 / 5.4, 1536 x 1024 9.2 / 6.9, 4096 x 4096 16.4 / 12.1, but 96 x 11008 11.2 / 14.7, 5000 x
// 5000 16.0 / 17.0 (fold deferred), 9342 x 6400 38.6 / 48.4; FP8 4096 x 512 12.4 / 8.0, 4096 x 4096 15.9 / 13.1, 1536 x 8192
// 13.7 / 13.7, 8661 x 4096 17.5 / 19.6; FP32 1536 x 1024 8.5 / 6.7, 4096 x 4096 19.7 / 15.3, 96 x 4096 8.3 / 8.7, 8301 x 7262
// 56 / 78, 4890 x 2902 (306 panels) 20 / 23; FP64 96 x 1024 8.1 / 6.7, 4126 x 1024 (258 panels) 15.2 / 17.8.  600 problems of up
// to 12000 x 11264 take 0.82 (BF16), 0.76 (FP8), 0.90 and 0.91 (FP64) of the time of two launches, six of them longer.
// (With the matrix in a cache.  From memory rows at a pitch of whole 512 bytes meet in the same channels, and of a row a panel has
// 16 to 64 bytes.  One launch in times of two, own fold and deferred, from memory / in a cache: BF16 1024 x 3072 1.18 and 1.29 / 0.87
// and 0.83, 1536 x 3584 1.27 and 1.44 / 0.86 and 0.84, 2560 x 4096 1.26 and 1.45 / 0.82 and 0.77, but 4096 x 4096 1.00 and 1.13 / 0.74
// and 0.65; FP8 2048 x 5120 1.23 and 1.34 / 0.89 and 0.87, x 4096 1.10 and 1.23 / 0.86 and 0.84; FP32 1536 x 2560 1.15 and 1.28 / 0.85
// and 0.83, x 2048 1.06 and 1.19 / 0.85 and 0.81.  Both folds take the same launches, for the same bits: one where the four gain
// together.  At other pitches they do up to the lines for a cache: BF16 4080 x 4096 0.85 and 0.80 from memory.)
template <typename T> static bool panel_pays(int64_t cols, int64_t rows, int64_t ld) {
    constexpr int V = Elem<T>::vec;
    int64_t most = V == 4 ? 2048 + cols * 3 / 5 : 1024 + cols * 3 / 5;
    if (V == 8) most = cols <= 4096 ? 2560 + cols * 7 / 10 : 3072;
    if (V == 16) most = cols <= 4096 ? 4096 + cols * 4 / 5 : std::min<int64_t>(2048 + cols * 3 / 5, 5000);
    if (V >= 4 && ld * Elem<T>::bytes >= 1536 && ld * Elem<T>::bytes % 512 == 0) {
        const int64_t least = V == 4 ? 2048 : V == 8 ? 2560 : 4096, more = V == 4 ? 512 : V == 8 ? 1024 : 1536;
        most = std::min(most, std::max(least, more + cols));
    }
    if (cols > 8192) most = V >= 8 ? 1024 : 256;
    const int64_t panels = (cols - 1) / Panel<T, V == 2 ? 8 : 4>::COLS + 1, rounds = (panels + 255) / 256;
    const bool tail = rounds > 1 && 5 * 256 * rounds > (V == 2 ? 6 : 7) * panels && rows > 256;
    const bool large = rounds > 1 && (double)cols * (double)rows * Elem<T>::bytes > (V >= 8 ? 72e6 : 60e6);
    return cols >= V && !tail && !large && rows <= most;
}
template <typename T, bool W, typename Out>
static void panel_launch(const void* src, int cols, int rows, int64_t ld, const Out& out, hipStream_t st) {
    const auto launch = [&](auto lpr) {
        constexpr int LPR = decltype(lpr)::value;
        // (whole chunks of the workgroups' order, so that all panels of a line have their XCD, where there is much to read:
        // FP8 1536 x 5000 11.9 us against 9.0)
        const unsigned panels = (unsigned)((cols - 1) / Panel<T, LPR>::COLS + 1), chunk = 8 * 128 / (16 * LPR);
        const unsigned blocks = rows >= 1024 ? (panels + chunk - 1) / chunk * chunk : panels;
        panel_kernel<T, W, LPR, Out><<<dim3(blocks), dim3(64 * PANEL_WAVES), 0, st>>>(src, cols, rows, ld, out);
    };
    // 16-bit and FP8: half as wide for long columns, where the chip holds all panels at once (32 bytes of a row against 64:
    // BF16 1536 x 4096 9.7 against 12.5, 4096 x 512 8.4 / 7.2, 8192 x 4096 20.6 / 16.2; FP8 4096 x 2048 10.8 / 13.0, x 64
    // 8.0 / 7.0); FP8, with the most arithmetic to a byte, a quarter (16 bytes: 4096 x 4096 9.2 against 11.0 with the fold
    // deferred; but 4096 columns of 2048, with a fold of its own, 11.3 / 10.6)
    if constexpr (Elem<T>::vec == 16) {
        if (cols <= 256 * Panel<T, 1>::COLS && rows >= std::max(1024, cols / 4 * 3)) return launch(std::integral_constant<int, 1>());
    }
    if constexpr (Elem<T>::vec >= 8) {
        constexpr bool fp8 = Elem<T>::vec == 16;
        if (cols <= 256 * Panel<T, 2>::COLS && rows >= (fp8 ? std::max(256, cols / 6) : std::max(384, cols / 2)))
            return launch(std::integral_constant<int, 2>());
    }
    launch(std::integral_constant<int, Elem<T>::vec == 2 ? 8 : 4>());
}

template <typename T, bool W>
static int encode_launch(const vabft_problem* p, const void* dB, void* d_Be, void* d_Be2, void* d_bstat, double* d_S,
                         double* s_partial, void* ws, int32_t* ticket, hipStream_t st) {
    using acc_t = typename Elem<T>::acc_t;
    if (!p->transB) {
        const int waves = encode_rows_waves(p, d_S == nullptr);
        const int rpb = encode_rows_per_block(p, waves);
        const int kblocks = (p->K + rpb - 1) / rpb;
#define VABFT_ENC_ROWS(R, WV)                                                                                    \
    if constexpr (R <= WV)                                                                                       \
        encode_rows_kernel<T, W, R, WV><<<dim3(kblocks), dim3(64 * WV), 0, st>>>(                                \
            dB, p->K, p->N, p->ldb, (acc_t*)d_Be, (acc_t*)d_Be2, (acc_t*)d_bstat, s_partial, ticket, d_S)
#define VABFT_ENC_ROWS_SWITCH(WV)                 \
    switch (rpb) {                                \
        case 16: VABFT_ENC_ROWS(16, WV); break;   \
        case 8: VABFT_ENC_ROWS(8, WV); break;     \
        case 4: VABFT_ENC_ROWS(4, WV); break;     \
        case 2: VABFT_ENC_ROWS(2, WV); break;     \
        default: VABFT_ENC_ROWS(1, WV); break;    \
    }
        if (waves == ENC_WAVES_OWN_FOLD) {
            VABFT_ENC_ROWS_SWITCH(ENC_WAVES_OWN_FOLD)
        } else {
            VABFT_ENC_ROWS_SWITCH(ENC_WAVES_DEFERRED)
        }
#undef VABFT_ENC_ROWS_SWITCH
#undef VABFT_ENC_ROWS
    } else if (panel_pays<T>(p->K, p->N, p->ldb)) {
        const PanelEncode<acc_t> out = {(acc_t*)d_Be, (acc_t*)d_Be2, (acc_t*)d_bstat, s_partial, ticket, d_S};
        panel_launch<T, W>(dB, p->K, p->N, p->ldb, out, st);
    } else {
        constexpr int V = Elem<T>::vec;
        const int rpb = col_rows_per_block(p->dtype, p->N, p->K);
        const int nsplit = (p->N + rpb - 1) / rpb;
        acc_t* part = reinterpret_cast<acc_t*>(ws);
        dim3 grid((p->K + 64 * V - 1) / (64 * V), nsplit);
        if (rpb == 64)
            encode_cols_kernel<T, W, 8><<<grid, dim3(256), 0, st>>>(dB, p->K, p->N, p->ldb, rpb, part, nullptr);
        else
            encode_cols_kernel<T, W, 4><<<grid, dim3(256), 0, st>>>(dB, p->K, p->N, p->ldb, rpb, part, nullptr);
        const int kblocks = s_partial_count(p);
        encode_cols_combine_kernel<acc_t, W><<<dim3(kblocks), dim3(256), 0, st>>>(
            part, nsplit, p->K, p->N, (acc_t*)d_Be, (acc_t*)d_Be2, (acc_t*)d_bstat, s_partial, ticket, d_S);
    }
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

// d_Be2 == nullptr: plain encode; otherwise the weighted checksum is produced in the same pass
// d_S == nullptr: S1..S3 stay as the s_partial_count() per-workgroup partials in s_partial
// ws: scratch of encode_workspace_bytes(); ticket: one int32 that is zero between launches
int encode_dispatch(const vabft_problem* p, const void* dB, void* d_Be, void* d_Be2, void* d_bstat, double* d_S,
                    double* s_partial, void* ws, int32_t* ticket, hipStream_t st) {
#define VABFT_ENC_CASE(T)                                                                               \
    return d_Be2 ? encode_launch<T, true>(p, dB, d_Be, d_Be2, d_bstat, d_S, s_partial, ws, ticket, st) \
                 : encode_launch<T, false>(p, dB, d_Be, nullptr, d_bstat, d_S, s_partial, ws, ticket, st)
    switch (p->dtype) {
        case VABFT_F64: VABFT_ENC_CASE(double);
        case VABFT_F32: VABFT_ENC_CASE(float);
        case VABFT_F16: VABFT_ENC_CASE(f16_t);
        case VABFT_BF16: VABFT_ENC_CASE(bf16_t);
        case VABFT_F8E4M3: VABFT_ENC_CASE(f8_t);
        case VABFT_F8E5M2: VABFT_ENC_CASE(bf8_t);
    }
#undef VABFT_ENC_CASE
    return VABFT_EINVAL;
}

// Rows of a launch with a wavefront each, at most: a launch holds fewer than 2^32 threads.
constexpr int64_t ROWS_MOST = 1 << 25;

template <typename T, bool W>
static int threshold_launch(const vabft_problem* p, const void* dA, const void* d_Be, const void* d_Be2,
                            const double* d_S, double e_max, double c_sigma, void* d_astat, void* d_expected,
                            void* d_expected2, void* d_T, hipStream_t st) {
    using acc_t = typename Elem<T>::acc_t;
    for (int64_t m = 0; m < p->M; m += ROWS_MOST) {
        const int rows = (int)std::min<int64_t>(ROWS_MOST, p->M - m);
        const void* A = (const char*)dA + m * p->lda * Elem<T>::bytes;
        acc_t *astat = (acc_t*)d_astat + 3 * m, *expected = (acc_t*)d_expected + m, *Tout = (acc_t*)d_T + m;
        acc_t* expected2 = W ? (acc_t*)d_expected2 + m : nullptr;
        auto kern = p->K / Elem<T>::vec >= 1024 ? threshold_rows_kernel<T, W, 4> : threshold_rows_kernel<T, W, 2>;
        kern<<<dim3((rows + 3) / 4), dim3(256), 0, st>>>(A, rows, p->K, p->N, p->lda, (const acc_t*)d_Be,
                                                         (const acc_t*)d_Be2, d_S, e_max, c_sigma, astat, expected,
                                                         expected2, Tout);
    }
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

// d_Be2 / d_expected2 == nullptr: plain pass; otherwise A (B r2) rides in the same read of A
int threshold_dispatch(const vabft_problem* p, const void* dA, const void* d_Be, const void* d_Be2, const double* d_S,
                       double e_max, double c_sigma, void* d_astat, void* d_expected, void* d_expected2, void* d_T,
                       hipStream_t st) {
#define VABFT_THR_CASE(T)                                                                                          \
    return d_Be2 ? threshold_launch<T, true>(p, dA, d_Be, d_Be2, d_S, e_max, c_sigma, d_astat, d_expected,        \
                                             d_expected2, d_T, st)                                                 \
                 : threshold_launch<T, false>(p, dA, d_Be, nullptr, d_S, e_max, c_sigma, d_astat, d_expected,      \
                                              nullptr, d_T, st)
    switch (p->dtype) {
        case VABFT_F64: VABFT_THR_CASE(double);
        case VABFT_F32: VABFT_THR_CASE(float);
        case VABFT_F16: VABFT_THR_CASE(f16_t);
        case VABFT_BF16: VABFT_THR_CASE(bf16_t);
        case VABFT_F8E4M3: VABFT_THR_CASE(f8_t);
        case VABFT_F8E5M2: VABFT_THR_CASE(bf8_t);
    }
#undef VABFT_THR_CASE
    return VABFT_EINVAL;
}

// ---------------------------------------------------------------------------
// Column checksums (section 2.2: c1 = [1 .. 1], A^c = [A; c1 A], C^{c1} = c1 A B).  By the symmetry
// C^T = B^T A^T the column check is Algorithm 1 with the roles exchanged: column j of B (K entries) plays
// the row of A, column k of A (M entries) plays the row of B, and M replaces N.
// ---------------------------------------------------------------------------

// Column threshold and expected column checksum from (sum, max, min, dot with c1 A) of a column of B
template <typename acc_t> struct PanelThreshold {
    const acc_t* eA;
    const double* SA;
    int M;
    double e_max, c_sigma;
    acc_t* colstat;
    acc_t* expected_col;
    acc_t* Tcol;
    static constexpr bool AGGREGATES = false;
    __device__ const acc_t* weights() const { return eA; }
    __device__ void column(int n, int K, acc_t sum, acc_t mx, acc_t mn, acc_t dot) const {
        const double mu = (double)sum / (double)K;
        double var = ((double)mx - mu) * (mu - (double)mn);
        var = var > 0 ? var : 0;
        const double S1 = SA[0], S2 = SA[1], S3 = SA[2], dM = (double)M;
        const double t_det = dM * fabs(mu) * S1;
        const double t_var23 = c_sigma * sqrt(dM * mu * mu * S2 + dM * dM * var * S3);
        const double t_var4 = c_sigma * sqrt(dM) * sqrt(var) * sqrt(S2);
        colstat[3 * (int64_t)n + 0] = mx;
        colstat[3 * (int64_t)n + 1] = mn;
        colstat[3 * (int64_t)n + 2] = (acc_t)mu;
        expected_col[n] = dot;
        Tcol[n] = (acc_t)(e_max * (t_det + t_var23 + t_var4));
    }
};

// Per column n of a K x N row-major B: fold the row-slab partials (sum, max, min, dot with c1 A) in slab
// order and evaluate the column threshold.
template <typename acc_t>
__global__ __launch_bounds__(256) void threshold_cols_finish_kernel(const acc_t* __restrict__ part, int nsplit,
                                                                    int N, int K, int M, const double* __restrict__ SA,
                                                                    double e_max, double c_sigma,
                                                                    acc_t* __restrict__ colstat,
                                                                    acc_t* __restrict__ expected_col,
                                                                    acc_t* __restrict__ Tcol) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= N) return;
    acc_t sum = 0, dot = 0, mx = -type_max<acc_t>(), mn = type_max<acc_t>();
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        // eight slabs' loads in flight at once; folded in slab order
        acc_t v[8][4];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int sc = s0 + u < nsplit ? s0 + u : nsplit - 1;
            const acc_t* q = part + (int64_t)sc * 4 * N;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[u][c] = q[c * (int64_t)N + n];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (s0 + u < nsplit) {
                sum += v[u][0];
                mx = fmax(mx, v[u][1]);
                mn = fmin(mn, v[u][2]);
                dot += v[u][3];
            }
    }
    const PanelThreshold<acc_t> out = {nullptr, SA, M, e_max, c_sigma, colstat, expected_col, Tcol};
    out.column(n, K, sum, mx, mn, dot);
}

static vabft_problem swapped_problem(const vabft_problem* p, int32_t M, int32_t N, int32_t transB, int64_t lda,
                                     int64_t ldb) {
    vabft_problem q = *p;
    q.M = M;
    q.N = N;
    q.transB = transB;
    q.lda = lda;
    q.ldb = ldb;
    return q;
}

// scratch of the two column-side passes: encode of A as an (M rows) x (K columns) "weight layout" matrix, and
// the slab partials of the column reduction over a K x N B
size_t cols_workspace_bytes(const vabft_problem* p) {
    const vabft_problem qa = swapped_problem(p, p->M, p->M, 1, p->lda, p->lda);
    const size_t a = encode_workspace_bytes(&qa);
    const size_t acc_bytes = p->dtype == VABFT_F64 ? 8 : 4;
    const size_t rpb = col_rows_per_block(p->dtype, p->K, p->N);
    const size_t nsplit = ((size_t)p->K + rpb - 1) / rpb;
    const size_t b = p->transB ? 0 : nsplit * 4 * (size_t)p->N * acc_bytes;
    return a > b ? a : b;
}

// c1 A, column statistics of A and their aggregates: the encode of the N x K layout applied to A (M x K)
int encode_a_dispatch(const vabft_problem* p, const void* dA, void* d_eA, void* d_acolstat, double* d_SA,
                      double* s_partial, void* ws, int32_t* ticket, hipStream_t st) {
    const vabft_problem q = swapped_problem(p, p->M, p->M, 1, p->lda, p->lda);
    return encode_dispatch(&q, dA, d_eA, nullptr, d_acolstat, d_SA, s_partial, ws, ticket, st);
}

template <typename T>
static int threshold_cols_launch(const vabft_problem* p, const void* dB, const void* d_eA, const double* d_SA,
                                 double e_max, double c_sigma, void* d_bcolstat, void* d_expected_col, void* d_Tcol,
                                 void* ws, hipStream_t st) {
    using acc_t = typename Elem<T>::acc_t;
    constexpr int V = Elem<T>::vec;
    if (panel_pays<T>(p->N, p->K, p->ldb)) {
        const PanelThreshold<acc_t> out = {(const acc_t*)d_eA, d_SA, p->M, e_max, c_sigma, (acc_t*)d_bcolstat,
                                           (acc_t*)d_expected_col, (acc_t*)d_Tcol};
        panel_launch<T, true>(dB, p->N, p->K, p->ldb, out, st);
        return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
    }
    const int rpb = col_rows_per_block(p->dtype, p->K, p->N);
    const int nsplit = (p->K + rpb - 1) / rpb;
    acc_t* part = reinterpret_cast<acc_t*>(ws);
    dim3 grid((p->N + 64 * V - 1) / (64 * V), nsplit);
    // rows of the reduction = k (K of them), columns = n (N of them), weight of row k = (c1 A)[k]
    encode_cols_kernel<T, true, 4><<<grid, dim3(256), 0, st>>>(dB, p->N, p->K, p->ldb, rpb, part,
                                                            (const acc_t*)d_eA);
    threshold_cols_finish_kernel<acc_t><<<dim3((p->N + 255) / 256), dim3(256), 0, st>>>(
        part, nsplit, p->N, p->K, p->M, d_SA, e_max, c_sigma, (acc_t*)d_bcolstat, (acc_t*)d_expected_col,
        (acc_t*)d_Tcol);
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

int threshold_cols_dispatch(const vabft_problem* p, const void* dB, const void* d_eA, const double* d_SA, double e_max,
                            double c_sigma, void* d_bcolstat, void* d_expected_col, void* d_Tcol, void* ws,
                            hipStream_t st) {
    if (p->transB) {
        // B stored N x K: its rows are the columns of the logical B, so this is the row pass with M := N, N := M
        const vabft_problem q = swapped_problem(p, p->N, p->M, 0, p->ldb, p->ldb);
        return threshold_dispatch(&q, dB, d_eA, nullptr, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, nullptr,
                                  d_Tcol, st);
    }
    switch (p->dtype) {
        case VABFT_F64:
            return threshold_cols_launch<double>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                                 ws, st);
        case VABFT_F32:
            return threshold_cols_launch<float>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                                ws, st);
        case VABFT_F16:
            return threshold_cols_launch<f16_t>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                                ws, st);
        case VABFT_BF16:
            return threshold_cols_launch<bf16_t>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                                 ws, st);
        case VABFT_F8E4M3:
            return threshold_cols_launch<f8_t>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                               ws, st);
        case VABFT_F8E5M2:
            return threshold_cols_launch<bf8_t>(p, dB, d_eA, d_SA, e_max, c_sigma, d_bcolstat, d_expected_col, d_Tcol,
                                                ws, st);
    }
    return VABFT_EINVAL;
}

int check_offline_dispatch(const vabft_problem* p, const void* dC, const void* d_expected, const void* d_T,
                           void* d_rowsum, void* d_E, int32_t* d_flags, int32_t* d_nflag, hipStream_t st) {
#define VABFT_OFF_CASE(T)                                                                                           \
    {                                                                                                               \
        using acc_t = typename Elem<T>::acc_t;                                                                      \
        for (int64_t m = 0; m < p->M; m += ROWS_MOST) {                                                             \
            const int rows = (int)std::min<int64_t>(ROWS_MOST, p->M - m);                                           \
            check_offline_kernel<T><<<dim3((rows + 3) / 4), dim3(256), 0, st>>>(                                    \
                (const char*)dC + m * p->ldc * Elem<T>::bytes, rows, p->N, p->ldc, (const acc_t*)d_expected + m,    \
                (const acc_t*)d_T + m, (acc_t*)d_rowsum + m, (acc_t*)d_E + m, d_flags + m, d_nflag);                \
        }                                                                                                           \
        break;                                                                                                      \
    }
    switch (p->dtype) {
        case VABFT_F64: VABFT_OFF_CASE(double)
        case VABFT_F32: VABFT_OFF_CASE(float)
        case VABFT_F16: VABFT_OFF_CASE(f16_t)
        case VABFT_F8E4M3:
        case VABFT_F8E5M2: VABFT_OFF_CASE(f16_t)  // the stored product of an FP8 problem is FP16
        case VABFT_BF16: VABFT_OFF_CASE(bf16_t)
        default: return VABFT_EINVAL;
    }
#undef VABFT_OFF_CASE
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

}  // namespace vabft
