// One row of A per wavefront: (sum, max, min), dot product with Be (and Be2), and the threshold T_m of Algorithm 1
// (section 3.4 boxed formula).  Shared by the streaming pass over A and by the GEMM launches that carry that pass in
// workgroups of their own.
#pragma once
#include <type_traits>

#include "unpack.h"

namespace vabft {

template <typename acc_t> struct RowSums {
    acc_t sum, dot, dot2, mx, mn;
};

// W: also the dot product with Be2.  NL: 16-byte pieces of the row in flight per lane.  LW: lanes per row (lane is the
// number among them), 64 or, for rows of that many pieces at most, fewer: the same bits, as what the other lanes would add
// is zero.  The pieces need no alignment beyond the element's.  sink(c, piece) is handed every whole piece.
struct NoSink {
    __device__ __forceinline__ void operator()(int, const raw16&) const {}
};
template <typename T, bool W, int NL, int LW = WAVE, typename SINK = NoSink>
__device__ __forceinline__ RowSums<typename Elem<T>::acc_t> row_sums(const char* row, int K, int lane,
                                                                     const typename Elem<T>::acc_t* __restrict__ Be,
                                                                     const typename Elem<T>::acc_t* __restrict__ Be2,
                                                                     SINK sink = SINK{}) {
    using acc_t = typename Elem<T>::acc_t;
    constexpr int V = Elem<T>::vec;
    acc_t sum = 0, dot = 0, dot2 = 0, mx = -type_max<acc_t>(), mn = type_max<acc_t>();
    const int nchunks = K / V;
    int c = lane;
    // the matching pieces of Be come from the caches
    for (; c + LW * (NL - 1) < nchunks; c += LW * NL) {
        raw16 r[NL];
#pragma unroll
        for (int u = 0; u < NL; ++u) r[u] = ld16u<T>(row + (int64_t)(c + LW * u) * 16);
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            acc_t v[V], b[V];
#pragma unroll
            for (int e = 0; e < V; ++e) b[e] = Be[(int64_t)(c + LW * u) * V + e];
            sink(c + LW * u, r[u]);
            Unpack<T>::run(r[u], v);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sum += v[e];
                dot = fma(v[e], b[e], dot);
                if constexpr (W) dot2 = fma(v[e], Be2[(int64_t)(c + LW * u) * V + e], dot2);
                mx = fmax(mx, v[e]);
                mn = fmin(mn, v[e]);
            }
        }
    }
    for (; c < nchunks; c += LW) {
        raw16 r0 = ld16u<T>(row + (int64_t)c * 16);
        acc_t v0[V];
        sink(c, r0);
        Unpack<T>::run(r0, v0);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const acc_t b = Be[(int64_t)c * V + e];
            sum += v0[e];
            dot = fma(v0[e], b, dot);
            if constexpr (W) dot2 = fma(v0[e], Be2[(int64_t)c * V + e], dot2);
            mx = fmax(mx, v0[e]);
            mn = fmin(mn, v0[e]);
        }
    }
    for (int k = nchunks * V + lane; k < K; k += LW) {
        acc_t x = Unpack<T>::one(row, k);
        sum += x;
        dot = fma(x, Be[k], dot);
        if constexpr (W) dot2 = fma(x, Be2[k], dot2);
        mx = fmax(mx, x);
        mn = fmin(mn, x);
    }
    RowSums<acc_t> o;
    o.sum = group_sum<LW>(sum);
    o.dot = group_sum<LW>(dot);
    o.dot2 = W ? group_sum<LW>(dot2) : (acc_t)0;
    o.mx = group_max<LW>(mx);
    o.mn = group_min<LW>(mn);
    return o;
}

// T_m in double precision from the row's (sum, max, min) and S1, S2, S3; mu receives the mean
template <typename acc_t>
__device__ __forceinline__ double row_threshold(const RowSums<acc_t>& r, int K, int N, double S1, double S2, double S3,
                                                double e_max, double c_sigma, double& mu) {
    mu = (double)r.sum / (double)K;
    double var = ((double)r.mx - mu) * (mu - (double)r.mn);
    var = var > 0 ? var : 0;
    const double dN = (double)N;
    const double t_det = dN * fabs(mu) * S1;
    const double t_var23 = c_sigma * sqrt(dN * mu * mu * S2 + dN * dN * var * S3);
    // c sqrt(N) sigma_A sqrt(S2).  What FP32 sums can hold stays far from the ends of FP64's range, so one root does; FP64
    // data may not (below 1e-81 var * S2 is zero), so its factors keep roots of their own.
    const double t_var4 = std::is_same<acc_t, double>::value ? c_sigma * sqrt(dN) * sqrt(var) * sqrt(S2)
                                                             : c_sigma * sqrt(dN * var * S2);
    return e_max * (t_det + t_var23 + t_var4);
}

}  // namespace vabft
