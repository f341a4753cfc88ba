// Operands whose rows the tiled kernels cannot read -- at odd addresses, of a length that is no multiple of 16 bytes, FP8 of
// any size but whole tiles -- laid out once for the GEMM behind: 16-bit elements (FP8 as FP16: exact), rows of whole 128-byte
// lines, zeros behind their end.  What is read is a wavefront's pieces of 16 bytes in a row wherever they start; what is
// written is aligned.  Bound by memory, and at a few MB by the launch: 1021 x 2047 and 2047 x 1531 BF16 4.4 us.  The direct
// kernels read each such piece as two lines, once per tile: BF16 3708 x 1873 x 10496 352 us, with this pass and the tiled
// kernel 151.
//
// With the A-side pass fused the rows of A, copied or not, give their statistics, expected checksum and threshold on the way
// (row_threshold.h, the same bits as the pass by itself).
#include "row_threshold.h"
#include "vabft_host.h"

namespace vabft {

struct PackStats {  // the A-side pass; Be null: none
    const float* Be;
    double* S;  // with s_nparts > 0 an output, or null: the sums are folded from s_partial[s_nparts][3]
    const double* s_partial;
    int32_t s_nparts, N;
    double e_max, c_sigma;
    float *astat, *expected, *T;
};

template <typename T> __device__ __forceinline__ void store_piece(raw16* dst, int c, const raw16& r) {
    if constexpr (Elem<T>::bytes == 2) {
        dst[c] = r;
    } else {
        dst[2 * c] = raw16{{widen2<T>(r.w[0], false), widen2<T>(r.w[0], true), widen2<T>(r.w[1], false), widen2<T>(r.w[1], true)}};
        dst[2 * c + 1] = raw16{{widen2<T>(r.w[2], false), widen2<T>(r.w[2], true), widen2<T>(r.w[3], false), widen2<T>(r.w[3], true)}};
    }
}
template <typename T> __device__ __forceinline__ uint16_t element16(const char* row, int k) {
    if constexpr (Elem<T>::bytes == 2)
        return reinterpret_cast<const uint16_t*>(row)[k];
    else
        return (uint16_t)widen2<T>(reinterpret_cast<const uint8_t*>(row)[k], false);
}

// one row by LW lanes (rows behind the matrix's last one are zeros)
template <typename T, int LW, bool STATS>
__device__ __forceinline__ void pack_row(const PackArgs& p, int row, const PackStats& q, double S1, double S2, double S3) {
    constexpr int V = Elem<T>::vec, NL = 4;
    const int lane = threadIdx.x % LW;
    if (row >= p.rows_out) {
        if (!STATS) return;  // (the exchanges of the statistics need every lane)
        row = p.rows_out - 1;
    }
    const int len = row < p.rows ? p.len : 0, nchunks = len / V;
    const char* src = reinterpret_cast<const char*>(p.src) + (int64_t)(row < p.rows ? row : 0) * p.ld * Elem<T>::bytes;
    uint16_t* const dst = reinterpret_cast<uint16_t*>(p.dst) + (int64_t)row * p.pitch;
    raw16* const out = reinterpret_cast<raw16*>(dst);
    const bool copy = p.dst != nullptr;
    if constexpr (STATS) {
        const RowSums<float> r = row_sums<T, false, NL, LW>(src, len, lane, q.Be, nullptr,
                                                            [&](int c, const raw16& x) {
                                                                if (copy) store_piece<T>(out, c, x);
                                                            });
        if (lane == 0) {
            double mu;
            const double t = row_threshold(r, len, q.N, S1, S2, S3, q.e_max, q.c_sigma, mu);
            q.astat[3 * (int64_t)row + 0] = r.mx;
            q.astat[3 * (int64_t)row + 1] = r.mn;
            q.astat[3 * (int64_t)row + 2] = (float)mu;
            q.expected[row] = r.dot;
            q.T[row] = (float)t;
        }
    } else {
        int c = lane;
        for (; c + LW * (NL - 1) < nchunks; c += LW * NL) {
            raw16 r[NL];
#pragma unroll
            for (int u = 0; u < NL; ++u) r[u] = ld16u<T>(src + (int64_t)(c + LW * u) * 16);
#pragma unroll
            for (int u = 0; u < NL; ++u) store_piece<T>(out, c + LW * u, r[u]);
        }
        for (; c < nchunks; c += LW) store_piece<T>(out, c, ld16u<T>(src + (int64_t)c * 16));
    }
    if (!copy) return;
    // the elements behind the last whole piece, zeros up to the next 16 bytes, and zeros to the end
    const int whole = nchunks * V, stop = (len + 7) / 8 * 8;
    for (int k = whole + lane; k < stop; k += LW) dst[k] = k < len ? element16<T>(src, k) : (uint16_t)0;
    for (int c = stop / 8 + lane; c < p.pitch / 8; c += LW) out[c] = raw16{{0u, 0u, 0u, 0u}};
}

template <typename T, bool STATS>
__device__ __forceinline__ void pack_rows(const PackArgs& p, int block, const PackStats& q, double S1, double S2, double S3) {
    const int first = block * p.block_rows;
    if (p.block_rows == 4)
        pack_row<T, 64, STATS>(p, first + threadIdx.x / 64, q, S1, S2, S3);
    else if (p.block_rows == 8)
        pack_row<T, 32, STATS>(p, first + threadIdx.x / 32, q, S1, S2, S3);
    else
        pack_row<T, 16, STATS>(p, first + threadIdx.x / 16, q, S1, S2, S3);
}

template <typename T> __global__ __launch_bounds__(256) void pack_kernel(const PackArgs a, const PackArgs b, const PackStats q) {
    __shared__ double s_red[12];
    if ((int)blockIdx.x >= a.blocks) {
        pack_rows<T, false>(b, blockIdx.x - a.blocks, q, 0, 0, 0);
    } else if (q.Be) {
        const bool fold = q.s_nparts != 0;
        if (fold) {
            fold_s_partials_to_lds(q.s_partial, q.s_nparts, threadIdx.x, s_red);
            __syncthreads();
            if (blockIdx.x == 0 && threadIdx.x < 3 && q.S) q.S[threadIdx.x] = folded_s(s_red, threadIdx.x);
        }
        const double S1 = fold ? folded_s(s_red, 0) : q.S[0], S2 = fold ? folded_s(s_red, 1) : q.S[1],
                     S3 = fold ? folded_s(s_red, 2) : q.S[2];
        pack_rows<T, true>(a, blockIdx.x, q, S1, S2, S3);
    } else {
        pack_rows<T, false>(a, blockIdx.x, q, 0, 0, 0);
    }
}

// (rows of up to 16 or 32 pieces share a wavefront)
static PackArgs with_blocks(PackArgs p, int eb, bool read) {
    const int pieces = p.len * eb / 16;
    p.block_rows = pieces <= 16 ? 16 : pieces <= 32 ? 8 : 4;
    p.blocks = p.dst || read ? (p.rows_out + p.block_rows - 1) / p.block_rows : 0;
    return p;
}

int pack_dispatch(int dtype, const PackArgs& a0, const PackArgs& b0, const FusedArgs* fused, const double* s_partial,
                  int s_nparts, int N, void* d_expected, void* d_T, hipStream_t st) {
    const int eb = dtype == VABFT_F8E4M3 || dtype == VABFT_F8E5M2 ? 1 : 2;
    const PackArgs a = with_blocks(a0, eb, fused != nullptr), b = with_blocks(b0, eb, false);
    PackStats q = {};
    if (fused) {
        q.Be = (const float*)fused->d_Be;
        q.S = fused->d_S ? const_cast<double*>(fused->d_S) : fused->d_S_out;
        q.s_partial = s_partial;
        q.s_nparts = fused->d_S ? 0 : s_nparts;
        q.N = N;
        q.e_max = fused->e_max;
        q.c_sigma = fused->c_sigma;
        q.astat = (float*)fused->d_astat;
        q.expected = (float*)d_expected;
        q.T = (float*)d_T;
    }
    const dim3 grid(a.blocks + b.blocks), block(256);
    switch (dtype) {
        case VABFT_BF16: pack_kernel<bf16_t><<<grid, block, 0, st>>>(a, b, q); break;
        case VABFT_F16: pack_kernel<f16_t><<<grid, block, 0, st>>>(a, b, q); break;
        case VABFT_F8E4M3: pack_kernel<f8_t><<<grid, block, 0, st>>>(a, b, q); break;
        case VABFT_F8E5M2: pack_kernel<bf8_t><<<grid, block, 0, st>>>(a, b, q); break;
        default: return VABFT_EINVAL;
    }
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

}  // namespace vabft
