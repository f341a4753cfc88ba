// Epilogue of the whole-tile GEMM kernels whose accumulator tiles are 32 x 32 (the FP8 kernel), and the tile geometry
// that the 16-bit whole-tile kernel shares: row sums of the FP32 accumulator tile before output quantisation (paper
// section 3.6 "Online (Fused Kernel) ABFT"; section 2.2 C^{r1'} = C r1), the accumulator bit-flip injector (section
// 6.1), and the store of C.
//
// Tile 256 x 256 per workgroup of 4 wavefronts (2 x 2), 128 x 128 per wavefront as 4 x 4 MFMA tiles.  The MFMA is
// issued with the roles of A and B swapped (D' = B^T A^T), which puts one C row in one lane: lane l of a tile owns row
// (l % 32) and the 16 registers run along 16 of the tile's 32 columns, the other 16 sit in lane l ^ 32.  A row sum is
// therefore 16 in-register adds per tile plus one cross-lane add.
#pragma once
#include "gemm_common.h"

namespace vabft {

namespace g16 {
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
constexpr int STAGE = A_BYTES + B_BYTES;
constexpr int LDS_BYTES = 2 * STAGE;  // double buffered: 128 KiB
// epilogue scratch (the operand stages are free by then): row-sum staging at 0, the C staging slabs
// from 4096, the fused A-statistics staging at 40960 and the weighted row sums behind it
constexpr int SRED_OFFSET = 40960;
constexpr int RED2_OFFSET = SRED_OFFSET + 2 * 4 * BM * 4;
constexpr int CRED_OFFSET = RED2_OFFSET + 2 * BM * 4;  // column sums, [2 wm][256 columns]

}  // namespace g16

// Pieces of the epilogue of the 16-bit GEMM kernels.  Accumulator element (mi, ni, r) of a
// wavefront is
//   C[row0 + wm*128 + mi*32 + lane%32][col0 + wn*128 + ni*32 + 8*(r/4) + 4*(lane/32) + r%4].

// Fault injector on the accumulator registers (paper section 6.1 "Error injection").
template <bool INJECT>
__device__ __forceinline__ void gemm16_inject(const GemmArgs& g, f32x16_t (&acc)[4][4], int row0, int col0, int wm,
                                              int wn, int l32, int lh) {
    using namespace g16;
    const int rl_base = wm * 128 + l32;
    const int cl_base = wn * 128 + 4 * lh;
    if (INJECT) {
        const InjectArgs& inj = g.inj;
        if (inj.mode == 1) {
            for (int e = 0; e < inj.n_list; ++e) {
                const int fr = inj.d_list[3 * e], fc = inj.d_list[3 * e + 1], fb = inj.d_list[3 * e + 2];
                if (fr < row0 || fr >= row0 + BM || fc < col0 || fc >= col0 + BN) continue;
                if (fr >= g.M || fc >= g.N || fb < 0 || fb > 31) continue;
                const int rl = fr - row0, cl = fc - col0;
                const bool own = (rl >> 7) == wm && (cl >> 7) == wn && (rl & 31) == l32 && ((cl >> 2) & 1) == lh;
                if (own) {
                    const int idx = ((rl >> 5) & 3) * 64 + ((cl >> 5) & 3) * 16 + ((cl & 31) >> 3) * 4 + (cl & 3);
                    float before = 0.f, after = 0.f;
                    static_for<0, 4>([&](auto mi_c) {
                        static_for<0, 4>([&](auto ni_c) {
                            static_for<0, 16>([&](auto r_c) {
                                constexpr int mi = decltype(mi_c)::value, ni = decltype(ni_c)::value,
                                              r = decltype(r_c)::value;
                                if (idx == mi * 64 + ni * 16 + r) {
                                    before = acc[mi][ni][r];
                                    after = flip_bit(before, fb);
                                    acc[mi][ni][r] = after;
                                }
                            });
                        });
                    });
                    log_fault(inj, fr, fc, fb, (double)before, (double)after);
                }
            }
        } else if (inj.mode == 2) {
            static_for<0, 4>([&](auto mi_c) {
                static_for<0, 4>([&](auto ni_c) {
                    static_for<0, 16>([&](auto r_c) {
                        constexpr int mi = decltype(mi_c)::value, ni = decltype(ni_c)::value, r = decltype(r_c)::value;
                        const int gi = row0 + rl_base + mi * 32;
                        const int gj = col0 + cl_base + ni * 32 + 8 * (r >> 2) + (r & 3);
                        if (gi < g.M && gj < g.N) {
                            const int bit = bernoulli_bit(inj, gi, gj, g.N);
                            if (bit >= 0) acc[mi][ni][r] = flip_and_log<float>(inj, acc[mi][ni][r], gi, gj, bit);
                        }
                    });
                });
            });
        }
    }

}

// Row sums of the wavefront's accumulator tile, taken before quantisation (section 2.2
// C^{r1'} = C r1 on the tile; section 3.6 fused check): 63 in-register adds per row, arranged
// pairwise, plus one cross-lane add.  Lanes 0..31 leave the sum of row (wm*128 + mi*32 + lane) over the
// wavefront's 128 columns in red[wn][row].
__device__ __forceinline__ void gemm16_rowsum_to_lds(const f32x16_t (&acc)[4][4], float* red, int wm, int wn, int l32,
                                                     int lh) {
    using namespace g16;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        // pairwise over the 16 registers of a tile, then pairwise over the 4 tiles: a short
        // rounding-error chain (depth 7 with the cross-lane add) instead of 64 sequential adds
        float t[4];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            float q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                q[k] = (acc[mi][ni][4 * k] + acc[mi][ni][4 * k + 1]) + (acc[mi][ni][4 * k + 2] + acc[mi][ni][4 * k + 3]);
            t[ni] = (q[0] + q[1]) + (q[2] + q[3]);
        }
        float s = (t[0] + t[1]) + (t[2] + t[3]);
        s += __shfl_xor(s, 32, WAVE);
        if (lh == 0) red[wn * BM + wm * 128 + mi * 32 + l32] = s;
    }
}

// Position-weighted row sums of the wavefront's accumulator tile (section 2.2 C^{r2'} = C r2,
// r2 = [1..N]): sum_j (j + 1) acc[i][j].  Inside the tile the weights are small compile-time
// constants; the offset of the lane's first column is applied once to the plain partial sum.
// Lanes 0..31 leave the result over the wavefront's 128 columns in red2[wn][row].
__device__ __forceinline__ void gemm16_rowsum2_to_lds(const f32x16_t (&acc)[4][4], float* red2, int col0, int wm,
                                                      int wn, int l32, int lh) {
    using namespace g16;
    const float w0 = (float)(col0 + wn * 128 + 4 * lh + 1);  // weight of the lane's first column
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        float t1[4], t2[4];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            float a1 = 0.f, a2 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                a1 += acc[mi][ni][r];
                a2 = fmaf((float)(ni * 32 + 8 * (r >> 2) + (r & 3)), acc[mi][ni][r], a2);
            }
            t1[ni] = a1;
            t2[ni] = a2;
        }
        float s = fmaf(w0, (t1[0] + t1[1]) + (t1[2] + t1[3]), (t2[0] + t2[1]) + (t2[2] + t2[3]));
        s += __shfl_xor(s, 32, WAVE);
        if (lh == 0) red2[wn * BM + wm * 128 + mi * 32 + l32] = s;
    }
}

// Column sums of the wavefront's accumulator tile (section 2.2 C^{c1'} = c1 C): the four row blocks in
// registers first (64 values per lane, index v = ni*16 + r), then a reduce-scatter butterfly over the 32
// lanes that hold the 32 rows of a block: in step s the lanes that differ in bit 4-s exchange the half of
// their values whose index bit 5-s belongs to the partner and add what they receive, so the number of
// values per lane halves in every step (62 exchanges instead of 320).  Lane l ends with the complete sums
// of values 2*(l%32) and 2*(l%32)+1 and stores them to cred[wm][column].
template <int NV> struct ColReduce {
    static __device__ __forceinline__ void run(const float (&cur)[NV], int l32, float (&out)[2]) {
        constexpr int H = NV / 2;
        // NV = 64, 32, 16, 8, 4 pairs with lane bit 4, 3, 2, 1, 0
        constexpr int BIT = NV == 64 ? 4 : NV == 32 ? 3 : NV == 16 ? 2 : NV == 8 ? 1 : 0;
        const bool up = (l32 >> BIT) & 1;
        float nxt[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const float lo = cur[i], hi = cur[i + H];
            const float keep = up ? hi : lo, send = up ? lo : hi;
            nxt[i] = keep + __shfl_xor(send, 1 << BIT, WAVE);
        }
        if constexpr (H == 2) {
            out[0] = nxt[0];
            out[1] = nxt[1];
        } else {
            ColReduce<H>::run(nxt, l32, out);
        }
    }
};

__device__ __forceinline__ void gemm16_colsum_to_lds(const f32x16_t (&acc)[4][4], float* cred, int wm, int wn, int l32,
                                                     int lh) {
    using namespace g16;
    float v[64];
#pragma unroll
    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            v[ni * 16 + r] = (acc[0][ni][r] + acc[1][ni][r]) + (acc[2][ni][r] + acc[3][ni][r]);
    float out[2];
    ColReduce<64>::run(v, l32, out);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int idx = 2 * l32 + e, ni = idx >> 4, r = idx & 15;
        cred[wm * BN + wn * 128 + ni * 32 + 8 * (r >> 2) + 4 * lh + (r & 3)] = out[e];
    }
}

// Quantise and store the wavefront's tile of C.
template <typename T>
__device__ __forceinline__ void gemm16_store_c(const GemmArgs& g, const f32x16_t (&acc)[4][4], unsigned char* smem,
                                               int row0, int col0, int lane, int wm, int wn, int l32, int lh) {
    using namespace g16;
    uint16_t* __restrict__ C = reinterpret_cast<uint16_t*>(g.C);
    // Whole tiles: pass each 32 x 128 slab of the wavefront's tile through a private LDS
    // buffer so that global stores are 16 bytes per lane and 256 contiguous bytes per row
    // (a lane owns 4 consecutive columns of one row, which alone would give 8-byte pieces
    // scattered over 32 rows).  Row pitch 264 B keeps the ds_write_b64 conflict free.
    constexpr int PITCH = 264;
    unsigned char* stage = smem + 4096 + (wm * 2 + wn) * (32 * PITCH);
    const int srow = lane >> 4, schunk = lane & 15;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint16_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = Elem<T>::from_acc(acc[mi][ni][4 * q + e]);
                uint2 v;
                v.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
                v.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
                *reinterpret_cast<uint2*>(stage + l32 * PITCH + ni * 64 + q * 16 + lh * 8) = v;
            }
        // LDS operations of one wavefront complete in order; only the compiler must not
        // move the reads above the writes (or the next slab's writes above these reads)
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int r = srow + 4 * t;
            const raw16 v = *reinterpret_cast<const raw16*>(stage + r * PITCH + schunk * 16);
            const int gi = row0 + wm * 128 + mi * 32 + r;
            const int gj = col0 + wn * 128 + schunk * 8;
            // C is not read again by this kernel: non-temporal store (measured 1.3 % of kernel time)
            typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_st;
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4_st, v),
                                        reinterpret_cast<u32x4_st*>(C + (int64_t)gi * g.ldc + gj));
        }
        asm volatile("" ::: "memory");
    }
}

}  // namespace vabft
