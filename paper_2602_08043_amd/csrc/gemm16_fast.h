// BF16 / FP16 GEMM on v_mfma_f32_16x16x32: 256 x 256 x 64 tile per workgroup of 4 wavefronts (2 x 2), 128 x 128 per
// wavefront = 8 x 8 MFMA tiles of 16 x 16, 256 accumulator registers, one wavefront per SIMD.  Rows of A and B are 16-byte aligned;
// products without injector and K-blocks take any M and N (EDGE), the plain and the checked one also tiles of 192 or 128
// columns where those fill the chip better (NF = 6, 4).
//
// Why the 16 x 16 x 32 instruction: on N(0,1)-like operands the chip is power-limited, not issue-limited, and
// this shape moves half the accumulator bytes per flop of the 32 x 32 x 16 one (a register-only loop of it
// sustains 2035 TFLOP/s at 2.04 GHz against 1792 at 1.78 GHz).
//
// The MFMA is issued with the operands swapped (D' = B^T A^T): lane l of a 16 x 16 result tile then owns
// C row (l % 16) and the four consecutive columns 4 * (l / 16) + 0..3, so a row sum of the accumulator tile
// (section 2.2 C^{r1'} = C r1, taken before quantisation: section 3.6 fused check) is in-register adds plus
// two cross-lane adds.  Accumulator element (mi, ni, r) of a wavefront is
//   C[row0 + wm*128 + mi*16 + lane%16][col0 + wn*128 + ni*16 + 4*(lane/16) + r].
//
// LDS (two stages per operand, 32 KiB each, [A0 | A1 | B0 | B1] so that the stages of an operand are an
// instruction immediate apart):
//   A tile, and B tile when B is stored N x K:  [256 rows][8 chunks of 16 B], chunk c of row r at position
//       c ^ ((r >> 1) & 7); a 16 x 32 fragment is one ds_read_b128 (lane: row l%16, chunk 4*ks + l/16), whose
//       16 lanes of a row group hit 16 distinct 16-byte slots of a 256-byte window.
//   B tile when B is stored K x N:  [64 k][32 chunks of 16 B] (n contiguous), chunk c of row k at position
//       c ^ 2*((k & 3) | 4*((k >> 3) & 1)) (narrow tiles: see the kernel); a fragment is two ds_read_b64_tr_b16, each handing lane i of a
//       16-lane block the 4 k-consecutive values of column i of a 4(k) x 16(n) sub-tile.
// Global memory -> LDS without passing through registers (global_load_lds_dwordx4), issued from inline
// assembly with a scalar base and a 32-bit lane offset: four loads share one M0 (LDS base) through their
// immediate offsets, so a load costs one issue slot and the address arithmetic is four scalar adds per k-tile.
//
// The MFMAs are inline assembly with the accumulator tied to its register ("+a"): left to the register
// allocator, a quarter of the 64 accumulator tiles changed registers every iteration and were copied
// through the vector file.  The compiler's hazard handling does not see into them; the hazards in reach are at
// the ends of the loop (operands written by vector code in front of an MFMA, accumulators read by vector code
// behind one: settle_accumulators) and are padded by hand; asm_lint.py checks the generated assembly.
//
// Kernel modes: 0 plain; 1 row check; 2 injector (with every kind of sum); 3 + position-weighted row sums; 4 +
// column sums; 5 partial row sums only (block-wise check by a kernel of its own); 6 / 7 prefix row sums at every
// K-block boundary (block-wise check with K split as well; 7 with the injector).
// Check-side work fused into this kernel (MODE >= 1): see gemm_tile32.h.  FUSED adds the A-side of Algorithm 1
// on the matrix cores: tile-column bn folds the k-units (128 k) u = bn, bn + tiles_n, ... of its rows of A.
// For those units a 16-column panel [1, Be_hi, Be_mid, Be_lo, 0 ...] (Be split into three pieces of the
// input type, so that the FP32-accumulated products carry Be to FP32 precision) is multiplied like one more
// B fragment: its result tile holds sum_k A[i][k] and the three partial dot products A[i] . Be.  Only max and
// min of the row stay in the vector ALU, as packed 16-bit operations on the fragment registers.
#pragma once
#include "gemm_tile32.h"
#include "row_threshold.h"

namespace vabft {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) short s16x2_t;
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;

// v_mfma_f32_16x16x32 as inline assembly with the accumulator tied to its registers.  The compiler's hazard
// handling does not see into it: a vector instruction that writes one of its operands must not sit within a
// few issue slots in front of it (measured: a v_cndmask three slots ahead corrupted the product), and to the
// compiler the statement has read its operands once it is issued, so the next vector instruction may get
// their registers.  acc_a (the GEMM tiles, AGPRs): its operands only ever come from LDS reads, and nothing but
// loads (whose results land later), scalar code and other MFMAs follows it.  acc_v4 (the four statistics tiles,
// VGPRs, amid ordinary vector code): eight idle issue slots behind the group, and the caller puts five in
// front of it.
template <typename T> struct Mfma16x;
template <> struct Mfma16x<bf16_t> {
    static __device__ __forceinline__ void acc_a(f32x4_t& c, const raw16& a, const raw16& b) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(c)
                     : "v"(__builtin_bit_cast(u32x4_t, a)), "v"(__builtin_bit_cast(u32x4_t, b)));
    }
    // c[j] += x * b[j], j = 0..3, as one statement (nothing can be scheduled between the four)
    static __device__ __forceinline__ void acc_v4(f32x4_t (&c)[4], const raw16& x, const raw16 (&b)[4]) {
        asm volatile(
            "v_mfma_f32_16x16x32_bf16 %0, %4, %5, %0\n\tv_mfma_f32_16x16x32_bf16 %1, %4, %6, %1\n\t"
            "v_mfma_f32_16x16x32_bf16 %2, %4, %7, %2\n\tv_mfma_f32_16x16x32_bf16 %3, %4, %8, %3\n\ts_nop 7"
            : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3])
            : "v"(__builtin_bit_cast(u32x4_t, x)), "v"(__builtin_bit_cast(u32x4_t, b[0])),
              "v"(__builtin_bit_cast(u32x4_t, b[1])), "v"(__builtin_bit_cast(u32x4_t, b[2])),
              "v"(__builtin_bit_cast(u32x4_t, b[3])));
    }
};
template <> struct Mfma16x<f16_t> {
    static __device__ __forceinline__ void acc_a(f32x4_t& c, const raw16& a, const raw16& b) {
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0"
                     : "+a"(c)
                     : "v"(__builtin_bit_cast(u32x4_t, a)), "v"(__builtin_bit_cast(u32x4_t, b)));
    }
    static __device__ __forceinline__ void acc_v4(f32x4_t (&c)[4], const raw16& x, const raw16 (&b)[4]) {
        asm volatile(
            "v_mfma_f32_16x16x32_f16 %0, %4, %5, %0\n\tv_mfma_f32_16x16x32_f16 %1, %4, %6, %1\n\t"
            "v_mfma_f32_16x16x32_f16 %2, %4, %7, %2\n\tv_mfma_f32_16x16x32_f16 %3, %4, %8, %3\n\ts_nop 7"
            : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3])
            : "v"(__builtin_bit_cast(u32x4_t, x)), "v"(__builtin_bit_cast(u32x4_t, b[0])),
              "v"(__builtin_bit_cast(u32x4_t, b[1])), "v"(__builtin_bit_cast(u32x4_t, b[2])),
              "v"(__builtin_bit_cast(u32x4_t, b[3])));
    }
};

namespace g16x {
using namespace g16;
using namespace g16f;
// Schedule of the 16 global -> LDS loads of the next tile inside a tile body of 128 MFMA slots: load j goes out at
// slot LOFF + j * LSTRIDE.  Measured on BF16 4096^3 (plain GEMM, same box, alternating): one load every 8 slots (the
// last one 7 slots in front of the barrier, which then waits for it) 95.8 us; every 4 slots (all inside the first
// step) 90.0 us, every 5 or 6 the same; every 2 slots 99.0 us (64 lanes x 16 B every 32 cycles from each of four
// wavefronts is more than the compute unit's vector memory path takes, and the queue stalls the MFMA issue).
constexpr int LSTRIDE = 4;
constexpr int LOFF = 1;      // >= 1: the M0 of a group of four rides one slot ahead of its first load
constexpr int HALF = 32768;  // a stage of A, and of a 256-wide B
// FUSED: behind the operand stages, the panel [1, Be_hi, Be_mid, Be_lo] of every k32-step this tile-column
// folds: per folded unit (slot) 4 steps x 4 panel rows x 32 k x 2 B = 1 KiB, at most PANEL_UNITS_* units;
// behind it 12 doubles for the fold of the S1..S3 partials and 5 floats: per-wavefront max |Be|, the scale
// LDS of a tile with NF column fragments per wavefront.  A k-tile of a narrow tile has fewer MFMA cycles (1536 and 1024
// instead of 2048) to hide the way of the next one's operands from memory, about 1700 cycles from the first load's issue
// to the barrier; a third stage for A (and for a 128-wide B) sends those loads out one k-tile earlier.  With two stages
// each: 1024 x 4096 x 4096 in 128-wide tiles 60.5 us, now 49; in 192-wide ones 66.7, now 62.
template <int NF> struct Lds16 {
    static constexpr bool NARROW = NF < 8;
    static constexpr int A_STAGES = NARROW ? 3 : 2, B_STAGES = NF == 4 ? 3 : 2;
    static constexpr int B_STAGE = 4096 * NF;
    static constexpr int B_AT = A_STAGES * HALF;
    static constexpr int PANEL = B_AT + B_STAGES * B_STAGE, SLOTS = NARROW ? PANEL_UNITS_NARROW : PANEL_UNITS_WIDE;
    static constexpr int S_RED = PANEL + SLOTS * 1024, SCALE = S_RED + 128;
    static constexpr int BYTES = PANEL, BYTES_FUSED = SCALE + 64;
    static_assert(BYTES_FUSED <= 160 * 1024, "LDS of a compute unit");
};

// a wave-uniform pointer, made visibly so (the inline assembly below needs it in scalar registers)
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
}
// Pins two uniform pointers in scalar registers and keeps the following instructions clear of whatever produced
// them: a scalar register written by the vector ALU (v_readfirstlane, v_readlane) must not be read by a memory
// instruction within five issue slots.  The compiler pads that hazard for instructions it knows, but it cannot
// see that the assembly statements below are memory instructions (measured: a load issued right behind the
// v_readfirstlane of its base took a stale base and faulted).
__device__ __forceinline__ void settle_bases(const unsigned char*& a, const unsigned char*& b) {
    asm volatile("s_nop 4" : "+s"(a), "+s"(b));
}
// M0 <- LDS base of the next group of four loads (one issue slot must separate it from the load that uses it)
__device__ __forceinline__ void set_m0(uint32_t lds_addr) { asm volatile("s_mov_b32 m0, %0" ::"s"(lds_addr)); }
// 16 bytes per lane: global (scalar base + lane offset + IMM) -> LDS (M0 + IMM + lane * 16)
template <int IMM> __device__ __forceinline__ void g2l16_m0(uint32_t voff, const unsigned char* sbase) {
    static_assert(IMM >= 0 && IMM < 4096, "13-bit signed immediate");
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(voff), "s"(sbase), "n"(IMM));
}
// Registers a128 .. a255 for the sums of the chains of a narrow tile (FORM16_128_CHAINS), named here and not by the compiler:
// as variables beside the 128 accumulators they spilled into scratch memory in any arrangement tried, 60 us a launch.  The
// compiler needs no accumulation register from a128 on (build.py fails if it uses one: asm_lint.py).
template <int I> __device__ __forceinline__ void chain_clear() { asm volatile("v_accvgpr_write_b32 a[%0], 0" ::"n"(128 + I)); }
template <int I> __device__ __forceinline__ void chain_add(float x) {
    float t;
    asm volatile("v_accvgpr_read_b32 %0, a[%2]\n\tv_add_f32 %0, %0, %1\n\tv_accvgpr_write_b32 a[%2], %0" : "=&v"(t) : "v"(x), "n"(128 + I));
}
template <int I> __device__ __forceinline__ float chain_sum() {
    float t;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(t) : "n"(128 + I));
    return t;
}
__device__ __forceinline__ void chain_reserve() {
    asm volatile("" ::: "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141",
                 "a142", "a143", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155",
                 "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169",
                 "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183",
                 "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", "a197",
                 "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211",
                 "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225",
                 "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239",
                 "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253",
                 "a254", "a255");
}
}  // namespace g16x

// ---- epilogue pieces for the 16 x 16 accumulator layout -------------------------------------------------------

// Fault injector on the accumulator registers (section 6.1 "Error injection").
template <bool INJECT>
__device__ __forceinline__ void gemm16x_inject(const GemmArgs& g, f32x4_t (&acc)[8][8], int row0, int col0, int wm,
                                               int wn, int l16, int lq) {
    using namespace g16;
    if (INJECT) {
        const InjectArgs& inj = g.inj;
        if (inj.mode == 1) {
            for (int e = 0; e < inj.n_list; ++e) {
                const int fr = inj.d_list[3 * e], fc = inj.d_list[3 * e + 1], fb = inj.d_list[3 * e + 2];
                if (fr < row0 || fr >= row0 + BM || fc < col0 || fc >= col0 + BN) continue;
                if (fr >= g.M || fc >= g.N || fb < 0 || fb > 31) continue;
                const int rl = fr - row0, cl = fc - col0;
                const bool own = (rl >> 7) == wm && (cl >> 7) == wn && (rl & 15) == l16 && ((cl >> 2) & 3) == lq;
                if (own) {
                    const int idx = ((rl >> 4) & 7) * 32 + ((cl >> 4) & 7) * 4 + (cl & 3);
                    float before = 0.f, after = 0.f;
                    static_for<0, 8>([&](auto mi_c) {
                        static_for<0, 8>([&](auto ni_c) {
                            static_for<0, 4>([&](auto r_c) {
                                constexpr int mi = decltype(mi_c)::value, ni = decltype(ni_c)::value,
                                              r = decltype(r_c)::value;
                                if (idx == mi * 32 + ni * 4 + r) {
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
            static_for<0, 8>([&](auto mi_c) {
                static_for<0, 8>([&](auto ni_c) {
                    static_for<0, 4>([&](auto r_c) {
                        constexpr int mi = decltype(mi_c)::value, ni = decltype(ni_c)::value, r = decltype(r_c)::value;
                        const int gi = row0 + wm * 128 + mi * 16 + l16;
                        const int gj = col0 + wn * 128 + ni * 16 + 4 * lq + r;
                        const int bit = bernoulli_bit(inj, gi, gj, g.N);
                        if (bit >= 0) acc[mi][ni][r] = flip_and_log<float>(inj, acc[mi][ni][r], gi, gj, bit);
                    });
                });
            });
        }
    }
}

// Row sums of the wavefront's accumulator tile, taken before quantisation: 31 in-register adds per row,
// arranged pairwise, plus two cross-lane adds.  Lanes 0..15 leave the sum of row wm*128 + mi*16 + lane over
// the wavefront's 128 columns in red[wn][row].
template <int NF>
__device__ __forceinline__ void gemm16x_rowsum_to_lds(const f32x4_t (&acc)[8][NF], float* red, int wm, int wn, int l16,
                                                      int lq) {
    using namespace g16;
    // the eight row fragments side by side: their cross-lane exchanges are in flight together (one wait per
    // exchange round instead of one per fragment); the order of the additions of a row is unchanged
    float s[8];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) {
        float t[NF];
#pragma unroll
        for (int ni = 0; ni < NF; ++ni) t[ni] = (acc[mi][ni][0] + acc[mi][ni][1]) + (acc[mi][ni][2] + acc[mi][ni][3]);
        s[mi] = (t[0] + t[1]) + (t[2] + t[3]);
        if constexpr (NF == 8) s[mi] += (t[4] + t[5]) + (t[6] + t[7]);
        if constexpr (NF == 6) s[mi] += t[4] + t[5];
    }
    float x[8];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) x[mi] = __shfl_xor(s[mi], 16, WAVE);
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) s[mi] += x[mi];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) x[mi] = __shfl_xor(s[mi], 32, WAVE);
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) s[mi] += x[mi];
    if (lq == 0) {
#pragma unroll
        for (int mi = 0; mi < 8; ++mi) red[wn * BM + wm * 128 + mi * 16 + l16] = s[mi];
    }
}

// Plain and position-weighted row sums together (section 2.2 C^{r2'} = C r2, r2 = [1..N]: sum_j (j + 1) acc[i][j]):
// every accumulator value is read once for both.  Inside the tile the weights are small compile-time constants;
// the offset of the lane's first column is applied once to the plain partial sum, which is formed exactly as
// gemm16x_rowsum_to_lds forms it (same tree, same bits).
__device__ __forceinline__ void gemm16x_rowsums12_to_lds(const f32x4_t (&acc)[8][8], float* red, float* red2, int col0,
                                                         int wm, int wn, int l16, int lq) {
    using namespace g16;
    const float w0 = (float)(col0 + wn * 128 + 4 * lq + 1);  // weight of the lane's first column
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) {
        float t1[8], t2[8];
#pragma unroll
        for (int ni = 0; ni < 8; ++ni) {
            const float a0 = acc[mi][ni][0], a1 = acc[mi][ni][1], a2 = acc[mi][ni][2], a3 = acc[mi][ni][3];
            t1[ni] = (a0 + a1) + (a2 + a3);
            t2[ni] = fmaf((float)(ni * 16 + 3), a3, fmaf((float)(ni * 16 + 2), a2, fmaf((float)(ni * 16 + 1), a1, (float)(ni * 16) * a0)));
        }
        const float p1 = ((t1[0] + t1[1]) + (t1[2] + t1[3])) + ((t1[4] + t1[5]) + (t1[6] + t1[7]));
        const float p2 = ((t2[0] + t2[1]) + (t2[2] + t2[3])) + ((t2[4] + t2[5]) + (t2[6] + t2[7]));
        float s1 = p1;
        s1 += __shfl_xor(s1, 16, WAVE);
        s1 += __shfl_xor(s1, 32, WAVE);
        float s2 = fmaf(w0, p1, p2);
        s2 += __shfl_xor(s2, 16, WAVE);
        s2 += __shfl_xor(s2, 32, WAVE);
        if (lq == 0) {
            red[wn * BM + wm * 128 + mi * 16 + l16] = s1;
            red2[wn * BM + wm * 128 + mi * 16 + l16] = s2;
        }
    }
}

// Column sums of the wavefront's accumulator tile (section 2.2 C^{c1'} = c1 C): the eight row blocks in
// registers first (32 values per lane, index v = ni*4 + r), then a reduce-scatter butterfly over the 16 lanes
// that hold the 16 rows of a block.  Lane l ends with the complete sums of values 2*(l%16) and 2*(l%16)+1.
template <int NV> struct ColReduce16 {
    static __device__ __forceinline__ void run(const float (&cur)[NV], int l16, float (&out)[2]) {
        constexpr int H = NV / 2;
        constexpr int BIT = NV == 32 ? 3 : NV == 16 ? 2 : NV == 8 ? 1 : 0;
        const bool up = (l16 >> BIT) & 1;
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
            ColReduce16<H>::run(nxt, l16, out);
        }
    }
};
__device__ __forceinline__ void gemm16x_colsum_to_lds(const f32x4_t (&acc)[8][8], float* cred, int wm, int wn, int l16,
                                                      int lq) {
    using namespace g16;
    float v[32];
#pragma unroll
    for (int ni = 0; ni < 8; ++ni)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            v[ni * 4 + r] = ((acc[0][ni][r] + acc[1][ni][r]) + (acc[2][ni][r] + acc[3][ni][r])) +
                            ((acc[4][ni][r] + acc[5][ni][r]) + (acc[6][ni][r] + acc[7][ni][r]));
    float out[2];
    ColReduce16<32>::run(v, l16, out);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int idx = 2 * l16 + e, ni = idx >> 2, r = idx & 3;
        cred[wm * BN + wn * 128 + ni * 16 + 4 * lq + r] = out[e];
    }
}

// two accumulator values -> packed pair of output elements, round to nearest even (v_cvt_pk_bf16_f32 /
// v_cvt_pk_f16_f32)
template <typename T> __device__ __forceinline__ uint32_t pack2(float a, float b);
template <> __device__ __forceinline__ uint32_t pack2<bf16_t>(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}
template <> __device__ __forceinline__ uint32_t pack2<f16_t>(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, f16x2_t));
}

// Quantise and store the wavefront's tile of C: each 16 x 128 slab passes through a private LDS buffer so
// that global stores are 16 bytes per lane and 256 contiguous bytes per row (a lane owns 4 consecutive
// columns of one row, which alone would give 8-byte pieces scattered over 16 rows).
// EDGE: rows and columns past the end are left out; C is aligned to its elements only (a last group of fewer than eight
// columns goes out element by element).
template <typename T, bool EDGE, int NF>
__device__ __forceinline__ void gemm16x_store_c(const GemmArgs& g, const f32x4_t (&acc)[8][NF], unsigned char* smem,
                                                int row0, int col0, int lane, int wm, int wn, int l16, int lq) {
    // row pitch 272 B: the 8-byte writes of 16 rows x 2 column groups hit 32 distinct bank pairs
    constexpr int PITCH = 272;
    constexpr int SLAB = 16 * PITCH;
    unsigned char* stage = smem + 4096 + (wm * 2 + wn) * (2 * SLAB);
    uint16_t* __restrict__ C = reinterpret_cast<uint16_t*>(g.C);
    constexpr int LPR = NF > 4 ? 16 : 8;  // lanes per row (a row of six fragments leaves four of them idle)
    const int srow = lane / LPR, schunk = lane % LPR;
    const int gj = col0 + wn * (16 * NF) + schunk * 8;
    const bool in_row = (2 * NF == LPR || schunk < 2 * NF) && (!EDGE || gj < g.N);
#pragma unroll
    for (int mi = 0; mi < 8; ++mi) {
        unsigned char* sl = stage + (mi & 1) * SLAB;
#pragma unroll
        for (int ni = 0; ni < NF; ++ni) {
            uint2 v;
            v.x = pack2<T>(acc[mi][ni][0], acc[mi][ni][1]);
            v.y = pack2<T>(acc[mi][ni][2], acc[mi][ni][3]);
            *reinterpret_cast<uint2*>(sl + l16 * PITCH + ni * 32 + lq * 8) = v;
        }
        // LDS operations of one wavefront complete in order; only the compiler must not move the reads
        // above the writes
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < LPR / 4; ++t) {
            const int r = srow + (64 / LPR) * t;
            const raw16 v = *reinterpret_cast<const raw16*>(sl + r * PITCH + schunk * 16);
            const int gi = row0 + wm * 128 + mi * 16 + r;
            // C is not read again by this kernel: non-temporal store
            typedef uint32_t u32x4_al __attribute__((ext_vector_type(4)));
            typedef uint32_t u32x4_un __attribute__((ext_vector_type(4), aligned(2)));
            using u32x4_st = typename std::conditional<EDGE, u32x4_un, u32x4_al>::type;
            uint16_t* c = C + (int64_t)gi * g.ldc + gj;
            if (in_row && (!EDGE || (gi < g.M && gj + 8 <= g.N)))
                __builtin_nontemporal_store(__builtin_bit_cast(u32x4_st, v), reinterpret_cast<u32x4_st*>(c));
            else if (EDGE && in_row && gi < g.M) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (gj + e < g.N) c[e] = (uint16_t)(v.w[e >> 1] >> (16 * (e & 1)));
            }
        }
        asm volatile("" ::: "memory");
    }
}

// ---- fused A-side statistics: helpers ---------------------------------------------------------------------

// Running (max, min) of 16-bit floating-point values held two per dword.
// BF16 has no packed max / min: with the bit patterns read as integers, non-negative values order like
// signed integers and negative values order reversed, so three integer trackers suffice:
//   smax = signed max, smin = signed min, umax = unsigned max;
//   max = smax >= 0 ? smax : smin  (no non-negative value: the negative of smallest magnitude),
//   min = umax has its sign bit ? umax : smin  (a negative value exists: the one of largest magnitude).
template <typename T> struct MinMax16;
template <> struct MinMax16<bf16_t> {
    uint32_t smax, smin, umax;
    __device__ __forceinline__ void init() {
        smax = 0x80008000u;
        smin = 0x7fff7fffu;
        umax = 0u;
    }
    __device__ __forceinline__ void fold(uint32_t d) {
        smax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2_t, smax),
                                                                     __builtin_bit_cast(s16x2_t, d)));
        smin = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(s16x2_t, smin),
                                                                     __builtin_bit_cast(s16x2_t, d)));
        umax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, umax),
                                                                     __builtin_bit_cast(u16x2_t, d)));
    }
    // the tracker of the lane `off` away, combined kind by kind
    __device__ __forceinline__ void merge_xor(int off) {
        const uint32_t a = __shfl_xor(smax, off, WAVE), b = __shfl_xor(smin, off, WAVE), c = __shfl_xor(umax, off, WAVE);
        smax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2_t, smax),
                                                                     __builtin_bit_cast(s16x2_t, a)));
        smin = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(s16x2_t, smin),
                                                                     __builtin_bit_cast(s16x2_t, b)));
        umax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, umax),
                                                                     __builtin_bit_cast(u16x2_t, c)));
    }
    // the two halves of the trackers, then as floats
    __device__ __forceinline__ void result(float& mx, float& mn) const {
        const int a = (int)(short)(smax & 0xffffu), b = (int)(short)(smax >> 16);
        const int c = (int)(short)(smin & 0xffffu), d = (int)(short)(smin >> 16);
        const uint32_t e = umax & 0xffffu, f = umax >> 16;
        const int sM = a > b ? a : b, sm = c < d ? c : d;
        const uint32_t uM = e > f ? e : f;
        const uint32_t bmx = (uint32_t)(sM >= 0 ? sM : sm) & 0xffffu;
        const uint32_t bmn = (uM & 0x8000u) ? uM : ((uint32_t)sm & 0xffffu);
        mx = __uint_as_float(bmx << 16);
        mn = __uint_as_float(bmn << 16);
    }
};
template <> struct MinMax16<f16_t> {
    uint32_t vmax, vmin;
    __device__ __forceinline__ void init() {
        vmax = 0xfbfffbffu;  // -65504
        vmin = 0x7bff7bffu;  // +65504
    }
    __device__ __forceinline__ void fold(uint32_t d) {
        vmax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(f16x2_t, vmax),
                                                                     __builtin_bit_cast(f16x2_t, d)));
        vmin = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(f16x2_t, vmin),
                                                                     __builtin_bit_cast(f16x2_t, d)));
    }
    __device__ __forceinline__ void merge_xor(int off) {
        const uint32_t a = __shfl_xor(vmax, off, WAVE), b = __shfl_xor(vmin, off, WAVE);
        vmax = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(f16x2_t, vmax),
                                                                     __builtin_bit_cast(f16x2_t, a)));
        vmin = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(f16x2_t, vmin),
                                                                     __builtin_bit_cast(f16x2_t, b)));
    }
    __device__ __forceinline__ void result(float& mx, float& mn) const {
        const f16x2_t a = __builtin_bit_cast(f16x2_t, vmax), b = __builtin_bit_cast(f16x2_t, vmin);
        mx = fmaxf((float)a[0], (float)a[1]);
        mn = fminf((float)b[0], (float)b[1]);
    }
};

// x as three pieces of the input type whose sum is x to (at least) FP32 precision
template <typename T> __device__ __forceinline__ void split3(float x, uint16_t (&p)[3]) {
    p[0] = Elem<T>::from_acc(x);
    const float r1 = x - Elem<T>::to_acc(p[0]);
    p[1] = Elem<T>::from_acc(r1);
    const float r2 = r1 - Elem<T>::to_acc(p[1]);
    p[2] = Elem<T>::from_acc(r2);
}
template <typename T> __device__ __forceinline__ uint16_t one16();
template <> __device__ __forceinline__ uint16_t one16<bf16_t>() { return 0x3f80; }
template <> __device__ __forceinline__ uint16_t one16<f16_t>() { return 0x3c00; }

// The assembly MFMAs are opaque to the compiler's hazard handling: before vector code reads the accumulators, idle
// slots let the last results land.  The empty statements behind them redefine every accumulator as far as the
// compiler can tell, so no read of one can be scheduled in front of the idle slots (register reads are not
// ordered against an assembly statement by its memory clobber).
template <int NF> __device__ __forceinline__ void settle_accumulators(f32x4_t (&acc)[8][NF]) {
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int ni = 0; ni < NF; ++ni) asm volatile("" : "+a"(acc[mi][ni]));
}

// The tile of rows row0 .. row0 + 255 and columns col0 .. col0 + 32 NF - 1; bm, bn: its tile-row and tile-column.
// NF: column fragments per wavefront.  8 is the 256 x 256 tile; 6 and 4 (256 x 192, 256 x 128) serve the plain and the
// checked product where wide tiles would leave compute units without work (gemm16_columns in api.hip).
// EDGE: M and N need not be multiples of the tile nor K of 64 (K is a multiple of 8, with B stored K x N N as well, K is at
// least 64).  Rows and
// columns past the end are read from the last valid ones -- the lane offsets are clamped once, the main loop is the
// same -- and dropped in the epilogue; the k past the last whole tile are multiplied by a step of their own behind the
// loop, zero-filled on their way to LDS.
// CHAINS: K in four chains behind each other, added up in registers that only the narrowest tile has (3 x 1.3 us a tile):
// the rounding error of the direct kernels, where copies of their operands come here (row sums of BF16 2049 x 2303 x 1001
// against 64 bits 1.3e-7, in one chain 2.0e-7; FP16 1001 x 5001 x 9001 3.8e-7, 7.3e-7).
template <typename T, int TRANSB, int MODE, bool FUSED, bool EDGE, int NF, bool CHAINS>
__device__ __forceinline__ void gemm16_fast_tile(const GemmArgs& g, int bm, int bn, int row0, int col0) {
    static_assert(!EDGE || MODE <= 1 || (NF == 8 && MODE >= 3 && MODE <= 5), "no injector and no K-blocks at other sizes");
    static_assert(NF == 8 || (EDGE && (NF == 6 || NF == 4)), "narrow tiles");
    static_assert(!CHAINS || (NF == 4 && MODE <= 1 && !FUSED), "registers for the sum of the chains");
    using namespace g16x;
    // MODE 6 / 7: block-wise check with K split as well (7: with the injector).  The kernel leaves the row sums of
    // the accumulator tile at every K-block boundary and at the end, in double; a kernel of its own forms the
    // K-block shares as differences of consecutive prefixes and compares them.
    constexpr bool KSNAP = MODE == 6 || MODE == 7;
    constexpr bool VERIFY = MODE >= 1 && !KSNAP, INJECT = MODE == 2 || MODE == 7, WSUM = MODE == 2 || MODE == 3;
    constexpr bool CSUM = MODE == 2 || MODE == 4;
    static_assert(!FUSED || VERIFY, "fused statistics belong to the verified kernel");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    lds_u8* const lds = (lds_u8*)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, lq = lane >> 4;
    const int l32 = lane & 31, lh = lane >> 5;
    if (CSUM && blockIdx.x == 0 && tid == 0 && g.d_ncolflag) *g.d_ncolflag = 0;
    if ((MODE == 5 || MODE == 2 || KSNAP) && blockIdx.x == 0 && tid == 0 && (g.block_mode || KSNAP)) {
        *g.d_nflag = 0;
        *g.d_nblockflag = 0;
    }
    constexpr int TN = 32 * NF;               // columns of the tile
    constexpr int NLOAD = 8 + NF, NSLOT = 8 * NF;
    using L = Lds16<NF>;
    constexpr int B_BASE = L::B_AT;
    const unsigned char* __restrict__ A = reinterpret_cast<const unsigned char*>(g.A);
    const unsigned char* __restrict__ B = reinterpret_cast<const unsigned char*>(g.B);

    f32x4_t acc[8][NF];
#pragma unroll
    for (int mi = 0; mi < 8; ++mi)
#pragma unroll
        for (int ni = 0; ni < NF; ++ni)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.f;

    // ---- global -> LDS: each wavefront issues 8 + NF loads of 1 KiB per k-tile ----------------------------
    // A (and an N x K B): load l covers rows wave*64 (B: wave*8 NF) + 8l .. +7; lane sits at row lane/8, chunk position lane%8
    // and fetches chunk (lane%8) ^ ((row>>1)&7), (row>>1)&7 = 4*(l&1) + lane/16.
    // K x N B: rows of 4 NF chunks, 16 k rows per wavefront; chunk position pos of row k holds chunk pos ^ f(k).
    // Rows of 512 or 256 bytes: f = 2*((k&3) | 4*((k>>3)&1)), so that the eight rows of a transposing read hit distinct
    // slots; rows of 384 bytes start half a window apart by themselves: f = 2*(((k>>1)&1) | 2*((k>>3)&1)).
    // Load l of a tile lands at LDS offset l*1024 of the wavefront's area: M0 holds the base of a group of
    // four, the immediate (l&3)*1024 is added to both addresses, so the lane offset carries -(l&3)*1024.
    // (EDGE: offsets are taken from the tile's first row and column; 4096 more on the lane's side than on the base's
    // keeps them positive where clamped rows no longer outweigh the immediates)
    constexpr int BIAS = EDGE ? 4096 : 0;
    const unsigned char* const a_base =
        uniform_ptr((EDGE ? A + (int64_t)row0 * g.lda * 2 : A + (int64_t)(row0 + wave * 64) * g.lda * 2) - BIAS);
    const unsigned char* const b_base =
        uniform_ptr((TRANSB ? (EDGE ? B + (int64_t)col0 * g.ldb * 2 : B + (int64_t)(col0 + wave * 8 * NF) * g.ldb * 2)
                            : B + ((int64_t)(wave * 16) * g.ldb + col0) * 2) - BIAS);
    uint32_t a_voff[8], b_voff[NF];
    const auto kn_swz = [](int k) {
        return NF == 6 ? 2 * (((k >> 1) & 1) | 2 * ((k >> 3) & 1)) : 2 * ((k & 3) | 4 * ((k >> 3) & 1));
    };
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        const uint32_t rk = ((lane & 7) ^ (lane >> 4) ^ (4 * (l & 1))) << 4;
        const int q = (lane >> 3) + 8 * l;
        const int ar = EDGE ? min(wave * 64 + q, g.M - 1 - row0) : q;
        a_voff[l] = (uint32_t)ar * (uint32_t)g.lda * 2 + rk - (l & 3) * 1024 + BIAS;
        if (TRANSB) {
            const int br = EDGE ? min(wave * 8 * NF + q, g.N - 1 - col0) : q;
            if (l < NF) b_voff[l] = (uint32_t)br * (uint32_t)g.ldb * 2 + rk - (l & 3) * 1024 + BIAS;
        } else {
            int k = (l * 64 + lane) / (4 * NF), n = ((l * 64 + lane) % (4 * NF) ^ kn_swz(k)) << 3;
            if (NF == 8) {  // the same, written so that the compiler sees what the loads have in common
                k = lh + 2 * l;
                n = (l32 ^ 2 * ((2 * (l & 1) + lh) | (4 * (l >> 2)))) << 3;
            }
            const int bc = EDGE ? min(n, g.b_cols - 8 - col0) : n;
            if (l < NF) b_voff[l] = (uint32_t)k * (uint32_t)g.ldb * 2 + bc * 2 - (l & 3) * 1024 + BIAS;
        }
    }
    const int64_t b_ktile = TRANSB ? (int64_t)(BK * 2) : (int64_t)BK * g.ldb * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const uint32_t a_dst = __builtin_amdgcn_readfirstlane(lds0 + wave * 8192);
    const uint32_t b_dst = __builtin_amdgcn_readfirstlane(lds0 + B_BASE + wave * NF * 1024);
    // Load number j of a k-tile; M0 must hold the base of its group of four (set_group).  256-wide tiles load A, then
    // B, narrow ones B first: the youngest loads are the ones with the longer lead (see Lds16).
    // The stage they go to: LS, and for narrow tiles wr_a, wr_b (LDS offsets).
    constexpr int B_FIRST = L::NARROW ? 0 : 8, A_FIRST = L::NARROW ? NF : 0;
    const auto is_b = [](int j) { return j >= B_FIRST && j < B_FIRST + NF; };
    const auto in_op = [](int j) { return j >= B_FIRST && j < B_FIRST + NF ? j - B_FIRST : j - A_FIRST; };
    uint32_t wr_a = 0, wr_b = 0;
    auto set_group = [&](auto ls_c, auto j_c) {
        constexpr int LS = decltype(ls_c)::value, j = decltype(j_c)::value, l = in_op(j);
        if constexpr (L::NARROW)
            set_m0((is_b(j) ? b_dst + wr_b : a_dst + wr_a) + (l >> 2) * 4096);
        else
            set_m0((is_b(j) ? b_dst : a_dst) + LS * HALF + (l >> 2) * 4096);
    };
    auto issue_load = [&](auto j_c, const unsigned char* ap, const unsigned char* bp) {
        constexpr int j = decltype(j_c)::value, l = in_op(j);
        if constexpr (!is_b(j))
            g2l16_m0<(l & 3) * 1024>(a_voff[l], ap);
        else
            g2l16_m0<(l & 3) * 1024>(b_voff[l], bp);
    };

    // ---- LDS -> fragments ---------------------------------------------------------------------------------
    const int f_swz = (l16 >> 1) & 7;
    lds_u8* a_rd[2];  // [k32-step]: row wm*128 + l16, chunk 4*ks + lq; fragment mi and the stage are immediates
    lds_u8* b_rd[NF];  // N x K B: [k32-step] (first two);  K x N B: [ni]
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) a_rd[ks] = lds + (wm * 128 + l16) * 128 + (((ks * 4 + lq) ^ f_swz) << 4);
    if (TRANSB) {
#pragma unroll
        for (int q = 0; q < NF; ++q)
            b_rd[q] = lds + B_BASE + (wn * 16 * NF + l16) * 128 + ((((q & 1) * 4 + lq) ^ f_swz) << 4);
    } else {
        // 16-lane block lq reads the 4(k) x 16(n) sub-tile at k = 8*lq + s/4 (+4 for the second half),
        // n = 16*ni + 4*(s%4), s = l16 (f of both is the same)
        const int k_l = 8 * lq + (l16 >> 2);
        const int f = kn_swz(k_l);
#pragma unroll
        for (int ni = 0; ni < NF; ++ni) {
            const int chunk = wn * 2 * NF + 2 * ni + ((l16 & 3) >> 1);
            b_rd[ni] = lds + B_BASE + k_l * (64 * NF) + ((chunk ^ f) << 4) + 8 * (l16 & 1);
        }
    }
    // Fragment read `op` of k32-step KS of stage S: 8 A fragments, then NF B fragments (N x K B) or 2 NF
    // transposing 8-byte reads (K x N B: the low halves of all fragments, then the high halves).
    constexpr int NRD = 8 + (TRANSB ? 1 : 2) * NF;
    static_assert(2 * NRD <= NSLOT, "a read every other slot");
    auto frag_op = [&](auto s_c, auto ks_c, auto op_c, raw16 (&af)[8], raw16 (&bf)[NF]) {
        constexpr int S = decltype(s_c)::value, KS = decltype(ks_c)::value, op = decltype(op_c)::value;
        constexpr int SO = L::NARROW ? 0 : S * HALF;  // (narrow tiles move the addresses from stage to stage)
        if constexpr (op < 8) {
            af[op] = lds_read16(a_rd[KS] + SO + op * 2048);
        } else if constexpr (TRANSB != 0) {
            bf[op - 8] = lds_read16(b_rd[KS] + SO + (op - 8) * 2048);
        } else {
            constexpr int ni = (op - 8) % NF, hi = (op - 8) / NF;
            const uint64_t v = lds_read_tr16_b64<SO + KS * 2048 * NF + hi * 256 * NF>(b_rd[ni]);
            bf[ni].w[2 * hi] = (uint32_t)v;
            bf[ni].w[2 * hi + 1] = (uint32_t)(v >> 32);
        }
    };

    // ---- fused A-side statistics (FUSED) ----------------------------------------------------------------
    // Both wavefronts of a wm pair hold the same A fragments; wavefront wn takes fragments 4*wn .. 4*wn+3.
    // sacc[t][j]: result tile of panel x fragment 4*wn + j, accumulated over the steps t (of four) of the folded
    // units: four short accumulation chains per row, added as a tree at the end, instead of one chain over all
    // steps (every MFMA rounds the running sum once; the chain was the largest term of the check's rounding
    // noise at sizes where one tile-column folds a whole row).  Lanes 0..15 hold (sum, dot_hi, dot_mid, dot_lo) of
    // row wm*128 + (4*wn + j)*16 + lane.
    f32x4_t sacc[4][4];
    MinMax16<T> mm[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int t = 0; t < 4; ++t) sacc[t][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        mm[j].init();
    }
    const lds_u8* const panel_rd = lds + L::PANEL + (l16 & 3) * 64 + lq * 16;
    const lds_u8* a_rd_st[2] = {a_rd[0] + wn * 8192, a_rd[1] + wn * 8192};
    // The statistics of k32-step KS of the tile in stage S (step t = 2S + KS of folded unit number hj) ride in the
    // slots of the k-step that runs while that tile is in LDS, instead of standing between
    // two k-steps with the matrix cores idle: the wavefront's four fragments and the panel fragment are read once
    // more from LDS in five early slots (the pipeline's own fragment registers are not touched), the panel rows
    // 4..15 are zeroed well ahead of their use (a vector write of an MFMA operand must not sit within a few slots of
    // the MFMA), the 16 fragment dwords fold into the max / min trackers one per slot (narrow tiles: two) in the last slots, when every
    // read of the step has been issued, and the four statistics MFMAs follow the step's last slot.
    raw16 st_x;
    raw16 st_a[4];
    auto stats_slot = [&](auto s_c, auto ks_c, auto slot_c, int hj) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value, KS = decltype(ks_c)::value, slot = decltype(slot_c)::value;
        if constexpr (slot == 3) st_x = lds_read16(panel_rd + hj * 1024 + (2 * S + KS) * 256);
        if constexpr (slot == 7 || slot == 11 || slot == 15 || slot == 19)
            st_a[(slot - 7) / 4] = lds_read16(a_rd_st[KS] + (L::NARROW ? 0 : S * HALF) + ((slot - 7) / 4) * 2048);
        constexpr int ZERO = NF == 8 ? 24 : 20, FPS = NF == 8 ? 1 : 2, FOLD = NSLOT - 16 / FPS;
        if constexpr (slot >= ZERO && slot < ZERO + 4) st_x.w[slot - ZERO] = l16 < 4 ? st_x.w[slot - ZERO] : 0u;
        if constexpr (slot >= FOLD)
            static_for<FPS * (slot - FOLD), FPS * (slot - FOLD + 1)>([&](auto d_c) {
                constexpr int d = decltype(d_c)::value;
                mm[d >> 2].fold(st_a[d >> 2].w[d & 3]);
            });
    };
    auto stats_mfma = [&](auto s_c, auto ks_c) __attribute__((always_inline)) {
        constexpr int S = decltype(s_c)::value, KS = decltype(ks_c)::value;
        // vector code wrote the panel fragment (see Mfma16x): the idle slots are tied to its final value
        u32x4_t xv = __builtin_bit_cast(u32x4_t, st_x);
        asm volatile("s_nop 4" : "+v"(xv));
        st_x = __builtin_bit_cast(raw16, xv);
        Mfma16x<T>::acc_v4(sacc[2 * S + KS], st_x, st_a);
    };

    // One k32-step = 8 NF slots of one MFMA (16 cycles, four issue cycles).  Even slots issue fragment read
    // slot/2 of the NEXT step (stage S, step KS, into the other register set).  LBASE is the step's first slot
    // within the tile body (0 or NSLOT): the loads of the next tile go into stage S^1.
    auto kstep = [&](auto s_c, auto ks_c, auto lbase_c, auto st_c, int hj, const raw16 (&af)[8], const raw16 (&bf)[NF],
                     raw16 (&naf)[8], raw16 (&nbf)[NF], const unsigned char* ap, const unsigned char* bp) {
        constexpr int S = decltype(s_c)::value, LBASE = decltype(lbase_c)::value;
        constexpr bool STATS = FUSED && decltype(st_c)::value != 0;
        if (!TRANSB) wait_lgkmcnt0();  // the assembly reads of (af, bf) issued during the previous step
        static_for<0, NSLOT>([&](auto slot_c) {
            constexpr int slot = decltype(slot_c)::value;
            constexpr int mi = slot / NF, ni = slot % NF;
            Mfma16x<T>::acc_a(acc[mi][ni], bf[ni], af[mi]);
            __builtin_amdgcn_sched_barrier(0);  // MFMA first, the rest of the slot in its shadow
            if constexpr ((slot & 1) == 0 && slot / 2 < NRD)
                frag_op(s_c, ks_c, std::integral_constant<int, slot / 2>{}, naf, nbf);
            // G: slot within the tile body (two steps); load j goes out at G = LOFF + j * LSTRIDE, the M0 of its
            // group of four one slot ahead of the group's first load
            constexpr int G = LBASE + slot;
            static_assert(LOFF >= 1 && LOFF + (NLOAD - 1) * LSTRIDE < 2 * NSLOT, "all loads inside the tile body");
            if constexpr (G + 1 >= LOFF && (G + 1 - LOFF) % LSTRIDE == 0 && (G + 1 - LOFF) / LSTRIDE < NLOAD) {
                constexpr int j = (G + 1 - LOFF) / LSTRIDE;
                if constexpr ((in_op(j) & 3) == 0) set_group(std::integral_constant<int, S ^ 1>{}, std::integral_constant<int, j>{});
            }
            if constexpr (G >= LOFF && (G - LOFF) % LSTRIDE == 0 && (G - LOFF) / LSTRIDE < NLOAD)
                issue_load(std::integral_constant<int, (G - LOFF) / LSTRIDE>{}, ap, bp);
            if constexpr (STATS) stats_slot(s_c, ks_c, slot_c, hj);
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (STATS) stats_mfma(s_c, ks_c);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using IStep = std::integral_constant<int, NSLOT>;

    if constexpr (CHAINS) {
        chain_reserve();
        static_for<0, 32 * NF>([&](auto i_c) { chain_clear<decltype(i_c)::value>(); });
    }
    const int nk = g.K / BK;
    raw16 af0[8], bf0[NF], af1[8], bf1[NF];
    // first tile; narrow tiles: and the second one's A (and B) where there is a stage for it
    static_for<0, L::A_STAGES - 1>([&](auto t_c) {
        constexpr int t = decltype(t_c)::value;
        const unsigned char* ap = uniform_ptr(a_base + (t < nk ? t : nk - 1) * (BK * 2));
        const unsigned char* bp = uniform_ptr(b_base + (t < nk ? t : nk - 1) * b_ktile);
        if constexpr (L::NARROW) {
            wr_a = t * HALF;
            wr_b = t * L::B_STAGE;
        }
        settle_bases(ap, bp);
        static_for<0, NLOAD>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value;
            if constexpr (is_b(j) && t >= L::B_STAGES - 1) return;
            if constexpr ((in_op(j) & 3) == 0) {
                set_group(I0{}, j_c);
                asm volatile("s_nop 0");
            }
            issue_load(j_c, ap, bp);
        });
    });
    int n_slots = 0;  // FUSED: number of k-units this tile-column folds
    if (FUSED) {
        // Panel cache: for slot j (unit u = bn + j*tiles_n), step t, k = 128u + 32t + q: rows
        // (1, Be_hi, Be_mid, Be_lo) of 32 k each.  Be is scaled by a
        // power of two sigma so that its pieces fit the input type's range (FP16); the dot product is scaled
        // back when it is published.
        const float* const Be = reinterpret_cast<const float*>(g.Be);
        const int nunits = nk >> 1;
        if (bn < nunits) {
            n_slots = (nunits - bn + g.tiles_n - 1) / g.tiles_n;
            n_slots = n_slots < L::SLOTS ? n_slots : L::SLOTS;
        }
        // the Be values of this thread (k = 128u + tid of every folded unit), all loads in flight together
        float bek[L::SLOTS];
#pragma unroll
        for (int j = 0; j < L::SLOTS; ++j)
            bek[j] = (j < n_slots && tid < 128) ? Be[128 * (bn + j * g.tiles_n) + tid] : 0.f;
        float* const s_scale = reinterpret_cast<float*>(smem + L::SCALE);
        // S1..S3 still in partials: every workgroup folds them here, under the latency of its first tile
        if (g.s_nparts) fold_s_partials_to_lds(g.s_partial, g.s_nparts, tid, reinterpret_cast<double*>(smem + L::S_RED));
        // sigma = 2^(exponent(max |Be|) - 13): |Be / sigma| < 2^14 (BF16 shares FP32's exponent range: sigma = 1)
        float inv_sigma = 1.f;
        if constexpr (std::is_same<T, f16_t>::value) {
            float m = 0.f;
#pragma unroll
            for (int j = 0; j < L::SLOTS; ++j) m = fmaxf(m, fabsf(bek[j]));
            m = wave_max(m);
            if (lane == 0) s_scale[wave] = m;
            __syncthreads();
            m = fmaxf(fmaxf(s_scale[0], s_scale[1]), fmaxf(s_scale[2], s_scale[3]));
            if (m > 0.f && m < 3.0e38f) inv_sigma = ldexpf(1.f, 13 - ilogbf(m));
        }
        uint16_t* const panel = reinterpret_cast<uint16_t*>(smem + L::PANEL);
#pragma unroll
        for (int j = 0; j < L::SLOTS; ++j) {
            if (j < n_slots && tid < 128) {
                uint16_t p[3];
                split3<T>(bek[j] * inv_sigma, p);
                uint16_t* dst = panel + (j * 4 + (tid >> 5)) * 128 + (tid & 31);
                dst[0] = one16<T>();
                dst[32] = p[0];
                dst[64] = p[1];
                dst[96] = p[2];
            }
        }
        if (tid == 0) s_scale[4] = 1.f / inv_sigma;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    // the very first step multiplies register set 1 before any tile has been read into it: zeros
#pragma unroll
    for (int i = 0; i < 8; ++i) af1[i] = raw16{{0u, 0u, 0u, 0u}};
#pragma unroll
    for (int i = 0; i < NF; ++i) bf1[i] = raw16{{0u, 0u, 0u, 0u}};
    asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");  // vector code wrote these operands: see Mfma16x

    // KSNAP: prefix row sums of the accumulator tile (section 5.2, K split as well).  Lane l owns C row l % 16 of
    // each of its 8 row fragments and 4 columns of each of the 8 column fragments: 32 values per row fragment,
    // added as a tree, then across the four lanes that share the row.  The two wavefronts of
    // a tile-column (wn = 0, 1) leave one partial each.  The assembly MFMAs are opaque to the compiler's hazard
    // handling, so idle slots let their results land first; outstanding LDS reads land before compiler-generated
    // code runs between two k-steps.
    int ksnap_idx = 0;
    auto snapshot = [&](int idx) __attribute__((always_inline)) {
        if constexpr (KSNAP) {
        wait_lgkmcnt0();
        settle_accumulators(acc);
        // (opaque to the optimiser, so that none of the address arithmetic below is hoisted out of this block and
        // kept in registers across the main loop)
        idx = __builtin_amdgcn_readfirstlane(idx);
        asm volatile("" : "+s"(idx));
        double tot[8];
#pragma unroll
        for (int mi = 0; mi < 8; ++mi) {
            // the lane's 32 values as a tree in FP32 (five roundings deep), then double across fragments' halves and
            // lanes: the prefixes of consecutive K-blocks are subtracted, so what is kept between kernels is double
            float q[8];
#pragma unroll
            for (int ni = 0; ni < 8; ++ni) q[ni] = (acc[mi][ni][0] + acc[mi][ni][1]) + (acc[mi][ni][2] + acc[mi][ni][3]);
            double s = (double)((q[0] + q[1]) + (q[2] + q[3])) + (double)((q[4] + q[5]) + (q[6] + q[7]));
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            tot[mi] = s;
            asm volatile("" : "+v"(tot[mi]));  // one row fragment at a time: keeps the live set small
        }
        if (lq == 0) {
            double* dst = g.kprefix + ((int64_t)idx * (2 * g.tiles_n) + 2 * bn + wn) * g.M + row0 + wm * 128 + l16;
#pragma unroll
            for (int mi = 0; mi < 8; ++mi) dst[mi * 16] = tot[mi];
        }
        }
    };

    // Body of k-tile kt (stage kt & 1), from barrier to barrier: step (kt-1, 1) multiplies register set 1 while
    // the fragments of (kt, 0) arrive in set 0, then step (kt, 0) multiplies set 0 while (kt, 1) arrives in set
    // 1.  The 16 loads of tile kt+1 (clamped at the last tile; the reload is harmless) go to the other stage,
    // whose last reads completed before the barrier that opened this body.  STATS: the tile belongs to a k-unit
    // this tile-column folds (unit u = kt/2, its steps t = 2*(kt&1), +1: the statistics read the tile itself, not
    // the pipeline's registers, so they are not one step behind).
    // Narrow tiles: A of tile kt+2 (and B, with three stages) goes out here, and the closing barrier leaves those loads in
    // flight; their stage is the one that tile kt-1 was read from.
    uint32_t rd_a = 0, rd_b = 0;  // narrow tiles: the stages that tile kt lies in
    const auto next_stage = [](uint32_t at, uint32_t bytes, uint32_t n) { return at + bytes == n * bytes ? 0u : at + bytes; };
    auto tile_body = [&](auto s_c, auto st_c, int kt, int hj) {
        constexpr bool STATS = decltype(st_c)::value != 0;
        const int kta = kt + L::A_STAGES - 1 < nk ? kt + L::A_STAGES - 1 : nk - 1;
        const int ktb = kt + L::B_STAGES - 1 < nk ? kt + L::B_STAGES - 1 : nk - 1;
        const unsigned char* ap = uniform_ptr(a_base + (int64_t)kta * (BK * 2));
        const unsigned char* bp = uniform_ptr(b_base + ktb * b_ktile);
        if constexpr (L::NARROW) {
            wr_a = rd_a == 0 ? (L::A_STAGES - 1) * HALF : rd_a - HALF;
            wr_b = rd_b == 0 ? (L::B_STAGES - 1) * L::B_STAGE : rd_b - L::B_STAGE;
            if constexpr (FUSED && STATS) {
                a_rd_st[0] = a_rd[0] + wn * 8192;
                a_rd_st[1] = a_rd[1] + wn * 8192;
            }
        }
        settle_bases(ap, bp);
        kstep(s_c, I0{}, I0{}, st_c, hj, af1, bf1, af0, bf0, ap, bp);   // step (kt-1, 1)
        kstep(s_c, I1{}, IStep{}, st_c, hj, af0, bf0, af1, bf1, ap, bp);  // step (kt, 0)
        if constexpr (L::NARROW) {
            asm volatile("" ::: "memory");
            // what this body sent out for tile kt+2 may be in flight: the youngest 8 (A) or 8 + NF (A and B) loads
            __builtin_amdgcn_s_waitcnt(0x70 | (L::B_STAGES == 3 ? 8 + NF : 8));  // vmcnt, lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const uint32_t na = next_stage(rd_a, HALF, L::A_STAGES), nb = next_stage(rd_b, L::B_STAGE, L::B_STAGES);
            const uint32_t da = na - rd_a, db = nb - rd_b;
            rd_a = na;
            rd_b = nb;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) a_rd[ks] = a_rd[ks] + (int)da;
#pragma unroll
            for (int q = 0; q < (TRANSB ? 2 : NF); ++q) b_rd[q] = b_rd[q] + (int)db;
        } else {
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
    };
    if (FUSED) {
        // Tiles are walked in units of two (so the stage parity stays a compile-time constant): plain units in
        // an inner loop, the folded unit between two such loops.  K is a multiple of 128 here (the host checks).
        const int nunits = nk >> 1;
        int hu = bn, hj = 0;
        int u = 0;
        for (;;) {
            const int stop = hu < nunits ? hu : nunits;
            for (; u < stop; ++u) {
                tile_body(I0{}, I0{}, 2 * u, 0);
                tile_body(I1{}, I0{}, 2 * u + 1, 0);
            }
            if (u >= nunits) break;
            tile_body(I0{}, I1{}, 2 * u, hj);
            tile_body(I1{}, I1{}, 2 * u + 1, hj);
            ++u;
            hu += g.tiles_n;
            ++hj;
        }
        if (!TRANSB) wait_lgkmcnt0();
#pragma unroll
        for (int mi = 0; mi < 8; ++mi)
#pragma unroll
            for (int ni = 0; ni < NF; ++ni) Mfma16x<T>::acc_a(acc[mi][ni], bf1[ni], af1[mi]);
    } else if constexpr (KSNAP) {
        // One loop nest per K-block: the plain loop over the block's k-tiles, then the fragment pipeline is drained
        // (the pending second step of the block's last tile is multiplied), the prefix is taken with no fragment
        // live, and the pipeline restarts on zeros like at the kernel's start (one idle step per K-block).  The
        // global -> LDS prefetch runs through: the next block's first tile is already on its way.
        int kt = 0;
        for (;;) {
            const int kt_end = kt + g.kblock_tiles < nk ? kt + g.kblock_tiles : nk;  // kblock_tiles is even
            for (; kt + 1 < kt_end; kt += 2) {
                tile_body(I0{}, I0{}, kt, 0);
                tile_body(I1{}, I0{}, kt + 1, 0);
            }
            if (kt < kt_end) {  // an odd tile count only in the last K-block
                tile_body(I0{}, I0{}, kt, 0);
                ++kt;
            }
            if (!TRANSB) wait_lgkmcnt0();
#pragma unroll
            for (int mi = 0; mi < 8; ++mi)
#pragma unroll
                for (int ni = 0; ni < NF; ++ni) Mfma16x<T>::acc_a(acc[mi][ni], bf1[ni], af1[mi]);
            if (kt >= nk) break;  // the last prefix is taken in the epilogue, behind the injector
            snapshot(ksnap_idx);
            ++ksnap_idx;
#pragma unroll
            for (int i = 0; i < 8; ++i) af1[i] = bf1[i] = raw16{{0u, 0u, 0u, 0u}};
            asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");  // vector code wrote these operands: see Mfma16x
        }
    } else {
        int kt = 0;
        if constexpr (CHAINS) {
            // the first three chains, of an even number of k-tiles; the last one goes on to the end
            const int per = (nk + 7) / 8 * 2;
            for (int stop = per; stop < nk; stop += per) {
                do {
                    chain_reserve();
                    tile_body(I0{}, I0{}, kt, 0);
                    tile_body(I1{}, I0{}, kt + 1, 0);
                    kt += 2;
                    // the last results land before the compiler may move an accumulator (24 of 2048 cycles)
                    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                } while (kt < stop);
                // (the fragments on their way land first, as in front of any vector code here)
                wait_lgkmcnt0();
                settle_accumulators(acc);
                static_for<0, 32 * NF>([&](auto i_c) {
                    constexpr int i = decltype(i_c)::value, mi = i / (4 * NF), ni = i / 4 % NF, r = i % 4;
                    chain_add<i>(acc[mi][ni][r]);
                    acc[mi][ni][r] = 0.f;
                    if constexpr (r == 3) {
                        asm volatile("" : "+a"(acc[mi][ni]));
                        chain_reserve();
                    }
                });
                asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");  // vector code wrote the accumulators: see Mfma16x
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        for (; kt + 1 < nk; kt += 2) {
            if constexpr (CHAINS) chain_reserve();
            tile_body(I0{}, I0{}, kt, 0);
            tile_body(I1{}, I0{}, kt + 1, 0);
        }
        if (kt < nk) tile_body(I0{}, I0{}, kt, 0);
        if constexpr (CHAINS) chain_reserve();
        if (!TRANSB) wait_lgkmcnt0();
#pragma unroll
        for (int mi = 0; mi < 8; ++mi)
#pragma unroll
            for (int ni = 0; ni < NF; ++ni) Mfma16x<T>::acc_a(acc[mi][ni], bf1[ni], af1[mi]);
    }
    if constexpr (CHAINS) chain_reserve();
    if constexpr (EDGE) {
        const int kt0 = nk * BK, klen = g.K - kt0;  // the k past the last whole tile: a multiple of 8, below 64
        if (klen > 0) {
            // registers -> stage 0 (its last reads completed before the loop's closing barrier), zero past K
            if constexpr (L::NARROW) {
                __builtin_amdgcn_s_waitcnt(0);  // the loop's last loads have landed, here and in the other wavefronts
                __syncthreads();
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) a_rd[ks] = a_rd[ks] - (int)rd_a;
#pragma unroll
                for (int q = 0; q < (TRANSB ? 2 : NF); ++q) b_rd[q] = b_rd[q] - (int)rd_b;
            }
            const raw16 z = {{0u, 0u, 0u, 0u}};
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                const int q = wave * 64 + (lane >> 3) + 8 * l;
                const int c = (lane & 7) ^ (lane >> 4) ^ (4 * (l & 1));  // chunk of 8 k at LDS position lane % 8
                const unsigned char* pa = A + ((int64_t)min(row0 + q, g.M - 1) * g.lda + kt0 + c * 8) * 2;
                *reinterpret_cast<raw16*>(smem + wave * 8192 + l * 1024 + lane * 16) = c * 8 < klen ? ld16(pa) : z;
                if (l >= NF) continue;
                raw16 vb;
                if (TRANSB) {
                    const int qb = wave * 8 * NF + (lane >> 3) + 8 * l;
                    const unsigned char* pb = B + ((int64_t)min(col0 + qb, g.N - 1) * g.ldb + kt0 + c * 8) * 2;
                    vb = c * 8 < klen ? ld16(pb) : z;
                } else {
                    const int kl = (l * 64 + lane) / (4 * NF), n = ((l * 64 + lane) % (4 * NF) ^ kn_swz(kl)) << 3;
                    const int k = wave * 16 + kl;
                    const unsigned char* pb = B + ((int64_t)(kt0 + k) * g.ldb + min(col0 + n, g.b_cols - 8)) * 2;
                    vb = k < klen ? ld16(pb) : z;
                }
                *reinterpret_cast<raw16*>(smem + B_BASE + wave * NF * 1024 + l * 1024 + lane * 16) = vb;
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            static_for<0, 2>([&](auto ks_c) {
                static_for<0, NRD>([&](auto op_c) { frag_op(I0{}, ks_c, op_c, af1, bf1); });
                wait_lgkmcnt0();
                // (the transposing reads are assembly: the fragments are tied behind the wait, and idle slots keep
                // whatever moved them clear of the MFMAs)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    u32x4_t x = __builtin_bit_cast(u32x4_t, af1[i]);
                    asm volatile("" : "+v"(x));
                    af1[i] = __builtin_bit_cast(raw16, x);
                }
#pragma unroll
                for (int i = 0; i < NF; ++i) {
                    u32x4_t x = __builtin_bit_cast(u32x4_t, bf1[i]);
                    asm volatile("" : "+v"(x));
                    bf1[i] = __builtin_bit_cast(raw16, x);
                }
                asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
                for (int mi = 0; mi < 8; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NF; ++ni) Mfma16x<T>::acc_a(acc[mi][ni], bf1[ni], af1[mi]);
                asm volatile("s_nop 7\n\ts_nop 7" ::: "memory");
                if constexpr (CHAINS) chain_reserve();
            });
            __syncthreads();  // the epilogue reuses the operand stages
        }
    }
    if constexpr (L::NARROW) {
        __builtin_amdgcn_s_waitcnt(0);  // the epilogue reuses the stages that the loop's last loads went to
        __syncthreads();
    }
    settle_accumulators(acc);
    if constexpr (CHAINS) chain_reserve();
    if constexpr (CHAINS)
        static_for<0, 32 * NF>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value, mi = i / (4 * NF), ni = i / 4 % NF, r = i % 4;
            acc[mi][ni][r] += chain_sum<i>();
            if constexpr (r == 3) {
                asm volatile("" : "+a"(acc[mi][ni]));
                chain_reserve();
            }
        });
    if constexpr (EDGE && MODE >= 1) {
        // columns past the end count as zero in the row sums, rows past it in the column sums
        if (col0 + TN > g.N || (CSUM && row0 + BM > g.M)) {
            static_for<0, 8>([&](auto mi_c) {
                static_for<0, NF>([&](auto ni_c) {
                    static_for<0, 4>([&](auto r_c) {
                        constexpr int mi = decltype(mi_c)::value, ni = decltype(ni_c)::value, r = decltype(r_c)::value;
                        const bool in = col0 + wn * (16 * NF) + ni * 16 + 4 * lq + r < g.N &&
                                        (!CSUM || row0 + wm * 128 + mi * 16 + l16 < g.M);
                        acc[mi][ni][r] = in ? acc[mi][ni][r] : 0.f;
                    });
                });
            });
        }
    }

    // ---- epilogue -------------------------------------------------------------------------------------------
    if constexpr (INJECT) gemm16x_inject<INJECT>(g, acc, row0, col0, wm, wn, l16, lq);
    if constexpr (KSNAP) snapshot(ksnap_idx);  // the last K-block's prefix is the whole row sum
    if (VERIFY) {
        float* red = reinterpret_cast<float*>(smem);                 // [2 wn][256 rows]
        float* sred = reinterpret_cast<float*>(smem + SRED_OFFSET);  // [4][256 rows]
        float* red2 = reinterpret_cast<float*>(smem + RED2_OFFSET);  // [2 wn][256 rows]
        float* cred = reinterpret_cast<float*>(smem + CRED_OFFSET);  // [2 wm][256 columns]
        if constexpr (WSUM)
            gemm16x_rowsums12_to_lds(acc, red, red2, col0, wm, wn, l16, lq);
        else
            gemm16x_rowsum_to_lds<NF>(acc, red, wm, wn, l16, lq);
        if constexpr (CSUM) gemm16x_colsum_to_lds(acc, cred, wm, wn, l16, lq);
        if (FUSED) {
            const float sigma = reinterpret_cast<const float*>(smem + L::SCALE)[4];
            // the four k-chunk lanes of a row hold partial (max, min); lanes 0..15 hold the panel's result
#pragma unroll
            for (int j = 0; j < 4; ++j) mm[j].merge_xor(16);
#pragma unroll
            for (int j = 0; j < 4; ++j) mm[j].merge_xor(32);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float mx, mn;
                mm[j].result(mx, mn);
                if (lq == 0) {
                    const int r = wm * 128 + (4 * wn + j) * 16 + l16;
                    const bool any = n_slots > 0;  // a tile-column beyond the last k-unit folds nothing
                    f32x4_t q;
#pragma unroll
                    for (int e = 0; e < 4; ++e) q[e] = (sacc[0][j][e] + sacc[1][j][e]) + (sacc[2][j][e] + sacc[3][j][e]);
                    sred[0 * BM + r] = q[0];
                    sred[1 * BM + r] = sigma * (q[1] + (q[2] + q[3]));
                    sred[2 * BM + r] = any ? mx : -3.402823466e+38f;
                    sred[3 * BM + r] = any ? mn : 3.402823466e+38f;
                }
            }
        }
        __syncthreads();
        const int gi = row0 + tid;
        float* rowpart = reinterpret_cast<float*>(g.rowpart);
        float* apart = reinterpret_cast<float*>(g.apart);
        float* rowpart2 = reinterpret_cast<float*>(g.rowpart2);
        if (!EDGE || gi < g.M) st_agent(rowpart + (int64_t)bn * g.M + gi, red[tid] + red[BM + tid]);
        if (WSUM && (!EDGE || gi < g.M)) st_agent(rowpart2 + (int64_t)bn * g.M + gi, red2[tid] + red2[BM + tid]);
        // column-sum partials are compared by a kernel of their own after this one: plain stores
        if (CSUM && (!EDGE || col0 + tid < g.N))
            reinterpret_cast<float*>(g.colpart)[(int64_t)bm * g.N + col0 + tid] = cred[tid] + cred[BN + tid];
        if (FUSED && (!EDGE || gi < g.M)) {
            float* ap = apart + (int64_t)bn * 4 * g.M + gi;
            st_agent(ap, sred[0 * BM + tid]);
            st_agent(ap + (int64_t)g.M, sred[1 * BM + tid]);
            st_agent(ap + 2 * (int64_t)g.M, sred[2 * BM + tid]);
            st_agent(ap + 3 * (int64_t)g.M, sred[3 * BM + tid]);
        }
        // block-wise check: the partials are all this kernel leaves; a later kernel compares them per block
        const bool partials_only = MODE == 5 || (MODE == 2 && g.block_mode);
        if (!partials_only)
            gemm_tile_row_check<WSUM, FUSED, EDGE>(g, smem, reinterpret_cast<const double*>(smem + L::S_RED), bm, gi, tid);
        __syncthreads();  // the store below reuses the LDS the reductions read
    }
    gemm16x_store_c<T, EDGE, NF>(g, acc, smem, row0, col0, lane, wm, wn, l16, lq);
}

// The A-side pass (Algorithm 1 for the rows of A) in workgroups of its own behind the tiles', on compute units that have no tile
// of the last round: `share` of the -g.fused_stats of a tile-row, a wavefront per row at a time.  An arrival of its tile-row.
template <typename T, bool EDGE> __device__ __forceinline__ void gemm16_stats(const GemmArgs& g, int bm, int share) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, w = -g.fused_stats;
    double* const s_red = reinterpret_cast<double*>(smem);
    const bool fold = g.s_nparts != 0;
    if (fold) {
        fold_s_partials_to_lds(g.s_partial, g.s_nparts, tid, s_red);
        __syncthreads();
        if (bm == 0 && share == 0 && tid < 3 && g.S) g.S[tid] = folded_s(s_red, tid);
    }
    const double S1 = fold ? folded_s(s_red, 0) : g.S[0], S2 = fold ? folded_s(s_red, 1) : g.S[1],
                 S3 = fold ? folded_s(s_red, 2) : g.S[2];
    const int rows = (256 + w - 1) / w, first = bm * 256 + share * rows, end = min(min(first + rows, bm * 256 + 256), g.M);
    for (int m = first + wave; m < end; m += 4) {
        const char* const row = reinterpret_cast<const char*>(g.A) + (int64_t)m * g.lda * 2;
        const RowSums<float> r = row_sums<T, false, 4>(row, g.K, lane, reinterpret_cast<const float*>(g.Be), nullptr);
        if (lane == 0) {
            double mu;
            const float t = (float)row_threshold(r, g.K, g.N, S1, S2, S3, g.e_max, g.c_sigma, mu);
            float* const astat = reinterpret_cast<float*>(g.astat) + 3 * (int64_t)m;
            astat[0] = r.mx;
            astat[1] = r.mn;
            astat[2] = (float)mu;
            st_agent(reinterpret_cast<float*>(const_cast<void*>(g.expected)) + m, r.dot);
            st_agent(reinterpret_cast<float*>(const_cast<void*>(g.T)) + m, t);
        }
    }
    gemm_tile_row_check<false, false, EDGE>(g, smem, nullptr, bm, bm * 256 + tid, tid);
}

template <typename T, int TRANSB, int MODE, bool FUSED, bool EDGE, int NF, bool CHAINS = false>
__global__ __launch_bounds__(256) void gemm16_fast_kernel(const GemmArgs g) {
    if constexpr (MODE == 1 && !FUSED && !CHAINS) {
        const int behind = (int)blockIdx.x - g.tiles_m * g.tiles_n;
        if (behind >= 0) {
            gemm16_stats<T, EDGE>(g, behind / -g.fused_stats, behind % -g.fused_stats);
            return;
        }
    }
    int bm, bn;
    tile_of_block(blockIdx.x, g.tiles_m, g.tiles_n, bm, bn);
    gemm16_fast_tile<T, TRANSB, MODE, FUSED, EDGE, NF, CHAINS>(g, bm, bn, bm * 256, bn * 32 * NF);
}

template <typename KERN> static int gemm16_start(KERN kern, const GemmArgs& a, size_t lds, bool& attr_set, hipStream_t st) {
    if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return VABFT_EDEVICE;
        attr_set = true;
    }
    const int behind = a.fused_stats < 0 ? -a.fused_stats * a.tiles_m : 0;
    kern<<<dim3(a.tiles_m * a.tiles_n + behind), dim3(256), lds, st>>>(a);
    return hipGetLastError() == hipSuccess ? VABFT_OK : VABFT_EDEVICE;
}

// form: see Form16; the tile's width is 256, 192 or 128
template <typename T, int TRANSB>
static int gemm16_fast_launch_tb(const GemmArgs& a, int mode, int form, hipStream_t st) {
    const int fused = a.fused_stats > 0 ? 1 : 0;
    const auto bytes = [&](auto l) { return (size_t)(fused ? decltype(l)::BYTES_FUSED : decltype(l)::BYTES); };
    using g16x::Lds16;
    const size_t lds = form >= FORM16_128 ? bytes(Lds16<4>{}) : form == FORM16_192 ? bytes(Lds16<6>{}) : bytes(Lds16<8>{});
#define VABFT_G16F_CASE(VF, FU, FORM, ...)                \
    if (mode == VF && fused == FU && form == FORM) {      \
        static bool attr_set = false;                     \
        return gemm16_start(__VA_ARGS__, a, lds, attr_set, st); \
    }
#define VABFT_G16F_WHOLE(VF, FU) VABFT_G16F_CASE(VF, FU, FORM16_WHOLE, gemm16_fast_kernel<T, TRANSB, VF, FU != 0, false, 8>)
#define VABFT_G16F_EDGE(VF, FU)                                                                         \
    VABFT_G16F_WHOLE(VF, FU)                                                                            \
    VABFT_G16F_CASE(VF, FU, FORM16_EDGE, gemm16_fast_kernel<T, TRANSB, VF, FU != 0, true, 8>)
#define VABFT_G16F_SIZES(VF, FU)                                                                        \
    VABFT_G16F_EDGE(VF, FU)                                                                             \
    VABFT_G16F_CASE(VF, FU, FORM16_192, gemm16_fast_kernel<T, TRANSB, VF, FU != 0, true, 6>)           \
    VABFT_G16F_CASE(VF, FU, FORM16_128, gemm16_fast_kernel<T, TRANSB, VF, FU != 0, true, 4>)
    VABFT_G16F_SIZES(0, 0)
    VABFT_G16F_SIZES(1, 0)
    VABFT_G16F_CASE(0, 0, FORM16_128_CHAINS, gemm16_fast_kernel<T, TRANSB, 0, false, true, 4, true>)
    VABFT_G16F_CASE(1, 0, FORM16_128_CHAINS, gemm16_fast_kernel<T, TRANSB, 1, false, true, 4, true>)
    VABFT_G16F_SIZES(1, 1)
    VABFT_G16F_WHOLE(2, 0)
    VABFT_G16F_EDGE(3, 0)
    VABFT_G16F_EDGE(4, 0)
    VABFT_G16F_EDGE(5, 0)
    VABFT_G16F_WHOLE(6, 0)
    VABFT_G16F_WHOLE(7, 0)
    VABFT_G16F_WHOLE(2, 1)
#undef VABFT_G16F_SIZES
#undef VABFT_G16F_EDGE
#undef VABFT_G16F_WHOLE
#undef VABFT_G16F_CASE
    return VABFT_EINVAL;
}

}  // namespace vabft
