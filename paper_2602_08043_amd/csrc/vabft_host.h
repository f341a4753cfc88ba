// Host-side declarations shared by the translation units of libvabft.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "vabft.h"

namespace vabft {

// encode.hip
size_t encode_workspace_bytes(const vabft_problem* p);
int s_partial_count(const vabft_problem* p);  // per-workgroup partials of S1..S3 an encode leaves: [count][3] double
// d_Be2 / d_expected2 may be null (no position-weighted checksum); d_S null: S1..S3 stay as partials in s_partial
int encode_dispatch(const vabft_problem* p, const void* dB, void* d_Be, void* d_Be2, void* d_bstat, double* d_S,
                    double* s_partial, void* ws, int32_t* ticket, hipStream_t st);
// folds the partials an encode left into S[3] (the same fixed order the encode itself uses)
void fold_s_launch(const double* s_partial, int count, double* S, hipStream_t st);
int threshold_dispatch(const vabft_problem* p, const void* dA, const void* d_Be, const void* d_Be2, const double* d_S,
                       double e_max, double c_sigma, void* d_astat, void* d_expected, void* d_expected2, void* d_T,
                       hipStream_t st);
// column checksums (c1 A, per-column thresholds)
size_t cols_workspace_bytes(const vabft_problem* p);
int encode_a_dispatch(const vabft_problem* p, const void* dA, void* d_eA, void* d_acolstat, double* d_SA,
                      double* s_partial, void* ws, int32_t* ticket, hipStream_t st);
int threshold_cols_dispatch(const vabft_problem* p, const void* dB, const void* d_eA, const double* d_SA, double e_max,
                            double c_sigma, void* d_bcolstat, void* d_expected_col, void* d_Tcol, void* ws,
                            hipStream_t st);
// blocks.hip: block-wise verification
int block_width(int dtype);
size_t blocks_workspace_bytes(const vabft_problem* p);
int encode_blocks_dispatch(const vabft_problem* p, const void* dB, void* d_Be_blk, double* d_S_blk, void* ws,
                           hipStream_t st);
int threshold_blocks_dispatch(const vabft_problem* p, const void* dA, const void* d_Be_blk, const double* d_S_blk,
                              double e_max, double c_sigma, void* d_astat, void* d_expected_blk, void* d_T_blk,
                              hipStream_t st);
int finalize_blocks_dispatch(const vabft_problem* p, const void* rowpart, const void* d_expected_blk,
                             const void* d_T_blk, void* d_rowsum_blk, void* d_E_blk, int32_t* d_blockflags, void* d_E,
                             int32_t* d_flags, int32_t* d_nflag, int32_t* d_nblockflag, int sub, int nparts,
                             hipStream_t st);
int finalize_blocks_k_dispatch(const vabft_problem* p, int nkb, const double* kprefix, const void* d_expected_blk,
                               const void* d_T_blk, void* d_rowsum_blk, void* d_E_blk, int32_t* d_blockflags,
                               void* d_E, int32_t* d_flags, int32_t* d_nflag, int32_t* d_nblockflag, hipStream_t st);
int check_offline_dispatch(const vabft_problem* p, const void* dC, const void* d_expected, const void* d_T,
                           void* d_rowsum, void* d_E, int32_t* d_flags, int32_t* d_nflag, hipStream_t st);

// gemm*.hip
struct InjectArgs {
    int32_t mode;
    int32_t bit_lo, bit_span;
    int32_t n_list;
    uint64_t seed;
    uint64_t hit_limit;  // floor(rate * 2^53)
    const int32_t* d_list;
    int32_t log_capacity;
    vabft_inject_rec* d_log;
    int32_t* d_ninj;
};

// a weighted call of a direct kernel, in the injector's place (which is off): what its A-side pass forms too, and, with
// DirectArgs::wsum == 2, what the localisation of flagged rows writes
struct WeightedArgs {
    int32_t mode;      // InjectArgs::mode: 0
    int32_t correct;
    const void* Be2;   // [K] acc
    void* expected2;   // [M] acc
    int32_t* loc;      // [M]
    void* delta;       // [M] acc
    int32_t* ncorrected;
};

struct GemmArgs {
    const void* A;
    const void* B;
    void* C;
    int32_t M, N, K;
    int64_t lda, ldb, ldc;
    int32_t tiles_m, tiles_n;
    void* rowpart;    // [tiles_n][M] acc: per-tile-column partial row sums
    int32_t* d_nflag; // number of flagged rows
    union {
        InjectArgs inj;
        WeightedArgs w;
    };
    // in-kernel compare-and-flag (whole-tile kernels): the last workgroup to finish a
    // tile-row combines the partials of that row block
    const void* expected;  // [M] acc: input, or output when fused_stats
    const void* T;         // [M] acc: input, or output when fused_stats
    void* rowsum;          // [M] acc
    void* E;               // [M] acc
    int32_t* flags;        // [M]
    int32_t* tickets;      // [tiles_m] arrival counters, then (8-byte aligned) one 64-bit word:
                           // finished row blocks << 32 | flagged rows; all zero between launches
    int32_t ticket_stride; // int32 from one tile-row's arrival counter to the next
    // fused A-side statistics (Algorithm 1 for the rows of A, inside the GEMM).  Tiled kernels: 1 on the operand tiles, -w in w
    // workgroups per tile-row of their own, the launch's last
    int32_t fused_stats;
    const void* Be;   // [K] acc
    double* S;        // [3]; with s_nparts > 0 an output, or null: the sums are folded from s_partial
    const double* s_partial;  // [s_nparts][3], left by an encode with a deferred fold
    int32_t s_nparts;
    double e_max, c_sigma;
    void* astat;      // [M][3] acc, output
    void* apart;      // [tiles_n][4][M] acc: per-K-slice (sum, dot, max, min) of the rows of A (fused_stats)
    // position-weighted row sums C r2 (kernel modes 2 and 3)
    void* rowpart2;   // partials, same shape as rowpart
    void* rowsum2;    // [M] acc, output; may be null
    // column sums c1 C (kernel modes 2 and 4): [tiles_m][N] acc partials
    void* colpart;
    int32_t* d_ncolflag;  // zeroed by the GEMM kernel for the column compare that follows it; may be null
    // block-wise check: the kernels only leave their partial row sums; a kernel of its own compares per block
    int32_t block_mode;
    int32_t* d_nblockflag;  // block mode: zeroed (with d_nflag) by the GEMM kernel for the compare that follows
    // block-wise check with K split as well (kernel modes 6 and 7 of the 16-bit whole-tile kernel): the row sums of
    // the accumulator tile taken every kblock_tiles k-tiles, in double
    double* kprefix;        // [K-blocks][2 * tiles_n][M]: prefix row sums (one per wavefront column of a tile-column)
    int32_t kblock_tiles;   // k-tiles (of 64) per K-block; even
    int32_t b_cols;  // elements that a row of B holds (16-bit tiled kernels, B stored K x N): N, in a copy more
};

size_t gemm_workspace_bytes(const vabft_problem* p);
struct FusedArgs {  // non-null d_Be selects the fused A-side path
    const void* d_Be;
    const double* d_S;  // null: S1..S3 are still the partials of the preceding encode,
    double* d_S_out;    // and what they fold to is wanted here (may be null)
    double e_max, c_sigma;
    void* d_astat;
    const WeightedArgs* w = nullptr;  // a weighted call that localises (and corrects) behind the check
};
// d_rowsum2 non-null selects the kernels that also form the position-weighted row sums; cols non-null those
// that also form the column sums and compares them
struct BlockArgs {
    const void* d_expected_blk;  // [nblocks][M] acc
    const void* d_T_blk;         // [nblocks][M] acc
    void* d_rowsum_blk;          // [nblocks][M] acc
    void* d_E_blk;               // [nblocks][M] acc
    int32_t* d_blockflags;       // [nblocks][M]
    int32_t* d_nblockflag;       // [1]
    // K split as well: kblock > 0, every array above is [K-blocks][nblocks][M], kprefix as in GemmArgs
    int32_t kblock = 0;
    double* kprefix = nullptr;
};
struct ColArgs {
    const void* d_expected_col;  // [N] acc
    const void* d_Tcol;          // [N] acc
    void* d_colsum;              // [N] acc
    void* d_Ecol;                // [N] acc
    int32_t* d_colflags;         // [N]
    int32_t* d_ncolflag;         // [1]
};
// pack.hip: copies of operands in the tiled kernels' layout
struct PackArgs {
    const void* src;
    void* dst;               // null: nothing to do
    int32_t rows, len;       // of the matrix
    int64_t ld;
    int32_t rows_out, pitch; // of the copy: rows (zeros behind the matrix's), elements from row to row (a multiple of 64)
    int32_t block_rows, blocks;  // set by pack_dispatch
};
// a, b: the copies of A and B.  fused: with the A-side pass (over all of A, whether a copies it or not).
int pack_dispatch(int dtype, const PackArgs& a, const PackArgs& b, const FusedArgs* fused, const double* s_partial,
                  int s_nparts, int N, void* d_expected, void* d_T, hipStream_t st);
int gemm_dispatch(const vabft_problem* p, const void* dA, const void* dB, void* dC, void* d_expected, void* d_T,
                  int verify, const FusedArgs* fused, const vabft_inject* inj, void* d_rowsum, void* d_rowsum2,
                  void* d_E, int32_t* d_flags, int32_t* d_nflag, vabft_inject_rec* d_injlog, int32_t* d_ninj,
                  void* ws, size_t ws_bytes, hipStream_t st, const ColArgs* cols = nullptr,
                  const BlockArgs* blocks = nullptr);
void workspace_init_launch(void* ws, size_t bytes, hipStream_t st);

// gemm_direct.h: workgroup tiles of 16 x 32 (K x N B: 16 x 64), 32 x 32 (32 x 64), 32 x 64 (ANY: rows of any length and
// distance) and 64 x 64, K shared by the wavefronts; four wavefronts side by side with 32 x 64 or 64 x 64 each
enum DirectShape { DIRECT_NONE = -1, DIRECT_16 = 0, DIRECT_32 = 1, DIRECT_32W = 2, DIRECT_ANY = 3, DIRECT_64 = 4,
                   DIRECT_OWN32 = 5, DIRECT_OWN64 = 6 };
struct DirectArgs {
    GemmArgs g;
    int8_t verify, wsum, csum;   // the check; with position-weighted row sums (2: localisation too); with column sums
    int8_t mirror;               // 0: the A-side pass's are the launch's first workgroups; -1: its last, the order being reversed
    int32_t stat_blocks;         // > 0: that many workgroups run that pass,
    int16_t stat_rows;           // of so many rows each: one, two or four per wavefront
    int16_t split;               // workgroups that share the K of a tile (> 1: g.apart holds [tile][split] tiles of
                                 // accumulator words, and an arrival counter per tile lies behind the tile-rows')
    int32_t first_block;         // of this launch (set by the launcher)
    int32_t tile_blocks;         // workgroups of the tiles, tiles_m * tiles_n * split
};
// The workgroup's size, which the compare at a launch's end asks for, lies 12 bytes behind the record: in the record's last
// cache line up to here.  16 bytes more were a fetch of another one there, 0.06 us of every short call's 7.
static_assert(sizeof(DirectArgs) <= 0x168, "");
int gemm_direct_launch_bf16(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_f16(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_f8(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_bf8(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_f32(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_f64(const DirectArgs& d, int shape, int transB, hipStream_t st);
// with position-weighted row sums (DirectArgs::wsum)
int gemm_direct_launch_w_bf16(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_w_f16(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_w_f8(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_w_bf8(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_w_f32(const DirectArgs& d, int shape, int transB, hipStream_t st);
int gemm_direct_launch_w_f64(const DirectArgs& d, int shape, int transB, hipStream_t st);

// per-dtype launchers (one translation unit each, to compile in parallel)
// mode: 0 plain, 1 check, 2 check + injector + weighted row sums + column sums, 3 check + weighted row
// sums, 4 check + column sums, 5 row-sum partials only (block-wise check), 6 prefix row sums per K-block, 7 the same with
// the injector.
// form (16-bit types): whole 256 x 256 tiles; the same for sizes that are no multiples of them (modes 0, 1 and 3 to 5);
// tiles of 256 rows and 192 or 128 columns (any size, modes 0 and 1), the last also with K in four chains (copied operands).
// The kernels do the compare-and-flag step themselves and, with GemmArgs::fused_stats, the A-side statistics and
// thresholds.
// k-units of 128 that the fused 16-bit kernels fold per tile-column at most (256-wide tiles alone; with narrow ones)
constexpr int PANEL_UNITS_WIDE = 16, PANEL_UNITS_NARROW = 15;
enum Form16 { FORM16_WHOLE = 0, FORM16_EDGE = 1, FORM16_192 = 2, FORM16_128 = 3, FORM16_128_CHAINS = 4 };
int gemm16_launch_bf16_nn(const GemmArgs& a, int mode, int form, hipStream_t st);
int gemm16_launch_bf16_nt(const GemmArgs& a, int mode, int form, hipStream_t st);
int gemm16_launch_f16_nn(const GemmArgs& a, int mode, int form, hipStream_t st);
int gemm16_launch_f16_nt(const GemmArgs& a, int mode, int form, hipStream_t st);
int gemm8_launch_f8_nt(const GemmArgs& a, int mode, hipStream_t st);   // E4M3, whole tiles only
int gemm8_launch_bf8_nt(const GemmArgs& a, int mode, hipStream_t st);  // E5M2, whole tiles only

}  // namespace vabft
