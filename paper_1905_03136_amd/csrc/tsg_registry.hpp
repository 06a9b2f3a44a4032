// tsg_registry.hpp -- host-side description of the generated kernel variants.
// The code generator emits one Variant record (and one launcher) per
// instantiated kernel; the runtime picks a record for each call.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsg {

// Arguments of one launch.  For TSMTTSM, X/ldx is B and Y/ldy is C; for TSMM,
// X/ldx is C and Y/ldy is B.
struct Launch {
    hipStream_t stream;
    int grid;
    int64_t K;
    int M, N;
    int conj;
    int opc;  // TSMM small operand: 0 C, 1 C^T, 2 C^H
    const void* A;
    int64_t lda;
    const void* X;
    int64_t ldx;
    void* Y;
    int64_t ldy;
    double alpha, beta;
    double* ws;  // TSMTTSM: one slot of M*N (x2 complex) doubles per block
    size_t lds;  // bytes of LDS of a block, for kernels that size it at run time
    unsigned* arrived;  // TSMTTSM: counter of the blocks, zero (null: the slots are summed by another kernel)
};

enum OpKind { OP_TSMTTSM = 0, OP_TSMM = 1 };

struct Variant {
    int op;             // OpKind
    int dt;             // tsg_dtype of the tall matrices
    int M, N;           // exact widths served, or 0 for a run-time-width variant
    int maxM, maxN;     // largest widths served (run-time-width variants)
    int pairA;          // needs 16-byte paired loads of A (even lda, aligned A)
    int pairX;          // TSMTTSM: paired loads of B; TSMM: paired stores of B
    int evenW;          // run-time-width variant that needs even widths (paired access)
    int threads;        // block size
    int rows_per_tile;  // rows consumed by one block per grid-stride iteration (for P = 1)
    int pack;           // row packing: 0 none, 1 P = 16 / max(M, N) (TSMTTSM), 2 P = 16 / N (TSMM)
    int flatA;          // reads the tall operands as runs of rows: needs lda == M (TSMTTSM: and ldb == N)
    int readB;          // TSMM reading the old B with A (serves only calls with beta != 0)
    int align16;        // needs A and X 16-byte aligned (direct 16-byte loads into LDS)
    const char* name;
    const void* (*kernel)(); // device function, for occupancy queries
    void (*launch)(const Launch&);
    // TSMTTSM with the rows staged in LDS by direct loads, run-time widths:
    // 1 for any two matrices, 2 for a matrix with itself; serves the widths
    // whose 16-column blocks (wider matrix) and 4-column groups (narrower one)
    // are exactly maxM / 16 and maxN / 4 (0: not such a kernel)
    int stage;
    int stages;         // its stages in LDS
    int gauss;          // it forms complex products from three real ones
    int fold;           // LDS bytes of its sum over row groups
    // TSMM of one small tile a wave (run-time widths): rows of a wave's tile
    // (0: not such a kernel), LDS bytes of its copy of C
    int once;
    int once_c;
    int once_db;  // two tiles of a wave in LDS, persistent blocks
    int once_m, once_n;  // it serves widths above these: those of the next smaller class, or nearer
    // the calls for which no other kernel was faster by more than 5% (1% at its
    // largest widths; timings differ by as much from run to run): 1 beta = 0,
    // 2 beta = 0 and its largest widths, 4 and 8 the same for beta != 0
    int once_for;
    int sums;  // TSMTTSM: takes Launch.arrived
};

// LDS bytes of a block of the staged kernel: NS stages of RT rows of both
// matrices in whole 1 KB pieces (sym: of one matrix), and 1 KB past the last,
// where the operand reads of columns past a width may reach; at least `fold`
// bytes, which the sum over row groups takes after the last stage.
inline size_t stage_lds_bytes(int wide, int narrow, size_t es, int RT, int NS, bool sym, size_t fold)
{
    const size_t x = (wide * es * RT + 1023) / 1024, y = sym ? 0 : (narrow * es * RT + 1023) / 1024;
    const size_t b = (x + y) * 1024 * NS + 1024;
    return b > fold ? b : fold;
}

// LDS bytes of a wave of the one-tile kernel: the tile's rows of A, then of B,
// in pieces of 1 KB 16 bytes apart (and room for reads of columns past a
// width); with beta != 0 the old rows of B too.
inline size_t once_wave_bytes(int M, int N, size_t es, int rows, bool beta_nz)
{
    const size_t a = (M * es * rows + 1023) / 1024 * 1040, b = (N * es * rows + 1023) / 1024 * 1040;
    return (a > b ? a : b) + 256 + (beta_nz ? b + 256 : 0);
}

extern const Variant kVariants[];
extern const int kNumVariants;

// Batched orthogonalisation parameters chosen by the autotuner (generated):
// input bytes per slab under automatic sizing, and the queue interleave
// (instances between an instance's slab items and its update items; 0: every
// slab item before any update item).
extern const int64_t kOrthItemBytes;
extern const int kOrthLag;

}  // namespace tsg
