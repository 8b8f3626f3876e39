// Tiled MFMA GEMM used by every dense contraction of the training step.
#pragma once
#include <hip/hip_runtime.h>

namespace blstm {

enum DType { DT_F32 = 0, DT_BF16 = 1 };

// One (A, B) operand pair contributing  sum_k A(m,k) * B(n,k)  to C(m,n).
//   A(m,k) = atrans ? A[k*lda + m] : A[m*lda + k]
//   B(n,k) = btrans ? B[k*ldb + n] : B[n*ldb + k]
// sA/sB are element strides added per batch index (blockIdx.z); they may be negative.
struct GemmSeg {
    const void* A;
    const void* B;
    long long lda, ldb, sA, sB;
    int K;
};

struct GemmDesc {
    GemmSeg seg[2];
    int nseg;                 // 1 or 2; both segments accumulate into the same C tile
    void* C;                  // [M][N] row-major, leading dimension ldc, element type out_type
    long long ldc, sC;
    const void* bias;         // per column n, element type in_type, or null
    long long sBias;
    const float* add;         // float [M][N] added to the product, or null
    long long ldadd, sAdd;
    float* rowsum;            // rowsum[m] = sum_k A(m,k) of segment 0 (bias gradients), or null
    long long sRowsum;
    float* partial;           // scratch for split-K partial tiles (float), or null: never split
    size_t partial_bytes;
    int M, N, batch;
    int Npad;                 // 0, or a multiple of the tile width >= N up to which B(n, .) may be read (it holds zeros or
                              // anything there): the product runs on whole tiles, C keeps its N columns
    bool a_pad;               // rows of A (as they lie in memory) may be read up to the next 16-byte boundary and hold finite values there
    bool c_pad;               // rows of C may be written up to the next multiple of eight columns
    bool long_parts;          // K is split, if at all, into parts of at least eight slabs (see make_plan)
    bool guarded_parts;       // K is split as the guarded kernel takes it (set by launch_gemm where that runs; by the caller for a product
                              // that has to give the bits of one on unaligned operands)
    bool atrans, btrans;
    DType in_type, out_type;  // in_type is the element type of A and B
};

// How a product is run: the tile shape, and into how many K ranges it is split.
enum GemmTile { GEMM_TILE_128 = 0,        // 128x128, every element type and shape
                GEMM_TILE_256 = 1,        // 256x256, bf16, few tiles and a long contraction
                GEMM_TILE_256X128 = 2,    // 256x128, bf16
                GEMM_TILE_64 = 3,         // 64x64, where larger tiles leave CUs idle or fill them unevenly
                GEMM_TILE_128X64 = 4,     // 128x64, bf16: too many tiles for 64x64, too few for 128x128
                GEMM_TILE_128S = 5,       // 128x128 with one LDS buffer, bf16, short contractions
                GEMM_TILE_RESIDENT = 6 }; // a workgroup keeps 128 columns' weights and walks down the rows, bf16, contractions of up to 256
struct GemmPlan {
    int tile;                 // a GemmTile
    bool deep;                // bf16 dA^T X, 128x128 tile with the loads further ahead (launches of at most one workgroup per CU)
    int splits;
    size_t partial_bytes;     // scratch the split needs (0 when splits == 1)
};
// Scratch bytes a product of this shape would use if it were given unlimited scratch.
size_t gemm_partial_bytes(int M, int N, int K, int batch, DType in_type, bool long_parts = false);
// The scratch softmax_xent_fwd_bwd_noalloc sets aside for one of its products when it decides whether a call fits.
size_t noalloc_partial_bytes(int M, int N, int K, DType in_type);

// Validates nothing (the caller's shapes are trusted); returns the launch status.
hipError_t launch_gemm(const GemmDesc& d, hipStream_t stream);
// n independent products of the A^T B form (atrans and btrans, operands of one type, float result, optional row sums, no
// bias, one segment): those the grouped kernel can take (gemm_group_ok) in one launch, which never splits along K, the others one
// by one.  So may the former be where they are faster split, each in its descriptor's scratch.
bool gemm_group_ok(const GemmDesc* d, int n);
hipError_t launch_gemm_group(const GemmDesc* d, int n, hipStream_t stream);

}  // namespace blstm
