// Launchers of the non-GEMM kernels.  All pointers are device pointers unless said otherwise.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include "gemm.hpp"

namespace blstm {

constexpr int BLSTM_MAX_PAIRS = 32;                  // pairs of one matching (64 replicas)
constexpr int BLSTM_MAX_REPLICA_PTRS = 64;           // replicas of one average (equals BLSTM_MAX_REPLICAS of the C header)

// ---- LSTM cell, one visited frame of both directions ---------------------------------
// Index d = direction.  Row strides are in elements.
struct CellFwdArgs {
    const float* pre[2];      // pre-activations a = W_x x + U_h h_prev + b, [B][4H] rows of stride ld_pre
    long long ld_pre;
    const float* c_prev[2];   // [B][H] rows of stride 2H, or null at the first visited frame
    float* c[2];              // [B][H] rows of stride 2H
    void* gates[2];           // activations i,f,g,o: [B][4H] rows of stride 8H (storage type)
    void* y[2];               // h: [B][H] rows of stride 2H (storage type)
    int B, H;
};
hipError_t launch_cell_fwd(const CellFwdArgs& a, DType store, hipStream_t s);

struct CellBwdArgs {
    const void* dy[2];        // dE/dh from the layer above, rows of stride 2H (storage type)
    const float* dh_rec[2];   // [B][H] contiguous, or null at the last visited frame
    float* dc_rec[2];         // [B][H] contiguous, read (unless first != 0) and overwritten
    const void* gates[2];     // rows of stride 8H
    const float* c[2];        // rows of stride 2H
    const float* c_prev[2];   // rows of stride 2H, or null at the first visited frame
    void* da[2];              // dE/da: [B][4H] rows of stride 8H (storage type)
    int B, H;
    int first;                // != 0: dc_rec is taken as zero (last visited frame)
};
hipError_t launch_cell_bwd(const CellBwdArgs& a, DType store, hipStream_t s);

// ---- persistent recurrent kernels (bf16 storage, H a multiple of 8 up to 1024) -------------------
struct RecFwdArgs {
    const unsigned short* uh[2];  // U_h per direction, [4H][H]
    const float* ax;              // W_x x + b for every frame, [M][8H]
    unsigned short* y;            // layer output h, [M][2H]
    unsigned short* z;            // the same once more, or null (honoured by launch_rec_small_fwd only)
    unsigned short* hx;           // h again in exchange order, [T][2][tiles][H/16][2][32][8]; pre-filled with 0xFFFF in sentinel mode
    unsigned short* gates;        // gate activations for rec_bwd_kernel only, as per-lane records [T][2][tiles][H/32][2][256] 16-byte words (not the per-frame path's [M][8H])
    float* c;                     // cell states, records [T][2][tiles][H/32][256] of four floats; both sized for whole 32-row tiles
    unsigned* cnt;                // [2*nbg][tiles_per_group] counters, zero before the launch
    unsigned* abort_word;         // raised when a wait ran out of time
    unsigned long long limit_ticks;   // wait limit in ticks of the 100 MHz wall clock
    // fill_words 16-byte words at `fill` are set to 0xFF bytes while the kernel runs (the backward kernel's exchange copy
    // of this layer, marked "not written yet" off the frame-to-frame path instead of by a launch of its own); null: none
    void* fill;
    unsigned long long fill_words;
    int T, B, H, nbg, tiles_per_group;
    unsigned* xcd;                // XCD_TABLE_BYTES of words, all ones (xcd.hpp), or null
    bool ask;                     // host only: launch nothing, only say whether it would be
};
struct RecBwdArgs {
    const unsigned short* uht[2]; // U_h^T per direction, [H][4H]
    const unsigned short* dy;     // dE/dh from above, [M][2H]
    const unsigned short* gates;  // as rec_fwd_kernel wrote them (per-lane records)
    const float* c;               // likewise
    unsigned short* da;           // dE/da, [M][8H]
    unsigned short* dax;          // dE/da again in exchange order, [T][2][tiles][4H/16][2][32][8]; pre-filled with 0xFFFF in sentinel mode
    float* dc;                    // carried dE/dc, records [2][tiles][H/32][256] of four floats (whole 32-row tiles)
    unsigned* cnt;
    unsigned* abort_word;
    unsigned long long limit_ticks;
    int T, B, H, nbg, tiles_per_group;
    unsigned* xcd;                // as above
    bool ask;                     // as above
};
bool rec_supported(int H);                  // whether the persistent kernels take this width
bool rec_takes(int T, int B, int H);        // ... and whether they are the faster path for so many frames and sequences
bool rec_fenced(int H);                     // whether they are built with the fenced protocol too
int rec_groups(int H, int tiles, int per_cu = 1);   // batch groups per direction for so many 32-row tiles and workgroups per CU
bool rec_narrow(int B, int H);              // a layer of up to 288 units that recurrent.hip runs (its forward kernel honours RecFwdArgs::fill there and wherever a workgroup has several tiles)
// *launched is false (and nothing was enqueued) when the grid cannot be co-resident on this device.
hipError_t launch_rec_fwd(const RecFwdArgs& a, bool sentinel, hipStream_t st, bool* launched);
hipError_t launch_rec_bwd(const RecBwdArgs& a, bool sentinel, hipStream_t st, bool* launched);
// The same for few sequences (recurrent_small.hip; sentinel protocol, nbg and tiles_per_group not used).  The saved records
// and exchange copies have an order of their own: forward and backward go together.
bool rec_small_supported(int B, int H);
hipError_t launch_rec_small_fwd(const RecFwdArgs& a, hipStream_t st, bool* launched);
hipError_t launch_rec_small_bwd(const RecBwdArgs& a, hipStream_t st, bool* launched);
// The same on 16-row tiles (recurrent_tile.hip; nbg and tiles_per_group set by the launcher, a counter per direction and tile):
// units of a workgroup, 32 or 64, or 0 if these kernels do not take the shape.
int rec_tile_units(int B, int H);
hipError_t launch_rec_tile_fwd(const RecFwdArgs& a, bool sentinel, hipStream_t st, bool* launched);
hipError_t launch_rec_tile_bwd(const RecBwdArgs& a, bool sentinel, hipStream_t st, bool* launched);

// ---- persistent recurrent kernels in float (H up to 1024) ------------------------------
struct Rec32FwdArgs {
    const float* uh[2];           // U_h per direction, [4H][H]
    const float* ax;              // W_x x + b for every frame, [M][8H]
    float* y;                     // h, [M][2H]
    float* z;                     // the same once more, or null (honoured where rec32_fwd_one says so)
    float* c;                     // cell states, [M][2H]
    float* gates;                 // gate activations, [M][8H]
    float* hx;                    // exchange copy of h, rec32_hx_bytes, filled with 0xFF bytes before the launch
    unsigned* abort_word;         // as in RecFwdArgs
    unsigned long long limit_ticks;
    void* fill;                   // fill_words 16-byte words to set to 0xFF bytes on the side, or null (honoured where rec32_fwd_one says so)
    unsigned long long fill_words;
    int T, B, H;
    int nu, nbg, tiles_per_group; // set by the launcher
    bool ask;                     // as in RecFwdArgs
};
struct Rec32BwdArgs {
    const float* uh[2];
    const float* dy;              // dE/dh from above, [M][2H]
    const float* gates;
    const float* c;
    float* da;                    // dE/da, [M][8H]
    float* dc;                    // carried dE/dc, [2][B][H]
    float* dax;                   // exchange copy of dE/da, rec32_dax_bytes, filled with 0xFF bytes before the launch
    unsigned* abort_word;
    unsigned long long limit_ticks;
    int T, B, H;
    int nu, nbg, tiles_per_group; // set by the launcher
    bool ask;                     // as in RecFwdArgs
};
// Whether the persistent kernel takes this shape (and is the faster of the two paths).
bool rec32_fwd_supported(int B, int H);
bool rec32_fwd_one(int B, int H);           // forward: the kernel with wavefronts for what is not the exchange runs it
bool rec32_bwd_supported(int B, int H);
size_t rec32_hx_bytes(int T, int B, int H);
size_t rec32_dax_bytes(int T, int B, int H);
hipError_t launch_rec32_fwd(Rec32FwdArgs a, hipStream_t st, bool* launched);   // *launched as for launch_rec_fwd
hipError_t launch_rec32_bwd(Rec32BwdArgs a, hipStream_t st, bool* launched);

// Transposes `count` matrices U_h [4H][H] (one per layer and direction) into dst + k * 4H*H.
struct TransposeUhArgs {
    const unsigned short* src[128];
    unsigned short* dst;
    int count;
};
hipError_t launch_transpose_uh(const TransposeUhArgs& a, int H, hipStream_t st);
hipError_t launch_fill_u32(unsigned* p, int n, unsigned v, hipStream_t st);
// Copies up to three row-major 16-bit matrices [rows][cols] (leading dimension ld) into [rows][cols_p] ones
// with zeros in columns cols .. cols_p - 1 (cols_p a multiple of 8, dst 16-byte aligned).
struct PadColsArgs {
    const unsigned short* src[3];
    unsigned short* dst[3];
    long long ld[3];
    int rows[3];
    int count, cols, cols_p;
    void* fill;                                // 16-byte words to set to all ones on the way
    size_t fill_words;
};
hipError_t launch_pad_cols(const PadColsArgs& a, hipStream_t st);
// Fills bytes/16 16-byte words with the 32-bit pattern v.
hipError_t launch_fill_bytes16(void* p, size_t bytes, unsigned v, hipStream_t st);

// ---- copies between compact and zero-padded tensors ----------------------------------------------
// A matrix of rg groups of r rows, each of cs segments of c columns, and its padded form with rp rows a group and cp
// columns a segment (offsets in elements; where there are two segments cp is a whole number of 16-byte words).
struct BlockTensor {
    size_t compact, padded;
    int rg, r, rp, cs, c, cp;
};
constexpr int BLOCK_COPIES_MAX = 64;
struct BlockCopies { BlockTensor t[BLOCK_COPIES_MAX]; };
hipError_t launch_pad_blocks(const BlockTensor* t, int n, const void* compact, void* padded, DType type, hipStream_t st);
// Columns h .. hp - 1 of `blocks` consecutive blocks of hp floats become zero.
hipError_t launch_zero_columns(float* p, long long blocks, int hp, int h, hipStream_t st);
hipError_t launch_compact_blocks(const BlockTensor* t, int n, const void* padded, void* compact, DType type, hipStream_t st);

// ---- softmax cross-entropy over rows of the logit matrix -----------------------------
// u [M][V] (storage type) is overwritten by dE/du = s (p - onehot); row_loss[m] = -s log p[label].
hipError_t launch_softmax_rows(void* u, long long ldu, const int32_t* labels, float* row_loss,
                               int M, int V, float s, DType store, hipStream_t st);
// out[0] = sum_m v[m], one workgroup, fixed summation order.
hipError_t launch_sum_to_scalar(const float* v, int M, float* out, hipStream_t st);

// ---- weight update and replica averaging ---------------------------------------------
hipError_t launch_sgd(float* theta, unsigned short* shadow, const float* grad, size_t n, float lr, float mu,
                      float* vel, hipStream_t st);
struct MixPairs {
    float* a[BLSTM_MAX_PAIRS];
    float* b[BLSTM_MAX_PAIRS];
    unsigned short* sa[BLSTM_MAX_PAIRS];
    unsigned short* sb[BLSTM_MAX_PAIRS];
    int npairs;
};
hipError_t launch_mix(const MixPairs& p, size_t n, hipStream_t st);
hipError_t launch_shadow(const float* theta, unsigned short* shadow, size_t n, hipStream_t st);
hipError_t launch_sgd_mix_pair(float* ti, float* tj, const float* gi, const float* gj, float* vi, float* vj,
                               unsigned short* si, unsigned short* sj, size_t n, float lr, float mu, hipStream_t st);
struct ReplicaSet {
    float* t[BLSTM_MAX_REPLICA_PTRS];
    unsigned short* s[BLSTM_MAX_REPLICA_PTRS];
    int R;
};
hipError_t launch_sync_average(const ReplicaSet& p, size_t n, hipStream_t st);

}  // namespace blstm
