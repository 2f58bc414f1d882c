// Row blocks of bf16 models on matrix cores, the prefill's chunks of up to kPrefillRows prompt rows and
// (where the stages do not hide its vector form) the draft module's in-flight rows: the launchers of spd_prefill.hip and the scratch they use.
// Internal; not part of the C ABI.
#pragma once
#include "spd_dev.h"

namespace spd {

// Prompt rows of one chunk: 2048 where their scratch stays within kPrefillBytes, else fewer, but never fewer
// than 1024, whatever that takes (4B class: 1024 rows, 149 MB; 9B class: 192 MB; more where a model is wider). A
// layer's weights are read once per chunk, which at 1024 rows is far below the matrix cores' time; narrow models
// need the rows to fill 256 CUs (1024 wide, 6000 tokens: 36.3 ms at 2048 rows, 44.7 ms at 1024).
constexpr int kPrefillRows = 2048, kPrefillMinRows = 1024;
constexpr size_t kPrefillBytes = (size_t)160 << 20;
constexpr int kPrefillMaxSplit = 16;  // K splits of one projection

// An fp32 activation matrix [rows][K] as three bf16 planes whose sum is the fp32 value exactly:
// element (p, m, k) at p + p * stride + m * K + k.
struct Planes {
  uint16_t* p;
  size_t stride;
};

// Scratch of the prefill, and of the draft module in a step (in the workspace).
struct PrefillBufs {
  int rows;          // row capacity, a multiple of 128: a chunk's, or max_tokens' where that is less
  size_t part_cap;   // floats in part
  float* x;          // [rows][d] residual rows of the target
  float* px;         // [rows][d] residual rows of the draft module
  float* q;          // [rows][Hq*dh] rotated queries, in pb's memory: read by the attention, before gate/up writes pb
  float* part;       // K-split partial sums, [split][row][column]
  float* rs;         // [rows] 1 / rms of the normalised rows
  uint16_t* pa;      // planes of [rows][max(d, Hq*dh)]: normalised rows, attention outputs
  uint16_t* pb;      // planes of [rows][max(d, F)]: SwiGLU activations, raw stage inputs
  uint16_t* zeros;   // 256 bytes of zeros
};

// Rows of a chunk and floats of partial sums for a model. Neither depends on a handle's max_tokens: the K splits
// follow from the partial sums that fit, and handles of any capacity store the same bits for a prompt.
int prefill_chunk_rows(int d, int F, int qdim, int qkv_cols);
size_t prefill_part_floats(int chunk_rows, int d, int F, int qkv_cols);

// The whole prompt: C.tok[0, len) through the target and the draft module's caches; the last row's
// residual ends in row *last_row of B.x. Asynchronous on stream.
void prefill_mfma(const Ctx& C, const PrefillBufs& B, const LayerDesc* layers, int len, void* stream, int* last_row);

// The draft module of one step: its feature projection and layers over the in-flight rows (Eq. agg-main,
// Eq. input-seq), the rows ending in C.pdm_x. max_rows: the SPD width; cap: at most this many workgroups
// per projection launch (0: no cap). Asynchronous on stream; nothing depends on host state.
void pdm_rows_mfma(const Ctx& C, const PrefillBufs& B, const LayerDesc* layers, int max_rows, int cap, void* stream);

}  // namespace spd
