// Ragged paged decode attention as a call of its own: up to eight query rows of one layer, row i
// attending keys [0, lens[i]) of a paged KV pool (Section 3.1: each in-flight token attends, at its
// own position, over the cache of the layer it is on). It runs the step's attention split
// (attn_split_g): one workgroup per (key split, KV head, row), the split that finishes last merging
// the row's splits in split order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "spd_dev.h"
#include "spd_devfn.h"
#include "spd_attn.h"

namespace spd {

void set_call_error(const std::string& msg);  // spd_last_error(NULL) (spd_api.cpp)

namespace {

struct RaggedRows {
  int lens[kMaxRows];
};

// Grid: x = key split, y = KV head, z = row. Workgroups past a row's last split return at once.
template <typename KVT, int DH, int GP>
__global__ __launch_bounds__(kWG) void k_attn_ragged(Ctx C, const float* q, const KVT* kv, float* out, float* part,
                                                     int* cnt, RaggedRows R, int smax) {
  extern __shared__ __align__(16) float lds[];
  const int split = blockIdx.x, g = blockIdx.y, z = blockIdx.z;
  const int k0 = split * C.chunk;
  const int page0 = C.page_table[min((k0 + (int)threadIdx.x / kAttnTPK) / C.page, C.max_pages - 1)];
  const int len = R.lens[z];
  const int nsplit = (len + C.chunk - 1) / C.chunk;
  if (split >= nsplit) return;
  const int k1 = min(len, k0 + C.chunk);
  constexpr int RS = kAttnMaxQ * (DH + 2);
  const size_t row = (size_t)z * C.qdim + (size_t)g * C.G * DH;
  const int cidx = z * C.hkv + g;
  attn_split_g<KVT, DH, GP>(C, kv, q + row, out + row, part + (size_t)cidx * smax * RS, cnt + cidx, g, split,
                            nsplit, k0, k1, len - 1, page0, lds);
}

// bf16 pools: rows of one KV head share its pages, so a workgroup serves 32 / G rows of a (key split, KV
// head) on matrix cores. Grid: x = key split, y = KV head, z = row group.
struct LimLens {
  const int* lens;
  __device__ __forceinline__ int operator()(int r) const { return lens[r] - 1; }
};

template <int DH>
__global__ __launch_bounds__(kWG, 2) void k_attn_ragged_mfma(Ctx C, const float* q, const uint16_t* kv, float* out,
                                                          float* part, RaggedRows R, int nrows) {
  extern __shared__ __align__(16) float lds[];
  __shared__ int s_lens[kMaxRows];
  const int rpg = 32 / C.G, r0 = blockIdx.z * rpg, nr = min(rpg, nrows - r0), split = blockIdx.x;
  int kend = 0;
  for (int i = 0; i < nr; i++) kend = max(kend, R.lens[r0 + i]);
  if (split * C.chunk >= kend) return;
  const int page0 = attn_mfma_page0(C, split);
  if (threadIdx.x < nr) s_lens[threadIdx.x] = R.lens[r0 + threadIdx.x];
  __syncthreads();
  const size_t rec0 = (size_t)r0 * C.hkv;
  attn_split_mfma<DH>(C, kv, q + (size_t)r0 * C.qdim, FloatOut{out + (size_t)r0 * C.qdim},
                      part + rec0 * C.max_splits * (kAttnMaxQ * (DH + 2)), blockIdx.y, split, nr, kend,
                      LimLens{s_lens}, page0, lds);
}

// The rows' split records into their outputs. Grid: x = KV head, y = row.
template <int DH>
__global__ __launch_bounds__(kWG) void k_attn_ragged_merge(Ctx C, float* out, const float* part, RaggedRows R) {
  __shared__ __align__(16) float sm[2 * kMaxSplits * kAttnMaxQ];
  attn_merge_row<DH>(C, part, FloatOut{out}, blockIdx.y, blockIdx.x, R.lens[blockIdx.y], sm);
}

__global__ __launch_bounds__(kWG) void k_zero_i32(int* p, int n) {
  for (int i = blockIdx.x * kWG + threadIdx.x; i < n; i += gridDim.x * kWG) p[i] = 0;
}

// A checked request: shapes, split count and the scratch it needs.
struct Request {
  Ctx C;
  RaggedRows R;
  int nrows, smax, dh, g4, bf16, vec;
  size_t rec_floats;  // split records
  int tickets;        // one per (row, KV head)
};

// bf16: whether the rows take the vector split, one workgroup per (key split, KV head, row) and the merge by
// tickets, and not the matrix-core one with its merge launch. The vector form is the quicker one while a split is a
// few rounds of 64 keys (fewer of them the more heads a round has), there are several splits to merge and
// about one workgroup a CU: 8 rows of 300 keys, splits of 64, 8 and 2 heads of 128: 13.4 us against 16.1; 2 rows
// of 1500 keys: 13.5 against 15.3; 8 rows, splits of 256: 16.4 against 18.8. Past that it is not: 8 rows of 1500
// keys with 32 and 8 heads 30.5 against 19.4, 4 rows of 300 keys with 8 heads on one 25.0 against 19.7 (splits of
// 256). At 64 dims the two differ by less than the call's own time varies.
bool vector_form(const Request& r, int chunk) {
  const int keys = r.nrows > 4 ? 1024 : r.nrows > 2 ? 512 : 256;
  return r.dh == 128 && r.smax > 1 && r.nrows * r.smax > 8 && (long long)r.nrows * r.smax * r.C.hkv <= 320 &&
         (long long)chunk * r.C.G <= keys;
}

spd_status check(const float* q, const void* kv, const int32_t* page_table, int32_t num_pages, const int32_t* lens,
                 int32_t nrows, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int32_t dtype,
                 int32_t chunk, const float* out, Request* rq) {
  auto bad = [](const char* m) {
    set_call_error(m);
    return SPD_E_INVAL;
  };
  if (!q || !kv || !page_table || !lens || !out) return bad("decode attention: NULL pointer");
  if (nrows < 1 || nrows > kMaxRows) return bad("decode attention: nrows must be in [1, 8]");
  if (head_dim != 64 && head_dim != 128) return bad("decode attention: head_dim must be 64 or 128");
  if (n_kv_heads < 1 || n_q_heads < 1 || n_q_heads % n_kv_heads) return bad("decode attention: bad head counts");
  const int G = n_q_heads / n_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8) return bad("decode attention: n_q_heads / n_kv_heads must be 1, 2, 4 or 8");
  if (dtype != SPD_F32 && dtype != SPD_BF16) return bad("decode attention: dtype must be SPD_F32 or SPD_BF16");
  if (chunk < 16 || chunk % 16) return bad("decode attention: chunk must be a positive multiple of 16");
  if (num_pages < 1) return bad("decode attention: num_pages must be positive");
  int maxlen = 0;
  for (int i = 0; i < nrows; i++) {
    if (lens[i] < 1 || (long long)lens[i] > 16LL * num_pages)
      return bad("decode attention: every length must be in [1, 16 * num_pages]");
    maxlen = std::max(maxlen, (int)lens[i]);
  }
  const int smax = (maxlen + chunk - 1) / chunk;
  if (smax > kMaxSplits) return bad("decode attention: more than 64 key splits per row (raise chunk)");
  Request& r = *rq;
  std::memset(&r.C, 0, sizeof(Ctx));
  r.C.hq = n_q_heads;
  r.C.hkv = n_kv_heads;
  r.C.dh = head_dim;
  r.C.qdim = n_q_heads * head_dim;
  r.C.kvdim = n_kv_heads * head_dim;
  r.C.G = G;
  r.C.page = 16;
  r.C.chunk = chunk;
  r.C.max_pages = num_pages;
  r.C.max_splits = smax;
  r.C.scale = (float)(1.0 / std::sqrt((double)head_dim));
  r.C.page_table = page_table;
  std::memset(&r.R, 0, sizeof(RaggedRows));
  for (int i = 0; i < nrows; i++) r.R.lens[i] = lens[i];
  r.nrows = nrows;
  r.smax = smax;
  r.dh = head_dim;
  r.g4 = G <= 4;
  r.bf16 = dtype == SPD_BF16;
  r.vec = !r.bf16 || vector_form(r, chunk);
  r.rec_floats = (size_t)nrows * n_kv_heads * smax * kAttnMaxQ * (head_dim + 2);
  r.tickets = nrows * n_kv_heads;
  return SPD_OK;
}

template <typename KVT, int DH>
void launch_ragged_vec(const Request& r, const float* q, const void* kv, float* out, float* part, int* cnt,
                       hipStream_t s) {
  const dim3 grid(r.smax, r.C.hkv, r.nrows);
  const size_t shm = attn_split_lds<KVT, DH>();
  if (r.g4)
    hipLaunchKernelGGL((k_attn_ragged<KVT, DH, 4>), grid, dim3(kWG), shm, s, r.C, q, (const KVT*)kv, out, part, cnt,
                       r.R, r.smax);
  else
    hipLaunchKernelGGL((k_attn_ragged<KVT, DH, 8>), grid, dim3(kWG), shm, s, r.C, q, (const KVT*)kv, out, part, cnt,
                       r.R, r.smax);
}

template <int DH>
void launch_ragged_mfma(const Request& r, const float* q, const void* kv, float* out, float* part, hipStream_t s) {
  const int rpg = 32 / r.C.G;
  const dim3 grid(r.smax, r.C.hkv, (r.nrows + rpg - 1) / rpg);
  hipLaunchKernelGGL((k_attn_ragged_mfma<DH>), grid, dim3(kWG), attn_mfma_lds<DH>(std::min(r.nrows, rpg) * r.C.G), s, r.C,
                     q, (const uint16_t*)kv, out, part, r.R, r.nrows);
  if (r.smax > 1)
    hipLaunchKernelGGL((k_attn_ragged_merge<DH>), dim3(r.C.hkv, r.nrows), dim3(kWG), 0, s, r.C, out,
                       (const float*)part, r.R);
}

// Matrix cores: the splits, then (with more than one) their merge. Vector form: the tickets are cleared (a fill
// kernel, so that a captured call replays correctly), then the attention, whose last splits merge.
spd_status run(const Request& r, const float* q, const void* kv, float* out, float* part, int* cnt, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (!r.vec) {
    if (r.dh == 128)
      launch_ragged_mfma<128>(r, q, kv, out, part, s);
    else
      launch_ragged_mfma<64>(r, q, kv, out, part, s);
  } else {
    hipLaunchKernelGGL(k_zero_i32, dim3((r.tickets + kWG - 1) / kWG), dim3(kWG), 0, s, cnt, r.tickets);
    if (r.bf16)
      launch_ragged_vec<uint16_t, 128>(r, q, kv, out, part, cnt, s);
    else if (r.dh == 128)
      launch_ragged_vec<float, 128>(r, q, kv, out, part, cnt, s);
    else
      launch_ragged_vec<float, 64>(r, q, kv, out, part, cnt, s);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_call_error(std::string("decode attention launch: ") + hipGetErrorString(e));
    return SPD_E_HIP;
  }
  return SPD_OK;
}

size_t rec_bytes(const Request& r) { return (r.rec_floats * sizeof(float) + 255) / 256 * 256; }

// Scratch of spd_decode_attention_noalloc: the split records of at most kNoAllocRecords (row, KV head,
// split) triples at head_dim 128, then one ticket per (row, KV head). Each GPU the library runs on holds
// its own copy until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device (the array's name is a host-side stand-in).
constexpr int kNoAllocRecords = 2048;
constexpr size_t kNoAllocRecBytes = (size_t)kNoAllocRecords * kAttnMaxQ * (128 + 2) * sizeof(float);
constexpr size_t kNoAllocBytes = kNoAllocRecBytes + sizeof(int) * (size_t)kNoAllocRecords;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up once per device with that device current.
spd_status scratch_of_current_device(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    set_call_error(std::string("decode attention (no allocation): hipGetDevice: ") + hipGetErrorString(e));
    return SPD_E_HIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_call_error(std::string("decode attention (no allocation): hipGetSymbolAddress: ") + hipGetErrorString(e));
      return SPD_E_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return SPD_OK;
}

}  // namespace
}  // namespace spd

using namespace spd;

extern "C" spd_status spd_decode_attention(const float* q, const void* kv, const int32_t* page_table,
                                           int32_t num_pages, const int32_t* lens, int32_t nrows, int32_t n_q_heads,
                                           int32_t n_kv_heads, int32_t head_dim, int32_t dtype, int32_t chunk,
                                           float* out, void* workspace, size_t ws_bytes, void* stream) {
  Request r;
  spd_status st = check(q, kv, page_table, num_pages, lens, nrows, n_q_heads, n_kv_heads, head_dim, dtype, chunk, out,
                        &r);
  if (st != SPD_OK) return st;
  if (!workspace || ((uintptr_t)workspace & 255)) {
    set_call_error("decode attention: workspace must be non-NULL and 256-byte aligned");
    return SPD_E_INVAL;
  }
  const size_t need = rec_bytes(r) + sizeof(int) * (size_t)r.tickets;
  if (ws_bytes < need) {
    set_call_error("decode attention: workspace too small, " + std::to_string(need) + " bytes needed");
    return SPD_E_CAPACITY;
  }
  char* ws = (char*)workspace;
  return run(r, q, kv, out, (float*)ws, (int*)(ws + rec_bytes(r)), stream);
}

extern "C" spd_status spd_decode_attention_noalloc(const float* q, const void* kv, const int32_t* page_table,
                                                   int32_t num_pages, const int32_t* lens, int32_t nrows,
                                                   int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                                   int32_t dtype, int32_t chunk, float* out, void* stream) {
  Request r;
  spd_status st = check(q, kv, page_table, num_pages, lens, nrows, n_q_heads, n_kv_heads, head_dim, dtype, chunk, out,
                        &r);
  if (st != SPD_OK) return st;
  const size_t records = (size_t)r.nrows * r.C.hkv * r.smax;
  if (records > (size_t)kNoAllocRecords) {
    set_call_error("decode attention (no allocation): nrows * n_kv_heads * splits = " + std::to_string(records) +
                   " exceeds the " + std::to_string(kNoAllocRecords) + " split records of the static scratch");
    return SPD_E_CAPACITY;
  }
  void* base = nullptr;
  st = scratch_of_current_device(&base);
  if (st != SPD_OK) return st;
  char* ws = (char*)base;
  return run(r, q, kv, out, (float*)ws, (int*)(ws + kNoAllocRecBytes), stream);
}
