// Row blocks of bf16 models on matrix cores: the prompt's prefill, and the draft module's rows in a step.
//
// A chunk of prompt rows goes through a layer as four dense projections and one causal attention. The
// activations stay fp32 in value: every fp32 operand x is cut into three bf16 planes by truncation,
// hi + mid + lo == x exactly (24 significant bits in three groups of eight), and each product runs as
// three bf16 MFMAs against the bf16 weights (or keys, or values), which are exact too. Only the order
// of the sums differs from an fp32 GEMV. v_mfma_f32_32x32x16_bf16 moves 16 times the multiplies of the
// fp32 instruction, so three of them are still five times faster.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "spd_attn.h"
#include "spd_devfn.h"
#include "spd_prefill.h"

namespace spd {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(1))) const void gbytes;
typedef __attribute__((address_space(3))) void lbytes;

// x as bf16 bits hi, mid, lo with hi + mid + lo == x (the parts below the smallest bf16 excepted).
// Truncation: no part overflows, and an infinity or NaN stays in hi alone.
__device__ __forceinline__ void split3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  const uint32_t u = __float_as_uint(x) & 0xffff0000u;
  const bool fin = (u & 0x7f800000u) != 0x7f800000u;
  const float r = fin ? x - __uint_as_float(u) : 0.f;
  const uint32_t m = __float_as_uint(r) & 0xffff0000u;
  hi = u >> 16;
  // a NaN whose payload sits in the low half would read as an infinity
  if (!fin && (__float_as_uint(x) & 0x7fffffu) != 0) hi |= 0x40u;
  mid = m >> 16;
  lo = __float_as_uint(r - __uint_as_float(m)) >> 16;
}

// Four consecutive elements into the three planes (8-byte aligned).
__device__ __forceinline__ void store_planes4(const Planes& P, size_t at, float a, float b, float c, float d) {
  uint32_t h[4], m[4], l[4];
  split3(a, h[0], m[0], l[0]);
  split3(b, h[1], m[1], l[1]);
  split3(c, h[2], m[2], l[2]);
  split3(d, h[3], m[3], l[3]);
  *reinterpret_cast<uint2*>(P.p + at) = make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
  *reinterpret_cast<uint2*>(P.p + P.stride + at) = make_uint2(m[0] | m[1] << 16, m[2] | m[3] << 16);
  *reinterpret_cast<uint2*>(P.p + 2 * P.stride + at) = make_uint2(l[0] | l[1] << 16, l[2] | l[3] << 16);
}

// ------------------------------------------------------------------------------- residual and norm
// One row per workgroup: v = x (or the token's embedding, or nothing) + the S partial sums of the
// projection before it, in split order; v becomes x. With a gain, v * gain goes to the planes of the
// next projection and 1 / rms(v) to rs; raw: v's own planes (the draft module's stage input).
struct NormArgs {
  const DevState* st;    // rows: the in-flight tokens of a step (null: the grid's rows)
  float* x;
  int d, S, base;        // base: 0 x, 1 the token's embedding, 2 zero
  const float* part;     // [S][rows][d], row stride d
  size_t part_stride;    // floats per split
  const int32_t* tok;
  const uint16_t* embed;
  const float* gain;     // null: no norm
  float eps;
  Planes out, raw;       // raw.p null: none
  float* rs;
};

constexpr int kPartBatch = 8;                  // partial sums loaded at once
constexpr int kNormVec = 8192 / 4 / kWG;  // float4 groups per thread at the largest d

__global__ __launch_bounds__(kWG) void k_pf_norm(NormArgs A) {
  __shared__ float red[4];
  const int m = blockIdx.x, d = A.d, n4 = d >> 2;
  if (A.st != nullptr && m >= A.st->a) return;
  float* x = A.x + (size_t)m * d;
  const uint16_t* E = A.base == 1 ? A.embed + (size_t)A.tok[m] * d : nullptr;
  float4 v[kNormVec];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kNormVec; i++) {
    const int k4 = threadIdx.x + i * kWG;
    if (k4 >= n4) break;
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (A.base == 0) {
      t = *reinterpret_cast<const float4*>(x + k4 * 4);
    } else if (A.base == 1) {
      const uint2 e = *reinterpret_cast<const uint2*>(E + k4 * 4);
      t = make_float4(bf_lo(e.x), bf_hi(e.x), bf_lo(e.y), bf_hi(e.y));
    }
    const float* pp = A.part + (size_t)m * d + k4 * 4;
    for (int s0 = 0; s0 < A.S; s0 += kPartBatch) {  // a batch's loads are in flight together
      float4 p[kPartBatch];
#pragma unroll
      for (int j = 0; j < kPartBatch; j++)
        if (s0 + j < A.S) p[j] = *reinterpret_cast<const float4*>(pp + (s0 + j) * A.part_stride);
#pragma unroll
      for (int j = 0; j < kPartBatch; j++)
        if (s0 + j < A.S) {
          t.x += p[j].x;
          t.y += p[j].y;
          t.z += p[j].z;
          t.w += p[j].w;
        }
    }
    ss = fmaf(t.x, t.x, ss);
    ss = fmaf(t.y, t.y, ss);
    ss = fmaf(t.z, t.z, ss);
    ss = fmaf(t.w, t.w, ss);
    v[i] = t;
    *reinterpret_cast<float4*>(x + k4 * 4) = t;
  }
  if (A.gain == nullptr) return;
#pragma unroll
  for (int i = 0; i < kNormVec; i++) {
    const int k4 = threadIdx.x + i * kWG;
    if (k4 >= n4) break;
    const float4 g = *reinterpret_cast<const float4*>(A.gain + k4 * 4);
    const float4 t = v[i];
    const size_t at = (size_t)m * d + k4 * 4;
    store_planes4(A.out, at, t.x * g.x, t.y * g.y, t.z * g.z, t.w * g.w);
    if (A.raw.p != nullptr) store_planes4(A.raw, at, t.x, t.y, t.z, t.w);
  }
  const float tot = block_sum(ss, red);
  if (threadIdx.x == 0) A.rs[m] = 1.0f / sqrtf(tot / (float)d + A.eps);
}

// ------------------------------------------------------------------------------------- projections
enum GemmKind { GK_PLAIN = 0, GK_QKV = 1, GK_GATEUP = 2 };

// Where a pair's two columns go: QKV pairs are a head's RoPE partners (q to the query rows, k and v to
// the paged cache), gate/up pairs the two factors of one SwiGLU activation.
struct PairOut {
  const float* rs;            // row scales
  float* q;                   // QKV
  uint16_t* kv;
  const int32_t* page_table;
  const float2* rope;
  int pos0, hq, hkv, dh, page;
  Planes act;                 // gate/up
  int F;
};

__device__ __forceinline__ void qkv_store(const PairOut& O, int m, int q, float lo, float hi) {
  const int half = O.dh >> 1, head = q / half, j = q - head * half, pos = O.pos0 + m;
  if (head < O.hq + O.hkv) {  // q and k are rotated at the row's position
    const float2 r = O.rope[(size_t)pos * half + j];
    const float a = lo * r.x - hi * r.y, b = hi * r.x + lo * r.y;
    lo = a;
    hi = b;
  }
  if (head < O.hq) {
    float* o = O.q + (size_t)m * O.hq * O.dh + head * O.dh;
    o[j] = lo;
    o[j + half] = hi;
  } else {
    const int is_v = head >= O.hq + O.hkv, hk = head - O.hq - (is_v ? O.hkv : 0);
    const size_t off = ((size_t)O.page_table[pos / O.page] * 2 + is_v) * O.hkv * O.page * O.dh +
                       ((size_t)hk * O.page + pos % O.page) * O.dh + j;
    st1<uint16_t>(O.kv, off, lo);
    st1<uint16_t>(O.kv, off + half, hi);
  }
}

__device__ __forceinline__ void act_store(const PairOut& O, int m, int q, float g, float u) {
  uint32_t h, mi, l;
  split3(g / (1.0f + expf(-g)) * u, h, mi, l);
  const size_t at = (size_t)m * O.F + q;
  O.act.p[at] = (uint16_t)h;
  O.act.p[O.act.stride + at] = (uint16_t)mi;
  O.act.p[2 * O.act.stride + at] = (uint16_t)l;
}

struct GemmArgs {
  Planes a;                       // [M][K]
  const uint16_t *w0, *w1, *w2;   // plain: w0; QKV: wq, wk, wv; gate/up: wg, wu
  const uint16_t* zeros;
  int M, K, ldw;
  int cols;                       // plain: columns; pair kinds: pairs (two columns each)
  int KS, S;                      // K range of a split, a multiple of 64; splits
  int mt, nt;                     // tiles
  float* part;                    // null: the pair epilogue
  PairOut out;
  const DevState* st;             // row GEMM: M is the step's in-flight tokens (null: M)
  unsigned long long* trace;      // row GEMM: launch-trace slot (null: none)
};

// Source row of tile row rb of the weights (rows past the matrix re-read its last one; their results are
// not stored). Pair kinds interleave the two matrices' rows, or a head's RoPE partners, by 32.
template <int KIND>
__device__ __forceinline__ const uint16_t* weight_row(const GemmArgs& G, int n0, int rb) {
  if (KIND == GK_PLAIN) return G.w0 + (size_t)min(n0 + rb, G.cols - 1) * G.ldw;
  const int which = (rb >> 5) & 1, q = min((n0 >> 1) + (rb >> 6) * 32 + (rb & 31), G.cols - 1);
  if (KIND == GK_GATEUP) return (which ? G.w1 : G.w0) + (size_t)q * G.ldw;
  const int half = G.out.dh >> 1, head = q / half, j = q - head * half;
  const uint16_t* W = G.w0;
  int hr = head;
  if (head >= G.out.hq) {
    hr -= G.out.hq;
    W = G.w1;
    if (hr >= G.out.hkv) {
      hr -= G.out.hkv;
      W = G.w2;
    }
  }
  return W + ((size_t)hr * G.out.dh + j + which * half) * G.ldw;
}

// C = A W^T over a BM x BN tile: a workgroup of NWM x NWN waves, each WM x WN in 32 x 32 MFMA tiles.
// The three A planes and the W rows of a K step of BK go to LDS with direct 16-byte global loads
// (double buffered; the 16-byte chunks of a row are permuted so that eight consecutive rows read eight
// different bank groups). Pair kinds interleave the weights' rows by 32 so that a lane holds both
// columns of its pairs in neighbouring MFMA tiles.
//
// Sums: a block of 64 inputs starts from zero and adds its lo products first, then mid, then hi, so
// that only the 4 hi MFMAs round at the block's magnitude; the blocks then add up in fp32. One running
// accumulator over all of K instead rounds three times per 16 inputs: relative error 5.5e-7 at K = 2560
// and 1.1e-6 at 9728, against 1.3e-7 and 2.3e-7 for the 64-lane fp32 GEMV and 1.3e-7 and 2.3e-7 (less
// with K splits) this way, at the same speed.
//
// Bound: the chain from LDS to MFMA between barriers (three planes of A against one of W: a 64 x 64 wave tile
// reads 16 operands per 24 MFMAs), then the last round of workgroups. Counters at 768 rows of the 4B class: the
// matrix cores run half of a busy CU's cycles, the LDS a third (half of that bank conflicts), and the CUs are busy
// 0.82 (gate/up), 0.73 (O-proj, down) and 0.50 (QKV) of a launch. A workgroup of eight waves over 128 x 256 shares
// each A tile between four waves: the 4B-class projections of 1501 rows in one chunk took 434 us (gate/up, 345
// TFLOP/s of products, 1034 of MFMA), 87 (O-proj) and 209 (down), against 510, 103 and 236 for four waves over
// 128 x 128 twice per CU; a large bf16 library product reaches 1375 TFLOP/s on the same card. Three and four buffers
// were slower than two (457 to 479 us for gate/up).
//
// Workgroup b runs on XCD b % 8: each XCD takes a contiguous range of the tiles, rows fastest, so the
// row tiles that share a weight tile share an L2.
template <int WM, int WN, int NWM, int NWN, int BK, int KIND>
__global__ __launch_bounds__(64 * NWM * NWN, 2) void k_pf_gemm(GemmArgs G) {
  constexpr int NTH = 64 * NWM * NWN;
  constexpr int BM = WM * NWM, BN = WN * NWN, NCH = BK / 8, ROWS = 3 * BM + BN, CPT = ROWS * NCH / NTH;
  constexpr int BUF = ROWS * BK * 2, TM = WM / 32, TN = WN / 32, NS = BK / 16;
  static_assert(ROWS * NCH % NTH == 0, "whole loads");
  static_assert(BK == 32 || BK == 64, "a block of 64 inputs is one or two steps");
  extern __shared__ __align__(16) char plds[];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  int b = blockIdx.x;
  {
    const int T = gridDim.x, per = T / 8, rem = T % 8, xcd = b % 8, j = b / 8;
    b = xcd * per + min(xcd, rem) + j;
  }
  const int mi = b % G.mt, ni = (b / G.mt) % G.nt, z = b / (G.mt * G.nt);
  const int m0 = mi * BM, n0 = ni * BN;
  const int kb = z * G.KS, ke = min(G.K, kb + G.KS);

  // source of this thread's chunk i: row R = plane * BM + row, or a weight row
  const uint16_t* src[CPT];
  int kc[CPT];
#pragma unroll
  for (int i = 0; i < CPT; i++) {
    const int t = i * NTH + tid, row = t / NCH, c = (t % NCH) ^ (NCH == 4 ? (row >> 1) & 3 : row & 7);
    kc[i] = c * 8;
    src[i] = (row < 3 * BM ? G.a.p + (row / BM) * G.a.stride + (size_t)min(m0 + row % BM, G.M - 1) * G.K
                           : weight_row<KIND>(G, n0, row - 3 * BM)) + c * 8;
  }
  auto issue = [&](int buf, int k) {  // inputs k .. k + BK (zeros past the split's end)
#pragma unroll
    for (int i = 0; i < CPT; i++) {
      const uint16_t* p = k + kc[i] < ke ? src[i] + k : G.zeros;
      __builtin_amdgcn_global_load_lds((gbytes*)p, (lbytes*)(plds + buf * BUF + (i * NTH + w * 64) * 16), 16, 0, 0);
    }
  };
  // every wave's loads have landed, and every wave is done with the buffer that is loaded next
  auto arrive = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  const int wm = w % NWM, wn = w / NWM, r = lane & 31, h = lane >> 5;
  const int sw = NCH == 4 ? (r >> 1) & 3 : r & 7;
  auto frag = [&](const char* base, int row, int s) {  // MFMA operand of inputs 16 s ..: lane row r, half h
    return *reinterpret_cast<const bf16x8*>(base + (row + r) * BK * 2 + (((2 * s + h) ^ sw) << 4));
  };
  f32x16 tot[TM][TN], acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) tot[i][j] = (f32x16)(0.f);
  auto mul = [&](const bf16x8 (&a)[TM], const bf16x8 (&bw)[TN], bool first) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bw[j], first ? (f32x16)(0.f) : acc[i][j], 0, 0, 0);
  };
  auto load_w = [&](const char* base, bf16x8 (&bw)[NS][TN]) {
#pragma unroll
    for (int s = 0; s < NS; s++)
#pragma unroll
      for (int j = 0; j < TN; j++) bw[s][j] = frag(base, 3 * BM + wn * WN + j * 32, s);
  };
  auto load_a = [&](const char* base, int p, int s, bf16x8 (&a)[TM]) {
#pragma unroll
    for (int i = 0; i < TM; i++) a[i] = frag(base, p * BM + wm * WM + i * 32, s);
  };
  auto planes = [&](const char* base, int p_last, const bf16x8 (&bw)[NS][TN], bool fresh) {  // lo, mid(, hi)
#pragma unroll
    for (int p = 2; p >= p_last; p--)
#pragma unroll
      for (int s = 0; s < NS; s++) {
        bf16x8 a[TM];
        load_a(base, p, s, a);
        mul(a, bw[s], fresh && p == 2 && s == 0);
      }
  };
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) tot[i][j][v] += acc[i][j][v];
  };

  issue(0, kb);
  if constexpr (BK == 64) {
    int buf = 0;
    for (int k = kb; k < ke; k += BK, buf ^= 1) {
      arrive();
      if (k + BK < ke) issue(buf ^ 1, k + BK);
      bf16x8 bw[NS][TN];
      load_w(plds + buf * BUF, bw);
      planes(plds + buf * BUF, 0, bw, true);
      fold();
    }
  } else {
    for (int k = kb; k < ke; k += 2 * BK) {
      bf16x8 w0[NS][TN], w1[NS][TN], hi0[NS][TM];
      arrive();
      if (k + BK < ke) issue(1, k + BK);
      load_w(plds, w0);
#pragma unroll
      for (int s = 0; s < NS; s++) load_a(plds, 0, s, hi0[s]);  // hi waits for the block's small products
      planes(plds, 1, w0, true);
      const bool second = k + BK < ke;
      if (second) {
        arrive();
        if (k + 2 * BK < ke) issue(0, k + 2 * BK);
        load_w(plds + BUF, w1);
        planes(plds + BUF, 1, w1, false);
      }
#pragma unroll
      for (int s = 0; s < NS; s++) mul(hi0[s], w0[s], false);
      if (second) {
#pragma unroll
        for (int s = 0; s < NS; s++) {
          bf16x8 a[TM];
          load_a(plds + BUF, 0, s, a);
          mul(a, w1[s], false);
        }
      }
      fold();
    }
  }

  // register v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
  const int mr = m0 + wm * WM + 4 * h;
  if (KIND == GK_PLAIN || G.part != nullptr) {
    const int ncol = KIND == GK_PLAIN ? G.cols : 2 * G.cols;
    float* o = G.part + (size_t)z * G.M * ncol;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int cb = wn * WN + j * 32;  // column block of the tile
      int col;
      bool ok;
      if (KIND == GK_PLAIN) {
        col = n0 + cb + r;
        ok = col < G.cols;
      } else {  // both columns of pair q at q and cols + q
        const int q = (n0 >> 1) + (cb >> 6) * 32 + r;
        col = ((cb >> 5) & 1) * G.cols + q;
        ok = q < G.cols;
      }
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int m = mr + i * 32 + 8 * (v >> 2) + (v & 3);
          if (ok && m < G.M) o[(size_t)m * ncol + col] = tot[i][j][v];
        }
    }
  } else if constexpr (KIND != GK_PLAIN && TN % 2 == 0) {
#pragma unroll
    for (int jp = 0; jp < TN / 2; jp++) {
      const int q = ((n0 + wn * WN) >> 1) + jp * 32 + r;
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int m = mr + i * 32 + 8 * (v >> 2) + (v & 3);
          if (q >= G.cols || m >= G.M) continue;
          const float sc = G.out.rs[m], s0 = tot[i][2 * jp][v] * sc, s1 = tot[i][2 * jp + 1][v] * sc;
          if (KIND == GK_QKV)
            qkv_store(G.out, m, q, s0, s1);
          else
            act_store(G.out, m, q, s0, s1);
        }
    }
  }
}

// The same product for up to eight rows (the draft module's in-flight rows, a prompt's last or only
// rows): the three planes of the eight rows are 24 of the 32 rows of ONE MFMA operand, so a weight takes
// one MFMA and a lane ends with the three planes' sums of its rows in registers v, v + 4 and v + 8. Four
// waves x 32 weight rows, steps of 64 inputs through kRowBufs LDS buffers; partial sums [split][8][column].
// Workgroup b takes jobs b, b + grid, .. of the tiles x splits.
// Bound: the weights' stream. In a step of the 4B class, beside the stage compute, the draft module's
// gate/up (99.6 MB) takes 24 us, where a vector GEMV held to 32 workgroups so as to leave the stages
// their LDS took 278. A cap on the workgroups (spd_set_pdm_grid) only lengthens the step: 4B n = 4
// 36.0 ms per 24 steps without one, 36.4 at 64 workgroups; 9B n = 8 34.6 per 20 steps, 36.0 at 64.
constexpr int kRowBufs = 3;
template <int KIND>
__global__ __launch_bounds__(kWG, 2) void k_pf_rows(GemmArgs G) {
  constexpr int BN = 128, BK = 64, ROWS = 32 + BN, CPT = ROWS * 8 / kWG, BUF = ROWS * BK * 2, NS = BK / 16;
  extern __shared__ __align__(16) char plds[];
  const int M = G.st != nullptr ? G.st->a : G.M;
  if (M <= 0) return;
  if (G.trace != nullptr && blockIdx.x == 0 && threadIdx.x == 0) G.trace[0] = (unsigned long long)wall_clock64();
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 31, h = lane >> 5;
  const int ncol = KIND == GK_PLAIN ? G.cols : 2 * G.cols, jobs = G.nt * G.S;
  for (int job = blockIdx.x; job < jobs; job += gridDim.x) {
    const int n0 = (job % G.nt) * BN, z = job / G.nt, kb = z * G.KS, ke = min(G.K, kb + G.KS);
    const uint16_t* src[CPT];
    int kc[CPT];
#pragma unroll
    for (int i = 0; i < CPT; i++) {
      const int t = i * kWG + tid, row = t / 8, c = (t % 8) ^ (row & 7);
      kc[i] = c * 8;
      src[i] = (row < 32 ? G.a.p + min(row >> 3, 2) * G.a.stride + (size_t)min(row & 7, M - 1) * G.K
                         : weight_row<KIND>(G, n0, row - 32)) + c * 8;
    }
    auto issue = [&](int buf, int k) {  // zeros past the split's end, so that every step waits for as many loads
#pragma unroll
      for (int i = 0; i < CPT; i++) {
        const uint16_t* p = k + kc[i] < ke ? src[i] + k : G.zeros;
        lbytes* const to = (lbytes*)(plds + buf * BUF + (i * kWG + w * 64) * 16);
        if (i == 0)  // the activations' 32 rows
          __builtin_amdgcn_global_load_lds((gbytes*)p, to, 16, 0, 0);
        else  // weights, read once: non-temporal
          __builtin_amdgcn_global_load_lds((gbytes*)p, to, 16, 0, 2);
      }
    };
    auto frag = [&](const char* base, int row, int s) {
      return *reinterpret_cast<const bf16x8*>(base + (row + r) * BK * 2 + (((2 * s + h) ^ (r & 7)) << 4));
    };
    float tot[12];
#pragma unroll
    for (int v = 0; v < 12; v++) tot[v] = 0.f;
#pragma unroll
    for (int i = 0; i < kRowBufs - 1; i++) issue(i, kb + i * BK);
    int rd = 0, wr = kRowBufs - 1;
    for (int k = kb; k < ke; k += BK) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((kRowBufs - 2) * CPT) : "memory");
      issue(wr, k + (kRowBufs - 1) * BK);
      wr = wr + 1 == kRowBufs ? 0 : wr + 1;
      const char* base = plds + rd * BUF;
      rd = rd + 1 == kRowBufs ? 0 : rd + 1;
      f32x16 acc;
#pragma unroll
      for (int s = 0; s < NS; s++)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(base, 0, s), frag(base, 32 + w * 32, s),
                                                      s == 0 ? (f32x16)(0.f) : acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 12; v++) tot[v] += acc[v];
    }
    // the zero loads past the end have landed and every wave is done with the buffers
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    int col;
    bool ok;
    if (KIND == GK_PLAIN) {
      col = n0 + w * 32 + r;
      ok = col < G.cols;
    } else {
      const int q = (n0 >> 1) + (w >> 1) * 32 + r;
      col = (w & 1) * G.cols + q;
      ok = q < G.cols;
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int m = 4 * h + e;
      if (ok && m < M) G.part[((size_t)z * kMaxRows + m) * ncol + col] = (tot[8 + e] + tot[4 + e]) + tot[e];
    }
  }
  if (G.trace != nullptr && threadIdx.x == 0)
    __hip_atomic_fetch_max(G.trace + 1, (unsigned long long)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The pair epilogue of a K-split projection: the splits added in order. Grid: x pairs, y rows. part:
// [split][prows][column].
template <int KIND>
__global__ __launch_bounds__(kWG) void k_pf_pairs(PairOut O, const float* part, int S, int prows, int pairs,
                                                  const DevState* st) {
  const int q = blockIdx.x * kWG + threadIdx.x, m = blockIdx.y;
  if (st != nullptr) {
    if (m >= st->a) return;
    O.pos0 = st->c;
  }
  if (q >= pairs) return;
  float s0 = 0.f, s1 = 0.f;
  const float* pp = part + (size_t)m * 2 * pairs + q;
  const size_t stride = (size_t)prows * 2 * pairs;
  for (int b = 0; b < S; b += kPartBatch) {
    float p0[kPartBatch], p1[kPartBatch];
#pragma unroll
    for (int j = 0; j < kPartBatch; j++)
      if (b + j < S) {
        p0[j] = pp[(b + j) * stride];
        p1[j] = pp[(b + j) * stride + pairs];
      }
#pragma unroll
    for (int j = 0; j < kPartBatch; j++)
      if (b + j < S) {
        s0 += p0[j];
        s1 += p1[j];
      }
  }
  const float sc = O.rs[m];
  if (KIND == GK_QKV)
    qkv_store(O, m, q, s0 * sc, s1 * sc);
  else
    act_store(O, m, q, s0 * sc, s1 * sc);
}

// --------------------------------------------------------------------------- draft module's features
// The in-flight rows' anchors as planes [a][n * d], zeros for the anchors a row has not reached: row i at
// depth a - 1 - i before the step (one deeper in the post-step schedule). Grid: x columns, y rows.
__global__ __launch_bounds__(kWG) void k_pdm_feat(Ctx C, Planes out) {
  const int i = blockIdx.y, a = C.st->a, k = (blockIdx.x * kWG + threadIdx.x) * 4, K = C.n * C.d;
  if (i >= a || k >= K) return;
  const int depth = a - 1 - i + C.post_step, nelig = (min(depth, C.n - 1) + 1) * C.d;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (k < nelig) v = *reinterpret_cast<const float4*>(C.anchors + (size_t)((C.st->c + i) % C.n) * K + k);
  store_planes4(out, (size_t)i * K + k, v.x, v.y, v.z, v.w);
}

// The draft module's row attention (attn_split_mfma): one workgroup per (key split, KV head, group of
// 32 / G rows); splits past the group's last key return at once. Outputs as planes [a][Hq*dh].
struct PlaneOut {
  Planes P;
  __device__ __forceinline__ void operator()(size_t at, float a, float b) const {
    uint32_t h[2], m[2], l[2];
    split3(a, h[0], m[0], l[0]);
    split3(b, h[1], m[1], l[1]);
    *reinterpret_cast<uint32_t*>(P.p + at) = h[0] | h[1] << 16;
    *reinterpret_cast<uint32_t*>(P.p + P.stride + at) = m[0] | m[1] << 16;
    *reinterpret_cast<uint32_t*>(P.p + 2 * P.stride + at) = l[0] | l[1] << 16;
  }
};

template <int DH>
__global__ __launch_bounds__(kWG, 2) void k_pdm_attn(Ctx C, const uint16_t* kv, Planes out) {
  extern __shared__ __align__(16) float lds[];
  const int rpg = 32 / C.G, r0 = blockIdx.z * rpg, split = blockIdx.x;
  const int page0 = attn_mfma_page0(C, split);
  const int nr = min(rpg, C.st->a - r0), pos0 = C.st->c + r0;
  if (nr <= 0 || split * C.chunk >= pos0 + nr) return;
  const BufSet& B = C.b[1];
  out.p += (size_t)r0 * C.qdim;
  attn_split_mfma<DH>(C, kv, B.q + (size_t)r0 * C.qdim, PlaneOut{out},
                      B.part + (size_t)r0 * C.hkv * C.max_splits * (kAttnMaxQ * (DH + 2)), blockIdx.y, split, nr,
                      pos0 + nr, LimPos{pos0}, page0, lds);
}

// The rows' split records into their output planes. Grid: x = KV head, y = row.
template <int DH>
__global__ __launch_bounds__(kWG) void k_pdm_attn_merge(Ctx C, Planes out) {
  __shared__ __align__(16) float sm[2 * kMaxSplits * kAttnMaxQ];
  const int r = blockIdx.y;
  if (r >= C.st->a) return;
  attn_merge_row<DH>(C, C.b[1].part, PlaneOut{out}, r, blockIdx.x, C.st->c + r + 1, sm);
}

// --------------------------------------------------------------------------------- causal attention
// Rows at positions pos0 .. pos0 + M - 1 over one layer's paged bf16 cache, which already holds their
// keys. A workgroup serves 128 queries (128 / G rows x the G heads of KV head g), 32 per wave, and
// walks the keys in tiles of 64 up to its last row's position:
//   * S^T = K Q^T (lane l: query l % 32, 16 keys per 32-key block), q in registers as three planes;
//   * the softmax of a query is a max and a sum over the lane's keys and one exchange with lane l ^ 32
//     (base 2: the queries are scaled by log2(e) / sqrt(dh));
//   * O^T += V^T P^T with p cut into planes in registers: the eight keys that half h of k step s needs
//     are the ones the lane already holds, if V^T keeps its key quads in the order 0, 2, 1, 3.
// K goes to LDS with direct loads, V through registers, where 4 x 8 blocks are transposed.
// A workgroup's rows share its key tiles, so 0 * v of a value past a row's own position, or 0 * k of a query
// plane, makes NaN of a row whose own keys and values do not: a query that ends as NaN is computed again over
// its own keys by plain FMAs (attn_query_plain).
// Bound: MFMA (48 per 32 keys, a quarter of a busy CU's cycles) beside the softmax's vector work, and CUs without a
// workgroup (768 rows of the 4B class are 192). A layer of the 4B class takes 35 us for 384 rows and 60 + 100 us for
// the chunks of 768 and 733 rows of 1501; the wide model's chunks of 2048, 2048 and 1904 rows 131, 243 and 349 us.
// With the page of each tile read where it is used, behind the keys in flight, they took 1.3 to 1.5 times as long.
struct AttnArgs {
  const float* q;
  Planes out;                 // [M][Hq*dh]
  const uint16_t* kv;
  const int32_t* page_table;
  int M, pos0, G, hkv, max_pages;
  float scale, qscale;        // 1 / sqrt(dh), and the same times log2(e)
  float4* tot;                // sums of earlier segments: a wave's [DH/8][64 lanes], then its (m, l)
};

// Key tiles of a segment, after which the sums restart from zero and the segment's join those before it, kept
// in global memory (the registers hold one set); up to kPfSegLast more tiles at the end make no segment of their own.
// One accumulator over the whole prompt rounds every product's sum at the running total's magnitude; relative error
// on flat scores (and at scores of deviation 1.5):
//   keys       one accumulator       256-key segments      fp32 MFMA, splits of 64 (6000: 128) keys
//    760       1.3e-7 (3.3e-7)       1.1e-7 (3.2e-7)       1.2e-7 (5.3e-7)
//   1501       1.6e-7 (3.8e-7)       1.2e-7 (3.5e-7)       1.3e-7 (5.7e-7)
//   6000       2.8e-7 (5.2e-7)       1.4e-7 (3.9e-7)       1.4e-7 (6.4e-7)
// 384-key segments are at 1.5e-7 at 6000 keys. A segment costs 1.5 us, half of it the round trip of the earlier sums
// (eight loads at once; four took longer and sixteen spill): the wide model's three chunks of 6000 tokens took 118,
// 219 and 317 us a layer with one accumulator. expf and a scale without log2(e) change none of the errors.
constexpr int kPfSeg = 4, kPfSegLast = 2;

template <int DH>
__global__ __launch_bounds__(kWG, 2) void k_pf_attn(AttnArgs A) {
  constexpr int KT = 64, NT = DH / 32, KS = DH / 16, NCH = DH / 8, PAGE = 16;
  constexpr int KBUF = KT * DH * 2, VBUF = DH * KT * 2, BUF = KBUF + VBUF;
  constexpr int KPT = KT * NCH / kWG;          // K chunks per thread (one page each pass)
  constexpr int VTH = KT / 4 * (DH / 8);       // threads with a 4 x 8 block of V
  constexpr int UB = DH == 64 ? 2 : 1;         // 32-key blocks unrolled: at 128 dims two spill
  extern __shared__ __align__(16) char plds[];
  __shared__ uint32_t s_nan[kWG / 64];  // per wave, its queries whose result is NaN
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, col = lane & 31, h = lane >> 5;
  const int g = blockIdx.x, G = A.G, rpw = 128 / G;
  const int row0 = ((int)gridDim.y - 1 - (int)blockIdx.y) * rpw;  // the longest rows first
  const int qd = A.hkv * G * DH;
  const int qi = w * 32 + col, qr = min(row0 + qi / G, A.M - 1), qh = g * G + qi % G;
  const int qlim = A.pos0 + qr;                                   // last key of this lane's query
  const int kend = A.pos0 + min(row0 + rpw, A.M);                 // keys of the workgroup: [0, kend)
  const int tiles = (kend + KT - 1) / KT;
  const size_t page_elems = (size_t)2 * A.hkv * PAGE * DH, head_off = (size_t)g * PAGE * DH;
  const size_t voff = (size_t)A.hkv * PAGE * DH;

  bf16x8 qf[3][KS];
  {
    const float* qp = A.q + (size_t)qr * qd + (size_t)qh * DH + h * 8;
#pragma unroll
    for (int s = 0; s < KS; s++) {
      union { uint16_t u[8]; bf16x8 f; } t[3];
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        const float4 v = *reinterpret_cast<const float4*>(qp + s * 16 + e);
        const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; k++) {
          uint32_t a, b, c;
          split3(f[k] * A.qscale, a, b, c);
          t[0].u[e + k] = (uint16_t)a;
          t[1].u[e + k] = (uint16_t)b;
          t[2].u[e + k] = (uint16_t)c;
        }
      }
#pragma unroll
      for (int p = 0; p < 3; p++) qf[p][s] = t[p].f;
    }
  }

  // The four pages of a key tile, one per lane (mod 4), are read a tile ahead of their use, so that no
  // wait for a page ever waits for keys or values in flight.
  auto pages = [&](int t) { return A.page_table[min(t * (KT / PAGE) + (lane & 3), A.max_pages - 1)]; };
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const int wlast = A.pos0 + min(row0 + (wu * 32 + 31) / G, A.M - 1);  // last key of the wave's last row
  auto issue_k = [&](int buf, int pg) {
#pragma unroll
    for (int i = 0; i < KPT; i++) {
      const int ch = i * kWG + tid, key = ch / NCH, c = (ch % NCH) ^ (key & 7);
      const int page = __builtin_amdgcn_readlane(pg, (i * kWG + wu * 64) / (NCH * PAGE));
      const uint16_t* p = A.kv + (size_t)page * page_elems + head_off + (key % PAGE) * DH + c * 8;
      __builtin_amdgcn_global_load_lds((gbytes*)p, (lbytes*)(plds + buf * BUF + (i * kWG + w * 64) * 16), 16, 0, 0);
    }
  };
  // V block of this thread: keys 4 kq .. + 3, dims 8 dg .. + 7
  const int kq = tid / (DH / 8), dg = tid % (DH / 8);
  uint4 vr[4];
  auto load_v = [&](int pg) {
    if (tid >= VTH) return;
    int page = __builtin_amdgcn_readlane(pg, wu * 64 / (DH / 2));
    if (DH == 64 && lane >= 32) page = __builtin_amdgcn_readlane(pg, wu * 2 + 1);
    const uint16_t* p = A.kv + (size_t)page * page_elems + head_off + voff + ((kq & 3) * 4) * DH + dg * 8;
#pragma unroll
    for (int j = 0; j < 4; j++) vr[j] = *reinterpret_cast<const uint4*>(p + j * DH);
  };
  auto store_v = [&](int buf, int t) {
    if (tid >= VTH) return;
    if ((t + 1) * KT > kend) {  // keys past the end may hold anything: zeros, so that 0 * v is 0
#pragma unroll
      for (int j = 0; j < 4; j++)
        if (t * KT + kq * 4 + j >= kend) vr[j] = make_uint4(0u, 0u, 0u, 0u);
    }
    const int slot = (kq & ~3) + ((kq & 1) << 1) + ((kq >> 1) & 1);
    char* vt = plds + buf * BUF + KBUF;
    const uint32_t* a = reinterpret_cast<const uint32_t*>(&vr[0]);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      const uint32_t x = __builtin_amdgcn_perm(a[4 + (e >> 1)], a[e >> 1], sel);
      const uint32_t y = __builtin_amdgcn_perm(a[12 + (e >> 1)], a[8 + (e >> 1)], sel);
      const int dim = dg * 8 + e, ch = (slot >> 1) ^ ((dim ^ (dim >> 3)) & 7);
      *reinterpret_cast<uint2*>(vt + dim * (KT * 2) + ch * 16 + (slot & 1) * 8) = make_uint2(x, y);
    }
  };

  f32x16 o[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) o[t] = (f32x16)(0.f);
  float m_run = -INFINITY, l_run = 0.f;
  // the earlier segments' sums join this one's; keep: the result goes back and this segment's sums start over
  auto fold = [&](bool first, bool keep) {
    float4* tot = A.tot + (((size_t)blockIdx.y * gridDim.x + blockIdx.x) * (kWG / 64) + wu) * ((NT * 4 + 1) * 64) + lane;
    if (!first) {
      const float2 ml = *reinterpret_cast<const float2*>(tot + NT * 4 * 64);
      const float al = __builtin_amdgcn_exp2f(ml.x - m_run);
      l_run = fmaf(ml.y, al, l_run);
#pragma unroll
      for (int b = 0; b < NT * 4; b += 8) {
        float4 x[8];  // a round trip for eight of them
#pragma unroll
        for (int i = 0; i < 8; i++) x[i] = tot[(b + i) * 64];
#pragma unroll
        for (int i = 0; i < 8; i++) {
          const int tt = (b + i) / 4, v = (b + i) % 4 * 4;
          o[tt][v] = fmaf(x[i].x, al, o[tt][v]);
          o[tt][v + 1] = fmaf(x[i].y, al, o[tt][v + 1]);
          o[tt][v + 2] = fmaf(x[i].z, al, o[tt][v + 2]);
          o[tt][v + 3] = fmaf(x[i].w, al, o[tt][v + 3]);
        }
      }
    }
    if (keep) {
#pragma unroll
      for (int tt = 0; tt < NT; tt++) {
#pragma unroll
        for (int i = 0; i < 4; i++)
          tot[(tt * 4 + i) * 64] = make_float4(o[tt][4 * i], o[tt][4 * i + 1], o[tt][4 * i + 2], o[tt][4 * i + 3]);
        o[tt] = (f32x16)(0.f);
      }
      *reinterpret_cast<float2*>(tot + NT * 4 * 64) = make_float2(m_run, l_run);
      l_run = 0.f;
    }
  };

  int pg = pages(0);
  issue_k(0, pg);
  load_v(pg);
  pg = pages(1);
  store_v(0, 0);
  for (int t = 0; t < tiles; t++) {
    const int buf = t & 1;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const bool more = t + 1 < tiles;
    if (more) {
      issue_k(buf ^ 1, pg);
      load_v(pg);
      pg = pages(t + 2);
    }
    const char* kt = plds + buf * BUF;
    const char* vt = kt + KBUF;
#pragma unroll UB
    for (int b = 0; b < 2; b++) {  // 32 keys at a time
      if (t * KT + b * 32 > wlast) continue;  // past every row of the wave
      const int key = b * 32 + col;
      f32x16 s;
#pragma unroll
      for (int k = 0; k < KS; k++) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(kt + key * DH * 2 + (((2 * k + h) ^ (col & 7)) << 4));
#pragma unroll
        for (int p = 2; p >= 0; p--)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[p][k], (p == 2 && k == 0) ? (f32x16)(0.f) : s, 0, 0, 0);
      }
      if (t * KT + b * 32 + 31 > A.pos0 + row0) {  // keys past some row of the workgroup
#pragma unroll
        for (int v = 0; v < 16; v++)
          if (t * KT + b * 32 + 8 * (v >> 2) + 4 * h + (v & 3) > qlim) s[v] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int v = 1; v < 16; v++) mx = fmaxf(mx, s[v]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float mn = fmaxf(m_run, mx);  // finite: key 0 is every row's
      if (__any(mn > m_run)) {
        const float al = __builtin_amdgcn_exp2f(m_run - mn);
        l_run *= al;
#pragma unroll
        for (int tt = 0; tt < NT; tt++)
#pragma unroll
          for (int v = 0; v < 16; v++) o[tt][v] *= al;
        m_run = mn;
      }
      float ps = 0.f;
#pragma unroll
      for (int k = 0; k < 2; k++) {
        union { uint32_t u[4]; bf16x8 f; } pf[3];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(s[8 * k + e] - m_run);
          const float p1 = __builtin_amdgcn_exp2f(s[8 * k + e + 1] - m_run);
          ps += p0 + p1;
          // truncated planes of a finite p >= 0
          const uint32_t h0 = __float_as_uint(p0), h1 = __float_as_uint(p1);
          const float r0 = p0 - __uint_as_float(h0 & 0xffff0000u), r1 = p1 - __uint_as_float(h1 & 0xffff0000u);
          const uint32_t m0 = __float_as_uint(r0), m1 = __float_as_uint(r1);
          const uint32_t l0 = __float_as_uint(r0 - __uint_as_float(m0 & 0xffff0000u));
          const uint32_t l1 = __float_as_uint(r1 - __uint_as_float(m1 & 0xffff0000u));
          pf[0].u[e >> 1] = __builtin_amdgcn_perm(h1, h0, 0x07060302u);
          pf[1].u[e >> 1] = __builtin_amdgcn_perm(m1, m0, 0x07060302u);
          pf[2].u[e >> 1] = __builtin_amdgcn_perm(l1, l0, 0x07060302u);
        }
        const int c = 2 * (2 * b + k) + h;  // 16-byte chunk of V^T's row: this half's eight keys
#pragma unroll
        for (int tt = 0; tt < NT; tt++) {
          const int dim = tt * 32 + col;
          const bf16x8 vf = *reinterpret_cast<const bf16x8*>(vt + dim * (KT * 2) + ((c ^ ((dim ^ (dim >> 3)) & 7)) << 4));
#pragma unroll
          for (int p = 2; p >= 0; p--) o[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[p].f, o[tt], 0, 0, 0);
        }
      }
      l_run += ps + __shfl_xor(ps, 32, 64);
    }
    if (more) store_v(buf ^ 1, t + 1);
    if (t + 1 + kPfSegLast < tiles && (t + 1) % kPfSeg == 0) fold(t + 1 == kPfSeg, true);
  }
  if (tiles > kPfSeg + kPfSegLast) fold(false, false);
  bool nan = l_run != l_run;
#pragma unroll
  for (int tt = 0; tt < NT; tt++)
#pragma unroll
    for (int v = 0; v < 16; v++) nan = nan || o[tt][v] != o[tt][v];
  const bool mine = row0 + qi / G < A.M;
  const unsigned long long nans = __ballot(nan && mine);
  if (lane == 0) s_nan[w] = (uint32_t)nans | (uint32_t)(nans >> 32);
  if (mine) {
    const float inv = 1.0f / l_run;
    const size_t at = (size_t)qr * qd + (size_t)qh * DH + 4 * h;
#pragma unroll
    for (int tt = 0; tt < NT; tt++)
#pragma unroll
      for (int v = 0; v < 16; v += 4)
        store_planes4(A.out, at + tt * 32 + 2 * v, o[tt][v] * inv, o[tt][v + 1] * inv, o[tt][v + 2] * inv,
                      o[tt][v + 3] * inv);
  }
  __syncthreads();  // every wave's queries are stored, and the key tiles are free
  for (int ww = 0; ww < kWG / 64; ww++)
    for (uint32_t m = __builtin_amdgcn_readfirstlane(s_nan[ww]); m != 0u; m &= m - 1u) {
      const int j = ww * 32 + __builtin_ctz(m), row = row0 + j / G;
      const size_t at = (size_t)row * qd + (size_t)(g * G + j % G) * DH;
      float a[4], M, L;
      if (attn_query_plain<DH>(A.kv, A.page_table, A.hkv, g, A.q + at, A.scale, 0, A.pos0 + row + 1,
                               reinterpret_cast<float*>(plds), M, L, a)) {
        const float inv = 1.0f / L;
        store_planes4(A.out, at + 4 * (tid % (DH / 4)), a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv);
      }
    }
}

// ---------------------------------------------------------------------------------------- launches
// Tile and K splits of a projection. Up to eight rows take the row GEMM (k_pf_rows). Above 192 rows the tiles are 128 x 256, one eight-wave workgroup
// per CU; up to 192 rows 64 x 128 and up to 32 rows 32 x 128, two workgroups per CU: fewer padding rows
// and more workgroups where the weights' stream is the bound (19456 x 2560 at 128 rows: 55 us against
// 107 us; at 45 rows 39 us). The splits are those of the least cost, in inputs of one tile: a round of
// workgroups costs its inputs plus about 288 of prologue and epilogue, a split the traffic of its
// partial sums (QKV at 1501 rows: one split 205 us, two 156 + 22 us of pair epilogue).
struct GemmPlan {
  int bm, S, KS;
};

GemmPlan plan_gemm(int M, int cols, int K, size_t part_cap) {
  GemmPlan p;
  p.bm = M <= kMaxRows ? kMaxRows : M <= 32 ? 32 : M <= 192 ? 64 : 128;
  const int bn = p.bm == 128 ? 256 : 128, slots = p.bm == 128 ? 256 : 512;
  const long long tiles = (long long)((M + p.bm - 1) / p.bm) * ((cols + bn - 1) / bn);
  double best = 0.0;
  p.S = 1;
  for (int S = 1; S <= kPrefillMaxSplit; S++) {
    const int KS = ((K + S - 1) / S + 63) / 64 * 64;
    if (S > 1 && ((size_t)S * std::max(M, kMaxRows) * cols > part_cap || KS < 256 || (S - 1) * KS >= K)) continue;
    const double cost = (double)((tiles * S + slots - 1) / slots) * (KS + 288) + (S > 1 ? S * 3.3e-5 * M * cols : 0.0);
    if (S == 1 || cost < best) {
      best = cost;
      p.S = S;
    }
  }
  p.KS = ((K + p.S - 1) / p.S + 63) / 64 * 64;
  return p;
}

template <int WM, int WN, int NWM, int NWN, int BK, int KIND>
void launch_gemm(GemmArgs G, int S, hipStream_t s) {
  constexpr int BM = WM * NWM, BN = WN * NWN;
  const int ncol = KIND == GK_PLAIN ? G.cols : 2 * G.cols;
  G.mt = (G.M + BM - 1) / BM;
  G.nt = (ncol + BN - 1) / BN;
  const size_t shm = (size_t)2 * (3 * BM + BN) * BK * 2;
  launch_timed((k_pf_gemm<WM, WN, NWM, NWN, BK, KIND>), dim3(G.mt * G.nt * S), dim3(64 * NWM * NWN), shm, s, G);
}

// One projection; returns the number of partial sums left in B.part (0: the pair epilogue has run). rows:
// G.M, or the most rows G.st can say. cap: at most this many workgroups of the row GEMM (0: no cap).
template <int KIND>
int gemm(const PrefillBufs& B, GemmArgs G, hipStream_t s, int cap = 0) {
  const int ncol = KIND == GK_PLAIN ? G.cols : 2 * G.cols;
  const GemmPlan p = plan_gemm(G.M, ncol, G.K, B.part_cap);
  G.KS = p.KS;
  G.S = p.S;
  G.zeros = B.zeros;
  // pairs meet in one lane only in the two-tile waves of the taller shapes
  const bool direct = KIND != GK_PLAIN && p.S == 1 && p.bm > 32;
  G.part = direct ? nullptr : B.part;
  int prows = G.M;
  if (p.bm == kMaxRows) {
    prows = kMaxRows;
    G.nt = (ncol + 127) / 128;
    const int jobs = G.nt * p.S;
    launch_timed((k_pf_rows<KIND>), dim3(cap > 0 ? std::min(cap, jobs) : jobs), dim3(kWG),
                 (size_t)kRowBufs * (32 + 128) * 64 * 2, s, G);
  } else if (p.bm == 32) {
    launch_gemm<32, 32, 1, 4, 64, KIND>(G, p.S, s);
  } else if (p.bm == 64) {
    launch_gemm<32, 64, 2, 2, 64, KIND>(G, p.S, s);
  } else {
    launch_gemm<64, 64, 2, 4, 32, KIND>(G, p.S, s);
  }
  if constexpr (KIND == GK_PLAIN) {
    return p.S;
  } else {
    if (!direct)
      launch_timed((k_pf_pairs<KIND>), dim3((G.cols + kWG - 1) / kWG, G.M), dim3(kWG), 0, s, G.out,
                   (const float*)B.part, p.S, prows, G.cols, G.st);
    return 0;
  }
}

// Floats of one split of a plain projection of `rows` rows: see k_pf_rows and k_pf_gemm.
size_t part_stride(int rows, int d) { return (size_t)(rows <= kMaxRows ? kMaxRows : rows) * d; }

void attention(const Ctx& C, AttnArgs A, hipStream_t s) {
  const int rpw = 128 / A.G;
  const dim3 grid(A.hkv, (A.M + rpw - 1) / rpw);
  const size_t shm = (size_t)2 * 2 * 64 * C.dh * 2;
  if (C.dh == 128)
    launch_timed((k_pf_attn<128>), grid, dim3(kWG), shm, s, A);
  else
    launch_timed((k_pf_attn<64>), grid, dim3(kWG), shm, s, A);
}

}  // namespace

int prefill_chunk_rows(int d, int F, int qdim, int qkv_cols) {
  auto bytes = [&](size_t rows) {
    return 4 * (2 * rows * d + prefill_part_floats((int)rows, d, F, qkv_cols) + rows) + 6 * rows * std::max(d, qdim) +
           std::max(6 * rows * std::max(d, F), 4 * rows * qdim);
  };
  int rows = kPrefillRows;
  while (rows > kPrefillMinRows && bytes(rows) > kPrefillBytes) rows -= 128;
  return rows;
}

// Partial sums: four splits of the narrow projections and two of QKV over a full chunk, and four of the
// wide ones over a chunk of 128 rows (longer chunks have tiles enough without splitting those).
size_t prefill_part_floats(int rows, int d, int F, int qkv_cols) {
  return std::max(std::max((size_t)4 * rows * d, (size_t)2 * rows * qkv_cols),
                  (size_t)4 * 128 * std::max(2 * F, qkv_cols));
}

void prefill_mfma(const Ctx& C, const PrefillBufs& B, const LayerDesc* layers, int len, void* stream, int* last_row) {
  hipStream_t s = (hipStream_t)stream;
  const int d = C.d, qkv_pairs = (C.hq + 2 * C.hkv) * (C.dh / 2);
  const int nch = (len + B.rows - 1) / B.rows;
  const int step = ((len + nch - 1) / nch + 127) / 128 * 128;  // equal chunks
  const size_t pa_w = std::max(d, C.qdim), pb_w = std::max(d, C.F);
  const Planes pa{B.pa, (size_t)B.rows * pa_w}, pb{B.pb, (size_t)B.rows * pb_w};

  for (int t0 = 0; t0 < len; t0 += step) {
    const int M = std::min(step, len - t0);
    const bool last = t0 + M == len;
    int S = 0;  // partial sums that wait in B.part
    auto norm = [&](float* x, int rows, int base, const float* gain, bool raw) {
      NormArgs N{};
      N.x = x;
      N.d = d;
      N.S = S;
      N.base = base;
      N.part = B.part;
      N.part_stride = part_stride(rows, d);
      N.tok = C.tok + t0;
      N.embed = (const uint16_t*)C.embed;
      N.gain = gain;
      N.eps = C.eps;
      N.out = pa;
      if (raw) N.raw = pb;
      N.rs = B.rs;
      launch_timed(k_pf_norm, dim3(rows), dim3(kWG), 0, s, N);
      S = 0;
    };
    auto plain = [&](const Planes& a, int rows, int K, const void* w, int ldw) {
      GemmArgs G{};
      G.a = a;
      G.w0 = (const uint16_t*)w;
      G.M = rows;
      G.K = K;
      G.ldw = ldw;
      G.cols = d;
      S = gemm<GK_PLAIN>(B, G, s);
    };
    auto qkv = [&](const LayerDesc& L) {
      GemmArgs G{};
      G.a = pa;
      G.w0 = (const uint16_t*)L.wq;
      G.w1 = (const uint16_t*)L.wk;
      G.w2 = (const uint16_t*)L.wv;
      G.M = M;
      G.K = d;
      G.ldw = d;
      G.cols = qkv_pairs;
      G.out.rs = B.rs;
      G.out.q = B.q;
      G.out.kv = (uint16_t*)L.kv;
      G.out.page_table = C.page_table;
      G.out.rope = C.rope;
      G.out.pos0 = t0;
      G.out.hq = C.hq;
      G.out.hkv = C.hkv;
      G.out.dh = C.dh;
      G.out.page = C.page;
      gemm<GK_QKV>(B, G, s);
    };
    // attention, O-proj, MLP of rows r0 .. M - 1; leaves the down projection's partial sums
    auto rest = [&](const LayerDesc& L, float* x, int r0) {
      const int rows = M - r0;
      AttnArgs A{};
      A.q = B.q + (size_t)r0 * C.qdim;
      A.out = pa;
      A.kv = (const uint16_t*)L.kv;
      A.page_table = C.page_table;
      A.M = rows;
      A.pos0 = t0 + r0;
      A.G = C.G;
      A.hkv = C.hkv;
      A.max_pages = C.max_pages;
      A.scale = C.scale;
      A.tot = reinterpret_cast<float4*>(B.part);  // free here; fits: rows (a multiple of 128) * qdim * 9/8 floats at most
      A.qscale = C.scale * 1.44269504088896340736f;
      attention(C, A, s);
      plain(pa, rows, C.qdim, L.wo, C.qdim);
      norm(x + (size_t)r0 * d, rows, 0, L.mlp_norm, false);
      GemmArgs G{};
      G.a = pa;
      G.w0 = (const uint16_t*)L.wg;
      G.w1 = (const uint16_t*)L.wu;
      G.M = rows;
      G.K = d;
      G.ldw = d;
      G.cols = C.F;
      G.out.rs = B.rs;
      G.out.act = pb;
      G.out.F = C.F;
      gemm<GK_GATEUP>(B, G, s);
      plain(pb, rows, C.F, L.wd, C.F);
    };

    int stage = 0;
    for (int l = 0; l < C.L; l++) {
      const bool opens = stage < C.n && l == C.beta[stage];  // a stage's input is an anchor
      norm(B.x, M, l == 0 ? 1 : 0, layers[l].attn_norm, opens);
      if (opens) {  // the draft module's feature projection, one anchor's columns at a time
        plain(pb, M, d, (const uint16_t*)C.w_in + (size_t)stage * d, C.n * d);
        norm(B.px, M, stage == 0 ? 2 : 0, nullptr, false);
        stage++;
      }
      qkv(layers[l]);
      if (l + 1 < C.L)
        rest(layers[l], B.x, 0);
      else if (last) {  // only the prompt's last row is read past the last layer's keys and values
        rest(layers[l], B.x, M - 1);
        norm(B.x + (size_t)(M - 1) * d, 1, 0, nullptr, false);
        *last_row = M - 1;
      }
    }
    for (int i = 0; i < C.ls; i++) {
      const LayerDesc& L = layers[C.L + i];
      norm(B.px, M, 0, L.attn_norm, false);
      qkv(L);
      if (i + 1 < C.ls) rest(L, B.px, 0);  // the last layer's rows are not read: its caches only
    }
  }
}

void pdm_rows_mfma(const Ctx& C, const PrefillBufs& B, const LayerDesc* layers, int max_rows, int cap, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int d = C.d, K = C.n * d;
  const Planes pa{B.pa, (size_t)kMaxRows * std::max(d, C.qdim)}, pb{B.pb, (size_t)kMaxRows * std::max(K, C.F)};
  int S = 0;
  auto norm = [&](int base, const float* gain) {
    NormArgs N{};
    N.st = C.st;
    N.x = C.pdm_x;
    N.d = d;
    N.S = S;
    N.base = base;
    N.part = B.part;
    N.part_stride = part_stride(max_rows, d);
    N.gain = gain;
    N.eps = C.eps;
    N.out = pa;
    N.rs = B.rs;
    launch_timed(k_pf_norm, dim3(max_rows), dim3(kWG), 0, s, N);
  };
  auto args = [&](const Planes& a, int k, const void* w, int ldw, int cols) {
    GemmArgs G{};
    G.st = C.st;
    G.a = a;
    G.w0 = (const uint16_t*)w;
    G.M = max_rows;
    G.K = k;
    G.ldw = ldw;
    G.cols = cols;
    G.out.rs = B.rs;
    return G;
  };
  launch_timed(k_pdm_feat, dim3((K / 4 + kWG - 1) / kWG, max_rows), dim3(kWG), 0, s, C, pb);
  {
    GemmArgs G = args(pb, K, C.w_in, K, d);
    if (C.ktrace != nullptr) G.trace = C.ktrace + 2 * (5 * C.J * C.n + KT_PDM);
    S = gemm<GK_PLAIN>(B, G, s, cap);
  }
  for (int i = 0; i < C.ls; i++) {
    const LayerDesc& L = layers[C.L + i];
    norm(i == 0 ? 2 : 0, L.attn_norm);
    GemmArgs Q = args(pa, d, L.wq, d, (C.hq + 2 * C.hkv) * (C.dh / 2));
    Q.w1 = (const uint16_t*)L.wk;
    Q.w2 = (const uint16_t*)L.wv;
    Q.out.q = C.b[1].q;
    Q.out.kv = (uint16_t*)L.kv;
    Q.out.page_table = C.page_table;
    Q.out.rope = C.rope;
    Q.out.hq = C.hq;
    Q.out.hkv = C.hkv;
    Q.out.dh = C.dh;
    Q.out.page = C.page;
    gemm<GK_QKV>(B, Q, s, cap);
    const int rpg = 32 / C.G, M = std::min(max_rows, rpg) * C.G;
    const dim3 grid(C.max_splits, C.hkv, (max_rows + rpg - 1) / rpg), mgrid(C.hkv, max_rows);
    if (C.dh == 128) {
      launch_timed((k_pdm_attn<128>), grid, dim3(kWG), attn_mfma_lds<128>(M), s, C, (const uint16_t*)L.kv, pa);
      if (C.max_splits > 1) launch_timed((k_pdm_attn_merge<128>), mgrid, dim3(kWG), 0, s, C, pa);
    } else {
      launch_timed((k_pdm_attn<64>), grid, dim3(kWG), attn_mfma_lds<64>(M), s, C, (const uint16_t*)L.kv, pa);
      if (C.max_splits > 1) launch_timed((k_pdm_attn_merge<64>), mgrid, dim3(kWG), 0, s, C, pa);
    }
    S = gemm<GK_PLAIN>(B, args(pa, C.qdim, L.wo, C.qdim, d), s, cap);
    norm(0, L.mlp_norm);
    GemmArgs U = args(pa, d, L.wg, d, C.F);
    U.w1 = (const uint16_t*)L.wu;
    U.out.act = pb;
    U.out.F = C.F;
    gemm<GK_GATEUP>(B, U, s, cap);
    S = gemm<GK_PLAIN>(B, args(pb, C.F, L.wd, C.F, d), s, cap);
  }
  norm(0, nullptr);
}

}  // namespace spd
