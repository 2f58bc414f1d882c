// Decode attention of one token over one KV head's paged cache, one key split per workgroup. The stage
// launches, the row blocks in vector form and the ragged calls in vector form share it, so they compute
// the same bits; the second half of the file is the form for rows that share a cache, on matrix cores.
//
// The token at position pos0 attends to keys 0..pos0 of its own layer (Section 3.1: each stage's
// token reads the cache of the layer it is on). Its G query heads share KV head g (grouped-query
// attention). A split covers keys [k0, k1) in rounds of 64 keys, 16 per wave, and the waves never
// wait for each other inside the split:
//   * lane l of a wave owns key l/4 of the wave's 16 and a quarter of the head dimension, for K and V
//     alike (one page-table lookup serves both); a round's loads are issued two rounds ahead and the
//     page of the round after is requested before them, so no wait for a page ever waits for K or V;
//   * scores are dot products over the quarter, summed across the four lanes of a key with DPP; the
//     lanes of a key then split the heads between them (head h on lane h mod 4), so the online
//     softmax of a head is a 16-lane max and sum;
//   * P.V goes through a wave-private LDS tile: lane l accumulates one head's slice of dimensions over
//     the wave's keys in key order.
// Each wave keeps its own running (m, l, o); the four are combined in wave order at the end of the
// split (one barrier). With one split the workgroup writes the output; otherwise the split that
// finishes last (a ticket per stage and head) merges every split in split order, its loads for up to
// 32 splits issued at once. The split size is a function of the configuration only, so a token's
// result never depends on how many stages run.
#pragma once
#include <type_traits>

#include "spd_devfn.h"

namespace spd {

constexpr int kAttnTPK = 4;                   // lanes per key
constexpr int kAttnWaveKeys = 64 / kAttnTPK;  // keys per wave per round
constexpr int kAttnPass = kWG / kAttnTPK;     // keys per round
constexpr int kAttnMaxQ = 8;                  // query heads per KV head
constexpr int kAttnMergeBatch = 32;           // splits whose partial outputs the merge loads at once

// LDS: pre-scaled queries, then per wave a V tile (reused for the wave's o at the end), its
// probabilities, and its rescale factors and (m, l).
template <typename KVT, int DH>
struct AttnLds {
  static constexpr int kWaves = kWG / 64;
  static constexpr size_t kQ = (size_t)kAttnMaxQ * DH * 4;
  static constexpr size_t kTile = (size_t)kAttnWaveKeys * DH * sizeof(KVT);
  static constexpr size_t kO = (size_t)kAttnMaxQ * DH * 4;
  static constexpr size_t kVt = kTile > kO ? kTile : kO;
  static constexpr size_t kP = (size_t)kAttnMaxQ * kAttnWaveKeys * 4;
  static constexpr size_t kA = (size_t)kAttnMaxQ * 4 * 3;  // alpha, m, l
  static constexpr size_t kWave = kVt + kP + kA;
  static constexpr size_t kTotal = kQ + kWaves * kWave;
};

template <typename KVT, int DH>
constexpr size_t attn_split_lds() {
  return AttnLds<KVT, DH>::kTotal;
}

// KV cache reads. Ordinary loads: a round's keys come back faster than with the non-temporal hint.
__device__ __forceinline__ uint4 ldkv16(const void* p) { return *reinterpret_cast<const uint4*>(p); }

__device__ __forceinline__ void st_dev2f(float* p, float x, float y) {  // p 8-byte aligned
  const unsigned long long u = (unsigned long long)__float_as_uint(x) | ((unsigned long long)__float_as_uint(y) << 32);
  __hip_atomic_store((unsigned long long*)p, u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over the four lanes of a quad (DPP quad permutes); all four lanes get the same bits.
__device__ __forceinline__ float quad_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));  // lane ^ 1
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));  // lane ^ 2
  return v;
}

// Max / sum over the 16 lanes of a wave that share lane mod 4; every such lane gets the same bits.
__device__ __forceinline__ float key_max(float v) {
#pragma unroll
  for (int m = 4; m < 64; m <<= 1) v = fmaxf(v, __shfl_xor(v, m, 64));
  return v;
}
__device__ __forceinline__ float key_sum(float v) {
#pragma unroll
  for (int m = 4; m < 64; m <<= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Orders the wave's LDS writes before its later LDS reads of other lanes' data (one wave executes
// its LDS operations in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// N consecutive KV elements from LDS as floats (N * sizeof(T): 8 bytes or a multiple of 16, aligned).
template <typename T, int N>
__device__ __forceinline__ void lds_row(const T* p, float* o) {
  constexpr int BYTES = N * (int)sizeof(T);
  if constexpr (BYTES % 16 == 0) {
#pragma unroll
    for (int c = 0; c < BYTES / 16; c++)
      unpack16<T>(reinterpret_cast<const uint4*>(p)[c], o + c * (16 / (int)sizeof(T)));
  } else {
    static_assert(BYTES == 8, "row of 8 bytes or a multiple of 16");
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    if constexpr (sizeof(T) == 2) {
      o[0] = bf_lo(u.x);
      o[1] = bf_hi(u.x);
      o[2] = bf_lo(u.y);
      o[3] = bf_hi(u.y);
    } else {
      o[0] = __uint_as_float(u.x);
      o[1] = __uint_as_float(u.y);
    }
  }
}

// Where an attention writes its output: two consecutive values at an (even) element offset.
struct FloatOut {
  float* p;
  __device__ __forceinline__ void operator()(size_t at, float a, float b) const {
    *reinterpret_cast<float2*>(p + at) = make_float2(a, b);
  }
};
template <typename Out>
struct ShiftedOut {  // Out, from an element offset on
  Out out;
  size_t base;
  __device__ __forceinline__ void operator()(size_t at, float a, float b) const { out(base + at, a, b); }
};

// Merge of one (token, KV head)'s nsplit split records (o[8][DH], m[8], l[8]; every split has a key,
// so each m is finite) in split order into its G output rows. Every thread of the workgroup calls it.
// All (m, l) pairs are requested first, then the first batch of partial outputs (only the entries
// that exist: the records are read past the L2, where a repeated address costs as much as a new
// one), then the (m, l) pairs go to LDS (sm: 2 * kMaxSplits * kAttnMaxQ floats). DEV: the records come
// from workgroups of the same launch (device-scope loads); else from an earlier launch.
template <int DH, bool DEV, typename Out>
__device__ __forceinline__ void attn_merge(const float* rec_base, int nsplit, int G, const Out out, float* sm) {
  constexpr int MAXQ = kAttnMaxQ, RS = MAXQ * (DH + 2);
  constexpr int NPAIR = MAXQ * DH / 2;
  constexpr int PPT = (NPAIR + kWG - 1) / kWG;
  const int tid = threadIdx.x;
  auto get = [](const float* p) { return DEV ? ld_dev(p) : *p; };
  auto get2 = [](const float* p) { return DEV ? ld_dev2(p) : *reinterpret_cast<const float2*>(p); };
  constexpr int MB = kAttnMergeBatch;
  constexpr int MLT = (kMaxSplits * MAXQ + kWG - 1) / kWG;
  float* sl = sm + kMaxSplits * MAXQ;
  float mlm[MLT], mll[MLT];
#pragma unroll
  for (int i = 0; i < MLT; i++) {
    const int t = tid + i * kWG, sp = t / G, qi = t % G;
    mlm[i] = mll[i] = 0.f;
    if (t < nsplit * G) {
      mlm[i] = get(rec_base + (size_t)sp * RS + MAXQ * DH + qi);
      mll[i] = get(rec_base + (size_t)sp * RS + MAXQ * DH + MAXQ + qi);
    }
  }
  const int qi0 = tid / (DH / 2), dp0 = tid % (DH / 2);
  const int qc0 = min(qi0, G - 1);
  float2 ob[MB];
#pragma unroll
  for (int j = 0; j < MB; j++)
    ob[j] = (j < nsplit && qi0 < G) ? get2(rec_base + (size_t)j * RS + qc0 * DH + 2 * dp0) : make_float2(0.f, 0.f);
#pragma unroll
  for (int i = 0; i < MLT; i++) {
    const int t = tid + i * kWG;
    if (t < nsplit * G) {
      sm[(t / G) * MAXQ + t % G] = mlm[i];
      sl[(t / G) * MAXQ + t % G] = mll[i];
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < PPT; i++) {
    const int e = tid + i * kWG, qi = e / (DH / 2), dp = e % (DH / 2);
    if (qi < G) {
      float M = -INFINITY;
      for (int sp = 0; sp < nsplit; sp++) M = fmaxf(M, sm[sp * MAXQ + qi]);
      float L = 0.f, a0 = 0.f, a1 = 0.f;
      for (int sp0 = 0; sp0 < nsplit; sp0 += MB) {
        if (i > 0 || sp0 > 0) {
#pragma unroll
          for (int j = 0; j < MB; j++)
            ob[j] = get2(rec_base + (size_t)min(sp0 + j, nsplit - 1) * RS + qi * DH + 2 * dp);
        }
#pragma unroll
        for (int j = 0; j < MB; j++) {
          if (sp0 + j < nsplit) {
            const float f = expf(sm[(sp0 + j) * MAXQ + qi] - M);
            L = fmaf(sl[(sp0 + j) * MAXQ + qi], f, L);
            a0 = fmaf(ob[j].x, f, a0);
            a1 = fmaf(ob[j].y, f, a1);
          }
        }
      }
      const float inv = 1.0f / L;
      if constexpr (std::is_same<Out, float*>::value)
        *reinterpret_cast<float2*>(out + qi * DH + 2 * dp) = make_float2(a0 * inv, a1 * inv);
      else
        out((size_t)qi * DH + 2 * dp, a0 * inv, a1 * inv);
    }
  }
}

// One split with GP head slots (4: G <= 4, 8: G <= 8). Arguments as for attn_split.
template <typename KVT, int DH, int GP>
__device__ bool attn_split_g(const Ctx& C, const KVT* kvb, const float* q, float* out, float* rec_base, int* cnt,
                             int g, int split, int nsplit, int k0, int k1, int pos0, int page0, float* lds) {
  constexpr int TPK = kAttnTPK, NE = DH / TPK, VE = Elt<KVT>::VE, KCH = NE / VE;
  constexpr int WK = kAttnWaveKeys, PASS = kAttnPass, MAXQ = kAttnMaxQ, NJ = GP / 4;
  constexpr int LPH = 64 / GP, DPL = DH / LPH;  // P.V: lanes per head, dimensions per lane
  constexpr int KUNR = DPL > 8 ? 2 : 4;          // P.V keys in flight
  constexpr int RS = MAXQ * (DH + 2);
  using LA = AttnLds<KVT, DH>;
  __shared__ int s_last;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int kk = lane / TPK, qq = lane % TPK;
  const int G = C.G;
  char* const lbase = reinterpret_cast<char*>(lds);
  float* qs = lds;                                                  // [MAXQ][DH] pre-scaled queries
  char* wbase = lbase + LA::kQ + (size_t)w * LA::kWave;
  KVT* vt = reinterpret_cast<KVT*>(wbase);                          // [WK][DH] V tile, then o [MAXQ][DH]
  float* pt = reinterpret_cast<float*>(wbase + LA::kVt);            // [MAXQ][WK] probabilities
  float* at = reinterpret_cast<float*>(wbase + LA::kVt + LA::kP);   // alpha[MAXQ], m[MAXQ], l[MAXQ]
  const size_t page_elems = (size_t)2 * C.hkv * C.page * DH;
  const size_t head_off = (size_t)g * C.page * DH;
  const size_t voff = (size_t)C.hkv * C.page * DH;
  const int R = (k1 - k0 + PASS - 1) / PASS;  // rounds
  const int my = w * WK + kk;                 // this lane's key within a round

  // Every global load below is unconditional (keys past the split read the slot of key k1 - 1, in
  // round 0 of the page their own key falls in, and are masked later), so the count of loads issued after any given load is the same on every path and each
  // wait covers exactly the loads it needs: queries first, then the page of round 1, round 0, the
  // page of round 2, round 1.
  constexpr int QPT = (MAXQ * DH + kWG - 1) / kWG;
  float qv[QPT];
#pragma unroll
  for (int i = 0; i < QPT; i++) {
    const int e = min(tid + i * kWG, G * DH - 1);
    qv[i] = q[e];
  }
  auto page_of = [&](int r) { return C.page_table[min(k0 + r * PASS + my, k1 - 1) / C.page]; };
  int pg_next = page_of(1);
  uint4 kb0[KCH], vb0[KCH], kb1[KCH], vb1[KCH];
  auto issue = [&](int r, int page, uint4* kr, uint4* vr) {
    const int key = min(k0 + r * PASS + my, k1 - 1);
    const KVT* base = kvb + (size_t)page * page_elems + head_off + (size_t)(key % C.page) * DH + qq * NE;
#pragma unroll
    for (int c = 0; c < KCH; c++) kr[c] = ldkv16(reinterpret_cast<const uint4*>(base) + c);
#pragma unroll
    for (int c = 0; c < KCH; c++) vr[c] = ldkv16(reinterpret_cast<const uint4*>(base + voff) + c);
  };
  issue(0, page0, kb0, vb0);
  {
    const int pg1 = pg_next;
    pg_next = page_of(2);
    issue(1, pg1, kb1, vb1);
  }
#pragma unroll
  for (int i = 0; i < QPT; i++) qs[tid + i * kWG] = qv[i] * C.scale;  // slots >= G: unused
  __syncthreads();  // queries staged

  float m_run[NJ], l_run[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    m_run[j] = -INFINITY;
    l_run[j] = 0.f;
  }
  const int ph = lane / LPH, pd = (lane % LPH) * DPL;  // P.V: head slot and first dimension
  float o[DPL];
#pragma unroll
  for (int e = 0; e < DPL; e++) o[e] = 0.f;

  auto round = [&](int r, uint4* kr_raw, uint4* vr_raw) {
    const int kbase = k0 + r * PASS + w * WK;  // the wave's first key in this round
    const int nkw = min(WK, k1 - kbase);       // wave-uniform
    float kf[NE];
#pragma unroll
    for (int c = 0; c < KCH; c++) unpack16<KVT>(kr_raw[c], kf + c * VE);
    // a key past the end may come from a page beyond the cache's length (round 0's page is looked up
    // before the length is known), whose contents are arbitrary: its V row enters the tile as zeros,
    // so that its zero probability keeps the sums exact even if those bytes are not a finite number
    const bool kin = kk < nkw;
#pragma unroll
    for (int c = 0; c < KCH; c++)
      reinterpret_cast<uint4*>(vt + kk * DH + qq * NE)[c] = kin ? vr_raw[c] : make_uint4(0u, 0u, 0u, 0u);
    {  // the buffers are free again: round r + 2, and the page of round r + 3 (past the end: key k1 - 1)
      const int pg = pg_next;
      pg_next = page_of(r + 3);
      issue(r + 2, pg, kr_raw, vr_raw);
    }
    if (nkw > 0) {  // else the wave has no key in this round
      const bool valid = kk < nkw;
      float sel[NJ];
#pragma unroll
      for (int j = 0; j < NJ; j++) sel[j] = -INFINITY;
#pragma unroll
      for (int qi = 0; qi < GP; qi++) {
        if (qi < G) {
          const float* qp = qs + qi * DH + qq * NE;
          float dsum = 0.f;
#pragma unroll
          for (int e = 0; e < NE; e += 4) {
            const float4 q4 = *reinterpret_cast<const float4*>(qp + e);
            dsum = fmaf(q4.x, kf[e], dsum);
            dsum = fmaf(q4.y, kf[e + 1], dsum);
            dsum = fmaf(q4.z, kf[e + 2], dsum);
            dsum = fmaf(q4.w, kf[e + 3], dsum);
          }
          dsum = quad_sum(dsum);
          if ((qi & 3) == qq) sel[qi >> 2] = valid ? dsum : -INFINITY;
        }
      }
      // online softmax of head qq + 4j over the wave's keys (key 0 of the round is valid, so mn is
      // finite for every head h < G unless its scores are all -inf, which leaves l as it was, or NaN,
      // which makes l NaN)
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        const int h = qq + 4 * j;
        const float mx = key_max(sel[j]);
        const float mn = fmaxf(m_run[j], mx);
        const float al = m_run[j] == -INFINITY ? 0.f : expf(m_run[j] - mn);
        const float p = sel[j] == -INFINITY ? 0.f : expf(sel[j] - mn);  // past the end, h >= G, or a score of -inf
        const float ps = key_sum(p);
        l_run[j] = l_run[j] * al + ps;
        m_run[j] = mn;
        if (h < G) {
          pt[h * WK + kk] = p;
          if (kk == 0) at[h] = al;
        }
      }
      wave_lds_sync();
      if (ph < G) {
        const float al = at[ph];
#pragma unroll
        for (int e = 0; e < DPL; e++) o[e] *= al;
        const float* pp = pt + ph * WK;
#pragma unroll KUNR
        for (int k = 0; k < WK; k++) {
          float v[DPL];
          lds_row<KVT, DPL>(vt + k * DH + pd, v);
          const float pk = pp[k];
#pragma unroll
          for (int e = 0; e < DPL; e++) o[e] = fmaf(pk, v[e], o[e]);
        }
      }
    }
    wave_lds_sync();  // the tile and probabilities are rewritten next round
  };
  for (int r = 0; r < R; r += 2) {  // an odd count ends with a round that has no key
    round(r, kb0, vb0);
    round(r + 1, kb1, vb1);
  }

  // the wave's (m, l, o) to LDS; o reuses the V tile
  float* ow = reinterpret_cast<float*>(vt);
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    const int h = qq + 4 * j;
    if (kk == 0 && h < G) {
      at[MAXQ + h] = m_run[j];
      at[2 * MAXQ + h] = l_run[j];
    }
  }
  if (ph < G) {
#pragma unroll
    for (int e = 0; e < DPL; e++) ow[ph * DH + pd + e] = o[e];
  }
  __syncthreads();

  // combine the waves in wave order: (A, M, L) of the split per (head, dimension pair); a wave with
  // no key has l = 0 and weight 0 (a NaN l counts even where the wave's maximum is still -inf)
  constexpr int NW = LA::kWaves;
  constexpr int NPAIR = MAXQ * DH / 2;
  constexpr int PPT = (NPAIR + kWG - 1) / kWG;
  float A0[PPT], A1[PPT], Ms[PPT], Ls[PPT];
#pragma unroll
  for (int i = 0; i < PPT; i++) {
    const int e = tid + i * kWG, qi = e / (DH / 2), dp = e % (DH / 2);
    A0[i] = A1[i] = Ms[i] = Ls[i] = 0.f;
    if (qi < G) {
      float M = -INFINITY;
#pragma unroll
      for (int wv = 0; wv < NW; wv++)
        M = fmaxf(M, reinterpret_cast<const float*>(lbase + LA::kQ + (size_t)wv * LA::kWave + LA::kVt + LA::kP)[MAXQ + qi]);
      float L = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; wv++) {
        const char* wb = lbase + LA::kQ + (size_t)wv * LA::kWave;
        const float* aw = reinterpret_cast<const float*>(wb + LA::kVt + LA::kP);
        const float lw = aw[2 * MAXQ + qi];
        if (lw != 0.f) {
          const float f = expf(aw[MAXQ + qi] - M);
          L = fmaf(lw, f, L);
          const float2 ov = *reinterpret_cast<const float2*>(reinterpret_cast<const float*>(wb) + qi * DH + 2 * dp);
          a0 = fmaf(ov.x, f, a0);
          a1 = fmaf(ov.y, f, a1);
        }
      }
      A0[i] = a0;
      A1[i] = a1;
      Ms[i] = M;
      Ls[i] = L;
    }
  }
  if (nsplit == 1) {
#pragma unroll
    for (int i = 0; i < PPT; i++) {
      const int e = tid + i * kWG, qi = e / (DH / 2), dp = e % (DH / 2);
      if (qi < G) {
        const float inv = 1.0f / Ls[i];
        *reinterpret_cast<float2*>(out + qi * DH + 2 * dp) = make_float2(A0[i] * inv, A1[i] * inv);
      }
    }
    return true;
  }
  float* rec = rec_base + (size_t)split * RS;
#pragma unroll
  for (int i = 0; i < PPT; i++) {
    const int e = tid + i * kWG, qi = e / (DH / 2), dp = e % (DH / 2);
    if (qi < G) {
      st_dev2f(rec + qi * DH + 2 * dp, A0[i], A1[i]);
      if (dp == 0) {
        st_dev(rec + MAXQ * DH + qi, Ms[i]);
        st_dev(rec + MAXQ * DH + MAXQ + qi, Ls[i]);
      }
    }
  }
  wait_own_stores();
  __syncthreads();
  if (tid == 0) {
    const int t = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (t == nsplit - 1);
  }
  __syncthreads();
  if (!s_last) return false;

  attn_merge<DH, true>(rec_base, nsplit, G, out, reinterpret_cast<float*>(lbase + LA::kQ));
  if (tid == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// ------------------------------------------------------------------ bf16 caches on matrix cores
// One key split [k0, k0 + chunk) of KV head g for up to 32 / G rows that read the same cache: row r's G
// query heads attend keys 0 .. lim(r). The nrows * G <= 32 queries (query j = r * G + h) are the columns
// of 32 x 32 MFMA tiles (v_mfma_f32_32x32x16_bf16: lane l supplies 8 consecutive k of A row l % 32 and
// of B column l % 32, from k = 8 (l / 32); accumulator register v of lane l is row 8 (v / 4) + 4 (l / 32)
// + v % 4, column l % 32). The fp32 queries and probabilities are cut into three bf16 planes by
// truncation (their sum is the fp32 value exactly) and the cache is bf16, so every product is exact and
// only the order of the sums differs from fp32 FMAs. Each wave takes 32-key tiles of the split:
//   * S^T = K Q^T: a lane loads its key's dims 16 s + 8 (l / 32) .. + 8 straight into the A operand;
//     the query planes sit in LDS;
//   * online softmax per query: a max and a sum over the lane's 16 scores and one exchange with lane
//     l ^ 32, which holds the query's other 16;
//   * O^T += V^T P^T: k step s of half h contracts the eight keys whose probabilities the lane already
//     holds (registers 8 s .. 8 s + 7); A row i of dim tile t stands for dim i * DH/32 + t, so a lane
//     reads the DH/32 values of all tiles of a key as one run of its V row (a wave-private LDS tile)
//     and transposes 8 keys x DH/32 dims in registers.
// The four waves' (m, l, o) combine in wave order; a row with one split writes its output, otherwise its
// split record, which attn_merge_row of the launch that follows merges in split order. (With tickets, the
// workgroup that finished last merged every row of the block one after the other, about 4.6 us each:
// four rows at 2051 keys took 28.9 us in that form.)
// Why matrix cores even for one row: a tile costs 48 MFMAs of 32 cycles whatever the number of columns,
// 0.6 us for 32 keys, where the vector form spends about 2 us of dependent work on 16 keys of a wave;
// and rows that share a cache read it once. Rows of a launch whose number of queries passes 32 take
// several workgroups.
typedef float mfma_acc16 __attribute__((ext_vector_type(16)));
typedef __bf16 mfma_bf8 __attribute__((ext_vector_type(8)));

// LDS bytes for M queries: query planes and V tiles, reused for the waves' o, then (m, l).
template <int DH>
constexpr size_t attn_mfma_lds(int M) {
  const size_t qp = (size_t)3 * M * DH * 2, vt = (size_t)(kWG / 64) * 32 * (DH * 2 + 16);
  const size_t o = (size_t)(kWG / 64) * M * DH * 4;
  return (qp + vt > o ? qp + vt : o) + (size_t)(kWG / 64) * 64 * 4;
}

// Rows at consecutive positions (a row block).
struct LimPos {
  int pos0;
  __device__ __forceinline__ int operator()(int r) const { return pos0 + r; }
};

// The page of the first key a lane reads of its wave's first tile.
__device__ __forceinline__ int attn_mfma_page0(const Ctx& C, int split) {
  const int key = split * C.chunk + (int)(threadIdx.x >> 6) * 32 + (int)(threadIdx.x & 31);
  return C.page_table[min(key / C.page, C.max_pages - 1)];
}

// Query q (one head, fp32) over the keys [k0, k1) of KV head g in plain fp32, by the whole workgroup: what a
// query, key or value that is not finite needs. There a plane's 0 * inf, or a value past a shorter row's last
// key, makes the matrix form NaN where the products themselves are not. M, L and a (dims 4 d4 .. + 3 of thread
// d4 = tid % (DH / 4)) are the split's maximum, sum and output; true in the threads that hold them. A score
// that is NaN or +inf makes every dim NaN, which the first pass finds: the values are then not read.
// The scores are computed twice rather than kept, 256 keys at a time: time grows with the keys, 128 FMAs for
// each 256 of them and pass, and memory does not. lds: kWG * 6 floats.
template <int DH>
__device__ __forceinline__ bool attn_query_plain(const uint16_t* kvb, const int* page_table, int hkv, int g,
                                                 const float* q, float scale, int k0, int k1, float* lds, float& M,
                                                 float& L, float (&a)[4]) {
  constexpr int PAGE = 16, TPQ = DH / 4, NG = kWG / TPQ;  // threads per key's value row, keys at once
  const int tid = threadIdx.x, d4 = tid % TPQ, grp = tid / TPQ;
  float* sp = lds;        // [kWG] probabilities
  float* sr = lds + kWG;  // [NG][TPQ][5] sums of the key groups
  auto row = [&](int key) {
    return kvb + ((size_t)page_table[key / PAGE] * 2 * hkv + g) * PAGE * DH + (key % PAGE) * DH;
  };
  auto score = [&](int key) {
    const uint4* k = reinterpret_cast<const uint4*>(row(key));
    float s = 0.f;
#pragma unroll 4
    for (int c = 0; c < DH / 8; c++) {
      float f[8];
      unpack16<uint16_t>(k[c], f);
#pragma unroll
      for (int e = 0; e < 8; e++) s = fmaf(q[c * 8 + e] * scale, f[e], s);
    }
    return s;
  };
  float m = -INFINITY;
  bool sound = true;
  for (int key = k0 + tid; key < k1; key += kWG) {
    const float s = score(key);
    m = fmaxf(m, s);
    sound = sound && s < INFINITY;
  }
#pragma unroll
  for (int i = 1; i < 64; i <<= 1) m = fmaxf(m, __shfl_xor(m, i, 64));
  const bool wave_sound = __all(sound);
  __syncthreads();  // the area's earlier readers are done
  if ((tid & 63) == 0) {
    sp[tid >> 6] = m;
    sp[4 + (tid >> 6)] = wave_sound ? 0.f : 1.f;
  }
  __syncthreads();
  M = fmaxf(fmaxf(sp[0], sp[1]), fmaxf(sp[2], sp[3]));
  const bool all_sound = sp[4] + sp[5] + sp[6] + sp[7] == 0.f;
  __syncthreads();
  if (!all_sound) {  // the same in every thread
    L = a[0] = a[1] = a[2] = a[3] = NAN;
    return grp == 0;
  }
  L = a[0] = a[1] = a[2] = a[3] = 0.f;
  for (int base = k0; base < k1; base += kWG) {
    float p = 0.f;
    if (base + tid < k1) {
      const float s = score(base + tid);
      p = s == -INFINITY ? 0.f : expf(s - M);
    }
    sp[tid] = p;
    __syncthreads();
    const int n = min(kWG, k1 - base);
    for (int i = grp; i < n; i += NG) {
      const uint2 v = *reinterpret_cast<const uint2*>(row(base + i) + (size_t)hkv * PAGE * DH + 4 * d4);
      const float pk = sp[i];
      L += pk;
      a[0] = fmaf(pk, bf_lo(v.x), a[0]);
      a[1] = fmaf(pk, bf_hi(v.x), a[1]);
      a[2] = fmaf(pk, bf_lo(v.y), a[2]);
      a[3] = fmaf(pk, bf_hi(v.y), a[3]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; i++) sr[tid * 5 + i] = a[i];
  sr[tid * 5 + 4] = L;
  __syncthreads();
  if (grp != 0) return false;
#pragma unroll 1
  for (int i = 1; i < NG; i++) {
    const float* o = sr + (i * TPQ + d4) * 5;
#pragma unroll
    for (int k = 0; k < 4; k++) a[k] += o[k];
    L += o[4];
  }
  return true;
}

// kvb: the layer's bf16 cache; q, out: query and output rows (row r at r * qdim, head g's G heads
// contiguous); part: the split records of (row r, KV head g) at index r * hkv + g;
// page0: attn_mfma_page0, requested by the caller; kend: the longest row's keys, [0, kend).
template <int DH, typename Out, typename Lim>
__device__ void attn_split_mfma(const Ctx& C, const uint16_t* kvb, const float* q, const Out out, float* part, int g,
                                int split, int nrows, int kend, const Lim lim, int page0, float* lds) {
  constexpr int NT = DH / 32, KS = DH / 16, KV16 = DH / 16;  // dim tiles, k steps of S, 16-byte loads per half row
  constexpr int MAXQ = kAttnMaxQ, RS = MAXQ * (DH + 2), NWV = kWG / 64, VROW = DH * 2 + 16;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int col = lane & 31, hf = lane >> 5;
  const int G = C.G, lg = __builtin_ctz(G), M = nrows * G;  // G is a power of two
  const int k0 = split * C.chunk, k1 = min(kend, k0 + C.chunk);
  __shared__ uint32_t s_bad;  // queries whose result here is not a number
  if (tid == 0) s_bad = 0u;
  char* const lbase = reinterpret_cast<char*>(lds);
  char* const qpl = lbase;                                                  // [3][M][DH] bf16, chunks permuted
  char* const vt = lbase + (size_t)3 * M * DH * 2 + (size_t)w * 32 * VROW;  // this wave's V tile
  const size_t page_elems = (size_t)2 * C.hkv * C.page * DH;
  const size_t head_off = (size_t)g * C.page * DH;
  const size_t voff = (size_t)C.hkv * C.page * DH;
  const int ntiles = (k1 - k0 + 31) / 32;

  // A lane reads its key of a tile as it comes: a key past the end lies in some page of the table, its
  // score is masked and its V row enters the tile as zeros.
  uint4 kr[KV16], vr[KV16];
  auto page_of = [&](int t) { return C.page_table[min((k0 + t * 32 + col) / C.page, C.max_pages - 1)]; };
  auto issue = [&](int t, int page) {
    const int key = k0 + t * 32 + col;
    const uint16_t* base = kvb + (size_t)page * page_elems + head_off + (size_t)(key % C.page) * DH + hf * 8;
#pragma unroll
    for (int c = 0; c < KV16; c++) kr[c] = ldkv16(base + c * 16);
#pragma unroll
    for (int c = 0; c < KV16; c++) vr[c] = ldkv16(base + voff + c * 16);
  };
  int t = w;
  int pg_next = page_of(t + NWV);
  issue(t, page0);

  // query planes: thread e takes eight dims of a query
  for (int e = tid; e < M * (DH / 8); e += kWG) {
    const int j = e / (DH / 8), c = e % (DH / 8), r = j >> lg, h = j & (G - 1);
    const float* qp = q + (size_t)r * C.qdim + (size_t)(g * G + h) * DH + c * 8;
    const float4 a = *reinterpret_cast<const float4*>(qp), b = *reinterpret_cast<const float4*>(qp + 4);
    const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t pl[3][4];
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const float x = f[k] * C.scale;
      const uint32_t hi = __float_as_uint(x);
      const float r1 = x - __uint_as_float(hi & 0xffff0000u);
      const uint32_t mi = __float_as_uint(r1);
      const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mi & 0xffff0000u));
      if (k & 1) {
        pl[0][k >> 1] |= hi & 0xffff0000u;
        pl[1][k >> 1] |= mi & 0xffff0000u;
        pl[2][k >> 1] |= lo & 0xffff0000u;
      } else {
        pl[0][k >> 1] = hi >> 16;
        pl[1][k >> 1] = mi >> 16;
        pl[2][k >> 1] = lo >> 16;
      }
    }
#pragma unroll
    for (int p = 0; p < 3; p++)
      *reinterpret_cast<uint4*>(qpl + ((size_t)p * M + j) * DH * 2 + ((c ^ (j & 7)) << 4)) =
          make_uint4(pl[p][0], pl[p][1], pl[p][2], pl[p][3]);
  }
  // this lane's query: column col; columns past M repeat the last one, and are not used
  const bool qon = col < M;
  const int qc = min(col, M - 1);
  const int qlim = lim(qc >> lg);
  __syncthreads();  // queries staged

  float m_run = -INFINITY, l_run = 0.f;
  mfma_acc16 o[NT];
#pragma unroll
  for (int tt = 0; tt < NT; tt++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[tt][v] = 0.f;

  for (; t < ntiles; t += NWV) {
    const int kb = k0 + t * 32;  // the tile's first key
    const bool kin = kb + col < k1;
#pragma unroll
    for (int c = 0; c < KV16; c++)  // dims 16 c + 8 hf of key col
      *reinterpret_cast<uint4*>(vt + (size_t)col * VROW + c * 32 + hf * 16) = kin ? vr[c] : make_uint4(0u, 0u, 0u, 0u);
    mfma_acc16 s;
#pragma unroll
    for (int v = 0; v < 16; v++) s[v] = 0.f;
#pragma unroll
    for (int p = 2; p >= 0; p--)  // the small products first
#pragma unroll
      for (int k = 0; k < KS; k++) {
        union { uint4 u; mfma_bf8 f; } ka;
        ka.u = kr[k];
        const mfma_bf8 qf = *reinterpret_cast<const mfma_bf8*>(qpl + ((size_t)p * M + qc) * DH * 2 +
                                                               (((2 * k + hf) ^ (qc & 7)) << 4));
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka.f, qf, s, 0, 0, 0);
      }
    if (t + NWV < ntiles) {  // the registers are free again: the next tile, and the page of the one after
      issue(t + NWV, pg_next);
      pg_next = page_of(t + 2 * NWV);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int key = kb + 8 * (v >> 2) + 4 * hf + (v & 3);
      s[v] = (key < k1 && key <= qlim) ? s[v] : -INFINITY;
      mx = fmaxf(mx, s[v]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m_run, mx);
    if (__any(mn > m_run)) {
      const float al = m_run == -INFINITY ? 0.f : expf(m_run - mn);
      l_run *= al;
#pragma unroll
      for (int tt = 0; tt < NT; tt++)
#pragma unroll
        for (int v = 0; v < 16; v++) o[tt][v] *= al;
      m_run = mn;
    }
    wave_lds_sync();  // the V tile is written
    float ps = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
      union { uint32_t u[4]; mfma_bf8 f; } pf[3];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const float s0 = s[8 * ks + e], s1 = s[8 * ks + e + 1];
        const float p0 = s0 == -INFINITY ? 0.f : expf(s0 - m_run), p1 = s1 == -INFINITY ? 0.f : expf(s1 - m_run);
        ps += p0 + p1;
        const uint32_t h0 = __float_as_uint(p0), h1 = __float_as_uint(p1);
        const float r0 = p0 - __uint_as_float(h0 & 0xffff0000u), r1 = p1 - __uint_as_float(h1 & 0xffff0000u);
        const uint32_t m0 = __float_as_uint(r0), m1 = __float_as_uint(r1);
        const uint32_t l0 = __float_as_uint(r0 - __uint_as_float(m0 & 0xffff0000u));
        const uint32_t l1 = __float_as_uint(r1 - __uint_as_float(m1 & 0xffff0000u));
        pf[0].u[e >> 1] = __builtin_amdgcn_perm(h1, h0, 0x07060302u);
        pf[1].u[e >> 1] = __builtin_amdgcn_perm(m1, m0, 0x07060302u);
        pf[2].u[e >> 1] = __builtin_amdgcn_perm(l1, l0, 0x07060302u);
      }
      uint32_t vw[8][NT / 2];  // the eight keys' NT dims of this lane's row
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const char* vp = vt + (size_t)(16 * ks + 8 * (e >> 2) + 4 * hf + (e & 3)) * VROW + col * NT * 2;
        if constexpr (NT == 4) {
          const uint2 u = *reinterpret_cast<const uint2*>(vp);
          vw[e][0] = u.x;
          vw[e][1] = u.y;
        } else {
          vw[e][0] = *reinterpret_cast<const uint32_t*>(vp);
        }
      }
#pragma unroll
      for (int tt = 0; tt < NT; tt++) {
        union { uint32_t u[4]; mfma_bf8 f; } va;
        const uint32_t sel = (tt & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
        for (int e = 0; e < 4; e++) va.u[e] = __builtin_amdgcn_perm(vw[2 * e + 1][tt >> 1], vw[2 * e][tt >> 1], sel);
#pragma unroll
        for (int p = 2; p >= 0; p--) o[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va.f, pf[p].f, o[tt], 0, 0, 0);
      }
    }
    l_run += ps + __shfl_xor(ps, 32, 64);
    wave_lds_sync();  // the tile is rewritten next step
  }
  __syncthreads();  // every wave is done with the planes and its V tile: the area holds the waves' o now

  float* ow = reinterpret_cast<float*>(lbase) + (size_t)w * M * DH;  // o[query][dim]
  const size_t main_bytes = attn_mfma_lds<DH>(M) - (size_t)NWV * 64 * 4;
  float* mlw = reinterpret_cast<float*>(lbase + main_bytes) + (size_t)w * 64;
  if (hf == 0) {
    mlw[col] = m_run;
    mlw[32 + col] = l_run;
  }
  if (qon) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int i = 8 * (v >> 2) + 4 * hf + (v & 3);
      if constexpr (NT == 4) {
        *reinterpret_cast<float4*>(ow + (size_t)col * DH + i * 4) = make_float4(o[0][v], o[1][v], o[2][v], o[3][v]);
      } else {
        *reinterpret_cast<float2*>(ow + (size_t)col * DH + i * 2) = make_float2(o[0][v], o[1][v]);
      }
    }
  }
  __syncthreads();

  // Combine the waves in wave order per (query, four dims); write a one-split row's output, else the row's
  // split record. A query of a row that has keys in this split has a valid key in wave 0's first tile (key
  // k0), so its maximum is finite. Lane l works out the waves' factors of query l % 32 once and hands them
  // over by shuffles: 32 queries of 128 dims with the factors per (query, dim pair), and divisions by G and
  // the chunk, took 14.9 us per launch at 8 rows of 200 keys.
  const float* mlb = reinterpret_cast<const float*>(lbase + main_bytes);
  float fw[NWV], Mq = -INFINITY, Lq = 0.f;
#pragma unroll
  for (int wv = 0; wv < NWV; wv++) Mq = fmaxf(Mq, mlb[wv * 64 + col]);
#pragma unroll
  for (int wv = 0; wv < NWV; wv++) {
    const float lw = mlb[wv * 64 + 32 + col];
    fw[wv] = lw != 0.f ? expf(mlb[wv * 64 + col] - Mq) : 0.f;  // 0: the wave had no key of this row
    Lq = fmaf(lw, fw[wv], Lq);
  }
  constexpr int TPQ = DH / 4, QPI = kWG / TPQ;  // threads per query, queries at once
  const int d4 = tid % TPQ;
  auto put = [&](int r, int h, const float (&a)[4], float Mr, float Lr) {
    if (lim(r) < C.chunk) {  // one split
      const float inv = 1.0f / Lr;
      const size_t at = (size_t)r * C.qdim + (size_t)(g * G + h) * DH + 4 * d4;
      out(at, a[0] * inv, a[1] * inv);
      out(at + 2, a[2] * inv, a[3] * inv);
    } else {
      float* rec = part + ((size_t)(r * C.hkv + g) * C.max_splits + split) * RS;
      *reinterpret_cast<float4*>(rec + h * DH + 4 * d4) = make_float4(a[0], a[1], a[2], a[3]);
      if (d4 == 0) {
        rec[MAXQ * DH + h] = Mr;
        rec[MAXQ * DH + MAXQ + h] = Lr;
      }
    }
  };
  for (int jb = 0; jb < M; jb += QPI) {
    const int j = jb + tid / TPQ, r = j >> lg, h = j & (G - 1);
    float f[NWV];
#pragma unroll
    for (int wv = 0; wv < NWV; wv++) f[wv] = __shfl(fw[wv], j & 31, 64);
    const float Mx = __shfl(Mq, j & 31, 64), L = __shfl(Lq, j & 31, 64);
    if (j >= M || k0 > lim(r)) continue;  // no key of this split for the row
    float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < NWV; wv++) {
      const float4 ov =
          *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(lbase) + ((size_t)wv * M + j) * DH + 4 * d4);
      a[0] = fmaf(ov.x, f[wv], a[0]);
      a[1] = fmaf(ov.y, f[wv], a[1]);
      a[2] = fmaf(ov.z, f[wv], a[2]);
      a[3] = fmaf(ov.w, f[wv], a[3]);
    }
    if (L != L || a[0] != a[0] || a[1] != a[1] || a[2] != a[2] || a[3] != a[3])
      atomicOr(&s_bad, 1u << j);
    else
      put(r, h, a, Mx, L);
  }
  __syncthreads();
  // Queries with a NaN, one after the other in plain fp32.
  for (uint32_t bad = __builtin_amdgcn_readfirstlane(s_bad); bad != 0u; bad &= bad - 1u) {
    const int j = __builtin_ctz(bad), r = j >> lg, h = j & (G - 1);
    float a[4], Mr, Lr;
    if (attn_query_plain<DH>(kvb, C.page_table, C.hkv, g, q + (size_t)r * C.qdim + (size_t)(g * G + h) * DH, C.scale, k0,
                             min(k1, lim(r) + 1), lds, Mr, Lr, a))
      put(r, h, a, Mr, Lr);
  }
}

// Row r's KV head g of a split launch: merges its split records (nothing to do if it has one split).
template <int DH, typename Out>
__device__ __forceinline__ void attn_merge_row(const Ctx& C, const float* part, const Out out, int r, int g, int len,
                                               float* sm) {
  const int nsplit = (len + C.chunk - 1) / C.chunk;
  if (nsplit > 1)
    attn_merge<DH, false>(part + (size_t)(r * C.hkv + g) * C.max_splits * kAttnMaxQ * (DH + 2), nsplit, C.G,
                          ShiftedOut<Out>{out, (size_t)r * C.qdim + (size_t)g * C.G * DH}, sm);
}

// One split. kvb: the layer's
// cache; q: the G rotated query rows of this head group; out: their G output rows; rec_base: the
// (o[8][DH], m[8], l[8]) records of this (stage, head), one per split; cnt: its split ticket (zero at
// rest); page0: the physical page of this thread's key in the first round (key k0 + threadIdx.x / 4,
// clamped; requested by the caller before anything else). Returns true when this workgroup wrote the
// final output.
template <typename KVT, int DH>
__device__ bool attn_split(const Ctx& C, const KVT* kvb, const float* q, float* out, float* rec_base, int* cnt, int g,
                           int split, int nsplit, int k0, int k1, int pos0, int page0, float* lds) {
  if (C.G <= 4)
    return attn_split_g<KVT, DH, 4>(C, kvb, q, out, rec_base, cnt, g, split, nsplit, k0, k1, pos0, page0, lds);
  return attn_split_g<KVT, DH, 8>(C, kvb, q, out, rec_base, cnt, g, split, nsplit, k0, k1, pos0, page0, lds);
}

}  // namespace spd
