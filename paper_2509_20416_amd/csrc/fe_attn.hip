// fe_attn.hip -- GQA decode attention of a cascade layer over its prefix KV
// cache plus the cascade entries, in one launch (gfx950).
//
// Layer i's query (one row per sequence, H_q heads) attends to the P_b cached
// prefix keys of its own cache and to the nctx keys it projected from the
// cascade states (Section 2.1; the cache is per layer because every L_i has
// its own parameters).
//
//  * fp32 caches (k_attn): one workgroup (4 waves) per (sequence, KV head,
//    head group, span of chunks of kAttnChunk prefix keys), heads fastest in
//    the grid; the GH query heads sharing a KV head are done together so every
//    K/V byte is read once.  A key row is split in 16-byte pieces over
//    RL = D*sizeof(T)/16 lanes, so one load instruction covers 64/RL whole
//    rows; K and V are loaded together.  A score is reduced over its RL lanes
//    with DPP row operations and leaves every lane of the row with the same
//    value, which is exactly what the value pass needs: each lane accumulates
//    p*V for its own dims and key rows, so the value sums need no cross-lane
//    traffic.  Row-group maxima use gfx950's permlane swaps.  The
//    per-(wave, row group) sums meet in LDS.  Chunk 0 also takes the nctx
//    cascade keys (fp32, one extra load per lane).
//  * bf16 caches (k_attn_mma): one-wave workgroups on the matrix cores with a
//    direct-to-LDS ring; see the comment above that kernel.
//  * A span that is not the whole sequence leaves o[D] (scaled to its max)
//    and (max, sum) per head in the workspace, and a second launch
//    (k_attn_merge) combines them in a fixed order: no atomics, no fences, the
//    result does not depend on scheduling.  A sequence with an empty prefix
//    still runs chunk 0 for its cascade keys.
#include "fe_attn_unit.h"
#include <algorithm>

namespace fe {

constexpr int kWaveKeys = kAttnChunk / 4;   // keys per wave

__device__ __forceinline__ float scaled_exp(float m, float M) {
  return m == -INFINITY ? 0.f : expf(m - M);
}

// element e of a 16-byte piece holding 16/sizeof(T) values
template <typename T> __device__ __forceinline__ float piece_at(const u32x4 &w, int e) {
  const uint32_t u = (e >> (sizeof(T) == 2 ? 1 : 0)) == 0   ? w.x
                     : (e >> (sizeof(T) == 2 ? 1 : 0)) == 1 ? w.y
                     : (e >> (sizeof(T) == 2 ? 1 : 0)) == 2 ? w.z
                                                            : w.w;
  if constexpr (sizeof(T) == 2) return (e & 1) ? __uint_as_float(u & 0xffff0000u) : __uint_as_float(u << 16);
  else return __uint_as_float(u);
}

template <typename T, int D, int GH>
__global__ __launch_bounds__(256) void k_attn(const T *__restrict__ Kc, const T *__restrict__ Vc,
                                              Seqs cu,
                                              const float *__restrict__ q,
                                              const float *__restrict__ knew,
                                              const float *__restrict__ vnew, int nctx,
                                              float *__restrict__ part, int nch, int nch_ld,
                                              int cpw,
                                              T *__restrict__ out, int Hq, int Hkv, int pmax) {
  constexpr int RL = D * (int)sizeof(T) / 16;  // lanes per key row
  constexpr int KPL = 64 / RL;                  // key rows per load instruction
  constexpr int DPL = 16 / (int)sizeof(T);      // dims per lane
  constexpr int NLD = kWaveKeys / KPL;          // K (and V) loads per lane per sub-chunk
  constexpr int CW = DPL / 4;                   // fp32 16-byte pieces per lane of a cascade row
  constexpr int NCX = (kMaxLayers + 4 * KPL - 1) / (4 * KPL);  // cascade rows per lane (chunk 0)
  __shared__ float s_o[4][KPL][GH][D];
  __shared__ float s_l[4][KPL][GH];
  __shared__ float s_m[4][GH];

  const int G = Hq / Hkv, ngrp = G / GH;
  // heads fastest: the workgroups that run side by side read neighbouring
  // head segments of the same token rows
  const int ch = blockIdx.y, c = blockIdx.x / ngrp, hg = blockIdx.x % ngrp, b = blockIdx.z;
  bool bad;
  const int start = cu.start(b), P = attn_prefix(cu, b, pmax, bad);
  const int span = kAttnChunk * cpw;  // prefix keys per workgroup
  const int nv = max(1, min((P + span - 1) / span, nch));
  if (ch >= nv) return;  // chunk beyond this sequence's prefix
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kg = lane / RL, dl = lane % RL;
  const int h0 = c * G + hg * GH;
  const float scale = rsqrtf((float)D);
  const int base = ch * span;
  // sub-chunks of kAttnChunk keys this workgroup visits (0 for an empty prefix)
  const int nsc = P > 0 ? min(cpw, (P - base + kAttnChunk - 1) / kAttnChunk) : 0;
  const int lkey = wave * kWaveKeys + kg;  // this lane's first key within a sub-chunk; step KPL
  const bool casc = ch == 0;
  float *part_o = part;
  float *part_ml = part + (size_t)gridDim.z * Hq * nch_ld * D;

  const size_t rs = (size_t)Hkv * D;
  const T *kb = Kc + ((size_t)start * Hkv + c) * D + dl * DPL;
  const T *vb = Vc + ((size_t)start * Hkv + c) * D + dl * DPL;
  // rows of sub-chunk `sc` at clamped in-bounds keys (masked when scored)
  auto load_rows = [&](int sc, u32x4 (&kr)[NLD], u32x4 (&vr)[NLD]) {
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      const size_t key = (size_t)min(base + sc * kAttnChunk + lkey + t * KPL, P - 1);
      kr[t] = *reinterpret_cast<const u32x4 *>(kb + key * rs);
      vr[t] = *reinterpret_cast<const u32x4 *>(vb + key * rs);
    }
  };
  u32x4 kr[NLD], vr[NLD];
  if (nsc > 0) load_rows(0, kr, vr);
  float qv[GH][DPL];
#pragma unroll
  for (int gh = 0; gh < GH; ++gh) {
    const f32x4 *qp = reinterpret_cast<const f32x4 *>(q + ((size_t)b * Hq + h0 + gh) * D + dl * DPL);
#pragma unroll
    for (int w = 0; w < DPL / 4; ++w) {
      const f32x4 v = qp[w];
      qv[gh][4 * w + 0] = v.x;
      qv[gh][4 * w + 1] = v.y;
      qv[gh][4 * w + 2] = v.z;
      qv[gh][4 * w + 3] = v.w;
    }
  }

  // running softmax state of this lane's row group, per head: m (uniform over
  // the wave), l and o (the group's own keys)
  float m[GH], l[GH], o[GH][DPL];
#pragma unroll
  for (int gh = 0; gh < GH; ++gh) {
    m[gh] = -INFINITY;
    l[gh] = 0.f;
#pragma unroll
    for (int e = 0; e < DPL; ++e) o[gh][e] = 0.f;
  }
  // online update with NS scored keys: s[t][gh] (masked -inf), value dims val(t, e)
  auto absorb = [&](auto &s, auto val) {
    constexpr int NS = sizeof(s) / sizeof(s[0]);
#pragma unroll
    for (int gh = 0; gh < GH; ++gh) {
      float mx = m[gh];
#pragma unroll
      for (int t = 0; t < NS; ++t) mx = fmaxf(mx, s[t][gh]);
      mx = across_groups_max<RL>(mx);
      const float alpha = scaled_exp(m[gh], mx);
      m[gh] = mx;
      float sum = l[gh] * alpha;
#pragma unroll
      for (int e = 0; e < DPL; ++e) o[gh][e] *= alpha;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        s[t][gh] = scaled_exp(s[t][gh], mx);
        sum += s[t][gh];
      }
      l[gh] = sum;
    }
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
      for (int e = 0; e < DPL; ++e) {
        const float ve = val(t, e);
#pragma unroll
        for (int gh = 0; gh < GH; ++gh) o[gh][e] += s[t][gh] * ve;  // weight 0 when masked
      }
  };

  // ---- chunk 0: the cascade keys (fp32) --------------------------------------
  if (casc) {
    f32x4 kx[NCX][CW], vx[NCX][CW];
#pragma unroll
    for (int t = 0; t < NCX; ++t) {
      const int j = min((t * 4 + wave) * KPL + kg, nctx - 1);
      const size_t off = (((size_t)b * nctx + j) * Hkv + c) * D + dl * DPL;
#pragma unroll
      for (int w = 0; w < CW; ++w) {
        kx[t][w] = reinterpret_cast<const f32x4 *>(knew + off)[w];
        vx[t][w] = reinterpret_cast<const f32x4 *>(vnew + off)[w];
      }
    }
    float sx[NCX][GH];
#pragma unroll
    for (int t = 0; t < NCX; ++t)
#pragma unroll
      for (int gh = 0; gh < GH; ++gh) {
        float acc = 0.f;
#pragma unroll
        for (int w = 0; w < CW; ++w)
          acc += qv[gh][4 * w] * kx[t][w].x + qv[gh][4 * w + 1] * kx[t][w].y +
                 qv[gh][4 * w + 2] * kx[t][w].z + qv[gh][4 * w + 3] * kx[t][w].w;
        acc = group_sum<RL>(acc);
        sx[t][gh] = (t * 4 + wave) * KPL + kg < nctx ? acc * scale : -INFINITY;
      }
    absorb(sx, [&](int t, int e) {
      const f32x4 &v = vx[t][e >> 2];
      return (e & 3) == 0 ? v.x : (e & 3) == 1 ? v.y : (e & 3) == 2 ? v.z : v.w;
    });
  }

  // ---- prefix keys, sub-chunk by sub-chunk (next rows in flight) -------------
  // The prefetch is unconditional (the last one re-reads clamped in-bounds
  // rows): under a branch the compiler would wait for it before the compute.
  for (int sc = 0; sc < nsc; ++sc) {
    u32x4 kn[NLD], vn[NLD];
    load_rows(sc + 1, kn, vn);
    const int key0 = base + sc * kAttnChunk + lkey;
    float s[NLD][GH];
#pragma unroll
    for (int t = 0; t < NLD; ++t)
#pragma unroll
      for (int gh = 0; gh < GH; ++gh) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < DPL; ++e) acc += qv[gh][e] * piece_at<T>(kr[t], e);
        acc = group_sum<RL>(acc);
        s[t][gh] = key0 + t * KPL < P ? acc * scale : -INFINITY;
      }
    absorb(s, [&](int t, int e) { return piece_at<T>(vr[t], e); });
#pragma unroll
    for (int t = 0; t < NLD; ++t) {
      kr[t] = kn[t];
      vr[t] = vn[t];
    }
  }

#pragma unroll
  for (int gh = 0; gh < GH; ++gh) {
#pragma unroll
    for (int w = 0; w < DPL / 4; ++w)
      *reinterpret_cast<f32x4 *>(&s_o[wave][kg][gh][dl * DPL + 4 * w]) =
          f32x4{o[gh][4 * w], o[gh][4 * w + 1], o[gh][4 * w + 2], o[gh][4 * w + 3]};
    if (dl == 0) s_l[wave][kg][gh] = l[gh];
    if (lane == 0) s_m[wave][gh] = m[gh];
  }
  __syncthreads();

  // ---- this workgroup's result: the output row when it holds the whole
  //      sequence, else its partial (o scaled to its max, (max, sum))
  const bool whole = nv == 1;
  for (int idx = tid; idx < GH * D; idx += 256) {
    const int gh = idx / D, e = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_m[w][gh]);
    float acc = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      float g = 0.f, gl = 0.f;
#pragma unroll
      for (int k = 0; k < KPL; ++k) {
        g += s_o[w][k][gh][e];
        gl += s_l[w][k][gh];
      }
      const float sw = scaled_exp(s_m[w][gh], M);
      acc += sw * g;
      L += sw * gl;
    }
    if (bad) {  // P_b outside [0, pmax]: the sequence's output is NaN
      acc = __int_as_float(0x7fc00000);
      L = whole ? 1.f : acc;
      M = 0.f;
    }
    if (whole) {
      out[(size_t)b * Hq * D + (size_t)(h0 + gh) * D + e] = Elt<T>::from_f(acc / L);
    } else {
      part_o[(((size_t)b * Hq + h0 + gh) * nch_ld + ch) * D + e] = acc;
      if (e == 0) {
        float *ml = part_ml + (((size_t)b * Hq + h0 + gh) * nch_ld + ch) * 2;
        ml[0] = M;
        ml[1] = L;
      }
    }
  }
}


// ---- bf16 caches: both contractions on the matrix cores -------------------------
//
// One wave per workgroup, so up to four run on a CU side by side and the set-up
// and write-out of one overlap the streaming of the others; each covers a span
// of prefix keys of one (sequence, KV head, head group).  K and V rows reach
// LDS by direct-to-LDS loads through a per-wave ring of DEPTH stages of 16 keys
// (DEPTH-1 stages in flight), with an XOR swizzle of the 16-byte pieces that
// keeps both operand gathers free of bank conflicts.
// Per stage, QK^T runs with the keys as MFMA rows (A = 16-byte pieces of K
// rows) and the GH query heads as columns (B = q, zero-padded to 16 heads).  q
// is split into a bf16 high part and a bf16 remainder, two MFMAs each, which
// keeps the scores at fp32-level accuracy against the bf16 keys.  q is
// pre-scaled by log2(e)/sqrt(D), so scores are in log2 units and every
// exponential is one v_exp_f32.  The result leaves each lane with 4 scores of
// one head, which is exactly the B operand of the 16-key value product
// O^T = V^T P^T, so the probabilities never move between lanes; V^T is
// gathered from the ring with 16-bit reads.  The probabilities enter the
// product as bf16 and the running sum adds the same rounded values, so the
// output is an exact weighted mean of V.  The running maximum is raised only
// when a score exceeds it by more than kLazyMax (probabilities stay below
// 2^kLazyMax), so the accumulators are rescaled on few stages.
// The nctx cascade keys (fp32) are done on the vector ALU by chunk 0 and merged
// into its result at the end.



template <int D, int GH, int DEPTH, int NCX>
__global__ __launch_bounds__(64) void k_attn_mma(const bf16_t *__restrict__ Kc,
                                                 const bf16_t *__restrict__ Vc,
                                                 Seqs cu,
                                                 const float *__restrict__ q,
                                                 const float *__restrict__ knew,
                                                 const float *__restrict__ vnew, int nctx,
                                                 float *__restrict__ part, int nch, int nch_ld,
                                                 int cpw, bf16_t *__restrict__ out, int Hq,
                                                 int Hkv, const float *__restrict__ rope,
                                                 int cascade, int nseq, int persist,
                                                 int csplit, int pmax) {
  __shared__ AttnLds<D, GH, DEPTH> lds;
  const int G = Hq / Hkv, ngrp = G / GH, ncols = Hkv * ngrp;
  const int lane = threadIdx.x;
  const int span = kAttnChunk * cpw;
  float *part_o = part;
  float *part_ml = part + (size_t)nseq * Hq * nch_ld * D;

  // One piece of work: prefix chunks [ch0, ch0 + nchunk) (kAttnChunk keys
  // each) of sequence b for the query heads of column col (KV head c, head
  // group hg), plus the (at most NCX) cascade keys when casc.  The result goes
  // to the output when `whole`, else to partial slot `slot`; npieces > 0
  // (given to the first piece of a segment) is stored as the segment's
  // partial count.
  auto unit = [&](const int b, const int col, const int ch0, const int nchunk, const int slot,
                  const bool whole, const int npieces, const bool casc) {
    const int c = col / ngrp, hg = col % ngrp;
    const int h0 = c * G + hg * GH;
    bool bad;
    const int start = cu.start(b), P = attn_prefix(cu, b, pmax, bad);
    const size_t row0 = (size_t)b * Hq + h0;
    attn_unit<D, GH, DEPTH, NCX>(
        Kc + ((size_t)start * Hkv + c) * D, Vc + ((size_t)start * Hkv + c) * D, (size_t)Hkv * D,
        P, bad, q + row0 * D, knew + ((size_t)b * nctx * Hkv + c) * D,
        vnew + ((size_t)b * nctx * Hkv + c) * D, (size_t)Hkv * D, nctx, rope, cascade, ch0, nchunk,
        whole, casc, part_o + (row0 * nch_ld + slot) * D, nch_ld * D,
        part_ml + (row0 * nch_ld + slot) * 2, nch_ld * 2, out + row0 * D,
        part_ml + (size_t)nseq * Hq * nch_ld * 2 + row0, npieces, lds);
  };


  if (!persist) {
    // one workgroup per span of cpw chunks: grid (columns, spans, sequences),
    // heads fastest so the workgroups that run side by side read neighbouring
    // head segments of the same token rows; partial slot = span index
    const int b = blockIdx.z, col = blockIdx.x, ch = blockIdx.y;
    bool bad;
    const int P = attn_prefix(cu, b, pmax, bad);
    const int nv = max(1, min((P + span - 1) / span, nch));
    if (csplit) {
      // the cascade keys as a unit of their own (grid y = nch), off the
      // prefix units' critical path; every sequence leaves nv + 1 partials,
      // the cascade's last
      if (ch == nch) unit(b, col, 0, 0, nv, false, 0, true);
      else if (ch < nv) unit(b, col, ch * cpw, cpw, ch, false, 0, false);
      return;
    }
    if (ch < nv) unit(b, col, ch * cpw, cpw, ch, nv == 1, 0, ch == 0);
    return;
  }
  // Persistent: a grid of resident waves, each taking one range of the
  // equal-chunk split (AttnSplit; W = the grid, or the chunk count if
  // smaller), so the waves finish together however ragged the sequences are.
  // Up to 256 sequences (4 per lane).
  int ucnt[4], uend[4];  // chunks of sequence lane + 64 i (all columns), running total
  int run = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = lane + 64 * i;
    int n = 0;
    if (b < nseq) {
      bool bad;
      n = attn_seg_chunks(attn_prefix(cu, b, pmax, bad), nch_ld) * ncols;
    }
    // inclusive scan over the wave, then add the totals of earlier blocks
    int x = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    ucnt[i] = n;
    uend[i] = run + x;
    run += __shfl(x, 63, 64);
  }
  const AttnSplit eq{run, min((long)gridDim.x, (long)run)};
  if ((long)blockIdx.x >= eq.W) return;
  int x = eq.begin(blockIdx.x);
  const int xe = eq.begin(blockIdx.x + 1);
  while (x < xe) {
    // sequence b: the number of sequences whose chunks all come before x
    int b = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) b += __popcll(__ballot(uend[i] <= x));
    int first = 0, cnt = 0;  // chunks before sequence b, and its own
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = __shfl(uend[i], b & 63, 64), n = __shfl(ucnt[i], b & 63, 64);
      if ((b >> 6) == i) {
        first = e - n;
        cnt = n;
      }
    }
    int col, ch0, n, slot, np;
    eq.piece(x, xe, first, cnt, ncols, col, ch0, n, slot, np);
    // items [ch0, ch0 + n) of the segment: prefix chunks below its last item,
    // which stands for the cascade keys
    const int items = cnt / ncols, pre = min(ch0 + n, items - 1) - ch0;
    unit(b, col, ch0, pre > 0 ? pre : 0, slot, false, np, ch0 + n == items);
    x += n;
  }
}


// ---- chunk merge (second launch) -------------------------------------------------
// A sequence whose prefix spans several workgroups leaves one partial per
// workgroup: o (scaled to that workgroup's max), max and sum per head.  This
// launch combines them in chunk order, 32 per round trip.  Sequences that fit
// one workgroup wrote their rows directly and are skipped.  Keeping the merge in
// its own launch means no workgroup ever waits on another: the kernel boundary
// publishes the partials once, where per-workgroup device-scope fences would
// write back the L2 once per workgroup.  LOG2: maxima in log2 units.
template <typename T, bool LOG2>
__global__ __launch_bounds__(256) void k_attn_merge(const float *__restrict__ part, int nch_ld,
                                                    Seqs cu, int span,
                                                    int nwg, T *__restrict__ out, int Hq, int D,
                                                    int counted, int csplit, int pmax) {
  const int b = blockIdx.y;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= Hq * D / 2) return;
  const int h = (2 * idx) / D, e = (2 * idx) % D;
  // partials of (b, h): one per span (sequences within one span wrote their
  // rows directly) and, with csplit, the cascade keys' one after them, or as
  // counted by the persistent attention
  int nv;
  if (counted) {
    nv = (int)part[(size_t)gridDim.y * Hq * nch_ld * (D + 2) + (size_t)b * Hq + h];
  } else {
    bool bad;
    const int P = attn_prefix(cu, b, pmax, bad);
    nv = max(1, min((P + span - 1) / span, nwg)) + csplit;
    if (nv == 1) return;
  }
  const float *po = part + ((size_t)b * Hq + h) * nch_ld * D + e;
  const float *pml = part + (size_t)gridDim.y * Hq * nch_ld * D + ((size_t)b * Hq + h) * nch_ld * 2;
  auto ex = [](float m, float M) {
    return m == -INFINITY ? 0.f : (LOG2 ? __builtin_amdgcn_exp2f(m - M) : expf(m - M));
  };
  float M = -INFINITY, L = 0.f, ax = 0.f, ay = 0.f;
  constexpr int R = 32;  // partials per round trip
  for (int c0 = 0; c0 < nv; c0 += R) {
    float2 ov[R], ml[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int k = min(c0 + u, nv - 1);
      ov[u] = *reinterpret_cast<const float2 *>(po + (size_t)k * D);
      ml[u] = *reinterpret_cast<const float2 *>(pml + 2 * k);
    }
    float Mn = M;
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (c0 + u < nv) Mn = fmaxf(Mn, ml[u].x);
    const float rr = ex(M, Mn);
    L *= rr;
    ax *= rr;
    ay *= rr;
#pragma unroll
    for (int u = 0; u < R; ++u)
      if (c0 + u < nv) {
        const float w = ex(ml[u].x, Mn);
        L += w * ml[u].y;
        ax += w * ov[u].x;
        ay += w * ov[u].y;
      }
    M = Mn;
  }
  T *op = out + (size_t)b * Hq * D + (size_t)h * D + e;
  op[0] = Elt<T>::from_f(ax / L);
  op[1] = Elt<T>::from_f(ay / L);
}

// ---- tiles of query rows (bf16 multi-position prefill) ---------------------------
// The rows of a prefill share their sequence's cache rows: row m sees
// keys start .. start + P_m - 1.  Done row by row (k_attn_mma) every row
// streams its own prefix through LDS, so a 1024-row prompt reads its keys 512
// times over and each MFMA carries GH live columns of 16.  Here a workgroup
// takes a tile of up to kTileQ / GH consecutive rows with one start and the GH
// heads of a head group, i.e. kTileQ (row, head) columns, streams the union
// of their keys once, and masks each column's scores past its own P.
//
// Four waves of 16 columns, one per SIMD, stages of 32 keys in a four-slot
// ring (64 KB at D = 128: two workgroups per CU, which hide each other's
// latencies).  The arithmetic is k_attn_mma's: q split into a bf16 high and
// low part, lazily raised maxima, probabilities as bf16 whose sum (a product
// with ones) adds the same rounded values; the row's own key (fp32) joins at
// the end, unrotated, since rotating it and the query by the same position
// leaves their product unchanged.
// Bound by the chain read - score - maximum - exponential - product of a
// stage, not by bytes: 1024 rows at the 8B shapes (32 query, 8 KV heads, D 128)
// take 41 us per layer, against 315 us for the row-by-row launches and their
// merges; tiles of 128 columns took 52 us with four waves (two column tiles
// each) and 46 us with eight, because a prompt's last tile sees twice the
// average keys and only two small workgroups per CU even that out.
//
// A workgroup walks a tile's keys by itself, 0.7 us a stage, so a long history
// behind few tiles (few rows or KV heads, or one sequence longer than the rest)
// left most CUs idle behind it.  Such tiles are cut into pieces of keys, a
// workgroup each, whose partial sums k_attn_tile_merge adds.  The plan decides
// on the device, where the histories are known: all tiles stay whole where the
// longest takes at most twice what the launch's stages are per resident
// workgroup (the short tiles then fill its time), or at most kWholeStages.
// Updates of three 1024-wide layers, us a call (row by row / whole tiles / cut):
// 64 rows after 8192 keys, one KV head of 8 query heads 297 / 549 / 209, 8 KV
// heads of 4 696 / 559 / 229; 256 rows of which one sequence has 8192 keys and
// the others 64, 8 KV heads of 4 551 / 654 / 327; 64 rows with no history 253 /
// 180 / 185: the merge's launch finds nothing to do there, 2 to 4 us a layer.
// (The last piece to be done adding the sums saved that launch, but a release
// fence per piece writes back the L2: 292 where the launch gives 229.)
constexpr int kTileQ = 64, kTileWaves = 4, kTileKeys = 32;
constexpr int kPieceStages = 16, kWholeStages = 32;  // shortest piece, longest tile never cut
constexpr int kTilePieces = 64;                      // pieces of one tile, at most
static_assert(kTilePlanSplit * 2 == kTilePlanPieces, "a cut tile has fewer than 2 nst / L pieces");

// Inclusive sum of x over the workgroup's 1024 threads; the last one's in total.
__device__ __forceinline__ int plan_scan(int x, int *s_w, int &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) s_w[wave] = x;
  __syncthreads();
  total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) x += s_w[w];
    total += s_w[w];
  }
  return x;
}

// The plan (TilePlan) of rows that see keys ranges[2m] .. ranges[2m + 1] - 1.  A
// tile is at most tq consecutive rows of one run: rows with the same
// start whose ranges are valid (an invalid row is a tile of its own).  One
// workgroup; per 1024 rows a scan for the run's first row and one for the
// tile's index, and where tiles are cut three per 1024 tiles for the lists.
// `slots`: partial results the scratch has room for (0: no tile is cut).
__global__ __launch_bounds__(1024) void k_attn_tile_plan(const int32_t *__restrict__ ranges, int M,
                                                         int pmax, int tq, int ncols, int slots,
                                                         int wgs, int32_t *__restrict__ plan) {
  __shared__ int s_w[16], s_carry[2], s_max[16], s_stg[1025];
  __shared__ long s_sum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const TilePlan pl{plan, M};
  int32_t *tiles = pl.first(), *stg = pl.stages();
  if (tid == 0) s_carry[0] = s_carry[1] = 0;
  for (int m0 = 0; m0 < M; m0 += 1024) {
    const int m = m0 + tid, mc = min(m, M - 1), mp = max(mc - 1, 0);
    const int start = ranges[2 * mc], P = ranges[2 * mc + 1] - start;
    const int start0 = ranges[2 * mp], P0 = ranges[2 * mp + 1] - start0;
    const bool bad = P < 0 || P > pmax, bad0 = P0 < 0 || P0 > pmax;
    const bool first = m < M && (m == 0 || bad || bad0 || start != start0);
    s_stg[tid + 1] = 0;
    if (tid == 0) s_stg[0] = 0;
    // the run's first row: the largest row <= m that starts one
    int x = first ? m : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x = max(x, y);
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    x = max(x, s_carry[0]);
    for (int w = 0; w < wave; ++w) x = max(x, s_w[w]);
    const bool head = m < M && (m - x) % tq == 0;
    const int before = s_carry[1];  // tiles of the rounds before; the last of them may go on
    int total;
    const int idx = plan_scan(head ? 1 : 0, s_w, total);  // the row's tile is before + idx - 1
    if (head) tiles[before + idx - 1] = m;
    if (m < M && !bad) atomicMax(&s_stg[idx], (P + kTileKeys - 1) / kTileKeys);
    __syncthreads();
    if (tid == 1023) s_carry[0] = x;
    if (tid < total) stg[before + tid] = s_stg[tid + 1];
    if (tid == 0) {
      s_carry[1] = before + total;
      if (before > 0) stg[before - 1] = max(stg[before - 1], s_stg[0]);
    }
    __syncthreads();
  }
  const int nt = s_carry[1];
  if (tid == 0) tiles[nt] = M;
  // the tiles' stages: their sum and the largest
  long sum = 0;
  int most = 0;
  if (slots > 0) {
    for (int t = tid; t < nt; t += 1024) {
      sum += stg[t];
      most = max(most, stg[t]);
    }
    for (int o = 1; o < 64; o <<= 1) {
      sum += __shfl_xor(sum, o, 64);
      most = max(most, __shfl_xor(most, o, 64));
    }
    if (lane == 0) {
      s_sum[wave] = sum;
      s_max[wave] = most;
    }
  }
  __syncthreads();
  if (slots > 0) {
    sum = 0;
    most = 0;
    for (int w = 0; w < 16; ++w) {
      sum += s_sum[w];
      most = max(most, s_max[w]);
    }
    sum *= ncols;
  }
  // stages of a piece: an even share of the work or more, so that fewer than
  // kTilePlanSplit tiles are cut, into at most kTilePlanPieces pieces; at most
  // `slots` of them (a tile that is cut has n > L stages and ceil(n / L) <=
  // 2 n / L pieces)
  const long share = (sum + wgs - 1) / wgs;
  const bool cuts = most > kWholeStages && most > 2 * share;
  int ne = nt, ns = 0;
  if (!cuts) {
    // the last tile first (a prompt's last tiles see the most keys)
    for (int j = tid; j < nt; j += 1024) {
      const int t = nt - 1 - j, row0 = tiles[t];
      pl.pieces()[j] = int4{row0, tiles[t + 1] - row0, 0, stg[t]};
    }
  } else {
    const long room = (2 * sum + slots - 1) / slots;
    long want = share > kPieceStages ? share : kPieceStages;
    want = want > room ? want : room;
    const int fewest = (most + kTilePieces - 1) / kTilePieces;
    const int L = want > most ? most : max((int)want, fewest);
    int nslot = 0;
    ne = 0;
    for (int j0 = 0; j0 < nt; j0 += 1024) {
      const int t = nt - 1 - (j0 + tid);
      const int n = t >= 0 ? stg[t] : 0, np = t < 0 ? 0 : n > L ? (n + L - 1) / L : 1;
      const bool cut = np > 1;
      int te, tsl, ts;
      const int e = ne + plan_scan(np, s_w, te) - np;
      const int sl = nslot + plan_scan(cut ? np : 0, s_w, tsl) - (cut ? np : 0);
      const int si = ns + plan_scan(cut ? 1 : 0, s_w, ts) - (cut ? 1 : 0);
      if (t >= 0) {
        const int row0 = tiles[t], rows = tiles[t + 1] - row0;
        // stages n / np each, one more in the first n % np
        const int each = n / np, more = n % np;
        for (int k = 0; k < np; ++k)
          pl.pieces()[e + k] = int4{row0, rows | (cut ? sl + k + 1 : 0) << 8, k * each + min(k, more),
                                    each + (k < more ? 1 : 0)};
        if (cut) pl.cut()[si] = int4{row0, rows, sl, np};
      }
      ne += te;
      nslot += tsl;
      ns += ts;
    }
  }
  if (tid == 0) {
    plan[0] = ne;
    plan[1] = ns;
  }
}

template <int D, int GH>
__global__ __launch_bounds__(64 * kTileWaves, 2) void k_attn_tile(const bf16_t *__restrict__ Kc,
                                                      const bf16_t *__restrict__ Vc,
                                                      const int32_t *__restrict__ ranges,
                                                      const int32_t *__restrict__ plan, int M,
                                                      const float *__restrict__ q,
                                                      const float *__restrict__ knew,
                                                      const float *__restrict__ vnew,
                                                      bf16_t *__restrict__ out,
                                                      float *__restrict__ parts, int Hq, int Hkv,
                                                      const float *__restrict__ rope, int pmax) {
  constexpr int NKC = D / 32, NDT = D / 16, VPR = D / 8, RB = 2 * D, HD = D / 2;
  constexpr int RPW = 256 / RB, LQ = VPR == 16 ? 3 : 2;
  constexpr int SK = kTileKeys, HALF = SK * RB, STAGE = 2 * HALF, S = 4;
  constexpr int NL = STAGE / 1024 / kTileWaves;  // 1 KB loads per wave per stage
  constexpr int CT = kTileQ / 16 / kTileWaves;   // 16-column tiles per wave
  static_assert((S - 1) * NL <= 63, "outstanding loads stay within the vmcnt range");
  __shared__ __attribute__((aligned(16))) unsigned char ring[S][STAGE];
  __shared__ int s_p[kTileWaves];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int G = Hq / Hkv, ngrp = G / GH, ncols = Hkv * ngrp;
  const size_t rs = (size_t)Hkv * D;
  const float qscale = 1.4426950408889634f * rsqrtf((float)D);
  // 16-byte piece p of row R sits at p ^ swzk(R) (K) or p ^ swz(R) (V, as in
  // attn_unit), rows mod 16.  A 16-byte read is served to lanes 0-3, 12-15 and
  // 20-27 together, then 4-11, 16-19 and 28-31, and so on: under swzk those
  // sixteen (row, piece) pairs of a K operand lie in distinct banks, under swz
  // they met in pairs.
  auto swz = [](int R) {
    const int Q = (R & 15) / RPW;
    return (2 * Q + (Q >> LQ)) & (VPR - 1);
  };
  auto swzk = [](int R) { return (R / RPW) & (VPR - 1); };
  // this lane's row and element offset in each of its loads (a stage's K rows,
  // then its V rows)
  int lrow[NL], loff[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int o = (j * kTileWaves + wave) * 1024 + 16 * lane, R = (o % HALF) / RB, sl = (o % RB) / 16;
    lrow[j] = R;
    loff[j] = 8 * (sl ^ (o < HALF ? swzk(R) : swz(R)));
  }
  // byte offsets of this lane's operand reads in a stage: 16-byte piece 4kc + g
  // of K row r (kc: ^ 64 kc), 8 bytes of V row 4g + r / 4 (dim tile dt: ^ 32 dt);
  // the second 16 rows lie 16 RB further (the swizzle repeats)
  const int koff = r * RB + 16 * (g ^ swzk(r));
  const int voff = HALF + (4 * g + (r >> 2)) * RB + 16 * (((r & 3) >> 1) ^ swz(4 * g + (r >> 2))) + 8 * (r & 1);
  const uint32_t ring0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)&ring[0][0]) + wave * 1024);
  const TilePlan pl{const_cast<int32_t *>(plan), M};
  const int nitems = plan[0] * ncols;
  // The last tiles of a prompt see the most keys and go first; the second
  // half of the grid, which shares the compute units of the first, takes its
  // items in the opposite order, so a unit gets a long item and a short one.
  const int half = gridDim.x / 2, wg = blockIdx.x;
  const int first = wg < half ? wg : (int)gridDim.x - 1 - (wg - half);
  for (int it = first; it < nitems; it += gridDim.x) {
    const int4 pc = pl.pieces()[it / ncols];
    const int col = it % ncols, row0 = pc.x, n = pc.y & 255, slot = (pc.y >> 8) - 1, st0 = pc.z, nst = pc.w;
    const int c = col / ngrp, h0 = c * G + (col % ngrp) * GH;
    const int start = ranges[2 * row0];
    // column 16 i + r of this wave: row mrow[i], head mh[i], its prefix length
    int mrow[CT], mh[CT], P[CT];
    bool bad[CT], live[CT];
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int cidx = wave * 16 * CT + 16 * i + r;
      live[i] = cidx / GH < n;
      mrow[i] = row0 + min(cidx / GH, n - 1);
      mh[i] = h0 + cidx % GH;
      P[i] = attn_prefix(Seqs{ranges, 1}, mrow[i], pmax, bad[i]);
    }
    int pmx = P[0], pmn = P[0];
#pragma unroll
    for (int i = 1; i < CT; ++i) {
      pmx = max(pmx, P[i]);
      pmn = min(pmn, P[i]);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      pmx = max(pmx, __shfl_xor(pmx, o, 64));
      pmn = min(pmn, __shfl_xor(pmn, o, 64));
    }
    pmx = __builtin_amdgcn_readfirstlane(pmx);  // this wave's columns: most and fewest keys
    pmn = __builtin_amdgcn_readfirstlane(pmn);
    __syncthreads();  // the ring and s_p of the last item are free
    if (lane == 0) s_p[wave] = pmx;
    __syncthreads();
    int Pt = s_p[0];  // keys of the tile
#pragma unroll
    for (int w = 1; w < kTileWaves; ++w) Pt = max(Pt, s_p[w]);
    const bf16_t *kb = Kc + ((size_t)start * Hkv + c) * D, *vb = Vc + ((size_t)start * Hkv + c) * D;
    // stage st (clamped: past the end the last one again, so every wave
    // issues the same count), rows clamped inside the tile's keys
    auto issue = [&](int st) {
      const int k0 = (st0 + min(st, nst - 1)) * SK;
      const uint32_t dst = ring0 + (st % S) * STAGE;
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const bf16_t *src = (j * kTileWaves + wave) * 1024 < HALF ? kb : vb;  // uniform
        ring_dma16(src + (size_t)min(k0 + lrow[j], Pt - 1) * rs + loff[j], dst + j * (kTileWaves * 1024));
      }
    };
    if (nst > 0)
#pragma unroll
      for (int st = 0; st < S - 1; ++st) issue(st);

    // q as B operands (high and low bf16 parts, rotated at P and scaled), and
    // the score of the row's own key, from the unrotated values
    u32x4 qh[CT][NKC], ql[CT][NKC];
    float sown[CT];
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const float *qp = q + ((size_t)mrow[i] * Hq + mh[i]) * D + 8 * g;
      const float *kp = knew + ((size_t)mrow[i] * Hkv + c) * D + 8 * g;
      float qf[NKC][8], dot = 0.f;
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
        for (int w = 0; w < 2; ++w) {
          const f32x4 a = *reinterpret_cast<const f32x4 *>(qp + 32 * kc + 4 * w);
          const f32x4 b = *reinterpret_cast<const f32x4 *>(kp + 32 * kc + 4 * w);
          qf[kc][4 * w] = a.x; qf[kc][4 * w + 1] = a.y; qf[kc][4 * w + 2] = a.z; qf[kc][4 * w + 3] = a.w;
          dot += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
        }
      sown[i] = xor32_sum(xor16_sum(dot)) * qscale;
#pragma unroll
      for (int kc = 0; kc < NKC / 2; ++kc)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const f32x4 cw = *reinterpret_cast<const f32x4 *>(rope + ((size_t)P[i] * HD + 32 * kc + 8 * g) * 2 + 4 * w);
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int e = 2 * w + u;
            const float cs = u ? cw.z : cw.x, sn = u ? cw.w : cw.y;
            const float x1 = qf[kc][e], x2 = qf[kc + NKC / 2][e];
            qf[kc][e] = x1 * cs - x2 * sn;
            qf[kc + NKC / 2][e] = x2 * cs + x1 * sn;
          }
        }
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc) {
        uint32_t hw[4], lw[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float a0 = qf[kc][e] * qscale, a1 = qf[kc][e + 1] * qscale;
          hw[e / 2] = pack_bf16(a0, a1);
          lw[e / 2] = pack_bf16(a0 - __uint_as_float(hw[e / 2] << 16),
                                a1 - __uint_as_float(hw[e / 2] & 0xffff0000u));
        }
        qh[i][kc] = u32x4{hw[0], hw[1], hw[2], hw[3]};
        ql[i][kc] = u32x4{lw[0], lw[1], lw[2], lw[3]};
      }
    }

    // lacc: the probabilities' sums, as the product with a row of ones
    float mx_[CT];
    f32x4 oacc[CT][NDT], lacc[CT];
    const u32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      mx_[i] = -INFINITY;
      lacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) oacc[i][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int st = 0; st < nst; ++st) {
      // stage st has landed (this wave's part) and this wave's reads of the
      // slot that is refilled next are done; the barrier extends both
      __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 2) * NL, 0));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      issue(st + S - 1);
      const int k0 = (st0 + st) * SK;
      if (k0 >= pmx) continue;  // no column of this wave sees this stage
      const unsigned char *ringp = &ring[0][0];
      const int kst = (st % S) * STAGE + koff, vst = (st % S) * STAGE + voff;
      f32x4 s[2][CT];  // [16-key half][column tile]
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < CT; ++i) s[h][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const u32x4 ka = *reinterpret_cast<const u32x4 *>(ringp + (kst ^ (64 * kc)) + 16 * h * RB);
#pragma unroll
          for (int i = 0; i < CT; ++i) {
            s[h][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ka), __builtin_bit_cast(bf16x8, ql[i][kc]), s[h][i], 0, 0, 0);
            s[h][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, ka), __builtin_bit_cast(bf16x8, qh[i][kc]), s[h][i], 0, 0, 0);
          }
        }
      const bool masked = k0 + SK > pmn;  // some column sees only part of the stage
      if (masked) {
#pragma unroll
        for (int i = 0; i < CT; ++i) {
          const int left = P[i] - k0 - 4 * g;  // this lane's keys 16h + v below it are seen
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (16 * h + v >= left) s[h][i][v] = -INFINITY;
        }
      }
      u32x4 pb[CT];  // lane (r, g): keys 4g + e of the first half, then of the second
#pragma unroll
      for (int i = 0; i < CT; ++i) {
        float mx = fmaxf(fmaxf(fmaxf(s[0][i].x, s[0][i].y), fmaxf(s[0][i].z, s[0][i].w)),
                         fmaxf(fmaxf(s[1][i].x, s[1][i].y), fmaxf(s[1][i].z, s[1][i].w)));
        mx = xor32_max(xor16_max(mx));
        const bool up = mx > mx_[i] + kLazyMax;
        if (__builtin_amdgcn_ballot_w64(up)) {
          const float mn = up ? mx : mx_[i];
          const float alpha = sexp2(mx_[i], mn);
          mx_[i] = mn;
          lacc[i] *= alpha;
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) oacc[i][dt] *= alpha;
        }
        // a column that has seen no key yet has the maximum -inf: subtract 0
        const float m = mx_[i] == -INFINITY ? 0.f : mx_[i];
        auto p2 = [&](float a, float b) {
          return pack_bf16(__builtin_amdgcn_exp2f(a - m), __builtin_amdgcn_exp2f(b - m));
        };
        pb[i] = u32x4{p2(s[0][i].x, s[0][i].y), p2(s[0][i].z, s[0][i].w),
                      p2(s[1][i].x, s[1][i].y), p2(s[1][i].z, s[1][i].w)};
        lacc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, pb[i]), lacc[i], 0, 0, 0);
      }
      if (masked) {
        uint32_t odd = 0;  // a non-finite value in the stage's V rows
#pragma unroll 2
        for (int o = 16 * lane; o < HALF; o += 1024) {
          const u32x4 w4 = *reinterpret_cast<const u32x4 *>(ringp + (st % S) * STAGE + HALF + o);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t x = w4[w];
            odd |= (uint32_t)((x & 0x7f80u) == 0x7f80u) | (uint32_t)((x & 0x7f800000u) == 0x7f800000u);
          }
        }
        if (__builtin_amdgcn_ballot_w64(odd != 0)) {
          // some column must not see a value row that holds an infinity or
          // NaN, and 0 * inf would reach it through the product: key by key,
          // each column over its own keys only
          const unsigned char *vr = ringp + (st % S) * STAGE + HALF;
#pragma unroll 1
          for (int key = 0; key < SK; ++key) {
            const int h = key >> 4, gg = (key & 15) >> 2, e = key & 3;
            float p[CT];
#pragma unroll
            for (int i = 0; i < CT; ++i) {
              const uint32_t w0 = h ? pb[i].z : pb[i].x, w1 = h ? pb[i].w : pb[i].y;
              const uint32_t pw = __shfl((e >> 1) ? w1 : w0, r + 16 * gg, 64);
              p[i] = (e & 1) ? __uint_as_float(pw & 0xffff0000u) : __uint_as_float(pw << 16);
            }
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
              const u32x2 vw = *reinterpret_cast<const u32x2 *>(
                  vr + key * RB + 16 * ((2 * dt + (g >> 1)) ^ swz(key)) + 8 * (g & 1));
              const f32x4 vf = {__uint_as_float(vw.x << 16), __uint_as_float(vw.x & 0xffff0000u),
                                __uint_as_float(vw.y << 16), __uint_as_float(vw.y & 0xffff0000u)};
#pragma unroll
              for (int i = 0; i < CT; ++i)
                if (k0 + key < P[i]) oacc[i][dt] += vf * p[i];
            }
          }
          continue;
        }
      }
      // V^T by the transposing read (see attn_unit), for the two 16-key halves
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const unsigned char *vp = ringp + (vst ^ (32 * dt));
        const u32x2 a0 = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                       (__attribute__((address_space(3))) i16x4 *)vp));
        const u32x2 a1 = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                       (__attribute__((address_space(3))) i16x4 *)(vp + 16 * RB)));
        const u32x4 av = {a0.x, a0.y, a1.x, a1.y};
#pragma unroll
        for (int i = 0; i < CT; ++i)
          oacc[i][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, pb[i]), oacc[i][dt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));  // the stages fetched past the end

    // the row's own key and value, then the output row
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const float lt = lacc[i].x;  // every row of the product with ones is the column's sum
      if (slot >= 0 && st0 > 0) {  // a later piece of a cut tile: its sums as they are
        if (!live[i]) continue;
        const int cidx = wave * 16 * CT + 16 * i + r;
        float *ps = parts + ((size_t)slot * ncols + col) * (kTileQ * (D + 2));
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) *reinterpret_cast<f32x4 *>(ps + cidx * D + 16 * dt + 4 * g) = oacc[i][dt];
        if (g == 0) *reinterpret_cast<float2 *>(ps + kTileQ * D + 2 * cidx) = float2{mx_[i], lt};
        continue;
      }
      const float M = fmaxf(mx_[i], sown[i]);
      const float sp = sexp2(mx_[i], M), sc = __builtin_amdgcn_exp2f(sown[i] - M);
      float inv = 1.f / (lt * sp + sc);
      if (bad[i]) inv = __int_as_float(0x7fc00000);  // P outside [0, pmax]
      if (!live[i]) continue;
      const float *vp = vnew + ((size_t)mrow[i] * Hkv + c) * D + 4 * g;
      if (slot >= 0) {  // the first piece of a cut tile, which takes the own key
        const int cidx = wave * 16 * CT + 16 * i + r;
        float *ps = parts + ((size_t)slot * ncols + col) * (kTileQ * (D + 2));
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
          *reinterpret_cast<f32x4 *>(ps + cidx * D + 16 * dt + 4 * g) =
              oacc[i][dt] * sp + *reinterpret_cast<const f32x4 *>(vp + 16 * dt) * sc;
        if (g == 0) *reinterpret_cast<float2 *>(ps + kTileQ * D + 2 * cidx) = float2{M, lt * sp + sc};
        continue;
      }
      bf16_t *op = out + ((size_t)mrow[i] * Hq + mh[i]) * D + 4 * g;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const f32x4 o = (oacc[i][dt] * sp + *reinterpret_cast<const f32x4 *>(vp + 16 * dt) * sc) * inv;
        *reinterpret_cast<u32x2 *>(op + 16 * dt) = u32x2{pack_bf16(o.x, o.y), pack_bf16(o.z, o.w)};
      }
    }
  }
}

// Rows of the cut tiles from their pieces' partials: a thread takes four dims
// of a (row, head) column, 256 threads a share of a (tile, head group).
template <int D, int GH>
__global__ __launch_bounds__(256) void k_attn_tile_merge(const int32_t *__restrict__ plan, int M,
                                                         const float *__restrict__ parts,
                                                         bf16_t *__restrict__ out, int Hq, int Hkv) {
  constexpr int TPC = D / 4, SHARES = kTileQ * TPC / 256, SLOT = kTileQ * (D + 2);
  const TilePlan pl{const_cast<int32_t *>(plan), M};
  const int G = Hq / Hkv, ngrp = G / GH, ncols = Hkv * ngrp, units = plan[1] * ncols * SHARES;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const int item = u / SHARES, col = item % ncols;
    const int4 ct = pl.cut()[item / ncols];
    const int idx = (u % SHARES) * 256 + threadIdx.x, cidx = idx / TPC, e = idx % TPC * 4;
    if (cidx / GH >= ct.y) continue;
    const int m = ct.x + cidx / GH, h = col / ngrp * G + col % ngrp * GH + cidx % GH, np = ct.w;
    const float *ps = parts + ((size_t)ct.z * ncols + col) * SLOT;
    const size_t step = (size_t)ncols * SLOT;
    float mx = -INFINITY, L = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    constexpr int R = 8;  // partials per round trip
    for (int k0 = 0; k0 < np; k0 += R) {
      f32x4 ov[R];
      float2 ml[R];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const float *p = ps + min(k0 + k, np - 1) * step;
        ov[k] = *reinterpret_cast<const f32x4 *>(p + cidx * D + e);
        ml[k] = *reinterpret_cast<const float2 *>(p + kTileQ * D + 2 * cidx);
      }
      float mn = mx;
#pragma unroll
      for (int k = 0; k < R; ++k) mn = fmaxf(mn, ml[k].x);
      const float old = sexp2(mx, mn);
      o *= old;
      L *= old;
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (k0 + k < np) {
          const float w = sexp2(ml[k].x, mn);
          o += ov[k] * w;
          L += ml[k].y * w;
        }
      mx = mn;
    }
    o *= 1.f / L;
    *reinterpret_cast<u32x2 *>(out + ((size_t)m * Hq + h) * D + e) =
        u32x2{pack_bf16(o.x, o.y), pack_bf16(o.z, o.w)};
  }
}

template <typename T, int D>
static hipError_t attn_t(const void *K, const void *V, Seqs cu, const float *q,
                         const float *knew, const float *vnew, int nctx, float *part, int nch,
                         int nch_ld, int cpw, void *out, int B, int Hq, int Hkv, int pmax,
                         hipStream_t s) {
  const int G = Hq / Hkv;
  const int GH = (G % 4 == 0) ? 4 : (G % 2 == 0 ? 2 : 1);
  const int nwg = nch < 1 ? 1 : (nch + cpw - 1) / cpw;
  const dim3 grid(Hkv * (G / GH), nwg, B);
#define FE_ATTN(GHV)                                                                            \
  hipLaunchKernelGGL((k_attn<T, D, GHV>), grid, dim3(256), 0, s, (const T *)K, (const T *)V, cu, \
                     q, knew, vnew, nctx, part, nwg, nch_ld, cpw, (T *)out, Hq, Hkv, pmax)
  if (GH == 4) FE_ATTN(4);
  else if (GH == 2) FE_ATTN(2);
  else FE_ATTN(1);
#undef FE_ATTN
  return hipGetLastError();
}

// Waves that stay resident at once: four one-wave workgroups per CU.
static int resident_waves() {
  static int n[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1024;
  if (n[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    n[dev] = 4 * cus;
  }
  return n[dev];
}

template <int D>
static hipError_t attn_mma_t(const void *K, const void *V, Seqs cu, const float *q,
                             const float *knew, const float *vnew, int nctx, float *part, int nch,
                             int nch_ld, int cpw, void *out, int B, int Hq, int Hkv,
                             const float *rope, int cascade, int pmax, int *persisted,
                             int *csplit, hipStream_t s) {
  const int G = Hq / Hkv;
  // query heads per wave (the MFMA tiles have 16 columns; more than 8 heads
  // would spill the cascade step's registers)
  const int GH = G % 8 == 0 ? 8 : G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1;
  const int nwg = nch < 1 ? 1 : (nch + cpw - 1) / cpw;
  const int ncols = Hkv * (G / GH);
  // persistent waves when the units outnumber the resident waves
  const int waves = resident_waves();
  const int persist = B <= 256 && (long)B * ncols * nwg > waves ? 1 : 0;
  *persisted = persist;
  // a launch whose partials are merged anyway gives the cascade keys units of
  // their own (one more partial slot per sequence)
  const int split = !persist && nwg > 1 ? 1 : 0;
  *csplit = split;
  const dim3 grid = persist ? dim3(waves) : dim3(ncols, nwg + split, B);
  // a span of at most 4 stages is requested whole by the ring's prologue
  const bool short_span = cpw * (kAttnChunk / 16) <= 4;
#define FE_ATTN(GHV, DEP, NCXV)                                                                  \
  hipLaunchKernelGGL((k_attn_mma<D, GHV, DEP, NCXV>), grid, dim3(64), 0, s, (const bf16_t *)K,   \
                     (const bf16_t *)V, cu, q, knew, vnew, nctx, part, nwg, nch_ld, cpw,         \
                     (bf16_t *)out, Hq, Hkv, rope, cascade, B, persist, split, pmax)
#define FE_ATTN_NCX(GHV, DEP)                                                                    \
  if (nctx <= 8) FE_ATTN(GHV, DEP, 8);                                                           \
  else FE_ATTN(GHV, DEP, kMaxLayers)
#define FE_ATTN_GH(GHV)                                                                          \
  if (short_span) { FE_ATTN_NCX(GHV, 5); }                                                       \
  else { FE_ATTN_NCX(GHV, 4); }
  switch (GH) {
    case 8: FE_ATTN_GH(8); break;
    case 4: FE_ATTN_GH(4); break;
    case 2: FE_ATTN_GH(2); break;
    default: FE_ATTN_GH(1); break;
  }
#undef FE_ATTN_GH
#undef FE_ATTN_NCX
#undef FE_ATTN
  return hipGetLastError();
}

// Enough workgroups to keep every CU busy with several at a time until the
// end (one-wave workgroups, four per CU) and no more: a sequence split over
// more workgroups only adds set-up work and partials to merge.
// A launch of at most a few rounds of resident waves (batch 1 at every model
// shape) instead takes the fewest chunks per unit that keep it to one round
// and its merge to one round trip (32 partials per head): measured at batch 1,
// 13B-shaped (40 KV heads, P 2048) 16.3 us per layer against 31.1 with one
// chunk per unit, 70B-shaped (P 4096) 16.2 against 19.0, 8B-shaped unchanged.
int attention_cpw(int B, int Hkv, int ngroups, int nch) {
  constexpr long kTargetWorkgroups = 4096;
  const long cols = (long)B * Hkv * ngroups, units = cols * nch;
  long cpw = (units + kTargetWorkgroups - 1) / kTargetWorkgroups;
  if (units <= kTargetWorkgroups) {
    const long waves = resident_waves();
    const long one_round = (units + waves - 1) / waves, one_trip = (nch + 31) / 32;
    cpw = one_round > one_trip ? one_round : one_trip;
  }
  if (cpw > nch) cpw = nch;
  return cpw < 1 ? 1 : (int)cpw;
}

// query heads of one column group: the tiles carry kTileQ / GH rows
static int tile_heads(int G) { return G % 8 == 0 ? 8 : G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1; }

// Partial results that fit behind the plan; none where no history is long
// enough for a tile to be cut.
static int tile_slots(int M, int pmax, int D, size_t floats) {
  if ((pmax + kTileKeys - 1) / kTileKeys <= kWholeStages) return 0;
  const size_t n = (floats - tile_plan_ints(M)) / ((size_t)kTileQ * (D + 2));
  return (int)std::min<size_t>(n, kTilePlanPieces);
}

hipError_t attn_tile_plan(const int32_t *ranges, int M, int pmax, int Hq, int Hkv, int D,
                          float *scratch, size_t floats, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (floats < tile_plan_ints(M)) return hipErrorInvalidValue;
  const int GH = tile_heads(Hq / Hkv);
  hipLaunchKernelGGL(k_attn_tile_plan, dim3(1), dim3(1024), 0, s, ranges, M, pmax, kTileQ / GH, Hq / GH,
                     tile_slots(M, pmax, D, floats), std::min(resident_waves() / 2, kTilePlanSplit),
                     (int32_t *)scratch);
  return hipGetLastError();
}

hipError_t attention_tiles(const void *K, const void *V, const int32_t *ranges, float *scratch,
                           size_t floats, int M, const float *q, const float *knew,
                           const float *vnew, void *out, int Hq, int Hkv, int D,
                           const float *rope, int pmax, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (floats < tile_plan_ints(M)) return hipErrorInvalidValue;
  const int GH = tile_heads(Hq / Hkv);
  const bool cut = tile_slots(M, pmax, D, floats) > 0;  // the plan may have cut tiles
  // two workgroups per CU; each takes every gridDim.x-th (piece, head group)
  const long items = (long)M * (Hq / GH), wgs = resident_waves() / 2;
  const dim3 grid((unsigned)(cut || items > wgs ? wgs : items));
  const int32_t *plan = (const int32_t *)scratch;
  float *parts = scratch + tile_plan_ints(M);
#define FE_ATTN_TILE(DV, GHV)                                                                     \
  hipLaunchKernelGGL((k_attn_tile<DV, GHV>), grid, dim3(64 * kTileWaves), 0, s, (const bf16_t *)K, \
                     (const bf16_t *)V, ranges, plan, M, q, knew, vnew, (bf16_t *)out, parts, Hq,  \
                     Hkv, rope, pmax);                                                             \
  if (cut)                                                                                         \
    hipLaunchKernelGGL((k_attn_tile_merge<DV, GHV>), dim3((wgs + 1) / 2), dim3(256), 0, s, plan, M, parts, \
                       (bf16_t *)out, Hq, Hkv)
#define FE_ATTN_TILE_D(DV)                 \
  switch (GH) {                            \
    case 8: FE_ATTN_TILE(DV, 8); break;    \
    case 4: FE_ATTN_TILE(DV, 4); break;    \
    case 2: FE_ATTN_TILE(DV, 2); break;    \
    default: FE_ATTN_TILE(DV, 1); break;   \
  }
  if (D == 128) FE_ATTN_TILE_D(128) else FE_ATTN_TILE_D(64)
#undef FE_ATTN_TILE_D
#undef FE_ATTN_TILE
  return hipGetLastError();
}

hipError_t attention(int dt, const void *K, const void *V, Seqs cu, const float *q,
                     const float *knew, const float *vnew, int nctx, float *part, int nch,
                     int nch_ld, int cpw, void *out, int B, int Hq, int Hkv, int D,
                     const float *rope, int cascade, int pmax, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  if (cpw < 1) cpw = 1;
  hipError_t e;
  int persisted = 0, csplit = 0;
  if (nctx < 1 || nctx > kMaxLayers) return hipErrorInvalidValue;
  if (dt)
    e = D == 128 ? attn_mma_t<128>(K, V, cu, q, knew, vnew, nctx, part, nch, nch_ld, cpw, out, B,
                                   Hq, Hkv, rope, cascade, pmax, &persisted, &csplit, s)
                 : attn_mma_t<64>(K, V, cu, q, knew, vnew, nctx, part, nch, nch_ld, cpw, out, B,
                                  Hq, Hkv, rope, cascade, pmax, &persisted, &csplit, s);
  else
    e = D == 128 ? attn_t<float, 128>(K, V, cu, q, knew, vnew, nctx, part, nch, nch_ld, cpw, out,
                                      B, Hq, Hkv, pmax, s)
                 : attn_t<float, 64>(K, V, cu, q, knew, vnew, nctx, part, nch, nch_ld, cpw, out,
                                     B, Hq, Hkv, pmax, s);
  if (e != hipSuccess) return e;
  const int nwg = nch < 1 ? 1 : (nch + cpw - 1) / cpw;
  if (nwg == 1 && !persisted) return hipSuccess;  // every sequence fits one workgroup
  const dim3 grid((Hq * D / 2 + 255) / 256, B);
  if (dt)
    hipLaunchKernelGGL((k_attn_merge<bf16_t, true>), grid, dim3(256), 0, s, part, nch_ld, cu,
                       kAttnChunk * cpw, nwg, (bf16_t *)out, Hq, D, persisted, csplit, pmax);
  else
    hipLaunchKernelGGL((k_attn_merge<float, false>), grid, dim3(256), 0, s, part, nch_ld, cu,
                       kAttnChunk * cpw, nwg, (float *)out, Hq, D, 0, 0, pmax);
  return hipGetLastError();
}

}  // namespace fe
