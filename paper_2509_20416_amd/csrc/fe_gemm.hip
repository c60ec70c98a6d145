// fe_gemm.hip -- weight-streaming MFMA GEMM for gfx950 with fused epilogues.
//
// Every FC of the drafter (feature fusion and input FC of Eq. 1; Q/K/V, O,
// gate/up and down projections of each cascade layer; the shared LM head) is
// Y[M, C] = A[M, K] * W[C, K]^T with a weight matrix that is read exactly once
// per pass and a handful of activation rows (M = batch, or batch x cascade
// rows).  The kernel is built around streaming W from HBM:
//
//  * A wave owns NT tiles of 16 output columns and a K slice.  Lane (r, g)
//    (r = lane % 16, g = lane / 16) loads 16 contiguous bytes of weight row
//    r at K offset g*E of every K step (E = 8 bf16 or 4 fp32 elements), which
//    is exactly the B operand of v_mfma_f32_16x16x32_bf16 (one MFMA per step)
//    or of four v_mfma_f32_16x16x4_f32.  No LDS staging for weights, no
//    re-reads: each weight byte is loaded by one lane once.
//  * Activation rows are the A operand, loaded with the same (g, element) ->
//    k mapping, so the products pair up correctly whatever order the matrix
//    core sums the K elements in.  Rows beyond M are fed as zeros.
//  * Loads are double-buffered in registers: the next U steps of weights and
//    activations are in flight while the current U steps run on the MFMA.
//  * WK waves of a workgroup split K; their partial tiles are summed in LDS in
//    a fixed order (deterministic, no atomics), then an epilogue functor
//    consumes the [M, span] fp32 tile.
//  * Which weight row feeds a "virtual column" is the epilogue's choice:
//    Q/K tiles pair rotary halves (dims m and m + D/2) inside one 16-column
//    tile; gate/up tiles pair gate row c with up row c.
#include "fe_internal.h"
#include <algorithm>
#include <type_traits>
#include <utility>

namespace fe {

template <typename T> __device__ __forceinline__ void mma16(f32x4 &acc, u32x4 a, u32x4 b);

template <> __device__ __forceinline__ void mma16<uint16_t>(f32x4 &acc, u32x4 a, u32x4 b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// Four K=4 fp32 MFMAs, one per element of the lanes' 16-byte fragments.  The
// elements are named explicitly: a loop over a vector element index here was
// compiled to four uses of element 0.
template <> __device__ __forceinline__ void mma16<float>(f32x4 &acc, u32x4 a, u32x4 b) {
  const f32x4 af = __builtin_bit_cast(f32x4, a), bf = __builtin_bit_cast(f32x4, b);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af.x, bf.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af.y, bf.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af.z, bf.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af.w, bf.w, acc, 0, 0, 0);
}

__device__ __forceinline__ u32x4 ldg_stream(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// ---------------------------------------------------------------------------
// Accumulation (up to 32 rows).  Leaves, in lane (r, g) of a wave, the 16x16
// tiles acc[i][f] = rows 16i.. of A times weight rows of virtual columns
// c0+16f.., summed over this wave's share of K.
// ---------------------------------------------------------------------------

// Staged path (M <= 32): weights are read as 512-byte contiguous pieces of
// two rows per load instruction (the access pattern HBM streams best), parked
// in the wave's own padded LDS tile, and read back as MFMA B fragments; the
// next 512-byte chunk of every row is in flight while the current one is
// multiplied.  K is walked in chunks of KC elements, split over WK waves.
constexpr int kStageRowBytes = 512 + 16;  // padded LDS row: 16 rows hit distinct banks

template <typename T, int MT, int NT, class Epi>
__device__ __forceinline__ void accum_staged(const T *__restrict__ A, int lda, const ARows &ar_,
                                             int M, int K, const Epi &epi, int c0, int wk,
                                             int WKn, char *stage, f32x4 (&acc)[MT][NT]) {
  constexpr int E = Elt<T>::kPer16B;
  constexpr int KC = 32 * E;       // elements per chunk: 512 bytes of a row
  constexpr int KS = 4 * E;        // elements per MFMA step
  constexpr int STEPS = KC / KS;   // 8
  constexpr int NLD = NT * 8;      // load instructions per chunk (2 rows each)
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int half = lane >> 5, l32 = lane & 31;
  const int nchunk = (K + KC - 1) / KC;
  const int ch0 = (int)(((long)nchunk * wk) / WKn), ch1 = (int)(((long)nchunk * (wk + 1)) / WKn);
  if (ch0 >= ch1) return;
  const u32x4 *src[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j)
    src[j] = reinterpret_cast<const u32x4 *>(epi.wrow(c0 + 2 * j + half)) + l32;
  const u32x4 *ap[MT];
  bool am[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = i * 16 + r;
    am[i] = m < M;
    ap[i] = reinterpret_cast<const u32x4 *>(A + (size_t)(am[i] ? ar_.row(m) : 0) * lda) + g;
  }
  const u32x4 zero = {0u, 0u, 0u, 0u};
  u32x4 wr[NLD], ar[STEPS][MT];
  auto load = [&](int ch) {
    const int kb = ch * KC;
    const bool wok = kb + l32 * E < K;
#pragma unroll
    for (int j = 0; j < NLD; ++j) wr[j] = wok ? ldg_stream(src[j] + ch * 32) : zero;
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
#pragma unroll
      for (int i = 0; i < MT; ++i)
        ar[st][i] = (am[i] && kb + st * KS + g * E < K) ? ap[i][ch * 32 + st * 4] : zero;
  };
  load(ch0);
  for (int ch = ch0; ch < ch1; ++ch) {
    // the previous chunk's LDS reads are complete before its rows are overwritten
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int j = 0; j < NLD; ++j)
      *reinterpret_cast<u32x4 *>(stage + (2 * j + half) * kStageRowBytes + l32 * 16) = wr[j];
    u32x4 ac[STEPS][MT];
#pragma unroll
    for (int st = 0; st < STEPS; ++st)
#pragma unroll
      for (int i = 0; i < MT; ++i) ac[st][i] = ar[st][i];
    // this chunk's rows are in LDS before any lane reads them
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (ch + 1 < ch1) load(ch + 1);
    const int nst = min(STEPS, (K - ch * KC) / KS);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st < nst) {
#pragma unroll
        for (int f = 0; f < NT; ++f) {
          const u32x4 bfr = *reinterpret_cast<const u32x4 *>(
              stage + (f * 16 + r) * kStageRowBytes + st * 64 + g * 16);
#pragma unroll
          for (int i = 0; i < MT; ++i) mma16<T>(acc[i][f], ac[st][i], bfr);
        }
      }
    }
  }
}

// Epilogues with kSliced = true cover many row blocks (and groups) in one
// launch: a grid dimension (z for k_gemm_mid, y for k_gemm) enumerates them
// and slice() moves A, M and the epilogue's outputs to its block before
// anything else runs.
template <class E, class = void> struct SlicedEpi { static constexpr bool value = false; };
template <class E> struct SlicedEpi<E, decltype((void)E::kSliced)> {
  static constexpr bool value = E::kSliced;
};

// Epilogues with a member bx, the storing ones: the workgroup's column block,
// where it is not blockIdx.x (k_gemm_tile), by which it picks embedding rows.
template <class E, class = void> struct HasBlock { static constexpr bool value = false; };
template <class E> struct HasBlock<E, decltype((void)std::declval<E>().bx)> {
  static constexpr bool value = true;
};

// ---------------------------------------------------------------------------
// The GEMM body: WN x WK waves; wave (wn, wk) owns NT 16-column tiles and the
// wk-th share of K.  Partial tiles are summed over wk in LDS in a fixed order
// (deterministic, no atomics), then the epilogue consumes the [M, span] tile.
// ---------------------------------------------------------------------------
template <typename T, int MT, int NT, int WK, int WN, bool NORM, class Epi>
__global__ __launch_bounds__(64 * WK * WN) void k_gemm(const T *__restrict__ A, int lda, ARows arows,
                                                       int M, int K, NormA na, Epi epi) {
  static_assert(MT <= 2, "more than 32 rows take k_gemm_mid");
  static_assert(!NORM || MT == 1, "fused RMSNorm is for M <= 16");
  constexpr int NTHR = 64 * WK * WN;
  constexpr int SPAN = WN * NT * 16;
  constexpr int LDT = SPAN + 1;
  constexpr int kStageBytes = WK * WN * NT * 16 * kStageRowBytes;
  constexpr int kRedBytes = WK * MT * 16 * LDT * 4;
  constexpr int kSmem = kStageBytes > kRedBytes ? kStageBytes : kRedBytes;
  __shared__ __attribute__((aligned(16))) char smem[kSmem];
  __shared__ float s_inv[16];
  float(*red)[MT * 16][LDT] = reinterpret_cast<float(*)[MT * 16][LDT]>(smem);

  if constexpr (SlicedEpi<Epi>::value) {  // grid y: the epilogue's slices
    const T *a = A;
    epi.slice(blockIdx.y, MT * 16, a, M);
    A = a;
    if (M <= 0) return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wn = wave % WN, wk = wave / WN;
  const int r = lane & 15, g = lane >> 4;
  const int c0_wg = blockIdx.x * SPAN;
  const int c0 = c0_wg + wn * NT * 16;

  // Fused RMSNorm: A holds gamma * x rows; each row's 1/rms comes from the
  // producer's per-tile sums of squares.  Thread t sums tiles p, p+PARTS, ...
  // of row t / PARTS; the loads are issued here and consumed after the main
  // loop, so their latency hides behind the weight stream.
  constexpr int PARTS = NTHR / 16;
  constexpr int kNormLoads = 16;  // tiles per thread covered by the unrolled loads
  float nv[NORM ? kNormLoads : 1];
  const int nrow = threadIdx.x / PARTS, npart = threadIdx.x % PARTS;
  if constexpr (NORM) {
    const float *sr = na.ssq + (size_t)na.row(min(nrow, M - 1)) * na.ntile;
#pragma unroll
    for (int u = 0; u < kNormLoads; ++u) nv[u] = sr[min(npart + PARTS * u, na.ntile - 1)];
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < NT; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};

  const typename Epi::Pre pre{};  // the epilogue loads its own values here
  if (c0 < epi.nvcols)
    accum_staged<T, MT, NT>(A, lda, arows, M, K, epi, c0, wk, WK,
                            smem + wave * NT * 16 * kStageRowBytes, acc);
  if constexpr (NORM) {
    float ssum = 0.f;
#pragma unroll
    for (int u = 0; u < kNormLoads; ++u) ssum += (npart + PARTS * u < na.ntile) ? nv[u] : 0.f;
    const float *sr = na.ssq + (size_t)na.row(min(nrow, M - 1)) * na.ntile;
    for (int t = npart + PARTS * kNormLoads; t < na.ntile; t += PARTS) ssum += sr[t];
    static_assert(PARTS >= 8 && PARTS <= 64, "row partials reduce over 8..64 lanes");
    ssum = group_sum<PARTS>(ssum);
    if (npart == 0 && nrow < M) s_inv[nrow] = 1.0f / sqrtf(ssum / (float)na.d + na.eps);
  }
  __syncthreads();  // staging tiles are dead; the buffer becomes the reduction tile

  // Lane (r, g) holds C[row 4g+v][col r] of each 16x16 tile.
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < NT; ++f)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wk][i * 16 + 4 * g + v][wn * NT * 16 + f * 16 + r] = acc[i][f][v];
  __syncthreads();
  if (WK > 1 || NORM) {
    for (int idx = threadIdx.x; idx < MT * 16 * SPAN; idx += NTHR) {
      const int m = idx / SPAN, c = idx % SPAN;
      float sum = red[0][m][c];
#pragma unroll
      for (int w = 1; w < WK; ++w) sum += red[w][m][c];
      if constexpr (NORM) sum *= (m < M ? s_inv[m] : 0.f);
      red[0][m][c] = sum;
    }
    __syncthreads();
  }
  epi.finish(&red[0][0][0], LDT, M, c0_wg, SPAN, pre);
}

// ---------------------------------------------------------------------------
// Row-streaming path for 1..4 input rows (batch-1 layers): no matrix cores, no
// weight staging.  A workgroup of W waves owns SPAN = 4W
// virtual columns; wave w takes weight rows 4w..4w+3 with 16 lanes per row,
// so every load instruction reads 256 contiguous bytes of each of 4 rows and
// a lane only ever accumulates its own row.  The input rows are in LDS in the
// storage type (zero-padded to whole pieces) and meet the weights in
// v_dot2c_f32_bf16, or in fp32 multiply-adds, as they arrive; two register banks of kGvDepth pieces per
// lane alternate, one in flight while the other is consumed.  Each row's sum
// is reduced over its 16 lanes with DPP; the [M, SPAN] tile goes to the same
// epilogues as the matrix-core paths.
// ---------------------------------------------------------------------------
constexpr int kGvDepth = 8;
constexpr int kGvMaxLds = 64 * 1024;  // bytes of input rows in LDS

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// Each 32-bit word goes through a scalar before the bit cast: a bit cast of a
// vector element (w.y) itself is compiled as a read of element 0.
__device__ __forceinline__ float dot8(u32x4 w, u32x4 x, float acc) {
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
  const uint32_t x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w0), __builtin_bit_cast(bf16x2_t, x0), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w1), __builtin_bit_cast(bf16x2_t, x1), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w2), __builtin_bit_cast(bf16x2_t, x2), acc, false);
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w3), __builtin_bit_cast(bf16x2_t, x3), acc, false);
}

// One 16-byte piece of a weight row times the same piece of an input row.
__device__ __forceinline__ float dot_piece(bf16_t, u32x4 w, u32x4 x, float acc) { return dot8(w, x, acc); }
__device__ __forceinline__ float dot_piece(float, u32x4 w, u32x4 x, float acc) {
  const f32x4 a = __builtin_bit_cast(f32x4, w), b = __builtin_bit_cast(f32x4, x);
  acc = fmaf(a.x, b.x, acc);
  acc = fmaf(a.y, b.y, acc);
  acc = fmaf(a.z, b.z, acc);
  return fmaf(a.w, b.w, acc);
}

template <typename T, int MR, int W, bool NORM, class Epi>
__global__ __launch_bounds__(64 * W) void k_gemv(const T *__restrict__ A, int lda, ARows arows,
                                                 int M, int K, NormA na, Epi epi) {
  constexpr int E = Elt<T>::kPer16B;  // elements per 16-byte piece
  constexpr int PE = 16 * E;          // a row's elements per load instruction
  constexpr int SPAN = 4 * W;
  constexpr int NTHR = 64 * W;
  extern __shared__ __attribute__((aligned(16))) char xs_raw[];
  __shared__ float tile[MR][SPAN + 1];
  __shared__ float s_inv[MR];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, rq = lane >> 4, l16 = lane & 15;
  const int c0 = blockIdx.x * SPAN;
  // unsigned: a signed division by the runtime xper below is twice the
  // instructions, all of them ahead of the input rows' loads
  const unsigned kpad = ((unsigned)K + PE - 1) / PE * PE;
  const int npc = kpad / PE;  // 16-byte pieces per lane per row
  T *xs = reinterpret_cast<T *>(xs_raw);

  // weight row of this lane (clamped; columns past the end are dropped at the end)
  const int col = c0 + wave * 4 + rq;
  const T *wr = epi.wrow(min(col, epi.nvcols - 1));
  // piece p of the row: elements p*PE + E*l16 ..; past K the address is
  // clamped in bounds and the (finite) weights meet zero-padded inputs
  auto ldw = [&](int p) {
    return ldg_stream(reinterpret_cast<const u32x4 *>(wr + min(p * PE + l16 * E, K - E)));
  };
  // every independent load is issued before anything is consumed, so the
  // whole prologue costs one memory round trip: the first weight pieces, the
  // input rows (registers, then LDS), the norm partials, the epilogue's values
  u32x4 ba[kGvDepth], bb[kGvDepth];
#pragma unroll
  for (int i = 0; i < kGvDepth; ++i) ba[i] = ldw(min(i, npc - 1));

  constexpr int XPT = kGvMaxLds / 16 / NTHR;  // input pieces per thread, at most
  const unsigned xper = kpad / E;
  const int xtot = MR * xper;
  // input piece idx: row m, elements e .. of it
  auto xrow = [&](int idx) { return MR == 1 ? 0 : (int)((unsigned)idx / xper); };
  auto xel = [&](int idx) { return (MR == 1 ? idx : (int)((unsigned)idx % xper)) * E; };
  u32x4 xr[XPT];
#pragma unroll
  for (int u = 0; u < XPT; ++u)
    if (NTHR * u < xtot) {  // uniform: batch u holds at least one piece
      const int idx = min(tid + NTHR * u, xtot - 1);
      const int m = xrow(idx), e = min(xel(idx), K - E);
      xr[u] = *reinterpret_cast<const u32x4 *>(A + (size_t)arows.row(min(m, M - 1)) * lda + e);
    }

  constexpr int PARTS = NTHR / 16;
  constexpr int kNormLoads = 16;
  float nv[NORM ? kNormLoads : 1];
  const int nrow = tid / PARTS, npart = tid % PARTS;
  if constexpr (NORM) {
    const float *sr = na.ssq + (size_t)na.row(min(nrow, M - 1)) * na.ntile;
#pragma unroll
    for (int u = 0; u < kNormLoads; ++u) nv[u] = sr[min(npart + PARTS * u, na.ntile - 1)];
  }
  const typename Epi::Pre pre = epi.prefetch(M, c0, SPAN);

  // input rows -> LDS, zero past K and past M
  const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int u = 0; u < XPT; ++u) {
    const int idx = tid + NTHR * u;
    if (NTHR * u < xtot && idx < xtot) {
      const int m = xrow(idx), e = xel(idx);
      *reinterpret_cast<u32x4 *>(xs + (size_t)m * kpad + e) = (m < M && e < K) ? xr[u] : zero;
    }
  }
  if constexpr (NORM) {
    float ssum = 0.f;
#pragma unroll
    for (int u = 0; u < kNormLoads; ++u) ssum += (npart + PARTS * u < na.ntile) ? nv[u] : 0.f;
    const float *sr = na.ssq + (size_t)na.row(min(nrow, M - 1)) * na.ntile;
    for (int t = npart + PARTS * kNormLoads; t < na.ntile; t += PARTS) ssum += sr[t];
    static_assert(PARTS >= 8 && PARTS <= 64, "row partials reduce over 8..64 lanes");
    ssum = group_sum<PARTS>(ssum);
    if (npart == 0 && nrow < MR) s_inv[nrow] = nrow < M ? 1.0f / sqrtf(ssum / (float)na.d + na.eps) : 0.f;
  }
  __syncthreads();

  float acc[MR];
#pragma unroll
  for (int m = 0; m < MR; ++m) acc[m] = 0.f;
  const T *xl = xs + l16 * E;
  auto consume = [&](const u32x4 (&bw)[kGvDepth], int p0) {
#pragma unroll
    for (int i = 0; i < kGvDepth; ++i) {
      const int p = p0 + i;
      if (p < npc) {
#pragma unroll
        for (int m = 0; m < MR; ++m)
          acc[m] = dot_piece(T(), bw[i], *reinterpret_cast<const u32x4 *>(xl + (size_t)m * kpad + p * PE), acc[m]);
      }
    }
  };
  for (int p0 = 0; p0 < npc; p0 += 2 * kGvDepth) {
#pragma unroll
    for (int i = 0; i < kGvDepth; ++i) bb[i] = ldw(min(p0 + kGvDepth + i, npc - 1));
    consume(ba, p0);
#pragma unroll
    for (int i = 0; i < kGvDepth; ++i) ba[i] = ldw(min(p0 + 2 * kGvDepth + i, npc - 1));
    consume(bb, p0 + kGvDepth);
  }
#pragma unroll
  for (int m = 0; m < MR; ++m) {
    float v = group_sum<16>(acc[m]);
    if constexpr (NORM) v *= s_inv[m];
    if (l16 == 0) tile[m][wave * 4 + rq] = v;
  }
  __syncthreads();
  epi.finish(&tile[0][0], SPAN + 1, M, c0, SPAN, pre);
}

// ---------------------------------------------------------------------------
// Batched rows (17..256): one workgroup owns BN = 16*NTW*WN output columns and
// every row; its four waves form WM = 4/WN row groups of 64 rows and WN column
// groups of 16*NTW columns.  K advances in chunks of 128 bytes per row.  The
// chunks of A (all rows) and of the BN weight rows go straight from memory to
// an S-stage LDS ring with direct-to-LDS loads (global_load_lds_dwordx4), so
// S-1 chunks are in flight without holding registers.  One load instruction
// fills 1 KB of LDS contiguously (lane l -> byte 16l); 16-byte piece p of row
// R sits at slot p ^ ((R >> 1) & 7) of its row, which keeps the MFMA fragment
// reads free of bank conflicts without padding.  Weights are read from HBM
// once; A (at most 256/WN rows) is served by L2 to every workgroup.
// Synchronisation is a plain s_barrier after an explicit vmcnt wait: the
// workgroup fence of __syncthreads would drain every load in flight.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wg_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ int ring_slot(int row, int piece) { return row * 8 + (piece ^ ((row >> 1) & 7)); }

template <typename T, int NTW, int WN, int S, class Epi, int RT = 4>
__global__ __launch_bounds__(256) void k_gemm_mid(const T *__restrict__ A, int lda, ARows arows,
                                                  int M, int K, Epi epi, float *__restrict__ splitp,
                                                  int ldp) {
  // RT: 16-row tiles per wave (4; 2 when at most 32 rows are live, so that the
  // ring does not carry duplicated rows of A)
  static_assert(RT == 4 || RT == 2, "row tiles per wave");
  constexpr int WM = 4 / WN;
  constexpr int MROWS = 16 * RT * WM;  // rows this configuration holds
  if constexpr (SlicedEpi<Epi>::value) {
    const T *a = A;
    epi.slice(blockIdx.z, MROWS, a, M);
    A = a;
    if (M <= 0) return;  // the whole workgroup: past the last row block
  }
  constexpr int E = Elt<T>::kPer16B;  // elements per 16-byte piece
  constexpr int KC = 8 * E;           // elements of K per chunk
  constexpr int BN = NTW * WN * 16;
  static_assert(BN % 32 == 0, "weight slots must split evenly over the four waves");
  constexpr int AI = MROWS / 32;      // A load instructions per wave per stage
  constexpr int WI = BN / 32;         // weight load instructions per wave per stage
  constexpr int CNT = AI + WI;
  static_assert((S - 2) * CNT <= 63, "vmcnt range");
  constexpr int ABYTES = MROWS * 128, STAGE = ABYTES + BN * 128;
  constexpr int LDT = BN + 1;
  constexpr int TILE = MROWS * LDT * 4;
  constexpr int SMEM = S * STAGE > TILE ? S * STAGE : TILE;
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int c0 = blockIdx.x * BN;
  // split K over gridDim.y: this workgroup's chunks [cb, cb + nch)
  const int nchk = (K + KC - 1) / KC;
  const int cb = (int)((long)nchk * blockIdx.y / gridDim.y);
  const int nch = (int)((long)nchk * (blockIdx.y + 1) / gridDim.y) - cb;

  // the lane's slot in each of its load instructions, and the source row and
  // piece offset that belong there (rows past M repeat row M-1: their products
  // land in output rows that are never stored)
  const T *asrc[AI];
  int aoff[AI];
#pragma unroll
  for (int j = 0; j < AI; ++j) {
    const int q = (j * 4 + wave) * 64 + lane, row = q >> 3;
    asrc[j] = A + (size_t)arows.row(min(row, M - 1)) * lda;
    aoff[j] = ((q & 7) ^ ((row >> 1) & 7)) * E;
  }
  const T *wsrc[WI];
  int woff[WI];
#pragma unroll
  for (int j = 0; j < WI; ++j) {
    const int q = (j * 4 + wave) * 64 + lane, n = q >> 3;
    wsrc[j] = epi.wrow(min(c0 + n, epi.nvcols - 1));
    woff[j] = ((q & 7) ^ ((n >> 1) & 7)) * E;
  }
  // chunk ch (clamped: past the end the last chunk is fetched again, so every
  // wave issues the same count), addresses clamped inside the rows
  auto issue = [&](int ch) {
    char *st = smem + (ch % S) * STAGE;
    const int k = (cb + min(ch, nch - 1)) * KC;
#pragma unroll
    for (int j = 0; j < AI; ++j)
      lds_dma16(asrc[j] + min(k + aoff[j], K - E), st + (j * 4 + wave) * 1024);
#pragma unroll
    for (int j = 0; j < WI; ++j)
      lds_dma16(wsrc[j] + min(k + woff[j], K - E), st + ABYTES + (j * 4 + wave) * 1024);
  };

  f32x4 acc[RT][NTW];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int f = 0; f < NTW; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int mrow0 = wm * 16 * RT, ncol0 = wn * NTW * 16;
  const int mtiles = min(RT, (M - mrow0 + 15) / 16);  // this wave's live 16-row tiles (may be <= 0)

#pragma unroll
  for (int st = 0; st < S - 1; ++st) issue(st);
  for (int ch = 0; ch < nch; ++ch) {
    wait_vmcnt<(S - 2) * CNT>();  // this wave's part of chunk ch has landed
    wg_barrier();                 // so has everyone's; ring slot of chunk ch-1 is free
    issue(ch + S - 1);
    const char *st = smem + (ch % S) * STAGE;
    if (cb + ch == nchk - 1 && K % KC) {  // ragged last chunk: zero the pieces past K
      const int k = (cb + ch) * KC;
      for (int q = tid; q < (MROWS + BN) * 8; q += 256) {
        const int row = q >> 3, piece = (q & 7) ^ ((row >> 1) & 7);
        if (k + piece * E >= K) *reinterpret_cast<u32x4 *>(const_cast<char *>(st) + q * 16) = u32x4{0u, 0u, 0u, 0u};
      }
      wg_barrier();
    }
    // every fragment of the chunk is read before the first product (the ring
    // holds all MROWS rows, so the reads need no guard and are in flight
    // together); only the products skip the wave's dead row tiles
    u32x4 bf[2][NTW], af[2][RT];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int f = 0; f < NTW; ++f)
        bf[ks][f] = *reinterpret_cast<const u32x4 *>(st + ABYTES + ring_slot(ncol0 + f * 16 + r, ks * 4 + g) * 16);
#pragma unroll
      for (int i = 0; i < RT; ++i)
        af[ks][i] = *reinterpret_cast<const u32x4 *>(st + ring_slot(mrow0 + i * 16 + r, ks * 4 + g) * 16);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < RT; ++i)
        if (i < mtiles)
#pragma unroll
          for (int f = 0; f < NTW; ++f) mma16<T>(acc[i][f], af[ks][i], bf[ks][f]);
  }
  wait_vmcnt<0>();  // the chunks fetched past the end land before the ring is reused or freed
  if (splitp) {  // split K: this slice's fp32 sums, reduced (and finished) by a second launch
    float *dst = splitp + (size_t)blockIdx.y * M * ldp + c0;
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (i < mtiles)
#pragma unroll
        for (int f = 0; f < NTW; ++f)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int m = mrow0 + i * 16 + 4 * g + v;
            if (m < M) dst[(size_t)m * ldp + ncol0 + f * 16 + r] = acc[i][f][v];
          }
    return;
  }
  wg_barrier();
  float(*tile)[LDT] = reinterpret_cast<float(*)[LDT]>(smem);
#pragma unroll
  for (int i = 0; i < RT; ++i)
    if (i < mtiles)
#pragma unroll
      for (int f = 0; f < NTW; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v) tile[mrow0 + i * 16 + 4 * g + v][ncol0 + f * 16 + r] = acc[i][f][v];
  __syncthreads();
  epi.finish(&tile[0][0], LDT, M, c0, BN, typename Epi::Pre{});
}

// ---------------------------------------------------------------------------
// Many rows, matrix-core bound (the cache update, the prefill, the batched
// Q/K/V and LM head: bf16, K a multiple of 64).  Eight waves, two per SIMD, WM
// row groups x WN column groups of RT x NTW 16 x 16 tiles; column tile f of
// wave column wn is tile f * WN + wn of the workgroup.  The ring and its
// swizzle are k_gemm_mid's; the schedule is software-pipelined over the two
// 32-wide K steps of a chunk:
//   read step-1 fragments of chunk c | products of step 0 (read last round)
//   wait: chunk c+1 landed, every read of chunk c done; barrier
//   refill chunk c's slot with chunk c+S, read step-0 fragments of chunk c+1 |
//   products of step 1
// with the loads and reads of a phase woven between the products, one row of
// tiles at a time.  A wave issues in order: with all loads and reads ahead of
// the products, every wave queued behind the others' at the same moment and
// the matrix cores waited (256 x 256 tiles, K 12288: 274 us a tile, woven 236;
// 128 x 128: 124 and 119).  Waits are compiler-visible s_waitcnt immediates and
// the phases are fenced with scheduling barriers: with inline-asm waits the
// compiler hoisted the barrier (and its lgkmcnt(0)) above the products.
// What bounds it is the loop inside a CU, not memory: 64 workgroups take as
// long as 256, and a deeper ring changes nothing.  Larger tiles read fewer
// fragments per product, so they run at a higher rate while they fill the
// chip (1024 rows x 28672 columns, K 4096: 315 us with 128 x 128, 213 with
// 256 x 256, 200 with 256 x 224 tiles, whose last round is full).
// ---------------------------------------------------------------------------
//
// SPLIT: K is split over grid y and each slice's fp32 sums go to splitp
// (slice y at y * M * ldp, row m at m * ldp) for a second launch that sums them
// and runs the epilogue; the row blocks of grid z then cover rows
// arows.row(m) of A directly (no epilogue slicing).
template <int RT, int NTW, int WM, int WN, int S, class Epi, bool SPLIT = false>
__global__ __launch_bounds__(512) void k_gemm_tile(const bf16_t *__restrict__ A, int lda, ARows arows,
                                                   int M, int K, Epi epi, float *__restrict__ splitp,
                                                   int ldp, int nb) {
  constexpr int NW = WM * WN;
  static_assert(NW == 8, "eight waves");
  constexpr int BM = 16 * RT * WM, BN = 16 * NTW * WN, KC = 64;
  constexpr int ABYTES = BM * 128, STAGE = ABYTES + BN * 128;
  // 1 KB loads of a chunk: AN + WI, dealt to the waves in turn; CNT per wave
  constexpr int AN = BM / 8, LN = AN + BN / 8, CNT = (LN + NW - 1) / NW;
  static_assert(S >= 2 && (S - 1) * CNT <= 63, "vmcnt range");
  // The epilogue takes FP of the NTW column tiles per pass.  Its tile rows are
  // 4 floats longer than the span: 16-byte aligned for the vector reads, and
  // the accumulator writes (4 rows x 16 columns per instruction) land on
  // distinct banks
  constexpr int kMaxTile = 140 * 1024;
  constexpr int FP = BM * (BN + 4) * 4 <= kMaxTile ? NTW : (NTW + 1) / 2;
  constexpr int PN = 16 * FP * WN, LDT = PN + 4, TILE = BM * LDT * 4;
  static_assert(TILE <= kMaxTile && PN % 32 == 0, "epilogue passes");
  constexpr int SMEM = SPLIT || S * STAGE > TILE ? S * STAGE : TILE;
  static_assert(SMEM <= 160 * 1024, "LDS of a compute unit");
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  // Which tile: workgroups are dealt to the 8 XCDs in turn, so XCD i's share
  // of the launch order is every 8th; it takes a contiguous run of the tiles in
  // the order row block (nb per group), columns, K slice, group, whose tiles
  // share their weights and A rows in the XCD's L2 (K/V of five layers, 1024
  // rows: 114 us in launch order, 107 so).
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (gridDim.y * gridDim.z > 1) {
    const int total = gridDim.x * gridDim.y * gridDim.z;
    const int pid = bx + gridDim.x * (by + gridDim.y * bz), xcd = pid & 7;
    int id = xcd * (total >> 3) + min(xcd, total & 7) + (pid >> 3);
    bz = id % nb;
    id /= nb;
    bx = id % gridDim.x;
    id /= gridDim.x;
    by = id % gridDim.y;
    bz += (id / gridDim.y) * nb;
  }
  if constexpr (HasBlock<Epi>::value) epi.bx = bx;
  int m0 = 0, Mb = M;  // first row of this block, rows in it
  if constexpr (SPLIT) {
    m0 = bz * BM;
    Mb = min(BM, M - m0);
  } else if constexpr (SlicedEpi<Epi>::value) {
    const bf16_t *a = A;
    epi.slice(bz, BM, a, M);
    A = a;
    Mb = M;
  }  // else one row block of at most BM rows
  if (Mb <= 0) return;  // the whole workgroup: past the last row block
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int c0 = bx * BN;
  // this workgroup's chunks of K: [cb, cb + nch)
  const int nchk = K / KC;
  const int cb = SPLIT ? (int)((long)nchk * by / gridDim.y) : 0;
  const int nch = SPLIT ? (int)((long)nchk * (by + 1) / gridDim.y) - cb : nchk;
  // the lane's source in each of its loads: load j of a wave fills the 1 KB
  // (eight rows) j * NW + wave of the stage, A rows first (rows past M repeat
  // row M-1, columns past the end the last column: their products land in
  // outputs that are never stored).  Where the loads don't divide evenly, the
  // last ones repeat the stage's last kilobyte, so every wave issues CNT.
  const bf16_t *src[CNT];
  int dst[CNT];
#pragma unroll
  for (int j = 0; j < CNT; ++j) {
    const int q = min(j * NW + wave, LN - 1), row = (q < AN ? q : q - AN) * 8 + (lane >> 3);
    const int piece = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    src[j] = q < AN ? A + (size_t)arows.row(m0 + min(row, Mb - 1)) * lda + piece
                    : epi.wrow(min(c0 + row, epi.nvcols - 1)) + piece;
    dst[j] = q * 1024;
  }
  auto issue1 = [&](int j, char *st, int k) { lds_dma16(src[j] + k, st + dst[j]); };
  // K offset of chunk ch (past the end the last chunk is fetched again)
  auto koff = [&](int ch) { return (cb + min(ch, nch - 1)) * KC; };
  f32x4 acc[RT][NTW];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int f = 0; f < NTW; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int mrow0 = wm * 16 * RT;
  auto afrag = [&](const char *st, int ks, int i) {
    return *reinterpret_cast<const u32x4 *>(st + ring_slot(mrow0 + i * 16 + r, ks * 4 + g) * 16);
  };
  auto bfrag = [&](const char *st, int ks, int f) {
    return *reinterpret_cast<const u32x4 *>(
        st + ABYTES + ring_slot((f * WN + wn) * 16 + r, ks * 4 + g) * 16);
  };
  u32x4 a0[RT], b0[NTW], a1[RT], b1[NTW];
  // the products of fragments (ca, cb_), and between them the reads of step ks
  // of the chunk at `rd` into (na, nb) and, with LOAD, the loads into `ld`
  auto phase = [&](auto load, const u32x4 (&ca)[RT], const u32x4 (&cb_)[NTW], const char *rd, int ks,
                   u32x4 (&na)[RT], u32x4 (&nb)[NTW], char *ld, int k) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      if constexpr (decltype(load)::value)
#pragma unroll
        for (int j = i * CNT / RT; j < (i + 1) * CNT / RT; ++j) issue1(j, ld, k);
#pragma unroll
      for (int f = i * NTW / RT; f < (i + 1) * NTW / RT; ++f) nb[f] = bfrag(rd, ks, f);
      na[i] = afrag(rd, ks, i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < NTW; ++f) mma16<bf16_t>(acc[i][f], ca[i], cb_[f]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
#pragma unroll
  for (int st = 0; st < S; ++st)
#pragma unroll
    for (int j = 0; j < CNT; ++j) issue1(j, smem + st * STAGE, koff(st));
  __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 1) * CNT, 15));  // chunk 0 (this wave's part)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < NTW; ++f) b0[f] = bfrag(smem, 0, f);
#pragma unroll
  for (int i = 0; i < RT; ++i) a0[i] = afrag(smem, 0, i);
  for (int ch = 0; ch < nch; ++ch) {
    // the step-0 fragments (read during the last products) are in
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, 0));
    __builtin_amdgcn_sched_barrier(0);
    char *slot = smem + (ch % S) * STAGE;
    phase(std::false_type{}, a0, b0, slot, 1, a1, b1, nullptr, 0);
    // chunk ch+1 landed (this wave's part) and every read of chunk ch is done;
    // the barrier extends both to the workgroup
    __builtin_amdgcn_s_waitcnt(waitcnt_imm((S - 2) * CNT, 0));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // after the last chunk the reads take what its refetch left: unused
    phase(std::true_type{}, a1, b1, smem + ((ch + 1) % S) * STAGE, 0, a0, b0, slot, koff(ch + S));
  }
  // the chunks fetched past the end land before the ring becomes the tile
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
  if constexpr (SPLIT) {
    float *out = splitp + ((size_t)by * M + m0) * ldp + c0;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int f = 0; f < NTW; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = mrow0 + i * 16 + 4 * g + v;
          if (m < Mb) out[(size_t)m * ldp + (f * WN + wn) * 16 + r] = acc[i][f][v];
        }
    return;
  }
  float(*tile)[LDT] = reinterpret_cast<float(*)[LDT]>(smem);
#pragma unroll
  for (int f0 = 0; f0 < NTW; f0 += FP) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int f = f0; f < f0 + FP && f < NTW; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          tile[mrow0 + i * 16 + 4 * g + v][((f - f0) * WN + wn) * 16 + r] = acc[i][f][v];
    __syncthreads();
    epi.finish(&tile[0][0], LDT, Mb, c0 + f0 * WN * 16, 16 * WN * min(FP, NTW - f0), typename Epi::Pre{});
    if constexpr (HasBlock<Epi>::value) epi.embed = nullptr;  // its rows are copied by the first pass
  }
}

// split-K slices the reductions sum (k_splitk_finish, k_resid_rows)
constexpr int kMaxSlices = 8;

// Tile shapes of the many-row GEMMs and what a 64-wide K chunk of one tile
// takes (ns, 32 to 64 workgroups, K 12288).  A launch takes the shape whose
// rounds of workgroups cost least; K may be split over as many workgroups per
// tile (at most kMaxSlices) as slices of its padded columns fit in `floats`,
// where the caller sums the slices, which costs a write and a read of each.
// The first shapes are for up to 160 rows only: one row block holds them all,
// so that every weight is read once, and a narrow one spreads few columns over
// the chip.  Measured with one workgroup per CU: 147 rows x 4096 columns,
// K 12288 in 8 slices 28 us with 160 x 128 against 32 with 256 x 128; the K/V
// rows of seven layers (2048 columns each, K 4096) 38 us with 160 x 64 against
// 46 with two row blocks of 128 x 128.
enum TileShape {
  kTile64x64 = 0, kTile96x64, kTile128x64, kTile160x64, kTile64x128, kTile96x128, kTile160x128,
  kTile128x128, kTile128x192, kTile128x256, kTile256x224, kTile256x256, kTileShapes
};
constexpr int kTileFirstMany = kTile128x128;  // the shapes before serve as many rows as they are high
struct TilePick {
  int shape, ks;
};
constexpr int kTileM[kTileShapes] = {64, 96, 128, 160, 64, 96, 160, 128, 128, 128, 256, 256};
constexpr int kTileN[kTileShapes] = {64, 64, 64, 64, 128, 128, 128, 128, 192, 256, 224, 256};
constexpr int kTileNs[kTileShapes] = {320, 385, 436, 517, 480, 577, 676, 615, 750, 830, 1180, 1240};
// columns of a slice: whole tiles
static int tile_ld(int shape, int ncols) {
  return (ncols + kTileN[shape] - 1) / kTileN[shape] * kTileN[shape];
}
static TilePick pick_tile(int M, int ncols, int K, int groups, size_t floats) {
  const long nch = K / 64;
  const double wbytes = 2.0 * groups * ncols * K;
  TilePick best{kTile128x128, 1};
  double cost = 1e30;
  for (int t = M <= kGemmMaxRows ? 0 : kTileFirstMany; t < kTileShapes; ++t) {
    if (t < kTileFirstMany && M > kTileM[t]) continue;
    const size_t slice = (size_t)M * tile_ld(t, ncols);
    for (int ks = 1; ks <= kMaxSlices; ++ks) {
      if (ks > 1 && (nch / ks < 8 || ks * slice > floats)) break;  // at least 8 chunks of K per slice
      const long wgs = (long)((M + kTileM[t] - 1) / kTileM[t]) * groups * ((ncols + kTileN[t] - 1) / kTileN[t]) * ks;
      const double rounds = (double)((wgs + 255) / 256);
      // ns: a full chip runs at about 1 / 1.2 of the rate above, the weights
      // stream at 4.8 TB/s at most, a round fills and drains its ring and
      // writes its tile (about 6 us), and slices move at about 4 TB/s
      double c = rounds * (double)((nch + ks - 1) / ks) * kTileNs[t] * 1.2;
      c = (c > wbytes / 4800 ? c : wbytes / 4800) + rounds * 6000.0;
      if (ks > 1) c += (double)ks * M * ncols * 8 / 4000.0;
      if (c < cost) {
        cost = c;
        best = {t, ks};
      }
    }
  }
  return best;
}

// Launch of k_gemm_tile over ncols virtual columns of M rows (and `groups`
// groups of them, TileKv's layers), grid z over the row blocks.  128 x 128
// tiles take a three-stage ring when the grid is about one workgroup per CU
// (96 KB of LDS), else two stages, which lets two workgroups share a CU (1024
// rows x 6144 columns, K 4096: 75 us with three stages, 59 with two).  FEW: the
// shapes of up to 160 rows are built for this epilogue.
template <class Epi, bool SPLIT, bool FEW>
static hipError_t launch_tile(const TilePick &p, const bf16_t *A, int lda, int M, int K, const Epi &e,
                              int groups, float *sp, int ldp, hipStream_t s) {
  const int nb = (M + kTileM[p.shape] - 1) / kTileM[p.shape];  // row blocks per group
  const dim3 grid((e.nvcols + kTileN[p.shape] - 1) / kTileN[p.shape], p.ks, nb * groups);
#define FE_TILE(RT, NTW, WM, WN, S)                                                             \
  hipLaunchKernelGGL((k_gemm_tile<RT, NTW, WM, WN, S, Epi, SPLIT>), grid, dim3(512), 0, s, A,   \
                     lda, kDenseRows, M, K, e, sp, ldp, nb)
  if constexpr (FEW) {
    switch (p.shape) {
      case kTile64x64: FE_TILE(2, 1, 2, 4, 4); break;
      case kTile96x64: FE_TILE(3, 1, 2, 4, 4); break;
      case kTile128x64: FE_TILE(4, 1, 2, 4, 4); break;
      case kTile160x64: FE_TILE(5, 1, 2, 4, 4); break;
      case kTile64x128: FE_TILE(2, 2, 2, 4, 4); break;
      case kTile96x128: FE_TILE(3, 2, 2, 4, 4); break;
      case kTile160x128: FE_TILE(5, 2, 2, 4, 4); break;
      default: break;
    }
    if (p.shape < kTileFirstMany) return hipGetLastError();
  }
  switch (p.shape) {
    case kTile128x128:
      if ((long)grid.x * grid.y * grid.z <= 288) FE_TILE(4, 2, 2, 4, 3);
      else FE_TILE(4, 2, 2, 4, 2);
      break;
    case kTile128x192: FE_TILE(4, 3, 2, 4, 3); break;
    case kTile128x256: FE_TILE(4, 4, 2, 4, 3); break;
    case kTile256x224: FE_TILE(4, 7, 4, 2, 2); break;
    case kTile256x256: FE_TILE(8, 4, 2, 4, 2); break;
    default: return hipErrorInvalidValue;
  }
#undef FE_TILE
  return hipGetLastError();
}

// Split-K reduction: sums the ks partial slices of a 16-column span in a fixed
// order and hands the span to the epilogue, like k_gemm_mid would.  A thread
// takes 4 adjacent columns of a row and issues all of its slice loads before
// adding.
template <class Epi>
__global__ __launch_bounds__(256) void k_splitk_finish(const float *__restrict__ splitp, int ldp,
                                                       int ks, int M, Epi epi) {
  constexpr int BNR = 16, LDT = BNR + 1;
  __shared__ float tile[256 * LDT];
  const int c0 = blockIdx.x * BNR;
  const size_t slice = (size_t)M * ldp;
  for (int q = threadIdx.x; q < M * (BNR / 4); q += 256) {
    const int m = q / (BNR / 4), c = (q % (BNR / 4)) * 4;
    if constexpr (Epi::kQkv)
      if (!epi.row_used(m, c0)) continue;  // the epilogue never reads this row here
    const float *src = splitp + (size_t)m * ldp + c0 + c;
    f32x4 part[kMaxSlices];
#pragma unroll
    for (int y = 0; y < kMaxSlices; ++y)
      part[y] = y < ks ? *reinterpret_cast<const f32x4 *>(src + y * slice) : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 v = part[0];
#pragma unroll
    for (int y = 1; y < kMaxSlices; ++y) v += part[y];
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[m * LDT + c + e] = v[e];
  }
  __syncthreads();
  epi.finish(tile, LDT, M, c0, BNR, typename Epi::Pre{});
}

// Row finish of a residual GEMM whose rows feed only RMSNorms: one workgroup
// of 1024 threads per row sums the ks fp32 slices in slice order and adds the
// residual (the value EpiResid gives), stores it, and writes
// gamma_q * (v / rms(v)) in the storage type to every copy q (fixed-order
// reductions; four adjacent columns per thread, packed loads and stores).
// ks = 0: the GEMM's own epilogue stored v; it is read back.
template <typename T> __device__ __forceinline__ void store4(T *y, const f32x4 &v);
template <> __device__ __forceinline__ void store4<float>(float *y, const f32x4 &v) {
  *reinterpret_cast<f32x4 *>(y) = v;
}
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t *y, const f32x4 &v) {
  *reinterpret_cast<u32x2 *>(y) = u32x2{f2bf2(v.x, v.y), f2bf2(v.z, v.w)};
}
// Eight adjacent values: one 16-byte store (bf16) or two (fp32).
template <typename T> __device__ __forceinline__ void store8(T *y, const float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    *reinterpret_cast<u32x4 *>(y) =
        u32x4{f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7])};
  } else {
    *reinterpret_cast<f32x4 *>(y) = f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4 *>(y + 4) = f32x4{v[4], v[5], v[6], v[7]};
  }
}
__device__ __forceinline__ bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
// Eight adjacent floats of an epilogue tile row: two 16-byte LDS reads when
// the tile's row stride is a multiple of 4 floats (the caller's column is a
// multiple of 8), else eight scalar reads.
__device__ __forceinline__ void tile8(const float *t, int ldt, float (&v)[8]) {
  if ((ldt & 3) == 0) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(t), b = *reinterpret_cast<const f32x4 *>(t + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = t[j];
  }
}
template <typename T> __device__ __forceinline__ f32x4 load4(const T *g);
template <> __device__ __forceinline__ f32x4 load4<float>(const float *g) {
  return *reinterpret_cast<const f32x4 *>(g);
}
template <> __device__ __forceinline__ f32x4 load4<bf16_t>(const bf16_t *g) {
  const u32x2 w = *reinterpret_cast<const u32x2 *>(g);
  return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
               __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u)};
}

constexpr int kRowThreads = 1024;
template <typename T, int NV>
__global__ __launch_bounds__(kRowThreads) void k_resid_rows(const float *__restrict__ splitp,
                                                            int ldp, int ks, int M, int d,
                                                            const float *__restrict__ resid,
                                                            long ldr, float *__restrict__ out,
                                                            long ldo, GainCopies gc, float eps) {
  constexpr int NW = kRowThreads / 64;
  __shared__ float red[NW];
  const int m = blockIdx.x, tid = threadIdx.x;
  const size_t slice = (size_t)M * ldp;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 v[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int e = 4 * (tid + kRowThreads * u), ec = min(e, d - 4);
    if (ks > 0) {
      const float *src = splitp + (size_t)m * ldp + ec;
      f32x4 part[kMaxSlices];
#pragma unroll
      for (int y = 0; y < kMaxSlices; ++y) part[y] = y < ks ? *reinterpret_cast<const f32x4 *>(src + y * slice) : zero;
      f32x4 t = part[0];
#pragma unroll
      for (int y = 1; y < kMaxSlices; ++y) t += part[y];
      if (resid) t = *reinterpret_cast<const f32x4 *>(resid + (size_t)m * ldr + ec) + t;
      v[u] = t;
    } else {
      v[u] = *reinterpret_cast<const f32x4 *>(out + (size_t)m * ldo + ec);
    }
    if (e >= d) v[u] = zero;
  }
  float ss = 0.f;
#pragma unroll
  for (int u = 0; u < NV; ++u) ss += v[u].x * v[u].x + v[u].y * v[u].y + v[u].z * v[u].z + v[u].w * v[u].w;
  ss = group_sum<64>(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int e = 4 * (tid + kRowThreads * u);
    if (e >= d) continue;
    if (ks > 0) *reinterpret_cast<f32x4 *>(out + (size_t)m * ldo + e) = v[u];
    const f32x4 xn = v[u] * inv;
#pragma unroll
    for (int q = 0; q < kMaxLayers + 1; ++q) {
      if (q >= gc.n) break;
      const f32x4 g = load4((const T *)gc.gamma[q] + e);
      store4((T *)gc.dst[q] + (size_t)m * gc.ld[q] + e, g * xn);
    }
  }
}

// Row finish of a many-row storing GEMM (the fusion FC): sums the ks fp32
// slices of a row in slice order, stores the row in bf16 and copies the
// embedding row of its token next to it (NaN for a token outside [0, vocab)).
// One workgroup per row, eight adjacent columns per thread.
__global__ __launch_bounds__(256) void k_store_rows(const float *__restrict__ splitp, int ldp, int ks,
                                                    int M, int ncols, bf16_t *__restrict__ out,
                                                    int ldo, const bf16_t *__restrict__ embed,
                                                    const int32_t *__restrict__ tokens, int vocab,
                                                    bf16_t *__restrict__ gather_out, int ld_gather,
                                                    int d) {
  const int m = blockIdx.x;
  const size_t slice = (size_t)M * ldp;
  const int tok = embed ? tokens[m] : -1;
  for (int e = 8 * threadIdx.x; e < ncols; e += 8 * 256) {
    const float *src = splitp + (size_t)m * ldp + e;
    float v[8];
    tile8(src, 4, v);
    for (int y = 1; y < ks; ++y) {
      float w[8];
      tile8(src + y * slice, 4, w);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] += w[j];
    }
    store8<bf16_t>(out + (size_t)m * ldo + e, v);
  }
  if (!embed) return;
  const bool bad = tok < 0 || tok >= vocab;
  const u32x4 nan8 = {0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u, 0x7fc07fc0u};
  const u32x4 *src = reinterpret_cast<const u32x4 *>(embed + (size_t)(bad ? 0 : tok) * d);
  u32x4 *dst = reinterpret_cast<u32x4 *>(gather_out + (size_t)m * ld_gather);
  for (int e = threadIdx.x; e < d / 8; e += 256) dst[e] = bad ? nan8 : src[e];
}

// ---------------------------------------------------------------------------
// Epilogues.
// ---------------------------------------------------------------------------
// kMidNtw: 16-column tiles per workgroup on the batched-rows path (0 = chosen
// from the column count); kMidNtwMin: the smallest the epilogue accepts.
// prefetch() runs before the main loop and may load, into registers, what
// finish() needs for this thread's first output element (Pre::ok), so those
// loads ride along with the first weight chunk.
struct NoPre {
  bool ok = false;
};
template <typename T> struct EpiStore {
  static constexpr bool kRowStream = true, kSplitK = true, kQkv = false;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  const T *w;
  int ldw, nvcols;
  T *out;
  int ldo;
  const T *embed;
  const int32_t *tokens;
  int vocab;
  T *gather_out;
  int ld_gather, d, B;
  int bx = -1;
  __device__ const T *wrow(int c) const { return w + (size_t)c * ldw; }
  // a thread per element when that is one round, else per (row, 8 adjacent
  // columns) with one vector store where aligned
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    const int gpr = span >> 3;
    if (M * span <= (int)blockDim.x) {
      const int idx = threadIdx.x, m = idx / span, c = idx % span;
      if (idx < M * span && c0 + c < nvcols) out[(size_t)m * ldo + c0 + c] = Elt<T>::from_f(tile[m * ldt + c]);
    }
    for (int idx = threadIdx.x; M * span > (int)blockDim.x && idx < M * gpr; idx += blockDim.x) {
      const int m = idx / gpr, c = (idx % gpr) * 8;
      T *y = out + (size_t)m * ldo + c0 + c;
      const float *t = tile + m * ldt + c;
      if (c0 + c + 8 <= nvcols && aligned16(y)) {
        float v[8];
        tile8(t, ldt, v);
        store8<T>(y, v);
      } else {
        for (int j = 0; j < 8 && c0 + c + j < nvcols; ++j) y[j] = Elt<T>::from_f(t[j]);
      }
    }
    if (embed) {  // the embedding row e_{t+1} of every sequence, copied next to g_t
      constexpr int E = Elt<T>::kPer16B;
      for (int b = bx < 0 ? (int)blockIdx.x : bx; b < B; b += gridDim.x) {
        const int tok = tokens[b];
        T *dst = gather_out + (size_t)b * ld_gather;
        if (tok < 0 || tok >= vocab) {
          for (int e = threadIdx.x; e < d; e += blockDim.x) dst[e] = Elt<T>::from_f(__int_as_float(0x7fc00000));
          continue;
        }
        const u32x4 *src = reinterpret_cast<const u32x4 *>(embed + (size_t)tok * d);
        u32x4 *dv = reinterpret_cast<u32x4 *>(dst);
        for (int e = threadIdx.x; e < d / E; e += blockDim.x) dv[e] = src[e];
      }
    }
  }
};

template <typename T> struct EpiResid {
  static constexpr bool kRowStream = true, kSplitK = true, kQkv = false;
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  const T *w;
  int ldw, nvcols;
  float *out;
  long ldo;
  const float *resid;
  long ldr;
  float *ssq;  // optional per-(row, 16-column tile) sums of squares of the output
  int ssq_rs, ssq_off;
  GainCopies gc;
  struct Pre {  // raw values: converted where used, so no load is waited for early
    bool ok = false;
    float r = 0.f;
    T g[kMaxLayers + 1];
  };
  __device__ const T *wrow(int c) const { return w + (size_t)c * ldw; }
  // residual and gains of element idx = threadIdx.x, when every element has
  // its own thread (clamped in-bounds loads)
  __device__ Pre prefetch(int M, int c0, int span) const {
    Pre p;
    const int idx = threadIdx.x;
    if (M * span > (int)blockDim.x || idx >= M * span) return p;
    const int m = idx / span, cc = min(c0 + idx % span, nvcols - 1);
    p.ok = true;
    if (resid) p.r = resid[(size_t)m * ldr + cc];
    if (gc.n > 0) {
#pragma unroll
      for (int q = 0; q < kMaxLayers + 1; ++q)
        p.g[q] = ((const T *)gc.gamma[min(q, gc.n - 1)])[cc];
    }
    return p;
  }
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &pre) const {
    for (int idx = threadIdx.x; idx < M * span; idx += blockDim.x) {
      const int m = idx / span, c = idx % span;
      if (c0 + c >= nvcols) continue;
      const bool own = pre.ok && idx == (int)threadIdx.x;
      float v = tile[m * ldt + c];
      if (resid) v = (own ? pre.r : resid[(size_t)m * ldr + c0 + c]) + v;
      out[(size_t)m * ldo + c0 + c] = v;
      tile[m * ldt + c] = v;
      if (own) {
#pragma unroll
        for (int q = 0; q < kMaxLayers + 1; ++q)
          if (q < gc.n)
            ((T *)gc.dst[q])[(size_t)m * gc.ld[q] + c0 + c] = Elt<T>::from_f(Elt<T>::to_f(pre.g[q]) * v);
      } else {
        for (int q = 0; q < gc.n; ++q)
          ((T *)gc.dst[q])[(size_t)m * gc.ld[q] + c0 + c] =
              Elt<T>::from_f(Elt<T>::to_f(((const T *)gc.gamma[q])[c0 + c]) * v);
      }
    }
    if (ssq) {
      __syncthreads();
      const int ntile = nvcols / 16;
      for (int idx = threadIdx.x; idx < M * (span / 16); idx += blockDim.x) {
        const int m = idx / (span / 16), t = idx % (span / 16);
        if (c0 + 16 * t >= nvcols) continue;
        float sq = 0.f;
        for (int c = 16 * t; c < 16 * t + 16; ++c) sq += tile[m * ldt + c] * tile[m * ldt + c];
        ssq[((size_t)m * ssq_rs + ssq_off) * ntile + c0 / 16 + t] = sq;
      }
    }
  }
};

// Within a head, 16-column tile t holds rotary pairs 8t..8t+7: column n < 8 is
// dim 8t+n, column n >= 8 is its partner dim D/2 + 8t + (n-8).
__device__ __forceinline__ int rope_dim(int cc, int D) {
  const int t = cc >> 4, n = cc & 15;
  return ((n & 8) ? (D >> 1) : 0) + 8 * t + (n & 7);
}

template <typename T> struct EpiQkv {
  static constexpr bool kRowStream = true, kSplitK = true, kQkv = true;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  QkvArgs a;
  int nvcols;
  __device__ const T *wrow(int c) const {
    const int qd = a.Hq * a.D, kvd = a.Hkv * a.D;
    const T *base;
    int row;
    if (c < qd) {
      base = (const T *)a.wq;
      row = (c / a.D) * a.D + rope_dim(c % a.D, a.D);
    } else if (c < qd + kvd) {
      c -= qd;
      base = (const T *)a.wk;
      row = (c / a.D) * a.D + rope_dim(c % a.D, a.D);
    } else {
      base = (const T *)a.wv;
      row = c - qd - kvd;
    }
    return base + (size_t)row * a.d;
  }
  // only the last context row of a sequence carries a query
  __device__ bool row_used(int m, int c0) const {
    return c0 >= a.Hq * a.D || m % a.nctx == a.nctx - 1;
  }
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &p) const {
    if (M * span > (int)blockDim.x) {
      finish8(tile, ldt, M, c0, span);
      return;
    }
    const int qd = a.Hq * a.D, kvd = a.Hkv * a.D, D = a.D;
    for (int idx = threadIdx.x; idx < M * span; idx += blockDim.x) {
      const int m = idx / span, c = idx % span;
      int vc = c0 + c;
      if (vc >= nvcols) continue;
      const int b = m / a.nctx, t = m % a.nctx, j = a.j0 + t;
      const float val = tile[m * ldt + c];
      if (vc < qd + kvd) {
        const bool isq = vc < qd;
        if (isq && t != a.nctx - 1) continue;
        const int lc = isq ? vc : vc - qd;
        const int h = lc / D, cc = lc % D, dd = rope_dim(cc, D);
        if (!a.rotate) {  // attention rotates
          if (isq)
            a.q_out[((size_t)b * a.Hq + h) * D + dd] = val;
          else
            a.k_out[(((size_t)b * a.nctx + t) * a.Hkv + h) * D + dd] = val;
          continue;
        }
        const float pv = tile[m * ldt + (c ^ 8)];
        const int P = a.seqs.end(b) - a.seqs.start(b);
        const int pos = min(a.cascade ? P + j : P, a.rope_npos - 1);
        const int pm = 8 * (cc >> 4) + (cc & 7);
        const float c_ = a.rope[((size_t)pos * (D / 2) + pm) * 2];
        const float s_ = a.rope[((size_t)pos * (D / 2) + pm) * 2 + 1];
        const float o = (cc & 8) ? (val * c_ + pv * s_) : (val * c_ - pv * s_);
        if (isq)
          a.q_out[((size_t)b * a.Hq + h) * D + dd] = o;
        else
          a.k_out[(((size_t)b * a.nctx + t) * a.Hkv + h) * D + dd] = o;
      } else {
        vc -= qd + kvd;
        a.v_out[((size_t)b * a.nctx + t) * kvd + vc] = val;
      }
    }
  }
  // Many rows: a thread per (row, 8 adjacent virtual columns), which are 8
  // adjacent dimensions of one head's query or key (one rotary half, paired
  // with the 8 columns 8 away in the same 16-column tile) or of a value row.
  __device__ void finish8(const float *tile, int ldt, int M, int c0, int span) const {
    const int qd = a.Hq * a.D, kvd = a.Hkv * a.D, D = a.D;
    const int gpr = span >> 3;
    for (int idx = threadIdx.x; idx < M * gpr; idx += blockDim.x) {
      const int m = idx / gpr, c = (idx % gpr) * 8, vc = c0 + c;
      if (vc >= nvcols) continue;
      const int b = m / a.nctx, t = m % a.nctx;
      const float *tv = tile + m * ldt + c;
      float o[8];
      float *y;
      if (vc < qd + kvd) {
        const bool isq = vc < qd;
        if (isq && t != a.nctx - 1) continue;
        const int lc = isq ? vc : vc - qd;
        const int h = lc / D, cc = lc % D;
        if (!a.rotate) {  // attention rotates
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = tv[e];
        } else {
          const float *pt = tile + m * ldt + (c ^ 8);
          const int P = a.seqs.end(b) - a.seqs.start(b);
          const int pos = min(a.cascade ? P + a.j0 + t : P, a.rope_npos - 1);
          // rotary pair index 8 (cc >> 4) + e of dims rope_dim(cc, D) + e
          const float *rp = a.rope + ((size_t)pos * (D / 2) + 8 * (cc >> 4)) * 2;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float cs = rp[2 * e], sn = rp[2 * e + 1];
            o[e] = (cc & 8) ? (tv[e] * cs + pt[e] * sn) : (tv[e] * cs - pt[e] * sn);
          }
        }
        y = isq ? a.q_out + ((size_t)b * a.Hq + h) * D + rope_dim(cc, D)
                : a.k_out + (((size_t)b * a.nctx + t) * a.Hkv + h) * D + rope_dim(cc, D);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = tv[e];
        y = a.v_out + ((size_t)b * a.nctx + t) * kvd + (vc - qd - kvd);
      }
      if (aligned16(y)) {
        store8<float>(y, o);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = o[e];
      }
    }
  }
};

// Cache rows of verified positions: virtual columns [0, kvd) are the key
// rows of W_k (rotary pairs packed per 16-column tile as for EpiQkv), then
// the value rows; row m is rotated at positions[m] and stored in the storage
// type at cache row dst_rows[m].
template <typename T> struct EpiKvCache {
  static constexpr bool kRowStream = true, kSplitK = true, kQkv = false;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  KvCacheArgs a;
  int nvcols;  // 2 * Hkv * D
  __device__ const T *wrow(int c) const {
    const int kvd = a.Hkv * a.D;
    if (c < kvd) return (const T *)a.wk + (size_t)((c / a.D) * a.D + rope_dim(c % a.D, a.D)) * a.d;
    return (const T *)a.wv + (size_t)(c - kvd) * a.d;
  }
  // A thread per (row, 8 adjacent virtual columns): those are 8 adjacent
  // dimensions of one head's key (inside one rotary half, paired with the 8
  // columns 8 away in the same 16-column tile) or of a value row, so each
  // group is one vector store of the cache row piece.
  // With at most one element per thread the thread takes one element.
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    const int kvd = a.Hkv * a.D, D = a.D;
    const float qnan = __int_as_float(0x7fc00000);
    if (M * span <= (int)blockDim.x) {  // a single element
      const int m = threadIdx.x / span, c = threadIdx.x % span, vc = c0 + c;
      if (m >= M || vc >= nvcols) return;
      const long dst = a.dst_rows[m];
      if (dst < 0 || dst >= a.cache_rows) return;  // nowhere to write
      const int pos = a.positions[m];
      const bool bad = pos < 0 || pos >= a.pos_limit;
      const float *t = tile + m * ldt + c;
      if (vc < kvd) {
        const int h = vc / D, cc = vc % D;
        const int pc = min(max(pos, 0), a.pos_limit - 1);
        const float *rp = a.rope + ((size_t)pc * (D / 2) + 8 * (cc >> 4) + (cc & 7)) * 2;
        const float pv = tile[m * ldt + (c ^ 8)];
        const float v = bad ? qnan : ((cc & 8) ? (t[0] * rp[0] + pv * rp[1]) : (t[0] * rp[0] - pv * rp[1]));
        ((T *)a.k_cache)[(size_t)dst * kvd + (size_t)h * D + rope_dim(cc, D)] = Elt<T>::from_f(v);
      } else {
        ((T *)a.v_cache)[(size_t)dst * kvd + (vc - kvd)] = Elt<T>::from_f(bad ? qnan : t[0]);
      }
      return;
    }
    // U groups at a time, first their rows' positions and destinations, then
    // their rotary coefficients, then the stores: one chain of loads per U
    // groups where a group by itself paid it each time
    constexpr int U = 4;
    const int gpr = span >> 3, n = M * gpr;
    for (int i0 = threadIdx.x; i0 < n; i0 += U * blockDim.x) {
      int pos[U];
      long dst[U];
      f32x4 rp[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int m = min(i0 + u * (int)blockDim.x, n - 1) / gpr;
        pos[u] = a.positions[m];
        dst[u] = a.dst_rows[m];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // rotary pair index 8 (cc >> 4) + j of dims rope_dim(cc, D) + j (value
        // columns read the table too, and leave it)
        const int vc = c0 + (min(i0 + u * (int)blockDim.x, n - 1) % gpr) * 8, cc = vc % D;
        const int pc = min(max(pos[u], 0), a.pos_limit - 1);
        const float *r = a.rope + ((size_t)pc * (D / 2) + 8 * (cc >> 4)) * 2;
#pragma unroll
        for (int w = 0; w < 4; ++w) rp[u][w] = *reinterpret_cast<const f32x4 *>(r + 4 * w);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int idx = i0 + u * (int)blockDim.x;
        if (idx >= n) break;
        const int m = idx / gpr, c = (idx % gpr) * 8, vc = c0 + c;
        if (vc >= nvcols || dst[u] < 0 || dst[u] >= a.cache_rows) continue;  // nowhere to write
        const bool bad = pos[u] < 0 || pos[u] >= a.pos_limit;
        const float *t = tile + m * ldt + c;
        float o[8];
        T *y;
        if (vc < kvd) {
          const int h = vc / D, cc = vc % D;
          float tv[8], pv[8];
          tile8(t, ldt, tv);
          tile8(tile + m * ldt + (c ^ 8), ldt, pv);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const f32x4 w = rp[u][j >> 1];
            const float cs = (j & 1) ? w.z : w.x, sn = (j & 1) ? w.w : w.y;
            o[j] = bad ? qnan : ((cc & 8) ? (tv[j] * cs + pv[j] * sn) : (tv[j] * cs - pv[j] * sn));
          }
          y = (T *)a.k_cache + (size_t)dst[u] * kvd + (size_t)h * D + rope_dim(cc, D);
        } else {
          tile8(t, ldt, o);
#pragma unroll
          for (int j = 0; j < 8; ++j) o[j] = bad ? qnan : o[j];
          y = (T *)a.v_cache + (size_t)dst[u] * kvd + (vc - kvd);
        }
        if (aligned16(y)) {
          store8<T>(y, o);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) y[j] = Elt<T>::from_f(o[j]);
        }
      }
    }
  }
};

// Row-block slices of the cache update's GEMMs (bf16, many rows per launch).
// Fusion FC: EpiStore with the embedding gather of the block's own rows.
struct TileStore : EpiStore<bf16_t> {
  static constexpr bool kSliced = true;
  int lda;
  __device__ void slice(int z, int mrows, const bf16_t *&A, int &M) {
    const int m0 = z * mrows;
    A += (size_t)m0 * lda;
    M = min(mrows, M - m0);
    out += (size_t)m0 * ldo;
    if (embed) {
      tokens += m0;
      gather_out += (size_t)m0 * ld_gather;
      B = M;
    }
  }
};
// Input FC into fp32 rows (out = A W^T), or with `resid` a residual FC
// (out = resid + A W^T).
struct TileF32 {
  static constexpr bool kRowStream = true, kSplitK = false, kSliced = true;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  const bf16_t *w;
  int ldw, nvcols;
  float *out;
  long ldo;
  int lda;
  const float *resid = nullptr;
  long ldr = 0;
  __device__ const bf16_t *wrow(int c) const { return w + (size_t)c * ldw; }
  __device__ void slice(int z, int mrows, const bf16_t *&A, int &M) {
    const int m0 = z * mrows;
    A += (size_t)m0 * lda;
    M = min(mrows, M - m0);
    out += (size_t)m0 * ldo;
    if (resid) resid += (size_t)m0 * ldr;
  }
  // a thread per (row, 4 adjacent columns): vector loads and stores where aligned
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    const int gpr = span >> 2;
    for (int idx = threadIdx.x; idx < M * gpr; idx += blockDim.x) {
      const int m = idx / gpr, c = (idx % gpr) * 4;
      float *y = out + (size_t)m * ldo + c0 + c;
      const float *rr = resid ? resid + (size_t)m * ldr + c0 + c : nullptr;
      const float *t = tile + m * ldt + c;
      if (c0 + c + 4 <= nvcols && aligned16(y) && (!rr || aligned16(rr))) {
        f32x4 v = (ldt & 3) == 0 ? *reinterpret_cast<const f32x4 *>(t) : f32x4{t[0], t[1], t[2], t[3]};
        if (rr) v += *reinterpret_cast<const f32x4 *>(rr);
        *reinterpret_cast<f32x4 *>(y) = v;
      } else {
        for (int j = 0; j < 4 && c0 + c + j < nvcols; ++j) y[j] = t[j] + (rr ? rr[j] : 0.f);
      }
    }
  }
};
// Q/K/V projections of a prefill's rows in one launch (fp32, unrotated): the
// rows of W_q, W_k, W_v as virtual columns, each projection's rows dense.
// Four adjacent columns lie in one projection (head dims are multiples of 64).
struct TileQkv {
  static constexpr bool kRowStream = true, kSplitK = false, kSliced = true;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  const bf16_t *w[3];
  float *out[3];
  int end[3];  // virtual columns below: W_q, then W_k, then W_v
  int ldw, nvcols, lda;
  __device__ const bf16_t *wrow(int c) const {
    return c < end[0]   ? w[0] + (size_t)c * ldw
           : c < end[1] ? w[1] + (size_t)(c - end[0]) * ldw
                        : w[2] + (size_t)(c - end[1]) * ldw;
  }
  __device__ void slice(int z, int mrows, const bf16_t *&A, int &M) {
    const int m0 = z * mrows;
    A += (size_t)m0 * lda;
    M = min(mrows, M - m0);
    out[0] += (size_t)m0 * end[0];
    out[1] += (size_t)m0 * (end[1] - end[0]);
    out[2] += (size_t)m0 * (end[2] - end[1]);
  }
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    const int gpr = span >> 2;
    for (int idx = threadIdx.x; idx < M * gpr; idx += blockDim.x) {
      const int m = idx / gpr, c = (idx % gpr) * 4, vc = c0 + c;
      if (vc >= nvcols) continue;
      const float *t = tile + m * ldt + c;
      float *y = vc < end[0]   ? out[0] + (size_t)m * end[0] + vc
                 : vc < end[1] ? out[1] + (size_t)m * (end[1] - end[0]) + vc - end[0]
                               : out[2] + (size_t)m * (end[2] - end[1]) + vc - end[1];
      *reinterpret_cast<f32x4 *>(y) =
          (ldt & 3) == 0 ? *reinterpret_cast<const f32x4 *>(t) : f32x4{t[0], t[1], t[2], t[3]};
    }
  }
};
// K/V cache rows of every layer: slice z = layer * row blocks + block, A
// holds the layers' normalised rows a_layer_stride elements apart.  The layers
// differ only in their weights and caches; those pointers travel in the kernel
// arguments and a slice picks its layer's with an unrolled select (a uniform
// choice: no indexed copy of the arguments).
struct KvGroup {
  int nblocks, lda;
  long a_layer_stride;
  const void *wk[kMaxLayers], *wv[kMaxLayers];
  void *kc[kMaxLayers], *vc[kMaxLayers];
};
struct TileKv {
  static constexpr bool kRowStream = true, kSplitK = false, kSliced = true;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 1;
  EpiKvCache<bf16_t> cur;
  int nvcols;
  KvGroup g;
  __device__ void slice(int z, int mrows, const bf16_t *&A, int &M) {
    const int l = z / g.nblocks, m0 = (z % g.nblocks) * mrows;
#pragma unroll
    for (int q = 0; q < kMaxLayers; ++q)
      if (q == l) {
        cur.a.wk = g.wk[q];
        cur.a.wv = g.wv[q];
        cur.a.k_cache = g.kc[q];
        cur.a.v_cache = g.vc[q];
      }
    cur.a.positions += m0;
    cur.a.dst_rows += m0;
    A += l * g.a_layer_stride + (size_t)m0 * g.lda;
    M = min(mrows, M - m0);
  }
  __device__ const bf16_t *wrow(int c) const { return cur.wrow(c); }
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &p) const {
    cur.finish(tile, ldt, M, c0, span, p);
  }
};

template <typename T> struct EpiSwiglu {
  static constexpr bool kRowStream = true, kSplitK = false;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 0, kMidNtwMin = 2;  // gate/up tile pairs
  const T *wg, *wu;
  int ldw, I, nvcols;  // nvcols = 2*I
  T *out;
  int ldo;
  // virtual tile pair (2p, 2p+1) = gate rows and up rows 16p..16p+15
  __device__ const T *wrow(int c) const {
    const int p = c >> 5, f = (c >> 4) & 1, n = c & 15;
    return (f ? wu : wg) + (size_t)(p * 16 + n) * ldw;
  }
  // a thread per output when that is one round, else per (row, 8 adjacent
  // gate columns): 8 adjacent outputs, one vector store where aligned
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    const int half = span >> 1, gpr = span >> 4;
    if (M * half <= (int)blockDim.x) {
      const int idx = threadIdx.x, m = idx / half, q = idx % half;
      const int c = (q >> 4) * 32 + (q & 15);  // gate column inside the tile
      const int vc = c0 + c;
      if (idx < M * half && vc < nvcols) {
        const float gt = tile[m * ldt + c], up = tile[m * ldt + c + 16];
        const float s = gt / (1.f + expf(-gt)) * up;
        out[(size_t)m * ldo + (vc >> 5) * 16 + (vc & 15)] = Elt<T>::from_f(s);
      }
      return;
    }
    for (int idx = threadIdx.x; idx < M * gpr; idx += blockDim.x) {
      const int m = idx / gpr, q = (idx % gpr) * 8;
      const int c = (q >> 4) * 32 + (q & 15);  // first gate column inside the tile
      const int vc = c0 + c;
      if (vc >= nvcols) continue;
      const float *t = tile + m * ldt + c;
      float gt[8], up[8], s[8];
      tile8(t, ldt, gt);
      tile8(t + 16, ldt, up);
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] = gt[j] / (1.f + expf(-gt[j])) * up[j];
      T *y = out + (size_t)m * ldo + (vc >> 5) * 16 + (vc & 15);
      if (vc + 8 <= nvcols && aligned16(y)) {
        store8<T>(y, s);
      } else {
        for (int j = 0; j < 8 && vc + j < nvcols; ++j) y[j] = Elt<T>::from_f(s[j]);
      }
    }
  }
};

// Gate/up + SwiGLU over row blocks (the multi-position prefill's MLP).
struct TileSwiglu : EpiSwiglu<bf16_t> {
  static constexpr bool kSliced = true;
  int lda;
  __device__ void slice(int z, int mrows, const bf16_t *&A, int &M) {
    const int m0 = z * mrows;
    A += (size_t)m0 * lda;
    M = min(mrows, M - m0);
    out += (size_t)m0 * ldo;
  }
};

// Maximum / minimum over 16 lanes (one DPP row), in every lane of the row.
__device__ __forceinline__ uint32_t row16_max(uint32_t x) {
  auto d = [](uint32_t v, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  x = max(x, d(x, std::integral_constant<int, 0xB1>{}));
  x = max(x, d(x, std::integral_constant<int, 0x4E>{}));
  x = max(x, d(x, std::integral_constant<int, 0x141>{}));
  return max(x, d(x, std::integral_constant<int, 0x128>{}));
}

// Shared LM head: per (row, 64-column tile) max, sum of exp(z - max) and the
// top-k (largest key first, equal keys by lower draft id); logits optionally
// kept.  Sixteen lanes take a (row, tile), four adjacent columns each, so a wave
// does four at a time, whatever the row count: the logits leave as whole
// vectors, a generator block's four draws are a lane's four columns, and a
// selection round is one DPP maximum of 32-bit keys.  (A thread per row, as
// rows above 16 had it, left most of a workgroup idle while 64 or 128 columns
// went by one after the other: the 30-row LM head of 32000 x 4096 took 93 us,
// the 224-row one 111.)
template <typename T> struct EpiLm {
  static constexpr bool kRowStream = false, kSplitK = false;
  using Pre = NoPre;
  __device__ Pre prefetch(int, int, int) const { return {}; }
  static constexpr int kMidNtw = 4, kMidNtwMin = 4;  // 64-column tiles, as lmhead_tiles counts
  LmArgs a;
  int ldw, nvcols;
  __device__ const T *wrow(int c) const { return (const T *)a.w + (size_t)c * ldw; }

  // Selection key of tempered logit x: x, or with draws x + Gumbel(u) = x -
  // log(-log(u)) (sampling without replacement).  Ordered as 32-bit integers:
  // 0 is no candidate, 1 a NaN, the rest the order-preserving bits of the
  // float.  Up to 16 rows list -inf (a draw of u = 0) and NaN, after every
  // other key; above, neither is a candidate.
  __device__ void finish(float *tile, int ldt, int M, int c0, int span, const Pre &) const {
    // with more items than one round of the waves, two at a time: a round's
    // maxima are a chain, and the other item's fill its gaps
    if (M * (span >> 6) > (int)(blockDim.x >> 4)) finish_items<2>(tile, ldt, M, c0, span);
    else finish_items<1>(tile, ldt, M, c0, span);
  }
  template <int U>
  __device__ void finish_items(const float *tile, int ldt, int M, int c0, int span) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int l16 = lane & 15, base = lane & 48;
    const int nseg = span >> 6, items = M * nseg, ntile = (nvcols + 63) >> 6;
    const bool vec = aligned16(a.logits), gen = a.draws.so != nullptr, on = a.draws.on();
    const uint32_t nan_key = M <= 16 ? 1u : 0u;
    const uint32_t none = M <= 16 ? 0u : 0x007fffffu;  // a winner up to this key (-inf) is no candidate
    const uint64_t seed = gen ? a.draws.so[0] : 0, offset = gen ? a.draws.so[1] : 0;
    for (int i0 = 4 * U * wave; i0 < items; i0 += 4 * U * nw) {
      float v[U][4], mx[U], se[U];
      uint32_t key[U][4];
      bool live[U];
      size_t pb[U];
      int cs[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + 4 * u + (lane >> 4), it = min(i, items - 1), m = it / nseg, seg = it % nseg;
        cs[u] = c0 + 64 * seg;                                 // the tile's first column
        live[u] = i < items && cs[u] < nvcols;
        const bool ok = live[u] && cs[u] + 4 * l16 < nvcols;   // the vocabulary is a multiple of 16
        pb[u] = (size_t)m * ntile + (cs[u] >> 6);
        const float *t = tile + m * ldt + 64 * seg + 4 * l16;
        const size_t e0 = (size_t)m * nvcols + cs[u] + 4 * l16;
        if ((ldt & 3) == 0) {
          const f32x4 x = *reinterpret_cast<const f32x4 *>(t);
          v[u][0] = x.x; v[u][1] = x.y; v[u][2] = x.z; v[u][3] = x.w;
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) v[u][q] = t[q];
        }
        if (a.logits && ok) {
          if (vec) {
            *reinterpret_cast<f32x4 *>(a.logits + e0) = f32x4{v[u][0], v[u][1], v[u][2], v[u][3]};
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) a.logits[e0 + q] = v[u][q];
          }
        }
        mx[u] = -INFINITY;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          v[u][q] = ok ? v[u][q] * a.inv_temp : -INFINITY;  // statistics and candidates at temperature T
          mx[u] = fmaxf(mx[u], v[u][q]);
        }
        mx[u] = group_max<16>(mx[u]);
        se[u] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) se[u] += ok ? expf(v[u][q] - mx[u]) : 0.f;
        se[u] = group_sum<16>(se[u]);
        float n[4];
        if (gen) {
          philox_block(seed, offset, (uint64_t)e0 >> 2, n);  // columns 4 l16 .. + 3 of the row
        } else if (on) {
#pragma unroll
          for (int q = 0; q < 4; ++q) n[q] = ok ? a.draws.u[e0 + q] : 0.5f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float kf = on ? v[u][q] - logf(-logf(n[q])) : v[u][q];
          const uint32_t w = __float_as_uint(kf);
          key[u][q] = !ok ? 0u : kf != kf ? nan_key : (w & 0x80000000u) ? ~w : (w | 0x80000000u);
        }
      }
      uint32_t got[U];  // lane r: the r-th best key, its column and its z / T
      int gcol[U];
      float gz[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        got[u] = 0;
        gcol[u] = 0;
        gz[u] = -INFINITY;
      }
      for (int r = 0; r < a.topk; ++r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          uint32_t(&k)[4] = key[u];
          const uint32_t best = row16_max(max(max(k[0], k[1]), max(k[2], k[3])));
          // the lowest column that holds it (as 64 - column, so a maximum finds it)
          uint32_t inv = 0;
#pragma unroll
          for (int q = 3; q >= 0; --q) inv = k[q] == best ? 64u - 4 * l16 - q : inv;
          const int col = 64 - (int)row16_max(inv);
          if (on) {
            const int q = col & 3;
            const float z = __shfl(q == 0 ? v[u][0] : q == 1 ? v[u][1] : q == 2 ? v[u][2] : v[u][3],
                                   base + (col >> 2), 64);
            if (l16 == r) gz[u] = z;
          }
          if (l16 == r) {
            got[u] = best;
            gcol[u] = col;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) k[q] = col == 4 * l16 + q ? 0u : k[q];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!live[u]) continue;
        if (l16 == 0) {
          a.part_max[pb[u]] = mx[u];
          a.part_sum[pb[u]] = se[u];
        }
        if (l16 < a.topk) {
          const uint32_t g = got[u] > none ? got[u] : 0u;
          const float val = g == 1u ? __int_as_float(0x7fc00000)
                                    : __uint_as_float((g & 0x80000000u) ? (g & 0x7fffffffu) : ~g);
          a.cand_val[pb[u] * kMaxTopk + l16] = g ? val : -INFINITY;
          a.cand_idx[pb[u] * kMaxTopk + l16] = g ? cs[u] + gcol[u] : 0x7fffffff;
          if (on) a.cand_z[pb[u] * kMaxTopk + l16] = g ? gz[u] : -INFINITY;
        }
      }
    }
  }
};

// ---------------------------------------------------------------------------
// Dispatch.
// ---------------------------------------------------------------------------
// Split-K width of the up-to-32-row kernel.
template <int WKmax, int MT> struct SplitK {
  static constexpr int cap = 8;
  static constexpr int value = WKmax < cap ? WKmax : cap;
};

template <typename T, class Epi>
static hipError_t run_gemv(const T *A, int lda, const ARows &arows, int M, int K,
                           const Epi &epi, const NormA *na, int mr, size_t lds, hipStream_t s) {
  constexpr int W = 4 * (Epi::kMidNtwMin > 1 ? Epi::kMidNtwMin : 1);  // SPAN = 16 * kMidNtwMin
  constexpr int SPAN = 4 * W;
  const int grid = (epi.nvcols + SPAN - 1) / SPAN;
  const NormA n0 = na ? *na : NormA{nullptr, 0, 1, 0, 1, 1, 0.f};
#define FE_GEMV(MRV, NORMV)                                                                      \
  hipLaunchKernelGGL((k_gemv<T, MRV, W, NORMV, Epi>), dim3(grid), dim3(64 * W), lds, s, A, lda, arows, \
                     M, K, n0, epi)
#define FE_GEMV_M(NORMV)              \
  switch (mr) {                       \
    case 1: FE_GEMV(1, NORMV); break; \
    case 2: FE_GEMV(2, NORMV); break; \
    default: FE_GEMV(4, NORMV); break; \
  }
  if (na) FE_GEMV_M(true) else FE_GEMV_M(false)
#undef FE_GEMV_M
#undef FE_GEMV
  return hipGetLastError();
}

// Where a split-K GEMM left its fp32 slices when the caller finishes them
// itself (ks = 0: the GEMM was not split and its epilogue ran).
struct SplitOut {
  const float *p = nullptr;
  int ldp = 0, ks = 0;
};

// batched rows above this go to k_gemm_tile's split-K path when the epilogue
// allows (measured at batch 32: the Q/K/V GEMM from 32 rows, 15.7 us against
// 18.4 on k_gemm_mid; the 32-row residual GEMMs stay on k_gemm_mid, whose
// half-height tiles were 8 % faster there)
constexpr int kTileSplitMinRows = 32, kTileSplitMinRowsQkv = 16;

// split-K slices of the narrow batched-rows GEMMs (at most 128 rows): up to
// kSliceCap32 slices, about kSliceWgs workgroups
constexpr int kSliceCap32 = 8, kSliceWgs = 256;

// ring stages of the at-most-32-row configuration: four keep two workgroups
// per CU (measured at the 8B batch-32 shapes: 1962 us per pass, against 1992
// with six stages and 1996 with 64-row tiles)
constexpr int kHalfStages = 4;

template <typename T, int NT, int WKmax, int WN, class Epi>
static hipError_t run_gemm(const T *A, int lda, const ARows &arows, int M, int K, const Epi &epi,
                           const NormA *na, hipStream_t s, const SplitScratch *ss = nullptr,
                           SplitOut *so = nullptr) {
  if (so) *so = SplitOut{};
  constexpr int SPAN = WN * NT * 16;
  const int grid = (epi.nvcols + SPAN - 1) / SPAN;
  const int mt = (M + 15) / 16;
  const NormA n0 = na ? *na : NormA{nullptr, 0, 1, 0, 1, 1, 0.f};
  // up to 4 rows whose padded input rows fit the LDS budget: row streaming
  // (the LM head's per-row top-k is cheaper on the matrix-core tiles).  fp32
  // rows took the matrix-core tiles before: their launches are all latency,
  // and those load the epilogue's values only after the products (the tiny
  // drafter's 256- to 768-wide rows: 6.2 us a launch, 4.6 so).
  if constexpr (Epi::kRowStream) {
    constexpr int PE = 16 * Elt<T>::kPer16B;
    const int mr = M <= 1 ? 1 : M <= 2 ? 2 : 4;
    const size_t lds = (size_t)mr * ((K + PE - 1) / PE * PE) * sizeof(T);
    if (M <= 4 && lds <= (size_t)kGvMaxLds && K >= Elt<T>::kPer16B)
      return run_gemv<T>(A, lda, arows, M, K, epi, na, mr, lds, s);
  }
  if (na) {
    if (mt != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm<T, 1, NT, SplitK<WKmax, 1>::value, WN, true, Epi>), dim3(grid),
                       dim3(64 * SplitK<WKmax, 1>::value * WN), 0, s, A, lda, arows, M, K, n0, epi);
    return hipGetLastError();
  }
  // 17..32 rows over wide outputs (the batch-32 gate/up): the LDS-ring kernel
  // with column-split waves beats the per-wave staging; narrow outputs take
  // it too when their epilogue can follow a split-K reduction, else they
  // would leave it too few workgroups
  bool splittable = false;
  if constexpr (Epi::kSplitK) splittable = ss != nullptr && ss->p != nullptr;
  const bool ring_wide = mt == 2 && (epi.nvcols >= 64 * 256 || splittable);
  // 5..16 rows: k_gemm's 16-column workgroups are few, and when they don't fill
  // whole rounds of CUs, those with one more set the time (5120 columns: 320
  // workgroups on 256 CUs, 12 rows: 2.8 TB/s against 4.3 for 4096 columns).
  // Split-K slices spread the columns evenly for a finish launch of about 6 us,
  // which the lost share of the stream (at 4.3 TB/s) has to exceed.  Without
  // room for two slices (a workspace for at most 16 rows holds none) k_gemm stays.
  bool uneven = false;
  int ks = 1, ldp = 0;  // slices of the launches below: 128-column tiles
  if (splittable) {
    constexpr int KC = 8 * Elt<T>::kPer16B;
    const int gx = (epi.nvcols + 127) / 128, nchk = (K + KC - 1) / KC;
    // about one workgroup per CU (k_splitk_finish sums at most 8 slices); many
    // rows make each slice heavier and its partial sums larger: fewer slices
    ks = min(M > 128 ? 4 : kSliceCap32, max(1, kSliceWgs / gx));
    ks = min(ks, kMaxSlices);
    ks = min(ks, max(1, nchk / 4));  // a few chunks per slice for the ring
    ldp = gx * 128;
    if ((size_t)ks * M * ldp > ss->floats) ks = 1;
  }
  if (sizeof(T) == 2 && mt == 1 && ks > 1) {
    const double fill = (double)grid / ((grid + 255) / 256 * 256);
    uneven = 2.0 * epi.nvcols * K / 4.3e6 * (1.0 / fill - 1.0) > 6.0;
  }
  if (mt <= 2 && !ring_wide && !uneven) {
    if (mt <= 1)
      hipLaunchKernelGGL((k_gemm<T, 1, NT, SplitK<WKmax, 1>::value, WN, false, Epi>), dim3(grid),
                         dim3(64 * SplitK<WKmax, 1>::value * WN), 0, s, A, lda, arows, M, K, n0, epi);
    else
      hipLaunchKernelGGL((k_gemm<T, 2, NT, SplitK<WKmax, 2>::value, WN, false, Epi>), dim3(grid),
                         dim3(64 * SplitK<WKmax, 2>::value * WN), 0, s, A, lda, arows, M, K, n0, epi);
    return hipGetLastError();
  }
  // batched rows: all M rows per workgroup, columns split over the grid; the
  // waves split columns as well when the rows do not fill four row groups
  if (M > 256) return hipErrorInvalidValue;
  if constexpr (sizeof(T) == 2 && Epi::kSplitK) {
    // More than 32 rows (bf16, K a multiple of 64), when the epilogue can
    // follow a split-K reduction: k_gemm_tile's 256 x 128 tiles (128 x 128 up
    // to 128 rows; all rows in one block, so the weights are streamed once), K split so that the grid
    // is about one workgroup per CU (k_gemm_mid has only one column wave
    // here); the slices are summed, in a fixed order, by the finish launch.
    // The Q/K/V GEMM (6144 columns) aims at fewer slices: six cost more to
    // write and sum than they save (layers of 160-224 rows at batch 32: 33.5
    // us per launch with six, 25.3 with four, 30.3 on k_gemm_mid).
    if (M > (Epi::kQkv ? kTileSplitMinRowsQkv : kTileSplitMinRows) && K % 64 == 0 && ss != nullptr &&
        ss->p != nullptr) {
      const int gx = (epi.nvcols + 127) / 128;
      int ksb = ((Epi::kQkv ? 192 : 288) + gx - 1) / gx;
      ksb = min(ksb, kMaxSlices);
      ksb = max(1, min(ksb, (K / 64) / 8));  // at least 8 chunks of K per slice
      const int ldpb = gx * 128;
      if ((size_t)ksb * M * ldpb <= ss->floats) {
        if (M > 128)
          hipLaunchKernelGGL((k_gemm_tile<4, 4, 4, 2, 3, Epi, true>), dim3(gx, ksb, 1), dim3(512), 0, s,
                             A, lda, arows, M, K, epi, ss->p, ldpb, 1);
        else  // 128 x 128 tiles
          hipLaunchKernelGGL((k_gemm_tile<4, 2, 2, 4, 3, Epi, true>), dim3(gx, ksb, 1), dim3(512), 0, s,
                             A, lda, arows, M, K, epi, ss->p, ldpb, 1);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || so) {  // the caller sums the slices
          if (so) *so = SplitOut{ss->p, ldpb, ksb};
          return e;
        }
        hipLaunchKernelGGL((k_splitk_finish<Epi>), dim3((epi.nvcols + 15) / 16), dim3(256), 0, s,
                           (const float *)ss->p, ldpb, ksb, M, epi);
        return hipGetLastError();
      }
    }
  }
  const int wn = M <= 64 ? 4 : (M <= 128 ? 2 : 1);
  int tt = Epi::kMidNtw;  // 16-column tiles per workgroup
  if (tt == 0) {
    tt = 2;
    while (tt < 4 && (epi.nvcols + 32 * tt - 1) / (32 * tt) >= 192) tt *= 2;
  }
  if (tt < Epi::kMidNtwMin) tt = Epi::kMidNtwMin;
  if (tt < wn) tt = wn;  // a tile per column group at least
  if (tt < 2) tt = 2;    // weight slots split evenly over the waves
  const int ntw = tt / wn;
  // Narrow outputs whose epilogue allows it: 128-column tiles (a quarter of
  // the re-reading of A that 32-column tiles cost) and K split over enough
  // workgroups to cover the CUs; the fp32 slices are summed, in a fixed order,
  // by a second launch that runs the epilogue.
  float *sp = ks > 1 ? ss->p : nullptr;
#define FE_GEMM_MID_RT(NTWV, WNV, SV, RTV)                                                           \
  hipLaunchKernelGGL((k_gemm_mid<T, NTWV, WNV, SV, Epi, RTV>),                                      \
                     dim3((epi.nvcols + 16 * NTWV * WNV - 1) / (16 * NTWV * WNV), ks), dim3(256), 0,  \
                     s, A, lda, arows, M, K, epi, sp, ldp)
#define FE_GEMM_MID(NTWV, WNV, SV) FE_GEMM_MID_RT(NTWV, WNV, SV, 4)
  // at most 32 rows: two 16-row tiles per wave, so the ring carries no
  // duplicated rows of A, and the stages it frees go to a deeper ring
  const bool half = wn == 4 && M <= 32;
  if constexpr (Epi::kSplitK) {
    if (sp) {
      if (wn == 4 && half) FE_GEMM_MID_RT(2, 4, kHalfStages, 2);
      else if (wn == 4) FE_GEMM_MID(2, 4, 4);
      else if (wn == 2) FE_GEMM_MID(4, 2, 4);
      else FE_GEMM_MID(8, 1, 3);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess || so) {  // the caller sums the slices
        if (so) *so = SplitOut{sp, ldp, ks};
        return e;
      }
      hipLaunchKernelGGL((k_splitk_finish<Epi>), dim3((epi.nvcols + 15) / 16), dim3(256), 0, s,
                         (const float *)sp, ldp, ks, M, epi);
      return hipGetLastError();
    }
  }
  if (wn == 4 && half) {
    if (ntw >= 2) FE_GEMM_MID_RT(2, 4, kHalfStages, 2);
    else FE_GEMM_MID_RT(1, 4, kHalfStages, 2);
  } else if (wn == 4) {
    if (ntw >= 2) FE_GEMM_MID(2, 4, 4);
    else FE_GEMM_MID(1, 4, 4);
  } else if (wn == 2) {
    if (ntw >= 2) FE_GEMM_MID(2, 2, 4);
    else FE_GEMM_MID(1, 2, 4);
  } else {
    if (ntw >= 4) FE_GEMM_MID(4, 1, 2);  // the LM head's grid is wide: two workgroups per CU
    else FE_GEMM_MID(2, 1, 3);
  }
#undef FE_GEMM_MID
#undef FE_GEMM_MID_RT
  return hipGetLastError();
}

hipError_t gemm_store(int dt, const void *A, int lda, int M, int K, const void *W, int ncols,
                      void *out, int ldo, const void *embed, const int32_t *tokens, int vocab,
                      void *gather_out, int ld_gather, int d, int B, hipStream_t s,
                      const SplitScratch *ss) {
  if (dt) {
    EpiStore<bf16_t> e{(const bf16_t *)W, K, ncols, (bf16_t *)out, ldo, (const bf16_t *)embed,
                       tokens, vocab, (bf16_t *)gather_out, ld_gather, d, B};
    return run_gemm<bf16_t, 1, 8, 1>((const bf16_t *)A, lda, kDenseRows, M, K, e, nullptr, s, ss);
  }
  EpiStore<float> e{(const float *)W, K, ncols, (float *)out, ldo, (const float *)embed,
                    tokens, vocab, (float *)gather_out, ld_gather, d, B};
  return run_gemm<float, 1, 8, 1>((const float *)A, lda, kDenseRows, M, K, e, nullptr, s, ss);
}

// The row pass of a residual GEMM: sums its slices (so.ks > 0; else out already
// holds the rows), adds the residual, stores the rows and writes their
// normalised copies (none: the rows alone).
template <typename T>
static hipError_t resid_rows(const SplitOut &so, int M, int ncols, const float *resid, long ldr,
                             float *out, long ldo, const GainCopies &gains, float eps, hipStream_t s) {
  if (so.ks == 0 && gains.n == 0) return hipSuccess;
#define FE_RROWS(NVV)                                                                            \
  hipLaunchKernelGGL((k_resid_rows<T, NVV>), dim3(M), dim3(kRowThreads), 0, s, so.p, so.ldp,      \
                     so.ks, M, ncols, resid, ldr, out, ldo, gains, eps)
  if (ncols <= 4 * kRowThreads) FE_RROWS(1);
  else FE_RROWS(2);
#undef FE_RROWS
  return hipGetLastError();
}

template <typename T>
static hipError_t resid_norm_rows(const T *A, int lda, int M, int K, const T *W, int ncols,
                                  float *out, long ldo, const float *resid, long ldr,
                                  const GainCopies &gains, float eps, hipStream_t s,
                                  const SplitScratch *ss) {
  if (M <= 0) return hipSuccess;
  if (ncols > 8192 || ncols % 4) return hipErrorInvalidValue;
  EpiResid<T> e{W, K, ncols, out, ldo, resid, ldr, nullptr, 1, 0, GainCopies{}};
  SplitOut so;
  const hipError_t ge = run_gemm<T, 1, 8, 1>(A, lda, kDenseRows, M, K, e, nullptr, s, ss, &so);
  if (ge != hipSuccess) return ge;
  return resid_rows<T>(so, M, ncols, resid, ldr, out, ldo, gains, eps, s);
}

hipError_t gemm_resid(int dt, const void *A, int lda, int M, int K, const void *W, int ncols,
                      float *out, long ldo, const float *resid, long ldr, float *ssq, int ssq_rs,
                      int ssq_off, const GainCopies *gains, hipStream_t s, const SplitScratch *ss,
                      float norm_eps) {
  if (norm_eps >= 0.f && gains && gains->n > 0) {
    if (dt)
      return resid_norm_rows<bf16_t>((const bf16_t *)A, lda, M, K, (const bf16_t *)W, ncols, out,
                                     ldo, resid, ldr, *gains, norm_eps, s, ss);
    return resid_norm_rows<float>((const float *)A, lda, M, K, (const float *)W, ncols, out, ldo,
                                  resid, ldr, *gains, norm_eps, s, ss);
  }
  GainCopies gc{};
  if (gains) gc = *gains;
  if (dt) {
    EpiResid<bf16_t> e{(const bf16_t *)W, K, ncols, out, ldo, resid, ldr, ssq, ssq_rs, ssq_off, gc};
    return run_gemm<bf16_t, 1, 8, 1>((const bf16_t *)A, lda, kDenseRows, M, K, e, nullptr, s, ss);
  }
  EpiResid<float> e{(const float *)W, K, ncols, out, ldo, resid, ldr, ssq, ssq_rs, ssq_off, gc};
  return run_gemm<float, 1, 8, 1>((const float *)A, lda, kDenseRows, M, K, e, nullptr, s, ss);
}

hipError_t gemm_qkv(int dt, const void *A, int lda, const ARows &arows, int M, const QkvArgs &a,
                    const NormA *na, hipStream_t s, const SplitScratch *ss) {
  const int nv = (a.Hq + 2 * a.Hkv) * a.D;
  if (dt) {
    EpiQkv<bf16_t> e{a, nv};
    return run_gemm<bf16_t, 1, 4, 1>((const bf16_t *)A, lda, arows, M, a.d, e, na, s, ss);
  }
  EpiQkv<float> e{a, nv};
  return run_gemm<float, 1, 8, 1>((const float *)A, lda, arows, M, a.d, e, na, s, ss);
}

hipError_t gemm_kvcache(int dt, const void *A, int lda, int M, const KvCacheArgs &a,
                        hipStream_t s, const SplitScratch *ss) {
  if (M <= 0) return hipSuccess;
  const int nv = 2 * a.Hkv * a.D;
  if (dt) {
    EpiKvCache<bf16_t> e{a, nv};
    return run_gemm<bf16_t, 1, 4, 1>((const bf16_t *)A, lda, kDenseRows, M, a.d, e, nullptr, s, ss);
  }
  EpiKvCache<float> e{a, nv};
  return run_gemm<float, 1, 8, 1>((const float *)A, lda, kDenseRows, M, a.d, e, nullptr, s, ss);
}

// Many rows at once (bf16).  K a multiple of 64: k_gemm_tile in the shape
// pick_tile finds, K split into slices where a row kernel can sum them; else
// k_gemm_mid's 128 x 64 tiles.  grid z covers the row blocks (and layers).
constexpr int kTileNtw = 2, kTileWn = 2, kTileStages = 3, kTileRows = 64 * (4 / kTileWn),
              kTileCols = 16 * kTileNtw * kTileWn;

template <class Epi>
static hipError_t rows_unsplit(const bf16_t *A, int lda, int M, int K, const Epi &e, hipStream_t s) {
  if (K % 64 == 0)
    return launch_tile<Epi, false, false>(pick_tile(std::max(M, kGemmMaxRows + 1), e.nvcols, K, 1, 0), A,
                                          lda, M, K, e, 1, nullptr, 0, s);
  const dim3 grid((e.nvcols + kTileCols - 1) / kTileCols, 1, (M + kTileRows - 1) / kTileRows);
  hipLaunchKernelGGL((k_gemm_mid<bf16_t, kTileNtw, kTileWn, kTileStages, Epi>), grid, dim3(256), 0, s,
                     A, lda, kDenseRows, M, K, e, nullptr, 0);
  return hipGetLastError();
}
hipError_t gemm_store_rows(const void *A, int lda, int M, int K, const void *W, int ncols, void *out,
                           int ldo, const void *embed, const int32_t *tokens, int vocab,
                           void *gather_out, int ld_gather, int d, hipStream_t s,
                           const SplitScratch *ss) {
  if (M <= 0) return hipSuccess;
  TileStore e;
  static_cast<EpiStore<bf16_t> &>(e) = EpiStore<bf16_t>{(const bf16_t *)W, K, ncols, (bf16_t *)out,
                                                        ldo, (const bf16_t *)embed, tokens, vocab,
                                                        (bf16_t *)gather_out, ld_gather, d, M};
  e.lda = lda;
  if (K % 64 == 0 && ncols % 8 == 0 && ss && ss->p) {
    const TilePick p = pick_tile(M, ncols, K, 1, ss->floats);
    const int ldp = tile_ld(p.shape, ncols);
    if (p.ks > 1 || (M <= kGemmMaxRows && (size_t)M * ldp <= ss->floats)) {
      const hipError_t err = launch_tile<EpiStore<bf16_t>, true, true>(p, (const bf16_t *)A, lda, M, K, e, 1,
                                                                 ss->p, ldp, s);
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(k_store_rows, dim3(M), dim3(256), 0, s, (const float *)ss->p, ldp, p.ks, M,
                         ncols, (bf16_t *)out, ldo, (const bf16_t *)embed, tokens, vocab,
                         (bf16_t *)gather_out, ld_gather, d);
      return hipGetLastError();
    }
  }
  return rows_unsplit((const bf16_t *)A, lda, M, K, e, s);
}

hipError_t gemm_swiglu_rows(const void *A, int lda, int M, int K, const void *w_gate,
                            const void *w_up, int I, void *out, int ldo, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  TileSwiglu e;
  static_cast<EpiSwiglu<bf16_t> &>(e) = EpiSwiglu<bf16_t>{(const bf16_t *)w_gate, (const bf16_t *)w_up,
                                                          K, I, 2 * I, (bf16_t *)out, ldo};
  e.lda = lda;
  return rows_unsplit((const bf16_t *)A, lda, M, K, e, s);
}

hipError_t gemm_resid_rows(const void *A, int lda, int M, int K, const void *W, int ncols, float *out,
                           long ldo, hipStream_t s, const float *resid, long ldr,
                           const GainCopies &norms, float eps, const SplitScratch *ss) {
  if (M <= 0) return hipSuccess;
  if (ncols > 8192 || ncols % 4) return hipErrorInvalidValue;
  SplitOut so;
  TilePick p{kTile128x128, 1};
  const size_t floats = ss && ss->p ? ss->floats : 0;
  if (K % 64 == 0) p = pick_tile(M, ncols, K, 1, floats);
  if (p.ks > 1 || (K % 64 == 0 && M <= kGemmMaxRows && (size_t)M * tile_ld(p.shape, ncols) <= floats)) {
    const EpiResid<bf16_t> e{(const bf16_t *)W, K, ncols, out, ldo, resid, ldr, nullptr, 1, 0, GainCopies{}};
    so = SplitOut{ss->p, tile_ld(p.shape, ncols), p.ks};
    const hipError_t err = launch_tile<EpiResid<bf16_t>, true, true>(p, (const bf16_t *)A, lda, M, K, e, 1,
                                                               ss->p, so.ldp, s);
    if (err != hipSuccess) return err;
  } else {
    TileF32 e{(const bf16_t *)W, K, ncols, out, ldo, lda};
    e.resid = resid;
    e.ldr = ldr;
    const hipError_t err = rows_unsplit((const bf16_t *)A, lda, M, K, e, s);
    if (err != hipSuccess) return err;
  }
  return resid_rows<bf16_t>(so, M, ncols, resid, ldr, out, ldo, norms, eps, s);
}

hipError_t gemm_qkv_rows(const void *A, int lda, int M, int K, const void *wq, const void *wk,
                         const void *wv, int qd, int kvd, float *q, float *k, float *v,
                         hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const TileQkv e{{(const bf16_t *)wq, (const bf16_t *)wk, (const bf16_t *)wv}, {q, k, v},
                  {qd, qd + kvd, qd + 2 * kvd}, K, qd + 2 * kvd, lda};
  return rows_unsplit((const bf16_t *)A, lda, M, K, e, s);
}

hipError_t gemm_kv_rows(const void *A, int lda, long a_layer_stride, int M, int nlayers,
                        const KvCacheArgs *layers, const NormA *na, hipStream_t s) {
  if (M <= 0 || nlayers <= 0) return hipSuccess;
  if (nlayers > kMaxLayers || (na && M > 16)) return hipErrorInvalidValue;
  TileKv e{};
  e.cur = EpiKvCache<bf16_t>{layers[0], 2 * layers[0].Hkv * layers[0].D};
  e.nvcols = e.cur.nvcols;
  e.g.lda = lda;
  e.g.a_layer_stride = a_layer_stride;
  for (int l = 0; l < nlayers; ++l) {
    e.g.wk[l] = layers[l].wk;
    e.g.wv[l] = layers[l].wv;
    e.g.kc[l] = layers[l].k_cache;
    e.g.vc[l] = layers[l].v_cache;
  }
  if (na) {
    // up to 16 rows, A = gamma * x per layer and the rows' sums of squares:
    // 16-column workgroups with K split over their four waves, grid y = layer
    e.g.nblocks = 1;
    const dim3 grid((e.nvcols + 15) / 16, nlayers);
    hipLaunchKernelGGL((k_gemm<bf16_t, 1, 1, 4, 1, true, TileKv>), grid, dim3(256), 0, s,
                       (const bf16_t *)A, lda, kDenseRows, M, layers[0].d, *na, e);
    return hipGetLastError();
  }
  if (layers[0].d % 64 == 0) {
    const TilePick p = pick_tile(M, e.nvcols, layers[0].d, nlayers, 0);
    e.g.nblocks = (M + kTileM[p.shape] - 1) / kTileM[p.shape];
    return launch_tile<TileKv, false, true>(p, (const bf16_t *)A, lda, M, layers[0].d, e, nlayers, nullptr, 0, s);
  }
  e.g.nblocks = (M + kTileRows - 1) / kTileRows;
  const dim3 grid((e.nvcols + kTileCols - 1) / kTileCols, 1, e.g.nblocks * nlayers);
  hipLaunchKernelGGL((k_gemm_mid<bf16_t, kTileNtw, kTileWn, kTileStages, TileKv>), grid, dim3(256), 0,
                     s, (const bf16_t *)A, lda, kDenseRows, M, layers[0].d, e, nullptr, 0);
  return hipGetLastError();
}

hipError_t gemm_swiglu(int dt, const void *A, int lda, const ARows &arows, int M, int K,
                       const void *w_gate, const void *w_up, int I, void *s_out, int lds,
                       const NormA *na, hipStream_t s) {
  if (dt) {
    EpiSwiglu<bf16_t> e{(const bf16_t *)w_gate, (const bf16_t *)w_up, K, I, 2 * I,
                        (bf16_t *)s_out, lds};
    return run_gemm<bf16_t, 2, 4, 1>((const bf16_t *)A, lda, arows, M, K, e, na, s);
  }
  EpiSwiglu<float> e{(const float *)w_gate, (const float *)w_up, K, I, 2 * I, (float *)s_out, lds};
  return run_gemm<float, 2, 4, 1>((const float *)A, lda, arows, M, K, e, na, s);
}

// LM head: 64-column tiles, four waves of 16 weight rows each over all of K
// (bf16; 8B batch 1: 49.5 us against 51.7 us for 2 x 2 waves of 32 rows x
// half of K, and 55-88 us for the 8- and 16-wave shapes).
constexpr int kLmWN = 4, kLmNT = 1;
int lmhead_tiles(int V) { return (V + kLmWN * kLmNT * 16 - 1) / (kLmWN * kLmNT * 16); }

hipError_t gemm_lmhead(int dt, const void *A, int lda, const ARows &arows, int M, int K,
                       const LmArgs &a, const NormA *na, int *nwg_out, hipStream_t s) {
  *nwg_out = lmhead_tiles(a.V);
  if (dt && !na && M > 128 && M <= 256 && K % 64 == 0) {
    // many rows (batched drafting, B x N of them): every row in one 256 x 128
    // tile of k_gemm_tile, so the head is streamed once (two of lmhead_tiles'
    // tiles per workgroup)
    EpiLm<bf16_t> e{a, K, a.V};
    const int gx = (a.V + 127) / 128;
    hipLaunchKernelGGL((k_gemm_tile<4, 4, 4, 2, 3, EpiLm<bf16_t>>), dim3(gx), dim3(512), 0, s,
                       (const bf16_t *)A, lda, arows, M, K, e, nullptr, 0, 1);
    return hipGetLastError();
  }
  if (dt) {
    EpiLm<bf16_t> e{a, K, a.V};
    return run_gemm<bf16_t, kLmNT, 1, kLmWN>((const bf16_t *)A, lda, arows, M, K, e, na, s);
  }
  EpiLm<float> e{a, K, a.V};
  return run_gemm<float, kLmNT, 2, kLmWN>((const float *)A, lda, arows, M, K, e, na, s);
}

}  // namespace fe
