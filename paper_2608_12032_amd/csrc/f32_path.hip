// fp32 inputs: block masses (Sec. 3.1, Eq. (1)) and frozen-support attention
// (Sec. 4.2, Eq. (4)) on the fp32 matrix instructions (fp32 products, fp32
// accumulation; no input is rounded).
//
// Tiles.  A wave owns groups of M query rows (attention and normalisers: one or
// two groups of 16; masses: one of 32) and walks 32-key sub-tiles.  It computes
// S^T = K Q^T, so that a lane holds scores of ONE query of each group (column =
// lane % M) and the online softmax is in-lane plus an exchange between the lane
// groups (lane / M), and O^T = V^T P^T, whose B operand of k-step t is register t
// of the score tile as it stands:
//   score register t of lane group g  <->  key (t/4) * 4G + 4g + t%4,  G = 64/M.
// The contraction order over d is free, so lane group g takes
// d = 4 (G i + g) .. + 3 and one 16-byte load of a K row feeds four matrix
// instructions per row group; row m of O^T block b stands for
// d = 4 (16 (b / 4) + m) + b % 4, so a 16-byte load of V feeds four d blocks.
// K and V go from global memory straight to registers: a 32-key sub-tile is 32
// KiB for 8,192 matrix cycles (two groups, d = 128), 16 bytes per clock and CU
// (32 with one group), so staging in LDS would save nothing.  A sub-tile's loads
// form one stream, K then V, and run kLead loads ahead of the products that use
// them, across sub-tiles.  A row's arithmetic is the same in either group and with
// either number of them, so the number may follow from the size of the call
// without any effect on a row's bits.
//
// Split.  The waves of a workgroup share its rows and take the row's
// sub-tiles in turn; their softmax states (max, sum, O) are merged in a fixed
// order through LDS at the end; two waves per SIMD cover each other's softmax.
//
// Bound: the fp32 matrix rate (157 TFLOP/s).  Attention over full rows, d =
// 128: 123 TFLOP/s at N = 8,192 x 3 heads, 118 at 4,096 x 4, 100 at 4,437 x 4
// (the last round a fifth full), 33 at 512 x 4 (128 tiles of one round).  A thread
// per query row with plain fma and its keys in LDS, which this replaced, ran 7.7
// TFLOP/s at N = 4,437 x 4 (5.2 ms, now 0.40).  Two groups of 16 rows on 16x16x4
// instructions against one of 32 on 32x32x2, whose rows round differently from
// those of a 16-row tile: 2 % slower at d = 128 (1,090 / 1,072 us at 12 x 4,437),
// 4 % faster at d = 64 (590 / 614).
// The construction step's masses take one sweep over the keys (186 us at N =
// 4,437 x 4 heads and 15 us for their reduction; the calibration's two: 421).
//
// Masking and padding follow the bf16 kernels: keys >= N never enter a
// softmax, query rows >= N read Q as 0 and get O = 0 and lse = -inf, and so do
// rows whose key set is empty; col_idx entries outside [0, n_k) are ignored, a
// repeated entry counts once (the row's ids are flagged in LDS and listed in
// ascending order), and row bounds are clamped to [0, col_idx_len].
//
// Row sums.  The softmax normaliser is summed per lane and sub-tile in fp32
// and carried in an fp64 running sum (and merged in fp64).  Added one by one
// to an fp32 accumulator, the many small terms of far keys fall below half
// its ulp and are lost: over 131k keys that biases the sum low by ~2e-4.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace losa {

namespace {

constexpr int CK = 32;    // keys per sub-tile
constexpr int kLead = 8;  // loads in flight ahead of their use, per wave

// Shapes of a wave's groups of M query rows.  A sub-tile's operands arrive as a
// stream of KC chunks of K, then (M = 16) VN of V, 16 bytes a lane.
template <int D, int M>
struct F32Tile {
  static constexpr int G = 64 / M;             // lane groups
  static constexpr int SR = M * M / 64;        // score registers per M-key tile
  static constexpr int KT = CK / M;            // M-key tiles per sub-tile
  static constexpr int QI = D / (4 * G);       // 16-byte chunks of a row per lane
  static constexpr int DB = D / M;             // d blocks of O^T
  static constexpr int VP = DB / 4;            // V loads per score register
  static constexpr int KC = KT * QI;
  static constexpr int VN = KT * SR * VP;
  static_assert(KC % kLead == 0 && VN % kLead == 0, "the stream fills the ring evenly");
};

template <int M>
struct F32Acc;
template <>
struct F32Acc<32> {
  typedef f32x16_t type;
  static __device__ __forceinline__ type mfma(float a, float b, type c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct F32Acc<16> {
  typedef f32x4_t type;
  static __device__ __forceinline__ type mfma(float a, float b, type c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Key of score register t in lane group g, inside an M-key tile.
template <int M>
__device__ __forceinline__ int score_key(int t, int g) {
  return (t >> 2) * (256 / M) + 4 * g + (t & 3);
}

// Chunk c of the stream of the sub-tile that starts at key0: rows
// key0 + kt*M + lane%M of K (chunk i of the row), or a piece of V's row of one
// score register.
template <int D, int M>
__device__ __forceinline__ f32x4_t load_k(const float* K, int key0, int c, int lm, int g) {
  using T = F32Tile<D, M>;
  const int kt = c % T::KT, i = c / T::KT;
  return *reinterpret_cast<const f32x4_t*>(K + (size_t)(key0 + lm) * D + 4 * g + kt * M * D +
                                           4 * T::G * i);
}
template <int D, int M>
__device__ __forceinline__ f32x4_t load_v(const float* V, int key0, int c, int lm, int g) {
  using T = F32Tile<D, M>;
  const int t = c / T::VP % T::SR, kt = c / T::VP / T::SR;
  return *reinterpret_cast<const f32x4_t*>(V + (size_t)(key0 + 4 * g) * D + lm * 4 +
                                           (kt * M + score_key<M>(t, 0)) * D + c % T::VP * 4 * M);
}

// The query operand, scaled; padding rows (!valid) read as 0, so that their
// scores stay finite whatever the padding holds.
template <int D, int M>
__device__ __forceinline__ void load_q(f32x4_t* qr, const float* Q, int row, int g, bool valid,
                                       float scale_log2) {
  using T = F32Tile<D, M>;
  const float* p = Q + (size_t)row * D + 4 * g;
#pragma unroll
  for (int i = 0; i < T::QI; ++i) {
    const f32x4_t x = *reinterpret_cast<const f32x4_t*>(p + 4 * T::G * i);
#pragma unroll
    for (int e = 0; e < 4; ++e) qr[i][e] = valid ? x[e] * scale_log2 : 0.f;
  }
}

// Scores of a sub-tile in log2 units: chunk c of K, in ring[c % kLead], against
// the query operands of RG row groups (group r's at qr[r * QI], its scores at
// s[r * KT]; two accumulation chains each, so that no product waits for the one
// before it).  issue(c) refills the slot just used.  Keys at or beyond kvalid get
// -inf.
template <int D, int M, int RG, typename Issue>
__device__ __forceinline__ void scores(f32x4_t* ring, const f32x4_t* qr, int g, int kvalid,
                                       typename F32Acc<M>::type* s, Issue&& issue) {
  using T = F32Tile<D, M>;
  using A = F32Acc<M>;
  typename A::type odd[RG * T::KT];
#pragma unroll
  for (int x = 0; x < RG * T::KT; ++x) {
    s[x] = typename A::type{};
    odd[x] = typename A::type{};
  }
#pragma unroll
  for (int c = 0; c < T::KC; ++c) {
    const int kt = c % T::KT, i = c / T::KT;
    const f32x4_t a = ring[c % kLead];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int r = 0; r < RG; ++r) {
        typename A::type& x = (e & 1) == 0 ? s[r * T::KT + kt] : odd[r * T::KT + kt];
        x = A::mfma(a[e], qr[r * T::QI + i][e], x);
      }
    issue(c);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int x = 0; x < RG * T::KT; ++x) s[x] += odd[x];
  if (kvalid < CK) {
#pragma unroll
    for (int x = 0; x < RG * T::KT; ++x)
#pragma unroll
      for (int t = 0; t < T::SR; ++t)
        if (x % T::KT * M + score_key<M>(t, g) >= kvalid) s[x][t] = -INFINITY;
  }
}

template <int M>
__device__ __forceinline__ float group_max(float x) {
  x = max_with_partner(x);
  if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return x;
}
template <int M>
__device__ __forceinline__ double group_sum(double x) {
  x += __shfl_xor(x, 32);
  if constexpr (M == 16) x += __shfl_xor(x, 16);
  return x;
}

// Maximum of the sub-tile's scores of this lane's query.
template <int D, int M>
__device__ __forceinline__ float tile_max(const typename F32Acc<M>::type* s) {
  using T = F32Tile<D, M>;
  float mx = s[0][0];
#pragma unroll
  for (int kt = 0; kt < T::KT; ++kt)
#pragma unroll
    for (int t = 0; t < T::SR; ++t) mx = fmaxf(mx, s[kt][t]);
  return group_max<M>(mx);
}

// s <- 2^(s - m); returns this lane's sum.
template <int D, int M>
__device__ __forceinline__ float tile_exp(typename F32Acc<M>::type* s, float m) {
  using T = F32Tile<D, M>;
  float part = 0.f;
#pragma unroll
  for (int kt = 0; kt < T::KT; ++kt)
#pragma unroll
    for (int t = 0; t < T::SR; ++t) {
      s[kt][t] = fast_exp2(s[kt][t] - m);
      part += s[kt][t];
    }
  return part;
}

// The row's distinct valid key blocks, ascending, into list; returns their
// count.  flag and wcount are LDS scratch; n_k <= kSparseFwdMaxNk, which flag and
// list have room for.  All NT threads call it.
template <int NT>
__device__ int block_list(int n_k, const int32_t* __restrict__ row_ptr,
                          const int32_t* __restrict__ col_idx, int64_t col_len, int r,
                          uint8_t* flag, uint16_t* list, int* wcount) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int j = tid; j < n_k; j += NT) flag[j] = 0;
  __syncthreads();
  int64_t e0 = row_ptr[r], e1 = row_ptr[r + 1];
  e0 = e0 < 0 ? 0 : (e0 > col_len ? col_len : e0);
  e1 = e1 < e0 ? e0 : (e1 > col_len ? col_len : e1);
  for (int64_t e = e0 + tid; e < e1; e += NT) {
    const int j = col_idx[e];
    if (j >= 0 && j < n_k) flag[j] = 1;
  }
  __syncthreads();
  int nb = 0;
  for (int c0 = 0; c0 < n_k; c0 += NT) {
    const int j = c0 + tid;
    const bool f = (j < n_k) && flag[j] != 0;
    const uint64_t bal = __ballot(f);
    const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0));
    if (lane == 0) wcount[w] = __popcll(bal);
    __syncthreads();
    int before = 0, total = 0;
    for (int x = 0; x < NT / 64; ++x) {
      before += (x < w) ? wcount[x] : 0;
      total += wcount[x];
    }
    if (f) list[nb + before + below] = (uint16_t)j;
    nb += total;
    __syncthreads();
  }
  return nb;
}

constexpr int kF32Waves = 8;  // waves of a workgroup (key splits): two per SIMD

// Attention of 16 RG query rows over their query block's key blocks (bk_sub
// 32-key sub-tiles each).  PV: O and, if given, lse (natural log).  !PV: only
// the normaliser, in log2 units, to lse.  DENSE: every sub-tile that holds a valid
// key, in order and from no list, so that no number of key blocks is too large
// (the calibration takes any).
template <int D, int RG, bool PV, bool DENSE>
__global__ void __launch_bounds__(64 * kF32Waves) __attribute__((amdgpu_waves_per_eu(2)))
    attn_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                    const float* __restrict__ V, const int32_t* __restrict__ row_ptr,
                    const int32_t* __restrict__ col_idx, int64_t col_len, float* __restrict__ O,
                    float* __restrict__ lse, int tile0, int blk, int bk_sub, int n_k, int N,
                    int n_pad, float scale_log2) {
  constexpr int M = 16;
  constexpr int ROWS = M * RG;
  using T = F32Tile<D, M>;
  using A = F32Acc<M>;
  constexpr int NWV = kF32Waves;
  constexpr int NT = 64 * NWV;
  constexpr int LD = D + 4;  // floats of a row of a partial output in LDS
  __shared__ uint8_t flag[kSparseFwdMaxNk];
  __shared__ uint16_t list[kSparseFwdMaxNk];
  __shared__ int wcount[NWV];
  __shared__ float mpart[NWV * ROWS];
  __shared__ double lpart[NWV * ROWS];
  __shared__ __attribute__((aligned(16))) float opart[PV ? NWV * ROWS * LD : 4];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lm = lane % M, g = lane / M;
  const int tiles = n_pad / ROWS;  // per head
  const int x0 = tile0 + xcd_remap(blockIdx.x, gridDim.x);
  const int bh = x0 / tiles;
  const int row0 = (x0 - bh * tiles) * ROWS;
  const int r = bh * (n_pad / blk) + row0 / blk;
  const size_t head = (size_t)bh * n_pad * D;

  f32x4_t qr[RG * T::QI];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    const int qrow = row0 + rg * M + lm;
    load_q<D, M>(qr + rg * T::QI, Q + head, qrow, g, qrow < N, scale_log2);
  }
  const int bk = bk_sub * CK;
  int S;
  if constexpr (DENSE)
    S = (N + CK - 1) / CK;
  else
    S = block_list<NT>(n_k, row_ptr, col_idx, col_len, r, flag, list, wcount) * bk_sub;
  auto key_of = [&](int x) -> int {
    const int y = x < S ? x : S - 1;
    if constexpr (DENSE) return y * CK;
    const int j = y / bk_sub;
    return __builtin_amdgcn_readfirstlane((int)list[j]) * bk + (y - j * bk_sub) * CK;
  };

  float m[RG];
  double l[RG];
  typename A::type o[RG][T::DB];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    m[rg] = kNegBig;
    l[rg] = 0.0;
    if constexpr (PV) {
#pragma unroll
      for (int b = 0; b < T::DB; ++b) o[rg][b] = typename A::type{};
    }
  }
  constexpr int NC = T::KC + (PV ? T::VN : 0);  // chunks of a sub-tile
  const float* Kh = K + head;
  const float* Vh = V + head;
  f32x4_t ring[kLead];
  int key0 = 0;
  if (w < S) {
    key0 = key_of(w);
#pragma unroll
    for (int c = 0; c < kLead; ++c) ring[c] = load_k<D, M>(Kh, key0, c, lm, g);
  }
  for (int x = w; x < S; x += NWV) {
    const int next = key_of(x + NWV);  // past the end: the last sub-tile again
    // chunk c's slot takes chunk c + kLead of the stream
    auto issue = [&](int c) {
      const int n = c + kLead;
      if (n < T::KC)
        ring[c % kLead] = load_k<D, M>(Kh, key0, n, lm, g);
      else if (n < NC)
        ring[c % kLead] = load_v<D, M>(Vh, key0, n - T::KC, lm, g);
      else
        ring[c % kLead] = load_k<D, M>(Kh, next, n - NC, lm, g);
    };
    typename A::type s[RG * T::KT];
    scores<D, M, RG>(ring, qr, g, N - key0, s, issue);
    float mx[RG];
    bool raise = false;
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      mx[rg] = tile_max<D, M>(s + rg * T::KT);
      raise = raise || mx[rg] > m[rg];
    }
    if (__ballot(raise) != 0) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        const float m_new = fmaxf(m[rg], mx[rg]);
        const float alpha = fast_exp2(m[rg] - m_new);  // 1 where the max stays
        m[rg] = m_new;
        l[rg] *= (double)alpha;
        if constexpr (PV) {
#pragma unroll
          for (int b = 0; b < T::DB; ++b) o[rg][b] *= alpha;
        }
      }
    }
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) l[rg] += (double)tile_exp<D, M>(s + rg * T::KT, m[rg]);
    if constexpr (PV) {
#pragma unroll
      for (int c = 0; c < T::VN; ++c) {
        const int p = c % T::VP, t = c / T::VP % T::SR, kt = c / T::VP / T::SR;
        const f32x4_t a = ring[(T::KC + c) % kLead];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int rg = 0; rg < RG; ++rg)
            o[rg][p * 4 + e] = A::mfma(a[e], s[rg * T::KT + kt][t], o[rg][p * 4 + e]);
        issue(T::KC + c);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    key0 = next;
  }

  // merge the waves' states: the common max, then sums and outputs rescaled to
  // it, added in wave order
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    const int at = w * ROWS + rg * M + lm;
    const double lw = group_sum<M>(l[rg]);
    if (g == 0) {
      mpart[at] = m[rg];
      lpart[at] = lw;
    }
    if constexpr (PV) {
      // register t of d block b holds d = 4 (16 (b / 4) + row) + b % 4
#pragma unroll
      for (int t = 0; t < T::SR; ++t)
#pragma unroll
        for (int b = 0; b < T::DB; ++b)
          opart[at * LD + 4 * (b / 4 * M + score_key<M>(t, g)) + b % 4] = o[rg][b][t];
    }
  }
  __syncthreads();
  auto merged = [&](int row, float* wgt) -> double {  // sum of row `row`, weight of each wave
    float mm = kNegBig;
#pragma unroll
    for (int y = 0; y < NWV; ++y) mm = fmaxf(mm, mpart[y * ROWS + row]);
    double lt = 0.0;
#pragma unroll
    for (int y = 0; y < NWV; ++y) {
      wgt[y] = fast_exp2(mpart[y * ROWS + row] - mm);
      lt += lpart[y * ROWS + row] * (double)wgt[y];
    }
    wgt[NWV] = mm;
    return lt;
  };
  float wgt[NWV + 1];
  if (tid < ROWS && lse != nullptr) {
    const float lf = (float)merged(tid, wgt);
    const float l2 = wgt[NWV] + __log2f(lf);
    const bool ok = row0 + tid < N && lf > 0.f;
    lse[(size_t)bh * n_pad + row0 + tid] = PV ? (ok ? l2 * kLn2 : -INFINITY) : l2;
  }
  if constexpr (PV) {
    for (int idx = tid; idx < ROWS * D / 4; idx += NT) {
      const int row = idx / (D / 4), d4 = (idx % (D / 4)) * 4;
      const float lf = (float)merged(row, wgt);
      const float inv = (row0 + row < N && lf > 0.f) ? 1.0f / lf : 0.f;
      f32x4_t acc = f32x4_t{};
#pragma unroll
      for (int y = 0; y < NWV; ++y) {
        const f32x4_t p = *reinterpret_cast<const f32x4_t*>(opart + (y * ROWS + row) * LD + d4);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = fmaf(p[e], wgt[y], acc[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] *= inv;
      *reinterpret_cast<f32x4_t*>(O + head + (size_t)(row0 + row) * D + d4) = acc;
    }
  }
}

// Block masses of one query block (blockIdx.x) over a range of per_wg key
// blocks (blockIdx.y).  Four waves: BLK/32 of them own 32 query rows each, and
// with 64-row blocks two such pairs take the key blocks in turn.  lse2 (log2
// units) comes from attn_f32_kernel, or (OWN: the caller gives no buffer to
// hold it; one workgroup per query block) from a first sweep over the keys.
template <int D, int BLK, bool OWN>
__global__ void __launch_bounds__(256)
    mass_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                    const float* __restrict__ lse2_in, float* __restrict__ mass, int bk_sub,
                    int per_wg, int n_k, int N, int n_pad, float scale_log2) {
  constexpr int M = 32;
  constexpr int RW = BLK / M;   // row waves
  constexpr int KSP = 4 / RW;   // waves that share rows and split the keys
  using T = F32Tile<D, M>;
  using A = F32Acc<M>;
  __shared__ float mpart[4 * M];
  __shared__ double lpart[4 * M];
  __shared__ float part[4];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = w % RW, sp = w / RW;
  const int lm = lane % M, g = lane / M;
  const int n_q = n_pad / BLK;
  const int r = blockIdx.x;
  const int bh = r / n_q;
  const int i = r - bh * n_q;
  const size_t head = (size_t)bh * n_pad * D;
  const int rows_valid = min(BLK, N - i * BLK);
  const int bk = bk_sub * CK;
  const int j0 = blockIdx.y * per_wg, j1 = min(n_k, j0 + per_wg);
  float* mrow = mass + (size_t)r * n_k;
  if (rows_valid <= 0) {  // a query block made only of padding
    for (int j = j0 + tid; j < j1; j += 256) mrow[j] = 0.f;
    return;
  }
  const int qrow = i * BLK + rw * M + lm;
  const bool qvalid = qrow < N;
  f32x4_t qr[T::QI];
  load_q<D, M>(qr, Q + head, qrow, g, qvalid, scale_log2);
  const float* Kh = K + head;
  f32x4_t ring[kLead];
  typename A::type s[T::KT];
  // first chunks of the sub-tile at key0, and the refill while it is worked on
  // (its own later chunks, then the first of the one at `next`)
  auto lead = [&](int key0) {
#pragma unroll
    for (int c = 0; c < kLead; ++c) ring[c] = load_k<D, M>(Kh, key0, c, lm, g);
  };
  auto sub_scores = [&](int key0, int next) {
    scores<D, M, 1>(ring, qr, g, N - key0, s, [&](int c) {
      const int n = c + kLead;
      ring[c % kLead] = load_k<D, M>(Kh, n < T::KC ? key0 : next, n % T::KC, lm, g);
    });
  };

  float lse2;
  if constexpr (OWN) {
    float m = kNegBig;
    double l = 0.0;
    const int S = (N + CK - 1) / CK;
    if (sp < S) lead(sp * CK);
    for (int x = sp; x < S; x += KSP) {
      sub_scores(x * CK, (x + KSP < S ? x + KSP : x) * CK);
      const float m_new = fmaxf(m, tile_max<D, M>(s));
      l *= (double)fast_exp2(m - m_new);
      m = m_new;
      l += (double)tile_exp<D, M>(s, m);
    }
    l = group_sum<M>(l);
    if (g == 0) {
      mpart[w * M + lm] = m;
      lpart[w * M + lm] = l;
    }
    __syncthreads();
    float mm = kNegBig;
#pragma unroll
    for (int y = 0; y < KSP; ++y) mm = fmaxf(mm, mpart[(y * RW + rw) * M + lm]);
    double lt = 0.0;
#pragma unroll
    for (int y = 0; y < KSP; ++y)
      lt += lpart[(y * RW + rw) * M + lm] *
            (double)fast_exp2(mpart[(y * RW + rw) * M + lm] - mm);
    lse2 = mm + __log2f((float)lt);
  } else {
    lse2 = lse2_in[(size_t)bh * n_pad + qrow];
  }
  // padding rows (Q = 0, finite scores) contribute exp2(-inf) = 0 to every mass
  const float sub = qvalid ? lse2 : INFINITY;

  // this wave's key blocks: j0 + sp, j0 + sp + KSP, ...; the trip count is the
  // same for every wave (barriers inside)
  const float inv_rows = 1.0f / (float)rows_valid;
  const int trips = (j1 - j0 + KSP - 1) / KSP;
  auto sub_key = [&](int y) -> int {  // first key of this wave's y-th sub-tile
    const int c = y / bk_sub;
    return (j0 + sp + c * KSP) * bk + (y - c * bk_sub) * CK;
  };
  // (a key block at or past j1 is not this workgroup's: nothing is read; the
  // refill past the last sub-tile reads the current one again)
  const int mine = max(0, (j1 - j0 - sp + KSP - 1) / KSP) * bk_sub;  // sub-tiles of this wave
  if (mine > 0) lead(sub_key(0));
  for (int c = 0; c < trips; ++c) {
    const int j = j0 + sp + c * KSP;
    float acc = 0.f;
    for (int u = 0; u < bk_sub; ++u) {
      const int y = c * bk_sub + u;
      if (y >= mine || sub_key(y) >= N) continue;
      const int next = y + 1 < mine ? sub_key(y + 1) : 0;
      sub_scores(sub_key(y), next < N ? next : 0);
      acc += tile_exp<D, M>(s, sub);
    }
    acc = wave_sum(acc);
    if (lane == 0) part[w] = acc;
    __syncthreads();
    if (lane == 0 && rw == 0 && j < j1) {
      float tot = 0.f;
#pragma unroll
      for (int y = 0; y < RW; ++y) tot += part[sp * RW + y];
      mrow[j] = tot * inv_rows;
    }
    __syncthreads();
  }
}

// Block statistics of one query block over a range of key blocks, for query
// blocks i0 .. i0 + n_i - 1 of every head: for query q of these and key block j
// its largest score, stat[bh][j][0][q] (log2 units), and the sum of its
// probabilities against that maximum, stat[bh][j][1][q], carried across the
// block's 32-key sub-tiles in fp64.  (One number, log2(sum) + maximum, has
// no room for the sum's 24 bits beside the maximum's size.)  Waves and key blocks
// as in mass_f32_kernel.
template <int D, int BLK>
__global__ void __launch_bounds__(256)
    stat_f32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                    float* __restrict__ stat, int i0, int n_i, int bk_sub, int per_wg, int n_k,
                    int n_kb, int N, int n_pad, float scale_log2) {
  constexpr int M = 32;
  constexpr int RW = BLK / M;
  constexpr int KSP = 4 / RW;
  using T = F32Tile<D, M>;
  using A = F32Acc<M>;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = w % RW, sp = w / RW;
  const int lm = lane % M, g = lane / M;
  const int bh = blockIdx.x / n_i;
  const int i = blockIdx.x - bh * n_i;  // from i0
  const int bk = bk_sub * CK;
  const int j0 = blockIdx.y * per_wg + sp, j1 = min(n_kb, (int)(blockIdx.y + 1) * per_wg);
  if (j0 >= j1) return;
  const int qrow = (i0 + i) * BLK + rw * M + lm;
  const float* Kh = K + (size_t)bh * n_pad * D;
  f32x4_t qr[T::QI];
  load_q<D, M>(qr, Q + (size_t)bh * n_pad * D, qrow, g, qrow < N, scale_log2);
  f32x4_t ring[kLead];
#pragma unroll
  for (int c = 0; c < kLead; ++c) ring[c] = load_k<D, M>(Kh, j0 * bk, c, lm, g);
  for (int j = j0; j < j1; j += KSP) {
    // m: reference of the block's sum, the same in both lanes of a query
    float m = kNegBig;
    double l = 0.0;
    const int subs = min(bk_sub, (N - j * bk + CK - 1) / CK);  // those that hold a valid key
    for (int u = 0; u < subs; ++u) {
      const int key0 = j * bk + u * CK;
      const int next = u + 1 < subs ? key0 + CK : (j + KSP < j1 ? (j + KSP) * bk : key0);
      typename A::type s[T::KT];
      scores<D, M, 1>(ring, qr, g, N - key0, s, [&](int c) {
        const int n = c + kLead;
        ring[c % kLead] = load_k<D, M>(Kh, n < T::KC ? key0 : next, n % T::KC, lm, g);
      });
      const float m_new = fmaxf(m, tile_max<D, M>(s));
      l = l * (double)fast_exp2(m - m_new) + (double)tile_exp<D, M>(s, m_new);
      m = m_new;
    }
    const double sum = group_sum<M>(l);
    if (g == 0) {
      float* const at = stat + ((size_t)bh * n_k + j) * 2 * n_i * BLK + i * BLK + rw * M + lm;
      at[0] = m;
      at[n_i * BLK] = (float)sum;
    }
  }
}

// Masses of one query block from its block statistics: each query's maximum and
// normaliser over the n_kb key blocks (fp64 sums), then per key block the mean
// over the valid queries.  Blocks past n_kb hold no valid key.
template <int BLK>
__global__ void __launch_bounds__(256)
    mass_of_stat_f32_kernel(const float* __restrict__ stat, float* __restrict__ mass, int i0,
                            int n_i, int n_k, int n_kb, int N, int n_pad) {
  constexpr int PT = 256 / BLK;  // threads per query
  __shared__ float mx[256];
  __shared__ double sm[256];
  __shared__ float qmax[BLK], qinv[BLK];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int n_q = n_pad / BLK;
  const int bh = blockIdx.x / n_i;
  const int i = i0 + blockIdx.x - bh * n_i;
  const int row = n_i * BLK;  // floats of a row of statistics
  const float* base = stat + (size_t)bh * n_k * 2 * row + (i - i0) * BLK;
  const size_t step = 2 * (size_t)row;
  float* mrow = mass + ((size_t)bh * n_q + i) * n_k;
  const int rows_valid = min(BLK, N - i * BLK);
  if (rows_valid <= 0) {
    for (int j = t; j < n_k; j += 256) mrow[j] = 0.f;
    return;
  }
  const int q = t % BLK, part = t / BLK;
  float m = kNegBig;
  for (int j = part; j < n_kb; j += PT) m = fmaxf(m, base[j * step + q]);
  double l = 0.0;
  for (int j = part; j < n_kb; j += PT)
    l += (double)base[j * step + row + q] * (double)fast_exp2(base[j * step + q] - m);
  mx[t] = m;
  sm[t] = l;
  __syncthreads();
  if (t < BLK) {
    float mm = m;
#pragma unroll
    for (int y = 1; y < PT; ++y) mm = fmaxf(mm, mx[y * BLK + t]);
    double lt = 0.0;
#pragma unroll
    for (int y = 0; y < PT; ++y) lt += sm[y * BLK + t] * (double)fast_exp2(mx[y * BLK + t] - mm);
    qmax[t] = mm;
    qinv[t] = 1.0f / (float)lt;
  }
  __syncthreads();
  const float inv_rows = 1.0f / (float)rows_valid;
  for (int j = w; j < n_k; j += 4) {
    float acc = 0.f;
    if (j < n_kb) {
#pragma unroll
      for (int e = 0; e < BLK / 64; ++e) {
        const int x = lane + 64 * e;
        if (x < rows_valid)
          acc += base[j * step + row + x] * (fast_exp2(base[j * step + x] - qmax[x]) * qinv[x]);
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) mrow[j] = acc * inv_rows;
  }
}

// log2 normalisers -> natural logs, -inf on padding rows.
__global__ void __launch_bounds__(256)
    lse_natural_kernel(float* __restrict__ lse, int N, int n_pad, int64_t total) {
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (x < total) lse[x] = x % n_pad < N ? lse[x] * kLn2 : -INFINITY;
}

// Tile heights of a call with `tiles` 32-row tiles: how many of them run as such
// (two row groups a wave), the rest as twice as many 16-row tiles (one).  A
// row's keys are not split over workgroups, and 256 tiles fill the matrix cores
// of the CUs (where two 16-row tiles share one, at d = 64, each runs half as
// fast), so the time goes in rounds of 256 tiles; a round of 16-row tiles has half
// the work but the same K/V traffic.  Full rows of 32 64-key blocks, one round of
// 32-row against one of 16-row tiles: 78 / 45 us at d = 128, 43 / 25 us at d = 64.
// So at d = 128 whole rounds are 32 rows high, and what is left over, if it is 128
// tiles or fewer, one round of 16 rows (8 rounds and 64 tiles: 663 us, all 32 rows
// 688, all 16 rows 759).  At d = 64 such a call takes 16 rows throughout: the
// second launch costs more than the better rounds give, up to 16 rounds (2 rounds
// and 64 tiles: 108 us, mixed 111, all 32 rows 125; 16 and 64: 711, 721, 732).
// Scores only take one height for all (N = 4,437, 4 heads, d = 128: 421 us a
// calibration with 32 rows, 497 with 16; N = 4,096, one head: 118 / 103).
template <bool PV>
int64_t wide_tiles(int d, int64_t tiles) {
  const int64_t rest = tiles % 256;
  if (PV) return rest > 128 || rest == 0 ? tiles : (d == 64 ? 0 : tiles - rest);
  const int64_t r32 = (tiles + 255) / 256, r16 = (2 * tiles + 255) / 256;
  return 5 * r32 <= 4 * r16 ? tiles : 0;
}

template <int D, int RG, bool PV, bool DENSE>
hipError_t launch_attn(const void* q, const void* k, const void* v, int tile0, int64_t tiles,
                       int blk, int blk_k, int N, int n_pad, float scale, const int32_t* row_ptr,
                       const int32_t* col_idx, int64_t col_len, void* o, float* lse,
                       hipStream_t stream) {
  if (tiles == 0) return hipSuccess;
  hipLaunchKernelGGL((attn_f32_kernel<D, RG, PV, DENSE>), dim3((uint32_t)tiles), dim3(64 * kF32Waves), 0,
                     stream, static_cast<const float*>(q), static_cast<const float*>(k),
                     static_cast<const float*>(v), row_ptr, col_idx, col_len,
                     static_cast<float*>(o), lse, tile0, blk, blk_k / CK, n_pad / blk_k, N, n_pad,
                     scale * kLog2e);
  return hipGetLastError();
}

template <bool PV, bool DENSE>
hipError_t launch_attn_any(int d, int blk, int blk_k, const void* q, const void* k, const void* v,
                           int BH, int N, int n_pad, float scale, const int32_t* row_ptr,
                           const int32_t* col_idx, int64_t col_len, void* o, float* lse,
                           hipStream_t stream) {
  const int64_t tiles = (int64_t)BH * (n_pad / 32), wide = wide_tiles<PV>(d, tiles);
  const int rest0 = (int)(2 * wide);  // first 16-row tile
  hipError_t err = hipErrorInvalidValue;
#define LOSA_F32_ATTN(DD)                                                                         \
  if (d == DD) {                                                                                  \
    err = launch_attn<DD, 2, PV, DENSE>(q, k, v, 0, wide, blk, blk_k, N, n_pad, scale, row_ptr,   \
                                        col_idx, col_len, o, lse, stream);                        \
    if (err == hipSuccess)                                                                        \
      err = launch_attn<DD, 1, PV, DENSE>(q, k, v, rest0, 2 * (tiles - wide), blk, blk_k, N,      \
                                          n_pad, scale, row_ptr, col_idx, col_len, o, lse, stream); \
  }
  LOSA_F32_ATTN(64)
  LOSA_F32_ATTN(128)
#undef LOSA_F32_ATTN
  return err;
}

// Key blocks per workgroup of the kernels that split a query block's keys over
// workgroups: enough workgroups for four per CU, each with 256 keys at least.
int key_blocks_per_wg(int rows, int n_k, int blk_k) {
  const int want = rows < 1024 ? (1024 + rows - 1) / rows : 1;
  const int least = 256 / blk_k > 1 ? 256 / blk_k : 1;
  const int per_wg = (n_k + want - 1) / want;
  return per_wg < least ? least : per_wg;
}

template <int D, int BLK>
hipError_t launch_mass(const void* q, const void* k, const float* lse2, float* mass, int BH,
                       int blk_k, int N, int n_pad, float scale, hipStream_t stream) {
  const int rows = BH * (n_pad / BLK);
  const int n_k = n_pad / blk_k;
  const float* qf = static_cast<const float*>(q);
  const float* kf = static_cast<const float*>(k);
  if (lse2 == nullptr) {
    hipLaunchKernelGGL((mass_f32_kernel<D, BLK, true>), dim3(rows, 1), dim3(256), 0, stream, qf,
                       kf, nullptr, mass, blk_k / CK, n_k, n_k, N, n_pad, scale * kLog2e);
    return hipGetLastError();
  }
  const int per_wg = key_blocks_per_wg(rows, n_k, blk_k);
  hipLaunchKernelGGL((mass_f32_kernel<D, BLK, false>), dim3(rows, (n_k + per_wg - 1) / per_wg),
                     dim3(256), 0, stream, qf, kf, lse2, mass, blk_k / CK, per_wg, n_k, N, n_pad,
                     scale * kLog2e);
  return hipGetLastError();
}

// Masses in one sweep over the keys: block statistics into `stat`, which has
// room for `room` floats per query of the call, then their reduction.  They take 2
// n_k floats per query, so where that is more than there are, the query blocks go
// in parts (two at most: n_k <= room, and `part` is a whole number of blocks for
// every block shape).
template <int D, int BLK>
hipError_t launch_stat(const void* q, const void* k, float* stat, int room, float* mass, int BH,
                       int blk_k, int N, int n_pad, float scale, hipStream_t stream) {
  const int n_q = n_pad / BLK;
  const int n_k = n_pad / blk_k, n_kb = (N + blk_k - 1) / blk_k;
  const int part = (int)std::min<int64_t>(n_q, (int64_t)n_q * room / (2 * n_k));
  for (int i0 = 0; i0 < n_q; i0 += part) {
    const int n_i = std::min(part, n_q - i0), rows = BH * n_i;
    const int per_wg = key_blocks_per_wg(rows, n_kb, blk_k);
    hipLaunchKernelGGL((stat_f32_kernel<D, BLK>), dim3(rows, (n_kb + per_wg - 1) / per_wg),
                       dim3(256), 0, stream, static_cast<const float*>(q),
                       static_cast<const float*>(k), stat, i0, n_i, blk_k / CK, per_wg, n_k, n_kb,
                       N, n_pad, scale * kLog2e);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(mass_of_stat_f32_kernel<BLK>, dim3(rows), dim3(256), 0, stream, stat, mass,
                       i0, n_i, n_k, n_kb, N, n_pad);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

// Masses, given room for the log2 normalisers (one float per token; written
// here) or none (scratch == nullptr).
hipError_t masses(int d, int blk, int blk_k, const void* q, const void* k, int BH, int N,
                  int n_pad, float scale, float* mass, float* scratch, hipStream_t stream) {
  if (scratch != nullptr) {
    const hipError_t err =
        launch_attn_any<false, true>(d, blk, blk_k, q, k, nullptr, BH, N, n_pad, scale, nullptr, nullptr,
                               0, nullptr, scratch, stream);
    if (err != hipSuccess) return err;
  }
#define LOSA_F32_MASS(DD, BB)  \
  if (d == DD && blk == BB)    \
    return launch_mass<DD, BB>(q, k, scratch, mass, BH, blk_k, N, n_pad, scale, stream);
  LOSA_F32_MASS(64, 64)
  LOSA_F32_MASS(64, 128)
  LOSA_F32_MASS(128, 64)
  LOSA_F32_MASS(128, 128)
#undef LOSA_F32_MASS
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_sparse_fwd_f32(int d, int blk, int blk_k, const void* q, const void* k,
                                 const void* v, int B, int H, int N, int n_pad, float scale,
                                 const int32_t* row_ptr, const int32_t* col_idx, int64_t col_len,
                                 void* o, float* lse, hipStream_t stream) {
  return launch_attn_any<true, false>(d, blk, blk_k, q, k, v, B * H, N, n_pad, scale, row_ptr,
                                      col_idx, col_len, o, lse, stream);
}

hipError_t launch_calibrate_f32(int d, int blk, int blk_k, const void* q, const void* k, int B,
                                int H, int N, int n_pad, float scale, float* mass, float* lse,
                                hipStream_t stream) {
  // the caller's lse holds the log2 normalisers until the masses are formed
  hipError_t err = masses(d, blk, blk_k, q, k, B * H, N, n_pad, scale, mass, lse, stream);
  if (err != hipSuccess || lse == nullptr) return err;
  const int64_t total = (int64_t)B * H * n_pad;
  hipLaunchKernelGGL(lse_natural_kernel, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, stream, lse, N,
                     n_pad, total);
  return hipGetLastError();
}

hipError_t launch_construct_f32(int d, int blk, int blk_k, const void* q, const void* k,
                                const void* v, int B, int H, int N, int n_pad, float scale,
                                void* o, float* mass, float* lse, hipStream_t stream) {
  // O is written last: until then it holds the block statistics, two floats per
  // query and key block, of all query blocks or one half and then the other, where
  // there are d key blocks or fewer, and the log2 normalisers otherwise (the masses
  // then take a sweep of their own)
  // (over an input it can hold neither: the mass kernel then finds its own
  // normalisers)
  const size_t bytes = (size_t)B * H * n_pad * d * sizeof(float);
  float* const scratch =
      overlap(o, q, bytes) || overlap(o, k, bytes) || overlap(o, v, bytes) ? nullptr
                                                                           : static_cast<float*>(o);
  hipError_t err = hipErrorInvalidValue;
  if (scratch != nullptr && n_pad / blk_k <= d) {
#define LOSA_F32_STAT(DD, BB) \
  if (d == DD && blk == BB)   \
    err = launch_stat<DD, BB>(q, k, scratch, d, mass, B * H, blk_k, N, n_pad, scale, stream);
    LOSA_F32_STAT(64, 64)
    LOSA_F32_STAT(64, 128)
    LOSA_F32_STAT(128, 64)
    LOSA_F32_STAT(128, 128)
#undef LOSA_F32_STAT
  } else {
    err = masses(d, blk, blk_k, q, k, B * H, N, n_pad, scale, mass, scratch, stream);
  }
  if (err != hipSuccess) return err;
  return launch_attn_any<true, true>(d, blk, blk_k, q, k, v, B * H, N, n_pad, scale, nullptr,
                                     nullptr, 0, o, lse, stream);
}

}  // namespace losa
