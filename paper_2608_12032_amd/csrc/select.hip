// Shortest-prefix block selection (Sec. 4.1, Eq. (3)) and CSR emission.
//
// Three launches:
//   select_rows  one wave per row r = (b*H + h)*n_q + i, the row's masses in
//                its registers.  Masses are >= 0, so their float bits order
//                like the values; the order is decreasing mass, ties by the
//                smaller block index.  The cut is found without sorting the
//                row: a search from the highest bit finds the largest pattern
//                T whose blocks (bits >= T) weigh at least the target, and
//                once 64 blocks or fewer share T's bits so far, those alone
//                are put in order.  Blocks that agree in all bits are taken by
//                index.  The threshold rule weighs a block by its mass, the
//                fixed-ratio top-k rule (TOPK; the ablation of Sec. 5, Table
//                2) by 1 with target min(topk, blocks holding a real key).
//                tau >= 1 keeps every key block that holds a real key, and so
//                does a row that never reaches tau.  The kept blocks go to a
//                bit mask per row, and the mask's bits counted to the row's
//                count.
//   scan_counts  one workgroup: exclusive scan of the counts -> row_ptr.
//   compact_rows one wave per row: the flagged block ids, ascending, at
//                col_idx[row_ptr[r] ...].
//
// Sums.  What decides is the sum of integer weights, masses in units of 2^-56
// of the least power of two 2^-e above tau (a mass of 2^-e and more counts as
// 2^-e, which reaches tau): independent of the order and within n_k 2^-55 tau of
// the exact sum, whatever the size of tau.  A step of the search first adds fp32
// masses and turns to the integers only where that sum is within 2^-19 tau of
// tau.  Its rounding error is less than that by 2^-21 tau, far more than the
// integers truncate: what the fp32 sum says is reached or not, the integers say
// too, so the cut is always among the blocks in play.
//
// Bound: the search's compare, select and add per block and step, and reading
// the masses.  At 22,296 rows of 3,716 masses (331 MB): select_rows 163 us
// (2.0 TB/s), where a bitonic sort of each row's 4,096 keys in LDS took 2,314
// us of barrier steps; compact_rows 33 us (110 us from byte flags), scan_counts
// 7 us (29 us with one row per load).
#include <cmath>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace losa {

namespace {

constexpr int SEL_T = 256;
constexpr int SEL_ROWS = SEL_T / 64;  // rows per workgroup, one per wave

__device__ __forceinline__ uint32_t mass_bits(float m) {  // negative and NaN -> 0
  return m > 0.f ? __float_as_uint(m) : 0u;
}

// m 2^e in units of 2^-56, truncated: hi in units of 2^-30 and lo < 2^26.
__device__ __forceinline__ void split_mass(float m, int e, uint32_t* hi, uint32_t* lo) {
  const float x = __builtin_ldexpf(m, e + 30);
  *hi = (uint32_t)x;
  *lo = (uint32_t)(__builtin_amdgcn_fractf(x) * 0x1p26f);
}
__device__ __forceinline__ uint64_t mass_weight(uint32_t bits, int e) {
  uint32_t hi, lo;
  split_mass(fminf(__builtin_ldexpf(__uint_as_float(bits), e), 1.f), 0, &hi, &lo);
  return ((uint64_t)hi << 26) + lo;
}

// Sum over the wave, the same in every lane.
template <typename T>
__device__ __forceinline__ T wave_total(T v) {
  auto bits = [](T x) { return __builtin_bit_cast(int, x); };
  auto val = [](int x) { return __builtin_bit_cast(T, x); };
  v += val(__builtin_amdgcn_update_dpp(0, bits(v), 0x128, 0xf, 0xf, false));  // row_ror:8
  v += val(__builtin_amdgcn_update_dpp(0, bits(v), 0x124, 0xf, 0xf, false));
  v += val(__builtin_amdgcn_update_dpp(0, bits(v), 0x122, 0xf, 0xf, false));
  v += val(__builtin_amdgcn_update_dpp(0, bits(v), 0x121, 0xf, 0xf, false));
  auto r = __builtin_amdgcn_permlane16_swap(bits(v), bits(v), false, false);
  v = val(r[0]) + val(r[1]);
  r = __builtin_amdgcn_permlane32_swap(bits(v), bits(v), false, false);
  return val(r[0]) + val(r[1]);
}

// Maximum over the wave, the same in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  auto dpp = [](uint32_t x, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  v = max(v, dpp(v, std::integral_constant<int, 0x128>{}));  // row_ror:8
  v = max(v, dpp(v, std::integral_constant<int, 0x124>{}));
  v = max(v, dpp(v, std::integral_constant<int, 0x122>{}));
  v = max(v, dpp(v, std::integral_constant<int, 0x121>{}));
  auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max((uint32_t)r[0], (uint32_t)r[1]);
  r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __builtin_amdgcn_readfirstlane(max((uint32_t)r[0], (uint32_t)r[1]));
}

__device__ __forceinline__ uint64_t read_lane(uint64_t x, int y) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, y) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), y) << 32;
}
__device__ __forceinline__ int bits_below(uint64_t m, int lane) {
  return __popcll(m & ((1ull << lane) - 1ull));
}

// The same value, but opaque: the compiler would otherwise keep what one pass
// over the row's blocks derives from each of them (split masses, ballots) for
// the next pass, 64 times over, and spill.
__device__ __forceinline__ uint32_t fresh(uint32_t& x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Bytes of a row's bit mask: whole 64-bit words, or one byte for fewer than
// eight blocks (never more than one byte per block).
__host__ __device__ inline size_t mask_stride(int n_k) {
  return n_k < 8 ? 1 : (size_t)((n_k + 63) / 64) * 8;
}

// V: blocks per lane, j = lane + 64 u
template <int V, bool TOPK>
__global__ void __launch_bounds__(SEL_T) __attribute__((amdgpu_waves_per_eu(V < 64 ? 1 : (TOPK ? 3 : 4))))
    select_rows_kernel(const float* __restrict__ mass, int rows, int n_q, int n_k, int n_kv, int N,
                       int block_q, float tau, int e, int topk, int32_t* __restrict__ counts,
                       uint8_t* __restrict__ masks) {
  __shared__ uint64_t keys[SEL_ROWS][64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.x * SEL_ROWS + w;
  if (r >= rows) return;
  const bool empty = (r % n_q) * block_q >= N;  // a query block made only of padding
  bool all = empty || (!TOPK && tau >= 1.0f);   // keep the blocks holding a real key (none if empty)

  uint32_t bits[V];
  uint32_t cut = 0;  // kept: bits > cut, or equal and j <= cut_j
  int cut_j = -1;
  if (!all) {
    // (past the row's end the resource reads zero: a branch per load would
    // wait out each one's latency)
    const __amdgpu_buffer_rsrc_t mrs = make_rsrc(mass + (size_t)r * n_k, (uint32_t)n_k * 4);
#pragma unroll
    for (int u = 0; u < V; ++u)
      bits[u] = __builtin_amdgcn_raw_buffer_load_b32(mrs, 4 * lane, 256 * u, 0);
#pragma unroll
    for (int u = 0; u < V; ++u) bits[u] = mass_bits(__uint_as_float(bits[u]));
    const uint64_t target =
        TOPK ? (uint64_t)min(topk, n_kv) : mass_weight(__float_as_uint(tau), e);
    // (the lambdas are inlined in every place: called, they would take the row's
    // registers through memory, 970 us instead of 195 at the size above)
    // weight of the blocks with bits >= c, c > 0 (threshold rule: if it is
    // below 2^57; the high parts then add up to less than 2^32)
    auto weight_from = [&](uint32_t c) __attribute__((always_inline)) -> uint64_t {
      uint32_t hi = 0, lo = 0;
#pragma unroll
      for (int u = 0; u < V; ++u) {
        if constexpr (TOPK) {
          hi += bits[u] >= c;
        } else {
          uint32_t h, l;
          const uint32_t b = fresh(bits[u]);
          split_mass(b >= c ? __uint_as_float(b) : 0.f, e, &h, &l);
          hi += h;
          lo += l;
        }
      }
      if constexpr (TOPK) return wave_total(hi);
      return ((uint64_t)wave_total(hi) << 26) + ((uint64_t)wave_total(lo >> 16) << 16) +
             wave_total(lo & 0xffffu);
    };
    auto reached = [&](uint32_t c) __attribute__((always_inline)) -> bool {
      if constexpr (!TOPK) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < V; ++u) s[u & 3] += bits[u] >= c ? __uint_as_float(bits[u]) : 0.f;
        const float d = wave_total((s[0] + s[1]) + (s[2] + s[3])) - tau;
        // V/4 + 8 additions deep: within 2^-19 of the sum
        static_assert(V / 4 + 8 <= 1 << 5, "rounding error of the fp32 sum");
        if (!(fabsf(d) <= tau * 0x1p-19f)) return __builtin_amdgcn_readfirstlane(d > 0.f);
      }
      return weight_from(c) >= target;
    };
    // Bounds that settle a step without a pass over the blocks: nothing weighs
    // in at more than the heaviest mass, and the blocks below c weigh less than
    // n_k c together (the fp32 total is within 2^-17 of the exact one; a
    // mass over 1 counts as 1: then neither bound is used).
    uint32_t top = 0x7fffffffu;
    float spare = 0.f;  // weight that can be left out for certain, per block
    if constexpr (!TOPK) {
      float sum = 0.f;
      top = 0;
#pragma unroll
      for (int u = 0; u < V; ++u) {
        sum += __uint_as_float(bits[u]);
        top = max(top, bits[u]);
      }
      top = wave_max(top);
      sum = wave_total(sum);
      spare = top <= 0x3f800000u ? (sum * (1.f - 0x1p-16f) - tau) / (float)n_k : 0.f;
    }
    uint32_t T = 0;
    int shift = 31;      // T's bits from here up are settled
    // whether block u of this lane shares them (threshold rule: a block of
    // mass 0 cannot move the cut; top-k: it can, if there is such a block)
    auto shares = [&](int u) __attribute__((always_inline)) -> bool {
      const uint32_t lo = TOPK ? T : max(T, 1u);
      return fresh(bits[u]) - lo < T + (1u << shift) - lo && (!TOPK || lane < n_k - 64 * u);
    };
    int in_play = 0;     // blocks that share them
    do {
      const int stop = shift == 31 ? 18 : (shift == 18 ? 9 : 0);
      while (shift > stop) {
        --shift;
        const uint32_t c = T | 1u << shift;
        if (c > top) continue;
        if (__uint_as_float(c) < spare || reached(c)) T = c;
      }
      if (!TOPK && T == 0 && !reached(1)) {  // the row never reaches tau
        all = true;
        break;
      }
      in_play = 0;
#pragma unroll
      for (int u = 0; u < V; ++u)
        in_play += __popcll(__ballot(shares(u)));
    } while (in_play > 64 && shift > 0);

    if (!all) {
      const uint64_t base = weight_from(T + (1u << shift));  // heavier than those in play
      if (in_play <= 64) {
        // one block in play per lane, and the weight before it
        int at = 0;
        uint32_t id = lane;
#pragma unroll
        for (int u = 0; u < V; ++u) {
          const bool mine = shares(u);
          const uint64_t bal = __ballot(mine);
          if (mine)
            keys[w][at + bits_below(bal, lane)] =
                ((uint64_t)(~bits[u]) << 32) | (64 * u + fresh(id));
          at += __popcll(bal);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint64_t key = keys[w][lane < in_play ? lane : 0];
        const uint64_t own = TOPK ? 1 : mass_weight(~(uint32_t)(key >> 32), e);
        uint64_t before = base;
        for (int y = 0; y < in_play; ++y)
          before += read_lane(key, y) < key ? read_lane(own, y) : 0;
        const int at_cut = __builtin_ctzll(
            __ballot(lane < in_play && before < target && before + own >= target));
        const uint64_t cut_key = read_lane(key, at_cut);
        cut = ~(uint32_t)(cut_key >> 32);
        cut_j = (int)(uint32_t)cut_key;
      } else {
        // more than 64 blocks of mass T: the first of them by index
        const uint64_t each = TOPK ? 1 : mass_weight(T, e);
        int need = (int)((target - base + each - 1) / each);
        cut = T;
#pragma unroll
        for (int u = 0; u < V; ++u) {
          const uint64_t bal = __ballot(shares(u));
          const int n = __popcll(bal);
          if (need > 0 && need <= n)
            cut_j = 64 * u + __builtin_ctzll(__ballot(((bal >> lane) & 1) != 0 &&
                                                      bits_below(bal, lane) == need - 1));
          need -= n;
        }
      }
    }
  }

  uint64_t word = 0;  // lane u: word u of the row's mask
  int count = 0;      // its bits, so that the compaction writes as many ids as it has room for
#pragma unroll
  for (int u = 0; u < V; ++u) {
    const uint32_t b = all ? 0 : fresh(bits[u]);
    const bool kept = all ? !empty && lane < n_kv - 64 * u
                          : lane < n_k - 64 * u &&
                                (b > cut || (b == cut && lane <= cut_j - 64 * u));
    const uint64_t bal = __ballot(kept);
    if (lane == u) word = bal;
    count += __popcll(bal);
  }
  uint8_t* mask = masks + (size_t)r * mask_stride(n_k);
  if (lane < (n_k + 63) / 64) {
    if (n_k < 8)
      *mask = (uint8_t)word;
    else
      reinterpret_cast<uint64_t*>(mask)[lane] = word;
  }
  if (lane == 0) counts[r] = count;
}

constexpr int SCAN_T = 1024;

__global__ void __launch_bounds__(SCAN_T)
    scan_counts_kernel(const int32_t* __restrict__ counts, int rows, int32_t* __restrict__ row_ptr) {
  __shared__ int32_t wtot[2][SCAN_T / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  int32_t run = 0;
  int par = 0;
  for (int64_t r0 = 0; r0 < rows; r0 += 4 * SCAN_T, par ^= 1) {
    const int64_t r = r0 + 4 * t;  // four consecutive rows per thread
    i32x4 c = i32x4{};
    if (r + 4 <= rows) {
      c = *reinterpret_cast<const i32x4*>(counts + r);
    } else {
      for (int e = 0; e < 4; ++e)
        if (r + e < rows) c[e] = counts[r + e];
    }
    const int32_t own = c[0] + c[1] + c[2] + c[3];
    int32_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t y = __shfl_up(incl, o);
      incl += lane >= o ? y : 0;
    }
    if (lane == 63) wtot[par][w] = incl;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int y = 0; y < SCAN_T / 64; ++y) {
      before += y < w ? wtot[par][y] : 0;
      total += wtot[par][y];
    }
    int32_t at = run + before + incl - own;
    i32x4 o4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o4[e] = at;
      at += c[e];
    }
    if (r + 4 <= rows) {
      *reinterpret_cast<i32x4*>(row_ptr + r) = o4;
    } else {
      for (int e = 0; e < 4; ++e)
        if (r + e < rows) row_ptr[r + e] = o4[e];
    }
    run += total;
  }
  if (t == 0) row_ptr[rows] = run;
}

// One wave per row: lane w holds word w of the row's mask (n_k <= 4,096), and
// each word's ids leave in one contiguous store.
__global__ void __launch_bounds__(SEL_T)
    compact_rows_kernel(const uint8_t* __restrict__ masks, const int32_t* __restrict__ row_ptr,
                        int rows, int n_k, int32_t* __restrict__ col_idx) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * SEL_ROWS + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (r >= rows) return;
  const int words = (n_k + 63) / 64;
  const uint8_t* mrow = masks + (size_t)r * mask_stride(n_k);
  uint64_t mine = 0;
  if (lane < words) mine = n_k < 8 ? *mrow : reinterpret_cast<const uint64_t*>(mrow)[lane];
  int32_t* out = col_idx + row_ptr[r];
  for (int w = 0; w < words; ++w) {
    const uint64_t m = read_lane(mine, w);
    if ((m >> lane) & 1) out[bits_below(m, lane)] = w * 64 + lane;
    out += __popcll(m);
  }
}

template <int V>
void launch_sel(const float* mass, int rows, int n_q, int n_k, int n_kv, int N, int block_q,
                float tau, int topk, int32_t* counts, uint8_t* masks, hipStream_t stream) {
  const dim3 grid((rows + SEL_ROWS - 1) / SEL_ROWS);
  int tau_exp = 0;  // tau in [2^(tau_exp - 1), 2^tau_exp)
  frexpf(tau, &tau_exp);
  if (topk > 0)
    hipLaunchKernelGGL((select_rows_kernel<V, true>), grid, dim3(SEL_T), 0, stream, mass, rows,
                       n_q, n_k, n_kv, N, block_q, tau, -tau_exp, topk, counts, masks);
  else
    hipLaunchKernelGGL((select_rows_kernel<V, false>), grid, dim3(SEL_T), 0, stream, mass, rows,
                       n_q, n_k, n_kv, N, block_q, tau, -tau_exp, topk, counts, masks);
}

}  // namespace

size_t select_workspace_bytes(int rows, int n_k) {
  // row counts, then one byte per block (the bit masks take an eighth of it)
  const size_t counts = ((size_t)rows * 4 + 255) & ~(size_t)255;
  return counts + (size_t)rows * n_k;
}

int select_max_nk() { return 4096; }

hipError_t launch_select(const float* mass, int B, int H, int N, int block_q, int block_k,
                         float tau, int topk, int32_t* row_ptr, int32_t* col_idx, void* workspace,
                         hipStream_t stream) {
  const int n_pad = padded_len(N, block_q, block_k);
  const int n_q = n_pad / block_q, n_k = n_pad / block_k;
  const int n_kv = (N + block_k - 1) / block_k;
  const int rows = B * H * n_q;
  int32_t* counts = static_cast<int32_t*>(workspace);
  uint8_t* masks =
      static_cast<uint8_t*>(workspace) + (((size_t)rows * 4 + 255) & ~(size_t)255);
  if (n_k <= 64) launch_sel<1>(mass, rows, n_q, n_k, n_kv, N, block_q, tau, topk, counts, masks, stream);
  else if (n_k <= 256) launch_sel<4>(mass, rows, n_q, n_k, n_kv, N, block_q, tau, topk, counts, masks, stream);
  else if (n_k <= 1024) launch_sel<16>(mass, rows, n_q, n_k, n_kv, N, block_q, tau, topk, counts, masks, stream);
  else if (n_k <= 2048) launch_sel<32>(mass, rows, n_q, n_k, n_kv, N, block_q, tau, topk, counts, masks, stream);
  else if (n_k <= 4096) launch_sel<64>(mass, rows, n_q, n_k, n_kv, N, block_q, tau, topk, counts, masks, stream);
  else return hipErrorInvalidValue;
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(SCAN_T), 0, stream, counts, rows, row_ptr);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(compact_rows_kernel, dim3((rows + SEL_ROWS - 1) / SEL_ROWS),
                     dim3(SEL_T), 0, stream, masks, row_ptr, rows, n_k, col_idx);
  return hipGetLastError();
}

}  // namespace losa
