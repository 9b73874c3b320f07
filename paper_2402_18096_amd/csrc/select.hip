// Top-k re-ranking with a recent window, demotion of tokens that fall out of
// the importance cache to the retained cache (re-quantized with Eq. 1), and
// the first selection after prefill (Fig. 3 right; Sections 2.1, 3.1).  The
// per-head device code is in select_device.h.
#include <algorithm>

#include "select_device.h"

namespace mikv {

namespace {

// (Register budget: five blocks per CU, so 1280 heads take one round.)
template <int HI_BITS, int LO_BITS>
__global__ __launch_bounds__(kSel) __attribute__((amdgpu_waves_per_eu(5))) void select_kernel(SelArgs A) {
  select_head<HI_BITS, LO_BITS>(A, blockIdx.x);
}

// First selection: one block per head finds the cut, the rank key of the
// n_dem-th least important eligible token, by radix select, and writes the
// mask.  The scores' order-preserving bits stay in registers (ITEMS per thread;
// a longer prompt's tail is read again in each pass), digits are 11 bits wide,
// and the passes end as soon as the digit's whole bin lies below the cut: a
// third digit is rare, the position digits follow only where equal scores
// straddle the cut.  Bound: the passes' barriers and LDS atomics (equal
// exponents meet in few bins) at one or two blocks per CU.  Against 256 threads
// that read the scores again for eight 8-bit passes: 128 heads x 32768 tokens
// 277 -> 46 us, 1280 x 8192 175 -> 54 us, 4 x 512 39 -> 5.4 us.
// Once the score is known the next digit starts at the highest bit that a
// position of this prompt can have.  Blocks have 1024 threads, or 256 for
// prompts of up to 1024 tokens with heads enough to fill the chip, where four
// times the blocks fit a CU (8192 heads x 16
// tokens, all scores equal: 157 -> 27 us; 93 with the 8-bit passes).
constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;

template <int kPre, int ITEMS>
__global__ __launch_bounds__(kPre) void select_prefill_kernel(const float *scores, int length, int k_heavy, int window,
                                                              uint8_t *hi_mask) {
  __shared__ uint32_t s_hist[kBins];
  __shared__ uint32_t s_wave[kPre / 64];
  __shared__ uint32_t s_pick[3];  // digit, rank inside its bin, the bin's count
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float *sc = scores + (int64_t)h * length;
  uint8_t *mask = hi_mask + (int64_t)h * length;
  const int thr = length - window > 0 ? length - window : 0;
  const int n_dem = thr - k_heavy;
  if (n_dem <= 0) {
    for (int j = tid; j < length; j += kPre) mask[j] = 1;
    return;
  }
  uint32_t ord[ITEMS];  // of the tokens tid + kPre u
#pragma unroll
  for (int u = 0; u < ITEMS; ++u) {
    const int i = u * kPre + tid;
    ord[u] = i < thr ? ordered_bits(sc[i]) : 0u;
  }
  // every eligible token's (ordered score bits, position)
  auto each = [&](auto f) {
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int i = u * kPre + tid;
      if (i < thr) f(ord[u], (uint32_t)i);
    }
    for (int i = ITEMS * kPre + tid; i < thr; i += kPre) f(ordered_bits(sc[i]), (uint32_t)i);
  };
  // The key (score bits, position) is 64 bits: digits from `shift` on, `known`
  // the bits of the prefix that earlier digits fixed.
  uint64_t prefix = 0, known = 0;
  uint32_t rank = (uint32_t)n_dem;
  const int pos_bits = thr > 1 ? 32 - __clz(thr - 1) : 0;  // positions are below 2^pos_bits
  for (int shift = 64 - kDigitBits;;) {
    for (int b = tid; b < kBins; b += kPre) s_hist[b] = 0u;
    __syncthreads();
    each([&](uint32_t o, uint32_t i) {
      const uint64_t key = ((uint64_t)o << 32) | i;
      if (((key ^ prefix) & known) == 0) atomicAdd(&s_hist[(uint32_t)(key >> shift) & (kBins - 1)], 1u);
    });
    __syncthreads();
    // the bin that holds the rank: a few bins per thread, an inclusive scan
    constexpr int PER = kBins / kPre;
    uint32_t c[PER], incl = 0u;
#pragma unroll
    for (int e = 0; e < PER; ++e) incl += c[e] = s_hist[PER * tid + e];
    const uint32_t own = incl;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += s_wave[w];
    uint32_t before = incl - own;
    if (before < rank && rank <= incl) {  // one thread
      bool found = false;
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        if (!found && rank <= before + c[e]) {
          found = true;
          s_pick[0] = PER * tid + e;
          s_pick[1] = rank - before;
          s_pick[2] = c[e];
        }
        if (!found) before += c[e];
      }
    }
    __syncthreads();
    prefix |= (uint64_t)s_pick[0] << shift;  // (the last digit's upper bits are known ones again)
    known = ~0ull << shift;
    rank = s_pick[1];
    if (rank == s_pick[2] || shift == 0) {
      prefix |= ((uint64_t)1 << shift) - 1;  // the whole bin leaves
      break;
    }
    const int next = shift - kDigitBits;
    shift = max(0, shift <= 32 ? min(next, pos_bits - kDigitBits) : next);
  }
  const uint64_t cut = prefix;
  each([&](uint32_t o, uint32_t i) { mask[i] = ((((uint64_t)o << 32) | i) <= cut) ? 0 : 1; });
  for (int j = thr + tid; j < length; j += kPre) mask[j] = 1;
}

// The sorted heavy-token list (Fig. 3 right: the tokens the re-rank kept
// for their accumulated attention): per head, the importance-pool tokens
// outside the window, most important first by the rank key (score
// descending, an exact tie to the newer token).  One block per head sorts
// the pool's keys in LDS with a bitonic network (window tokens and empty
// slots get key 0, below every real key, so they sort last).
constexpr int kHeavyMaxSlots = 8192;  // importance-pool slots a head may hold for the list (64 KiB of keys)

__global__ __launch_bounds__(kSel) void heavy_list_kernel(const int32_t *n_hi, const int32_t *hi_pos,
                                                          const float *hi_acc, int cap_hi, int P, int thr, int k_heavy,
                                                          int32_t *heavy_idx) {
  extern __shared__ uint64_t s_key[];  // [P], P a power of two >= cap_hi
  const int h = blockIdx.x;
  const int n = min(n_hi[h], cap_hi);
  const int32_t *pos = hi_pos + (int64_t)h * cap_hi;
  const float *acc = hi_acc + (int64_t)h * cap_hi;
  for (int i = threadIdx.x; i < P; i += kSel) {
    uint64_t k = 0;
    if (i < n) {
      const int p = pos[i];
      if (p < thr) k = rank_key(acc[i], p);
    }
    s_key[i] = k;
  }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += kSel) {
        const int l = i ^ j;
        if (l > i) {
          const uint64_t a = s_key[i], b = s_key[l];
          // descending overall: runs with (i & k) == 0 descend, the others ascend
          const bool swap = (i & k) == 0 ? a < b : a > b;
          if (swap) {
            s_key[i] = b;
            s_key[l] = a;
          }
        }
      }
      __syncthreads();
    }
  }
  int32_t *out = heavy_idx + (int64_t)h * k_heavy;
  for (int r = threadIdx.x; r < k_heavy; r += kSel) {
    const uint64_t k = r < P ? s_key[r] : 0;
    out[r] = k != 0 ? (int32_t)(uint32_t)(k & 0xffffffffu) : -1;
  }
}

template <int HI, int LO>
void launch_select(const SelArgs &A, int NH, hipStream_t st) {
  hipLaunchKernelGGL((select_kernel<HI, LO>), dim3(NH), dim3(kSel), 0, st, A);
}

}  // namespace

}  // namespace mikv

using namespace mikv;

extern "C" size_t mikv_select_workspace_size(const mikv_cache *c) {
  if (!c) return 0;
  return (size_t)2 * 4 * (size_t)c->batch * c->kv_heads * (size_t)std::max(c->cap_hi, 1);
}

namespace mikv {

int select_topk(const mikv_cache *c, int32_t length, int32_t k_heavy, int32_t window, void *ws, size_t ws_bytes,
                bool appended, hipStream_t st) {
  int rc = validate_cache(c);
  if (rc) return rc;
  if (k_heavy < 0 || window < 0) return set_error(MIKV_ERR_INVALID_ARG, "mikv_select_topk: negative k_heavy/window");
  if (length < 1 || length > c->max_len)
    return set_error(length < 1 ? MIKV_ERR_INVALID_ARG : MIKV_ERR_CAPACITY,
                     "mikv_select_topk: length %d outside [1, max_len]", length);
  if (!ws || ws_bytes < mikv_select_workspace_size(c))
    return set_error(MIKV_ERR_CAPACITY, "mikv_select_topk: workspace too small");
  if (c->key_block && window < kKeyBlock)
    return set_error(MIKV_ERR_INVALID_ARG, "mikv_select_topk: per-channel keys need a window >= %d (got %d)",
                     kKeyBlock, window);
  SelArgs A = make_sel_args(c, length, k_heavy, window, ws);
  A.pending = appended ? 1 : 0;
  const int NH = n_heads_of(c);
  switch (format_key(c)) {
    case 1602: launch_select<16, 2>(A, NH, st); break;
    case 1604: launch_select<16, 4>(A, NH, st); break;
    case 1608: launch_select<16, 8>(A, NH, st); break;
    case 802: launch_select<8, 2>(A, NH, st); break;
    case 1603: launch_select<16, 3>(A, NH, st); break;
    case 803: launch_select<8, 3>(A, NH, st); break;
    case 402: launch_select<4, 2>(A, NH, st); break;
    case 804: launch_select<8, 4>(A, NH, st); break;
    default: launch_select<8, 8>(A, NH, st); break;
  }
  return check_launch("mikv_select_topk");
}

}  // namespace mikv

extern "C" int mikv_select_topk(const mikv_cache *c, int32_t length, int32_t k_heavy, int32_t window,
                                int32_t *heavy_idx, void *ws, size_t ws_bytes, void *stream) {
  if (heavy_idx && c && c->cap_hi > kHeavyMaxSlots)
    return set_error(MIKV_ERR_UNSUPPORTED, "mikv_select_topk: the heavy list needs cap_hi <= %d (got %d)",
                     kHeavyMaxSlots, c->cap_hi);
  int rc = select_topk(c, length, k_heavy, window, ws, ws_bytes, false, (hipStream_t)stream);
  if (rc || !heavy_idx || k_heavy == 0) return rc;
  int P = 1;
  while (P < c->cap_hi) P <<= 1;
  const int thr = std::max(0, length - window);
  hipLaunchKernelGGL(heavy_list_kernel, dim3(n_heads_of(c)), dim3(kSel), (size_t)P * sizeof(uint64_t),
                     (hipStream_t)stream, c->n_hi, c->hi_pos, c->hi_acc, c->cap_hi, P, thr, k_heavy, heavy_idx);
  return check_launch("mikv_select_topk (heavy list)");
}

extern "C" int32_t mikv_heavy_budget(int32_t length, int32_t ratio_num, int32_t ratio_den, int32_t window,
                                     int32_t window_in_ratio) {
  if (length < 0 || ratio_num < 0 || ratio_den < 1 || window < 0) return -1;
  int64_t k = (int64_t)ratio_num * length / ratio_den;
  if (window_in_ratio) k -= window;
  return (int32_t)std::max<int64_t>(0, k);
}

extern "C" int mikv_select_prefill(const float *scores, int32_t n_heads, int32_t length, int32_t k_heavy,
                                   int32_t window, uint8_t *hi_mask, void *stream) {
  if (!scores || !hi_mask) return set_error(MIKV_ERR_INVALID_ARG, "mikv_select_prefill: NULL pointer");
  if (n_heads < 1 || length < 1 || k_heavy < 0 || window < 0)
    return set_error(MIKV_ERR_INVALID_ARG, "mikv_select_prefill: bad sizes");
  const int threads = n_heads >= 512 && length <= 1024 ? 256 : 1024;
  auto kernel = threads == 256         ? select_prefill_kernel<256, 4>
                : length <= 4 * 1024  ? select_prefill_kernel<1024, 4>
                : length <= 16 * 1024 ? select_prefill_kernel<1024, 16>
                                      : select_prefill_kernel<1024, 32>;
  constexpr int kMost = 1 << 20;  // heads per launch: a grid's threads stay below 2^32
  for (int64_t h0 = 0; h0 < n_heads; h0 += kMost)
    hipLaunchKernelGGL(kernel, dim3((int)std::min<int64_t>(kMost, n_heads - h0)), dim3(threads), 0, (hipStream_t)stream,
                       scores + h0 * length, length, k_heavy, window, hi_mask + h0 * length);
  return check_launch("mikv_select_prefill");
}
