// Streaming kernels for one GEMV whose rows two waves share (bitcos_fast.h:
// LONG), by words per lane: bf16 rows above 16384 weights, int8 rows above
// 32768.
#include "bitcos_fast.h"

namespace bitcos_k {

template <bool BF16, int W0, int... Ws>
static FastFn pick_long_w(int w, std::integer_sequence<int, Ws...>) {
  FastFn fn = nullptr;
  ((w == W0 + Ws ? (fn = bitcos_fast_kernel<W0 + Ws, 64, BF16, false, true>, 0) : 0), ...);
  return fn;
}

// Kernel for rows of up to 128 * per_lane words; nullptr if there is none.
FastFn pick_fast_long(int per_lane, bool bf16) {
  constexpr int kB = bitcos::kMaxWordsBf16 / 2 + 1, kI = bitcos::kMaxWordsI8 / 2 + 1;
  return bf16 ? pick_long_w<true, kB>(per_lane, std::make_integer_sequence<int, bitcos::kMaxWordsBf16 - kB + 1>{})
              : pick_long_w<false, kI>(per_lane, std::make_integer_sequence<int, bitcos::kMaxWordsI8 - kI + 1>{});
}

}  // namespace bitcos_k
