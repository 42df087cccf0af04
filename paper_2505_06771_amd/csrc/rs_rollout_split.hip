// rs_rollout_split.hip -- the fused rollout's kernels for launches whose full
// wavefronts would leave SIMDs idle: fewer envs per wavefront, one wavefront
// per SIMD. They are a translation unit of their own so that the out-of-line
// parts of the certificate they share with the full kernels are compiled for
// their register budget here and for the full kernels' there.
#include "rs_rollout.hpp"

namespace rs {

template <bool PP> static const void *split_kernel(int N) {
  const void *k = nullptr;
  static_for<2, 15>([&](auto nc) {
    constexpr int n = decltype(nc)::value;
    constexpr int g = n <= 2 ? 2 : (n <= 4 ? 4 : (n <= 8 ? 8 : 16));
    if (N == n) k = reinterpret_cast<const void *>(&k_rollout<g, n, PP, false, true>);
  });
  return k;
}

const void *rollout_split_kernel(int N, bool predator_prey) {
  return predator_prey ? split_kernel<true>(N) : split_kernel<false>(N);
}

}  // namespace rs
