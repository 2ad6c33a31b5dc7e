// f(integral_constant 0) ... f(integral_constant N - 1), for bodies whose index has to be a constant.
#pragma once
#include <type_traits>
#include <utility>

#include <hip/hip_runtime.h>

namespace br {

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace br
