// An axis that a wave knows, as a compile-time constant.
#pragma once

#include <hip/hip_runtime.h>

namespace mg {

template <int A> struct Axis { static constexpr int a = A; };
// fn(Axis<w>()), w wave-uniform
template <typename F> __device__ __forceinline__ void with_axis(int w, F fn) {
    if (w == 0)
        fn(Axis<0>());
    else if (w == 1)
        fn(Axis<1>());
    else
        fn(Axis<2>());
}

}  // namespace mg
