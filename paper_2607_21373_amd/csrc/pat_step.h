// Device helpers shared by the step kernels (pat_kernels.hip) and the resident sweeps of
// small meshes (pat_small.hip): one row's arithmetic, so that both give the same bits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace pat {

__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The value a boundary slot multiplies: S - S_prev in a step, -S_prev in the
// transpose sweep's closing launch (only_prev).
template <typename T>
__device__ __forceinline__ T bdiff(T x, T y, bool only_prev) { return only_prev ? -y : x - y; }

// One row of a three-level step: S' = S + (d - (dt/m)(dt K S + B d - src)), d = S - Sp,
// from acc = (K S)_row, bacc = (B d)_row and the source src (0 forward).
template <typename T>
__device__ __forceinline__ T step_update_d(T cur, T d, T acc, T bacc, T src, T dm, T dt) {
    const T f = mad(dt, acc, bacc) - src;
    return cur + mad(-dm, f, d);
}
template <typename T>
__device__ __forceinline__ T step_update(T cur, T prev, T acc, T bacc, T src, T dm, T dt) {
    return step_update_d(cur, cur - prev, acc, bacc, src, dm, dt);
}
// The transpose sweep's result, (q - q_prev) m/dt - (dt K q - B q_prev - src), from
// acc = (K q)_row and bacc = -(B q_prev)_row.
template <typename T>
__device__ __forceinline__ T adj_result(T cur, T prev, T acc, T bacc, T src, T dm, T dt) {
    const T f = mad(dt, acc, bacc) - src;
    return (cur - prev) / dm - f;
}

// B values from bslot[bo], nb slots of them nonzero (nb = 0: interior row); entries
// beyond the padded slots [x0, x1); sensor weights [e0, e1)
struct RowSpec {
    int bo = 0, nb = 0, x0 = 0, x1 = 0, e0 = 0, e1 = 0;
    __device__ __forceinline__ void load(const int4 *spec, int k) {
        const int4 u = spec[2 * (k - 1)], v = spec[2 * (k - 1) + 1];
        bo = u.x; nb = u.y; x0 = u.z; x1 = u.w;
        e0 = v.x; e1 = v.y;
    }
    // from the table by row; the sensor weights' range is not in it
    __device__ __forceinline__ void load_direct(const int4 *rdir, int row) {
        const int4 u = rdir[row];
        bo = u.x; nb = u.y; x0 = u.z; x1 = u.w;
    }
    __device__ __forceinline__ void load_inject(const int32_t *injptr, int row) {
        int32_t e[2];  // one 8-byte load
        __builtin_memcpy(e, injptr + row, sizeof(e));
        e0 = e[0]; e1 = e[1];
    }
    __device__ __forceinline__ bool any() const { return nb || x1 > x0 || e1 > e0; }
};

// the four values of one quad
template <typename T>
__device__ __forceinline__ void load_quad(const T *p, T v[4]) {
    if constexpr (sizeof(T) == 4) {
        const auto q = *reinterpret_cast<const T __attribute__((ext_vector_type(4))) *>(p);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
        using V2 = T __attribute__((ext_vector_type(2)));
        const V2 q0 = reinterpret_cast<const V2 *>(p)[0], q1 = reinterpret_cast<const V2 *>(p)[1];
        v[0] = q0.x; v[1] = q0.y; v[2] = q1.x; v[3] = q1.y;
    }
}

// Compile-time loop: f(std::integral_constant<int, I>) for I = B, B + S, ... < E.
template <int B, int E, int S = 1, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + S, E, S>(f);
    }
}

}  // namespace pat
