// Four consecutive rows (a "quad") per lane: the accesses, the LDS staging and
// the H_up term that the column kernels and the batched product share.
#pragma once
#include <cstdint>

#include "internal.h"

namespace hub {
namespace {

// one fused multiply-add, a * b + c
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T, int TB>
struct Vec {
    T v[TB];
};

// ---- 16-byte accesses ---------------------------------------------------
template <typename T>
struct Q4 {
    T v[4];
};

template <typename T>
__device__ __forceinline__ Q4<T> ld_q4(const T *p)
{
    Q4<T> r;
    if constexpr (sizeof(T) == 4) {
        const float4 q = *reinterpret_cast<const float4 *>(p);
        r.v[0] = q.x;
        r.v[1] = q.y;
        r.v[2] = q.z;
        r.v[3] = q.w;
    } else {
        const double2 q0 = reinterpret_cast<const double2 *>(p)[0], q1 = reinterpret_cast<const double2 *>(p)[1];
        r.v[0] = q0.x;
        r.v[1] = q0.y;
        r.v[2] = q1.x;
        r.v[3] = q1.y;
    }
    return r;
}

template <typename T>
__device__ __forceinline__ void st_q4(T *p, const T (&v)[4])
{
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        reinterpret_cast<double2 *>(p)[0] = make_double2(v[0], v[1]);
        reinterpret_cast<double2 *>(p)[1] = make_double2(v[2], v[3]);
    }
}

// Quads of columns whose length is no multiple of 4: element-aligned 16-byte
// accesses, and the first nv (1..3) rows alone in a column's last quad.
template <typename T>
__device__ __forceinline__ Q4<T> ld_q4e(const T *p, int nv)
{
    constexpr int N = 16 / (int)sizeof(T);
    typedef T VecU __attribute__((ext_vector_type(N), aligned(sizeof(T))));
    Q4<T> r;
    if (nv >= 4) {
#pragma unroll
        for (int h = 0; h < 4 / N; ++h) {
            const VecU q = *reinterpret_cast<const VecU *>(p + h * N);
#pragma unroll
            for (int i = 0; i < N; ++i) r.v[h * N + i] = q[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) r.v[i] = i < nv ? p[i] : (T)0;
    }
    return r;
}

template <typename T>
__device__ __forceinline__ void st_q4e(T *p, const T (&v)[4], int nv)
{
    constexpr int N = 16 / (int)sizeof(T);
    typedef T VecU __attribute__((ext_vector_type(N), aligned(sizeof(T))));
    if (nv >= 4) {
#pragma unroll
        for (int h = 0; h < 4 / N; ++h) {
            VecU q;
#pragma unroll
            for (int i = 0; i < N; ++i) q[i] = v[h * N + i];
            *reinterpret_cast<VecU *>(p + h * N) = q;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < nv) p[i] = v[i];
    }
}

// Alignment of N interleaved columns' values of one row: whole accesses where N is a power of two
template <typename T, int N>
constexpr int vec_align = (N & (N - 1)) != 0 ? (int)sizeof(T) : sizeof(T) * N < 16 ? (int)sizeof(T) * N : 16;

// Distance in LDS between the four rows of quad q of nq staged quads (lds_slot)
__device__ __forceinline__ int quad_pitch(int q, int nq) { return min(64, nq - (q & ~63)); }

// N interleaved columns' values of one row, as one LDS access where N is a power of two
template <typename T, int N>
__device__ __forceinline__ Vec<T, N> ld_vec(const T *p)
{
    struct alignas(vec_align<T, N>) V {
        Vec<T, N> v;
    };
    return reinterpret_cast<const V *>(p)->v;
}

// Quad q of nq staged quads of TB columns, interleaved by column, to its lds_slot
template <typename T, int TB>
__device__ __forceinline__ void put_quad(T *xs, const Q4<T> (&v)[TB], int q, int nq)
{
    struct alignas(vec_align<T, TB>) V {
        Vec<T, TB> v;
    };
    const int s0 = lds_slot(4 * q, 4 * nq), sw = quad_pitch(q, nq);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        V o;
#pragma unroll
        for (int t = 0; t < TB; ++t) o.v.v[t] = v[t].v[r];
        *reinterpret_cast<V *>(xs + (s0 + r * sw) * TB) = o;
    }
}

// acc[r][t] += the H_up entries of a quad's four rows (entry k of the four in
// e4[16 k]), two entry columns at a time, the next two loaded meanwhile.  Bound
// by the LDS: two reads an entry, 62 % of a CU's busy cycles on the 4x4 torus (FP32,
// two columns), half of them bank conflicts; without the next entries' loads 1.24
// instead of 1.20 ms a product.
template <typename T, int TB>
__device__ __forceinline__ void up_quad(T (&acc)[4][TB], const T *xs, const T *tab, const uint4 *__restrict__ e4,
                                        int len)
{
    auto use = [&](const uint4 &q) {
        const uint32_t e[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const T v = tab[e[i] >> 24];
            const Vec<T, TB> xr = ld_vec<T, TB>(xs + (e[i] & 0xFFFFFFu) * TB);
#pragma unroll
            for (int t = 0; t < TB; ++t) acc[i][t] = mad(v, xr.v[t], acc[i][t]);
        }
    };
    if (len <= 0) return;
    uint4 na = e4[0], nb = e4[16 * min(1, len - 1)];
    int k = 0;
    for (; k + 2 <= len; k += 2) {
        const uint4 ea = na, eb = nb;
        na = e4[16 * min(k + 2, len - 1)];
        nb = e4[16 * min(k + 3, len - 1)];
        use(ea);
        use(eb);
    }
    if (k < len) use(na);
}

}  // namespace
}  // namespace hub
