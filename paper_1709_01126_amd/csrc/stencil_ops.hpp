// stencil_ops.hpp -- device helpers shared by the kernels.
#pragma once

#include <type_traits>

#include "solver.hpp"

namespace pot3d {

// Checked builds (-DPOT3D_CHECKED, libpot3d_checked.so) test every global
// index of the stencil kernels against its array size.  An index out of range
// is replaced by 0 and the source line is recorded in g_oob_line, which the
// host reads after each solve.  Normal builds compile CHK(i, n) to i.
#ifdef POT3D_CHECKED
static __device__ unsigned int g_oob_line = 0;   // one per source file
__device__ __forceinline__ long long chk_index(long long i, long long n, unsigned line)
{
    if (i < 0 || i >= n) {
        g_oob_line = line;
        return 0;
    }
    return i;
}
#define CHK(i, n) chk_index((long long)(i), (long long)(n), __LINE__)
#else
#define CHK(i, n) (i)
#endif

// The line that this source file's kernels have recorded (0: none), cleared.
static inline unsigned read_oob_line()
{
    unsigned line = 0;
#ifdef POT3D_CHECKED
    const unsigned zero = 0;
    if (hipMemcpyFromSymbol(&line, HIP_SYMBOL(g_oob_line), sizeof(line)) != hipSuccess) return ~0u;
    if (line) (void)hipMemcpyToSymbol(HIP_SYMBOL(g_oob_line), &zero, sizeof(zero));
#endif
    return line;
}

template <typename V> __device__ __forceinline__ V vfma(V a, V b, V c);
template <> __device__ __forceinline__ double vfma<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <> __device__ __forceinline__ float vfma<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Pointer to global memory, typed as such.
template <typename T>
using GPtr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ GPtr<T> to_global(T *p)
{
    return (GPtr<T>)p;
}

// Pointer to memory that no kernel writes while this one runs (row tables,
// the scalar block): uniform loads through it become scalar loads.
template <typename T>
using CPtr = __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ CPtr<T> to_const(T *p)
{
    return (CPtr<T>)p;
}

// Streaming accesses: vectors that a pass reads or writes once per cell use
// the non-temporal policy, so they do not displace the lines that are read
// again soon (the operand's halo rows and layers, and the tiles the next pass
// starts on).  Measured: 393 -> 369 us per FP64 iteration at 151 x 301 x 601,
// 3.72 -> 3.48 ms at 301 x 641 x 1281, FP32-refined solve 1.28 -> 1.23 s.
template <typename P>
__device__ __forceinline__ auto stream_load(P p)
{
    return __builtin_nontemporal_load(p);
}
template <typename P, typename T>
__device__ __forceinline__ void stream_store(P p, T v)
{
    __builtin_nontemporal_store(v, p);
}

__device__ __forceinline__ RowCoef load_row(CPtr<const RowCoef> rows, long long idx)
{
    RowCoef r;
    r.rm = rows[idx].rm;
    r.rp = rows[idx].rp;
    r.tm = rows[idx].tm;
    r.tp = rows[idx].tp;
    r.s = rows[idx].s;
    r.pq = rows[idx].pq;
    r.pad0 = r.pad1 = 0.0;
    return r;
}

// Reciprocal of a positive normal value: the hardware estimate refined by
// two Newton steps y <- y + y (1 - d y), each of which squares the relative
// error (within about an ulp of 1/d).
__device__ __forceinline__ double recip(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    double e = __builtin_fma(-d, y, 1.0);
    y = __builtin_fma(y, e, y);
    e = __builtin_fma(-d, y, 1.0);
    return __builtin_fma(y, e, y);
}
// FP32: the estimate and one Newton step (about an ulp; the IEEE division
// is three times the instructions).
__device__ __forceinline__ float recip(float d)
{
    const float y = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(y, __builtin_fmaf(-d, y, 1.0f), y);
}

// A double moved across lanes by a DPP row shift (row_shr:n is 0x110 + n,
// row_shl:n is 0x100 + n; rows are 16 lanes).  Lanes whose source lies
// outside their row receive 0.
template <int CTRL>
__device__ __forceinline__ double row_shift(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Lane l receives lane l-1 (shr) or l+1 (shl); the lane past the wavefront's
// end receives 0 (DPP bound control: no initialised destination needed).
__device__ __forceinline__ double shr1(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x138, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x138, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double shl1(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x130, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x130, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float shl1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xF, 0xF, true));
}

// The value of v in lane l (uniform l), as a wave-uniform double.
__device__ __forceinline__ double lane_value(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ double wave_uniform(double v)
{
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float wave_uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Element at a 32-bit byte offset from a vector's base: the access takes the
// base in scalar registers and a 32-bit offset per lane.  (The one-sweep
// path is used for vectors under 4 GiB.)
template <typename T>
__device__ __forceinline__ GPtr<T> at_byte(GPtr<T> base, unsigned boff)
{
    using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return (GPtr<T>)((__attribute__((address_space(1))) C *)base + boff);
}

// Orders one wavefront's LDS accesses across lanes (a row moving between
// layouts): release and acquire fences at wavefront scope around a wave barrier.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The ring buffer that sweep j uses as p_{j-off} (off = 0: the one it writes).
template <typename V>
__device__ __forceinline__ V *ring_at(const SweepVecs<V> &v, int sweep, int off)
{
    const int q = (sweep % 3 + 3 - off) % 3;
    return q == 0 ? v.ring[0] : (q == 1 ? v.ring[1] : v.ring[2]);
}

}  // namespace pot3d
