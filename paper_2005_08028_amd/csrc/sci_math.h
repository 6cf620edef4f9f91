// Per-voxel arithmetic of the TV denoiser (and the workgroup numbering),
// shared by every HIP kernel of the library so that the streaming and the
// fused schedules evaluate identical expressions (the build disables floating-point contraction; every fused
// multiply-add below is explicit).
//
// Notation follows Algorithm 1 (FGP box) of the paper: w is the extrapolated
// dual, theta = x - lambda D^T w, z = D theta, q = w + z / (8 lambda),
// p = projection of q onto the unit ball of the TV's dual norm.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sci {

enum { TV_ATV = 0, TV_ITV2D = 1, TV_VTV = 2 };
enum { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2 };

// ---- dual storage types ---------------------------------------------------

template <int DT> struct Dual;

template <> struct Dual<DT_F32> {
    using T = float;
    __device__ static inline float cvt(T v) { return v; }
    __device__ static inline float ld(const T *p, uint32_t i) { return p[i]; }
    __device__ static inline T to(float v) { return v; }
    __device__ static inline void st(T *p, uint32_t i, float v) { p[i] = v; }
};

// bfloat16: upper half of a float32; stores round to nearest even.
template <> struct Dual<DT_BF16> {
    using T = uint16_t;
    __device__ static inline float cvt(T v) { return __uint_as_float((uint32_t)v << 16); }
    __device__ static inline float ld(const T *p, uint32_t i) { return cvt(p[i]); }
    __device__ static inline T to(float v)
    {
        uint32_t u = __float_as_uint(v);
        uint32_t r = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
        if ((u & 0x7fffffffu) > 0x7f800000u) r = (u >> 16) | 0x40u; // keep NaN a NaN
        return (uint16_t)r;
    }
    __device__ static inline void st(T *p, uint32_t i, float v) { p[i] = to(v); }
};

// IEEE binary16: hardware conversion (round to nearest even).
template <> struct Dual<DT_F16> {
    using T = _Float16;
    __device__ static inline float cvt(T v) { return (float)v; }
    __device__ static inline float ld(const T *p, uint32_t i) { return cvt(p[i]); }
    __device__ static inline T to(float v) { return (_Float16)v; }
    __device__ static inline void st(T *p, uint32_t i, float v) { p[i] = to(v); }
};

// ---- the FGP step ---------------------------------------------------------

// Extrapolated dual w = p + beta (p - p_prev).
__device__ inline float extrapolate(float p, float pp, float beta) { return fmaf(beta, p - pp, p); }

// theta = x - lambda (D^T w) with
// (D^T w)(i,j) = (w_h(i,j-1) - w_h(i,j)) + (w_v(i-1,j) - w_v(i,j));
// missing neighbours enter as 0.
__device__ inline float theta_of(float x, float wh_left, float wh, float wv_up, float wv, float lam)
{
    return fmaf(-lam, (wh_left - wh) + (wv_up - wv), x);
}

// q = w + step * z. Entries of the dual that carry no difference take
// step = 0 (so q = w, which is 0 there) instead of a masked z.
__device__ inline float ascend(float w, float z, float step) { return fmaf(step, z, w); }

// Cross-lane neighbours along j, as DPP wavefront shifts folded into the
// consuming instruction: the value held by lane l-1 (0 in lane 0), and by
// lane l+1 (0 in lane 63).
__device__ inline float from_left(float v) { return __builtin_amdgcn_update_dpp(0.0f, v, 0x138, 0xF, 0xF, true); }
__device__ inline float from_right(float v) { return __builtin_amdgcn_update_dpp(0.0f, v, 0x130, 0xF, 0xF, true); }

// ATV projection q / max(1, |q|): equal to clamping q to [-1, 1]. One v_med3_f32
// (a NaN gives -1, as the pair fmaxf, fminf does, which also costs a
// canonicalising v_max_f32).
__device__ inline float proj_atv(float q) { return __builtin_amdgcn_fmed3f(q, -1.0f, 1.0f); }

// Isotropic scale 1 / max(1, sqrt(n2)) = min(1, 1/sqrt(n2)) for a squared norm
// n2 >= 0. A NaN norm gives 1 (fminf returns its other operand): the finite
// components of that pixel, with VTV the other frames', stay as they are.
__device__ inline float iso_scale(float n2) { return fminf(1.0f, __builtin_amdgcn_rsqf(n2)); }
// The same for a norm that is no NaN: the median with 0 and 1 becomes the output
// clamp of v_rsq_f32 and costs no instruction (fminf is one of the 19 of an
// ITV2D voxel-iteration), but turns a NaN into 0.
__device__ inline float iso_scale_no_nan(float n2)
{
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_rsqf(n2), 0.0f, 1.0f);
}
// A pass that starts from a zero dual meets no NaN norm while every pixel it
// reads is at most this: |w| <= 3, so |theta| <= |x| + 12 lambda and
// |q| <= 3 + (|x| + 12 lambda) / (4 lambda) stay finite. One comparison per pixel
// and pass then saves an instruction per pixel and iteration. (Starting duals
// would need two to four comparisons more; those passes keep iso_scale.)
__device__ inline float no_nan_limit(float lam)
{
    return lam > 1e-37f && lam < 1e30f ? 1e37f * fminf(1.0f, lam) : -1.0f;
}

// Semi-implicit (Chambolle 2004) scale 1 / (1 + sqrt(n2)) for the squared
// norm n2 of z/(8 lambda), with the hardware square root and reciprocal
// (v_sqrt_f32, v_rcp_f32: about 1 ulp each, in place of the IEEE-exact
// sequences, which cost several times the instructions).
__device__ inline float semi_implicit_scale(float n2)
{
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_sqrtf(n2));
}

// The same step per component (ATV): q / (1 + |s|) for s = z/(8 lambda).
__device__ inline float semi_implicit_atv(float q, float s) { return q * __builtin_amdgcn_rcpf(1.0f + fabsf(s)); }

// Squared-norm accumulation (h^2 + v^2 added to acc).
__device__ inline float norm2_add(float acc, float h, float v) { return fmaf(v, v, fmaf(h, h, acc)); }

// The step of a row's vertical differences: step where 0 <= r < nx - 1, else 0,
// for a row r that is uniform over the wavefront. Selected as an integer, which
// the scalar unit does (a float select takes a vector instruction).
__device__ inline float row_step(int r, int nx, float step)
{
    return __int_as_float(__float_as_int(step) & -(int)((uint32_t)r < (uint32_t)(nx - 1)));
}

// ---- image rows as bounded buffers ------------------------------------------
//
// The columns of an image row that a strip of lanes covers, as a raw buffer
// resource: the address is wavefront-uniform (scalar), a lane gives its byte
// offset in 32 bits, and the hardware's range check stands in for the masks of
// a stencil's edges: a load at an offset >= `bytes` returns 0 and a store there
// is dropped. bytes = 0 makes a row that does not exist. This spares the
// 64-bit vector address of every access, the selects on the loaded values and
// the execution masks around the stores.
using RowBuf = __amdgpu_buffer_rsrc_t;
constexpr uint32_t kNoColumn = 1u << 27; // element offset of a lane that takes no part: past any strip

template <typename T> __device__ inline RowBuf row_buf(const T *row, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)const_cast<T *>(row), 0, (int)bytes, 0x00020000);
}
__device__ inline float row_ld(RowBuf b, uint32_t off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)off, 0, 0));
}
__device__ inline void row_st(RowBuf b, uint32_t off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), b, (int)off, 0, 0);
}

// Keep a prefetch where it stands: memory reads above cannot sink below (the
// compiler otherwise moves loads whose values only the next loop iteration
// uses to the loop's end, where their latency is exposed).
__device__ __forceinline__ void issued() { asm volatile("" ::: "memory"); }
// Wait here for the load that fills v.
__device__ __forceinline__ void settle(float &v) { asm volatile("" : "+v"(v)); }

// ---- work mapping -----------------------------------------------------------

// Workgroups are handed to the 8 XCDs of the chip round-robin by linear id;
// renumber them so that XCD c gets one contiguous run of tiles (raster order
// within a frame), and tiles that share halos or cache lines share that
// XCD's L2.
__device__ inline int xcd_contiguous(int wg, int nwg)
{
    constexpr int kXcd = 8;
    const int q = nwg / kXcd, r = nwg % kXcd;
    const int c = wg % kXcd, idx = wg / kXcd;
    return c < r ? c * (q + 1) + idx : r * (q + 1) + (c - r) * q + idx;
}

// Workgroup barrier over LDS only: waits for this wavefront's LDS accesses
// (lgkmcnt), not for its global loads and stores; the signal fences keep the
// compiler from moving memory accesses across it.
__device__ __forceinline__ void lds_barrier()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F); // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

} // namespace sci
