// Sensing-operator kernels: Phi (Eq. (3)-(4)), Phi^T, the diagonal of
// Phi Phi^T, and the element-wise GAP / ADMM projections (Eq. (21), Eq. (24)).
//
// All of them are HBM streams over [B][nx][ny] volumes: one thread per pixel
// (i, j), consecutive threads on consecutive columns (coalesced), looping
// over the B frames. The per-pixel sum over frames stays in a register.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sci_internal.h"
#include "sci_math.h"

namespace sci {
namespace {

constexpr int kBlock = 256;
constexpr int kProjBlock = 64; // projection: one wavefront per workgroup

inline unsigned grid_for(size_t n)
{
    size_t g = (n + kBlock - 1) / kBlock;
    return (unsigned)(g > 0 ? g : 1);
}

__global__ __launch_bounds__(kBlock) void k_forward(uint32_t npix, int B, const float *__restrict__ C,
                                                    const float *__restrict__ X, float *__restrict__ Y)
{
    uint32_t pix = blockIdx.x * kBlock + threadIdx.x;
    if (pix >= npix) return;
    float acc = 0.0f;
    for (int k = 0; k < B; ++k) {
        uint32_t o = (uint32_t)k * npix + pix;
        acc = fmaf(C[o], X[o], acc);
    }
    Y[pix] = acc;
}

__global__ __launch_bounds__(kBlock) void k_adjoint(uint32_t npix, int B, const float *__restrict__ C,
                                                    const float *__restrict__ Y, float *__restrict__ X)
{
    uint32_t pix = blockIdx.x * kBlock + threadIdx.x;
    if (pix >= npix) return;
    float y = Y[pix];
    for (int k = 0; k < B; ++k) {
        uint32_t o = (uint32_t)k * npix + pix;
        X[o] = C[o] * y;
    }
}

__global__ __launch_bounds__(kBlock) void k_weights(uint32_t npix, int B, const float *__restrict__ C, float rho,
                                                    float *__restrict__ Sinv)
{
    uint32_t pix = blockIdx.x * kBlock + threadIdx.x;
    if (pix >= npix) return;
    float s = 0.0f;
    for (int k = 0; k < B; ++k) {
        float c = C[(uint32_t)k * npix + pix];
        s = fmaf(c, c, s);
    }
    s = s + rho;
    Sinv[pix] = s > 0.0f ? 1.0f / s : 0.0f;
}

// A solve's setup in one pass over the masks: Sinv = 1 / (sum_k C_k^2 + rho)
// (nullable), theta = Phi^T Y (nullable), u = 0 (nullable), the masks packed
// one bit per frame, and one flag per kProjBlock pixels: 1 when all their
// entries are 0 or 1, else 0 (the projection of that block then reads C). All
// masks of a pixel are loaded before their first use, into KB >= B registers.
// A memory stream with a launch's latency under it. Weights, packing, a global
// flag, theta and u as kernels of their own read C three times; with the copy
// of theta that ends a solve of no iterations, 10.8 -> 5.8 us at 256x256x8,
// 25.4 -> 17.7 us at 512x512x16, 126 -> 88 us at 1024x1024x24. The plain
// forward and adjoint products gain nothing from the same form (2.4 -> 2.0 and
// 2.6 -> 2.8 us at 256x256x8, 36.4 -> 37.6 and 44.5 -> 47.5 at 1024x1024x24).
template <int KB>
__global__ __launch_bounds__(kProjBlock) void k_setup_reg(uint32_t npix, int B, const float *__restrict__ C,
                                                          const float *__restrict__ Y, float rho,
                                                          float *__restrict__ Sinv, float *__restrict__ theta,
                                                          float *__restrict__ u, uint32_t *__restrict__ bits,
                                                          int *__restrict__ flags)
{
    const int block = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const uint32_t pix = (uint32_t)block * kProjBlock + threadIdx.x;
    bool binary = true;
    if (pix < npix) {
        float c[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) c[k] = C[(uint32_t)min(k, B - 1) * npix + pix];
        const float y = theta ? Y[pix] : 0.0f;
        float s = 0.0f;
        uint32_t m = 0u;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (k >= B) continue;
            const uint32_t o = (uint32_t)k * npix + pix;
            s = fmaf(c[k], c[k], s);
            if (c[k] == 1.0f) m |= 1u << k;
            else if (c[k] != 0.0f) binary = false;
            if (theta) theta[o] = c[k] * y;
            if (u) u[o] = 0.0f;
        }
        s = s + rho;
        if (Sinv) Sinv[pix] = s > 0.0f ? 1.0f / s : 0.0f;
        bits[pix] = m;
    }
    const bool all = __all(binary);
    if (threadIdx.x == 0) flags[block] = all ? 1 : 0;
}

// Calls f(integral_constant<int, KB>) with the smallest even KB that holds B frames (B <= 32).
template <int KB = 2, typename F> void with_slots(int B, F &&f)
{
    if constexpr (KB < 32) {
        if (B > KB) {
            with_slots<KB + 2>(B, f);
            return;
        }
    }
    f(std::integral_constant<int, KB>{});
}
inline dim3 proj_grid(uint32_t npix) { return dim3((npix + kProjBlock - 1) / kProjBlock); }

// Projection modes: what the kernels take as v, the point they project.
//   kProjGap    v = theta (Eq. (21))
//   kProjAdmm   v = theta - u (Eq. (24)); the kernel also writes the denoiser
//               input s = u + x, and x only when x is non-null
//   kProjFista  v = theta + ex (theta - u), FISTA's extrapolated point formed
//               on load from the newest iterate (theta) and the one before (u),
//               the same expression as k_extrapolate (Sec. 2.2)
//   kProjTwist  v = a2 w + a1 theta + ex u, TwIST's two-step update from the
//               denoised point (w), the newest iterate (theta) and the one
//               before (u), the same expression as k_two_step (Sec. 2.2); the
//               kernel also stores v, the new iterate, to svol
constexpr int kProjGap = 0, kProjAdmm = 1, kProjFista = 2, kProjTwist = 3;

__device__ inline float fista_point(float x, float xp, float ex) { return fmaf(ex, x - xp, x); }
__device__ inline float twist_point(float xp, float x, float th, float a0, float a1, float a2)
{
    return fmaf(a2, th, fmaf(a1, x, a0 * xp));
}

// x_k = v_k + C_k r with r = (Y - sum_k C_k v_k) Sinv.
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_project(uint32_t npix, int B, float ex, float a1, float a2, const float *__restrict__ w, const float *__restrict__ theta,
                                                    const float *__restrict__ u, const float *__restrict__ C,
                                                    const float *__restrict__ Y, const float *__restrict__ Sinv,
                                                    float *__restrict__ x, float *__restrict__ svol)
{
    uint32_t pix = blockIdx.x * kBlock + threadIdx.x;
    if (pix >= npix) return;
    constexpr bool ADMM = MODE == kProjAdmm;
    float acc = 0.0f;
    for (int k = 0; k < B; ++k) {
        uint32_t o = (uint32_t)k * npix + pix;
        float v = MODE == kProjGap    ? theta[o]
                : ADMM                ? theta[o] - u[o]
                : MODE == kProjFista ? fista_point(theta[o], u[o], ex)
                                     : twist_point(u[o], theta[o], w[o], ex, a1, a2);
        acc = fmaf(C[o], v, acc);
    }
    float r = (Y[pix] - acc) * Sinv[pix];
    for (int k = 0; k < B; ++k) {
        uint32_t o = (uint32_t)k * npix + pix;
        float v = MODE == kProjGap    ? theta[o]
                : ADMM                ? theta[o] - u[o]
                : MODE == kProjFista ? fista_point(theta[o], u[o], ex)
                                     : twist_point(u[o], theta[o], w[o], ex, a1, a2);
        float xv = fmaf(C[o], r, v);
        if (!ADMM || x) x[o] = xv;
        if (ADMM) svol[o] = u[o] + xv;
        if (MODE == kProjTwist) svol[o] = v;
    }
}

// The projection with every frame of a pixel in registers (B <= KB <= 32), so
// that each volume is read once. HBM stream (GAP: read theta, write x); below
// a few million voxels its time is the latency of its loads. All of them are
// issued before the first use: every slot k < KB loads unconditionally (a slot
// past the last frame repeats frame B - 1 and drops out of the sum). A test of
// k < B around each load puts the load and its use in a basic block of their
// own, and the frames then come in one latency after another: with that, GAP
// took 5.1 / 10.3 / 39.6 us inside a solve at 256x256x8 / 512x512x10 /
// 1024x1024x24 (5.1 TB/s), without it 3.3 / 5.8 / 32.4 us (6.2 TB/s; back to
// back 2.6 / 4.1 / 27.1 us). One pixel per thread and one wavefront per
// workgroup were as fast as any other split up to 512x512x24 and faster at
// 1024x1024x24 (256 threads 30.1 us back to back, two pixels per thread 28.4
// to 33.0 us): the finest grain leaves the shortest last round. Workgroups are
// numbered XCD-contiguously, so that an XCD projects the band of rows whose
// theta the row-major denoisers (VTV) left in its L2: 8.6 -> 5.8 us at
// 512x512x10.
//
// Binary masks come as packed bits (flags[block] != 0, see k_setup_reg): C_k is
// 0 or 1, so fmaf(C_k, v, acc) and fmaf(C_k, r, v) give the same values as with
// the float masks, which are read where the block's flag is 0.
template <int MODE, int KB>
__global__ __launch_bounds__(kProjBlock) void k_project_reg(uint32_t npix, int B, float ex, float a1, float a2,
                                                            const float *__restrict__ w,
                                                            const float *__restrict__ theta,
                                                            const float *__restrict__ u, const float *__restrict__ C,
                                                            const uint32_t *__restrict__ bits,
                                                            const int *__restrict__ flags,
                                                            const float *__restrict__ Y,
                                                            const float *__restrict__ Sinv, float *__restrict__ x,
                                                            float *__restrict__ svol)
{
    const int block = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const uint32_t pix = (uint32_t)block * kProjBlock + threadIdx.x;
    if (pix >= npix) return;
    constexpr bool ADMM = MODE == kProjAdmm;
    float v[KB], uu[KB], ww[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const uint32_t o = (uint32_t)min(k, B - 1) * npix + pix;
        v[k] = theta[o];
        if (MODE != kProjGap) uu[k] = u[o];
        if (MODE == kProjTwist) ww[k] = w[o];
    }
    const uint32_t m = bits[pix];
    const float yv = Y[pix], sv = Sinv[pix];
    // the rest, with C_k from cof(k)
    auto finish = [&](auto cof) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (ADMM) v[k] = v[k] - uu[k];
            else if (MODE == kProjFista) v[k] = fista_point(v[k], uu[k], ex);
            else if (MODE == kProjTwist) v[k] = twist_point(uu[k], v[k], ww[k], ex, a1, a2);
            if (k < B) acc = fmaf(cof(k), v[k], acc);
        }
        const float r = (yv - acc) * sv;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            if (k < B) {
                const uint32_t o = (uint32_t)k * npix + pix;
                const float xv = fmaf(cof(k), r, v[k]);
                if (!ADMM || x) x[o] = xv;
                if (ADMM) svol[o] = uu[k] + xv;
                if (MODE == kProjTwist) svol[o] = v[k];
            }
        }
    };
    if (flags[block] != 0) { // uniform over the workgroup
        finish([&](int k) { return (m >> k) & 1u ? 1.0f : 0.0f; });
    } else {
        float c[KB];
#pragma unroll
        for (int k = 0; k < KB; ++k) c[k] = C[(uint32_t)min(k, B - 1) * npix + pix];
        finish([&](int k) { return c[k]; });
    }
}

struct ProjArgs {
    uint32_t npix;
    int B;
    float ex, a1, a2;
    const float *w, *theta, *u, *C;
    const uint32_t *bits;
    const int *flags;
    const float *Y, *Sinv;
    float *x, *svol;
    hipStream_t s;
};

template <int MODE> void launch_project_reg(const ProjArgs &a)
{
    with_slots(a.B, [&](auto kb) {
        hipLaunchKernelGGL((k_project_reg<MODE, decltype(kb)::value>), proj_grid(a.npix), dim3(kProjBlock), 0, a.s, a.npix,
                           a.B, a.ex, a.a1, a.a2, a.w, a.theta, a.u, a.C, a.bits, a.flags, a.Y, a.Sinv, a.x, a.svol);
    });
}

// At most 32 frames, as many as a mask word has bits: registers; beyond, the
// loop over frames.
template <int MODE>
void launch_project(uint32_t npix, int B, float ex, const float *theta, const float *u, const float *C,
                    const float *Y, const float *Sinv, float *x, float *svol, hipStream_t s, const uint32_t *cbits,
                    const int *cflags, float a1 = 0.0f, float a2 = 0.0f, const float *w = nullptr)
{
    if (B <= 32)
        launch_project_reg<MODE>(ProjArgs{npix, B, ex, a1, a2, w, theta, u, C, cbits, cflags, Y, Sinv, x, svol, s});
    else
        hipLaunchKernelGGL((k_project<MODE>), dim3(grid_for(npix)), dim3(kBlock), 0, s, npix, B, ex, a1, a2, w, theta,
                           u, C, Y, Sinv, x, svol);
}

__global__ __launch_bounds__(kBlock) void k_copy4(uint32_t n4, const uint32_t *__restrict__ src,
                                                  uint32_t *__restrict__ dst)
{
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n4) dst[i] = src[i];
}

__global__ __launch_bounds__(kBlock) void k_copy1(uint32_t n, const uint8_t *__restrict__ src,
                                                  uint8_t *__restrict__ dst)
{
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ __launch_bounds__(kBlock) void k_zero4(uint32_t n4, uint32_t *__restrict__ dst)
{
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n4) dst[i] = 0u;
}

__global__ __launch_bounds__(kBlock) void k_zero1(uint32_t n, uint8_t *__restrict__ dst)
{
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dst[i] = 0;
}

__global__ __launch_bounds__(kBlock) void k_fill(uint32_t n, float v, float *__restrict__ dst)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dst[i] = v;
}

// FISTA extrapolation theta = x + c (x - x_prev).
__global__ __launch_bounds__(kBlock) void k_extrapolate(uint32_t n, float c, const float *__restrict__ x,
                                                        const float *__restrict__ xp, float *__restrict__ th)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const float xv = x[i];
    th[i] = fmaf(c, xv - xp[i], xv);
}

// TwIST two-step update out = a0 x_prev + a1 x + a2 theta.
__global__ __launch_bounds__(kBlock) void k_two_step(uint32_t n, float a0, float a1, float a2,
                                                     const float *__restrict__ xp, const float *__restrict__ x,
                                                     const float *__restrict__ th, float *__restrict__ out)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    out[i] = fmaf(a2, th[i], fmaf(a1, x[i], a0 * xp[i]));
}

} // namespace

void launch_fill(float *dst, float v, size_t n, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n)), dim3(kBlock), 0, s, (uint32_t)n, v, dst);
}

void launch_extrapolate(size_t n, float c, const float *x, const float *xp, float *th, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_extrapolate, dim3(grid_for(n)), dim3(kBlock), 0, s, (uint32_t)n, c, x, xp, th);
}

void launch_two_step(size_t n, float a0, float a1, float a2, const float *xp, const float *x, const float *th,
                     float *out, hipStream_t s)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_two_step, dim3(grid_for(n)), dim3(kBlock), 0, s, (uint32_t)n, a0, a1, a2, xp, x, th, out);
}

void launch_forward(int nx, int ny, int B, const float *C, const float *X, float *Y, hipStream_t s)
{
    uint32_t npix = (uint32_t)nx * (uint32_t)ny;
    hipLaunchKernelGGL(k_forward, dim3(grid_for(npix)), dim3(kBlock), 0, s, npix, B, C, X, Y);
}

void launch_adjoint(int nx, int ny, int B, const float *C, const float *Y, float *X, hipStream_t s)
{
    uint32_t npix = (uint32_t)nx * (uint32_t)ny;
    hipLaunchKernelGGL(k_adjoint, dim3(grid_for(npix)), dim3(kBlock), 0, s, npix, B, C, Y, X);
}

size_t mask_flags_count(size_t npix) { return (npix + kProjBlock - 1) / kProjBlock; }

void launch_setup(int nx, int ny, int B, const float *C, const float *Y, float rho, float *Sinv, float *theta, float *u,
                  uint32_t *bits, int *flags, hipStream_t s)
{
    const uint32_t npix = (uint32_t)nx * (uint32_t)ny;
    if (B > 32) { // no packed masks: the projection loops over the frames
        if (Sinv) hipLaunchKernelGGL(k_weights, dim3(grid_for(npix)), dim3(kBlock), 0, s, npix, B, C, rho, Sinv);
        if (theta) launch_adjoint(nx, ny, B, C, Y, theta, s);
        if (u) launch_zero(u, (size_t)npix * B * sizeof(float), s);
        return;
    }
    with_slots(B, [&](auto kb) {
        hipLaunchKernelGGL(k_setup_reg<decltype(kb)::value>, proj_grid(npix), dim3(kProjBlock), 0, s, npix, B, C, Y, rho,
                           Sinv, theta, u, bits, flags);
    });
}

void launch_gap_project(int nx, int ny, int B, const float *theta, const float *C, const float *Y,
                        const float *Sinv, float *x, hipStream_t s, const uint32_t *cbits, const int *cflags)
{
    launch_project<kProjGap>((uint32_t)nx * (uint32_t)ny, B, 0.0f, theta, nullptr, C, Y, Sinv, x, nullptr, s, cbits,
                             cflags);
}

void launch_admm_project(int nx, int ny, int B, const float *theta, const float *u, const float *C,
                         const float *Y, const float *Sinv, float *x, float *svol, hipStream_t s,
                         const uint32_t *cbits, const int *cflags)
{
    launch_project<kProjAdmm>((uint32_t)nx * (uint32_t)ny, B, 0.0f, theta, u, C, Y, Sinv, x, svol, s, cbits, cflags);
}

void launch_fista_project(int nx, int ny, int B, const float *x, const float *x_prev, float ex, const float *C,
                          const float *Y, const float *W, float *z, hipStream_t s, const uint32_t *cbits,
                          const int *cflags)
{
    launch_project<kProjFista>((uint32_t)nx * (uint32_t)ny, B, ex, x, x_prev, C, Y, W, z, nullptr, s, cbits, cflags);
}

void launch_twist_project(int nx, int ny, int B, const float *x, const float *x_prev, const float *theta, float a0,
                          float a1, float a2, const float *C, const float *Y, const float *W, float *z, float *x_next,
                          hipStream_t s, const uint32_t *cbits, const int *cflags)
{
    launch_project<kProjTwist>((uint32_t)nx * (uint32_t)ny, B, a0, x, x_prev, C, Y, W, z, x_next, s, cbits, cflags, a1,
                               a2, theta);
}

// Device-to-device copy and zero fill as plain kernels, so that they can be
// captured into HIP graphs (no memset / memcpy nodes).
void launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return;
    if ((bytes & 3) == 0 && ((uintptr_t)src & 3) == 0 && ((uintptr_t)dst & 3) == 0) {
        uint32_t n4 = (uint32_t)(bytes / 4);
        hipLaunchKernelGGL(k_copy4, dim3(grid_for(n4)), dim3(kBlock), 0, s, n4, (const uint32_t *)src,
                           (uint32_t *)dst);
    } else {
        hipLaunchKernelGGL(k_copy1, dim3(grid_for(bytes)), dim3(kBlock), 0, s, (uint32_t)bytes,
                           (const uint8_t *)src, (uint8_t *)dst);
    }
}

void launch_zero(void *dst, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return;
    if ((bytes & 3) == 0 && ((uintptr_t)dst & 3) == 0) {
        uint32_t n4 = (uint32_t)(bytes / 4);
        hipLaunchKernelGGL(k_zero4, dim3(grid_for(n4)), dim3(kBlock), 0, s, n4, (uint32_t *)dst);
    } else {
        hipLaunchKernelGGL(k_zero1, dim3(grid_for(bytes)), dim3(kBlock), 0, s, (uint32_t)bytes, (uint8_t *)dst);
    }
}

} // namespace sci
