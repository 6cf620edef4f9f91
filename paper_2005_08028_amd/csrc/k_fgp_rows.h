// Row-pipelined fused-schedule TV denoiser kernel (template), instantiated in
// the k_fgp_rows_*.hip translation units; its body also serves the batched
// launch (k_batched.hip).
//
// The same M FGP iterations per pass over HBM as the tiled kernel
// (Algorithm 1, FGP box; projections of Eq. (29)-(30)), decomposed by
// temporal wavefront blocking (Wellein et al., "Efficient temporal blocking
// for stencil computations by multicore-aware wavefront parallelization",
// COMPSAC 2009) instead of overlapped 2D tiles. One wavefront owns a strip of
// 64*C columns of one frame (C adjacent columns per lane; a recomputed halo of
// M+1 columns on the left and M on the right, as in the tiles) and a segment
// of H rows, and walks the segment from top to bottom. Iteration level t
// (0 <= t < M) trails level t-1 by one row: in step k, level t is on row
// r = k - t; it takes w_t and p_t of row r+1, just produced by level t-1 in
// the same step, forms theta_t of row r+1, and with its own theta_t, w_t, p_t
// of row r (kept from the previous step) produces p_{t+1} and w_{t+1} of
// row r for level t+1. All levels of a column live in the lane's registers,
// so rows are recomputed only in the pipeline fill above a segment
// (M+2 rows) and below it (M rows), and no workgroup barrier is needed:
// vertical neighbours are earlier steps of the same lane and horizontal ones
// come from DPP shifts. x of the last rows sits in a ring in LDS private to
// the wavefront, written twice so that every level reads it at a fixed
// offset.
//
// Pixels outside the image hold x = p = 0 and, with the step set to 0 on
// every dual entry that carries no difference, keep p = 0: the zero padding
// of the difference operators. Rows a level computes before the fill has
// reached it hold meaningless values that never enter a stored result (each
// stored value depends only on rows inside its dependency cone). The
// per-voxel arithmetic is that of the streaming and tiled kernels (same
// helpers, same operand order, no contraction), so results are
// bit-identical to theirs with float32 dual storage.
//
// What bounds it: vector instruction issue (17 per voxel-iteration for ITV2D,
// v_rsq_f32 taking two slots), two wavefronts per SIMD. A cold 10-iteration
// ITV2D pass at 1024x1024x24 (128-row segments, 1,920 wavefronts) takes 169 us;
// three things brought it there from 189 us (their figures without the case of
// a NaN norm, which adds 3 us):
//   * The SIMD serves the older of its two wavefronts first. That one then
//     runs as if alone (119 us) and the other is left to finish alone (185
//     us), with the vector unit 70 % busy to the end. A priority that falls
//     along each chunk of rows lets the one behind catch up: both end
//     together, 187 -> 166 us (one change per chunk 171, none but a quarter
//     of the segment 177).
//   * Rows are read and written as bounded buffers (RowBuf): no masks, no
//     vector addresses (748 -> 687 vector instructions per chunk).
//   * The loads of a chunk are issued at its start and waited for at its end
//     before the last stores, instead of behind them (200 -> 187 us).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "k_fgp_tile_shapes.h"
#include "sci_internal.h"
#include "sci_math.h"

namespace sci {

constexpr int kRowChunk = 2; // rows loaded per chunk (one chunk ahead)

// f(integral_constant<int, I>) for I = I0 .. N-1, unrolled at compile time.
template <int I0, int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I0 < N) {
        f(std::integral_constant<int, I0>{});
        static_for<I0 + 1, N>(f);
    }
}

// LDS ring of rows (x, or starting duals) private to one wavefront.
template <int M, int C> struct alignas(16) RowRing {
    float v[2 * (M + kRowChunk)][64 * C];
};

// The ring padded to 1/8 of a CU's 160 KB of LDS.
template <int M, int C> struct alignas(16) RowRingPadded {
    static constexpr size_t kEighth = 160 * 1024 / 8;
    RowRing<M, C> ring;
    char pad[sizeof(RowRing<M, C>) < kEighth ? kEighth - sizeof(RowRing<M, C>) : 16];
};

// One wavefront's segment: strip sx, segment seg (rows [seg*H, seg*H + H)) of
// the frame at element offset fo; V = elements per dual channel of the whole
// video. MODE: 0 w = 0; 1 w = p^(s0); 2 w = p^(s0) + b[0] (p^(s0) - p^(s0-1)).
// CH_STEP = 1 replaces the projection of q by Chambolle's (2004) semi-implicit step
// p = (w + z/(8 lambda)) / (1 + |z/(8 lambda)|), |.| per component (ATV) or
// per voxel (ITV2D), with the operations of the streaming pass.
// MOM = 0 (no momentum: every beta of the pass is 0, MODE < 2, no p_prev
// output) takes w = p at every level; the extrapolation and the previous
// duals it would read drop out, with identical results.
template <int TV, int M, int DT, int C, int MODE, int CH_STEP = 0, int MOM = 1>
__device__ __forceinline__ void fgp_rows_body(int nx, int ny, int sx, int seg, int H, uint32_t fo, uint32_t V,
                                              const float *__restrict__ x,
                                              const typename Dual<DT>::T *__restrict__ pc,
                                              const typename Dual<DT>::T *__restrict__ pp, const TileBeta &bt,
                                              float lam, float step, typename Dual<DT>::T *__restrict__ pn_out,
                                              typename Dual<DT>::T *__restrict__ pp_out,
                                              float *__restrict__ theta_out, float *__restrict__ u_out,
                                              RowRing<M, C> &rr)
{
    using T = typename Dual<DT>::T;
    constexpr int CH = kRowChunk;
    constexpr int TW = 64 * C;
    constexpr int TXO = TW - 2 * M - 1; // interior columns per strip
    constexpr int P = M + CH;           // ring period: rows k+1-M .. k+1 and the chunk written ahead
    static_assert(TXO > 0, "strip too narrow for the pass length");
    auto &ring = rr.v;

    const int lane = threadIdx.x & 63;
    const int a = seg * H;               // first row of the segment
    const int hi = min(a + H, nx);       // one past its last row
    const int j0 = sx * TXO - (M + 1) + lane * C;

    // the strip's columns inside the image: jb .. jb + ncol, of which the first
    // nhor carry a horizontal difference
    const int jb = max(sx * TXO - (M + 1), 0);
    const uint32_t ncol = (uint32_t)min(ny - jb, TW), nhor = (uint32_t)min(ny - 1 - jb, TW);
    float step_h[C];
    uint32_t off_in[C], off_out[C]; // columns loaded and stored, from jb, in elements; kNoColumn: none
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int j = j0 + c;
        const bool hj = j >= 0 && j < ny - 1; // horizontal differences exist for 0 <= j < ny-1
        step_h[c] = hj ? step : 0.0f;
        off_in[c] = j >= jb && j < ny ? (uint32_t)(j - jb) : kNoColumn;
        const int cw = lane * C + c;
        off_out[c] = cw >= M + 1 && cw <= TW - 1 - M && j < ny ? (uint32_t)(j - jb) : kNoColumn;
    }
    static_assert(DT == DT_F32, "16-bit duals run the tiles");
    constexpr uint32_t SZ = (uint32_t)sizeof(T);
#pragma unroll
    for (int s = 0; s < 2 * P; ++s)
#pragma unroll
        for (int c = 0; c < C; ++c) ring[s][lane * C + c] = 0.0f;

    // level t's state on its current row r: theta_t(r), w_t(r), p_t(r)
    float cth[M][C], cwh[M][C], cwv[M][C], cph[M][C], cpv[M][C];
#pragma unroll
    for (int t = 0; t < M; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) cth[t][c] = cwh[t][c] = cwv[t][c] = cph[t][c] = cpv[t][c] = 0.0f;
    float cpm[C]; // p_v^(s0+M) of the row above the theta row
#pragma unroll
    for (int c = 0; c < C; ++c) cpm[c] = 0.0f;

    // Chunk loads: x and (MODE >= 1) the starting duals of CH rows. Pixels
    // outside the image and dual entries that carry no difference (column
    // ny-1 of the horizontal channel, row nx-1 of the vertical one) lie
    // outside their row's buffer and come back as 0.
    float xn[CH][C], lh[CH][C], lv[CH][C], mh[CH][C], mv[CH][C];
    auto load_chunk = [&](int i0) {
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int i = i0 + s;
            const bool iin = i >= 0 && i < nx;
            const uint32_t rowo = fo + (iin ? (uint32_t)i : 0u) * (uint32_t)ny + (uint32_t)jb;
            const uint32_t nh = iin ? nhor : 0u;                                // entries of p_h
            const uint32_t nv = (uint32_t)i < (uint32_t)(nx - 1) ? ncol : 0u;   // and of p_v
            const RowBuf xb = row_buf(x + rowo, iin ? ncol * 4u : 0u);
#pragma unroll
            for (int c = 0; c < C; ++c) xn[s][c] = row_ld(xb, off_in[c] * 4u);
            if (MODE >= 1) {
                const RowBuf hb = row_buf(pc + rowo, nh * SZ), vb = row_buf(pc + (size_t)V + rowo, nv * SZ);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    lh[s][c] = row_ld(hb, off_in[c] * SZ);
                    lv[s][c] = row_ld(vb, off_in[c] * SZ);
                }
            }
            if (MODE == 2) {
                const RowBuf hb = row_buf(pp + rowo, nh * SZ), vb = row_buf(pp + (size_t)V + rowo, nv * SZ);
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    mh[s][c] = row_ld(hb, off_in[c] * SZ);
                    mv[s][c] = row_ld(vb, off_in[c] * SZ);
                }
            }
        }
    };

    // Step k runs level t on row k - t. The first stored row a needs level 0
    // from row a - M, primed two steps earlier (theta_0 and w_0 of the row
    // above); the last stored row a+H-1 leaves level M-1 at step a+H+M-2.
    //
    // Relative to k_start, level t first matters at step 2t (it takes in w_t
    // of the row that primes its theta); the first NPRO chunks, where some
    // level is still idle, are unrolled with those levels and the theta
    // stage (whose rows lie above the segment there) left out. Every later
    // chunk runs all levels.
    const int k_start = a - M - 2;
    const int nsteps = H + 2 * M + 1;
    const int nchunk = (nsteps + CH - 1) / CH; // >= M + 1 > NPRO
    constexpr int NPRO = (2 * (M - 1) + CH - 1) / CH;
    // Cold ITV2D passes take the scale without a NaN case up to the first chunk
    // that has a pixel beyond the limit. 1024x1024x24, 10 iterations: 176.8 us
    // with iso_scale throughout, 167.4 like this; 5 iterations 82.3 and 79.0.
    constexpr bool TAME = MODE == 0 && TV != TV_ATV && !CH_STEP;
    const float limit = no_nan_limit(lam);
    uint64_t tame = ~0ull; // lanes, ANDed as masks: no branch
    // The rows loaded during a chunk go to the ring (and are waited for) at its
    // end, before its last stores: a wait further on would wait for those
    // stores too, which vmcnt counts with the loads. (Not the duals of a warm
    // momentum pass of 10: held that much longer, ATV needs two to four of its
    // 256 registers more and spills.)
    constexpr bool SETTLE = MODE < 2 || M < kTileMaxM;
    auto settle_chunk = [&](int i0) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TAME) {
#pragma unroll
            for (int s = 0; s < CH; ++s)
#pragma unroll
                for (int c = 0; c < C; ++c) tame &= __ballot(fabsf(xn[s][c]) <= limit);
        }
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int slot = (((i0 + s) % P) + P) % P;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (MODE >= 1 && SETTLE) {
                    settle(lh[s][c]);
                    settle(lv[s][c]);
                }
                if (MODE == 2 && SETTLE) {
                    settle(mh[s][c]);
                    settle(mv[s][c]);
                }
                ring[slot][lane * C + c] = xn[s][c];
                ring[slot + P][lane * C + c] = xn[s][c];
            }
        }
    };
    load_chunk(k_start + 1);
    settle_chunk(k_start + 1);
    auto chunk = [&](int b, auto pro, auto no_nan) {
        constexpr int PB = decltype(pro)::value;  // prologue chunk index, or -1
        constexpr bool NN = decltype(no_nan)::value; // no norm of the chunk is NaN
        const int k0 = k_start + b * CH;
        // level-0 inputs of the chunk's rows k0+1 .. k0+CH
        float i0h[CH][C], i0v[CH][C], j0h[CH][C], j0v[CH][C];
#pragma unroll
        for (int s = 0; s < CH; ++s) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (MODE == 0) {
                    i0h[s][c] = i0v[s][c] = j0h[s][c] = j0v[s][c] = 0.0f;
                } else {
                    j0h[s][c] = lh[s][c];
                    j0v[s][c] = lv[s][c];
                    i0h[s][c] = MODE == 2 ? extrapolate(lh[s][c], mh[s][c], bt.b[0]) : lh[s][c];
                    i0v[s][c] = MODE == 2 ? extrapolate(lv[s][c], mv[s][c], bt.b[0]) : lv[s][c];
                }
            }
        }
        load_chunk(k0 + CH + 1);
        issued();
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int k = k0 + s;
            const int base = (((k + 1) % P) + P) % P + P; // x(k+1) in the second copy; x(k+1-t) at base - t
            // inputs of level t: w_t, p_t of row k - t + 1
            float ih[C], iv[C], jh[C], jv[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                ih[c] = i0h[s][c];
                iv[c] = i0v[s][c];
                jh[c] = j0h[s][c];
                jv[c] = j0v[s][c];
            }
            float qph[C], qpv[C]; // p^(s0+M-1) of the output row
#pragma unroll
            for (int t = 0; t < M; ++t) {
                if (PB >= 0 && PB * CH + s < 2 * t) break; // this level and the later ones are idle
                // priority falls along a chunk, half a step at a time (see the
                // header comment): the co-resident wavefront that is behind in
                // its chunk goes first
                if (t == 0) {
                    if (s == 0) __builtin_amdgcn_s_setprio(3);
                    else __builtin_amdgcn_s_setprio(1);
                }
                if (t == M / 2) {
                    if (s == 0) __builtin_amdgcn_s_setprio(2);
                    else __builtin_amdgcn_s_setprio(0);
                }
                const int r = k - t;
                // theta_t of row r+1 = x - lambda D^T w_t
                float thn[C];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float whl = c > 0 ? ih[c - 1] : from_left(ih[C - 1]);
                    thn[c] = theta_of(ring[base - t][lane * C + c], whl, ih[c], cwv[t][c], iv[c], lam);
                }
                const float step_v = row_step(r, nx, step);
                const float bnext = bt.b[t + 1];
                float oh[C], ov[C], nh[C], nv[C];
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const float thr = c < C - 1 ? cth[t][c + 1] : from_right(cth[t][0]);
                    const float zh = thr - cth[t][c];
                    const float zv = thn[c] - cth[t][c];
                    if (CH_STEP) {
                        const float sh = step_h[c] * zh, sv = step_v * zv;
                        const float qh = cwh[t][c] + sh, qv = cwv[t][c] + sv;
                        if (TV == TV_ATV) {
                            nh[c] = semi_implicit_atv(qh, sh);
                            nv[c] = semi_implicit_atv(qv, sv);
                        } else {
                            const float s1 = semi_implicit_scale(norm2_add(0.0f, sh, sv));
                            nh[c] = qh * s1;
                            nv[c] = qv * s1;
                        }
                    } else {
                        const float qh = ascend(cwh[t][c], zh, step_h[c]);
                        const float qv = ascend(cwv[t][c], zv, step_v);
                        if (TV == TV_ATV) {
                            nh[c] = proj_atv(qh);
                            nv[c] = proj_atv(qv);
                        } else {
                            const float n2 = norm2_add(0.0f, qh, qv);
                            const float sc = NN ? iso_scale_no_nan(n2) : iso_scale(n2);
                            nh[c] = qh * sc;
                            nv[c] = qv * sc;
                        }
                    }
                    if (MOM) {
                        oh[c] = extrapolate(nh[c], cph[t][c], bnext);
                        ov[c] = extrapolate(nv[c], cpv[t][c], bnext);
                    } else {
                        oh[c] = nh[c];
                        ov[c] = nv[c];
                    }
                }
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if (t == M - 1) {
                        qph[c] = cph[t][c];
                        qpv[c] = cpv[t][c];
                    }
                    cth[t][c] = thn[c];
                    cwh[t][c] = ih[c];
                    cwv[t][c] = iv[c];
                    cph[t][c] = jh[c];
                    cpv[t][c] = jv[c];
                    ih[c] = oh[c];
                    iv[c] = ov[c];
                    jh[c] = nh[c];
                    jv[c] = nv[c];
                }
            }
            if (PB >= 0) { // the theta row is above the segment
                if (s == CH - 1) settle_chunk(k0 + CH + 1);
                continue;
            }
            // row r = k - M + 1 now has p^(s0+M) in jh, jv: theta = x - lambda D^T p
            const int r = k - M + 1;
            float th[C], xr[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float phl = c > 0 ? jh[c - 1] : from_left(jh[C - 1]);
                xr[c] = ring[base - M][lane * C + c];
                th[c] = theta_of(xr[c], phl, jh[c], cpm[c], jv[c], lam);
                cpm[c] = jv[c];
            }
            if (s == CH - 1) settle_chunk(k0 + CH + 1);
            if (r >= a && r < hi) { // uniform
                const uint32_t rowo = fo + (uint32_t)r * (uint32_t)ny + (uint32_t)jb;
                auto put = [&](float *out, const float(&v)[C]) {
                    const RowBuf b = row_buf(out + rowo, ncol * 4u);
#pragma unroll
                    for (int c = 0; c < C; ++c) row_st(b, off_out[c] * 4u, v[c]);
                };
                auto put_dual = [&](T *out, const float(&h)[C], const float(&v)[C]) {
                    const RowBuf hb = row_buf(out + rowo, ncol * SZ);
                    const RowBuf vb = row_buf(out + (size_t)V + rowo, ncol * SZ);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        row_st(hb, off_out[c] * SZ, h[c]);
                        row_st(vb, off_out[c] * SZ, v[c]);
                    }
                };
                if (theta_out) put(theta_out, th);
                if (u_out) {
                    float uu[C];
#pragma unroll
                    for (int c = 0; c < C; ++c) uu[c] = xr[c] - th[c];
                    put(u_out, uu);
                }
                if (pn_out) put_dual(pn_out, jh, jv);
                if (MOM && pp_out) put_dual(pp_out, qph, qpv);
            }
        }
    };
    static_for<0, NPRO>([&](auto pb) { chunk(decltype(pb)::value, pb, std::false_type{}); });
    int b = NPRO;
    if constexpr (TAME)
        for (; b < nchunk && tame == ~0ull; ++b) chunk(b, std::integral_constant<int, -1>{}, std::true_type{});
    for (; b < nchunk; ++b) chunk(b, std::integral_constant<int, -1>{}, std::false_type{});
}

// One pass over every frame: a one-wavefront workgroup per (frame, segment,
// strip), numbered XCD-contiguously.
template <int TV, int M, int DT, int C, int MODE, int CH_STEP, int MOM>
__global__ __launch_bounds__(64, 2) void k_fgp_rows(int nx, int ny, int nstrip, int nseg, int H,
                                                    const float *__restrict__ x,
                                                    const typename Dual<DT>::T *__restrict__ pc,
                                                    const typename Dual<DT>::T *__restrict__ pp, TileBeta bt,
                                                    float lam, float step, typename Dual<DT>::T *__restrict__ pn_out,
                                                    typename Dual<DT>::T *__restrict__ pp_out,
                                                    float *__restrict__ theta_out, float *__restrict__ u_out)
{
    const int lin = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    const int per_frame = nstrip * nseg;
    const int frame = lin / per_frame, rem = lin % per_frame;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    auto body = [&](RowRing<M, C> &ring) {
        fgp_rows_body<TV, M, DT, C, MODE, CH_STEP, MOM>(nx, ny, rem % nstrip, rem / nstrip, H,
                                                        (uint32_t)frame * plane,
                                                        plane * (gridDim.x / (uint32_t)per_frame), x, pc, pp, bt, lam,
                                                        step, pn_out, pp_out, theta_out, u_out, ring);
    };
    if constexpr (MOM) {
        __shared__ RowRing<M, C> ring;
        body(ring);
    } else {
        // The momentum-free kernel needs few enough registers for three
        // wavefronts per SIMD; its one-wavefront workgroups then spread
        // unevenly over the SIMDs (some run three: 309 against 238 us for a
        // 10-iteration ITV2D pass at 1024x1024x24 inside GAP), so its LDS is
        // padded to admit at most eight workgroups (two wavefronts per SIMD)
        // per CU. The asm keeps the unused padding allocated.
        __shared__ RowRingPadded<M, C> lds;
        asm volatile("; lds padding %0" ::"v"((uint32_t)(size_t)&lds.pad[0]));
        body(lds.ring);
    }
}

// Launch of one pass over every frame: strips of 64*C - 2M - 1 interior
// columns, segments of H rows. The Chambolle-2004 step without momentum
// runs the MOM = 0 instantiation.
template <int TV, int M, int DT, int C, int CH_STEP>
void launch_rows_m(int H, int nx, int ny, int B, const float *x, const TilePass &tp, float lam, hipStream_t s)
{
    using T = typename Dual<DT>::T;
    constexpr int TXO = 64 * C - 2 * M - 1;
    const int nstrip = (ny + TXO - 1) / TXO, nseg = (nx + H - 1) / H;
    const dim3 g(nstrip * nseg * B), b(64);
    const float step = 1.0f / (8.0f * lam);
    bool mom = tp.mode == 2 || tp.pp_out != nullptr;
    for (int t = 1; t <= M; ++t) mom = mom || tp.beta.b[t] != 0.0f;
#define SCI_ROWS_MODE(md, mo)                                                                                       \
    hipLaunchKernelGGL((k_fgp_rows<TV, M, DT, C, md, CH_STEP, mo>), g, b, 0, s, nx, ny, nstrip, nseg, H, x,          \
                       (const T *)tp.pc, (const T *)tp.pp, tp.beta, lam, step, (T *)tp.pn_out, (T *)tp.pp_out,      \
                       tp.theta, tp.u_out)
    if (CH_STEP && !mom) {
        if (tp.mode == 0) SCI_ROWS_MODE(0, 0);
        else SCI_ROWS_MODE(1, 0);
    } else if (tp.mode == 0) SCI_ROWS_MODE(0, 1);
    else if (tp.mode == 1) SCI_ROWS_MODE(1, 1);
    else SCI_ROWS_MODE(2, 1);
#undef SCI_ROWS_MODE
}

// Dispatch on the pass length m = 1..kTileMaxM.
template <int TV, int DT, int CH_STEP = 0>
int launch_rows(int H, int m, int nx, int ny, int B, const float *x, const TilePass &tp, float lam, hipStream_t s)
{
    static_assert(kTileMaxM == 10, "pass lengths dispatched below");
    constexpr int C = kRowCols;
    switch (m) {
    case 1: launch_rows_m<TV, 1, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 2: launch_rows_m<TV, 2, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 3: launch_rows_m<TV, 3, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 4: launch_rows_m<TV, 4, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 5: launch_rows_m<TV, 5, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 6: launch_rows_m<TV, 6, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 7: launch_rows_m<TV, 7, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 8: launch_rows_m<TV, 8, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 9: launch_rows_m<TV, 9, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    case 10: launch_rows_m<TV, 10, DT, C, CH_STEP>(H, nx, ny, B, x, tp, lam, s); return SCI_OK;
    }
    return SCI_ERR_INVALID_ARG;
}

} // namespace sci
