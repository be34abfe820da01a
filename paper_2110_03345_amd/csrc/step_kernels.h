// HIP kernels for gfx950 (CDNA4): leapfrog step of the acoustic wave
// equation with a 2r-order Laplacian and a sponge layer, fused with point
// injection, point sampling and (adjoint variant) the imaging condition.
//
// Forward (paper Sec. 2.4, constant density, no attenuation; second order in
// time):   C = a (2 A + k (L A + S)) - b B,          a = b = 1 outside the sponge
// Adjoint (exact transpose, Sec. 2.2 adjoint PDE):  the same update with
//          A = w^{m+1}, B = w^{m+2}, S = R^T g^m,  plus the imaging term
//          G += w^{m+1} (L u^m + S^m)   (gradient w.r.t. k; Sec. 2.2 reduced
//          gradient <grad_m L* w, dm>).
//
// A step launch is HBM-bound (16 B per forward update, 28 B per adjoint update):
// no MFMA.  Tiles are 64 wide along the contiguous axis; the u^n tile plus its
// halo sits in LDS.  2D: 16 rows, one wave64 per tile row.  3D: a thread owns four
// or two points of a row, a wave as many rows, and each block marches along axis
// 0 over a chunk of planes, keeping the 2r+1 values of its columns in registers
// (2.5D blocking), so that the axis-0 neighbours never touch LDS.
//
// This header holds the step kernels and their launch templates; the
// translation units step2d.hip, step3d_fwd.hip and step3d_adj.hip each
// instantiate one family, so that they compile in parallel.
#pragma once

#include "common.h"

// Implicit contraction is off: every fused multiply-add is written out as
// fmaf, so the arithmetic of a point does not depend on how the compiler
// schedules the surrounding code (any two kernels that evaluate the same
// expressions compute the same bits).
#pragma clang fp contract(off)

#include <type_traits>

namespace stride {
namespace {


constexpr int kXcds = 8;  // MI355X: workgroups go round-robin over 8 XCDs

// Hardware places block b on XCD b % 8.  Map blocks so that each XCD owns a
// contiguous range of logical tiles: neighbouring tiles then share halo rows
// through the same L2.
__device__ __forceinline__ int xcd_logical(int b, int nblk_pad)
{
    int per = nblk_pad / kXcds;
    return (b % kXcds) * per + b / kXcds;
}

// Calls fn(integral_constant<I>) for I = 0..N-1 while it returns true; every
// I is a compile-time constant in the body (used to index register queues).
template <int N, int I = 0, class Fn>
__device__ __forceinline__ void unrolled_while(Fn&& fn)
{
    if constexpr (I < N) {
        if (fn(std::integral_constant<int, I>{}))
            unrolled_while<N, I + 1>(fn);
    }
}

// Raw buffer access (CDNA): a descriptor over [base, base + bytes) returns 0
// for any byte offset at or beyond `bytes`, so loads of points outside the
// grid need no branch: their offset is set beyond any field (0xffffffff for single
// values, kNoByte for vectors), and a plane outside the grid gets bytes = 0.  Third descriptor word of the gfx9 family.
constexpr int kBufWord3 = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const float* base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, bytes, kBufWord3);
}

__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, int byte_off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, byte_off, 0, 0);
}

// Store with the non-temporal policy (results are read back only in a later
// launch): a 32-bit offset into a per-plane descriptor, no 64-bit address.
__device__ __forceinline__ void bstore_nt(__amdgpu_buffer_rsrc_t r, int byte_off, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, byte_off, 0, 2);
}

// The builtin returns the raw 32 bits; reinterpret them (no numeric conversion).
__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t r, int byte_off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0));
}

// Streamed operands (read once per step: u^{n-1}, k, G) are loaded with the
// non-temporal cache policy so they do not evict the stencil field's halo.
#ifndef STRIDE_STREAM_AUX
#define STRIDE_STREAM_AUX 2
#endif
__device__ __forceinline__ float bload_stream(__amdgpu_buffer_rsrc_t r, int byte_off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, STRIDE_STREAM_AUX));
}

__device__ __forceinline__ int layer_depth(int i, int n, int nb)
{
    int hi = n - 1 - nb;
    return i < nb ? nb - i : (i > hi ? i - hi : 0);
}

__device__ __forceinline__ void sample_block(const SampleSet& smp, const float* field, int step,
                                             int sb)
{
    if (sample_lanes(smp.ntap) == 1) {
        const int r = sb * (int)blockDim.x + (int)threadIdx.x;
        if (r >= smp.count)
            return;
        float acc = 0.f;
        const long long base = (long long)r * smp.ntap;
        for (int t = 0; t < smp.ntap; ++t)
            acc = fmaf(smp.w[base + t], field[smp.idx[base + t]], acc);
        float* o = smp.out + (long long)r * smp.out_stride + step;
        *o = smp.accumulate ? fmaf(smp.scale, acc, *o) : smp.scale * acc;
        return;
    }
    // one wave per point: lane l sums taps l, l + 64, ...; then a butterfly
    // reduction over the wave (a fixed order, so results are reproducible)
    const int lane = (int)threadIdx.x & 63;
    const int r = sb * ((int)blockDim.x >> 6) + ((int)threadIdx.x >> 6);
    if (r >= smp.count)
        return;
    const long long base = (long long)r * smp.ntap;
    float acc = 0.f;
    for (int t = lane; t < smp.ntap; t += 64)
        acc = fmaf(smp.w[base + t], field[smp.idx[base + t]], acc);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        acc += __shfl_xor(acc, off, 64);
    if (lane == 0) {
        float* o = smp.out + (long long)r * smp.out_stride + step;
        *o = smp.accumulate ? fmaf(smp.scale, acc, *o) : smp.scale * acc;
    }
}

constexpr float kTwelfth = 1.f / 12.f;

// Leapfrog update with the sponge's damping: a = 1 / (1 + eta dt/2) by the
// hardware reciprocal (within 1 ulp; an IEEE division would cost about ten
// instructions per point, and most waves of a 3D grid touch the sponge).
__device__ __forceinline__ float leapfrog(float ctr, float prev, float kk, float rhs, float eta,
                                          float half_dt)
{
    if (eta == 0.f)
        return fmaf(kk, rhs, fmaf(2.f, ctr, -prev));
    const float a = __builtin_amdgcn_rcpf(fmaf(eta, half_dt, 1.f));
    const float b = fmaf(-eta, half_dt, 1.f) * a;
    return fmaf(a, fmaf(kk, rhs, 2.f * ctr), -(b * prev));
}

// 2D Laplacian at S[0] of an LDS tile with row length LW_.
template <int R, int LW_>
__device__ __forceinline__ float lap2d(const float* S, const StencilCoef& cf)
{
    float ay = 0.f, ax = 0.f;
#pragma unroll
    for (int q = R; q >= 1; --q) {
        ay = fmaf(cf.c[0][q], S[q * LW_] + S[-q * LW_], ay);
        ax = fmaf(cf.c[1][q], S[q] + S[-q], ax);
    }
    return fmaf(cf.c0, S[0], ay + ax);
}

// ----------------------------------------------------------------------- 2D
//
// One block = one 64 x TY tile, TY = WAVES * RY rows (RY per thread).  The
// tile of A (and U) with its R-wide halo is staged in LDS row by row: wave w
// loads tile rows w, w + WAVES, ..., each lane one column and lanes 0..2R-1
// one halo column as well.  Every load of the step is issued up front: the
// point values of B, K (and G), the LDS tile, and the tile's injection
// entries with their signal samples (the entry range comes from a uniform
// table read), so a tile with injected points costs two dependent round trips
// and any other tile one.  Injected values reach their points through a small
// LDS array, used only by tiles that have entries.  The 2D field fits one
// buffer descriptor (at most 2 GiB): offsets of points outside the grid are
// set to 0xffffffff and read 0.

// Signal sample of row `id`: s[step], or with FILT (the fourth-order step's
// source) (s[step-1] + 10 s[step] + s[step+1]) / 12, zero outside the record.
template <bool FILT>
__device__ __forceinline__ float sig_at(const float* sig, int id, int stride, int step)
{
    const float* s = sig + (long long)id * stride;
    if constexpr (!FILT) {
        return s[step];
    } else {
        const float sm = step >= 1 ? s[step - 1] : 0.f;
        const float sp = step + 1 < stride ? s[step + 1] : 0.f;
        return fmaf(10.f, s[step], sm + sp) / 12.f;
    }
}

// Sum of the signals of the point whose first entry is `head` (entry order).
template <bool FILT = false>
__device__ __forceinline__ float tile_point_signal(const TileEntry* ent, TileEntry head,
                                                   const float* sig, int stride, int step)
{
    float v = head.w * sig_at<FILT>(sig, head.id, stride, step);
    for (int k = 1; k < head.run; ++k) {
        const TileEntry e = ent[k];
        v = fmaf(e.w, sig_at<FILT>(sig, e.id, stride, step), v);
    }
    return v;
}

// Output of a step launch at one point (see StepMode).  ctr and lap: centre
// and Laplacian of the stencil field A, with the injected value already added
// except in the adjoint correction, which takes it apart as inj and adds it
// as k inj (A = q = k L w^{m+1}, D = w^{m+1}):
//   w^m = a (2 w^{m+1} + q + (k/12) L q + k inj) - b w^{m+2}.
// uu: the point field D; bb, kk: B and k.
template <int MODE>
constexpr bool kIsMedium = MODE == kMedium || MODE == kMediumY0;

template <bool ADJ, int MODE>
constexpr bool kInjApart = (ADJ && MODE == kCorrect) || kIsMedium<MODE>;

template <bool ADJ, int MODE>
__device__ __forceinline__ float step_out(float ctr, float lap, float inj, float uu, float bb,
                                          float kk, float eta, float half_dt)
{
    if constexpr (MODE == kStep || MODE == kStepV || MODE == kImageV || MODE == kAdjPlain) {
        return leapfrog(ctr, bb, kk, lap, eta, half_dt);
    } else if constexpr (MODE == kPrep) {
        return kk * lap;
    } else {
        float rhs = fmaf(kk * kTwelfth, lap, ctr);
        if constexpr (ADJ)
            rhs = fmaf(kk, inj, rhs);
        return leapfrog(uu, bb, 1.f, rhs, eta, half_dt);
    }
}

// Output of a medium step.  lap = L u, dens = sum_a gamma_a D_a u, inj the
// injected value, lapb = L u^{n-1}, prev = u^{n-1}; at is the attenuation
// field: weighting L u - L u^{n-1} (Y2) or added to the damping (y = 0).
template <bool Y2>
__device__ __forceinline__ float medium_out(float ctr, float lap, float dens, float inj,
                                            float lapb, float prev, float kk, float at, float eta,
                                            float half_dt)
{
    float rhs = lap + dens + inj;
    if constexpr (Y2)
        rhs = fmaf(at, lap - lapb, rhs);
    else
        eta += at;
    return leapfrog(ctr, prev, kk, rhs, eta, half_dt);
}

// Imaging factor of a medium step for the gradient with respect to vp,
// dJ/dvp = (2/vp) sum_n w^{n+1} h^n (stored by the forward when V is given):
//   y = 2:  h = v + (att/2) (L u - L u^{n-1})                (att = beta = 2 alpha0 vp / dt),
//   y = 0:  h = v + (att a dt/4) ((2 u^{n-1} - 2 u) / k - v)  (att = 2 alpha0 vp, a the
//           step's damping factor with the attenuation),
// v the step's right-hand side L u + sum_a gamma_a D_a u + S (+ beta (L u - L u^{n-1})).
template <bool Y2>
__device__ __forceinline__ float medium_h(float ctr, float lap, float dens, float inj, float lapb,
                                          float prev, float kk, float at, float eta, float half_dt)
{
    float v = lap + dens + inj;
    if constexpr (Y2) {
        const float dl = lap - lapb;
        v = fmaf(at, dl, v);
        return fmaf(0.5f * at, dl, v);
    }
    const float a = __builtin_amdgcn_rcpf(fmaf(eta + at, half_dt, 1.f));
    const float du = 2.f * (prev - ctr) / kk;
    return fmaf(at * a * (0.5f * half_dt), du - v, v);
}

// Imaging accumulator update of an adjoint launch.  Second order:
// G += w^{m+1} (L u^m + S^m) with ctr = w^{m+1}, lu = L u^m + S^m.  Fourth
// order accumulates k G, the gradient with respect to k times k:
//   H += p (w + q/12) + (k/12) w L p,   p = k (L u^m + St^m), q = k L w,
// with ctr = q, pc = p, lu = L p and uu = w = w^{m+1}.
template <int MODE>
__device__ __forceinline__ float image_out(float ctr, float pc, float lu, float uu, float kk,
                                           float gg)
{
    if constexpr (MODE == kCorrect)
        return fmaf((kk * kTwelfth) * uu, lu, fmaf(pc, fmaf(ctr, kTwelfth, uu), gg));
    else
        return fmaf(ctr, lu, gg);
}

template <int R, bool ADJ, int RY, int WAVES, int MODE = kStep>
__device__ __forceinline__ void step2d_body(const Dims& d, const StencilCoef& cf,
                                            const SpongeCoef& sp, const StepParams& p,
                                            const LaunchShape& ls, const int b)
{
    constexpr int NT = 64 * WAVES;
    constexpr int TY = WAVES * RY;
    constexpr int LW = kTileX + 2 * R;
    constexpr int LH = TY + 2 * R;
    constexpr int RW = (LH + WAVES - 1) / WAVES;    // tile rows loaded per wave
    constexpr bool MED = kIsMedium<MODE>;
    constexpr bool MED2 = MODE == kMedium;          // B a stencil field
    constexpr bool ONE = MODE == kImageV || MODE == kAdjPlain;      // adjoint with one stencil field
    constexpr int NF = (ADJ && !ONE) || MED2 ? 2 : 1;  // stencil fields A (and U, or B)
    __shared__ float sF[NF][LH * LW];
    __shared__ float sS[NF][TY * kTileX];           // injected signal per tile point

    if (b >= ls.tile_blocks_pad) {
        sample_block(p.smp, p.A, p.step, b - ls.tile_blocks_pad);
        return;
    }
    const int tile = xcd_logical(b, ls.tile_blocks_pad);
    if (tile >= ls.tile_blocks)
        return;
    const int tyi = tile / ls.tiles_x;
    const int y0 = tyi * TY;
    const int x0 = (tile - tyi * ls.tiles_x) * kTileX;
    const int tid = threadIdx.x;
    const int lx = tid & 63;
    const int wy = tid >> 6;
    const int n0 = d.n[0], n1 = d.n[1];
    const int s0 = (int)d.st[0];
    const int fbytes = (int)(d.total * 4);
    const int gx = x0 + lx;
    const bool xin = gx < n1;

    // entry ranges of the tile (uniform); the forward correction pass injects
    // nothing, the adjoint one its receivers, and it images without a source term
    constexpr bool INJ = MODE != kCorrect || ADJ;
    constexpr bool IMG = ADJ && MODE != kCorrect && !ONE;
    int eb0 = 0, ne0 = 0;
    if constexpr (INJ) {
        eb0 = p.inj.ptr[tile];
        ne0 = p.inj.ptr[tile + 1] - eb0;
    }
    int eb1 = 0, ne1 = 0;
    if constexpr (IMG) {
        eb1 = p.img.ptr[tile];
        ne1 = p.img.ptr[tile + 1] - eb1;
    }

    // tile rows with halo: byte offsets of the column and the halo column
    const int hcol = lx < R ? x0 - R + lx : x0 + kTileX - R + lx;
    const int hlds = lx < R ? lx : kTileX + lx;
    const bool hin = lx < 2 * R && hcol >= 0 && hcol < n1;
    int ro[RW], ho[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int r = wy + i * WAVES;
        const int gy = y0 - R + r;
        const bool rok = r < LH && gy >= 0 && gy < n0;
        ro[i] = rok && xin ? (gy * s0 + gx) * 4 : -1;
        ho[i] = rok && hin ? (gy * s0 + hcol) * 4 : -1;
    }
    float va[NF][RW], vh[NF][RW];
    const float* F1 = ADJ ? p.U : p.B;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const auto rf = plane_rsrc(f == 0 ? p.A : F1, fbytes);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            va[f][i] = bload(rf, ro[i]);
            vh[f][i] = bload(rf, ho[i]);
        }
    }
    int po[RY];
    float bb[RY], kk[RY], gg[RY], uu[RY], mgy[RY], mgx[RY], mat[RY], vv[RY], v2[RY];
    {
        const auto rb = plane_rsrc(p.B, fbytes);
        const auto rk = plane_rsrc(p.K, fbytes);
        const auto ru = plane_rsrc(p.D, fbytes);
#pragma unroll
        for (int j = 0; j < RY; ++j) {
            const int gy = y0 + wy * RY + j;
            po[j] = xin && gy < n0 ? gy * s0 + gx : -1;
            const int bo = po[j] >= 0 ? po[j] * 4 : -1;
            if constexpr (MODE != kPrep && !MED2)
                bb[j] = bload(rb, bo);
            kk[j] = bload(rk, bo);
            if constexpr (MODE == kCorrect)
                uu[j] = bload(ru, bo);
            if constexpr (MED) {
                mgy[j] = bload(plane_rsrc(p.gam[0], fbytes), bo);
                mgx[j] = bload(plane_rsrc(p.gam[1], fbytes), bo);
                mat[j] = bload(plane_rsrc(p.att, fbytes), bo);
            }
        }
        if constexpr (ADJ && MODE != kAdjPlain) {
            const auto rg = plane_rsrc(p.G, fbytes);
#pragma unroll
            for (int j = 0; j < RY; ++j)
                gg[j] = bload(rg, po[j] >= 0 ? po[j] * 4 : -1);
        }
        if constexpr (MODE == kImageV) {
            const auto rv = plane_rsrc(p.V, fbytes);
            const auto r2 = plane_rsrc(p.V2 ? p.V2 : p.V, p.V2 ? fbytes : 0);
#pragma unroll
            for (int j = 0; j < RY; ++j) {
                vv[j] = bload(rv, po[j] >= 0 ? po[j] * 4 : -1);
                v2[j] = bload(r2, po[j] >= 0 ? po[j] * 4 : -1);
            }
        }
    }

    // one entry per thread (more only in tiles with over NT entries)
    int il0 = -1, il1 = -1;
    float iv0 = 0.f, iv1 = 0.f;
    if (tid < ne0) {
        const TileEntry e = p.inj.ent[eb0 + tid];
        if (e.run > 0) {
            il0 = e.local;
            iv0 = tile_point_signal<MODE == kPrep>(p.inj.ent + eb0 + tid, e, p.inj_sig,
                                                   p.inj_stride, p.step);
        }
    }
    if constexpr (IMG) {
        if (tid < ne1) {
            const TileEntry e = p.img.ent[eb1 + tid];
            if (e.run > 0) {
                il1 = e.local;
                iv1 = tile_point_signal(p.img.ent + eb1 + tid, e, p.img_sig, p.img_stride, p.step);
            }
        }
    }

#pragma unroll
    for (int f = 0; f < NF; ++f) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = wy + i * WAVES;
            if (r < LH) {
                sF[f][r * LW + lx + R] = va[f][i];
                if (lx < 2 * R)
                    sF[f][r * LW + hlds] = vh[f][i];
            }
        }
    }
    const bool inj_any = ne0 > 0;
    const bool img_any = IMG && ne1 > 0;
    if (inj_any)
#pragma unroll
        for (int j = 0; j < RY; ++j)
            sS[0][(wy * RY + j) * kTileX + lx] = 0.f;
    if (img_any)
#pragma unroll
        for (int j = 0; j < RY; ++j)
            sS[NF - 1][(wy * RY + j) * kTileX + lx] = 0.f;
    __syncthreads();
    if (inj_any || img_any) {
        if (il0 >= 0)
            sS[0][il0] = iv0;
        for (int e = tid + NT; e < ne0; e += NT) {
            const TileEntry en = p.inj.ent[eb0 + e];
            if (en.run > 0)
                sS[0][en.local] = tile_point_signal<MODE == kPrep>(p.inj.ent + eb0 + e, en, p.inj_sig,
                                                                   p.inj_stride, p.step);
        }
        if constexpr (IMG) {
            if (il1 >= 0)
                sS[1][il1] = iv1;
            for (int e = tid + NT; e < ne1; e += NT) {
                const TileEntry en = p.img.ent[eb1 + e];
                if (en.run > 0)
                    sS[1][en.local] =
                        tile_point_signal(p.img.ent + eb1 + e, en, p.img_sig, p.img_stride, p.step);
            }
        }
        __syncthreads();
    }

    if (!xin)
        return;
    const int dxd = layer_depth(gx, n1, d.nb);
    const float ex = sp.e[1] * (float)(dxd * dxd);
#pragma unroll
    for (int j = 0; j < RY; ++j) {
        if (po[j] < 0)
            break;
        const int ly = wy * RY + j;
        const float* SA = &sF[0][(ly + R) * LW + lx + R];
        const float ctr = SA[0];
        float lap = lap2d<R, LW>(SA, cf);
        float inj = 0.f;
        if (inj_any) {
            if constexpr (kInjApart<ADJ, MODE>)
                inj = sS[0][ly * kTileX + lx];
            else
                lap += sS[0][ly * kTileX + lx];
        }
        const int dyd = layer_depth(y0 + ly, n0, d.nb);
        const float eta = fmaf(sp.e[0], (float)(dyd * dyd), ex);
        if constexpr (MED) {
            float dy = 0.f, dx = 0.f;
#pragma unroll
            for (int q = R; q >= 1; --q) {
                dy = fmaf(cf.d[0][q], SA[q * LW] - SA[-q * LW], dy);
                dx = fmaf(cf.d[1][q], SA[q] - SA[-q], dx);
            }
            float prev, lapb = 0.f;
            if constexpr (MED2) {
                const float* SB = &sF[NF - 1][(ly + R) * LW + lx + R];
                lapb = lap2d<R, LW>(SB, cf);
                prev = SB[0];
            } else {
                prev = bb[j];
            }
            const float dens = fmaf(mgy[j], dy, mgx[j] * dx);
            p.C[po[j]] = medium_out<MED2>(ctr, lap, dens, inj, lapb, prev, kk[j], mat[j], eta,
                                          sp.half_dt);
            if (p.V)   // gradient forward: the imaging factor, read once by the adjoint
                __builtin_nontemporal_store(medium_h<MED2>(ctr, lap, dens, inj, lapb, prev, kk[j],
                                                           mat[j], eta, sp.half_dt),
                                            p.V + po[j]);
            continue;
        }
        p.C[po[j]] = step_out<ADJ, MODE>(ctr, lap, inj, uu[j], bb[j], kk[j], eta, sp.half_dt);
        if constexpr (MODE == kStepV)   // read once, by the adjoint much later
            __builtin_nontemporal_store(lap, p.V + po[j]);
        if constexpr (MODE == kImageV) {
            // with V2 absent its loads read 0 (empty descriptor): fma(B, 0, G) = G
            p.G[po[j]] = fmaf(ctr, vv[j], fmaf(bb[j], v2[j], gg[j]));
        } else if constexpr (ADJ && MODE != kAdjPlain) {
            const float* SU = &sF[NF - 1][(ly + R) * LW + lx + R];
            float lu = lap2d<R, LW>(SU, cf);
            if (img_any)
                lu += sS[NF - 1][ly * kTileX + lx];
            p.G[po[j]] = image_out<MODE>(ctr, SU[0], lu, uu[j], kk[j], gg[j]);
        }
    }
}

// ----------------------------------------------------------------------- 3D
#include "step3d_body.h"

// ------------------------------------------------------------ kernel entry points
//
// Single shot: parameters by value.  Batched: blockIdx.y selects a slot whose
// parameters (and sponge, which depends on the slot's dt) are read from a
// device table; inactive slots exit at once.  Both run the same body, so a
// shot computes the same bits alone and in a batch.

template <int R, bool ADJ, int RY, int WAVES, int MODE = kStep>
__global__ __launch_bounds__(64 * WAVES) void step2d_kernel(Dims d, StencilCoef cf, SpongeCoef sp,
                                                            StepParams p, LaunchShape ls)
{
    step2d_body<R, ADJ, RY, WAVES, MODE>(d, cf, sp, p, ls, blockIdx.x);
}

template <int R, bool ADJ, int RY, int WAVES, int MODE>
__global__ __launch_bounds__(64 * WAVES) void step2d_batched(Dims d, StencilCoef cf, LaunchShape ls,
                                                             const SlotStep* table)
{
    const SlotStep st = table[blockIdx.y];
    if (!st.active)
        return;
    step2d_body<R, ADJ, RY, WAVES, MODE>(d, cf, st.sp, st.p, ls, blockIdx.x);
}

// Occupancy of the 3D kernels: the leapfrog steps, the fourth-order launches with
// one stencil field and the y = 0 medium step stay within 128 VGPRs (4 waves per
// SIMD) by themselves; the attribute holds the compiler to it for a single shot,
// whose launch shapes count on it.
template <bool ADJ, int MODE>
constexpr int min_waves_3d()
{
    return MODE == kMedium || MODE == kMediumY0 || (ADJ && MODE == kCorrect) ? 1 : 4;
}

template <int R, bool ADJ, int VX, int WAVES, int MODE, bool STREAM>
__global__ __launch_bounds__(64 * WAVES)
__attribute__((amdgpu_waves_per_eu(min_waves_3d<ADJ, MODE>())))
void step3d_kernel(Dims d, StencilCoef cf, SpongeCoef sp, StepParams p, LaunchShape ls)
{
    step3d_body<R, ADJ, VX, WAVES, MODE, STREAM>(d, cf, sp, p, ls, blockIdx.x);
}

template <int R, bool ADJ, int VX, int WAVES, int MODE>
__global__ __launch_bounds__(64 * WAVES) void step3d_batched(Dims d, StencilCoef cf, LaunchShape ls,
                                                             const SlotStep* table)
{
    // as constant memory, so that the parameters are loaded where they are used, like
    // a single shot's: a copy of them lives in registers throughout (131 VGPRs at
    // order 10 with one stencil field, three waves per SIMD, instead of 110 and four)
    const SlotStep& st =
        (const SlotStep&)((const __attribute__((address_space(4))) SlotStep*)(uintptr_t)table)[blockIdx.y];
    if (!st.active)
        return;
    step3d_body<R, ADJ, VX, WAVES, MODE, true>(d, cf, st.sp, st.p, ls, blockIdx.x);
}

// Points per thread of a 3D step: four with one stencil field, two with two
// (whose register queues would otherwise leave one wave per SIMD).
template <bool ADJ, int MODE>
constexpr int vec3d()
{
    constexpr bool one = MODE == kImageV || MODE == kAdjPlain;
    return (ADJ && !one) || MODE == kMedium ? kVx3dTwo : kVx3dOne;
}

// 2D tile shapes with compiled kernels (rows per thread, waves); tile_shape_2d()
// returns one of these.  Without STRIDE_TILE_SWEEP: the shape of common.h.
#ifdef STRIDE_TILE_SWEEP
#define STRIDE_DISPATCH2D(L)                                                                      \
    do {                                                                                          \
        if (ls.waves == 8)                                                                        \
            L(4, 8);                                                                              \
        else if (ls.ry == 2)                                                                      \
            L(2, 4);                                                                              \
        else if (ls.ry == 8)                                                                      \
            L(8, 4);                                                                              \
        else                                                                                      \
            L(4, 4);                                                                              \
    } while (0)
#else
#define STRIDE_DISPATCH2D(L) L(kRy2d, kWaves2d)
#endif

// Launch of one step kernel family: the tile blocks, then the sample blocks.
template <int R, bool ADJ, int MODE>
void launch2d_t(const Dims& d, const StencilCoef& cf, const SpongeCoef& sp, const LaunchShape& ls,
                const StepParams& p, hipStream_t s)
{
    const int nt = 64 * ls.waves;
    int smp_blocks = (p.smp.count * sample_lanes(p.smp.ntap) + nt - 1) / nt;
    dim3 grid(ls.tile_blocks_pad + smp_blocks);
#define STRIDE_LAUNCH2D(RY_, W_)                                                                  \
    hipLaunchKernelGGL((step2d_kernel<R, ADJ, RY_, W_, MODE>), grid, dim3(64 * (W_)), 0, s, d, cf, sp, \
                       p, ls)
    STRIDE_DISPATCH2D(STRIDE_LAUNCH2D);
#undef STRIDE_LAUNCH2D
}

template <int R, bool ADJ, int MODE>
void launch3d_t(const Dims& d, const StencilCoef& cf, const SpongeCoef& sp, const LaunchShape& ls,
                const StepParams& p, hipStream_t s)
{
    const int nt = 64 * kWaves3d;
    int smp_blocks = (p.smp.count * sample_lanes(p.smp.ntap) + nt - 1) / nt;
    dim3 grid(ls.tile_blocks_pad + smp_blocks);
    constexpr int VX = vec3d<ADJ, MODE>();
    if (stream_3d(d, ADJ, MODE))
        hipLaunchKernelGGL((step3d_kernel<R, ADJ, VX, kWaves3d, MODE, true>), grid, dim3(nt), 0, s, d,
                           cf, sp, p, ls);
    else
        hipLaunchKernelGGL((step3d_kernel<R, ADJ, VX, kWaves3d, MODE, false>), grid, dim3(nt), 0, s, d,
                           cf, sp, p, ls);
}

template <int R, bool ADJ, int MODE>
void batched2d_t(const Dims& d, const StencilCoef& cf, const LaunchShape& ls, const SlotStep* table,
                 int nslots, int max_sample_threads, hipStream_t s)
{
    const int nt = 64 * ls.waves;
    int smp_blocks = (max_sample_threads + nt - 1) / nt;
    dim3 grid(ls.tile_blocks_pad + smp_blocks, nslots);
#define STRIDE_LAUNCH2DB(RY_, W_)                                                                  \
    hipLaunchKernelGGL((step2d_batched<R, ADJ, RY_, W_, MODE>), grid, dim3(64 * (W_)), 0, s, d, cf, ls, \
                       table)
    STRIDE_DISPATCH2D(STRIDE_LAUNCH2DB);
#undef STRIDE_LAUNCH2DB
}

template <int R, bool ADJ, int MODE>
void batched3d_t(const Dims& d, const StencilCoef& cf, const LaunchShape& ls, const SlotStep* table,
                 int nslots, int max_sample_threads, hipStream_t s)
{
    const int nt = 64 * kWaves3d;
    int smp_blocks = (max_sample_threads + nt - 1) / nt;
    dim3 grid(ls.tile_blocks_pad + smp_blocks, nslots);
    hipLaunchKernelGGL((step3d_batched<R, ADJ, vec3d<ADJ, MODE>(), kWaves3d, MODE>), grid, dim3(nt), 0,
                       s, d, cf, ls, table);
}

// Runtime (R, mode) to template arguments for one family.  Forward modes:
// kStep, kPrep, kCorrect, kMedium, kMediumY0, kStepV; adjoint modes: kStep, kCorrect,
// kImageV, kAdjPlain.
template <bool THREE_D, bool ADJ, int R>
void launch_mode_r(int mode, const Dims& d, const StencilCoef& cf, const SpongeCoef& sp,
                   const LaunchShape& ls, const StepParams& p, hipStream_t s)
{
#define STRIDE_MODE_CASE(M_)                                                                      \
    case M_:                                                                                      \
        if constexpr (THREE_D)                                                                    \
            launch3d_t<R, ADJ, M_>(d, cf, sp, ls, p, s);                                          \
        else                                                                                      \
            launch2d_t<R, ADJ, M_>(d, cf, sp, ls, p, s);                                          \
        return;
    if constexpr (ADJ) {
        switch (mode) {
            STRIDE_MODE_CASE(kStep)
            STRIDE_MODE_CASE(kCorrect)
            STRIDE_MODE_CASE(kImageV)
            STRIDE_MODE_CASE(kAdjPlain)
        default:
            return;
        }
    } else {
        switch (mode) {
            STRIDE_MODE_CASE(kStep)
            STRIDE_MODE_CASE(kPrep)
            STRIDE_MODE_CASE(kCorrect)
            STRIDE_MODE_CASE(kMedium)
            STRIDE_MODE_CASE(kMediumY0)
            STRIDE_MODE_CASE(kStepV)
        default:
            return;
        }
    }
#undef STRIDE_MODE_CASE
}

// Runtime mode to template arguments for the batched launches of one
// family.  Forward modes: kStep, kStepV, kPrep, kCorrect; adjoint modes:
// kStep, kImageV, kAdjPlain, kCorrect.
template <bool THREE_D, bool ADJ, int R>
void batched_mode_r(int mode, const Dims& d, const StencilCoef& cf, const LaunchShape& ls,
                    const SlotStep* table, int nslots, int max_sample_threads, hipStream_t s)
{
#define STRIDE_BMODE_CASE(M_)                                                                     \
    case M_:                                                                                      \
        if constexpr (THREE_D)                                                                    \
            batched3d_t<R, ADJ, M_>(d, cf, ls, table, nslots, max_sample_threads, s);             \
        else                                                                                      \
            batched2d_t<R, ADJ, M_>(d, cf, ls, table, nslots, max_sample_threads, s);             \
        return;
    if constexpr (ADJ) {
        switch (mode) {
            STRIDE_BMODE_CASE(kStep)
            STRIDE_BMODE_CASE(kImageV)
            STRIDE_BMODE_CASE(kAdjPlain)
            STRIDE_BMODE_CASE(kCorrect)
        default:
            return;
        }
    } else {
        switch (mode) {
            STRIDE_BMODE_CASE(kStep)
            STRIDE_BMODE_CASE(kStepV)
            STRIDE_BMODE_CASE(kPrep)
            STRIDE_BMODE_CASE(kCorrect)
        default:
            return;
        }
    }
#undef STRIDE_BMODE_CASE
}

}  // namespace
}  // namespace stride
