// 3D step kernel (every mode of StepMode), included by step_kernels.h.
//
// One block = one 64 x TY column tile marching along axis 0 over a chunk of
// planes; a thread owns VX consecutive points of a tile row (64 / VX lanes per
// row, VX rows per wave), so that a field is read, staged and written in whole
// vectors.  Each thread keeps the 2R+1 axis-0 neighbours of its points in a
// rotating register queue (the march is unrolled by 2R+1 so that the queue
// never shifts).  The plane tile with its halo goes to a double-buffered LDS
// slot, so one barrier per plane suffices; the in-plane taps are LDS vector
// reads, 2R rows for the y taps and 2 HQ / VX vectors for the x taps, shared
// by the VX points of the thread.
//
// What bounds it, and why vectors: with one point per lane and four rows per
// thread the same march read 20 LDS words a point and spent about 55 VALU
// instructions on it, which at grids of up to about 252^3 is more time than
// the memory traffic; with VX = 4 a point costs 12.5 LDS words, a quarter of
// the memory instructions and about 42 VALU instructions.
//
// Software pipeline: while plane z is computed, the queue's lead plane and the
// halo of plane z+1 are in flight; the point values (B, K, G, ...) of plane
// z+1 are issued right after those of plane z were used, into the same
// registers, which is as far ahead of their use and keeps the kernels with
// one stencil field within 128 VGPRs (4 waves per SIMD).
//
// All global accesses are raw buffer accesses with per-plane descriptors:
// offsets outside the grid read 0 and drop stores, so no access needs a
// branch.  A vector that straddles the end of a row lies within the row's
// pitch (a multiple of 16 floats); what it reads there is overwritten by 0 in
// the LDS tile, and what it writes there is never used.
#pragma once

template <int VX>
using StepVec = float __attribute__((ext_vector_type(VX)));

// Byte offset of a vector outside any field or plane (their sizes are multiples
// of 64 below 2^31).  Not -1: the compiler narrows a load of which only some
// values are used, and -1 plus their offset wraps round into the field.
constexpr int kNoByte = 0x7ffffff0;

template <int VX, int AUX>
__device__ __forceinline__ StepVec<VX> bloadv(__amdgpu_buffer_rsrc_t r, int byte_off)
{
    static_assert(VX == 2 || VX == 4, "vector accesses of 8 or 16 bytes");
    if constexpr (VX == 4)
        return __builtin_bit_cast(StepVec<4>,
                                  __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, AUX));
    else
        return __builtin_bit_cast(StepVec<2>,
                                  __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, AUX));
}

template <int VX, int AUX = 0>
__device__ __forceinline__ void bstorev(__amdgpu_buffer_rsrc_t r, int byte_off, StepVec<VX> v)
{
    using U = unsigned __attribute__((ext_vector_type(VX)));
    if constexpr (VX == 4)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U, v), r, byte_off, 0, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U, v), r, byte_off, 0, AUX);
}

// Non-temporal store: results are read back only in a later launch.
template <int VX>
__device__ __forceinline__ void bstorev_nt(__amdgpu_buffer_rsrc_t r, int byte_off, StepVec<VX> v)
{
    bstorev<VX, 2>(r, byte_off, v);
}

// STREAM: the point values are loaded with the non-temporal policy (grids
// whose fields do not stay in the Infinity Cache from step to step).
template <int R, bool ADJ, int VX, int WAVES, int MODE, bool STREAM>
__device__ __forceinline__ void step3d_body(const Dims& d, const StencilCoef& cf,
                                            const SpongeCoef& sp, const StepParams& p,
                                            const LaunchShape& ls, const int b)
{
    using V = StepVec<VX>;
    constexpr int NT = 64 * WAVES;
    constexpr int LPR = kTileX / VX;                // lanes per tile row
    constexpr int TY = WAVES * VX;
    constexpr int HQ = (R + VX - 1) / VX * VX;      // halo columns, in whole vectors
    constexpr int LW = kTileX + 2 * HQ;
    constexpr int LH = TY + 2 * R;
    constexpr int Q = 2 * R + 1;
    constexpr int NYH = 2 * R * LPR;                // halo vectors above and below
    constexpr int XPR = 2 * HQ / VX;                // halo vectors left and right of a row
    constexpr int NH = NYH + XPR * TY;
    constexpr int HL = (NH + NT - 1) / NT;
    constexpr bool MED = kIsMedium<MODE>;
    constexpr bool MED2 = MODE == kMedium;          // B a stencil field
    constexpr bool ONE = MODE == kImageV || MODE == kAdjPlain;      // adjoint with one stencil field
    constexpr int NF = (ADJ && !ONE) || MED2 ? 2 : 1;  // stencil fields: A (and U, or B)
    constexpr bool HAS_B = MODE != kPrep && !MED2;  // B a point value
    constexpr bool HAS_G = ADJ && MODE != kAdjPlain;
    constexpr int PLANE = LH * LW;
    constexpr int PL = TY * kTileX;                 // block-local points per plane
    constexpr int AUX = STREAM ? STRIDE_STREAM_AUX : 0;
    __shared__ __align__(16) float sF[2][NF][PLANE];
    __shared__ __align__(16) float sS[2][NF][PL];   // injected signal per plane point
    __shared__ int2 sE[NF][NT];                     // entry (local point, value) per thread

    if (b >= ls.tile_blocks_pad) {
        sample_block(p.smp, p.A, p.step, b - ls.tile_blocks_pad);
        return;
    }
    const int lb = xcd_logical(b, ls.tile_blocks_pad);
    if (lb >= ls.tile_blocks)
        return;
    const int zci = lb / ls.tiles_xy;
    const int tile = lb - zci * ls.tiles_xy;
    const int y0 = (tile / ls.tiles_x) * TY;
    const int x0 = (tile % ls.tiles_x) * kTileX;
    const int n0 = d.n[0], n1 = d.n[1], n2 = d.n[2];
    const int z0 = zci * ls.zc;
    const int z1 = min(z0 + ls.zc, n0);
    const long long s0 = d.st[0];
    const int s1 = (int)d.st[1];
    const int tid = threadIdx.x;
    const int row = tid / LPR;
    const int col = (tid % LPR) * VX;
    const int gx = x0 + col, gy = y0 + row;
    const float* F[2] = {p.A, ADJ ? p.U : (MED2 ? p.B : p.A)};

    // plane-independent geometry: byte offsets within a plane (kNoByte: outside)
    const int plane_bytes = (int)(s0 * 4);
    const int bo = gx < n2 && gy < n1 ? (gy * s1 + gx) * 4 : kNoByte;
    const int lo = (row + R) * LW + col + HQ;       // own points in the LDS tile
    float ey[VX];
    {
        const int dyd = layer_depth(gy, n1, d.nb);
#pragma unroll
        for (int k = 0; k < VX; ++k) {
            const int dxd = layer_depth(gx + k, n2, d.nb);
            ey[k] = fmaf(sp.e[1], (float)(dyd * dyd), sp.e[2] * (float)(dxd * dxd));
        }
    }
    // rows that end inside a vector of this tile or its halo (uniform)
    const bool ragged = n2 % VX != 0 && x0 + kTileX + HQ > n2;
    int hl[HL], ho[HL], hx[HL];
#pragma unroll
    for (int h = 0; h < HL; ++h) {
        const int i = tid + h * NT;
        hl[h] = -1;
        ho[h] = kNoByte;
        hx[h] = 0;
        if (i < NH) {
            int ly, lx;
            if (i < NYH) {
                const int hr = i / LPR;
                ly = hr < R ? hr - R : TY + hr - R;
                lx = (i % LPR) * VX;
            } else {
                const int c = (i - NYH) % XPR;
                ly = (i - NYH) / XPR;
                lx = c < XPR / 2 ? c * VX - HQ : kTileX + (c - XPR / 2) * VX;
            }
            const int g = x0 + lx, y = y0 + ly;
            hl[h] = (ly + R) * LW + lx + HQ;
            hx[h] = g;
            if (y >= 0 && y < n1 && g >= 0 && g < n2)
                ho[h] = (y * s1 + g) * 4;
        }
    }
    // descriptor of plane z of a field, z in the grid
    auto rsrc_in = [&](const float* f, int z) { return plane_rsrc(f + z * s0, plane_bytes); };
    auto rsrc = [&](const float* f, int z) {
        const bool in = z >= 0 && z < n0;
        return plane_rsrc(f + (in ? z : 0) * s0, in ? plane_bytes : 0);
    };

    // queue slot (i + t) % Q holds plane z0 + i + t - R at march iteration i
    V q[NF][Q];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < 2 * R; ++t)
            q[f][t] = bloadv<VX, 0>(rsrc(F[f], z0 - R + t), bo);

    V pl[NF], ph[NF][HL], pb, pk, pg, pu, pm[4], pv, pv2;
    // lead plane and halo of plane z
    auto prefetch = [&](int z) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            pl[f] = bloadv<VX, 0>(rsrc(F[f], z + R), bo);
            const auto rz = rsrc_in(F[f], z);
#pragma unroll
            for (int h = 0; h < HL; ++h)
                ph[f][h] = bloadv<VX, 0>(rz, ho[h]);
        }
    };
    // point values of plane z
    auto prefetch_points = [&](int z) {
        if constexpr (HAS_B)
            pb = bloadv<VX, AUX>(rsrc_in(p.B, z), bo);
        pk = bloadv<VX, AUX>(rsrc_in(p.K, z), bo);
        if constexpr (MED) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                pm[m] = bloadv<VX, AUX>(rsrc_in(m < 3 ? p.gam[m] : p.att, z), bo);
        }
        if constexpr (MODE == kCorrect)
            pu = bloadv<VX, AUX>(rsrc_in(p.D, z), bo);
        if constexpr (HAS_G)
            pg = bloadv<VX, AUX>(rsrc_in(p.G, z), bo);
        if constexpr (MODE == kImageV) {
            // kept states: read once per sweep; with V2 absent the descriptor
            // is empty and its loads read 0
            pv = bloadv<VX, STRIDE_STREAM_AUX>(rsrc_in(p.V, z), bo);
            pv2 = bloadv<VX, STRIDE_STREAM_AUX>(p.V2 ? rsrc_in(p.V2, z) : plane_rsrc(p.V, 0), bo);
        }
    };

    // Injection entries of the block (uniform range).  Thread t takes entry t,
    // sums the signal over the point's run and parks (local point, value) in
    // LDS; before the barrier of each plane it writes the value of its entry
    // of that plane to the LDS plane array, where the point's thread takes
    // (and clears) it after the barrier.  Blocks with more than NT entries
    // read the rest at every plane.
    constexpr bool INJ = MODE != kCorrect || ADJ;
    constexpr bool IMG = ADJ && MODE != kCorrect && !ONE;
    int eb0 = 0, ne0 = 0;
    if constexpr (INJ) {
        eb0 = p.inj.ptr[lb];
        ne0 = p.inj.ptr[lb + 1] - eb0;
    }
    int eb1 = 0, ne1 = 0;
    if constexpr (IMG) {
        eb1 = p.img.ptr[lb];
        ne1 = p.img.ptr[lb + 1] - eb1;
    }
    const bool inj_any = ne0 > 0;
    const bool img_any = IMG && ne1 > 0;
    prefetch(z0);
    prefetch_points(z0);
    if (inj_any || img_any) {
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
        for (int bsel = 0; bsel < 2; ++bsel)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                *(V*)&sS[bsel][f][row * kTileX + col] = V(0.f);
        sE[0][tid] = make_int2(il0, __float_as_int(iv0));
        if constexpr (IMG)
            sE[1][tid] = make_int2(il1, __float_as_int(iv1));
        __syncthreads();
        if (il0 >= 0 && il0 < PL)
            sS[0][0][il0] = iv0;
        if constexpr (IMG)
            if (il1 >= 0 && il1 < PL)
                sS[0][1][il1] = iv1;
    }
    // Entries beyond the first NT of the block, written at their plane.  A
    // block's entries are sorted by point, so their planes never decrease.
    // The adjoint (receiver sets of up to 512 taps a point fill some blocks
    // with thousands of entries) keeps a cursor per thread over its entries
    // (tid + NT, tid + 2 NT, ...) and at plane pz takes them until the first
    // of a later plane: every entry is read once per chunk, plus one
    // look-ahead per plane.  The forward step, whose source entries rarely
    // overflow, scans them at every plane and keeps its registers.
    int oc0 = tid + NT, oc1 = tid + NT;
    auto overflow = [&](auto filt, const InjTable& T, int eb, int ne, int& oc, const float* sig,
                        int stride, int pz, float* dst) {
        if constexpr (ADJ) {
            for (; oc < ne; oc += NT) {
                const TileEntry en = T.ent[eb + oc];
                const int ez = en.local / PL;
                if (ez > pz)
                    break;
                if (en.run > 0 && ez == pz)
                    dst[en.local - pz * PL] = tile_point_signal<decltype(filt)::value>(
                        T.ent + eb + oc, en, sig, stride, p.step);
            }
        } else {
            for (int e = tid + NT; e < ne; e += NT) {
                const TileEntry en = T.ent[eb + e];
                if (en.run > 0 && en.local / PL == pz)
                    dst[en.local - pz * PL] = tile_point_signal<decltype(filt)::value>(
                        T.ent + eb + e, en, sig, stride, p.step);
            }
        }
    };

    int buf = 0;
    for (int zb = z0; zb < z1; zb += Q) {
        unrolled_while<Q>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr int slot_lead = (u + 2 * R) % Q;
            constexpr int slot_c = (u + R) % Q;
            const int z = zb + u;
            if (z >= z1)
                return false;
            float* S = &sF[buf][0][0];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                float* Sf = S + f * PLANE;
                q[f][slot_lead] = pl[f];
                *(V*)&Sf[lo] = q[f][slot_c];
#pragma unroll
                for (int h = 0; h < HL; ++h)
                    if (hl[h] >= 0)
                        *(V*)&Sf[hl[h]] = ph[f][h];
                if (ragged) {
#pragma unroll
                    for (int k = 1; k < VX; ++k) {
                        if (gx + k >= n2)
                            Sf[lo + k] = 0.f;
#pragma unroll
                        for (int h = 0; h < HL; ++h)
                            if (hl[h] >= 0 && hx[h] + k >= n2)
                                Sf[hl[h] + k] = 0.f;
                    }
                }
            }
            if (z + 1 < z1)
                prefetch(z + 1);
            const int pz = z - z0;
            if (pz > 0 && (inj_any || img_any)) {
                // parked entry sets: the injection, and the imaging source term
#pragma unroll
                for (int f = 0; f < (IMG ? 2 : 1); ++f) {
                    const int2 e = sE[f][tid];
                    if (e.x >= 0 && e.x / PL == pz)
                        sS[buf][f][e.x - pz * PL] = __int_as_float(e.y);
                }
            }
            if (ne0 > NT)
                overflow(std::integral_constant<bool, MODE == kPrep>{}, p.inj, eb0, ne0, oc0,
                         p.inj_sig, p.inj_stride, pz, &sS[buf][0][0]);
            if constexpr (IMG)
                if (ne1 > NT)
                    overflow(std::false_type{}, p.img, eb1, ne1, oc1, p.img_sig, p.img_stride, pz,
                             &sS[buf][NF - 1][0]);
            __syncthreads();

            // Sums over the taps of field f per axis (second derivative s, and
            // with DIFF the first derivative g), outermost taps first.  The
            // scheduling barriers bound how many LDS vectors are in flight.
            auto taps = [&](auto fc, auto diffc, V* s, V* g) {
                constexpr int f = decltype(fc)::value;
                constexpr bool DIFF = decltype(diffc)::value;
                const float* Sf = S + f * PLANE + lo;
                float xs[VX + 2 * HQ];
#pragma unroll
                for (int i = 0; i < HQ / VX; ++i) {
                    const V l = *(const V*)(Sf - HQ + i * VX);
                    const V r = *(const V*)(Sf + VX + i * VX);
#pragma unroll
                    for (int k = 0; k < VX; ++k) {
                        xs[i * VX + k] = l[k];
                        xs[HQ + VX + i * VX + k] = r[k];
                    }
                }
                V own = q[f][slot_c];
                if (ragged)     // with its points beyond the row's end at 0
                    own = *(const V*)Sf;
#pragma unroll
                for (int k = 0; k < VX; ++k)
                    xs[HQ + k] = own[k];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    s[a] = V(0.f);
                    if constexpr (DIFF)
                        g[a] = V(0.f);
                }
#pragma unroll
                for (int t = R; t >= 1; --t)
#pragma unroll
                    for (int k = 0; k < VX; ++k) {
                        const float xp = xs[HQ + k + t], xm = xs[HQ + k - t];
                        s[2][k] = fmaf(cf.c[2][t], xp + xm, s[2][k]);
                        if constexpr (DIFF)
                            g[2][k] = fmaf(cf.d[2][t], xp - xm, g[2][k]);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = R; t >= 1; --t) {
                    const V yp = *(const V*)(Sf + t * LW), ym = *(const V*)(Sf - t * LW);
                    const V zp = q[f][(u + R + t) % Q], zm = q[f][(u + R - t) % Q];
#pragma unroll
                    for (int k = 0; k < VX; ++k) {
                        s[0][k] = fmaf(cf.c[0][t], zp[k] + zm[k], s[0][k]);
                        s[1][k] = fmaf(cf.c[1][t], yp[k] + ym[k], s[1][k]);
                        if constexpr (DIFF) {
                            g[0][k] = fmaf(cf.d[0][t], zp[k] - zm[k], g[0][k]);
                            g[1][k] = fmaf(cf.d[1][t], yp[k] - ym[k], g[1][k]);
                        }
                    }
                    if (t == 3)
                        __builtin_amdgcn_sched_barrier(0);
                }
            };
            using F0 = std::integral_constant<int, 0>;
            using F1 = std::integral_constant<int, NF - 1>;
            V s[3], g[3], lap, inj = V(0.f);
            taps(F0{}, std::integral_constant<bool, MED>{}, s, g);
            const V ctr = q[0][slot_c];
#pragma unroll
            for (int k = 0; k < VX; ++k)
                lap[k] = fmaf(cf.c0, ctr[k], s[0][k] + s[1][k] + s[2][k]);
            if (inj_any) {
                V* si = (V*)&sS[buf][0][row * kTileX + col];
                const V t = *si;
                if constexpr (kInjApart<ADJ, MODE>)
                    inj = t;
                else
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        lap[k] += t[k];
                *si = V(0.f);
            }
            const int dzd = layer_depth(z, n0, d.nb);
            const float ez = sp.e[0] * (float)(dzd * dzd);
            V eta;
#pragma unroll
            for (int k = 0; k < VX; ++k)
                eta[k] = ez + ey[k];
            if constexpr (MED) {
                V dens, lapb = V(0.f), prev, out;
#pragma unroll
                for (int k = 0; k < VX; ++k)
                    dens[k] = fmaf(pm[0][k], g[0][k], fmaf(pm[1][k], g[1][k], pm[2][k] * g[2][k]));
                if constexpr (MED2) {
                    taps(F1{}, std::false_type{}, s, g);
                    prev = q[NF - 1][slot_c];
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        lapb[k] = fmaf(cf.c0, prev[k], s[0][k] + s[1][k] + s[2][k]);
                } else {
                    prev = pb;
                }
#pragma unroll
                for (int k = 0; k < VX; ++k)
                    out[k] = medium_out<MED2>(ctr[k], lap[k], dens[k], inj[k], lapb[k], prev[k], pk[k],
                                              pm[3][k], eta[k], sp.half_dt);
                bstorev_nt<VX>(rsrc_in(p.C, z), bo, out);
                if (p.V) {   // gradient forward: the imaging factor
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        out[k] = medium_h<MED2>(ctr[k], lap[k], dens[k], inj[k], lapb[k], prev[k],
                                                pk[k], pm[3][k], eta[k], sp.half_dt);
                    bstorev_nt<VX>(rsrc_in(p.V, z), bo, out);
                }
            } else {
                V out;
                // a wave with no point in the layer takes the undamped update
                // without the per-point branches (the same operations)
                bool damped = false;
#pragma unroll
                for (int k = 0; k < VX; ++k)
                    damped = damped || eta[k] != 0.f;
                const V bv = HAS_B ? pb : V(0.f), uv = MODE == kCorrect ? pu : V(0.f);
                if (MODE == kPrep || !__any(damped)) {
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        out[k] = step_out<ADJ, MODE>(ctr[k], lap[k], inj[k], uv[k], bv[k], pk[k], 0.f,
                                                     sp.half_dt);
                } else {
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        out[k] = step_out<ADJ, MODE>(ctr[k], lap[k], inj[k], uv[k], bv[k], pk[k],
                                                     eta[k], sp.half_dt);
                }
                bstorev_nt<VX>(rsrc_in(p.C, z), bo, out);
                if constexpr (MODE == kStepV)
                    bstorev_nt<VX>(rsrc_in(p.V, z), bo, lap);
                if constexpr (MODE == kImageV) {
                    V gn;
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        gn[k] = fmaf(ctr[k], pv[k], fmaf(pb[k], pv2[k], pg[k]));
                    bstorev_nt<VX>(rsrc_in(p.G, z), bo, gn);
                } else if constexpr (HAS_G) {
                    taps(F1{}, std::false_type{}, s, g);
                    const V uc0 = q[NF - 1][slot_c];
                    V lu, gn;
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        lu[k] = fmaf(cf.c0, uc0[k], s[0][k] + s[1][k] + s[2][k]);
                    if (img_any) {
                        V* si = (V*)&sS[buf][NF - 1][row * kTileX + col];
                        const V t = *si;
#pragma unroll
                        for (int k = 0; k < VX; ++k)
                            lu[k] += t[k];
                        *si = V(0.f);
                    }
#pragma unroll
                    for (int k = 0; k < VX; ++k)
                        gn[k] = image_out<MODE>(ctr[k], uc0[k], lu[k], uv[k], pk[k], pg[k]);
                    bstorev_nt<VX>(rsrc_in(p.G, z), bo, gn);
                }
            }
            if (z + 1 < z1)
                prefetch_points(z + 1);
            buf ^= 1;
            return true;
        });
    }
}
