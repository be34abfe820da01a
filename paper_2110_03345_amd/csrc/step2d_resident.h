// 2D leapfrog sweeps with the state kept on the chip (kStep, kStepV and the
// adjoint steps imaging from a stored v), included by step2d.hip.
//
// A single 2D step is bound by its launch and one load phase (6.1 us at 1104^2,
// 4.1 us at 240^2), while u^n, u^{n-1} and k of a grid of up to about two
// million points fit the registers of the 256 CUs.  So one launch runs a whole
// sweep: each block owns one tile, keeps u^{n-1}, u^n and k of its points in
// registers and u^n of the tile and its frame in LDS, and per step exchanges
// only the frame of R cells with its eight neighbours.  Measured, whole solves
// with their sources and receivers: 2.1 us a step at 1104^2 (single steps: 5.9),
// 1.6 at 240^2 (4.3); forward and adjoint together 5.0 at 1104^2 (14.1).
//
// Exchange: a block publishes each of its outer quads as three 64-bit words (a
// value, a third of the fourth value's bits, 21 bits of the step's number) with
// device-scope atomic stores into its slots of a double-buffered area, and takes
// its frame from the neighbours' slots, polling until the words carry the number.
// Value and number travel in one word, so no fence and no flag is needed: 1.75 us
// for 1152 words between 256 blocks, against 2.5 us with a flag per block.  The
// outer quads are computed first, so that the rest of the tile is computed while
// the words are on their way.  A block overwrites its words of exchange n with
// those of n + 2 only after taking every neighbour's words of n + 1, which each
// neighbour publishes after taking all its words of n.
//
// T = 2: one exchange for two steps.  The frame is twice as wide, and the first
// step is computed on the tile and a ring of R cells around it, whose u^n and
// u^{n-1} need no exchange of their own.  At 240^2 an exchange and two small
// computations take 2.8 us (1.4 a step) where two exchanges take 3.6.
//
// Every block must be resident at once: the launch is cooperative, and every
// wait is bounded; a block that waits too long sets p.err, which ends the
// waits of all others.  The bound counts polls, not time: a process whose queues
// are set aside for another's does not poll meanwhile.  Steps compute the operations of the single-step kernel
// in the same order: the same bits.
#pragma once

// Points of a tile whose bilinear taps are kept in LDS.
constexpr int kResidentSampled = 64;

// J: quads per thread; T: steps per exchange (2: order 8, one quad)
template <int R, int MODE, int J, int T>
__global__ __launch_bounds__(kResidentThreads) void step2d_resident(Dims d, StencilCoef cf,
                                                                    ResidentShape rs, ResidentBatch batch)
{
    using V = StepVec<4>;
    using Word = unsigned long long;
    constexpr int NT = kResidentThreads;
    constexpr bool ADJ = MODE == kImageV;
    constexpr int HB = (R + 3) / 4, HQ = 4 * HB;    // quads and columns the row taps reach
    constexpr int FR = T * R, FB = (T * R + 3) / 4; // frame rows, frame quads of a row
    constexpr int ER = FR - R, EB = (T - 1) * HB;   // ring rows, ring quads of a row
    // centre values: in registers, or with two steps per exchange (whose ring
    // takes them from the frame) in LDS
    constexpr bool CEN = T == 1;
    extern __shared__ __align__(16) float lds[];
    // one past the step in which the block gave up, 0: none.  (Not a flag: a wave may
    // reach the next step's wait before another has looked at this step's)
    __shared__ int bad;
    __shared__ int ti[4 * kResidentSampled];         // bilinear taps of the tile's points
    __shared__ float tw[4 * kResidentSampled];
    __shared__ int tr[kResidentSampled];
    __shared__ float ey[kResidentSide];
    __shared__ __align__(16) float ex[kResidentSide];
    const int block = xcd_logical(blockIdx.x, gridDim.x), slot = block / rs.tiles;
    if (slot >= batch.n)
        return;
    const int tile = block - slot * rs.tiles;
    const ResidentParams& p = batch.p[slot];
    const SpongeCoef sp = p.sp;
    const int tid = threadIdx.x;
    const int txq = rs.tx / 4, ty = rs.ty;
    const int W = rs.tx + 8 * FB;
    const int area = W * (ty + 2 * FR);
    float* const buf = lds;                          // two buffers of u^n
    float* const sS = lds + 2 * area;                // two buffers of injected values
    float* const sK = lds + (p.injects ? 4 : 2) * area;     // k (adjoint, two quads a thread)
    const int tyi = tile / rs.tiles_x, txi = tile - tyi * rs.tiles_x;
    const int y0 = tyi * ty, x0 = txi * rs.tx;
    const int n0 = d.n[0], n1 = d.n[1];
    const int s0 = (int)d.st[0];
    const int fbytes = (int)(d.total * 4);
    const int nbq = resident_outer_quads(R, rs);     // published quads
    const int ws = resident_word_stride(R, rs);
    const int nq = txq * ty, items = (txq + 2 * EB) * (ty + 2 * ER);
    const bool state = p.A != nullptr;

    const int eb = p.inj.ptr[tile];
    const int ne = p.inj.ptr[tile + 1] - eb;
    int sb = 0, ns = 0;
    if (p.smp.out) {
        sb = p.smp.ptr[tile];
        ns = p.smp.ptr[tile + 1] - sb;
    }
    const bool ragged = n1 % 4 != 0 && x0 + rs.tx + 4 * FB > n1;    // rows ending inside a quad

    // zero everything, then the state of the tile and its frame
    for (int i = tid; i < (ne > 0 ? 4 : 2) * area / 4; i += NT)
        *(V*)&lds[4 * i] = V(0.f);
    if (tid == 0)
        bad = 0;
    __syncthreads();

    // items: outer quads first (thread i), then the inner ones and the ring, on the
    // lowest threads that can hold them, the second round from the highest of
    // those down
    const int nc = resident_compute_threads(items, nbq, J);
    // the adjoint, with G and v in registers, derives places and damping anew
    // every step and (two quads a thread) keeps k in LDS, to stay within 128
    // VGPRs; the forward sweeps hold them
    constexpr bool LEAN = ADJ && J > 1, KEEP_K = !LEAN;
    V uc[J], up[J], kk[J], eta[J], gg[J], vv[J], v2[J];     // vv, v2: v of the steps
    int rq[J];                                      // row << 16 | quad, from the ring's first; -1: none
    int li_[J], bo_[J];
    bool damped[J], own[J];
    auto place_of = [&](int rq) {
        return ((rq >> 16) + R) * W + 4 * ((rq & 0xffff) + FB - EB);
    };
    // its own quads' byte offset in a field
    auto field_of = [&](int rq, bool own) {
        return rq < 0 || !own ? kNoByte
                              : ((y0 + (rq >> 16) - ER) * s0 + x0 + 4 * ((rq & 0xffff) - EB)) * 4;
    };
    auto place = [&](int j) { return LEAN ? place_of(rq[j]) : li_[j]; };
    auto field = [&](int j) { return LEAN ? field_of(rq[j], own[j]) : bo_[j]; };
    const auto rK = plane_rsrc(p.K, fbytes);
    const auto rA = plane_rsrc(state ? p.A : p.K, state ? fbytes : 0);
    const auto rB = plane_rsrc(state ? p.B : p.K, state ? fbytes : 0);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = tid >= nc ? items : j == 0 ? tid : j * nc + (nc - 1 - tid);
        int r = 0, q = 0;
        if (i < nbq) {
            if (i < FR * txq) {
                r = i / txq;
                q = i - r * txq;
            } else if (i < 2 * FR * txq) {
                const int e = i - FR * txq;
                r = ty - FR + e / txq;
                q = e % txq;
            } else {
                const int e = i - 2 * FR * txq;
                r = FR + e / (2 * FB);
                q = e % (2 * FB);
                q = q < FB ? q : txq - 2 * FB + q;
            }
        } else if (i < nq) {
            const int e = i - nbq, wi = txq - 2 * FB;
            r = FR + e / wi;
            q = FB + e % wi;
        } else if constexpr (T > 1) {
            const int e = i - nq, row = txq + 2 * EB;
            if (e < 2 * ER * row) {
                r = e / row;
                q = e - r * row - EB;
                r = r < ER ? r - ER : ty + r - ER;
            } else {
                r = (e - 2 * ER * row) / (2 * EB);
                q = (e - 2 * ER * row) % (2 * EB);
                q = q < EB ? q - EB : txq + q - EB;
            }
        }
        const int gy = y0 + r, gx = x0 + 4 * q;
        const bool in = i < items && gy >= 0 && gy < n0 && gx >= 0 && gx < n1;
        own[j] = T == 1 || i < nq;
        rq[j] = in ? (r + ER) << 16 | (q + EB) : -1;
        li_[j] = place_of(rq[j]);
        bo_[j] = field_of(rq[j], own[j]);
        const int so = in ? (gy * s0 + gx) * 4 : kNoByte;
        uc[j] = bloadv<4, 0>(rA, so);
        up[j] = bloadv<4, 0>(rB, so);
        kk[j] = bloadv<4, 0>(rK, so);
        if constexpr (!KEEP_K)
            if (in)
                *(V*)&sK[4 * i] = kk[j];
        const int dyd = layer_depth(gy, n0, d.nb);
        bool any = dyd != 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int dxd = layer_depth(gx + k, n1, d.nb);
            any = any || dxd != 0;
            eta[j][k] = fmaf(sp.e[0], (float)(dyd * dyd), sp.e[1] * (float)(dxd * dxd));
        }
        damped[j] = __any(in && any);
        if constexpr (ADJ)
            gg[j] = bloadv<4, 0>(plane_rsrc(p.G, fbytes), bo_[j]);
    }
    // points beyond the end of a row stay 0
    auto clip = [&](V& v, int l) {
        const int gx = x0 + l % W - 4 * FB;
#pragma unroll
        for (int k = 1; k < 4; ++k)
            v[k] = gx + k < n1 ? v[k] : 0.f;
    };
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (rq[j] >= 0) {
            const int li = li_[j];
            if (ragged) {
                clip(uc[j], li);
                clip(up[j], li);
            }
            if (own[j])
                *(V*)&buf[li] = uc[j];
        }
    // sponge: squared depth per row, e_x depth^2 per column of the tile and ring
    for (int i = tid; i < ty + 2 * ER; i += NT) {
        const int dyd = layer_depth(y0 + i - ER, n0, d.nb);
        ey[i] = (float)(dyd * dyd);
    }
    for (int i = tid; i < rs.tx + 8 * EB; i += NT) {
        const int dxd = layer_depth(x0 + i - 4 * EB, n1, d.nb);
        ex[i] = sp.e[1] * (float)(dxd * dxd);
    }

    // frame quad of this thread: its place in LDS and in the owner's slots.
    // The last waves with items poll: they finish their items last, when the
    // words are about to arrive (waves without items, polling all along, slow
    // the exchange: 2.6 us a step at 592^2 with 48 x 54 tiles, 1.8 this way)
    int hl = -1, first;
    const Word* hw = nullptr;
    {
        const int nrow = txq + 2 * FB, nh = 2 * FR * nrow + 2 * FB * ty;
        const int nhw = (nh + 63) / 64 * 64;
        first = nc > nhw ? nc - nhw : 0;
        const int h = tid - first;
        if (h >= 0 && h < nh) {
            int rr, qq;
            if (h < FR * nrow) {
                rr = h / nrow - FR;
                qq = h % nrow - FB;
            } else if (h < 2 * FR * nrow) {
                const int e = h - FR * nrow;
                rr = ty + e / nrow;
                qq = e % nrow - FB;
            } else {
                const int e = h - 2 * FR * nrow;
                rr = e / (2 * FB);
                qq = e % (2 * FB);
                qq = qq < FB ? qq - FB : txq + qq - FB;
            }
            const int gy = y0 + rr, gx = x0 + 4 * qq;
            if (gy >= 0 && gy < n0 && gx >= 0 && gx < n1) {
                const int oy = rr < 0 ? -1 : (rr >= ty ? 1 : 0), ox = qq < 0 ? -1 : (qq >= txq ? 1 : 0);
                const int r = rr - oy * ty, q = qq - ox * txq;
                const int id = r < FR         ? r * txq + q
                               : r >= ty - FR ? (r - (ty - 2 * FR)) * txq + q
                                              : 2 * FR * txq + (r - FR) * 2 * FB + (q < FB ? q : q - (txq - 2 * FB));
                hl = (rr + FR) * W + 4 * (qq + FB);
                hw = p.words + (long long)(tile + oy * rs.tiles_x + ox) * 3 * ws + id;
                if (state) {
                    V v = bloadv<4, 0>(rA, (gy * s0 + gx) * 4);
                    if (ragged)
                        clip(v, hl);
                    *(V*)&buf[hl] = v;
                }
            }
        }
    }
    Word* const mine = p.words + (long long)tile * 3 * ws + tid;
    const long long parity = (long long)rs.tiles * 3 * ws;
    const int look = p.patience < 1024 ? 0 : 1023;   // polls between looks at p.err

    // the order in which threads take entries and points: from the last before
    // the polling waves down (past `skip`), those waves at the end
    auto turn_of = [&](int skip) { return (first - skip - 1 - tid) & (NT - 1); };
    // this thread's injection entry (tiles with more than NT read the rest
    // every step)
    const int et = turn_of(64);
    TileEntry en{};
    if (et < ne)
        en = p.inj.ent[eb + et];
    // its next signal sample, loaded a step ahead of its use
    auto raw = [&](int t) {
        return en.run > 0 && t < p.count
                   ? p.inj_sig[(long long)en.id * p.inj_stride + p.step + p.dir * t]
                   : 0.f;
    };
    auto inject = [&](int t, float head) {
        float* s = sS + (t & 1) * area;
        const int step = p.step + p.dir * t;
        if (en.run > 0) {
            float v = en.w * head;
            for (int k = 1; k < en.run; ++k) {
                const TileEntry x = p.inj.ent[eb + et + k];
                v = fmaf(x.w, sig_at<false>(p.inj_sig, x.id, p.inj_stride, step), v);
            }
            s[en.local] = v;
        }
        for (int e = et + NT; e < ne; e += NT) {
            const TileEntry x = p.inj.ent[eb + e];
            if (x.run > 0)
                s[x.local] = tile_point_signal(p.inj.ent + eb + e, x, p.inj_sig, p.inj_stride, step);
        }
    };
    // samples of the state in S (LDS taps where they fit: a global load per tap
    // and step would outlast the exchange)
    auto sample = [&](const float* S, int step) {
        const int nt = p.smp.ntap;
        const int* idx = p.smp.idx + (long long)sb * nt;
        const float* w = p.smp.w + (long long)sb * nt;
        if (sample_lanes(nt) == 1) {
            for (int r = turn_of(0); r < ns; r += NT) {
                float acc = 0.f;
                int row;
                if (r < kResidentSampled) {
                    row = tr[r];
                    for (int k = 0; k < nt; ++k)
                        acc = fmaf(tw[r * 4 + k], S[ti[r * 4 + k]], acc);
                } else {
                    row = p.smp.id[sb + r];
                    for (int k = 0; k < nt; ++k)
                        acc = fmaf(w[r * nt + k], S[idx[r * nt + k]], acc);
                }
                p.smp.out[(long long)row * p.smp.out_stride + step] = acc;
            }
        } else {
            // one wave per point, lanes over the taps (the order of sample_block)
            for (int r = turn_of(0) >> 6; r < ns; r += NT / 64) {
                float acc = 0.f;
                for (int k = tid & 63; k < nt; k += 64)
                    acc = fmaf(w[r * nt + k], S[idx[r * nt + k]], acc);
#pragma unroll
                for (int off = 32; off > 0; off >>= 1)
                    acc += __shfl_xor(acc, off, 64);
                if ((tid & 63) == 0)
                    p.smp.out[(long long)p.smp.id[sb + r] * p.smp.out_stride + step] = acc;
            }
        }
    };
    if (p.smp.ntap == 4 && tid < 4 * min(ns, kResidentSampled)) {
        ti[tid] = p.smp.idx[(long long)sb * 4 + tid];
        tw[tid] = p.smp.w[(long long)sb * 4 + tid];
    }
    if (tid < min(ns, kResidentSampled))
        tr[tid] = p.smp.id[sb + tid];
    float sig = 0.f;
    if (ne > 0) {
        inject(0, raw(0));
        sig = raw(1);
    }
    __syncthreads();

    auto load_v = [&](V* v, int t) {
        const auto rV = plane_rsrc(p.V + t * p.vstride, fbytes);
#pragma unroll
        for (int j = 0; j < J; ++j)
            v[j] = bloadv<4, STRIDE_STREAM_AUX>(rV, field(j));
    };
    auto image = [&](int j, const V& u, const V& v) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            gg[j][k] = fmaf(u[k], v[k], gg[j][k]);
    };
    // with two steps per exchange both steps' terms are added at the second,
    // from v loaded at the second before
    if constexpr (ADJ && T > 1) {
        load_v(vv, 0);
        if (p.count > 1)
            load_v(v2, 1);
    }
    // Step t + s of the sweep, s < T; false: it was the last, or the blocks gave up.
    auto step = [&](auto sc, int t0) {
        constexpr int s = decltype(sc)::value;
        constexpr bool LAST = s == T - 1;       // of an exchange
        const int t = t0 + s;
        const int from = T == 1 ? t & 1 : s;
        const float* S = buf + from * area;
        float* Sn = buf + (1 - from) * area;
        const bool more = t + 1 < p.count;
        // (a sweep of one exchange: before its blocks store the state others
        // still load)
        const bool exchange = LAST && (more || p.sample_last || p.count <= T);
        Word* const out = mine + (t0 / T & 1) * parity;
        auto next_inject = [&]() {
            if (ne > 0 && more) {
                inject(t + 1, sig);
                sig = raw(t + 2);
            }
        };
        // first with two quads a thread (a step at 1104^2 is 0.05 us shorter), else
        // after the words (0.02 us at 240^2)
        if constexpr (J > 1)
            next_inject();
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (rq[j] < 0 || (T > 1 && LAST && !own[j]))
                continue;
            const int li = place(j);
            const float* Sc = S + li;
            const V kq = KEEP_K ? kk[j] : *(const V*)&sK[4 * (j == 0 ? tid : 2 * nc - 1 - tid)];
            const V cen = CEN ? uc[j] : *(const V*)Sc;
            float xs[4 + 2 * HQ];
#pragma unroll
            for (int i = 0; i < HB; ++i) {
                const V l = *(const V*)(Sc - HQ + 4 * i), r = *(const V*)(Sc + 4 + 4 * i);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    xs[4 * i + k] = l[k];
                    xs[HQ + 4 + 4 * i + k] = r[k];
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                xs[HQ + k] = cen[k];
            V ay = V(0.f), ax = V(0.f), lap, un;
#pragma unroll
            for (int q = R; q >= 1; --q)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    ax[k] = fmaf(cf.c[1][q], xs[HQ + k + q] + xs[HQ + k - q], ax[k]);
            __builtin_amdgcn_sched_barrier(0);   // bounds the LDS vectors in flight
#pragma unroll
            for (int q = R; q >= 1; --q) {
                const V yp = *(const V*)(Sc + q * W), ym = *(const V*)(Sc - q * W);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    ay[k] = fmaf(cf.c[0][q], yp[k] + ym[k], ay[k]);
                if (q == 3)
                    __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                lap[k] = fmaf(cf.c0, cen[k], ay[k] + ax[k]);
            if (ne > 0) {
                const V si = *(const V*)&sS[(t & 1) * area + li];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    lap[k] += si[k];
            }
            if (damped[j]) {
                V et = eta[j];
                if constexpr (LEAN) {
                    const float dy2 = ey[rq[j] >> 16];
                    const V exv = *(const V*)&ex[4 * (rq[j] & 0xffff)];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        et[k] = fmaf(sp.e[0], dy2, exv[k]);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    un[k] = leapfrog(cen[k], up[j][k], kq[k], lap[k], et[k], sp.half_dt);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    un[k] = leapfrog(cen[k], up[j][k], kq[k], lap[k], 0.f, sp.half_dt);
            }
            if (ragged)
                clip(un, li);
            if (j == 0 && tid < nbq && exchange) {
                const unsigned v3 = __float_as_uint(un[3]), tag = (p.tag + t + 1) << 11;
                const unsigned hi[3] = {tag | (v3 & 0x7ff), tag | (v3 >> 11 & 0x7ff), tag | v3 >> 22};
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    __hip_atomic_store(out + k * ws, (Word)__float_as_uint(un[k]) | (Word)hi[k] << 32,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            *(V*)&Sn[li] = un;
            if constexpr (MODE == kStepV)
                vv[j] = lap;
            if constexpr (ADJ && T == 1) {
                if (t > 0)
                    image(j, up[j], vv[j]);     // the previous step's term
            }
            if constexpr (ADJ && T > 1 && LAST) {
                image(j, up[j], vv[j]);
                image(j, cen, v2[j]);
            }
            // (a ring quad's next step has the same u^{n-1} two steps on)
            up[j] = CEN || own[j] ? cen : un;
            if constexpr (CEN)
                uc[j] = un;
        }
        if (ns > 0)
            sample(S, p.step + p.dir * t);
        if constexpr (J == 1)
            next_inject();
        if (exchange && hl >= 0) {
            const Word* w = hw + (t0 / T & 1) * parity;
            const unsigned want = (p.tag + t + 1) << 11;
            V v;
            for (int tries = 1;; ++tries) {
                unsigned hi[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const Word x = __hip_atomic_load(w + k * ws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    hi[k] = (unsigned)(x >> 32) ^ want;     // < 2^11: of this step
                    v[k] = __uint_as_float((unsigned)x);
                }
                if ((hi[0] | hi[1] | hi[2]) < 0x800u) {
                    v[3] = __uint_as_float(hi[0] | hi[1] << 11 | hi[2] << 22);
                    break;
                }
                if ((tries & look) == 0) {
                    const bool late = tries >= p.patience;
                    if (late)
                        __hip_atomic_store(p.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (late || __hip_atomic_load(p.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        bad = t + 1;
                        break;
                    }
                }
            }
            *(V*)&Sn[hl] = v;
        }
        // v after the poll: loads return in order, and a poll would wait for v
        if constexpr (MODE == kStepV) {
            if (t >= p.v_from) {
                const auto rV = plane_rsrc(p.V + (t - p.v_from) * p.vstride, fbytes);
#pragma unroll
                for (int j = 0; j < J; ++j)
                    bstorev_nt<4>(rV, field(j), vv[j]);
            }
        }
        if constexpr (ADJ && T == 1)
            load_v(vv, t);
        if constexpr (ADJ && T > 1 && LAST)
            if (t + 1 < p.count) {
                load_v(vv, t + 1);
                if (t + 2 < p.count)
                    load_v(v2, t + 2);
            }
        __syncthreads();
        return more && bad != t + 1;
    };
    for (int t = 0;; t += T) {
        if (!step(std::integral_constant<int, 0>{}, t))
            break;
        if constexpr (T > 1)
            if (!step(std::integral_constant<int, T - 1>{}, t))
                break;
    }
    if (bad)
        return;
    const int end = T == 1 ? p.count & 1 : p.count % T;      // buffer of the final state
    if (p.sample_last && ns > 0)
        sample(buf + end * area, p.step + p.dir * p.count);
    if constexpr (ADJ)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            // the last step's term, unless a second step has added it
            if (rq[j] >= 0 && (T == 1 || end == 1))
                image(j, up[j], vv[j]);
            bstorev<4>(plane_rsrc(p.G, fbytes), field(j), gg[j]);
        }
    if (p.A2)
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if constexpr (!CEN)
                if (rq[j] >= 0)
                    uc[j] = *(const V*)&buf[end * area + place(j)];
            bstorev<4>(plane_rsrc(p.A2, fbytes), field(j), uc[j]);
            bstorev<4>(plane_rsrc(p.B2, fbytes), field(j), up[j]);
        }
}
