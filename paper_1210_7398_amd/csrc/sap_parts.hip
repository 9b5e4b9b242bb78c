// SAP phase kernel with two lanes per site, for blocks whose SSOR iterate does not fit
// LDS as a whole: the block is split along t into two workgroups ("parts"), each holding
// the iterate of its own half in LDS.  It computes exactly what k_sap_phase computes
// (Algorithm 1 fused with the M_SAP update, the locally-lexicographic SSOR in hyperplane
// order of the sub-block-local coordinates, section 3 "Inverse of block operator" and Fig. 1):
//   v_c = r_c + kappa F sum_{hops leaving the block} H x_other
//   x_c = n_ssor forward + backward sweeps from 0,  y_c += x_c,  r_c = v_c - D_cc x_c.
//
// Lanes.  Lane d = 0 of a pair takes the four forward hops of its site, lane d = 1 the
// four backward hops.  Both run the same instructions: the projection sign is s = +1 / -1,
// and lane 1 reads U_mu at its backward neighbour, transposes it with selects and works on
// conjugates, whose signs ride on multiply-adds (a daggered copy of the links at the site would
// cost a quarter more bytes per sweep).  After
// the pair's sum each lane owns one chiral half (spins 2d and 2d + 1), applies its 6x6
// block of F and updates those six components.
//
// Parts.  The sub-block layers along t are split in halves.  Only hops in t cross between
// the halves, and they connect the last t-layer of a sub-block to the first one of the
// next, whose hyperplanes differ by S_t - 1: the data one part needs from the other were
// produced S_t - 1 steps earlier (new values) or in the previous sweep (old values).
// Each part publishes its boundary layer after every update into a global array of
// 64-bit words (value, tag), the tag naming launch and sweep; the other part copies the
// words it needs for its next step into LDS halo slots, waiting (bounded) on the tag.
// Sweep w's words go to slot w mod 3, which a part can only reuse after the reader has
// moved on (writing sweep w + 3 needs the reader's sweep w + 2 data).  The two parts of a
// block take their block from a ticket counter in start order, so a part only ever waits
// on a part that is already running; the last workgroup resets the counter.
//
// What bounds it: the dependent chain of a hyperplane step (table entries, loads, LDS reads, about
// 800 vector instructions of a site update per lane, LDS store, barrier), with one or two waves a
// SIMD.  Cycle stamps of the 24^3x48 launch showed 2700 of a step's 13000 cycles outside the
// update: every wave copied a share of the halo words (with integer divisions by their number),
// read the hyperplane starts from LDS, and a pointer choice between LDS and global memory made flat
// loads, after which every wait is for all loads in flight.  With a wave of its own for the halo
// words, the starts in registers (v_readlane), record-wise LDS, the dagger of the backward links
// folded into signs the instructions take anyway (902 -> 760, 798 in the present lane order) and no
// relaxation arithmetic at omega = 1, a launch takes 458 us instead of 533 (FP32, 6^3x12 blocks,
// the same bits), now 450 to 458.  Its requests leaving the L2s are 2.7 GB, 6.0 TB/s, which the
// last-level cache and memory serve together (a colour's links, clover and v are 191 MB); with
// every load an L2 hit it would take 390, so the chain is the larger part.  Measured and not kept:
// a site's links, or all it needs, loaded a step ahead (507 us with two hops' links, 10% slower
// than without once the waits were exact; all of it spills in FP32 and gains nothing in FP16).
#include <algorithm>
#include <type_traits>

#include "twolane.h"

namespace sapq {

struct PartArgs {
    int colour, gather, first, ssor_only, n_ssor;
    float kappa, omega;
    int Vp, Hp;
    int sweep_waves, halo_wave;  // waves that update sites; the wave that copies halo words
    const int *gslot;         // [NP][Vp] block slot of each part-local site
    const uint2 *pnb;         // [NP][Vp][2] LDS slots of the 4 neighbours of lane d (16 bits each)
    const uint2 *gnb;         // [NP][Vp] block slots of the 4 backward neighbours (16 bits each)
    const int *pstart;        // [MAX_PLANES + 1] part-local hyperplane starts
    const int *exp_idx;       // [NP][Vp] index in the part's boundary layer, or -1
    const int *imp;           // [NP][Hp] halo slots, ordered by the hyperplane that reads them
    const int *imp_start;     // [NP][MAX_PLANES + 1]
    unsigned long long *xch;  // [NBc][NP][3][24][Hp]
    unsigned *sync;           // [0] ticket, [1] done, [2] epoch, [3] error
    int spin_limit;           // bounded wait on a halo word, in polls
    unsigned wait_xor;        // 0; nonzero only where a test forces the time-out path (no
                              // written word then carries the awaited tag)
};

__device__ __forceinline__ unsigned xch_tag(unsigned epoch, int sweep) {
    return 0x80000000u | ((epoch & 0x1ffffffu) << 6) | (unsigned)(sweep & 63);
}
__device__ __forceinline__ void xch_put(unsigned long long *p, float v, unsigned tag) {
    const unsigned long long w = ((unsigned long long)tag << 32) | __float_as_uint(v);
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long xch_get(unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the word at p once it carries `tag`; on time-out the error flag is raised and the caller
// stops waiting for the rest of the launch (the result is then discarded by the host)
__device__ __forceinline__ float xch_wait(unsigned long long w, unsigned long long *p, unsigned tag, bool &gave_up,
                                          const PartArgs &a) {
    tag ^= a.wait_xor;
    if ((unsigned)(w >> 32) != tag && !gave_up) {
        int it = 0;
        do {
            __builtin_amdgcn_s_sleep(2);
            w = xch_get(p);
        } while ((unsigned)(w >> 32) != tag && ++it < a.spin_limit);
        if ((unsigned)(w >> 32) != tag) {
            gave_up = true;
            __hip_atomic_store(&a.sync[3], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    return __uint_as_float((unsigned)w);
}

// barrier for LDS traffic only: global loads (halo words) and stores stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ALONE: the workgroup has a CU to itself.  A whole block (NP = 1) then takes four lanes per site on the
// hyperplanes that its waves hold that way, and up to 12 waves: on an idle CU a step lasts as long as
// one wave's instructions and their latency (5900 cycles at 4^4 blocks with two lanes), and
// the wider planes need fewer passes.  Measured, M_SAP in FP32 unless said, two lanes -> four:
// 4^4 blocks 813 -> 696 us (8 workgroups), 842 -> 733 (128), 963 -> 793 (256), but 1191 -> 1485
// (384, where CUs are shared and issue slots are what is short: that kernel stays at
// two lanes); 6^4 2115 -> 1968 (8), 5794 -> 5692 (384, alone by its LDS), in BF16 5107 -> 4627
// (512); 6x4x10x6 in BF16 2342 -> 2011 (24).  A split block waits on its halo words, not on its own update
// (two lanes 2773, four 2936 us at 12^3x24): it keeps two lanes, and where it is alone the
// staged load order (block_hop_clover_impl), whose 40 registers more are free there.
template <int P, int NP, bool ALONE>
__global__ void __launch_bounds__(NP == 1 && ALONE ? 768 : 512, NP == 2 && ALONE ? 2 : 3) k_sap_phase_parts(GeomDev g, PartArgs a, const typename Prec<P>::S2 *rsrc,
                                                         typename Prec<P>::S2 *r, typename Prec<P>::S2 *x,
                                                         typename Prec<P>::S2 *y,
                                                         const typename Prec<P>::S2 *__restrict__ U,
                                                         const typename Prec<P>::S2 *__restrict__ F) {
    using S2 = typename Prec<P>::S2;
    constexpr bool FOUR = NP == 1 && ALONE, STAGED = NP == 2 && ALONE;
    extern __shared__ float4 xs[];
    __shared__ unsigned sh_ticket;
    const int Vb = g.Vb, Vp = a.Vp, Hp = a.Hp;
    int blk = blockIdx.x, part = 0;
    unsigned epoch = 0;
    if (NP == 2) {
        if (threadIdx.x == 0) sh_ticket = atomicAdd(&a.sync[0], 1u);
        __syncthreads();
        const unsigned t = sh_ticket;
        if (t >= gridDim.x) {  // counter out of step with the launch: flag it and do nothing
            if (threadIdx.x == 0) __hip_atomic_store(&a.sync[3], 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        blk = (int)(t >> 1);
        part = (int)(t & 1u);
        epoch = __hip_atomic_load(&a.sync[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int ib = a.colour * g.NBc + blk;
    const int d = pair_dir(threadIdx.x);
    const int q0 = pair_site(threadIdx.x), nq = blockDim.x >> 1;
    const float sg = d ? -1.f : 1.f;
    const float kappa = a.kappa, omega = a.omega;
    const int *gslot = a.gslot + (size_t)part * Vp;
    const uint2 *pnb = a.pnb + (size_t)part * Vp * 2;
    const int *expi = a.exp_idx + (size_t)part * Vp;
    const int *imp = a.imp + (size_t)part * Hp;
    const int *imps = a.imp_start + (size_t)part * (MAX_PLANES + 1);
    const size_t xstride = (size_t)3 * 24 * Hp;
    unsigned long long *xo = a.xch + ((size_t)blk * NP + part) * xstride;
    unsigned long long *xi = a.xch + ((size_t)blk * NP + (part ^ 1)) * xstride;
    const uint2 *gnb = a.gnb + (size_t)part * Vp;
    const S2 *Fk = F + ((size_t)ib * 2 + d) * 18 * Vb;
    const S2 *vb = a.ssor_only ? rsrc : r;
    float *xsf = reinterpret_cast<float *>(xs);
    bool gave_up = false;

    // 1. v_c (gathering the other colour), zero the iterate, the halo slots and the zero slot
    {
        int bl[4];
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) bl[mu] = g.blk_nbr[(2 * mu + d) * g.NB + ib];
        for (int i = q0; i < Vp; i += nq) {
            const int s = gslot[i];
            if (!a.ssor_only) {
                cx<float> v[6];
                load6(v, rsrc, ib, s, d, Vb);
                if (a.gather) {
                    cx<float> acc[12];
#pragma unroll
                    for (int c = 0; c < 12; ++c) acc[c] = cxz<float>();
                    gather_hop<0>(acc, g, x, U, ib, s, d, bl[0], sg);
                    gather_hop<1>(acc, g, x, U, ib, s, d, bl[1], sg);
                    gather_hop<2>(acc, g, x, U, ib, s, d, bl[2], sg);
                    gather_hop<3>(acc, g, x, U, ib, s, d, bl[3], sg);
                    cx<float> own[6], out[6];
                    pair_reduce(own, acc);
                    clover_block(out, own, Fk + s, Vb);
#pragma unroll
                    for (int e = 0; e < 6; ++e) v[e] = v[e] + kappa * out[e];
                }
                store6(r, ib, s, d, Vb, v);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) xs[6 * i + 3 * d + q] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int t = threadIdx.x; t < 6 * (Hp + 1); t += blockDim.x) xs[6 * Vp + t] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();

    // 2. sweeps: x_n <- (1 - omega) x_n + omega (v_n + kappa F(n) sum_{m in block} H_nm x_m)
    const int H = g.nplanes, nsw = 2 * a.n_ssor;
    // The hyperplane and halo-import starts, lane l holding entries l and l + 1: a step reads them
    // with v_readlane, where LDS or global reads would put a round trip at the head of every step.
    const int lane = threadIdx.x & 63;
    const int pl0 = a.pstart[lane], pl1 = a.pstart[lane + 1];
    const int im0 = imps[lane], im1 = imps[lane + 1];
    auto at = [](int v, int h) { return __builtin_amdgcn_readlane(v, h); };
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nwv = blockDim.x >> 6;
    const QuadLane Q = quad_lane(lane);
    // hyperplane h by four lanes per site
    auto by_four = [&](int h) { return FOUR && at(pl1, h) - at(pl0, h) <= 16 * a.sweep_waves; };
    // the boundary words of a site, tagged with the sweep
    auto publish = [&](const cx<float> xn[6], int kx, int w) {
        if (kx < 0) return;
        const unsigned wt = xch_tag(epoch, w);
        unsigned long long *dst = xo + ((w % 3) * 24 + 12 * d) * Hp + kx;
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            xch_put(dst + (2 * e) * Hp, xn[e].r, wt);
            xch_put(dst + (2 * e + 1) * Hp, xn[e].i, wt);
        }
    };
    // The table entries of a site (LDS slots of its neighbours, block slots of its backward
    // neighbours, boundary index) are read one step ahead, for this thread's first site of
    // the coming hyperplane: read at the start of their own step they would put a load round
    // trip ahead of every other load of the step.
    uint2 nb_n = make_uint2(0u, 0u), gl_n = make_uint2(0u, 0u);
    int kx_n = -1;
    auto tables_for = [&](int h) {
        if (by_four(h)) {
            const int i = at(pl0, h) + 16 * wv + (lane & 15);
            if (i < at(pl1, h)) {
                nb_n.x = reinterpret_cast<const unsigned *>(pnb)[4 * i + 2 * Q.d + Q.m];
                gl_n.x = reinterpret_cast<const unsigned *>(gnb)[2 * i + Q.m];
            }
            return;
        }
        const int i = at(pl0, h) + q0;
        if (i < at(pl1, h)) {
            nb_n = pnb[2 * i + d];
            gl_n = gnb[i];
            kx_n = NP == 2 ? expi[i] : -1;
        }
    };
    tables_for(0);
    // The halo words of `n` slots (slot index k(e)) from sweep slot `src`, checked against `tag`, into
    // LDS, one slot per lane: all 24 loads in flight, then the waits.
    auto import_words = [&](int n, auto k_of, int src, unsigned tag) {
        for (int e = lane; e < n; e += 64) {
            const int k = k_of(e);
            unsigned long long *p = xi + (src + k), word[24];
#pragma unroll
            for (int c = 0; c < 24; ++c) word[c] = xch_get(p + c * Hp);
#pragma unroll
            for (int c = 0; c < 24; ++c) xsf[24 * (Vp + k) + c] = xch_wait(word[c], p + c * Hp, tag, gave_up, a);
        }
    };
    for (int w = 0; w < nsw; ++w) {
        const bool fwd = (w & 1) == 0;
        for (int pi = 0; pi < H; ++pi) {
            const int h = fwd ? pi : H - 1 - pi, hn = pi + 1 == H ? h : fwd ? h + 1 : h - 1;
            // (1) the updates; a part-local site i of plane h sits at block slot
            // i + pst[h] + part (pst[h + 1] - pst[h]) (each part owns one contiguous slot
            // range of every hyperplane, part 0 first)
            if (wv < a.sweep_waves) {
                const int i_lo = at(pl0, h), i_hi = at(pl1, h), shift = NP == 2 ? i_lo + part * (i_hi - i_lo) : 0;
                // this thread's first site with the tables read a step ahead, then those of the
                // coming step (at a turn the plane repeats, and so do its tables), then any further
                // sites (a hyperplane with more sites than the workgroup has lane pairs)
                const uint2 nb0 = nb_n, gl0 = gl_n;
                const int kx0 = kx_n, i0 = i_lo + q0, ns = 32 * a.sweep_waves;
                tables_for(hn);
                // At the turn of a sweep (w > 0, pi = 0) the plane repeats: the top corner of the
                // sub-blocks after a forward sweep, the bottom corner after a backward one.  Every
                // neighbour of such a site lies on the side just swept and has not changed since
                // the site's last update, so with omega = 1 (no (1 - omega) x term) the update
                // would give the same value bit for bit: it is skipped and only the boundary
                // words are published again under the new sweep's tag.
                // the new value of N components of site i from component c0 on, from F of its hops and its v
                auto relax = [&](auto n, cx<float> *xn, const cx<float> *out, const cx<float> *v, int i, int c0) {
                    constexpr int N = decltype(n)::value;
#pragma unroll
                    for (int e = 0; e < N; ++e) xn[e] = v[e] + kappa * out[e];
                    if (omega != 1.f) {
                        const float2 *xf = reinterpret_cast<const float2 *>(xs) + 12 * i + c0;
#pragma unroll
                        for (int e = 0; e < N; ++e) {
                            const float2 ov = xf[e];
                            xn[e] = {(1.f - omega) * ov.x + omega * xn[e].r, (1.f - omega) * ov.y + omega * xn[e].i};
                        }
                    }
                };
                if (omega == 1.f && w > 0 && pi == 0) {
                    for (int i = i0; NP == 2 && i < i_hi; i += ns) {
                        cx<float> xn[6];
                        lds_get6(xn, xs, d, i);
                        publish(xn, i == i0 ? kx0 : expi[i], w);
                    }
                } else if (by_four(h)) {
                    const int i = i_lo + 16 * wv + (lane & 15), c0 = 6 * Q.d + 3 * Q.m;
                    if (i < i_hi) {
                        cx<float> out[3], v[3], xn[3];
                        quad_hop_clover_v(out, v, vb, xs, nb0.x, gl0.x, U, F, ib, i + shift, Q, Vb);
                        relax(std::integral_constant<int, 3>(), xn, out, v, i, c0);
                        float2 *xf = reinterpret_cast<float2 *>(xs) + 12 * i + c0;
#pragma unroll
                        for (int e = 0; e < 3; ++e) xf[e] = make_float2(xn[e].r, xn[e].i);
                    }
                } else {
                    auto update = [&](int i, uint2 nb, uint2 gl, int kx) {
                        cx<float> out[6], v[6], xn[6];
                        block_hop_clover_v<STAGED>(out, v, vb, xs, nb, gl, U, Fk, ib, i + shift, d, Vb, sg);
                        relax(std::integral_constant<int, 6>(), xn, out, v, i, 6 * d);
                        lds_put6(xs, d, i, xn);
                        if constexpr (NP == 2) publish(xn, kx, w);
                    };
                    if (i0 < i_hi) update(i0, nb0, gl0, kx0);
                    for (int i = i0 + ns; i < i_hi; i += ns) update(i, pnb[2 * i + d], gnb[i], NP == 2 ? expi[i] : -1);
                }
            }
            // (2) the halo words that the next step reads (each by one site of its plane, so they
            // can be stored while others update), by a wave of their own where the workgroup has
            // room for one: 2700 of the 13000 cycles of a step went into every wave copying a
            // share of them.  A wave that does both updates first, since the other part may be
            // waiting for what it publishes.  At the turn of a sweep the plane repeats and its halo
            // slots already hold the right sweep (or the plane reads none), so nothing is fetched.
            if (NP == 2 && wv == a.halo_wave) {
                // part 0 reads part 1 through +t (lower hyperplane: this sweep's values in a
                // forward sweep); part 1 reads part 0 through -t (higher hyperplane); before the
                // first sweep the halo is zero
                const int ver = ((part == 0) == fwd) ? w : w - 1;
                if (pi + 1 < H && ver >= 0) {
                    const int e0 = at(im0, hn);
                    import_words(at(im1, hn) - e0, [&](int e) { return imp[e0 + e]; }, (ver % 3) * 24 * Hp, xch_tag(epoch, ver));
                }
            }
            lds_barrier();
        }
    }

    // 3. the whole halo at the last sweep, then outputs
    if (NP == 2) {
        const int src = ((nsw - 1) % 3) * 24 * Hp;
        const unsigned tag = xch_tag(epoch, nsw - 1);
        for (int c = wv; c < 24; c += nwv)
            for (int k = lane; k < Hp; k += 64) {
                unsigned long long *p = xi + (src + c * Hp + k);
                xsf[24 * (Vp + k) + c] = xch_wait(xch_get(p), p, tag, gave_up, a);
            }
        __syncthreads();
    }
    for (int i = q0; i < Vp; i += nq) {
        const int s = gslot[i];
        cx<float> xv[6];
        lds_get6(xv, xs, d, i);
        store6(x, ib, s, d, Vb, xv);
        if (a.ssor_only) continue;
        cx<float> yv[6];
        if (a.first) {
#pragma unroll
            for (int e = 0; e < 6; ++e) yv[e] = xv[e];
        } else {
            load6(yv, y, ib, s, d, Vb);
#pragma unroll
            for (int e = 0; e < 6; ++e) yv[e] = yv[e] + xv[e];
        }
        store6(y, ib, s, d, Vb, yv);
        cx<float> out[6], v[6];
        block_hop_clover_v<STAGED>(out, v, r, xs, pnb[2 * i + d], gnb[i], U, Fk, ib, s, d, Vb, sg);
#pragma unroll
        for (int e = 0; e < 6; ++e) v[e] = v[e] - xv[e] + kappa * out[e];
        store6(r, ib, s, d, Vb, v);
    }

    // 4. the last workgroup to finish resets the ticket counter and advances the epoch
    if (NP == 2) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned done = atomicAdd(&a.sync[1], 1u);
            if (done == gridDim.x - 1) {
                __hip_atomic_store(&a.sync[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.sync[2], epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// r_c += kappa F sum_{hops leaving the block} H x  (r_c -= D_{c,other} x_other, the last step
// of M_SAP), two lanes per site; a site with no hop leaving its block is left alone.
template <int P>
__global__ void __launch_bounds__(256) k_sap_face_2l(GeomDev g, int colour, float kappa, typename Prec<P>::S2 *r,
                                                     const typename Prec<P>::S2 *x,
                                                     const typename Prec<P>::S2 *__restrict__ U,
                                                     const typename Prec<P>::S2 *__restrict__ F) {
    const long i = xcd_site_base(128) + pair_site(threadIdx.x);
    const int d = pair_dir(threadIdx.x);
    const long nc = (long)g.NBc * g.Vb;
    if (i >= nc) return;
    const int ib = colour * g.NBc + (int)(i / g.Vb), s = (int)(i % g.Vb);
    bool outside = false;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const unsigned w = g.nbr16[mu * g.Vb + s];
        outside |= !((d ? (w >> 16) : w) & 0x8000u);
    }
    if (!pair_any(outside)) return;  // both lanes of the pair leave together
    const float sg = d ? -1.f : 1.f;
    cx<float> acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = cxz<float>();
    gather_hop<0>(acc, g, x, U, ib, s, d, g.blk_nbr[(2 * 0 + d) * g.NB + ib], sg);
    gather_hop<1>(acc, g, x, U, ib, s, d, g.blk_nbr[(2 * 1 + d) * g.NB + ib], sg);
    gather_hop<2>(acc, g, x, U, ib, s, d, g.blk_nbr[(2 * 2 + d) * g.NB + ib], sg);
    gather_hop<3>(acc, g, x, U, ib, s, d, g.blk_nbr[(2 * 3 + d) * g.NB + ib], sg);
    cx<float> own[6], out[6], v[6];
    pair_reduce(own, acc);
    clover_block(out, own, F + ((size_t)ib * 2 + d) * 18 * g.Vb + s, g.Vb);
    load6(v, r, ib, s, d, g.Vb);
#pragma unroll
    for (int e = 0; e < 6; ++e) v[e] = v[e] + kappa * out[e];
    store6(r, ib, s, d, g.Vb, v);
}

void launch_sap_face_2l(Ctx *c, int colour, void *r, const void *x) {
    const long nc = (long)c->g.NBc * c->g.Vb;
    const unsigned grid = (unsigned)((2 * nc + 255) / 256 + N_XCD - 1) / N_XCD * N_XCD;
    INNER_SWITCH(c->prm.prec_inner, (k_sap_face_2l<P_><<<grid, 256, 0, c->stream>>>(
                                         c->g, colour, (float)c->prm.kappa, (typename Prec<P_>::S2 *)r,
                                         (const typename Prec<P_>::S2 *)x, (const typename Prec<P_>::S2 *)c->Uin,
                                         (const typename Prec<P_>::S2 *)c->Fin)));
}

template <int P> static void *parts_kernel(int np, bool alone) {
    return np == 2 ? (alone ? (void *)k_sap_phase_parts<P, 2, true> : (void *)k_sap_phase_parts<P, 2, false>)
                   : (alone ? (void *)k_sap_phase_parts<P, 1, true> : (void *)k_sap_phase_parts<P, 1, false>);
}
static void *parts_kernel(const Ctx *c) {
    void *fn = nullptr;
    INNER_SWITCH(c->prm.prec_inner, fn = parts_kernel<P_>(c->sap_np, c->parts_alone));
    return fn;
}

void launch_sap_phase_parts(Ctx *c, int colour, int gather, int first, int ssor_only, const void *rsrc, void *r,
                            void *x, void *y) {
    PartArgs a;
    a.colour = colour;
    a.gather = gather;
    a.first = first;
    a.ssor_only = ssor_only;
    a.n_ssor = c->prm.n_ssor;
    a.kappa = (float)c->prm.kappa;
    a.omega = (float)c->prm.omega;
    a.Vp = c->part_Vp;
    a.Hp = c->part_Hp;
    a.gslot = c->part_gslot;
    a.pnb = c->part_nb;
    a.gnb = c->part_gnb;
    a.pstart = c->part_pstart;
    a.exp_idx = c->part_exp;
    a.imp = c->part_imp;
    a.imp_start = c->part_imps;
    a.xch = c->xch;
    a.sync = c->xsync;
    a.spin_limit = c->halo_spin_limit;
    a.wait_xor = c->halo_wait_xor;
    // two lanes per site of the widest hyperplane, and for a split block a wave for the halo words
    // (the last one does both where the sweeps take all eight); with four lanes per site up to the 12 waves
    // that the kernel's registers allow
    const bool four = c->sap_np == 1 && c->parts_alone;
    a.sweep_waves = four ? std::min(12, (c->part_max_plane + 15) / 16) : c->part_threads / 64;
    const int waves = c->sap_np == 2 ? std::min(8, a.sweep_waves + 1) : a.sweep_waves;
    a.halo_wave = waves - 1;
    const dim3 grid(c->g.NBc * c->sap_np), block(64 * waves);
    void *fn = parts_kernel(c);
    GeomDev g = c->g;
    void *args[] = {&g, &a, &rsrc, &r, &x, &y, &c->Uin, &c->Fin};
    (void)hipLaunchKernel(fn, grid, block, args, c->parts_lds, c->stream);
}

int set_parts_lds_limit(Ctx *c) {
    if (!c->use_parts || c->parts_lds <= 65536) return 0;
    (void)hipFuncSetAttribute(parts_kernel(c), hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->parts_lds);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace sapq
