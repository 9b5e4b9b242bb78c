// The SAP phase of one block in the even-odd site order at omega = 1, for FP16 / BF16 storage:
// the body shared by the single-source kernel (csrc/sap_eo.hip) and the batched one
// (csrc/batch.hip).  It computes what k_sap_phase_parts computes (Algorithm 1 fused with the
// M_SAP update, SSOR block inverse in even-odd order, section 3 "Inverse of block operator").
//
// One lane per site; a thread keeps one even and one odd site for the whole phase, with their
// sixteen links (96 registers, two 16-bit reals each) and clover blocks (72).  So the sweeps read
// nothing but the neighbours' iterate in LDS, every lane has work in every half-update, and four
// 4^4 blocks (of two waves) share a CU.  The two-lane kernel reloads links and clover rows in
// every half-sweep (450 KB per 4^4 block, more than the L2 holds for the blocks in flight) and
// needs 1.27 times the vector instructions per site in FP16 (two lanes of 848 against 1336: its
// lanes transpose links with selects, both compute addresses, and add two halves).  A phase at 32^3x64
// in 4^4 blocks of FP16 took 538 us and takes 303, 278 in the cycles between a call's first and last
// (BF16 263).  From 4 to 8 SSOR iterations one adds 41 us (BF16 30), so the four take about 155:
// bound by the issue of their vector instructions, of which FP16 has 864 v_fma_mix_f32 at 4.4
// cycles and 472 plain ones at 2.7 (two waves a SIMD), BF16 1528 with 96 shifts at 4.4.  The other
// 123 us are the first loads and the gather, the residual's half-update (20) and the outputs,
// 432 bytes per site in all.  One site per thread, with half the waves idle in each half-update,
// took 365.
//
// At omega = 1 the sweeps are 2 n_ssor half-updates o, e, o, e, ...: the first update of the even
// sites from x = 0 gives x_e = v_e, and the plane at each turn of a sweep keeps its values.  After
// the last one x_e = v_e + K_eo x_o, so the block residual of the even sites is zero (or x not finite)
// and only the odd sites' is computed.
//
// The gather of the other colour runs over the block's faces, one direction pair at a time
// (forward and backward faces of a direction share no site), into accumulators in LDS: a face of
// a 4^4 block is one wave, where a loop over sites would run every direction with three lanes in
// four masked.
#pragma once

#include "twolane.h"

namespace sapq {

// tables of the even-odd kernel, from the context (device pointers)
struct EoTables {
    int Ve, T;             // even sites; threads
    const uint4 *nb;       // [Vb] LDS slots of the neighbours +x -x +y -y +z -z +t -t (16 bits each),
                           // Vb (the zero slot) for a neighbour outside the block
    const unsigned *face;  // [4][2 Vb] per direction the sites of the forward face, then those of the
                           // backward one: slot | slot of the neighbour in the next block << 16
    int nface[4];          // sites of a face of direction mu
};

EoTables eo_tables(const Ctx *c);

constexpr int EO_THREADS = 512;  // at two waves per SIMD, which 256 registers allow

// LDS: the iterate (or the gather's accumulators) float4 [6][NS] (slot Vb stays zero, Vb + 1 is
// spare), then v uint4 [2][3][T].  The pitch NS is a compile-time constant, the smallest of three
// that holds the block, so that the six reads of a neighbour share one address.
constexpr int EO_NS[3] = {258, 514, 1026};
inline int eo_class(int Vb) { return Vb + 2 <= EO_NS[0] ? 0 : Vb + 2 <= EO_NS[1] ? 1 : 2; }
inline size_t eo_lds_bytes(int Vb, int T) { return (size_t)96 * EO_NS[eo_class(Vb)] + (size_t)96 * T; }
// the most that any block of Vb's pitch takes: the limit to set for the kernel they share
inline int eo_lds_limit(int Vb) {
    const int most = EO_NS[eo_class(Vb)] - 2;
    return (int)eo_lds_bytes(most, most / 2);
}

__device__ __forceinline__ unsigned raw2(__half2 v) { return *reinterpret_cast<unsigned *>(&v); }
__device__ __forceinline__ unsigned raw2(__hip_bfloat162 v) { return *reinterpret_cast<unsigned *>(&v); }
template <typename S2> __device__ __forceinline__ cx<float> from_raw(unsigned w) {
    const S2 v = *reinterpret_cast<const S2 *>(&w);
    return ld(&v);
}
template <typename S2> __device__ __forceinline__ unsigned to_raw(cx<float> v) {
    S2 o;
    st(&o, v);
    return raw2(o);
}
// the iterate of this kernel is planar, float4 [6][NS]
__device__ __forceinline__ void lds_planar(cx<float> psi[12], const float4 *xs, int NS, int slot) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const float4 f = xs[q * NS + slot];
        psi[2 * q] = {f.x, f.y};
        psi[2 * q + 1] = {f.z, f.w};
    }
}
// keeps the compiler from hoisting what it derives from w (conversions, third link rows) out of
// the sweep loop, where it would have to spill them
__device__ __forceinline__ void opaque(unsigned &w) { asm volatile("" : "+v"(w)); }

// Products whose first factor comes from 16-bit storage.  The first product of a sum is a fused
// multiply-add onto zero, not a multiply, so that the compiler can read the factor from its FP16
// half (v_fma_mix_f32) instead of converting it first: 1336 vector instructions a site update
// instead of 1420.  (BF16 converts by shifts and masks, and has the same 1528 either way.)
__device__ __forceinline__ cx<float> emul(cx<float> a, cx<float> b) {
    return {fmx(a.r, b.r, -fmx(a.i, b.i, 0.f)), fmx(a.r, b.i, fmx(a.i, b.r, 0.f))};
}
__device__ __forceinline__ cx<float> emulc(cx<float> a, cx<float> b) {  // conj(a) b
    return {fmx(a.r, b.r, fmx(a.i, b.i, 0.f)), fmx(a.r, b.i, -fmx(a.i, b.r, 0.f))};
}

// g = U h or U^+ h from the rows 0 and 1 of U; row 2 = conj(row 0 x row 1)
__device__ __forceinline__ void eo_row2(cx<float> u[9]) {
    const cx<float> m1 = {-u[1].r, -u[1].i}, m2 = {-u[2].r, -u[2].i}, m0 = {-u[0].r, -u[0].i};
    u[6] = conjx(cfma(m2, u[4], emul(u[1], u[5])));
    u[7] = conjx(cfma(m0, u[5], emul(u[2], u[3])));
    u[8] = conjx(cfma(m1, u[3], emul(u[0], u[4])));
}
template <bool DAG> __device__ __forceinline__ void eo_mul(cx<float> g[3], const cx<float> u[9], const cx<float> h[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
        g[a] = DAG ? cfmac(u[6 + a], h[2], cfmac(u[3 + a], h[1], emulc(u[a], h[0])))
                   : cfma(u[3 * a + 2], h[2], cfma(u[3 * a + 1], h[1], emul(u[3 * a], h[0])));
}

// acc (+)= (1 -+ gamma_mu) W psi, W = U (forward) or U^+ (backward), from the stored rows of U
template <int MU, bool BWD, bool FIRST>
__device__ __forceinline__ void hop_site(cx<float> acc[12], const cx<float> psi[12], cx<float> u[9]) {
    constexpr float s = BWD ? -1.f : 1.f;
    eo_row2(u);
    cx<float> h0[3], h1[3], g0[3], g1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<float> p0 = psi[a], p1 = psi[3 + a], p2 = psi[6 + a], p3 = psi[9 + a];
        if (MU == 0) { h0[a] = rfma(s, itimes(p3), p0);  h1[a] = rfma(s, itimes(p2), p1); }
        if (MU == 1) { h0[a] = rfma(s, p3, p0);          h1[a] = rfma(-s, p2, p1); }
        if (MU == 2) { h0[a] = rfma(s, itimes(p2), p0);  h1[a] = rfma(-s, itimes(p3), p1); }
        if (MU == 3) { h0[a] = rfma(-s, p2, p0);         h1[a] = rfma(-s, p3, p1); }
    }
    eo_mul<BWD>(g0, u, h0);
    eo_mul<BWD>(g1, u, h1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        cx<float> l2, l3;
        if (MU == 0) { l2 = -s * itimes(g1[a]); l3 = -s * itimes(g0[a]); }
        if (MU == 1) { l2 = -s * g1[a];         l3 = s * g0[a]; }
        if (MU == 2) { l2 = -s * itimes(g0[a]); l3 = s * itimes(g1[a]); }
        if (MU == 3) { l2 = -s * g0[a];         l3 = -s * g1[a]; }
        acc[a] = FIRST ? g0[a] : acc[a] + g0[a];
        acc[3 + a] = FIRST ? g1[a] : acc[3 + a] + g1[a];
        acc[6 + a] = FIRST ? l2 : acc[6 + a] + l2;
        acc[9 + a] = FIRST ? l3 : acc[9 + a] + l3;
    }
}

// a block's site in registers
struct EoSite {
    unsigned u[8][6];  // U_mu at the site and at its backward neighbour, mu = x, y, z, t
    unsigned f[2][18]; // the two chiral blocks of F
};

template <typename S2, int NS, int D>
__device__ __forceinline__ void eo_hop(cx<float> acc[12], const EoSite &q, uint4 nb, const float4 *xs) {
    const unsigned w = D < 4 ? (D < 2 ? nb.x : nb.y) : (D < 6 ? nb.z : nb.w);
    cx<float> psi[12], u[9];
    lds_planar(psi, xs, NS, (int)(D % 2 ? w >> 16 : w & 0xffffu));
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = from_raw<S2>(q.u[D][e]);
    hop_site<D / 2, D % 2 == 1, D == 0>(acc, psi, u);
}

// out = F in for both chiral blocks (clover_apply with conversion-free first products)
template <typename S2> __device__ __forceinline__ void eo_clover(cx<float> out[12], const cx<float> in[12], const EoSite &q) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        cx<float> f[18];
#pragma unroll
        for (int e = 0; e < 18; ++e) f[e] = from_raw<S2>(q.f[k][e]);
        const cx<float> *B = f + 9, *u = in + 6 * k, *l = u + 3;
        cx<float> *o = out + 6 * k;
        auto d = [](float w, cx<float> v) { return cx<float>{fmx(w, v.r, 0.f), fmx(w, v.i, 0.f)}; };
        o[0] = cfma(B[2], l[2], cfma(B[1], l[1], cfma(B[0], l[0], cfmac(f[4], u[2], cfmac(f[3], u[1], d(f[0].r, u[0]))))));
        o[1] = cfma(B[5], l[2], cfma(B[4], l[1], cfma(B[3], l[0], cfmac(f[5], u[2], cfma(f[3], u[0], d(f[0].i, u[1]))))));
        o[2] = cfma(B[8], l[2], cfma(B[7], l[1], cfma(B[6], l[0], cfma(f[5], u[1], cfma(f[4], u[0], d(f[1].r, u[2]))))));
        o[3] = cfmac(f[7], l[2], cfmac(f[6], l[1], cfmac(B[6], u[2], cfmac(B[3], u[1], cfmac(B[0], u[0], d(f[1].i, l[0]))))));
        o[4] = cfmac(f[8], l[2], cfma(f[6], l[0], cfmac(B[7], u[2], cfmac(B[4], u[1], cfmac(B[1], u[0], d(f[2].r, l[1]))))));
        o[5] = cfma(f[8], l[1], cfma(f[7], l[0], cfmac(B[8], u[2], cfmac(B[5], u[1], cfmac(B[2], u[0], d(f[2].i, l[2]))))));
    }
}

// out = F sum of the site's in-block hops of the iterate
template <typename S2, int NS>
__device__ __forceinline__ void eo_apply(cx<float> out[12], EoSite &q, uint4 nb, const float4 *xs) {
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
        for (int e = 0; e < 6; ++e) opaque(q.u[m][e]);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 18; ++e) opaque(q.f[k][e]);
    cx<float> acc[12];
#define EO_HOP(D) eo_hop<S2, NS, D>(acc, q, nb, xs); __builtin_amdgcn_sched_barrier(0);
    EO_HOP(0) EO_HOP(1) EO_HOP(2) EO_HOP(3) EO_HOP(4) EO_HOP(5) EO_HOP(6) EO_HOP(7)
#undef EO_HOP
    eo_clover<S2>(out, acc, q);
}

// A hop of the gather, one of direction MU that leaves the block: its site, the neighbour's spinor
// and the link as stored.  Each thread takes one per direction (a few more where two faces have
// more sites than the workgroup has threads), and all four directions' loads are issued before
// the first is used.
struct EoFace {
    int s;  // slot of the site, -1: none
    unsigned psi[12], u[6];
};

template <int MU, typename S2>
__device__ __forceinline__ void eo_face_load(EoFace &f, const GeomDev &g, const EoTables &t, const S2 *x, const S2 *U, int ib,
                                             int k) {
    const int nf = t.nface[MU];
    f.s = -1;
    if (k >= 2 * nf) return;
    const unsigned w = t.face[2 * MU * g.Vb + k];
    const bool bwd = k >= nf;
    const int bl = (bwd ? g.blk_nbr[(2 * MU + 1) * g.NB + ib] : g.blk_nbr[(2 * MU) * g.NB + ib]) & BLK_MASK;
    const int sn = (int)(w >> 16);
    f.s = (int)(w & 0xffffu);
    const S2 *p = x + (size_t)bl * 12 * g.Vb + sn;
#pragma unroll
    for (int c = 0; c < 12; ++c) f.psi[c] = raw2(p[(size_t)c * g.Vb]);
    const S2 *l = U + ((size_t)(bwd ? bl : ib) * 4 + MU) * 6 * g.Vb + (bwd ? sn : f.s);
#pragma unroll
    for (int e = 0; e < 6; ++e) f.u[e] = raw2(l[(size_t)e * g.Vb]);
}

// the hop added into the accumulators of its site
template <int MU, bool BWD, typename S2, int NS>
__device__ __forceinline__ void eo_face_hop(float4 *xs, const EoFace &f, const GeomDev &g, int ib) {
    const float ph = (g.blk_nbr[(2 * MU + BWD) * g.NB + ib] & WRAP_BIT) ? g.bc[MU] : 1.f;
    cx<float> psi[12], u[9], acc[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = ph * from_raw<S2>(f.psi[c]);
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = from_raw<S2>(f.u[e]);
    hop_site<MU, BWD, true>(acc, psi, u);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        float4 *o = &xs[q * NS + f.s];
        const float4 a = *o;
        *o = make_float4(a.x + acc[2 * q].r, a.y + acc[2 * q].i, a.z + acc[2 * q + 1].r, a.w + acc[2 * q + 1].i);
    }
}

// both faces of direction MU, whose sites differ; f: this thread's first hop, already loaded
template <int MU, typename S2, int NS>
__device__ __forceinline__ void eo_faces(float4 *xs, EoFace &f, const GeomDev &g, const EoTables &t, const S2 *x, const S2 *U,
                                         int ib) {
    const int nf = t.nface[MU];
    for (int k = threadIdx.x;;) {
        // the two faces in separate branches: a wave mostly holds one of them
        if (f.s >= 0) {
            if (k < nf)
                eo_face_hop<MU, false, S2, NS>(xs, f, g, ib);
            else
                eo_face_hop<MU, true, S2, NS>(xs, f, g, ib);
        }
        k += blockDim.x;
        if (k >= 2 * nf) break;
        eo_face_load<MU>(f, g, t, x, U, ib, k);
    }
    __syncthreads();
}

template <typename S2>
__device__ __forceinline__ void eo_load(EoSite &q, const EoTables &t, const S2 *U, const S2 *F, int ib, int Vb, int s) {
    const uint4 nb = t.nb[s];
    const size_t lstride = (size_t)6 * Vb;
    const S2 *Ub = U + (size_t)ib * 4 * lstride;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const unsigned w = mu == 0 ? nb.x : mu == 1 ? nb.y : mu == 2 ? nb.z : nb.w;
        const int sb = min((int)(w >> 16), Vb - 1);  // outside: any link, the spinor is the zero slot
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            q.u[2 * mu][e] = raw2(Ub[mu * lstride + (size_t)e * Vb + s]);
            q.u[2 * mu + 1][e] = raw2(Ub[mu * lstride + (size_t)e * Vb + sb]);
        }
    }
    const S2 *Fb = F + (size_t)ib * 36 * Vb + s;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 18; ++e) q.f[k][e] = raw2(Fb[(size_t)(18 * k + e) * Vb]);
}

// v of a site in storage precision, to and from LDS (read back by the same thread only)
template <typename S2> __device__ __forceinline__ void eo_put_v(uint4 *vs, int n, const cx<float> v[12]) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
        vs[k * n] = make_uint4(to_raw<S2>(v[4 * k]), to_raw<S2>(v[4 * k + 1]), to_raw<S2>(v[4 * k + 2]), to_raw<S2>(v[4 * k + 3]));
}
template <typename S2> __device__ __forceinline__ void eo_get_v(cx<float> v[12], const uint4 *vs, int n) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint4 w = vs[k * n];
        v[4 * k] = from_raw<S2>(w.x);
        v[4 * k + 1] = from_raw<S2>(w.y);
        v[4 * k + 2] = from_raw<S2>(w.z);
        v[4 * k + 3] = from_raw<S2>(w.w);
    }
}
template <int NS> __device__ __forceinline__ void eo_put_x(float4 *xs, int s, const cx<float> v[12]) {
#pragma unroll
    for (int c = 0; c < 6; ++c) xs[c * NS + s] = make_float4(v[2 * c].r, v[2 * c].i, v[2 * c + 1].r, v[2 * c + 1].i);
}

// x <- v + kappa F H x at the site, x in v
template <typename S2, int NS>
__device__ __forceinline__ void eo_update(cx<float> v[12], EoSite &q, const EoTables &t, const float4 *xs, const uint4 *vs,
                                          int n, int s, float kappa) {
    cx<float> fh[12];
    eo_apply<S2, NS>(fh, q, t.nb[s], xs);
    eo_get_v<S2>(v, vs, n);
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = rfma(kappa, fh[c], v[c]);
}

// a spinor of the solver's layout as stored
template <typename S2> __device__ __forceinline__ void eo_fetch(unsigned w[12], const S2 *f, int ib, int Vb, int s) {
#pragma unroll
    for (int c = 0; c < 12; ++c) w[c] = raw2(f[((size_t)ib * 12 + c) * Vb + s]);
}

// The phase of block ib.  rsrc: the vector the block's v is taken from; r, x, y as in
// k_sap_phase_parts; ssor_only: v = rsrc and only x is written.  NS: pitch of the LDS rows.
// After a phase the residual of the even sites is zero, so the next phase of the colour does not
// read it (EO_R_ZERO) and it is only written by the last one (EO_LAST), for whoever reads r then.
enum { EO_GATHER = 1, EO_FIRST = 2, EO_SSOR_ONLY = 4, EO_R_ZERO = 8, EO_LAST = 16 };

template <int P, int NS>
__device__ __forceinline__ void eo_phase(const GeomDev &g, const EoTables &t, float4 *xs, int ib, int mode, int n_ssor,
                                         float kappa, const typename Prec<P>::S2 *rsrc, typename Prec<P>::S2 *r,
                                         typename Prec<P>::S2 *x, typename Prec<P>::S2 *y,
                                         const typename Prec<P>::S2 *__restrict__ U,
                                         const typename Prec<P>::S2 *__restrict__ F) {
    using S2 = typename Prec<P>::S2;
    const int Vb = g.Vb, n = blockDim.x;
    const int se = min((int)threadIdx.x, t.Ve - 1), so = min(t.Ve + (int)threadIdx.x, Vb - 1);
    // threads without a site work on the last one's data and put it into the spare slot
    const bool live_e = (int)threadIdx.x < t.Ve, live_o = t.Ve + (int)threadIdx.x < Vb;
    const int we = live_e ? se : Vb + 1, wo = live_o ? so : Vb + 1;
    uint4 *ve = reinterpret_cast<uint4 *>(xs + 6 * NS) + threadIdx.x, *vo = ve + 3 * n;

    // 1. v = r + kappa F (hops leaving the block), kept in storage precision; x_e = v_e
    EoFace f0, f1, f2, f3;
    if (mode & EO_GATHER) {
        eo_face_load<0>(f0, g, t, x, U, ib, threadIdx.x);
        eo_face_load<1>(f1, g, t, x, U, ib, threadIdx.x);
        eo_face_load<2>(f2, g, t, x, U, ib, threadIdx.x);
        eo_face_load<3>(f3, g, t, x, U, ib, threadIdx.x);
    }
    unsigned re[12], ro[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) re[c] = 0;
    if (!(mode & EO_R_ZERO)) eo_fetch(re, rsrc, ib, Vb, se);
    eo_fetch(ro, rsrc, ib, Vb, so);
    EoSite qe, qo;
    eo_load(qe, t, U, F, ib, Vb, se);
    for (int k = threadIdx.x; k < 6 * NS; k += n) xs[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    if (mode & EO_GATHER) {
        eo_faces<0, S2, NS>(xs, f0, g, t, x, U, ib);
        eo_faces<1, S2, NS>(xs, f1, g, t, x, U, ib);
        eo_faces<2, S2, NS>(xs, f2, g, t, x, U, ib);
        eo_faces<3, S2, NS>(xs, f3, g, t, x, U, ib);
    }
    eo_load(qo, t, U, F, ib, Vb, so);
    auto start = [&](EoSite &q, const unsigned *rw, int s, int w, uint4 *vs) {
        cx<float> v[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = from_raw<S2>(rw[c]);
        if (mode & EO_GATHER) {
            cx<float> h[12], fh[12];
            lds_planar(h, xs, NS, s);
            eo_clover<S2>(fh, h, q);
#pragma unroll
            for (int c = 0; c < 12; ++c) v[c] = rfma(kappa, fh[c], v[c]);
        }
        eo_put_v<S2>(vs, n, v);
        eo_get_v<S2>(v, vs, n);
        eo_put_x<NS>(xs, w, v);
    };
    start(qe, re, se, we, ve);
    start(qo, ro, so, wo, vo);
    __syncthreads();

    // 2. half-updates x <- v + kappa F H x, odd sites first
    for (int k = 0; k < n_ssor; ++k) {
        cx<float> v[12];
        eo_update<S2, NS>(v, qo, t, xs, vo, n, so, kappa);
        eo_put_x<NS>(xs, wo, v);
        __syncthreads();
        eo_update<S2, NS>(v, qe, t, xs, ve, n, se, kappa);
        eo_put_x<NS>(xs, we, v);
        __syncthreads();
    }

    // 3. outputs: x, y += x, r = v - A x (zero on the even sites)
    unsigned ye[12], yo[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) ye[c] = yo[c] = 0;
    if (!(mode & (EO_FIRST | EO_SSOR_ONLY))) {
        eo_fetch(ye, y, ib, Vb, se);
        eo_fetch(yo, y, ib, Vb, so);
    }
    auto finish = [&](const unsigned *yw, int s) {
        cx<float> xv[12], yv[12];
        lds_planar(xv, xs, NS, s);
        store_spinor(x, g, ib, s, xv);
        if (mode & EO_SSOR_ONLY) return;
#pragma unroll
        for (int c = 0; c < 12; ++c) yv[c] = from_raw<S2>(yw[c]) + xv[c];
        store_spinor(y, g, ib, s, yv);
    };
    if (live_e) {
        finish(ye, se);
        if ((mode & (EO_LAST | EO_SSOR_ONLY)) == EO_LAST) {
            // 0, and not a number where x is infinite or none, as v - A x would be
            cx<float> z[12];
            lds_planar(z, xs, NS, se);
#pragma unroll
            for (int c = 0; c < 12; ++c) z[c] = z[c] - z[c];
            store_spinor(r, g, ib, se, z);
        }
    }
    if (live_o) finish(yo, so);
    if (mode & EO_SSOR_ONLY) return;
    cx<float> v[12], xv[12];
    eo_update<S2, NS>(v, qo, t, xs, vo, n, so, kappa);
    lds_planar(xv, xs, NS, so);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        v[c] = v[c] - xv[c];
        asm volatile("" : "+v"(v[c].r), "+v"(v[c].i));  // or the whole update would sink into the branch
    }
    if (live_o) store_spinor(r, g, ib, so, v);
}

}  // namespace sapq
