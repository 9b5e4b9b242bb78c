// Two lanes per site: the per-site building blocks of the two-lane SAP phase kernels (one
// source, csrc/sap_parts.hip; several sources, csrc/batch.hip).  Lane d = 0 of a pair takes
// the four forward hops (1 - gamma_mu) U_mu(n) psi(n + mu), lane d = 1 the four backward hops
// (1 + gamma_mu) U_mu(n - mu)^+ psi(n - mu), with U_mu(n - mu) read at the neighbour; both lanes run the same instructions (projection sign s = +1 / -1).
// A pair butterfly adds the two halves, and lane d then owns chiral half d (spins 2d, 2d + 1).
#pragma once

#include "sitecore.h"

namespace sapq {

// (1 - s gamma_mu) W psi accumulated into acc (FIRST: acc is set), W = U on the lanes with s = 1 and
// U^+ on those with s = -1, by the same instructions on both; the projection and the rebuild of
// the lower spins follow the chiral-basis gamma matrices (see sitecore.h).  The backward lanes
// work on conjugates, conj(U^+ h) = U^T conj(h): the transpose is a swap of the off-diagonal
// elements (link_swap), and the sign of the imaginary parts rides on the multiply-adds of the
// projection and of the sums, which take a factor s anyway (conjugating the link itself took
// nine more instructions per hop).  The helpers below are written for the compute type C (float,
// or double for the FP64 operator); the SSOR iterate in LDS is always float.
template <int MU, bool FIRST, typename C>
__device__ __forceinline__ void hop_lane(cx<C> acc[12], const cx<C> psi[12], const cx<C> u[9], C s) {
    cx<C> h0[3], h1[3], g0[3], g1[3];  // conjugated where s = -1
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<C> p0 = psi[a], p1 = psi[3 + a], p2 = psi[6 + a], p3 = psi[9 + a];
        if (MU == 0) { h0[a] = {fmx(-s, p3.i, p0.r), fmx(s, p0.i, p3.r)}; h1[a] = {fmx(-s, p2.i, p1.r), fmx(s, p1.i, p2.r)}; }
        if (MU == 1) { h0[a] = {fmx(s, p3.r, p0.r), fmx(s, p0.i, p3.i)};  h1[a] = {fmx(-s, p2.r, p1.r), fmx(s, p1.i, -p2.i)}; }
        if (MU == 2) { h0[a] = {fmx(-s, p2.i, p0.r), fmx(s, p0.i, p2.r)}; h1[a] = {fmx(s, p3.i, p1.r), fmx(s, p1.i, -p3.r)}; }
        if (MU == 3) { h0[a] = {fmx(-s, p2.r, p0.r), fmx(s, p0.i, -p2.i)}; h1[a] = {fmx(-s, p3.r, p1.r), fmx(s, p1.i, -p3.i)}; }
    }
    su3_mul(g0, u, h0, false);
    su3_mul(g1, u, h1, false);
    // acc + (x, y) or acc + (s x, y), (x, s y) with a sign
    auto ps = [&](cx<C> &o, C x, C y) { o = FIRST ? cx<C>{x, s * y} : cx<C>{o.r + x, fmx(s, y, o.i)}; };
    auto sp = [&](cx<C> &o, C x, C y) { o = FIRST ? cx<C>{s * x, y} : cx<C>{fmx(s, x, o.r), o.i + y}; };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ps(acc[a], g0[a].r, g0[a].i);
        ps(acc[3 + a], g1[a].r, g1[a].i);
        if (MU == 0) { ps(acc[6 + a], g1[a].i, -g1[a].r);  ps(acc[9 + a], g0[a].i, -g0[a].r); }
        if (MU == 1) { sp(acc[6 + a], -g1[a].r, -g1[a].i); sp(acc[9 + a], g0[a].r, g0[a].i); }
        if (MU == 2) { ps(acc[6 + a], g0[a].i, -g0[a].r);  ps(acc[9 + a], -g1[a].i, g1[a].r); }
        if (MU == 3) { sp(acc[6 + a], -g0[a].r, -g0[a].i); sp(acc[9 + a], -g1[a].r, -g1[a].i); }
    }
}

// rows 0, 1 of a stored link and row 2 = conj(row0 x row1)
template <typename C> __device__ __forceinline__ void link_rebuild(cx<C> u[9]) { su3_row2(u); }
template <typename S2, typename C>
__device__ __forceinline__ void link_rows(cx<C> u[9], const S2 *p, int Vb) {
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = ld(p + (size_t)e * Vb);
    link_rebuild(u);
}

// u <- u^T on the lanes with swap set, u unchanged on the others (same instructions on both)
template <typename C> __device__ __forceinline__ void link_swap(cx<C> u[9], bool swap) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a + 1; b < 3; ++b) {
            const cx<C> up = u[3 * a + b], lo = u[3 * b + a];
            u[3 * a + b] = sel(swap, lo, up);
            u[3 * b + a] = sel(swap, up, lo);
        }
}

// one hermitian chiral block [[A, B], [B^+, C]] of F (18 slots, see k_pack_clover)
template <typename C = float> struct Clov { cx<C> f[18]; };

template <typename S2, typename C>
__device__ __forceinline__ void load_clov(Clov<C> &F, const S2 *p, int Vb) {
#pragma unroll
    for (int e = 0; e < 18; ++e) F.f[e] = ld(p + (size_t)e * Vb);
}

// out = F_k in:  slots 0-2 the six real diagonal entries pairwise, 3-5 / 6-8 the strict
// lower triangles of A / C, 9-17 B row by row
template <typename C> __device__ __forceinline__ void clover_apply(cx<C> out[6], const cx<C> in[6], const Clov<C> &F) {
    const cx<C> d01 = F.f[0], d23 = F.f[1], d45 = F.f[2];
    const cx<C> a10 = F.f[3], a20 = F.f[4], a21 = F.f[5], c10 = F.f[6], c20 = F.f[7], c21 = F.f[8];
    const cx<C> *B = F.f + 9;
    const cx<C> u0 = in[0], u1 = in[1], u2 = in[2], l0 = in[3], l1 = in[4], l2 = in[5];
    out[0] = cfma(B[2], l2, cfma(B[1], l1, cfma(B[0], l0, cfmac(a20, u2, cfmac(a10, u1, d01.r * u0)))));
    out[1] = cfma(B[5], l2, cfma(B[4], l1, cfma(B[3], l0, cfmac(a21, u2, cfma(a10, u0, d01.i * u1)))));
    out[2] = cfma(B[8], l2, cfma(B[7], l1, cfma(B[6], l0, cfma(a21, u1, cfma(a20, u0, d23.r * u2)))));
    out[3] = cfmac(c20, l2, cfmac(c10, l1, cfmac(B[6], u2, cfmac(B[3], u1, cfmac(B[0], u0, d23.i * l0)))));
    out[4] = cfmac(c21, l2, cfma(c10, l0, cfmac(B[7], u2, cfmac(B[4], u1, cfmac(B[1], u0, d45.r * l1)))));
    out[5] = cfma(c21, l1, cfma(c20, l0, cfmac(B[8], u2, cfmac(B[5], u1, cfmac(B[2], u0, d45.i * l2)))));
}

template <typename S2, typename C>
__device__ __forceinline__ void clover_block(cx<C> out[6], const cx<C> in[6], const S2 *p, int Vb) {
    Clov<C> F;
    load_clov(F, p, Vb);
    clover_apply(out, in, F);
}

// The two lanes of a site are lanes l and l + 32 of a wave: thread t of a workgroup (of whole
// waves) takes direction pair_dir(t) of site pair_site(t), so that a wave's loads are two runs of
// 32 sites and coalesce.  (With the two lanes of a site next to each other four neighbouring
// lanes touched two lines, 18 cache accesses a load instead of about 5, and the address unit was
// busy 87% of the FP16 operator's time.  A call of it at 32^3x64 took 582 us and takes 501, M_SAP
// in FP32 at 24^3x48 4035 and 3910, on ragged BF16 blocks 2625 and 2357.)
__device__ __forceinline__ int pair_dir(int t) { return (t >> 5) & 1; }
__device__ __forceinline__ int pair_site(int t) { return (t >> 6) * 32 + (t & 31); }

// the swap leaves lane l with both lanes' a, lane l + 32 with both lanes' b: their sum
__device__ __forceinline__ float pair_sum(float a, float b) {
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}
__device__ __forceinline__ double pair_sum(double a, double b) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// the lane's chiral half of the hops' sum over the pair
template <typename C> __device__ __forceinline__ void pair_reduce(cx<C> own[6], const cx<C> acc[12]) {
#pragma unroll
    for (int c = 0; c < 6; ++c) own[c] = {pair_sum(acc[c].r, acc[6 + c].r), pair_sum(acc[c].i, acc[6 + c].i)};
}
// the row swap leaves a's sum over lanes l and l + 16 in the even rows of 16 lanes, b's in the odd ones
__device__ __forceinline__ float row_sum(float a, float b) {
    const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}
// whether p holds in either lane of the pair
__device__ __forceinline__ bool pair_any(bool p) {
    const auto w = __builtin_amdgcn_permlane32_swap(p, p, false, false);
    return w[0] | w[1];
}

// the six components (spins 2d, 2d + 1) of site (ib, s) owned by lane d
template <typename S2, typename C>
__device__ __forceinline__ void load6(cx<C> v[6], const S2 *f, int ib, int s, int d, int Vb) {
    const S2 *p = f + ((size_t)ib * 12 + 6 * d) * Vb + s;
#pragma unroll
    for (int e = 0; e < 6; ++e) v[e] = ld(p + (size_t)e * Vb);
}
template <typename S2, typename C>
__device__ __forceinline__ void store6(S2 *f, int ib, int s, int d, int Vb, const cx<C> v[6]) {
    S2 *p = f + ((size_t)ib * 12 + 6 * d) * Vb + s;
#pragma unroll
    for (int e = 0; e < 6; ++e) st(p + (size_t)e * Vb, v[e]);
}

// iterate in LDS: records of six float4 per slot, float4 q holding components 2q and 2q + 1, so
// that a neighbour's six reads share one address (eight lanes of a 16-byte read, the LDS's width,
// start at eight different banks whenever their slots are consecutive)
__device__ __forceinline__ void lds_spinor(cx<float> psi[12], const float4 *xs, int slot) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const float4 f = xs[6 * slot + q];
        psi[2 * q] = {f.x, f.y};
        psi[2 * q + 1] = {f.z, f.w};
    }
}
// lane d's half of the record (components 6d .. 6d + 5)
__device__ __forceinline__ void lds_get6(cx<float> v[6], const float4 *xs, int d, int slot) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const float4 f = xs[6 * slot + 3 * d + q];
        v[2 * q] = {f.x, f.y};
        v[2 * q + 1] = {f.z, f.w};
    }
}
__device__ __forceinline__ void lds_put6(float4 *xs, int d, int slot, const cx<float> v[6]) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
        xs[6 * slot + 3 * d + q] = make_float4(v[2 * q].r, v[2 * q].i, v[2 * q + 1].r, v[2 * q + 1].i);
}

// One in-block hop of the lane: the neighbour spinor from LDS slot `slot` and the lane's
// link rows u (U_mu at the site for lane 0, at the backward neighbour for lane 1), already loaded.
template <int MU, bool FIRST = false>
__device__ __forceinline__ void lds_hop(cx<float> acc[12], const float4 *xs, unsigned slot, cx<float> u[9],
                                        float sg) {
    cx<float> psi[12];
    lds_spinor(psi, xs, (int)slot);
    link_rebuild(u);
    link_swap(u, sg < 0.f);
    hop_lane<MU, FIRST>(acc, psi, u, sg);
}

// the six stored rows of link U_mu at block slot sl of block ib
template <typename S2>
__device__ __forceinline__ void link_load(cx<float> u[9], const S2 *U, int ib, int mu, int sl, int Vb) {
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = ld(U + ((size_t)ib * 4 + mu) * 6 * Vb + sl + (size_t)e * Vb);
}

// sum over the lane's in-block hops of site (ib, s), reduced over the pair, and F of the
// lane's chiral half:  out = (F sum_{m in block} H_nm x_m) restricted to spins 2d, 2d + 1;
// with WITH_V also the lane's six components of the field vf at the site.
// gl: block slots of the backward neighbours, where lane 1 finds its links.
// Load order (STAGED): the link rows of all four hops before any product, the clover rows
// after the second hop, v after the third, so that each group arrives while earlier hops
// compute.  A wait on a load also waits on every load issued before it, so the groups are
// issued in the order they are used; issuing everything at once, or each hop's links just
// before the hop (the unstaged order, for kernels short of registers), leaves more of the
// latency exposed.  Both orders compute the same values.
template <bool WITH_V, bool STAGED, typename S2>
__device__ __forceinline__ void block_hop_clover_impl(cx<float> out[6], cx<float> v[6], const S2 *vf, const float4 *xs,
                                                      uint2 nb, uint2 gl, const S2 *U, const S2 *Fk, int ib,
                                                      int s, int d, int Vb, float sg) {
    cx<float> acc[12];
    const bool at_site = d == 0;
    const int sl[4] = {at_site ? s : (int)(gl.x & 0xffffu), at_site ? s : (int)(gl.x >> 16),
                       at_site ? s : (int)(gl.y & 0xffffu), at_site ? s : (int)(gl.y >> 16)};
    cx<float> u[4][9];
    Clov<float> F;
    if constexpr (STAGED) {
#pragma unroll
        for (int m = 0; m < 4; ++m) link_load(u[m], U, ib, m, sl[m], Vb);
    }
    if constexpr (!STAGED) link_load(u[0], U, ib, 0, sl[0], Vb);
    lds_hop<0, true>(acc, xs, nb.x & 0xffffu, u[0], sg);
    if constexpr (!STAGED) link_load(u[1], U, ib, 1, sl[1], Vb);
    lds_hop<1>(acc, xs, nb.x >> 16, u[1], sg);
    if constexpr (STAGED) load_clov(F, Fk + s, Vb);
    if constexpr (!STAGED) link_load(u[2], U, ib, 2, sl[2], Vb);
    lds_hop<2>(acc, xs, nb.y & 0xffffu, u[2], sg);
    if constexpr (STAGED && WITH_V) load6(v, vf, ib, s, d, Vb);
    if constexpr (!STAGED) link_load(u[3], U, ib, 3, sl[3], Vb);
    lds_hop<3>(acc, xs, nb.y >> 16, u[3], sg);
    if constexpr (!STAGED) {
        load_clov(F, Fk + s, Vb);
        if constexpr (WITH_V) load6(v, vf, ib, s, d, Vb);
    }
    cx<float> own[6];
    pair_reduce(own, acc);
    clover_apply(out, own, F);
}
template <typename S2>
__device__ __forceinline__ void block_hop_clover(cx<float> out[6], const float4 *xs, uint2 nb, uint2 gl,
                                                 const S2 *U, const S2 *Fk, int ib, int s, int d, int Vb, float sg) {
    block_hop_clover_impl<false, true>(out, (cx<float> *)nullptr, (const S2 *)nullptr, xs, nb, gl, U, Fk, ib, s, d,
                                       Vb, sg);
}
// the unstaged order
template <typename S2>
__device__ __forceinline__ void block_hop_clover_seq(cx<float> out[6], const float4 *xs, uint2 nb, uint2 gl,
                                                     const S2 *U, const S2 *Fk, int ib, int s, int d, int Vb, float sg) {
    block_hop_clover_impl<false, false>(out, (cx<float> *)nullptr, (const S2 *)nullptr, xs, nb, gl, U, Fk, ib, s, d,
                                        Vb, sg);
}
// the same and v = the lane's six components of vf at (ib, s), in either order
template <bool STAGED, typename S2>
__device__ __forceinline__ void block_hop_clover_v(cx<float> out[6], cx<float> v[6], const S2 *vf, const float4 *xs,
                                                   uint2 nb, uint2 gl, const S2 *U, const S2 *Fk, int ib, int s,
                                                   int d, int Vb, float sg) {
    block_hop_clover_impl<true, STAGED>(out, v, vf, xs, nb, gl, U, Fk, ib, s, d, Vb, sg);
}

// ================================================================ four lanes per site
// The same update by four lanes: rows of 16 lanes (d, m) = (0, 0), (0, 1), (1, 0), (1, 1) of a wave share 16
// sites, lane m taking the hops mu = 2m and 2m + 1 of direction d and then spin 2d + m of the
// result.  Directions x and z (J = 0), and y and t (J = 1), have the same spin structure up to
// the order of the lower spins, which lane m = 1 reads as (2, 3) and lane m = 0 as (3, 2), and the sign
// t = +1 / -1 of one of the two half spinors.  acc: spins 0, 1 and the lower spins in that order.
struct QuadLane {
    int d, m;
    float s, t, st;  // s = +1 / -1: direction, t: row pair, their product
};
__device__ __forceinline__ QuadLane quad_lane(int lane) {
    QuadLane q;
    q.d = lane >> 5;
    q.m = (lane >> 4) & 1;
    q.s = q.d ? -1.f : 1.f;
    q.t = q.m ? -1.f : 1.f;
    q.st = q.s * q.t;
    return q;
}
template <int J>
__device__ __forceinline__ void quad_hop(cx<float> acc[12], const float4 *xs, unsigned slot, cx<float> u[9], const QuadLane &Q) {
    const float s = Q.s, t = Q.t, st = Q.st;
    cx<float> p[6], q0[3], q1[3], h0[3], h1[3], g0[3], g1[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const float4 f = xs[6 * slot + q];
        p[2 * q] = {f.x, f.y};
        p[2 * q + 1] = {f.z, f.w};
    }
    const float2 *lo = reinterpret_cast<const float2 *>(xs) + 12 * slot;
    const int o0 = Q.m ? 6 : 9;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float2 f0 = lo[o0 + a], f1 = lo[15 - o0 + a];
        q0[a] = {f0.x, f0.y};
        q1[a] = {f1.x, f1.y};
    }
    link_rebuild(u);
    link_swap(u, Q.d != 0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<float> p0 = p[a], p1 = p[3 + a];
        if (J == 0) {
            h0[a] = {fmx(-s, q0[a].i, p0.r), fmx(s, p0.i, q0[a].r)};
            h1[a] = {fmx(-st, q1[a].i, p1.r), fmx(s, p1.i, t * q1[a].r)};
        } else {
            h0[a] = {fmx(st, q0[a].r, p0.r), fmx(s, p0.i, t * q0[a].i)};
            h1[a] = {fmx(-s, q1[a].r, p1.r), fmx(s, p1.i, -q1[a].i)};
        }
    }
    su3_mul(g0, u, h0, false);
    su3_mul(g1, u, h1, false);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (J == 0) {
            acc[a] = {g0[a].r, s * g0[a].i};
            acc[3 + a] = {g1[a].r, s * g1[a].i};
            acc[6 + a] = {g0[a].i, -s * g0[a].r};
            acc[9 + a] = {t * g1[a].i, -st * g1[a].r};
        } else {
            acc[a] = {acc[a].r + g0[a].r, fmx(s, g0[a].i, acc[a].i)};
            acc[3 + a] = {acc[3 + a].r + g1[a].r, fmx(s, g1[a].i, acc[3 + a].i)};
            acc[6 + a] = {fmx(st, g0[a].r, acc[6 + a].r), fmx(t, g0[a].i, acc[6 + a].i)};
            acc[9 + a] = {fmx(-s, g1[a].r, acc[9 + a].r), acc[9 + a].i - g1[a].i};
        }
    }
}

// out = spin 2d + m of F sum_{m in block} H_nm x_m at site (ib, s), v = that spin of vf.  nb, gl: the lane's two
// neighbour slots in LDS and backward neighbours' block slots (16 bits each).  Row m of the chiral block is [A B] or [B^+ C], so lane m = 1 reads B transposed
// and takes its conjugate.
template <typename S2>
__device__ __forceinline__ void quad_hop_clover_v(cx<float> out[3], cx<float> v[3], const S2 *vf, const float4 *xs,
                                                  unsigned nb, unsigned gl, const S2 *U, const S2 *F, int ib, int s,
                                                  const QuadLane &Q, int Vb) {
    const S2 *Ub = U + (size_t)ib * 24 * Vb, *Fb = F + (size_t)ib * 36 * Vb, *vb = vf + (size_t)ib * 12 * Vb;
    cx<float> u0[9], u1[9], acc[12];
    const int l0 = 12 * Q.m * Vb + (Q.d ? (int)(gl & 0xffffu) : s), l1 = (12 * Q.m + 6) * Vb + (Q.d ? (int)(gl >> 16) : s);
#pragma unroll
    for (int e = 0; e < 6; ++e) u0[e] = ld(Ub + (l0 + e * Vb));
#pragma unroll
    for (int e = 0; e < 6; ++e) u1[e] = ld(Ub + (l1 + e * Vb));
    quad_hop<0>(acc, xs, nb & 0xffffu, u0, Q);
    const int f0 = 18 * Q.d * Vb + s;
    const cx<float> d23 = ld(Fb + (f0 + Vb)), dd = ld(Fb + (f0 + 2 * Q.m * Vb));
    cx<float> T[3], B[9];
#pragma unroll
    for (int e = 0; e < 3; ++e) T[e] = ld(Fb + (f0 + (3 + 3 * Q.m + e) * Vb));
    const int sa = Q.m ? Vb : 3 * Vb, sb = Q.m ? 3 * Vb : Vb, f9 = f0 + 9 * Vb;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) B[3 * a + b] = ld(Fb + (f9 + a * sa + b * sb));
    const int v0 = (6 * Q.d + 3 * Q.m) * Vb + s;
#pragma unroll
    for (int e = 0; e < 3; ++e) v[e] = ld(vb + (v0 + e * Vb));
    quad_hop<1>(acc, xs, nb >> 16, u1, Q);
    cx<float> half[6], x[3], y[3];  // x: the lane's spin of the sum, y: the other one of its chiral half
    pair_reduce(half, acc);
    const bool swap = Q.d && !Q.m;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const cx<float> ev = sel(swap, half[3 + a], half[a]), od = sel(swap, half[a], half[3 + a]);
        x[a] = {row_sum(ev.r, od.r), row_sum(ev.i, od.i)};
        y[a] = {row_sum(od.r, ev.r), row_sum(od.i, ev.i)};
    }
    const float e0 = Q.m ? d23.i : dd.r, e1 = Q.m ? dd.r : dd.i, e2 = Q.m ? dd.i : d23.r;
    out[0] = cfmac(T[1], x[2], cfmac(T[0], x[1], e0 * x[0]));
    out[1] = cfmac(T[2], x[2], cfma(T[0], x[0], e1 * x[1]));
    out[2] = cfma(T[2], x[1], cfma(T[1], x[0], e2 * x[2]));
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) out[a] = cfma(cx<float>{B[3 * a + b].r, Q.t * B[3 * a + b].i}, y[b], out[a]);
}

// one hop leaving the block (neighbour in another block, from the global iterate x)
template <int MU, typename S2>
__device__ __forceinline__ void gather_hop(cx<float> acc[12], const GeomDev &g, const S2 *x, const S2 *U, int ib,
                                           int s, int d, int bl, float sg) {
    const unsigned w = g.nbr16[MU * g.Vb + s];
    const unsigned hw = d ? (w >> 16) : (w & 0xffffu);
    if (hw & 0x8000u) return;  // inside the block: not part of the gather
    const int sn = (int)(hw & 0x7fffu), ibn = bl & BLK_MASK;
    const float ph = (bl & WRAP_BIT) ? g.bc[MU] : 1.f;
    cx<float> psi[12], u[9];
    load_spinor(psi, x, g, ibn, sn);
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = ph * psi[c];
    const bool at_site = d == 0;
    link_rows(u, U + ((size_t)(at_site ? ib : ibn) * 4 + MU) * 6 * g.Vb + (at_site ? s : sn), g.Vb);
    link_swap(u, d != 0);
    hop_lane<MU, false>(acc, psi, u, sg);
}

// one hop of the lane to a neighbour inside or outside the block, read from the global field x
// (the full operator; the hop of MU = 0 sets acc); outside neighbours across the lattice boundary
// take the fermion phase
template <int MU, typename S2, typename C>
__device__ __forceinline__ void hop_any(cx<C> acc[12], const GeomDev &g, const S2 *x, const S2 *U, int ib, int s, int d,
                                        C sg) {
    const unsigned w = g.nbr16[MU * g.Vb + s];
    const unsigned hw = d ? (w >> 16) : (w & 0xffffu);
    const int sn = (int)(hw & 0x7fffu);
    int ibn = ib;
    C ph = C(1);
    if (!(hw & 0x8000u)) {
        const int bl = g.blk_nbr[(2 * MU + d) * g.NB + ib];
        ibn = bl & BLK_MASK;
        ph = (bl & WRAP_BIT) ? C(g.bc[MU]) : C(1);
    }
    cx<C> psi[12], u[9];
    load_spinor(psi, x, g, ibn, sn);
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = ph * psi[c];
    const bool at_site = d == 0;
    link_rows(u, U + ((size_t)(at_site ? ib : ibn) * 4 + MU) * 6 * g.Vb + (at_site ? s : sn), g.Vb);
    link_swap(u, d != 0);
    hop_lane<MU, MU == 0>(acc, psi, u, sg);
}

}  // namespace sapq
