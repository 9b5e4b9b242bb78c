// Single-source SAP phase in the even-odd site order, one lane per site (csrc/sapeo.h): one
// workgroup per block of the phase's colour.
#include "sapeo.h"

namespace sapq {

template <int P, int NS>
__global__ void __attribute__((amdgpu_waves_per_eu(2))) __launch_bounds__(EO_THREADS)
k_sap_phase_eo(GeomDev g, EoTables t, int colour, int mode, int n_ssor, float kappa,
               const typename Prec<P>::S2 *rsrc, typename Prec<P>::S2 *r, typename Prec<P>::S2 *x,
               typename Prec<P>::S2 *y, const typename Prec<P>::S2 *__restrict__ U,
               const typename Prec<P>::S2 *__restrict__ F) {
    extern __shared__ float4 xs[];
    eo_phase<P, NS>(g, t, xs, colour * g.NBc + (int)xcd_site_base(1), mode, n_ssor, kappa, rsrc, r, x, y, U, F);
}

EoTables eo_tables(const Ctx *c) {
    EoTables t;
    const int *B = c->geom.block;
    t.Ve = (c->g.Vb + 1) / 2;
    t.T = (t.Ve + 63) / 64 * 64;
    t.nb = c->eo_nb;
    t.face = c->eo_face;
    for (int m = 0; m < 4; ++m) t.nface[m] = c->g.Vb / B[m];
    return t;
}

// The rule: the even-odd site order at omega = 1 in a 16-bit storage precision (whose links and
// clover blocks fit the registers of one lane), blocks of two or more sites in every direction (so
// that the two faces of a direction share no site), more than EO_MIN_SITES sites and at most
// EO_THREADS threads.  Every other phase keeps the kernels that reload a site's links: at omega !=
// 1 the turn planes change, FP32 fields would take twice the registers, and a small block is one
// wave, partly idle, with 31 KB of LDS, of which a CU holds five.  Measured, a SAP cycle in FP16,
// here and with the two-lane or four-lane form: 2x2x2x4 blocks 1079 and 494 us (14112 of a colour),
// 2x2x4x4 594 and 396 (7200), 2x3x4x4 197 and 176 (1536) but 455 and 469 (5000), 3x3x3x4 144 and
// 154 (1152), 2x4x4x4 319 and 364 (3200), 4^4 297 and 403 (2048), 4x4x4x8 519 and 811 (2048),
// 4x4x6x6 1102 and 1024 (2048; BF16 953 and 1432), 4x4x8x8 636 and 919 (1024). With few blocks (up
// to 256 of a colour, four lanes per site) 4x4x4x6 85 and 104, 4^4 79 and 80 (BF16 83 and 75),
// 2x4x4x4 81 and 59.
constexpr int EO_MIN_SITES = 96;
bool eo_supported(const Ctx *c) {
    const int Vb = c->g.Vb, Ve = (Vb + 1) / 2, *B = c->geom.block;
    return c->use_parts && c->sap_np == 1 && eo_order(&c->geom) && !(c->prm.flags & SAPQ_FLAG_EOMR) && c->prm.omega == 1.0 &&
           c->prm.prec_inner != SAPQ_FP32 && B[0] > 1 && B[1] > 1 && B[2] > 1 && B[3] > 1 &&
           Vb > EO_MIN_SITES && Ve <= EO_THREADS;
}

template <int P> static void *eo_kernel(int cls) {
    return cls == 0 ? (void *)k_sap_phase_eo<P, EO_NS[0]> : cls == 1 ? (void *)k_sap_phase_eo<P, EO_NS[1]>
                                                                     : (void *)k_sap_phase_eo<P, EO_NS[2]>;
}
static void *eo_kernel(const Ctx *c) {
    const int cls = eo_class(c->g.Vb);
    return c->prm.prec_inner == SAPQ_FP16 ? eo_kernel<SAPQ_FP16>(cls) : eo_kernel<SAPQ_BF16>(cls);
}

void launch_sap_phase_eo(Ctx *c, int colour, bool gather, bool first, bool last, bool ssor_only, const void *rsrc, void *r,
                         void *x, void *y) {
    EoTables t = eo_tables(c);
    int mode = (gather ? EO_GATHER : 0) | (first ? EO_FIRST : EO_R_ZERO) | (last ? EO_LAST : 0) | (ssor_only ? EO_SSOR_ONLY : 0);
    float kappa = (float)c->prm.kappa;
    void *args[] = {&c->g, &t, &colour, &mode, &c->prm.n_ssor, &kappa, &rsrc, &r, &x, &y, &c->Uin, &c->Fin};
    (void)hipLaunchKernel(eo_kernel(c), dim3(c->g.NBc), dim3(t.T), args, eo_lds_bytes(c->g.Vb, t.T), c->stream);
}

int set_eo_lds_limit(Ctx *c) {
    const int bytes = eo_lds_limit(c->g.Vb);
    if (c->prm.prec_inner == SAPQ_FP32 || bytes <= 65536) return 0;
    if (hipFuncSetAttribute(eo_kernel(c), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess) return 0;
    (void)hipGetLastError();  // clears the runtime's last-error slot
    return -1;
}

}  // namespace sapq
