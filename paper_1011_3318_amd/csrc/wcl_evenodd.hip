// Even-odd reduction of D phi = eta (not in the paper; a standard
// accelerator of the same solve).  With even extents every hop joins sites of
// opposite parity (x+y+z+t mod 2), so with H = the hopping part of D,
//   D = [[A_ee, H_eo], [H_oe, A_oo]],
//   Dhat = A_ee - H_eo A_oo^{-1} H_oe          (Schur complement, even sites)
//   Dhat phi_e = eta_e - H_eo A_oo^{-1} eta_o,
//   phi_o = A_oo^{-1} (eta_o - H_oe phi_e).
// A^{-1} is the per-site inverse of the two 6x6 Hermitian site-term blocks,
// built once per (kappa, c_SW).
//
// Half fields hold the sites of one parity: in the device order the sites
// 2h and 2h + 1 differ only in the lowest bit of x (the column cross-section
// c_x is even when L_x is), so exactly one of them has each parity, and the
// site of parity p is stored at half index h.  A half field is a spinor field
// of V/2 sites in the usual tiled layout.
#include "wcl_device.h"
#include "wcl_kernels.h"

// full index and coordinates of half site h of parity p
WCL_DEV int eo_full(const Geom& g, int h, int p, int x[4]) {
    int i = 2 * h;
    geom_coords(g, i, x);
    if (((x[0] + x[1] + x[2] + x[3]) & 1) != p) {
        ++i;
        x[0] += 1;   // the partner differs in the lowest bit of x only (x even -> x + 1)
    }
    return i;
}

// Spinor and link (rows 0, 1) of hop K at half site h of parity p: neighbour
// from the half field `in` (FULL: from a full-lattice field), link from the
// parity-split copy (SL) or the full-lattice field.  In the split copy the
// links of 64 consecutive half sites are 64 consecutive elements; in the full
// field they alternate with the other parity's, so that half of every line a
// wavefront loads belongs to other hops.
template <int K, int P, bool SL, bool FULL, bool LINK_NT, typename T>
WCL_DEV void eo_fetch(const EoArgs& a, const char* in, int h, int p, const int nbr[8], const int lnk[8], T s[24],
                      T u[18]) {
    if constexpr (FULL) SpinorIO<P>::load(in, a.g.V, nbr[K], s);
    else SpinorIO<P>::load(in, a.Vh, nbr[K] >> 1, s);
    if constexpr (SL) {
        constexpr bool fwd = K % 2 == 0;
        const char* base = (const char*)a.links + (size_t)(fwd ? p : 1 - p) * a.links_stride;
        GaugeIO<P>::template load_raw<LINK_NT>(base, a.Vh, K / 2, fwd ? h : nbr[K] >> 1, u);
    } else {
        GaugeIO<P>::template load_raw<false>(a.gauge, a.g.V, K / 2, lnk[K], u);
    }
}

// acc = H in at half site h (full site i) of parity p: the eight hops,
// reading the neighbours (all of the other parity), two-deep load pipeline.
template <int P, bool SL, bool FULL, bool LINK_NT, typename T>
WCL_DEV void eo_hops(const EoArgs& a, const char* in, int h, int p, int i, const int x[4], T acc[24]) {
    int nbr[8], lnk[8];
    T ph[8];
    hop_sites(a.g, i, x, nbr, lnk, ph);
    const T mk = T(-a.kappa);
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = T(0);
    T s0[24], u0[18], s1[24], u1[18];
    eo_fetch<0, P, SL, FULL, LINK_NT>(a, in, h, p, nbr, lnk, s0, u0);
#define WCL_EHOP(K, SC, UC, SN, UN)                                                                \
    if ((K) < 7) eo_fetch<((K) + 1) & 7, P, SL, FULL, LINK_NT>(a, in, h, p, nbr, lnk, SN, UN);     \
    hop_compute<(K) / 2, ((K) % 2) == 0>(SC, UC, mk * ph[K], acc);
    WCL_EHOP(0, s0, u0, s1, u1)
    WCL_EHOP(1, s1, u1, s0, u0)
    WCL_EHOP(2, s0, u0, s1, u1)
    WCL_EHOP(3, s1, u1, s0, u0)
    WCL_EHOP(4, s0, u0, s1, u1)
    WCL_EHOP(5, s1, u1, s0, u0)
    WCL_EHOP(6, s0, u0, s1, u1)
    WCL_EHOP(7, s1, u1, s0, u0)
#undef WCL_EHOP
}

// y = M z at half site h for the packed Hermitian blocks of one parity:
// site = true: M = A = 1 + csw kappa C (a.clover, even sites), else
// M = A^{-1} (a.ainv, odd sites)
template <int P, bool SITE, bool NT, typename T>
WCL_DEV void eo_site(const EoArgs& a, int h, const T z[24], T y[24]) {
    const T ck = T(a.csw * a.kappa);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        T c[36], w[12];
        CloverBlk<P>::template load<NT>(SITE ? a.clover : a.ainv, a.Vh, h, b, c);
        herm6_apply(c, z + 12 * b, w);
#pragma unroll
        for (int j = 0; j < 12; ++j) y[12 * b + j] = SITE ? fmad(ck, w[j], z[12 * b + j]) : w[j];
    }
}

// One kernel for every step of the reduction; half sites of parity a.parity,
// one per lane, right-hand side from the workgroup index:
//   EO_INV     out_h = A^{-1} H in                 (A_oo^{-1} H_oe psi_e)
//   EO_SCHUR   out_h = A in2_h - H in              (Dhat psi_e, with in = A_oo^{-1} H_oe psi_e)
//              epilogue DS_AXPY: out_h = y_h - that; DS_DOT: partials of <a_h, out_h>, |out_h|^2
//   EO_PREP    out_h = y(i) - H in                 (eta_e - H_eo A_oo^{-1} eta_o; y full)
//   EO_RECON   out(i) = A^{-1} (y(i) - H in) and out(i') = in_h at the even
//              site i' of the pair                 (the whole phi into the full field)
//   EO_SITEINV out_h = A^{-1} y(i)                 (A_oo^{-1} eta_o)
// FULL (EO_INV, EO_SCHUR): psi_e is a full-lattice field (in of EO_INV, in2
// of EO_SCHUR) and the result too, with zeros on the odd sites.
//
// Bound by HBM.  Fields and links come from parity-split copies: with the
// full-lattice ones each line of the clover and of the forward links is half
// unused.  Dhat in FP32 on 24^3x48 (apply_schur; 541 MB at least): 271 us in
// five launches from the full fields, 156 us in two from the split ones (163
// with several configurations in rotation, when nothing stays in a cache).
template <int P, int MODE, int EPI, bool SL, bool FULL, bool NT, bool LINK_NT>
__global__ __launch_bounds__(256, P == WCL_F64 ? 2 : 4) void k_eo(EoArgs a) {
    using T = typename Real<P>::T;
    int tile;
    const int rhs = walk_rhs(a.walk, xcd_remap(blockIdx.x, gridDim.x), gridDim.x / a.nrhs, a.nrhs, &tile);
    if (a.sc && !a.sc[rhs].active) return;   // uniform over the workgroup
    const int h = walk_site(a.walk, tile);
    const bool active = h < a.Vh;
    T acc[24];
    if (active) {
        int x[4];
        const int i = eo_full(a.g, h, a.parity, x);
        const char* in = (const char*)a.in + rhs * a.in_stride;
        const char* y = (const char*)a.y + rhs * a.y_stride;
        char* out = (char*)a.out + rhs * a.out_stride;
        if constexpr (MODE == EO_INV) {
            T w[24];
            eo_hops<P, SL, FULL, LINK_NT>(a, in, h, a.parity, i, x, w);
            eo_site<P, false, NT>(a, h, w, acc);
            SpinorIO<P>::store(out, a.Vh, h, acc);
        } else if constexpr (MODE == EO_SCHUR) {
            T w[24], s[24];
            eo_hops<P, SL, false, LINK_NT>(a, in, h, a.parity, i, x, w);
            const char* in2 = (const char*)a.in2 + rhs * a.in2_stride;
            if constexpr (FULL) SpinorIO<P>::load(in2, a.g.V, i, s);
            else SpinorIO<P>::load(in2, a.Vh, h, s);
            eo_site<P, true, NT>(a, h, s, acc);
#pragma unroll
            for (int k = 0; k < 24; ++k) acc[k] -= w[k];
            if constexpr (EPI == DS_AXPY) {
                SpinorIO<P>::load(y, a.Vh, h, s);
#pragma unroll
                for (int k = 0; k < 24; ++k) acc[k] = s[k] - acc[k];
            }
            if constexpr (FULL) {
                // the pair's sites 2h, 2h + 1 are neighbours in memory
                T z[24];
#pragma unroll
                for (int k = 0; k < 24; ++k) z[k] = T(0);
                SpinorIO<P>::template store<false>(out, a.g.V, i, acc);
                SpinorIO<P>::template store<false>(out, a.g.V, i ^ 1, z);
            } else {
                SpinorIO<P>::store(out, a.Vh, h, acc);
            }
        } else if constexpr (MODE == EO_PREP || MODE == EO_RECON) {
            T w[24], s[24];
            eo_hops<P, SL, false, LINK_NT>(a, in, h, a.parity, i, x, w);
            SpinorIO<P>::load(y, a.g.V, i, s);
#pragma unroll
            for (int k = 0; k < 24; ++k) s[k] -= w[k];
            if constexpr (MODE == EO_PREP) {
                SpinorIO<P>::store(out, a.Vh, h, s);
            } else {
                eo_site<P, false, NT>(a, h, s, acc);
                SpinorIO<P>::load(in, a.Vh, h, s);
                SpinorIO<P>::template store<false>(out, a.g.V, i, acc);
                SpinorIO<P>::template store<false>(out, a.g.V, i ^ 1, s);
            }
        } else {   // EO_SITEINV
            T s[24];
            SpinorIO<P>::load(y, a.g.V, i, s);
            eo_site<P, false, NT>(a, h, s, acc);
            SpinorIO<P>::store(out, a.Vh, h, acc);
        }
    }
    if constexpr (MODE == EO_SCHUR && EPI == DS_DOT) {
        double d[3] = {0.0, 0.0, 0.0};
        if (active) {
            T v[24];
            SpinorIO<P>::load((const char*)a.a + rhs * a.a_stride, a.Vh, h, v);
            site_dot3(v, acc, d);
        }
        block_reduce3(d, a.partial + 3 * ((size_t)tile + (size_t)rhs * (gridDim.x / a.nrhs)));
    }
}

int eo_partials_per_rhs(int Vh) { return (Vh + 255) / 256; }

template <int P, int MODE, int EPI, bool SL, bool FULL>
static int launch_eo_n(const EoArgs& a0, hipStream_t st) {
    EoArgs a = a0;
    a.walk = tile_walk(a.g, 64, 2, a.nrhs, 2 * site_vec_bytes(P), site_field_bytes(P), false);
    const int grid = (a.Vh + 255) / 256 * a.nrhs;
    // Non-temporal field loads only for one rhs streaming more than the 256 MB
    // Infinity Cache holds.  A launch reads each split link once, the next
    // launch (the other parity) reads it again: links that take no more than
    // half of that cache stay in it for a solve, which applies one operator over
    // and over.  Cached / non-temporal links, FP32 24^3x48 (127 MB): solve 14.5 /
    // 15.1 ms, apply_schur with changing fields 162 / 164 us; apply_schur of one
    // field again and again, FP64 24^3x48 (255 MB) 363 / 341 us, FP32 32^4
    // (201 MB) 239 / 223.
    const size_t links = 2 * gauge_bytes(P, a.Vh);
    const bool nt = a.nrhs == 1 && links + clover_bytes(P, a.Vh) + 2 * spinor_rhs_bytes(P, a.Vh) > (256u << 20);
    if (!nt) k_eo<P, MODE, EPI, SL, FULL, false, false><<<grid, 256, 0, st>>>(a);
    else if (SL && links > (128u << 20)) k_eo<P, MODE, EPI, SL, FULL, true, SL><<<grid, 256, 0, st>>>(a);
    else k_eo<P, MODE, EPI, SL, FULL, true, false><<<grid, 256, 0, st>>>(a);
    WCL_HIP(hipGetLastError());
    return WCL_OK;
}

template <int P, int MODE, int EPI, bool FULL>
static int launch_eo_t(const EoArgs& a, hipStream_t st) {
    return a.links ? launch_eo_n<P, MODE, EPI, true, FULL>(a, st) : launch_eo_n<P, MODE, EPI, false, FULL>(a, st);
}

// The forms that are called: the operator between full-lattice fields
// (wcl_apply_schur) at both precisions, a solve's FP32 level with its dot
// products, and its FP64 level, which reads full-lattice links only.
int launch_eo(const EoArgs& a, int prec, int mode, int epi, hipStream_t st) {
    if (a.g.V % 2 || a.Vh * 2 != a.g.V) {
        wcl_set_error("even-odd: half volume %d does not match the lattice", a.Vh);
        return WCL_EINVAL;
    }
    if (a.full && epi == DS_PLAIN) {
        if (prec == WCL_F64 && mode == EO_INV) return launch_eo_t<WCL_F64, EO_INV, DS_PLAIN, true>(a, st);
        if (prec == WCL_F64 && mode == EO_SCHUR) return launch_eo_t<WCL_F64, EO_SCHUR, DS_PLAIN, true>(a, st);
        if (prec == WCL_F32 && mode == EO_INV) return launch_eo_t<WCL_F32, EO_INV, DS_PLAIN, true>(a, st);
        if (prec == WCL_F32 && mode == EO_SCHUR) return launch_eo_t<WCL_F32, EO_SCHUR, DS_PLAIN, true>(a, st);
    } else if (!a.full && prec == WCL_F32) {
        if (mode == EO_INV && epi == DS_PLAIN) return launch_eo_t<WCL_F32, EO_INV, DS_PLAIN, false>(a, st);
        if (mode == EO_SCHUR && epi == DS_DOT) return launch_eo_t<WCL_F32, EO_SCHUR, DS_DOT, false>(a, st);
    } else if (!a.full && prec == WCL_F64 && !a.links) {
        if (epi == DS_PLAIN) switch (mode) {
                case EO_INV: return launch_eo_n<WCL_F64, EO_INV, DS_PLAIN, false, false>(a, st);
                case EO_PREP: return launch_eo_n<WCL_F64, EO_PREP, DS_PLAIN, false, false>(a, st);
                case EO_RECON: return launch_eo_n<WCL_F64, EO_RECON, DS_PLAIN, false, false>(a, st);
                case EO_SITEINV: return launch_eo_n<WCL_F64, EO_SITEINV, DS_PLAIN, false, false>(a, st);
                default: break;
            }
        if (mode == EO_SCHUR && epi == DS_DOT) return launch_eo_n<WCL_F64, EO_SCHUR, DS_DOT, false, false>(a, st);
        if (mode == EO_SCHUR && epi == DS_AXPY) return launch_eo_n<WCL_F64, EO_SCHUR, DS_AXPY, false, false>(a, st);
    }
    wcl_set_error("even-odd: no launch of precision %d, mode %d, epilogue %d", prec, mode, epi);
    return WCL_EINVAL;
}
