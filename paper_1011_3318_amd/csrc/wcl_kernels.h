// Kernel launch interfaces shared between the HIP sources.
#pragma once

#include <algorithm>

#include "wcl_internal.h"

enum { DS_PLAIN = 0, DS_AXPY = 1, DS_DOT = 2 };

// BiCGStab scalars of one right-hand side, resident on the device.
struct Scal {
    double rho[2], rho_old[2], alpha[2], omega[2], rv[2];
    double tt, rr, rr0, pp;
    int active, breakdown;
};

// ------------------------------------------------- host transfers ------
// Copies between host memory of the caller (pageable or not) and the device,
// ordered on st (wcl_stage.cpp).  stage_to_device: the source is read until st
// has been waited for (a pinned one is copied in place); stage_to_host: the
// destination is complete on return.
int stage_to_device(int device, void* dev, const void* host, size_t bytes, hipStream_t st);
int stage_to_host(int device, void* host, const void* dev, size_t bytes, hipStream_t st);
void stage_ref();     // one per context: the staging memory is freed with the last
void stage_unref();

// Order in which a launch walks the tiles of a lattice field (or of a half
// field) and the right-hand sides: rhs group, z range, part of the z range, t,
// (x, y) column, tile, rhs of the group.
//
// Storage order runs a column through all of t before the next one.  When the
// cross-section is cut in x or y too (extents such as 24: columns of 8 x 8 x 8),
// the x and y neighbours outside the column are then a whole column away and
// every one of them is fetched again after it left the L2; so the columns of
// one z range are walked side by side.  On 24^3x48 that fetches 1.12 instead of
// 1.37 GB per FP64 D-apply, 450 + 360 instead of 520 + 427 MB per FP32 Dhat.
struct TileWalk {
    int tiles;   // tiles of one column at one t; 0: storage order
    int zt;      // of these, tiles walked together (divides tiles)
    int nxy;     // columns of one z range
    int Lt;
    int group;   // right-hand sides walked together (the last group may have fewer)
    unsigned m_zt, m_nxy, m_Lt, m_nsub, m_group;   // walk_magic of the divisors
};

// Quotients by the walk's divisors, uniform over a wavefront: one scalar
// multiplication instead of a division's 20 to 30 vector instructions (six of
// them were 0.2 us of a 7 us launch).  Exact for n * d < 2^32.
inline unsigned walk_magic(int d) { return d == 1 ? 0u : (unsigned)(((1ull << 32) + d - 1) / d); }
__host__ __device__ inline int walk_div(int n, unsigned magic) {
    return magic == 0u ? n : (int)(((uint64_t)(unsigned)n * magic) >> 32);
}

__host__ __device__ inline int walk_tile(const TileWalk& k, int w) {
    if (k.tiles == 0) return w;
    // q / d and q % d in turn
    const int q0 = walk_div(w, k.m_zt), piece = w - q0 * k.zt;
    const int q1 = walk_div(q0, k.m_nxy), cxy = q0 - q1 * k.nxy;
    const int q2 = walk_div(q1, k.m_Lt), t = q1 - q2 * k.Lt;
    const int z = walk_div(q2, k.m_nsub), sub0 = q2 * k.zt - z * k.tiles;   // (q2 - z * nsub) * zt
    return ((z * k.nxy + cxy) * k.Lt + t) * k.tiles + sub0 + piece;
}

// Launch position lb of n walk positions times nrhs: the right-hand side, and
// the walk position in *pos.
__host__ __device__ inline int walk_rhs(const TileWalk& k, int lb, int n, int nrhs, int* pos) {
    if (nrhs == 1) {
        *pos = lb;
        return 0;
    }
    if (k.group == nrhs) {
        *pos = walk_div(lb, k.m_group);
        return lb - *pos * nrhs;
    }
    const int g = lb / (n * k.group), rem = lb - g * (n * k.group);
    const int left = nrhs - g * k.group, size = left < k.group ? left : k.group;
    *pos = rem / size;
    return g * k.group + rem - *pos * size;
}

// tile: sites per tile of the launch; sites: lattice sites per element of the
// field (1: lattice fields, 2: half fields); vec, fields: bytes per element of
// the vectors of one rhs and of the links and clover.
//
// What the t neighbours find in the 4 MB of an XCD's L2 is what one t slice of
// the walk moves: above 3 MB its z range is halved as long as four planes
// remain (below that the z neighbours at the ranges' ends cost more).
// Right-hand sides go in groups of at most 6, each a walk of its own.
// Measured, D-apply, whole ranges and groups / this rule: 32^4 FP32 131 / 126 us
// (two planes: 150), FP64 285 / 278, 3 rhs FP32 298 / 282, FP64 631 / 590;
// 16^3x32 with 12 rhs FP32 125 / 110 (groups of 4: 114, of 2: 129), FP64 263 / 247.
// Columns are walked side by side only where an XCD's eighth of the launch is
// more than 1.25 t slices of a z range (Lt * nCz / 8): in less, nearly every t
// neighbour belongs to another XCD, while storage order has whole columns in
// one.  Storage order / side by side, 3 rhs: 48x24x8x5 FP32 17.4 / 18.5 us, FP64
// 35.0 / 37.5; 20x28x16x4 12.7 / 13.5 and 24.8 / 25.8; 32x21x4x10 10.8 / 11.2 and
// 21.4 / 22.8; but 28x28x8x12 24.8 / 23.6 and 63.0 / 60.5, 48x6x8x16 12.9 / 12.0
// and 25.6 / 24.5, 24^3x6 25.3 / 24.8 and 66.3 / 62.1.
// by_nrhs = false keeps the walk of the tiles the same for every nrhs, for
// launches whose workgroups sum over several tiles.  The multi-rhs figures above
// are the exchange kernel's, which counts them; in the others counting them makes
// no difference (24^4, 28x20x16x38, 20x20x16x20, 12x20x24x18, FP32, FP64 and FP16,
// 2 to 12 rhs: within 3 % either way).
inline TileWalk tile_walk(const Geom& g, int tile, int sites, int nrhs, size_t vec, size_t fields, bool by_nrhs) {
    const int groups = (nrhs + 5) / 6;
    TileWalk k{};
    k.zt = 1;
    k.nxy = g.nC[0] * g.nC[1];
    k.Lt = g.L[3];
    k.group = (nrhs + groups - 1) / groups;
    k.m_group = walk_magic(k.group);
    const int s = tile * sites;
    if (g.S % s != 0) return k;
    k.tiles = k.zt = g.S / s;
    const size_t per_tile = (size_t)tile * k.nxy * ((by_nrhs ? k.group : 1) * vec + fields);
    while (k.zt % 2 == 0 && k.zt * per_tile > (3u << 20) && k.zt / 2 * s >= 4 * g.c[0] * g.c[1]) k.zt /= 2;
    if (k.nxy == 1 && k.zt == k.tiles) k.tiles = 0;   // that is storage order
    if (k.nxy > 1 && g.L[3] * g.nC[2] <= 10) k.tiles = 0;
    const int nsub = k.tiles / k.zt, widest = std::max(std::max(k.tiles, k.nxy), k.Lt);
    if ((uint64_t)(g.V / s) * widest >> 32) k.tiles = 0;   // past the range of walk_div
    k.m_zt = walk_magic(k.zt);
    k.m_nxy = walk_magic(k.nxy);
    k.m_Lt = walk_magic(k.Lt);
    k.m_nsub = nsub > 0 ? walk_magic(nsub) : 0;
    return k;
}

// Lanes per site that a launch takes for a lattice's setting, which may come
// from an autotuner's file: anything but 2 and 4 is 1.
inline int dslash_lanes(int lps) { return lps == 2 || lps == 4 ? lps : 1; }

// What a workgroup needs to find its tile stands together at the front: one
// round of scalar loads before the first field load instead of two (12^4, one
// rhs, FP32 6.6 -> 6.3 us, FP16 6.0 -> 5.8; 10x24x9x18, FP16, 2 rhs 9.6 -> 9.3).
struct DslashArgs {
    Geom g;
    TileWalk walk;       // set by launch_dslash
    int nrhs;
    int lps;             // lanes per site (see dslash_lanes)
    const Scal* sc;      // optional: right-hand sides with sc[rhs].active == 0 are skipped
    const void* gauge;
    const void* clover;
    const void* in;
    void* out;
    const void* y;       // DS_AXPY source
    const void* a;       // DS_DOT left vector
    size_t in_stride, out_stride, y_stride, a_stride;  // bytes per rhs
    double kappa, csw;
    double* partial;     // DS_DOT: [nrhs][tiles][3]
};

int launch_pack_spinor(const Geom& g, int prec, int nrhs, const double* aos, void* soa, size_t stride,
                       hipStream_t st);
int launch_unpack_spinor(const Geom& g, int prec, int nrhs, const void* soa, size_t stride, double* aos,
                         hipStream_t st);
// *bad = 1 when some of the n links (AoS) is further than bound from SU(3)
int launch_check_links(int64_t n, const double* aos, double bound, int* bad, hipStream_t st);
int launch_pack_gauge(const Geom& g, const double* aos, void* g64, void* g32, void* g16, hipStream_t st);
int launch_clover_build(const Geom& g, const void* g64, void* c64, void* c32, void* c16, hipStream_t st);
int launch_pack_clover(const Geom& g, const double* host_dev, void* c64, void* c32, void* c16, hipStream_t st);
int launch_unpack_clover(const Geom& g, const void* c64, double* host_dev, hipStream_t st);

int dslash_partials_per_rhs(int V, int lps);
int launch_dslash(const DslashArgs& a, int gp, int spi, int spo, int epi, int spy, hipStream_t st);

// --------------------------------------------------------- even-odd ----
// Steps of the even-odd reduction (wcl_evenodd.hip); "half" fields hold the
// V/2 sites of one parity, the site of parity p in pair (2h, 2h+1) at index h.
enum { EO_INV = 0, EO_SCHUR = 1, EO_PREP = 2, EO_RECON = 3, EO_SITEINV = 4 };
struct EoArgs {
    Geom g;
    TileWalk walk;       // set by launch_eo
    int Vh;              // V / 2
    int parity;          // parity of the sites the launch computes
    int full;            // EO_INV, EO_SCHUR: psi_e and Dhat psi_e are full-lattice fields
    const void* gauge;   // full-lattice links, precision of the launch
    const void* links;   // optional: parity-split links (even half field, then odd), used instead
    size_t links_stride; // bytes of one of them
    const void* clover;  // clover of the even sites, half field
    const void* ainv;    // site-term inverse of the odd sites, half field, clover layout
    const void* in;      // half field of the other parity (hop source; EO_INV with full: full field)
    const void* in2;     // half field of `parity` (EO_SCHUR site-term operand; with full: full field)
    const void* y;       // full field (EO_PREP/RECON/SITEINV) or half field (EO_SCHUR axpy)
    const void* a;       // half field: left vector of the DS_DOT partials
    void* out;           // half field, or full field (EO_RECON; EO_SCHUR with full)
    size_t in_stride, in2_stride, y_stride, a_stride, out_stride;   // bytes per rhs
    double kappa, csw;
    int nrhs;
    double* partial;     // DS_DOT: [nrhs][tiles][3]
    const Scal* sc;      // optional: right-hand sides with sc[rhs].active == 0 are skipped
};
int eo_partials_per_rhs(int Vh);
int launch_eo(const EoArgs& a, int prec, int mode, int epi, hipStream_t st);

// ------------------------------------------------------------- solvers --
enum { FIN_RHO = 2, FIN_PP = 3, FIN_RR = 4, FIN_RR0 = 5 };

int blas_partials(int prec, int64_t V);
int blas_p_update(int prec, int64_t V, int nrhs, const Scal* sc, const void* r, void* p, const void* v,
                  hipStream_t st);
// s = r - alpha v, alpha formed from the partials pv of <rhat, v> (Gv per rhs)
int blas_s_update_fin(int prec, int64_t V, int nrhs, Scal* sc, const double* pv, int Gv, const void* r,
                      const void* v, void* s, hipStream_t st);
// x += alpha p^ + omega s^, r = s - omega t, partials of <rhat, r>, |r|^2 into
// `partial` (which must not alias pw); omega formed from the partials pw of
// <s, t>, |t|^2 (Gw per rhs)
int blas_xr_update_fin(int prec, int64_t V, int nrhs, Scal* sc, const double* pw, int Gw, void* x, const void* ph,
                       const void* sh, const void* s, const void* t, void* r, const void* rh, double* partial,
                       hipStream_t st);
int blas_dot(int prec, int64_t V, int nrhs, const Scal* sc, const void* a, const void* b, double* partial,
             hipStream_t st);
// x = p = v = 0, r = rhat = b, partials of <b, b> for the active rhs
int blas_init(int prec, int64_t V, int nrhs, const Scal* sc, const void* b, void* x, void* r, void* rh, void* p,
              void* v, double* partial, hipStream_t st);
int blas_to_f32_scaled(int64_t V, int nrhs, const Scal* sc, const void* a64, void* y32, hipStream_t st);
int blas_to_f64_scaled(int64_t V, int nrhs, const Scal* sc, const void* a32, void* y64, hipStream_t st);
// mirror (optional): device-visible pinned host array that also receives the
// updated scalars of the active rhs
int blas_finalize(const double* partial, int G, int nrhs, Scal* sc, int kind, hipStream_t st,
                  Scal* mirror = nullptr);

// ------------------------------------------------------ domain solves ---
struct BlockArgs {
    Geom g;
    Blocks B;
    const void* gauge;   // storage precision of the domain solver
    const void* clover;
    const void* src;     // projection source
    size_t src_stride;
    void* rho;           // workspace float4 [rhs][6][NE]
    void* q;
    void* x;
    size_t ws_stride;    // float4 elements per rhs
    int NE;              // nblocks * ev
    int wpb;             // workgroups per domain (split path)
    void* out;           // K_RAS output (FP32), owned sites
    size_t out_stride;
    void* vj;            // optional copy of this sweep's correction (storage precision)
    size_t vj_stride;
    int accumulate;      // out += x instead of out = x
    // fused residual update (on-chip path, sweeps after the first), with
    // vprev = v_{j-1}:
    //   res_boundary == 0: src = r_{j-1}; the kernel forms r_j = src - D vprev
    //     and writes r_j to rout at the owned sites;
    //   res_boundary == 1 (no overlap): src = the previous sweep's final MR
    //     residual rho_N = r_{j-1} - D_Omega v_{j-1}; the kernel adds only the
    //     hops that leave the domain, and writes its own final rho_N to rout.
    const void* vprev;   // storage precision
    size_t vprev_stride;
    void* rout;          // storage precision
    size_t rout_stride;
    int res_boundary;
    double kappa, csw;
    int nrhs;
    double* partial;     // [rhs][nblocks][wpb][3]
    const Scal* sc;      // optional: right-hand sides with sc[rhs].active == 0 are skipped
    // split-path variants (the other readings of Sec. 1-2):
    const void* dhat;    // k_blk_dslash: when set, the dot products are <dhat, q> and |q|^2
                         // instead of <q, rho> and |q|^2 (truncated BiCGStab's <rhat, v>)
    int colour;          // -1: every domain; 0 or 1: only the domains of that colour
                         // (multiplicative Schwarz); the others write zeros at their owned sites
    int whole;           // 1: the last step keeps the whole extended solution in x and the additive
                         // gather sums it (overlaps add up); 0: restriction to the owned sites
    const void* ainv;    // block Jacobi: site-term inverse A^{-1}, clover layout, storage precision
    void* bp;            // truncated BiCGStab workspaces (float4 [rhs][6][NE]): p, s, t, rhat
    void* bs;
    void* bt;
    void* brh;
    double* bpart[3];    // truncated BiCGStab partial sums: <rhat, r>, <rhat, v>, (<t, s>, |t|^2)
    double* dsc;         // truncated BiCGStab per-(rhs, domain) scalars [rhs][nblocks][8]:
                         // rho, alpha, omega, rho_old (complex)
    int dot2;            // on-chip MR steps with binary16 operands and FP32 sums (FP16 storage only)
    // on-chip path, output of the sweeps: skip_out = 1 writes no output (the
    // sweep's correction goes to vj only); vsum_n > 0 writes
    // out = vsum[0] + ... + vsum[vsum_n - 1] + x, vsum[j] at vsum + j * vsum_step
    // (storage precision, per-rhs stride vj_stride)
    int skip_out;
    const void* vsum;
    int vsum_n;
    size_t vsum_step;
};

int launch_blk_project(const BlockArgs& a, int src_prec, int bicgstab, hipStream_t st);
// src: -1, or the precision of the projection source that the first MR step
// reads in place of rho in the workspace
int launch_blk_dslash(const BlockArgs& a, int gp, int src, hipStream_t st);
int launch_blk_update(const BlockArgs& a, int vj_prec, int src, int last, hipStream_t st);
// block Jacobi step: x = x + A^{-1} (b - q) (first: x = A^{-1} b), b = rho
int launch_blk_jacobi(const BlockArgs& a, int gp, int vj_prec, int first, int last, hipStream_t st);
// truncated BiCGStab: p update, s update, x/r update (see wcl_block.hip)
int launch_bcg_p(const BlockArgs& a, int it, hipStream_t st);
int launch_bcg_s(const BlockArgs& a, hipStream_t st);
int launch_bcg_xr(const BlockArgs& a, int vj_prec, int last, hipStream_t st);
// additive Schwarz: v(x) = sum of the extended solutions of every domain whose
// Omega' holds x, out (+)= v, vj = v
int launch_blk_gather(const BlockArgs& a, int vj_prec, hipStream_t st);
// A^{-1} = (1 + csw kappa C)^{-1} per site, stored like the clover field in
// FP64, FP32 and FP16; *bad (device int) is set when some A(x) is singular
int launch_site_inverse(const Geom& g, const void* c64, double kappa, double csw, void* a64, void* a32, void* a16,
                        int* bad, hipStream_t st);
// Fields of the even-odd reduction at precision prec (FP64 or FP32), as half
// fields: ainv = A^{-1} of the odd sites, clov = C of the even sites, links
// (optional) = the links of the even sites, then of the odd ones, links_stride
// bytes apart.  *bad is set when A is singular at some site of either parity.
int launch_eo_fields(const Geom& g, int prec, const void* c64, const void* clover, const void* gauge, double kappa,
                     double csw, void* ainv, void* clov, void* links, size_t links_stride, int* bad, hipStream_t st);
int launch_blk_unpack(const BlockArgs& a, const float* ws, double* out, hipStream_t st);
// ------------------------------------------------------------- solvers --
struct Workspace;
Workspace* wcl_workspace_new(wcl_ctx* ctx);
void wcl_workspace_delete(Workspace* w);
void workspace_begin(Workspace* w);   // a new call: buffers it does not ask for may be given up
size_t workspace_bytes(const Workspace* w);
void workspace_get(Workspace* w, const char* name, size_t bytes, void** out, int* rc);
// Nested RAS-BiCGStab on an explicit workspace and stream (Sec. 3).
// resid_rhs (optional, nrhs values): |eta_i - D phi_i| / |eta_i| per rhs
// (0 for a zero rhs, -1 where the solve ended on a hard error).
int nested_solve(wcl_lattice* lat, Workspace* ws, const wcl_solver_params* prm, double kappa, double csw,
                 const void* eta, void* phi, int nrhs, wcl_solve_stats* stats, hipStream_t st,
                 double* resid_rhs = nullptr);
// Device bytes a nested solve needs on a fresh workspace (estimate, upper bound).
size_t nested_workspace_bytes(const wcl_lattice* lat, const wcl_solver_params* prm, int nrhs);
int fused_threads(int ev);   // workgroup size of the fused domain solver, 0 if it does not fit
int launch_blk_fused(const BlockArgs& a, int gp, int src_prec, hipStream_t st);
int blas_restart(int prec, int64_t V, int nrhs, const Scal* sc, const void* src, void* r, void* rh, void* p, void* v,
                 hipStream_t st);
