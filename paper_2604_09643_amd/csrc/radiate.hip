// radiate.hip -- gfx950 kernels and C ABI of the differentiable acoustic radiation model.
//
// Model (main text Eq. (1); kernel from Appendix A, Eq. (A13) with K_G):
//   s[e,k] = sum_v p0[v] * phi(d - c t_k) / (2 d),  phi(u) = u exp(-u^2/(2 sigma^2)),
//   t_k = k/fs, terms kept iff |d - c t_k| <= trunc*sigma, e = f*M + m,
//   x_e = R_f e_m + t_f (rigid array of Stage 4).
//
// GPU formulation (FP32 VALU; the model is a windowed sum, and only the expansion of the
// forward's moments into samples is a contraction, done on the matrix cores).
//   * Voxels are processed in regions: boxes of voxels around a common centre.
//     One workgroup owns one region.  Its four wavefronts take 64-element
//     chunks in turn, one element per lane, and walk the region's voxels in
//     lock-step.  Voxel offsets and p0 values are wave-uniform (loads of a
//     wave-uniform address).
//   * Distances.  Each (region, element) pair gets a reference distance d_c
//     to the region centre, computed in double-float (pairs of FP32 values).
//     Each (voxel, element) pair then forms d_v - d_c from
//     N = |D+o|^2 - |D|^2 = 2 D.o + o.o and one Newton step on
//     y = sqrt(dh^2 + N).  So u = d - c t keeps ~1e-10 m absolute accuracy
//     although d ~ 1e-2 m.
//   * Samples.  Around the centre sample k0 = round(d/delta) with offset
//     u0 = d - k0 delta, the Gaussian of sample k0 +- j factorises as
//     e0 * H^{+-j} * Gamma_j, with e0 = exp(-u0^2/2s^2), H = exp(u0 delta/s^2)
//     and Gamma_j = exp(-j^2 delta^2/2s^2) a per-call table.  So each sample
//     costs one multiply of a running power of H plus one or two FMAs, with
//     no transcendental; two or three exponentials are evaluated per pair.
//   * Forward in moment form (Gaussian, exponential, power law): every pair adds NM polynomial
//     moments of its offset from its centre sample into fixed-point sums in LDS, which a region's
//     workgroup expands into signal rows and adds to the signals with global atomics (k_forward_mom).
//   * Forward otherwise (uniform sphere, short windows, coarse sampling or spacing): every lane owns a private
//     row of signal samples in LDS (layout [sample][lane], bank = lane, no conflicts) and updates it by
//     read-modify-write; two z-neighbouring voxels share one pass over the rows (the Gaussian's rows
//     about each voxel's centre sample are taken whole).  At the end of each region the rows are added
//     into the signals with global atomics (transposed, so each atomic instruction covers consecutive
//     samples of one element).
//   * Sums of the regions' rows: FP32 up to 4096 row-form regions, FP64 sums beyond.
//   * Adjoints in moment form: a table of dL/ds's local expansions per sample, built once per
//     call, two LDS reads and a Horner sum per pair, with its derivative for the element gradients
//     (am_regions).
//   * Adjoints otherwise: each lane stages its element's dL/ds window in the same
//     private-row layout and gathers.  dL/dp0 of a voxel is summed across the
//     64 lanes with DPP and across the four wavefronts in LDS.  It is written
//     once, with no atomics.  The element gradient is accumulated per lane in
//     FP64 over the region's voxels.  It goes to a per-region partial buffer,
//     then to a deterministic FP64 reduction over regions and the per-frame
//     chain rule to (dL/dR, dL/dt).
//   * The other source profiles of Appendix A (exponential, power law, uniform
//     sphere) swap the pair functions; the exponential factorises per leg.
//   * Around the model: the Stage 2/4 negative-correlation loss (FP64 row
//     statistics), the TGV regulariser (one marching pass), the axis-angle and
//     Euler-angle pose maps, and the batched serving step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>

#include "moment_series.h"
#include "radiate.h"

// Scratch of radiate_forward_static, for callers that cannot allocate: one copy per device
// (each device that loads the library holds it until the process ends), shared by every call
// on that device.  Host code never passes this name to a kernel: it resolves the device's
// address once (static_scratch_of, at ra_create) and uses that.
constexpr size_t STATIC_SCRATCH_BYTES = RA_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[STATIC_SCRATCH_BYTES];

namespace {

constexpr int WAVE = 64;
constexpr int WAVES = 4;              // wavefronts per region workgroup
constexpr int BLOCK = WAVE * WAVES;
constexpr int GEN_STEP = 8;           // spacing of the generic window bounds (8, 16, ..., 40)
#ifdef RA_FAST_BUILD
constexpr int EXP_STEP = 8;           // spacing of the exponential profile's window bounds
#else
constexpr int EXP_STEP = 4;
#endif
constexpr int RS_MAX = 47;            // largest |row - kc| of the row-referenced dL/dp0 adjoint
constexpr int PAIR_D = 3;             // largest centre-sample spread of two voxels the paired forward takes
constexpr int NC_THREADS = 256;       // workgroup of the negative-correlation row kernel
constexpr int NXCD = 8;               // MI355X compute dies; workgroups are dealt round-robin
constexpr int NCU = 256;              // its compute units
constexpr int RESID_BLOCKS = 1024;    // partial sums of the loss
constexpr int FWD_F32_MAX_REGIONS = 4096;   // forward regions up to which partial rows are summed in FP32
constexpr size_t LDS_FWD_BUDGET = 80 * 1024;   // forward: two region workgroups per CU
constexpr size_t LDS_ADJ_BUDGET = 80 * 1024;   // adjoint with element gradients: two per CU
constexpr size_t LDS_ADJ0_BUDGET = 53 * 1024;  // adjoint for dL/dp0 only: three per CU
constexpr int BATCH_BINS_MAX = 40;    // centre samples of a region the batched step's moment form takes
constexpr int FM_WAVES = 8;           // wavefronts of the moment-form forward's region workgroup, two per CU
constexpr int FM_WAVES_BIG = 16;      // and where its LDS leaves room for one per CU
constexpr int FM_REFS = 2;            // element chunks whose references it computes at a time
constexpr int FM_FIELDS = 13;         // floats of a reference
constexpr int FM_RZ = 8;              // voxels of a column it unrolls
constexpr int FM_SIDE = 16;           // its largest region side
constexpr float FM_FAINT = 0x1p-14f;  // largest |p0| of a line over the bound of its region's bins below which it is faint
constexpr size_t AM_TABLE_MAX = (size_t)16 << 30;   // bytes of the moment table (wide Gaussians: any)
constexpr int AM_WAVES = 16;          // wavefronts of the moment-form adjoints' region workgroup, one per CU
constexpr int AM_REFS = 3;            // references held: this chunk's, the next one's and the one after
constexpr size_t LDS_FM_BUDGET = 80 * 1024;    // two of its workgroups per CU

// ------------------------------------------------------------------------------------------
// double-float arithmetic (value = h + l, |l| <= ulp(h)/2)
// ------------------------------------------------------------------------------------------
// Double-float (hi + lo) arithmetic.  Each helper turns off FMA contraction: fusing a
// product of one step into the sum of the next (e.g. the rounded product of two_prod into the
// quick_two_sum that follows) silently breaks the error-free transformations, leaving FP32
// precision (about one ulp of a 60 mm distance, 4e-9 m).
struct DF {
    float h, l;
};
__device__ __forceinline__ DF two_sum(float a, float b) {
#pragma clang fp contract(off)
    float s = a + b;
    float v = s - a;
    float e = (a - (s - v)) + (b - v);
    return {s, e};
}
__device__ __forceinline__ DF quick_two_sum(float a, float b) {
#pragma clang fp contract(off)
    float s = a + b;
    float e = b - (s - a);
    return {s, e};
}
__device__ __forceinline__ DF two_prod(float a, float b) {
#pragma clang fp contract(off)
    float p = a * b;
    float e = fmaf(a, b, -p);
    return {p, e};
}
__device__ __forceinline__ DF df_add(DF a, DF b) {
#pragma clang fp contract(off)
    DF s = two_sum(a.h, b.h);
    return quick_two_sum(s.h, s.l + (a.l + b.l));
}
__device__ __forceinline__ DF df_neg(DF a) { return {-a.h, -a.l}; }
__device__ __forceinline__ DF df_mul(DF a, DF b) {
#pragma clang fp contract(off)
    DF p = two_prod(a.h, b.h);
    return quick_two_sum(p.h, p.l + (a.h * b.l + a.l * b.h));
}
__device__ __forceinline__ DF df_sqrt(DF a) {
#pragma clang fp contract(off)
    float s = sqrtf(a.h);
    DF p = two_prod(s, s);
    float r = ((a.h - p.h) - p.l) + a.l;
    return quick_two_sum(s, s == 0.0f ? 0.0f : r / (2.0f * s));   // an element may sit at the centre of a region that ends short
}
__device__ __forceinline__ DF df_from_double(double x) {
#pragma clang fp contract(off)
    float h = (float)x;
    return {h, (float)(x - (double)h)};
}

// ------------------------------------------------------------------------------------------
// per-call constants
// ------------------------------------------------------------------------------------------
struct Geo {
    int nx, ny, nz;
    long long vsx, vsy;    // element strides of p0 along x and y (z is contiguous)
    long long gsx, gsy;    // element strides of dL/dp0 along x and y
    int rx, ry, rz;        // region size in voxels
    int nrx, nry, nrz;     // regions per axis
    int nreg;
    int K, E, M, F;
    int jin;               // steps |j| <= jin always lie inside the window
    int jclamp;            // |k0 - kc| bound within a region
    float jclampf;
    int kmargin;           // row index of the region's reference sample kc
    int L;                 // LDS row length in samples
    int nvpad;             // voxels per region, padded to a multiple of 4
    int zero;              // always 0 (keeps table loads per-lane, see forward_region)
    float org_h[3], org_l[3];
    float sp_h, sp_l;
    float dlt_h, dlt_l, inv_dlt;   // sample length delta = c/fs
    float tsig;                    // trunc*sigma
    float kappa;                   // e0 = exp2(kappa * u0^2)
    float alpha;                   // H = exp2(alpha * u0)
    float inv_s2;                  // 1/sigma^2
    float gmin;                    // geometry check: minimum element-to-grid distance
    float edge;                    // JT delta - trunc sigma: sample k0 +- JT is in the window iff +-u0 >= edge
    float gam[JMAX + 1];           // Gamma_j
    float jdg[JMAX + 1];           // j delta Gamma_j
    float jjdg[JMAX + 1];          // (j delta)^2 Gamma_j
    float gamr[RS_MAX + 1];        // Gamma_m = exp(-m^2 delta^2 / 2 sigma^2) by LDS row offset m from kc
    int ktype;                     // source profile, RA_KERNEL_*
    int jwin;                      // other profiles: window half-width in steps (JT = 0 kernels)
    float kexp;                    // exponential: K(x) = exp2(kexp x)
    float kinv_w, kinv_w2;         // 1/w, 1/w^2
    float knu, k2nu;               // power law: K(x) = exp2(knu log2(1 + x^2/w^2)), knu = -nu; 2 nu
    // moment forms: lengths in units of delta / 2
    int jt;                        // window half-width in samples
    int nbin;                      // centre samples of a region, 2 jclamp + 1
    float unit_h, unit_l;          // 2 / delta
    float hs_u, hs_l;              // grid spacing in units (double-float)
    // terms of the other profiles that no polynomial in t holds: of the window's outermost samples kc +- jt, in the
    // window for some offsets only, and of the exponential's kink at kc (see edge_phi)
    int xkind;                     // 0 none, 1 an outermost sample, 2 that and the centre
    float thr, ev[4], es;
    unsigned flip;                 // 0: the outermost sample on t's side; sign bit: the one on the other side
    float kx;                      // centre: t/2 exp2(kx |t|)
};

// Workgroup -> region, so that each compute die (XCD) gets a contiguous run of
// regions: neighbouring regions read overlapping signal windows, which then
// hit in that die's L2.
__device__ __forceinline__ int region_of_block(int b, int nreg) {
    int q = nreg / NXCD, rm = nreg % NXCD;
    int x = b % NXCD, i = b / NXCD;
    return x * q + min(x, rm) + i;
}

struct Region {
    int i0, j0, k0;        // first voxel
    int ni, nj, nk;        // voxels inside the grid
    DF cx, cy, cz;         // centre
};

__device__ __forceinline__ Region region_info(const Geo& g, int reg) {
    Region R;
    int a = reg / (g.nry * g.nrz), b = (reg / g.nrz) % g.nry, c = reg % g.nrz;
    R.i0 = a * g.rx; R.j0 = b * g.ry; R.k0 = c * g.rz;
    R.ni = min(g.rx, g.nx - R.i0); R.nj = min(g.ry, g.ny - R.j0); R.nk = min(g.rz, g.nz - R.k0);
    DF sp{g.sp_h, g.sp_l};
    R.cx = df_add(DF{g.org_h[0], g.org_l[0]}, df_mul(DF{(float)R.i0 + 0.5f * (float)(g.rx - 1), 0.f}, sp));
    R.cy = df_add(DF{g.org_h[1], g.org_l[1]}, df_mul(DF{(float)R.j0 + 0.5f * (float)(g.ry - 1), 0.f}, sp));
    R.cz = df_add(DF{g.org_h[2], g.org_l[2]}, df_mul(DF{(float)R.k0 + 0.5f * (float)(g.rz - 1), 0.f}, sp));
    return R;
}

// Per (region, element) reference: D = centre - x_e, d_c = |D| = dh + dl,
// kc = round(dh/delta), uc0 = d_c - kc*delta.
struct Ref {
    float Dx, Dy, Dz;
    float dh, dh2, uc0;
    float hdh;             // dh / 2
    int kbase;             // sample index of LDS row 0
};

__device__ __forceinline__ Ref make_ref(const Geo& g, const float* __restrict__ xe, int e, const Region& R) {
#pragma clang fp contract(off)
    const float* x = xe + 6 * e;
    DF Dx = df_add(R.cx, df_neg(DF{x[0], x[3]}));
    DF Dy = df_add(R.cy, df_neg(DF{x[1], x[4]}));
    DF Dz = df_add(R.cz, df_neg(DF{x[2], x[5]}));
    DF d2 = df_add(df_add(df_mul(Dx, Dx), df_mul(Dy, Dy)), df_mul(Dz, Dz));
    DF d = df_sqrt(d2);
    float kc = rintf(d.h * g.inv_dlt);
    DF kd = df_add(two_prod(kc, g.dlt_h), DF{kc * g.dlt_l, 0.f});
    DF u = df_add(d, df_neg(kd));
    Ref r;
    r.Dx = Dx.h; r.Dy = Dy.h; r.Dz = Dz.h;
    r.dh = d.h;
    r.dh2 = d.h * d.h;
    r.uc0 = u.h;
    r.hdh = 0.5f * d.h;
    r.kbase = (int)kc - g.kmargin;
    return r;
}

// Per (voxel, element) pair: centre-sample offset j0 (relative to kc), residual u0,
// 1/(2d), and the Gaussian factors e0, H, 1/H.
struct Pair {
    int j0;
    float u0, hr, e0, H, Hi;
};

// Copy a wave-uniform value into a VGPR.
__device__ __forceinline__ float to_vgpr(float x) {
    float v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
    return v;
}

// Per-call constants of the pair loops.  With VG they are copied into vector registers
// once (VALU instructions then read no scalar register), otherwise they stay in scalar
// registers; which is faster depends on the kernel's register pressure and schedule, and
// was measured per kernel.
template <int JT, bool M2>
struct VConst {
    float gam[JT + 1], jdg[JT + 1], jjdg[M2 ? JT + 1 : 1];
    float inv_dlt, dlt_h, dlt_l, kappa, alpha, jclampf, njclampf, edge, nedge, tsig, inv_s2;
};

template <bool VG>
__device__ __forceinline__ float cst_copy(float x) {
    if constexpr (VG) return to_vgpr(x);
    return x;
}

template <bool VG, int JT, bool M2>
__device__ __forceinline__ void load_vconst(VConst<JT, M2>& v, const Geo& g) {
#pragma unroll
    for (int j = 0; j <= JT; ++j) {
        v.gam[j] = cst_copy<VG>(g.gam[j]);
        v.jdg[j] = cst_copy<VG>(g.jdg[j]);
        if (M2) v.jjdg[j] = cst_copy<VG>(g.jjdg[j]);
    }
    v.inv_dlt = cst_copy<VG>(g.inv_dlt);
    v.dlt_h = cst_copy<VG>(g.dlt_h);
    v.dlt_l = cst_copy<VG>(g.dlt_l);
    v.kappa = cst_copy<VG>(g.kappa);
    v.alpha = cst_copy<VG>(g.alpha);
    v.jclampf = cst_copy<VG>(g.jclampf);
    v.njclampf = cst_copy<VG>(-g.jclampf);
    v.edge = cst_copy<VG>(g.edge);
    v.nedge = cst_copy<VG>(-g.edge);
    v.tsig = cst_copy<VG>(g.tsig);
    v.inv_s2 = cst_copy<VG>(g.inv_s2);
}

// Distance part of a pair: uc = d_v - kc delta (compensated), 1/d_v and 1/(2 d_v).  The voxel
// table holds o and |o|^2 / 2, so Nh = D.o + |o|^2/2 = (|D+o|^2 - |D|^2) / 2 is three FMAs; with
// y = sqrt(dh^2 + 2 Nh) ~ d_v, a = y - dh (exact), one Newton step gives d_v - dh = a + (N - a (y
// + dh)) / (2 y), carried here in halves.
struct Dist {
    float uc, rs, hr;
};

__device__ __forceinline__ Dist pair_dist(const Ref& r, float4 o) {
#pragma clang fp contract(off)    // a = y - dh must be exact (Sterbenz) for the Newton step
    const float Nh = fmaf(r.Dx, o.x, fmaf(r.Dy, o.y, fmaf(r.Dz, o.z, o.w)));
    const float S = fmaf(2.0f, Nh, r.dh2);
    Dist q;
    q.rs = __builtin_amdgcn_rsqf(S);          // 1/d_v
    const float y = S * q.rs;                 // ~ d_v
    const float a = y - r.dh;                 // exact (Sterbenz)
    const float bh = fmaf(0.5f, y, r.hdh);    // (y + dh) / 2
    const float th = fmaf(-a, bh, Nh);        // (N - a (y + dh)) / 2
    q.hr = 0.5f * q.rs;                       // 1/(2 d_v)
    q.uc = r.uc0 + fmaf(th, q.rs, a);         // d_v - kc delta
    return q;
}

// Nearest sample offset from kc, as a float.  |j| <= jclamp holds by the triangle
// inequality; the clamp keeps LDS indices in range whatever the inputs (NaN converts to 0).
template <int NJ, bool M2>
__device__ __forceinline__ float centre_step(const VConst<NJ, M2>& c, float uc) {
    return __builtin_amdgcn_fmed3f(rintf(uc * c.inv_dlt), c.njclampf, c.jclampf);
}

// uc - j delta with delta in double-float.
template <int NJ, bool M2>
__device__ __forceinline__ float residual(const VConst<NJ, M2>& c, float uc, float jf) {
    return fmaf(-jf, c.dlt_l, fmaf(-jf, c.dlt_h, uc));
}

template <int JT, bool M2>
__device__ __forceinline__ Pair make_pair(const VConst<JT, M2>& c, const Ref& r, float4 o) {
    const Dist q = pair_dist(r, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    Pair p;
    p.j0 = (int)jf;
    p.u0 = u0;
    p.hr = q.hr;
    p.e0 = __builtin_amdgcn_exp2f(c.kappa * (u0 * u0));
    float au = c.alpha * u0;
    p.H = __builtin_amdgcn_exp2f(au);
    p.Hi = __builtin_amdgcn_exp2f(-au);
    return p;
}

// 64-lane sum; the total lands in lane 63 (other lanes hold partial sums).  Every step writes all
// rows with zeros for lanes without a source, so each folds into one v_add_f32_dpp: after the four
// row shifts lane 15 of a row holds the row's total, and lane 63 then adds lane 47 (row 2) and
// lane 31 (rows 0 and 1).
__device__ __forceinline__ float wave_sum_to_63(float v) {
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x111, 0xf, 0xf, true);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x112, 0xf, 0xf, true);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x114, 0xf, 0xf, true);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x118, 0xf, 0xf, true);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x142, 0xf, 0xf, true);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0.0f, v, 0x143, 0xf, 0xf, true);  // row_bcast:31
    return v;
}

// Sums of four values over the 64 lanes, left as one partial per row of 16 lanes: on return lanes
// 12..15 of row r hold row r's sums of v0, v2, v1, v3 (in that order).  Two exchange steps within
// quads leave each lane with one quad sum (lane & 3 = 0, 1, 2, 3: v0, v2, v1, v3), then two row
// shifts add the four quads of a row: 11 VALU for four values where four full sums take 24.
__device__ __forceinline__ float wave_sum4_rows(float v0, float v1, float v2, float v3, int lane) {
    const bool odd = lane & 1, hi2 = lane & 2;
    // quad_perm [1,0,3,2]: even lanes add their odd neighbour's v0 / v1, odd lanes the even one's v2 / v3
    const float s02 = (odd ? v2 : v0) + __builtin_amdgcn_update_dpp(0.0f, odd ? v0 : v2, 0xB1, 0xf, 0xf, true);
    const float s13 = (odd ? v3 : v1) + __builtin_amdgcn_update_dpp(0.0f, odd ? v1 : v3, 0xB1, 0xf, 0xf, true);
    // quad_perm [2,3,0,1]: lanes 0, 1 of a quad keep s02 and add lanes 2, 3's; lanes 2, 3 keep s13
    float s = (hi2 ? s13 : s02) + __builtin_amdgcn_update_dpp(0.0f, hi2 ? s02 : s13, 0x4E, 0xf, 0xf, true);
    s += __builtin_amdgcn_update_dpp(0.0f, s, 0x114, 0xf, 0xf, true);   // row_shr:4
    s += __builtin_amdgcn_update_dpp(0.0f, s, 0x118, 0xf, 0xf, true);   // row_shr:8
    return s;
}

// ------------------------------------------------------------------------------------------
// element positions (prologue) and geometry check
// ------------------------------------------------------------------------------------------
__global__ void k_elements(Geo g, const double* __restrict__ elem, const double* __restrict__ poses,
                           float* __restrict__ xe, int* __restrict__ status, float3 box_lo, float3 box_hi) {
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= g.E) return;
    int f = e / g.M, m = e % g.M;
    const double* P = poses + 12 * f;
    const double* em = elem + 3 * m;
    DF ev[3] = {df_from_double(em[0]), df_from_double(em[1]), df_from_double(em[2])};
    float out[6];
    for (int i = 0; i < 3; ++i) {
        DF acc = df_from_double(P[9 + i]);
        for (int j = 0; j < 3; ++j) acc = df_add(acc, df_mul(df_from_double(P[3 * i + j]), ev[j]));
        out[i] = acc.h;
        out[3 + i] = acc.l;
    }
    for (int q = 0; q < 6; ++q) xe[6 * e + q] = out[q];
    float dx = fmaxf(fmaxf(box_lo.x - out[0], out[0] - box_hi.x), 0.f);
    float dy = fmaxf(fmaxf(box_lo.y - out[1], out[1] - box_hi.y), 0.f);
    float dz = fmaxf(fmaxf(box_lo.z - out[2], out[2] - box_hi.z), 0.f);
    if (dx * dx + dy * dy + dz * dz < g.gmin * g.gmin) atomicOr(status, 1);
}

// Voxels of a region, in the order they are visited: offset from the region centre and
// |o|^2 (vtab), and region-relative indices plus the p0 offset from the region's first
// voxel (itab).  Entries past rx*ry*rz (padding to a multiple of 4) sit at the centre
// with index -1, i.e. outside every region.
__global__ void k_voxel_table(Geo g, float4* __restrict__ vtab, int4* __restrict__ itab) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    int n = g.rx * g.ry * g.rz;
    if (t >= g.nvpad) return;
    if (t >= n) {
        vtab[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        itab[t] = make_int4(1 << 30, 1 << 30, 1 << 30, 0);
        return;
    }
    int i = t / (g.ry * g.rz), j = (t / g.rz) % g.ry, k = t % g.rz;
    itab[t] = make_int4(i, j, k, (int)(i * g.vsx + j * g.vsy + k));
    DF sp{g.sp_h, g.sp_l};
    float ox = (float)i - 0.5f * (float)(g.rx - 1);
    float oy = (float)j - 0.5f * (float)(g.ry - 1);
    float oz = (float)k - 0.5f * (float)(g.rz - 1);
    DF x = df_mul(DF{ox, 0.f}, sp), y = df_mul(DF{oy, 0.f}, sp), z = df_mul(DF{oz, 0.f}, sp);
    DF oo = df_add(df_add(df_mul(x, x), df_mul(y, y)), df_mul(z, z));
    vtab[t] = make_float4(x.h, y.h, z.h, 0.5f * oo.h);       // |o|^2 / 2
}

__global__ void k_fill(float* __restrict__ p, size_t n, float v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_f64(double* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

__global__ void k_to_f32(const double* __restrict__ a, size_t n, float* __restrict__ out) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = (float)a[i];
}

__global__ void k_copy(const float* __restrict__ a, size_t n, float* __restrict__ out) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = a[i];
}

// Fixed-order FP64 sum of the loss partials (one workgroup of 256 threads, n <= 1024 floats).
__global__ __launch_bounds__(256) void k_loss_total(const float* __restrict__ part, int n,
                                                    double* __restrict__ out) {
    __shared__ double red[256];
    double a = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) a += (double)part[i];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// ------------------------------------------------------------------------------------------
// forward
// ------------------------------------------------------------------------------------------
// With EXACT, JT = floor(T sigma / delta + 1/2) is the largest |j| any pair's window can reach,
// and the Gaussian forward takes the 2 JT + 1 rows about the centre sample whole: every term of
// the window is among them, and the ones they add beyond |u| = T sigma are each below psi(T) of
// the kernel's peak (1.5e-7 at T = 6), below the FP32 rounding of a signal sample, so no row
// carries a window test.  Otherwise JT comes from a list spaced GEN_STEP apart, so every step up
// to JT - GEN_STEP lies inside (the host checks it) and only the last GEN_STEP steps are tested,
// each with a compile-time decision.

// One (voxel, element) pair of the forward model: add p0 * phi(u_k)/(2d) to the lane's
// private LDS row for the 2*JT+1 samples around the centre sample.
template <int JT, bool EXACT>
__device__ __forceinline__ void fwd_pair(const Geo& g, const VConst<JT, false>& c, const Ref& ref, float4 o,
                                         float pv, float* lane_rows) {
    const Pair p = make_pair(c, ref, o);
    const float A = pv * p.hr;
    float Rf = A * p.e0, Rb = Rf;
    float* lo = lane_rows + p.j0 * WAVE;
    float rw[2 * JT + 1];                  // rows j0-JT .. j0+JT: all reads issued first
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) rw[i] = lo[i * WAVE];
    rw[JT] = fmaf(p.u0, Rf, rw[JT]);
#pragma unroll
    for (int jj = 1; jj <= JT; ++jj) {
        Rf *= p.H;
        Rb *= p.Hi;
        // (u0 -+ j delta) Gamma_j, one FMA each
        float wf = fmaf(p.u0, c.gam[jj], -c.jdg[jj]), wb = fmaf(p.u0, c.gam[jj], c.jdg[jj]);
        if (!EXACT && jj > JT - GEN_STEP) {
            const float uf = fmaf(-(float)jj, c.dlt_h, p.u0), ub = fmaf((float)jj, c.dlt_h, p.u0);
            wf = fabsf(uf) <= c.tsig ? wf : 0.0f;
            wb = fabsf(ub) <= c.tsig ? wb : 0.0f;
        }
        rw[JT + jj] = fmaf(wf, Rf, rw[JT + jj]);
        rw[JT - jj] = fmaf(wb, Rb, rw[JT - jj]);
    }
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) lo[i * WAVE] = rw[i];
}

// Source profiles other than the Gaussian (Appendix A, normalised to K(0) = 1, width w):
// K(x) at x = |u|, and phi'(u) = K(x) + x K'(x) given k = K(x).  KT_POWER2 is the power law
// with nu = 2, K = 1/(1 + x^2/w^2)^2 by one reciprocal instead of a logarithm and an exponential
// (the host picks it when nu is exactly 2).
constexpr int KT_POWER2 = 4;

template <int KT>
__device__ __forceinline__ float prof(const Geo& g, float x) {
    if constexpr (KT == RA_KERNEL_EXPONENTIAL) return __builtin_amdgcn_exp2f(g.kexp * x);
    if constexpr (KT == RA_KERNEL_POWER)
        return __builtin_amdgcn_exp2f(g.knu * __builtin_amdgcn_logf(fmaf(x * x, g.kinv_w2, 1.0f)));
    if constexpr (KT == KT_POWER2) {
        const float r = __builtin_amdgcn_rcpf(fmaf(x * x, g.kinv_w2, 1.0f));
        return r * r;
    }
    return 1.0f;
}

template <int KT>
__device__ __forceinline__ float dprof(const Geo& g, float x, float k) {
    if constexpr (KT == RA_KERNEL_EXPONENTIAL) return k * fmaf(-x, g.kinv_w, 1.0f);
    if constexpr (KT == RA_KERNEL_POWER || KT == KT_POWER2) {
        const float q = x * x * g.kinv_w2;
        return k * fmaf(-g.k2nu * q, __builtin_amdgcn_rcpf(1.0f + q), 1.0f);
    }
    return 1.0f;
}

// One (voxel, element) pair of the forward model for a profile other than the Gaussian.
// These do not factor into a per-pair constant times fixed weights, so every sample of the
// window, |j| <= g.jwin steps from the centre sample, evaluates K(|u|) and its own window
// test |u| <= trunc sigma.  `centre` points at the lane's row of the reference sample kc.
template <int KT>
__device__ __forceinline__ void fwd_pair_var(const Geo& g, const VConst<0, false>& c, const Ref& ref, float4 o,
                                             float pv, float* centre) {
    const Dist q = pair_dist(ref, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    const float A = pv * q.hr;
    float* lo = centre + (int)jf * WAVE;
    const int jw = g.jwin;
#pragma unroll 4
    for (int jj = -jw; jj <= jw; ++jj) {
        const float u = residual(c, u0, (float)jj);      // u0 - jj delta
        const float x = fabsf(u);
        const float t = x <= c.tsig ? u * prof<KT>(g, x) : 0.0f;
        lo[jj * WAVE] = fmaf(A, t, lo[jj * WAVE]);
    }
}

// One pair of the forward model for the exponential profile.  Its exponent is linear in
// |u|, so each leg factors exactly: at step j >= 1 after the centre sample u = u0 - j delta
// < 0 and K = exp(u0/w) G_j, before it u = u0 + j delta > 0 and K = exp(-u0/w) G_j, with
// G_j = exp(-j delta/w) in the per-call table gam[] (jdg[] = j delta G_j).  Each sample then
// costs one FMA for its weight (u0 -+ j delta) G_j and one to accumulate, with no
// recurrence.  JT comes from a list spaced EXP_STEP apart; the last EXP_STEP steps carry their
// own window test.
template <int JT>
__device__ __forceinline__ void fwd_pair_exp(const Geo& g, const VConst<JT, false>& c, const Ref& ref, float4 o,
                                             float pv, float* lane_rows) {
    const Dist q = pair_dist(ref, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    const float A = pv * q.hr;
    const float x0 = u0 * g.kexp;                         // u0/w in log2 units
    const float Rf = A * __builtin_amdgcn_exp2f(-x0);     // A exp(u0/w)
    const float Rb = A * __builtin_amdgcn_exp2f(x0);      // A exp(-u0/w)
    float* lo = lane_rows + (int)jf * WAVE;
    float rw[2 * JT + 1];
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) rw[i] = lo[i * WAVE];
    rw[JT] = fmaf(u0 * A, __builtin_amdgcn_exp2f(fabsf(u0) * g.kexp), rw[JT]);
#pragma unroll
    for (int jj = 1; jj <= JT; ++jj) {
        float wf = fmaf(u0, c.gam[jj], -c.jdg[jj]), wb = fmaf(u0, c.gam[jj], c.jdg[jj]);
        if (jj > JT - EXP_STEP) {
            const float uf = fmaf(-(float)jj, c.dlt_h, u0), ub = fmaf((float)jj, c.dlt_h, u0);
            wf = fabsf(uf) <= c.tsig ? wf : 0.0f;
            wb = fabsf(ub) <= c.tsig ? wb : 0.0f;
        }
        rw[JT + jj] = fmaf(wf, Rf, rw[JT + jj]);
        rw[JT - jj] = fmaf(wb, Rb, rw[JT - jj]);
    }
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) lo[i * WAVE] = rw[i];
}

// Forward contributions of two neighbouring voxels a, b, added to the rows in one pass.  Both are
// expanded about the smaller of their centre samples, base: with u' = d - (kc + base) delta, the
// kernel value at row base + j is R_j (u' - j delta) Gamma_j with R_j = e0' H'^j (e0' =
// exp(-u'^2/2s^2), H' = exp(u' delta/s^2)), so each row is read and written once for both voxels.
// The voxel whose centre sample is the base ("lo", |u'| <= delta/2) takes its own rows -JT .. JT;
// the other ("hi", u' in [-delta/2, (D + 1/2) delta]) takes rows -JT .. JT + D, which hold its
// own 2 JT + 1 rows; its rows beyond those lie further out than any window row (|u| > (JT + 1/2)
// delta), each below the bound of the whole-row reading above.  Each voxel's R_j is one chain of
// multiplies by H' from row -JT, started at p exp2(u'(kappa u' - JT alpha) - 1) / d (the -1
// halves 1/d to 1/(2d)): two exponentials per voxel.  Requires |j0(a) - j0(b)| <= D, which
// holds when a and b are grid neighbours and spacing < D delta.
template <int JT, int D>
__device__ __forceinline__ void fwd_two(const VConst<JT + D, false>& c, const Ref& ref, float4 oa, float pa,
                                        float4 ob, float pb, float* lane_rows) {
    const Dist A = pair_dist(ref, oa), B = pair_dist(ref, ob);
    const float ja = rintf(A.uc * c.inv_dlt), jb = rintf(B.uc * c.inv_dlt);
    // |j| <= jclamp by the triangle inequality; the clamp keeps LDS indices in range whatever the
    // inputs (NaN converts to 0)
    const float bf = __builtin_amdgcn_fmed3f(fminf(ja, jb), c.njclampf, c.jclampf);
    const float ua = residual(c, A.uc, bf), ub = residual(c, B.uc, bf);
    const bool alo = ja <= jb;
    const float ul = alo ? ua : ub, uh = alo ? ub : ua;
    const float al = alo ? pa * A.rs : pb * B.rs, ah = alo ? pb * B.rs : pa * A.rs;
    const float ctop = -(float)JT * c.alpha;
    const float Hl = __builtin_amdgcn_exp2f(c.alpha * ul), Hh = __builtin_amdgcn_exp2f(c.alpha * uh);
    float Rl = al * __builtin_amdgcn_exp2f(fmaf(ul, fmaf(c.kappa, ul, ctop), -1.0f));
    float Rh = ah * __builtin_amdgcn_exp2f(fmaf(uh, fmaf(c.kappa, uh, ctop), -1.0f));
    float* lo = lane_rows + (int)bf * WAVE;
    constexpr int NR = 2 * JT + 1 + D;
    float rw[NR];                          // rows base-JT .. base+JT+D: all reads issued first
#pragma unroll
    for (int i = 0; i < NR; ++i) rw[i] = lo[i * WAVE];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int j = i - JT;
        // (u' - j delta) Gamma_j, one FMA
        const float wh = j == 0 ? uh : (j > 0 ? fmaf(uh, c.gam[j], -c.jdg[j]) : fmaf(uh, c.gam[-j], c.jdg[-j]));
        if (i > 0) Rh *= Hh;
        if (j <= JT) {
            const float wl = j == 0 ? ul : (j > 0 ? fmaf(ul, c.gam[j], -c.jdg[j]) : fmaf(ul, c.gam[-j], c.jdg[-j]));
            if (i > 0) Rl *= Hl;
            rw[i] = fmaf(wl, Rl, fmaf(wh, Rh, rw[i]));
        } else {
            rw[i] = fmaf(wh, Rh, rw[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) lo[i * WAVE] = rw[i];
}

// The forward work of one region: every element chunk of the region, shared among the
// workgroup's wavefronts (chunks wave, wave + WAVES, ...).  `rows` is the calling
// wavefront's private LDS block of g.L sample rows, zero on entry and on exit.
template <int JT, bool EXACT, int D, typename SumT, int KT = RA_KERNEL_GAUSSIAN>
__device__ __forceinline__ void forward_region(const Geo& g, int reg, const float* __restrict__ p0,
                                               const float* __restrict__ xe, const float4* __restrict__ vtab,
                                               const int4* __restrict__ itab, SumT* __restrict__ s,
                                               float* rows, int lane, int wave) {
    const Region R = region_info(g, reg);
    const float* pbase = p0 + (size_t)R.i0 * g.vsx + (size_t)R.j0 * g.vsy + R.k0;
    const int nchunk = (g.E + WAVE - 1) / WAVE;
    VConst<JT + D, false> cst;
    // per-call constants in VGPRs where the register file allows it (measured faster for the
    // Gaussian up to 24 steps; beyond that they would cost occupancy)
    load_vconst<KT == RA_KERNEL_GAUSSIAN && JT + D <= 27>(cst, g);
    // g.zero is 0: the per-lane index makes the voxel loads vector loads (VGPR results)
    const int zl = lane * g.zero;
    // regions wholly inside the grid whose z-rows hold a multiple of 4 voxels skip the per-voxel
    // bounds tests
    const bool interior = R.ni == g.rx && R.nj == g.ry && R.nk == g.rz && (g.rz & 3) == 0;

    for (int c = wave; c < nchunk; c += WAVES) {
        const int e = c * WAVE + lane;
        const bool valid = e < g.E;
        // lanes past the last element model element 0; their rows are cleared, not flushed
        const Ref ref = make_ref(g, xe, valid ? e : 0, R);
        float* lane_rows = rows + lane + (g.kmargin - JT) * WAVE;
        // voxels four at a time, the next four loading while the current are processed
        float4 oa[4], ob[4];
        float pa[4], pb[4];
        auto fetch = [&](float4* o, float* pv, int t) {
            if (interior) {            // four consecutive voxels along z, all inside the grid
                const int off = itab[t].w;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = vtab[t + q + zl];
                    pv[q] = pbase[off + q + zl];
                }
                return;
            }
            // a voxel that is not there (an element may be) stands at the first of its pair, or of the region
            const float4 first = vtab[zl];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int4 ix = itab[t + q];
                const bool inside = ix.x < R.ni && ix.y < R.nj && ix.z < R.nk;
                o[q] = vtab[t + q + zl];
                if (!inside) o[q] = (q & 1) ? o[q - 1] : first;
                const float v = pbase[(inside ? ix.w : 0) + zl];
                pv[q] = inside ? v : 0.0f;
            }
        };
        auto work = [&](const float4* o, const float* pv) {
            if constexpr (KT == RA_KERNEL_EXPONENTIAL) {
#pragma unroll
                for (int q = 0; q < 4; ++q) fwd_pair_exp<JT>(g, cst, ref, o[q], pv[q], lane_rows);
            } else if constexpr (KT != RA_KERNEL_GAUSSIAN) {
#pragma unroll
                for (int q = 0; q < 4; ++q) fwd_pair_var<KT>(g, cst, ref, o[q], pv[q], lane_rows);
            } else if constexpr (D == 0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) fwd_pair<JT, EXACT>(g, cst, ref, o[q], pv[q], lane_rows);
            } else {
                fwd_two<JT, D>(cst, ref, o[0], pv[0], o[1], pv[1], lane_rows);
                fwd_two<JT, D>(cst, ref, o[2], pv[2], o[3], pv[3], lane_rows);
            }
        };
        fetch(oa, pa, 0);
        for (int t = 0; t < g.nvpad; t += 8) {
            const bool more = t + 4 < g.nvpad;
            if (more) fetch(ob, pb, t + 4);
            work(oa, pa);
            if (!more) break;
            if (t + 8 < g.nvpad) fetch(oa, pa, t + 8);
            work(ob, pb);
        }
        // Add the rows to HBM and clear them.  The single-call forward adds into FP64 sums, so
        // that its rounding does not grow with the number of regions whose partial rows meet in
        // one sample (thousands at 256^3 seen from 60 mm).  Lane ix takes
        // row ix of four elements at a time (one 16-byte LDS access: all lanes read the same four
        // banks, so four elements cost what one did); each atomic instruction covers consecutive
        // samples of one element.
        for (int qb = 0; qb < WAVE; qb += 4) {
            int kb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) kb[i] = __builtin_amdgcn_readlane(ref.kbase, qb + i);
            for (int ix = lane; ix < g.L; ix += WAVE) {
                float4* slot = reinterpret_cast<float4*>(rows + ix * WAVE + qb);
                const float4 v4 = *slot;
                *slot = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int eq = c * WAVE + qb + i;
                    const int k = kb[i] + ix;
                    if (eq < g.E && v[i] != 0.0f && k >= 0 && k < g.K)
                        atomicAdd(&s[(size_t)eq * g.K + k], (SumT)v[i]);
                }
            }
        }
    }
}

// SumT: the type the region's partial rows are added into in memory (float: straight into the
// caller's signals; double: FP64 sums converted afterwards).
template <int JT, bool EXACT, int D, int KT = RA_KERNEL_GAUSSIAN, typename SumT = double>
__global__ __launch_bounds__(BLOCK) void k_forward(Geo g, const float* __restrict__ p0,
                                                   const float* __restrict__ xe,
                                                   const float4* __restrict__ vtab,
                                                   const int4* __restrict__ itab,
                                                   SumT* __restrict__ s) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    float* rows = lds + (size_t)wave * g.L * WAVE;
    for (int ix = 0; ix < g.L; ++ix) rows[ix * WAVE + lane] = 0.0f;
    forward_region<JT, EXACT, D, SumT, KT>(g, region_of_block(blockIdx.x, g.nreg), p0, xe, vtab, itab, s, rows,
                                           lane, wave);
}

// ------------------------------------------------------------------------------------------
// forward in moment form (Gaussian, exponential and power-law profiles)
// ------------------------------------------------------------------------------------------
// With lengths in units of delta / 2, a pair's distance is d = 2 kc + t with kc its nearest sample and
// |t| <= 1.  The window row kc + j carries phi((t/2 - j) delta), which on |t| <= 1 is a polynomial
// sum_n D_n(j) t^n of NM terms: its Chebyshev series, cut after NM terms on the host, which takes
// the form only where the cut part is below FM_TOL of the pulse's peak.  So a pair needs only add
// a t^n (a = p0/(2d), n < NM) to NM sums of its centre sample, and the region's signal rows follow
// from all pairs' sums at once:
//   s[kc + r] = sum_{|j| <= jt} sum_n D_n(j) M_n[r - j].
//
// The scatter.  A workgroup owns one region and one chunk of 64 elements at a time; its wavefronts share
// one set of sums in LDS, [centre sample][n][lane = element], and take different columns of the region.
// The adds are LDS atomics: ds_add_f32 takes 193 cycles a wavefront here (it serialises the lanes),
// ds_add_u32 4.7, a private read-modify-write 5.7 (and then every wavefront would need its own set), so
// the sums are 32-bit fixed point.  Their unit is chosen per region and element so that no sum can
// overflow.  The voxels of one bin lie within one sample of each other, so of a line of voxels along an
// axis the bin holds at most 1 + delta / (h c) of them, c the least |cosine| between the axis and the
// direction to the element over the region; with B the sum over the lines of the largest |p0| in each,
// the bin's sum is at most that count times B / d_low, d_low being the element's distance to the
// region's box.  The best of the three axes, or sum |p0| / d_low, becomes 2^31 units: for 16^3 equal
// voxels a term is rounded to 1.2e-7 of itself, as one FP32 addition would.  Regions whose p0 is not
// finite, and elements inside or within half a voxel of the region's box, or not finite, take FP32 sums
// by ds_add_f32 instead (slow, and the values then propagate as they would in FP32).  A region whose
// voxels differ by many orders of magnitude is summed in classes of size (fm_bound).
//
// The expansion into rows is a banded Toeplitz product, [rows x 64] = D [rows x (bins NM)] M: FP32
// matrix instructions (16 rows x 16 elements x 4 bins each), whose result has consecutive samples
// of an element in consecutive lanes, as the atomic adds into the signals want them.
//
// Distances.  A region is up to 1.3 mm in radius, 67 units, where FP32 rounds u = d - c t to 4e-6 units;
// so each column of 8 voxels first takes its own distance and nearest sample, with D.o split into a
// part that adds exactly and the rest, and its voxels count from there: rms error of t 0.9e-6 over
// 16^3 voxels, against 1.4e-6 in the row form over 8x8x16.  With edge terms the column's distance is
// FP64 and the same in every region (fm_col_f64).
//
// Bounds: 24 VALU instructions (one at a quarter of the rate) and NM ds_add_u32 (33 LDS cycles at NM = 7)
// per pair and wavefront plus about 40 per column, against 104 VALU and 58 LDS cycles per pair in the
// row form.  On the sweep (128x128x64 voxels of 0.1 mm, 8192 elements, sigma 0.08 mm) the adds take
// about 8 ms of 9.9, the row form 26.9.  The FP32 matrix instructions share the VALU's time, so the
// expansion adds to that: 5.7 ms with 8x8x8 regions, two workgroups to a CU; hence the largest regions
// that the LDS holds, one workgroup of 16 wavefronts to a CU.
__device__ __forceinline__ float mom_coef(const MomCoef& m, int n, int j, int jt) {
    const int a = j < 0 ? -j : j;
    if (a > jt) return 0.0f;
    const float v = m.d[a * MOM_MAX + n];
    return (j < 0 && !(n & 1)) ? -v : v;
}

// Four floats as a native vector: copies of it are plain vector moves (no byte copies through
// memory), so arrays of it stay in registers.
typedef float vf4 __attribute__((ext_vector_type(4)));

constexpr int FM_PAD = 20;                                   // zeros before D_n(-jt) in its LDS table
constexpr int fm_stride(int nm) { return nm * WAVE + 16; }   // LDS words per bin: 4 bins read at once hit 32 banks
constexpr int fm_dlen(int jt) { return 2 * jt + 1 + FM_PAD + 16; }
// Its LDS in floats: sums and one zero bin, references, voxel offsets per axis, |p0| sums, D table.
constexpr size_t fm_off_ref(int nm, int nbin) { return (size_t)(nbin + 1) * fm_stride(nm); }
constexpr size_t fm_off_axis(int nm, int nbin) { return fm_off_ref(nm, nbin) + FM_REFS * FM_FIELDS * WAVE; }
constexpr size_t fm_off_red(int nm, int nbin) { return fm_off_axis(nm, nbin) + 3 * FM_SIDE * 4; }
constexpr size_t fm_off_dt(int nm, int nbin) { return fm_off_red(nm, nbin) + 4 * FM_WAVES_BIG + 4; }
constexpr size_t fm_off_edge(int nm, int nbin, int jt) { return fm_off_dt(nm, nbin) + (nm * fm_dlen(jt) + 63) / 64 * 64; }
constexpr size_t fm_lds(int nm, int nbin, int jt, bool edge) {       // with edge sums, [row][lane]
    return (fm_off_edge(nm, nbin, jt) + (edge ? (size_t)(nbin + 2 * jt) * WAVE : 0)) * sizeof(float);
}

// What bounds the sums of a region's bins: sum |p0|, and per axis the sum over the lines along it of the
// largest |p0| in each (NaN if any p0 is not finite).
struct FmBound {
    float all, line[3], low;               // low: see fm_bound
};

// Reference of a (region, element) pair in units: D = centre - x_e in double-float, dh = |D| rounded,
// uc0 = dh - 2 kc, n0 = (|D|^2 - dh^2) / 2, and the quantum of the column sums.
struct MomRef {
    float D[3], Dl[3], dh, uc0, n0, magic;
    int kc;                                // nearest sample
};

__device__ __forceinline__ MomRef mom_make_ref(const Geo& g, const float* __restrict__ x, const Region& R) {
#pragma clang fp contract(off)
    const DF u{g.unit_h, g.unit_l};
    const DF D[3] = {df_mul(df_add(R.cx, df_neg(DF{x[0], x[3]})), u), df_mul(df_add(R.cy, df_neg(DF{x[1], x[4]})), u),
                     df_mul(df_add(R.cz, df_neg(DF{x[2], x[5]})), u)};
    const DF d = df_sqrt(df_add(df_add(df_mul(D[0], D[0]), df_mul(D[1], D[1])), df_mul(D[2], D[2])));
    const float kc = rintf(0.5f * d.h);
    MomRef r;
    float h2 = 0.0f;
    const int n[3] = {g.rx, g.ry, g.rz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.D[a] = D[a].h;
        r.Dl[a] = D[a].l;
        const float half = 0.5f * (float)(n[a] - 1) * g.hs_u;
        h2 += half * half;
    }
    r.dh = d.h;
    r.uc0 = d.h - 2.0f * kc;
    r.n0 = d.h * d.l;
    r.kc = (int)kc;
    // |D.o + o.o/2| < 2^e of this product, so multiples of 2^(e - 22) below it add exactly
    const float rad = sqrtf(h2) + 4.0f * g.hs_u;
    r.magic = 1.5f * __builtin_amdgcn_ldexpf(1.0f, __builtin_amdgcn_frexp_expf(rad * (d.h + rad)) + 1);
    return r;
}

// The scale of a pair's fixed-point sums and its inverse; 0 where FP32 sums are taken.
struct FmScale {
    float scale, inv;
};

__device__ __forceinline__ FmScale fm_scale(const Geo& g, const Region& R, const MomRef& m, const FmBound& bd) {
#pragma clang fp contract(off)
    const float half[3] = {0.5f * (float)(g.rx - 1) * g.hs_u, 0.5f * (float)(g.ry - 1) * g.hs_u,
                           0.5f * (float)(g.rz - 1) * g.hs_u};
    const float far = m.dh + sqrtf(half[0] * half[0] + half[1] * half[1] + half[2] * half[2]);
    const int n[3] = {R.ni, R.nj, R.nk};
    float dl2 = 0.0f, most = bd.all;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // distance past the region's voxels along the axis, before the first or beyond the last
        const float out = fmaxf(m.D[a] - half[a], half[a] - (float)(n[a] - 1) * g.hs_u - m.D[a]);
        if (!(out > 0.0f)) continue;
        dl2 += out * out;
        const float gap = g.hs_u * 0.999f * out / far;       // least difference in distance of two voxels of a line
        const float cnt = floorf(2.0f / gap) + 1.0f;         // voxels of a line within one bin (2 units)
        most = fminf(most, cnt * bd.line[a]);
    }
    most = bd.all - bd.all == 0.0f ? most * 1.001f : bd.all;  // fminf drops NaN
    const float dlow = sqrtf(dl2) * 0.999f;
    // 1/d <= 1/dlow for every term of the region; scale 0 (take FP32 sums) where that says nothing
    const bool ok = dlow >= 0.5f * g.hs_u && m.dh < 1e15f;
    FmScale r;
    r.scale = ok ? 2.147e9f * dlow / most : 0.0f;
    r.inv = most / (2.147e9f * dlow);
    if (!(r.scale > 0.0f && r.scale < 1e37f && r.inv > 1e-37f && r.inv < 1e37f)) r.scale = r.inv = 0.0f;
    return r;
}

// One axis' share of N = D.o + o.o/2 for the voxel offset o = t.x + t.y (t.z = o^2/2): hi, a multiple
// of the quantum that `magic` rounds to, and what is left.
__device__ __forceinline__ void fm_axis(float4 t, float D, float Dl, float magic, float& hi, float& lo) {
#pragma clang fp contract(off)
    const float p = t.x * D, e = fmaf(t.x, D, -p);
    const float w = p + t.z;
    hi = (w + magic) - magic;
    lo = fmaf(t.y, D, fmaf(t.x, Dl, ((p - hi) + t.z) + e));
}

__device__ __forceinline__ int cvt_round_i32(float x) {      // floor(x + 1/2)
    int v;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(v) : "v"(x));
    return v;
}

// Offsets of a region's voxels from its centre along each axis, [axis][index] (along z: of the centres of its
// columns), as fm_axis takes them.  A column holds FM_RZ voxels, the last of a region that ends short those up to nk: its
// centre is that of its own voxels, since an element may be where the missing ones would be.  Where regions are one
// column deep, index 1 along z is for the grid's last ones.
__device__ __forceinline__ void fm_axis_table(const Geo& g, int nk, int tid, float4* axis) {
    if (tid >= 3 * FM_SIDE) return;
    const int a = tid / FM_SIDE, i = tid % FM_SIDE;
    const bool last = g.rz <= FM_RZ && i == 1;
    const int z0 = last ? 0 : i * FM_RZ, len = last ? g.nz - (g.nrz - 1) * g.rz : min(FM_RZ, max(nk - z0, 1));
    const float n = a == 0 ? (float)i - 0.5f * (float)(g.rx - 1)
                           : a == 1 ? (float)i - 0.5f * (float)(g.ry - 1)
                                    : (float)z0 + 0.5f * (float)(len - 1) - 0.5f * (float)(g.rz - 1);
    const DF o = df_mul(DF{n, 0.0f}, DF{g.hs_u, g.hs_l});
    axis[tid] = make_float4(o.h, o.l, 0.5f * o.h * o.h, 0.0f);
}

// N of each of a column's nz voxels about the column's centre, which is tz along z from the region's; the rest of the
// FM_RZ repeat the last one (with no weight).
__device__ __forceinline__ void fm_column_n(const Geo& g, int nz, float4 tz, float Dz, float Dzl, float (&ez)[FM_RZ]) {
#pragma clang fp contract(off)
    const DF Dc = df_add(DF{Dz, Dzl}, DF{tz.x, tz.y});
    auto at = [&](float k) {
        const DF o = df_mul(DF{k, 0.0f}, DF{g.hs_u, g.hs_l});
        return fmaf(o.h, Dc.l, fmaf(o.l, Dc.h, o.h * fmaf(0.5f, o.h, Dc.h)));
    };
    if (nz >= FM_RZ) {                                       // with constant offsets, which leave the loops over chunks
#pragma unroll
        for (int k = 0; k < FM_RZ; ++k) ez[k] = at((float)k - 0.5f * (float)(FM_RZ - 1));
    } else {
#pragma unroll
        for (int k = 0; k < FM_RZ; ++k) ez[k] = at((float)min(k, nz - 1) - 0.5f * (float)(nz - 1));
    }
}

constexpr float FM_MAGIC = 25165824.0f;    // 1.5 * 2^24: adding it rounds to a multiple of 2 (a sample)

// A column of FM_RZ voxels: its centre's distance dc, that distance from the column's own nearest sample
// (uc), and FM_MAGIC plus that sample's offset from kc.
struct FmCol {
    float dc, uc, magic;
};

// bh + bl = N at the column's centre; bh is exact.  One Newton step from y = sqrt(dh^2 + 2 bh), with
// a = y - dh exact: d = y + (N - a dh - a^2/2) / y.
__device__ __forceinline__ FmCol fm_col(float bh, float bl, float dh, float dh2, float uc0) {
#pragma clang fp contract(off)
    const float S = fmaf(2.0f, bh, dh2);
    const float rs = __builtin_amdgcn_rsqf(S);
    const float y = S * rs;
    const float a = y - dh;
    const float th = fmaf(-0.5f, a * a, fmaf(-a, dh, bh)) + bl;
    const float corr = fmaf(th, rs, uc0);
    FmCol c;
    c.magic = (a + corr) + FM_MAGIC;
    c.uc = (a - (c.magic - FM_MAGIC)) + corr;
    c.dc = y;
    return c;
}

// The same for the profiles with edge terms, from the column's and the element's own positions in FP64, so that it depends
// on nothing of the region: the forward and the adjoints, on regions of different sizes, then find the same t of a
// pair to the last bit and put an outermost sample in or out alike (from each region's centre, a pair within
// rounding of the edge fell in on one side and out on the other: <A p, r> and <p, A^T r> apart by 1e-3 of |A p| where
// all pairs are at the edge).  c: the column's centre from the element, in units.
struct FmElem {
    double x, y, z, h;                     // grid origin from the element, spacing; units
};

__device__ __forceinline__ FmElem fm_elem(const Geo& g, const float* __restrict__ x) {
#pragma clang fp contract(off)
    const double u = (double)g.unit_h + (double)g.unit_l;
    double o[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        o[a] = (((double)g.org_h[a] + (double)g.org_l[a]) - ((double)x[a] + (double)x[3 + a])) * u;
    return {o[0], o[1], o[2], ((double)g.sp_h + (double)g.sp_l) * u};
}

__device__ __forceinline__ FmCol fm_col_f64(double cx2z2, double cy, int kc) {
#pragma clang fp contract(off)
    const double S = fma(cy, cy, cx2z2);
    const double y0 = __builtin_amdgcn_rsq(S);
    double d = S * y0, hf = 0.5 * y0;
    const double r = fma(-hf, d, 0.5);
    d = fma(d, r, d);
    hf = fma(hf, r, hf);
    d = S > 0.0 ? fma(fma(-d, d, S), hf, d) : S;             // 0, and NaN as it is
    const double k = __builtin_rint(0.5 * d);
    FmCol c;
    c.dc = (float)d;
    c.uc = (float)fma(-2.0, k, d);
    c.magic = FM_MAGIC + 2.0f * (float)(k - (double)kc);
    return c;
}

__device__ __forceinline__ double fm_square_add(double c, double s) { return fma(c, c, s); }

// N of a column's voxels about its centre, cz along z from the element.
__device__ __forceinline__ void fm_column_n(const Geo& g, int nz, double cz, float (&ez)[FM_RZ]) {
    const float h = (float)cz;
    fm_column_n(g, nz, make_float4(0.0f, 0.0f, 0.0f, 0.0f), h, (float)(cz - (double)h), ez);
}

// A voxel of the column: rs = 1/d, t, and FM_MAGIC plus its nearest sample's offset from kc (kept in
// [lo, hi] whatever the inputs).
struct FmPair {
    float rs, t, rm;
};

__device__ __forceinline__ FmPair fm_pair(const FmCol& c, float dc2, float hdc, float ez, float lo, float hi) {
#pragma clang fp contract(off)                 // the distance's Newton step, as pair_dist
    FmPair p;
    const float S = fmaf(2.0f, ez, dc2);
    p.rs = __builtin_amdgcn_rsqf(S);
    const float y = S * p.rs;
    const float a = y - c.dc;
    const float bh = fmaf(0.5f, y, hdc);
    const float th = fmaf(-a, bh, ez);
    const float uc = c.uc + fmaf(th, p.rs, a);
    p.rm = __builtin_amdgcn_fmed3f(uc + c.magic, lo, hi);      // NaN lands in range too
    p.t = uc - (p.rm - c.magic);
    return p;
}

// What a pair adds beyond its polynomial, at one of the window's outermost samples kc +- jt, each of which is in
// the window for |u| <= T w only.  If the window reaches less than half a sample past kc + jt - 1/2 .. (thr > 0, the
// polynomial holds |j| < jt), that is the sample on t's side, for |t| >= thr; otherwise the polynomial holds |j| <= jt and
// the sample on the other side is taken back for |t| > thr.  phi is odd, so both are sgn(t) F(|t|); F: four terms.
struct Edge {
    float v, d;                            // value and its derivative in t (0 inside thr)
    unsigned row;                          // 0: kc - jt, or the byte offset of kc + jt
};

struct EdgeCoef {
    float thr, e0, e1, e2, e3;
    unsigned flip, far;
};

__device__ __forceinline__ EdgeCoef edge_coef(const Geo& g, float scale) {     // in vector registers
    EdgeCoef c{g.thr, g.ev[0] * scale, g.ev[1] * scale, g.ev[2] * scale, g.ev[3] * scale, g.flip,
               (unsigned)g.jt * 2u * WAVE * 4u};
    asm volatile("" : "+v"(c.thr), "+v"(c.e0), "+v"(c.e1), "+v"(c.e2), "+v"(c.e3), "+v"(c.flip), "+v"(c.far));
    return c;
}

__device__ __forceinline__ Edge edge_phi(const EdgeCoef& c, float t) {
    const float a = fabsf(t);
    const bool in = a >= c.thr;
    const float f = fmaf(a, fmaf(a, fmaf(a, c.e3, c.e2), c.e1), c.e0);
    const float d = fmaf(a, fmaf(3.0f * a, c.e3, 2.0f * c.e2), c.e1);
    Edge e;
    e.v = in ? copysignf(1.0f, t) * f : 0.0f;
    e.d = in ? d : 0.0f;
    e.row = ~(unsigned)((int)(__float_as_uint(t) ^ c.flip) >> 31) & c.far;
    return e;
}

// The adds of one column of FM_RZ voxels (p0 values pv, zero past the grid); ez: N of each voxel about
// the column's centre.  INT: fixed-point sums.
template <int NM, bool INT, int X>
__device__ __forceinline__ void fm_column(const Geo& g, const EdgeCoef& xc, unsigned eoff, const float (&pv)[FM_RZ],
                                          const float (&ez)[FM_RZ], const FmCol& c, float scale, float lo, float hi,
                                          unsigned off0, unsigned str, char* sums) {
    const float dc2 = c.dc * c.dc, hdc = 0.5f * c.dc;
#pragma unroll
    for (int k = 0; k < FM_RZ; ++k) {
        const FmPair p = fm_pair(c, dc2, hdc, ez[k], lo, hi);
        // the low 24 bits of rm are 0xC00000 + (centre sample offset)
        const unsigned off = __umul24(__float_as_uint(p.rm), str) + off0;
        float q = pv[k] * p.rs;
        if (INT) q *= scale;
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            if (INT) {
                int* dst = reinterpret_cast<int*>(sums + off) + n * WAVE;
                __hip_atomic_fetch_add(dst, cvt_round_i32(q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                float* dst = reinterpret_cast<float*>(sums + off) + n * WAVE;
                __hip_atomic_fetch_add(dst, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if (n + 1 < NM) q *= p.t;
        }
        if (X) {                               // sums of single rows: of kc - jt at er
            const float a = INT ? pv[k] * p.rs * scale : pv[k] * p.rs;
            const unsigned er = (__float_as_uint(p.rm) << 8) + eoff;
            const Edge e = edge_phi(xc, p.t);
            auto add = [&](unsigned at, float v) {
                if (INT)
                    __hip_atomic_fetch_add(reinterpret_cast<int*>(sums + at), cvt_round_i32(v), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                else if (v != 0.0f)
                    __hip_atomic_fetch_add(reinterpret_cast<float*>(sums + at), v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            add(er + e.row, INT || e.v != 0.0f ? a * e.v : 0.0f);
            if (X == 2)
                add(er + xc.far / 2u, (a * 0.5f * g.es) * (p.t * __builtin_amdgcn_exp2f(g.kx * fabsf(p.t))));
        }
    }
}

// A value that the whole wavefront has, in a scalar register.
__device__ __forceinline__ float to_scalar(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// Sum |p0| and the line bounds of a region's voxels with |p0| below top by the whole workgroup (`red`: LDS, 4 floats a
// wavefront and 3), and from where on its voxels make a class of their own (FmBound's `low`, 0: they are taken together).
// One unit for all sums of a region suits voxels of like size.  A line is faint if its largest |p0| is below FM_FAINT
// of what bounds the region's bins, so that the unit would exceed 2^-17 of it; where one line in 16 along any axis is,
// the voxels from FM_FAINT of the bound on are summed first and the rest after them, in a unit of their own.  One voxel
// of 1e4 over a background of 0.01: the samples that it does not reach are off by 2.5e-4 of themselves in one unit.
template <int NW>
__device__ __forceinline__ FmBound fm_bound(const Geo& g, const Region& R, const float* __restrict__ pbase, float top,
                                            float* red) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
    const int n[3] = {R.ni, R.nj, R.nk};
    const long long st[3] = {g.vsx, g.vsy, 1};
    float b[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float most[3] = {0.0f, 0.0f, 0.0f};                      // of this thread's line: at most FM_SIDE^2 of them along an axis
    static_assert(NW * WAVE >= FM_SIDE * FM_SIDE, "a thread per line");
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int p = a == 0 ? 1 : 0, q = a == 2 ? 1 : 2;    // the other two axes
        if (tid < n[p] * n[q]) {
            const float* line = pbase + (size_t)(tid / n[q]) * st[p] + (size_t)(tid % n[q]) * st[q];
            float sum = 0.0f;
            for (int i = 0; i < n[a]; ++i) {
                float v = fabsf(line[(size_t)i * st[a]]);
                v = v >= top ? 0.0f : v;                     // with top NaN all stay, and NaN does
                most[a] = fmaxf(most[a], v);
                sum += v;
            }
            b[a] = most[a];
            if (a == 2) b[3] = sum;
        }
    }
    int* few = reinterpret_cast<int*>(red + 4 * FM_WAVES_BIG);   // per axis: 16 times the faint lines, less the lines with any voxel
    if (tid < 3) few[tid] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        b[i] = wave_sum_to_63(b[i]);
        if (lane == WAVE - 1) red[4 * wv + i] = b[i];
    }
    __syncthreads();
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] += red[4 * w + i];
    FmBound r{to_scalar(t[3]), {to_scalar(t[0]), to_scalar(t[1]), to_scalar(t[2])}, 0.0f};
    const bool finite = r.all - r.all == 0.0f;
    const float low = FM_FAINT * fminf(fminf(r.line[0], r.line[1]), fminf(r.line[2], r.all));
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int faint = __popcll(__ballot(most[a] > 0.0f && most[a] < low)), any = __popcll(__ballot(most[a] > 0.0f));
        if (lane == 0 && any) __hip_atomic_fetch_add(few + a, 16 * faint - any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    if (finite && max(few[0], max(few[1], few[2])) > 0) r.low = low;
    r.low = to_scalar(r.low);
    return r;
}

// The forward work of one region for element chunks c0, c0 + cstep, ...  `lds` is the workgroup's LDS
// (fm_lds bytes) with the D table in place.  Every thread of the workgroup must call it.
template <int NM, int NW, int X, typename SumT>
__device__ __forceinline__ void fm_region(const Geo& g, int reg, int c0, int cstep, const float* __restrict__ p0,
                                          const float* __restrict__ xe, SumT* __restrict__ s, float* lds) {
    constexpr int STR = fm_stride(NM);
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int nbin = g.nbin, jt = g.jt, K = g.K;
    const int rows = nbin + 2 * jt;
    float* refs = lds + fm_off_ref(NM, nbin);                // [slot][field][lane]
    float4* axis = reinterpret_cast<float4*>(lds + fm_off_axis(NM, nbin));
    const float* dt = lds + fm_off_dt(NM, nbin);
    float* edge = lds + fm_off_edge(NM, nbin, jt);           // sums of single rows, [row][lane]
    const Region R = region_info(g, reg);
    const float* pbase = p0 + (size_t)R.i0 * g.vsx + (size_t)R.j0 * g.vsy + R.k0;
    const int nchunk = (g.E + WAVE - 1) / WAVE;
    const int ncol = R.ni * R.nj, mine = (ncol + NW - 1) / NW;
    for (int i = tid; i < (nbin + 1) * STR / 4; i += NW * WAVE)
        reinterpret_cast<float4*>(lds)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (X)
        for (int i = tid; i < rows * WAVE; i += NW * WAVE) edge[i] = 0.0f;
    fm_axis_table(g, R.nk, tid, axis);
    const float rlo = FM_MAGIC - 2.0f * g.jclampf, rhi = FM_MAGIC + 2.0f * g.jclampf;
    const float ies = X ? 1.0f / g.es : 0.0f;

    // classes of voxels, the largest first (see fm_bound): those from low on and below top (NaN: no limit)
    float top = __builtin_nanf("");
    for (bool more = true; more;) {
        const FmBound bound = fm_bound<NW>(g, R, pbase, top, lds + fm_off_red(NM, nbin));
        const float low = bound.low;
        const bool part = low > 0.0f || top == top;
        int slot = FM_REFS;
        for (int c = c0; c < nchunk; c += cstep, ++slot) {
            if (slot == FM_REFS) {                               // references of the next FM_REFS chunks
                slot = 0;
                if (c != c0) __syncthreads();                    // the last ones have been read
                if (wv < FM_REFS) {
                    const int e = (c + wv * cstep) * WAVE + lane;
                    const MomRef r = mom_make_ref(g, xe + 6 * (size_t)min(e, g.E - 1), R);
                    const FmScale q = fm_scale(g, R, r, bound);
                    float* f = refs + wv * FM_FIELDS * WAVE + lane;
                    const float v[FM_FIELDS] = {r.D[0], r.D[1], r.D[2],  r.Dl[0], r.Dl[1],
                                                r.Dl[2], r.dh,  r.uc0,   r.n0,    q.scale,
                                                r.magic, q.inv, __int_as_float(r.kc - g.jclamp - jt)};
#pragma unroll
                    for (int i = 0; i < FM_FIELDS; ++i) f[i * WAVE] = v[i];
                }
                __syncthreads();
            }
            const float* rf = refs + slot * FM_FIELDS * WAVE;
            const float* rl = rf + lane;
            const float dh = rl[6 * WAVE], scale = rl[9 * WAVE];
            const int kb = __float_as_int(rl[12 * WAVE]);
            const bool valid = c * WAVE + lane < g.E;
            const bool finite = dh < 1e15f;
            // nothing to add: every window of the chunk misses the record, or the region is all zero
            const bool hit = valid && (!finite || (kb + rows > 0 && kb < K && bound.all != 0.0f));
            if (!__any(hit)) continue;
            const bool fixed = !__any(valid && scale == 0.0f);
            const float Dx = rl[0], Dy = rl[WAVE], Dz = rl[2 * WAVE], Dxl = rl[3 * WAVE], Dyl = rl[4 * WAVE];
            const float Dzl = rl[5 * WAVE], uc0 = rl[7 * WAVE], magic = rl[10 * WAVE], dh2 = dh * dh;
            unsigned off0 = (unsigned)lane * 4u + (unsigned)g.jclamp * (STR * 4u) - 0xC00000u * (STR * 4u);
            unsigned str = STR * 4u;
            asm volatile("" : "+v"(off0), "+v"(str));            // in vector registers: scalar operands halve the issue rate
            // row of a bin's sample kc - jt; FM_MAGIC << 8 is 0xC0000000
            unsigned eoff = (unsigned)(fm_off_edge(NM, nbin, jt) + lane + g.jclamp * WAVE) * 4u - 0xC0000000u;
            asm volatile("" : "+v"(eoff));
            const EdgeCoef xc = edge_coef(g, g.es);
            FmElem fe{};
            if (X) fe = fm_elem(g, xe + 6 * (size_t)min(c * WAVE + lane, g.E - 1));
            for (int z0 = 0; z0 < R.nk; z0 += FM_RZ) {
                const int nz = R.nk - z0;
                const float4 tz = axis[2 * FM_SIDE + z0 / FM_RZ];
                float zh, zl, ez[FM_RZ];
                double cz2 = 0.0, cx2 = 0.0;
                if (X) {
                    const double cz = fma((double)(R.k0 + z0) + 0.5 * (double)(min(nz, FM_RZ) - 1), fe.h, fe.z);
                    cz2 = cz * cz;
                    fm_column_n(g, nz, cz, ez);
                } else {
                    fm_axis(tz, Dz, Dzl, magic, zh, zl);
                    zl += rl[8 * WAVE];
                    fm_column_n(g, nz, tz, Dz, Dzl, ez);
                }
                int ix = -1;
                float xh = 0.0f, xl = 0.0f;
                for (int col = wv * mine; col < min((wv + 1) * mine, ncol); ++col) {
                    const int i = col / R.nj, j = col - i * R.nj;
                    const float* pc = pbase + (size_t)i * g.vsx + (size_t)j * g.vsy + z0;
                    float pv[FM_RZ];
                    if (nz >= FM_RZ) {
#pragma unroll
                        for (int k = 0; k < FM_RZ; ++k) pv[k] = pc[k];
                    } else {
#pragma unroll
                        for (int k = 0; k < FM_RZ; ++k) pv[k] = k < nz ? pc[min(k, nz - 1)] : 0.0f;
                    }
                    if (part) {                              // the column's voxels of this class, if any (kept in scalar registers)
                        bool any = false;
#pragma unroll
                        for (int k = 0; k < FM_RZ; ++k) {
                            const float v = fabsf(pv[k]);
                            const bool in = v >= low && !(v >= top);
                            pv[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(in ? pv[k] : 0.0f)));
                            any = any || in;
                        }
                        if (!__any(any)) continue;
                    }
                    FmCol cl;
                    if (X) {
                        if (i != ix) cx2 = fm_square_add(fma((double)(R.i0 + i), fe.h, fe.x), cz2);
                        ix = i;
                        cl = fm_col_f64(cx2, fma((double)(R.j0 + j), fe.h, fe.y), kb + g.jclamp + jt);
                    } else {
                        if (i != ix) {                           // the wavefront's columns run along y
                            ix = i;
                            fm_axis(axis[i], Dx, Dxl, magic, xh, xl);
                            xh += zh;
                            xl += zl;
                        }
                        float yh, yl;
                        fm_axis(axis[FM_SIDE + j], Dy, Dyl, magic, yh, yl);
                        cl = fm_col(xh + yh, xl + yl, dh, dh2, uc0);
                    }
                    if (fixed)
                        fm_column<NM, true, X>(g, xc, eoff, pv, ez, cl, scale, rlo, rhi, off0, str, reinterpret_cast<char*>(lds));
                    else
                        fm_column<NM, false, X>(g, xc, eoff, pv, ez, cl, 1.0f, rlo, rhi, off0, str, reinterpret_cast<char*>(lds));
                }
            }
            __syncthreads();
            if (fixed) {
                // [16 rows x 16 elements] tiles: wavefront w takes elements 16 (w & 3).. and row tiles w / 4,
                // w / 4 + NW / 4, .., two at a time (they share the D operand)
                const int eg = wv & 3, li = lane & 15, lk = lane >> 4;
                const int nq = (2 * jt + 16 + 3) / 4;
                const int* acc = reinterpret_cast<const int*>(lds) + 16 * eg + li;
                const float* db = dt + 2 * jt + FM_PAD + li - lk;          // D_n(jt + li - lk - 4 q)
                const int dl = fm_dlen(jt);
                const int e0 = 16 * eg + 4 * lk;
                const vf4 inv = *reinterpret_cast<const vf4*>(rf + 11 * WAVE + e0);
                const vf4 kbe = *reinterpret_cast<const vf4*>(rf + 12 * WAVE + e0);
                auto add_rows = [&](vf4 v, int r0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int e = c * WAVE + e0 + i, k = __float_as_int(kbe[i]) + r0 + li;
                        float x = v[i] * inv[i];
                        if (X && r0 + li < rows)
                            x = fmaf((float)reinterpret_cast<const int*>(edge)[(r0 + li) * WAVE + e0 + i], inv[i] * ies, x);
                        if (e < g.E && x != 0.0f && r0 + li < rows && k >= 0 && k < K)
                            atomicAdd(s + (size_t)e * K + k, (SumT)x);
                    }
                };
                for (int r0 = 16 * (wv >> 2); r0 < rows; r0 += 8 * NW) {
                    const int r1 = r0 + 4 * NW;
                    vf4 s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = {0.0f, 0.0f, 0.0f, 0.0f};
                    const int b0 = r0 - 2 * jt + lk;
                    // bins that do not exist read the zero bin
                    auto bin = [&](int b) { return acc + (b >= 0 && b < nbin ? b : nbin) * STR; };
                    if (r1 < rows) {
                        for (int q = 0; q < nq; ++q) {
                            const int* a0 = bin(b0 + 4 * q);
                            const int* a1 = bin(b0 + 4 * q + 4 * NW);
#pragma unroll
                            for (int n = 0; n < NM; ++n) {
                                const float bv = db[n * dl - 4 * q];
                                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32((float)a0[n * WAVE], bv, s0, 0, 0, 0);
                                s1 = __builtin_amdgcn_mfma_f32_16x16x4f32((float)a1[n * WAVE], bv, s1, 0, 0, 0);
                            }
                        }
                        add_rows(s1, r1);
                    } else {
                        for (int q = 0; q < nq; ++q) {
                            const int* a0 = bin(b0 + 4 * q);
#pragma unroll
                            for (int n = 0; n < NM; ++n)
                                s0 = __builtin_amdgcn_mfma_f32_16x16x4f32((float)a0[n * WAVE], db[n * dl - 4 * q], s0, 0, 0, 0);
                        }
                    }
                    add_rows(s0, r0);
                }
            } else {
                // FP32 sums: plain sums over the window rows, lane = element
                const float* acc = lds + lane;
                for (int r = wv; r < rows; r += NW) {
                    float v = X ? edge[r * WAVE + lane] * ies : 0.0f;
                    for (int b = max(r - 2 * jt, 0); b <= min(r, nbin - 1); ++b)
#pragma unroll
                        for (int n = 0; n < NM; ++n)
                            v = fmaf(acc[b * STR + n * WAVE], dt[n * fm_dlen(jt) + FM_PAD + r - b], v);
                    const int k = kb + r;
                    if (valid && v != 0.0f && k >= 0 && k < K) atomicAdd(s + (size_t)(c * WAVE + lane) * K + k, (SumT)v);
                }
            }
            __syncthreads();
            for (int i = tid; i < nbin * STR / 4; i += NW * WAVE)
                reinterpret_cast<float4*>(lds)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (X)
                for (int i = tid; i < rows * WAVE; i += NW * WAVE) edge[i] = 0.0f;
            __syncthreads();
        }        __syncthreads();                                     // the bound has been read
        more = low > 0.0f;
        top = low;
    }
}

template <int NM, int NW, int X, typename SumT>
__global__ __launch_bounds__(NW * WAVE) __attribute__((amdgpu_waves_per_eu(4))) void k_forward_mom(
    Geo g, MomCoef mc, int nslice, const float* __restrict__ p0, const float* __restrict__ xe, SumT* __restrict__ s) {
    extern __shared__ float lds[];
    const int dl = fm_dlen(g.jt);
    float* dt = lds + fm_off_dt(NM, g.nbin);
    for (int i = threadIdx.x; i < NM * dl; i += NW * WAVE)
        dt[i] = mom_coef(mc, i / dl, i % dl - FM_PAD - g.jt, g.jt);
    const int b = region_of_block(blockIdx.x, gridDim.x);
    fm_region<NM, NW, X, SumT>(g, b / nslice, b % nslice, nslice, p0, xe, s, lds);
}

// ------------------------------------------------------------------------------------------
// adjoint: dL/dp0 and/or per-region element-gradient partials
// ------------------------------------------------------------------------------------------
// Moments of one (voxel, element) pair over its sample window, with r = dL/ds:
//   M0 = sum r e0 H^j G_j,  M1 = sum (j delta) r e0 H^j G_j (sign by side),  M2 = sum (j delta)^2 ...
// so that sum r u e = u0 M0 - M1 and sum r u^2 e = u0^2 M0 - 2 u0 M1 + M2.
struct Moments {
    float M0, M1, M2;
};

template <int JT, bool EXACT, bool WANT_M2>
__device__ __forceinline__ Moments adj_moments(const Geo& g, const VConst<JT, WANT_M2>& c, const Pair& p,
                                               const float* lane_rows) {
    const float* lo = lane_rows + p.j0 * WAVE;
    float rw[2 * JT + 1];                  // the window's residuals, all reads issued first
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) rw[i] = lo[i * WAVE];
    // residual at row j0 + jj, zero outside the window
    auto inwin = [&](int jj) -> float {
        const int a = jj < 0 ? -jj : jj;
        float rv = rw[JT + jj];
        if (EXACT && a == JT) {
            rv = (jj > 0 ? p.u0 >= c.edge : p.u0 <= c.nedge) ? rv : 0.0f;
        } else if (!EXACT && a > JT - GEN_STEP) {
            const float uj = fmaf(-(float)jj, c.dlt_h, p.u0);
            rv = fabsf(uj) <= c.tsig ? rv : 0.0f;
        }
        return rv;
    };
    Moments m;
    if constexpr (!WANT_M2) {
        // Both sums by Horner's rule in H (rows j0 + j, j >= 0) and in 1/H (rows j0 - j, j >= 1):
        // P(H) = sum Gamma_j r_j H^j, Q(1/H) = sum Gamma_j r_-j H^-(j-1), with their derivatives,
        // give sum Gamma r H^jj = P + Q/H and sum jj Gamma r H^jj = H P' - (Q + Q'/H)/H.
        float pf = c.gam[JT] * inwin(JT), df = 0.0f;
#pragma unroll
        for (int j = JT - 1; j >= 0; --j) {
            df = fmaf(df, p.H, pf);
            pf = fmaf(pf, p.H, j == 0 ? inwin(0) : c.gam[j] * inwin(j));
        }
        float qb = c.gam[JT] * inwin(-JT), db = 0.0f;
#pragma unroll
        for (int j = JT - 1; j >= 1; --j) {
            db = fmaf(db, p.Hi, qb);
            qb = fmaf(qb, p.Hi, c.gam[j] * inwin(-j));
        }
        m.M0 = p.e0 * fmaf(p.Hi, qb, pf);
        const float gb = p.Hi * fmaf(p.Hi, db, qb);
        m.M1 = (c.dlt_h * p.e0) * fmaf(p.H, df, -gb);
        m.M2 = 0.0f;
        return m;
    }
    float Rf = p.e0, Rb = p.e0;
    m.M0 = rw[JT] * Rf;
    m.M1 = 0.0f;
    m.M2 = 0.0f;
#pragma unroll
    for (int jj = 1; jj <= JT; ++jj) {
        Rf *= p.H;
        Rb *= p.Hi;
        const float rf = inwin(jj), rb = inwin(-jj);
        const float tb = rb * Rb;
        const float sp = fmaf(rf, Rf, tb), sm = fmaf(rf, Rf, -tb);
        m.M0 = fmaf(c.gam[jj], sp, m.M0);
        m.M1 = fmaf(c.jdg[jj], sm, m.M1);
        if (WANT_M2) m.M2 = fmaf(c.jjdg[jj], sp, m.M2);
    }
    return m;
}

// dL/dp0 part of one pair with the Gaussian referenced to the region's sample kc instead of
// the pair's centre.  Row m (from kc) of the window has weight exp(-(uc - m delta)^2 / 2 s^2)
// = E_c Hc^m Gamma_m, with uc = d - kc delta, Hc = exp(uc delta / s^2), E_c = exp(-uc^2 / 2 s^2);
// Gamma_m depends on the row alone and was multiplied into the staged residuals (with the
// lane's power-of-two scale), so that over the window's rows i = 0..2 JT (m = mlow + i)
//   A = sum r phi / K = E_c Hc^mlow [ (uc - mlow delta) S0 - delta S1 ],
//   S0 = sum c_i Hc^i, S1 = sum i c_i Hc^i,
// by Horner's rule in Hc: two FMAs per sample and two exponentials per pair.  The host admits
// this form only where every factor stays inside the FP32 range.  Returns A / (lane scale).
template <int JT>
__device__ __forceinline__ float adj_rowref(const VConst<JT, false>& c, const Ref& ref, float4 o,
                                            const float* lane_rows, float& hr) {
    const Dist q = pair_dist(ref, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    const float* lo = lane_rows + (int)jf * WAVE;
    float rw[2 * JT + 1];
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) rw[i] = lo[i * WAVE];
    // the outermost rows j0 -+ JT are inside the window iff u0 <= -edge / u0 >= edge
    rw[0] = u0 <= c.nedge ? rw[0] : 0.0f;
    rw[2 * JT] = u0 >= c.edge ? rw[2 * JT] : 0.0f;
    const float mlow = jf - (float)JT;
    const float xa = c.alpha * q.uc;
    const float Hc = __builtin_amdgcn_exp2f(xa);
    const float pref = __builtin_amdgcn_exp2f(fmaf(c.kappa * q.uc, q.uc, xa * mlow));
    float p = rw[2 * JT], dv = 0.0f;
#pragma unroll
    for (int i = 2 * JT - 1; i >= 0; --i) {
        dv = fmaf(dv, Hc, p);
        p = fmaf(p, Hc, rw[i]);
    }
    const float ulow = residual(c, q.uc, mlow);               // uc - mlow delta
    hr = q.hr;
    return pref * fmaf(ulow, p, -c.dlt_h * (Hc * dv));
}

// Window sums of one pair for a profile other than the Gaussian: A = sum r phi(u) and,
// with WANT_B, B = sum r phi'(u), each sample with its own window test.
struct VarSums {
    float A, B, hr;
};

template <int KT, bool WANT_B>
__device__ __forceinline__ VarSums adj_var(const Geo& g, const VConst<0, WANT_B>& c, const Ref& ref, float4 o,
                                           const float* centre) {
    const Dist q = pair_dist(ref, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    const float* lo = centre + (int)jf * WAVE;
    const int jw = g.jwin;
    VarSums v{0.0f, 0.0f, q.hr};
#pragma unroll 4
    for (int jj = -jw; jj <= jw; ++jj) {
        const float u = residual(c, u0, (float)jj);
        const float x = fabsf(u);
        const float rv = x <= c.tsig ? lo[jj * WAVE] : 0.0f;
        const float k = prof<KT>(g, x);
        v.A = fmaf(rv * u, k, v.A);
        if (WANT_B) v.B = fmaf(rv, dprof<KT>(g, x, k), v.B);
    }
    return v;
}

// Window sums of one pair for the exponential profile, by the leg factorisation of
// fwd_pair_exp: per leg S0 = sum r G_j and S1 = sum r j delta G_j (two FMAs per sample), then
//   A = exp(u0/w) (u0 S0f - S1f) + exp(-u0/w) (u0 S0b + S1b) + r_0 u0 K(|u0|),
//   B = exp(u0/w) ((1 + u0/w) S0f - S1f/w) + exp(-u0/w) ((1 - u0/w) S0b - S1b/w)
//       + r_0 K(|u0|) (1 - |u0|/w),
// from phi'(u) = K(|u|) (1 - |u|/w).
template <int JT, bool WANT_B>
__device__ __forceinline__ VarSums adj_exp(const Geo& g, const VConst<JT, WANT_B>& c, const Ref& ref, float4 o,
                                           const float* lane_rows) {
    const Dist q = pair_dist(ref, o);
    const float jf = centre_step(c, q.uc);
    const float u0 = residual(c, q.uc, jf);
    const float* lo = lane_rows + (int)jf * WAVE;
    float rw[2 * JT + 1];
#pragma unroll
    for (int i = 0; i <= 2 * JT; ++i) rw[i] = lo[i * WAVE];
    float s0f = 0.0f, s1f = 0.0f, s0b = 0.0f, s1b = 0.0f;
#pragma unroll
    for (int jj = 1; jj <= JT; ++jj) {
        float rf = rw[JT + jj], rb = rw[JT - jj];
        if (jj > JT - EXP_STEP) {
            const float uf = fmaf(-(float)jj, c.dlt_h, u0), ub = fmaf((float)jj, c.dlt_h, u0);
            rf = fabsf(uf) <= c.tsig ? rf : 0.0f;
            rb = fabsf(ub) <= c.tsig ? rb : 0.0f;
        }
        s0f = fmaf(rf, c.gam[jj], s0f);
        s1f = fmaf(rf, c.jdg[jj], s1f);
        s0b = fmaf(rb, c.gam[jj], s0b);
        s1b = fmaf(rb, c.jdg[jj], s1b);
    }
    const float x0 = u0 * g.kexp;                         // -u0/w in log2 units
    const float Ef = __builtin_amdgcn_exp2f(-x0), Eb = __builtin_amdgcn_exp2f(x0);
    const float a0 = fabsf(u0);
    const float K0 = __builtin_amdgcn_exp2f(a0 * g.kexp);
    VarSums v;
    v.hr = q.hr;
    v.A = fmaf(Ef, fmaf(u0, s0f, -s1f), fmaf(Eb, fmaf(u0, s0b, s1b), rw[JT] * u0 * K0));
    if (WANT_B) {
        const float iw = g.kinv_w, t = u0 * iw;
        const float bf = fmaf(1.0f + t, s0f, -s1f * iw), bb = fmaf(1.0f - t, s0b, -s1b * iw);
        v.B = fmaf(Ef, bf, fmaf(Eb, bb, rw[JT] * K0 * fmaf(-a0, iw, 1.0f)));
    } else {
        v.B = 0.0f;
    }
    return v;
}

// The adjoint work of one region.  dL/dp0 of each voxel is summed over the element
// chunks of the region in LDS (`gsum`, one array of g.nvpad values per wavefront, then
// across wavefronts) and written once; element gradients go to pose_part[reg][e].
// Contains workgroup barriers: every thread of the workgroup must call it.
template <int JT, bool EXACT, bool WANT_P0, bool WANT_POSE, int KT = RA_KERNEL_GAUSSIAN, bool RS = false>
__device__ __forceinline__ void adjoint_region(const Geo& g, int reg, const float* __restrict__ p0,
                                               const float* __restrict__ xe, const float4* __restrict__ vtab,
                                               const int4* __restrict__ itab, const float* __restrict__ r,
                                               float* __restrict__ grad_p0, int accumulate,
                                               double* __restrict__ pose_part, float* rows, float* gsum_all,
                                               int lane, int wave) {
    float* gsum = gsum_all + (size_t)wave * g.nvpad;
    if (WANT_P0)
        for (int t = lane; t < g.nvpad; t += WAVE) gsum[t] = 0.0f;

    const Region R = region_info(g, reg);
    const float* pbase = p0 ? p0 + (size_t)R.i0 * g.vsx + (size_t)R.j0 * g.vsy + R.k0 : nullptr;
    const int nchunk = (g.E + WAVE - 1) / WAVE;
    VConst<JT, WANT_POSE> cst;
    load_vconst<false>(cst, g);
    const bool interior = R.ni == g.rx && R.nj == g.ry && R.nk == g.rz && (g.rz & 3) == 0;

    for (int c = wave; c < nchunk; c += WAVES) {
        const int e = c * WAVE + lane;
        const bool valid = e < g.E;
        const Ref ref = make_ref(g, xe, valid ? e : 0, R);
        int rs_exp = 0;                    // row-referenced form: the lane's window scale 2^-rs_exp
        {   // stage this lane's window of dL/ds in its private row (zeros past the last element
            // and outside [0, K)); loads go out 16 at a time, clamped into the row, before any
            // is waited for
            const float* rrow = r + (size_t)(valid ? e : 0) * g.K;
            float vmax = 0.0f;
            for (int ix0 = 0; ix0 < g.L; ix0 += 16) {
                float v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int k = min(max(ref.kbase + ix0 + q, 0), g.K - 1);
                    v[q] = rrow[k];
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int ix = ix0 + q, k = ref.kbase + ix;
                    const float x = (valid && k >= 0 && k < g.K) ? v[q] : 0.0f;
                    if (ix < g.L) rows[ix * WAVE + lane] = x;
                    if (RS) vmax = fmaxf(vmax, fabsf(x));
                }
            }
            if constexpr (RS) {
                // row-referenced form: scale the lane's window by a power of two (largest value in
                // [1/2, 1)) and by Gamma of each row's offset from kc
                rs_exp = vmax > 0.0f ? __builtin_amdgcn_frexp_expf(vmax) : 0;
                for (int ix0 = 0; ix0 < g.L; ix0 += 16) {      // 16 rows in flight
                    float v[16];
#pragma unroll
                    for (int q = 0; q < 16; ++q)
                        if (ix0 + q < g.L) v[q] = rows[(ix0 + q) * WAVE + lane];
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int ix = ix0 + q, m = ix - g.kmargin;
                        if (ix < g.L)
                            rows[ix * WAVE + lane] = __builtin_amdgcn_ldexpf(v[q], -rs_exp) * g.gamr[m < 0 ? -m : m];
                    }
                }
            }
        }
        const float* lane_rows = rows + lane + (g.kmargin - JT) * WAVE;
        double gx = 0.0, gy = 0.0, gz = 0.0;
        for (int t = 0; t < g.nvpad; t += 4) {
            float G[4];
            float fx = 0.0f, fy = 0.0f, fz = 0.0f;     // four pairs in FP32, then into FP64
            float pv4[4];
            int at[4] = {t, t + 1, t + 2, t + 3};
            if (WANT_POSE) {
                if (interior) {                          // four consecutive voxels along z
                    const int off = itab[t].w;
#pragma unroll
                    for (int q = 0; q < 4; ++q) pv4[q] = pbase[off + q];
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int4 ix = itab[t + q];
                        const bool inside = ix.x < R.ni && ix.y < R.nj && ix.z < R.nk;
                        const float v = pbase[inside ? ix.w : 0];
                        pv4[q] = inside ? v : 0.0f;
                        at[q] = inside ? t + q : 0;          // as in the forward
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 o = vtab[at[q]];
                float A, B = 0.0f, hr;             // sum_k r phi(u), sum_k r phi'(u), 1/(2d)
                if constexpr (RS) {
                    A = __builtin_amdgcn_ldexpf(adj_rowref<JT>(cst, ref, o, lane_rows, hr), rs_exp);
                } else if constexpr (KT == RA_KERNEL_GAUSSIAN) {
                    const Pair p = make_pair(cst, ref, o);
                    const Moments m = adj_moments<JT, EXACT, WANT_POSE>(g, cst, p, lane_rows);
                    A = fmaf(p.u0, m.M0, -m.M1);                                       // sum r u e
                    if (WANT_POSE) {
                        const float Su2 = fmaf(p.u0, fmaf(p.u0, m.M0, -2.0f * m.M1), m.M2);  // sum r u^2 e
                        B = fmaf(-Su2, cst.inv_s2, m.M0);
                    }
                    hr = p.hr;
                } else {
                    VarSums v;
                    if constexpr (KT == RA_KERNEL_EXPONENTIAL)
                        v = adj_exp<JT, WANT_POSE>(g, cst, ref, o, lane_rows);
                    else
                        v = adj_var<KT, WANT_POSE>(g, cst, ref, o, lane_rows);
                    A = v.A;
                    B = v.B;
                    hr = v.hr;
                }
                G[q] = A * hr;                     // sum_k r phi / (2d); 0 for lanes past the last element
                if (WANT_POSE) {
                    const float pv = pv4[q];
                    const float twohr = 2.0f * hr;                                          // 1/d
                    // p0 (B/(2d) - A/(2d^2)) / d times (x_e - x_v) = -(D + o)
                    const float coef = -pv * hr * twohr * fmaf(-twohr, A, B);
                    fx = fmaf(coef, ref.Dx + o.x, fx);
                    fy = fmaf(coef, ref.Dy + o.y, fy);
                    fz = fmaf(coef, ref.Dz + o.z, fz);
                }
            }
            if (WANT_POSE) {
                gx += (double)fx;
                gy += (double)fy;
                gz += (double)fz;
            }
            if (WANT_P0) {
#pragma unroll
                for (int q = 0; q < 4; ++q) G[q] = wave_sum_to_63(G[q]);
                if (lane == WAVE - 1) {
                    float4* dst = reinterpret_cast<float4*>(gsum + t);
                    float4 a = *dst;
                    a.x += G[0]; a.y += G[1]; a.z += G[2]; a.w += G[3];
                    *dst = a;
                }
            }
        }
        if (WANT_POSE && valid) {
            double* out = pose_part + ((size_t)reg * g.E + e) * 3;
            out[0] = gx; out[1] = gy; out[2] = gz;
        }
    }
    if (WANT_P0) {
        __syncthreads();
        float* gbase = grad_p0 + (size_t)R.i0 * g.gsx + (size_t)R.j0 * g.gsy + R.k0;
        for (int t = threadIdx.x; t < g.nvpad; t += BLOCK) {
            const int4 ix = itab[t];
            if (!(ix.x < R.ni && ix.y < R.nj && ix.z < R.nk)) continue;
            const float v = gsum_all[t] + gsum_all[g.nvpad + t] + gsum_all[2 * g.nvpad + t] +
                            gsum_all[3 * g.nvpad + t];
            float* dst = gbase + ix.x * g.gsx + ix.y * g.gsy + ix.z;
            *dst = accumulate ? *dst + v : v;
        }
        __syncthreads();
    }
}

template <int JT, bool EXACT, bool WANT_P0, bool WANT_POSE, int KT = RA_KERNEL_GAUSSIAN, bool RS = false>
__global__ __launch_bounds__(BLOCK) void k_adjoint(Geo g, const float* __restrict__ p0,
                                                   const float* __restrict__ xe,
                                                   const float4* __restrict__ vtab,
                                                   const int4* __restrict__ itab,
                                                   const float* __restrict__ r,
                                                   float* __restrict__ grad_p0, int accumulate,
                                                   double* __restrict__ pose_part) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    float* rows = lds + (size_t)wave * g.L * WAVE;
    float* gsum = lds + (size_t)WAVES * g.L * WAVE;
    adjoint_region<JT, EXACT, WANT_P0, WANT_POSE, KT, RS>(g, region_of_block(blockIdx.x, g.nreg), p0, xe, vtab,
                                                           itab, r, grad_p0, accumulate, pose_part, rows, gsum,
                                                           lane, wave);
}

// ------------------------------------------------------------------------------------------
// adjoints in moment form (Gaussian, exponential and power-law profiles)
// ------------------------------------------------------------------------------------------
// The transpose of the forward's moment form: the window sum of a pair with nearest sample kc and offset t is
//   sum_j r[kc + j] phi((t/2 - j) delta) = delta sum_n t^n Q_n[kc],  Q_n[k] = sum_j r[k + j] D_n(j) / delta,
// so a pair costs its distance, two LDS reads and Horner's rule instead of a pass over its 2 JT + 1 window
// rows.  Rows are taken whole about kc, so a term with T sigma < |u| <= (JT + 1/2) delta (at most psi(T) ~ 1e-7
// of the peak at T = 6) is added where the exact window leaves it out.
//
// The table built once per call from dL/ds: rows
// Q[e][kk][n] = sum_{|j| <= jt} r[e][k + j] D_n(j) / delta for kk in [0, K + 2 jt), k = kk - jt, with dL/ds
// zero outside [0, K); each row is NQ float4 (4 terms each).  One zero row follows the last element's
// rows.  The window's two legs are taken together, since D_n(-j) = (-1)^(n+1) D_n(j): 10 VALU for two
// samples.  A row of dL/ds is staged in LDS; the bound is writing the table (275 MB on the sweep: 0.118 ms
// with a thread's 25 taps read from memory, 0.069 ms so).
constexpr int MT_ROWS = 256;          // table rows per workgroup

template <int NQ>
__global__ __launch_bounds__(MT_ROWS) void k_moment_series(int E, int K, int jt, MomCoef mc, const float* __restrict__ r,
                                                           float4* __restrict__ q) {
    __shared__ float row[MT_ROWS + 2 * JMAX];
    const int kq = K + 2 * jt, per = (kq + MT_ROWS - 1) / MT_ROWS;
    const int e = blockIdx.x / per, kk0 = (blockIdx.x - e * per) * MT_ROWS;
    const float* re = r + (size_t)e * K;
    for (int i = threadIdx.x; i < MT_ROWS + 2 * jt; i += MT_ROWS) {
        const int k = kk0 - 2 * jt + i;                      // row[i] = r[kk0 - 2 jt + i]
        row[i] = k >= 0 && k < K ? re[k] : 0.0f;
    }
    __syncthreads();
    const int kk = kk0 + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < NQ) q[(size_t)E * kq * NQ + threadIdx.x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (kk >= kq) return;
    const float* w = row + threadIdx.x + jt;                 // r at the row's own sample
    float acc[4 * NQ];
#pragma unroll
    for (int n = 0; n < 4 * NQ; ++n) acc[n] = w[0] * mc.d[n];
    for (int j = 1; j <= jt; ++j) {
        const float a = w[j], b = w[-j], sum = a + b, dif = a - b;
#pragma unroll
        for (int n = 0; n < 4 * NQ; ++n) acc[n] = fmaf(n & 1 ? sum : dif, mc.d[j * MOM_MAX + n], acc[n]);
    }
    float4* out = q + NQ * ((size_t)e * kq + kk);
#pragma unroll
    for (int i = 0; i < NQ; ++i) out[i] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
}

// Adjoints from those tables: dL/dp0 (WANT_P0) and/or the element gradients (WANT_POSE) of regions reg0 ..
// reg1 - 1.  The workgroup's 16 wavefronts take the element chunks together, each of them CPW columns of 8
// voxels; lane = element.  The chunk's table rows for the region's nbin centre samples are in LDS,
// [bin][half][lane] float4, so that a wavefront reads one half at 1 KiB contiguous; they arrive by direct
// loads to LDS, those of the next chunk while this one's voxels run where two windows fit (nbuf 2).  A pair
// costs its distance and offset as in the forward, two LDS reads and Horner's rule.  Each lane keeps the sum
// over its chunks' elements of every voxel it visits in a register, and the 64 lanes meet once, after the
// last chunk.  With WANT_POSE the sum runs together with its derivative in t, P and P':
//   dL/dx_e = - sum_v p0 (2 / delta) / d^2 (P' - P / d) (D + o), d and o in units;
// the terms of four voxels add in FP32, those sums in FP64, the wavefronts' sums of a chunk meet in LDS (in the
// window just used) in wavefront order, and a workgroup adds its regions into one row of partials in their
// order (or each into its own row, row_step apart), so no result depends on timing.
// Bounds: VALU.  About 19 instructions per pair for dL/dp0 and 36 per column of 8 pairs, 34 per pair with
// the element gradients too.  On this chip FP32 adds, multiplies and FMAs of vector registers issue at up to
// 1.5 a clock and CU, those with a scalar operand, med3, conversions and shifts at 0.9, v_rsq_f32 at 0.5: the
// sum over a pair comes to 25 cycles, 28 measured (sweep of 128x128x64 voxels and 8192 elements: 7.14 ms
// before, with 35 instructions per pair, 6.5 ms now; with the element gradients 12.4 -> 10.4 ms).
constexpr int AM_FIELDS = 11;         // floats of a reference
constexpr int am_nq(int nm) { return (nm + 3) / 4; }         // float4 per table row
// float4 per window: the table rows (at least what the wavefronts' partials need), then the samples of dL/ds that
// the profiles with edge terms read, [row][lane] (xrows of them, 0 for the Gaussian)
constexpr int am_rows(int nbin, int nq) { return nbin * nq * WAVE > 1536 ? nbin * nq * WAVE : 1536; }
constexpr int am_win(int nbin, int nq, int xrows) { return am_rows(nbin, nq) + xrows * WAVE / 4; }
constexpr size_t am_off_axis(int nbin, int nq, int xrows, int nbuf) {
    return (size_t)nbuf * am_win(nbin, nq, xrows) * 4 + AM_REFS * AM_FIELDS * WAVE;
}
constexpr size_t am_lds(int nbin, int nq, int xrows, int nbuf) {
    return (am_off_axis(nbin, nq, xrows, nbuf) + 3 * FM_SIDE * 4) * sizeof(float);
}

template <int NM, int CPW, bool WANT_P0, bool WANT_POSE, int X>
__device__ __forceinline__ void am_regions(const Geo& g, int reg0, int reg1, int nbuf, const float* __restrict__ p0,
                                           const float* __restrict__ xe, const float4* __restrict__ q,
                                           const float* __restrict__ r, float* __restrict__ grad_p0, int accumulate,
                                           double* __restrict__ pose_part, size_t row_step, float* lds) {
    constexpr int NQ = am_nq(NM);
    // With edge terms (compiled for 4 columns a wavefront alone) the columns go round the wavefronts, so that regions of 16
    // or 32 columns occupy all of them too (exponential, 40^3 voxels of 0.3 mm, 256 elements: 352 us with 4 of 16 at work)
    constexpr bool STRIDED = X != 0;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int nbin = g.nbin, jt = g.jt, kq = g.K + 2 * jt;
    const int xrows = X ? nbin + 2 * jt : 0;
    const int win = am_win(nbin, NQ, xrows);
    float4* qw = reinterpret_cast<float4*>(lds);
    float* refs = lds + (size_t)nbuf * win * 4;              // [slot][field][lane]
    float4* axis = reinterpret_cast<float4*>(lds + am_off_axis(nbin, NQ, xrows, nbuf));
    const int nchunk = (g.E + WAVE - 1) / WAVE;
    const int iters = (reg1 - reg0) * nchunk;                // (region, chunk) pairs, one after the other

    auto make_refs = [&](int it) {                           // by one wavefront
        const int rr = it / nchunk, c = it - rr * nchunk;
        const MomRef r = mom_make_ref(g, xe + 6 * (size_t)min(c * WAVE + lane, g.E - 1), region_info(g, reg0 + rr));
        float* f = refs + (it % AM_REFS) * AM_FIELDS * WAVE + lane;
        const float v[AM_FIELDS] = {r.D[0], r.D[1], r.D[2], r.Dl[0], r.Dl[1], r.Dl[2],
                                    r.dh,   r.uc0,  r.n0,   r.magic, __int_as_float(r.kc)};
#pragma unroll
        for (int i = 0; i < AM_FIELDS; ++i) f[i * WAVE] = v[i];
    };
    // whether any window of the chunk meets the record (an element that is not finite counts)
    auto hits = [&](int it) -> bool {
        const float* rl = refs + (it % AM_REFS) * AM_FIELDS * WAVE + lane;
        const int b0 = __float_as_int(rl[10 * WAVE]) - g.jclamp + jt;   // table row of bin 0
        const bool finite = rl[6 * WAVE] < 1e15f;
        return __any((it % nchunk) * WAVE + lane < g.E && (!finite || (b0 < kq && b0 + nbin > 0)));
    };
    // issue the loads of this wavefront's bins
    auto fetch = [&](int it) {
        const float* rl = refs + (it % AM_REFS) * AM_FIELDS * WAVE + lane;
        const int b0 = __float_as_int(rl[10 * WAVE]) - g.jclamp + jt;
        const int e = (it % nchunk) * WAVE + lane;
        const float4* qe = q + (size_t)min(e, g.E - 1) * kq * NQ;
        const float4* zrow = q + (size_t)g.E * kq * NQ;      // what does not exist reads the zero row
        float4* dst = qw + (nbuf == 2 ? (it & 1) : 0) * win;
        typedef const __attribute__((address_space(1))) void* gptr;
        typedef __attribute__((address_space(3))) void* lptr;
        for (int b = wv; b < nbin; b += AM_WAVES) {
            const int kk = b0 + b;
            const float4* src = e < g.E && kk >= 0 && kk < kq ? qe + (size_t)kk * NQ : zrow;
#pragma unroll
            for (int i = 0; i < NQ; ++i)
                __builtin_amdgcn_global_load_lds((gptr)(src + i), (lptr)(dst + (b * NQ + i) * WAVE), 16, 0, 0);
        }
        if (X) {                                             // row x of the samples is kc - jclamp - jt + x
            const float* re = r + (size_t)min(e, g.E - 1) * g.K;
            float* rdst = reinterpret_cast<float*>(dst + am_rows(nbin, NQ));
            for (int x = wv; x < xrows; x += AM_WAVES) {
                const int k = b0 - 2 * jt + x;
                const float* src = e < g.E && k >= 0 && k < g.K ? re + k : reinterpret_cast<const float*>(zrow);
                __builtin_amdgcn_global_load_lds((gptr)src, (lptr)(rdst + x * WAVE), 4, 0, 0);
            }
        }
    };

    fm_axis_table(g, g.rz, tid, axis);
    if (wv == 0 && iters > 0) make_refs(0);
    if (wv == 1 && iters > 1) make_refs(1);
    __syncthreads();
    if (nbuf == 2 && iters > 0 && hits(0)) fetch(0);

    float acc[WANT_P0 ? CPW * FM_RZ : 1];
#pragma unroll
    for (int i = 0; i < (WANT_P0 ? CPW * FM_RZ : 1); ++i) acc[i] = 0.0f;
    const float rlo = FM_MAGIC - 2.0f * g.jclampf, rhi = FM_MAGIC + 2.0f * g.jclampf;
    int reg = reg0, c = 0;
    Region R = region_info(g, reg0);

    for (int it = 0; it < iters; ++it) {
        const bool hit = hits(it);
        if (nbuf == 1) {
            __syncthreads();                                 // the window has been read
            if (hit) fetch(it);
        }
        __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0): this wavefront's loads to LDS have landed
        __syncthreads();                                     // and everyone's; the other window has been read
        if (wv == (it & (AM_WAVES - 1)) && it + 2 < iters) make_refs(it + 2);
        if (nbuf == 2 && it + 1 < iters && hits(it + 1)) fetch(it + 1);
        float4* const used = qw + (nbuf == 2 ? (it & 1) : 0) * win;
        const int ncol = R.ni * R.nj;
        double Sx = 0.0, Sy = 0.0, Sz = 0.0;                 // sum over this wavefront's voxels of f (D + o)
        const float* rl = refs + (it % AM_REFS) * AM_FIELDS * WAVE + lane;
        if (hit) {
            const float Dx = rl[0], Dy = rl[WAVE], Dz = rl[2 * WAVE], Dxl = rl[3 * WAVE], Dyl = rl[4 * WAVE];
            const float Dzl = rl[5 * WAVE];
            const float dh = rl[6 * WAVE], uc0 = rl[7 * WAVE], magic = rl[9 * WAVE], dh2 = dh * dh;
            const float* pbase = WANT_POSE ? p0 + (size_t)R.i0 * g.vsx + (size_t)R.j0 * g.vsy + R.k0 : nullptr;
            const float4 tz = axis[2 * FM_SIDE + (R.nk < g.rz)];
            float zh, zl, ez[FM_RZ];
            FmElem fe{};
            double cz2 = 0.0, cx2 = 0.0;
            if (X) {                                         // as the forward, to the last bit
                fe = fm_elem(g, xe + 6 * (size_t)min(c * WAVE + lane, g.E - 1));
                const double cz = fma((double)R.k0 + 0.5 * (double)(R.nk - 1), fe.h, fe.z);
                cz2 = cz * cz;
                fm_column_n(g, R.nk, cz, ez);
            } else {
                fm_axis(tz, Dz, Dzl, magic, zh, zl);
                zl += rl[8 * WAVE];
                fm_column_n(g, R.nk, tz, Dz, Dzl, ez);
            }
            const float zmid = 0.5f * (float)(FM_RZ - R.nk);     // a whole column's middle from this one's, in voxels
            // a bin's table row, from the low 24 bits of rm, 0xC00000 + (centre sample offset).  Kept in vector
            // registers, so that a pair's address is one instruction without scalar operands
            constexpr unsigned STEP = NQ * WAVE * 16u;
            const unsigned wbase = (nbuf == 2 ? (it & 1) : 0) * win * 16u;
            unsigned off0 = (unsigned)lane * 16u + (NQ == 2 ? (unsigned)g.jclamp : (unsigned)g.jclamp - 0xC00000u) * STEP + wbase, step = STEP;
            // row of a bin's sample kc - jt among the samples of dL/ds; FM_MAGIC << 8 is 0xC0000000
            unsigned xoff = wbase + (unsigned)am_rows(nbin, NQ) * 16u + (unsigned)(lane + g.jclamp * WAVE) * 4u - 0xC0000000u;
            asm volatile("" : "+v"(off0), "+v"(step), "+v"(xoff));
            const EdgeCoef xc = edge_coef(g, 1.0f);
            int ix = -1;
            float xh = 0.0f, xl = 0.0f, ox = 0.0f;
#pragma unroll
            for (int cc = 0; cc < CPW; ++cc) {
                const int col = STRIDED ? cc * AM_WAVES + wv : wv * CPW + cc;
                if (col >= ncol) continue;
                const int i = col / R.nj, j = col - i * R.nj;
                const float4 ty = axis[FM_SIDE + j];
                FmCol cl;
                if (i != ix) {                               // a wavefront's columns run along y
                    const float4 tx = axis[i];
                    ox = tx.x;
                    if (X) {
                        cx2 = fm_square_add(fma((double)(R.i0 + i), fe.h, fe.x), cz2);
                    } else {
                        fm_axis(tx, Dx, Dxl, magic, xh, xl);
                        xh += zh;
                        xl += zl;
                    }
                    ix = i;
                }
                if (X) {
                    cl = fm_col_f64(cx2, fma((double)(R.j0 + j), fe.h, fe.y), __float_as_int(rl[10 * WAVE]));
                } else {
                    float yh, yl;
                    fm_axis(ty, Dy, Dyl, magic, yh, yl);
                    cl = fm_col(xh + yh, xl + yl, dh, dh2, uc0);
                }
                const float dc2 = cl.dc * cl.dc, hdc = 0.5f * cl.dc;
                float pv[FM_RZ];
                if (WANT_POSE) {
                    const float* pc = pbase + (size_t)i * g.vsx + (size_t)j * g.vsy;
                    if (R.nk == FM_RZ) {
#pragma unroll
                        for (int k = 0; k < FM_RZ; ++k) pv[k] = pc[k];
                    } else {
#pragma unroll
                        for (int k = 0; k < FM_RZ; ++k) pv[k] = k < R.nk ? pc[min(k, R.nk - 1)] : 0.0f;
                    }
                }
                float c0[2] = {0.0f, 0.0f}, cz[2] = {0.0f, 0.0f};         // of four voxels each
#pragma unroll
                for (int k = 0; k < FM_RZ; ++k) {
                    const FmPair p = fm_pair(cl, dc2, hdc, ez[k], rlo, rhi);
                    const unsigned off = NQ == 2 ? (__float_as_uint(p.rm) << 11) + off0
                                                 : __umul24(__float_as_uint(p.rm), step) + off0;
                    const vf4* row = reinterpret_cast<const vf4*>(reinterpret_cast<const char*>(lds) + off);
                    vf4 m4[NQ];
#pragma unroll
                    for (int i = 0; i < NQ; ++i) m4[i] = row[i * WAVE];
                    float h = m4[(NM - 1) / 4][(NM - 1) % 4], dd = 0.0f;
#pragma unroll
                    for (int n = NM - 2; n >= 0; --n) {
                        if (WANT_POSE) dd = n == NM - 2 ? h : fmaf(dd, p.t, h);
                        h = fmaf(h, p.t, m4[n / 4][n % 4]);
                    }
                    if (X) {                                 // an outermost sample and the centre
                        const char* rx = reinterpret_cast<const char*>(lds) + ((__float_as_uint(p.rm) << 8) + xoff);
                        const Edge e = edge_phi(xc, p.t);
                        float rv = *reinterpret_cast<const float*>(rx + e.row);
                        rv = e.v != 0.0f ? rv : 0.0f;        // dL/ds outside the window may be anything
                        h = fmaf(rv, e.v, h);
                        if (WANT_POSE) dd = fmaf(rv, e.d, dd);
                        if (X == 2) {                        // exp2(kx |t|) = exp(-|t| delta / 2w)
                            const float r0 = 0.5f * *reinterpret_cast<const float*>(rx + xc.far / 2u), ta = fabsf(p.t);
                            const float x0 = r0 * __builtin_amdgcn_exp2f(g.kx * ta);
                            h = fmaf(x0, p.t, h);
                            if (WANT_POSE) dd = fmaf(x0, fmaf(0.6931471805599453f * g.kx, ta, 1.0f), dd);
                        }
                    }
                    if (WANT_P0) acc[cc * FM_RZ + k] = fmaf(h, p.rs, acc[cc * FM_RZ + k]);
                    if (WANT_POSE) {
                        const float w = (pv[k] * p.rs) * p.rs;
                        const float f = w * fmaf(-h, p.rs, dd);
                        c0[k / 4] += f;
                        cz[k / 4] = fmaf(f, (float)k - 0.5f * (float)(FM_RZ - 1), cz[k / 4]);
                    }
                }
                if (WANT_POSE) {
                    const double C = (double)c0[0] + (double)c0[1];
                    Sx = fma((double)(Dx + ox), C, Sx);
                    Sy = fma((double)(Dy + ty.x), C, Sy);
                    Sz = fma((double)fmaf(zmid, g.hs_u, Dz + tz.x), C, fma((double)g.hs_u, (double)cz[0] + (double)cz[1], Sz));
                }
            }
        }
        if (WANT_POSE) {
            double* part = reinterpret_cast<double*>(used);  // [wave][3][lane]
            __syncthreads();                                 // the window has been read
            const double u = -((double)g.unit_h + (double)g.unit_l);
            part[(wv * 3 + 0) * WAVE + lane] = u * Sx;
            part[(wv * 3 + 1) * WAVE + lane] = u * Sy;
            part[(wv * 3 + 2) * WAVE + lane] = u * Sz;
            __syncthreads();
            if (tid < 3 * WAVE && c * WAVE + lane < g.E) {   // wavefront w: component w
                double* row = pose_part + (reg - reg0) * row_step + (size_t)(c * WAVE + lane) * 3 + wv;
                double a = reg == reg0 || row_step ? 0.0 : *row;
                for (int w = 0; w < AM_WAVES; ++w) a += part[(w * 3 + wv) * WAVE + lane];
                *row = a;
            }
        }
        if (++c < nchunk) continue;
        // the region's last chunk
        c = 0;
        if (WANT_P0) {
            // sums over the lanes: rows of 16 lanes, then the four rows
            constexpr int NV = AM_WAVES * CPW * FM_RZ;
            float* part = reinterpret_cast<float*>(used);    // [row][voxel], columns of FM_RZ
            const int vsel = (lane & 3) == 1 ? 2 : ((lane & 3) == 2 ? 1 : (lane & 3));
            __syncthreads();                                 // the window (or the partials in it) has been read
#pragma unroll
            for (int i = 0; i < CPW * FM_RZ; i += 4) {
                const float v = wave_sum4_rows(acc[i], acc[i + 1], acc[i + 2], acc[i + 3], lane);
                const int at = STRIDED ? (i / FM_RZ * AM_WAVES + wv) * FM_RZ + i % FM_RZ : wv * CPW * FM_RZ + i;
                if ((lane & 15) >= 12) part[(lane >> 4) * NV + at + vsel] = v;
                acc[i] = acc[i + 1] = acc[i + 2] = acc[i + 3] = 0.0f;
            }
            __syncthreads();
            float* gbase = grad_p0 + (size_t)R.i0 * g.gsx + (size_t)R.j0 * g.gsy + R.k0;
            for (int t = tid; t < ncol * FM_RZ; t += AM_WAVES * WAVE) {
                const int col = t / FM_RZ, k = t % FM_RZ;
                if (k >= R.nk) continue;
                const float v = (part[t] + part[NV + t]) + (part[2 * NV + t] + part[3 * NV + t]);
                float* dst = gbase + (size_t)(col / R.nj) * g.gsx + (size_t)(col % R.nj) * g.gsy + k;
                *dst = accumulate ? *dst + v : v;
            }
        }
        R = region_info(g, ++reg);
    }
    __syncthreads();                                         // the LDS is free for the next call
}

// One workgroup per CU at most, each with an even share of consecutive regions, so that a region's first
// loads run behind the one before (back-projection of 99 elements, two chunks, into 161x147x130 voxels:
// 471 us with a workgroup per region, 415 us so).
template <int NM, int CPW, bool WANT_P0, bool WANT_POSE, int X>
__global__ __launch_bounds__(AM_WAVES * WAVE) __attribute__((amdgpu_waves_per_eu(4))) void k_adjoint_series(
    Geo g, int nbuf, const float* __restrict__ p0, const float* __restrict__ xe, const float4* __restrict__ q,
    const float* __restrict__ r, float* __restrict__ grad_p0, int accumulate, double* __restrict__ pose_part) {
    extern __shared__ float4 lds4[];
    const int b = region_of_block(blockIdx.x, gridDim.x);
    const int r0 = (int)((long long)g.nreg * b / gridDim.x), r1 = (int)((long long)g.nreg * (b + 1) / gridDim.x);
    am_regions<NM, CPW, WANT_P0, WANT_POSE, X>(g, r0, r1, nbuf, p0, xe, q, r, grad_p0, accumulate,
                                            WANT_POSE ? pose_part + (size_t)blockIdx.x * g.E * 3 : nullptr, 0,
                                            reinterpret_cast<float*>(lds4));
}

// Sum the rows of element-gradient partials in FP64 and a fixed order: a workgroup takes 16
// consecutive gradient components; its 16 phases each sum every 16th row (loads of 16
// consecutive doubles), then the phases are added in order.
constexpr int PR_T = 16, PR_P = 16;
__global__ __launch_bounds__(PR_T * PR_P) void k_pose_reduce(Geo g, int rows, const double* __restrict__ part,
                                                            double* __restrict__ ge, double* __restrict__ grad_elem,
                                                            int accumulate) {
    __shared__ double red[PR_P][PR_T];
    const int tl = threadIdx.x % PR_T, ph = threadIdx.x / PR_T;
    const int n3 = 3 * g.E;
    const int t = blockIdx.x * PR_T + tl;
    double acc = 0.0;
    if (t < n3)
        for (int rg = ph; rg < rows; rg += PR_P) acc += part[(size_t)rg * n3 + t];
    red[ph][tl] = acc;
    __syncthreads();
    if (ph == 0 && t < n3) {
        double sum = 0.0;
        for (int p = 0; p < PR_P; ++p) sum += red[p][tl];
        ge[t] = sum;
        if (grad_elem) grad_elem[t] = accumulate ? grad_elem[t] + sum : sum;
    }
}

// Per frame: dL/dR = sum_m g_e e_m^T, dL/dt = sum_m g_e (FP64 block reduction).
__global__ __launch_bounds__(256) void k_pose_frame(Geo g, const double* __restrict__ ge,
                                                    const double* __restrict__ elem,
                                                    double* __restrict__ grad_pose, int accumulate) {
    __shared__ double red[12][256];
    const int f = blockIdx.x;
    double acc[12];
    for (int q = 0; q < 12; ++q) acc[q] = 0.0;
    for (int m = threadIdx.x; m < g.M; m += blockDim.x) {
        const double* gv = ge + 3 * ((size_t)f * g.M + m);
        const double* em = elem + 3 * m;
        for (int i = 0; i < 3; ++i) {
            for (int j = 0; j < 3; ++j) acc[3 * i + j] += gv[i] * em[j];
            acc[9 + i] += gv[i];
        }
    }
    for (int q = 0; q < 12; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 12; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 12) {
        double v = red[threadIdx.x][0];
        double* out = grad_pose + 12 * f + threadIdx.x;
        *out = accumulate ? *out + v : v;
    }
}

// r = 2 (s - y) in place; per-block FP32 partial sums of (s - y)^2.
__global__ __launch_bounds__(256) void k_residual(float* __restrict__ s, const float* __restrict__ y, size_t n,
                                                  float* __restrict__ partial) {
    __shared__ float red[256];
    float acc = 0.0f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        float d = s[i] - y[i];
        acc = fmaf(d, d, acc);
        s[i] = 2.0f * d;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Stage 2 negative correlation, one workgroup per signal row (one element): the row's
// means, then its spreads and covariance (two passes, FP64 sums), L_e = -Cov/(sigma_s sigma_y),
// and in place dL/ds = w_e (-(y - ybar) / (K sigma_s sigma_y) + Cov (s - sbar) / (K sigma_s^3
// sigma_y)).  A row with zero spread in either signal gets L_e = 0 and a zero gradient.
__device__ __forceinline__ double block_sum_f64(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = NC_THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double t = red[0];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(NC_THREADS) void k_nc_residual(float* __restrict__ s, const float* __restrict__ y,
                                                            const float* __restrict__ weight, int E, int K,
                                                            double* __restrict__ loss_e,
                                                            double* __restrict__ wloss_e) {
    __shared__ double red[NC_THREADS];
    for (int e = blockIdx.x; e < E; e += gridDim.x) {
        float* se = s + (size_t)e * K;
        const float* ye = y + (size_t)e * K;
        double as = 0.0, ay = 0.0;
        for (int k = threadIdx.x; k < K; k += NC_THREADS) {
            as += (double)se[k];
            ay += (double)ye[k];
        }
        const double ms = block_sum_f64(as, red) / K, my = block_sum_f64(ay, red) / K;
        double c = 0.0, vs = 0.0, vy = 0.0;
        for (int k = threadIdx.x; k < K; k += NC_THREADS) {
            const double ds = (double)se[k] - ms, dy = (double)ye[k] - my;
            c = fma(ds, dy, c);
            vs = fma(ds, ds, vs);
            vy = fma(dy, dy, vy);
        }
        const double C = block_sum_f64(c, red) / K;
        const double Vs = block_sum_f64(vs, red) / K, Vy = block_sum_f64(vy, red) / K;
        const double w = weight ? (double)weight[e] : 1.0;
        double a = 0.0, b = 0.0, L = 0.0;
        if (Vs > 0.0 && Vy > 0.0) {
            const double ss = sqrt(Vs), sy = sqrt(Vy);
            L = -C / (ss * sy);
            a = w / (K * ss * sy);
            b = w * C / (K * ss * Vs * sy);
        }
        if (threadIdx.x == 0) {
            if (loss_e) loss_e[e] = L;
            wloss_e[e] = w * L;
        }
        for (int k = threadIdx.x; k < K; k += NC_THREADS) {
            const double ds = (double)se[k] - ms, dy = (double)ye[k] - my;
            se[k] = (float)(fma(b, ds, -a * dy));
        }
    }
}

// Fixed-order FP64 sum of n values into *out (one workgroup).
__global__ __launch_bounds__(NC_THREADS) void k_sum_f64(const double* __restrict__ v, int n,
                                                        double* __restrict__ out) {
    __shared__ double red[NC_THREADS];
    double a = 0.0;
    for (int i = threadIdx.x; i < n; i += NC_THREADS) a += v[i];
    const double t = block_sum_f64(a, red);
    if (threadIdx.x == 0) *out = t;
}

// Second-order TGV regulariser of the Stage 1 / Stage 5 objectives, for a volume u and its
// auxiliary vector field w, the discretisation written out: alpha1 sum |D+ u - w|_eps + alpha0 sum |E(w)|_eps, D+ forward
// differences (zero at the last index), E(w) = (D-_a w_b + D-_b w_a) / 2 with backward
// differences (zero at the first index), |x|_eps = sqrt(|x|^2 + eps^2) - eps.  With the
// normalised fields q = alpha1 g/|g|_eps (g = D+u - w) and Q = alpha0 E/|E|_eps the gradients are
//   dR/du   = sum_a [q_a(v - e_a) (v_a >= 1) - q_a(v) (v_a <= n_a - 2)],
//   dR/dw_b = -q_b(v) + sum_a [Q_ab(v) (v_a >= 1) - Q_ab(v + e_a) (v_a <= n_a - 2)],
// so a voxel needs q at itself and its three lower neighbours and Q at itself and its three
// upper neighbours: everything within one voxel of it.  One pass computes them from u and w.
struct TgvDims {
    int nx, ny, nz;
    int n, sx, sy;           // voxels (< 2^31); strides of x and y (z contiguous)
    int bz, by, xc;          // tiles along z and y, planes of a tile
    float a0, a1, eps;
};

// Bound by memory: 16 bytes read and 16 written a voxel.  A workgroup marches along x over rows of z: L lanes hold a
// row's 4 L voxels, 4 each, and its first and last row are halo.  Each voxel's q and Q are computed once and passed to
// the neighbours that need them: along x in registers, along z within the lane or by a lane shift, along y through LDS,
// as are the inputs' own neighbours.  The next plane's loads are in flight meanwhile.  256^3: 108 us, 5.0 TB/s, of them
// 17 us by stores that do not allocate in L2 (the results are not read again here); computing q and Q again for each
// neighbour from a tile of u and w in LDS took 214 us, bound by its 106 instructions a voxel and their LDS reads.
constexpr int TGV_V = 4;               // voxels of a lane
constexpr int TGV_TILE = 62 * TGV_V;   // voxels along z of a workgroup where a row of z does not fit into 64 lanes
constexpr int TGV_NW = 12;             // wavefronts of a workgroup: 16 spill (256^3: 196 us), 8 have more halo (149 us)
constexpr int TGV_LDS = 9;             // float4 per thread: u twice, w, and what a row passes on

typedef float tgv4 __attribute__((ext_vector_type(4)));
typedef tgv4 tgv4u __attribute__((aligned(4)));        // rows start at any voxel

// Norms and their reciprocals by the hardware square root and reciprocal (about 1 ulp each;
// the arguments are at least eps^2, far from the denormal range).
__device__ __forceinline__ float tgv_n1(const TgvDims& d, const float g[3]) {
    return __builtin_amdgcn_sqrtf(g[0] * g[0] + g[1] * g[1] + g[2] * g[2] + d.eps * d.eps);
}

__device__ __forceinline__ float tgv_n0(const TgvDims& d, const float E[6]) {
    return __builtin_amdgcn_sqrtf(E[0] * E[0] + E[1] * E[1] + E[2] * E[2] +
                                  2.0f * (E[3] * E[3] + E[4] * E[4] + E[5] * E[5]) + d.eps * d.eps);
}

__device__ __forceinline__ float tgv_ratio(float a, float n) {
    return a * __builtin_amdgcn_rcpf(n);
}

// The previous and the next lane's value (0 beyond the wavefront); called with all lanes active.
__device__ __forceinline__ float tgv_lower(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));
}

__device__ __forceinline__ float tgv_upper(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// Four voxels from index i on of an array of n; those that are not wanted may come from the next row.
__device__ __forceinline__ tgv4 tgv_load(const float* __restrict__ src, int i, int n) {
    if (i <= n - TGV_V) return *reinterpret_cast<const tgv4u*>(src + i);
    tgv4 v;
#pragma unroll
    for (int e = 0; e < TGV_V; ++e) v[e] = src[i + min(e, n - 1 - i)];
    return v;
}

__device__ __forceinline__ void tgv_store(float* __restrict__ dst, int k, int nz, tgv4 v, float scale, int accumulate) {
    if (k <= nz - TGV_V) {
        tgv4u* p = reinterpret_cast<tgv4u*>(dst + k);
        if (accumulate) {
            const tgv4 o = *p;
#pragma unroll
            for (int e = 0; e < TGV_V; ++e) v[e] = fmaf(scale, v[e], o[e]);
        } else {
            v *= scale;
        }
        __builtin_nontemporal_store(v, p);
        return;
    }
#pragma unroll
    for (int e = 0; e < TGV_V; ++e)
        if (k < nz - e) dst[k + e] = accumulate ? fmaf(scale, v[e], dst[k + e]) : scale * v[e];
}

// Value partials (one per workgroup) and, when asked, both gradients, in one pass.
template <int L>
__global__ __launch_bounds__(64 * TGV_NW) void k_tgv(TgvDims d, const float* __restrict__ u, const float* __restrict__ w,
                                                 float scale, int accumulate, float* __restrict__ gu,
                                                 float* __restrict__ gw, double* __restrict__ partial) {
    constexpr int NT = 64 * TGV_NW, R = NT / L;
    extern __shared__ char tgv_smem[];
    tgv4* T = reinterpret_cast<tgv4*>(tgv_smem);       // [0, 1] u by plane parity, [2 + b] w_b, [5] q_y, [6 + b] Q_yb
    // tiles in x order, each compute die (XCD) taking a contiguous run of them so that the
    // halo rows and planes shared with the neighbouring tiles stay in that die's L2
    const int blk = region_of_block(blockIdx.x, gridDim.x);
    const int bk = blk % d.bz, bj = (blk / d.bz) % d.by, bi = blk / (d.bz * d.by);
    const int t = threadIdx.x, r = t / L, l = t % L;
    const bool split = d.bz > 1;                       // then the first and the last lane are halo
    const int k = split ? bk * TGV_TILE + TGV_V * (l - 1) : TGV_V * l;
    const int j = bj * (R - 2) + r - 1;
    const int x0 = bi * d.xc, x1 = x0 + min(d.xc, d.nx - x0);
    const int tm = r > 0 ? t - L : t, tp = r < R - 1 ? t + L : t;
    const bool row = j >= 0 && j < d.ny && k >= 0;
    const bool out = row && r > 0 && r < R - 1 && (!split || (l > 0 && l < L - 1)) && k < d.nz;
    const int jc = min(max(j, 0), d.ny - 1) * d.sy, kc = k >= 0 && k < d.nz ? k : 0;
    tgv4 pu, pw[3], cu, cw[3], A[3];        // A: what dR/dw of plane i has from Q of planes up to i
    float qx[TGV_V] = {0.0f, 0.0f, 0.0f, 0.0f};
    double acc = 0.0;
    auto load = [&](int x, tgv4& lu, tgv4 lw[3]) {
        const int o = min(max(x, 0), d.nx - 1) * d.sx + jc + kc;
        lu = tgv_load(u, o, d.n);
#pragma unroll
        for (int b = 0; b < 3; ++b) lw[b] = tgv_load(w + (size_t)b * d.n, o, d.n);
    };
    load(x0 - 1, pu, pw);
    load(x0, cu, cw);
#pragma unroll
    for (int b = 0; b < 3; ++b) A[b] = 0.0f;
    T[((x0 - 1) & 1) * NT + t] = pu;
    for (int i = x0 - 1; i < x1; ++i) {
        // planes i (pu, pw) and i + 1 (cu, cw): Q of plane i + 1, q and the results of plane i
        T[((i + 1) & 1) * NT + t] = cu;
#pragma unroll
        for (int b = 0; b < 3; ++b) T[(2 + b) * NT + t] = cw[b];
        __syncthreads();
        tgv4 nu, nw[3];
        load(min(i + 2, x1), nu, nw);
        tgv4 gs;
        {
            // q of plane i; q_a counts in dR/du only where v_a <= n_a - 2
            const tgv4 uy = T[(i & 1) * NT + tp];
            const float uz = tgv_upper(pu[0]);
            const bool ux = i >= 0 && i < d.nx - 1;
            tgv4 qy, qz;
#pragma unroll
            for (int e = 0; e < TGV_V; ++e) {
                float g[3];
                g[0] = (ux ? cu[e] - pu[e] : 0.0f) - pw[0][e];
                g[1] = (j < d.ny - 1 ? uy[e] - pu[e] : 0.0f) - pw[1][e];
                g[2] = (k < d.nz - 1 - e ? (e < TGV_V - 1 ? pu[(e + 1) % TGV_V] : uz) - pu[e] : 0.0f) - pw[2][e];
                const float n1 = tgv_n1(d, g), s1 = tgv_ratio(d.a1, n1);
                if (out && i >= x0 && k < d.nz - e) acc += (double)d.a1 * (double)(n1 - d.eps);
#pragma unroll
                for (int b = 0; b < 3; ++b) A[b][e] -= s1 * g[b];
                const float qh = ux ? s1 * g[0] : 0.0f;
                gs[e] = qx[e] - qh;
                qx[e] = qh;
                qy[e] = row && j < d.ny - 1 && k < d.nz - e ? s1 * g[1] : 0.0f;
                qz[e] = row && k < d.nz - 1 - e ? s1 * g[2] : 0.0f;
            }
            const float ql = tgv_lower(qz[TGV_V - 1]), qb = k > 0 ? ql : 0.0f;
#pragma unroll
            for (int e = 0; e < TGV_V; ++e) gs[e] += ((e ? qz[(e + TGV_V - 1) % TGV_V] : qb) - qz[e]) - qy[e];
            T[5 * NT + t] = qy;
        }
        tgv4 gb[3];
        {
            // Q of plane i + 1
            const bool px = i + 1 < d.nx, lx = i >= 0 && px;
            tgv4 Q[6], wy[3];
            float wz[3];
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                wy[b] = T[(2 + b) * NT + tm];
                wz[b] = tgv_lower(cw[b][TGV_V - 1]);
            }
#pragma unroll
            for (int e = 0; e < TGV_V; ++e) {
                const bool in = row && px && k < d.nz - e;
                float D[3][3], E[6];
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    D[0][b] = in && lx ? cw[b][e] - pw[b][e] : 0.0f;
                    D[1][b] = in && j > 0 ? cw[b][e] - wy[b][e] : 0.0f;
                    D[2][b] = in && k + e > 0 ? cw[b][e] - (e ? cw[b][e - 1] : wz[b]) : 0.0f;
                }
                E[0] = D[0][0];
                E[1] = D[1][1];
                E[2] = D[2][2];
                E[3] = 0.5f * (D[0][1] + D[1][0]);
                E[4] = 0.5f * (D[0][2] + D[2][0]);
                E[5] = 0.5f * (D[1][2] + D[2][1]);
                const float n0 = tgv_n0(d, E), s0 = tgv_ratio(d.a0, n0);
                if (out && in && i + 1 < x1) acc += (double)d.a0 * (double)(n0 - d.eps);
#pragma unroll
                for (int c = 0; c < 6; ++c) Q[c][e] = s0 * E[c];
            }
            // Q_ab as an index into Q by (a, b)
            constexpr int qi[3][3] = {{0, 3, 4}, {3, 1, 5}, {4, 5, 2}};
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const tgv4 Qx = Q[qi[0][b]], Qy = Q[qi[1][b]], Qz = Q[qi[2][b]];
                T[(6 + b) * NT + t] = Qy;
                const float Ql = tgv_upper(Qz[0]), Qn = k < d.nz - TGV_V ? Ql : 0.0f;
                gb[b] = A[b] - Qx;
#pragma unroll
                for (int e = 0; e < TGV_V; ++e)
                    A[b][e] = (i >= 0 ? Qx[e] : 0.0f) + (j > 0 ? Qy[e] : 0.0f) +
                              ((k + e > 0 ? Qz[e] : 0.0f) - (e < TGV_V - 1 ? Qz[(e + 1) % TGV_V] : Qn));
            }
        }
        __syncthreads();
        const bool store = out && i >= x0;
        const size_t o = (size_t)(i * d.sx + jc);
        if (gu && store) {
            gs += T[5 * NT + tm];
            tgv_store(gu + o, k, d.nz, gs, scale, accumulate);
        }
        if (gw) {
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                A[b] -= T[(6 + b) * NT + tp];
                if (store) tgv_store(gw + (size_t)b * d.n + o, k, d.nz, gb[b], scale, accumulate);
            }
        }
        pu = cu;
        cu = nu;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            pw[b] = cw[b];
            cw[b] = nw[b];
        }
    }
    __syncthreads();
    double* red = reinterpret_cast<double*>(tgv_smem);
    red[t] = acc;
    __syncthreads();
    for (int s2 = 512; s2 > 0; s2 >>= 1) {
        if (t < s2 && t + s2 < NT) red[t] += red[t + s2];
        __syncthreads();
    }
    if (t == 0) partial[blk] = red[0];
}

// How a volume is cut: lanes of a row (the fewest of 16, 32, 64 that hold it, so that short rows share a wavefront;
// longer ones are cut with a halo lane on either side), tiles along z, y and x, and planes of a tile.
struct TgvCut {
    int lanes, bz, by, bx, xc;
};

static TgvCut tgv_cut(int nx, int ny, int nz) {
    TgvCut c;
    c.lanes = nz <= 16 * TGV_V ? 16 : nz <= 32 * TGV_V ? 32 : 64;
    c.bz = nz <= 64 * TGV_V ? 1 : (nz - 1) / TGV_TILE + 1;
    const int rows = 64 * TGV_NW / c.lanes - 2;
    c.by = (ny - 1) / rows + 1;
    // planes of a tile: the fewest steps over the rounds of workgroups, each tile taking one step more than planes
    const long long slots = NCU, cols = (long long)c.by * c.bz, first = (cols + slots - 1) / slots;
    long long best = -1;
    for (long long m = first; m < first + 4; ++m) {
        const int xc = (int)std::max(1LL, (nx + m * slots / cols - 1) / (m * slots / cols));
        if (best < 0 || m * (xc + 2) < best) {
            best = m * (xc + 2);
            c.xc = xc;
        }
    }
    c.bx = (nx - 1) / c.xc + 1;
    return c;
}

static inline unsigned tgv_blocks(int nx, int ny, int nz) {
    const TgvCut c = tgv_cut(nx, ny, nz);
    return (unsigned)c.bx * c.by * c.bz;
}

// ------------------------------------------------------------------------------------------
// axis-angle poses.  R = exp([w]x) = I + a [w]x + b [w]x^2, and
// dL/dw = J_r(w)^T vee(R^T G - G^T R) / 1 with J_r the right Jacobian of SO(3):
//   J_r = I - b [w]x + c [w]x^2,  a = sin th/th, b = (1-cos th)/th^2, c = (th - sin th)/th^3.
// ------------------------------------------------------------------------------------------
__device__ void so3_coefs(double th, double& a, double& b, double& c) {
    double t2 = th * th;
    if (th < 0.05) {
        a = 1.0 - t2 / 6.0 * (1.0 - t2 / 20.0 * (1.0 - t2 / 42.0 * (1.0 - t2 / 72.0)));
        b = 0.5 * (1.0 - t2 / 12.0 * (1.0 - t2 / 30.0 * (1.0 - t2 / 56.0 * (1.0 - t2 / 90.0))));
        c = (1.0 / 6.0) * (1.0 - t2 / 20.0 * (1.0 - t2 / 42.0 * (1.0 - t2 / 72.0 * (1.0 - t2 / 110.0))));
    } else {
        double sn = sin(th), cs = cos(th);
        a = sn / th;
        b = (1.0 - cs) / t2;
        c = (th - sn) / (t2 * th);
    }
}

__device__ void so3_exp(const double* w, double* R) {
    const double w0 = w[0], w1 = w[1], w2 = w[2];
    const double th = sqrt(w0 * w0 + w1 * w1 + w2 * w2);
    double a, b, c;
    so3_coefs(th, a, b, c);
    const double K[9] = {0, -w2, w1, w2, 0, -w0, -w1, w0, 0};
    const double W[3] = {w0, w1, w2};
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const double k2 = W[i] * W[j] - (i == j ? th * th : 0.0);  // [w]x^2 = w w^T - th^2 I
            R[3 * i + j] = (i == j ? 1.0 : 0.0) + a * K[3 * i + j] + b * k2;
        }
}

// gw = J_r(w)^T vee(R^T G - G^T R)... with M = R^T G and m = vee(M - M^T).
__device__ void so3_vjp(const double* w, const double* G, double* gw) {
    double R[9];
    so3_exp(w, R);
    const double w0 = w[0], w1 = w[1], w2 = w[2];
    const double th = sqrt(w0 * w0 + w1 * w1 + w2 * w2);
    double a, b, c;
    so3_coefs(th, a, b, c);
    double Mx[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) Mx[3 * i + j] = R[i] * G[j] + R[3 + i] * G[3 + j] + R[6 + i] * G[6 + j];
    const double m[3] = {Mx[7] - Mx[5], Mx[2] - Mx[6], Mx[3] - Mx[1]};
    // J_r^T m = m + b [w]x m + c [w]x^2 m
    const double Km[3] = {w1 * m[2] - w2 * m[1], w2 * m[0] - w0 * m[2], w0 * m[1] - w1 * m[0]};
    const double KKm[3] = {w1 * Km[2] - w2 * Km[1], w2 * Km[0] - w0 * Km[2], w0 * Km[1] - w1 * Km[0]};
    for (int i = 0; i < 3; ++i) gw[i] = m[i] + b * Km[i] + c * KKm[i];
}

// Euler angles of Stage 4 (extrinsic x, then y, then z): R = Rz(a2) Ry(a1) Rx(a0).
__device__ void mat3_mul(const double* A, const double* B, double* C) {
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}

// Elementary rotations about x, y, z and their derivatives with respect to the angle.
__device__ void euler_factors(const double* a, double* Rx, double* Ry, double* Rz, double* Dx, double* Dy,
                              double* Dz) {
    const double cx = cos(a[0]), sx = sin(a[0]), cy = cos(a[1]), sy = sin(a[1]), cz = cos(a[2]), sz = sin(a[2]);
    const double rx[9] = {1, 0, 0, 0, cx, -sx, 0, sx, cx}, dx[9] = {0, 0, 0, 0, -sx, -cx, 0, cx, -sx};
    const double ry[9] = {cy, 0, sy, 0, 1, 0, -sy, 0, cy}, dy[9] = {-sy, 0, cy, 0, 0, 0, -cy, 0, -sy};
    const double rz[9] = {cz, -sz, 0, sz, cz, 0, 0, 0, 1}, dz[9] = {-sz, -cz, 0, cz, -sz, 0, 0, 0, 0};
    for (int i = 0; i < 9; ++i) {
        Rx[i] = rx[i]; Ry[i] = ry[i]; Rz[i] = rz[i];
        Dx[i] = dx[i]; Dy[i] = dy[i]; Dz[i] = dz[i];
    }
}

__global__ void k_pose_from_euler(const double* __restrict__ pose6, int F, double* __restrict__ poses) {
    int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const double* p = pose6 + 6 * f;
    double Rx[9], Ry[9], Rz[9], Dx[9], Dy[9], Dz[9], T[9];
    euler_factors(p, Rx, Ry, Rz, Dx, Dy, Dz);
    double* R = poses + 12 * f;
    mat3_mul(Ry, Rx, T);
    mat3_mul(Rz, T, R);
    R[9] = p[3]; R[10] = p[4]; R[11] = p[5];
}

__global__ void k_pose_grad_euler(const double* __restrict__ pose6, const double* __restrict__ gpose, int F,
                                  double* __restrict__ g6) {
    int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const double* G = gpose + 12 * f;
    double Rx[9], Ry[9], Rz[9], Dx[9], Dy[9], Dz[9], T[9], U[9];
    euler_factors(pose6 + 6 * f, Rx, Ry, Rz, Dx, Dy, Dz);
    double* out = g6 + 6 * f;
    double acc[3];
    mat3_mul(Ry, Dx, T);                   // dR/da0 = Rz Ry Dx
    mat3_mul(Rz, T, U);
    acc[0] = 0.0;
    for (int i = 0; i < 9; ++i) acc[0] += G[i] * U[i];
    mat3_mul(Dy, Rx, T);                   // dR/da1 = Rz Dy Rx
    mat3_mul(Rz, T, U);
    acc[1] = 0.0;
    for (int i = 0; i < 9; ++i) acc[1] += G[i] * U[i];
    mat3_mul(Ry, Rx, T);                   // dR/da2 = Dz Ry Rx
    mat3_mul(Dz, T, U);
    acc[2] = 0.0;
    for (int i = 0; i < 9; ++i) acc[2] += G[i] * U[i];
    out[0] = acc[0]; out[1] = acc[1]; out[2] = acc[2];
    out[3] = G[9]; out[4] = G[10]; out[5] = G[11];
}

__global__ void k_pose_from_aa(const double* __restrict__ pose6, int F, double* __restrict__ poses) {
    int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const double* p = pose6 + 6 * f;
    double* R = poses + 12 * f;
    so3_exp(p, R);
    R[9] = p[3]; R[10] = p[4]; R[11] = p[5];
}

__global__ void k_pose_grad_aa(const double* __restrict__ pose6, const double* __restrict__ gpose, int F,
                               double* __restrict__ g6) {
    int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= F) return;
    const double* G = gpose + 12 * f;
    double* out = g6 + 6 * f;
    so3_vjp(pose6 + 6 * f, G, out);
    out[3] = G[9]; out[4] = G[10]; out[5] = G[11];
}

// ------------------------------------------------------------------------------------------
// exact update count (FP64, decided as |d - c*(k/fs)| <= trunc*sigma)
// ------------------------------------------------------------------------------------------
__global__ void k_elements_f64(int M, int E, const double* __restrict__ elem, const double* __restrict__ poses,
                               double* __restrict__ xe) {
#pragma clang fp contract(off)
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= E) return;
    int f = e / M, m = e % M;
    const double* R = poses + 12 * f;
    const double* em = elem + 3 * m;
    for (int i = 0; i < 3; ++i)
        xe[3 * e + i] = R[3 * i + 0] * em[0] + R[3 * i + 1] * em[1] + R[3 * i + 2] * em[2] + R[9 + i];
}

__global__ __launch_bounds__(256) void k_count(int nx, int ny, int nz, double ox, double oy, double oz, double h,
                                               int E, const double* __restrict__ xe, double c, double fs, int K,
                                               double tsig, unsigned long long* __restrict__ total) {
#pragma clang fp contract(off)
    __shared__ unsigned long long red[256];
    long long nvox = (long long)nx * ny * nz;
    long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    unsigned long long cnt = 0;
    if (v < nvox) {
        long long i = v / ((long long)ny * nz), j = (v / nz) % ny, k = v % nz;
        double px = ox + (double)i * h, py = oy + (double)j * h, pz = oz + (double)k * h;
        for (int e = 0; e < E; ++e) {
            double dx = px - xe[3 * e], dy = py - xe[3 * e + 1], dz = pz - xe[3 * e + 2];
            double d = sqrt(dx * dx + dy * dy + dz * dz);
            long a = (long)ceil((d - tsig) * fs / c) - 1;
            long b = (long)floor((d + tsig) * fs / c) + 1;
            if (a < 0) a = 0;
            if (b > K - 1) b = K - 1;
            while (a <= b && !(fabs(d - c * ((double)a / fs)) <= tsig)) ++a;
            while (b >= a && !(fabs(d - c * ((double)b / fs)) <= tsig)) --b;
            if (b >= a) cnt += (unsigned long long)(b - a + 1);
        }
    }
    red[threadIdx.x] = cnt;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(total, red[0]);
}


// ------------------------------------------------------------------------------------------
// issue-rate probes (calibration of the roofline figures): every thread runs PROBE_CHAINS
// independent chains of FP32 FMAs, or of v_exp_f32, so the issue rate, not latency, bounds them
// ------------------------------------------------------------------------------------------
constexpr int PROBE_CHAINS = 8;
constexpr int PROBE_BLOCKS = 4096;

__global__ __launch_bounds__(256) void k_probe_fma(float* __restrict__ out, int iters, float a, float b) {
    float x[PROBE_CHAINS];
#pragma unroll
    for (int c = 0; c < PROBE_CHAINS; ++c) x[c] = 1e-3f * (float)(threadIdx.x + c);
#pragma unroll 4
    for (int i = 0; i < iters; ++i)
#pragma unroll
        for (int c = 0; c < PROBE_CHAINS; ++c) x[c] = fmaf(x[c], a, b);
    float t = 0.0f;
#pragma unroll
    for (int c = 0; c < PROBE_CHAINS; ++c) t += x[c];
    out[blockIdx.x * blockDim.x + threadIdx.x] = t;
}

__global__ __launch_bounds__(256) void k_probe_exp(float* __restrict__ out, int iters) {
    float x[PROBE_CHAINS];
#pragma unroll
    for (int c = 0; c < PROBE_CHAINS; ++c) x[c] = 1e-3f * (float)(threadIdx.x + c);
#pragma unroll 4
    for (int i = 0; i < iters; ++i)
#pragma unroll
        for (int c = 0; c < PROBE_CHAINS; ++c) x[c] = __builtin_amdgcn_exp2f(-x[c]);    // stays in (1/2, 1]
    float t = 0.0f;
#pragma unroll
    for (int c = 0; c < PROBE_CHAINS; ++c) t += x[c];
    out[blockIdx.x * blockDim.x + threadIdx.x] = t;
}

// ==========================================================================================
// batched steps (serving): one gradient step for every request of a batch, each request
// with its own array size, sample count and box of the resident volume.  Work lists and
// their lengths live in device memory and every launch uses a fixed grid that walks its
// list, so a captured HIP graph replays the step for whatever batch the lists describe.
// ==========================================================================================
constexpr int BATCH_THREADS = 256;

// A request's descriptor: its geometry and the moment forms' series (nm terms for the forward, 8 for the adjoints).  The
// adjoints take a region of 16 voxels along z as two of 8, those of ga.
struct BatchGeo {
    Geo g, ga;
    int nm;
    MomCoef series, series8;
};

// Element positions of every request, by threads t0, t0 + stride, ..
__device__ __forceinline__ void batch_elements(const ra_batch_request* __restrict__ reqs, const int2* __restrict__ items,
                                               int n, int t0, int stride) {
    for (int it = t0; it < n; it += stride) {
        const int2 w = items[it];
        const ra_batch_request& q = reqs[w.x];
        double R[9];
        so3_exp(q.pose6, R);
        const double* em = q.elem + 3 * w.y;
        const DF ev[3] = {df_from_double(em[0]), df_from_double(em[1]), df_from_double(em[2])};
        float* out = q.xe + 6 * w.y;
        for (int i = 0; i < 3; ++i) {
            DF acc = df_from_double(q.pose6[3 + i]);
            for (int j = 0; j < 3; ++j) acc = df_add(acc, df_mul(df_from_double(R[3 * i + j]), ev[j]));
            out[i] = acc.h;
            out[3 + i] = acc.l;
        }
    }
}

__global__ void k_batch_elements(const ra_batch_request* __restrict__ reqs, const int2* __restrict__ items,
                                 const int* __restrict__ counts) {
    batch_elements(reqs, items, counts[3], blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// zero the signal buffer of every request (slot-major, one workgroup per slot at a time)
__global__ void k_batch_zero(const BatchGeo* __restrict__ geos, const ra_batch_request* __restrict__ reqs,
                             const int* __restrict__ counts) {
    const int ns = counts[4];
    for (int slot = blockIdx.x; slot < ns; slot += gridDim.x) {
        if (reqs[slot].kind < 0) continue;      // slot not in this batch
        const Geo& g = geos[slot].g;
        float* s = reqs[slot].s;
        const int n = g.E * g.K;
        for (int i = threadIdx.x; i < n; i += blockDim.x) s[i] = 0.0f;
    }
}

// r = 2 (s - y) in place and the loss sum (s - y)^2 of every request
__global__ __launch_bounds__(BATCH_THREADS) void k_batch_residual(const BatchGeo* __restrict__ geos,
                                                                  const ra_batch_request* __restrict__ reqs,
                                                                  const int* __restrict__ counts) {
    __shared__ float red[BATCH_THREADS];
    const int ns = counts[4];
    for (int slot = blockIdx.x; slot < ns; slot += gridDim.x) {
        const ra_batch_request& q = reqs[slot];
        if (q.kind < 0) continue;               // slot not in this batch (uniform per block)
        const Geo& g = geos[slot].g;
        const int n = g.E * g.K;
        float acc = 0.0f;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const float d = q.s[i] - q.y[i];
            acc = fmaf(d, d, acc);
            q.s[i] = 2.0f * d;
        }
        red[threadIdx.x] = acc;
        __syncthreads();
        for (int w = BATCH_THREADS / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) q.loss[0] = red[0];
        __syncthreads();
    }
}

template <int JT, bool EXACT, int D>
__global__ __launch_bounds__(BLOCK) void k_forward_batch(const BatchGeo* __restrict__ geos,
                                                         const ra_batch_request* __restrict__ reqs,
                                                         const float4* __restrict__ vtab,
                                                         const int4* __restrict__ itab,
                                                         const int2* __restrict__ items,
                                                         const int* __restrict__ counts, int lmax) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    float* rows = lds + (size_t)wave * lmax * WAVE;
    for (int ix = 0; ix < lmax; ++ix) rows[ix * WAVE + lane] = 0.0f;
    const int n = counts[0];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = items[it];
        const ra_batch_request& q = reqs[w.x];
        forward_region<JT, EXACT, D, float>(geos[w.x].g, w.y, q.p0, q.xe, vtab, itab, q.s, rows, lane, wave);
    }
}

template <int JT, bool EXACT, bool WANT_P0, bool WANT_POSE>
__global__ __launch_bounds__(BLOCK) void k_adjoint_batch(const BatchGeo* __restrict__ geos,
                                                         const ra_batch_request* __restrict__ reqs,
                                                         const float4* __restrict__ vtab,
                                                         const int4* __restrict__ itab,
                                                         const int2* __restrict__ items,
                                                         const int* __restrict__ counts, int which, int lmax) {
    extern __shared__ float lds[];
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    float* rows = lds + (size_t)wave * lmax * WAVE;
    float* gsum = lds + (size_t)WAVES * lmax * WAVE;
    const int n = counts[which];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = items[it];
        const ra_batch_request& q = reqs[w.x];
        adjoint_region<JT, EXACT, WANT_P0, WANT_POSE>(geos[w.x].g, w.y, q.p0, q.xe, vtab, itab, q.s, q.grad_p0, 0,
                                                       q.pose_part, rows, gsum, lane, wave);
    }
}

// Moment form of the batched step.  Element positions of every request, and cleared signals.
__global__ __launch_bounds__(BATCH_THREADS) void k_batch_begin(const BatchGeo* __restrict__ geos,
                                                               const ra_batch_request* __restrict__ reqs,
                                                               const int2* __restrict__ items,
                                                               const int* __restrict__ counts) {
    const int ns = counts[4], stride = gridDim.x * BATCH_THREADS, t0 = blockIdx.x * BATCH_THREADS + threadIdx.x;
    batch_elements(reqs, items, counts[3], t0, stride);
    for (int slot = 0; slot < ns; ++slot) {
        if (reqs[slot].kind < 0) continue;
        const long long n = (long long)geos[slot].g.E * geos[slot].g.K;
        float* s = reqs[slot].s;
        for (long long i = t0; i < n; i += stride) s[i] = 0.0f;
    }
}

template <int NM>
__device__ __forceinline__ void batch_forward_item(const BatchGeo& bg, const ra_batch_request& rq, int reg, bool same, float* lds) {
    const int dl = fm_dlen(bg.g.jt);
    float* dt = lds + fm_off_dt(NM, bg.g.nbin);
    if (!same)                                               // the last item's table, if it was of the same request, is in place
        for (int i = threadIdx.x; i < NM * dl; i += FM_WAVES * WAVE)
            dt[i] = mom_coef(bg.series, i / dl, i % dl - FM_PAD - bg.g.jt, bg.g.jt);
    fm_region<NM, FM_WAVES, 0, float>(bg.g, reg, 0, 1, rq.p0, rq.xe, rq.s, lds);
    __syncthreads();                                         // the LDS is free for the next item
}

// lds_bytes: this launch's LDS; a request that needs more (a descriptor from another batch layout) is skipped.
__global__ __launch_bounds__(FM_WAVES * WAVE) __attribute__((amdgpu_waves_per_eu(4))) void k_forward_mom_batch(
    const BatchGeo* __restrict__ geos, const ra_batch_request* __restrict__ reqs, const int2* __restrict__ items,
    const int* __restrict__ counts, int lds_bytes) {
    extern __shared__ float lds[];
    const int n = counts[0];
    int last = -1;
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = items[it];
        const BatchGeo& bg = geos[w.x];
        const bool same = w.x == last;
        if ((int)fm_lds(bg.nm, bg.g.nbin, bg.g.jt, false) > lds_bytes) continue;      // uniform per workgroup
        if (bg.nm == 6) batch_forward_item<6>(bg, reqs[w.x], w.y, same, lds);
        else if (bg.nm == 7) batch_forward_item<7>(bg, reqs[w.x], w.y, same, lds);
        else batch_forward_item<8>(bg, reqs[w.x], w.y, same, lds);
        last = w.x;
    }
}

// dL/ds = 2 (s - y) in place, each element's loss, and the table of dL/ds, as k_moment_series: a workgroup takes an
// element's row from its start, and the window of table row kk ends at r[kk], so each segment needs only the tail of
// the one before.  The loss of element e goes behind the table (the batch's residual and table kernels took
// 0.204 and 0.013 ms a step, one workgroup a request; 0.018 ms so).
__global__ __launch_bounds__(MT_ROWS) void k_batch_series(const BatchGeo* __restrict__ geos,
                                                          const ra_batch_request* __restrict__ reqs,
                                                          const int2* __restrict__ items, const int* __restrict__ counts) {
    __shared__ float row[MT_ROWS + 2 * JMAX];
    __shared__ float red[MT_ROWS / WAVE];
    const int n = counts[3], tid = threadIdx.x;
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = items[it];
        const BatchGeo& bg = geos[w.x];
        const ra_batch_request& rq = reqs[w.x];
        const int E = bg.g.E, K = bg.g.K, jt = bg.g.jt, kq = K + 2 * jt, e = w.y;
        float* s = rq.s + (size_t)e * K;
        const float* y = rq.y + (size_t)e * K;
        float4* q = reinterpret_cast<float4*>(rq.q);
        float loss = 0.0f;
        __syncthreads();                                     // the last item's row has been read
        if (tid < 2 * jt) row[tid] = 0.0f;
        for (int kk0 = 0; kk0 < kq; kk0 += MT_ROWS) {
            const int kk = kk0 + tid;
            float r = 0.0f;
            if (kk < K) {
                const float d = s[kk] - y[kk];
                loss = fmaf(d, d, loss);
                r = 2.0f * d;
                s[kk] = r;
            }
            row[2 * jt + tid] = r;                           // row[2 jt + i] = r[kk0 + i]
            __syncthreads();
            const float* c = row + tid + jt;                 // r at the row's own sample kk - jt
            float acc[MOM_G];
#pragma unroll
            for (int m = 0; m < MOM_G; ++m) acc[m] = c[0] * bg.series8.d[m];
            for (int j = 1; j <= jt; ++j) {
                const float a = c[j], b = c[-j], sum = a + b, dif = a - b;
#pragma unroll
                for (int m = 0; m < MOM_G; ++m) acc[m] = fmaf(m & 1 ? sum : dif, bg.series8.d[j * MOM_MAX + m], acc[m]);
            }
            if (kk < kq) {
                float4* out = q + 2 * ((size_t)e * kq + kk);
                out[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
                out[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
            }
            float tail = 0.0f;
            if (tid < 2 * jt) tail = row[MT_ROWS + tid];
            __syncthreads();
            if (tid < 2 * jt) row[tid] = tail;
        }
        loss = wave_sum_to_63(loss);
        if ((tid & (WAVE - 1)) == WAVE - 1) red[tid / WAVE] = loss;
        __syncthreads();
        if (tid == 0) {
            float t = 0.0f;
            for (int i = 0; i < MT_ROWS / WAVE; ++i) t += red[i];
            rq.q[((size_t)E * kq + 1) * MOM_G + e] = t;
        }
        if (e == 0 && tid < 2) q[(size_t)E * kq * 2 + tid] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);     // the zero row
    }
}

// The moment-form adjoints of every request: the pose items, then the volume items.  A workgroup takes units of
// BATCH_UNIT consecutive items, far apart in the list, and in each the runs of consecutive regions of a request
// together: items differ in cost by their element count and by the windows that miss the record (six requests of 61 to
// 127 voxels a side, 64 to 256 elements: 1.50 ms with an even share of consecutive items per workgroup, 1.10 ms so).
constexpr int BATCH_UNIT = 8;

template <int CPW, bool WANT_P0, bool WANT_POSE>
__device__ __forceinline__ void batch_adjoint_run(const BatchGeo& bg, const ra_batch_request& rq, int reg, int cnt, int nbuf,
                                                  float* lds) {
    const size_t row = (size_t)bg.g.E * 3;
    if (bg.g.rz > FM_RZ) {                                   // a region's halves add into one row of partials
        for (int i = 0; i < cnt; ++i, ++reg) {
            const int c = 2 * (reg % bg.g.nrz), half = reg / bg.g.nrz * bg.ga.nrz + c;
            am_regions<MOM_G, CPW, WANT_P0, WANT_POSE, 0>(bg.ga, half, half + min(2, bg.ga.nrz - c), nbuf, rq.p0, rq.xe,
                                                          reinterpret_cast<const float4*>(rq.q), nullptr, rq.grad_p0, 0,
                                                          WANT_POSE ? rq.pose_part + reg * row : nullptr, 0, lds);
        }
        return;
    }
    am_regions<MOM_G, CPW, WANT_P0, WANT_POSE, 0>(bg.g, reg, reg + cnt, nbuf, rq.p0, rq.xe,
                                                   reinterpret_cast<const float4*>(rq.q), nullptr, rq.grad_p0, 0,
                                                   WANT_POSE ? rq.pose_part + reg * row : nullptr, row, lds);
}

__global__ __launch_bounds__(AM_WAVES * WAVE) __attribute__((amdgpu_waves_per_eu(4))) void k_adjoint_series_batch(
    const BatchGeo* __restrict__ geos, const ra_batch_request* __restrict__ reqs, const int2* __restrict__ ipose,
    const int2* __restrict__ ivol, const int* __restrict__ counts, int nbin, int nbuf) {
    extern __shared__ float4 lds4[];
    float* lds = reinterpret_cast<float*>(lds4);
    const int lane = threadIdx.x & (WAVE - 1);
    const int np = counts[1], n = np + counts[2];
    int i = 0, end = 0;
    for (int unit = blockIdx.x;;) {
        if (i >= end) {
            if ((long long)unit * BATCH_UNIT >= n) break;
            i = unit * BATCH_UNIT;
            end = min(i + BATCH_UNIT, n);
            unit += gridDim.x;
        }
        const bool pose = i < np;
        const int2* list = pose ? ipose : ivol - np;         // indexed by i
        const int stop = pose ? min(end, np) : end;
        const int2 w = list[i];
        const int j = i + lane;
        const int2 v = list[min(j, stop - 1)];
        const unsigned long long other = __ballot(j >= stop || v.x != w.x || v.y != w.y + lane);
        const int cnt = __builtin_amdgcn_readfirstlane(other ? __builtin_ctzll(other) : WAVE);
        const int x = __builtin_amdgcn_readfirstlane(w.x), reg = __builtin_amdgcn_readfirstlane(w.y);
        const BatchGeo& bg = geos[x];
        i += cnt;
        if (bg.g.nbin > nbin) continue;                      // the LDS windows hold nbin bins
        const int cols = bg.g.rx * bg.g.ry;
        if (pose) {
            if (cols > 2 * AM_WAVES) batch_adjoint_run<4, false, true>(bg, reqs[x], reg, cnt, nbuf, lds);
            else if (cols > AM_WAVES) batch_adjoint_run<2, false, true>(bg, reqs[x], reg, cnt, nbuf, lds);
            else batch_adjoint_run<1, false, true>(bg, reqs[x], reg, cnt, nbuf, lds);
        } else {
            if (cols > 2 * AM_WAVES) batch_adjoint_run<4, true, false>(bg, reqs[x], reg, cnt, nbuf, lds);
            else if (cols > AM_WAVES) batch_adjoint_run<2, true, false>(bg, reqs[x], reg, cnt, nbuf, lds);
            else batch_adjoint_run<1, true, false>(bg, reqs[x], reg, cnt, nbuf, lds);
        }
    }
}

// Pose requests: element gradients summed over regions (FP64, fixed order), chained to
// (dL/dR, dL/dt), then to (dL/dw, dL/dt), followed by one Adam step on the pose.
// First stage of the pose update: the per-region element gradients of a pose request are
// summed in POSE_CHUNKS fixed chunks of regions, each into the chunk's first row (FP64, in
// region order), so that the per-request stage below adds POSE_CHUNKS rows instead of
// nreg.  A workgroup's threads take consecutive components of one chunk (coalesced rows).
constexpr int POSE_CHUNKS = 32;
__global__ __launch_bounds__(BATCH_THREADS) void k_batch_pose_chunks(const BatchGeo* __restrict__ geos,
                                                                     const ra_batch_request* __restrict__ reqs,
                                                                     const int* __restrict__ counts) {
    const int ns = counts[4];
    for (int it = blockIdx.x; it < ns * POSE_CHUNKS; it += gridDim.x) {
        const int slot = it / POSE_CHUNKS, c = it % POSE_CHUNKS;
        const ra_batch_request& q = reqs[slot];
        if (q.kind != RA_REQ_POSE) continue;
        const int n3 = 3 * geos[slot].g.E;
        const int cs = (q.nreg + POSE_CHUNKS - 1) / POSE_CHUNKS;
        const int r0 = c * cs, r1 = min(r0 + cs, q.nreg);
        if (r0 >= r1) continue;
        for (int t = threadIdx.x; t < n3; t += BATCH_THREADS) {
            double* col = q.pose_part + t;
            double a = 0.0;
#pragma unroll 4
            for (int rg = r0; rg < r1; ++rg) a += col[(size_t)rg * n3];
            col[(size_t)r0 * n3] = a;
        }
    }
}

__global__ __launch_bounds__(BATCH_THREADS) void k_batch_pose_update(const BatchGeo* __restrict__ geos,
                                                                     const ra_batch_request* __restrict__ reqs,
                                                                     const int* __restrict__ counts, int moment) {
    __shared__ double red[12][BATCH_THREADS];
    const int ns = counts[4];
    for (int slot = blockIdx.x; slot < ns; slot += gridDim.x) {
        const ra_batch_request& q = reqs[slot];
        if (moment && q.kind >= 0) {             // the loss: the elements' sums behind the moment table, in FP64
            const Geo& gl = geos[slot].g;
            const float* le = q.q + ((size_t)gl.E * (gl.K + 2 * gl.jt) + 1) * MOM_G;
            double a = 0.0;
            for (int e = threadIdx.x; e < gl.E; e += BATCH_THREADS) a += (double)le[e];
            red[0][threadIdx.x] = a;
            __syncthreads();
            for (int w = BATCH_THREADS / 2; w > 0; w >>= 1) {
                if ((int)threadIdx.x < w) red[0][threadIdx.x] += red[0][threadIdx.x + w];
                __syncthreads();
            }
            if (threadIdx.x == 0) q.loss[0] = (float)red[0][0];
            __syncthreads();
        }
        if (q.kind != RA_REQ_POSE) continue;
        const Geo& g = geos[slot].g;
        double acc[12];
        for (int i = 0; i < 12; ++i) acc[i] = 0.0;
        const int cs = (q.nreg + POSE_CHUNKS - 1) / POSE_CHUNKS;      // chunk sums from k_batch_pose_chunks
        for (int m = threadIdx.x; m < g.M; m += blockDim.x) {
            double ge[3] = {0.0, 0.0, 0.0};
            for (int rg = 0; rg < q.nreg; rg += cs) {
                const double* pp = q.pose_part + ((size_t)rg * g.E + m) * 3;
                ge[0] += pp[0]; ge[1] += pp[1]; ge[2] += pp[2];
            }
            const double* em = q.elem + 3 * m;
            for (int i = 0; i < 3; ++i) {
                for (int j = 0; j < 3; ++j) acc[3 * i + j] += ge[i] * em[j];
                acc[9 + i] += ge[i];
            }
        }
        for (int i = 0; i < 12; ++i) red[i][threadIdx.x] = acc[i];
        __syncthreads();
        for (int w = BATCH_THREADS / 2; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w)
                for (int i = 0; i < 12; ++i) red[i][threadIdx.x] += red[i][threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            double G[9], g6[6];
            for (int i = 0; i < 9; ++i) G[i] = red[i][0];
            so3_vjp(q.pose6, G, g6);
            g6[3] = red[9][0]; g6[4] = red[10][0]; g6[5] = red[11][0];
            double* st = q.adam;                 // m[6], v[6], step
            const double b1 = 0.9, b2 = 0.999, eps = 1e-8;     // torch.optim.Adam's defaults
            const double t = st[12] + 1.0;
            st[12] = t;
            const double c1 = 1.0 - pow(b1, t), c2 = 1.0 - pow(b2, t);
            for (int i = 0; i < 6; ++i) {
                st[i] = b1 * st[i] + (1.0 - b1) * g6[i];
                st[6 + i] = b2 * st[6 + i] + (1.0 - b2) * g6[i] * g6[i];
                const double lr = i < 3 ? q.lr_w : q.lr_t;
                q.pose6[i] -= lr * (st[i] / c1) / (sqrt(st[6 + i] / c2) + eps);
            }
        }
        __syncthreads();
    }
}

// Volume requests: p0 -= lr * dL/dp0 over the request's box (atomic: boxes may overlap).
__global__ __launch_bounds__(BLOCK) void k_batch_volume_apply(const BatchGeo* __restrict__ geos,
                                                              const ra_batch_request* __restrict__ reqs,
                                                              const int4* __restrict__ itab,
                                                              const int2* __restrict__ items,
                                                              const int* __restrict__ counts) {
    const int n = counts[2];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const int2 w = items[it];
        const Geo& g = geos[w.x].g;
        const ra_batch_request& q = reqs[w.x];
        const Region R = region_info(g, w.y);
        float* pbase = q.p0 + (size_t)R.i0 * g.vsx + (size_t)R.j0 * g.vsy + R.k0;
        const float* gbase = q.grad_p0 + (size_t)R.i0 * g.gsx + (size_t)R.j0 * g.gsy + R.k0;
        const float lr = (float)q.lr_w;
        for (int t = threadIdx.x; t < g.nvpad; t += blockDim.x) {
            const int4 ix = itab[t];
            if (!(ix.x < R.ni && ix.y < R.nj && ix.z < R.nk)) continue;
            atomicAdd(pbase + ix.w, -lr * gbase[ix.x * g.gsx + ix.y * g.gsy + ix.z]);
        }
    }
}

}  // namespace

// ==============================================================================================
// host side
// ==============================================================================================
struct ra_ctx {
    int device = 0;
    int* d_status = nullptr;
    char* arena = nullptr;                  // the context's scratch (grown by ensure_scratch)
    size_t arena_bytes = 0;
    char* static_scratch = nullptr;         // this device's static array (radiate_forward_static)
    // the moment forms' series for the last few samplings used, and that of the current call (10 to 22 us of host time to make
    // one, against calls of 20 us on: a program may go through several widths or profiles in turn)
    MomSeries series[8];
    int series_oldest = 0;
    const MomSeries* now = nullptr;
    unsigned long long* h_count = nullptr;  // pinned
    double* h_f64 = nullptr;                // pinned, one value
    double* d_f64 = nullptr;                // device, one value
    int sums_mode = RA_SUMS_AUTO;           // how the forward adds its partial rows (ra_set_forward_sums)
    std::string err;
};

namespace {

int fail(ra_ctx* ctx, int code, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return code;
}

#define RA_HIP(ctx, call)                                                                   \
    do {                                                                                    \
        hipError_t e_ = (call);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail(ctx, RA_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));  \
    } while (0)

bool finite_pos(double x) { return std::isfinite(x) && x > 0.0; }

// Window half-widths with a kernel compiled for exactly that many steps.  Others run
// the next larger generic kernel, which tests its last GEN_STEP steps.
#ifdef RA_FAST_BUILD
#define RA_EXACT_LIST(X) X(12) X(16)
#else
#define RA_EXACT_LIST(X) \
    X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20) X(21) X(22) X(23) X(24)
#endif
#define RA_GENERIC_LIST(X) X(8) X(16) X(24) X(32) X(40)
#ifdef RA_FAST_BUILD
#define RA_EXP_LIST(X) X(8) X(16) X(24) X(32) X(40)
#else
#define RA_EXP_LIST(X) X(4) X(8) X(12) X(16) X(20) X(24) X(28) X(32) X(36) X(40)
#endif
// Window bounds of the per-sample kernels of the other source profiles.

void choose_jt(int jout, int& jt, bool& exact) {
#define RA_TRY_EXACT(n) \
    if (jout == n) {    \
        jt = n;         \
        exact = true;   \
        return;         \
    }
    RA_EXACT_LIST(RA_TRY_EXACT)
#undef RA_TRY_EXACT
    exact = false;
    jt = -1;
#define RA_TRY_GENERIC(n) \
    if (jt < 0 && jout <= n) jt = n;
    RA_GENERIC_LIST(RA_TRY_GENERIC)
#undef RA_TRY_GENERIC
}

// Per-call plan.  The forward and the adjoint use different region sizes: the forward
// keeps only sample rows in LDS and can afford larger regions (fewer partial rows to
// add into HBM); the adjoint also keeps per-voxel dL/dp0 sums.
struct Plan {
    Geo g;              // adjoint regions (element gradients: per-region partials are kept, so larger)
    Geo ga;             // adjoint regions for dL/dp0 alone
    Geo gf;             // forward regions
    int jt;
    bool exact;
    int pair_d;         // forward takes voxels two at a time with this spread (0: one at a time)
    bool pair_ok;       // sampling and spacing allow pairs (regions with an even depth still needed)
    bool rowref;        // the dL/dp0-only adjoint may use the row-referenced form (adj_rowref)
    bool f64_sums;      // the forward adds its partial rows into FP64 sums (else FP32, straight into s)
    bool fm;            // the forward takes the moment form (k_forward_mom) on regions gm
    Geo gm;
    int fm_slices;      // workgroups that share a region's element chunks
    MomTerms terms;     // terms of the moment forms' series
    bool am, am_pose;   // dL/dp0 alone / the element gradients take the moment form
    Geo ga1, ga2;       // on regions ga1 (dL/dp0 alone) and ga2 (element gradients, with dL/dp0 or without)
    int am_nbuf[2];     // table windows in LDS, of each
    int part_rows;      // rows of element-gradient partials: a region's each, or in moment form a workgroup's
    size_t lds_fm;
    size_t lds_adj, lds_adj0, lds_fwd;
    // scratch layout (byte offsets)
    size_t off_xe, off_vtab, off_itab, off_vtab_a, off_itab_a, off_vtab_f, off_itab_f, off_part, off_ge, off_s,
        off_partial, off_nc, off_ncw, off_nct, off_s64, off_q, total;
    size_t kept;        // bytes a forward-only call reserves beyond what it needs: the adjoints' but for tables the row forms do without
};

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int validate(ra_ctx* ctx, const ra_grid* grid, int32_t M, int32_t F, const ra_sampling* samp) {
    if (!ctx) return RA_EINVAL;
    if (!grid || !samp) return fail(ctx, RA_EINVAL, "grid and sampling descriptors are required");
    if (grid->nx <= 0 || grid->ny <= 0 || grid->nz <= 0)
        return fail(ctx, RA_EINVAL, "grid dimensions must be positive");
    if ((long long)grid->nx * grid->ny * grid->nz >= (1LL << 31))
        return fail(ctx, RA_EINVAL, "grid has 2^31 or more voxels");
    if (!finite_pos(grid->spacing)) return fail(ctx, RA_EINVAL, "grid spacing must be finite and positive");
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(grid->origin[a])) return fail(ctx, RA_EINVAL, "grid origin must be finite");
    if (M <= 0 || F <= 0) return fail(ctx, RA_EINVAL, "M and F must be positive");
    if ((long long)M * F >= (1LL << 31)) return fail(ctx, RA_EINVAL, "M*F too large");
    if (samp->K <= 0) return fail(ctx, RA_EINVAL, "K must be positive");
    if (!finite_pos(samp->c) || !finite_pos(samp->fs) || !finite_pos(samp->sigma) || !finite_pos(samp->trunc))
        return fail(ctx, RA_EINVAL, "c, fs, sigma and trunc must be finite and positive");
    double delta = samp->c / samp->fs;
    double tsig = samp->trunc * samp->sigma;
    if (tsig < 0.5 * delta) return fail(ctx, RA_EINVAL, "trunc*sigma must be at least half a sample length");
    int jout = (int)std::floor(tsig / delta + 0.5);
    if (jout > JMAX) return fail(ctx, RA_EINVAL, "trunc*sigma exceeds 40 sample lengths");
    if (samp->kernel < RA_KERNEL_GAUSSIAN || samp->kernel > RA_KERNEL_UNIFORM)
        return fail(ctx, RA_EINVAL, "unknown source profile (kernel)");
    if (samp->kernel == RA_KERNEL_POWER && !(std::isfinite(samp->nu) && samp->nu > 0.5))
        return fail(ctx, RA_EINVAL, "power-law exponent nu must be finite and above 1/2");
    return RA_OK;
}

// Region size: the largest candidate box whose LDS footprint (sample rows of every
// wavefront, plus per-voxel sums for the adjoint) fits the byte budget per workgroup.
size_t set_regions(Geo& g, const ra_grid* grid, double delta, int jt, bool with_gsum, int extra_rows,
                   size_t budget) {
    static const int cand[][3] = {{8, 8, 16}, {8, 8, 8}, {4, 8, 8}, {4, 4, 8}, {4, 4, 4},
                                  {2, 4, 4},  {2, 2, 4}, {2, 2, 2}, {1, 1, 2}, {1, 1, 1}};
    size_t lds = 0;
    for (const auto& c : cand) {
        int rx = std::min(c[0], g.nx), ry = std::min(c[1], g.ny), rz = std::min(c[2], g.nz);
        double rad = 0.5 * grid->spacing *
                     std::sqrt((double)(rx - 1) * (rx - 1) + (double)(ry - 1) * (ry - 1) + (double)(rz - 1) * (rz - 1));
        int jclamp = (int)std::ceil(rad / delta * (1.0 + 1e-6)) + 1;
        int L = 2 * (jclamp + jt) + 1 + extra_rows;
        int nvpad = (rx * ry * rz + 3) & ~3;
        lds = (size_t)WAVES * L * WAVE * sizeof(float) + (with_gsum ? (size_t)WAVES * nvpad * sizeof(float) : 0);
        g.rx = rx; g.ry = ry; g.rz = rz;
        g.nvpad = nvpad;
        g.jclamp = jclamp;
        g.jclampf = (float)jclamp;
        g.kmargin = jclamp + jt;
        g.L = L;
        if (lds <= budget) break;
    }
    g.nrx = (g.nx + g.rx - 1) / g.rx;
    g.nry = (g.ny + g.ry - 1) / g.ry;
    g.nrz = (g.nz + g.rz - 1) / g.rz;
    g.nreg = g.nrx * g.nry * g.nrz;
    return lds;
}

// This sampling's series, kept in the context with those of the last seven others.
const MomSeries& series_of(ra_ctx* ctx, const ra_sampling* samp, bool exact) {
    const double key[4] = {(double)samp->kernel + (exact ? 0.5 : 0.0), samp->c / samp->fs / samp->sigma, samp->trunc, samp->nu};
    for (const MomSeries& m : ctx->series)
        if (std::memcmp(key, m.key, sizeof(key)) == 0) return *(ctx->now = &m);
    constexpr int kept = sizeof(ctx->series) / sizeof(ctx->series[0]);
    MomSeries& m = ctx->series[ctx->series_oldest];
    ctx->series_oldest = (ctx->series_oldest + 1) % kept;
    ctx->now = &m;
    make_series(samp, exact, m);
    std::memcpy(m.key, key, sizeof(key));
    return m;
}

// Moment forms: lengths in units of delta / 2.
void set_units(Geo& g, const ra_grid* grid, double delta) {
    const double unit = 2.0 / delta;
    g.unit_h = (float)unit;
    g.unit_l = (float)(unit - (double)g.unit_h);
    g.hs_u = (float)(grid->spacing * unit);
    g.hs_l = (float)(grid->spacing * unit - (double)g.hs_u);
}

void set_terms(Geo& g, const MomTerms& t) {
    g.xkind = t.xkind;
    g.thr = t.thr;
    g.flip = t.flip;
    for (int i = 0; i < 4; ++i) g.ev[i] = t.ev[i];
    g.es = t.es;
    g.kx = t.kx;
}

// Estimated cycles of the Gaussian's row-form forward: its wavefronts take 57 cycles per voxel and window row (32 where voxels
// go in pairs), a third of that hidden behind the atomics of other workgroups, of which the chip does 108 a cycle; and 20 us
// of start-up.  Within 25 % of what 30 calls took (spacings 0.05 to 1.2 mm, widths 0.06 to 0.15 mm, 64 and 256 elements).
double row_forward_cost(const Geo& g, int jt, int pair_d) {
    const double rows = 2.0 * jt + 1 + pair_d, chunks = (g.E + WAVE - 1) / WAVE;
    const double work = std::ceil(g.nreg / 512.0) * std::ceil(chunks / WAVES) * g.nvpad * rows * (pair_d ? 32.0 : 57.0);
    return 48000.0 + 0.7 * work + (double)g.nreg * g.E * g.L / 108.0;
}

// The moment-form forward of a call, with nm terms: on which regions.
// Those that make the estimated time least.  Per pair and wavefront a CU spends about 34 cycles on the
// adds; per region and chunk the expansion takes row tiles x quads x NM matrix instructions of 32 cycles
// on each SIMD (measured: 1.45 times that, with the operand conversions and the atomics), and barriers and
// clearing about 2500 cycles where one workgroup has the CU, 800 where two share it.  Large grids take
// 16x16x16; a box of 32^3 voxels seen by one chunk takes small ones, which fill the chip.  Coarse spacings leave regions of
// few voxels, for each of which a window is expanded: there the Gaussian's row form is the faster one, and is taken where
// its estimate is below 1.1 times this one's with 17 us a workgroup for references, bounds and clearing (sigma 0.1 mm, 40^3
// voxels, 256 elements: 69 us against 150 in rows at 0.25 mm, 354 against 366 at 0.46, 1263 against 375 at 0.5).
void plan_forward_mom(const ra_grid* grid, const ra_sampling* samp, const MomTerms& mt, Plan& P) {
    P.fm = false;
    const int nm = mt.fwd;
    if (!nm) return;
    const double delta = samp->c / samp->fs;
    const int jt = (int)std::floor(samp->trunc * samp->sigma / delta + 0.5);
    static const int cand[][3] = {{16, 16, 16}, {16, 16, 8}, {8, 16, 8}, {8, 8, 16}, {8, 8, 8}, {4, 8, 8},
                                  {4, 4, 8},    {2, 4, 8},   {2, 2, 8},  {1, 2, 8},  {1, 1, 8}};
    const int nchunk = (P.g.E + WAVE - 1) / WAVE;
    double best = 0.0, start = 0.0;
    for (const auto& cd : cand) {
        Geo g = P.g;
        // as many regions along x and y as the candidate's size gives, of even size
        g.nrx = (g.nx + cd[0] - 1) / cd[0]; g.nry = (g.ny + cd[1] - 1) / cd[1]; g.nrz = (g.nz + cd[2] - 1) / cd[2];
        g.rx = (g.nx + g.nrx - 1) / g.nrx; g.ry = (g.ny + g.nry - 1) / g.nry; g.rz = std::min(cd[2], g.nz);
        const double rad = 0.5 * grid->spacing * std::sqrt((double)(g.rx - 1) * (g.rx - 1) + (double)(g.ry - 1) * (g.ry - 1) +
                                                           (double)(g.rz - 1) * (g.rz - 1));
        if (rad / delta > 1e4) continue;                   // never fits; keeps the bin count an int
        g.jclamp = (int)std::ceil(rad / delta * (1.0 + 1e-6)) + 1;
        g.jclampf = (float)g.jclamp;
        g.jt = jt;
        g.nbin = 2 * g.jclamp + 1;
        const size_t lds = fm_lds(nm, g.nbin, jt, mt.xkind != 0);
        if (lds > 160 * 1024) continue;
        g.nrx = (g.nx + g.rx - 1) / g.rx; g.nry = (g.ny + g.ry - 1) / g.ry;
        g.nreg = g.nrx * g.nry * g.nrz;
        const int per_cu = lds <= LDS_FM_BUDGET ? 2 : 1;
        const int slices = std::min(nchunk, std::max(1, (2048 + g.nreg - 1) / g.nreg));
        const double expand = ((g.nbin + 2 * jt + 15) / 16) * ((2 * jt + 19) / 4) * nm * 32.0 * 1.45;
        const int zl = g.nz - (g.nrz - 1) * g.rz;          // columns run in steps of FM_RZ voxels
        const double zpad = (g.nrz - 1.0) * ((g.rz + FM_RZ - 1) / FM_RZ * FM_RZ) + (zl + FM_RZ - 1) / FM_RZ * FM_RZ;
        const double pairs = (double)g.nx * g.ny * zpad / g.nreg * 34.0;
        const double each = pairs + expand + (per_cu == 2 ? 800.0 : 2500.0);   // CU cycles per region and chunk
        const double wgs = (double)g.nreg * slices, per_wg = (double)((nchunk + slices - 1) / slices);
        // the last round of workgroups; a CU with one where two fit runs it about 1.6 times as fast
        const double full = std::floor(wgs / (256.0 * per_cu)), left = wgs - full * 256.0 * per_cu;
        const double last = left == 0.0 ? 0.0 : (left <= 256.0 && per_cu == 2 ? 0.62 : 1.0);
        const double cost = (full + last) * per_cu * per_wg * each;
        if (P.fm && cost >= best) continue;
        best = cost;
        start = (full + last) * 40000.0;
        P.fm = true;
        P.gm = g;
        P.fm_slices = slices;
        P.lds_fm = lds;
    }
    if (samp->kernel == RA_KERNEL_GAUSSIAN && best + start > 0.9 * row_forward_cost(P.gf, P.jt, P.pair_d)) P.fm = false;
    if (!P.fm) return;
    set_units(P.gm, grid, delta);
    set_terms(P.gm, mt);
}

// Estimated cycles of the Gaussian's row-form adjoints: 46 per voxel and window row of a wavefront and 600 per row staged, and
// 20 us of start-up; `slots` workgroups run at once.
double row_adjoint_cost(const Geo& g, int jt, double slots) {
    const double chunks = (g.E + WAVE - 1) / WAVE;
    return 48000.0 + std::ceil(g.nreg / slots) * std::ceil(chunks / WAVES) * (g.nvpad * (2.0 * jt + 1) * 46.0 + g.L * 600.0);
}

// The moment-form adjoint's regions: columns of up to 8 voxels, up to 64 of them, those that make the estimated
// time least (`pair`: CU cycles per pair and wavefront, 30 for dL/dp0, 44 with the element gradients).  Two
// table windows in LDS let a chunk's loads run behind the previous chunk's voxels; where the spacing is so
// coarse that only one fits, the loads (about 41 cycles per bin, and their latency) add to the time.  Columns of 4 and 2
// voxels cost what one of 8 does, and are for spacings where the table window of 8 would not fit (40^3 voxels of 0.42 mm,
// 256 elements: the row form took 528 us, these 107).  `rows`: the row form's estimate; it keeps the call where 1.5 times
// this one's and 15 us exceed it, as with narrow Gaussians (19 rows) at coarse spacings: sigma 0.06 mm at 0.42 mm, element
// gradients 107 us in rows and 132 in moments, at 0.3 mm 103 and 76.
bool plan_adjoint_mom(const ra_grid* grid, const ra_sampling* samp, const Geo& base, double pair, int nq, bool edge, double rows,
                      Geo& out, int& nbuf) {
    // with edge terms whole columns only, which are the forward's
    static const int cand[][3] = {{8, 8, 8}, {4, 8, 8}, {4, 4, 8}, {2, 4, 8}, {2, 2, 8}, {1, 2, 8}, {1, 1, 8}, {8, 8, 4}, {4, 8, 4},
                                  {4, 4, 4}, {2, 4, 4}, {2, 2, 4}, {4, 4, 2}, {2, 4, 2}, {2, 2, 2}, {1, 2, 2}, {1, 1, 2}, {1, 1, 1}};
    const double delta = samp->c / samp->fs;
    const int nchunk = (base.E + WAVE - 1) / WAVE;
    double best = 0.0;
    bool found = false;
    for (const auto& cd : cand) {
        if (edge && cd[2] < FM_RZ) break;
        Geo g = base;
        g.nrx = (g.nx + cd[0] - 1) / cd[0]; g.nry = (g.ny + cd[1] - 1) / cd[1]; g.nrz = (g.nz + cd[2] - 1) / cd[2];
        g.rx = (g.nx + g.nrx - 1) / g.nrx; g.ry = (g.ny + g.nry - 1) / g.nry; g.rz = std::min(cd[2], g.nz);
        g.nrx = (g.nx + g.rx - 1) / g.rx; g.nry = (g.ny + g.ry - 1) / g.ry;
        g.nreg = g.nrx * g.nry * g.nrz;
        const double rad = 0.5 * grid->spacing * std::sqrt((double)(g.rx - 1) * (g.rx - 1) + (double)(g.ry - 1) * (g.ry - 1) +
                                                           (double)(g.rz - 1) * (g.rz - 1));
        if (rad / delta > 1e4) continue;
        g.jclamp = (int)std::ceil(rad / delta * (1.0 + 1e-6)) + 1;
        g.jclampf = (float)g.jclamp;
        g.jt = (int)std::floor(samp->trunc * samp->sigma / delta + 0.5);
        g.nbin = 2 * g.jclamp + 1;
        const int xrows = edge ? g.nbin + 2 * g.jt : 0;
        const int nb = am_lds(g.nbin, nq, xrows, 2) <= 160 * 1024 ? 2 : 1;
        if (am_lds(g.nbin, nq, xrows, nb) > 160 * 1024) continue;
        const int cols = (g.rx * g.ry + AM_WAVES - 1) / AM_WAVES * AM_WAVES;     // a round of wavefronts is the least
        const double each = cols * FM_RZ * pair + 900.0 + (nb == 1 ? 1500.0 + 41.0 * g.nbin : 0.0);
        const double cost = std::ceil(g.nreg / (double)NCU) * (nchunk * each + 3000.0) + 5000.0;
        if (found && cost >= best) continue;
        best = cost;
        found = true;
        out = g;
        nbuf = nb;
    }
    if (1.5 * best + 36000.0 > rows) found = false;
    if (found) set_units(out, grid, delta);
    return found;
}

// Calls that return the sum of the elements' negative correlations: that sum is signed and may cancel to 1e-3 of its
// terms or less, where what the two forms of the forward round differently (1e-6 of a signal) shows in its digits
// (boxes of 36 to 82 voxels a side, 24 to 106 elements: up to 9e-5 of the sum, above 2e-5 for 4 of 150 inputs; row
// form against itself 2e-6).  They keep the row form, so that their losses compare with recorded ones, and with edge
// terms the adjoints' row forms, which decide the window's edge as that forward does.  Scores and gradients
// without the sum take the moment forms.
constexpr unsigned PLAN_ROW_FORWARD = 1u;
constexpr unsigned PLAN_NO_TABLE = 2u;     // adjoints without a moment table (see plan_call)

// The context keeps the moment forms' series; without one (the batched step) the plan has the row forms only.
void make_plan(ra_ctx* ctx, const ra_grid* grid, int32_t M, int32_t F, const ra_sampling* samp, Plan& P,
               int sums_mode = RA_SUMS_AUTO, unsigned only = 0) {
    Geo& g = P.g;
    std::memset(&g, 0, sizeof(g));
    g.nx = grid->nx; g.ny = grid->ny; g.nz = grid->nz;
    g.vsx = (long long)grid->ny * grid->nz;
    g.vsy = grid->nz;
    g.gsx = g.vsx;
    g.gsy = g.vsy;
    g.K = samp->K; g.M = M; g.F = F; g.E = M * F;
    const double delta = samp->c / samp->fs;
    const double sigma = samp->sigma;
    const double tsig = samp->trunc * sigma;
    const int jout = (int)std::floor(tsig / delta + 0.5);
    choose_jt(jout, P.jt, P.exact);
    g.ktype = samp->kernel;
    if (g.ktype != RA_KERNEL_GAUSSIAN) {
        P.exact = false;
        if (g.ktype == RA_KERNEL_EXPONENTIAL) {
            // factorised legs (fwd_pair_exp): the smallest listed window bound, tables of
            // G_j = exp(-j delta/w)
            P.jt = -1;
#define RA_TRY_EXP(n) \
    if (P.jt < 0 && jout <= n) P.jt = n;
            RA_EXP_LIST(RA_TRY_EXP)
#undef RA_TRY_EXP
        } else {
            // per-sample kernels with a run-time window of jout steps either side
            P.jt = jout;
        }
        g.jwin = jout;
        const double log2e = 1.4426950408889634;
        g.kexp = (float)(-log2e / sigma);
        g.kinv_w = (float)(1.0 / sigma);
        g.kinv_w2 = (float)(1.0 / (sigma * sigma));
        g.knu = (float)(-samp->nu);
        g.k2nu = (float)(2.0 * samp->nu);
    }
    g.edge = (float)(P.jt * delta - tsig);
    g.jin = (int)std::floor(tsig / delta - 0.5);
    for (int a = 0; a < 3; ++a) {
        g.org_h[a] = (float)grid->origin[a];
        g.org_l[a] = (float)(grid->origin[a] - (double)g.org_h[a]);
    }
    g.sp_h = (float)grid->spacing;
    g.sp_l = (float)(grid->spacing - (double)g.sp_h);
    g.dlt_h = (float)delta;
    g.dlt_l = (float)(delta - (double)g.dlt_h);
    g.inv_dlt = (float)(1.0 / delta);
    g.tsig = (float)tsig;
    const double log2e = 1.4426950408889634;
    g.kappa = (float)(-log2e / (2.0 * sigma * sigma));
    g.alpha = (float)(log2e * delta / (sigma * sigma));
    g.inv_s2 = (float)(1.0 / (sigma * sigma));
    g.gmin = (float)(10.0 * sigma);
    for (int j = 0; j <= JMAX; ++j) {
        double gj = g.ktype == RA_KERNEL_EXPONENTIAL ? std::exp(-(double)j * delta / sigma)
                                                     : std::exp(-(double)j * j * delta * delta / (2.0 * sigma * sigma));
        g.gam[j] = (float)gj;
        g.jdg[j] = (float)(j * delta * gj);
        g.jjdg[j] = (float)((j * delta) * (j * delta) * gj);
    }
    for (int m = 0; m <= RS_MAX; ++m) {
        g.gamr[m] = (float)std::exp(-(double)m * m * delta * delta / (2.0 * sigma * sigma));
    }
    // Paired forward: z-neighbours (distance h) have centre samples at most D apart when
    // h < D delta.
    P.pair_d = 0;
    P.pair_ok = P.exact && g.ktype == RA_KERNEL_GAUSSIAN && grid->spacing <= (PAIR_D - 0.01) * delta;
    if (P.pair_ok) P.pair_d = PAIR_D;
    P.gf = g;
    P.ga = g;
    P.lds_adj = set_regions(g, grid, delta, P.jt, true, 0, LDS_ADJ_BUDGET);
    P.lds_adj0 = set_regions(P.ga, grid, delta, P.jt, true, 0, LDS_ADJ0_BUDGET);
    // Row-referenced dL/dp0 adjoint: its factors reach exp(+-(kmargin + 1)^2 (delta/sigma)^2 / 2)
    // (Hc^(2 JT), E_c Hc^mlow and Gamma_m at the window's ends), which must stay well inside the
    // FP32 range (e^88); the staged window is normalised to [1/2, 1).
    {
        const double km = P.ga.kmargin + 1.0, ds = delta / sigma;
        P.rowref = P.exact && g.ktype == RA_KERNEL_GAUSSIAN && P.ga.kmargin <= RS_MAX && km * km * ds * ds / 2.0 <= 75.0;
    }
    P.lds_fwd = set_regions(P.gf, grid, delta, P.jt, false, P.pair_d, LDS_FWD_BUDGET);
    // pairs are (k, k+1) of the visiting order, so the forward region needs an even rz
    if (P.pair_d && (P.gf.rz & 1)) {
        P.pair_d = 0;
        P.lds_fwd = set_regions(P.gf, grid, delta, P.jt, false, 0, LDS_FWD_BUDGET);
    }
    // Profiles that do not vanish at the window edge (RA_KERNEL_* other than the Gaussian): the
    // dL/dp0 adjoint takes the forward's regions where they fit its LDS budget, so that both compute
    // every pair's u from the same reference, bit for bit, and decide its window edge alike (then
    // <A p0, r> = <p0, A^T r> holds to summation rounding; with other regions an edge term within
    // rounding of the edge can fall in on one side and out on the other).
    if (g.ktype != RA_KERNEL_GAUSSIAN) {
        Geo ga2 = P.ga;
        const size_t lds2 = set_regions(ga2, grid, delta, P.jt, true, 0, LDS_FWD_BUDGET);
        if (lds2 <= LDS_FWD_BUDGET && ga2.rx == P.gf.rx && ga2.ry == P.gf.ry && ga2.rz == P.gf.rz) {
            P.ga = ga2;
            P.lds_adj0 = lds2;
        }
    }
    // FP32 rounding of the forward's sums grows with the number of regions whose partial rows
    // meet in one sample; past FWD_F32_MAX_REGIONS forward regions the rows go into FP64 sums.
    P.f64_sums = sums_mode == RA_SUMS_F64 || (sums_mode == RA_SUMS_AUTO && P.gf.nreg > FWD_F32_MAX_REGIONS);

    static const MomTerms none{};
    const MomTerms& mt = ctx ? series_of(ctx, samp, P.exact).terms : none;
    P.terms = mt;
    P.fm = P.am = P.am_pose = false;
    if (mt.fwd) {
        const bool x = mt.xkind != 0;
        plan_forward_mom(grid, samp, mt, P);
        // Up to 48 bytes of table per sample of dL/ds, where the row forms need none: beyond AM_TABLE_MAX those
        // serve the other profiles and narrow Gaussians, so that a sweep whose signals fill the memory still has
        // room.  Wider Gaussians have always taken a table: their row form is 3 times slower.
        const size_t table = (size_t)g.E * (g.K + 2 * jout) * am_nq(MOM_MAX) * sizeof(float4);
        const bool room = !(only & PLAN_NO_TABLE) &&
                          (table <= AM_TABLE_MAX || (g.ktype == RA_KERNEL_GAUSSIAN && delta <= WIDE_GAUSS * sigma));
        const double any = INFINITY;
        P.am = room && mt.vol && plan_adjoint_mom(grid, samp, g, x ? 45.0 : 30.0, am_nq(mt.vol), x,
                                                  x ? any : row_adjoint_cost(P.ga, P.jt, 768.0), P.ga1, P.am_nbuf[0]);
        P.am_pose = room && mt.pose && plan_adjoint_mom(grid, samp, g, x ? 60.0 : 43.0, am_nq(mt.pose), x,
                                                        x ? any : row_adjoint_cost(g, P.jt, 512.0), P.ga2, P.am_nbuf[1]);
        set_terms(P.ga1, mt);
        set_terms(P.ga2, mt);
        // with edge terms the forward and the dL/dp0 adjoint take the same form, so that they decide the edges alike
        if (x && !(P.fm && P.am)) P.fm = P.am = P.am_pose = false;
        if (only & PLAN_ROW_FORWARD) {
            P.fm = false;
            if (x) P.am = P.am_pose = false;
        }
    }
    P.part_rows = P.am_pose ? std::min(P.ga2.nreg, NCU) : g.nreg;

    size_t o = 0;
    P.off_xe = o; o = align_up(o + (size_t)g.E * 6 * sizeof(float));
    P.off_vtab = o; o = align_up(o + (size_t)g.nvpad * sizeof(float4));
    P.off_itab = o; o = align_up(o + (size_t)g.nvpad * sizeof(int4));
    P.off_vtab_a = o; o = align_up(o + (size_t)P.ga.nvpad * sizeof(float4));
    P.off_itab_a = o; o = align_up(o + (size_t)P.ga.nvpad * sizeof(int4));
    P.off_vtab_f = o; o = align_up(o + (size_t)P.gf.nvpad * sizeof(float4));
    P.off_itab_f = o; o = align_up(o + (size_t)P.gf.nvpad * sizeof(int4));
    P.off_part = o; o = align_up(o + (size_t)P.part_rows * g.E * 3 * sizeof(double));
    P.off_ge = o; o = align_up(o + (size_t)g.E * 3 * sizeof(double));
    P.off_s = o; o = align_up(o + (size_t)g.E * g.K * sizeof(float));
    P.off_partial = o; o = align_up(o + RESID_BLOCKS * sizeof(float));
    P.off_nc = o; o = align_up(o + (size_t)g.E * sizeof(double));
    P.off_ncw = o; o = align_up(o + (size_t)g.E * sizeof(double));
    P.off_nct = o; o = align_up(o + sizeof(double));
    P.off_s64 = o; o = align_up(o + (P.f64_sums ? (size_t)g.E * g.K * sizeof(double) : 0));
    const int nq = std::max(P.am ? am_nq(mt.vol) : 0, P.am_pose ? am_nq(mt.pose) : 0);
    P.off_q = o; o = align_up(o + ((size_t)g.E * (g.K + 2 * jout) + 1) * nq * sizeof(float4));
    P.total = o;
    const bool own = g.ktype == RA_KERNEL_GAUSSIAN && delta <= WIDE_GAUSS * sigma;
    P.kept = own || nq == 0 ? o : P.off_q + align_up((size_t)g.nreg * g.E * 3 * sizeof(double));
}

int ensure_scratch(ra_ctx* ctx, size_t bytes, hipStream_t stream) {
    if (bytes <= ctx->arena_bytes) return RA_OK;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
        return fail(ctx, RA_ENOMEM, "scratch must be reserved (ra_reserve) before stream capture");
    RA_HIP(ctx, hipStreamSynchronize(stream));
    if (ctx->arena) RA_HIP(ctx, hipFree(ctx->arena));
    ctx->arena = nullptr;
    ctx->arena_bytes = 0;
    if (hipMalloc(&ctx->arena, bytes) != hipSuccess) {
        ctx->arena = nullptr;
        (void)hipGetLastError();
        return fail(ctx, RA_ENOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes of scratch failed");
    }
    ctx->arena_bytes = bytes;
    return RA_OK;
}

// Plan of a call with an adjoint, and its scratch.  Where there is no room for the moment table (up to 48 bytes per
// sample of dL/ds), the row forms, which need none, take the call.
int plan_call(ra_ctx* ctx, const ra_grid* grid, int32_t M, int32_t F, const ra_sampling* samp, Plan& P, hipStream_t stream,
              unsigned only = 0) {
    make_plan(ctx, grid, M, F, samp, P, ctx->sums_mode, only);
    int rc = ensure_scratch(ctx, P.total, stream);
    if (rc != RA_ENOMEM || !(P.am || P.am_pose)) return rc;
    make_plan(ctx, grid, M, F, samp, P, ctx->sums_mode, only | PLAN_NO_TABLE);
    if ((rc = ensure_scratch(ctx, P.total, stream)) == RA_OK) ctx->err.clear();
    return rc;
}

// Allow a kernel the full LDS of a CU, once per kernel (so not again under stream capture).
template <typename K>
hipError_t allow_full_lds(K kern) {
    static std::mutex mu;
    static std::set<const void*> done;
    const void* f = (const void*)kern;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count(f)) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e == hipSuccess) done.insert(f);
    return e;
}

template <typename T>
T* at(ra_ctx* ctx, size_t off) {
    return reinterpret_cast<T*>(ctx->arena + off);
}

template <typename T>
T* at(char* base, size_t off) {
    return reinterpret_cast<T*>(base + off);
}

int prologue(ra_ctx* ctx, char* base, const ra_grid* grid, const Plan& P, const double* elem, const double* poses,
             hipStream_t stream, bool forward_only = false) {
    const Geo& g = P.g;
    float3 lo = make_float3((float)grid->origin[0], (float)grid->origin[1], (float)grid->origin[2]);
    float3 hi = make_float3((float)(grid->origin[0] + (g.nx - 1) * grid->spacing),
                            (float)(grid->origin[1] + (g.ny - 1) * grid->spacing),
                            (float)(grid->origin[2] + (g.nz - 1) * grid->spacing));
    hipLaunchKernelGGL(k_elements, dim3((g.E + 255) / 256), dim3(256), 0, stream, g, elem, poses,
                       at<float>(base, P.off_xe), ctx->d_status, lo, hi);
    if (!forward_only && !P.am_pose)
        hipLaunchKernelGGL(k_voxel_table, dim3((g.nvpad + 255) / 256), dim3(256), 0, stream, g,
                           at<float4>(base, P.off_vtab), at<int4>(base, P.off_itab));
    if (!forward_only && !P.am) {
        hipLaunchKernelGGL(k_voxel_table, dim3((P.ga.nvpad + 255) / 256), dim3(256), 0, stream, P.ga,
                           at<float4>(base, P.off_vtab_a), at<int4>(base, P.off_itab_a));
    }
    if (!P.fm)
        hipLaunchKernelGGL(k_voxel_table, dim3((P.gf.nvpad + 255) / 256), dim3(256), 0, stream, P.gf,
                           at<float4>(base, P.off_vtab_f), at<int4>(base, P.off_itab_f));
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

// Scratch layout of a forward-only call (element positions, the forward's voxel tables and, with
// FP64 sums, the sums): the offsets of P the forward reads, rewritten from 0; returns the bytes.
size_t forward_layout(Plan& P) {
    size_t o = 0;
    P.off_xe = o; o = align_up(o + (size_t)P.g.E * 6 * sizeof(float));
    P.off_vtab_f = o; o = align_up(o + (size_t)P.gf.nvpad * sizeof(float4));
    P.off_itab_f = o; o = align_up(o + (size_t)P.gf.nvpad * sizeof(int4));
    P.off_s64 = o; o = align_up(o + (P.f64_sums ? (size_t)P.g.E * P.g.K * sizeof(double) : 0));
    return o;
}

// Device address of this device's static scratch array, resolved once per device (the
// current device must be `device`).
hipError_t static_scratch_of(int device, char** out) {
    static std::mutex mu;
    static std::map<int, char*> addr;
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(device);
    if (it == addr.end()) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        it = addr.emplace(device, static_cast<char*>(p)).first;
    }
    *out = it->second;
    return hipSuccess;
}

template <int JT, bool EXACT, int D, int KT = RA_KERNEL_GAUSSIAN>
int launch_forward_t(ra_ctx* ctx, char* base, const Plan& P, const float* p0, float* s, hipStream_t stream) {
    const size_t n = (size_t)P.g.E * P.g.K;
    if (!P.f64_sums) {
        auto kern = k_forward<JT, EXACT, D, KT, float>;
        RA_HIP(ctx, allow_full_lds(kern));
        hipLaunchKernelGGL(k_fill, dim3(1024), dim3(256), 0, stream, s, n, 0.0f);
        hipLaunchKernelGGL(kern, dim3(P.gf.nreg), dim3(BLOCK), P.lds_fwd, stream, P.gf, p0,
                           at<float>(base, P.off_xe), at<float4>(base, P.off_vtab_f), at<int4>(base, P.off_itab_f), s);
        RA_HIP(ctx, hipGetLastError());
        return RA_OK;
    }
    auto kern = k_forward<JT, EXACT, D, KT, double>;
    RA_HIP(ctx, allow_full_lds(kern));
    double* s64 = at<double>(base, P.off_s64);
    hipLaunchKernelGGL(k_fill_f64, dim3(1024), dim3(256), 0, stream, s64, n);
    hipLaunchKernelGGL(kern, dim3(P.gf.nreg), dim3(BLOCK), P.lds_fwd, stream, P.gf, p0, at<float>(base, P.off_xe),
                       at<float4>(base, P.off_vtab_f), at<int4>(base, P.off_itab_f), s64);
    hipLaunchKernelGGL(k_to_f32, dim3(1024), dim3(256), 0, stream, s64, n, s);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

template <int NM, int NW, int X>
int launch_forward_mom(ra_ctx* ctx, char* base, const Plan& P, const float* p0, float* s, hipStream_t stream) {
    const size_t n = (size_t)P.g.E * P.g.K;
    const dim3 grid((unsigned)(P.gm.nreg * P.fm_slices)), block(NW * WAVE);
    const float* xe = at<float>(base, P.off_xe);
    if (!P.f64_sums) {
        auto kern = k_forward_mom<NM, NW, X, float>;
        RA_HIP(ctx, allow_full_lds(kern));
        hipLaunchKernelGGL(k_fill, dim3(1024), dim3(256), 0, stream, s, n, 0.0f);
        hipLaunchKernelGGL(kern, grid, block, P.lds_fm, stream, P.gm, ctx->now->fwd, P.fm_slices, p0, xe, s);
        RA_HIP(ctx, hipGetLastError());
        return RA_OK;
    }
    auto kern = k_forward_mom<NM, NW, X, double>;
    RA_HIP(ctx, allow_full_lds(kern));
    double* s64 = at<double>(base, P.off_s64);
    hipLaunchKernelGGL(k_fill_f64, dim3(1024), dim3(256), 0, stream, s64, n);
    hipLaunchKernelGGL(kern, grid, block, P.lds_fm, stream, P.gm, ctx->now->fwd, P.fm_slices, p0, xe, s64);
    hipLaunchKernelGGL(k_to_f32, dim3(1024), dim3(256), 0, stream, s64, n, s);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

// Kernels with a listed window bound JT test only their last GEN_STEP (Gaussian) or
// EXP_STEP (exponential) steps, which needs every earlier step inside the window.
bool generic_bound_ok(const Plan& P) {
    if (P.g.ktype == RA_KERNEL_EXPONENTIAL) return P.g.jin >= P.jt - EXP_STEP;
    return P.exact || P.g.ktype != RA_KERNEL_GAUSSIAN || P.g.jin >= P.jt - GEN_STEP;
}

int launch_forward(ra_ctx* ctx, char* base, const Plan& P, const float* p0, float* s, hipStream_t stream) {
    if (P.fm) {
        const bool big = P.lds_fm > LDS_FM_BUDGET;
#define RA_CASE(n, x)                                                                    \
    if (P.terms.fwd == n && P.terms.xkind == x)                                          \
        return big ? launch_forward_mom<n, FM_WAVES_BIG, x>(ctx, base, P, p0, s, stream) \
                   : launch_forward_mom<n, FM_WAVES, x>(ctx, base, P, p0, s, stream);
        RA_CASE(6, 0) RA_CASE(7, 0) RA_CASE(8, 0)
        RA_CASE(8, 1) RA_CASE(10, 1) RA_CASE(12, 1) RA_CASE(6, 2) RA_CASE(8, 2)
#undef RA_CASE
    }
    if (!generic_bound_ok(P)) return fail(ctx, RA_ENOTSUP, "window half-width not supported");
    // other profiles; the per-sample kernels index from the centre row kmargin (JT = 0)
    switch (P.g.ktype) {
        case RA_KERNEL_EXPONENTIAL:
#define RA_CASE(n) \
    if (P.jt == n) return launch_forward_t<n, false, 0, RA_KERNEL_EXPONENTIAL>(ctx, base, P, p0, s, stream);
            RA_EXP_LIST(RA_CASE)
#undef RA_CASE
            break;
        case RA_KERNEL_POWER:
            if (P.g.knu == -2.0f) return launch_forward_t<0, false, 0, KT_POWER2>(ctx, base, P, p0, s, stream);
            return launch_forward_t<0, false, 0, RA_KERNEL_POWER>(ctx, base, P, p0, s, stream);
        case RA_KERNEL_UNIFORM: return launch_forward_t<0, false, 0, RA_KERNEL_UNIFORM>(ctx, base, P, p0, s, stream);
        default: break;
    }
#define RA_CASE(n)                                                                       \
    if (P.exact && P.jt == n)                                                            \
        return P.pair_d ? launch_forward_t<n, true, PAIR_D>(ctx, base, P, p0, s, stream)       \
                        : launch_forward_t<n, true, 0>(ctx, base, P, p0, s, stream);
    RA_EXACT_LIST(RA_CASE)
#undef RA_CASE
#define RA_CASE(n) \
    if (!P.exact && P.jt == n) return launch_forward_t<n, false, 0>(ctx, base, P, p0, s, stream);
    RA_GENERIC_LIST(RA_CASE)
#undef RA_CASE
    return fail(ctx, RA_ENOTSUP, "window half-width not supported");
}

template <int JT, bool EXACT, bool P0, bool POSE, int KT = RA_KERNEL_GAUSSIAN>
int launch_adjoint_t(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, int acc,
                     hipStream_t stream) {
    auto kern = k_adjoint<JT, EXACT, P0, POSE, KT>;
    if constexpr (P0 && !POSE && EXACT && KT == RA_KERNEL_GAUSSIAN)
        if (P.rowref) kern = k_adjoint<JT, EXACT, P0, POSE, KT, true>;
    RA_HIP(ctx, allow_full_lds(kern));
    const bool alone = P0 && !POSE;        // dL/dp0 alone: the smaller regions
    const Geo& g = alone ? P.ga : P.g;
    hipLaunchKernelGGL(kern, dim3(g.nreg), dim3(BLOCK), alone ? P.lds_adj0 : P.lds_adj, stream, g, p0,
                       at<float>(ctx, P.off_xe), at<float4>(ctx, alone ? P.off_vtab_a : P.off_vtab),
                       at<int4>(ctx, alone ? P.off_itab_a : P.off_itab), r, gp0, acc, at<double>(ctx, P.off_part));
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

template <int JT, bool EXACT, int KT = RA_KERNEL_GAUSSIAN>
int launch_adjoint_j(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, bool pose, int acc,
                     hipStream_t stream) {
    if (gp0 && pose) return launch_adjoint_t<JT, EXACT, true, true, KT>(ctx, P, p0, r, gp0, acc, stream);
    if (gp0) return launch_adjoint_t<JT, EXACT, true, false, KT>(ctx, P, p0, r, gp0, acc, stream);
    return launch_adjoint_t<JT, EXACT, false, true, KT>(ctx, P, p0, r, gp0, acc, stream);
}

template <int NM, int CPW, bool P0, bool POSE, int X>
int launch_adjoint_series_t(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, int acc,
                            hipStream_t stream) {
    const Geo& g = POSE ? P.ga2 : P.ga1;
    const int nbuf = P.am_nbuf[POSE ? 1 : 0], xrows = X ? g.nbin + 2 * g.jt : 0;
    auto kern = k_adjoint_series<NM, CPW, P0, POSE, X>;
    RA_HIP(ctx, allow_full_lds(kern));
    hipLaunchKernelGGL(kern, dim3(std::min(g.nreg, NCU)), dim3(AM_WAVES * WAVE), am_lds(g.nbin, am_nq(NM), xrows, nbuf),
                       stream, g, nbuf, p0, at<float>(ctx, P.off_xe), at<float4>(ctx, P.off_q), r, gp0, acc,
                       at<double>(ctx, P.off_part));
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

template <int NM, bool P0, bool POSE, int X>
int launch_adjoint_series_c(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, int acc,
                            hipStream_t stream) {
    const Geo& g = POSE ? P.ga2 : P.ga1;
    const int cpw = (g.rx * g.ry + AM_WAVES - 1) / AM_WAVES;
    if constexpr (X == 0) {
        if (cpw <= 1) return launch_adjoint_series_t<NM, 1, P0, POSE, X>(ctx, P, p0, r, gp0, acc, stream);
        if (cpw <= 2) return launch_adjoint_series_t<NM, 2, P0, POSE, X>(ctx, P, p0, r, gp0, acc, stream);
    }
    return launch_adjoint_series_t<NM, 4, P0, POSE, X>(ctx, P, p0, r, gp0, acc, stream);
}

// The adjoints in moment form: the table of dL/ds, then the regions.
int launch_adjoint_series(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, bool pose, int acc,
                          hipStream_t stream) {
    const int K = P.g.K, jt = pose ? P.ga2.jt : P.ga1.jt, per = (K + 2 * jt + MT_ROWS - 1) / MT_ROWS;
    const int nm = pose ? P.terms.pose : P.terms.vol;
    auto table = am_nq(nm) == 2 ? k_moment_series<2> : k_moment_series<3>;
    hipLaunchKernelGGL(table, dim3((unsigned)P.g.E * per), dim3(MT_ROWS), 0, stream, P.g.E, K, jt,
                       pose ? ctx->now->pose : ctx->now->vol, r, at<float4>(ctx, P.off_q));
#define RA_CASE(n, x)                                                                                    \
    if (nm == n && P.terms.xkind == x && pose)                                                           \
        return gp0 ? launch_adjoint_series_c<n, true, true, x>(ctx, P, p0, r, gp0, acc, stream)          \
                   : launch_adjoint_series_c<n, false, true, x>(ctx, P, p0, r, gp0, acc, stream);
    RA_CASE(8, 0) RA_CASE(8, 1) RA_CASE(12, 1) RA_CASE(8, 2)
#undef RA_CASE
#define RA_CASE(n, x) \
    if (nm == n && P.terms.xkind == x && !pose)  \
        return launch_adjoint_series_c<n, true, false, x>(ctx, P, p0, r, gp0, acc, stream);
    RA_CASE(6, 0) RA_CASE(7, 0) RA_CASE(8, 0) RA_CASE(8, 1) RA_CASE(12, 1) RA_CASE(8, 2)
#undef RA_CASE
    return fail(ctx, RA_ENOTSUP, "moment form without a kernel for its terms");
}

int launch_adjoint(ra_ctx* ctx, const Plan& P, const float* p0, const float* r, float* gp0, bool pose, int acc,
                   hipStream_t stream) {
    if (pose ? P.am_pose : P.am) return launch_adjoint_series(ctx, P, p0, r, gp0, pose, acc, stream);
    if (!generic_bound_ok(P)) return fail(ctx, RA_ENOTSUP, "window half-width not supported");
    switch (P.g.ktype) {
        case RA_KERNEL_EXPONENTIAL:
#define RA_CASE(n) \
    if (P.jt == n) return launch_adjoint_j<n, false, RA_KERNEL_EXPONENTIAL>(ctx, P, p0, r, gp0, pose, acc, stream);
            RA_EXP_LIST(RA_CASE)
#undef RA_CASE
            break;
        case RA_KERNEL_POWER:
            if (P.g.knu == -2.0f) return launch_adjoint_j<0, false, KT_POWER2>(ctx, P, p0, r, gp0, pose, acc, stream);
            return launch_adjoint_j<0, false, RA_KERNEL_POWER>(ctx, P, p0, r, gp0, pose, acc, stream);
        case RA_KERNEL_UNIFORM:
            return launch_adjoint_j<0, false, RA_KERNEL_UNIFORM>(ctx, P, p0, r, gp0, pose, acc, stream);
        default: break;
    }
#define RA_CASE(n) \
    if (P.exact && P.jt == n) return launch_adjoint_j<n, true>(ctx, P, p0, r, gp0, pose, acc, stream);
    RA_EXACT_LIST(RA_CASE)
#undef RA_CASE
#define RA_CASE(n) \
    if (!P.exact && P.jt == n) return launch_adjoint_j<n, false>(ctx, P, p0, r, gp0, pose, acc, stream);
    RA_GENERIC_LIST(RA_CASE)
#undef RA_CASE
    return fail(ctx, RA_ENOTSUP, "window half-width not supported");
}

int adjoint_body(ra_ctx* ctx, const Plan& P, const float* p0, const double* elem, const float* r,
                 float* grad_p0, double* grad_pose, double* grad_elem, uint32_t flags, hipStream_t stream) {
    const int acc = (flags & RA_ACCUMULATE) ? 1 : 0;
    const bool pose = grad_pose || grad_elem;
    if (!grad_p0 && !pose) return RA_OK;
    int rc = launch_adjoint(ctx, P, p0, r, grad_p0, pose, acc, stream);
    if (rc != RA_OK) return rc;
    if (pose) {
        const Geo& g = P.g;
        hipLaunchKernelGGL(k_pose_reduce, dim3((3 * g.E + PR_T - 1) / PR_T), dim3(PR_T * PR_P), 0, stream, g, P.part_rows,
                           at<double>(ctx, P.off_part), at<double>(ctx, P.off_ge), grad_elem, acc);
        if (grad_pose)
            hipLaunchKernelGGL(k_pose_frame, dim3(g.F), dim3(256), 0, stream, g, at<double>(ctx, P.off_ge), elem,
                               grad_pose, acc);
        RA_HIP(ctx, hipGetLastError());
    }
    return RA_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// exported API
// ---------------------------------------------------------------------------------------------
extern "C" {

int ra_create(ra_ctx** out, int device) {
    if (!out) return RA_EINVAL;
    *out = nullptr;
    ra_ctx* ctx = new (std::nothrow) ra_ctx();
    if (!ctx) return RA_ENOMEM;
    ctx->device = device;
    if (hipSetDevice(device) != hipSuccess || hipMalloc(&ctx->d_status, sizeof(int)) != hipSuccess ||
        hipMemset(ctx->d_status, 0, sizeof(int)) != hipSuccess ||
        hipHostMalloc((void**)&ctx->h_count, sizeof(unsigned long long), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&ctx->h_f64, sizeof(double), hipHostMallocDefault) != hipSuccess ||
        hipMalloc(&ctx->d_f64, sizeof(double)) != hipSuccess ||
        static_scratch_of(device, &ctx->static_scratch) != hipSuccess) {
        (void)hipGetLastError();
        ra_destroy(ctx);
        return RA_EHIP;
    }
    *out = ctx;
    return RA_OK;
}

void ra_destroy(ra_ctx* ctx) {
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    if (ctx->arena) (void)hipFree(ctx->arena);
    if (ctx->d_status) (void)hipFree(ctx->d_status);
    if (ctx->h_count) (void)hipHostFree(ctx->h_count);
    if (ctx->h_f64) (void)hipHostFree(ctx->h_f64);
    if (ctx->d_f64) (void)hipFree(ctx->d_f64);
    delete ctx;
}

const char* ra_last_error(const ra_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int ra_status(ra_ctx* ctx, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    hipStream_t st = (hipStream_t)stream;
    int h = 0;
    RA_HIP(ctx, hipMemcpyAsync(&h, ctx->d_status, sizeof(int), hipMemcpyDeviceToHost, st));
    RA_HIP(ctx, hipStreamSynchronize(st));
    RA_HIP(ctx, hipMemsetAsync(ctx->d_status, 0, sizeof(int), st));
    RA_HIP(ctx, hipStreamSynchronize(st));
    if (h) return fail(ctx, RA_EGEOM, "an element came closer than 10 sigma to the voxel grid");
    return RA_OK;
}

int ra_reserve(ra_ctx* ctx, size_t bytes) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    RA_HIP(ctx, hipSetDevice(ctx->device));
    return ensure_scratch(ctx, bytes, nullptr);
}

size_t ra_scratch_bytes(const ra_grid* grid, int32_t M, int32_t F, const ra_sampling* samp) {
    ra_ctx tmp;
    if (validate(&tmp, grid, M, F, samp) != RA_OK) return 0;
    size_t most = 0;
    for (unsigned only : {0u, PLAN_ROW_FORWARD}) {
        Plan P;
        make_plan(&tmp, grid, M, F, samp, P, RA_SUMS_F64, only);      // the largest of the forward's sum modes
        most = std::max(most, P.total);
    }
    return most;
}

int ra_set_forward_sums(ra_ctx* ctx, int32_t mode) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (mode != RA_SUMS_AUTO && mode != RA_SUMS_F32 && mode != RA_SUMS_F64)
        return fail(ctx, RA_EINVAL, "mode must be RA_SUMS_AUTO, RA_SUMS_F32 or RA_SUMS_F64");
    ctx->sums_mode = mode;
    return RA_OK;
}

int radiate_forward(ra_ctx* ctx, const ra_grid* grid, const float* p0, int32_t M, const double* elem,
                    const double* poses, int32_t F, const ra_sampling* samp, float* s, void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!p0 || !elem || !poses || !s) return fail(ctx, RA_EINVAL, "p0, elem, poses and s are required");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    Plan P;
    make_plan(ctx, grid, M, F, samp, P, ctx->sums_mode);
    // a later call with an adjoint may be captured, and finds its scratch; but a forward that fits runs
    rc = ensure_scratch(ctx, std::min(P.total, P.kept), st);
    if (rc == RA_ENOMEM && (rc = ensure_scratch(ctx, forward_layout(P), st)) == RA_OK) ctx->err.clear();
    if (rc != RA_OK) return rc;
    if ((rc = prologue(ctx, ctx->arena, grid, P, elem, poses, st, true)) != RA_OK) return rc;
    return launch_forward(ctx, ctx->arena, P, p0, s, st);
}

int radiate_forward_static(ra_ctx* ctx, const ra_grid* grid, const float* p0, int32_t M, const double* elem,
                           const double* poses, int32_t F, const ra_sampling* samp, float* s, void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!p0 || !elem || !poses || !s) return fail(ctx, RA_EINVAL, "p0, elem, poses and s are required");
    if (!ctx->static_scratch) return fail(ctx, RA_EHIP, "the static scratch of this device was not resolved");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    Plan P;
    make_plan(ctx, grid, M, F, samp, P, ctx->sums_mode);
    const size_t need = forward_layout(P);
    if (need > STATIC_SCRATCH_BYTES)
        return fail(ctx, RA_ENOMEM, "radiate_forward_static needs " + std::to_string(need) +
                                        " bytes of scratch; its static array holds " +
                                        std::to_string(STATIC_SCRATCH_BYTES));
    if ((rc = prologue(ctx, ctx->static_scratch, grid, P, elem, poses, st, true)) != RA_OK) return rc;
    return launch_forward(ctx, ctx->static_scratch, P, p0, s, st);
}

int radiate_adjoint(ra_ctx* ctx, const ra_grid* grid, const float* p0, int32_t M, const double* elem,
                    const double* poses, int32_t F, const ra_sampling* samp, const float* r, float* grad_p0,
                    double* grad_pose, double* grad_elem, uint32_t flags, void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!elem || !poses || !r) return fail(ctx, RA_EINVAL, "elem, poses and r are required");
    if ((grad_pose || grad_elem) && !p0) return fail(ctx, RA_EINVAL, "p0 is required for pose gradients");
    if (flags & ~RA_ACCUMULATE) return fail(ctx, RA_EINVAL, "unknown flag bits");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    Plan P;
    if ((rc = plan_call(ctx, grid, M, F, samp, P, st)) != RA_OK) return rc;
    if ((rc = prologue(ctx, ctx->arena, grid, P, elem, poses, st)) != RA_OK) return rc;
    return adjoint_body(ctx, P, p0, elem, r, grad_p0, grad_pose, grad_elem, flags, st);
}

int loss_and_grad(ra_ctx* ctx, const ra_grid* grid, const float* p0, int32_t M, const double* elem,
                  const double* poses, int32_t F, const ra_sampling* samp, const float* y, double* loss,
                  float* s_out, float* grad_p0, double* grad_pose, double* grad_elem, uint32_t flags,
                  void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!p0 || !elem || !poses || !y) return fail(ctx, RA_EINVAL, "p0, elem, poses and y are required");
    if (flags & ~(RA_ACCUMULATE | RA_LOSS_ON_DEVICE | RA_SIGNALS_GIVEN))
        return fail(ctx, RA_EINVAL, "unknown flag bits");
    const bool given = (flags & RA_SIGNALS_GIVEN) != 0;
    if (given && !s_out) return fail(ctx, RA_EINVAL, "RA_SIGNALS_GIVEN needs the signals in s_out");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    Plan P;
    if ((rc = plan_call(ctx, grid, M, F, samp, P, st)) != RA_OK) return rc;
    if ((rc = prologue(ctx, ctx->arena, grid, P, elem, poses, st)) != RA_OK) return rc;
    float* s = at<float>(ctx, P.off_s);
    const size_t n = (size_t)P.g.E * P.g.K;
    if (given) {
        // the caller's signals; the residual below overwrites the scratch copy, not them
        hipLaunchKernelGGL(k_copy, dim3(1024), dim3(256), 0, st, s_out, n, s);
    } else {
        if ((rc = launch_forward(ctx, ctx->arena, P, p0, s, st)) != RA_OK) return rc;
        if (s_out) hipLaunchKernelGGL(k_copy, dim3(1024), dim3(256), 0, st, s, n, s_out);
    }
    float* partial = at<float>(ctx, P.off_partial);
    hipLaunchKernelGGL(k_residual, dim3(RESID_BLOCKS), dim3(256), 0, st, s, y, n, partial);
    RA_HIP(ctx, hipGetLastError());
    if ((rc = adjoint_body(ctx, P, p0, elem, s, grad_p0, grad_pose, grad_elem, flags & RA_ACCUMULATE, st)) != RA_OK)
        return rc;
    if (loss) {
        // FP64 sum of the per-block FP32 partials, in a fixed order, on the device
        double* dst = (flags & RA_LOSS_ON_DEVICE) ? loss : ctx->d_f64;
        hipLaunchKernelGGL(k_loss_total, dim3(1), dim3(256), 0, st, partial, RESID_BLOCKS, dst);
        RA_HIP(ctx, hipGetLastError());
        if (!(flags & RA_LOSS_ON_DEVICE)) {
            RA_HIP(ctx, hipMemcpyAsync(ctx->h_f64, ctx->d_f64, sizeof(double), hipMemcpyDeviceToHost, st));
            RA_HIP(ctx, hipStreamSynchronize(st));
            *loss = *ctx->h_f64;
        }
    }
    return RA_OK;
}

int nc_loss_and_grad(ra_ctx* ctx, const ra_grid* grid, const float* p0, int32_t M, const double* elem,
                     const double* poses, int32_t F, const ra_sampling* samp, const float* y,
                     const float* weight, double* loss, double* loss_elem, float* s_out, float* grad_p0,
                     double* grad_pose, double* grad_elem, uint32_t flags, void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!p0 || !elem || !poses || !y) return fail(ctx, RA_EINVAL, "p0, elem, poses and y are required");
    if (flags & ~RA_ACCUMULATE) return fail(ctx, RA_EINVAL, "unknown flag bits");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    Plan P;
    if ((rc = plan_call(ctx, grid, M, F, samp, P, st, loss ? PLAN_ROW_FORWARD : 0)) != RA_OK) return rc;
    if ((rc = prologue(ctx, ctx->arena, grid, P, elem, poses, st)) != RA_OK) return rc;
    float* s = at<float>(ctx, P.off_s);
    if ((rc = launch_forward(ctx, ctx->arena, P, p0, s, st)) != RA_OK) return rc;
    const int E = P.g.E;
    if (s_out) hipLaunchKernelGGL(k_copy, dim3(1024), dim3(256), 0, st, s, (size_t)E * P.g.K, s_out);
    double* wl = at<double>(ctx, P.off_ncw);
    hipLaunchKernelGGL(k_nc_residual, dim3(std::min(E, 65536)), dim3(NC_THREADS), 0, st, s, y, weight, E, P.g.K,
                       loss_elem, wl);
    RA_HIP(ctx, hipGetLastError());
    if ((rc = adjoint_body(ctx, P, p0, elem, s, grad_p0, grad_pose, grad_elem, flags, st)) != RA_OK) return rc;
    if (loss) {
        double* d_total = at<double>(ctx, P.off_nct);
        hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(NC_THREADS), 0, st, wl, E, d_total);
        RA_HIP(ctx, hipMemcpyAsync(ctx->h_f64, d_total, sizeof(double), hipMemcpyDeviceToHost, st));
        RA_HIP(ctx, hipStreamSynchronize(st));
        *loss = *ctx->h_f64;
    }
    return RA_OK;
}

int ra_pose_from_axis_angle(ra_ctx* ctx, const double* pose6, int32_t F, double* poses, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!pose6 || !poses || F <= 0) return fail(ctx, RA_EINVAL, "pose6, poses and F > 0 are required");
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_pose_from_aa, dim3((F + 127) / 128), dim3(128), 0, (hipStream_t)stream, pose6, F, poses);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

int ra_pose_grad_axis_angle(ra_ctx* ctx, const double* pose6, const double* grad_pose, int32_t F, double* grad6,
                            void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!pose6 || !grad_pose || !grad6 || F <= 0)
        return fail(ctx, RA_EINVAL, "pose6, grad_pose, grad6 and F > 0 are required");
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_pose_grad_aa, dim3((F + 127) / 128), dim3(128), 0, (hipStream_t)stream, pose6, grad_pose, F,
                       grad6);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

size_t ra_tgv_scratch_bytes(int32_t nx, int32_t ny, int32_t nz) {
    if (nx <= 0 || ny <= 0 || nz <= 0) return 0;
    return align_up((size_t)tgv_blocks(nx, ny, nz) * sizeof(double));
}

int tgv_loss_and_grad(ra_ctx* ctx, int32_t nx, int32_t ny, int32_t nz, const float* u, const float* w,
                      double alpha0, double alpha1, double eps, double scale, double* loss, float* grad_u,
                      float* grad_w, uint32_t flags, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (nx <= 0 || ny <= 0 || nz <= 0) return fail(ctx, RA_EINVAL, "grid dimensions must be positive");
    if ((long long)nx * ny * nz >= (1LL << 31)) return fail(ctx, RA_EINVAL, "grid has 2^31 or more voxels");
    if (!u || !w) return fail(ctx, RA_EINVAL, "u and w are required");
    if (!(alpha0 >= 0.0) || !(alpha1 >= 0.0) || !(eps >= 1e-18) || !std::isfinite(scale) || !std::isfinite(alpha0) ||
        !std::isfinite(alpha1) || !std::isfinite(eps))
        return fail(ctx, RA_EINVAL, "alpha0, alpha1 >= 0, eps >= 1e-18 and a finite scale are required");
    if (flags & ~RA_ACCUMULATE) return fail(ctx, RA_EINVAL, "unknown flag bits");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    int rc = ensure_scratch(ctx, ra_tgv_scratch_bytes(nx, ny, nz), st);
    if (rc != RA_OK) return rc;
    TgvDims d;
    d.nx = nx; d.ny = ny; d.nz = nz;
    d.n = nx * ny * nz;
    d.sy = nz;
    d.sx = ny * nz;
    const TgvCut cut = tgv_cut(nx, ny, nz);
    d.bz = cut.bz;
    d.by = cut.by;
    d.xc = cut.xc;
    d.a0 = (float)alpha0; d.a1 = (float)alpha1; d.eps = (float)eps;
    const unsigned nblocks = (unsigned)cut.bx * cut.by * cut.bz;      // at most one per voxel: below 2^31
    double* partial = at<double>(ctx, 0);
    constexpr int nt = 64 * TGV_NW;
    constexpr size_t lds = (size_t)nt * TGV_LDS * sizeof(tgv4);
    auto kernel = cut.lanes == 16 ? k_tgv<16> : cut.lanes == 32 ? k_tgv<32> : k_tgv<64>;
    RA_HIP(ctx, allow_full_lds(kernel));
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(nt), lds, st, d, u, w, (float)scale,
                       (flags & RA_ACCUMULATE) ? 1 : 0, grad_u, grad_w, partial);
    RA_HIP(ctx, hipGetLastError());
    if (loss) {
        hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(NC_THREADS), 0, st, partial, (int)nblocks, ctx->d_f64);
        RA_HIP(ctx, hipMemcpyAsync(ctx->h_f64, ctx->d_f64, sizeof(double), hipMemcpyDeviceToHost, st));
        RA_HIP(ctx, hipStreamSynchronize(st));
        *loss = scale * *ctx->h_f64;
    }
    return RA_OK;
}

int ra_pose_from_euler(ra_ctx* ctx, const double* pose6, int32_t F, double* poses, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!pose6 || !poses || F <= 0) return fail(ctx, RA_EINVAL, "pose6, poses and F > 0 are required");
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_pose_from_euler, dim3((F + 127) / 128), dim3(128), 0, (hipStream_t)stream, pose6, F, poses);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

int ra_pose_grad_euler(ra_ctx* ctx, const double* pose6, const double* grad_pose, int32_t F, double* grad6,
                       void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!pose6 || !grad_pose || !grad6 || F <= 0)
        return fail(ctx, RA_EINVAL, "pose6, grad_pose, grad6 and F > 0 are required");
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_pose_grad_euler, dim3((F + 127) / 128), dim3(128), 0, (hipStream_t)stream, pose6, grad_pose,
                       F, grad6);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

int ra_count_updates(ra_ctx* ctx, const ra_grid* grid, int32_t M, const double* elem, const double* poses,
                     int32_t F, const ra_sampling* samp, long long* count, void* stream) {
    int rc = validate(ctx, grid, M, F, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!elem || !poses || !count) return fail(ctx, RA_EINVAL, "elem, poses and count are required");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    const int E = M * F;
    const size_t off_count = align_up((size_t)E * 3 * sizeof(double));
    if ((rc = ensure_scratch(ctx, off_count + sizeof(unsigned long long), st)) != RA_OK) return rc;
    double* xe64 = at<double>(ctx, 0);
    unsigned long long* d_count = at<unsigned long long>(ctx, off_count);
    hipLaunchKernelGGL(k_elements_f64, dim3((E + 255) / 256), dim3(256), 0, st, M, E, elem, poses, xe64);
    hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, st, reinterpret_cast<float*>(d_count), (size_t)2, 0.0f);
    long long nvox = (long long)grid->nx * grid->ny * grid->nz;
    hipLaunchKernelGGL(k_count, dim3((unsigned)((nvox + 255) / 256)), dim3(256), 0, st, grid->nx, grid->ny, grid->nz,
                       grid->origin[0], grid->origin[1], grid->origin[2], grid->spacing, E, xe64, samp->c,
                       samp->fs, samp->K, samp->trunc * samp->sigma, d_count);
    RA_HIP(ctx, hipGetLastError());
    RA_HIP(ctx, hipMemcpyAsync(ctx->h_count, d_count, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    RA_HIP(ctx, hipStreamSynchronize(st));
    *count = (long long)*ctx->h_count;
    return RA_OK;
}

int ra_probe_rates(ra_ctx* ctx, double* fma_per_s, double* exp_per_s, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!fma_per_s || !exp_per_s) return fail(ctx, RA_EINVAL, "fma_per_s and exp_per_s are required");
    hipStream_t st = (hipStream_t)stream;
    RA_HIP(ctx, hipSetDevice(ctx->device));
    int rc = ensure_scratch(ctx, align_up((size_t)PROBE_BLOCKS * 256 * sizeof(float)), st);
    if (rc != RA_OK) return rc;
    float* out = at<float>(ctx, 0);
    const int it_fma = 16384, it_exp = 4096;
    hipEvent_t e0, e1;
    RA_HIP(ctx, hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(ctx, RA_EHIP, "hipEventCreate failed");
    }
    auto timed = [&](bool exp_probe, int iters, double& rate) -> hipError_t {
        for (int rep = 0; rep < 2; ++rep) {          // the first launch warms up; the second is timed
            hipError_t e = hipEventRecord(e0, st);
            if (e != hipSuccess) return e;
            if (exp_probe)
                hipLaunchKernelGGL(k_probe_exp, dim3(PROBE_BLOCKS), dim3(256), 0, st, out, iters);
            else
                hipLaunchKernelGGL(k_probe_fma, dim3(PROBE_BLOCKS), dim3(256), 0, st, out, iters, 0.999f, 1e-3f);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = hipEventRecord(e1, st)) != hipSuccess) return e;
            if ((e = hipEventSynchronize(e1)) != hipSuccess) return e;
        }
        float ms = 0.0f;
        hipError_t e = hipEventElapsedTime(&ms, e0, e1);
        rate = (double)PROBE_BLOCKS * 256.0 * PROBE_CHAINS * iters / (ms * 1e-3);
        return e;
    };
    hipError_t e = timed(false, it_fma, *fma_per_s);
    if (e == hipSuccess) e = timed(true, it_exp, *exp_per_s);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return fail(ctx, RA_EHIP, std::string("rate probe: ") + hipGetErrorString(e));
    return RA_OK;
}

}  // extern "C"

extern "C" {

size_t ra_batch_geo_bytes(void) { return sizeof(BatchGeo); }

int ra_batch_describe(ra_ctx* ctx, const ra_grid* box, int64_t stride_x, int64_t stride_y, int32_t M,
                      const ra_sampling* samp, void* geo, ra_batch_info* info) {
    int rc = validate(ctx, box, M, 1, samp);
    if (rc != RA_OK) return rc;
    ctx->err.clear();
    if (!geo || !info) return fail(ctx, RA_EINVAL, "geo and info are required");
    if (samp->kernel != RA_KERNEL_GAUSSIAN)
        return fail(ctx, RA_ENOTSUP, "the batched step supports the Gaussian profile only");
    if (stride_y < box->nz || stride_x < (int64_t)stride_y * box->ny)
        return fail(ctx, RA_EINVAL, "volume strides smaller than the box");
    Plan P;
    make_plan(nullptr, box, M, 1, samp, P);
    BatchGeo bg;
    std::memset(&bg, 0, sizeof(bg));
    Geo& g = bg.g;
    g = P.g;
    g.vsx = stride_x;
    g.vsy = stride_y;
    g.gsx = (long long)box->ny * box->nz;
    g.gsy = box->nz;
    // the batched row-form forward pairs z-neighbours when it can: D more rows (the adjoint stages
    // them too, and never reads them)
    const int pd = (P.pair_ok && !(g.rz & 1)) ? PAIR_D : 0;
    g.L += pd;
    // the moment forms on the same regions, where their series and LDS allow it
    const double delta = samp->c / samp->fs;
    g.jt = P.jt;
    g.nbin = 2 * g.jclamp + 1;
    set_units(g, box, delta);
    bg.ga = g;
    if (g.rz > FM_RZ) {
        bg.ga.rz = FM_RZ;
        bg.ga.nrz = (g.nz + FM_RZ - 1) / FM_RZ;
        bg.ga.nreg = g.nrx * g.nry * bg.ga.nrz;
    }
    const MomTerms mt = P.exact ? series_of(ctx, samp, true).terms : MomTerms{};
    bg.nm = mt.fwd;
    const size_t lds = fm_lds(bg.nm, g.nbin, g.jt, false);
    const bool moment = mt.fwd && mt.pose && g.nbin <= BATCH_BINS_MAX && lds <= 160 * 1024 && am_lds(g.nbin, 2, 0, 1) <= 160 * 1024;
    if (moment) {
        bg.series = ctx->now->fwd;
        bg.series8 = ctx->now->pose;
    }
    // Regions of few voxels (coarse spacings) keep the row form in the forward: per region and chunk, CU cycles of the adds and
    // the expansion (see plan_forward_mom) against those of the rows and their atomics (see row_forward_cost).  2x2x4 voxels
    // of 0.4 mm: 26.3 ms a step of six requests of 96^3 voxels and 128 elements in moments, 17.3 in rows.
    const double mom = g.rx * g.ry * ((g.rz + FM_RZ - 1) / FM_RZ * FM_RZ) * 34.0 +
                       ((g.nbin + 2 * g.jt + 15) / 16) * ((2 * g.jt + 19) / 4) * bg.nm * 32.0 * 1.45 + (lds <= LDS_FM_BUDGET ? 800.0 : 2500.0);
    const double rows = g.nvpad * (2 * g.jt + 1 + pd) * 0.7 * (pd ? 32.0 : 57.0) / 8.0 + g.L * 152.0;
    std::memcpy(geo, &bg, sizeof(BatchGeo));
    info->nreg = g.nreg;
    info->jt = P.jt;
    info->exact = P.exact ? 1 : 0;
    info->pair_d = pd;
    // rows of LDS of 1 KiB: the row form's samples, or what the moment-form forward needs
    info->moment = moment ? (mom <= 1.1 * rows ? 1 : 2) : 0;
    info->lmax = info->moment == 1 ? std::max(g.L, (int)((lds + 1023) / 1024)) : g.L;
    info->nvpad = g.nvpad;
    info->rx = g.rx; info->ry = g.ry; info->rz = g.rz;
    info->nbin = g.nbin;
    // the table with its zero row, then one loss per element
    info->q_bytes = moment ? (((int64_t)M * (samp->K + 2 * P.jt) + 1) * MOM_G + M) * (int64_t)sizeof(float) : 0;
    return RA_OK;
}

int ra_batch_tables(ra_ctx* ctx, const void* geo, void* vtab, void* itab, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!geo || !vtab || !itab) return fail(ctx, RA_EINVAL, "geo, vtab and itab are required");
    Geo g;
    std::memcpy(&g, geo, sizeof(Geo));
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipLaunchKernelGGL(k_voxel_table, dim3((g.nvpad + 255) / 256), dim3(256), 0, (hipStream_t)stream, g,
                       (float4*)vtab, (int4*)itab);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

}  // extern "C"

namespace {

// Pose updates, losses of the moment form, and volume updates.
int batch_finish(ra_ctx* ctx, const ra_batch* b, uint32_t flags, hipStream_t st) {
    const BatchGeo* geos = (const BatchGeo*)b->geos;
    const int grid = b->grid_blocks > 0 ? b->grid_blocks : 1024;
    hipLaunchKernelGGL(k_batch_pose_chunks, dim3(grid), dim3(BATCH_THREADS), 0, st, geos, b->reqs, b->counts);
    hipLaunchKernelGGL(k_batch_pose_update, dim3(grid), dim3(BATCH_THREADS), 0, st, geos, b->reqs, b->counts, b->moment);
    if (flags & RA_BATCH_APPLY_UPDATES)
        hipLaunchKernelGGL(k_batch_volume_apply, dim3(grid), dim3(BLOCK), 0, st, geos, b->reqs, (const int4*)b->itab,
                           (const int2*)b->items_vol, b->counts);
    RA_HIP(ctx, hipGetLastError());
    return RA_OK;
}

// Residuals with losses and tables, both kinds of adjoint in one launch, and what follows them.
int batch_adjoints_mom(ra_ctx* ctx, const ra_batch* b, uint32_t flags, hipStream_t st) {
    const BatchGeo* geos = (const BatchGeo*)b->geos;
    const int grid = b->grid_blocks > 0 ? b->grid_blocks : 1024;
    const int nbuf = am_lds(b->nbin, 2, 0, 2) <= 160 * 1024 ? 2 : 1;
    RA_HIP(ctx, allow_full_lds(k_adjoint_series_batch));
    hipLaunchKernelGGL(k_batch_series, dim3(grid), dim3(MT_ROWS), 0, st, geos, b->reqs, (const int2*)b->items_elem, b->counts);
    hipLaunchKernelGGL(k_adjoint_series_batch, dim3(std::min(grid, NCU)), dim3(AM_WAVES * WAVE), am_lds(b->nbin, 2, 0, nbuf), st,
                       geos, b->reqs, (const int2*)b->items_pose, (const int2*)b->items_vol, b->counts, b->nbin, nbuf);
    return batch_finish(ctx, b, flags, st);
}

template <int JT, bool EXACT, int D>
int batch_step_t(ra_ctx* ctx, const ra_batch* b, uint32_t flags, hipStream_t st) {
    const BatchGeo* geos = (const BatchGeo*)b->geos;
    const float4* vtab = (const float4*)b->vtab;
    const int4* itab = (const int4*)b->itab;
    const int2* ifwd = (const int2*)b->items_fwd;
    const int2* ipose = (const int2*)b->items_pose;
    const int2* ivol = (const int2*)b->items_vol;
    const int2* ielem = (const int2*)b->items_elem;
    const int grid = b->grid_blocks > 0 ? b->grid_blocks : 1024;
    const size_t lds_f = (size_t)WAVES * b->lmax * WAVE * sizeof(float);
    const size_t lds_a = lds_f + (size_t)WAVES * b->nvpad * sizeof(float);
    auto kf = k_forward_batch<JT, EXACT, D>;
    auto kp = k_adjoint_batch<JT, EXACT, false, true>;
    auto kv = k_adjoint_batch<JT, EXACT, true, false>;
    RA_HIP(ctx, allow_full_lds(kf));
    RA_HIP(ctx, allow_full_lds(kp));
    RA_HIP(ctx, allow_full_lds(kv));
    hipLaunchKernelGGL(k_batch_elements, dim3(64), dim3(256), 0, st, b->reqs, ielem, b->counts);
    hipLaunchKernelGGL(k_batch_zero, dim3(grid), dim3(256), 0, st, geos, b->reqs, b->counts);
    hipLaunchKernelGGL(kf, dim3(grid), dim3(BLOCK), lds_f, st, geos, b->reqs, vtab, itab, ifwd, b->counts, b->lmax);
    if (b->moment) return batch_adjoints_mom(ctx, b, flags, st);
    hipLaunchKernelGGL(k_batch_residual, dim3(grid), dim3(BATCH_THREADS), 0, st, geos, b->reqs, b->counts);
    hipLaunchKernelGGL(kp, dim3(grid), dim3(BLOCK), lds_a, st, geos, b->reqs, vtab, itab, ipose, b->counts, 1,
                       b->lmax);
    hipLaunchKernelGGL(kv, dim3(grid), dim3(BLOCK), lds_a, st, geos, b->reqs, vtab, itab, ivol, b->counts, 2,
                       b->lmax);
    return batch_finish(ctx, b, flags, st);
}

// The moment form: positions and cleared signals, the forward, then the adjoints.
int batch_step_mom(ra_ctx* ctx, const ra_batch* b, uint32_t flags, hipStream_t st) {
    const BatchGeo* geos = (const BatchGeo*)b->geos;
    const int grid = b->grid_blocks > 0 ? b->grid_blocks : 1024;
    const size_t lds_f = (size_t)b->lmax * 1024;
    RA_HIP(ctx, allow_full_lds(k_forward_mom_batch));
    hipLaunchKernelGGL(k_batch_begin, dim3(grid), dim3(BATCH_THREADS), 0, st, geos, b->reqs, (const int2*)b->items_elem, b->counts);
    hipLaunchKernelGGL(k_forward_mom_batch, dim3(grid), dim3(FM_WAVES * WAVE), lds_f, st, geos, b->reqs,
                       (const int2*)b->items_fwd, b->counts, (int)lds_f);
    return batch_adjoints_mom(ctx, b, flags, st);
}

}  // namespace

extern "C" int ra_batch_step(ra_ctx* ctx, const ra_batch* b, uint32_t flags, void* stream) {
    if (!ctx) return RA_EINVAL;
    ctx->err.clear();
    if (!b || !b->geos || !b->reqs || !b->vtab || !b->itab || !b->items_fwd || !b->items_pose || !b->items_vol ||
        !b->items_elem || !b->counts)
        return fail(ctx, RA_EINVAL, "every table of the batch is required");
    if (flags & ~RA_BATCH_APPLY_UPDATES) return fail(ctx, RA_EINVAL, "unknown flag bits");
    if (b->lmax <= 0 || b->nvpad <= 0 || b->nvpad % 4) return fail(ctx, RA_EINVAL, "bad lmax or nvpad");
    if ((size_t)WAVES * b->lmax * WAVE * sizeof(float) + (size_t)WAVES * b->nvpad * sizeof(float) > 160 * 1024)
        return fail(ctx, RA_EINVAL, "lmax / nvpad exceed the LDS of a workgroup");
    const bool ex = b->exact != 0;
    if (b->moment) {
        // the moment form exists for the exact Gaussian window only; its LDS windows hold nbin bins
        if (!b->coef) return fail(ctx, RA_EINVAL, "the moment form needs the coefficient scratch (coef)");
        if (!ex || b->jt < 1 || b->jt > JMAX) return fail(ctx, RA_EINVAL, "moment form with a window it does not cover");
        if (b->nbin < 1 || b->nbin > BATCH_BINS_MAX)
            return fail(ctx, RA_EINVAL, "nbin must be the value ra_batch_describe reported");
        if (am_lds(b->nbin, 2, 0, 1) > 160 * 1024) return fail(ctx, RA_EINVAL, "nbin exceeds the LDS of a workgroup");
    }
    RA_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    if (b->pair_d != 0 && (b->pair_d != PAIR_D || !ex))
        return fail(ctx, RA_EINVAL, "pair_d must be the value ra_batch_describe reported");
    if (b->moment && b->moment != 2) return batch_step_mom(ctx, b, flags, st);
#define RA_CASE(n)                                                                                      \
    if (ex && b->jt == n)                                                                               \
        return b->pair_d ? batch_step_t<n, true, PAIR_D>(ctx, b, flags, st)                             \
                         : batch_step_t<n, true, 0>(ctx, b, flags, st);
    RA_EXACT_LIST(RA_CASE)
#undef RA_CASE
#define RA_CASE(n) \
    if (!ex && b->jt == n) return batch_step_t<n, false, 0>(ctx, b, flags, st);
    RA_GENERIC_LIST(RA_CASE)
#undef RA_CASE
    return fail(ctx, RA_ENOTSUP, "window half-width not supported");
}
