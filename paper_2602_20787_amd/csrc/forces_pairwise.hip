// Forces of all N particles with every unordered pair evaluated once
// (Sect. 2.1, eqs. ComovingEquationsOfMotion and ForceCylindrical; with a
// table, the far images of Sect. 2.2, eq. S1R2EwaldCorrectionTable).  The
// pair term is odd in the separation: the image set {d - nL, |n| <= n_img}
// of the pair (j, i) is the negated set of (i, j), so S and P are shared and
// F_z, dx, dy change sign; the table's far-image term is odd in d along z
// and even across, so the same holds with it.  The exception is an axial
// separation of L/2 (up to rounding), where both particles may take a
// minimum image of the same sign; F_z then keeps its sign.  Evaluating each
// pair once halves the arithmetic of the per-target kernels
// (forces_exact.hip, table.hip).
//
// Layout and schedule: pair_schedule.h, with parts of 64 records (kSortMin: few
// particles keep their own order).
//
// What bounds a call is the number of waves in flight: a wave alone takes 37
// us for its 64 steps at |n| <= 8 where five on its SIMD take 15 us each, and
// every launch ends in a tail of half-empty SIMDs.  So as many rounds share a
// launch as the slots' memory allows (kSlotBytes), up to one launch of one
// group of all parts (flat: S = P, every slot written once), and where even
// that has too few tiles each is split over the two or four waves of a workgroup.
//
// Workgroup.  One wave owns its part, one particle per lane, in registers;
// the tile's sources come through LDS: at step s lane l takes source l xor s,
// so no two lanes meet the same source at once.  The reaction on a source is
// summed in FP64 in an LDS slot that the lanes update in turn (64 steps visit
// every lane).  Of Q waves each takes n = 64/Q of the sources, held Q times over,
// in n steps; the Q reactions on a source are added at the end, and wave 0 adds
// the waves' sums of the part (in slots of their own they would take Q times the
// workspace).  A
// tile whose sources' box is far from the wave's (no pair closer than
// the sum of the largest softenings, no axial separation near L/2) skips the
// softening and half-period screens and the per-pair minimum image; the pair
// arithmetic is the same either way.  Waves share nothing up to that last sum, so
// their steps need no barrier.  Small register sets let several of them share a SIMD,
// which hides the latency of the transcendentals (17 reciprocal square
// roots per pair) and of the LDS traffic behind the other waves' work.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "pair_f64.h"
#include "pair_fp32.h"
#include "pair_schedule.h"
#include "table_pair.h"

namespace steps {

namespace {

constexpr int kPart = 64;  // particles per part, one per lane
constexpr int kSplit = 4;  // most waves of a split tile
// The one-launch form, without workspace, up to this many particles.  Per call (us,
// |n| <= 8 with the potential), one launch against tiles: N = 500 13 and 36, 1000 13
// and 36, 2000 29 and 36, 2300 43 and 36, 2500 47 and 37 (38 to 42 before tiles were
// split over four waves; calls up to here need no workspace, so the line stays).
constexpr int kSmallMax = 2304;
// Waves per SIMD.  Measured per call at N = 2^20, |n| <= 8 with the potential
// (ms) with one launch per round: 1 particle per lane at 4, 5, 6 and 8 waves
// 1994, 1891, 1895 and 1918; 2 per lane at 2 and 3 waves 2067 and 2110; 4 per
// lane at 2 waves (256 VGPRs) 2182.  The extra VALU work of one particle per
// lane (139 instructions per pair in the far loop against 134.5 with four, for
// the reaction's LDS update and the loop) costs less than the latency the
// extra waves hide.  With a table a bound of 4 waves (78 VGPRs, 6 waves; 98
// with the potential, where a bound of 5 changed CIC by -2 to +1.5 %): before the
// lookup was trimmed CIC 1436 and TSC 2042 ms, against 1473 and 2200 with 2 per
// lane at 3 waves and 1441 and 2075 with the bound at 6 waves; CIC now 1192.
constexpr int waves_per_simd(int torder) { return torder > 0 ? 4 : 5; }

struct PairwiseArgs {
    const SrcRec *rec;   // [N] records in spatial order
    const double *box;   // [ceil(N/64)][8] bounding boxes of aligned runs of 64 records
    double *sum;         // [M S][4][N] FP64 sums in spatial order (x, y, z, potential)
    double L, invL, halfL, tie;  // tie: |d| within this of L/2 takes the check
    double far_h;                // largest softening sum for which the fast path is allowed
    float tie32;                 // FP32 screen for it: 0.5 L (1 - 1e-6), below every such |d|
    ImageConsts c;
    TableView tv;  // far-image table (table paths only)
    float invLf, invL2f;
    int N;
    Rounds rd;  // this launch's meetings
};

// Exact band 2 <= |n| <= n_far of one pair in one lane (delta = d/L signed,
// r = rho/L; per unit G m / L^2): the rare fallback of band tables for
// pairs beyond the table's rho range.
__device__ __noinline__ void band_serial(float delta, float r, int n_far, float &fz, float &fr) {
    const float r2 = r * r;
    float sz = 0.f, sr = 0.f;
    for (int q = n_far; q >= 2; --q) {
        const float qf = (float)q;
        const float up = delta - qf, um = delta + qf;
        const float ip = __builtin_amdgcn_rsqf(__builtin_fmaf(up, up, r2));
        const float im = __builtin_amdgcn_rsqf(__builtin_fmaf(um, um, r2));
        const float ip3 = ip * ip * ip, im3 = im * im * im;
        sz = __builtin_fmaf(-up, ip3, __builtin_fmaf(-um, im3, sz));
        sr = __builtin_fmaf(-r, ip3 + im3, sr);
    }
    fz = sz;
    fr = sr;
}

// a wave's particle
struct Owned {
    double x, y, z, m;
    float h;
    int t;  // record index, or N for an empty lane
};

struct WaveBox {
    double x0, x1, y0, y1, z0, z1, h;
};

// How the pairs between the wave's particles (box w) and the records of box b
// are evaluated.  kNear: a pair may be softened.  The others: the boxes are
// apart by more than the sum of their largest softenings (with that sum below
// L/2, so that no image n != 0 is softened either); kWrap: some axial separation
// may come near L/2, each pair takes its own minimum image and the half-period
// screen; kFar: none does, and every axial separation t = z_i - z_j of the two
// boxes has the same minimum image t - kL, returned as kL.  Evaluated alike by
// every lane.
enum { kNear = 0, kWrap = 1, kFar = 2 };

__device__ __forceinline__ int tile_kind(const PairwiseArgs &a, const WaveBox &w, const double *b, double &kL) {
    const double hs = w.h + b[6];
    if (hs > a.far_h) return kNear;
    const double gx = fmax(0.0, fmax(w.x0 - b[1], b[0] - w.x1));
    const double gy = fmax(0.0, fmax(w.y0 - b[3], b[2] - w.y1));
    // axial separations t = z_i - z_j lie in [tl, th], inside (-L, L)
    const double tl = w.z0 - b[5], th = w.z1 - b[4];
    double gz;
    if (ceil(tl * a.invL) <= floor(th * a.invL)) {
        gz = 0.0;  // a multiple of L inside: some pair may be axially aligned
    } else {
        const double el = fabs(tl - a.L * rint(tl * a.invL)), eh = fabs(th - a.L * rint(th * a.invL));
        gz = fmin(el, eh);
    }
    if (!(gx * gx + gy * gy + gz * gz > hs * hs * (1.0 + 1e-4) + 1e-300)) return kNear;
    // a separation within 1e-5 L of a half period (the screen is 5e-7 L)
    const double m = 1e-5 * a.L;
    if (ceil((tl - m) * a.invL - 0.5) <= floor((th + m) * a.invL - 0.5)) return kWrap;
    kL = a.L * floor(tl * a.invL + 0.5);
    return kFar;
}

// LDS of a workgroup: its tile's sources (SoA) and their FP64 reaction slots.
// The masses are FP32 values; with a table they are held in FP64, which saves a
// conversion and an address per pair (CIC, N = 131072: 20.6 -> 20.0 ms).  The
// exact pair keeps them in FP32: 120.6 against 127.3 ms at 262144 particles in
// clumps, |n| <= 8 with the potential (though 66.3 against 64.8 us at 4096).
template <int TORDER>
struct Stage {
    using Mass = typename std::conditional<(TORDER > 0), double, float>::type;
    double x[64], y[64], z[64];
    Mass m[64];
    double r[4][64];  // reactions, FP64
    float h[64];
};

// Reaction on the source from an evaluated pair, in the owned sums'
// orientation (dx = x_i - x_j): the source sees -dx, -dy and -d, except
// where |d| = L/2 up to rounding and its own minimum image has the sign of d.
__device__ __forceinline__ double tie_fz(const PairwiseArgs &a, double zi, double zj, double Fz64) {
    const double d64 = min_image(zi - zj, a.L, a.invL);
    if (__builtin_fabs(__builtin_fabs(d64) - a.halfL) <= a.tie) {
        const double dji = min_image(zj - zi, a.L, a.invL);
        if ((dji < 0.0) == (d64 < 0.0)) return -Fz64;
    }
    return Fz64;
}

// The table's far images of one pair (Sect. 2.2, eq. S1R2EwaldCorrectionTable)
// added to (S, Fz): R_z is odd in d and R_rho even, so the corrected pair
// keeps the symmetry of the exact one.  `self`: the pair of a particle with
// itself (no correction).
template <int TORDER, bool COMPLETE, class Nodes>
__device__ __forceinline__ void table_far(const PairwiseArgs &a, const Nodes &nodes, float dx, float dy, float d,
                                          bool self, float &S, float &Fz) {
    float rho, rinv;
    rho_of(__builtin_fmaf(dx, dx, dy * dy), rho, rinv);
    const float rr = rho * a.invLf;
    const float delta = __builtin_fabsf(d) * a.invLf;
    const bool inside = (rr <= a.tv.r_max) && !self;
    float tz, tr;
    lookup<(TORDER > 0 ? TORDER : 1)>(a.tv, nodes, delta, rr, tz, tr);
    float Rz = signed_tz(tz, d);
    float Rr = tr;
    if (!inside) {
        Rz = 0.f;
        Rr = 0.f;
        if (!self) {
            const float ds = d * a.invLf;
            if (COMPLETE) {
                // line-mass limit of the complete sum minus the images |n| <= 1
                const float r2 = rr * rr;
                float nz = 0.f, nr = 0.f;
#pragma unroll
                for (int n = -1; n <= 1; ++n) {
                    const float u = ds - (float)n;
                    const float iq = __builtin_amdgcn_rsqf(__builtin_fmaf(u, u, r2));
                    const float iq3 = iq * iq * iq;
                    nz = __builtin_fmaf(-u, iq3, nz);
                    nr = __builtin_fmaf(-rr, iq3, nr);
                }
                Rz = -nz;
                Rr = -2.f * __builtin_amdgcn_rcpf(rr) - nr;
            } else {
                band_serial(ds, rr, a.tv.n_far, Rz, Rr);
            }
        }
    }
    S = __builtin_fmaf(-Rr * a.invL2f, rinv, S);
    Fz = __builtin_fmaf(-Rz, a.invL2f, Fz);
}

// One wave's passage over a tile's sources where none is softened: n steps, lane
// l taking source l xor step.  kFar: the separation is the FP64 difference of
// the positions, with the minimum image's shift kL taken off the owned z once
// per tile, rounded to FP32 (as exact as in near_pass, with no per-pair floor);
// no half-period screen.  kWrap: both per pair (a near_pass without its screens
// for softening: N = 30011 with 4 images 1107 -> 1071 us, 200000 with 8 70.9 ->
// 69.6 ms).  FP32 pair terms, FP64 sums and reactions as in near_pass.
template <int NIMG, bool POT, int TORDER, bool COMPLETE, int KIND>
__device__ __forceinline__ void far_pass(const PairwiseArgs &a, const Owned &o, Stage<TORDER> &st, int n, double kL,
                                         double *acc) {
    const int lane = threadIdx.x & 63;
    const double zs = o.z - kL;
    for (int step = 0; step < n; ++step) {
        const int k = lane ^ step;
        const double sxj = st.x[k], syj = st.y[k], szj = st.z[k];
        const double ms = (double)st.m[k];
        double jx = 0.0, jy = 0.0, jz = 0.0, jp = 0.0;
        if (step > 0) {
            // the slot as the previous lane left it
            jx = st.r[0][k];
            jy = st.r[1][k];
            jz = st.r[2][k];
            if (POT) jp = st.r[3][k];
        }
        const double dx64 = o.x - sxj, dy64 = o.y - syj;
        const float dx = (float)dx64, dy = (float)dy64;
        const float d = (float)(KIND == kFar ? zs - szj : min_image(o.z - szj, a.L, a.invL));
        float S, Fz, P = 0.f;
        pair_fast<NIMG, POT>(dx, dy, d, a.c, S, Fz, P);
        if (TORDER > 0) table_far<TORDER, COMPLETE>(a, GlobalNodes{a.tv.T, a.tv.w}, dx, dy, d, false, S, Fz);
        const double S64 = (double)S, Fz64 = (double)Fz;
        const double mS = ms * S64;
        acc[0] = __builtin_fma(mS, dx64, acc[0]);
        acc[1] = __builtin_fma(mS, dy64, acc[1]);
        acc[2] = __builtin_fma(ms, Fz64, acc[2]);
        if (POT) acc[3] = __builtin_fma(ms, (double)P, acc[3]);
        const double miS = o.m * S64;
        st.r[0][k] = __builtin_fma(miS, dx64, jx);
        st.r[1][k] = __builtin_fma(miS, dy64, jy);
        const double fz = KIND == kWrap && __builtin_fabsf(d) >= a.tie32 ? tie_fz(a, o.z, szj, Fz64) : Fz64;
        st.r[2][k] = __builtin_fma(o.m, fz, jz);
        if (POT) st.r[3][k] = __builtin_fma(o.m, (double)P, jp);
        hand_over();
    }
}

// A pair in general position: FP64 separation and minimum image, FP32 terms.
// The n = 0 image of a pair inside its softening length takes the spline in
// FP32 (selected per pair; the separation is the FP64 one cast); with a
// softening sum above L/2 the images n != 0 may be softened too and the pair
// is evaluated in FP64 with the spline on every image (rare).  `wide`, `thr2`:
// the pair may be softened, from a bound; `self`: no term at all, images
// included.  MIRROR: evaluated at |d|, F_z then given the sign of d (0 at d = 0),
// so that a pair has the same terms bit for bit from either side (as written, sums
// over +n and -n and the compiler's contractions in them round differently at -d).
struct PairTerms {
    double dx, dy;
    float d, S, Fz, P;
};

template <int NIMG, bool POT, int TORDER, bool COMPLETE, bool MIRROR = false, class Nodes>
__device__ __forceinline__ PairTerms general_pair(const PairwiseArgs &a, const Nodes &nodes, double xi, double yi, double zi, float hi,
                                                  const SrcRec &src, float thr2, bool wide, bool self) {
    PairTerms t;
    t.dx = xi - src.x;
    t.dy = yi - src.y;
    const double signed_d = min_image(zi - src.z, a.L, a.invL);
    const double d64 = MIRROR ? __builtin_fabs(signed_d) : signed_d;
    const float dx = (float)t.dx, dy = (float)t.dy, d = (float)d64;
    t.d = d;
    const float rho2 = __builtin_fmaf(dx, dx, dy * dy);
    const float r2_0 = __builtin_fmaf(d, d, rho2);
    float T, U, Q;
    pair_images<NIMG, POT>(rho2, d, r2_0, a.c, T, U, Q);
    const float hij = hi + src.h;
    const bool near = (wide || r2_0 < thr2) && (r2_0 < hij * hij || hij > (float)a.halfL);
    float s0, p0;
    if (__ballot(near && !self) != 0) {
        float sf, pf;
        spline_n0(r2_0, hij, sf, pf);
        const float ri0 = __builtin_amdgcn_rsqf(r2_0);
        s0 = near ? sf : ri0 * ri0 * ri0;
        p0 = near ? pf : ri0;
    } else {
        const float ri0 = __builtin_amdgcn_rsqf(r2_0);
        s0 = ri0 * ri0 * ri0;
        p0 = ri0;
    }
    t.S = s0 + T;
    t.Fz = __builtin_fmaf(d, t.S, -a.c.Lf * U);
    t.P = p0 + Q;
    if (self) {
        t.S = 0.f;
        t.Fz = 0.f;
        t.P = 0.f;
    }
    if (near && hij > (float)a.halfL && !self) {
        // rare and divergent
        double gs, gf, gp;
        pair_spline_f64(t.dx, t.dy, d64, (double)hi + (double)src.h, a.L, (NIMG >= 0) ? NIMG : a.c.n_img, gs, gf, gp);
        t.S = (float)gs;
        t.Fz = (float)gf;
        t.P = (float)gp;
    }
    if (TORDER > 0) table_far<TORDER, COMPLETE>(a, nodes, dx, dy, d, self, t.S, t.Fz);
    if (MIRROR) t.Fz = signed_tz(t.Fz, (float)signed_d);
    return t;
}

// One wave's passage over a tile's sources in general position, summed in
// FP64 (the records are in spatial order, so a particle's near neighbours
// arrive together and an FP32 partial would lose their cancellation).  REACT:
// the sources are another part's and their reactions are summed in the FP64
// LDS slots; otherwise (a part against itself; the tile's first record is
// `base`, `cnt` of its sources are real) the self pair and the padding are
// skipped.
template <int NIMG, bool POT, int TORDER, bool COMPLETE, bool REACT>
__device__ __forceinline__ void near_pass(const PairwiseArgs &a, const Owned &o, Stage<TORDER> &st, int n, int base, int cnt,
                                          float hmax, double *acc) {
    const int lane = threadIdx.x & 63;
    const float hb = o.h + hmax;  // >= h_i + h_j for every source of the tile
    const float thr2 = hb * hb;
    const bool wide = hb > (float)a.halfL;
    for (int step = 0; step < n; ++step) {
        const int k = lane ^ step;
        SrcRec src;
        src.x = st.x[k];
        src.y = st.y[k];
        src.z = st.z[k];
        src.h = st.h[k];
        const int ks = k & (n - 1);  // source of the tile
        const bool self = !REACT && (base + ks == o.t || ks >= cnt);
        const PairTerms t =
            general_pair<NIMG, POT, TORDER, COMPLETE>(a, GlobalNodes{a.tv.T, a.tv.w}, o.x, o.y, o.z, o.h, src, thr2, wide, self);
        const double ms = (double)st.m[k];
        double jx = 0.0, jy = 0.0, jz = 0.0, jp = 0.0;
        if (REACT && step > 0) {
            // the slot as the previous lane left it
            jx = st.r[0][k];
            jy = st.r[1][k];
            jz = st.r[2][k];
            if (POT) jp = st.r[3][k];
        }
        const double S64 = (double)t.S, Fz64 = (double)t.Fz;
        const double mS = ms * S64;
        acc[0] = __builtin_fma(mS, t.dx, acc[0]);
        acc[1] = __builtin_fma(mS, t.dy, acc[1]);
        acc[2] = __builtin_fma(ms, Fz64, acc[2]);
        if (POT) acc[3] = __builtin_fma(ms, (double)t.P, acc[3]);
        if (REACT) {
            const double fz = __builtin_fabsf(t.d) >= a.tie32 ? tie_fz(a, o.z, src.z, Fz64) : Fz64;
            const double miS = o.m * S64;
            st.r[0][k] = __builtin_fma(miS, t.dx, jx);
            st.r[1][k] = __builtin_fma(miS, t.dy, jy);
            st.r[2][k] = __builtin_fma(o.m, fz, jz);
            if (POT) st.r[3][k] = __builtin_fma(o.m, (double)t.P, jp);
            hand_over();
        }
    }
}

// Few particles (N <= kSmallMax): every ordered pair, one wave per target with
// the sources over its lanes, straight from the caller's arrays to the
// outputs.  What bounds such a call is the chain of launches and the workspace
// around it (N = 500, |n| <= 2: 66 us in ten launches), so this form has one
// launch and no workspace (13 us, most of it the host's).  Two targets per
// wave took 33 us against 29 at N = 2000.  The pair term of (j, i) is that of
// (i, j) with the signs turned, bit for bit (MIRROR), so momentum is conserved as
// in the pairwise form.  The lanes' FP64 sums are added in a fixed tree.
struct SmallArgs {
    PairwiseArgs a;
    const double *pos, *mass, *eps;
    float *acc, *pot;
};

template <int NIMG, bool POT, int TORDER, bool COMPLETE>
__global__ __launch_bounds__(256) void forces_small_kernel(SmallArgs p) {
    const PairwiseArgs &a = p.a;
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= a.N) return;  // whole wave
    const double *x = p.pos, *y = p.pos + a.N, *z = p.pos + 2 * a.N;
    const double xi = x[i], yi = y[i], zi = wrap_z(z[i], a.L);
    const float hi = (float)p.eps[i];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int j0 = 0; j0 < a.N; j0 += 64) {
        const int j = j0 + lane;
        const bool live = j < a.N;
        const int js = live ? j : a.N - 1;
        SrcRec src;
        src.x = x[js];
        src.y = y[js];
        src.z = wrap_z(z[js], a.L);
        src.m = (float)p.mass[js];
        src.h = (float)p.eps[js];
        const PairTerms t =
            general_pair<NIMG, POT, TORDER, COMPLETE, true>(a, GlobalNodes{a.tv.T, a.tv.w}, xi, yi, zi, hi, src, 0.f,
                                                            true, !live || j == i);
        const double ms = (double)src.m, mS = ms * (double)t.S;
        acc[0] = __builtin_fma(mS, t.dx, acc[0]);
        acc[1] = __builtin_fma(mS, t.dy, acc[1]);
        acc[2] = __builtin_fma(ms, (double)t.Fz, acc[2]);
        if (POT) acc[3] = __builtin_fma(ms, (double)t.P, acc[3]);
    }
#pragma unroll
    for (int c = 0; c < (POT ? 4 : 3); ++c) {
        for (int off = 32; off >= 1; off >>= 1) acc[c] += __shfl_xor(acc[c], off);
        if (lane == 0) {
            float *o = c < 3 ? p.acc + (int64_t)c * a.N : p.pot;
            o[i] = (float)(-acc[c]);
        }
    }
}

// One tile: tiles i <= j of every group (round 0), then S^2 per meeting of the
// launch's other rounds.  SPLIT: by several waves, in flat calls.  In the one-wave
// form n is left to run time and barriers stand where a fence would do, for what the
// compiler makes of the loops: with 64 for n and fences N = 131072, |n| <= 8, takes
// 28.0 ms without the potential in place of 27.0, with 64 and barriers 32.1 in place
// of 30.0 with it.
template <int NIMG, bool POT, int TORDER, bool COMPLETE, bool SPLIT>
__global__ __launch_bounds__(SPLIT ? 64 * kSplit : 64, waves_per_simd(TORDER)) void forces_pairwise_kernel(
    PairwiseArgs a) {
    __shared__ Stage<TORDER> one;
    extern __shared__ double each[];  // SPLIT: a Stage per wave
    Stage<TORDER> *const stages = SPLIT ? reinterpret_cast<Stage<TORDER> *>(each) : &one;
    const int lane = SPLIT ? threadIdx.x & 63 : threadIdx.x;
    const int wave = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    Stage<TORDER> &st = stages[wave];
    const Tile t = tile_of(a.rd, blockIdx.x);
    const int n = kPart / (SPLIT ? (int)blockDim.x / 64 : a.rd.Q);              // sources of the wave
    const int64_t g0 = min((int64_t)a.N, (int64_t)t.pa * kPart);                // first owned record
    const int64_t b0 = min((int64_t)a.N, (int64_t)t.pb * kPart + wave * n);     // first source record
    const int ocnt = (int)min((int64_t)kPart, (int64_t)a.N - g0);               // owned records
    const int cnt = (int)min((int64_t)n, (int64_t)a.N - b0);                    // sources
    const bool react = t.pa != t.pb;
    // the owned particles' slot and the sources'
    double *pa = a.sum + (int64_t)t.slot_a * 4 * a.N + g0;
    double *pb = a.sum + (int64_t)t.slot_b * 4 * a.N + b0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int out = lane;
    if (ocnt > 0 && cnt > 0) {
        // an empty lane copies the part's first record with no mass (it sits
        // where a particle is, so every pair distance stays that of a real pair)
        Owned o;
        const bool real = lane < ocnt;
        const SrcRec rr = a.rec[real ? g0 + lane : g0];
        o.t = real ? (int)g0 + lane : a.N;
        o.x = rr.x;
        o.y = rr.y;
        o.z = rr.z;
        o.h = rr.h;
        o.m = real ? (double)rr.m : 0.0;
        // a partly filled tile is padded with massless copies of its first record
        const int ks = lane & (n - 1);
        const bool live = ks < cnt;
        const SrcRec sr = a.rec[live ? b0 + ks : b0];
        st.x[lane] = sr.x;
        st.y[lane] = sr.y;
        st.z[lane] = sr.z;
        st.m[lane] = live ? sr.m : 0.f;
        st.h[lane] = sr.h;
        const double *w = a.box + (g0 >> 6) * kBox, *b = a.box + (b0 >> 6) * kBox;
        const WaveBox wb = {w[0], w[1], w[2], w[3], w[4], w[5], w[6]};
        if (SPLIT)
            hand_over();
        else
            __syncthreads();
        double kL = 0.0;
        const int kind = react ? __builtin_amdgcn_readfirstlane(tile_kind(a, wb, b, kL)) : kNear;
        if (!react)
            near_pass<NIMG, POT, TORDER, COMPLETE, false>(a, o, st, n, (int)b0, cnt, (float)b[6], acc);
        else if (kind == kFar)
            far_pass<NIMG, POT, TORDER, COMPLETE, kFar>(a, o, st, n, kL, acc);
        else if (kind == kWrap)
            far_pass<NIMG, POT, TORDER, COMPLETE, kWrap>(a, o, st, n, kL, acc);
        else
            near_pass<NIMG, POT, TORDER, COMPLETE, true>(a, o, st, n, (int)b0, cnt, (float)b[6], acc);
        if (SPLIT)
            hand_over();
        else
            __syncthreads();
        // the lane's addresses are formed here: held over the loops they would cost 4 VGPRs
        asm volatile("" : "+v"(out));
        if (react && out < cnt) {
            // reactions on the sources, in the owned sums' orientation
#pragma unroll
            for (int c = 0; c < (POT ? 4 : 3); ++c) {
                double v = st.r[c][out];
                for (int e = n; e < kPart; e += n) v += st.r[c][out + e];
                if (c < 3) v = -v;
                double *p = pb + (int64_t)c * a.N;
                p[out] = a.rd.first ? v : p[out] + v;
            }
        }
    } else if (a.rd.first && react && lane < cnt) {
#pragma unroll
        for (int c = 0; c < (POT ? 4 : 3); ++c) pb[(int64_t)c * a.N + lane] = 0.0;
    }
    if (SPLIT) {
        // the waves' sums of the part, in wave order
        hand_over();
        double *const mine[4] = {st.x, st.y, st.z, st.r[3]};
#pragma unroll
        for (int c = 0; c < (POT ? 4 : 3); ++c) mine[c][lane] = acc[c];
        __syncthreads();
        if (wave > 0) return;
        for (int w = 1; w < (int)blockDim.x / 64; ++w) {
            const double *const other[4] = {stages[w].x, stages[w].y, stages[w].z, stages[w].r[3]};
#pragma unroll
            for (int c = 0; c < (POT ? 4 : 3); ++c) acc[c] += other[c][lane];
        }
    }
    if (out < ocnt && (a.rd.first || cnt > 0)) {
#pragma unroll
        for (int c = 0; c < (POT ? 4 : 3); ++c) {
            double *p = pa + (int64_t)c * a.N;
            p[out] = a.rd.first ? acc[c] : p[out] + acc[c];
        }
    }
}

// ---------------------------------------------------------------------------
// TSC tables that fit the LDS.  A TSC pair gathers nine nodes in six loads, 56
// cache accesses each, and what bounds it is the rate of those (address units
// 77% busy, VALU 56%, 930 cycles a step where the VALU work takes 430), so here
// the whole table sits in the LDS of a workgroup of 16 waves, one to a CU, each
// walking its share of the launch's tiles.  That leaves no room for staged
// sources: a lane holds one source and its reaction sums in registers, and after
// each step they move to another lane, by a Gray code of exchanges (DPP for two
// out of three, a permute for each fourth step), so that every lane meets every
// source.  us per call: N = 10000 393 -> 269, 20011 (with the potential) 1272 ->
// 1024, 40000 4342 -> 3332, 100000 23800 -> 19100; what bounds it then is bank
// conflicts of the gathers and the VALU (124 instructions) about alike, and with the
// potential 128 registers: 68 bytes of scratch a lane with a complete table, 80 with
// a band, four of whose loads and stores fall in each step of the far loop (20011
// particles, complete: 962 us).
constexpr int kLdsWaves = 16;
constexpr int kLdsNodes = 20480;  // 160 KiB
constexpr int kLdsGroups = 256;   // one per CU
// From this many particles on: 4096 waves with 55 us a tile (us per call from L2
// and from LDS: N = 4000 80 and 86, 5000 121 and 83, 6000 153 and 141).
constexpr int kLdsMin = 4500;

inline bool lds_table(const TableView &tv, int64_t N) {
    return N >= kLdsMin && tv.w * (tv.n_r + 3) <= kLdsNodes;
}

// The mass moves in FP32, which leaves the form with the potential a register more
// (32 x 32 nodes, N = 6000: 150 us, with an FP64 mass 155 to 185 by what else spills).
struct MovingSource {
    double x, y, z;
    double r[4];  // reactions
    float m, h;
};

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t u) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)u, CTRL, 0xf, 0xf, true);
}

template <class F>
__device__ __forceinline__ void each_dword(double &v, F &&f) {
    const uint64_t u = __double_as_longlong(v);
    v = __longlong_as_double((long long)((uint64_t)f((uint32_t)u) | (uint64_t)f((uint32_t)(u >> 32)) << 32));
}

template <bool POT, bool NEAR, class F>
__device__ __forceinline__ void move_source(MovingSource &s, F &&f) {
    each_dword(s.x, f);
    each_dword(s.y, f);
    each_dword(s.z, f);
    s.m = __uint_as_float(f(__float_as_uint(s.m)));
#pragma unroll
    for (int c = 0; c < (POT ? 4 : 3); ++c) each_dword(s.r[c], f);
    if (NEAR) s.h = __uint_as_float(f(__float_as_uint(s.h)));
}

// One wave's passage over the 64 sources of a tile of a kind (kFar: image shift
// kL); the tile's first record is `base`, `cnt` of its sources are real.
// Returns the source that the lane ends with.
template <bool POT, bool COMPLETE, int KIND>
__device__ __forceinline__ int lds_pass(const PairwiseArgs &a, const LdsNodes &nodes, const Owned &o, MovingSource &s,
                                         double kL, bool react, int base, int cnt, double *acc) {
    const int lane = threadIdx.x & 63;
    const double zs = o.z - kL;
    int at = lane;  // the source that this lane holds
    auto step = [&] {
        double dx, dy;
        float S, Fz, P = 0.f, d;
        if (KIND != kNear) {
            dx = o.x - s.x;
            dy = o.y - s.y;
            d = (float)(KIND == kFar ? zs - s.z : min_image(o.z - s.z, a.L, a.invL));
            pair_fast<1, POT>((float)dx, (float)dy, d, a.c, S, Fz, P);
            table_far<2, COMPLETE>(a, nodes, (float)dx, (float)dy, d, false, S, Fz);
        } else {
            const SrcRec src = {s.x, s.y, s.z, 0.f, s.h};
            const bool self = !react && (base + at == o.t || at >= cnt);
            const PairTerms t =
                general_pair<1, POT, 2, COMPLETE>(a, nodes, o.x, o.y, o.z, o.h, src, 0.f, true, self);
            dx = t.dx;
            dy = t.dy;
            d = t.d;
            S = t.S;
            Fz = t.Fz;
            P = t.P;
        }
        const double S64 = (double)S, Fz64 = (double)Fz;
        const double ms = (double)s.m, mS = ms * S64;
        acc[0] = __builtin_fma(mS, dx, acc[0]);
        acc[1] = __builtin_fma(mS, dy, acc[1]);
        acc[2] = __builtin_fma(ms, Fz64, acc[2]);
        if (POT) acc[3] = __builtin_fma(ms, (double)P, acc[3]);
        const double fz = KIND != kFar && react && __builtin_fabsf(d) >= a.tie32 ? tie_fz(a, o.z, s.z, Fz64) : Fz64;
        const double miS = o.m * S64;
        s.r[0] = __builtin_fma(miS, dx, s.r[0]);
        s.r[1] = __builtin_fma(miS, dy, s.r[1]);
        s.r[2] = __builtin_fma(o.m, fz, s.r[2]);
        if (POT) s.r[3] = __builtin_fma(o.m, (double)P, s.r[3]);
    };
    auto permute = [&](int mask) {
        const int from = (lane ^ mask) * 4;
        move_source<POT, KIND == kNear>(s, [&](uint32_t u) { return (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)u); });
        at ^= mask;
    };
    auto by1 = [&] {  // lane xor 1
        move_source<POT, KIND == kNear>(s, [](uint32_t u) { return dpp_move<0xB1>(u); });
        at ^= 1;
    };
    auto by2 = [&] {  // lane xor 2
        move_source<POT, KIND == kNear>(s, [](uint32_t u) { return dpp_move<0x4E>(u); });
        at ^= 2;
    };
    for (int k = 1;; ++k) {
        step();
        by1();
        step();
        by2();
        step();
        by1();
        step();
        if (k == 16) break;
        permute(4 << __builtin_ctz(k));  // lane xor 4, 8, 4, 16, 4, 8, 4, 32, ...
    }
    return at;
}

template <bool POT, bool COMPLETE>
__global__ __launch_bounds__(64 * kLdsWaves) void forces_pairwise_lds_kernel(PairwiseArgs a, unsigned tiles) {
    __shared__ float2 T[kLdsNodes];
    const int nodes = a.tv.w * (a.tv.n_r + 3);
    for (int i = threadIdx.x; i < nodes; i += 64 * kLdsWaves) T[i] = a.tv.T[i];
    __syncthreads();
    const LdsNodes table = {T, a.tv.w};
    const int lane = threadIdx.x & 63;
    const unsigned wave = __builtin_amdgcn_readfirstlane(blockIdx.x * kLdsWaves + (threadIdx.x >> 6));
    for (unsigned at = wave; at < tiles; at += gridDim.x * kLdsWaves) {
        const Tile t = tile_of(a.rd, at);
        const int64_t g0 = min((int64_t)a.N, (int64_t)t.pa * kPart);   // first owned record
        const int64_t b0 = min((int64_t)a.N, (int64_t)t.pb * kPart);   // first source record
        const int ocnt = (int)min((int64_t)kPart, (int64_t)a.N - g0);  // owned records
        const int cnt = (int)min((int64_t)kPart, (int64_t)a.N - b0);   // sources
        const bool react = t.pa != t.pb;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        double *pa = a.sum + (int64_t)t.slot_a * 4 * a.N + g0;
        double *pb = a.sum + (int64_t)t.slot_b * 4 * a.N + b0;
        int source = lane;  // the source whose reaction this lane ends with
        MovingSource s;
#pragma unroll
        for (int c = 0; c < 4; ++c) s.r[c] = 0.0;
        if (ocnt > 0 && cnt > 0) {
            // empty lanes as in forces_pairwise_kernel
            Owned o;
            const bool real = lane < ocnt, live = lane < cnt;
            const SrcRec rr = a.rec[real ? g0 + lane : g0], sr = a.rec[live ? b0 + lane : b0];
            o.t = real ? (int)g0 + lane : a.N;
            o.x = rr.x;
            o.y = rr.y;
            o.z = rr.z;
            o.h = rr.h;
            o.m = real ? (double)rr.m : 0.0;
            s.x = sr.x;
            s.y = sr.y;
            s.z = sr.z;
            s.h = sr.h;
            s.m = live ? sr.m : 0.f;
            const double *w = a.box + (g0 >> 6) * kBox;
            const WaveBox wb = {w[0], w[1], w[2], w[3], w[4], w[5], w[6]};
            double kL = 0.0;
            const int kind =
                react ? __builtin_amdgcn_readfirstlane(tile_kind(a, wb, a.box + (b0 >> 6) * kBox, kL)) : kNear;
            if (kind == kFar)
                source = lds_pass<POT, COMPLETE, kFar>(a, table, o, s, kL, true, (int)b0, cnt, acc);
            else if (kind == kWrap)
                source = lds_pass<POT, COMPLETE, kWrap>(a, table, o, s, 0.0, true, (int)b0, cnt, acc);
            else
                source = lds_pass<POT, COMPLETE, kNear>(a, table, o, s, 0.0, react, (int)b0, cnt, acc);
        }
        if (react && source < cnt && (a.rd.first || ocnt > 0)) {
#pragma unroll
            for (int c = 0; c < (POT ? 4 : 3); ++c) {
                const double v = c < 3 ? -s.r[c] : s.r[c];
                double *p = pb + (int64_t)c * a.N + source;
                *p = a.rd.first ? v : *p + v;
            }
        }
        if (lane < ocnt && (a.rd.first || cnt > 0)) {
#pragma unroll
            for (int c = 0; c < (POT ? 4 : 3); ++c) {
                double *p = pa + (int64_t)c * a.N + lane;
                *p = a.rd.first ? acc[c] : *p + acc[c];
            }
        }
    }
}

template <int NIMG, bool POT, int TORDER, bool COMPLETE>
struct Launcher {
    static hipError_t small(const SmallArgs &p, hipStream_t stream) {
        hipLaunchKernelGGL((forces_small_kernel<NIMG, POT, TORDER, COMPLETE>), dim3((p.a.N + 3) / 4), dim3(256), 0,
                           stream, p);
        return hipGetLastError();
    }

    static hipError_t run(PairwiseArgs a, const Schedule &s, hipStream_t stream) {
        if constexpr (TORDER == 2) {
            if (lds_table(a.tv, a.N))
                return each_launch(s, a.N, kPart, [&](const Rounds &rd, unsigned tiles) {
                    a.rd = rd;
                    hipLaunchKernelGGL((forces_pairwise_lds_kernel<POT, COMPLETE>), dim3(kLdsGroups),
                                       dim3(64 * kLdsWaves), 0, stream, a, tiles);
                    return hipGetLastError();
                });
        }
        // Tiles are split while they would not fill the device (us per call over 1, 2
        // and 4 waves: |n| <= 8 N = 4096 75, 65, 59; 6000 111, 102, 101; 8000 161, 160,
        // 158; 9000 196, 196, 198; CIC 4096 58, 59, 54; 8000 131, 131, 136; TSC from the
        // caches, which more waves share, 2800 55, 46, 47).
        const int64_t tiles = (int64_t)s.S * (s.S + 1) / 2;
        const int waves = !s.flat ? 1 : tiles <= (TORDER == 2 ? 1024 : 4096) ? kSplit : tiles <= 8192 ? 2 : 1;
        return each_launch(s, a.N, kPart, [&](const Rounds &rd, unsigned blocks) {
            a.rd = rd;
            if (waves > 1)
                hipLaunchKernelGGL((forces_pairwise_kernel<NIMG, POT, TORDER, COMPLETE, true>), dim3(blocks),
                                   dim3(64 * waves), waves * sizeof(Stage<TORDER>), stream, a);
            else
                hipLaunchKernelGGL((forces_pairwise_kernel<NIMG, POT, TORDER, COMPLETE, false>), dim3(blocks), dim3(64),
                                   0, stream, a);
            return hipGetLastError();
        });
    }
};

// Calls f(Launcher<...>{}) for the kernel instance of (n_img, pot, table order, complete).
template <class F>
auto dispatch(int n_img, bool pot, int order, bool complete, F &&f) {
    if (order == 0) {
        // image counts unrolled at compile time, the others by the run-time loop
        if (pot) {
            switch (n_img) {
                case 0: return f(Launcher<0, true, 0, false>{});
                case 1: return f(Launcher<1, true, 0, false>{});
                case 2: return f(Launcher<2, true, 0, false>{});
                case 4: return f(Launcher<4, true, 0, false>{});
                case 8: return f(Launcher<8, true, 0, false>{});
                default: return f(Launcher<-1, true, 0, false>{});
            }
        }
        switch (n_img) {
            case 0: return f(Launcher<0, false, 0, false>{});
            case 1: return f(Launcher<1, false, 0, false>{});
            case 2: return f(Launcher<2, false, 0, false>{});
            case 4: return f(Launcher<4, false, 0, false>{});
            case 8: return f(Launcher<8, false, 0, false>{});
            default: return f(Launcher<-1, false, 0, false>{});
        }
    }
    if (order == 1) {
        if (pot) return complete ? f(Launcher<1, true, 1, true>{}) : f(Launcher<1, true, 1, false>{});
        return complete ? f(Launcher<1, false, 1, true>{}) : f(Launcher<1, false, 1, false>{});
    }
    if (pot) return complete ? f(Launcher<1, true, 2, true>{}) : f(Launcher<1, true, 2, false>{});
    return complete ? f(Launcher<1, false, 2, true>{}) : f(Launcher<1, false, 2, false>{});
}

}  // namespace

namespace {

Schedule pairwise_schedule(int64_t N, size_t budget) {
    // groups of 16 parts, 8 above 2^21 particles, where a call has enough
    // meetings and the slots would grow past 1 GiB
    return make_schedule(N, kPart, N <= ((int64_t)1 << 21) ? 16 : 8, budget);
}

// The schedule in a workspace too small for the default one: two sets of slots
// (1 KiB per particle up to 2^21), one with a table.  It takes a launch per round
// or two (us per call, default and this one, |n| <= 8: N = 4096 59 and 91, 15000
// 482 and 707, 30000 1770 and 2115, 60000 6800 and 7120).
Schedule lean_schedule(int64_t N, bool table) {
    const int S = N <= ((int64_t)1 << 21) ? 16 : 8;
    return make_schedule(N, kPart, S, (size_t)(table ? 1 : 2) * S * N * kSetBytes);
}

size_t schedule_bytes(int64_t N, const Schedule &s) {
    if (N <= kSmallMax) return 0;
    const int64_t nbox = (N + 63) / 64;
    return ws_total({N >= kSortMin ? order_targets_bytes(N) : 0, (size_t)N * sizeof(SrcRec),
                     (size_t)nbox * kBox * sizeof(double), slot_bytes(s, N)});
}

}  // namespace

size_t pairwise_bytes(int64_t N, size_t slot_budget) { return schedule_bytes(N, pairwise_schedule(N, slot_budget)); }

// Launches the pairwise path for all N particles: exact images |n| <= n_img,
// or (table non-null) images |n| <= 1 plus the table's far images with CIC
// (order 1) or TSC (order 2) interpolation.  Arguments already validated.
// Scratch (spatial order, records, boxes, FP64 sums) comes from `ws`.
int launch_forces_pairwise(const double *pos, const double *mass, const double *eps, int64_t N, double L,
                           int n_img, const steps_cyl_table *table, int order, float *out_acc, float *out_pot,
                           Workspace &ws, hipStream_t stream, size_t slot_budget) {
    Schedule sch = pairwise_schedule(N, slot_budget);
    if (slot_budget == 0 && ws.size < schedule_bytes(N, sch)) {
        const Schedule lean = lean_schedule(N, table != nullptr);
        if (schedule_bytes(N, lean) < schedule_bytes(N, sch)) sch = lean;
    }
    int rc = check_workspace(ws, schedule_bytes(N, sch));
    if (rc) return rc;
    PairwiseArgs a;
    a.L = L;
    a.invL = 1.0 / L;
    a.halfL = 0.5 * L;
    a.tie = 1e-12 * L;
    a.far_h = 0.49 * L;
    a.tie32 = (float)(0.5 * L * (1.0 - 1e-6));
    a.c.Lf = (float)L;
    a.c.L2f = (float)(L * L);
    a.c.m2Lf = (float)(-2.0 * L);
    a.c.n_img = table ? 1 : n_img;
    a.invLf = (float)(1.0 / L);
    a.invL2f = (float)(1.0 / (L * L));
    if (table) a.tv = table_view(table);
    a.N = (int)N;
    const int ord = table ? order : 0;
    const bool complete = table && table->complete != 0;

    if (N <= kSmallMax) {
        SmallArgs p;
        p.a = a;
        p.pos = pos;
        p.mass = mass;
        p.eps = eps;
        p.acc = out_acc;
        p.pot = out_pot;
        return hip_status(
            dispatch(a.c.n_img, out_pot != nullptr, ord, complete, [&](auto l) { return l.small(p, stream); }),
            "forces_pairwise launch");
    }
    const int *perm = nullptr;
    if (N >= kSortMin && (rc = order_targets(pos, N, L, nullptr, N, stream, ws, &perm))) return rc;
    const int64_t nbox = (N + 63) / 64;
    SrcRec *rec = (SrcRec *)ws.take((size_t)N * sizeof(SrcRec));
    double *box = (double *)ws.take((size_t)nbox * kBox * sizeof(double));
    double *sum = (double *)ws.take(slot_bytes(sch, N));
    if (!rec || !box || !sum) return fail(STEPS_EINVAL, "workspace too small for the pairwise path");
    a.rec = rec;
    a.box = box;
    a.sum = sum;
    hipError_t e = launch_stage(pos, mass, eps, (int)N, L, perm, rec, box, stream);
    if (e == hipSuccess)
        e = dispatch(a.c.n_img, out_pot != nullptr, ord, complete, [&](auto l) { return l.run(a, sch, stream); });
    if (e == hipSuccess) e = launch_finish(sch, a.sum, kPart, perm, (int)N, out_acc, N, out_pot, stream);
    return hip_status(e, "forces_pairwise launch");
}

}  // namespace steps
