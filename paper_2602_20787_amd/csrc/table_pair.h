// Device side of the tabulated far-image correction, shared by the table
// force kernel and the octree walk: the table object, a view of it for
// kernels, the CIC/TSC lookup, the exact band shared by a wave, and the pair
// interaction of the tabulated scheme (exact images |n| <= 1, softened, plus
// the interpolated band; Sect. 2.2, eq. S1R2EwaldCorrectionTable).
#pragma once

#include "common.h"
#include "pair_f64.h"
#include "pair_fp32.h"

struct steps_cyl_table {
    float2 *nodes = nullptr;     // [(n_r + 3) * (n_d + 3)], node (i, j) at (j + 1) * (n_d + 3) + i + 1
    double2 *nodes64 = nullptr;  // the same nodes in FP64
    int n_d = 0, n_r = 0, n_far = 0;
    int complete = 0;            // 1: every image |n| >= 2 (Ewald build)
    double r_max = 0.0;
};

namespace steps {

// what a kernel needs of a table (passed by value)
struct TableView {
    const float2 *T;
    float inv_hd, inv_hr, r_max;
    int n_d, n_r, n_far, w, complete;
};

inline TableView table_view(const steps_cyl_table *t) {
    TableView v;
    v.T = t->nodes;
    v.inv_hd = (float)(2.0 * t->n_d);
    v.inv_hr = (float)(t->n_r / t->r_max);
    v.r_max = (float)t->r_max;
    v.n_d = t->n_d;
    v.n_r = t->n_r;
    v.n_far = t->n_far;
    v.w = t->n_d + 3;
    v.complete = t->complete;
    return v;
}

// period-dependent constants of the pair interaction
struct PeriodConsts {
    double L, invL, halfL;
    float invLf, invL2f;
    ImageConsts c;  // n_img = 1
};

inline PeriodConsts period_consts(double L) {
    PeriodConsts p;
    p.L = L;
    p.invL = 1.0 / L;
    p.halfL = 0.5 * L;
    p.invLf = (float)(1.0 / L);
    p.invL2f = (float)(1.0 / (L * L));
    p.c.Lf = (float)L;
    p.c.L2f = (float)(L * L);
    p.c.m2Lf = (float)(-2.0 * L);
    p.c.n_img = 1;
    return p;
}

// exact band of one pair shared by the wave (see the learned kernel)
__device__ __forceinline__ void band_wave(float delta, float r, int n_far, float &fz, float &fr) {
    const int lane = threadIdx.x & 63;
    const float r2 = r * r;
    float sz = 0.f, sr = 0.f;
    for (int q = 2 + lane + 64 * ((n_far - 2 - lane) / 64 + 1); q >= 2; q -= 64) {
        if (q <= n_far) {
            const float qf = (float)q;
            const float up = delta - qf, um = delta + qf;
            const float ip = __builtin_amdgcn_rsqf(__builtin_fmaf(up, up, r2));
            const float im = __builtin_amdgcn_rsqf(__builtin_fmaf(um, um, r2));
            const float ip3 = ip * ip * ip, im3 = im * im * im;
            sz = __builtin_fmaf(-up, ip3, __builtin_fmaf(-um, im3, sz));
            sr = __builtin_fmaf(-r, ip3 + im3, sr);
        }
    }
    for (int off = 32; off >= 1; off >>= 1) {
        sz += __shfl_xor(sz, off);
        sr += __shfl_xor(sr, off);
    }
    fz = sz;
    fr = sr;
}

// rho and 1/rho of a pair (both 0 on the axis) from one reciprocal square root:
// the correctly rounded square root and the reciprocal of it took 18 VALU
// instructions more, of the 107 of a CIC pair in the pairwise kernel.  rho is within
// 1.5 ulp, 1/rho within one where the reciprocal of the root was within 1.5.  With
// rho correctly rounded (a Newton step, 1.4 % longer) the accelerations' rms error
// against 64 bits is the same within 3 % and larger in 21 of 24 calls (272 to 24893
// particles, both orders and kinds of table, 3.3e-8 to 9.4e-8).
__device__ __forceinline__ void rho_of(float rho2, float &rho, float &rinv) {
    rinv = rho2 >= 1.17549435e-38f ? __builtin_amdgcn_rsqf(rho2) : 0.f;
    rho = rho2 * rinv;
}

// The correctly rounded square root: a Newton step on the hardware's reciprocal
// square root gives it for every finite x >= 2^-64 (compared with the library's
// for every such float), in 5 instructions against 19.
constexpr float kSqrtMin = 0x1p-64f;

__device__ __forceinline__ float sqrt_newton(float x) {
    const float q = __builtin_amdgcn_rsqf(x);
    const float s = x * q;
    return __builtin_fmaf(__builtin_fmaf(-s, s, x), 0.5f * q, s);
}

__device__ __forceinline__ float sqrt_exact(float x) {
    float r = sqrt_newton(x);
    if (__builtin_expect(!(x >= kSqrtMin && x < __builtin_inff()), 0)) r = __builtin_sqrtf(x);
    return r;
}

// T_z carries the sign of d (odd in d, 0 at d = 0)
__device__ __forceinline__ float signed_tz(float tz, float d) {
    const float v = __uint_as_float(__float_as_uint(tz) ^ (__float_as_uint(d) & 0x80000000u));
    return d != 0.f ? v : 0.f;
}

// two neighbouring nodes of a row, one load
struct __attribute__((packed, aligned(8))) NodePair {
    float2 a, b;
};

// Byte offsets are 32-bit from uniform row pointers, so that a node costs one
// multiply-add and its rows share the offset.
template <class T>
__device__ __forceinline__ T node_at(const float2 *row, unsigned off) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(row) + off);
}

// Where a lookup reads the nodes: two neighbours, or one, of row `row` and the
// columns from `col` on, at byte offset `off`.
struct GlobalNodes {
    const float2 *T;
    int w;
    __device__ NodePair pair(int row, int col, unsigned off) const { return node_at<NodePair>(T + row * w + col, off); }
    __device__ float2 one(int row, int col, unsigned off) const { return node_at<float2>(T + row * w + col, off); }
};

struct LdsNodes {
    const float2 *T;
    int w;
    __device__ NodePair pair(int row, int col, unsigned off) const {
        const float2 *p = T + row * w + col + off / (unsigned)sizeof(float2);
        return NodePair{p[0], p[1]};
    }
    __device__ float2 one(int row, int col, unsigned off) const {
        return T[row * w + col + off / (unsigned)sizeof(float2)];
    }
};

// The instruction's own conversion: NaN and negative numbers give 0, larger ones
// than fit 2^32 - 1.  In the language a number beyond the range has none.  (Bounded
// in FP32 before the conversion instead, the TSC kernel with the potential spills
// eight registers more: band tables of 32 x 32, N = 6000, 157 -> 195 us.)
__device__ __forceinline__ unsigned saturated(float x) {
    unsigned v;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(v) : "v"(x));
    return v;
}

template <int ORDER, class Nodes>
__device__ __forceinline__ void lookup(const TableView &a, const Nodes &nodes, float delta, float r, float &tz,
                                       float &tr) {
    // the positions in the cell by explicit fused operations: they do not depend
    // on what the compiler can contract
    const float x = delta * a.inv_hd, y = r * a.inv_hr;
    tz = 0.f;
    tr = 0.f;
    if (ORDER == 1) {
        // indices clamped into the table whatever the input
        const unsigned i0 = min(saturated(x), (unsigned)(a.n_d - 1)), j0 = min(saturated(y), (unsigned)(a.n_r - 1));
        const float fx = __builtin_fmaf(delta, a.inv_hd, -(float)i0), fy = __builtin_fmaf(r, a.inv_hr, -(float)j0);
        const unsigned off = (__umul24(j0, (unsigned)a.w) + i0) * (unsigned)sizeof(float2);
        const NodePair lo = nodes.pair(1, 1, off), hi = nodes.pair(2, 1, off);
        const float z0 = __builtin_fmaf(fx, lo.b.x - lo.a.x, lo.a.x), z1 = __builtin_fmaf(fx, hi.b.x - hi.a.x, hi.a.x);
        const float r0 = __builtin_fmaf(fx, lo.b.y - lo.a.y, lo.a.y), r1 = __builtin_fmaf(fx, hi.b.y - hi.a.y, hi.a.y);
        tz = __builtin_fmaf(fy, z1 - z0, z0);
        tr = __builtin_fmaf(fy, r1 - r0, r0);
    } else {
        const unsigned i0 = min(saturated(__builtin_rintf(x)), (unsigned)a.n_d);
        const unsigned j0 = min(saturated(__builtin_rintf(y)), (unsigned)a.n_r);
        const float fx = __builtin_fmaf(delta, a.inv_hd, -(float)i0), fy = __builtin_fmaf(r, a.inv_hr, -(float)j0);
        const float ax0 = 0.5f - fx, ax2 = 0.5f + fx, ay0 = 0.5f - fy, ay2 = 0.5f + fy;
        const float wx[3] = {0.5f * ax0 * ax0, __builtin_fmaf(-fx, fx, 0.75f), 0.5f * ax2 * ax2};
        const float wy[3] = {0.5f * ay0 * ay0, __builtin_fmaf(-fy, fy, 0.75f), 0.5f * ay2 * ay2};
        const unsigned off = (__umul24(j0, (unsigned)a.w) + i0) * (unsigned)sizeof(float2);  // node (i0 - 1, j0 - 1)
#pragma unroll
        for (int dj = 0; dj < 3; ++dj) {
            const NodePair p = nodes.pair(dj, 0, off);
            const float2 q = nodes.one(dj, 2, off);
            const float rz = __builtin_fmaf(wx[2], q.x, __builtin_fmaf(wx[1], p.b.x, wx[0] * p.a.x));
            const float rr = __builtin_fmaf(wx[2], q.y, __builtin_fmaf(wx[1], p.b.y, wx[0] * p.a.y));
            tz = __builtin_fmaf(wy[dj], rz, tz);
            tr = __builtin_fmaf(wy[dj], rr, tr);
        }
    }
}

struct TableTerms {
    float dx, dy, S, Fz, P;  // S_eff, F_z,eff and (POT) P
};

// A pair of the tabulated scheme that is not softened, lies inside the table
// and off the axis: table_terms without its branches, so that several pairs
// can be in flight at once.  False where it is not such a pair (the terms are
// then meaningless); the same values, bit for bit, where it is.
template <int ORDER>
__device__ __forceinline__ bool table_terms_inside(const TableView &a, const PeriodConsts &pc, double xi, double yi,
                                                   double zi, const SrcRec &src, TableTerms &t) {
    const double dx64 = xi - src.x, dy64 = yi - src.y;
    const double d64 = min_image(zi - src.z, pc.L, pc.invL);
    const float dx = (float)dx64, dy = (float)dy64, d = (float)d64;
    const float rho2 = __builtin_fmaf(dx, dx, dy * dy);
    // pair_fast<1, false> with the contractions the compiler makes of it spelled out
    const float ri0 = __builtin_amdgcn_rsqf(__builtin_fmaf(d, d, rho2));
    const float dzp = d - pc.c.Lf, dzm = d + pc.c.Lf;
    const float rip = __builtin_amdgcn_rsqf(__builtin_fmaf(dzp, dzp, rho2));
    const float rim = __builtin_amdgcn_rsqf(__builtin_fmaf(dzm, dzm, rho2));
    const float rip2 = rip * rip, rim3 = rim * rim * rim;
    const float S = __builtin_fmaf(ri0 * ri0, ri0, __builtin_fmaf(rip2, rip, rim3));
    const float Fz = __builtin_fmaf(d, S, -pc.c.Lf * __builtin_fmaf(rip2, rip, -rim3));
    const float rho = sqrt_newton(rho2);
    const float r = rho * pc.invLf;
    const float delta = __builtin_fabsf(d) * pc.invLf;
    float tz, Rr;
    lookup<ORDER>(a, GlobalNodes{a.T, a.w}, delta, r, tz, Rr);
    const float Rz = signed_tz(tz, d);
    const float rinv = __builtin_amdgcn_rcpf(rho);
    t = TableTerms{dx, dy, __builtin_fmaf(-Rr * pc.invL2f, rinv, S), __builtin_fmaf(-Rz, pc.invL2f, Fz), 0.f};
    return r <= a.r_max && rho2 >= kSqrtMin;
}

// One pair of the tabulated scheme.  Every lane of the wave must call it
// together (the exact band beyond a band table's rho_max is shared by the
// wave); ``active`` marks lanes with a real target.  COMPLETE: the table holds
// every image |n| >= 2 (pairs beyond rho_max take the line-mass limit) rather
// than a band.
template <int ORDER, bool POT, bool COMPLETE, class Nodes>
__device__ __forceinline__ TableTerms table_terms(const TableView &a, const Nodes &nodes, const PeriodConsts &pc,
                                                  double xi, double yi, double zi, float hi, const SrcRec &src,
                                                  bool self, bool active) {
    const int lane = threadIdx.x & 63;
    const double dx64 = xi - src.x, dy64 = yi - src.y;
    const double d64 = min_image(zi - src.z, pc.L, pc.invL);
    const float dx = (float)dx64, dy = (float)dy64, d = (float)d64;
    float S, Fz, Pn = 0.f;
    pair_fast<1, POT>(dx, dy, d, pc.c, S, Fz, Pn);
    const float rho2 = __builtin_fmaf(dx, dx, dy * dy);
    const float r2_0 = __builtin_fmaf(d, d, rho2);
    const float hij = hi + src.h;
    if (r2_0 < hij * hij || hij > (float)pc.halfL) {
        if (self) {
            S = 0.f;
            Fz = 0.f;
            Pn = 0.f;
        } else {
            // inlined: a call's register convention would raise the walk from 96 to 131 VGPRs
            double gs, gf, gp;
            pair_spline_f64(dx64, dy64, d64, (double)hi + (double)src.h, pc.L, 1, gs, gf, gp);
            S = (float)gs;
            Fz = (float)gf;
            Pn = (float)gp;
        }
    }
    const float rho = sqrt_exact(rho2);
    const float r = rho * pc.invLf;
    const float delta = __builtin_fabsf(d) * pc.invLf;
    const bool inside = (r <= a.r_max) && !self;
    float tz, tr;
    lookup<ORDER>(a, nodes, delta, r, tz, tr);
    float Rz = signed_tz(tz, d);
    float Rr = tr;
    if (!inside) {
        Rz = 0.f;
        Rr = 0.f;
    }
    if (COMPLETE) {
        // line-mass limit of the complete sum minus the three nearest images
        if (!inside && !self) {
            const float ds = d * pc.invLf, r2 = r * r;
            float nz = 0.f, nr = 0.f;
#pragma unroll
            for (int n = -1; n <= 1; ++n) {
                const float u = ds - (float)n;
                const float iq = __builtin_amdgcn_rsqf(__builtin_fmaf(u, u, r2));
                const float iq3 = iq * iq * iq;
                nz = __builtin_fmaf(-u, iq3, nz);
                nr = __builtin_fmaf(-r, iq3, nr);
            }
            Rz = -nz;
            Rr = -2.f * __builtin_amdgcn_rcpf(r) - nr;
        }
    }
    uint64_t outside = COMPLETE ? 0 : __ballot(!inside && !self && active);
    while (outside) {
        const int c = __builtin_ctzll(outside);
        outside &= outside - 1;
        const float dc = __shfl(d * pc.invLf, c), rc = __shfl(r, c);
        float bz, br;
        band_wave(dc, rc, a.n_far, bz, br);
        if (lane == c) {
            Rz = bz;
            Rr = br;
        }
    }
    const float rinv = rho > 0.f ? __builtin_amdgcn_rcpf(rho) : 0.f;
    return TableTerms{dx, dy, __builtin_fmaf(-Rr * pc.invL2f, rinv, S), __builtin_fmaf(-Rz, pc.invL2f, Fz), Pn};
}

// (px, py) += m S_eff (dx, dy), pz += m Fz_eff, pp += m P (the caller negates
// at the end).
template <bool POT>
__device__ __forceinline__ void table_add(const TableTerms &t, float m, float &px, float &py, float &pz, float &pp) {
    const float mS = m * t.S;
    px = __builtin_fmaf(mS, t.dx, px);
    py = __builtin_fmaf(mS, t.dy, py);
    pz = __builtin_fmaf(m, t.Fz, pz);
    if (POT) pp = __builtin_fmaf(m, t.P, pp);
}

}  // namespace steps
