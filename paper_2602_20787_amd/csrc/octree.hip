// Barnes-Hut octree force in the S1 x R2 topology (Sect. 2.4, "Octree"):
// cubic cells, a root cell twice the largest linear size of the volume
// (S0 = 2 max(L, 2 R_dom)), a random shift of the domain along the axis and
// a rotation about it at every call, cell monopoles, and a radial correction
// table measured on the initial load and subtracted from the tree forces.
//
// Build (FP64, all on the GPU, two host synchronisations: the number of cells
// and of groups):
//  1. rotate by the given angle, shift and wrap z, and form 63-bit Morton
//     keys of the integer cell coordinates q = floor((p - lo) 2^21 / S0)
//     (x bit above y above z per level); radix-sort (key, index);
//  2. the cells, of all levels at once, from the sorted keys.  lcp(i, j) is
//     the number of 3-bit digits in which keys i and j agree.  A cell of level
//     l that holds more than leaf_size particles (and l < 21) is open; so the
//     cells around particle i are open down to level D(i) = max over the runs
//     of leaf_size + 1 particles with i among them of the lcp of their ends.
//     A cell of level l >= 1 starts at i where its parent is open and i differs
//     from i - 1 above: lcp(i - 1, i) < l <= D(i) + 1.  A scan of these counts
//     numbers the cells in depth-first order, (start, level); the "skip" of a
//     cell is the first cell of the order that starts at its end.  (Level by
//     level, with three scans and two synchronisations each, the build took 1.3
//     ms at 2^20 particles and 0.75 at 100,003: now 0.6 and 0.35.)
//  3. mass, mass-weighted position, largest softening and quadrupole
//     bottom-up: the leaves from their particles, then, a launch per level,
//     cells from their children.
//
// Groups: for every cell holding more than 64 particles, its children that
// hold at most 64 are packed greedily, in order, into runs of at most 64
// particles (a leaf holding more is cut into runs of 64); a tree of at most
// 64 particles is one group.  Groups are thus made of whole sibling cells
// and stay compact where 64 consecutive particles in key order would not
// (the key order jumps between distant octants).
//
// Walk: one 64-lane wave per group.  A cell is accepted for the whole group
// when size^2 < theta^2 d^2 and d^2 > (h_group + h_cell)^2, d the distance
// (periodic in z) from its centre of mass to the group's bounding box; an
// accepted cell adds its monopole, an opened leaf its particles, both through
// the pair interaction of the tabulated scheme (exact images |n| <= 1 plus the
// table's far images).  The lanes take turns as tests and as targets: the wave
// keeps the frontier of the walk in depth-first order on an LDS stack, tests
// its next 64 cells at once (one per lane), replaces the opened ones by their
// children in place, and hands what lies before the first opened one to a list
// of cells and leaves that is staged 64 sources at a time in LDS and then
// evaluated with a target per lane.  The list is in depth-first order and so
// are the sums.  Accelerations are rotated back and written in the caller's
// particle order.
#include <cmath>
#include <type_traits>
#include <vector>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include "table_pair.h"

namespace steps {
namespace {

constexpr int kLevels = 21;
constexpr int kBlock = 256;
constexpr int kMaxBins = 256;
constexpr int kGroup = 64;
// The walk's waves share nothing: workgroups of one are dealt out evenly (N =
// 2^20 11.3 -> 10.8 ms, with quadrupoles 22.6 -> 21.0, against workgroups of four).
constexpr int kWalkBlock = 64;

// one cell in depth-first order (88 B): monopole, and the traceless
// quadrupole about the centre of mass (xx, yy, zz, xy, xz, yz) when enabled
struct CellRec {
    double cx, cy, cz, mass, hmax, size;
    int start, count, skip, leaf;
    float q[6];
};

// what the walk needs of a cell; siblings are contiguous, in order
struct alignas(64) WalkNode {
    double cx, cy, cz, hmax, size2;  // centre of mass, largest softening, size^2
    float m, h;                      // mass and largest softening, FP32
    int first, count;                // children, or particles with the top bit of count set
};
constexpr int kLeafBit = (int)0x80000000u;

}  // namespace
}  // namespace steps

struct steps_cyl_tree {
    int leaf_size = 16;
    int quadrupole = 0;
    int64_t cap_n = 0, cap_cells = 0;
    size_t cub_bytes = 0;
    void *cub_tmp = nullptr;
    // particles
    double *tx = nullptr, *ty = nullptr, *tz = nullptr;
    uint64_t *key_in = nullptr, *key_out = nullptr;
    int *idx_in = nullptr, *idx_out = nullptr;
    double *sx = nullptr, *sy = nullptr, *sz = nullptr, *sm = nullptr, *sh = nullptr;
    int *depth = nullptr;                              // per particle: open levels around it (-1: none)
    int64_t *first = nullptr, *first_sum = nullptr;    // cells that start at it, running total
    int *levels = nullptr;                             // [2][32] open cells per level: number, cursor
    // cells, depth-first
    double *c_m = nullptr, *c_mx = nullptr, *c_my = nullptr, *c_mz = nullptr, *c_h = nullptr;
    double *c_q = nullptr;  // [6][cap_cells] quadrupoles (when enabled)
    int *open_cells = nullptr;                // by level
    uint64_t *n_in = nullptr, *n_sum = nullptr;  // children << 32 | groups that a cell packs, running total
    steps::WalkNode *nodes = nullptr;
    float *node_q = nullptr;  // [cap_cells][8] quadrupoles (when enabled)
    steps::CellRec *cells = nullptr;
    int *cell_level = nullptr;
    int *g_start = nullptr, *g_count = nullptr;  // per group: particle range
    int64_t n_cells = 0, n = 0, n_groups = 0;
    // walk statistics, per wave
    int *wave_cells = nullptr, *wave_parts = nullptr;
    // radial correction
    double *corr = nullptr;
    int n_bins = 0;
    double corr_rdom = 0.0;
    // calibration scratch
    double *bin_sum = nullptr, *bin_cnt = nullptr;
    float *acc_dir = nullptr, *acc_tree = nullptr;
    int64_t cap_cal = 0;
};

namespace steps {
namespace {

template <typename T>
hipError_t grow(T *&p, int64_t n) {
    (void)hipFree(p);
    p = nullptr;
    return hipMalloc(&p, (size_t)std::max<int64_t>(n, 1) * sizeof(T));
}

hipError_t ensure_scratch(steps_cyl_tree *t, size_t need) {
    if (need <= t->cub_bytes) return hipSuccess;
    t->cub_bytes = 0;
    char *p = (char *)t->cub_tmp;
    const hipError_t e = grow(p, (int64_t)need);
    t->cub_tmp = p;
    if (e == hipSuccess) t->cub_bytes = need;
    return e;
}

hipError_t ensure_particles(steps_cyl_tree *t, int64_t n) {
    if (n <= t->cap_n) return hipSuccess;
    const int64_t c = n + n / 4 + 1024;
    t->cap_n = 0;
    hipError_t e = hipSuccess;
#define G(p) \
    if (e == hipSuccess) e = grow(t->p, c);
    G(tx) G(ty) G(tz) G(key_in) G(key_out) G(idx_in) G(idx_out) G(sx) G(sy) G(sz) G(sm) G(sh)
    G(depth) G(first) G(first_sum) G(wave_cells) G(wave_parts) G(g_start) G(g_count)
#undef G
    if (e == hipSuccess) e = grow(t->levels, 64);
    // scratch of the library sort and scan, sized for c items
    size_t b1 = 0, b2 = 0;
    if (e == hipSuccess)
        e = rocprim::radix_sort_pairs(nullptr, b1, t->key_in, t->key_out, t->idx_in, t->idx_out, (int)c, 0, 63);
    if (e == hipSuccess)
        e = rocprim::inclusive_scan(nullptr, b2, t->first, t->first_sum, (size_t)c, rocprim::plus<int64_t>(), 0);
    if (e == hipSuccess) e = ensure_scratch(t, std::max(b1, b2));
    if (e == hipSuccess) t->cap_n = c;
    return e;
}

hipError_t ensure_cells(steps_cyl_tree *t, int64_t n) {
    if (n <= t->cap_cells) return hipSuccess;
    const int64_t c = n + n / 4 + 64;
    t->cap_cells = 0;
    hipError_t e = hipSuccess;
#define G(p) \
    if (e == hipSuccess) e = grow(t->p, c);
    G(c_m) G(c_mx) G(c_my) G(c_mz) G(c_h) G(open_cells) G(n_in) G(n_sum) G(nodes) G(cells) G(cell_level)
#undef G
    if (e == hipSuccess) e = grow(t->c_q, t->quadrupole ? 6 * c : 1);
    if (e == hipSuccess) e = grow(t->node_q, t->quadrupole ? 8 * c : 1);
    size_t b = 0;
    if (e == hipSuccess)
        e = rocprim::inclusive_scan(nullptr, b, t->n_in, t->n_sum, (size_t)c, rocprim::plus<uint64_t>(), 0);
    if (e == hipSuccess) e = ensure_scratch(t, b);
    if (e == hipSuccess) t->cap_cells = c;
    return e;
}

struct Frame {
    double c, s, shift, L, lo[3], scale;
};

// rotation, shift and wrap as separately rounded operations (no contraction),
// so that keys and cells do not depend on the compiler's choices
// (the workgroup holds at least 64 threads)
__global__ void keys_kernel(const double *pos, int64_t N, Frame f, double *tx, double *ty, double *tz,
                            uint64_t *key, int *idx, int *levels) {
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 64) levels[i] = 0;
    if (i >= N) return;
    const double X = pos[i], Y = pos[N + i], Z = pos[2 * N + i];
    const double x = f.c * X - f.s * Y;
    const double y = f.s * X + f.c * Y;
    double z = Z + f.shift;
    z = z - f.L * floor(z / f.L);
    if (z >= f.L) z = 0.0;
    tx[i] = x;
    ty[i] = y;
    tz[i] = z;
    const double p[3] = {x, y, z};
    uint64_t q[3];
    for (int a = 0; a < 3; ++a) {
        double v = floor((p[a] - f.lo[a]) * f.scale);
        v = v < 0.0 ? 0.0 : (v > (double)((1 << kLevels) - 1) ? (double)((1 << kLevels) - 1) : v);
        q[a] = (uint64_t)v;
    }
    uint64_t k = 0;
    for (int b = 0; b < kLevels; ++b) {
        k |= ((q[0] >> b) & 1ull) << (3 * b + 2);
        k |= ((q[1] >> b) & 1ull) << (3 * b + 1);
        k |= ((q[2] >> b) & 1ull) << (3 * b);
    }
    key[i] = k;
    idx[i] = (int)i;
}

// number of 3-bit digits in which two keys agree
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x ? (__builtin_clzll(x) - 1) / 3 : kLevels;
}

// Particles in key order, the levels open around each (at most level 20: a cell
// of level 21 is a leaf), the number of cells that start at it, and how many
// open cells each level has.
__global__ __launch_bounds__(kBlock) void gather_kernel(const int *idx, int N, const double *tx, const double *ty,
                                                        const double *tz, const double *mass, const double *eps,
                                                        double *sx, double *sy, double *sz, double *sm, double *sh,
                                                        const uint64_t *key, int leaf_size, int *depth, int64_t *first,
                                                        int *levels) {
    __shared__ int run[kBlock + 64];  // lcp of the run of leaf_size + 1 particles from i0 - leaf_size + k, or -1
    __shared__ int hist[kLevels];
    const int i0 = blockIdx.x * kBlock;
    const int i = i0 + threadIdx.x;
    if (threadIdx.x < kLevels) hist[threadIdx.x] = 0;
    for (int k = threadIdx.x; k < kBlock + leaf_size; k += kBlock) {
        const int64_t j = (int64_t)i0 - leaf_size + k;
        run[k] = j >= 0 && j + leaf_size < N ? common_digits(key[j], key[j + leaf_size]) : -1;
    }
    __syncthreads();
    if (i < N) {
        const int j = idx[i];
        sx[i] = tx[j];
        sy[i] = ty[j];
        sz[i] = tz[j];
        sm[i] = mass[j];
        sh[i] = eps[j];
        int d = -1;
        for (int k = 0; k <= leaf_size; ++k) d = max(d, run[threadIdx.x + k]);
        d = min(d, kLevels - 1);
        const int lo = i > 0 ? common_digits(key[i - 1], key[i]) + 1 : 1;
        depth[i] = d;
        first[i] = d < 0 ? 0 : max(0, d + 2 - lo);
        for (int l = lo; l <= d; ++l) atomicAdd(&hist[l], 1);
        if (i == 0 && d >= 0) atomicAdd(&hist[0], 1);
    }
    __syncthreads();
    if (threadIdx.x < kLevels && hist[threadIdx.x]) atomicAdd(&levels[threadIdx.x], hist[threadIdx.x]);
}

// first open cell of each level in the list of open cells
struct LevelStarts {
    int at[kLevels];
};

// The cells that start at each particle; open cells are listed by level (in
// any order: the sums over a level do not depend on it).
__global__ __launch_bounds__(kBlock) void cells_kernel(const uint64_t *key, const int *depth, const int64_t *first,
                                                       const int64_t *first_sum, int N, int n_cells, int leaf_size,
                                                       double side, LevelStarts ls, int *cursor, CellRec *cells,
                                                       int *cell_level, int *open_cells) {
    __shared__ int hist[kLevels], base[kLevels];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (threadIdx.x < kLevels) hist[threadIdx.x] = 0;
    __syncthreads();
    // this particle's cells: levels lo .. hi at positions p .. (the root before them)
    const int n = i < N ? (int)first[i] : 0;
    const int d = i < N ? depth[i] : -1;
    const int hi = d + 1, lo = hi - n + 1;
    const int p = i < N ? 1 + (int)(first_sum[i] - n) : 0;
    const bool root = i == 0;
    for (int l = lo; l <= min(hi, d); ++l) atomicAdd(&hist[l], 1);
    if (root && d >= 0) atomicAdd(&hist[0], 1);
    __syncthreads();
    if (threadIdx.x < kLevels) {
        base[threadIdx.x] = hist[threadIdx.x] ? ls.at[threadIdx.x] + atomicAdd(&cursor[threadIdx.x], hist[threadIdx.x]) : 0;
        hist[threadIdx.x] = 0;
    }
    __syncthreads();
    auto write = [&](int at, int l, int end) {
        const bool leaf = l > d;
        CellRec &c = cells[at];
        c.size = side / (double)(1ull << l);
        c.start = i;
        c.count = end - i;
        c.skip = end < N ? 1 + (int)(first_sum[end] - first[end]) : n_cells;
        c.leaf = leaf ? 1 : 0;
        cell_level[at] = l;
        if (!leaf) open_cells[base[l] + atomicAdd(&hist[l], 1)] = at;
    };
    if (root) write(0, 0, N);
    for (int l = lo; l <= hi; ++l) {
        // the end: the first particle beyond whose prefix of l digits is larger
        const int shift = 3 * (kLevels - l);
        const uint64_t prefix = key[i] >> shift;
        int a = i + 1, b = l > d && l < kLevels ? min(N, i + leaf_size) : N;
        while (a < b) {
            const int mid = a + (b - a) / 2;
            if ((key[mid] >> shift) > prefix) b = mid; else a = mid + 1;
        }
        write(p + (l - lo), l, a);
    }
}

// geometric centre of a cell from its key prefix (massless cells only)
__device__ void cell_centre(uint64_t key, int level, const Frame &f, double side, double *c) {
    uint64_t q[3] = {0, 0, 0};
    for (int b = 0; b < level; ++b) {
        const uint64_t digit = (key >> (3 * (kLevels - 1 - b))) & 7ull;
        q[0] = 2 * q[0] + ((digit >> 2) & 1);
        q[1] = 2 * q[1] + ((digit >> 1) & 1);
        q[2] = 2 * q[2] + (digit & 1);
    }
    const double h = side / (double)(1ull << level);
    for (int a = 0; a < 3; ++a) c[a] = f.lo[a] + ((double)q[a] + 0.5) * h;
}

// Mass, mass-weighted position and largest softening of the leaves (list null:
// every cell that is one, from its particles) or of one level's open cells
// (from their children), and (QUAD) the traceless quadrupole about the centre
// of mass, from the particles or by the parallel-axis shift of the children's.
template <bool QUAD>
__global__ void moments_kernel(const int *list, int n, int64_t cap, const CellRec *cells, double *c_m, double *c_mx,
                               double *c_my, double *c_mz, double *c_h, double *c_q, const double *sx,
                               const double *sy, const double *sz, const double *sm, const double *sh) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int c = list ? list[k] : k;
    if (!list && !cells[c].leaf) return;
    const int s = cells[c].start, e = s + cells[c].count, skip = cells[c].skip;
    double m = 0.0, mx = 0.0, my = 0.0, mz = 0.0, h = 0.0;
    if (!list) {
        for (int j = s; j < e; ++j) {
            m += sm[j];
            mx += sm[j] * sx[j];
            my += sm[j] * sy[j];
            mz += sm[j] * sz[j];
            h = fmax(h, sh[j]);
        }
    } else {
        for (int q = c + 1; q < skip; q = cells[q].skip) {
            m += c_m[q];
            mx += c_mx[q];
            my += c_my[q];
            mz += c_mz[q];
            h = fmax(h, c_h[q]);
        }
    }
    c_m[c] = m;
    c_mx[c] = mx;
    c_my[c] = my;
    c_mz[c] = mz;
    c_h[c] = h;
    if (!QUAD) return;
    double q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (m > 0.0) {
        const double gx = mx / m, gy = my / m, gz = mz / m;
        auto add = [&](double w, double x, double y, double z) {
            const double r2 = x * x + y * y + z * z;
            q[0] += w * (3.0 * x * x - r2);
            q[1] += w * (3.0 * y * y - r2);
            q[2] += w * (3.0 * z * z - r2);
            q[3] += w * 3.0 * x * y;
            q[4] += w * 3.0 * x * z;
            q[5] += w * 3.0 * y * z;
        };
        if (!list) {
            for (int j = s; j < e; ++j) add(sm[j], sx[j] - gx, sy[j] - gy, sz[j] - gz);
        } else {
            for (int ch = c + 1; ch < skip; ch = cells[ch].skip) {
                const double mc = c_m[ch];
                for (int a = 0; a < 6; ++a) q[a] += c_q[(size_t)a * cap + ch];
                if (mc > 0.0) add(mc, c_mx[ch] / mc - gx, c_my[ch] / mc - gy, c_mz[ch] / mc - gz);
            }
        }
    }
    for (int a = 0; a < 6; ++a) c_q[(size_t)a * cap + c] = q[a];
}

// groups packed by cell c (see the file comment); with out < 0 only counted
__device__ int pack_groups(const CellRec *cells, int c, int *g_start, int *g_count, int out) {
    const CellRec r = cells[c];
    int n = 0;
    auto emit = [&](int s, int k) {
        if (out >= 0) {
            g_start[out + n] = s;
            g_count[out + n] = k;
        }
        ++n;
    };
    if (r.count <= kGroup) {
        if (c == 0) emit(0, r.count);  // the whole tree is one group
        return n;
    }
    if (r.leaf) {
        for (int s = r.start; s < r.start + r.count; s += kGroup) emit(s, min(kGroup, r.start + r.count - s));
        return n;
    }
    int run_s = 0, run_n = 0;
    for (int ch = c + 1; ch < r.skip; ch = cells[ch].skip) {
        const int cc = cells[ch].count;
        if (cc > kGroup) {
            if (run_n) emit(run_s, run_n);
            run_n = 0;
        } else {
            if (run_n + cc > kGroup) {
                emit(run_s, run_n);
                run_n = 0;
            }
            if (run_n == 0) run_s = cells[ch].start;
            run_n += cc;
        }
    }
    if (run_n) emit(run_s, run_n);
    return n;
}

// children and groups of each cell
__global__ void count_kernel(const CellRec *cells, int n, uint64_t *n_in) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    uint64_t children = 0;
    if (!cells[c].leaf)
        for (int ch = c + 1; ch < cells[c].skip; ch = cells[ch].skip) ++children;
    n_in[c] = children << 32 | (uint64_t)(uint32_t)pack_groups(cells, c, nullptr, nullptr, -1);
}

// The moments of each cell into its record, its groups, and its children (the
// root by itself) as nodes of the walk.
__global__ void nodes_kernel(CellRec *cells, const int *cell_level, int n, const double *c_m, const double *c_mx,
                             const double *c_my, const double *c_mz, const double *c_h, const double *c_q,
                             int64_t cap, int quad, const uint64_t *pkey, Frame f, double side, const uint64_t *n_in,
                             const uint64_t *n_sum, int *g_start, int *g_count, WalkNode *nodes, float *node_q) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint64_t mine = n_in[p], before = n_sum[p] - mine;
    if ((uint32_t)mine) pack_groups(cells, p, g_start, g_count, (int)(uint32_t)before);
    auto centre = [&](int c, double g[3]) {
        const double m = c_m[c];
        if (m > 0.0) {
            g[0] = c_mx[c] / m;
            g[1] = c_my[c] / m;
            g[2] = c_mz[c] / m;
        } else {
            cell_centre(pkey[cells[c].start], cell_level[c], f, side, g);
        }
    };
    {
        double g[3];
        centre(p, g);
        CellRec &r = cells[p];
        r.cx = g[0];
        r.cy = g[1];
        r.cz = g[2];
        r.mass = c_m[p];
        r.hmax = c_h[p];
        for (int a = 0; a < 6; ++a) r.q[a] = quad ? (float)c_q[(size_t)a * cap + p] : 0.f;
    }
    auto node = [&](int at, int c) {
        double g[3];
        centre(c, g);
        const double size = cells[c].size;
        const int leaf = cells[c].leaf;
        WalkNode w;
        w.cx = g[0];
        w.cy = g[1];
        w.cz = g[2];
        w.hmax = c_h[c];
        w.size2 = size * size;
        w.m = (float)c_m[c];
        w.h = (float)c_h[c];
        w.first = leaf ? cells[c].start : 1 + (int)((n_sum[c] - n_in[c]) >> 32);
        w.count = leaf ? (cells[c].count | kLeafBit) : (int)(n_in[c] >> 32);
        nodes[at] = w;
        if (quad)
            for (int a = 0; a < 6; ++a) node_q[(size_t)at * 8 + a] = (float)c_q[(size_t)a * cap + c];
    };
    if (p == 0) node(0, 0);
    if (cells[p].leaf) return;
    int at = 1 + (int)(before >> 32);
    for (int ch = p + 1; ch < cells[p].skip; ch = cells[ch].skip) node(at++, ch);
}

// ---------------------------------------------------------------- walk
struct WalkArgs {
    const WalkNode *nodes;
    const float *node_q;
    const double *sx, *sy, *sz, *sm, *sh;
    const int *idx, *g_start, *g_count;
    float *ax, *ay, *az;
    int *wave_cells, *wave_parts;
    const double *corr;
    TableView tv;
    PeriodConsts pc;
    double theta2, c, s, corr_step;
    int n_groups, n_bins;
};

__device__ __forceinline__ double wave_min(double v) {
    for (int off = 32; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
    return v;
}

// squared distance from c to the box [lo, hi], periodic along z (no
// contraction, so that the acceptance decisions round as written)
__device__ double box_distance2(double cx, double cy, double cz, const double lo[3], const double hi[3],
                                double L) {
#pragma clang fp contract(off)
    const double dx = fmax(0.0, fmax(lo[0] - cx, cx - hi[0]));
    const double dy = fmax(0.0, fmax(lo[1] - cy, cy - hi[1]));
    double dz = 1e300;
    for (int k = -1; k <= 1; ++k) {
        const double z = cz + k * L;
        dz = fmin(dz, fmax(0.0, fmax(lo[2] - z, z - hi[2])));
    }
    return dx * dx + dy * dy + dz * dz;
}

// no pair at d^2 >= d2 with softening sum <= hs is softened, by a margin over
// FP32 rounding
__device__ __forceinline__ bool far_apart(double d2, double hs, double L) {
    return d2 > hs * hs * 1.00001 && hs < 0.49999 * L;
}

// size^2 < theta^2 d^2 and d^2 > (h_group + h_cell)^2, compared squared; `far`
// as above for the cell with the group
__device__ bool accept_cell(const WalkNode &r, const double lo[3], const double hi[3], double hg, double theta2,
                            double L, bool &far) {
#pragma clang fp contract(off)
    const double d2 = box_distance2(r.cx, r.cy, r.cz, lo, hi, L);
    const double hs = hg + r.hmax;
    far = far_apart(d2, hs, L);
    return r.size2 < theta2 * d2 && d2 > hs * hs;
}

// quadrupole term of an accepted cell for the images |n| <= 4 about the
// minimum image (beyond, the term falls as 1/n^4), subtracted from the
// partial sums (which carry the opposite sign of the acceleration):
// a += Q s / r^5 - (5/2) (s.Q.s) s / r^7.  Q s_n = Q s_0 - n L Q e_z.
constexpr int kQuadImages = 4;

__device__ __forceinline__ void quadrupole_term(const SrcRec &r, const float *q, double xi, double yi, double zi,
                                                const PeriodConsts &pc, float &px, float &py, float &pz) {
    const float sx = (float)(xi - r.x), sy = (float)(yi - r.y);
    const float d = (float)min_image(zi - r.z, pc.L, pc.invL);
    const float rho2 = __builtin_fmaf(sx, sx, sy * sy);
    const float bx = __builtin_fmaf(q[0], sx, __builtin_fmaf(q[3], sy, q[4] * d));
    const float by = __builtin_fmaf(q[3], sx, __builtin_fmaf(q[1], sy, q[5] * d));
    const float bz = __builtin_fmaf(q[4], sx, __builtin_fmaf(q[5], sy, q[2] * d));
#pragma unroll
    for (int n = -kQuadImages; n <= kQuadImages; ++n) {
        const float nL = (float)n * pc.c.Lf;
        const float sz = d - nL;
        const float qx = __builtin_fmaf(-nL, q[4], bx);
        const float qy = __builtin_fmaf(-nL, q[5], by);
        const float qz = __builtin_fmaf(-nL, q[2], bz);
        const float r2 = __builtin_fmaf(sz, sz, rho2);
        const float ri = __builtin_amdgcn_rsqf(r2);
        const float ri2 = ri * ri;
        const float ri5 = ri2 * ri2 * ri;
        const float sqs = __builtin_fmaf(sx, qx, __builtin_fmaf(sy, qy, sz * qz));
        const float c = -2.5f * sqs * ri2;
        px = __builtin_fmaf(-ri5, __builtin_fmaf(c, sx, qx), px);
        py = __builtin_fmaf(-ri5, __builtin_fmaf(c, sy, qy), py);
        pz = __builtin_fmaf(-ri5, __builtin_fmaf(c, sz, qz), pz);
    }
}

// v of the lanes' F groups of 64 / F, in every lane: out[k] is the value that
// lane k (64 / F) + lane mod (64 / F) holds.
template <int F>
__device__ __forceinline__ void spread(float v, float *out) {
    if (F == 1) {
        out[0] = v;
    } else {
        const unsigned u = __float_as_uint(v);
        const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        if (F == 2) {
            out[0] = __uint_as_float(h[0]);
            out[1] = __uint_as_float(h[1]);
        } else {
            const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
            const auto up = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
            out[0] = __uint_as_float(lo[0]);
            out[1 % F] = __uint_as_float(lo[1]);
            out[2 % F] = __uint_as_float(up[0]);
            out[3 % F] = __uint_as_float(up[1]);
        }
    }
}

// The frontier: cells still to be tested or resolved, the next in depth-first
// order on top.  A step pops n of them and pushes at most 8 n, so with
// n <= (kStack - kStackRest - size)/8 (at least 1) the wide steps stay below
// kStack - kStackRest, and popping one by one from there adds at most 7 per
// level: 147 entries.
constexpr int kStack = 768, kStackRest = 160;
enum { kOpen = 0, kFar = 1, kNear = 2, kLeaf = 3 };  // kind of an entry, its top two bits

struct alignas(16) WalkSrc {
    SrcRec r;
    int own;        // its particle index (-1: a cell)
    unsigned flag;  // its entry's kind, | kFarSrc: no pair with the group is softened, | flush
};
constexpr unsigned kFarSrc = 4, kFlush = 8;

template <bool QUAD>
struct WalkLds {
    double box[7];       // the group's bounding box (low, high) and largest softening
    unsigned stack[kStack];
    unsigned list[128];  // resolved cells and leaves, in order
    int start[64];       // a batch: first source of each entry
    unsigned kind[64];   // and the flags of its last source
    int first[64];       // and its node or first particle
    WalkSrc src[64];     // a stage of the batch's sources
    float q[QUAD ? 64 : 1][6];
};

__device__ __forceinline__ unsigned lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Exclusive sum over the lanes of v < 2^BITS; `total` of all.
template <int BITS>
__device__ __forceinline__ int small_scan(int v, int &total) {
    int e = 0;
    total = 0;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint64_t m = __ballot((v >> b) & 1);
        e += (int)lanes_below(m) << b;
        total += __builtin_popcountll(m) << b;
    }
    return e;
}

// Waves per SIMD that the registers are bounded for.  CIC at 4 and 5: 12.55 and
// 12.28 ms at N = 2^20; with quadrupoles at 4 and 3: 4.08 and 3.95 ms a step at
// N = 100,003, where there are two waves per SIMD in any case.
constexpr int walk_waves(int order, bool quad, int split) {
    return split > 1 ? 2 : quad ? 3 : order == 1 ? 5 : 4;
}

// A wave tested one cell at a time, all lanes alike, and read sources one at a
// time from memory (148 VALU instructions per interaction of a wave, 34 of them
// tests; N = 2^20, theta 0.5: 15.7 -> 11.0 ms).
//
// SPLIT waves per group, each for 64 / SPLIT of its targets: the lanes then hold
// them SPLIT times over, take one of SPLIT sources each and hand each other the
// terms, which every lane adds in order.  A source costs a wave less and a group
// more: this is for trees of few groups, which leave SIMDs idle (see walk()).  Not
// with quadrupoles, whose 36 terms per cell cost more to hand over than to repeat.
template <int ORDER, bool QUAD, bool COMPLETE, int SPLIT>
__global__ __launch_bounds__(kWalkBlock, walk_waves(ORDER, QUAD, SPLIT)) void tree_walk_kernel(WalkArgs a) {
    static_assert(SPLIT == 1 || !QUAD, "quadrupoles take whole groups");
    __shared__ WalkLds<QUAD> lds[kWalkBlock / 64];
    constexpr int kOwned = 64 / SPLIT;  // targets of a wave
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * kWalkBlock + threadIdx.x) >> 6;
    const int group = (int)(wave / SPLIT), slice = (int)(wave % SPLIT);
    if (group >= a.n_groups) return;  // whole wave (and the waves share nothing)
    WalkLds<QUAD> &w = lds[threadIdx.x >> 6];
    const int g0 = a.g_start[group], g_n = a.g_count[group];
    if (slice * kOwned >= g_n) return;
    {
        const int j = g0 + min(lane, g_n - 1);
        const double x = a.sx[j], y = a.sy[j], z = a.sz[j];
        const double b[7] = {wave_min(x), wave_min(y), wave_min(z), wave_max(x),
                             wave_max(y), wave_max(z), wave_max(a.sh[j])};
        if (lane == 0)
            for (int c = 0; c < 7; ++c) w.box[c] = b[c];
    }
    const int own = slice * kOwned + lane % kOwned;
    const bool active = own < g_n;
    const int i = g0 + own;
    const int ii = active ? i : g0;
    const double xi = a.sx[ii], yi = a.sy[ii], zi = a.sz[ii];
    const float hi = (float)a.sh[ii];
    const GlobalNodes nodes = {a.tv.T, a.tv.w};
    float sx = 0.f, sy = 0.f, sz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
    float px = 0.f, py = 0.f, pz = 0.f;
    int pending = 0, n_cell = 0, n_part = 0;
    int size = 1, listed = 0;
    if (lane == 0) w.stack[0] = 0;  // the root, unresolved
    for (;;) {
        asm volatile("" ::: "memory");
        if (listed < 64 && size > 0) {
            // ---- one step of the frontier
            const int n = min(min(64, size), max(1, (kStack - kStackRest - size) >> 3));
            unsigned e = lane < n ? w.stack[size - 1 - lane] : 0u;
            int first = 0, count = 1;  // what replaces the entry: itself, or `count` children from `first`
            bool open = false;
            if (lane < n && (e >> 30) == kOpen) {
                const WalkNode r = a.nodes[e];
                bool far;
                if (accept_cell(r, w.box, w.box + 3, w.box[6], a.theta2, a.pc.L, far)) {
                    e |= (unsigned)(far ? kFar : kNear) << 30;
                } else if (r.count < 0) {
                    e |= (unsigned)kLeaf << 30;
                } else {
                    open = true;
                    first = r.first;
                    count = r.count;
                }
            }
            const uint64_t opened = __ballot(open);
            const int f = opened ? __builtin_ctzll(opened) : n;  // entries that are next in the list
            if (lane < f) w.list[listed + lane] = e;
            listed += f;
            if (lane < f || lane >= n) count = 0;
            int total;
            const int before = small_scan<4>(count, total);
            size += total - n;
            const int top = size - 1 - before;
            if (open) {
                for (int k = 0; k < count; ++k) w.stack[top - k] = (unsigned)(first + k);
            } else if (count) {
                w.stack[top] = e;
            }
            continue;
        }
        if (listed == 0) break;
        // ---- a batch of the list
        const int n = min(64, listed);
        const unsigned e = lane < n ? w.list[lane] : 0u;
        const unsigned next = lane + 64 < listed ? w.list[lane + 64] : 0u;
        const unsigned kind = e >> 30;
        const bool leaf = lane < n && kind == kLeaf;
        int first = (int)(e & 0x3fffffffu), count = lane < n ? 1 : 0;
        if (leaf) {
            const WalkNode &r = a.nodes[first];
            first = r.first;
            count = r.count & ~kLeafBit;
        }
        // the partial sums are flushed after a leaf and after 16 cells in a row
        const uint64_t leaves = __ballot(leaf);
        const uint64_t below = leaves & ((1ull << lane) - 1);
        const int row = below ? lane - 64 + __builtin_clzll(below) : pending + lane;
        const bool flush = leaf || (row & 15) == 15;
        pending = (leaves ? n - 64 + (int)__builtin_clzll(leaves) : pending + n) & 15;
        int total, start;
        if (__ballot(count > 127) == 0) {
            start = small_scan<7>(count, total);
        } else {
            int s = count;
            for (int off = 1; off < 64; off <<= 1) {
                const int v = __shfl_up(s, off);
                if (lane >= off) s += v;
            }
            start = s - count;
            total = __shfl(s, 63);
        }
        total = __builtin_amdgcn_readfirstlane(total);
        n_cell += n - __builtin_popcountll(leaves);
        n_part += total - (n - __builtin_popcountll(leaves));
        w.start[lane] = start;
        w.kind[lane] = kind | (kind == kFar ? kFarSrc : 0u) | (flush ? kFlush : 0u);
        w.first[lane] = first;
        if (lane < 64) w.list[lane] = next;
        listed -= n;
        for (int base = 0; base < total; base += 64) {
            asm volatile("" ::: "memory");
            // ---- stage up to 64 sources
            const int m = min(64, total - base);
            if (lane < m) {
                const int t = base + lane;
                int k = 0;  // the entry: the last that starts at or before t
#pragma unroll
                for (int b = 32; b >= 1; b >>= 1)
                    if (k + b < n && w.start[k + b] <= t) k += b;
                const unsigned kd = w.kind[k];
                const int at = t - w.start[k];
                SrcRec r;
                int own = -1;
                unsigned flag = kd;
                if ((kd & 3) == kLeaf) {
                    own = w.first[k] + at;
                    r.x = a.sx[own];
                    r.y = a.sy[own];
                    r.z = a.sz[own];
                    r.m = (float)a.sm[own];
                    r.h = (float)a.sh[own];
                    const int end = k + 1 < n ? w.start[k + 1] : total;
                    if (t + 1 < end) flag = kLeaf;
                    if (far_apart(box_distance2(r.x, r.y, r.z, w.box, w.box + 3, a.pc.L), w.box[6] + a.sh[own], a.pc.L))
                        flag |= kFarSrc;
                } else {
                    const int c = w.first[k];
                    const WalkNode &q = a.nodes[c];
                    r.x = q.cx;
                    r.y = q.cy;
                    r.z = q.cz;
                    r.m = q.m;
                    r.h = q.h;
                    if (QUAD)
                        for (int b = 0; b < 6; ++b) w.q[lane][b] = a.node_q[(size_t)c * 8 + b];
                }
                w.src[lane] = WalkSrc{r, own, flag};
            }
            asm volatile("" ::: "memory");
            // ---- and evaluate them
            auto add = [&](float mS, float m, float dx, float dy, float Fz) {
                px = __builtin_fmaf(mS, dx, px);
                py = __builtin_fmaf(mS, dy, py);
                pz = __builtin_fmaf(m, Fz, pz);
            };
            auto flush = [&](unsigned flag) {
                if (flag & kFlush) {
                    kahan_add(sx, cx, px);
                    kahan_add(sy, cy, py);
                    kahan_add(sz, cz, pz);
                    px = py = pz = 0.f;
                }
            };
            if (SPLIT == 1) {
                // a target per lane: two sources at once where neither needs a
                // branch, to hide the latency of the table's gathers
                auto one = [&](const SrcRec &r, const TableTerms &t, unsigned flag, int s) {
                    add(r.m * t.S, r.m, t.dx, t.dy, t.Fz);
                    if (QUAD && (flag & 3) != kLeaf) quadrupole_term(r, w.q[QUAD ? s : 0], xi, yi, zi, a.pc, px, py, pz);
                    flush(flag);
                };
                for (int s = 0; s < m;) {
                    const SrcRec r0 = w.src[s].r, r1 = w.src[min(s + 1, m - 1)].r;
                    const unsigned f0 = __builtin_amdgcn_readfirstlane(w.src[s].flag);
                    const unsigned f1 = s + 1 < m ? __builtin_amdgcn_readfirstlane(w.src[s + 1].flag) : 0u;
                    if (f0 & f1 & kFarSrc) {
                        TableTerms t0, t1;
                        const bool ok0 = table_terms_inside<ORDER>(a.tv, a.pc, xi, yi, zi, r0, t0);
                        const bool ok1 = table_terms_inside<ORDER>(a.tv, a.pc, xi, yi, zi, r1, t1);
                        if (__ballot(!(ok0 && ok1)) == 0) {
                            one(r0, t0, f0, s);
                            one(r1, t1, f1, s + 1);
                            s += 2;
                            continue;
                        }
                    }
                    one(r0, table_terms<ORDER, false, COMPLETE>(a.tv, nodes, a.pc, xi, yi, zi, hi, r0,
                                                                w.src[s].own == i, active),
                        f0, s);
                    ++s;
                }
            } else {
                // this lane's source of each SPLIT, the terms added in order
                for (int s = 0; s < m; s += SPLIT) {
                    const int mine = min(s + lane / kOwned, m - 1);
                    const WalkSrc src = w.src[mine];
                    TableTerms t;
                    bool ok = (src.flag & kFarSrc) != 0;
                    if (__ballot(!ok) == 0) ok = table_terms_inside<ORDER>(a.tv, a.pc, xi, yi, zi, src.r, t);
                    if (__ballot(!ok) != 0)
                        t = table_terms<ORDER, false, COMPLETE>(a.tv, nodes, a.pc, xi, yi, zi, hi, src.r, src.own == i,
                                                                  active);
                    float mS[SPLIT], mm[SPLIT], dx[SPLIT], dy[SPLIT], Fz[SPLIT];
                    spread<SPLIT>(src.r.m * t.S, mS);
                    spread<SPLIT>(src.r.m, mm);
                    spread<SPLIT>(t.dx, dx);
                    spread<SPLIT>(t.dy, dy);
                    spread<SPLIT>(t.Fz, Fz);
#pragma unroll
                    for (int k = 0; k < SPLIT; ++k) {
                        if (s + k >= m) break;
                        add(mS[k], mm[k], dx[k], dy[k], Fz[k]);
                        flush(__builtin_amdgcn_readfirstlane(w.src[s + k].flag));
                    }
                }
            }
        }
    }
    kahan_add(sx, cx, px);
    kahan_add(sy, cy, py);
    kahan_add(sz, cz, pz);
    if (wave % SPLIT == 0 && lane == 0) {
        a.wave_cells[group] = n_cell;
        a.wave_parts[group] = n_part;
    }
    if (!active || lane >= kOwned) return;
    // acceleration in the rotated frame (the sums carry the opposite sign)
    double gx = -(double)(sx - cx), gy = -(double)(sy - cy);
    const float gz = -(sz - cz);
    if (a.n_bins > 0) {  // radial correction, linear between bin centres
        const double rho = sqrt(xi * xi + yi * yi);
        if (rho > 0.0) {
            const double t = rho / a.corr_step - 0.5;
            double dlt;
            if (t <= 0.0) {
                dlt = a.corr[0];
            } else if (t >= a.n_bins - 1) {
                dlt = a.corr[a.n_bins - 1];
            } else {
                const int k = (int)t;
                const double fr = t - k;
                dlt = (1.0 - fr) * a.corr[k] + fr * a.corr[k + 1];
            }
            gx -= dlt * xi / rho;
            gy -= dlt * yi / rho;
        }
    }
    const int o = a.idx[i];
    a.ax[o] = (float)(a.c * gx + a.s * gy);
    a.ay[o] = (float)(-a.s * gx + a.c * gy);
    a.az[o] = gz;
}

// ---------------------------------------------------------------- calibration
// per-bin sum and count of the radial error, one block per bin (fixed order)
__global__ __launch_bounds__(kBlock) void radial_bins_kernel(const double *pos, const float *at, const float *ad,
                                                             int N, double rdom, int n_bins, double *sum,
                                                             double *cnt) {
    __shared__ double s_sum[kBlock], s_cnt[kBlock];
    const int b = blockIdx.x;
    double su = 0.0, cn = 0.0;
    for (int i = threadIdx.x; i < N; i += kBlock) {
        const double x = pos[i], y = pos[N + i];
        const double rho = sqrt(x * x + y * y);
        int k = (int)floor(rho / rdom * n_bins);
        k = k < 0 ? 0 : (k > n_bins - 1 ? n_bins - 1 : k);
        if (k != b) continue;
        if (rho > 0.0) {
            const double ex = (double)at[i] - (double)ad[i], ey = (double)at[N + i] - (double)ad[N + i];
            su += (ex * x + ey * y) / rho;
        }
        cn += 1.0;
    }
    s_sum[threadIdx.x] = su;
    s_cnt[threadIdx.x] = cn;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            s_sum[threadIdx.x] += s_sum[threadIdx.x + w];
            s_cnt[threadIdx.x] += s_cnt[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sum[b] += s_sum[0];
        cnt[b] += s_cnt[0];
    }
}

__global__ void zero_kernel(double *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

unsigned blocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

#define TRY(x)                                                   \
    do {                                                         \
        hipError_t e_ = (x);                                     \
        if (e_ != hipSuccess) return hip_status(e_, #x);         \
    } while (0)

int build(steps_cyl_tree *t, const double *pos, const double *mass, const double *eps, int64_t N, double L,
          double R_dom, double shift, double angle, hipStream_t stream, Frame &f, double &side) {
    const int n = (int)N;
    TRY(ensure_particles(t, N));
    side = 2.0 * std::fmax(L, 2.0 * R_dom);
    f.c = std::cos(angle);
    f.s = std::sin(angle);
    f.shift = shift;
    f.L = L;
    f.lo[0] = -0.5 * side;
    f.lo[1] = -0.5 * side;
    f.lo[2] = 0.5 * L - 0.5 * side;
    f.scale = (double)(1 << kLevels) / side;
    hipLaunchKernelGGL(keys_kernel, dim3(blocks(N)), dim3(kBlock), 0, stream, pos, N, f, t->tx, t->ty, t->tz,
                       t->key_in, t->idx_in, t->levels);
    TRY(hipGetLastError());
    size_t bytes = t->cub_bytes;
    TRY(rocprim::radix_sort_pairs(t->cub_tmp, bytes, t->key_in, t->key_out, t->idx_in, t->idx_out, n, 0, 63,
                                           stream));
    hipLaunchKernelGGL(gather_kernel, dim3(blocks(N)), dim3(kBlock), 0, stream, t->idx_out, n, t->tx, t->ty, t->tz,
                       mass, eps, t->sx, t->sy, t->sz, t->sm, t->sh, t->key_out, t->leaf_size, t->depth, t->first,
                       t->levels);
    TRY(hipGetLastError());
    bytes = t->cub_bytes;
    TRY(rocprim::inclusive_scan(t->cub_tmp, bytes, t->first, t->first_sum, (size_t)n, rocprim::plus<int64_t>(),
                                stream));
    int64_t below = 0;  // cells below the root
    int open[kLevels];
    TRY(hipMemcpyAsync(&below, t->first_sum + (n - 1), sizeof(below), hipMemcpyDeviceToHost, stream));
    TRY(hipMemcpyAsync(open, t->levels, sizeof(open), hipMemcpyDeviceToHost, stream));
    TRY(hipStreamSynchronize(stream));
    if (below + 1 > ((int64_t)1 << 30))
        return fail(STEPS_EINVAL, "more than 2^30 tree cells (coincident particles?)");
    const int total = (int)below + 1;
    TRY(ensure_cells(t, total));
    LevelStarts ls;
    for (int l = 0, at = 0; l < kLevels; at += open[l++]) ls.at[l] = at;
    hipLaunchKernelGGL(cells_kernel, dim3(blocks(N)), dim3(kBlock), 0, stream, t->key_out, t->depth, t->first,
                       t->first_sum, n, total, t->leaf_size, side, ls, t->levels + 32, t->cells, t->cell_level,
                       t->open_cells);
    TRY(hipGetLastError());
    // moments: the leaves, then the open cells bottom-up
    for (int l = kLevels; l >= 0; --l) {
        const int *list = l < kLevels ? t->open_cells + ls.at[l] : nullptr;
        const int cnt = l < kLevels ? open[l] : total;
        if (!cnt) continue;
        hipLaunchKernelGGL((t->quadrupole ? moments_kernel<true> : moments_kernel<false>), dim3(blocks(cnt)),
                           dim3(kBlock), 0, stream, list, cnt, t->cap_cells, t->cells, t->c_m, t->c_mx, t->c_my,
                           t->c_mz, t->c_h, t->c_q, t->sx, t->sy, t->sz, t->sm, t->sh);
        TRY(hipGetLastError());
    }
    // target groups and the walk's nodes
    hipLaunchKernelGGL(count_kernel, dim3(blocks(total)), dim3(kBlock), 0, stream, t->cells, total, t->n_in);
    TRY(hipGetLastError());
    bytes = t->cub_bytes;
    TRY(rocprim::inclusive_scan(t->cub_tmp, bytes, t->n_in, t->n_sum, (size_t)total, rocprim::plus<uint64_t>(),
                                stream));
    hipLaunchKernelGGL(nodes_kernel, dim3(blocks(total)), dim3(kBlock), 0, stream, t->cells, t->cell_level, total,
                       t->c_m, t->c_mx, t->c_my, t->c_mz, t->c_h, t->c_q, t->cap_cells, t->quadrupole, t->key_out, f,
                       side, t->n_in, t->n_sum, t->g_start, t->g_count, t->nodes, t->node_q);
    TRY(hipGetLastError());
    uint64_t sums = 0;
    TRY(hipMemcpyAsync(&sums, t->n_sum + (total - 1), sizeof(sums), hipMemcpyDeviceToHost, stream));
    TRY(hipStreamSynchronize(stream));
    const int ng = (int)(uint32_t)sums;
    t->n_groups = ng;
    t->n_cells = total;
    t->n = N;
    return STEPS_OK;
}

int walk(steps_cyl_tree *t, const steps_cyl_table *table, int order, double L, double theta, const Frame &f,
         bool correct, float *out_acc, hipStream_t stream) {
    WalkArgs a;
    a.nodes = t->nodes;
    a.node_q = t->node_q;
    a.sx = t->sx;
    a.sy = t->sy;
    a.sz = t->sz;
    a.sm = t->sm;
    a.sh = t->sh;
    a.idx = t->idx_out;
    a.g_start = t->g_start;
    a.g_count = t->g_count;
    a.n_groups = (int)t->n_groups;
    a.ax = out_acc;
    a.ay = out_acc + t->n;
    a.az = out_acc + 2 * t->n;
    a.wave_cells = t->wave_cells;
    a.wave_parts = t->wave_parts;
    a.corr = t->corr;
    a.tv = table_view(table);
    a.pc = period_consts(L);
    a.theta2 = theta * theta;
    a.c = f.c;
    a.s = f.s;
    a.n_bins = correct ? t->n_bins : 0;
    a.corr_step = t->n_bins ? t->corr_rdom / t->n_bins : 1.0;
    // Waves per group, by the number of groups (about N / 45; there are 1024
    // SIMDs) and what a source costs.  ms per call at SPLIT 1, 2, 4: CIC N =
    // 20000 1.41, 1.07, 0.91, 50000 1.66, 1.32, 1.30, 100003 2.08, 1.85, 2.08,
    // 200000 2.90, 3.01, 3.54; TSC 50000 1.82, 1.20, 1.16, 100003 2.21, 1.84,
    // 1.87, 400000 5.38, 4.97, 5.77, 2^20 12.3, 12.2, 15.1.
    const int64_t g = t->n_groups;
    const int split = t->quadrupole ? 1 : order == 1 ? (g <= 1100 ? 4 : g <= 3300 ? 2 : 1) : (g <= 1600 ? 4 : g <= 16384 ? 2 : 1);
    const int64_t threads = t->n_groups * 64 * split;
    const dim3 grid((unsigned)((threads + kWalkBlock - 1) / kWalkBlock)), block(kWalkBlock);
    auto launch = [&](auto order_c, auto quad_c, auto complete_c) {
        constexpr int O = decltype(order_c)::value;
        constexpr bool Q = decltype(quad_c)::value, C = decltype(complete_c)::value;
        if (Q || split == 1)
            hipLaunchKernelGGL((tree_walk_kernel<O, Q, C, 1>), grid, block, 0, stream, a);
        else if (split == 2)
            hipLaunchKernelGGL((tree_walk_kernel<O, false, C, 2>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((tree_walk_kernel<O, false, C, 4>), grid, block, 0, stream, a);
    };
    auto with_table = [&](auto order_c, auto quad_c) {
        if (a.tv.complete)
            launch(order_c, quad_c, std::true_type{});
        else
            launch(order_c, quad_c, std::false_type{});
    };
    auto with_quad = [&](auto order_c) {
        if (t->quadrupole)
            with_table(order_c, std::true_type{});
        else
            with_table(order_c, std::false_type{});
    };
    if (order == 2)
        with_quad(std::integral_constant<int, 2>{});
    else
        with_quad(std::integral_constant<int, 1>{});
    return hip_status(hipGetLastError(), "tree walk");
}

int check_common(const double *pos, const double *mass, const double *eps, int64_t N, double L, double R_dom,
                 const steps_cyl_table *table, int order, double theta) {
    if (!pos || !mass || !eps || !table) return fail(STEPS_EINVAL, "pos, mass, eps and table must be non-null");
    if (N < 1 || N > STEPS_MAX_N) return fail(STEPS_EINVAL, "N=%lld outside [1, 2^29]", (long long)N);
    if (!finite_positive(L) || !finite_positive(R_dom)) return fail(STEPS_EINVAL, "L and R_dom must be finite and > 0");
    if (order != 1 && order != 2) return fail(STEPS_EINVAL, "order=%d: 1 (CIC) or 2 (TSC)", order);
    if (!std::isfinite(theta) || theta < 0.0) return fail(STEPS_EINVAL, "theta must be finite and >= 0");
    return STEPS_OK;
}

}  // namespace
}  // namespace steps

using namespace steps;

STEPS_API int steps_cyl_tree_create(int leaf_size, int quadrupole, steps_cyl_tree **out) {
    if (!out) return fail(STEPS_EINVAL, "out must be non-null");
    if (leaf_size < 1 || leaf_size > 64) return fail(STEPS_EINVAL, "leaf_size=%d outside [1, 64]", leaf_size);
    if (quadrupole != 0 && quadrupole != 1) return fail(STEPS_EINVAL, "quadrupole must be 0 or 1");
    clear_error();
    steps_cyl_tree *t = new (std::nothrow) steps_cyl_tree();
    if (!t) return fail(STEPS_ENOMEM, "out of host memory");
    t->leaf_size = leaf_size;
    t->quadrupole = quadrupole;
    *out = t;
    return STEPS_OK;
}

STEPS_API void steps_cyl_tree_destroy(steps_cyl_tree *t) {
    if (!t) return;
    void *ptrs[] = {t->cub_tmp, t->tx, t->ty, t->tz, t->key_in, t->key_out, t->idx_in, t->idx_out, t->sx, t->sy,
                    t->sz, t->sm, t->sh, t->depth, t->first, t->first_sum, t->levels, t->c_m, t->c_mx, t->c_my, t->c_mz,
                    t->c_h, t->c_q, t->open_cells, t->n_in, t->n_sum, t->nodes, t->node_q, t->cells, t->cell_level,
                    t->wave_cells, t->wave_parts, t->corr, t->bin_sum, t->g_start, t->g_count, t->bin_cnt, t->acc_dir,
                    t->acc_tree};
    for (void *p : ptrs) (void)hipFree(p);
    delete t;
}

STEPS_API int steps_cyl_tree_forces(steps_cyl_tree *t, const double *pos, const double *mass, const double *eps,
                                    int64_t N, double L, double R_dom, const steps_cyl_table *table, int order,
                                    double theta, double shift, double angle, int correct, float *out_acc,
                                    hipStream_t stream) {
    if (!t || !out_acc) return fail(STEPS_EINVAL, "tree and out_acc must be non-null");
    int rc = check_common(pos, mass, eps, N, L, R_dom, table, order, theta);
    if (rc) return rc;
    if (!std::isfinite(shift) || !std::isfinite(angle)) return fail(STEPS_EINVAL, "shift and angle must be finite");
    if (correct && t->n_bins == 0) return fail(STEPS_EINVAL, "no radial correction has been set");
    if ((rc = require_device())) return rc;
    clear_error();
    Frame f;
    double side;
    if ((rc = build(t, pos, mass, eps, N, L, R_dom, shift, angle, stream, f, side))) return rc;
    return walk(t, table, order, L, theta, f, correct != 0, out_acc, stream);
}

STEPS_API int steps_cyl_tree_set_correction(steps_cyl_tree *t, const double *corr, int n_bins, double R_dom) {
    if (!t) return fail(STEPS_EINVAL, "tree must be non-null");
    if (n_bins == 0) {
        clear_error();
        t->n_bins = 0;
        return STEPS_OK;
    }
    if (!corr || n_bins < 1 || n_bins > kMaxBins || !finite_positive(R_dom))
        return fail(STEPS_EINVAL, "need corr, 1 <= n_bins <= %d and R_dom > 0", kMaxBins);
    for (int k = 0; k < n_bins; ++k)
        if (!std::isfinite(corr[k])) return fail(STEPS_EINVAL, "non-finite correction");
    int rc = require_device();
    if (rc) return rc;
    clear_error();
    if (!t->corr) STEPS_CHECK_HIP(hipMalloc(&t->corr, kMaxBins * sizeof(double)));
    STEPS_CHECK_HIP(hipMemcpy(t->corr, corr, n_bins * sizeof(double), hipMemcpyHostToDevice));
    t->n_bins = n_bins;
    t->corr_rdom = R_dom;
    return STEPS_OK;
}

STEPS_API int steps_cyl_tree_calibrate(steps_cyl_tree *t, const double *pos, const double *mass, const double *eps,
                                       int64_t N, double L, double R_dom, const steps_cyl_table *table, int order,
                                       double theta, const double *shifts, const double *angles, int n_real,
                                       int n_bins, double *out_corr, hipStream_t stream) {
    if (!t || !shifts || !angles) return fail(STEPS_EINVAL, "tree, shifts and angles must be non-null");
    int rc = check_common(pos, mass, eps, N, L, R_dom, table, order, theta);
    if (rc) return rc;
    if (n_real < 1 || n_real > 1024) return fail(STEPS_EINVAL, "n_real=%d outside [1, 1024]", n_real);
    if (n_bins < 1 || n_bins > kMaxBins) return fail(STEPS_EINVAL, "n_bins=%d outside [1, %d]", n_bins, kMaxBins);
    for (int k = 0; k < n_real; ++k)
        if (!std::isfinite(shifts[k]) || !std::isfinite(angles[k]))
            return fail(STEPS_EINVAL, "shifts and angles must be finite");
    if ((rc = require_device())) return rc;
    clear_error();
    if (N > t->cap_cal) {
        (void)hipFree(t->acc_dir);
        (void)hipFree(t->acc_tree);
        t->acc_dir = t->acc_tree = nullptr;
        t->cap_cal = 0;
        STEPS_CHECK_HIP(hipMalloc(&t->acc_dir, 3 * N * sizeof(float)));
        STEPS_CHECK_HIP(hipMalloc(&t->acc_tree, 3 * N * sizeof(float)));
        t->cap_cal = N;
    }
    if (!t->bin_sum) {
        STEPS_CHECK_HIP(hipMalloc(&t->bin_sum, kMaxBins * sizeof(double)));
        STEPS_CHECK_HIP(hipMalloc(&t->bin_cnt, kMaxBins * sizeof(double)));
    }
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(kBlock), 0, stream, t->bin_sum, kMaxBins);
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(kBlock), 0, stream, t->bin_cnt, kMaxBins);
    STEPS_CHECK_HIP(hipGetLastError());
    rc = steps_cyl_forces_table(pos, mass, eps, N, L, table, order, nullptr, N, t->acc_dir, nullptr, stream);
    if (rc) return rc;
    for (int k = 0; k < n_real; ++k) {
        Frame f;
        double side;
        if ((rc = build(t, pos, mass, eps, N, L, R_dom, shifts[k], angles[k], stream, f, side))) return rc;
        if ((rc = walk(t, table, order, L, theta, f, false, t->acc_tree, stream))) return rc;
        hipLaunchKernelGGL(radial_bins_kernel, dim3(n_bins), dim3(kBlock), 0, stream, pos, t->acc_tree, t->acc_dir,
                           (int)N, R_dom, n_bins, t->bin_sum, t->bin_cnt);
        STEPS_CHECK_HIP(hipGetLastError());
    }
    std::vector<double> s(n_bins), c(n_bins), corr(n_bins);
    STEPS_CHECK_HIP(hipMemcpyAsync(s.data(), t->bin_sum, n_bins * sizeof(double), hipMemcpyDeviceToHost, stream));
    STEPS_CHECK_HIP(hipMemcpyAsync(c.data(), t->bin_cnt, n_bins * sizeof(double), hipMemcpyDeviceToHost, stream));
    STEPS_CHECK_HIP(hipStreamSynchronize(stream));
    for (int k = 0; k < n_bins; ++k) corr[k] = c[k] > 0.0 ? s[k] / c[k] : 0.0;
    if (out_corr)
        for (int k = 0; k < n_bins; ++k) out_corr[k] = corr[k];
    return steps_cyl_tree_set_correction(t, corr.data(), n_bins, R_dom);
}

STEPS_API int steps_cyl_tree_info(const steps_cyl_tree *t, int64_t *n_cells, int64_t *cell_interactions,
                                  int64_t *particle_interactions) {
    if (!t) return fail(STEPS_EINVAL, "tree must be non-null");
    clear_error();
    if (n_cells) *n_cells = t->n_cells;
    if (cell_interactions || particle_interactions) {
        const int64_t waves = t->n_groups;
        std::vector<int> wc(waves), wp(waves), gc(waves);
        if (waves) {
            STEPS_CHECK_HIP(hipMemcpy(wc.data(), t->wave_cells, waves * sizeof(int), hipMemcpyDeviceToHost));
            STEPS_CHECK_HIP(hipMemcpy(wp.data(), t->wave_parts, waves * sizeof(int), hipMemcpyDeviceToHost));
            STEPS_CHECK_HIP(hipMemcpy(gc.data(), t->g_count, waves * sizeof(int), hipMemcpyDeviceToHost));
        }
        int64_t sc = 0, sp = 0;
        for (int64_t w = 0; w < waves; ++w) {
            sc += (int64_t)gc[w] * wc[w];
            sp += (int64_t)gc[w] * wp[w];
        }
        if (cell_interactions) *cell_interactions = sc;
        if (particle_interactions) *particle_interactions = sp;
    }
    return STEPS_OK;
}

STEPS_API int steps_cyl_tree_cells(const steps_cyl_tree *t, int *host_level, int *host_start, int *host_count,
                                   int *host_skip, int *host_leaf, double *host_mass, double *host_com,
                                   int *host_order) {
    if (!t) return fail(STEPS_EINVAL, "tree must be non-null");
    clear_error();
    const int64_t n = t->n_cells;
    std::vector<CellRec> r(n);
    if (n) STEPS_CHECK_HIP(hipMemcpy(r.data(), t->cells, n * sizeof(CellRec), hipMemcpyDeviceToHost));
    if (host_level && n) STEPS_CHECK_HIP(hipMemcpy(host_level, t->cell_level, n * sizeof(int), hipMemcpyDeviceToHost));
    for (int64_t k = 0; k < n; ++k) {
        if (host_start) host_start[k] = r[k].start;
        if (host_count) host_count[k] = r[k].count;
        if (host_skip) host_skip[k] = r[k].skip;
        if (host_leaf) host_leaf[k] = r[k].leaf;
        if (host_mass) host_mass[k] = r[k].mass;
        if (host_com) {
            host_com[k] = r[k].cx;
            host_com[n + k] = r[k].cy;
            host_com[2 * n + k] = r[k].cz;
        }
    }
    if (host_order && t->n)
        STEPS_CHECK_HIP(hipMemcpy(host_order, t->idx_out, t->n * sizeof(int), hipMemcpyDeviceToHost));
    return STEPS_OK;
}
