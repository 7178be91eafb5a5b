// What the pairwise force paths share (forces_pairwise.hip, forces_learned.hip):
// the schedule of their tiles, the staged records and the last pass.
//
// Layout.  The particles are put in spatial (Morton) order and staged as 32-byte
// records {x, y, z wrapped, m, h}, with a bounding box per run of 64 records.  A
// part is a run of records that a workgroup owns, a group S parts.  Each particle
// has M sets of S slots of FP64 sums (x, y, z, potential).
//
// Schedule (bitwise deterministic, no atomics).  G groups meet in G' rounds (G' =
// G rounded up to even): in round 0 every group meets itself, and rounds 1 ..
// G'-1 are a round-robin tournament: in round r + 1 group G'-1 meets group r and,
// for k = 1 .. G'/2 - 1, group (r + k) mod (G'-1) meets group (r - k) mod (G'-1),
// so every unordered pair of groups meets exactly once and no group appears twice
// in a round.  A meeting of groups a and b takes S^2 tiles: tile (i, j) holds part
// i of a and streams part j of b, adding a's sums into slot j of part i and b's
// reactions into slot i of part j.  A group meets itself in the S (S + 1)/2 tiles
// i <= j; tile (i, i) is one-sided and adds to slot i alone.  So within a round
// each slot has one writer.  A launch runs up to M rounds, each in a slot set of
// its own; the first launch writes its sets (zeros where a partner is missing),
// later ones add to them in launch order.  A last pass adds the slots in order
// and writes FP32 outputs at the particles' own positions.
//
// As many rounds share a launch as the slots' memory allows, up to one launch of
// one group of all parts (flat: S = P, every slot written once); there each tile
// may be split over Q workgroups of 1/Q of its sources (the learned path; the others
// split it over the waves of a workgroup).
#pragma once

#include <algorithm>

#include "common.h"
#include "pair_f64.h"
#include "pair_fp32.h"

namespace steps {
namespace {

// Bytes of FP64 sum slots of a call.  Up to kScratchN particles the slots (and
// what else a call takes) fit the 128 MiB array of steps_cyl_forces_noalloc,
// which then runs the same schedule; above, more rounds share a launch.
constexpr int64_t kScratchN = 125000;
constexpr size_t kSlotBytesScratch = (size_t)112 << 20, kSlotBytes = (size_t)256 << 20;
constexpr size_t kSetBytes = 32;  // per particle and slot

// Below this many particles the parts are runs of the particles' own order:
// what the order saves in near tiles is less than the 60 us that sorting costs
// (us per call without and with it: N = 8000 160 and 191, 10000 247 and 266, 12000
// 331 and 349, 14000 432 and 436; with a CIC table 130 and 152, 205 and 207, 273 and
// 262; learned 1879 and 1910, 2932 and 2956, 4226 and 4237).
constexpr int64_t kSortMin = 10240;

struct Schedule {
    int S, M, Q;  // parts per group, slot sets, workgroups per tile (Q > 1: flat)
    bool flat;    // one group
};

// Groups of `S` parts of `part` particles, as many sets as fit `budget` bytes (0:
// the default); a budget above kScratchN that holds no set of S (the static
// array's) takes fewer parts per group.  Flat where all parts' slots fit.
inline Schedule make_schedule(int64_t N, int part, int S, size_t budget) {
    const int64_t P = (N + part - 1) / part;
    const bool fixed = budget > 0 && N > kScratchN;
    if (budget == 0) budget = N <= kScratchN ? kSlotBytesScratch : kSlotBytes;
    Schedule s = {S, 1, 1, false};
    if (N <= kScratchN && (size_t)P * N * kSetBytes <= budget) {
        s.S = (int)P;
        s.flat = true;
        return s;
    }
    while (fixed && s.S > 1 && (size_t)s.S * N * kSetBytes > budget) s.S >>= 1;
    s.M = (int)std::max<int64_t>(1, (int64_t)(budget / ((size_t)s.S * N * kSetBytes)));
    const int64_t G = (P + s.S - 1) / s.S;
    const int rounds = G > 1 ? (int)(G + (G & 1)) : 1;
    const int launches = (rounds + s.M - 1) / s.M;
    s.M = (rounds + launches - 1) / launches;  // launches of equal length, every set written by the first
    return s;
}

inline size_t slot_bytes(const Schedule &s, int64_t N) { return (size_t)s.S * s.M * s.Q * N * kSetBytes; }

// the meetings of one launch
struct Rounds {
    int S, Q, G, Gp;  // parts per group, workgroups per tile, groups, groups rounded up to even
    int round;        // first round of the launch (0: the groups' own meetings)
    int first;        // the slots are written, not added to
    unsigned own;     // workgroups of round 0 in this launch
};

struct Tile {
    int64_t pa, pb;      // owned part, source part (past the last part: none)
    int q;               // which 1/Q of its sources
    int slot_a, slot_b;  // slot of the owned sums, of the reactions
};

// Tile `at` of a launch: round 0's first (tiles i <= j of every group, Q
// workgroups each), then S^2 per meeting of the launch's other rounds.
__device__ __forceinline__ Tile tile_of(const Rounds &r, unsigned at) {
    Tile t;
    const int S = r.S, Q = r.Q;
    int ga, gb, pi, pj, set = 0;
    t.q = 0;
    if (at < r.own) {
        const unsigned T = (unsigned)S * (S + 1) / 2;
        const unsigned tile = at / Q;
        t.q = (int)(at % Q);
        ga = gb = (int)(tile / T);
        const unsigned c = tile % T;  // by columns: c = j (j + 1)/2 + i, i <= j
        pj = (int)((__builtin_sqrtf(8.f * (float)c + 1.f) - 1.f) * 0.5f);
        while ((unsigned)(pj + 1) * (pj + 2) / 2 <= c) ++pj;
        while ((unsigned)pj * (pj + 1) / 2 > c) --pj;
        pi = (int)(c - (unsigned)pj * (pj + 1) / 2);
    } else {
        const unsigned w = at - r.own;
        const unsigned per = (unsigned)S * S, half = r.Gp / 2;
        const unsigned meeting = w / per;
        const int meet = (int)(meeting % half);
        set = (int)(meeting / half) + (r.own ? 1 : 0);
        const int round = r.round + set - 1;
        const int M = r.Gp - 1;
        if (meet == 0) {
            ga = M;
            gb = round;
        } else {
            ga = (round + meet) % M;
            gb = (round - meet + M) % M;
        }
        pi = (int)((w % per) / S);
        pj = (int)((w % per) % S);
    }
    // the empty group of an odd count lies past the last part
    t.pa = (int64_t)ga * S + pi;
    t.pb = (int64_t)gb * S + pj;
    t.slot_a = (set * S + pj) * Q + t.q;
    t.slot_b = (set * S + pi) * Q;
    return t;
}

// Calls launch(rounds, workgroups) for each launch of the schedule.
template <class F>
hipError_t each_launch(const Schedule &s, int N, int part, F &&launch) {
    Rounds rd;
    const int64_t group = (int64_t)part * s.S;
    rd.S = s.S;
    rd.Q = s.Q;
    rd.G = (int)((N + group - 1) / group);
    rd.Gp = rd.G + (rd.G & 1);
    const int rounds = rd.G > 1 ? rd.Gp : 1;
    hipError_t e = hipSuccess;
    for (int r = 0; e == hipSuccess && r < rounds; r += s.M) {
        const int k = std::min(s.M, rounds - r);
        rd.round = r;
        rd.first = r == 0;
        rd.own = r == 0 ? (unsigned)rd.G * s.S * (s.S + 1) / 2 * s.Q : 0;
        e = launch(rd, rd.own + (unsigned)(k - (r == 0)) * (rd.Gp / 2) * s.S * s.S);
    }
    return e;
}

// Ends a step of a wave that hands LDS slots from lane to lane: what the next
// step reads another lane has written in this one, which the compiler, following
// one lane, cannot see.  It must keep the steps' LDS accesses in program order
// (the wave's LDS operations then complete in issue order); no instruction.
__device__ __forceinline__ void hand_over() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

constexpr int kBox = 8;  // doubles per 64-record box

// Records in the order of `perm` (null: the particles' own) and, with `box`, the
// bounding box {x_lo, x_hi, y_lo, y_hi, z_lo, z_hi, h_max, 0} of every aligned run
// of 64; one wave per run.
__global__ __launch_bounds__(256) void stage_kernel(const double *pos, const double *mass, const double *eps, int N,
                                                    double L, const int *perm, SrcRec *rec, double *box) {
    const int b = blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const int64_t k = (int64_t)b * 64 + (threadIdx.x & 63);
    if ((int64_t)b * 64 >= N) return;  // whole wave leaves together
    double v[7];
    if (k < N) {
        const int64_t p = perm ? perm[k] : k;
        SrcRec r;
        r.x = pos[p];
        r.y = pos[N + p];
        r.z = wrap_z(pos[2 * (int64_t)N + p], L);
        r.m = (float)mass[p];
        r.h = (float)eps[p];
        rec[k] = r;
        v[0] = r.x;
        v[1] = -r.x;
        v[2] = r.y;
        v[3] = -r.y;
        v[4] = r.z;
        v[5] = -r.z;
        v[6] = (double)r.h;
    } else {
        for (int c = 0; c < 6; ++c) v[c] = HUGE_VAL;  // neutral for the minima
        v[6] = 0.0;
    }
    if (!box) return;
    // minima of (x, -x, y, -y, z, -z), maximum of h, over the wave
    for (int off = 32; off >= 1; off >>= 1) {
        for (int c = 0; c < 6; ++c) v[c] = fmin(v[c], __shfl_xor(v[c], off));
        v[6] = fmax(v[6], __shfl_xor(v[6], off));
    }
    if ((threadIdx.x & 63) == 0) {
        double *o = box + (int64_t)b * kBox;
        o[0] = v[0];
        o[1] = -v[1];
        o[2] = v[2];
        o[3] = -v[3];
        o[4] = v[4];
        o[5] = -v[5];
        o[6] = v[6];
        o[7] = 0.0;
    }
}

// One component of 64 particles per workgroup, whose waves take
// equal runs of the slots (added in order, then the runs in order): few
// particles have many slots, and what bounds the pass is the loads in flight
// (N = 4096, 128 slots: 17 us with one thread per particle, 4.6 us in 16 runs).  With
// Q > 1 waves per tile (one group) slot o Q + q is written for every q where
// the particle's own part p <= o acted, and for q = 0 alone where it reacted.
__global__ __launch_bounds__(1024) void finish_kernel(const double *sum, int slots, int Q, int part_size,
                                                      const int *perm, int N, float *ax, float *ay, float *az,
                                                      float *pot) {
    __shared__ double run[16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int c = blockIdx.y;
    const int k = blockIdx.x * 64 + lane;
    double s = 0.0;
    if (k < N) {
        const double *p = sum + (int64_t)c * N + k;
        const int64_t stride = 4 * (int64_t)N;
        const int skip = Q > 1 ? blockIdx.x * 64 / part_size : 0;  // parts that hold one slot
        const int total = skip + (slots - skip) * Q;
        const int each = (total + waves - 1) / waves;
        const int end = min(total, (wave + 1) * each);
#pragma unroll 8
        for (int e = wave * each; e < end; ++e) s += p[(e < skip ? e * Q : skip * Q + (e - skip)) * stride];
    }
    run[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && k < N) {
        for (int w = 1; w < waves; ++w) s += run[w][lane];
        const int64_t i = perm ? perm[k] : k;
        // attraction: a = -sum m_j S (x_i - x_j), potential = -sum m_j / r
        float *out = c == 0 ? ax : c == 1 ? ay : c == 2 ? az : pot;
        out[i] = (float)(-s);
    }
}

// ---- per-target lists: source chunks, whose totals are slots of launch_finish

inline int finish_waves(int slots) { return slots > 64 ? 16 : 4; }

// Up to this many sources a target's bits do not depend on the list.
constexpr int64_t kSameBits = 4096;

struct Chunks {
    int n;
    bool folded;    // a workgroup takes every chunk and adds their totals itself
    int64_t piece;  // targets per launch
};

// Source chunks for n_tgt targets of N sources in blocks of `block`: enough
// (target block, chunk) pairs for 8192 workgroups (eight to a CU's four resident
// ones, so that the last to finish cost little), chunks of at least min_chunk
// sources; one chunk once the targets fill the device.  The exact kernel's us per
// call with 2048 workgroups and 4096 sources, and so: 256 of 262144 particles 1428
// -> 321, 4096 of them 4215 -> 3945, 1000 of 50000 1365 -> 282, 300 of 10000 484 ->
// 50.  Where `room` bytes do not hold the totals the former two numbers apply.  Up to
// kSameBits sources the chunks are the same in any case: long lists go in pieces that
// fill the device, and where the totals have no room they are folded (140,003
// targets of 4096, |n| <= 8: 2321 and 3240 us).
inline Chunks target_chunks(int64_t N, int64_t n_tgt, int block, int min_chunk, size_t room) {
    const int64_t blocks = (n_tgt + block - 1) / block;
    auto chunks = [&](int64_t groups, int64_t least) {
        return (int)std::min((groups + blocks - 1) / blocks, (N + least - 1) / least);
    };
    if (N > kSameBits) {
        const int c = chunks(8192, min_chunk);
        return {(size_t)c * 4 * n_tgt * sizeof(double) <= room ? c : chunks(2048, 4096), false, n_tgt};
    }
    const int all = (int)((N + min_chunk - 1) / min_chunk);
    const int64_t pieces = all > 1 ? (blocks * all + 8191) / 8192 : 1;
    const int64_t piece = std::min(n_tgt, (blocks + pieces - 1) / pieces * block);
    const bool folded = all > 1 && (size_t)all * 4 * piece * sizeof(double) > room;
    return {all, folded, folded ? n_tgt : piece};
}

// Bytes of a launch's totals, and of those and a list's spatial order.
inline size_t totals_bytes(const Chunks &c) {
    return c.n > 1 && !c.folded ? (size_t)c.n * 4 * c.piece * sizeof(double) : 0;
}

inline size_t list_bytes(int64_t n_tgt, const Chunks &c) {
    return ws_total({per_target_bytes(n_tgt), totals_bytes(c)});
}

// The chunks that a workspace of `size` bytes has room for.
inline Chunks chunks_in(size_t size, int64_t N, int64_t n_tgt, int block, int min_chunk) {
    const Chunks c = target_chunks(N, n_tgt, block, min_chunk, SIZE_MAX);
    return size < list_bytes(n_tgt, c) ? target_chunks(N, n_tgt, block, min_chunk, 0) : c;
}

// Adds a chunk's totals as finish_kernel adds slots: in runs, then the runs in
// order.  f: LDS, [8][stride], the run's sums and the total's; `ends`: of the run.
__device__ __forceinline__ void fold_chunk(double *f, int stride, double x, double y, double z, double p, bool ends) {
    const double v[4] = {x, y, z, p};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double r = f[c * stride] + v[c];
        if (ends) f[(4 + c) * stride] += r;
        f[c * stride] = ends ? 0.0 : r;
    }
}

hipError_t launch_stage(const double *pos, const double *mass, const double *eps, int N, double L, const int *perm,
                        SrcRec *rec, double *box, hipStream_t stream) {
    const int nbox = (N + 63) / 64;
    hipLaunchKernelGGL(stage_kernel, dim3((nbox + 3) / 4), dim3(256), 0, stream, pos, mass, eps, N, L, perm, rec, box);
    return hipGetLastError();
}

// `stride`: elements between the components of out_acc
hipError_t launch_finish(const Schedule &s, const double *sum, int part, const int *perm, int N, float *out_acc,
                         int64_t stride, float *out_pot, hipStream_t stream) {
    const int slots = s.S * s.M;
    hipLaunchKernelGGL(finish_kernel, dim3((N + 63) / 64, out_pot ? 4 : 3), dim3(64 * finish_waves(slots * s.Q)), 0,
                       stream, sum, slots, s.Q, part, perm, N, out_acc, out_acc + stride, out_acc + 2 * stride, out_pot);
    return hipGetLastError();
}

}  // namespace
}  // namespace steps
