// Cell-to-cell transport on gfx950 (paper: section "Transport Algorithm", its four stages; the
// track-length flux estimator of eqs. 5-7).
//
// A "world" holds a structure-of-arrays particle bank shared by any number of problems (each a
// grid of square cells with its own materials, source, seed and FP64 tallies), so one sampler
// launch serves particles of different problems and cells together.  One transport step:
//   gather  (stage 1)  bank -> canonical left-entry conditions, per-particle random stream ids;
//   sample  (stage 2)  the generative sampler (gmc_transmit kernels), or stages 1-2 in one, the
//            analog walk started from the bank;
//   apply   (stages 3-4)  FP64 rescale of the path to physical units, weight attenuation and
//            flux / absorption tallies (FP64 atomics), rotation back to the global frame, move
//            to the neighbour cell or leave / cut off, and compaction of the survivors into the
//            other bank with one atomic per workgroup's tile of particles.
// Volumetric births draw a source particle and take its first leg inside the birth cell with the
// analog walk or the internal (volumetric-source) model; surface-source births enter their
// boundary cell directly.
// Random numbers depend only on (problem seed, history id, cell-visit index): a history's
// result does not depend on which other problems share the bank or on its slot.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/gmc.h"
#include "gmc_device.hpp"
#include "gmc_internal.hpp"
#include "gmc_walk.hpp"

namespace gmc {
namespace {

struct ProblemDev {
    int32_t nx, ny;
    double L, Ly;                  // cell width (along x) and height
    float lr;                      // ln(Ly / L): 0 for square cells
    int64_t cell0;                 // first global cell index of this problem
    int32_t sx0, sy0, snx, sny;    // source block
    int32_t reflect;
    double w_min;
    uint64_t seed;
    int32_t src_face;              // -1 volumetric, else the domain side of a surface source
    int32_t xy;                    // XY geometry: directions on the sphere, projected
    uint32_t max_visits;           // a history is cut off before its cell visit of this number
};

struct BankDev {
    int32_t *cell, *pid, *entry;
    float *yin, *gx, *gy;
    double *w;
    uint32_t *hist, *event;
};

// Tallies of every cell visit, side by side per cell: deposited weight, sum of w_in * l_phys, sum
// of l_phys, number of visits.  The flux follows from the first two (eq. 7: deposit / (V sigma_a),
// or sum of w l / V where sigma_a = 0) and is formed when the tallies are read.
constexpr int kVisitTallies = 4;

// Material of a cell as a crossing needs it: the sampler's conditions ln tau and c in FP32, and
// sigma_a = (1 - c) tau / L for the tallies.
struct CellMat {
    float lt, c;
    double siga;
};

struct CellsDev {
    const double *tau;             // per global cell (births)
    const CellMat *mat;            // per global cell
    double *visit;                 // [cells][kVisitTallies]
    double *leak, *cutoff;
    // weight and number of generative samples rejected by the decoder (a part of the cutoff)
    double *rej_w, *rej_n;
    const ProblemDev *prob;
};

// Threads of a workgroup that tallies, and cells of its table.  Large launches: one workgroup of 1,024
// to a compute unit, which takes tiles of that many particles in turn, so that each fills one table:
// what a launch adds to the global tallies grows with the number of tables (the checkerboard's 128
// steps take 17.6 ms with one table of 4,096 cells to a CU and 18.1 ms with two of 2,048; the lattice's
// 30 smaller ones 16.3 and 16.1 ms).  Small ones: a workgroup of 256 to each 256 particles.
constexpr int kTallyThreads = 1024;
constexpr int kSmallTallyThreads = 256;
constexpr int tally_slots(int threads) { return threads == kTallyThreads ? 4096 : 512; }

// Per-workgroup tally staging: the visit tallies of a workgroup's particles are summed per cell in
// an LDS hash table and added to the global ones at its end.  Particles near a source crowd into
// few cells, whose same-address global atomics complete one in 12 ns.  A cell that finds neither
// its slot nor a free one within kTallyProbes probes adds to the global tallies directly.
constexpr int kTallyProbes = 4;
template <int SLOTS>
struct TallyTable {
    static constexpr int kShift = 32 - __builtin_ctz(SLOTS);   // multiplicative hash to log2(SLOTS) bits
    int32_t key[SLOTS];
    double v[SLOTS * kVisitTallies];
};
template <int SLOTS>
__device__ __forceinline__ void tally_init(TallyTable<SLOTS> &tl)
{
    for (int s = threadIdx.x; s < SLOTS; s += blockDim.x) tl.key[s] = -1;
    for (int s = threadIdx.x; s < SLOTS * kVisitTallies; s += blockDim.x) tl.v[s] = 0.0;
}

template <int SLOTS>
__device__ __forceinline__ void tally_add(TallyTable<SLOTS> &tl, const CellsDev &cd, int cell, double dw, double wl,
                                          double l)
{
    uint32_t s = ((uint32_t)cell * 2654435761u) >> TallyTable<SLOTS>::kShift;
    for (int k = 0; k < kTallyProbes; ++k) {
        const int prev = atomicCAS(&tl.key[s], -1, cell);
        if (prev == -1 || prev == cell) {
            double *v = tl.v + s * kVisitTallies;
            if (dw != 0.0) atomicAdd(v, dw);       // 0 without absorption
            atomicAdd(v + 1, wl);
            atomicAdd(v + 2, l);
            atomicAdd(v + 3, 1.0);
            return;
        }
        s = (s + 1) & (SLOTS - 1);
    }
    double *v = cd.visit + (int64_t)cell * kVisitTallies;
    if (dw != 0.0) atomicAdd(v, dw);
    atomicAdd(v + 1, wl);
    atomicAdd(v + 2, l);
    atomicAdd(v + 3, 1.0);
}

// The table to the global tallies, four lanes to a cell: the atomics of neighbouring lanes on
// neighbouring addresses travel as one request, and requests are what bounds them (scattered
// FP64 atomics 18-24 G/s; four side by side 0.012 ns each, against 0.044 ns in four arrays).
template <int SLOTS>
__device__ __forceinline__ void tally_flush(TallyTable<SLOTS> &tl, const CellsDev &cd)
{
    for (int e = threadIdx.x; e < SLOTS * kVisitTallies; e += blockDim.x) {
        const int cell = tl.key[e / kVisitTallies];
        const double v = tl.v[e];
        if (cell >= 0 && v != 0.0) atomicAdd(&cd.visit[(int64_t)cell * kVisitTallies + e % kVisitTallies], v);
    }
}

// Stage 3 for one cell visit: w_out = w e^{-sigma_a l} (eq. 5) and deposit dw (eq. 6) in FP64
// with the physical path (path_units in units of `unit`, the length of the face the walk's frame
// took as its height), plus the path tallies w l, l and one visit.
template <int SLOTS>
__device__ __forceinline__ double visit_tally(const CellsDev &cd, int cell, double sig_a, double w, float path_units,
                                              double unit, TallyTable<SLOTS> &tl)
{
    const double ls = (double)path_units * unit;
    const double dw = sig_a > 0.0 ? w * (-expm1(-sig_a * ls)) : 0.0;
    tally_add(tl, cd, cell, dw, w * ls, ls);
    return w - dw;
}

// The first-flight split's xi of one particle's cell visits (split_draw of stream hist + 2^32 visit):
// only the second counter word, the visit, changes, so two Philox rounds' other halves are the
// particle's own.
__device__ __forceinline__ DrawPrefix split_prefix(uint32_t hist, uint32_t k0, uint32_t k1)
{
    const uint64_t p0 = (uint64_t)kPhiloxM0 * hist;
    const uint64_t p1 = (uint64_t)kPhiloxM1 * ((uint32_t)(p0 >> 32) ^ kTagSplit ^ k1);
    return DrawPrefix{k0, (uint32_t)(p1 >> 32) ^ (k0 + kPhiloxW0), (uint32_t)p1, (uint32_t)p0 ^ (k1 + kPhiloxW1)};
}

__device__ __forceinline__ float split_draw(const DrawPrefix &q, uint32_t k0, uint32_t k1, uint32_t visit)
{
    const uint64_t g = (uint64_t)kPhiloxM0 * (visit ^ q.a);
    return u01(philox_rest(U4{q.b, q.c, (uint32_t)(g >> 32) ^ q.d, (uint32_t)g}, k0, k1).a);
}

struct Next {
    int32_t cell, entry;
    float yin, gx, gy;
    bool alive;
};

// Stage 4: after leaving `cell` through local face `face` at counter-clockwise position pos
// with global direction (gx, gy) and weight w_out: cut off, leak, reflect or enter the
// neighbour (whose entry face is the opposite one, entered at position 1 - pos in its own
// counter-clockwise orientation, i.e. canonical height y = pos).
__device__ __forceinline__ Next move_on(const CellsDev &cd, const ProblemDev &P, int cell, int &ci, int &cj, int face,
                                        float pos, float gx, float gy, double w_out)
{
    Next nx{cell, 0, 0.0f, gx, gy, false};
    if (face < 0 || face > 3) {              // capped walk or rejected sample: drop its weight
        atomicAdd(&cd.cutoff[cell], w_out);  // with the cutoff
        if (face == -1) {
            atomicAdd(&cd.rej_w[cell], w_out);
            atomicAdd(&cd.rej_n[cell], 1.0);
        }
        return nx;
    }
    if (w_out < P.w_min) {
        atomicAdd(&cd.cutoff[cell], w_out);
        return nx;
    }
    const int ni = ci + (face == 1) - (face == 3), nj = cj + (face == 2) - (face == 0);
    if (ni < 0 || nj < 0 || ni >= P.nx || nj >= P.ny) {
        if (!P.reflect) {
            atomicAdd(&cd.leak[cell], w_out);
            return nx;
        }
        nx.entry = face;                     // specular reflection back into the same cell
        nx.yin = 1.0f - pos;
        if (face == 0 || face == 2) nx.gy = -gy;
        else nx.gx = -gx;
    } else {
        nx.cell = (int32_t)(P.cell0 + (int64_t)nj * P.nx + ni);
        nx.entry = (face + 2) & 3;
        nx.yin = pos;
        ci = ni;
        cj = nj;
    }
    nx.alive = true;
    return nx;
}

__device__ __forceinline__ Next move_on(const CellsDev &cd, const ProblemDev &P, int cell, int face, float pos,
                                        float gx, float gy, double w_out)
{
    const uint32_t local = (uint32_t)(cell - P.cell0);
    int cj = (int)(local / (uint32_t)P.nx), ci = (int)(local - (uint32_t)cj * (uint32_t)P.nx);
    return move_on(cd, P, cell, ci, cj, face, pos, gx, gy, w_out);
}

// What a workgroup's append shares: survivors of each wave and their first index, and the
// survivors per problem in a hash table.
template <int THREADS>
struct AppendLds {
    uint32_t wave[THREADS / 64];
    unsigned long long base;
    int32_t pid[THREADS];
    uint32_t count[THREADS];
};

template <int THREADS>
__device__ __forceinline__ void append_init(AppendLds<THREADS> &al)
{
    al.pid[threadIdx.x] = -1;
    al.count[threadIdx.x] = 0;
}

// Append the alive threads' particles to `out` and count them per problem.  One atomic on the
// counter per call (a wave's own would queue up: one in 12 ns), none on the problems' counts until
// append_flush, but for problems that find neither their slot nor a free one within kTallyProbes
// probes: those count globally.  Called by all threads of the workgroup.
template <int THREADS>
__device__ __forceinline__ void append(AppendLds<THREADS> &al, bool alive, const Next &nx, int32_t pid, double w,
                                       uint32_t hist, uint32_t event, BankDev out,
                                       unsigned long long *counter, unsigned long long *pcount)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t mask = __ballot(alive);
    if (lane == 0) al.wave[wave] = (uint32_t)__popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int k = 0; k < THREADS / 64; ++k) {
            const uint32_t c = al.wave[k];
            al.wave[k] = total;
            total += c;
        }
        al.base = total ? atomicAdd(counter, (unsigned long long)total) : 0ull;
    }
    __syncthreads();
    if (alive) {
        const int64_t j = (int64_t)(al.base + al.wave[wave]) + rank_in(mask);
        out.cell[j] = nx.cell;
        out.pid[j] = pid;
        out.entry[j] = nx.entry;
        out.yin[j] = nx.yin;
        out.gx[j] = nx.gx;
        out.gy[j] = nx.gy;
        out.w[j] = w;
        out.hist[j] = hist;
        out.event[j] = event;
    }
    // one lane of each distinct problem counts for all of its survivors in the wave
    uint32_t mine = 0;
    for (uint64_t m = mask; m;) {
        const int l0 = __ffsll((unsigned long long)m) - 1;
        const int p0 = __shfl(pid, l0);
        const uint64_t same = __ballot(alive && pid == p0);
        if (lane == l0) mine = (uint32_t)__popcll(same);
        m &= ~same;
    }
    if (mine > 0) {
        uint32_t s = (uint32_t)pid % THREADS;
        int k = 0;
        for (; k < kTallyProbes; ++k) {
            const int prev = atomicCAS(&al.pid[s], -1, pid);
            if (prev == -1 || prev == pid) break;
            s = (s + 1) % THREADS;
        }
        if (k < kTallyProbes) atomicAdd(&al.count[s], mine);
        else atomicAdd(&pcount[pid], (unsigned long long)mine);
    }
    __syncthreads();       // al.wave and al.base are read before the next call writes them
}

template <int THREADS>
__device__ __forceinline__ void append_flush(AppendLds<THREADS> &al, unsigned long long *pcount)
{
    __syncthreads();
    if (al.pid[threadIdx.x] >= 0)
        atomicAdd(&pcount[al.pid[threadIdx.x]], (unsigned long long)al.count[threadIdx.x]);
}

// Volumetric births of histories [h0, h0 + count) of problem pid, first leg by the analog walk in
// the birth cell (global orientation): the source sample of history h0 + t and its walk's exit
// record at index t.  A lane group's walk, not a lane's, bounds the launch (see gmc_walk.hpp).
template <bool XY>
__global__ __launch_bounds__(256, kWalkBlocksPerCu) void birth_walk_kernel(CellsDev cd, int32_t pid, uint32_t h0, int64_t count,
                                                            int32_t *face, float *pos, float *dcos, float *dsin,
                                                            float *path)
{
    __shared__ WalkGroups groups[4];
    __shared__ uint32_t pool;
    const ProblemDev P = cd.prob[pid];
    run_walks<false, XY, false>(
        count, P.seed, groups, &pool,
        [&](int64_t t) {
            const uint32_t h = h0 + (uint32_t)t;
            const U4 r = draw4(P.seed, (uint64_t)h, 0u, kTagSource);
            const uint32_t nsrc = (uint32_t)(P.snx * P.sny);
            const uint32_t pick = __umulhi(r.a, nsrc);
            const int ci = P.sx0 + (int)(pick % (uint32_t)P.snx), cj = P.sy0 + (int)(pick / (uint32_t)P.snx);
            const int cell = (int)(P.cell0 + (int64_t)cj * P.nx + ci);
            const float ph = u01(r.d);
            // the cell's own frame [0, L / Ly] x [0, 1], lengths in units of its height Ly
            float st = 1.0f;
            if constexpr (XY) {              // isotropic on the sphere: mu from a second draw
                const U4 r2 = draw4(P.seed, (uint64_t)h, 1u, kTagSource);
                const float mu = 2.0f * u01(r2.a) - 1.0f;
                st = sqrtf(fmaxf(1.0f - mu * mu, 0.0f));
            }
            WalkStart w;
            w.wa = (float)(P.L / P.Ly);
            w.x = w.wa * u01_open(r.b);
            w.y = u01_open(r.c);
            w.u = st * cos_turns(ph);
            w.v = st * sin_turns(ph);
            w.tau = (float)(cd.tau[cell] * (P.Ly / P.L));
            w.c = cd.mat[cell].c;
            w.stream = (uint64_t)h;
            w.key = P.seed;
            return w;
        },
        [&](int64_t t, int f, float ps, float u, float v, float len, uint32_t) {
            face[t] = f;
            pos[t] = ps;
            dcos[t] = u;
            dsin[t] = v;
            path[t] = len;
        });
}

// Surface-source births of histories [h0, h0 + count): a uniformly picked cell of the source
// strip, entered through side f of the domain at a uniform canonical height with a cosine-law
// canonical direction (sin theta = 2u - 1), rotated to the global frame; no tally yet, the
// first transmission (cell visit 1) is the next transport step's.
__global__ __launch_bounds__(kTallyThreads) void surface_birth_kernel(CellsDev cd, int32_t pid, uint32_t h0,
                                                                      int64_t count, BankDev out,
                                                                      unsigned long long *counter,
                                                                      unsigned long long *pcount)
{
    __shared__ AppendLds<kTallyThreads> al;
    append_init(al);
    __syncthreads();
    const ProblemDev P = cd.prob[pid];
    for (int64_t t0 = (int64_t)blockIdx.x * kTallyThreads; t0 < count; t0 += (int64_t)gridDim.x * kTallyThreads) {
        const int64_t t = t0 + threadIdx.x;
        bool alive = false;
        Next nx{};
        uint32_t h = 0;
        if (t < count) {
            h = h0 + (uint32_t)t;
            const U4 r = draw4(P.seed, (uint64_t)h, 0u, kTagSource);
            const uint32_t nsrc = (uint32_t)(P.snx * P.sny);
            const uint32_t pick = __umulhi(r.a, nsrc);
            const int ci = P.sx0 + (int)(pick % (uint32_t)P.snx), cj = P.sy0 + (int)(pick / (uint32_t)P.snx);
            const int f = P.src_face;
            float s, cth;
            if (P.xy) {      // isotropic incident flux on the sphere: cosine sqrt(xi), azimuth psi
                const float xi = u01_open(r.c);
                cth = sqrtf(xi);
                s = sqrtf(fmaxf(1.0f - xi, 0.0f)) * cos_turns(u01(r.d));
            } else {
                s = 2.0f * u01_open(r.c) - 1.0f;
                cth = sqrtf(fmaxf(1.0f - s * s, 0.0f));
            }
            nx.cell = (int32_t)(P.cell0 + (int64_t)cj * P.nx + ci);
            nx.entry = f;
            nx.yin = u01_open(r.b);
            rot_quarter((f + 1) & 3, cth, s, nx.gx, nx.gy);
            alive = true;
        }
        append(al, alive, nx, pid, 1.0, h, 1u, out, counter, pcount);
    }
    append_flush(al, pcount);
}

// Source births for the generative internal model: birth cell, position and direction of
// histories [h0, h0 + count) (the same Philox draw as birth_walk_kernel) as internal-model
// conditions in the cell's own frame; the birth event uses random stream id h.
__global__ __launch_bounds__(256) void source_kernel(CellsDev cd, int32_t pid, uint32_t h0, int64_t count,
                                                     float *ltau, float *cc, float *xb, float *yb,
                                                     float *cosb, float *sinb, uint64_t *ids, uint64_t *keys)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const ProblemDev P = cd.prob[pid];
    const uint32_t h = h0 + (uint32_t)t;
    const U4 r = draw4(P.seed, (uint64_t)h, 0u, kTagSource);
    const uint32_t nsrc = (uint32_t)(P.snx * P.sny);
    const uint32_t pick = __umulhi(r.a, nsrc);
    const int ci = P.sx0 + (int)(pick % (uint32_t)P.snx), cj = P.sy0 + (int)(pick / (uint32_t)P.snx);
    const int cell = (int)(P.cell0 + (int64_t)cj * P.nx + ci);
    const float ph = u01(r.d);
    const CellMat m = cd.mat[cell];
    ltau[t] = m.lt;
    cc[t] = m.c;
    xb[t] = u01_open(r.b);
    yb[t] = u01_open(r.c);
    cosb[t] = cos_turns(ph);
    sinb[t] = sin_turns(ph);
    ids[t] = (uint64_t)h;
    keys[t] = P.seed;
}

// Stages 3-4 of the volumetric births (exits in the cell's own frame, which is the global
// orientation): tally, move, append.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void birth_apply_kernel(CellsDev cd, int32_t pid, uint32_t h0,
                                                                    int64_t count, const int32_t *face_c,
                                                                    const float *pos, const float *dcos,
                                                                    const float *dsin, const float *path,
                                                                    BankDev out, unsigned long long *counter,
                                                                    unsigned long long *pcount)
{
    __shared__ TallyTable<tally_slots(THREADS)> tl;
    __shared__ AppendLds<THREADS> al;
    tally_init(tl);
    append_init(al);
    __syncthreads();
    const ProblemDev P = cd.prob[pid];
    for (int64_t t0 = (int64_t)blockIdx.x * THREADS; t0 < count; t0 += (int64_t)gridDim.x * THREADS) {
        const int64_t t = t0 + threadIdx.x;
        bool alive = false;
        Next nx{};
        double w_out = 0.0;
        uint32_t h = 0;
        if (t < count) {
            h = h0 + (uint32_t)t;
            const U4 r = draw4(P.seed, (uint64_t)h, 0u, kTagSource);
            const uint32_t nsrc = (uint32_t)(P.snx * P.sny);
            const uint32_t pick = __umulhi(r.a, nsrc);
            const int ci = P.sx0 + (int)(pick % (uint32_t)P.snx), cj = P.sy0 + (int)(pick / (uint32_t)P.snx);
            const int cell = (int)(P.cell0 + (int64_t)cj * P.nx + ci);
            w_out = visit_tally(cd, cell, cd.mat[cell].siga, 1.0, path[t], P.Ly, tl);
            nx = move_on(cd, P, cell, face_c[t], pos[t], dcos[t], dsin[t], w_out);
            alive = nx.alive;
        }
        append(al, alive, nx, pid, w_out, h, 1u, out, counter, pcount);
    }
    append_flush(al, pcount);
    tally_flush(tl, cd);
}

// Where stage 1 leaves the canonical conditions of the particles to sample.
struct CondDev {
    float *ltau, *cc, *yin, *sth, *laspect, *omx;
    uint64_t *ids, *keys;
};

// Stage 1 of one particle: its canonical conditions.  Entry face e maps to the canonical left face
// by the rotation of k = (e + 1) mod 4 quarter turns (canonical -> local).
// The canonical cell takes the entry face as its height: left and right faces have length Ly,
// bottom and top length L, so entries through a vertical face see tau * Ly / L and aspect
// A = L / Ly, entries through a horizontal face tau and A = Ly / L.
struct Canonical {
    float lt, la, c, s, ox;
};

__device__ __forceinline__ Canonical canonical(const CellMat &m, float lr, int e, float gx, float gy)
{
    const int k = (e + 1) & 3;
    float U, V;
    rot_quarter((4 - k) & 3, gx, gy, U, V);
    return Canonical{(e & 1) ? m.lt + lr : m.lt, (e & 1) ? -lr : lr, m.c, fminf(fmaxf(V, -1.0f), 1.0f), U};
}

// Conditions of particle i of the bank to place j.
__device__ __forceinline__ void put_conditions(const BankDev &b, int64_t i, const CellsDev &cd, const CondDev &o,
                                               int64_t j)
{
    const ProblemDev &P = cd.prob[b.pid[i]];
    const Canonical q = canonical(cd.mat[b.cell[i]], P.lr, b.entry[i], b.gx[i], b.gy[i]);
    o.ltau[j] = q.lt;
    o.laspect[j] = q.la;
    o.omx[j] = q.ox;                     // read only in XY geometry
    o.cc[j] = q.c;
    o.yin[j] = b.yin[i];
    o.sth[j] = q.s;
    o.ids[j] = (uint64_t)b.hist[i] | ((uint64_t)b.event[i] << 32);
    o.keys[j] = P.seed;
}

// Stages 1-2 of an analog step: every alive particle's crossing by the walk, started from the bank
// and the cell's material as it is taken (the conditions of put_conditions, never written).  KEYS:
// the world holds several problems, each with its key; otherwise key `seed`.  The checkerboard's 128
// steps: 19.9 -> 18.6 ms with the gather kernel and the conditions' way through memory gone.
template <bool XY, bool KEYS>
__global__ __launch_bounds__(256, kWalkBlocksPerCu) void walk_step_kernel(BankDev b, int64_t n_arg,
                                                                          const unsigned long long *n_dev, CellsDev cd,
                                                                          float lr, uint64_t seed, int32_t *face,
                                                                          float *pos, float *dcos, float *dsin,
                                                                          float *path)
{
    __shared__ WalkGroups groups[4];
    __shared__ uint32_t pool;
    run_walks<false, XY, KEYS>(
        n_dev ? (int64_t)*n_dev : n_arg, seed, groups, &pool,
        [&](int64_t i) {
            const ProblemDev *P = KEYS ? &cd.prob[b.pid[i]] : nullptr;
            const float lri = KEYS ? P->lr : lr;
            const Canonical q = canonical(cd.mat[b.cell[i]], lri, b.entry[i], b.gx[i], b.gy[i]);
            WalkStart w;
            w.wa = q.la == 0.0f ? 1.0f : expf(q.la);
            w.x = 0.0f;
            w.y = b.yin[i];
            w.u = XY ? q.ox : sqrtf(fmaxf(1.0f - q.s * q.s, 0.0f));
            w.v = q.s;
            w.tau = expf(q.lt);
            w.c = q.c;
            w.stream = (uint64_t)b.hist[i] | ((uint64_t)b.event[i] << 32);
            w.key = KEYS ? P->seed : 0u;
            return w;
        },
        [&](int64_t i, int f, float ps, float u, float v, float len, uint32_t) {
            face[i] = f;
            pos[i] = ps;
            dcos[i] = u;
            dsin[i] = v;
            path[i] = len;
        });
}

// Stage 1: canonical conditions of every alive particle.
__global__ __launch_bounds__(256) void gather_kernel(BankDev b, int64_t n_arg, const unsigned long long *n_dev,
                                                     CellsDev cd, CondDev o)
{
    const int64_t n = n_dev ? (int64_t)*n_dev : n_arg;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) put_conditions(b, i, cd, o, i);
}

// Exit-record faces the split gather leaves for the apply stage: the particle's history ended in
// it; its crossing is collided, the exit record is the sampler's at the particle's slot.
constexpr int32_t kFaceEnded = -1000, kFaceCollided = -1001;

// Stage 1 with the first-flight split (models fitted on collided exits, blob flag bit 1).  Each
// particle draws its crossing's split (uncollided_exit, keyed by history and cell visit); while
// the crossings stay uncollided it is streamed through up to ff_max cells inside this kernel:
// stages 3-4 of each such crossing (FP64 attenuation and tallies, staged in the workgroup's LDS
// table, and the move to the neighbour) exactly as the apply stage would do them with the same
// random numbers, its bank slot then updated in place.  The crossing that ends the loop is
//   * collided: face kFaceCollided, canonical conditions compacted into the sampler's staging,
//     their place in `slot`;
//   * the ff_max-th uncollided one: its exit record written at the particle's own index, for
//     the apply stage;
//   * one that ended the history (leak, cutoff): face kFaceEnded.
// ff_max = 1 is one crossing per particle per step.  `streamed` counts the crossings finished here.
//
// How many crossings a particle streams through varies (geometric: on the lattice 16 in the mean,
// the longest of 64 lanes about 60), so lanes are not bound to particles: a workgroup takes its
// share (BlockShare) through a counter in LDS, and a wave stops for new particles when
// kStreamRefill of its lanes idle.  One workgroup per CU with a table of 4,096 cells (147 KB): what
// spills over such a table goes out as scattered FP64 atomics (0.055 ns each on the whole
// chip), which bounded the kernel with a table of 1,024 and three workgroups per CU.  A step then
// takes as long as its longest streams, 64 crossings of 1.5 us (instructions in sequence).
// Measured, 2 10^5 particles on the lattice: 549 us with one particle to a lane and the smaller
// table, 240 us; the mean over a run's 30 steps 172 -> 104 us (1,024 threads 125, 256 threads 123,
// two workgroups of half the table 139; idle lanes to refill 8 / 16 / 32 the same).
// ONE: all particles belong to problem `only`, whose description then stays in scalar registers
// (otherwise a lane holds its particle's).
constexpr int kStreamThreads = 512;
constexpr int kStreamBlocksPerCu = 1;
constexpr int kStreamRefill = 16;
using TallyStream = TallyTable<4096>;
// Largest bank of a world and most cells that a particle streams through in a step: together the
// crossings that one workgroup may count.
constexpr int64_t kMaxBank = (int64_t)1 << 31;
constexpr int kMaxStreaming = 1024;
using StreamCount = unsigned long long;
static_assert((unsigned long long)kMaxBank * kMaxStreaming <= ~(StreamCount)0, "a workgroup's count of crossings");

template <bool ONE>
__global__ __launch_bounds__(kStreamThreads) void gather_split_kernel(BankDev b, int64_t n_arg,
                                                                      const unsigned long long *n_dev, CellsDev cd,
                                                                      CondDev o, int32_t *slot,
                                                                      unsigned long long *count, int32_t *e_face,
                                                                      float *e_pos, float *e_dcos, float *e_dsin,
                                                                      float *e_path, int ff_max, int32_t only,
                                                                      unsigned long long *streamed)
{
    __shared__ TallyStream tl;
    __shared__ uint32_t pool, waves[kStreamThreads / 64];
    __shared__ StreamCount beyond;
    __shared__ unsigned long long first;
    tally_init(tl);
    if (threadIdx.x == 0) {
        pool = 0;
        beyond = 0;
    }
    __syncthreads();
    const int64_t n = n_dev ? (int64_t)*n_dev : n_arg;
    const BlockShare mine(n);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // lanes of a wave that take a particle: where there are few, every wave gets its share
    const uint32_t share = (mine.items + kStreamThreads / 64 - 1) / (kStreamThreads / 64);
    const int lanes = share < 64 ? (int)share : 64;

    bool active = false, held = false;
    int64_t i = 0;
    ProblemDev P = cd.prob[ONE ? only : 0];
    int cell = 0, ci = 0, cj = 0, e = 0;
    float gx = 0.0f, gy = 0.0f, yy = 0.0f;
    double w = 0.0;
    uint32_t ev = 0, hist = 0, passed = 0;
    StreamCount tot = 0;
    int32_t fate = 0;
    DrawPrefix q{};
    bool dry = mine.items == 0;
    for (;;) {
        if (held && !active) {               // the particle's streaming is over
            if (fate != 0) e_face[i] = fate;
            if (passed > 0 && fate != kFaceEnded) {
                b.cell[i] = cell;
                b.entry[i] = e;
                b.yin[i] = yy;
                b.gx[i] = gx;
                b.gy[i] = gy;
                b.w[i] = w;
                b.event[i] = ev;
            }
            // crossings beyond the one per particle that the step counts (a history that ended
            // here finished its step's own crossing in the loop)
            tot += fate == kFaceEnded ? passed - 1 : passed;
            held = false;
        }
        const uint64_t needs = __ballot(!active && lane < lanes);
        if (!dry) {
            const uint32_t cnt = (uint32_t)__popcll(needs);
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&pool, cnt);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
            dry = at >= mine.items || mine.items - at <= cnt;
            const uint32_t item = at + (uint32_t)rank_in(needs);
            if (!active && lane < lanes && at < mine.items && item < mine.items) {
                i = mine.index(item);
                if (i < n) {
                    if constexpr (!ONE) P = cd.prob[b.pid[i]];
                    cell = b.cell[i];
                    e = b.entry[i];
                    gx = b.gx[i];
                    gy = b.gy[i];
                    yy = b.yin[i];
                    w = b.w[i];
                    ev = b.event[i];
                    hist = b.hist[i];
                    const uint32_t local = (uint32_t)(cell - P.cell0);
                    cj = (int)(local / (uint32_t)P.nx);
                    ci = (int)(local - (uint32_t)cj * (uint32_t)P.nx);
                    q = split_prefix(hist, (uint32_t)P.seed, (uint32_t)(P.seed >> 32));
                    passed = 0;
                    active = held = true;
                }
            }
        }
        int live = __popcll(__ballot(active));
        if (live == 0) {
            if (dry) break;
            continue;
        }
        const int stop = dry ? 0 : lanes - kStreamRefill;
        for (int it = 0; live > 0 && (live > stop || it == 0); ++it) {
            if (active) {
                const CellMat m = cd.mat[cell];
                const Canonical a = canonical(m, P.lr, e, gx, gy);
                const float u = P.xy ? a.ox : sqrtf(fmaxf(1.0f - a.s * a.s, 0.0f));
                const float xi = split_draw(q, (uint32_t)P.seed, (uint32_t)(P.seed >> 32), ev);
                Exit ex;
                const float wa = P.lr == 0.0f ? 1.0f : expf(a.la);
                if (!uncollided_exit(expf(a.lt), a.c, yy, u, a.s, wa, xi, ex)) {
                    active = false;
                    fate = kFaceCollided;
                } else if (passed + 1 >= (uint32_t)ff_max) {
                    e_face[i] = ex.face;
                    e_pos[i] = ex.pos;
                    e_dcos[i] = ex.u;
                    e_dsin[i] = ex.v;
                    e_path[i] = ex.path;
                    active = false;
                    fate = 0;
                } else {
                    const int k = (e + 1) & 3;
                    const double w_out = visit_tally(cd, cell, m.siga, w, ex.path, (e & 1) ? P.Ly : P.L, tl);
                    float ngx, ngy;
                    rot_quarter(k, ex.u, ex.v, ngx, ngy);
                    const Next nx = move_on(cd, P, cell, ci, cj, (ex.face + k) & 3, ex.pos, ngx, ngy, w_out);
                    ++passed;
                    if (nx.alive && ev + 1 >= P.max_visits) {
                        atomicAdd(&cd.cutoff[cell], w_out);
                        active = false;
                    }
                    if (!nx.alive) active = false;
                    if (!active) fate = kFaceEnded;
                    cell = nx.cell;
                    e = nx.entry;
                    yy = nx.yin;
                    gx = nx.gx;
                    gy = nx.gy;
                    w = w_out;
                    ++ev;
                }
            }
            live = __popcll(__ballot(active));
        }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) tot += __shfl_xor(tot, m);
    if (lane == 0 && tot > 0) atomicAdd(&beyond, tot);
    __syncthreads();                         // also: the bank's and e_face's new values
    if (threadIdx.x == 0 && beyond > 0) atomicAdd(streamed, beyond);
    tally_flush(tl, cd);
    // the collided particles of this share to the sampler's staging, one atomic per workgroup tile
    for (uint32_t v0 = 0; v0 < mine.items; v0 += kStreamThreads) {
        const uint32_t v = v0 + threadIdx.x;
        const int64_t p = v < mine.items ? mine.index(v) : n;
        const bool take = p < n && e_face[p] == kFaceCollided;
        const uint64_t mask = __ballot(take);
        if (lane == 0) waves[wave] = (uint32_t)__popcll(mask);
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t total = 0;
            for (int k = 0; k < kStreamThreads / 64; ++k) {
                const uint32_t c = waves[k];
                waves[k] = total;
                total += c;
            }
            first = total ? atomicAdd(count, (unsigned long long)total) : 0ull;
        }
        __syncthreads();
        if (take) {
            const int64_t j = (int64_t)(first + waves[wave]) + rank_in(mask);
            put_conditions(b, p, cd, o, j);
            slot[p] = (int32_t)j;
        }
        __syncthreads();
    }
}

// Exit records of the split's collided particles, at their slots.
struct ExitDev {
    const int32_t *face;
    const float *pos, *dcos, *dsin, *path;
};

// Stages 3-4 for every alive particle, survivors compacted into `out`.  Bound by its global atomics
// (5 a cell of a workgroup's table and 2 a wave of survivors in an earlier form): 10^6 particles on
// the 32 x 32 checkerboard 409 -> 37 us, 2 10^5 on the lattice 123 -> 26 us.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void apply_kernel(BankDev in, int64_t n_arg,
                                                              const unsigned long long *n_dev,
                                                              const int32_t *face_c, const float *pos,
                                                              const float *dcos, const float *dsin,
                                                              const float *path, const int32_t *slot, ExitDev split,
                                                              CellsDev cd, BankDev out, unsigned long long *counter,
                                                              unsigned long long *pcount)
{
    __shared__ TallyTable<tally_slots(THREADS)> tl;
    __shared__ AppendLds<THREADS> al;
    tally_init(tl);
    append_init(al);
    __syncthreads();
    const int64_t n = n_dev ? (int64_t)*n_dev : n_arg;
    for (int64_t i0 = (int64_t)blockIdx.x * THREADS; i0 < n; i0 += (int64_t)gridDim.x * THREADS) {
        const int64_t i = i0 + threadIdx.x;
        bool alive = false;
        Next nx{};
        double w_out = 0.0;
        int32_t pid = 0;
        uint32_t hist = 0, event = 0;
        int fc = i < n ? face_c[i] : kFaceEnded;
        if (fc != kFaceEnded) {
            float ps, dc, ds, pl;
            if (fc == kFaceCollided) {       // the sampler's exit of the particle's slot
                const int64_t j = slot[i];
                fc = split.face[j];
                ps = split.pos[j];
                dc = split.dcos[j];
                ds = split.dsin[j];
                pl = split.path[j];
            } else {
                ps = pos[i];
                dc = dcos[i];
                ds = dsin[i];
                pl = path[i];
            }
            pid = in.pid[i];
            const ProblemDev P = cd.prob[pid];
            const int cell = in.cell[i];
            const int k = (in.entry[i] + 1) & 3;
            hist = in.hist[i];
            event = in.event[i] + 1;
            w_out = visit_tally(cd, cell, cd.mat[cell].siga, in.w[i], pl, (in.entry[i] & 1) ? P.Ly : P.L, tl);
            float gx, gy;
            rot_quarter(k, dc, ds, gx, gy);
            nx = move_on(cd, P, cell, fc >= 0 ? (fc + k) & 3 : fc, ps, gx, gy, w_out);
            if (nx.alive && event >= P.max_visits) {
                atomicAdd(&cd.cutoff[cell], w_out);
                nx.alive = false;
            }
            alive = nx.alive;
        }
        append(al, alive, nx, pid, w_out, hist, event, out, counter, pcount);
    }
    append_flush(al, pcount);
    tally_flush(tl, cd);
}

// Ends a step or an injection: the bank's counters and the streamed crossings to the host's pinned
// copy (a store over the bus; the stream's end makes it visible), the other bank's counters and the
// split's count cleared for the next step.  One kernel of 3 us in the place of two that cleared and
// two copies; a thread a counter (a step of 1,000 particles in a world of 16,384 / 65,536 problem
// slots 44 / 95 us, with one workgroup for all of them 53 / 123).
__global__ __launch_bounds__(256) void finish_kernel(const unsigned long long *ctr, unsigned long long *other,
                                                     unsigned long long *split_count,
                                                     const unsigned long long *streamed, unsigned long long *host, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        host[i] = ctr[i];
        other[i] = 0ull;
    }
    if (i == 0) {
        host[n] = *streamed;
        *split_count = 0ull;
    }
}

// After a step or injection that failed part way: the counters as its successor expects them, of
// the particles alive before it (in all and per problem).
__global__ __launch_bounds__(256) void reset_kernel(const unsigned long long *alive, unsigned long long *ctr,
                                                    unsigned long long *other, unsigned long long *split_count, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) {
        ctr[i] = alive[i];
        other[i] = 0ull;
    }
    if (i == 0) *split_count = 0ull;
}

// Materials of cells [cell0, cell0 + n) of width L: tau is in place, c and ln tau were uploaded to the
// cells' own places for cutoff and leak tallies (cleared afterwards).
__global__ __launch_bounds__(256) void materials_kernel(CellsDev cd, CellMat *mat, int64_t cell0, int64_t n, double L)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double c = cd.cutoff[cell0 + i];
    mat[cell0 + i] = CellMat{((const float *)(cd.leak + cell0))[i], (float)c, (1.0 - c) * cd.tau[cell0 + i] / L};
}

// Clears the tallies of cells [cell0, cell0 + n).
__global__ void zero_tallies_kernel(CellsDev cd, int64_t cell0, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int k = 0; k < kVisitTallies; ++k) cd.visit[(cell0 + i) * kVisitTallies + k] = 0.0;
    cd.leak[cell0 + i] = 0.0;
    cd.cutoff[cell0 + i] = 0.0;
    cd.rej_w[cell0 + i] = 0.0;
    cd.rej_n[cell0 + i] = 0.0;
}

// The tallies as the host reads them, a column per quantity.
enum class Column : int8_t { Flux, Absorbed, Leak, Cutoff, WeightPath, Path, Visits, RejectedW, RejectedN };
struct Columns {
    int count = 0;
    Column col[5];
};

// Columns of cells [cell0, cell0 + n), of volume V each, one after another to `out`.  The flux is the
// deposit over V sigma_a, or the sum of w l over V without absorption (eq. 7).
__global__ __launch_bounds__(256) void columns_kernel(CellsDev cd, int64_t cell0, int64_t n, double V, Columns q,
                                                      double *out)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t cell = cell0 + i;
    const double *t = cd.visit + cell * kVisitTallies;
    for (int k = 0; k < q.count; ++k) {
        double v = 0.0;
        switch (q.col[k]) {
        case Column::Flux: {
            const double sa = cd.mat[cell].siga;
            v = sa > 0.0 ? t[0] / (V * sa) : t[1] / V;
            break;
        }
        case Column::Absorbed: v = t[0]; break;
        case Column::WeightPath: v = t[1]; break;
        case Column::Path: v = t[2]; break;
        case Column::Visits: v = t[3]; break;
        case Column::Leak: v = cd.leak[cell]; break;
        case Column::Cutoff: v = cd.cutoff[cell]; break;
        case Column::RejectedW: v = cd.rej_w[cell]; break;
        case Column::RejectedN: v = cd.rej_n[cell]; break;
        }
        out[k * n + i] = v;
    }
}

int blocks_for(int64_t n) { return (int)((n + 255) / 256); }

// Whether a launch over n particles on a device of cu compute units takes small workgroups: with
// at most 128 particles to a compute unit.  A large one clears and looks through 147 KB for its few
// particles and adds 1,024 of them to the source's few cells one after another.  Births of 300 / 4,000 /
// 16,000 histories on the lattice, large -> small: 27.8 -> 26.3 / 30.6 -> 28.0 / 32.7 -> 30.5 us, in a
// source of one cell 29.3 -> 27.6 / 35.7 -> 29.4 / 37.2 -> 31.2; 33,000 on the lattice the same with
// both, 65,536 34 against 39.
bool small_tally(int64_t n, int cu) { return n <= (int64_t)128 * cu; }

// Its grid.
int tally_blocks(int64_t n, int cu)
{
    if (small_tally(n, cu)) return (int)((n + kSmallTallyThreads - 1) / kSmallTallyThreads);
    return (int)std::min<int64_t>((n + kTallyThreads - 1) / kTallyThreads, (int64_t)cu);
}

}  // namespace
}  // namespace gmc

using namespace gmc;

struct gmc_world {
    int device = 0;
    int64_t cap = 0;
    int32_t max_problems = 0;
    int64_t max_cells = 0;
    void *mem = nullptr;
    BankDev bank[2]{};
    int cur = 0;
    int integrator = GMC_EULER;   // ODE integrator of the generative sampler
    const gmc_model *src_model = nullptr;   // internal model for births (else analog first leg)
    int src_K = 16;
    // sampler staging
    float *c_ltau = nullptr, *c_c = nullptr, *c_yin = nullptr, *c_sth = nullptr;
    float *c_x = nullptr, *c_cos = nullptr;      // internal-model births
    float *c_la = nullptr;                       // canonical ln aspect (rectangular cells)
    float *c_ox = nullptr;                       // canonical in-plane x direction (XY geometry)
    // first-flight split: place of each collided particle among the compacted ones, their exits, count
    int32_t *s_slot = nullptr, *s_face = nullptr;
    float *s_pos = nullptr, *s_dcos = nullptr, *s_dsin = nullptr, *s_path = nullptr;
    unsigned long long *s_count = nullptr;
    unsigned long long *n_large = nullptr;       // sampler's device-side tile choice (two count handoffs)
    unsigned long long *streamed = nullptr;      // crossings finished inside split gathers
    int ff_max = 64;                             // cells a particle may stream through per step
    int64_t stepped = 0;                         // particles stepped (one crossing each)
    uint64_t *ids = nullptr, *keys = nullptr;
    int32_t *e_face = nullptr;
    float *e_pos = nullptr, *e_dcos = nullptr, *e_dsin = nullptr, *e_path = nullptr;
    // cells and tallies
    double *tau = nullptr;
    CellMat *mat = nullptr;
    double *visit = nullptr, *leak = nullptr, *cutoff = nullptr, *rej_w = nullptr, *rej_n = nullptr;
    ProblemDev *prob = nullptr;
    unsigned long long *counters = nullptr;   // [2][1 + max_problems]: n_alive, per-problem
    unsigned long long *host_counters = nullptr;
    double *host_columns = nullptr;           // host_doubles of pinned memory, after the counters
    // captured transport steps, one per (sampler, model, K, integrator, bank parity, bucket)
    struct StepGraph {
        int sampler, K, integrator, cur, ff, xy;
        uint64_t model;        // serial of the model (0 for the analog walk)
        int64_t bucket;
        hipGraph_t graph;
        hipGraphExec_t exec;
    };
    bool graphs = false;
    hipStream_t capture_stream = nullptr;
    std::vector<StepGraph> step_graphs;
    // host bookkeeping
    int64_t n_alive = 0;
    bool broken = false;                      // the last step or injection failed part way
    std::vector<int64_t> alive_pp;
    std::vector<ProblemDev> prob_host;
    std::vector<char> in_use;
    int32_t problems = 0, only = -1;    // problems held; the one held, -1 if not exactly one
    std::vector<int32_t> src_face;      // per problem slot: -1 volumetric, else a surface side
    std::vector<char> rect;             // per problem slot: non-square cells
    std::vector<char> xyg;              // per problem slot: XY geometry
    std::vector<std::pair<int64_t, int64_t>> free_cells;   // [begin, end) ranges
    std::mutex mu;

    unsigned long long *cnt(int which) { return counters + (size_t)which * (1 + max_problems); }
    CellsDev cells() const { return CellsDev{tau, mat, visit, leak, cutoff, rej_w, rej_n, prob}; }
};

namespace {

// Doubles of a world's pinned memory (at most 4 MB; five columns of its cells if that is less) through
// which tallies are read: the kernel that forms their columns stores them there, a part of the
// cells at a time, and the host copies them on.
// Four columns / one of 112^2 cells 33 / 18 us, 362^2 195 / 57 us, 3000^2 16.2 / 4.3 ms; by a copy of
// each column from an array of its own on the device 52 / 14 us, 203 / 53 us, 16.1 / 4.0 ms; by a copy
// of the cells' four tallies, taken apart on the host, 63 / 36 us, 484 / 349 us, 93 / 81 ms.
int64_t host_doubles(int64_t max_cells) { return std::min<int64_t>((int64_t)1 << 19, 5 * max_cells); }

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Byte layout of one world allocation (also used to report the footprint).
struct Layout {
    size_t total = 0;
    std::vector<std::pair<void **, size_t>> parts;
    void add(void **p, size_t bytes) { parts.push_back({p, total}); total += align256(bytes); }
};

void plan(gmc_world *w, Layout &L)
{
    const size_t C = (size_t)w->cap, P = (size_t)w->max_problems, N = (size_t)w->max_cells;
    for (int b = 0; b < 2; ++b) {
        BankDev &k = w->bank[b];
        L.add((void **)&k.cell, 4 * C);
        L.add((void **)&k.pid, 4 * C);
        L.add((void **)&k.entry, 4 * C);
        L.add((void **)&k.yin, 4 * C);
        L.add((void **)&k.gx, 4 * C);
        L.add((void **)&k.gy, 4 * C);
        L.add((void **)&k.w, 8 * C);
        L.add((void **)&k.hist, 4 * C);
        L.add((void **)&k.event, 4 * C);
    }
    L.add((void **)&w->c_ltau, 4 * C);
    L.add((void **)&w->c_c, 4 * C);
    L.add((void **)&w->c_yin, 4 * C);
    L.add((void **)&w->c_sth, 4 * C);
    L.add((void **)&w->c_x, 4 * C);
    L.add((void **)&w->c_la, 4 * C);
    L.add((void **)&w->c_ox, 4 * C);
    L.add((void **)&w->s_slot, 4 * C);
    L.add((void **)&w->s_face, 4 * C);
    L.add((void **)&w->s_pos, 4 * C);
    L.add((void **)&w->s_dcos, 4 * C);
    L.add((void **)&w->s_dsin, 4 * C);
    L.add((void **)&w->s_path, 4 * C);
    L.add((void **)&w->c_cos, 4 * C);
    L.add((void **)&w->ids, 8 * C);
    L.add((void **)&w->keys, 8 * C);
    L.add((void **)&w->e_face, 4 * C);
    L.add((void **)&w->e_pos, 4 * C);
    L.add((void **)&w->e_dcos, 4 * C);
    L.add((void **)&w->e_dsin, 4 * C);
    L.add((void **)&w->e_path, 4 * C);
    L.add((void **)&w->tau, 8 * N);
    L.add((void **)&w->mat, sizeof(CellMat) * N);
    L.add((void **)&w->visit, 8 * kVisitTallies * N);
    L.add((void **)&w->leak, 8 * N);
    L.add((void **)&w->cutoff, 8 * N);
    L.add((void **)&w->rej_w, 8 * N);
    L.add((void **)&w->rej_n, 8 * N);
    L.add((void **)&w->prob, sizeof(ProblemDev) * P);
    // cleared together when the world is made
    L.add((void **)&w->s_count, 8);
    L.add((void **)&w->streamed, 8);
    L.add((void **)&w->n_large, 16);
    L.add((void **)&w->counters, 8 * 2 * (1 + P));
}

// Enqueue the end of a step or injection that left the particles in bank `which`.
hipError_t enqueue_finish(gmc_world *w, int which, hipStream_t s)
{
    const int n = 1 + w->max_problems;
    hipLaunchKernelGGL(finish_kernel, dim3(blocks_for(n)), dim3(256), 0, s, w->cnt(which), w->cnt(1 - which),
                       w->s_count, w->streamed, w->host_counters, n);
    return hipGetLastError();
}

// Before a step or injection: the counters put right if the last one failed (its kernels no longer
// run, see failed_call, so the host's copy of the counters is free).  Until sync_counters has run,
// this one counts as failed.
hipError_t begin_counters(gmc_world *w, hipStream_t s)
{
    const bool was = w->broken;
    w->broken = true;
    if (!was) return hipSuccess;
    w->host_counters[0] = (unsigned long long)w->n_alive;
    for (int p = 0; p < w->max_problems; ++p) w->host_counters[1 + p] = (unsigned long long)w->alive_pp[p];
    const int n = 1 + w->max_problems;
    hipLaunchKernelGGL(reset_kernel, dim3(blocks_for(n)), dim3(256), 0, s, w->host_counters, w->cnt(w->cur),
                       w->cnt(1 - w->cur), w->s_count, n);
    return hipGetLastError();
}

// Ends a step or injection that failed after begin_counters: waits for what it had enqueued, and
// leaves no error behind for the next call to find.  The bank, the counts and the number of steps
// stay as they were before it; tallies its kernels made stand.
int failed_call(hipStream_t s, int rc)
{
    (void)hipStreamSynchronize(s);
    (void)hipGetLastError();
    return rc;
}

// Wait for it and take its counts over.
int sync_counters(gmc_world *w, hipStream_t s)
{
    const hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return set_hip_error(e, "transport: reading counters");
    w->broken = false;
    w->n_alive = (int64_t)w->host_counters[0];
    for (int p = 0; p < w->max_problems; ++p) w->alive_pp[p] = (int64_t)w->host_counters[1 + p];
    return GMC_OK;
}

}  // namespace

extern "C" {

int gmc_world_footprint(int64_t bank_capacity, int32_t max_problems, int64_t max_cells, size_t *bytes)
{
    if (!bytes || bank_capacity <= 0 || max_problems <= 0 || max_cells <= 0)
        return set_error(GMC_EINVAL, "gmc_world_footprint: bad argument");
    gmc_world w;
    w.cap = bank_capacity;
    w.max_problems = max_problems;
    w.max_cells = max_cells;
    Layout L;
    plan(&w, L);
    *bytes = L.total;
    return GMC_OK;
}

int gmc_world_create(int64_t bank_capacity, int32_t max_problems, int64_t max_cells, gmc_world **out)
{
    if (!out) return set_error(GMC_EINVAL, "gmc_world_create: null output");
    *out = nullptr;
    if (bank_capacity <= 0 || bank_capacity > kMaxBank || max_problems <= 0 ||
        max_problems > 65536 || max_cells <= 0 || max_cells > ((int64_t)1 << 31))
        return set_error(GMC_EINVAL, "gmc_world_create: capacity out of range");
    const int irc = gmc_device_init();
    if (irc != GMC_OK) return irc;
    gmc_world *w = new gmc_world();
    w->cap = bank_capacity;
    w->max_problems = max_problems;
    w->max_cells = max_cells;
    Layout L;
    plan(w, L);
    hipError_t e = hipGetDevice(&w->device);
    if (e != hipSuccess) { delete w; return set_hip_error(e, "gmc_world_create: hipGetDevice"); }
    e = hipMalloc(&w->mem, L.total);
    if (e != hipSuccess) { delete w; return set_error(GMC_ENOMEM, "gmc_world_create: device allocation failed"); }
    for (auto &pr : L.parts) *pr.first = (char *)w->mem + pr.second;
    e = hipHostMalloc((void **)&w->host_counters, 8 * ((size_t)(2 + max_problems) + host_doubles(max_cells)),
                      hipHostMallocDefault);
    if (e != hipSuccess) {
        (void)hipFree(w->mem);
        delete w;
        return set_error(GMC_ENOMEM, "gmc_world_create: pinned host allocation failed");
    }
    std::memset(w->host_counters, 0, 8 * (size_t)(2 + max_problems));
    w->host_columns = (double *)(w->host_counters + 2 + max_problems);
    e = hipMemset(w->s_count, 0, (size_t)((char *)w->mem + L.total - (char *)w->s_count));
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        (void)hipHostFree(w->host_counters);
        (void)hipFree(w->mem);
        delete w;
        return set_hip_error(e, "gmc_world_create: clearing counters");
    }
    w->alive_pp.assign(max_problems, 0);
    w->prob_host.assign(max_problems, ProblemDev{});
    w->in_use.assign(max_problems, 0);
    w->src_face.assign(max_problems, -1);
    w->rect.assign(max_problems, 0);
    w->xyg.assign(max_problems, 0);
    w->free_cells.push_back({0, max_cells});
    *out = w;
    return GMC_OK;
}

int gmc_world_destroy(gmc_world *w)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_world_destroy: null world");
    hipError_t e1 = hipSuccess, e2 = hipSuccess;
    for (auto &g : w->step_graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    if (w->capture_stream) (void)hipStreamDestroy(w->capture_stream);
    if (w->host_counters) e1 = hipHostFree(w->host_counters);
    if (w->mem) e2 = hipFree(w->mem);
    delete w;
    if (e1 != hipSuccess) return set_hip_error(e1, "gmc_world_destroy");
    if (e2 != hipSuccess) return set_hip_error(e2, "gmc_world_destroy");
    return GMC_OK;
}

int gmc_problem_add(gmc_world *w, const gmc_problem_desc *d, int32_t *pid_out, void *stream)
{
    if (!w || !d || !pid_out) return set_error(GMC_EINVAL, "gmc_problem_add: null pointer");
    if (d->nx <= 0 || d->ny <= 0 || !(d->L > 0.0) || !d->tau || !d->c)
        return set_error(GMC_EINVAL, "gmc_problem_add: bad grid or materials");
    if (d->src_nx <= 0 || d->src_ny <= 0 || d->src_x0 < 0 || d->src_y0 < 0 ||
        d->src_x0 + d->src_nx > d->nx || d->src_y0 + d->src_ny > d->ny)
        return set_error(GMC_EINVAL, "gmc_problem_add: source block outside the grid");
    if (!(d->Ly >= 0.0) || !std::isfinite(d->Ly))
        return set_error(GMC_EINVAL, "gmc_problem_add: Ly must be 0 (square cells) or positive");
    const double Ly = d->Ly > 0.0 ? d->Ly : d->L;
    if (d->xy != 0 && d->xy != 1)
        return set_error(GMC_EINVAL, "gmc_problem_add: xy must be 0 (flatland) or 1 (XY geometry)");
    if (d->max_visits != 0 && (d->max_visits < 2 || d->max_visits > ((int64_t)1 << 31)))
        return set_error(GMC_EINVAL, "gmc_problem_add: max_visits must be 0 (2^24) or in 2..2^31");
    if (d->src_face < -1 || d->src_face > 3)
        return set_error(GMC_EINVAL, "gmc_problem_add: src_face must be -1 (volumetric) or a side 0..3");
    if (d->src_face >= 0) {
        const int f = d->src_face;
        const bool strip = (f == 3) ? (d->src_x0 == 0 && d->src_nx == 1)
                         : (f == 1) ? (d->src_x0 == d->nx - 1 && d->src_nx == 1)
                         : (f == 0) ? (d->src_y0 == 0 && d->src_ny == 1)
                                    : (d->src_y0 == d->ny - 1 && d->src_ny == 1);
        if (!strip || d->reflect)
            return set_error(GMC_EINVAL, "gmc_problem_add: a surface source needs a one-cell strip "
                                         "along its side of the domain and vacuum boundaries");
    }
    const int64_t n = (int64_t)d->nx * d->ny;
    for (int64_t i = 0; i < n; ++i)
        if (!(d->tau[i] >= 0.0) || !std::isfinite(d->tau[i]) || !(d->c[i] >= 0.0) || !(d->c[i] <= 1.0))
            return set_error(GMC_EINVAL, "gmc_problem_add: tau must be finite >= 0 and c in [0, 1]");
    std::lock_guard<std::mutex> lk(w->mu);
    for (int q = 0; q < w->max_problems; ++q)
        if (w->in_use[q] && w->xyg[q] != (d->xy ? 1 : 0))
            return set_error(GMC_EINVAL, "gmc_problem_add: the world's problems share one geometry (flatland or XY)");
    int pid = -1;
    for (int p = 0; p < w->max_problems; ++p)
        if (!w->in_use[p]) { pid = p; break; }
    if (pid < 0) return set_error(GMC_ENOMEM, "gmc_problem_add: no free problem slot");
    std::vector<float> lt;
    try {
        lt.resize(n);
    } catch (const std::bad_alloc &) {
        return set_error(GMC_ENOMEM, "gmc_problem_add: host staging");
    }
    for (int64_t i = 0; i < n; ++i) lt[i] = d->tau[i] > 0.0 ? (float)std::log(d->tau[i]) : -1.0e4f;
    int64_t cell0 = -1;
    for (auto &r : w->free_cells)
        if (r.second - r.first >= n) {
            cell0 = r.first;
            r.first += n;
            break;
        }
    if (cell0 < 0) return set_error(GMC_ENOMEM, "gmc_problem_add: no room for the cells");
    w->free_cells.erase(std::remove_if(w->free_cells.begin(), w->free_cells.end(),
                                       [](const std::pair<int64_t, int64_t> &r) { return r.first >= r.second; }),
                        w->free_cells.end());
    const uint32_t max_visits = d->max_visits == 0 ? (1u << 24) : (uint32_t)d->max_visits;
    ProblemDev P{d->nx, d->ny, d->L, Ly, (float)std::log(Ly / d->L), cell0, d->src_x0, d->src_y0,
                 d->src_nx, d->src_ny, d->reflect ? 1 : 0, d->w_min, d->seed, d->src_face, d->xy ? 1 : 0,
                 max_visits};
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(w->tau + cell0, d->tau, 8 * n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(w->cutoff + cell0, d->c, 8 * n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(w->leak + cell0, lt.data(), 4 * n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(w->prob + pid, &P, sizeof P, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(materials_kernel, dim3(blocks_for(n)), dim3(256), 0, s, w->cells(), w->mat, cell0, n, d->L);
        hipLaunchKernelGGL(zero_tallies_kernel, dim3(blocks_for(n)), dim3(256), 0, s, w->cells(), cell0, n);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);      // the host staging vector goes away
    if (e != hipSuccess) {
        w->free_cells.push_back({cell0, cell0 + n});
        return set_hip_error(e, "gmc_problem_add: upload");
    }
    w->in_use[pid] = 1;
    w->only = ++w->problems == 1 ? pid : -1;
    w->src_face[pid] = d->src_face;
    w->rect[pid] = Ly != d->L;
    w->xyg[pid] = d->xy ? 1 : 0;
    w->prob_host[pid] = P;
    w->alive_pp[pid] = 0;
    *pid_out = pid;
    return GMC_OK;
}

int gmc_problem_remove(gmc_world *w, int32_t pid)
{
    if (!w || pid < 0 || pid >= (w ? w->max_problems : 0) || !w->in_use[pid])
        return set_error(GMC_EINVAL, "gmc_problem_remove: no such problem");
    std::lock_guard<std::mutex> lk(w->mu);
    if (w->alive_pp[pid] != 0)
        return set_error(GMC_EINVAL, "gmc_problem_remove: the problem still has particles in flight");
    const ProblemDev &P = w->prob_host[pid];
    w->free_cells.push_back({P.cell0, P.cell0 + (int64_t)P.nx * P.ny});
    std::sort(w->free_cells.begin(), w->free_cells.end());
    std::vector<std::pair<int64_t, int64_t>> merged;
    for (auto &r : w->free_cells) {
        if (!merged.empty() && merged.back().second >= r.first) merged.back().second = std::max(merged.back().second, r.second);
        else merged.push_back(r);
    }
    w->free_cells.swap(merged);
    w->in_use[pid] = 0;
    w->only = --w->problems == 1 ? (int32_t)(std::find(w->in_use.begin(), w->in_use.end(), 1) - w->in_use.begin()) : -1;
    w->rect[pid] = 0;
    w->xyg[pid] = 0;
    return GMC_OK;
}

int gmc_world_inject(gmc_world *w, int32_t pid, uint64_t h_begin, int64_t count, void *stream,
                     int64_t *n_alive_out)
{
    if (!w || pid < 0 || pid >= w->max_problems || !w->in_use[pid])
        return set_error(GMC_EINVAL, "gmc_world_inject: no such problem");
    if (count < 0 || h_begin + (uint64_t)count > ((uint64_t)1 << 32))
        return set_error(GMC_EINVAL, "gmc_world_inject: history ids must stay below 2^32");
    if (count > w->cap - w->n_alive)
        return set_error(GMC_ENOMEM, "gmc_world_inject: not enough free bank slots");
    if (w->src_face[pid] < 0 && w->src_model && (w->rect[pid] || w->xyg[pid]))
        return set_error(GMC_EINVAL, "gmc_world_inject: the internal model serves flatland square cells only");
    hipStream_t s = (hipStream_t)stream;
    if (count > 0) {
        const int cu = device_cu_count();
        if (cu <= 0) return set_error(GMC_EDEVICE, "gmc_world_inject: cannot query the device");
        const int which = w->cur;
        unsigned long long *ctr = w->cnt(which);
        // the bank's counters stand at the particles alive, in all and per problem, and continue
        const hipError_t eb = begin_counters(w, s);
        if (eb != hipSuccess) return failed_call(s, set_hip_error(eb, "gmc_world_inject: launch"));
        if (w->src_face[pid] >= 0) {
            hipLaunchKernelGGL(surface_birth_kernel, dim3((unsigned)std::min<int64_t>((count + kTallyThreads - 1) / kTallyThreads, cu)),
                               dim3(kTallyThreads), 0, s, w->cells(),
                               pid, (uint32_t)h_begin, count, w->bank[which], ctr, ctr + 1);
        } else if (!w->src_model) {
            const dim3 grid(walk_grid(count, cu));
            if (w->xyg[pid])
                hipLaunchKernelGGL(birth_walk_kernel<true>, grid, dim3(256), 0, s, w->cells(), pid, (uint32_t)h_begin,
                                   count, w->e_face, w->e_pos, w->e_dcos, w->e_dsin, w->e_path);
            else
                hipLaunchKernelGGL(birth_walk_kernel<false>, grid, dim3(256), 0, s, w->cells(), pid, (uint32_t)h_begin,
                                   count, w->e_face, w->e_pos, w->e_dcos, w->e_dsin, w->e_path);
        } else {
            hipLaunchKernelGGL(source_kernel, dim3(blocks_for(count)), dim3(256), 0, s, w->cells(), pid,
                               (uint32_t)h_begin, count, w->c_ltau, w->c_c, w->c_x, w->c_yin, w->c_cos,
                               w->c_sth, w->ids, w->keys);
            const gmc_model *m = w->src_model;
            MlpParams p = m->tmpl;
            p.log_tau = w->c_ltau;
            p.c = w->c_c;
            p.x_in = w->c_x;
            p.y_in = w->c_yin;
            p.cos_phi = w->c_cos;
            p.sin_th = w->c_sth;
            p.noise = nullptr;
            p.raw = nullptr;
            p.ids = w->ids;
            p.keys = w->keys;
            p.face = w->e_face;
            p.pos = w->e_pos;
            p.dcos = w->e_dcos;
            p.dsin = w->e_dsin;
            p.path = w->e_path;
            p.n = count;
            p.n_dev = nullptr;
            p.K = w->src_K;
            p.integrator = w->integrator;
            p.seed = 0;
            p.id_base = 0;
            hipError_t e = launch_mlp_ode(m->precision, m->hidden, p, cu, s);
            if (e != hipSuccess) return failed_call(s, set_hip_error(e, "gmc_world_inject: internal sampler"));
        }
        if (w->src_face[pid] < 0) {
            const bool small = small_tally(count, cu);
            auto *kernel = small ? birth_apply_kernel<kSmallTallyThreads> : birth_apply_kernel<kTallyThreads>;
            hipLaunchKernelGGL(kernel, dim3(tally_blocks(count, cu)), dim3(small ? kSmallTallyThreads : kTallyThreads), 0,
                               s, w->cells(), pid, (uint32_t)h_begin, count, w->e_face, w->e_pos, w->e_dcos, w->e_dsin,
                               w->e_path, w->bank[which], ctr, ctr + 1);
        }
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = enqueue_finish(w, which, s);
        if (e != hipSuccess) return failed_call(s, set_hip_error(e, "gmc_world_inject: launch"));
        const int rc = sync_counters(w, s);
        if (rc != GMC_OK) return failed_call(s, rc);
    }
    if (n_alive_out) *n_alive_out = w->n_alive;
    return GMC_OK;
}

int gmc_world_set_source_model(gmc_world *w, const gmc_model *m, int K)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_world_set_source_model: null world");
    if (m && (m->n_in != 12 || K < 1 || K > 1024))
        return set_error(GMC_EINVAL, "gmc_world_set_source_model: needs an internal model (12 inputs) and K in 1..1024");
    std::lock_guard<std::mutex> lk(w->mu);
    w->src_model = m;
    w->src_K = K;
    return GMC_OK;
}

int gmc_world_set_integrator(gmc_world *w, int integrator)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_world_set_integrator: null world");
    if (integrator != GMC_EULER && integrator != GMC_RK4)
        return set_error(GMC_EINVAL, "gmc_world_set_integrator: integrator must be GMC_EULER or GMC_RK4");
    std::lock_guard<std::mutex> lk(w->mu);
    w->integrator = integrator;
    return GMC_OK;
}

int gmc_world_set_streaming(gmc_world *w, int max_crossings)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_world_set_streaming: null world");
    if (max_crossings < 1 || max_crossings > kMaxStreaming)
        return set_error(GMC_EINVAL, "gmc_world_set_streaming: max_crossings must be in 1..1024");
    std::lock_guard<std::mutex> lk(w->mu);
    w->ff_max = max_crossings;
    return GMC_OK;
}

int gmc_world_transmissions(const gmc_world *w, int64_t *count)
{
    if (!w || !count) return set_error(GMC_EINVAL, "gmc_world_transmissions: null argument");
    *count = w->stepped + (int64_t)w->host_counters[1 + w->max_problems];
    return GMC_OK;
}

int gmc_world_set_graphs(gmc_world *w, int enable)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_world_set_graphs: null world");
    std::lock_guard<std::mutex> lk(w->mu);
    if (enable && !w->capture_stream) {
        hipError_t e = hipStreamCreateWithFlags(&w->capture_stream, hipStreamNonBlocking);
        if (e != hipSuccess) {
            w->capture_stream = nullptr;
            return set_hip_error(e, "gmc_world_set_graphs: capture stream");
        }
    }
    w->graphs = enable != 0;
    return GMC_OK;
}

namespace {

// XY geometry of the world's problems (they all share one geometry)
bool world_xy(const gmc_world *w)
{
    for (int p = 0; p < w->max_problems; ++p)
        if (w->in_use[p] && w->xyg[p]) return true;
    return false;
}

// Enqueue one transport step on `s`: gather, sampler, apply, counters to the host.  Grids are sized for
// `n_launch` particles; the kernels process n_dev[0] of them when n_dev is given (a captured step
// serves every count up to its bucket), else n_launch.
int enqueue_step(gmc_world *w, int sampler, const gmc_model *m, int K, hipStream_t s, int64_t n_launch,
                 const unsigned long long *n_dev)
{
    const int cur = w->cur, nxt = 1 - cur;
    const bool split = sampler == GMC_SAMPLER_GMC && m->collided;
    const int cu = device_cu_count();
    if (cu <= 0) return set_error(GMC_EDEVICE, "gmc_transport_step: cannot query the device");
    const CondDev o{w->c_ltau, w->c_c, w->c_yin, w->c_sth, w->c_la, w->c_ox, w->ids, w->keys};
    if (split) {
        const dim3 grid((unsigned)std::min<int64_t>((n_launch + 63) / 64, (int64_t)cu * kStreamBlocksPerCu));
        const int32_t only = w->graphs ? -1 : w->only;
        if (only >= 0)
            hipLaunchKernelGGL(gather_split_kernel<true>, grid, dim3(kStreamThreads), 0, s, w->bank[cur], n_launch,
                               n_dev, w->cells(), o, w->s_slot, w->s_count, w->e_face, w->e_pos, w->e_dcos, w->e_dsin,
                               w->e_path, w->ff_max, only, w->streamed);
        else
            hipLaunchKernelGGL(gather_split_kernel<false>, grid, dim3(kStreamThreads), 0, s, w->bank[cur], n_launch,
                               n_dev, w->cells(), o, w->s_slot, w->s_count, w->e_face, w->e_pos, w->e_dcos, w->e_dsin,
                               w->e_path, w->ff_max, only, w->streamed);
    } else if (sampler == GMC_SAMPLER_GMC) {
        hipLaunchKernelGGL(gather_kernel, dim3(blocks_for(n_launch)), dim3(256), 0, s, w->bank[cur], n_launch,
                           n_dev, w->cells(), o);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_hip_error(e, "gmc_transport_step: gather");
    if (sampler == GMC_SAMPLER_GMC) {
        MlpParams p = m->tmpl;
        p.log_tau = w->c_ltau;
        p.c = w->c_c;
        p.y_in = w->c_yin;
        p.sin_th = w->c_sth;
        p.log_aspect = (m->n_in == 11 && !m->xy) ? w->c_la : nullptr;
        p.omega_x = m->xy ? w->c_ox : nullptr;
        p.noise = nullptr;
        p.raw = nullptr;
        p.ids = w->ids;
        p.keys = w->keys;
        p.face = split ? w->s_face : w->e_face;
        p.pos = split ? w->s_pos : w->e_pos;
        p.dcos = split ? w->s_dcos : w->e_dcos;
        p.dsin = split ? w->s_dsin : w->e_dsin;
        p.path = split ? w->s_path : w->e_path;
        p.n = n_launch;
        p.n_dev = split ? w->s_count : n_dev;
        p.n_dev_large = p.n_dev ? w->n_large : nullptr;
        p.K = K;
        p.integrator = w->integrator;
        p.seed = 0;
        p.id_base = 0;
        e = launch_mlp_ode(m->precision, m->hidden, p, cu, s);
    } else {
        // one problem alone: its key and shape are the launch's (a captured step serves any set of
        // problems)
        const int32_t only = w->graphs ? -1 : w->only;
        const float lr = only >= 0 ? w->prob_host[only].lr : 0.0f;
        const uint64_t seed = only >= 0 ? w->prob_host[only].seed : 0;
        const bool xy = world_xy(w);
        auto *kernel = xy ? (only >= 0 ? walk_step_kernel<true, false> : walk_step_kernel<true, true>)
                          : (only >= 0 ? walk_step_kernel<false, false> : walk_step_kernel<false, true>);
        hipLaunchKernelGGL(kernel, dim3(walk_grid(n_launch, cu)), dim3(256), 0, s, w->bank[cur], n_launch, n_dev,
                           w->cells(), lr, seed, w->e_face, w->e_pos, w->e_dcos, w->e_dsin, w->e_path);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return set_hip_error(e, "gmc_transport_step: sampler");
    unsigned long long *ctr = w->cnt(nxt);
    const bool small = small_tally(n_launch, cu);
    auto *kernel = small ? apply_kernel<kSmallTallyThreads> : apply_kernel<kTallyThreads>;
    hipLaunchKernelGGL(kernel, dim3(tally_blocks(n_launch, cu)), dim3(small ? kSmallTallyThreads : kTallyThreads), 0, s,
                       w->bank[cur], n_launch, n_dev, w->e_face, w->e_pos, w->e_dcos, w->e_dsin, w->e_path, w->s_slot,
                       ExitDev{w->s_face, w->s_pos, w->s_dcos, w->s_dsin, w->s_path}, w->cells(), w->bank[nxt], ctr,
                       ctr + 1);
    e = hipGetLastError();
    if (e == hipSuccess) e = enqueue_finish(w, nxt, s);
    if (e != hipSuccess) return set_hip_error(e, "gmc_transport_step: apply");
    return GMC_OK;
}

// Bucket of a particle count: the next power of two (at least 1024), capped at the capacity.
int64_t step_bucket(const gmc_world *w, int64_t n)
{
    int64_t b = 1024;
    while (b < n) b <<= 1;
    return std::min<int64_t>(b, w->cap);
}

// The captured step for this configuration and bucket, captured (and instantiated) on first use.
// The captured kernels read the particle count from the current bank's device counter.
int step_graph(gmc_world *w, int sampler, const gmc_model *m, int K, int64_t bucket, hipGraphExec_t *exec)
{
    const int integ = (sampler == GMC_SAMPLER_GMC) ? w->integrator : 0;
    const uint64_t mm = (sampler == GMC_SAMPLER_GMC) ? m->serial : 0;
    const int KK = (sampler == GMC_SAMPLER_GMC) ? K : 0;
    const int ff = (sampler == GMC_SAMPLER_GMC && m->collided) ? w->ff_max : 0;
    // the captured launches bake in the world's geometry (the analog walk reads omega_x only in
    // XY geometry), so the key holds it too
    const int xy = world_xy(w) ? 1 : 0;
    for (auto &g : w->step_graphs)
        if (g.sampler == sampler && g.model == mm && g.K == KK && g.integrator == integ && g.cur == w->cur &&
            g.ff == ff && g.xy == xy && g.bucket == bucket) {
            *exec = g.exec;
            return GMC_OK;
        }
    hipStream_t cs = w->capture_stream;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return set_hip_error(e, "gmc_transport_step: begin capture");
    const int rc = enqueue_step(w, sampler, m, K, cs, bucket, w->cnt(w->cur));
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(cs, &graph);
    if (rc != GMC_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (e != hipSuccess) return set_hip_error(e, "gmc_transport_step: end capture");
    hipGraphExec_t x = nullptr;
    e = hipGraphInstantiate(&x, graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGraphDestroy(graph);
        return set_hip_error(e, "gmc_transport_step: instantiate");
    }
    w->step_graphs.push_back({sampler, KK, integ, w->cur, ff, xy, mm, bucket, graph, x});
    *exec = x;
    return GMC_OK;
}

}  // namespace

int gmc_transport_step(gmc_world *w, int sampler, const gmc_model *m, int K, void *stream,
                       int64_t *n_alive_out)
{
    if (!w) return set_error(GMC_EINVAL, "gmc_transport_step: null world");
    if (sampler != GMC_SAMPLER_GMC && sampler != GMC_SAMPLER_MC)
        return set_error(GMC_EINVAL, "gmc_transport_step: sampler must be GMC or MC");
    if (sampler == GMC_SAMPLER_GMC && (!m || K < 1 || K > 1024))
        return set_error(GMC_EINVAL, "gmc_transport_step: GMC needs a model and K in 1..1024");
    if (sampler == GMC_SAMPLER_GMC && m->n_in != 10 && m->n_in != 11)
        return set_error(GMC_EINVAL, "gmc_transport_step: the model is not a boundary model (10 or 11 inputs)");
    if (sampler == GMC_SAMPLER_GMC && m->n_in == 10 &&
        std::any_of(w->rect.begin(), w->rect.end(), [](char r) { return r != 0; }))
        return set_error(GMC_EINVAL, "gmc_transport_step: rectangular cells need an 11-input boundary model");
    if (sampler == GMC_SAMPLER_GMC && world_xy(w) != m->xy)
        return set_error(GMC_EINVAL, "gmc_transport_step: the model's geometry (flatland / XY) differs from the world's");
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = w->n_alive;
    if (n > 0) {
        int rc = GMC_OK;
        hipError_t e = begin_counters(w, s);
        if (e != hipSuccess) return failed_call(s, set_hip_error(e, "gmc_transport_step: launch"));
        if (w->graphs) {
            hipGraphExec_t x = nullptr;
            rc = step_graph(w, sampler, m, K, step_bucket(w, n), &x);
            if (rc == GMC_OK && (e = hipGraphLaunch(x, s)) != hipSuccess)
                rc = set_hip_error(e, "gmc_transport_step: graph launch");
        } else {
            rc = enqueue_step(w, sampler, m, K, s, n, nullptr);
        }
        if (rc == GMC_OK) rc = sync_counters(w, s);
        if (rc != GMC_OK) return failed_call(s, rc);
        w->cur = 1 - w->cur;
        w->stepped += n;
    }
    if (n_alive_out) *n_alive_out = w->n_alive;
    return GMC_OK;
}

int gmc_problem_alive(const gmc_world *w, int32_t pid, int64_t *n_alive)
{
    if (!w || !n_alive || pid < 0 || pid >= w->max_problems || !w->in_use[pid])
        return set_error(GMC_EINVAL, "gmc_problem_alive: no such problem");
    *n_alive = w->alive_pp[pid];
    return GMC_OK;
}

namespace {

// Columns cols[0 .. k-1] of problem pid's tallies to the host arrays dst (NULL: not wanted).
int read_columns(gmc_world *w, int32_t pid, const Column *cols, double *const *dst, int k, hipStream_t s,
                 const char *who)
{
    std::lock_guard<std::mutex> lk(w->mu);       // one reader at a time: the pinned memory is the world's
    const ProblemDev &P = w->prob_host[pid];
    const int64_t n = (int64_t)P.nx * P.ny;
    const double V = P.L * P.Ly;
    Columns q;
    double *to[5];
    for (int i = 0; i < k; ++i)
        if (dst[i]) {
            q.col[q.count] = cols[i];
            to[q.count++] = dst[i];
        }
    const int64_t most = host_doubles(w->max_cells) / (q.count > 0 ? q.count : 1);
    for (int64_t i0 = 0; q.count > 0 && i0 < n; i0 += most) {
        const int64_t m = std::min(most, n - i0);
        hipLaunchKernelGGL(columns_kernel, dim3(blocks_for(m)), dim3(256), 0, s, w->cells(), P.cell0 + i0, m, V, q,
                           w->host_columns);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return set_hip_error(e, who);
        for (int k = 0; k < q.count; ++k) std::memcpy(to[k] + i0, w->host_columns + k * m, 8 * (size_t)m);
    }
    if (q.count == 0) {
        const hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return set_hip_error(e, who);
    }
    return GMC_OK;
}

}  // namespace

int gmc_problem_tally(gmc_world *w, int32_t pid, double *flux, double *absorbed, double *leak,
                      double *cutoff, void *stream)
{
    if (!w || pid < 0 || pid >= w->max_problems || !w->in_use[pid])
        return set_error(GMC_EINVAL, "gmc_problem_tally: no such problem");
    constexpr Column cols[4] = {Column::Flux, Column::Absorbed, Column::Leak, Column::Cutoff};
    double *const dst[4] = {flux, absorbed, leak, cutoff};
    return read_columns(w, pid, cols, dst, 4, (hipStream_t)stream, "gmc_problem_tally: copy");
}

int gmc_problem_path_tally(gmc_world *w, int32_t pid, double *wpath, double *path, double *visits,
                           double *rejected_w, double *rejected_n, void *stream)
{
    if (!w || pid < 0 || pid >= w->max_problems || !w->in_use[pid])
        return set_error(GMC_EINVAL, "gmc_problem_path_tally: no such problem");
    constexpr Column cols[5] = {Column::WeightPath, Column::Path, Column::Visits, Column::RejectedW,
                                Column::RejectedN};
    double *const dst[5] = {wpath, path, visits, rejected_w, rejected_n};
    return read_columns(w, pid, cols, dst, 5, (hipStream_t)stream, "gmc_problem_path_tally: copy");
}

}  // extern "C"
