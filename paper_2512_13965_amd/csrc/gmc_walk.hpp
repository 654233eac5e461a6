// Analog random walk through a cell (paper: section "Monte Carlo Method", eq. 4), as a device
// engine over whole waves, shared by the walk kernel (gmc_walk.hip) and the analog source births
// (gmc_transport.hip).
//
// A walk is a serial chain of flights whose number has a heavy tail (mean 1 + pi tau_s / 4, the
// longest of 2^20 walks at tau = 100 about 10^4), so a launch has two regimes, and a wave goes
// from the first to the second when its share of the walks runs out:
//   * one lane per walk while there are walks to start.  Bound by vector issue: about 110
//     instructions a flight, of which the Philox block takes 40 (19 wide multiplies, 20
//     three-way exclusive ors).  A lane whose walk has ended waits until kRefill lanes of its
//     wave do: the exit records and the next conditions are then handled for all of them at
//     once, as that path costs a wave the same for one lane as for 64.
//   * a group of g lanes per walk (g = 4 .. 64, a power of two) once at most 16 walks are left
//     in the wave.  The random numbers of a flight depend on its index alone, so the group
//     draws its walk's next g flights side by side; only the positions form a chain, which
//     three lanes of the group follow, one for x, one for y and one for the path length, a
//     fused multiply-add a flight; then each lane tests its own flight for the cell's boundary
//     and the first one that ends the walk writes its record.  Every value is the one that the
//     first regime computes, bit for bit: all fused multiply-adds are written as such, none is
//     left to the compiler's choice.
// The walks are dealt out to blocks in advance (BlockShare), and the waves of a block take from
// its share through a counter in LDS.  One counter for the whole launch costs more than the walks where they are
// short: same-address atomics complete one in 13 ns (2^23 walks at tau = 1, 64 to an atomic:
// 1.7 ms).
// Measured, against one lane per walk throughout and a launch-wide counter: 2^20 walks of mixed
// cells (longest 5,200 flights) 2.96 -> 0.11 ms, 10^6 at tau = 100, c = 0.99 (12,000) 8.5 ->
// 0.59 ms, 2^23 at tau = 100 12.7 -> 2.7 ms (2.4e11 flights/s), 2^23 at tau = 1 1.7 -> 0.25 ms.
// The longest walk of a launch costs 11 ns a flight in the end.
#pragma once

#include "gmc_device.hpp"

namespace gmc {
namespace {

// Idle lanes that make a wave stop for the next walks.  8 / 16 / 24 / 32 / 40, 2^23 walks each:
// tau = 100 2.75 / 2.69 / 2.72 / 2.89 / 3.30 ms, tau = 10 0.67 / 0.53 / 0.44 / 0.40 / 0.42 ms.
constexpr int kRefill = 24;
// Walks left in a wave that make it share lanes out (8 instead of 16: 2^20 walks at tau = 100
// 0.76 -> 0.83 ms), and flights after the last refill before it may (0 to 16 measure the same;
// six end most walks of thin cells).
constexpr int kGroupWalks = 16;
constexpr int kGroupAfter = 6;

// End of a walk (besides the exit faces 0..3): absorbed in the cell, or cut off at kMaxFlights.
constexpr int kAbsorbed = -1, kCapped = -2, kAtFace = -4;

// One walk before its first flight: position and direction in the cell [0, wa] x [0, 1] (lengths
// in units of its height), tau over that height, scattering ratio, random stream.
struct WalkStart {
    float x, y, u, v, tau, c, wa;
    uint64_t stream, key;
};

// Shared memory of one wave's lane groups: per coordinate (x, y, path length) the step of each
// flight as (length, direction component), and the coordinate before each flight.
typedef float f32v2 __attribute__((ext_vector_type(2)));
typedef float f32v4 __attribute__((ext_vector_type(4)));
struct __attribute__((aligned(16))) WalkGroups {
    f32v2 step[3][66];
    float at[3][64];
};

// N flights of the chain: the coordinate before each of them to at[0 .. N-1], and after them.
// s holds their steps, two to a vector.
template <int N>
__device__ __forceinline__ float walk_chain(float val, const f32v4 (&s)[N / 2], float *at)
{
    float a[N + 1];
    a[0] = val;
#pragma unroll
    for (int k = 0; k < N; ++k)
        a[k + 1] = __builtin_fmaf(s[k / 2][2 * (k & 1)], s[k / 2][2 * (k & 1) + 1], a[k]);
#pragma unroll
    for (int k = 0; k < N; k += 4) *(f32v4 *)(at + k) = f32v4{a[k], a[k + 1], a[k + 2], a[k + 3]};
    return a[N];
}

// Compiler barrier between a wave's accesses to WalkGroups from different lanes (LDS accesses of
// one wave complete in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int rank_in(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// What the first two Philox rounds of a walk's draws take from its stream and key alone (only
// the third counter word, the flight, changes from draw to draw).
struct DrawPrefix {
    uint32_t a, b, c, d;
};

__device__ __forceinline__ DrawPrefix draw_prefix(uint64_t stream, uint32_t k0, uint32_t k1)
{
    const uint64_t p0 = (uint64_t)kPhiloxM0 * (uint32_t)stream;
    const uint64_t p1 = (uint64_t)kPhiloxM1 * ((uint32_t)(p0 >> 32) ^ kTagWalk ^ k1);
    return DrawPrefix{(uint32_t)(stream >> 32) ^ k0, (uint32_t)(p1 >> 32) ^ (k0 + kPhiloxW0), (uint32_t)p1,
                      (uint32_t)p0 ^ (k1 + kPhiloxW1)};
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Round r (from 0) of a Philox block.
__device__ __forceinline__ void philox_round(U4 &c, uint32_t k0, uint32_t k1, uint32_t r)
{
    const uint64_t p0 = (uint64_t)kPhiloxM0 * c.a, p1 = (uint64_t)kPhiloxM1 * c.c;
    c.a = xor3((uint32_t)(p1 >> 32), c.b, k0 + r * kPhiloxW0);
    c.c = xor3((uint32_t)(p0 >> 32), c.d, k1 + r * kPhiloxW1);
    c.b = (uint32_t)p1;
    c.d = (uint32_t)p0;
}

// Rounds 3 to 10 of a Philox block.
__device__ __forceinline__ U4 philox_rest(U4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (uint32_t r = 2; r < 10; ++r) philox_round(c, k0, k1, r);
    return c;
}

// draw4(key, stream, flight, kTagWalk) from the prefix of (stream, key): its first two rounds, and all.
__device__ __forceinline__ U4 draw_begin(const DrawPrefix &q, uint32_t flight)
{
    const uint64_t f = (uint64_t)kPhiloxM1 * flight;
    const uint64_t g = (uint64_t)kPhiloxM0 * ((uint32_t)(f >> 32) ^ q.a);
    return U4{q.b ^ (uint32_t)f, q.c, (uint32_t)(g >> 32) ^ q.d, (uint32_t)g};
}

__device__ __forceinline__ U4 draw_flight(const DrawPrefix &q, uint32_t k0, uint32_t k1, uint32_t flight)
{
    return philox_rest(draw_begin(q, flight), k0, k1);
}

// The walks or particles 0 .. n-1 that a block of a launch takes: granules of consecutive ones,
// block b the granules b, b + nb, b + 2 nb, ...; a granule halves from 64 until every block has
// four.  Item v of the block is index(v), none if that lies beyond n.
struct BlockShare {
    int shift;
    uint32_t items;
    __device__ __forceinline__ explicit BlockShare(int64_t n) : shift(6)
    {
        while (shift > 0 && ((int64_t)gridDim.x << (shift + 2)) > n) --shift;
        const int64_t nb = gridDim.x, granules = (n + (1 << shift) - 1) >> shift;
        items = (uint32_t)(granules > blockIdx.x ? (granules - blockIdx.x + nb - 1) / nb : 0) << shift;
    }
    __device__ __forceinline__ int64_t index(uint32_t item) const
    {
        return (((int64_t)(item >> shift) * gridDim.x + blockIdx.x) << shift) + (item & ((1u << shift) - 1u));
    }
};

// Distance to the cell's boundary along (u, v); xface: the ray leaves through a vertical face.
__device__ __forceinline__ float walk_boundary(float x, float y, float u, float v, float wa, bool &xface)
{
    const float kInf = __builtin_inff();
    const float tx = fabsf(u) > 0.0f ? (u > 0.0f ? wa - x : -x) * fast_rcp(u) : kInf;
    const float ty = fabsf(v) > 0.0f ? (v > 0.0f ? 1.0f - y : -y) * fast_rcp(v) : kInf;
    xface = tx <= ty;
    return fmaxf(xface ? tx : ty, 0.0f);
}

// Face and counter-clockwise position (a fraction of the face) of the exit after `db`.
__device__ __forceinline__ int walk_exit(float x, float y, float u, float v, float wa, float db, bool xface,
                                         float &pos)
{
    if (xface) {
        const float ye = fminf(fmaxf(__builtin_fmaf(db, v, y), 0.0f), 1.0f);
        pos = u > 0.0f ? ye : 1.0f - ye;
        return u > 0.0f ? 1 : 3;
    }
    const float xe = fminf(fmaxf(__builtin_fmaf(db, u, x), 0.0f), wa);
    pos = v > 0.0f ? (wa - xe) / wa : xe / wa;
    return v > 0.0f ? 2 : 0;
}

// Length of a flight (word 0) where the walk scatters: inv_sig = 1 / sigma, negative in a cell
// without collisions.
__device__ __forceinline__ float flight_length(const U4 &r, float inv_sig)
{
    return inv_sig >= 0.0f ? neg_log(u01(r.a)) * inv_sig : __builtin_inff();
}

// Direction after a scattering (word 1): isotropic in the plane, or, in XY geometry, on the
// sphere (mu = 2 xi - 1 from word 3), projected.
template <bool XY>
__device__ __forceinline__ void scatter_direction(const U4 &r, float &u, float &v)
{
    const float ph = u01(r.b);
    u = cos_turns(ph);
    v = sin_turns(ph);
    if constexpr (XY) {
        const float mu = __builtin_fmaf(2.0f, u01(r.d), -1.0f);
        const float st = sqrtf(fmaxf(__builtin_fmaf(-mu, mu, 1.0f), 0.0f));
        u *= st;
        v *= st;
    }
}

// Walks 0 .. n-1, by all waves of the grid.  fetch(i) gives the start of walk i; emit(i, face, pos,
// u, v, path, collisions) takes its end.  Flight j of a walk draws Philox (key, (stream, j, walk
// tag)): word 0 -> length, 1 -> direction, 2 -> absorption test (ANALOG: a collision absorbs when
// xi > c, flights ~ Exp(tau); otherwise flights ~ Exp(c tau)), 3 -> mu (XY).  KEYS: every walk has
// a key of its own, else key `seed`.  groups: one per wave of the block; pool: the block's counter.
template <bool ANALOG, bool XY, bool KEYS, typename Fetch, typename Emit>
__device__ __forceinline__ void run_walks(int64_t n, uint64_t seed, WalkGroups *groups, uint32_t *pool,
                                          Fetch &&fetch, Emit &&emit)
{
    const int lane = threadIdx.x & 63;
    const int waves = blockDim.x / 64;
    WalkGroups &G = groups[threadIdx.x >> 6];
    if (threadIdx.x == 0) *pool = 0;
    __syncthreads();

    const BlockShare mine(n);
    const uint32_t items = mine.items;
    // lanes of a wave that start a walk: where there are few walks, every wave gets its share
    const uint32_t share = (items + waves - 1) / waves;
    const int lanes = share < 64 ? (int)share : 64;

    const uint32_t s0 = (uint32_t)seed, s1 = (uint32_t)(seed >> 32);
    uint32_t key0 = s0, key1 = s1;
    DrawPrefix q{};
    float x = 0.0f, y = 0.0f, u = 1.0f, v = 0.0f, len = 0.0f, inv_sig = -1.0f, cs = 0.0f, wa = 1.0f;
    uint32_t flight = 0;
    int64_t idx = 0;
    int end = kAtFace;
    bool alive = false, started = false;
    bool dry = items == 0;

    // ---- one lane per walk
    for (;;) {
        if (started && !alive) {
            if (end == kAtFace) {
                bool xface;
                float pos;
                const float db = walk_boundary(x, y, u, v, wa, xface);
                const int face = walk_exit(x, y, u, v, wa, db, xface, pos);
                emit(idx, face, pos, u, v, len + db, flight);
            } else {
                emit(idx, end, 0.0f, u, v, len, flight);
            }
            started = false;
        }
        const bool need = !alive && lane < lanes;
        const uint64_t needs = __ballot(need);
        const int cnt = __popcll(needs);
        if (!dry) {
            uint32_t first = 0;
            if (lane == 0) first = atomicAdd(pool, (uint32_t)cnt);
            first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
            dry = first >= items || items - first <= (uint32_t)cnt;
            const uint32_t item = first + (uint32_t)rank_in(needs);
            if (need && first < items && item < items) {
                idx = mine.index(item);
                if (idx < n) {
                    const WalkStart w = fetch(idx);
                    const float sig = ANALOG ? w.tau : w.c * w.tau;
                    inv_sig = sig > 1e-30f ? 1.0f / sig : -1.0f;    // 1 / sig would overflow below
                    cs = w.c;
                    x = w.x;
                    y = w.y;
                    u = w.u;
                    v = w.v;
                    wa = w.wa;
                    len = 0.0f;
                    flight = 0;
                    if constexpr (KEYS) {
                        key0 = (uint32_t)w.key;
                        key1 = (uint32_t)(w.key >> 32);
                    }
                    q = draw_prefix(w.stream, KEYS ? key0 : s0, KEYS ? key1 : s1);
                    alive = started = true;
                    end = kAtFace;
                }
            }
        }
        int active = __popcll(__ballot(alive));
        if (active == 0) {
            if (dry) return;
            continue;
        }
        // on until enough lanes idle, or, with few walks left, once more to the pool, until it is dry
        const int stop = dry ? 0 : lanes - kRefill;
        for (int it = 0; active > 0; ++it) {
            if ((active <= stop && it > 0) || (active <= kGroupWalks && it >= kGroupAfter)) break;
            if (alive) {
                bool xface;
                const float db = walk_boundary(x, y, u, v, wa, xface);
                const U4 r = draw_flight(q, KEYS ? key0 : s0, KEYS ? key1 : s1, flight);
                const float ds = flight_length(r, inv_sig);
                if (ds >= db) {
                    alive = false;
                } else {
                    len += ds;
                    x = __builtin_fmaf(ds, u, x);
                    y = __builtin_fmaf(ds, v, y);
                    flight += 1;
                    if (ANALOG && u01(r.c) > cs) {
                        alive = false;
                        end = kAbsorbed;
                    } else {
                        scatter_direction<XY>(r, u, v);
                        if (flight >= kMaxFlights) {
                            alive = false;
                            end = kCapped;
                        }
                    }
                }
            }
            active = __popcll(__ballot(alive));
        }
        if (dry && active > 0) break;
    }
    if (started && !alive) {
        if (end == kAtFace) {
            bool xface;
            float pos;
            const float db = walk_boundary(x, y, u, v, wa, xface);
            const int face = walk_exit(x, y, u, v, wa, db, xface, pos);
            emit(idx, face, pos, u, v, len + db, flight);
        } else {
            emit(idx, end, 0.0f, u, v, len, flight);
        }
    }

    // ---- a group of g lanes per walk: lane `base` + j holds flight `flight` + j; lanes j = 0, 1, 2
    // carry x, y and the path length along the chain in `val`
    int g = 1, base = lane, j = 0;
    float val = 0.0f;
    for (;;) {
        const uint64_t leaders = __ballot(alive && j == 0);
        const int walks = __popcll(leaders);
        if (walks == 0) return;
        if (g == 1 || 2 * walks * g <= 64) {
            if (g > 1) {
                x = __shfl(val, base);
                y = __shfl(val, base + 1);
                len = __shfl(val, base + 2);
                u = G.step[0][base].y;
                v = G.step[1][base].y;
            }
            while (2 * walks * g <= 64) g *= 2;
            float *from = G.at[0];
            wave_sync();
            if (alive && j == 0) from[rank_in(leaders)] = __int_as_float(lane);
            wave_sync();
            const int w = lane / g;
            alive = w < walks;
            const int src = alive ? __float_as_int(from[w]) : lane;
            base = lane & ~(g - 1);
            j = lane - base;
            x = __shfl(x, src);
            y = __shfl(y, src);
            len = __shfl(len, src);
            u = __shfl(u, src);
            v = __shfl(v, src);
            wa = __shfl(wa, src);
            inv_sig = __shfl(inv_sig, src);
            if constexpr (ANALOG) cs = __shfl(cs, src);
            flight = (uint32_t)__shfl((int)flight, src);
            q.a = (uint32_t)__shfl((int)q.a, src);
            q.b = (uint32_t)__shfl((int)q.b, src);
            q.c = (uint32_t)__shfl((int)q.c, src);
            q.d = (uint32_t)__shfl((int)q.d, src);
            if constexpr (KEYS) {
                key0 = (uint32_t)__shfl((int)key0, src);
                key1 = (uint32_t)__shfl((int)key1, src);
            }
            idx = (int64_t)__shfl((long long)idx, src);
            val = j == 1 ? y : (j == 2 ? len : x);
            wave_sync();
            if (j == 0) {
                G.step[0][lane].y = u;
                G.step[1][lane].y = v;
            }
        }
        if (g == 64) break;
        bool ends = false, xface = false, absorbed = false;
        float db = 0.0f, ds = 0.0f, un = 0.0f, vn = 0.0f;
        if (alive) {
            const U4 r = draw_flight(q, KEYS ? key0 : s0, KEYS ? key1 : s1, flight + (uint32_t)j);
            ds = flight_length(r, inv_sig);
            scatter_direction<XY>(r, un, vn);
            if constexpr (ANALOG) absorbed = u01(r.c) > cs;
            G.step[0][lane].x = ds;
            G.step[1][lane].x = ds;
            G.step[2][lane] = f32v2{ds, 1.0f};
            if (j + 1 < g) {               // the next flight's direction
                G.step[0][lane + 1].y = un;
                G.step[1][lane + 1].y = vn;
            }
            wave_sync();
            const int coord = j == 1 ? 1 : (j == 2 ? 2 : 0);
            const f32v4 *step = (const f32v4 *)&G.step[coord][base];
            float *at = &G.at[coord][base];    // the lanes from j = 3 on repeat lane 0
            if (g == 4) {
                const f32v4 s[2] = {step[0], step[1]};
                val = walk_chain<4>(val, s, at);
            } else {
                // eight flights at a time, the next eight steps on their way meanwhile
                f32v4 s[4] = {step[0], step[1], step[2], step[3]};
#pragma unroll 1                               // unrolled further, it spills
                for (int k = 8; k < g; k += 8) {
                    const f32v4 t[4] = {step[k / 2], step[k / 2 + 1], step[k / 2 + 2], step[k / 2 + 3]};
                    val = walk_chain<8>(val, s, at + k - 8);
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[i] = t[i];
                }
                val = walk_chain<8>(val, s, at + g - 8);
            }
            wave_sync();
            x = G.at[0][lane];
            y = G.at[1][lane];
            len = G.at[2][lane];
            u = G.step[0][lane].y;
            v = G.step[1][lane].y;
            db = walk_boundary(x, y, u, v, wa, xface);
            ends = ds >= db || absorbed || flight + (uint32_t)j + 1u >= kMaxFlights;
        }
        const uint64_t all = __ballot(ends);
        if (alive) {
            const uint64_t ours = (all >> base) & ((1ull << g) - 1ull);
            if (ours) {
                if (j == __ffsll((unsigned long long)ours) - 1) {
                    const uint32_t f = flight + (uint32_t)j;
                    if (ds >= db) {
                        float pos;
                        const int face = walk_exit(x, y, u, v, wa, db, xface, pos);
                        emit(idx, face, pos, u, v, len + db, f);
                    } else if (absorbed) {
                        emit(idx, kAbsorbed, 0.0f, u, v, len + ds, f + 1u);
                    } else {
                        emit(idx, kCapped, 0.0f, un, vn, len + ds, f + 1u);
                    }
                }
                alive = false;
            } else {
                flight += (uint32_t)g;
                if (j == g - 1) {          // the first direction of the next round
                    G.step[0][base].y = un;
                    G.step[1][base].y = vn;
                }
            }
        }
        wave_sync();
    }

    // ---- the wave's last walk, by all its lanes (base = 0, j = lane; what belongs to the walk is
    // uniform): a chain of 64 flights, eight at a time and unrolled, with the next eight's steps on
    // their way (24 steps on their way spill) and, in the shadow of each eight, one of the last eight
    // Philox rounds of the next 64 flights' draws.  A flight of the longest walk: 20 ns in the loop
    // above, 15 unrolled, 11 with the draws in the shadow (2^16 walks at tau = 1000 7.8 -> 5.9 ms).
    auto uniform = [](uint32_t a) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)a); };
    auto uniform_f = [](float a) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(a))); };
    q = DrawPrefix{uniform(q.a), uniform(q.b), uniform(q.c), uniform(q.d)};
    key0 = uniform(KEYS ? key0 : s0);
    key1 = uniform(KEYS ? key1 : s1);
    flight = uniform(flight);
    wa = uniform_f(wa);
    inv_sig = uniform_f(inv_sig);
    if constexpr (ANALOG) cs = uniform_f(cs);
    const int coord = lane == 1 ? 1 : (lane == 2 ? 2 : 0);
    const f32v4 *step = (const f32v4 *)&G.step[coord][0];
    float *at = &G.at[coord][0];               // the lanes from 3 on repeat lane 0
    U4 r = draw_flight(q, key0, key1, flight + (uint32_t)lane);
    for (;;) {
        float un, vn;
        const float ds = flight_length(r, inv_sig);
        scatter_direction<XY>(r, un, vn);
        const bool absorbed = ANALOG && u01(r.c) > cs;
        G.step[0][lane].x = ds;
        G.step[1][lane].x = ds;
        G.step[2][lane] = f32v2{ds, 1.0f};
        G.step[0][lane + 1].y = un;
        G.step[1][lane + 1].y = vn;
        wave_sync();
        f32v4 s[2][4];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[c][i] = step[4 * c + i];
        r = draw_begin(q, flight + 64u + (uint32_t)lane);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            val = walk_chain<8>(val, s[c % 2], at + 8 * c);
            if (c + 2 < 8) {
#pragma unroll
                for (int i = 0; i < 4; ++i) s[c % 2][i] = step[4 * (c + 2) + i];
            }
            philox_round(r, key0, key1, 2u + c);
            __builtin_amdgcn_sched_barrier(0);
        }
        wave_sync();
        x = G.at[0][lane];
        y = G.at[1][lane];
        len = G.at[2][lane];
        u = G.step[0][lane].y;
        v = G.step[1][lane].y;
        bool xface;
        const float db = walk_boundary(x, y, u, v, wa, xface);
        const uint32_t f = flight + (uint32_t)lane;
        const uint64_t ends = __ballot(ds >= db || absorbed || f + 1u >= kMaxFlights);
        if (ends) {
            if (lane == __ffsll((unsigned long long)ends) - 1) {
                if (ds >= db) {
                    float pos;
                    const int face = walk_exit(x, y, u, v, wa, db, xface, pos);
                    emit(idx, face, pos, u, v, len + db, f);
                } else if (absorbed) {
                    emit(idx, kAbsorbed, 0.0f, u, v, len + ds, f + 1u);
                } else {
                    emit(idx, kCapped, 0.0f, un, vn, len + ds, f + 1u);
                }
            }
            return;
        }
        flight += 64u;
        if (lane == 63) {                      // the first direction of the next round
            G.step[0][0].y = un;
            G.step[1][0].y = vn;
        }
        wave_sync();
    }
}

}  // namespace
}  // namespace gmc
