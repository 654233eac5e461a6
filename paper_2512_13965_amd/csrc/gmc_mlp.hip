// Fused velocity-MLP + ODE sampler for gfx950 (paper: section "Conditional Flow
// Matching", eq. 8; network of section "Network Architecture and Inputs"; decoding of eq. 11).
//
// BF16 and FP8 models of width 128 run mlp_wave_kernel (below).  The others: persistent workgroups
// (four waves for FP32, eight in the two-group schedule of BF16 / FP8 models) each own a tile of
// samples at a time and carry it through all ODE steps (Euler x <- x + v(x, k/K | c) / K, or
// classic RK4):
//   * the tile's activations live in LDS (128 x H), the ODE state x and the condition in LDS;
//   * each hidden layer is a [H x H] x [H x 128] contraction on MFMA; each wave owns a set of
//     32-row output tiles (four-wave kernels: wave w the rows [w*H/4, (w+1)*H/4); two-group
//     schedule: see Cfg) and keeps its 32x32 accumulator tiles in registers;
//   * weights stream from L2 straight into MFMA operand registers, pre-arranged on the host in
//     per-lane fragment order so each lane issues one 16-byte load per 32-row tile and k-block
//     and a wave's loads are one contiguous 1 KB line;
//   * the epilogue (bias already in the accumulator, SiLU, cast to the next layer's operand
//     type) writes each accumulator tile back into the LDS activation tile in the column order
//     the next layer's operand reads expect, so the next layer's B-operand reads are contiguous
//     16-byte LDS reads; the host permutes the next layer's weight columns to match.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "gmc_device.hpp"
#include "gmc_internal.hpp"
#include "gmc_mma.hpp"

namespace gmc {
namespace {

// BF16 and FP8 models carry every hidden activation scaled by -log2(e): the host scales the
// first layer's weights and every hidden bias by -log2(e) and the output layer's weights by
// -ln 2 (the same network in exact arithmetic), so an accumulator holds a' = -log2(e) a, and
// the scaled activation -log2(e) SiLU(a) is a' / (1 + 2^a'): the exponential takes the
// accumulator as it is.  FP8 models (SCALE) store half of it divided by the next layer's
// activation scale (a power of two, folded into the reciprocal's argument) and their e4m3
// layers apply 2 sw sa through the matrix core's operand scale.  FP32 models keep plain
// activations.

// One epilogue unit of an FP32 model: the activation of accumulator values 4g .. 4g+3.
__device__ __forceinline__ void epi_unit(const f32x16 &acc, int g, uint32_t *w)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = __builtin_bit_cast(uint32_t, silu(acc[4 * g + j]));
}

// The SiLU epilogue of the NT accumulator tiles a(t) of a BF16 or FP8 model (16 values each, value
// i = 16 t + i % 16), software-pipelined: iteration j issues the exponential of value j - D, the add of
// value j - 2D, the reciprocal of value j - 3D and the final multiply of value j - 4D -- independent
// instructions -- and packs groups of values as they complete; store(t, words) receives each
// tile's packed words once its last value is done.  With per-layer scales the output factor
// oscale * inv_next (a power of two) goes into the reciprocal's argument, acc * rcp((1 + e) / c)
// being exactly (acc * c) * rcp(1 + e).
// hook(j) runs in iteration j (matrix work of the same wave, spread over the pipeline).
constexpr int kPipeD = 1;
struct NoHook {
    template <typename J> __device__ __forceinline__ void operator()(J) const {}
};
template <int PO, bool SCALE, int NT, typename Val, typename Store, typename Hook = NoHook>
__device__ __forceinline__ void drain_pipe(Val &&val, float oscale, float inv_next, Store &&store, Hook &&hook = Hook{})
{
    constexpr int NV = NT * 16;
    constexpr int D = kPipeD;
    static_assert(PO == kBF16 || PO == kFP8, "FP32 models take epi_unit");
    const float k = SCALE ? 1.0f / (oscale * inv_next) : 1.0f;
    float t[NV], y[NV];
    uint32_t wd[NT][4 * words_per_unit(PO)];
    sfor<NV + 4 * D>([&](auto J) {
        constexpr int j = decltype(J)::value;
        if constexpr (j < NV) t[j] = val(std::integral_constant<int, j>{});
        if constexpr (j - D >= 0 && j - D < NV) t[j - D] = __builtin_amdgcn_exp2f(t[j - D]);
        if constexpr (j - 2 * D >= 0 && j - 2 * D < NV) {
            if constexpr (SCALE) t[j - 2 * D] = __builtin_fmaf(t[j - 2 * D], k, k);
            else t[j - 2 * D] = 1.0f + t[j - 2 * D];
        }
        if constexpr (j - 3 * D >= 0 && j - 3 * D < NV) t[j - 3 * D] = __builtin_amdgcn_rcpf(t[j - 3 * D]);
        if constexpr (j - 4 * D >= 0 && j - 4 * D < NV) {
            constexpr int i = j - 4 * D;
            y[i] = val(std::integral_constant<int, i>{}) * t[i];
            constexpr int tt = i / 16, v = i % 16;
            if constexpr (PO == kBF16) {
                if constexpr (v % 2 == 1) wd[tt][v / 2] = pack_bf16(y[i - 1], y[i]);
            } else {
                if constexpr (v % 4 == 3) wd[tt][v / 4] = pack_fp8x4(y[i - 3], y[i - 2], y[i - 1], y[i]);
            }
            if constexpr (v == 15) store(std::integral_constant<int, tt>{}, wd[tt]);
        }
        hook(J);
        __builtin_amdgcn_sched_barrier(0);
    });
}


// One dense layer + SiLU of an FP32 model for this wave's RTW row tiles and all CT column tiles of
// samples.  The rows are done in NP passes of RP row tiles; the epilogue of pass p runs interleaved with the
// MFMA k-loop of pass p + 1 (it only reads pass p's accumulators), so the SiLU transcendentals
// overlap the matrix unit.  Those results are held packed in registers until every wave has
// finished reading the input tile (barrier, when `out` aliases the input); the last pass's
// epilogue is computed and stored after that barrier.
template <int RTW, int CT, int NKB, bool IN_PLACE>
__device__ __forceinline__ void dense_silu(Rsrc wA, Rsrc bias, int T0, const char *in, int in_stride, char *out,
                                           int out_stride, int lane)
{
    constexpr int RP = RTW >= 4 ? RTW / 2 : 1;     // row tiles per pass
    constexpr int NP = RTW / RP;                   // passes
    constexpr int UNITS = RP * CT * 4;             // epilogue units (4 values) per pass
    constexpr int WPU = words_per_unit(kF32);
    constexpr int UPK = (UNITS + NKB - 1) / NKB;   // epilogue units per k-block
    uint32_t pk[NP > 1 ? NP - 1 : 1][UNITS * WPU];
    f32x16 acc[2][RP][CT];
    auto epi = [&](auto PP, int u) {
        constexpr int pp = decltype(PP)::value;
        const int r = u / (4 * CT), c = (u / 4) % CT, g = u % 4;
        epi_unit(acc[pp % 2][r][c], g, &pk[pp][u * WPU]);
    };
    sfor<NP>([&](auto P) {
        constexpr int p = decltype(P)::value;
        init_bias<RP, CT>(acc[p % 2], bias, T0 + p * RP, lane);
        mma_pass<kF32, RP, CT, NKB>(acc[p % 2], wA, T0 + p * RP, in, in_stride, 0, lane, [&](auto KB) {
            constexpr int kb = decltype(KB)::value;
            if constexpr (p > 0) {
                sfor<UPK>([&](auto J) {
                    constexpr int u = kb * UPK + decltype(J)::value;
                    if constexpr (u < UNITS) epi(std::integral_constant<int, p - 1>{}, u);
                });
            }
        });
        if constexpr (p > 0 && NKB * UPK < UNITS) {
            sfor<UNITS - NKB * UPK>([&](auto J) {
                epi(std::integral_constant<int, p - 1>{}, NKB * UPK + decltype(J)::value);
            });
        }
    });
    if constexpr (IN_PLACE) __syncthreads();
    sfor<NP - 1>([&](auto P) {
        constexpr int p = decltype(P)::value;
        sfor<RP * CT>([&](auto TC) {
            constexpr int r = decltype(TC)::value / CT, c = decltype(TC)::value % CT;
            store_tile<kF32>(&pk[p][(r * CT + c) * 4 * WPU], T0 + p * RP + r, c, out, out_stride, lane);
        });
    });
    constexpr int pl = NP - 1;
    sfor<RP * CT>([&](auto TC) {
        constexpr int r = decltype(TC)::value / CT, c = decltype(TC)::value % CT;
        uint32_t w[4 * WPU];
#pragma unroll
        for (int g = 0; g < 4; ++g) epi_unit(acc[pl % 2][r][c], g, &w[g * WPU]);
        store_tile<kF32>(w, T0 + pl * RP + r, c, out, out_stride, lane);
    });
}

// Part J of NJ of draining accumulator tiles src[RP][CT] through the epilogue into packed words.
template <int NJ, int J, int RP, int CT>
__device__ __forceinline__ void drain_step(const f32x16 (&src)[RP][CT], uint32_t *pk)
{
    constexpr int UNITS = RP * CT * 4;
    constexpr int UPK = (UNITS + NJ - 1) / NJ;
    constexpr int WPU = words_per_unit(kF32);
    sfor<UPK>([&](auto U) {
        constexpr int u = J * UPK + decltype(U)::value;
        if constexpr (u < UNITS) epi_unit(src[u / (4 * CT)][(u / 4) % CT], u % 4, &pk[u * WPU]);
    });
}

// Store the packed outputs of one row pass (row tiles Tb .. Tb + RP - 1, all column tiles).
template <int RP, int CT>
__device__ __forceinline__ void store_pass(const uint32_t *pk, int Tb, char *act, int stride, int lane)
{
    constexpr int WPU = words_per_unit(kF32);
    sfor<RP * CT>([&](auto TC) {
        constexpr int r = decltype(TC)::value / CT, c = decltype(TC)::value % CT;
        store_tile<kF32>(&pk[(r * CT + c) * 4 * WPU], Tb + r, c, act, stride, lane);
    });
}

template <int MP, int H, int TM = kTileM>
struct Cfg {
    static constexpr int P1 = layer_prec(MP, 0);            // layer 1 operand precision
    static constexpr int PH = layer_prec(MP, 1);            // hidden layers' operand precision
    static constexpr int P5 = layer_prec(MP, 4);            // last layer operand precision
    static constexpr bool SCALE = (MP == kFP8);             // per-layer FP8 scales
    static constexpr int ACT_ELEM = (MP == kF32) ? 4 : 2;   // widest type stored in the tile
    static constexpr int ACT_STRIDE = H * ACT_ELEM + 16;    // +16 B: conflict-free row reads
    static constexpr int IN_STRIDE = 16 * elem_bytes(P1) + 16;
    // Two-group schedule (BF16 / FP8, H >= 256): eight waves, two per SIMD.  Group 0 owns the
    // first half of every layer's output rows, group 1 the second half; while one group's
    // waves run the matrix k-loop, the other group's waves run the SiLU epilogue on the same
    // SIMDs, so vector and matrix work overlap across waves.
    static constexpr bool GROUPS = (MP != kF32);
    static_assert(!GROUPS || H >= 256, "width 128 has kernels of its own");
    static constexpr int W = GROUPS ? 8 : kWaves;
    static constexpr int THREADS = 64 * W;
    static constexpr int NT = H / 32;                       // row tiles of a hidden layer
    static constexpr int RTW = NT / W;                      // row tiles per wave
    static constexpr int RPG = NT / 8;                      // row tiles per wave (two-group schedule)
    static constexpr int NKB1 = 16 / kb_width(P1);
    static constexpr int NKBH = H / kb_width(PH);
    static constexpr int NKB5 = H / kb_width(P5);
    static constexpr int RP = RTW >= 4 ? RTW / 2 : 1;       // row tiles per pass
    static constexpr int NP = RTW / RP;                     // row passes per layer
    // Cross-layer pipelining (FP32): pass p of wave w computes row tiles p * NT / 2 + w * RP + r, so
    // the first passes of all waves fill the first half of the consumer's k-blocks and the
    // second passes the other half; each half must be whole k-blocks.
    static constexpr bool PIPE = !GROUPS && NP == 2 && NKBH % 2 == 0 && NKB5 % 2 == 0;
    static constexpr int GH = PIPE ? NKBH / 2 : 1;
    static constexpr int G5 = PIPE ? NKB5 / 2 : 1;
    static constexpr int CT = TM / 32;                      // sample column tiles of a tile
    static constexpr int LDS_ACT = TM * ACT_STRIDE;
    static constexpr int LDS_IN = TM * IN_STRIDE;
    // two-group schedule: the hidden layers' and the output layer's biases stay in LDS
    static constexpr int BIAS = GROUPS ? 4 * H + 32 : 0;
    static constexpr int LDS_BYTES = LDS_ACT + LDS_IN + (5 + 6 + 5 + 5) * TM * 4 + BIAS * 4;
    // k-blocks of weight fragments a wave keeps on their way (two-group schedule).  A CU takes
    // 64 bytes of them a cycle some 700 cycles after it asks; small tiles multiply a k-block too fast
    // to load ahead by two of them, and have the registers for more.  RK4 x 12 at width 512, ring of
    // 2 or 4 / 8 / 16 k-blocks: 10,000 samples (64 to a tile) BF16 862 / 923 / 1,028 us, FP8 676 (2) /
    // 727 (4); 1,000 samples (32) BF16 625 / 627 / 803 us.  Full tiles keep 2: 4 spill (2^20 samples,
    // Euler K = 16: BF16 21.2 / 21.4 ms, FP8 with 1 / 2 14.4 / 16.1 ms).
    static constexpr int NJ = NKBH / 2 > 0 ? NKBH / 2 : 1;
    static constexpr int WANT = (TM >= kWideTileM ? 2 : TM == kMidTileM ? 4 : 8) / (PH == kFP8 ? 2 : 1);
    static constexpr int RING = WANT < NJ ? WANT : NJ;
};

template <int MP, int H, int RK, int TM>
__global__ __launch_bounds__((Cfg<MP, H, TM>::THREADS), 1) void mlp_ode_kernel(MlpParams p)
{
    using C = Cfg<MP, H, TM>;
    static_assert(C::LDS_BYTES <= 160 * 1024, "LDS budget");
    static_assert(C::RTW >= 1 && C::NT % C::W == 0, "row tiles must split evenly over the waves");
    static_assert(C::GROUPS || C::W >= C::CT, "one wave per column tile in layer 5");
    static_assert(!C::GROUPS || (C::RPG >= 1 && C::NKBH % 2 == 0 && C::NKB5 % 2 == 0),
                  "two-group schedule: each group's rows fill whole k-blocks of the consumer");
    __shared__ __attribute__((aligned(16))) char smem[C::LDS_BYTES];
    char *act = smem;
    char *in0 = smem + C::LDS_ACT;
    float *xs = (float *)(smem + C::LDS_ACT + C::LDS_IN);   // [5][128] ODE state
    float *cf = xs + 5 * TM;                              // [6][128] condition features
    float *ksum = cf + 6 * TM;                            // [5][128] RK4 stage sum
    float *vout = ksum + 5 * TM;                          // [5][128] last network output
    float *biases = vout + 5 * TM;                        // [4][H], [32] (two-group schedule)

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // samples to process: the launch's own count, or one the device holds (a captured graph
    // sized for a bucket of counts); noise and raw keep the row stride p.n
    const int64_t n_items = p.n_dev ? (int64_t)*p.n_dev : p.n;
    if constexpr (TM != kTileM) {
        if (p.n_dev_large) {
            const bool large = n_items > p.small_max;
            if (blockIdx.x == 0 && threadIdx.x == 0) *p.n_dev_large = large ? (unsigned long long)n_items : 0ull;
            if (large) return;
        }
    }
    const int64_t ntiles = (n_items + TM - 1) / TM;
    const float dt = 1.0f / (float)p.K;
    constexpr bool rk4 = (RK == 1);
    const int nevals = rk4 ? 4 * p.K : p.K;
    // Euler: the lane that holds output d of sample sn applies x += dt v at once.  Classic RK4:
    // the output goes to vout; before the next evaluation the thread of sample tid forms the
    // stage input (stages at t, t + dt/2, t + dt/2, t + dt take x, x + dt/2 k1, x + dt/2 k2,
    // x + dt k3) and after the fourth stage x += dt/6 (k1 + 2 k2 + 2 k3 + k4).
    auto emit = [&](int d, int sn, float v) {
        const int o = d * TM + sn;
        if constexpr (rk4) vout[o] = v;
        else xs[o] += v * dt;
    };
    auto advance = [&](int e, float xi[5]) {
        const int stage = e & 3;
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            const int o = d * TM + tid;
            const float v = vout[o];
            if (stage < 3) {
                ksum[o] = stage == 0 ? v : ksum[o] + 2.0f * v;
                xi[d] = xs[o] + (stage == 2 ? dt : 0.5f * dt) * v;
            } else {
                xi[d] = xs[o] = xs[o] + (dt * (1.0f / 6.0f)) * (ksum[o] + v);
            }
        }
    };
    // two-group schedule: this wave's weight fragments of the hidden layers' next k-blocks (wrapping
    // from the last hidden layer to the first of the next evaluation), and those of layer 1
    using FragH = typename Mma<C::PH>::Frag;
    using Frag1 = typename Mma<C::P1>::Frag;
    FragH ring[C::RING][C::GROUPS ? C::RPG : 1];
    Frag1 first[C::GROUPS ? C::RPG : 1];
    const int tb = __builtin_amdgcn_readfirstlane((wave >> 2) * (C::NT / 2) + (wave & 3) * C::RPG);
    auto load_hidden = [&](FragH (&slot)[C::GROUPS ? C::RPG : 1], Rsrc w, int kb) {
#pragma unroll
        for (int r = 0; r < C::RPG; ++r)
            slot[r] = Mma<C::PH>::load_g(w, lane * frag_bytes(C::PH), ((tb + r) * C::NKBH + kb) * 64 * frag_bytes(C::PH));
    };
    auto load_first = [&] {
        const Rsrc w = make_rsrc(p.wA[0], p.wA_bytes[0]);
#pragma unroll
        for (int r = 0; r < C::RPG; ++r)
            first[r] = Mma<C::P1>::load_g(w, lane * frag_bytes(C::P1), (tb + r) * 64 * frag_bytes(C::P1));
    };
    if constexpr (C::GROUPS) {
        for (int l = 0; l < 4; ++l)
            for (int k = tid; k < H; k += C::THREADS) biases[l * H + k] = p.bias[l][k];
        if (tid < 32) biases[4 * H + tid] = p.bias[4][tid];
        const Rsrc w1 = make_rsrc(p.wA[1], p.wA_bytes[1]);
        sfor<C::RING>([&](auto D) { load_hidden(ring[decltype(D)::value], w1, decltype(D)::value); });
        load_first();
        // visible after the barrier that follows the first tile's inputs
    }
    // This lane's index for the addresses of one phase.  The FP8 kernel of width 512 forms them
    // anew in each: held through the other phases they spill (58 registers; 2 now; 2^20 samples
    // 14.8 -> 14.3 ms).  The others have the registers, and would pay 1.8 % in vector instructions.
    auto here = [&] {
        int l = tid & 63;
        if constexpr (MP == kFP8 && H == 512 && TM == kTileM) asm volatile("" : "+v"(l));
        return l;
    };
    const int T0 = wave * C::RTW;                    // first row tile (layer-by-layer path)
    const int TX = wave * C::RP, TY = C::NT / 2 + wave * C::RP;   // pass row tiles (pipelined path)

    // The two groups of the two-group schedule run separate code (the same barriers in the same
    // order): one code for both holds each group's registers through the other's phases (48
    // registers spilled of the BF16 kernel of width 512; 4 now).  With the weights of the next
    // phase on their way across the barriers, half of the output layer's at once and the biases in
    // LDS: BF16 width 512, 2^20 samples, Euler K = 16 21.75 -> 21.16 ms (the library's own product
    // of two 8192 x 8192 matrices runs at the rate of 22.1 ms: the power limit holds the clock),
    // RK4 x 12 50,003 samples 3.62 -> 3.42 ms, 10,000 (64-sample tiles) 947 -> 862 us, 1,000 (32-sample
    // tiles, their weights at 80 % of a CU's 64 bytes a cycle) 760 -> 626 us; FP8 1,000 531 -> 417 us.
    auto tiles = [&](auto GRP) {
        constexpr int grp = decltype(GRP)::value;
        for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
            const int64_t base = tile * TM;
            if ((!C::GROUPS || grp == 0) && tid < TM) {
                const int64_t i = base + tid;
                float z[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
                float lt = 0.f, cc = 0.f, yy = 0.5f, ss = 0.f, xx = 0.5f, co = 1.f, la = 0.f;
                if (i < n_items) {
                    lt = p.log_tau[i];
                    cc = p.c[i];
                    yy = p.y_in[i];
                    ss = p.sin_th[i];
                    if (p.n_cond == 6) {
                        xx = p.x_in[i];
                        co = p.cos_phi[i];
                    }
                    if (p.log_aspect) la = p.log_aspect[i];
                    else if (p.omega_x) la = p.omega_x[i];     // XY model: fifth feature omega_x
                    if (p.noise) {
#pragma unroll
                        for (int d = 0; d < 5; ++d) z[d] = p.noise[d * p.n + i];
                    } else {
                        normal5(p.keys ? p.keys[i] : p.seed, p.ids ? p.ids[i] : p.id_base + (uint64_t)i, z);
                    }
                }
#pragma unroll
                for (int d = 0; d < 5; ++d) xs[d * TM + tid] = z[d];
                // boundary model: (ln tau, c, 2 y_in - 1, sin th), rectangular cells add ln A, an
                // XY-geometry model the entry direction's in-plane x component omega_x;
                // internal model: (ln tau, c, 2 x - 1, 2 y - 1, cos phi, sin phi)
                cf[0 * TM + tid] = lt;
                cf[1 * TM + tid] = cc;
                if (p.n_cond == 6) {
                    cf[2 * TM + tid] = 2.0f * xx - 1.0f;
                    cf[3 * TM + tid] = 2.0f * yy - 1.0f;
                    cf[4 * TM + tid] = co;
                    cf[5 * TM + tid] = ss;
                } else {
                    cf[2 * TM + tid] = 2.0f * yy - 1.0f;
                    cf[3 * TM + tid] = ss;
                    cf[4 * TM + tid] = la;
                    cf[5 * TM + tid] = 0.0f;
                }
            }
            __syncthreads();

            // Two-group schedule: the layer-5 lanes apply the integrator's update (Euler step, RK4
            // stage) and write the next input row themselves, so the input row is assembled here
            // only for the first evaluation.
            for (int e = 0; e < nevals; ++e) {
                const int stage = rk4 ? (e & 3) : 0;
                const int k = rk4 ? (e >> 2) : e;
                const float t = ((float)k + (stage == 0 ? 0.0f : (stage == 3 ? 1.0f : 0.5f))) * dt;
                // layer-1 input row of sample tid: [x0..x4, t, ln tau, c, 2y-1, sin th, 0 x 6]
                if ((!C::GROUPS || (e == 0 && grp == 0)) && tid < TM) {
                    float v[16];
                    if (!rk4 || e == 0) {
#pragma unroll
                        for (int d = 0; d < 5; ++d) v[d] = xs[d * TM + tid];
                    } else {
                        advance(e - 1, v);
                    }
                    v[5] = t;
#pragma unroll
                    for (int d = 0; d < 6; ++d) v[6 + d] = cf[d * TM + tid];   // zero past n_cond
#pragma unroll
                    for (int d = 12; d < 16; ++d) v[d] = 0.0f;
                    char *row = in0 + tid * C::IN_STRIDE;
                    if constexpr (C::P1 == kF32) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *(f32x4 *)(row + 16 * q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                    } else {
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            *(u32x4 *)(row + 16 * q) =
                                u32x4{pack_bf16(v[8 * q], v[8 * q + 1]), pack_bf16(v[8 * q + 2], v[8 * q + 3]),
                                      pack_bf16(v[8 * q + 4], v[8 * q + 5]), pack_bf16(v[8 * q + 6], v[8 * q + 7])};
                    }
                }
                if (!C::GROUPS || e == 0) __syncthreads();

                if constexpr (C::GROUPS) {
                    // Two-group schedule.  Per hidden layer, three barrier-separated phases:
                    //   P1: group 0 multiplies over the k-blocks of the first half of the input
                    //       features; group 1 runs the epilogue of its previous-layer rows (layer 1
                    //       included) and writes them over the second half (nobody reads it in P1)
                    //   P2: group 0 over the second half; group 1 over the first half
                    //   P3: group 0 runs its epilogue into the first half; group 1 over the
                    //       second half
                    // Every accumulator sums its k-blocks in natural order.
                    constexpr int RG = C::RPG;
                    // FP8 models: the last hidden layer writes BF16, two bytes per feature, whose
                    // first half would cover the FP8 second half that group 1 still reads in P3.
                    // Its outputs are therefore stored with the two halves swapped (row tile
                    // T -> T ^ NT/2) and layer 5 reads k-block kb from position kb ^ NKB5/2.
                    constexpr int XT = (C::PH != C::P5) ? C::NT / 2 : 0;
                    constexpr int SW5 = (C::PH != C::P5) ? C::NKB5 / 2 : 0;
                    const int wg = wave & 3;
                    const int TB = tb;                                // first row tile of this wave
                    f32x16 acc[RG][C::CT];
                    // SiLU epilogue of accumulator tiles a[r][c] (row tile T0 + r, column tile c0 + c)
                    // into the activation tile, row tile index xor xt
                    auto drain_tiles = [&](auto POC, auto &a, int T0, int c0, float osc, float inv, int xt) {
                        constexpr int PO = decltype(POC)::value;
                        using A = std::remove_reference_t<decltype(a)>;
                        constexpr int RX = std::extent_v<A, 0>, CX = std::extent_v<A, 1>;
                        drain_pipe<PO, C::SCALE, RX * CX>(
                            [&](auto I) {
                                constexpr int i = decltype(I)::value;
                                return a[(i / 16) / CX][(i / 16) % CX][i % 16];
                            },
                            osc, inv,
                            [&](auto TT, const uint32_t *wd) {
                                constexpr int tt = decltype(TT)::value;
                                store_tile<PO>(wd, (T0 + tt / CX) ^ xt, c0 + tt % CX, act, C::ACT_STRIDE, lane);
                            });
                    };
                    auto drain = [&](auto POC, float osc, float inv, int xt = 0) {
                        const int lane = here();
                        constexpr int PO = decltype(POC)::value;
                        drain_pipe<PO, C::SCALE, RG * C::CT>(
                            [&](auto I) {
                                constexpr int i = decltype(I)::value;
                                return acc[(i / 16) / C::CT][(i / 16) % C::CT][i % 16];
                            },
                            osc, inv,
                            [&](auto TT, const uint32_t *wd) {
                                constexpr int tt = decltype(TT)::value;
                                store_tile<PO>(wd, (TB + tt / C::CT) ^ xt, tt % C::CT, act, C::ACT_STRIDE, lane);
                            });
                    };
                    // layer 1 (10 -> H): both groups multiply their own rows; group 0 writes them now,
                    // group 1 during the first hidden layer's P1.  FP8 models (whose epilogue has
                    // the most vector work) split group 0's rows between the two waves of each SIMD
                    // instead: group 1 recomputes the second half of them (a single k-block of
                    // MFMAs) and runs that half's epilogue.
                    auto layer1 = [&] {
                        static_assert(C::NKB1 == 1, "layer 1 is one k-block");
                        init_bias_lds<RG, C::CT>(acc, biases, TB, lane);
                        const char *sb = in0 + (lane & 31) * C::IN_STRIDE + (lane >> 5) * 16;
#pragma unroll
                        for (int c = 0; c < C::CT; ++c) {
                            const Frag1 b = Mma<C::P1>::load_s(sb + c * 32 * C::IN_STRIDE);
#pragma unroll
                            for (int r = 0; r < RG; ++r) Mma<C::P1>::run(acc[r][c], first[r], b, 127);
                        }
                    };
                    if constexpr (MP != kFP8 || C::CT < 4) {
                        layer1();
                        if constexpr (grp == 0) drain(std::integral_constant<int, C::PH>{}, p.oscale[0], p.inv_in_scale[1]);
                    } else {
                        constexpr int RS = RG >= 2 ? RG / 2 : 1;       // row tiles of each share
                        constexpr int CS = RG >= 2 ? 4 : 2;            // column tiles of each share
                        constexpr int R_OFF = RG >= 2 ? RG / 2 : 0, C_OFF = RG >= 2 ? 0 : 2;
                        const Rsrc w0 = make_rsrc(p.wA[0], p.wA_bytes[0]);
                        f32x16 part[RS][CS];
                        const int TS0 = wg * RG + (grp == 0 ? 0 : R_OFF), CS0 = (grp == 0) ? 0 : C_OFF;
                        if constexpr (grp != 0) layer1();
                        init_bias_lds<RS, CS>(part, biases, TS0, lane);
                        mma_seq<C::P1, RS, CS, C::NKB1, C::NKB1, MapAll>(part, w0, TS0, in0, C::IN_STRIDE, CS0, lane,
                                                                         [](auto) {});
                        drain_tiles(std::integral_constant<int, C::PH>{}, part, TS0, CS0, p.oscale[0],
                                    p.inv_in_scale[1], 0);
                    }
                    __syncthreads();
                    auto hidden = [&](int l, auto OUTP) {
                        const int ln = l < 3 ? l + 1 : 1;
                        const Rsrc wl = make_rsrc(p.wA[l], p.wA_bytes[l]), wn = make_rsrc(p.wA[ln], p.wA_bytes[ln]);
                        const int sc = (C::PH == kFP8) ? p.mscale[l] : 127;
                        constexpr int NJ = C::NJ, D = C::RING;
                        auto products0 = [&] {
                            const int lane = here();
                            init_bias_lds<RG, C::CT>(acc, biases + l * H, TB, lane);
                            mma_ring<C::PH, RG, C::CT, NJ, D>(acc, ring, act, C::ACT_STRIDE, 0, 0, lane, sc, [&](auto J) {
                                constexpr int j = decltype(J)::value;
                                load_hidden(ring[j % D], wl, j + D);
                            });
                        };
                        auto products1 = [&] {
                            const int lane = here();
                            mma_ring<C::PH, RG, C::CT, NJ, D>(acc, ring, act, C::ACT_STRIDE, NJ, 0, lane, sc, [&](auto J) {
                                constexpr int j = decltype(J)::value;
                                if constexpr (j + D < NJ) load_hidden(ring[j % D], wl, NJ + j + D);
                                else load_hidden(ring[j % D], wn, j + D - NJ);
                            });
                        };
                        if constexpr (grp == 0) products0();
                        else drain(std::integral_constant<int, C::PH>{}, p.oscale[l - 1], p.inv_in_scale[l]);
                        __syncthreads();
                        if constexpr (grp == 0) products1();
                        else products0();
                        __syncthreads();
                        if constexpr (grp == 0)
                            drain(OUTP, p.oscale[l], (l < 3) ? p.inv_in_scale[l + 1] : 1.0f,
                                  decltype(OUTP)::value != C::PH ? XT : 0);
                        else
                            products1();
                        __syncthreads();
                    };
                    constexpr int NSAME = (C::PH == C::P5) ? 3 : 2;
#pragma unroll 1
                    for (int l = 1; l <= NSAME; ++l) hidden(l, std::integral_constant<int, C::PH>{});
                    if constexpr (NSAME == 2) hidden(3, std::integral_constant<int, C::P5>{});
                    // layer 5 (5 x H): group 0 wave w owns sample column tile w (with small tiles the
                    // waves beyond the last one repeat it); group 1 writes its layer-4 rows meanwhile.
                    // A k-block is one product of a single chain, and no time to load the next one in:
                    // eight k-blocks of fragments are on their way, the second half's before the barrier.
                    constexpr int N5 = C::NKB5 / 2, D5 = N5 < 8 ? N5 : 8;
                    using Frag5 = typename Mma<C::P5>::Frag;
                    f32x16 out[1][1];
                    Frag5 w5[D5][1];
                    const Rsrc w4 = make_rsrc(p.wA[4], p.wA_bytes[4]);
                    auto load5 = [&](int kb) {
                        return Mma<C::P5>::load_g(w4, lane * frag_bytes(C::P5), kb * 64 * frag_bytes(C::P5));
                    };
                    const int wc = C::CT == 4 || wg < C::CT ? wg : C::CT - 1;
                    if constexpr (grp == 0) {
                        sfor<D5>([&](auto J) { w5[decltype(J)::value][0] = load5(decltype(J)::value); });
                        init_bias_lds<1, 1>(out, biases + 4 * H, 0, lane);
                        mma_ring<C::P5, 1, 1, N5, D5, SW5>(out, w5, act, C::ACT_STRIDE, 0, wc, lane, 127, [&](auto J) {
                            w5[decltype(J)::value % D5][0] = load5(D5 + decltype(J)::value);
                        });
                    } else {
                        drain(std::integral_constant<int, C::P5>{}, p.oscale[3], 1.0f, XT);
                    }
                    load_first();
                    __syncthreads();
                    if constexpr (grp == 0) {
                        mma_ring<C::P5, 1, 1, N5, D5, SW5>(out, w5, act, C::ACT_STRIDE, N5, wc, lane, 127, [&](auto J) {
                            constexpr int k = decltype(J)::value;
                            if constexpr (k + D5 < N5) w5[k % D5][0] = load5(N5 + D5 + k);
                        });
                    }
                    if (grp == 0 && (C::CT == 4 || wg < C::CT)) {
                        const int sn = wg * 32 + (lane & 31);
                        if constexpr (!rk4) {
                            // x += dt v, then the next input row's x (and t) in BF16
                            char *row = in0 + sn * C::IN_STRIDE;
                            if (lane < 32) {
                                float x[4];
#pragma unroll
                                for (int d = 0; d < 4; ++d) {
                                    x[d] = xs[d * TM + sn] + out[0][0][d] * dt;
                                    xs[d * TM + sn] = x[d];
                                }
                                *(u32x2 *)row = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
                            } else {
                                const float x4 = xs[4 * TM + sn] + out[0][0][0] * dt;
                                xs[4 * TM + sn] = x4;
                                *(uint32_t *)(row + 8) = pack_bf16(x4, (float)(e + 1) * dt);
                            }
                        } else {
                            // RK4 (the arithmetic of advance): stages 0..2 add v to the stage sum
                            // and give the next stage's input, stage 3 finishes the step; then the
                            // next input row's x (and t) in BF16
                            auto update = [&](int d, float v) {
                                const int o = d * TM + sn;
                                if (stage < 3) {
                                    ksum[o] = stage == 0 ? v : ksum[o] + 2.0f * v;
                                    return xs[o] + (stage == 2 ? dt : 0.5f * dt) * v;
                                }
                                return xs[o] = xs[o] + (dt * (1.0f / 6.0f)) * (ksum[o] + v);
                            };
                            const int e1 = e + 1, st1 = e1 & 3;
                            const float t1 = ((float)(e1 >> 2) + (st1 == 0 ? 0.0f : (st1 == 3 ? 1.0f : 0.5f))) * dt;
                            char *row = in0 + sn * C::IN_STRIDE;
                            if (lane < 32) {
                                float x[4];
#pragma unroll
                                for (int d = 0; d < 4; ++d) x[d] = update(d, out[0][0][d]);
                                *(u32x2 *)row = u32x2{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])};
                            } else {
                                const float x4 = update(4, out[0][0][0]);
                                *(uint32_t *)(row + 8) = pack_bf16(x4, t1);
                            }
                        }
                    }
                    __syncthreads();
                    continue;
                }

                if constexpr (C::PIPE) {
                    // Cross-layer pipeline.  X holds a layer's first row pass, Y its second.  Each
                    // layer's second-pass epilogue runs inside the next layer's MFMA loop over the
                    // k-blocks holding first-pass outputs (already in LDS); its results are stored
                    // and the remaining k-blocks follow after a barrier.
                    constexpr int RP = C::RP, CT = C::CT;
                    f32x16 X[RP][CT], Y[RP][CT];
                    uint32_t pk[RP * CT * 4 * words_per_unit(kF32)];
                    const Rsrc w0 = make_rsrc(p.wA[0], p.wA_bytes[0]), b0 = make_rsrc(p.bias[0], p.bias_bytes[0]);
                    init_bias<RP, CT>(X, b0, TX, lane);
                    mma_seq<kF32, RP, CT, C::NKB1, C::NKB1, MapAll>(X, w0, TX, in0, C::IN_STRIDE, 0, lane, [](auto) {});
                    init_bias<RP, CT>(Y, b0, TY, lane);
                    mma_seq<kF32, RP, CT, C::NKB1, C::NKB1, MapAll>(Y, w0, TY, in0, C::IN_STRIDE, 0, lane, [&](auto J) {
                        drain_step<C::NKB1, decltype(J)::value>(X, pk);
                    });
                    store_pass<RP, CT>(pk, TX, act, C::ACT_STRIDE, lane);
                    __syncthreads();
#pragma unroll 1
                    for (int l = 1; l <= 3; ++l) {
                        const Rsrc wl = make_rsrc(p.wA[l], p.wA_bytes[l]), bl = make_rsrc(p.bias[l], p.bias_bytes[l]);
                        init_bias<RP, CT>(X, bl, TX, lane);
                        mma_seq<kF32, RP, CT, C::NKBH, C::NKBH / 2, MapHalf0<C::GH>>(
                            X, wl, TX, act, C::ACT_STRIDE, 0, lane, [&](auto J) {
                                drain_step<C::NKBH / 2, decltype(J)::value>(Y, pk);
                            });
                        store_pass<RP, CT>(pk, TY, act, C::ACT_STRIDE, lane);
                        __syncthreads();
                        mma_seq<kF32, RP, CT, C::NKBH, C::NKBH / 2, MapHalf1<C::GH>>(
                            X, wl, TX, act, C::ACT_STRIDE, 0, lane, [](auto) {});
                        init_bias<RP, CT>(Y, bl, TY, lane);
                        mma_seq<kF32, RP, CT, C::NKBH, C::NKBH, MapAll>(
                            Y, wl, TY, act, C::ACT_STRIDE, 0, lane, [&](auto J) {
                                drain_step<C::NKBH, decltype(J)::value>(X, pk);
                            });
                        __syncthreads();
                        store_pass<RP, CT>(pk, TX, act, C::ACT_STRIDE, lane);
                        __syncthreads();
                    }
                    // layer 5 (5 x H, rows padded to one tile) over the first-pass k-blocks while
                    // layer 4's second pass drains; wave w < CT owns sample column tile w, further
                    // waves only drain
                    f32x16 out[1][1];
                    const Rsrc w4 = make_rsrc(p.wA[4], p.wA_bytes[4]);
                    auto drain4 = [&](auto J) { drain_step<C::NKB5 / 2, decltype(J)::value>(Y, pk); };
                    if (C::W == CT || wave < CT) {
                        init_bias<1, 1>(out, make_rsrc(p.bias[4], p.bias_bytes[4]), 0, lane);
                        mma_seq<kF32, 1, 1, C::NKB5, C::NKB5 / 2, MapHalf0<C::G5>>(
                            out, w4, 0, act, C::ACT_STRIDE, wave, lane, drain4);
                    } else {
                        sfor<C::NKB5 / 2>(drain4);
                    }
                    store_pass<RP, CT>(pk, TY, act, C::ACT_STRIDE, lane);
                    __syncthreads();
                    if (C::W == CT || wave < CT) {
                        mma_seq<kF32, 1, 1, C::NKB5, C::NKB5 / 2, MapHalf1<C::G5>>(
                            out, w4, 0, act, C::ACT_STRIDE, wave, lane, [](auto) {});
                        const int sn = wave * 32 + (lane & 31);
                        if (lane < 32) {
#pragma unroll
                            for (int d = 0; d < 4; ++d) emit(d, sn, out[0][0][d]);
                        } else {
                            emit(4, sn, out[0][0][0]);
                        }
                    }
                    __syncthreads();
                    continue;
                }

                // layer 1: 10 -> H (reads in0, writes the activation tile: no barrier before writing)
                dense_silu<C::RTW, C::CT, C::NKB1, false>(
                    make_rsrc(p.wA[0], p.wA_bytes[0]), make_rsrc(p.bias[0], p.bias_bytes[0]), T0, in0, C::IN_STRIDE, act,
                    C::ACT_STRIDE, lane);
                __syncthreads();
                // hidden layers 2..4: H -> H, in place
#pragma unroll 1
                for (int l = 1; l <= 3; ++l) {
                    dense_silu<C::RTW, C::CT, C::NKBH, true>(
                        make_rsrc(p.wA[l], p.wA_bytes[l]), make_rsrc(p.bias[l], p.bias_bytes[l]), T0,
                        act, C::ACT_STRIDE, act, C::ACT_STRIDE, lane);
                    __syncthreads();
                }
                // layer 5: H -> 5 (rows padded to 32); wave w handles sample column tile w
                if (C::W == C::CT || wave < C::CT) {
                    f32x16 out[1][1];
                    init_bias<1, 1>(out, make_rsrc(p.bias[4], p.bias_bytes[4]), 0, lane);
                    mma_pass<kF32, 1, 1, C::NKB5>(out, make_rsrc(p.wA[4], p.wA_bytes[4]), 0, act,
                                                   C::ACT_STRIDE, wave, lane, [](auto) {});
                    const int sn = wave * 32 + (lane & 31);
                    if (lane < 32) {
#pragma unroll
                        for (int d = 0; d < 4; ++d) emit(d, sn, out[0][0][d]);
                    } else {
                        emit(4, sn, out[0][0][0]);
                    }
                }
                __syncthreads();
            }

            if ((!C::GROUPS || grp == 0) && tid < TM) {
                const int64_t i = base + tid;
                float xk[5];
                if constexpr (rk4 && !C::GROUPS) {
                    advance(nevals - 1, xk);
                } else {
#pragma unroll
                    for (int d = 0; d < 5; ++d) xk[d] = xs[d * TM + tid];
                }
                if (i < n_items) {
                    const float a0 = xk[0], a1 = xk[1], a2 = xk[2], a3 = xk[3], a4 = xk[4];
                    if (p.raw) {
                        p.raw[0 * p.n + i] = a0;
                        p.raw[1 * p.n + i] = a1;
                        p.raw[2 * p.n + i] = a2;
                        p.raw[3 * p.n + i] = a3;
                        p.raw[4 * p.n + i] = a4;
                    }
                    Exit e;
                    decode_exit(a0, a1, a2, a3, a4, e, p.xy != 0);
                    p.face[i] = e.face;
                    p.pos[i] = e.pos;
                    p.dcos[i] = e.u;
                    p.dsin[i] = e.v;
                    p.path[i] = e.path;
                }
            }
            __syncthreads();
        }
    };
    if constexpr (C::GROUPS) {
        if (wave < 4) tiles(std::integral_constant<int, 0>{});
        else tiles(std::integral_constant<int, 1>{});
    } else {
        tiles(std::integral_constant<int, 0>{});
    }
}

// Width 128 with BF16 or FP8 operands: a wave carries 32 samples through all evaluations by
// itself.  The accumulator values lane (n, h) holds of a layer are the operand values lane (n, h)
// reads for the next one (phys_to_feature), so with all of a layer's rows in one wave the
// activations never leave its registers: no activation tile, no barrier, and the state of the ODE
// stays in registers too.  The weights of all layers (BF16 108 KB) are copied into LDS once per
// workgroup, of which a CU holds one with three waves to a SIMD.  Bound by the SiLU (two
// transcendentals of 8 cycles an activation, 26 cycles with the rest: 6.7k cycles per 32 samples and
// evaluation against 3.5k of matrix work; vector units busy 84 % of a full launch), so a layer's
// two pairs of row tiles, X and Y, take turns: Y's products run in the iterations of X's SiLU, and
// the next layer's X over the k-blocks that X gave in those of Y's.
// Measured, against four waves to 128 samples with the activations in LDS (three such workgroups
// to a CU): BF16 RK4 x 12, 2^20 samples 7.33 -> 6.27 ms, 2^18 1.77 -> 1.59 ms, 1,000 343 -> 224 us;
// FP8 Euler K = 16, 2^20 samples 2.52 -> 2.01 ms.  (Two waves to a SIMD: 6.43 ms; without the
// products in the SiLU's iterations: 6.87 ms; the biases read from memory: 6.45 ms.)
template <int MP>
struct WaveCfg {
    static constexpr int H = 128;
    static constexpr int PH = layer_prec(MP, 1), P5 = layer_prec(MP, 4);
    static constexpr bool SCALE = (MP == kFP8);
    static constexpr int NT = H / 32;
    static constexpr int NKBH = H / kb_width(PH), NKB5 = H / kb_width(P5);
    static constexpr int W = 12, THREADS = 64 * W;
    static constexpr int TILE = 64 * 16;                       // one fragment line of 64 lanes
    static constexpr int LDS_1 = NT * TILE;                    // layer 1: one BF16 k-block
    static constexpr int LDS_H = NT * NKBH * 64 * frag_bytes(PH);
    static constexpr int LDS_5 = NKB5 * TILE;
    static constexpr int OFF_H = LDS_1, OFF_5 = LDS_1 + 3 * LDS_H, OFF_B = OFF_5 + LDS_5;
    static constexpr int LDS_BYTES = OFF_B + (4 * H + 32) * 4;
};

// Lane n + 32's value in lane n.
__device__ __forceinline__ float upper_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x),
                                                    false, false);
    return __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Layer 1's operand of 32 samples in one wave: the input row [x0..x4, t, cf0..cf5, 0 x 4], of which
// lanes 0-31 hold features 0-7 and lanes 32-63 features 8-15; of the state xi lanes 0-31 hold x0..x3
// and lanes 32-63 x4 (as the output layer's rows fall).  c01, c23, c45: the condition in pairs.
__device__ __forceinline__ u32x4 wave_input(const float (&xi)[4], float t, uint32_t c01, uint32_t c23, uint32_t c45,
                                            int half)
{
    const uint32_t x4t = pack_bf16(upper_half(xi[0]), t);
    return half ? u32x4{c23, c45, 0u, 0u} : u32x4{pack_bf16(xi[0], xi[1]), pack_bf16(xi[2], xi[3]), x4t, c01};
}

// x <- x + dt v, or the RK4 stage (as in mlp_ode_kernel); xi: the next evaluation's input.
template <bool rk4>
__device__ __forceinline__ void wave_update(float (&x)[4], float (&xi)[4], float (&ks)[4], const f32x16 &out, int stage,
                                            float dt)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const float v = out[d];
        if constexpr (!rk4) {
            x[d] += v * dt;
            xi[d] = x[d];
        } else if (stage < 3) {
            ks[d] = stage == 0 ? v : ks[d] + 2.0f * v;
            xi[d] = x[d] + (stage == 2 ? dt : 0.5f * dt) * v;
        } else {
            xi[d] = x[d] = x[d] + (dt * (1.0f / 6.0f)) * (ks[d] + v);
        }
    }
}

// Four packed words as a BF16 operand fragment.
template <typename F>
__device__ __forceinline__ void put16(F &f, const uint32_t *w)
{
    if constexpr (std::is_same_v<F, u32x4>) f = u32x4{w[0], w[1], w[2], w[3]};
}

template <int MP, int RK>
__global__ __launch_bounds__((WaveCfg<MP>::THREADS), WaveCfg<MP>::W / 4) void mlp_wave_kernel(MlpParams p)
{
    using C = WaveCfg<MP>;
    using M1 = Mma<kBF16>;
    using MH = Mma<C::PH>;
    constexpr bool rk4 = (RK == 1);
    static_assert(C::LDS_BYTES <= 160 * 1024, "LDS budget");
    __shared__ __attribute__((aligned(16))) char smem[C::LDS_BYTES];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;

    const int64_t n_items = p.n_dev ? (int64_t)*p.n_dev : p.n;
    if (n_items == 0) return;                              // taken by the teams
    // weights and biases to LDS; FP8 fragments (32 bytes a lane) as two lines of 16-byte halves
    auto copy = [&](int off, const void *src, int bytes) {
        for (int b = tid * 16; b < bytes; b += C::THREADS * 16)
            *(u32x4 *)(smem + off + b) = *(const u32x4 *)((const char *)src + b);
    };
    copy(0, p.wA[0], C::LDS_1);
    for (int l = 0; l < 3; ++l) {
        if constexpr (C::PH == kFP8) {
            for (int q = tid; q < C::LDS_H / 16; q += C::THREADS) {
                const int line = q >> 7, in = q & 127;         // source: lane in / 2, half in % 2
                *(u32x4 *)(smem + C::OFF_H + l * C::LDS_H + line * 2048 + (in & 1) * 1024 + (in >> 1) * 16) =
                    *(const u32x4 *)((const char *)p.wA[1 + l] + q * 16);
            }
        } else {
            copy(C::OFF_H + l * C::LDS_H, p.wA[1 + l], C::LDS_H);
        }
    }
    copy(C::OFF_5, p.wA[4], C::LDS_5);
    for (int l = 0; l < 4; ++l) copy(C::OFF_B + l * C::H * 4, p.bias[l], C::H * 4);
    copy(C::OFF_B + 4 * C::H * 4, p.bias[4], 32 * 4);
    __syncthreads();

    const int64_t ntiles = (n_items + 31) / 32;
    const float dt = 1.0f / (float)p.K;
    const int nevals = rk4 ? 4 * p.K : p.K;
    int at_lane = lane * 16, at_half = half * 16;     // offsets of this lane in a line, in a bias row
    const char *frag = smem + at_lane;
    auto load_h = [&](int l, int T, int kb) {
        const char *f = frag + C::OFF_H + l * C::LDS_H + (T * C::NKBH + kb) * 64 * frag_bytes(C::PH);
        if constexpr (C::PH == kFP8) return MH::cat(*(const u32x4 *)f, *(const u32x4 *)(f + 1024));
        else return *(const u32x4 *)f;
    };
    auto load_bias = [&](int off) {          // the accumulator's start for one row tile
        const float *b = (const float *)(smem + C::OFF_B + at_half) + off;
        f32x16 v;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 q = *(const f32x4 *)(b + 8 * g);
            v[4 * g + 0] = q.x;
            v[4 * g + 1] = q.y;
            v[4 * g + 2] = q.z;
            v[4 * g + 3] = q.w;
        }
        return v;
    };
    for (int64_t tile = (int64_t)wave * gridDim.x + blockIdx.x; tile < ntiles; tile += (int64_t)gridDim.x * C::W) {
        const int64_t i = tile * 32 + (lane & 31);
        float z[5], cf[6];
        sampler_inputs(p, i, n_items, z, cf);
        const uint32_t c01 = pack_bf16(cf[0], cf[1]), c23 = pack_bf16(cf[2], cf[3]), c45 = pack_bf16(cf[4], cf[5]);
        float x[4], ks[4], xi[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            x[d] = half ? (d == 0 ? z[4] : 0.0f) : z[d];
            xi[d] = x[d];
            ks[d] = 0.0f;
        }
#pragma unroll 1
        for (int e = 0; e < nevals; ++e) {
            // the weights do not change from one evaluation to the next: keep the compiler from
            // loading them ahead of the loop, for which there are no registers
            asm volatile("" : "+v"(at_lane), "+v"(at_half));
            frag = smem + at_lane;
            const int stage = rk4 ? (e & 3) : 0;
            const int k = rk4 ? (e >> 2) : e;
            const float t = ((float)k + (stage == 0 ? 0.0f : (stage == 3 ? 1.0f : 0.5f))) * dt;
            const u32x4 in = wave_input(xi, t, c01, c23, c45, half);
            f32x16 X[2], Y[2], out;
            typename MH::Frag B[2][C::NKBH];          // operands of the layer read, of the one written
            u32x4 b5[C::NKB5];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                X[r] = load_bias(32 * r);
                Y[r] = load_bias(64 + 32 * r);
                M1::run(X[r], *(const u32x4 *)(frag + r * C::TILE), in, 127);
                M1::run(Y[r], *(const u32x4 *)(frag + (2 + r) * C::TILE), in, 127);
            }
            // packed words of row tile T to the operands of the layer that reads them
            auto put = [&](auto PO, auto SLOT, auto TT, const uint32_t *w) {
                constexpr int T = decltype(TT)::value, q = decltype(SLOT)::value;
                if constexpr (decltype(PO)::value == kBF16 && C::PH == kBF16 && q < 2) {
                    put16(B[q][2 * T], w);
                    put16(B[q][2 * T + 1], w + 4);
                } else if constexpr (decltype(PO)::value == kBF16) {
                    put16(b5[2 * T], w);
                    put16(b5[2 * T + 1], w + 4);
                } else {
#pragma unroll
                    for (int m = 0; m < 4; ++m) B[q][T / 2][4 * (T % 2) + m] = (int)w[m];
                }
            };
            // the products of hidden layer l, row tiles T0 and T0 + 1, over k-blocks K0 .. K1 - 1, as a
            // list of 2 (K1 - K0): fragments are read PF places ahead
            constexpr int PF = C::PH == kFP8 ? 2 : 4;
            typename MH::Frag a[PF];
            auto fetch = [&](auto L, auto T0, auto K0, auto M) {
                constexpr int m = decltype(M)::value;
                a[m % PF] = load_h(decltype(L)::value, decltype(T0)::value + m % 2, decltype(K0)::value + m / 2);
            };
            auto product = [&](f32x16 (&acc)[2], auto L, auto Q, auto T0, auto K0, auto K1, auto M) {
                constexpr int m = decltype(M)::value, n = 2 * (decltype(K1)::value - decltype(K0)::value);
                if constexpr (m < n) {
                    const int sc = (C::PH == kFP8) ? p.mscale[1 + decltype(L)::value] : 127;
                    MH::run(acc[m % 2], a[m % PF], B[decltype(Q)::value][decltype(K0)::value + m / 2], sc);
                    if constexpr (m + PF < n) fetch(L, T0, K0, std::integral_constant<int, m + PF>{});
                }
            };
            using I0 = std::integral_constant<int, 0>;
            using I2 = std::integral_constant<int, 2>;
            using KH = std::integral_constant<int, C::NKBH / 2>;
            using KN = std::integral_constant<int, C::NKBH>;
            constexpr int STEPS = 32 + 4 * kPipeD, LEAD = 4;   // iterations of a pair's SiLU
            // SiLU of the pair `src` (row tiles T0, T0 + 1) with a list of n products in its iterations
            auto silu_pair = [&](f32x16 (&src)[2], auto PO, auto SLOT, auto T0, float osc, float inv, auto N, auto &&run) {
                constexpr int n = decltype(N)::value, every = (STEPS - LEAD) / (n > 0 ? n : 1);
                drain_pipe<decltype(PO)::value, C::SCALE, 2>(
                    [&](auto I) { return src[decltype(I)::value / 16][decltype(I)::value % 16]; }, osc, inv,
                    [&](auto TT, const uint32_t *w) {
                        put(PO, SLOT, std::integral_constant<int, decltype(T0)::value + decltype(TT)::value>{}, w);
                    },
                    [&](auto J) {
                        constexpr int j = decltype(J)::value - LEAD;
                        if constexpr (n > 0 && j >= 0 && j % every == 0 && j / every < n)
                            run(std::integral_constant<int, j / every>{});
                    });
            };
            using PHC = std::integral_constant<int, C::PH>;
            silu_pair(X, PHC{}, I0{}, I0{}, p.oscale[0], p.inv_in_scale[1], I0{}, [](auto) {});
            sfor<3>([&](auto L) {
                constexpr int l = decltype(L)::value;
                using Q = std::integral_constant<int, l % 2>;                       // operands read
                using R = std::integral_constant<int, l == 2 ? 2 : (l + 1) % 2>;    // and written
                using PO = std::integral_constant<int, l == 2 ? C::P5 : C::PH>;
                // the previous layer's Y, with X over the first half of the k-blocks
#pragma unroll
                for (int r = 0; r < 2; ++r) X[r] = load_bias(C::H * (1 + l) + 32 * r);
                sfor<PF>([&](auto M) { if constexpr (decltype(M)::value < C::NKBH) fetch(L, I0{}, I0{}, M); });
                silu_pair(Y, PHC{}, Q{}, I2{}, p.oscale[l], p.inv_in_scale[1 + l], KN{},
                          [&](auto M) { product(X, L, Q{}, I0{}, I0{}, KH{}, M); });
                sfor<PF>([&](auto M) { if constexpr (decltype(M)::value < C::NKBH) fetch(L, I0{}, KH{}, M); });
#pragma unroll
                for (int r = 0; r < 2; ++r) Y[r] = load_bias(C::H * (1 + l) + 64 + 32 * r);
                sfor<C::NKBH>([&](auto M) {
                    product(X, L, Q{}, I0{}, KH{}, KN{}, M);
                    __builtin_amdgcn_sched_barrier(0);
                });
                // X, with Y over all k-blocks
                sfor<PF>([&](auto M) { fetch(L, I2{}, I0{}, M); });
                silu_pair(X, PO{}, R{}, I0{}, p.oscale[1 + l], l < 2 ? p.inv_in_scale[2 + l] : 1.0f,
                          std::integral_constant<int, 2 * C::NKBH>{},
                          [&](auto M) { product(Y, L, Q{}, I2{}, I0{}, KN{}, M); });
            });
            // the last Y, with the output layer over the first half
            out = load_bias(4 * C::H);
            auto last = [&](auto KB) {
                constexpr int kb = decltype(KB)::value;
                M1::run(out, *(const u32x4 *)(frag + C::OFF_5 + kb * C::TILE), b5[kb], 127);
            };
            silu_pair(Y, std::integral_constant<int, C::P5>{}, I2{}, I2{}, p.oscale[3], 1.0f,
                      std::integral_constant<int, C::NKB5 / 2>{}, last);
            sfor<C::NKB5 / 2>([&](auto M) { last(std::integral_constant<int, C::NKB5 / 2 + decltype(M)::value>{}); });
            wave_update<rk4>(x, xi, ks, out, stage, dt);
        }
        const float x4 = upper_half(x[0]);
        if (half == 0 && i < n_items) {
            const float xk[5] = {x[0], x[1], x[2], x[3], x4};
            sampler_outputs(p, i, xk);
        }
    }
}

// The same network and arithmetic for launches of few tiles, where a wave by itself (mlp_wave_kernel)
// takes as long as its 256 activations a lane in sequence: a team of four waves, one to a SIMD,
// shares 32 samples.  Wave T holds the fragments of row tile T of every layer in registers (BF16
// 132), so nothing is loaded in the loop; a layer's packed outputs pass through LDS in operand
// order, two buffers in turn, with one barrier a layer; the output layer and the state's update
// run in all four waves alike, so the state is not exchanged.  Bound by latency (a layer's eight
// products of one chain, 16 activations, the exchange).
// Measured, RK4 x 12, a wave each -> a team: 1,000 samples BF16 227 -> 112 us, FP8 222 -> 104; 8,192
// BF16 233 -> 120; 16,384 (two teams to a CU) BF16 237 -> 158, FP8 225 -> 155.  The lattice of 200,000
// particles, whose late steps hold few: 16.0 -> 14.0 ms.
template <int MP, int RK>
__global__ __launch_bounds__(256, 2) void mlp_team_kernel(MlpParams p)
{
    using C = WaveCfg<MP>;
    using M1 = Mma<kBF16>;
    using MH = Mma<C::PH>;
    constexpr bool rk4 = (RK == 1);
    constexpr int EX = 8 * 64 * 16;                        // one buffer: 128 BF16 values of 32 samples
    __shared__ __attribute__((aligned(16))) char ex[2 * EX];
    __shared__ __attribute__((aligned(16))) float biases[4 * C::H + 32];
    const int tid = threadIdx.x, T = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5;

    const int64_t n_items = p.n_dev ? (int64_t)*p.n_dev : p.n;
    if (p.n_dev_large) {
        const bool large = n_items > p.small_max;
        if (blockIdx.x == 0 && tid == 0) *p.n_dev_large = large ? (unsigned long long)n_items : 0ull;
        if (large) return;
    }
    const int64_t ntiles = (n_items + 31) / 32;
    if (blockIdx.x >= ntiles) return;
    const float dt = 1.0f / (float)p.K;
    const int nevals = rk4 ? 4 * p.K : p.K;
    for (int l = 0; l < 4; ++l)
        if (tid < C::H) biases[l * C::H + tid] = p.bias[l][tid];
    if (tid < 32) biases[4 * C::H + tid] = p.bias[4][tid];
    u32x4 w1 = M1::load_g(make_rsrc(p.wA[0], p.wA_bytes[0]), lane * 16, T * C::TILE);
    typename MH::Frag wh[3][C::NKBH];
    u32x4 w5[C::NKB5];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        const Rsrc w = make_rsrc(p.wA[1 + l], p.wA_bytes[1 + l]);
#pragma unroll
        for (int kb = 0; kb < C::NKBH; ++kb)
            wh[l][kb] = MH::load_g(w, lane * frag_bytes(C::PH), (T * C::NKBH + kb) * 64 * frag_bytes(C::PH));
    }
    {
        const Rsrc w = make_rsrc(p.wA[4], p.wA_bytes[4]);
#pragma unroll
        for (int kb = 0; kb < C::NKB5; ++kb) w5[kb] = M1::load_g(w, lane * 16, kb * C::TILE);
    }
    __syncthreads();
    auto load_bias = [&](int off) {          // the accumulator's start for one row tile
        const float *b = biases + off + 4 * half;
        f32x16 v;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 q = *(const f32x4 *)(b + 8 * g);
            v[4 * g + 0] = q.x;
            v[4 * g + 1] = q.y;
            v[4 * g + 2] = q.z;
            v[4 * g + 3] = q.w;
        }
        return v;
    };
    // SiLU of the row tile to buffer `to`: BF16, its two k-blocks' 16 bytes a lane each; FP8, its half
    // of a k-block's 32 bytes
    auto silu_out = [&](f32x16 &acc, auto PO, char *to, float osc, float inv) {
        drain_pipe<decltype(PO)::value, C::SCALE, 1>(
            [&](auto I) { return acc[decltype(I)::value]; }, osc, inv,
            [&](auto, const uint32_t *w) {
                if constexpr (decltype(PO)::value == kBF16) {
                    *(u32x4 *)(to + 2 * T * C::TILE + lane * 16) = u32x4{w[0], w[1], w[2], w[3]};
                    *(u32x4 *)(to + (2 * T + 1) * C::TILE + lane * 16) = u32x4{w[4], w[5], w[6], w[7]};
                } else {
                    *(u32x4 *)(to + T * C::TILE + lane * 16) = u32x4{w[0], w[1], w[2], w[3]};
                }
            });
    };

    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t i = tile * 32 + (lane & 31);
        float z[5], cf[6];
        sampler_inputs(p, i, n_items, z, cf);
        const uint32_t c01 = pack_bf16(cf[0], cf[1]), c23 = pack_bf16(cf[2], cf[3]), c45 = pack_bf16(cf[4], cf[5]);
        float x[4], ks[4], xi[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            x[d] = half ? (d == 0 ? z[4] : 0.0f) : z[d];
            xi[d] = x[d];
            ks[d] = 0.0f;
        }
#pragma unroll 1
        for (int e = 0; e < nevals; ++e) {
            const int stage = rk4 ? (e & 3) : 0;
            const int k = rk4 ? (e >> 2) : e;
            const float t = ((float)k + (stage == 0 ? 0.0f : (stage == 3 ? 1.0f : 0.5f))) * dt;
            const u32x4 in = wave_input(xi, t, c01, c23, c45, half);
            f32x16 acc = load_bias(32 * T);
            M1::run(acc, w1, in, 127);
            silu_out(acc, std::integral_constant<int, C::PH>{}, ex, p.oscale[0], p.inv_in_scale[1]);
            sfor<3>([&](auto L) {
                constexpr int l = decltype(L)::value;
                using PO = std::integral_constant<int, l == 2 ? C::P5 : C::PH>;
                const char *from = ex + (l % 2) * EX + lane * 16;
                acc = load_bias(C::H * (1 + l) + 32 * T);
                const int sc = (C::PH == kFP8) ? p.mscale[1 + l] : 127;
                __syncthreads();
#pragma unroll
                for (int kb = 0; kb < C::NKBH; ++kb) {
                    if constexpr (C::PH == kFP8)
                        MH::run(acc, wh[l][kb],
                                MH::cat(*(const u32x4 *)(from + 2 * kb * C::TILE), *(const u32x4 *)(from + (2 * kb + 1) * C::TILE)), sc);
                    else
                        MH::run(acc, wh[l][kb], *(const u32x4 *)(from + kb * C::TILE), sc);
                }
                silu_out(acc, PO{}, ex + ((l + 1) % 2) * EX, p.oscale[1 + l], l < 2 ? p.inv_in_scale[2 + l] : 1.0f);
            });
            f32x16 out = load_bias(4 * C::H);
            __syncthreads();
#pragma unroll
            for (int kb = 0; kb < C::NKB5; ++kb)
                M1::run(out, w5[kb], *(const u32x4 *)(ex + EX + kb * C::TILE + lane * 16), 127);
            wave_update<rk4>(x, xi, ks, out, stage, dt);
        }
        const float x4 = upper_half(x[0]);
        if (T == 0 && half == 0 && i < n_items) {
            const float xk[5] = {x[0], x[1], x[2], x[3], x4};
            sampler_outputs(p, i, xk);
        }
    }
}

// Launches of at most 64 samples per compute unit (two teams to a CU: 158 us against 237 at 16,384; a
// third round of teams would take longer than the 234 us that a wave each takes up to twelve to a CU)
// run teams; a count known only on the device chooses there, as in launch_one.
template <int MP>
hipError_t launch_wave(const MlpParams &p_in, int cu, hipStream_t s)
{
    using C = WaveCfg<MP>;
    MlpParams p = p_in;
    p.n_dev_large = nullptr;
    const int64_t few = (int64_t)64 * cu;
    if (p.n <= few || p_in.n_dev_large) {
        const bool chain = p.n > few;
        MlpParams q = p;
        q.n_dev_large = chain ? p_in.n_dev_large : nullptr;
        q.small_max = few;
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((p.n + 31) / 32, (int64_t)2 * cu));
        if (p.integrator == 1) hipLaunchKernelGGL((mlp_team_kernel<MP, 1>), dim3(grid), dim3(256), 0, s, q);
        else hipLaunchKernelGGL((mlp_team_kernel<MP, 0>), dim3(grid), dim3(256), 0, s, q);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !chain) return e;
        p.n_dev = p_in.n_dev_large;
    }
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((p.n + 31) / 32, cu));
    if (p.integrator == 1) hipLaunchKernelGGL((mlp_wave_kernel<MP, 1>), dim3(grid), dim3(C::THREADS), 0, s, p);
    else hipLaunchKernelGGL((mlp_wave_kernel<MP, 0>), dim3(grid), dim3(C::THREADS), 0, s, p);
    return hipGetLastError();
}

// grid: one persistent workgroup per tile of a launch of at most `bound` samples, at most one per
// compute unit (whose LDS it fills)
template <int MP, int H, int TM>
hipError_t launch_tiles(const MlpParams &p, int64_t bound, int cu, hipStream_t s)
{
    constexpr int threads = Cfg<MP, H, TM>::THREADS;
    const int64_t ntiles = (bound + TM - 1) / TM;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(ntiles, cu));
    if (p.integrator == 1) hipLaunchKernelGGL((mlp_ode_kernel<MP, H, 1, TM>), dim3(grid), dim3(threads), 0, s, p);
    else hipLaunchKernelGGL((mlp_ode_kernel<MP, H, 0, TM>), dim3(grid), dim3(threads), 0, s, p);
    return hipGetLastError();
}

// The same launch over samples [off, off + cnt) of p: every per-sample array moves by off (the
// [5][n] noise and raw arrays, whose row stride is p.n, are not used with it).
inline MlpParams sample_range(const MlpParams &p, int64_t off, int64_t cnt)
{
    MlpParams q = p;
    auto mv = [off](auto *&ptr) { if (ptr) ptr += off; };
    mv(q.log_tau); mv(q.c); mv(q.y_in); mv(q.sin_th); mv(q.x_in); mv(q.cos_phi);
    mv(q.log_aspect); mv(q.omega_x); mv(q.ids); mv(q.keys);
    mv(q.face); mv(q.pos); mv(q.dcos); mv(q.dsin); mv(q.path);
    if (!p.ids) q.id_base = p.id_base + (uint64_t)off;
    q.n = cnt;
    return q;
}

// Launches with at most kSmallTileM (kMidTileM, kWideTileM) samples per compute unit (the tail steps
// of a transport run, small requests) take 32-sample (64-, 96-sample) tiles: one round of them
// covers the launch on every CU, and a tile's latency falls with its matrix work (an evaluation of
// 32 / 64 / 96 / 128 samples takes 13 / 18 / 29 / 40 us in BF16 at width 512 and 30 / 55 / 79 / 104 us
// in FP32 at width 256).  When only the device knows the count (n_dev) and its bound p.n is larger,
// the choice is made on the device (MlpParams::n_dev_large; between 32, 64 and 128) without a
// read-back; a sample's result is the same with every tile size.  A count known on the host whose
// last round of 128-sample tiles would hold at most 96 samples per CU runs that remainder as one
// round of smaller tiles.
template <int MP, int H>
hipError_t launch_one(const MlpParams &p, int cu, hipStream_t s)
{
    MlpParams q = p;
    q.n_dev_large = nullptr;
    const int64_t small = (int64_t)kSmallTileM * cu, mid = (int64_t)kMidTileM * cu, wide = (int64_t)kWideTileM * cu;
    if (p.n <= small) return launch_tiles<MP, H, kSmallTileM>(q, p.n, cu, s);
    if (!p.n_dev) {
        if (p.n <= mid) return launch_tiles<MP, H, kMidTileM>(q, p.n, cu, s);
        if (p.n <= wide) return launch_tiles<MP, H, kWideTileM>(q, p.n, cu, s);
        const int64_t round = (int64_t)kTileM * cu, rem = p.n % round;
        if (!p.noise && !p.raw && rem > 0 && rem <= wide) {
            const MlpParams head = sample_range(q, 0, p.n - rem);
            const hipError_t e = launch_tiles<MP, H, kTileM>(head, head.n, cu, s);
            if (e != hipSuccess) return e;
            const MlpParams tail = sample_range(q, p.n - rem, rem);
            return rem <= small ? launch_tiles<MP, H, kSmallTileM>(tail, rem, cu, s)
                   : rem <= mid ? launch_tiles<MP, H, kMidTileM>(tail, rem, cu, s)
                                : launch_tiles<MP, H, kWideTileM>(tail, rem, cu, s);
        }
    } else if (p.n_dev_large) {
        // 32-sample kernel, then the 64-sample one, each handing on what it does not take
        q.n_dev_large = p.n_dev_large;
        q.small_max = small;
        hipError_t e = launch_tiles<MP, H, kSmallTileM>(q, small, cu, s);
        if (e != hipSuccess) return e;
        q.n_dev = p.n_dev_large;
        q.n_dev_large = p.n <= mid ? nullptr : p.n_dev_large + 1;
        q.small_max = mid;
        e = launch_tiles<MP, H, kMidTileM>(q, std::min<int64_t>(p.n, mid), cu, s);
        if (e != hipSuccess || p.n <= mid) return e;
        q.n_dev = p.n_dev_large + 1;
        q.n_dev_large = nullptr;
    }
    return launch_tiles<MP, H, kTileM>(q, p.n, cu, s);
}

}  // namespace

bool mlp_supported(int prec, int hidden)
{
    if (prec == kF32) return hidden == 128 || hidden == 256;
    if (prec == kBF16 || prec == kFP8) return hidden == 128 || hidden == 256 || hidden == 512;
    return false;
}

hipError_t launch_mlp_ode(int prec, int hidden, const MlpParams &p, int cu, hipStream_t s)
{
    if (p.net == 1) return launch_film_ode(prec, hidden, p, cu, s);
    switch (prec * 1000 + hidden) {
    case kF32 * 1000 + 128: return launch_one<kF32, 128>(p, cu, s);
    case kF32 * 1000 + 256: return launch_one<kF32, 256>(p, cu, s);
    case kBF16 * 1000 + 128: return launch_wave<kBF16>(p, cu, s);
    case kBF16 * 1000 + 256: return launch_one<kBF16, 256>(p, cu, s);
    case kBF16 * 1000 + 512: return launch_one<kBF16, 512>(p, cu, s);
    case kFP8 * 1000 + 128: return launch_wave<kFP8>(p, cu, s);
    case kFP8 * 1000 + 256: return launch_one<kFP8, 256>(p, cu, s);
    case kFP8 * 1000 + 512: return launch_one<kFP8, 512>(p, cu, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gmc
