// scan_tiled.hpp -- two kernels beside the ring kernel of the forward (dstate 16): the
// scan of a 16-timestep sequence (the verify shape), and the pre-pass over time segments.
//
// Each wavefront works alone: it owns 8 channels of one batch element, and lane
// l = 8 j + q holds channel j's states 2q and 2q+1 of eq. (2) in VGPRs.  In
// scan_fwd_short it
//
//   A  does the per-element work once: lane (j, q) widens u, delta and z of
//      channel j at timesteps 2q and 2q + 1, computes dlt = softplus(delta + dt_bias)
//      (eq. (3)), dx = dlt * u and silu(z) (Table 8), and publishes (dlt, dx) in its
//      private LDS area; the wave also stages the B and C rows there, time-major and
//      widened to fp32;
//   B  runs the recurrence for its two states over the 16 timesteps --
//      abar = 2^(dlt A log2 e) (zero-order hold on A), h = abar h + dx B
//      (simplified Euler on B) -- reading the next four timesteps' operands
//      from LDS while computing the current four, and publishes its partial
//      contraction C_t[2q] h_t[2q] + C_t[2q+1] h_t[2q+1] per timestep;
//   C  lane (j, q) sums channel j's partials at its own timesteps, adds Dskip * u,
//      applies the gate and stores y.
//
// Arithmetic is fp32; the state never leaves VGPRs except through h0 / h_last.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.hpp"
#include "scan_params.hpp"

#include <type_traits>

namespace mbs {
namespace tiled {

constexpr int kN = 16;                // states per channel
constexpr int kCh = 8;                // channels per wave
constexpr int kQ = 8;                 // state pairs per channel (lanes per channel)
constexpr int kT = 32;                // timesteps per chunk of the pre-pass
constexpr int kWavesPerGroup = 4;     // independent waves per workgroup
constexpr int kThreads = kWavesPerGroup * 64;

// 4 consecutive activations of one row, which may start at any element: they are only
// aligned to theirs (the hardware takes such loads).
typedef u32x2 u32x2_e2 __attribute__((aligned(2)));
typedef f32x4 f32x4_e4 __attribute__((aligned(4)));
template <int IN> struct Raw4;
template <> struct Raw4<1> {
    u32x2 v;
    __device__ __forceinline__ void load(const void *base, uint32_t off) {
        v = *reinterpret_cast<const u32x2_e2 *>(static_cast<const char *>(base) + off * 2u);
    }
    __device__ __forceinline__ float get(int i) const {
        const uint32_t w = (i >> 1) ? v.y : v.x;
        return (i & 1) ? bf16_hi(w) : bf16_lo(w);
    }
};
template <> struct Raw4<0> {
    f32x4 v;
    __device__ __forceinline__ void load(const void *base, uint32_t off) {
        v = *reinterpret_cast<const f32x4_e4 *>(static_cast<const char *>(base) + off * 4u);
    }
    __device__ __forceinline__ float get(int i) const { return v[i]; }
};

// 2 consecutive activations of one row (4 bytes bf16, 8 bytes fp32): the
// per-lane share of a 16-timestep sequence.
template <int IN> struct Raw2;
template <> struct Raw2<1> {
    uint32_t v;
    __device__ __forceinline__ void load(const void *base, uint32_t off) {
        v = *reinterpret_cast<const uint32_t *>(static_cast<const char *>(base) + off * 2u);
    }
    __device__ __forceinline__ float get(int i) const { return i ? bf16_hi(v) : bf16_lo(v); }
};
template <> struct Raw2<0> {
    float2 v;
    __device__ __forceinline__ void load(const void *base, uint32_t off) {
        v = *reinterpret_cast<const float2 *>(static_cast<const char *>(base) + off * 4u);
    }
    __device__ __forceinline__ float get(int i) const { return i ? v.y : v.x; }
};

// Private LDS areas of a wave.  A 16-byte write serves 8 consecutive lanes at a time from
// 32 banks (a 128-byte period, measured), and every row write below covers 8 consecutive
// entries or is spread by the pads and the order of rows.
// ShortSmem: the tables of 16 timesteps; 5.6 KB, so that 7 workgroups fit a CU's LDS.
//   dd    row r = timesteps 2r, 2r+1; entry j = (dlt, dx, dlt, dx) of channel j
//   bc    row t; entry q = (B[2q], B[2q+1], C[2q], C[2q+1]) at timestep t
//   part  row 4 j + tq = channel j, timesteps 4 tq .. 4 tq + 3; lanes q and q ^ 1 add their
//         partial outputs in registers first, so a row holds 4 sums (+ 1 pad entry)
constexpr int kDdRow = 9;       // 16-byte entries per row: 8 used + 1 pad
constexpr int kShort = 16;      // timesteps
struct ShortSmem {
    f32x4 dd[kShort / 2][kDdRow];                    // 1.1 KB
    f32x4 bc[kShort][kQ];                            // 2 KB
    f32x4 part[kCh * (kShort / 4)][kQ / 2 + 1];      // 2.5 KB
};
static_assert(sizeof(ShortSmem) * kWavesPerGroup * 7 <= 160 * 1024,
              "seven workgroups of the 16-timestep tables fit the 160 KB of a CU's LDS");

// The row of timestep pair r in the pre-pass's tables: lane q writes pairs 2q and 2q + 1,
// which go to rows q and 8 + q, so that the 8 lanes of a channel write 8 different bank
// quads.
__device__ __forceinline__ constexpr int pair_row(int r) { return (r >> 1) + (r & 1) * (kT / 4); }

// v + the value of lane l ^ 1 (a DPP quad permutation): the same sum in both lanes.
__device__ __forceinline__ float add_lane_xor1(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));
}
// The segment aggregate pass (scan_seg_agg) stages B two timesteps per entry:
//   b2    row pair_row(r) = timesteps 2r, 2r+1; entry q = (B[2q], B[2q+1]) at 2r, then at 2r+1
// (and dd rows in the same order)
struct WaveSmemPre {
    f32x4 dd[kT / 2][kDdRow];                 // 2.25 KB
    f32x4 b2[kT / 2][kDdRow];                 // 2.25 KB
};

// Wait until at most N of this wave's LDS operations are outstanding (they complete in
// order); vmcnt and expcnt are left alone.
template <int N> __device__ __forceinline__ void lds_wait() {
    static_assert(N >= 0 && N < 16, "lgkmcnt is a 4-bit field");
    // nothing may be scheduled across the wait, so that the reads issued after
    // it stay after it and the operands read before it need no further wait
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
    __builtin_amdgcn_sched_barrier(0);
}

// The scan of a sequence of 16 timesteps (one slice per chain: the verify shape), where
// thousands of short waves run once each.  What bounds it is the waves' set-up and first
// memory round trip, so it uses few registers (7 waves per SIMD) and small tables: 11.3 us
// for (32, 3584, 16), bf16 in, in a loop (9.6 at least), where the ring kernel with one wave per chain (128 VGPRs,
// 4 waves per SIMD) takes 12.9 us.
// POS = true: also record the states at p.pos (p.npos > 0).
// The grid is two-dimensional (channel groups x batch), so that a wave finds its group
// without a division.
template <int IN, int OUT, bool GATE, bool SOFTPLUS, bool POS>
__global__ __launch_bounds__(kThreads) void scan_fwd_short(ScanParams p) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ShortSmem &sm = reinterpret_cast<ShortSmem *>(smem_raw)[wave];

    const int lane = threadIdx.x & 63;
    const int j = lane >> 3;          // channel within the wave
    const int q = lane & 7;           // state pair; also the timestep pair of phases A and C
    const uint32_t n_cg = (uint32_t)((p.dim + kCh - 1) / kCh);
    const uint32_t cg32 = blockIdx.x * kWavesPerGroup + wave;
    if (cg32 >= n_cg) return;                        // whole wave leaves together
    const int64_t cg = cg32, b = blockIdx.y;

    const int64_t d = cg * kCh + j;
    const bool live = d < p.dim;
    const int64_t dcl = live ? d : p.dim - 1;           // dead lanes read a valid row, never store
    const int64_t row = b * p.dim + dcl;
    constexpr int64_t L = kShort;
    const int n0 = 2 * q;

    // Wave-uniform 64-bit bases plus 32-bit lane offsets in elements, so the loads use
    // the scalar-base form.
    constexpr int kEl = IN == 1 ? 2 : 4;
    const int64_t act0 = (b * p.dim + cg * kCh) * L;                 // wave-uniform
    const int64_t bc0 = b * kN * L;
    const char *ub = static_cast<const char *>(p.u) + act0 * kEl;
    const char *db = static_cast<const char *>(p.delta) + act0 * kEl;
    const char *zb = GATE ? static_cast<const char *>(p.z) + act0 * kEl : nullptr;
    const char *bb = static_cast<const char *>(p.Bm) + bc0 * kEl;
    const char *cb = static_cast<const char *>(p.Cm) + bc0 * kEl;
    char *yb = static_cast<char *>(p.y) + act0 * (OUT == 1 ? 2 : 4);
    const uint32_t act_row = (uint32_t)((dcl - cg * kCh) * L);       // lane's channel row

    // The activation loads go out before the per-row operands below, whose loads are
    // conditional (null pointers are allowed): in the other order the compiler made the
    // activation addresses wait for them, two memory round trips.
    // B/C staging: lane (j, q) moves timesteps 2j, 2j + 1 of state rows 2q and 2q + 1.
    struct Slot { Raw2<IN> u, dl, z, B0, B1, C0, C1; } sl;
    {
        const uint32_t oa = act_row + 2 * q, ob = (uint32_t)(2 * q * L) + 2 * j;
        sl.u.load(ub, oa);
        sl.dl.load(db, oa);
        if (GATE) sl.z.load(zb, oa);
        sl.B0.load(bb, ob);
        sl.B1.load(bb, ob + (uint32_t)L);
        sl.C0.load(cb, ob);
        sl.C1.load(cb, ob + (uint32_t)L);
    }
    float a2[2], h[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        a2[s] = p.A[dcl * kN + n0 + s] * kLog2e;
        h[s] = p.h0 ? p.h0[row * kN + n0 + s] : 0.0f;
    }
    const float dskip = p.Dskip ? p.Dskip[dcl] : 0.0f;
    const float bias = p.dt_bias ? p.dt_bias[dcl] : 0.0f;

    // Phase B step TQ: timesteps 4 TQ .. 4 TQ + 3, operands already in registers.
    auto recur4 = [&](const f32x4 (&ddv)[2], const f32x4 (&bcv)[4], auto tq_c) {
        constexpr int TQ = decltype(tq_c)::value;
        float acc4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float dl = (k & 1) ? ddv[k >> 1].z : ddv[k >> 1].x;
            const float dx = (k & 1) ? ddv[k >> 1].w : ddv[k >> 1].y;
            h[0] = __builtin_fmaf(hw_exp2(dl * a2[0]), h[0], dx * bcv[k][0]);
            h[1] = __builtin_fmaf(hw_exp2(dl * a2[1]), h[1], dx * bcv[k][1]);
            acc4[k] = __builtin_fmaf(bcv[k][3], h[1], bcv[k][2] * h[0]);
        }
        // state pairs q and q ^ 1 summed; both lanes write the same entry
#pragma unroll
        for (int k = 0; k < 4; ++k) acc4[k] = add_lane_xor1(acc4[k]);
        sm.part[(kShort / 4) * j + TQ][q >> 1] = f32x4{acc4[0], acc4[1], acc4[2], acc4[3]};
    };
    auto load4 = [&](f32x4 (&ddv)[2], f32x4 (&bcv)[4], auto tq_c) {
        constexpr int TQ = decltype(tq_c)::value;
#pragma unroll
        for (int k = 0; k < 2; ++k) ddv[k] = sm.dd[2 * TQ + k][j];
#pragma unroll
        for (int k = 0; k < 4; ++k) bcv[k] = sm.bc[4 * TQ + k][q];
    };
    constexpr int kW = 1;      // one partial row is written per step
    // Order this wave's LDS writes before its later reads of other lanes' data.
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // ---- A
    float xs[2], gs[2];
    {
        float dl[2], dx[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float x = sl.u.get(k);
            const float v = sl.dl.get(k) + bias;
            dl[k] = SOFTPLUS ? softplus_f32(v) : v;
            dx[k] = dl[k] * x;
            xs[k] = x;
            if (GATE) gs[k] = silu_f32(sl.z.get(k));
        }
        sm.dd[q][j] = f32x4{dl[0], dx[0], dl[1], dx[1]};
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
        sm.bc[2 * j + k][q] = f32x4{sl.B0.get(k), sl.B1.get(k), sl.C0.get(k), sl.C1.get(k)};
    wave_sync();

    // ---- B.  One wait per step: before step i computes, its operands (read during step
    // i - 1) must have arrived, while the partial row that step i - 1 wrote may still be
    // in flight.
    const float hs0 = POS ? h[0] : 0.0f;        // the state before the sequence
    const float hs1 = POS ? h[1] : 0.0f;
    {
        f32x4 ddA[2], bcA[4], ddB[2], bcB[4];
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
        load4(ddA, bcA, I0{});
        lds_wait<0>();
        load4(ddB, bcB, I1{});
        recur4(ddA, bcA, I0{});
        lds_wait<kW>();
        load4(ddA, bcA, I2{});
        recur4(ddB, bcB, I1{});
        lds_wait<kW>();
        load4(ddB, bcB, I3{});
        recur4(ddA, bcA, I2{});
        lds_wait<kW>();
        recur4(ddB, bcB, I3{});
    }
    wave_sync();

    // ---- C: sum the 4 partial sums of channel j at timesteps 2q, 2q+1, one half of entry
    // (j, q >> 1) each
    {
        const float2 *src = reinterpret_cast<const float2 *>(&sm.part[(kShort / 4) * j + (q >> 1)][0]) + (q & 1);
        float2 acc = src[0];
#pragma unroll
        for (int w = 1; w < kQ / 2; ++w) {
            acc.x += src[2 * w].x;
            acc.y += src[2 * w].y;
        }
        float yv[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float y = __builtin_fmaf(dskip, xs[k], k ? acc.y : acc.x);
            if (GATE) y *= gs[k];
            yv[k] = y;
        }
        if (live) {
            const uint32_t oy = act_row + 2 * q;
            if (OUT == 0)
                *reinterpret_cast<float2 *>(yb + oy * 4u) = float2{yv[0], yv[1]};
            else
                *reinterpret_cast<uint32_t *>(yb + oy * 2u) = bf16x2_pack(yv[0], yv[1]);
        }
    }

    // States at requested positions, 64 at a time: lane l holds position k0 + l (-2 past the
    // last).  One replay of the timesteps from the tables, with phase B's operations in the
    // same order, so that a recorded state equals the one the scan carries; a ballot finds the
    // positions of a timestep.  With a replay for each position, fp32 (30, 32, 16) with 16
    // positions took 23.6 us, this way 6.4; with one (32, 3584, 16), bf16, 16.3 either way.
    if constexpr (POS) for (int64_t k0 = 0; k0 < p.npos; k0 += 64) {
        const int pk = k0 + lane < p.npos ? p.pos[(k0 + lane) * p.batch + b] : -2;
        auto record = [&](uint64_t hit, float g0, float g1) {
            for (; hit; hit &= hit - 1) {
                float *dst = p.h_pos + (((k0 + __builtin_ctzll(hit)) * p.batch + b) * p.dim + d) * kN + n0;
                if (live) {
                    dst[0] = g0;
                    dst[1] = g1;
                }
            }
        };
        // position -1 is the state before the first timestep, one past either end reads NaN
        record(__ballot(pk == -1), hs0, hs1);
        record(__ballot(k0 + lane < p.npos && (pk < -1 || pk >= kShort)), __builtin_nanf(""), __builtin_nanf(""));
        uint64_t todo = __ballot(pk >= 0 && pk < kShort);
        float g0 = hs0, g1 = hs1;
        for (int i = 0; todo; ++i) {                            // todo is empty after timestep 15
            const f32x4 dv = sm.dd[i >> 1][j];
            const float dl = (i & 1) ? dv.z : dv.x;
            const float dx = (i & 1) ? dv.w : dv.y;
            const f32x4 bv = sm.bc[i][q];
            g0 = __builtin_fmaf(hw_exp2(dl * a2[0]), g0, dx * bv[0]);
            g1 = __builtin_fmaf(hw_exp2(dl * a2[1]), g1, dx * bv[1]);
            const uint64_t hit = __ballot(pk == i);
            record(hit, g0, g1);
            todo &= ~hit;
        }
    }

    if (p.h_last && live) {
#pragma unroll
        for (int s = 0; s < 2; ++s) p.h_last[row * kN + n0 + s] = h[s];
    }
}

// ---- segment aggregates ------------------------------------------------------
//
// The scan's segments but the last are cut into pieces of piece_len timesteps
// (a multiple of 32), npieces in all.  For every piece and every state n of a
// row, the piece's element of the associative operator of
// Section 2 ("Implementation"):
//   P[n] = prod_t abar_t[n] = 2^(A[n] log2 e sum_t dlt_t),
//   H[n] = sum_t (prod_{r > t} abar_r[n]) dlt_t B_t[n] x_t,
// so that the state at the piece's end is P h_start + H.  H is the state the
// recurrence reaches from a zero state at the piece's start; P is one
// exponential of the piece's summed dlt, not a product of hundreds of
// hardware exponentials near 1, whose rounding would drift and be carried into
// every later segment by the fold P h + H.  The pairs (P, H) go to
// carry[((piece * rows + row) * 16 + n) * 2 + {0, 1}].
//
// Pieces smaller than the scan's segments give a SIMD several waves of this pass, which
// fill each other's waits (plan::segments has the rule and what it measured).
//
// A walk from the segment's end that stops once the running product of abar is
// exactly zero in fp32 gives the same (P, H) with fewer timesteps, but with the
// timestep bias of the MambaByte layers (dt down to 1e-3) some channel of almost
// every 8-channel wave decays too slowly for that within a segment, and the walk
// costs a multiply more per step: measured slower on the 1.6B layer.
//
// The waves of piece 0 also copy h0 (or zeros) into plane npieces as the pairs
// (1, h0[n]), which the scan folds first.
//
// Lane l = 8 j + q as in the scan: channel j, states 2q and 2q+1.  Per chunk,
// lane (j, q) forms dlt and dx of channel j at timesteps 4q .. 4q+3 and stages B
// rows 2j and 2j+1 at those timesteps (the dd and b2 tables of WaveSmemPre).
template <int IN, bool SOFTPLUS>
__global__ __launch_bounds__(kThreads) void scan_seg_agg(ScanParams p, int64_t piece_len, int64_t npieces,
                                                    float *carry) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WaveSmemPre &sm = reinterpret_cast<WaveSmemPre *>(smem_raw)[wave];

    const int lane = threadIdx.x & 63;
    const int j = lane >> 3;
    const int q = lane & 7;
    const uint32_t n_cg = (uint32_t)((p.dim + kCh - 1) / kCh);
    const uint32_t nsg = (uint32_t)npieces;             // the pieces that have an aggregate
    const uint32_t per_xcd = gridDim.x / 8;
    const uint32_t blk = blockIdx.x;
    const uint32_t lwg = blk < per_xcd * 8 ? (blk % 8) * per_xcd + blk / 8 : blk;
    const uint32_t wid = lwg * kWavesPerGroup + wave;
    if (wid >= n_cg * (uint32_t)p.batch * nsg) return;   // whole wave leaves together
    const uint32_t rest = wid / nsg;
    const int64_t piece = wid - rest * nsg;
    const uint32_t bq = rest / n_cg;
    const int64_t cg = rest - bq * n_cg;
    const int64_t b = bq;
    const int64_t t_begin = piece * piece_len;

    const int64_t d = cg * kCh + j;
    const bool live = d < p.dim;
    const int64_t dcl = live ? d : p.dim - 1;           // dead lanes read a valid row, never store
    const int64_t row = b * p.dim + dcl;
    const int64_t L = p.seqlen;
    const int n0 = 2 * q;
    const int64_t rows = p.batch * p.dim;

    float a2[2], h[2] = {0.0f, 0.0f};
    float dsum = 0.0f;      // this lane's share of the piece's sum of dlt
#pragma unroll
    for (int s = 0; s < 2; ++s) a2[s] = p.A[dcl * kN + n0 + s] * kLog2e;
    if (piece == 0 && live) {
        const float g0 = p.h0 ? p.h0[row * kN + n0] : 0.0f;
        const float g1 = p.h0 ? p.h0[row * kN + n0 + 1] : 0.0f;
        *reinterpret_cast<f32x4 *>(carry + (((int64_t)nsg * rows + row) * kN + n0) * 2) =
            f32x4{1.0f, g0, 1.0f, g1};
    }
    const float bias = p.dt_bias ? p.dt_bias[dcl] : 0.0f;

    constexpr int kEl = IN == 1 ? 2 : 4;
    const int64_t row0 = b * p.dim + cg * kCh;                       // wave-uniform
    const int64_t act0 = row0 * L + t_begin;
    const char *ub = static_cast<const char *>(p.u) + act0 * kEl;
    const char *db = static_cast<const char *>(p.delta) + act0 * kEl;
    const char *bb = static_cast<const char *>(p.Bm) + (b * kN * L + t_begin) * kEl;
    const uint32_t act_row = (uint32_t)((dcl - cg * kCh) * L);       // lane's channel row
    const uint32_t bc_row = (uint32_t)(2 * j * L);                   // B rows 2j, 2j+1
    const uint32_t nch = (uint32_t)(piece_len / kT);

    struct Slot { Raw4<IN> u, dl, B0, B1; };
    Slot s0, s1;
    // Chunk k starts at 32 k; past the piece's end the loads read the last
    // chunk again (never consumed).
    auto issue_loads = [&](Slot &sl, uint32_t k) {
        const uint32_t tr = (k < nch ? k : nch - 1) * kT + 4 * q;
        sl.u.load(ub, act_row + tr);
        sl.dl.load(db, act_row + tr);
        sl.B0.load(bb, bc_row + tr);
        sl.B1.load(bb, bc_row + tr + (uint32_t)L);
    };
    // Four timesteps: table rows 2 TQ and 2 TQ + 1, the even timestep of a row first.
    auto fwd4 = [&](const f32x4 (&dv)[2], const f32x4 (&bv)[2]) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const float dl = o ? dv[k].z : dv[k].x;
                const float dx = o ? dv[k].w : dv[k].y;
                const float b0 = o ? bv[k].z : bv[k].x;
                const float b1 = o ? bv[k].w : bv[k].y;
                h[0] = __builtin_fmaf(hw_exp2(dl * a2[0]), h[0], dx * b0);
                h[1] = __builtin_fmaf(hw_exp2(dl * a2[1]), h[1], dx * b1);
            }
        }
    };
    auto load2 = [&](f32x4 (&dv)[2], f32x4 (&bv)[2], int tq) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            dv[k] = sm.dd[pair_row(2 * tq + k)][j];
            bv[k] = sm.b2[pair_row(2 * tq + k)][q];
        }
    };
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    auto chunk = [&](Slot &sl, uint32_t k) {
        float dl[4], dx[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = sl.dl.get(i) + bias;
            dl[i] = SOFTPLUS ? softplus_f32(v) : v;
            dx[i] = dl[i] * sl.u.get(i);
        }
        // pairwise within the quad, then across chunks and lanes: the rounding
        // of the piece's sum stays small
        dsum += (dl[0] + dl[1]) + (dl[2] + dl[3]);
        sm.dd[pair_row(2 * q)][j] = f32x4{dl[0], dx[0], dl[1], dx[1]};
        sm.dd[pair_row(2 * q + 1)][j] = f32x4{dl[2], dx[2], dl[3], dx[3]};
        sm.b2[pair_row(2 * q)][j] = f32x4{sl.B0.get(0), sl.B1.get(0), sl.B0.get(1), sl.B1.get(1)};
        sm.b2[pair_row(2 * q + 1)][j] = f32x4{sl.B0.get(2), sl.B1.get(2), sl.B0.get(3), sl.B1.get(3)};
        wave_sync();
        issue_loads(sl, k + 2);
        {
            f32x4 dA[2], bA[2], dB[2], bB[2];
            load2(dA, bA, 0);
            lds_wait<0>();
            load2(dB, bB, 1);
            fwd4(dA, bA);
            lds_wait<0>();
            load2(dA, bA, 2);
            fwd4(dB, bB);
            lds_wait<0>();
            load2(dB, bB, 3);
            fwd4(dA, bA);
            lds_wait<0>();
            load2(dA, bA, 4);
            fwd4(dB, bB);
            lds_wait<0>();
            load2(dB, bB, 5);
            fwd4(dA, bA);
            lds_wait<0>();
            load2(dA, bA, 6);
            fwd4(dB, bB);
            lds_wait<0>();
            load2(dB, bB, 7);
            fwd4(dA, bA);
            lds_wait<0>();
            fwd4(dB, bB);
        }
        wave_sync();                                  // dd / b2 are rewritten by the next chunk
    };

    issue_loads(s0, 0);
    issue_loads(s1, 1);
    uint32_t k = 0;
    for (; k + 2 <= nch; k += 2) {                  // pairs of chunks
        chunk(s0, k);
        chunk(s1, k + 1);
    }
    if (k < nch) chunk(s0, k);                      // an odd chunk count leaves one
    // the eight lanes of channel j hold its timesteps 4q .. 4q+3 of every chunk:
    // after the butterfly each holds the whole piece's sum
    dsum += __shfl_xor(dsum, 1);
    dsum += __shfl_xor(dsum, 2);
    dsum += __shfl_xor(dsum, 4);
    if (live) {
        const float P0 = hw_exp2(a2[0] * dsum), P1 = hw_exp2(a2[1] * dsum);
        *reinterpret_cast<f32x4 *>(carry + ((piece * rows + row) * kN + n0) * 2) = f32x4{P0, h[0], P1, h[1]};
    }
}

// ---- host side: launch configuration -------------------------------------

// Compute units of the current device; 256 (MI355X) if the runtime cannot say.
inline int64_t device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    return cus;
}

// Waves resident at once on the current device at 2 per SIMD.
inline int64_t resident_waves() { return 8 * device_cus(); }

template <int IN, int OUT, bool GATE, bool SP>
hipError_t fwd_short_sp(ScanParams &p, void *stream) {
    const unsigned n_cg = (unsigned)((p.dim + kCh - 1) / kCh);
    void *args[] = {&p};
    const void *fn = p.npos > 0 ? reinterpret_cast<const void *>(&scan_fwd_short<IN, OUT, GATE, SP, true>)
                                : reinterpret_cast<const void *>(&scan_fwd_short<IN, OUT, GATE, SP, false>);
    return hipLaunchKernel(fn, dim3((n_cg + kWavesPerGroup - 1) / kWavesPerGroup, (unsigned)p.batch), dim3(kThreads),
                           args, sizeof(ShortSmem) * kWavesPerGroup, static_cast<hipStream_t>(stream));
}

template <int IN, int OUT, bool GATE>
hipError_t fwd_short(ScanParams &p, void *stream) {
    return p.delta_softplus ? fwd_short_sp<IN, OUT, GATE, true>(p, stream)
                            : fwd_short_sp<IN, OUT, GATE, false>(p, stream);
}

}  // namespace tiled
}  // namespace mbs
