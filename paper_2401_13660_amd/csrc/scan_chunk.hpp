// scan_chunk.hpp -- the forward selective scan for dstate = 16, one wave per chain in chunks
// of 32 timesteps.
//
// For problems that the ring kernel streams from memory more slowly, and fp32 ones whose chains
// fill the chip evenly: the ring kernel's slices of 16 timesteps ask for half a 128-byte line of
// an fp32 row at a time, and with more data than the 256 MB of the Infinity Cache it reaches
// about 3.0 TB/s where this kernel, a line at a time, reaches 3.7 ((16, 3584, 1024) fp32: 318 us
// and 263; with checkpoints 361 and 280; bf16 with checkpoints, (16, 3584, 2048): 574 and 525).
// plan::chunk_is_faster has the rule.
//
// Each wave works alone: it owns 8 channels of one batch element over one time segment, and
// lane l = 8 j + q holds channel j's states 2q and 2q + 1 in VGPRs.  Per chunk it
//   A  does the per-element work of channel j at timesteps 4q .. 4q + 3 and publishes (dlt,
//      dlt u) in its LDS area; stages the chunk's B and C rows there, widened to fp32;
//   B  runs the recurrence over the 32 timesteps, reading the next four timesteps' operands
//      while computing the current four, and publishes its partial outputs;
//   C  sums the eight partials of channel j at timesteps 4q .. 4q + 3, adds Dskip u, applies
//      the gate and stores y.
// Global loads run two chunks ahead.  Every state and output comes from the ring kernel's
// operations in the same order: the same bits.
// Requires seqlen % 16 == 0 and 16-byte aligned rows.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.hpp"
#include "fwd_plan.hpp"
#include "scan_params.hpp"
#include "scan_ring.hpp"
#include "scan_tiled.hpp"

#include <type_traits>

namespace mbs {
namespace chunk {

using tiled::kCh;
using tiled::kN;
using tiled::kQ;
using tiled::kT;
using tiled::kThreads;
using tiled::kWavesPerGroup;
using tiled::pair_row;

// Private LDS area of one wave.  Rows are padded so that the reads of every table touch
// distinct banks; the dd rows are in pair_row's order so that its writes do too.
//   dd    row pair_row(r) = timesteps 2r, 2r+1; entry j = (dlt, dx, dlt, dx) of channel j
//   bc    row t; entry q = (B[2q], B[2q+1], C[2q], C[2q+1]) at timestep t
//   part  row 8 j + tq = channel j, timesteps 4 tq .. 4 tq + 3; entry q = the partial output
//         of state pair q at those four timesteps
struct WaveSmem {
    f32x4 dd[kT / 2][tiled::kDdRow];                 // 2.25 KB
    f32x4 bc[kT][kQ + 2];                            // 5 KB
    f32x4 part[kCh * (kT / 4)][kQ + 1];              // 9 KB
};

template <int IN, int OUT, bool GATE, bool SOFTPLUS, int REC>
__global__ __launch_bounds__(kThreads) void scan_fwd_chunk(ScanParams p, int64_t seg_len, int64_t pieces,
                                                      const float *carry) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    WaveSmem &sm = reinterpret_cast<WaveSmem *>(smem_raw)[wave];
    constexpr int kPS = kT / 4;                         // part rows per channel

    const int lane = threadIdx.x & 63;
    const int j = lane >> 3;          // channel within the wave
    const int q = lane & 7;           // state pair; also the timestep quad of phases A and C
    const uint32_t n_cg = (uint32_t)((p.dim + kCh - 1) / kCh);
    const uint32_t nseg = ((uint32_t)p.seqlen + (uint32_t)seg_len - 1) / (uint32_t)seg_len;
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2): renumber them so
    // that an XCD works on a contiguous range of channel groups and the B/C rows of a batch
    // element stay in one or two L2s.  Time segment innermost: the waves resident together
    // work on every segment, and their loads spread over the L2 sets even when the row
    // stride is a multiple of 128 KB.
    const uint32_t per_xcd = gridDim.x / 8, blk = blockIdx.x;
    const uint32_t lwg = blk < per_xcd * 8 ? (blk % 8) * per_xcd + blk / 8 : blk;
    const uint32_t wid = lwg * kWavesPerGroup + wave;
    if (wid >= n_cg * (uint32_t)p.batch * nseg) return;      // whole wave leaves together
    const uint32_t rest = wid / nseg, b32 = rest / n_cg;
    const int64_t seg = wid - rest * nseg, cg = rest - b32 * n_cg, b = b32;
    const int64_t t_begin = seg * seg_len;
    const int64_t t_end = t_begin + seg_len < p.seqlen ? t_begin + seg_len : p.seqlen;

    const int64_t d = cg * kCh + j;
    const bool live = d < p.dim;
    const int64_t dcl = live ? d : p.dim - 1;           // dead lanes read a valid row, never store
    const int64_t row = b * p.dim + dcl, rows = p.batch * p.dim;
    const int64_t L = p.seqlen;
    const int n0 = 2 * q;

    // Wave-uniform 64-bit bases (the wave's first channel row, or state row 0 of B and C, at
    // the segment start) plus 32-bit lane offsets in elements.
    constexpr int kEl = IN == 1 ? 2 : 4;
    const int64_t act0 = (b * p.dim + cg * kCh) * L + t_begin, bc0 = b * kN * L + t_begin;
    const char *ub = static_cast<const char *>(p.u) + act0 * kEl;
    const char *db = static_cast<const char *>(p.delta) + act0 * kEl;
    const char *zb = GATE ? static_cast<const char *>(p.z) + act0 * kEl : nullptr;
    const char *bb = static_cast<const char *>(p.Bm) + bc0 * kEl;
    const char *cb = static_cast<const char *>(p.Cm) + bc0 * kEl;
    char *yb = static_cast<char *>(p.y) + act0 * (OUT == 1 ? 2 : 4);
    const uint32_t seg_n = (uint32_t)(t_end - t_begin);             // a multiple of 16
    const uint32_t act_row = (uint32_t)((dcl - cg * kCh) * L);       // lane's channel row
    // B/C staging: lane (j, q) moves timesteps 4j .. 4j + 3 of state rows 2q and 2q + 1
    const uint32_t bc_row = (uint32_t)(2 * q * L);

    struct Slot { tiled::Raw4<IN> u, dl, z, B0, B1, C0, C1; };
    Slot s0, s1;
    // Loads never branch: past the end of the segment they read its last quad again (never
    // consumed).
    auto issue_loads = [&](Slot &sl, uint32_t tr) {            // tr: chunk start within the segment
        const uint32_t ta = tr + 4 * q < seg_n - 4 ? tr + 4 * q : seg_n - 4;
        sl.u.load(ub, act_row + ta);
        sl.dl.load(db, act_row + ta);
        if (GATE) sl.z.load(zb, act_row + ta);
        const uint32_t tb = tr + 4 * j < seg_n - 4 ? tr + 4 * j : seg_n - 4;
        sl.B0.load(bb, bc_row + tb);
        sl.B1.load(bb, bc_row + tb + (uint32_t)L);
        sl.C0.load(cb, bc_row + tb);
        sl.C1.load(cb, bc_row + tb + (uint32_t)L);
    };
    // The first chunks' loads go out before the per-row operands below, whose loads are
    // conditional.
    issue_loads(s0, 0);
    issue_loads(s1, kT);

    float a2[2], h[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        a2[s] = p.A[dcl * kN + n0 + s] * kLog2e;
        h[s] = (nseg == 1 && p.h0) ? p.h0[row * kN + n0 + s] : 0.0f;
    }
    if (nseg > 1) {
        // carry-in: the pre-pass's copy of h0 (the wave of the last segment may write h_last
        // over h0 before this one starts), then the aggregates of the earlier segments'
        // pieces; folding (1, h0) into the zero state gives h0 exactly
        auto fold = [&](int64_t plane) {
            const f32x4 ph = *reinterpret_cast<const f32x4 *>(carry + ((plane * rows + row) * kN + n0) * 2);
            h[0] = __builtin_fmaf(ph.x, h[0], ph.y);
            h[1] = __builtin_fmaf(ph.z, h[1], ph.w);
        };
        fold(pieces * (nseg - 1));
        for (int64_t i = 0; i < pieces * seg; ++i) fold(i);
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
        sm.part[kPS * j + TQ][q] = f32x4{acc4[0], acc4[1], acc4[2], acc4[3]};
    };
    auto load4 = [&](f32x4 (&ddv)[2], f32x4 (&bcv)[4], auto tq_c) {
        constexpr int TQ = decltype(tq_c)::value;
#pragma unroll
        for (int k = 0; k < 2; ++k) ddv[k] = sm.dd[pair_row(2 * TQ + k)][j];
#pragma unroll
        for (int k = 0; k < 4; ++k) bcv[k] = sm.bc[4 * TQ + k][q];
    };

    // Positions to record, 64 at a time as in the ring kernel.  The states of those in the
    // chunk at t0: from the state before the chunk, its first timesteps once more from the
    // tables, with phase B's operations in the same order.
    auto positions = [&](int64_t k0) {
        return k0 + lane < p.npos ? (int)p.pos[(k0 + lane) * p.batch + b] : -2;
    };
    const int pos0 = REC == ring::kPositions ? positions(0) : -2;
    auto record_positions = [&](int64_t t0, int nt, float r0, float r1) {
        for (int64_t k0 = 0; k0 < p.npos; k0 += 64) {
            const int pk = k0 == 0 ? pos0 : positions(k0);
            for (uint64_t hit = __ballot(pk >= (int)t0 && pk < (int)t0 + nt); hit; hit &= hit - 1) {
                const int l = __builtin_ctzll(hit);
                const int last = __builtin_amdgcn_readlane(pk, l) - (int)t0;
                float g0 = r0, g1 = r1;
                for (int i = 0; i <= last; ++i) {
                    const f32x4 dv = sm.dd[pair_row(i >> 1)][j];
                    const float dl = (i & 1) ? dv.z : dv.x;
                    const float dx = (i & 1) ? dv.w : dv.y;
                    const f32x4 bv = sm.bc[i][q];
                    g0 = __builtin_fmaf(hw_exp2(dl * a2[0]), g0, dx * bv[0]);
                    g1 = __builtin_fmaf(hw_exp2(dl * a2[1]), g1, dx * bv[1]);
                }
                if (live) {
                    float *dst = p.h_pos + (((k0 + l) * p.batch + b) * p.dim + d) * kN + n0;
                    dst[0] = g0;
                    dst[1] = g1;
                }
            }
        }
    };

    // Checkpoints are stored in time order, one per 16 timesteps, so a lane's pointer steps by
    // one plane (rows x kN floats) per store.
    float *ck_at = REC == ring::kCheckpoints ? p.ck + ((t_begin / 16) * rows + row) * kN + n0 : nullptr;
    auto store_ck = [&] {                            // the state before the next 16 timesteps
        if (live) *reinterpret_cast<float2 *>(ck_at) = float2{h[0], h[1]};
        ck_at += rows * kN;
    };

    auto chunk = [&](Slot &sl, int64_t t0) {
        const int nt = (int)(t_end - t0 < kT ? t_end - t0 : kT);       // 32, or 16 at the end

        // ---- A
        float xs[4], gs[4], dl[4], dx[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float x = sl.u.get(k), v = sl.dl.get(k) + bias;
            dl[k] = SOFTPLUS ? softplus_f32(v) : v;
            dx[k] = dl[k] * x;
            xs[k] = x;
            if (GATE) gs[k] = silu_f32(sl.z.get(k));
        }
        sm.dd[pair_row(2 * q)][j] = f32x4{dl[0], dx[0], dl[1], dx[1]};
        sm.dd[pair_row(2 * q + 1)][j] = f32x4{dl[2], dx[2], dl[3], dx[3]};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            sm.bc[4 * j + k][q] = f32x4{sl.B0.get(k), sl.B1.get(k), sl.C0.get(k), sl.C1.get(k)};
        ring::wave_sync();
        issue_loads(sl, (uint32_t)(t0 - t_begin) + 2 * kT);            // the chunk after next

        // ---- B.  One wait per step: before step i computes, its operands (read during step
        // i - 1) must have arrived, while the partial row that step i - 1 wrote may still be
        // in flight.
        const float hs0 = h[0], hs1 = h[1];             // the state before this chunk
        if (REC == ring::kCheckpoints) store_ck();
        {
            f32x4 ddA[2], bcA[4], ddB[2], bcB[4];
            using I0 = std::integral_constant<int, 0>;
            using I1 = std::integral_constant<int, 1>;
            using I2 = std::integral_constant<int, 2>;
            using I3 = std::integral_constant<int, 3>;
            using I4 = std::integral_constant<int, 4>;
            using I5 = std::integral_constant<int, 5>;
            using I6 = std::integral_constant<int, 6>;
            using I7 = std::integral_constant<int, 7>;
            load4(ddA, bcA, I0{});
            tiled::lds_wait<0>();
            load4(ddB, bcB, I1{});
            recur4(ddA, bcA, I0{});
            tiled::lds_wait<1>();
            load4(ddA, bcA, I2{});
            recur4(ddB, bcB, I1{});
            tiled::lds_wait<1>();
            load4(ddB, bcB, I3{});
            recur4(ddA, bcA, I2{});
            tiled::lds_wait<1>();
            if (nt == kT) {
                load4(ddA, bcA, I4{});
                recur4(ddB, bcB, I3{});
                if (REC == ring::kCheckpoints) store_ck();
                tiled::lds_wait<1>();
                load4(ddB, bcB, I5{});
                recur4(ddA, bcA, I4{});
                tiled::lds_wait<1>();
                load4(ddA, bcA, I6{});
                recur4(ddB, bcB, I5{});
                tiled::lds_wait<1>();
                load4(ddB, bcB, I7{});
                recur4(ddA, bcA, I6{});
                tiled::lds_wait<1>();
                recur4(ddB, bcB, I7{});
            } else {
                recur4(ddB, bcB, I3{});
            }
        }
        ring::wave_sync();

        // ---- C
        if (4 * q < nt) {
            f32x4 acc = sm.part[kPS * j + q][0];
#pragma unroll
            for (int w = 1; w < kQ; ++w) acc += sm.part[kPS * j + q][w];
            float yv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float y = __builtin_fmaf(dskip, xs[k], acc[k]);
                if (GATE) y *= gs[k];
                yv[k] = y;
            }
            if (live) {
                const uint32_t oy = act_row + (uint32_t)(t0 - t_begin) + 4 * q;
                if (OUT == 0)
                    *reinterpret_cast<f32x4 *>(yb + oy * 4u) = f32x4{yv[0], yv[1], yv[2], yv[3]};
                else
                    *reinterpret_cast<u32x2 *>(yb + oy * 2u) = u32x2{bf16x2_pack(yv[0], yv[1]), bf16x2_pack(yv[2], yv[3])};
            }
        }
        if (REC == ring::kPositions) record_positions(t0, nt, hs0, hs1);
        ring::wave_sync();                              // part / dd / bc are rewritten by the next chunk
    };

    int64_t t0 = t_begin;
    for (; t0 + 2 * kT <= t_end; t0 += 2 * kT) {       // pairs of full chunks
        chunk(s0, t0);
        chunk(s1, t0 + kT);
    }
    if (t0 < t_end) chunk(s0, t0);                      // a full chunk and/or a half chunk remain
    if (t0 + kT < t_end) chunk(s1, t0 + kT);

    if (p.h_last && live && seg == nseg - 1) {
#pragma unroll
        for (int s = 0; s < 2; ++s) p.h_last[row * kN + n0 + s] = h[s];
    }
}

// ---- host side ------------------------------------------------------------------

template <int IN, int OUT, bool GATE, bool SP>
hipError_t fwd_chunk(ScanParams &p, const plan::Fwd &f, hipStream_t st, const float *carry) {
    const void *fn = reinterpret_cast<const void *>(&scan_fwd_chunk<IN, OUT, GATE, SP, ring::kCheckpoints>);
    if constexpr (IN == 0) {                            // bf16 comes here with checkpoints only
        if (p.npos > 0) fn = reinterpret_cast<const void *>(&scan_fwd_chunk<IN, OUT, GATE, SP, ring::kPositions>);
        else if (!p.ck) fn = reinterpret_cast<const void *>(&scan_fwd_chunk<IN, OUT, GATE, SP, ring::kPlain>);
    }
    int64_t seg_len = f.seg_len, pieces = f.pieces;
    void *args[] = {&p, &seg_len, &pieces, &carry};
    return hipLaunchKernel(fn, dim3((unsigned)f.workgroups), dim3(f.threads), args, sizeof(WaveSmem) * kWavesPerGroup, st);
}

}  // namespace chunk
}  // namespace mbs
