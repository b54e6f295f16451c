// scan_ring.hpp -- the forward selective scan for dstate = 16, time slices dealt
// round the waves of a workgroup.
//
// The recurrence of eq. (2) is serial in time, but only its last operation is: the
// exponentials, softplus, the gate, the products with B and C and the sums over
// states need no state.  A chain (8 channels of one batch element over one time
// segment) is therefore cut into slices of 16 timesteps, and W waves of a workgroup
// take its slices in turn (wave r: slices r, r + W, ...).  A wave prepares its slice
// alone, waits for the state that the slice before it ends in, runs the 16-step
// chain h = abar h + bx (one FMA per state and step), hands the state on through LDS
// and finishes its outputs while the next wave runs the next slice's chain.  Every
// wait ends: slice 0 waits for nothing, slice s for slice s - 1 only, a wave takes
// its slices in rising order, and the waves of a workgroup are resident together.
//
// What bounds it: instruction issue (an exponential or an MFMA holds its SIMD for 8 cycles, the
// VALU instructions beside them take 4; 171 of these, 40 and 12 of those per slice make 1,100
// cycles, the 972M layer takes about 1,280).  With one wave per 8 channels for a whole sequence the
// number of waves is batch * dim / 8, so that most shapes left SIMDs with one wave or two,
// unevenly, or paid a pre-pass that repeated every exponential to cut the sequence.  Here
// the waves per SIMD are a free choice (4, as many as 128 VGPRs allow), and with W a
// multiple of 4 every SIMD of a compute unit has the same share of every chain.
// Measured, bf16 in and fp32 out, before (one wave per 8 channels, time slices inside the
// wave or segments with a pre-pass, by shape) and now:
//   (4, 3584, 8192)    541 -> 470-490 us        (4, 2048, 8192)   341 -> 290
//   (1, 4608, 65536)  1999 -> 1560-1580         (1, 3584, 8192)   214 -> 148
//   (1, 2048, 8192)    132 -> 109               (1, 3584, 1013), by the row kernel: 2330 -> 24
//
// Lane l = 8 j + q holds channel j's states 2q and 2q + 1.  Per slice the wave
//   A  does the per-element work of channel j at timesteps 2q, 2q + 1: dlt, dx = dlt u
//      and silu(z); and stages the slice's B and C rows in LDS, widened to fp32;
//   E  forms abar = 2^(dlt A log2 e) and bx = dx B for its two states and all 16
//      timesteps.  The products dlt A are outer products (time x state) per channel:
//      v_mfma_f32_4x4x1 forms 4 timesteps of a state per instruction and takes each
//      lane's dlt to all 8 lanes of the channel on the way (A-operand broadcast over
//      pairs of blocks; its products are the VALU's bit for bit).  dx is spread the
//      same way, times 1;
//   H  runs the chain from the state handed over, keeping h_t in bx's registers;
//   C  forms the partial outputs C_t[2q] h_t[2q] + C_t[2q+1] h_t[2q+1] and hands them
//      through LDS to lane (j, t / 2), which sums the eight of its own two timesteps,
//      adds Dskip u, applies the gate and stores y.
//
// Up to 15 timesteps after the last full slice are run one by one by the wave whose turn
// it is, so any length goes, at any row alignment.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.hpp"
#include "fwd_plan.hpp"
#include "scan_params.hpp"
#include "scan_tiled.hpp"

#include <type_traits>

namespace mbs {
namespace ring {

constexpr int kN = 16;                // states per channel
constexpr int kCh = 8;                // channels per chain
constexpr int kQ = 8;                 // state pairs per channel (lanes per channel)
constexpr int kS = 16;                // timesteps per slice
constexpr int kMaxWaves = 16;         // per workgroup: 4 per SIMD at 128 VGPRs

// What the launch adds to the problem.
struct RingParams {
    uint32_t n_cg;        // channel groups of 8 per batch element
    uint32_t nseg;        // time segments (1: none)
    uint32_t seg_len;     // timesteps per segment, a multiple of 32 when nseg > 1
    uint32_t pieces;      // pre-pass pieces per segment
    uint32_t chains;      // n_cg * batch * nseg
    uint32_t log_w;       // waves per chain: 1 << log_w
    const float *carry;   // pre-pass aggregates (nseg > 1), see scan_seg_agg
};

// Two consecutive activations of one row, which may start at any element: the pair is
// only aligned to its element (the hardware takes such loads).
typedef uint32_t u32_e2 __attribute__((aligned(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef f32x2 f32x2_e4 __attribute__((aligned(4)));
template <int IN> struct Pair;
template <> struct Pair<1> {
    uint32_t v;
    __device__ __forceinline__ void load(const char *base, uint32_t off) {
        v = *reinterpret_cast<const u32_e2 *>(base + off * 2u);
    }
    // the first n of the two; what is read for the others is the row's element n - 1 again.
    // BOTH: the second is read at all.
    template <bool BOTH> __device__ __forceinline__ void load_first(const char *base, uint32_t off, int n) {
        v = *reinterpret_cast<const uint16_t *>(base + (off + (n > 0 ? 0 : n - 1)) * 2u);
        if constexpr (BOTH) v |= (uint32_t)*reinterpret_cast<const uint16_t *>(base + (off + (n > 1 ? 1 : n - 1)) * 2u) << 16;
    }
    __device__ __forceinline__ float get(int i) const { return i ? bf16_hi(v) : bf16_lo(v); }
};
template <> struct Pair<0> {
    f32x2 v;
    __device__ __forceinline__ void load(const char *base, uint32_t off) {
        v = *reinterpret_cast<const f32x2_e4 *>(base + off * 4u);
    }
    template <bool BOTH> __device__ __forceinline__ void load_first(const char *base, uint32_t off, int n) {
        v.x = v.y = *reinterpret_cast<const float *>(base + (off + (n > 0 ? 0 : n - 1)) * 4u);
        if constexpr (BOTH) v.y = *reinterpret_cast<const float *>(base + (off + (n > 1 ? 1 : n - 1)) * 4u);
    }
    __device__ __forceinline__ float get(int i) const { return i ? v.y : v.x; }
};
template <int OUT> __device__ __forceinline__ void store_pair(char *base, uint32_t off, float a, float b) {
    if constexpr (OUT == 0) *reinterpret_cast<f32x2_e4 *>(base + off * 4u) = f32x2{a, b};
    else *reinterpret_cast<u32_e2 *>(base + off * 2u) = bf16x2_pack(a, b);
}

// LDS of one wave.  Writes of b2 and c2 fill a row of 8 entries from 8 consecutive
// lanes, reads broadcast a row's entries; partial rows of 9 entries spread the
// 8-byte reads of 32 lanes over all 64 banks.  No access meets another in a bank.
struct WaveSmem {
    f32x4 b2[kS / 2][kQ];             // row r, entry q: (B[2q], B[2q+1]) at 2r, then at 2r + 1
    f32x4 c2[kS / 2][kQ];             // the same of C
    f32x4 part[kCh * (kS / 4)][kQ + 1];  // row 4 j + t / 4, entry q: 4 timesteps' partial outputs
    float2 hand[64];                  // the state after this wave's last finished slice
};
static_assert(sizeof(WaveSmem) % 16 == 0, "areas of a workgroup follow each other");

// LDS order within one wave: its own operations complete in order, so ordering the
// compiler is enough.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 4 products per lane: a (this channel's lanes 4 HALF .. 4 HALF + 3, in that order)
// times b (this lane).
template <int HALF> __device__ __forceinline__ f32x4 outer4(float a, float b) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 1, HALF, 0);
}

enum Record { kPlain = 0, kCheckpoints = 1, kPositions = 2 };

template <int IN, int OUT, bool GATE, bool SOFTPLUS, int REC>
__global__ __launch_bounds__(kMaxWaves * 64) void scan_fwd_ring(ScanParams p, RingParams g) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_waves = blockDim.x >> 6;
    WaveSmem *areas = reinterpret_cast<WaveSmem *>(smem_raw);
    uint32_t *done = reinterpret_cast<uint32_t *>(areas + n_waves);   // per wave: its last finished slice + 1
    WaveSmem &sm = areas[wave];
    const int lane = threadIdx.x & 63;
    if (lane == 0) done[wave] = 0;
    __syncthreads();

    const int j = lane >> 3;          // channel within the chain
    const int q = lane & 7;           // state pair; also the timestep pair of A and C
    const int W = 1 << g.log_w;
    const int r = wave & (W - 1);
    const int before = (wave & ~(W - 1)) | ((wave - 1) & (W - 1));    // the wave of the slice before
    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2): renumber
    // them so that an XCD works on a contiguous range of channel groups and the B/C
    // rows of a batch element stay in one or two L2s.  Segments innermost.
    const uint32_t per_xcd = gridDim.x / 8, blk = blockIdx.x;
    const uint32_t lwg = blk < per_xcd * 8 ? (blk % 8) * per_xcd + blk / 8 : blk;
    const uint32_t chain = lwg * (n_waves >> g.log_w) + (wave >> g.log_w);
    if (chain >= g.chains) return;                       // whole waves; no barrier follows
    const uint32_t rest = g.nseg == 1 ? chain : chain / g.nseg;
    const uint32_t seg = chain - rest * g.nseg;
    const uint32_t b32 = rest / g.n_cg;
    const int64_t cg = rest - b32 * g.n_cg, b = b32;
    const uint32_t L = (uint32_t)p.seqlen;
    const uint32_t t_begin = seg * g.seg_len;
    const uint32_t t_end = L - t_begin > g.seg_len ? t_begin + g.seg_len : L;
    const uint32_t nfull = (t_end - t_begin) / kS;       // full slices
    const int nt = (int)((t_end - t_begin) % kS);        // timesteps of the short one after them
    const bool owns_tail = nt > 0 && (nfull & (W - 1)) == (uint32_t)r;
    if ((uint32_t)r >= nfull && !owns_tail) return;

    const int64_t dcl = cg * kCh + j < p.dim ? cg * kCh + j : p.dim - 1;   // dead lanes: the last row again
    const int64_t row = b * p.dim + dcl, rows = p.batch * p.dim;
    const int n0 = 2 * q;

    // Wave-uniform 64-bit bases plus 32-bit lane offsets in elements.
    constexpr int kEl = IN == 1 ? 2 : 4;
    const int64_t act0 = (b * p.dim + cg * kCh) * p.seqlen, bc0 = b * kN * p.seqlen;
    const char *ub = static_cast<const char *>(p.u) + act0 * kEl;
    const char *db = static_cast<const char *>(p.delta) + act0 * kEl;
    const char *zb = GATE ? static_cast<const char *>(p.z) + act0 * kEl : nullptr;
    const char *bb = static_cast<const char *>(p.Bm) + bc0 * kEl;
    const char *cb = static_cast<const char *>(p.Cm) + bc0 * kEl;
    char *yb = static_cast<char *>(p.y) + act0 * (OUT == 1 ? 2 : 4);
    const uint32_t act_row = (uint32_t)(dcl - cg * kCh) * L;         // lane's channel row
    const uint32_t bc_row = 2u * q * L;                              // B/C rows 2q, 2q + 1 ...

    // B/C staging: lane (j, q) moves timesteps 2j, 2j + 1 of state rows 2q and 2q + 1.
    using Raw = Pair<IN>;
    struct Slot { Raw u, dl, z, B0, B1, C0, C1; } sl;
    // Loads never branch: past the last full slice a wave reads its first again (never
    // consumed).  A wave's next slice is asked for as soon as the last one's registers are
    // free, except where the 128 VGPRs do not hold it beside the exponentials (14 registers
    // of fp32, or what checkpoints with a gate, or positions, need): then after them, before the
    // wait for the state.  Spilled instead, (4, 3584, 2048) fp32 took 242 us, this way 156; bf16
    // with checkpoints (4, 3584, 8192) 577 and 564.  Without a gate checkpoints spill nothing, and
    // (1, 3584, 46656) took 843 us with early loads and 916 with late ones.
    constexpr bool kLateLoads = IN == 0 || REC == kPositions || (REC == kCheckpoints && GATE);
    const uint32_t oa = act_row + 2 * q, ob = bc_row + 2 * j;
    auto issue_loads = [&](uint32_t i) {
        const uint32_t t0 = t_begin + (i < nfull ? i : (uint32_t)r) * kS;
        sl.u.load(ub, oa + t0);
        sl.dl.load(db, oa + t0);
        if (GATE) sl.z.load(zb, oa + t0);
        sl.B0.load(bb, ob + t0);
        sl.B1.load(bb, ob + t0 + L);
        sl.C0.load(cb, ob + t0);
        sl.C1.load(cb, ob + t0 + L);
    };
    if ((uint32_t)r < nfull) issue_loads(r);

    float a2[2], h[2] = {0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 2; ++s) a2[s] = p.A[dcl * kN + n0 + s] * kLog2e;
    if (r == 0) {
        if (g.nseg == 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) h[s] = p.h0 ? p.h0[row * kN + n0 + s] : 0.0f;
        } else {
            // carry-in: the pre-pass's copy of h0, then the aggregates of the earlier
            // segments' pieces; folding (1, h0) into the zero state gives h0 exactly
            auto fold = [&](int64_t plane) {
                const f32x4 ph = *reinterpret_cast<const f32x4 *>(g.carry + ((plane * rows + row) * kN + n0) * 2);
                h[0] = __builtin_fmaf(ph.x, h[0], ph.y);
                h[1] = __builtin_fmaf(ph.z, h[1], ph.w);
            };
            fold((int64_t)g.pieces * (g.nseg - 1));
            for (uint32_t i = 0; i < g.pieces * seg; ++i) fold(i);
        }
    }
    const float dskip = p.Dskip ? p.Dskip[dcl] : 0.0f;
    const float bias = p.dt_bias ? p.dt_bias[dcl] : 0.0f;

    // Positions to record, 64 at a time: lane l holds this batch element's position k0 + l
    // (-2 past the last: no timestep), the first 64 read once.  A ballot finds those of a
    // slice.  Read one by one in every slice, on the chain's critical path, 1, 16, 64 and 256
    // positions made the scan of (1, 4608, 8192), bf16, take 270, 451, 1094 and 3440 us; this
    // way 245, 242, 267 and 376.
    auto positions = [&](int64_t k0) {
        return k0 + lane < p.npos ? (int)p.pos[(k0 + lane) * p.batch + b] : -2;
    };
    const int pos0 = REC == kPositions ? positions(0) : -2;
    const uint32_t lane_state = (uint32_t)((dcl - cg * kCh) * kN + n0);
    auto record = [&](int64_t k, float g0, float g1) {
        float *dst = p.h_pos + ((k * p.batch + b) * p.dim + cg * kCh) * kN;
        dst[lane_state] = g0;
        dst[lane_state + 1] = g1;
    };
    // Positions that no timestep holds: -1 is the state before the first, (g0, g1), one past
    // either end reads NaN.
    auto record_others = [&](float g0, float g1) {
        for (int64_t k0 = 0; k0 < p.npos; k0 += 64) {
            const int pk = k0 == 0 ? pos0 : positions(k0);
            for (uint64_t hit = __ballot(k0 + lane < p.npos && (pk < 0 || pk >= (int)L)); hit; hit &= hit - 1) {
                const int l = __builtin_ctzll(hit);
                const bool start = __builtin_amdgcn_readlane(pk, l) == -1;
                record(k0 + l, start ? g0 : __builtin_nanf(""), start ? g1 : __builtin_nanf(""));
            }
        }
    };

    // The state that slice s starts from, handed over by the wave of slice s - 1.  The
    // flag is read before the state it vouches for, and a wave's LDS operations are
    // carried out in order.
    auto take_state = [&](uint32_t s) {
        if (s == 0 || W == 1) return;
        uint64_t hv;
        for (;;) {
            const uint32_t f = __hip_atomic_load(&done[before], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("" ::: "memory");
            hv = __hip_atomic_load(reinterpret_cast<uint64_t *>(&areas[before].hand[lane]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            if ((uint32_t)__builtin_amdgcn_readfirstlane(f) == s) break;
            __builtin_amdgcn_s_sleep(1);
        }
        h[0] = __uint_as_float((uint32_t)hv);
        h[1] = __uint_as_float((uint32_t)(hv >> 32));
    };

    for (uint32_t s = r; s < nfull; s += W) {
        const uint32_t t0 = t_begin + s * kS;

        // ---- A: per-element work of timesteps t0 + 2q, t0 + 2q + 1; B/C staging
        float xs[2], gs[2], dl[2], dx[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float x = sl.u.get(k), v = sl.dl.get(k) + bias;
            dl[k] = SOFTPLUS ? softplus_f32(v) : v;
            dx[k] = dl[k] * x;
            xs[k] = x;
            if (GATE) gs[k] = silu_f32(sl.z.get(k));
        }
        // the gate now, so that z's register is free for the next slice's load
        if (GATE) asm volatile("" : "+v"(gs[0]), "+v"(gs[1]));
        sm.b2[j][q] = f32x4{sl.B0.get(0), sl.B1.get(0), sl.B0.get(1), sl.B1.get(1)};
        sm.c2[j][q] = f32x4{sl.C0.get(0), sl.C1.get(0), sl.C0.get(1), sl.C1.get(1)};
        wave_sync();
        if constexpr (!kLateLoads) issue_loads(s + W);   // the wave's next slice

        // ---- E: abar and bx of all 16 timesteps
        float ab[kS][2], hx[kS][2];
        {
            float xbv[kS];
            f32x4 bv[kS / 2];
#pragma unroll
            for (int i = 0; i < kS / 2; ++i) bv[i] = sm.b2[i][q];
            auto half = [&](auto half_c) {
                constexpr int HALF = decltype(half_c)::value;
#pragma unroll
                for (int k = 0; k < 2; ++k) {            // timesteps 8 HALF + 2 i + k
                    const f32x4 e0 = outer4<HALF>(dl[k], a2[0]);
                    const f32x4 e1 = outer4<HALF>(dl[k], a2[1]);
                    const f32x4 xb = outer4<HALF>(dx[k], 1.0f);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int t = 8 * HALF + 2 * i + k;
                        ab[t][0] = e0[i];
                        ab[t][1] = e1[i];
                        xbv[t] = xb[i];
                    }
                }
            };
            half(std::integral_constant<int, 0>{});
            half(std::integral_constant<int, 1>{});
            // The exponentials together, at raised priority: while one wave of a SIMD issues
            // exponentials nothing pairs with them, and two waves' other instructions issue in
            // pairs (2.1 cycles each instead of 4.4, measured) only while no wave is at its
            // exponentials, so they are got over with.
#pragma unroll
            for (int t = 0; t < kS; ++t) asm volatile("" : "+v"(ab[t][0]), "+v"(ab[t][1]), "+v"(xbv[t]));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int t = 0; t < kS; ++t) {
                ab[t][0] = hw_exp2(ab[t][0]);
                ab[t][1] = hw_exp2(ab[t][1]);
            }
#pragma unroll
            for (int t = 0; t < kS; ++t) asm volatile("" : "+v"(ab[t][0]), "+v"(ab[t][1]));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int i = 0; i < kS / 2; ++i) {
                hx[2 * i][0] = xbv[2 * i] * bv[i][0];
                hx[2 * i][1] = xbv[2 * i] * bv[i][1];
                hx[2 * i + 1][0] = xbv[2 * i + 1] * bv[i][2];
                hx[2 * i + 1][1] = xbv[2 * i + 1] * bv[i][3];
            }
        }
        // All of it before the wait: the compiler would sink the exponentials past it,
        // and the slices would take turns at them too.
#pragma unroll
        for (int t = 0; t < kS; ++t)
            asm volatile("" : "+v"(ab[t][0]), "+v"(ab[t][1]), "+v"(hx[t][0]), "+v"(hx[t][1]));

        if constexpr (kLateLoads) issue_loads(s + W);

        // ---- H: the state before the slice, the chain, the hand-over
        take_state(s);
        const float hs0 = h[0], hs1 = h[1];
        __builtin_amdgcn_s_setprio(1);                   // the other waves of the chain wait for this
#pragma unroll
        for (int t = 0; t < kS; ++t) {
            h[0] = hx[t][0] = __builtin_fmaf(ab[t][0], h[0], hx[t][0]);
            h[1] = hx[t][1] = __builtin_fmaf(ab[t][1], h[1], hx[t][1]);
        }
        if (W > 1) {
            const uint64_t hv = (uint64_t)__float_as_uint(h[0]) | ((uint64_t)__float_as_uint(h[1]) << 32);
            __hip_atomic_store(reinterpret_cast<uint64_t *>(&sm.hand[lane]), hv, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("" ::: "memory");
            __hip_atomic_store(&done[wave], s + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __builtin_amdgcn_s_setprio(0);

        if constexpr (REC == kCheckpoints) {             // the state before the slice's first timestep
            *reinterpret_cast<float2 *>(p.ck + ((int64_t)(t0 / kS) * rows + row) * kN + n0) = float2{hs0, hs1};
        }
        if constexpr (REC == kPositions) {
            if (s == 0 && seg == 0) record_others(hs0, hs1);
            for (int64_t k0 = 0; k0 < p.npos; k0 += 64) {
                const int pk = k0 == 0 ? pos0 : positions(k0);
                for (uint64_t hit = __ballot(pk >= (int)t0 && pk < (int)t0 + kS); hit; hit &= hit - 1) {
                    const int l = __builtin_ctzll(hit);
                    const uint32_t at = (uint32_t)__builtin_amdgcn_readlane(pk, l) - t0;
                    float g0 = hx[0][0], g1 = hx[0][1];
#pragma unroll
                    for (int t = 1; t < kS; ++t)
                        if (at == (uint32_t)t) { g0 = hx[t][0]; g1 = hx[t][1]; }
                    record(k0 + l, g0, g1);
                }
            }
        }

        f32x4 cvs[kS / 2];
#pragma unroll
        for (int i = 0; i < kS / 2; ++i) cvs[i] = sm.c2[i][q];
#pragma unroll
        for (int i = 0; i < kS / 2; ++i) asm volatile("" : "+v"(cvs[i]));
        // ---- C: partial outputs, their sum over the state pairs, skip, gate, store
#pragma unroll
        for (int tq = 0; tq < kS / 4; ++tq) {
            float acc[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4 cv = cvs[2 * tq + i];
                const int t = 4 * tq + 2 * i;
                acc[2 * i] = __builtin_fmaf(cv.y, hx[t][1], cv.x * hx[t][0]);
                acc[2 * i + 1] = __builtin_fmaf(cv.w, hx[t + 1][1], cv.z * hx[t + 1][0]);
            }
            sm.part[(kS / 4) * j + tq][q] = f32x4{acc[0], acc[1], acc[2], acc[3]};
        }
        wave_sync();
        const float2 *src = reinterpret_cast<const float2 *>(&sm.part[(kS / 4) * j + (q >> 1)][0]) + (q & 1);
        float2 acc = src[0];
#pragma unroll
        for (int w = 1; w < kQ; ++w) {
            acc.x += src[2 * w].x;
            acc.y += src[2 * w].y;
        }
        float y0 = __builtin_fmaf(dskip, xs[0], acc.x), y1 = __builtin_fmaf(dskip, xs[1], acc.y);
        if (GATE) {
            y0 *= gs[0];
            y1 *= gs[1];
        }
        // Dead lanes (channels past dim) work on the last channel's row and store its
        // values again: a store under a condition would leave the compiler unsure how many
        // operations are outstanding, and it would wait for the store before the next
        // slice's data.
        store_pair<OUT>(yb, oa + t0, y0, y1);
        wave_sync();                                     // the tables are rewritten by the next slice
    }

    // ---- the sequence's last nt < 16 timesteps, one after the other
    if (owns_tail) {
        const uint32_t t0 = t_begin + nfull * kS;
        const int na = nt - 2 * q, nb = nt - 2 * j;
        // Every load at once, none under a lane's condition, or each waited for the one before:
        // bf16 (28, 4608, 4) with a first state took 16.5 us so, 15.0 this way, (200, 3584, 2)
        // 90 and 67.
        auto load_first = [&](auto both) {
            constexpr bool BOTH = decltype(both)::value;
            sl.u.template load_first<BOTH>(ub, oa + t0, na);
            sl.dl.template load_first<BOTH>(db, oa + t0, na);
            if (GATE) sl.z.template load_first<BOTH>(zb, oa + t0, na);
            sl.B0.template load_first<BOTH>(bb, ob + t0, nb);
            sl.B1.template load_first<BOTH>(bb, ob + t0 + L, nb);
            sl.C0.template load_first<BOTH>(cb, ob + t0, nb);
            sl.C1.template load_first<BOTH>(cb, ob + t0 + L, nb);
        };
        if (nt > 1) load_first(std::integral_constant<bool, true>{});
        else load_first(std::integral_constant<bool, false>{});
        sm.b2[j][q] = f32x4{sl.B0.get(0), sl.B1.get(0), sl.B0.get(1), sl.B1.get(1)};
        sm.c2[j][q] = f32x4{sl.C0.get(0), sl.C1.get(0), sl.C0.get(1), sl.C1.get(1)};
        // the partials' area: (dlt, dx) of timestep t, channel j, then the sums over states
        float2 *dd = reinterpret_cast<float2 *>(&sm.part[0][0]);
        float *sums = reinterpret_cast<float *>(&sm.part[kCh * 2][0]);
        float xs[2], gs[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float x = sl.u.get(k), v = sl.dl.get(k) + bias;
            const float dl = SOFTPLUS ? softplus_f32(v) : v;
            xs[k] = x;
            if (GATE) gs[k] = silu_f32(sl.z.get(k));
            dd[(2 * q + k) * kCh + j] = float2{dl, dl * x};
        }
        wave_sync();
        take_state(nfull);
        if (REC == kPositions && nfull == 0) record_others(h[0], h[1]);   // seg is 0
        for (int t = 0; t < nt; ++t) {
            const float2 dv = dd[t * kCh + j];
            const float2 bv = reinterpret_cast<const float2 *>(&sm.b2[t >> 1][q])[t & 1];
            const float2 cv = reinterpret_cast<const float2 *>(&sm.c2[t >> 1][q])[t & 1];
            h[0] = __builtin_fmaf(hw_exp2(dv.x * a2[0]), h[0], dv.y * bv.x);
            h[1] = __builtin_fmaf(hw_exp2(dv.x * a2[1]), h[1], dv.y * bv.y);
            float acc = __builtin_fmaf(cv.y, h[1], cv.x * h[0]);
            acc += __shfl_xor(acc, 1);
            acc += __shfl_xor(acc, 2);
            acc += __shfl_xor(acc, 4);
            if (q == 0) sums[t * kCh + j] = acc;
            if constexpr (REC == kPositions) {
                for (int64_t k0 = 0; k0 < p.npos; k0 += 64) {
                    const int pk = k0 == 0 ? pos0 : positions(k0);
                    for (uint64_t hit = __ballot(pk == (int)t0 + t); hit; hit &= hit - 1)
                        record(k0 + __builtin_ctzll(hit), h[0], h[1]);
                }
            }
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (2 * q + k >= nt) continue;
            float y = __builtin_fmaf(dskip, xs[k], sums[(2 * q + k) * kCh + j]);
            if (GATE) y *= gs[k];
            st_out<OUT>(yb, oa + t0 + k, y);
        }
    }

    // the wave of the last slice
    if (p.h_last && seg == g.nseg - 1 && (nt > 0 ? owns_tail : (nfull - 1 - r) % W == 0)) {
        p.h_last[row * kN + n0] = h[0];
        p.h_last[row * kN + n0 + 1] = h[1];
    }
}

// ---- host side ------------------------------------------------------------------

template <int IN, int OUT, bool GATE, bool SP>
hipError_t fwd_ring(ScanParams &p, const plan::Fwd &f, hipStream_t st, const float *carry) {
    RingParams g{};
    g.n_cg = (uint32_t)((p.dim + kCh - 1) / kCh);
    g.nseg = (uint32_t)f.nseg;
    g.seg_len = (uint32_t)f.seg_len;
    g.pieces = (uint32_t)f.pieces;
    g.chains = (uint32_t)f.chains;
    g.log_w = f.log_w;
    g.carry = carry;
    void *args[] = {&p, &g};
    const void *fn = p.npos > 0 ? reinterpret_cast<const void *>(&scan_fwd_ring<IN, OUT, GATE, SP, kPositions>)
                     : p.ck     ? reinterpret_cast<const void *>(&scan_fwd_ring<IN, OUT, GATE, SP, kCheckpoints>)
                                : reinterpret_cast<const void *>(&scan_fwd_ring<IN, OUT, GATE, SP, kPlain>);
    return hipLaunchKernel(fn, dim3((unsigned)f.workgroups), dim3(f.threads), args,
                           sizeof(WaveSmem) * (f.threads / 64) + 4 * kMaxWaves, st);
}

}  // namespace ring
}  // namespace mbs
