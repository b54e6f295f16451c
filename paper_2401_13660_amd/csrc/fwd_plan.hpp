// fwd_plan.hpp -- which kernel a forward scan takes and how its work is cut: rules on
// sizes and alignment, in host code without a GPU call.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace mbs {
namespace plan {

constexpr int64_t kCh = 8;            // channels per chain
constexpr int64_t kSlice = 16;        // timesteps per slice of the ring kernel

enum Kernel {
    kRow,                             // one thread per row (scan_rowwise.hpp)
    kShort,                           // a sequence of 16 timesteps (scan_tiled.hpp)
    kRing,                            // slices dealt round the waves of a workgroup (scan_ring.hpp)
    kChunk,                           // one wave per chain, chunks of 32 timesteps (scan_chunk.hpp)
};

struct Shape {
    int64_t batch, dim, L, dstate;
    int in_bytes, out_bytes;          // per activation
    bool gate;
    bool aligned16;                   // every activation and y on a 16-byte boundary
    bool ckpt;                        // checkpoints are stored
    int64_t npos;                     // states recorded per batch element
    bool h0;                          // a first state is given
};

struct Fwd {
    Kernel kernel;
    int64_t chains;                   // of all time segments (kRing, kChunk)
    int64_t nseg, seg_len, pieces;    // time segments (1: none), their length, pre-pass pieces per segment
    uint32_t log_w;                   // waves per chain: 1 << log_w
    int64_t workgroups;
    uint32_t threads;                 // per workgroup
};

// HIP refuses a launch whose workgroups times threads along a grid dimension do not fit
// 32 bits.
inline bool launch_fits(int64_t workgroups, uint32_t threads) {
    return workgroups <= int64_t(0xFFFFFFFF) / threads;
}

// Chains of W waves in workgroups of 4 waves, or of W if that is more.
inline uint32_t ring_threads(uint32_t log_w) { return 64u * (log_w > 2 ? 1u << log_w : 4u); }
inline int64_t ring_workgroups(int64_t chains, uint32_t log_w) {
    const int64_t per_wg = log_w > 2 ? 1 : 4 >> log_w;
    return (chains + per_wg - 1) / per_wg;
}

// Waves per chain.  4 (one per SIMD) for most: measured with 1, 2, 4 and 8, bf16 in and
// fp32 out, (4, 3584, 8192) took 546, 541, 492 and 559 us, (4, 2048, 8192) 410, 306, 292 and
// 316, (1, 4608, 65536) 3123, 2296, 1583 and 1999, (1, 3584, 1013) 56, 34, 24 and 25: fewer
// waves leave SIMDs unevenly filled or idle, more make the chain's hand-overs its pace.
// 8 with at most one chain per CU ((1, 2048, 8192): 115 us with 4, 109 with 8).
// The waves of short sequences come in several rounds where chains are many, and each
// wave's start-up counts.  Measured with 1, 2, 4 waves, in us:
//   from 3 chains per CU    2 up to 8 slices     (2, 3584, 96)     8.5,  7.8,  8.3
//                           4 above              (2, 3584, 192)   13.0, 11.3, 10.9
//   from 4 chains per CU    1 up to 4 slices     (16, 3584, 48)   17.1, 19.6, 25.1
//                           2 up to 16           (2, 4608, 256)   20.0, 17.0, 16.3
//   from 7 chains per CU    1 up to 8            (4, 3584, 128)   12.2, 12.5, 14.4
//   from 8 chains per CU    2 up to 32           (8, 3584, 512)   63.4, 59.5, 60.4
//                           4 above              (8, 3584, 2048)   280,  243,  237
//   from 16 chains per CU   1 up to 16           (16, 3584, 256)  58.1, 59.6, 65.4
//                           2 up to 32           (32, 3584, 272)   151,  150,  162
// Fewer where the launch would not fit a grid dimension otherwise.
inline uint32_t waves_per_chain_log2(int64_t chains, int64_t slices, int64_t cus) {
    uint32_t lw = chains <= cus ? 3 : 2;
    if (chains > 4 * cus && slices <= 16)
        lw = slices <= 4 || (slices <= 8 && chains >= 7 * cus) || chains > 24 * cus ? 0 : 1;
    else if ((chains > 3 * cus && slices <= 8) || (chains > 11 * cus && slices <= 32))
        lw = 1;
    while (lw > 0 && ((int64_t(1) << lw) > slices || !launch_fits(ring_workgroups(chains, lw), ring_threads(lw)))) --lw;
    return lw;
}

// Time segments of the forward (1: none), their length and the pre-pass pieces per segment.
// A pre-pass computes each segment's aggregate from a zero state; the scan of segment s then
// starts from h0 folded with the aggregates of segments 0 .. s-1.  The pre-pass repeats the
// exponentials of all segments but the last, so the sequence is cut only where its chains
// leave the chip unevenly or hardly filled (bf16 in, us unsegmented and cut):
// - fewer than 7/8 of a chain per CU, into about 4 CUs' worth of chains, the fewer the
//   earlier: up to half a chain per CU from 2048 timesteps ((1, 1024, 2048), 128 chains, 30
//   and 26; (1, 64, 2048) 30 and 23, (1, 64, 1536) 23 either way); up to 5/8 from 3072 ((1,
//   1280, 3056), 160 chains, 43 and 40, (1, 1280, 2048) 30 either way); below 3/4 from 4096
//   ((1, 1528, 6000), 191 chains, 80 and 75, (1, 1528, 3056) 43 and 45); below 7/8 from 16384
//   ((1, 1536, 16384), 192 chains, 207 and 164, (1, 1792, 16384), 224 chains, 208 and 210), and
//   from 4/5 into 8 for evenness ((1, 1664, 16384), 208 chains, 209 in 4 and 191).
// - just over one chain per CU, where a few CUs take two and set the time, from 8192
//   timesteps into 8: (1, 2112, 8192), 264 chains, 146 and 129, (1, 2304, 32768), 288 chains,
//   571 and 492; (1, 2432, 16384), 304 chains, 287 and 307.
// Segments have at least 256 timesteps and number at most 128, for the fold over the earlier
// ones is serial: (1, 8, 65536) took 131 us in 256 segments of 2 pieces and 58 in 128.
// One wave of the pre-pass runs per piece and 8 channels; alone on its SIMD it waits on its
// chain of dependent operations.  A segment is cut into 2 or 4 pieces while that makes at
// most 4 waves per SIMD, of at least 512 and 768 timesteps: (1, 1024, 32768), 8 segments in
// 1, 2 and 4 pieces, 271, 249 and 248; (1, 1536, 16384), 5 segments in 2 and 4, 189 and 164;
// (1, 512, 8192), 16 segments of 512 timesteps in 1 and 2, 44 and 47; (1, 512, 32768), 16 of
// 2048 in 2 and 4, 125 and 128.  Shorter ones into 2 while there are at most 16 of them and that
// makes no more than one wave per SIMD: (1, 512, 2048), 8 of 256, 21.8 and 19.2; (1, 320, 4096),
// 16 of 256, 23.2 and 22.6, (1, 640, 4096), 16, 25.9 and 26.4, (1, 80, 6144), 24, 23.5 and 24.1.
inline int64_t segments(int64_t chains, int64_t L, int64_t cus, int64_t *seg_len, int64_t *pieces) {
    int64_t n = 1, m = 1;
    const int64_t least_L = chains * 8 <= cus * 4 ? 2048 : chains * 8 <= cus * 5 ? 3072
                            : chains * 8 < cus * 6 ? 4096 : 16384;
    if (chains * 8 < cus * 7 && L >= least_L) n = 4 * cus / chains;
    if (chains * 5 >= cus * 4 && n > 1) n = 8;
    if (chains > cus && chains * 8 <= cus * 9 && L >= 8192) n = 8;
    if (n > L / 256) n = L / 256;
    if (n > 128) n = 128;
    *seg_len = L;
    *pieces = 1;
    if (n <= 1) return 1;
    const int64_t least = (L + n - 1) / n;
    while (m < 4 && 2 * m * chains * (n - 1) <= 16 * cus && least >= (m == 1 ? 1024 : 3072)) m *= 2;
    if (m == 1 && n <= 16 && 2 * chains * (n - 1) <= 4 * cus) m = 2;
    const int64_t unit = 32 * m;                        // pieces of a multiple of 32 timesteps
    const int64_t len = (least + unit - 1) / unit * unit;
    *seg_len = len;
    *pieces = m;
    return (L + len - 1) / len;
}

// Time segments of the chunk kernel: with fewer than 3/8 of the waves that fill the chip at 2
// per SIMD, the most that make at most twice as many, of at least 256 timesteps; the pre-pass
// in 2 pieces per segment where that shortens the busiest SIMD's work, ceil(2 w / simds) / 2
// below ceil(w / simds) for the w waves of whole segments.
inline int64_t chunk_segments(int64_t chains, int64_t L, int64_t cus, int64_t *seg_len, int64_t *pieces) {
    const int64_t resident = 8 * cus, simds = 4 * cus;
    int64_t n = chains * 8 < resident * 3 ? 2 * resident / chains : 1, m = 1;
    if (n > L / 256) n = L / 256;
    *seg_len = L;
    *pieces = 1;
    if (n <= 1) return 1;
    const int64_t w = chains * (n - 1);
    if ((2 * w + simds - 1) / simds < 2 * ((w + simds - 1) / simds)) m = 2;
    const int64_t unit = 32 * m, len = ((L + n - 1) / n + unit - 1) / unit * unit;
    *seg_len = len;
    *pieces = m;
    return (L + len - 1) / len;
}

// The chunk kernel takes whole slices in aligned rows where it is the faster one: where a
// problem moves more bytes than the 256 MB of the Infinity Cache hold, or where its one wave
// per chain, 8 per CU at a time, fills the chip evenly.  In rows of an odd number of slices its
// loads of 32 timesteps straddle lines, and some of the rules leave those out.  In us, ring and
// chunk:
// - fp32 in, rounds of 8 chains per CU at least 7/8 full, even rows of 192 timesteps and more,
//   of any size: (4, 4096, 384) 34.1 and 30.7, (16, 4096, 256) 85 and 77, (4, 3840, 1024) 79
//   and 71; without recorded positions, for which this kernel takes a launch more;
// - fp32 in, more than 256 MB, above 6 chains per CU, rounds of 8 at least 5/8 full: (3, 4608,
//   2048) 164 and 145, (4, 3072, 2048), 6 exactly, 140 either way, (5, 3584, 8160) with
//   checkpoints, 8.75, 901 and 953, without a gate (5, 3584, 11072) 948 and 1084;
// - the same with checkpoints, also above 3 and up to 4: (4, 2048, 2304) 125 and 113, (1, 6144,
//   8160), 3 exactly, 320 and 377; and in even rows above 5: (1, 10648, 5632) 413 and 387, (2,
//   5632, 2640) 202 and 215;
// - bf16 in, with checkpoints, more than 256 MB: above 16 chains per CU, (16, 3584, 512) 150 and
//   138, (64, 3584, 256) 327 and 299; and above 4 where rounds of 4 chains per CU are at least
//   7/8 full, (8, 2048, 8160) 715 and 606, (7, 4608, 2304) 382 and 338, (5, 3584, 8160), 8.75
//   per CU, 782 and 880; with bf16 out 15/16, (8, 3072, 2304) 268 and 251, (7, 4096, 1024), 14
//   per CU, 138 and 144; from 192 timesteps, (91, 4608, 64) 162 and 183;
// - where states are recorded only with 128 timesteps for each, as it runs up to 32 timesteps
//   again for one: fp32 (38, 6304, 80) with 16 positions 459 and 616;
// - fp32 in, more than 256 MB beside the checkpoints, few chains, which both cut into segments:
//   from 1/4 to 7/8 of a chain per CU, (1, 1280, 65536) 700 and 631, (1, 512, 65536) 293 and 286,
//   (1, 1792, 65536) 819 and 883, of more than 768 MB from 1/8, (1, 256, 468736) 1092 and 1021;
//   and above 1, up to 1.2, (1, 2112, 16384) 307 and 268, (1, 2688, 16384) 315 and 326.
// The two kernels give the same bits except where they cut a sequence into other segments, and
// storing checkpoints or recording positions must not change them: only the last rule chooses
// for a problem that is cut, and it asks for neither.
inline bool chunk_is_faster(const Shape &s, int64_t chains, int64_t cus) {
    if (!s.aligned16 || s.L % kSlice != 0) return false;
    const bool even = s.L % 32 == 0;
    const int64_t per_step = s.in_bytes * (s.gate ? 3 : 2) + s.out_bytes;
    auto moves_more_than = [&](int64_t mib, int64_t bytes) { return s.batch * s.dim > (mib << 20) / (s.L * bytes); };
    // do the chains fill num/den of their rounds of k per CU?
    auto filled = [&](int64_t k, int64_t num, int64_t den) {
        const int64_t round = k * cus, rounds = (chains + round - 1) / round;
        return chains * den >= rounds * round * num;
    };
    if (chains <= 3 * cus) {
        if (s.in_bytes == 2 || !moves_more_than(256, per_step)) return false;
        if (chains < cus) return chains * (moves_more_than(768, per_step) ? 8 : 4) >= cus && chains * 8 < cus * 7;
        return chains > cus && chains * 5 <= cus * 6;
    }
    if (s.in_bytes == 4 && s.npos == 0 && even && s.L >= 192 && filled(8, 7, 8)) return true;
    if (!moves_more_than(256, per_step + (s.ckpt ? 4 : 0)) || s.L < 128 * s.npos) return false;
    if (s.in_bytes == 2)
        return s.ckpt && s.L >= 192 && (chains > 16 * cus || (chains > 4 * cus && (s.out_bytes == 4 ? filled(4, 7, 8) : filled(4, 15, 16))));
    return (chains > 6 * cus && filled(8, 5, 8)) || (s.ckpt && (chains <= 4 * cus || (even && chains > 5 * cus)));
}

// The row kernel takes a few timesteps of many rows that start from zero: a wave of the ring
// kernel is set up for 8 channels, one of the row kernel for 64 rows, but it reads first states
// row by row.  In us, ring and row, with a gate, y in the inputs' type:
// - bf16 in, up to 8 timesteps, from 16 chains per CU and 16 more per timestep: (16, 4608, 1), 36
//   per CU, 8.0 and 7.4, with 2 8.7 and 8.9; (28, 4608, 2), 63, 13.1 and 11.7, with 3 13.8 and
//   13.7; (64, 4608, 8), 144, 42 and 39; (200, 3584, 2), 350, 62 and 45;
// - fp32 in, up to 4, from 8 and 24 more: (16, 4608, 1) 7.7 and 7.3, (28, 4608, 2) 12.5 and 11.7,
//   with 3 13.4 and 14.2; (200, 3584, 3) 63 and 52, with 6 77 and 90;
// - with a first state, bf16 (64, 4608, 2) 29.5 and 29.8, (200, 3584, 4) 75 either way.
// Not where states are recorded: bf16 (31, 5112, 1) with 8 positions 26 and 60.  The row kernel
// forms its sums in the order of the ring kernel's last timesteps, so that recording changes no
// bit.
inline bool row_is_faster(const Shape &s, int64_t chains, int64_t cus) {
    if (s.h0 || s.npos > 0) return false;
    return s.in_bytes == 2 ? s.L <= 8 && chains >= (16 + 16 * s.L) * cus : s.L <= 4 && chains >= (8 + 24 * s.L) * cus;
}

// The plan of a scan with at least one row and one timestep; cus_of says how many compute
// units the device has, asked only where a rule needs it.
inline Fwd fwd(const Shape &s, int64_t (*cus_of)()) {
    Fwd f{kRow, 0, 1, s.L, 1, 0, 0, 64};
    const int64_t rows = s.batch * s.dim, base = s.batch * ((s.dim + kCh - 1) / kCh);
    f.workgroups = (rows + 63) / 64;
    // The kernels of dstate 16 take any length below 2^25 (32-bit lane offsets inside a
    // wave's rows: 16 rows x L x 4 bytes < 2^32) and as many chains as one wave each fits a
    // launch (below 2^26); the row kernel's launch holds 8 times as many.
    if (s.dstate != 16 || s.L >= (int64_t(1) << 25) || !launch_fits(ring_workgroups(base, 0), ring_threads(0))) return f;
    // The 16-timestep kernel takes the verify shape: one slice, 16-byte aligned rows (its
    // loads are wider), no checkpoints, the batch in the grid's second dimension.
    if (s.L == 16 && s.aligned16 && !s.ckpt && s.batch <= 65535) {
        f.kernel = kShort;
        f.workgroups = ((s.dim + kCh - 1) / kCh + 3) / 4;
        f.threads = 256;
        return f;
    }
    const int64_t cus = cus_of();
    if (row_is_faster(s, base, cus)) return f;
    if (chunk_is_faster(s, base, cus)) {
        f.kernel = kChunk;
        f.nseg = chunk_segments(base, s.L, cus, &f.seg_len, &f.pieces);
        f.chains = base * f.nseg;
        f.workgroups = (f.chains + 3) / 4;
        f.threads = 256;
        return f;
    }
    f.kernel = kRing;
    f.nseg = segments(base, s.L, cus, &f.seg_len, &f.pieces);
    f.chains = base * f.nseg;
    f.log_w = waves_per_chain_log2(f.chains, (f.seg_len + kSlice - 1) / kSlice, cus);
    f.workgroups = ring_workgroups(f.chains, f.log_w);
    f.threads = ring_threads(f.log_w);
    return f;
}

// Device bytes of the segment carry: the aggregates of the pieces of segments
// 0 .. nseg-2, then the copy of h0 (rows x 16 states x 2 floats per plane).
inline size_t carry_bytes(int64_t rows, const Fwd &f) {
    return f.nseg > 1 ? (size_t)(f.pieces * (f.nseg - 1) + 1) * (size_t)rows * 16 * 2 * sizeof(float) : 0;
}

}  // namespace plan
}  // namespace mbs
