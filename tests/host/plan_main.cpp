// Prints the forward's plan for each input line "batch dim L dstate in_bytes out_bytes gate aligned16 ckpt
// positions h0 cus" as "kernel nseg seg_len pieces waves_per_chain workgroups threads carry_bytes"; host code only.
#include <cstdio>

#include "fwd_plan.hpp"

static long long cus;

int main() {
    long long b, d, L, n;
    int in, out, gate, aligned, ckpt, positions, h0;
    while (std::scanf("%lld %lld %lld %lld %d %d %d %d %d %d %d %lld", &b, &d, &L, &n, &in, &out, &gate, &aligned, &ckpt,
                      &positions, &h0, &cus) == 12) {
        const mbs::plan::Fwd f = mbs::plan::fwd({b, d, L, n, in, out, gate != 0, aligned != 0, ckpt != 0, positions, h0 != 0},
                                               [] { return (int64_t)cus; });
        static const char *const names[] = {"row", "short", "ring", "chunk"};
        std::printf("%s %lld %lld %lld %u %lld %u %zu\n", names[f.kernel], (long long)f.nseg, (long long)f.seg_len,
                    (long long)f.pieces, 1u << f.log_w, (long long)f.workgroups, f.threads,
                    mbs::plan::carry_bytes(b * d, f));
    }
    return 0;
}
