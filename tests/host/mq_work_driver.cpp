// The work of the many-row kernel's workgroups, on the CPU by the code the kernel compiles (csrc/octopus_decode_mq.hpp).  Arguments: sequences,
// KV heads, splits, row blocks, 1 if the order is spread; one line per workgroup that has work: die, pair, split, block; "spreads" and the same but
// max_len in the last place: whether the kernel spreads the call.  Built by tests/test_many_rows_work.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "octopus_decode.hpp"
#include "octopus_decode_mq.hpp"

int main(int argc, char **argv) {
    const bool ask = argc == 7 && std::strcmp(argv[1], "spreads") == 0;
    if (argc != 6 && !ask) return 2;
    char **a = argv + (ask ? 2 : 1);
    const uint32_t seqs = std::atoi(a[0]), kv = std::atoi(a[1]), splits = std::atoi(a[2]), blocks = std::atoi(a[3]), n = seqs * kv * splits * blocks;
    if (ask) {
        std::printf("%d\n", octopus::mq_spreads(seqs, splits, std::atoi(a[4]), n) ? 1 : 0);
        return 0;
    }
    for (uint32_t b = 0; b < (n + 7) / 8 * 8; ++b) {
        const uint32_t at = octopus::mq_position(b, n);
        if (at >= n) continue;
        const octopus::MqWork w = octopus::mq_work(at, seqs, kv, splits, blocks, std::atoi(a[4]) != 0);
        std::printf("%u %u %u %u\n", b % 8, w.pair, w.split, w.grp);
    }
    return 0;
}
