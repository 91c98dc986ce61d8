// Host-only checks of the attention's split (wq_attn_plan.h) over the ranges
// that the entry point accepts (built with g++ by tests/test_host_logic.py).
#include <cstdio>
#include <initializer_list>

#include "wq_attn_plan.h"

static int failures = 0;

static void check(bool ok, const char* what, long long seqs, long long hkv, long long group, long long page, long long len) {
    if (!ok && ++failures <= 10)
        std::printf("FAIL %s: %lld sequences, %lld kv heads x %lld, page %lld, max_seq_len %lld\n", what, seqs, hkv, group, page, len);
}

int main() {
    using namespace wq::attn;
    for (int64_t seqs : {1, 2, 3, 16, 31, 32, 33, 64, 200, 511, 1024, 1025, 5000})
        for (int64_t hkv : {1, 2, 3, 4, 8, 16, 100, 256})
            for (int64_t group = 1; group <= 8; ++group)
                for (int64_t page = 1; page <= 1024; page *= 2)
                    for (int64_t len : {0, 1, 64, 192, 193, 512, 4096, 4097, 8191, 8193, 40960, 65536, 131072, 590000,
                                        1 << 20, (1 << 22) - 1, 1 << 22}) {
                        auto ck = [&](bool ok, const char* what) { check(ok, what, seqs, hkv, group, page, len); };
                        const Plan pl = make_plan(seqs, group * hkv, hkv, len, page, 512, true);
                        const Plan fixed = make_plan(seqs, group * hkv, hkv, len, page, 512, false);
                        ck(pl.chunk == fixed.chunk && pl.splits == fixed.splits, "the workspace depends on the lengths' split");
                        ck(make_plan(seqs, group * hkv, hkv, len, 1, 512, true).splits == pl.splits, "the workspace depends on the page");
                        // LDS of a workgroup: block-table entries and the states of four waves, in 64 KiB.
                        ck(chunk_pages(pl, page) * 4 + 16 + 4 * group * 130 * 4 <= 64 * 1024, "LDS");
                        if (!pl.units) continue;
                        const int64_t l = len > 1 ? len : 1;
                        ck(pl.units > seqs && pl.units <= seqs * pl.splits, "units");
                        // Cutting all sequences at their longest by the largest chunk takes no more than the units.
                        ck(seqs * ((l + pl.max_chunk - 1) / pl.max_chunk) <= pl.units, "longest chunk");
                        ck(pl.max_chunk % kChunkQuantum == 0, "quantum");
                    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
