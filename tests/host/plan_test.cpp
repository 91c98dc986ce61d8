// Host-only checks of how a descriptor list is split into launches
// (wq_plan.h), built with g++ by tests/test_host_logic.py.  Addresses are
// made up; nothing is dereferenced.
#include <cstdio>
#include <vector>

#include "wq_plan.h"

static int failures = 0;

static void expect(bool got, bool want, const char* what) {
    if (got != want) {
        std::printf("FAIL %s: got %d, want %d\n", what, (int)got, (int)want);
        ++failures;
    }
}

static std::vector<wq::plan::Group> split(const std::vector<wq_linear>& lin, int64_t m) {
    std::vector<wq::plan::Group> groups;
    wq::plan::SpanSet reads, writes;
    wq::plan::split_groups(lin.data(), (int)lin.size(), m, reads, writes,
                           [&](const wq::plan::Group& g) { groups.push_back(g); });
    return groups;
}

// A linear whose buffers lie in a region of its own.
static wq_linear linear(int i, int64_t n, int64_t k) {
    const uintptr_t base = (uintptr_t)(i + 1) << 42;
    wq_linear l{};
    l.packed_w = reinterpret_cast<const uint32_t*>(base);
    l.scales = reinterpret_cast<const uint16_t*>(base + ((uintptr_t)1 << 40));
    l.x = reinterpret_cast<const uint16_t*>(base + ((uintptr_t)2 << 40));
    l.y = reinterpret_cast<uint16_t*>(base + ((uintptr_t)3 << 40));
    l.N = n;
    l.K = k;
    return l;
}

int main() {
    // x of m rows behind one 32-bit buffer: K where it ends, one group below
    // and above; batches
    // of the matrix-core plans and lists.
    for (int64_t m : {2, 3, 4, 16, 64, 65, 128}) {
        const int64_t k_at = (int64_t)wq::kPrefillOutOffset / 2 / m / 32 * 32;
        expect(wq::gemm_fits(1, k_at, m), true, "x at the out-of-range offset");
        expect(wq::gemm_fits(1, k_at + 32, m), false, "x one group past it");
        for (int64_t k : {k_at - 32, k_at, k_at + 32}) {
            const auto g = split({linear(0, 512, 4096), linear(1, 1, k), linear(2, 512, 4096)}, m);
            char what[96];
            std::snprintf(what, sizeof(what), "M=%d K=%lld in a matrix-core launch", (int)m, (long long)k);
            bool grouped = false;
            for (const auto& x : g)
                if (x.begin <= 1 && 1 < x.end) grouped = x.grouped;
            expect(grouped, k <= k_at, what);
        }
    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
