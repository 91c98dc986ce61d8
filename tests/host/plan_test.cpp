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
    // Two rows of x: a linear alone in its launch takes the kernel that
    // wq_gemv picks for it; with others, or at other batches, the planned one.
    struct {
        int64_t n, k;
        bool vector;
    } const pairs[] = {
        {1, 3104, true},      {2048, 3104, true},    {2048, 3072, false},  {2049, 4096, false},   {512, 16384, true},
        {2049, 8192, true},   {3072, 6176, true},    {3072, 6144, false},  {3073, 8192, false},   {4096, 14336, true},
        {6144, 14336, true},  {7168, 14336, false},  {4096, 10240, false}, {4096, 4096, false},   {8192, 4096, false},
        {10240, 4096, true},  {10241, 4096, false},  {9216, 4096, false},  {12288, 4096, true},   {14336, 4096, false},
        {10240, 14336, true}, {12288, 14336, false}, {14336, 8192, true},  {14592, 8192, false},  {24576, 4096, true},
        {25600, 4096, false}, {28672, 4096, false},  {40960, 8192, true},  {41984, 8192, false},  {28928, 3584, false},
        {20480, 5120, false}, {128256, 3072, false}, {3072, 3072, false},  {16384, 3072, false},  {3200, 7168, false},
    };
    for (const auto& p : pairs) {
        char what[96];
        std::snprintf(what, sizeof(what), "%lld x %lld alone at M=2 by the vector kernel", (long long)p.n, (long long)p.k);
        expect(wq::vector_takes_pair(p.n, p.k), p.vector, what);
        expect(!split({linear(0, p.n, p.k)}, 2)[0].grouped, p.vector, what);
        // A list that closes before it: the second linear reads the first one's y.
        wq_linear dep = linear(1, p.n, p.k);
        const wq_linear before = linear(0, 64, 64);
        dep.x = before.y;
        const auto g = split({before, dep}, 2);
        expect(g.size() == 2 && g[0].grouped && !g[1].grouped, p.vector, what);
        expect(split({linear(0, p.n, p.k), linear(1, 64, 64)}, 2)[0].grouped, true, "two linears");
        expect(split({linear(0, p.n, p.k)}, 3)[0].grouped, true, "three rows");
    }
    if (failures) return 1;
    std::printf("ok\n");
    return 0;
}
