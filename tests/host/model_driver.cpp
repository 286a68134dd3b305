// Runs the host code that chooses plans, cuts and grids, without a GPU, for
// tests/test_plan_model.py: one command per line of standard input, one line of
// results each.  Built together with the library's host source.
#include <cstdio>
#include <cstring>
#include <string>

#include "hmsv_host.cpp"

namespace {

int no_blocks(int, int) { return 0; }

// A database of the given lengths (any order), host side only.
hmsv_db make_db(std::vector<int64_t> len, bool degenerate) {
    std::sort(len.begin(), len.end(), [](int64_t a, int64_t b) { return a > b; });
    hmsv_db db;
    db.nseq = (int64_t)len.size();
    db.table_rows = degenerate ? kDegenRows : kRows;
    db.cum_rows.assign(1, 0);
    for (int64_t l : len)
        db.cum_rows.push_back(db.cum_rows.back() + std::max<int64_t>(4, (l + 3) & ~(int64_t)3));
    return db;
}

}  // namespace

int main() {
    static const KernelEntry none{0, 1, 1, nullptr, no_blocks};
    for (int is_msv = 0; is_msv < 2; ++is_msv)
        for (int g = 1; g <= 64; g *= 2)
            for (int q = 1; q <= (g == 1 ? 32 : g == 32 ? 60 : g == 64 ? 30 : 64); ++q) {
                const KernelEntry k{is_msv, g, q, nullptr, no_blocks};
                register_kernels(&k, 1);
            }
    for (int g = 4; g <= 64; g *= 2)
        for (int q = 1; q <= (g == 64 ? 22 : 16); ++q) {
            const P7KernelEntry k{g, q, nullptr, nullptr};
            register_p7_kernels(&k, 1);
        }
    char line[256];
    while (std::fgets(line, sizeof line, stdin)) {
        long long n = 0, len = 0;
        int G = 0, Q = 0, w = 0, blocks = 0, M = 0;
        if (std::sscanf(line, "grid %lld %lld %d %d %d %d %d", &n, &len, &M, &G, &Q, &w, &blocks) == 7) {
            // the blocks of a call with a plan's own grid on n sequences of len residues
            const hmsv_db db = make_db(std::vector<int64_t>((size_t)n, len), false);
            const hmsv_plan plan{G, Q, w, blocks};
            KArgs a{};
            int b = blocks;
            plan_split(&db, 0, db.nseq, &none, plan, M, &b, a, 256);
            std::printf("%d %d %d\n", b, a.nsegs, a.nlong);
        } else if (std::sscanf(line, "lds %lld", &n) == 1) {
            // blocks of n bytes of LDS that fit a CU
            std::printf("%d\n", lds_blocks((size_t)n));
        } else if (std::sscanf(line, "waves %d %d %d %lld %d", &G, &Q, &w, &n, &blocks) == 5) {
            // wavefronts per block of an untuned plan: w table rows, n sequences
            std::printf("%d\n", block_waves(G, Q, w, n, blocks));
        } else if (std::sscanf(line, "plan %d %d %d %lld %d", &w, &M, &G, &n, &blocks) == 5) {
            // the plan and cut of filter w (0 SSV, 1 MSV, 2 P7Viterbi) at M on G compute
            // units, for `blocks` copies of n sequences of 40..1039 residues
            std::vector<int64_t> lens;
            for (int64_t i = 0; i < n; ++i)
                for (int c = 0; c < blocks; ++c) lens.push_back(40 + (i * 997) % 1000);
            const hmsv_db db = make_db(lens, false);
            hmsv_plan p{};
            if (w == 2) {
                if (hmsv_p7_default_plan(M, &p) != HMSV_OK) return 1;
                p7_choose(&db, M, &p, G);
                std::printf("%d %d %d 0 0\n", p.G, p.Q, p.waves_per_block);
                continue;
            }
            const Range r{db.cum_rows.data(), db.nseq};
            if (resolve_plan(w, M, db.table_rows, r, nullptr, &p, G) != HMSV_OK) return 1;
            const int64_t groups =
                (int64_t)G * resident_waves(p.G, p.Q, p.waves_per_block, kRows) * (64 / p.G);
            const Cut c = choose_cut(r, M, p.G, p.Q, groups, G);
            std::printf("%d %d %d %lld %lld\n", p.G, p.Q, p.waves_per_block, (long long)c.limit,
                        (long long)c.seg);
        } else {
            std::printf("? %s", line);
        }
    }
    return 0;
}
