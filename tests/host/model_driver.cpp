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
            plan_split(&db, 0, db.nseq, &none, plan, M, &b, a);
            std::printf("%d %d %d\n", b, a.nsegs, a.nlong);
        } else {
            std::printf("? %s", line);
        }
    }
    return 0;
}
