// Host check of qf::collect_size: a reverse walk that empties the buffer when the
// next gate's values do not fit never writes past it, in either order of the gates.
#include <cstdio>

#include "../paper_2409_17716_amd/csrc/qf_internal.h"

namespace qf {
qf_status set_error(qf_status st, const char*, ...) { return st; }
}

// Highest value written when the gates' values are laid down in order.
static size_t walk(const std::vector<size_t>& needs, size_t cap) {
    size_t used = 0, top = 0;
    for (size_t n : needs) {
        if (used + n > cap) used = 0;
        used += n;
        top = used > top ? used : top;
    }
    return top;
}

int main() {
    const size_t limit = size_t(8) << 20;
    // the rows of runs on registers of one large qudit and many small ones, and of
    // small ones only: 16 x 2^17 with 40 registers, 11 x 2^18 with 60, ...
    std::vector<std::vector<size_t>> lists = {{},
                                              {0},
                                              {1},
                                              {limit},
                                              {limit + 1, 1},
                                              {1, limit + 1},
                                              {10485760, 327680, 327680, 327680},
                                              {327680, 10485760, 327680},
                                              {8448000, 132000},
                                              std::vector<size_t>(40, 327680),
                                              {3 * limit, 2 * limit, limit, 5, limit / 2, limit / 2 + 1, 7}};
    uint64_t x = 88172645463325252ull;
    auto next = [&](uint64_t m) {
        x ^= x << 13;
        x ^= x >> 7;
        x ^= x << 17;
        return x % m;
    };
    for (int i = 0; i < 2000; ++i) {
        std::vector<size_t> l(1 + next(30));
        for (size_t& n : l) n = next(next(2) ? 2 * limit : limit / 8);
        lists.push_back(l);
    }
    long bad = 0;
    for (std::vector<size_t> l : lists)
        for (int rev = 0; rev < 2; ++rev) {
            const size_t cap = qf::collect_size(l, limit);
            size_t sum = 0, most = 1;
            for (size_t n : l) {
                sum += n;
                most = n > most ? n : most;
            }
            if (walk(l, cap) > cap || cap > (most > limit ? most : limit) || (sum > 0 && sum <= limit && cap < sum)) ++bad;
            l = std::vector<size_t>(l.rbegin(), l.rend());
        }
    std::printf("%s (%ld of %zu lists)\n", bad ? "FAIL" : "OK", bad, lists.size());
    return bad ? 1 : 0;
}
