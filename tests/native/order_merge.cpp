// The merge of the ordering's sequences against a plain one, its entries coming in piece by piece, and no call of it longer
// than it was allowed to be (built and run by tests/test_order_native.py; no GPU).
#include <cstdio>
#include <numeric>
#include <random>

#include "bgl_order_merge.h"

int main()
{
    std::mt19937_64 rng(7);
    auto below = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
    int64_t longest_run = 0;
    for (int round = 0; round < 400; ++round) {
        const int sequences = 1 + (int)below(round % 2 ? 3 : 20);
        const int64_t num_train = 1 + below(round % 5 ? 300 : 20'000), num_nodes = num_train + below(100);
        const int64_t num_out = round % 3 ? num_train : below(num_train + 1);
        std::vector<int32_t> ids((size_t)num_nodes);
        std::iota(ids.begin(), ids.end(), 0);
        std::shuffle(ids.begin(), ids.end(), rng);
        ids.resize((size_t)num_train);
        std::vector<int32_t> seqs;
        std::vector<int64_t> shifts;
        for (int s = 0; s < sequences; ++s) {
            // alike, reversed, in parts that others have in another place (long runs of taken entries), or in no order
            std::vector<int32_t> one = ids;
            if (round % 4 == 1) std::reverse(one.begin(), one.end());
            if (round % 4 == 2) std::rotate(one.begin(), one.begin() + s * num_train / sequences, one.end());
            if (round % 4 == 3 && s) std::shuffle(one.begin(), one.end(), rng);
            seqs.insert(seqs.end(), one.begin(), one.end());
            shifts.push_back(below(3) ? below(num_train) : 0);
        }
        std::vector<int32_t> want, order((size_t)num_train, -1);
        std::vector<char> taken((size_t)num_nodes, 0);
        std::vector<int64_t> at = shifts;
        for (int64_t t = 0; t < num_out; ++t) {
            const int s = (int)(t % sequences);
            int64_t run = 0;
            for (;; ++run) {
                const int32_t v = seqs[(size_t)(s * num_train + at[s])];
                at[s] = (at[s] + 1) % num_train;
                if (taken[(size_t)v]) continue;
                taken[(size_t)v] = 1;
                want.push_back(v);
                break;
            }
            longest_run = std::max(longest_run, run);
        }
        want.resize((size_t)num_train, -1);
        bgl::OrderMerge merge(seqs.data(), sequences, shifts.data(), num_train, num_nodes, num_out, order.data(), 0);
        for (bool all = false; !all;) {
            all = true;
            for (int64_t &n : merge.there) {
                n = std::min(num_train, n + below(2) * below(num_train / 4 + 2));
                all &= n == num_train;
            }
            const int64_t most = 1 + below(200), made = merge.go_on(most);
            if (made < 0 || made > most) {
                printf("round %d: %lld entries instead of %lld\n", round, (long long)made, (long long)most);
                return 1;
            }
        }
        if (round % 7 == 0)
            for (int64_t made = 1; made > 0;) {
                made = merge.go_on(100);
                if (made > 100) return printf("round %d: %lld entries instead of 100\n", round, (long long)made), 1;
            }
        else
            merge.finish();
        if (order != want) return printf("round %d: another order\n", round), 1;
    }
    if (longest_run < 5'000) return printf("no long run of taken entries: %lld\n", (long long)longest_run), 1;
    printf("ok %lld\n", (long long)longest_run);
    return 0;
}
