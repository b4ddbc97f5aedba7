// Merge of the ordering's sequences into one order (BGL paper, Sec. 3.2.2).  Host code only, so that it can be tested without
// a GPU.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace bgl {

// Turn t takes the next node of sequence t mod S that no earlier turn has taken.  One bit per
// node says which are taken (a byte each is eight times the cache: 2.45 M nodes, two sequences of 204,800: 0.4 ms instead of
// 0.9).  Many sequences are looked through 64 entries at a time, without a branch for each: all of them are read almost to
// their end, and most entries are taken (ten of 100,000 on 1 M nodes: a call 6.4 -> 6.1 ms; two of 500,000 3.6 -> 3.75).
// It goes on as far as the sequences are there, so that most of it is done by the time the traversals end, and looks at no more
// than so many entries at a time, however many in a row are taken: nobody enqueues work for the device meanwhile.
class OrderMerge {
    static constexpr size_t ONE_BY_ONE = 3;  // sequences that are looked through entry by entry
    struct Reader {
        int64_t at;         // next place to look at, cyclically from the shift
        int64_t first = 0;  // the last 64 looked at begin here
        uint64_t open = 0;  // those of them that were not taken then and have not been looked at again
    };
    const int32_t *seqs;
    int64_t num_train, num_out;
    int32_t *order;
    std::vector<uint64_t> used;
    std::vector<Reader> readers;
    int64_t k = 0;             // turns taken
    size_t j = 0;              // whose turn it is

    // What a run of turns works on, in registers: the marks of taken nodes could be any of the members otherwise.
    struct Run {
        uint64_t *const used;
        const int64_t num_train;
        int64_t left;  // entries that may still be looked at
        bool taken(int32_t v) const { return used[(size_t)v / 64] >> (v % 64) & 1u; }
        // The next node of a sequence that nobody has taken, or -1 if its entry is not there yet or none may be looked at any
        // more.  (What has been passed over is taken and stays so.)
        int32_t next(Reader &r, const int32_t *seq, int64_t limit)
        {
            int64_t c = r.at, n = left;
            int32_t v;
            do {
                if (c >= limit || n == 0) {
                    r.at = c;
                    left = n;
                    return -1;
                }
                v = seq[c];
                --n;
                c = c + 1 == num_train ? 0 : c + 1;
            } while (taken(v));
            r.at = c;
            left = n;
            return v;
        }
        int32_t next_of_64(Reader &r, const int32_t *seq, int64_t limit)
        {
            for (;;) {
                for (; r.open; r.open &= r.open - 1) {
                    const int32_t v = seq[r.first + __builtin_ctzll(r.open)];
                    if (!taken(v)) {
                        r.open &= r.open - 1;
                        return v;
                    }
                }
                const int64_t n = std::min<int64_t>(std::min<int64_t>(limit - r.at, left), 64);
                if (n <= 0) return -1;
                for (int64_t i = 0; i < n; ++i) r.open |= (uint64_t)!taken(seq[r.at + i]) << i;
                left -= n;
                r.first = r.at;
                r.at = r.at + n == num_train ? 0 : r.at + n;
            }
        }
    };

public:
    std::vector<int64_t> there;  // leading entries of each sequence that may be read

    OrderMerge(const int32_t *seqs_, int32_t num_sequences, const int64_t *shifts, int64_t num_train_, int64_t num_nodes,
               int64_t num_out_, int32_t *order_, int64_t there_)
        : seqs(seqs_), num_train(num_train_), num_out(num_out_), order(order_), used((size_t)((num_nodes + 63) / 64), 0),
          there((size_t)num_sequences, there_)
    {
        for (int32_t s = 0; s < num_sequences; ++s) readers.push_back(Reader{shifts[s]});
    }
    // Looks at so many entries at most; those it has looked at.  0: there was nothing to do.
    int64_t go_on(int64_t entries)
    {
        Run run{used.data(), num_train, entries};
        const size_t sequences = readers.size();
        Reader *const reader = readers.data();
        const int64_t *const limits = there.data();
        int64_t turn = k;
        size_t s = j;
        while (turn < num_out) {
            const int32_t *seq = seqs + s * (size_t)num_train;
            const int32_t v = sequences > ONE_BY_ONE ? run.next_of_64(reader[s], seq, limits[s]) : run.next(reader[s], seq, limits[s]);
            if (v < 0) break;
            run.used[(size_t)v / 64] |= 1ull << (v % 64);
            order[turn++] = v;
            s = s + 1 == sequences ? 0 : s + 1;
        }
        k = turn;
        j = s;
        return entries - run.left;
    }
    // To the end; all entries have to be there.
    void finish() { go_on(INT64_MAX); }
};

}  // namespace bgl
