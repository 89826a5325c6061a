// The library's own classical CF splitting: the Ruge-Stueben first pass
// without a second pass (the splitting the paper uses, Sec. 4).  It is a
// greedy sequential algorithm, so it runs on the host between the device
// strength kernel and the device neighbourhood kernels.
//
// Measure lambda_i = number of points that strongly depend on i.  Points
// with no strong connection in either direction are F.  Repeatedly the
// undecided point with the largest measure (smallest index among equals)
// becomes C; the undecided points depending on it become F and every
// undecided point those new F-points depend on gains one; the undecided
// points the new C-point depends on lose one.  When the largest remaining
// measure is zero the rest become F.
//
// The points of one measure are a set of bits with two levels of summary
// bits: a point moves between measures in a few word operations, and the
// smallest index of the largest measure is three find-first steps.  (A binary
// heap of (measure, index) with stale entries: a 97 x 97 five-point grid 1.17 ms,
// 1000 x 1000 259 ms; the sets 0.37 and 72 ms.)  Measures of MAX_SETS and more, rare, wait in such a
// heap.
#include <cstddef>
#include <cstdint>
#include <queue>
#include <utility>
#include <vector>

namespace lair {

namespace {

// A set of the integers 0 .. n - 1.
class BitSet {
public:
    explicit BitSet(int64_t n)
        : n0_((size_t)((n + 63) >> 6)), n1_((n0_ + 63) >> 6), n2_((n1_ + 63) >> 6),
          w_(n0_ + n1_ + n2_, 0) {}
    bool empty() const { return count_ == 0; }
    void insert(int64_t i) {
        w_[(size_t)(i >> 6)] |= bit(i);
        w_[n0_ + (size_t)(i >> 12)] |= bit(i >> 6);
        w_[n0_ + n1_ + (size_t)(i >> 18)] |= bit(i >> 12);
        ++count_;
    }
    void erase(int64_t i) {
        --count_;
        if (w_[(size_t)(i >> 6)] &= ~bit(i)) return;
        if (w_[n0_ + (size_t)(i >> 12)] &= ~bit(i >> 6)) return;
        w_[n0_ + n1_ + (size_t)(i >> 18)] &= ~bit(i >> 12);
    }
    int64_t smallest() const {               // not empty
        size_t k = 0;
        while (w_[n0_ + n1_ + k] == 0) ++k;
        int64_t i = (int64_t)(k << 6) + __builtin_ctzll(w_[n0_ + n1_ + k]);
        i = (i << 6) + __builtin_ctzll(w_[n0_ + (size_t)i]);
        return (i << 6) + __builtin_ctzll(w_[(size_t)i]);
    }

private:
    static uint64_t bit(int64_t i) { return (uint64_t)1 << (i & 63); }
    size_t n0_, n1_, n2_;
    std::vector<uint64_t> w_;
    int64_t count_ = 0;
};

constexpr int32_t MAX_SETS = 64;

}  // namespace

void rs_first_pass(int64_t n, const int32_t *rp, const int32_t *cj,
                   const uint8_t *sm, int8_t *cf) {
    // the strong entries, and their transpose
    std::vector<int32_t> sp((size_t)n + 1), sj, tp((size_t)n + 1, 0);
    sj.reserve((size_t)rp[n]);
    for (int64_t i = 0; i < n; ++i) {
        sp[(size_t)i] = (int32_t)sj.size();
        for (int32_t p = rp[i]; p < rp[i + 1]; ++p)
            if (sm[p]) {
                sj.push_back(cj[p]);
                tp[(size_t)cj[p] + 1]++;
            }
    }
    sp[(size_t)n] = (int32_t)sj.size();
    for (int64_t i = 0; i < n; ++i) tp[(size_t)i + 1] += tp[(size_t)i];
    std::vector<int32_t> tj(sj.size());
    {
        std::vector<int32_t> fill(tp.begin(), tp.end() - 1);
        for (int64_t i = 0; i < n; ++i)
            for (int32_t p = sp[(size_t)i]; p < sp[(size_t)i + 1]; ++p)
                tj[(size_t)fill[(size_t)sj[(size_t)p]]++] = (int32_t)i;
    }
    enum : int8_t { UNDECIDED = -1, FPT = 0, CPT = 1 };
    std::vector<int8_t> st((size_t)n, UNDECIDED);
    std::vector<int32_t> lam((size_t)n, 0);
    std::vector<BitSet> sets;
    using Key = std::pair<int32_t, int32_t>;   // (measure, -index)
    std::priority_queue<Key> high;             // entries may be stale
    int32_t top = -1;                          // no set above it has a member
    auto enter = [&](int32_t k) {
        const int32_t m = lam[(size_t)k];
        if (m >= MAX_SETS) {
            high.push(Key(m, -k));
            return;
        }
        while ((int32_t)sets.size() <= m) sets.emplace_back(n);
        sets[(size_t)m].insert(k);
        if (m > top) top = m;
    };
    auto leave = [&](int32_t k) {
        if (lam[(size_t)k] < MAX_SETS) sets[(size_t)lam[(size_t)k]].erase(k);
    };
    for (int32_t i = 0; i < n; ++i) {
        lam[(size_t)i] = tp[(size_t)i + 1] - tp[(size_t)i];
        if (sp[(size_t)i + 1] == sp[(size_t)i] && lam[(size_t)i] == 0) st[(size_t)i] = FPT;
        else enter(i);
    }
    auto bump = [&](int32_t k, int32_t d) {
        leave(k);
        lam[(size_t)k] += d;
        enter(k);
    };
    for (;;) {
        int32_t i = -1;
        while (!high.empty() && i < 0) {
            const Key key = high.top();
            high.pop();
            const int32_t k = -key.second;
            if (st[(size_t)k] == UNDECIDED && lam[(size_t)k] == key.first) i = k;
        }
        if (i < 0) {
            while (top >= 0 && sets[(size_t)top].empty()) --top;
            if (top <= 0) break;             // the rest become F
            i = (int32_t)sets[(size_t)top].smallest();
            sets[(size_t)top].erase(i);
        }
        st[(size_t)i] = CPT;
        for (int32_t q = tp[(size_t)i]; q < tp[(size_t)i + 1]; ++q) {
            const int32_t j = tj[(size_t)q];
            if (st[(size_t)j] != UNDECIDED) continue;
            st[(size_t)j] = FPT;
            leave(j);
            for (int32_t p = sp[(size_t)j]; p < sp[(size_t)j + 1]; ++p)
                if (st[(size_t)sj[(size_t)p]] == UNDECIDED) bump(sj[(size_t)p], +1);
        }
        for (int32_t p = sp[(size_t)i]; p < sp[(size_t)i + 1]; ++p)
            if (st[(size_t)sj[(size_t)p]] == UNDECIDED) bump(sj[(size_t)p], -1);
    }
    for (int64_t i = 0; i < n; ++i) cf[i] = st[(size_t)i] == CPT ? 1 : 0;
}

}  // namespace lair
