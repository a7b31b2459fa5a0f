// CPU-only driver of the batch assembly's rounds (csrc/pod_plan.*), built with
// g++ by tests/test_host_rounds.py.  Prints one line per failed check.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "pod.h"
#include "pod_plan.h"

namespace {

int failures = 0;
void check(bool ok, const char* what, int line) {
    if (!ok) {
        std::printf("FAIL line %d: %s\n", line, what);
        ++failures;
    }
}
#define CHECK(x) check((x), #x, __LINE__)

struct Cells {
    std::vector<int> coff{0}, off{0}, longest;
    int n() const { return static_cast<int>(coff.size()) - 1; }
    void add(const std::vector<int>& lists) {
        for (int l : lists) off.push_back(off.back() + l);
        coff.push_back(static_cast<int>(off.size()) - 1);
        longest.push_back(lists.empty() ? 0 : *std::max_element(lists.begin(), lists.end()));
    }
};

constexpr size_t ENT = 100, ATOM = 1000;

size_t need(const Cells& s, int c) {
    const size_t nc = s.coff[c + 1] - s.coff[c];
    return nc * s.longest[c] * ENT + nc * ATOM;
}

// every cell is in one round, entries follow each other, no round of several
// cells is beyond the cap, and bytes is the largest round
void consistent(const Cells& s, const pod::BatchRounds& r, size_t cap) {
    const int nr = static_cast<int>(r.first.size()) - 1;
    CHECK(r.first.front() == 0 && r.first.back() == s.n() && static_cast<int>(r.n_ent.size()) == nr);
    size_t most = 0;
    for (int k = 0; k < nr; ++k) {
        CHECK(r.first[k] < r.first[k + 1]);
        size_t bytes = 0;
        long ent = 0, big = 0;
        for (int c = r.first[k]; c < r.first[k + 1]; ++c) {
            CHECK(r.ebase[c] == ent);
            const size_t nc = s.coff[c + 1] - s.coff[c];
            const long e = static_cast<long>((need(s, c) - nc * ATOM) / ENT);
            ent += e;
            big = std::max(big, e);
            bytes += need(s, c);
        }
        CHECK(r.n_ent[k] == ent && r.ent_max[k] == big);
        CHECK(bytes <= cap || r.first[k + 1] == r.first[k] + 1 || need(s, r.first[k]) > cap);
        most = std::max(most, bytes);
    }
    CHECK(r.bytes == most);
}

}  // namespace

int main() {
    Cells s;
    for (int c = 0; c < 37; ++c) {
        std::vector<int> lists(c % 5 == 4 ? 0 : 1 + (7 * c) % 11);
        for (size_t a = 0; a < lists.size(); ++a) lists[a] = static_cast<int>((13 * c + 5 * a) % 17);
        s.add(lists);
    }
    pod::BatchPlan plan;
    CHECK(pod::plan_batch(s.n(), s.coff.back(), s.off.back(), s.coff.data(), s.off.data(), 20, 160 * 1024, nullptr,
                          &plan) == POD_OK && plan.longest == s.longest);
    size_t all = 0, largest = 0;
    for (int c = 0; c < s.n(); ++c) {
        all += need(s, c);
        largest = std::max(largest, need(s, c));
    }
    pod::BatchRounds r;
    for (size_t cap : {all, all - 1, all / 2, all / 7, largest, largest - 1, size_t(1), size_t(0)}) {
        pod::plan_rounds(s.n(), s.coff.data(), s.longest.data(), ENT, ATOM, cap, &r);
        consistent(s, r, cap);
        if (cap >= all) CHECK(r.first.size() == 2);
        if (cap >= largest) CHECK(r.bytes <= cap);
    }
    // a device with `have` bytes: the rounds get smaller until they fit, and are
    // refused only when the largest cell alone does not
    for (size_t have : {all, all - 1, all / 3, 2 * largest, largest, largest - 1, size_t(0)}) {
        int calls = 0;
        const int rc = pod::fit_rounds(
            s.n(), s.coff.data(), s.longest.data(), ENT, ATOM, size_t(1) << 31,
            [&](size_t bytes) {
                ++calls;
                return bytes <= have ? POD_OK : POD_ENOMEM;
            },
            &r);
        CHECK(rc == (have >= largest ? POD_OK : POD_ENOMEM));
        CHECK(calls < 64);
        if (rc == POD_OK) CHECK(r.bytes <= have);
        consistent(s, r, size_t(-1));
    }
    // a round has at most BATCH_MAX_CELLS cells, whatever they need
    Cells empty;
    empty.coff.assign(2 * pod::BATCH_MAX_CELLS + 4, 0);
    empty.longest.assign(empty.n(), 0);
    pod::plan_rounds(empty.n(), empty.coff.data(), empty.longest.data(), ENT, ATOM, all, &r);
    CHECK((r.first == std::vector<int>{0, pod::BATCH_MAX_CELLS, 2 * pod::BATCH_MAX_CELLS, empty.n()}) && r.bytes == 0);
    // another answer ends the search
    int calls = 0;
    CHECK(pod::fit_rounds(s.n(), s.coff.data(), s.longest.data(), ENT, ATOM, all,
                          [&](size_t) { ++calls; return POD_EHIP; }, &r) == POD_EHIP && calls == 1);
    if (failures == 0) std::printf("host rounds: all checks passed\n");
    return failures == 0 ? 0 : 1;
}
