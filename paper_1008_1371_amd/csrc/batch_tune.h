// Speed-only choices of a batched solve: threads per workgroup of the persistent
// launch, and the sweep schedule (that launch, or launches grouped by order).
// Host code without HIP.
#pragma once
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <utility>

namespace hsvd {

// Before tuning: threads per workgroup for `problems` of at most nmax columns
// on `cus` compute units.  Threads beyond 256 work on further block pairs of
// the same problem, so a workgroup is no wider than the largest problem's
// pairs; few problems want the shortest solve, many the smallest workgroups (a
// compute unit then holds four problems in different phases).
// FP64, n ~ U{8..256}, 256 compute units, ms at 256 / 512 / 1024 threads:
// 300 problems 23.6 / 17.9 / 15.7, 600 29.1 / 23.8 / 19.6, 1000 39.1 / 28.7 /
// 29.8, 1500 46.8 / 42.0 / 44.1, 2200 58.9 / 61.3 / 65.4; U{8..128}, 400
// problems 6.0 / 4.4 / 4.4; mixed precision in the same proportions.
inline int default_threads(int problems, int nmax, int cus)
{
    const int widest = nmax <= 64 ? 256 : (nmax <= 128 ? 512 : 1024);
    return std::min(widest, problems <= 3 * cus ? 1024 : (problems <= 7 * cus ? 512 : 256));
}

// Before tuning: the persistent launch (0), but for few FP64 problems
// (bit-identical in both) the grouped ones (1), whose launches spread a
// problem's block pairs over the chip.  ms, persistent / grouped: 16 problems
// of n ~ U{8..256} 13.5 / 5.5, 300 15.6 / 11.6, 500 18.1 / 17.7; U{250..256} 16
// 14.0 / 5.0, 300 33.0 / 22.9, 500 37.6 / 35.1; U{100..220} 300 16.7 / 12.4,
// 500 20.0 / 21.8; U{65..128} 100 4.0 / 3.0, 200 4.2 / 4.3, 300 5.3 / 5.4;
// U{8..64} 100 1.7 / 1.6, 300 1.9 / 2.2.
inline int default_schedule(int problems, int nmax, int cus, bool mixed)
{
    return !mixed && problems <= (nmax > 128 ? 5 * cus / 4 : cus / 2) ? 1 : 0;
}

// What the autotuner chose.  A choice holds for the class of batch that it was
// timed on: by the number of problems per compute unit (the lines of the rules
// above), the width also by the largest order.  Timed on thousands of problems,
// the persistent launch at 256 threads wins; forced on 16 of order 250 to 256
// it takes 20.2 ms where the grouped launches take 4.6.
struct BatchTune {
    static constexpr int kOrders = 4, kCounts = 5;
    int threads[kOrders][kCounts] = {};  // 0: not tuned
    int sched[2][kCounts];               // FP64, mixed; -1: not tuned
    int last[2] = {-1, -1};              // the schedule tuned or read last

    BatchTune()
    {
        for (auto &of : sched) std::fill(of, of + kCounts, -1);
    }
    static int order_class(int nmax) { return std::min(kOrders - 1, (nmax - 1) / 64); }
    static int count_class(long long problems, int cus)
    {
        if (2 * problems <= cus) return 0;
        if (4 * problems <= 5 * cus) return 1;
        return problems <= 3 * cus ? 2 : (problems <= 7 * cus ? 3 : 4);
    }
    int threads_for(int problems, int nmax, int cus) const
    {
        const int t = threads[order_class(nmax)][count_class(problems, cus)];
        return t ? t : default_threads(problems, nmax, cus);
    }
    int schedule_for(int problems, int nmax, int cus, bool mixed) const
    {
        const int s = sched[mixed ? 1 : 0][count_class(problems, cus)];
        return s >= 0 ? s : default_schedule(problems, nmax, cus, mixed);
    }

    // Entries {"batched_bucket": B, "threads": T, "problems_class": C} and
    // {"batched_schedule": P, "mode": M, "problems_class": C}; without the class
    // they hold for every one.
    void read(const char *text)
    {
        auto classes = [](int items, int c) {
            return items == 2 ? std::make_pair(0, kCounts) : std::make_pair(c, c + 1);
        };
        for (const char *q = strstr(text, "\"batched_bucket\""); q; q = strstr(q + 1, "\"batched_bucket\"")) {
            int b = -1, t = 0, c = 0;
            const int items = sscanf(q, "\"batched_bucket\": %d, \"threads\": %d, \"problems_class\": %d", &b, &t, &c);
            if (items < 2 || b < 0 || b >= kOrders || c < 0 || c >= kCounts || (t != 256 && t != 512 && t != 1024)) continue;
            const auto cl = classes(items, c);
            std::fill(threads[b] + cl.first, threads[b] + cl.second, t);
        }
        for (const char *q = strstr(text, "\"batched_schedule\""); q; q = strstr(q + 1, "\"batched_schedule\"")) {
            int p = -1, m = -1, c = 0;
            const int items = sscanf(q, "\"batched_schedule\": %d, \"mode\": %d, \"problems_class\": %d", &p, &m, &c);
            if (items < 2 || (p != 0 && p != 1) || (m != 0 && m != 1) || c < 0 || c >= kCounts) continue;
            const auto cl = classes(items, c);
            std::fill(sched[p] + cl.first, sched[p] + cl.second, m);
            last[p] = m;
        }
    }
    // The entries, each after a comma but the file's first.
    void write(FILE *f, bool &first) const
    {
        auto next = [&] {
            const char *const sep = first ? "" : ",";
            first = false;
            return sep;
        };
        for (int b = 0; b < kOrders; ++b)
            for (int c = 0; c < kCounts; ++c)
                if (threads[b][c])
                    fprintf(f, "%s\n  {\"batched_bucket\": %d, \"threads\": %d, \"problems_class\": %d}", next(), b,
                            threads[b][c], c);
        for (int p = 0; p < 2; ++p)
            for (int c = 0; c < kCounts; ++c)
                if (sched[p][c] >= 0)
                    fprintf(f, "%s\n  {\"batched_schedule\": %d, \"mode\": %d, \"problems_class\": %d}", next(), p,
                            sched[p][c], c);
    }
};

}  // namespace hsvd
