// Every order in which the workgroups that carry the second phase of a
// re-layout can run (pic_relayout.hpp): drawn schedules in which a workgroup
// may be held up before each thing it does while others start or go on.
#include <cstdio>
#include <functional>
#include <random>
#include <vector>

#include "pic_relayout.hpp"

struct State {
    bool rebin;
    int step = 0, finished = 0, ticket = 0, copied = 0;
    bool bad = false;
    std::vector<bool> part;
};

struct Wg {
    State &s;
    std::function<void()> &others;     // lets other workgroups run meanwhile
    bool rebin()
    {
        others();
        const bool r = s.rebin;
        others();
        return r;
    }
    void copy(int bid, int nb)
    {
        if (bid < 0 || bid >= nb || s.part[bid] || s.finished || s.step) s.bad = true;   // a part twice, or bins gone
        else s.part[bid] = true;
        others();
        ++s.copied;
    }
    bool arrive(int nb)
    {
        others();
        const bool last = ++s.ticket == nb;
        if (last && s.copied != nb) s.bad = true;
        return last;
    }
    void finish()
    {
        others();
        ++s.finished;
    }
    void advance()
    {
        others();
        if (s.rebin && s.finished != 1) s.bad = true;
        s.rebin = false;
        ++s.step;
    }
};

template <bool ADV>
int failures(bool rebin, int nb, int draws)
{
    std::mt19937 rng(1);
    int bad = 0;
    for (int k = 0; k < draws; ++k) {
        State s{rebin};
        s.part.assign(nb, false);
        std::vector<int> left(nb);
        for (int i = 0; i < nb; ++i) left[i] = i;
        std::function<void()> others;
        auto start = [&] {
            const int j = rng() % left.size(), bid = left[j];
            left.erase(left.begin() + j);
            Wg wg{s, others};
            pic::relayout_end<ADV>(wg, bid, nb);
        };
        others = [&] {
            while (!left.empty() && rng() % 3 == 0) start();
        };
        while (!left.empty()) start();
        bad += s.bad || s.step != (ADV ? 1 : 0) || s.finished != (rebin ? 1 : 0);
    }
    return bad;
}

int main()
{
    int bad = 0;
    for (int nb : {2, 3, 5, 9})
        for (int rebin : {0, 1}) bad += failures<true>(rebin, nb, 20000) + failures<false>(rebin, nb, 20000);
    printf("%d\n", bad);
    return 0;
}
