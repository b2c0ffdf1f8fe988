// Work whose stages are handed out one at a time, to launches that have room for the next stage of a few pieces of it. Host code only.
#pragma once

template <typename Work, int ENTRIES, int STAGES>
struct FgStageQueue {
    struct Entry {
        Work work;
        int stage[STAGES];
        int n, next;      // stages, and those handed out

        void then(int s) { stage[n++] = s; }
    } e[ENTRIES];
    int first = 0, count = 0;

    bool empty() const { return count == 0; }
    Entry& add(const Work& work) {      // at most ENTRIES over the queue's life; the caller appends at least one stage
        Entry& y = e[first + count++];
        y.work = work;
        y.n = y.next = 0;
        return y;
    }
    // f(work, stage) for the next stage of the first `most` entries that have one left, oldest first (an entry may have fewer stages
    // than one before it has left: it is passed over until that one is done)
    template <typename F>
    void take(int most, F f) {
        int taken = 0;
        for (int i = first; i < first + count && taken < most; ++i) {
            if (e[i].next == e[i].n) continue;
            f(e[i].work, e[i].stage[e[i].next++]);
            ++taken;
        }
        while (count > 0 && e[first].next == e[first].n) ++first, --count;
    }
};
