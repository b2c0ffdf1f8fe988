// Drives FgStageQueue over every order of up to four pieces of work of 1 to 4 stages, with 0 to 3 launches behind each that is added:
// every stage is handed out once and in order, by at most one launch each, at most `most` to a launch, and the queue ends empty.
#include <cstdio>
#include <cstring>

#include "stage_queue.h"

namespace {
constexpr int PIECES = 4, MOST = 2;

bool check(const int* stages, const int* launches, int pieces) {
    FgStageQueue<int, PIECES, 4> q;
    memset((void*)&q.e, 0x55, sizeof(q.e));
    int given[PIECES] = {0}, total = 0, handed = 0;
    bool fine = true;
    auto launch = [&] {
        int here = 0, seen = 0;
        q.take(MOST, [&](int work, int stage) {
            const bool known = work >= 0 && work < pieces;
            fine = fine && known && given[work] < stages[work] && stage == 10 * work + given[work] && !(seen >> work & 1);
            if (known) {
                ++given[work];
                seen |= 1 << work;
            }
            ++here;
        });
        handed += here;
        fine = fine && here <= MOST;
        return here;
    };
    for (int i = 0; i < pieces; ++i) {
        auto& e = q.add(i);
        for (int s = 0; s < stages[i]; ++s) e.then(10 * i + s);
        total += stages[i];
        for (int k = 0; k < launches[i] && fine; ++k) launch();
    }
    for (int k = 0; fine && !q.empty(); ++k) fine = k < total && launch() > 0;
    return fine && handed == total;
}
}  // namespace

int main() {
    int cases = 0, wrong = 0;
    for (int pieces = 1; pieces <= PIECES; ++pieces)
        for (int code = 0; code < 1 << 4 * pieces; ++code) {
            int stages[PIECES], launches[PIECES];
            for (int i = 0; i < pieces; ++i) {
                stages[i] = 1 + (code >> 4 * i & 3);
                launches[i] = code >> (4 * i + 2) & 3;
            }
            ++cases;
            if (check(stages, launches, pieces)) continue;
            if (wrong++ < 5) {
                printf("wrong:");
                for (int i = 0; i < pieces; ++i) printf(" %d stages, %d launches;", stages[i], launches[i]);
                printf("\n");
            }
        }
    printf("%d of %d orders wrong\n", wrong, cases);
    return wrong != 0;
}
