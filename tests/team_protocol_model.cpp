// Walks through every interleaving of a team's exchange (verify_tree.hip) on the host, with the kernel's own tags and boxes:
// members start whenever they like, publish, look a bounded number of times, compute what did not arrive and leave; then the
// same launch runs again on the mailbox as it was left.  A member that takes a message of another step, or of an earlier run,
// for the one it waits for is what must not happen.
//   team_protocol_model <members> <steps> <polls> <runs> <bits>   bits: of the step number in the tag (8 as in the kernel)
// Prints the number of states and of wrong messages taken.
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <unordered_set>
#include <string>
#include <vector>

#include "team_protocol.h"

static int C, STEPS, POLLS, RUNS, BITS;

// What a message means, beside its tag: the model checks it, no workgroup sees it.
struct Word { uint64_t tag; uint8_t run, step; };
struct Member { uint8_t phase, step, polls, got, alone; uint8_t epoch; };       // phase: 0 not started, 1 publish, 2 look, 3 left
struct State {
    Word box[2][4][4];                                       // [box][reader][writer]
    Member m[4];
    uint8_t run, exits;
};

static uint64_t tag_of(const State &, const Member &m)
{
    return team_tag(m.epoch, 5, m.step & ((1u << BITS) - 1));
}

int main(int argc, char **argv)
{
    if (argc != 6) return 2;
    C = atoi(argv[1]); STEPS = atoi(argv[2]); POLLS = atoi(argv[3]); RUNS = atoi(argv[4]); BITS = atoi(argv[5]);
    std::unordered_set<std::string> seen;
    std::vector<State> todo;
    long wrong = 0;
    auto push = [&](const State &s) {
        if (seen.emplace((const char *)&s, sizeof s).second) todo.push_back(s);
    };
    State first;
    memset(&first, 0, sizeof first);
    push(first);
    while (!todo.empty()) {
        const State s = todo.back();
        todo.pop_back();
        bool all_left = true;
        for (int i = 0; i < C; ++i) all_left = all_left && s.m[i].phase == 3;
        if (all_left) {                                      // stream order: the next run begins when this one has ended
            if (s.run + 1 >= RUNS) continue;
            State t = s;
            t.run += 1;
            memset(t.m, 0, sizeof t.m);
            push(t);
            continue;
        }
        for (int i = 0; i < C; ++i) {
            if (s.m[i].phase == 3) continue;
            State t = s;
            Member &m = t.m[i];
            if (m.phase == 0) {
                m.epoch = t.exits;
                m.phase = 1;
            } else if (m.phase == 1) {
                for (int r = 0; r < C; ++r) {
                    Word &w = t.box[team_box(m.step)][r][i];
                    w.tag = tag_of(t, m);
                    w.run = t.run;
                    w.step = m.step;
                }
                m.phase = 2;
                m.polls = 0;
                m.got = 0;
            } else {
                // one look: every other member's word
                m.got = 0;
                for (int o = 0; o < C; ++o) {
                    if (o == i) continue;
                    const Word &w = t.box[team_box(m.step)][i][o];
                    if (!team_carries(w.tag, tag_of(t, m))) continue;
                    m.got |= 1 << o;
                    if (w.run != t.run || w.step != m.step) ++wrong;
                }
                const bool all = m.got == (((1 << C) - 1) & ~(1 << i));
                if (!all && !m.alone && m.polls < POLLS) {
                    m.polls += 1;
                } else {
                    if (!all) m.alone = 1;                   // computes the rest itself and does not wait again
                    m.step += 1;
                    m.phase = 1;
                    m.polls = m.got = 0;
                    if (m.step == STEPS) {
                        m.phase = 3;
                        m.step = 0;
                        t.exits += 1;
                    }
                }
            }
            push(t);
        }
    }
    printf("states %zu wrong %ld\n", seen.size(), wrong);
    return 0;
}
