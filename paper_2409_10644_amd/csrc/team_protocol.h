// How the workgroups that share a verification walk name their messages (see verify_tree.hip).  Plain arithmetic, so that a
// host program can step through the exchange with the same functions.
#pragma once
#include <stdint.h>

constexpr int TEAM_MAX = 16;             // workgroups per team
constexpr int TEAM_MAILBOXES = 512;      // a ring: walk w of the process uses mailbox w % TEAM_MAILBOXES

// A message says in full what it is: which walk (`nonce`, one per walk ever launched), which run of it (`epoch`, the
// mailbox's exit count when the launch began: a replay of a captured launch has the nonce of the first run), which step.
// Nothing may be left to the order in which workgroups get on: one that has given up waiting runs ahead of the others by any
// number of steps and goes on publishing.  A walk has at most one step per node of a path's contexts and one for the
// distribution it ends in; the largest tree (level sizes of at most MCSD_MAX_BRANCH children, MCSD_MAX_NODES nodes,
// MCSD_MAX_LEVELS levels) has 157, so eight bits number the steps, from 1 on: no tag is all zeros, what a mailbox holds at first.
constexpr int TEAM_STEP_BITS = 8, TEAM_NONCE_BITS = 17, TEAM_PIECE_BITS = 16;      // and the epoch in the 23 bits above

// The words of a step's message carry this tag and 16 bits of the sum each.
constexpr uint64_t team_tag(unsigned epoch, uint64_t nonce, unsigned step)
{
    return (((uint64_t)epoch << TEAM_NONCE_BITS | (nonce / TEAM_MAILBOXES & ((1ull << TEAM_NONCE_BITS) - 1))) << TEAM_STEP_BITS |
            ((step + 1) & ((1u << TEAM_STEP_BITS) - 1))) << TEAM_PIECE_BITS;
}
constexpr bool team_carries(uint64_t word, uint64_t tag) { return (word ^ tag) >> TEAM_PIECE_BITS == 0; }

// Two boxes in turn: a workgroup that waits for everyone's step s + 1 before it writes step s + 2 overwrites nothing that is
// still wanted; one that does not wait may, and then the reader finds another tag and computes the sum itself.
constexpr unsigned team_box(unsigned step) { return step & 1; }
