// seq_types.h - the sequence engine: one component's search by many
// wavefronts, with the sequential search's result to the last node.
//
// A component's search is kept as a list of tasks in search order.  A task is
// a piece of the sequential search's stack: the state at its top and some of
// the untried rows below it.  Its wave searches on from there for at most
// `cap` nodes.  If that does not exhaust the piece, the stack that is left is
// cut into pieces again - the deepest few untried levels together, then one
// level each, then the rest - which take the task's place in the list, right
// after the nodes it has counted.  So the list always reads in the
// sequential order: node counts (and trace hashes) of finished tasks add up
// from the front, and a component is done when the front meets a solution
// (FEASIBLE), the end of the list (INFEASIBLE), or the task in which the
// budget runs out, which is searched once more with what is left of it for
// the depth at the stop.  Each round runs the first tasks of every list, as
// many as the device takes at once: the ones that the sequential search
// would reach next.
#pragma once

#include <cstdint>

#include "device_types.h"

namespace mpld {

// One run list per kernel: the register tier's, and the CSR tiers' (both
// one-wave layouts in one kernel, so that a round is one launch).
enum SeqTier : int32_t { kSeqReg = 0, kSeqCsr = 1, kSeqTiers = 2 };
enum SeqKind : int32_t {
  kSeqRoot = 0,   // the component from its root
  kSeqNode = 1,   // on from the saved state, at a node
  kSeqNext = 2    // from the saved state's deepest untried row
};
// SeqResult.status besides the search's own
constexpr int32_t kSeqCapped = -1, kSeqWaiting = -2, kSeqLost = -3;

// Run-list entries: the task, and what becomes of it at its cap.  Tasks at
// the front of their list are cut, the ones behind saved whole, so that
// memory goes where the sequential search is; where there is no room for that
// either, the first task goes on to its end and the others wait.
constexpr int32_t kSeqTaskMask = (1 << 28) - 1, kSeqCut = 1 << 28, kSeqForce = 1 << 29;

constexpr int32_t kSeqPieces = 24;        // most pieces of one cut
constexpr int32_t kSeqFirstLevels = 1;    // untried levels of the deepest piece

struct SeqTask {
  int32_t comp, kind;
  uint32_t dbase;      // CSR tiers: depth below the piece's stack
  uint32_t levels;     // CSR tiers: its levels ...
  uint32_t nent;       // ... and undo-log entries
  uint32_t row_in;     // CSR tiers, kSeqNode: the row that led to the node
  int64_t at;          // arena: register tier: the saved state; CSR tiers: planes, headers, log
  int64_t col;         // arena, CSR tiers: colors of the nodes covered below the piece, -1 none
  uint64_t open;       // register tier: the piece's untried levels
};
static_assert(sizeof(SeqTask) == 48, "task is 48 bytes");
struct SeqResult {
  int32_t status;      // search status, kSeqCapped, kSeqWaiting or kSeqLost (no memory for it)
  int32_t depth;
  uint64_t nodes, hash;
  int64_t sol;         // arena: colors of a solution
  int32_t child, nchild;
};
static_assert(sizeof(SeqResult) == 40, "result is 40 bytes");
struct SeqComp {
  int32_t pos;         // launch position (register tier: item)
  int32_t tier, running, count;   // count: tasks in the list
  uint64_t acc, hash;  // nodes (and their trace hash) before the list
  // once done
  int32_t status, depth;
  int64_t sol;
  int32_t cross;       // the task in which the budget runs out, -1 none
  int32_t wide;        // CSR tiers: the wide layout
  uint64_t left;       // what it has left of it
};
static_assert(sizeof(SeqComp) == 64, "component is 64 bytes");
struct SeqHead {
  unsigned long long arena;                // bytes taken
  int32_t tasks;                           // tasks taken
  int32_t lost;                            // components given up
  int32_t active[kSeqTiers], next[kSeqTiers];   // components still searched: of the last round, of this
  int32_t share[kSeqTiers];                // first tasks of a list that run in a round
  int32_t run[2][kSeqTiers];               // lengths of the run lists
  int32_t pop[2][kSeqTiers];               // entries taken beyond each workgroup's first
  int32_t ticket, rounds;
};
struct SeqArgs {
  SeqHead* head;
  SeqComp* comps;
  SeqTask* tasks;
  SeqResult* results;
  int32_t* lists;      // [2][ncomps][list_cap]
  int32_t* runs;       // [2][kSeqTiers][run_cap]
  uint8_t* arena;
  int64_t arena_cap;
  int32_t ncomps, task_cap, list_cap, run_cap;
  int32_t slots[kSeqTiers];   // tasks that the device takes at once
  int32_t cap[kSeqTiers];     // nodes a task may count
  int32_t least[kSeqTiers];   // least share
  int32_t trace;
};

// Bytes of a saved register-tier state of K planes (reg_save's layout).
constexpr int64_t seq_reg_state_bytes(int32_t k, bool stitch) {
  return stitch ? (int64_t)kRegStateBytes : 128 + 64 * 4 * (3 + 2 * (int64_t)k);
}

}  // namespace mpld
