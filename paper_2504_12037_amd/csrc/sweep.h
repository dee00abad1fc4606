// Level schedule of a single-spin elimination program.
//
// The steps of an elimination tree whose messages do not depend on each
// other can run at the same time.  A step's level is one more than the
// highest level of the steps whose messages it reads (0 without inputs); a
// workgroup of the level kernels (sweep.hip) takes a tile of S samples
// through the levels in order, forward, and back for the adjoint, with one
// barrier per phase of a level instead of several per step.  Most steps of a
// sparse graph are tiny (on the 256-spin random 3-regular graph at width 10,
// 160 of the 217 steps leave a message of at most 8 entries, in 24 levels).
//
// The work of a level is cut into units, each done by one wave: the
// wave's lanes hold S samples (fastest) times E = 64 / S consecutive output
// entries, and the unit walks its entries E at a time.  The index into an
// input message follows from the output entry bit by bit, so it is a base
// (in the record), a part of the lane's bits (one word per lane for all
// inputs, from a table that steps share) and a part of the walk bits (4-bit
// positions in the record).
//
// Each wave has its own program: records of kSweepRec words in the order it
// runs them, each saying how many workgroup barriers come before it, so a
// wave loads its records ahead of time through any barrier.  Every wave of a
// program passes the same number of barriers.
//
// This header is shared by the host schedule (sweep.cpp, no HIP) and the
// kernels.
#pragma once
#include <stdint.h>

#include <vector>

#include "program.h"

namespace tnvan {

constexpr int kSweepIn = 4;      // most inputs of a step
constexpr int kSweepEdges = 4;   // most R-R edges a step consumes
constexpr int kSweepWalk = 3;    // a unit walks at most 2^kSweepWalk passes of E entries
// walk bits by mode (0 forward, 1 adjoint, 2 jets) and bytes per number: the
// passes' operands are held in registers at once
constexpr int sweep_walk(int mode, int real_size) {
  return mode != 0 ? 1 : real_size == 8 ? 2 : 3;
}
constexpr int kSweepWaves = 8;   // most waves per workgroup
constexpr int kSweepTile = 8;    // most samples per tile

// Records.  Word 0: operation (4 bits), barriers before it (8 bits), then
// the fields below; positions are 4 bits each, 15 for a bit without effect.
// Words 16 to 18 are about the next record (zeros when it is no unit): its
// transfer table offset, its w | log2 entries << 8, its lane words; so what
// it needs from memory is loaded one record ahead.
constexpr int kSweepRec = 20;
enum SweepOp : int32_t {
  SWEEP_END = 0,
  // a range of output entries of a step; SWEEP_JOINT: its joint weights
  //   0: w << 12 | inputs << 16 | dense << 19 | edges << 20 | log2 entries << 24
  //   1: arena offset of the first entry   2: the same in the transfer table
  //   3: the same in the scratch (joint weights with spin -1 lie 2^w further)
  //   4: step | position << 16             5: first partial sum
  //   6: output bit of each edge, 8 bits each   7: first entry
  //   8 + 2k: input k: arena offset at the first entry; positions of the
  //   walk bits in its index | bit of the eliminated spin << 12 | producing
  //   step << 16.  Lane word: the lane's index into input k in byte k
  SWEEP_FWD = 1,
  SWEEP_JOINT = 2,
  // rho of a range of entries of one input
  //   0: log2 lanes per sum << 12 | log2 items << 16
  //   1: scratch offset of the first item   2: positions of the walk bits
  //   3: arena offset of the first entry    4: producing step
  //   5: output bits each lane sums over.   Lane word: the lane's offset
  SWEEP_MARG = 3,
  // per-sample sums of a step over its units
  //   0: edges << 20   1: first partial sum   2: stride   3: units
  //   4: position      5..8: R-R edges
  SWEEP_SUM = 4,
  SWEEP_LOGZ = 5,   // ln Z_R from the closing entries
  SWEEP_WAIT = 6,   // barriers alone, or nothing: ahead of a first record that is no unit
};

struct SweepInst {
  int32_t prog[kSweepWaves];    // first record of each wave's program
  int32_t arena;    // entries per sample of the arena
  int32_t scr;      // adjoint scratch entries per sample
  int32_t slots;    // adjoint partial sums per sample
  int32_t n_close, close_off;   // closing steps: pairs (arena entry, step)
};

// The programs of every instance for S samples per tile and one mode.
struct SweepPlan {
  std::vector<SweepInst> insts;
  std::vector<int32_t> prog;
  std::vector<int32_t> lanes;   // lane words, E of a kind in a row
  std::vector<int32_t> close;
};

// Programs with wide steps run in segments: the steps of kWideStep bits or
// more spread over the chip, one launch per group of independent ones
// (wide.hip), and between them the light steps in level programs, one
// workgroup per sample.  A segment's light steps need only wide steps of the
// segments before; its wide steps follow in groups by their inputs.
//
// A workgroup of a wide step takes 2^kWideChunk output entries o: the chunk
// position i = thread + kWideThreads * r, whose bits stand on the output bits
// the schedule picks (the five lowest, for runs of 32 entries, then those
// that the inputs don't have, the largest input first, so that the sums over
// them stay in the workgroup).  What depends on o bit by bit (o itself, the
// index into each input) is a table of the thread's, of the r's and of the
// workgroup's part.
constexpr int kWideStep = 12;
constexpr int kWideChunk = 11;
constexpr int kWideThreads = 256;
constexpr int kWideRegs = (1 << kWideChunk) / kWideThreads;
struct WideInput {
  int32_t off, step, xbit, bits;
  int32_t idx;      // table of its index: [kWideThreads][kWideRegs][workgroups]
  int32_t free;     // chunk positions' bits not in its scope
  int32_t dep;      // table, per entry of the chunk in its scope: position | index << kWideChunk
  int32_t row;      // table [workgroups]: which partial sum it holds
  int32_t part;     // partial sums [row][entry], or -1: the workgroup has the whole sums
};
struct WideStep {
  int32_t step, gpos, w, n_in, n_edge, off;
  int32_t edge_off;
  int32_t out;      // table of o, as WideInput::idx
  int64_t t_off;    // transfer table, or -1: formed from the edges
  int32_t red;      // sums [workgroup][1 + edges] (spin, edge correlations)
  int32_t pad;
  WideInput in[kWideIn];
};
// an input's rho from its partial sums; a wide step's sums over its workgroups
struct WideFin { int32_t part, off, step, nbits, rows, first; };   // first: workgroup of the launch
struct WideSum { int32_t first, stride, n, edge; };   // edge: R-R edge, or -1 - position
struct WideGroup {
  int32_t w0, w1, blocks;      // steps and their workgroups
  int32_t f0, f1, fblocks;     // WideFin and their workgroups
};
struct WideSegment {
  int32_t fwd[kSweepWaves], bwd[kSweepWaves];   // first records of the light programs
  std::vector<WideGroup> groups;                // after the light steps
};
struct WidePlan {
  std::vector<std::vector<WideSegment>> segs;   // per instance
  std::vector<WideStep> steps;
  std::vector<WideFin> fins;
  std::vector<WideSum> sums;
  std::vector<int32_t> sum_lo;                  // per instance, and the end
  std::vector<int32_t> tab;
  std::vector<SweepInst> insts;                 // (prog unused)
  std::vector<int32_t> part, red;               // scratch words per sample
  std::vector<int32_t> prog, lanes, close;
};

struct HostProgram;
// Whether instance q can run in segments (single-spin steps within the
// limits above and those of the wide steps); and their schedule.
bool wide_fits(const HostProgram &P, int q);
void build_wide(const HostProgram &P, const std::vector<int32_t> &run, WidePlan &out);

// Whether instance q is a single-spin program with full tables within the
// limits above.
bool sweep_fits(const HostProgram &P, int q);

// run[q] != 0: schedule instance q (sweep_fits holds); others get no
// program.  bwd: forward and reverse, else forward alone.  waves: per
// workgroup, 1 to kSweepWaves.
void build_sweep(const HostProgram &P, const std::vector<int32_t> &run, int S, int waves, bool bwd,
                 int max_walk, SweepPlan &out);

}  // namespace tnvan
