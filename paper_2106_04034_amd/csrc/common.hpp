// Internal structures shared by the HIP kernels and the host runtime of
// libgsgp.so.  Nothing here is part of the public ABI (include/gsgp.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gsgp.h"

namespace gsgp {

// Canonical case chunk: fitness partial sums are formed over these runs of
// consecutive cases of one segment (train or test), in a fixed order, and
// combined in FP64 in chunk order.  Launch shapes never change the chunking,
// so fitness bits (and therefore selection) do not depend on tuning.  A
// chunk is 2 KiB of one semantic row (512 FP32 or 256 FP64 cases): each
// offspring task then reads and writes 2 KiB contiguous per row, which keeps
// HBM efficient under the random row order of the operators, and one chunk
// column of a large population (its distinct parent and pool rows) stays
// closer to an XCD's L2 (2 KiB against 4 KiB chunks: 1-2 % less time per
// generation on 256-, 1,024- and 2,048-row populations).
constexpr int kChunkBytes = 2048;
constexpr int chunk_cases(int storage_bytes) { return kChunkBytes / storage_bytes; }
// Each segment (train, test) of a semantic row is padded with zeros to a
// multiple of this many cases; rows therefore start 256-byte aligned.
constexpr int kSegPad = 64;
constexpr int kWave = 64;
// Threads of one launch in a dimension: HIP takes fewer than 2^32.  Launches that
// could have more go in pieces of at most this many.
constexpr int64_t kMaxThreads = (int64_t)1 << 31;
// Interpreter work unit: a block of kInterpCases cases (kWave lanes x 2 cases).
constexpr int kInterpCases = 128;
// X is stored in tiles of kXTile cases, each tile feature-major: element
// (case c, feature f) at ((c / kXTile) * l + f) * kXTile + c % kXTile.  One
// tile's features (l x 2 KiB) are contiguous, so the rows an interpreter
// block reads spread over every L2 channel and few pages, where a
// feature-major [l][ld] layout put them ld x 8 bytes apart.
constexpr int kXTile = 256;
__host__ __device__ constexpr int64_t x_index(int64_t c, int64_t f, int64_t l) {
  return ((c / kXTile) * l + f) * kXTile + c % kXTile;
}
constexpr int kMaxTournament = 64;
// The interpreter of the deep programs keeps the top two stack values in
// registers and the rest (depth - 2 values per lane) in a lane-strided column:
// in LDS up to this many values (63 x 2 cases x 64 lanes x 8 B = 63 KiB, one
// wave per block),
// beyond it in a global-memory region of the workspace that a spill pass of
// kSpillWaves waves shares, one column per wave.
constexpr int kMaxLdsSlots = 63;
constexpr int kSpillWaves = 128;
// Stack values below the top two that a genome of k genes can need: its
// deepest stack up to its last valid function is at most k - 1 values.
constexpr int64_t max_need(int64_t k) { return k > 3 ? k - 3 : 0; }
// The compile step files each run's programs into kLists lists by stack need
// (values below the top two), so that a CU keeps as many waves resident as the
// programs' LDS columns allow: list b < kLists - 1 holds the programs whose
// need lies in (kListSlots[b - 1], kListSlots[b]] (list 0: need <=
// kListSlots[0]).  Those lists' interpreter keeps one value more in registers:
// list 0 needs no LDS (82 % of random programs of 127 genes, 22 % of 1,023),
// the others 2, 4 and 8 KiB a wave.  The last list holds every deeper program
// (two-cases-per-lane passes with columns up to kMaxLdsSlots, then the spill
// pass): 0.3 % at 127 genes, 1.3 % at 2,047.
constexpr int kLists = 5;
constexpr int kListSlots[kLists - 1] = {1, 2, 3, 5};
__host__ __device__ constexpr int list_of(int need) {
  return need <= 1 ? 0 : need == 2 ? 1 : need == 3 ? 2 : need <= 5 ? 3 : 4;
}
static_assert(list_of(kListSlots[0]) == 0 && list_of(kListSlots[1]) == 1 && list_of(kListSlots[2]) == 2 &&
                  list_of(kListSlots[3]) == 3 && list_of(kListSlots[3] + 1) == kLists - 1,
              "list_of must follow kListSlots");
// A compiled op.  `word`:
//   bits 0..1   the function (OpFn), or for a push which terminal (OpPush);
//   bits 2..3   the class (OpClass);
//   bits 4..15  stack depth before the op (values, top included);
//   bits 16..31 feature index.
// A push directly followed by a function it feeds is compiled into one op
// (kClsFeature / kClsConst) that applies the function to the top of the
// stack and the terminal, leaving the rest of the stack untouched.  `value`
// holds the constant of a constant op and, for an op that uses a feature, the
// bits of the byte offset, in a tile of X, of the row that the next such op
// uses (0 for the last one).  A program's first entry is no op: its `value` is
// the first such row.  The op after a program's last one is an end word (push
// class, bit 1 set).  `code` is the byte offset of the op's handler in
// eval_program_threaded's table.
struct CompiledOp {
  int32_t code, word;
  double value;
};
static_assert(sizeof(CompiledOp) == 16, "four ops a 64-byte line");
// The interpreters read a program's ops eight at a time, up to two batches
// ahead: programs start on a multiple of four ops (op_stride), and kOpTail
// entries follow the last program.
constexpr int kOpPad = 8;
constexpr int kOpTail = 3 * kOpPad;
// the header, at most k - 1 ops and the end word
__host__ __device__ constexpr int64_t op_stride(int64_t k) { return (k + 1 + 3) / 4 * 4; }

enum OpClass : int32_t { kClsPush = 0, kClsStack = 1, kClsFeature = 2, kClsConst = 3 };
enum OpFn : int32_t { kFnAdd = 0, kFnSub = 1, kFnMul = 2, kFnDiv = 3 };
enum OpPush : int32_t { kPushFeature = 0, kPushConst = 1 };
constexpr int kOpDepthMax = 0xFFF;

// After the state words of all runs: programs that each launch of the wide
// interpreter has given up so far, a cache line of words for every XCD.
constexpr int kWideLaunches = 2;
constexpr int kGivenUpStride = 32;
constexpr int kGivenUpWords = 8 * kGivenUpStride;  // a launch

// Per-run device state words.
enum StateWord : int {
  kStGen = 0,           // last completed generation
  kStDone = 1,          // arrival counter of the survival kernel's blocks
  kStReplaySelect = 2,  // 1: variation draws are supplied, do not draw
  kStReplayElite = 3,   // 1: survival decisions are supplied
  kStMaxDepth = 4,      // deepest stack of the compiled genomes
  kStNonFinite = 5,     // set when X or y holds NaN / Inf
  kStList0 = 6,         // kLists words: the number of programs in each stack-need list
  kStXBig = 11,         // set when X holds a value beyond 2^128 in magnitude
  kStWords = 12
};

// Best and worst train fitness of kFitGroup consecutive individuals (lowest
// index on ties): the fitness kernel leaves one per group for survival.
constexpr int kFitGroup = 16;
struct Extremes {
  double min, max;
  int32_t min_i, max_i;
};

// The loop without selection (tournament_size 0, no local search) runs up to
// kBlockGens generations at a time (see k_mutate_block).  A copy of the best
// parent over the worst offspring makes that individual leave its own line:
// its values are then those of generation-0-of-the-block individual `root`,
// taken through the recorded mutations of individual by[s] at step s (-1: the
// copy itself, nothing applied).
constexpr int kBlockGens = 15;
struct BlockState {
  int32_t base;                  // generation the block started from
  int32_t n;                     // individuals that have left their line
  int32_t dst;                   // the one the last step's copy overwrote, -1: no copy
  int32_t who[kBlockGens];       // [n]
  int32_t root[kBlockGens];
  int32_t by[kBlockGens][kBlockGens + 1];
};

// Everything a kernel needs to know about one run; lives in the workspace.
struct RunDev {
  void* S[2];               // population semantics ping-pong, [m][ld], storage type
  void* sigR;               // squashed pool semantics, [r][ld]
  void* y;                  // target, [ld], storage type, zero pads
  double* X;                // features in case tiles, [ceil(ld / kXTile)][l][kXTile], pads repeat a case (see k_prep)
  double* part;             // chunk partial sums of squared residuals, [nch][m]; with local
                            // search the generation's sums of o, o^2 and o * t, [nch][3][m];
                            // for blocks of generations [generations a block][nch][m]
  double* F[2];             // train RMSE ping-pong, [m]
  double* Ft[2];            // test RMSE ping-pong, [m]
  Extremes* extremes;       // of the newest fitness, [ceil(m / kFitGroup)]
  double* block_F;          // blocks of generations: train, then test RMSE of steps 1 .. kBlockGens - 1, [2][kBlockGens - 1][m]
  BlockState* block;        // blocks of generations, else NULL
  gsgp_record* rec;         // variation draws, [gmax][m]; generation g at g - 1
  gsgp_gen_stats* stats;    // [gmax + 1]
  gsgp_gen_stats* elite_in; // supplied survival decisions, [gmax]
  int32_t* code;            // genomes, [m + r][k]
  double* cval;             // [m + r][k]
  CompiledOp* ops;          // compiled genomes, [m + r][op_stride(k)] + kOpTail
  int32_t* nops;            // [m + r]
  int32_t* need;            // LDS stack values per lane each program needs, [m + r]
  int32_t* lists;           // programs list by list, [m + r] (counts in kStList0 ..)
  int32_t* state;           // [kStWords]
  double* ls;               // local search: (alpha, beta) of every individual, [gmax + 1][m][2]
  double* tsum;             // local search: sum t and sum t^2 over train, then over test cases
  int64_t n_train, n_test;  // real cases
  int64_t tr_pad, te_pad;   // padded segment lengths
  int64_t ld;               // row stride (tr_pad + te_pad)
  int32_t l;                // features
  int32_t nch_tr, nch_te, nch;  // chunks per segment and in total
  uint32_t run_id;
  int32_t surv_blk0, surv_blks; // survival kernel blocks of this run
  int32_t x_big;            // X holds a value beyond 2^128 in magnitude (no short division by features)
  int32_t row_blk0;         // first block of this run in the row kernel of a block of generations
  int64_t vary_task0;       // first task of this run in the variation launch
  int64_t cblk0;            // first 128-case block of this run (interpreter)
  int64_t cblk0w;           // first 256-case block of this run (wide interpreter)
  int64_t col0;             // first column of this run's X tiles over all runs (data prep)
};

// Run-independent parameters, passed by value to every kernel.
struct Params {
  int32_t m, r, k, gmax;
  int32_t tsize, ms_random;
  int32_t n_runs, precision;
  int32_t ls, pad1;                // ls: least-squares scaling of every variation offspring
  uint64_t t_xo, t_func, t_feat;  // event thresholds floor(p * 2^32)
  double ms, erc_lo, erc_hi;
  uint32_t seed;
  int32_t pad;
};

// Chunk-tiled layout of every semantic buffer (population, pool): the
// padded columns of a run are cut into chunks (train segment first, then
// test), and each chunk stores the slices of all rows one after another.
// Element (row i, column col) of a buffer with `rows` rows lives at
//   rows * cs + i * len + (col - cs)
// where cs and len are the first column and the length of col's chunk.  One
// chunk's parents, pool trees and offspring thus sit in three contiguous
// blocks, which keeps address translation and DRAM pages local while the
// operators pick rows at random.
struct ChunkGeom {
  int64_t cs;   // first padded column of the chunk
  int64_t len;  // columns in the chunk (a multiple of kSegPad)
};

__host__ __device__ inline ChunkGeom chunk_geom(int64_t tr_pad, int64_t te_pad, int32_t nch_tr, int32_t c,
                                                int64_t chunk) {
  ChunkGeom g;
  if (c < nch_tr) {
    g.cs = (int64_t)c * chunk;
    g.len = tr_pad - g.cs;
  } else {
    const int64_t k = (int64_t)(c - nch_tr) * chunk;
    g.cs = tr_pad + k;
    g.len = te_pad - k;
  }
  if (g.len > chunk) g.len = chunk;
  return g;
}

// Index of (row i, padded column col) in a chunk-tiled buffer of `rows` rows.
__host__ __device__ inline int64_t tiled_index(int64_t tr_pad, int64_t te_pad, int32_t nch_tr, int64_t chunk,
                                               int64_t rows, int64_t i, int64_t col) {
  const int32_t c = col < tr_pad ? (int32_t)(col / chunk) : nch_tr + (int32_t)((col - tr_pad) / chunk);
  const ChunkGeom g = chunk_geom(tr_pad, te_pad, nch_tr, c, chunk);
  return rows * g.cs + i * g.len + (col - g.cs);
}

// Launch shape of the variation kernel.
struct VaryLaunch {
  int32_t waves;         // waves per block
  int32_t opb;           // offspring per block task
  int32_t ogroups;       // ceil(m / opb)
  int32_t remap;         // 1: XCD-aware block order
  int64_t total_tasks;   // sum over runs of nch * ogroups
  int64_t grid;          // blocks launched
};

enum SurviveMode : int32_t { kSurvInit = 0, kSurvGen = 1, kSurvSelectOnly = 2 };

// Host-side launchers (kernels.hip).  All enqueue on `s` and return the
// launch status.
hipError_t launch_prep(const RunDev* d_runs, const Params& p, int64_t total_cols,
                       const double* const* Xsrc, const double* const* ysrc, hipStream_t s);
hipError_t launch_set_state(const RunDev* d_runs, int32_t n_runs, int32_t word, int32_t value,
                            hipStream_t s);
hipError_t launch_reset_state(const RunDev* d_runs, int32_t n_runs, int32_t* given_up, hipStream_t s);
hipError_t launch_genome(const RunDev* d_runs, const Params& p, hipStream_t s);
hipError_t launch_compile(const RunDev* d_runs, const Params& p, hipStream_t s);
// Interpreter passes.  launch_interpret_wide: the programs of the stack-need
// lists first .. last (< kLists - 1; at most `progs` per run together), four
// cases per lane, case_blocks blocks of kXTile cases over all runs; a wave takes
// per_wave (<= 32) programs one after the other on its block.  given_up:
// kGivenUpWords of the launch's own, zero before it.
// launch_interpret: the last list's programs with a need of at most `slots`
// (<= kMaxLdsSlots), two cases per lane, blocks of kInterpCases cases.
hipError_t launch_interpret_wide(const RunDev* d_runs, const Params& p, int64_t case_blocks, int first, int last,
                                 int64_t progs, int32_t per_wave, int32_t* given_up, hipStream_t s);
hipError_t launch_interpret(const RunDev* d_runs, const Params& p, int64_t case_blocks, int slots, int32_t progs,
                            hipStream_t s);
// Last pass: every program of the last list whose need exceeds kMaxLdsSlots,
// with its stack in `spill` (kSpillWaves columns of slots x 2 x 64 doubles).
hipError_t launch_interpret_spill(const RunDev* d_runs, const Params& p, double* spill, int slots,
                                  hipStream_t s);
hipError_t launch_vary(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, bool rows_only,
                       hipStream_t s);
hipError_t launch_fitness(const RunDev* d_runs, const Params& p, bool init, hipStream_t s);
// `gens` (odd, at most kBlockGens) generations of the loop without selection.
hipError_t launch_block(const RunDev* d_runs, const Params& p, const VaryLaunch& lc, int32_t gens,
                        int32_t row_blocks, hipStream_t s);
// Local search: sums of the stored target over each run's train and test cases.
hipError_t launch_target_sums(const RunDev* d_runs, const Params& p, hipStream_t s);
hipError_t launch_survive(const RunDev* d_runs, const Params& p, int32_t total_blocks, int mode,
                          hipStream_t s);
// Read-back into contiguous arrays (device memory or mapped host memory).
hipError_t launch_fetch_semantics(int32_t precision, const RunDev& R, const void* buf, int64_t rows, int64_t row0,
                                  int64_t case0, int64_t n_cases, int64_t e0, int64_t count, const double* ls,
                                  double* out, hipStream_t s);
hipError_t launch_fetch_stats(const RunDev* d_runs, int32_t run0, int32_t gen0, int32_t n, int64_t e0, int64_t count,
                              gsgp_gen_stats* out, hipStream_t s);
hipError_t launch_fetch_pair(const double* a, const double* b, int32_t n, double* out, hipStream_t s);
// Reconstruction helpers.
hipError_t launch_transpose(const double* X, int64_t n, int32_t l, double* Xfm, int64_t ld,
                            hipStream_t s);
// The n0 generation-0 trees tree0[] to out0 and the np pool trees pool[],
// squashed, to outp ([program][ld]).
hipError_t launch_interpret_list(const CompiledOp* ops, const int32_t* nops, int32_t k, int32_t m,
                                 const int32_t* tree0, int32_t n0, const int32_t* pool, int32_t np, const double* Xfm,
                                 int64_t ld, int64_t n, double* out0, double* outp, int slots, double* spill,
                                 hipStream_t s);
struct alignas(16) ReplayNode {
  int32_t op;     // 0 mutation, 1 crossover, 2 copy
  int32_t a, b;   // source slots (previous generation); b is 0 unless crossover
  int32_t r1, r2; // pool slots, 0 where the operation reads none
  int32_t out;    // destination slot
  double ms;
  double alpha, beta;  // local search: the offspring is alpha + beta * (operator output)
};
// The part of an ancestry that one individual depends on, walked on the device
// (see k_lineage): lineage_lds bytes of LDS must not exceed kReplayLdsBytes,
// and the population not kLineagePop.  `slots`, lineage_slots int32 or null, is
// what the nodes are made from: those of generation g go to begin[gen - g] ..
// begin[gen - g + 1] - 1.
struct LineageSummary {
  int32_t max_slots, n0, np, total_nodes;
};
constexpr int32_t kLineagePop = 8192;
constexpr int64_t lineage_lds(int64_t m, int64_t r) { return 4 * (2 * m + r); }
constexpr int64_t lineage_slots(int64_t m, int64_t r, int64_t gen) { return (gen + 1) * m + r; }
hipError_t launch_lineage(const RunDev& R, const Params& p, int32_t gen, int32_t individual, int32_t* begin,
                          int32_t* tree0, int32_t* pool, int32_t* slots, LineageSummary* out, hipStream_t s);
hipError_t launch_lineage_nodes(const RunDev& R, const Params& p, int32_t gen, const int32_t* begin,
                                const int32_t* slots, ReplayNode* nodes, hipStream_t s);
// A whole lineage of `gen` generations in one launch: nodes of generation g at
// begin[gen - g] .. begin[gen - g + 1] - 1 (device array of gen + 1), at most
// `slots` rows a generation; replay_cases(slots, n) must not be 0.
constexpr int64_t kReplayLdsBytes = 128 << 10;
int replay_cases(int64_t slots, int64_t n);
hipError_t launch_replay_lineage(const ReplayNode* nodes, const int32_t* begin, int32_t gen, int32_t n0, int32_t np,
                                 int32_t slots, int32_t out_slot, const double* first,
                                 const double* pool, int64_t ld, int64_t n, double* out, hipStream_t s);
hipError_t launch_replay_nodes(const ReplayNode* nodes, int32_t nnodes, const double* prev,
                               const double* pool, double* next, int64_t ld, int64_t n,
                               hipStream_t s);

}  // namespace gsgp
