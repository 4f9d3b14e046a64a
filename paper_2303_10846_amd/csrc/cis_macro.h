// The coloured PR-SGS sweeps of the macroscopic systems in one launch (kernels in cis_macro.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cis_internal.h"

namespace cis {

constexpr int kSweepWords = 16;   // 64-bit words per cell in the exchange buffer (12 used): a 128-byte line
constexpr int kSweepColors = 16;  // most non-empty colours

// The non-empty colours of a mesh: colour k's cells are off[k] .. off[k] + n[k] - 1, in one workgroup those of
// wavefronts wave0[k] .. wave0[k + 1] - 1 (64 / lanes-per-cell cells each).
struct SweepPlan {
  int m = 0;           // non-empty colours; 0: the mesh keeps a launch per colour
  bool local = false;  // the whole mesh in one workgroup of up to kLocalThreads threads; else in blocks
  int32_t off[kSweepColors], n[kSweepColors], wave0[kSweepColors + 1];
};
constexpr int kLocalThreads = 1024;

// The sweeps in blocks: `blocks` workgroups own equal parts of the cells in spatial order, and each relaxes in LDS
// what its cells' values of the next h steps depend on, cells of others included, so that increments are exchanged
// once in h steps.  The colours of the steps repeat after a period of 2(m - 1), of which h is a divisor or a multiple.
constexpr int kBlockWaves = 8;            // wavefronts of a workgroup, each with cells of one colour
constexpr int kWideBlockWaves = 16;       // .. of meshes whose blocks do not fit 8
constexpr int kBlockVals = 512;           // increments in LDS: of its wavefronts' slots, then of other cells read
constexpr int kBlockReads = 256;          // increments read from other workgroups per window
// Largest mesh: 3 bytes of LDS a cell while the plan is made; with 6 face slots the wavefronts end it earlier: 16 of 8
// cells, so 256 blocks of 128 own cells, 32 768, could hold no neighbours (24 389 fit)
constexpr int kBlockCells = 54000;
constexpr int kBlockSlots = 16 * kWideBlockWaves;  // cells that a workgroup relaxes (half of them with 6 face slots)
constexpr int kBlockMax = 256;            // workgroups
struct BlockRecord {
  int32_t reads, acks;                 // entries of read[] and ack[]
  int32_t color[kWideBlockWaves];      // a wavefront's colour, -1: none
  int32_t cell[kBlockVals];            // the cell of an increment, -1: none
  int16_t nb[kBlockSlots][kMaxFaces];  // increments of a slot's neighbours, -1: none
  uint8_t own[kBlockSlots];
  int16_t read[kBlockReads];           // increments that other workgroups own, and their colours
  uint8_t read_color[kBlockReads];
  int16_t ack[kBlockMax];              // the workgroups that read this one's
};
constexpr int kBlockCands = 8;  // most windows tried: the divisors of a period of up to 30
struct BlockPlan {
  int blocks = 0;    // 0: the mesh is too large or runs in one workgroup
  int h = 0;
  bool wide = false;
  BlockRecord* rec = nullptr;  // [blocks], device
  int32_t* owner = nullptr;    // [nc] block of a cell
  int32_t* most = nullptr;     // [kBlockCands] wavefronts that each window asks of the largest block
  uint32_t* link = nullptr;    // [kBlockMax][kBlockMax / 32] bit b of row a: block b reads increments of block a
};
constexpr int kBlockLink = kBlockMax * kBlockMax / 32;
// 64-bit words of the exchange buffer: [2][nc][kSweepWords], then one word per block a 64-byte line, [2][kBlockMax][8]
inline __host__ __device__ int64_t sweep_words(int64_t nc) { return 2 * (kSweepWords * nc + 8 * kBlockMax); }

// Polls of one wait before a block gives up (each at least a memory round trip, 0.5 us: 0.1 to 0.3 s).  A wait that
// long means that a workgroup is kept off the device, by a kernel of another stream or process, so the flag turns the
// rest of the call to a launch per colour, which waits for nothing.
constexpr uint32_t kSweepPolls = 1u << 18;

// Largest tag of a window: tags are compared as increasing numbers; a launch (up to 3 million steps) takes one a step.
constexpr uint32_t kSweepTagMax = 0x7fffffffu;

// State of the sweeps of one cis_state: the plans, the exchange buffer (device) and the tag of
// the last window published in it.
struct MacroSweeps {
  SweepPlan plan;
  BlockPlan block;
  bool laid_out = false;
  uint64_t* words = nullptr;
  uint32_t tag = 0;
  uint32_t polls = kSweepPolls;  // limit of a wait, but for the first polls_from launches (tests set both)
  int64_t polls_from = 0;
  int32_t redone = 0;  // calls that went on with a launch per colour after a wait ran out
  bool ready() const { return plan.m > 0 && (plan.local || laid_out); }  // the sweeps can be one launch
  bool in_blocks() const { return ready() && !plan.local; }
};

// Tag 0, that of no window, in every word of the exchange buffer (and the links of the layout, used before any tag)
void clear_sweep_words(const MacroSweeps& f, int64_t nc, hipStream_t st);

// The colours of a mesh: m = 0 where there are more than kSweepColors.
SweepPlan sweep_plan(const Dev& d, const int64_t* color_off, int64_t n_colors);

// Blocks for a mesh of nc cells on the current device (0: none, the mesh is too large or runs in one workgroup).
int block_count(const SweepPlan& pl, const Dev& d, int64_t nc);

// Before the first sweeps of a state (its other calls don't pay for it: 0.1 ms on 1 296 cells, 0.35 on 50 400): finds
// the longest window that fits and lays out f.block.rec on the stream, which it waits for.  Where none fits, or the
// device refuses a launch, the state keeps a launch per colour (plan.m = 0).
void lay_out_blocks(const Dev& d, MacroSweeps& f, hipStream_t st);

// Bit of Work::flag[0] set when a wait of the sweeps in blocks ran out.  Its results are then not valid, and from there
// on nothing in the call may write the state: a launch that finds the bit set returns at once, the update leaves G, R,
// W and q alone, and the host redoes the iteration (or the Krylov step) and the rest with a launch per colour.
constexpr int32_t kSweepStuck = 8;

// Whether the sweeps in blocks pay for n_pairs pairs in an iteration of `others` further launches.  Their launch is
// cooperative, on a hardware queue of its own: besides the 20 us around it every later launch of the stream starts
// 1.2 us later, until the host next waits (1 000 cells, 21 micro relaxations: 82 -> 109 us).  They save about 10 us and
// 2 us a relaxation (stage on 1 000 hexahedra 49 -> 31 us with 3 relaxations, 104 -> 52 with 21; on 1 296 tetrahedra
// 47 -> 32 with 5, 143 -> 60 with 41).
bool blocks_pay(const MacroSweeps& f, int n_pairs, int64_t others);

// Step 4 in one launch (spectral radii, right-hand side, n_macro forward + backward sweep pairs and the
// predicted equilibrium), after lay_out_blocks.  false: not launched, the mesh takes a launch per colour.
bool launch_macro_sweeps(const Dev& d, const Bufs& b, const Work& w, MacroSweeps& f, int n_macro, hipStream_t st);

// Mac^T u = t of the adjoint's block preconditioner, n_pairs sweep pairs from u = 0, likewise.  flag: as Work::flag.
bool launch_adj_macro_sweeps(const Dev& d, const Bufs& b, MacroSweeps& f, const double* t, double* u, int n_pairs,
                             int32_t* flag, hipStream_t st);

}  // namespace cis
