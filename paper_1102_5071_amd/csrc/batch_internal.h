// Internal declarations of the batched path: many independent trajectories
// advanced together, one kernel per Lanczos phase over all of them.
//
// Instances that share their driven operators (and the dimension) form a
// group of at most 64; a group's vectors are stored interleaved, element
// (row r, instance j) at voff + r * B + j, so one wavefront lane per instance
// gathers the same column of all instances in one contiguous request and the
// shared operator row is read once for the whole group (an SpMM over the
// group).  The instances' own H0 is kept as a dense diagonal plus, if any, an
// off-diagonal CSR per instance.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cfet_internal.h"

namespace cfet {

constexpr int kBatchMaxGroup = 64;  // instances per group (one wavefront lane each)
// wavefronts per block of the row kernels: chosen at create among these
// (with the rows each lane covers); every row kernel of a batch uses the
// same block layout, since the block partials follow it
constexpr int kBatchWaveChoices[] = {2, 4, 8};
constexpr int kBatchDefaultWaves = 4;
constexpr int kBatchMaxK1 = 8;      // 1 + driven terms

// Tiles of the flip sweeps (batch.hip): elements of a packed vector.
constexpr int kFlipBits = 12;
constexpr int kFlipMaxBits = 21;    // packed elements of a group they serve
// elements of a batch from which the flip sweeps are used: one tile per CU.
// Below, they leave CUs idle and their extra launch shows (three steps of 64
// chains of 2^12 and 2^13 rows, 0.4 M elements: 2.2 ms with k_b_spmm, 2.8 with
// the sweeps; at 0.9 M, 64 of 2^11 to 2^15, 3.2 and 3.1; four of 2^18, 1.0 M, 3.4
// and 2.8)
constexpr int64_t kFlipMinElements = int64_t(1) << 20;
// ... and flips per row, on average: k_b_spmm reads a neighbour for each, the sweeps
// cost the same for all (two steps of 64 chains of 2^13 to 2^18 rows, one driven site
// 3.84 ms with k_b_spmm, 4.48 with the sweeps; six 4.57 and 4.58; eight 4.73 and 4.55)
constexpr int kFlipMinPerRow = 7;
constexpr int kFlipGather = 3;      // bits above a tile that the low sweep gathers itself

struct BGroup {
  int64_t n;            // rows
  int64_t voff;         // element offset of the group's vectors
  int B;                // instances in the group
  int lpr;              // lanes per row: smallest power of two >= B
  int rows_per_block;   // rows handled by one block of the row kernels
  int nblocks;          // blocks of the group in the row-kernel grid
  int block0;           // first block of the group in that grid
  int slot0;            // first instance slot of the group
  int shared_h0;        // 1: H0 is term 0 of the shared operator
  int pad;
  const int64_t* rowptr;  // shared operator, n + 1 row pointers
  const uint32_t* colt;   // column | term << kTermShift
  const double2* val;
  const double2* diag;    // [n][B] H0 diagonal of each instance (shared_h0 == 0)
  const int64_t* orp;     // [B][n + 1] H0 off-diagonal rows per instance, or null
  const int32_t* ocol;
  const double2* oval;
};

// What the flip sweeps read of a group besides (an array of its own: the row
// kernels load a BGroup in every block).
struct BFlip {
  int nv;               // n * B = 2^nv elements
  int sblocks, sblock0; // tiles of the low sweep (all groups) and
  int hblocks, hblock0; // of the high sweep (0: the low sweep gathers)
  int pad;
  const double* coef;   // factor of the flip of element bit v < 24
  const double* diagr;  // [n][B] real H0 diagonal
};

// Per-slot Lanczos state and statistics (slot = instance in group order).
struct BSlots {
  double* alpha;    // [slot][kMaxM]
  double* beta;     // [slot][kMaxM]
  double* inv;      // [slot][kMaxM] 1 / norm of stored basis vector l
  double2* coef;    // [slot][kMaxM] recombination coefficients
  double* beta0;    // [slot]
  int* m_eff;       // [slot]
  int* done;        // [slot] 1 once the running exponential's basis is complete
  int* mcap;        // [slot] min(m, n)
  long long* matvecs;     // [slot] cumulative
  long long* expos;       // [slot]
  long long* breakdowns;  // [slot] stopped by the breakdown rule
  long long* early;       // [slot] stopped by the error estimate
  int* min_m;             // [slot]
  int* max_m;             // [slot]
};

// Parameters read by every launch from device memory, so that a captured
// step graph stays valid across calls.
struct BState {
  const double* wts;   // [expo][slot][K1] weights in application order
  long long cursor;    // exponential index into wts (advanced on the device)
  double dt;
  double tol;
  int nslots;
  int K1;
  int status;          // latched device status: last field, never rewritten by the
                       // per-call parameter upload (cleared when reported)
};

struct BLaunch {
  const BGroup* groups;  // device array
  int ngroups;
  int total_blocks;
  int nslots;
  int64_t ntot;          // elements of one packed vector
  double2* V;            // basis: vector l at V + l * ntot (vector 0 = psi)
  double2* Y;            // H v_k
  double* part;          // [slot][pstride] partial sums: instance slot, block of its group
  int64_t pstride;
  int waves;             // wavefronts per block of the row kernels (2, 4 or 8)
  BSlots S;
  BState* st;
  const BFlip* flips;    // flip sweeps, by group (null: k_b_spmm), and
  int low_blocks;        //   blocks of the low sweep
  int high_blocks;       //   and of the high sweep
};

// (kBAlphaFlip: the partials of the low sweep's tiles)
enum BScalarMode { kBStart = 0, kBAlpha = 1, kBBeta = 2, kBAlphaFlip = 3 };

hipError_t batch_norm(const BLaunch& L, hipStream_t s);
hipError_t batch_scalars(const BLaunch& L, int mode, int k, hipStream_t s);
hipError_t batch_spmm(const BLaunch& L, int k, hipStream_t s);
hipError_t batch_axpy(const BLaunch& L, int k, hipStream_t s);
hipError_t batch_combine(const BLaunch& L, hipStream_t s);
hipError_t batch_advance(const BLaunch& L, hipStream_t s);
hipError_t batch_set_cursor(const BLaunch& L, long long v, hipStream_t s);
hipError_t batch_pack(const BLaunch& L, const double2* user, const int64_t* uoff, hipStream_t s);
hipError_t batch_unpack(const BLaunch& L, double2* user, const int64_t* uoff, hipStream_t s);
hipError_t batch_stats_reset(const BLaunch& L, hipStream_t s);

}  // namespace cfet
