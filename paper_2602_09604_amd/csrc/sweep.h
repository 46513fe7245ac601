// Sweeps: several consecutive matrix passes applied in one trip through
// memory.  A workgroup stages a tile of 2^T amplitudes in LDS (the L lowest
// state bits plus T - L chosen higher bits), applies every pass of the sweep
// whose targets lie in the tile to it, one after another, and writes the tile
// back.  sweep.cpp plans and encodes sweeps, k_sweep.hip runs them.
#pragma once
#include "sv_internal.h"

namespace sv {

constexpr int kSweepMaxBits = 13;  // largest tile: 2^13 amplitudes, 64 KiB of LDS
constexpr int kSweepMinBits = 8;   // one matrix-core unit of a k = 4 pass
constexpr size_t kSweepLds = 163840;  // what a workgroup may take: a CU's 160 KiB
// LDS for the matrices of a sweep of an n-qubit state: so that two workgroups
// share a CU's 160 KiB (a sweep of one larger matrix takes more and runs
// alone), or all of it where the state is a single tile and, for split
// matrices (64 KiB at k = 6), up to 20 qubits, where a CU has one tile anyway,
// and from 25, where the sweep saved is worth more than the second workgroup
// (16 FP16X3 passes with k = 6, all in pairs / a quantum volume in blocks of 6, us
// with all of the LDS and half of it: 20 qubits 122, 185 / 150, 190; 22: 322, 278 /
// 372, 355; 23: 516, 445 / 558, 536; 24: 862, 854 / 1066, 1060; 25: 1546, 1527 / 1941,
// 1991; 26: 2795, 3123 / 4328, 4420; at 21, 237, 276 / 242, 273, but there it would
// change the order of passes, and with it the rounding of a BF16X3 circuit by 2.5e-5).
inline size_t sweep_mat_room(int n, int T, int precision) {
  const bool split = precision == SV_PREC_BF16X3 || precision == SV_PREC_FP16X3;
  const bool all = T == n || (split && (n <= 20 || n >= 25));
  return (all ? kSweepLds : kSweepLds / 2) - ((size_t)8 << T);
}
constexpr int kSweepLow = 4;       // low state bits in every tile: whole 128-byte lines
constexpr int kSweepMaxK = 6;

// Kind of a K-qubit pass in the sweep's split precision.
constexpr int kSweepSplit = 8;

// One pass of a sweep on the device.  Tile bits are numbered in the order
// in-lane bits (K - 2 of them; for K = 2 both local bits), two lane bits h,
// four lane bits j, then unit bits; mask[b] is what bit b adds (by XOR) to a
// byte address in the tile: the swizzle of the tile's slots is linear over
// the bits, so any assignment of state bits to these roles is one table.
struct alignas(64) SweepOp {  // 64 bytes, no padding: graph keys compare the data
  uint32_t mask[kSweepMaxBits];
  uint32_t kind;   // 1, 2: vector ALUs; 3..6: FP32 matrix cores; kSweepSplit + 4..6: split operands
  uint32_t mat;    // byte offset of the matrix: kinds 1, 2 from the sweep's data, the others in the LDS copy
  uint32_t unused;
};

// Launch arguments of a sweep.  hi packs the state bits of the tile above its
// L low bits, ascending, six bits each: tile bit L + i is state bit
// (hi >> 6 i) & 63.
struct SweepArgs {
  uint64_t tiles = 0;
  uint64_t hi = 0;
  int32_t low = 0;      // L
  int32_t nh = 0;       // T - L
  int32_t nops = 0;
  int32_t mat16 = 0;    // LDS copy of the matrices of kinds 3 and up, in 16-byte units
  uint32_t mat_off = 0; // where they start in the data (the passes come first)
};

// A planned sweep: its tile and its passes (in order), indices into the
// caller's list.
struct Sweep {
  int T = 0;
  int low = 0;
  uint64_t bits = 0;            // state bits in the tile
  std::vector<int> members;
  int precision = SV_PREC_FP32_MFMA;  // of the k >= 4 passes
  size_t mat_bytes = 0;         // LDS bytes of the matrices
  size_t data_bytes = 0;        // device data: the passes and every matrix
};

// One sweep of one state of a batch: workgroups first .. first + groups - 1
// of the launch walk its tiles.
struct BatchSweep {
  float4* psi;
  uint64_t data;   // where its passes start in the batch's data
  SweepArgs args;
  uint32_t first;
  uint32_t groups;
  int32_t T;
};

// A pass as the planner sees it: its qubits and its kind (0: not for a sweep).
struct SweepItem {
  uint64_t mask = 0;
  int kind = 0;
};

int sweep_tile_bits(int n, int precision);
// Device kind of a k-target pass in a sweep with tiles of T bits; 0: it does not run in one.
int sweep_kind(int T, int k, int precision);
// Whether a pass (sorted targets) that shares its sweep with no other still runs
// as one; graph: its data may be on the device from an earlier call.
bool sweep_alone(int n, int k, const int* s, int precision, bool graph);
// T: tile size, at most n; mat_room: LDS bytes for the matrices of a sweep.
void plan_sweeps(const std::vector<SweepItem>& items, int n, int T, size_t mat_room, int precision,
                 std::vector<Sweep>& out);
SweepArgs sweep_args(const Sweep& sw, int n);
// Encode one sweep: targets (sorted) and matrix of every pass, in order.
void encode_sweep(const Sweep& sw, const std::vector<const Pass*>& passes, const std::vector<const double*>& mats,
                  unsigned char* dst);
void launch_sweep(const Sweep& sw, int n, void* psi, const unsigned char* data, hipStream_t st);

void launch_sweep_batch(const BatchSweep* table, int count, unsigned groups, size_t lds, bool nt,
                        const unsigned char* data, hipStream_t st);

}  // namespace sv
