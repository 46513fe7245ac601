// Host side of the tile sweeps (see sweep.h): which passes share a sweep, and
// the device data of one.
#include "sweep.h"

#include <algorithm>
#include <cstring>
#include <stdexcept>

namespace sv {

namespace {
bool split_precision(int precision) { return precision == SV_PREC_BF16X3 || precision == SV_PREC_FP16X3; }
// Device kind of a k-target pass: 1 and 2 on the vector ALUs, the others on
// the matrix cores (k = 3 always in FP32).
int op_kind(int k, int precision) { return k >= 4 && split_precision(precision) ? kSweepSplit + k : k; }
int kind_bits(int kind) { return kind > kSweepSplit ? kind - kSweepSplit : kind; }
size_t op_mat_bytes(int kind) {  // complex64, or the real 2^(K+1) square matrix in two halves
  return (size_t)(kind > kSweepSplit ? 16 : 8) << (2 * kind_bits(kind));
}
size_t lds_mat_bytes(int kind) { return kind > 2 ? op_mat_bytes(kind) : 0; }

// What a matrix counts for when the sweeps of a circuit are planned.  BF16X3: a k
// = 3 one as a k = 4 one, so that the same passes share a sweep as when it was
// padded to that; another order of passes moves a BF16X3 result by as much as its
// error (2 to 3e-5 after a few dozen passes).
size_t planned_mat_bytes(int kind, int precision) {
  return lds_mat_bytes(kind == 3 && precision == SV_PREC_BF16X3 ? 4 : kind);
}

// byte-address mask of tile bit b (the swizzle of k_sweep.hip on one bit)
uint32_t bit_mask(int b) {
  if (b == 0) return 8;
  const int e = 1 << (b - 1);
  return (uint32_t)((e ^ (((e >> 4) ^ (e >> 8)) & 15)) * 16);
}
}  // namespace

// Tile size of an n-qubit state.  FP32: 2^12 amplitudes while a workgroup has at
// most two tiles, 2^13 above, where fewer sweeps count for more (grid at greedy
// k = 4 / grid unfused / quantum volume in blocks of 5, us with 2^12 and 2^13: 20
// qubits 225, 293 / 396, 538 / 136, 202; 21: 377, 369 / 566, 662 / 220, 263; 22: 444,
// 426 / 1002, 866 / 357, 367; 23: 491, 445 / 1694, 1480 / 612, 569; 25: 3500, 3255 /
// 8429, 7197 / 2195, 2008).
int sweep_tile_bits(int n, int precision) {
  if (split_precision(precision)) return std::min(n, 12);  // room for two 64 KiB matrices
  return n <= 21 ? std::min(n, 12) : 13;
}

// The FP32 passes of every size (the split precisions keep their own kernels
// for k >= 4), as long as the tile holds one unit of 16 groups.
int sweep_kind(int T, int k, int precision) {
  if (std::max(k, 4) + 4 > T) return 0;
  return op_kind(k, precision);
}

// From k = 5; at k = 4 the pass kernels are as fast.
// FP32_VALU: the register kernel is bound by its ALUs there (5 qubits, 12 to 20
// qubits of state: 60-72 us, here 12-15; 24: 104, 65; 26: 241-414, 197-271; 6
// qubits, 24 qubits of state: 214-366, 118-132).  At k = 5 its 3M form streams
// as fast in the end: with bit 0 and no target in bits 1..3, where its
// elements are halves of groups, from 28 qubits (760-822 us against 875-1086;
// 30 qubits: 3.1-3.4 ms against 4.5-4.9, since a tile with few long rows far
// apart reads memory more slowly), and for any targets from 32 (12.4-16.0 ms
// against 11.8-16.9, 0.6 % apart on average; at 30 the sweep is 8 % faster).
// FP32_MFMA: the pass of k_mfma.hip from 21 qubits (22 qubits: 23-28 us against 28
// at k = 5, 35-41 against 46 at k = 6; 6 qubits, 28 qubits of state: 1.30-1.59 ms
// against 1.50, 32: 17.9-20.9 against 23.5), except 5-qubit passes on bit 0 and
// bits 1..3 of a streamed state, where it exchanges lanes (26 and 28 qubits:
// 0.68-0.96 of its time here), and except 6-qubit passes below 24 qubits that
// are encoded for the call: a call of them is bound by the host, which writes
// 64 KiB for a pass there and 32 here (21 / 22 / 23 qubits of quantum volume at
// depth 10: 1.69 / 1.83 / 2.02 ms a call there, 1.44 / 1.60 / 1.81 here; as a kept
// graph 0.57 against 0.81 at 22).
// Split precisions: up to 20 qubits (6 qubits: 18.4-23.8 us there, 14.5-17.7 here;
// 5 qubits 10.4-14.6, 11.0-14.7); above, k_mfma.hip's passes stream better (28
// qubits 711 against 892 us).
bool sweep_alone(int n, int k, const int* s, int precision, bool graph) {
  if (k < 5) return false;
  if (split_precision(precision)) return n <= 20;
  const bool low = s[0] == 0 && s[1] <= 3;  // bit 0 and one of bits 1..3
  if (precision == SV_PREC_FP32_MFMA && n > 20) return k == 5 ? low && n >= 26 : n < 24 && !graph;
  return k >= 6 || (n < 32 && (n < 28 || s[0] != 0 || low));
}

// Greedy in passes: a sweep is seeded with the first pass left and takes
// every later eligible pass whose targets still fit in the tile and which
// shares no qubit with a pass skipped before it (so it commutes with all of
// those).  A pass that is not eligible is a sweep of its own (T = 0) and keeps
// its place in the order.
void plan_sweeps(const std::vector<SweepItem>& items, int n, int T, size_t mat_room, int precision,
                 std::vector<Sweep>& out) {
  out.clear();
  const int low = T == n ? T : kSweepLow;
  const uint64_t low_mask = ((uint64_t)1 << low) - 1;
  std::vector<char> used(items.size(), 0);
  for (size_t s = 0; s < items.size(); ++s) {
    if (used[s]) continue;
    Sweep sw;
    sw.members.push_back((int)s);
    used[s] = 1;
    if (items[s].kind) {
      sw.T = T;
      if (split_precision(precision)) sw.precision = precision;
      sw.low = low;
      sw.bits = low_mask | items[s].mask;
      size_t mat = lds_mat_bytes(items[s].kind), planned = planned_mat_bytes(items[s].kind, precision);
      sw.data_bytes = sizeof(SweepOp) + op_mat_bytes(items[s].kind);
      uint64_t blocked = 0;
      for (size_t h = s + 1; h < items.size(); ++h) {
        if (used[h]) continue;
        const uint64_t m = items[h].mask;
        const size_t mb = planned_mat_bytes(items[h].kind, precision);
        if (items[h].kind && (m & blocked) == 0 && __builtin_popcountll(sw.bits | m) <= T &&
            planned + mb <= mat_room) {
          sw.bits |= m;
          planned += mb;
          mat += lds_mat_bytes(items[h].kind);
          sw.data_bytes += sizeof(SweepOp) + op_mat_bytes(items[h].kind);
          sw.members.push_back((int)h);
          used[h] = 1;
        } else {
          blocked |= m;
          if ((sw.bits & ~blocked) == 0 && __builtin_popcountll(sw.bits) == T) break;  // nothing more can join
        }
      }
      sw.mat_bytes = mat;
      // fill the tile with the lowest bits left
      for (int b = low; b < n && __builtin_popcountll(sw.bits) < T; ++b) sw.bits |= (uint64_t)1 << b;
    }
    out.push_back(std::move(sw));
  }
}

SweepArgs sweep_args(const Sweep& sw, int n) {
  SweepArgs a;
  a.tiles = (uint64_t)1 << (n - sw.T);
  a.low = sw.low;
  for (int b = sw.low; b < n; ++b)
    if ((sw.bits >> b) & 1) a.hi |= (uint64_t)b << (6 * a.nh++);
  a.nops = (int32_t)sw.members.size();
  a.mat16 = (int32_t)(sw.mat_bytes / 16);
  a.mat_off = (uint32_t)(sw.data_bytes - sw.mat_bytes);
  return a;
}

void encode_sweep(const Sweep& sw, const std::vector<const Pass*>& passes, const std::vector<const double*>& mats,
                  unsigned char* dst) {
  int tile_bit[64], tb = 0;
  for (int b = 0; b < 64; ++b) tile_bit[b] = (sw.bits >> b) & 1 ? tb++ : -1;
  // the passes, the matrices of kinds 1 and 2, then the block that goes to LDS
  size_t at = passes.size() * sizeof(SweepOp), big = 0;
  const size_t big_off = sw.data_bytes - sw.mat_bytes;
  for (size_t p = 0; p < passes.size(); ++p) {
    const Pass& ps = *passes[p];
    const int K = ps.k, kind = op_kind(K, ps.precision);
    SweepOp op{};
    op.kind = (uint32_t)kind;
    op.mat = (uint32_t)(K <= 2 ? at : big);
    // roles of the tile bits: the local bits (targets; for K = 1 one more in-lane
    // bit), lane bits, unit bits.  The lane bits j, and with them h, should fall on
    // different banks: bit 0 and tile bits b with different (b - 1) % 4.
    const int nl = std::max(K, 2);  // in-lane and h bits for K >= 3; the two in-lane bits for K <= 2
    bool taken[kSweepMaxBits] = {};
    int role[kSweepMaxBits], nr = 0;
    for (int j = 0; j < K; ++j) {
      role[nr++] = tile_bit[ps.s[j]];
      taken[role[nr - 1]] = true;
    }
    auto cls = [](int b) { return b == 0 ? 4 : (b - 1) & 3; };
    for (int b = sw.T - 1; b >= 0 && nr < nl; --b)  // the in-lane bit left at K = 1, from the top
      if (!taken[b]) taken[role[nr++] = b] = true;
    bool cls_used[5] = {};
    const int lanes = K <= 2 ? 6 : 4;
    if (K >= 3) cls_used[cls(role[K - 2])] = true;  // h bit 0
    int got = 0;
    for (int pass = 0; pass < 2 && got < lanes; ++pass)  // distinct classes first, then any
      for (int b = 0; b < sw.T && got < lanes; ++b) {
        if (taken[b] || (pass == 0 && cls_used[cls(b)])) continue;
        cls_used[cls(b)] = true;
        taken[b] = true;
        role[nr++] = b;
        ++got;
      }
    for (int b = 0; b < sw.T; ++b)
      if (!taken[b]) role[nr++] = b;
    for (int b = 0; b < sw.T; ++b) op.mask[b] = bit_mask(role[b]);
    std::memcpy(dst + p * sizeof(SweepOp), &op, sizeof(op));
    const double* m = mats[p];
    float* f = reinterpret_cast<float*>(dst + (K <= 2 ? at : big_off + big));
    (K <= 2 ? at : big) += op_mat_bytes(kind);
    if (K <= 2) {
      for (size_t e = 0; e < (size_t)2 << (2 * K); ++e) f[e] = (float)m[e];
      continue;
    }
    if (kind > kSweepSplit) {
      // [row tile t][k-step s][hi, lo][lane][e]: entry e of lane (h, j) is row
      // (amplitude (j / 4) N + 2 t + (j / 2) % 2, part j % 2), column
      // (amplitude h N + 4 s + e / 2, part e % 2)
      const int N = 1 << (K - 2), D = 1 << K;
      uint16_t* o = reinterpret_cast<uint16_t*>(f);
      for (int t = 0; t < N / 2; ++t)
        for (int s = 0; s < N / 4; ++s, o += 2 * 64 * 8)
          for (int lane = 0; lane < 64; ++lane) {
            const int h = lane >> 4, j = lane & 15;
            const int row = (j >> 2) * N + 2 * t + ((j >> 1) & 1), rp = j & 1;
            for (int e = 0; e < 8; ++e) {
              const int col = h * N + 4 * s + (e >> 1), cp = e & 1;
              const double ur = m[2 * ((size_t)row * D + col)], ui = m[2 * ((size_t)row * D + col) + 1];
              split_entry(ps.precision, rp == cp ? ur : rp == 0 ? -ui : ui, o[lane * 8 + e], o[64 * 8 + lane * 8 + e]);
            }
          }
      continue;
    }
    // [row tile t][column pair i2][h][row r of 8]: lane h holds the
    // amplitudes h N + i; row r of tile t is amplitude (r / 2) N + 2 t + r % 2
    const int N = 1 << (K - 2), D = 1 << K;
    for (int t = 0; t < N / 2; ++t)
      for (int i2 = 0; i2 < N / 2; ++i2)
        for (int h = 0; h < 4; ++h)
          for (int r = 0; r < 8; ++r)
            for (int w = 0; w < 2; ++w, f += 2) {
              const int row = (r >> 1) * N + 2 * t + (r & 1), col = h * N + 2 * i2 + w;
              const size_t e = (size_t)2 * (row * D + col);
              f[0] = (float)m[e];
              f[1] = (float)m[e + 1];
            }
  }
  if (at != big_off || big != sw.mat_bytes) throw std::logic_error("sweep matrices do not match their plan");
}

}  // namespace sv
