// Tile sweeps: several gate passes in one read and write of the state (see
// sweep.h for the scheme).
//
// Every pass of a sweep runs on the tile in LDS, so a sweep of m passes moves
// 16 bytes per amplitude through HBM once instead of m times.  A k = 3..6
// pass is a real GEMM in the 4M form ([Yr; Yi] = [[Ur, -Ui], [Ui, Ur]] [Xr; Xi]) on
// v_mfma_f32_16x16x4_f32: FP32 products and FP32 accumulation.  Lane (h, j)
// of a unit (16 groups of 2^K amplitudes) holds the amplitudes h 2^(K-2) + i of
// group j: the rows and columns of the real matrix are ordered on the host so
// that a lane's inputs and its outputs are the same amplitudes, and a pass
// reads and writes its tile in place with no exchange between lanes.  No pass
// is padded to a larger one: products with the zeros of a padding would carry an
// infinite or NaN amplitude out of its group.  k = 1, 2 passes multiply on the
// vector ALUs, each lane on four amplitudes of its own.
#include <type_traits>

#include "k_common.h"
#include "sweep.h"

namespace sv {

namespace {
using namespace kern;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;

// Slots are float4 (two amplitudes); slot bits 0..3 are XORed with bits 4..7
// and 8..11 so that strided accesses spread over the LDS banks.
__device__ __forceinline__ int swz(int e) { return e ^ (((e >> 4) ^ (e >> 8)) & 15); }

// Barrier between the passes on a tile: orders the LDS accesses of the
// workgroup only, so the loads of the next tile stay in flight across it.
__device__ __forceinline__ void tile_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// XOR of the masks of the set bits of v (NB bits, starting at mask[from])
template <int NB>
__device__ __forceinline__ uint32_t mix(const SweepOp& op, int from, int v) {
  uint32_t a = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) a ^= ((v >> b) & 1) ? op.mask[from + b] : 0u;
  return a;
}

__device__ __forceinline__ float2& amp(unsigned char* t, uint32_t byte) { return *reinterpret_cast<float2*>(t + byte); }

// A K-qubit pass on the matrix cores.  A wave takes UPW whole units, or, when
// the tile has fewer units than the workgroup waves, WPU waves share a unit
// and split its output rows (all of them read the unit before any writes it).
// PAIRS (K = 3 in BF16X3 sweeps): each instruction adds two products, amplitudes
// a and a + 4, instead of four, the others being 0 * 0: the order in which the
// sums were formed when these passes ran as K = 4.  A last bit that falls
// differently here moves the 16-bit splits of the passes that follow by up to
// 1.7e-5 of the result.
template <int T, int NW, int K, bool PAIRS = false>
__device__ __forceinline__ void op_mfma(unsigned char* tile, const SweepOp& op, const unsigned char* mats, int wave,
                                        int lane) {
  if constexpr (T >= K + 4) {
    constexpr int IB = K - 2, N = 1 << IB, R = 2 * N, RT = N / 2;
    constexpr int UB = T - K - 4, UNITS = 1 << UB;
    constexpr int UPW = UNITS >= NW ? UNITS / NW : 1;
    constexpr int WPU = UNITS >= NW ? 1 : (NW / UNITS < RT ? NW / UNITS : RT);
    constexpr int RTW = RT / WPU;                   // row tiles per wave
    constexpr int TB = UPW == 1 && RTW > 1 ? 2 : 1; // row tiles at a time
    const bool on = wave < UNITS / UPW * WPU;
    float b[UPW][R];
    uint32_t up[UPW];
    if (on) {
      const uint32_t lp = mix<6>(op, IB, ((lane & 15) << 2) | (lane >> 4));
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        up[u] = lp ^ mix<UB>(op, IB + 6, wave / WPU * UPW + u);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float2 v = amp(tile, up[u] ^ mix<IB>(op, 0, i));
          b[u][2 * i] = v.x;
          b[u][2 * i + 1] = v.y;
        }
      }
    }
    if constexpr (WPU > 1) tile_sync();
    if (!on) return;
    // row tile t, columns 2 i2, 2 i2 + 1 of this lane's h: (ur, ui) pairs of
    // amplitude row (lane & 15) >> 1; rows come as (re, im) = (ur, -ui), (ui, ur)
    const float4* A = reinterpret_cast<const float4*>(mats + op.mat) + ((lane >> 4) * 8 + ((lane & 15) >> 1));
    const bool im = lane & 1;
    const int t0 = (wave % WPU) * RTW;
#pragma unroll
    for (int tt = 0; tt < RTW; tt += TB) {
      f32x4 acc[TB][UPW];
#pragma unroll
      for (int q = 0; q < TB; ++q)
#pragma unroll
        for (int u = 0; u < UPW; ++u) acc[q][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i2 = 0; i2 < N / 2; ++i2) {
        float a[TB][4];
#pragma unroll
        for (int q = 0; q < TB; ++q) {
          const float4 f = A[((t0 + tt + q) * (N / 2) + i2) * 32];
          a[q][0] = im ? f.y : f.x;
          a[q][1] = im ? f.x : -f.y;
          a[q][2] = im ? f.w : f.z;
          a[q][3] = im ? f.z : -f.w;
        }
#pragma unroll
        for (int half = 0; half < (PAIRS ? 2 : 1); ++half) {
          const bool in = !PAIRS || ((lane >> 4) & 1) == half;
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int q = 0; q < TB; ++q)
#pragma unroll
              for (int u = 0; u < UPW; ++u)
                acc[q][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? a[q][s] : 0.f, in ? b[u][4 * i2 + s] : 0.f,
                                                                 acc[q][u], 0, 0, 0);
        }
      }
#pragma unroll
      for (int q = 0; q < TB; ++q)
#pragma unroll
        for (int u = 0; u < UPW; ++u)
#pragma unroll
          for (int w = 0; w < 2; ++w) {
            // in-lane index 2 t + w; t0 is only known at run time when waves share a unit
            const uint32_t at = up[u] ^ mix<IB>(op, 0, 2 * (t0 + tt + q) + w);
            amp(tile, at) = make_float2(acc[q][u][2 * w], acc[q][u][2 * w + 1]);
          }
    }
  }
}

// The same pass with split operands (x = hi + lo, three products) on
// v_mfma_f32_16x16x32: a k-step is four amplitudes of every lane.  The tile
// holds FP32 amplitudes between passes, split as k_mfma.hip splits them.
template <int T, int NW, int K, int PREC>
__device__ __forceinline__ void op_split(unsigned char* tile, const SweepOp& op, const unsigned char* mats, int wave,
                                         int lane) {
  if constexpr (T >= K + 4) {
    using frag = typename std::conditional<PREC == SV_PREC_BF16X3, bf16x8, f16x8>::type;
    constexpr int IB = K - 2, N = 1 << IB, S = N / 4, RT = N / 2;
    constexpr int UB = T - K - 4, UNITS = 1 << UB;
    constexpr int UPW = UNITS >= NW ? UNITS / NW : 1;
    constexpr int WPU = UNITS >= NW ? 1 : (NW / UNITS < RT ? NW / UNITS : RT);
    constexpr int RTW = RT / WPU;
    const bool on = wave < UNITS / UPW * WPU;
    frag hi[UPW][S], lo[UPW][S];
    uint32_t up[UPW];
    if (on) {
      const uint32_t lp = mix<6>(op, IB, ((lane & 15) << 2) | (lane >> 4));
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        up[u] = lp ^ mix<UB>(op, IB + 6, wave / WPU * UPW + u);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float2 v = amp(tile, up[u] ^ mix<IB>(op, 0, i));
#pragma unroll
          for (int part = 0; part < 2; ++part) {
            const float x = part ? v.y : v.x;
            const int s = i / 4, e = 2 * (i % 4) + part;
            if constexpr (PREC == SV_PREC_BF16X3) {
              const short h = __builtin_bit_cast(short, (__bf16)x);
              hi[u][s][e] = h;
              lo[u][s][e] = __builtin_bit_cast(short, (__bf16)(x - __uint_as_float((uint32_t)(uint16_t)h << 16)));
            } else {
              const float xs = x * kSplitF16Scale;
              const _Float16 h = (_Float16)xs;
              hi[u][s][e] = h;
              lo[u][s][e] = (_Float16)((xs - (float)h) * kSplitF16LoScale);
            }
          }
        }
      }
    }
    if constexpr (WPU > 1) tile_sync();
    if (!on) return;
    const frag* A = reinterpret_cast<const frag*>(mats + op.mat) + lane;  // [row tile][k-step][hi, lo][lane]
    const int t0 = (wave % WPU) * RTW;
#pragma unroll
    for (int tt = 0; tt < RTW; ++tt) {
      f32x4 acc[UPW], cor[UPW];
#pragma unroll
      for (int u = 0; u < UPW; ++u) acc[u] = cor[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const frag ah = A[(((t0 + tt) * S + s) * 2) * 64], al = A[(((t0 + tt) * S + s) * 2 + 1) * 64];
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
          if constexpr (PREC == SV_PREC_BF16X3) {
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, hi[u][s], acc[u], 0, 0, 0);
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, lo[u][s], acc[u], 0, 0, 0);
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, hi[u][s], acc[u], 0, 0, 0);
          } else {
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, hi[u][s], acc[u], 0, 0, 0);
            cor[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, lo[u][s], cor[u], 0, 0, 0);
            cor[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, hi[u][s], cor[u], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < UPW; ++u) {
        float y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          y[q] = PREC == SV_PREC_BF16X3 ? acc[u][q]
                                        : (acc[u][q] + cor[u][q] * (1.f / kSplitF16LoScale)) * (1.f / kSplitF16Scale);
#pragma unroll
        for (int w = 0; w < 2; ++w)
          amp(tile, up[u] ^ mix<IB>(op, 0, 2 * (t0 + tt) + w)) = make_float2(y[2 * w], y[2 * w + 1]);
      }
    }
  }
}

// A one- or two-qubit pass on the vector ALUs: local bits are in-lane bits.
template <int T, int NW, int K>
__device__ __forceinline__ void op_valu(unsigned char* tile, const SweepOp& op, const unsigned char* __restrict__ data,
                                        int wave, int lane) {
  constexpr int D = 1 << K;
  constexpr int UNITS = 1 << (T - 8);
  constexpr int UPW = UNITS >= NW ? UNITS / NW : 1;
  if (wave * UPW >= UNITS) return;
  const float2* __restrict__ U = reinterpret_cast<const float2*>(data + op.mat);
  const uint32_t lp = mix<6>(op, 2, lane);
  constexpr int UC = UPW > 2 ? 2 : UPW;  // units at a time
#pragma unroll
  for (int u0 = 0; u0 < UPW; u0 += UC) {
    uint32_t up[UC];
    float2 v[UC][4];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      up[u] = lp ^ mix<T - 8>(op, 8, wave * UPW + u0 + u);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[u][i] = amp(tile, up[u] ^ mix<2>(op, 0, i));
    }
#pragma unroll
    for (int u = 0; u < UC; ++u)
#pragma unroll
      for (int g = 0; g < 4; g += D)
#pragma unroll
        for (int r = 0; r < D; ++r) {
          float2 o = make_float2(0.f, 0.f);
#pragma unroll
          for (int c = 0; c < D; ++c) cmac(o, U[r * D + c], v[u][g + c]);
          amp(tile, up[u] ^ mix<2>(op, 0, g + r)) = o;
        }
  }
}

// A workgroup walks tiles t, t + stride, ...: the next
// tile's loads are issued before the passes run on the current one, so memory
// and the matrix cores work at the same time (with one tile per workgroup the
// workgroups of a launch stayed in step, all loading and then all
// multiplying: 56 ms against 48 for a 28-qubit grid of 103 k = 4 passes in 46
// sweeps).  The matrices of the k >= 3 passes are copied to LDS once.  At 28
// qubits a sweep's traffic alone takes 0.80-0.82 ms (5.3 TB/s); a k = 4 pass
// adds 0.25-0.30 ms of matrix-core time once there are more than two, so three
// passes take about 1.0 ms where they took 2.4 as launches.
// PREC: the split precision of the k >= 4 passes, or SV_PREC_FP32_MFMA.
template <int T, int NW, bool NT, int PREC>
__device__ __forceinline__ void sweep_tiles(float4* __restrict__ psi, const unsigned char* __restrict__ data,
                                            const SweepArgs& d, uint64_t t, uint64_t stride, unsigned char* smem) {
  unsigned char* tile = smem;
  unsigned char* mats = smem + ((size_t)8 << T);
  constexpr int SLOTS = 1 << (T - 1);
  constexpr int NTHR = 64 * NW;
  constexpr int PER = SLOTS >= NTHR ? SLOTS / NTHR : 1;
  const int tid = threadIdx.x;
  const int L = d.low, nh = d.nh, nops = d.nops;
  // first element of a tile: its number spread over the state bits outside it
  auto first = [&](uint64_t t) {
    uint64_t b = t << L, hi = d.hi;
    for (int i = 0; i < nh; ++i, hi >>= 6) {
      const uint64_t lm = ((uint64_t)1 << (hi & 63)) - 1;
      b = ((b & ~lm) << 1) | (b & lm);
    }
    return b >> 1;
  };
  // amplitude offset of tile index x
  auto spread = [&](uint32_t x) {
    uint64_t o = x & ((1u << L) - 1);
    uint64_t hi = d.hi;
    for (int i = 0; i < nh; ++i, hi >>= 6) o |= (uint64_t)((x >> (L + i)) & 1) << (hi & 63);
    return o;
  };
  const uint64_t own = spread(2 * tid) >> 1;
  uint64_t off[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) off[i] = spread(2 * NTHR * i) >> 1;
  float4* slots = reinterpret_cast<float4*>(tile);
  const bool mine = SLOTS >= NTHR || tid < SLOTS;
  const SweepOp* __restrict__ ops = reinterpret_cast<const SweepOp*>(data);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  float4 r[PER];
  float4* cur = psi + first(t) + own;
  if (mine) {
#pragma unroll
    for (int i = 0; i < PER; ++i) r[i] = gld<NT>(cur + off[i]);
  }
  {
    const float4* from = reinterpret_cast<const float4*>(data + d.mat_off);
    float4* to = reinterpret_cast<float4*>(mats);
    for (int i = tid; i < d.mat16; i += NTHR) to[i] = from[i];
  }
  while (true) {
    // a thread's slots are its own between the store and the next load
    if (mine) {
#pragma unroll
      for (int i = 0; i < PER; ++i) slots[swz(tid + NTHR * i)] = r[i];
    }
    tile_sync();
    const uint64_t tn = t + stride;
    float4* next = psi + first(tn) + own;
    if (mine && tn < d.tiles) {
#pragma unroll
      for (int i = 0; i < PER; ++i) r[i] = gld<NT>(next + off[i]);
    }
    SweepOp op = ops[0];
    for (int o = 0; o < nops; ++o) {
      const SweepOp ahead = ops[o + 1 < nops ? o + 1 : o];  // its scalar loads run beside this pass
      switch (op.kind) {
        case 1: op_valu<T, NW, 1>(tile, op, data, wave, lane); break;
        case 2: op_valu<T, NW, 2>(tile, op, data, wave, lane); break;
        case 4: op_mfma<T, NW, 4>(tile, op, mats, wave, lane); break;
        default:  // kinds are set on the host
          if constexpr (PREC != SV_PREC_FP32_MFMA) {
            if (op.kind == kSweepSplit + 4) op_split<T, NW, 4, PREC>(tile, op, mats, wave, lane);
            else if (op.kind == kSweepSplit + 5) op_split<T, NW, 5, PREC>(tile, op, mats, wave, lane);
            else if (op.kind == kSweepSplit + 6) op_split<T, NW, 6, PREC>(tile, op, mats, wave, lane);
          }
          if (op.kind == 3) op_mfma<T, NW, 3, PREC == SV_PREC_BF16X3>(tile, op, mats, wave, lane);
          else if (op.kind == 5) op_mfma<T, NW, 5>(tile, op, mats, wave, lane);
          else if (op.kind == 6) op_mfma<T, NW, 6>(tile, op, mats, wave, lane);
      }
      tile_sync();
      op = ahead;
    }
    if (mine) {
#pragma unroll
      for (int i = 0; i < PER; ++i) gst<NT>(cur + off[i], slots[swz(tid + NTHR * i)]);
    }
    if (tn >= d.tiles) break;
    t = tn;
    cur = next;
  }
}

template <int T, int NW, bool NT, int PREC>
__global__ __launch_bounds__(64 * NW) void k_sweep(float4* __restrict__ psi, const unsigned char* __restrict__ data,
                                                   const SweepArgs d) {
  extern __shared__ __align__(16) unsigned char smem[];
  sweep_tiles<T, NW, NT, PREC>(psi, data, d, blockIdx.x, gridDim.x, smem);
}

// The same sweeps of many states in one launch: entry e of the table owns
// workgroups first[e] .. first[e + 1) - 1.  Tiles of at most 2^12 amplitudes.
template <bool NT>
__global__ __launch_bounds__(512) void k_sweep_batch(const unsigned char* __restrict__ data,
                                                     const BatchSweep* __restrict__ table, int count) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t b = blockIdx.x;
  int lo = 0, hi = count - 1;  // last entry with first <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (table[mid].first <= b) lo = mid;
    else hi = mid - 1;
  }
  const BatchSweep e = table[lo];
  const uint64_t t = b - e.first;
  switch (e.T) {
    case 8: sweep_tiles<8, 8, NT, SV_PREC_FP32_MFMA>(e.psi, data + e.data, e.args, t, e.groups, smem); break;
    case 9: sweep_tiles<9, 8, NT, SV_PREC_FP32_MFMA>(e.psi, data + e.data, e.args, t, e.groups, smem); break;
    case 10: sweep_tiles<10, 8, NT, SV_PREC_FP32_MFMA>(e.psi, data + e.data, e.args, t, e.groups, smem); break;
    case 11: sweep_tiles<11, 8, NT, SV_PREC_FP32_MFMA>(e.psi, data + e.data, e.args, t, e.groups, smem); break;
    case 12: sweep_tiles<12, 8, NT, SV_PREC_FP32_MFMA>(e.psi, data + e.data, e.args, t, e.groups, smem); break;
    default: break;  // tile sizes are set on the host
  }
}

// Lets a kernel take the most dynamic LDS any sweep asks for.  The limit belongs
// to the kernel, not to a launch: threads launch sweeps of different sizes at
// the same time, so every one of them sets the same value.
void allow_lds(const void* kernel, size_t lds) {
  if (lds > kSweepLds) throw DeviceError{hipErrorInvalidValue, "k_sweep: LDS of a workgroup"};
  if (lds > 65536)  // above the default limit
    SV_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSweepLds));
}

constexpr uint64_t kSweepGroups = 512;  // workgroups of a launch: two per CU

template <int T, int NW, int PREC>
void launch_p(const Sweep& sw, int n, void* psi, const unsigned char* data, hipStream_t st) {
  const SweepArgs a = sweep_args(sw, n);
  const dim3 grid((unsigned)(a.tiles < kSweepGroups ? a.tiles : kSweepGroups));
  const size_t lds = ((size_t)8 << T) + sw.mat_bytes;
  auto* kernel = n >= kNtMinQubits ? k_sweep<T, NW, true, PREC> : k_sweep<T, NW, false, PREC>;
  allow_lds((const void*)kernel, lds);
  hipLaunchKernelGGL(kernel, grid, dim3(64 * NW), lds, st, (float4*)psi, data, a);
}

template <int T, int NW>
void launch_t(const Sweep& sw, int n, void* psi, const unsigned char* data, hipStream_t st) {
  if constexpr (T <= 12) {
    if (sw.precision == SV_PREC_FP16X3) return launch_p<T, NW, SV_PREC_FP16X3>(sw, n, psi, data, st);
    if (sw.precision == SV_PREC_BF16X3) return launch_p<T, NW, SV_PREC_BF16X3>(sw, n, psi, data, st);
  }
  if (sw.precision != SV_PREC_FP32_MFMA) throw DeviceError{hipErrorInvalidValue, "k_sweep: precision"};
  launch_p<T, NW, SV_PREC_FP32_MFMA>(sw, n, psi, data, st);
}

}  // namespace

void launch_sweep(const Sweep& sw, int n, void* psi, const unsigned char* data, hipStream_t st) {
  if (sw.T > n) throw DeviceError{hipErrorInvalidValue, "k_sweep: tile larger than the state"};
  switch (sw.T) {
    case 8: launch_t<8, 8>(sw, n, psi, data, st); break;
    case 9: launch_t<9, 8>(sw, n, psi, data, st); break;
    case 10: launch_t<10, 8>(sw, n, psi, data, st); break;
    case 11: launch_t<11, 8>(sw, n, psi, data, st); break;
    case 12: launch_t<12, 8>(sw, n, psi, data, st); break;
    case 13: launch_t<13, 8>(sw, n, psi, data, st); break;
    default: throw DeviceError{hipErrorInvalidValue, "k_sweep: tile bits"};
  }
  SV_HIP(hipGetLastError());
}

void launch_sweep_batch(const BatchSweep* table, int count, unsigned groups, size_t lds, bool nt,
                        const unsigned char* data, hipStream_t st) {
  auto* kernel = nt ? k_sweep_batch<true> : k_sweep_batch<false>;
  allow_lds((const void*)kernel, lds);
  hipLaunchKernelGGL(kernel, dim3(groups), dim3(512), lds, st, data, table, count);
  SV_HIP(hipGetLastError());
}

}  // namespace sv
