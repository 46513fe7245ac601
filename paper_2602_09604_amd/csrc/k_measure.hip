// Reads of the state that write nothing back (the expectation-value kernel
// of Sec. IV, and the Born probabilities of Eq. 1 behind measurement):
// Pauli-string expectations, marginal probabilities and inverse-CDF
// sampling.  Every sum is in FP64 in a fixed order, so results do not vary
// between runs; squares and products of complex64 amplitudes are formed in
// FP64, where they are exact.
#include <algorithm>

#include "k_common.h"

namespace sv {

namespace {
using kern::gld;

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 2048;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double sq(const float2 a) {
  return (double)a.x * (double)a.x + (double)a.y * (double)a.y;
}

// ------------------------------------------------------------ Pauli strings
// Up to kTerms strings that share the flip mask f = X|Y part.  For P = i^ny
// X^f Z^z: <psi|P|psi> = i^ny sum_i (-1)^{|(i^f) & z|} conj(c_i) c_{i^f}.
// With f != 0 the sum runs over pairs (i, j = i^f) with bit h (the highest
// bit of f) clear in i; the pair contributes s_i w + s_j conj(w), w =
// conj(c_i) c_j, s_j = (-1)^{|i & z|} and s_i = s_j (-1)^{|f & z|}.  So a
// term with |f & z| even collects 2 s_j Re w (a real sum) and one with
// |f & z| odd collects -2i s_j Im w.  Each amplitude is read once.
constexpr int kTerms = 8;
struct PauliArgs {
  uint64_t f;
  uint64_t items;          // float4 elements (f == 0 or f == 1) or element quads; a power of two
  uint64_t lowmask;        // ones below bit h
  uint64_t z[kTerms];
  uint32_t chi[kTerms][4]; // high words of the FP64 coefficients (+-1 or 0) of each item value
  uint32_t odd;            // bit t: |f & z_t| is odd
};

// First amplitude index of item x: 2x for elements; for quads, 2x with a
// zero inserted at bit h (the bit-h-clear member of the pair).
template <int MODE>
__device__ __forceinline__ uint64_t first_amp(const PauliArgs& a, uint64_t x) {
  const uint64_t g = 2 * x;
  return MODE == 2 ? ((g & ~a.lowmask) << 1) | (g & a.lowmask) : g;
}

__device__ __forceinline__ uint32_t sign_bits(const PauliArgs& a, uint64_t i, int terms) {
  uint32_t s = 0;
#pragma unroll
  for (int t = 0; t < kTerms; ++t)
    if (t < terms) s |= (uint32_t)(__popcll(i & a.z[t]) & 1) << t;
  return s;
}

__device__ __forceinline__ double coef(uint32_t hi, uint32_t sign) {
  return __longlong_as_double((long long)((uint64_t)(hi ^ (sign << 31)) << 32));
}

// The values an item contributes, before signs: MODE 0, the two Born
// probabilities |c_i|^2, |c_{i+1}|^2; MODE 1, Re and Im of w = conj(c_i)
// c_{i+1}; MODE 2, Re and Im of w for the pairs at i and i + 1.
template <int MODE>
__device__ __forceinline__ void item_values(const float4 A, const float4 B, bool fodd, double* v) {
  if (MODE == 0) {
    v[0] = sq(make_float2(A.x, A.y));
    v[1] = sq(make_float2(A.z, A.w));
  } else if (MODE == 1) {
    v[0] = (double)A.x * A.z + (double)A.y * A.w;
    v[1] = (double)A.x * A.w - (double)A.y * A.z;
  } else {
    const float2 c0 = make_float2(A.x, A.y), c1 = make_float2(A.z, A.w);
    const float2 p0 = fodd ? make_float2(B.z, B.w) : make_float2(B.x, B.y);
    const float2 p1 = fodd ? make_float2(B.x, B.y) : make_float2(B.z, B.w);
    v[0] = (double)c0.x * p0.x + (double)c0.y * p0.y;
    v[1] = (double)c0.x * p0.y - (double)c0.y * p0.x;
    v[2] = (double)c1.x * p1.x + (double)c1.y * p1.y;
    v[3] = (double)c1.x * p1.y - (double)c1.y * p1.x;
  }
}

__device__ __forceinline__ double flip_if(double x, uint32_t bit) {
  return __longlong_as_double(__double_as_longlong(x) ^ (long long)((uint64_t)bit << 63));
}

// Two ways to apply the per-m signs (bit t of bits for term t):
// - SIGNS: bits are this item's signs; the coefficients take them (a sign
//   flip of each coefficient's high word, scalar work per value and term);
// - FLIPS: the accumulator holds B_t = (sign of the last item) * (sum so
//   far) and bits are where the sign changed since the last item: B_t is
//   turned over (one vector XOR per term), then the values are added with
//   fixed coefficients.
// Quads (mode 2: four values per item) measured faster with FLIPS (5.7
// against 6.1 ms for 8 terms at 32 qubits), elements (two values) with
// SIGNS (5.6-5.7 against 6.3 ms).
template <int MODE>
constexpr bool kFlips = MODE == 2;

template <int MODE, int TERMS>
__device__ __forceinline__ void accumulate(double* acc, const PauliArgs& a, uint32_t bits, const double* v) {
  constexpr int NV = MODE == 2 ? 4 : 2;
#pragma unroll
  for (int t = 0; t < TERMS; ++t) {
    const uint32_t b = (bits >> t) & 1u;
    if constexpr (kFlips<MODE>) {
      acc[t] = flip_if(acc[t], b);
#pragma unroll
      for (int c = 0; c < NV; ++c) acc[t] = fma(coef(a.chi[t][c], 0u), v[c], acc[t]);
    } else {
#pragma unroll
      for (int c = 0; c < NV; ++c) acc[t] = fma(coef(a.chi[t][c], b), v[c], acc[t]);
    }
  }
}

// Apply each thread's own signs (bit t of own), then sum the block's
// threads in a fixed order into row[t].  `part` is free again after the next
// call on another buffer.
using BlockPart = double[kThreads / 64][kTerms];
template <int TERMS>
__device__ __forceinline__ void block_partials(const double* acc, uint32_t own, BlockPart& part,
                                               double* __restrict__ row) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < TERMS; ++t) {
    const double r = wave_sum(((own >> t) & 1) ? -acc[t] : acc[t]);
    if (lane == 0) part[w][t] = r;
  }
  __syncthreads();
  if (threadIdx.x < TERMS) {
    double v = 0.0;
    for (int x = 0; x < kThreads / 64; ++x) v += part[x][threadIdx.x];
    row[threadIdx.x] = v;
  }
}

// The sums of several sweeps of a state held in the caches, in one launch:
// blockIdx.y is the sweep.  A sweep by itself is 4 to 8 us of launch and
// latency at 20 qubits whatever it reads, so an Ising Hamiltonian's 24 sweeps in
// a launch each, with a column sum behind every one, took 302 us; as three
// launches and a wait it takes 42.
template <int TERMS>
struct PauliSweeps {
  static constexpr int kMax = 3072 / (8 + 8 * TERMS);  // sweeps in one launch's arguments
  uint64_t f[kMax];
  uint64_t z[kMax][TERMS];
};

// coefficients, masks and walk of one sweep (host and device)
template <int TERMS>
__host__ __device__ inline int pauli_args(PauliArgs& a, int n, uint64_t f, const uint64_t* z) {
  a.f = f;
  a.odd = 0;
  const int mode = f > 1 ? 2 : (int)f;
  a.lowmask = 0;
  a.items = (uint64_t)1 << (n - 1);  // n = 1: one element
  if (mode == 2) {
    const int h = 63 - __builtin_clzll(f);  // h >= 1, so n >= 2
    a.lowmask = ((uint64_t)1 << h) - 1;
    a.items = (uint64_t)1 << (n - 2);
  }
  // mode 0 (|c_i|^2, |c_{i+1}|^2): the sign of z_t bit 0 on the second; modes
  // 1, 2: Re w for an even |f & z_t|, Im w for an odd one, and in mode 2 the
  // pair at i + 1 again signed by bit 0
  constexpr uint32_t kOne = 0x3FF00000u, kNeg = 0x80000000u;
#pragma unroll
  for (int t = 0; t < TERMS; ++t) {
    a.z[t] = z[t];
    const bool im = __builtin_popcountll(f & z[t]) & 1;
    a.odd |= (uint32_t)im << t;
    const uint32_t zeta = (z[t] & 1) ? kNeg : 0u;
    if (mode == 0) {
      a.chi[t][0] = kOne;
      a.chi[t][1] = kOne | zeta;
      a.chi[t][2] = a.chi[t][3] = 0u;
    } else {
      a.chi[t][0] = im ? 0u : kOne;
      a.chi[t][1] = im ? kOne : 0u;
      a.chi[t][2] = a.chi[t][0] ? a.chi[t][0] | zeta : 0u;
      a.chi[t][3] = a.chi[t][1] ? a.chi[t][1] | zeta : 0u;
    }
  }
  return mode;
}

// Block b of the walk owns M kThreads consecutive items (M and the number of
// blocks are powers of two) and its thread u the items T + m kThreads, T = b M
// kThreads + u, m < M.  The bits of first_amp(T) and first_amp(m kThreads) are
// disjoint, so the sign (-1)^{|i & z_t|} of every pair
// splits into a per-thread sign and a per-m sign that is the same for every
// lane; it reaches the sums through wave-uniform coefficients (+-1 or 0:
// the real-or-imaginary choice and the sign of bit 0 of z_t folded in), in
// one of the two ways described at accumulate, and the thread's own sign is
// applied once at the end.  Mode 0 and 1 items are float4 elements
// (amplitudes 2x, 2x + 1); mode 2 items are quads: the element at i (bit h
// clear, i even) and the element holding its partners i ^ f and
// (i + 1) ^ f.  Every thread keeps two items in flight.
// `blocks` follows from the state's size alone, and with it the order of every
// sum: a term rounds the same whatever else the call asks for.  A launch of
// many sweeps has fewer workgroups per sweep, each walking several blocks.
template <int MODE, int TERMS>
__device__ __forceinline__ void pauli_walk(const float4* __restrict__ psi, const PauliArgs& a, unsigned blocks,
                                           BlockPart* part, double* __restrict__ partials) {
  constexpr int NV = MODE == 2 ? 4 : 2;
  const uint64_t nth = (uint64_t)blocks * kThreads, M = a.items >= nth ? a.items / nth : 1;
  const uint64_t i_step = first_amp<MODE>(a, kThreads);
  const uint32_t step = sign_bits(a, i_step, TERMS);  // m even: m + 1 flips these
  const bool fodd = a.f & 1;  // the partner of i is the odd amplitude of its element
  int buffer = 0;
  for (unsigned block = blockIdx.x; block < blocks; block += gridDim.x, buffer ^= 1) {
    double acc[TERMS];
#pragma unroll
    for (int t = 0; t < TERMS; ++t) acc[t] = 0.0;
    const uint64_t T = (uint64_t)block * (kThreads * M) + threadIdx.x;
    const uint64_t iT = first_amp<MODE>(a, T);
    uint32_t last = 0;  // per-m sign bits of the last item added (FLIPS)
    if (T < a.items) {  // false only past the end of a state of fewer than nth items
      // the trip count and has1 are the same for every lane, so the four
      // loads of an iteration issue back to back (a lone last item loads
      // its own element twice)
      for (uint64_t m = 0; m < M; m += 2) {
        const bool has1 = m + 1 < M;
        const uint64_t im = first_amp<MODE>(a, m * kThreads);
        const uint64_t i0 = iT | im, i1 = has1 ? i0 | i_step : i0;
        const float4 A0 = gld<false>(psi + (i0 >> 1));
        const float4 A1 = gld<false>(psi + (i1 >> 1));
        float4 B0 = A0, B1 = A1;
        if (MODE == 2) {
          B0 = gld<false>(psi + (((i0 ^ a.f) & ~(uint64_t)1) >> 1));
          B1 = gld<false>(psi + (((i1 ^ a.f) & ~(uint64_t)1) >> 1));
        }
        const uint32_t sig = sign_bits(a, im, TERMS);
        double v[NV];
        item_values<MODE>(A0, B0, fodd, v);
        accumulate<MODE, TERMS>(acc, a, kFlips<MODE> ? sig ^ last : sig, v);
        last = sig;
        if (has1) {
          item_values<MODE>(A1, B1, fodd, v);
          accumulate<MODE, TERMS>(acc, a, kFlips<MODE> ? step : sig ^ step, v);
          last = sig ^ step;
        }
      }
    }
    const uint32_t own = sign_bits(a, iT, TERMS) ^ (kFlips<MODE> ? last : 0u);
    block_partials<TERMS>(acc, own, part[buffer], partials + (size_t)block * kTerms);
  }
}

template <int TERMS>
__global__ __launch_bounds__(kThreads) void k_pauli_sweeps(const float4* __restrict__ psi, int n,
                                                          const PauliSweeps<TERMS> s, int first, unsigned blocks,
                                                          double* __restrict__ partials) {
  __shared__ BlockPart part[2];
  PauliArgs a;
  const int mode = pauli_args<TERMS>(a, n, s.f[blockIdx.y], s.z[blockIdx.y]);
  double* out = partials + (size_t)(first + blockIdx.y) * blocks * kTerms;
  if (mode == 0) pauli_walk<0, TERMS>(psi, a, blocks, part, out);
  else if (mode == 1) pauli_walk<1, TERMS>(psi, a, blocks, part, out);
  else pauli_walk<2, TERMS>(psi, a, blocks, part, out);
}

// The same sums on a streamed state, walked the way the sampling chunk sums
// walk it: wave W of NW takes chunks of R = 2048 consecutive items, W,
// W + NW, W + 2 NW, ..., each in 32 steps of 64 lanes, two steps in flight
// (so the waves in flight read a moving window of the state, each its own
// 32 KiB run; a grid-stride walk spreads every wave over the whole state).  Item x = c NW R + W R + k 64 + lane splits into disjoint bit
// fields, so the per-thread part of every sign comes from W R + lane and
// the wave-uniform part from c NW R + k 64.  Needs items to be a multiple
// of NW R.
constexpr uint64_t kChunkItems = 2048;
template <int MODE, int TERMS>
__global__ __launch_bounds__(kThreads) void k_pauli_chunks(const float4* __restrict__ psi, const PauliArgs a,
                                                          double* __restrict__ partials) {
  constexpr int NV = MODE == 2 ? 4 : 2;
  __shared__ BlockPart part;
  double acc[TERMS];
#pragma unroll
  for (int t = 0; t < TERMS; ++t) acc[t] = 0.0;
  const uint64_t NW = (uint64_t)gridDim.x * (kThreads / 64);
  const uint64_t W = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const uint64_t iT = first_amp<MODE>(a, W * kChunkItems + lane);
  const uint64_t rounds = a.items / (NW * kChunkItems);
  const bool fodd = a.f & 1;
  uint32_t last = 0;
  for (uint64_t c = 0; c < rounds; ++c) {
    for (uint64_t k = 0; k < kChunkItems / 64; k += 2) {
      const uint64_t im0 = first_amp<MODE>(a, c * NW * kChunkItems + k * 64);
      const uint64_t im1 = first_amp<MODE>(a, c * NW * kChunkItems + (k + 1) * 64);
      const uint64_t i0 = iT | im0, i1 = iT | im1;
      const float4 A0 = gld<true>(psi + (i0 >> 1));
      const float4 A1 = gld<true>(psi + (i1 >> 1));
      float4 B0 = A0, B1 = A1;
      if (MODE == 2) {
        B0 = gld<true>(psi + (((i0 ^ a.f) & ~(uint64_t)1) >> 1));
        B1 = gld<true>(psi + (((i1 ^ a.f) & ~(uint64_t)1) >> 1));
      }
      const uint32_t sig0 = sign_bits(a, im0, TERMS), sig1 = sign_bits(a, im1, TERMS);
      double v[NV];
      item_values<MODE>(A0, B0, fodd, v);
      accumulate<MODE, TERMS>(acc, a, kFlips<MODE> ? sig0 ^ last : sig0, v);
      item_values<MODE>(A1, B1, fodd, v);
      accumulate<MODE, TERMS>(acc, a, kFlips<MODE> ? sig1 ^ sig0 : sig1, v);
      last = sig1;
    }
  }
  const uint32_t own = sign_bits(a, iT, TERMS) ^ (kFlips<MODE> ? last : 0u);
  block_partials<TERMS>(acc, own, part, partials + (size_t)blockIdx.x * kTerms);
}

// Column sums of the blocks x width matrix of per-block partials, in a fixed
// order: workgroup g owns columns 64 g .. 64 g + 63 (one per lane); each of
// its 16 waves sums a contiguous run of rows, and wave 0 then adds the 16
// wave sums in wave order.
constexpr int kFinalWaves = 16;
__global__ __launch_bounds__(64 * kFinalWaves) void k_column_sums(const double* __restrict__ partials, int blocks,
                                                                  int width, double* __restrict__ out) {
  __shared__ double part[kFinalWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + lane;
  const int per = (blocks + kFinalWaves - 1) / kFinalWaves;
  const int b0 = w * per, b1 = b0 + per < blocks ? b0 + per : blocks;
  double s = 0.0;
  if (col < width) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += partials[(size_t)b * width + col];
  }
  part[w][lane] = s;
  __syncthreads();
  if (w != 0 || col >= width) return;
  double t = 0.0;
  for (int x = 0; x < kFinalWaves; ++x) t += part[x][lane];
  out[col] = t;
}

// The Pauli sums of every sweep: workgroup s adds the blocks x kTerms partials
// of sweep s in a fixed order, 128 rows at a time (columns past a sweep's terms
// hold nothing and reach nothing).
constexpr int kFinalRows = 128;
__global__ __launch_bounds__(kFinalRows * kTerms) void k_pauli_final(const double* __restrict__ partials, int blocks,
                                                                    double* __restrict__ out) {
  __shared__ double part[kFinalRows * kTerms];
  const double* p = partials + (size_t)blockIdx.x * blocks * kTerms;
  double s = 0.0;
#pragma unroll 8
  for (int i = threadIdx.x; i < blocks * kTerms; i += kFinalRows * kTerms) s += p[i];
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;  // 8 runs of 16 rows, then across the runs
  double t = 0.0;
#pragma unroll
  for (int r = 0; r < kFinalRows / 8; ++r) t += part[((threadIdx.x >> 3) * (kFinalRows / 8) + r) * kTerms + (threadIdx.x & 7)];
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
  if (threadIdx.x < kTerms) out[(size_t)blockIdx.x * kTerms + threadIdx.x] = t;
}

// ------------------------------------------------------- marginal probabilities
// Chunks of 64 consecutive amplitudes are visited in the order c' = (oh,
// free): chunk c = deposit(free, fc) | deposit(oh, hc), where hc holds the
// measured qubits at or above bit 6 (in chunk units) and fc the others.
// Each wave walks a contiguous range of c', so within a run of equal oh its
// lanes accumulate privately (lane = index bits 0..5).  When oh changes, a
// butterfly over the lane bits that are not measured leaves, in the lanes
// whose unmeasured lane bits are zero, the sum over lanes sharing their
// measured low bits; those lanes (distinct outcomes) add it to the wave's
// own LDS histogram, so no two lanes update one bin at once and the order of
// every sum is fixed.
constexpr int kMaxMeasured = 10;
struct MargArgs {
  uint64_t len;          // 2^n
  uint64_t nchunks;      // 2^(n-6), or 1 for n < 6
  uint64_t fc;           // chunk-index bits that are not measured
  uint64_t hc;           // chunk-index bits that are measured (qubit q >= 6 -> bit q - 6)
  int free_bits;         // popcount(fc)
  int m;
  int q[kMaxMeasured];
  uint32_t low_meas;     // measured qubits among bits 0..5
};

__device__ __forceinline__ uint64_t deposit(uint64_t x, uint64_t mask) {
  uint64_t r = 0;
  for (uint64_t m = mask; m; m &= m - 1, x >>= 1)
    if (x & 1) r |= m & (~m + 1);
  return r;
}

__device__ __forceinline__ int outcome(uint64_t i, const MargArgs& a) {
  int o = 0;
#pragma unroll
  for (int j = 0; j < kMaxMeasured; ++j)
    if (j < a.m) o |= (int)((i >> a.q[j]) & 1) << j;
  return o;
}

template <bool NT>
__global__ __launch_bounds__(kThreads) void k_marginal_partial(const float2* __restrict__ psi, const MargArgs a,
                                                              double* __restrict__ partials) {
  extern __shared__ double hist[];  // [4 waves][2^m]
  const int M = 1 << a.m;
  for (int x = threadIdx.x; x < 4 * M; x += kThreads) hist[x] = 0.0;
  __syncthreads();
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* __restrict__ h = hist + w * M;
  const bool owner = ((uint32_t)lane & ~a.low_meas & 63u) == 0;
  const uint64_t waves = (uint64_t)gridDim.x * 4;
  const uint64_t per = (a.nchunks + waves - 1) / waves;
  const uint64_t c0 = ((uint64_t)blockIdx.x * 4 + w) * per;
  const uint64_t c1 = c0 + per < a.nchunks ? c0 + per : a.nchunks;
  if (c0 < c1) {
    uint64_t oh = c0 >> a.free_bits;
    uint64_t cf = deposit(c0 & (((uint64_t)1 << a.free_bits) - 1), a.fc);
    uint64_t ch = deposit(oh, a.hc);
    for (uint64_t cp = c0; cp < c1;) {
      const uint64_t run_end = ((oh + 1) << a.free_bits) < c1 ? ((oh + 1) << a.free_bits) : c1;
      double acc = 0.0;
      for (; cp + 4 <= run_end; cp += 4) {
        uint64_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          c[u] = cf | ch;
          cf = ((cf | ~a.fc) + 1) & a.fc;
        }
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = sq(gld<NT>(psi + (c[u] << 6) + lane));
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += v[u];
      }
      for (; cp < run_end; ++cp) {
        const uint64_t i = ((cf | ch) << 6) + lane;
        acc += i < a.len ? sq(psi[i]) : 0.0;
        cf = ((cf | ~a.fc) + 1) & a.fc;
      }
#pragma unroll
      for (int b = 0; b < 6; ++b)
        if (!((a.low_meas >> b) & 1)) acc += __shfl_xor(acc, 1 << b, 64);
      if (owner) h[outcome((ch << 6) + lane, a)] += acc;
      ++oh;
      ch = deposit(oh, a.hc);
    }
  }
  __syncthreads();
  for (int o = threadIdx.x; o < M; o += kThreads) {
    double v = 0.0;
    for (int x = 0; x < 4; ++x) v += hist[x * M + o];
    partials[(size_t)blockIdx.x * M + o] = v;
  }
}

// ------------------------------------------------------------------ sampling
// 1. sums of |c_i|^2 over chunks of 2^c amplitudes (one wave per chunk) and
//    over the 2^b equal parts of each (up to eight parts of at least 512);
// 2. inclusive prefix sums of the chunk sums (blocks of 2048, then the block
//    totals, then the offsets added back);
// 3. per shot, a binary search for the first chunk whose inclusive prefix
//    exceeds u * total (one thread per shot);
// 4. per shot (one wave), a scan over that chunk's parts and one over the
//    part, eight amplitudes per lane, for the first amplitude that crosses
//    the remainder.
// A wave of step 4 is a chain of three dependent loads and reads 4 KB of the
// state.  At 28 qubits and 100000 shots a wave that searched by itself and
// stepped through the chunk 64 amplitudes at a time took 666 us; steps 3 and 4
// take 9 + 108 us (159 with 8-byte loads in step 4), and the parts cost step 1
// 12 us of 328.
template <bool NT>
__global__ __launch_bounds__(kThreads) void k_chunk_sums(const float2* __restrict__ psi, int cbits, int bbits,
                                                        uint64_t nchunks, double* __restrict__ sums,
                                                        double* __restrict__ parts) {
  const uint64_t ch = ((uint64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (ch >= nchunks) return;  // whole waves leave together
  // 16-byte loads (two amplitudes per lane), several in flight: the sum
  // order per lane stays fixed (cbits >= 1, so a chunk is whole elements)
  const uint64_t len4 = (uint64_t)1 << (cbits - 1 - bbits);  // elements of a part
  const float4* __restrict__ p = reinterpret_cast<const float4*>(psi + (ch << cbits));
  double total = 0.0;
  for (int b = 0; b < 1 << bbits; ++b, p += len4) {
    double v = 0.0;
#pragma unroll 4
    for (uint64_t i = lane; i < len4; i += 64) {
      const float4 a = gld<NT>(p + i);
      v += sq(make_float2(a.x, a.y));
      v += sq(make_float2(a.z, a.w));
    }
    v = wave_sum(v);
    if (lane == 0) parts[(ch << bbits) + b] = v;
    total += v;
  }
  if (lane == 0) sums[ch] = total;
}

constexpr int kScanPer = 8;                       // elements per thread
constexpr int kScanBlock = kThreads * kScanPer;   // 2048 elements per block

__device__ double block_exclusive_scan(double v, double* total) {
  __shared__ double wsum[kThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  double off = 0.0, all = 0.0;
  for (int i = 0; i < kThreads / 64; ++i) {
    if (i < w) off += wsum[i];
    all += wsum[i];
  }
  __syncthreads();
  *total = all;
  return off + x - v;
}

// In place: inclusive prefix within each block of kScanBlock; block totals out.
__global__ __launch_bounds__(kThreads) void k_scan_blocks(double* __restrict__ x, uint64_t count,
                                                         double* __restrict__ totals) {
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanPer;
  double loc[kScanPer];
  double run = 0.0;
#pragma unroll
  for (int e = 0; e < kScanPer; ++e) {
    loc[e] = base + e < count ? x[base + e] : 0.0;
    run += loc[e];
    loc[e] = run;
  }
  double total;
  const double off = block_exclusive_scan(run, &total);
#pragma unroll
  for (int e = 0; e < kScanPer; ++e)
    if (base + e < count) x[base + e] = off + loc[e];
  if (threadIdx.x == 0 && totals) totals[blockIdx.x] = total;
}

__global__ __launch_bounds__(kThreads) void k_scan_add(double* __restrict__ x, uint64_t count,
                                                      const double* __restrict__ incl_totals) {
  if (blockIdx.x == 0) return;
  const double off = incl_totals[blockIdx.x - 1];
  const uint64_t base = (uint64_t)blockIdx.x * kScanBlock;
  for (int e = threadIdx.x; e < kScanBlock; e += kThreads)
    if (base + e < count) x[base + e] += off;
}

constexpr uint64_t kNoSample = ~(uint64_t)0;

__device__ __forceinline__ double wave_inclusive(double x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// The chunk of every shot, one thread each: the first with incl > target (or,
// past the end, the first reaching total).
__global__ __launch_bounds__(kThreads) void k_find_chunks(const double* __restrict__ incl, uint64_t nchunks,
                                                         const double* __restrict__ u, uint64_t shots,
                                                         uint64_t* __restrict__ out) {
  const uint64_t shot = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (shot >= shots) return;
  const double total = incl[nchunks - 1];
  if (!(total > 0.0)) {
    out[shot] = kNoSample;
    return;
  }
  const double target = u[shot] * total;
  const bool past_end = !(target < total);
  uint64_t lo = 0, hi = nchunks - 1;
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo) / 2;
    const bool go_left = past_end ? !(incl[mid] < total) : incl[mid] > target;
    if (go_left) hi = mid;
    else lo = mid + 1;
  }
  out[shot] = lo;
}

// in: out[shot] is the shot's chunk; out: the amplitude it picks in it
__global__ __launch_bounds__(kThreads) void k_sample(const float2* __restrict__ psi, int cbits, int bbits,
                                                    const double* __restrict__ incl, const double* __restrict__ parts,
                                                    uint64_t nchunks, const double* __restrict__ u, uint64_t shots,
                                                    uint64_t* __restrict__ out) {
  const uint64_t shot = ((uint64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (shot >= shots) return;  // whole waves leave together
  const uint64_t ch = out[shot];
  if (ch == kNoSample) return;
  const double total = incl[nchunks - 1];
  const double target = u[shot] * total;
  const bool past_end = !(target < total);
  // what is left of the target inside the chunk; past the end nothing crosses
  // and the last amplitude with p > 0 is taken
  double r = target - (ch > 0 ? incl[ch - 1] : 0.0);
  const int nparts = 1 << bbits;
  double v = lane < nparts ? parts[(ch << bbits) + lane] : 0.0;
  double x = wave_inclusive(v, lane);
  uint64_t cross = __ballot(!past_end && x > r && v > 0.0);
  uint64_t nz = __ballot(v > 0.0);
  if (!nz) {
    if (lane == 0) out[shot] = kNoSample;
    return;
  }
  const bool last_part = !cross;
  const int part = cross ? __ffsll((long long)cross) - 1 : 63 - __clzll(nz);
  r -= __shfl(x - v, part, 64);
  const uint64_t len = (uint64_t)1 << (cbits - bbits);
  const uint64_t base = (ch << cbits) + (uint64_t)part * len;
  double acc = 0.0;
  uint64_t last_nz = kNoSample, found = kNoSample;
  for (uint64_t s = 0; s < len && found == kNoSample; s += 512) {
    double p[8];
    v = 0.0;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {  // 16-byte loads; a part is whole elements
      const uint64_t i = s + (uint64_t)lane * 8 + e;
      const float4 a = i < len ? *reinterpret_cast<const float4*>(psi + base + i) : make_float4(0.f, 0.f, 0.f, 0.f);
      p[e] = sq(make_float2(a.x, a.y));
      p[e + 1] = sq(make_float2(a.z, a.w));
      v += p[e];
      v += p[e + 1];
    }
    x = wave_inclusive(v, lane);
    cross = __ballot(!past_end && !last_part && acc + x > r && v > 0.0);
    nz = __ballot(v > 0.0);
    const int owner = cross ? __ffsll((long long)cross) - 1 : nz ? 63 - __clzll(nz) : -1;
    if (owner >= 0) {
      // the owner lane walks its eight amplitudes
      const double before = acc + (x - v);
      double run = 0.0;
      int hit = -1, last = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        run += p[e];
        if (p[e] > 0.0) {
          last = e;
          if (hit < 0 && before + run > r) hit = e;
        }
      }
      const int pick = __shfl(cross && hit >= 0 ? hit : last, owner, 64);
      const uint64_t i = base + s + (uint64_t)owner * 8 + pick;
      if (cross) found = i;
      else last_nz = i;
    }
    acc += __shfl(x, 63, 64);
  }
  if (lane == 0) out[shot] = found != kNoSample ? found : last_nz;
}

unsigned blocks_for(uint64_t items, uint64_t per_thread) {
  uint64_t b = (items + kThreads * per_thread - 1) / (kThreads * per_thread);
  if (b > (uint64_t)kMaxBlocks) b = kMaxBlocks;
  return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

namespace {
// one class of sweeps (all of at most TERMS terms): partials of sweep i at
// (first + i) * blocks * kTerms
template <int TERMS>
void pauli_class(const void* psi, int n, const PauliSweep* sweeps, const std::vector<int>& which, int first,
                 unsigned blocks, unsigned groups, double* partials, hipStream_t st) {
  if (n >= kern::kNtMinQubits) {  // streamed: a launch per sweep, each bound by memory
    for (size_t i = 0; i < which.size(); ++i) {
      PauliArgs a{};
      const int mode = pauli_args<TERMS>(a, n, sweeps[which[i]].f, sweeps[which[i]].z);
      auto* kernel = mode == 0 ? k_pauli_chunks<0, TERMS> : mode == 1 ? k_pauli_chunks<1, TERMS> : k_pauli_chunks<2, TERMS>;
      hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), 0, st, (const float4*)psi, a,
                         partials + (first + i) * blocks * kTerms);
    }
    return;
  }
  for (size_t i0 = 0; i0 < which.size(); i0 += PauliSweeps<TERMS>::kMax) {
    PauliSweeps<TERMS> s;
    const size_t m = std::min(which.size() - i0, (size_t)PauliSweeps<TERMS>::kMax);
    for (size_t i = 0; i < m; ++i) {
      s.f[i] = sweeps[which[i0 + i]].f;
      std::copy(sweeps[which[i0 + i]].z, sweeps[which[i0 + i]].z + TERMS, s.z[i]);
    }
    hipLaunchKernelGGL(k_pauli_sweeps<TERMS>, dim3(groups, (unsigned)m), dim3(kThreads), 0, st, (const float4*)psi, n,
                       s, first + (int)i0, blocks, partials);
  }
}
}  // namespace

// Blocks of a sweep's walk.  Streamed states: all that are resident, each wave
// walking whole chunks.  Cached ones: a power of two (the walk's split of signs
// needs it) of at least 4 items a thread up to 256 blocks, 16 up to 512 and 32
// beyond: a call of one sweep wants many blocks, one of many sweeps few
// reductions (us a call of one term / 8 diagonal terms / an Ising
// Hamiltonian, with 256, 512, 1024 blocks: 22 qubits 24 / 31 / 76, 24 / 29 / 84,
// 24 / 29 / 89; 24 qubits 45 / 70 / 350, 40 / 51 / 336, 40 / 44 / 356).
static unsigned pauli_blocks(int n) {
  if (n >= kern::kNtMinQubits) return kMaxBlocks;
  unsigned b = 1;
  const uint64_t items = n > 1 ? (uint64_t)1 << (n - 2) : 1;
  while ((uint64_t)b * 2 * kThreads * (b < 256 ? 4 : b < 512 ? 16 : 32) <= items) b *= 2;
  return b;
}
// Sweeps that share the partials' scratch: 8 MiB of it, 256 at most.
static size_t pauli_group(int n) {
  return std::min<size_t>(256, ((size_t)8 << 20) / (sizeof(double) * kTerms * pauli_blocks(n)));
}
size_t pauli_scratch_bytes(int n, size_t sweeps) {
  return sizeof(double) * kTerms * std::min(sweeps, pauli_group(n)) * pauli_blocks(n);
}

// Sums of every sweep: out[8 w + t] = sum over pairs (or amplitudes) of term t
// of sweep order[w].  `order` receives the sweeps' order.
void launch_pauli(const void* psi, int n, const std::vector<PauliSweep>& sweeps, std::vector<int>& order,
                  double* scratch, double* out, hipStream_t st) {
  if (n < 1) throw DeviceError{hipErrorInvalidValue, "k_pauli: n"};
  const unsigned blocks = pauli_blocks(n);
  order.clear();
  for (size_t w0 = 0; w0 < sweeps.size(); w0 += pauli_group(n)) {
    const size_t count = std::min(pauli_group(n), sweeps.size() - w0);
    // Workgroups of a launch of several sweeps: up to 22 qubits the state stays
    // in the L2s whatever the order; above, sweeps that are resident together
    // read the same part of it at the same time (24 masks at 24 qubits: 336 us
    // with 4096 workgroups, 446 with 8192; 22 masks at 22: 86 and 75).
    const size_t resident = n <= 22 ? 8192 : 4096;
    unsigned groups = blocks;
    while (n < kern::kNtMinQubits && groups > 1 && groups * count > resident) groups /= 2;
    std::vector<int> cls[4];
    for (size_t w = 0; w < count; ++w) {
      const PauliSweep& s = sweeps[w0 + w];
      if (s.terms < 1 || s.terms > kTerms) throw DeviceError{hipErrorInvalidValue, "k_pauli: 1..8 terms per sweep"};
      if (n < 64 && (s.f >> n) != 0) throw DeviceError{hipErrorInvalidValue, "k_pauli: flip mask past n"};
      cls[s.terms <= 1 ? 0 : s.terms <= 2 ? 1 : s.terms <= 4 ? 2 : 3].push_back((int)w);
    }
    int first = 0;
    for (int c = 0; c < 4; ++c) {
      const PauliSweep* g = sweeps.data() + w0;
      if (c == 0) pauli_class<1>(psi, n, g, cls[c], first, blocks, groups, scratch, st);
      else if (c == 1) pauli_class<2>(psi, n, g, cls[c], first, blocks, groups, scratch, st);
      else if (c == 2) pauli_class<4>(psi, n, g, cls[c], first, blocks, groups, scratch, st);
      else pauli_class<8>(psi, n, g, cls[c], first, blocks, groups, scratch, st);
      for (int w : cls[c]) order.push_back((int)w0 + w);
      first += (int)cls[c].size();
    }
    hipLaunchKernelGGL(k_pauli_final, dim3((unsigned)count), dim3(kFinalRows * kTerms), 0, st, (const double*)scratch,
                       (int)blocks, out + kTerms * w0);
  }
  SV_HIP(hipGetLastError());
}

int marginal_max_qubits() { return kMaxMeasured; }
size_t marginal_scratch_bytes(int m) { return sizeof(double) * (size_t)kMaxBlocks << m; }

void launch_marginal(const void* psi, int n, int m, const int* qubits, double* scratch, double* out,
                     hipStream_t st) {
  if (m < 1 || m > kMaxMeasured || m > n) throw DeviceError{hipErrorInvalidValue, "k_marginal: bad m"};
  MargArgs a{};
  a.len = (uint64_t)1 << n;
  const int cbits = n > 6 ? n - 6 : 0;
  a.nchunks = (uint64_t)1 << cbits;
  a.m = m;
  for (int j = 0; j < m; ++j) {
    if (qubits[j] < 0 || qubits[j] >= n) throw DeviceError{hipErrorInvalidValue, "k_marginal: qubit past n"};
    a.q[j] = qubits[j];
    if (qubits[j] < 6) a.low_meas |= 1u << qubits[j];
    else a.hc |= (uint64_t)1 << (qubits[j] - 6);
  }
  a.fc = (a.nchunks - 1) & ~a.hc;
  a.free_bits = __builtin_popcountll(a.fc);
  const unsigned blocks = blocks_for(a.nchunks * 64, 16);
  const int M = 1 << m;
  if (n >= kern::kNtMinQubits)
    hipLaunchKernelGGL(k_marginal_partial<true>, dim3(blocks), dim3(kThreads), sizeof(double) * 4 * M, st,
                       (const float2*)psi, a, scratch);
  else
    hipLaunchKernelGGL(k_marginal_partial<false>, dim3(blocks), dim3(kThreads), sizeof(double) * 4 * M, st,
                       (const float2*)psi, a, scratch);
  hipLaunchKernelGGL(k_column_sums, dim3((M + 63) / 64), dim3(64 * kFinalWaves), 0, st, (const double*)scratch,
                     (int)blocks, M, out);
  SV_HIP(hipGetLastError());
}

// Chunk size 2^c: 4096 amplitudes, or larger so that at most 2^22 chunks
// (2048 scan blocks) exist.
int sample_chunk_bits(int n) {
  int c = n < 12 ? n : 12;
  if (n - c > 22) c = n - 22;
  return c;
}
// Parts of a chunk, 2^b of at least 512 amplitudes: one load and scan finds
// the part.
int sample_part_bits(int n) {
  const int c = sample_chunk_bits(n);
  return c <= 9 ? 0 : c - 9 < 3 ? c - 9 : 3;
}
size_t sample_scratch_bytes(int n) {
  const uint64_t nchunks = (uint64_t)1 << (n - sample_chunk_bits(n));
  return sizeof(double) * (nchunks + kMaxBlocks + (nchunks << sample_part_bits(n)));
}

// prepare: build the chunk prefix sums in scratch (needed once per state);
// then draw `shots` samples.  uniforms / out: device arrays of `shots`; out
// gets all ones for a zero state.
void launch_sample(const void* psi, int n, bool prepare, const double* uniforms, uint64_t shots, uint64_t* out,
                   double* scratch, hipStream_t st) {
  const int c = sample_chunk_bits(n);
  if (c < 1) throw DeviceError{hipErrorInvalidValue, "k_sample: a chunk must hold whole 16-byte elements"};
  const uint64_t nchunks = (uint64_t)1 << (n - c);
  const int b = sample_part_bits(n);
  double* incl = scratch;
  double* totals = scratch + nchunks;
  double* parts = totals + kMaxBlocks;
  if (prepare) {
    const uint64_t waves_blocks = (nchunks * 64 + kThreads - 1) / kThreads;
    if (n >= kern::kNtMinQubits)
      hipLaunchKernelGGL(k_chunk_sums<true>, dim3((unsigned)waves_blocks), dim3(kThreads), 0, st,
                         (const float2*)psi, c, b, nchunks, incl, parts);
    else
      hipLaunchKernelGGL(k_chunk_sums<false>, dim3((unsigned)waves_blocks), dim3(kThreads), 0, st,
                         (const float2*)psi, c, b, nchunks, incl, parts);
    const uint64_t sblocks = (nchunks + kScanBlock - 1) / kScanBlock;
    if (sblocks > (uint64_t)kScanBlock) throw DeviceError{hipErrorInvalidValue, "k_sample: too many chunks"};
    hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)sblocks), dim3(kThreads), 0, st, incl, nchunks, totals);
    if (sblocks > 1) {
      hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(kThreads), 0, st, totals, sblocks, (double*)nullptr);
      hipLaunchKernelGGL(k_scan_add, dim3((unsigned)sblocks), dim3(kThreads), 0, st, incl, nchunks,
                         (const double*)totals);
    }
  }
  if (shots) {
    hipLaunchKernelGGL(k_find_chunks, dim3((unsigned)((shots + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       (const double*)incl, nchunks, uniforms, shots, out);
    const uint64_t blocks = (shots * 64 + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(k_sample, dim3((unsigned)blocks), dim3(kThreads), 0, st, (const float2*)psi, c, b,
                       (const double*)incl, (const double*)parts, nchunks, uniforms, shots, out);
  }
  SV_HIP(hipGetLastError());
}

}  // namespace sv
