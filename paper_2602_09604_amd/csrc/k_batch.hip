// Batched simulation of many independent small circuits.
//
// Every circuit of at least 8 qubits runs as tile sweeps (sweep.h): launch L
// covers sweep L of every circuit that has one, each workgroup walking tiles
// of one circuit, so the grid is filled by the whole batch instead of by one
// state.  The kernel boundary is the barrier between dependent sweeps of a
// circuit (it also makes every XCD's writes visible to the next sweep without
// spinning on device flags).  A state of up to 12 qubits is one tile, and its
// sweeps take as many passes as their matrices fit in LDS.
// k_batch_lds runs the circuits no tile takes (fewer than 8 qubits, or a gate
// too wide for the tile of an 8- or 9-qubit state): one workgroup per circuit
// loads the state into LDS once, applies every fused pass and stores it once.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <exception>
#include <thread>
#include <cstring>

#include <stdexcept>

#include "k_common.h"
#include "sweep.h"

namespace sv {

void* state_psi(sv_state* s);
int state_n(sv_state* s);
hipStream_t state_stream(sv_state* s);
int state_device(sv_state* s);
bool state_poisoned(sv_state* s);
void state_poison(sv_state* s);
void state_staging(sv_state* s, size_t bytes, unsigned char** host, unsigned char** dev);
void state_staging_trim(sv_state* s, size_t keep);
void state_note_gates(sv_state* s, const sv_gate* g, size_t n);

namespace {
using namespace kern;

// One fused pass of one circuit, in element space (see k_apply_reg modes).
struct BPass {
  uint64_t items;             // lane work items
  uint64_t lowmask[SV_MAX_K];
  uint64_t stride[SV_MAX_K];
  uint32_t mat;               // float2 index of the complex64 matrix
  int mode, K;
};

struct BCirc {
  float2* psi;
  int n;
  int pass0, npass;
};

template <int K, int MODE, typename PTR2, typename PTR4>
__device__ __forceinline__ void apply_item(PTR2 psi2, PTR4 psi4, const float2* __restrict__ U, const BPass& p,
                                           uint64_t g) {
  constexpr int D = 1 << K;
  uint64_t base = g;
#pragma unroll
  for (int j = 0; j < K; ++j) base = ((base & ~p.lowmask[j]) << 1) | (base & p.lowmask[j]);
  if constexpr (MODE == 2) {
    float2 v[D];
#pragma unroll
    for (int l = 0; l < D; ++l) v[l] = psi2[base + local_offset<K, uint64_t>(l, p.stride)];
#pragma unroll
    for (int r = 0; r < D; ++r) {
      float2 acc = make_float2(0.f, 0.f);
#pragma unroll
      for (int c = 0; c < D; ++c) cmac(acc, U[r * D + c], v[c]);
      psi2[base + local_offset<K, uint64_t>(r, p.stride)] = acc;
    }
  } else {
    float4 v[D];
#pragma unroll
    for (int l = 0; l < D; ++l) v[l] = psi4[base + local_offset<K, uint64_t>(l, p.stride)];
#pragma unroll
    for (int r = 0; r < D; ++r)
      psi4[base + local_offset<K, uint64_t>(r, p.stride)] = pair_row<K, MODE>(v, U, r);
  }
}

// Dispatch on the pass shape (uniform across the workgroup).
template <typename PTR2, typename PTR4>
__device__ void apply_dispatch(PTR2 psi2, PTR4 psi4, const float2* __restrict__ U, const BPass& p, uint64_t g) {
  switch (p.mode * 8 + p.K) {
    case 0 * 8 + 1: apply_item<1, 0>(psi2, psi4, U, p, g); break;
    case 0 * 8 + 2: apply_item<2, 0>(psi2, psi4, U, p, g); break;
    case 0 * 8 + 3: apply_item<3, 0>(psi2, psi4, U, p, g); break;
    case 0 * 8 + 4: apply_item<4, 0>(psi2, psi4, U, p, g); break;
    case 0 * 8 + 5: apply_item<5, 0>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 0: apply_item<0, 1>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 1: apply_item<1, 1>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 2: apply_item<2, 1>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 3: apply_item<3, 1>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 4: apply_item<4, 1>(psi2, psi4, U, p, g); break;
    case 1 * 8 + 5: apply_item<5, 1>(psi2, psi4, U, p, g); break;
    case 2 * 8 + 6: apply_item<6, 2>(psi2, psi4, U, p, g); break;
    default: break;  // shapes are checked on the host
  }
}

// One workgroup per circuit.
__global__ __launch_bounds__(256) void k_batch_lds(const BCirc* __restrict__ circs, const BPass* __restrict__ passes,
                                                   const float2* __restrict__ mats) {
  extern __shared__ float4 st4[];
  float2* st2 = reinterpret_cast<float2*>(st4);
  const BCirc c = circs[blockIdx.x];
  const int pairs = 1 << (c.n - 1);
  float4* g4 = reinterpret_cast<float4*>(c.psi);
  for (int i = threadIdx.x; i < pairs; i += 256) st4[i] = g4[i];
  __syncthreads();
  for (int pi = 0; pi < c.npass; ++pi) {
    const BPass p = passes[c.pass0 + pi];
    for (uint64_t g = threadIdx.x; g < p.items; g += 256) apply_dispatch(st2, st4, mats + p.mat, p, g);
    __syncthreads();
  }
  for (int i = threadIdx.x; i < pairs; i += 256) g4[i] = st4[i];
}

bool shape_supported(int mode, int K) {
  return (mode == 0 && K >= 1 && K <= 5) || (mode == 1 && K >= 0 && K <= 5) || (mode == 2 && K == 6);
}

constexpr int kBatchTileBits = 12;
constexpr int kBatchAloneQubits = 9;     // circuits k_batch_lds may run
constexpr uint64_t kBatchGroups = 256;   // workgroups per state in a launch
// Staging that stays with the first handle: 512 circuits of 10 to 22 qubits take
// a ring of 64 MiB, which costs about 1 ms to allocate anew.
constexpr size_t kBatchKeepBytes = (size_t)64 << 20;

void fill_pass(BPass& bp, int n, const FusedGate& f, uint32_t mat) {
  int pos[SV_MAX_K];
  if (f.q[0] == 0) {
    bp.mode = 1;
    bp.K = f.k - 1;
    for (int j = 0; j < bp.K; ++j) pos[j] = f.q[j + 1] - 1;
    bp.items = (uint64_t)1 << (n - 1 - bp.K);
  } else if (f.k <= 5) {
    bp.mode = 0;
    bp.K = f.k;
    for (int j = 0; j < bp.K; ++j) pos[j] = f.q[j] - 1;
    bp.items = (uint64_t)1 << (n - 1 - bp.K);
  } else {
    bp.mode = 2;
    bp.K = f.k;
    for (int j = 0; j < bp.K; ++j) pos[j] = f.q[j];
    bp.items = (uint64_t)1 << (n - bp.K);
  }
  for (int j = 0; j < SV_MAX_K; ++j) {
    bp.lowmask[j] = j < bp.K ? ((uint64_t)1 << pos[j]) - 1 : 0;
    bp.stride[j] = j < bp.K ? (uint64_t)1 << pos[j] : 0;
  }
  bp.mat = mat;
}

}  // namespace

int plan_fusion(const sv_gate* g, size_t n, int n_qubits, const sv_run_opts& o, std::vector<FusedGate>& fused,
                std::vector<int32_t>& block_of, int max_ctrl);

namespace {
// What one circuit runs as: its sweeps, or (whole) its passes in k_batch_lds.
struct CircPlan {
  std::vector<FusedGate> fused;
  std::vector<Pass> passes;
  std::vector<Sweep> sweeps;
  std::vector<size_t> off;  // data of each sweep, from the start of the circuit's data
  size_t bytes = 0;
  bool whole = false;
};

void plan_circuit(const sv_gate* g, size_t ng, int n, const sv_run_opts& o, CircPlan& c) {
  std::vector<int32_t> block_of;
  plan_fusion(g, ng, n, o, c.fused, block_of, 0);  // batched passes take no controls
  const int T = std::min(n, kBatchTileBits);
  std::vector<SweepItem> items(c.fused.size());
  c.passes.resize(c.fused.size());
  for (size_t i = 0; i < c.fused.size(); ++i) {
    const FusedGate& f = c.fused[i];
    if (f.cmask)
      throw std::invalid_argument("sv_batch_run: a controlled gate wider than max_k qubits (targets plus "
                                  "controls) cannot run in the batched kernel");
    c.passes[i].k = f.k;
    std::copy(f.q, f.q + f.k, c.passes[i].s);
    for (int j = 0; j < f.k; ++j) items[i].mask |= (uint64_t)1 << f.q[j];
    items[i].kind = sweep_kind(T, f.k, SV_PREC_FP32_VALU);
    if (!items[i].kind) c.whole = true;
  }
  if (c.whole) return;
  plan_sweeps(items, n, T, sweep_mat_room(SV_MAX_QUBITS, T, SV_PREC_FP32_VALU), SV_PREC_FP32_VALU, c.sweeps);
  for (Sweep& s : c.sweeps) {
    c.off.push_back(c.bytes);
    c.bytes += (s.data_bytes + 255) / 256 * 256;
  }
}

void encode_circuit(const CircPlan& c, unsigned char* dst) {
  std::vector<const Pass*> ps;
  std::vector<const double*> ms;
  for (size_t i = 0; i < c.sweeps.size(); ++i) {
    ps.clear();
    ms.clear();
    for (int m : c.sweeps[i].members) {
      ps.push_back(&c.passes[m]);
      ms.push_back(c.fused[m].mat.data());
    }
    encode_sweep(c.sweeps[i], ps, ms, dst + c.off[i]);
  }
}

// body(c) for every circuit on host threads
template <class F>
void for_circuits(size_t n_circ, F&& body) {
  const unsigned hw = std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
  const unsigned nt = (unsigned)std::min<size_t>(hw, std::max<size_t>(1, n_circ / 2));
  std::atomic<size_t> next{0};
  std::vector<std::exception_ptr> errs(nt);
  auto worker = [&](unsigned w) {
    set_host_pool_worker(true);
    struct Reset {
      ~Reset() { set_host_pool_worker(false); }
    } reset;
    try {
      for (size_t c = next++; c < n_circ; c = next++) body(c);
    } catch (...) {
      errs[w] = std::current_exception();
      next = n_circ;
    }
  };
  std::vector<std::thread> pool;
  for (unsigned w = 1; w < nt; ++w) pool.emplace_back(worker, w);
  worker(0);
  for (auto& t : pool) t.join();
  for (auto& e : errs)
    if (e) std::rethrow_exception(e);
}

struct BatchOut {
  double gpu_s = 0, fuse_s = 0;
  uint64_t passes = 0, bytes = 0, launches = 0;
};

BatchOut batch_run_impl(sv_state* const* states, const int* ns, const sv_gate* const* circuits, const size_t* n_gates,
                        size_t n_circ, const sv_run_opts& o) {
  BatchOut out;
  const auto t0 = std::chrono::steady_clock::now();
  std::vector<CircPlan> plans(n_circ);
  for_circuits(n_circ, [&](size_t c) { plan_circuit(circuits[c], n_gates[c], ns[c], o, plans[c]); });
  out.fuse_s = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();

  // circuits of k_batch_lds: tables and matrices
  std::vector<BCirc> alone;
  std::vector<BPass> passes;
  std::vector<float> mats;  // complex64, interleaved
  int alone_n = 1;
  // launch L: sweep L of every circuit that has one
  struct Level {
    std::vector<BatchSweep> table;
    uint64_t groups = 0;
    size_t lds = 0, at = 0;
  };
  std::vector<Level> levels;
  std::vector<size_t> data_off(n_circ, 0);
  size_t data = 0, table_bytes = 0;
  uint64_t state_bytes = 0;
  for (size_t c = 0; c < n_circ; ++c) {
    const CircPlan& pl = plans[c];
    out.passes += pl.fused.size();
    out.bytes += ((uint64_t)16 << ns[c]) * pl.fused.size();
    if (pl.whole) {
      if (ns[c] > kBatchAloneQubits) throw DeviceError{hipErrorInvalidValue, "batch: a pass no tile takes"};
      alone.push_back(BCirc{(float2*)state_psi(states[c]), ns[c], (int)passes.size(), (int)pl.fused.size()});
      alone_n = std::max(alone_n, ns[c]);
      for (const FusedGate& f : pl.fused) {
        BPass bp{};
        fill_pass(bp, ns[c], f, (uint32_t)(mats.size() / 2));
        if (!shape_supported(bp.mode, bp.K)) throw std::invalid_argument("sv_batch_run: unsupported pass shape");
        passes.push_back(bp);
        for (double v : f.mat) mats.push_back((float)v);
      }
      continue;
    }
    state_bytes += (uint64_t)8 << ns[c];
    data_off[c] = data;
    data += pl.bytes;
    for (size_t L = 0; L < pl.sweeps.size(); ++L) {
      const Sweep& sw = pl.sweeps[L];
      if (L >= levels.size()) levels.emplace_back();
      Level& l = levels[L];
      BatchSweep e{};
      e.psi = (float4*)state_psi(states[c]);
      e.data = data_off[c] + pl.off[L];
      e.args = sweep_args(sw, ns[c]);
      e.T = sw.T;
      e.first = (uint32_t)l.groups;
      e.groups = (uint32_t)std::min(e.args.tiles, kBatchGroups);
      l.groups += e.groups;
      l.lds = std::max(l.lds, ((size_t)8 << sw.T) + sw.mat_bytes);
      l.table.push_back(e);
      table_bytes += sizeof(BatchSweep);
    }
  }
  // one staging area: sweep data | sweep tables | k_batch_lds circuits, passes, matrices
  auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const size_t off_table = al(data);
  const size_t off_circ = al(off_table + table_bytes);
  const size_t off_pass = al(off_circ + sizeof(BCirc) * alone.size());
  const size_t off_mat = al(off_pass + sizeof(BPass) * passes.size());
  const size_t total = al(off_mat + sizeof(float) * mats.size());
  if (levels.empty() && alone.empty()) {  // nothing to launch, but the handles' queued work is waited for
    SV_HIP(hipStreamSynchronize(state_stream(states[0])));
    return out;
  }
  unsigned char *host = nullptr, *dev = nullptr;
  state_staging(states[0], total, &host, &dev);
  for_circuits(n_circ, [&](size_t c) {
    if (!plans[c].whole) encode_circuit(plans[c], host + data_off[c]);
  });
  size_t at = off_table;
  for (Level& l : levels) {
    l.at = at;
    std::memcpy(host + at, l.table.data(), sizeof(BatchSweep) * l.table.size());
    at += sizeof(BatchSweep) * l.table.size();
  }
  if (!alone.empty()) {
    std::memcpy(host + off_circ, alone.data(), sizeof(BCirc) * alone.size());
    std::memcpy(host + off_pass, passes.data(), sizeof(BPass) * passes.size());
    std::memcpy(host + off_mat, mats.data(), sizeof(float) * mats.size());
  }
  const hipStream_t st = state_stream(states[0]);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  struct Events {
    hipEvent_t &a, &b;
    ~Events() {
      if (a) (void)hipEventDestroy(a);
      if (b) (void)hipEventDestroy(b);
    }
  } events{e0, e1};
  SV_HIP(hipEventCreate(&e0));
  SV_HIP(hipEventCreate(&e1));
  SV_HIP(hipMemcpyAsync(dev, host, total, hipMemcpyHostToDevice, st));
  SV_HIP(hipEventRecord(e0, st));
  if (!alone.empty()) {
    hipLaunchKernelGGL(k_batch_lds, dim3((unsigned)alone.size()), dim3(256), (size_t)8 << alone_n, st,
                       (const BCirc*)(dev + off_circ), (const BPass*)(dev + off_pass), (const float2*)(dev + off_mat));
    SV_HIP(hipGetLastError());
    ++out.launches;
  }
  const bool nt = state_bytes >= ((uint64_t)8 << kNtMinQubits);  // the states exceed the last-level cache
  for (const Level& l : levels) {
    if (l.groups >= ((uint64_t)1 << 31)) throw DeviceError{hipErrorInvalidValue, "batch level too large"};
    launch_sweep_batch((const BatchSweep*)(dev + l.at), (int)l.table.size(), (unsigned)l.groups, l.lds, nt, dev, st);
    ++out.launches;
  }
  SV_HIP(hipEventRecord(e1, st));
  SV_HIP(hipStreamSynchronize(st));
  float ms = 0.f;
  SV_HIP(hipEventElapsedTime(&ms, e0, e1));
  out.gpu_s = ms * 1e-3;
  state_staging_trim(states[0], kBatchKeepBytes);
  return out;
}
}  // namespace

int validate_gates(const sv_gate* g, size_t n, int n_qubits);

}  // namespace sv

using namespace sv;

extern "C" int sv_batch_run(sv_state* const* states, const sv_gate* const* circuits, const size_t* n_gates,
                            size_t n_circuits, const sv_run_opts* opts, sv_run_stats* stats) {
  if (n_circuits == 0) return SV_OK;
  if (!states || !circuits || !n_gates) return fail(SV_EINVAL, "NULL argument");
  sv_run_opts o{};
  if (opts) {
    o = *opts;
  } else {
    o.max_k = 4;
    o.fusion = SV_FUSE_GREEDY;
  }
  if (o.fusion < SV_FUSE_NONE || o.fusion > SV_FUSE_BLOCK || (o.fusion != SV_FUSE_NONE && (o.max_k < 1 || o.max_k > SV_MAX_K)))
    return fail(SV_EINVAL, "opts invalid");
  std::vector<int> ns(n_circuits);
  for (size_t c = 0; c < n_circuits; ++c) {
    if (!states[c]) return fail(SV_EINVAL, "states[" + std::to_string(c) + "] is NULL");
    if (state_poisoned(states[c])) return fail(SV_ESTATE, "a handle is poisoned");
    ns[c] = state_n(states[c]);
    if (ns[c] > 30) return fail(SV_EINVAL, "batched circuits are limited to 30 qubits");
    if (int rc = validate_gates(circuits[c], n_gates[c], ns[c])) return rc;
  }
  // batched passes multiply in FP32, whatever the options say
  o.precision = SV_PREC_FP32_VALU;
  std::vector<hipEvent_t> waits;
  try {
    SV_HIP(hipSetDevice(state_device(states[0])));  // its staging ring outlives the call
    // work already queued on the other handles' streams (initialisation,
    // earlier passes) must finish before the batch touches their states
    const hipStream_t st0 = state_stream(states[0]);
    std::vector<hipStream_t> seen{st0};
    for (size_t c = 1; c < n_circuits; ++c) {
      const hipStream_t sc = state_stream(states[c]);
      if (std::find(seen.begin(), seen.end(), sc) != seen.end()) continue;
      seen.push_back(sc);
      hipEvent_t ev = nullptr;
      SV_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
      waits.push_back(ev);
      SV_HIP(hipEventRecord(ev, sc));
      SV_HIP(hipStreamWaitEvent(st0, ev, 0));
    }
    const BatchOut out = batch_run_impl(states, ns.data(), circuits, n_gates, n_circuits, o);
    for (hipEvent_t ev : waits) (void)hipEventDestroy(ev);
    waits.clear();
    for (size_t c = 0; c < n_circuits; ++c) state_note_gates(states[c], circuits[c], n_gates[c]);
    if (stats) {
      *stats = sv_run_stats{};
      uint64_t gi = 0;
      for (size_t c = 0; c < n_circuits; ++c) gi += n_gates[c];
      stats->gates_in = gi;
      stats->passes = out.passes;
      stats->gpu_s = out.gpu_s;
      stats->fuse_s = out.fuse_s;
      stats->bytes = out.bytes;
      stats->launches = out.launches;
    }
    return SV_OK;
  } catch (const DeviceError& e) {
    for (hipEvent_t ev : waits) (void)hipEventDestroy(ev);
    for (size_t c = 0; c < n_circuits; ++c) state_poison(states[c]);
    return fail(SV_EDEVICE, std::string(e.what) + ": " + hipGetErrorString(e.err));
  } catch (const std::bad_alloc&) {
    for (hipEvent_t ev : waits) (void)hipEventDestroy(ev);
    return fail(SV_ENOMEM, "host allocation failed");
  } catch (const std::exception& e) {
    for (hipEvent_t ev : waits) (void)hipEventDestroy(ev);
    return fail(SV_EINVAL, e.what());
  } catch (...) {
    for (hipEvent_t ev : waits) (void)hipEventDestroy(ev);
    return fail(SV_EINVAL, "unknown failure");
  }
}
