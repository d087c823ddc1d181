// Routing-aware adaptive speculative expansion (Sec. "Routing-aware Adaptive
// Speculative Expansion"): best-first selection of draft-tree tokens by the
// utility U_i = p_i T_AR / (|E_i \ U| T_exp + C_i^draft) while U_i >= 1.
//
// One workgroup of 256 threads per tree.  U only grows and U_i falls with
// |E_i \ U|, so a node with p_i T_AR / C_i^draft < 1, and every node below it,
// can never be selected: only the others ("viable", in index order: slots)
// take part, and only their ids are read.  In LDS, E rounded up to a power of
// two >= 32 is EW words:
//   pv[i]            p_i (0 for nodes that are not viable), later pv[slot] =
//                    p T_AR;  cdr[slot] = C^draft
//   rows[slot][l][w] the experts the slot's node is predicted to use at layer l
//   uni[l][w]        the union U of the selected tokens' (layer, expert) pairs,
//                    a copy per wave or one for all
// so that repeated ids collapse by themselves, |E_i \ U| is
// sum_l popcount(rows[i][l] & ~uni[l]) and U grows by a word-wise OR.
// Phases: (1) per-node validity and the root's experts into U; (2) prefix
// confidences and viability; (3) slots; (4) the slots' ids -> bitsets; (5) the
// greedy loop: each wave lists and scores the candidates among its own slots
// (those v with v % 4 = wave, so that siblings spread over the waves), each
// 16-lane row of it one at a time; the block takes the largest U_i (ties:
// smaller index) and, if U_i >= 1, adds the node's experts to U.  With a copy
// of U per wave a step has one workgroup barrier, with a single U two.
//
// What bounds it is each tree's chain of dependent steps, not bytes, so with
// more trees than compute units several workgroups share a unit
// (launch_expand).  Measured on MI355X, one launch that reads all nodes' ids,
// keeps one U and rebuilds a candidate list between three barriers a step,
// against this: one OLMoE-shaped tree 24.1 -> 15.9 us, one Qwen3-shaped tree
// 18.9 -> 11.3, 300 of them 61 -> 21, 1024 118 -> 27 us; at T_AR = 100000 (57 to
// 68 selections a tree) 124 -> 102, 440 -> 440 and 820 -> 712 us.  Trees that
// fill the LDS, every node selected: 8 nodes at L = 128, E = 1024, k = 32
// 54 -> 45 us, 104 at L = 48, E = 256 220 -> 195, 1024 at L = 35, E = 32
// 5.8 -> 5.8 ms; where every node is viable and none is selected the ids are
// read for nothing after the confidences instead of beside them: 16.6 -> 18.9
// us for the first of these shapes, 16.0 -> 16.6 for the second.
#include "common.h"
#include "kernels.h"

namespace s2moe {
namespace {

constexpr int kLeft = -1;  // n_admit of a tree that a launch leaves to the next one

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
static_assert(kWaves == kExpandWaves, "copies of the union in LDS");

// A wave's best candidate of a step: U_i and (slot << kNewBits | |E_i \ U|).
constexpr int kNewBits = 18;  // L E <= 128 * 1024 pairs
constexpr uint32_t kNone = ~0u;

struct Misc {
  union {
    int viable[4 * kWaves];  // viable nodes per (256-node block, wave)
    struct {
      double u[2][kWaves];  // per step parity and wave
      uint32_t sn[2][kWaves];
    } best;
  };
  int status;
};
static_assert(sizeof(Misc) <= 112, "Misc must fit its LDS slot");

// U_i from the node's benefit, current new-pair count and C^draft, in the
// order B / (n * T_exp + c) with no fused multiply-add.
__device__ __forceinline__ double utility(double ben, int n_new, double t_exp, double c) {
#pragma clang fp contract(off)
  const double cost = (double)n_new * t_exp + c;
  return ben / cost;
}

// (u, sn) beats (bu, bsn): larger utility, then smaller slot (= node index).
__device__ __forceinline__ bool better(double u, uint32_t sn, double bu, uint32_t bsn) {
  return u > bu || (u == bu && sn < bsn);
}

__device__ __forceinline__ int wave_sum_int(int v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

// Sum over each 16-lane row (DPP row shifts); the total lands in the row's
// last lane.
__device__ __forceinline__ int row16_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  return v;
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// popcount(a & ~b) over one EW-word bitset pair, read as aligned vectors.
template <int EW>
__device__ __forceinline__ int count_new(const uint32_t* a, const uint32_t* b) {
  int c = 0;
  if constexpr (EW == 1) {
    c = __popc(a[0] & ~b[0]);
  } else if constexpr (EW == 2) {
    const uint64_t x = *reinterpret_cast<const uint64_t*>(a);
    const uint64_t y = *reinterpret_cast<const uint64_t*>(b);
    c = __popcll(x & ~y);
  } else {
#pragma unroll
    for (int q = 0; q < EW / 4; ++q) {
      const u32x4 x = reinterpret_cast<const u32x4*>(a)[q];
      const u32x4 y = reinterpret_cast<const u32x4*>(b)[q];
#pragma unroll
      for (int w = 0; w < 4; ++w) c += __popc(x[w] & ~y[w]);
    }
  }
  return c;
}

// dst |= src (or dst = src) over W words, by `step` threads of which this is
// number `at`.
template <bool kAssign>
__device__ __forceinline__ void or_words(uint32_t* dst, const uint32_t* src, int W, int at,
                                         int step) {
  if ((W & 3) == 0) {  // then every bitset is 16-byte aligned
    u32x4* d = reinterpret_cast<u32x4*>(dst);
    const u32x4* s = reinterpret_cast<const u32x4*>(src);
    for (int w = at; w < (W >> 2); w += step) d[w] = kAssign ? s[w] : (d[w] | s[w]);
  } else {
    for (int w = at; w < W; w += step) dst[w] = kAssign ? src[w] : (dst[w] | src[w]);
  }
}

// Orders a wave's LDS accesses before and after it (each wave works on its own
// LDS copies, so no other wave takes part).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// One 8-byte LDS access that the compiler neither keeps in a register nor
// splits: p values pass between waves that are not at a barrier.
__device__ __forceinline__ double lds_load(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lds_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int NPT, int EW>
__device__ __forceinline__ void expand_tree(const ExpandArgs& a, unsigned char* lds, int t) {
  const ExpandLds lay = expand_lds(a.N, a.L, a.E, a.cap, a.copies);
  Misc* misc = reinterpret_cast<Misc*>(lds + lay.misc);
  uint32_t* rows = reinterpret_cast<uint32_t*>(lds + lay.rows);
  uint32_t* uni0 = reinterpret_cast<uint32_t*>(lds + lay.uni);
  double* pv = reinterpret_cast<double*>(lds + lay.pv);
  float* cdr = reinterpret_cast<float*>(lds + lay.cdr);
  uint16_t* node_of = reinterpret_cast<uint16_t*>(lds + lay.node);
  uint16_t* slot_of = reinterpret_cast<uint16_t*>(pv);  // between phases 2 and 4
  int16_t* par_of = reinterpret_cast<int16_t*>(lds + lay.list);  // before phase 5

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int L = a.L, E = a.E, k = a.k, N = a.N;
  const int Lk = L * k, W = L * EW;  // ids and bitset words of a node
  const bool copies = a.copies > 1;
  uint16_t* list =
      reinterpret_cast<uint16_t*>(lds + lay.list) + wave * ((N + kWaves - 1) / kWaves);
  uint32_t* uni = uni0 + (copies ? wave * W : 0);
  const size_t node0 = (size_t)t * N;

  // (1) per-node records (also the padding's, so that they need not wait for
  // the node count) and the root's ids: one round of loads.
  int par[NPT];
  float qd[NPT], cd[NPT];
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const size_t i = node0 + min(tid + m * kThreads, N - 1);
    par[m] = a.parent[i];
    qd[m] = a.q[i];
    cd[m] = a.c_draft[i];
  }
  constexpr int kRootPer = 4096 / kThreads;  // L * k <= 4096
  int rv[kRootPer];
#pragma unroll
  for (int r = 0; r < kRootPer; ++r) {
    const int j = tid + r * kThreads;
    rv[r] = -1;
    if (a.root_eid != nullptr && j < Lk) rv[r] = a.root_eid[(size_t)t * Lk + j];
  }
  const int n_in = a.n_nodes[t];
  const int n = min(max(n_in, 0), N);
  int status = n_in < 0 || n_in > N ? 8 : 0;
  uint32_t pending = 0, viable = 0;  // bit m: node tid + 256 m
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const int i = tid + m * kThreads;
    if (i < n) {
      bool ok = true;
      if (!(par[m] == -1 || (par[m] >= 0 && par[m] < i))) { ok = false; status |= 1; }
      if (!(qd[m] >= 0.f && qd[m] <= 1.f)) { ok = false; status |= 2; }
      if (!(cd[m] > 0.f && cd[m] < INFINITY)) { ok = false; status |= 4; }
      pv[i] = ok ? -1.0 : 0.0;  // -1: not resolved yet
      if (ok) pending |= 1u << m;
    }
  }
  for (int w = tid; w < W; w += kThreads) uni0[w] = 0u;
  if (tid == 0) misc->status = 0;
  __syncthreads();
  if (status) atomicOr(&misc->status, status);
  auto layer_of = [&](uint32_t f) { return (uint32_t)(((uint64_t)f * a.k_div) >> 42); };
#pragma unroll
  for (int r = 0; r < kRootPer; ++r) {
    const int j = tid + r * kThreads;
    const int e = rv[r];
    if (j < Lk && e >= 0 && e < E) atomicOr(&uni0[layer_of(j) * EW + (e >> 5)], 1u << (e & 31));
  }

  // (2) prefix confidences, root-down: p_i = p_parent * q_i.  Each wave
  // re-reads its nodes' parents until all are resolved.  A parent has a
  // smaller index, so the unresolved node of smallest index always has a
  // resolved parent (or none), whichever wave holds it: some wave gets on
  // with every reading, and every wait ends.  A node whose utility is below 1
  // even with every expert in U, or whose parent is such a node or invalid,
  // can never be selected: its p becomes 0, which makes its children's 0 as
  // well.
  double ben[NPT];
  while (__ballot(pending != 0)) {
#pragma unroll
    for (int m = 0; m < NPT; ++m) {
      if ((pending >> m) & 1u) {
        const double pp = par[m] < 0 ? 1.0 : lds_load(pv + par[m]);
        if (pp >= 0.0) {
          const double p = pp * (double)qd[m];
          ben[m] = p * a.t_ar;
          const bool v = utility(ben[m], 0, a.t_exp, (double)cd[m]) >= 1.0;
          lds_store(pv + tid + m * kThreads, v ? p : 0.0);
          pending &= ~(1u << m);
          if (v) viable |= 1u << m;
        }
      }
    }
  }

  // (3) viable nodes get slots in index order.
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const int c = __popcll(__ballot((viable >> m) & 1u));
    if (lane == 0) misc->viable[m * kWaves + wave] = c;
  }
  __syncthreads();
  int nv = 0;
  int slot[NPT];
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    int base = nv;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int c = misc->viable[m * kWaves + w];
      if (w < wave) base += c;
      nv += c;
    }
    slot[m] = base + __popcll(__ballot((viable >> m) & 1u) & below);
  }
  if (a.leave && nv > a.cap) {  // for the launch that follows
    if (tid == 0) a.n_admit[t] = kLeft;
    return;
  }
#pragma unroll
  for (int m = 0; m < NPT; ++m)
    if ((viable >> m) & 1u) {
      node_of[slot[m]] = (uint16_t)(tid + m * kThreads);
      slot_of[tid + m * kThreads] = (uint16_t)slot[m];
    }
  {
    const int words = nv * W;
    u32x4* r4 = reinterpret_cast<u32x4*>(rows);
    for (int w = tid; w < (words >> 2); w += kThreads) r4[w] = u32x4{0u, 0u, 0u, 0u};
    for (int w = (words & ~3) + tid; w < words; w += kThreads) rows[w] = 0u;
  }
  __syncthreads();
  // The parent of a viable node is viable.
#pragma unroll
  for (int m = 0; m < NPT; ++m)
    if ((viable >> m) & 1u) par_of[slot[m]] = par[m] < 0 ? -1 : (int16_t)slot_of[par[m]];

  // (4) the viable nodes' ids -> bitsets; ids outside [0, E) are padding
  // (they OR 0 into word 0: no branch).
  const int32_t* ids = a.eid + node0 * (size_t)Lk;
  auto set_bit = [&](uint32_t row, int e) {
    const bool ok = (uint32_t)e < (uint32_t)E;
    const uint32_t w = ok ? row * EW + ((uint32_t)e >> 5) : 0u;
    atomicOr(&rows[w], ok ? 1u << (e & 31) : 0u);
  };
  const int cpn = (Lk + 3) >> 2;  // 4-id chunks of a node
  const int n_chunks = nv * cpn;
  auto slot_of_chunk = [&](uint32_t c) { return (uint32_t)(((uint64_t)c * a.cpn_div) >> 42); };
  if ((Lk & 3) == 0) {
    // Chunks are 16-byte aligned (eid is); with k a multiple of 4 the four
    // ids of a chunk share a layer.
    constexpr int kBatch = 8;
    const bool same_layer = (k & 3) == 0;
    for (int c0 = tid; c0 < n_chunks; c0 += kThreads * kBatch) {
      u32x4 v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int c = c0 + u * kThreads;
        if (c < n_chunks) {
          const uint32_t sl = slot_of_chunk(c);
          v[u] = __builtin_nontemporal_load(
              reinterpret_cast<const u32x4*>(ids + (size_t)node_of[sl] * Lk) + (c - sl * cpn));
        }
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int c = c0 + u * kThreads;
        if (c < n_chunks) {
          const uint32_t sl = slot_of_chunk(c);
          const uint32_t f = 4 * (c - sl * cpn);
          uint32_t l = layer_of(f), pos = f - l * k;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            set_bit(sl * L + l, (int)v[u][x]);
            if (!same_layer && ++pos == (uint32_t)k) {
              pos = 0;
              ++l;
            }
          }
        }
      }
    }
  } else {
    for (int c = tid; c < n_chunks; c += kThreads) {
      const uint32_t sl = slot_of_chunk(c);
      const int f = 4 * (c - sl * cpn);
      const int32_t* src = ids + (size_t)node_of[sl] * Lk;
      int e[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) e[x] = f + x < Lk ? src[f + x] : -1;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (f + x < Lk) set_bit(sl * L + layer_of(f + x), e[x]);
    }
  }
  if (copies && wave > 0) or_words<true>(uni, uni0, W, lane, kWave);
  __syncthreads();
  // Each wave's own slots: bit q of a lane is slot 4 (lane + 64 q) + wave.
  int par_s[NPT];
  uint32_t avail = 0, done = 0;
#pragma unroll
  for (int q = 0; q < NPT; ++q) {
    const int v = kWaves * (lane + q * kWave) + wave;
    par_s[q] = v < nv ? par_of[v] : -2;
    if (par_s[q] == -1) avail |= 1u << q;
  }
#pragma unroll
  for (int m = 0; m < NPT; ++m)
    if ((viable >> m) & 1u) {
      pv[slot[m]] = ben[m];
      cdr[slot[m]] = cd[m];
    }
  __syncthreads();

  // (5) greedy selection.
  const int sub = lane & 15;
  const int nq = (nv + kThreads - 1) / kThreads;
  int s = 0;
  for (; s < nv; ++s) {
    if (a.max_admit > 0 && s >= a.max_admit) break;
    // Candidates: unselected, parent selected or the root.
    int nf = 0;
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      if (q < nq) {
        const bool cand = ((avail & ~done) >> q) & 1u;
        const uint64_t mask = __ballot(cand);
        if (cand)
          list[nf + __popcll(mask & below)] = (uint16_t)(kWaves * (lane + q * kWave) + wave);
        nf += __popcll(mask);
      }
    }
    if (copies) wave_sync();
    else __syncthreads();  // U is everybody's
    // Each 16-lane row scores one candidate at a time, a lane per layer; the
    // row's last lane keeps the row's best.
    double bu = -1.0;
    uint32_t bsn = kNone;
    for (int x0 = 0; x0 < nf; x0 += 4) {
      const int x = x0 + (lane >> 4);
      int c = 0, v = 0;
      if (x < nf) {
        v = list[x];
        const uint32_t* rv_ = rows + (size_t)v * W;
        for (int l = sub; l < L; l += 16) c += count_new<EW>(rv_ + l * EW, uni + l * EW);
      }
      c = row16_sum(c);
      if (x < nf && sub == 15) {
        const double u = utility(pv[v], c, a.t_exp, (double)cdr[v]);
        const uint32_t sn = ((uint32_t)v << kNewBits) | (uint32_t)c;
        if (better(u, sn, bu, bsn)) {
          bu = u;
          bsn = sn;
        }
      }
    }
    // The wave's best of its four row leaders.
    {
      double wu = readlane_f64(bu, 15);
      uint32_t wsn = __builtin_amdgcn_readlane(bsn, 15);
#pragma unroll
      for (int g = 1; g < 4; ++g) {
        const double gu = readlane_f64(bu, 16 * g + 15);
        const uint32_t gsn = __builtin_amdgcn_readlane(bsn, 16 * g + 15);
        if (better(gu, gsn, wu, wsn)) {
          wu = gu;
          wsn = gsn;
        }
      }
      bu = wu;
      bsn = wsn;
    }
    // Two buffers by step parity: a wave that is a step ahead writes the
    // other one, and none can be two steps ahead of the barrier.
    const int z = s & 1;
    if (lane == 0) {
      misc->best.u[z][wave] = bu;
      misc->best.sn[z][wave] = bsn;
    }
    __syncthreads();
    bu = misc->best.u[z][0];
    bsn = misc->best.sn[z][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w)
      if (better(misc->best.u[z][w], misc->best.sn[z][w], bu, bsn)) {
        bu = misc->best.u[z][w];
        bsn = misc->best.sn[z][w];
      }
    if (bsn == kNone || !(bu >= 1.0)) break;  // same decision in every thread
    const int j = (int)(bsn >> kNewBits);
    if (tid == 0) {
      a.order[node0 + s] = node_of[j];
      a.util[node0 + s] = bu;
      a.n_new[node0 + s] = (int)(bsn & ((1u << kNewBits) - 1));
    }
#pragma unroll
    for (int q = 0; q < NPT; ++q) {
      if (par_s[q] == j) avail |= 1u << q;
      if (kWaves * (lane + q * kWave) + wave == j) done |= 1u << q;
    }
    // U gains the selected node's experts; the next step's wave_sync or
    // barrier orders this before its scoring.
    const uint32_t* rj = rows + (size_t)j * W;
    if (copies) or_words<false>(uni, rj, W, lane, kWave);
    else or_words<false>(uni, rj, W, tid, kThreads);
  }
  if (copies) wave_sync();
  else __syncthreads();

  // Epilogue: padding of the per-selection outputs, union size, status.
  for (int x = s + tid; x < N; x += kThreads) {
    a.order[node0 + x] = -1;
    a.util[node0 + x] = 0.0;
    a.n_new[node0 + x] = 0;
  }
  if (wave == 0) {
    int pc = 0;
    for (int w = lane; w < W; w += kWave) pc += __popc(uni[w]);
    pc = wave_sum_int(pc);
    if (lane == 0) {
      a.n_admit[t] = s;
      a.n_pairs[t] = pc;
      a.status[t] = misc->status;
    }
  }
}

// A workgroup per tree, dealt to whichever unit is free.  kLeftOnly: a later
// launch, where only those whose tree was left do anything.
template <int NPT, int EW, bool kLeftOnly>
__global__ __launch_bounds__(kThreads, 4) void expand_kernel(ExpandArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  if (kLeftOnly && a.n_admit[blockIdx.x] != kLeft) return;
  expand_tree<NPT, EW>(a, lds, blockIdx.x);
}

// Bitsets that a workgroup of at most `budget` bytes of LDS holds.
int slots_in(const ExpandArgs& a, size_t budget, int copies) {
  int c = a.N;
  const size_t all = expand_lds(a.N, a.L, a.E, c, copies).total;
  const size_t row = (size_t)a.L * expand_words(a.E) * 4;
  if (all > budget) c = (int)max((long)0, (long)c - (long)((all - budget + row - 1) / row));
  while (c > 0 && expand_lds(a.N, a.L, a.E, c, copies).total > budget) --c;
  return c;
}

template <int NPT, int EW>
hipError_t launch_ew(const ExpandArgs& a, size_t lds_bytes, hipStream_t s) {
  const auto kernel =
      a.left_only ? expand_kernel<NPT, EW, true> : expand_kernel<NPT, EW, false>;
  if (lds_bytes > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(a.T), dim3(kThreads), lds_bytes, s, a);
  return hipGetLastError();
}

template <int NPT>
hipError_t launch_npt(const ExpandArgs& a, size_t lds_bytes, hipStream_t s) {
  switch (expand_words(a.E)) {
    case 1: return launch_ew<NPT, 1>(a, lds_bytes, s);
    case 2: return launch_ew<NPT, 2>(a, lds_bytes, s);
    case 4: return launch_ew<NPT, 4>(a, lds_bytes, s);
    case 8: return launch_ew<NPT, 8>(a, lds_bytes, s);
    case 16: return launch_ew<NPT, 16>(a, lds_bytes, s);
    case 32: return launch_ew<NPT, 32>(a, lds_bytes, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_one(const ExpandArgs& a, hipStream_t s) {
  const size_t lds_bytes = expand_lds(a.N, a.L, a.E, a.cap, a.copies).total;
  if (a.N <= kThreads) return launch_npt<1>(a, lds_bytes, s);
  if (a.N <= 2 * kThreads) return launch_npt<2>(a, lds_bytes, s);
  return launch_npt<4>(a, lds_bytes, s);
}

}  // namespace

// The launches of a call: one that keeps the bitsets of every node, unless
// the trees outnumber the compute units.  Then first one whose workgroups take
// half of a unit's LDS each (a quarter from two trees a unit on), which leaves
// the trees with more viable nodes than its bitsets to the next.
// Measured on MI355X, 1024 Qwen3-shaped trees (116 nodes of 768 bytes; 46
// bitsets in a quarter, 100 in a half) by T_AR, against one launch of one
// workgroup a unit: 512 27 us (118), 8192, where most trees pass the quarter,
// 234 (440; 299 without the half), 100000 712 (820).  Empty later launches cost
// about 1 us each.  Where each launch leaves every tree and the last one selects
// nothing, the others are lost: 300 trees of 28 nodes of 4 KB 35 us (26).
//
// The copies of U: one per wave up to kCopyWords words, where it does not
// cost the last bitset.  One Qwen3-shaped tree of 57 selections (192 words)
// 102 us against 104 with a single U; L = 48, E = 256, 52 selections (384 words)
// 91.4 against 89.9, L = 64, E = 512, 28 selections (1024 words) 64 against 60.
constexpr size_t kQuarterLds = 40 * 1024, kHalfLds = 80 * 1024;
constexpr int kMinSlots = 16;     // a launch with fewer bitsets would leave nearly every tree
constexpr int kCopyWords = 256;

hipError_t launch_expand(const ExpandArgs& a_in, size_t lds_limit, hipStream_t s) {
  if (a_in.T == 0) return hipSuccess;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  ExpandArgs a = a_in;
  a.left_only = false;
  const int words = a.L * expand_words(a.E);
  const struct {
    size_t lds;
    int min_slots;  // fewer bitsets than this: not this launch
    int trees;      // nor for this many trees or fewer
  } launches[] = {{kQuarterLds, min(kMinSlots, a.N), 2 * cus},
                  {kHalfLds, min(kMinSlots, a.N), cus},
                  {lds_limit, a.N, 0}};
  for (const auto& l : launches) {
    if (a.T <= l.trees) continue;
    const int single = slots_in(a, l.lds, 1), copied = slots_in(a, l.lds, kExpandWaves);
    const bool all = single == a.N && copied < a.N;  // the copies would cost the last bitset
    a.copies = words <= kCopyWords && !all && copied >= l.min_slots ? kExpandWaves : 1;
    a.cap = a.copies == 1 ? single : copied;
    if (a.cap < l.min_slots) continue;
    a.leave = a.cap < a.N;
    if ((e = launch_one(a, s)) != hipSuccess || !a.leave) return e;
    a.left_only = true;
  }
  // An accepted shape's N bitsets and one union fit the last launch.
  return hipErrorInvalidValue;
}

}  // namespace s2moe
