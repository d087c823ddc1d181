// Routing-aware adaptive speculative expansion (Sec. "Routing-aware Adaptive
// Speculative Expansion"): best-first selection of draft-tree tokens by the
// utility U_i = p_i T_AR / (|E_i \ U| T_exp + C_i^draft) while U_i >= 1.
//
// One workgroup of 256 threads per tree.  U only grows and U_i falls with
// |E_i \ U|, so a node with p_i T_AR / C_i^draft < 1, and every node below it,
// can never be selected: only the others ("viable", in index order: slots)
// take part, and only their ids are read.  In LDS, E rounded up to a power of
// two >= 32 is EW words:
//   pv[i]            p_i (0 for nodes that are not viable);  cdr[i] = C_i^draft
//   rows[slot][l][w] the experts the slot's node is predicted to use at layer l
//   uni[wave][l][w]  the union U of the selected tokens' (layer, expert) pairs,
//                    a copy per wave
// so that repeated ids collapse by themselves, |E_i \ U| is
// sum_l popcount(rows[i][l] & ~uni[l]) and U grows by a word-wise OR.
// Phases: (1) per-node validity and the root's experts into U; (2) prefix
// confidences and viability; (3) slots; (4) the slots' ids -> bitsets; (5) the
// greedy loop: each wave lists the candidates from its own flags, each 16-lane
// row of each wave scores one candidate at a time, the block takes the
// largest U_i (ties: smaller index) and, if U_i >= 1, every wave adds the
// node's experts to its copy of U.  A step has one workgroup barrier.
//
// What bounds it is each tree's chain of dependent steps, not bytes, so with
// more trees than compute units several workgroups share a unit
// (launch_expand); slots beyond the bitsets in LDS are counted from their ids
// in memory.  Measured on MI355X against all nodes' ids and bitsets, a
// candidate list and three barriers per step: one OLMoE-shaped tree
// 24.0 -> 17.2 us, one Qwen3-shaped tree 20.5 -> 13.5, 400 of them 66 -> 23,
// 1024 120 -> 26 us; 1024 OLMoE-shaped trees 71 -> 26, GPT-OSS-shaped
// 73 -> 30 us.
#include "common.h"
#include "kernels.h"

namespace s2moe {
namespace {

// Which trees a launch takes: all; those whose viable nodes fit its bitsets
// (the others get n_admit = kLeft); those left.
enum : int { kAllTrees = 0, kFitting = 1, kRest = 2 };
constexpr int kLeft = -1;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
static_assert(kWaves == kExpandWaves, "copies of the union in LDS");

struct Misc {
  double red_u[2][kWaves];  // per step parity and wave: the wave's best candidate
  int red_i[2][kWaves];
  int red_n[2][kWaves];
  int viable[4 * kWaves];  // viable nodes per (256-node block, wave)
  int status;
};
static_assert(sizeof(Misc) <= 256, "Misc must fit its LDS slot");

// U_i from the node's benefit, current new-pair count and C^draft, in the
// order B / (n * T_exp + c) with no fused multiply-add.
__device__ __forceinline__ double utility(double ben, int n_new, double t_exp, double c) {
#pragma clang fp contract(off)
  const double cost = (double)n_new * t_exp + c;
  return ben / cost;
}

// (u, i) beats (bu, bi): larger utility, then smaller node index.
__device__ __forceinline__ bool better(double u, int i, double bu, int bi) {
  return u > bu || (u == bu && i < bi);
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

// The same count from the layer's k ids (a slot without a bitset): ids
// outside [0, E) are padding, repeats count once.
__device__ __forceinline__ int count_new_ids(const int32_t* e, int k, int E, const uint32_t* u) {
  int c = 0;
  for (int x = 0; x < k; ++x) {
    const int ex = e[x];
    if ((uint32_t)ex >= (uint32_t)E || ((u[ex >> 5] >> (ex & 31)) & 1u)) continue;
    bool first = true;
    for (int y = 0; y < x; ++y) first = first && e[y] != ex;
    c += first;
  }
  return c;
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
__global__ __launch_bounds__(kThreads) void expand_kernel(ExpandArgs a) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int Q = NPT * kWaves;  // slots per lane
  const ExpandLds lay = expand_lds(a.N, a.L, a.E, a.cap);
  double* pv = reinterpret_cast<double*>(lds + lay.pv);
  uint32_t* rows = reinterpret_cast<uint32_t*>(lds + lay.rows);
  uint32_t* uni0 = reinterpret_cast<uint32_t*>(lds + lay.uni);
  float* cdr = reinterpret_cast<float*>(lds + lay.cdr);
  uint16_t* node_of = reinterpret_cast<uint16_t*>(lds + lay.node);
  uint16_t* slot_of = reinterpret_cast<uint16_t*>(lds + lay.slot);
  int16_t* par_of = reinterpret_cast<int16_t*>(lds + lay.par);
  Misc* misc = reinterpret_cast<Misc*>(lds + lay.misc);

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int L = a.L, E = a.E, k = a.k, N = a.N;
  const int Lk = L * k, W = L * EW;  // ids and bitset words of a node
  uint16_t* list = reinterpret_cast<uint16_t*>(lds + lay.list) + wave * N;
  uint32_t* uni = uni0 + wave * W;

  const int t = blockIdx.x;
  if (a.pass == kRest && a.n_admit[t] != kLeft) return;
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
      cdr[i] = cd[m];
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
  // re-reads its nodes' parents until all are resolved; a parent has a
  // smaller index, so the wave that holds it never waits for this one and
  // every wait ends.  A node whose utility is below 1 even with every expert
  // in U, or whose parent is such a node or invalid, can never be selected:
  // its p becomes 0, which makes its children's 0 as well.
  while (__ballot(pending != 0)) {
#pragma unroll
    for (int m = 0; m < NPT; ++m) {
      if ((pending >> m) & 1u) {
        const double pp = par[m] < 0 ? 1.0 : lds_load(pv + par[m]);
        if (pp >= 0.0) {
          const double p = pp * (double)qd[m];
          const bool v = utility(p * a.t_ar, 0, a.t_exp, (double)cd[m]) >= 1.0;
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
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    int base = nv;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int c = misc->viable[m * kWaves + w];
      if (w < wave) base += c;
      nv += c;
    }
    const uint64_t mask = __ballot((viable >> m) & 1u);
    if ((viable >> m) & 1u) {
      const int i = tid + m * kThreads;
      const int v = base + __popcll(mask & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
      node_of[v] = (uint16_t)i;
      slot_of[i] = (uint16_t)v;
      par_of[v] = (int16_t)par[m];
    }
  }
  if (a.pass == kFitting && nv > a.cap) {  // left to the launch that follows
    if (tid == 0) a.n_admit[t] = kLeft;
    return;
  }
  const int nr = min(nv, a.cap);  // slots with a bitset in LDS
  {
    const int words = nr * W;
    u32x4* r4 = reinterpret_cast<u32x4*>(rows);
    for (int w = tid; w < (words >> 2); w += kThreads) r4[w] = u32x4{0u, 0u, 0u, 0u};
    for (int w = (words & ~3) + tid; w < words; w += kThreads) rows[w] = 0u;
  }
  __syncthreads();

  // (4) the ids of those slots' nodes -> bitsets; ids outside [0, E) are
  // padding (they OR 0 into word 0: no branch).
  const int32_t* ids = a.eid + node0 * (size_t)Lk;
  auto set_bit = [&](uint32_t row, int e) {
    const bool ok = (uint32_t)e < (uint32_t)E;
    const uint32_t w = ok ? row * EW + ((uint32_t)e >> 5) : 0u;
    atomicOr(&rows[w], ok ? 1u << (e & 31) : 0u);
  };
  const int cpn = (Lk + 3) >> 2;  // 4-id chunks of a node
  const int n_chunks = nr * cpn;
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
  // Every wave keeps its own copy of U and of the candidate flags.
  if (wave > 0)
    for (int w = lane; w < W; w += kWave) uni[w] = uni0[w];
  const int nq = (nv + kWave - 1) / kWave;
  int par_s[Q];
  uint32_t avail = 0, done = 0;  // bit q: slot lane + 64 q
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    par_s[q] = -2;
    const int v = lane + q * kWave;
    if (q < nq && v < nv) {
      const int pn = par_of[v];
      par_s[q] = pn < 0 ? -1 : (int)slot_of[pn];
      if (pn < 0) avail |= 1u << q;
    }
  }
  __syncthreads();

  // (5) greedy selection, one workgroup barrier per step.
  const int sub = lane & 15;
  int s = 0;
  for (; s < nv; ++s) {
    if (a.max_admit > 0 && s >= a.max_admit) break;
    // Candidates: unselected, parent selected or the root.
    int nf = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q < nq) {
        const bool cand = ((avail & ~done) >> q) & 1u;
        const uint64_t mask = __ballot(cand);
        if (cand)
          list[nf + __popcll(mask & (lane == 0 ? 0ull : (~0ull >> (64 - lane))))] =
              (uint16_t)(lane + q * kWave);
        nf += __popcll(mask);
      }
    }
    wave_sync();
    if (nf == 0) break;  // the same in every wave
    // Each 16-lane row of each wave scores one candidate at a time, a lane
    // per layer; the row's last lane keeps the row's best.
    double bu = -1.0;
    int bi = INT32_MAX, bn = 0;
    for (int x0 = wave * 4; x0 < nf; x0 += kWaves * 4) {
      const int x = x0 + (lane >> 4);
      int c = 0, v = 0, node = 0;
      if (x < nf) {
        v = list[x];
        node = node_of[v];
        if (v < nr) {
          const uint32_t* rv_ = rows + (size_t)v * W;
          for (int l = sub; l < L; l += 16) c += count_new<EW>(rv_ + l * EW, uni + l * EW);
        } else {
          for (int l = sub; l < L; l += 16)
            c += count_new_ids(ids + (size_t)node * Lk + l * k, k, E, uni + l * EW);
        }
      }
      c = row16_sum(c);
      if (x < nf && sub == 15) {
        const double u = utility(pv[node] * a.t_ar, c, a.t_exp, (double)cdr[node]);
        if (better(u, v, bu, bi)) {
          bu = u;
          bi = v;
          bn = c;
        }
      }
    }
    // The wave's best of its four row leaders.
    {
      double wu = readlane_f64(bu, 15);
      int wi = __builtin_amdgcn_readlane(bi, 15), wn = __builtin_amdgcn_readlane(bn, 15);
#pragma unroll
      for (int g = 1; g < 4; ++g) {
        const double gu = readlane_f64(bu, 16 * g + 15);
        const int gi = __builtin_amdgcn_readlane(bi, 16 * g + 15);
        if (better(gu, gi, wu, wi)) {
          wu = gu;
          wi = gi;
          wn = __builtin_amdgcn_readlane(bn, 16 * g + 15);
        }
      }
      bu = wu;
      bi = wi;
      bn = wn;
    }
    // Two buffers by step parity: a wave that is a step ahead writes the
    // other one, and none can be two steps ahead of the barrier.
    const int z = s & 1;
    if (lane == 0) {
      misc->red_u[z][wave] = bu;
      misc->red_i[z][wave] = bi;
      misc->red_n[z][wave] = bn;
    }
    __syncthreads();
    bu = misc->red_u[z][0];
    bi = misc->red_i[z][0];
    bn = misc->red_n[z][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w)
      if (better(misc->red_u[z][w], misc->red_i[z][w], bu, bi)) {
        bu = misc->red_u[z][w];
        bi = misc->red_i[z][w];
        bn = misc->red_n[z][w];
      }
    if (bi == INT32_MAX || !(bu >= 1.0)) break;  // same decision in every thread
    const int j = bi, node = node_of[j];
    if (tid == 0) {
      a.order[node0 + s] = node;
      a.util[node0 + s] = bu;
      a.n_new[node0 + s] = bn;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (par_s[q] == j) avail |= 1u << q;
      if (lane + q * kWave == j) done |= 1u << q;
    }
    // U gains the selected node's experts.
    if (j < nr) {
      const uint32_t* rj = rows + (size_t)j * W;
      for (int w = lane; w < W; w += kWave) uni[w] |= rj[w];
    } else {
      for (int f = lane; f < Lk; f += kWave) {
        const int e = ids[(size_t)node * Lk + f];
        if ((uint32_t)e < (uint32_t)E)
          atomicOr(&uni[layer_of(f) * EW + (e >> 5)], 1u << (e & 31));
      }
    }
    // The next step's wave_sync orders U before its scoring.
  }
  wave_sync();

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

// Bitsets that a workgroup of at most `budget` bytes of LDS holds.
int slots_in(const ExpandArgs& a, size_t budget) {
  const size_t row = (size_t)a.L * expand_words(a.E) * 4;
  const size_t fixed = expand_lds(a.N, a.L, a.E, 0).total;
  return (int)min((size_t)a.N, budget > fixed ? (budget - fixed) / row : (size_t)0);
}

template <int NPT, int EW>
hipError_t launch_ew(const ExpandArgs& a, size_t lds_bytes, hipStream_t s) {
  const void* fn = reinterpret_cast<const void*>(&expand_kernel<NPT, EW>);
  if (lds_bytes > 65536) {
    const hipError_t e =
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((expand_kernel<NPT, EW>), dim3(a.T), dim3(kThreads), lds_bytes, s, a);
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
  const size_t lds_bytes = expand_lds(a.N, a.L, a.E, a.cap).total;
  if (a.N <= kThreads) return launch_npt<1>(a, lds_bytes, s);
  if (a.N <= 2 * kThreads) return launch_npt<2>(a, lds_bytes, s);
  return launch_npt<4>(a, lds_bytes, s);
}

}  // namespace

// Trees that do not fill the compute units, and trees whose bitsets all fit a
// quarter of a unit's LDS, take one launch.  Otherwise one launch with a
// quarter (four workgroups a unit) takes the trees whose viable nodes fit,
// and a second one with half takes the rest.  Measured on MI355X, 1024
// Qwen3-shaped trees (768 bytes a node, 44 slots in 40 KB) by T_AR: 512 26
// us with the two launches (41 with one at half), 8192, where most trees are
// left, 256 (188); one launch at a quarter with the nodes beyond it counted
// from their ids 25 and 672, the bitsets of all nodes in one workgroup a unit
// with the next tree's ids prefetched 121 and 432.
constexpr size_t kQuarterLds = 40 * 1024, kHalfLds = 80 * 1024;
constexpr int kMinSlots = 16;

hipError_t launch_expand(const ExpandArgs& a_in, size_t lds_limit, hipStream_t s) {
  if (a_in.T == 0) return hipSuccess;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  ExpandArgs a = a_in;
  const int most = slots_in(a, lds_limit);  // the fixed part alone is at most 66000 bytes
  const int quarter = slots_in(a, kQuarterLds);
  a.pass = kAllTrees;
  a.cap = most;
  if (a.T <= cus || quarter >= a.N) {
    if (a.T > cus) a.cap = a.N;
    return launch_one(a, s);
  }
  if (quarter >= kMinSlots) {
    a.pass = kFitting;
    a.cap = quarter;
    if ((e = launch_one(a, s)) != hipSuccess) return e;
    a.pass = kRest;
  }
  a.cap = min(most, max(slots_in(a, kHalfLds), kMinSlots));
  return launch_one(a, s);
}

}  // namespace s2moe
