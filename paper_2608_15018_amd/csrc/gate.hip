// Reuse-aware expert gating and token->expert bucketing (Sec. "Reuse-aware
// Expert Gating": cross-token expert importance aggregation, global
// preferred expert selection, soft routing bias for reuse promotion).
//
// One workgroup of 16 waves handles the whole verify batch (B <= 256,
// E <= 256): the decisions couple all tokens through g, and the batch is
// small.  Nothing here is a serial loop over assignments:
//   * g: a few threads per expert sum runs of tokens, runs added in order;
//   * TopCap: one wave's exact top-cap of the candidates' g by (g desc, id
//     asc), the threshold search used for the per-token top-k;
//   * per token (a team of lanes: a wave, or a 16-lane row of one so that the
//     workgroup takes 64 tokens at a time): biased order keys, the exact top-k
//     by taking the team's largest key k times (ties to the lower expert id),
//     or by the threshold search where k is large (team_max_k), ascending-id
//     order, a softmax over the team;
//   * buckets: a B-bit token mask per expert (LDS 64-bit ORs), so an
//     assignment's position in its expert's list is the popcount of the mask
//     below its token.
// Measured on MI355X, this kernel: 256 tokens over 8 experts 25 -> 10.6 us, 64
// over 64 experts 11.1 -> 8.3, 37 over 128 experts 12.5 -> 9.6, against a
// bitwise threshold search by ballots, one token per wave at a time, which the
// one scalar unit of the compute unit bound.
// Every result is deterministic: integer atomics only (bitwise OR), fixed
// floating-point summation orders, rank-based placement.
#include "small_batch.h"

namespace s2moe {

constexpr int kStage = 10240;  // logits staged in LDS up to B * E = 10240

// A token's logits in this lane's slots (experts e0 .. e0 + S - 1); slots past
// E are left 0.
template <int S>
__device__ __forceinline__ void load_row(const float* ell, int e0, int E, bool real, float (&l)[S]) {
  if (S % 4 == 0 && (E & 3) == 0) {
#pragma unroll
    for (int s = 0; s < S; s += 4) {
      const f32x4 v = real && e0 + s < E ? *reinterpret_cast<const f32x4*>(ell + e0 + s)
                                         : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (s + q < S) l[s + q] = v[q];
    }
  } else {
#pragma unroll
    for (int s = 0; s < S; ++s) l[s] = real && e0 + s < E ? ell[e0 + s] : 0.f;
  }
}

// kG = lanes of a token's team, kS = expert slots per lane (E <= kG kS).
// kNT = 0: teams rank by taking maxima; else whole waves (kG = 64), kNT tokens
// at a time, by the threshold search.  kSelect (with kStaged): the kernel first
// ranks every token's staged logits itself and writes plain_idx and gap,
// instead of reading them from a routing launch (ra: the routing step's
// arguments).
template <bool kStaged, int kG, int kS, int kNT, bool kSelect>
__global__ __launch_bounds__(1024) void reuse_gate_kernel(GateArgs a, RouteArgs ra) {
  static_assert(kStaged || !kSelect, "ranking reads the staged logits");
  static_assert(kNT == 0 || kG == kWave, "the search ranks by wave");
  constexpr int kMaskWords = kMaxTokens / 64;
  constexpr int kNJ = (kG * kS + 63) / 64;  // expert slots per lane of TopCap's wave
  __shared__ __align__(16) float ell_s[kStaged ? kStage : 1];
  __shared__ float w_s[kMaxTokens];
  __shared__ float gap_s[kMaxTokens];
  __shared__ float gm_s[kMaxExperts];                  // g of every expert
  __shared__ int pref_s[kMaxExperts];
  __shared__ int count_s[kMaxExperts];
  __shared__ int offset_s[kMaxExperts + 1];
  __shared__ uint64_t mask_s[kMaxExperts][kMaskWords];
  // [part][E] partial sums of g first, the selected expert ids later.
  static_assert(kMaxTokens * kMaxTopK == 4 * 1024, "shared buffer size");
  __shared__ float gpart_s[1024];
  uint8_t* idx_s = reinterpret_cast<uint8_t*>(gpart_s);
  __shared__ int cand_s[kMaxExperts];
  __shared__ uint8_t plain_s[kSelect ? kMaxTokens * kMaxTopK : 1];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = wave_id();
  const int n_waves = blockDim.x >> 6;
  const int B = a.B, E = a.E, k = a.k;

  // Non-negative confidences w_b; logits to LDS; cleared masks and ranks.
  int positive = 0;
  if (tid < B) {
    const float w = fmaxf(a.conf_w[tid], 0.f);
    w_s[tid] = w;
    if (!kSelect) gap_s[tid] = a.gap[tid];
    positive = w > 0.f;
  }
  if (kStaged) {
    // All loads first, then the LDS writes (10 per thread at most).
    constexpr int kPer = kStage / 1024;
    float v[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = tid + q * 1024;
      v[q] = i < B * E ? a.logits[i] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int i = tid + q * 1024;
      if (i < B * E) ell_s[i] = v[q];
    }
  }
  for (int i = tid; i < kMaxExperts * kMaskWords; i += blockDim.x)
    (&mask_s[0][0])[i] = 0ull;
  if (tid < kMaxExperts) {
    cand_s[tid] = (!(a.flags & kPrefActivatedOnly) && tid < E) ? 1 : 0;
  }
  const int active = __syncthreads_or(positive);
  const float* ell = kStaged ? static_cast<const float*>(ell_s) : a.logits;

  // Team t of wave w takes tokens kTeams w + t, + kTeams n_waves, ...
  constexpr int kTeams = kWave / kG;
  const int team = lane / kG, e0 = (lane % kG) * kS;
  if (kSelect && kNT > 0) {
    for (int b = wave; b < B; b += n_waves)
      wave_select_plain<kNJ>(E, k, ell + (size_t)b * E, plain_s + b * k, gap_s + b,
                             ra.plain_idx + (size_t)b * k, ra.gap + b);
    __syncthreads();
  } else if (kSelect) {
    // Exact top-(k+1) by (value desc, id asc): the last one taken is the
    // (k+1)-th, the others are the plain top-k.
    for (int b0 = wave * kTeams; b0 < B; b0 += n_waves * kTeams) {
      const int b = b0 + team;
      float l[kS];
      load_row<kS>(ell + (size_t)min(b, B - 1) * E, e0, E, b < B, l);
      uint32_t key[kS];
#pragma unroll
      for (int s = 0; s < kS; ++s) key[s] = b < B && e0 + s < E ? order_key(l[s]) : 0u;
      uint32_t bits = 0, rest = 0;
      const uint32_t first = team_take_max<kG, kS>(key, bits);
      for (int j = 1; j < k; ++j) team_take_max<kG, kS>(key, bits);
      const float gv = key_value(first) - key_value(team_take_max<kG, kS>(key, rest));
      int pos = b * k + team_exclusive_scan<kG>(__popc(bits));
#pragma unroll
      for (int s = 0; s < kS; ++s)
        if ((bits >> s) & 1u) {
          ra.plain_idx[pos] = e0 + s;
          plain_s[pos++] = (uint8_t)(e0 + s);
        }
      if (b < B && lane % kG == 0) {
        gap_s[b] = gv;
        ra.gap[b] = gv;
      }
    }
    __syncthreads();
  }

  // TopCap candidates: all experts, or those in some token's plain top-k.
  if (a.flags & kPrefActivatedOnly) {
    for (int i = tid; i < B * k; i += blockDim.x) {
      const int e = kSelect ? (int)plain_s[i] : a.plain_idx[i];
      if (e >= 0 && e < E) cand_s[e] = 1;
    }
  }

  // g_e = sum_b w_b * ell_{b,e}: `parts` threads per expert each sum a
  // contiguous run of tokens in order, then the runs are added in order.
  int parts = 1;
  while (parts * 2 * E <= 1024 && parts * 2 <= B) parts *= 2;
  const int run = (B + parts - 1) / parts;
  if (tid < parts * E) {
    const int e = tid % E, part = tid / E;
    const int b_lo = part * run, b_hi = min(B, b_lo + run);
    float s = 0.f;
#pragma unroll 4
    for (int b = b_lo; b < b_hi; ++b) s = fmaf(w_s[b], ell[(size_t)b * E + e], s);
    gpart_s[part * E + e] = s;
  }
  __syncthreads();
  if (tid < E) {
    float s = gpart_s[tid];
    for (int part = 1; part < parts; ++part) s += gpart_s[part * E + tid];
    a.g[tid] = s;
    gm_s[tid] = s;
  }
  __syncthreads();

  // E* = TopCap(g): the cap candidates of largest g (ties: lower id), by one
  // wave; all candidates when there are at most cap.
  if (wave == 0) {
    uint32_t key[1][kNJ];
    int n_cand = 0;
#pragma unroll
    for (int j = 0; j < kNJ; ++j) {
      const int e = lane + kWave * j;
      key[0][j] = e < E && cand_s[e] ? order_key(gm_s[e]) : 0u;
      n_cand += __popcll(__ballot(key[0][j] != 0u));
    }
    uint32_t pref_bits = 0;
    if (active) {
      if (n_cand <= a.cap) {
#pragma unroll
        for (int j = 0; j < kNJ; ++j)
          if (key[0][j] != 0u) pref_bits |= 1u << j;
      } else {
        uint32_t sel[1];
        wave_top_k<1, kNJ>(key, a.cap, sel);
        pref_bits = sel[0];
      }
    }
#pragma unroll
    for (int j = 0; j < kNJ; ++j) {
      const int e = lane + kWave * j;
      if (e < E) {
        const int p = (pref_bits >> j) & 1u;
        pref_s[e] = p;
        a.pref[e] = p;
      }
    }
  }
  __syncthreads();

  // Per token: lambda_b, biased keys, biased top-k, gate weights, masks.
  const bool from_biased = (a.flags & kGateFromBiased) != 0;
  if constexpr (kNT > 0) {
    // Wave w takes tokens w, w + 16, ...; kNT of them at a time.
    for (int b0 = wave; b0 < B; b0 += n_waves * kNT) {
      float l[kNT][kNJ], lb[kNT][kNJ];
      uint32_t key[kNT][kNJ];
#pragma unroll
      for (int t = 0; t < kNT; ++t) {
        const int b = b0 + t * n_waves;
        float lam = 0.f;
        if (active && b < B) lam = (a.flags & kBiasAbsolute) ? a.alpha : a.alpha * gap_s[b];
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
          const int e = lane + kWave * j;
          l[t][j] = 0.f;
          lb[t][j] = 0.f;
          key[t][j] = 0;
          if (b < B && e < E) {
            l[t][j] = ell[(size_t)b * E + e];
            lb[t][j] = pref_s[e] ? l[t][j] + lam : l[t][j];
            key[t][j] = order_key(lb[t][j]);
          }
        }
      }
      uint32_t bits[kNT];
      wave_top_k<kNT, kNJ>(key, k, bits);
      float ez[kNT][kNJ], sum[kNT], inv_s[kNT];
#pragma unroll
      for (int t = 0; t < kNT; ++t) {
        uint32_t mk = 0;
#pragma unroll
        for (int j = 0; j < kNJ; ++j)
          if ((bits[t] >> j) & 1u) mk = max(mk, from_biased ? key[t][j] : order_key(l[t][j]));
        const float m = key_value(wave_max_key_dpp(mk));
        sum[t] = 0.f;
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
          const float x = from_biased ? lb[t][j] : l[t][j];
          ez[t][j] = ((bits[t] >> j) & 1u) ? __builtin_amdgcn_exp2f((x - m) * kLog2e) : 0.f;
          sum[t] += ez[t][j];
        }
      }
#pragma unroll
      for (int t = 0; t < kNT; ++t) inv_s[t] = __builtin_amdgcn_rcpf(wave_sum_dpp(sum[t]));
#pragma unroll
      for (int t = 0; t < kNT; ++t) {
        const int b = b0 + t * n_waves;
        if (b >= B) break;
        int rank[kNJ];
        wave_rank_flagged<kNJ>(bits[t], rank);
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
          if ((bits[t] >> j) & 1u) {
            const int pos = b * k + rank[j];
            const int e = lane + kWave * j;
            a.idx[pos] = e;
            a.gate_w[pos] = ez[t][j] * inv_s[t];
            idx_s[pos] = (uint8_t)e;
            atomicOr(reinterpret_cast<unsigned long long*>(&mask_s[e][b >> 6]),
                     1ull << (b & 63));
          }
        }
      }
    }
  }
  for (int b0 = kNT > 0 ? B : wave * kTeams; b0 < B; b0 += n_waves * kTeams) {
    const int b = b0 + team;
    const bool real = b < B;
    float lam = 0.f;
    if (active && real) lam = (a.flags & kBiasAbsolute) ? a.alpha : a.alpha * gap_s[b];
    float l[kS], x[kS];  // x: what the gate weights are taken from
    uint32_t key[kS], xkey[kS];
    load_row<kS>(ell + (size_t)min(b, B - 1) * E, e0, E, real, l);
#pragma unroll
    for (int s = 0; s < kS; ++s) {
      const bool in = real && e0 + s < E;
      const float lb = in && pref_s[e0 + s] ? l[s] + lam : l[s];
      x[s] = from_biased ? lb : l[s];
      key[s] = in ? order_key(lb) : 0u;
      xkey[s] = from_biased ? key[s] : order_key(l[s]);
    }
    uint32_t bits = 0;
    for (int j = 0; j < k; ++j) team_take_max<kG, kS>(key, bits);
    // Softmax over the selected k: max through the order keys (exact),
    // then exp, a team sum and one reciprocal.
    uint32_t mk = 0;
#pragma unroll
    for (int s = 0; s < kS; ++s)
      if ((bits >> s) & 1u) mk = max(mk, xkey[s]);
    const float m = key_value(team_max_key<kG>(mk));
    float ez[kS], sum = 0.f;
#pragma unroll
    for (int s = 0; s < kS; ++s) {
      // exp(x - m) as 2^((x - m) log2 e) on the hardware exp2 (about 1e-6
      // relative error for |x - m| < 20)
      ez[s] = ((bits >> s) & 1u) ? __builtin_amdgcn_exp2f((x[s] - m) * kLog2e) : 0.f;
      sum += ez[s];
    }
    const float inv_s = __builtin_amdgcn_rcpf(team_sum<kG>(sum));
    int pos = b * k + team_exclusive_scan<kG>(__popc(bits));
#pragma unroll
    for (int s = 0; s < kS; ++s) {
      if ((bits >> s) & 1u) {
        const int e = e0 + s;
        a.idx[pos] = e;
        a.gate_w[pos] = ez[s] * inv_s;
        idx_s[pos] = (uint8_t)e;
        ++pos;
        atomicOr(reinterpret_cast<unsigned long long*>(&mask_s[e][b >> 6]), 1ull << (b & 63));
      }
    }
  }
  __syncthreads();

  // Counts from the masks; exclusive offsets and the activated-expert list.
  if (tid < E) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) c += __popcll(mask_s[tid][w]);
    count_s[tid] = c;
    a.count[tid] = c;
  }
  __syncthreads();
  if (wave == 0) {
    int c[4], f[4], sum_c = 0, sum_f = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = lane * 4 + j;
      c[j] = e < E ? count_s[e] : 0;
      f[j] = c[j] > 0;
      sum_c += c[j];
      sum_f += f[j];
    }
    const int incl_c = wave_inclusive_scan_dpp(sum_c);
    const int incl_f = wave_inclusive_scan_dpp(sum_f);
    const int total_c = __builtin_amdgcn_readlane(incl_c, 63);
    const int total_f = __builtin_amdgcn_readlane(incl_f, 63);
    int run_c = incl_c - sum_c, run_f = incl_f - sum_f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = lane * 4 + j;
      if (e < E) {
        offset_s[e] = run_c;
        a.offset[e] = run_c;
        if (f[j]) a.uniq[run_f] = e;
      }
      run_c += c[j];
      run_f += f[j];
    }
    for (int i = total_f + lane; i < E; i += kWave) a.uniq[i] = -1;
    if (lane == 0) {
      offset_s[E] = total_c;
      a.offset[E] = total_c;
      *a.n_uniq = total_f;
    }
  }
  __syncthreads();

  // Stable expert-major slot list: assignment (b, j) of expert e goes after
  // the assignments of e by tokens b' < b.  Every idx_s entry was written
  // above with an id below E, and offset_s[e] + before < B k for each of
  // them, so the two clamps below never change a result the kernel computes.
  // They are defence only: they keep the addressing inside offset_s and slot
  // should that invariant ever be broken by a change to this kernel.
  for (int i = tid; i < B * k; i += blockDim.x) {
    const int b = i / k;
    const int e = min((int)idx_s[i], E - 1);
    int before = 0;
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) {
      const uint64_t m = mask_s[e][w];
      if (w < (b >> 6)) before += __popcll(m);
      else if (w == (b >> 6)) before += __popcll(m & ((1ull << (b & 63)) - 1ull));
    }
    a.slot[min(offset_s[e] + before, B * k - 1)] = i;
  }
}

// Small batches without a bias that can change the selection (alpha = 0,
// or a single token): one wave (small_gate) computes g and E* as the kernel
// above does, takes the plain top-k, forms the gate weights with the same
// arithmetic and buckets the B k <= 64 assignments, with no workgroup
// barriers between the phases.
template <int kNJ>
__global__ __launch_bounds__(kWave) void reuse_gate_small_kernel(GateArgs a) {
  __shared__ SmallGateLds s;
  small_gate<kNJ>(a, a.plain_idx, a.gap, s, true);
}

// The same, ranking the tokens' logits first (small_route_gate): the
// routing launch's ranking and this gating in one single-wave launch.
template <int kNJ>
__global__ __launch_bounds__(kWave) void route_gate_small_kernel(RouteArgs ra, GateArgs a) {
  __shared__ SmallGateLds s;
  small_route_gate<kNJ>(ra, a, s, true);
}

template <bool kStaged, bool kSelect, int kG, int kS, int kNT = 0>
void launch_gate_team(const GateArgs& a, const RouteArgs& ra, hipStream_t s) {
  hipLaunchKernelGGL((reuse_gate_kernel<kStaged, kG, kS, kNT, kSelect>), dim3(1), dim3(1024), 0, s,
                     a, ra);
}

// Largest k that the teams rank by taking maxima; more go to the threshold
// search, whose length does not depend on k.  A line lies where the gating
// launches cross; MI355X, us by the search and by taking maxima: 8 tokens, 64
// experts, k = 3 / 4 / 8 / 16 5.8 / 5.8 / 6.0 / 6.0 and 5.6 / 5.9 / 6.3 / 7.0;
// 16 tokens, 128 experts, k = 7 / 8 / 16 7.5 / 7.4 / 7.6 and 7.5 / 7.5 / 8.8;
// 32 tokens, 256 experts, k = 6 / 8 / 16 12.1 / 12.2 / 12.7 and 11.9 / 12.6 /
// 15.3; 64 tokens, 128 experts, k = 8 / 13 / 16 12.6 / 12.8 / 12.8 and 10.8 /
// 12.6 / 13.5; 256 tokens, 64 experts, k = 8 / 16 24.3 / 25.5 and 17.5 / 24.8.
int team_max_k(int B, int E) {
  if (E <= 16) return B <= 8 ? 8 : kMaxTopK;
  if (B <= 8) return E <= 64 ? 3 : E <= 128 ? 6 : 7;
  if (B <= 16) return E <= 64 ? 5 : E <= 128 ? 7 : 8;
  if (B <= 32) return E <= 64 ? 12 : E <= 128 ? 8 : 6;
  return E <= 64 ? kMaxTopK : 13;
}

bool gate_by_search(const GateArgs& a) { return a.k > team_max_k(a.B, a.E); }

// Waves take 1, 2 or 4 tokens at a time, so that their searches' chains
// overlap.  Logits that are not staged are those of 41 tokens and more.
template <bool kStaged, bool kSelect, int kNJ>
void launch_gate_search(const GateArgs& a, const RouteArgs& ra, hipStream_t s) {
  if constexpr (kSelect)
    launch_gate_team<kStaged, true, 64, kNJ, 1>(a, ra, s);  // at most 16 tokens
  else if constexpr (!kStaged)
    launch_gate_team<false, false, 64, kNJ, 4>(a, ra, s);
  else if (a.B <= 16)
    launch_gate_team<true, false, 64, kNJ, 1>(a, ra, s);
  else if (a.B <= 32)
    launch_gate_team<true, false, 64, kNJ, 2>(a, ra, s);
  else
    launch_gate_team<true, false, 64, kNJ, 4>(a, ra, s);
}

// Up to 16 tokens each of the 16 waves has at most one, and a whole wave per
// token is the shorter chain (16 tokens over 128 experts: the call takes 39.8
// us against 41.4 with 16-lane rows); above, rows take four tokens a wave (32
// tokens 93.1 against 94.7 us, 64 tokens 65.9 against 72.8).  16 experts or
// fewer need one slot a lane either way.
constexpr int kWaveTeamMaxTokens = 16;

template <bool kStaged, bool kSelect>
void launch_gate_staged(const GateArgs& a, const RouteArgs& ra, hipStream_t s) {
  if (gate_by_search(a)) {
    if (a.E <= 64) launch_gate_search<kStaged, kSelect, 1>(a, ra, s);
    else if (a.E <= 128) launch_gate_search<kStaged, kSelect, 2>(a, ra, s);
    else launch_gate_search<kStaged, kSelect, 4>(a, ra, s);
    return;
  }
  if constexpr (kStaged) {
    if (a.E <= 16) return launch_gate_team<true, kSelect, 16, 1>(a, ra, s);
    if (a.B <= kWaveTeamMaxTokens) {
      if (a.E <= 64) launch_gate_team<true, kSelect, 64, 1>(a, ra, s);
      else if (a.E <= 128) launch_gate_team<true, kSelect, 64, 2>(a, ra, s);
      else launch_gate_team<true, kSelect, 64, 4>(a, ra, s);
      return;
    }
  }
  if (a.E <= 64) launch_gate_team<kStaged, kSelect, 16, 4>(a, ra, s);
  else if (a.E <= 128) launch_gate_team<kStaged, kSelect, 16, 8>(a, ra, s);
  else launch_gate_team<kStaged, kSelect, 16, 16>(a, ra, s);
}

bool small_gate_applies(const GateArgs& a) {
  return a.B <= kSmallMaxTokens && (a.alpha == 0.f || a.B == 1);
}

hipError_t launch_reuse_gate(const GateArgs& a, hipStream_t s) {
  if (small_gate_applies(a)) {
    if (a.E <= 64)
      hipLaunchKernelGGL(reuse_gate_small_kernel<1>, dim3(1), dim3(kWave), 0, s, a);
    else if (a.E <= 128)
      hipLaunchKernelGGL(reuse_gate_small_kernel<2>, dim3(1), dim3(kWave), 0, s, a);
    else
      hipLaunchKernelGGL(reuse_gate_small_kernel<4>, dim3(1), dim3(kWave), 0, s, a);
    return hipGetLastError();
  }
  const RouteArgs none{};
  if (a.B * a.E <= kStage)
    launch_gate_staged<true, false>(a, none, s);
  else
    launch_gate_staged<false, false>(a, none, s);
  return hipGetLastError();
}

// The workgroup gating kernel ranks the tokens itself, after the logits-only
// launch, up to this many of them: more would wait for the one workgroup
// longer than the launch saved.  Measured on MI355X, calls with a ranking of
// their own against this: 128 experts, where it is a launch, at 32 tokens
// 94.6 against 92.6 us, but at 64 tokens 65.7 against 66.6; 64 experts, where
// one workgroup per token also computes the logits, at 12 / 24 / 64 tokens
// 39.5 / 56.6 / 142 against 37.5 / 54.4 / 140 us, at 100 tokens 81.2 against
// 82.6, and at 64 tokens of a small layer by k = 6 / 8 / 9 / 12 / 16 30.0 /
// 30.7 / 31.7 / 33.2 / 34.0 against 29.3 / 30.5 / 31.7 / 33.8 / 35.5.
int gate_select_max_tokens(const GateArgs& a) {
  if (gate_by_search(a)) return 16;  // a token a wave
  if (a.E > 64) return 32;
  return a.E <= 16 || a.k <= 8 ? 64 : 32;
}

hipError_t launch_route_and_gate(const RouteArgs& ra, const GateArgs& a, hipStream_t s) {
  const bool small = small_gate_applies(a) && route_ranks_separately(ra);
  const bool select = (route_ranks_separately(ra) || route_rows_same_bits(ra)) &&
                      a.B * a.E <= kStage &&
                      a.B <= gate_select_max_tokens(a);
  if (!small && !select) {
    const hipError_t err = launch_route(ra, s);
    return err != hipSuccess ? err : launch_reuse_gate(a, s);
  }
  const hipError_t err = launch_route_rows(ra, s);
  if (err != hipSuccess) return err;
  if (small) {
    if (a.E <= 64)
      hipLaunchKernelGGL(route_gate_small_kernel<1>, dim3(1), dim3(kWave), 0, s, ra, a);
    else if (a.E <= 128)
      hipLaunchKernelGGL(route_gate_small_kernel<2>, dim3(1), dim3(kWave), 0, s, ra, a);
    else
      hipLaunchKernelGGL(route_gate_small_kernel<4>, dim3(1), dim3(kWave), 0, s, ra, a);
  } else {
    launch_gate_staged<true, true>(a, ra, s);
  }
  return hipGetLastError();
}

}  // namespace s2moe
