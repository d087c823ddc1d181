// bf16 expert FFN of large batches: weights stream from HBM to registers
// once, the tokens' activations are shared through LDS.
//
// Unit of work: 64 rows of one expert matrix pair (gate and up) or one down
// matrix, for all tokens routed to that expert (at most 256).  A workgroup is
// two groups of 4 waves; wave w of a group owns 16 rows.  The groups take the
// two halves of the reduction dimension K, dealt in runs of two steps so that
// they read consecutive kilobytes of a row tile at a time, and add their
// partial tiles through LDS at the end.  Gate-up buckets of more than 128
// tokens, whose two accumulators per tile would not fit, are halved by token
// instead: both groups then read all of K, the same weights in step.
//
// Per 32-wide K step a lane loads 16 bytes of its row of each matrix (the A
// operand of v_mfma_f32_16x16x32_bf16); the group's token tiles (B operand)
// are staged in LDS one chunk of C steps ahead, double-buffered with one
// barrier per chunk, in fragment order (16 bytes of token r, K slice g at
// block 16 g + r of a tile), so that a fragment is one contiguous read.
//
// The SwiGLU activations are kept step-major: the 32 values that K step s of
// the down projection takes from row r lie at [s][r][32].  A bucket's share
// of a step is then one contiguous run, where row-major rows a multiple of
// 4 KB apart put it all on a few L2 channels (down launch at 256 tokens over
// 7 experts of F = 14336: 270 -> 249 us).
//
// What bounds it: the weight stream, in rounds of at most two workgroups per
// compute unit (registers: 8 waves of 128).  Measured on MI355X, gate-up +
// down launch, against the register-only kernel that splits K over the waves
// of a workgroup and takes 64 tokens per pass over the weights
// (ffn_bf16.hip): H = 4096, F = 14336, 7 experts, 256 tokens 566 + 372 ->
// 329 + 220 us, 128 tokens 352 + 231 -> 308 + 165 us; row-major weights,
// H = F = 2880, 79 experts, 37 tokens 249 + 140 -> 218 + 131 us.  Contiguous
// K halves instead of dealt runs: 326 us for 300 at 64 tokens.  Deeper
// weight rings (3 or 4 chunks), 32-row units and a persistent grid with equal
// shares were 5-25 % slower.
#include "ffn_common.h"

namespace s2moe {

using namespace ffn;

namespace {

constexpr int kGroups = 2;       // wave groups of a workgroup
constexpr int kGroupWaves = 4;   // waves of a group, 16 rows each
constexpr int kGroupThreads = kGroupWaves * kWave;
constexpr int kThreads = kGroups * kGroupThreads;
constexpr int kRows = 16 * kGroupWaves;  // rows of a unit
constexpr int kLdsBlocks = 4096;         // 16-byte blocks of LDS: two workgroups fit a CU

template <bool kPacked>
__device__ __forceinline__ u32x4 load_weights(const u32x4* p, int s) {
  if (kPacked) return __builtin_nontemporal_load(p + 64 * s);
  return p[4 * s];
}

// Offset of row r's 32 activations of step s in the step-major Hh.
__device__ __forceinline__ size_t hh_offset(const FfnArgs& a, int s, int r) {
  return ((size_t)s * (a.B * (a.k + a.S)) + r) * 32;
}

// One unit with T token tiles per group (kt token parts, 1 or 2, the other
// split being over K); A chunks of activations in flight in registers.
template <int kMode, int T, int A, int C, bool kPacked>
__device__ __forceinline__ void wide_pass(const FfnArgs& a, const Segment& seg, int kt, int r0,
                                          int K, const uint16_t* W0, const uint16_t* W1,
                                          u32x4* lds) {
  constexpr int NM = kMode == 0 ? 2 : 1;
  constexpr int kBlocks = T * C * 64;  // 16-byte blocks of a chunk of one group
  constexpr int P = (kBlocks + kGroupThreads - 1) / kGroupThreads;  // per thread
  constexpr int kBuf = P * kGroupThreads;
  constexpr int kTilesPad = kBuf / (64 * C);  // staged tiles, pad included
  static_assert(kGroups * 2 * kBuf <= kLdsBlocks, "double-buffered chunks");
  static_assert(kGroupWaves * NM * T * kWave <= kLdsBlocks, "exchange of the K halves");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = wave_id();
  const int grp = wave / kGroupWaves, w = wave % kGroupWaves;
  const int rA = lane & 15, gK = lane >> 4;
  const int kk = kGroups / kt;
  const int gt = grp / kk, gk = grp % kk;  // the group's token part and K part
  const int rw = r0 + 16 * w;              // the wave's first row
  const int nks = K / 32, last = nks - 1;
  const int n_chunks = (nks + 2 * kk - 1) / (2 * kk) * (2 / C);
  // K is dealt to the K parts in runs of two steps.
  auto step_of = [&](int c, int cs) {
    const int j = c * C + cs;
    return ((j / 2) * kk + gk) * 2 + (j & 1);
  };
  const int t_first = gt * 16 * T;
  u32x4* buf = lds + grp * 2 * kBuf;

  // Staging: block q = thread + p kGroupThreads of a chunk is 16-byte block
  // q % (4 C) of token q / (4 C).
  const int th = threadIdx.x % kGroupThreads;
  const int xj = th % (4 * C), x_step = xj / 4;
  const u32x4* xs[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int tok = (th + p * kGroupThreads) / (4 * C);
    const int row = x_row(a, kMode, seg, min(t_first + tok, seg.n - 1));
    const uint16_t* X = kMode == 0 ? static_cast<const uint16_t*>(a.x) + (size_t)row * a.H
                                   : static_cast<const uint16_t*>(a.hh) + hh_offset(a, 0, row);
    xs[p] = reinterpret_cast<const u32x4*>(X) + (xj & 3);
  }
  const size_t x_stride = kMode == 0 ? 4 : hh_offset(a, 1, 0) / 8;  // blocks from step to step
  auto lds_of = [&](int p) {
    const int tok = (th + p * kGroupThreads) / (4 * C);
    return (x_step * kTilesPad + tok / 16) * 64 + (xj & 3) * 16 + (tok & 15);
  };
  const u32x4* pa[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const uint16_t* M = m == 1 ? W1 : W0;
    if (kPacked)
      pa[m] = reinterpret_cast<const u32x4*>(M) + (size_t)(rw / 16) * nks * 64 + lane;
    else
      pa[m] = reinterpret_cast<const u32x4*>(M + (size_t)(rw + rA) * K) + gK;
  }

  f32x4 acc[NM][T];
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int tt = 0; tt < T; ++tt) acc[m][tt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Steps past the end reload the last one, so every load is unconditional.
  u32x4 ring[2][NM][C];
  u32x4 stg[A][P];
  auto load_x = [&](u32x4 (&d)[P], int c) {
    const int s = min(step_of(c, x_step), last);
#pragma unroll
    for (int p = 0; p < P; ++p) d[p] = xs[p][x_stride * s];
  };
  auto load_w = [&](u32x4 (&d)[NM][C], int c) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int cs = 0; cs < C; ++cs)
        d[m][cs] = load_weights<kPacked>(pa[m], min(step_of(c, cs), last));
  };
#pragma unroll
  for (int g = 0; g < A; ++g) load_x(stg[g], g);
  load_w(ring[0], 0);
#pragma unroll
  for (int p = 0; p < P; ++p) buf[lds_of(p)] = stg[0][p];
  __syncthreads();
  for (int base = 0; base < n_chunks; base += 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int c = base + d;
      if (c >= n_chunks) break;
      // The vector-memory counter completes loads in issue order: the
      // activations are requested before the weights of the same turn, so
      // the wait for them leaves the newer weights in flight.
      load_x(stg[d % A], c + A);  // into the slot staged at the end of chunk c - 1
      load_w(ring[(d + 1) & 1], c + 1);
      pipe_barrier();
      const u32x4* b0 = buf + (c & 1) * kBuf + lane;
#pragma unroll
      for (int cs = 0; cs < C; ++cs) {
        if (step_of(c, cs) < nks) {
#pragma unroll
          for (int tt = 0; tt < T; ++tt) {
            const bf16x8 b = as_bf16x8(b0[(cs * kTilesPad + tt) * 64]);
#pragma unroll
            for (int m = 0; m < NM; ++m)
              acc[m][tt] = mfma(as_bf16x8(ring[d & 1][m][cs]), b, acc[m][tt]);
          }
        }
      }
      // The other buffer was last read in chunk c - 1, before the barrier
      // that ended it.
#pragma unroll
      for (int p = 0; p < P; ++p) buf[((c + 1) & 1) * kBuf + lds_of(p)] = stg[(d + 1) % A][p];
      __syncthreads();
    }
  }

  // K halves: tile tt is finished by the group of K half tt % 2; the other
  // group hands its partial tile over through LDS.
  if (kk > 1) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int tt = 0; tt < T; ++tt)
        if ((tt & 1) != gk) lds[((w * NM + m) * T + tt) * kWave + lane] = acc[m][tt];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int tt = 0; tt < T; ++tt) {
        if ((tt & 1) != gk) continue;
        const f32x4 p = lds[((w * NM + m) * T + tt) * kWave + lane];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[m][tt][i] += p[i];
      }
  }
  // Lane holds D[m][n] for token n = rA of each tile and rows rw + 4 gK + i.
#pragma unroll
  for (int tt = 0; tt < T; ++tt) {
    if ((tt & (kk - 1)) != gk) continue;
    const int t = t_first + tt * 16 + rA;
    if (t >= seg.n) continue;
    if (kMode == 0) {
      uint16_t* dst = static_cast<uint16_t*>(a.hh) + hh_offset(a, rw / 32, seg.base + t);
      uint32_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] = f32_to_bf16(silu(acc[0][tt][i]) * acc[NM - 1][tt][i]);
      uint2 v;
      v.x = h[0] | (h[1] << 16);
      v.y = h[2] | (h[3] << 16);
      *reinterpret_cast<uint2*>(dst + (rw & 16) + 4 * gK) = v;
    } else {
      float* dst = a.out + (size_t)out_row(a, seg, t) * a.H;
      *reinterpret_cast<f32x4*>(dst + rw + 4 * gK) = acc[0][tt];
    }
  }
}

// Token tiles are rounded up to a compiled count: chunks of two steps up to
// 4 tiles, of one above (LDS).  Gate-up keeps two accumulators per tile, so
// it stops at 8 tiles per group (128 registers a wave).
template <int kMode, bool kPacked>
__global__ __launch_bounds__(kThreads, 4) void ffn_bf16_wide_kernel(FfnArgs a) {
  __shared__ u32x4 lds[kLdsBlocks];
  Segment seg;
  int unit;
  if (!resolve_block(a, kMode, kRows, &seg, &unit) || seg.n > kMaxTokens) return;
  const int rows = kMode == 0 ? (seg.shared ? a.Fs : a.F) : a.H;
  const int K = kMode == 0 ? a.H : (seg.shared ? a.Fs : a.F);
  const size_t mat = (size_t)rows * K;
  const uint16_t *W0, *W1;
  if (kMode == 0) {
    W0 = static_cast<const uint16_t*>(seg.shared ? a.sh_gate : a.gate) + seg.id * mat;
    W1 = static_cast<const uint16_t*>(seg.shared ? a.sh_up : a.up) + seg.id * mat;
  } else {
    W0 = W1 = static_cast<const uint16_t*>(seg.shared ? a.sh_down : a.down) + seg.id * mat;
  }
  const int r0 = unit * kRows;
  const int tiles = (seg.n + 15) / 16;
  const int kt = kMode == 0 && tiles > 8 ? 2 : 1;
  const int T = (tiles + kt - 1) / kt;
  constexpr int A = kMode == 0 ? 1 : 2;
  if (T <= 1) wide_pass<kMode, 1, A, 2, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  else if (T == 2) wide_pass<kMode, 2, A, 2, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  else if (T == 3) wide_pass<kMode, 3, A, 2, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  else if (T == 4) wide_pass<kMode, 4, A, 2, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  else if (T <= 6) wide_pass<kMode, 6, A, 1, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  else if (T <= 8) wide_pass<kMode, 8, A, 1, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  if constexpr (kMode == 1) {
    if (T > 12) wide_pass<kMode, 16, A, 1, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
    else if (T > 8) wide_pass<kMode, 12, A, 1, kPacked>(a, seg, kt, r0, K, W0, W1, lds);
  }
}

template <int kMode>
hipError_t launch_wide_mode(const FfnArgs& a, hipStream_t s) {
  const dim3 grid(n_blocks(a, kMode, kRows)), block(kThreads);
  if (a.packed)
    hipLaunchKernelGGL((ffn_bf16_wide_kernel<kMode, true>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((ffn_bf16_wide_kernel<kMode, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_bf16_wide(const FfnArgs& a, hipStream_t s) {
  const hipError_t err = launch_wide_mode<0>(a, s);
  return err != hipSuccess ? err : launch_wide_mode<1>(a, s);
}

}  // namespace s2moe
