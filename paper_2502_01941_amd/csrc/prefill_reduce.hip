// Normalisation of the window-softmax partials (Section 5.1, Eq. 3): per (problem, chunk, KV head) the attention
// mass sum over the head's query rows of 2^(lse_chunk - lse_row), where lse_row is the log2 of the row's softmax
// denominator over all of its keys.
//
// A workgroup takes a tile of the chunks of one KV head.  It first combines the head's row denominators from the
// slices' statistics - a few KB that every tile of the head reads again, out of cache, which costs less than a
// launch of its own (a dependent kernel ends no earlier than 4-5 us after its predecessor) - and then sums its
// chunks, a group of lanes per chunk with 16-byte loads.  All sums are in fixed order (no atomics), so results
// are reproducible run to run.
#include "common.hpp"

namespace shotkv {

namespace {

constexpr int kMassThreads = 256;
constexpr int kMaxRows = 256;

// Sum over groups of LANES lanes, widest exchange first, off the LDS pipe.
template <int LANES>
__device__ __forceinline__ float sum_over_lanes(float x) {
  if constexpr (LANES == 1) {
    return x;
  } else {
    return sum_over_lanes<LANES / 2>(x + __uint_as_float(lane_xor<LANES / 2>(__float_as_uint(x))));
  }
}

// LANES: lanes per chunk, R / 4 rounded up to a power of two.  AHEAD: the team's first chunks are requested ahead of the
// slices' statistics.
template <int LANES, bool AHEAD>
__global__ __launch_bounds__(kMassThreads) void chunk_mass_kernel(const float* __restrict__ partial,
                                                                  const float* __restrict__ group_stat, int H_kv,
                                                                  int R, int n_valid, int n_groups, int max_c,
                                                                  int tile, float* __restrict__ chunk_mass) {
  const int g = blockIdx.y, p = blockIdx.z, tid = threadIdx.x;
  const size_t head = static_cast<size_t>(p) * H_kv + g;
  constexpr int kTeams = kMassThreads / LANES;  // lane groups: one slice, later one chunk each
  const int team = tid / LANES, row0 = 4 * (tid % LANES);
  const bool has_rows = row0 < R;

  const float* rows = partial + head * max_c * R + row0;
  const int c_end = min((static_cast<int>(blockIdx.x) + 1) * tile, max_c);
  constexpr int kChunks = 4;  // chunks a team has in flight
  float4 x[kChunks];
  auto load_chunks = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kChunks; ++j) {
      const int c = min(c0 + j * kTeams, c_end - 1);
      x[j] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (has_rows) x[j] = *reinterpret_cast<const float4*>(rows + static_cast<size_t>(c) * R);
    }
  };
  const int c_first = blockIdx.x * tile + team;
  if constexpr (AHEAD) load_chunks(c_first);

  // ---- row denominators: every team combines its share of the slices, then the teams are combined ------
  __shared__ float s_max[kTeams][4 * LANES];
  __shared__ float s_sum[kTeams][4 * LANES];
  __shared__ __attribute__((aligned(16))) float s_lse[4 * LANES];
  {
    float M[4], L[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) { M[e] = -INFINITY; L[e] = 0.f; }
    const float* stat = group_stat + head * n_groups * R + row0;
    constexpr int kBatch = 4;  // loads in flight
    for (int s0 = team; s0 < n_groups; s0 += kTeams * kBatch) {
      float4 y[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        y[j] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        const int sl = s0 + j * kTeams;
        if (has_rows && sl < n_groups) y[j] = *reinterpret_cast<const float4*>(stat + static_cast<size_t>(sl) * R);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float m = M[e];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) m = fmaxf(m, reinterpret_cast<const float*>(&y[j])[e]);
        if (m > -INFINITY) {
          L[e] *= exp2f(M[e] - m);
#pragma unroll
          for (int j = 0; j < kBatch; ++j) L[e] += exp2f(reinterpret_cast<const float*>(&y[j])[e] - m);  // 2^-inf = 0
          M[e] = m;
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) { s_max[team][row0 + e] = M[e]; s_sum[team][row0 + e] = L[e]; }
  }
  __syncthreads();
  if (tid < 4 * LANES) {
    float M = -INFINITY, L = 0.f;
#pragma unroll
    for (int t = 0; t < kTeams; ++t) M = fmaxf(M, s_max[t][tid]);
    if (M > -INFINITY)
#pragma unroll
      for (int t = 0; t < kTeams; ++t) L += s_sum[t][tid] * exp2f(s_max[t][tid] - M);
    // log2 of the row's softmax denominator; +inf for a row without keys so that its weights vanish
    s_lse[tid] = L > 0.f && tid < n_valid ? add_log2(M, L) : INFINITY;
  }
  __syncthreads();

  // ---- masses -------------------------------------------------------------------------------------------
  const float4 lse = *reinterpret_cast<const float4*>(&s_lse[row0]);
  for (int c0 = c_first; c0 < c_end; c0 += kTeams * kChunks) {
    if (!AHEAD || c0 != c_first) load_chunks(c0);
#pragma unroll
    for (int j = 0; j < kChunks; ++j) {
      float m = row0 + 0 < n_valid ? exp2f(x[j].x - lse.x) : 0.f;  // 2^-inf = 0
      m += row0 + 1 < n_valid ? exp2f(x[j].y - lse.y) : 0.f;
      m += row0 + 2 < n_valid ? exp2f(x[j].z - lse.z) : 0.f;
      m += row0 + 3 < n_valid ? exp2f(x[j].w - lse.w) : 0.f;
      m = sum_over_lanes<LANES>(m);
      const int c = c0 + j * kTeams;
      if (row0 == 0 && c < c_end) chunk_mass[(static_cast<size_t>(p) * max_c + c) * H_kv + g] = m;
    }
  }
}

}  // namespace

hipError_t launch_chunk_mass(const PrefillDims& d, int n_valid, const PrefillWorkspace& w, hipStream_t s) {
  { KernelTimer stat_timer(d.timing, kKernelRowStats, s); }  // the row denominators are part of the same kernel
  KernelTimer timer(d.timing, kKernelChunkMass, s);
  if (d.R % 4 || d.R > kMaxRows) return hipErrorInvalidValue;
  // small tiles spread few problems over the chip, large ones share the row denominators of many
  const int heads = d.P * d.H_kv;
  const int tiles = max(1, min(ceil_div(w.max_c, 32), ceil_div(2048, heads)));
  const int tile = ceil_div(w.max_c, tiles);
  const dim3 grid(ceil_div(w.max_c, tile), d.H_kv, d.P);
  // Up to one workgroup per CU the kernel is two trips to memory, so the first chunks are asked for with the statistics
  // (whole call, us, without and with: 8192 tokens in 40 shots 23.7 and 23.3, four of them 45.5 and 45.1, 32768 tokens 39.6
  // and 39.3; 384 workgroups 129.8 and 129.5).  Many workgroups all asking before the first can go on to its sums lose
  // (the kernel alone, 1216 workgroups 8.6 and 10.0, 2048 19.7 and 22.9).
  const bool ahead = grid.x * static_cast<long>(heads) <= 256;
#define SHOTKV_LAUNCH_MASS(LL)                                                                                          \
  hipLaunchKernelGGL((ahead ? chunk_mass_kernel<LL, true> : chunk_mass_kernel<LL, false>), grid, dim3(kMassThreads), 0, \
                     s, w.partial, w.group_stat, d.H_kv, d.R, n_valid, w.n_groups, w.max_c, tile, w.chunk_mass)
  if (d.R <= 32) SHOTKV_LAUNCH_MASS(8);
  else if (d.R <= 64) SHOTKV_LAUNCH_MASS(16);
  else if (d.R <= 128) SHOTKV_LAUNCH_MASS(32);
  else SHOTKV_LAUNCH_MASS(64);
#undef SHOTKV_LAUNCH_MASS
  return hipGetLastError();
}

}  // namespace shotkv
