// Causal attention forward of the whole prompt that also emits the window-softmax partials of Eq. 3
// (Section 5.1; the appendix on limitations leaves kernel-level optimisation of the scoring step open).
//
// The prefill phase of a decoder computes softmax(Q K^T) V for every prompt position anyway.  The last W
// query rows of that pass are the observation-window rows whose weights Eq. 3 pools per shot, so this
// kernel writes, next to the attention output, the same per-(window row, chunk) statistic the
// stand-alone score kernel writes - log2 of the chunk's sum of exponentials - plus each window row's
// log2 denominator.  The per-shot reduction, selection and compaction kernels then run unchanged, and
// K is not read a second time for scoring.
//
// Shape: bf16, head_dim 128.  A workgroup of four waves owns 128 consecutive queries of one query head,
// each wave 32 of them, and walks the keys 0..last query in blocks of 32.
//   S^T = K_blk Q^T   v_mfma_f32_32x32x16_bf16, keys along the accumulator registers, queries along the
//                     lanes (the window queries' layout of the score kernel), so the online softmax is
//                     in-lane and its statistics are per-lane scalars.
//   O^T += V_blk^T P^T  the same instruction with d along the accumulator registers and queries still
//                     along the lanes: the weights a lane holds after the softmax ARE its B operand, and
//                     rescaling the output is a per-lane multiply.  The A operand needs V with keys
//                     contiguous; a small pre-pass packs V once into 32-key blocks [d][key] in exactly the
//                     key order the accumulator registers have.
//   precision         this product runs in fp16 (v_mfma_f32_32x32x16_f16): a weight keeps 11 significant bits
//                     instead of bf16's 8, which holds the output within 4.6e-4 of its row maximum with one
//                     instruction per step (a bf16 weight is off by up to 2^-9; bf16 hi + lo would cost a
//                     second instruction).  fp16's narrow range is dealt with by two exact power-of-two
//                     scalings: the softmax reference sits 15 below the running maximum, so weights lie
//                     in (0, 2^15] and anything above 2^-39 of the largest survives; and the pre-pass
//                     scales every KV-head plane of V so that its largest finite |v| lands in [2^14, 2^15).
//                     Sums of weights stay in fp32, add the weights before they are rounded, and carry the same
//                     reference.
// K and packed-V blocks are streamed global -> LDS with direct-to-LDS loads into a ring of three stages
// shared by the four waves (one barrier per block); the LDS layouts are bank-conflict free for the
// 128-bit operand reads (K as in the score kernel; V^T rows of 64 bytes with a two-bit XOR of the
// 16-byte column).  The grid puts the query tile in its slowest dimension, longest tiles first, so that
// every head's long tiles are dispatched before anybody's short ones.
#include "common.hpp"

namespace shotkv {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) float floatx2;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((address_space(3))) const char lds_cchar;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) const f16x8 lds_f16x8;

constexpr int kD = 128;
constexpr int kBlockKeys = 32;
constexpr int kRowBytes = kD * 2;
constexpr int kGroupBytes = 4 * kRowBytes + 64;       // K: four rows + pad = one direct-to-LDS instruction
constexpr int kKBytes = 8 * kGroupBytes;              // 8704
constexpr int kVtBytes = kD * kBlockKeys * 2;         // 8192: [128 d][32 keys] fp16
// Softmax reference = running maximum - kWeightShift (log2 domain), in every block: the largest weight is then a power
// of two, which fp16 holds exactly, and weights keep their 11 bits down to 2^-29 of it.  A reference that stays where it
// is for a while is faster, and loses precision.  One that stays until a weight passes fp16's range (8192 tokens 570 us,
// 587 as it is, 32768 7900 and 8215, whole calls) has a largest weight that is rounded, and sums that need no maximum, of
// the rounded weights, put the same error in the denominator: rows that two keys share are off by up to twice as much.  One
// with more headroom (8 below the maximum, 2^7; 8192 tokens 550) loses bits from 2^-22 on - a weight of 2^-26 is off by up
// to 0.8 %, one of 2^-30 by 11 % - and where the heaviest keys carry small values those weights make the output.
constexpr int kWeightShift = 15;
constexpr int kStageBytes = kKBytes + kVtBytes;
constexpr int kRing = 3;
constexpr int kTileQ = 128;
constexpr int kWavesQ = 4;
constexpr int kThreadsQ = kWavesQ * kWave;
constexpr int kLoadsPerWave = 4;                      // 2 K groups + 2 V^T slabs per wave per block

// ---- V packing -----------------------------------------------------------------------------------
// Largest finite |v| of every share of every KV-head plane, as bf16 bits (their order is the order of the
// magnitudes); the packing kernel takes the maximum over a plane's shares.
__global__ __launch_bounds__(256) void v_absmax_kernel(const bf16_t* __restrict__ v, int n_tokens,
                                                       uint32_t* __restrict__ v_share_max) {
  const size_t plane = blockIdx.y;
  const size_t n16 = static_cast<size_t>(n_tokens) * kD / 8;  // 16-byte pieces of the plane
  const size_t per = (n16 + gridDim.x - 1) / gridDim.x;       // a contiguous share per workgroup
  const size_t lo = blockIdx.x * per, hi = min(n16, lo + per);
  const u32x4* src = reinterpret_cast<const u32x4*>(v + plane * n_tokens * kD);
  uint32_t best = 0u;
  auto fold = [&](const u32x4& raw) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t a = raw[e] & 0x7fffu, b = (raw[e] >> 16) & 0x7fffu;
      if (a < 0x7f80u) best = max(best, a);  // infinities and NaNs do not set the scale
      if (b < 0x7f80u) best = max(best, b);
    }
  };
  size_t i = lo + threadIdx.x;
  for (; i + 3 * 256 < hi; i += 4 * 256) {  // four loads in flight per thread
    const u32x4 r0 = src[i], r1 = src[i + 256], r2 = src[i + 512], r3 = src[i + 768];
    fold(r0); fold(r1); fold(r2); fold(r3);
  }
  for (; i < hi; i += 256) fold(src[i]);
  __shared__ uint32_t wave_best[256 / kWave];
  best = wave_max(best);
  if (threadIdx.x % kWave == 0) wave_best[threadIdx.x / kWave] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 256 / kWave; ++w) best = max(best, wave_best[w]);
    v_share_max[plane * kVShares + blockIdx.x] = best;
  }
}

// The power of two that brings a plane's largest |v| (bf16 bits) into [2^14, 2^15): multiply V by
// plane_scale(bits, false) when packing, the output by plane_scale(bits, true).  Both are exact.
__device__ __forceinline__ float plane_scale(uint32_t absmax_bits, bool inverse) {
  int e = static_cast<int>(absmax_bits >> 7);  // biased exponent of the largest magnitude
  e = min(max(e, 15), 254);                    // all-zero, denormal or absurdly small planes: a fixed scale
  return __uint_as_float(static_cast<uint32_t>(inverse ? e - 14 : 268 - e) << 23);
}

// vt[p][g][block][d][c][j] = scale * V[p][g][32*block + 8*(2*(c/2) + j/4) + 4*(c%2) + j%4][d] as fp16: column
// c = 2*s + half holds, in order, the eight keys whose weights a lane of half `half` feeds to matrix step s.
// Keys past n_tokens are zero.
__global__ __launch_bounds__(256) void pack_vt_kernel(const bf16_t* __restrict__ v, int n_tokens, int n_blocks,
                                                      const uint32_t* __restrict__ v_share_max, int n_shares,
                                                      uint32_t* __restrict__ v_absmax,
                                                      uint16_t* __restrict__ vt) {
  const int blk = blockIdx.x;
  const size_t plane = blockIdx.y;  // p * H_kv + g
  uint32_t absmax = 0u;
  for (int i = threadIdx.x % kWave; i < n_shares; i += kWave) absmax = max(absmax, v_share_max[plane * kVShares + i]);
  absmax = wave_max(absmax);
  if (blk == 0 && threadIdx.x == 0) v_absmax[plane] = absmax;  // for the attention kernel
  __shared__ uint16_t tile[kBlockKeys][kD + 2];
  const float scale = plane_scale(absmax, false);
  const bf16_t* src = v + plane * n_tokens * kD;
  for (int i = threadIdx.x; i < kBlockKeys * kD / 8; i += 256) {
    const int key = i / (kD / 8), d8 = i % (kD / 8);
    const int t = blk * kBlockKeys + key;
    u32x4 raw = {0u, 0u, 0u, 0u};
    if (t < n_tokens) raw = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + static_cast<size_t>(t) * kD + d8 * 8));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const floatx2 f = {__uint_as_float(raw[e] << 16) * scale, __uint_as_float(raw[e] & 0xffff0000u) * scale};
      const f16x2 hh = __builtin_convertvector(f, f16x2);
      const uint32_t bits = __builtin_bit_cast(uint32_t, hh);
      tile[key][d8 * 8 + 2 * e] = static_cast<uint16_t>(bits & 0xffffu);
      tile[key][d8 * 8 + 2 * e + 1] = static_cast<uint16_t>(bits >> 16);
    }
  }
  __syncthreads();
  uint16_t* dst = vt + (plane * n_blocks + blk) * (kD * kBlockKeys);
  for (int i = threadIdx.x; i < kD * 4; i += 256) {  // one 16-byte column per thread
    const int d = i / 4, c = i % 4, s = c >> 1, half = c & 1;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j0 = 2 * e, j1 = 2 * e + 1;
      const int k0 = 8 * (2 * s + j0 / 4) + 4 * half + j0 % 4;
      const int k1 = 8 * (2 * s + j1 / 4) + 4 * half + j1 % 4;
      w[e] = static_cast<uint32_t>(tile[k0][d]) | (static_cast<uint32_t>(tile[k1][d]) << 16);
    }
    *reinterpret_cast<u32x4*>(dst + d * kBlockKeys + c * 8) = u32x4{w[0], w[1], w[2], w[3]};
  }
}

// ---- streaming helpers ---------------------------------------------------------------------------
__device__ __forceinline__ void load_lds(const char* base, uint32_t off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_addr), "v"(off), "s"(base)
               : "memory", "m0");
}
// Where a lane fetches from, within the KB that one instruction brings, for both kinds of block: lane l fills LDS slot
// l, and 16-byte column x of a K row (four rows to an instruction) sits in slot x ^ row, column x of a V^T row (d;
// sixteen rows to an instruction) in slot x ^ (d / 4): sixteen consecutive V^T rows, read 16 bytes each by sixteen
// lanes, then cover the 64 LDS banks exactly once.
__device__ __forceinline__ uint32_t piece_offset(int lane) { return (lane << 4) ^ ((lane >> 4) << 4); }

// K groups [g0, g0 + 2) of a block: group i fills rows 4i..4i+3.  Rows past the last token re-read it (they are masked
// by causality); only the last block of the prompt has any.
template <bool CLAMP>
__device__ __forceinline__ void issue_k(const char* __restrict__ k_plane, int key0, int n_tokens,
                                        uint32_t lds_addr, int g0, uint32_t piece, int lane) {
  const char* base = k_plane + static_cast<size_t>(key0 + 4 * g0) * kRowBytes;
  if (CLAMP && key0 + kBlockKeys > n_tokens) {
    const uint32_t col_bytes = piece & (kRowBytes - 1);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = min(4 * (g0 + i) + (lane >> 4), n_tokens - 1 - key0);
      load_lds(k_plane + static_cast<size_t>(key0) * kRowBytes, static_cast<uint32_t>(row) * kRowBytes + col_bytes,
               lds_addr + (g0 + i) * kGroupBytes);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) load_lds(base + i * 1024, piece, lds_addr + (g0 + i) * kGroupBytes);
}
// V^T slabs [i0, i0 + 2) of a packed block: slab i fills rows (d) 16i..16i+15 of 64 bytes
__device__ __forceinline__ void issue_vt(const char* __restrict__ vt_block, uint32_t lds_addr, int i0, uint32_t piece) {
#pragma unroll
  for (int i = 0; i < 2; ++i) load_lds(vt_block + (i0 + i) * 1024, piece, lds_addr + (i0 + i) * 1024);
}

__device__ __forceinline__ f16x2 to_f16x2(float x0, float x1) {
  const floatx2 f = {x0, x1};
  return __builtin_convertvector(f, f16x2);  // round to nearest even
}

// The lane number made afresh: a value that is needed again after a loop need not hold a register through it.
__device__ __forceinline__ int lane_again() {
  uint32_t zero = 0;
  asm volatile("" : "+s"(zero));
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero)));
}

struct AttentionArgs {
  const bf16_t* q;
  const bf16_t* k;
  const uint16_t* vt;
  const uint32_t* v_absmax;
  int n_tokens, n_blocks_total, H, H_kv, W;
  float c;  // softmax scale in the log2 domain
  float* o_out;
  const int32_t* shot_offsets;
  int share, n_shots, max_c, R;
  float* partial;
  float* row_stat;
};

// One tile: 128 consecutive queries from q0 on, each wave 32 of them.  EMIT: the tile may hold window rows, or end the
// prompt; its weights are kept in fp32 for the statistics.
template <bool EMIT>
__device__ __forceinline__ void attention_tile(const AttentionArgs& x, int h, int p, int q0, lds_cchar* lds_base) {
  // Operands read from LDS ahead of the matrix instructions that take them, those of O^T ahead of the softmax: as many
  // as three waves per SIMD have registers for.  Read two at a time where they are taken, as the compiler does by itself,
  // 8192 tokens take 572 us instead of 567, 1500 tokens 79 instead of 76.
  constexpr int kKAhead = 6, kVAhead = 4;
  const int n_tokens = x.n_tokens, W = x.W, R = x.R, max_c = x.max_c;
  const float c = x.c;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int G = x.H / x.H_kv, g = h / G;
  const int half = lane >> 5;
  const int wave_min_q = q0 + 32 * wave;
  const int wave_max_q = min(wave_min_q + 31, n_tokens - 1);
  const int last_q = min(q0 + kTileQ, n_tokens) - 1;
  const int n_blocks = last_q / kBlockKeys + 1;         // keys 0..last_q
  // the window rows of this wave, if any, take part in Eq. 3
  const int win0 = n_tokens - W;
  const bool wave_emits = EMIT && wave_max_q >= win0 && wave_min_q < n_tokens;
  const int q_row = wave_min_q + (lane & 31);           // this lane's query
  const int q_eff = EMIT ? min(q_row, n_tokens - 1) : q_row;  // rows past the prompt repeat the last one, unstored
  const bool lane_emits = EMIT && q_row >= win0 && q_row < n_tokens && half == 0;

  const size_t plane = static_cast<size_t>(p) * x.H_kv + g;
  const char* k_plane = reinterpret_cast<const char*>(x.k) + plane * n_tokens * kRowBytes;
  const char* vt_plane = reinterpret_cast<const char*>(x.vt) + plane * x.n_blocks_total * kVtBytes;
  // B operands of S^T: query q_eff, head-dim slice 16*ks + 8*half .. +8
  bf16x8 bq[8];
  const bf16_t* q_ptr = x.q + ((static_cast<size_t>(p) * x.H + h) * n_tokens + q_eff) * kD + half * 8;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) bq[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(q_ptr + ks * 16));
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) asm volatile("" ::"v"(bq[ks]));  // landed before the hand-tracked loads start

  const uint32_t lds_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds_base));
  const uint32_t piece = piece_offset(lane);
  auto issue = [&](int b, int slot) {
    issue_k<EMIT>(k_plane, b * kBlockKeys, n_tokens, lds_addr + slot * kStageBytes, 2 * wave, piece, lane);
    issue_vt(vt_plane + static_cast<size_t>(b) * kVtBytes, lds_addr + slot * kStageBytes + kKBytes, 2 * wave, piece);
  };

  float m_run = -INFINITY, l_run = 0.f, l_chunk = 0.f;
  floatx16 ot[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) ot[t][v] = 0.f;

  // Eq. 3 bookkeeping (emitting waves only): the segment whose sum is being collected, see max_chunks().  (Offsets
  // that are out of order give wrong statistics in range; the problem's scores are discarded.)
  // The ends of 64 segments at a time sit in the lanes, one load for all of them.
  const int32_t* off = x.shot_offsets + static_cast<size_t>(p / x.share) * (x.n_shots + 1);
  const int n_seg = wave_emits ? x.n_shots + 2 : 0;
  int ends = 0;
  auto segment_end = [&](int sg) {
    const int at = sg & (kWave - 1);
    if (at == 0) {
      const int i = sg + lane;
      ends = i <= x.n_shots ? off[i] : n_tokens;
      asm volatile("" : "+v"(ends));  // waited for here: not at every end, with the store just issued and the stream
    }
    return __builtin_amdgcn_readlane(ends, at);
  };
  int cur_c = 0, cur_s = 0, cur_e = wave_emits ? segment_end(0) : 0;
  const int h_local = h - g * G;
  float* part_row = x.partial + plane * max_c * R + h_local * W + (q_row - win0);  // + segment * R
  auto finish_chunk = [&]() {
    const float tot = sum_across_halves(l_chunk);
    if (lane_emits) part_row[static_cast<size_t>(cur_c) * R] = tot > 0.f ? add_log2(m_run, tot) : -INFINITY;
    l_chunk = 0.f;
    ++cur_c;
    if (cur_c < n_seg) { cur_s = cur_e; cur_e = segment_end(cur_c); }
  };

  issue(0, 0);
  if (n_blocks > 1) issue(1, 1);
  // where a lane reads the first operand of S^T and of O^T in a stage: 16-byte column half of row lane % 32, XOR-swizzled
  const uint32_t k_read = (lane & 31) * kRowBytes + ((lane & 31) >> 2) * 64 + ((half ^ (lane & 3)) << 4);
  const uint32_t v_read = (lane & 31) * 64 + ((half ^ ((lane >> 2) & 3)) << 4);
  int slot = 0, slot2 = 2;  // of blocks b and b + 2
  for (int b = 0; b < n_blocks; ++b) {
    // this wave's loads of block b have landed once only those of block b+1 can be outstanding
    if (b + 1 < n_blocks) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoadsPerWave) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // ... and after the barrier so have the other waves'; everybody is also done with block b-1
    asm volatile("s_barrier" ::: "memory");
    if (b + 2 < n_blocks) issue(b + 2, slot2);
    const uint32_t blk = lds_addr + slot * kStageBytes;
    slot = slot + 1 == kRing ? 0 : slot + 1;
    slot2 = slot2 + 1 == kRing ? 0 : slot2 + 1;
    const int key0 = b * kBlockKeys;
    const bool has_work = key0 <= wave_max_q;
    if (!has_work && !wave_emits) continue;
    floatx16 acc;
    f16x8 p16[2];
    f16x8 va[8];  // A operands of O^T: step i % 2 of head-dim rows 32 * (i / 2) ..
    uint32_t v_even = blk + kKBytes + v_read;
    asm("" : "+v"(v_even));
    auto load_v = [&](int i) {
      return *reinterpret_cast<lds_f16x8*>(static_cast<uintptr_t>((i & 1 ? v_even ^ 32 : v_even) + 2048 * (i >> 1)));
    };
    if (has_work) {
      // ---- S^T: keys along registers (row 8*(v/4) + 4*half + v%4), queries along lanes -------------
      uint32_t even = blk + k_read, odd;
      asm("" : "+v"(even));  // one register through the loop, not one for each
      odd = even ^ 32;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const bf16x8 a = *reinterpret_cast<lds_bf16x8*>(static_cast<uintptr_t>(((ks & 1) ? odd : even) + 64 * (ks >> 1)));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bq[ks], acc, 0, 0, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, kKAhead, 0);
#pragma unroll
      for (int i = 0; i < 8 - kKAhead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kKAhead, 0);
      // ---- causal mask, online softmax ---------------------------------------------------------
      if (key0 + kBlockKeys - 1 > wave_min_q) {
        const int limit = q_eff - key0 + 1 - 4 * half;  // rows below this are visible
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (8 * (v >> 2) + (v & 3) >= limit) acc[v] = -INFINITY;
      }
#pragma unroll
      for (int i = 0; i < kVAhead; ++i) va[i] = load_v(i);
      __builtin_amdgcn_sched_barrier(0);
      float bm = max_of_two(acc[0], acc[1]);
#pragma unroll
      for (int v = 2; v < 16; v += 2) bm = fmaxf(fmaxf(bm, acc[v]), acc[v + 1]);
      const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
      bm = max_of_two(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
      // (max_of_two and sums that start from the first weights: seven vector instructions of a block, which wait for one
      // another; whole calls, 8192 tokens 561 and 551 us, 32768 7870 and 7750, 1500 73.8 and 72.5, 8 of 5000 with 8 heads
      // 461 and 452)
      // finite from the first block on: key 0 is always visible
      const float m_new = max_of_two(m_run, fmaf(bm, c, -static_cast<float>(kWeightShift)));
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // 0 from -inf
        l_run *= alpha;
        if (EMIT) l_chunk *= alpha;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int v = 0; v < 16; ++v) ot[t][v] *= alpha;
        m_run = m_new;
      }
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float w0 = __builtin_amdgcn_exp2f(fmaf(acc[v], c, -m_run));
        const float w1 = __builtin_amdgcn_exp2f(fmaf(acc[v + 1], c, -m_run));
        const f16x2 w = to_f16x2(w0, w1);
        p16[v / 8][v % 8] = w[0];
        p16[v / 8][v % 8 + 1] = w[1];
        s0 = v == 0 ? w0 : s0 + w0;  // (zero and a weight is an addition that the compiler keeps)
        s1 = v == 0 ? w1 : s1 + w1;
        if (EMIT) {  // the statistics take the weights as well
          acc[v] = w0;
          acc[v + 1] = w1;
        }
      }
      l_run += s0 + s1;
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    }
    // ---- Eq. 3: this block's weights credited to the chunks it overlaps --------------------------
    // The tiles with window rows are the longest and wait for the waves that do this, three instructions per weight and
    // segment.  Whole call, with compares against both ends of a segment and a scalar load at each, and this: 8192 tokens in
    // 2000 units 1276 and 963 us, in 320 640 and 621; 5000 tokens of 8 heads in 600 units 429 and 318, in 27 shots 204 and
    // 169; with compares and all vector memory waited for at every end 469 and 176.
    if (cur_c < n_seg && cur_s <= key0 && cur_e >= key0 + kBlockKeys) {  // one segment: the sum below without masks
      float sum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) sum += acc[v];
      l_chunk += sum;
      if (cur_e == key0 + kBlockKeys) finish_chunk();
    } else if (wave_emits) {
      while (cur_c < n_seg && cur_s < key0 + kBlockKeys) {
        // the segment's rows of the block, a bit each; this lane holds rows 4 * half + 8 * (v / 4) + v % 4
        auto below = [](int n) { return n > 0 ? ~0u >> (kBlockKeys - n) : 0u; };
        const uint32_t rows = (below(min(cur_e - key0, kBlockKeys)) & ~below(cur_s - key0)) >> (4 * half);
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int in = __builtin_amdgcn_sbfe(static_cast<int>(rows), 8 * (v >> 2) + (v & 3), 1);  // all ones or zeros
          sum += __int_as_float(__float_as_int(acc[v]) & in);
        }
        l_chunk += sum;
        if (cur_e <= key0 + kBlockKeys) finish_chunk();
        else break;
      }
    }
    // ---- O^T += V_blk^T P^T in fp16 -------------------------------------------------------------------
    if (has_work) {
#pragma unroll
      for (int i = kVAhead; i < 8; ++i) va[i] = load_v(i);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        ot[i >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[i], p16[i & 1], ot[i >> 1], 0, 0, 0);
#pragma unroll
      for (int i = kVAhead; i < 8; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kVAhead, 1);
    }
  }

  // ---- results -------------------------------------------------------------------------------------
  if (wave_emits) {
    // chunks that reach past this tile's keys hold what their visible part gave; later ones nothing
    while (cur_c < n_seg) finish_chunk();
    const float l_row = sum_across_halves(l_run);
    if (lane_emits) x.row_stat[plane * R + h_local * W + (q_row - win0)] = add_log2(m_run, l_row);
  }
  // undoes V's scale; applied after the normalisation, because up / l_tot can fall below the normal range
  const float up = plane_scale(x.v_absmax[plane], true);
  const float l_tot = sum_across_halves(l_run);
  const int row_out = wave_min_q + (lane_again() & 31);
  if (!EMIT || row_out < n_tokens) {
    const float inv = 1.f / l_tot;
    float* dst = x.o_out + ((static_cast<size_t>(p) * x.H + h) * n_tokens + row_out) * kD + 4 * (lane_again() >> 5);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<float4*>(dst + 32 * t + 8 * a) =
            make_float4(ot[t][4 * a] * inv * up, ot[t][4 * a + 1] * inv * up, ot[t][4 * a + 2] * inv * up,
                        ot[t][4 * a + 3] * inv * up);
  }
}

// n_plain tiles of queries that are not in the window, then the rest; the longest first.
//
// Bound by matrix and vector issue, which add up, at a power-limited clock.  Operands read ahead of the softmax, segment
// ends in the lanes, 168 registers and the heads of all problems in one order for the XCDs; whole call, 32 query / 8 KV
// heads, without all of that and with it: 1500 tokens 87 and 73 us, 3000 156 and 135, 8192 588 and 570, 32768 8080 and
// 7930; 8 problems of 5000 with 8 heads 508 and 476.  Outputs are the same bits.  Waves of 64 queries, which read LDS half
// as often, have registers for two per SIMD: 3 - 5 % faster at 32768 tokens, but 6 % slower at 6000 and slower in most
// calls below (measured with a reference that stays), so there is one kernel.
__global__ __launch_bounds__(kThreadsQ, 3) void attention_scores_kernel(AttentionArgs x, int n_plain) {
  __shared__ __attribute__((aligned(64))) char lds[kRing][kStageBytes];
  lds_cchar* lds_base = (lds_cchar*)&lds[0][0];
  // Workgroups are dealt to the eight XCDs round-robin: query heads that read one KV head go to one XCD, whose L2
  // then holds that head's K and V once instead of every XCD all of them (8192 tokens 601 -> 596 us, 20000 tokens
  // 3262 -> 3137, 32768 tokens 8618 -> 8236, 64 heads at 6000 tokens 672 -> 638).  Where the heads of all problems
  // together are no multiple of eight they keep their order.
  const int total = gridDim.x * gridDim.y;
  int head = blockIdx.x + gridDim.x * blockIdx.y;
  if (total % 8 == 0) head = (head % 8) * (total / 8) + head / 8;
  const int p = head / gridDim.x, h = head - p * gridDim.x;
  const int tile = gridDim.z - 1 - blockIdx.z;  // long tiles first, for all heads and problems
  if (tile < n_plain) attention_tile<false>(x, h, p, tile * kTileQ, lds_base);
  else attention_tile<true>(x, h, p, tile * kTileQ, lds_base);
}

}  // namespace

bool attention_supported(const PrefillDims& d) {
  return d.dtype == SHOTKV_BF16 && d.D == kD && d.W <= kTileQ &&
         static_cast<long>(d.n_tokens) * kRowBytes < (1L << 32);
}

int attention_key_blocks(int n_tokens) { return ceil_div(n_tokens, kBlockKeys); }

hipError_t launch_pack_vt(const PrefillDims& d, const void* v, const PrefillWorkspace& w, hipStream_t s) {
  const int nb = attention_key_blocks(d.n_tokens);
  KernelTimer timer(d.timing, kKernelPackVt, s);
  // enough workgroups to fill the chip a few times over, each with at least 128 rows of a plane
  const int planes = d.P * d.H_kv;
  const int shares = max(1, min(min(ceil_div(d.n_tokens, 128), ceil_div(1024, planes)), kVShares));
  hipLaunchKernelGGL(v_absmax_kernel, dim3(shares, planes), dim3(256), 0, s, static_cast<const bf16_t*>(v),
                     d.n_tokens, w.v_share_max);
  hipLaunchKernelGGL(pack_vt_kernel, dim3(nb, d.P * d.H_kv), dim3(256), 0, s, static_cast<const bf16_t*>(v),
                     d.n_tokens, nb, w.v_share_max, shares, w.v_absmax, static_cast<uint16_t*>(w.vt));
  return hipGetLastError();
}

hipError_t launch_attention_scores(const PrefillDims& d, const void* q, const void* k, const void* vt,
                                   const int32_t* shot_offsets, float* attn_out, const PrefillWorkspace& w,
                                   hipStream_t s) {
  const int nb = attention_key_blocks(d.n_tokens);
  { KernelTimer plan_timer(d.timing, kKernelPlan, s); }  // the kernel walks the shot boundaries itself
  KernelTimer timer(d.timing, kKernelAttention, s);
  const AttentionArgs args = {static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                              static_cast<const uint16_t*>(vt), w.v_absmax, d.n_tokens, nb, d.H, d.H_kv, d.W,
                              d.sm_scale * kLog2e, attn_out, shot_offsets, d.share, d.n_shots, w.max_c, d.R, w.partial,
                              w.group_stat};
  const dim3 grid(d.H, d.P, ceil_div(d.n_tokens, kTileQ));
  hipLaunchKernelGGL(attention_scores_kernel, grid, dim3(kThreadsQ), 0, s, args, (d.n_tokens - d.W) / kTileQ);
  return hipGetLastError();
}

}  // namespace shotkv
