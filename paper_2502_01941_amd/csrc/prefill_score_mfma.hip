// Window-attention softmax partials on the gfx950 matrix cores (Section 5.1, Eq. 3: alpha_{t,h}).
//
// Shape: bf16 or fp32, head_dim 64 or 128, up to 256 query rows (G*W) per KV head, instantiated for 1, 2, 4, 6
// (bf16) or 8 blocks of 32 rows; rows past G*W are zero operands whose statistics are written as -inf.
//
// A workgroup is one to eight waves (one per row block for one or two blocks and in fp32; two, or four in small
// launches, for 128 rows in bf16, two for 192 and four for 256) that take one slice of a KV head's key axis and walk it
// in blocks of 32 keys.  It finds the shot boundaries inside its slice itself (one pass over the offsets, in flight
// together with the queries and the first blocks).  Each wave keeps its share of the window queries in registers as
// MFMA B operands and computes S^T[32 keys x 32 queries] = K_blk * Q^T per row block with v_mfma_f32_32x32x16_bf16
// (fp32 inputs: six of them per step, see below).  Keys run along the accumulator registers and queries along the
// lanes, so the row-softmax statistics (max and sum over keys) are in-lane reductions; only the two lane halves are
// merged, once per chunk.  A block that contains a chunk boundary credits its weights to the chunks on either side
// with masked in-lane sums.
//
// K blocks are streamed global -> LDS with 16-byte direct-to-LDS loads (whole 256-byte rows, fully
// coalesced; each wave fetches its share of every block) into a ring of three buffers, so two blocks are
// in flight while one is being consumed; all waves read the whole block back in MFMA A-operand
// layout.  One s_barrier per block tells the waves that a block has landed and that the buffer of the
// block before it may be refilled.  With ~166 registers per wave three waves fit on a SIMD.
//
// LDS layout of a block (KeyLayout): a direct-to-LDS instruction writes 64 consecutive 16-byte slots, so a
// lane chooses which 16-byte column of its row it fetches; the choice makes the 128-bit operand reads, which
// the LDS serves sixteen lanes (rows r..r+15, one column) at a time from 64 banks, free of conflicts.
//   256-byte rows (head_dim 128): row r starts at r*256 + (r/4)*64 and column c sits in slot c ^ (r%4).  The
//     64-byte pad per four rows plus the two-bit XOR cover all banks, while the address of MFMA step ks
//     stays (lane base for ks parity) + 64*(ks/2), i.e. an immediate offset - no per-step address registers.
//   128-byte rows (head_dim 64): row r starts at r*128 and column c sits in slot c ^ ((r/2)%8): two rows
//     share the 256 bytes of the banks, so eight pairs of rows have to differ in the slot.  Half the bytes
//     and half the matrix steps per key, but the same exponentials: bound by vector issue (16 problems of
//     16001 tokens, 8 KV heads, 128 query rows: 72 us = 3.6 TB/s; plain vector arithmetic took 2427 us).
//   512-byte rows (fp32, head_dim 128): row r starts at r*512 + (r/2)*32 and column c sits in slot c ^ (r%2);
//     sixteen rows then cover the banks and every step is an immediate offset from one lane base.
//
// fp32: the matrix unit's own fp32 form takes 16 times as long per product as bf16, so both operands are split
// into three bf16 parts (split_f32) and six products of parts are summed in fp32, 0.37 of that time; the few values
// that bf16 parts cannot hold take the fp32 form (logits_block).  Splitting is as much vector work (350 instructions a
// block) as the products are matrix work, so four and eight waves split a block between them and read each other's parts
// from LDS, for a second barrier and 26 KB more LDS, where that pays (share_parts).  Error of the scores against float64 over head
// layouts, windows and 1001 .. 65000 tokens: 0.3 - 0.8e-7 of the norm.  One query block per wave (96 operand
// registers at head_dim 128), up to eight waves per workgroup.  4 problems of 4001 tokens, 8 KV heads, 128 query rows,
// head_dim 128: 33 us, 37 if each wave splits for itself, with the fp32 form 48, with plain vector arithmetic 394.  Whole
// calls, shared and each for itself: 16 of 8192 tokens 302 and 321 us, head_dim 64 4 of 9000 with 256 rows 103 and 112,
// one of 100000 with 224 rows 247 and 277.
//
// The direct-to-LDS loads are written as inline assembly and their completion is tracked by hand with
// s_waitcnt vmcnt: when they are visible to the compiler it makes every LDS read wait for all loads
// in flight, including the prefetched blocks, which serialises load and compute.  Unknown
// vector-memory operations can only make the compiler's own waits stricter, never too weak, because
// loads complete in order.
#include "common.hpp"

namespace shotkv {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float floatx2;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) const char lds_cchar;  // keeps LDS reads as ds_read, not flat
typedef __attribute__((address_space(3))) const int lds_cint;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8_out;

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float floatx4;

constexpr int kBlockKeys = 32;

// How a 32-key block lies in LDS; see the top of the file.
template <int ROW_BYTES> struct KeyLayout;
template <> struct KeyLayout<512> {
  static constexpr int kLoadBytes = 2 * 512 + 32;    // LDS stride of one direct-to-LDS instruction: two rows + pad
  // slot of lane l in instruction i: row 2i + l/32, slot l%32, which holds column (l%32) ^ (l/32)
  __device__ static uint32_t fetch_column(int, int lane) { return (lane & 31) ^ (lane >> 5); }
  __device__ static int operand_base(int row, int half) {
    return row * 512 + (row >> 1) * 32 + ((half ^ (row & 1)) << 4);
  }
  __device__ static int operand(int base, int ks) { return base + 32 * ks; }
};
template <> struct KeyLayout<256> {
  static constexpr int kLoadBytes = 4 * 256 + 64;    // four rows + pad
  // row 4i + l/16, slot l%16, which holds column (l%16) ^ (l/16)
  __device__ static uint32_t fetch_column(int, int lane) { return (lane & 15) ^ (lane >> 4); }
  __device__ static int operand_base(int row, int half) {
    return row * 256 + (row >> 2) * 64 + ((half ^ (row & 3)) << 4);
  }
  __device__ static int operand(int base, int ks) { return ((ks & 1) ? base ^ 32 : base) + 64 * (ks >> 1); }
};
template <> struct KeyLayout<128> {
  static constexpr int kLoadBytes = 8 * 128;         // eight rows
  // row 8i + l/8, slot l%8, which holds column (l%8) ^ ((row/2)%8)
  __device__ static uint32_t fetch_column(int i, int lane) { return (lane & 7) ^ ((4 * i + (lane >> 4)) & 7); }
  __device__ static int operand_base(int row, int half) { return row * 128 + ((half ^ ((row >> 1) & 7)) << 4); }
  __device__ static int operand(int base, int ks) { return base ^ (ks << 5); }
};

// Element type of Q and K with the head dimension: row sizes, operand registers and the matrix instruction.
// Step ks of a row is its 32 bytes at 32*ks; the lanes of half h hold the 16 bytes at 32*ks + 16*h of it.
template <typename T> struct Operand;                       // 16 bytes of a row as one lane holds them
template <> struct Operand<bf16_t> { typedef bf16x8 Vec; };
template <> struct Operand<float> { typedef floatx4 Vec; };
template <typename T, int D> struct Element {
  typedef typename Operand<T>::Vec Vec;
  static constexpr int kRowBytes = D * static_cast<int>(sizeof(T));
  static constexpr int kSteps = kRowBytes / 32;
  // query operand registers (vectors of 8 bf16): one per step in bf16, three parts per pair of steps in fp32
  static constexpr int kQueryVecs = sizeof(T) == 2 ? kSteps : 3 * kSteps / 2;
  static constexpr int kLoadsPerBlock = kBlockKeys * kRowBytes / 1024;  // 1 KB direct-to-LDS instructions
  static constexpr int kBufBytes = kLoadsPerBlock * KeyLayout<kRowBytes>::kLoadBytes;
  typedef KeyLayout<kRowBytes> Layout;
  // fp32: the three bf16 parts of a block lie in LDS like three bf16 blocks
  typedef KeyLayout<2 * D> PartLayout;
  static constexpr int kPartBytes = kBlockKeys * 2 * D / 1024 * PartLayout::kLoadBytes;
};
__device__ __forceinline__ floatx16 multiply_step(bf16x8 a, bf16x8 b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
// fp32 as three bf16 parts, each what the ones before leave rounded to nearest: |mid| <= 2^-8 and |lo| <= 2^-17 of the
// element's leading power of two, both of either sign, and nothing is left.  Every product of two parts is exact in
// fp32.  Of the nine the six largest are taken; the dropped mid * lo, lo * mid and lo * lo together stay below 2^-23.9
// of |q||k| per element with no preferred sign - the rounding of one fp32 multiply-add.  (Truncated parts cost the same
// instructions, but there the dropped products reach 2^-21 and all have the sign of q * k.)
// Two things a bf16 part cannot hold: infinities, as well as elements above 2^128 - 2^119, which round up to one (the
// parts behind them are NaN), and the last bits of elements below 2^-100 (logits_block).
struct Split { bf16x8 hi, mid, lo; };
__device__ __forceinline__ Split split_f32(floatx4 a, floatx4 b) {
  u32x4 h, m, l;
  auto round2 = [](float x0, float x1) __attribute__((always_inline)) {
    const floatx2 f = {x0, x1};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
  };
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x0 = e < 2 ? a[2 * e] : b[2 * e - 4], x1 = e < 2 ? a[2 * e + 1] : b[2 * e - 3];
    h[e] = round2(x0, x1);
    const float r0 = x0 - __uint_as_float(h[e] << 16), r1 = x1 - __uint_as_float(h[e] & 0xffff0000u);
    m[e] = round2(r0, r1);
    l[e] = round2(r0 - __uint_as_float(m[e] << 16), r1 - __uint_as_float(m[e] & 0xffff0000u));
  }
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
__device__ __forceinline__ floatx16 multiply_split(const Split& a, bf16x8 bh, bf16x8 bm, bf16x8 bl, floatx16 acc) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo, bh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, bm, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, bl, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, bh, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, bm, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, bh, acc, 0, 0, 0);
}
#ifndef SHOTKV_SCORE_RING
#define SHOTKV_SCORE_RING 3
#endif
#ifndef SHOTKV_SCORE_WAVES_PER_SIMD
#define SHOTKV_SCORE_WAVES_PER_SIMD 3
#endif
constexpr int kRing = SHOTKV_SCORE_RING;  // LDS buffers per workgroup: kRing - 1 blocks in flight
static_assert(kRing >= 2 && kRing <= 5, "ring depth");

// Issue this wave's share of the direct-to-LDS loads of one 32-key block: instructions [i0, i0 + NL).
// Rows past the end of the span (rem keys are left in it) re-read its last key (they are masked later), so
// every address stays inside it.
// The loads carry the non-temporal hint: K is read exactly once, and a stream that does not settle in L2
// and the memory-side cache leaves them to the statistics this kernel writes and the next kernels read
// (measured: 8 % faster here, and the per-chunk reduction that follows finds its input in cache).
template <typename E, int NL>
__device__ __forceinline__ void issue_block(const char* __restrict__ k_plane, int key0, int rem,
                                            uint32_t lds_addr, int i0, int lane) {
  typedef typename E::Layout L;
  constexpr int kRows = 1024 / E::kRowBytes;  // rows per instruction
  const int last = rem - 1;  // rem >= 1
  const char* base = k_plane + static_cast<size_t>(key0) * E::kRowBytes;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int rr = min(kRows * (i0 + i) + lane / (kWave / kRows), last);
    const uint32_t off = static_cast<uint32_t>(rr) * E::kRowBytes + (L::fetch_column(i0 + i, lane) << 4);
    // M0 = LDS address of the instruction's slots (wave-uniform); lane l lands at M0 + 16*l
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :
                 : "s"(lds_addr + (i0 + i) * L::kLoadBytes), "v"(off), "s"(base)
                 : "memory", "m0");
  }
}

// Fold the 16 logits a lane holds for one query (key rows 8*(v/4) + 4*half + v%4 of the block) into
// that query's running (reference, sum) in the log2 domain: sum = sum_k 2^(z_k - reference).
//
// Any reference gives the same softmax once the chunks are combined, so the reference found so far -
// the largest logit of some earlier block, carried over from chunk to chunk - is kept and the
// exponentials are summed against it directly.  That is safe unless a logit exceeds the reference by
// ~2^100 (or there is no reference yet); the case is caught on the sum, wave-uniformly, and the block
// is then redone as the usual online-softmax update, which raises the reference to the block maximum.
// A reference far above a chunk's logits costs nothing that the result could show: it is at most the
// row maximum, so a term that underflows against it underflows in the normalised weight as well.
// Both lane halves of a query always hold the same reference (the maximum is taken over both).
// l_grp is the sum over the workgroup's finished chunks against the same reference; it follows every
// change of the reference.
template <bool MASKED, bool EXACT>
__device__ __forceinline__ void softmax_fold(floatx16 acc, float c, int half, int rem, int key0,
                                             int last_visible, float& m_run, float& l_run, float& l_grp) {
  if (MASKED) {
    // row 8*(v/4) + v%4 + 4*half is masked when it is past the chunk or past the query's position:
    // one per-lane limit, compared against compile-time row constants
    const int limit = min(rem, last_visible - key0 + 1) - 4 * half;
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (8 * (v >> 2) + (v & 3) >= limit) acc[v] = -INFINITY;
  }
  if (!EXACT) {
    // (starting from the first two: zero and a weight is an addition that the compiler keeps)
    float s0 = __builtin_amdgcn_exp2f(fmaf(acc[0], c, -m_run)), s1 = __builtin_amdgcn_exp2f(fmaf(acc[1], c, -m_run));
#pragma unroll
    for (int v = 2; v < 16; v += 2) {
      s0 += __builtin_amdgcn_exp2f(fmaf(acc[v], c, -m_run));
      s1 += __builtin_amdgcn_exp2f(fmaf(acc[v + 1], c, -m_run));
    }
    const float s = s0 + s1;
    // wave-uniform decision, so the exact path below is taken by all lanes or none (a lane without a
    // reference yet gets inf or NaN here)
    if (__builtin_amdgcn_ballot_w64(!(s < 0x1p100f)) == 0) {
      l_run += s;
      return;
    }
  }
  float bm = fmaxf(acc[0], acc[1]);
#pragma unroll
  for (int v = 2; v < 16; v += 2) bm = fmaxf(fmaxf(bm, acc[v]), acc[v + 1]);
  bm = max_across_halves(bm);
  const float m_new = fmaxf(m_run, bm * c);
  const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
  float s0 = 0.f, s1 = 0.f;
#pragma unroll
  for (int v = 0; v < 16; v += 2) {
    s0 += __builtin_amdgcn_exp2f(fmaf(acc[v], c, -m_safe));
    s1 += __builtin_amdgcn_exp2f(fmaf(acc[v + 1], c, -m_safe));
  }
  l_run = l_run * alpha + (s0 + s1);
  l_grp *= alpha;
  m_run = m_new;
}

// Where the wave's queries lie in memory, and whether their logits may be taken from bf16 parts (fp32 only): every
// query element is zero or between 2^-100 and 2^50, so that its parts are exact and that what a tiny key element's
// parts lose (below 2^-126) cannot show, and the scale is below 2^30.
template <typename T> struct Queries {
  const T* rows;
  int qb0, n_rows;
  bool plain;
};

// S^T of one 32-key block and this wave's NQW query blocks.  fp32: from the bf16 parts; an infinite key element, or one
// that rounds up to infinity, makes its logits NaN, and the block is then taken again in the matrix unit's fp32 form,
// as every block is for queries that are not plain.
//
// SHARED (fp32): the workgroup's waves have put the block's bf16 parts at `parts` (split_block); otherwise every wave splits
// for itself.  (A null pointer would not tell: it is the address of the first LDS variable.)
template <typename T, int D, int NQW, bool SHARED>
__device__ __forceinline__ void logits_block(lds_cchar* lds_buf, lds_cchar* parts, const bf16x8 (&bq)[NQW][Element<T, D>::kQueryVecs],
                                             const Queries<T>& src, int lane, floatx16 (&acc)[NQW]) {
  typedef typename Element<T, D>::Layout L;
  typedef typename Element<T, D>::Vec Vec;
  typedef __attribute__((address_space(3))) const Vec lds_vec;
  const int base = L::operand_base(lane & 31, lane >> 5);
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQW; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
  };
  clear();
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int ks = 0; ks < Element<T, D>::kSteps; ++ks) {
      const Vec a = *reinterpret_cast<lds_vec*>(lds_buf + L::operand(base, ks));
#pragma unroll
      for (int q = 0; q < NQW; ++q) acc[q] = multiply_step(a, bq[q][ks], acc[q]);
    }
  } else {
    if (src.plain) {
      typedef typename Element<T, D>::PartLayout P;
      const int part_base = P::operand_base(lane & 31, lane >> 5);
#pragma unroll
      for (int kp = 0; kp < Element<T, D>::kSteps / 2; ++kp) {
        Split a;
        if constexpr (SHARED) {
          lds_cchar* at = parts + P::operand(part_base, kp);
          a.hi = *reinterpret_cast<lds_bf16x8*>(at);
          a.mid = *reinterpret_cast<lds_bf16x8*>(at + Element<T, D>::kPartBytes);
          a.lo = *reinterpret_cast<lds_bf16x8*>(at + 2 * Element<T, D>::kPartBytes);
        } else {
          const Vec a0 = *reinterpret_cast<lds_vec*>(lds_buf + L::operand(base, 2 * kp));
          const Vec a1 = *reinterpret_cast<lds_vec*>(lds_buf + L::operand(base, 2 * kp + 1));
          a = split_f32(a0, a1);
        }
#pragma unroll
        for (int q = 0; q < NQW; ++q)
          acc[q] = multiply_split(a, bq[q][3 * kp], bq[q][3 * kp + 1], bq[q][3 * kp + 2], acc[q]);
      }
      float any = acc[0][0];  // NaN if one of the logits is
#pragma unroll
      for (int q = 0; q < NQW; ++q)
#pragma unroll
        for (int v = 0; v < 16; v += 2)
          any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(any, acc[q][v]), acc[q][v + 1]);
      if (__builtin_amdgcn_ballot_w64(any != any) == 0) return;
      clear();
    }
#pragma clang loop unroll(disable)
    for (int ks = 0; ks < Element<T, D>::kSteps; ++ks) {
      const Vec a = *reinterpret_cast<lds_vec*>(lds_buf + L::operand(base, ks));
#pragma unroll
      for (int q = 0; q < NQW; ++q) {
        const int qi = (src.qb0 + q) * 32 + (lane & 31);
        Vec b = {0.f, 0.f, 0.f, 0.f};
        if (qi < src.n_rows) b = *reinterpret_cast<const Vec*>(src.rows + qi * D + ks * 8 + (lane >> 5) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc[q], 0, 0, 0);
      }
    }
  }
}

// fp32: this wave's share of splitting a block for all waves of the workgroup: pairs of steps wave, wave + WAVES, ...
// Every lane takes the elements that it needs as an operand, so the parts keep the operands' order.
template <int D, int WAVES>
__device__ __forceinline__ void split_block(lds_cchar* lds_buf, lds_char* parts, int wave, int lane) {
  typedef Element<float, D> E;
  typedef __attribute__((address_space(3))) const floatx4 lds_floatx4;
  const int base = E::Layout::operand_base(lane & 31, lane >> 5);
  const int part_base = E::PartLayout::operand_base(lane & 31, lane >> 5);
  constexpr int kPairs = E::kSteps / 2;
#pragma unroll
  for (int i = 0; i < (kPairs + WAVES - 1) / WAVES; ++i) {
    const int kp = wave + i * WAVES;
    if (kPairs % WAVES != 0 && kp >= kPairs) break;
    const Split a = split_f32(*reinterpret_cast<lds_floatx4*>(lds_buf + E::Layout::operand(base, 2 * kp)),
                              *reinterpret_cast<lds_floatx4*>(lds_buf + E::Layout::operand(base, 2 * kp + 1)));
    lds_char* at = parts + E::PartLayout::operand(part_base, kp);
    *reinterpret_cast<lds_bf16x8_out*>(at) = a.hi;
    *reinterpret_cast<lds_bf16x8_out*>(at + E::kPartBytes) = a.mid;
    *reinterpret_cast<lds_bf16x8_out*>(at + 2 * E::kPartBytes) = a.lo;
  }
}

// One 32-key block against this wave's NQW query blocks.
template <typename T, int D, int NQW, bool SHARED, bool MASKED, bool EXACT>
__device__ __forceinline__ void compute_block(lds_cchar* lds_buf, lds_cchar* parts, const bf16x8 (&bq)[NQW][Element<T, D>::kQueryVecs],
                                              const Queries<T>& src, int lane, int key0, int rem, int causal_base, int W, float c,
                                              float (&m_run)[NQW], float (&l_run)[NQW], float (&l_grp)[NQW]) {
  const int row = lane & 31, half = lane >> 5;
  floatx16 acc[NQW];
  logits_block<T, D, NQW, SHARED>(lds_buf, parts, bq, src, lane, acc);
#pragma unroll
  for (int q = 0; q < NQW; ++q) {
    const int last_visible = causal_base + ((src.qb0 + q) * 32 + row) % W;
    softmax_fold<MASKED, EXACT>(acc[q], c, half, rem, key0, last_visible, m_run[q], l_run[q], l_grp[q]);
  }
}

// The same block when a chunk ends inside it: the exact online-softmax update, then the sixteen weights
// 2^(z - reference) of every query stay in `e` so that the caller can credit them to the chunks on either
// side of each boundary.  Nothing is added to l_run here.
template <typename T, int D, int NQW, bool SHARED, bool MASKED>
__device__ __forceinline__ void weights_block(lds_cchar* lds_buf, lds_cchar* parts, const bf16x8 (&bq)[NQW][Element<T, D>::kQueryVecs],
                                              const Queries<T>& src, int lane, int key0, int rem, int causal_base, int W, float c,
                                              float (&m_run)[NQW], float (&l_run)[NQW], float (&l_grp)[NQW],
                                              floatx16 (&e)[NQW]) {
  const int row = lane & 31, half = lane >> 5;
  logits_block<T, D, NQW, SHARED>(lds_buf, parts, bq, src, lane, e);
#pragma unroll
  for (int q = 0; q < NQW; ++q) {
    if (MASKED) {
      const int last_visible = causal_base + ((src.qb0 + q) * 32 + row) % W;
      const int limit = min(rem, last_visible - key0 + 1) - 4 * half;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (8 * (v >> 2) + (v & 3) >= limit) e[q][v] = -INFINITY;
    }
    float bm = fmaxf(e[q][0], e[q][1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) bm = fmaxf(fmaxf(bm, e[q][v]), e[q][v + 1]);
    bm = max_across_halves(bm);
    const float m_new = fmaxf(m_run[q], bm * c);
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run[q] - m_safe);
    l_run[q] *= alpha;
    l_grp[q] *= alpha;
    m_run[q] = m_new;
#pragma unroll
    for (int v = 0; v < 16; ++v) e[q][v] = __builtin_amdgcn_exp2f(fmaf(e[q][v], c, -m_safe));
  }
}

// Crediting the weights of a block to the chunks on either side of a boundary.  A lane holds key rows
// 8*i + 4*half + v of the block in elements 4*i + v, so eight consecutive rows are four elements of both lane halves: a
// group.  Groups without a boundary are added whole; in one with a boundary the elements of an interval are added under an
// execution mask.  A boundary is the same for the whole wave, so "row r of the group lies in the interval" is bit r of a
// scalar, rows 0..3 of it the lower lane half's and 4..7 the upper one's: s_bfe_i32 gives 0 or -1 for exec_lo / exec_hi,
// and no vector compares or selects are needed.  The two scalar instructions per element are what masked adds cost: with
// all sixteen elements masked for every interval a block with an end took 73 of them on average where units are 25 tokens,
// and 20 so (and 26 vector adds instead of 36).  This kernel, 8 problems of 16384 tokens in 600 units, per KV head, 83.5
// and 74.0 us; 16 x 16001 tokens of head_dim 64 in 80 units 75.1 and 71.4; whole calls, 16 x 8192 of head_dim 64 in units
// of 6 tokens 177 and 150, 2 x 32768 in units of 15 108 and 101.  Weights of such a block against the carried reference,
// without the block's maximum, are slower (sentences 142.9 and 145.5, head_dim 64 115 and 139).
#define SHOTKV_MASKED_STEP2(V, U, ACC_A, ACC_B, XA, XB)                       \
  "s_bfe_i32 exec_lo, %[m], 0x1000" #V "\n\t"                                \
  "s_bfe_i32 exec_hi, %[m], 0x1000" #U "\n\t"                                \
  "v_add_f32 %[" #ACC_A "], %[" #ACC_A "], %[" #XA "]\n\t"                    \
  "v_add_f32 %[" #ACC_B "], %[" #ACC_B "], %[" #XB "]\n\t"
#define SHOTKV_MASKED_STEP1(V, U, ACC_A, XA)                                  \
  "s_bfe_i32 exec_lo, %[m], 0x1000" #V "\n\t"                                \
  "s_bfe_i32 exec_hi, %[m], 0x1000" #U "\n\t"                                \
  "v_add_f32 %[" #ACC_A "], %[" #ACC_A "], %[" #XA "]\n\t"

// sums += the rows of a group that `rows` names
__device__ __forceinline__ void masked_add4(float& a, float& b, float a0, float a1, float a2, float a3, float b0, float b1,
                                            float b2, float b3, uint32_t rows) {
  uint64_t save;
  asm volatile("s_mov_b64 %[save], exec\n\t"
               SHOTKV_MASKED_STEP2(0, 4, a, b, a0, b0) SHOTKV_MASKED_STEP2(1, 5, a, b, a1, b1)
               SHOTKV_MASKED_STEP2(2, 6, a, b, a2, b2) SHOTKV_MASKED_STEP2(3, 7, a, b, a3, b3)
               "s_mov_b64 exec, %[save]"
               : [a] "+v"(a), [b] "+v"(b), [save] "=&s"(save)
               : [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3), [b0] "v"(b0), [b1] "v"(b1), [b2] "v"(b2),
                 [b3] "v"(b3), [m] "s"(rows)
               : "scc");
}
__device__ __forceinline__ void masked_add4(float& a, float a0, float a1, float a2, float a3, uint32_t rows) {
  uint64_t save;
  asm volatile("s_mov_b64 %[save], exec\n\t"
               SHOTKV_MASKED_STEP1(0, 4, a, a0) SHOTKV_MASKED_STEP1(1, 5, a, a1)
               SHOTKV_MASKED_STEP1(2, 6, a, a2) SHOTKV_MASKED_STEP1(3, 7, a, a3)
               "s_mov_b64 exec, %[save]"
               : [a] "+v"(a), [save] "=&s"(save)
               : [a0] "v"(a0), [a1] "v"(a1), [a2] "v"(a2), [a3] "v"(a3), [m] "s"(rows)
               : "scc");
}
#undef SHOTKV_MASKED_STEP2
#undef SHOTKV_MASKED_STEP1

// sum[q] += the rows of group i of e[q] that `rows` names
template <int NQW>
__device__ __forceinline__ void credit_rows(const floatx16 (&e)[NQW], int i, uint32_t rows, float (&sum)[NQW]) {
#pragma unroll
  for (int q = 0; q + 1 < NQW; q += 2)
    masked_add4(sum[q], sum[q + 1], e[q][4 * i], e[q][4 * i + 1], e[q][4 * i + 2], e[q][4 * i + 3], e[q + 1][4 * i],
                e[q + 1][4 * i + 1], e[q + 1][4 * i + 2], e[q + 1][4 * i + 3], rows);
  if (NQW & 1) {
    constexpr int q = NQW - 1;
    masked_add4(sum[q], e[q][4 * i], e[q][4 * i + 1], e[q][4 * i + 2], e[q][4 * i + 3], rows);
  }
}

constexpr int kEndCache = 128;  // shot boundaries of a slice kept in LDS

template <typename T, int D, int NQB, int WAVES, bool SHARED>
struct GroupShape {
  static constexpr int kWaves = WAVES;                                      // waves per workgroup
  static constexpr int kNQW = NQB / kWaves;                                 // query blocks per wave
  static constexpr int kLoads = Element<T, D>::kLoadsPerBlock / kWaves;     // load instructions per wave per block
  static_assert(NQB % kWaves == 0 && Element<T, D>::kLoadsPerBlock % kWaves == 0, "even shares");
  static constexpr int kThreads = kWaves * kWave;
  // Waves per SIMD the registers are budgeted for: what the query operands leave room for (bf16, head_dim 128:
  // three waves with up to two query blocks per wave, two with more), and no more than the LDS admits.
  static constexpr int kQueryRegs = kNQW * Element<T, D>::kQueryVecs * 4;
  static constexpr int kRegWaves =
      (kQueryRegs > 64 || kNQW > 2) ? 2 : kQueryRegs > 32 ? SHOTKV_SCORE_WAVES_PER_SIMD : SHOTKV_SCORE_WAVES_PER_SIMD + 1;
  static constexpr int kPartsBytes = SHARED ? 3 * Element<T, D>::kPartBytes : 16;
  static constexpr int kLdsWaves = 160 * 1024 / (kRing * Element<T, D>::kBufBytes + kPartsBytes + 1024) * kWaves / 4;
  static constexpr int kMinWavesPerSimd = kLdsWaves < 1 ? 1 : kLdsWaves < kRegWaves ? kLdsWaves : kRegWaves;
};

template <typename T, int D, int NQB, int WAVES, bool SHARED>
__global__ __launch_bounds__((GroupShape<T, D, NQB, WAVES, SHARED>::kThreads),
                             (GroupShape<T, D, NQB, WAVES, SHARED>::kMinWavesPerSimd)) void
score_partials_mfma_kernel(
    const T* __restrict__ q_obs, const T* __restrict__ k, int n_tokens, int H, int H_kv, int W,
    int n_rows, float c, const int32_t* __restrict__ shot_offsets, int share, int n_shots, int group_keys,
    int max_c, float* __restrict__ partial, float* __restrict__ group_stat) {
  typedef GroupShape<T, D, NQB, WAVES, SHARED> S;
  typedef Element<T, D> E;
  constexpr int NQW = S::kNQW;
  constexpr int R = NQB * 32;
  __shared__ __attribute__((aligned(64))) char lds[kRing][E::kBufBytes];
  __shared__ __attribute__((aligned(64))) char lds_parts[S::kPartsBytes];
  __shared__ int s_end[kEndCache];
  __shared__ int s_count[S::kWaves][2];

  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = blockIdx.y, p = blockIdx.z;
  const int32_t* off = shot_offsets + static_cast<size_t>(p / share) * (n_shots + 1);
  const int k_begin = blockIdx.x * group_keys, k_end = min(k_begin + group_keys, n_tokens);
  const char* k_plane =
      reinterpret_cast<const char*>(k) + (static_cast<size_t>(p) * H_kv + g) * n_tokens * E::kRowBytes;
  const int G = H / H_kv;
  const T* q_rows = q_obs + (static_cast<size_t>(p) * H + static_cast<size_t>(g) * G) * W * D;
  float* out = partial + (static_cast<size_t>(p) * H_kv + g) * max_c * R;  // chunk c of this head: + c * R
  const int qb0 = wave * NQW;

  // B operands: query row (qb0+q)*32 + lane%32, the lane half's 16 bytes of every step
  // Query rows past n_rows = G*W (a row count that is not one of the instantiated ones) are zero operands; their
  // statistics are written as -inf, so they carry no weight further down.
  constexpr int kVec = 16 / sizeof(T);
  bf16x8 bq[NQW][E::kQueryVecs];
  // of the query elements' magnitudes, fp32 only: the largest, and the smallest as twice its bits less one (a zero wraps
  // to the top); an element costs two instructions
  float largest = 0.f;
  uint32_t smallest = UINT32_MAX;
#pragma unroll
  for (int q = 0; q < NQW; ++q) {
    const int qi = (qb0 + q) * 32 + (lane & 31);
    auto query = [&](int ks) __attribute__((always_inline)) {
      u32x4 raw = {0u, 0u, 0u, 0u};
      if (qi < n_rows) raw = *reinterpret_cast<const u32x4*>(q_rows + qi * D + ks * (2 * kVec) + (lane >> 5) * kVec);
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          largest = fmaxf(largest, fabsf(__uint_as_float(raw[e])));  // (NaNs are found in the logits)
          smallest = min(smallest, (raw[e] << 1) - 1u);
        }
      }
      return __builtin_bit_cast(typename E::Vec, raw);
    };
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int ks = 0; ks < E::kSteps; ++ks) bq[q][ks] = query(ks);
    } else {
#pragma unroll
      for (int kp = 0; kp < E::kSteps / 2; ++kp) {
        const Split b = split_f32(query(2 * kp), query(2 * kp + 1));
        bq[q][3 * kp] = b.hi;
        bq[q][3 * kp + 1] = b.mid;
        bq[q][3 * kp + 2] = b.lo;
      }
    }
  }
  Queries<T> src{q_rows, qb0, n_rows, true};
  if constexpr (sizeof(T) == 4)
    src.plain = __builtin_amdgcn_ballot_w64(largest > 0x1p50f || smallest < 2 * __float_as_uint(0x1p-100f) - 1u) == 0 &&
                c < 0x1p30f;
  lds_cchar* lds_base = (lds_cchar*)&lds[0][0];
  const uint32_t lds_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds_base));
  const int causal_base = n_tokens - W;
  const int g0 = wave * S::kLoads;

  // The slice is walked in blocks of 32 keys that take no notice of chunk boundaries: a block that contains a
  // boundary credits its weights to the chunks on either side with masked in-lane sums (sentence-sized units end
  // inside most blocks, shots of hundreds of tokens inside few), and no block carries padding except the last.
  // `cur` sits in ring slot cur_buf; up to kLook = kRing - 1 requested blocks follow it in the next slots.
  // A new block is requested each iteration, right after the barrier that frees the slot of the block
  // before cur.
  constexpr int kLook = kRing - 1;
  auto ring_slot = [](int sl) { return sl >= kRing ? sl - kRing : sl; };
  int cur_key0 = k_begin, next_key0 = k_begin + kBlockKeys;  // next block to request
  issue_block<E, S::kLoads>(k_plane, k_begin, k_end - k_begin, lds_addr, g0, lane);
  int n_q = 0;
#pragma unroll
  for (int i = 0; i < kLook - 1; ++i) {
    if (next_key0 < k_end) {
      issue_block<E, S::kLoads>(k_plane, next_key0, k_end - next_key0, lds_addr + (i + 1) * E::kBufBytes, g0, lane);
      n_q = i + 1;
      next_key0 += kBlockKeys;
    }
  }

  // Shot boundaries: segment of a key = offsets that are not above it.  The ends inside the slice go to LDS, one
  // read per boundary instead of a dependent trip to memory.  (Offsets that are out of order give a wrong but
  // harmless set of chunk numbers in range; the problem's scores are discarded.)
  int seg0 = 0, seg1 = 0;
  constexpr int kOffBatch = 8;  // loads in flight
#pragma clang loop unroll(disable)
  for (int i0 = wave * kWave; i0 <= n_shots; i0 += S::kThreads * kOffBatch) {
    int o[kOffBatch];
#pragma unroll
    for (int j = 0; j < kOffBatch; ++j) o[j] = off[min(i0 + j * S::kThreads + lane, n_shots)];
#pragma unroll
    for (int j = 0; j < kOffBatch; ++j) {
      const int i = i0 + j * S::kThreads + lane;
      if (i > n_shots) o[j] = INT32_MAX;
      seg0 += __popcll(__builtin_amdgcn_ballot_w64(o[j] <= k_begin));
      seg1 += __popcll(__builtin_amdgcn_ballot_w64(o[j] < k_end));
      if (o[j] > k_begin && o[j] < k_end) s_end[i % kEndCache] = o[j];
    }
  }
  if (lane == 0) { s_count[wave][0] = seg0; s_count[wave][1] = seg1; }
  // the query loads must have landed before the streaming loop starts: inside the loop the only vector-memory loads are
  // the block loads, whose completion is tracked by hand, and the queries of the fp32 form, which wait for all of them
#pragma unroll
  for (int q = 0; q < NQW; ++q)
#pragma unroll
    for (int ks = 0; ks < E::kQueryVecs; ++ks) asm volatile("" ::"v"(bq[q][ks]));
  __syncthreads();
  seg0 = seg1 = 0;
#pragma unroll
  for (int w = 0; w < S::kWaves; ++w) {
    seg0 += s_count[w][0];
    seg1 += s_count[w][1];
  }
  seg0 = __builtin_amdgcn_readfirstlane(seg0);
  seg1 = __builtin_amdgcn_readfirstlane(seg1);
  const bool ends_in_lds = seg1 - seg0 <= kEndCache;
  // Two loads, each through a pointer of its own address space: as one load through a generic pointer to either, every
  // boundary would wait for all vector memory, the blocks in flight included (whole call, 8 problems of 16384 tokens in
  // 600 units, per KV head: 159.7 us that way, 157.2 like this; 32 of 32768 tokens in 1240 units 951 and 941).
  lds_cint* ends = (lds_cint*)&s_end[0];
  auto segment_end = [&](int sg) {
    if (sg >= seg1) return k_end;
    if (ends_in_lds) return __builtin_amdgcn_readfirstlane(ends[sg % kEndCache]);
    return __builtin_amdgcn_readfirstlane(off[sg]);
  };

  float m_run[NQW], l_run[NQW], l_grp[NQW];
#pragma unroll
  for (int q = 0; q < NQW; ++q) { m_run[q] = -INFINITY; l_run[q] = 0.f; l_grp[q] = 0.f; }

  // A finished chunk's statistic, log2(sum_k 2^z_k) per query, waits in registers until kStash chunks
  // have finished (or the stream ends) and is then stored right after a barrier, ahead of that
  // iteration's loads: vector stores share the loads' completion counter, so a store inside the
  // streaming loop puts its own latency into the wait for the next block, and the fewer of them the
  // better.  Both lane halves hold a query's value; chunk j of the batch is kept by the lanes of half
  // j / 4 in slot j % 4.  Row r of the partial array is query (lane%32)*NQB + qb.
  constexpr int kStash = 8;
  float stash[4][NQW];
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
#pragma unroll
    for (int q = 0; q < NQW; ++q) stash[sl][q] = 0.f;
  int n_stash = 0, stash_c0 = 0;
  const int my_half = lane >> 5;
  auto stash_put = [&](const float (&val)[NQW], int chunk) {
    if (n_stash == 0) stash_c0 = chunk;
    const bool mine = (n_stash >> 2) == my_half;
    const int slot = n_stash & 3;
#pragma unroll
    for (int sl = 0; sl < 4; ++sl)
#pragma unroll
      for (int q = 0; q < NQW; ++q) stash[sl][q] = (mine && sl == slot) ? val[q] : stash[sl][q];
    ++n_stash;
  };
  auto flush = [&]() {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const int j = sl + 4 * my_half;
      if (j < n_stash) {
        float* dst = out + static_cast<size_t>(stash_c0 + j) * R + (lane & 31) * NQB + qb0;
        if (NQW == 2) {
          *reinterpret_cast<float2*>(dst) = make_float2(stash[sl][0], stash[sl][NQW - 1]);
        } else {
#pragma unroll
          for (int q = 0; q < NQW; ++q) dst[q] = stash[sl][q];
        }
      }
    }
    n_stash = 0;
  };

  int cur_buf = 0;
  bool first_block = true;
  int cur_seg = seg0, cur_end = segment_end(seg0);

  // the current chunk is complete: add up the lane halves (same reference), keep its statistic
  auto finish_chunk = [&]() {
    float val[NQW];
#pragma unroll
    for (int q = 0; q < NQW; ++q) {
      const float l = sum_across_halves(l_run[q]);
      // log2(0) = -inf: a query that saw none of the chunk's keys; so is a padding query row
      val[q] = (l > 0.f && (qb0 + q) * 32 + (lane & 31) < n_rows) ? add_log2(m_run[q], l)
                                                                   : -INFINITY;
      l_grp[q] += l;
      l_run[q] = 0.f;  // the reference carries over to the next chunk
    }
    if (n_stash == kStash) flush();  // several chunks can end inside one block
    stash_put(val, blockIdx.x + cur_seg);
    ++cur_seg;
    cur_end = cur_seg <= seg1 ? segment_end(cur_seg) : INT32_MAX;
  };

#pragma clang loop unroll(disable)
  while (true) {
    // this wave's share of `cur` has landed once only the loads of the queued blocks are outstanding
    // (stores of statistics issued meanwhile are younger than those loads and only make the wait stricter)
    if (n_q == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (n_q == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::kLoads) : "memory");
    else if (n_q == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * S::kLoads) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * S::kLoads) : "memory");
    // ... and after the barrier so has the other waves'; all are also done reading the block before
    if (SHARED) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else if (S::kWaves > 1) asm volatile("s_barrier" ::: "memory");
    if (n_stash == kStash) flush();
    if (next_key0 < k_end) {
      issue_block<E, S::kLoads>(k_plane, next_key0, k_end - next_key0,
                             lds_addr + ring_slot(cur_buf + n_q + 1) * E::kBufBytes, g0, lane);
      ++n_q;
      next_key0 += kBlockKeys;
    }
    // keys past the end of the span and keys a window query may not see yet are masked; both only
    // happen in the span's last block or in the last W keys, so the common block takes the plain path.
    // The workgroup's first block has no reference yet and takes the exact update straight away.
    const int cur_rem = min(kBlockKeys, k_end - cur_key0);
    const bool masked = cur_rem < kBlockKeys || cur_key0 + kBlockKeys - 1 > causal_base;
    lds_cchar* blk = lds_base + cur_buf * E::kBufBytes;
    lds_cchar* parts = (lds_cchar*)&lds_parts[0];
    if constexpr (SHARED) {
      // (the waves have read the parts of the block before: the barrier above)
      split_block<D, S::kWaves>(blk, (lds_char*)&lds_parts[0], wave, lane);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (cur_end >= cur_key0 + cur_rem) {  // no chunk ends inside the block
      if (first_block)
        compute_block<T, D, NQW, SHARED, true, true>(blk, parts, bq, src, lane, cur_key0, cur_rem, causal_base, W, c, m_run, l_run, l_grp);
      else if (masked)
        compute_block<T, D, NQW, SHARED, true, false>(blk, parts, bq, src, lane, cur_key0, cur_rem, causal_base, W, c, m_run, l_run, l_grp);
      else
        compute_block<T, D, NQW, SHARED, false, false>(blk, parts, bq, src, lane, cur_key0, cur_rem, causal_base, W, c, m_run, l_run, l_grp);
    } else {
      floatx16 e[NQW];
      if (masked)
        weights_block<T, D, NQW, SHARED, true>(blk, parts, bq, src, lane, cur_key0, cur_rem, causal_base, W, c, m_run, l_run, l_grp, e);
      else
        weights_block<T, D, NQW, SHARED, false>(blk, parts, bq, src, lane, cur_key0, cur_rem, causal_base, W, c, m_run, l_run, l_grp, e);
      float sum[NQW];  // of the current chunk's rows in this block
      auto add_sum = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NQW; ++q) { l_run[q] += sum[q]; sum[q] = 0.f; }
      };
#pragma unroll
      for (int q = 0; q < NQW; ++q) sum[q] = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row0 = cur_key0 + 8 * i;
        if (cur_end >= row0 + 8) {  // the group has no end inside
#pragma unroll
          for (int q = 0; q < NQW; ++q) sum[q] += (e[q][4 * i] + e[q][4 * i + 1]) + (e[q][4 * i + 2] + e[q][4 * i + 3]);
        } else {
          uint32_t open = 0xffu;  // rows not yet credited
          do {
            const uint32_t behind = 0xffu << max(cur_end - row0, 0);  // (offsets that are out of order may end before)
            credit_rows<NQW>(e, i, open & ~behind, sum);
            open = behind;
            add_sum();
            finish_chunk();
          } while (cur_end < row0 + 8);
          credit_rows<NQW>(e, i, open, sum);
        }
        if (i == 3) add_sum();
        else if (cur_end == row0 + 8) { add_sum(); finish_chunk(); }
      }
    }
    first_block = false;
    if (cur_end == cur_key0 + cur_rem) finish_chunk();  // the chunk ends with the block
    if (n_q == 0) break;
    cur_key0 += kBlockKeys;
    --n_q;
    cur_buf = ring_slot(cur_buf + 1);
  }
  if (n_stash > 0) flush();
  // the same statistic over all of the workgroup's chunks, from which the row denominators are built
  if (lane < 32) {
    float* dst = group_stat + ((static_cast<size_t>(p) * H_kv + g) * gridDim.x + blockIdx.x) * R +
                 (lane & 31) * NQB + qb0;
#pragma unroll
    for (int q = 0; q < NQW; ++q)
      dst[q] = (l_grp[q] > 0.f && (qb0 + q) * 32 + lane < n_rows) ? add_log2(m_run[q], l_grp[q])
                                                                 : -INFINITY;
  }
}

}  // namespace

int score_group_keys(int P, int H_kv, int row_blocks, int n_tokens, int n_shots) {
#ifdef SHOTKV_SCORE_GROUP_KEYS
  return SHOTKV_SCORE_GROUP_KEYS;
#else
  // A workgroup takes one slice of the key axis.  Long slices amortise its
  // query registers and its start-up, but the chip wants a thousand workgroups or more: measured on
  // batches of 1 to 128 problems of 32K tokens, 2048-key slices win from about four thousand workgroups
  // on, 1024-key slices from about one thousand on, and below that the count matters more than the length: one
  // problem of 2000 / 4000 tokens (8 KV heads) takes 24.3 / 26.0 us with 128-key slices, 27.2 / 28.5 us with 256;
  // from 8192 tokens on 256 is faster (31.7 against 32.5 us), 16384 tokens 36.1 with 256 and 37.6 with 512,
  // 32768 tokens 47.4 and 43.6 (128 query rows on four waves; 32 or 160 rows on fewer: 38.6 and 40.3, 59.1 and 60.5).
  const long total_keys = static_cast<long>(n_tokens) * H_kv * P;
  long keys = total_keys < 48L * 1024L ? 128 : 256;
  if (total_keys >= 2048L * 4096L) keys = 2048;
  else if (total_keys >= 1024L * 1024L) keys = 1024;
  else if (total_keys >= ((row_blocks & 3) ? 512L : 256L) * 1024L) keys = 512;
  // sentence-sized units: most blocks hold a boundary and cost twice a plain block, so the workgroups'
  // run times differ more and shorter ones balance better (3 % at 1240 units per 32K tokens)
  if (n_shots > 0 && n_tokens / n_shots < 64 && keys > 512) keys = 512;
  return static_cast<int>(keys);
#endif
}

int score_row_blocks(int dtype, int rows) {
  // what the kernel is instantiated for; fp32, with one block per wave, has no six-block form
  const int need = ceil_div(rows, 32);
  return need <= 2 ? need : need <= 4 ? 4 : (need <= 6 && dtype == SHOTKV_BF16) ? 6 : 8;
}

template <typename T, int D, int NQB, int WAVES, bool SHARED = false>
static void launch_score(const PrefillDims& d, const void* q_obs, const void* k, const int32_t* off,
                         const PrefillWorkspace& w, hipStream_t s) {
  hipLaunchKernelGGL((score_partials_mfma_kernel<T, D, NQB, WAVES, SHARED>), dim3(w.n_groups, d.H_kv, d.P),
                     dim3(GroupShape<T, D, NQB, WAVES, SHARED>::kThreads), 0, s, static_cast<const T*>(q_obs),
                     static_cast<const T*>(k), d.n_tokens, d.H, d.H_kv, d.W, d.R_rows, d.sm_scale * kLog2e,
                     off, d.share, d.n_shots, w.group_keys, w.max_c, w.partial, w.group_stat);
}

// Waves that share the query blocks of a workgroup.  With four (one block each at 128 rows) a launch of few
// workgroups reaches all SIMDs and a block of keys takes half as long; with two every block of keys is read from LDS
// half as often, which is what counts once the chip is full.  Whole compression, four against two waves, 8 KV heads,
// 128 rows, head_dim 128: 8192 tokens 29.6 / 31.5 us, 4 x 32768 93 / 99, 32 x 32768 545 / 550, 64 x 32768 1074 / 1071,
// 128 x 32768 2080 / 2049; units of 25 tokens 4 x 32768 173 / 177, 32 x 32768 986 / 946; head_dim 64: 8 x 16384
// 75 / 81, 16 x 16001 122 / 118.  A unit's end costs a wave the same whatever share of the rows it has, so with several
// ends in a block two waves are better early: units of 8 tokens, 32768 tokens 143 / 154, 4 x 32768 266 / 256, at
// head_dim 64 238 / 199, 16 x 8192 in units of 6 278 / 262, 2 x 32768 in units of 15 146 / 148.  256 rows always take four (two blocks each instead of four, which spills):
// 32 x 32768 805 / 924 us.
static bool four_waves(const PrefillDims& d) {
  const long total_keys = static_cast<long>(d.n_tokens) * d.H_kv * d.P;
  const int unit = d.n_shots > 0 ? d.n_tokens / d.n_shots : INT32_MAX;  // tokens, on average
  return total_keys < (unit < 16 ? 1L << 19 : d.D == 64 ? 3L << 19 : unit < 64 ? 2L << 20 : 12L << 20);
}

// Whether the four or eight waves of a workgroup split fp32 blocks between them.  (Two waves gain less from it than the
// second barrier costs: 8 problems of 8000 tokens, 16 query / 8 KV heads, head_dim 128, 157 us a call, 150 if each splits for
// itself.)  Four waves at head_dim 128 that share leave room for two workgroups per CU, three where each wave splits for
// itself: launches that are one round of three but not of two mostly lose.  Whole call, 128 rows, 8 KV heads, shared and
// each for itself, by workgroups with a whole slice: 512 62.0 and 68.4 us, 528 69.5 and 67.8, 560 72.8 and 70.9, 640 120.2
// and 119.0 (2 x 20000 tokens), 720 77.0 and 77.4, 744 83.1 and 79.6, 760 79.3 and 80.4, 768 80.2 and 81.5, 776 86.8 and
// 92.6, 1000 92.4 and 96.6, 1250 197.6 and 203.  head_dim 64 (four per CU either way) 624 66.9 and 71.9, eight waves 624
// 180 and 201.
static bool share_parts(const PrefillDims& d, const PrefillWorkspace& w) {
  const long workgroups = static_cast<long>(d.n_tokens / w.group_keys) * d.H_kv * d.P;
  return d.D == 64 || workgroups <= 2 * 256 || workgroups >= 3 * 256;
}

template <typename T, int D>
static hipError_t launch_score_rows(const PrefillDims& d, const void* q_obs, const void* k, const int32_t* off,
                                    const PrefillWorkspace& w, hipStream_t s) {
  constexpr bool kF32 = sizeof(T) == 4;
  switch (d.R / 32) {
    case 1: launch_score<T, D, 1, 1>(d, q_obs, k, off, w, s); break;
    case 2: launch_score<T, D, 2, 2>(d, q_obs, k, off, w, s); break;
    case 4:
      if constexpr (!kF32)
        if (!four_waves(d)) { launch_score<T, D, 4, 2>(d, q_obs, k, off, w, s); break; }
      if constexpr (kF32)
        if (share_parts(d, w)) { launch_score<T, D, 4, 4, true>(d, q_obs, k, off, w, s); break; }
      if constexpr (!kF32 || D == 128) launch_score<T, D, 4, 4>(d, q_obs, k, off, w, s);
      break;
    case 6:
      if constexpr (!kF32) { launch_score<T, D, 6, 2>(d, q_obs, k, off, w, s); break; }
      return hipErrorInvalidValue;
    case 8:
      launch_score<T, D, 8, kF32 ? 8 : 4, kF32>(d, q_obs, k, off, w, s);  // fp32 operands: one block per wave
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_score_partials(const PrefillDims& d, const void* q_obs, const void* k, const int32_t* off,
                                 const PrefillWorkspace& w, hipStream_t s) {
  { KernelTimer plan_timer(d.timing, kKernelPlan, s); }  // the kernel finds the shot boundaries of its slices itself
  KernelTimer timer(d.timing, kKernelScore, s);
  if (d.dtype == SHOTKV_BF16) {
    if (d.D == 128) return launch_score_rows<bf16_t, 128>(d, q_obs, k, off, w, s);
    if (d.D == 64) return launch_score_rows<bf16_t, 64>(d, q_obs, k, off, w, s);
  } else {
    if (d.D == 128) return launch_score_rows<float, 128>(d, q_obs, k, off, w, s);
    if (d.D == 64) return launch_score_rows<float, 64>(d, q_obs, k, off, w, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace shotkv
