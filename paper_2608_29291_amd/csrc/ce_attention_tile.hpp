// One tile of routed attention: 128 queries of one (sequence, head) against the
// sequence's keys, by a workgroup of 4 waves. The prefill and generation kernel
// runs nothing else; the decode kernel runs it for the long sequences of a mixed
// batch.
//
// bf16 in and out, fp32 accumulation, head_dim 128; 32 queries per wave, keys in
// tiles of 64, two workgroups per CU:
//   * S^T = K Q^T on MFMA 32x32x16 (keys are the A operand, queries the B
//     operand, held in registers for the whole loop), so each lane owns one
//     query: its 16 scores of a block of 32 keys sit in the lane and the other
//     16 in lane l ^ 32, and the online softmax (running max m, rescale of the
//     output by 2^(m_old - m_new)) needs one cross-lane exchange; the running
//     sum l stays per lane until the end;
//   * P (bf16, the lane's probabilities in MFMA operand order) times V^T:
//     O^T = V^T P^T with the key index of the product permuted to match the
//     layout of the score accumulators;
//   * K and V tiles reach LDS by whole-line DMA (a row of 128 bf16 is 256
//     bytes): chunk c of K row r at c ^ (r & 15), so 16 consecutive rows read
//     by one 16-byte fragment load cover all 64 banks; chunk c of V row r at
//     c ^ 4 (r & 3), so the four keys that half a wave's transposing 8-byte
//     reads touch cover them too. Q comes and O leaves through LDS as whole
//     lines as well;
//   * what bounds it: per wave and tile 32 MFMAs (1024 clocks) and about 190
//     VALU instructions (about 900 clocks, 32 of them exp2) that the same SIMD
//     issues. A stage therefore carries one block of 32 keys through the
//     softmax, one probability after each MFMA of two independent products: the
//     scores of the block after it and the output of the block before it. With
//     blocks of 64 keys this pipeline needs more than 256 registers (it
//     spilled); with 32 it takes 196;
//   * two stages per barrier; K and V are double-buffered. With causal masking
//     the tiles after the workgroup's last query are skipped, and only blocks
//     that reach past a wave's first visible limit are masked element by
//     element;
//   * the scale is folded into the exponent, p = 2^(s c - m c) with c = scale
//     log2 e > 0 and m a running maximum of the raw scores that moves (and
//     rescales the output and the sum) only when some lane's block maximum
//     exceeds it by more than 8 / c, so p < 2^8 and most blocks skip the
//     rescale.
// Measured, kernel alone, 12 heads over 2: 4 x 2176 bidirectional 144 -> 125 us
// (930 TFLOP/s; 816 workgroups on 512 places, so the second round is 60% full),
// 8 x 551 causal 25 -> 22 us, against one stage of 64 keys whose MFMAs and
// softmax the compiler kept apart, V transposed through registers, and Q and O
// in 16- and 8-byte pieces of a row (these alone 5 us and 3 us). Without any
// softmax the MFMAs, waits and barriers of the same loop take 99 us.
#pragma once

#include <type_traits>

#include "ce_device.hpp"

namespace ce {

namespace attn {

constexpr int kDh = 128;       // head dimension
constexpr int kQT = 128;       // queries per workgroup
constexpr int kKT = 64;        // keys per tile
constexpr int kBK = 32;        // keys per block: one pass of the softmax
constexpr int kKRow = kDh * 2; // bytes per key row
constexpr int kKBytes = kKT * kKRow;       // 16 KB
constexpr int kAhead = 3;                  // MFMA operands read from LDS this many products ahead
constexpr float kLazy = 8.0f;              // headroom of the running maximum (exponent of 2)

struct AttnArgs {
  const char* q;
  const char* k;
  const char* v;
  char* o;
  const int32_t* qo;
  const int32_t* ko;
  int B, H, Hkv, q_cap, kv_cap, causal;
  float scale_log2;  // scale * log2(e)
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// 8-byte LDS read that transposes 4 x 16 blocks of 16-bit values inside groups
// of 16 lanes: lane i gets value i % 4 of the 8 bytes that lanes i / 4, + 4,
// + 8, + 12 of its group point at.
__device__ __forceinline__ u32x2_t lds_read_tr(const char* __restrict__ p) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                         (__attribute__((address_space(3))) s16x4_t*)(p)));
}

// smem: 4 kKBytes, 1024-byte aligned, free at entry (every wave past a barrier);
// kShared: the kernel has other arrays in LDS.
template <bool kShared>
__device__ __forceinline__ void attention_tile(const AttnArgs& a, char* const smem, int b, int h, int q0, int nq,
                                               int qbase) {
  // Beside other arrays in LDS the compiler ties the DMAs to the fragment reads
  // and drains them before each stage (1.7 us a tile of keys instead of 1.1),
  // unless their base passes through an empty asm; alone that costs 2%.
  typedef __attribute__((address_space(3))) char lds_char;
  lds_char* ring = (lds_char*)smem;
  if constexpr (kShared) asm volatile("" : "+s"(ring));
  char* const kbuf = smem;
  char* const vbuf = smem + 2 * kKBytes;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kvh = h / (a.H / a.Hkv);
  const int klo = clampi(a.ko[b], 0, a.kv_cap), khi = clampi(a.ko[b + 1], klo, a.kv_cap);
  const int nk = khi - klo;
  const int off = nk - nq;  // end alignment of the causal mask

  // tiles of keys this query block can see
  int ntiles = (nk + kKT - 1) / kKT;
  if (a.causal) {
    const int jmax = min(nq - 1, q0 + kQT - 1) + off;  // last key the block's last query sees
    ntiles = jmax < 0 ? 0 : min(ntiles, jmax / kKT + 1);
  }

  // ---- this lane's query: row q0 + 32 wave + (lane % 32), K-chunks of (lane / 32) ----
  const int lrow = lane & 31;
  const int lhalf = lane >> 5;
  const int qi = q0 + 32 * wave + lrow;  // query index inside the sequence
  auto opaque = [](uint32_t x) __attribute__((always_inline)) {
    asm volatile("" : "+v"(x));
    return x;
  };
  const int64_t kv_row = (int64_t)a.Hkv * kKRow;  // bytes between consecutive keys
  const int64_t tile_bytes = kKT * kv_row;

  // ---- K tile DMA: wave w fetches key rows 16 w .. +15, four rows of 256 B
  //      per instruction; full tiles add the tile offset as a scalar ----
  const __amdgpu_buffer_rsrc_t krs = make_rsrc(a.k, (uint32_t)((int64_t)a.kv_cap * kv_row));
  const int kr_sub = lane >> 4;   // row within the instruction
  const int kpc = lane & 15;      // physical chunk this lane fills
  uint32_t kvo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * wave + 4 * i + kr_sub;
    kvo[i] = opaque((uint32_t)((int64_t)(klo + r) * kv_row) + (uint32_t)(kvh * kKRow + ((kpc ^ (r & 15)) << 4)));
  }
  // Keys of a ragged last tile past the sequence's end are fetched as they
  // are (the next sequence's rows, or zeros past the buffer): every score of
  // a key at or past n_kv is replaced by -inf before the softmax reads it.
  auto dma_k = [&](int tile, int buf) __attribute__((always_inline)) {
    lds_char* region = ring + buf * kKBytes + 16 * wave * kKRow;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, region + 4 * i * kKRow, 16, (int)kvo[i], (int)(tile * tile_bytes), 0, 0);
  };
  // ---- V tile DMA: the same rows, chunk c of row r at c ^ 4 (r & 3). Keys of
  //      a ragged last tile past the sequence's end fetch its last key instead
  //      (finite values: their probabilities are 0, and 0 * NaN is not) ----
  const __amdgpu_buffer_rsrc_t vrs = make_rsrc(a.v, (uint32_t)((int64_t)a.kv_cap * kv_row));
  const uint32_t vcol = (uint32_t)(kvh * kKRow + ((kpc ^ (kr_sub << 2)) << 4));
  const uint32_t vvo = (uint32_t)((int64_t)(klo + 16 * wave + kr_sub) * kv_row) + vcol;
  auto dma_v = [&](int tile, int buf) __attribute__((always_inline)) {
    lds_char* region = ring + (2 + buf) * kKBytes + 16 * wave * kKRow;
    auto put = [&](int i, uint32_t vo, int so) __attribute__((always_inline)) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vrs, region + 4 * i * kKRow, 16, (int)vo, so, 0, 0);
    };
    if ((tile + 1) * kKT <= nk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) put(i, vvo, (int)(tile * tile_bytes + 4 * i * kv_row));
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = klo + min(tile * kKT + 16 * wave + 4 * i + kr_sub, nk - 1);
        put(i, (uint32_t)((int64_t)key * kv_row) + vcol, 0);
      }
    }
  };

  u32x4_t qf[8];  // this lane's query, K steps of 16
  // ---- per-lane LDS fragment offsets ----
  uint32_t koff[8];  // K: row lrow, chunk (2 s + lhalf), swizzled
#pragma unroll
  for (int s2 = 0; s2 < 8; ++s2)
    koff[s2] = opaque((uint32_t)(lrow * kKRow + ((((uint32_t)(2 * s2 + lhalf)) ^ (uint32_t)(lrow & 15)) << 4)));
  // V: a transposing read gives 16 lanes the 16 dims of four keys; this lane
  // supplies 8 bytes of key 4 lhalf + (lane / 4) % 4. One register per block of
  // 32 dims (the swizzle moves it), the key is an immediate.
  uint32_t voff[4];
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    const int key = (lane >> 2) & 3;
    const int c = ((db ^ key) << 2) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    voff[db] = opaque((uint32_t)(2 * kKBytes + (4 * lhalf + key) * kKRow + (c << 4) + 8 * (lane & 1)));
  }

  f32x16_t oacc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) oacc[i] = f32x16_t{};
  float m_run = -__builtin_inff(), l_run = 0.0f;  // l_run: this lane's keys only until the epilogue
  const int vis = a.causal ? min(nk, qi + off + 1) : nk;              // keys [0, vis) are visible
  const int vis0 = a.causal ? min(nk, q0 + 32 * wave + off + 1) : nk;  // the wave's smallest

  using Half0 = std::integral_constant<int, 0>;
  using Half1 = std::integral_constant<int, 1>;
  using Yes = std::true_type;
  using No = std::false_type;
  auto tile_max = [&](const f32x16_t& sc) __attribute__((always_inline)) {
    float m = -__builtin_inff();
#pragma unroll
    for (int v = 0; v < 16; ++v) m = fmaxf(m, sc[v]);
    return m;
  };
  // hide the keys of block `blk` this lane may not see (ragged end, causal cut)
  auto mask = [&](int blk, f32x16_t& sc, float& mt) __attribute__((always_inline)) {
    const int kbase = blk * kBK;
    if (kbase + kBK > vis0) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (kbase + 8 * (v >> 2) + 4 * lhalf + (v & 3) >= vis) sc[v] = -__builtin_inff();
      mt = tile_max(sc);
    }
  };
  // operand of MFMA j of a stage: 0..7 the scores (32-byte K step j), 8..15
  // the output (16 keys (j - 8) / 4, 32 dims j % 4)
  auto frag = [&](int j, int khalf, int vhalf) __attribute__((always_inline)) {
    if (j < 8) return lds_read16(smem + koff[j], khalf * kBK * kKRow);
    const char* p = smem + voff[j & 3] + (vhalf * kBK + 16 * ((j - 8) >> 2)) * kKRow;
    const u32x2_t lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * kKRow);
    return u32x4_t{lo.x, lo.y, hi.x, hi.y};
  };
  // One stage takes block blk (32 keys, half blk % 2 of its tile) through the
  // softmax (scores sc, lane maximum mt; probabilities to pn) while the matrix
  // cores compute the scores of block blk + 1 (into sn, lane maximum to mn) and
  // then the output of block blk - 1 (probabilities pp): one probability after
  // each MFMA, in program order. The fences keep the compiler from sorting the
  // two kinds of instructions apart again.
  auto stage = [&](auto half_c, auto first_c, auto last_c, int blk, f32x16_t& sc, f32x16_t& sn, u32x4_t (&pp)[2],
                   u32x4_t (&pn)[2], float mt, float& mn) __attribute__((always_inline)) {
    constexpr int kHalf = decltype(half_c)::value;
    constexpr bool kFirst = decltype(first_c)::value, kLast = decltype(last_c)::value;
    constexpr int kLo = kLast ? 8 : 0, kHi = kFirst ? 8 : 16;  // MFMAs of this stage
    constexpr int kPer = 16 / (kHi - kLo);                     // probabilities after each
    u32x4_t fr[16];
#pragma unroll
    for (int j = kLo; j < kLo + kAhead; ++j) fr[j] = frag(j, kHalf ^ 1, kHalf ^ 1);
    // The running maximum moves (and the output is rescaled) only when some
    // lane's block maximum exceeds it by more than kLazy in the exponent, so
    // probabilities stay below 2^kLazy; the sum l uses the same maximum, so
    // the quotient O / l does not depend on it. The output still lacks block
    // blk - 1, whose probabilities have the old maximum: it is rescaled after
    // this stage's MFMAs.
    {
      const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt), false, false);
      mt = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
    }
    float alpha = 1.0f;
    const bool move = __builtin_amdgcn_ballot_w64((mt - m_run) * a.scale_log2 > kLazy) != 0;
    if (move) {
      const float m_new = fmaxf(m_run, mt);
      if (m_new != -__builtin_inff()) alpha = __builtin_amdgcn_exp2f((m_run - m_new) * a.scale_log2);
      l_run *= alpha;
      m_run = m_new;
    }
    const float mc = m_run == -__builtin_inff() ? 0.0f : m_run * a.scale_log2;
    float rs = 0.0f, even = 0.0f;
    auto prob = [&](int e) __attribute__((always_inline)) {
      float p = __builtin_amdgcn_exp2f(fmaf(sc[e], a.scale_log2, -mc));
      asm volatile("" : "+v"(p));  // this and the next keep the value between its fences
      if (e & 1) {
        rs += even + p;
        uint32_t w = pack_bf16(even, p);
        asm volatile("" : "+v"(w), "+v"(rs));
        pn[e >> 3][(e & 7) >> 1] = w;
      } else {
        even = p;
      }
    };
    float mx = -__builtin_inff();
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = kLo; j < kHi; ++j) {
      if (j + kAhead < kHi) fr[j + kAhead] = frag(j + kAhead, kHalf ^ 1, kHalf ^ 1);
      if (j == 0) sn = f32x16_t{};
      if (j < 8)
        mfma_step<true>(sn, fr[j], qf[j]);
      else
        mfma_step<true>(oacc[j & 3], fr[j], pp[(j - 8) >> 2]);
#pragma unroll
      for (int e = (j - kLo) * kPer; e < (j - kLo + 1) * kPer; ++e) prob(e);
      if (!kLast && !kFirst && j >= 12) {
#pragma unroll
        for (int v = 4 * (j - 12); v < 4 * (j - 11); ++v) mx = fmaxf(mx, sn[v]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    l_run += rs;
    if constexpr (!kFirst) {
      if (move) {
#pragma unroll
        for (int i = 0; i < 4; ++i) oacc[i] *= alpha;
      }
    }
    if constexpr (!kLast) {
      mn = kFirst ? tile_max(sn) : mx;
      mask(blk + 1, sn, mn);
    }
  };

  // tile t: buffer t % 2 of K and of V. Scores run one block ahead and the
  // output one block behind, so between two barriers the second half of tile t
  // and the first of tile t + 1 meet K of t + 1 and V of t only, and the DMA of
  // K of t + 2 and V of t + 1 has that time to arrive.
  if (ntiles > 0) {
    f32x16_t sa = f32x16_t{}, sb;
    u32x4_t pa[2], pb[2];
    float ma, mb;
    // The wave's 32 queries come by whole-line DMA as well (rows past the end of
    // the sequence as zeros), chunk c of row r at c ^ (r & 15), into the parts
    // of the two V buffers that this wave itself fills later.
    {
      const int64_t q_row = (int64_t)a.H * kKRow;
      const char* qp = a.q + (int64_t)(qbase + q0) * q_row + (int64_t)h * kKRow;
      const int rows = min(nq - q0, kQT);
      const __amdgpu_buffer_rsrc_t qrs = make_rsrc(qp, (uint32_t)((rows - 1) * q_row + kKRow));
      const int qb = 2 * kKBytes + 16 * wave * kKRow;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = 4 * i + kr_sub;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            qrs, ring + qb + (i >> 2) * kKBytes + 4 * (i & 3) * kKRow, 16,
            (int)((32 * wave + r) * q_row + ((kpc ^ (r & 15)) << 4)), 0, 0, 0);
      }
      dma_k(0, 0);
      if (ntiles > 1) {
        dma_k(1, 1);
        wait_vmcnt<8>();
      } else {
        wait_vmcnt<4>();
      }
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s2 = 0; s2 < 8; ++s2)
        qf[s2] = lds_read16(smem + qb + (lrow >> 4) * kKBytes + (lrow & 15) * kKRow,
                            ((2 * s2 + lhalf) ^ (lrow & 15)) << 4);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before V takes their place
    }
    dma_v(0, 0);
    wait_vmcnt<4>();  // K
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) mfma_step<true>(sa, frag(j, 0, 0), qf[j]);
    ma = tile_max(sa);
    mask(0, sa, ma);
    stage(Half0{}, Yes{}, No{}, 0, sa, sb, pb, pa, ma, mb);
    wait_vmcnt<0>();
    __syncthreads();  // every wave has read K of tile 0; V of tile 0 is there
    for (int t = 0; t + 1 < ntiles; ++t) {
      if (t + 2 < ntiles) dma_k(t + 2, t & 1);
#pragma unroll
      for (int s2 = 0; s2 < 8; ++s2) koff[s2] ^= kKBytes;
      stage(Half1{}, No{}, No{}, 2 * t + 1, sb, sa, pa, pb, mb, ma);
      dma_v(t + 1, (t + 1) & 1);
      stage(Half0{}, No{}, No{}, 2 * t + 2, sa, sb, pb, pa, ma, mb);
#pragma unroll
      for (int db = 0; db < 4; ++db) voff[db] ^= kKBytes;
      wait_vmcnt<0>();
      __syncthreads();
    }
    stage(Half1{}, No{}, Yes{}, 2 * ntiles - 1, sb, sa, pa, pb, mb, ma);
#pragma unroll
    for (int j = 8; j < 16; ++j) mfma_step<true>(oacc[j & 3], frag(j, 0, 1), pb[(j - 8) >> 2]);
  }

  // ---- epilogue: O = O^T / l, turned through LDS into whole rows (256 bytes
  //      by 16 lanes). The wave uses its own 8 KB of the K buffers, which no
  //      wave reads after the last barrier. ----
  l_run += __shfl_xor(l_run, 32);
  const float inv = l_run > 0.0f ? 1.0f / l_run : 0.0f;
  char* const ob = kbuf + wave * 32 * kKRow;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      store4<true>(ob + lrow * kKRow + (((4 * db + g) ^ (lrow & 15)) << 4) + 8 * lhalf, oacc[db][4 * g] * inv,
                   oacc[db][4 * g + 1] * inv, oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 4 * i + kr_sub;
    const u32x4_t w = lds_read16(ob, r * kKRow + (kpc << 4));
    const int row = q0 + 32 * wave + r;
    if (row < nq)
      *reinterpret_cast<u32x4_t*>(a.o + ((int64_t)(qbase + row) * a.H + h) * kKRow + ((kpc ^ (r & 15)) << 4)) = w;
  }
}

}  // namespace attn

}  // namespace ce
