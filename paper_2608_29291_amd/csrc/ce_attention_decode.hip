// Routed attention for few queries per sequence (decode steps over the
// compressed key-value cache): softmax(scale Q K^T + M) V as ce_attention.hip
// defines it, bf16 in and out, head_dim 128.
//
// Bound: memory. A decode step reads every key and value of the cache once for
// a handful of queries, so the kernel is built to have the whole cache in
// flight and to read it once:
//   * the query heads that share a key/value head are columns of one MFMA
//     operand: 32 columns hold up to 32 (query, head) rows, row r = query
//     r / g, head r % g of the group of g = H / H_kv, so K and V are read once
//     per key/value head and not once per query head;
//   * a sequence's keys are cut into chunks, one workgroup each (work items are
//     enumerated on the device from the offsets, so ragged caches balance);
//     inside a chunk the 4 waves take tiles of 32 keys in turn and share
//     nothing until the end (no barrier in the loop);
//   * K goes from memory straight to registers in operand order, V through
//     registers and a wave-private LDS tile that transposes it; the next
//     tile's loads are issued as soon as the registers are free.
// The waves meet in LDS (their running maxima, sums and outputs); with more
// than one chunk the fp32 results go to the workspace and a second launch
// combines them in chunk order, so the result does not depend on which
// workgroup finished first.
//
// The launch takes whole batches, chosen by their rows on average, so these may
// come mixed with others: a sequence with several items' rows (a few more
// queries) is cut into as many workgroups in all, its tiles of 32 rows times
// longer chunks; a prefill runs the 128-query tiles of ce_attention_tile.hpp in
// the same launch, which read its keys once per 128 queries. us, 28 / 4 heads,
// (every sequence on 128-query tiles /) all in uncut tiles of 32 rows / now:
// 1023 empty sequences and a prefill of 4681 (353 /) 610 / 244, 255 and one of
// 1170 (45 /) 66 / 40, 255 of one query over 300 keys and a prefill of 915 (185 /)
// 72 / 54, two sequences of 8000 keys with 5 queries and 1 (138 /) 238 / 37, 8 of
// 2000 with 4 (41 /) 30 / 19, 64 queries over 8000 and 14 empty (181 /) 119 / 78,
// 300 over 300 and 65 empty (14.4 /) 17.8 / 14.4.
//
// Measured (16 queries, 28 / 4 heads, caches of 551 to 3100 keys, 48 MB of keys
// and values): 14.8 us + 5.8 us for the combination, 3.3 TB/s in the first
// launch; the 128-query kernel took 90 us (one workgroup per query head walked
// a whole cache, each key was read by the 7 heads of its group, and one row of
// 128 was a query).
#include "ce_attention_tile.hpp"
#include "ce_host.hpp"
#include "ce_launch.hpp"

namespace ce {

namespace {

using attn::clampi;
using attn::kDh;
using attn::kLazy;

constexpr int kRowB = kDh * 2;           // bytes per key row and head
constexpr int kRows = kAttnRows;         // (query, head) rows per work item
constexpr int kKT = 32;                  // keys per tile of a wave
constexpr int kVRow = kKT * 2;           // bytes per row of V^T
constexpr int kVTile = kDh * kVRow;      // 8 KB
constexpr int kOLd = kDh + 4;            // floats per row of the waves' outputs in LDS
// A sequence of kLongQ queries whose keys would be cut in fewer chunks than
// kLongC takes 128-query tiles; its g per tile are then no more items than its
// tiles of 32 rows, which the grid has room for. us, 28 / 4 heads, row tiles and
// 128-query tiles: 64 queries over 64 keys 8.2 and 6.7, 32 over 1000 in two
// chunks 29.6 and 24.2, 100 over 8000 in three 112 and 138, 32 over 8000 51 and
// 139.
constexpr int kLongQ = 32;
constexpr int kLongC = 3;

struct DecodeArgs : attn::AttnArgs {
  int chunk;        // keys per work item (a multiple of 4 kKT)
  int items;        // work items the grid has room for
  int part_rows;    // rows of a partial result
  float* part;      // [slots x Hkv x part_rows x (kDh + 2)] output, maximum, sum
};

// Partial result of row r of item i of a sequence whose keys begin at klo
// (its slots begin at 2 klo / chunk: see attention_split).
__device__ __forceinline__ float* part_at(const DecodeArgs& a, int klo, int i, int kvh, int r) {
  return a.part + (((int64_t)(2 * klo / a.chunk + i) * a.Hkv + kvh) * a.part_rows + r) * (kDh + 2);
}

// How a sequence of nq queries (g rows each) and nk keys is cut: T tiles of 32
// rows times C chunks of T a.chunk keys, or 128-query tiles of one head each.
struct Cut {
  bool by_query;
  int T, C, n_items;
};
__device__ __forceinline__ Cut cut_of(int nq, int g, int nk, int chunk) {
  Cut c = {false, (nq * g + kRows - 1) / kRows, 1, 0};
  if (nk > chunk) c.C = (nk + chunk - 1) / chunk;
  if (c.T > 1) c.C = (c.C + c.T - 1) / c.T;
  c.by_query = c.T > 1 && nq >= kLongQ && c.C < kLongC;
  if (c.by_query) c.C = 1;
  c.n_items = c.by_query ? (nq + attn::kQT - 1) / attn::kQT * g : c.T * c.C;
  return c;
}

// Byte offset of unit u (4 keys) of V^T row d in a wave's tile. A write covers
// rows 8 apart and a read 32 consecutive rows; rows sit in 64-byte slots, four
// to a 256-byte bank line, and the slot and unit keys give both all 64 banks.
__device__ __forceinline__ uint32_t vt_off(int d, uint32_t u) {
  return (uint32_t)(((d & ~3) | ((d ^ (d >> 3)) & 3)) * kVRow) + ((u ^ (uint32_t)((d >> 2) & 7)) << 3);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attention_decode_kernel(
    DecodeArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kRows * kOLd * 4];  // V^T tiles, then outputs
  __shared__ float ml[2][4][kRows];
  __shared__ int wsh[8];
  static_assert(4 * kRows * kOLd * 4 >= 4 * kVTile && 4 * kRows * kOLd * 4 >= 4 * attn::kKBytes, "the tiles fit");

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = a.H / a.Hkv;
  const int kvh = blockIdx.y;
  const int item = blockIdx.x;

  // ---- the sequence and chunk of this item: item counts of 256 sequences at
  //      a time (one per thread), prefix sums by wave and over the waves ----
  int base = 0;
  bool found = false;
  for (int s0 = 0; s0 < a.B; s0 += 256) {
    const int s = s0 + tid;
    int lo = 0, nq = 0, klo = 0, nk = 0, n = 0;
    if (s < a.B) {
      const int q0 = a.qo[s], q1 = a.qo[s + 1], k0 = a.ko[s], k1 = a.ko[s + 1];
      lo = clampi(q0, 0, a.q_cap);
      nq = clampi(q1, lo, a.q_cap) - lo;
      klo = clampi(k0, 0, a.kv_cap);
      nk = clampi(k1, klo, a.kv_cap) - klo;
      n = cut_of(nq, g, nk, a.chunk).n_items;
    }
    int x = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsh[wave] = x;
    __syncthreads();
    int before = base;
    for (int w = 0; w < wave; ++w) before += wsh[w];
    const int total = (wsh[0] + wsh[1]) + (wsh[2] + wsh[3]);
    __syncthreads();
    const int ex = before + x - n;
    if (item >= ex && item < ex + n) {
      wsh[0] = s;
      wsh[1] = item - ex;
      wsh[2] = lo;
      wsh[3] = nq;
      wsh[4] = klo;
      wsh[5] = nk;
    }
    __syncthreads();
    if (item < base + total) {
      found = true;
      break;
    }
    base += total;
  }
  if (!found) return;
  const int b = __builtin_amdgcn_readfirstlane(wsh[0]);
  const int sub = __builtin_amdgcn_readfirstlane(wsh[1]);
  const int qbase = __builtin_amdgcn_readfirstlane(wsh[2]);
  const int nq = __builtin_amdgcn_readfirstlane(wsh[3]);
  const int klo = __builtin_amdgcn_readfirstlane(wsh[4]);
  const int nk = __builtin_amdgcn_readfirstlane(wsh[5]);
  const Cut ct = cut_of(nq, g, nk, a.chunk);
  if (ct.by_query) {
    // the workgroups of one x, which share an XCD (the grid's x is a multiple of
    // its count), take heads of one key/value head as far as they go; last tiles
    // first: under a causal mask they see the most keys
    const int u = sub * a.Hkv + kvh;
    const int tile = (nq + attn::kQT - 1) / attn::kQT - 1 - u / a.H;
    attn::attention_tile<true>(a, smem, b, u % a.H, tile * attn::kQT, nq, qbase);
    return;
  }
  const bool cut = ct.C > 1;
  const int tile = ct.T == 1 ? 0 : ct.C == 1 ? sub : sub / ct.C;
  const int r0 = tile * kRows;
  const int rows = min(kRows, nq * g - r0);
  const int kbeg = (sub - tile * ct.C) * (cut ? a.chunk * ct.T : 0);
  const int kend = cut ? min(nk, kbeg + a.chunk * ct.T) : nk;
  const int off = nk - nq;  // end alignment of the causal mask

  // ---- the query row of this lane, K-chunks of (lane / 32) ----
  const int lrow = lane & 31;
  const int lhalf = lane >> 5;
  const int rr = r0 + min(lrow, rows - 1);
  const int qi = rr / g;  // query inside the sequence
  const int hq = kvh * g + (rr - qi * g);
  u32x4_t qf[8];
  {
    const char* qp = a.q + ((int64_t)(qbase + qi) * a.H + hq) * kRowB + lhalf * 16;
#pragma unroll
    for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const u32x4_t*>(qp + s * 32);
  }
  const int vis = a.causal ? min(kend, qi + off + 1) : kend;               // keys [0, vis) are visible
  const int vis0 = a.causal ? min(kend, r0 / g + off + 1) : kend;          // the item's first query
  const int vis1 = a.causal ? min(kend, (r0 + rows - 1) / g + off + 1) : kend;  // and its last

  const int64_t kv_row = (int64_t)a.Hkv * kRowB;
  const char* const kp = a.k + (int64_t)klo * kv_row + (int64_t)kvh * kRowB;
  const char* const vp = a.v + (int64_t)klo * kv_row + (int64_t)kvh * kRowB;
  char* const vt = smem + wave * kVTile;
  const int vkg = lane & 7;   // keys 4 vkg .. +3 of the tile
  const int vdg = lane >> 3;  // dims 8 vdg .. +7 and 64 + 8 vdg .. +7
  // keys past the sequence's end read its last key (their scores become -inf
  // and their probabilities 0)
  u32x4_t kf[8], vr[8];
  auto load_k = [&](int k0) __attribute__((always_inline)) {
    const char* p = kp + (int64_t)min(k0 + lrow, nk - 1) * kv_row + lhalf * 16;
#pragma unroll
    for (int s = 0; s < 8; ++s) kf[s] = *reinterpret_cast<const u32x4_t*>(p + s * 32);
  };
  auto load_v = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* p = vp + (int64_t)min(k0 + 4 * vkg + i, nk - 1) * kv_row + vdg * 16;
      vr[i] = *reinterpret_cast<const u32x4_t*>(p);
      vr[4 + i] = *reinterpret_cast<const u32x4_t*>(p + 128);
    }
  };

  f32x16_t oacc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) oacc[i] = f32x16_t{};
  float m_run = -__builtin_inff(), l_run = 0.0f;

  const int step = 4 * kKT;
  int k0 = kbeg + wave * kKT;
  if (k0 < vis1) {
    load_k(k0);
    load_v(k0);
  }
  for (; k0 < vis1; k0 += step) {
    const bool more = k0 + step < vis1;
    // scores: S^T = K Q^T (keys are the A operand), two chains
    f32x16_t sc = {}, s2 = {};
#pragma unroll
    for (int s = 0; s < 8; s += 2) {
      mfma_step<true>(sc, kf[s], qf[s]);
      mfma_step<true>(s2, kf[s + 1], qf[s + 1]);
    }
    if (more) load_k(k0 + step);
    sc += s2;
    if (k0 + kKT > vis0) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (k0 + 8 * (v >> 2) + 4 * lhalf + (v & 3) >= vis) sc[v] = -__builtin_inff();
    }
    // online softmax (lane = row; its keys sit in the lane and in lane ^ 32)
    float mt = sc[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mt = fmaxf(mt, sc[v]);
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    if (__builtin_amdgcn_ballot_w64((mt - m_run) * a.scale_log2 > kLazy)) {
      const float m_new = fmaxf(m_run, mt);
      const float alpha = m_new == -__builtin_inff() ? 1.0f : __builtin_amdgcn_exp2f((m_run - m_new) * a.scale_log2);
#pragma unroll
      for (int i = 0; i < 4; ++i) oacc[i] *= alpha;
      l_run *= alpha;
      m_run = m_new;
    }
    const float mc = m_run == -__builtin_inff() ? 0.0f : m_run * a.scale_log2;
    float rs = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      sc[v] = __builtin_amdgcn_exp2f(fmaf(sc[v], a.scale_log2, -mc));
      rs += sc[v];
    }
    l_run += rs + __shfl_xor(rs, 32);
    u32x4_t pf[2];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i) pf[st][i] = pack_bf16(sc[8 * st + 2 * i], sc[8 * st + 2 * i + 1]);
    // V tile to LDS, transposed (a wave's own tile: its LDS operations are in
    // order, so no barrier)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        const u32x2_t w = {__builtin_amdgcn_perm(vr[4 * c + 1][e >> 1], vr[4 * c][e >> 1], sel),
                           __builtin_amdgcn_perm(vr[4 * c + 3][e >> 1], vr[4 * c + 2][e >> 1], sel)};
        *reinterpret_cast<u32x2_t*>(vt + vt_off(64 * c + 8 * vdg + e, (uint32_t)vkg)) = w;
      }
    if (more) load_v(k0 + step);
    // O^T += V^T P^T over 2 steps of 16 keys, in the scores' key order
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const u32x2_t lo = *reinterpret_cast<const u32x2_t*>(vt + vt_off(32 * db + lrow, (uint32_t)(4 * st + lhalf)));
        const u32x2_t hi =
            *reinterpret_cast<const u32x2_t*>(vt + vt_off(32 * db + lrow, (uint32_t)(4 * st + lhalf + 2)));
        const u32x4_t vf = {lo.x, lo.y, hi.x, hi.y};
        mfma_step<true>(oacc[db], vf, pf[st]);
      }
  }

  // ---- the four waves meet: common maximum, scaled outputs through LDS ----
  if (lhalf == 0) {
    ml[0][wave][lrow] = m_run;
    ml[1][wave][lrow] = l_run;
  }
  __syncthreads();  // also: every wave is done with its V tile
  float m_all = ml[0][0][lrow];
#pragma unroll
  for (int w = 1; w < 4; ++w) m_all = fmaxf(m_all, ml[0][w][lrow]);
  const float al = m_run == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_all) * a.scale_log2);
  float* const ob = reinterpret_cast<float*>(smem);
  if (lrow < rows) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4_t x = {oacc[db][4 * g4] * al, oacc[db][4 * g4 + 1] * al, oacc[db][4 * g4 + 2] * al,
                           oacc[db][4 * g4 + 3] * al};
        *reinterpret_cast<f32x4_t*>(ob + (wave * kRows + lrow) * kOLd + 32 * db + 8 * g4 + 4 * lhalf) = x;
      }
  }
  __syncthreads();
  // thread: row tid / 32 (+ 8, 16, 24), dims 4 (tid % 32) .. +3
  for (int r = tid >> 5; r < rows; r += 8) {
    const int d0 = 4 * (tid & 31);
    float mr = ml[0][0][r], lr = 0.0f;
#pragma unroll
    for (int w = 1; w < 4; ++w) mr = fmaxf(mr, ml[0][w][r]);
    f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float mw = ml[0][w][r];
      lr += mw == -__builtin_inff() ? 0.0f : ml[1][w][r] * __builtin_amdgcn_exp2f((mw - mr) * a.scale_log2);
      x += *reinterpret_cast<const f32x4_t*>(ob + (w * kRows + r) * kOLd + d0);
    }
    if (cut) {
      float* const p = part_at(a, klo, sub, kvh, r);
      *reinterpret_cast<u32x2_t*>(p + d0) = u32x2_t{__float_as_uint(x.x), __float_as_uint(x.y)};
      *reinterpret_cast<u32x2_t*>(p + d0 + 2) = u32x2_t{__float_as_uint(x.z), __float_as_uint(x.w)};
      if (d0 == 0) {
        p[kDh] = mr;
        p[kDh + 1] = lr;
      }
    } else {
      const int q2 = (r0 + r) / g;
      const float inv = lr > 0.0f ? 1.0f / lr : 0.0f;
      store4<true>(a.o + ((int64_t)(qbase + q2) * a.H + kvh * g + (r0 + r - q2 * g)) * kRowB + d0 * 2, x.x * inv,
                   x.y * inv, x.z * inv, x.w * inv);
    }
  }
}

// Chunk results of the sequences that were cut, added in chunk order:
// workgroups per sequence and key/value head, a wave per row (4 at a time and
// workgroup), two dims per lane; eight chunks' loads in flight.
__global__ __launch_bounds__(256) void attention_combine_kernel(DecodeArgs a) {
  const int b = blockIdx.x, kvh = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = a.H / a.Hkv;
  const int lo = clampi(a.qo[b], 0, a.q_cap);
  const int nq = clampi(a.qo[b + 1], lo, a.q_cap) - lo;
  const int klo = clampi(a.ko[b], 0, a.kv_cap);
  const int nk = clampi(a.ko[b + 1], klo, a.kv_cap) - klo;
  const Cut ct = cut_of(nq, g, nk, a.chunk);
  if (nq <= 0 || ct.C <= 1) return;
  const int rows = nq * g, n = ct.C;
  const int64_t stride = (int64_t)a.Hkv * a.part_rows * (kDh + 2);  // floats between chunks
  for (int r = wave + 4 * (int)blockIdx.z; r < rows; r += 4 * (int)gridDim.z) {
    const float* const p = part_at(a, klo, r / kRows * n, kvh, r % kRows);
    float m = -__builtin_inff(), l = 0.0f, x0 = 0.0f, x1 = 0.0f;
    for (int c0 = 0; c0 < n; c0 += 8) {
      float mc[8], lc[8], y0[8], y1[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float* const pc = p + min(c0 + i, n - 1) * stride;
        mc[i] = pc[kDh];
        lc[i] = pc[kDh + 1];
        y0[i] = pc[2 * lane];
        y1[i] = pc[2 * lane + 1];
      }
      float m_new = m;
#pragma unroll
      for (int i = 0; i < 8; ++i) m_new = fmaxf(m_new, mc[i]);
      // (a maximum of -inf is a chunk whose keys are hidden or whose scores are
      // all NaN: its output, 0 or NaN, counts with weight 0, as a wave's does in
      // the launch before; loads repeated past the last chunk don't count)
      const float al = m_new == -__builtin_inff() ? 1.0f : __builtin_amdgcn_exp2f((m - m_new) * a.scale_log2);
      l *= al;
      x0 *= al;
      x1 *= al;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool in = c0 + i < n;
        const float w = in && mc[i] != -__builtin_inff() ? __builtin_amdgcn_exp2f((mc[i] - m_new) * a.scale_log2) : 0.0f;
        l = fmaf(in ? lc[i] : 0.0f, w, l);
        x0 = fmaf(in ? y0[i] : 0.0f, w, x0);
        x1 = fmaf(in ? y1[i] : 0.0f, w, x1);
      }
      m = m_new;
    }
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    const int q2 = r / g;
    *reinterpret_cast<uint32_t*>(a.o + ((int64_t)(lo + q2) * a.H + kvh * g + (r - q2 * g)) * kRowB + 4 * lane) =
        pack_bf16(x0 * inv, x1 * inv);
  }
}

}  // namespace

hipError_t launch_attention_decode(const char* q, const char* k, const char* v, char* o, const int32_t* q_offsets,
                                   const int32_t* kv_offsets, int B, int H, int Hkv, int q_cap, int kv_cap, bool causal,
                                   float scale, void* ws, hipStream_t stream) {
  if (q_cap <= 0) return hipSuccess;
  DecodeArgs args{{q, k, v, o, q_offsets, kv_offsets, B, H, Hkv, q_cap, kv_cap, causal ? 1 : 0,
                   scale * 1.4426950408889634f}, 0, 0, 0, nullptr};
  AttnSplit sp = attention_split(B, H, Hkv, q_cap, kv_cap, ws != nullptr);
  args.chunk = sp.chunk;
  args.items = sp.items;
  args.part_rows = sp.part_rows;
  args.part = static_cast<float*>(ws);
  const int items = (sp.items + kXcdCount - 1) / kXcdCount * kXcdCount;
  hipLaunchKernelGGL(attention_decode_kernel, dim3(items, Hkv), dim3(256), 0, stream, args);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !sp.cuts) return e;
  // a sequence may have several tiles of rows when there are more queries than
  // sequences (else one would have to be empty for each query more)
  const int g = H / Hkv;
  const int tiles = q_cap <= B ? 1 : ((q_cap < kLongQ ? q_cap : kLongQ - 1) * g + kRows - 1) / kRows;
  hipLaunchKernelGGL(attention_combine_kernel, dim3(B, Hkv, tiles < 8 ? tiles : 8), dim3(256), 0, stream, args);
  return hipGetLastError();
}

}  // namespace ce
