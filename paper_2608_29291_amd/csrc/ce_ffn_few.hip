// SwiGLU FFN GEMMs for few packed rows (decode steps: one token per running
// request; small fp32 batches, in tiles of 16 or 32 rows): the same gate/up and
// down products as ce_ffn.hip with the same row maps and epilogues.
//
// Bound: the weights, each read once. A 256 x 256 tile kernel streams 256
// token rows through LDS for a handful of rows and fills a fraction of the
// CUs; here a workgroup owns 16 output features (or 32, gate/up above 16 rows)
// of all the rows and its waves split K by 128-byte lines (wave w of W takes
// lines w, w + W, ...: consecutive lines of a weight row are in flight at
// once). Every wave has an LDS ring of its own, filled by whole-line DMA, so
// the K loop has no barrier; the waves' sums meet in LDS at the end, added in
// wave order (deterministic), where the epilogue runs. Operands loaded
// straight to registers in MFMA order touch 16 lines per quarter wave and
// reached 4.2 TB/s; the DMA takes 5.3.
//
// Measured at the 7B width (d 3584, d_ff 18944, 407 MB of weights), gate/up +
// down in us, this kernel and the 256 x 256 tiles: 4 rows 50 + 28 and 85 + 64,
// 16 rows 51 + 31 and 86 + 62, 32 rows 62 + 43 and 88 + 63, 64 rows 72 + 55 and
// 88 + 77; at d 1536, d_ff 8960: 16 rows 13 + 10 and 29 + 35, 64 rows 22 + 18
// and 34 + 48. Two workgroups on a CU hide each other's start (gate/up with
// one of 8 waves per CU: 60 us).
#include "ce_device.hpp"
#include "ce_host.hpp"
#include "ce_launch.hpp"

namespace ce {

namespace {

constexpr int kLine = 128;  // bytes of K per step of a wave: two 16x16x32 MFMAs
constexpr int kBlk = 16 * kLine;  // one block of 16 rows in LDS

// One 16-byte chunk per lane of both operands on a 16 x 16 block: lane l holds
// chunk l / 16 of row l % 16 (bf16: K = 32; fp32: four products of K = 4).
template <bool kBF16>
__device__ __forceinline__ void mfma16_step(f32x4_t& acc, const u32x4_t& a, const u32x4_t& b) {
  if constexpr (kBF16) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                  acc, 0, 0, 0);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
  }
}

__device__ __forceinline__ int map_row(int j, const int32_t* m1, const int32_t* m2) {
  const int r = m1 ? m1[j] : j;
  return m2 ? m2[r] : r;
}

// kMode 0: gate/up + SwiGLU over kF blocks of 16 features (blocks 2i: gate,
// 2i + 1: up); 1: down (+ residual, layer-gap sums) over one block.
// kNB: blocks of 16 token rows. kW waves, each with a ring of kD steps.
template <bool kBF16, int kMode, int kF, int kNB, int kW, int kD>
__global__ __launch_bounds__(64 * kW) void ffn_few_kernel(FfnGemmArgs a) {
  constexpr int kR = kMode == 0 ? 2 * kF : kF;  // blocks of 16 weight rows
  static_assert(kMode == 0 || kF == 1, "down: one block of features");
  constexpr int kStep = (kR + kNB) * kBlk;  // bytes of one step of a wave
  constexpr int kLoads = 2 * (kR + kNB);    // DMA instructions of one step
  __shared__ __attribute__((aligned(1024))) char smem[kW * kD * kStep];
  static_assert(kW * kR * kNB * 1024 <= kW * kD * kStep, "the sums fit where the rings were");

  const int tid = threadIdx.x;
  if (kMode == 0 && (int)blockIdx.x >= a.copy.first) {
    if (blockIdx.y == 0 && blockIdx.z == 0)
      copy_bypass_rows<kW>(a.copy.src, a.copy.dst, a.copy.row_bytes, a.copy.T, a.copy.token_pos,
                           (int)blockIdx.x - a.copy.first, a.copy.blocks);
    return;
  }
  if (a.clear_cnt && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
    for (int i = tid; i < a.clear_n; i += 64 * kW) a.clear_cnt[i] = 0;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = blockIdx.y;

  int kt = *a.kt_ptr;
  const bool two_sets = a.n_sets == 2 && a.n0_ptr;
  int n0 = *(two_sets ? a.n0_ptr : a.kt_ptr);
  kt = kt < 0 ? 0 : (kt > a.cap ? a.cap : kt);
  n0 = two_sets ? (n0 < 0 ? 0 : (n0 > kt ? kt : n0)) : kt;
  constexpr int kElem = kBF16 ? 2 : 4;
  const int row_lo = (set ? n0 : 0) + (int)blockIdx.z * (16 * kNB);
  const int row_hi = min(row_lo + 16 * kNB, set ? kt : n0);
  if (row_lo >= row_hi) return;

  // ---- DMA plan: an instruction moves 8 rows x 128 bytes, whole lines; lane
  //      (r8, p) fills chunk p of row r8 with source chunk p ^ key(row), so
  //      that the 16 rows of a fragment read cover all LDS banks ----
  const int f0 = blockIdx.x * (16 * kF);
  const int r8 = lane >> 3;
  const int pch = lane & 7;
  uint32_t wo[kR][2], to[kNB][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = 8 * h + r8;  // row of the block
    const uint32_t c = (uint32_t)(pch ^ ((r >> 1) & 7)) * 16;
#pragma unroll
    for (int b = 0; b < kR; ++b)
      wo[b][h] = (uint32_t)((int64_t)(f0 + 16 * (kMode == 0 ? b >> 1 : b) + r) * a.w_ld) + c;
    // rows past the last one read zeros (past the buffer's end)
#pragma unroll
    for (int n = 0; n < kNB; ++n) {
      const int j = row_lo + 16 * n + r;
      to[n][h] = j < row_hi ? (uint32_t)((int64_t)map_row(j, a.map1, a.map2) * a.tok_ld) + c : 0x80000000u;
    }
  }
  const char* const w0 = set ? a.w0[1] : a.w0[0];
  const char* const w1 = set ? a.w1[1] : a.w1[0];
  const uint32_t w_bytes = (uint32_t)(a.n_feat * a.w_ld), t_bytes = (uint32_t)(a.tok_rows * a.tok_ld);
  // pruned FFN (down): rows that run pruned read zeros from line ns_keep on, and
  // K ends there when all rows do
  int ns = a.k_bytes / kLine;
  int keep = ns;
  uint32_t cut[kNB][2];
#pragma unroll
  for (int n = 0; n < kNB; ++n) cut[n][0] = to[n][0], cut[n][1] = to[n][1];
  if (kMode == 1 && a.row_flag) {
    keep = min(ns, a.ns_keep);
    auto flag = [&](int j) __attribute__((always_inline)) { return a.row_flag[a.omap1 ? a.omap1[j] : j] != 0; };
#pragma unroll
    for (int n = 0; n < kNB; ++n)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = row_lo + 16 * n + 8 * h + r8;
        if (j < row_hi && flag(j)) cut[n][h] = 0x80000000u;
      }
    if (__ballot(row_lo + lane < row_hi && !flag(min(row_lo + lane, row_hi - 1))) == 0ull) ns = keep;
  }
  char* const ring = smem + wave * (kD * kStep);

  // step s of this wave into ring slot d; past the last step an empty buffer
  // (zeros, no traffic) keeps the loop free of branches
  auto dma = [&](int s, int d) __attribute__((always_inline)) {
    const bool in = s < ns;
    const bool tail = kMode == 1 && s >= keep;
    const __amdgpu_buffer_rsrc_t r0 = make_rsrc(w0, in ? w_bytes : 0u);
    const __amdgpu_buffer_rsrc_t r1 = make_rsrc(kMode == 0 ? w1 : w0, in ? w_bytes : 0u);
    const __amdgpu_buffer_rsrc_t rt = make_rsrc(a.tok, in ? t_bytes : 0u);
    char* const to_lds = ring + d * kStep;
#pragma unroll
    for (int b = 0; b < kR + kNB; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            b >= kR ? rt : ((kMode == 0 && (b & 1)) ? r1 : r0),
            (__attribute__((address_space(3))) void*)(to_lds + b * kBlk + h * (kBlk / 2)), 16,
            (int)(b >= kR ? (tail ? cut : to)[b >= kR ? b - kR : 0][h] : wo[b < kR ? b : 0][h]), s * kLine, 0, 0);
  };

  f32x4_t acc[kR][kNB];
#pragma unroll
  for (int r = 0; r < kR; ++r)
#pragma unroll
    for (int n = 0; n < kNB; ++n) acc[r][n] = f32x4_t{};

  const int l16 = lane & 15;
  const int lq = lane >> 4;
#pragma unroll
  for (int d = 0; d < kD; ++d) {
    dma(wave + kW * d, d);
    __builtin_amdgcn_sched_barrier(0);  // in slot order: the loop waits for the oldest only
  }
  for (int s = wave; s < ns; s += kW * kD) {
#pragma unroll
    for (int d = 0; d < kD; ++d) {
      wait_vmcnt<(kD - 1) * kLoads>();
      __builtin_amdgcn_sched_barrier(0);
      // (the fragment offset through an empty asm: the compiler would drain
      // every DMA in flight before an LDS read it can tie to the ring)
      uint32_t fo = (uint32_t)(l16 * kLine) + ((uint32_t)(lq ^ ((l16 >> 1) & 7)) << 4);
      asm volatile("" : "+v"(fo));
      const char* const base = ring + d * kStep;
      u32x4_t f[2][kR + kNB];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < kR + kNB; ++b)
          f[h][b] = *reinterpret_cast<const u32x4_t*>(base + (fo ^ (64 * h)) + b * kBlk);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < kR; ++r)
#pragma unroll
          for (int n = 0; n < kNB; ++n)
            mfma16_step<kBF16>(acc[r][n], f[h][r], f[h][kR + n]);
      // every fragment is in registers: the slot takes the step kD ahead
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      dma(s + kW * (kD + d), d);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  wait_vmcnt<0>();  // the last steps' zeros
  __syncthreads();
  f32x4_t (*const red)[kR * kNB][64] = reinterpret_cast<f32x4_t(*)[kR * kNB][64]>(smem);

  // ---- the waves' sums: lane l, element v of block (r, n) is feature
  //      16 r + 4 (l / 16) + v of row 16 n + l % 16 ----
#pragma unroll
  for (int r = 0; r < kR; ++r)
#pragma unroll
    for (int n = 0; n < kNB; ++n) red[wave][r * kNB + n][lane] = acc[r][n];
  __syncthreads();
  auto total = [&](int t) __attribute__((always_inline)) {
    f32x4_t x = red[0][t][lane];
#pragma unroll
    for (int w = 1; w < kW; ++w) x += red[w][t][lane];
    return x;
  };
  for (int u = wave; u < kF * kNB; u += kW) {
    const int i = u / kNB, n = u - i * kNB;  // feature block, row block
    const int jr = row_lo + 16 * n + l16;
    const int f = f0 + 16 * i + 4 * lq;
    if constexpr (kMode == 0) {
      const f32x4_t g = total(2 * i * kNB + n), up = total((2 * i + 1) * kNB + n);
      if (jr < row_hi)
        store4<kBF16>(a.out + (int64_t)map_row(jr, a.omap1, a.omap2) * a.out_ld + (int64_t)f * kElem,
                      silu_f32(g.x) * up.x, silu_f32(g.y) * up.y, silu_f32(g.z) * up.z, silu_f32(g.w) * up.w);
    } else {
      f32x4_t v = total(n);
      const bool in = jr < row_hi;
      double gdot = 0.0, gin = 0.0, gout = 0.0;  // layer-gap sums over this lane's features
      if (in) {
        const int64_t oi = map_row(jr, a.omap1, a.omap2);
        char* const orow = a.out + oi * a.out_ld + (int64_t)f * kElem;
        f32x4_t res = {0.0f, 0.0f, 0.0f, 0.0f};
        if (a.res) res = load4<kBF16>(a.res + oi * a.res_ld + (int64_t)f * kElem);
        v += res;
        store4<kBF16>(orow, v.x, v.y, v.z, v.w);
        if (a.gap_part) {
          // the values as stored (bf16: after the one rounding)
          float y[4] = {v.x, v.y, v.z, v.w};
          if constexpr (kBF16) {
            const u32x2_t pk = {pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
            y[0] = bf16_to_f32(pk.x & 0xffffu), y[1] = bf16_to_f32(pk.x >> 16);
            y[2] = bf16_to_f32(pk.y & 0xffffu), y[3] = bf16_to_f32(pk.y >> 16);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            gdot = fma((double)res[e], (double)y[e], gdot);
            gin = fma((double)res[e], (double)res[e], gin);
            gout = fma((double)y[e], (double)y[e], gout);
          }
        }
      }
      if (a.gap_part) {
        // lanes 16 apart hold the row's other features of this block
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
          gdot += __shfl_xor(gdot, o);
          gin += __shfl_xor(gin, o);
          gout += __shfl_xor(gout, o);
        }
        if (in && lq == 0) {
          const int prow = a.omap1 ? a.omap1[jr] : jr;
          double* gp = a.gap_part + ((int64_t)prow * a.gap_np + blockIdx.x) * 4;
          gp[0] = gdot;
          gp[1] = gin;
          gp[2] = gout;
        }
      }
    }
  }
}

template <bool kBF16, int kMode, int kF, int kNB, int kW, int kD>
hipError_t launch_few(FfnGemmArgs a, hipStream_t stream) {
  const int grid = grid_with_copy(a.copy, a.n_feat / (16 * kF));
  hipLaunchKernelGGL((ffn_few_kernel<kBF16, kMode, kF, kNB, kW, kD>), dim3(grid, a.n_sets, (a.cap + 16 * kNB - 1) / (16 * kNB)), dim3(64 * kW), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_few(const FfnGemmArgs& a, int mode, bool bf16, hipStream_t stream) {
  if (!bf16) return mode == 0 ? launch_few<false, 0, 1, 2, 4, 2>(a, stream) : launch_few<false, 1, 1, 1, 8, 3>(a, stream);
  if (mode == 0) {
    if (a.cap <= 16) return launch_few<true, 0, 1, 1, 4, 3>(a, stream);
    if (a.cap <= 32) return launch_few<true, 0, 2, 2, 4, 3>(a, stream);
    return launch_few<true, 0, 2, 4, 4, 2>(a, stream);
  }
  if (a.cap <= 16) return launch_few<true, 1, 1, 1, 8, 4>(a, stream);
  if (a.cap <= 32) return launch_few<true, 1, 1, 2, 8, 3>(a, stream);
  return launch_few<true, 1, 1, 4, 8, 2>(a, stream);
}

}  // namespace ce
