// SwiGLU FFN GEMMs for packed counts between a decode step and a batch (bf16):
// the same gate/up and down products as ce_ffn.hip with the same row maps and
// epilogues, for launches whose 256 x 256 tiles are too few for the chip.
//
// A workgroup of 8 waves owns a tile of 64 kWB weight rows x 32 kM token rows
// (wave (ww, wt): 16 kWB weight rows x 16 kM token rows, MFMA 16x16x32); the
// plan picks the tile so that the workgroups come out in whole rounds of the
// CUs (mid_plan). K streams in 128-byte lines by whole-line DMA through a ring
// of three or four stages; a wave reads its fragments half a stage ahead of the
// products, and one barrier per stage says that the next stage has landed and
// this one is read. Down runs each tile in pieces over K; the pieces' fp32 sums
// go to the workspace and a second launch adds them in piece order, one
// workgroup per row, with the residual and the layer-gap sums (all CUs add,
// where a last-arriving workgroup per tile adds a whole tile by itself).
//
// Bound: the weights from memory below about 160 rows, then the operands' way
// from L2 into LDS. Measured, us, this kernel (down with its second launch) and
// the 256 x 256 tiles: d 1536, d_ff 8960, gate/up 96 rows 16.8 and 32.5, 256
// rows 24 and 37.5, 402 rows 34 and 38; down 96 rows 16 and 48, 402 rows 28 and
// 64, 1024 rows 46 and 77, 2400 rows 78 and 90; d 3584, d_ff 18944, gate/up 96
// rows 71 and 94, 402 rows 139 and 155; down 96 rows 43 and 80, 256 rows 58 and
// 101, 640 rows 120 and 135, 1600 rows 275 and 242 (not taken).
#include <type_traits>

#include "ce_device.hpp"
#include "ce_host.hpp"
#include "ce_launch.hpp"

namespace ce {

namespace {

constexpr int kLine = 128;  // bytes of K per stage and row

__device__ __forceinline__ int map_row(int j, const int32_t* m1, const int32_t* m2) {
  const int r = m1 ? m1[j] : j;
  return m2 ? m2[r] : r;
}

__device__ __forceinline__ void row_counts(const FfnGemmArgs& a, int* kt, int* n0) {
  const bool two_sets = a.n_sets == 2 && a.n0_ptr;
  int k = *a.kt_ptr;
  int n = *(two_sets ? a.n0_ptr : a.kt_ptr);
  k = k < 0 ? 0 : (k > a.cap ? a.cap : k);
  *kt = k;
  *n0 = two_sets ? (n < 0 ? 0 : (n > k ? k : n)) : k;
}

// kMode 0: gate/up + SwiGLU (weight blocks 2i: gate, 2i + 1: up); 1: down
template <int kMode, int kWB, int kM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void ffn_mid_kernel(FfnGemmArgs a,
                                                                                                 int n_tt, int n_ft,
                                                                                                 int pieces) {
  constexpr int kWR = 64 * kWB;  // weight rows of the tile
  constexpr int kTR = 32 * kM;   // token rows
  constexpr int kFT = kMode == 0 ? kWR / 2 : kWR;
  constexpr int kStage = (kWR + kTR) * kLine;
  constexpr int kWI = kWR / 64;          // weight DMA instructions of a wave
  constexpr int kTI = (kTR / 8 + 7) / 8;  // token DMA instructions of a wave
  constexpr int kLoads = kWI + kTI;
  constexpr int kSlots = 4 * kStage <= 160 * 1024 ? 4 : 3;  // stages in the ring
  __shared__ __attribute__((aligned(1024))) char smem[kSlots * kStage];

  const int tid = threadIdx.x;
  if (kMode == 0 && (int)blockIdx.x >= a.copy.first) {
    copy_bypass_rows<8>(a.copy.src, a.copy.dst, a.copy.row_bytes, a.copy.T, a.copy.token_pos,
                        (int)blockIdx.x - a.copy.first, a.copy.blocks);
    return;
  }
  if (a.clear_cnt && blockIdx.x == 0)
    for (int i = tid; i < a.clear_n; i += 512) a.clear_cnt[i] = 0;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ww = wave & 3;
  const int wt = wave >> 2;

  // ---- work item: XCD x = blockIdx % 8 takes a contiguous range of (piece,
  //      feature tile, token tile), token tiles fastest, so the workgroups of
  //      an XCD share weight tiles and a K range through its L2 ----
  const int total = n_tt * n_ft * pieces;
  const int per = (total + kXcdCount - 1) / kXcdCount;
  const int w = (int)(blockIdx.x % kXcdCount) * per + (int)(blockIdx.x / kXcdCount);
  if (w >= total || (int)(blockIdx.x / kXcdCount) >= per) return;
  const int piece = w / (n_tt * n_ft);
  const int rem = w - piece * (n_tt * n_ft);
  const int ft = rem / n_tt;
  const int tt = rem - ft * n_tt;

  int kt, n0;
  row_counts(a, &kt, &n0);
  const int tiles0 = (n0 + kTR - 1) / kTR;
  const int set = tt < tiles0 ? 0 : 1;
  const int row_lo = set ? n0 + (tt - tiles0) * kTR : tt * kTR;
  const int row_hi = set ? min(row_lo + kTR, kt) : min(row_lo + kTR, n0);
  if (row_lo >= row_hi) return;
  const int f0 = ft * kFT;

  // ---- DMA plan: an instruction moves 8 rows x 128 bytes; lane (r8, p) fills
  //      chunk p of its row with source chunk p ^ key(row), so that the 16
  //      rows of a fragment read cover all LDS banks ----
  const int r8 = lane >> 3;
  const int pch = lane & 7;
  const __amdgpu_buffer_rsrc_t wr0 = make_rsrc(set ? a.w0[1] : a.w0[0], (uint32_t)(a.n_feat * a.w_ld));
  const __amdgpu_buffer_rsrc_t wr1 =
      kMode == 0 ? make_rsrc(set ? a.w1[1] : a.w1[0], (uint32_t)(a.n_feat * a.w_ld)) : wr0;
  const __amdgpu_buffer_rsrc_t trs = make_rsrc(a.tok, (uint32_t)(a.tok_rows * a.tok_ld));
  // wave w's weight rows 8 (w + 8 i) .. +7: with gate/up blocks alternating
  // every 16 rows, waves 2, 3, 6, 7 read up rows only
  const bool up = kMode == 0 && (wave & 2) != 0;
  uint32_t wo[kWI], to[kTI], cut[kTI];  // cut: `to` in the channels that pruned rows skip
#pragma unroll
  for (int i = 0; i < kWI; ++i) {
    const int r = 8 * (wave + 8 * i) + r8;
    const int feat = f0 + (kMode == 0 ? 16 * (r >> 5) + (r & 15) : r);
    // features past the last one read zeros (past the buffer's end)
    wo[i] = feat < a.n_feat ? (uint32_t)((int64_t)feat * a.w_ld) + (uint32_t)(pch ^ ((r >> 1) & 7)) * 16 : 0x80000000u;
  }
  auto dma_w = [&](int s, int slot) __attribute__((always_inline)) {
    char* const st = smem + slot * kStage;
#pragma unroll
    for (int i = 0; i < kWI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          up ? wr1 : wr0, (__attribute__((address_space(3))) void*)(st + 8 * (wave + 8 * i) * kLine), 16, (int)wo[i],
          s * kLine, 0, 0);
  };
  // pruned FFN (down): rows that run pruned read zeros from stage ns_keep on,
  // and K ends there for a tile whose rows all do
  int ns = a.k_bytes / kLine;
  int keep = ns;
  if (kMode == 1 && a.row_flag) {
    keep = min(ns, a.ns_keep);
    bool all = true;
#pragma unroll
    for (int i = 0; i < (kTR + 63) / 64; ++i) {
      const int j = row_lo + 64 * i + lane;
      if (j < row_hi) all = all && a.row_flag[a.omap1 ? a.omap1[j] : j] != 0;
    }
    if (__ballot(!all) == 0ull) ns = keep;
  }
  // the first stages' weights go out before the index maps are read
  const int s0 = (int)((int64_t)ns * piece / pieces), s1 = (int)((int64_t)ns * (piece + 1) / pieces);
#pragma unroll
  for (int d = 0; d < kSlots; ++d)
    if (s0 + d < s1) dma_w(s0 + d, d);

  // token instructions past the tile's last one repeat it (same bytes, same place)
  auto tok_q = [&](int i) __attribute__((always_inline)) { return min(wave + 8 * i, kTR / 8 - 1); };
  {
    int src[kTI];
#pragma unroll
    for (int i = 0; i < kTI; ++i) {
      const int j = row_lo + 8 * tok_q(i) + r8;
      src[i] = j < row_hi ? j : -1;
    }
    if (a.map1) {
#pragma unroll
      for (int i = 0; i < kTI; ++i) {
        const int v = a.map1[src[i] < 0 ? 0 : src[i]];
        src[i] = src[i] < 0 ? -1 : v;
      }
    }
    if (a.map2) {
#pragma unroll
      for (int i = 0; i < kTI; ++i) {
        const int v = a.map2[src[i] < 0 ? 0 : src[i]];
        src[i] = src[i] < 0 ? -1 : v;
      }
    }
#pragma unroll
    for (int i = 0; i < kTI; ++i) {
      const int r = 8 * tok_q(i) + r8;
      to[i] = src[i] < 0 ? 0x80000000u
                         : (uint32_t)((int64_t)src[i] * a.tok_ld) + (uint32_t)(pch ^ ((r >> 1) & 7)) * 16;
      cut[i] = to[i];
      const int j = row_lo + r;
      if (kMode == 1 && a.row_flag && j < row_hi && a.row_flag[a.omap1 ? a.omap1[j] : j] != 0) cut[i] = 0x80000000u;
    }
  }
  auto dma_t = [&](int s, int slot) __attribute__((always_inline)) {
    char* const st = smem + slot * kStage;
    const bool tail = kMode == 1 && s >= keep;
#pragma unroll
    for (int i = 0; i < kTI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          trs, (__attribute__((address_space(3))) void*)(st + (kWR + 8 * tok_q(i)) * kLine), 16,
          (int)(tail ? cut[i] : to[i]), s * kLine,
          0, 0);
  };
#pragma unroll
  for (int d = 0; d < kSlots; ++d)
    if (s0 + d < s1) dma_t(s0 + d, d);

  f32x4_t acc[kWB][kM];
#pragma unroll
  for (int i = 0; i < kWB; ++i)
#pragma unroll
    for (int j = 0; j < kM; ++j) acc[i][j] = f32x4_t{};
  const int l16 = lane & 15;
  const int lq = lane >> 4;

  // this wave's part of stage s + 1 has landed: behind it are in flight the
  // later stages up to s + kSlots - 1, of which those of the prologue count
  // with their token part only (all weights went out before)
  auto landed = [&](int s) __attribute__((always_inline)) {
    const int later = min(kSlots - 2, s1 - 2 - s);
    const int pro = kSlots - 2 - (s - s0);  // of those, the prologue's
    if (later >= 2) {
      if (pro <= 0) wait_vmcnt<2 * kLoads>();
      else if (pro == 1) wait_vmcnt<kLoads + kTI>();
      else wait_vmcnt<2 * kTI>();
    } else if (later == 1) {
      if (pro <= 0) wait_vmcnt<kLoads>();
      else wait_vmcnt<kTI>();
    } else {
      wait_vmcnt<0>();
    }
  };
  u32x4_t fa[2][kWB], fb[2][kM];
  // fragments of K half h of the stage in `slot` (their offset through an
  // empty asm: the compiler would drain every DMA in flight before an LDS read
  // it can tie to the ring)
  auto frags = [&](int slot, auto hc) __attribute__((always_inline)) {
    constexpr int H = decltype(hc)::value;
    uint32_t fo = (uint32_t)(slot * kStage + l16 * kLine) + ((uint32_t)((lq + 4 * H) ^ ((l16 >> 1) & 7)) << 4);
    asm volatile("" : "+v"(fo));
#pragma unroll
    for (int j = 0; j < kM; ++j)
      fb[H][j] = *reinterpret_cast<const u32x4_t*>(smem + fo + (kWR + 16 * (kM * wt + j)) * kLine);
#pragma unroll
    for (int i = 0; i < kWB; ++i)
      fa[H][i] = *reinterpret_cast<const u32x4_t*>(smem + fo + (16 * (kWB * ww + i)) * kLine);
  };
  auto mul = [&](auto hc) __attribute__((always_inline)) {
    constexpr int H = decltype(hc)::value;
#pragma unroll
    for (int i = 0; i < kWB; ++i)
#pragma unroll
      for (int j = 0; j < kM; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fa[H][i]),
                                                            __builtin_bit_cast(bf16x8_t, fb[H][j]), acc[i][j], 0, 0, 0);
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  // (tokens follow all weights here: stage s0 has landed when the token parts
  // of the later stages are all that is in flight)
  if (s0 < s1) {
    const int later = min(kSlots - 1, s1 - 1 - s0);
    if (later >= 3) wait_vmcnt<3 * kTI>();
    else if (later == 2) wait_vmcnt<2 * kTI>();
    else if (later == 1) wait_vmcnt<kTI>();
    else wait_vmcnt<0>();
  }
  lds_barrier();
  frags(0, H0{});
  // (scalar loads still in flight share the LDS reads' counter and would make
  // the loop wait for every read)
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14));
  int slot = 0;
  // the second half's reads run under the first half's products, and the next
  // stage's first reads under the second half's (the last stage apart: a
  // branch in the loop would make the compiler wait for both at once)
  for (int s = s0; s < s1 - 1; ++s) {
    frags(slot, H1{});
    __builtin_amdgcn_sched_barrier(0);
    mul(H0{});
    __builtin_amdgcn_sched_barrier(0);
    landed(s);
    lds_barrier();  // stage s + 1 is there and every wave has read stage s
    __builtin_amdgcn_sched_barrier(0);
    if (s + kSlots < s1) {
      dma_w(s + kSlots, slot);
      dma_t(s + kSlots, slot);
    }
    slot = slot == kSlots - 1 ? 0 : slot + 1;
    frags(slot, H0{});
    __builtin_amdgcn_sched_barrier(0);
    mul(H1{});
    __builtin_amdgcn_sched_barrier(0);
  }
  if (s0 < s1) {  // (a piece of a pruned tile can be empty: its sums are zero)
    frags(slot, H1{});
    mul(H0{});
    mul(H1{});
  }

  // ---- epilogue: lane l, element v of block (i, j) is weight row
  //      16 i + 4 (l / 16) + v of the wave's, token row 16 j + l % 16 ----
#pragma unroll
  for (int j = 0; j < kM; ++j) {
    const int jr = row_lo + 16 * (kM * wt + j) + l16;
    if (jr >= row_hi) continue;
    if constexpr (kMode == 0) {
      char* const orow = a.out + (int64_t)map_row(jr, a.omap1, a.omap2) * a.out_ld;
#pragma unroll
      for (int i = 0; i < kWB / 2; ++i) {
        const int f = f0 + 16 * (kWB / 2 * ww + i) + 4 * lq;
        if (f >= a.n_feat) continue;
        const f32x4_t g = acc[2 * i][j], u = acc[2 * i + 1][j];
        store4<true>(orow + (int64_t)f * 2, silu_f32(g.x) * u.x, silu_f32(g.y) * u.y, silu_f32(g.z) * u.z,
                     silu_f32(g.w) * u.w);
      }
    } else {
      float* const prow = a.part + ((int64_t)piece * a.cap + jr) * a.n_feat;
#pragma unroll
      for (int i = 0; i < kWB; ++i) {
        const int f = f0 + 16 * (kWB * ww + i) + 4 * lq;
        if (f < a.n_feat) *reinterpret_cast<f32x4_t*>(prow + f) = acc[i][j];
      }
    }
  }
}

// out[row] = sum of the pieces in order (+ residual), one workgroup per packed
// row, four features per thread; with gap_part the row's layer-gap sums in one slot.
__global__ __launch_bounds__(256) void ffn_mid_add_kernel(FfnGemmArgs a, int pieces) {
  __shared__ double red[4][3];
  const int j = blockIdx.x;
  int kt, n0;
  row_counts(a, &kt, &n0);
  if (j >= kt) return;
  const int64_t oi = map_row(j, a.omap1, a.omap2);
  char* const orow = a.out + oi * a.out_ld;
  const float* const p = a.part + (int64_t)j * a.n_feat;
  const int64_t step = (int64_t)a.cap * a.n_feat;  // floats between pieces
  double gdot = 0.0, gin = 0.0, gout = 0.0;
  for (int f = 4 * (int)threadIdx.x; f < a.n_feat; f += 1024) {
    f32x4_t res = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.res) res = load4<true>(a.res + oi * a.res_ld + (int64_t)f * 2);
    f32x4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int c0 = 0; c0 < pieces; c0 += 8) {
      f32x4_t x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        x[i] = *reinterpret_cast<const f32x4_t*>(p + min(c0 + i, pieces - 1) * step + f);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (c0 + i < pieces) v += x[i];
    }
    v += res;
    const u32x2_t pk = {pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
    *reinterpret_cast<u32x2_t*>(orow + (int64_t)f * 2) = pk;
    if (a.gap_part) {
      // the values as stored, after the one rounding
      const float y[4] = {bf16_to_f32(pk.x & 0xffffu), bf16_to_f32(pk.x >> 16), bf16_to_f32(pk.y & 0xffffu),
                          bf16_to_f32(pk.y >> 16)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        gdot = fma((double)res[e], (double)y[e], gdot);
        gin = fma((double)res[e], (double)res[e], gin);
        gout = fma((double)y[e], (double)y[e], gout);
      }
    }
  }
  if (!a.gap_part) return;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    gdot += __shfl_xor(gdot, o);
    gin += __shfl_xor(gin, o);
    gout += __shfl_xor(gout, o);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[wave][0] = gdot;
    red[wave][1] = gin;
    red[wave][2] = gout;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int prow = a.omap1 ? a.omap1[j] : j;
    a.gap_part[(int64_t)prow * a.gap_np * 4 + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
  }
}

template <int kMode, int kWB, int kM>
hipError_t launch_mid(FfnGemmArgs a, int pieces, hipStream_t stream) {
  constexpr int kFT = kMode == 0 ? 32 * kWB : 64 * kWB;
  const int n_tt = (a.cap + 32 * kM - 1) / (32 * kM) + (a.n_sets - 1);
  const int n_ft = (a.n_feat + kFT - 1) / kFT;
  const int grid = grid_with_copy(a.copy, (n_tt * n_ft * pieces + kXcdCount - 1) / kXcdCount * kXcdCount);
  hipLaunchKernelGGL((ffn_mid_kernel<kMode, kWB, kM>), dim3(grid), dim3(512), 0, stream, a, n_tt, n_ft, pieces);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || kMode == 0) return e;
  hipLaunchKernelGGL(ffn_mid_add_kernel, dim3(a.cap), dim3(256), 0, stream, a, pieces);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_mid(const FfnGemmArgs& a, int mode, const MidPlan& p, hipStream_t stream) {
  if (mode == 0 && p.wb == 4) {
    switch (p.m) {
      case 3: return launch_mid<0, 4, 3>(a, 1, stream);
      case 4: return launch_mid<0, 4, 4>(a, 1, stream);
      default: return launch_mid<0, 4, 5>(a, 1, stream);
    }
  }
  if (mode == 0) {
    switch (p.m) {
      case 2: return launch_mid<0, 2, 2>(a, 1, stream);
      case 3: return launch_mid<0, 2, 3>(a, 1, stream);
      case 4: return launch_mid<0, 2, 4>(a, 1, stream);
      case 5: return launch_mid<0, 2, 5>(a, 1, stream);
      case 6: return launch_mid<0, 2, 6>(a, 1, stream);
      default: return launch_mid<0, 2, 8>(a, 1, stream);
    }
  }
  switch (p.m) {
    case 2: return launch_mid<1, 2, 2>(a, p.pieces, stream);
    case 3: return launch_mid<1, 2, 3>(a, p.pieces, stream);
    case 4: return launch_mid<1, 2, 4>(a, p.pieces, stream);
    case 5: return launch_mid<1, 2, 5>(a, p.pieces, stream);
    case 6: return launch_mid<1, 2, 6>(a, p.pieces, stream);
    default: return launch_mid<1, 2, 8>(a, p.pieces, stream);
  }
}

}  // namespace ce
