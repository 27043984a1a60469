// Attention over the packed retained tokens of a routed layer (paper section
// 3.4, task-adaptive token compaction: the retained tokens are packed into a
// shorter sequence for the layer's attention and FFN; for understanding the
// packed keys / values of the routed layers are the compressed key-value cache
// that decoding reuses).
//
//   O_b[:, h] = softmax(scale * Q_b[:, h] K_b[:, kv(h)]^T + M) V_b[:, kv(h)]
//
// per sequence b (packed rows q_offsets[b] .. q_offsets[b+1] of Q / O and
// kv_offsets[b] .. of K / V), query head h, key/value head kv(h) = h / (H / H_kv).
// M is 0, or with causal masking -inf for keys after the query, end-aligned:
// query i of n_q sits at key position n_kv - n_q + i. A query that sees no key
// outputs zeros.
//
// The kernel looks its query tile up and runs it (ce_attention_tile.hpp: the
// tile's design, its bounds and what it measured).
#include "ce_attention_tile.hpp"
#include "ce_launch.hpp"

namespace ce {

namespace {

using namespace attn;

// Exclusive prefix sum over the 256 threads of the workgroup, plus the total
// (scr: 4 ints of LDS). Every thread must call it.
__device__ __forceinline__ int excl_scan256(int v, int* scr, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) scr[wave] = x;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before += scr[w];
  total = (scr[0] + scr[1]) + (scr[2] + scr[3]);
  __syncthreads();
  return before + x - v;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attention_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) char smem[4 * kKBytes];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- which sequence and query tile: up to 64 sequences by a scan of their
  //      tile counts inside each wave (one load and no barrier); more, 256 at a
  //      time (one per thread, a block scan; a chunk below this workgroup's tile
  //      is skipped whole, and the next chunk's offsets are loaded before the
  //      scan). The LDS is free until the first K tile. ----
  const int t = blockIdx.x;
  int b = -1, q0 = 0, nq = 0, qbase = 0;
  if (a.B <= 64) {
    int lo = 0, hi = 0;
    if (lane < a.B) {
      lo = clampi(a.qo[lane], 0, a.q_cap);
      hi = clampi(a.qo[lane + 1], lo, a.q_cap);
    }
    const int nt = (hi - lo + kQT - 1) / kQT;
    int end = nt;  // tiles up to and with this lane's sequence
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(end, o);
      if (lane >= o) end += y;
    }
    const uint64_t past = __builtin_amdgcn_ballot_w64(t < end);
    if (past) {
      b = __builtin_ctzll(past);
      q0 = (__builtin_amdgcn_readlane(end, b) - 1 - t) * kQT;  // last tiles first: under a causal mask they see the most keys
      qbase = __builtin_amdgcn_readlane(lo, b);
      nq = __builtin_amdgcn_readlane(hi, b) - qbase;
    }
  } else {
    int* const wsh = reinterpret_cast<int*>(smem);
    int lo = 0, hi = 0;
    if (tid < a.B) {
      lo = clampi(a.qo[tid], 0, a.q_cap);
      hi = clampi(a.qo[tid + 1], lo, a.q_cap);
    }
    int base = 0;  // tiles of the chunks before
    for (int s0 = 0; s0 < a.B; s0 += 256) {
      const int cnt = min(256, a.B - s0);
      const int clo = lo, chi = hi;
      if (s0 + 256 + tid < a.B) {
        lo = clampi(a.qo[s0 + 256 + tid], 0, a.q_cap);
        hi = clampi(a.qo[s0 + 256 + tid + 1], lo, a.q_cap);
      }
      const int nt = tid < cnt ? (chi - clo + kQT - 1) / kQT : 0;
      int total;
      const int ex = excl_scan256(nt, wsh, total);
      if (t < base + total) {
        if (tid < cnt && t >= base + ex && t < base + ex + nt) {
          wsh[4] = s0 + tid;
          wsh[5] = (nt - 1 - (t - base - ex)) * kQT;  // last tiles first: under a causal mask they see the most keys
          wsh[6] = chi - clo;
          wsh[7] = clo;
        }
        __syncthreads();
        b = wsh[4];
        q0 = wsh[5];
        nq = wsh[6];
        qbase = wsh[7];
        __syncthreads();  // the LDS goes to the K / V tiles
        break;
      }
      base += total;
    }
  }
  if (b < 0) return;
  b = __builtin_amdgcn_readfirstlane(b);
  q0 = __builtin_amdgcn_readfirstlane(q0);
  nq = __builtin_amdgcn_readfirstlane(nq);
  qbase = __builtin_amdgcn_readfirstlane(qbase);
  attention_tile<false>(a, smem, b, blockIdx.y, q0, nq, qbase);
}

}  // namespace

hipError_t launch_attention(const char* q, const char* k, const char* v, char* o, const int32_t* q_offsets,
                            const int32_t* kv_offsets, int B, int H, int Hkv, int q_cap, int kv_cap, bool causal,
                            float scale, hipStream_t stream) {
  if (q_cap <= 0) return hipSuccess;
  const int tiles = (q_cap + kQT - 1) / kQT + B;  // each sequence adds at most one partial tile
  AttnArgs args{q, k, v, o, q_offsets, kv_offsets, B, H, Hkv, q_cap, kv_cap, causal ? 1 : 0,
                scale * 1.4426950408889634f};
  hipLaunchKernelGGL(attention_kernel, dim3(tiles, H), dim3(256), 0, stream, args);
  return hipGetLastError();
}

}  // namespace ce
