// fcm_kernels_v10.h -- DW->PW for few pixels: NHWC, bf16, 3x3 (gfx950).
//
// k_few10<PBK, CT>
//   A workgroup of eight waves computes PBK blocks of 16 consecutive output pixels (of the
//   whole batch: blocks run over rows and images, none is left half empty by a tile's
//   shape) and a block of 16 * CT output channels (PBK * CT <= 8). With a few hundred pixels
//   the persistent and deep kernels have a handful of workgroups, each taking the chunks of
//   input channels one after another, so a launch is that chain: the copies' latency, the
//   stencil, a barrier and the MFMAs per chunk. Here the chunks of the depthwise stage go
//   to the waves in parallel:
//   * DW: wave w takes pixel block w % PBK and the 32-channel chunks w / PBK, + 8 / PBK, ...
//     A lane is an output pixel (l % 16) and an 8-channel slot (l / 16) of the chunk and
//     loads its nine taps (16 bytes each, out-of-range offsets for the padding) from memory
//     to registers, a chunk ahead of the one it filters; one more load brings the slot's
//     weights and biases to the lanes of its 16-lane row, from where DPP broadcasts them as
//     in k_deep7. The result is written to LDS as the MFMA's B operand.
//   * one barrier
//   * PW: wave w < PBK * CT contracts block w / CT with the 16 output channels w % CT over
//     all chunks; the first kPre10 chunks' weights were loaded to registers before the DW
//     stage, each later one is loaded kPre10 chunks ahead.
//   Sums run in the order of k_deep7 (taps in pairs, chunks in sequence, the bias last): a
//   chain gives the same bits whichever of the two runs a pair of layers. (k_fused3 adds the
//   taps one by one: about one output in 1e5 differs in its last place.)
//
//   What bounds it: the launch, then the CU's address unit, 16 cycles a load instruction
//   and as much again where it misses: ten a chunk and pixel block and one a chunk and
//   output tile (7x7x960 -> 160 with eight tiles: 17.7 us, without the tiles' loads 13.1,
//   without eight of nine taps 14.0, without the stencil's arithmetic 17.7). So narrow blocks of
//   output channels pay while CUs are idle although each repeats the DW stage, and the
//   kernel as a whole only until the chip is full (the planner's time model).
#pragma once

#include "fcm_kernels_v8.h"

namespace fcm {

// 16 bytes at a 4-byte boundary
typedef uint32_t u32x4w __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kPre10 = 16;  // chunks of PW weights in flight or in registers

template <int PBK, int CT>
__global__ __launch_bounds__(512) void k_few10(KArgs a) {
  extern __shared__ __align__(16) char smem[];
  constexpr int K = 3, E = 2, MC = 32, DS = 8 / PBK;  // (DS: waves that share a pixel block's chunks)
  using Dw = DwLanes8<TBF16, K>;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int ci_b = a.Ci * E, nch = ceil_div(a.Ci, MC);
  const int np = a.N * a.Ho * a.Wo;

  // ---- this workgroup's pixels and output channels ----
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int cb = lid % a.n_cb, p0 = (lid / a.n_cb) * 16 * PBK;

  // ---- the lane's pixel of the DW stage: the nine taps' offsets ----
  const int db = wave % PBK;
  const rsrc_t rx = make_rsrc(a.x, (uint32_t)(a.N * a.H * a.W * ci_b));
  uint32_t toff[9];
  {
    const int p = p0 + db * 16 + r16, n = p / (a.Ho * a.Wo), q = p - n * a.Ho * a.Wo;
    const int oy = q / a.Wo, ox = q - oy * a.Wo;
    const int iy = oy * a.stride - a.pad, ix = ox * a.stride - a.pad;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int gy = iy + t / K, gx = ix + t % K;
      const bool ok = p < np && (unsigned)gy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W;
      toff[t] = ok ? (uint32_t)(((n * a.H + gy) * a.W + gx) * ci_b + 16 * g) : kOob;
    }
  }
  // weights and biases: lanes 0..8 of a row the slot's 36 words, lanes 9 and 10 its biases
  const char* wbp = r16 < 9 ? (const char*)a.w1 + g * 144 + r16 * 16 : (const char*)a.b1 + g * 32 + (r16 - 9) * 16;
  const int wbs = r16 < 9 ? 576 : 128;  // bytes of a chunk
  const bool wbl = r16 < 9 || (r16 < 11 && a.b1);
  struct Chunk {
    u32x4 x[9], w[1];
  };
  auto load = [&](Chunk& k, int c) {
    const bool in = c * MC + 8 * g < a.Ci;  // (input channels come in eights)
#pragma unroll
    for (int t = 0; t < 9; ++t)
      k.x[t] = __builtin_amdgcn_raw_buffer_load_b128(rx, in ? toff[t] : kOob, (uint32_t)(c * 64), 0);
    k.w[0] = u32x4{0u, 0u, 0u, 0u};
    if (wbl && in) k.w[0] = *(const u32x4w*)(wbp + c * wbs);
  };
  Chunk ka, kb;
  const int c0 = wave / PBK;
  if (c0 < nch) load(ka, c0);

  // ---- the wave's PW role: its weights ahead of the DW stage ----
  const int pb = wave / CT % PBK, tile = cb * CT + wave % CT;
  const bool pw = wave < PBK * CT && tile * 16 < a.Co;  // (uniform)
  const rsrc_t rw = make_rsrc(a.w2, (uint32_t)(a.Co * ci_b));
  const uint32_t woff = tile * 16 + r16 < a.Co ? (uint32_t)((tile * 16 + r16) * ci_b + 16 * g) : kOob;
  auto load_w = [&](int c) {
    return __builtin_amdgcn_raw_buffer_load_b128(rw, c * MC + 8 * g < a.Ci ? woff : kOob, (uint32_t)(c * 64), 0);
  };
  u32x4 wq[kPre10];
#pragma unroll
  for (int k = 0; k < kPre10; ++k) wq[k] = u32x4{0u, 0u, 0u, 0u};
  if (pw) {
#pragma unroll
    for (int k = 0; k < kPre10; ++k)
      if (k < nch) wq[k] = load_w(k);
  }

  // ---- DW ----
  const EpiF8 e1 = make_epif8(a.act[0]);
  auto filter = [&](const Chunk& k, int c) {
    float acc[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[e] = bcast7<9>(k.w[0][e]);
      acc[4 + e] = bcast7<10>(k.w[0][e]);
    }
    static_for7<0, 8>([&](auto jc) {
      constexpr int J = decltype(jc)::value;
      Dw::template channel<J>(acc[J], k.x, k.w);
    });
    u32x4 d;
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = bf16x2_8(acc[2 * q], acc[2 * q + 1], e1);
    *(u32x4*)(smem + (db * nch + c) * 1024 + lane * 16) = d;
  };
  for (int c = c0; c < nch; c += 2 * DS) {
    if (c + DS < nch) load(kb, c + DS);
    filter(ka, c);
    if (c + DS >= nch) break;
    if (c + 2 * DS < nch) load(ka, c + 2 * DS);
    filter(kb, c + DS);
  }
  wait_lgkm0();
  barrier3();
  if (!pw) return;

  // ---- PW ----
  f32x4 acc = {0, 0, 0, 0};
  const char* dl = smem + pb * nch * 1024 + lane * 16;
  for (int c1 = 0; c1 < nch; c1 += kPre10) {
    u32x4 xb[kPre10];
#pragma unroll
    for (int k = 0; k < kPre10; ++k) xb[k] = *(const u32x4*)(dl + min(c1 + k, nch - 1) * 1024);
#pragma unroll
    for (int k = 0; k < kPre10; ++k) {
      if (c1 + k < nch) mma16(TBF16{}, acc, wq[k], xb[k]);
      if (c1 + k + kPre10 < nch) wq[k] = load_w(c1 + k + kPre10);
    }
  }

  const int p = p0 + pb * 16 + r16, co = tile * 16 + 4 * g;
  if (p >= np || co >= a.Co) return;
  const EpiF8 e2 = make_epif8(a.act[1]);
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] += load_bias<TBF16>(a.b2, co + q);
  *(u32x2*)((char*)a.y + ((size_t)p * a.Co + co) * E) =
      u32x2{bf16x2_8(acc[0], acc[1], e2), bf16x2_8(acc[2], acc[3], e2)};
}

template <int PBK, int CT>
int launch_few10(const KArgs& a, int grid, void* stream) {
  const void* fn = (const void*)k_few10<PBK, CT>;
  const int lds = a.L.bytes;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
  }
  return launch_args(fn, grid, 512, lds, stream, a);
}

}  // namespace fcm
