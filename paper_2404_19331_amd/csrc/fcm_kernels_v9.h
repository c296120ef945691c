// fcm_kernels_v9.h -- DW->PW module on NCHW, every element type (gfx950).
//
// k_dwpw9<DT, K, CT, PB>
//   A workgroup of four waves computes one TH x TW output tile (run time) of one image and a
//   block of 16 * CT output channels. The input channels go through it in chunks of MC = 64
//   bytes: the chunk's haloed window and its pointwise weight rows are loaded into registers
//   while the previous chunk is computed, then written to LDS (both double buffered, one
//   barrier a chunk; loads two chunks ahead were no faster); the depthwise stage reads the window and its result is the MFMA's B
//   operand without leaving the registers. GW waves form a group (a 16-pixel block or two
//   each) and the J = 4 / GW groups share the chunks, as in k_ir8.
//
//   The window is held [position][16-byte slots of channels] (int8 in the order of k_ir8's
//   exchange: byte 4t + v of slot s is channel 16t + 4s + v): a lane gathers
//   the channels of its slot at one position, one element load each with the channel in the
//   scalar offset, so that a wave's lanes read consecutive pixels of a plane, no alignment
//   of planes or rows is needed, and the loop has no index arithmetic. (Element-wise
//   staging with three divisions an element bounded the first-generation kernel.) Weight
//   rows of any length are read as 16 bytes, words or elements.
//
//   Depthwise: bf16 dot instructions on pairs of taps and fp32 multiply-adds take the
//   weights by DPP broadcast within the 16-lane rows, each row holding its own slot's;
//   int8 runs on the matrix cores with diagonal weights (see k_ir8).
//
//   What bounds it: the chain of chunks (element loads, one instruction per element of the
//   window; barrier; stencil), with one or two workgroups on a CU.
#pragma once

#include "fcm_kernels_v8.h"

namespace fcm {

// How the rows of a matrix can be read: whole 16 bytes, words, or elements.
enum { ROWS_VEC = 0, ROWS_WORDS = 1, ROWS_ELEMENTS = 2 };

template <class DT, int K, int CT, int PB>
__global__ __launch_bounds__(256) void k_dwpw9(KArgs a) {
  extern __shared__ __align__(16) char smem[];
  constexpr bool I8 = std::is_same<DT, TI8>::value;
  constexpr bool F32 = std::is_same<DT, TF32>::value;
  using AccV = typename DT::AccV;
  constexpr int E = DT::ELT, MC = 64 / E, CPG = 16 / E;
  constexpr int KK = K * K;
  constexpr int EP = kPitchE8;
  constexpr int NX = window_vecs9(dtype_id<DT>()), NWV = kWeightVecs9;

  const int S = a.stride, TW = a.TW, P = a.TH * TW;
  const int IH = (a.TH - 1) * S + K, IW = (TW - 1) * S + K, Q = IH * IW;
  const int J = a.splits, GW = a.gw;
  const Lds9 lay = lds9(dtype_id<DT>(), K, S, a.TH, TW, a.Ci, GW, J, PB, CT);
  const int ci_b = a.Ci * E, hw = a.H * a.W;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int nw = GW * J;
  const int j = wave / GW, w = wave % GW;
  const int gt = w * 64 + lane, ng = 64 * GW;  // thread of the group, threads per group

  // ---- this workgroup's tile and output-channel block ----
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int co0 = (lid % a.n_cb) * 16 * CT;
  int t = lid / a.n_cb;
  const int tx = t % a.tiles_x;
  t /= a.tiles_x;
  const int ty = t % a.tiles_y, n = t / a.tiles_y;
  const int oy0 = ty * a.TH, ox0 = tx * TW;
  const int iy0 = oy0 * S - a.pad, ix0 = ox0 * S - a.pad;
  const int nch = ceil_div(a.Ci, MC);

  // ---- the group's share of a chunk: window slots (i: position and slot), weight slots
  // (i: row of the block and slot); offsets without the chunk ----
  const size_t img = (size_t)hw * ci_b;
  const rsrc_t rx = make_rsrc((const char*)a.x + (size_t)n * img, (uint32_t)img);
  const rsrc_t rw = make_rsrc(a.w2, (uint32_t)(a.Co * ci_b));
  uint32_t xoff[NX], woff[NWV];
  int xdst[NX], wdst[NWV];
#pragma unroll
  for (int k = 0; k < NX; ++k) {
    const int i = gt + k * ng;
    const int pos = i % lay.nqp, sl = i / lay.nqp;
    const int qy = pos / IW, qx = pos - qy * IW;
    const int gy = iy0 + qy, gx = ix0 + qx;
    const bool ok = pos < Q && (unsigned)gy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W;
    xdst[k] = i < 4 * lay.nqp ? pos * EP + sl * 16 : -1;
    xoff[k] = ok && i < 4 * lay.nqp ? (uint32_t)((sl * (I8 ? 4 : CPG) * hw + gy * a.W + gx) * E) : kOob;
  }
#pragma unroll
  for (int k = 0; k < NWV; ++k) {
    const int i = gt + k * ng, row = i >> 2, sl = i & 3;
    wdst[k] = row < 16 * CT ? row * EP + sl * 16 : -1;
    woff[k] = row < 16 * CT && co0 + row < a.Co ? (uint32_t)((co0 + row) * ci_b + sl * 16) : kOob;
  }
  const int wrows = a.vec_w2 ? ROWS_VEC : (ci_b % 4 == 0 ? ROWS_WORDS : ROWS_ELEMENTS);
  uint32_t xr[NX][CPG];
  u32x4 wr[NWV];
  auto load_chunk = [&](int c) {
    const uint32_t so = (uint32_t)(c * MC * hw * E);
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      if (k * ng >= 4 * lay.nqp) break;  // (uniform)
#pragma unroll
      for (int e = 0; e < CPG; ++e) {
        const int ch = I8 ? 16 * (e >> 2) + (e & 3) : e;  // (from the slot's first channel)
        xr[k][e] = load_elem8<DT>(rx, xoff[k], so + (uint32_t)(ch * hw * E));
      }
    }
    const int left = ci_b - c * 64 - 16 * (gt & 3);  // bytes of the row from this lane's slot on
#pragma unroll
    for (int k = 0; k < NWV; ++k) {
      if (k * ng >= 64 * CT) break;
      if (wrows != ROWS_ELEMENTS) {
        wr[k] = load_row8(rw, wrows == ROWS_VEC, woff[k], (uint32_t)(c * 64), left);
      } else if constexpr (E < 4) {
        uint32_t v[CPG];
#pragma unroll
        for (int e = 0; e < CPG; ++e)
          v[e] = load_elem8<DT>(rw, e * E < left ? woff[k] + e * E : kOob, (uint32_t)(c * 64));
        wr[k] = pack_slot8<DT>(v);
      }
    }
  };
  auto store_chunk = [&](char* eb) {
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      if (k * ng >= 4 * lay.nqp) break;
      if (xdst[k] >= 0) *(u32x4*)(eb + xdst[k]) = pack_slot8<DT>(xr[k]);
    }
#pragma unroll
    for (int k = 0; k < NWV; ++k) {
      if (k * ng >= 64 * CT) break;
      if (wdst[k] >= 0) *(u32x4*)(eb + lay.e_bytes + wdst[k]) = wr[k];
    }
  };
  if (j < nch) load_chunk(j);

  // ---- depthwise weights ([channel][tap] elements) and biases, zero beyond the channels ----
  {
    const int nel = nch * MC * KK, real = a.Ci * KK;
    const rsrc_t rd = make_rsrc(a.w1, (uint32_t)(real * E));
    const rsrc_t rb = make_rsrc(a.b1 ? a.b1 : a.w1, a.b1 ? (uint32_t)(a.Ci * 4) : 0u);
    for (int i = threadIdx.x; i < nel; i += 64 * nw) {
      const uint32_t v = load_elem8<DT>(rd, i < real ? (uint32_t)(i * E) : kOob, 0u);
      char* p = smem + lay.dww_off + i * E;
      if constexpr (E == 4) *(uint32_t*)p = v;
      else if constexpr (E == 2) *(uint16_t*)p = (uint16_t)v;
      else *(uint8_t*)p = (uint8_t)v;
    }
    for (int i = threadIdx.x; i < nch * MC; i += 64 * nw)
      *(uint32_t*)(smem + lay.b1_off + i * 4) = __builtin_amdgcn_raw_buffer_load_b32(rb, i < a.Ci ? i * 4 : kOob, 0, 0);
  }

  // ---- the wave's output pixels ----
  int ebase[PB], opix[PB];
#pragma unroll
  for (int b = 0; b < PB; ++b) {
    const int p = (b * GW + w) * 16 + r16, pc = min(p, P - 1);
    const int py = pc / TW, px = pc - py * TW;
    ebase[b] = (py * S * IW + px * S) * EP + (I8 ? 0 : 16 * g);
    opix[b] = p < P && oy0 + py < a.Ho && ox0 + px < a.Wo ? ((oy0 + py) * a.Wo + ox0 + px) : -1;
  }
  const DwLanes8<DT, K> dl(IW, g, r16);

  AccV acc2[PB][CT];
#pragma unroll
  for (int b = 0; b < PB; ++b)
#pragma unroll
    for (int u = 0; u < CT; ++u) acc2[b][u] = AccV{0, 0, 0, 0};
  const EpiF8 e1 = make_epif8(a.act[0]);
  const Rq8 q1 = make_rq8(a.rq[0], a.act[0]);

  char* ebuf = smem + 2 * j * lay.buf;
  if (j < nch) store_chunk(ebuf);
  wait_lgkm0();
  barrier3();

  const int niter = ceil_div(nch, J);
  for (int it = 0; it < niter; ++it) {
    const int c = j + J * it;
    const char* eb = ebuf + (it & 1) * lay.buf;
    if (c + J < nch) load_chunk(c + J);
    if (c < nch) {
      u32x4 d[PB];
      dl.template run<PB>(d, eb, ebase, smem + lay.dww_off + c * MC * KK * E, smem + lay.b1_off + c * MC * 4, e1, q1);
      const char* wp = eb + lay.e_bytes + r16 * EP + 16 * g;
#pragma unroll
      for (int u = 0; u < CT; ++u) {
        const u32x4 av = *(const u32x4*)(wp + u * 16 * EP);
#pragma unroll
        for (int b = 0; b < PB; ++b) mma16(DT{}, acc2[b][u], av, d[b]);
      }
    }
    if (c + J < nch) store_chunk(ebuf + ((it + 1) & 1) * lay.buf);
    wait_lgkm0();
    barrier3();
  }

  if (J > 1) {  // the groups' sums, in group order
    AccV* red = (AccV*)smem;
    if (j > 0) {
#pragma unroll
      for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int u = 0; u < CT; ++u) red[(((wave - GW) * PB + b) * CT + u) * 64 + lane] = acc2[b][u];
    }
    wait_lgkm0();
    barrier3();
    if (j > 0) return;
    for (int jj = 1; jj < J; ++jj)
#pragma unroll
      for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int u = 0; u < CT; ++u) acc2[b][u] += red[((((jj - 1) * GW + w) * PB + b) * CT + u) * 64 + lane];
  }
  const EpiF8 e2 = make_epif8(a.act[1]);
  const Rq8 q2 = make_rq8(a.rq[1], a.act[1]);
#pragma unroll
  for (int u = 0; u < CT; ++u) {
    const int co = co0 + 16 * u + 4 * g;
    if (co >= a.Co) continue;
    AccV bb;
#pragma unroll
    for (int q = 0; q < 4; ++q) bb[q] = load_bias<DT>(a.b2, min(co + q, a.Co - 1));
#pragma unroll
    for (int b = 0; b < PB; ++b) {
      const AccV v = acc2[b][u] + bb;
      u32x4 o = {0u, 0u, 0u, 0u};  // the four results, packed from word 0
      if constexpr (I8) {
        o[0] = rq8x4(v, q2);
      } else if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float f = v[q];
          o[q] = __float_as_uint(e2.none ? f : __builtin_amdgcn_fmed3f(f, e2.lo, e2.hi));
        }
      } else {
        o[0] = bf16x2_8(v[0], v[1], e2);
        o[1] = bf16x2_8(v[2], v[3], e2);
      }
      if (opix[b] < 0) continue;
      store_planes8<DT, 4>((char*)a.y + (((size_t)n * a.Co + co) * a.Ho * a.Wo + opix[b]) * E,
                           (size_t)a.Ho * a.Wo * E, o, a.Co - co);
    }
  }
}

template <class DT, int K, int CT, int PB>
int launch_dwpw9(const KArgs& a, int grid, void* stream) {
  const void* fn = (const void*)k_dwpw9<DT, K, CT, PB>;
  const int lds = a.L.bytes;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
  }
  return launch_args(fn, grid, 64 * a.gw * a.splits, lds, stream, a);
}

}  // namespace fcm
