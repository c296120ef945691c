// fcm_kernels_v8.h -- PW->DW and PW->DW->PW modules (gfx950), NHWC and NCHW.
//
// k_ir8<DT, K, KS, CT, PB, NCHW>
//   A workgroup computes one TH x TW output tile (run time) of one image. The intermediate
//   channels go through it in chunks of MC = 64 bytes (one MFMA k-step of the last
//   convolution): the first PW expands a chunk on the tile's haloed window into an LDS
//   buffer E, the depthwise stage filters it, and the result is either stored (PW -> DW,
//   CT = 0) or contracted into output accumulators that stay in registers
//   (output-stationary, Sec. III-A OS-LWS). GW waves (1, 2 or 4) form a group; J groups of
//   one workgroup take chunks j, j + J, ... and add their accumulators through LDS at the
//   end, which keeps the chain of chunks short where a launch has few tiles.
//
//   Per chunk and wave:
//   * PW1: the wave's 16-position tiles of the window (w, w + GW, ...). The window sits in
//     LDS ([position][channel slots], staged once), the chunk's weight rows in A-operand
//     registers, loaded a chunk ahead. The lane (position l % 16, group l / 16) collects
//     its accumulators (bias as the MFMA's C operand), activation and cast into the 16-byte
//     slot l / 16 of E's position: bf16 rows are taken in the order that makes the slot 8
//     consecutive channels; int8 takes natural rows, byte 4t + v of slot s being channel
//     16t + 4s + v. Positions outside the image are written as real 0 (the DW's padding,
//     Sec. III-A PWDW_R).
//   * one barrier (E is double buffered)
//   * DW: lane = output pixel l % 16 of the wave's own 16-pixel blocks, slot l / 16.
//     bf16: dot instructions on pairs of taps, weights broadcast within 16-lane rows by
//     DPP, each row holding its own slot's weights. int8: on the matrix
//     cores. For slot s the A operand is diagonal, row m holding the weight of tap
//     4 kk + l / 16 at byte m of the slot, zero elsewhere; the B operand is E's slot s at
//     that tap's position. Row m of slot s is channel 16 (m / 4) + 4s + m % 4, so after the
//     four slots the lane holds channels 16 (l / 16) .. + 15 of its pixel: 16 contiguous
//     bytes to store, or the B operand of PW2. (Integer zeros cannot pick up a NaN or
//     infinity of a neighbouring channel, so only int8 can use the diagonal form.)
//   * PW2: the DW result is the MFMA's B operand without leaving the registers.
//
//   NCHW gathers the window transposed, one element load per channel and position (lanes
//   along the pixels of a plane), and stores each channel's pixels to its plane; all between
//   is the same. fp32: 16-channel chunks, four 16x16x4 MFMAs a k-step, FMA stencils.
//
//   E and the window have a pitch of 16 bytes more than a multiple of 64, an odd number of
//   16-byte units: 16 lanes at consecutive positions reach every LDS bank once.
//
//   What bounds it: the vector ALU (the epilogues of PW1 on the haloed window and of DW),
//   then launch and the chain of chunks for small batches; LDS and the matrix cores are
//   below half busy.
#pragma once

#include "fcm_kernels_v7.h"
#include "fcm_kernels_v4.h"

namespace fcm {

constexpr int kMaxWaves8 = 8;

// Two float results as packed bf16. Without an activation the value passes as it is (a
// median with infinite ends would turn a NaN into one of them).
struct EpiF8 {
  bool none;
  float lo, hi;
};
__device__ __forceinline__ EpiF8 make_epif8(int act) {
  return EpiF8{act == ACT_NONE, 0.0f, act == ACT_RELU6 ? 6.0f : __builtin_huge_valf()};
}
__device__ __forceinline__ uint32_t bf16x2_8(float v0, float v1, const EpiF8& e) {
  if (e.none) return pack_bf16x2(v0, v1);  // (uniform)
  return pack_bf16x2(__builtin_amdgcn_fmed3f(v0, e.lo, e.hi), __builtin_amdgcn_fmed3f(v1, e.lo, e.hi));
}

// 16 bytes at voff (+ soff) of a row-major matrix whose rows are multiples of 16 bytes
// (vec) or of 4 bytes; nb: bytes of the row left from voff on (the rest reads as zero).
__device__ __forceinline__ u32x4 load_row8(rsrc_t r, bool vec, uint32_t voff, uint32_t soff, int nb) {
  if (vec) return __builtin_amdgcn_raw_buffer_load_b128(r, nb > 0 ? voff : kOob, soff, 0);
  u32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    v[e] = __builtin_amdgcn_raw_buffer_load_b32(r, 4 * e < nb ? voff + 4 * e : kOob, soff, 0);
  return v;
}

// One element of a buffer as a 32-bit value (bf16 bits, int8 byte, fp32 bits).
template <class DT>
__device__ __forceinline__ uint32_t load_elem8(rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (DT::ELT == 4) return __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
  else if constexpr (DT::ELT == 2) return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
  else return (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, voff, soff, 0);
}
// The 16 / ELT elements of a slot packed into 16 bytes.
template <class DT>
__device__ __forceinline__ u32x4 pack_slot8(const uint32_t (&v)[16 / DT::ELT]) {
  u32x4 o;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    if constexpr (DT::ELT == 4) o[d] = v[d];
    else if constexpr (DT::ELT == 2) o[d] = v[2 * d] | (v[2 * d + 1] << 16);
    else o[d] = v[4 * d] | (v[4 * d + 1] << 8) | (v[4 * d + 2] << 16) | (v[4 * d + 3] << 24);
  }
  return o;
}

// The first `valid` of N packed elements, one to each of consecutive planes.
template <class DT, int N>
__device__ __forceinline__ void store_planes8(char* y, size_t plane, const u32x4& o, int valid) {
#pragma unroll
  for (int q = 0; q < N; ++q) {
    if (q >= valid) break;
    if constexpr (DT::ELT == 4) *(uint32_t*)(y + q * plane) = o[q];
    else if constexpr (DT::ELT == 2) *(uint16_t*)(y + q * plane) = (uint16_t)(o[q >> 1] >> (16 * (q & 1)));
    else *(uint8_t*)(y + q * plane) = (uint8_t)(o[q >> 2] >> (8 * (q & 3)));
  }
}

// The depthwise stage of one wave: lane = output pixel l % 16 of each of PB blocks, slot
// l / 16 of a 64-byte chunk held [position][slots] in LDS. d[b] = the 16 bytes of the lane's
// slot (int8: of channels 16 (l / 16) .. + 15; see above), +bias, activation and cast.
// wts: the chunk's weights [channel][tap], bias: its biases, both in LDS.
template <class DT, int K>
struct DwLanes8 {
  static constexpr int KK = K * K, NKK = (KK + 3) / 4, EP = kPitchE8;
  int IW, g, r16;
  int tko[NKK];       // int8: offset of the lane group's tap of each k-step
  uint32_t dmask[4];  // int8: the diagonal byte of each operand word

  __device__ __forceinline__ DwLanes8(int IW_, int g_, int r16_) : IW(IW_), g(g_), r16(r16_) {
    if constexpr (DT::ELT == 1) {
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        const int tap = min(4 * kk + g, KK - 1);
        tko[kk] = ((tap / K) * IW + tap % K) * EP;
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) dmask[d] = (r16 >> 2) == d ? 0xffu << (8 * (r16 & 3)) : 0u;
    }
  }

  template <int PB>
  __device__ __forceinline__ void run(u32x4 (&d)[PB], const char* eb, const int (&ebase)[PB], const char* wts,
                                      const char* bias, const EpiF8& ef, const Rq8& eq) const {
    using AccV = typename DT::AccV;
    if constexpr (DT::ELT == 1) {
      const char* wb = wts + (16 * (r16 >> 2) + (r16 & 3)) * KK;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        AccV acc[PB];
        const AccV bv = *(const AccV*)(bias + (16 * g + 4 * s) * 4);
#pragma unroll
        for (int b = 0; b < PB; ++b) acc[b] = bv;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
          const int tap = 4 * kk + g;
          uint32_t wt = *(const uint8_t*)(wb + 4 * s * KK + min(tap, KK - 1));
          if (4 * kk + 3 >= KK) wt = tap < KK ? wt : 0u;
          wt = __builtin_amdgcn_perm(wt, wt, 0u);  // the byte in all four places
          const u32x4 av = {wt & dmask[0], wt & dmask[1], wt & dmask[2], wt & dmask[3]};
#pragma unroll
          for (int b = 0; b < PB; ++b) mma16(DT{}, acc[b], av, *(const u32x4*)(eb + ebase[b] + tko[kk] + 16 * s));
        }
#pragma unroll
        for (int b = 0; b < PB; ++b) d[b][s] = rq8x4(acc[b], eq);
      }
    } else {
      // the slot's CPG * KK weights as words, 64 of them (four a lane) to a register set
      constexpr int CPG = 16 / DT::ELT, NWORD = CPG * KK * DT::ELT / 4, NS = (NWORD + 63) / 64;
      u32x4 wv[NS];
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const int off = 256 * k + 16 * r16;
        wv[k] = *(const u32x4*)(wts + g * (NWORD * 4) + (off < NWORD * 4 ? off : 0));
      }
      float bv[CPG];
#pragma unroll
      for (int q = 0; q < CPG / 4; ++q) {
        const f32x4 b4 = *(const f32x4*)(bias + (CPG * g + 4 * q) * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) bv[4 * q + e] = b4[e];
      }
#pragma unroll
      for (int b = 0; b < PB; ++b) {
        u32x4 xv[KK];
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
          for (int kx = 0; kx < K; ++kx) xv[K * ky + kx] = *(const u32x4*)(eb + ebase[b] + (ky * IW + kx) * EP);
        float acc[CPG];
#pragma unroll
        for (int e = 0; e < CPG; ++e) acc[e] = bv[e];
        static_for7<0, CPG>([&](auto jc) {
          constexpr int J = decltype(jc)::value;
          channel<J>(acc[J], xv, wv);
        });
        if constexpr (DT::ELT == 2) {
#pragma unroll
          for (int q = 0; q < 4; ++q) d[b][q] = bf16x2_8(acc[2 * q], acc[2 * q + 1], ef);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            d[b][q] = __float_as_uint(ef.none ? acc[q] : __builtin_amdgcn_fmed3f(acc[q], ef.lo, ef.hi));
        }
      }
    }
  }

  // Channel J of the slot: word q of the weights sits in set q / 64, lane (q % 64) / 4,
  // component q % 4. bf16 (KK odd): an even channel's taps pair up from its first, an odd
  // one's first tap is the high half of a word it shares (as dw_channel7).
  template <int J, int NS>
  __device__ static __forceinline__ void channel(float& acc, const u32x4 (&xv)[KK], const u32x4 (&wv)[NS]) {
    if constexpr (DT::ELT == 4) {
      static_for7<0, KK>([&](auto tc) {
        constexpr int T = decltype(tc)::value, q = J * KK + T;
        acc = __builtin_fmaf(bcast7<(q % 64) / 4>(wv[q / 64][q % 4]), __uint_as_float(xv[T][J]), acc);
      });
    } else {
      constexpr int k = J >> 1, odd = J & 1, q0 = (KK * J - odd) / 2, NP = (KK + 1) / 2;
      static_for7<0, NP>([&](auto pc) {
        constexpr int i = decltype(pc)::value, q = q0 + i;
        uint32_t x;
        if constexpr (odd) {
          if constexpr (i == 0) x = xv[0][k] & 0xffff0000u;
          else x = __builtin_amdgcn_perm(xv[2 * i][k], xv[2 * i - 1][k], 0x07060302u);
        } else {
          if constexpr (i == NP - 1) x = xv[KK - 1][k] & 0xffffu;
          else x = __builtin_amdgcn_perm(xv[2 * i + 1][k], xv[2 * i][k], 0x05040100u);
        }
        dot_bcast7<(q % 64) / 4, i == NP - 1>(acc, wv[q / 64][q % 4], x);
      });
    }
  }
};

template <class DT, int K, int KS, int CT, int PB, bool NCHW>
__global__ __launch_bounds__(64 * kMaxWaves8) void k_ir8(KArgs a) {
  extern __shared__ __align__(16) char smem[];
  constexpr bool I8 = std::is_same<DT, TI8>::value, F32 = std::is_same<DT, TF32>::value;
  using AccV = typename DT::AccV;
  constexpr int E = DT::ELT, MC = 64 / E, TPC = 4 / E, CPG = 16 / E;
  constexpr int KK = K * K;
  constexpr int EP = kPitchE8;
  constexpr int NU = CT > 0 ? CT : 1;

  const int S = a.stride, TW = a.TW, P = a.TH * TW;
  const int IH = (a.TH - 1) * S + K, IW = (TW - 1) * S + K, Q = IH * IW;
  const int J = a.splits, GW = a.gw;
  const int MB = CT > 0 ? a.Cm : a.COB;  // intermediate channels of this workgroup
  const Lds8 lay = lds8(dtype_id<DT>(), K, S, a.TH, TW, a.Ci, MB, GW, J, PB, CT);
  const int ci_b = a.Ci * E, cm_b = a.Cm * E;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, g = lane >> 4;
  const int nw = GW * J;
  const int j = wave / GW, w = wave % GW;

  // ---- this workgroup's tile ----
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int cb = CT > 0 ? 0 : lid % a.n_cb;
  int t = CT > 0 ? lid : lid / a.n_cb;
  const int tx = t % a.tiles_x;
  t /= a.tiles_x;
  const int ty = t % a.tiles_y, n = t / a.tiles_y;
  const int oy0 = ty * a.TH, ox0 = tx * TW;
  const int iy0 = oy0 * S - a.pad, ix0 = ox0 * S - a.pad;
  const int cm0 = cb * MB;                       // first intermediate channel
  const int mb = min(MB, a.Cm - cm0);            // of this workgroup
  const int nch = ceil_div(mb, MC);

  // ---- depthwise weights and both biases of the workgroup's channels: flat copies ----
  {
    const rsrc_t rd = make_rsrc((const char*)a.w2 + (size_t)cm0 * KK * E, (uint32_t)(mb * KK * E));
    const rsrc_t r1 = make_rsrc(a.b1 ? (const char*)a.b1 + (size_t)cm0 * 4 : (const char*)a.w1, a.b1 ? mb * 4u : 0u);
    const rsrc_t r2 = make_rsrc(a.b2 ? (const char*)a.b2 + (size_t)cm0 * 4 : (const char*)a.w1, a.b2 ? mb * 4u : 0u);
    const int nd = (lay.b1_off - lay.dww_off) >> 10, nb = (lay.b2_off - lay.b1_off) >> 10;
    for (int i = wave; i < nd + 2 * nb; i += nw) {
      if (i < nd)
        dma16(rd, smem + lay.dww_off + i * 1024, (uint32_t)(i * 1024 + lane * 16));
      else if (i < nd + nb)
        dma16(r1, smem + lay.b1_off + (i - nd) * 1024, (uint32_t)((i - nd) * 1024 + lane * 16));
      else
        dma16(r2, smem + lay.b2_off + (i - nd - nb) * 1024, (uint32_t)((i - nd - nb) * 1024 + lane * 16));
    }
  }
  // ---- first chunk's PW1 weights (A operands), a chunk ahead of their use ----
  const rsrc_t rw1 = make_rsrc(a.w1, (uint32_t)(a.Cm * ci_b));
  uint32_t aoff[KS];
  int anb[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int row = I8 ? r16 : CPG * (r16 >> 2) + (r16 & 3);
    aoff[s] = (uint32_t)(row * ci_b + 64 * s + 16 * g);
    anb[s] = ci_b - (64 * s + 16 * g);
  }
  u32x4 a1[TPC][KS];
  auto load_a1 = [&](int c) {
#pragma unroll
    for (int tt = 0; tt < TPC; ++tt) {
      const uint32_t so = (uint32_t)((cm0 + c * MC + (I8 ? 16 : 4) * tt) * ci_b);
#pragma unroll
      for (int s = 0; s < KS; ++s) a1[tt][s] = load_row8(rw1, a.vec_w1, aoff[s], so, anb[s]);
    }
  };
  if (j < nch) load_a1(j);

  // ---- the haloed window: [position][16-byte slots], zero outside the image and beyond
  // the input channels ----
  {
    const size_t img = (size_t)a.H * a.W * ci_b;
    const rsrc_t rx = make_rsrc((const char*)a.x + (size_t)n * img, (uint32_t)img);
    const int nsl = 4 * ceil_div(ci_b, 64), items = lay.nqp * nsl, step = 64 * nw;
    constexpr int B = 4;
    for (int i0 = threadIdx.x; i0 < items; i0 += step * B) {
      u32x4 v[B];
      int dst[B];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int i = i0 + b * step;
        const int pos = NCHW ? i % lay.nqp : i / nsl, sl = NCHW ? i / lay.nqp : i - pos * nsl;
        const int qy = pos / IW, qx = pos - qy * IW;
        const int gy = iy0 + qy, gx = ix0 + qx;
        const bool ok = pos < Q && (unsigned)gy < (unsigned)a.H && (unsigned)gx < (unsigned)a.W;
        dst[b] = i < items ? pos * lay.xp + sl * 16 : -1;
        if constexpr (NCHW) {  // (channels beyond the last lie beyond the image's buffer)
          uint32_t el[CPG];
          const uint32_t off = ok ? (uint32_t)(((sl * CPG * a.H + gy) * a.W + gx) * E) : kOob;
#pragma unroll
          for (int e = 0; e < CPG; ++e) el[e] = load_elem8<DT>(rx, off, (uint32_t)(e * a.H * a.W * E));
          v[b] = pack_slot8<DT>(el);
        } else {
          v[b] = load_row8(rx, a.vec_x, (uint32_t)((gy * a.W + gx) * ci_b + sl * 16), 0u, ok ? ci_b - sl * 16 : 0);
        }
      }
#pragma unroll
      for (int b = 0; b < B; ++b)
        if (dst[b] >= 0) *(u32x4*)(smem + dst[b]) = v[b];
    }
  }

  // ---- the wave's window tiles and output pixels ----
  const int nqt = lay.nqp >> 4;
  uint32_t inside = 0;  // bit i: this lane's position of the wave's i-th tile lies in the image
  for (int i = 0, qt = w; qt < nqt; ++i, qt += GW) {
    const int pos = qt * 16 + r16;
    const int qy = pos / IW, qx = pos - qy * IW;
    const bool ok = pos < Q && (unsigned)(iy0 + qy) < (unsigned)a.H && (unsigned)(ix0 + qx) < (unsigned)a.W;
    inside |= (ok ? 1u : 0u) << i;
  }
  int ebase[PB], opix[PB];  // E position of the pixel's first tap; output pixel or -1
#pragma unroll
  for (int b = 0; b < PB; ++b) {
    const int p = (b * GW + w) * 16 + r16, pc = min(p, P - 1);
    const int py = pc / TW, px = pc - py * TW;
    ebase[b] = (py * S * IW + px * S) * EP + (I8 ? 0 : 16 * g);
    opix[b] = p < P && oy0 + py < a.Ho && ox0 + px < a.Wo ? ((oy0 + py) * a.Wo + ox0 + px) : -1;
  }
  const DwLanes8<DT, K> dl(IW, g, r16);

  AccV acc2[PB][NU];
#pragma unroll
  for (int b = 0; b < PB; ++b)
#pragma unroll
    for (int u = 0; u < NU; ++u) acc2[b][u] = AccV{0, 0, 0, 0};

  const EpiF8 e1 = make_epif8(a.act[0]), e2 = make_epif8(a.act[1]);
  const Rq8 q1 = make_rq8(a.rq[0], a.act[0]);
  const Rq8 q2 = make_rq8(a.rq[1], a.act[1]);
  const rsrc_t rw3 = make_rsrc(CT > 0 ? a.w3 : a.w1, CT > 0 ? (uint32_t)(a.Co * cm_b) : 0u);
  const uint32_t a2off = (uint32_t)(r16 * cm_b + 16 * g);
  const int nks = ceil_div(ci_b, 64);  // k-steps of PW1 (staged ones)

  wait_vm_n<0>();
  wait_lgkm0();
  barrier3();

  const int niter = ceil_div(nch, J);
  for (int it = 0; it < niter; ++it) {
    const int c = j + J * it;
    const bool active = c < nch;
    char* eb = smem + lay.e_off + (2 * j + (it & 1)) * lay.e_buf;
    const int m0 = c * MC;  // within the workgroup's channels
    u32x4 a2[NU];
    if (active) {
      if constexpr (CT > 0) {
        const uint32_t vo = m0 * E + 16 * g < cm_b ? a2off : kOob;
#pragma unroll
        for (int u = 0; u < CT; ++u)
          a2[u] = __builtin_amdgcn_raw_buffer_load_b128(rw3, vo, (uint32_t)(u * 16 * cm_b + m0 * E), 0);
      }
      // ---- PW1 on the wave's window tiles ----
      AccV b1[TPC];
#pragma unroll
      for (int tt = 0; tt < TPC; ++tt) {
        const int ch = I8 ? m0 + 16 * tt + 4 * g : m0 + CPG * g + 4 * tt;
        b1[tt] = *(const AccV*)(smem + lay.b1_off + ch * 4);
      }
      const char* xp = smem + (w * 16 + r16) * lay.xp + 16 * g;
      char* ep = eb + (w * 16 + r16) * EP + 16 * g;
#pragma unroll 2
      for (int i = 0, qt = w; qt < nqt; ++i, qt += GW) {
        AccV acc[TPC];
#pragma unroll
        for (int tt = 0; tt < TPC; ++tt) acc[tt] = b1[tt];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if (s > 0 && s >= nks) break;  // (uniform; nothing is staged there)
          const u32x4 xb = *(const u32x4*)(xp + 64 * s);
#pragma unroll
          for (int tt = 0; tt < TPC; ++tt) mma16(DT{}, acc[tt], a1[tt][s], xb);
        }
        u32x4 o;
        if constexpr (I8) {
#pragma unroll
          for (int tt = 0; tt < TPC; ++tt) o[tt] = rq8x4(acc[tt], q1);
        } else if constexpr (F32) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float f = acc[0][q];
            o[q] = __float_as_uint(e1.none ? f : __builtin_amdgcn_fmed3f(f, e1.lo, e1.hi));
          }
        } else {
#pragma unroll
          for (int tt = 0; tt < TPC; ++tt)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              o[2 * tt + h] = bf16x2_8(acc[tt][2 * h], acc[tt][2 * h + 1], e1);
        }
        const bool in = (inside >> i) & 1u;
#pragma unroll
        for (int d = 0; d < 4; ++d) o[d] = in ? o[d] : 0u;
        *(u32x4*)ep = o;
        xp += GW * 16 * lay.xp;
        ep += GW * 16 * EP;
      }
    }
    wait_lgkm0();
    barrier3();
    if (active) {
      if (c + J < nch) load_a1(c + J);
      // ---- DW on the wave's pixel blocks, PW2 or the store ----
      u32x4 d[PB];
      dl.template run<PB>(d, eb, ebase, smem + lay.dww_off + m0 * KK * E, smem + lay.b2_off + m0 * 4, e2, q2);
      if constexpr (CT > 0) {
#pragma unroll
        for (int u = 0; u < CT; ++u) {
#pragma unroll
          for (int b = 0; b < PB; ++b) mma16(DT{}, acc2[b][u], a2[u], d[b]);
        }
      } else {
        const int ch = m0 + CPG * g;
#pragma unroll
        for (int b = 0; b < PB; ++b)
          if (opix[b] >= 0 && ch < mb) {
            if constexpr (NCHW)
              store_planes8<DT, CPG>((char*)a.y + (((size_t)n * a.Cm + cm0 + ch) * a.Ho * a.Wo + opix[b]) * E,
                                     (size_t)a.Ho * a.Wo * E, d[b], mb - ch);
            else
              *(u32x4*)((char*)a.y + (((size_t)n * a.Ho * a.Wo + opix[b]) * a.Cm + cm0 + ch) * E) = d[b];
          }
      }
    }
  }

  if constexpr (CT > 0) {
    if (J > 1) {  // the groups' sums, in group order
      wait_lgkm0();
      barrier3();
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
          for (int u = 0; u < CT; ++u)
            acc2[b][u] += red[((((jj - 1) * GW + w) * PB + b) * CT + u) * 64 + lane];
    }
    const EpiF8 e3 = make_epif8(a.act[2]);
    const Rq8 q3 = make_rq8(a.rq[2], a.act[2]);
#pragma unroll
    for (int u = 0; u < CT; ++u) {
      const int co = 16 * u + 4 * g;
      if (co >= a.Co) continue;
      AccV bb;
#pragma unroll
      for (int q = 0; q < 4; ++q) bb[q] = load_bias<DT>(a.b3, min(co + q, a.Co - 1));
#pragma unroll
      for (int b = 0; b < PB; ++b) {
        const AccV v = acc2[b][u] + bb;
        u32x4 o = {0u, 0u, 0u, 0u};  // the four results, packed from word 0
        if constexpr (I8) {
          o[0] = rq8x4(v, q3);
        } else if constexpr (F32) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float f = v[q];
            o[q] = __float_as_uint(e3.none ? f : __builtin_amdgcn_fmed3f(f, e3.lo, e3.hi));
          }
        } else {
          o[0] = bf16x2_8(v[0], v[1], e3);
          o[1] = bf16x2_8(v[2], v[3], e3);
        }
        if (opix[b] < 0) continue;
        if constexpr (NCHW) {
          store_planes8<DT, 4>((char*)a.y + (((size_t)n * a.Co + co) * a.Ho * a.Wo + opix[b]) * E,
                               (size_t)a.Ho * a.Wo * E, o, a.Co - co);
        } else {
          char* y = (char*)a.y + (((size_t)n * a.Ho * a.Wo + opix[b]) * a.Co + co) * E;
          if constexpr (I8) *(uint32_t*)y = o[0];
          else if constexpr (F32) *(u32x4*)y = o;
          else *(u32x2*)y = u32x2{o[0], o[1]};
        }
      }
    }
  }
}

template <class DT, int K, int KS, int CT, int PB, bool NCHW>
int launch_ir8(const KArgs& a, int grid, void* stream) {
  const void* fn = (const void*)k_ir8<DT, K, KS, CT, PB, NCHW>;
  const int lds = a.L.bytes;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return (int)e;
  }
  return launch_args(fn, grid, 64 * a.gw * a.splits, lds, stream, a);
}

}  // namespace fcm
