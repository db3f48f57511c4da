// zq_kernels.hip -- gfx950 kernels of the qwZ / qgZ compression path.
//
// Block-wise symmetric quantisation as ZeRO++ applies it to the weight
// Allgather (INT8) and the gradient all-to-all reduce-scatter (INT4), per the
// paper's Background (ZeRO++ subsection) and Design (Weight / Gradient
// Partitioning).  The exact definition every kernel reproduces bit for bit is
// written out in include/zq.h.
//
// All kernels are streaming, HBM-bound work (no contraction, so no MFMA):
//   * one tile of 64 lanes x E elements per wave, launches covering the whole
//     tensor, nontemporal loads and stores (data is touched once);
//   * per-block absmax reduced across the lanes of a block with DPP row
//     permutes (quad_perm, row_half_mirror, row_mirror) -- no LDS round trip;
//   * rounding to nearest-even by adding 1.5*2^23, which leaves the code as
//     two's complement in the low mantissa bits, then byte/nibble packing
//     with v_perm_b32;
//   * the reduce level, the one kernel with real arithmetic per byte (P
//     multiplies and adds per output element), converts a nibble with one
//     v_cvt_off_f32_i4 (q/16 exactly) and multiplies by 16*s, which is exact,
//     so every product is still fl(q*s).
//
// Floating point: built with -ffp-contract=off (and the pragma below) so a*b+c
// is never fused; fp32 division is the correctly rounded sequence; fp32 and
// fp16 denormals are preserved (default HIP mode).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "zq.h"
#include "zq_device.h"
#include "zq_internal.h"

#pragma clang fp contract(off)

// Nontemporal hints per kernel family: bit 0 = loads, bit 1 = stores.  Data
// streamed once gains from them; a kernel whose input was just written by the
// previous call (the dequantiser after a reduce level) loses its cache hits.
// The quantisers: INT8 output measured faster with plain stores (the
// degree-2 half shard 100.3 against 104.9 us), INT4 output with nontemporal
// ones (the fp32 gradient 310.0 against 312.0 us).
// Wave priority while a wave issues its loads (s_setprio, within the
// kernel): raised so that the loads of a newly started wave go out ahead of
// other waves' arithmetic, then back to normal for the wave's own arithmetic.
#ifndef ZQ_PRIO_QUANT
#define ZQ_PRIO_QUANT 1
#endif
#ifndef ZQ_PRIO_DEQ
#define ZQ_PRIO_DEQ 0
#endif
template <int ON>
__device__ __forceinline__ void prio_issue() {
  if constexpr (ON) __builtin_amdgcn_s_setprio(3);
}
template <int ON>
__device__ __forceinline__ void prio_compute() {
  if constexpr (ON) __builtin_amdgcn_s_setprio(0);
}
#ifndef ZQ_NT_QUANT8
#define ZQ_NT_QUANT8 1
#endif
#ifndef ZQ_NT_QUANT4
#define ZQ_NT_QUANT4 3
#endif
#ifndef ZQ_NT_DEQ8
#define ZQ_NT_DEQ8 3
#endif
#ifndef ZQ_NT_DEQ4
#define ZQ_NT_DEQ4 0
#endif
#ifndef ZQ_NT_REDUCE
#define ZQ_NT_REDUCE 3
#endif
// Dequantisers with more than 16 output bytes per thread stage them in LDS.
#ifndef ZQ_DEQ_STAGE
#define ZQ_DEQ_STAGE 1
#endif
// Scale arrays are written 4 bytes per block, i.e. in partial cache lines:
// plain stores let L2 merge them into full lines before write-back.
#ifndef ZQ_NT_SCALES
#define ZQ_NT_SCALES 0
#endif
namespace zq {
namespace {


constexpr float kRoundMagic = 12582912.0f;  // 1.5 * 2^23
constexpr float kFlushBelow = 0x1p-119f;    // absmax below this: zero block
constexpr float kMaxFloat = 3.40282346638528859812e+38f;

template <int NT, typename T>
__device__ __forceinline__ T ld(const T* p) {
  if constexpr (NT & 1) return __builtin_nontemporal_load(p);
  else return *p;
}
template <int NT, typename T>
__device__ __forceinline__ void st(T* p, T v) {
  if constexpr (NT & 2) __builtin_nontemporal_store(v, p);
  else *p = v;
}


// fl(fl(v * r) + 1.5*2^23): for |fl(v*r)| < 2^22 the sum lies in [2^23, 2^24)
// where binary32 spacing is 1, so it is 1.5*2^23 + rint_even(fl(v*r)); the
// integer sits in the low mantissa bits as two's complement.
__device__ __forceinline__ uint32_t code_bits(float v, float r) {
  float t = v * r;
  return f2u(t + kRoundMagic);
}

// Block scale fl(a / qmax) for a normal a >= 2^-119, via one binary64
// multiply: a/qmax is either a binary32 value or lies at least
// ulp(a/qmax) / (2 qmax) >= (a/qmax) * 2^-32 away from every binary32 rounding
// boundary (qmax is odd, so a/qmax is not dyadic unless qmax divides a's
// significand), while a * fl64(1/qmax) is within 2^-52 relative of a/qmax.
// Rounding that to binary32 (nearest even) therefore gives fl(a / qmax),
// the correctly rounded quotient, in 3 instructions instead of a division.
template <int QMAX>
__device__ __forceinline__ float scale_of(float amax) {
  return (float)((double)amax * (1.0 / (double)QMAX));
}

// INT4 code (two's complement nibble k of w) as float.
__device__ __forceinline__ float nib_to_f32(uint32_t w, int k) {
  return (float)((int32_t)(w << (28 - 4 * k)) >> 28);
}

// q/16 for the two's-complement low nibble of byte BYTE of w, in one
// instruction (v_cvt_off_f32_i4 with an SDWA byte select).
template <int BYTE>
__device__ __forceinline__ float nib_over_16(uint32_t w) {
  float f;
  if constexpr (BYTE == 0)
    asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_0" : "=v"(f) : "v"(w));
  else if constexpr (BYTE == 1)
    asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1" : "=v"(f) : "v"(w));
  else if constexpr (BYTE == 2)
    asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2" : "=v"(f) : "v"(w));
  else
    asm("v_cvt_off_f32_i4_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3" : "=v"(f) : "v"(w));
  return f;
}

// The 8 nibbles of w, each as q/16 (element order: low nibble of byte 0 first).
__device__ __forceinline__ void nibbles_over_16(uint32_t w, float* o) {
  const uint32_t h = w >> 4;
  o[0] = nib_over_16<0>(w); o[1] = nib_over_16<0>(h);
  o[2] = nib_over_16<1>(w); o[3] = nib_over_16<1>(h);
  o[4] = nib_over_16<2>(w); o[5] = nib_over_16<2>(h);
  o[6] = nib_over_16<3>(w); o[7] = nib_over_16<3>(h);
}

// Max over the L lanes of an aligned lane group (L a power of two <= 64).
// Non-negative binary32 values order like their bit patterns.
template <int L>
__device__ __forceinline__ uint32_t group_max(uint32_t v) {
  static_assert(L >= 1 && L <= 64 && (L & (L - 1)) == 0, "lane group");
  if constexpr (L >= 2) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
  if constexpr (L >= 4) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
  if constexpr (L >= 8) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));  // row_half_mirror
  if constexpr (L >= 16) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false)); // row_mirror
  if constexpr (L >= 32) v = max(v, (uint32_t)__shfl_xor((int)v, 16, 64));
  if constexpr (L >= 64) v = max(v, (uint32_t)__shfl_xor((int)v, 32, 64));
  return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return group_max<64>(v); }

// byte 0 of m0..m3 -> bytes 0..3
__device__ __forceinline__ uint32_t pack_bytes4(uint32_t m0, uint32_t m1, uint32_t m2, uint32_t m3) {
  uint32_t lo = __builtin_amdgcn_perm(m1, m0, 0x0c0c0400u);
  uint32_t hi = __builtin_amdgcn_perm(m3, m2, 0x0c0c0400u);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// low nibble of m[0..7] -> nibbles 0..7 (element 2j low, 2j+1 high of byte j)
__device__ __forceinline__ uint32_t pack_nibbles8(const uint32_t* m) {
  uint32_t ev = pack_bytes4(m[0], m[2], m[4], m[6]);
  uint32_t od = pack_bytes4(m[1], m[3], m[5], m[7]);
  return (ev & 0x0f0f0f0fu) | ((od << 4) & 0xf0f0f0f0u);
}

// ------------------------------------------------------------------ raw I/O

template <int NT, int NW>
__device__ __forceinline__ void load_words(const void* p, uint32_t (&w)[NW]) {
  if constexpr (NW % 4 == 0) {
#pragma unroll
    for (int k = 0; k < NW / 4; ++k) {
      const u32x4 t = ld<NT>(static_cast<const u32x4*>(p) + k);
      w[4 * k] = t.x; w[4 * k + 1] = t.y; w[4 * k + 2] = t.z; w[4 * k + 3] = t.w;
    }
  } else if constexpr (NW == 2) {
    const u32x2 t = ld<NT>(static_cast<const u32x2*>(p));
    w[0] = t.x; w[1] = t.y;
  } else {
    static_assert(NW == 1, "words");
    w[0] = ld<NT>(static_cast<const uint32_t*>(p));
  }
}

template <int NT, int NW>
__device__ __forceinline__ void store_words(void* p, const uint32_t (&w)[NW]) {
  if constexpr (NW % 4 == 0) {
#pragma unroll
    for (int k = 0; k < NW / 4; ++k)
      st<NT>(static_cast<u32x4*>(p) + k, u32x4{w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]});
  } else if constexpr (NW == 2) {
    st<NT>(static_cast<u32x2*>(p), u32x2{w[0], w[1]});
  } else {
    static_assert(NW == 1, "words");
    st<NT>(static_cast<uint32_t*>(p), w[0]);
  }
}

// ------------------------------------------------------------------ element formats

template <int DT>
constexpr int elem_size() { return DT == ZQ_F32 ? 4 : 2; }

// E consecutive elements from element index i, widened to binary32 (exact).
template <int NT, int DT, int E>
__device__ __forceinline__ void load_elems(const void* p, int64_t i, float (&v)[E]) {
  constexpr int NW = E * elem_size<DT>() / 4;
  uint32_t w[NW];
  load_words<NT, NW>(static_cast<const char*>(p) + i * elem_size<DT>(), w);
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    if constexpr (DT == ZQ_F32) {
      v[k] = u2f(w[k]);
    } else if constexpr (DT == ZQ_BF16) {
      v[2 * k] = u2f(w[k] << 16);
      v[2 * k + 1] = u2f(w[k] & 0xffff0000u);
    } else {
      v[2 * k] = h2f(w[k] & 0xffffu);
      v[2 * k + 1] = h2f(w[k] >> 16);
    }
  }
}

// E binary32 values narrowed (nearest even) and stored from element index i.
template <int NT, int DT, int E>
__device__ __forceinline__ void store_elems(void* p, int64_t i, const float (&v)[E]) {
  constexpr int NW = E * elem_size<DT>() / 4;
  uint32_t w[NW];
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    if constexpr (DT == ZQ_F32) w[k] = f2u(v[k]);
    else if constexpr (DT == ZQ_BF16) w[k] = bf16x2_bits(v[2 * k], v[2 * k + 1]);
    else w[k] = f2h(v[2 * k]) | (f2h(v[2 * k + 1]) << 16);
  }
  store_words<NT, NW>(static_cast<char*>(p) + i * elem_size<DT>(), w);
}

template <int DT>
__device__ __forceinline__ float load1(const void* p, int64_t i) {
  if constexpr (DT == ZQ_F32) return static_cast<const float*>(p)[i];
  else if constexpr (DT == ZQ_BF16) return u2f((uint32_t)static_cast<const uint16_t*>(p)[i] << 16);
  else return h2f(static_cast<const uint16_t*>(p)[i]);
}

template <int DT>
__device__ __forceinline__ void store1(void* p, int64_t i, float v) {
  if constexpr (DT == ZQ_F32) static_cast<float*>(p)[i] = v;
  else if constexpr (DT == ZQ_BF16) static_cast<uint16_t*>(p)[i] = (uint16_t)(bf16x2_bits(v, 0.0f) & 0xffffu);
  else static_cast<uint16_t*>(p)[i] = (uint16_t)f2h(v);
}


}  // namespace

// ------------------------------------------------------------------ quantise
// Full blocks only.  A lane owns E elements of one block, as C = E*size/16
// chunks of 16 bytes: L = B/E lanes hold the block, and chunk j of the
// block's lane i is the block's chunk j*L + i, so each load instruction of a
// wave reads whole runs of L*16 bytes while the block's absmax, scale and
// reciprocal are computed once per lane for all E elements.  One wave tile
// is 64/L blocks; a workgroup's tiles are adjacent.  The codes and scales of
// a workgroup are staged in LDS and written back as one contiguous run of
// 16-byte stores: at this kernel's ~8:1 read:write mix
// that keeps the write stream from slowing the reads (per-lane 2-byte stores
// measured ~10% slower).  A workgroup holding the last, partial tile stores
// straight from its lanes instead.  When n is not a multiple of B, one more
// workgroup quantises the short last block, in the same launch.

// The one short block [start, start + len), len < B <= 1024, quantised by
// one wave; the scale goes to *scale.
template <int DT, int QBITS>
__device__ __forceinline__ void quantize_tail(const void* __restrict__ x, int64_t start, int len,
                                              uint8_t* __restrict__ out, float* __restrict__ scale) {
  constexpr float QMAX = QBITS == 8 ? 127.0f : 7.0f;
  const int lane = threadIdx.x & 63;
  float a = 0.0f;
  for (int j = lane; j < len; j += 64) a = fmaxf(a, fabsf(load1<DT>(x, start + j)));
  const float amax = u2f(wave_max(f2u(a)));
  float s = 0.0f, r = 0.0f;
  if (amax >= kFlushBelow) {
    s = scale_of<(int)QMAX>(amax);
    r = QMAX / amax;
  }
  if constexpr (QBITS == 8) {
    for (int j = lane; j < len; j += 64) out[start + j] = (uint8_t)code_bits(load1<DT>(x, start + j), r);
  } else {
    for (int k = lane; 2 * k < len; k += 64) {
      uint32_t lo = code_bits(load1<DT>(x, start + 2 * k), r);
      uint32_t hi = (2 * k + 1 < len) ? code_bits(load1<DT>(x, start + 2 * k + 1), r) : 0u;
      out[(start >> 1) + k] = (uint8_t)((lo & 0xfu) | ((hi & 0xfu) << 4));
    }
  }
  if (lane == 0) *scale = s;
}

template <int DT, int QBITS, int B>
__global__ void __launch_bounds__(kQuantThreads) k_quantize(const void* __restrict__ x, int64_t nfull,
                                                            uint8_t* __restrict__ out, float* __restrict__ scales,
                                                            int tail) {
  constexpr int E = quant_elems(elem_size<DT>(), B), L = B / E, BPW = 64 / L;
  constexpr int CE = 16 / elem_size<DT>(), C = E / CE;          // elements per chunk, chunks per lane
  constexpr int T = quant_tiles(elem_size<DT>()), WAVES = kQuantThreads / 64;
  constexpr float QMAX = QBITS == 8 ? 127.0f : 7.0f;
  constexpr int NT = QBITS == 8 ? ZQ_NT_QUANT8 : ZQ_NT_QUANT4;
  constexpr int OB = QBITS == 8 ? E : E / 2;                    // code bytes per lane and tile
  constexpr int OBC = OB / C;                                   // code bytes per chunk
  constexpr int BB = B * OB / E;                                // code bytes per block
  constexpr int WG_BLOCKS = WAVES * T * BPW;                    // blocks per workgroup
  constexpr int WG_BYTES = WAVES * T * 64 * OB;                 // code bytes per workgroup
  constexpr int NWO = OB >= 4 ? OB / 4 : 1;
  static_assert(E % CE == 0 && L >= 1 && L <= 64 && WG_BYTES % 16 == 0, "lane layout");
  static_assert(OBC == 2 || OBC % 4 == 0, "chunk codes");
  __shared__ u32x4 obuf[WG_BYTES / 16];
  __shared__ float sbuf[WG_BLOCKS];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // with a short last block (tail > 0 elements) the launch has one workgroup
  // more than the full blocks need: the last one quantises that block with
  // its first wave (scalar test: 32-bit workgroup indices)
  if (tail > 0 && blockIdx.x == gridDim.x - 1) {
    if (wave == 0) quantize_tail<DT, QBITS>(x, nfull * B, tail, out, scales + nfull);
    return;
  }
  // workgroup g owns tiles [g*WAVES*T, (g+1)*WAVES*T); its t-th round of loads
  // covers WAVES adjacent tiles, one per wave
  const int64_t wg_blk0 = (int64_t)blockIdx.x * WG_BLOCKS;
  const int li = lane % L;  // the lane's index within its block
  prio_issue<ZQ_PRIO_QUANT>();
  float v[T][E];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int64_t blk = wg_blk0 + (t * WAVES + wave) * BPW + lane / L;
#pragma unroll
    for (int j = 0; j < C; ++j) {
      float c[CE];
      if (blk < nfull) {
        load_elems<NT, DT, CE>(x, blk * B + (int64_t)(j * L + li) * CE, c);
      } else {
#pragma unroll
        for (int k = 0; k < CE; ++k) c[k] = 0.0f;
      }
#pragma unroll
      for (int k = 0; k < CE; ++k) v[t][j * CE + k] = c[k];
    }
  }
  prio_compute<ZQ_PRIO_QUANT>();
  const bool full = wg_blk0 + WG_BLOCKS <= nfull;  // workgroup-uniform
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int slot = t * WAVES + wave;              // tile index within the workgroup
    const int64_t blk = wg_blk0 + slot * BPW + lane / L;
    float a = fabsf(v[t][0]);
#pragma unroll
    for (int k = 1; k < E; ++k) a = fmaxf(a, fabsf(v[t][k]));
    const float amax = u2f(group_max<L>(f2u(a)));
    float s = 0.0f, r = 0.0f;
    if (amax >= kFlushBelow) {
      s = scale_of<(int)QMAX>(amax);
      r = QMAX / amax;
    }
    uint32_t m[E];
#pragma unroll
    for (int k = 0; k < E; ++k) m[k] = code_bits(v[t][k], r);

    // this lane's packed codes: OB bytes in element order (chunk j's codes are
    // bytes [j*OBC, (j+1)*OBC)), little-endian in w
    uint32_t w[NWO];
    if constexpr (QBITS == 8) {
#pragma unroll
      for (int k = 0; k < E / 4; ++k) w[k] = pack_bytes4(m[4 * k], m[4 * k + 1], m[4 * k + 2], m[4 * k + 3]);
    } else if constexpr (E == 4) {
      w[0] = (m[0] & 0xfu) | ((m[1] & 0xfu) << 4) | ((m[2] & 0xfu) << 8) | ((m[3] & 0xfu) << 12);
    } else {
#pragma unroll
      for (int k = 0; k < E / 8; ++k) w[k] = pack_nibbles8(m + 8 * k);
    }

    // chunk j's codes go to byte (j*L + li)*OBC of the block's codes
    if (full) {
      char* ob = reinterpret_cast<char*>(obuf) + (slot * BPW + lane / L) * BB;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        char* d = ob + (j * L + li) * OBC;
        if constexpr (OBC == 2) {
          *reinterpret_cast<uint16_t*>(d) = (uint16_t)(w[j / 2] >> (16 * (j % 2)));
        } else {
#pragma unroll
          for (int k = 0; k < OBC / 4; ++k) reinterpret_cast<uint32_t*>(d)[k] = w[j * (OBC / 4) + k];
        }
      }
      if (li == 0) sbuf[slot * BPW + lane / L] = s;
    } else if (blk < nfull) {
      uint8_t* ob = out + blk * BB;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        uint8_t* d = ob + (j * L + li) * OBC;
        if constexpr (OBC == 2) {
          st<NT>(reinterpret_cast<uint16_t*>(d), (uint16_t)(w[j / 2] >> (16 * (j % 2))));
        } else {
          uint32_t wc[OBC / 4];
#pragma unroll
          for (int k = 0; k < OBC / 4; ++k) wc[k] = w[j * (OBC / 4) + k];
          store_words<NT, OBC / 4>(d, wc);
        }
      }
      if (li == 0) st<2 * ZQ_NT_SCALES>(scales + blk, s);
    }
  }
  if (full) {
    __syncthreads();
    u32x4* dst = reinterpret_cast<u32x4*>(out + wg_blk0 * BB);
#pragma unroll
    for (int c = tid; c < WG_BYTES / 16; c += kQuantThreads) st<NT>(dst + c, obuf[c]);
    if (tid < WG_BLOCKS) st<2 * ZQ_NT_SCALES>(scales + wg_blk0 + tid, sbuf[tid]);
  }
}

// ------------------------------------------------------------------ dequantise
// INT8 (QBITS 8) or INT4 (QBITS 4) codes -> binary32 products -> DT.  Thread g
// < n/E owns elements [gE, gE + E) (one block, since E <= B); the n % E
// leftover elements go to the following threads, one each.  When a thread's
// output is wider than 16 bytes, a workgroup stages its outputs in LDS and
// writes them back as wave-contiguous 16-byte stores (wide per-lane writes
// lose bandwidth); the workgroup holding the end of the tensor stores
// directly.

template <int DT, int QBITS>
__global__ void __launch_bounds__(kDeqThreads) k_dequant(const uint8_t* __restrict__ codes,
                                                      const float* __restrict__ scales, int64_t n, int lgB,
                                                      void* __restrict__ y) {
  constexpr int E = QBITS == 8 ? deq8_elems(elem_size<DT>()) : deq4_elems(elem_size<DT>());
  constexpr int NT = QBITS == 8 ? ZQ_NT_DEQ8 : ZQ_NT_DEQ4;
  constexpr int IB = QBITS == 8 ? E : E / 2;  // code bytes per thread
  constexpr int OB = E * elem_size<DT>();     // output bytes per thread
  constexpr bool STAGE = ZQ_DEQ_STAGE && OB > 16;
  static_assert(IB % 4 == 0 && OB % 16 == 0, "lane layout");
  __shared__ u32x4 ybuf[STAGE ? kDeqThreads * OB / 16 : 1];

  const int64_t ngroups = n / E;
  const int64_t g0 = (int64_t)blockIdx.x * kDeqThreads;
  const int64_t gid = g0 + threadIdx.x;
  if (STAGE && g0 + kDeqThreads <= ngroups) {  // workgroup-uniform
    const int64_t e0 = gid * E;
    uint32_t w[IB / 4];
    prio_issue<ZQ_PRIO_DEQ>();
    load_words<NT, IB / 4>(codes + (e0 * IB) / E, w);
    const float s = ld<NT>(scales + (e0 >> lgB));
    prio_compute<ZQ_PRIO_DEQ>();
    float v[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      if constexpr (QBITS == 8) v[k] = (float)(int32_t)(int8_t)(w[k >> 2] >> (8 * (k & 3))) * s;
      else v[k] = nib_to_f32(w[k >> 3], k & 7) * s;
    }
    store_elems<0, DT, E>(reinterpret_cast<char*>(ybuf) + threadIdx.x * OB, 0, v);
    __syncthreads();
    u32x4* dst = reinterpret_cast<u32x4*>(static_cast<char*>(y) + g0 * OB);
#pragma unroll
    for (int c = 0; c < OB / 16; ++c) st<NT>(dst + c * kDeqThreads + threadIdx.x, ybuf[c * kDeqThreads + threadIdx.x]);
  } else if (gid < ngroups) {
    const int64_t e0 = gid * E;
    uint32_t w[IB / 4];
    prio_issue<ZQ_PRIO_DEQ>();
    load_words<NT, IB / 4>(codes + (e0 * IB) / E, w);
    const float s = ld<NT>(scales + (e0 >> lgB));
    prio_compute<ZQ_PRIO_DEQ>();
    float v[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      if constexpr (QBITS == 8) v[k] = (float)(int32_t)(int8_t)(w[k >> 2] >> (8 * (k & 3))) * s;
      else v[k] = nib_to_f32(w[k >> 3], k & 7) * s;
    }
    store_elems<NT, DT, E>(y, e0, v);
  } else if (gid - ngroups < n - ngroups * E) {
    const int64_t i = ngroups * E + (gid - ngroups);
    float prod;
    if constexpr (QBITS == 8) prod = (float)(int32_t)(int8_t)codes[i] * scales[i >> lgB];
    else prod = nib_to_f32(codes[i >> 1], (int)(i & 1)) * scales[i >> lgB];
    store1<DT>(y, i, prod);
  }
}

// ------------------------------------------------------------------ reduce level
// Vector path: the full blocks [0, nfull), nfull >= the group size GB below.
// A lane owns E consecutive elements (E/2 bytes of every slice: consecutive
// lanes read consecutive bytes); L = B/E lanes hold one block; a wave tile is
// 64 lanes = BPW blocks.  The 4 waves of a workgroup take 4 adjacent tiles (a
// group of GB blocks).  Every load and store is addressed from a wave-uniform
// base plus the lane's offset, with no predicates: where GB does not divide
// nfull the last group is moved back to end at nfull and recomputes some of
// its neighbour's blocks, rewriting identical values.  Large levels use E = 32
// (16 B per slice per lane), small levels (few waves, often many slices)
// E = 8, so that four times as many waves run.
//
// Slices start where ceil(m/2) puts them, at any byte address when m % 32 is
// not 0, so slice words are loaded through types of alignment 1 (one
// global_load_dwordx4 all the same: the gfx9 ABI runs with unaligned global
// access on); outputs are always aligned.  A short last block (tail elements)
// is reduced by the first wave of one more workgroup of the same launch.
// Bound by HBM and, at few waves, by latency.  One launch over all of an odd
// level (P = 8, m = 15,432,099, B = 64: 17 us, 4.6 TB/s) replaced a wave per
// block with byte loads (171 us); the blocks after the last whole group used to
// take such waves too, one slice after the other (P = 64, m = 1,000,000,
// B = 256: 36.6 -> 14.1 us).
//
// Per slice and element: one v_cvt_off_f32_i4 (q/16), one multiply by 16*s
// ((q/16)*(16 s) is the exact real q*s, so the rounded product is fl(q*s)),
// one add.  16*s is exact unless it overflows (s > 2^123, i.e. inputs above
// ~7e37); a wave holding such a scale multiplies by 16 first instead.  The
// first slice initialises the sum with its product: +0 + x = x for every x but
// -0, and a -0 sum and a +0 sum requantise to the same code and scale.  Slices
// are summed in ascending order, exactly as defined.
//
// YDT >= 0 adds the fused final dequantisation: the requantised codes are
// turned back into fl(code * s_out) in YDT (the value qgz_dequantize would
// produce from this level's output) and written to y; out / sout may then be
// null, in which case the INT4 result is not stored.  Outputs wider than 16
// bytes per lane are staged in LDS and written as workgroup-contiguous
// 16-byte stores, as in the dequantiser.

// A wave-uniform value, held in scalar registers from here on.
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// The words at a wave-uniform address plus a lane's byte offset, from any byte
// address: one global load whose 64-bit part is in scalar registers.  (The
// builtin has to see the unaligned type, and the address space, which the
// conversion to scalar registers hides from the compiler.)
#define ZQ_GLOBAL __attribute__((address_space(1)))
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
template <int NW>
__device__ __forceinline__ void load_words_any(const void* base, uint32_t lane_byte, uint32_t (&w)[NW]) {
  static_assert(ZQ_NT_REDUCE & 1, "nontemporal loads");
  const ZQ_GLOBAL char* p =
      reinterpret_cast<const ZQ_GLOBAL char*>(uniform((int64_t)reinterpret_cast<uintptr_t>(base))) + lane_byte;
  if constexpr (NW == 4) {
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const ZQ_GLOBAL u32x4_any*>(p));
    w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
  } else {
    static_assert(NW == 1, "words");
    w[0] = __builtin_nontemporal_load(reinterpret_cast<const ZQ_GLOBAL u32_any*>(p));
  }
}

// The slices of one wave tile (up to U): words and scales.  Each slice's scale
// is loaded right after its words, so that its arithmetic starts when the two are
// there, and not when the last slice's are (all words first: P = 8, m =
// 100,663,296, B = 128 takes 86 us in place of 80).  Where a block spans the wave
// its scale is wave-uniform and a scalar load: a 64-lane load of one word costs the
// vector memory path as much as a row of them.
template <int U, int NW>
struct SliceBatch {
  uint32_t w[U][NW];
  float s[U];
};
template <int L, int NW>
__device__ __forceinline__ void load_slice(const uint8_t* bytes, uint32_t lane_byte, const float* scales,
                                           uint32_t lane_scale, uint32_t (&w)[NW], float& s) {
  load_words_any(bytes, lane_byte, w);
  if constexpr (L == 64) {
    s = *reinterpret_cast<const ZQ_GLOBAL float*>(uniform((int64_t)reinterpret_cast<uintptr_t>(scales)));
  } else {
    uint32_t sw[1];
    load_words_any(scales, 4 * lane_scale, sw);
    s = u2f(sw[0]);
  }
}

// One slice into a lane's sum: acc[k] = fl(acc[k] + fl(q_k * s)) for the E
// codes of the NW words ww (FIRST: acc[k] = fl(q_k * s)).  KEEP: an empty asm
// keeps each slice's additions where they are: the compiler otherwise moves
// those of a whole loop body behind its last slice and holds all products in
// registers meanwhile (two batches of 4: 325 registers, one wave per SIMD,
// against 122 and four).  It stands behind both branches, so that they meet in
// the products: with the additions inside the branches the 32 sums of a lane
// were copied between registers at every slice (P = 4, m = 100,663,296, B =
// 512: 59 us a level, 48 so).
template <int E, int NW, bool FIRST, bool KEEP = false>
__device__ __forceinline__ void add_slice(float (&acc)[E], const uint32_t (&ww)[NW], float sc) {
  const float s16 = sc * 16.0f;
  if (__all(s16 <= kMaxFloat)) {  // wave-uniform: 16*s exact for every lane
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      float f[8];
      nibbles_over_16(ww[j], f);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float prod = f[k] * s16;
        acc[8 * j + k] = FIRST ? prod : acc[8 * j + k] + prod;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      float f[8];
      nibbles_over_16(ww[j], f);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float prod = (f[k] * 16.0f) * sc;
        acc[8 * j + k] = FIRST ? prod : acc[8 * j + k] + prod;
      }
    }
  }
  if constexpr (KEEP) {
#pragma unroll
    for (int k = 0; k < E; ++k) asm volatile("" : "+v"(acc[k]));
  }
}

// Requantise one wave tile (blocks from blk0, in the group that starts at
// block gblk) and store its INT4 codes and scales (when out is not null) and, for YDT >= 0, the fused
// dequantisation fl(code * s_out) in YDT.  ybuf: the workgroup's LDS staging
// buffer for dequantised outputs wider than 16 bytes per lane; then every
// wave of the workgroup must call this for the same group.
template <int B, int E, int YDT>
__device__ __forceinline__ void requant_tile(const float (&acc)[E], int64_t blk0, int64_t gblk, int lane,
                                             uint8_t* __restrict__ out, float* __restrict__ sout,
                                             void* __restrict__ y, u32x4* ybuf) {
  constexpr int L = B / E, NW = E / 8;
  constexpr int YB = YDT < 0 ? 0 : E * elem_size<(YDT < 0 ? 0 : YDT)>();  // dequantised bytes per lane
  float a = fabsf(acc[0]);
#pragma unroll
  for (int k = 1; k < E; ++k) a = fmaxf(a, fabsf(acc[k]));
  const float amax = u2f(group_max<L>(f2u(a)));
  float so = 0.0f, r = 0.0f;
  if (amax >= kFlushBelow) {
    so = scale_of<7>(amax);
    r = 7.0f / amax;
  }
  uint32_t m[E];
#pragma unroll
  for (int k = 0; k < E; ++k) m[k] = code_bits(acc[k], r);
  if (out != nullptr) {
    uint32_t o[NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) o[j] = pack_nibbles8(m + 8 * j);
    store_words<ZQ_NT_REDUCE, NW>(out + blk0 * (B / 2) + lane * (E / 2), o);
    if (lane % L == 0) st<2 * ZQ_NT_SCALES>(sout + blk0 + lane / L, so);
  }
  if constexpr (YDT >= 0) {
    // code as float: (1.5*2^23 + q) - 1.5*2^23 = q exactly; then fl(q * s_out)
    float v[E];
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = (u2f(m[k]) - kRoundMagic) * so;
    if constexpr (YB > 16) {  // every wave of the workgroup is here, at the same group
      store_elems<0, YDT, E>(reinterpret_cast<char*>(ybuf) + threadIdx.x * YB, 0, v);
      __syncthreads();
      u32x4* dst = reinterpret_cast<u32x4*>(static_cast<char*>(y) + gblk * B * elem_size<YDT>());
#pragma unroll
      for (int c = 0; c < YB / 16; ++c)
        st<ZQ_NT_DEQ4>(dst + c * kThreads + threadIdx.x, ybuf[c * kThreads + threadIdx.x]);
      __syncthreads();
    } else {
      store_elems<ZQ_NT_DEQ4, YDT, E>(y, blk0 * B + (int64_t)lane * E, v);
    }
  }
}

// One block of len <= B elements by one wave (the short last block of a level,
// and every block of a level smaller than one group): plain arithmetic, the
// definition as written, sum from +0, one multiply and one add per slice.  A
// lane owns byte j = lane + 64 i of the block (elements 2j, 2j + 1).  The
// loads of U slices are in flight together (past the end: byte nbytes - 1 and
// slice P - 1 again, unused): 8, fewer where a lane has more than two bytes of each,
// so that this path does not set the registers of the kernels it is part of.
template <int B, typename Src>
__device__ __forceinline__ void reduce_block(const Src& src, int P, int64_t blk, int len, uint8_t* __restrict__ out,
                                             float* __restrict__ sout, void* __restrict__ y, int ydt) {
  constexpr int I = B > 128 ? B / 128 : 1, U = I > 2 ? 16 / I : 8;
  const int lane = threadIdx.x & 63;
  const int nbytes = (len + 1) >> 1;
  const int64_t base = blk * B;
  float acc[2 * I];
#pragma unroll
  for (int k = 0; k < 2 * I; ++k) acc[k] = 0.0f;
#pragma unroll 1
  for (int p0 = 0; p0 < P; p0 += U) {
    uint32_t w[U][I];
    float s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u < P ? p0 + u : P - 1;
      const uint8_t* b = src.bytes(p) + (base >> 1);
      s[u] = src.scales(p)[blk];
#pragma unroll
      for (int i = 0; i < I; ++i) {
        const int j = lane + 64 * i;
        w[u][i] = b[j < nbytes ? j : nbytes - 1];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p0 + u < P) {
#pragma unroll
        for (int i = 0; i < I; ++i) {
          acc[2 * i] = acc[2 * i] + nib_to_f32(w[u][i], 0) * s[u];
          acc[2 * i + 1] = acc[2 * i + 1] + nib_to_f32(w[u][i], 1) * s[u];
        }
      }
    }
  }
  float a = 0.0f;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = lane + 64 * i;
    if (j < nbytes) {
      a = fmaxf(a, fabsf(acc[2 * i]));
      if (2 * j + 1 < len) a = fmaxf(a, fabsf(acc[2 * i + 1]));
    }
  }
  const float amax = u2f(wave_max(f2u(a)));
  float so = 0.0f, r = 0.0f;
  if (amax >= kFlushBelow) {
    so = scale_of<7>(amax);
    r = 7.0f / amax;
  }
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int j = lane + 64 * i;
    if (j < nbytes) {
      const uint32_t lo = code_bits(acc[2 * i], r);
      const uint32_t hi = (2 * j + 1 < len) ? code_bits(acc[2 * i + 1], r) : 0u;
      if (out != nullptr) out[(base >> 1) + j] = (uint8_t)((lo & 0xfu) | ((hi & 0xfu) << 4));
      if (ydt >= 0) {
        const float v0 = (u2f(lo) - kRoundMagic) * so, v1 = (u2f(hi) - kRoundMagic) * so;
        const int64_t i0 = base + 2 * j;
        if (ydt == ZQ_F32) store1<ZQ_F32>(y, i0, v0);
        else if (ydt == ZQ_F16) store1<ZQ_F16>(y, i0, v0);
        else store1<ZQ_BF16>(y, i0, v0);
        if (2 * j + 1 < len) {
          if (ydt == ZQ_F32) store1<ZQ_F32>(y, i0 + 1, v1);
          else if (ydt == ZQ_F16) store1<ZQ_F16>(y, i0 + 1, v1);
          else store1<ZQ_BF16>(y, i0 + 1, v1);
        }
      }
    }
  }
  if (lane == 0 && out != nullptr) sout[blk] = so;
}

// Levels smaller than one group: one wave per block, the last one short when
// B does not divide m.
template <int B, typename Src>
__global__ void __launch_bounds__(64) k_reduce_blocks(Src src, int P, int64_t m, uint8_t* __restrict__ out,
                                                      float* __restrict__ sout, void* __restrict__ y, int ydt) {
  const int64_t blk = blockIdx.x, rest = m - blk * B;
  reduce_block<B>(src, P, blk, (int)(rest < B ? rest : B), out, sout, y, ydt);
}

// Any slice count, by batches of U slices in two register buffers, the loads of
// the next batch in flight while one is summed.  The first batch takes the slices
// that U does not divide (1 .. U of them, one copy of its code for each count), so
// that every other batch is whole, no load is repeated, and in the loop none is
// predicated: the compiler waits for exactly those it needs.  (With a last batch that
// loads slice P - 1 again in place of those it lacks, P = 9, m = 6,291,456, B =
// 128 took 11.4 us, 9.6 so.)
template <int B, int E, int U, int YDT, typename Src>
__global__ void __launch_bounds__(kThreads) k_reduce(Src src, int P, int64_t nfull, int tail, unsigned tail_wg,
                                                     uint8_t* __restrict__ out, float* __restrict__ sout,
                                                     void* __restrict__ y) {
  constexpr int L = B / E, BPW = 64 / L, NW = E / 8, WPG = kThreads / 64, GB = WPG * BPW;
  static_assert(L >= 1 && L <= 64 && (NW == 1 || NW == 4), "lane layout");
  constexpr int YB = YDT < 0 ? 0 : E * elem_size<(YDT < 0 ? 0 : YDT)>();  // dequantised bytes per lane
  __shared__ u32x4 ybuf[YB > 16 ? kThreads * YB / 16 : 1];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x == tail_wg) {
    if (wv == 0) reduce_block<B>(src, P, nfull, tail, out, sout, y, YDT);
    return;
  }
  const unsigned lane_byte = lane * (E / 2), lane_scale = lane / L;
  const int64_t last = nfull - GB, first = (int64_t)blockIdx.x * GB;
  const int64_t gblk = uniform(first < last ? first : last), blk0 = gblk + wv * BPW;
  const int whole = (P - 1) / U, first_n = P - whole * U;  // whole batches after the first one; its slices

  // N slices from slice p0 on of this wave's tile
  auto issue = [&](SliceBatch<U, NW>& X, int p0, auto n) {
#pragma unroll
    for (int u = 0; u < decltype(n)::value; ++u)
      load_slice<L>(src.bytes(p0 + u) + blk0 * (B / 2), lane_byte, src.scales(p0 + u) + blk0, lane_scale, X.w[u],
                    X.s[u]);
  };
  auto next = [&](SliceBatch<U, NW>& X, int b) { issue(X, first_n + b * U, std::integral_constant<int, U>{}); };
  float acc[E];
  auto sum = [&](const SliceBatch<U, NW>& X) {
#pragma unroll
    for (int u = 0; u < U; ++u) add_slice<E, NW, false, true>(acc, X.w[u], X.s[u]);
  };

  SliceBatch<U, NW> X0, X1;
  auto start = [&](auto n) {
    issue(X1, 0, n);
    if (whole > 0) next(X0, 0);
    add_slice<E, NW, true, true>(acc, X1.w[0], X1.s[0]);
#pragma unroll
    for (int u = 1; u < decltype(n)::value; ++u) add_slice<E, NW, false, true>(acc, X1.w[u], X1.s[u]);
  };
  static_assert(U == 3 || U == 4 || U == 6, "first batch");
  if (first_n == 1) start(std::integral_constant<int, 1>{});
  else if (first_n == 2) start(std::integral_constant<int, 2>{});
  else if (U == 3 || first_n == 3) start(std::integral_constant<int, 3>{});
  else if (U == 4 || first_n == 4) start(std::integral_constant<int, U < 4 ? U : 4>{});
  else if (first_n == 5) start(std::integral_constant<int, U < 5 ? U : 5>{});
  else start(std::integral_constant<int, U>{});
  int b = 0;
#pragma unroll 1
  for (; b + 2 < whole; b += 2) {
    next(X1, b + 1);
    sum(X0);
    next(X0, b + 2);
    sum(X1);
  }
  if (b + 1 < whole) {
    next(X1, b + 1);
    sum(X0);
    sum(X1);
  } else if (b < whole) {
    sum(X0);
  }
  requant_tile<B, E, YDT>(acc, blk0, gblk, lane, out, sout, y, ybuf);
}

// The slice count fixed at compile time (PC = 1 .. 8; E = 32 on large levels, E =
// 8 on small ones of 2, 4 and 8 slices).  Same lane layout, arithmetic and order as
// k_reduce, with all of a tile's slices loaded at once: the compiler waits for
// each slice's data on its own (s_waitcnt vmcnt(n) counting the loads issued
// after it), and the sum of slice 0 starts while the others are still
// arriving.  A workgroup takes TRC consecutive groups; with TRC > 1 the loads
// of a wave's next tile are issued before its current tile is summed, so they
// arrive while it computes (two register buffers).  The last workgroup clamps
// its group index to the last group and recomputes it.
template <int B, int E, int PC, int TRC, int YDT, typename Src>
__global__ void __launch_bounds__(kThreads) k_reduce_p(Src src, int, int64_t nfull, int tail, unsigned tail_wg,
                                                       uint8_t* __restrict__ out, float* __restrict__ sout,
                                                       void* __restrict__ y) {
  constexpr int L = B / E, BPW = 64 / L, NW = E / 8, WPG = kThreads / 64, GB = WPG * BPW, NBUF = TRC > 1 ? 2 : 1;
  static_assert(L >= 1 && L <= 64 && (NW == 1 || NW == 4) && PC >= 1 && TRC >= 1, "lane layout");
  constexpr int YB = YDT < 0 ? 0 : E * elem_size<(YDT < 0 ? 0 : YDT)>();
  __shared__ u32x4 ybuf[YB > 16 ? kThreads * YB / 16 : 1];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x == tail_wg) {
    if (wv == 0) reduce_block<B>(src, PC, nfull, tail, out, sout, y, YDT);
    return;
  }
  const unsigned lane_byte = lane * (E / 2), lane_scale = lane / L;
  const int64_t last = nfull - GB, first = (int64_t)blockIdx.x * (TRC * GB);
  auto group_blk = [&](int t) { return uniform(first + t * GB < last ? first + t * GB : last); };

  SliceBatch<PC, NW> X[NBUF];
  auto issue = [&](int buf, int64_t gblk) {
    const int64_t blk0 = gblk + wv * BPW;
#pragma unroll
    for (int p = 0; p < PC; ++p)
      load_slice<L>(src.bytes(p) + blk0 * (B / 2), lane_byte, src.scales(p) + blk0, lane_scale, X[buf].w[p],
                    X[buf].s[p]);
  };

  issue(0, group_blk(0));
#pragma unroll
  for (int t = 0; t < TRC; ++t) {
    if (t + 1 < TRC) issue((t + 1) % NBUF, group_blk(t + 1));
    float acc[E];
    add_slice<E, NW, true>(acc, X[t % NBUF].w[0], X[t % NBUF].s[0]);
#pragma unroll
    for (int p = 1; p < PC; ++p) add_slice<E, NW, false>(acc, X[t % NBUF].w[p], X[t % NBUF].s[p]);
    const int64_t gblk = group_blk(t);
    requant_tile<B, E, YDT>(acc, gblk + wv * BPW, gblk, lane, out, sout, y, ybuf);
  }
}

// ------------------------------------------------------------------ address tables
// Writes count (<= kTableChunk) 64-bit entries carried in the kernel
// arguments to dst[0, count): lane t stores entry t with a vector store.
__global__ void __launch_bounds__(kTableChunk) k_fill_table(uint64_t* __restrict__ dst, TableChunk chunk, int count) {
  const int t = threadIdx.x;
  if (t < count) dst[t] = chunk.v[t];
}

FillTableKernel fill_table_kernel() { return &k_fill_table; }

// ------------------------------------------------------------------ instantiation tables

template <int DT, int QB>
static QuantKernel quant_kernel_for(int lgB) {
  switch (lgB) {
    case 5: return &k_quantize<DT, QB, 32>;
    case 6: return &k_quantize<DT, QB, 64>;
    case 7: return &k_quantize<DT, QB, 128>;
    case 8: return &k_quantize<DT, QB, 256>;
    case 9: return &k_quantize<DT, QB, 512>;
    default: return &k_quantize<DT, QB, 1024>;
  }
}

QuantKernel quant_kernel(int dt, int qbits, int lgB) {
  if (qbits == 8) {
    if (dt == ZQ_F32) return quant_kernel_for<ZQ_F32, 8>(lgB);
    if (dt == ZQ_F16) return quant_kernel_for<ZQ_F16, 8>(lgB);
    return quant_kernel_for<ZQ_BF16, 8>(lgB);
  }
  if (dt == ZQ_F32) return quant_kernel_for<ZQ_F32, 4>(lgB);
  if (dt == ZQ_F16) return quant_kernel_for<ZQ_F16, 4>(lgB);
  return quant_kernel_for<ZQ_BF16, 4>(lgB);
}

DequantKernel dequant_kernel(int dt, int qbits) {
  if (qbits == 8) {
    if (dt == ZQ_F32) return &k_dequant<ZQ_F32, 8>;
    if (dt == ZQ_F16) return &k_dequant<ZQ_F16, 8>;
    return &k_dequant<ZQ_BF16, 8>;
  }
  if (dt == ZQ_F32) return &k_dequant<ZQ_F32, 4>;
  if (dt == ZQ_F16) return &k_dequant<ZQ_F16, 4>;
  return &k_dequant<ZQ_BF16, 4>;
}

// The reduce kernel of a level.  Large levels: the slice count fixed at compile
// time up to 8 (with two slices at B = 64 .. 256 a workgroup takes four groups),
// at or above the batches at every count and block size (1 slice, m =
// 100,663,296, B = 1024: 38.4 us by batches of 4, 23.2 fixed; 3 slices, B = 128:
// 48 and 39; 7, B = 512: 84 and 71); batches of 4 for 9 to 12 slices, where batches
// of 3 are up to 4% slower at 50 million elements and more, and of 3 beyond, which
// are level with them there and faster below (13 slices, m = 20,971,520, B = 128:
// 28.9 us, 30.1 with 4).  Small levels, which latency binds: 2, 4 and 8 fixed for B
// = 64 .. 256, else batches of 6 (64 slices, m = 1,048,576: B = 128 12.1 us, 13.4 by
// single buffers of 8; B = 512 12.3 and 14.8; with two buffers of 8 up to 8% slower
// at 13 slices and 6 million elements).
template <int B, int YDT, typename Src>
static ReduceKernel<Src> reduce_kernel_for(int P, bool small) {
  constexpr int EL = kReduceElems, ES = kReduceElemsSmall;
  if constexpr (B >= 64 && B <= 256) {
    if (small && P == 2) return &k_reduce_p<B, ES, 2, 1, YDT, Src>;
    if (small && P == 4) return &k_reduce_p<B, ES, 4, 1, YDT, Src>;
    if (small && P == 8) return &k_reduce_p<B, ES, 8, 1, YDT, Src>;
  }
  if constexpr (B <= 512) {
    if (small) return &k_reduce<B, ES, 6, YDT, Src>;
  }
  switch (P) {
    case 1: return &k_reduce_p<B, EL, 1, 1, YDT, Src>;
    case 2: return &k_reduce_p<B, EL, 2, reduce_groups(2, B, false), YDT, Src>;
    case 3: return &k_reduce_p<B, EL, 3, 1, YDT, Src>;
    case 4: return &k_reduce_p<B, EL, 4, 1, YDT, Src>;
    case 5: return &k_reduce_p<B, EL, 5, 1, YDT, Src>;
    case 6: return &k_reduce_p<B, EL, 6, 1, YDT, Src>;
    case 7: return &k_reduce_p<B, EL, 7, 1, YDT, Src>;
    case 8: return &k_reduce_p<B, EL, 8, 1, YDT, Src>;
    default: return P <= 12 ? &k_reduce<B, EL, 4, YDT, Src> : &k_reduce<B, EL, 3, YDT, Src>;
  }
}

template <int YDT, typename Src>
static ReduceKernel<Src> reduce_kernel_b(int lgB, int P, bool small) {
  switch (lgB) {
    case 5: return reduce_kernel_for<32, YDT, Src>(P, small);
    case 6: return reduce_kernel_for<64, YDT, Src>(P, small);
    case 7: return reduce_kernel_for<128, YDT, Src>(P, small);
    case 8: return reduce_kernel_for<256, YDT, Src>(P, small);
    case 9: return reduce_kernel_for<512, YDT, Src>(P, small);
    default: return reduce_kernel_for<1024, YDT, Src>(P, small);
  }
}

template <>
ReduceKernel<SlicesInRow> reduce_kernel(int lgB, int P, bool small, int ydt) {
  switch (ydt) {
    case ZQ_F32: return reduce_kernel_b<ZQ_F32, SlicesInRow>(lgB, P, small);
    case ZQ_F16: return reduce_kernel_b<ZQ_F16, SlicesInRow>(lgB, P, small);
    case ZQ_BF16: return reduce_kernel_b<ZQ_BF16, SlicesInRow>(lgB, P, small);
    default: return reduce_kernel_b<-1, SlicesInRow>(lgB, P, small);
  }
}

template <>
ReduceKernel<SlicesInTable> reduce_kernel(int lgB, int P, bool small, int) {
  return reduce_kernel_b<-1, SlicesInTable>(lgB, P, small);
}

template <>
ReduceKernel<SlicesInArgs> reduce_kernel(int lgB, int P, bool small, int) {
  return reduce_kernel_b<-1, SlicesInArgs>(lgB, P, small);
}

template <typename Src>
static ReduceBlocksKernel<Src> reduce_blocks_b(int lgB) {
  switch (lgB) {
    case 5: return &k_reduce_blocks<32, Src>;
    case 6: return &k_reduce_blocks<64, Src>;
    case 7: return &k_reduce_blocks<128, Src>;
    case 8: return &k_reduce_blocks<256, Src>;
    case 9: return &k_reduce_blocks<512, Src>;
    default: return &k_reduce_blocks<1024, Src>;
  }
}

template <>
ReduceBlocksKernel<SlicesInRow> reduce_blocks_kernel(int lgB) { return reduce_blocks_b<SlicesInRow>(lgB); }
template <>
ReduceBlocksKernel<SlicesInTable> reduce_blocks_kernel(int lgB) { return reduce_blocks_b<SlicesInTable>(lgB); }
template <>
ReduceBlocksKernel<SlicesInArgs> reduce_blocks_kernel(int lgB) { return reduce_blocks_b<SlicesInArgs>(lgB); }

}  // namespace zq
