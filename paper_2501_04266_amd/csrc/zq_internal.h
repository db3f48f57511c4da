// zq_internal.h -- launch geometry and kernel handles shared by the kernel and
// API translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zq {

constexpr int kThreads = 256;  // threads per workgroup of the streaming kernels (4 waves)
#ifndef ZQ_QUANT_THREADS
#define ZQ_QUANT_THREADS 256
#endif
constexpr int kQuantThreads = ZQ_QUANT_THREADS;
// wave tiles per wave in the quantiser: one for either input width (two
// tiles on 16-bit input measured slower than one tile of 16 elements per
// lane; on fp32 input two tiles measured slower too)
#ifndef ZQ_QUANT_TILES_F32
#define ZQ_QUANT_TILES_F32 1
#endif
#ifndef ZQ_QUANT_TILES_16
#define ZQ_QUANT_TILES_16 1
#endif
constexpr int quant_tiles(int dt_bytes) { return dt_bytes == 4 ? ZQ_QUANT_TILES_F32 : ZQ_QUANT_TILES_16; }
#ifndef ZQ_DEQ_THREADS
#define ZQ_DEQ_THREADS 256
#endif
constexpr int kDeqThreads = ZQ_DEQ_THREADS;


// Elements per lane.  Each wave handles one tile of 64 lanes x E elements and
// each workgroup four tiles; launches cover the whole tensor (no grid-stride
// loop), which measured fastest for streaming on gfx950.  Loads are 16 B per
// lane and instruction (a quantiser lane holding more takes several 16-byte
// chunks of its block, so each load instruction stays contiguous across the
// block's lanes) and each lane writes at most 32 contiguous bytes (wider
// per-lane writes lose bandwidth).  Quantiser: 4 elements per lane on fp32
// input (8 or 16, with half or a quarter of the VALU instructions per
// element, measured 3-5% slower), 16 on 16-bit input (2-3% faster than 8).
#ifndef ZQ_QUANT_E_F32
#define ZQ_QUANT_E_F32 4
#endif
#ifndef ZQ_QUANT_E_16
#define ZQ_QUANT_E_16 16
#endif
constexpr int quant_elems(int dt_bytes, int block) {
  int e = dt_bytes == 4 ? ZQ_QUANT_E_F32 : ZQ_QUANT_E_16;
  return block / e > 64 ? block / 64 : e;  // a block may span at most one wave
}
#ifndef ZQ_DEQ8_E_F32
#define ZQ_DEQ8_E_F32 8
#endif
#ifndef ZQ_DEQ8_E_16
#define ZQ_DEQ8_E_16 8
#endif
#ifndef ZQ_DEQ4_E_F32
#define ZQ_DEQ4_E_F32 16
#endif
#ifndef ZQ_DEQ4_E_16
#define ZQ_DEQ4_E_16 16
#endif
constexpr int deq8_elems(int out_bytes) { return out_bytes == 4 ? ZQ_DEQ8_E_F32 : ZQ_DEQ8_E_16; }
constexpr int deq4_elems(int out_bytes) { return out_bytes == 4 ? ZQ_DEQ4_E_F32 : ZQ_DEQ4_E_16; }
#ifndef ZQ_REDUCE_E
#define ZQ_REDUCE_E 32
#endif
constexpr int kReduceElems = ZQ_REDUCE_E;  // 16 bytes of every slice per lane
constexpr int kReduceElemsSmall = 8;  // 4 bytes per slice per lane, for small levels
// A level whose E = 32 launch would have fewer waves than this runs the small
// variant (4x the waves, more slices in flight per wave).
#ifndef ZQ_REDUCE_SMALL_WAVES
#define ZQ_REDUCE_SMALL_WAVES 4096
#endif

// (x, full blocks, out, scales, length of the short last block or 0)
using QuantKernel = void (*)(const void*, int64_t, uint8_t*, float*, int);
using DequantKernel = void (*)(const uint8_t*, const float*, int64_t, int, void*);

// Where the P slices of a reduce level are: back to back from one address each
// for bytes and scales, or at the addresses that two device tables hold (the
// peers' buffers mapped into this GPU's address space).
struct SlicesInRow {
  const uint8_t* in;
  const float* sin;
  int64_t slice_bytes, slice_scales;
  __device__ const uint8_t* bytes(int p) const { return in + p * slice_bytes; }
  __device__ const float* scales(int p) const { return sin + p * slice_scales; }
};
struct SlicesInTable {
  const uint8_t* const* in;
  const float* const* sin;
  __device__ const uint8_t* bytes(int p) const { return in[p]; }
  __device__ const float* scales(int p) const { return sin[p]; }
};
// The addresses themselves, as kernel arguments (1 KiB of them), for up to
// kArgSlices slices.
constexpr int kArgSlices = 64;
struct SlicesInArgs {
  const uint8_t* in[kArgSlices];
  const float* sin[kArgSlices];
  __device__ const uint8_t* bytes(int p) const { return in[p]; }
  __device__ const float* scales(int p) const { return sin[p]; }
};
// (slices, P, full blocks, length of the short last block and the workgroup that
// takes it (past the grid when there is none), out, scales, y)
template <typename Src>
using ReduceKernel = void (*)(Src, int, int64_t, int, unsigned, uint8_t*, float*, void*);
// (slices, P, m, out, scales, y, dtype of y or -1)
template <typename Src>
using ReduceBlocksKernel = void (*)(Src, int, int64_t, uint8_t*, float*, void*, int);

QuantKernel quant_kernel(int dt, int qbits, int lgB);
DequantKernel dequant_kernel(int dt, int qbits);
// Groups per workgroup of the kernel of a level (its launch covers the full
// blocks in groups of 4 wave tiles): four on large levels of two slices in blocks
// of 64 to 256, else one.
constexpr int reduce_groups(int P, int block, bool small) {
  return !small && block >= 64 && block <= 256 && P == 2 ? 4 : 1;
}
// ydt < 0: INT4 output only; otherwise also the fused dequantisation to ydt
// (slices in a row only)
template <typename Src>
ReduceKernel<Src> reduce_kernel(int lgB, int P, bool small, int ydt);
// one wave per block, for levels smaller than one group
template <typename Src>
ReduceBlocksKernel<Src> reduce_blocks_kernel(int lgB);
template <>
ReduceKernel<SlicesInRow> reduce_kernel(int lgB, int P, bool small, int ydt);
template <>
ReduceKernel<SlicesInTable> reduce_kernel(int lgB, int P, bool small, int ydt);
template <>
ReduceKernel<SlicesInArgs> reduce_kernel(int lgB, int P, bool small, int ydt);
template <>
ReduceBlocksKernel<SlicesInRow> reduce_blocks_kernel(int lgB);
template <>
ReduceBlocksKernel<SlicesInTable> reduce_blocks_kernel(int lgB);
template <>
ReduceBlocksKernel<SlicesInArgs> reduce_blocks_kernel(int lgB);
// a chunk of 64-bit table entries passed by value to the table-fill kernel
constexpr int kTableChunk = 64;
struct TableChunk {
  uint64_t v[kTableChunk];
};
using FillTableKernel = void (*)(uint64_t*, TableChunk, int);
FillTableKernel fill_table_kernel();

}  // namespace zq
