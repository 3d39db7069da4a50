// Tiles of the prefill GEMM kernels: sizes, activation rows, the order in
// which persistent workgroups walk the tiles, and the epilogue.
#pragma once

#include "sharq_dequant16.hpp"
#include "sharq_plan.hpp"

#include <type_traits>

namespace sharq {

constexpr int kBM = 128;          // tile rows: 4 wavefronts x 32
constexpr int kBK = 128;          // K per step: 4 scale blocks, 64 bytes of codes per row

// Activation rows live in panel-major buffers: K is cut into panels of 128
// positions (one K step; the last panel may be narrower) and panel p stores
// all R rows' bytes for its K range back to back, so the 32 rows of a
// wavefront are 2 KB (codes), 1 KB (backbone), 512 B (metadata) and 128 B
// (scales) of contiguous memory per step.
struct ARow {
  const uint8_t *dn, *spc, *spm, *dns, *sps;   // buffer bases
  int64_t r, R;                                // this lane's activation row, rows in the buffers
};

#define SHARQ_FENCE() __builtin_amdgcn_sched_barrier(0)

// f(std::integral_constant<int, I>{}) for I, ..., N - 1, unrolled.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Place of part q (16 bytes) of a staged 64-byte row in the 8-wavefront kernels:
// q ^ swz_row(row).  Reads of 32 rows and writes of 16 rows then have no bank
// conflict (with the places of the bf16 kernels they took 17% of the cycles).
__device__ __forceinline__ int swz_row(int row) { return ((row >> 2) ^ ((row >> 1) & 1)) & 3; }

template <typename OutT>
__device__ __forceinline__ void store_out(OutT* p, float v);
template <>
__device__ __forceinline__ void store_out<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_out<uint16_t>(uint16_t* p, float v) { *p = f32_to_bf16_rne(v); }
template <>
__device__ __forceinline__ void store_out<_Float16>(_Float16* p, float v) { *p = (_Float16)v; }

// Four consecutive outputs of one row.
template <typename OutT>
struct Vec4Out;
template <>
struct Vec4Out<float> {
  static __device__ __forceinline__ void put(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
  }
  static constexpr int kAlign = 16;
};
template <>
struct Vec4Out<uint16_t> {
  static __device__ __forceinline__ void put(uint16_t* p, float a, float b, float c, float d) {
    // v_cvt_pk_bf16_f32: two round-to-nearest-even conversions per instruction
    typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
    bf4 v;
    v[0] = (__bf16)a; v[1] = (__bf16)b; v[2] = (__bf16)c; v[3] = (__bf16)d;
    *reinterpret_cast<bf4*>(p) = v;
  }
  static constexpr int kAlign = 8;
};
template <>
struct Vec4Out<_Float16> {
  static __device__ __forceinline__ void put(_Float16* p, float a, float b, float c, float d) {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    h4 v;
    v[0] = (_Float16)a; v[1] = (_Float16)b; v[2] = (_Float16)c; v[3] = (_Float16)d;
    *reinterpret_cast<h4*>(p) = v;
  }
  static constexpr int kAlign = 8;
};

// A value that is the same in every lane, read from the first active one.
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Fourth dword of a raw buffer resource (no stride, no swizzle, 32-bit
// data format: the range check is on the byte offset).
constexpr int kBufferWord3 = 0x00020000;
typedef uint32_t v4u32_t __attribute__((ext_vector_type(4)));

constexpr int kEpiStride = 528;            // bytes per staged row: 512 + 16 (spreads rows over banks)
constexpr int kEpiWave = 32 * kEpiStride;  // one wavefront's region

// Epilogue of a wavefront's 32 x 256 block of 2-byte outputs through LDS.
// In the accumulator layout a lane holds 8-byte pieces of one output row, so
// direct stores put 32 scattered 16-byte pieces in every instruction (rows
// are N outputs apart); measured on the Llama prefill shapes this cost about
// 5 us per round of tiles.  Here the block is staged in LDS and read back
// along rows: each store instruction then writes two whole 512-byte row
// segments.  The wavefront owns its LDS region, and its LDS accesses execute
// in order, so no barrier is needed inside.
template <typename OutT, int NF>
__device__ __forceinline__ void store_tile_lds(const v16f (&acc)[NF], OutT* Y, int64_t ldy, int64_t row0,
                                               int64_t row_hi, int n0, int N, uint8_t* buf, int lane) {
  // a staged row is 64 NF bytes (+16); 4 NF lanes read it back, 16 / NF rows
  // per instruction (NF 3: 5 rows, the last 4 lanes and rows past 32 idle)
  constexpr int stride = 64 * NF + 16, lpr = 4 * NF, rpi = 64 / lpr;
  constexpr bool kEven = 32 % rpi == 0 && 64 % lpr == 0;
  const int r = lane & 31, half = lane >> 5;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      Vec4Out<OutT>::put(reinterpret_cast<OutT*>(buf + r * stride + (32 * f + 8 * g + 4 * half) * 2),
                         acc[f][4 * g], acc[f][4 * g + 1], acc[f][4 * g + 2], acc[f][4 * g + 3]);
    }
  }
  // every read back first: a store under a per-row condition would take its
  // read into its own branch and wait for it there, one LDS round trip per
  // store
  constexpr int kReads = (32 + rpi - 1) / rpi;
  uint4 v[kReads];
#pragma unroll
  for (int i = 0; i < kReads; ++i)
    v[i] = *reinterpret_cast<const uint4*>(buf + (rpi * i + lane / lpr) * stride + (lane % lpr) * 16);
  // row0 and row_hi are the same in every lane; the compiler cannot see it,
  // and a buffer resource held in vector registers would cost a loop over
  // lanes around every store
  row0 = uniform64(row0);
  row_hi = uniform64(row_hi);
  const int64_t rows = row_hi - row0 < 32 ? row_hi - row0 : 32;   // the wavefront's rows in the tile
  if (rows <= 0) return;
  const int64_t span = rows * ldy * (int64_t)sizeof(OutT);
  const int ch = lane % lpr, col = n0 + 8 * ch;
  const bool idle = !kEven && lane >= rpi * lpr;
  if (span <= (int64_t)1 << 30) {
    // Unconditional buffer stores over a range of exactly the wavefront's
    // rows: the range check drops a store to a row past the tile, and a
    // column past N gets an offset (2^31 - 16) past any such range.
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(Y + row0 * ldy, (short)0, (int)span,
                                                                        kBufferWord3);
#pragma unroll
    for (int i = 0; i < kReads; ++i) {
      const int rr = rpi * i + lane / lpr;
      const int off = col < N && (kEven || (!idle && rr < 32)) ? (int)(((int64_t)rr * ldy + col) * (int64_t)sizeof(OutT)) : 0x7FFFFFF0;
      v4u32_t q;
      q[0] = v[i].x; q[1] = v[i].y; q[2] = v[i].z; q[3] = v[i].w;
      __builtin_amdgcn_raw_buffer_store_b128(q, rs, off, 0, 0);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kReads; ++i) {
      const int rr = rpi * i + lane / lpr;
      if (rr < rows && col < N && !idle) *reinterpret_cast<uint4*>(Y + (row0 + rr) * ldy + col) = v[i];
    }
  }
}

// Epilogue.  2-byte outputs go through the wavefront's LDS region `epi` as
// whole row segments when the output allows 16-byte stores (every
// workgroup-uniform condition); otherwise each lane stores its own row, four
// consecutive columns per store.  The caller makes `epi` free.
template <typename OutT, int NF>
__device__ __forceinline__ void il_epilogue(const v16f (&acc)[NF], OutT* Y, int64_t ldy, int64_t row_lo,
                                            int64_t row_hi, int n0, int N, uint8_t* epi, int wave, int lane) {
  const int half = lane >> 5;
  if constexpr (sizeof(OutT) == 2) {
    if (((reinterpret_cast<uintptr_t>(Y) | (uintptr_t)(ldy * 2)) & 15u) == 0 && N % 8 == 0) {
      store_tile_lds<OutT, NF>(acc, Y, ldy, row_lo + wave * 32, row_hi, n0, N, epi, lane);
      return;
    }
  }
  const int64_t row = row_lo + wave * 32 + (lane & 31);
  if (row >= row_hi) return;
  OutT* yr = Y + row * ldy;
  const bool vec = ((reinterpret_cast<uintptr_t>(Y) | (uintptr_t)(ldy * (int64_t)sizeof(OutT))) &
                    (uintptr_t)(Vec4Out<OutT>::kAlign - 1)) == 0;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int col = n0 + f * 32 + 8 * g + 4 * half;
      if (vec && col + 3 < N) {
        Vec4Out<OutT>::put(yr + col, acc[f][4 * g], acc[f][4 * g + 1], acc[f][4 * g + 2], acc[f][4 * g + 3]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < N) store_out<OutT>(yr + col + e, acc[f][4 * g + e]);
      }
    }
  }
}

// Tile order.  Workgroups are dispatched round-robin over the 8 XCDs
// (workgroup id mod 8), each with its own L2.  The ids are renumbered so that
// each XCD walks a contiguous range of tiles, ordered in blocks of 4 M-tiles
// x 8 N-tiles: the 32 workgroups an XCD runs at once then share 4 activation
// tiles and 8 weight tiles in its L2.  Other grid shapes keep row-major order.
__device__ __forceinline__ void tile_of(int id, int gx, int gy, int& mt, int& nt) {
  const int total = gx * gy;
  if ((gx & 7) == 0 && (gy & 3) == 0) {
    const int per = total >> 3;
    const int idp = (id & 7) * per + (id >> 3);
    const int blk = idp >> 5, in = idp & 31;
    const int bx = gx >> 3;
    mt = (blk / bx) * 4 + (in & 3);
    nt = (blk % bx) * 8 + (in >> 2);
  } else {
    mt = id / gx;
    nt = id - mt * gx;
  }
}

// Half tile u of a last round run as `halves` half tiles behind `full` whole
// ones: tile t, columns 128 h on.
__device__ __forceinline__ void half_unit(int u, int full, int halves, int& t, int& h) {
  if ((halves & 15) == 0 && (full & 7) == 0) {
    t = full + ((u >> 4) << 3) + (u & 7);
    h = (u >> 3) & 1;
  } else {
    t = full + (u >> 1);
    h = u & 1;
  }
}

// Compute units of the current device (queried once per device).
inline int device_cus() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cache[dev] = n;
  }
  return cache[dev];
}

// Work units of the persistent kernel: whole tiles, with a last round that
// would be at most half full run as twice as many half tiles.
struct PersistPlan {
  int grid, full, halves;
};

inline PersistPlan persist_plan(int gx, int gy) {
  const int tiles = gx * gy, cus = device_cus();
  PersistPlan p{tiles < cus ? tiles : cus, tiles, 0};
  const int r = tiles % p.grid;
  if (tiles > p.grid && r > 0 && 2 * r <= p.grid) {
    p.full = tiles - r;
    p.halves = 2 * r;
  }
  return p;
}

// The NVFP4 weight tile of a 32-position step in the double-buffered pipelines
// (any K): one row per thread, dequantized to bf16 in LDS.
struct NvW {         // one thread's weight row for one block
  uint4 codes;
  uint32_t sc;
};

template <int NF>
__device__ __forceinline__ void load_nv_w(NvW& w, const uint8_t* wc, const uint8_t* ws, int n0, int N, int K,
                                          int ks) {
  static_assert(NF == 8, "one weight row per thread");
  const int p = ks >> 2, j = ks & 3, wp = min(128, K - 128 * p);
  const int64_t pn = (int64_t)p * N;
  const int n = min(n0 + (int)threadIdx.x, N - 1);
  w.codes = *reinterpret_cast<const uint4*>(wc + pn * 64 + (int64_t)n * (wp / 2) + 16 * j);
  w.sc = ws[pn * 4 + (int64_t)n * (wp / 32) + j];
}

// Dequantize this thread's weight row (32 values) into the LDS tile as bf16.
__device__ __forceinline__ void store_nv_w(const NvW& w, uint8_t* lds) {
  const int row = threadIdx.x;
  const float d = e4m3_value(w.sc);
  const uint32_t c[4] = {w.codes.x, w.codes.y, w.codes.z, w.codes.w};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<uint4*>(lds + row * 64 + 16 * (q ^ swz_nv(row))) = dequant8_bf16(c[q], d);
}

}  // namespace sharq
