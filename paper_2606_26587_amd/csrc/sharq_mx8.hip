// MXFP4 two-path GEMM on the dense backbone copy with 8 wavefronts per
// workgroup (gfx950; SharQ Sec. 3.3 eq. "sharq-output", Sec. 3.4).
//
// A workgroup computes 256 rows x 64 NF columns, each of its 8 wavefronts (two
// per SIMD) 64 x 32 NF.  One K step is a 128-position panel: both paths'
// activation codes, the weight codes and their scales go from global memory
// straight into LDS (three stages, 153 KB), two steps ahead of their use, so
// the step itself is 32 MFMAs, 20 LDS reads and ~17 VALU instructions per
// wavefront (NF 4) with no staging registers.  The MFMA order per output is
// that of the 4-wavefront kernel, so both give the same bits.
//
// What bounds it: the FP4 MFMA at the clock the part holds under it.  With
// neither loads nor LDS reads the gate/up shape below takes 172 us, without
// loads 184; with every load from one cached panel 204.
// Measured against the 4-wavefront kernel (us, weights streamed): M 2048, N 6144, K
// 4096 52.4 -> 47.9 (NF 3: one round of 256 tiles); N 28672 219.9 -> 210.8; M 4096,
// N 4096, K 4096 65.7 -> 59.7; M 2048, N 4096, K 14336 102.5, 111.3 here (NF 2).

#include "sharq_tile.hpp"

namespace sharq {

constexpr int kT8 = 512;                          // threads
constexpr int kOp8 = 256 * 64;                    // one operand of a 128-position step: 256 rows x 64 bytes
constexpr int kScale8 = 256 * 4;                  // its E8M0 scales
constexpr int kStage8 = 3 * kOp8 + 3 * kScale8;   // backbone, residual, weight; their scales
constexpr int kLds8 = 3 * kStage8;                // 153 KB; the epilogue reuses it

struct Args8 {
  const uint8_t *spd, *sps, *dnc, *dns, *wc, *ws;
  int64_t M;
  int N, K;
};

// Direct loads from global memory to LDS: lane l's 16 (4) bytes at base + off
// go to LDS address lds + 16 l (4 l).
__device__ __forceinline__ void dma16(uint32_t lds, uint64_t base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0");
}
__device__ __forceinline__ void dma4(uint32_t lds, uint64_t base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0");
}
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int SUB>
__device__ __forceinline__ v16f mma8(const uint4& b, const uint4& a, v16f c, uint32_t sb, uint32_t sa) {
  const auto op = [](const uint4& q) {
    v8i v;
    v[0] = (int)q.x; v[1] = (int)q.y; v[2] = (int)q.z; v[3] = (int)q.w;
    v[4] = 0; v[5] = 0; v[6] = 0; v[7] = 0;
    return v;
  };
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(op(b), op(a), c, 4, 4, SUB, (int)sb, SUB, (int)sa);
}

// This wavefront's share of a step's loads: 16-row slices (1 KB) w and w + 8
// of each operand, and a 64-row slice of the scales.
template <int NF>
struct Loader8 {
  uint64_t spd, dnc, wc, sps, dns, ws;   // at the tile's first row / column (uniform)
  uint32_t a0, a1, w0, w1, sa, sw;       // this lane's offsets
  int wave;
  int64_t R, N;

  __device__ __forceinline__ void issue(uint32_t stage, int step) const {
    const uint64_t pa = (uint64_t)step * (uint64_t)R, pn = (uint64_t)step * (uint64_t)N;
    const uint32_t l = stage + 1024u * (uint32_t)wave;
    dma16(l, spd + pa * 64, a0);
    dma16(l + 8192, spd + pa * 64, a1);
    dma16(l + kOp8, dnc + pa * 64, a0);
    dma16(l + kOp8 + 8192, dnc + pa * 64, a1);
    dma16(l + 2 * kOp8, wc + pn * 64, w0);
    if (NF > 2 && wave + 8 < 4 * NF) dma16(l + 2 * kOp8 + 8192, wc + pn * 64, w1);
    const uint32_t s = stage + 3 * kOp8 + 256u * (uint32_t)(wave & 3);
    if (wave < 4) dma4(s, sps + pa * 4, sa);
    else dma4(s + kScale8, dns + pa * 4, sa);
    if (wave < NF) dma4(s + 2 * kScale8, ws + pn * 4, sw);
  }
};

__device__ __forceinline__ uint4 lds8(const uint8_t* p) { return *reinterpret_cast<const uint4*>(p); }

template <int NF>
struct Scales8 {
  uint32_t sp[2], dn[2], w[NF];
};

template <int NF>
__device__ __forceinline__ void read_scales8(Scales8<NF>& s, const uint8_t* stage, int arow, int wrow, int half) {
  const uint8_t* p = stage + 3 * kOp8;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    s.sp[r] = *reinterpret_cast<const uint32_t*>(p + (arow + 32 * r) * 4) >> (16 * half);
    s.dn[r] = *reinterpret_cast<const uint32_t*>(p + kScale8 + (arow + 32 * r) * 4) >> (16 * half);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f)
    s.w[f] = *reinterpret_cast<const uint32_t*>(p + 2 * kScale8 + (wrow + 32 * f) * 4) >> (16 * half);
}

template <int NF>
struct Ops8 {
  uint4 sp[2], dn[2], b[NF];
};

// Operand J of a sub-step in the order of use (backbone, weights, residual)
template <int NF, int J>
__device__ __forceinline__ void read_op8(Ops8<NF>& o, const uint8_t* stage, uint32_t rd, uint32_t rd_a, uint32_t rd_w) {
  if constexpr (J < 2) o.sp[J] = lds8(stage + rd_a + 2048 * J + rd);
  else if constexpr (J < 2 + NF) o.b[J - 2] = lds8(stage + 2 * kOp8 + rd_w + 2048 * (J - 2) + rd);
  else o.dn[J - 2 - NF] = lds8(stage + kOp8 + rd_a + 2048 * (J - 2 - NF) + rd);
}

template <int NF, int SUB>
__device__ __forceinline__ void sub8(v16f (&acc)[2][NF], const Ops8<NF>& o, const Scales8<NF>& s, Ops8<NF>& n,
                                     const uint8_t* from, uint32_t rd, uint32_t rd_a, uint32_t rd_w) {
  static_for<0, 4 * NF>([&](auto ic) {
    constexpr int i = decltype(ic)::value, j = i % (2 * NF), f = j >> 1, r = j & 1;
    if constexpr (i < 2 * NF) acc[r][f] = mma8<SUB>(o.b[f], o.sp[r], acc[r][f], s.w[f], s.sp[r]);
    else acc[r][f] = mma8<SUB>(o.b[f], o.dn[r], acc[r][f], s.w[f], s.dn[r]);
    if constexpr (i < NF + 4) read_op8<NF, i>(n, from, rd, rd_a, rd_w);
  });
}

struct Tile8 {
  int64_t row_lo;
  int n0;
};

// This wavefront's loader for a tile.
template <int NF>
__device__ __forceinline__ void set_loader8(Loader8<NF>& ld, const Args8& p, const Tile8& t, int wave, int lane) {
  const int rows = (int)(p.M - t.row_lo < kRows8 ? p.M - t.row_lo : kRows8), cols = p.N - t.n0;
  const auto slice = [&](int row, int have) {   // rows past the last one reread it
    return (uint32_t)((row < have ? row : have - 1) * 64 + 16 * ((lane & 3) ^ swz_row(lane >> 2)));
  };
  ld.wave = wave;
  ld.R = p.M;
  ld.N = p.N;
  ld.a0 = slice(16 * wave + (lane >> 2), rows);
  ld.a1 = slice(16 * wave + 128 + (lane >> 2), rows);
  ld.w0 = slice(16 * wave + (lane >> 2), cols);
  ld.w1 = slice(16 * wave + 128 + (lane >> 2), cols);
  const int srow = 64 * (wave & 3) + lane;
  ld.sa = 4u * (uint32_t)(srow < rows ? srow : rows - 1);
  ld.sw = 4u * (uint32_t)(srow < cols ? srow : cols - 1);
  const auto at = [](const uint8_t* q) { return (uint64_t)uniform64((int64_t)reinterpret_cast<uintptr_t>(q)); };
  ld.spd = at(p.spd + t.row_lo * 64);
  ld.dnc = at(p.dnc + t.row_lo * 64);
  ld.wc = at(p.wc + (int64_t)t.n0 * 64);
  ld.sps = at(p.sps + t.row_lo * 4);
  ld.dns = at(p.dns + t.row_lo * 4);
  ld.ws = at(p.ws + (int64_t)t.n0 * 4);
}

// Tiles of 256 x 64 NF back to back, as handed out by next(Tile8&).  (Loading a
// tile's first steps before the previous tile's epilogue measured the same.)
template <typename OutT, int NF, class Next>
__device__ __forceinline__ void tiles8(const Args8& p, OutT* Y, int64_t ldy, uint8_t* lds, Next next) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1, col = lane & 31, half = lane >> 5;
  const int nks = p.K / 128;
  const uint32_t rd0 = (uint32_t)(col * 64 + 16 * ((2 * half) ^ swz_row(col)));
  const uint32_t rd1 = (uint32_t)(col * 64 + 16 * ((2 * half + 1) ^ swz_row(col)));
  const uint32_t rd_a = (uint32_t)(wm * 64 * 64), rd_w = (uint32_t)(wn * 32 * NF * 64);
  const int arow = wm * 64 + col, wrow = wn * 32 * NF + col;
  const uint32_t l0 =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;   // LDS address of the stages

  for (Tile8 t; next(t);) {
    Loader8<NF> ld;
    set_loader8<NF>(ld, p, t, wave, lane);
    ld.issue(l0, 0);
    if (nks > 1) ld.issue(l0 + kStage8, 1);
    dma_wait();
    __syncthreads();
    uint32_t q0 = l0, q1 = l0 + kStage8, q2 = l0 + 2 * kStage8;
    uint8_t *st0 = lds, *st1 = lds + kStage8, *st2 = lds + 2 * kStage8;
    v16f acc[2][NF];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[r][f][e] = 0.0f;
    Ops8<NF> x, y;
    Scales8<NF> sc, sn;
    static_for<0, NF + 4>([&](auto j) { read_op8<NF, decltype(j)::value>(x, st0, rd0, rd_a, rd_w); });
    read_scales8<NF>(sc, st0, arow, wrow, half);
    for (int s = 0; s < nks; ++s) {
      if (s + 2 < nks) ld.issue(q2, s + 2);
      sub8<NF, 0>(acc, x, sc, y, st0, rd1, rd_a, rd_w);
      read_scales8<NF>(sn, st1, arow, wrow, half);
      sub8<NF, 1>(acc, y, sc, x, st1, rd0, rd_a, rd_w);
      dma_wait();
      __syncthreads();
      sc = sn;
      uint8_t* m = st0;
      st0 = st1;
      st1 = st2;
      st2 = m;
      const uint32_t u = q0;
      q0 = q1;
      q1 = q2;
      q2 = u;
    }
    // every wavefront is past its last LDS read: the stages are free
    const int64_t row_hi = t.row_lo + kRows8 < p.M ? t.row_lo + kRows8 : p.M;
#pragma unroll
    for (int r = 0; r < 2; ++r)
      il_epilogue<OutT, NF>(acc[r], Y, ldy, t.row_lo, row_hi, t.n0 + wn * 32 * NF, p.N,
                            lds + wave * (32 * (64 * NF + 16)), 2 * wm + r, lane);
    __syncthreads();   // the LDS is free before the next tile's loads
  }
}

template <typename OutT, int NF>
__global__ __launch_bounds__(kT8) void k_linear_mx8(Args8 p, OutT* Y, int64_t ldy, int gx, int gy, int full) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kLds8];
  int id = (int)blockIdx.x;
  tiles8<OutT, NF>(p, Y, ldy, lds, [&](Tile8& t) {
    if (id >= full) return false;
    int mt, nt;
    tile_in_groups(xcd_unit(id, full), gx, gy, mt, nt);
    id += (int)gridDim.x;
    t.row_lo = (int64_t)mt * kRows8;
    t.n0 = nt * 64 * NF;
    return true;
  });
  if constexpr (NF == 4) {
    int u = (int)blockIdx.x;
    tiles8<OutT, 2>(p, Y, ldy, lds, [&](Tile8& t) {
      for (; u < 2 * (gx * gy - full); u += (int)gridDim.x) {
        int mt, nt;
        tile_in_groups(full + (u >> 1), gx, gy, mt, nt);
        t.n0 = nt * 256 + 128 * (u & 1);
        if (t.n0 >= p.N) continue;
        t.row_lo = (int64_t)mt * kRows8;
        u += (int)gridDim.x;
        return true;
      }
      return false;
    });
  }
}

template <typename OutT>
static hipError_t go8(const Args8& a, void* Y, int64_t ldy, hipStream_t st) {
  const Plan8 p = plan8(a.M, a.N, device_cus());
  OutT* y = reinterpret_cast<OutT*>(Y);
  const dim3 grid((unsigned)p.grid), block(kT8);
  if (p.nf == 4) k_linear_mx8<OutT, 4><<<grid, block, 0, st>>>(a, y, ldy, p.gx, p.gy, p.full);
  else k_linear_mx8<OutT, 3><<<grid, block, 0, st>>>(a, y, ldy, p.gx, p.gy, p.full);
  return hipGetLastError();
}

hipError_t launch_linear_mx8(int ydt, const uint8_t* spd, const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns,
                             int64_t M, const uint8_t* wc, const uint8_t* ws, int N, int K, void* Y, int64_t ldy,
                             hipStream_t st) {
  const Args8 a{spd, sps, dnc, dns, wc, ws, M, N, K};
  if (ydt == 2) return go8<float>(a, Y, ldy, st);
  if (ydt == 1) return go8<_Float16>(a, Y, ldy, st);
  return go8<uint16_t>(a, Y, ldy, st);
}

}  // namespace sharq
