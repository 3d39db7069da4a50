// NVFP4 two-path prefill GEMM for gfx950 (SharQ Sec. 3.3 eq. "sharq-output";
// Sec. 3.4 "Shared FP4 weights with path-specific scales").
//
// NVFP4 block scales are E4M3 (not powers of two), which the block-scaled FP4
// MFMA cannot apply, so both operands are dequantized exactly (q * d) and
// multiplied on 16-bit MFMA; the per-tensor scales S_x * S_w are applied once
// in the epilogue.  K a multiple of 128 runs on the persistent kernel below in
// fp16; other K on a double-buffered one in bf16.

#include "sharq_tile.hpp"

namespace sharq {

// The small-M kernel of the formats on 16-bit MFMA (sharq_skinny16.hip).
hipError_t launch_linear_skinny16(bool nv, int pat, int ydt, const uint8_t* spc, const uint8_t* spm,
                                  const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns, const float* tsx,
                                  int64_t M, const uint8_t* wc, const uint8_t* ws, const float* tsw, int N, int K,
                                  void* Y, int64_t ldy, hipStream_t st);

// ---------------------------------------------------------------------------
// K not a multiple of 128
// ---------------------------------------------------------------------------
//
// One K step is one 32-position block.  Activation fragments are dequantized
// in the registers of the wavefront that owns the rows; the weight tile is
// dequantized once per workgroup into LDS (bf16, 64 bytes per row, parts
// XOR-swizzled).
//
// bf16 32x32x16 operand layout: lane l holds row l % 32 and K values
// 8 (l / 32) + 0..7; the accumulator layout is that of the FP4 MFMA.

struct NvA {         // one lane's activation data for one 32-position block
  uint4 dn;          // residual codes
  uint2 spc;         // compressed backbone codes
  uint32_t spm;      // backbone metadata
  uint32_t ssc;      // backbone E4M3 scale (byte 0)
  uint32_t dsc;      // residual E4M3 scales of the two 16-halves (bytes 0, 1)
};

__device__ __forceinline__ void load_nv_a(NvA& s, const ARow& a, int ks, int K) {
  const int p = ks >> 2, j = ks & 3, wp = min(128, K - 128 * p);
  const int64_t pr = (int64_t)p * a.R;
  s.dn = *reinterpret_cast<const uint4*>(a.dn + pr * 64 + a.r * (wp / 2) + 16 * j);
  s.spc = *reinterpret_cast<const uint2*>(a.spc + pr * 32 + a.r * (wp / 4) + 8 * j);
  s.spm = *reinterpret_cast<const uint32_t*>(a.spm + pr * 16 + a.r * (wp / 8) + 4 * j);
  s.ssc = a.sps[pr * 4 + a.r * (wp / 32) + j];
  s.dsc = *reinterpret_cast<const uint16_t*>(a.dns + pr * 8 + a.r * (wp / 16) + 2 * j);
}

template <int PAT, int NF>
__device__ __forceinline__ void step_nv(v16f (&acc)[NF], const NvA& a, const uint8_t* lw, int lane) {
  const int half = lane >> 5, col = lane & 31;
  const uint4 sp = expand_block<PAT>(a.spc, a.spm);
  const float dsp = e4m3_value(a.ssc & 0xFFu);
  const float d0 = e4m3_value(a.dsc & 0xFFu), d1 = e4m3_value((a.dsc >> 8) & 0xFFu);
  const uint32_t spw[4] = {sp.x, sp.y, sp.z, sp.w};
  const uint32_t dnw[4] = {a.dn.x, a.dn.y, a.dn.z, a.dn.w};
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    // K values 8 half + 16 t + 0..7: dword (half + 2 t) of the block; the
    // residual's 16-half is t
    const bf16x8 asp = as_bf16x8(dequant8_bf16(spw[half + 2 * t], dsp));
    const bf16x8 adn = as_bf16x8(dequant8_bf16(dnw[half + 2 * t], t ? d1 : d0));
    bf16x8 b[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int row = f * 32 + col;
      b[f] = as_bf16x8(*reinterpret_cast<const uint4*>(lw + row * 64 + 16 * ((half + 2 * t) ^ swz_nv(row))));
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(asp, b[f], acc[f], 0, 0, 0);
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(adn, b[f], acc[f], 0, 0, 0);
  }
}

template <int NF, int PAT, typename OutT>
__global__ __launch_bounds__(256) void k_linear_nv(const uint8_t* sp_codes, const uint8_t* sp_meta,
                                                   const uint8_t* sp_scale, const uint8_t* dn_codes,
                                                   const uint8_t* dn_scale, const float* ts_x, int64_t M,
                                                   const uint8_t* wc, const uint8_t* ws, const float* ts_w, int N,
                                                   int K, OutT* Y, int64_t ldy, int gx, int gy) {
  constexpr int BN = 32 * NF;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BN * 64];
  int mt, nt;
  tile_of(blockIdx.x, gx, gy, mt, nt);
  const int n0 = nt * BN;
  const int64_t row_lo = (int64_t)mt * kBM;
  const int64_t row_hi = row_lo + kBM < M ? row_lo + kBM : M;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  const int nks = K / 32;

  int64_t orow = row_lo + wave * 32 + (lane & 31);
  if (orow >= row_hi) orow = row_hi - 1;
  ARow a;
  a.r = orow;
  a.R = M;
  a.dn = dn_codes;
  a.spc = sp_codes;
  a.spm = sp_meta;
  a.dns = dn_scale;
  a.sps = sp_scale;

  v16f acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[f][r] = 0.0f;

  NvA a0, a1;
  NvW wn;
  const int last = nks - 1;
  load_nv_w<NF>(wn, wc, ws, n0, N, K, 0);
  load_nv_a(a0, a, 0, K);
  store_nv_w(wn, lds);
  load_nv_w<NF>(wn, wc, ws, n0, N, K, min(1, last));
  load_nv_a(a1, a, min(1, last), K);
  int ks = 0;
  for (; ks + 1 < nks; ks += 2) {
    __syncthreads();
    step_nv<PAT, NF>(acc, a0, lds, lane);
    store_nv_w(wn, lds + BN * 64);
    load_nv_w<NF>(wn, wc, ws, n0, N, K, min(ks + 2, last));
    load_nv_a(a0, a, min(ks + 2, last), K);
    __syncthreads();
    step_nv<PAT, NF>(acc, a1, lds + BN * 64, lane);
    store_nv_w(wn, lds);
    load_nv_w<NF>(wn, wc, ws, n0, N, K, min(ks + 3, last));
    load_nv_a(a1, a, min(ks + 3, last), K);
  }
  if (ks < nks) {
    __syncthreads();
    step_nv<PAT, NF>(acc, a0, lds, lane);
  }

  const float scale = *ts_x * *ts_w;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int col = n0 + f * 32 + (lane & 31);
    if (col >= N) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = row_lo + wave * 32 + 8 * (r / 4) + 4 * half + (r % 4);
      if (row < row_hi) store_out<OutT>(Y + row * ldy + col, acc[f][r] * scale);
    }
  }
}

// ---------------------------------------------------------------------------
// Persistent kernel (K a multiple of 128): NVFP4 on fp16 MFMA, HiF4 on bf16
// ---------------------------------------------------------------------------
//
// A workgroup of 8 wavefronts (two per SIMD: one's VALU and LDS work issues
// under the other's MFMAs) computes 64 WM rows x 64 NC columns, each wavefront 64
// rows x 32 NF columns: 256 rows x 256, 192 or 128 columns (WM 4, NF = NC), or 128
// x 256 (WM 2, NC 4, NF 2; the first four wavefronts dequantize the activations).
// One K step is one 32-position block.  Both operands of a step are
// dequantized once per workgroup into LDS, 16 activation values and 4 NC
// weight values a thread, two steps ahead of their use (three stages).  With 64 rows per
// wavefront a weight fragment read from LDS feeds two MFMAs; with 32 rows the
// reads alone need the whole LDS bandwidth at the MFMA's rate.
//
// NVFP4: both paths multiply the same weight, so where the two activation
// operands add up exactly in fp16 one MFMA does the work of two:
//   a_sp w + a_dn w = (a_sp + a_dn) w.
// a_sp = q1 d1 and a_dn = q2 d2 with E2M1 codes and E4M3 scales.  With E the
// smaller scale's exponent (at least -6, the subnormals'), both are multiples
// of 2^(E-4) and |a_sp + a_dn| <= 6 (d1 + d2), so the sum is exact in fp16 (11
// significant bits) when 6 (d1 + d2) < 2^(E+7), that is, in the scales' own
// steps of 2^(E-3), d1 + d2 <= 21.25 * 2^E.  It holds while the two scales are
// within about a factor of 16: for nearly every block but those with an
// outlier channel, whose backbone scale is far above its residual's.  The test
// is taken for 32 rows of a block together (one wavefront's share of the
// dequantization); where it fails the operands stay apart and the consumers
// run both MFMAs.  The fp32 sums then hold the same exact products either
// way, with fewer roundings where merged.  The choice depends on the scales
// alone, so every storage form of the backbone gives the same bits.
// HiF4 values are exact in bf16 only, whose 8 bits rarely hold such a sum: its
// operands always stay apart.
//
// What bounds it: the 16-bit MFMA.  An MFMA keeps the VALU port for about 16
// of its 32 cycles (measured: MFMAs with 8 and 12 VALU instructions each take
// 50 and 64 cycles with two wavefronts per SIMD), so per wavefront and step
// (256 x 256) 16 to 18 NVFP4 MFMAs leave room for about 70 VALU instructions; the
// dequantization takes 32 + 16 of them and its scales and addresses the rest.

constexpr int kFmtNv = 0, kFmtHf = 1;
constexpr int kT16 = 512;                     // threads
constexpr int kPart16 = 256 * 64;             // one operand of a step: 256 rows x 32 positions x 2 bytes
constexpr int kStage16 = 3 * kPart16;         // activation (merged, or backbone), weight, residual
constexpr int kLds16 = 3 * kStage16;          // 144 KB; the epilogue reuses it

struct Args16 {
  const uint8_t *spc, *spm, *sps, *dnc, *dns, *wc, *ws;
  const float *ts_x, *ts_w;   // NVFP4
  int64_t M;
  int N, K;
};

// A thread's codes of one step, from global memory: half h of a block of one
// activation row, and its share of a weight row's block.
struct Raw16 {
  uint2 dn;                  // residual codes
  uint32_t c0, c1;           // backbone: dense codes (pattern 0), or compressed codes and metadata
  uint2 w;                   // weight codes (one dword with 128 columns)
  uint32_t ssp, sdn, sw;     // NVFP4: E4M3 scales; HiF4: the units' metadata words
};

// Uniform bases (first row or column of the tile) and this thread's row and
// part in them; rows past the last one reread it.
template <int NC>
struct Tile16 {
  // threads that share a weight row's block: 16 values each, 8 with 128 columns
  static constexpr int kPerRow = NC == 2 ? 4 : 2;
  const uint8_t *dn, *spc, *spm, *dns, *sps, *wc, *ws;
  uint32_t arow, half, wrow, wpart;
  bool wactive, aactive;     // the same in every lane of a wavefront (192 columns: 6 wavefronts; 128 rows: 4)
};

// Block BLK of the panel with pm rows (pn columns) before it.
template <int FMT, int PAT, int NC, int BLK>
__device__ __forceinline__ void load16(Raw16& r, const Tile16<NC>& t, int64_t pm, int64_t pn, int part) {
  const uint32_t at = t.arow * 64 + 8 * t.half, wat = t.wrow * 64 + (NC == 2 ? 4 : 8) * t.wpart;
  if (part == 0) r.dn = *reinterpret_cast<const uint2*>(t.dn + pm * 64 + 16 * BLK + at);
  if (part == 1) {
    if (PAT == 0) {
      const uint2 c = *reinterpret_cast<const uint2*>(t.spc + pm * 64 + 16 * BLK + at);
      r.c0 = c.x;
      r.c1 = c.y;
    } else {
      r.c0 = *reinterpret_cast<const uint32_t*>(t.spc + pm * 32 + 8 * BLK + (at >> 1));
      r.c1 = *reinterpret_cast<const uint16_t*>(t.spm + pm * 16 + 4 * BLK + (at >> 2));
    }
  }
  if (part == 2) {
    if (NC == 2) r.w.x = *reinterpret_cast<const uint32_t*>(t.wc + pn * 64 + 16 * BLK + wat);
    else r.w = *reinterpret_cast<const uint2*>(t.wc + pn * 64 + 16 * BLK + wat);
  }
  if (FMT == kFmtNv) {
    if (part == 3) r.ssp = *(t.sps + pm * 4 + BLK + t.arow * 4);
    if (part == 4) r.sdn = *(t.dns + pm * 8 + 2 * BLK + (t.arow * 8 + t.half));
    if (part == 5) r.sw = *(t.ws + pn * 4 + BLK + t.wrow * 4);
  } else {   // a unit's word is at its even block
    if (part == 3) r.ssp = *reinterpret_cast<const uint32_t*>(t.sps + pm * 8 + 4 * (BLK >> 1) + t.arow * 8);
    if (part == 4) r.sdn = *reinterpret_cast<const uint32_t*>(t.dns + pm * 8 + 4 * (BLK >> 1) + t.arow * 8);
    if (part == 5) r.sw = *reinterpret_cast<const uint32_t*>(t.ws + pn * 8 + 4 * (BLK >> 1) + t.wrow * 8);
  }
}

// Where a thread writes: its activation row's two 16-byte parts (2 h, 2 h + 1)
// and its weight row's, at stage + these offsets.
struct Put16 {
  uint32_t a0, a1, w0, w1;
};

// Dequantization of a step into its LDS stage, in pieces that fill MFMA slots.
// BLK: block of the panel (HiF4: its parity is the half of the unit).
template <int FMT, int PAT, int NC, int BLK>
struct Fill16 {
  f16x2 dsp, ddn, addend, dw;
  bool merged;
  uint32_t h0, h1, h2;   // pairs waiting for their 16-byte part

  static __device__ __forceinline__ uint32_t backbone(const Raw16& r, int d) {
    if (PAT == 0) return d == 0 ? r.c0 : r.c1;
    return d == 0 ? expand_dw<PAT == 0 ? 24 : PAT, 0>(make_uint2(r.c0, 0u), r.c1)
                  : expand_dw<PAT == 0 ? 24 : PAT, 1>(make_uint2(r.c0, 0u), r.c1);
  }

  template <int I>
  __device__ __forceinline__ uint32_t pair(uint32_t e, uint32_t c) const {
    const f16x2 q1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(e, 1.0f, I);
    const f16x2 q2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(c, 1.0f, I);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(q1, dsp, q2 * addend));
  }

  // NVFP4: scales and the merge test; the flag of the wavefront's 32 rows goes to the stage's flags.
  __device__ __forceinline__ void scales(const Raw16& r, uint32_t* flags, int wave, int lane) {
    const float d1 = e4m3_value(r.ssp), d2 = e4m3_value(r.sdn);
    const _Float16 a = (_Float16)d1, b = (_Float16)d2;
    dsp = f16x2{a, a};
    ddn = f16x2{b, b};
    const float pe = fmaxf(__uint_as_float(__float_as_uint(fminf(d1, d2)) & 0x7F800000u), 0x1p-6f);   // 2^E
    merged = __builtin_amdgcn_ballot_w64(d1 + d2 <= pe * 21.25f) == ~0ull;
    addend = __builtin_bit_cast(f16x2, __builtin_bit_cast(uint32_t, ddn) & (merged ? ~0u : 0u));
    if (lane == 0) flags[wave] = merged ? 0u : 1u;
  }

  // Pieces 0..7: the activation (NVFP4, piece 0 with its scales); 8..11: the weight.
  template <int I>
  __device__ __forceinline__ void piece(const Raw16& r, uint8_t* stage, const Put16& put, const Tile16<NC>& t,
                                        uint32_t* flags, int wave, int lane) {
    if constexpr (I < 8) {
      if (!t.aactive) return;
    }
    if constexpr (FMT == kFmtNv) {
      if constexpr (I == 0) scales(r, flags, wave, lane);
      if constexpr (I < 8) {
        constexpr int d = I >> 2, i = I & 3;
        const uint32_t v = pair<i>(backbone(r, d), d == 0 ? r.dn.x : r.dn.y);
        if constexpr (i == 0) h0 = v;
        if constexpr (i == 1) h1 = v;
        if constexpr (i == 2) h2 = v;
        if constexpr (i == 3)
          *reinterpret_cast<uint4*>(stage + (d == 0 ? put.a0 : put.a1)) = make_uint4(h0, h1, h2, v);
        if constexpr (I == 7) {
          if (!merged) {
            *reinterpret_cast<uint4*>(stage + 2 * kPart16 + put.a0) = nv_dequant8(r.dn.x, ddn);
            *reinterpret_cast<uint4*>(stage + 2 * kPart16 + put.a1) = nv_dequant8(r.dn.y, ddn);
          }
        }
      } else if (t.wactive) {
        if constexpr (I == 8) dw = nv_scale2(r.sw);
        if constexpr (I == 9) *reinterpret_cast<uint4*>(stage + kPart16 + put.w0) = nv_dequant8(r.w.x, dw);
        if constexpr (I == 11 && NC != 2) *reinterpret_cast<uint4*>(stage + kPart16 + put.w1) = nv_dequant8(r.w.y, dw);
      }
    } else {
      constexpr int hb = BLK & 1;
      const int q = 2 * (int)t.half;
      if constexpr (I == 0)
        *reinterpret_cast<uint4*>(stage + put.a0) = hf_dequant8(backbone(r, 0), hf_scales(r.ssp, hb, q));
      if constexpr (I == 2)
        *reinterpret_cast<uint4*>(stage + put.a1) = hf_dequant8(backbone(r, 1), hf_scales(r.ssp, hb, q + 1));
      if constexpr (I == 4)
        *reinterpret_cast<uint4*>(stage + 2 * kPart16 + put.a0) = hf_dequant8(r.dn.x, hf_scales(r.sdn, hb, q));
      if constexpr (I == 6)
        *reinterpret_cast<uint4*>(stage + 2 * kPart16 + put.a1) = hf_dequant8(r.dn.y, hf_scales(r.sdn, hb, q + 1));
      if constexpr (I >= 8) {
        if (t.wactive) {
          const int wq = NC == 2 ? (int)t.wpart : 2 * (int)t.wpart;
          if constexpr (I == 8)
            *reinterpret_cast<uint4*>(stage + kPart16 + put.w0) = hf_dequant8(r.w.x, hf_scales(r.sw, hb, wq));
          if constexpr (I == 10 && NC != 2)
            *reinterpret_cast<uint4*>(stage + kPart16 + put.w1) = hf_dequant8(r.w.y, hf_scales(r.sw, hb, wq + 1));
        }
      }
    }
  }
};

template <int FMT>
__device__ __forceinline__ v16f mma16(const uint4& b, const uint4& a, v16f c) {
  if constexpr (FMT == kFmtNv) return __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(b), as_f16x8(a), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(b), as_bf16x8(a), c, 0, 0, 0);
}

__device__ __forceinline__ uint4 lds16(const uint8_t* p) { return *reinterpret_cast<const uint4*>(p); }

// One step on the stage at `cur` (its first sub-step's operands in a0 / b0),
// with the fill of the stage two steps ahead and the loads of the step after
// that in its slots.  rd0, rd1: this lane's offsets of sub-steps 0 and 1 in an
// operand's fragment.  The stage's residual products follow each sub-step:
// always (HiF4), or for the row fragments whose paths stay apart.
template <int FMT, int PAT, int NC, int NF, int FB, class Load>
__device__ __forceinline__ void step16(v16f (&acc)[2][NF], uint4 (&a0)[2], uint4 (&b0)[NF], const uint8_t* cur,
                                       const uint8_t* nxt, uint8_t* fill, uint32_t rd0, uint32_t rd1, uint32_t rd_w,
                                       uint32_t rd_a, const uint32_t* cur_flags, uint32_t* fill_flags,
                                       const Raw16& raw, const Put16& put, const Tile16<NC>& t, int wave, int lane,
                                       Load load) {
  constexpr int kSlots = 4 * NF;
  Fill16<FMT, PAT, NC, FB> fl;
  uint4 a1[2], b1[NF], d[2];
  uint32_t apart0 = 0u, apart1 = 0u;
  if constexpr (FMT == kFmtNv) {
    apart0 = cur_flags[0];
    apart1 = cur_flags[1];
  }
  const uint8_t *ca = cur + rd_a, *cw = cur + kPart16 + rd_w, *cd = cur + 2 * kPart16 + rd_a;
  const uint8_t *na = nxt + rd_a, *nw = nxt + kPart16 + rd_w;
  static_for<0, 2>([&](auto tc) {
    constexpr int T = decltype(tc)::value;
    uint4(&a)[2] = T ? a1 : a0;
    uint4(&b)[NF] = T ? b1 : b0;
    uint4(&an)[2] = T ? a0 : a1;
    uint4(&bn)[NF] = T ? b0 : b1;
    const uint32_t rn = T ? rd0 : rd1;
    if constexpr (FMT == kFmtHf) {
      d[0] = lds16(cd + (T ? rd1 : rd0));
      d[1] = lds16(cd + 2048 + (T ? rd1 : rd0));
    }
    static_for<0, 2 * NF>([&](auto sc) {
      constexpr int i = decltype(sc)::value, f = i >> 1, r = i & 1, slot = T * 2 * NF + i;
      acc[r][f] = mma16<FMT>(b[f], a[r], acc[r][f]);
      // the operands of the next sub-step, in the order of their use
      if constexpr (FMT == kFmtNv) {
        if constexpr (i < 2) an[i] = lds16((T ? na : ca) + 2048 * i + rn);
        else if constexpr (i < 2 + NF) bn[i - 2] = lds16((T ? nw : cw) + 2048 * (i - 2) + rn);
      }
      load(std::integral_constant<int, slot>{});
      static_for<slot * 12 / kSlots, (slot + 1) * 12 / kSlots>([&](auto pc) {
        fl.template piece<decltype(pc)::value>(raw, fill, put, t, fill_flags, wave, lane);
      });
    });
    if constexpr (FMT == kFmtHf) {
      static_for<0, 2 * NF>([&](auto sc) {
        constexpr int i = decltype(sc)::value, f = i >> 1, r = i & 1;
        acc[r][f] = mma16<FMT>(b[f], d[r], acc[r][f]);
        if constexpr (i < 2) an[i] = lds16((T ? na : ca) + 2048 * i + rn);
        else if constexpr (i < 2 + NF) bn[i - 2] = lds16((T ? nw : cw) + 2048 * (i - 2) + rn);
      });
    } else {
      const uint32_t rt = T ? rd1 : rd0;
      if (__builtin_amdgcn_readfirstlane((int)apart0)) {
        const uint4 x = lds16(cd + rt);
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[0][f] = mma16<FMT>(b[f], x, acc[0][f]);
      }
      if (__builtin_amdgcn_readfirstlane((int)apart1)) {
        const uint4 x = lds16(cd + 2048 + rt);
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[1][f] = mma16<FMT>(b[f], x, acc[1][f]);
      }
      SHARQ_FENCE();
    }
  });
}

// One tile of 64 WM rows x 64 NC columns, rows from row_lo, columns from n0: WM by
// 8 / WM wavefronts of 64 rows x 32 NF columns.
template <int FMT, int PAT, typename OutT, int NC, int WM>
__device__ __forceinline__ void tile16(const Args16& p, OutT* Y, int64_t ldy, int64_t row_lo, int n0, uint8_t* lds,
                                       uint32_t* flags) {
  constexpr int WN = 8 / WM, NF = 2 * NC / WN, kRows = 64 * WM;
  const int64_t row_hi = row_lo + kRows < p.M ? row_lo + kRows : p.M;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave / WN, wn = wave % WN;
  const int panels = p.K / 128;

  Tile16<NC> t;
  const int arow = (tid >> 1) % kRows, arows = (int)(row_hi - row_lo);
  t.arow = (uint32_t)(arow < arows ? arow : arows - 1);
  t.half = (uint32_t)(tid & 1);
  constexpr int kPerRow = Tile16<NC>::kPerRow;
  const int lrow = tid / kPerRow, wrows = p.N - n0;
  t.wrow = (uint32_t)(lrow < wrows ? lrow : wrows - 1);
  t.wpart = (uint32_t)(tid % kPerRow);
  t.wactive = NC != 3 || wave < 6;
  t.aactive = WM == 4 || wave < 2 * WM;
  constexpr int kSc = FMT == kFmtNv ? 1 : 2;   // scale bytes per block in sps and ws
  t.dn = p.dnc + row_lo * 64;
  t.spc = p.spc + row_lo * (PAT == 0 ? 64 : 32);
  t.spm = PAT == 0 ? nullptr : p.spm + row_lo * 16;
  t.dns = p.dns + row_lo * 8;
  t.sps = p.sps + row_lo * (4 * kSc);
  t.wc = p.wc + (int64_t)n0 * 64;
  t.ws = p.ws + (int64_t)n0 * (4 * kSc);

  Put16 put;
  put.a0 = (uint32_t)(arow * 64 + 16 * ((2 * (tid & 1)) ^ swz_row(arow)));
  put.a1 = (uint32_t)(arow * 64 + 16 * ((2 * (tid & 1) + 1) ^ swz_row(arow)));
  const int wq = NC == 2 ? tid % 4 : 2 * (tid & 1);
  put.w0 = (uint32_t)(lrow * 64 + 16 * (wq ^ swz_row(lrow)));
  put.w1 = (uint32_t)(lrow * 64 + 16 * (((wq + 1) & 3) ^ swz_row(lrow)));

  // sub-step T: lane half h takes part 2 h + T of its row; fragments start at multiples of 32 rows
  const int col = lane & 31, half = lane >> 5;
  const uint32_t rd0 = (uint32_t)(col * 64 + 16 * ((2 * half) ^ swz_row(col)));
  const uint32_t rd1 = (uint32_t)(col * 64 + 16 * ((2 * half + 1) ^ swz_row(col)));
  const uint32_t rd_a = (uint32_t)(wm * 64 * 64), rd_w = (uint32_t)(wn * 32 * NF * 64);

  v16f acc[2][NF];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[r][f][e] = 0.0f;

  // Invariant at step s: stages s and s + 1 (mod 3) are filled; a0, b0 hold
  // step s's first operands; x (s even) or y holds the codes of step s + 2.
  Raw16 x, y;
  uint4 a0[2], b0[NF];
  uint8_t *st0 = lds, *st1 = lds + kStage16, *st2 = lds + 2 * kStage16;
  uint32_t *fg0 = flags, *fg1 = flags + 8, *fg2 = flags + 16;
  static_for<0, 6>([&](auto i) { load16<FMT, PAT, NC, 0>(x, t, 0, 0, decltype(i)::value); });
  static_for<0, 6>([&](auto i) { load16<FMT, PAT, NC, 1>(y, t, 0, 0, decltype(i)::value); });
  {
    Fill16<FMT, PAT, NC, 0> f0;
    Fill16<FMT, PAT, NC, 1> f1;
    static_for<0, 12>([&](auto i) { f0.template piece<decltype(i)::value>(x, st0, put, t, fg0, wave, lane); });
    static_for<0, 6>([&](auto i) { load16<FMT, PAT, NC, 2>(x, t, 0, 0, decltype(i)::value); });
    static_for<0, 12>([&](auto i) { f1.template piece<decltype(i)::value>(y, st1, put, t, fg1, wave, lane); });
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 2; ++r) a0[r] = lds16(st0 + rd_a + 2048 * r + rd0);
#pragma unroll
  for (int f = 0; f < NF; ++f) b0[f] = lds16(st0 + kPart16 + rd_w + 2048 * f + rd0);

  for (int k = 0; k < panels; ++k) {
    // the codes of the next panel's blocks; past the last panel it is reread and not used
    const int64_t k0 = k, k1 = k + 1 < panels ? k + 1 : panels - 1;
    const int64_t m0 = k0 * p.M, m1 = k1 * p.M, c0 = k0 * p.N, c1 = k1 * p.N;
#define SHARQ_STEP16(FB, LB, FROM, INTO, PM, PN)                                                                  \
  step16<FMT, PAT, NC, NF, FB>(acc, a0, b0, st0, st1, st2, rd0, rd1, rd_w, rd_a, fg0 + 2 * wm, fg2, FROM, put, t, wave, \
                           lane, [&](auto slot) {                                                                 \
                             constexpr int i = decltype(slot)::value;                                             \
                             if constexpr (i < 6) load16<FMT, PAT, NC, LB>(INTO, t, PM, PN, i);                   \
                           });                                                                                    \
  __syncthreads();                                                                                                \
  {                                                                                                               \
    uint8_t* s_ = st0;                                                                                            \
    st0 = st1;                                                                                                    \
    st1 = st2;                                                                                                    \
    st2 = s_;                                                                                                     \
    uint32_t* f_ = fg0;                                                                                           \
    fg0 = fg1;                                                                                                    \
    fg1 = fg2;                                                                                                    \
    fg2 = f_;                                                                                                     \
  }
    // step 4k + i fills block i + 2 and loads block i + 3 (of this panel or the next)
    SHARQ_STEP16(2, 3, x, y, m0, c0)
    SHARQ_STEP16(3, 0, y, x, m1, c1)
    SHARQ_STEP16(0, 1, x, y, m1, c1)
    SHARQ_STEP16(1, 2, y, x, m1, c1)
#undef SHARQ_STEP16
  }

  if constexpr (FMT == kFmtNv) {
    const float scale = *p.ts_x * *p.ts_w;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[r][f][e] *= scale;
  }
  // every wavefront is past its last LDS read: the stages are free
  uint8_t* epi = lds + wave * (32 * (64 * NF + 16));
#pragma unroll
  for (int r = 0; r < 2; ++r)
    il_epilogue<OutT, NF>(acc[r], Y, ldy, row_lo, row_hi, n0 + wn * 32 * NF, p.N, epi, 2 * wm + r, lane);
}

// At most one workgroup per CU walks the units b, b + G, ....  Units [0, full)
// are whole tiles, each XCD (id mod 8) taking a contiguous range of them; with
// 256 x 256 tiles the rest run as two half tiles of 128 columns each.
template <int FMT, int PAT, typename OutT, int NC, int WM>
__global__ __launch_bounds__(kT16) void k_linear16(Args16 p, OutT* Y, int64_t ldy, int gx, int gy, int full) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kLds16];
  __shared__ uint32_t flags[24];
  for (int id = (int)blockIdx.x; id < full; id += (int)gridDim.x) {
    int mt, nt;
    tile_in_groups(xcd_unit(id, full), gx, gy, mt, nt);
    tile16<FMT, PAT, OutT, NC, WM>(p, Y, ldy, (int64_t)mt * (64 * WM), nt * 64 * NC, lds, flags);
    __syncthreads();   // the LDS is free before the next tile's prologue
  }
  if constexpr (NC == 4 && WM == 4) {
    for (int u = (int)blockIdx.x; u < 2 * (gx * gy - full); u += (int)gridDim.x) {
      int mt, nt;
      tile_in_groups(full + (u >> 1), gx, gy, mt, nt);
      const int n0 = nt * 256 + 128 * (u & 1);
      if (n0 < p.N) tile16<FMT, PAT, OutT, 2, 4>(p, Y, ldy, (int64_t)mt * 256, n0, lds, flags);
      __syncthreads();
    }
  }
}

template <int FMT, int PAT, typename OutT>
static hipError_t go_linear16(const Args16& a, void* Y, int64_t ldy, hipStream_t st) {
  const Plan16 p = plan16(a.M, a.N, form16(FMT == kFmtNv, PAT), device_cus());
  OutT* y = reinterpret_cast<OutT*>(Y);
  const dim3 grid((unsigned)p.grid), block(kT16);
  const auto kernel = p.rows == 128 ? k_linear16<FMT, PAT, OutT, 4, 2>
                      : p.nf == 4   ? k_linear16<FMT, PAT, OutT, 4, 4>
                      : p.nf == 3   ? k_linear16<FMT, PAT, OutT, 3, 4>
                                    : k_linear16<FMT, PAT, OutT, 2, 4>;
  kernel<<<grid, block, 0, st>>>(a, y, ldy, p.gx, p.gy, p.full);
  return hipGetLastError();
}

template <int PAT, typename OutT>
static hipError_t go_nv(const uint8_t* spc, const uint8_t* spm, const uint8_t* sps, const uint8_t* dnc,
                        const uint8_t* dns, const float* tsx, int64_t M, const uint8_t* wc, const uint8_t* ws,
                        const float* tsw, int N, int K, void* Y, int64_t ldy, hipStream_t st) {
  if (K % kBK == 0)
    return go_linear16<kFmtNv, PAT, OutT>(Args16{spc, spm, sps, dnc, dns, wc, ws, tsx, tsw, M, N, K}, Y, ldy, st);
  if constexpr (PAT == 0) {
    return hipErrorInvalidValue;   // the dense backbone copy needs K a multiple of 128
  } else {
    constexpr int NF = 8;
    const int gx = (N + 32 * NF - 1) / (32 * NF), gy = (int)((M + kBM - 1) / kBM);
    k_linear_nv<NF, PAT, OutT><<<dim3((unsigned)(gx * gy)), dim3(256), 0, st>>>(
        spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, reinterpret_cast<OutT*>(Y), ldy, gx, gy);
    return hipGetLastError();
  }
}

template <int PAT>
static hipError_t go_nv_dt(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps, const uint8_t* dnc,
                           const uint8_t* dns, const float* tsx, int64_t M, const uint8_t* wc, const uint8_t* ws,
                           const float* tsw, int N, int K, void* Y, int64_t ldy, hipStream_t st) {
  if (ydt == 2) return go_nv<PAT, float>(spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
  if (ydt == 1) return go_nv<PAT, _Float16>(spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
  return go_nv<PAT, uint16_t>(spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
}

hipError_t launch_linear_nv(int pat, int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                            const uint8_t* dnc, const uint8_t* dns, const float* tsx, int64_t M, const uint8_t* wc,
                            const uint8_t* ws, const float* tsw, int N, int K, void* Y, int64_t ldy,
                            const uint8_t* spd, hipStream_t st) {
  const bool dense = spd && K % kBK == 0;
  if ((dense || spc != nullptr) && use_skinny16(M, N, K, form16(true, dense ? 0 : pat), device_cus()))
    return launch_linear_skinny16(true, dense ? 0 : pat, ydt, dense ? spd : spc, spm, sps, dnc, dns, tsx, M, wc, ws,
                                  tsw, N, K, Y, ldy, st);
  if (dense) return go_nv_dt<0>(ydt, spd, nullptr, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
  if (spc == nullptr) return hipErrorInvalidValue;   // rejected by the C ABI (K not a multiple of 128)
  return pat == 24 ? go_nv_dt<24>(ydt, spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st)
                   : go_nv_dt<48>(ydt, spc, spm, sps, dnc, dns, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
}

// HiF4 with K a multiple of 128.
hipError_t launch_linear16_hif4(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                                const uint8_t* dnc, const uint8_t* dns, int64_t M, const uint8_t* wc,
                                const uint8_t* ws, int N, int K, void* Y, int64_t ldy, hipStream_t st) {
  const Args16 a{spc, spm, sps, dnc, dns, wc, ws, nullptr, nullptr, M, N, K};
  if (ydt == 2) return go_linear16<kFmtHf, 24, float>(a, Y, ldy, st);
  if (ydt == 1) return go_linear16<kFmtHf, 24, _Float16>(a, Y, ldy, st);
  return go_linear16<kFmtHf, 24, uint16_t>(a, Y, ldy, st);
}

}  // namespace sharq
