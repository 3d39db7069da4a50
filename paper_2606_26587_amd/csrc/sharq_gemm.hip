// SharQ two-path FP4 GEMM for gfx950 (SharQ Sec. 3.3 eq. "sharq-output";
// Sec. 3.4 "Shared FP4 weights with path-specific scales" and "Residual path
// compensation by accumulation").
//
//   Y = dequant(backbone) * dequant(W)^T + dequant(residual) * dequant(W)^T
//
// Both products run on the CDNA4 block-scaled MFMA
// v_mfma_scale_f32_32x32x64_f8f6f4 with E2M1 operands and E8M0 scales, into
// ONE fp32 accumulator; Y is written once.
//
// gfx950 has no sparse MFMA for FP4 operands (the sparse smfmac forms take
// 8/16-bit inputs only), so the 2:4 or 4:8 backbone enters the MFMA as dense
// E2M1 nibbles with zeros at the dropped positions: either expanded from its
// compressed form in the registers of the wavefront that owns the rows (each
// wavefront owns 32 distinct rows of the 128-row tile, so a row is expanded
// once per tile and never goes through LDS), or read from the dense copy the
// preparation wrote (pattern 0), which spares every column tile the
// expansion.  The shared weight tile (E2M1 payload + E8M0 scales) is staged
// through LDS once per K step and read by both MFMAs of every fragment.
// Also here: the small-M kernel for decode, the grouped (MoE) forms, the HiF4
// kernel for larger M with K not a multiple of 128, and the generic kernels of
// the ablation path combinations.

// MFMA 32x32x64 FP4 operand layout (lane l, 64-wide wavefront): lane l holds
// row (l % 32) and the 32 K values of block (l / 32) of the 64-wide K slice as
// 32 nibbles in its first four dwords (lower K in the lower nibble); its
// 32-bit scale operand supplies, through op_sel, the E8M0 byte of that row and
// block.  Accumulator element r of lane l is output row
// 8 (r / 4) + 4 (l / 32) + (r % 4), column l % 32.

#include "sharq_tile.hpp"

namespace sharq {

constexpr int kLdsStride = 80;    // bytes per staged weight row (64 + 16 to spread LDS banks)

__device__ __forceinline__ v8i as_operand(uint4 q) {
  v8i v;
  v[0] = (int)q.x; v[1] = (int)q.y; v[2] = (int)q.z; v[3] = (int)q.w;
  v[4] = 0; v[5] = 0; v[6] = 0; v[7] = 0;
  return v;
}

// ---------------------------------------------------------------------------
// Per-lane activation fragment of one K step (two 64-wide MFMA sub-steps)
// ---------------------------------------------------------------------------

struct AStep {
  uint4 dn[2];       // residual codes, sub-step 0 / 1
  uint2 spc[2];      // compressed backbone codes
  uint32_t spm[2];   // backbone metadata
  uint32_t sdn, ssp; // E8M0 scales of the step's 4 blocks (byte j = block 4 ks + j)
  uint4 spd[2];      // the dense backbone codes instead (pattern 0: a dense copy was prepared)
};

template <bool SCALE_DW>
__device__ __forceinline__ void load_a(AStep& s, const ARow& a, int ks, int half, int nblk, int K) {
  // SCALE_DW: K is a multiple of 128, every panel is full and every block exists
  const int wp = SCALE_DW ? 128 : min(128, K - 128 * ks);
  const int64_t pr = (int64_t)ks * a.R;
  const uint8_t* dn = a.dn + pr * 64 + a.r * (wp / 2);
  const uint8_t* spc = a.spc + pr * 32 + a.r * (wp / 4);
  const uint8_t* spm = a.spm + pr * 16 + a.r * (wp / 8);
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int j = 2 * sub + half;   // block within the panel
    if (SCALE_DW || 4 * ks + j < nblk) {
      s.dn[sub] = *reinterpret_cast<const uint4*>(dn + 16 * j);
      s.spc[sub] = *reinterpret_cast<const uint2*>(spc + 8 * j);
      s.spm[sub] = *reinterpret_cast<const uint32_t*>(spm + 4 * j);
    } else {
      s.dn[sub] = make_uint4(0u, 0u, 0u, 0u);
      s.spc[sub] = make_uint2(0u, 0u);
      s.spm[sub] = 0x44444444u;   // 2:4: a valid (0,1) pair; 4:8 ignores it with zero codes
    }
  }
  const uint8_t* dns = a.dns + pr * 4 + a.r * (wp / 32);
  const uint8_t* sps = a.sps + pr * 4 + a.r * (wp / 32);
  if (SCALE_DW) {
    // raw dwords: the per-lane byte shift is applied at the point of use so
    // that no instruction waits on these loads before the MFMAs need them
    s.sdn = *reinterpret_cast<const uint32_t*>(dns);
    s.ssp = *reinterpret_cast<const uint32_t*>(sps);
  } else {
    // same byte order as the dword form: byte j = block 4 ks + j (127 past K)
    s.sdn = 0u;
    s.ssp = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool ok = 4 * ks + j < nblk;
      s.sdn |= (uint32_t)(ok ? dns[j] : 127u) << (8 * j);
      s.ssp |= (uint32_t)(ok ? sps[j] : 127u) << (8 * j);
    }
  }
}

// The weight tile of one K step held in registers between its global load and
// its LDS store: BN rows x 64 bytes of codes (16 bytes per thread and chunk)
// plus one dword of four E8M0 scales per row.
template <int NF>
struct WStep {
  uint4 q[NF / 2];
  uint32_t s;
};

template <int NF, bool SCALE_DW>
__device__ __forceinline__ void load_w(WStep<NF>& w, const uint8_t* wc, const uint8_t* ws, int n0, int N, int K,
                                       int ks, int nblk) {
  // panel-major weight: panel ks holds all N rows' 64 bytes (or fewer for a
  // narrow last panel), so a full tile of BN rows is one contiguous run
  constexpr int BN = 32 * NF;
  const int tid = threadIdx.x;
  const int wp = SCALE_DW ? 128 : min(128, K - 128 * ks);
  const int64_t pn = (int64_t)ks * N;
#pragma unroll
  for (int j = 0; j < BN / 64; ++j) {
    const int c = tid + 256 * j;
    const int row = c >> 2, part = c & 3;
    const int n = min(n0 + row, N - 1);
    w.q[j] = (SCALE_DW || 4 * ks + part < nblk)
                 ? *reinterpret_cast<const uint4*>(wc + pn * 64 + (int64_t)n * (wp / 2) + 16 * part)
                 : make_uint4(0u, 0u, 0u, 0u);
  }
  // one scale dword per weight row (threads 0 .. BN-1).  Threads past BN
  // reread row BN-1 and never store it: no branch, which keeps the
  // interleaved K step one basic block (the compiler would otherwise move its
  // MFMAs out of their slots), and no select on the loaded value, which
  // would make the thread wait for the load where it is issued
  const int n = min(n0 + (BN >= 256 ? tid : min(tid, BN - 1)), N - 1);
  const uint8_t* sr = ws + pn * 4 + (int64_t)n * (wp / 32);
  uint32_t sv = 0u;
  if (SCALE_DW) {
    sv = *reinterpret_cast<const uint32_t*>(sr);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) sv |= (uint32_t)(4 * ks + j < nblk ? sr[j] : 127u) << (8 * j);
  }
  w.s = sv;
}

// Weight scales in LDS are laid out per (column, lane half): lane (col, h)
// finds, at byte 2f + sub of its 2 NF-byte record, the E8M0 scale of weight row
// f*32 + col for block 4 ks + 2 sub + h -- exactly the byte its MFMA for
// fragment f, sub-step sub needs -- so one LDS read fetches all of them and
// op_sel selects the byte.
template <int NF>
__device__ __forceinline__ void store_w(const WStep<NF>& w, uint8_t* lds_w, uint8_t* lds_s) {
  constexpr int BN = 32 * NF;
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < BN / 64; ++j) {
    const int c = tid + 256 * j;
    const int row = c >> 2, part = c & 3;
    *reinterpret_cast<uint4*>(lds_w + row * kLdsStride + 16 * part) = w.q[j];
  }
  if (BN >= 256 || tid < BN) {
    const int f = tid >> 5, col = tid & 31;
    // blocks 0 and 2 of the step go to half 0, blocks 1 and 3 to half 1
    const uint32_t h0 = __builtin_amdgcn_perm(0u, w.s, 0x0c0c0200u);   // b0 | b2 << 8
    const uint32_t h1 = __builtin_amdgcn_perm(0u, w.s, 0x0c0c0301u);   // b1 | b3 << 8
    *reinterpret_cast<uint16_t*>(lds_s + (2 * col + 0) * (2 * NF) + 2 * f) = (uint16_t)h0;
    *reinterpret_cast<uint16_t*>(lds_s + (2 * col + 1) * (2 * NF) + 2 * f) = (uint16_t)h1;
  }
}

template <int SA, int SB>
__device__ __forceinline__ v16f mfma_fp4(v8i a, v8i b, v16f c, uint32_t sa, uint32_t sb) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 4, 4, SA, (int)sa, SB, (int)sb);
}

template <int SUB, int NF>
__device__ __forceinline__ void mma_sub(v16f (&acc)[NF], const uint8_t* lds_w, const uint32_t (&bw)[NF / 2],
                                        v8i a_sp, v8i a_dn, uint32_t ssp, uint32_t sdn, int lane) {
  const int half = lane >> 5, col = lane & 31;
  v8i b[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f)
    b[f] = as_operand(*reinterpret_cast<const uint4*>(lds_w + (f * 32 + col) * kLdsStride + 32 * SUB + 16 * half));
  // backbone products first, then the residual products into the same
  // accumulators: consecutive MFMAs never depend on each other.  The weight
  // scale of fragment f is byte 2 (f & 1) + SUB of word f / 2.
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    if (f & 1) acc[f] = mfma_fp4<2 * SUB, 2 + SUB>(a_sp, b[f], acc[f], ssp, bw[f >> 1]);
    else       acc[f] = mfma_fp4<2 * SUB, SUB>(a_sp, b[f], acc[f], ssp, bw[f >> 1]);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    if (f & 1) acc[f] = mfma_fp4<2 * SUB, 2 + SUB>(a_dn, b[f], acc[f], sdn, bw[f >> 1]);
    else       acc[f] = mfma_fp4<2 * SUB, SUB>(a_dn, b[f], acc[f], sdn, bw[f >> 1]);
  }
}

// One K step: expand the backbone of both sub-steps, then 2 x NF backbone and
// 2 x NF residual MFMAs against the staged weight tile.
template <int NF, int PAT>
__device__ __forceinline__ void step_mx(v16f (&acc)[NF], const AStep& cur, const uint8_t* lw, const uint8_t* ls,
                                        int lane) {
  static_assert(NF == 8 || NF == 4, "scale record is read as 16 or 8 bytes");
  const int half = lane >> 5, col = lane & 31;
  uint32_t bw[NF / 2];
  if (NF == 8) {
    const uint4 q = *reinterpret_cast<const uint4*>(ls + (2 * col + half) * (2 * NF));
    bw[0] = q.x; bw[1] = q.y; bw[NF / 2 > 2 ? 2 : 0] = q.z; bw[NF / 2 > 3 ? 3 : 0] = q.w;
  } else {
    const uint2 q = *reinterpret_cast<const uint2*>(ls + (2 * col + half) * (2 * NF));
    bw[0] = q.x; bw[NF / 2 > 1 ? 1 : 0] = q.y;
  }
  // op_sel 0 / 2 then picks block 4 ks + half (sub-step 0) / 4 ks + 2 + half (sub-step 1)
  const uint32_t ssp = cur.ssp >> (8 * half), sdn = cur.sdn >> (8 * half);
  {
    const v8i a_sp = as_operand(expand_block<PAT>(cur.spc[0], cur.spm[0]));
    mma_sub<0, NF>(acc, lw, bw, a_sp, as_operand(cur.dn[0]), ssp, sdn, lane);
  }
  {
    const v8i a_sp = as_operand(expand_block<PAT>(cur.spc[1], cur.spm[1]));
    mma_sub<1, NF>(acc, lw, bw, a_sp, as_operand(cur.dn[1]), ssp, sdn, lane);
  }
}

// One 128 x (32 NF) output tile.  Rows of the tile are output rows
// [row_lo, row_lo + 128) clipped at row_hi; the activation row of output row
// i is row_index[i] when row_index is given, else i - out_base + act_base.
template <int NF, int PAT, bool SCALE_DW, typename OutT>
__device__ __forceinline__ void tile_mx(const uint8_t* sp_codes, const uint8_t* sp_meta, const uint8_t* sp_scale,
                                        const uint8_t* dn_codes, const uint8_t* dn_scale, const int32_t* row_index,
                                        int64_t act_rows, int64_t row_lo, int64_t row_hi, const uint8_t* wc,
                                        const uint8_t* ws, int n0,
                                        int N, int K, OutT* Y, int64_t ldy, uint8_t* lds_w, uint8_t* lds_s) {
  constexpr int BN = 32 * NF;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  const int nblk = K / 32, nks = (K + kBK - 1) / kBK;

  int64_t orow = row_lo + wave * 32 + (lane & 31);
  if (orow >= row_hi) orow = row_hi - 1;   // clamp: loads stay in bounds, stores are masked
  ARow a;
  a.r = row_index ? (int64_t)row_index[orow] : orow;
  a.R = act_rows;
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

  // Software pipeline over K steps, unrolled by two so that the two
  // activation register sets alternate by position instead of being copied.
  // Step ks computes from LDS buffer ks & 1 and register set ks & 1; after
  // its MFMAs the weight tile of step ks+1 (loaded one step earlier) goes to
  // the other LDS buffer and the loads of step ks+2 are issued, so every
  // global load has one full step of MFMA work to arrive.  Loads past the
  // last step re-read the last step (clamped) and are never used.
  AStep a0, a1;
  WStep<NF> wn;
  const int last = nks - 1;
  load_w<NF, SCALE_DW>(wn, wc, ws, n0, N, K, 0, nblk);
  load_a<SCALE_DW>(a0, a, 0, half, nblk, K);
  store_w<NF>(wn, lds_w, lds_s);
  load_w<NF, SCALE_DW>(wn, wc, ws, n0, N, K, min(1, last), nblk);
  load_a<SCALE_DW>(a1, a, min(1, last), half, nblk, K);
  // The scheduling fences keep each phase in place: without them the
  // compiler hoists ALU work on freshly issued loads into the preceding MFMA
  // phase, which then has to wait for those loads.
  constexpr int SREC = 64 * 2 * NF;   // bytes of one buffer's scale records
  int ks = 0;
  for (; ks + 1 < nks; ks += 2) {   // one exit: the accumulators stay in place
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    step_mx<NF, PAT>(acc, a0, lds_w, lds_s, lane);
    __builtin_amdgcn_sched_barrier(0);
    store_w<NF>(wn, lds_w + BN * kLdsStride, lds_s + SREC);
    load_w<NF, SCALE_DW>(wn, wc, ws, n0, N, K, min(ks + 2, last), nblk);
    load_a<SCALE_DW>(a0, a, min(ks + 2, last), half, nblk, K);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    step_mx<NF, PAT>(acc, a1, lds_w + BN * kLdsStride, lds_s + SREC, lane);
    __builtin_amdgcn_sched_barrier(0);
    store_w<NF>(wn, lds_w, lds_s);
    load_w<NF, SCALE_DW>(wn, wc, ws, n0, N, K, min(ks + 3, last), nblk);
    load_a<SCALE_DW>(a1, a, min(ks + 3, last), half, nblk, K);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (ks < nks) {   // odd number of steps: the last one is in buffer 0 / set 0
    __syncthreads();
    step_mx<NF, PAT>(acc, a0, lds_w, lds_s, lane);
  }

#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int col = n0 + f * 32 + (lane & 31);
    if (col >= N) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = row_lo + wave * 32 + 8 * (r / 4) + 4 * half + (r % 4);
      if (row < row_hi) store_out<OutT>(Y + row * ldy + col, acc[f][r]);
    }
  }
}

// ---------------------------------------------------------------------------
// Interleaved main loop (full 128-wide panels, 256 output columns)
// ---------------------------------------------------------------------------
//
// With one wavefront per SIMD the matrix core idles whenever the wavefront
// issues anything but MFMAs, unless that work sits between MFMAs it does not
// feed and is short enough (a wave64 VALU instruction takes 4 cycles, one
// FP4 32x32x64 MFMA 32) to finish before the next MFMA may issue.  Each K step
// therefore runs its 32 MFMAs as fixed slots and spreads the preparation of
// later steps thinly between them: the weight reads of its second sub-step,
// the expansion of the next step's backbone (one 16-bit piece, ~8 VALU, per
// slot), the copy of its residual operand, the LDS store of the weight tile
// two steps ahead and the reads of the next step's first weight operands.
// The weight tile goes through three LDS stages, so the tile of step k+1 is
// published one barrier before step k ends and its first operands are already
// in registers when step k+1 begins.  The global loads of later steps (the
// weights three steps ahead, the activations two steps ahead) go out in six
// parts behind the first six MFMAs rather than as one block before the first:
// measured on the Llama prefill shapes, a block of ~10 loads and their
// address arithmetic ahead of every step left the matrix core idle, and
// spreading them took the three GEMMs from ~450 to ~420-430 us.
// Scheduling fences keep every slot in place.

struct AOps {        // MFMA-ready activation operands of one K step
  uint4 sp[2], dn[2];
  uint32_t ssp, sdn; // E8M0 scale dwords shifted to this lane's half
};

constexpr int kStageW = 256 * kLdsStride;        // weight codes of one stage
constexpr int kStageBytes = kStageW + 64 * 16;   // + the 64 scale records

// 4:8 expansion through a table.  For a keep mask m, entry m holds two
// v_perm selectors: byte i of the first picks the code for position 2 i (its
// index among the kept codes, or 0x0C = zero if position 2 i is dropped), the
// second the code for position 2 i + 1.  The group's four codes are spread to
// bytes, permuted twice (once shifted into the high nibbles) and OR-ed.
__device__ __forceinline__ uint2 lut48_entry(uint32_t m) {
  uint32_t se = 0u, so = 0u, idx = 0u;
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    uint32_t sel = 0x0Cu;
    if ((m >> p) & 1u) sel = idx++;
    if (p & 1) so |= sel << (8 * (p >> 1));
    else se |= sel << (8 * (p >> 1));
  }
  return make_uint2(se, so);
}

__device__ __forceinline__ uint32_t expand48_lut(uint32_t c16, uint2 sel) {
  uint32_t x = (c16 | (c16 << 8)) & 0x00FF00FFu;   // bytes 0, 2: code pairs (0, 1), (2, 3)
  x = (x | (x << 4)) & 0x0F0F0F0Fu;                 // byte i: code i
  return __builtin_amdgcn_perm(0u, x, sel.x) | __builtin_amdgcn_perm(0u, x << 4, sel.y);
}

// Fill a workgroup's 256-entry table (one entry per thread); the caller
// synchronizes before the first use.
__device__ __forceinline__ void lut48_fill(uint2* lut) {
  if (threadIdx.x < 256) lut[threadIdx.x] = lut48_entry(threadIdx.x);
}

// Piece Q (0..15) of the next step's expanded backbone: block Q / 8, output
// dword (Q % 8) / 2, 16-bit half Q % 2 (returned in place within the dword).
template <int PAT, int Q>
__device__ __forceinline__ uint32_t exp_piece(const AStep& r) {
  constexpr int B = Q / 8, D = (Q % 8) / 2, H = Q % 2;
  const uint2 c = r.spc[B];
  const uint32_t meta = r.spm[B];
  if (PAT == 24) {
    constexpr int G = 2 * D + H;   // group of 4 positions
    const uint32_t cw = G < 4 ? c.x : c.y;
    const uint32_t byte = (cw >> (8 * (G & 3))) & 0xFFu;
    const uint32_t nib = (meta >> (4 * G)) & 0xFu;
    return ((byte & 0xFu) << (4 * (nib & 3u) + 16 * H)) | ((byte >> 4) << (4 * (nib >> 2) + 16 * H));
  } else {
    constexpr int G = D;           // group of 8 positions, half H of it
    const uint32_t cw = G < 2 ? c.x : c.y;
    uint32_t c16 = (cw >> (16 * (G & 1))) & 0xFFFFu;
    const uint32_t mask = (meta >> (8 * G)) & 0xFFu;
    if (H == 1) c16 >>= 4 * __builtin_popcount(mask & 0xFu);
    uint32_t out = 0u;
#pragma unroll
    for (int p = 4 * H; p < 4 * H + 4; ++p) {
      if ((mask >> p) & 1u) {
        out |= (c16 & 0xFu) << (4 * p);
        c16 >>= 4;
      }
    }
    return out;
  }
}

template <int PAT, int Q>
__device__ __forceinline__ void put_piece(AOps& o, const AStep& r, const uint2 (&sel)[8]) {
  if (PAT == 0) return;   // the backbone arrives dense
  constexpr int B = Q / 8, D = (Q % 8) / 2, H = Q % 2;
  uint32_t& d = D == 0 ? o.sp[B].x : D == 1 ? o.sp[B].y : D == 2 ? o.sp[B].z : o.sp[B].w;
  if (PAT == 48) {
    // a whole group (output dword) per even piece, from its table entry
    if (H == 0) {
      const uint32_t cw = D < 2 ? r.spc[B].x : r.spc[B].y;
      d = expand48_lut((cw >> (16 * (D & 1))) & 0xFFFFu, sel[4 * B + D]);
    }
  } else {
    const uint32_t v = exp_piece<PAT, Q>(r);
    d = H == 0 ? v : (d | v);
  }
}

// The weight is the MFMA's first operand and the activation its second, so
// the accumulator is the transposed tile: lane l holds activation row
// l % 32 and, in element r, output column 8 (r / 4) + 4 (l / 32) + r % 4 of
// the fragment -- four consecutive columns per group of four elements.
template <int SUB, int F, int NF>
__device__ __forceinline__ void mma_sp(v16f (&acc)[NF], const AOps& a, const uint4 (&b)[NF],
                                       const uint32_t (&bw)[NF / 2]) {
  acc[F] = mfma_fp4<(F & 1) ? 2 + SUB : SUB, SUB>(as_operand(b[F]), as_operand(a.sp[SUB]), acc[F], bw[F >> 1],
                                                 a.ssp);
}

template <int SUB, int F, int NF>
__device__ __forceinline__ void mma_dn(v16f (&acc)[NF], const AOps& a, const uint4 (&b)[NF],
                                       const uint32_t (&bw)[NF / 2]) {
  acc[F] = mfma_fp4<(F & 1) ? 2 + SUB : SUB, SUB>(as_operand(b[F]), as_operand(a.dn[SUB]), acc[F], bw[F >> 1],
                                                 a.sdn);
}

template <int SUB, int F0, int F1, int NB>
__device__ __forceinline__ void read_b(uint4 (&b)[NB], const uint8_t* lw, int lane) {
  const int half = lane >> 5, col = lane & 31;
#pragma unroll
  for (int f = F0; f < F1; ++f)
    b[f] = *reinterpret_cast<const uint4*>(lw + (f * 32 + col) * kLdsStride + 32 * half + 16 * SUB);
}

__device__ __forceinline__ void read_bw(uint32_t (&bw)[4], const uint8_t* stage, int lane) {
  const int half = lane >> 5, col = lane & 31;
  const uint4 q = *reinterpret_cast<const uint4*>(stage + kStageW + (2 * col + half) * 16);
  bw[0] = q.x; bw[1] = q.y; bw[2] = q.z; bw[3] = q.w;
}

// half tiles (fragments 0-3): the first 8 bytes of the record
__device__ __forceinline__ void read_bw(uint32_t (&bw)[2], const uint8_t* stage, int lane) {
  const int half = lane >> 5, col = lane & 31;
  const uint2 q = *reinterpret_cast<const uint2*>(stage + kStageW + (2 * col + half) * 16);
  bw[0] = q.x; bw[1] = q.y;
}

// One K step k.  In: b0 / bw = sub-step 0 weight operands and scale records
// of step k (read from stage `cur`); ops = expanded activations of step k.
// Out: b0 / bwn = those of step k+1 (from stage `nxt`); opsn.sp and scales =
// expansion of raw (step k+1; its residual codes are loaded into opsn.dn by
// `issue`); wst (step k+2) stored to stage `wr`.  issue(part) issues part
// 0-5 of the step's global loads (a std::integral_constant argument).
// SPR = 0: the six parts go out behind the first six MFMAs; SPR = 1: spread
// over the whole step, two slots of each group of eight apart (the schedule of
// the row-gathering grouped GEMM, whose scattered activation rows make each
// load slower to issue; for contiguous rows the burst is faster).
template <int PAT, int SPR = 0, class Issue>
__device__ __forceinline__ void step5(v16f (&acc)[8], const AOps& ops, uint4 (&b0)[8], const uint32_t (&bw)[4],
                                      uint32_t (&bwn)[4], const uint8_t* cur, const uint8_t* nxt, uint8_t* wr,
                                      AOps& opsn, const AStep& raw, const WStep<8>& wst, int lane, Issue issue,
                                      const uint2* lut) {
  const int half = lane >> 5, tid = threadIdx.x;
  uint4 b1[8];
  uint2 sel[8];
  if (PAT == 48) {   // table entries of the next step's eight 4:8 groups
#pragma unroll
    for (int i = 0; i < 8; ++i) sel[i] = lut[(raw.spm[i >> 2] >> (8 * (i & 3))) & 0xFFu];
  }
  // LDS traffic is spread at about one instruction per slot (a 1 KB
  // wavefront access keeps the LDS busy for several MFMA-lengths when four
  // wavefronts burst together); VALU work stays under ~8 instructions per slot.
  // ---- sub-step 0, backbone: second sub-step's weight operands; the
  // global loads of later steps go out in six parts behind the first MFMAs
  mma_sp<0, 0>(acc, ops, b0, bw); issue(std::integral_constant<int, 0>()); read_b<1, 0, 1>(b1, cur, lane);
  put_piece<PAT, 0>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 1>(acc, ops, b0, bw);
  if constexpr (SPR == 0) issue(std::integral_constant<int, 1>());
  read_b<1, 1, 2>(b1, cur, lane);
  SHARQ_FENCE();
  mma_sp<0, 2>(acc, ops, b0, bw);
  if constexpr (SPR == 0) issue(std::integral_constant<int, 2>());
  read_b<1, 2, 3>(b1, cur, lane);
  put_piece<PAT, 1>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 3>(acc, ops, b0, bw);
  if constexpr (SPR == 0) issue(std::integral_constant<int, 3>());
  read_b<1, 3, 4>(b1, cur, lane);
  SHARQ_FENCE();
  mma_sp<0, 4>(acc, ops, b0, bw);
  if constexpr (SPR == 0) issue(std::integral_constant<int, 4>());
  read_b<1, 4, 5>(b1, cur, lane);
  put_piece<PAT, 2>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 5>(acc, ops, b0, bw);
  if constexpr (SPR == 0) issue(std::integral_constant<int, 5>());
  else issue(std::integral_constant<int, 1>());
  read_b<1, 5, 6>(b1, cur, lane);
  SHARQ_FENCE();
  mma_sp<0, 6>(acc, ops, b0, bw); read_b<1, 6, 7>(b1, cur, lane); put_piece<PAT, 3>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 7>(acc, ops, b0, bw); read_b<1, 7, 8>(b1, cur, lane); SHARQ_FENCE();
  // ---- sub-step 0, residual: the weight tile two steps ahead to LDS
  mma_dn<0, 0>(acc, ops, b0, bw); put_piece<PAT, 4>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<0, 1>(acc, ops, b0, bw);
  *reinterpret_cast<uint4*>(wr + (tid >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[0];
  SHARQ_FENCE();
  mma_dn<0, 2>(acc, ops, b0, bw); put_piece<PAT, 5>(opsn, raw, sel);
  if constexpr (SPR == 1) issue(std::integral_constant<int, 2>());
  SHARQ_FENCE();
  mma_dn<0, 3>(acc, ops, b0, bw);
  *reinterpret_cast<uint4*>(wr + ((tid + 256) >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[1];
  SHARQ_FENCE();
  mma_dn<0, 4>(acc, ops, b0, bw); put_piece<PAT, 6>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<0, 5>(acc, ops, b0, bw);
  *reinterpret_cast<uint4*>(wr + ((tid + 512) >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[2];
  SHARQ_FENCE();
  mma_dn<0, 6>(acc, ops, b0, bw); put_piece<PAT, 7>(opsn, raw, sel);
  if constexpr (SPR == 1) issue(std::integral_constant<int, 3>());
  SHARQ_FENCE();
  mma_dn<0, 7>(acc, ops, b0, bw);
  *reinterpret_cast<uint4*>(wr + ((tid + 768) >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[3];
  SHARQ_FENCE();
  // ---- sub-step 1, backbone: weight scales, then the next step's operands
  mma_sp<1, 0>(acc, ops, b1, bw); put_piece<PAT, 8>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<1, 1>(acc, ops, b1, bw);
  {
    const int f = tid >> 5, c = tid & 31;
    // record (c, h) byte 2 (f & 1) + sub <- block 2 h + sub of weight row 32 f + c
    *reinterpret_cast<uint16_t*>(wr + kStageW + (2 * c + 0) * 16 + 2 * f) = (uint16_t)wst.s;
    *reinterpret_cast<uint16_t*>(wr + kStageW + (2 * c + 1) * 16 + 2 * f) = (uint16_t)(wst.s >> 16);
  }
  SHARQ_FENCE();
  mma_sp<1, 2>(acc, ops, b1, bw); put_piece<PAT, 9>(opsn, raw, sel);
  if constexpr (SPR == 1) issue(std::integral_constant<int, 4>());
  SHARQ_FENCE();
  mma_sp<1, 3>(acc, ops, b1, bw); read_b<0, 0, 1>(b0, nxt, lane); SHARQ_FENCE();
  mma_sp<1, 4>(acc, ops, b1, bw); put_piece<PAT, 10>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<1, 5>(acc, ops, b1, bw); read_b<0, 1, 2>(b0, nxt, lane); SHARQ_FENCE();
  mma_sp<1, 6>(acc, ops, b1, bw); put_piece<PAT, 11>(opsn, raw, sel);
  if constexpr (SPR == 1) issue(std::integral_constant<int, 5>());
  SHARQ_FENCE();
  mma_sp<1, 7>(acc, ops, b1, bw); read_b<0, 2, 3>(b0, nxt, lane); SHARQ_FENCE();
  // ---- sub-step 1, residual
  mma_dn<1, 0>(acc, ops, b1, bw); put_piece<PAT, 12>(opsn, raw, sel); read_b<0, 3, 4>(b0, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 1>(acc, ops, b1, bw); read_b<0, 4, 5>(b0, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 2>(acc, ops, b1, bw); put_piece<PAT, 13>(opsn, raw, sel); read_b<0, 5, 6>(b0, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 3>(acc, ops, b1, bw); read_b<0, 6, 7>(b0, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 4>(acc, ops, b1, bw); put_piece<PAT, 14>(opsn, raw, sel); read_b<0, 7, 8>(b0, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 5>(acc, ops, b1, bw); read_bw(bwn, nxt, lane); SHARQ_FENCE();
  mma_dn<1, 6>(acc, ops, b1, bw); put_piece<PAT, 15>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<1, 7>(acc, ops, b1, bw);
  opsn.ssp = raw.ssp >> (16 * half);
  opsn.sdn = raw.sdn >> (16 * half);
  if (PAT == 0) {
    opsn.sp[0] = raw.spd[0];
    opsn.sp[1] = raw.spd[1];
  }
  SHARQ_FENCE();
}

// The same K step for a half tile (128 output columns, fragments 0-3): 16
// MFMA slots.  The weight stage keeps the full tile's layout with rows 0-127
// (and bytes 0-7 of each scale record) filled, so the operand reads are the
// full tile's; the extra work per slot is about twice as dense.
template <int PAT, class Issue>
__device__ __forceinline__ void step5h(v16f (&acc)[4], const AOps& ops, uint4 (&b0)[4], const uint32_t (&bw)[2],
                                       uint32_t (&bwn)[2], const uint8_t* cur, const uint8_t* nxt, uint8_t* wr,
                                       AOps& opsn, const AStep& raw, const WStep<4>& wst, int lane, Issue issue,
                                       const uint2* lut) {
  const int half = lane >> 5, tid = threadIdx.x;
  uint4 b1[4];
  uint2 sel[8];
  if (PAT == 48) {
#pragma unroll
    for (int i = 0; i < 8; ++i) sel[i] = lut[(raw.spm[i >> 2] >> (8 * (i & 3))) & 0xFFu];
  }
  // ---- sub-step 0: the second sub-step's weight operands and the global
  // loads of later steps, then the weight tile two steps ahead to LDS
  mma_sp<0, 0>(acc, ops, b0, bw); issue(std::integral_constant<int, 0>()); read_b<1, 0, 1>(b1, cur, lane);
  put_piece<PAT, 0>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 1>(acc, ops, b0, bw); issue(std::integral_constant<int, 1>()); read_b<1, 1, 2>(b1, cur, lane);
  put_piece<PAT, 1>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 2>(acc, ops, b0, bw); issue(std::integral_constant<int, 2>()); read_b<1, 2, 3>(b1, cur, lane);
  put_piece<PAT, 2>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<0, 3>(acc, ops, b0, bw); issue(std::integral_constant<int, 3>()); read_b<1, 3, 4>(b1, cur, lane);
  put_piece<PAT, 3>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<0, 0>(acc, ops, b0, bw); issue(std::integral_constant<int, 4>()); put_piece<PAT, 4>(opsn, raw, sel);
  *reinterpret_cast<uint4*>(wr + (tid >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[0];
  SHARQ_FENCE();
  mma_dn<0, 1>(acc, ops, b0, bw); issue(std::integral_constant<int, 5>()); put_piece<PAT, 5>(opsn, raw, sel);
  *reinterpret_cast<uint4*>(wr + ((tid + 256) >> 2) * kLdsStride + 16 * (tid & 3)) = wst.q[1];
  SHARQ_FENCE();
  mma_dn<0, 2>(acc, ops, b0, bw); put_piece<PAT, 6>(opsn, raw, sel);
  {
    // threads 128-255 hold a copy of column 127's scales and write bytes 8-15
    // of the records, which a half tile never reads: no branch, so the step
    // stays one basic block and the compiler keeps every MFMA in its slot
    const int f = tid >> 5, c = tid & 31;
    *reinterpret_cast<uint16_t*>(wr + kStageW + (2 * c + 0) * 16 + 2 * f) = (uint16_t)wst.s;
    *reinterpret_cast<uint16_t*>(wr + kStageW + (2 * c + 1) * 16 + 2 * f) = (uint16_t)(wst.s >> 16);
  }
  SHARQ_FENCE();
  mma_dn<0, 3>(acc, ops, b0, bw); put_piece<PAT, 7>(opsn, raw, sel); SHARQ_FENCE();
  // ---- sub-step 1: the next step's first operands and scale records
  mma_sp<1, 0>(acc, ops, b1, bw); put_piece<PAT, 8>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<1, 1>(acc, ops, b1, bw); read_b<0, 0, 1>(b0, nxt, lane); put_piece<PAT, 9>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<1, 2>(acc, ops, b1, bw); read_b<0, 1, 2>(b0, nxt, lane); put_piece<PAT, 10>(opsn, raw, sel); SHARQ_FENCE();
  mma_sp<1, 3>(acc, ops, b1, bw); read_b<0, 2, 3>(b0, nxt, lane); put_piece<PAT, 11>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<1, 0>(acc, ops, b1, bw); read_b<0, 3, 4>(b0, nxt, lane); put_piece<PAT, 12>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<1, 1>(acc, ops, b1, bw); read_bw(bwn, nxt, lane); put_piece<PAT, 13>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<1, 2>(acc, ops, b1, bw); put_piece<PAT, 14>(opsn, raw, sel); SHARQ_FENCE();
  mma_dn<1, 3>(acc, ops, b1, bw); put_piece<PAT, 15>(opsn, raw, sel);
  opsn.ssp = raw.ssp >> (16 * half);
  opsn.sdn = raw.sdn >> (16 * half);
  if (PAT == 0) {
    opsn.sp[0] = raw.spd[0];
    opsn.sp[1] = raw.spd[1];
  }
  SHARQ_FENCE();
}

// Residual codes of step ks straight into the operand registers, and the
// backbone codes / metadata / scales of step ks into a raw set (panel-major,
// K a multiple of 128).
// In this loop lane half h takes blocks 2h and 2h+1 of each 128-position
// step (sub-step s uses block 2h + s), so a lane's bytes of every buffer are
// contiguous: 32 bytes of residual codes, 16 of backbone codes, 8 of metadata.
__device__ __forceinline__ void load_a_dn(AOps& o, const ARow& a, int ks, int half) {
  const uint8_t* dn = a.dn + (int64_t)ks * a.R * 64 + a.r * 64 + 32 * half;
  o.dn[0] = *reinterpret_cast<const uint4*>(dn);
  o.dn[1] = *reinterpret_cast<const uint4*>(dn + 16);
}

// PAT 0: a.spc is the dense backbone copy, laid out like the residual codes.
template <int PAT>
__device__ __forceinline__ void load_a_meta(AStep& s, const ARow& a, int ks, int half) {
  const int64_t pr = (int64_t)ks * a.R;
  if (PAT == 0) {
    const uint8_t* sp = a.spc + pr * 64 + a.r * 64 + 32 * half;
    s.spd[0] = *reinterpret_cast<const uint4*>(sp);
    s.spd[1] = *reinterpret_cast<const uint4*>(sp + 16);
  } else {
    const uint4 c = *reinterpret_cast<const uint4*>(a.spc + pr * 32 + a.r * 32 + 16 * half);
    const uint2 m = *reinterpret_cast<const uint2*>(a.spm + pr * 16 + a.r * 16 + 8 * half);
    s.spc[0] = make_uint2(c.x, c.y);
    s.spc[1] = make_uint2(c.z, c.w);
    s.spm[0] = m.x;
    s.spm[1] = m.y;
  }
  s.sdn = *reinterpret_cast<const uint32_t*>(a.dns + pr * 4 + a.r * 4);
  s.ssp = *reinterpret_cast<const uint32_t*>(a.sps + pr * 4 + a.r * 4);
}

// Parts of one K step's global loads (K a multiple of 128), so that the
// interleaved loop can spread them over its MFMA slots: the backbone codes
// (or the dense copy) and the two scale dwords of the activations; two halves
// of the weight codes and the weight scales (load_w's bytes, in parts).
template <int PAT, int P>
__device__ __forceinline__ void load_a_meta_part(AStep& s, const ARow& a, int ks, int half) {
  const int64_t pr = (int64_t)ks * a.R;
  if constexpr (P == 0) {
    if (PAT == 0) {
      const uint8_t* sp = a.spc + pr * 64 + a.r * 64 + 32 * half;
      s.spd[0] = *reinterpret_cast<const uint4*>(sp);
      s.spd[1] = *reinterpret_cast<const uint4*>(sp + 16);
    } else {
      const uint4 c = *reinterpret_cast<const uint4*>(a.spc + pr * 32 + a.r * 32 + 16 * half);
      const uint2 m = *reinterpret_cast<const uint2*>(a.spm + pr * 16 + a.r * 16 + 8 * half);
      s.spc[0] = make_uint2(c.x, c.y);
      s.spc[1] = make_uint2(c.z, c.w);
      s.spm[0] = m.x;
      s.spm[1] = m.y;
    }
  } else {
    s.sdn = *reinterpret_cast<const uint32_t*>(a.dns + pr * 4 + a.r * 4);
    s.ssp = *reinterpret_cast<const uint32_t*>(a.sps + pr * 4 + a.r * 4);
  }
}

template <int NF, int P>
__device__ __forceinline__ void load_w_part(WStep<NF>& w, const uint8_t* wc, const uint8_t* ws, int n0, int N,
                                            int ks) {
  constexpr int BN = 32 * NF;
  const int tid = threadIdx.x;
  const int64_t pn = (int64_t)ks * N;
  if constexpr (P < 2) {
#pragma unroll
    for (int j = P * NF / 4; j < (P + 1) * NF / 4; ++j) {
      const int c = tid + 256 * j;
      const int row = c >> 2, part = c & 3;
      const int n = min(n0 + row, N - 1);
      w.q[j] = *reinterpret_cast<const uint4*>(wc + pn * 64 + (int64_t)n * 64 + 16 * part);
    }
  } else {
    // In a half tile threads BN..255 load column BN - 1's scales again: their
    // copy lands in record bytes that a half tile never reads.  Selecting 0
    // for them instead would make the value depend on the load at issue time,
    // and the wait for it (the newest load) drained every load in flight once
    // per step: 57.5 -> 53.5 us on the Llama qkv shape, whose last round runs
    // as half tiles.
    const int n = min(n0 + (BN >= 256 ? tid : min(tid, BN - 1)), N - 1);
    w.s = *reinterpret_cast<const uint32_t*>(ws + pn * 4 + (int64_t)n * 4);
  }
}

template <int NF>
__device__ __forceinline__ void store_w_stage(const WStep<NF>& w, uint8_t* stage) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < NF / 2; ++j) {
    const int c = tid + 256 * j;
    *reinterpret_cast<uint4*>(stage + (c >> 2) * kLdsStride + 16 * (c & 3)) = w.q[j];
  }
  if (NF == 8 || tid < 32 * NF) {
    const int f = tid >> 5, c = tid & 31;
    *reinterpret_cast<uint16_t*>(stage + kStageW + (2 * c + 0) * 16 + 2 * f) = (uint16_t)w.s;
    *reinterpret_cast<uint16_t*>(stage + kStageW + (2 * c + 1) * 16 + 2 * f) = (uint16_t)(w.s >> 16);
  }
}

constexpr int kTileLds = 4 * kEpiWave > 3 * kStageBytes ? 4 * kEpiWave : 3 * kStageBytes;
constexpr int kPersistLds = 3 * kStageBytes + 4 * kEpiWave;   // stages and epilogue apart: 129 KB

// One K step of a full (NF = 8) or half (NF = 4) tile; SPR: the load
// schedule of step5.
template <int PAT, int SPR = 0, int NF, class Issue>
__device__ __forceinline__ void step_il(v16f (&acc)[NF], const AOps& ops, uint4 (&b0)[NF],
                                        const uint32_t (&bw)[NF / 2], uint32_t (&bwn)[NF / 2], const uint8_t* cur,
                                        const uint8_t* nxt, uint8_t* wr, AOps& opsn, const AStep& raw,
                                        const WStep<NF>& wst, int lane, Issue issue, const uint2* lut) {
  if constexpr (NF == 8)
    step5<PAT, SPR>(acc, ops, b0, bw, bwn, cur, nxt, wr, opsn, raw, wst, lane, issue, lut);
  else
    step5h<PAT>(acc, ops, b0, bw, bwn, cur, nxt, wr, opsn, raw, wst, lane, issue, lut);
}

// The register sets of the interleaved pipeline.  They rotate with period
// three, so the main loop is unrolled by three and the LDS stages are fixed
// per unrolled step.  Invariant at the start of step k (sets indexed by
// k mod 3): stages k, k+1 hold W(k), W(k+1); b0 / bw hold step k's first
// weight operands; o[k] is complete; o[k+1].dn = residual codes of step k+1
// (in flight); r[k+1], r[k+2] = raw backbone data of steps k+1, k+2; w[k+2],
// w[k] = raw W(k+2), W(k+3).  Step k loads the residual codes of step k+2, the
// raw backbone of step k+3 and W(k+4): every load has two full steps to
// arrive.  Loads past the last step re-read it (clamped) and their results
// are never used.
template <int NF>
struct IlSets {
  AStep r0, r1, r2;
  WStep<NF> w0, w1, w2;
  AOps o0, o1, o2;
};

// A tile's first global loads: W(0..2), the residual codes of steps 0 and 1,
// the raw backbone of steps 0..2.  They touch no LDS, so a persistent loop can
// issue them for its next tile before the current tile's output stores.
template <int PAT, int NF>
__device__ __forceinline__ void il_issue(IlSets<NF>& p, const ARow& a, const uint8_t* wc, const uint8_t* ws,
                                         int n0, int N, int K, int half) {
  const int nblk = K / 32, last = K / kBK - 1;
  const auto cl = [&](int k) { return k < last ? k : last; };
  load_w<NF, true>(p.w0, wc, ws, n0, N, K, 0, nblk);
  load_a_meta<PAT>(p.r0, a, 0, half);
  load_a_dn(p.o0, a, 0, half);
  load_w<NF, true>(p.w1, wc, ws, n0, N, K, cl(1), nblk);
  load_a_dn(p.o1, a, cl(1), half);
  load_a_meta<PAT>(p.r1, a, cl(1), half);
  load_a_meta<PAT>(p.r2, a, cl(2), half);
  load_w<NF, true>(p.w2, wc, ws, n0, N, K, cl(2), nblk);
}

// The rest of a tile's prologue: W(0), W(1) into stages 0 and 1, step 0's
// backbone operands, the load of W(3), and step 0's first weight operands.
// The stages must be free (a barrier after the previous tile's last step).
template <int PAT, int NF>
__device__ __forceinline__ void il_start(IlSets<NF>& p, const uint8_t* wc, const uint8_t* ws, int n0, int N,
                                         int K, uint8_t* lds, uint4 (&b0)[NF], uint32_t (&bwa)[NF / 2], int lane,
                                         int half) {
  const int nblk = K / 32, last = K / kBK - 1;
  store_w_stage(p.w0, lds);
  store_w_stage(p.w1, lds + kStageBytes);
  if (PAT == 0) {
    p.o0.sp[0] = p.r0.spd[0];
    p.o0.sp[1] = p.r0.spd[1];
  } else {
    p.o0.sp[0] = expand_block<PAT>(p.r0.spc[0], p.r0.spm[0]);
    p.o0.sp[1] = expand_block<PAT>(p.r0.spc[1], p.r0.spm[1]);
  }
  p.o0.ssp = p.r0.ssp >> (16 * half);
  p.o0.sdn = p.r0.sdn >> (16 * half);
  load_w<NF, true>(p.w0, wc, ws, n0, N, K, 3 < last ? 3 : last, nblk);
  __syncthreads();
  read_bw(bwa, lds, lane);
  read_b<0, 0, NF>(b0, lds, lane);
}

// Every K step of a started tile into acc.
template <int PAT, int NF, int SPR = 0>
__device__ __forceinline__ void il_main(v16f (&acc)[NF], IlSets<NF>& p, uint4 (&b0)[NF], uint32_t (&bwa)[NF / 2],
                                        const ARow& a, const uint8_t* wc, const uint8_t* ws, int n0, int N, int K,
                                        uint8_t* lds, int lane, int half, const uint2* lut) {
  const int nks = K / kBK, last = nks - 1;
  const auto cl = [&](int k) { return k < last ? k : last; };
  uint8_t* const st0 = lds;
  uint8_t* const st1 = lds + kStageBytes;
  uint8_t* const st2 = lds + 2 * kStageBytes;
  uint32_t bwb[NF / 2];
  int ks = 0;
  for (; ks + 2 < nks; ks += 3) {
    step_il<PAT, SPR>(acc, p.o0, b0, bwa, bwb, st0, st1, st2, p.o1, p.r1, p.w2, lane, [&](auto part) {
      constexpr int P = decltype(part)::value;
      if constexpr (P == 0) load_a_dn(p.o2, a, cl(ks + 2), half);
      else if constexpr (P == 1) load_a_meta_part<PAT, 0>(p.r0, a, cl(ks + 3), half);
      else if constexpr (P == 2) load_a_meta_part<PAT, 1>(p.r0, a, cl(ks + 3), half);
      else load_w_part<NF, P - 3>(p.w1, wc, ws, n0, N, cl(ks + 4));
    }, lut);
    __syncthreads();
    step_il<PAT, SPR>(acc, p.o1, b0, bwb, bwa, st1, st2, st0, p.o2, p.r2, p.w0, lane, [&](auto part) {
      constexpr int P = decltype(part)::value;
      if constexpr (P == 0) load_a_dn(p.o0, a, cl(ks + 3), half);
      else if constexpr (P == 1) load_a_meta_part<PAT, 0>(p.r1, a, cl(ks + 4), half);
      else if constexpr (P == 2) load_a_meta_part<PAT, 1>(p.r1, a, cl(ks + 4), half);
      else load_w_part<NF, P - 3>(p.w2, wc, ws, n0, N, cl(ks + 5));
    }, lut);
    __syncthreads();
    step_il<PAT, SPR>(acc, p.o2, b0, bwa, bwb, st2, st0, st1, p.o0, p.r0, p.w1, lane, [&](auto part) {
      constexpr int P = decltype(part)::value;
      if constexpr (P == 0) load_a_dn(p.o1, a, cl(ks + 4), half);
      else if constexpr (P == 1) load_a_meta_part<PAT, 0>(p.r2, a, cl(ks + 5), half);
      else if constexpr (P == 2) load_a_meta_part<PAT, 1>(p.r2, a, cl(ks + 5), half);
      else load_w_part<NF, P - 3>(p.w0, wc, ws, n0, N, cl(ks + 6));
    }, lut);
    __syncthreads();
    // bw alternates with period two: after three steps the roles swap
#pragma unroll
    for (int i = 0; i < NF / 2; ++i) {
      const uint32_t t = bwa[i];
      bwa[i] = bwb[i];
      bwb[i] = t;
    }
  }
  if (ks < nks) {   // one or two steps left, in sets 0 and 1
    step_il<PAT, SPR>(acc, p.o0, b0, bwa, bwb, st0, st1, st2, p.o1, p.r1, p.w2, lane, [](auto) {}, lut);
    if (ks + 1 < nks) {
      __syncthreads();
      step_il<PAT, SPR>(acc, p.o1, b0, bwb, bwa, st1, st2, st0, p.o2, p.r2, p.w0, lane, [](auto) {}, lut);
    }
  }
}

// This lane's activation row in a tile of rows [row_lo, row_hi): rows past
// the end are clamped (loads stay in bounds, stores are masked).
__device__ __forceinline__ int64_t il_row(const int32_t* row_index, int64_t row_lo, int64_t row_hi) {
  int64_t orow = row_lo + (threadIdx.x >> 6) * 32 + (threadIdx.x & 31);
  if (orow >= row_hi) orow = row_hi - 1;
  return row_index ? (int64_t)row_index[orow] : orow;
}

// The last panel of a K that is not a multiple of 128 (1 to 3 blocks), after
// the tile's full panels: its few operands come straight from global memory,
// block 2 SUB + half per lane; lanes past K reread block 0 and zero the weight.
// Beside ~30 full steps its latency is small (about one step), and the full
// panels keep the interleaved pipeline: M 1024, N 5000, K 2080, 50 us on the
// double-buffered kernel that handled such K before.
template <int PAT, int NF>
__device__ __forceinline__ void il_tail(v16f (&acc)[NF], const ARow& a, const uint8_t* wc, const uint8_t* ws, int n0,
                                        int N, int K, int lane, int half) {
  const int ks = K / kBK, nb = (K - kBK * ks) >> 5, col = lane & 31;
  const int64_t pr = (int64_t)ks * a.R * 4 + a.r * nb, pn = (int64_t)ks * N * 4;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    if (2 * sub >= nb) break;   // the same in every lane
    const bool in = 2 * sub + half < nb;
    const int j = in ? 2 * sub + half : 0;
    const uint4 dn = *reinterpret_cast<const uint4*>(a.dn + (pr + j) * 16);
    const uint2 c = *reinterpret_cast<const uint2*>(a.spc + (pr + j) * 8);
    const uint32_t meta = *reinterpret_cast<const uint32_t*>(a.spm + (pr + j) * 4);
    const uint32_t ssp = a.sps[pr + j], sdn = a.dns[pr + j];
    uint4 b[NF];
    uint32_t sw[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int64_t V = pn + (int64_t)min(n0 + 32 * f + col, N - 1) * nb + j;
      b[f] = *reinterpret_cast<const uint4*>(wc + V * 16);
      sw[f] = ws[V];
    }
    const v8i sp = as_operand(expand_block<PAT>(c, meta)), rs = as_operand(dn);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      if (!in) b[f] = make_uint4(0u, 0u, 0u, 0u);
      acc[f] = mfma_fp4<0, 0>(as_operand(b[f]), sp, acc[f], sw[f], ssp);
    }
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = mfma_fp4<0, 0>(as_operand(b[f]), rs, acc[f], sw[f], sdn);
  }
}

// One tile of the interleaved pipeline, alone: its LDS stages at lds, its
// epilogue staged over them once every wavefront is done with them.
template <int PAT, typename OutT, int NF, bool TAIL = false>
__device__ __forceinline__ void tile_mx_il(const uint8_t* sp_codes, const uint8_t* sp_meta, const uint8_t* sp_scale,
                                           const uint8_t* dn_codes, const uint8_t* dn_scale, const int32_t* row_index,
                                           int64_t act_rows, int64_t row_lo, int64_t row_hi, const uint8_t* wc,
                                           const uint8_t* ws, int n0, int N, int K, OutT* Y, int64_t ldy,
                                           uint8_t* lds, const uint2* lut) {
  static_assert(NF == 8 || NF == 4, "full (256-column) or half tile");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  ARow a;
  a.r = il_row(row_index, row_lo, row_hi);
  a.R = act_rows;
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
  IlSets<NF> p;
  uint4 b0[NF];
  uint32_t bwa[NF / 2];
  il_issue<PAT, NF>(p, a, wc, ws, n0, N, K, half);
  il_start<PAT, NF>(p, wc, ws, n0, N, K, lds, b0, bwa, lane, half);
  il_main<PAT, NF>(acc, p, b0, bwa, a, wc, ws, n0, N, K, lds, lane, half, lut);
  if constexpr (TAIL) il_tail<PAT, NF>(acc, a, wc, ws, n0, N, K, lane, half);
  __syncthreads();   // every wavefront is done with the weight stages
  il_epilogue<OutT, NF>(acc, Y, ldy, row_lo, row_hi, n0, N, lds + wave * kEpiWave, wave, lane);
}

// A tile of the persistent loops: output rows [row_lo, row_hi), this lane's
// activation row r, weight columns n0.. of the payload at wc / ws.
struct IlTile {
  int64_t row_lo, row_hi, r;
  const uint8_t *wc, *ws;
  int n0;
};

// Full tiles back to back, as handed out by next(IlTile&) until it returns
// false.  The next tile's first loads go out after the current tile's last
// step and before its output stores: the vector-memory counter completes in
// issue order, so loads issued behind the stores would first wait for the
// stores (64 KB per tile) to drain.  The epilogue therefore has its own LDS
// region `epi` (4 kEpiWave bytes) beside the three stages at `lds`.
template <int PAT, typename OutT, bool TAIL, int SPR = 0, class Next>
__device__ __forceinline__ void tiles_mx_il(const uint8_t* sp_codes, const uint8_t* sp_meta, const uint8_t* sp_scale,
                                            const uint8_t* dn_codes, const uint8_t* dn_scale, int64_t act_rows, int N,
                                            int K, OutT* Y, int64_t ldy, uint8_t* lds, uint8_t* epi,
                                            const uint2* lut, Next next) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  IlTile t;
  if (!next(t)) return;
  ARow a;
  a.r = t.r;
  a.R = act_rows;
  a.dn = dn_codes;
  a.spc = sp_codes;
  a.spm = sp_meta;
  a.dns = dn_scale;
  a.sps = sp_scale;
  IlSets<8> p;
  il_issue<PAT, 8>(p, a, t.wc, t.ws, t.n0, N, K, half);
  for (;;) {
    uint4 b0[8];
    uint32_t bwa[4];
    il_start<PAT, 8>(p, t.wc, t.ws, t.n0, N, K, lds, b0, bwa, lane, half);
    IlTile tn;
    const bool more = next(tn);   // the row-index load has the whole tile to arrive
    v16f acc[8];
#pragma unroll
    for (int f = 0; f < 8; ++f)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[f][r] = 0.0f;
    il_main<PAT, 8, SPR>(acc, p, b0, bwa, a, t.wc, t.ws, t.n0, N, K, lds, lane, half, lut);
    if constexpr (TAIL) il_tail<PAT, 8>(acc, a, t.wc, t.ws, t.n0, N, K, lane, half);
    if (more) {
      a.r = tn.r;
      il_issue<PAT, 8>(p, a, tn.wc, tn.ws, tn.n0, N, K, half);
    }
    il_epilogue<OutT, 8>(acc, Y, ldy, t.row_lo, t.row_hi, t.n0, N, epi + wave * kEpiWave, wave, lane);
    if (!more) return;
    t = tn;
    __syncthreads();   // every wavefront is done with the stages before they are refilled
  }
}

// One tile per workgroup, for K below 128 (the simpler pipeline of tile_mx,
// which needs no full panel).
template <int NF, int PAT, bool SCALE_DW, typename OutT>
__global__ __launch_bounds__(256) void k_linear_mx(const uint8_t* sp_codes, const uint8_t* sp_meta,
                                                   const uint8_t* sp_scale, const uint8_t* dn_codes,
                                                   const uint8_t* dn_scale, int64_t M, const uint8_t* wc,
                                                   const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy, int gx,
                                                   int gy) {
  constexpr int BN = 32 * NF;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BN * kLdsStride + 2 * 64 * 2 * NF];
  uint8_t* lds_w = lds;
  uint8_t* lds_s = lds + 2 * BN * kLdsStride;
  int mt, nt;
  tile_of(blockIdx.x, gx, gy, mt, nt);
  const int n0 = nt * BN;
  const int64_t m0 = (int64_t)mt * kBM;
  const int64_t m1 = m0 + kBM < M ? m0 + kBM : M;
  tile_mx<NF, PAT, SCALE_DW, OutT>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, nullptr, M, m0, m1, wc, ws, n0, N,
                                   K, Y, ldy, lds_w, lds_s);
}

// Persistent dense kernel (K of at least 128): at most one workgroup per
// CU, walking the work units b, b + G, b + 2G, ... (G workgroups).  A tile's
// output stores then drain while the same CU starts its next tile instead of
// the whole grid waiting at the end of every round (3% on the Llama gate/up
// shape, 7 rounds).  With G a multiple of 8 every tile an XCD runs keeps the
// XCD of its number, so the tile_of blocks still share an L2.
//
// Units [0, full) are whole tiles.  When the last round would be at most
// half full (tiles = full + r, 0 < r <= G / 2), its r tiles run instead as
// 2 r half tiles of 128 columns, units [full, full + 2 r): every CU then
// runs a half tile instead of half of the CUs running a whole one (the
// Llama qkv shape: 384 tiles on 256 CUs).  Half tile u covers tile t(u),
// columns 128 h(u) on; with r a multiple of 8, t(u) keeps the XCD of u.

template <int PAT, typename OutT, bool TAIL>
__global__ __launch_bounds__(256) void k_linear_mx_persist(const uint8_t* sp_codes, const uint8_t* sp_meta,
                                                           const uint8_t* sp_scale, const uint8_t* dn_codes,
                                                           const uint8_t* dn_scale, int64_t M, const uint8_t* wc,
                                                           const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy,
                                                           int gx, int gy, int full, int halves) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kPersistLds];
  __shared__ uint2 lut48[256];
  if (PAT == 48) {
    lut48_fill(lut48);
    __syncthreads();
  }
  int id = (int)blockIdx.x;
  tiles_mx_il<PAT, OutT, TAIL>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, M, N, K, Y, ldy, lds,
                         lds + 3 * kStageBytes, lut48, [&](IlTile& t) {
                           if (id >= full) return false;
                           int mt, nt;
                           tile_of(id, gx, gy, mt, nt);
                           t.row_lo = (int64_t)mt * kBM;
                           t.row_hi = t.row_lo + kBM < M ? t.row_lo + kBM : M;
                           t.r = il_row(nullptr, t.row_lo, t.row_hi);
                           t.wc = wc;
                           t.ws = ws;
                           t.n0 = nt * 256;
                           id += (int)gridDim.x;
                           return true;
                         });
  for (; id < full + halves; id += (int)gridDim.x) {
    int t, h, mt, nt;
    half_unit(id - full, full, halves, t, h);
    tile_of(t, gx, gy, mt, nt);
    const int64_t m0 = (int64_t)mt * kBM;
    const int64_t m1 = m0 + kBM < M ? m0 + kBM : M;
    __syncthreads();   // the LDS stages are free before this tile's prologue
    tile_mx_il<PAT, OutT, 4, TAIL>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, nullptr, M, m0, m1, wc, ws,
                             nt * 256 + 128 * h, N, K, Y, ldy, lds, lut48);
  }
}

// Grouped (MoE) form.  The grid is (column tiles) x (items); an item is a
// 128-row tile of one expert's slice [off[e], off[e+1]) of the output.  The
// tile-to-expert map is rebuilt on the device from expert_offsets (an
// exclusive scan of ceil(rows_e / 128)), so the host never reads the
// routing.  Items past the last tile exit before any barrier.
template <int NF, int PAT, bool SCALE_DW, typename OutT>
__global__ __launch_bounds__(256) void k_linear_mx_grouped(
    const uint8_t* sp_codes, const uint8_t* sp_meta, const uint8_t* sp_scale, const uint8_t* dn_codes,
    const uint8_t* dn_scale, const int32_t* row_index, int64_t act_rows, const int32_t* offs, int E,
    const uint8_t* wc, const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy, int gx) {
  constexpr int BN = 32 * NF;
  constexpr int kOld = 2 * BN * kLdsStride + 2 * 64 * 2 * NF;
  __shared__ __attribute__((aligned(16))) uint8_t lds[kOld > kTileLds ? kOld : kTileLds];
  uint8_t* lds_w = lds;
  uint8_t* lds_s = lds + 2 * BN * kLdsStride;
  __shared__ int s_first[1025];
  const int tid = threadIdx.x;
  // tiles per expert, then an inclusive scan (Hillis-Steele) over <= 1024 experts
  for (int e = tid; e < E; e += 256) {
    const int rows = offs[e + 1] - offs[e];
    s_first[e + 1] = rows > 0 ? (rows + kBM - 1) / kBM : 0;
  }
  if (tid == 0) s_first[0] = 0;
  __syncthreads();
  for (int step = 1; step < E; step <<= 1) {
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j + 1;
      v[j] = (e <= E && e - step >= 1) ? s_first[e - step] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j + 1;
      if (e <= E) s_first[e] += v[j];
    }
    __syncthreads();
  }
  // Workgroups go round-robin over the 8 XCDs; renumber so that each XCD
  // walks a contiguous range of (column tile, item) pairs in column-major
  // order: the few row tiles of one expert that share a weight tile then run
  // back to back on one XCD and reuse it from that XCD's L2.
  const int items = (int)gridDim.x / gx;
  const int total_wg = (int)gridDim.x;
  int idp = blockIdx.x;
  if ((total_wg & 7) == 0) idp = (blockIdx.x & 7) * (total_wg >> 3) + (blockIdx.x >> 3);
  const int xt = idp / items, item = idp - xt * items;
  if (item >= s_first[E]) return;   // uniform across the workgroup
  int lo = 0, hi = E;               // find e with s_first[e] <= item < s_first[e+1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (s_first[mid] <= item) lo = mid; else hi = mid;
  }
  const int e = lo;
  const int64_t r0 = (int64_t)offs[e] + (int64_t)(item - s_first[e]) * kBM;
  const int64_t r_end = offs[e + 1];
  const int64_t r1 = r0 + kBM < r_end ? r0 + kBM : r_end;
  const int n0 = xt * BN;
  const uint8_t* wce = wc + (int64_t)e * N * (K / 2);
  const uint8_t* wse = ws + (int64_t)e * N * (K / 32);
  if constexpr (SCALE_DW && NF == 8)
  {
    __shared__ uint2 lut48[256];
    if (PAT == 48) {
      lut48_fill(lut48);
      __syncthreads();
    }
    tile_mx_il<PAT, OutT, 8>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, row_index, act_rows, r0, r1, wce, wse, n0,
                          N, K, Y, ldy, lds, lut48);
  }
  else
    tile_mx<NF, PAT, SCALE_DW, OutT>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, row_index, act_rows, r0, r1,
                                     wce, wse, n0, N, K, Y, ldy, lds_w, lds_s);
}

// Persistent grouped form (K of at least 128): at most one workgroup per
// CU walks the real (column tile, item) pairs -- their count comes from the
// same on-device scan -- so a CU starts its next tile without a new
// workgroup launch and the padding items of the launch-per-tile form cost
// nothing.  The order is XCD-contiguous and item-major: the column tiles of
// one row tile, and the few row tiles of one expert, run at the same time on
// one XCD and share its L2 (an item's gathered activation rows and the
// expert's weight tiles).  Measured on the Qwen3-30B-A3B experts (4096
// tokens, top-8): gate_up 190.7 -> 173.7 us, bit-identical; its 1902 units
// had fallen outside the earlier numbering, which required a multiple of 8,
// and were spread round-robin over the XCDs.  A last round at most half
// full runs as half tiles, as in the dense kernel (gate_up's 110 leftover
// units as 220 halves: 164.4 -> 162.8 us).  GATHER (a row map is given):
// full tiles take the spread load schedule of step5 (gate_up 165 -> 154 us,
// bit-identical; contiguous rows keep the burst, which is faster for them).
template <int PAT, typename OutT, bool TAIL, bool GATHER>
__global__ __launch_bounds__(256) void k_linear_mx_grouped_persist(
    const uint8_t* sp_codes, const uint8_t* sp_meta, const uint8_t* sp_scale, const uint8_t* dn_codes,
    const uint8_t* dn_scale, const int32_t* row_index, int64_t act_rows, const int32_t* offs, int E,
    const uint8_t* wc, const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy, int gx) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kPersistLds];
  __shared__ int s_first[1025];
  __shared__ uint2 lut48[256];
  const int tid = threadIdx.x;
  for (int e = tid; e < E; e += 256) {
    const int rows = offs[e + 1] - offs[e];
    s_first[e + 1] = rows > 0 ? (rows + kBM - 1) / kBM : 0;
  }
  if (tid == 0) s_first[0] = 0;
  if (PAT == 48) lut48_fill(lut48);
  __syncthreads();
  for (int step = 1; step < E; step <<= 1) {
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j + 1;
      v[j] = (e <= E && e - step >= 1) ? s_first[e - step] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = tid + 256 * j + 1;
      if (e <= E) s_first[e] += v[j];
    }
    __syncthreads();
  }
  const int items = s_first[E];
  const int total = gx * items;
  // When the last round would be at most half full, its units run as twice
  // as many half tiles of 128 columns (as in k_linear_mx_persist).
  const int G = (int)gridDim.x, rem = total % G;
  const int halves = rem > 0 && 2 * rem <= G ? 2 * rem : 0;
  const int full = total - halves / 2;
  // unit u (item-major: item u / gx, column tile u mod gx) -> expert, rows
  const auto locate = [&](int u, int& e, int64_t& row_lo, int64_t& row_hi) {
    const int item = u / gx;
    int lo = 0, hi = E;   // e with s_first[e] <= item < s_first[e+1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_first[mid] <= item) lo = mid; else hi = mid;
    }
    e = lo;
    row_lo = (int64_t)offs[e] + (int64_t)(item - s_first[e]) * kBM;
    const int64_t r_end = offs[e + 1];
    row_hi = row_lo + kBM < r_end ? row_lo + kBM : r_end;
  };
  // each XCD takes a contiguous range of the whole-tile units (xcd_unit)
  int id = (int)blockIdx.x;
  tiles_mx_il<PAT, OutT, TAIL, GATHER ? 1 : 0>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, act_rows, N, K, Y, ldy, lds,
                         lds + 3 * kStageBytes, lut48, [&](IlTile& t) {
                           if (id >= full) return false;
                           const int u = xcd_unit(id, full);
                           id += G;
                           int e;
                           locate(u, e, t.row_lo, t.row_hi);
                           t.r = il_row(row_index, t.row_lo, t.row_hi);
                           t.wc = wc + (int64_t)e * N * (K / 2);
                           t.ws = ws + (int64_t)e * N * (K / 32);
                           t.n0 = (u % gx) * 256;
                           return true;
                         });
  if ((int)blockIdx.x < halves) {
    int u, h, e;
    half_unit((int)blockIdx.x, full, halves, u, h);
    int64_t row_lo, row_hi;
    locate(u, e, row_lo, row_hi);
    __syncthreads();   // the LDS stages are free before this tile's prologue
    tile_mx_il<PAT, OutT, 4, TAIL>(sp_codes, sp_meta, sp_scale, dn_codes, dn_scale, row_index, act_rows, row_lo, row_hi,
                             wc + (int64_t)e * N * (K / 2), ws + (int64_t)e * N * (K / 32), (u % gx) * 256 + 128 * h,
                             N, K, Y, ldy, lds, lut48);
  }
}

// ---------------------------------------------------------------------------
// Small-M (decode) MXFP4 GEMM
// ---------------------------------------------------------------------------
//
// With few activation rows the layer streams its weight from HBM and the
// prefill tile (128 x 256 outputs) leaves most CUs idle.  Here a workgroup
// owns 16 NB output columns and all M <= 16 MF rows, on the FP4 MFMA
// v_mfma_scale_f32_16x16x128_f8f6f4 (lane l holds row / column l % 16 and
// the 32 K values of block l / 16 of a 128-position panel; accumulator
// element r of lane l is row 4 (l / 16) + r, column l % 16).  Its KS
// wavefronts split K into KS ranges; each streams its weight slice straight
// from HBM into MFMA operands (1 KB loads per panel, coalesced by the
// panel-major layout) with a two-deep register prefetch, expands each
// activation block once for all NB column fragments, and the KS partial
// tiles are added in LDS in a fixed order.

typedef float v4f_t __attribute__((ext_vector_type(4)));

template <int MF, int NB>
struct SkinnyStage {
  uint4 w[NB];             // weight codes: column 16 n + l % 16, block l / 16
  uint32_t ws[NB];         // their E8M0 scales (bytes)
  uint4 dn[MF];            // residual codes of row 16 m + l % 16, block l / 16
  uint2 spc[MF];           // backbone codes and metadata of the same block
  uint32_t spm[MF];
  uint4 spd[MF];           // or (pattern 0) its dense backbone codes
  uint32_t sdn[MF], ssp[MF];
};

struct SkinnyArgs {
  const uint8_t *spc, *spm, *sps, *dnc, *dns, *wc, *ws;
  int64_t M;
  int N, K;
};

// PAT 0: spc is the dense backbone copy (16 bytes per block, the residual
// codes' layout) and spm is unused.  RAG: K is not a multiple of 128; in the
// narrower last panel, lanes whose block lies past K reread block 0 (and zero
// its weight codes in skinny_step).
template <int MF, int NB, int PAT, bool RAG>
__device__ __forceinline__ void skinny_load(SkinnyStage<MF, NB>& st, const SkinnyArgs& p, const int64_t (&row)[MF],
                                            int n0, int ks, int lane) {
  const int nb = RAG ? min(128, p.K - 128 * ks) >> 5 : 4;   // blocks of this panel
  const int j = RAG && (lane >> 4) >= nb ? 0 : lane >> 4;   // block within the panel
  const int64_t pn = (int64_t)ks * p.N * 4, pm = (int64_t)ks * p.M * 4;   // blocks before it
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int64_t V = pn + (int64_t)min(n0 + 16 * n + (lane & 15), p.N - 1) * nb + j;
    st.w[n] = *reinterpret_cast<const uint4*>(p.wc + V * 16);
    st.ws[n] = p.ws[V];
  }
#pragma unroll
  for (int m = 0; m < MF; ++m) {
    const int64_t V = pm + row[m] * nb + j;   // block-major index of (row, block)
    st.dn[m] = *reinterpret_cast<const uint4*>(p.dnc + V * 16);
    if (PAT == 0) {
      st.spd[m] = *reinterpret_cast<const uint4*>(p.spc + V * 16);
    } else {
      st.spc[m] = *reinterpret_cast<const uint2*>(p.spc + V * 8);
      st.spm[m] = *reinterpret_cast<const uint32_t*>(p.spm + V * 4);
    }
    st.sdn[m] = p.dns[V];
    st.ssp[m] = p.sps[V];
  }
}

// The weight is the MFMA's first operand: accumulator element r of lane l is
// then output column 4 (l / 16) + r of the fragment and activation row l % 16.
template <int MF, int NB, int PAT, bool RAG>
__device__ __forceinline__ void skinny_step(v4f_t (&acc)[MF][NB], SkinnyStage<MF, NB>& st, int K, int ks, int lane) {
  if (RAG) {
    const uint32_t in = 32 * (lane >> 4) < K - 128 * ks ? ~0u : 0u;
#pragma unroll
    for (int n = 0; n < NB; ++n)
      st.w[n] = make_uint4(st.w[n].x & in, st.w[n].y & in, st.w[n].z & in, st.w[n].w & in);
  }
#pragma unroll
  for (int m = 0; m < MF; ++m) {
    const v8i asp = as_operand(PAT == 0 ? st.spd[m] : expand_block<PAT>(st.spc[m], st.spm[m]));
    const v8i adn = as_operand(st.dn[m]);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const v8i b = as_operand(st.w[n]);
      acc[m][n] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, asp, acc[m][n], 4, 4, 0, (int)st.ws[n], 0,
                                                                  (int)st.ssp[m]);
      acc[m][n] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, adn, acc[m][n], 4, 4, 0, (int)st.ws[n], 0,
                                                                  (int)st.sdn[m]);
    }
  }
}

// Workgroup id -> (column group, row tile).  Workgroups are dispatched
// round-robin over the 8 XCDs; with several row tiles the ids are renumbered
// to give each XCD a contiguous range in which the row tiles of one column
// group follow each other, so the workgroups that read the same weight
// columns share an L2.
__device__ __forceinline__ void skinny_tile(int id, int ncg, int nrt, int& cg, int& rt) {
  if (nrt == 1) {
    cg = id;
    rt = 0;
    return;
  }
  const int total = ncg * nrt;
  const int idp = (total & 7) == 0 ? (id & 7) * (total >> 3) + (id >> 3) : id;
  cg = idp / nrt;
  rt = idp - cg * nrt;
}

// One tile of 16 MF rows (the lane's are `row`) x 16 NB columns by the KS
// wavefronts of a workgroup, into Y rows [y0, y_end).
template <int MF, int NB, int KS, int PAT, bool RAG>
__device__ __forceinline__ void skinny_compute(const SkinnyArgs& p, const int64_t (&row)[MF], int64_t y0,
                                               int64_t y_end, int n0, void* Y, int ydt, int64_t ldy,
                                               float (&part)[KS][MF * NB][256]) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nks = (p.K + kBK - 1) / kBK;
  const int per = (nks + KS - 1) / KS;
  const int k0 = wave * per, k1 = min(nks, k0 + per);

  v4f_t acc[MF][NB];
#pragma unroll
  for (int m = 0; m < MF; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[m][n] = v4f_t{0.0f, 0.0f, 0.0f, 0.0f};

  // The order of a panel's loads and MFMAs.  Left alone, the compiler moves both
  // stages' conditional loads behind both stages' MFMAs and then waits for all of
  // them, which suits few rows (more wavefronts stream); with 64 rows a CU has one
  // wavefront per SIMD and its own MFMAs have to cover its loads.  Fences keep them
  // between; with the backbone to expand, loads without a branch (past the
  // range the last panel again) do better.  N 4096, K 14336, M 256, us: dense copy
  // 42.0 plain, 43.0 clamped, 36.8 fenced; 2:4 54.1, 40.3, 49.6; 4:8 75.1, 62.5, 73.3.
  constexpr int kPlain = 0, kFenced = 1, kClamped = 2;
  constexpr int kOrder = MF == 4 && PAT == 0 ? kFenced : PAT != 0 && NB == 4 && MF * KS >= 16 ? kClamped : kPlain;
  SkinnyStage<MF, NB> s0, s1;
  if (k0 < k1) skinny_load<MF, NB, PAT, RAG>(s0, p, row, n0, k0, lane);
  if (k0 + 1 < k1) skinny_load<MF, NB, PAT, RAG>(s1, p, row, n0, k0 + 1, lane);
  int ks = k0;
  if constexpr (kOrder == kFenced) {
    for (; ks + 1 < k1; ks += 2) {
      skinny_step<MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);
      SHARQ_FENCE();
      if (ks + 2 < k1) skinny_load<MF, NB, PAT, RAG>(s0, p, row, n0, ks + 2, lane);
      SHARQ_FENCE();
      skinny_step<MF, NB, PAT, RAG>(acc, s1, p.K, ks + 1, lane);
      SHARQ_FENCE();
      if (ks + 3 < k1) skinny_load<MF, NB, PAT, RAG>(s1, p, row, n0, ks + 3, lane);
      SHARQ_FENCE();
    }
  } else if constexpr (kOrder == kClamped) {
    constexpr int kMore = MF == 2 && !RAG ? 2 : 1;   // 2: no loads after the last panels
    for (; ks + kMore < k1; ks += 2) {
      skinny_step<MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);
      skinny_load<MF, NB, PAT, RAG>(s0, p, row, n0, min(ks + 2, k1 - 1), lane);
      skinny_step<MF, NB, PAT, RAG>(acc, s1, p.K, ks + 1, lane);
      skinny_load<MF, NB, PAT, RAG>(s1, p, row, n0, min(ks + 3, k1 - 1), lane);
    }
    if (kMore == 2 && ks + 1 < k1) {
      skinny_step<MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);
      skinny_step<MF, NB, PAT, RAG>(acc, s1, p.K, ks + 1, lane);
      ks += 2;
    }
  } else {
    for (; ks + 1 < k1; ks += 2) {
      skinny_step<MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);
      if (ks + 2 < k1) skinny_load<MF, NB, PAT, RAG>(s0, p, row, n0, ks + 2, lane);
      skinny_step<MF, NB, PAT, RAG>(acc, s1, p.K, ks + 1, lane);
      if (ks + 3 < k1) skinny_load<MF, NB, PAT, RAG>(s1, p, row, n0, ks + 3, lane);
    }
  }
  if (ks < k1) skinny_step<MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);

  // the KS partial tiles, added by all threads in the order of K
#pragma unroll
  for (int m = 0; m < MF; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) *reinterpret_cast<v4f_t*>(&part[wave][m * NB + n][4 * lane]) = acc[m][n];
  __syncthreads();
  for (int q = tid; q < MF * NB * 256; q += 64 * KS) {
    const int f = q >> 8, e = q & 255, m = f / NB, n = f - m * NB;
    const int r = e >> 4, c = e & 15;                      // row and column of the fragment
    const int at = 64 * (c >> 2) + 4 * r + (c & 3);        // its place in the accumulator layout
    float v = part[0][f][at];
    for (int w = 1; w < KS; ++w) v += part[w][f][at];
    const int64_t yr = y0 + 16 * m + r;
    const int col = n0 + 16 * n + c;
    if (yr < y_end && col < p.N) {
      if (ydt == 2) reinterpret_cast<float*>(Y)[yr * ldy + col] = v;
      else if (ydt == 1) reinterpret_cast<_Float16*>(Y)[yr * ldy + col] = (_Float16)v;
      else reinterpret_cast<uint16_t*>(Y)[yr * ldy + col] = f32_to_bf16_rne(v);
    }
  }
}

template <int MF, int NB, int KS, int PAT, bool RAG>
__global__ __launch_bounds__(64 * KS) void k_linear_mx_skinny(SkinnyArgs p, void* Y, int ydt, int64_t ldy, int ncg,
                                                              int nrt) {
  __shared__ float part[KS][MF * NB][256];
  const int lane = threadIdx.x & 63;
  int cg, rt;
  skinny_tile(blockIdx.x, ncg, nrt, cg, rt);
  const int64_t r0 = (int64_t)rt * 16 * MF;
  int64_t row[MF];
#pragma unroll
  for (int m = 0; m < MF; ++m) {
    row[m] = r0 + 16 * m + (lane & 15);
    if (row[m] >= p.M) row[m] = p.M - 1;   // loads stay in bounds, stores are masked
  }
  skinny_compute<MF, NB, KS, PAT, RAG>(p, row, r0, p.M, cg * 16 * NB, Y, ydt, ldy, part);
}

// Grouped forms for few rows (MoE decode), where the launch streams the
// experts' weights: a workgroup takes 16 NB columns and up to CH rows of one
// expert, with no 128-row tiles and, for an expert's first CH rows, no scan over
// the experts.  The rows of a popular expert beyond those go to total / CH
// further slots, the first of the grid, which find theirs by a scan (most end
// there): walking them in one workgroup took 55 us instead of 7.6 where all 512
// rows have one expert of 128 (N 2048, K 768).  extra >= the sum over experts
// of (rows - 1) / CH.  K is split over KS wavefronts: where routing leaves few
// workgroups with rows, their loads in flight bound the launch (without a split
// E 8, N 28672, K 4096, 64 rows of one expert 41.0 us, 18.3 with 8 rows; E 128, N
// 1536, K 2048, 128 rows 35.9, 28.6 split in four).
template <int CH>
__device__ __forceinline__ bool grouped_chunk(const int32_t* offs, int E, int extra, int slot, int& e, int& lo,
                                              int& hi) {
  int skip = 0;   // chunks of the expert before this one
  if (slot >= extra) {
    e = slot - extra;
  } else {
    const int lane = threadIdx.x & 63;
    int base = 0, before = 0;
    for (;; base += 64) {   // the same in every lane
      if (base >= E) return false;
      const int ex = base + lane;
      const int rows = ex < E ? offs[ex + 1] - offs[ex] : 0;
      const int more = rows > CH ? (rows - 1) / CH : 0;
      int sum = more;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(sum, d);
        if (lane >= d) sum += up;
      }
      const uint64_t in = __ballot(slot < before + sum);
      if (in != 0) {
        const int l = __builtin_ctzll(in);
        e = base + l;
        skip = slot - before - __shfl(sum - more, l) + 1;
        break;
      }
      before += __shfl(sum, 63);
    }
    e = __builtin_amdgcn_readfirstlane(e);
    skip = __builtin_amdgcn_readfirstlane(skip);
  }
  lo = offs[e] + skip * CH;
  hi = offs[e + 1];
  if (hi - lo > CH) hi = lo + CH;
  return hi > lo;
}

template <int MF, int NB, int KS, int PAT, bool RAG>
__global__ __launch_bounds__(64 * KS) void k_linear_mx_grouped_skinny(SkinnyArgs p, const int32_t* ridx,
                                                                      const int32_t* offs, int E, int extra, void* Y,
                                                                      int ydt, int64_t ldy, int ncg) {
  __shared__ float part[KS][MF * NB][256];
  const int lane = threadIdx.x & 63;
  const int slot = (int)blockIdx.x / ncg, cg = (int)blockIdx.x - slot * ncg;
  int e, lo, hi;
  if (!grouped_chunk<16 * MF>(offs, E, extra, slot, e, lo, hi)) return;   // the same in every wavefront
  p.wc += (int64_t)e * p.N * (p.K / 2);
  p.ws += (int64_t)e * p.N * (p.K / 32);
  int64_t row[MF];
#pragma unroll
  for (int m = 0; m < MF; ++m) {
    int i = lo + 16 * m + (lane & 15);
    if (i >= hi) i = hi - 1;   // loads stay in bounds, stores are masked
    row[m] = ridx ? (int64_t)ridx[i] : (int64_t)i;
  }
  skinny_compute<MF, NB, KS, PAT, RAG>(p, row, lo, hi, cg * 16 * NB, Y, ydt, ldy, part);
}

template <int MF, int NB, int KS, int PAT>
static hipError_t go_skinny(const SkinnyArgs& p, void* Y, int ydt, int64_t ldy, hipStream_t st) {
  const int ncg = (p.N + 16 * NB - 1) / (16 * NB);
  const int nrt = (int)((p.M + 16 * MF - 1) / (16 * MF));
  const dim3 grid((unsigned)(ncg * nrt)), block(64 * KS);
  if constexpr (PAT != 0) {
    if (p.K % kBK != 0) {
      k_linear_mx_skinny<MF, NB, KS, PAT, true><<<grid, block, 0, st>>>(p, Y, ydt, ldy, ncg, nrt);
      return hipGetLastError();
    }
  }
  k_linear_mx_skinny<MF, NB, KS, PAT, false><<<grid, block, 0, st>>>(p, Y, ydt, ldy, ncg, nrt);
  return hipGetLastError();
}

// K split: about 8192 weight streams in flight (wavefronts x column
// fragments per wavefront, for M > 16 wavefronts alone) to keep HBM busy,
// at least 4 panels per wavefront, at most `cap` wavefronts per workgroup.
static int skinny_split(int wgs, int K, int cap) {
  const int nks = (K + kBK - 1) / kBK;
  int ks = 4;
  while (ks < cap && wgs * ks * 2 <= 8192 && nks >= 4 * ks * 2) ks *= 2;
  return ks;
}

// (row fragments, column fragments, K splits) by M: every activation block
// expansion feeds NB column fragments; the K split keeps enough wavefronts
// streaming the weight.  Above 16 rows the workgroups tile M by 32 or 64.
template <int PAT>
static hipError_t go_skinny_m(const SkinnyArgs& p, void* Y, int ydt, int64_t ldy, hipStream_t st) {
  const int64_t M = p.M;
  const int N = p.N, K = p.K;
  if (M <= 16) {
    // Column fragments: as many as leave at least 192 workgroups (one
    // workgroup runs on one CU), since each activation block loaded and
    // expanded then feeds more weight columns.
    // Measured on the Llama decode shapes with the weight streamed from HBM
    // (µs, M = 1 / 16): qkv 6.3 / 7.6 -> 5.7 / 6.3 with 2 fragments, gate_up
    // 19.3 / 24.2 -> 16.3 / 17.3 with 4.  Sixteen wavefronts of 4 fragments
    // spill registers, hence the cap of 8.
    const int nb = (N + 63) / 64 >= 192 ? 4 : (N + 31) / 32 >= 192 ? 2 : 1;
    const int ks = skinny_split((N + 15) / 16, K, nb == 4 ? 8 : 16);
#define SHARQ_SKINNY1(NB_, KS_) \
  if (nb == NB_ && ks == KS_) return go_skinny<1, NB_, KS_, PAT>(p, Y, ydt, ldy, st);
    SHARQ_SKINNY1(4, 4) SHARQ_SKINNY1(4, 8)
    SHARQ_SKINNY1(2, 4) SHARQ_SKINNY1(2, 8) SHARQ_SKINNY1(2, 16)
    SHARQ_SKINNY1(1, 4) SHARQ_SKINNY1(1, 8) SHARQ_SKINNY1(1, 16)
#undef SHARQ_SKINNY1
    return hipErrorInvalidValue;   // unreachable: (nb, ks) is one of the above
  }
  if (M <= 32) {
    // As at M <= 16, 4 column fragments when N leaves 192 workgroups of 64
    // columns (M = 32 gate_up from HBM: 32.1 -> 26.0 µs), else 2.
    const int ks = skinny_split((N + 15) / 16, K, 8);
    if ((N + 63) / 64 >= 192)
      return ks == 8 ? go_skinny<2, 4, 8, PAT>(p, Y, ydt, ldy, st)
                     : go_skinny<2, 4, 4, PAT>(p, Y, ydt, ldy, st);
    return ks == 8 ? go_skinny<2, 2, 8, PAT>(p, Y, ydt, ldy, st)
                   : go_skinny<2, 2, 4, PAT>(p, Y, ydt, ldy, st);
  }
  const SkinnyWide w = skinny_wide(M, N, K, backbone_form(PAT), device_cus());
#define SHARQ_SKINNY(MF_, NB_, KS_) \
  if (w.mf == MF_ && w.nb == NB_ && w.ks == KS_) return go_skinny<MF_, NB_, KS_, PAT>(p, Y, ydt, ldy, st);
  SHARQ_SKINNY(1, 1, 8) SHARQ_SKINNY(2, 1, 8) SHARQ_SKINNY(2, 2, 8) SHARQ_SKINNY(2, 4, 8) SHARQ_SKINNY(2, 4, 4)
  SHARQ_SKINNY(4, 4, 4)
#undef SHARQ_SKINNY
  return hipErrorInvalidValue;   // unreachable
}

// ---------------------------------------------------------------------------
// Path combinations (Sec. 4.4, table "ablation-combination"): the sum of up
// to two paths, each sparse (compressed codes + metadata, expanded in
// registers; scale per 32 logical positions) or dense (plain codes), into one
// accumulator.  Path 1 reads the sp_* buffers, path 2 the dn_* buffers.  A
// slot kind is 0 (absent), kSlotDense, or the sparse metadata layout (24 for
// 2:4, 48 for 4:8).  Generic kernels -- one tile per workgroup, double-
// buffered weight stages, any K a multiple of 32 -- since the combinations
// other than SharQ's exist for ablation.
// ---------------------------------------------------------------------------

constexpr int kSlotDense = 1;

struct SlotBuf {
  const uint8_t *c, *m, *s;   // codes, metadata (sparse only), scales
};

// One slot's data of one MXFP4 K step for this lane: per sub-step the codes
// (dense: 16 bytes; sparse: 8 bytes in .x/.y and the metadata dword in .z)
// and the four E8M0 scales of the step's blocks (byte j = block 4 ks + j).
struct SlotStep {
  uint4 c[2];
  uint32_t s;
};

template <int KIND>
__device__ __forceinline__ void load_slot_mx(SlotStep& d, const SlotBuf& b, int64_t r, int64_t R, int ks, int half,
                                             int nblk, int K) {
  if (KIND == 0) return;
  const int wp = min(128, K - 128 * ks);
  const int64_t pr = (int64_t)ks * R;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    const int j = 2 * sub + half;
    const bool ok = 4 * ks + j < nblk;
    if (KIND == kSlotDense) {
      d.c[sub] = ok ? *reinterpret_cast<const uint4*>(b.c + pr * 64 + r * (wp / 2) + 16 * j) : make_uint4(0u, 0u, 0u, 0u);
    } else {
      const uint2 c = ok ? *reinterpret_cast<const uint2*>(b.c + pr * 32 + r * (wp / 4) + 8 * j) : make_uint2(0u, 0u);
      const uint32_t m = ok ? *reinterpret_cast<const uint32_t*>(b.m + pr * 16 + r * (wp / 8) + 4 * j) : 0x44444444u;
      d.c[sub] = make_uint4(c.x, c.y, m, 0u);
    }
  }
  const uint8_t* sr = b.s + pr * 4 + r * (wp / 32);
  d.s = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) d.s |= (uint32_t)(4 * ks + j < nblk ? sr[j] : 127u) << (8 * j);
}

template <int KIND>
__device__ __forceinline__ v8i slot_operand(const uint4& c) {
  if (KIND == kSlotDense) return as_operand(c);
  return as_operand(expand_block<KIND>(make_uint2(c.x, c.y), c.z));
}

template <int SUB, int KIND>
__device__ __forceinline__ void mma_slot(v16f (&acc)[8], const v8i (&b)[8], const SlotStep& a, const uint32_t (&bw)[4],
                                         int half) {
  if (KIND == 0) return;
  const v8i op = slot_operand<KIND>(a.c[SUB]);
  const uint32_t sa = a.s >> (8 * half);
#pragma unroll
  for (int f = 0; f < 8; ++f) {
    if (f & 1) acc[f] = mfma_fp4<2 * SUB, 2 + SUB>(op, b[f], acc[f], sa, bw[f >> 1]);
    else       acc[f] = mfma_fp4<2 * SUB, SUB>(op, b[f], acc[f], sa, bw[f >> 1]);
  }
}

template <int K1, int K2>
__device__ __forceinline__ void step_slots(v16f (&acc)[8], const SlotStep& a1, const SlotStep& a2, const uint8_t* lw,
                                           const uint8_t* ls, int lane) {
  const int half = lane >> 5, col = lane & 31;
  uint32_t bw[4];
  const uint4 q = *reinterpret_cast<const uint4*>(ls + (2 * col + half) * 16);
  bw[0] = q.x; bw[1] = q.y; bw[2] = q.z; bw[3] = q.w;
#pragma unroll
  for (int sub = 0; sub < 2; ++sub) {
    v8i b[8];
#pragma unroll
    for (int f = 0; f < 8; ++f)
      b[f] = as_operand(*reinterpret_cast<const uint4*>(lw + (f * 32 + col) * kLdsStride + 32 * sub + 16 * half));
    if (sub == 0) {
      mma_slot<0, K1>(acc, b, a1, bw, half);
      mma_slot<0, K2>(acc, b, a2, bw, half);
    } else {
      mma_slot<1, K1>(acc, b, a1, bw, half);
      mma_slot<1, K2>(acc, b, a2, bw, half);
    }
  }
}

template <int K1, int K2, typename OutT>
__global__ __launch_bounds__(256) void k_linear_slots_mx(SlotBuf p1, SlotBuf p2, int64_t M, const uint8_t* wc,
                                                         const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy,
                                                         int gx, int gy) {
  constexpr int NF = 8, BN = 256;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BN * kLdsStride + 2 * 64 * 16];
  uint8_t* const lds_w = lds;
  uint8_t* const lds_s = lds + 2 * BN * kLdsStride;
  constexpr int SREC = 64 * 16;
  int mt, nt;
  tile_of(blockIdx.x, gx, gy, mt, nt);
  const int n0 = nt * BN;
  const int64_t row_lo = (int64_t)mt * kBM;
  const int64_t row_hi = row_lo + kBM < M ? row_lo + kBM : M;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  const int nblk = K / 32, nks = (K + kBK - 1) / kBK;
  int64_t r = row_lo + wave * 32 + (lane & 31);
  if (r >= row_hi) r = row_hi - 1;   // clamp: loads stay in bounds, stores are masked

  v16f acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[f][e] = 0.0f;

  // the double-buffered pipeline of tile_mx: step ks computes from buffer
  // ks & 1 while the weight tile of ks + 1 goes to the other buffer and the
  // loads of ks + 2 are issued
  SlotStep a0[2], a1[2];
  WStep<NF> wn;
  const int last = nks - 1;
  load_w<NF, false>(wn, wc, ws, n0, N, K, 0, nblk);
  load_slot_mx<K1>(a0[0], p1, r, M, 0, half, nblk, K);
  load_slot_mx<K2>(a0[1], p2, r, M, 0, half, nblk, K);
  store_w<NF>(wn, lds_w, lds_s);
  load_w<NF, false>(wn, wc, ws, n0, N, K, min(1, last), nblk);
  load_slot_mx<K1>(a1[0], p1, r, M, min(1, last), half, nblk, K);
  load_slot_mx<K2>(a1[1], p2, r, M, min(1, last), half, nblk, K);
  int ks = 0;
  for (; ks + 1 < nks; ks += 2) {
    __syncthreads();
    step_slots<K1, K2>(acc, a0[0], a0[1], lds_w, lds_s, lane);
    store_w<NF>(wn, lds_w + BN * kLdsStride, lds_s + SREC);
    load_w<NF, false>(wn, wc, ws, n0, N, K, min(ks + 2, last), nblk);
    load_slot_mx<K1>(a0[0], p1, r, M, min(ks + 2, last), half, nblk, K);
    load_slot_mx<K2>(a0[1], p2, r, M, min(ks + 2, last), half, nblk, K);
    __syncthreads();
    step_slots<K1, K2>(acc, a1[0], a1[1], lds_w + BN * kLdsStride, lds_s + SREC, lane);
    store_w<NF>(wn, lds_w, lds_s);
    load_w<NF, false>(wn, wc, ws, n0, N, K, min(ks + 3, last), nblk);
    load_slot_mx<K1>(a1[0], p1, r, M, min(ks + 3, last), half, nblk, K);
    load_slot_mx<K2>(a1[1], p2, r, M, min(ks + 3, last), half, nblk, K);
  }
  if (ks < nks) {
    __syncthreads();
    step_slots<K1, K2>(acc, a0[0], a0[1], lds_w, lds_s, lane);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int col = n0 + f * 32 + (lane & 31);
    if (col >= N) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t row = row_lo + wave * 32 + 8 * (e / 4) + 4 * half + (e % 4);
      if (row < row_hi) store_out<OutT>(Y + row * ldy + col, acc[f][e]);
    }
  }
}

// NVFP4: one K step is one 32-position block; both operands are exactly
// dequantized to bf16 (see k_linear_nv).  A dense slot has two E4M3 scales
// per block (halves of 16), a sparse slot one.
struct SlotNv {
  uint4 c;      // dense: codes; sparse: codes in .x/.y, metadata in .z
  uint32_t s;   // scale byte(s)
};

template <int KIND>
__device__ __forceinline__ void load_slot_nv(SlotNv& d, const SlotBuf& b, int64_t r, int64_t R, int ks, int K) {
  if (KIND == 0) return;
  const int p = ks >> 2, j = ks & 3, wp = min(128, K - 128 * p);
  const int64_t pr = (int64_t)p * R;
  if (KIND == kSlotDense) {
    d.c = *reinterpret_cast<const uint4*>(b.c + pr * 64 + r * (wp / 2) + 16 * j);
    d.s = *reinterpret_cast<const uint16_t*>(b.s + pr * 8 + r * (wp / 16) + 2 * j);
  } else {
    const uint2 c = *reinterpret_cast<const uint2*>(b.c + pr * 32 + r * (wp / 4) + 8 * j);
    d.c = make_uint4(c.x, c.y, *reinterpret_cast<const uint32_t*>(b.m + pr * 16 + r * (wp / 8) + 4 * j), 0u);
    d.s = b.s[pr * 4 + r * (wp / 32) + j];
  }
}

// this lane's bf16 operand of sub-step t: K values 8 half + 16 t + 0..7
template <int KIND>
__device__ __forceinline__ bf16x8 slot_nv_operand(const SlotNv& a, int t, int half) {
  if (KIND == kSlotDense) {
    const uint32_t w[4] = {a.c.x, a.c.y, a.c.z, a.c.w};
    const float d = e4m3_value(t ? (a.s >> 8) & 0xFFu : a.s & 0xFFu);
    return as_bf16x8(dequant8_bf16(w[half + 2 * t], d));
  }
  const uint4 e = expand_block<KIND>(make_uint2(a.c.x, a.c.y), a.c.z);
  const uint32_t w[4] = {e.x, e.y, e.z, e.w};
  return as_bf16x8(dequant8_bf16(w[half + 2 * t], e4m3_value(a.s & 0xFFu)));
}

template <int K1, int K2>
__device__ __forceinline__ void step_slots_nv(v16f (&acc)[8], const SlotNv& a1, const SlotNv& a2, const uint8_t* lw,
                                              int lane) {
  const int half = lane >> 5, col = lane & 31;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    bf16x8 b[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) {
      const int row = f * 32 + col;
      b[f] = as_bf16x8(*reinterpret_cast<const uint4*>(lw + row * 64 + 16 * ((half + 2 * t) ^ swz_nv(row))));
    }
    if (K1 != 0) {
      const bf16x8 a = slot_nv_operand<K1>(a1, t, half);
#pragma unroll
      for (int f = 0; f < 8; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[f], acc[f], 0, 0, 0);
    }
    if (K2 != 0) {
      const bf16x8 a = slot_nv_operand<K2>(a2, t, half);
#pragma unroll
      for (int f = 0; f < 8; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b[f], acc[f], 0, 0, 0);
    }
  }
}

template <int K1, int K2, typename OutT>
__global__ __launch_bounds__(256) void k_linear_slots_nv(SlotBuf p1, SlotBuf p2, const float* ts_x, int64_t M,
                                                         const uint8_t* wc, const uint8_t* ws, const float* ts_w,
                                                         int N, int K, OutT* Y, int64_t ldy, int gx, int gy) {
  constexpr int NF = 8, BN = 256;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BN * 64];
  int mt, nt;
  tile_of(blockIdx.x, gx, gy, mt, nt);
  const int n0 = nt * BN;
  const int64_t row_lo = (int64_t)mt * kBM;
  const int64_t row_hi = row_lo + kBM < M ? row_lo + kBM : M;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, half = lane >> 5;
  const int nks = K / 32;
  int64_t r = row_lo + wave * 32 + (lane & 31);
  if (r >= row_hi) r = row_hi - 1;

  v16f acc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[f][e] = 0.0f;

  SlotNv a0[2], a1[2];
  NvW wn;
  const int last = nks - 1;
  load_nv_w<NF>(wn, wc, ws, n0, N, K, 0);
  load_slot_nv<K1>(a0[0], p1, r, M, 0, K);
  load_slot_nv<K2>(a0[1], p2, r, M, 0, K);
  store_nv_w(wn, lds);
  load_nv_w<NF>(wn, wc, ws, n0, N, K, min(1, last));
  load_slot_nv<K1>(a1[0], p1, r, M, min(1, last), K);
  load_slot_nv<K2>(a1[1], p2, r, M, min(1, last), K);
  int ks = 0;
  for (; ks + 1 < nks; ks += 2) {
    __syncthreads();
    step_slots_nv<K1, K2>(acc, a0[0], a0[1], lds, lane);
    store_nv_w(wn, lds + BN * 64);
    load_nv_w<NF>(wn, wc, ws, n0, N, K, min(ks + 2, last));
    load_slot_nv<K1>(a0[0], p1, r, M, min(ks + 2, last), K);
    load_slot_nv<K2>(a0[1], p2, r, M, min(ks + 2, last), K);
    __syncthreads();
    step_slots_nv<K1, K2>(acc, a1[0], a1[1], lds + BN * 64, lane);
    store_nv_w(wn, lds);
    load_nv_w<NF>(wn, wc, ws, n0, N, K, min(ks + 3, last));
    load_slot_nv<K1>(a1[0], p1, r, M, min(ks + 3, last), K);
    load_slot_nv<K2>(a1[1], p2, r, M, min(ks + 3, last), K);
  }
  if (ks < nks) {
    __syncthreads();
    step_slots_nv<K1, K2>(acc, a0[0], a0[1], lds, lane);
  }
  const float scale = *ts_x * *ts_w;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int col = n0 + f * 32 + (lane & 31);
    if (col >= N) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t row = row_lo + wave * 32 + 8 * (e / 4) + 4 * half + (e % 4);
      if (row < row_hi) store_out<OutT>(Y + row * ldy + col, acc[f][e] * scale);
    }
  }
}

// The small-M kernel of the formats on 16-bit MFMA (sharq_skinny16.hip).
hipError_t launch_linear_skinny16(bool nv, int pat, int ydt, const uint8_t* spc, const uint8_t* spm,
                                  const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns, const float* tsx,
                                  int64_t M, const uint8_t* wc, const uint8_t* ws, const float* tsw, int N, int K,
                                  void* Y, int64_t ldy, hipStream_t st);

// HiF4 with K a multiple of 128 (sharq_linear16.hip).
hipError_t launch_linear16_hif4(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                                const uint8_t* dnc, const uint8_t* dns, int64_t M, const uint8_t* wc,
                                const uint8_t* ws, int N, int K, void* Y, int64_t ldy, hipStream_t st);

// ---------------------------------------------------------------------------
// HiF4 two-path GEMM (2:4 backbone + dense residual).  No matrix instruction
// takes HiF4, but every HiF4 value E6M2 * 2^(E1_8 + E1_16) * S1P2 has at most
// 6 significant bits and an exponent in [-50, 17], so both operands are
// dequantized exactly to bf16 and multiplied on v_mfma_f32_32x32x16_bf16, as
// in the NVFP4 kernel (one K step = one 32-position block, the weight tile
// dequantized once per workgroup into LDS).  A unit's 4 metadata bytes
// [E6M2, E1_8, E1_16 low, E1_16 high] sit at its even block's 2-byte slots.
// ---------------------------------------------------------------------------

// The unit metadata word of block j of panel row (pr, r).
__device__ __forceinline__ uint32_t hif4_word_at(const uint8_t* sc, int64_t pr, int64_t r, int wp, int j) {
  return *reinterpret_cast<const uint32_t*>(sc + (pr * 4 + r * (wp / 32) + (j & ~1)) * 2);
}

// Eight codes (dword q of block half hb of a unit) -> eight exact bf16 values.
__device__ __forceinline__ uint4 hif4_dequant8_bf16(uint32_t codes, uint32_t word, int hb, int q) {
  const float base = e6m2_value(word & 0xFFu);
  const int l2 = 4 * hb + q, l3 = 8 * hb + 2 * q;
  const int e8 = (int)((word >> (8 + l2)) & 1u);
  const float sc0 = base * exp2_int(e8 + (int)((word >> (16 + l3)) & 1u));
  const float sc1 = base * exp2_int(e8 + (int)((word >> (17 + l3)) & 1u));
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float sc = i < 2 ? sc0 : sc1;
    const float a = s1p2_value((codes >> (8 * i)) & 0xFu, sc), b = s1p2_value((codes >> (8 * i + 4)) & 0xFu, sc);
    o[i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

struct HfA {           // one lane's activation data for one block
  uint4 dn;            // residual codes
  uint2 spc;           // compressed backbone codes
  uint32_t spm;        // backbone metadata (2:4)
  uint32_t sw, dw;     // backbone and residual unit words
};

struct HfW {           // one thread's weight row for one block
  uint4 codes;
  uint32_t word;
};

__device__ __forceinline__ void load_hf_a(HfA& s, const ARow& a, int ks, int K) {
  const int p = ks >> 2, j = ks & 3, wp = min(128, K - 128 * p);
  const int64_t pr = (int64_t)p * a.R;
  s.dn = *reinterpret_cast<const uint4*>(a.dn + pr * 64 + a.r * (wp / 2) + 16 * j);
  s.spc = *reinterpret_cast<const uint2*>(a.spc + pr * 32 + a.r * (wp / 4) + 8 * j);
  s.spm = *reinterpret_cast<const uint32_t*>(a.spm + pr * 16 + a.r * (wp / 8) + 4 * j);
  s.sw = hif4_word_at(a.sps, pr, a.r, wp, j);
  s.dw = hif4_word_at(a.dns, pr, a.r, wp, j);
}

__device__ __forceinline__ void load_hf_w(HfW& w, const uint8_t* wc, const uint8_t* ws, int n0, int N, int K, int ks) {
  const int p = ks >> 2, j = ks & 3, wp = min(128, K - 128 * p);
  const int64_t pn = (int64_t)p * N;
  const int n = min(n0 + (int)threadIdx.x, N - 1);
  w.codes = *reinterpret_cast<const uint4*>(wc + pn * 64 + (int64_t)n * (wp / 2) + 16 * j);
  w.word = hif4_word_at(ws, pn, n, wp, j);
}

__device__ __forceinline__ void store_hf_w(const HfW& w, uint8_t* lds, int hb) {
  const int row = threadIdx.x;
  const uint32_t c[4] = {w.codes.x, w.codes.y, w.codes.z, w.codes.w};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<uint4*>(lds + row * 64 + 16 * (q ^ swz_nv(row))) = hif4_dequant8_bf16(c[q], w.word, hb, q);
}

__device__ __forceinline__ void step_hf(v16f (&acc)[8], const HfA& a, int hb, const uint8_t* lw, int lane) {
  const int half = lane >> 5, col = lane & 31;
  const uint4 sp = expand_block<24>(a.spc, a.spm);
  const uint32_t spw[4] = {sp.x, sp.y, sp.z, sp.w};
  const uint32_t dnw[4] = {a.dn.x, a.dn.y, a.dn.z, a.dn.w};
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int q = half + 2 * t;   // K values 8 q .. 8 q + 7 of the block
    const bf16x8 asp = as_bf16x8(hif4_dequant8_bf16(spw[q], a.sw, hb, q));
    const bf16x8 adn = as_bf16x8(hif4_dequant8_bf16(dnw[q], a.dw, hb, q));
    bf16x8 b[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) {
      const int row = f * 32 + col;
      b[f] = as_bf16x8(*reinterpret_cast<const uint4*>(lw + row * 64 + 16 * (q ^ swz_nv(row))));
    }
#pragma unroll
    for (int f = 0; f < 8; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(asp, b[f], acc[f], 0, 0, 0);
#pragma unroll
    for (int f = 0; f < 8; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(adn, b[f], acc[f], 0, 0, 0);
  }
}

template <typename OutT>
__global__ __launch_bounds__(256) void k_linear_hif4(const uint8_t* sp_codes, const uint8_t* sp_meta,
                                                     const uint8_t* sp_scale, const uint8_t* dn_codes,
                                                     const uint8_t* dn_scale, int64_t M, const uint8_t* wc,
                                                     const uint8_t* ws, int N, int K, OutT* Y, int64_t ldy, int gx,
                                                     int gy) {
  constexpr int NF = 8, BN = 256;
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
    for (int e = 0; e < 16; ++e) acc[f][e] = 0.0f;

  // the double-buffered pipeline of k_linear_nv; block ks is half ks & 1 of its unit
  HfA a0, a1;
  HfW wn;
  const int last = nks - 1;
  load_hf_w(wn, wc, ws, n0, N, K, 0);
  load_hf_a(a0, a, 0, K);
  store_hf_w(wn, lds, 0);
  load_hf_w(wn, wc, ws, n0, N, K, min(1, last));
  load_hf_a(a1, a, min(1, last), K);
  int ks = 0;
  for (; ks + 1 < nks; ks += 2) {   // nks is even: blocks ks, ks + 1 are the halves of one unit
    __syncthreads();
    step_hf(acc, a0, 0, lds, lane);
    store_hf_w(wn, lds + BN * 64, 1);
    load_hf_w(wn, wc, ws, n0, N, K, min(ks + 2, last));
    load_hf_a(a0, a, min(ks + 2, last), K);
    __syncthreads();
    step_hf(acc, a1, 1, lds + BN * 64, lane);
    store_hf_w(wn, lds, 0);
    load_hf_w(wn, wc, ws, n0, N, K, min(ks + 3, last));
    load_hf_a(a1, a, min(ks + 3, last), K);
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int col = n0 + f * 32 + (lane & 31);
    if (col >= N) continue;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t row = row_lo + wave * 32 + 8 * (e / 4) + 4 * half + (e % 4);
      if (row < row_hi) store_out<OutT>(Y + row * ldy + col, acc[f][e]);
    }
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------

template <int NF, int PAT, bool SDW, typename OutT>
static hipError_t go_linear(const uint8_t* spc, const uint8_t* spm, const uint8_t* sps, const uint8_t* dnc,
                            const uint8_t* dns, int64_t M, const uint8_t* wc, const uint8_t* ws, int N, int K,
                            void* Y, int64_t ldy, hipStream_t st) {
  const int gx = (N + 32 * NF - 1) / (32 * NF), gy = (int)((M + kBM - 1) / kBM);
  if constexpr (SDW && NF == 8) {
    const PersistPlan pl = persist_plan(gx, gy);
    const auto kernel = K % kBK == 0 ? k_linear_mx_persist<PAT, OutT, false>
                                     : k_linear_mx_persist<PAT, OutT, PAT != 0>;
    kernel<<<dim3((unsigned)pl.grid), dim3(256), 0, st>>>(spc, spm, sps, dnc, dns, M, wc, ws, N, K,
                                                          reinterpret_cast<OutT*>(Y), ldy, gx, gy, pl.full, pl.halves);
  } else {
    k_linear_mx<NF, PAT, SDW, OutT><<<dim3((unsigned)(gx * gy)), dim3(256), 0, st>>>(
        spc, spm, sps, dnc, dns, M, wc, ws, N, K, reinterpret_cast<OutT*>(Y), ldy, gx, gy);
  }
  return hipGetLastError();
}

template <int NF, int PAT, bool SDW>
static hipError_t go_linear_dt(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                               const uint8_t* dnc, const uint8_t* dns, int64_t M, const uint8_t* wc,
                               const uint8_t* ws, int N, int K, void* Y, int64_t ldy, hipStream_t st) {
  if (ydt == 2) return go_linear<NF, PAT, SDW, float>(spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
  if (ydt == 1) return go_linear<NF, PAT, SDW, _Float16>(spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
  return go_linear<NF, PAT, SDW, uint16_t>(spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
}

// The persistent interleaved kernel on a dense backbone copy (pattern 0).
template <typename OutT>
static hipError_t go_dense_backbone(const uint8_t* spd, const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns,
                                    int64_t M, const uint8_t* wc, const uint8_t* ws, int N, int K, void* Y,
                                    int64_t ldy, hipStream_t st) {
  const int gx = (N + 255) / 256, gy = (int)((M + kBM - 1) / kBM);
  const PersistPlan pl = persist_plan(gx, gy);
  k_linear_mx_persist<0, OutT, false><<<dim3((unsigned)pl.grid), dim3(256), 0, st>>>(
      spd, nullptr, sps, dnc, dns, M, wc, ws, N, K, reinterpret_cast<OutT*>(Y), ldy, gx, gy, pl.full, pl.halves);
  return hipGetLastError();
}

// The 8-wavefront kernel on a dense backbone copy (sharq_mx8.hip).
hipError_t launch_linear_mx8(int ydt, const uint8_t* spd, const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns,
                             int64_t M, const uint8_t* wc, const uint8_t* ws, int N, int K, void* Y, int64_t ldy,
                             hipStream_t st);

// spd (optional): the backbone's dense copy; used by the main kernels (K a
// multiple of 128, M beyond the small-M kernel's range), which then skip the
// expansion, and by the small-M kernel when it is the only form.
hipError_t launch_linear_mx(int pat, int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                            const uint8_t* dnc, const uint8_t* dns, int64_t M, const uint8_t* wc, const uint8_t* ws,
                            int N, int K, void* Y, int64_t ldy, const uint8_t* spd, hipStream_t st) {
  const bool sdw = K >= kBK;   // at least one full panel
  constexpr int NF = 8;
  const bool dense = spd && K % kBK == 0;
  const bool skinny = use_skinny(M, N, K, backbone_form(spc ? pat : 0), backbone_form(dense ? 0 : pat), device_cus());
  if (dense && !skinny) {
    if (use_mx8(M, N, device_cus())) return launch_linear_mx8(ydt, spd, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
    if (ydt == 2) return go_dense_backbone<float>(spd, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
    if (ydt == 1) return go_dense_backbone<_Float16>(spd, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
    return go_dense_backbone<uint16_t>(spd, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
  }
  if (skinny) {
    if (spc == nullptr)   // the backbone exists as its dense copy only
      return go_skinny_m<0>(SkinnyArgs{spd, nullptr, sps, dnc, dns, wc, ws, M, N, K}, Y, ydt, ldy, st);
    const SkinnyArgs p{spc, spm, sps, dnc, dns, wc, ws, M, N, K};
    return pat == 24 ? go_skinny_m<24>(p, Y, ydt, ldy, st) : go_skinny_m<48>(p, Y, ydt, ldy, st);
  }
  if (spc == nullptr) return hipErrorInvalidValue;   // rejected by the C ABI (K not a multiple of 128)
  if (pat == 24) {
    return sdw ? go_linear_dt<NF, 24, true>(ydt, spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st)
               : go_linear_dt<NF, 24, false>(ydt, spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
  }
  return sdw ? go_linear_dt<NF, 48, true>(ydt, spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st)
             : go_linear_dt<NF, 48, false>(ydt, spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
}

template <int MF, int NB, int KS, int PAT>
static hipError_t go_grouped_skinny(const SkinnyArgs& p, const int32_t* ridx, const int32_t* offs, int E,
                                    int64_t total, void* Y, int ydt, int64_t ldy, hipStream_t st) {
  const int ncg = (p.N + 16 * NB - 1) / (16 * NB);
  const int extra = (int)(total / (16 * MF));
  const dim3 grid((unsigned)ncg * (unsigned)(E + extra)), block(64 * KS);
  if constexpr (PAT != 0) {
    if (p.K % kBK != 0) {
      k_linear_mx_grouped_skinny<MF, NB, KS, PAT, true><<<grid, block, 0, st>>>(p, ridx, offs, E, extra, Y, ydt, ldy, ncg);
      return hipGetLastError();
    }
  }
  k_linear_mx_grouped_skinny<MF, NB, KS, PAT, false><<<grid, block, 0, st>>>(p, ridx, offs, E, extra, Y, ydt, ldy, ncg);
  return hipGetLastError();
}

template <int PAT>
static hipError_t go_grouped_skinny_cfg(const SkinnyArgs& p, const int32_t* ridx, const int32_t* offs, int E,
                                        int64_t total, void* Y, int ydt, int64_t ldy, hipStream_t st) {
  const GroupedCfg c = grouped_cfg(total, E, p.N, p.K, device_cus());
  if (c.nb == 2) return go_grouped_skinny<1, 2, 4, PAT>(p, ridx, offs, E, total, Y, ydt, ldy, st);
  if (c.ks == 2) return go_grouped_skinny<1, 4, 2, PAT>(p, ridx, offs, E, total, Y, ydt, ldy, st);
  return go_grouped_skinny<1, 4, 4, PAT>(p, ridx, offs, E, total, Y, ydt, ldy, st);
}

template <int NF, int PAT, bool SDW, typename OutT>
static hipError_t go_grouped(const uint8_t* spc, const uint8_t* spm, const uint8_t* sps, const uint8_t* dnc,
                             const uint8_t* dns, const int32_t* ridx, int64_t act_rows, const int32_t* offs, int E,
                             int64_t total, const uint8_t* wc, const uint8_t* ws, int N, int K, void* Y, int64_t ldy,
                             hipStream_t st) {
  // upper bound on the number of 128-row tiles over all experts
  const int64_t items = (total + kBM - 1) / kBM + E;
  const int gx = (N + 32 * NF - 1) / (32 * NF);
  if ((int64_t)gx * items > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  if constexpr (SDW && NF == 8) {
    const int64_t bound = (int64_t)gx * items, cus = device_cus();
    const unsigned g = (unsigned)(bound < cus ? bound : cus);
    constexpr bool kTail = PAT != 0;   // the dense backbone copy needs K a multiple of 128
    const bool tail = K % kBK != 0;
    const auto kernel = ridx ? (tail ? k_linear_mx_grouped_persist<PAT, OutT, kTail, true>
                                     : k_linear_mx_grouped_persist<PAT, OutT, false, true>)
                             : (tail ? k_linear_mx_grouped_persist<PAT, OutT, kTail, false>
                                     : k_linear_mx_grouped_persist<PAT, OutT, false, false>);
    kernel<<<dim3(g), dim3(256), 0, st>>>(spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, wc, ws, N, K,
                                          reinterpret_cast<OutT*>(Y), ldy, gx);
    return hipGetLastError();
  }
  dim3 grid((unsigned)(gx * items)), block(256);
  k_linear_mx_grouped<NF, PAT, SDW, OutT><<<grid, block, 0, st>>>(spc, spm, sps, dnc, dns, ridx, act_rows, offs, E,
                                                                  wc, ws, N, K, reinterpret_cast<OutT*>(Y), ldy, gx);
  return hipGetLastError();
}

template <int NF, int PAT, bool SDW>
static hipError_t go_grouped_dt(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                                const uint8_t* dnc, const uint8_t* dns, const int32_t* ridx, int64_t act_rows,
                                const int32_t* offs, int E, int64_t total, const uint8_t* wc, const uint8_t* ws, int N,
                                int K, void* Y, int64_t ldy, hipStream_t st) {
  if (ydt == 2)
    return go_grouped<NF, PAT, SDW, float>(spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y, ldy, st);
  if (ydt == 1)
    return go_grouped<NF, PAT, SDW, _Float16>(spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y, ldy,
                                              st);
  return go_grouped<NF, PAT, SDW, uint16_t>(spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y, ldy,
                                            st);
}

// spd (optional): the backbone's dense copy, read instead of expanding the
// compressed backbone when K is a multiple of 128.
hipError_t launch_linear_mx_grouped(int pat, int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps,
                                    const uint8_t* dnc, const uint8_t* dns, const int32_t* ridx, int64_t act_rows,
                                    const int32_t* offs, int E, int64_t total, const uint8_t* wc, const uint8_t* ws,
                                    int N, int K, void* Y, int64_t ldy, const uint8_t* spd, hipStream_t st) {
  // at least one full panel, and every expert's scales at a multiple of 4
  // bytes (K not a multiple of 128 can leave them anywhere), as the
  // interleaved pipeline's loads need
  const bool sdw = K >= kBK && ((int64_t)N * (K / 32)) % 4 == 0;
  constexpr int NF = 8;
  if (use_grouped_skinny(total, E, N, device_cus())) {
    if (spd && K % kBK == 0)
      return go_grouped_skinny_cfg<0>(SkinnyArgs{spd, nullptr, sps, dnc, dns, wc, ws, act_rows, N, K}, ridx, offs, E,
                                      total, Y, ydt, ldy, st);
    const SkinnyArgs p{spc, spm, sps, dnc, dns, wc, ws, act_rows, N, K};
    return pat == 24 ? go_grouped_skinny_cfg<24>(p, ridx, offs, E, total, Y, ydt, ldy, st)
                     : go_grouped_skinny_cfg<48>(p, ridx, offs, E, total, Y, ydt, ldy, st);
  }
  if (spd && K % kBK == 0)
    return go_grouped_dt<NF, 0, true>(ydt, spd, nullptr, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K,
                                      Y, ldy, st);
  if (pat == 24) {
    return sdw ? go_grouped_dt<NF, 24, true>(ydt, spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y,
                                             ldy, st)
               : go_grouped_dt<NF, 24, false>(ydt, spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y,
                                              ldy, st);
  }
  return sdw ? go_grouped_dt<NF, 48, true>(ydt, spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y, ldy,
                                           st)
             : go_grouped_dt<NF, 48, false>(ydt, spc, spm, sps, dnc, dns, ridx, act_rows, offs, E, total, wc, ws, N, K, Y, ldy,
                                            st);
}

template <int K1, int K2, typename OutT>
static hipError_t go_slots(bool nv, const SlotBuf& p1, const SlotBuf& p2, const float* tsx, int64_t M,
                           const uint8_t* wc, const uint8_t* ws, const float* tsw, int N, int K, void* Y, int64_t ldy,
                           hipStream_t st) {
  const int gx = (N + 255) / 256, gy = (int)((M + kBM - 1) / kBM);
  const dim3 grid((unsigned)(gx * gy)), block(256);
  if (nv)
    k_linear_slots_nv<K1, K2, OutT><<<grid, block, 0, st>>>(p1, p2, tsx, M, wc, ws, tsw, N, K,
                                                            reinterpret_cast<OutT*>(Y), ldy, gx, gy);
  else
    k_linear_slots_mx<K1, K2, OutT><<<grid, block, 0, st>>>(p1, p2, M, wc, ws, N, K, reinterpret_cast<OutT*>(Y), ldy,
                                                            gx, gy);
  return hipGetLastError();
}

template <int K1, int K2>
static hipError_t go_slots_dt(int ydt, bool nv, const SlotBuf& p1, const SlotBuf& p2, const float* tsx, int64_t M,
                              const uint8_t* wc, const uint8_t* ws, const float* tsw, int N, int K, void* Y,
                              int64_t ldy, hipStream_t st) {
  if (ydt == 2) return go_slots<K1, K2, float>(nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
  if (ydt == 1) return go_slots<K1, K2, _Float16>(nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
  return go_slots<K1, K2, uint16_t>(nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
}

// Path combinations (modes 1-4 of the C interface): 1 sparse, 2 dense (RTN),
// 3 dense + dense, 4 sparse + sparse.  pat: 24 or 48 (the sparse metadata
// layout).  nv: NVFP4 (the weight's sparse view `ws` serves every path: its
// per-16 dense view holds the same values).
hipError_t launch_linear_slots(int mode, int pat, int ydt, bool nv, const uint8_t* c1, const uint8_t* m1,
                               const uint8_t* s1, const uint8_t* c2, const uint8_t* m2, const uint8_t* s2,
                               const float* tsx, int64_t M, const uint8_t* wc, const uint8_t* ws, const float* tsw,
                               int N, int K, void* Y, int64_t ldy, hipStream_t st) {
  const SlotBuf p1{c1, m1, s1}, p2{c2, m2, s2};
  const bool p24 = pat == 24;
  switch (mode) {
    case 1: return p24 ? go_slots_dt<24, 0>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st)
                       : go_slots_dt<48, 0>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
    case 2: return go_slots_dt<0, kSlotDense>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
    case 3: return go_slots_dt<kSlotDense, kSlotDense>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
    case 4: return p24 ? go_slots_dt<24, 24>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st)
                       : go_slots_dt<48, 48>(ydt, nv, p1, p2, tsx, M, wc, ws, tsw, N, K, Y, ldy, st);
    default: return hipErrorInvalidValue;
  }
}

// HiF4 (2:4 backbone, K a multiple of 64).
hipError_t launch_linear_hif4(int ydt, const uint8_t* spc, const uint8_t* spm, const uint8_t* sps, const uint8_t* dnc,
                              const uint8_t* dns, int64_t M, const uint8_t* wc, const uint8_t* ws, int N, int K,
                              void* Y, int64_t ldy, hipStream_t st) {
  if (use_skinny16(M, N, K, form16(false, 24), device_cus()))
    return launch_linear_skinny16(false, 24, ydt, spc, spm, sps, dnc, dns, nullptr, M, wc, ws, nullptr, N, K, Y, ldy,
                                  st);
  if (K % kBK == 0) return launch_linear16_hif4(ydt, spc, spm, sps, dnc, dns, M, wc, ws, N, K, Y, ldy, st);
  const int gx = (N + 255) / 256, gy = (int)((M + kBM - 1) / kBM);
  const dim3 grid((unsigned)(gx * gy)), block(256);
  if (ydt == 2)
    k_linear_hif4<float><<<grid, block, 0, st>>>(spc, spm, sps, dnc, dns, M, wc, ws, N, K,
                                                 reinterpret_cast<float*>(Y), ldy, gx, gy);
  else if (ydt == 1)
    k_linear_hif4<_Float16><<<grid, block, 0, st>>>(spc, spm, sps, dnc, dns, M, wc, ws, N, K,
                                                    reinterpret_cast<_Float16*>(Y), ldy, gx, gy);
  else
    k_linear_hif4<uint16_t><<<grid, block, 0, st>>>(spc, spm, sps, dnc, dns, M, wc, ws, N, K,
                                                    reinterpret_cast<uint16_t*>(Y), ldy, gx, gy);
  return hipGetLastError();
}

}  // namespace sharq
