// Small-M NVFP4 and HiF4 two-path GEMM for gfx950 (decode; SharQ Sec. 3.3
// eq. "sharq-output", Sec. 3.4 "Residual path compensation by accumulation").
//
// The block scales of both formats are not powers of two, so, as in the
// prefill kernels, both operands are dequantized exactly (NVFP4 to fp16, HiF4
// to bf16) and multiplied on 16-bit MFMA.  With few rows the layer streams its
// weight: the floor is the weight's bytes (0.53 or 0.56 per value), and the
// 128 x 256 prefill tile leaves most CUs idle (N = 4096 has 16 such tiles).
// As in the MXFP4 small-M kernel a workgroup therefore owns 16 NB output
// columns and 16 MF rows, and its KS wavefronts split K, each streaming its
// weight panels straight from HBM into MFMA operands with a two-deep register
// prefetch; the KS partial tiles are added in LDS in a fixed order.
//
// v_mfma_f32_16x16x32_{f16,bf16}: lane l holds row / column l % 16 and 8 K
// values of group l / 16; accumulator element r of lane l is row 4 (l / 16) +
// r of the first operand and column l % 16 of the second.  Which 8 positions a
// group holds is free as long as both operands agree: group j takes block j of
// the 128-wide panel, and MFMA t of a panel its dword t (positions 32 j + 8 t
// ..+7), so a lane needs one 16-byte load and one scale per block.
//
// Any K the formats allow: in a last panel narrower than 128, lanes whose
// block lies past K reread block 0 and zero its weight codes.

#include "sharq_tile.hpp"

namespace sharq {

typedef float v4f_s __attribute__((ext_vector_type(4)));

constexpr int kFmtNv = 0, kFmtHf = 1;

template <int MF, int NB>
struct Skinny16Stage {
  uint4 w[NB];          // weight codes: column 16 n + l % 16, block l / 16
  uint32_t ws[NB];      // NVFP4: their E4M3 scale; HiF4: the unit's metadata word
  uint4 dn[MF];         // residual codes of row 16 m + l % 16, block l / 16
  uint4 sp[MF];         // backbone: dense codes (PAT 0), or codes (x, y) and metadata (z)
  uint32_t sdn[MF];     // NVFP4: two E4M3 scales (bytes 0, 1); HiF4: the unit's word
  uint32_t ssp[MF];     // NVFP4: one E4M3 scale; HiF4: the unit's word
};

struct Skinny16Args {
  const uint8_t *spc, *spm, *sps, *dnc, *dns, *wc, *ws;
  int64_t M;
  int N, K;
};

template <int FMT, int MF, int NB, int PAT, bool RAG>
__device__ __forceinline__ void s16_load(Skinny16Stage<MF, NB>& st, const Skinny16Args& p, int64_t r0, int n0, int ks,
                                         int lane) {
  const int wp = RAG ? min(128, p.K - 128 * ks) : 128;   // width of this panel
  const int j = RAG && 32 * (lane >> 4) >= wp ? 0 : lane >> 4;
  const int nb = wp >> 5;                                // its blocks
  const int64_t pn = (int64_t)ks * p.N * 4, pm = (int64_t)ks * p.M * 4;   // blocks before this panel
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int col = min(n0 + 16 * n + (lane & 15), p.N - 1);
    const int64_t V = pn + (int64_t)col * nb + j;
    st.w[n] = *reinterpret_cast<const uint4*>(p.wc + V * 16);
    if (FMT == kFmtNv) st.ws[n] = p.ws[V];
    else st.ws[n] = *reinterpret_cast<const uint32_t*>(p.ws + (V - (j & 1)) * 2);
  }
#pragma unroll
  for (int m = 0; m < MF; ++m) {
    int64_t row = r0 + 16 * m + (lane & 15);
    if (row >= p.M) row = p.M - 1;
    const int64_t V = pm + row * nb + j;
    st.dn[m] = *reinterpret_cast<const uint4*>(p.dnc + V * 16);
    if (PAT == 0) {
      st.sp[m] = *reinterpret_cast<const uint4*>(p.spc + V * 16);
    } else {
      const uint2 c = *reinterpret_cast<const uint2*>(p.spc + V * 8);
      st.sp[m].x = c.x;
      st.sp[m].y = c.y;
      st.sp[m].z = *reinterpret_cast<const uint32_t*>(p.spm + V * 4);
    }
    if (FMT == kFmtNv) {
      st.sdn[m] = *reinterpret_cast<const uint16_t*>(p.dns + V * 2);
      st.ssp[m] = p.sps[V];
    } else {
      st.sdn[m] = *reinterpret_cast<const uint32_t*>(p.dns + (V - (j & 1)) * 2);
      st.ssp[m] = *reinterpret_cast<const uint32_t*>(p.sps + (V - (j & 1)) * 2);
    }
  }
}

__device__ __forceinline__ uint32_t dword_of(const uint4& q, int t) {
  return t == 0 ? q.x : t == 1 ? q.y : t == 2 ? q.z : q.w;
}

template <int FMT>
__device__ __forceinline__ v4f_s s16_mma(const uint4& b, const uint4& a, v4f_s c) {
  if constexpr (FMT == kFmtNv) return __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(b), as_f16x8(a), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b), as_bf16x8(a), c, 0, 0, 0);
}

// Per MFMA t: the weight operands of the NB fragments, then both paths of
// every row fragment against them.
template <int FMT, int MF, int NB, int PAT, bool RAG>
__device__ __forceinline__ void s16_step(v4f_s (&acc)[MF][NB], const Skinny16Stage<MF, NB>& st, int K, int ks,
                                         int lane) {
  const int j = lane >> 4;
  const int hb = j & 1;   // HiF4: which half of its unit the lane's block is
  const uint32_t wmask = RAG && 32 * j >= K - 128 * ks ? 0u : ~0u;
  uint4 sp[MF];
#pragma unroll
  for (int m = 0; m < MF; ++m)
    sp[m] = PAT == 0 ? st.sp[m] : expand_block<PAT == 0 ? 24 : PAT>(make_uint2(st.sp[m].x, st.sp[m].y), st.sp[m].z);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    uint4 b[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      uint32_t c = dword_of(st.w[n], t);
      if (RAG) c &= wmask;
      b[n] = FMT == kFmtNv ? nv_dequant8(c, nv_scale2(st.ws[n])) : hf_dequant8(c, hf_scales(st.ws[n], hb, t));
    }
#pragma unroll
    for (int m = 0; m < MF; ++m) {
      uint4 a, d;
      if (FMT == kFmtNv) {
        a = nv_dequant8(dword_of(sp[m], t), nv_scale2(st.ssp[m]));
        d = nv_dequant8(dword_of(st.dn[m], t), nv_scale2((st.sdn[m] >> (8 * (t >> 1))) & 0xFFu));
      } else {
        a = hf_dequant8(dword_of(sp[m], t), hf_scales(st.ssp[m], hb, t));
        d = hf_dequant8(dword_of(st.dn[m], t), hf_scales(st.sdn[m], hb, t));
      }
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[m][n] = s16_mma<FMT>(b[n], a, acc[m][n]);
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[m][n] = s16_mma<FMT>(b[n], d, acc[m][n]);
    }
  }
}

template <int FMT, int MF, int NB, int KS, int PAT, bool RAG>
__global__ __launch_bounds__(64 * KS) void k_linear_skinny16(Skinny16Args p, const float* ts_x, const float* ts_w,
                                                             void* Y, int ydt, int64_t ldy, int ncg, int nrt) {
  __shared__ float part[KS][MF * NB][256];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // the row tiles of one column group follow each other on one XCD (workgroups
  // are dealt round-robin over the 8) and share the weight panels in its L2
  int cg = blockIdx.x, rt = 0;
  if (nrt > 1) {
    const int total = ncg * nrt, id = blockIdx.x;
    const int idp = (total & 7) == 0 ? (id & 7) * (total >> 3) + (id >> 3) : id;
    cg = idp / nrt;
    rt = idp - cg * nrt;
  }
  const int n0 = cg * 16 * NB;
  const int64_t r0 = (int64_t)rt * 16 * MF;
  const int nks = (p.K + 127) >> 7;
  const int per = (nks + KS - 1) / KS;
  const int k0 = wave * per, k1 = min(nks, k0 + per);

  v4f_s acc[MF][NB];
#pragma unroll
  for (int m = 0; m < MF; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[m][n] = v4f_s{0.0f, 0.0f, 0.0f, 0.0f};

  Skinny16Stage<MF, NB> s0, s1;
  if (k0 < k1) s16_load<FMT, MF, NB, PAT, RAG>(s0, p, r0, n0, k0, lane);
  if (k0 + 1 < k1) s16_load<FMT, MF, NB, PAT, RAG>(s1, p, r0, n0, k0 + 1, lane);
  int ks = k0;
  for (; ks + 1 < k1; ks += 2) {
    s16_step<FMT, MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);
    if (ks + 2 < k1) s16_load<FMT, MF, NB, PAT, RAG>(s0, p, r0, n0, ks + 2, lane);
    s16_step<FMT, MF, NB, PAT, RAG>(acc, s1, p.K, ks + 1, lane);
    if (ks + 3 < k1) s16_load<FMT, MF, NB, PAT, RAG>(s1, p, r0, n0, ks + 3, lane);
  }
  if (ks < k1) s16_step<FMT, MF, NB, PAT, RAG>(acc, s0, p.K, ks, lane);

  // the KS partial tiles, added by all threads in the order of K
#pragma unroll
  for (int m = 0; m < MF; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n)
      *reinterpret_cast<v4f_s*>(&part[wave][m * NB + n][4 * lane]) = acc[m][n];
  __syncthreads();
  const float scale = FMT == kFmtNv ? *ts_x * *ts_w : 1.0f;
  for (int q = tid; q < MF * NB * 256; q += 64 * KS) {
    const int f = q >> 8, e = q & 255, m = f / NB, n = f - m * NB;
    const int r = e >> 4, c = e & 15;                      // row and column of the fragment
    const int at = 64 * (c >> 2) + 4 * r + (c & 3);        // its place in the accumulator layout
    float v = part[0][f][at];
    for (int w = 1; w < KS; ++w) v += part[w][f][at];
    if (FMT == kFmtNv) v *= scale;
    const int64_t row = r0 + 16 * m + r;
    const int col = n0 + 16 * n + c;
    if (row < p.M && col < p.N) {
      if (ydt == 2) reinterpret_cast<float*>(Y)[row * ldy + col] = v;
      else if (ydt == 1) reinterpret_cast<_Float16*>(Y)[row * ldy + col] = (_Float16)v;
      else reinterpret_cast<uint16_t*>(Y)[row * ldy + col] = f32_to_bf16_rne(v);
    }
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

template <int FMT, int MF, int NB, int KS, int PAT>
static hipError_t go_s16(const Skinny16Args& p, const float* tsx, const float* tsw, void* Y, int ydt, int64_t ldy,
                         hipStream_t st) {
  const int ncg = (p.N + 16 * NB - 1) / (16 * NB);
  const int nrt = (int)((p.M + 16 * MF - 1) / (16 * MF));
  if constexpr (PAT != 0) {
    if (p.K % 128 != 0) {
      k_linear_skinny16<FMT, MF, NB, KS, PAT, true>
          <<<dim3((unsigned)(ncg * nrt)), dim3(64 * KS), 0, st>>>(p, tsx, tsw, Y, ydt, ldy, ncg, nrt);
      return hipGetLastError();
    }
  }
  k_linear_skinny16<FMT, MF, NB, KS, PAT, false>
      <<<dim3((unsigned)(ncg * nrt)), dim3(64 * KS), 0, st>>>(p, tsx, tsw, Y, ydt, ldy, ncg, nrt);
  return hipGetLastError();
}

// (row fragments, column fragments, K splits).  Up to 32 rows, column fragments:
// as many as leave at least 192 workgroups, since every activation block loaded
// and dequantized then feeds more weight columns; up to 16 rows the K split of
// the MXFP4 kernel (about 8192 weight streams in flight, at least 4 panels per
// wavefront).  Measured with the weight streamed from HBM, us for (N, K) =
// (6144, 4096) / (28672, 4096) / (4096, 14336) / (1024, 4096), M = 16, NVFP4:
// (1,1,16) 8.0/28.7/11.2/4.6, (1,2,8) 6.2/19.1/15.5/5.6, (1,4,4) 11.4/17.9/29.9/10.7,
// where the 128 x 256 prefill tile took 92/109/298/89.
struct S16Cfg {
  int mf, nb, ks;
};

static S16Cfg s16_config(int form, int64_t M, int N, int K) {
  if (M > 32) {
    const Wide16 w = wide16(M, N, K, form, device_cus());
    return {w.mf, w.nb, w.ks};
  }
  const int mf = M <= 16 ? 1 : 2;
  int nb = 4;
  while (nb > 1 && (N + 16 * nb - 1) / (16 * nb) < 192) nb >>= 1;
  if (mf > 1) return {mf, nb, nb == 4 ? 4 : 8};
  const int nks = (K + 127) / 128, cap = nb == 4 ? 8 : 16, streams = (N + 15) / 16;
  int ks = 4;
  while (ks < cap && streams * ks * 2 <= 8192 && nks >= 4 * ks * 2) ks *= 2;
  return {mf, nb, ks};
}

template <int FMT, int PAT>
static hipError_t go_s16_cfg(const Skinny16Args& p, const float* tsx, const float* tsw, void* Y, int ydt, int64_t ldy,
                             hipStream_t st, S16Cfg c) {
#define SHARQ_S16(MF_, NB_, KS_) \
  if (c.mf == MF_ && c.nb == NB_ && c.ks == KS_) return go_s16<FMT, MF_, NB_, KS_, PAT>(p, tsx, tsw, Y, ydt, ldy, st);
  SHARQ_S16(1, 1, 4) SHARQ_S16(1, 1, 8) SHARQ_S16(1, 1, 16)
  SHARQ_S16(1, 2, 4) SHARQ_S16(1, 2, 8) SHARQ_S16(1, 2, 16)
  SHARQ_S16(1, 4, 4) SHARQ_S16(1, 4, 8)
  SHARQ_S16(2, 1, 8) SHARQ_S16(2, 2, 8) SHARQ_S16(2, 4, 4)
  if constexpr (FMT == kFmtHf || PAT == 48) { SHARQ_S16(4, 4, 4) }
#undef SHARQ_S16
  return hipErrorInvalidValue;   // unreachable: s16_config gives one of the above
}

hipError_t launch_linear_skinny16(bool nv, int pat, int ydt, const uint8_t* spc, const uint8_t* spm,
                                  const uint8_t* sps, const uint8_t* dnc, const uint8_t* dns, const float* tsx,
                                  int64_t M, const uint8_t* wc, const uint8_t* ws, const float* tsw, int N, int K,
                                  void* Y, int64_t ldy, hipStream_t st) {
  const Skinny16Args p{spc, spm, sps, dnc, dns, wc, ws, M, N, K};
  const S16Cfg c = s16_config(form16(nv, pat), M, N, K);
  if (!nv) return go_s16_cfg<kFmtHf, 24>(p, tsx, tsw, Y, ydt, ldy, st, c);
  if (pat == 0) return go_s16_cfg<kFmtNv, 0>(p, tsx, tsw, Y, ydt, ldy, st, c);
  if (pat == 24) return go_s16_cfg<kFmtNv, 24>(p, tsx, tsw, Y, ydt, ldy, st, c);
  return go_s16_cfg<kFmtNv, 48>(p, tsx, tsw, Y, ydt, ldy, st, c);
}

}  // namespace sharq
