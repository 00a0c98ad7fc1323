// HIP kernels for gfx950 (CDNA4): shared-prefix continuous-sampling decode.
//
// One launch per layer-step does all the device work of that layer:
//   * append: each live slot's new K/V row goes into its response pages;
//   * split-K attention over the shared prefix: one work-group per
//     (prompt, KV head, prefix chunk: 128 tokens on MFMA tiles, `split`
//     tokens otherwise).  Every K/V byte of the chunk is read from HBM once
//     and used by all m * hpk query rows of that
//     KV head -- the rows of every live slot of the prompt.  With >= 16 rows
//     the two contractions run on MFMA tiles (v_mfma_f32_16x16x32_bf16);
//     below that, and in fp32, on one 16-row tile per wavefront over plain rows;
//   * split-K attention over each live slot's private response (hpk rows per
//     KV byte): MFMA tiles for bf16 and E4M3 pages, row tiles or wavefront dot
//     products for fp32 pages;
//   * log-sum-exp merge: one work-group per live (slot, KV head), placed at
//     the end of the grid, waits (bounded) until every chunk of that slot has
//     published its partial, combines the partial softmaxes and writes O.
// Short responses and their merges take a wavefront each, four to a work-group,
// where the launch would not fit the GPU at once (StepArgs::resp_cut).
// Idle slots get O = 0.
//
// A partial over a key set J is (M, L, O) with scores in log2 units
// (s_j = scale * log2(e) * q.k_j): M = max_j s_j, L = sum_j 2^(s_j - M),
// O = sum_j 2^(s_j - M) v_j.  Two partials combine exactly as
// M = max(M1, M2), L = 2^(M1-M) L1 + 2^(M2-M) L2, O likewise, and the result
// is O / L.
//
// This header holds the device code; every kernel translation unit includes it
// and instantiates the shapes it serves (its copies have internal linkage).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.h"

namespace infs {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

#define NEG_INF (-__builtin_huge_valf())

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Lane permutations inside 16-lane DPP rows (row_mask = bank_mask = all).
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Sum over each aligned group of N consecutive lanes; every lane gets its group's sum.
template <int N>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(N == 2 || N == 4 || N == 8 || N == 16 || N == 32 || N == 64, "group size");
  x += dpp<0xB1>(x);                       // quad_perm [1,0,3,2]: lane ^ 1
  if constexpr (N >= 4) x += dpp<0x4E>(x); // quad_perm [2,3,0,1]: lane ^ 2
  if constexpr (N == 8) x += dpp<0x141>(x);  // row_half_mirror: quad 0 <-> quad 1
  if constexpr (N >= 16) {
    x += dpp<0x124>(x);                    // row_ror:4
    x += dpp<0x128>(x);                    // row_ror:8
  }
  if constexpr (N >= 32) x += __shfl_xor(x, 16);
  if constexpr (N >= 64) x += __shfl_xor(x, 32);
  return x;
}

// Combine partial (m2, l2) into (m, l); returns the weights of the old and new parts.
__device__ __forceinline__ void lse_combine(float& m, float& l, float m2, float l2, float& a, float& b) {
  const float mn = fmaxf(m, m2);
  const float mu = (mn == NEG_INF) ? 0.f : mn;
  a = exp2_fast(m - mu);
  b = exp2_fast(m2 - mu);
  l = l * a + l2 * b;
  m = mn;
}

// 16-byte chunk helpers: 8 bf16 or 4 fp32 elements.
template <bool BF>
__device__ __forceinline__ float dot16B(const u32x4& k, const u32x4& q) {
  if constexpr (BF) {
    // Pairs are taken with shufflevector from a whole-vector cast: casting the
    // individual 32-bit lanes to bf16x2 is mis-lowered by this compiler (all
    // four dots read the same dword).
    const bf16x8 kv = __builtin_bit_cast(bf16x8, k), qv = __builtin_bit_cast(bf16x8, q);
    float s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kv, kv, 0, 1), __builtin_shufflevector(qv, qv, 0, 1), 0.f, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kv, kv, 2, 3), __builtin_shufflevector(qv, qv, 2, 3), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kv, kv, 4, 5), __builtin_shufflevector(qv, qv, 4, 5), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kv, kv, 6, 7), __builtin_shufflevector(qv, qv, 6, 7), s, false);
    return s;
  } else {
    float s = __uint_as_float(k.x) * __uint_as_float(q.x);
    s = fmaf(__uint_as_float(k.y), __uint_as_float(q.y), s);
    s = fmaf(__uint_as_float(k.z), __uint_as_float(q.z), s);
    s = fmaf(__uint_as_float(k.w), __uint_as_float(q.w), s);
    return s;
  }
}

__device__ __forceinline__ void axpy16B(float* o, float p, const u32x4& v) {
  o[0] = fmaf(p, __uint_as_float(v.x), o[0]); o[1] = fmaf(p, __uint_as_float(v.y), o[1]);
  o[2] = fmaf(p, __uint_as_float(v.z), o[2]); o[3] = fmaf(p, __uint_as_float(v.w), o[3]);
}

// Compile-time shape of one kernel instantiation.
template <bool BF_, int D_, int HPK_, bool MFMA_, int PR_, bool KV8_ = false>
struct Shape {
  static constexpr bool BF = BF_;
  // KV8: the prefix store and the pages hold K/V as E4M3 bytes; the kernels
  // widen them to bf16 in registers (exact) and compute as for bf16.
  static constexpr bool KV8 = KV8_;
  static constexpr int D = D_;
  static constexpr int HPK = HPK_;
  static constexpr bool MFMA = MFMA_;
  static constexpr int PR = PR_;                  // prefix rows per record group (padded)
  static constexpr int ES = BF ? 2 : 4;            // element bytes
  static constexpr int EPL = 16 / ES;              // elements per lane chunk
  static constexpr int ROWB = D * ES;              // bytes of one K or V row of one head
  static constexpr int LPT = ROWB / 16;            // lanes per token (16-byte units of a row)
  static constexpr int TPI = 64 / LPT;             // tokens per load instruction
  static constexpr int KES = KV8 ? 1 : ES;        // bytes per stored K/V element
  static constexpr int KROWB = D * KES;            // bytes of one stored K or V row of one head
  static constexpr int LANEB = EPL * KES;          // stored bytes behind one lane's EPL elements
  static constexpr int PAGEB = kPageTokens * KROWB; // bytes of one page of one head, K or V
  static constexpr int NB = PR / 16;               // MFMA row blocks
  static constexpr int KB = D / 32;                // MFMA k-blocks over head_dim
  static constexpr int DB = D / 16;                // MFMA 16-wide head_dim blocks
  // MFMA prefix work split over the four wavefronts: RG row groups of NBW
  // 16-row tiles times TG token groups of BPW 32-token blocks of the chunk
  // (16 rows: 1 x 4, 32 rows: 2 x 2, 64 rows: 4 x 1, 128 rows: 4 x 1 with two
  // tiles per wavefront).  Token groups of one row group combine through LDS.
  static constexpr int NBW = NB >= 8 ? 2 : 1;
  static constexpr int RG = MFMA ? NB / NBW : 1;
  static constexpr int TG = kWaves / RG;
  static constexpr int BPW = (kMfmaPrefixSplit / kMfmaBlock) / TG;
  static constexpr int WAVE_NR = (!MFMA && PR > HPK) ? PR : HPK;
  static constexpr int WAVE_SMEM = 4 * WAVE_NR * (D + 6);  // see RowTile::SMEM
  // fp32 responses of 4 or 8 rows run on row tiles.  A tile costs the same for
  // any row count, the wavefront dot products cost by the row: with 2 rows a
  // small group's step (d = 64) takes 8.3 us with them and 10.8 us with tiles, a
  // four-layer group decode (P = 1328) 42.2 and 47.1 ms.
  static constexpr bool RESP_ROWS = !BF && HPK >= 4;
  static constexpr int MFMA_SLOT = (MFMA && TG > 1) ? (NBW * DB * 64 * 4 + 2 * NBW * 64) : 0;
  static constexpr int MFMA_SMEM = kWaves * MFMA_SLOT;
  static constexpr int SMEM = WAVE_SMEM > MFMA_SMEM ? WAVE_SMEM : MFMA_SMEM;
  // wavefronts per SIMD the kernels are compiled for
  static constexpr int MIN_WAVES = 2;
  static_assert(LPT >= 2 && LPT <= 64, "row size");
  static_assert(!MFMA || BF, "MFMA path is bf16");
  static_assert(!KV8 || (BF && MFMA), "FP8 KV on the bf16 MFMA shapes");
  static_assert(!MFMA || (PR % 16 == 0), "MFMA rows");
  static_assert(!MFMA || (NB % NBW == 0 && kWaves % RG == 0 && DB % TG == 0 && BPW >= 1), "MFMA work split");
};

// ----------------------------------------------------------------------------
// Partial exchange between work-groups.  Producers store their partials, wait
// until the stores have completed and count an arrival; a merge reads them
// once its counters show every arrival.  Two cache policies:
//  * coherent: stores write through to the device coherence point and loads
//    bypass the XCD's L2 (the policy of agent-scope atomic stores and loads),
//    for producers and merges on any XCDs;
//  * XCD-local (StepArgs::l2_xcds > 0): stores stop in the XCD's L2 and loads
//    are served by the XCD's L2 or by the CU's L1.  The L1 is clean when a
//    launch starts, and a merge first reads a record line only after every
//    producer of that line has arrived, so the L1 never returns an older
//    copy within one launch that writes each record once.  Valid when every
//    work-group of a KV head runs on one XCD: work-group b on XCD
//    b % l2_xcds with Hkv a multiple of l2_xcds, which the host verified
//    when it created the context and which every work-group checks again (a
//    mismatch sets the status word).
// Neither needs an agent-scope fence (on this chip one writes back the whole
// L2).  Raw buffer resources over the workspace let a lane's 16 bytes leave
// as one write; offsets are in bytes and below ws_o_bytes / ws_ml_bytes.  The
// policy is a template parameter: the kernel picks one instantiation of its
// work-group body per launch, so no load or store waits behind a branch.
// ----------------------------------------------------------------------------
constexpr int kRawBufferWord3 = 0x00020000;
constexpr int kStoreThrough = 16;  // sc1
constexpr int kLoadCoherent = 16;  // sc1
constexpr int kStoreL2 = 0;
constexpr int kLoadL2 = 1;         // sc0: coherent at work-group scope: may hit the CU's L1 (clean at a launch's start), else the XCD's L2
constexpr int kXccIdReg = 20 | (3 << 11);  // s_getreg operand: HW_REG_XCC_ID bits 3:0

// MISS_L1: loads miss the CU's L1 also in the XCD-local exchange (sc0 loads
// are coherent only at work-group scope and may hit a line the L1 kept from
// an earlier read; a launch that rewrites and rereads the same records, as
// the step launch through every layer does, needs this).  Stores are the same
// either way.
template <bool L2, bool MISS_L1 = false>
struct Exchange {
  static constexpr int kStore = L2 ? kStoreL2 : kStoreThrough;
  static constexpr int kLoad = (L2 && !MISS_L1) ? kLoadL2 : kLoadCoherent;
  __amdgpu_buffer_rsrc_t o, ml;
  __device__ explicit Exchange(const StepArgs& a)
      : o(__builtin_amdgcn_make_buffer_rsrc(a.ws_o, 0, (int)a.ws_o_bytes, kRawBufferWord3)),
        ml(__builtin_amdgcn_make_buffer_rsrc(a.ws_ml, 0, (int)a.ws_ml_bytes, kRawBufferWord3)) {}
  __device__ void store(uint32_t off, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), o, off, 0, kStore);
  }
  __device__ void store4(uint32_t off, f32x4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), o, off, 0, kStore);
  }
  // (M, L) of record rec.
  __device__ void store_ml(int64_t rec, float m, float l) const {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(m), __float_as_uint(l)}, ml, (uint32_t)(rec * 8), 0,
                                          kStore);
  }
  __device__ f32x4 load4(uint32_t off) const {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(o, off, 0, kLoad));
  }
  __device__ u32x2 load_ml(int64_t rec) const {
    return __builtin_amdgcn_raw_buffer_load_b64(ml, (uint32_t)(rec * 8), 0, kLoad);
  }
};

// E4M3 (OCP) <-> bf16.  Widening is exact: every E4M3 value is a bf16 value.
// Narrowing rounds to nearest even; magnitudes beyond 448 are clamped first,
// so the conversion saturates instead of producing NaN.
__device__ __forceinline__ u32x4 widen_e4m3(uint2 w) {
  u32x4 r;
  r.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w.x, 1.0f, false));
  r.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w.x, 1.0f, true));
  r.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w.y, 1.0f, false));
  r.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w.y, 1.0f, true));
  return r;
}
__device__ __forceinline__ float sat_e4m3(float x) { return fminf(fmaxf(x, -448.f), 448.f); }
__device__ __forceinline__ uint32_t narrow4_e4m3(uint32_t lo, uint32_t hi) {  // 4 bf16 -> 4 E4M3 bytes
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(sat_e4m3(__uint_as_float(lo << 16)), sat_e4m3(__uint_as_float(lo & 0xffff0000u)),
                                          0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(sat_e4m3(__uint_as_float(hi << 16)), sat_e4m3(__uint_as_float(hi & 0xffff0000u)),
                                      w, true);
  return (uint32_t)w;
}
__device__ __forceinline__ uint2 narrow_e4m3(const u32x4& v) {  // 8 bf16 -> 8 E4M3 bytes
  return uint2{narrow4_e4m3(v.x, v.y), narrow4_e4m3(v.z, v.w)};
}
// One lane's EPL stored elements as a 16-byte register of the compute type.
// Load one lane's EPL stored elements, widened to the compute type.  Every
// K/V byte is read once per launch.  Response K/V (NT) is loaded
// non-temporal, so its stream through the XCD's L2 does not push out the
// split-K partials that the merges read back from there; the shared prefix,
// a fifth of the bytes and read again by every step, keeps the default policy
// (measured slightly faster than non-temporal).
template <class SH, bool NT>
__device__ __forceinline__ u32x4 ld_kv(const char* p) {
  if constexpr (SH::KV8) {
    u32x2 w;
    if constexpr (NT)
      w = __builtin_nontemporal_load((const u32x2*)p);
    else
      w = *(const u32x2*)p;
    return widen_e4m3(uint2{w.x, w.y});
  } else if constexpr (NT) {
    return __builtin_nontemporal_load((const u32x4*)p);
  } else {
    return *(const u32x4*)p;
  }
}
// Store one lane's EPL elements (given in the compute type) into a stored row.
template <class SH>
__device__ __forceinline__ void st_kv(char* p, const u32x4& v) {
  if constexpr (SH::KV8)
    *(uint2*)p = narrow_e4m3(v);
  else
    *(u32x4*)p = v;
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) x = fmaxf(x, __shfl_xor(x, s));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) x += __shfl_xor(x, s);
  return x;
}

// ----------------------------------------------------------------------------
// Wavefront dot products: NR query rows over the token range [t0, t1) of one KV head.
// LPT consecutive lanes hold one token's row (16 B each), so a load
// instruction covers TPI tokens; U loads per lane for K and for V are issued
// together before any arithmetic.  Each token group keeps its own running
// (m, l, o); the groups are combined at the end.  t0 must be a multiple of 16
// (page-aligned) so that every load instruction stays inside one page.
// ----------------------------------------------------------------------------
template <class SH, int NR>
struct WaveCfg {
  // Loads per lane per iteration, sized so that K/V buffers, scores and
  // accumulators of NR rows stay within the two-wavefronts-per-SIMD budget.
  static constexpr int UMAX = NR <= 2 ? 16 : NR <= 4 ? 8 : 4;
  static constexpr int U = (64 / SH::TPI) < UMAX ? (64 / SH::TPI) : UMAX;
  static_assert(16 % SH::TPI == 0, "a load instruction must not straddle a page");
};

template <class SH, int NR, class Addr>
__device__ __forceinline__ void wave_partial(const Addr& ad, int t0, int t1, const u32x4 (&q)[NR], float sl2,
                                             float (&m)[NR], float (&l)[NR], float (&o)[NR][SH::EPL]) {
  constexpr int LPT = SH::LPT, TPI = SH::TPI, EPL = SH::EPL, U = WaveCfg<SH, NR>::U;
  // Loads are issued in sub-blocks of SB per lane (K, then V) and the online
  // softmax runs per sub-block, so the arithmetic on early sub-blocks overlaps
  // the arrival of later ones.  Every load is unconditional: tokens past t1
  // read a valid row (Addr keeps addresses in bounds) and are masked to -inf.
  constexpr int SB = U >= 8 ? 4 : U;
  constexpr int NSB = U / SB;
  static_assert(U % SB == 0 && SB % 2 == 0, "sub-blocks of token pairs");
  const int lane = threadIdx.x & 63, ts = lane / LPT;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    m[r] = NEG_INF;
    l[r] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[r][e] = 0.f;
  }
  constexpr int PGI = (U * TPI + 15) / 16;  // 16-token pages touched per iteration
  for (int base = t0; base < t1; base += U * TPI) {
    // Page numbers first, in straight-line code: the compiler then waits for
    // the page-table load once instead of before every K/V load.
    int pg[PGI];
#pragma unroll
    for (int i = 0; i < PGI; ++i) pg[i] = ad.page(((base - t0) >> 4) + i);
    u32x4 kk[U], vv[U];
#pragma unroll
    for (int b = 0; b < NSB; ++b) {
#pragma unroll
      for (int kind = 0; kind < 2; ++kind)
#pragma unroll
        for (int u = b * SB; u < b * SB + SB; ++u) {
          u32x4& dst = kind ? vv[u] : kk[u];
          dst = ld_kv<SH, Addr::kNonTemporal>(ad.row(kind, base + u * TPI, base - t0 + u * TPI, pg[(u * TPI) >> 4], t1));
        }
    }
#pragma unroll
    for (int b = 0; b < NSB; ++b) {
      float s[SB][NR];
#pragma unroll
      for (int x = 0; x < SB; ++x) {
        const int u = b * SB + x;
        const bool ok = base + u * TPI + ts < t1;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const float y = group_sum<LPT>(dot16B<SH::BF>(kk[u], q[r])) * sl2;
          s[x][r] = ok ? y : NEG_INF;
        }
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        float mb = s[0][r];
#pragma unroll
        for (int x = 1; x < SB; ++x) mb = fmaxf(mb, s[x][r]);
        const float mn = fmaxf(m[r], mb);
        const float mu = (mn == NEG_INF) ? 0.f : mn;
        const float corr = exp2_fast(m[r] - mu);
        m[r] = mn;
        l[r] *= corr;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[r][e] *= corr;
#pragma unroll
        for (int x = 0; x < SB; ++x) {
          const float p = exp2_fast(s[x][r] - mu);
          l[r] += p;
          axpy16B(o[r], p, vv[b * SB + x]);
        }
      }
    }
  }
}

// Fold one token (K row chunk k, V row chunk v held by every token group) into
// token group 0's running partial.  All lanes take part in the reduction.
template <class SH, int NR>
__device__ __forceinline__ void fold_token(const u32x4& k, const u32x4& v, const u32x4 (&q)[NR], float sl2,
                                           float (&m)[NR], float (&l)[NR], float (&o)[NR][SH::EPL]) {
  const bool mine = (threadIdx.x & 63) < SH::LPT;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float x = group_sum<SH::LPT>(dot16B<SH::BF>(k, q[r])) * sl2;
    if (mine) {
      const float mn = fmaxf(m[r], x);
      const float corr = exp2_fast(m[r] - mn);
      const float p = exp2_fast(x - mn);
      m[r] = mn;
      l[r] = l[r] * corr + p;
#pragma unroll
      for (int e = 0; e < SH::EPL; ++e) o[r][e] *= corr;
      axpy16B(o[r], p, v);
    }
  }
}

// Combine the TPI token groups of a wavefront (lanes ch, ch+LPT, ...).
template <class SH, int NR>
__device__ __forceinline__ void wave_combine_groups(float (&m)[NR], float (&l)[NR], float (&o)[NR][SH::EPL]) {
#pragma unroll
  for (int mask = SH::LPT; mask < 64; mask <<= 1) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const float m2 = __shfl_xor(m[r], mask);
      const float l2 = __shfl_xor(l[r], mask);
      float a, b;
      lse_combine(m[r], l[r], m2, l2, a, b);
#pragma unroll
      for (int e = 0; e < SH::EPL; ++e) o[r][e] = o[r][e] * a + __shfl_xor(o[r][e], mask) * b;
    }
  }
}

template <class SH, int NR, bool L2>
__device__ __forceinline__ void combine_store_partial(float* smem, const Exchange<L2>& ex, int64_t rec0);

// Combine the four wavefronts' partials through LDS and store the block's
// partial rows [0, NR) at records rec0 + r.
template <class SH, int NR, bool L2>
__device__ __forceinline__ void block_store_partial(float* smem, const float (&m)[NR], const float (&l)[NR],
                                                    const float (&o)[NR][SH::EPL], const Exchange<L2>& ex,
                                                    int64_t rec0) {
  constexpr int D = SH::D, EPL = SH::EPL;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float* so = smem;                   // [4][NR][D]
  float* sml = smem + 4 * NR * D;     // [4][NR][2]
  if (lane < SH::LPT) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int e = 0; e < EPL; ++e) so[(w * NR + r) * D + lane * EPL + e] = o[r][e];
  }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      sml[(w * NR + r) * 2 + 0] = m[r];
      sml[(w * NR + r) * 2 + 1] = l[r];
    }
  }
  combine_store_partial<SH, NR, L2>(smem, ex, rec0);
}

// Second half of block_store_partial: after every wavefront has published its
// partial rows to LDS (so = [4][NR][D] unnormalised outputs, then
// sml = [4][NR][2] (m, l)), combine them and store rows [0, NR) at records
// rec0 + r.
template <class SH, int NR, bool L2>
__device__ __forceinline__ void combine_store_partial(float* smem, const Exchange<L2>& ex, int64_t rec0) {
  constexpr int D = SH::D;
  const float* so = smem;
  const float* sml = smem + 4 * NR * D;
  __syncthreads();
  for (int idx = threadIdx.x; idx < NR * D; idx += kBlockThreads) {
    const int r = idx / D, d = idx - r * D;
    float M = NEG_INF;
#pragma unroll
    for (int v = 0; v < 4; ++v) M = fmaxf(M, sml[(v * NR + r) * 2]);
    const float Mu = (M == NEG_INF) ? 0.f : M;
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float wgt = exp2_fast(sml[(v * NR + r) * 2] - Mu);
      L += wgt * sml[(v * NR + r) * 2 + 1];
      O += wgt * so[(v * NR + r) * D + d];
    }
    ex.store((uint32_t)(((rec0 + r) * D + d) * 4), O);
    if (d == 0) ex.store_ml(rec0 + r, M, L);
  }
}

// Addressing of a slot's stored response tokens: pages [page][kv][K|V][16][D].
// Lane i of `pages` holds the page of the wave's i-th 16-token group.  A load
// instruction covers TPI consecutive tokens of one page, so its address is
// (page base) + (token in page) * KROWB + lane * LANEB -- uniform plus lane offset.
template <class SH>
struct SuffixAddr {
  static constexpr bool kNonTemporal = true;
  const char* pool;
  int pages;
  int hkv, g;
  __device__ int page(int pslot) const { return __builtin_amdgcn_readlane(pages, pslot); }
  __device__ const char* row(int kind, int tokbase, int, int pg, int) const {
    const int lane = threadIdx.x & 63;
    return pool + ((int64_t)(pg * hkv + g) * 2 + kind) * SH::PAGEB + (tokbase & 15) * SH::KROWB + lane * SH::LANEB;
  }
};

// ----------------------------------------------------------------------------
// Response chunk on MFMA tiles (bf16 and E4M3 pages).  A page holds 16 tokens
// of one KV head, K then V, each in MFMA operand order:
//   K unit (kb, lane), 8 elements: token lane%16, dims 32kb + 8(lane/16) + e;
//   V unit (db, lane), 4 elements: dim 16db + lane%16, tokens 4(lane/16) + e;
// so a wavefront reads one operand tile with one coalesced load per lane
// (16 / 8 bytes for bf16).  Per page, S^T[tok][col] = K[tok] . Q[col] is one
// 16x16 tile (A = K units, B = Q^T, col = query row of the KV head: HPK of
// the 16 columns carry rows, the rest are zero).  Two consecutive pages form
// one 32-token k-block of O^T[d][col] += V^T[d][tok] P^T[tok][col]: the P^T
// operand is the eight probabilities a lane holds after the pages' two S^T
// tiles (the first page's four, then the second's) and the V^T operand is the
// two pages' V units side by side, so the contraction index is the same
// token permutation on both operands.  The running (m, l) and O^T are indexed
// by col = lane % 16 as on the prefix tiles; l is a per-lane sum until
// publish() adds the four lane groups.
// ----------------------------------------------------------------------------
template <class SH>
struct RespMfma {
  static constexpr int D = SH::D, KB = SH::KB, DB = SH::DB, HPK = SH::HPK, KES = SH::KES;
  static constexpr int NPG = D >= 128 ? 4 : 8;        // pages per load round
  static constexpr int TOK = 16 * NPG;                // tokens per load round
  static constexpr int KUB = 8 * KES, VUB = 4 * KES;  // bytes of one K / V unit
  using KUnit = std::conditional_t<SH::KV8, u32x2, u32x4>;
  using VUnit = std::conditional_t<SH::KV8, uint32_t, u32x2>;
  using VPair = std::conditional_t<SH::KV8, u32x2, u32x4>;  // two pages' V units, side by side
  struct Regs {
    KUnit k[NPG][KB];
    VPair v[NPG / 2][DB];
  };
  // Running partial: O^T tiles, m per column and, in lt, the column's sum of
  // probabilities (every element; an all-ones V^T tile through the same MFMA).
  struct Acc {
    f32x4 o[DB];
    f32x4 lt;
    float m;
  };
  // The newest token's rows, loaded with the queries: kq[kb] = K dims
  // 32kb + 8(lane/16) .. +7 and vq[db] = V dims 16db + 4(lane/16) .. +3.
  struct NewRows {
    u32x4 kq[KB];
    u32x2 vq[DB];
  };
  static_assert(HPK <= 16 && KB * 32 == D && DB * 16 == D, "response tile shape");

  __device__ __forceinline__ static int k_unit(int kb, int lane) { return (kb * 64 + lane) * KUB; }
  __device__ __forceinline__ static int v_unit(int db, int lane) { return (db * 64 + lane) * VUB; }
  // Page pg of KV head g: K at the returned address, V PAGEB bytes later.
  __device__ __forceinline__ static const char* page(const char* pool, int pg, int hkv, int g) {
    return pool + (int64_t)(pg * hkv + g) * 2 * SH::PAGEB;
  }

  // Loads of the round whose first page is entry ps of the wavefront's page
  // list (lane i of `pages`: its i-th page; entries past the range name page
  // 0, so every load stays inside the pool).  K of every page, then V, each
  // pair's V units straight into one MFMA operand register.
  __device__ __forceinline__ static void load_round(const char* pool, int pages, int hkv, int g, int ps, Regs& R) {
    const int lane = threadIdx.x & 63;
    const char* pp[NPG];
#pragma unroll
    for (int pr = 0; pr < NPG; ++pr) pp[pr] = page(pool, __builtin_amdgcn_readlane(pages, min(ps + pr, 63)), hkv, g);
#pragma unroll
    for (int pr = 0; pr < NPG; ++pr)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) R.k[pr][kb] = __builtin_nontemporal_load((const KUnit*)(pp[pr] + k_unit(kb, lane)));
#pragma unroll
    for (int j = 0; j < NPG / 2; ++j)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const VUnit a0 = __builtin_nontemporal_load((const VUnit*)(pp[2 * j] + SH::PAGEB + v_unit(db, lane)));
        const VUnit a1 = __builtin_nontemporal_load((const VUnit*)(pp[2 * j + 1] + SH::PAGEB + v_unit(db, lane)));
        if constexpr (SH::KV8)
          R.v[j][db] = u32x2{a0, a1};
        else
          R.v[j][db] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3);
      }
  }

  __device__ __forceinline__ static bf16x8 k_op(const KUnit& u) {
    if constexpr (SH::KV8)
      return __builtin_bit_cast(bf16x8, widen_e4m3(uint2{u.x, u.y}));
    else
      return __builtin_bit_cast(bf16x8, u);
  }
  __device__ __forceinline__ static u32x4 v_op(const VPair& u) {  // eight elements as bf16
    if constexpr (SH::KV8)
      return widen_e4m3(uint2{u.x, u.y});
    else
      return u;
  }
  // Bits of elements 2k and 2k + 1 of a four-element V unit that belong to
  // the first n tokens.
  __device__ __forceinline__ static uint32_t keep(int n, int k) {
    return (n > 2 * k ? 0x0000ffffu : 0u) | (n > 2 * k + 1 ? 0xffff0000u : 0u);
  }

  // Q^T operand: lane l holds query row row0 + l%16 (zero from HPK on), dims
  // 32kb + 8(l/16) .. +7.
  __device__ __forceinline__ static void load_q(const void* q, int64_t row0, bf16x8 (&bq)[KB]) {
    const int lane = threadIdx.x & 63, col = lane & 15, h = lane >> 4;
    const uint16_t* qr = (const uint16_t*)q + (row0 + col) * D + h * 8;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) bq[kb] = col < HPK ? *(const bf16x8*)(qr + kb * 32) : bf16x8{};
  }
  // The newest token's K / V rows (bf16, the caller's row layout), rounded to
  // E4M3 and back for E4M3 pages: the token is attended as its page stores it.
  __device__ __forceinline__ static void load_new(const char* krow, const char* vrow, NewRows& N) {
    const int h = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) N.kq[kb] = *(const u32x4*)(krow + (kb * 32 + h * 8) * 2);
#pragma unroll
    for (int db = 0; db < DB; ++db) N.vq[db] = *(const u32x2*)(vrow + (db * 16 + h * 4) * 2);
  }
  __device__ __forceinline__ static void round_new(NewRows& N) {
    if constexpr (SH::KV8) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) N.kq[kb] = widen_e4m3(narrow_e4m3(N.kq[kb]));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const int b = (int)narrow4_e4m3(N.vq[db].x, N.vq[db].y);
        N.vq[db] = u32x2{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 1.0f, false)),
                         __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 1.0f, true))};
      }
    }
  }

  // A partial that holds only the newest token (A's first contribution).
  __device__ __forceinline__ static void start_new(const NewRows& N, const bf16x8 (&bq)[KB], float sl2, Acc& A) {
    float s = 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) s += dot16B<true>(N.kq[kb], __builtin_bit_cast(u32x4, bq[kb]));
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    // the token's own weight is 2^(x - m) = 1 with m = x
    A.m = s * sl2;
    A.lt = f32x4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
    for (int db = 0; db < DB; ++db) A.o[db] = f32x4{bf_lo(N.vq[db].x), bf_hi(N.vq[db].x), bf_lo(N.vq[db].y), bf_hi(N.vq[db].y)};
  }

  __device__ __forceinline__ static void init(Acc& A) {
    A.m = NEG_INF;
    A.lt = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < DB; ++db) A.o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Tokens base .. base + TOK - 1 (the round held in R), of which those below
  // t1 count: one online-softmax step per page pair (32 tokens).
  __device__ __forceinline__ static void round(const Regs& R, const bf16x8 (&bq)[KB], int base, int t1, float sl2,
                                               Acc& A) {
    const int lane = threadIdx.x & 63, h = lane >> 4;
    const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
#pragma unroll
    for (int j = 0; j < NPG / 2; ++j) {
      const int pb0 = base + 32 * j;
      if (pb0 >= t1) break;
      // a pair that reaches past t1 masks its tail (scores and V elements)
      const bool edge = pb0 + 32 > t1;
      f32x4 st[2];
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
          t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_op(R.k[2 * j + mb][kb]), bq[kb], t, 0, 0, 0);
        t *= sl2;
        if (edge) {
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = (pb0 + 16 * mb + 4 * h + e < t1) ? t[e] : NEG_INF;
        }
        st[mb] = t;
      }
      float mx = fmaxf(fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3])),
                       fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = fmaxf(A.m, mx);
      const float mu = (mn == NEG_INF) ? 0.f : mn;
      const float corr = exp2_fast(A.m - mu);
      A.m = mn;
      A.lt *= corr;
#pragma unroll
      for (int db = 0; db < DB; ++db) A.o[db] *= corr;
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pb[e] = (__bf16)exp2_fast(st[0][e] - mu);
        pb[4 + e] = (__bf16)exp2_fast(st[1][e] - mu);
      }
      A.lt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb, A.lt, 0, 0, 0);
      // V elements of tokens at or past t1 (a page's unused tail holds whatever
      // was there) are cleared so that their zero weights give exact zeros.
      const int n0 = min(max(t1 - (pb0 + 4 * h), 0), 4), n1 = min(max(t1 - (pb0 + 16 + 4 * h), 0), 4);
      const u32x4 vm = {keep(n0, 0), keep(n0, 1), keep(n1, 0), keep(n1, 1)};
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        u32x4 va = v_op(R.v[j][db]);
        if (edge) va &= vm;
        A.o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, va), pb, A.o[db], 0, 0, 0);
      }
    }
  }

  // Store the newest token (position t, 0..15, of the page at pgk) in operand
  // order from the rows in N: K unit (kb, 16h + t) from the lanes with
  // lane % 16 == 0 (lane group h), V element (dim 16db + 4h + i, token t) from
  // lane 16h + i, i < 4.
  __device__ __forceinline__ static void store_new(char* pgk, int t, const NewRows& N) {
    const int lane = threadIdx.x & 63, h = lane >> 4, i = lane & 15;
    if (i == 0) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) st_kv<SH>(pgk + k_unit(kb, h * 16 + t), N.kq[kb]);
    }
    if (i < 4) {
      char* vb = pgk + SH::PAGEB + (t & 3) * KES;
      const int l0 = 16 * (t >> 2) + 4 * h + i;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const uint32_t w = (i & 2) ? N.vq[db].y : N.vq[db].x;
        const uint32_t bits = (i & 1) ? (w >> 16) : (w & 0xffffu);
        if constexpr (SH::KV8) {
          // N.vq holds E4M3 values widened to bf16: narrowing again is exact
          const uint32_t b = narrow4_e4m3(bits, 0u) & 0xffu;
          *(uint8_t*)(vb + v_unit(db, l0)) = (uint8_t)b;
        } else {
          *(uint16_t*)(vb + v_unit(db, l0)) = (uint16_t)bits;
        }
      }
    }
  }

  // Publish the wavefront's partial rows to LDS in block_store_partial's
  // layout (finish with combine_store_partial<SH, HPK, L2>).
  __device__ __forceinline__ static void publish(float* smem, const Acc& A) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, col = lane & 15, h = lane >> 4;
    float* so = smem;
    float* sml = smem + 4 * HPK * D;
    if (col < HPK) {
#pragma unroll
      for (int db = 0; db < DB; ++db) *(f32x4*)(so + (w * HPK + col) * D + db * 16 + h * 4) = A.o[db];
      if (h == 0) {
        sml[(w * HPK + col) * 2 + 0] = A.m;
        sml[(w * HPK + col) * 2 + 1] = A.lt[0];
      }
    }
  }
};

// ----------------------------------------------------------------------------
// Row tile: up to 16 query rows over tokens whose K and V are stored as plain
// rows (the prefix store below 16 MFMA rows or in fp32, and fp32 pages).  One
// wavefront, S^T[tok][row] = K[tok] . Q[row] and O^T[d][row] += V^T[d][tok]
// P^T[tok][row] on 16x16 matrix tiles: fp32 on v_mfma_f32_16x16x4_f32 (fp32
// products and sums), bf16 on v_mfma_f32_16x16x32_bf16.  row = lane % 16 on
// S^T, O^T and the running (m, l), h = lane / 16 below.
//   K operand: 16 bytes at chunk 4kb + h of token lane % 16 -- an element e of
//     it belongs to dim (4kb + h) * EPL + e, and the query operand holds the
//     same, so the order of the contraction does not matter.
//   V operand: token 4h + r (r = 0..3, what a lane's scores of a 16-token tile
//     are), VB bytes at chunk c = 16nv + lane % 16.  Element e of the chunk is
//     one output tile: its row i is dim (16nv + i) * VE + e.  fp32 takes the
//     lane's element as it is (one k-step per r); bf16 packs the eight tokens of
//     a 32-token group (16mb + 4h + r) per element with v_perm.
// Every load is 16 bytes a lane (8 for bf16 rows of 64) of whole 64-byte pieces
// of rows.  Bound by the matrix unit in fp32 (2048 cycles per 16 tokens and 16
// rows at d = 128), by loads in bf16.  The wavefront dot products it replaces
// spent their time summing across lanes: a 28-layer fp32 step of 8 slots (2
// rows each, 16 prefix rows, P = 1000) took 1834 us with them at one wavefront
// per SIMD and takes 487 us with tiles at two; bf16 with 2 rows (8 layers,
// P = 2483) took 213 us and takes 151.  Short chains keep the fp32 error where
// it was (1.8e-7 against 1.9e-7 relative); one chain of D is 465 us and 2.1e-7.
// ----------------------------------------------------------------------------
template <class SH, int NR>
struct RowTile {
  static constexpr bool BF = SH::BF;
  static constexpr int D = SH::D, EPL = SH::EPL, KB = SH::LPT / 4;
  static constexpr int GT = BF ? 32 : 16, MBS = GT / 16;                 // tokens and 16-token tiles of a group
  static constexpr int VB = SH::ROWB >= 256 ? 16 : 8, VE = VB / SH::ES;  // V bytes / elements of a lane's load
  static constexpr int NV = SH::ROWB / (16 * VB);
  static constexpr int NT = D / 16;                                      // output tiles: nv * VE + e
  static constexpr int NG = 128 / (GT * SH::ROWB * 2 / 256);             // groups per load round: 128 registers
  static constexpr int TOK = NG * GT;
  static constexpr int PITCH = D + 4;                 // LDS floats per published row: rows on different banks
  static constexpr int SMEM = kWaves * NR * (PITCH + 2);
  static_assert(NR <= 16 && NV * VE == NT && KB >= 1 && NG >= 1, "tile shape");
  using VReg = std::conditional_t<VB == 16, u32x4, u32x2>;
  struct Regs {
    u32x4 k[NG][MBS][KB];
    VReg v[NG][MBS][4][NV];
  };
  struct Acc {
    f32x4 o[NT];
    float m, l;  // l: this lane's share of the row's sum
  };

  // Loads of tokens base .. base + TOK - 1; ad.row(kind, t16, off) is the row of
  // token t16 + off (t16 a uniform multiple of 16, off < 16), any readable row
  // past the range's end.
  template <class Addr>
  __device__ __forceinline__ static void load_round(const Addr& ad, int base, Regs& R) {
    const int lane = threadIdx.x & 63, i = lane & 15, h = lane >> 4;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int mb = 0; mb < MBS; ++mb) {
        const char* kr = ad.row(0, base + g * GT + mb * 16, i) + h * 16;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) R.k[g][mb][kb] = Addr::template load<u32x4>(kr + kb * 64);
      }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int mb = 0; mb < MBS; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const char* vr = ad.row(1, base + g * GT + mb * 16, 4 * h + r) + i * VB;
#pragma unroll
          for (int nv = 0; nv < NV; ++nv) R.v[g][mb][r][nv] = Addr::template load<VReg>(vr + nv * 16 * VB);
        }
  }

  // Query operand from row pointer qr of this lane's row (null: a zero row).
  __device__ __forceinline__ static void load_q(const char* qr, u32x4 (&q)[KB]) {
    const int h = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) q[kb] = qr ? *(const u32x4*)(qr + (4 * kb + h) * 16) : u32x4{0, 0, 0, 0};
  }

  __device__ __forceinline__ static void init(Acc& A) {
    A.m = NEG_INF;
    A.l = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) A.o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // A partial that holds one token, given by its rows (fp32 pages: the newest token).
  __device__ __forceinline__ static void start_row(const char* krow, const char* vrow, const u32x4 (&q)[KB], float sl2,
                                                   Acc& A) {
    static_assert(!BF, "fp32 rows");
    const int h = (threadIdx.x & 63) >> 4;
    float s = 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) s += dot16B<false>(*(const u32x4*)(krow + (4 * kb + h) * 16), q[kb]);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    A.m = s * sl2;
    A.l = h == 0 ? 1.f : 0.f;
#pragma unroll
    for (int nv = 0; nv < NV; ++nv)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 x = *(const f32x4*)(vrow + (nv * 16 + 4 * h + r) * VB);
#pragma unroll
        for (int e = 0; e < VE; ++e) A.o[nv * VE + e][r] = x[e];
      }
  }

  // Two bf16 numbers with those that are infinite or NaN cleared.
  __device__ __forceinline__ static uint32_t finite_part(uint32_t w) {
    const uint32_t lo = (w & 0x7f80u) == 0x7f80u ? 0u : 0x0000ffffu, hi = (w & 0x7f800000u) == 0x7f800000u ? 0u : 0xffff0000u;
    return w & (lo | hi);
  }

  // Tokens base .. base + TOK - 1 (the round held in R), of which those below t1
  // count: one online-softmax step per group.  INF (bf16): V may hold infinities.
  template <bool INF = false>
  __device__ __forceinline__ static void round(Regs& R, const u32x4 (&q)[KB], int base, int t1, float sl2, Acc& A) {
    const int h = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int gb = base + g * GT;
      if (gb >= t1) break;
      f32x4 st[MBS];
#pragma unroll
      for (int mb = 0; mb < MBS; ++mb) {
        // short chains of products, added pairwise: sums of few terms round less than
        // one of D, and no product waits for the last
        constexpr int NC = BF ? KB : 2 * KB;
        f32x4 t[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          t[c] = f32x4{0.f, 0.f, 0.f, 0.f};
          if constexpr (BF) {
            t[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, R.k[g][mb][c]),
                                                           __builtin_bit_cast(bf16x8, q[c]), t[c], 0, 0, 0);
          } else {
#pragma unroll
            for (int e = 2 * (c & 1); e < 2 * (c & 1) + 2; ++e)
              t[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(R.k[g][mb][c / 2][e]),
                                                          __uint_as_float(q[c / 2][e]), t[c], 0, 0, 0);
          }
#pragma unroll
          for (int n = 1; (c + 1) % (2 * n) == 0; n *= 2) t[c + 1 - 2 * n] += t[c + 1 - n];
        }
        st[mb] = t[0] * sl2;
      }
      if (gb + GT > t1) {  // the range ends inside: mask scores, clear V (0 * whatever is there must be 0)
#pragma unroll
        for (int mb = 0; mb < MBS; ++mb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const bool in = gb + mb * 16 + 4 * h + r < t1;
            st[mb][r] = in ? st[mb][r] : NEG_INF;
#pragma unroll
            for (int nv = 0; nv < NV; ++nv) R.v[g][mb][r][nv] = in ? R.v[g][mb][r][nv] : VReg{};
          }
      }
      float mx = fmaxf(fmaxf(st[0][0], st[0][1]), fmaxf(st[0][2], st[0][3]));
      if constexpr (MBS == 2) mx = fmaxf(mx, fmaxf(fmaxf(st[1][0], st[1][1]), fmaxf(st[1][2], st[1][3])));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mn = fmaxf(A.m, mx);
      const float mu = (mn == NEG_INF) ? 0.f : mn;
      const float corr = exp2_fast(A.m - mu);
      A.m = mn;
      if constexpr (BF) {
        // A probability is weighed as the sum of two bf16 numbers (its rounding and
        // what that leaves), so it keeps 16 bits of mantissa on bf16 products.
        bf16x8 ph, pl;
        A.l *= corr;
#pragma unroll
        for (int t = 0; t < NT; ++t) A.o[t] *= corr;
#pragma unroll
        for (int mb = 0; mb < MBS; ++mb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x = exp2_fast(st[mb][r] - mu);
            ph[mb * 4 + r] = (__bf16)x;
            pl[mb * 4 + r] = (__bf16)(x - (float)(__bf16)x);
            A.l += x;
          }
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
          u32x4 a;
#pragma unroll
          for (int y = 0; y < 4; ++y)  // tokens (16mb + 4h) + 2(y%2), +1 with mb = y/2
            a[y] = __builtin_amdgcn_perm(R.v[g][y / 2][2 * (y & 1) + 1][0][e / 2], R.v[g][y / 2][2 * (y & 1)][0][e / 2], sel);
          u32x4 al = a;
          if constexpr (INF) {
#pragma unroll
            for (int y = 0; y < 4; ++y) al[y] = finite_part(a[y]);
          }
          A.o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, al), pl, A.o[e], 0, 0, 0);
          A.o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), ph, A.o[e], 0, 0, 0);
        }
      } else {
        // the group's sum starts from zero and joins the running one as a whole:
        // short chains, as for the scores
        float x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = exp2_fast(st[0][r] - mu);
        A.l = A.l * corr + ((x[0] + x[1]) + (x[2] + x[3]));
#pragma unroll
        for (int nv = 0; nv < NV; ++nv)
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r)
              c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(R.v[g][0][r][nv][e]), x[r], c, 0, 0, 0);
            A.o[nv * VE + e] = A.o[nv * VE + e] * corr + c;
          }
      }
    }
  }

  // Partial of stored tokens [t0, t1), the first round of which R holds.  In bf16
  // what the rounding of a probability leaves is zero or of either sign: times an
  // infinite V it would turn the infinity into NaN.  A partial that is not finite
  // is therefore taken once more, with that product over the finite V only (a
  // weight's own rounding times infinity stays infinity).  The look costs 0.1 us a
  // layer: 12 layers, 7 slots of 2 rows, P = 1500, d = 128: 107.1 us a step without
  // it, 108.6 with.
  template <class Addr>
  __device__ __forceinline__ static void stored(const Addr& ad, int t0, int t1, const u32x4 (&q)[KB], float sl2, Regs& R,
                                                Acc& A) {
    init(A);
    for (int base = t0; base < t1; base += TOK) {
      if (base != t0) load_round(ad, base, R);
      round(R, q, base, t1, sl2, A);
    }
    if constexpr (BF) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};  // NaN where an element is infinite or NaN
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = fmaf(A.o[t][r], 0.f, z[r]);
      if (__builtin_expect(__any((z[0] + z[1]) + (z[2] + z[3]) != 0.f), 0)) {
        init(A);
        for (int base = t0; base < t1; base += TOK) {
          load_round(ad, base, R);
          round<true>(R, q, base, t1, sl2, A);
        }
      }
    }
  }

  // Combine the four wavefronts' partials through LDS and store rows [0, NR) at
  // records rec0 + row.
  template <bool L2>
  __device__ __forceinline__ static void store(float* smem, Acc& A, const Exchange<L2>& ex, int64_t rec0) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 15, h = lane >> 4;
    float* sml = smem + kWaves * NR * PITCH;
    A.l += __shfl_xor(A.l, 16);
    A.l += __shfl_xor(A.l, 32);
    if (row < NR) {
      float* so = smem + (w * NR + row) * PITCH;
#pragma unroll
      for (int nv = 0; nv < NV; ++nv)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int e = 0; e < VE; e += 4)  // dims (16nv + 4h + r) * VE + e .. + 3
            *(f32x4*)(so + (nv * 16 + 4 * h + r) * VE + e) =
                f32x4{A.o[nv * VE + e][r], A.o[nv * VE + e + 1][r], A.o[nv * VE + e + 2][r], A.o[nv * VE + e + 3][r]};
      if (h == 0) {
        sml[(w * NR + row) * 2 + 0] = A.m;
        sml[(w * NR + row) * 2 + 1] = A.l;
      }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < NR * (D / 4); x += kBlockThreads) {
      const int r = x / (D / 4), d = (x - r * (D / 4)) * 4;
      float M = NEG_INF;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) M = fmaxf(M, sml[(v * NR + r) * 2]);
      const float Mu = (M == NEG_INF) ? 0.f : M;
      float L = 0.f;
      f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        const float wgt = exp2_fast(sml[(v * NR + r) * 2] - Mu);
        L += wgt * sml[(v * NR + r) * 2 + 1];
        O += *(const f32x4*)(smem + (v * NR + r) * PITCH + d) * wgt;
      }
      ex.store4((uint32_t)(((rec0 + r) * D + d) * 4), O);
      if (d == 0) ex.store_ml(rec0 + r, M, L);
    }
  }
};

// Rows of the plain prefix store: [prompt][kv][K|V][max_prompt_len][D].  Tokens
// past `end` read its last row (masked by the tile), inside this head's region.
template <class SH>
struct PrefixRows {
  const char* base[2];
  int end;
  __device__ PrefixRows(const StepArgs& a, const char* prefix, int p, int g, int end_) : end(end_) {
    const int64_t head = ((int64_t)p * a.Hkv + g) * 2;
    base[0] = prefix + head * a.max_prompt_len * SH::KROWB;
    base[1] = prefix + (head + 1) * a.max_prompt_len * SH::KROWB;
  }
  __device__ const char* row(int kind, int t16, int off) const {
    return base[kind] + (int64_t)min(t16 + off, end - 1) * SH::KROWB;
  }
  template <class T>
  __device__ static T load(const char* p) {
    return *(const T*)p;
  }
};
// Rows of a response in fp32 pages [page][kv][K|V][16][D]; lane i of `pages`
// holds the page of the wavefront's i-th 16-token group (entries past its range
// name page 0).  Non-temporal, as all response K/V.
template <class SH>
struct PageRows {
  const char* pool;
  int pages, hkv, g, first;  // first: the wavefront's first token
  __device__ const char* row(int kind, int t16, int off) const {
    const int pg = __builtin_amdgcn_readlane(pages, min((t16 - first) >> 4, 63));
    return pool + ((int64_t)(pg * hkv + g) * 2 + kind) * SH::PAGEB + off * SH::KROWB;
  }
  template <class T>
  __device__ static T load(const char* p) {
    return __builtin_nontemporal_load((const T*)p);
  }
};

__device__ __forceinline__ int64_t prefix_records(const StepArgs& a, int pr) {
  return (int64_t)a.num_prompts * a.prefix_chunks_max * a.Hkv * pr;
}

// ----------------------------------------------------------------------------
// Prefix chunk on row tiles (fp32, or fewer than 16 rows): rows r =
// slot_in_prompt * hpk + j, a quarter of the chunk's tokens per wavefront.
// ----------------------------------------------------------------------------
// This lane's query row of prefix work item (prompt p, KV head g): null for
// padding rows and rows of idle slots.
template <class SH>
__device__ __forceinline__ const char* prefix_query(const StepArgs& a, const void* q, int p, int g) {
  const int r = threadIdx.x & 15, si = r / SH::HPK, j = r - si * SH::HPK, s = p * a.m + min(si, a.m - 1);
  return r < a.prefix_rows && a.slot[s].len > 0 ? (const char*)q + ((int64_t)s * a.Hq + g * SH::HPK + j) * SH::ROWB
                                                : nullptr;
}

template <class SH, bool L2>
__device__ void prefix_rows(const StepArgs& a, int p, int c, int g, float* smem) {
  using T = RowTile<SH, SH::PR>;
  const int w = threadIdx.x >> 6;
  const int t0 = c * a.prefix_split, t1 = min(t0 + a.prefix_split, a.prompt[p].plen), sub = a.prefix_split / kWaves;
  const int wt0 = min(t0 + w * sub, t1), wt1 = min(wt0 + sub, t1);
  const PrefixRows<SH> ad(a, (const char*)a.prefix, p, g, wt1);
  typename T::Regs R;
  T::load_round(ad, wt0, R);
  u32x4 q[T::KB];
  T::load_q(prefix_query<SH>(a, a.q, p, g), q);
  typename T::Acc A;
  T::stored(ad, wt0, wt1, q, a.scale_log2, R, A);
  T::template store<L2>(smem, A, Exchange<L2>(a), (((int64_t)p * a.Hkv + g) * a.prefix_chunks_max + c) * SH::PR);
}

// ----------------------------------------------------------------------------
// Prefix chunk, MFMA path (R = NB*16 rows).  Per 32-token block:
//   S^T[tok][row] = K[tok][:] . Q[row][:]     (A = K block, B = Q^T; 2 x NB tiles of 16x16)
//   O^T[d][row]  += V^T[d][tok] P^T[tok][row] (A = V^T, B = P^T; NB x DB tiles)
// With S^T, O^T and the running (m, l) all indexed by row = lane % 16, the
// online-softmax rescale needs no cross-lane transpose.  The P^T operand takes
// the 8 probabilities a lane already holds; the contraction index (token) is
// the same permutation on both operands, and the prefix store keeps V in that
// order (see prefill_mfma_kernel).  Each wavefront keeps one block in flight
// (the accumulators of 32+ rows leave no registers for a second).
// ----------------------------------------------------------------------------
template <class SH>
__device__ __forceinline__ void mfma_block(const bf16x8 (&ka)[2][SH::KB], const bf16x8 (&va)[SH::DB],
                                           const bf16x8 (&bq)[SH::NB][SH::KB], int tb, int t1, float sl2,
                                           f32x4 (&acc)[SH::NB][SH::DB], float (&mrow)[SH::NB],
                                           float (&lrow)[SH::NB]) {
  constexpr int NB = SH::NB, KB = SH::KB, DB = SH::DB;
  const int lane = threadIdx.x & 63, q4 = lane >> 4;
  f32x4 st[2][NB];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[mb][kb], bq[nb][kb], t, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int tok = tb + mb * 16 + q4 * 4 + e;
        t[e] = (tok < t1) ? t[e] * sl2 : NEG_INF;
      }
      st[mb][nb] = t;
    }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float mb_ = fmaxf(fmaxf(fmaxf(st[0][nb][0], st[0][nb][1]), fmaxf(st[0][nb][2], st[0][nb][3])),
                      fmaxf(fmaxf(st[1][nb][0], st[1][nb][1]), fmaxf(st[1][nb][2], st[1][nb][3])));
    mb_ = fmaxf(mb_, __shfl_xor(mb_, 16));
    mb_ = fmaxf(mb_, __shfl_xor(mb_, 32));
    const float mn = fmaxf(mrow[nb], mb_);
    const float mu = (mn == NEG_INF) ? 0.f : mn;
    const float corr = exp2_fast(mrow[nb] - mu);
    mrow[nb] = mn;
    lrow[nb] *= corr;
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[nb][db] *= corr;
    bf16x8 pb;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const __bf16 h = (__bf16)exp2_fast(st[mb][nb][e] - mu);
        pb[mb * 4 + e] = h;
        lrow[nb] += (float)h;
      }
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[nb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[db], pb, acc[nb][db], 0, 0, 0);
  }
}

// ----------------------------------------------------------------------------
// Prefix chunk on MFMA tiles.  Wavefront w takes row group rg = w % RG (its
// NBW 16-row tiles) and token group tg = w / RG (BPW consecutive 32-token
// blocks of the chunk), walking its blocks with the next block's loads in
// flight while the current one is multiplied (with two tiles per wavefront,
// only the next K).  With one token group the
// wavefront stores its rows' partial directly; otherwise the token groups of
// a row group publish their partials to LDS and, after one barrier, each
// combines DB / TG of the head-dimension blocks of its row group and stores
// them.
// ----------------------------------------------------------------------------
template <class SH, bool L2>
__device__ void prefix_mfma(const StepArgs& a, int p, int c, int g, float* smem) {
  constexpr int D = SH::D, KB = SH::KB, DB = SH::DB, HPK = SH::HPK;
  constexpr int NBW = SH::NBW, RG = SH::RG, TG = SH::TG, BPW = SH::BPW;
  using WS = Shape<true, D, HPK, true, NBW * 16>;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, q4 = lane >> 4, r16 = lane & 15;
  const int rg = w % RG, tg = w / RG;
  const int plen = a.prompt[p].plen;
  const int t0 = c * a.prefix_split, t1 = min(t0 + a.prefix_split, plen);
  const int nblk = (t1 - t0 + kMfmaBlock - 1) / kMfmaBlock;
  const int b0 = tg * BPW, b1 = min(b0 + BPW, nblk);
  const float sl2 = a.scale_log2;

  bf16x8 bq[NBW][KB];
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) {
    const int row = (rg * NBW + nb) * 16 + r16, si = row / HPK, j = row - si * HPK, s = p * a.m + min(si, a.m - 1);
    const bool ok = row < a.prefix_rows && a.slot[s].len > 0;
    const uint16_t* qr = (const uint16_t*)a.q + ((int64_t)s * a.Hq + g * HPK + j) * D;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) bq[nb][kb] = ok ? *(const bf16x8*)(qr + kb * 32 + q4 * 8) : bf16x8{};
  }
  f32x4 acc[NBW][DB];
  float mrow[NBW], lrow[NBW];
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) {
    mrow[nb] = NEG_INF;
    lrow[nb] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[nb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const char* head = (const char*)a.prefix +
                     ((int64_t)(p * a.Hkv + g) * (a.max_prompt_len / kMfmaBlock)) * (2 * kMfmaBlock * D * SH::KES);
  auto fetch_k = [&](int b, bf16x8 (&ka)[2][KB]) {
    const char* kblk = head + (int64_t)((t0 + b * kMfmaBlock) / kMfmaBlock) * (2 * kMfmaBlock * D * SH::KES);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
        ka[mb][kb] = __builtin_bit_cast(bf16x8, ld_kv<SH, false>(kblk + ((mb * KB + kb) * 64 + lane) * 8 * SH::KES));
  };
  auto fetch_v = [&](int b, bf16x8 (&va)[DB]) {
    const char* vblk = head + (int64_t)((t0 + b * kMfmaBlock) / kMfmaBlock) * (2 * kMfmaBlock * D * SH::KES) +
                       kMfmaBlock * D * SH::KES;
#pragma unroll
    for (int db = 0; db < DB; ++db) va[db] = __builtin_bit_cast(bf16x8, ld_kv<SH, false>(vblk + (db * 64 + lane) * 8 * SH::KES));
  };
  // With two tiles per wavefront the accumulators leave room to prefetch only
  // the next block's K; its V is fetched once the current block is done.
  constexpr bool PREFETCH_V = NBW == 1;
  if (b0 < b1) {
    bf16x8 ka[2][KB], va[DB];
    fetch_k(b0, ka);
    fetch_v(b0, va);
    for (int b = b0; b < b1; ++b) {
      const bool more = b + 1 < b1;
      bf16x8 kn[2][KB], vn[DB];
      if (more) {
        fetch_k(b + 1, kn);
        if constexpr (PREFETCH_V) fetch_v(b + 1, vn);
      }
      mfma_block<WS>(ka, va, bq, t0 + b * kMfmaBlock, t1, sl2, acc, mrow, lrow);
      if (more) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int kb = 0; kb < KB; ++kb) ka[mb][kb] = kn[mb][kb];
        if constexpr (PREFETCH_V) {
#pragma unroll
          for (int db = 0; db < DB; ++db) va[db] = vn[db];
        } else {
          fetch_v(b + 1, va);
        }
      }
    }
  }
#pragma unroll
  for (int nb = 0; nb < NBW; ++nb) {
    lrow[nb] += __shfl_xor(lrow[nb], 16);
    lrow[nb] += __shfl_xor(lrow[nb], 32);
  }
  const int64_t rec0 = (((int64_t)p * a.Hkv + g) * a.prefix_chunks_max + c) * SH::PR;
  const Exchange<L2> ex(a);
  if constexpr (TG == 1) {
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      const int64_t rec = rec0 + (rg * NBW + nb) * 16 + r16;
#pragma unroll
      for (int db = 0; db < DB; ++db) ex.store4((uint32_t)((rec * D + db * 16 + q4 * 4) * 4), acc[nb][db]);
      if (q4 == 0) ex.store_ml(rec, mrow[nb], lrow[nb]);
    }
  } else {
    constexpr int OFL = NBW * DB * 64 * 4;
    {
      float* sl = smem + w * SH::MFMA_SLOT;
#pragma unroll
      for (int nb = 0; nb < NBW; ++nb) {
#pragma unroll
        for (int db = 0; db < DB; ++db) *(f32x4*)(sl + ((nb * DB + db) * 64 + lane) * 4) = acc[nb][db];
        sl[OFL + nb * 64 + lane] = mrow[nb];
        sl[OFL + NBW * 64 + nb * 64 + lane] = lrow[nb];
      }
    }
    __syncthreads();
    constexpr int DBW = DB / TG;  // head-dim blocks this wavefront combines and stores
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      float M = NEG_INF;
#pragma unroll
      for (int t = 0; t < TG; ++t) M = fmaxf(M, smem[(t * RG + rg) * SH::MFMA_SLOT + OFL + nb * 64 + lane]);
      const float Mu = (M == NEG_INF) ? 0.f : M;
      float wv[TG], L = 0.f;
#pragma unroll
      for (int t = 0; t < TG; ++t) {
        const float* sl = smem + (t * RG + rg) * SH::MFMA_SLOT;
        wv[t] = exp2_fast(sl[OFL + nb * 64 + lane] - Mu);
        L += wv[t] * sl[OFL + NBW * 64 + nb * 64 + lane];
      }
      const int64_t rec = rec0 + (rg * NBW + nb) * 16 + r16;
#pragma unroll
      for (int x = 0; x < DBW; ++x) {
        const int db = tg * DBW + x;
        f32x4 acc4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < TG; ++t)
          acc4 += *(const f32x4*)(smem + (t * RG + rg) * SH::MFMA_SLOT + ((nb * DB + db) * 64 + lane) * 4) * wv[t];
        ex.store4((uint32_t)((rec * D + db * 16 + q4 * 4) * 4), acc4);
      }
      if (tg == 0 && q4 == 0) ex.store_ml(rec, M, L);
    }
  }
}

// ----------------------------------------------------------------------------
// Response chunk of one live slot (hpk rows), plus the append of this step's
// K/V when the chunk holds the newest position.
// ----------------------------------------------------------------------------
// One wavefront copies the newest token's fp32 K and V rows into its page row.
template <class SH>
__device__ __forceinline__ void store_row(char* page_row, const char* krow, const char* vrow) {
  const int lane = threadIdx.x & 63;
  for (int x = lane; x < 2 * SH::LPT; x += 64) {
    const int kind = x / SH::LPT, ch = x - kind * SH::LPT;
    *(u32x4*)(page_row + kind * SH::PAGEB + ch * 16) = *(const u32x4*)((kind ? vrow : krow) + ch * 16);
  }
}

template <class SH, bool L2>
__device__ void suffix_chunk_mfma(const StepArgs& a, int s, int c, int g, float* smem);
template <class SH, bool L2>
__device__ void suffix_chunk_rows(const StepArgs& a, int s, int c, int g, float* smem);

template <class SH, bool L2>
__device__ void suffix_chunk(const StepArgs& a, int s, int c, int g, float* smem) {
  if constexpr (SH::BF) {
    suffix_chunk_mfma<SH, L2>(a, s, c, g, smem);
    return;
  }
  if constexpr (SH::RESP_ROWS) {
    suffix_chunk_rows<SH, L2>(a, s, c, g, smem);
    return;
  }
  constexpr int HPK = SH::HPK;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, ch = lane % SH::LPT;
  const SlotPlan& sp = a.slot[s];
  const int len = sp.len;
  const int t0 = c * a.split, t1 = min(t0 + a.split, len);
  const int sub = a.split / 4;
  const int wt0 = min(t0 + w * sub, t1), wt1 = min(wt0 + sub, t1);
  // Page indices of this wavefront's range (lane i: the i-th 16-token group) and
  // the query rows, loaded together.
  const int npg = (wt1 - wt0 + kPageTokens - 1) / kPageTokens;
  const int32_t* ptab = a.page_table + (int64_t)sp.seq * a.pages_per_slot + (wt0 >> 4);
  const int pages = lane < npg ? ptab[lane] : 0;
  u32x4 q[HPK];
#pragma unroll
  for (int r = 0; r < HPK; ++r)
    q[r] = *((const u32x4*)((const char*)a.q + ((int64_t)s * a.Hq + g * HPK + r) * SH::ROWB) + ch);
  // The newest token (position len-1) comes from the caller's rows: the wave
  // whose range holds it loads it up front, folds it in after the stored
  // tokens, and stores it into its page.
  const int last = len - 1;
  const bool has_new = last >= wt0 && last < wt1;
  const int64_t newrow = ((int64_t)s * a.Hkv + g) * SH::ROWB;
  u32x4 knew = u32x4{0, 0, 0, 0}, vnew = u32x4{0, 0, 0, 0};
  if (has_new) {
    knew = *((const u32x4*)((const char*)a.knew + newrow) + ch);
    vnew = *((const u32x4*)((const char*)a.vnew + newrow) + ch);
  }
  SuffixAddr<SH> ad{(const char*)a.pool, pages, a.Hkv, g};
  float m[HPK], l[HPK], o[HPK][SH::EPL];
  wave_partial<SH, HPK>(ad, wt0, has_new ? last : wt1, q, a.scale_log2, m, l, o);
  if (has_new) {
    fold_token<SH, HPK>(knew, vnew, q, a.scale_log2, m, l, o);
    if (lane < SH::LPT) {
      char* row = (char*)a.pool + (int64_t)(sp.cur_page * a.Hkv + g) * 2 * SH::PAGEB + (last & 15) * SH::KROWB +
                  ch * SH::LANEB;
      st_kv<SH>(row, knew);
      st_kv<SH>(row + SH::PAGEB, vnew);
    }
  }
  wave_combine_groups<SH, HPK>(m, l, o);
  const int64_t rec0 = prefix_records(a, SH::PR) + (((int64_t)s * a.Hkv + g) * a.suffix_chunks_max + c) * HPK;
  block_store_partial<SH, HPK, L2>(smem, m, l, o, Exchange<L2>(a), rec0);

  if (t1 == len && g == 0 && threadIdx.x == 0) {  // bookkeeping of this step's token (K/V stored above)
    const int pos = len - 1;
    a.page_table[(int64_t)sp.seq * a.pages_per_slot + (pos >> 4)] = sp.cur_page;
    if (a.count_tokens)
      __hip_atomic_fetch_add(&a.tokens[(s / a.m) * a.G + sp.sample], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Response chunk of one live slot on MFMA tiles (bf16 and E4M3 pages; see
// RespMfma): wavefront w takes tokens [wt0, wt1) of the chunk in rounds of
// RespMfma::TOK; the wavefront whose range holds the newest position starts
// from that token (read from the caller's rows together with the queries) and
// stores it into its page; the four wavefronts' partials combine through LDS.
template <class SH, bool L2>
__device__ void suffix_chunk_mfma(const StepArgs& a, int s, int c, int g, float* smem) {
  using RM = RespMfma<SH>;
  constexpr int HPK = SH::HPK;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const SlotPlan& sp = a.slot[s];
  const int len = sp.len;
  const int t0 = c * a.split, t1 = min(t0 + a.split, len);
  const int sub = a.split / 4;
  const int wt0 = min(t0 + w * sub, t1), wt1 = min(wt0 + sub, t1);
  const int npg = (wt1 - wt0 + kPageTokens - 1) / kPageTokens;
  const int32_t* ptab = a.page_table + (int64_t)sp.seq * a.pages_per_slot + (wt0 >> 4);
  const int pages = lane < npg ? ptab[lane] : 0;
  const int last = len - 1;
  const bool has_new = last >= wt0 && last < wt1;
  const int te = has_new ? last : wt1;  // stored tokens of this wavefront: [wt0, te)
  typename RM::Regs R;
  RM::load_round((const char*)a.pool, pages, a.Hkv, g, 0, R);
  // queries and the newest token's rows in one batch of loads; that token is
  // folded in first and stored into its page
  bf16x8 bq[SH::KB];
  RM::load_q(a.q, (int64_t)s * a.Hq + g * HPK, bq);
  typename RM::NewRows N;
  if (has_new) {
    const int64_t newrow = ((int64_t)s * a.Hkv + g) * SH::ROWB;
    RM::load_new((const char*)a.knew + newrow, (const char*)a.vnew + newrow, N);
  }
  typename RM::Acc A;
  if (has_new) {
    RM::round_new(N);
    RM::start_new(N, bq, a.scale_log2, A);
    RM::store_new((char*)RM::page((const char*)a.pool, sp.cur_page, a.Hkv, g), last & 15, N);
  } else {
    RM::init(A);
  }
  for (int base = wt0; base < te; base += RM::TOK) {
    if (base != wt0) RM::load_round((const char*)a.pool, pages, a.Hkv, g, (base - wt0) >> 4, R);
    RM::round(R, bq, base, te, a.scale_log2, A);
  }
  RM::publish(smem, A);
  const int64_t rec0 = prefix_records(a, SH::PR) + (((int64_t)s * a.Hkv + g) * a.suffix_chunks_max + c) * HPK;
  combine_store_partial<SH, HPK, L2>(smem, Exchange<L2>(a), rec0);

  if (t1 == len && g == 0 && threadIdx.x == 0) {  // bookkeeping of this step's token (K/V stored above)
    const int pos = len - 1;
    a.page_table[(int64_t)sp.seq * a.pages_per_slot + (pos >> 4)] = sp.cur_page;
    if (a.count_tokens)
      __hip_atomic_fetch_add(&a.tokens[(s / a.m) * a.G + sp.sample], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// fp32 response chunk on a row tile: the wavefront whose range holds the newest
// position starts from that token's rows and stores them into its page.
template <class SH, bool L2>
__device__ void suffix_chunk_rows(const StepArgs& a, int s, int c, int g, float* smem) {
  using T = RowTile<SH, SH::HPK>;
  constexpr int HPK = SH::HPK;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const SlotPlan& sp = a.slot[s];
  const int len = sp.len, last = len - 1;
  const int t0 = c * a.split, t1 = min(t0 + a.split, len), sub = a.split / kWaves;
  const int wt0 = min(t0 + w * sub, t1), wt1 = min(wt0 + sub, t1);
  const int npg = (wt1 - wt0 + kPageTokens - 1) / kPageTokens;
  const int32_t* ptab = a.page_table + (int64_t)sp.seq * a.pages_per_slot + (wt0 >> 4);
  const PageRows<SH> ad{(const char*)a.pool, lane < npg ? ptab[lane] : 0, a.Hkv, g, wt0};
  const bool has_new = last >= wt0 && last < wt1;
  const int te = has_new ? last : wt1;  // stored tokens of this wavefront: [wt0, te)
  typename T::Regs R;
  T::load_round(ad, wt0, R);
  u32x4 q[T::KB];
  const int row = lane & 15;
  T::load_q(row < HPK ? (const char*)a.q + ((int64_t)s * a.Hq + g * HPK + row) * SH::ROWB : nullptr, q);
  typename T::Acc A;
  if (has_new) {
    const int64_t newrow = ((int64_t)s * a.Hkv + g) * SH::ROWB;
    T::start_row((const char*)a.knew + newrow, (const char*)a.vnew + newrow, q, a.scale_log2, A);
    store_row<SH>((char*)a.pool + (int64_t)(sp.cur_page * a.Hkv + g) * 2 * SH::PAGEB + (last & 15) * SH::KROWB,
                  (const char*)a.knew + newrow, (const char*)a.vnew + newrow);
  } else {
    T::init(A);
  }
  for (int base = wt0; base < te; base += T::TOK) {
    if (base != wt0) T::load_round(ad, base, R);
    T::round(R, q, base, te, a.scale_log2, A);
  }
  T::template store<L2>(smem, A, Exchange<L2>(a),
                        prefix_records(a, SH::PR) + (((int64_t)s * a.Hkv + g) * a.suffix_chunks_max + c) * HPK);

  if (t1 == len && g == 0 && threadIdx.x == 0) {  // bookkeeping of this step's token (K/V stored above)
    a.page_table[(int64_t)sp.seq * a.pages_per_slot + (last >> 4)] = sp.cur_page;
    if (a.count_tokens)
      __hip_atomic_fetch_add(&a.tokens[(s / a.m) * a.G + sp.sample], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ----------------------------------------------------------------------------
// Merge all partials of (slot s, KV head g) and write O rows g*hpk .. +hpk-1
// (the log-sum-exp combination of split-K partial softmaxes).  Partial c < nP
// is prefix chunk c, then the response chunks.  The hpk*d outputs are cut into
// 4-float vectors, one per lane (MV vectors per lane when they exceed 64); the
// partials are dealt round-robin to the four wavefronts, each of which loads a
// round of MCU partials at once (16-byte loads, no load waits on another) and
// folds them into a running (max, sum, output); the four wavefronts' results
// are then combined through LDS.
// ----------------------------------------------------------------------------
template <class SH>
struct MergeShape {
  static constexpr int OPP = SH::HPK * SH::D;          // outputs per partial
  static constexpr int NVEC = OPP / 4;                 // 4-float vectors per partial
  static constexpr int MV = (NVEC + 63) / 64;          // vectors per lane
  static constexpr int MCU = MV == 1 ? 8 : 4;          // partials per load round and wavefront
  static constexpr int SMEM = 4 * 64 * MV * 8;         // per wave and lane vector: max, sum, 2 pad, 4 outputs
  static_assert(SH::D % 4 == 0, "vectors");
};

template <class SH, bool L2>
__device__ void merge_outputs(const StepArgs& a, int s, int g, float* smem) {
  using MS = MergeShape<SH>;
  constexpr int D = SH::D, HPK = SH::HPK, MV = MS::MV, MCU = MS::MCU;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = s / a.m, si = s - p * a.m;
  const int nP = a.prompt[p].nchunks;
  const int n = nP + (a.slot[s].len + a.split - 1) / a.split;
  const int64_t pbase = ((int64_t)p * a.Hkv + g) * a.prefix_chunks_max * SH::PR + si * HPK;
  const int64_t pstride = SH::PR;
  const int64_t sbase = prefix_records(a, SH::PR) + ((int64_t)s * a.Hkv + g) * a.suffix_chunks_max * HPK;
  const int64_t sstride = HPK;
  auto rec = [&](int c, int j) -> int64_t { return (c < nP ? pbase + c * pstride : sbase + (c - nP) * sstride) + j; };
  const Exchange<L2> ex(a);

  float M[MV], L[MV];
  f32x4 O[MV];
#pragma unroll
  for (int v = 0; v < MV; ++v) {
    M[v] = NEG_INF;
    L[v] = 0.f;
    O[v] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c0 = w; c0 < n; c0 += 4 * MCU) {
    u32x2 ml[MCU][MV];
    f32x4 ov[MCU][MV];
#pragma unroll
    for (int u = 0; u < MCU; ++u) {
      const int c = c0 + 4 * u;
#pragma unroll
      for (int v = 0; v < MV; ++v) {
        const int x = (v * 64 + lane) * 4, j = x / D, d = x - j * D;
        if (c < n && x < MS::OPP) {
          const int64_t r = rec(c, j);
          ml[u][v] = ex.load_ml(r);
          ov[u][v] = ex.load4((uint32_t)((r * D + d) * 4));
        } else {
          ml[u][v] = u32x2{__float_as_uint(NEG_INF), 0u};
          ov[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
#pragma unroll
    for (int u = 0; u < MCU; ++u)
#pragma unroll
      for (int v = 0; v < MV; ++v) {
        const float mc = __uint_as_float(ml[u][v].x), lc = __uint_as_float(ml[u][v].y);
        const float nm = fmaxf(M[v], mc);
        const float base = nm == NEG_INF ? 0.f : nm;
        const float al = exp2_fast(M[v] - base), be = mc == NEG_INF ? 0.f : exp2_fast(mc - base);
        L[v] = L[v] * al + lc * be;
        O[v] = O[v] * al + ov[u][v] * be;
        M[v] = nm;
      }
  }
#pragma unroll
  for (int v = 0; v < MV; ++v) {
    float* e = smem + ((w * MV + v) * 64 + lane) * 8;
    e[0] = M[v];
    e[1] = L[v];
    *(f32x4*)(e + 4) = O[v];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < MS::NVEC; t += kBlockThreads) {
    const int v = t >> 6, ln = t & 63;
    float mw[4], mx = NEG_INF;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mw[q] = smem[((q * MV + v) * 64 + ln) * 8];
      mx = fmaxf(mx, mw[q]);
    }
    const float base = mx == NEG_INF ? 0.f : mx;
    float Lt = 0.f;
    f32x4 Ot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float* e = smem + ((q * MV + v) * 64 + ln) * 8;
      const float wq = mw[q] == NEG_INF ? 0.f : exp2_fast(mw[q] - base);
      Lt += wq * e[1];
      Ot += *(const f32x4*)(e + 4) * wq;
    }
    const int x = t * 4, j = x / D, d = x - j * D;
    *(f32x4*)(a.o + ((int64_t)s * a.Hq + g * HPK + j) * D + d) = Ot * (1.f / Lt);
  }
}

// A producer block has stored its partial: once every thread's stores have
// completed, count one arrival on the counter of each live slot among slots
// first .. first + n - 1 (lane i adds for slot first + i; n <= 64).  A
// response chunk counts on its own slot, a prefix chunk on every live slot of
// its prompt, so a merge waits on a single counter that no other merge polls.
__device__ __forceinline__ void arrive(const StepArgs& a, int first, int n, int g) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);  // this thread's partial stores have completed
  __syncthreads();                // ... and so have every thread's
  if ((int)threadIdx.x < n && a.slot[first + threadIdx.x].len > 0)
    __hip_atomic_fetch_add(a.counters + (int64_t)((first + threadIdx.x) * a.Hkv + g) * kCounterStride, 1,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t* slot_counter(const StepArgs& a, int s, int g) {
  return a.counters + (int64_t)(s * a.Hkv + g) * kCounterStride;
}
// Counters wrap: `reached` compares by the sign of the difference.
__device__ __forceinline__ bool reached(const int32_t* ctr, int32_t target) {
  const int32_t v = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (int32_t)((uint32_t)v - (uint32_t)target) >= 0;
}

// One lane: wait until *ctr has reached target, polling at most merge_polls
// times.  Gives up at once when merge_polls < 0 or, in a step launch,
// when the status word shows that another wait has given up.
__device__ bool bounded_wait(const StepArgs& a, const int32_t* ctr, int32_t target, bool step) {
  if (a.merge_polls < 0) return false;
  if (reached(ctr, target)) return true;
  if (step && __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
  for (int spins = 0; spins < a.merge_polls; ++spins) {
    __builtin_amdgcn_s_sleep(2);
    if (reached(ctr, target)) return true;
  }
  return false;
}

// Merge block of (slot s, KV head g): wait until the prefix chunks of its
// prompt and its own response chunks have all arrived on its counter
// (bounded), then merge.
template <class SH, bool L2>
__device__ void merge_block(const StepArgs& a, int s, int g, unsigned long long* flag, float* smem) {
  if (threadIdx.x == 0) *flag = bounded_wait(a, slot_counter(a, s, g), a.slot[s].target, false);
  __syncthreads();
  if (!*flag) {
    if (threadIdx.x == 0) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float* o = a.o + ((int64_t)s * a.Hq + g * SH::HPK) * SH::D;
    for (int idx = threadIdx.x; idx < SH::HPK * SH::D; idx += kBlockThreads) o[idx] = __builtin_nanf("");
    return;
  }
  merge_outputs<SH, L2>(a, s, g, smem);
}

// One wavefront merges every partial of (slot s, KV head g) of a layer and
// writes O rows g*hpk .. +hpk-1 (the log-sum-exp combination of the split-K
// partial softmaxes, in partial order).  Lane x of vector v holds outputs
// 4 * (v * 64 + x) .. +3; partials are loaded MCW at a time.
// STEP: one of many layers, so partials are read past the CU's L1 (records of the
// layer before may be there).
template <class SH>
struct MergeWaveShape {
  static constexpr int OPP = SH::HPK * SH::D;
  static constexpr int MV = (OPP / 4 + 63) / 64;
  static constexpr int MCW = merge_wave_partials(OPP);
};

template <class SH, bool L2, bool STEP>
__device__ void merge_wave(const StepArgs& a, float* out, int s, int g, int32_t target) {
  using MW = MergeWaveShape<SH>;
  constexpr int D = SH::D, HPK = SH::HPK, MV = MW::MV, MCW = MW::MCW;
  const int lane = threadIdx.x & 63;
  const int p = s / a.m, si = s - p * a.m;
  float* orow = out + ((int64_t)s * a.Hq + g * HPK) * D;
  int ok = 0;
  if (lane == 0) {
    ok = bounded_wait(a, slot_counter(a, s, g), target, STEP);
    if (!ok) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  ok = __builtin_amdgcn_readfirstlane(ok);
  if (!ok) {
#pragma unroll
    for (int v = 0; v < MV; ++v) {
      const int x = (v * 64 + lane) * 4;
      if (x < MW::OPP) *(f32x4*)(orow + x) = f32x4{1.f, 1.f, 1.f, 1.f} * __builtin_nanf("");
    }
    return;
  }
  const int nP = a.prompt[p].nchunks;
  const int n = nP + a.slot[s].pieces;
  const int64_t pbase = ((int64_t)p * a.Hkv + g) * a.prefix_chunks_max * SH::PR + si * HPK;
  const int64_t sbase = prefix_records(a, SH::PR) + ((int64_t)s * a.Hkv + g) * a.suffix_chunks_max * HPK;
  auto rec = [&](int c, int j) -> int64_t { return (c < nP ? pbase + (int64_t)c * SH::PR : sbase + (int64_t)(c - nP) * HPK) + j; };
  const Exchange<L2, STEP> ex(a);
  float M[MV], L[MV];
  f32x4 O[MV];
#pragma unroll
  for (int v = 0; v < MV; ++v) {
    M[v] = NEG_INF;
    L[v] = 0.f;
    O[v] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c0 = 0; c0 < n; c0 += MCW) {
    u32x2 ml[MCW][MV];
    f32x4 ov[MCW][MV];
#pragma unroll
    for (int u = 0; u < MCW; ++u) {
      const int c = c0 + u;
#pragma unroll
      for (int v = 0; v < MV; ++v) {
        const int x = (v * 64 + lane) * 4, j = x / D, d = x - j * D;
        if (c < n && x < MW::OPP) {
          const int64_t r = rec(c, j);
          ml[u][v] = ex.load_ml(r);
          ov[u][v] = ex.load4((uint32_t)((r * D + d) * 4));
        } else {
          ml[u][v] = u32x2{__float_as_uint(NEG_INF), 0u};
          ov[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
#pragma unroll
    for (int u = 0; u < MCW; ++u)
#pragma unroll
      for (int v = 0; v < MV; ++v) {
        const float mc = __uint_as_float(ml[u][v].x), lc = __uint_as_float(ml[u][v].y);
        const float nm = fmaxf(M[v], mc);
        const float base = nm == NEG_INF ? 0.f : nm;
        const float al = exp2_fast(M[v] - base), be = mc == NEG_INF ? 0.f : exp2_fast(mc - base);
        L[v] = L[v] * al + lc * be;
        O[v] = O[v] * al + ov[u][v] * be;
        M[v] = nm;
      }
  }
#pragma unroll
  for (int v = 0; v < MV; ++v) {
    const int x = (v * 64 + lane) * 4;
    if (x < MW::OPP) *(f32x4*)(orow + x) = O[v] * (1.f / L[v]);
  }
}

// One wavefront takes the whole response of slot s (bf16 and E4M3 pages; see
// StepArgs::resp_cut), from loads to arrival, apart from the other wavefronts.
template <class SH, bool L2>
__device__ void suffix_slot_wave(const StepArgs& a, int s, int g) {
  using RM = RespMfma<SH>;
  constexpr int D = SH::D, HPK = SH::HPK;
  const int lane = threadIdx.x & 63, col = lane & 15, h = lane >> 4;
  const SlotPlan& sp = a.slot[s];
  const int last = sp.len - 1, npages = (sp.len + kPageTokens - 1) / kPageTokens;
  int32_t* ptab = a.page_table + (int64_t)sp.seq * a.pages_per_slot;
  const int pages = lane < npages ? ptab[lane] : 0;
  typename RM::Regs R;
  RM::load_round((const char*)a.pool, pages, a.Hkv, g, 0, R);
  bf16x8 bq[SH::KB];
  RM::load_q(a.q, (int64_t)s * a.Hq + g * HPK, bq);
  typename RM::NewRows N;
  const int64_t newrow = ((int64_t)s * a.Hkv + g) * SH::ROWB;
  RM::load_new((const char*)a.knew + newrow, (const char*)a.vnew + newrow, N);
  typename RM::Acc A;
  RM::round_new(N);
  RM::start_new(N, bq, a.scale_log2, A);
  RM::store_new((char*)RM::page((const char*)a.pool, sp.cur_page, a.Hkv, g), last & 15, N);
  for (int base = 0; base < last; base += RM::TOK) {
    if (base != 0) RM::load_round((const char*)a.pool, pages, a.Hkv, g, base >> 4, R);
    RM::round(R, bq, base, last, a.scale_log2, A);
  }
  if (g == 0 && lane == 0) {  // bookkeeping of this step's token (K/V stored above)
    ptab[last >> 4] = sp.cur_page;
    if (a.count_tokens)
      __hip_atomic_fetch_add(&a.tokens[(s / a.m) * a.G + sp.sample], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const Exchange<L2> ex(a);
  const int64_t rec0 = prefix_records(a, SH::PR) + ((int64_t)s * a.Hkv + g) * a.suffix_chunks_max * HPK;
  if (col < HPK) {
#pragma unroll
    for (int db = 0; db < SH::DB; ++db) ex.store4((uint32_t)(((rec0 + col) * D + db * 16 + h * 4) * 4), A.o[db]);
    if (h == 0) ex.store_ml(rec0 + col, A.m, A.lt[0]);
  }
  // counted once this wavefront's stores have completed
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0);
  if (lane == 0) __hip_atomic_fetch_add(slot_counter(a, s, g), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <class SH, bool L2, bool WAVES>
__device__ __forceinline__ void decode_block(const StepArgs& a, float* smem, unsigned long long* flagp) {
  const int item = blockIdx.x / a.Hkv;
  const int g = blockIdx.x - item * a.Hkv;
  if (L2 && threadIdx.x == 0 &&
      (__builtin_amdgcn_s_getreg(kXccIdReg) & 15) != (int)((blockIdx.x + a.l2_check_shift) % a.l2_xcds))
    __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (item < a.n_prefix_items) {
    int p = 0;
    while (p < a.num_prompts - 1 && !(a.prompt[p].nchunks > 0 && item < a.prompt[p].item_begin + a.prompt[p].nchunks))
      ++p;
    const int c = item - a.prompt[p].item_begin;
    if constexpr (SH::MFMA)
      prefix_mfma<SH, L2>(a, p, c, g, smem);
    else
      prefix_rows<SH, L2>(a, p, c, g, smem);
    arrive(a, p * a.m, a.m, g);
    return;
  }
  int it = item - a.n_prefix_items;
  if constexpr (WAVES) {  // live slot i's response and merge: wavefront i % 4 of work-group i / 4 of either kind
    const int nw = (a.n_merge_items + kWaves - 1) / kWaves;
    const int i = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (it < nw) {
      if (it * kWaves + i < a.n_merge_items) suffix_slot_wave<SH, L2>(a, a.live_slot[it * kWaves + i], g);
      return;
    }
    const int e = (it - nw - a.n_zero_items) * kWaves + i;
    if (it >= nw + a.n_zero_items) {
      if (e < a.n_merge_items) merge_wave<SH, L2, false>(a, a.o, a.live_slot[e], g, a.slot[a.live_slot[e]].target);
      return;
    }
    const int s = a.zero_slot[it - nw];
    float* o = a.o + ((int64_t)s * a.Hq + g * SH::HPK) * SH::D;
    for (int idx = threadIdx.x; idx < SH::HPK * SH::D; idx += kBlockThreads) o[idx] = 0.f;
    return;
  }
  if (it < a.n_suffix_items) {
    const int lane = threadIdx.x & 63;
    bool hit = false;
    if (lane < a.S) {
      const int len = a.slot[lane].len, b = a.slot[lane].item_begin;
      hit = len > 0 && it >= b && it < b + (len + a.split - 1) / a.split;
    }
    const int s = __ffsll((long long)__ballot(hit)) - 1;
    if (s < 0) return;  // unreachable with a consistent plan
    const int c = it - a.slot[s].item_begin;
    suffix_chunk<SH, L2>(a, s, c, g, smem);
    arrive(a, s, 1, g);
    return;
  }
  it -= a.n_suffix_items;
  if (it < a.n_zero_items) {
    const int s = a.zero_slot[it];
    float* o = a.o + ((int64_t)s * a.Hq + g * SH::HPK) * SH::D;
    for (int idx = threadIdx.x; idx < SH::HPK * SH::D; idx += kBlockThreads) o[idx] = 0.f;
    return;
  }
  it -= a.n_zero_items;
  merge_block<SH, L2>(a, a.live_slot[it], g, flagp, smem);
}

// One kernel per shape and exchange policy (L2: partials through the XCD's
// L2; the host launches the one that matches StepArgs::l2_xcds), and for bf16 one more
// of each for StepArgs::resp_cut == 2 (WAVES; in one kernel it cost the other 1.5 %:
// 28 layers, 16 slots, 439.8 against 433.3 us).  Timing mode
// (a.clock_start != null): every block folds its start and end time (device
// wall clock) into one of this launch's start / end slots.
template <class SH, bool L2, bool WAVES>
__global__ __launch_bounds__(kBlockThreads, SH::MIN_WAVES) void decode_kernel(const StepArgs a) {
  constexpr int SMEM = SH::SMEM > MergeShape<SH>::SMEM ? SH::SMEM : MergeShape<SH>::SMEM;
  __shared__ __attribute__((aligned(16))) float smem[SMEM];
  __shared__ unsigned long long flag;
  const int cs = (blockIdx.x % kClockSlots) * kClockStride;
  if (a.clock_start && threadIdx.x == 0)
    __hip_atomic_fetch_min(a.clock_start + cs, (unsigned long long)__builtin_amdgcn_s_memrealtime(), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  decode_block<SH, L2, WAVES>(a, smem, &flag);
  if (a.clock_start) {
    __syncthreads();
    if (threadIdx.x == 0)
      __hip_atomic_fetch_max(a.clock_end + cs, (unsigned long long)__builtin_amdgcn_s_memrealtime(), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ----------------------------------------------------------------------------
// Prefill: [plen, Hkv, D] -> prefix store.  A copy: bound by HBM traffic (each
// element read once, stored once) and, at one prompt and layer a launch, by the
// latency of one read and one write.
// ----------------------------------------------------------------------------
// Plain layout: whole rows move, so a thread takes kPrefillUnits 16-byte units of
// the input in input order (coalesced reads, row-sized writes), all loads first.
// blockIdx.y: 0 K, 1 V.
constexpr int kPrefillUnits = 4;
template <class SH>
__global__ __launch_bounds__(256) void prefill_plain_kernel(char* store, const char* k, const char* v, int prompt,
                                                           int plen, int hkv, int pmax) {
  const int64_t units = (int64_t)plen * hkv * SH::LPT;
  const int kind = blockIdx.y;
  const u32x4* src = (const u32x4*)(kind ? v : k);
  for (int64_t u0 = (int64_t)blockIdx.x * (kPrefillUnits * 256) + threadIdx.x; u0 < units;
       u0 += (int64_t)gridDim.x * (kPrefillUnits * 256)) {
    u32x4 r[kPrefillUnits];
#pragma unroll
    for (int i = 0; i < kPrefillUnits; ++i) r[i] = src[min(u0 + i * 256, units - 1)];
#pragma unroll
    for (int i = 0; i < kPrefillUnits; ++i) {
      const int64_t u = u0 + i * 256;
      if (u >= units) break;
      const int ch = (int)(u % SH::LPT);
      const uint32_t row = (uint32_t)(u / SH::LPT);  // plen * hkv: a store of 2^32 rows is beyond any memory
      const uint32_t j = row / (uint32_t)hkv, g = row - j * (uint32_t)hkv;
      char* dst = store + ((((int64_t)prompt * hkv + g) * 2 + kind) * pmax + j) * SH::ROWB;
      *((u32x4*)dst + ch) = r[i];
    }
  }
}

// MFMA layout per (prompt, kv head), per 32-token block: a K block of
// [2 token halves][KB][64 lanes][8] and a V block of [DB][64 lanes][8].
// K unit (mb, kb, lane): tokens mb*16 + lane%16, dims kb*32 + 8*(lane/16) + e.
// V unit (db, lane): dim db*16 + lane%16, tokens tau(8*(lane/16) + e) where
// tau(8q+e) = 4q+e for e < 4 and 16+4q+(e-4) otherwise -- the order in which
// a lane holds probabilities after the S^T tiles.  Padding tokens are zero.
//
// One work-group per (block, KV head), KV heads fastest.  A K unit is 16
// contiguous bytes of the input; a V unit gathers one element of eight rows, so
// the block's V rows (16-byte loads) are turned in LDS.  The row pitch of 4
// dwords past the row puts the four token groups of a unit's 64 lanes on
// disjoint banks.  A prompt of 2048 tokens, 8 KV heads, d = 128, bf16 (16.8 MB
// moved) takes 5.5 us (rocprofv3; 3.0 TB/s) where a thread gathering each unit's
// eight elements one by one took 10.7 us; the copy alone is 3.5 us at the rate of
// a large copy.
template <class SH>
__global__ __launch_bounds__(256) void prefill_mfma_kernel(char* store, const uint16_t* k, const uint16_t* v,
                                                          int prompt, int plen, int hkv, int pmax) {
  constexpr int D = SH::D, KB = SH::KB, DB = SH::DB, KES = SH::KES;
  constexpr int KU = 2 * KB * 64, VU = DB * 64;  // units of a block
  constexpr int RU = D / 8, PITCH = D + 8;       // 16-byte units and LDS elements of a V row
  static_assert(KU % 256 == 0 && VU % 256 == 0 && kMfmaBlock * RU == VU, "whole rounds of a work-group");
  __shared__ __attribute__((aligned(16))) uint16_t vt[kMfmaBlock * PITCH];
  const int64_t items = (int64_t)hkv * ((plen + kMfmaBlock - 1) / kMfmaBlock);
  for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const int g = (int)(item % hkv), b = (int)(item / hkv), t0 = b * kMfmaBlock;
    char* blk = store + (((int64_t)prompt * hkv + g) * (pmax / kMfmaBlock) + b) * (2 * kMfmaBlock * D * KES);
    auto load = [&](const uint16_t* x, int tok, int d0) {  // eight elements of a row, zero past the prompt
      const u32x4 w = *(const u32x4*)(x + ((int64_t)min(tok, plen - 1) * hkv + g) * D + d0);
      return tok < plen ? w : u32x4{0, 0, 0, 0};
    };
    u32x4 vr[VU / 256], kr[KU / 256];
#pragma unroll
    for (int i = 0; i < VU / 256; ++i) {
      const int x = i * 256 + threadIdx.x;
      vr[i] = load(v, t0 + x / RU, (x % RU) * 8);
    }
#pragma unroll
    for (int i = 0; i < KU / 256; ++i) {
      const int x = i * 256 + threadIdx.x, lane = x & 63, sub = x >> 6, mb = sub / KB, kb = sub - mb * KB;
      kr[i] = load(k, t0 + mb * 16 + (lane & 15), kb * 32 + (lane >> 4) * 8);
    }
#pragma unroll
    for (int i = 0; i < VU / 256; ++i) {
      const int x = i * 256 + threadIdx.x;
      *(u32x4*)(vt + (x / RU) * PITCH + (x % RU) * 8) = vr[i];
    }
#pragma unroll
    for (int i = 0; i < KU / 256; ++i) st_kv<SH>(blk + (int64_t)(i * 256 + threadIdx.x) * 8 * KES, kr[i]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < VU / 256; ++i) {
      const int x = i * 256 + threadIdx.x, lane = x & 63, db = x >> 6, qq = lane >> 4;
      const uint16_t* col = vt + db * 16 + (lane & 15);
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const int tok = e < 4 ? 4 * qq + e : 16 + 4 * qq + (e - 4);
        w[e / 2] = col[tok * PITCH] | ((uint32_t)col[(tok + 1) * PITCH] << 16);
      }
      st_kv<SH>(blk + (int64_t)kMfmaBlock * D * KES + (int64_t)x * 8 * KES, u32x4{w[0], w[1], w[2], w[3]});
    }
    __syncthreads();  // the next block's rows overwrite vt
  }
}

}  // namespace
}  // namespace infs
