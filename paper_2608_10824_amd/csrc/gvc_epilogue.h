// Work-unit maps and fused epilogues shared by the GEMM kernels (k_gemm.hip,
// k_tile.hip).
#pragma once
#include "gvc_kernels.h"
#include "gvc_sync.h"

namespace gvc {

typedef unsigned u32x4b __attribute__((ext_vector_type(4)));
#define GPB(p) ((const void __attribute__((address_space(1)))*)(p))
#define LPB(p) ((void __attribute__((address_space(3)))*)(p))

__device__ __forceinline__ void map_pair(const GemmArgs& a, int pair, int& mat_a, int& blk_a, int& mat_b,
                                         int& blk_b, bool& b_ok) {
  b_ok = true;
  if (a.map == MAP_QKV) {
    const int dh = a.e.head_dim;
    const int per_mat = a.wblk[0] >> 1;        // pairs per d x d matrix
    const int m = pair / per_mat, pp = pair % per_mat;
    const int per_head = dh >> 5;              // pairs per head
    const int head = pp / per_head, j = pp % per_head;
    mat_a = mat_b = m;
    blk_a = head * (dh >> 4) + j;
    blk_b = blk_a + per_head;
  } else if (a.map == MAP_GU) {
    mat_a = 0; mat_b = 1; blk_a = blk_b = pair;
  } else if (a.map == MAP_SINGLE) {
    mat_a = mat_b = 0; blk_a = blk_b = pair; b_ok = false;
  } else if (a.map == MAP_QKV_SINGLE) {
    mat_a = mat_b = pair / a.wblk[0]; blk_a = blk_b = pair % a.wblk[0]; b_ok = false;
  } else {
    mat_a = mat_b = 0;
    blk_a = 2 * pair;
    blk_b = 2 * pair + 1;
    if (blk_b >= a.wblk[0]) { blk_b = blk_a; b_ok = false; }
  }
}

__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

// GELU, tanh form: x/2 (1 + tanh(sqrt(2/pi) (x + 0.044715 x^3))).
__device__ __forceinline__ float gelu_f(float x) {
  return 0.5f * x * (1.0f + tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x)));
}

__device__ __forceinline__ void add_bias(floatx4& v, const float* bias, int f) {
  const float4 b = *(const float4*)(bias + f);
  v[0] += b.x; v[1] += b.y; v[2] += b.z; v[3] += b.w;
}

// RoPE of the pair (a, b) of dims i and i + d_h/2.  The fused multiply-adds are
// written out: left to the compiler, two kernels could round differently.
__device__ __forceinline__ float rope_lo(float a, float b, float c, float s) { return __builtin_fmaf(a, c, -(b * s)); }
__device__ __forceinline__ float rope_hi(float a, float b, float c, float s) { return __builtin_fmaf(b, c, a * s); }

// Epilogue of one lane: 4 consecutive output features of block A and of
// block B for token row m.  Every lane of the wave calls it (some epilogues
// shuffle across lanes); `valid` says whether row m exists (m is already
// clamped into range for address arithmetic).  rs scales the accumulators
// (folded RMSNorm, 1 otherwise).
template <int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int pair, int lane, int m, floatx4 va, floatx4 vb,
                                         bool b_ok, bool valid, float rs) {
  const EpiArgs& e = a.e;
  int mat_a, blk_a, mat_b, blk_b; bool bo;
  map_pair(a, pair, mat_a, blk_a, mat_b, blk_b, bo);
  va *= rs;
  vb *= rs;
  const int sub = (lane >> 4) * 4;   // first of the 4 features this lane holds
  if constexpr (EPI == EPI_QKV) {
    if (!valid) return;
    const int dh = e.head_dim, half = dh >> 1;
    const int head = blk_a / (dh >> 4);
    const int ia = (blk_a % (dh >> 4)) * 16 + sub;   // dim within head, < half
    const int pos = e.rows.pos[m];
    const int b = e.rows.ep[m];
    if (e.bias[mat_a]) {
      add_bias(va, e.bias[mat_a], blk_a * 16 + sub);
      add_bias(vb, e.bias[mat_a], blk_b * 16 + sub);
    }
    float ra[4], rb[4];
    if (mat_a < 2 && e.rope) {
      const float2* cs = e.rope + (size_t)pos * half + ia;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 c = cs[i];
        ra[i] = rope_lo(va[i], vb[i], c.x, c.y);
        rb[i] = rope_hi(va[i], vb[i], c.x, c.y);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) { ra[i] = va[i]; rb[i] = vb[i]; }
    }
    if (mat_a == 0) {
      bf16* q = e.q + (size_t)m * e.d + head * dh;
      u16x4 oa = {f2bf(ra[0]), f2bf(ra[1]), f2bf(ra[2]), f2bf(ra[3])};
      u16x4 ob = {f2bf(rb[0]), f2bf(rb[1]), f2bf(rb[2]), f2bf(rb[3])};
      *(u16x4*)(q + ia) = oa;
      *(u16x4*)(q + ia + half) = ob;
    } else if (mat_a == 1) {
      bf16* k = e.kc + ((size_t)(b * e.n_heads + head) * e.kv_pad + pos) * dh;
      u16x4 oa = {f2bf(ra[0]), f2bf(ra[1]), f2bf(ra[2]), f2bf(ra[3])};
      u16x4 ob = {f2bf(rb[0]), f2bf(rb[1]), f2bf(rb[2]), f2bf(rb[3])};
      *(u16x4*)(k + ia) = oa;
      *(u16x4*)(k + ia + half) = ob;
    } else {
      bf16* v = e.vc + (size_t)(b * e.n_heads + head) * dh * e.kv_pad + pos;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[(size_t)(ia + i) * e.kv_pad] = f2bf(ra[i]);
        v[(size_t)(ia + half + i) * e.kv_pad] = f2bf(rb[i]);
      }
    }
  } else if constexpr (EPI == EPI_QKV_RAW) {
    // single block of q, k or v for decode rows: q and k stay fp32 and
    // un-rotated (the decode attention rotates them), v goes to the cache
    if (!valid) return;
    const int f = blk_a * 16 + sub;
    if (mat_a == 0) {
      *(float4*)(e.qraw + (size_t)m * e.d + f) = float4{va[0], va[1], va[2], va[3]};
    } else if (mat_a == 1) {
      *(float4*)(e.kraw + (size_t)m * e.d + f) = float4{va[0], va[1], va[2], va[3]};
    } else {
      const int dh = e.head_dim, head = f / dh, dim = f % dh;
      bf16* v = e.vc + ((size_t)(e.rows.ep[m] * e.n_heads + head) * dh + dim) * e.kv_pad + e.rows.pos[m];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[(size_t)i * e.kv_pad] = f2bf(va[i]);
    }
  } else if constexpr (EPI == EPI_RESID) {
    const int d = e.d;
    const size_t ri = (size_t)(e.resid_mapped ? e.rows.idx[m] : m) * d;
    const size_t oi = (size_t)(e.out_mapped ? e.rows.idx[m] : m) * d;
    const int fa = blk_a * 16 + sub, fb = blk_b * 16 + sub;
    if (e.bias[0]) {
      add_bias(va, e.bias[0], fa);
      if (b_ok) add_bias(vb, e.bias[0], fb);
    }
    const float4 r0 = *(const float4*)(e.resid + ri + fa);
    const float4 oa = {r0.x + va[0], r0.y + va[1], r0.z + va[2], r0.w + va[3]};
    float4 ob = {0.f, 0.f, 0.f, 0.f};
    if (b_ok) {
      const float4 r1 = *(const float4*)(e.resid + ri + fb);
      ob = float4{r1.x + vb[0], r1.y + vb[1], r1.z + vb[2], r1.w + vb[3]};
    }
    if (valid) {
      *(float4*)(e.out + oi + fa) = oa;
      if (b_ok) *(float4*)(e.out + oi + fb) = ob;
    }
    if (e.xn) {   // folded RMSNorm input of the next projection
      const float4 ga = *(const float4*)(e.xn_gain + fa);
      float ss = oa.x * oa.x + oa.y * oa.y + oa.z * oa.z + oa.w * oa.w;
      if (valid)
        *(u16x4*)(e.xn + frag_off(m, fa, e.xn_kb)) =
            u16x4{f2bf(oa.x * ga.x), f2bf(oa.y * ga.y), f2bf(oa.z * ga.z), f2bf(oa.w * ga.w)};
      if (b_ok) {
        const float4 gb = *(const float4*)(e.xn_gain + fb);
        ss += ob.x * ob.x + ob.y * ob.y + ob.z * ob.z + ob.w * ob.w;
        if (valid)
          *(u16x4*)(e.xn + frag_off(m, fb, e.xn_kb)) =
              u16x4{f2bf(ob.x * gb.x), f2bf(ob.y * gb.y), f2bf(ob.z * gb.z), f2bf(ob.w * gb.w)};
      }
      ss += __shfl_xor(ss, 16);
      ss += __shfl_xor(ss, 32);
      if (valid && lane < 16) e.ssq_out[(size_t)m * e.ssq_out_parts + pair] = ss;
    }
  } else if constexpr (EPI == EPI_SILU) {
    const int f = blk_a * 16 + sub;
    if (valid && f < e.n_feat) {
      u16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = f2bf(silu_f(va[i]) * vb[i]);
      *(u16x4*)(e.act + frag_off(m, f, e.kb_act)) = o;
    }
  } else if constexpr (EPI == EPI_GELU) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && !b_ok) break;
      const int f = (half ? blk_b : blk_a) * 16 + sub;
      floatx4 v = half ? vb : va;
      if (!valid || f >= e.n_feat) continue;
      if (e.bias[0]) add_bias(v, e.bias[0], f);
      const u16x4 o = {f2bf(gelu_f(v[0])), f2bf(gelu_f(v[1])), f2bf(gelu_f(v[2])), f2bf(gelu_f(v[3]))};
      *(u16x4*)(e.act + frag_off(m, f, e.kb_act)) = o;
    }
  } else if constexpr (EPI == EPI_PATCH) {
    if (!valid) return;
    const float inv255 = 1.0f / 255.0f;
    float* o = e.store + (size_t)m * e.ld_store;
    const float* pt = e.pos_tab + (size_t)e.rows.pos[m] * e.ld_store;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && !b_ok) break;
      const int f = (half ? blk_b : blk_a) * 16 + sub;
      const floatx4& v = half ? vb : va;
      const float4 bb = *(const float4*)(e.bias[0] + f), pp = *(const float4*)(pt + f);
      *(float4*)(o + f) = float4{v[0] * inv255 + bb.x + pp.x, v[1] * inv255 + bb.y + pp.y,
                                 v[2] * inv255 + bb.z + pp.z, v[3] * inv255 + bb.w + pp.w};
    }
  } else if constexpr (EPI == EPI_STORE) {
    if (!valid) return;
    float* o = e.store + (size_t)m * e.ld_store;
    const int fa = blk_a * 16 + sub;
    if (fa < a.n_out) *(float4*)(o + fa) = float4{va[0], va[1], va[2], va[3]};
    const int fb = blk_b * 16 + sub;
    if (b_ok && fb < a.n_out) *(float4*)(o + fb) = float4{vb[0], vb[1], vb[2], vb[3]};
  } else {  // EPI_EMBED
    if (!valid) return;
    const int d = e.d;
    const int pos = e.rows.pos[m], b = e.rows.ep[m];
    float* h = e.h0 + (size_t)e.rows.idx[m] * d;
    const float sc = e.vis_scale;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && !b_ok) break;
      const int f = (half ? blk_b : blk_a) * 16 + sub;
      const floatx4& v = half ? vb : va;
      float4 o;
      if (pos >= 1 && pos <= e.n_patches) {
        o.x = v[0] * sc; o.y = v[1] * sc; o.z = v[2] * sc; o.w = v[3] * sc;
        if (e.bias[0]) {
          const float4 bb = *(const float4*)(e.bias[0] + f);
          o.x += bb.x; o.y += bb.y; o.z += bb.z; o.w += bb.w;
        }
      } else if (pos < e.n_patches + e.n_text) {
        const int t = pos == 0 ? 0 : pos - e.n_patches;
        const bf16* er = e.embed + (size_t)min(max(e.text_ids[b * e.n_text + t], 0), e.n_vocab - 1) * d + f;
        o.x = bf2f(er[0]); o.y = bf2f(er[1]); o.z = bf2f(er[2]); o.w = bf2f(er[3]);
      } else {
        const float* xr = e.extra + ((size_t)b * e.n_extra + (pos - e.n_patches - e.n_text)) * d + f;
        o = *(const float4*)xr;
      }
      *(float4*)(h + f) = o;
    }
  }
}

}  // namespace gvc
