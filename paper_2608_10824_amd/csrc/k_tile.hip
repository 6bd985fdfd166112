// Tiled GEMM of the prompt pass for launches that fill the chip with whole
// tiles: every projection of the many-row sessions, and those launches of the
// others that gemm_route() gives it.
//
// A workgroup of WW x WT waves owns WW * WP weight pairs x WT * TB blocks of
// 16 token rows and walks the whole k range in order.  Every k step, both
// operands' fragments of the tile are copied straight into LDS
// (global_load_lds), S stages deep; wave (ww, wt) holds the fragments of step
// k in registers and multiplies them while those of step k + 1 are read from
// LDS, the reads spread between the MFMAs.  A wave tile of 2 WP x TB blocks
// reads 2 WP + TB fragments per 2 WP * TB MFMAs, and with the reads in front of
// the MFMAs (one register set, the kernel before this one) LDS and the matrix
// cores took turns.  7B projections alone, reads in front -> beside (best shape
// each): 2368 rows QKV 287 -> 234 us, output 94 -> 79, down 242 -> 191; 736 rows
// 98 -> 77, 45 -> 35, gate/up 148 -> 135, down 143 -> 87.  What bounds it now:
// at 2368 rows the matrix cores are busy 41-57% of the cycles and LDS reads 19-24%
// (no bank conflicts), while the tiles draw 9-11 TB/s from the L2s (gate/up 3.7 GB
// in 380 us, down 2.2 GB in 197); at 276 rows 24-36% and 17-25%, and the same 10
// TB/s.
// Against split-k with fp32 partial sums and a kernel that adds them: 589 rows
// QKV 147 -> 72 us, output 76 -> 32, gate/up 214 -> 123, down 121 -> 82; 282
// rows QKV 56 -> 47, gate/up 89 -> 60 (launches alone; gemm_route has passes).
// Ten shapes, because whole rounds of workgroups on 256 CUs leave a rest that
// depends on the sizes.
//
// A row's sum runs over k in order, so it does not depend on the tile.  With
// SL the sum is cut into the split-k launches' slices: a slice is summed from
// zero and added to the total, which gives bit for bit what those launches
// and k_gemm_ks (its k shares) give, so a session may choose by row count.
#include <algorithm>
#include <atomic>

#include "gvc_epilogue.h"

namespace gvc {

// Epilogue of one wave: accumulators v of WP pairs (from pair0) x TB token
// blocks (from tb0).  The fused epilogue of one (pair, block) loads its row's
// numbers, then what they point to (RoPE, residual), then stores; one after
// the other that chain cost a 7B QKV launch of 2368 rows 20 us per round of
// tiles.  For QKV and the residual the row numbers of all blocks are loaded
// first, and a block's operands while the block before it is stored (with
// RoPE, without biases and the folded norm: launch_gemm_tile sees to it).
template <int EPI, int WP, int TB>
__device__ __forceinline__ void tile_epilogue(const GemmArgs& a, int pair0, int lane, int tb0,
                                              const floatx4 (&v)[2 * WP][TB]) {
  const EpiArgs& e = a.e;
  const int col = lane & 15, sub = (lane >> 4) * 4;
  auto row = [&](int j) { return (tb0 + j) * 16 + col; };
  if constexpr (EPI == EPI_QKV) {
    const int dh = e.head_dim, half = dh >> 1;
    int pos[TB], ep[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int m = min(row(j), a.M - 1);
      pos[j] = e.rows.pos[m];
      ep[j] = e.rows.ep[m];
    }
    int mat[WP], head[WP], ia[WP];
#pragma unroll
    for (int p = 0; p < WP; ++p) {
      int mb, bb, ba; bool ok;
      map_pair(a, min(pair0 + p, a.n_pairs - 1), mat[p], ba, mb, bb, ok);
      head[p] = ba / (dh >> 4);
      ia[p] = (ba % (dh >> 4)) * 16 + sub;   // dim within head, < half
    }
    float4 cs[2][WP][2];   // (cos, sin) of 4 dims
    auto load = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int p = 0; p < WP; ++p) {
        const float4* r = (const float4*)(e.rope + (size_t)pos[j] * half + ia[p]);
        cs[j & 1][p][0] = r[0];
        cs[j & 1][p][1] = r[1];
      }
    };
    load(0);
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      if (j + 1 < TB) load(j + 1);
      const int m = row(j);
#pragma unroll
      for (int p = 0; p < WP; ++p) {
        if (pair0 + p >= a.n_pairs || m >= a.M) continue;
        const floatx4 va = v[2 * p][j], vb = v[2 * p + 1][j];
        if (mat[p] < 2) {
          const float4 c0 = cs[j & 1][p][0], c1 = cs[j & 1][p][1];
          const float c[4] = {c0.x, c0.z, c1.x, c1.z}, s[4] = {c0.y, c0.w, c1.y, c1.w};
          u16x4 oa, ob;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            oa[i] = f2bf(rope_lo(va[i], vb[i], c[i], s[i]));
            ob[i] = f2bf(rope_hi(va[i], vb[i], c[i], s[i]));
          }
          bf16* o = mat[p] == 0 ? e.q + (size_t)m * e.d + head[p] * dh
                                : e.kc + ((size_t)(ep[j] * e.n_heads + head[p]) * e.kv_pad + pos[j]) * dh;
          *(u16x4*)(o + ia[p]) = oa;
          *(u16x4*)(o + ia[p] + half) = ob;
        } else {
          bf16* o = e.vc + (size_t)(ep[j] * e.n_heads + head[p]) * dh * e.kv_pad + pos[j];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            o[(size_t)(ia[p] + i) * e.kv_pad] = f2bf(va[i]);
            o[(size_t)(ia[p] + half + i) * e.kv_pad] = f2bf(vb[i]);
          }
        }
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
    size_t ri[TB], oi[TB];
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      const int m = min(row(j), a.M - 1), x = e.resid_mapped || e.out_mapped ? e.rows.idx[m] : m;
      ri[j] = (size_t)(e.resid_mapped ? x : m) * e.d;
      oi[j] = (size_t)(e.out_mapped ? x : m) * e.d;
    }
    const int last = 16 * a.wblk[0] - 4;   // blocks past the matrix re-read its last features
    float4 r[2][2 * WP];
    auto load = [&](int j) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2 * WP; ++q)
        r[j & 1][q] = *(const float4*)(e.resid + ri[j] + min((2 * pair0 + q) * 16 + sub, last));
    };
    load(0);
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      if (j + 1 < TB) load(j + 1);
      if (row(j) >= a.M) continue;
#pragma unroll
      for (int q = 0; q < 2 * WP; ++q) {
        const float4 x = r[j & 1][q];
        const floatx4& y = v[q][j];
        if (2 * pair0 + q < a.wblk[0])
          *(float4*)(e.out + oi[j] + (2 * pair0 + q) * 16 + sub) =
              float4{x.x + y[0], x.y + y[1], x.z + y[2], x.w + y[3]};
      }
    }
  } else {
#pragma unroll
    for (int p = 0; p < WP; ++p) {
      if (pair0 + p >= a.n_pairs) continue;
      int ma, ba, mb, bb; bool b_ok;
      map_pair(a, pair0 + p, ma, ba, mb, bb, b_ok);
#pragma unroll
      for (int j = 0; j < TB; ++j) {
        const int m = row(j);
        epilogue<EPI>(a, pair0 + p, lane, min(m, a.M - 1), v[2 * p][j], v[2 * p + 1][j], b_ok, m < a.M, 1.0f);
      }
    }
  }
}

template <int EPI, int WP, int TB, int WW, int WT, int S, int OCC, bool SL>
__global__ __launch_bounds__(WW * WT * 64, OCC) void k_gemm_tile(const GemmArgs a, int mtiles, int ntiles) {
  constexpr int NW = WW * WT, WF = 2 * WW * WP, TF = WT * TB, FR = WF + TF;
  constexpr int LPW = (FR + NW - 1) / NW;   // fragment copies per wave per k step
  static_assert(S >= 3 && (S - 2) * LPW < 64, "vmcnt range");
  extern __shared__ u32x4b tile_lds[];      // [S][FR][64]
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ww = wv % WW, wt = wv / WW;
  // XCD-aware order: all tiles of one weight tile run on XCD (tile % 8) and
  // share its weights in that L2; within an XCD, jobs run in groups of 8
  // token tiles x all of the XCD's weight tiles, so the workgroups resident
  // at one time share both operands' tiles
  const int x = blockIdx.x, xcd = x & 7, i = x >> 3;
  const int nnt = (ntiles + 7) / 8, g = i / (8 * nnt), r = i % (8 * nnt);
  const int gs = min(8, mtiles - g * 8);
  const int nt = xcd + 8 * (r / gs), mt = g * 8 + r % gs;
  if (nt >= ntiles) return;
  const int pair0 = nt * WW * WP, tb0 = mt * TF, KB = a.KB;
  const bf16x8* src[LPW];
  int dst[LPW];
#pragma unroll
  for (int l = 0; l < LPW; ++l) {
    const int f = min(wv + l * NW, FR - 1);
    dst[l] = f;
    if (f < WF) {
      int ma, ba, mb, bb; bool ok;
      map_pair(a, min(pair0 + f / 2, a.n_pairs - 1), ma, ba, mb, bb, ok);
      src[l] = ((f & 1) ? a.w[mb] + (size_t)bb * KB * 64 : a.w[ma] + (size_t)ba * KB * 64) + lane;
    } else {
      src[l] = a.x + (size_t)min(tb0 + f - WF, a.mblocks - 1) * KB * 64 + lane;
    }
  }
  int fill = 0, fill_k = 0, rd_stage = 0;   // next stage to fill and its k step; next stage to read
  auto issue = [&]() __attribute__((always_inline)) {   // k steps past the end re-read the last one (in bounds)
    u32x4b* st = tile_lds + fill * FR * 64;
    const size_t o = (size_t)min(fill_k, KB - 1) * 64;
#pragma unroll
    for (int l = 0; l < LPW; ++l) __builtin_amdgcn_global_load_lds(GPB(src[l] + o), LPB(st + dst[l] * 64), 16, 0, 0);
    ++fill_k;
    fill = fill + 1 == S ? 0 : fill + 1;
  };
  floatx4 acc[2 * WP][TB], tot[SL ? 2 * WP : 1][SL ? TB : 1];
#pragma unroll
  for (int p = 0; p < 2 * WP; ++p)
#pragma unroll
    for (int j = 0; j < TB; ++j) {
      acc[p][j] = floatx4{0, 0, 0, 0};
      if constexpr (SL) tot[p][j] = floatx4{0, 0, 0, 0};
    }
  typedef bf16x8 WFrag[2 * WP];
  typedef bf16x8 XFrag[TB];
  auto read = [&](WFrag& w, XFrag& t) __attribute__((always_inline)) {
    const u32x4b* st = tile_lds + rd_stage * FR * 64;
#pragma unroll
    for (int j = 0; j < TB; ++j) t[j] = __builtin_bit_cast(bf16x8, st[(WF + wt * TB + j) * 64 + lane]);
#pragma unroll
    for (int p = 0; p < 2 * WP; ++p) w[p] = __builtin_bit_cast(bf16x8, st[(2 * ww * WP + p) * 64 + lane]);
    rd_stage = rd_stage + 1 == S ? 0 : rd_stage + 1;
  };
  auto multiply = [&](const WFrag& w, const XFrag& t) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 2 * WP; ++p)
#pragma unroll
      for (int j = 0; j < TB; ++j) acc[p][j] = mfma16(w[p], t[j], acc[p][j]);
  };
  int slice_end = SL ? a.sk_steps : 0;
  auto end_slice = [&](int k) __attribute__((always_inline)) {   // after the k-th step (from 1)
    if (!SL || (k != slice_end && k != KB)) return;
    slice_end += a.sk_steps;
    if constexpr (SL)
#pragma unroll
      for (int p = 0; p < 2 * WP; ++p)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          tot[p][j] += acc[p][j];
          acc[p][j] = floatx4{0, 0, 0, 0};
        }
  };
#pragma unroll
  for (int c = 0; c < S - 1; ++c) issue();
  wait_vmcnt<(S - 2) * LPW>();
  lds_barrier();
  WFrag wa, wb;
  XFrag xa, xb;
  read(wa, xa);
  // Step k: w0, x0 hold its fragments; those of step k + 1 are read beside its
  // MFMAs.  The stage filled here last held step k - 1, whose reads every
  // wave had finished before its MFMAs, so before this barrier.
  auto step = [&](const WFrag& w0, const XFrag& x0, WFrag& w1, XFrag& x1) __attribute__((always_inline)) {
    wait_vmcnt<(S - 3) * LPW>();
    lds_barrier();
    issue();
    read(w1, x1);
    multiply(w0, x0);
    constexpr int NR = 2 * WP + TB, NM = 2 * WP * TB;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);         // an LDS read,
      __builtin_amdgcn_sched_group_barrier(0x008, NM / NR, 0);   // then its share of the MFMAs
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NM - NM / NR * NR, 0);
  };
  int k = 0;
  for (; k + 2 <= KB; k += 2) {
    step(wa, xa, wb, xb);
    end_slice(k + 1);
    step(wb, xb, wa, xa);
    end_slice(k + 2);
  }
  if (k < KB) {
    multiply(wa, xa);
    end_slice(KB);
  }
  wait_vmcnt<0>();   // direct-to-LDS loads must land before the workgroup ends
  if constexpr (SL)
    tile_epilogue<EPI, WP, TB>(a, pair0 + ww * WP, lane, tb0 + wt * TB, tot);
  else
    tile_epilogue<EPI, WP, TB>(a, pair0 + ww * WP, lane, tb0 + wt * TB, acc);
}

// Shapes: weight blocks x token blocks of a workgroup's tile, workgroups per
// CU, and what a k step takes (ns) with one and with all of them resident,
// measured on the 7B projections at 148-2368 rows with most CUs busy.
struct TileShape {
  int wblk, tblk, occ;
  float one, all;
};
constexpr TileShape kTiles[] = {
    {6, 10, 1, 300, 300},  {4, 10, 2, 234, 370},  {12, 10, 1, 425, 435}, {8, 6, 2, 246, 390},  {12, 12, 1, 480, 510},
    {16, 10, 1, 520, 520}, {16, 16, 1, 740, 740}, {8, 10, 2, 370, 540},  {16, 14, 1, 680, 680}, {16, 12, 1, 600, 600},
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int kSlicedTiles = 5;   // the first ones also have an SL form (its totals fit the registers)

// Workgroups of a launch, as if the fullest XCD's were on each of the 8: all
// tiles of a weight tile run on one XCD (12-block tiles of the 7B output
// projection are 22 weight tiles, three on six XCDs and two on the others:
// 4416 rows take three rounds, 346 us on average with the down projection,
// where 16-block tiles take two, 262).
static int tile_count(const GemmArgs& a, const TileShape& t) {
  const int ntiles = (2 * a.n_pairs + t.wblk - 1) / t.wblk;
  return (ntiles + 7) / 8 * 8 * ((a.mblocks + t.tblk - 1) / t.tblk);
}

// Time of a launch in ns: whole rounds of resident workgroups, then the rest,
// at the measured step times, plus launch and epilogue.
static float tile_time(const GemmArgs& a, const TileShape& t, int cus) {
  const int n = tile_count(a, t), full = n / (t.occ * cus), rem = n % (t.occ * cus);
  float all = t.all;
  // 6-block tiles, two to a weight tile, on part of the CUs twice: 1.21 to 1.29
  // times that at widths 2560-5120 (7B gate/up at 164 rows: 73.5 us, 12 x 10 tiles 63)
  if (t.tblk == 6 && full == 0 && a.mblocks <= 12) all *= 1.25f;
  const float steps = full * all + (rem == 0 ? 0.f : (rem > cus ? all : t.one));
  return a.KB * steps + 10000.f + 4000.f * (full + (rem > 0) - 1);
}

hipError_t device_cus(int& cus) {
  static std::atomic<int> known{0};
  cus = known.load(std::memory_order_relaxed);
  if (cus > 0) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (cus <= 0) return hipErrorInvalidDevice;
  known.store(cus, std::memory_order_relaxed);
  return hipSuccess;
}

template <int EPI, int WP, int TB, int WW, int WT, int S, int OCC, bool SL>
static hipError_t launch_tile_one(const GemmArgs& a, hipStream_t s) {
  constexpr int lds = S * (2 * WW * WP + WT * TB) * 1024;
  static_assert(lds <= 160 * 1024, "LDS");
  static std::atomic<bool> attr{false};
  if (!attr.load(std::memory_order_acquire)) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_tile<EPI, WP, TB, WW, WT, S, OCC, SL>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr.store(true, std::memory_order_release);
  }
  const int mtiles = (a.mblocks + WT * TB - 1) / (WT * TB), ntiles = (a.n_pairs + WW * WP - 1) / (WW * WP);
  hipLaunchKernelGGL((k_gemm_tile<EPI, WP, TB, WW, WT, S, OCC, SL>), dim3(8 * ((ntiles + 7) / 8) * mtiles),
                     dim3(WW * WT * 64), lds, s, a, mtiles, ntiles);
  return hipGetLastError();
}

template <int EPI, bool SL>
static hipError_t launch_tile_shape(const GemmArgs& a, int shape, hipStream_t s) {
  switch (shape) {   // as in kTiles
    case 0: return launch_tile_one<EPI, 1, 5, 3, 2, 8, 1, SL>(a, s);
    case 1: return launch_tile_one<EPI, 1, 5, 2, 2, 5, 2, SL>(a, s);
    case 2: return launch_tile_one<EPI, 1, 5, 6, 2, 7, 2, SL>(a, s);
    case 3: return launch_tile_one<EPI, 2, 3, 2, 2, 5, 2, SL>(a, s);
    case 4: return launch_tile_one<EPI, 3, 3, 2, 4, 6, 2, SL>(a, s);
    default: break;
  }
  if constexpr (!SL) {
    switch (shape) {
      case 5: return launch_tile_one<EPI, 2, 5, 4, 2, 5, 2, SL>(a, s);
      case 6: return launch_tile_one<EPI, 4, 4, 2, 4, 5, 2, SL>(a, s);
      case 7: return launch_tile_one<EPI, 2, 5, 2, 2, 4, 2, SL>(a, s);
      case 8: return launch_tile_one<EPI, 2, 7, 4, 2, 5, 2, SL>(a, s);
      case 9: return launch_tile_one<EPI, 2, 6, 4, 2, 5, 2, SL>(a, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

// The shape that tile_time puts first.
static int best_tile(const GemmArgs& a, int n_shapes, int cus) {
  int best = 0;
  for (int i = 1; i < n_shapes; ++i)
    if (tile_time(a, kTiles[i], cus) < tile_time(a, kTiles[best], cus)) best = i;
  return best;
}

// Sliced launch, in us.  (Launches of the residual projections took 0.85 to 1.05
// of tile_time, 0.93 at the median of 800.)
static float gemm_tile_time(const GemmArgs& a, int cus) {
  return 0.93e-3f * tile_time(a, kTiles[best_tile(a, kSlicedTiles, cus)], cus);
}

hipError_t launch_gemm_tile(const GemmArgs& a, int epi, hipStream_t s) {
  if (a.map == MAP_SINGLE || a.map == MAP_QKV_SINGLE || a.e.ssq_in) return hipErrorInvalidValue;
  if (epi == EPI_QKV && (a.e.bias[0] || a.e.bias[1] || a.e.bias[2] || !a.e.rope)) return hipErrorInvalidValue;
  if (epi == EPI_RESID && (a.e.bias[0] || a.e.xn || a.map != MAP_PLAIN)) return hipErrorInvalidValue;
  int cus = 0;
  const hipError_t e = device_cus(cus);
  if (e != hipSuccess) return e;
  const bool sl = a.sk_steps > 0;
  const int n = sl ? kSlicedTiles : kNumTiles;
  const int shape = a.tile_shape >= 1 && a.tile_shape <= n ? a.tile_shape - 1 : best_tile(a, n, cus);
  switch (epi) {
    case EPI_QKV: return sl ? launch_tile_shape<EPI_QKV, true>(a, shape, s) : launch_tile_shape<EPI_QKV, false>(a, shape, s);
    case EPI_RESID:
      return sl ? launch_tile_shape<EPI_RESID, true>(a, shape, s) : launch_tile_shape<EPI_RESID, false>(a, shape, s);
    case EPI_SILU:
      return sl ? launch_tile_shape<EPI_SILU, true>(a, shape, s) : launch_tile_shape<EPI_SILU, false>(a, shape, s);
    case EPI_EMBED: return sl ? hipErrorInvalidValue : launch_tile_shape<EPI_EMBED, false>(a, shape, s);
    default: return hipErrorInvalidValue;
  }
}

// The kernel of a split-k session's launch.  Up to 10 token blocks a split-k
// launch is one token tile and level or ahead (7B gate/up at 148 rows 48 us in a
// prompt pass, tile kernel 52; QKV 40 and 40).  Above, QKV and gate/up launches
// fill the chip with whole tiles: split-k was behind at every width of 512-5120
// and 161-1000 rows (width 512: 18 us, tile kernel 13; 4096 at 176 rows 67, 47).
// A residual projection has a third or less of their tiles, and a workgroup of
// the tile kernel walks its whole k range, so it takes the kernel expected to be
// first, which at 190 of these widths and heights was never more than 1.6 us
// behind the best.  Prompt pass per layer in us with the output projection on
// tile / per-pair / tall split-k: width 1024 at 176 rows 84.3 / 78.8 / 86.0,
// 2048 at 320 145 / 138, at 752 190 / 202; 4096 at 208 255 / 253 / 247, at 350
// 291 / 303.  With the down projection on tile / split-k / tall split-k: 1536 (k
// 6144) at 176 122 / 97 / 100, at 900 194 / 203; 2048 (5504) at 320 145 / 127, at
// 752 190 / 208; 4096 (11008) at 276 259 / 240 / 226, at 350 291 / 298.
GemmRoute gemm_route(GemmArgs& a, int epi, bool pairs, int NT, int cus) {
  if (a.mblocks <= 10) return pairs ? GemmRoute::kPairs : GemmRoute::kSplit;
  if (epi != EPI_RESID) return GemmRoute::kTile;
  GemmRoute best = GemmRoute::kTile;
  float t = gemm_tile_time(a, cus);
  if (pairs) {
    const float tp = gemm_ks_time(a, NT, cus);
    if (tp < t) { t = tp; best = GemmRoute::kPairs; }
  }
  // (the per-pair kernel's k shares on split-k: in tall tiles of 8 slices only, as measured)
  for (int tall = pairs ? 1 : 0; tall < 2; ++tall) {
    if (tall && (!gemm_sk_tall_rows(a.M) || (pairs && a.splits != 8))) continue;
    const float ts = gemm_sk_narrow_time(a, tall, cus);
    if (ts < t) { t = ts; best = GemmRoute::kSplit; a.sk_tall = tall; }
  }
  return best;
}

}  // namespace gvc
