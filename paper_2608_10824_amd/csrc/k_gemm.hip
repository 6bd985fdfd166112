// Gathered-row GEMM for the projections and the FFN: C[m][n] = X[m][:] . W[n][:].
//
// Each projection of a (partial) prompt pass or of a single-token decode pass
// runs over the M recomputed token rows only (Alg. 1, partial forward pass).
// M is small next to the weight matrices (1 to a few hundred rows per episode),
// so the kernel is built around streaming the packed bf16 weights once:
//  * MFMA v_mfma_f32_16x16x32_bf16 with the weight block as the A operand
//    (16 output features) and 16 token rows as the B operand; every lane loads
//    16 contiguous bytes of both operands straight from their packed layouts;
//  * one workgroup owns a PAIR of 16-row weight blocks for all the tile's
//    token rows; the pair is chosen so that the epilogue's partner values
//    sit in the same lane and register: RoPE dims (i, i + d_h/2), SwiGLU
//    (gate j, up j);
//  * weight and token fragments are prefetched a chunk ahead in registers;
//  * the k range is split across the waves of one workgroup and summed in
//    LDS in a fixed order, so results are bitwise reproducible and no
//    workgroup ever waits on another.
#include "gvc_epilogue.h"

namespace gvc {

// One workgroup owns one pair of weight blocks (one block for the single
// maps) and a tile of KT x NT blocks of 16 token rows.  Its KT * KS waves are
// KT token groups (NT blocks each) times KS shares of the k range: the waves
// of one k share read the same weight fragments at the same time, so the
// weights leave HBM once per workgroup while each wave keeps only NT token
// blocks in registers.  The k shares are summed through LDS in a fixed order
// (deterministic, no cross-workgroup traffic).  Each wave streams its share
// in chunks of PF k-steps, double-buffered in registers with no branch
// between a chunk's loads and its MFMAs, so two chunks are in flight; the
// prefetch of the chunk after the last re-reads the last chunk instead of
// branching.  Token fragments come straight from the (L2-resident)
// activations.
// A launch of one token block (decode, the head rows) reads each weight once:
// marked non-temporal, the loads do not push the activations, keys and values
// out of L2 (three 7B episodes of 4 layers 4430 -> 4281 us per step, sixteen
// 5130 -> 4984).  With several token tiles the later ones find the weights
// in L2, where the hint costs more than it gives.
template <bool ONCE>
__device__ __forceinline__ bf16x8 weight_load(const bf16x8* p) {
  if constexpr (ONCE) return __builtin_bit_cast(bf16x8, __builtin_nontemporal_load((const u32x4b*)p));
  return *p;
}

template <int KS, int KT, int NT, int PF, int EPI, bool ONE>
__global__ __launch_bounds__(KS * KT * 64) void k_gemm_ks(const GemmArgs a) {
  constexpr int KW = KS * KT;
  __shared__ floatx4 red[KW][2][64];
  __shared__ float ssq_red[KW][16];
  __shared__ float rscale[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tg = wave / KS, ks = wave % KS;
  // XCD-aware order: workgroup ids go round-robin over the 8 XCDs, so the
  // token tiles of one work unit get ids 8 apart -- same XCD, dispatched
  // together -- and the later tiles find the unit's weights in that L2.
  const int grp = blockIdx.x / (8 * a.mtiles), r8 = blockIdx.x % (8 * a.mtiles);
  const int pair = grp * 8 + (r8 & 7), mt = r8 >> 3;
  if (pair >= a.n_pairs) return;
  // Folded RMSNorm (single token block): lane (row r = lane % 16, chunk
  // wave * 4 + lane / 16) loads up to SQ of the row's partial sums of squares
  // now and adds them after the main loop, so the loads overlap the stream.
  constexpr int SQ = 16;
  float sq[SQ];
  const bool fold = NT == 1 && KT == 1 && a.e.ssq_in != nullptr;
  if (fold) {
    const int r = min(lane & 15, a.M - 1);
    const int nch = KW * 4, ch = wave * 4 + (lane >> 4);
    const int per = (a.e.ssq_parts + nch - 1) / nch;
    const float* sp = a.e.ssq_in + (size_t)r * a.e.ssq_parts;
#pragma unroll
    for (int i = 0; i < SQ; ++i) {
      const int idx = ch * per + i;
      const float v = sp[min(idx, a.e.ssq_parts - 1)];
      sq[i] = (i < per && idx < a.e.ssq_parts) ? v : 0.f;
    }
  }
  int mat_a, blk_a, mat_b, blk_b; bool b_ok;
  map_pair(a, pair, mat_a, blk_a, mat_b, blk_b, b_ok);
  const bf16x8* wa = a.w[mat_a] + (size_t)blk_a * a.KB * 64 + lane;
  const bf16x8* wb = a.w[mat_b] + (size_t)blk_b * a.KB * 64 + lane;
  const int mb0 = (mt * KT + tg) * NT;   // first token block of this wave
  // Lanes of token rows >= M re-read the last valid row of their block:
  // those output columns are never stored, and the shared address keeps a
  // decode launch (M = 1) from fetching 15 padding rows per fragment.
  const bf16x8* xg[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int mb = min(mb0 + t, a.mblocks - 1);
    const int xl = (lane & 48) | min(lane & 15, a.M - 1 - mb * 16);
    xg[t] = a.x + (size_t)mb * a.KB * 64 + xl;
  }
  // this wave's contiguous share of the k range
  const int kb0 = min(a.KB, ks * a.kb_per_split);
  const int nsteps = min(a.KB, kb0 + a.kb_per_split) - kb0;
  const int nchunks = nsteps / PF;

  floatx4 acc_a[NT], acc_b[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) { acc_a[t] = floatx4{0, 0, 0, 0}; acc_b[t] = floatx4{0, 0, 0, 0}; }
  bf16x8 a0[PF], b0[PF], x0[PF][NT], a1[PF], b1[PF], x1[PF][NT];
  auto load = [&](bf16x8 (&A)[PF], bf16x8 (&Bv)[PF], bf16x8 (&X)[PF][NT], int c) {
    const size_t kb = (size_t)(kb0 + min(c, nchunks - 1) * PF) * 64;
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      const size_t o = kb + (size_t)p * 64;
      A[p] = weight_load<NT == 1>(wa + o);
      if constexpr (!ONE) Bv[p] = weight_load<NT == 1>(wb + o);
#pragma unroll
      for (int t = 0; t < NT; ++t) X[p][t] = xg[t][o];
    }
  };
  auto compute = [&](const bf16x8 (&A)[PF], const bf16x8 (&Bv)[PF], const bf16x8 (&X)[PF][NT]) {
#pragma unroll
    for (int p = 0; p < PF; ++p)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc_a[t] = mfma16(A[p], X[p][t], acc_a[t]);
        if constexpr (!ONE) acc_b[t] = mfma16(Bv[p], X[p][t], acc_b[t]);
      }
  };
  if (nchunks > 0) {
    load(a0, b0, x0, 0);
    int c = 0;
    for (; c + 1 < nchunks; c += 2) {
      load(a1, b1, x1, c + 1);
      compute(a0, b0, x0);
      load(a0, b0, x0, c + 2);
      compute(a1, b1, x1);
    }
    if (c < nchunks) compute(a0, b0, x0);
  }
  for (int s = nchunks * PF; s < nsteps; ++s) {   // ragged k tail
    const size_t kb = (size_t)(kb0 + s) * 64;
    const bf16x8 wva = wa[kb];
    const bf16x8 wvb = ONE ? wva : wb[kb];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bf16x8 xv = xg[t][kb];
      acc_a[t] = mfma16(wva, xv, acc_a[t]);
      if constexpr (!ONE) acc_b[t] = mfma16(wvb, xv, acc_b[t]);
    }
  }
  if (fold) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < SQ; ++i) t += sq[i];
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    if (lane < 16) ssq_red[wave][lane] = t;
    __syncthreads();
    if (wave == 0 && lane < 16) {
      float u = ssq_red[0][lane];
#pragma unroll
      for (int w = 1; w < KW; ++w) u += ssq_red[w][lane];
      rscale[lane] = 1.0f / sqrtf(u / (float)a.e.norm_dim + a.e.norm_eps);
    }
  }
  // Reduce over the KS k shares of each token group, one token block per
  // round; the wave with ks == t % KS keeps the sum of block t and runs its
  // epilogue.
  const int col = lane & 15;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    red[wave][0][lane] = acc_a[t];
    if constexpr (!ONE) red[wave][1][lane] = acc_b[t];
    __syncthreads();
    if (ks == t % KS) {
      floatx4 sa = red[tg * KS][0][lane], sb = ONE ? sa : red[tg * KS][1][lane];
#pragma unroll
      for (int w = 1; w < KS; ++w) {
        sa += red[tg * KS + w][0][lane];
        if constexpr (!ONE) sb += red[tg * KS + w][1][lane];
      }
      acc_a[t] = sa; acc_b[t] = sb;
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (ks != t % KS) continue;
    const int m = (mb0 + t) * 16 + col;
    const float rs = fold ? rscale[col] : 1.0f;
    epilogue<EPI>(a, pair, lane, min(m, a.M - 1), acc_a[t], acc_b[t], b_ok, m < a.M, rs);
  }
}

// Split-k variant for prompt-pass projections whose whole tiles would leave
// compute units idle: one workgroup per (group of NCW * PB consecutive weight
// blocks, of all the launch's matrices in order; k slice; tile of T token
// blocks).  NCW compute waves each stream their PB weight blocks through a
// private LDS ring of RW fragments (non-temporal direct-to-LDS loads, in k
// order), and NXW loader waves copy the tile's token fragments into DX LDS
// stages of KC k steps.  Partial sums go to part[slice][row][feature];
// k_gemm_sk_epi then adds the slices in order and runs the fused epilogue.
// The slices depend only on the matrix shape, so a row's result never depends
// on how many rows a pass recomputes.  Weight loads then never
// queue behind token loads in a wave's in-order memory counter, and a
// compute wave waits only for its own oldest weight fragment; one workgroup
// barrier per chunk hands the token stages over (the stage refilled after
// the barrier of chunk c last held chunk c - 1, which every compute wave
// finished before arriving).
template <int T, int NCW, int PB, int KC, int DX, int NXW, int RW>
__global__ __launch_bounds__((NCW + NXW) * 64) void k_gemm_dx(const GemmArgs a) {
  constexpr int NF = KC * T, ITOK = (NF + NXW - 1) / NXW;
  static_assert((DX - 2) * ITOK < 64 && RW < 64, "vmcnt range");
  extern __shared__ u32x4b dx_lds[];                 // [NCW][RW][64] rings, then [DX][NF][64] token stages
  u32x4b* const xst = dx_lds + NCW * RW * 64;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int id = blockIdx.x;
  const int g = id % a.sk_groups;
  id /= a.sk_groups;
  const int s = id % a.sk_slices, mt = id / a.sk_slices;
  const int kb0 = s * a.sk_steps, nk = min(a.KB, kb0 + a.sk_steps) - kb0;
  if (nk <= 0) return;
  const int nch = (nk + KC - 1) / KC;
  const int mb0 = mt * T, nT = min(T, a.mblocks - mb0);
  const int nblk = a.wblk[0] * (a.map == MAP_QKV ? 3 : (a.map == MAP_GU ? 2 : 1));
  if (wv >= NCW) {   // token loader
    const int x = wv - NCW;
    auto issue = [&](int c) {   // chunks past the end re-read the last k step (in bounds)
      u32x4b* st = xst + (c % DX) * NF * 64;
#pragma unroll
      for (int i = 0; i < ITOK; ++i) {
        const int f = min(x + i * NXW, NF - 1), kk = f / T, t = f % T;
        const int kb = kb0 + min(c * KC + kk, nk - 1);
        __builtin_amdgcn_global_load_lds(GPB(a.x + ((size_t)(mb0 + min(t, nT - 1)) * a.KB + kb) * 64 + lane),
                                         LPB(st + f * 64), 16, 0, 0);
      }
    };
#pragma unroll
    for (int c = 0; c < DX - 1; ++c) issue(c);
    for (int c = 0; c < nch; ++c) {
      wait_vmcnt<(DX - 2) * ITOK>();
      lds_barrier();
      issue(c + DX - 1);
    }
    wait_vmcnt<0>();
    return;
  }
  const bf16x8* wp[PB];
  int vbs[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    const int vb = (g * NCW + wv) * PB + p;
    vbs[p] = vb;
    const int vc = min(vb, nblk - 1), mat = vc / a.wblk[0], blk = vc % a.wblk[0];
    wp[p] = a.w[mat] + ((size_t)blk * a.KB + kb0) * 64 + lane;
  }
  u32x4b* const ring = dx_lds + wv * RW * 64;
  const int total = nk * PB;
  int next = 0;   // next fragment of this wave's stream (k major, block minor)
  auto refill = [&](int slot) {
    const int i = min(next, total - 1), k = i / PB, p = i - k * PB;
    const bf16x8* src = wp[0];
#pragma unroll
    for (int q = 1; q < PB; ++q)
      if (p == q) src = wp[q];
    __builtin_amdgcn_global_load_lds(GPB(src + (size_t)k * 64), LPB(ring + slot * 64), 16, 0, 2);
    ++next;
  };
#pragma unroll
  for (int r = 0; r < RW; ++r) refill(r);
  floatx4 acc[PB][T];
#pragma unroll
  for (int p = 0; p < PB; ++p)
#pragma unroll
    for (int t = 0; t < T; ++t) acc[p][t] = floatx4{0, 0, 0, 0};
  int slot = 0;
  for (int c = 0; c < nch; ++c) {
    lds_barrier();
    const u32x4b* st = xst + (c % DX) * NF * 64;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
      if (c * KC + kk >= nk) break;
      bf16x8 wf[PB];
#pragma unroll
      for (int p = 0; p < PB; ++p) {
        wait_vmcnt<RW - 1>();
        wf[p] = __builtin_bit_cast(bf16x8, ring[slot * 64 + lane]);
        __builtin_amdgcn_s_waitcnt(0xC07F);   // the read has left the slot before it is refilled
        refill(slot);
        slot = slot + 1 == RW ? 0 : slot + 1;
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const bf16x8 xf = __builtin_bit_cast(bf16x8, st[(kk * T + t) * 64 + lane]);
#pragma unroll
        for (int p = 0; p < PB; ++p) acc[p][t] = mfma16(wf[p], xf, acc[p][t]);
      }
    }
  }
  wait_vmcnt<0>();
  const int col = lane & 15, sub = (lane >> 4) * 4;
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    if (vbs[p] >= nblk) continue;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (t >= nT) continue;
      const int m = (mb0 + t) * 16 + col;
      if (m < a.M)   // rows past the last one are never summed
        *(floatx4*)(a.part + ((size_t)s * a.part_rows + m) * a.part_ld + vbs[p] * 16 + sub) = acc[p][t];
    }
  }
}

// Sums the k slices of k_gemm_dx in order and runs the epilogue: one wave
// per (work pair, block of 16 rows), in the lane layout of the MFMA result.
// The 4 waves of a workgroup take 4 consecutive pairs of one row block, so
// each row's partial sums are read as whole cache lines by one CU (C2
// gate/up: prompt pass 6.56 -> 6.48 ms against row-block-minor order).
template <int EPI>
__global__ __launch_bounds__(256) void k_gemm_sk_epi(const GemmArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= a.n_pairs * a.mblocks) return;
  const int pair = w % a.n_pairs, mb = w / a.n_pairs;
  int ma, ba, mb2, bb; bool b_ok;
  map_pair(a, pair, ma, ba, mb2, bb, b_ok);
  const int m = mb * 16 + (lane & 15), sub = (lane >> 4) * 4;
  const int fa = (ma * a.wblk[0] + ba) * 16 + sub, fb = (mb2 * a.wblk[0] + bb) * 16 + sub;
  floatx4 va = {0, 0, 0, 0}, vb = {0, 0, 0, 0};
  if (m < a.M)   // the cores store no partial sums for rows past the last one
    for (int s = 0; s < a.sk_slices; ++s) {
      const float* row = a.part + ((size_t)s * a.part_rows + m) * a.part_ld;
      va += *(const floatx4*)(row + fa);
      if (b_ok) vb += *(const floatx4*)(row + fb);
    }
  epilogue<EPI>(a, pair, lane, min(m, a.M - 1), va, vb, b_ok, m < a.M, 1.0f);
}

template <int EPI>
static hipError_t launch_sk_epi(const GemmArgs& a, hipStream_t s) {
  const int waves = a.n_pairs * a.mblocks;
  hipLaunchKernelGGL(k_gemm_sk_epi<EPI>, dim3((waves + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

// One weight block per compute wave, so that a launch of whole k slices
// fills the 256 compute units with one workgroup each at the 7B shape: wide
// (QKV, gate/up) 12 blocks, QKV 64 groups x 4 slices and gate/up 115 x 2;
// narrow (down) 32 groups of 8 blocks x 8 slices.  Chunks of 2 k steps in 4
// token stages of 10 token blocks, 2 loader waves, weight rings of 6 (wide,
// 152 KiB of LDS) and 8 fragments.
constexpr int kSkT = 10, kDxKC = 2, kDxD = 4, kDxNXW = 2;
constexpr int kDxWideW = 12, kDxWideR = 6, kDxNarrowW = 8, kDxNarrowR = 8;
// Tall tiles: a narrow launch of 11-18 token blocks (161-288 rows) as one tile
// of 18 blocks per k slice (2 token stages, 136 KiB), so each slice's weights
// leave HBM once instead of once per 160-row tile.  A slice's partial sums are
// the same MFMA sequence in either tiling, so they are bit-identical.
constexpr int kSkTallT = 18, kDxTallNarrowD = 2;

template <int T, int NCW, int PB, int KC, int DX, int NXW, int RW>
static hipError_t launch_dx_core(const GemmArgs& a, hipStream_t s) {
  constexpr int lds = (NCW * RW + DX * KC * T) * 1024;
  static_assert(lds <= 160 * 1024, "LDS");
  static bool attr = false;
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dx<T, NCW, PB, KC, DX, NXW, RW>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const int mtiles = (a.mblocks + T - 1) / T;
  hipLaunchKernelGGL((k_gemm_dx<T, NCW, PB, KC, DX, NXW, RW>), dim3(a.sk_groups * a.sk_slices * mtiles),
                     dim3((NCW + NXW) * 64), lds, s, a);
  return hipGetLastError();
}

bool gemm_sk_tall_rows(int M) {
  const int mblocks = (M + 15) / 16;
  return mblocks > kSkT && mblocks <= kSkTallT;
}

// Fitted to prompt passes of widths 512-5120 at 161-900 rows that differ in the
// kernel of one residual projection (see gemm_route): a ramp per round of
// workgroups, the weights and MFMAs of all workgroups spread over the CUs (tall
// tiles: of whole rounds), and the partial sums' way through memory.
float gemm_sk_narrow_time(const GemmArgs& a, bool tall, int cus) {
  const float mb = 4e-6f * a.M * a.wblk[0] * 16 * a.sk_slices;   // megabytes of partial sums
  const int n = a.sk_groups * a.sk_slices * (tall ? 1 : (a.mblocks + kSkT - 1) / kSkT);
  const int rounds = (n + cus - 1) / cus;
  if (tall) return 14.5f + 0.58f * rounds * a.sk_steps + 0.31f * mb;
  return 10.3f + 6.4f * rounds + 0.457f * n * a.sk_steps / cus + 0.16f * mb;
}

int gemm_sk_group_blocks(int sk_shape) { return sk_shape == SK_WIDE ? kDxWideW : kDxNarrowW; }

hipError_t launch_gemm_sk(const GemmArgs& a, int epi, hipStream_t s) {
  if (a.map == MAP_SINGLE || a.map == MAP_QKV_SINGLE || a.e.ssq_in || !a.part) return hipErrorInvalidValue;
  if (a.sk_tall && (a.sk_shape != SK_NARROW || !gemm_sk_tall_rows(a.M))) return hipErrorInvalidValue;
  hipError_t e;
  if (a.sk_shape == SK_WIDE)
    e = launch_dx_core<kSkT, kDxWideW, 1, kDxKC, kDxD, kDxNXW, kDxWideR>(a, s);
  else if (a.sk_tall)
    e = launch_dx_core<kSkTallT, kDxNarrowW, 1, kDxKC, kDxTallNarrowD, kDxNXW, kDxNarrowR>(a, s);
  else
    e = launch_dx_core<kSkT, kDxNarrowW, 1, kDxKC, kDxD, kDxNXW, kDxNarrowR>(a, s);
  if (e != hipSuccess) return e;
  switch (epi) {
    case EPI_QKV: return launch_sk_epi<EPI_QKV>(a, s);
    case EPI_RESID: return launch_sk_epi<EPI_RESID>(a, s);
    case EPI_SILU: return launch_sk_epi<EPI_SILU>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int EPI, int KT, int NT, bool ONE>
static hipError_t launch_one(const GemmArgs& a, hipStream_t s) {
  constexpr int PF = gemm_pf(NT);
  const dim3 grid((a.n_pairs + 7) / 8 * 8 * a.mtiles);
  const int ks = a.splits / KT;
  if constexpr (KT == 1) {
    if (ks == 8) {
      hipLaunchKernelGGL((k_gemm_ks<8, 1, NT, PF, EPI, ONE>), grid, dim3(8 * 64), 0, s, a);
      return hipGetLastError();
    }
    if (ks == 4) {
      hipLaunchKernelGGL((k_gemm_ks<4, 1, NT, PF, EPI, ONE>), grid, dim3(4 * 64), 0, s, a);
      return hipGetLastError();
    }
  } else {
    if (ks == 4) {
      hipLaunchKernelGGL((k_gemm_ks<4, KT, NT, PF, EPI, ONE>), grid, dim3(4 * KT * 64), 0, s, a);
      return hipGetLastError();
    }
    if (ks == 2) {
      hipLaunchKernelGGL((k_gemm_ks<2, KT, NT, PF, EPI, ONE>), grid, dim3(2 * KT * 64), 0, s, a);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

template <int EPI, int NT>
static hipError_t launch_nt(const GemmArgs& a, hipStream_t s) {
  const bool one = a.map == MAP_SINGLE || a.map == MAP_QKV_SINGLE;
  if constexpr (EPI == EPI_RESID || EPI == EPI_STORE || EPI == EPI_QKV_RAW) {
    if (one) return (NT == 1 && a.tgroups == 1) ? launch_one<EPI, 1, 1, true>(a, s) : hipErrorInvalidValue;
  }
  if (one) return hipErrorInvalidValue;
  if constexpr (EPI == EPI_QKV_RAW) {
    return hipErrorInvalidValue;
  } else {
    if (a.tgroups == 1) return launch_one<EPI, 1, NT, false>(a, s);
    return hipErrorInvalidValue;
  }
}

template <int EPI>
static hipError_t launch_epi(const GemmArgs& a, int NT, hipStream_t s) {
  switch (NT) {
    case 1: return launch_nt<EPI, 1>(a, s);
    case 2: return launch_nt<EPI, 2>(a, s);
    case 3: return launch_nt<EPI, 3>(a, s);
    case 4: return launch_nt<EPI, 4>(a, s);
    case 5: return launch_nt<EPI, 5>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// Fitted as gemm_sk_narrow_time: one workgroup of 8 waves to a CU, two of 4.
float gemm_ks_time(const GemmArgs& a, int NT, int cus) {
  const int n = a.n_pairs * a.mtiles;
  if (a.splits != 8) return 7.7f + 0.2f * a.KB * ((n + 2 * cus - 1) / (2 * cus));
  return 7.5f + (1.3f + (NT > 4 ? 0.108f : 0.076f) * a.KB) * ((n + cus - 1) / cus);
}

hipError_t launch_gemm(const GemmArgs& a, int epi, int NT, hipStream_t s) {
  switch (epi) {
    case EPI_QKV: return launch_epi<EPI_QKV>(a, NT, s);
    case EPI_RESID: return launch_epi<EPI_RESID>(a, NT, s);
    case EPI_SILU: return launch_epi<EPI_SILU>(a, NT, s);
    case EPI_STORE: return launch_epi<EPI_STORE>(a, NT, s);
    case EPI_EMBED: return launch_epi<EPI_EMBED>(a, NT, s);
    case EPI_QKV_RAW: return launch_epi<EPI_QKV_RAW>(a, NT, s);
    case EPI_PATCH: return launch_epi<EPI_PATCH>(a, NT, s);
    case EPI_GELU: return launch_epi<EPI_GELU>(a, NT, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gvc
