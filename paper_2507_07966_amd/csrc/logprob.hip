// Response-token log-probabilities: logp_n = z_{y_n} - ln sum_v exp(z_v), z = logit_scale * W h_n,
// without ever materialising the [tokens, vocabulary] logits.
//
// The GRPO objective (paper Eq. 1) needs the probabilities the policy, the old policy and the
// reference model give to the sampled response tokens; after the prefill each device computes the
// logits of its token slice (Sec. 5.2).  With a 7B-class model that is a [N, 3584] x [3584, 152064]
// product per model, 1.8e13 FLOP for 16K response tokens, and the logits (10 GB in fp32) are only
// ever reduced to two numbers per token.
//
// Kernel 1 (bf16 MFMA GEMM with a reducing epilogue), bound by MFMA power for many tokens and by reading W for
// few. A workgroup (8 wavefronts) computes one 256-vocabulary x 32 NB-token tile of Z^T = W H^T (NB = 8, 6, 4,
// 2; launch_logprob chooses): wavefront (wv, wt) owns 64 vocabulary rows x 16 NB tokens (4 x NB accumulator
// blocks of v_mfma_f32_16x16x32_bf16, 128 registers for NB = 8; that shape moves half the accumulator data per
// FLOP of the 32 x 32 x 16 one and sustains about 10 % more under the board's power limit).  W and H panels of
// 64 channels go global -> LDS through range-checked buffer loads (rows past the end of either matrix read as
// zero), double buffered, one barrier per 64 channels (a third buffer gained nothing at 64 and 128 tokens);
// for NB = 8, 12 LDS operand reads feed 32 MFMAs.  In the epilogue every lane holds 16 logits of each of NB
// tokens: it reduces them to a maximum and a sum of exponentials, combines with the three lanes holding the
// token's other rows and, through LDS, with the other three row blocks, so the tile writes one (m, l) pair per
// token; the lane that holds the target's logit writes it out.  Every XCD gets an equal, contiguous share of
// the tiles, walked in bands of four vocabulary tiles, so the 32 tiles running together on one XCD form an
// 8-token-tile x 4-vocabulary-tile block: 12 distinct panels per step share that XCD's L2 instead of 64.
// (Dealing whole token tiles to the XCDs instead left most of the chip idle when their number was not a
// multiple of 8: 2,100 tokens x 152,064 words 6.04 ms, now 1.95; 8,200 tokens 12.97, now 7.20; at 16,384 tokens,
// where it was balanced, the two are within 1 %, 13.97 and 13.83.)
// Kernel 2 combines the (m, l) pairs of a token over all vocabulary blocks: LSE = m + ln l,
// logp = z_target - LSE.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <utility>

#include "common.h"
#include "logprob.h"
#include "mfma_tiles.h"

namespace pa {
namespace {

using namespace mt;

constexpr int LP_WAVES = 8, LP_THREADS = LP_WAVES * 64;
constexpr int BK = 64;                      // channels per stage
constexpr int BAND = 4;                     // vocabulary tiles that are walked together
constexpr int PANEL_BYTES = LP_TILE * BK * 2;  // the 256-row x 64-channel panel of W
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// v_mfma_f32_16x16x32_bf16 (l16 = lane % 16, g4 = lane / 16): A: lane holds row l16, contraction indices
// 8*g4 .. 8*g4+7; B: column l16, the same indices; C: register i holds row 4*g4 + i, column l16.
// The four lanes l16, l16 + 16, l16 + 32, l16 + 48 hold the 16 rows of a column: maximum / sum over them.
__device__ inline void pair_values(float x, float& a, float& b) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const unsigned r0 = r[0], r1 = r[1];   // read through named temporaries, see attn_bf16.hip
  a = __uint_as_float(r0);
  b = __uint_as_float(r1);
}
__device__ inline float column_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  float u, w;
  pair_values(x, u, w);
  return fmaxf(u, w);
}
__device__ inline float column_sum(float x) {
  x += __shfl_xor(x, 16);
  float u, w;
  pair_values(x, u, w);
  return u + w;
}

template <int NB>
__global__ __launch_bounds__(LP_THREADS, NB == 2 ? 4 : 2) void logprob_tile_kernel(
    const __bf16* __restrict__ hidden, const __bf16* __restrict__ lm_head, const int32_t* __restrict__ targets,
    float2* __restrict__ partials, float* __restrict__ target_logit, int64_t N, int d, int V, int TM, int TV,
    float logit_scale) {
  constexpr int TT = 32 * NB;                           // tokens per tile
  constexpr int LP_STAGE = PANEL_BYTES + TT * BK * 2;   // W panel, H panel
  constexpr int HB = NB / 2;                            // 1 KiB blocks of the H panel per wavefront
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * LP_STAGE];

  // ---- which tile: XCD x = blockIdx % 8 computes a contiguous eighth of the tiles, numbered band by band (a band:
  //      four vocabulary tiles x all token tiles, vocabulary fastest; the last band may be narrower)
  int tm, tv;
  {
    const int per_xcd = gridDim.x >> 3;
    const int idx = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (idx >= TM * TV) return;
    const int whole = TV / BAND * BAND * TM;  // tiles in bands of full width
    const int width = idx < whole ? BAND : TV % BAND;
    const int r = idx < whole ? idx % (BAND * TM) : idx - whole;
    tm = r / width;
    tv = (idx < whole ? idx / (BAND * TM) * BAND : TV / BAND * BAND) + r % width;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int wv = wave & 3, wt = wave >> 2;
  const int64_t v0 = (int64_t)tv * LP_TILE, t0 = (int64_t)tm * TT;

  // ---- loads: the W panel is 256 rows x 128 bytes = 32 blocks of 1 KiB (8 rows each), 4 per wavefront, the H
  //      panel TT / 8 blocks, NB / 2 per wavefront
  const int64_t rowb = (int64_t)d * 2;
  const int64_t w_rows = V - v0 < LP_TILE ? V - v0 : LP_TILE, h_rows = N - t0 < TT ? N - t0 : TT;
  const rsrc_t r_w = make_rsrc(lm_head + v0 * d, w_rows * rowb);
  const rsrc_t r_h = make_rsrc(hidden + t0 * d, h_rows * rowb);
  unsigned loff[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    const int row = (wave * 4 + n) * 8 + lane / 8;
    const int chunk = (lane % 8) ^ swizzle_term(row, 128);  // logical chunk stored at this position
    loff[n] = (unsigned)(row * rowb + chunk * 16);
  }
  unsigned hoff[HB];
#pragma unroll
  for (int n = 0; n < HB; ++n) {
    const int row = (wave * HB + n) * 8 + lane / 8;
    const int chunk = (lane % 8) ^ swizzle_term(row, 128);
    hoff[n] = (unsigned)(row * rowb + chunk * 16);
  }
  auto issue = [&](int stage, int buf) {
    unsigned char* dst = smem + buf * LP_STAGE;
    const unsigned k_off = (unsigned)stage * (BK * 2);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      load_chunk_to_lds(r_w, dst + (wave * 4 + n) * 1024, loff[n], k_off);
      if (n < HB) load_chunk_to_lds(r_h, dst + PANEL_BYTES + (wave * HB + n) * 1024, hoff[n < HB ? n : 0], k_off);
    }
  };

  constexpr int NA = 4;   // 16-row blocks of the wavefront's 64 vocabulary rows; NB: of its 16 NB tokens
  f32x4 C[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) C[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Per-lane LDS addresses of the operand reads, one set per buffer (the second buffer lies 40 to 64 KiB on: with
  // the panels' own offsets beyond the reach of a read's 16-bit immediate), so the main loop itself holds no address
  // arithmetic.
  // (Row blocks of 16 share the swizzle of rows 0..15.)
  const unsigned char* wop[2][BK / 32];
  const unsigned char* hop[2][BK / 32];
#pragma unroll
  for (int bufi = 0; bufi < 2; ++bufi)
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      const int off = l16 * 128 + (((4 * ks + g4) ^ swizzle_term(l16, 128)) << 4);
      wop[bufi][ks] = smem + bufi * LP_STAGE + (wv * 64) * 128 + off;
      hop[bufi][ks] = smem + bufi * LP_STAGE + PANEL_BYTES + (wt * 16 * NB) * 128 + off;
    }

  const int nstages = (d + BK - 1) / BK;  // channels past d read as zero (range-checked loads)
  auto stage = [&](int s, auto buf_c) {
    constexpr int BUF = decltype(buf_c)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's share of stage s has landed
    __syncthreads();                      // everyone's share has; the other buffer is no longer read
    if (s + 1 < nstages) issue(s + 1, BUF ^ 1);
    // The MFMA part of a stage runs at wave priority 1, the wait, the barrier and the issue of the next stage's
    // loads at priority 0: of the two wavefronts sharing a SIMD, the one already in its MFMAs is served before
    // the one still issuing loads (+1.5 %; priority for the loads instead: -0.4 %).
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      bf16x8 wa[NA], hb[NB];
#pragma unroll
      for (int a = 0; a < NA; ++a) wa[a] = lds_operand(wop[BUF][ks] + a * 16 * 128);
#pragma unroll
      for (int b = 0; b < NB; ++b) hb[b] = lds_operand(hop[BUF][ks] + b * 16 * 128);
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int a = 0; a < NA; ++a) C[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[a], hb[b], C[a][b], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  issue(0, 0);
  {
    int s = 0;
    for (; s + 1 < nstages; s += 2) {
      stage(s, std::integral_constant<int, 0>{});
      stage(s + 1, std::integral_constant<int, 1>{});
    }
    if (s < nstages) stage(s, std::integral_constant<int, 0>{});
  }

  // ---- epilogue.  Register i of C[a][b]: vocabulary row v0 + wv*64 + a*16 + 4*g4 + i,
  //      token t0 + wt*16*NB + b*16 + l16.
  const float c2 = logit_scale * LOG2E;  // work in base 2
  __syncthreads();                        // every wavefront is done with the panels: reuse the LDS
  float2* stage_ml = reinterpret_cast<float2*>(smem);  // [4 row blocks][TT tokens] (m in base-2 units, l)
  const int64_t vlane = v0 + wv * 64 + 4 * g4;         // this lane's first vocabulary row
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int64_t tok = t0 + wt * 16 * NB + b * 16 + l16;
    float m = -INFINITY;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (vlane + a * 16 + i < V) m = fmaxf(m, C[a][b][i]);
    m = column_max(m) * c2;  // -inf only when none of the block's 64 rows exists
    float l = 0.f;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (vlane + a * 16 + i < V) l += __builtin_amdgcn_exp2f(__builtin_fmaf(C[a][b][i], c2, -m));
    l = column_sum(l);
    if (g4 == 0) stage_ml[wv * TT + wt * 16 * NB + b * 16 + l16] = float2{m, l};  // m = -inf, l = 0 for a block past V
    if (tok < N) {
      // the target's logit, if it lies in this wavefront's 64 rows and this lane's four of every 16
      const int64_t rel = (int64_t)targets[tok] - (v0 + wv * 64);
      if (rel >= 0 && rel < 64) {
        const int r = (int)rel & 15, a_t = (int)rel >> 4;
        if ((r >> 2) == g4) {
          const int i_t = r & 3;
          float z = 0.f;
#pragma unroll
          for (int a = 0; a < NA; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (a == a_t && i == i_t) z = C[a][b][i];
          target_logit[tok] = z * logit_scale;
        }
      }
    }
  }
  // one (m, l) pair per token for the tile's 256 vocabulary rows (block 0 always exists)
  __syncthreads();
  if (tid < TT && t0 + tid < N) {
    float m = stage_ml[tid].x;
#pragma unroll
    for (int k = 1; k < 4; ++k) m = fmaxf(m, stage_ml[k * TT + tid].x);
    float l = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2 v = stage_ml[k * TT + tid];
      l += v.y * __builtin_amdgcn_exp2f(v.x - m);
    }
    partials[(int64_t)tv * N + t0 + tid] = float2{m * LN2, l};
  }
}

// (m, l) pairs of a token over all vocabulary tiles -> LSE and log-probability.  A block handles 16 tokens (one
// 128-byte line of each row of pairs); each of its 16 thread groups takes every 16th row, eight loads in flight and
// one rescaling per eight, and the groups are merged through LDS.  (64 tokens per block and one load at a time took
// 69 us for 333 tokens x 594 rows on 6 CUs; now 9 us.)
constexpr int FIN_TOKENS = 16, FIN_GROUPS = 16, FIN_DEPTH = 8;
__global__ __launch_bounds__(FIN_TOKENS * FIN_GROUPS) void logprob_finalize_kernel(
    const float2* __restrict__ partials, const float* __restrict__ target_logit, const int32_t* __restrict__ targets,
    float* __restrict__ logprob, float* __restrict__ lse_out, int64_t N, int nparts, int V) {
  __shared__ float2 sm[FIN_GROUPS][FIN_TOKENS];
  const int tl = threadIdx.x % FIN_TOKENS, grp = threadIdx.x / FIN_TOKENS;
  const int64_t tok = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * FIN_TOKENS + tl;
  float m = -INFINITY, l = 0.f;
  if (tok < N)
    for (int p0 = grp; p0 < nparts; p0 += FIN_GROUPS * FIN_DEPTH) {
      float2 v[FIN_DEPTH];
#pragma unroll
      for (int i = 0; i < FIN_DEPTH; ++i) {
        const int p = p0 + i * FIN_GROUPS;
        v[i] = p < nparts ? partials[(int64_t)p * N + tok] : float2{-INFINITY, 0.f};
      }
      float mn = fmaxf(m, v[0].x);  // row p0 exists: finite
#pragma unroll
      for (int i = 1; i < FIN_DEPTH; ++i) mn = fmaxf(mn, v[i].x);
      l *= expf(m - mn);            // first time: 0 * exp(-inf) = 0
#pragma unroll
      for (int i = 0; i < FIN_DEPTH; ++i) l += v[i].y * expf(v[i].x - mn);
      m = mn;
    }
  sm[grp][tl] = float2{m, l};
  __syncthreads();
  if (grp == 0 && tok < N) {
    float mm = m;
#pragma unroll
    for (int k = 1; k < FIN_GROUPS; ++k) mm = fmaxf(mm, sm[k][tl].x);
    float ll = 0.f;
#pragma unroll
    for (int k = 0; k < FIN_GROUPS; ++k) {
      const float2 v = sm[k][tl];
      ll += v.y > 0.f ? v.y * expf(v.x - mm) : 0.f;  // a group that saw no tile holds (-inf, 0)
    }
    const float lse = mm + logf(ll);
    // no tile holds the logit of an id outside [0, V) (an ignore index, say): its slot was never written
    const int32_t y = targets[tok];
    logprob[tok] = (y >= 0 && y < V) ? target_logit[tok] - lse : __builtin_nanf("");
    if (lse_out) lse_out[tok] = lse;
  }
}

// Eq. 2: A_i = (r_i - mean) / std over one group of G rewards (population std; equal rewards -> 0).
__global__ __launch_bounds__(64) void group_advantages_kernel(const float* __restrict__ rewards,
                                                              float* __restrict__ adv, int G, int num_groups) {
  const int g = blockIdx.x * 64 + threadIdx.x;
  if (g >= num_groups) return;
  const float* r = rewards + (int64_t)g * G;
  float mean = 0.f;
  for (int i = 0; i < G; ++i) mean += r[i];
  mean /= (float)G;
  float var = 0.f;
  for (int i = 0; i < G; ++i) var += (r[i] - mean) * (r[i] - mean);
  const float sd = sqrtf(var / (float)G);
  for (int i = 0; i < G; ++i) adv[(int64_t)g * G + i] = sd > 0.f ? (r[i] - mean) / sd : 0.f;
}

}  // namespace

namespace {

// Compute units of the current device, asked once per device (a partitioned GPU has fewer than 256).
int compute_units() {
  static std::atomic<int> known[64];
  int device = 0, cus = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= 64) return NUM_CU;
  cus = known[device].load(std::memory_order_relaxed);
  if (cus > 0) return cus;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) {
    (void)hipGetLastError();
    return NUM_CU;
  }
  known[device].store(cus, std::memory_order_relaxed);
  return cus;
}

int64_t tile_rounds(int nb, int64_t N, int TV, int64_t cus) { return ((N + 32 * nb - 1) / (32 * nb) * TV + cus - 1) / cus; }

template <int NB>
int launch_tiles(const LogprobArgs& a, int TV, hipStream_t s) {
  const int TM = (int)((a.N + 32 * NB - 1) / (32 * NB));
  const int64_t grid = ((int64_t)TM * TV + 7) / 8 * 8;
  logprob_tile_kernel<NB><<<(unsigned)grid, LP_THREADS, 0, s>>>(
      static_cast<const __bf16*>(a.hidden), static_cast<const __bf16*>(a.lm_head), a.targets,
      reinterpret_cast<float2*>(a.partials), a.target_logit, a.N, a.d, a.V, TM, TV, a.logit_scale);
  return (int)hipGetLastError();
}

}  // namespace

int launch_logprob(const LogprobArgs& a, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int TV = (a.V + LP_TILE - 1) / LP_TILE;
  // Tokens per tile, 64 ... 256: the launch runs in rounds of one tile per CU (two for 64 tokens), so the tile with
  // the least rounds x time per round is taken.  Time of a round relative to 256 tokens, measured on launches of
  // whole rounds (d = 3584): 192 tokens 0.78, 128 tokens 0.62 (smaller tiles read more LDS operands per MFMA).
  // Against 256-token tiles, V = 152,064: 333 tokens 489 -> 447 us, 128 tokens 297 -> 276; V = 50,000, d = 1536:
  // 640 tokens 121 -> 101, 4100 tokens 568 -> 544.  A smaller tile has to promise 2 %.  Up to 64 tokens the call is
  // bound by reading W: two 64-token workgroups per CU keep more loads in flight (314 -> 229 us, 4.8 TB/s).
  const int cus = compute_units();
  int nb = 8;
  double best = 0.98 * tile_rounds(8, a.N, TV, cus);
  for (const auto& [smaller, t] : {std::pair{6, 0.78}, {4, 0.62}})
    if (const double cost = tile_rounds(smaller, a.N, TV, cus) * t; cost < best) {
      best = cost;
      nb = smaller;
    }
  if (a.N <= 64) nb = 2;
  const int st = nb == 8 ? launch_tiles<8>(a, TV, s)
               : nb == 6 ? launch_tiles<6>(a, TV, s)
               : nb == 4 ? launch_tiles<4>(a, TV, s) : launch_tiles<2>(a, TV, s);
  if (st != 0) return 1;
  const int64_t blocks = (a.N + FIN_TOKENS - 1) / FIN_TOKENS;
  const dim3 grid((unsigned)std::min(blocks, MAX_GRID_X), (unsigned)((blocks + MAX_GRID_X - 1) / MAX_GRID_X));
  logprob_finalize_kernel<<<grid, FIN_TOKENS * FIN_GROUPS, 0, s>>>(
      reinterpret_cast<const float2*>(a.partials), a.target_logit, a.targets, a.logprob, a.lse, a.N, TV, a.V);
  return (int)hipGetLastError();
}

int launch_group_advantages(const float* rewards, float* adv, int G, int num_groups, void* stream) {
  if (num_groups == 0) return 0;
  group_advantages_kernel<<<(unsigned)((num_groups + 63) / 64), 64, 0, static_cast<hipStream_t>(stream)>>>(
      rewards, adv, G, num_groups);
  return (int)hipGetLastError();
}

}  // namespace pa
