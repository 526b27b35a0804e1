// dfssm_mid.hip -- scaffold + LoRA linear from a few tokens to about a thousand
// on the gfx950 int8 matrix cores (v_mfma_i32_16x16x64_i8), one launch.
//
// At these sizes neither the arithmetic (1 us at 128 tokens of the 1.3B in_proj)
// nor the bytes (4 MB) take long; a call is the latency of its loads, of one
// reduction and of the LoRA exchange.  So:
//  * A workgroup owns a tile of 16*TT tokens x 16*RT output rows and splits K
//    over its KW waves: every byte of the tile's codes and signs is read by
//    one wave, through LDS (below), and all waves load at once.  The waves'
//    partial tiles meet in LDS after one barrier, and each wave finishes its
//    share of them.
//  * The sign bits are expanded to {0,1} bytes in registers, so the MFMA
//    gives D = sum_{bit=1} Q and acc_s = 2*D - sum_k Q.
//  * The LoRA down-projection acc_a = Q A^T and sum_k Q come from workgroups at
//    the front of the same grid (16*TT tokens x 16 ranks each, the same
//    staging), which publish them as 64-bit words {tag, 4 limb bytes} and
//    {tag, sum} with agent-scope stores; tags as in the few-token kernel.  The
//    words of a (token tile, 64-rank chunk) are laid out [16][64 lanes] as
//    their readers' lanes want them: a poll is 17 loads of 512 contiguous
//    bytes (the few-token kernel's lane-by-lane polls touch 64 lines each).
//    A wave whose words have not arrived after `spin` polls computes the same
//    integers itself, so no workgroup depends on another being scheduled.
//  * Up-projection and epilogue as in the few-token kernel: four limb MFMAs
//    per tile, exact int64 acc_b, the pinned fp32 order.
// Measured (us per call in a graph of calls, each on weights of its own, r = 64,
// before -> now; before: the few-token kernel in 64-token blocks or the former
// prefill path, whichever was faster): 1.3B in_proj at 9 / 48 / 128 / 301 tokens 9.4
// / 20.9 / 24.4 / 28.0 -> 7.1 / 8.4 / 11.8 / 19.5, out_proj at 9 / 64 / 301 / 1000 8.0
// / 14.5 / 33.2 / 40.6 -> 6.7 / 7.8 / 11.2 / 21.9, 130M out_proj at 1000 18.4 -> 9.3.
#include <algorithm>
#include <cmath>
#include <limits>

#include "dfssm_int4.hpp"
#include "dfssm_linear.hpp"

namespace {

using namespace dfssm_lin;

struct MidArgs {
  const int8_t* q;
  const float* s;
  int M, K, N, r, rp;
  const uint32_t* w_bits;
  const float* alpha;
  const int8_t* A;
  const int8_t* B;
  const float* beta;
  float* y;
  int32_t* acc_s_out;
  int32_t* acc_a_out;
  int64_t* acc_b_out;
  uint64_t* xw;     // limb words [group of token tiles][rank chunk of 64][16][64 lanes], then sum-Q words [token]
  uint64_t* epoch;  // device epoch words, or NULL: the call's tag is host_tag
  uint32_t host_tag;
  int arrivals;     // workgroups per call
  int tsh;          // 2^tsh token tiles per group: up to rank 16 (32) a tile has words for 16 (32) of the 64 lanes
  int nb_lora;      // LoRA workgroups at the front of the grid
  int nrt;          // 16-rank tiles they cover
  int ntb, nrb;     // token blocks, row blocks
  int spin;         // polls of a missing word before computing it locally
};

// The 16 words of a lane lie 512 bytes apart at every rank: 128 apart, calls of
// few tokens took 0.2 us longer.
__device__ __forceinline__ uint64_t* limb_words(const MidArgs& a, int tile, int chunk) {
  const int g = tile >> a.tsh, sub = tile - (g << a.tsh);
  return a.xw + ((int64_t)g * (a.rp >> 6) + chunk) * 1024 + (sub << (6 - a.tsh));
}
__device__ __forceinline__ uint64_t* sumq_words(const MidArgs& a) {
  const int tiles = (a.M + 15) >> 4;
  return a.xw + (a.r > 0 ? (int64_t)((tiles + (1 << a.tsh) - 1) >> a.tsh) * 16 * a.rp : 0);
}

// ---- direct-to-LDS staging.  An MFMA operand has one row per lane, so a load
// straight into operand registers touches 64 cache lines with every
// instruction, and a CU draws 16 bytes per clock from its L2 that way.  So each
// wave brings its own share of K through LDS in steps of 128 columns: lane i of a
// 16-byte load fetches piece i % 8 of row i / 8, whole 128-byte lines (60 bytes
// per clock per CU measured, against 36 with 64-byte pieces of rows).  The areas are private to the wave: no barrier, only the wave's own
// load counter.
// LDS of one wave: a ring of D steps of 16*TT token rows x 128 bytes, then two
// sign buffers of 16*RT rows x 32 bytes (2 steps).  The partial tiles overlay
// the ring once the wave is through with its K columns.
template <int TT, int RT, int D>
struct WaveLds {
  static constexpr int kStep = TT * 2048;
  static constexpr int kSign = D * kStep > TT * RT * 1024 ? D * kStep : TT * RT * 1024;
  static constexpr int kSignBuf = RT * 512;
  static constexpr int kBytes = kSign + (2 * kSignBuf > 2048 * D ? 2 * kSignBuf : 2048 * D);  // LoRA: A's ring
};

// LoRA workgroup: 16*TT tokens x 16 ranks, K split over the waves; the first
// rank tile's also sums Q.
template <int TT, int RT, int KW, int D, bool L4>
__device__ __forceinline__ void mid_lora(const MidArgs& a, int8_t* lds, uint32_t lds0, uint32_t* tag_lds) {
  using L = WaveLds<TT, RT, D>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rho = lane & 15, kg = lane >> 4;
  const int M = a.M, K = a.K, r = a.r;
  const int b = blockIdx.x;
  const int tb = b / a.nrt, jt = b - tb * a.nrt;
  uint64_t ep_old = 0;
  if (a.epoch && threadIdx.x == 0) ep_old = dfssm_dev::arrive(a.epoch, b);
  const int m0 = 16 * TT * tb;
  const int ng = (K + 127) >> 7;
  const int s0 = wave * ng / KW, n = (wave + 1) * ng / KW - s0;
  const int vlast = ((K - 1) & 127) / 16;  // last piece of a row's last step
  int8_t* const wl = lds + wave * L::kBytes;
  const uint32_t wl0 = lds0 + (uint32_t)(wave * L::kBytes);
  const int8_t* qb = a.q + (int64_t)m0 * K + 128 * s0;
  const int lrow = lane >> 3, lc = (lane & 7) ^ lrow;  // row of a load's 8, piece fetched
  uint32_t qoff[2 * TT];
#pragma unroll
  for (int i = 0; i < 2 * TT; ++i) qoff[i] = (uint32_t)(min(m0 + 8 * i + lrow, M - 1) - m0) * (uint32_t)K;
  const int apitch = L4 ? K / 2 : K;
  const int8_t* ab = a.A + (L4 ? 64 : 128) * s0;
  auto issue = [&](int k) {
    const uint32_t sb = wl0 + (uint32_t)(k % D) * L::kStep;
    const int lim = s0 + k == ng - 1 ? vlast : 7;  // pieces past K re-read the last (A is zeroed there)
#pragma unroll
    for (int i = 0; i < 2 * TT; ++i) dma16(qoff[i] + 16u * min(lc, lim), qb + 128 * k, sb + 1024u * i);
    if (r > 0) {
      const uint32_t ab0 = wl0 + L::kSign + (uint32_t)(k % D) * 2048u;
      if constexpr (L4) {
        // 64 packed bytes per row: piece i % 4 of row i / 4
        const int row = min(16 * jt + (lane >> 2), r - 1);
        dma16((uint32_t)row * (uint32_t)apitch + 16u * min(lane & 3, lim >> 1), ab + 64 * k, ab0);
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int row = min(16 * jt + 8 * h + lrow, r - 1);
          dma16((uint32_t)row * (uint32_t)apitch + 16u * min(lc, lim), ab + 128 * k, ab0 + 1024u * h);
        }
      }
    }
  };
  v4i acc[TT];
  int qs[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    acc[i] = zero4();
    qs[i] = 0;
  }
  constexpr int kLoads = 2 * TT + (L4 ? 1 : 2);  // per step
  for (int k = 0; k < D && k < n; ++k) issue(k);
  for (int k = 0; k < n; ++k) {
    const int y = min(D - 1, n - 1 - k);
    if (r > 0)
      wait_steps<kLoads>(y);
    else
      wait_steps<2 * TT>(y);
    const int8_t* st = wl + (k % D) * L::kStep + 128 * rho;
    const int8_t* as = wl + L::kSign + (k % D) * 2048;
    v4i x[2][TT], av[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int po = 16 * ((2 * kg + v) ^ swz8(rho));
#pragma unroll
      for (int i = 0; i < TT; ++i) x[v][i] = *reinterpret_cast<const v4i*>(st + 2048 * i + po);
      av[v] = zero4();
      if (r > 0) {
        if constexpr (L4) {
          const uint4 u = expand_i4(*reinterpret_cast<const uint2*>(as + 64 * rho + 16 * kg + 8 * v));
          av[v] = v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
        } else {
          av[v] = *reinterpret_cast<const v4i*>(as + 128 * rho + po);
        }
      }
    }
    wait_lds();
    if (k + D < n) issue(k + D);
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const bool past = s0 + k == ng - 1 && 2 * kg + v > vlast;
      if (past) av[v] = zero4();
      const uint32_t ones = past ? 0u : 0x01010101u;
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        acc[i] = mfma(av[v], x[v][i], acc[i]);
        if (jt == 0) {
#pragma unroll
          for (int t = 0; t < 4; ++t) qs[i] = sdot4((uint32_t)x[v][i][t], ones, qs[i]);
        }
      }
    }
  }
  // partial tiles, then per token the partial sums of Q
  int8_t* const wr = wl;
#pragma unroll
  for (int i = 0; i < TT; ++i) *reinterpret_cast<v4i*>(wr + 1024 * i + 16 * lane) = acc[i];
  if (jt == 0) {
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      int v = qs[i];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (kg == 0) *reinterpret_cast<int*>(wr + L::kSign + 64 * i + 4 * rho) = v;
    }
  }
  if (threadIdx.x == 0) {
    if (a.epoch) {
      *tag_lds = dfssm_dev::epoch_tag(ep_old);
      dfssm_dev::advance_if_last(a.epoch, b, ep_old, a.arrivals);
    } else {
      *tag_lds = a.host_tag;
    }
  }
  __syncthreads();
  const uint32_t tag = *tag_lds;
  if (wave >= TT || m0 + 16 * wave >= M) return;  // uniform
  // wave i finishes token tile i: lane (rho, kg) holds ranks 16jt + 4kg + v
  v4i d = zero4();
  for (int w = 0; w < KW; ++w) d += *reinterpret_cast<const v4i*>(lds + w * L::kBytes + 1024 * wave + 16 * lane);
  const int m = m0 + 16 * wave + rho;
  const int tile = (m0 >> 4) + wave;
  uint64_t* lw = limb_words(a, tile, jt >> 2) + 16 * (jt & 3) + rho;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int j = 16 * jt + 4 * kg + v;
    const int val = j < r ? d[v] : 0;
    if (r > 0) word_store(lw + 64 * (4 * kg + v), tag, pack_limbs(val));
    if (a.acc_a_out && j < r && m < M) a.acc_a_out[(int64_t)m * r + j] = val;
  }
  if (jt == 0 && kg == 0 && m < M) {
    int t = 0;
    for (int w = 0; w < KW; ++w) t += *reinterpret_cast<const int*>(lds + w * L::kBytes + L::kSign + 64 * wave + 4 * rho);
    word_store(sumq_words(a) + m, tag, (uint32_t)t);
  }
}

// BIG: ranks above 64 (rp > 64), a separate instantiation: its chunk loop costs
// registers
template <int TT, int RT, int KW, int D, bool L4, bool BIG>
__global__ __launch_bounds__(64 * KW, TT == 1 && !BIG ? 4 : 2) void mfma_mid(MidArgs a) {
  using L = WaveLds<TT, RT, D>;
  constexpr int kTiles = TT * RT;
  constexpr int P = kTiles >= KW ? kTiles / KW : 1;  // tiles a wave finishes
  static_assert(kTiles < KW || (kTiles % KW == 0 && RT % P == 0), "a wave finishes row tiles of one token tile");
  static_assert(D <= 4 && 64 * TT + 16 <= L::kBytes - L::kSign, "wait counts, LDS layout");
  __shared__ __attribute__((aligned(16))) int8_t lds[KW * L::kBytes];
  uint32_t* const tag_lds = reinterpret_cast<uint32_t*>(lds + L::kBytes - 16);  // past every wave's use of wave 0's area
  const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(lds_void*)lds);
  if ((int)blockIdx.x < a.nb_lora) {
    mid_lora<TT, RT, KW, D, L4>(a, lds, lds0, tag_lds);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rho = lane & 15, kg = lane >> 4;
  const int M = a.M, K = a.K, N = a.N, r = a.r, W = K >> 5;
  uint64_t ep_old = 0;
  if (a.epoch && threadIdx.x == 0) ep_old = dfssm_dev::arrive(a.epoch, blockIdx.x);
  // each XCD (workgroup id % 8) takes a contiguous run of the row-major tile
  // list: its sign rows come from memory once, into its own L2
  int tile_id;
  {
    const int idx = (int)blockIdx.x - a.nb_lora, cnt = a.ntb * a.nrb;
    const int per = cnt >> 3, rem = cnt & 7, x = idx & 7;
    tile_id = x * per + min(x, rem) + (idx >> 3);
  }
  const int rb = tile_id / a.ntb, tb = tile_id - rb * a.ntb;
  const int m0 = 16 * TT * tb, n0 = 16 * RT * rb;
  // this wave's steps of 128 columns
  const int ng = (K + 127) >> 7;
  const int s0 = wave * ng / KW, n = (wave + 1) * ng / KW - s0;
  const int vlast = ((K - 1) & 127) / 16;  // last 16-byte piece of a row's last step
  int8_t* const wl = lds + wave * L::kBytes;
  const uint32_t wl0 = lds0 + (uint32_t)(wave * L::kBytes);

  const int8_t* qb = a.q + (int64_t)m0 * K + 128 * s0;
  const uint32_t* wb = a.w_bits + (int64_t)n0 * W + 4 * s0;
  const int lrow = lane >> 3, lc = (lane & 7) ^ lrow;  // row of a load's 8, piece fetched
  uint32_t qoff[2 * TT];
#pragma unroll
  for (int i = 0; i < 2 * TT; ++i) qoff[i] = (uint32_t)(min(m0 + 8 * i + lrow, M - 1) - m0) * (uint32_t)K;
  // sign words of 2 steps: 32 bytes of each row as two 16-byte pieces, piece
  // p of row n at slot p ^ ((n >> 2) & 1).  Lane i of a load fetches slot i % 2
  // of row i / 2 (32 rows a load).  Rows of other than whole 16-byte pieces
  // (K % 128 != 0) go word by word, lane i: word i % 8 of row i / 8.
  const bool wvec = (W & 3) == 0;
  constexpr int kSignLoads = (RT + 1) / 2;
  auto issue_signs = [&](int c) {  // steps 2c, 2c+1 of this wave
    const uint32_t sb = wl0 + L::kSign + (uint32_t)(c & 1) * L::kSignBuf;
    const int w0 = 4 * s0 + 8 * c;  // first word
    if (wvec) {
#pragma unroll
      for (int j = 0; j < kSignLoads; ++j) {
        const int row = 32 * j + (lane >> 1);
        const int wd = min(4 * ((lane & 1) ^ ((row >> 2) & 1)), W - 4 - w0);
        const uint32_t o = (uint32_t)(min(n0 + row, N - 1) - n0) * (uint32_t)W + (uint32_t)wd;
        if (RT % 2 == 0 || j + 1 < kSignLoads || lane < 32) dma16(4u * o, wb + 8 * c, sb + 1024u * j);
      }
    } else {
      // words past the row re-read its last (zeroed when used)
#pragma unroll
      for (int j = 0; j < 2 * RT; ++j) {
        const int row = 8 * j + (lane >> 3);
        const int wd = min((lane & 3) + 4 * (((lane >> 2) & 1) ^ ((row >> 2) & 1)), W - 1 - w0);
        const uint32_t o = (uint32_t)(min(n0 + row, N - 1) - n0) * (uint32_t)W + (uint32_t)wd;
        dma4(4u * o, wb + 8 * c, sb + 256u * j);
      }
    }
  };
  auto issue = [&](int k) {
    if ((k & 1) == 0) issue_signs(k >> 1);
    const uint32_t sb = wl0 + (uint32_t)(k % D) * L::kStep;
    const int lim = s0 + k == ng - 1 ? vlast : 7;  // pieces past K re-read the last (their signs are zeroed)
#pragma unroll
    for (int i = 0; i < 2 * TT; ++i) dma16(qoff[i] + 16u * min(lc, lim), qb + 128 * k, sb + 1024u * i);
  };
  v4i acc[RT][TT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < TT; ++i) acc[t][i] = zero4();

  // ---- operands of the tiles this wave finishes go out first
  const bool fin = wave * P < kTiles;
  const int fi = (wave * P) / RT, ft = (wave * P) % RT;
  const int mtok = m0 + 16 * fi + rho;
  const int mc = min(mtok, M - 1);
  const bool ba = (r % 16) == 0;
  const int64_t bpitch = L4 ? r / 2 : r;
  v4i bop[P];
  float alv[P][4], bev[P][4];
  float sm = 0.f;

  if (fin) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int nt = n0 + 16 * (ft + p);
      bop[p] = r > 0 ? load16_row_guarded<L4>(a.B + (int64_t)min(nt + rho, N - 1) * bpitch, 16 * kg, r, ba) : zero4();
      const int nb = nt + 4 * kg;
      if ((N & 3) == 0 && nb + 3 < N) {
        const float4 al4 = *reinterpret_cast<const float4*>(a.alpha + nb);
        alv[p][0] = al4.x; alv[p][1] = al4.y; alv[p][2] = al4.z; alv[p][3] = al4.w;
        if (r > 0) {
          const float4 be4 = *reinterpret_cast<const float4*>(a.beta + nb);
          bev[p][0] = be4.x; bev[p][1] = be4.y; bev[p][2] = be4.z; bev[p][3] = be4.w;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int n = min(nb + v, N - 1);
          alv[p][v] = a.alpha[n];
          bev[p][v] = r > 0 ? a.beta[n] : 0.f;
        }
      }
    }
    sm = a.s[mc];
  }
  for (int k = 0; k < D && k < n; ++k) issue(k);
  for (int k = 0; k < n; ++k) {
    // sign loads among the younger ones only make this wait longer
    wait_steps<2 * TT>(min(D - 1, n - 1 - k));
    const int8_t* st = wl + (k % D) * L::kStep + 128 * rho;
    // lane group kg takes columns 32kg .. 32kg+31 of the step, 16 per MFMA:
    // word kg of the row's 4
    const int8_t* sg_ = wl + L::kSign + ((k >> 1) & 1) * L::kSignBuf + 32 * rho +
                        16 * ((k & 1) ^ ((rho >> 2) & 1)) + 4 * kg;
    v4i x[2][TT];
    uint32_t w[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) w[t] = *reinterpret_cast<const uint32_t*>(sg_ + 512 * t);
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int i = 0; i < TT; ++i)
        x[v][i] = *reinterpret_cast<const v4i*>(st + 2048 * i + 16 * ((2 * kg + v) ^ swz8(rho)));
    wait_lds();
    if (k + D < n) issue(k + D);
    if (s0 + k == ng - 1 && 2 * kg > vlast) {  // words past K count as 0 (K % 32 == 0: whole words)
#pragma unroll
      for (int t = 0; t < RT; ++t) w[t] = 0u;
    }
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const v4i sg = expand16_at(w[t], 16 * v);
#pragma unroll
        for (int i = 0; i < TT; ++i) acc[t][i] = mfma(sg, x[v][i], acc[t][i]);
      }
  }

  // this wave's partial tiles over its own ring
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < TT; ++i) *reinterpret_cast<v4i*>(wl + 1024 * (i * RT + t) + 16 * lane) = acc[t][i];

  // ---- the first poll of the LoRA words is on its way during the reduction
  const int tile = (m0 >> 4) + fi;
  const bool live = fin && m0 + 16 * fi < M;  // uniform
  uint64_t w[16], wq = 0;
  auto poll = [&](int chunk, bool want_q) {
    const uint64_t* lw = limb_words(a, tile, chunk) + lane;
    if (64 * chunk + 16 * kg < r) {
#pragma unroll
      for (int e = 0; e < 16; ++e) w[e] = word_load(lw + 64 * e);
    }
    if (want_q) wq = word_load(sumq_words(a) + mc);
  };
  if (live) poll(0, true);
  if (threadIdx.x == 0) {
    if (a.epoch) {
      *tag_lds = dfssm_dev::epoch_tag(ep_old);
      dfssm_dev::advance_if_last(a.epoch, blockIdx.x, ep_old, a.arrivals);
    } else {
      *tag_lds = a.host_tag;
    }
  }
  __syncthreads();
  if (!live) return;
  const uint32_t tag = *tag_lds;
  v4i d[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int8_t* rd = lds + 1024 * (fi * RT + ft + p) + 16 * lane;
    d[p] = *reinterpret_cast<const v4i*>(rd);
#pragma unroll
    for (int u = 1; u < KW; ++u) d[p] += *reinterpret_cast<const v4i*>(rd + u * L::kBytes);
    // summed before the wait for the LoRA words: left to itself the compiler
    // keeps all KW terms in registers across it, and spills
    asm volatile("" : "+v"(d[p]));
  }
  const bool keep = rb == 0 && ft == 0 && a.acc_a_out && mtok < M;  // values computed here go to acc_a_out
  int sq = 0;
  v4i lm[4];
  auto finish_poll = [&](int chunk, bool want_q) {
    const int j0 = 64 * chunk + 16 * kg;
    uint32_t val[16];
    auto arrived = [&] {
      uint32_t other = want_q ? (uint32_t)(wq >> 32) ^ tag : 0u;
      if (j0 < r) {
#pragma unroll
        for (int e = 0; e < 16; ++e) other |= (uint32_t)(w[e] >> 32) ^ tag;
      }
      return other == 0u;
    };
    bool have = arrived();
    for (int it = 0; !__all(have) && it < a.spin; ++it) {
      __builtin_amdgcn_s_sleep(1);
      poll(chunk, want_q);
      have = arrived();
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) val[e] = j0 < r ? (uint32_t)w[e] : 0u;
    if (want_q) sq = (int)(uint32_t)wq;
    if (!have) {
      // the LoRA workgroups' words did not arrive: compute them here
#pragma unroll 1
      for (int e = 0; e < 16; ++e) {
        const int v = j0 + e < r ? lane_dot<L4>(a.A, a.q, K, j0 + e, mc) : 0;
        const uint32_t pl = pack_limbs(v);
#pragma unroll
        for (int f = 0; f < 16; ++f) val[f] = f == e ? pl : val[f];
        if (keep && j0 + e < r) a.acc_a_out[(int64_t)mc * r + j0 + e] = v;
      }
      if (want_q) sq = lane_dot<L4>(a.A, a.q, K, -1, mc);
    }
    limb_operands(val, lm);
  };

  v4i ehi[P], elo[P];
#pragma unroll
  for (int p = 0; p < P; ++p) ehi[p] = elo[p] = zero4();
  auto up = [&] {  // one 64-rank chunk
#pragma unroll
    for (int p = 0; p < P; ++p) {
      ehi[p] = mfma(bop[p], lm[2], ehi[p] + (mfma(bop[p], lm[3], zero4()) << 8));
      elo[p] = mfma(bop[p], lm[0], elo[p] + (mfma(bop[p], lm[1], zero4()) << 8));
    }
  };
  if constexpr (!BIG) {
    finish_poll(0, true);
    if (r > 0) up();
  } else {
#pragma unroll 1
    for (int c = 0; c < a.rp >> 6; ++c) {
      if (c > 0) {
        poll(c, false);
#pragma unroll
        for (int p = 0; p < P; ++p)
          bop[p] = load16_row_guarded<L4>(a.B + (int64_t)min(n0 + 16 * (ft + p) + rho, N - 1) * bpitch,
                                          64 * c + 16 * kg, r, ba);
      }
      finish_poll(c, c == 0);
      up();
    }
  }
  if (mtok >= M) return;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int nb = n0 + 16 * (ft + p) + 4 * kg;
    float yv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t as = 2 * d[p][v] - sq;
      yv[v] = dfssm_dev::epilogue(sm, alv[p][v], bev[p][v], as, ehi[p][v], elo[p][v], r > 0);
      if (nb + v < N) {
        if (a.acc_s_out) a.acc_s_out[(int64_t)mtok * N + nb + v] = as;
        if (a.acc_b_out)
          a.acc_b_out[(int64_t)mtok * N + nb + v] = r > 0 ? (int64_t)elo[p][v] + ((int64_t)ehi[p][v] << 16) : 0;
      }
    }
    if (a.y) {
      float* dst = a.y + (int64_t)mtok * N + nb;
      if ((N & 3) == 0 && nb + 3 < N) {
        *reinterpret_cast<float4*>(dst) = make_float4(yv[0], yv[1], yv[2], yv[3]);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (nb + v < N) dst[v] = yv[v];
      }
    }
  }
}

template <int TT, int RT, int KW, int D, bool L4, bool BIG = false>
hipError_t launch_t(MidArgs a, hipStream_t st) {
  a.ntb = (int)dfssm::ceil_div(a.M, 16 * TT);
  a.nrb = (int)dfssm::ceil_div(a.N, 16 * RT);
  a.nrt = std::max(1, (a.r + 15) / 16);
  a.nb_lora = a.spin > 0 ? a.ntb * a.nrt : 0;
  a.arrivals = a.nb_lora + a.ntb * a.nrb;
  mfma_mid<TT, RT, KW, D, L4, BIG><<<dim3((unsigned)a.arrivals), dim3(64 * KW), 0, st>>>(a);
  return hipGetLastError();
}

// The tile forms and their modelled cost (us): with x = workgroups per CU, R = the
// workgroups that fit a CU at once (LDS and registers), e = ceil(x) - 1, s = max(0,
// x - 1), E = ceil(x / R) - 1, m = min(1, x) and k = K / 1024,
//   c0 + c1 k + (c2 + c3 k) e + (c4 + c5 k) s + (c6 + c7 k) E + (c8 + c9 k) m,
// that is one workgroup's chain of latencies, what further workgroups on a CU add,
// what they share, a step for every further round and how full the first is; c10 x
// where N % 16 != 0 (a token's outputs then start off the 64-byte segments of a
// tile's stores); c11 x l with l = M K / 4 MB - 1 within 0 .. 1 (the codes outgrow an
// XCD's L2); and (c12 + c13 min(1, e)) ceil(r / 16) / 4 up to rank 64, or above, with
// coefficients of their own, (c12 + c13 s) g for g further chunks of 64 ranks.  Fitted
// on MI355X, slopes held above 0, each call of a graph on weights of its own (400 MB
// of them in turn, as a decode step meets them): a grid of 3 to 4096 tokens on 19
// shapes (K = 512 to 16384 x N = 512 to 9600), r = 0 to 256, int8 and int4, and 1470
// calls drawn from 2 to 7001 tokens of the projections of d = 768 to 2560 in steps of
// 128.  On drawn calls that a fit had not seen, the choice between these forms and the
// many-token tiles takes 0.3% more time than the fastest form up to 64 tokens, 0.8%
// above; fitted on the grid alone, with neither E, m nor l, 2.2%, and 24% just short
// of a full round (957 x 1920 x 7996 44.0 us, the fastest 35.5).
struct MidForm {
  int tt, rt;
  int res[2];  // R up to rank 64, and above
  double c[2][14];
};
constexpr MidForm kMidForms[] = {
    // 64 x 64, 8 waves; 4 waves
    {4, 4, {1, 1},
     {{6.611, 1.031, 1.908, 1.042, 2.681, 0.504, 0, 0, 0.844, 0.243, -0.012, 1.142, -0.040, 0.980},
      {5.910, 1.099, 1.169, 0.486, 5.172, 1.082, 0, 0, 2.023, 0.071, 0.084, 0.651, 1.345, 1.152}}},
    {4, 4, {2, 2},
     {{8.533, 1.326, 0, 0.968, 1.903, 0.060, 2.538, 0, 0.658, 0.050, 0.018, 1.946, -1.389, -0.279},
      {6.751, 1.410, 0.724, 0.010, 0.638, 1.187, 3.523, 0, 1.032, -0.158, -0.126, 1.048, 1.472, 0.791}}},
    // 32 x 64, 8 waves; 4 waves
    {2, 4, {1, 1},
     {{5.288, 0.749, 2.034, 0.497, 1.359, 0.385, 0, 0, 0.737, -0.004, 0.059, 0.298, 0.272, 0.291},
      {5.127, 0.733, 0.619, 0.432, 3.698, 0.303, 0, 0, 1.252, 0.081, 0.248, 0, 1.251, 0.585}}},
    {2, 4, {3, 2},
     {{6.038, 0.988, 0, 0.325, 1.028, 0.379, 0.964, 0, 0.196, 0.016, 0.007, 0.568, -0.491, 0.003},
      {5.323, 0.998, 0.284, 0.018, 1.972, 0.358, 0.550, 0.515, 0.159, 0.004, -0.001, 1.872, 1.253, 0.339}}},
    // 16 x 64, 4 waves; 16 x 32 and 16 x 16, 8 waves
    {1, 4, {4, 3},
     {{4.829, 0.829, 0.236, 0.236, 0.463, 0.191, 0.764, 0.105, -0.043, -0.015, -0.015, 0.077, 0.494, -0.072},
      {5.335, 0.736, 0.214, 0.090, 1.382, 0.184, 0, 0.097, -0.034, -0.033, 0.146, 0.457, 1.188, 0.164}}},
    {1, 2, {2, 1},
     {{4.754, 0.431, 0.492, 0, 0.032, 0.124, 1.649, 0.133, -0.012, 0.082, 0.089, 0.656, 0.424, 0.498},
      {5.126, 0.420, 0.886, 0.389, 0.110, 0, 0, 0, -0.393, 0.096, 0.204, 0.284, 1.072, 0.174}}},
    {1, 1, {2, 1},
     {{4.242, 0.436, 0.421, 0, 0.035, 0.126, 1.803, 0, 0.092, 0.109, 0.112, 1.384, 0.441, 0.215},
      {4.634, 0.427, 0.390, 0.156, 0.603, 0.146, 0, 0, 0.086, 0.026, 0.083, 0, 1.006, 0.153}}},
};
struct MidPlan {
  int form;
  double us;
};
MidPlan plan_mid(int64_t M, int64_t K, int64_t N, int64_t r) {
  // test switch linear_kernel: form n - 2
  const int forced = dfssm::test_switch(DFSSM_TEST_LINEAR_KERNEL);
  if (forced >= 2) return {forced - 2, 0.0};
  MidPlan best{0, std::numeric_limits<double>::infinity()};
  const int cus = dfssm::device_cu_count();
  const double k = (double)K / 1024.0;
  const double l = std::min(1.0, std::max(0.0, (double)M * (double)K / 4194304.0 - 1.0));
  for (int f = 0; f < (int)(sizeof(kMidForms) / sizeof(kMidForms[0])); ++f) {
    const MidForm& F = kMidForms[f];
    const int64_t tb = dfssm::ceil_div(M, 16 * F.tt);
    const double blocks = (double)tb * (double)(dfssm::ceil_div(N, 16 * F.rt) + std::max<int64_t>(1, dfssm::ceil_div(r, 16)));
    const double x = blocks / cus, e = std::max(0.0, std::ceil(x) - 1.0), s = std::max(0.0, x - 1.0);
    const double E = std::max(0.0, std::ceil(x / F.res[r > 64]) - 1.0), m = std::min(1.0, x);
    const double* c = F.c[r > 64];
    const double rank = r <= 64 ? (c[12] + c[13] * std::min(1.0, e)) * (double)dfssm::ceil_div(r, 16) / 4.0
                                : (c[12] + c[13] * s) * (double)(dfssm::ceil_div(r, 64) - 1);
    const double us = c[0] + c[1] * k + (c[2] + c[3] * k) * e + (c[4] + c[5] * k) * s + (c[6] + c[7] * k) * E +
                      (c[8] + c[9] * k) * m + (N % 16 ? c[10] * x : 0.0) + c[11] * x * l + rank;
    if (us < best.us) best = {f, us};
  }
  return best;
}

template <bool L4, bool BIG>
hipError_t launch_form(int form, const MidArgs& a, hipStream_t st) {
  switch (form) {
    case 0: return launch_t<4, 4, 8, 2, L4, BIG>(a, st);
    case 1: return launch_t<4, 4, 4, 2, L4, BIG>(a, st);
    case 2: return launch_t<2, 4, 8, 2, L4, BIG>(a, st);
    case 3: return launch_t<2, 4, 4, 2, L4, BIG>(a, st);
    case 4: return launch_t<1, 4, 4, 2, L4, BIG>(a, st);
    case 5: return launch_t<1, 2, 8, 2, L4, BIG>(a, st);
    default: return launch_t<1, 1, 8, 2, L4, BIG>(a, st);
  }
}

int tile_shift(int64_t r) { return r <= 16 ? 2 : (r <= 32 ? 1 : 0); }

template <bool L4>
hipError_t mid_impl(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N, int64_t r,
                    const uint32_t* w_bits, const float* alpha, const int8_t* A, const int8_t* B,
                    const float* beta, float* y, int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                    const dfssm::LinearWorkspace& ws, hipStream_t st) {
  using namespace dfssm;
  if (M == 0 || N == 0) return hipSuccess;
  const int rp = (int)rank_padded(r);
  if (!mid_takes(M, r)) return hipErrorInvalidValue;
  // Test switch local_lora: no LoRA workgroups, every lane computes its LoRA
  // values itself at once (the path a lane takes when the words never arrive).
  const bool local_only = test_switch(DFSSM_TEST_LOCAL_LORA) == 1;
  const bool dev = wants_device_epoch(st);
  MidArgs a{q, s, (int)M, (int)K, (int)N, (int)r, rp, w_bits, alpha, A, B, beta, y, acc_s, r > 0 ? acc_a_out : nullptr,
            acc_b, ws.xw, dev ? ws.epoch : nullptr, dev ? 0u : next_host_tag(), 0, tile_shift(r), 0, 0, 0, 0,
            local_only ? 0 : (1 << 14)};
  const int form = plan_mid(M, K, N, r).form;
  return rp > 64 ? launch_form<L4, true>(form, a, st) : launch_form<L4, false>(form, a, st);
}

}  // namespace

namespace dfssm {

bool mid_takes(int64_t M, int64_t r) {
  const int64_t tiles = ceil_div(M, 16);
  return (r > 0 ? ceil_div(tiles, 1 << tile_shift(r)) * 16 * rank_padded(r) : 0) + 16 * tiles <= kXwWords;
}

double mid_cost_us(int64_t M, int64_t K, int64_t N, int64_t r) { return plan_mid(M, K, N, r).us; }

hipError_t launch_mid_linear(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N,
                             int64_t r, const uint32_t* w_bits, const float* alpha,
                             const int8_t* A, const int8_t* B, const float* beta, float* y,
                             int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                             const LinearWorkspace& ws, hipStream_t st) {
  return mid_impl<false>(q, s, M, K, N, r, w_bits, alpha, A, B, beta, y, acc_s, acc_a_out, acc_b, ws, st);
}

hipError_t launch_mid_linear_i4(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N,
                                int64_t r, const uint32_t* w_bits, const float* alpha,
                                const uint8_t* A4, const uint8_t* B4, const float* beta, float* y,
                                int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                                const LinearWorkspace& ws, hipStream_t st) {
  return mid_impl<true>(q, s, M, K, N, r, w_bits, alpha, reinterpret_cast<const int8_t*>(A4),
                        reinterpret_cast<const int8_t*>(B4), beta, y, acc_s, acc_a_out, acc_b, ws, st);
}

}  // namespace dfssm
