// dfssm_tile.hip -- scaffold + LoRA linear for many tokens (prefill) on the
// gfx950 int8 matrix cores (v_mfma_i32_16x16x64_i8), two launches.
//
// The sign bits are expanded on chip, in registers, to {0,1} bytes (a nibble
// n becomes bytes via (n * 0x00204081) & 0x01010101), so the MFMA computes
// D[n,m] = sum_{bit=1} Q[m,k] and acc_s = 2*D - sum_k Q[m,k]; the expanded signs
// never touch memory or LDS (the paper expands to int8 "on the fly" ahead of
// a library int8 GEMM, Sec. 4.1).
//
// lora_down computes acc_a = Q A^T with the same MFMA and writes it as 4
// signed base-256 int8 limbs, and sum_k Q.  mfma_tile gets the exact int64
// acc_b = sum_j B[n,j] acc_a[m,j] from four int8 MFMAs per 16x16 tile, E_hi =
// 256*(B.L3) + B.L2 and E_lo = 256*(B.L1) + B.L0 (each < 2^31 for r <= 256),
// acc_b = E_lo + 65536*E_hi; where a tile's acc_a are small enough for acc_b
// to fit 32 bits (they are for real activations) three MFMAs give it directly
// and the int64 -> fp32 conversion falls away.
//
// Operands of both kernels reach LDS by direct-to-LDS loads of whole 128-byte
// lines of Q (stages of 128 columns): a CU draws 60 bytes per clock from its
// L2 that way and 36 with 64-byte pieces of rows.  Signs come in groups of
// G stages, 16 G bytes of each row.  16-byte pieces of a row are stored
// swizzled (swz8).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "dfssm_int4.hpp"
#include "dfssm_linear.hpp"

namespace {

using namespace dfssm_lin;

// ------------------------------------------------------------ LoRA down
struct DownArgs {
  const int8_t* q;
  int M, K, r, rp;
  const int8_t* A;
  int8_t* limbs;     // [4][M][rp]
  int32_t* sumq;     // [M]
  int32_t* acc_a;    // [M][r], or NULL
};

// 16 tokens x 16*RA ranks per workgroup, K split over KW waves
template <int RA, int KW, bool L4>
__global__ __launch_bounds__(64 * KW, 2) void lora_down(DownArgs a) {
  constexpr int kStep = 2048 + RA * 2048;
  constexpr int D = 2;
  constexpr int kBytes = D * kStep;
  static_assert(kBytes >= RA * 1024 + 64, "partial tiles overlay the ring");
  __shared__ __attribute__((aligned(16))) int8_t lds[KW * kBytes];
  const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(lds_void*)lds);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rho = lane & 15, kg = lane >> 4;
  const int M = a.M, K = a.K, r = a.r;
  const int m0 = 16 * blockIdx.x, j0 = 16 * RA * blockIdx.y;
  const bool first = blockIdx.y == 0;
  const int ng = (K + 127) >> 7;
  const int s0 = wave * ng / KW, n = (wave + 1) * ng / KW - s0;
  const int vlast = ((K - 1) & 127) / 16;
  int8_t* const wl = lds + wave * kBytes;
  const uint32_t wl0 = lds0 + (uint32_t)(wave * kBytes);
  const int8_t* qb = a.q + (int64_t)m0 * K + 128 * s0;
  const int lrow = lane >> 3, lc = (lane & 7) ^ lrow;
  uint32_t qoff[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) qoff[i] = (uint32_t)(min(m0 + 8 * i + lrow, M - 1) - m0) * (uint32_t)K;
  const int apitch = L4 ? K / 2 : K;
  const int8_t* ab = a.A + (L4 ? 64 : 128) * s0;  // rows from 0: a workgroup may lie wholly past rank r
  auto issue = [&](int k) {
    const uint32_t sb = wl0 + (uint32_t)(k % D) * kStep;
    const int lim = s0 + k == ng - 1 ? vlast : 7;
#pragma unroll
    for (int i = 0; i < 2; ++i) dma16(qoff[i] + 16u * min(lc, lim), qb + 128 * k, sb + 1024u * i);
    if (r > 0) {
      if constexpr (L4) {
#pragma unroll
        for (int t = 0; t < RA; ++t) {
          const int row = min(j0 + 16 * t + (lane >> 2), r - 1);
          dma16((uint32_t)(row * apitch) + 16u * min(lane & 3, lim >> 1), ab + 64 * k, sb + 2048u + 1024u * t);
        }
      } else {
#pragma unroll
        for (int t = 0; t < 2 * RA; ++t) {
          const int row = min(j0 + 8 * t + lrow, r - 1);
          dma16((uint32_t)(row * apitch) + 16u * min(lc, lim), ab + 128 * k, sb + 2048u + 1024u * t);
        }
      }
    }
  };
  v4i acc[RA];
#pragma unroll
  for (int t = 0; t < RA; ++t) acc[t] = zero4();
  int qs = 0;
  for (int k = 0; k < D && k < n; ++k) issue(k);
  for (int k = 0; k < n; ++k) {
    const int y = min(D - 1, n - 1 - k);
    if (r > 0)
      wait_steps<2 + (L4 ? RA : 2 * RA)>(y);
    else
      wait_steps<2>(y);
    const int8_t* st = wl + (k % D) * kStep;
    v4i x[2], av[2][RA];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int po = 16 * ((2 * kg + v) ^ swz8(rho));
      x[v] = *reinterpret_cast<const v4i*>(st + 128 * rho + po);
#pragma unroll
      for (int t = 0; t < RA; ++t) {
        av[v][t] = zero4();
        if (r > 0) {
          if constexpr (L4) {
            const uint4 u = expand_i4(
                *reinterpret_cast<const uint2*>(st + 2048 + 1024 * t + 64 * rho + 16 * kg + 8 * v));
            av[v][t] = v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
          } else {
            av[v][t] = *reinterpret_cast<const v4i*>(st + 2048 + 2048 * t + 128 * rho + po);
          }
        }
      }
    }
    wait_lds();
    if (k + D < n) issue(k + D);
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      if (s0 + k == ng - 1 && 2 * kg + v > vlast) x[v] = zero4();  // columns past K
#pragma unroll
      for (int t = 0; t < RA; ++t) acc[t] = mfma(av[v][t], x[v], acc[t]);
      if (first) {
#pragma unroll
        for (int t = 0; t < 4; ++t) qs = sdot4((uint32_t)x[v][t], 0x01010101u, qs);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < RA; ++t) *reinterpret_cast<v4i*>(wl + 1024 * t + 16 * lane) = acc[t];
  if (first) {
    qs += __shfl_xor(qs, 16, 64);
    qs += __shfl_xor(qs, 32, 64);
    if (kg == 0) *reinterpret_cast<int*>(wl + 1024 * RA + 4 * rho) = qs;
  }
  __syncthreads();
  const int m = m0 + rho;
  if (RA == 1 && r > 0 && wave >= RA && wave < 4 && m < M) {
    // ranks 16 .. 63 of the padded rank: zero limbs
#pragma unroll
    for (int l = 0; l < 4; ++l)
      *reinterpret_cast<uint32_t*>(a.limbs + ((int64_t)l * M + m) * a.rp + j0 + 16 * wave + 4 * kg) = 0u;
  }
  if (wave < RA && m < M) {
    // wave t finishes rank tile t: lane (rho, kg) holds ranks 4kg .. 4kg+3
    v4i d = zero4();
    for (int w = 0; w < KW; ++w) d += *reinterpret_cast<const v4i*>(lds + w * kBytes + 1024 * wave + 16 * lane);
    const int j = j0 + 16 * wave + 4 * kg;
    uint32_t pl[4] = {0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int val = j + v < r ? d[v] : 0;
      const uint32_t p = pack_limbs(val);
#pragma unroll
      for (int l = 0; l < 4; ++l) pl[l] |= ((p >> (8 * l)) & 0xffu) << (8 * v);
      if (a.acc_a && j + v < r) a.acc_a[(int64_t)m * r + j + v] = val;
    }
    if (r > 0) {
#pragma unroll
      for (int l = 0; l < 4; ++l) *reinterpret_cast<uint32_t*>(a.limbs + ((int64_t)l * M + m) * a.rp + j) = pl[l];
    }
  }
  if (first && wave == KW - 1 && kg == 0 && m < M) {
    int t = 0;
    for (int w = 0; w < KW; ++w) t += *reinterpret_cast<const int*>(lds + w * kBytes + 1024 * RA + 4 * rho);
    a.sumq[m] = t;
  }
}

// ------------------------------------------------------------ scaffold tiles
struct TileArgs {
  const int8_t* q;
  const float* s;
  int M, K, N, r, rp;
  const uint32_t* w_bits;
  const float* alpha;
  const int8_t* limbs;
  const int8_t* B;
  const float* beta;
  const int32_t* sumq;
  float* y;
  int32_t* acc_s_out;
  int64_t* acc_b_out;
  int l4;        // B holds packed int4
  int ntb, nrb;  // token blocks, row blocks
  int run, runx; // row tiles per block; the first runx blocks hold one more
};

// Whether 128 * sum_j |acc_a[j]| < 2^31 for this lane's token, from its limb
// operands (16 ranks a lane, the four lanes rho + 16 kg of a token together)
__device__ __forceinline__ bool fits32(const v4i (&lm)[4]) {
  uint32_t sum = 0, top = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    sum = __builtin_amdgcn_sad_u8((uint32_t)lm[2][d] ^ 0x80808080u, 0x80808080u, sum);
    top |= (uint32_t)lm[3][d];
  }
  sum += top ? 256u : 16u;
  sum += (uint32_t)__shfl_xor((int)sum, 16, 64);
  sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
  return sum < 256u;
}

// bits [sh, sh+4) of w -> 4 bytes of {0,1}
__device__ __forceinline__ int expand4(uint32_t w, uint32_t sh) {
  return (int)((__builtin_amdgcn_ubfe(w, sh, 4) * 0x00204081u) & 0x01010101u);
}

// Tile index of block b among cnt blocks whose XCD is b % 8: each XCD gets a
// contiguous run of the token-major tile list
__device__ __forceinline__ int xcd_tile(int b, int cnt) {
  const int per = cnt >> 3, rem = cnt & 7, x = b & 7;
  return x * per + min(x, rem) + (b >> 3);
}

// Workgroup of WT x WR = 4 waves: 16*TT*WT tokens x 16*RT*WR rows, wave (wt, wr)
// owns 16*TT x 16*RT of them.  K in stages of 128 columns, a ring of D stages
// of Q; signs in groups of G stages, two buffers.
template <int TT, int RT, int WT, int D, int G, bool BIG>
__global__ __launch_bounds__(256, 2) void mfma_tile(TileArgs a) {
  constexpr int WR = 4 / WT;
  constexpr bool kX = WT == 1;  // runs of up to 4*RT + 1 row tiles, the last one shared by the waves
  constexpr int kRowsQ = 16 * TT * WT, kRowsS = 16 * RT * WR + (kX ? 16 : 0);
  constexpr int kQStage = kRowsQ * 128;
  constexpr int kSgRow = 16 * G;  // bytes of a sign row per group
  constexpr int kSgBuf = kRowsS * kSgRow;
  constexpr int kLq = kRowsQ / 32;              // Q loads per wave and stage
  constexpr int kSi = (kRowsS * kSgRow + 1023) / 1024;  // sign loads per group, all waves
  static_assert(kRowsQ % 32 == 0 && (G == 2 || G == 4) && D >= 2 && D <= 4 && G >= D - 1, "");
  constexpr int kLimb = 4 * kRowsQ * 64;  // the tile's limbs, then its B rows, over the ring
  static_assert((BIG ? kRowsS * 256 : kLimb + kRowsS * 64) <= D * kQStage + 2 * kSgBuf, "LoRA operands overlay the ring");
  __shared__ __attribute__((aligned(16))) int8_t lds[D * kQStage + 2 * kSgBuf];
  __shared__ __attribute__((aligned(16))) float al_lds[kRowsS], be_lds[kRowsS], s_lds[kRowsQ];
  __shared__ __attribute__((aligned(16))) int32_t sq_lds[kRowsQ];
  const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(lds_void*)lds);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wt = wave % WT, wr = wave / WT;
  const int rho = lane & 15, kg = lane >> 4;
  const int M = a.M, K = a.K, N = a.N, r = a.r, W = K >> 5;
  const int tile = xcd_tile(blockIdx.x, a.ntb * a.nrb);
  const int tb = tile / a.nrb, rb = tile - tb * a.nrb;
  const int m0 = kRowsQ * tb;
  // this block's run of row tiles: lengths differ by at most one
  const int rt0 = rb * a.run + min(rb, a.runx), cnt = a.run + (rb < a.runx ? 1 : 0);
  const int n0 = 16 * rt0;
  const bool extra = kX && cnt > RT * WR;
  const int ng = (K + 127) >> 7;
  const int vlast = ((K - 1) & 127) / 16;

  const int8_t* qb = a.q + (int64_t)m0 * K;
  const uint32_t* wb = a.w_bits + (int64_t)n0 * W;
  const int lrow = lane >> 3, lc = (lane & 7) ^ lrow;
  // Q rows 8 (wave + 4i) + lrow of the tile
  uint32_t qoff[kLq];
#pragma unroll
  for (int i = 0; i < kLq; ++i)
    qoff[i] = (uint32_t)(min(m0 + 8 * (wave + 4 * i) + lrow, M - 1) - m0) * (uint32_t)K + 16u * lc;
  // sign rows: 16-byte piece of stage p of a group at slot p ^ sswz(row)
  constexpr int kRpi = 1024 / kSgRow;  // rows per load
  constexpr int kSl = (kSi + 3) / 4;
  auto sswz = [](int row) { return G == 4 ? (row >> 1) & 3 : (row >> 2) & 1; };
  uint32_t soff[kSl];
  const int spc = (lane % G) ^ sswz(lane / G);
#pragma unroll
  for (int j = 0; j < kSl; ++j)
    soff[j] = (uint32_t)(min(n0 + kRpi * (wave + 4 * j) + lane / G, N - 1) - n0) * (uint32_t)W;
  const bool wvec = (W & 3) == 0;
  auto issue_signs = [&](int g) {
    const uint32_t sb = lds0 + D * kQStage + (uint32_t)(g & 1) * kSgBuf;
    const int w0 = 4 * G * g;
    if (wvec) {
      const int wd = min(4 * spc, W - 4 - w0);
#pragma unroll
      for (int j = 0; j < kSl; ++j)
        if (kRpi * (wave + 4 * j + 1) <= kRowsS || kRpi * (wave + 4 * j) + lane / G < kRowsS)
          dma16(4u * (soff[j] + (uint32_t)wd), wb + w0, sb + 1024u * (wave + 4 * j));
    } else {
      // word by word: lane i of a load fetches word slot i % 4G of row i / 4G
      constexpr int kR4 = 64 / (4 * G);
      int nn = n0;
      asm volatile("" : "+s"(nn));  // offsets formed here, not held through the K loop
#pragma unroll
      for (int j = 0; j < (kRowsS / kR4 + 3) / 4; ++j) {
        const int r0 = kR4 * (wave + 4 * j), row = r0 + lane / (4 * G);
        const int wd = min(4 * (((lane >> 2) % G) ^ sswz(row)) + (lane & 3), W - 1 - w0);
        const uint32_t o = (uint32_t)(min(nn + row, N - 1) - nn) * (uint32_t)W + (uint32_t)wd;
        if (r0 < kRowsS) dma4(4u * o, wb + w0, sb + (uint32_t)(kSgRow * r0));
      }
    }
  };
  auto issue = [&](int k, uint32_t slot) {
    if (k % G == 0) issue_signs(k / G);
    const uint32_t sb = lds0 + slot * kQStage + 1024u * wave;
    if (k == ng - 1 && vlast != 7) {  // uniform: pieces past K re-read the last
      uint32_t past = 16u * (uint32_t)max(lc - vlast, 0);
      asm volatile("" : "+v"(past));
#pragma unroll
      for (int i = 0; i < kLq; ++i) dma16(qoff[i] - past, qb + 128 * k, sb + 4096u * i);
    } else {
#pragma unroll
      for (int i = 0; i < kLq; ++i) dma16(qoff[i], qb + 128 * k, sb + 4096u * i);
    }
  };

  v4i acc[RT][TT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < TT; ++i) acc[t][i] = zero4();
  v4i accx[TT / 4 > 0 ? TT / 4 : 1];  // the shared tile's token tiles TT/4 * wave ..
#pragma unroll
  for (int i = 0; i < TT / 4; ++i) accx[i] = zero4();

  for (int p = 0; p < D - 1; ++p)
    if (p < ng) issue(p, p);
  // the block's scalars, read after the K loop
  for (int x = threadIdx.x; x < kRowsS; x += 256) {
    const int n = min(n0 + x, N - 1);
    al_lds[x] = a.alpha[n];
    be_lds[x] = r > 0 ? a.beta[n] : 0.f;
  }
  for (int x = threadIdx.x; x < kRowsQ; x += 256) {
    const int m = min(m0 + x, M - 1);
    s_lds[x] = a.s[m];
    sq_lds[x] = a.sumq[m];
  }
  const int8_t* qrd = lds + (16 * TT * wt + rho) * 128;
  const int8_t* srd = lds + D * kQStage + (16 * RT * wr + rho) * kSgRow + 4 * kg;
  // Wide form: a wave in its K loop goes before one that writes its tile out, so
  // the two blocks of a CU drift apart and one multiplies while the other stores
  // (us at r = 64, without / with: 2048 x 2048 x 8512 46.3 / 44.7, 2048 x 4096 x 8512
  // 71.5 / 69.3, 7001 x 2560 x 10576 203.9 / 202.7).  The 128 x 128 form, whose grids
  // here fill two rounds and more, loses by it: 2048 x 4096 x 2048 35.0 / 35.5.
  if constexpr (kX) __builtin_amdgcn_s_setprio(1);
  int slot = 0;
  for (int k = 0; k < ng; ++k) {
    // own loads of stage k landed (sign loads among the younger ones only
    // make the wait longer), own LDS reads of stage k - 1 done
    wait_lds();
    wait_steps<kLq>(min(D - 2, ng - 1 - k));
    asm volatile("s_barrier" ::: "memory");
    if (k + D - 1 < ng) issue(k + D - 1, slot == 0 ? D - 1 : slot - 1);
    const int8_t* st = qrd + slot * kQStage;
    const int8_t* sg_ = srd + ((k / G) & 1) * kSgBuf + 16 * ((k % G) ^ sswz(rho));
    slot = slot == D - 1 ? 0 : slot + 1;
    uint32_t w[RT], wx = 0;
#pragma unroll
    for (int t = 0; t < RT; ++t) w[t] = *reinterpret_cast<const uint32_t*>(sg_ + 16 * kSgRow * t);
    if (extra) wx = *reinterpret_cast<const uint32_t*>(sg_ + 16 * kSgRow * (RT * WR - RT * wr));
    if (k == ng - 1 && 2 * kg > vlast) {  // words past K (K % 32 == 0: whole words)
#pragma unroll
      for (int t = 0; t < RT; ++t) w[t] = 0u;
      wx = 0u;
    }
    // 2*TT groups of RT MFMAs (one token tile of one half of the stage each,
    // kept apart by sched_barrier); every group reads the operand of the
    // third group after it and expands its share of the second half's signs
    const int po[2] = {16 * ((2 * kg) ^ swz8(rho)), 16 * ((2 * kg + 1) ^ swz8(rho))};
    auto read_x = [&](int j) { return *reinterpret_cast<const v4i*>(st + 2048 * (j % TT) + po[j / TT]); };
    v4i x[4], sg[2][RT];
#pragma unroll
    for (int j = 0; j < 3; ++j) x[j] = read_x(j);
#pragma unroll
    for (int t = 0; t < RT; ++t) sg[0][t] = expand16_at(w[t], 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 2 * TT; ++j) {
      if (j + 3 < 2 * TT) x[(j + 3) & 3] = read_x(j + 3);
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[t][j % TT] = mfma(sg[j / TT][t], x[j & 3], acc[t][j % TT]);
      if (j < TT) {
#pragma unroll
        for (int u = 4 * RT * j / TT; u < 4 * RT * (j + 1) / TT; ++u) sg[1][u >> 2][u & 3] = expand4(w[u >> 2], 16 + 4 * (u & 3));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (extra) {  // uniform; its Q operands are read apart (a wave-indexed pick would be branches)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const v4i sx = expand16_at(wx, 16 * v);
#pragma unroll
        for (int i = 0; i < TT / 4; ++i)
          accx[i] = mfma(sx, *reinterpret_cast<const v4i*>(st + 2048 * (TT / 4 * wave + i) + po[v]), accx[i]);
      }
    }
  }

  if constexpr (kX) __builtin_amdgcn_s_setprio(0);

  // ---- epilogue: the block's LoRA operands into the ring's LDS, once for all
  // waves (loads between the stores of y would each wait for their own
  // round trip)
  __syncthreads();
  const bool lora = r > 0;
  const int64_t bpitch = a.l4 ? r / 2 : r;
  const bool ba = (r % 16) == 0;
  auto load_b = [&](int n, int j) -> v4i {
    const int8_t* row = a.B + (int64_t)min(n, N - 1) * bpitch;
    return a.l4 ? load16_row_guarded<true>(row, j, r, ba) : load16_row_guarded<false>(row, j, r, ba);
  };
  if (!BIG && lora) {
    v4i lv[kRowsQ / 16], bv[(kRowsS + 63) / 64];
#pragma unroll
    for (int u = 0; u < kRowsQ / 16; ++u) {
      const int idx = threadIdx.x + 256 * u;  // (limb, row, 16-byte piece)
      const int l = idx / (4 * kRowsQ), ml = (idx >> 2) % kRowsQ, c = idx & 3;
      lv[u] = load16(a.limbs + ((int64_t)l * M + min(m0 + ml, M - 1)) * a.rp + 16 * c);
    }
#pragma unroll
    for (int u = 0; u < (kRowsS + 63) / 64; ++u) {
      const int idx = threadIdx.x + 256 * u;
      bv[u] = load_b(n0 + (idx >> 2), 16 * (idx & 3));
    }
#pragma unroll
    for (int u = 0; u < kRowsQ / 16; ++u) {
      const int idx = threadIdx.x + 256 * u;
      const int l = idx / (4 * kRowsQ), ml = (idx >> 2) % kRowsQ, c = idx & 3;
      *reinterpret_cast<v4i*>(lds + (l * kRowsQ + ml) * 64 + 16 * (c ^ ((ml >> 1) & 3))) = lv[u];
    }
#pragma unroll
    for (int u = 0; u < (kRowsS + 63) / 64; ++u) {
      const int idx = threadIdx.x + 256 * u;
      if (kRowsS % 64 == 0 || idx < 4 * kRowsS)
      *reinterpret_cast<v4i*>(lds + kLimb + (idx >> 2) * 64 + 16 * ((idx & 3) ^ ((idx >> 3) & 3))) = bv[u];
    }
  }
  if (BIG && lora) {  // B alone, all ranks: 256 bytes a row, piece p at slot p ^ (row & 15)
    for (int idx = threadIdx.x; idx < kRowsS * (a.rp >> 4); idx += 256) {
      const int row = idx / (a.rp >> 4), pc = idx - row * (a.rp >> 4);
      *reinterpret_cast<v4i*>(lds + 256 * row + 16 * (pc ^ (row & 15))) = load_b(n0 + row, 16 * pc);
    }
  }
  __syncthreads();
  const int nl = 16 * RT * wr, ml = 16 * TT * wt;  // this wave's first row, token of the block
  if (m0 + ml >= M) return;
  const int l_off = rho * 64 + 16 * (kg ^ ((rho >> 1) & 3));
  const bool fast = (N & 3) == 0 && !a.acc_s_out && !a.acc_b_out && n0 + 16 * cnt <= N && lora && a.y;
  v4i bop[RT];
  if (!BIG && lora) {
#pragma unroll
    for (int t = 0; t < RT; ++t) bop[t] = *reinterpret_cast<const v4i*>(lds + kLimb + (nl + 16 * t) * 64 + l_off);
  }
  // acc_b of one 16 x 16 tile at ranks up to 64 (small: it fits 32 bits, elo
  // alone)
  auto up = [&](const v4i& bo, const v4i (&lm)[4], bool small, v4i& ehi, v4i& elo) {
    ehi = elo = zero4();
    if (!lora) return;
    if (small) {
      elo = mfma(bo, lm[2], elo);
      elo = mfma(bo, lm[1], elo << 8);
      elo = mfma(bo, lm[0], elo << 8);
    } else {
      ehi = mfma(bo, lm[3], ehi);
      elo = mfma(bo, lm[1], elo);
      ehi = mfma(bo, lm[2], ehi << 8);
      elo = mfma(bo, lm[0], elo << 8);
    }
  };
  // outputs of one 16 x 16 tile: row offset rl of the run, token offset tl of
  // the block
  auto tile_out = [&](auto is_fast, const v4i& c, const v4i& ehi, const v4i& elo, bool small, int rl, int tl) {
    constexpr bool kFast = decltype(is_fast)::value;
    const int m = m0 + tl + rho, n = n0 + rl + 4 * kg;
    const float sm = s_lds[tl + rho];
    const int nq = -sq_lds[tl + rho];
    const float4 al4 = *reinterpret_cast<const float4*>(&al_lds[rl + 4 * kg]);
    const float4 be4 = *reinterpret_cast<const float4*>(&be_lds[rl + 4 * kg]);
    const float alv[4] = {al4.x, al4.y, al4.z, al4.w}, bev[4] = {be4.x, be4.y, be4.z, be4.w};
    float yv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t as = (c[v] << 1) + nq;
      if (kFast && small)
        yv[v] = sm * (alv[v] * (float)as + bev[v] * (float)elo[v]);  // the epilogue's operations, acc_b in 32 bits
      else
        yv[v] = dfssm_dev::epilogue(sm, alv[v], bev[v], as, ehi[v], elo[v], kFast || lora);
      if (!kFast && m < M && n + v < N) {
        if (a.acc_s_out) a.acc_s_out[(int64_t)m * N + n + v] = as;
        if (a.acc_b_out) a.acc_b_out[(int64_t)m * N + n + v] = lora ? (int64_t)elo[v] + ((int64_t)ehi[v] << 16) : 0;
      }
    }
    if constexpr (kFast) {
      *reinterpret_cast<float4*>(a.y + (int64_t)m * N + n) = make_float4(yv[0], yv[1], yv[2], yv[3]);
    } else if (m < M && a.y) {
      float* dst = a.y + (int64_t)m * N + n;
      if ((N & 3) == 0 && n + 3 < N) {
        *reinterpret_cast<float4*>(dst) = make_float4(yv[0], yv[1], yv[2], yv[3]);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (n + v < N) dst[v] = yv[v];
      }
    }
  };
  auto load_lm = [&](int tl, v4i (&lm)[4]) {
    if (!BIG && lora) {
#pragma unroll
      for (int l = 0; l < 4; ++l) lm[l] = *reinterpret_cast<const v4i*>(lds + (l * kRowsQ + tl) * 64 + l_off);
    }
  };
  const int ntw = min(max(cnt - RT * wr, 0), RT);  // this wave's row tiles
  // whole token tiles without accumulator outputs go unchecked; the checked
  // form takes the others (all of them, or the block's partial token tile)
  auto finish = [&](auto is_fast) {
    constexpr bool kFast = decltype(is_fast)::value;
    auto mine = [&](int tl) {
      const bool whole = m0 + tl + 16 <= M;
      return kFast ? whole : m0 + tl < M && !(fast && whole);
    };
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const int tl = ml + 16 * i;
      if (!mine(tl)) continue;  // uniform
      if constexpr (BIG) {
        // the limbs of one 64-rank chunk at a time, the next one on its way
        v4i ehi[RT], elo[RT], nx[4];
#pragma unroll
        for (int t = 0; t < RT; ++t) ehi[t] = elo[t] = zero4();
        const int8_t* lp = a.limbs + (int64_t)min(m0 + tl + rho, M - 1) * a.rp + 16 * kg;
        auto fetch = [&](int j0) {
#pragma unroll
          for (int l = 0; l < 4; ++l) nx[l] = load16(lp + (int64_t)l * M * a.rp + j0);
        };
        if (lora) fetch(0);
        for (int j0 = 0; lora && j0 < a.rp; j0 += 64) {
          v4i lm[4];
#pragma unroll
          for (int l = 0; l < 4; ++l) lm[l] = nx[l];
          if (j0 + 64 < a.rp) fetch(j0 + 64);
#pragma unroll
          for (int t = 0; t < RT; ++t) {
            const v4i bo = *reinterpret_cast<const v4i*>(lds + 256 * (nl + 16 * t + rho) + 16 * (((j0 >> 4) + kg) ^ rho));
            ehi[t] = mfma(bo, lm[2], ehi[t] + (mfma(bo, lm[3], zero4()) << 8));
            elo[t] = mfma(bo, lm[0], elo[t] + (mfma(bo, lm[1], zero4()) << 8));
          }
        }
#pragma unroll
        for (int t = 0; t < RT; ++t)
          if (t < ntw) tile_out(is_fast, acc[t][i], ehi[t], elo[t], false, nl + 16 * t, tl);
        continue;
      }
      v4i lm[4], ehi, elo;
      load_lm(tl, lm);
      // sum_j |acc_a| < 2^24 for every token of the tile (no limb 3, sum of
      // (|limb 2| + 1) below 256): |acc_b| < 128 * 2^24, so 32 bits hold it
      const bool small = kFast && !BIG && __all(fits32(lm));
      if (kFast && small && ntw == RT) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          up(bop[t], lm, true, ehi, elo);
          tile_out(is_fast, acc[t][i], ehi, elo, true, nl + 16 * t, tl);
        }
      } else {
#pragma unroll
        for (int t = 0; t < RT; ++t)
          if (t < ntw) {
            up(bop[t], lm, false, ehi, elo);
            tile_out(is_fast, acc[t][i], ehi, elo, false, nl + 16 * t, tl);
          }
      }
    }
    if (extra) {
      constexpr int kXr = 16 * RT * WR;
      v4i bx = zero4();
      if (!BIG && lora) bx = *reinterpret_cast<const v4i*>(lds + kLimb + kXr * 64 + l_off);
#pragma unroll
      for (int i = 0; i < TT / 4; ++i) {
        const int tl = 16 * (TT / 4 * wave + i);
        if (!mine(tl)) continue;
        v4i lm[4], ehi, elo;
        load_lm(tl, lm);
        up(bx, lm, false, ehi, elo);
        tile_out(is_fast, accx[i], ehi, elo, false, kXr, tl);
      }
    }
  };
  if (fast) finish(std::true_type{});
  if (!fast || m0 + kRowsQ > M) finish(std::false_type{});
}

// Row blocks per token block of the wide form: runs of 16 row tiles, or of up
// to 17 (the last shared by the waves) where that saves a round of the chip's
// block slots (two per CU): 2048 tokens x 8512 rows then are 512 blocks.
int64_t wide_runs(int64_t tb, int64_t nt16) {
  const int64_t slots = 2 * dfssm::device_cu_count();
  const int64_t n16 = dfssm::ceil_div(nt16, 16), n17 = dfssm::ceil_div(nt16, 17);
  return dfssm::ceil_div(tb * n17, slots) < dfssm::ceil_div(tb * n16, slots) ? n17 : n16;
}

template <int TT, int RT, int WT, int D, int G, bool BIG = false>
hipError_t launch_tile(TileArgs a, hipStream_t st) {
  static_assert(WT != 1 || RT == 4, "wide_runs");
  a.ntb = (int)dfssm::ceil_div(a.M, 16 * TT * WT);
  const int nt16 = (int)dfssm::ceil_div(a.N, 16);
  a.nrb = WT == 1 ? (int)wide_runs(a.ntb, nt16) : (int)dfssm::ceil_div(nt16, RT * (4 / WT));
  a.run = nt16 / a.nrb;
  a.runx = nt16 % a.nrb;
  mfma_tile<TT, RT, WT, D, G, BIG><<<dim3((unsigned)(a.ntb * a.nrb)), dim3(256), 0, st>>>(a);
  return hipGetLastError();
}

// The two tile forms: 128 tokens x 256 rows (runs of up to 17 row tiles; a wave
// holds 128 x 64, each expanded sign operand feeds 8 MFMAs) and 128 x 128
// (a wave 64 x 64: twice the workgroups).  Modelled cost (us, both launches) with x =
// workgroups per CU, of which two fit at once, E = ceil(x / 2) - 1 and k = K / 1024:
//   c0 + c1 k + (c2 + c3 k) x + (c4 + c5 k) E, and c6 x where N % 16 != 0
// (a token's outputs then start off the 64-byte segments of a tile's stores: at x = 1,
// K = 2048 about 4 us of the wide form's 40); above rank 64, which takes the 128 x 128
// form, with g = further chunks of 64 ranks, coefficients of its own and
// g (c7 + c8 M / 1000) more.  Fitted on MI355X as the split-K tile kernel's cost is.
struct TilePlan {
  bool wide;
  double us;
};
TilePlan plan_tile(int64_t M, int64_t K, int64_t N, int64_t r) {
  static constexpr double kC[3][9] = {{12.535, 4.082, 3.424, 1.935, 0.853, 3.064, 0.948, 0, 0},
                                      {21.663, 4.499, 1.612, 3.777, 6.643, 3.516, 3.689, 0, 0},
                                      {8.939, 5.429, 4.744, 1.360, 3.143, 4.294, 2.012, 2.764, 1.617}};
  const int cus = dfssm::device_cu_count();
  const int64_t tb = dfssm::ceil_div(M, 128);
  const double k = (double)K / 1024.0, m = (double)M / 1000.0;
  const double g = (double)std::max<int64_t>(0, dfssm::ceil_div(r, 64) - 1);
  TilePlan p{false, 0.0};
  for (int f = 0; f < (r > 64 ? 1 : 2); ++f) {
    const int64_t rb = f ? wide_runs(tb, dfssm::ceil_div(N, 16)) : dfssm::ceil_div(N, 128);
    const double x = (double)(tb * rb) / cus, E = std::max(0.0, std::ceil(x / 2) - 1.0);
    const double* c = kC[r > 64 ? 2 : f];
    const double us = c[0] + c[1] * k + (c[2] + c[3] * k) * x + (c[4] + c[5] * k) * E + (N % 16 ? c[6] * x : 0.0) + g * (c[7] + c[8] * m);
    if (f == 0 || us < p.us) p = {f == 1, us};
  }
  // test switch prefill_kernel: 4 the 128 x 128 form, 8 the wide one
  const int forced = dfssm::test_switch(DFSSM_TEST_PREFILL_KERNEL);
  if (forced == 4) p.wide = false;
  if (forced == 8) p.wide = true;
  return p;
}

// 16 ranks per workgroup up to rank 16 (the whole rank), 64 above, or 32 while
// workgroups of 64 would leave half the CUs without one: us at r = 64 with 64 /
// 32 ranks, 1000 x 2048 4.2 / 2.7, 1536 x 1024 4.2 / 3.0, 3000 x 4096 7.6 / 9.3,
// 7001 x 2560 11.9 / 14.8.
template <bool L4>
hipError_t launch_down(const DownArgs& a, hipStream_t st) {
  const unsigned mb = (unsigned)dfssm::ceil_div(a.M, 16);
  if (a.r <= 16)
    lora_down<1, 8, L4><<<dim3(mb), dim3(512), 0, st>>>(a);
  else if (2 * (int64_t)mb * (a.rp / 64) <= dfssm::device_cu_count())
    lora_down<2, 8, L4><<<dim3(mb, (unsigned)(a.rp / 32)), dim3(512), 0, st>>>(a);
  else
    lora_down<4, 8, L4><<<dim3(mb, (unsigned)(a.rp / 64)), dim3(512), 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace

namespace dfssm {

double tile_cost_us(int64_t M, int64_t K, int64_t N, int64_t r) { return plan_tile(M, K, N, r).us; }

int device_cu_count() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int v = cache[dev].load(std::memory_order_relaxed);
  if (v <= 0) {
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cache[dev].store(v, std::memory_order_relaxed);
  }
  return v;
}

hipError_t launch_tile_linear(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N,
                              int64_t r, const uint32_t* w_bits, const float* alpha,
                              const int8_t* A, const int8_t* B, bool l4, const float* beta, float* y,
                              int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                              const LinearWorkspace& ws, hipStream_t st) {
  if (M == 0 || N == 0) return hipSuccess;
  const int rp = (int)rank_padded(r);
  DownArgs da{q, (int)M, (int)K, (int)r, rp, A, ws.limbs, ws.sumq, r > 0 ? acc_a_out : nullptr};
  hipError_t e = l4 ? launch_down<true>(da, st) : launch_down<false>(da, st);
  if (e != hipSuccess) return e;
  TileArgs ta{q, s, (int)M, (int)K, (int)N, (int)r, rp, w_bits, alpha, ws.limbs, B, beta, ws.sumq, y, acc_s, acc_b,
              l4 ? 1 : 0, 0, 0};
  if (rp > 64) return launch_tile<4, 4, 2, 3, 4, true>(ta, st);
  return plan_tile(M, K, N, r).wide ? launch_tile<8, 4, 1, 3, 2>(ta, st) : launch_tile<4, 4, 2, 3, 4>(ta, st);
}

}  // namespace dfssm
