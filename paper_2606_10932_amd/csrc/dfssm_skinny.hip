// dfssm_skinny.hip -- scaffold + LoRA linear for one or two tokens on the gfx950
// int8 matrix cores (v_mfma_i32_16x16x64_i8), at the sizes where it is faster than
// the split-K tile kernel (the choice and both sides' figures stand at the
// dispatch).
//
// The product is a contraction the matrix cores finish in a fraction of the time
// the sign bits take to stream.  Here a workgroup owns 16 output rows and every
// token, and its waves split K:
//  * each lane loads, before any arithmetic, 128 consecutive columns of its
//    row's sign bits (one 16-byte load) and the same columns of its token's
//    codes, then runs 8 MFMAs.  Inside one MFMA the order of the 64 contracted columns is free as
//    long as both operands use the same order, so lane (row, kg) feeds
//    columns kc(kg) + 16v .. +15 at step v and token lane (m, kg) feeds the
//    same columns;
//  * the signs are expanded to {0,1} bytes in registers (nibble n -> bytes
//    (n * 0x00204081) & 0x01010101), so the MFMA gives D = sum_{bit=1} Q and
//    acc_s = 2*D - sum_k Q;
//  * the waves' partial tiles are summed in LDS; one wave then does the
//    LoRA up-projection (four limb MFMAs: E_hi = 256*(B.L3) + B.L2,
//    E_lo = 256*(B.L1) + B.L0, exact int64 acc_b = E_lo + 65536*E_hi) and the
//    fp32 epilogue; its row operands were loaded at the start.
// One launch: the first nb_lora workgroups compute the LoRA down-projection
// acc_a = Q A^T (one wave per rank) and sum_k Q, and publish
// them as 64-bit words {tag, value} (value: acc_a's 4 signed base-256 limbs
// as bytes, or sum Q) with agent-scope stores; a word is valid once its tag
// is the call's.  A call enqueued directly takes its tag from a host counter
// (bit 31 set).  A call captured into a graph would replay with a frozen
// argument, so there the tag is the call's epoch + 1 (below 2^31), kept on
// the device so that every replay moves it on.  Every reader and writer of the words (each publishing LoRA
// wave, each output workgroup) is a member of the call with an index i, and
// arrives once, at its start, with a 64-bit fetch-add on epoch word i % 64
// of the workspace ({epoch, arrivals}, one per 128-byte line, so that
// arrivals meet at 64 addresses and not one), which hands it the epoch;
// the last member to arrive on a word stores {epoch + 1, 0} there, and
// member 0 stores it into every word no member of this call uses.  All 64
// words start at {0, 0} and each call moves every one of them on by one,
// so all of one call agree on its epoch, the next call (stream-ordered
// after it) starts from the next one, and a word left by an earlier call
// never validates.
// The other workgroups read the words they need after their scaffold
// product.  The wait is bounded:
// a lane whose words have not arrived after `spin` polls computes the values
// itself from A and Q (the integers are the same either way), so no
// workgroup depends on another being scheduled.
#include <algorithm>
#include <atomic>

#include "dfssm_int4.hpp"
#include "dfssm_linear.hpp"
#include "dfssm_persist.hpp"

namespace {

using namespace dfssm_lin;

constexpr int kMaxWaves = 8;

struct SkinnyArgs {
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
  int64_t* acc_b_out;
  int32_t* acc_a;  // [M][r], written by the LoRA workgroups (and by fallback lanes)
  uint64_t* xw;    // [xcopies][xstride]: [M][rp] limb words, then [M] sum-Q words
  int64_t xstride; // M * rp + M, rounded up to 32 words
  int xcopies;     // 8: one copy per XCD (every output workgroup reads the same
                   // words, so the copies spread its polls) at r > 32 when they
                   // fit; else 1
  uint64_t* epoch; // kEpochGroups words {epoch:32, arrivals:32}, kEpochStride apart;
                   // NULL: the call's tag is host_tag
  uint32_t host_tag;
  int arrivals;    // members per call: publishing LoRA waves, then output workgroups
  int lora_members;  // publishing LoRA waves (members 0 .. lora_members - 1)
  int nb_lora;     // LoRA workgroups at the front of the grid
  int spin;        // polls of a missing word before computing it locally
};


// whole-wave sum, the total in every lane (DPP inside 16-lane rows, then
// gfx950's permlane swaps across rows and halves)
__device__ __forceinline__ int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
  auto p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  v = (int)(p[0] + p[1]);
  p = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return (int)(p[0] + p[1]);
}

// LoRA workgroup: wave w takes rank b*nw + w for every token; the wave of rank 0
// also sums Q.  Every 16-byte load of a 4 KB column batch
// is issued before the first v_dot4.
constexpr int kPrepTokens = 2;
static_assert(kPrepTokens == dfssm::kSkinnyMaxTokens, "one LoRA wave per rank");
constexpr int kPrepBatch = 4;
template <bool L4>
__device__ void lora_block(const SkinnyArgs& a) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int M = a.M, K = a.K, r = a.r, rp = a.rp;
  const int j = (int)blockIdx.x * nw + wave;
  if (j >= rp) return;
  // a publishing wave arrives once, at its start (device-epoch calls); the
  // epoch is needed only when it publishes
  uint64_t ep_old = 0;
  if (a.epoch && lane == 0) ep_old = dfssm_dev::arrive(a.epoch, j);
  const int mt = min(kPrepTokens, M);
  const bool jr = j < r, qsum = j == 0;
  int acc[kPrepTokens], qs[kPrepTokens];
#pragma unroll
  for (int m = 0; m < kPrepTokens; ++m) acc[m] = qs[m] = 0;
  if (jr || qsum) {
    const int8_t* arow = a.A + (int64_t)(jr ? j : 0) * (L4 ? K / 2 : K);
    for (int kb = 0; kb < K; kb += 1024 * kPrepBatch) {
      // int4: the packed bytes are kept as loaded and expanded at their use,
      // so no expansion waits on a load before the batch's last load issues
      uint4 av[kPrepBatch], x[kPrepTokens][kPrepBatch];
      uint2 araw[kPrepBatch];
#pragma unroll
      for (int u = 0; u < kPrepBatch; ++u) {
        const int k = kb + 1024 * u + 16 * lane;
        const bool ok = k < K;  // K % 32 == 0: a 16-byte chunk is wholly in or out
        if constexpr (L4)
          araw[u] = (jr && ok) ? *reinterpret_cast<const uint2*>(arow + k / 2) : make_uint2(0, 0);
        else
          av[u] = (jr && ok) ? load_row16<false>(arow, k) : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int m = 0; m < kPrepTokens; ++m)
          x[m][u] = (ok && m < mt) ? *reinterpret_cast<const uint4*>(a.q + (int64_t)m * K + k)
                                   : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < kPrepBatch; ++u) {
        if constexpr (L4) av[u] = expand_i4(araw[u]);
#pragma unroll
        for (int m = 0; m < kPrepTokens; ++m) {
          acc[m] = sdot4(av[u].x, x[m][u].x, acc[m]);
          acc[m] = sdot4(av[u].y, x[m][u].y, acc[m]);
          acc[m] = sdot4(av[u].z, x[m][u].z, acc[m]);
          acc[m] = sdot4(av[u].w, x[m][u].w, acc[m]);
          if (qsum) {
            qs[m] = sdot4(0x01010101u, x[m][u].x, qs[m]);
            qs[m] = sdot4(0x01010101u, x[m][u].y, qs[m]);
            qs[m] = sdot4(0x01010101u, x[m][u].z, qs[m]);
            qs[m] = sdot4(0x01010101u, x[m][u].w, qs[m]);
          }
        }
      }
    }
  }
  int mine = 0, mine_q = 0;
#pragma unroll
  for (int m = 0; m < kPrepTokens; ++m) {
    if (m < mt) {  // uniform
      const int t = wave_sum(acc[m]);
      mine = lane == m ? t : mine;
      if (qsum) {
        const int tq = wave_sum(qs[m]);
        mine_q = lane == m ? tq : mine_q;
      }
    }
  }
  const uint64_t old = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ep_old >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)ep_old);
  const uint32_t tag = a.epoch ? dfssm_dev::epoch_tag(old) : a.host_tag;
  if (a.xcopies == 1) {
    if (lane < mt) {
      if (jr) a.acc_a[(int64_t)lane * r + j] = mine;
      word_store(a.xw + (int64_t)lane * rp + j, tag, pack_limbs(mine));  // zero limbs for ranks in [r, rp)
      if (qsum) word_store(a.xw + (int64_t)M * rp + lane, tag, (uint32_t)mine_q);
    }
  } else {
    // lane c*mt + i stores token i's words into copy c (lane i holds
    // them).  Every instruction here delays the words: this branch's
    // shuffles cost the single copy ~0.3 us a call at r = 16, and a lane
    // modulo in their place cost more.
    const int src = lane % mt;
    const int vm = __shfl(mine, src, 64), vq = __shfl(mine_q, src, 64);
    if (lane < mt && jr) a.acc_a[(int64_t)lane * r + j] = mine;
    if (lane < mt * a.xcopies) {
      const int cpy = lane / mt, m = lane - cpy * mt;
      uint64_t* xc = a.xw + (int64_t)cpy * a.xstride;
      word_store(xc + (int64_t)m * rp + j, tag, pack_limbs(vm));  // zero limbs for ranks in [r, rp)
      if (qsum) word_store(xc + (int64_t)M * rp + m, tag, (uint32_t)vq);
    }
  }
  if (a.epoch && lane == 0) dfssm_dev::advance_if_last(a.epoch, j, old, a.arrivals);
}

// The limbs of acc_a[m][j0 + 16kg .. +15] as 4 limb operands (byte e of limb
// t = limb t of rank j0 + 16kg + e) and, when sq is given, sum Q of token m, for
// the lane (rho, kg) (m = min(rho, M - 1)): from the LoRA workgroups' words, or
// computed here once `spin` polls have passed.
//   - CP: the words come in one copy per XCD, and this wave polls its XCD's
//     copy token by token.  Lane L reads rank j0 + L of each token (one 512-byte
//     load per token), lanes below M read the sum-Q words, and the words reach
//     their lanes through the wave's LDS tile wx [kPrepTokens][kWxPitch] (sq:
//     wq [kPrepTokens]).
//   - otherwise each lane polls its own 16 words and keeps them once in.
constexpr int kWxPitch = 68;  // words per token row of wx (16 bytes of skew)

// Polls of all tokens in the copy xc: lane L reads rank j0 + L of each, lanes
// below M the sum-Q words (want_sq).  On success the words are in wx rows 0 ..
// M-1 and wq[0 .. M-1]; false once `spin` polls have passed without all of them.
__device__ __forceinline__ bool poll_tokens(const SkinnyArgs& a, uint32_t tag, const uint64_t* xc, int j0,
                                            bool want_sq, uint32_t* wx, int* wq) {
  const int lane = threadIdx.x & 63;
  const int rp = a.rp, M = a.M;
  const uint64_t* wp = xc + j0 + lane;
  const uint64_t* sp = xc + (int64_t)M * rp + min(lane, M - 1);
  for (int it = 0;; ++it) {
    uint64_t w[kPrepTokens], wqv = 0;
#pragma unroll
    for (int i = 0; i < kPrepTokens; ++i)
      if (i < M) w[i] = word_load(wp + (int64_t)i * rp);  // M is uniform
    if (want_sq) wqv = word_load(sp);
    bool ok = !want_sq || (uint32_t)(wqv >> 32) == tag;
#pragma unroll
    for (int i = 0; i < kPrepTokens; ++i)
      if (i < M) ok = ok && (uint32_t)(w[i] >> 32) == tag;
    if (__all(ok)) {
#pragma unroll
      for (int i = 0; i < kPrepTokens; ++i)
        if (i < M) wx[i * kWxPitch + lane] = (uint32_t)w[i];
      if (want_sq && lane < M) wq[lane] = (int)(uint32_t)wqv;
      return true;
    }
    if (it >= a.spin) return false;
    __builtin_amdgcn_s_sleep(2);
  }
}

template <bool L4, bool CP>
__device__ __forceinline__ void fetch_lora(const SkinnyArgs& a, uint32_t tag, int j0, int rho, int kg, uint32_t* wx,
                                           int* wq, v4i (&lm)[4], int* sq, bool store_acc) {
  const int M = a.M, rp = a.rp;
  const int m = min(rho, M - 1);  // tokens past M repeat the last
  uint32_t val[16], vq = 0;
  bool have = false;
  if constexpr (CP) {
    have = poll_tokens(a, tag, a.xw + (int64_t)dfssm_px::xcc_id() * a.xstride, j0, sq != nullptr, wx, wq);
    if (have) {
      // the LDS writes above and these reads are the same wave's, in order
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint4 u = *reinterpret_cast<const uint4*>(wx + m * kWxPitch + 16 * kg + 4 * d);
        val[4 * d] = u.x; val[4 * d + 1] = u.y; val[4 * d + 2] = u.z; val[4 * d + 3] = u.w;
      }
      if (sq) vq = (uint32_t)wq[m];
      __builtin_amdgcn_wave_barrier();  // wx is written again by the next chunk's call
    }
  } else {
    const uint64_t* wp = a.xw + (int64_t)m * rp + j0 + 16 * kg;
    const uint64_t* sp = a.xw + (int64_t)M * rp + m;
    for (int it = 0;; ++it) {
      if (!have) {
        uint64_t w[16], wqv = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = word_load(wp + e);
        if (sq) wqv = word_load(sp);
        bool ok = !sq || (uint32_t)(wqv >> 32) == tag;
#pragma unroll
        for (int e = 0; e < 16; ++e) ok = ok && (uint32_t)(w[e] >> 32) == tag;
        if (ok) {
#pragma unroll
          for (int e = 0; e < 16; ++e) val[e] = (uint32_t)w[e];
          vq = (uint32_t)wqv;
          have = true;
        }
      }
      if (__all(have) || it >= a.spin) break;
      __builtin_amdgcn_s_sleep(2);
    }
  }
  if (!have) {
    // the LoRA workgroups' words did not arrive: compute them here
#pragma unroll 1
    for (int e = 0; e < 16; ++e) {
      const int j = j0 + 16 * kg + e;
      const int v = j < a.r ? lane_dot<L4>(a.A, a.q, a.K, j, m) : 0;
      val[e] = pack_limbs(v);
      if (store_acc && j < a.r) a.acc_a[(int64_t)m * a.r + j] = v;
    }
    if (sq) vq = (uint32_t)lane_dot<L4>(a.A, a.q, a.K, -1, m);
  }
  limb_operands(val, lm);
  if (sq) *sq = (int)vq;
}

// Block: 16 output rows, nw = blockDim.x / 64 waves, wave w takes iterations w,
// w + nw, ... of 128 columns per lane group, 512 in all.  CP: the LoRA words come
// in one copy per XCD (a.xcopies == 8).  The two ways to poll are separate
// instantiations: in one kernel their union of registers cost a wave per SIMD.
constexpr int kSteps = 8;           // MFMAs per iteration
constexpr int kCols = 64 * kSteps;  // columns per wave iteration
constexpr int kSignWords = kSteps / 2;

template <bool L4, bool CP>
__global__ __launch_bounds__(64 * kMaxWaves) void mfma_skinny(SkinnyArgs a) {
  __shared__ v4i red[kMaxWaves][64];
  __shared__ __align__(16) uint32_t wx[CP ? kPrepTokens * kWxPitch : 4];
  __shared__ int wq[CP ? kPrepTokens : 1];
  __shared__ uint32_t tag_lds;
  if ((int)blockIdx.x < a.nb_lora) {
    lora_block<L4>(a);
    return;
  }
  // an output workgroup arrives once, at its start (device-epoch calls); the
  // epoch is needed only after the scaffold product
  const int member = a.lora_members + ((int)blockIdx.x - a.nb_lora);
  uint64_t ep_old = 0;
  if (a.epoch && threadIdx.x == 0) ep_old = dfssm_dev::arrive(a.epoch, member);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int rho = lane & 15, kg = lane >> 4;
  const int M = a.M, K = a.K, N = a.N, r = a.r, W = K >> 5;
  const int n0 = 16 * ((int)blockIdx.x - a.nb_lora);
  const int nrow = min(n0 + rho, N - 1);  // sign / B row of this lane (rows past N are never stored)
  const uint32_t* wrow = a.w_bits + (int64_t)nrow * W;
  const int nit = (K + kCols - 1) / kCols;
  const bool wvec = (W % kSignWords) == 0;

  // ---- the row operands of the wave that finishes the tile go out first: B
  //      bytes of ranks 0..63, row scales, token scales
  const bool fin = wave == 0;
  const int mtok = rho;  // token of this lane
  const int mc = min(mtok, M - 1);
  const int nb = n0 + 4 * kg;  // this lane's output rows nb .. nb+3
  const bool ba = (r % 16) == 0;
  const int64_t bpitch = L4 ? r / 2 : r;  // bytes per B row
  // int4: the packed B bytes are held as loaded and expanded after the
  // scaffold loop, so the loop's loads do not wait for them
  v4i bop = zero4();
  uint2 braw = make_uint2(0, 0);
  bool bpacked = false;
  float alv[4] = {0.f, 0.f, 0.f, 0.f}, bev[4] = {0.f, 0.f, 0.f, 0.f};
  float sm = 0.f;
  if (fin) {
    if (r > 0) {
      if (L4 && 16 * kg + 16 <= r && ba) {
        braw = *reinterpret_cast<const uint2*>(a.B + (int64_t)nrow * bpitch + 8 * kg);
        bpacked = true;
      } else {
        bop = load16_row_guarded<L4>(a.B + (int64_t)nrow * bpitch, 16 * kg, r, ba);
      }
    }
    if ((N & 3) == 0 && nb + 3 < N) {
      const float4 al4 = *reinterpret_cast<const float4*>(a.alpha + nb);
      alv[0] = al4.x; alv[1] = al4.y; alv[2] = al4.z; alv[3] = al4.w;
      if (r > 0) {
        const float4 be4 = *reinterpret_cast<const float4*>(a.beta + nb);
        bev[0] = be4.x; bev[1] = be4.y; bev[2] = be4.z; bev[3] = be4.w;
      }
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = min(nb + v, N - 1);
        alv[v] = a.alpha[n];
        bev[v] = r > 0 ? a.beta[n] : 0.f;
      }
    }
    sm = a.s[mc];
  }

  // ---- scaffold: this wave's share of K
  v4i acc = zero4();
  for (int it = wave; it < nit; it += nw) {
    const int kc = it * kCols + kg * 16 * kSteps;  // first column of this lane
    const int wd0 = kc >> 5;
    uint32_t sw[kSignWords];
    if (wvec && wd0 + kSignWords <= W) {
      const uint4 t = *reinterpret_cast<const uint4*>(wrow + wd0);
      sw[0] = t.x; sw[1] = t.y; sw[2] = t.z; sw[3] = t.w;
    } else {
      // signs past K meet zero codes; only the load has to stay in the row
#pragma unroll
      for (int i = 0; i < kSignWords; ++i) sw[i] = wd0 + i < W ? wrow[wd0 + i] : 0u;
    }
    v4i x[kSteps];
    const int8_t* qrow = a.q + (int64_t)min(rho, M - 1) * K;
#pragma unroll
    for (int v = 0; v < kSteps; ++v) {
      const int col = kc + 16 * v;  // K % 32 == 0: 16 columns are wholly in or out
      x[v] = (rho < M && col < K) ? load16(qrow + col) : zero4();
    }
#pragma unroll
    for (int v = 0; v < kSteps; ++v) acc = mfma(expand16_at(sw[v >> 1], 16 * (v & 1)), x[v], acc);
  }

  // ---- sum the waves' partial tiles; wave 0 finishes the tile
  red[wave][lane] = acc;
  if (threadIdx.x == 0) {
    if (a.epoch) {
      tag_lds = dfssm_dev::epoch_tag(ep_old);
      dfssm_dev::advance_if_last(a.epoch, member, ep_old, a.arrivals);
    } else {
      tag_lds = a.host_tag;
    }
  }
  __syncthreads();
  const uint32_t tag = tag_lds;
  if (!fin) return;
  v4i d = red[0][lane];
  for (int w = 1; w < nw; ++w) d += red[w][lane];

  // LoRA limbs of ranks 0..63 and sum Q of this lane's token; the first block
  // also keeps acc_a for the caller if its words had to be computed here
  v4i lm[4];
  int sq = 0;
  const bool keep = (int)blockIdx.x == a.nb_lora && mtok < M;
  fetch_lora<L4, CP>(a, tag, 0, rho, kg, wx, wq, lm, &sq, keep);

  // LoRA up-projection, limbs 3, 2, 1, 0 over the 64-rank chunks
  if (L4 && bpacked) {
    // an opaque zero made after the polls: the expansion cannot be moved in
    // front of them, where it would wait for the B load before the first poll
    uint32_t z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    braw.x ^= z;
    braw.y ^= z;
    const uint4 u = expand_i4(braw);
    bop = v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
  }
  v4i ehi = zero4(), elo = zero4();
  if (r > 0) {
    v4i e3 = mfma(bop, lm[3], zero4()), e2 = mfma(bop, lm[2], zero4());
    v4i e1 = mfma(bop, lm[1], zero4()), e0 = mfma(bop, lm[0], zero4());
    for (int j0 = 64; j0 < a.rp; j0 += 64) {
      const v4i bl = load16_row_guarded<L4>(a.B + (int64_t)nrow * bpitch, j0 + 16 * kg, r, ba);
      v4i lj[4];
      fetch_lora<L4, CP>(a, tag, j0, rho, kg, wx, wq, lj, nullptr, keep);
      e3 = mfma(bl, lj[3], e3);
      e2 = mfma(bl, lj[2], e2);
      e1 = mfma(bl, lj[1], e1);
      e0 = mfma(bl, lj[0], e0);
    }
    ehi = (e3 << 8) + e2;
    elo = (e1 << 8) + e0;
  }

  // lane (rho, kg) holds D[row nb + v][token mtok]
  if (mtok >= M) return;
  float yv[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int32_t as = 2 * d[v] - sq;
    yv[v] = dfssm_dev::epilogue(sm, alv[v], bev[v], as, ehi[v], elo[v], r > 0);
    if (nb + v < N) {
      if (a.acc_s_out) a.acc_s_out[(int64_t)mtok * N + nb + v] = as;
      if (a.acc_b_out) a.acc_b_out[(int64_t)mtok * N + nb + v] = r > 0 ? (int64_t)elo[v] + ((int64_t)ehi[v] << 16) : 0;
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

template <bool L4>
hipError_t skinny_impl(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N, int64_t r,
                       const uint32_t* w_bits, const float* alpha, const int8_t* A, const int8_t* B,
                       const float* beta, float* y, int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                       const dfssm::LinearWorkspace& ws, hipStream_t st) {
  using namespace dfssm;
  if (M == 0 || N == 0) return hipSuccess;
  if (M > kSkinnyMaxTokens) return hipErrorInvalidValue;
  const int rp = (int)rank_padded(r);
  const int nw = (int)std::min<int64_t>(kMaxWaves, ceil_div(K, kCols));
  // Test switch local_lora: no LoRA workgroups, every lane computes its LoRA
  // values itself at once (the path a lane takes when the words never
  // arrive).
  const bool local_only = test_switch(DFSSM_TEST_LOCAL_LORA) == 1;
  const int lora_waves = local_only ? 0 : rp;
  const int nb_lora = (int)ceil_div(lora_waves, nw);
  const int64_t out_blocks = ceil_div(N, 16);
  // the call's tag: under graph capture from the device epoch (a replay
  // moves it on), otherwise from a host counter (no arrivals at all)
  const bool device_epoch = wants_device_epoch(st);
  // One copy of the LoRA words per XCD, each on a 256-byte boundary (no cache line
  // holds words of two copies), when the LoRA down-projection is the longer path
  // (r > 32): every output workgroup then waits on the words, and the copies took
  // 1.2-2.3 us off a call (1.3B projections, r = 64).  At r <= 32 the words are
  // mostly in before the first poll.
  const int64_t xstride = round_up(M * rp + M, 32);
  const int xcopies = r > 32 ? 8 : 1;
  static_assert(8 * (kSkinnyMaxTokens * (kMaxRank + 1) + 32) <= kXwWords, "the copies fit their region");
  const SkinnyArgs a{q, s, (int)M, (int)K, (int)N, (int)r, rp, w_bits, alpha, A, B, beta, y, acc_s, acc_b,
                     ws.acc_a, ws.xw, xstride, xcopies, device_epoch ? ws.epoch : nullptr,
                     device_epoch ? 0u : next_host_tag(), (int)(lora_waves + out_blocks), lora_waves, nb_lora,
                     local_only ? 0 : (1 << 14)};
  const dim3 grid((unsigned)(nb_lora + out_blocks)), block(64 * nw);
  if (xcopies == 1)
    mfma_skinny<L4, false><<<grid, block, 0, st>>>(a);
  else
    mfma_skinny<L4, true><<<grid, block, 0, st>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (acc_a_out && r > 0)
    e = hipMemcpyAsync(acc_a_out, ws.acc_a, (size_t)(M * r) * 4, hipMemcpyDeviceToDevice, st);
  return e;
}

}  // namespace

namespace dfssm {

uint32_t next_host_tag() {
  static std::atomic<uint32_t> seq{0};
  return 0x80000000u | (seq.fetch_add(1, std::memory_order_relaxed) & 0x7fffffffu);
}

bool wants_device_epoch(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
    (void)hipGetLastError();
    cap = hipStreamCaptureStatusActive;
  }
  return cap != hipStreamCaptureStatusNone;
}

hipError_t launch_skinny_linear(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N,
                                int64_t r, const uint32_t* w_bits, const float* alpha,
                                const int8_t* A, const int8_t* B, const float* beta, float* y,
                                int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                                const LinearWorkspace& ws, hipStream_t st) {
  return skinny_impl<false>(q, s, M, K, N, r, w_bits, alpha, A, B, beta, y, acc_s, acc_a_out, acc_b, ws, st);
}

hipError_t launch_skinny_linear_i4(const int8_t* q, const float* s, int64_t M, int64_t K, int64_t N,
                                   int64_t r, const uint32_t* w_bits, const float* alpha,
                                   const uint8_t* A4, const uint8_t* B4, const float* beta, float* y,
                                   int32_t* acc_s, int32_t* acc_a_out, int64_t* acc_b,
                                   const LinearWorkspace& ws, hipStream_t st) {
  return skinny_impl<true>(q, s, M, K, N, r, w_bits, alpha, reinterpret_cast<const int8_t*>(A4),
                           reinterpret_cast<const int8_t*>(B4), beta, y, acc_s, acc_a_out, acc_b, ws, st);
}

}  // namespace dfssm
