// dfssm_linear.hpp -- device helpers shared by the scaffold + LoRA linear
// kernels that exchange the LoRA down-projection inside one launch (the
// few-token and the split-K tile kernel): sign expansion, int8 / int4 row
// loads, tagged words.
#pragma once

#include "dfssm_internal.hpp"
#include "dfssm_persist.hpp"

namespace dfssm {

// Tag of a call enqueued outside graph capture: a process-wide counter with
// bit 31 set, so it never equals a device-epoch tag (below 2^31) or 0.  One
// counter for every kernel whose words share the workspace region xw: a word
// that another kernel left there, in whatever layout, never validates.
uint32_t next_host_tag();
// Whether a call on st has to take its tag from the device epoch: true while
// the stream is being captured (a replay would repeat a frozen argument), and
// if the query fails (the device epoch is right either way; the failed
// query's error is cleared so that the launch check does not see it).
bool wants_device_epoch(hipStream_t st);

}  // namespace dfssm

namespace dfssm_lin {

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4i mfma(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ v4i zero4() { return v4i{0, 0, 0, 0}; }

// bits [sh, sh+16) of w -> 16 bytes of {0,1}, byte b of dword t = bit sh+4t+b
__device__ __forceinline__ v4i expand16_at(uint32_t w, uint32_t sh) {
  v4i o;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const uint32_t nib = __builtin_amdgcn_ubfe(w, sh + 4 * t, 4);
    o[t] = (int)((nib * 0x00204081u) & 0x01010101u);
  }
  return o;
}

__device__ __forceinline__ v4i load16(const int8_t* p) {
  const uint4 u = *reinterpret_cast<const uint4*>(p);
  return v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
}

// 16 bytes of an int8 row, zero outside [0, len)
__device__ __forceinline__ v4i load16_guarded(const int8_t* row, int start, int len, bool aligned) {
  if (start + 16 <= len && aligned) return load16(row + start);
  v4i o = zero4();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = start + e;
    const uint32_t b = (i >= 0 && i < len) ? (uint32_t)(uint8_t)row[i] : 0u;
    o[e >> 2] |= (int)(b << (8 * (e & 3)));
  }
  return o;
}

// int4 factors: two's-complement nibbles, value 2i in the low nibble of byte
// i.  sext_nibbles turns 4 bytes holding nibble values 0..15 into the
// signed values -8..7 (XOR 8, then a subtraction that cannot borrow across
// bytes); expand_i4 turns 8 packed bytes into the 16 int8 values in order.
__device__ __forceinline__ uint32_t sext_nibbles(uint32_t t) {
  t ^= 0x08080808u;
  return ((t | 0x80808080u) - 0x08080808u) ^ 0x80808080u;
}

__device__ __forceinline__ uint4 expand_i4(uint2 p) {
  const uint32_t lo0 = p.x & 0x0F0F0F0Fu, hi0 = (p.x >> 4) & 0x0F0F0F0Fu;
  const uint32_t lo1 = p.y & 0x0F0F0F0Fu, hi1 = (p.y >> 4) & 0x0F0F0F0Fu;
  // v_perm_b32 interleaves the low-nibble and high-nibble bytes
  return make_uint4(sext_nibbles(__builtin_amdgcn_perm(hi0, lo0, 0x05010400u)),
                    sext_nibbles(__builtin_amdgcn_perm(hi0, lo0, 0x07030602u)),
                    sext_nibbles(__builtin_amdgcn_perm(hi1, lo1, 0x05010400u)),
                    sext_nibbles(__builtin_amdgcn_perm(hi1, lo1, 0x07030602u)));
}

// values start .. start+15 (start % 16 == 0) of a factor row, in bytes
// (L4: 8 packed bytes at start/2)
template <bool L4>
__device__ __forceinline__ uint4 load_row16(const int8_t* row, int start) {
  if constexpr (L4) return expand_i4(*reinterpret_cast<const uint2*>(row + start / 2));
  return *reinterpret_cast<const uint4*>(row + start);
}

// 16 values of a factor row of len values, zero outside [0, len)
template <bool L4>
__device__ __forceinline__ v4i load16_row_guarded(const int8_t* row, int start, int len, bool aligned) {
  if constexpr (!L4) {
    return load16_guarded(row, start, len, aligned);
  } else {
    if (start + 16 <= len && aligned) {
      const uint4 u = load_row16<true>(row, start);
      return v4i{(int)u.x, (int)u.y, (int)u.z, (int)u.w};
    }
    v4i o = zero4();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int i = start + e;
      uint32_t b = 0u;
      if (i >= 0 && i < len) {
        const int byte = (uint8_t)row[i >> 1];
        const int nib = (i & 1) ? (byte >> 4) : (byte & 15);
        b = (uint32_t)(uint8_t)(int8_t)(nib >= 8 ? nib - 16 : nib);
      }
      o[e >> 2] |= (int)(b << (8 * (e & 3)));
    }
    return o;
  }
}

__device__ __forceinline__ int sdot4(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot4((int)a, (int)b, c, false);
}

// agent scope: the words cross XCDs (each XCD has its own L2)
__device__ __forceinline__ void word_store(uint64_t* p, uint32_t tag, uint32_t v) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t word_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t pack_limbs(int32_t v) {
  int8_t d[4];
  dfssm_dev::split_limbs(v, d);
  return (uint32_t)(uint8_t)d[0] | ((uint32_t)(uint8_t)d[1] << 8) | ((uint32_t)(uint8_t)d[2] << 16) |
         ((uint32_t)(uint8_t)d[3] << 24);
}

// 16 words of 4 limb bytes (word e: rank e) -> 4 limb operands (byte e of
// limb t = limb t of rank e)
__device__ __forceinline__ void limb_operands(const uint32_t (&val)[16], v4i (&lm)[4]) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    // 4x4 byte transpose: pairs, then halves
    const uint32_t p0 = __builtin_amdgcn_perm(val[4 * d + 1], val[4 * d], 0x05010400u);
    const uint32_t p1 = __builtin_amdgcn_perm(val[4 * d + 1], val[4 * d], 0x07030602u);
    const uint32_t p2 = __builtin_amdgcn_perm(val[4 * d + 3], val[4 * d + 2], 0x05010400u);
    const uint32_t p3 = __builtin_amdgcn_perm(val[4 * d + 3], val[4 * d + 2], 0x07030602u);
    lm[0][d] = (int)__builtin_amdgcn_perm(p2, p0, 0x05040100u);
    lm[1][d] = (int)__builtin_amdgcn_perm(p2, p0, 0x07060302u);
    lm[2][d] = (int)__builtin_amdgcn_perm(p3, p1, 0x05040100u);
    lm[3][d] = (int)__builtin_amdgcn_perm(p3, p1, 0x07060302u);
  }
}

typedef __attribute__((address_space(3))) void lds_void;
// direct-to-LDS loads; the LDS address is uniform already, which the compiler
// may not see
__device__ __forceinline__ void dma16(uint32_t voff, const void* sbase, uint32_t lds) {
  dfssm_px::lds_dma16(voff, sbase, (uint32_t)__builtin_amdgcn_readfirstlane((int)lds));
}
__device__ __forceinline__ void dma4(uint32_t voff, const void* sbase, uint32_t lds) {
  dfssm_px::lds_dma4(voff, sbase, (uint32_t)__builtin_amdgcn_readfirstlane((int)lds));
}
// at most n of the wave's vector-memory operations still in flight
template <int n>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory");
}
// at most y * u in flight (u a constant, y < 4 uniform)
template <int u>
__device__ __forceinline__ void wait_steps(int y) {
  if (y >= 3)
    wait_vm<3 * u>();
  else if (y == 2)
    wait_vm<2 * u>();
  else if (y == 1)
    wait_vm<u>();
  else
    wait_vm<0>();
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// 16-byte piece c of row m of a 128-byte-row tile sits at slot c ^ (m & 7): without
// it the rows of one read would all meet in one slot of either half of the banks.
// Pairs of rows still meet (a read serves rows 0-3 and 12-15 of lane group kg with
// rows 4-11 of group kg + 1, which reads piece c + 2): SQ_LDS_BANK_CONFLICT is 0.4 of
// the LDS cycles.  A placement without conflicts ((m1, m2 ^ m3, m3) of m's bits)
// took that to 0 and no time off: 2048 x 2048 x 8512 47.4 -> 47.0 us, 2048 x 4096 x
// 2048 35.1 -> 35.7, 32 x 4096 x 2048 6.34 -> 6.39.
__device__ __forceinline__ int swz8(int row) { return row & 7; }

// sum_k A[j,k] Q[m,k] (j < r) or sum_k Q[m,k] (j < 0), one lane alone
template <bool L4>
__device__ int lane_dot(const int8_t* __restrict__ A, const int8_t* __restrict__ q, int K, int j, int m) {
  const int8_t* qrow = q + (int64_t)m * K;
  const int8_t* arow = A + (int64_t)(j < 0 ? 0 : j) * (L4 ? K / 2 : K);
  int acc = 0;
  for (int k = 0; k < K; k += 16) {
    const uint4 x = *reinterpret_cast<const uint4*>(qrow + k);
    const uint4 w = j < 0 ? make_uint4(0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u)
                          : load_row16<L4>(arow, k);
    acc = sdot4(w.x, x.x, acc);
    acc = sdot4(w.y, x.y, acc);
    acc = sdot4(w.z, x.z, acc);
    acc = sdot4(w.w, x.w, acc);
  }
  return acc;
}

}  // namespace dfssm_lin
