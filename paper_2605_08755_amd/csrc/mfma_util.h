// Helpers shared by the matrix-core kernels (device code only).
#pragma once

#include <type_traits>
#include <utility>

#include "laq_internal.h"

namespace laq {

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kBufferFlagsM = 0x00020000;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, kBufferFlagsM);
}

// (a & m) | c in one v_and_or_b32.  The mask lives in a scalar register and
// the magic constant in a vector register (a VOP3 instruction takes no
// literal on this target, and at most one scalar operand); left to itself the
// compiler emits a v_and_b32 and a v_or_b32 with literals instead.  The
// compiler does not know what the statement is, so it adds no wait states
// between it and a matrix instruction: its result goes through a packed add
// before it is an operand, and no register of a matrix result may be free
// while that result is on its way (every element of it is used afterwards).
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t m, uint32_t c) {
  uint32_t r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(m), "v"(c));  // mask from a scalar register
  return r;
}

__device__ __forceinline__ uint32_t pk_add_f16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, a) + __builtin_bit_cast(half2_t, b));
}

// fp16 bit patterns of -(2^(10-p) + z) in both halves, for the field
// offsets used by the layouts (ulp of 2^(10-p) is 2^-p, so + z is + z*2^p
// ulps).  zz holds z in both 16-bit halves; z << shift < 2^11, so no carry
// crosses between the halves.
__device__ __forceinline__ uint32_t neg_magic(uint32_t base_bits, uint32_t zz, uint32_t shift) {
  return (base_bits | (base_bits << 16)) + (zz << shift);
}

// Exact (q - z) pairs of one 32-code chunk, in natural order: pair t holds
// codes 2t (low half) and 2t+1 (high half).
template <int BITS>
__device__ __forceinline__ void unpack_chunk_exact(const uint32_t (&w)[BITS], uint32_t z1, uint32_t (&pr)[16]) {
  const uint32_t z = z1 | (z1 << 16);
  if constexpr (BITS == 3) {
    const uint32_t n0 = neg_magic(0xE400u, z, 0);  // -(1024 + z): fields at bits 0-2
    const uint32_t n3 = neg_magic(0xD800u, z, 3);  // -(128 + z):  bits 3-5
    const uint32_t n6 = neg_magic(0xCC00u, z, 6);  // -(16 + z):   bits 6-8
    const uint32_t n7 = neg_magic(0xC800u, z, 7);  // -(8 + z):    bits 7-9
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint32_t t = w[p] >> 10;
      pr[5 * p + 0] = pk_add_f16(and_or(w[p], 0x00070007u, 0x64006400u), n0);
      pr[5 * p + 1] = pk_add_f16(and_or(w[p], 0x00380038u, 0x58005800u), n3);
      pr[5 * p + 2] = pk_add_f16(and_or(w[p], 0x01C001C0u, 0x4C004C00u), n6);
      pr[5 * p + 3] = pk_add_f16(and_or(t, 0x00070007u, 0x64006400u), n0);
      pr[5 * p + 4] = pk_add_f16(and_or(t, 0x00380038u, 0x58005800u), n3);
    }
    // codes 30/31: code bit j is bit 9 / bit 25 of plane j -> field at bits 7-9
    const uint32_t spare = ((w[0] >> 2) & 0x00800080u) | ((w[1] >> 1) & 0x01000100u) | (w[2] & 0x02000200u);
    pr[15] = pk_add_f16(spare | 0x48004800u, n7);
  } else {
    const uint32_t n0 = neg_magic(0xE400u, z, 0);  // -(1024 + z): nibbles at bits 0-3
    const uint32_t n4 = neg_magic(0xD400u, z, 4);  // -(64 + z):   bits 4-7
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t t = w[p] >> 8;
      pr[4 * p + 0] = pk_add_f16(and_or(w[p], 0x000F000Fu, 0x64006400u), n0);
      pr[4 * p + 1] = pk_add_f16(and_or(w[p], 0x00F000F0u, 0x54005400u), n4);
      pr[4 * p + 2] = pk_add_f16(and_or(t, 0x000F000Fu, 0x64006400u), n0);
      pr[4 * p + 3] = pk_add_f16(and_or(t, 0x00F000F0u, 0x54005400u), n4);
    }
  }
}

__device__ __forceinline__ half8_t frag(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(half8_t, u32x4v{a, b, c, d});
}

// s_waitcnt vmcnt(N) (other counters unconstrained), N a compile-time constant <= 63.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (((N >> 4) & 3) << 14));
}

// f(std::integral_constant<int, I>{}) for I = 0 .. N-1, in order.
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// 4 x 4 transpose across the four 16-lane quarters of a wave: on entry
// register c of quarter j holds element (j, c); on exit register j of
// quarter c holds it.  Two rounds of lane-half swaps (32 lanes, then 16).
__device__ __forceinline__ void transpose_quarters(uint32_t& r0, uint32_t& r1, uint32_t& r2, uint32_t& r3) {
  auto a = __builtin_amdgcn_permlane32_swap(r0, r2, false, false);
  auto b = __builtin_amdgcn_permlane32_swap(r1, r3, false, false);
  auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  r0 = c[0];
  r1 = c[1];
  r2 = d[0];
  r3 = d[1];
}

// Codes of a quad (four groups of 16 rows) through LDS.  A 16-byte load whose
// consecutive lanes lie in different rows moves 15.6 bytes per clock and
// compute unit, one with four consecutive lanes on 64 contiguous bytes 53
// (measured on MI355X, L2-resident); the matrix core's operands want
// consecutive lanes in consecutive rows.  So the codes go straight from memory
// to LDS with four lanes per row, and from LDS to registers in operand order,
// which also needs no cross-lane transposes.  Unit of a quad: BITS planes of
// 16 rows x 64 bytes, then the 16 x 4 scales and the 16 x 4 zero points, a
// 32-bit word each.  Piece p (group) of row r sits at position p ^ (r >> 2), so
// that reading one group of all rows touches every LDS bank once.
__host__ __device__ constexpr int unit_bytes(int bits) { return bits * 1024 + 512; }

__device__ __forceinline__ uint32_t lds_byte(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Requests quad q of a 16-row tile into the unit at st: BITS + 2 loads.  Groups
// past G get bit 31 in their offsets (past every extent: zeros), rows past the
// tile's are past the extents.  AUX: cache policy of the code loads.
template <int BITS, int AUX>
__device__ __forceinline__ void request_quad(char* st, __amdgpu_buffer_rsrc_t qr, __amdgpu_buffer_rsrc_t sr,
                                             __amdgpu_buffer_rsrc_t zr, int lane, int q, int G, bool live) {
  typedef __attribute__((address_space(3))) void lds_void;
  const int r = lane >> 2;
  const int gc = 4 * q + ((lane & 3) ^ (r >> 2));
  const int gz = 4 * q + (lane & 3);
  const uint32_t wo = (uint32_t)((r * BITS * G + gc) * 16) | (uint32_t)!(live && gc < G) << 31;
  const uint32_t dead = (uint32_t)!(live && gz < G) << 31;
#pragma unroll
  for (int p = 0; p < BITS; ++p)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(qr, (lds_void*)(st + p * 1024), 16, wo + p * G * 16, 0, 0, AUX);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, (lds_void*)(st + BITS * 1024), 2, (uint32_t)(r * G + gz) * 2 | dead, 0,
                                           0, 0);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(zr, (lds_void*)(st + BITS * 1024 + 256), 1, (uint32_t)(r * G + gz) | dead,
                                           0, 0, 0);
}

// This lane's words of a unit (row n, chunk j of each of the four groups, at
// a[gi] + plane * 1024) and the row's four scales and zero points (at asc +
// BITS * 1024 and 256 further).  Planes 1024 bytes apart are offsets 0 and 4 of
// a read2st64.  Inline assembly because the compiler makes every LDS read that
// follows a direct-to-LDS load wait for all such loads in flight; the statement
// waits for its own reads.
template <int BITS>
__device__ __forceinline__ void read_unit(uint32_t (&w)[4][BITS], u32x4& sc, u32x4& zc, const uint32_t (&a)[4],
                                          uint32_t asc) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  u32x2 d0, d1, d2, d3;
  if constexpr (BITS == 3) {
    asm volatile(
        "ds_read2st64_b32 %0, %10 offset0:0 offset1:4\n\t"
        "ds_read_b32 %4, %10 offset:2048\n\t"
        "ds_read_b128 %8, %14 offset:3072\n\t"
        "ds_read_b128 %9, %14 offset:3328\n\t"
        "ds_read2st64_b32 %1, %11 offset0:0 offset1:4\n\t"
        "ds_read_b32 %5, %11 offset:2048\n\t"
        "ds_read2st64_b32 %2, %12 offset0:0 offset1:4\n\t"
        "ds_read_b32 %6, %12 offset:2048\n\t"
        "ds_read2st64_b32 %3, %13 offset0:0 offset1:4\n\t"
        "ds_read_b32 %7, %13 offset:2048\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3), "=&v"(w[0][2]), "=&v"(w[1][2]), "=&v"(w[2][2]),
          "=&v"(w[3][2]), "=&v"(sc), "=&v"(zc)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(asc)
        : "memory");
  } else {
    u32x2 e0, e1, e2, e3;
    asm volatile(
        "ds_read2st64_b32 %0, %10 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %4, %10 offset0:8 offset1:12\n\t"
        "ds_read_b128 %8, %14 offset:4096\n\t"
        "ds_read_b128 %9, %14 offset:4352\n\t"
        "ds_read2st64_b32 %1, %11 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %5, %11 offset0:8 offset1:12\n\t"
        "ds_read2st64_b32 %2, %12 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %6, %12 offset0:8 offset1:12\n\t"
        "ds_read2st64_b32 %3, %13 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %7, %13 offset0:8 offset1:12\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3), "=&v"(e0), "=&v"(e1), "=&v"(e2), "=&v"(e3), "=&v"(sc),
          "=&v"(zc)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(asc)
        : "memory");
    w[0][2] = e0.x, w[0][3] = e0.y, w[1][2] = e1.x, w[1][3] = e1.y;
    w[2][2] = e2.x, w[2][3] = e2.y, w[3][2] = e3.x, w[3][3] = e3.y;
  }
  w[0][0] = d0.x, w[0][1] = d0.y, w[1][0] = d1.x, w[1][1] = d1.y;
  w[2][0] = d2.x, w[2][1] = d2.y, w[3][0] = d3.x, w[3][1] = d3.y;
}

// The unit at st as request_quad fills it: row lane % 16, chunk lane / 16.
template <int BITS>
__device__ __forceinline__ void read_quad(uint32_t (&w)[4][BITS], u32x4& sc, u32x4& zc, uint32_t st, int lane) {
  const uint32_t n = lane & 15;
  uint32_t a[4];
#pragma unroll
  for (uint32_t gi = 0; gi < 4; ++gi) a[gi] = st + n * 64 + 16 * (gi ^ (n >> 2)) + 4 * (lane >> 4);
  read_unit<BITS>(w, sc, zc, a, st + n * 16);
}

}  // namespace

}  // namespace laq
