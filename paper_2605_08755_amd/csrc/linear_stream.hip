// Skinny GEMM on the matrix cores for rows of at most 16 quads (a quad is
// four 128-groups, 512 columns; K <= 8192):
//   y[m][n] = sum_g s[n][g] * sum_{k in g} x[m][k] * (q[n][k] - z[n][g])   (Eq. 1)
//
// A block is TS x nq waves: wave (t, q) owns quad q of the row and keeps that
// quad's activations in registers as matrix-core operands for the whole
// launch, while the block walks over groups of TS tiles of 16 weight rows.
// Per tile a wave multiplies its quad, the nq waves' partial sums meet in LDS
// and are added in quad order, so results are deterministic.
//
// What bounds it, and why it is built this way (MI355X, measured):
//  - Vector-memory address rate.  A 16-byte load whose consecutive lanes lie
//    in different rows moves 15.6 bytes per clock and compute unit; with four
//    consecutive lanes on 64 contiguous bytes it moves 53.  The matrix core's
//    operand layout wants consecutive lanes in consecutive rows, so the codes
//    go memory -> LDS with four lanes per row (direct-to-LDS, no registers)
//    and LDS -> registers in operand order, which also makes the cross-lane
//    transposes of a register path unnecessary.
//  - Vector ALU work per weight.  A code field masked out of its word is an
//    fp16 subnormal of value q * 2^(p-24), exact as a matrix-core operand, so
//    a pair of codes costs one v_and_b32 (and a third of a shift), with the
//    zero point entering once per group as z * sum x.  Fields are brought to
//    two offsets (class 0 and class C), each with an accumulator of its own:
//    26 instructions per 32 codes of W3, where forming exact (q - z) pairs
//    took 45.
//  - Activation traffic.  x is read once per block, not once per tile.
#include <algorithm>

#include "mfma_util.h"

namespace laq {

namespace {

constexpr int kStreamLdsBytes = 160 * 1024;
constexpr int kStreamWaves = 16;  // waves per block: 128 registers each at 4 per SIMD

// Lanes of a wave that hold valid results (lane (n, j) holds rows 4j..4j+3 of
// column n), result registers per lane, and bytes of one wave's partials.
__host__ __device__ constexpr int valid_lanes(int MT) { return MT == 16 ? 64 : MT == 8 ? 32 : 16; }
__host__ __device__ constexpr int result_regs(int MT) { return MT < 4 ? MT : 4; }
__host__ __device__ constexpr int partial_bytes(int MT) { return valid_lanes(MT) * result_regs(MT) * 4; }

// Activation pair held by position i of the operand registers: positions 0-7
// pair up with the class 0 codes, 8-15 with the class C codes, in the order in
// which code_pairs makes them.
template <int BITS>
__device__ constexpr int pair_at(int i) {
  constexpr int p3[16] = {0, 3, 2, 5, 8, 7, 10, 13, 1, 4, 6, 9, 11, 14, 12, 15};
  constexpr int p4[16] = {0, 2, 4, 6, 8, 10, 12, 14, 1, 3, 5, 7, 9, 11, 13, 15};
  return BITS == 3 ? p3[i] : p4[i];
}

// The 16 code pairs of a 32-code chunk as fp16 subnormals: b[0..7] of value
// q * 2^-24 (fields at bits 0-2, or 0-3), b[8..15] of value q * 2^(C-24)
// (fields at bits 3-5: C = 3, or 4-7: C = 4).
template <int BITS>
__device__ __forceinline__ void code_pairs(const uint32_t (&w)[BITS], uint32_t (&b)[16]) {
  if constexpr (BITS == 3) {
    constexpr uint32_t m0 = 0x00070007u, m3 = 0x00380038u;
    const uint32_t t0 = w[0] >> 10, t1 = w[1] >> 10, t2 = w[2] >> 10;
    const uint32_t u0 = w[0] >> 6, u1 = w[1] >> 6, u2 = w[2] >> 3;
    b[0] = w[0] & m0;
    b[1] = t0 & m0;
    b[2] = u0 & m0;
    b[3] = w[1] & m0;
    b[4] = t1 & m0;
    b[5] = u1 & m0;
    b[6] = w[2] & m0;
    b[7] = t2 & m0;
    b[8] = w[0] & m3;
    b[9] = t0 & m3;
    b[10] = w[1] & m3;
    b[11] = t1 & m3;
    b[12] = w[2] & m3;
    b[13] = t2 & m3;
    b[14] = u2 & m3;
    // codes 30/31: code bit j is bit 9 / bit 25 of plane j -> field at bits 3-5
    b[15] = and_or(w[2] >> 4, 0x00200020u, and_or(w[1] >> 5, 0x00100010u, u0 & 0x00080008u));
  } else {
    constexpr uint32_t m0 = 0x000F000Fu, m4 = 0x00F000F0u;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t t = w[p] >> 8;
      b[2 * p + 0] = w[p] & m0;
      b[2 * p + 1] = t & m0;
      b[8 + 2 * p + 0] = w[p] & m4;
      b[8 + 2 * p + 1] = t & m4;
    }
  }
}
template <int BITS>
constexpr float kClassRatio = BITS == 3 ? 0.125f : 0.0625f;  // 2^-C

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// LDS accesses of this kernel are inline assembly: the compiler makes every
// LDS access that follows a direct-to-LDS load wait for all such loads in
// flight, the next tiles' included.  Each statement waits for its own reads
// (lgkmcnt), and the data flow's other waits (vmcnt, barriers) are explicit.
template <int OFF>
__device__ __forceinline__ void lds_read4_b128(u32x4 (&f)[4], const uint32_t (&a)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\t"
      "ds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\t"
      "ds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "i"(OFF)
      : "memory");
}
// A stage's words of this lane (row n, chunk c of each of the four groups, at
// a[gi] + plane * 1024), row n's four scales (at asc + BITS * 1024), and the
// scale and zero point of group c (at aown + BITS * 1024, and 256 further).
// Planes 1024 bytes apart are offsets 0 and 4 of a read2st64.
template <int BITS>
__device__ __forceinline__ void lds_read_stage(uint32_t (&w)[4][BITS], u32x4& sc, uint32_t& so, uint32_t& zo,
                                               const uint32_t (&a)[4], uint32_t asc, uint32_t aown) {
  u32x2 d0, d1, d2, d3;
  if constexpr (BITS == 3) {
    asm volatile(
        "ds_read2st64_b32 %0, %11 offset0:0 offset1:4\n\t"
        "ds_read_b32 %4, %11 offset:2048\n\t"
        "ds_read_b128 %8, %15 offset:3072\n\t"
        "ds_read2st64_b32 %1, %12 offset0:0 offset1:4\n\t"
        "ds_read_b32 %5, %12 offset:2048\n\t"
        "ds_read2st64_b32 %2, %13 offset0:0 offset1:4\n\t"
        "ds_read_b32 %6, %13 offset:2048\n\t"
        "ds_read2st64_b32 %3, %14 offset0:0 offset1:4\n\t"
        "ds_read_b32 %7, %14 offset:2048\n\t"
        "ds_read_b32 %9, %16 offset:3072\n\t"
        "ds_read_b32 %10, %16 offset:3328\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3), "=&v"(w[0][2]), "=&v"(w[1][2]), "=&v"(w[2][2]),
          "=&v"(w[3][2]), "=&v"(sc), "=&v"(so), "=&v"(zo)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(asc), "v"(aown)
        : "memory");
  } else {
    u32x2 e0, e1, e2, e3;
    asm volatile(
        "ds_read2st64_b32 %0, %11 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %4, %11 offset0:8 offset1:12\n\t"
        "ds_read_b128 %8, %15 offset:4096\n\t"
        "ds_read2st64_b32 %1, %12 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %5, %12 offset0:8 offset1:12\n\t"
        "ds_read2st64_b32 %2, %13 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %6, %13 offset0:8 offset1:12\n\t"
        "ds_read2st64_b32 %3, %14 offset0:0 offset1:4\n\t"
        "ds_read2st64_b32 %7, %14 offset0:8 offset1:12\n\t"
        "ds_read_b32 %9, %16 offset:4096\n\t"
        "ds_read_b32 %10, %16 offset:4352\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3), "=&v"(e0), "=&v"(e1), "=&v"(e2), "=&v"(e3), "=&v"(sc),
          "=&v"(so), "=&v"(zo)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(asc), "v"(aown)
        : "memory");
    w[0][2] = e0.x, w[0][3] = e0.y, w[1][2] = e1.x, w[1][3] = e1.y;
    w[2][2] = e2.x, w[2][3] = e2.y, w[3][2] = e3.x, w[3][3] = e3.y;
  }
  w[0][0] = d0.x, w[0][1] = d0.y, w[1][0] = d1.x, w[1][1] = d1.y;
  w[2][0] = d2.x, w[2][1] = d2.y, w[3][0] = d3.x, w[3][1] = d3.y;
}
template <int OFF>
__device__ __forceinline__ void lds_write_b32(uint32_t addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1 offset:%2" ::"v"(addr), "v"(v), "i"(OFF) : "memory");
}
// Eight partials of one output, STRIDE bytes apart.
template <int STRIDE>
__device__ __forceinline__ void lds_read8_b32(float (&v)[8], uint32_t a) {
  asm volatile(
      "ds_read_b32 %0, %8\n\t"
      "ds_read_b32 %1, %8 offset:%9\n\t"
      "ds_read_b32 %2, %8 offset:%10\n\t"
      "ds_read_b32 %3, %8 offset:%11\n\t"
      "ds_read_b32 %4, %8 offset:%12\n\t"
      "ds_read_b32 %5, %8 offset:%13\n\t"
      "ds_read_b32 %6, %8 offset:%14\n\t"
      "ds_read_b32 %7, %8 offset:%15\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(a), "i"(STRIDE), "i"(2 * STRIDE), "i"(3 * STRIDE), "i"(4 * STRIDE), "i"(5 * STRIDE), "i"(6 * STRIDE),
        "i"(7 * STRIDE)
      : "memory");
}
// This wave's LDS accesses are done, then the block's barrier (a
// __syncthreads() would also wait for the loads in flight).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// Waits until at most `later` stages' loads (WL each) are outstanding.
template <int WL>
__device__ __forceinline__ void wait_stages(int later) {
  __builtin_amdgcn_sched_barrier(0);
  if (later <= 0) wait_vmcnt<0>();
  else if (later == 1) wait_vmcnt<WL>();
  else if (later == 2) wait_vmcnt<2 * WL>();
  else wait_vmcnt<3 * WL>();
  __builtin_amdgcn_sched_barrier(0);
}
// TS tiles per step, nb partial buffers (2: one barrier per step, 1: two), D
// ring stages, nq quads, and whether the sums are those of a K range.
constexpr int stream_cfg(int TS, int nb, int D, int nq, bool partial) {
  return TS | nb << 5 | D << 7 | nq << 10 | (int)partial << 15;
}
constexpr int kStreamStages = 4;  // most stages of the ring

// MT: activation rows staged (4, 8 or 16; rows past M read zeros).
// PH: groups of a quad staged at a time (4, or 2 or 1 where the waves' slabs of
// four groups do not fit in LDS).  cfg: stream_cfg().  The block's quads are
// q0 .. q0 + nq - 1 (those past the row read zeros); a range of them writes its
// fp32 partial sums to part [M][N] instead of the fp16 outputs to y.
template <int BITS, int MT, int PH>
__device__ __forceinline__ void stream_block(
    const uint16_t* __restrict__ x, const uint32_t* __restrict__ qw, const uint16_t* __restrict__ scales,
    const uint8_t* __restrict__ zeros, uint16_t* __restrict__ y, float* __restrict__ part, int M, int N, int G,
    int cfg, int b, int nblocks, int q0) {
  typedef __attribute__((address_space(3))) void lds_void;
  extern __shared__ u32x4 lds[];
  constexpr int SB = unit_bytes(BITS);
  constexpr int PB = partial_bytes(MT);
  constexpr int LV = valid_lanes(MT);
  constexpr int NR = result_regs(MT);
  constexpr int WL = BITS + 2;  // loads of a stage per wave
  constexpr int XR = PH * 16;   // 16-byte pieces of a slab row

  const int TS = cfg & 31, nb = (cfg >> 5) & 3, D = (cfg >> 7) & 7, nq = (cfg >> 10) & 31;
  const bool partial = cfg >> 15;
  const int W = TS * nq;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = TS == 1 ? 0 : w / nq;  // tile of the group
  const int q = w - t * nq;            // quad of the block's
  const int K = 128 * G;
  char* const ldsb = reinterpret_cast<char*>(lds);

  // 1. The quad's activations, PH groups at a time: rows 0..MT-1 of the slab
  //    (shared by the quad's TS waves, which split its rows; TS > 1 only with
  //    PH = 4), piece p of row m at position p ^ (m & 7).  The first stage of
  //    codes is requested behind the first slab's loads.
  const __amdgpu_buffer_rsrc_t xr = rsrc(x, (uint32_t)M * K * 2);
  char* const slab = ldsb + W * SB + q * (MT * PH * 256);
  auto fetch_slab = [&](int ph) {
    constexpr int RPI = 4 / PH;  // slab rows per load instruction
    for (int i = t; i < MT / RPI; i += TS) {
      const int m = i * RPI + lane / XR;
      const int col = 512 * (q0 + q) + 128 * PH * ph + 8 * ((lane % XR) ^ (m & 7));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void*)(slab + i * 1024), 16,
                                               (uint32_t)(m * K + col) * 2 | (uint32_t)!(m < M && col < K) << 31, 0,
                                               0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  fetch_slab(0);

  // Load roles.  Two neighbouring quads are the 128 contiguous bytes of a row
  // and plane that make a whole cache line, so their two waves share the
  // loads: each brings eight rows of the pair's eight groups, lane l 16 bytes
  // (one plane of one group) of row 8 h + l / 8 (h = q & 1).  (Measured at
  // 51200 x 5120, loads alone: 21.7 us with each wave its own 64-byte pieces,
  // 18.8 us with whole lines and the non-temporal policy, which only whole
  // lines can use.)  The last quad of an odd count brings its own 16 rows of
  // 64 bytes.  Piece p of row r sits at position p ^ swizzle(r), so that
  // reading one group of all 16 rows touches every LDS bank once.  Scales and
  // zero points: the same rows and groups, each lane's value in a word of its
  // own.  Groups past G get bit 31 in their offsets: past every extent, read
  // as zero.
  const bool paired = (q | 1) < nq;  // uniform over the wave
  const bool whole = (G & 7) == 0;    // rows of whole lines
  const int h = paired ? q & 1 : 0;
  const int lr = paired ? 8 * h + (lane >> 3) : lane >> 2;
  const int gb = 4 * (q0 + q - h);  // first group loaded
  const int gc = gb + (paired ? (lane & 7) ^ ((lr >> 1) & 7) : (lane & 3) ^ ((lr >> 2) & 3));
  const int gz = gb + (paired ? lane & 7 : lane & 3);
  uint32_t wo[BITS];
#pragma unroll
  for (int p = 0; p < BITS; ++p) wo[p] = (uint32_t)(((lr * BITS + p) * G + gc) * 16) | (uint32_t)(gc >= G) << 31;
  const uint32_t zo = (uint32_t)(lr * G + gz) | (uint32_t)(gz >= G) << 31;
  const uint32_t so = (uint32_t)((lr * G + gz) * 2) | (uint32_t)(gz >= G) << 31;
  // Requests this wave's quad of iteration i into ring stage S; tiles past
  // the last read zeros.  WL loads, none of them into registers.
  auto issue = [&](int i, int S) {
    const uint32_t r0 = (((uint32_t)(b + i * nblocks)) * (uint32_t)TS + (uint32_t)t) * 16u;
    const uint32_t rows = r0 < (uint32_t)N ? min(16u, (uint32_t)N - r0) : 0u;
    const int64_t row0 = rows ? (int64_t)r0 : 0;
    const __amdgpu_buffer_rsrc_t qr = rsrc(qw + row0 * BITS * 4 * G, rows * BITS * G * 16);
    const __amdgpu_buffer_rsrc_t sr = rsrc(scales + row0 * G, rows * G * 2);
    const __amdgpu_buffer_rsrc_t zr = rsrc(zeros + row0 * G, rows * G);
    char* const st = ldsb + (S * W + w) * SB;
#pragma unroll
    for (int p = 0; p < BITS; ++p)
      if (whole)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(qr, (lds_void*)(st + p * 1024), 16, wo[p], 0, 0, 2);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(qr, (lds_void*)(st + p * 1024), 16, wo[p], 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, (lds_void*)(st + BITS * 1024), 2, so, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(zr, (lds_void*)(st + BITS * 1024 + 256), 1, zo, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  const int groups = ((N + 15) / 16 + TS - 1) / TS;  // tile groups; block b takes b, b + nblocks, ...
  const int iters = (groups - b + nblocks - 1) / nblocks;
  issue(0, 0);
  const int nl = lane & 15;  // weight row / activation row / result column
  const int j = lane >> 4;   // chunk of a group
  const int arow = nl & (MT - 1);
  uint32_t xa[4];
#pragma unroll
  for (int jj = 0; jj < 4; ++jj) xa[jj] = lds_byte(slab) + arow * (XR * 16) + 16 * ((4 * j + jj) ^ (arow & 7));
  u32x4 af[4][4];  // [group][matrix-core step]
  float xs[4];     // this chunk's sum of x per group
  static_for<4 / PH>([&](auto pc) {
    constexpr int ph = decltype(pc)::value;
    if constexpr (ph > 0) fetch_slab(ph);  // this wave's reads of the slab have returned
    wait_stages<WL>(ph == 0 ? 1 : 0);
    if (TS > 1) lds_barrier();  // the other waves' rows of the slab
    static_for<PH>([&](auto gc2) {
      constexpr int gi = ph * PH + decltype(gc2)::value;
      u32x4 f[4];
      lds_read4_b128<256 * decltype(gc2)::value>(f, xa);
      uint32_t xp[16];
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        xp[4 * jj + 0] = f[jj].x;
        xp[4 * jj + 1] = f[jj].y;
        xp[4 * jj + 2] = f[jj].z;
        xp[4 * jj + 3] = f[jj].w;
      }
      float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        s0 = __builtin_amdgcn_fdot2(as_half2(xp[k]), as_half2(0x3C003C00u), s0, false);
        s1 = __builtin_amdgcn_fdot2(as_half2(xp[8 + k]), as_half2(0x3C003C00u), s1, false);
      }
      xs[gi] = s0 + s1;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        af[gi][k] = u32x4{xp[pair_at<BITS>(4 * k)], xp[pair_at<BITS>(4 * k + 1)], xp[pair_at<BITS>(4 * k + 2)],
                          xp[pair_at<BITS>(4 * k + 3)]};
    });
  });
  // Lane (m, j): the sum of row m over group j (chunks in order).
  float xsum;
  {
    uint32_t r0 = __builtin_bit_cast(uint32_t, xs[0]), r1 = __builtin_bit_cast(uint32_t, xs[1]);
    uint32_t r2 = __builtin_bit_cast(uint32_t, xs[2]), r3 = __builtin_bit_cast(uint32_t, xs[3]);
    transpose_quarters(r0, r1, r2, r3);
    xsum = (__builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1)) +
           (__builtin_bit_cast(float, r2) + __builtin_bit_cast(float, r3));
  }
  // The slabs' place becomes ring stages and partials once every wave has
  // read its operands.  (Slabs in LDS of their own, with every stage requested
  // before the activations are used, measured no faster.)
  lds_barrier();
  for (int i = 1; i < D && i < iters; ++i) issue(i, i);

  // 2. Tiles.
  // Where this lane's row nl lies in a stage: the codes of group gi, chunk j,
  // and the quad's four scales.
  uint32_t ca[4], sca;
  {
    const uint32_t st = lds_byte(ldsb + (w - h) * SB) + (paired ? (nl >> 3) * SB : 0);
    const int rowb = paired ? (nl & 7) * 128 : nl * 64;
    const int swz = paired ? (nl >> 1) & 7 : (nl >> 2) & 3;
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) ca[gi] = st + rowb + 16 * ((4 * h + gi) ^ swz) + 4 * j;
    sca = st + (paired ? (nl & 7) * 32 + 16 * h : nl * 16);
  }
  const uint32_t parts = lds_byte(ldsb + D * W * SB);
  int S = 0;  // ring stage of iteration i
  wait_stages<WL>(min(D, iters) - 1);
  lds_barrier();  // (the pair's other half)
  for (int i = 0; i < iters; ++i) {
    uint32_t cw[4][BITS], so_, zo_;
    u32x4 sc;
    {
      const uint32_t off = (uint32_t)(S * W * SB);
      const uint32_t a[4] = {ca[0] + off, ca[1] + off, ca[2] + off, ca[3] + off};
      lds_read_stage<BITS>(cw, sc, so_, zo_, a, sca + off, sca + off + 4 * j);
    }
    // In units of 2^-24 (the operands' subnormals): sum over the groups of
    // s * (sum_k q x), then - s z sum x of the four groups by one fp32 MFMA.
    float4_t acc = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) {
      uint32_t pr[16];
      code_pairs<BITS>(cw[gi], pr);
      float4_t c0 = float4_t{0.f, 0.f, 0.f, 0.f}, c1 = c0;
      c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, af[gi][0]), frag(pr[0], pr[1], pr[2], pr[3]), c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, af[gi][2]), frag(pr[8], pr[9], pr[10], pr[11]), c1, 0, 0, 0);
      c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, af[gi][1]), frag(pr[4], pr[5], pr[6], pr[7]), c0, 0, 0, 0);
      c1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, af[gi][3]), frag(pr[12], pr[13], pr[14], pr[15]), c1, 0, 0, 0);
      const uint32_t scg = gi == 0 ? sc.x : gi == 1 ? sc.y : gi == 2 ? sc.z : sc.w;
      const _Float16 s = __builtin_bit_cast(_Float16, (uint16_t)(scg & 0xFFFFu));
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[r] = fmaf((float)s, fmaf(c1[r], kClassRatio<BITS>, c0[r]), acc[r]);
    }
    const float sown = (float)__builtin_bit_cast(_Float16, (uint16_t)(so_ & 0xFFFFu));
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xsum, sown * (float)zo_ * -0x1p-24f, acc, 0, 0, 0);

    const uint32_t pbuf = parts + (uint32_t)(((nb - 1) & i) * W * PB);
    // (The products by 2^24 also stand between the matrix instruction and the
    // stores: the compiler inserts the wait states that a reader of its result
    // needs before instructions it knows, not before inline assembly.)
    if (LV == 64 || lane < LV) {
      const uint32_t pa = pbuf + w * PB + lane * 4;
      static_for<NR>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        lds_write_b32<r * LV * 4>(pa, __builtin_bit_cast(uint32_t, acc[r] * 0x1p24f));
      });
    }
    // The next iteration's stage has landed when only later stages' loads
    // are outstanding (the output stores issued meanwhile are older); the
    // barrier publishes it and the partials, and frees this iteration's stage.
    wait_stages<WL>(min(D, iters - i) - 2);
    lds_barrier();
    // Outputs: the nq waves' partials of a tile in quad order, read eight at
    // a time (the last eight overlap the ones before).
    constexpr int NO = LV * NR;
    for (int idx = threadIdx.x; idx < TS * NO; idx += 64 * W) {
      const int tt = idx / NO, e = idx % NO;
      const int r = e / LV, ln = e % LV;
      float v = 0.0f;
      for (int k = 0; k < nq; k += 8) {
        const int k0 = max(0, min(k, nq - 8));
        float p[8];
        lds_read8_b32<PB>(p, pbuf + (uint32_t)((tt * nq + k0) * PB + e * 4));
#pragma unroll
        for (int u = 0; u < 8; ++u) v += k0 + u >= k && k0 + u < nq ? p[u] : 0.0f;
      }
      const int m = 4 * (ln >> 4) + r;
      const int64_t n = ((int64_t)(b + i * nblocks) * TS + tt) * 16 + (ln & 15);
      if (m < M && n < N) {
        if (partial) part[(int64_t)m * N + n] = v;
        else y[(int64_t)m * N + n] = __builtin_bit_cast(uint16_t, (_Float16)v);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (i + D < iters) issue(i + D, S);
    if (nb == 1 && i + 1 < iters) lds_barrier();  // the partials are read before the next tile's are written
    S = S + 1 == D ? 0 : S + 1;
  }
}

// part: K ranges of nq quads, block b taking range b / nblocks and writing
// part[range][M][N]; or null (one range, outputs to y).
template <int BITS, int MT, int PH>
__global__ __launch_bounds__(64 * kStreamWaves) void linear_stream_kernel(
    const uint16_t* __restrict__ x, const uint32_t* __restrict__ qw, const uint16_t* __restrict__ scales,
    const uint8_t* __restrict__ zeros, int M, int N, int G, int cfg, int nblocks, uint16_t* __restrict__ y,
    float* __restrict__ part) {
  const int range = cfg >> 15 ? (int)blockIdx.x / nblocks : 0;
  stream_block<BITS, MT, PH>(x, qw, scales, zeros, y, part + (int64_t)range * M * N, M, N, G, cfg,
                             (int)blockIdx.x - range * nblocks, nblocks, range * ((cfg >> 10) & 31));
}

}  // namespace

StreamPlan stream_plan(int bits, int M, int64_t N, int G, int ranges) {
  StreamPlan p;
  // (ranges of an even number of quads, so that whole lines stay in one range)
  const int nq_all = (G + 3) / 4;
  const int nq = ranges == 1 ? nq_all : ((nq_all + ranges - 1) / ranges + 1) / 2 * 2;
  if (nq > kStreamWaves) return p;
  const int64_t tiles = (N + 15) / 16;
  const int MT = M <= 4 ? 4 : M <= 8 ? 8 : 16;
  const int SB = unit_bytes(bits), PB = partial_bytes(MT);
  auto lds = [&](int TS, int PH, int D, int nb) {
    const int W = TS * nq;
    // (a tile's partials are read in batches of eight quads)
    return W * SB + std::max(nq * MT * PH * 256, (D - 1) * W * SB + (nb * W + std::max(0, 8 - nq)) * PB);
  };
  int TS = (int)std::min<int64_t>(kStreamWaves / nq, (tiles + 255) / 256);
  TS = std::max(1, TS);
  while (TS > 1 && lds(TS, 4, 2, 1) > kStreamLdsBytes) --TS;
  int PH = 4;
  while (PH > 1 && lds(TS, PH, 2, 1) > kStreamLdsBytes) PH /= 2;
  if (lds(TS, PH, 2, 1) > kStreamLdsBytes) return p;
  const int64_t groups = (tiles + TS - 1) / TS;
  const int nblocks = (int)std::min<int64_t>(groups, 256 / ranges);
  const int64_t iters = (groups + nblocks - 1) / nblocks;
  p.D = 1;
  while (p.D < kStreamStages && p.D < iters && lds(TS, PH, p.D + 1, 1) <= kStreamLdsBytes) ++p.D;
  p.nb = lds(TS, PH, p.D, 2) <= kStreamLdsBytes ? 2 : 1;
  p.MT = MT;
  p.PH = PH;
  p.TS = TS;
  p.W = TS * nq;
  p.nblocks = nblocks;
  p.nq = nq;
  p.ranges = (nq_all + nq - 1) / nq;
  p.lds = (uint32_t)lds(TS, PH, p.D, p.nb);
  return p;
}

template <int BITS>
hipError_t launch_linear_stream(const StreamPlan& p, const uint16_t* x, const uint32_t* qweight,
                                const uint16_t* scales, const uint8_t* zeros, uint16_t* y, float* part, int M,
                                int64_t N, int G, hipStream_t stream, const LaunchEvents& ev) {
  const int cfg = stream_cfg(p.TS, p.nb, p.D, p.nq, part != nullptr);
#define LAQ_ST(MTV, PHV)                                                                                             \
  launch(linear_stream_kernel<BITS, MTV, PHV>, dim3(p.nblocks * p.ranges), dim3(64 * p.W), p.lds, stream, ev, x, \
         qweight, scales, zeros, M, (int)N, G, cfg, p.nblocks, y, part)
  if (p.MT == 16 && p.PH == 4) LAQ_ST(16, 4);
  else if (p.MT == 16 && p.PH == 2) LAQ_ST(16, 2);
  else if (p.MT == 16 && p.PH == 1) LAQ_ST(16, 1);
  else if (p.MT == 8 && p.PH == 4) LAQ_ST(8, 4);
  else if (p.MT == 8 && p.PH == 2) LAQ_ST(8, 2);
  else if (p.MT == 4 && p.PH == 4) LAQ_ST(4, 4);
  else return hipErrorInvalidValue;
#undef LAQ_ST
  return hipGetLastError();
}

template hipError_t launch_linear_stream<3>(const StreamPlan&, const uint16_t*, const uint32_t*, const uint16_t*,
                                            const uint8_t*, uint16_t*, float*, int, int64_t, int, hipStream_t,
                                            const LaunchEvents&);
template hipError_t launch_linear_stream<4>(const StreamPlan&, const uint16_t*, const uint32_t*, const uint16_t*,
                                            const uint8_t*, uint16_t*, float*, int, int64_t, int, hipStream_t,
                                            const LaunchEvents&);

}  // namespace laq
