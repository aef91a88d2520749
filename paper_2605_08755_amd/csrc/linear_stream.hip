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
//  - Vector ALU work per weight.  The products are of exact (q - z) values as
//    normal fp16 numbers (45 instructions per 32 codes of W3, 40 of W4), the
//    same as in the tile-by-tile kernels.  (Codes masked out of their words
//    alone, fp16 subnormals q * 2^(p-24), with z * sum x subtracted per group,
//    take 26 and ran 51200 x 5120 W3 at M = 16 in 28.6 us instead of 32.2, but
//    the matrix core keeps fewer bits of products with subnormal operands: the
//    error before the output's rounding was 2.4e-5 of its RMS for N(0, 1)
//    activations and 1.6e-4 for one-signed ones at K = 25600, against 1e-7, and
//    an infinite activation gave NaN in every output of its row.)
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
constexpr int kResultRegs = 4;
__host__ __device__ constexpr int partial_bytes(int MT) { return valid_lanes(MT) * kResultRegs * 4; }

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
  constexpr int NR = kResultRegs;
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
  static_for<4 / PH>([&](auto pc) {
    constexpr int ph = decltype(pc)::value;
    if constexpr (ph > 0) fetch_slab(ph);  // this wave's reads of the slab have returned
    wait_stages<WL>(ph == 0 ? 1 : 0);
    if (TS > 1) lds_barrier();  // the other waves' rows of the slab
    static_for<PH>([&](auto gc2) {
      lds_read4_b128<256 * decltype(gc2)::value>(af[ph * PH + decltype(gc2)::value], xa);
    });
  });
  // The slabs' place becomes ring stages and partials once every wave has
  // read its operands.  (Slabs in LDS of their own, with every stage requested
  // before the activations are used, measured no faster.)
  lds_barrier();
  for (int i = 1; i < D && i < iters; ++i) issue(i, i);

  // 2. Tiles.
  // Where this lane's row nl lies in a stage: the codes of group gi, chunk j,
  // and the row's four scales (zero points 256 bytes further).
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
    uint32_t cw[4][BITS];
    u32x4 sc, zc;
    {
      const uint32_t off = (uint32_t)(S * W * SB);
      const uint32_t a[4] = {ca[0] + off, ca[1] + off, ca[2] + off, ca[3] + off};
      read_unit<BITS>(cw, sc, zc, a, sca + off);
    }
    float4_t acc = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) {
      uint32_t pr[16];
      unpack_chunk_exact<BITS>(cw[gi], zc[gi], pr);
      float4_t c = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, af[gi][jj]),
                                                   frag(pr[4 * jj], pr[4 * jj + 1], pr[4 * jj + 2], pr[4 * jj + 3]), c,
                                                   0, 0, 0);
      acc += (float)__builtin_bit_cast(_Float16, (uint16_t)(sc[gi] & 0xFFFFu)) * c;
    }

    const uint32_t pbuf = parts + (uint32_t)(((nb - 1) & i) * W * PB);
    // (The vector addition above stands between the matrix instruction and the
    // stores: the compiler inserts the wait states that a reader of its result
    // needs before instructions it knows, not before inline assembly.)
    if (LV == 64 || lane < LV) {
      const uint32_t pa = pbuf + w * PB + lane * 4;
      static_for<NR>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const float v = acc[r];  // (a bit cast of the vector's element itself takes element 0)
        lds_write_b32<r * LV * 4>(pa, __builtin_bit_cast(uint32_t, v));
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
