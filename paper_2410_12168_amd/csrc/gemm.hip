// gemm.hip -- W4Ax mixed-precision GEMM for gfx950 (paper Sec. 4).
//
// Operand path.  Both operands arrive as sign-magnitude codes.  A 4-bit chunk
// becomes FP8-E4M3 subnormal bytes (code * 2^-9) with two masks and one
// rotate per 8 codes; an 8-bit activation byte (sign, 7-bit magnitude m)
// becomes two such FP8 bytes, hi = m >> 3 (0..15) and lo = m & 7, so that
// code = 8 * hi + lo.  Each 32x32 output block of one K-block is two chained
// v_mfma_f32_32x32x64_f8f6f4 for W4A4 (K = 128 = one block) and four for W4A8,
// the hi ones with an E8M0 block scale of 2^3 on A.  Products of such codes are
// integers times 2^-18 and their sums stay below 2^24 units, so the fp32 MFMA
// result is the exact block sum (the paper's integer tile result, Sec. 4.1) and
// needs no int->float convert.
// Dequantization (Sec. 4.3: the scale absorbs the conversion factor), once per
// output and K-block:
//     C += Y * P,   P = 2 sa * sw    (fp32; exact),
// with P from one v_mfma_f32_32x32x8_f16 per block (K = 2 of 8 used, twice the
// same product), which leaves one vector operation per output; C is kept in
// units of 2^-17, scaled once at the end.
//
// What bounds it: a SIMD issues MFMAs and vector operations in turn more than
// side by side.  A 16x16x128 MFMA with the eight vector operations of its
// dequantization measured 45 cycles at best (54 as the compiler orders them)
// for 32 of matrix work; a 32x32x64 reads half the operand registers per
// product, and with P on the matrix core the same work takes 43, 40 of them
// matrix work, if no wait falls between (register-only, 2.4 GHz).  The 256-row
// tile reaches 67: one of the two pipes is busy 88% of the time, the rest is LDS
// traffic (fragments, unpacking, direct loads) and barriers.  The 128-row tile is at
// 89, with both pipes idle nearly half of the time: four MFMA blocks a wave between
// barriers are too few to cover the fragment reads and waves 0-3's unpacking.
//
// Kernel structure (the gfx950 form of the paper's software pipeline,
// Sec. 4.2, and of its tile decomposition, Sec. 4.4):
//   * persistent workgroups of 8 waves walk a host-built list of work units
//     (tile, K-block range); full tiles go to one workgroup, the fractional
//     last wave of tiles is split over all of them by cost;
//   * packed weights and activation codes stream HBM -> LDS with direct
//     (register-free) loads, several K-blocks ahead: weights by waves 4-7 into
//     a ring, activations by waves 0-3, which unpack them once per workgroup
//     into a double-buffered stage of FP8 bytes; each wave unpacks the weight
//     fragments it uses;
//   * in the 256-row tile the two waves of a SIMD alternate, one computing
//     while the other prepares; in the 128-row tile all waves run in step;
//   * split tiles write fp32 partials; the last workgroup to finish a tile
//     (arrival counter, no waiting) adds the partials in slot order and
//     stores fp16, so the result does not depend on arrival order.
// Measured (LLaMA-3-70B, 1/16 of the blocks 8-bit): gate_up at 4096 tokens 1696 us,
// qkv 324 us; gate_up at 128 tokens 80 to 84 us; LLaMA-3-8B o at 2048 tokens 44 us.
// Steps on the way, each against its predecessor on one box, back to back:
// 32x32x64 MFMAs with P on the matrix core and phases, against 16x16x128 MFMAs with
// P on the vector ALU and one barrier per K-block for both tiles, gate_up 1895 ->
// 1783 us at 4096 tokens and 88.3 -> 84.5 us at 128, qkv 351 -> 317 us; one scale
// operand per column block (scale_products32) in place of both side by side, gate_up
// with its quantizer 1767 -> 1728 and 86.0 -> 82.6 us; one write of M0 for a wave's
// four weight panels (dma16_from4) in place of four, 1731 -> 1723 and 85.9 -> 81.3 us.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "fmpq.h"
#include "kernels.h"
#include "operand.h"
#include "swiglu.h"

namespace comet {

namespace {

constexpr int kWr = kTileN * 64;            // one packed weight K-block of a tile
constexpr int kOrderLds = 4 * kMaxBlocks;   // the kernel's LDS copy of the K-block order
constexpr int kARb = 4096 + 64;             // a row block's activation codes in a stage
constexpr int kSlot = kWr + 2 * kTileN;     // weight ring slot: packed weights + fp16 weight scales

// Geometry of a tile of TM rows: 256, or 128 where comet::choose_tile_m finds
// that faster (up to 128 rows, where half of a 256-row tile would be padding,
// and for some larger shapes).  The waves' quadrants are 128 x 64 in the
// 256-row tile and 64 x 64 in the 128-row tile (2 x 4 waves, two per SIMD).
// Waves 0-3 stage activations, waves 4-7 load weights.
// LDS: two stages of activation codes ready for the MFMAs, the packed codes of
// a later K-block (raw), a ring of four K-blocks' activation scales (32 bits
// each) and one of D K-blocks' weights, as deep as fits.
template <int TM>
struct Geo {
  static constexpr int Waves = 8;
  static constexpr int Threads = 64 * Waves;
  static constexpr int WCols = Waves / 2;          // waves side by side
  static constexpr int WN = kTileN / WCols;        // wave quadrant columns
  static constexpr int WM = TM / 2;                // and rows
  static constexpr int RB = WM / 32;               // 32-row blocks per quadrant
  static constexpr int CB = WN / 32;               // 32-column blocks
  static constexpr int NB = RB * CB;
  static constexpr int LW = Waves / 2;             // waves of a role
  static constexpr int RW = TM / LW;               // rows staged by an activation wave
  static constexpr int PW = kTileN / 16 / LW;      // weight panels loaded by a weight wave
  static constexpr int Loads = PW + 1;             // its loads per K-block
  static constexpr int A = TM / 32 * kARb;         // a stage
  static constexpr int D = TM == 256 ? 4 : 6;      // weight ring slots
  static constexpr int oRaw = 2 * A;
  static constexpr int oSa = oRaw + TM * 64;
  static constexpr int oRing = oSa + 4 * 4 * TM;
  static constexpr int Lds = oRing + D * kSlot;
  static_assert(TM == 256 || TM == 128, "tile heights");
  static_assert(Lds + kOrderLds + 64 <= 160 * 1024, "LDS");
  static_assert(TM * 136 * 2 <= Lds, "SwiGLU epilogue buffer fits in LDS");
};

// Weights in a ring slot, and an 8-bit block's activation codes in a stage
// (its two K-halves one after the other): 64 bytes per row (or weight column),
// row by row, as a direct load lands them; row r's 16-byte chunk j (of 4) is at
// r * 64 + ((j ^ (r / 4 % 4)) << 4).  The loads read whole rows (four lanes
// each fetch a row's chunks, swizzled), at 56 bytes per cycle and CU where
// 16-row columns of chunks run at 31; and a fragment read of 32 rows and two
// chunks, lane l taking row l % 32, is free of bank conflicts on gfx950, whose
// 16-byte reads are served in groups of lanes 0-3, 12-15, 20-27 and 4-11,
// 16-19, 28-31.
__device__ __forceinline__ int rpos(int r, int j) { return r * 64 + ((j ^ ((r >> 2) & 3)) << 4); }

// A 4-bit block's activation codes in a stage: FP8 bytes in fragment order.
// The 1 KB unit ((rb * 2 + h) * 2 + p) holds, for row block rb and K-half h
// (codes 64 h .. 64 h + 63), 16 bytes per lane: lane l's are codes 64 h + 32
// (l / 32) + 16 p .. + 15 of row 32 rb + l % 32, in place l ^ 2 (l / 32), K-half 1
// 64 bytes further on.  That spreads the writes of the unpacked codes, whose lanes
// hold the four chunks of two rows in eight lanes, over all banks, and leaves the
// reads spread.
__device__ __forceinline__ constexpr int aunit(int rb, int h, int p) {
  return rb * kARb + h * (2048 + 64) + p * 1024;
}

__device__ __forceinline__ i32x8 lds_frag(const uint8_t* p0, const uint8_t* p1) {
  const u32x4 x = *reinterpret_cast<const u32x4*>(p0);
  const u32x4 y = *reinterpret_cast<const u32x4*>(p1);
  i32x8 f;
  f[0] = (int)x[0]; f[1] = (int)x[1]; f[2] = (int)x[2]; f[3] = (int)x[3];
  f[4] = (int)y[0]; f[5] = (int)y[1]; f[6] = (int)y[2]; f[7] = (int)y[3];
  return f;
}

// One K-block position of the schedule is one int of the host's encoding (a
// code): bits 0..9 block index g, bit 10 set for an 8-bit activation block, bits
// 11.. the block's offset in A_packed in units of M*64 bytes.

// The plan (schedule, work units, split table) is read-only while the kernel
// runs.  Reading it through the constant address space keeps its loads on the
// scalar unit: a vector load here would come with a wait on the vector-memory
// counter, which also waits for every weight load in flight.
typedef const __attribute__((address_space(4))) int* cint_ptr;
__device__ __forceinline__ int plan_at(const int* a, int i) {
  return ((cint_ptr)a)[i];
}
__device__ __forceinline__ int order_at(const GemmArgs& p, int i) { return plan_at(p.order, i); }

// The thread index as a value the compiler cannot see through: what is
// computed from it is recomputed at each use (a few VALU operations) instead
// of held in registers across the K-loop, which has none to spare.
__device__ __forceinline__ int opaque_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Direct global -> LDS load of 16 bytes per lane: a scalar base and a 32-bit
// per-lane byte offset; the wave's 64 chunks land at LDS bytes lds .. lds +
// 1023, lane by lane.  Issued as inline assembly so that the compiler does
// not wait for it at LDS reads of other buffers; the K-loop waits for it
// explicitly before the barrier that publishes it.  The load must not follow the
// write of M0 directly, and within inline assembly nothing is put between them
// but what stands there: the s_nop.
__device__ __forceinline__ void dma16(const uint8_t* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
}
// Four kilobytes side by side in LDS, each from its own scalar base: one write of
// M0, and the instruction's offset, which counts for memory and for LDS, so base i
// is 1024 * i short of its kilobyte.  NT: with the non-temporal hint, for data used
// once (the weights of a single row of tiles), which then does not displace the
// activation codes, which every workgroup reads, from L2.
template <bool NT>
__device__ __forceinline__ void dma16_from4(const uint8_t* const (&b)[4], uint32_t voff,
                                            uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\t"
                 "global_load_lds_dwordx4 %0, %2 offset:1024 nt\n\t"
                 "global_load_lds_dwordx4 %0, %3 offset:2048 nt\n\t"
                 "global_load_lds_dwordx4 %0, %4 offset:3072 nt"
                 :: "v"(voff), "s"(b[0]), "s"(b[1]), "s"(b[2]), "s"(b[3]),
                    "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
  else
    asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                 "global_load_lds_dwordx4 %0, %2 offset:1024\n\t"
                 "global_load_lds_dwordx4 %0, %3 offset:2048\n\t"
                 "global_load_lds_dwordx4 %0, %4 offset:3072"
                 :: "v"(voff), "s"(b[0]), "s"(b[1]), "s"(b[2]), "s"(b[3]),
                    "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
}
// dma16 of N kilobytes in a row, in memory and in LDS (the instruction's offset
// counts for both).
template <int N>
__device__ __forceinline__ void dma16_run(const uint8_t* base, uint32_t voff, uint32_t lds) {
  static_assert(N == 2 || N == 4, "runs");
  if constexpr (N == 4)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:2048\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:3072"
                 :: "v"(voff), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:1024"
                 :: "v"(voff), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
}
// 16 bits per lane, zero-extended: lane l's lands at LDS bytes lds + 4 l .. + 3.
__device__ __forceinline__ void dma2(const uint8_t* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_ushort %0, %1"
               :: "v"(voff), "s"(base), "s"(__builtin_amdgcn_readfirstlane(lds)) : "m0");
}

__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Per-lane LDS offsets of a wave's fragments.  The lane holds row (or column)
// lane % 32 of a 32-row block in every fragment.
struct LaneOffsets {
  int a4;   // 4-bit activation fragment, in a stage: (+ aunit(rb, h, p)) ^ (h * 64)
  int a8;   // 8-bit, chunk 2 (lane / 32) + p of a K-half: (+ h * A / 2 + rb * 2048) ^ (p * 16)
  int w;    // weight fragment, in a slot, chunk 2 h + lane / 32: (+ cb * 2048) ^ (h * 32)
  int sa;   // activation scale, in a scale slot: + rb * 128
  int sw;   // weight scale of column wc + lane % 32, in a slot: + cb * 64
};
template <int TM>
__device__ __forceinline__ LaneOffsets lane_offsets() {
  const int lane = opaque_tid() & 63, wave = wave_id();
  using L = Geo<TM>;
  const int wr = wave / L::WCols * L::WM, wc = wave % L::WCols * L::WN;
  const int r = lane & 31;
  LaneOffsets o;
  o.a4 = aunit(wr / 32, 0, 0) + (lane ^ (2 * (lane >> 5))) * 16;
  o.a8 = wr * 64 + rpos(r, 2 * (lane >> 5));
  o.w = wc * 64 + rpos(r, lane >> 5);
  o.sa = 4 * (wr + r);
  o.sw = kWr + 2 * (wc + r);
  return o;
}

// A tile's place and the loads of the weight waves: wave LW + w loads panels
// PW w .. of the tile.  Panels past N are clamped (their outputs are never
// stored).
struct TileLoads {
  int m0, n0;
  const uint8_t* w[4];  // panel i, less 1024 * i (dma16_from4)
};
template <int TM>
__device__ __forceinline__ TileLoads tile_loads(const GemmArgs& p, int m0, int n0) {
  using L = Geo<TM>;
  const int NG = p.K / kG, last = p.N / 16 - 1;
  const int p0 = min(n0 / 16 + L::PW * (wave_id() % L::LW), last);
  static_assert(L::PW == 4, "panels of a weight wave");
  TileLoads t{m0, n0, {}};
  #pragma unroll
  for (int i = 0; i < L::PW; ++i) t.w[i] = p.W + (size_t)min(p0 + i, last) * NG * 1024 - 1024 * i;
  return t;
}

// The direct loads.  Each is a scalar base and a lane offset, with few scalar
// operations on purpose: a wave that computes addresses issues no MFMAs.
//
// Weights of K-block g, by the weight waves: 16 columns of 64 bytes to the
// kilobyte, and the scales of the wave's columns (8 per lane; columns past N
// re-read the last ones).
template <int TM>
__device__ __forceinline__ void load_weights(const GemmArgs& p, const TileLoads& t, int code,
                                             uint32_t slot) {
  using L = Geo<TM>;
  const int w = wave_id() % L::LW, lane = opaque_tid() & 63;
  const uint32_t g = code & 1023;
  const uint32_t off = (lane >> 2) * 64u + ((lane ^ (lane >> 4)) & 3) * 16u + g * 1024u;
  dma16_from4<TM == 128>(t.w, off, slot + L::PW * 1024 * w);
  constexpr int C = kTileN / L::LW;  // columns
  if (lane < C / 8)
    dma16(reinterpret_cast<const uint8_t*>(p.sw + (uint64_t)g * (uint32_t)p.N),
          2u * (uint32_t)min(t.n0 + C * w + 8 * lane, p.N - 8), slot + kWr + 2 * C * w);
}

// Start of a K-block's codes in A_packed, and of its activation scales.
__device__ __forceinline__ const uint8_t* codes_base(const GemmArgs& p, int code) {
  return p.A + (uint64_t)((uint32_t)p.M * 64u) * (uint32_t)(code >> 11);
}
__device__ __forceinline__ const uint8_t* sa_base(const GemmArgs& p, int code) {
  return reinterpret_cast<const uint8_t*>(p.sa + (uint64_t)(uint32_t)(code & 1023) * (uint32_t)p.M);
}

// Activation codes by the activation waves (wave w: rows RW w .. of the tile): of a 4-bit
// block, packed, into the raw area, to be unpacked by the same wave; of an
// 8-bit block, into a stage.  Rows past M re-read row M - 1; byte offsets
// within a block stay below 2^32 (at most 2^21 rows of 128 bytes).
template <int TM>
__device__ __forceinline__ void load_codes4(const GemmArgs& p, const TileLoads& t,
                                            const uint8_t* A, uint32_t raw) {
  constexpr int RW = Geo<TM>::RW;
  const int w = wave_id(), lane = opaque_tid() & 63;
  if (t.m0 + TM <= p.M) {
    dma16_run<RW / 16>(A, (t.m0 + RW * w) * 64u + lane * 16u, raw + RW * w * 64);
  } else {
    const int r = t.m0 + RW * w + (lane >> 2);
    #pragma unroll
    for (int i = 0; i < RW / 16; ++i)
      dma16(A, (uint32_t)min(r + 16 * i, p.M - 1) * 64u + (lane & 3) * 16u,
            raw + RW * w * 64 + 1024 * i);
  }
}
template <int TM>
__device__ __forceinline__ void load_codes8(const GemmArgs& p, const TileLoads& t, int code,
                                            uint32_t stage) {
  constexpr int RW = Geo<TM>::RW;
  const int w = wave_id(), lane = opaque_tid() & 63;
  const uint8_t* A = codes_base(p, code);
  const int r = t.m0 + RW * w + (lane >> 2);
  #pragma unroll
  for (int i = 0; i < RW / 16; ++i)
    #pragma unroll
    for (int h = 0; h < 2; ++h)
      dma16(A, (uint32_t)min(r + 16 * i, p.M - 1) * 128u + 64u * h + ((lane ^ (lane >> 4)) & 3) * 16u,
            stage + h * TM * 64 + RW * w * 64 + 1024 * i);
}
// Activation scales of the same rows, into a scale slot.
template <int TM>
__device__ __forceinline__ void load_sa(const GemmArgs& p, const TileLoads& t, const uint8_t* base,
                                        uint32_t slot) {
  constexpr int RW = Geo<TM>::RW;
  const int w = wave_id(), lane = opaque_tid() & 63;
  if (RW == 64 || lane < RW)
    dma2(base, 2u * (uint32_t)min(t.m0 + RW * w + lane, p.M - 1), slot + 4 * RW * w);
}

// Activation waves: unpack the 4-bit codes that this wave loaded into the raw area
// into activation stage `stage` (see aunit).
template <int TM>
__device__ __forceinline__ void unpack_codes(const uint8_t* raw, uint8_t* stage) {
  constexpr int RW = Geo<TM>::RW;
  const int lane = opaque_tid() & 63, w = wave_id();
  // all reads first: one LDS round trip
  u32x4 v[RW / 16];
  #pragma unroll
  for (int i = 0; i < RW / 16; ++i)
    v[i] = *reinterpret_cast<const u32x4*>(raw + RW * w * 64 + 1024 * i + lane * 16);
  // chunk c = lane % 4 of row 16 i + lane / 4: K-half c / 2, lane half c % 2
  const int c = lane & 3;
  uint8_t* d = stage + aunit(0, c >> 1, 0) + (((c & 1) * 32 + (lane >> 2)) ^ (2 * (c & 1))) * 16;
  #pragma unroll
  for (int i = 0; i < RW / 16; ++i) {
    u32x4 lo, hi;
    unpack4(v[i], lo, hi);
    const int r = RW * w + 16 * i;  // the kilobyte's first row
    uint8_t* q = d + aunit(r >> 5, 0, 0) + ((r >> 4) & 1) * 256;
    *reinterpret_cast<u32x4*>(q) = lo;
    *reinterpret_cast<u32x4*>(q + 1024) = hi;
  }
}

__device__ __forceinline__ void wait_vm_all() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Waits until the loads of at most n K-blocks of weights are in flight in this
// wave (any n; at most D - 2 are).
template <int TM>
__device__ __forceinline__ void wait_w(int n) {
  using L = Geo<TM>;
  static_assert(L::D <= 6, "counts below");
  if (L::D > 5 && n >= 4)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(4 * L::Loads) : "memory");
  else if (L::D > 4 && n >= 3)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(3 * L::Loads) : "memory");
  else if (L::D > 3 && n >= 2)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * L::Loads) : "memory");
  else if (n >= 1)
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(L::Loads) : "memory");
  else
    wait_vm_all();
}

__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Barrier that publishes this wave's LDS writes (ds_write completion) but
// leaves its outstanding global loads in flight.
__device__ __forceinline__ void barrier_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 16 bytes of 4-bit codes (32 channels) -> one MFMA operand of 32 FP8 bytes.
__device__ __forceinline__ i32x8 unpack_frag(u32x4 v) {
  i32x8 f;
  #pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = (int)(v[i] & kSignMag);
    f[2 * i + 1] = (int)(rotr4(v[i]) & kSignMag);
  }
  return f;
}

__device__ __forceinline__ void order_point() { __builtin_amdgcn_sched_barrier(0); }

// Accumulators of a wave's quadrant, in units of 2^-17 (the FP8 code
// encoding, and P = 2 sa sw, see scale_products32), and the block whose
// dequantization is still due, the last one of the K-block before:
// C[NB - 1] += y * P.  Block b is row block b / CB, column block b % CB.
template <int TM>
struct Acc {
  static constexpr int NB = Geo<TM>::NB;
  f32x16 C[NB];
  f32x16 y, P;
  __device__ __forceinline__ void clear_due() {
    #pragma unroll
    for (int i = 0; i < 16; ++i) y[i] = P[i] = 0.f;
  }
  __device__ __forceinline__ void clear() {
    clear_due();
    #pragma unroll
    for (int b = 0; b < NB; ++b) C[b] = f32x16{};
  }
  // elements [I0, I1) of block b += y * P
  template <int I0, int I1>
  __device__ __forceinline__ void dequant(int b) {
    #pragma unroll
    for (int i = I0; i < I1; ++i)
      C[b][i] = __builtin_fmaf(y[i], P[i], C[b][i]);
    // pin the updates here; otherwise the optimizer sinks them and keeps the
    // K-block's MFMA results live
    asm volatile("" : "+v"(C[b]));
  }
  // Adds the block still due (it stays in y and P: follow with clear_due()
  // unless the next K-block overwrites them).
  __device__ __forceinline__ void finish() { dequant<0, 16>(NB - 1); }
};

// Diagnostic form: block b's exact sums (y, units of 2^-18) into the window.
template <int TM>
__device__ __forceinline__ void store_sums(const GemmArgs& p, const f32x16& y, int b, int g, int NG,
                                           int m0, int n0) {
  using L = Geo<TM>;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int row0 = m0 + wave / L::WCols * L::WM + b / L::CB * 32 + 4 * (lane >> 5);
  const int col = n0 + wave % L::WCols * L::WN + b % L::CB * 32 + (lane & 31);
  #pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = row0 + 8 * (i >> 2) + (i & 3);
    if (row >= p.win_m0 && row < p.win_m1 && col >= p.win_n0 && col < p.win_n1) {
      const size_t idx = ((size_t)(row - p.win_m0) * (p.win_n1 - p.win_n0) +
                          (col - p.win_n0)) * NG + g;
      p.acc[idx] = (int32_t)(y[i] * kUnit);
    }
  }
}

// What a wave holds of a K-block when its compute phase starts: the weight
// fragments of its 64 columns and (4-bit blocks) the first row block's
// activation fragments, and the scales.
struct Frags {
  i32x8 wf[2][2];
  i32x8 af[2];
  uint32_t sa, sw[2];  // one fp16 scale each, the upper half zero
};

// The compute phase of one K-block: RB x 2 blocks of 32 x 32 of the wave's
// quadrant, from the fragments in f, the activation stage and the scale slot
// (the lane's offsets added).
//
// Order of issue.  4-bit block: the two MFMAs of block b with the
// dequantization of block b - 1 behind them, then block b's scale products;
// the last block's dequantization stays due.  The first MFMA's share of the
// dequantization is the smaller one, because it also waits for the scale
// products.  8-bit block: twice the MFMAs and the hi/lo split of the codes,
// whose registers leave room for one block's results only, so each block is
// dequantized right after its MFMAs.
template <int TM, bool DIAG, class Hook>
__device__ __forceinline__ void compute4(const uint8_t* a, const uint8_t* sap, Frags& f,
                                         int g, const GemmArgs& p, const TileLoads& t,
                                         Acc<TM>& acc, Hook&& hook) {
  constexpr int RB = Geo<TM>::RB, CB = Geo<TM>::CB, NB = RB * CB;
  if constexpr (!DIAG) acc.P = scale_products32(f.sa, f.sw[0]);
  order_point();
  i32x8 an[2];  // the next row block, read a whole row block ahead
  #pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int rb = b / CB, cb = b % CB;
    const bool last_cb = cb == CB - 1 && rb + 1 < RB;
    f32x16 y = mfma32_fp8(f.af[0], f.wf[cb][0], f32x16{});
    order_point();
    if (cb == 0 && rb + 1 < RB) {
      an[0] = lds_frag(a + aunit(rb + 1, 0, 0), a + aunit(rb + 1, 0, 1));
      if (TM == 128) an[1] = lds_frag(a + aunit(rb + 1, 1, 0), a + aunit(rb + 1, 1, 1));
    }
    // (K-half 1 only half a block ahead in the 256-row tile: registers)
    const i32x8 a1 = f.af[1];
    if (TM == 256 && last_cb) an[1] = lds_frag(a + aunit(rb + 1, 1, 0), a + aunit(rb + 1, 1, 1));
    if constexpr (!DIAG)
      if (b > 0) acc.template dequant<0, 4>(b - 1);
    order_point();
    y = mfma32_fp8(a1, f.wf[cb][1], y);
    order_point();
    if (last_cb) {
      f.af[0] = an[0];
      f.af[1] = an[1];
    }
    if constexpr (DIAG) {
      store_sums<TM>(p, y, b, g, p.K / kG, t.m0, t.n0);
    } else {
      if (b > 0) {
        acc.template dequant<4, 16>(b - 1);
        order_point();
        acc.P = scale_products32(f.sa, f.sw[cb]);
      }
      if (last_cb) f.sa = *reinterpret_cast<const uint32_t*>(sap + (rb + 1) * 128);
      acc.y = y;
    }
    order_point();
    hook(b);
    order_point();
  }
}

template <int TM, bool DIAG, class Hook>
__device__ __forceinline__ void compute8(const uint8_t* const (&a)[2], const uint8_t* sap, Frags& f,
                                         int g, const GemmArgs& p, const TileLoads& t,
                                         Acc<TM>& acc, Hook&& hook) {
  constexpr int RB = Geo<TM>::RB, CB = Geo<TM>::CB, NB = RB * CB, H = TM * 64;
  f.sa = *reinterpret_cast<const uint32_t*>(sap);
  #pragma unroll
  for (int h = 0; h < 2; ++h) f.af[h] = lds_frag(a[0] + h * H, a[1] + h * H);
  i32x8 ah[2];
  #pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int rb = b / CB, cb = b % CB;
    const bool last_cb = cb == CB - 1 && rb + 1 < RB;
    f32x16 y = {};
    if constexpr (!DIAG) acc.P = scale_products32(f.sa, f.sw[cb]);
    if (last_cb) f.sa = *reinterpret_cast<const uint32_t*>(sap + (rb + 1) * 128);
    #pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (cb == 0) {
        #pragma unroll
        for (int i = 0; i < 8; ++i) {
          ah[h][i] = (int)hi8((uint32_t)f.af[h][i]);
          f.af[h][i] = (int)lo8((uint32_t)f.af[h][i]);
        }
      }
      y = mfma32_fp8(f.af[h], f.wf[cb][h], y);
      y = mfma32_fp8_x8(ah[h], f.wf[cb][h], y);  // + 8 * hi, exact
      order_point();
      if (last_cb)
        f.af[h] = lds_frag(a[0] + h * H + (rb + 1) * 2048, a[1] + h * H + (rb + 1) * 2048);
      order_point();
    }
    if constexpr (DIAG) {
      store_sums<TM>(p, y, b, g, p.K / kG, t.m0, t.n0);
    } else {
      acc.y = y;
      acc.template dequant<0, 16>(b);
    }
    order_point();
    hook(b);
    order_point();
  }
}

// K-loop over schedule positions [pos, end), all 4-bit, of a unit [g_begin,
// g_end).  Relative position j = pos - g_begin uses activation stage
// j % 2, scale slot j % 4 and weight ring slot j % D.  An iteration is two
// phases, each ended by a barrier of all eight waves:
//   * prepare (no matrix work): finish the previous K-block's dequantization
//     and read the fragments of j.  Waves 0-3 (LEAD false) also unpack the
//     activation codes of j + 1 into stage (j + 1) % 2 (or start the direct
//     loads of an 8-bit block there) and start the loads of the codes of j + 2
//     into the raw area and of its scales; waves 4-7 (LEAD) start the loads of
//     weights j + D - 1 into the ring;
//   * compute: the MFMAs of j.
// Waves 0-3 run one phase behind waves 4-7, so that on every SIMD one wave
// prepares while the other computes.  In units of phases, waves 4-7 prepare j
// in phase 2 j and compute it in 2 j + 1, waves 0-3 in 2 j + 1 and 2 j + 2.
// What is written while others read:
//   * stage (j + 1) % 2 is written in phase 2 j + 1 (waves 0-3, prepare j);
//     its old content, j - 1, was last read in phase 2 j (waves 0-3, compute
//     j - 1); its new one is first read in phase 2 j + 2;
//   * the direct loads of an 8-bit block that follows the run are waited for at
//     the end of phase 2 j + 2, the run's last;
//   * the raw area belongs, part by part, to the wave that loads and unpacks it;
//   * scale slot (j + 2) % 4 is loaded from phase 2 j + 1 on, waited for in
//     phase 2 j + 3 (waves 0-3, prepare j + 1) and first read in 2 j + 4;
//   * ring slot (j + D - 1) % D is loaded from phase 2 j on (waves 4-7,
//     prepare j); its old content, j - 1, was last read in phase 2 j - 1
//     (waves 0-3, prepare j - 1).  Weights j + 1 are waited for at the end of
//     phase 2 j + 1 and first read in phase 2 j + 2.
template <int TM, bool DIAG, bool LEAD>
__device__ __forceinline__ void kloop_phases(const GemmArgs& p, uint8_t* smem, uint32_t lds,
                                             const int* order, int g_begin, int pos, int end,
                                             int g_end, const TileLoads& t, Acc<TM>& acc) {
  using L = Geo<TM>;
  int j = pos - g_begin;
  int slot = j % L::D;
  // order entries, read one iteration ahead: waves 4-7 need that of j + D - 1,
  // waves 0-3 those of j + 1 and j + 2
  constexpr int kAhead = LEAD ? L::D - 1 : 2;
  int c1 = LEAD ? 0 : __builtin_amdgcn_readfirstlane(order[min(pos + 1, g_end - 1)]);
  int ca = __builtin_amdgcn_readfirstlane(order[min(pos + kAhead, g_end - 1)]);
  const uint8_t* abase = codes_base(p, ca);
  const uint8_t* sbase = sa_base(p, ca);
  for (; pos < end; ++pos, ++j) {
    const LaneOffsets o = lane_offsets<TM>();
    const uint8_t* stage = smem + (j & 1) * L::A;
    const uint8_t* a = stage + o.a4;
    const uint8_t* sap = smem + L::oSa + (j & 3) * 4 * TM + o.sa;
    const uint8_t* w = smem + L::oRing + slot * kSlot;

    // prepare
    Frags f;
    u32x4 raw[Geo<TM>::CB][2];
    #pragma unroll
    for (int cb = 0; cb < Geo<TM>::CB; ++cb) {
      raw[cb][0] = *reinterpret_cast<const u32x4*>(w + o.w + cb * 2048);
      raw[cb][1] = *reinterpret_cast<const u32x4*>(w + (o.w ^ 32) + cb * 2048);
    }
    #pragma unroll
    for (int cb = 0; cb < 2; ++cb) f.sw[cb] = *reinterpret_cast<const uint16_t*>(w + o.sw + 64 * cb);
    f.sa = *reinterpret_cast<const uint32_t*>(sap);
    f.af[0] = lds_frag(a + aunit(0, 0, 0), a + aunit(0, 0, 1));
    f.af[1] = lds_frag(a + aunit(0, 1, 0), a + aunit(0, 1, 1));
    order_point();
    if constexpr (!DIAG) acc.finish();
    order_point();
    #pragma unroll
    for (int cb = 0; cb < Geo<TM>::CB; ++cb)
      #pragma unroll
      for (int h = 0; h < 2; ++h) {
        f.wf[cb][h] = unpack_frag(raw[cb][h]);
        asm volatile("" : "+v"(f.wf[cb][h]));  // here, not sunk into the compute phase
      }
    order_point();
    if (!LEAD && pos + 1 < g_end) {
      wait_vm_all();
      if (!(c1 & 1024))
        unpack_codes<TM>(smem + L::oRaw, smem + ((j & 1) ^ 1) * L::A);
      else
        load_codes8<TM>(p, t, c1, lds + ((j & 1) ^ 1) * L::A);
      order_point();  // the raw area has been read
      if (pos + 2 < g_end) {
        if (!(ca & 1024)) load_codes4<TM>(p, t, abase, lds + L::oRaw);
        load_sa<TM>(p, t, sbase, lds + L::oSa + ((j + 2) & 3) * 4 * TM);
      }
    }
    if (LEAD && pos + L::D - 1 < g_end)
      load_weights<TM>(p, t, ca, lds + L::oRing + (slot == 0 ? L::D - 1 : slot - 1) * kSlot);
    barrier_lds();
    order_point();

    // compute; waves 0-3 also find the addresses of the next loads
    int cn = 0;
    const int g = DIAG ? __builtin_amdgcn_readfirstlane(order[pos]) & 1023 : 0;
    auto hook = [&](int b) {
      if (b == 1) cn = order[min(pos + kAhead + 1, g_end - 1)];
      if (!LEAD && b == 2) {
        c1 = ca;
        ca = __builtin_amdgcn_readfirstlane(cn);
        abase = codes_base(p, ca);
        sbase = sa_base(p, ca);
      }
    };
    const bool next8 = !LEAD && pos + 1 < g_end && (c1 & 1024);
    compute4<TM, DIAG>(a, sap, f, g, p, t, acc, hook);
    if constexpr (LEAD) {
      ca = __builtin_amdgcn_readfirstlane(cn);
      wait_w<TM>(g_end - pos - 2);
    } else {
      if (next8) wait_vm_all();
    }
    barrier_lds();
    order_point();
    slot = slot + 1 == L::D ? 0 : slot + 1;
  }
}

// K-loop as kloop_phases, of precision B8, with all waves in step and one barrier
// per K-block: for the 128-row tile, and for 8-bit blocks, whose longer chains of
// MFMAs and dequantizations the SIMD's two waves fill better side by side.  In
// iteration j waves 0-3 (LEAD false) unpack the activation codes of j + 1, after
// computing, into the stage that j - 1 left free, and start the loads of j + 2;
// waves 4-7 load weights j + D - 1 into the ring slot of j - 1 and wait, at the
// end, for j + 1.
template <int TM, bool DIAG, bool B8, bool LEAD>
__device__ __forceinline__ void kloop_step(const GemmArgs& p, uint8_t* smem, uint32_t lds,
                                            const int* order, int g_begin, int pos, int end,
                                            int g_end, const TileLoads& t, Acc<TM>& acc) {
  using L = Geo<TM>;
  if constexpr (B8) acc.finish();
  const LaneOffsets o = lane_offsets<TM>();
  constexpr int kAhead = LEAD ? L::D - 1 : 2;
  int j = pos - g_begin;
  int slot = j % L::D;
  int c1 = LEAD ? 0 : __builtin_amdgcn_readfirstlane(order[min(pos + 1, g_end - 1)]);
  int ca = __builtin_amdgcn_readfirstlane(order[min(pos + kAhead, g_end - 1)]);
  for (; pos < end; ++pos, ++j) {
    const uint8_t* stage = smem + (j & 1) * L::A;
    const int next_stage = ((j & 1) ^ 1) * L::A;
    const uint8_t* a[2] = {stage + (B8 ? o.a8 : o.a4), stage + (o.a8 ^ 16)};
    const uint8_t* sap = smem + L::oSa + (j & 3) * 4 * TM + o.sa;
    const uint8_t* w = smem + L::oRing + slot * kSlot;
    const bool next8 = !LEAD && pos + 1 < g_end && (c1 & 1024);
    if (next8) load_codes8<TM>(p, t, c1, lds + next_stage);
    Frags f;
    u32x4 raw[2][2];
    f.sa = *reinterpret_cast<const uint32_t*>(sap);
    #pragma unroll
    for (int cb = 0; cb < 2; ++cb) f.sw[cb] = *reinterpret_cast<const uint16_t*>(w + o.sw + 64 * cb);
    raw[0][0] = *reinterpret_cast<const u32x4*>(w + o.w);
    if constexpr (!B8) f.af[0] = lds_frag(a[0] + aunit(0, 0, 0), a[0] + aunit(0, 0, 1));
    raw[0][1] = *reinterpret_cast<const u32x4*>(w + (o.w ^ 32));
    if constexpr (!B8) f.af[1] = lds_frag(a[0] + aunit(0, 1, 0), a[0] + aunit(0, 1, 1));
    raw[1][0] = *reinterpret_cast<const u32x4*>(w + o.w + 2048);
    raw[1][1] = *reinterpret_cast<const u32x4*>(w + (o.w ^ 32) + 2048);
    const int cn = order[min(pos + kAhead + 1, g_end - 1)];
    const int g = DIAG ? __builtin_amdgcn_readfirstlane(order[pos]) & 1023 : 0;
    order_point();
    if constexpr (!DIAG && !B8) acc.finish();
    order_point();
    #pragma unroll
    for (int cb = 0; cb < 2; ++cb)
      #pragma unroll
      for (int h = 0; h < 2; ++h) f.wf[cb][h] = unpack_frag(raw[cb][h]);
    auto hook = [&](int b) {
      if (LEAD && b == 0 && pos + L::D - 1 < g_end)
        load_weights<TM>(p, t, ca, lds + L::oRing + (slot == 0 ? L::D - 1 : slot - 1) * kSlot);
    };
    if constexpr (B8)
      compute8<TM, DIAG>(a, sap, f, g, p, t, acc, hook);
    else
      compute4<TM, DIAG>(a[0], sap, f, g, p, t, acc, hook);
    if constexpr (LEAD) {
      wait_w<TM>(g_end - pos - 2);
    } else if (pos + 1 < g_end) {
      wait_vm_all();
      if (!next8) unpack_codes<TM>(smem + L::oRaw, smem + next_stage);
      order_point();  // the raw area has been read
      if (pos + 2 < g_end) {
        if (!(ca & 1024)) load_codes4<TM>(p, t, codes_base(p, ca), lds + L::oRaw);
        load_sa<TM>(p, t, sa_base(p, ca), lds + L::oSa + ((j + 2) & 3) * 4 * TM);
      }
    }
    barrier_lds();
    order_point();
    c1 = ca;
    ca = __builtin_amdgcn_readfirstlane(cn);
    slot = slot + 1 == L::D ? 0 : slot + 1;
  }
  if constexpr (B8) acc.clear_due();
}

// A work unit's K-blocks: in natural order one K-loop per run of equal
// precision, else the 4-bit run, then the 8-bit run.  The 256-row tile runs in
// alternating phases, the 128-row tile in step: with half the MFMAs between
// barriers the extra barrier costs more than the overlap gives (LLaMA-3-70B
// gate_up at 128 tokens 95.7 us in phases, 84.5 in step), and in step the
// 256-row tile's gate_up at 4096 tokens takes 1863 us against 1783.
template <int TM, bool DIAG, bool NAT, bool LEAD>
__device__ __forceinline__ void run_unit(const GemmArgs& p, uint8_t* smem, uint32_t lds,
                                         const int* order, int g_begin, int g_end,
                                         const TileLoads& t, Acc<TM>& acc) {
  auto run4 = [&](int pos, int end) {
    if constexpr (TM == kTileMSmall) {
      kloop_step<TM, DIAG, false, LEAD>(p, smem, lds, order, g_begin, pos, end, g_end, t, acc);
    } else {
      if (!LEAD) barrier_lds();  // one phase behind waves 4-7
      order_point();
      kloop_phases<TM, DIAG, LEAD>(p, smem, lds, order, g_begin, pos, end, g_end, t, acc);
      if (LEAD) barrier_lds();  // the other waves' last compute phase
      order_point();
    }
  };
  auto run8 = [&](int pos, int end) {
    kloop_step<TM, DIAG, true, LEAD>(p, smem, lds, order, g_begin, pos, end, g_end, t, acc);
  };
  if constexpr (NAT) {
    auto run_end = [&](int pos, bool b8) {
      while (pos < g_end && ((order_at(p, pos) & 1024) != 0) == b8) ++pos;
      return pos;
    };
    for (int pos = g_begin; pos < g_end;) {
      const int mid = run_end(pos, false);
      if (pos < mid) run4(pos, mid);
      acc.finish();  // nothing due from here: no more registers live across the runs
      acc.clear_due();
      pos = run_end(mid, true);
      if (mid < pos) run8(mid, pos);
    }
  } else {
    const int split = min(max(p.n4, g_begin), g_end);
    if (g_begin < split) run4(g_begin, split);
    if (split < g_end) run8(split, g_end);
  }
}

// Row, within the wave's quadrant, of element i of row block rb for lane half
// q2 = lane / 32 (the 32x32 accumulator layout; its column is lane % 32).
__device__ __forceinline__ int block_row(int rb, int q2, int i) {
  return rb * 32 + 8 * (i >> 2) + 4 * q2 + (i & 3);
}

// An accumulator (units of 2^-17) as fp16.
__device__ __forceinline__ uint16_t out_f16(float c) {
  return __half_as_ushort(__float2half_rn(c * (kUnit / 2)));
}

// Epilogue of a work unit: a whole tile is stored as fp16; a split tile
// publishes this slot's fp32 partial, and the last workgroup to arrive adds
// the partials in slot order and stores fp16.
// SwiGLU epilogue (the step after the path, fused): the tile's columns 0-127
// are the gate and 128-255 the up outputs of channels 128 j .. 128 j + 127
// (j = n0 / 256).  The up waves put fp16(up) into LDS, the gate waves turn
// each entry into h = SiLU(fp16(gate)) * up (fp16), and then 16 lanes per row
// quantize the row's 128 channels of h as the activation quantizer does,
// into block j of the next layer's A_packed.  `lds` is free by now.
template <int TM>
__device__ __forceinline__ void swiglu_tile(const GemmArgs& p, int m0, int n0,
                                            const f32x16 (&C)[Geo<TM>::NB], uint8_t* lds) {
  using L = Geo<TM>;
  constexpr int kHalf = L::WCols / 2;  // waves over the gate columns
  constexpr int kHP = 136;  // row pitch in halves: 128 channels + 16 bytes
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c32 = lane & 31, q2 = lane >> 5;
  const int wr = wave / L::WCols * L::WM, wq = wave % L::WCols;
  uint16_t* H = reinterpret_cast<uint16_t*>(lds);
  __syncthreads();
  if (wq >= kHalf) {
    #pragma unroll
    for (int b = 0; b < L::NB; ++b)
      #pragma unroll
      for (int i = 0; i < 16; ++i)
        H[(wr + block_row(b / L::CB, q2, i)) * kHP + (wq - kHalf) * L::WN + b % L::CB * 32 + c32] =
            out_f16(C[b][i]);
  }
  __syncthreads();
  if (wq < kHalf) {
    #pragma unroll
    for (int b = 0; b < L::NB; ++b)
      #pragma unroll
      for (int i = 0; i < 16; ++i) {
        uint16_t* h =
            H + (wr + block_row(b / L::CB, q2, i)) * kHP + wq * L::WN + b % L::CB * 32 + c32;
        *h = swiglu_f16(out_f16(C[b][i]), *h);
      }
  }
  __syncthreads();
  const int j = n0 / kTileN;
  const bool b8 = (p.out_map.bits[j >> 6] >> (j & 63)) & 1;
  const size_t base = (size_t)p.M * 64 * (size_t)(j + n8_before(p.out_map, j));
  const int lane16 = threadIdx.x & 15;
  for (int r = threadIdx.x >> 4; r < TM; r += L::Threads / 16) {
    float x[8];
    load8(H + r * kHP + 8 * lane16, x);
    float a = 0.0f;
    #pragma unroll
    for (int i = 0; i < 8; ++i) a = fmaxf(a, fabsf(x[i]));
    a = max16(a);
    Codes c;
    const uint16_t s16 = quantize8(x, a, b8 ? 127.0f : 7.0f, c);
    const int m = m0 + r;
    if (m >= p.M) continue;
    if (b8)
      *reinterpret_cast<uint2*>(p.out_A + base + (size_t)m * 128 + 8 * lane16) = pack8(c);
    else
      *reinterpret_cast<uint32_t*>(p.out_A + base + (size_t)m * 64 + 4 * lane16) = pack4(c);
    if (lane16 == 0) p.out_sa[(size_t)j * p.M + m] = s16;
  }
}

template <int TM, bool SWIGLU>
__device__ __forceinline__ void store_tile(const GemmArgs& p, const WorkUnit& unit, int m0, int n0,
                                           f32x16 (&C)[Geo<TM>::NB], int* s_last,
                                           uint8_t* lds) {
  using L = Geo<TM>;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int c32 = lane & 31, q2 = lane >> 5;
  const int wr = wave / L::WCols * L::WM, wc = wave % L::WCols * L::WN;
  if (unit.nslots > 1) {
    // Split tile.  Each slot publishes its fp32 partial and counts in;
    // whichever counts in last adds the partials in slot order.  A tile of
    // two slots needs only the other slot's partial: the plan puts the
    // first slot early in its workgroup's list and the second at the end, so
    // the second usually finds the first arrived and then skips publishing
    // its own.  One device-scope release and one acquire per tile slot, by
    // one thread: on this multi-XCD part each is a write-back or invalidate
    // of the whole L2, too costly to issue from every wave.
    const int base = plan_at(p.split_index, unit.tile);
    const bool pair = unit.nslots == 2;
    if (threadIdx.x == 0) {
      *s_last = pair && __hip_atomic_load(p.counters + base, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) == 1;
      if (*s_last) __threadfence();  // acquire the other slot's partial
    }
    __syncthreads();
    if (!*s_last) {
      float* part = p.partials + (size_t)(base + unit.slot) * (TM * kTileN);
      #pragma unroll
      for (int b = 0; b < L::NB; ++b)
        #pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(part + (((wave * L::NB + b) * 4 + q) * 64 + lane) * 4) =
              f32x4{C[b][4 * q], C[b][4 * q + 1], C[b][4 * q + 2], C[b][4 * q + 3]};
      // the barrier orders every wave's partial stores before the first thread's
      // device-scope release below
      __syncthreads();
      if (threadIdx.x == 0) {
        __threadfence();
        const bool last = atomicAdd(p.counters + base, 1) == unit.nslots - 1;
        if (last) __threadfence();
        *s_last = last;
      }
      __syncthreads();
      if (!*s_last) return;
    }
    // A pair adds the other slot's partial to its registers (two terms: the
    // same sum whichever slot adds it); otherwise all partials in slot order.
    const int s_first = pair ? unit.slot ^ 1 : 0;
    const int s_end = pair ? s_first + 1 : unit.nslots;
    if (!pair) {
      #pragma unroll
      for (int b = 0; b < L::NB; ++b) C[b] = f32x16{};
    }
    for (int s = s_first; s < s_end; ++s) {
      const float* src = p.partials + (size_t)(base + s) * (TM * kTileN);
      #pragma unroll
      for (int b = 0; b < L::NB; ++b) {
        #pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(
              src + (((wave * L::NB + b) * 4 + q) * 64 + lane) * 4);
          #pragma unroll
          for (int i = 0; i < 4; ++i) C[b][4 * q + i] += v[i];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (threadIdx.x == 0) p.counters[base] = 0;  // ready for the next launch
  }
  if constexpr (SWIGLU) {
    swiglu_tile<TM>(p, m0, n0, C, lds);
    return;
  }
  #pragma unroll
  for (int b = 0; b < L::NB; ++b) {
    const int col = n0 + wc + b % L::CB * 32 + c32;
    #pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = m0 + wr + block_row(b / L::CB, q2, i);
      if (row < p.M && col < p.N) p.out[(size_t)row * p.N + col] = out_f16(C[b][i]);
    }
  }
}

// NAT: the schedule lists the K-blocks in the map's own order (the ablation
// baseline without tile remapping); otherwise all 4-bit blocks come first.
template <int TM, bool DIAG, bool SWIGLU, bool NAT>
__global__ __launch_bounds__(Geo<TM>::Threads) void gemm_kernel(GemmArgs p) {
  using L = Geo<TM>;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  __shared__ int s_last;
  __shared__ int s_order[kMaxBlocks];
  const int NG = p.K / kG;
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
  const int u_end = plan_at(p.wg_begin, blockIdx.x + 1);
  for (int i = threadIdx.x; i < NG; i += L::Threads) s_order[i] = p.order[i];
  __syncthreads();

  const bool lead = wave_id() >= L::LW;
  // The unit whose first K-block loads are in flight: they are issued before
  // the previous unit's epilogue, so their latency overlaps its stores.
  WorkUnit unit{};
  TileLoads t{};
  auto issue = [&](int uu) {
    const int* ue = reinterpret_cast<const int*>(p.units) + 5 * uu;
    unit = WorkUnit{plan_at(ue, 0), plan_at(ue, 1), plan_at(ue, 2), plan_at(ue, 3),
                    plan_at(ue, 4)};
    t = tile_loads<TM>(p, (unit.tile / p.tiles_n) * TM, (unit.tile % p.tiles_n) * kTileN);
    if (lead) {
      for (int d = 0; d < min(L::D - 1, unit.g_end - unit.g_begin); ++d)
        load_weights<TM>(p, t, order_at(p, unit.g_begin + d), lds + L::oRing + d * kSlot);
    } else {
      const int c0 = order_at(p, unit.g_begin);
      if (c0 & 1024)
        load_codes8<TM>(p, t, c0, lds);
      else
        load_codes4<TM>(p, t, codes_base(p, c0), lds + L::oRaw);
      load_sa<TM>(p, t, sa_base(p, c0), lds + L::oSa);
    }
  };
  int u = plan_at(p.wg_begin, blockIdx.x);
  if (u < u_end) issue(u);
  for (; u < u_end; ++u) {
    Acc<TM> acc;
    acc.clear();
    // the unit's first K-block in place, its second's activations on their way
    if (lead) {
      wait_w<TM>(min(unit.g_end - unit.g_begin - 1, L::D - 2));
      barrier_lds();
      order_point();
      run_unit<TM, DIAG, NAT, true>(p, smem, lds, s_order, unit.g_begin, unit.g_end, t, acc);
    } else {
      wait_vm_all();
      if (!(order_at(p, unit.g_begin) & 1024)) unpack_codes<TM>(smem + L::oRaw, smem);
      if (unit.g_begin + 1 < unit.g_end) {
        const int c1 = order_at(p, unit.g_begin + 1);
        wait_lds();
        order_point();
        if (!(c1 & 1024)) load_codes4<TM>(p, t, codes_base(p, c1), lds + L::oRaw);
        load_sa<TM>(p, t, sa_base(p, c1), lds + L::oSa + 4 * TM);
      }
      barrier_lds();
      order_point();
      run_unit<TM, DIAG, NAT, false>(p, smem, lds, s_order, unit.g_begin, unit.g_end, t, acc);
    }
    const WorkUnit cur = unit;
    const int m0 = t.m0, n0 = t.n0;
    if (!SWIGLU && u + 1 < u_end) issue(u + 1);  // LDS is free
    if (DIAG) continue;

    acc.finish();
    store_tile<TM, SWIGLU>(p, cur, m0, n0, acc.C, &s_last, smem);
    if (SWIGLU && u + 1 < u_end) {
      __syncthreads();  // that epilogue works in LDS
      issue(u + 1);
    }
  }
}

typedef void (*GemmKernelFn)(GemmArgs);

// The instantiations: production (plain, diagnostic; the SwiGLU epilogue for
// 128-row tiles only) and the natural-order ablation (plain, diagnostic), for
// both tile heights.  nullptr: not instantiated.
template <int TM>
GemmKernelFn gemm_kernel_of(bool diag, bool swiglu, bool natural) {
  if (natural) {
    if (swiglu) return nullptr;
    return diag ? gemm_kernel<TM, true, false, true> : gemm_kernel<TM, false, false, true>;
  }
  if (diag) return gemm_kernel<TM, true, false, false>;
  if (!swiglu) return gemm_kernel<TM, false, false, false>;
  if constexpr (TM == kTileMSmall) return gemm_kernel<TM, false, true, false>;
  return nullptr;  // the 256-row kernel's SwiGLU runs as its own kernel
}

GemmKernelFn gemm_kernel_fn(int tile_m, bool diag, bool swiglu, bool natural) {
  return tile_m == kTileMSmall ? gemm_kernel_of<kTileMSmall>(diag, swiglu, natural)
                               : gemm_kernel_of<kTileM>(diag, swiglu, natural);
}

}  // namespace

int gemm_lds_bytes(int tile_m) {
  return tile_m == kTileMSmall ? Geo<kTileMSmall>::Lds : Geo<kTileM>::Lds;
}

hipError_t launch_gemm(const GemmArgs& a, int num_wgs, bool diag, bool swiglu, bool natural,
                       int tile_m, hipStream_t stream) {
  const GemmKernelFn fn = gemm_kernel_fn(tile_m, diag, swiglu, natural);
  if (!fn) return hipErrorInvalidValue;  // not instantiated
  hipLaunchKernelGGL(fn, dim3(num_wgs),
                     dim3(tile_m == kTileMSmall ? Geo<kTileMSmall>::Threads : Geo<kTileM>::Threads),
                     gemm_lds_bytes(tile_m), stream, a);
  return hipGetLastError();
}

hipError_t set_gemm_attributes() {
  for (int tm : {kTileM, kTileMSmall})
    for (int v = 0; v < 5; ++v) {
      const bool diag = v == 1 || v == 4, swiglu = v == 2, natural = v >= 3;
      const GemmKernelFn fn = gemm_kernel_fn(tm, diag, swiglu, natural);
      if (!fn) continue;
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         gemm_lds_bytes(tm));
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

}  // namespace comet
