// Chip-wide variants of the two device-side loops, for shapes whose
// recurrent weights need more than one XCD (bf16 H in (1024, 2048], f32 H in
// (512, 1024], at most 256 sequences).  The weights stay in LDS for the whole
// loop, split over the work-groups of the chip, and the loop state crosses
// XCDs every step.
//
// Forward split.  A work-group takes the gate columns of KPC hidden units (8
// bf16, 4 f32) over the whole reduction, so nothing but h_t crosses
// work-groups: it streams all of h_{t-1} and its product needs no partner.
// Gradient split.  The reduction is four times as long there (K = 4H), so the
// output columns are cut into groups of 64 units and the reduction into KG
// slices (8 bf16, 16 f32); work-group (group, slice) holds a slice of H/32
// k-steps x 64 columns (64 H bytes of LDS) and runs the cell of CW of the
// group's units.  A group's KG work-groups sit on one XCD.
//
// Inside a work-group every wave runs the recurrence of its own rows alone:
// the batch is cut into groups of 32 rows, wave w takes row group w % RW and
// share w / RW of the work-group's reduction (RW KW = 8; c_kernels says how
// many and why, and where the float32 forward has sixteen waves).  No barrier stands in a
// step: the shares meet in LDS behind flags (forward) or as partial products
// of the group, like the KG slices (gradient), and the waves of a SIMD hide
// each other's waits.  Measured: the forward loop with a reduction split over
// KG = 2 / 4 work-groups and their partial products in the L2 took, per step,
// bf16 H = 2048 18.0 us (B = 64), 23.9 (128), H = 1536 15.7 (64), 19.1 (128),
// f32 H = 640 16.4 (64), 15.2 (128); with the whole reduction per work-group
// 11.7, 14.3, 10.0, 11.3, 10.4, 11.8.  Above 128 rows, where every work-group
// then streams up to 1 MB a step, the two are closer (inference of 40 steps,
// I = 512, split and whole: bf16 H = 2048 B = 160 913 and 846 us, 192 994 and
// 919, 256 1215 and 1157, H = 1536 B = 256 967 and 771; f32 H = 1024 B = 160
// 1192 and 1050, 224 1342 and 1384, 256 1444 and 1432).
//
// One step of a forward wave:
//   wait for the producers of its k-steps of h_{t-1} (the next step's input
//   projections are asked for first: left to the end of the product, the
//   publish waited for them, 2-3 us a step at 128 rows), stream the k-steps
//   from the exchange ring (device-scope loads, 8 k-steps of 2 KB in flight)
//   against the weights in LDS, add the shares, run the cell, store h_t into
//   the ring with device-scope stores (written through to where every XCD's
//   loads see it), set the wave's exchange flag; then the h history, stack
//   and y.
// One step of a gradient wave:
//   phase B': wait for the KG KW partial products of its column group, sum
//     them for its share of the cells, run the cell, dz into the ring, flag;
//   phase A': wait for the producers of its k-steps of dz_t, stream them
//     against the weights (32x32 MFMAs), store the 32 x 64 partial product
//     into the XCD's L2 and set the wave's partial flag.
//
// What is reused when.  Ring slot t % 2 is rewritten at step t + 2 (t - 2) by
// a cell wave whose shares have, taken together, waited for the exchange
// flags of step t + 1 (t - 1) of every producer of the row group, each set
// after all the shares of its work-group read slot t % 2.  Forward, a share's
// LDS slot is rewritten once the cell wave's flag says that it has read it.
// Gradient, there is one partial slot: a wave stores its partial of step t
// only after every wave of its column group has set its exchange flag of step
// t, which follows the reads of the previous partial.  Every wait has the
// loop's wall-clock limit and abort flag.
//
// Exchange blocks are 1 KB.  Forward: 16 rows of one k-step (32 bf16 or 16
// f32 columns), lane l's 16 bytes being row l % 16, chunk l / 16.  Gradient:
// 32 rows of 16 bf16 or 8 f32 columns, row l % 32, chunk l / 32.  The
// reduction runs over units forward and over 4 unit + gate in the gradient,
// so a unit's four dz values are adjacent.  W^T rows, the input projection's
// columns and the stack's gate values are in the same 4 unit + gate order:
// one 16-byte access per row and unit.
//
// Bound at bf16 H = 2048, B = 256, per step and compute unit: forward 1 MB of
// exchange blocks from the L2 (8.7 us at the measured 50 B/clk; the counters
// show 15 % of these requests waiting for a line on its way from the other
// XCDs), gradient 512 KB; 1 MB of LDS weight reads (3.4 us at 128 B/clk)
// beside 33.5 MFLOP (3.4 us).  A step of few rows is bound by the exchange
// itself: 7-8 us from one publish to the next at 32 rows.
#include <type_traits>

#include "ll_kernels.h"
#include "ll_exchange.h"

namespace ll {

namespace {

constexpr int CNW = 8;
constexpr int CNT = 64 * CNW;
constexpr int kPartFloats = 32 * 64;   // a wave's partial product
constexpr int kScratch = 2048;         // LDS bytes of a wave's layout changes

typedef __attribute__((ext_vector_type(16))) float f32x16;

// One k-step: every lane supplies a 16-byte chunk of A and of B (f32: four
// 32x32x2 MFMAs; element j of the lane's chunk is its k-slot in the j-th).
template <typename T>
__device__ __forceinline__ f32x16 mfma32(uint4 a, uint4 b, f32x16 c);
template <>
__device__ __forceinline__ f32x16 mfma32<bf16_t>(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                c, 0, 0, 0);
}
template <>
__device__ __forceinline__ f32x16 mfma32<float>(uint4 a, uint4 b, f32x16 c) {
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
  return c;
}

// The gradient's split.  KG: reduction slices; KW: waves that share a slice.
template <typename T, int KG_, int KW_>
struct CShape {
  static constexpr int KPC = Op<T>::kPerChunk;
  static constexpr int KG = KG_, KW = KW_;
  static constexpr int NGX = 32 / KG;          // column groups per XCD
  static constexpr int CW = KPC;               // cell units per work-group: one 16-byte chunk
  static constexpr int RW = CNW / KW;          // row groups
  static constexpr int RPK = 32 / KW;          // rows of a wave's cells
  static constexpr int RPL = CW * RPK > 64 ? CW * RPK / 64 : 1;   // rows per lane
  static constexpr int NP = KG * KW;           // partials of a column group
  static_assert(RPL == 1 || RPL == 2 || RPL == 4, "rows per lane");
  static_assert(NP <= 64, "one lane per partial flag");
};

__device__ __forceinline__ void c_fail(const CLoopArgs& a) {
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_or(a.err, LL_DEVERR_BARRIER_BIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Wait until flags[0 .. n) are all >= need, 64 at a time.
__device__ __forceinline__ void wait_range(const CLoopArgs& a, const unsigned* flags, int n, unsigned need) {
  const int lane = threadIdx.x & 63;
  unsigned long long t0 = 0;
  unsigned polls = 0;
  for (int i0 = 0; i0 < n;) {
    const bool mine = i0 + lane < n;
    const unsigned f =
        __hip_atomic_load(flags + (mine ? i0 + lane : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_ballot_w64(mine && f < need) == 0) {
      i0 += 64;
      continue;
    }
    if (polls == 0) t0 = wall_clock64();
    __builtin_amdgcn_s_sleep(1);
    if ((++polls & 255u) == 0) {
      if (__hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
      if (wall_clock64() - t0 > a.limit) {
        __hip_atomic_fetch_or(a.err, LL_DEVERR_BARRIER_BIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
      }
    }
  }
}

// LDS layout changes within one wave: its earlier LDS writes are ordered
// before its later reads (the hardware runs a wave's LDS operations in
// order; the fence keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void st16_dev(__amdgpu_buffer_rsrc_t r, unsigned off, uint4 v) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.x, v.y, v.z, v.w}, r, off, 0, kCpolStoreDev);
}

// k-steps of a wave's loop body and so of its loads in flight: a share is
// padded to whole bodies (with zero weights, and zeros for ring blocks).
template <typename T>
constexpr int c_unroll() { return sizeof(T) == 2 ? 8 : 4; }
template <typename T>
__host__ __device__ constexpr int c_share(int KS, int KW, int U = c_unroll<T>()) {   // padded k-steps of a share of the slice
  const int n = (KS + KW - 1) / KW;
  return (n + U - 1) / U * U;
}

// The wave's partial product: acc[ct] += ring blocks (rs, 1 KB each, zeros
// past the range) times the weight k-steps [0, U ng) in LDS (two column tiles
// of 1 KB each), in groups of U from group `rot` on, around: the work-groups
// of an XCD all read the same freshly written blocks, and each starts
// elsewhere so that they do not all wait for the same misses.  A block's
// registers are refilled as soon as its products are issued, and the weights
// come from LDS two k-steps ahead (left to the compiler, every pair of
// products waited for its own LDS reads: 218 clocks a k-step instead of 64).
// `behind` runs once the last blocks have been asked for.
template <typename T, typename Behind>
__device__ __forceinline__ void c_product(__amdgpu_buffer_rsrc_t rs, const uint4* w, int ng, int rot,
                                          f32x16 (&acc)[2], Behind behind) {
  constexpr int U = c_unroll<T>();
  const int lane = threadIdx.x & 63;
  uint4 b[U], wv[2][4];
  const uint4* wl = w + lane;
  auto rd = [&](uint4 (&v)[4], int g, int c) {   // weights of k-steps 2c, 2c + 1 of group g
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = wl[(g * U + 2 * c) * 128 + i * 64];
  };
  int cur = rot % ng;
#pragma unroll
  for (int i = 0; i < U; ++i) b[i] = ld_chunk_l2(rs, (unsigned)(((cur * U + i) << 10) + lane * 16));
  rd(wv[0], cur, 0);
  for (int left = ng; left > 0; --left) {
    const int nxt = cur + 1 < ng ? cur + 1 : 0;
    if (left == 1) behind();
#pragma unroll
    for (int c = 0; c < U / 2; ++c) {
      rd(wv[(c + 1) & 1], c + 1 < U / 2 ? cur : nxt, c + 1 < U / 2 ? c + 1 : 0);
      __builtin_amdgcn_sched_barrier(0);
      const uint4(&v)[4] = wv[c & 1];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        acc[0] = mfma32<T>(b[2 * c + k], v[2 * k], acc[0]);
        acc[1] = mfma32<T>(b[2 * c + k], v[2 * k + 1], acc[1]);
        // (the last group asks past the range: no traffic)
        b[2 * c + k] = ld_chunk_l2(rs, left > 1 ? (unsigned)(((nxt * U + 2 * c + k) << 10) + lane * 16) : kOOB);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  }
}

// Partial product of a wave to memory: element (column c, row r) at float
// ((((c/32) 4 + r/8) 32 + c%32) 2 + (r/4)%2) 4 + r%4, the result registers'
// own order, so that each store instruction writes 1 KB in one piece.
__device__ __forceinline__ unsigned part_off(int c, int r) {
  return (unsigned)((((((c >> 5) * 4 + (r >> 3)) * 32 + (c & 31)) * 2 + ((r >> 2) & 1)) * 4 + (r & 3)) * 4);
}
__device__ __forceinline__ void store_partial(float* p, const f32x16 (&acc)[2]) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, hf = lane >> 5;
  float4* p4 = reinterpret_cast<float4*>(p);
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      p4[((ct * 4 + q) * 32 + l32) * 2 + hf] =
          make_float4(acc[ct][4 * q], acc[ct][4 * q + 1], acc[ct][4 * q + 2], acc[ct][4 * q + 3]);
}
// RPL consecutive rows of one column of a partial.
template <int RPL>
__device__ __forceinline__ void load_partial(__amdgpu_buffer_rsrc_t r, unsigned off, float (&v)[RPL]) {
  if constexpr (RPL == 4) {
    const uint4 u = ld_chunk_l2(r, off);
    v[0] = __uint_as_float(u.x);
    v[1] = __uint_as_float(u.y);
    v[2] = __uint_as_float(u.z);
    v[3] = __uint_as_float(u.w);
  } else if constexpr (RPL == 2) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 u = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kCpolSc1));
    v[0] = __uint_as_float(u.x);
    v[1] = __uint_as_float(u.y);
  } else {
    v[0] = ld_f32_l2(r, off);
  }
}

// Length of the row group's longest row (its first: rows are in length
// order), capped at the trip count (0 when the lengths failed the range check).
__device__ __forceinline__ int group_len(const CLoopArgs& a, int rg, int T_eff) {
  if (rg * 32 >= a.B || T_eff <= 0) return 0;
  return uni(min(T_eff, a.seq_len[a.perm[rg * 32]]));
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward loop, chip-wide.  Work-group wg owns KPC hidden units (8 bf16, 4
// f32): the 16 NT gate columns of the whole reduction.  The weights are the
// first matrix-core operand, rows 4 unit + gate, and the 32 batch rows of a
// wave (RTL row tiles of 16: one for at most 16 rows) the columns, so a result register quad is the four gates of one
// (row, unit): the cell runs where the product ends.  One product step for
// lane 16 q + l: rows l of the two row tiles, units NT q .. NT q + NT - 1.
// ---------------------------------------------------------------------------
// k-steps (2 KB of ring blocks each) of a wave's loop body and in flight.  A
// share is padded to whole bodies: float32's short shares (KW >= 4) take 4,
// for there the products of the padding cost more than the loads in flight
// give (H = 640, B = 64 11.2 us a step with 8, 10.4 with 4; H = 1024 equal;
// the longer shares of B = 128, H = 1024 17.3 with 8, 19.9 with 4), and so do
// sixteen waves, which have 128 registers each.
template <typename T, int KW, int NW>
constexpr int cfwd_unroll() { return sizeof(T) == 4 && (KW >= 4 || NW == 16) ? 4 : 8; }
template <typename T, int KW_, int RTL_, int NW_ = 8>
struct CFwd {
  static constexpr int KPC = Op<T>::kPerChunk;
  static constexpr int KW = KW_, RTL = RTL_;     // shares; row tiles of a row group
  static constexpr int NW = NW_;
  static constexpr int RW = NW / KW;             // row groups
  static constexpr int NT = KPC / 4;             // weight tiles: units per lane and row
  static constexpr int NCF = KW == 1 ? 1 : RTL;  // cell waves (exchange flags) per row group
  static constexpr int RT = RTL / NCF;           // row tiles of a cell wave
};
// LDS of the forward kernel: weights, the shares' partial products on their
// way to the cell waves, the flags of that hand-over.
template <typename T, int KW, int NW>
__host__ __device__ constexpr int cfwd_weight_chunks(int KS) {
  return KW * c_share<T>(KS, KW, cfwd_unroll<T, KW, NW>()) * CFwd<T, KW, 2, NW>::NT * 64;
}
template <typename T, int KW, int NW>
__host__ __device__ constexpr int cfwd_part_chunks() {
  return CFwd<T, KW, 2, NW>::RW * 2 * (KW - 1) * CFwd<T, KW, 2, NW>::NT * 64;
}
template <typename T, int KW, int NW>
constexpr size_t cfwd_lds(int H) {
  const int KS = H / (4 * Op<T>::kPerChunk);
  return (size_t)(cfwd_weight_chunks<T, KW, NW>(KS) + cfwd_part_chunks<T, KW, NW>()) * 16 + 3 * NW * 4;
}

// Wait until the n <= 256 flags of the range are all >= need (n % 4 == 0, 16
// bytes per lane and poll).  A lane whose flags are there asks no more: every
// wave of the chip polls, beside the ring's loads (f32 H = 1024, inference of
// 40 steps, B = 64 643 -> 606 us, B = 128 810 -> 774; bf16 equal).
__device__ __forceinline__ void wait_quads(const CLoopArgs& a, __amdgpu_buffer_rsrc_t flags, int n, unsigned need) {
  const int lane = threadIdx.x & 63;
  bool mine = lane * 4 < n;
  unsigned long long t0 = 0;
  unsigned polls = 0;
  while (true) {
    const uint4 f = ld_chunk_l2(flags, mine ? (unsigned)(lane * 16) : kOOB);
    const bool late = mine && (f.x < need || f.y < need || f.z < need || f.w < need);
    if (__builtin_amdgcn_ballot_w64(late) == 0) break;
    mine = late;
    if (polls == 0) t0 = wall_clock64();
    __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");   // (every poll loads again)
    if ((++polls & 255u) == 0) {
      if (__hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      if (wall_clock64() - t0 > a.limit) {
        __hip_atomic_fetch_or(a.err, LL_DEVERR_BARRIER_BIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
  }
  asm volatile("" ::: "memory");
}
// The same for flags in LDS, one per lane with `mine` set.
__device__ __forceinline__ void wait_lds(const CLoopArgs& a, const unsigned* flags, int idx, bool mine, unsigned need) {
  unsigned long long t0 = 0;
  unsigned polls = 0;
  while (true) {
    const unsigned f = __hip_atomic_load(flags + (mine ? idx : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__builtin_amdgcn_ballot_w64(mine && f < need) == 0) break;
    if (polls == 0) t0 = wall_clock64();
    __builtin_amdgcn_s_sleep(1);
    if ((++polls & 255u) == 0) {
      if (__hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
      if (wall_clock64() - t0 > a.limit) {
        __hip_atomic_fetch_or(a.err, LL_DEVERR_BARRIER_BIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ void set_lds(unsigned* flag, unsigned value) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The wave's product: acc[nt][rt] += weight tile nt (LDS, NT KB per k-step)
// times row tile rt of the ring blocks (rs, 2 KB per k-step, zeros past the
// range), k-steps [0, U ng) in groups of U from group `rot` on, around (the
// work-groups of an XCD read the same freshly written blocks and start
// apart).  Even and odd k-steps sum apart (half the length of a rounding
// chain).
template <typename T, int NT, int RTL, int U>
__device__ __forceinline__ void cfwd_product(__amdgpu_buffer_rsrc_t rs, const uint4* w, int ng, int rot,
                                             f32x4 (&acc)[NT][RTL]) {
  const int lane = threadIdx.x & 63;
  uint4 b[U][RTL], wv[2][2 * NT];
  f32x4 s[2][NT][RTL];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int rt = 0; rt < RTL; ++rt) s[k][n][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint4* wl = w + lane;
  auto rd = [&](uint4 (&v)[2 * NT], int g, int c) {   // weights of k-steps 2c, 2c + 1 of group g
#pragma unroll
    for (int i = 0; i < 2 * NT; ++i) v[i] = wl[((g * U + 2 * c) * NT + i) * 64];
  };
  int cur = rot % ng;
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int rt = 0; rt < RTL; ++rt)
      b[i][rt] = ld_chunk_l2(rs, (unsigned)(((cur * U + i) * 2 + rt) << 10) + lane * 16);
  rd(wv[0], cur, 0);
  for (int left = ng; left > 0; --left) {
    const int nxt = cur + 1 < ng ? cur + 1 : 0;
#pragma unroll
    for (int c = 0; c < U / 2; ++c) {
      rd(wv[(c + 1) & 1], c + 1 < U / 2 ? cur : nxt, c + 1 < U / 2 ? c + 1 : 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int i = 2 * c + k;
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int rt = 0; rt < RTL; ++rt) s[k][n][rt] = Mfma<T>::step(wv[c & 1][k * NT + n], b[i][rt], s[k][n][rt]);
        // (the last group asks past the range: no traffic)
#pragma unroll
        for (int rt = 0; rt < RTL; ++rt)
          b[i][rt] = ld_chunk_l2(rs, left > 1 ? (unsigned)(((nxt * U + i) * 2 + rt) << 10) + lane * 16 : kOOB);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
  }
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int rt = 0; rt < RTL; ++rt) acc[n][rt] = s[0][n][rt] + s[1][n][rt];
}

template <typename T, int KW, int RTL, int NW>
__global__ __launch_bounds__(64 * NW, 1) void cfwd_kernel(CLoopArgs a) {
  using S = CFwd<T, KW, RTL, NW>;
  constexpr int KPC = S::KPC, RW = S::RW, NT = S::NT, RT = S::RT, NCF = S::NCF, U = cfwd_unroll<T, KW, NW>();
  extern __shared__ uint4 lds[];
  const int H = a.H, B = a.B, RGN = a.RGN;
  const int wg = blockIdx.x, jb = wg * KPC;
  if (RGN > RW || H > 256 * KPC || jb >= H) {
    if (jb < H) c_fail(a);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int q = lane >> 4, l16 = lane & 15;
  const int KS = H / (4 * KPC), KSP = c_share<T>(KS, KW, cfwd_unroll<T, KW, NW>());   // k-steps; of a share, padded
  const long G4 = 4L * H, H5 = 5L * H;
  uint4* parts = lds + cfwd_weight_chunks<T, KW, NW>(KS);
  unsigned* pf = reinterpret_cast<unsigned*>(parts + cfwd_part_chunks<T, KW, NW>());   // [wave]: partials stored
  unsigned* rf = pf + NW;                                                          // [row group][row tile]: read
  if (tid < 3 * NW) pf[tid] = 0u;
  {
    // weights: row m of tile n is gate m % 4 of unit NT (m / 4) + n
    const T* WT = reinterpret_cast<const T*>(a.W) + a.woff;
    for (int i = tid; i < KW * KSP * NT * 64; i += 64 * NW) {
      const int l = i & 63, m = l & 15, n = (i >> 6) % NT, kk = (i >> 6) / NT, sh = kk / KSP;
      const int ks = sh * KS / KW + kk - sh * KSP;
      lds[i] = ks < (sh + 1) * KS / KW
                   ? ld16(WT + (4L * (jb + NT * (m >> 2) + n) + (m & 3)) * a.ldw + (4 * ks + (l >> 4)) * KPC)
                   : zero4();
    }
  }
  __syncthreads();
  // (sixteen waves: neighbours share a row group, so that five or six groups
  // spread over the four SIMDs)
  const int rg = NW == 16 ? wave / KW : wave % RW;
  int kw = NW == 16 ? wave % KW : wave / RW;
  // (told that kw is 0 or 1, the compiler indexes acc with it, in scratch)
  if constexpr (NW == 16) asm("" : "+s"(kw));
  auto wave_of = [&](int k) { return NW == 16 ? rg * KW + k : k * RW + rg; };
  if (rg >= RGN) return;
  // cells: row tiles rt0 .. rt0 + RT - 1, row l16 of each, units j .. j + NT - 1
  const bool cellw = kw < NCF;
  const int rt0 = cellw && KW > 1 ? kw : 0;
  const int j = jb + NT * q;
  int b[RT];
  float hs[RT][NT], cs[RT][NT];
#pragma unroll
  for (int e = 0; e < RT; ++e) {
    const int r = rg * 32 + (rt0 + e) * 16 + l16;
    b[e] = cellw && r < B ? a.perm[r] : -1;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      hs[e][n] = b[e] >= 0 && a.h0 ? a.h0[(long)b[e] * H + j + n] : 0.f;
      cs[e][n] = b[e] >= 0 && a.c0 ? a.c0[(long)b[e] * H + j + n] : 0.f;
    }
  }

  const int T_eff = uni(a.meta[0]);
  const int len = group_len(a, rg, T_eff);
  // this wave's k-steps (a k-step is the units of four work-groups) and their
  // producers' flags
  const int ks0 = kw * KS / KW, nks = (kw + 1) * KS / KW - ks0;
  const int nfl = 4 * nks * NCF;
  const __amdgpu_buffer_rsrc_t rfl = make_rsrc(a.xflags + ((long)rg * 256 + 4 * ks0) * NCF, (unsigned)nfl * 4);
  unsigned* my_xflag = a.xflags + ((long)rg * 256 + wg) * NCF + (cellw ? kw : 0);
  const __amdgpu_buffer_rsrc_t rring = make_rsrc(a.ring, (unsigned)(2 * RGN * KS) << 11);
  const uint4* w = lds + kw * KSP * NT * 64;
  // ring dword of (row tile 0, row l16, the lane's units)
  const unsigned hoff = (unsigned)(((wg >> 2) << 11) + ((wg & 3) * 16 + l16) * 16 + q * 4);

  float4 zx[RT][NT];
  auto load_zx = [&](int A, long off) {
    const int nr = max(0, min(32, A - rg * 32));
    const __amdgpu_buffer_rsrc_t rz = make_rsrc(a.Zx + (off + rg * 32) * G4, (unsigned)(nr * G4 * 4));
#pragma unroll
    for (int e = 0; e < RT; ++e)
#pragma unroll
      for (int n = 0; n < NT; ++n)
        zx[e][n] = ld_f32x4(rz, cellw ? (unsigned)((((rt0 + e) * 16 + l16) * G4 + 4 * (j + n)) * 4) : kOOB);
  };
  int A_t = len > 0 ? uni(a.active[0]) : 0;
  long off_t = 0;
  if (len > 0) load_zx(A_t, 0);

  for (int t = 0; t < len; ++t) {
    const int A_n = uni(a.active[t + 1]);
    const int nr = min(32, A_t - rg * 32);                 // rows of the group running at t
    // the next step's input projections: asked for before the exchange wait,
    // so that the publish below does not wait for them
    float4 zc[RT][NT];
#pragma unroll
    for (int e = 0; e < RT; ++e)
#pragma unroll
      for (int n = 0; n < NT; ++n) zc[e][n] = zx[e][n];
    load_zx(A_n, off_t + A_t);
    if (t > 0 && nks > 0) wait_quads(a, rfl, nfl, (unsigned)(t + 1));
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(reinterpret_cast<char*>(a.ring) + (((long)((t + 1) & 1) * RGN + rg) * KS + ks0) * 2048,
                  (unsigned)nks << 11);
    f32x4 acc[NT][RTL];
    // sixteen waves are bound by the matrix cores enough to leave a row tile
    // out once its rows have finished (or for a last row group of one tile);
    // eight lose more by the second loop (bf16 H = 2048 B = 40 422 -> 498 us)
    if (NW == 16 && nr <= 16) {
      f32x4 first[NT][1];
      cfwd_product<T, NT, 1, U>(rs, w, KSP / U, wg >> 3, first);
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        acc[n][0] = first[n][0];
        acc[n][RTL - 1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    } else {
      cfwd_product<T, NT, RTL, U>(rs, w, KSP / U, wg >> 3, acc);
    }
    if constexpr (KW > 1) {
      // the shares meet in LDS: each stores its product of the row tiles that
      // are not its own (once their cell waves have read step t-1's), wave
      // kw < 2 adds those of row tile kw in share order
      wait_lds(a, rf, rg * 2 + (lane & 1), lane < NCF, (unsigned)t);
      float4* p4 = reinterpret_cast<float4*>(parts);
#pragma unroll
      for (int rt = 0; rt < RTL; ++rt)
        if (kw != rt)
#pragma unroll
          for (int n = 0; n < NT; ++n)
            p4[(((rg * 2 + rt) * (KW - 1) + (kw < rt ? kw : kw - 1)) * NT + n) * 64 + lane] =
                make_float4(acc[n][rt][0], acc[n][rt][1], acc[n][rt][2], acc[n][rt][3]);
      set_lds(pf + wave, (unsigned)(t + 1));
      if (!cellw) {
        off_t += A_t;
        A_t = A_n;
        continue;
      }
      wait_lds(a, pf, wave_of(lane % KW), lane < KW, (unsigned)(t + 1));
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        f32x4 v = rt0 ? acc[n][RTL - 1] : acc[n][0];
#pragma unroll
        for (int s = 0; s < KW - 1; ++s) {
          const float4 u = p4[(((rg * 2 + rt0) * (KW - 1) + s) * NT + n) * 64 + lane];
          v += f32x4{u.x, u.y, u.z, u.w};
        }
        acc[n][0] = v;
      }
      set_lds(rf + rg * 2 + kw, (unsigned)(t + 1));
    }
    float4 gv[RT][NT];
    unsigned hv[RT];
#pragma unroll
    for (int e = 0; e < RT; ++e) {
      const int r = (rt0 + e) * 16 + l16;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const float ig = sigmoidf_(acc[n][e][0] + zc[e][n].x), fg = sigmoidf_(acc[n][e][1] + zc[e][n].y);
        const float gg = tanhf_(acc[n][e][2] + zc[e][n].z), og = sigmoidf_(acc[n][e][3] + zc[e][n].w);
        const float cn = lstm_c(ig, fg, gg, cs[e][n]);
        const float hn = og * tanhf_(cn);
        if (r < nr) {
          cs[e][n] = cn;
          hs[e][n] = hn;
        }
        gv[e][n] = make_float4(ig, fg, gg, og);
      }
      if constexpr (NT == 1)
        hv[e] = __float_as_uint(hs[e][0]);
      else
        hv[e] = (unsigned)f32_to_bf16(hs[e][0]) | ((unsigned)f32_to_bf16(hs[e][NT - 1]) << 16);
      if (r < nr)
        st_dev(rring, (unsigned)((((t & 1) * RGN + rg) * KS) << 11) + ((unsigned)(rt0 + e) << 10) + hoff,
               __uint_as_float(hv[e]));
    }
    wait_all_vm();
    if (lane == 0) __hip_atomic_store(my_xflag, (unsigned)(t + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // h history, stack row and y of step t
#pragma unroll
    for (int e = 0; e < RT; ++e) {
      const int r = (rt0 + e) * 16 + l16;
      const long cr = off_t + rg * 32 + r;
      if (r < nr) {
        *reinterpret_cast<unsigned*>(reinterpret_cast<T*>(a.X) + cr * H + j) = hv[e];
        if (a.stack) {
          float* srow = a.stack + cr * H5;
#pragma unroll
          for (int n = 0; n < NT; ++n) *reinterpret_cast<float4*>(srow + 4 * (j + n)) = gv[e][n];
          if constexpr (NT == 1)
            srow[G4 + j] = cs[e][0];
          else
            *reinterpret_cast<float2*>(srow + G4 + j) = make_float2(cs[e][0], cs[e][NT - 1]);
        }
      }
      if (a.y && b[e] >= 0) {
        float* yp = a.y + ((long)t * B + b[e]) * H + j;
        if constexpr (NT == 1)
          yp[0] = r < nr ? hs[e][0] : 0.f;
        else
          *reinterpret_cast<float2*>(yp) = r < nr ? make_float2(hs[e][0], hs[e][NT - 1]) : make_float2(0.f, 0.f);
      }
    }
    off_t += A_t;
    A_t = A_n;
  }

#pragma unroll
  for (int e = 0; e < RT; ++e) {
    if (b[e] < 0) continue;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      a.hT[(long)b[e] * H + j + n] = hs[e][n];
      a.cT[(long)b[e] * H + j + n] = cs[e][n];
    }
  }
  // y past the group's last step: whole rows, the steps dealt to the
  // work-groups, the rows to the waves of the row group
  if (a.y) {
    const int nwg = H / KPC;
    const int rows = min(32, B - rg * 32);
    for (int t = len + wg; t < a.T_max; t += nwg)
      for (int r = kw; r < rows; r += KW) {
        float4* row = reinterpret_cast<float4*>(a.y + ((long)t * B + a.perm[rg * 32 + r]) * H);
        for (int i = lane; i < H / 4; i += 64) row[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
  }
}

// ---------------------------------------------------------------------------
// Gradient loop, chip-wide.  Step t (descending):
//   phase B': dh_t of the rows that ran at step t+1 is the sum of the KG KW
//     partial products of step t+1 (other rows keep dhT); with the values
//     popped for step t: dh_tot, dc, dz; dz into the ring, publish; then the
//     dz rows for the dW and dx products and db;
//   phase A': partial products of dh_{t-1} = dz_t W_h^T, published; the pops
//     of step t-1 behind its last ring loads.
// After the last step, dh0 of the rows that ran at step 0 is the sum of the
// partial products of step 0.
// ---------------------------------------------------------------------------
template <typename T, int KG, int KW>
__global__ __launch_bounds__(CNT, 1) void cbwd_kernel(CLoopArgs a) {
  using S = CShape<T, KG, KW>;
  constexpr int KPC = S::KPC, NGX = S::NGX, CW = S::CW, RW = S::RW, RPK = S::RPK, RPL = S::RPL, NP = S::NP;
  extern __shared__ uint4 lds[];
  __shared__ int s_info[2];
  join_group(a.rank_ctr, s_info);
  const int x = uni(s_info[0]), rank = uni(s_info[1]);
  const int H = a.H, B = a.B, RGN = a.RGN;
  if (x >= 8 || rank >= 32 || RGN > RW || H > 8 * 64 * NGX) {
    c_fail(a);
    return;
  }
  const int ngr = (H + 63) / 64;
  const int gpx = (ngr + 7) / 8;
  const int kq = rank / NGX, nq = rank % NGX, grp = x * gpx + nq;
  if (nq >= gpx || grp >= ngr) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int KS = H / 32, KSP = c_share<T>(KS, KW);   // k-steps of the slice (of 4H columns); of a share, padded
  const long G4 = 4L * H, H5 = 5L * H;
  const T* W = reinterpret_cast<const T*>(a.W);
  {
    // weights: output column c is unit grp * 64 + c; element k of a row is
    // W[unit][gate k % 4][unit' k / 4].  Eight neighbouring threads take
    // neighbouring chunks of one row (coalesced reads of each gate's run).
    constexpr int UPC = KPC / 4;                 // units per chunk
    typedef typename std::conditional<sizeof(T) == 2, unsigned, float>::type P4;   // a chunk's values of one gate
    const int nch = KS * 2;                      // chunks per row of the slice
    for (int i = tid; i < KW * KSP * 128; i += CNT) lds[i] = zero4();   // (the padding)
    __syncthreads();
    for (int i = tid; i < (nch + 7) / 8 * 512; i += CNT) {
      const int c8 = i & 7, c = (i >> 3) & 63, ch = (i >> 9) * 8 + c8;
      if (ch >= nch) continue;
      const int unit = grp * 64 + c;
      uint4 v = zero4();
      if (unit < H) {
        const T* src = W + (long)(a.woff + unit) * G4 + (long)(kq * nch + ch) * UPC;
        alignas(16) T tmp[KPC];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const P4 p = *reinterpret_cast<const P4*>(src + (long)g * H);
          if constexpr (sizeof(T) == 2) {
            tmp[g] = (T)(p & 0xffffu);
            tmp[4 + g] = (T)(p >> 16);
          } else {
            tmp[g] = p;
          }
        }
        v = *reinterpret_cast<const uint4*>(tmp);
      }
      const int ks = ch >> 1;
        int sh = 0;   // the share of k-step ks
#pragma unroll
        for (int k = 1; k < KW; ++k) sh += ks >= k * KS / KW;
        lds[((sh * KSP + ks - sh * KS / KW) * 2 + (c >> 5)) * 64 + (ch & 1) * 32 + (c & 31)] = v;
    }
  }
  __syncthreads();
  const int rg = wave % RW, kw = wave / RW;
  float* sc = reinterpret_cast<float*>(lds + KW * KSP * 128) + wave * (kScratch / 4);
  T* sc_dz = reinterpret_cast<T*>(sc);           // [RPK][4][CW] dz of the wave's cells

  const int uu = lane % CW, lr = kw * RPK + (lane / CW) * RPL;
  const int jb = grp * 64 + kq * CW, j = jb + uu;
  const bool has = rg < RGN && jb < H;           // the wave has cells (H % CW == 0: all of its units)
  const bool cellt = has && lane / CW < RPK / RPL;
  int b[RPL];
  float dh[RPL], dc[RPL];
#pragma unroll
  for (int e = 0; e < RPL; ++e) {
    const int r = rg * 32 + lr + e;
    b[e] = cellt && r < B ? a.perm[r] : -1;
    dh[e] = b[e] >= 0 && a.dhT ? a.dhT[(long)b[e] * H + j] : 0.f;
    dc[e] = b[e] >= 0 && a.dcT ? a.dcT[(long)b[e] * H + j] : 0.f;
  }
  float dbacc[4] = {0.f, 0.f, 0.f, 0.f};

  const int T_eff = uni(a.meta[0]);
  const int len = rg < RGN ? group_len(a, rg, T_eff) : 0;
  const int ks0 = kw * KS / KW, nks = (kw + 1) * KS / KW - ks0;
  const int ksg = kq * KS + ks0;
  const int KSR = KG * KS;
  // producers of the wave's k-steps: a k-step is KPC / 2 units, half of a
  // work-group's CW
  const int cb0 = ksg >> 1, cbn = ((ksg + nks - 1) >> 1) - cb0 + 1;
  const unsigned* in_flags = a.xflags + ((long)rg * 256 + cb0) * KW;
  const unsigned* grp_flags = a.xflags + ((long)rg * 256 + grp * KG) * KW;
  unsigned* my_xflag = a.xflags + ((long)rg * 256 + grp * KG + kq) * KW + kw;
  const long pbase = (((long)x * RGN + rg) * NGX + nq) * NP;
  unsigned* my_pflag = a.pflags + pbase + kq * KW + kw;
  float* my_part = a.part + (pbase + kq * KW + kw) * kPartFloats;
  const __amdgpu_buffer_rsrc_t rpart = make_rsrc(a.part + pbase * kPartFloats, NP * kPartFloats * 4);
  const __amdgpu_buffer_rsrc_t rring = make_rsrc(a.ring, (unsigned)(2 * RGN * KSR) << 10);
  const uint4* w = lds + kw * KSP * 128;
  T* DZ = reinterpret_cast<T*>(a.X);

  // popped for the step at hand: i, f, g, o; c_{t-1}; dy.  c_t is the c_{t-1}
  // of the step after it.
  float4 gt[RPL];
  float cc[RPL], cp[RPL], dyv[RPL];
  auto load_c = [&](float (&v)[RPL], int t, int A, long off) {   // c_t of the rows running at t (t < 0: c0)
    const int nr = max(0, min(32, A - rg * 32));
    const __amdgpu_buffer_rsrc_t rc = t >= 0 ? make_rsrc(a.stack + (off + rg * 32) * H5 + G4, (unsigned)(nr * H5 * 4))
                                             : make_rsrc(a.c0, a.c0 ? (unsigned)((long)B * H * 4) : 0u);
#pragma unroll
    for (int e = 0; e < RPL; ++e)
      v[e] = ld_f32(rc, b[e] < 0 ? kOOB : (unsigned)(((t >= 0 ? (lr + e) * H5 : (long)b[e] * H) + j) * 4));
  };
  auto load_step = [&](int t, int A, long off) {
    const int nr = max(0, min(32, A - rg * 32));
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.stack + (off + rg * 32) * H5, (unsigned)(nr * H5 * 4));
    const __amdgpu_buffer_rsrc_t rd =
        a.dy_compact ? make_rsrc(a.dy + (off + rg * 32) * H, (unsigned)(nr * H * 4))
                     : make_rsrc(a.dy ? a.dy + (long)t * B * H : nullptr, a.dy ? (unsigned)((long)B * H * 4) : 0u);
#pragma unroll
    for (int e = 0; e < RPL; ++e) {
      gt[e] = ld_f32x4(rs, b[e] < 0 ? kOOB : (unsigned)(((lr + e) * H5 + 4 * j) * 4));
      dyv[e] = ld_f32(rd, b[e] < 0 ? kOOB : (unsigned)(((a.dy_compact ? (long)(lr + e) * H : (long)b[e] * H) + j) * 4));
    }
  };
  // dh of the rows that ran at step t from the partial products of that step
  auto gather_dh = [&](int t, int nr) {
    wait_range(a, a.pflags + pbase, NP, (unsigned)(T_eff - t));
    constexpr int PB = NP * RPL > 32 ? 32 / RPL : NP;   // partials loaded at a time
    float s[RPL];
#pragma unroll
    for (int p0 = 0; p0 < NP; p0 += PB) {
      float pv[PB][RPL];
#pragma unroll
      for (int p = 0; p < PB; ++p)
        load_partial<RPL>(rpart, (p0 + p) * kPartFloats * 4 + part_off(kq * CW + uu, lr & 31), pv[p]);
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int e = 0; e < RPL; ++e) s[e] = p0 + p == 0 ? pv[p][e] : s[e] + pv[p][e];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int e = 0; e < RPL; ++e)
      if (lr + e < nr) dh[e] = s[e];
  };

  if (len > 0) {
    int A_t = uni(a.active[len - 1]), A_p = len > 1 ? uni(a.active[len - 2]) : 0, nr_next = 0;
    long off_t = uni(a.off[len - 1]);
    if (has) {
      load_c(cc, len - 1, A_t, off_t);
      load_step(len - 1, A_t, off_t);
      load_c(cp, len - 2, A_p, off_t - A_p);
    }
    for (int t = len - 1; t >= 0; --t) {
      const int nr = min(32, A_t - rg * 32);
      const int sl = t & 1;
      const int A_pp = t >= 2 ? uni(a.active[t - 2]) : 0;
      // ---- phase B'
      if (has) {
        if (t < len - 1) gather_dh(t + 1, nr_next);
        float dz[RPL][4];
#pragma unroll
        for (int e = 0; e < RPL; ++e) {
#pragma unroll
          for (int g = 0; g < 4; ++g) dz[e][g] = 0.f;
          if (lr + e < nr && cellt) {
            const float dht = dh[e] + dyv[e];
            const float ig = gt[e].x, fg = gt[e].y, gg = gt[e].z, og = gt[e].w;
            const float tc = tanhf_(cc[e]);
            const float d_o = dht * tc;
            const float dct = dc[e] + dht * og * (1.f - tc * tc);
            dz[e][0] = dct * gg * (ig * (1.f - ig));
            dz[e][1] = dct * cp[e] * (fg * (1.f - fg));
            dz[e][2] = dct * ig * (1.f - gg * gg);
            dz[e][3] = d_o * (og * (1.f - og));
            dc[e] = dct * fg;
          }
        }
        // ring: the four values of a unit side by side (bf16: two units per
        // 16-byte chunk, put together by the lanes of a pair, which swap
        // half of their rows)
        const unsigned rbase = (unsigned)((sl * RGN + rg) * KSR) * 1024u;
        if constexpr (sizeof(T) == 4) {
#pragma unroll
          for (int e = 0; e < RPL; ++e)
            if (cellt && lr + e < nr)
              st16_dev(rring, rbase + (unsigned)(((j >> 1) << 10) + ((j & 1) * 32 + lr + e) * 16),
                       make_uint4(__float_as_uint(dz[e][0]), __float_as_uint(dz[e][1]), __float_as_uint(dz[e][2]),
                                  __float_as_uint(dz[e][3])));
        } else {
          unsigned lo[RPL], hi[RPL];
#pragma unroll
          for (int e = 0; e < RPL; ++e) {
            lo[e] = (unsigned)Op<T>::from_f32(dz[e][0]) | ((unsigned)Op<T>::from_f32(dz[e][1]) << 16);
            hi[e] = (unsigned)Op<T>::from_f32(dz[e][2]) | ((unsigned)Op<T>::from_f32(dz[e][3]) << 16);
          }
          const unsigned ub = rbase + (unsigned)(((j >> 2) << 10) + (((j >> 1) & 1) * 32) * 16);
          const bool odd = (uu & 1) != 0;
          if constexpr (RPL == 1) {
            typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
            if (cellt && lr < nr)
              __builtin_amdgcn_raw_buffer_store_b64(u32x2{lo[0], hi[0]}, rring, ub + lr * 16 + (odd ? 8 : 0), 0,
                                                    kCpolStoreDev);
          } else {
#pragma unroll
            for (int e = 0; e < RPL / 2; ++e) {
              // even lane: rows 0 .. RPL/2 - 1 of both units; odd lane: the rest
              const int mine = odd ? RPL / 2 + e : e;
              const unsigned ml = odd ? lo[RPL / 2 + e] : lo[e], mh = odd ? hi[RPL / 2 + e] : hi[e];
              const unsigned gl = odd ? lo[e] : lo[RPL / 2 + e], gh = odd ? hi[e] : hi[RPL / 2 + e];
              const unsigned ol = __shfl_xor(gl, 1, 64), oh = __shfl_xor(gh, 1, 64);
              if (cellt && lr + mine < nr)
                st16_dev(rring, ub + (lr + mine) * 16, odd ? make_uint4(ol, oh, ml, mh) : make_uint4(ml, mh, ol, oh));
            }
          }
        }
        wait_all_vm();
        if (lane == 0) __hip_atomic_store(my_xflag, (unsigned)(T_eff - t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // dz rows (gate-major) through LDS: 16 bytes of one row and gate per lane
#pragma unroll
        for (int e = 0; e < RPL; ++e)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            dbacc[g] += dz[e][g];
            if (cellt) sc_dz[((lr - kw * RPK + e) * 4 + g) * CW + uu] = Op<T>::from_f32(dz[e][g]);
          }
        wave_lds_fence();
#pragma unroll
        for (int i = 0; i < (RPK * 4 + 63) / 64; ++i) {
          const int k = lane + 64 * i, row = kw * RPK + (k >> 2), g = k & 3;
          if (k < RPK * 4 && row < nr)
            *reinterpret_cast<uint4*>(DZ + (off_t + rg * 32 + row) * G4 + (long)g * H + jb) =
                *reinterpret_cast<const uint4*>(sc_dz + k * CW);
        }
        wave_lds_fence();
      } else {
        // a work-group of the last, half-filled group without units of its
        // own: nothing to publish, its flag only says how far it is
        if (lane == 0) __hip_atomic_store(my_xflag, (unsigned)(T_eff - t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // ---- phase A'
      wait_range(a, in_flags, cbn * KW, (unsigned)(T_eff - t));
      f32x16 acc[2] = {f32x16{}, f32x16{}};
      c_product<T>(make_rsrc(reinterpret_cast<char*>(a.ring) + (((long)sl * RGN + rg) * KSR + ksg) * 1024,
                             (unsigned)nks << 10),
                   w, KSP / c_unroll<T>(), nq * 2, acc, [&]() {
                     if (has && t >= 1) {   // pops of step t-1
#pragma unroll
                       for (int e = 0; e < RPL; ++e) cc[e] = cp[e];
                       load_step(t - 1, A_p, off_t - A_p);
                       load_c(cp, t - 2, A_pp, off_t - A_p - A_pp);
                     }
                   });
      wait_range(a, grp_flags, NP, (unsigned)(T_eff - t));
      store_partial(my_part, acc);
      wait_all_vm();
      if (lane == 0)
        __hip_atomic_store(my_pflag, (unsigned)(T_eff - t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      nr_next = nr;
      off_t -= A_p;
      A_t = A_p;
      A_p = A_pp;
    }
    if (has) gather_dh(0, nr_next);
  }

#pragma unroll
  for (int e = 0; e < RPL; ++e) {
    if (b[e] < 0) continue;
    if (a.dh0) a.dh0[(long)b[e] * H + j] = dh[e];
    if (a.dc0) a.dc0[(long)b[e] * H + j] = dc[e];
  }
  // db of the work-group's CW units (each unit's cells run on exactly one
  // work-group): sum over the waves and their row lanes, fixed order
  __syncthreads();
  float* red = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int g = 0; g < 4; ++g) red[g * CNT + tid] = cellt ? dbacc[g] : 0.f;
  __syncthreads();
  if (tid < 4 * CW && jb + tid % CW < H) {
    const int g = tid / CW, u = tid % CW;
    float s = 0.f;
    for (int i = u; i < CNT; i += CW) s += red[g * CNT + i];
    a.db[(long)g * H + jb + u] = s;
  }
}

// Set-up: h0 rows into ring slot 1 in the consumers' order, flags to zero.
//   f = (((m * KS + ks) * 2 + rt) * 64 + l) * KPC + e: row m*32 + rt*16 + l % 16,
//   unit (4 ks + l / 16) * KPC + e.
template <typename T>
__global__ __launch_bounds__(256) void c_prepare_kernel(const float* __restrict__ h0,
                                                        const int* __restrict__ perm, int B, int H, int RGN,
                                                        void* ring, unsigned* flags, int nflags) {
  constexpr int KPC = Op<T>::kPerChunk;
  const int KS = H / (4 * KPC);
  const long n = (long)RGN * KS * 128 * KPC;
  T* slot1 = reinterpret_cast<T*>(ring) + n;
  for (long f = blockIdx.x * 256L + threadIdx.x; f < n; f += gridDim.x * 256L) {
    const int e = (int)(f % KPC);
    const int l = (int)((f / KPC) % 64);
    const int rt = (int)((f / (64 * KPC)) & 1);
    const int ks = (int)((f / (128 * KPC)) % KS);
    const int m = (int)(f / (128L * KPC * KS));
    const int r = m * 32 + rt * 16 + (l & 15);
    const int u = (4 * ks + (l >> 4)) * KPC + e;
    slot1[f] = Op<T>::from_f32((h0 && r < B) ? h0[(long)perm[r] * H + u] : 0.f);
  }
  for (long i = blockIdx.x * 256L + threadIdx.x; i < nflags; i += gridDim.x * 256L) flags[i] = 0u;
}

template <typename T>
hipError_t launch_c_prepare(const float* h0, const int* perm, int B, int H, int rgn, void* ring,
                            unsigned* flags, int nflags, hipStream_t s) {
  const long n = (long)rgn * 32 * H;
  long blocks = (std::max(n, (long)nflags) + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(c_prepare_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, h0, perm, B, H, rgn, ring,
                     flags, nflags);
  return hipGetLastError();
}
template hipError_t launch_c_prepare<float>(const float*, const int*, int, int, int, void*, unsigned*, int,
                                            hipStream_t);
template hipError_t launch_c_prepare<bf16_t>(const float*, const int*, int, int, int, void*, unsigned*, int,
                                             hipStream_t);

namespace {
// KW, KWF: shares of the gradient's slices and of the forward's reduction
template <typename T, int KW, int KWF, int RTL = 2, int NW = 8>
CKernels c_make(int H, int rgn) {
  constexpr int KGB = sizeof(T) == 2 ? 8 : 16;
  CKernels k{};
  k.fwd = reinterpret_cast<const void*>(&cfwd_kernel<T, KWF, RTL, NW>);
  k.bwd = reinterpret_cast<const void*>(&cbwd_kernel<T, KGB, KW>);
  k.threads_fwd = 64 * NW;
  k.lds_fwd = cfwd_lds<T, KWF, NW>(H);
  k.lds_bwd = (size_t)KW * c_share<T>(H / 32, KW) * 2048 + CNW * kScratch;
  k.rgn = rgn;
  k.kw = KW;
  k.cw = Op<T>::kPerChunk;
  k.nwg_fwd = H / k.cw;
  k.part_floats = 8L * rgn * 32 * KW * kPartFloats;
  k.flag_words_fwd = 8 + rgn * 256 * CFwd<T, KWF, RTL, NW>::NCF;
  k.flag_words = std::max(k.flag_words_fwd, 8 + rgn * 256 * KW + 8 * rgn * 32 * KW);
  return k;
}
}  // namespace

// Kernels for a (dtype, H, B): H % 32 == 0, one work-group per compute unit
// for H = 2048 (bf16) / 1024 (f32), fewer below; at most 256 rows.
//
// Waves that share a slice of the gradient's reduction, us per step (rows: loop
// with KW = 1, 2, 4, 8): a share more is a partial product more for every cell
// to sum, so one wave per slice, bf16 H = 2048 16 rows: 7.5, 8.4, 7.7, 12.7;
// 40: 10.3, 12.5, 14.5; 96: 13.2, 15.5; f32 H = 640 16: 9.3, 10.9, 10.8; 64:
// 10.8, 13.1, 17.4; 96: 11.5, 17.5; only float32's long slices of one row
// group are faster shared by four (H = 1024 16 rows: 13.0, 13.2, 11.5;
// H = 768: 10.4, -, 10.5).
//
// Forward.  At most 16 rows leave the second row tile of the group out
// (inference of 40 steps, B = 16: bf16 H = 2048 370 -> 325 us, H = 1056
// 330 -> 278; f32 H = 1024 389 -> 327, H = 544 338 -> 275).  float32's five
// or six row groups: eight waves of a group each would put two on one SIMD
// and one on each of the others, at 6.8 us of matrix work a step (H = 1024);
// sixteen, two to a group, spread it (H = 1024 B = 144 1174 -> 994 us, 160
// 1221 -> 1050, 192 1307 -> 1084; seven or eight groups are even either way:
// 224 1410 -> 1495).
// bfloat16's products are a quarter as long and its weights and shares of two
// exceed the LDS.
template <typename T>
CKernels c_kernels(int H, int B) {
  const int rgn = (B + 31) / 32;
  if (H % 32 || H < 64 || H > (sizeof(T) == 2 ? 2048 : 1024) || rgn < 1 || rgn > 8) return CKernels{};
  if constexpr (sizeof(T) == 4) {
    if (rgn <= 1 && H > 768) return B <= 16 ? c_make<T, 4, 8, 1>(H, rgn) : c_make<T, 4, 8>(H, rgn);
    if (rgn == 5 || rgn == 6) return c_make<T, 1, 2, 2, 16>(H, rgn);
  }
  return B <= 16    ? c_make<T, 1, 8, 1>(H, rgn)
         : rgn <= 1 ? c_make<T, 1, 8>(H, rgn)
         : rgn <= 2 ? c_make<T, 1, 4>(H, rgn)
         : rgn <= 4 ? c_make<T, 1, 2>(H, rgn)
                    : c_make<T, 1, 1>(H, rgn);
}
template CKernels c_kernels<float>(int, int);
template CKernels c_kernels<bf16_t>(int, int);

hipError_t c_setup(const CKernels& k, int* occ_fwd, int* occ_bwd) {
  hipFuncAttributes fa{}, fb{};
  hipError_t e = hipFuncGetAttributes(&fa, k.fwd);
  if (e != hipSuccess) return e;
  e = hipFuncGetAttributes(&fb, k.bwd);
  if (e != hipSuccess) return e;
  if (fa.localSizeBytes > 32 || fb.localSizeBytes > 32) {
    *occ_fwd = 0;
    *occ_bwd = 0;
    return hipSuccess;
  }
  e = hipFuncSetAttribute(k.fwd, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds_fwd);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute(k.bwd, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds_bwd);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(occ_fwd, k.fwd, k.threads_fwd, k.lds_fwd);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(occ_bwd, k.bwd, CNT, k.lds_bwd);
}

hipError_t c_launch(const void* fn, const CLoopArgs& a, int nwg, int threads, size_t lds, hipStream_t s) {
  CLoopArgs copy = a;
  void* kargs[] = {&copy};
  return hipLaunchKernel(fn, dim3((unsigned)nwg), dim3((unsigned)threads), kargs, lds, s);
}

}  // namespace ll
