// float32 matrix-core products of the loop that do not sit on the recurrence
// (the same three as in ll_gemm.hip): both operands row-major along the
// reduction (NT: input projection, dx, gate recomputation) and both along
// the rows (TN: dW = [X; Hprev]^T DZ straight from the row-major operands).
//
// Bound: the float32 matrix cores (157 TFLOP/s; 64 clocks per 32x32x2
// instruction).  A 64x64 tile per work-group of four waves (one 32x32 block
// each) is enough for that: per k-step of 8 a wave reads 2 KB of LDS for 256
// clocks of matrix instructions, a compute unit 16 B/clk from the L2, and five
// work-groups of 32 KB LDS fit a compute unit, so the loads of one hide under
// the products of the others and small shapes still make enough tiles.
// Measured: the input projection 6400 x 2048 x 512 0.164 -> 0.140 ms against
// the 128x128 register-staged form this replaces (51200 rows: 0.93 ms for
// either, 115 TFLOP/s: the four waves of a work-group meet at a barrier per
// k-tile, and the SIMDs idle when their waves wait for another SIMD's); 128x128
// tiles here 0.157 and 0.94 ms, dx at 51200 rows 0.95 against 0.89.  dW
// reads its operands in place: three transposing copies (0.057 ms at
// 6400 rows, 0.235 at 51200) are gone.  Operands go straight into LDS (buffer
// loads with the LDS destination), two stages, one barrier per k-tile of 32.
#include <algorithm>

#include "ll_exchange.h"

namespace ll {

namespace {

constexpr int kK = 32;         // elements of the reduction per k-tile
constexpr int kThreads = 256;
constexpr int kGroupRows = 8;  // row tiles per group of the tile order

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void_t;

// Tile of work-group L: XCD L % 8 takes a contiguous share of the tiles, in
// groups of kGroupRows row tiles; false if there is none.
__device__ __forceinline__ bool tile_of(int L, int nmt, int nnt, int splits, int* mt, int* nt, int* z) {
  const int per_split = nmt * nnt, ntiles = per_split * splits;
  const int share = (ntiles + 7) / 8;
  const int t = (L & 7) * share + (L >> 3);
  if ((L >> 3) >= share || t >= ntiles) return false;
  *z = t / per_split;
  const int tt = t - *z * per_split;
  const int grp = tt / (kGroupRows * nnt), fm = grp * kGroupRows;
  const int gsz = min(nmt - fm, kGroupRows);
  const int within = tt - grp * kGroupRows * nnt;
  *mt = fm + within % gsz;
  *nt = within / gsz;
  return true;
}

}  // namespace

// ---------------------------------------------------------------------------
// C[crow(m)][n] = sum_k A[arow(m)][k] B[n][k] (+ bias, gate epilogue).
//
// LDS: per stage and operand 64 rows x 8 chunks of 16 bytes; chunk c of row r
// sits in slot c ^ swz(r), swz(r) = (r & 7) ^ ((r >> 3) & 1), so that the
// reads of 16 consecutive lanes (16 rows, one chunk) hit different bank
// groups.  A load instruction fills 8 rows: lane l writes slot l % 8 of row
// l / 8.  Lane l of a wave supplies row / column l % 32 and, in k-step ks,
// chunk 2 ks + l / 32; element j of the chunks feeds the j-th instruction.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void gemm32_nt_kernel(GemmArgs g, unsigned a_bytes, unsigned b_bytes) {
  constexpr int kT = 64, LI = 2;   // tile; load instructions per wave and operand
  // (an array per stage: the compiler then does not wait for the fills of the
  // other stage before it reads this one)
  __shared__ uint4 sA0[kT * 8], sA1[kT * 8], sB0[kT * 8], sB1[kT * 8];
  if ((int)blockIdx.x < g.pre_blocks) {   // the jobs carried by this launch
    pre_jobs_body<float>(g.pre, blockIdx.x, g.pre_blocks, kThreads);
    return;
  }
  const int M = g.M_dev ? min(*g.M_dev, g.M) : g.M;
  int mt, nt, z;
  if (!tile_of(blockIdx.x - g.pre_blocks, (M + kT - 1) / kT, (g.N + kT - 1) / kT, 1, &mt, &nt, &z)) return;
  const int m0 = mt * kT, n0 = nt * kT, K = g.K;
  const int nkt = (K + kK - 1) / kK;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, hf = lane >> 5;

  const __amdgpu_buffer_rsrc_t ra = make_rsrc(g.A, a_bytes), rb = make_rsrc(g.Bm, b_bytes);
  unsigned aoff[LI], boff[LI];
  int ch[LI];
#pragma unroll
  for (int i = 0; i < LI; ++i) {
    const int row = (i * 4 + wave) * 8 + (lane >> 3);
    const int m = m0 + row, n = n0 + row;
    ch[i] = (lane & 7) ^ ((row & 7) ^ ((row >> 3) & 1));
    aoff[i] = m < M ? (unsigned)((g.a_rowmap ? g.a_rowmap[m] : m) * (long)g.lda * 4 + ch[i] * 16) : kOOB;
    boff[i] = n < g.N ? (unsigned)(n * (long)g.ldb * 4 + ch[i] * 16) : kOOB;
  }
  auto fill = [&](int kt, uint4* a_dst, uint4* b_dst) {
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const bool past = kt * kK + ch[i] * 4 >= K;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(a_dst + (i * 4 + wave) * 64), 16,
                                               past ? kOOB : aoff[i] + kt * (kK * 4), 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)(b_dst + (i * 4 + wave) * 64), 16,
                                               past ? kOOB : boff[i] + kt * (kK * 4), 0, 0, 0);
    }
  };
  f32x16 acc = {};
  const int sw = (l32 & 7) ^ ((l32 >> 3) & 1);
  const int arow = (wm * 32 + l32) * 8, brow = (wn * 32 + l32) * 8;
  auto step = [&](int kt, const uint4* sa, const uint4* sb, uint4* a_next, uint4* b_next) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (kt + 1 < nkt) fill(kt + 1, a_next, b_next);
    uint4 a[4], b[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      a[ks] = sa[arow + ((2 * ks + hf) ^ sw)];
      b[ks] = sb[brow + ((2 * ks + hf) ^ sw)];
    }
    __builtin_amdgcn_sched_barrier(0);   // (every read of the k-tile before the first product)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[ks].x), __uint_as_float(b[ks].x), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[ks].y), __uint_as_float(b[ks].y), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[ks].z), __uint_as_float(b[ks].z), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[ks].w), __uint_as_float(b[ks].w), acc, 0, 0, 0);
    }
  };
  fill(0, sA0, sB0);
  for (int kt = 0; kt < nkt; kt += 2) {
    step(kt, sA0, sB0, sA1, sB1);
    if (kt + 1 < nkt) step(kt + 1, sA1, sB1, sA0, sB0);
  }

  // result register r of lane l: row (r % 4) + 8 (r / 4) + 4 (l / 32), column
  // l % 32.  Loads first, then stores.
  const int act_h = g.act_h;
  const int n = n0 + wn * 32 + l32;
  const bool nok = n < g.N;
  const float bn = g.bias && nok ? g.bias[g.bias_um ? (n & 3) * g.bias_um + (n >> 2) : n] : 0.f;
  int crow[16];
  float zin[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + (r & 3) + 8 * (r >> 2) + 4 * hf;
    crow[r] = m < M && nok ? (g.c_rowmap ? g.c_rowmap[m] : m) : -1;
  }
  if (act_h) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + wm * 32 + (r & 3) + 8 * (r >> 2) + 4 * hf;
      zin[r] = crow[r] < 0 ? 0.f
               : g.addend  ? g.addend[(long)g.add_rowmap[m] * g.ld_add + n]
                           : g.C[(long)crow[r] * g.ldc + n];
    }
  }
  __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0): those loads, ahead of any store
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (crow[r] < 0) continue;
    float v = acc[r] + bn;
    if (act_h) v = n / act_h == 2 ? tanhf_(v + zin[r]) : sigmoidf_(v + zin[r]);
    g.C[(long)crow[r] * g.ldc + n] = v;
  }
}

// ---------------------------------------------------------------------------
// C[m][n] = sum_k A[arow(k)][m] B[k][n'] over rows k < K of row-major
// operands; rows m >= M1 read a second operand (its own row tiles, so M1 can
// be anything), and for those n' = n + n_jump once n >= n_from (the GRU's
// candidate block differs between the two sides).
//
// LDS: per stage and operand 32 rows (k) x 16 chunks of 4 columns; chunk c of
// row k sits in slot c ^ 8 (k & 1), so the two rows a matrix instruction reads
// (k-slot l / 32) lie in different banks.  A load instruction fills 4 rows.
// The row map of a k-tile is read a k-tile ahead of its fill.
//
// The sums of kSpan k-tiles (256 rows) are gathered in a second set of
// registers: the rounding error of one float32 chain grows with the square
// root of its length (2-norm error of dW at 6400 rows of H = 256: 7.5e-7 with
// spans of 2048 rows, 5.6e-7 with these).  No split of the reduction is
// shorter than 256 rows, so no chain is longer than a split-K sum's.
// ---------------------------------------------------------------------------
constexpr int kSpan = 8;   // (even: a span starts on the first stage)

template <int S>
__global__ __launch_bounds__(kThreads) void gemm32_tn_kernel(GemmTnArgs g, unsigned a_bytes, unsigned b_bytes,
                                                             unsigned a2_bytes) {
  constexpr int kT = 64 * S, RC = 16 * S, LI = 2 * S;   // tile; chunks per LDS row; load instructions per wave
  __shared__ uint4 sA0[kK * RC], sA1[kK * RC], sB0[kK * RC], sB1[kK * RC];   // (an array per stage, as above)
  const int M1 = g.A2 ? g.M1 : g.M;
  const int nm1 = (M1 + kT - 1) / kT, nm2 = (g.M - M1 + kT - 1) / kT;
  int mt, nt, z;
  if (!tile_of(blockIdx.x, nm1 + nm2, (g.N + kT - 1) / kT, g.splits, &mt, &nt, &z)) return;
  const bool second = mt >= nm1;
  const int am0 = (second ? mt - nm1 : mt) * kT, aM = second ? g.M - M1 : M1;   // columns of the operand
  const int n0 = nt * kT, b0 = n0 + (second && n0 >= g.n_from ? g.n_jump : 0);
  const int K = g.K_dev ? min(*g.K_dev, g.K) : g.K;
  const int kper = ((K + g.splits - 1) / g.splits + kK - 1) / kK * kK;
  const int kb = min(K, z * kper), ke = min(K, kb + kper);
  const int nkt = (ke - kb + kK - 1) / kK;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, hf = lane >> 5;

  const __amdgpu_buffer_rsrc_t ra = second ? make_rsrc(g.A2, a2_bytes) : make_rsrc(g.A, a_bytes);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(g.Bm, b_bytes);
  const long lda = second ? g.lda2 : g.lda;
  const int* map = second ? g.a2_rowmap : g.a_rowmap;
  const bool has_map = map != nullptr;
  const __amdgpu_buffer_rsrc_t rmap = make_rsrc(map, has_map ? (unsigned)ke * 4u : 0u);
  // load instruction i: rows (i 4 + wave) 64 / RC + lane / RC, slot lane % RC
  int lrow[LI];
  unsigned acol[LI], bcol[LI], am[LI];
#pragma unroll
  for (int i = 0; i < LI; ++i) {
    lrow[i] = (i * 4 + wave) * (64 / RC) + lane / RC;
    const int c = ((lane % RC) ^ (8 * (lrow[i] & 1))) * 4;
    acol[i] = am0 + c < aM ? (unsigned)((am0 + c) * 4) : kOOB;
    bcol[i] = n0 + c < g.N ? (unsigned)((b0 + c) * 4) : kOOB;
  }
  auto load_map = [&](int kt) {
#pragma unroll
    for (int i = 0; i < LI; ++i)
      am[i] = __builtin_amdgcn_raw_buffer_load_b32(rmap, (unsigned)(kb + kt * kK + lrow[i]) * 4u, 0, 0);
  };
  auto fill = [&](int kt, uint4* a_dst, uint4* b_dst) {
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const int k = kb + kt * kK + lrow[i];
      const long ar = has_map ? (long)am[i] : (long)k;
      const unsigned ao = k < ke && acol[i] != kOOB ? (unsigned)(ar * lda * 4) + acol[i] : kOOB;
      const unsigned bo = k < ke && bcol[i] != kOOB ? (unsigned)((long)k * g.ldb * 4) + bcol[i] : kOOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(a_dst + (i * 4 + wave) * 64), 16, ao, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void_t*)(b_dst + (i * 4 + wave) * 64), 16, bo, 0, 0, 0);
    }
    load_map(kt + 1);
  };
  f32x16 acc[S][S] = {}, sum[S][S] = {};
  auto step = [&](int kt, const uint4* sa, const uint4* sb, uint4* a_next, uint4* b_next) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (kt + 1 < nkt) fill(kt + 1, a_next, b_next);
    const float* a = reinterpret_cast<const float*>(sa);
    const float* b = reinterpret_cast<const float*>(sb);
    const int ac = (wm * 32 * S + l32) ^ (32 * hf), bc = (wn * 32 * S + l32) ^ (32 * hf);
#pragma unroll
    for (int h = 0; h < S; ++h) {
      constexpr int P = 16 / S;
      float av[P][S], bv[P][S];
#pragma unroll
      for (int p = 0; p < P; ++p)   // rows 2p + hf
#pragma unroll
        for (int i = 0; i < S; ++i) {
          av[p][i] = a[(2 * (h * P + p) + hf) * kT + (ac ^ (32 * i))];
          bv[p][i] = b[(2 * (h * P + p) + hf) * kT + (bc ^ (32 * i))];
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
          for (int j = 0; j < S; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[p][i], bv[p][j], acc[i][j], 0, 0, 0);
    }
  };
  load_map(0);
  if (nkt > 0) fill(0, sA0, sB0);
  for (int k0 = 0; k0 < nkt; k0 += kSpan) {
    const int k1 = min(nkt, k0 + kSpan);
    for (int kt = k0; kt < k1; kt += 2) {
      step(kt, sA0, sB0, sA1, sB1);
      if (kt + 1 < k1) step(kt + 1, sA1, sB1, sA0, sB0);
    }
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = 0; j < S; ++j) {
        sum[i][j] += acc[i][j];
        acc[i][j] = f32x16{};
      }
  }
  float* C = g.C + (g.splits > 1 ? (long)z * g.split_stride : 0L);
  const int mc = (second ? M1 : 0) + am0;
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int n = n0 + (wn * S + j) * 32 + l32;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = (wm * S + i) * 32 + (r & 3) + 8 * (r >> 2) + 4 * hf;
        if (am0 + m < aM && n < g.N) C[(long)(mc + m) * g.ldc + n] = sum[i][j][r];
      }
    }
}

namespace {
long nt32_a_bytes(const GemmArgs& g) { return (long)(g.a_rows > 0 ? g.a_rows : g.M) * g.lda * 4; }
long tn32_a_bytes(const GemmTnArgs& g) { return (long)(g.a_rows > 0 ? g.a_rows : g.K) * g.lda * 4; }
}  // namespace

// 32-bit offsets, 16-byte rows, whole 16-byte chunks of the reduction; no
// split (every float32 NT product has enough tiles).
bool gemm32_nt_applies(const GemmArgs& g) {
  if (g.splits != 1 || g.K_dev || g.K % 4 || g.lda % 4 || g.ldb % 4) return false;
  if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.Bm)) & 15) return false;
  return nt32_a_bytes(g) < (long)kOOB && (long)g.N * g.ldb * 4 < (long)kOOB;
}

hipError_t launch_gemm32_nt(const GemmArgs& g, hipStream_t s) {
  if (!gemm32_nt_applies(g)) return hipErrorInvalidValue;
  const long tiles = (long)((g.M + 63) / 64) * ((g.N + 63) / 64);
  hipLaunchKernelGGL(gemm32_nt_kernel, dim3((unsigned)((tiles + 7) / 8 * 8 + g.pre_blocks)), dim3(kThreads), 0, s, g,
                     (unsigned)nt32_a_bytes(g), (unsigned)((long)g.N * g.ldb * 4));
  return hipGetLastError();
}

bool gemm32_tn_applies(const GemmTnArgs& g) {
  if (g.M % 4 || g.N % 4 || g.lda % 4 || g.ldb % 4 || g.splits < 1 || g.tile_flags) return false;
  if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.Bm) | reinterpret_cast<uintptr_t>(g.A2)) & 15)
    return false;
  if (g.A2 && (g.M1 <= 0 || g.M1 >= g.M || g.M1 % 4 || g.lda2 % 4)) return false;
  if (g.n_jump && (g.n_from % 64 || g.n_jump % 4)) return false;
  const long a2b = g.A2 ? (long)g.a2_rows * g.lda2 * 4 : 0;
  return tn32_a_bytes(g) < (long)kOOB && (long)g.b_rows * g.ldb * 4 < (long)kOOB && a2b < (long)kOOB;
}

// Tile edge of a TN product: 128 for long reductions whose 128x128 tiles,
// split up to four ways, still make two per compute unit (1024 x 2048 over
// 51 200 rows: 1.76 ms against 2.02 with 64); shorter ones take 64, which
// needs fewer splits and no sum over them (6 400 rows: training step 1.24 ms
// against 1.27).
long tn32_tiles(long t, int M, int M1, int N) { return ((M1 + t - 1) / t + (M - M1 + t - 1) / t) * ((N + t - 1) / t); }
bool tn32_big(int M, int M1, int N, int n_from, long K) {
  return n_from % 128 == 0 && K >= 16384 && tn32_tiles(128, M, M1, N) >= 128;
}
int gemm32_tn_splits(int M, int M1, int N, int n_from, long K, int n_cu) {
  const long tiles = tn32_tiles(tn32_big(M, M1, N, n_from, K) ? 128 : 64, M, M1, N);
  const long sp = (2L * n_cu + tiles - 1) / tiles;
  return (int)std::max(1L, std::min(16L, std::min(sp, std::max(1L, K / 256))));
}

hipError_t launch_gemm32_tn(const GemmTnArgs& g, hipStream_t s) {
  if (!gemm32_tn_applies(g)) return hipErrorInvalidValue;
  const int M1 = g.A2 ? g.M1 : g.M;
  const bool big = tn32_big(g.M, M1, g.N, g.n_from, g.K);
  const long n = (tn32_tiles(big ? 128 : 64, g.M, M1, g.N) * g.splits + 7) / 8 * 8;
  const unsigned ab = (unsigned)tn32_a_bytes(g), bb = (unsigned)((long)g.b_rows * g.ldb * 4),
                 a2b = (unsigned)(g.A2 ? (long)g.a2_rows * g.lda2 * 4 : 0);
  if (big)
    hipLaunchKernelGGL(gemm32_tn_kernel<2>, dim3((unsigned)n), dim3(kThreads), 0, s, g, ab, bb, a2b);
  else
    hipLaunchKernelGGL(gemm32_tn_kernel<1>, dim3((unsigned)n), dim3(kThreads), 0, s, g, ab, bb, a2b);
  return hipGetLastError();
}

}  // namespace ll
