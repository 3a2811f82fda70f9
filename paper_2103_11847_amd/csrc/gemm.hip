// Transform-domain frontal-slice products (Algorithm 1 step 2): the one
// dense contraction of the c-product, C~_k = op(A~_k) op(B~_k) for k < p,
// as batched GEMMs on the gfx950 matrix cores.
//
// Tile: BM x BN outputs per workgroup of 4 waves arranged 2 x 2, each wave
// owning (BM/2) x (BN/2) as 16 x 16 MFMA blocks.  Operands are staged through
// LDS as [rows][BK + pad] (contraction index contiguous) so each lane's MFMA
// operand is one LDS read: 1 element for the K = 4 FP32/FP64 instructions,
// 8 packed 16-bit elements for the K = 32 BF16/FP16 instructions of gfx950.
// Global loads are ordered along each operand's contiguous dimension; the
// next K-chunk is prefetched into registers while the current one is
// multiplied.  Ragged edges are zero-filled on load and masked on store.
#include <algorithm>
#include <type_traits>

#include "fastdct.h"
#include "mfma.h"

namespace dctk {

// batches of at least this many slices are placed per XCD (slice_block)
constexpr int kSliceXcdMin = 16;

struct GemmArgs {
  int gx, gy, gz;
  int M, N, K;
  const void* A;
  int64_t lda, sA;
  const void* B;
  int64_t ldb, sB;
  void* C;
  int64_t ldc, sC;
  Gate g;
  int nbatch;   // > 0: slices placed per XCD (see slice_block); the grid's z is padded to 8 ceil(nbatch / 8)
  OperandRange range;   // FP32, split kernel (last: in the middle it cost every small product 0.1 us of argument loads)
};

// XCD-aware slice placement of a plain batched launch.  Workgroups are dealt to
// the 8 XCDs round robin in dispatch order, and each XCD has its own L2.  With
// T = gx gy tiles per slice, dispatch slot `lin` goes to XCD lin % 8 and is
// given tile (lin / 8) % T of slice 8 ((lin / 8) / T) + lin % 8: every tile of
// a slice runs on one XCD, in consecutive slots, so the slice's operands are
// fetched into one L2 instead of eight.  Padding slots (slice >= nbatch) exit.
__device__ inline bool slice_block(const GemmArgs& ga, VBlock& vb) {
  if (ga.nbatch <= 0) return true;
  const int64_t T = (int64_t)ga.gx * ga.gy;
  const int64_t lin = vb.x + (int64_t)ga.gx * (vb.y + (int64_t)ga.gy * vb.z);
  const int64_t slot = lin >> 3;
  const int64_t z = (slot / T) * 8 + (lin & 7);
  if (z >= ga.nbatch) return false;
  const int64_t t = slot % T;
  vb.x = (int)(t % ga.gx);
  vb.y = (int)(t / ga.gx);
  vb.z = (int)z;
  return true;
}

// Eight 16-bit elements at any address (a 2-byte aligned 16-byte load).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_un __attribute__((ext_vector_type(4), aligned(2)));
template <typename TI>
__device__ __forceinline__ u32x4 load8(const TI* p) {
  return *reinterpret_cast<const u32x4_un*>(p);
}
// A unit of 8 elements whose load was moved back by n elements to end with its
// row: elements n .. 7 to the front, 0 behind them (n <= 0: as loaded).
__device__ __forceinline__ u32x4 drop8(u32x4 v, int n) {
  if (n <= 0) return v;
  if (n >= 8) return u32x4{0u, 0u, 0u, 0u};
  if (n & 4) v = u32x4{v.z, v.w, 0u, 0u};
  if (n & 2) v = u32x4{v.y, v.z, v.w, 0u};
  if (n & 1)
    v = u32x4{__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16),
              __builtin_amdgcn_alignbit(v.w, v.z, 16), v.w >> 16};
  return v;
}

// 16-bit slice GEMM, A~ contiguous in k.  VEC (K >= 8, and N >= 8 for B
// contiguous in n): operands move as 8-element units along their contiguous
// dimension, at any alignment and any size: rows beyond an operand are read
// from its last row, a unit that would cross the end of its row is loaded
// from the row's last 8 elements and put right when it is staged, where its
// wait is.  An operand contiguous in k goes to its LDS rows as one 16-byte
// store, one contiguous in n is transposed on the way, as eight stores into
// eight rows.  Sizes that were no multiple of 8 took 2-byte loads before:
// 64 x 637^3 BF16 200 us (640^3: 87), now 97 (85); 31 x 501^3 67 (504^3: 32), now
// 37 (31); 32 x 302^3, two products a slice, 51 (304^3: 25), now 27 (26).
template <typename TI, typename TO, int BM, int BN, bool TB, bool VEC>
__device__ __forceinline__ void gemm_kernel_body(const GemmArgs& ga, const VBlock vb) {
  const int M = ga.M, N = ga.N, K = ga.K;
  const TI* __restrict__ A = (const TI*)ga.A;
  const TI* __restrict__ B = (const TI*)ga.B;
  TO* __restrict__ C = (TO*)ga.C;
  const int64_t lda = ga.lda, sA = ga.sA, ldb = ga.ldb, sB = ga.sB, ldc = ga.ldc, sC = ga.sC;
  const Gate g = ga.g;
  typedef Mfma<TI> MF;
  typedef typename MF::acc_t acc_t;
  typedef typename MF::frag_t frag_t;
  constexpr int KSTEP = MF::KSTEP;
  // 256-row tiles: 32-wide contraction chunks (the two operand tiles of a
  // 256 x 128 chunk are 30 KB of LDS, so two workgroups share a CU)
  constexpr int BK = BM >= 256 ? 32 : 64;
  constexpr int LDS_LD = BK + 8;   // 16-byte pad
  constexpr int NT = 256, WGM = 2, WGN = NT / 128;   // threads, wave grid
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int FM = WM / 16, FN = WN / 16;

  if (!gate_open(g)) return;

  __shared__ __attribute__((aligned(16))) TI As[BM * LDS_LD];
  __shared__ __attribute__((aligned(16))) TI Bs[BN * LDS_LD];

  const int bz = vb.z;
  const int m0 = vb.y * BM;
  const int n0 = vb.x * BN;
  A += (int64_t)bz * sA;
  B += (int64_t)bz * sB;
  C += (int64_t)bz * sC;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;

  // scalar staging
  constexpr int A_PER = VEC ? 1 : BM * BK / NT, B_PER = VEC ? 1 : BN * BK / NT;  // elements per thread
  TI ra[A_PER], rb[B_PER];
  auto b_coord = [&](int u, int& c, int& kk) {
    const int idx = tid + u * NT;
    if (!TB) { kk = idx / BN; c = idx % BN; }   // contiguous along n
    else     { c = idx / BK; kk = idx % BK; }   // contiguous along k
  };
  auto load_tiles = [&](int k0) {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) {
      const int idx = tid + u * NT, gm = m0 + idx / BK, gk = k0 + idx % BK;
      TI v = (TI)0;
      if (gm < M && gk < K) v = A[(int64_t)gm * lda + gk];
      ra[u] = v;
    }
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
      int c, kk;
      b_coord(u, c, kk);
      const int gn = n0 + c, gk = k0 + kk;
      TI v = (TI)0;
      if (gn < N && gk < K) v = TB ? B[(int64_t)gn * ldb + gk] : B[(int64_t)gk * ldb + gn];
      rb[u] = v;
    }
  };
  auto store_tiles = [&]() {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) {
      const int idx = tid + u * NT;
      As[idx / BK * LDS_LD + idx % BK] = ra[u];
    }
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
      int c, kk;
      b_coord(u, c, kk);
      Bs[c * LDS_LD + kk] = rb[u];
    }
  };

  // vector staging: units of 8 k of a row, or of 8 rows x 8 k transposed in registers
  struct H8 { TI v[8]; };
  constexpr int A_NK = BM * BK / 8;                          // units of the A tile
  constexpr int B_NK = TB ? BN * BK / 8 : BN * BK / 64;
  constexpr int A_UV = VEC ? (A_NK + NT - 1) / NT : 1, B_UV = VEC ? (B_NK + NT - 1) / NT : 1;
  constexpr int B_L = TB ? 1 : 8;                            // loads per unit
  u32x4 va[A_UV], vbv[B_UV][B_L];
  // unit u of an operand tile of R rows: its first (row, k)
  auto unit = [&](int u, int R, bool kcontig, int& r, int& kk) {
    const int idx = tid + u * NT;
    if (kcontig) { r = idx / (BK / 8); kk = (idx % (BK / 8)) * 8; }
    else         { kk = (idx / (R / 8)) * 8; r = (idx % (R / 8)) * 8; }
  };
  auto at_most = [](int v, int lim) { return v < lim ? v : lim; };
  auto load_vec = [&](int k0) {
#pragma unroll
    for (int u = 0; u < A_UV; ++u) {
      int r, kk;
      unit(u, BM, true, r, kk);
      va[u] = load8(A + (int64_t)at_most(m0 + r, M - 1) * lda + at_most(k0 + kk, K - 8));
    }
#pragma unroll
    for (int u = 0; u < B_UV; ++u) {
      int c, kk;
      unit(u, BN, TB, c, kk);
      if (B_NK % NT != 0 && tid + u * NT >= B_NK) continue;
#pragma unroll
      for (int l = 0; l < B_L; ++l)
        vbv[u][l] = load8(B + (TB ? (int64_t)at_most(n0 + c, N - 1) * ldb + at_most(k0 + kk, K - 8)
                                  : (int64_t)at_most(k0 + kk + l, K - 1) * ldb + at_most(n0 + c, N - 8)));
    }
  };
  auto store_vec = [&](int k0) {
    const bool kend = k0 + BK > K, nend = n0 + BN > N;   // uniform
#pragma unroll
    for (int u = 0; u < A_UV; ++u) {
      if (A_NK % NT != 0 && tid + u * NT >= A_NK) continue;
      int r, kk;
      unit(u, BM, true, r, kk);
      u32x4 v = va[u];
      if (kend) v = drop8(v, k0 + kk - (K - 8));
      *reinterpret_cast<u32x4*>(&As[r * LDS_LD + kk]) = v;
    }
#pragma unroll
    for (int u = 0; u < B_UV; ++u) {
      if (B_NK % NT != 0 && tid + u * NT >= B_NK) continue;
      int c, kk;
      unit(u, BN, TB, c, kk);
      if constexpr (TB) {
        u32x4 v = vbv[u][0];
        if (kend) v = drop8(v, k0 + kk - (K - 8));
        *reinterpret_cast<u32x4*>(&Bs[c * LDS_LD + kk]) = v;
      } else {
        if (nend) {
#pragma unroll
          for (int l = 0; l < 8; ++l) vbv[u][l] = drop8(vbv[u][l], n0 + c - (N - 8));
        }
        if (kend) {
#pragma unroll
          for (int l = 0; l < 8; ++l)
            if (k0 + kk + l >= K) vbv[u][l] = u32x4{0u, 0u, 0u, 0u};
        }
        H8 h[8];
#pragma unroll
        for (int l = 0; l < 8; ++l) h[l] = __builtin_bit_cast(H8, vbv[u][l]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          H8 w;
#pragma unroll
          for (int l = 0; l < 8; ++l) w.v[l] = h[l].v[j];
          *reinterpret_cast<u32x4*>(&Bs[(c + j) * LDS_LD + kk]) = __builtin_bit_cast(u32x4, w);
        }
      }
    }
  };

  frag_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = (acc_t)0;

  const int lr = lane & 15;          // row (A) / column (B) within a 16-block
  const int lk = (lane >> 4) * MF::EPL;  // first contraction index of this lane

  if constexpr (VEC) load_vec(0);
  else load_tiles(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
    if constexpr (VEC) store_vec(k0);
    else store_tiles();
    __syncthreads();
    // prefetch the next chunk into registers
    if constexpr (VEC) {
      if (k0 + BK < K) load_vec(k0 + BK);
    } else {
      if (k0 + BK < K) load_tiles(k0 + BK);
    }
#pragma unroll
    for (int ks = 0; ks < BK; ks += KSTEP) {
      const TI* ap[FM];
      const TI* bp[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) ap[i] = &As[(wm * WM + i * 16 + lr) * LDS_LD + ks + lk];
#pragma unroll
      for (int j = 0; j < FN; ++j) bp[j] = &Bs[(wn * WN + j * 16 + lr) * LDS_LD + ks + lk];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = MF::mac(ap[i], bp[j], acc[i][j]);
    }
  }

  // D layout of the 16x16 instructions: column lane % 16; rows 4 (lane/16) + r, or
  // lane/16 + 4 r for FP64.
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * WN + j * 16 + (lane & 15);
      if (col >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + (MF::ROWS_STRIDED ? (lane >> 4) + 4 * r : (lane >> 4) * 4 + r);
        if (row < M) C[(int64_t)row * ldc + col] = out_cvt<TO, acc_t>(acc[i][j][r]);
      }
    }
}

template <typename TI, typename TO, int BM, int BN, bool TB, bool VEC, bool GROUPED>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs ga_, const GemmArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    VBlock vb = hw_block();
    if (!slice_block(ga_, vb)) return;
    gemm_kernel_body<TI, TO, BM, BN, TB, VEC>(ga_, vb);
  } else {
    VBlock vb;
    const GemmArgs g = group_args(grp, bmap, vb);
    if (!slice_block(g, vb)) return;   // the instance's grid may be padded
    gemm_kernel_body<TI, TO, BM, BN, TB, VEC>(g, vb);
  }
}

// The same with 64 x 64 or 32 x 32 tiles: the slices of video and of small
// cubes, a few chunks of K each, where the time is that of the loads' round
// trips.  So the next kRing chunks (64 k) of both operands are in flight in
// registers, and one barrier a chunk separates the two LDS buffers.  B
// contiguous in n moves in units of 2 k x 8 n, paired on the way into 8 LDS
// rows.  LDS rows are 8 blocks of 16 bytes, block b of row r at
// b ^ (r ^ r / 8) % 8: neither the stores of 8 rows 8 apart nor the operand
// reads of 8 neighbouring rows meet in a bank.  Two FP16 products
// a slice, with one chunk in flight and now: 32 x 256^3 18.7 -> 17.8 us, 20 x
// 320^3 31.8 -> 28.3.  The sums are those of gemm_kernel, bit for bit.
template <typename TI, typename TO, int BT, bool TB>
__device__ __forceinline__ void gemm_ring_body(const GemmArgs& ga, const VBlock vb) {
  typedef Mfma<TI> MF;
  constexpr int BK = 64, kRing = 4, U = BT / 32, F = BT / 32;   // row units of a thread; 16 x 16 blocks of a wave: F x F
  if (!gate_open(ga.g)) return;
  __shared__ u32x4 S[2][2][BT * 8];   // buffer, operand
  const int M = ga.M, N = ga.N, K = ga.K;
  const int64_t lda = ga.lda, ldb = ga.ldb;
  const int m0 = vb.y * BT, n0 = vb.x * BT;
  const TI* A = (const TI*)ga.A + (int64_t)vb.z * ga.sA;
  const TI* B = (const TI*)ga.B + (int64_t)vb.z * ga.sB;
  TO* __restrict__ C = (TO*)ga.C + (int64_t)vb.z * ga.sC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, lr = lane & 15, lg = lane >> 4;
  auto slot = [](int r, int b) { return r * 8 + (b ^ ((r ^ (r >> 3)) & 7)); };
  auto at_most = [](int v, int lim) { return v < lim ? v : lim; };
  // operands contiguous in k: rows ur + 32 u, k 8 ub; B contiguous in n: k 2 kr and 2 kr + 1, n 8 nb
  const int ur = tid >> 3, ub = tid & 7, kr = tid / (BT / 8), nb = tid % (BT / 8);
  const bool pairs = BT == 64 || kr < 32;
  const TI *pa[U], *pb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    pa[u] = A + (int64_t)at_most(m0 + ur + 32 * u, M - 1) * lda;
    pb[u] = TB ? B + (int64_t)at_most(n0 + ur + 32 * u, N - 1) * ldb : B + at_most(n0 + 8 * nb, N - 8);
  }
  constexpr int BU = TB ? U : 2;
  u32x4 ra[kRing][U], rb[kRing][BU];
  auto load = [&](int k0, u32x4 (&va)[U], u32x4 (&vb_)[BU]) {
    const int k = at_most(k0 + 8 * ub, K - 8);
#pragma unroll
    for (int u = 0; u < U; ++u) va[u] = load8(pa[u] + k);
    if constexpr (TB) {
#pragma unroll
      for (int u = 0; u < U; ++u) vb_[u] = load8(pb[u] + k);
    } else if (pairs) {
#pragma unroll
      for (int u = 0; u < 2; ++u) vb_[u] = load8(pb[0] + (int64_t)at_most(k0 + 2 * kr + u, K - 1) * ldb);
    }
  };
  auto store = [&](int k0, int b, const u32x4 (&va)[U], const u32x4 (&vb_)[BU]) {
    const bool kend = k0 + BK > K;   // uniform
#pragma unroll
    for (int u = 0; u < U; ++u) {
      u32x4 v = va[u];
      if (kend) v = drop8(v, k0 + 8 * ub - (K - 8));
      S[b][0][slot(ur + 32 * u, ub)] = v;
    }
    if constexpr (TB) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        u32x4 v = vb_[u];
        if (kend) v = drop8(v, k0 + 8 * ub - (K - 8));
        S[b][1][slot(ur + 32 * u, ub)] = v;
      }
    } else if (pairs) {
      u32x4 x = vb_[0], y = vb_[1];
      if (n0 + BT > N) {
        x = drop8(x, n0 + 8 * nb - (N - 8));
        y = drop8(y, n0 + 8 * nb - (N - 8));
      }
      if (kend) {
        x = k0 + 2 * kr < K ? x : u32x4{0u, 0u, 0u, 0u};
        y = k0 + 2 * kr + 1 < K ? y : u32x4{0u, 0u, 0u, 0u};
      }
      unsigned* w = reinterpret_cast<unsigned*>(&S[b][1][0]);
      const unsigned xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const unsigned a = xs[j / 2], c = ys[j / 2];
        w[slot(nb * 8 + j, kr >> 2) * 4 + (kr & 3)] = j & 1 ? a >> 16 | (c & 0xffff0000u) : (a & 0xffffu) | c << 16;
      }
    }
  };
  typename MF::frag_t acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;
  const int nc = (K + BK - 1) / BK;
#pragma unroll
  for (int d = 0; d < kRing; ++d)
    if (d < nc) load(d * BK, ra[d], rb[d]);
  store(0, 0, ra[0], rb[0]);
  if (kRing < nc) load(kRing * BK, ra[0], rb[0]);
  __syncthreads();
  for (int c0 = 0; c0 < nc; c0 += kRing) {
#pragma unroll
    for (int d = 0; d < kRing; ++d) {
      const int c = c0 + d;
      if (c >= nc) break;
      const int q = (d + 1) % kRing;
      if (c + 1 < nc) {
        store((c + 1) * BK, (c + 1) & 1, ra[q], rb[q]);
        if (c + 1 + kRing < nc) load((c + 1 + kRing) * BK, ra[q], rb[q]);
      }
      const u32x4 *SA = S[c & 1][0], *SB = S[c & 1][1];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const TI *ap[F], *bp[F];
#pragma unroll
        for (int i = 0; i < F; ++i) {
          ap[i] = reinterpret_cast<const TI*>(&SA[slot((wm * F + i) * 16 + lr, ks * 4 + lg)]);
          bp[i] = reinterpret_cast<const TI*>(&SB[slot((wn * F + i) * 16 + lr, ks * 4 + lg)]);
        }
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j) acc[i][j] = MF::mac(ap[i], bp[j], acc[i][j]);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) {
      const int col = n0 + (wn * F + j) * 16 + lr;
      if (col >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + (wm * F + i) * 16 + lg * 4 + r;
        if (row < M) C[(int64_t)row * ga.ldc + col] = out_cvt<TO, float>(acc[i][j][r]);
      }
    }
}

template <typename TI, typename TO, int BT, bool TB, bool GROUPED>
__global__ __launch_bounds__(256, 4) void gemm_ring_kernel(GemmArgs ga_, const GemmArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    VBlock vb = hw_block();
    if (!slice_block(ga_, vb)) return;
    gemm_ring_body<TI, TO, BT, TB>(ga_, vb);
  } else {
    VBlock vb;
    const GemmArgs g = group_args(grp, bmap, vb);
    if (!slice_block(g, vb)) return;
    gemm_ring_body<TI, TO, BT, TB>(g, vb);
  }
}

// FP32 / FP64 slice GEMM with 16-byte global loads (VW elements) along each
// operand's contiguous dimension and LDS tiles kept in that same orientation:
// A~ as [m][k] (or [k][m] when transposed), the right operand as [k][n] (or
// [n][k]).  Rows of the [.][k] tiles carry a 16-byte pad and those of the
// [k][.] tiles a 64-byte pad, so the 16-byte stores and the MFMA operand reads
// (16 rows x 4 k per instruction) hit distinct banks.  4 waves in 2 x 2, each
// owning (BM/2) x (BN/2) as 16 x 16 blocks; the next chunk is prefetched into
// registers while the current one is multiplied.  Out-of-range elements are
// loaded from a clamped address and replaced by zero (no branches per load).
template <typename T, int BM, int BN, int BK, bool TA, bool TB, int VW>
__device__ __forceinline__ void gemm_mn_kernel_body(const GemmArgs& ga, const VBlock vb) {
  typedef Mfma<T> MF;
  typedef typename MF::frag_t frag_t;
  constexpr int KSTEP = MF::KSTEP;
  static_assert(KSTEP == 4 && MF::EPL == 1, "32/64-bit MFMA only");
  constexpr int PADK = 16 / (int)sizeof(T), PADR = 64 / (int)sizeof(T);
  constexpr int LDAK = BK + PADK, LDAM = BM + PADR;   // A as [m][k] / [k][m]
  constexpr int LDBK = BK + PADK, LDBN = BN + PADR;   // B as [n][k] / [k][n]
  constexpr int A_LDS = TA ? BK * LDAM : BM * LDAK;
  constexpr int B_LDS = TB ? BN * LDBK : BK * LDBN;
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 16, FN = WN / 16;
  // vectors per chunk and per thread
  constexpr int A_V = BM * BK / VW, B_V = BN * BK / VW;
  constexpr int A_PER = (A_V + 255) / 256, B_PER = (B_V + 255) / 256;
  static_assert(FM >= 1 && FN >= 1, "tile");
  static_assert(BK % KSTEP == 0 && BK % VW == 0 && BM % VW == 0 && BN % VW == 0, "chunk");

  if (!gate_open(ga.g)) return;
  __shared__ __attribute__((aligned(16))) T As[A_LDS];
  __shared__ __attribute__((aligned(16))) T Bs[B_LDS];

  const int M = ga.M, N = ga.N, K = ga.K;
  const T* __restrict__ A = (const T*)ga.A + (int64_t)vb.z * ga.sA;
  const T* __restrict__ B = (const T*)ga.B + (int64_t)vb.z * ga.sB;
  T* __restrict__ C = (T*)ga.C + (int64_t)vb.z * ga.sC;
  const int64_t lda = ga.lda, ldb = ga.ldb, ldc = ga.ldc;
  const int m0 = vb.y * BM, n0 = vb.x * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int lr = lane & 15, lk = lane >> 4;

  // chunk coordinates of vector u of this thread: (row r, contiguous offset c)
  // A: TA -> rows are k (BK of them), vectors along m; else rows m, vectors along k
  constexpr int A_ROWV = TA ? BM / VW : BK / VW;
  constexpr int B_ROWV = TB ? BK / VW : BN / VW;
  T ra[A_PER][VW], rb[B_PER][VW];
  auto load_chunk = [&](int k0) {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) {
      const int idx = tid + u * 256;
      const int r = idx / A_ROWV, c = (idx - r * A_ROWV) * VW;
      const int gm = m0 + (TA ? c : r), gk = k0 + (TA ? r : c);
      const bool ok = (A_V % 256 == 0 || idx < A_V) && gm < M && gk < K;
      const int64_t off = ok ? (TA ? (int64_t)gk * lda + gm : (int64_t)gm * lda + gk) : 0;
      VecIO<T, VW>::ld(A + off, ra[u]);
      if (!ok) {
#pragma unroll
        for (int v = 0; v < VW; ++v) ra[u][v] = (T)0;
      }
    }
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
      const int idx = tid + u * 256;
      const int r = idx / B_ROWV, c = (idx - r * B_ROWV) * VW;
      const int gn = n0 + (TB ? r : c), gk = k0 + (TB ? c : r);
      const bool ok = (B_V % 256 == 0 || idx < B_V) && gn < N && gk < K;
      const int64_t off = ok ? (TB ? (int64_t)gn * ldb + gk : (int64_t)gk * ldb + gn) : 0;
      VecIO<T, VW>::ld(B + off, rb[u]);
      if (!ok) {
#pragma unroll
        for (int v = 0; v < VW; ++v) rb[u][v] = (T)0;
      }
    }
  };
  auto store_chunk = [&]() {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) {
      const int idx = tid + u * 256;
      if (A_V % 256 == 0 || idx < A_V) {
        const int r = idx / A_ROWV, c = (idx - r * A_ROWV) * VW;
        VecIO<T, VW>::st(&As[r * (TA ? LDAM : LDAK) + c], ra[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
      const int idx = tid + u * 256;
      if (B_V % 256 == 0 || idx < B_V) {
        const int r = idx / B_ROWV, c = (idx - r * B_ROWV) * VW;
        VecIO<T, VW>::st(&Bs[r * (TB ? LDBK : LDBN) + c], rb[u]);
      }
    }
  };

  frag_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = (T)0;

  load_chunk(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
    store_chunk();
    __syncthreads();
    if (k0 + BK < K) load_chunk(k0 + BK);
#pragma unroll
    for (int ks = 0; ks < BK; ks += KSTEP) {
      const T* ap[FM];
      const T* bp[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int m = wm * WM + i * 16 + lr;
        ap[i] = TA ? &As[(ks + lk) * LDAM + m] : &As[m * LDAK + ks + lk];
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = wn * WN + j * 16 + lr;
        bp[j] = TB ? &Bs[n * LDBK + ks + lk] : &Bs[(ks + lk) * LDBN + n];
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = MF::mac(ap[i], bp[j], acc[i][j]);
    }
  }

#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * WN + j * 16 + lr;
      if (col >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + (MF::ROWS_STRIDED ? lk + 4 * r : lk * 4 + r);
        if (row < M) C[(int64_t)row * ldc + col] = acc[i][j][r];
      }
    }
}

template <typename T, int BM, int BN, int BK, bool TA, bool TB, int VW, bool GROUPED>
__global__ __launch_bounds__(256) void gemm_mn_kernel(GemmArgs ga_, const GemmArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    VBlock vb = hw_block();
    if (!slice_block(ga_, vb)) return;
    gemm_mn_kernel_body<T, BM, BN, BK, TA, TB, VW>(ga_, vb);
  } else {
    VBlock vb;
    const GemmArgs g = group_args(grp, bmap, vb);
    if (!slice_block(g, vb)) return;   // the instance's grid may be padded
    gemm_mn_kernel_body<T, BM, BN, BK, TA, TB, VW>(g, vb);
  }
}

// FP32 slice GEMM on the BF16 matrix cores.  An FP32 number is the exact sum of
// three bfloat16 numbers (3 x 8 significant bits, each the round-to-nearest of
// what the ones before it leave), so the product of two is nine BF16 products,
// each exact in FP32.  The three smallest (second x third, third x second,
// third x third: below 2^-26 of the whole) are left out, the other six are
// accumulated in FP32, the small ones first, by the 16x16x32 instruction,
// which runs 16 times as many operations per cycle as the FP32 16x16x4: 6 / 16
// of its matrix-core time, with one rounding per 32 k and product where the
// FP32 instruction makes one per 4 k.  On uniform random operands the relative
// 2-norm error against FP64 is 3.35e-7 (FP32 instruction: 4.03e-7) at K = 512,
// 4.8e-7 (5.7e-7) at K = 1024, 2.3e-7 (2.9e-7) at K = 256, 1.3e-7 (1.8e-7) at
// K = 96.
//
// Tile: BM x BN outputs per workgroup.  A thread loads 8 consecutive k of one
// row of A~ (and of one column of the right operand: 8 loads, each coalesced
// along n), splits them in registers (5.5 VALU operations per element) and
// writes the three planes to LDS as 16-byte units of 8 k, so the MFMA operands
// are single 16-byte reads and the transposition of the right operand costs
// nothing.  Unit q of row r is stored at r * 4 + (q ^ (r / 2 % 4)): stores and
// reads of 8 consecutive lanes hit 8 different bank groups without padding.
// The next chunk's loads are in flight while the current one is multiplied.
// Bounds are the buffer descriptors': rows beyond the slice read as zeros.
// What is read beyond K in a row of A~ (the next row's start) meets a zero row
// of the right operand; with both operands contiguous in k (TB) the last chunk
// of A~ is zeroed explicitly.
// Bound: neither memory nor the matrix cores, which are busy 45 % of the time,
// but what happens between a chunk's two barriers (the splitting's vector work and
// the LDS traffic of three planes) and, with one tile per CU, the results leaving
// at the end (13 us of 64 x 512^3).  Kernel times, FP32 instruction before -> now:
// 64 x 512^3 139 -> 83 us, 3 x 1024^3 67 -> 46, 32 x 256^3 16.3 -> 12.4.
//
// The split does not represent infinities and NaN (their remainders are NaN),
// values that round to infinity in bfloat16, nor all 24 bits of numbers below
// 2^-110 (the third part ends at 2^-133: such a number loses up to 2^-134).  A
// tile in which that may show is computed again with the FP32 instruction, in
// the order of gemm_mn_kernel (split_again): where a result is not finite, and
// where K losses, times the largest number they can meet, reach 2^-26 of a
// result.  For losses of the data that number is the operator's largest, known
// since its creation, so only tiles with small results or zeros look at their
// data; an operator that holds such numbers has every tile do so.  In a Krylov
// step the data is of norm 1 and neither is needed.  No number is tested in the
// loop (that cost 49 -> 54 us at 3 x 1024^3), and results that are merely small
// cost nothing: the BF16 instruction keeps subnormal operands and results.
// Between events on random data, 64 x 512^3: 106 us, 126 where every tile looks
// at its data, 290 where every tile is computed again; 3 x 1024^3: 49, 59 and 140.
struct Split8 {
  uint4 h[3];
};
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  unsigned w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      const unsigned q = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
      w[h][i] = q;
      a -= __builtin_bit_cast(float, q << 16);
      b -= __builtin_bit_cast(float, q & 0xffff0000u);
    }
  }
  Split8 s;
#pragma unroll
  for (int h = 0; h < 3; ++h) s.h[h] = make_uint4(w[h][0], w[h][1], w[h][2], w[h][3]);
  return s;
}

// Raw buffer descriptor of `n` floats from p (at most 2 GiB).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t float_buffer(const float* p, int64_t n) {
  const int64_t cap = 0x1fffffff;
  n = n < 0 ? 0 : (n < cap ? n : cap);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), (short)0, (int)(n * 4), 0x00020000);
}

typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) unsigned lds_uint;
constexpr int kSplitSeen = 5;
// twice the bits of the least magnitude to which K losses of 2^-134 times `top` stay below 2^-26
__device__ inline unsigned split_reach(int K, float top) {
  return 2u * __builtin_bit_cast(unsigned, 0x1p-108f * (float)K * top);
}

// What follows a tile whose results may show a loss (seen[0]: one is not finite,
// seen[1]: one is within reach of the data's), or whose operator holds numbers
// that lose bits: the tile's data is read for its largest magnitude (seen[2])
// and numbers that lose bits (seen[3]), and if a result is within reach of
// either's losses, the tile is computed again with the FP32 instruction,
// operands staged as they are.  `least` is twice the bits of the least magnitude
// among the lane's results, `small` whether the operator holds such numbers.
// Nothing of the split loop is taken over, the arguments neither (they are read
// again through gp): what both would share cost registers in the loop (14.7 ->
// 15.9 us at 31 x 243 x 211 x 197).
template <int BM, int BN, int NT, int WGM, int WGN, bool TB>
__device__ __forceinline__ void split_again(const GemmArgs* gp, int bx, int by, int bz, unsigned least, unsigned small,
                                            lds_float* As, lds_float* Bs, lds_uint* seen) {
  constexpr int BK = 32, LD = BK + 4;
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  static_assert(LD <= 3 * BK / 2, "the rows fit the three planes");
  const GemmArgs& ga = *gp;
  const int M = ga.M, N = ga.N, K = ga.K;
  const int64_t lda = ga.lda, ldb = ga.ldb;
  const int m0 = by * BM, n0 = bx * BN;
  const float* A = (const float*)ga.A + (int64_t)bz * ga.sA;
  const float* B = (const float*)ga.B + (int64_t)bz * ga.sB;
  float* C = (float*)ga.C + (int64_t)bz * ga.sC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN, lr = lane & 15, lg = lane >> 4;

  if (seen[0] == 0) {
    unsigned top = 0, low = ~0u;   // twice the bits of the largest magnitude, of the least above 0 minus 1
    auto see = [&](float x) {
      const unsigned t = __builtin_bit_cast(unsigned, x) << 1;
      top = max(top, t);
      low = min(low, t - 1u);
    };
    // four elements of a row from i, or its last four (no branch per load: it would be waited for)
    auto see4 = [&](const float* row, int i, int len) {
      typedef float f32x4_un __attribute__((ext_vector_type(4), aligned(4)));
      const f32x4_un v = *reinterpret_cast<const f32x4_un*>(row + min(i, len - 4));
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float x = v[q];
        see(x);
      }
    };
    const int rows = min(BM, M - m0);
    if (!ga.range.right && N >= 4) {          // columns of B (never TB)
      constexpr int TPR = BN / 4;
#pragma unroll 16
      for (int k = tid / TPR; k < K; k += NT / TPR) see4(B + (int64_t)k * ldb, n0 + tid % TPR * 4, N);
    } else if (ga.range.right && K >= 4) {    // rows of A
      const int units = (K + 3) / 4;
      int r = tid / units, q = tid % units;
#pragma unroll 8
      for (int i = tid; i < rows * units; i += NT) {
        see4(A + (int64_t)(m0 + r) * lda, q * 4, K);
        q += NT;
        const int rr = q / units;
        r += rr;
        q -= rr * units;
      }
    } else if (!ga.range.right) {
      for (int i = tid; i < K * N; i += NT) see(B[(int64_t)(i / N) * ldb + i % N]);
    } else {
      for (int i = tid; i < rows * K; i += NT) see(A[(int64_t)(m0 + i / K) * lda + i % K]);
    }
    for (int d = 32; d > 0; d >>= 1) top = max(top, (unsigned)__shfl_xor((int)top, d));
    if (lane == 0) __hip_atomic_fetch_max(&seen[2], top >> 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (__any(low < 2u * kSplitLow - 1u)) seen[3] = 1;
    __syncthreads();
    if (small != 0 && __any(least < split_reach(K, __builtin_bit_cast(float, seen[2])))) seen[4] = 1;
    __syncthreads();
    if (seen[4] == 0 && (seen[1] == 0 || seen[3] == 0)) return;
  }

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // a chunk's operands in registers while the one before is multiplied; rows
  // and columns beyond an operand repeat its last one, k beyond K are zeros
  constexpr int RA = BM * BK / NT, RB = BN * BK / NT;
  const int kk = tid % BK, r0 = tid / BK, kb = tid / BN, cb = min(n0 + tid % BN, N - 1);
  float ra[RA], rb[RB];
  auto load = [&](int k0) {
    const int ka = min(k0 + kk, K - 1);
#pragma unroll
    for (int u = 0; u < RA; ++u) ra[u] = A[(int64_t)min(m0 + r0 + u * (NT / BK), M - 1) * lda + ka];
#pragma unroll
    for (int u = 0; u < RB; ++u)
      rb[u] = TB ? B[(int64_t)min(n0 + r0 + u * (NT / BK), N - 1) * ldb + ka]
                 : B[(int64_t)min(k0 + kb + u * (NT / BN), K - 1) * ldb + cb];
  };
  load(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < RA; ++u) As[(r0 + u * (NT / BK)) * LD + kk] = k0 + kk < K ? ra[u] : 0.0f;
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int k = TB ? kk : kb + u * (NT / BN), c = TB ? r0 + u * (NT / BK) : tid % BN;
      Bs[c * LD + k] = k0 + k < K ? rb[u] : 0.0f;
    }
    __syncthreads();
    if (k0 + BK < K) load(k0 + BK);
#pragma unroll 2
    for (int ks = 0; ks < BK; ks += 4) {
      float bf[FN];
#pragma unroll
      for (int j = 0; j < FN; ++j) bf[j] = Bs[(wn * WN + j * 16 + lr) * LD + ks + lg];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const float af = As[(wm * WM + i * 16 + lr) * LD + ks + lg];
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af, bf[j], acc[i][j], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * WN + j * 16 + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + lg * 4 + r;
        if (row < M && col < N) C[(int64_t)row * ga.ldc + col] = acc[i][j][r];
      }
    }
}

// The same through a call, for kernels whose loop takes every register (inlined,
// 256 x 256 spilled some of them, 3 MB a launch at 64 x 512^3, and five workgroups
// of 64 x 64 a CU lost 4 % to fewer registers in the loop); elsewhere the call's
// scratch costs more (batches 0.7 %).
template <int BM, int BN, int NT, int WGM, int WGN, bool TB>
static __device__ __attribute__((noinline)) void split_again_call(const GemmArgs* gp, int bx, int by, int bz, unsigned least,
                                                                  unsigned small, lds_float* As, lds_float* Bs, lds_uint* seen) {
  split_again<BM, BN, NT, WGM, WGN, TB>(gp, bx, by, bz, least, small, As, Bs, seen);
}

template <int BM, int BN, int NT, int WGM, int WGN, bool CALL, bool TB>
__device__ __forceinline__ void gemm_split_kernel_body(const GemmArgs& ga, const GemmArgs* gp, const VBlock vb) {
  constexpr int BK = 32;
  constexpr int WM = BM / WGM, WN = BN / WGN, FM = WM / 16, FN = WN / 16;
  constexpr int AU = BM * 4 / NT, BU = BN * 4 / NT;   // 8-element units per thread and chunk
  static_assert(WGM * WGN * 64 == NT && AU * NT == BM * 4 && BU * NT == BN * 4, "tile");
  static_assert(NT % BN == 0 || BN % NT == 0, "columns of a unit");
  if (!gate_open(ga.g)) return;
  __shared__ uint4 As[3][BM * 4];
  __shared__ uint4 Bs[3][BN * 4];
  __shared__ unsigned seen[kSplitSeen];
  const int M = ga.M, N = ga.N, K = ga.K;
  const float* A = (const float*)ga.A + (int64_t)vb.z * ga.sA;
  const float* B = (const float*)ga.B + (int64_t)vb.z * ga.sB;
  float* C = (float*)ga.C + (int64_t)vb.z * ga.sC;
  const int lda = (int)ga.lda, ldb = (int)ga.ldb;   // below 2^20 (split_shape_ok)
  const int m0 = vb.y * BM, n0 = vb.x * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int lr = lane & 15, lg = lane >> 4;

  // byte offsets from the tile's first row (A~, TB) or column of a chunk
  const int oa = ((tid >> 2) * lda + (tid & 3) * 8) * 4;
  const int ob = TB ? ((tid >> 2) * ldb + (tid & 3) * 8) * 4 : (tid / BN * 8 * ldb + tid % BN) * 4;
  const float* At = A + (int64_t)m0 * lda;
  const float* Bt = TB ? B + (int64_t)n0 * ldb : B + n0;
  const int64_t na = (int64_t)(M - 1 - m0) * lda + K, nb = TB ? (int64_t)(N - 1 - n0) * ldb + K : (int64_t)K * ldb - n0;
  float ra[AU][8], rb[BU][8];
  auto load8 = [&](const __amdgpu_buffer_rsrc_t& q, int o, float (&v)[8]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const f32x4 w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(q, o + 16 * h, 0, 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * h + i] = w[i];
    }
  };
  auto load_chunk = [&](int k0) {
    const __amdgpu_buffer_rsrc_t qa = float_buffer(At + k0, na - k0);
#pragma unroll
    for (int u = 0; u < AU; ++u) load8(qa, oa + u * (NT / 4) * lda * 4, ra[u]);
    if constexpr (TB) {
      const __amdgpu_buffer_rsrc_t qb = float_buffer(Bt + k0, nb - k0);
#pragma unroll
      for (int u = 0; u < BU; ++u) load8(qb, ob + u * (NT / 4) * ldb * 4, rb[u]);
      if (k0 + BK > K) {
#pragma unroll
        for (int u = 0; u < AU; ++u)
#pragma unroll
          for (int i = 0; i < 8; ++i) ra[u][i] = k0 + (tid & 3) * 8 + i < K ? ra[u][i] : 0.0f;
      }
    } else {
      const __amdgpu_buffer_rsrc_t qb = float_buffer(Bt + (int64_t)k0 * ldb, nb - (int64_t)k0 * ldb);
#pragma unroll
      for (int u = 0; u < BU; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          rb[u][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(qb, ob + (u * (NT / BN * 8) + i) * ldb * 4, 0, 0));
    }
  };
  auto put = [&](uint4* S, int plane, int r, int q, const float (&v)[8]) {
    const Split8 s = split8(v);
    const int at = r * 4 + (q ^ ((r >> 1) & 3));
#pragma unroll
    for (int h = 0; h < 3; ++h) S[h * plane + at] = s.h[h];
  };
  auto store_chunk = [&]() {
#pragma unroll
    for (int u = 0; u < AU; ++u) {
      const int i = tid + u * NT;
      put(&As[0][0], BM * 4, i >> 2, i & 3, ra[u]);
    }
#pragma unroll
    for (int u = 0; u < BU; ++u) {
      const int i = tid + u * NT;
      if (TB) put(&Bs[0][0], BN * 4, i >> 2, i & 3, rb[u]);
      else put(&Bs[0][0], BN * 4, i % BN, i / BN, rb[u]);
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // the operator's range, or, where the data has norm 1 and the operators are not tiny, one that nothing reaches
  const unsigned *rg = ga.range.at, both = ga.range.unit == 2 ? min(rg[0], rg[2]) : rg[0];
  const unsigned top_ = rg[2 * ga.range.right], low_ = ~rg[2 * ga.range.right + 1];
  load_chunk(0);
  const bool near = ga.range.unit != 0 && __builtin_amdgcn_readfirstlane(both) >= (127u - 40u) << 23;
  const unsigned top = near ? 0u : __builtin_amdgcn_readfirstlane(top_), small = !near && (unsigned)__builtin_amdgcn_readfirstlane(low_) < kSplitLow - 1u;
  if (tid < kSplitSeen) seen[tid] = 0;
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
    store_chunk();
    __syncthreads();
    if (k0 + BK < K) load_chunk(k0 + BK);
    bf16x8 bf[FN][3];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = wn * WN + j * 16 + lr;
#pragma unroll
      for (int h = 0; h < 3; ++h) bf[j][h] = __builtin_bit_cast(bf16x8, Bs[h][n * 4 + (lg ^ ((n >> 1) & 3))]);
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int m = wm * WM + i * 16 + lr;
      bf16x8 af[3];
#pragma unroll
      for (int h = 0; h < 3; ++h) af[h] = __builtin_bit_cast(bf16x8, As[h][m * 4 + (lg ^ ((m >> 1) & 3))]);
      constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[pa[q]], bf[j][pb[q]], acc[i][j], 0, 0, 0);
    }
  }

  // The least and the largest of twice the results' magnitudes in bits.  What lies
  // beyond the operands is zeros, which do not count, but for columns beyond a B
  // contiguous in n: those are the next row's data, and may stay.  Agreed on before
  // the results leave: a barrier after the stores would wait for them.
  unsigned least = ~0u, most = 0;
  auto look = [&](auto edge_c) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        unsigned l = ~0u;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const float v = acc[i][j][r];
          const unsigned t = __builtin_bit_cast(unsigned, v) << 1;
          l = min(l, !TB || !decltype(edge_c)::value || n0 + wn * WN + j * 16 + lr < N ? t : ~0u);
          most = max(most, t);
        }
        if (decltype(edge_c)::value) l = m0 + wm * WM + i * 16 + lg * 4 + r < M ? l : ~0u;
        least = min(least, l);
      }
  };
  if (m0 + BM <= M && (!TB || n0 + BN <= N)) look(std::false_type{});
  else look(std::true_type{});
  if (__any(most >= 0xff000000u)) seen[0] = 1;
  if (__any(least < split_reach(K, __builtin_bit_cast(float, top)))) seen[1] = 1;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int col = n0 + wn * WN + j * 16 + lr;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WM + i * 16 + lg * 4 + r;
        if (row < M && col < N) C[(int64_t)row * ga.ldc + col] = acc[i][j][r];
      }
    }
  if ((seen[0] | seen[1]) != 0 || small != 0) {
    lds_float *la = (lds_float*)&As[0][0], *lb = (lds_float*)&Bs[0][0];
    if constexpr (CALL) split_again_call<BM, BN, NT, WGM, WGN, TB>(gp, vb.x, vb.y, vb.z, least, small, la, lb, (lds_uint*)seen);
    else split_again<BM, BN, NT, WGM, WGN, TB>(gp, vb.x, vb.y, vb.z, least, small, la, lb, (lds_uint*)seen);
  }
}

template <int BM, int BN, int NT, int WGM, int WGN, int WAVES, bool TB, bool GROUPED>
__global__ __launch_bounds__(NT, WAVES) void gemm_split_kernel(GemmArgs ga_, const GemmArgs* grp, const int4* bmap) {
  constexpr bool CALL = BM >= 256 || WAVES > 4;   // no registers to spare
  if constexpr (!GROUPED) {
    VBlock vb = hw_block();
    if (!slice_block(ga_, vb)) return;
    // (the arguments where the kernel finds them: the first one, from the segment's start)
    gemm_split_kernel_body<BM, BN, NT, WGM, WGN, CALL, TB>(ga_, (const GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr(), vb);
  } else {
    VBlock vb;
    const GemmArgs g = group_args(grp, bmap, vb);
    if (!slice_block(g, vb)) return;   // the instance's grid may be padded
    gemm_split_kernel_body<BM, BN, NT, WGM, WGN, CALL, TB>(g, grp + bmap[blockIdx.x].x, vb);
  }
}

template <typename T, int BM, int BN, int BK>
static hipError_t launch_gemm_mn(dctk_ctx ctx, hipStream_t s, GemmArgs ga, int ta, int tb, bool vec,
                                 int batch) {
  ga.nbatch = batch >= kSliceXcdMin ? batch : 0;
  const int gz = ga.nbatch > 0 ? (batch + 7) / 8 * 8 : batch;
  const dim3 grid((unsigned)((ga.N + BN - 1) / BN), (unsigned)((ga.M + BM - 1) / BM), (unsigned)gz);
  constexpr int VW = 16 / (int)sizeof(T);
#define DCTK_GMN(TA_, TB_, VW_) return launch_kernel(ctx, s, gemm_mn_kernel<T, BM, BN, BK, TA_, TB_, VW_, false>, gemm_mn_kernel<T, BM, BN, BK, TA_, TB_, VW_, true>, grid, 256, 0, ga)
#define DCTK_GMN_V(TA_, TB_)    \
  do {                          \
    if (vec) DCTK_GMN(TA_, TB_, VW); \
    DCTK_GMN(TA_, TB_, 1);      \
  } while (0)
  if constexpr (sizeof(T) == 8) {   // FP32 operators keep A~ transposed
    if (ta && !tb) DCTK_GMN_V(true, false);
  }
  if (ta) return hipErrorInvalidValue;
  if (!tb) DCTK_GMN_V(false, false);
  DCTK_GMN_V(false, true);
#undef DCTK_GMN_V
#undef DCTK_GMN
}

template <int BM, int BN, int NT, int WGM, int WGN, int WAVES>
static hipError_t launch_gemm_split(dctk_ctx ctx, hipStream_t s, GemmArgs ga, int tb, int batch) {
  ga.nbatch = batch >= kSliceXcdMin ? batch : 0;
  const int gz = ga.nbatch > 0 ? (batch + 7) / 8 * 8 : batch;
  const dim3 grid((unsigned)((ga.N + BN - 1) / BN), (unsigned)((ga.M + BM - 1) / BM), (unsigned)gz);
#define DCTK_GSP(TB_) return launch_kernel(ctx, s, gemm_split_kernel<BM, BN, NT, WGM, WGN, WAVES, TB_, false>, gemm_split_kernel<BM, BN, NT, WGM, WGN, WAVES, TB_, true>, grid, NT, 0, ga)
  if (tb) DCTK_GSP(true);
  DCTK_GSP(false);
#undef DCTK_GSP
}

// The split kernel's offsets within a tile are 32-bit (256 rows of lda, or 32
// of ldb, floats).
static bool split_shape_ok(int64_t lda, int64_t ldb) { return lda < (1 << 20) && ldb < (1 << 20); }

// Output tile edge of the split kernel: 256, 128 or 64, the one of least
// estimated time per 32-long chunk, from what a tile of each takes while the
// chip is full (64 x 512^3: 94, 98 and 118 us, i.e. 5.9, 1.53 and 0.46 us per
// tile, chunk and CU) and from what a chunk takes at least, its loads' latency
// (2.0 us with 128 x 128 tiles, 3 x 1024^3: 63 us; 1.4 us with 64 x 64, 32 x
// 256^3: 12.4 us against 20.0).
static int split_tile(int M, int N, int batch, int num_cus) {
  auto rounds = [&](int t) {
    const int64_t tiles = (int64_t)((M + t - 1) / t) * ((N + t - 1) / t) * batch;
    return (double)((tiles + num_cus - 1) / num_cus);
  };
  const double c256 = 5.9 * rounds(256), c128 = std::max(2.0, 1.53 * rounds(128)), c64 = std::max(1.4, 0.46 * rounds(64));
  return c256 <= c128 && c256 <= c64 ? 256 : (c128 <= c64 ? 128 : 64);
}

// FP32 / FP64 GEMMs with the output in the input type.  FP32 takes the split
// kernel from 64 x 64 tiles up while those cover the CUs.  Below that (and for
// FP64 and operands the split kernel does not take) the FP32 / FP64
// instructions with 64 x 64 tiles while they cover the CUs, else 32 x 32 (31 x
// 96^3 FP32: 4.2 us, split 64 x 64 5.1: too few workgroups).  A tile of 128
// asked for takes 256 x 256 where that is the one of least estimated time.
template <typename T>
static hipError_t launch_gemm_vec(dctk_ctx ctx, hipStream_t s, int M, int N, int K, const void* A, int64_t lda,
                                  int64_t sA, int ta, const void* B, int64_t ldb, int64_t sB, int tb, void* C,
                                  int64_t ldc, int64_t sC, int batch, Gate g, int num_cus, int tile,
                                  const OperandRange& range) {
  GemmArgs ga{};
  ga.range = range;
  ga.M = M;
  ga.N = N;
  ga.K = K;
  ga.A = A;
  ga.lda = lda;
  ga.sA = sA;
  ga.B = B;
  ga.ldb = ldb;
  ga.sB = sB;
  ga.C = C;
  ga.ldc = ldc;
  ga.sC = sC;
  ga.g = g;
  constexpr int VW = 16 / (int)sizeof(T);
  const bool vec = M % VW == 0 && N % VW == 0 && K % VW == 0 && lda % VW == 0 && ldb % VW == 0 &&
                   sA % VW == 0 && sB % VW == 0 && ((uintptr_t)A % 16) == 0 && ((uintptr_t)B % 16) == 0;
  const int64_t t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch;
  constexpr int BK = sizeof(T) == 8 ? 16 : 32;
  if constexpr (sizeof(T) == 4) {
    if (split_shape_ok(lda, ldb)) {
      const int best = split_tile(M, N, batch, num_cus);
      if ((tile == 128 || (tile == 0 && t64 >= (int64_t)num_cus)) && best == 256)
        return launch_gemm_split<256, 256, 512, 2, 4, 2>(ctx, s, ga, tb, batch);
      if (tile == 128 || (tile == 0 && t64 >= (int64_t)num_cus && best == 128))
        return launch_gemm_split<128, 128, 256, 2, 2, 2>(ctx, s, ga, tb, batch);
      if (tile == 64 || (tile == 0 && t64 >= (int64_t)num_cus)) {
        // four workgroups a CU, or, where that saves a round, five in fewer registers (31 x 352^3: 32.4 us with
        // four, 30.7 with five; where it saves none, 32 x 256^3: 16.4 and 17.3)
        const int64_t r4 = (t64 + 4 * num_cus - 1) / (4 * num_cus), r5 = (t64 + 5 * num_cus - 1) / (5 * num_cus);
        if (r5 < r4) return launch_gemm_split<64, 64, 256, 2, 2, 5>(ctx, s, ga, tb, batch);
        return launch_gemm_split<64, 64, 256, 2, 2, 4>(ctx, s, ga, tb, batch);
      }
    }
  }
  if (tile == 64 || tile == 128 || (tile == 0 && t64 >= (int64_t)num_cus))
    return launch_gemm_mn<T, 64, 64, BK>(ctx, s, ga, ta, tb, vec, batch);
  return launch_gemm_mn<T, 32, 32, BK>(ctx, s, ga, ta, tb, vec, batch);
}

template <typename TI, typename TO>
static hipError_t launch_gemm_t(dctk_ctx ctx, hipStream_t s, int M, int N, int K, const void* A, int64_t lda, int64_t sA,
                                int ta, const void* B, int64_t ldb, int64_t sB, int tb, void* C, int64_t ldc,
                                int64_t sC, int batch, Gate g, int num_cus, int tile) {
  if (ta) return hipErrorInvalidValue;   // 16-bit operators keep A~ transposed
  GemmArgs ga{};
  ga.nbatch = batch >= kSliceXcdMin ? batch : 0;
  const int gz = ga.nbatch > 0 ? (batch + 7) / 8 * 8 : batch;
  ga.M = M;
  ga.N = N;
  ga.K = K;
  ga.A = A;
  ga.lda = lda;
  ga.sA = sA;
  ga.B = B;
  ga.ldb = ldb;
  ga.sB = sB;
  ga.C = C;
  ga.ldc = ldc;
  ga.sC = sC;
  ga.g = g;
  auto grid = [&](int bm, int bn) { return dim3((unsigned)((N + bn - 1) / bn), (unsigned)((M + bm - 1) / bm), (unsigned)gz); };
#define DCTK_GEMM16(KERNEL, BM, BN, ...)                                                                \
  do {                                                                                                  \
    if (tb) return launch_kernel(ctx, s, KERNEL(true, false, __VA_ARGS__), KERNEL(true, true, __VA_ARGS__), grid(BM, BN), 256, 0, ga); \
    return launch_kernel(ctx, s, KERNEL(false, false, __VA_ARGS__), KERNEL(false, true, __VA_ARGS__), grid(BM, BN), 256, 0, ga);       \
  } while (0)
#define DCTK_TILED(TB_, GR, BM, BN, VEC) gemm_kernel<TI, TO, BM, BN, TB_, VEC, GR>
#define DCTK_RING(TB_, GR, BT) gemm_ring_kernel<TI, TO, BT, TB_, GR>
  // shorter than a unit: scalar loads (32 x 32 tiles: the result is a few columns, or the sums short)
  if (K < 8 || (!tb && N < 8)) DCTK_GEMM16(DCTK_TILED, 32, 32, 32, 32, false);
  // 128 x 128 tiles while they give every CU two, then 64 x 64 when they
  // fill the chip, 32 x 32 otherwise.
  const int64_t tiles256 = (int64_t)((M + 255) / 256) * ((N + 255) / 256) * batch;
  const int64_t tiles128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128) * batch;
  int64_t tiles64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch;
  // 256 x 128 while 256 x 256 blocks still give every CU one (each operand
  // byte staged serves 4/3 the flops of a 128 x 128 tile, and two workgroups
  // of 4 waves per CU hide more latency than one of 8 with 256 x 256 tiles)
  if (tile == 256 || (tile == 0 && M >= 256 && N >= 256 && tiles256 >= (int64_t)num_cus))
    DCTK_GEMM16(DCTK_TILED, 256, 128, 256, 128, true);
  if (tile == 128 || (tile == 0 && tiles128 >= 2 * (int64_t)num_cus)) DCTK_GEMM16(DCTK_TILED, 128, 128, 128, 128, true);
  if (tile == 64 || (tile == 0 && tiles64 >= 2 * (int64_t)num_cus)) DCTK_GEMM16(DCTK_RING, 64, 64, 64);
  DCTK_GEMM16(DCTK_RING, 32, 32, 32);
#undef DCTK_RING
#undef DCTK_TILED
#undef DCTK_GEMM16
}

static int g_num_cus = 256;

hipError_t launch_gemm(dctk_ctx ctx, hipStream_t s, int in_dtype, int out_acc, int M, int N, int K,
                       const void* A, int64_t lda, int64_t sA, int ta,
                       const void* B, int64_t ldb, int64_t sB, int tb,
                       void* C, int64_t ldc, int64_t sC, int batch, Gate g, int tile, const OperandRange& range) {
  // out_acc = 1: output in the accumulator type; 0: output in the input type
  switch (in_dtype) {
    case DCTK_F64:
      return launch_gemm_vec<double>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile, range);
    case DCTK_F32:
      return launch_gemm_vec<float>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile, range);
    case DCTK_BF16:
      if (out_acc)
        return launch_gemm_t<bf16_t, float>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile);
      return launch_gemm_t<bf16_t, bf16_t>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile);
    case DCTK_F16:
      if (out_acc)
        return launch_gemm_t<f16_t, float>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile);
      return launch_gemm_t<f16_t, f16_t>(ctx, s, M, N, K, A, lda, sA, ta, B, ldb, sB, tb, C, ldc, sC, batch, g, g_num_cus, tile);
    default:
      return hipErrorInvalidValue;
  }
}

// ---- the c-product and its adjoint on an operator's workspaces ---------------
static size_t dtype_size(int dt) { return dt == DCTK_F64 ? 8 : (dt == DCTK_F32 ? 4 : 2); }

bool fused_eligible(dctk_op op) {
  const int64_t nmax = op->n1 > op->n2 ? op->n1 : op->n2;
  const bool small_offsets = op->p * op->n1 * op->n2 < (int64_t(1) << 31) && op->p * nmax * op->s < (int64_t(1) << 31);
  return !op->two_sided && op->p <= kFusedMaxP && small_offsets;
}

// Without a tuned choice: the fused product while the problem is small enough to
// be latency-bound (fewer 32 x 32 output tiles than CUs) and its in-register
// transforms are cheap (p <= 4; FP64, whose transforms cost the unfused path
// more, also p <= 8 with slices up to 112^3); else transform, GEMM, transform.
// Time per product, fused / three kernels (us): FP32 p = 3, n = 256: 6.7 /
// 12.9, n = 230: 12.9 / 14.6; p = 5, n = 64: 13.9 / 12.5; p = 8, n = 32: 18.5 /
// 13.7, n = 128: 29.0 / 15.7, n = 192: 40.5 / 18.1; BF16 p = 8, n = 128: 31.3 /
// 16.9; FP64 p = 8, n = 96: 17.3 / 19.0, n = 115: 29.2 / 23.9, p = 5, n = 153:
// 23.7 / 22.0.
bool use_fused(dctk_op op, int adjoint) {
  const int path = op->tune[adjoint ? 1 : 0][0];
  if (path >= 0) return path == 1;
  const int64_t M = adjoint ? op->n2 : op->n1, K = adjoint ? op->n1 : op->n2, N = op->s;
  const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32);
  return t32 < g_num_cus && (op->p <= 4 || (op->gemm_dtype == DCTK_F64 && M * N * K <= (int64_t)112 * 112 * 112));
}

// The GEMM's gate under a product's control block: it runs unless the process
// stopped at an earlier step.
static Gate gemm_gate(const Ctl& ctl) {
  Gate g{nullptr, 0, 0};
  if (ctl.kind != CTL_PLAIN) {
    g.st = ctl.st;
    g.j = ctl.kind == CTL_ARN_FWD ? ctl.j - 1 : ctl.j;
    const bool fwd = ctl.kind == CTL_GKB_FWD || ctl.kind == CTL_GKB_FWDU;
    g.mode = fwd ? 0 : 1;
    if (fwd) g.j = ctl.j;
  }
  return g;
}

// Step 2 of a three-kernel product: the slice products of X~ (op->xh) into op->ch.
// In a Krylov step X~ is that of a vector of norm 1, or near it (OperandRange's
// unit): what the FP32 operands lose below 2^-110 is then far below the product's
// rounding, unless an operator itself is that small (the kernel sees to that),
// and nothing has to be looked for.
static hipError_t slice_gemms(dctk_op op, hipStream_t s, int adjoint, const Ctl& ctl) {
  dctk_ctx ctx = op->ctx;
  const int tile = op->tune[adjoint ? 1 : 0][1];
  const int64_t p = op->p, n1 = op->n1, n2 = op->n2, sc = op->s;
  const int gdt = op->gemm_dtype;
  const int64_t rin = adjoint ? n1 : n2;
  const int64_t rout = adjoint ? n2 : n1;
  const int64_t sAh = n1 * n2;
  hipError_t e;
  prof_begin(ctx, PROF_GEMM);
  // the left operand: A~ (n1 x n2), or for the adjoint A~^T (n2 x n1) -- read
  // from the transposed copy that all but FP64 operators keep
  const bool tcopy = adjoint && op->AhT != nullptr;
  const void* Aop = tcopy ? op->AhT : op->Ah;
  const int64_t ldA = tcopy ? n1 : n2;
  const int tA = adjoint && !tcopy ? 1 : 0;
  const Gate g = gemm_gate(ctl);
  const int unit = ctl.kind != CTL_PLAIN ? 1 + op->two_sided : 0;
  const OperandRange ra{op->range, 0, unit}, rb{op->range, 1, unit};
  if (!op->two_sided) {
    // forward: (n1 x n2)(n2 x s);  adjoint: (n2 x n1 := A~^T)(n1 x s)
    e = launch_gemm(ctx, s, gdt, 1, (int)rout, (int)sc, (int)rin, Aop, ldA, sAh, tA,
                    op->xh, sc, rin * sc, 0, op->ch, sc, rout * sc, (int)p, g, tile, ra);
  } else {
    e = launch_gemm(ctx, s, gdt, 0, (int)rout, (int)sc, (int)rin, Aop, ldA, sAh, tA,
                    op->xh, sc, rin * sc, 0, op->th, sc, rout * sc, (int)p, g, tile, ra);
    // right factor: forward (rout x s)(s x s) with B~; adjoint with B~^T
    if (e == hipSuccess)
      e = launch_gemm(ctx, s, gdt, 1, (int)rout, (int)sc, (int)sc, op->th, sc, rout * sc, 0,
                      op->Bh, sc, sc * sc, adjoint ? 1 : 0, op->ch, sc, rout * sc, (int)p, g, tile,
                      rb);
  }
  prof_end(ctx, PROF_GEMM);
  return e;
}

bool pair_eligible(dctk_op op) {
  // short tubes only with FP32 slice products: pairing rounds the next product's
  // input from the unnormalised vector, and 16-bit short-tube solves keep their roundings
  if (op->p < 16 && op->gemm_dtype != DCTK_F32) return false;
  return !op->fast && tube_pair_ok(op->p, op->vec_dtype) &&
         !(fused_eligible(op) && (use_fused(op, 0) || use_fused(op, 1)));
}

hipError_t pair_first(dctk_op op, hipStream_t s, int adjoint, const void* X, const Ctl& ctl) {
  dctk_ctx ctx = op->ctx;
  const int64_t pp = op->p * op->p;
  const int64_t rin = adjoint ? op->n1 : op->n2;
  const int gi = adjoint ? 2 : 0;
  prof_begin(ctx, PROF_TUBE_FWD);
  hipError_t e = launch_tube(ctx, s, op->vec_dtype, op->gemm_dtype, op->p, rin * op->s, X, op->xh, op->Gd + gi * pp,
                             op->Gf + gi * pp, nullptr, nullptr, ctl, true, false, nullptr);
  prof_end(ctx, PROF_TUBE_FWD);
  if (e != hipSuccess) return e;
  return slice_gemms(op, s, adjoint, ctl);
}

hipError_t pair_gemm(dctk_op op, hipStream_t s, int adjoint, const Ctl& ctl) {
  return slice_gemms(op, s, adjoint, ctl);
}

hipError_t pair_transforms(dctk_op op, hipStream_t s, int adjoint, const void* src, void* Y, bool xin,
                           const Ctl& ctl, int* nblocks_out) {
  dctk_ctx ctx = op->ctx;
  const int64_t pp = op->p * op->p;
  const int64_t rout = adjoint ? op->n2 : op->n1;
  // this product's inverse (L^{-1}, or L^T for the adjoint); its transpose is the
  // next product's forward transform (L^{-T} for the adjoint after a forward
  // product, L after an adjoint)
  const int g1 = adjoint ? 3 : 1;
  prof_begin(ctx, PROF_TUBE_PAIR);
  hipError_t e = launch_tube_pair(ctx, s, op->gemm_dtype, op->p, rout * op->s, (const float*)op->ch,
                                  (const float*)src, (float*)Y, op->xh, op->Gf + g1 * pp, xin, ctl, nblocks_out);
  prof_end(ctx, PROF_TUBE_PAIR);
  return e;
}

hipError_t apply_op(dctk_op op, hipStream_t s, int adjoint, const void* X, void* Y, const void* src,
                    void* xnorm, const Ctl& ctl, int* nblocks_out) {
  dctk_ctx ctx = op->ctx;
  if (fused_eligible(op) && use_fused(op, adjoint)) return launch_fused(op, s, adjoint, X, Y, src, xnorm, ctl, nblocks_out);
  const int64_t p = op->p, n1 = op->n1, n2 = op->n2, sc = op->s;
  const int gdt = op->gemm_dtype, vdt = op->vec_dtype;
  const double* Gd = op->Gd;
  const float* Gf = op->Gf;
  const int64_t pp = p * p;
  hipError_t e;
  // rows of the input / output vectors
  const int64_t rin = adjoint ? n1 : n2;
  const int64_t rout = adjoint ? n2 : n1;
  // step 1: transform the input tubes (L, or L^{-T} for the adjoint) into the GEMM type;
  // this kernel evaluates the control block (input scale, recorded scalars)
  const int gi = adjoint ? 2 : 0;
  prof_begin(ctx, PROF_TUBE_FWD);
  if (op->fast)  // tubes longer than kMaxTube: the O(p log p) transform
    e = launch_tube_fast_ctl(ctx, s, op->tube, adjoint ? DCTK_MAT_LINVT : DCTK_MAT_L, vdt, gdt, p, rin * sc, X,
                             op->xh, nullptr, xnorm, ctl, true, false, nullptr);
  else
    e = launch_tube(ctx, s, vdt, gdt, p, rin * sc, X, op->xh, Gd + gi * pp, Gf + gi * pp, nullptr, xnorm, ctl, true,
                    false, nullptr);
  prof_end(ctx, PROF_TUBE_FWD);
  if (e != hipSuccess) return e;
  // later kernels read the recorded scalars from the state
  Ctl later = ctl;
  later.from_state = 1;
  // step 2: slice products
  e = slice_gemms(op, s, adjoint, ctl);
  if (e != hipSuccess) return e;
  // step 3: inverse transform (L^{-1}, or L^T for the adjoint) with the epilogue
  const int go = adjoint ? 3 : 1;
  prof_begin(ctx, PROF_TUBE_INV);
  if (op->fast)
    e = launch_tube_fast_ctl(ctx, s, op->tube, adjoint ? DCTK_MAT_LT : DCTK_MAT_LINV, vdt, vdt, p, rout * sc, op->ch,
                             Y, src, nullptr, later, false, true, nblocks_out);
  else
    e = launch_tube(ctx, s, vdt, vdt, p, rout * sc, op->ch, Y, Gd + go * pp, Gf + go * pp, src, nullptr, later, false,
                    true, nblocks_out);
  prof_end(ctx, PROF_TUBE_INV);
  return e;
}

void set_num_cus(int n) { if (n > 0) g_num_cus = n; }
int num_cus() { return g_num_cus; }
size_t elem_size(int dt) { return dtype_size(dt); }

}  // namespace dctk
