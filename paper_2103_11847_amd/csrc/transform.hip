// Tube transforms along mode 3 (Algorithm 1 steps 1 and 3; Remark 2.1).
//
// A tube transform is out = in x_3 G with G a small p x p matrix: for every
// position e of a frontal slice, out[k][e] = sum_t G[k][t] in[t][e].  With the
// slice-major layout the p inputs of a tube are p slices apart, so a thread
// streams VEC consecutive positions of every slice (coalesced 16-byte loads
// along the slice) and keeps its tubes in registers; G sits in LDS.  Tubes
// longer than 8 run on the matrix cores.  The work is HBM-bound for the p of
// colour images and video (2p flops per 2 elements moved).
#include <cmath>
#include <type_traits>
#include <vector>

#include "mfma.h"

namespace dctk {

// ---- host: the transform matrices, FP64 closed forms -----------------------
// C_n of eq. (dft1), 0-based: C[i][j] = sqrt((2 - [i == 0]) / n) cos(i (2j + 1) pi / (2n)).
static void dct_matrix(int64_t n, std::vector<double>& C) {
  C.assign((size_t)(n * n), 0.0);
  const double pi = 3.14159265358979323846264338327950288;
  for (int64_t i = 0; i < n; ++i) {
    double sc = std::sqrt((i == 0 ? 1.0 : 2.0) / (double)n);
    for (int64_t j = 0; j < n; ++j)
      C[(size_t)(i * n + j)] = sc * std::cos((double)i * (double)(2 * j + 1) * pi / (2.0 * (double)n));
  }
}

int build_tube_matrix(int tube, int which, int64_t p, double* out) {
  if (p <= 0) return DCTK_ESHAPE;
  if (out == nullptr) return DCTK_EINVAL;
  if (which < DCTK_MAT_L || which > DCTK_MAT_LT) return DCTK_EINVAL;
  std::vector<double> C, L((size_t)(p * p)), Li((size_t)(p * p));
  dct_matrix(p, C);
  if (tube == DCTK_TUBE_DCT2) {
    for (int64_t i = 0; i < p; ++i)
      for (int64_t j = 0; j < p; ++j) {
        L[(size_t)(i * p + j)] = C[(size_t)(i * p + j)];
        Li[(size_t)(i * p + j)] = C[(size_t)(j * p + i)];  // C^{-1} = C^T
      }
  } else if (tube == DCTK_TUBE_TH) {
    // M = W^{-1} C (I + Z): row i of C (I + Z) is C[i][j] + C[i][j-1], scaled by 1 / C[i][0].
    for (int64_t i = 0; i < p; ++i)
      for (int64_t j = 0; j < p; ++j) {
        double v = C[(size_t)(i * p + j)] + (j > 0 ? C[(size_t)(i * p + j - 1)] : 0.0);
        L[(size_t)(i * p + j)] = v / C[(size_t)(i * p)];
      }
    // M^{-1} = (I + Z)^{-1} C^T W with (I + Z)^{-1}[i][l] = (-1)^{l - i} for l >= i:
    // M^{-1}[i][j] = C[j][0] * sum_{l >= i} (-1)^{l - i} C[j][l].
    for (int64_t i = 0; i < p; ++i)
      for (int64_t j = 0; j < p; ++j) {
        double acc = 0.0, sg = 1.0;
        for (int64_t l = i; l < p; ++l, sg = -sg) acc += sg * C[(size_t)(j * p + l)];
        Li[(size_t)(i * p + j)] = acc * C[(size_t)(j * p)];
      }
  } else {
    return DCTK_EINVAL;
  }
  for (int64_t i = 0; i < p; ++i)
    for (int64_t j = 0; j < p; ++j) {
      double v;
      switch (which) {
        case DCTK_MAT_L: v = L[(size_t)(i * p + j)]; break;
        case DCTK_MAT_LINV: v = Li[(size_t)(i * p + j)]; break;
        case DCTK_MAT_LINVT: v = Li[(size_t)(j * p + i)]; break;
        default: v = L[(size_t)(j * p + i)]; break;
      }
      out[i * p + j] = v;
    }
  return DCTK_OK;
}

// ---- device: the streaming transform ----------------------------------------
// Four neighbouring positions of a slice in memory: one 16-byte (32, 8) access
// that needs no more than the element's own alignment, so slices of any size
// and buffers at any address move in vectors.
typedef float f32x4_un __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2_un __attribute__((ext_vector_type(2), aligned(8)));
typedef unsigned int u32x2_un __attribute__((ext_vector_type(2), aligned(2)));
typedef _Float16 f16x4_un __attribute__((ext_vector_type(4), aligned(2)));
__device__ inline void load4(const float* p, float (&v)[4]) {
  const f32x4_un q = *reinterpret_cast<const f32x4_un*>(p);
  v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
__device__ inline void load4(const double* p, double (&v)[4]) {
  const f64x2_un a = *reinterpret_cast<const f64x2_un*>(p), b = *reinterpret_cast<const f64x2_un*>(p + 2);
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ inline void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<f32x4_un*>(p) = f32x4_un{v[0], v[1], v[2], v[3]};
}
__device__ inline void store4(double* p, const double (&v)[4]) {
  *reinterpret_cast<f64x2_un*>(p) = f64x2_un{v[0], v[1]};
  *reinterpret_cast<f64x2_un*>(p + 2) = f64x2_un{v[2], v[3]};
}
__device__ inline void store4(bf16_t* p, const float (&v)[4]) {
  const unsigned lo = (unsigned)float_to_bf16(v[0]) | ((unsigned)float_to_bf16(v[1]) << 16);
  const unsigned hi = (unsigned)float_to_bf16(v[2]) | ((unsigned)float_to_bf16(v[3]) << 16);
  *reinterpret_cast<u32x2_un*>(p) = u32x2_un{lo, hi};
}
__device__ inline void store4(f16_t* p, const float (&v)[4]) {
  *reinterpret_cast<f16x4_un*>(p) = f16x4_un{(f16_t)v[0], (f16_t)v[1], (f16_t)v[2], (f16_t)v[3]};
}
// positions e .. e + 3 of a slice of `count`, or (inside) four that all lie in it
template <typename T, typename V>
__device__ inline void store_row(T* p, int64_t e, int64_t count, const V (&v)[4], bool inside = false) {
  if (inside || e + 4 <= count) {
    store4(p + e, v);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (e + i < count) p[e + i] = cvt<T, V>(v[i]);
  }
}
// Four values loaded n positions early, to end with their slice: entries n .. 3
// to the front, 0 behind them (n <= 0: as loaded).
template <typename T>
__device__ inline void drop4(T (&v)[4], int64_t n) {
  if (n <= 0) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T r = (T)0;
#pragma unroll
    for (int j = i + 1; j < 4; ++j) r = n == j - i ? v[j] : r;
    v[i] = r;
  }
}
// four values in LDS, 16-byte aligned
__device__ inline void lds_load4(const float* p, float (&v)[4]) {
  const float4 q = *reinterpret_cast<const float4*>(p);
  v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
__device__ inline void lds_load4(const double* p, double (&v)[4]) {
  const double2 a = *reinterpret_cast<const double2*>(p), b = *reinterpret_cast<const double2*>(p + 2);
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ inline void lds_store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void lds_store4(double* p, const double (&v)[4]) {
  *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
  *reinterpret_cast<double2*>(p + 2) = make_double2(v[2], v[3]);
}

// TIN: float or double; TOUT: float, double, bf16_t or f16_t; TC: compute type.
// SCALE: apply the control block's input scale (and write xnorm); EPI: apply
// its a/b/src epilogue and write per-block partials of out^2.
struct TubeArgs {
  int gx, gy, gz;
  int p;
  int64_t count;       // tube positions (elements per slice)
  const void* in;      // p x count, TIN
  void* out;           // p x count, TOUT
  const void* G;       // p x p, TC
  const void* src;     // p x count, TOUT, or null
  void* xnorm;         // p x count, TIN, or null
  Ctl ctl;
};

template <typename TIN, typename TOUT, typename TC, int KB, bool SCALE, bool EPI>
__device__ __forceinline__ void tube_kernel_body(const TubeArgs& ta, const VBlock vb) {
  __shared__ double sh[kShCtl];
  const int p = ta.p;
  const int64_t count = ta.count;
  const TIN* __restrict__ in = (const TIN*)ta.in;
  TOUT* out = (TOUT*)ta.out;
  const TC* __restrict__ G = (const TC*)ta.G;
  const TOUT* src = (const TOUT*)ta.src;
  TIN* xnorm = (TIN*)ta.xnorm;
  const Ctl& ctl = ta.ctl;
  double a_d, b_d, s_d;
  if (!ctl_begin(ctl, a_d, b_d, s_d, sh, vb)) return;
  if (!SCALE) s_d = 1.0;
  if (!EPI) { a_d = 1.0; b_d = 0.0; }
  const TC a = (TC)a_d, b = (TC)b_d, sc = (TC)s_d;
  extern __shared__ char smem_raw[];
  TC* sG = reinterpret_cast<TC*>(smem_raw);
  for (int i = threadIdx.x; i < p * p; i += blockDim.x) sG[i] = G[i];
  __syncthreads();
  double sq = 0.0;
  const int64_t stride = (int64_t)ta.gx * blockDim.x * 4;
  // all p tubes of a 4-position group at once: every input (and src) load
  // of the group is issued before the first use, from clamped addresses
  const bool use_src = EPI && src != nullptr && b != (TC)0;
  // positions e0 .. e0 + 3; tail_c: fewer of them lie in the slice
  auto do_group = [&](int64_t e0, auto tail_c) {
    constexpr bool tail = decltype(tail_c)::value;
    const int nv = tail ? (int)(count - e0) : 4;
    // rows of `q` (p x count) into v, zeros outside
    auto rows = [&](const auto* q, auto (&v)[KB][4]) {
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        const auto* r = q + (int64_t)(t < p ? t : 0) * count + e0;
        if constexpr (!tail) {
          load4(r, v[t]);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[t][i] = r[i < nv ? i : 0];
        }
      }
    };
    TIN xv[KB][4];
    rows(in, xv);
    TC sv[KB][4];
    if constexpr (EPI) {
      if (use_src) rows(src, sv);
    }
#pragma unroll
    for (int t = 0; t < KB; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (t >= p || (tail && v >= nv)) xv[t][v] = (TIN)0;
        if (!EPI || !use_src || t >= p || (tail && v >= nv)) sv[t][v] = (TC)0;
      }
    if (SCALE) {
#pragma unroll
      for (int t = 0; t < KB; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) xv[t][v] = (TIN)(sc * (TC)xv[t][v]);
      if (xnorm != nullptr) {
#pragma unroll
        for (int t = 0; t < KB; ++t)
          if (t < p) store_row(xnorm + (int64_t)t * count, e0, count, xv[t], !tail);
      }
    }
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k >= p) break;
      TC acc[4] = {(TC)0, (TC)0, (TC)0, (TC)0};
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        const TC gk = t < p ? sG[k * p + t] : (TC)0;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] += gk * (TC)xv[t][v];
      }
      TC ov[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        TC r = a * acc[v];
        if (EPI) r += b * sv[k][v];
        ov[v] = r;
        if (EPI && v < nv) sq += (double)r * (double)r;
      }
      store_row(out + (int64_t)k * count, e0, count, ov, !tail);
    }
  };
  for (int64_t e0 = ((int64_t)vb.x * blockDim.x + threadIdx.x) * 4; e0 < count; e0 += stride) {
    if (e0 + 4 <= count) do_group(e0, std::false_type{});
    else do_group(e0, std::true_type{});
  }
  if (EPI && ctl.part_out != nullptr) {
    const double tot = block_sum_all(sq, sh);
    if (threadIdx.x == 0) ctl.part_out[vb.x] = tot;
  }
}

template <typename TIN, typename TOUT, typename TC, int KB, bool SCALE, bool EPI, bool GROUPED>
__global__ __launch_bounds__(kThreads) void tube_kernel(TubeArgs ta_, const TubeArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    tube_kernel_body<TIN, TOUT, TC, KB, SCALE, EPI>(ta_, hw_block());
  } else {
    VBlock vb;
    const TubeArgs g = group_args(grp, bmap, vb);
    tube_kernel_body<TIN, TOUT, TC, KB, SCALE, EPI>(g, vb);
  }
}

// Tubes longer than 8: the transform out = G x in is a (p x p)(p x count)
// contraction, so it runs on the matrix cores (FP32 and FP64, each with its
// own 16x16x4 instruction).  A workgroup stages G (p x p,
// padded to a multiple of 16) in LDS once and then walks its 64-position tiles
// (grid stride).  Every global access of a tile is a row of 64 consecutive
// positions of one slice, moved as 16-byte vectors: the input (from clamped
// addresses, all issued together, scaled by the control block's s and
// written to xnorm on the way) and the epilogue's src are loaded before the
// tile is multiplied; wave w computes the 16 positions of column block w for
// every 16-row band of outputs with 16x16x4 MFMAs; the products return
// to LDS, and the epilogue reads them back as rows, applies a, b and src,
// stores the rows and accumulates the workgroup's partial sum of out^2.
// Without an epilogue (fewer registers live) the control block's loads, G
// and the first tile are in flight together, and the next tile's rows load
// while the current one is multiplied.
// VEC: count >= 4, at any alignment (a unit that would cross the end of its
// slice is read from the slice's last 4 positions and put right when staged).
// FP64 at 256 x 256 x 64 (67 MB moved): forward 296 us, inverse 202 before
// (vector units, the input read again for every 8 outputs), now 25 and 26
// (FP64 at 200 x 200 x 31: 67 / 52 -> 11.6 / 10.9; FP32 at 200 x 200 x 12: 18 / 15 -> 7.1 / 6.3).
// Slices of a size that is no multiple of 4 moved in single elements: FP32 at 333 x 333 x 64
// 26.0 / 26.0 us, now 20.5 / 20.5.  Whole tiles test no position and mask no load (the loads were
// waited for where they were masked, before the passes): 512 x 512 x 64 forward to FP32 36 -> 32.5 us,
// to BF16 39.5 -> 33..
template <typename T, typename TOUT, int PM, bool SCALE, bool EPI, bool VEC>
__device__ __forceinline__ void tube_mfma_kernel_body(const TubeArgs& ta, const VBlock vb) {
  typedef Mfma<T> MF;
  constexpr int NB = 64;            // positions per tile
  // G as [k][t], t contiguous (+16 bytes; FP64 +32, two rows' operands per 64 bytes),
  // input / products as [row][e], e contiguous (+16 bytes; FP64 +128, so that the
  // operand's rows alternate between the halves of the banks)
  constexpr int LDG = PM + 4;
  constexpr int LDX = sizeof(T) == 8 ? NB + 16 : NB + 4;
  constexpr int FR = PM / 16;       // row bands
  constexpr int XU = PM * (NB / 4) / 256;  // 4-position units of a tile per thread
  constexpr int GU = PM * PM / 256;        // G entries per thread
  static_assert(XU * 256 == PM * (NB / 4) && GU * 256 == PM * PM, "tile");
  __shared__ __attribute__((aligned(16))) T sG[PM * LDG];
  __shared__ __attribute__((aligned(16))) T sX[PM * LDX];
  __shared__ double sh[kShCtl];
  const int p = ta.p;
  const int64_t count = ta.count;
  const T* in = (const T*)ta.in;
  TOUT* out = (TOUT*)ta.out;
  const T* G = (const T*)ta.G;
  const T* src = (const T*)ta.src;   // outputs of type T only (launch_tube refuses src otherwise)
  T* xnorm = (T*)ta.xnorm;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t ntiles = (count + NB - 1) / NB;

  // a tile's input rows (rv), then its src rows (sv), which are waited for
  // later, into registers from clamped addresses; what lies outside is taken
  // out where they are used
  T rv[XU][4], sv[XU][4];
  auto load_rows = [&](const T* q, int64_t tile, T (&v)[XU][4]) {
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int t = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t row = (int64_t)(t < p ? t : 0) * count, e = tile * NB + c;
      if constexpr (VEC) {
        load4(q + row + (e + 4 <= count ? e : count - 4), v[u]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = q[row + (e + j < count ? e + j : count - 1)];
      }
    }
  };
  auto load_tile = [&](int64_t tile) {
    load_rows(in, tile, rv);
    if constexpr (EPI) {
      __builtin_amdgcn_sched_barrier(0);
      if (src != nullptr) load_rows(src, tile, sv);
    }
  };
  // entries of a unit at position e beyond the slice (the last tile's)
  auto tail = [&](int64_t e, T (&v)[4]) {
    if constexpr (VEC) drop4(v, e - (count - 4));
    else
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = e + i < count ? v[i] : (T)0;
  };

  // prologue: the control block's loads, G and the first tile's rows are all in
  // flight before the first of them is used
  const CtlLoad cl = ctl_load(ta.ctl);
  T gv[GU];
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int i = tid + u * 256, k = i / PM, t = i % PM;
    const bool ok = k < p && t < p;
    const T v = G[ok ? k * p + t : 0];
    gv[u] = ok ? v : (T)0;
  }
  int64_t tile = vb.x;
  if (!EPI && tile < ntiles) load_tile(tile);
  double a_d, b_d, s_d;
  if (!ctl_eval(ta.ctl, cl, a_d, b_d, s_d, sh, vb)) return;
  if (!SCALE) s_d = 1.0;
  if (!EPI) { a_d = 1.0; b_d = 0.0; }
  const T a = (T)a_d, b = (T)b_d, sc = (T)s_d;
  const bool use_src = EPI && src != nullptr && b != (T)0;   // b = 0: src never enters
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int i = tid + u * 256, k = i / PM, t = i % PM;
    sG[k * LDG + t] = gv[u];
  }
  const int lr = lane & 15, lk = lane >> 4;
  double sq = 0.0;
  // one tile; tail_c: it reaches beyond the slice (whole tiles test no position)
  auto do_tile = [&](auto tail_c) {
    constexpr bool last = decltype(tail_c)::value;
    const int64_t e0 = tile * NB;
    if (EPI) load_tile(tile);
    __syncthreads();  // the previous tile's products have been read from LDS (and G is staged)
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int t = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t e = e0 + c;
      if (last) {
        tail(e, rv[u]);
        if (EPI && use_src) tail(e, sv[u]);
      }
      if (SCALE) {
#pragma unroll
        for (int v = 0; v < 4; ++v) rv[u][v] *= sc;
        if (xnorm != nullptr && t < p) store_row(xnorm + (int64_t)t * count, e, count, rv[u], !last);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) rv[u][v] = t < p ? rv[u][v] : (T)0;
      lds_store4(&sX[t * LDX + c], rv[u]);
    }
    __syncthreads();
    // without an epilogue (fewer registers live) the next tile's rows load while
    // this one is multiplied; with it they load at the top of the next tile
    if (!EPI && tile + ta.gx < ntiles) load_tile(tile + ta.gx);
    typename MF::frag_t acc[FR];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[f][r] = (T)0;
#pragma unroll 4
    for (int t0 = 0; t0 < PM; t0 += 4) {
      const T* bp = &sX[(t0 + lk) * LDX + wave * 16 + lr];
#pragma unroll
      for (int f = 0; f < FR; ++f) acc[f] = MF::mac(&sG[(f * 16 + lr) * LDG + t0 + lk], bp, acc[f]);
    }
    // a wave reads and writes only its own 16 columns of sX, and a wave's LDS
    // accesses complete in order: no block barrier before its products go back
    __builtin_amdgcn_wave_barrier();
    // products back to LDS as [k][e]: lane holds rows 4 (lane / 16) + r (FP64: lane / 16
    // + 4 r) of column lane % 16
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) sX[(f * 16 + (MF::ROWS_STRIDED ? lk + 4 * r : lk * 4 + r)) * LDX + wave * 16 + lr] = acc[f][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int k = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t e = e0 + c;
      if (k >= p) continue;
      T y[4];
      lds_load4(&sX[k * LDX + c], y);
#pragma unroll
      for (int v = 0; v < 4; ++v) y[v] *= a;
      if (EPI) {
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] += use_src ? b * sv[u][v] : (T)0;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (!last || e + v < count) sq += (double)y[v] * (double)y[v];
      }
      store_row(out + (int64_t)k * count, e, count, y, !last);
    }
  };
  for (; tile < ntiles; tile += ta.gx) {
    if ((tile + 1) * NB <= count) do_tile(std::false_type{});
    else do_tile(std::true_type{});
  }
  if (EPI && ta.ctl.part_out != nullptr) {
    const double tot = block_sum_all(sq, sh);
    if (tid == 0) ta.ctl.part_out[vb.x] = tot;
  }
}

template <typename T, typename TOUT, int PM, bool SCALE, bool EPI, bool VEC, bool GROUPED>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? 2 : 4) void tube_mfma_kernel(TubeArgs ta_, const TubeArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    tube_mfma_kernel_body<T, TOUT, PM, SCALE, EPI, VEC>(ta_, hw_block());
  } else {
    VBlock vb;
    const TubeArgs g = group_args(grp, bmap, vb);
    tube_mfma_kernel_body<T, TOUT, PM, SCALE, EPI, VEC>(g, vb);
  }
}

template <typename T, typename TOUT>
static hipError_t launch_tube_mfma(dctk_ctx ctx, hipStream_t s, int64_t p, int64_t count, const void* in, void* out,
                                   const T* G, const void* src, void* xnorm, const Ctl& ctl, bool scale,
                                   bool epi, int* nblocks_out) {
  // a few workgroups per CU, each walking several 64-position tiles, so G
  // is staged once per workgroup rather than once per tile
  int64_t blocks = (count + 63) / 64;
  const int64_t cap = (sizeof(T) == 8 ? 2 : 4) * (int64_t)num_cus();   // what fits a CU's LDS
  if (blocks > cap) blocks = cap;
  if (nblocks_out) *nblocks_out = (int)blocks;
  if (epi && ctl.part_out != nullptr && blocks > kRedBlocks) return hipErrorInvalidConfiguration;
  const bool vec = count >= 4;
  TubeArgs ta{};
  ta.p = (int)p;
  ta.count = count;
  ta.in = in;
  ta.out = out;
  ta.G = G;
  ta.src = src;
  ta.xnorm = xnorm;
  ta.ctl = ctl;
  const dim3 grid((unsigned)blocks);
#define DCTK_TMV(PM_, SC_, EP_) \
  do { \
    if (vec) return launch_kernel(ctx, s, tube_mfma_kernel<T, TOUT, PM_, SC_, EP_, true, false>, tube_mfma_kernel<T, TOUT, PM_, SC_, EP_, true, true>, grid, 256, 0, ta); \
    return launch_kernel(ctx, s, tube_mfma_kernel<T, TOUT, PM_, SC_, EP_, false, false>, tube_mfma_kernel<T, TOUT, PM_, SC_, EP_, false, true>, grid, 256, 0, ta); \
  } while (0)
#define DCTK_TM(PM_) \
  do { \
    if (scale) DCTK_TMV(PM_, true, false); \
    if constexpr (sizeof(T) == sizeof(TOUT)) DCTK_TMV(PM_, false, true); \
  } while (0)
  if (p <= 16) DCTK_TM(16);
  if (p <= 32) DCTK_TM(32);
  if (p <= 48) DCTK_TM(48);
  DCTK_TM(64);
  return hipErrorInvalidValue;   // a 16-bit output is a slice product's operand: the input side
#undef DCTK_TM
#undef DCTK_TMV
}

// ---- the two transforms between consecutive slice products ---------------------
// Inside a Golub-Kahan step the inverse transform of one product and the
// forward transform of the next act on the same tubes: y = a (G1 c) + b src is
// the new basis vector (Algorithm 4's U~ or V~, kept unnormalised in its slot)
// and x = G1^T y is the next product's transformed input (its normalisation is
// applied by the next product's epilogue, as `a`).  The second matrix is always
// the transpose of the first: after a forward product G1 = L^{-1} and the
// adjoint's forward transform is L^{-T}; after an adjoint product G1 = L^T and
// the forward product's transform is L.  One pass over a 64-position tile does
// both: the slice products' rows and the src rows come in, y goes out (with
// the workgroup's partial sum of y^2), y returns to LDS, the second MFMA pass
// forms x reading the one staged copy of G1 transposed, and x goes out in the
// GEMM type -- y is never read back from memory.  The control block is the one
// of the first transform's product; the scale it returns for that product's
// input (1/alpha or 1/beta, as the input x of that product was stored
// unnormalised) joins `a`.
// x is stored as 2^-e G1^T y, 2^e the power of two below alpha_1, and the
// product's own pair (xin) multiplies `a` by 2^e: y has the operator's scale, so
// the slice product of G1^T y would hold the square of it, which FP32 does not
// from 1e-19 down and 1e19 up.  alpha_1 stands for y's norm, which is known only
// after the launch; a power of two leaves every bit in between as it was.  FP16
// operands, whose narrow range would turn a small alpha_1 into infinities, keep
// y's own scale (e = 0).
struct PairArgs {
  int gx, gy, gz;
  int p;
  int xin;           // 1: the slice products' operand carries 2^-e
  int64_t count;
  const float* c;    // p x count slice products (FP32)
  const float* src;  // p x count, or null
  float* y;          // p x count, the new basis vector
  void* x;           // p x count, TX: the next product's transformed input
  const float* G1;   // p x p
  Ctl ctl;
};

// e of PairArgs from alpha_1, within what FP32 powers of two reach
__device__ inline int pair_exp(double alpha1) {
  const int e = (int)((__builtin_bit_cast(unsigned long long, alpha1) >> 52) & 0x7ff) - 1023;
  return __builtin_amdgcn_readfirstlane(e < -120 ? -120 : (e > 120 ? 120 : e));
}
__device__ inline float pow2f(int e) { return __builtin_bit_cast(float, (127 + e) << 23); }

template <typename TX, int PM, bool VEC>
__device__ __forceinline__ void tube_pair_kernel_body(const PairArgs& pa, const VBlock vb) {
  typedef Mfma<float> MF;
  constexpr int NB = 64;
  // rows of G1 padded by 8: both the row reads of the first pass and the
  // column reads of the second spread over the banks
  constexpr int LDG = PM + 8;
  constexpr int LDX = NB + 4;
  constexpr int FR = PM / 16;
  constexpr int XU = PM * (NB / 4) / 256;
  constexpr int GU = PM * PM / 256;
  static_assert(XU * 256 == PM * (NB / 4) && GU * 256 == PM * PM, "tile");
  __shared__ __attribute__((aligned(16))) float sG1[PM * LDG];
  __shared__ __attribute__((aligned(16))) float sX[PM * LDX];
  __shared__ double sh[kShCtl];
  const int p = pa.p;
  const int64_t count = pa.count;
  const float* in = pa.c;
  const float* src = pa.src;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t ntiles = (count + NB - 1) / NB;

  // a tile's product rows (rv), then its src rows (sv), which are waited for
  // later, into registers from clamped addresses (what lies outside is taken
  // out where they are used); loading the next tile's rows during the passes
  // measured slower
  float rv[XU][4], sv[XU][4];
  auto load_rows = [&](const float* q, int64_t tile, float (&v)[XU][4]) {
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int t = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t row = (int64_t)(t < p ? t : 0) * count, e = tile * NB + c;
      if constexpr (VEC) {
        load4(q + row + (e + 4 <= count ? e : count - 4), v[u]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = q[row + (e + j < count ? e + j : count - 1)];
      }
    }
  };
  auto tail = [&](int64_t e, float (&v)[4]) {
    if constexpr (VEC) drop4(v, e - (count - 4));
    else
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = e + i < count ? v[i] : 0.0f;
  };
  // one MFMA pass: the products G x (tile in sX) back into sX as [k][e], with
  // G = G1, or (TR) its transpose read from the same LDS copy
  auto mfma_pass = [&](const float* sG, auto tr) {
    constexpr bool TR = decltype(tr)::value;
    typename MF::frag_t acc[FR];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[f][r] = 0.0f;
    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll 4
    for (int t0 = 0; t0 < PM; t0 += 4) {
      const float* bp = &sX[(t0 + lk) * LDX + wave * 16 + lr];
#pragma unroll
      for (int f = 0; f < FR; ++f)
        acc[f] = MF::mac(TR ? &sG[(t0 + lk) * LDG + f * 16 + lr] : &sG[(f * 16 + lr) * LDG + t0 + lk], bp, acc[f]);
    }
    // a wave reads and writes only its own 16 columns of sX, and a wave's LDS
    // accesses complete in order: no block barrier between its operand reads
    // and its product writes
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) sX[(f * 16 + lk * 4 + r) * LDX + wave * 16 + lr] = acc[f][r];
    __syncthreads();
  };

  // prologue: the control block's loads and the matrix in flight together
  const double alpha1 = pa.ctl.st->alpha[0];
  const CtlLoad cl = ctl_load(pa.ctl);
  float g1[GU];
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int i = tid + u * 256, k = i / PM, t = i % PM;
    const bool ok = k < p && t < p;
    const float v1 = pa.G1[ok ? k * p + t : 0];
    g1[u] = ok ? v1 : 0.0f;
  }
  double a_d, b_d, s_d;
  asm volatile("" ::"v"(alpha1));   // waited for with the control block's values, not on its own
  if (!ctl_eval(pa.ctl, cl, a_d, b_d, s_d, sh, vb)) return;
  const int ex = std::is_same<TX, f16_t>::value ? 0 : pair_exp(alpha1);
  const float xs = pow2f(-ex), b = (float)b_d;
  const float a = (float)(a_d * s_d * (double)(pa.xin ? pow2f(ex) : 1.0f));
  const bool use_src = src != nullptr && b != 0.0f;   // b = 0: src never enters
#pragma unroll
  for (int u = 0; u < GU; ++u) {
    const int i = tid + u * 256, k = i / PM, t = i % PM;
    sG1[k * LDG + t] = g1[u];
  }
  double sq = 0.0;
  // one tile; tail_c: it reaches beyond the slice (whole tiles test no position)
  auto do_tile = [&](int64_t tile, auto tail_c) {
    constexpr bool last = decltype(tail_c)::value;
    const int64_t e0 = tile * NB;
    load_rows(in, tile, rv);
    __builtin_amdgcn_sched_barrier(0);
    load_rows(src != nullptr ? src : in, tile, sv);
    __syncthreads();  // the previous tile's x rows have been read from sX (and G1 is staged)
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int t = i / (NB / 4), c = (i % (NB / 4)) * 4;
      if (last) {
        tail(e0 + c, rv[u]);
        tail(e0 + c, sv[u]);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        rv[u][v] = t < p ? rv[u][v] : 0.0f;
        sv[u][v] = t < p ? sv[u][v] : 0.0f;
      }
      lds_store4(&sX[t * LDX + c], rv[u]);
    }
    __syncthreads();
    mfma_pass(sG1, std::false_type{});
    // y = a (G1 c) + b src: written out, summed, and staged for the second pass
    // (rows k >= p are zero in both passes)
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int k = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t e = e0 + c;
      float4* rowp = reinterpret_cast<float4*>(&sX[k * LDX + c]);
      const float4 q = *rowp;
      float y[4] = {a * q.x, a * q.y, a * q.z, a * q.w};
#pragma unroll
      for (int v = 0; v < 4; ++v) y[v] += use_src ? b * sv[u][v] : 0.0f;
      if (k < p) {
        store_row(pa.y + (int64_t)k * count, e, count, y, !last);
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (!last || e + v < count) sq += (double)y[v] * (double)y[v];
      }
      // positions beyond the slice enter the second pass as zeros
#pragma unroll
      for (int v = 0; v < 4; ++v)
        y[v] = last && e + v >= count ? 0.0f : xs * y[v];
      *rowp = make_float4(y[0], y[1], y[2], y[3]);
    }
    __syncthreads();
    mfma_pass(sG1, std::true_type{});
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int i = tid + u * 256;
      const int k = i / (NB / 4), c = (i % (NB / 4)) * 4;
      const int64_t e = e0 + c;
      if (k >= p) continue;
      const float4 q = *reinterpret_cast<const float4*>(&sX[k * LDX + c]);
      const float xv[4] = {q.x, q.y, q.z, q.w};
      store_row((TX*)pa.x + (int64_t)k * count, e, count, xv, !last);
    }
  };
  for (int64_t tile = vb.x; tile < ntiles; tile += pa.gx) {
    if ((tile + 1) * NB <= count) do_tile(tile, std::false_type{});
    else do_tile(tile, std::true_type{});
  }
  if (pa.ctl.part_out != nullptr) {
    const double tot = block_sum_all(sq, sh);
    if (tid == 0) pa.ctl.part_out[vb.x] = tot;
  }
}

// The same pair of transforms for short tubes (p <= 8): a thread holds the p
// entries of four neighbouring tubes in registers, so y = a (G1 c) + b src and
// x = G1^T y follow each other without LDS or barriers, with every load of c
// and src in flight together (16 rows of 16 bytes per thread at p = 8).  Bound
// by memory (16 B/element at 4 p flops); inside a Golub-Kahan step it replaces
// the inverse and the forward transform's own launches and the re-read of y.
template <int KB>
__device__ __forceinline__ void tube_pair_small_body(const PairArgs& pa, const VBlock vb) {
  __shared__ float sG[KB * KB];
  __shared__ double sh[kShCtl];
  const int p = pa.p;
  const int64_t count = pa.count;
  const bool has_src = pa.src != nullptr;
  const float* in = pa.c;
  const float* src = has_src ? pa.src : pa.c;   // without src its loads read c again and are not used
  const int64_t stride = (int64_t)pa.gx * kThreads * 4;
  float cv[KB][4], sv[KB][4];
  auto load = [&](int64_t e0) {
    if (e0 + 4 <= count) {
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        const int64_t o = (int64_t)(t < p ? t : 0) * count + e0;
        load4(in + o, cv[t]);
        load4(src + o, sv[t]);
      }
    } else {   // the slice's last thread, and those beyond it
#pragma unroll
      for (int t = 0; t < KB; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t o = (int64_t)(t < p ? t : 0) * count + (e0 + v < count ? e0 + v : 0);
          cv[t][v] = in[o];
          sv[t][v] = src[o];
        }
    }
  };
  int64_t e0 = ((int64_t)vb.x * kThreads + threadIdx.x) * 4;
  // the first tubes, the matrix and the control block's values in flight together
  const double alpha1 = pa.ctl.st->alpha[0];
  const CtlLoad cl = ctl_load(pa.ctl);
  const int gi = (int)threadIdx.x;
  const float g = pa.G1[gi < p * p ? gi : 0];
  load(e0);
  double a_d, b_d, s_d;
  asm volatile("" ::"v"(alpha1));   // waited for with the control block's values, not on its own
  if (!ctl_eval(pa.ctl, cl, a_d, b_d, s_d, sh, vb)) return;
  const int ex = pair_exp(alpha1);
  const float xs = pow2f(-ex), b = has_src ? (float)b_d : 0.0f;
  const float a = (float)(a_d * s_d * (double)(pa.xin ? pow2f(ex) : 1.0f));
  const bool use_src = b != 0.0f;   // b = 0: src never enters
  if (gi < p * p) sG[gi / p * KB + gi % p] = g;
  __syncthreads();
  double sq = 0.0;
  for (; e0 < count; e0 += stride) {
    float y[KB][4];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (k < p) {
#pragma unroll
        for (int t = 0; t < KB; ++t)
          if (t < p) {
            const float w = sG[k * KB + t];
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += w * cv[t][v];
          }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float r = a * acc[v];
        if (use_src) r += b * sv[k][v];
        y[k][v] = r;
      }
    }
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k >= p) break;
      store_row(pa.y + (int64_t)k * count, e0, count, y[k]);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (e0 + v < count) sq += (double)y[k][v] * (double)y[k][v];
    }
    if (e0 + stride < count) load(e0 + stride);
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      if (k >= p) break;
      float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int t = 0; t < KB; ++t)
        if (t < p) {
          const float w = sG[t * KB + k];
#pragma unroll
          for (int v = 0; v < 4; ++v) x[v] += w * y[t][v];
        }
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] *= xs;
      store_row((float*)pa.x + (int64_t)k * count, e0, count, x);
    }
  }
  if (pa.ctl.part_out != nullptr) {
    const double tot = block_sum_all(sq, sh);
    if (threadIdx.x == 0) pa.ctl.part_out[vb.x] = tot;
  }
}

template <int KB, bool GROUPED>
__global__ __launch_bounds__(kThreads) void tube_pair_small_kernel(PairArgs pa_, const PairArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    tube_pair_small_body<KB>(pa_, hw_block());
  } else {
    VBlock vb;
    const PairArgs g = group_args(grp, bmap, vb);
    tube_pair_small_body<KB>(g, vb);
  }
}

template <typename TX, int PM, bool VEC, bool GROUPED>
__global__ __launch_bounds__(256, 4) void tube_pair_kernel(PairArgs pa_, const PairArgs* grp, const int4* bmap) {
  if constexpr (!GROUPED) {
    tube_pair_kernel_body<TX, PM, VEC>(pa_, hw_block());
  } else {
    VBlock vb;
    const PairArgs g = group_args(grp, bmap, vb);
    tube_pair_kernel_body<TX, PM, VEC>(g, vb);
  }
}

bool tube_pair_ok(int64_t p, int vec_dtype) { return vec_dtype == DCTK_F32 && p <= kMaxTube; }

hipError_t launch_tube_pair(dctk_ctx ctx, hipStream_t s, int x_dtype, int64_t p, int64_t count, const float* c,
                            const float* src, float* y, void* x, const float* G1, bool xin, const Ctl& ctl,
                            int* nblocks_out) {
  if (!tube_pair_ok(p, DCTK_F32)) return hipErrorInvalidValue;
  // four workgroups per CU (36 KB of LDS each), each walking several tiles of
  // 64 positions; short tubes: 1024 positions per workgroup and turn
  const bool small = p <= 8;
  int64_t blocks = small ? (count + 4 * kThreads - 1) / (4 * kThreads) : (count + 63) / 64;
  const int64_t cap = 4 * (int64_t)num_cus();
  if (blocks > cap) blocks = cap;
  if (nblocks_out) *nblocks_out = (int)blocks;
  if (ctl.part_out != nullptr && blocks > kRedBlocks) return hipErrorInvalidConfiguration;
  const bool vec = count >= 4;
  PairArgs pa{};
  pa.p = (int)p;
  pa.xin = xin ? 1 : 0;
  pa.count = count;
  pa.c = c;
  pa.src = src;
  pa.y = y;
  pa.x = x;
  pa.G1 = G1;
  pa.ctl = ctl;
  const dim3 grid((unsigned)blocks);
#define DCTK_PAIR_V(TX, PM_)                                                                                     \
  do {                                                                                                         \
    if (vec) return launch_kernel(ctx, s, tube_pair_kernel<TX, PM_, true, false>, tube_pair_kernel<TX, PM_, true, true>, grid, 256, 0, pa); \
    return launch_kernel(ctx, s, tube_pair_kernel<TX, PM_, false, false>, tube_pair_kernel<TX, PM_, false, true>, grid, 256, 0, pa); \
  } while (0)
#define DCTK_PAIR_S(KB_) \
  return launch_kernel(ctx, s, tube_pair_small_kernel<KB_, false>, tube_pair_small_kernel<KB_, true>, grid, kThreads, 0, pa)
#define DCTK_PAIR_P(TX)            \
  do {                             \
    if (p <= 16) DCTK_PAIR_V(TX, 16); \
    if (p <= 32) DCTK_PAIR_V(TX, 32); \
    if (p <= 48) DCTK_PAIR_V(TX, 48); \
    DCTK_PAIR_V(TX, 64);           \
  } while (0)
  if (small) {   // 16-bit products do not pair short tubes
    if (x_dtype != DCTK_F32) return hipErrorInvalidValue;
    if (p <= 4) DCTK_PAIR_S(4);
    DCTK_PAIR_S(8);
  }
  switch (x_dtype) {
    case DCTK_F32: DCTK_PAIR_P(float);
    case DCTK_BF16: DCTK_PAIR_P(bf16_t);
    case DCTK_F16: DCTK_PAIR_P(f16_t);
    default: return hipErrorInvalidValue;
  }
#undef DCTK_PAIR_P
#undef DCTK_PAIR_S
#undef DCTK_PAIR_V
}

template <typename TIN, typename TOUT, typename TC>
static hipError_t launch_tube_t(dctk_ctx ctx, hipStream_t s, int64_t p, int64_t count, const void* in, void* out,
                                const TC* G, const void* src, void* xnorm, const Ctl& ctl, bool scale, bool epi,
                                int* nblocks_out) {
  int64_t nthreads = (count + 3) / 4;
  int64_t blocks = (nthreads + kThreads - 1) / kThreads;
  if (blocks > kRedBlocks) blocks = kRedBlocks;
  if (blocks < 1) blocks = 1;
  if (nblocks_out) *nblocks_out = (int)blocks;
  size_t shmem = (size_t)(p * p) * sizeof(TC);
  TubeArgs ta{};
  ta.p = (int)p;
  ta.count = count;
  ta.in = in;
  ta.out = out;
  ta.G = G;
  ta.src = src;
  ta.xnorm = xnorm;
  ta.ctl = ctl;
  const dim3 grid((unsigned)blocks);
#define DCTK_TUBE_LAUNCH(KB, S, E) \
  return launch_kernel(ctx, s, tube_kernel<TIN, TOUT, TC, KB, S, E, false>, tube_kernel<TIN, TOUT, TC, KB, S, E, true>, grid, kThreads, (unsigned)shmem, ta)
#define DCTK_TUBE_SE(KB)                                                    \
  do {                                                                      \
    if (scale) DCTK_TUBE_LAUNCH(KB, true, false);                            \
    if constexpr (sizeof(TIN) == sizeof(TOUT)) DCTK_TUBE_LAUNCH(KB, false, true); \
  } while (0)
  if (p <= 4) DCTK_TUBE_SE(4);
  DCTK_TUBE_SE(8);
  return hipErrorInvalidValue;   // a 16-bit output is a slice product's operand: the input side
#undef DCTK_TUBE_SE
#undef DCTK_TUBE_LAUNCH
}

// in_dtype: element type of `in` (F64/F32); out_dtype: of `out` (F64, F32, BF16, F16).
// A transform whose output is a GEMM operand applies the input side of the
// control block (scale); one whose input is a GEMM result applies the epilogue
// side (epi).
hipError_t launch_tube(dctk_ctx ctx, hipStream_t s, int in_dtype, int out_dtype, int64_t p, int64_t count,
                       const void* in, void* out, const double* Gd, const float* Gf,
                       const void* src, void* xnorm, const Ctl& ctl, bool scale, bool epi, int* nblocks_out) {
  // the input side (scale, xnorm) or the output side (a, b, src, partials)
  if (scale == epi || p > kMaxTube) return hipErrorInvalidValue;
  const bool mfma = p > 8;
#define DCTK_TUBE(T, TO, G)                                                                                             \
  (mfma ? launch_tube_mfma<T, TO>(ctx, s, p, count, in, out, G, src, xnorm, ctl, scale, epi, nblocks_out)                \
        : launch_tube_t<T, TO, T>(ctx, s, p, count, in, out, G, src, xnorm, ctl, scale, epi, nblocks_out))
  if (in_dtype == DCTK_F64) {
    if (out_dtype != DCTK_F64) return hipErrorInvalidValue;
    return DCTK_TUBE(double, double, Gd);
  }
  switch (out_dtype) {
    case DCTK_F32: return DCTK_TUBE(float, float, Gf);
    case DCTK_BF16: return src ? hipErrorInvalidValue : DCTK_TUBE(float, bf16_t, Gf);
    case DCTK_F16: return src ? hipErrorInvalidValue : DCTK_TUBE(float, f16_t, Gf);
    default: return hipErrorInvalidValue;
  }
#undef DCTK_TUBE
}

}  // namespace dctk
