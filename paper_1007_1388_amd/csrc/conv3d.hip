// conv3d.hip -- gfx950 BF16 MFMA kernels of the learned warm start.
//
// Implicit-GEMM 3-D convolutions on channels-last BF16 tensors with FP32
// accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16):
//   forward      C[voxel][co]      = sum_k  patch(x)[voxel][k] * w[co][k]
//   bwd-data     C[voxel_in][ci]   = sum_k  patch^T(dy)[voxel_in][k] * wt[ci][k]
//   bwd-weight   C[co][k]          = sum_v  dy[v][co] * patch(x)[v][k]      (split over voxels)
// with k = tap * Cin + ci.  By shape (the launch_ functions below):
//   3x3x3, stride 1        k_conv_rows, k_conv_plane: source halos in LDS by direct loads
//   3x3x3, 8 channels      k_conv_fwd_c8, k_conv_wgrad_c8
//   stride-2 bwd-data      k_conv_up (all parities of a tile in one workgroup)
//   1x1x1                  k_conv_point, k_conv_wgrad_point
//   3x3x3 bwd-weight       k_conv_wgrad_rows
//   parts of bwd-weight    k_wgrad_sum: added in a fixed order
//   forward of stride 2 and what those leave, channels a multiple of 32: k_conv_tap
//   the rest               k_conv_gemm, k_conv_wgrad: a 128 x BN tile per workgroup
//                          (4 waves of 32 rows), operands staged in LDS with K fastest
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../../include/lbm_surrogate.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128;     // rows per workgroup tile
constexpr int BK = 32;      // K per MFMA step
constexpr int LDK = BK + 8; // LDS row length (bf16), padded against bank conflicts

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// round to nearest even by gfx950's conversion instruction
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

struct Geo {
  int n, d, h, w, c, ldc;
};

__device__ __forceinline__ long long vox(const Geo& g, int n, int d, int h, int w) {
  return (((long long)n * g.d + d) * g.h + h) * g.w + w;
}

// Decompose a voxel index of geometry g.
__device__ __forceinline__ void unvox(const Geo& g, long long m, int& n, int& d, int& h, int& w) {
  w = (int)(m % g.w);
  long long r = m / g.w;
  h = (int)(r % g.h);
  r /= g.h;
  d = (int)(r % g.d);
  n = (int)(r / g.d);
}

// ---------------------------------------------------------- fwd / bwd-data
// MODE 0: forward.  Row m = output voxel of y; k = tap*Cin + ci; A = x at
//         input position o*stride + tap - pad.
// MODE 1: input gradient.  Row m = input voxel of dx; k = tap*Cout + co;
//         A = dy at output position (i + pad - tap)/stride when integral.
template <int MODE, int BN>
__global__ void __launch_bounds__(256) k_conv_gemm(const uint16_t* __restrict__ src, Geo gs,  // gathered tensor
                                                  const uint16_t* __restrict__ wk, int kpad,   // [BNcols][kpad]
                                                  const float* __restrict__ bias, uint16_t* __restrict__ out,
                                                  Geo go,                                       // rows = voxels of go
                                                  const uint16_t* __restrict__ act, int act_ldc, int ksize,
                                                  int stride, int relu, int accumulate, int kin) {
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const long long M = (long long)go.n * go.d * go.h * go.w;
  const long long m0 = (long long)blockIdx.x * BM;
  const int n0 = blockIdx.y * BN;
  const int ncols = go.c;
  const int pad = ksize == 3 ? 1 : 0;
  const int taps = ksize * ksize * ksize;

  // A loads: BM rows x 4 chunks of 8 -> 512 chunks, 2 per thread
  int a_row[2], a_chk[2];
  int an[2], ad[2], ah[2], aw[2];
  bool a_ok[2];
  for (int q = 0; q < 2; ++q) {
    const int id = tid + q * 256;
    a_row[q] = id >> 2;
    a_chk[q] = id & 3;
    const long long m = m0 + a_row[q];
    a_ok[q] = m < M;
    unvox(go, a_ok[q] ? m : 0, an[q], ad[q], ah[q], aw[q]);
  }
  f32x4 acc[2][BN / 16];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < BN / 16; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = 0; k0 < kpad; k0 += BK) {
    // ---- stage A
    for (int q = 0; q < 2; ++q) {
      const int k = k0 + a_chk[q] * 8;
      const int tap = k / kin, c0 = k - tap * kin;
      u32x4 v = u32x4{0u, 0u, 0u, 0u};
      if (a_ok[q] && tap < taps) {
        const int kd = tap / (ksize * ksize), kh = (tap / ksize) % ksize, kw = tap % ksize;
        int sd, sh, sw;
        bool ok;
        if (MODE == 0) {
          sd = ad[q] * stride + kd - pad;
          sh = ah[q] * stride + kh - pad;
          sw = aw[q] * stride + kw - pad;
          ok = sd >= 0 && sd < gs.d && sh >= 0 && sh < gs.h && sw >= 0 && sw < gs.w;
        } else {
          const int td = ad[q] + pad - kd, th = ah[q] + pad - kh, tw = aw[q] + pad - kw;
          ok = td >= 0 && th >= 0 && tw >= 0 && (td % stride) == 0 && (th % stride) == 0 && (tw % stride) == 0;
          sd = td / stride;
          sh = th / stride;
          sw = tw / stride;
          ok = ok && sd < gs.d && sh < gs.h && sw < gs.w;
        }
        if (ok) v = *(const u32x4*)(src + vox(gs, an[q], sd, sh, sw) * gs.ldc + c0);
      }
      *(u32x4*)(As + a_row[q] * LDK + a_chk[q] * 8) = v;
    }
    // ---- stage B: BN rows x 4 chunks
    for (int id = tid; id < BN * 4; id += 256) {
      const int r = id >> 2, ch = id & 3;
      u32x4 v = u32x4{0u, 0u, 0u, 0u};
      if (n0 + r < ncols) v = *(const u32x4*)(wk + (long long)(n0 + r) * kpad + k0 + ch * 8);
      *(u32x4*)(Bs + r * LDK + ch * 8) = v;
    }
    __syncthreads();
    const int row = lane & 15, kg = (lane >> 4) * 8;
    bf16x8 a0 = *(const bf16x8*)(As + (wave * 32 + row) * LDK + kg);
    bf16x8 a1 = *(const bf16x8*)(As + (wave * 32 + 16 + row) * LDK + kg);
#pragma unroll
    for (int j = 0; j < BN / 16; ++j) {
      bf16x8 b = *(const bf16x8*)(Bs + (j * 16 + row) * LDK + kg);
      acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[0][j], 0, 0, 0);
      acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[1][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // ---- epilogue: lane holds D[(lane/16)*4 + r][lane%16] of each 16x16 tile
  for (int i = 0; i < 2; ++i) {
    for (int r = 0; r < 4; ++r) {
      const long long m = m0 + wave * 32 + i * 16 + (lane >> 4) * 4 + r;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < BN / 16; ++j) {
        const int n = n0 + j * 16 + (lane & 15);
        if (n >= ncols) continue;
        float v = acc[i][j][r];
        if (bias) v += bias[n];
        if (relu) v = v > 0.f ? v : 0.f;
        const long long o = m * go.ldc + n;
        if (act && !(bf2f(act[m * act_ldc + n]) > 0.f)) v = 0.f;
        if (accumulate) v += bf2f(out[o]);
        out[o] = f2bf(v);
      }
    }
  }
}

// ------------------------------------------- fwd / bwd-data, tap-major
// The same products with the K loop ordered tap by tap (C gathered channels
// per tap, C a multiple of 32), for the shapes where that holds:
//  * each wave's A operand goes straight from memory into the MFMA registers
//    (lane = row l%16, K group l/16: one 16-byte load of 8 channels of the
//    tap's source voxel), through a raw buffer resource whose range check
//    returns zeros for taps outside the volume;
//  * every row's tap validity is a bit mask computed once, and the tap
//    offset is uniform per K step, so a K step costs each lane one add, one
//    select and one load per A fragment;
//  * the weight tile (shared by the four waves) is double-buffered in LDS,
//    one barrier per K step, and the next step's loads are in flight while
//    the current step's MFMAs run;
//  * the stride-2 input gradient runs per output parity class (grid.z): an
//    input voxel i receives only from taps k with k = i + 1 mod 2 on every
//    axis, so each class runs its 1, 2, 4 or 8 taps instead of 27.
// A wave owns FM 16-row fragments and all 16*FN columns of the tile.
struct DArgs {
  const uint16_t* src;
  Geo gs;
  unsigned src_bytes;  // range of the gathered view, for the buffer resource
  const uint16_t* wk;
  int kstride;         // weight row length
  unsigned wk_bytes;
  const float* bias;
  uint16_t* out;
  Geo go;
  const uint16_t* act;
  int act_ldc;
  int ksize, stride, relu, accumulate, C;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, 0x00020000);
}

// Epilogue of eight consecutive channels of a voxel (lo: the first four):
// bias, ReLU, ReLU' mask, accumulation, rounding, one 16-byte store (channel
// counts are multiples of 8).
__device__ __forceinline__ void store8(const DArgs& a, long long vo, int col, f32x4 lo, f32x4 hi) {
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = k < 4 ? lo[k] : hi[k - 4];
  auto half = [](const u32x4& m, int k) { return bf2f((uint16_t)(m[k >> 1] >> (16 * (k & 1)))); };
  if (a.bias) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] += a.bias[col + k];
  }
  if (a.relu) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = v[k] > 0.f ? v[k] : 0.f;
  }
  if (a.act) {
    const u32x4 m = *(const u32x4*)(a.act + vo * a.act_ldc + col);
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (!(half(m, k) > 0.f)) v[k] = 0.f;
  }
  uint16_t* o = a.out + vo * a.go.ldc + col;
  if (a.accumulate) {
    const u32x4 p = *(const u32x4*)o;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] += half(p, k);
  }
  u32x4 q;
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = (unsigned)f2bf(v[2 * k]) | (unsigned)f2bf(v[2 * k + 1]) << 16;
  *(u32x4*)o = q;
}

// Row m of the tap-major kernels: its output voxel (-1 past the last row),
// the element offset of channel group kg of its source at tap (0, 0, 0), and
// the mask of the taps whose source lies in the volume.
template <int MODE, bool CLS>
__device__ __forceinline__ void tap_row(const DArgs& a, int m, int Mrows, int cd, int ch, int cw, const int (&pcl)[3],
                                        const int (&na)[3], int kg, int& base, int& voxel, unsigned& mask) {
  const Geo& gs = a.gs;
  const Geo& go = a.go;
  const int pad = a.ksize == 3 ? 1 : 0;
  const bool ok = m < Mrows;
  int r = ok ? m : 0;
  int c3[3];
  c3[2] = r % cw; r /= cw;
  c3[1] = r % ch; r /= ch;
  c3[0] = r % cd;
  const int n = r / cd;
  if (CLS)
    for (int x = 0; x < 3; ++x) c3[x] = 2 * c3[x] + pcl[x];
  voxel = ok ? ((n * go.d + c3[0]) * go.h + c3[1]) * go.w + c3[2] : -1;
  const int ext[3] = {gs.d, gs.h, gs.w};
  int b3[3];
  unsigned v3[3];
  for (int x = 0; x < 3; ++x) {
    b3[x] = MODE == 0 ? c3[x] * a.stride - pad : (CLS ? (c3[x] + 1) >> 1 : c3[x] + pad);
    unsigned v = 0;
    for (int j = 0; j < na[x]; ++j) {
      const int sx = MODE == 0 ? b3[x] + j : b3[x] - j;
      if (sx >= 0 && sx < ext[x]) v |= 1u << j;
    }
    v3[x] = v;
  }
  unsigned mm = 0;
  for (int jd = 0; jd < na[0]; ++jd)
    for (int jh = 0; jh < na[1]; ++jh)
      for (int jw = 0; jw < na[2]; ++jw)
        if ((v3[0] >> jd) & (v3[1] >> jh) & (v3[2] >> jw) & 1u) mm |= 1u << ((jd * na[1] + jh) * na[2] + jw);
  mask = ok ? mm : 0u;
  base = (((n * gs.d + b3[0]) * gs.h + b3[1]) * gs.w + b3[2]) * gs.ldc + kg * 8;
}

template <int MODE, bool CLS, int FM, int FN>
__global__ void __launch_bounds__(256) k_conv_tap(DArgs a) {
  constexpr int BN = 16 * FN, WM = 16 * FM, BMW = 4 * WM;
  constexpr int LDB = 40;  // padded weight-tile row (bf16)
  constexpr unsigned OOB = 0x80000000u;
  // weight chunks per thread (BN rows x 4 chunks of 8); rows past BN are
  // spare, so that every thread stores and the loop has no branch
  constexpr int NB = (BN * 4 + 255) / 256;
  constexpr int BROWS = NB * 64;
  __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BROWS * LDB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Geo gs = a.gs, go = a.go;
  const int pad = a.ksize == 3 ? 1 : 0;
  // parity class and its row grid (CLS), else the whole output grid
  int pcl[3] = {0, 0, 0};
  int cd = go.d, ch = go.h, cw = go.w;
  if (CLS) {
    pcl[0] = blockIdx.z & 1;
    pcl[1] = (blockIdx.z >> 1) & 1;
    pcl[2] = (blockIdx.z >> 2) & 1;
    cd = (go.d - pcl[0] + 1) >> 1;
    ch = (go.h - pcl[1] + 1) >> 1;
    cw = (go.w - pcl[2] + 1) >> 1;
  }
  // per-axis tap lists: entry j has kernel index kk(j) and source shift dl(j)
  //   MODE 0:        kk = j, source = o*stride - pad + j
  //   MODE 1, s = 1: kk = j, source = i + pad - j
  //   MODE 1, s = 2: kk = p ? 2j : 1, source = (i + 1)/2 - j  (p = i mod 2)
  int na[3];
  for (int x = 0; x < 3; ++x) na[x] = CLS ? (pcl[x] ? 2 : 1) : a.ksize;
  const int Mrows = go.n * cd * ch * cw;
  const int m0 = blockIdx.x * BMW + wave * WM;

  int basef[FM], voxf[FM];
  unsigned mskf[FM];
#pragma unroll
  for (int f = 0; f < FM; ++f)
    tap_row<MODE, CLS>(a, m0 + f * 16 + (lane & 15), Mrows, cd, ch, cw, pcl, na, lane >> 4, basef[f], voxf[f], mskf[f]);

  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
  const int n0 = blockIdx.y * BN;
  const int ncols = go.c;
  const int cpt = a.C >> 5;  // K steps per tap
  const int nsub = na[0] * na[1] * na[2] * cpt;

  // uniform K-step state: tap position (jd, jh, jw) and channel offset c0
  struct St {
    int jd, jh, jw, c0;
  };
  auto tap_of = [&](const St& q, int& off, int& bit, int& t) {
    int dd, dh, dw, kd, kh, kw;
    if (CLS) {
      dd = -q.jd; dh = -q.jh; dw = -q.jw;
      kd = pcl[0] ? 2 * q.jd : 1; kh = pcl[1] ? 2 * q.jh : 1; kw = pcl[2] ? 2 * q.jw : 1;
    } else {
      dd = MODE == 0 ? q.jd : -q.jd; dh = MODE == 0 ? q.jh : -q.jh; dw = MODE == 0 ? q.jw : -q.jw;
      kd = q.jd; kh = q.jh; kw = q.jw;
    }
    off = ((dd * gs.h + dh) * gs.w + dw) * gs.ldc + q.c0;
    bit = (q.jd * na[1] + q.jh) * na[2] + q.jw;
    t = (kd * a.ksize + kh) * a.ksize + kw;
  };
  // branch-free, so that the K loop stays one loop
  auto advance = [&](St& q) {
    q.c0 += 32;
    const int cw_ = q.c0 == a.C;
    q.c0 = cw_ ? 0 : q.c0;
    q.jw += cw_;
    const int ww = q.jw == na[2];
    q.jw = ww ? 0 : q.jw;
    q.jh += ww;
    const int hw = q.jh == na[1];
    q.jh = hw ? 0 : q.jh;
    q.jd += hw;
  };
  // An offset with the high bit set lies past the buffer's range, which
  // loads zeros without touching memory (proper offsets stay below 2^31).
  // `dead` is OOB for the step after the last, so every step issues the same
  // loads, with no branch, and the waits stay exact.
  auto load_a = [&](int off, int bit, unsigned dead, u32x4* dst) {
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      const unsigned vo = (unsigned)(basef[f] + off) * 2u | ((~(mskf[f] >> bit) & 1u) << 31) | dead;
      dst[f] = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, 0, 0);
    }
  };
  // per-thread weight offsets; the high bit sends a spare or missing row
  // out of range (offsets proper stay below 2^31)
  unsigned boff[NB], bpen[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int id = tid + i * 256;
    const int r = id >> 2, chk = id & 3;
    const bool ok = id < BN * 4 && n0 + r < ncols;
    boff[i] = (unsigned)((ok ? n0 + r : 0) * a.kstride + chk * 8) * 2u;
    bpen[i] = ok ? 0u : OOB;
  }
  auto load_b = [&](int t, int c0, unsigned dead, u32x4* dst) {
    const unsigned kb = (unsigned)(t * a.C + c0) * 2u;
#pragma unroll
    for (int i = 0; i < NB; ++i)
      dst[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (boff[i] + kb) | bpen[i] | dead, 0, 0);
  };
  auto store_b = [&](int buf, const u32x4* v) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int id = tid + i * 256;
      *(u32x4*)(&Bs[buf][(id >> 2) * LDB + (id & 3) * 8]) = v[i];
    }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[f][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  St st{0, 0, 0, 0};
  u32x4 acur[FM], anxt[FM], breg[NB];
  {
    int off, bit, t;
    tap_of(st, off, bit, t);
    load_b(t, 0, 0u, breg);
    load_a(off, bit, 0u, acur);
  }
  store_b(0, breg);
  __syncthreads();
  // K step s: issue the loads of step s + 1 (weights first, so that staging
  // them waits for no A load), multiply step s (operands in acur, weights in
  // LDS buffer s & 1), then stage the next weights
  // two steps per iteration, the A registers alternating between acur and
  // anxt, so that a load is first waited for one step after its issue
#define LBM_CONV_KSTEP(S, CUR, NXT)                                                                          \
  {                                                                                                        \
    advance(st);                                                                                           \
    const unsigned dead = (unsigned)(nsub - 2 - (S)) & OOB; /* S + 1 == nsub */                            \
    int off, bit, t;                                                                                       \
    tap_of(st, off, bit, t);                                                                               \
    load_b(t, st.c0, dead, breg);                                                                          \
    load_a(off, bit, dead, NXT);                                                                           \
    __builtin_amdgcn_sched_barrier(0); /* the loads stay ahead of the MFMAs */                             \
    const uint16_t* B = Bs[(S) & 1];                                                                       \
    _Pragma("unroll") for (int j = 0; j < FN; ++j) {                                                       \
      const bf16x8 b = *(const bf16x8*)(B + (j * 16 + (lane & 15)) * LDB + (lane >> 4) * 8);               \
      _Pragma("unroll") for (int f = 0; f < FM; ++f) acc[f][j] =                                           \
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, CUR[f]), b, acc[f][j], 0, 0, 0); \
    }                                                                                                      \
    store_b(((S) + 1) & 1, breg);                                                                          \
    __syncthreads();                                                                                       \
  }
  int s = 0;
  for (; s + 1 < nsub; s += 2) {
    LBM_CONV_KSTEP(s, acur, anxt)
    LBM_CONV_KSTEP(s + 1, anxt, acur)
  }
  if (s < nsub) LBM_CONV_KSTEP(s, acur, anxt)
#undef LBM_CONV_KSTEP
  // ---- epilogue: lane holds D[(lane/16)*4 + r][lane%16] of each 16x16 tile;
  // the voxel of D row q is held by lane q (A layout row q)
#pragma unroll
  for (int f = 0; f < FM; ++f) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int vo = __shfl(voxf[f], (lane >> 4) * 4 + r);
      if (vo < 0) continue;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = n0 + j * 16 + (lane & 15);
        if (n >= ncols) continue;
        float v = acc[f][j][r];
        if (a.bias) v += a.bias[n];
        if (a.relu) v = v > 0.f ? v : 0.f;
        const long long o = (long long)vo * go.ldc + n;
        if (a.act && !(bf2f(a.act[(long long)vo * a.act_ldc + n]) > 0.f)) v = 0.f;
        if (a.accumulate) v += bf2f(a.out[o]);
        a.out[o] = f2bf(v);
      }
    }
  }
}

// ------------------------------------------------------------- bwd-weight
// C[co][k] += sum over voxels v of dy[v][co] * patch(x)[v][k].  Rows = co
// (BM = 128 covers every Cout here in one or two tiles), columns = k
// (BN = 64), K loop over 32-voxel chunks of this workgroup's voxel range.
__global__ void __launch_bounds__(256) k_conv_wgrad(const uint16_t* __restrict__ x, Geo gx,
                                                    const uint16_t* __restrict__ dy, Geo gy, float* __restrict__ dw,
                                                    float* __restrict__ part, int kpad, int kin, int ksize, int stride,
                                                    long long vox_per_wg) {
  constexpr int BN = 64;
  __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDK];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN * LDK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int co0 = blockIdx.x * BM;
  const int k0c = blockIdx.y * BN;
  const long long V = (long long)gy.n * gy.d * gy.h * gy.w;
  const long long vbeg = (long long)blockIdx.z * vox_per_wg;
  const long long vend = vbeg + vox_per_wg < V ? vbeg + vox_per_wg : V;
  const int pad = ksize == 3 ? 1 : 0;
  const int taps = ksize * ksize * ksize;
  const int cout = gy.c;
  f32x4 acc[2][BN / 16];
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < BN / 16; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (long long v0 = vbeg; v0 < vend; v0 += BK) {
    // A[co][vox]: 32 voxels x 128 co -> 512 chunks of 8 co, 2 per thread
    for (int q = 0; q < 2; ++q) {
      const int id = tid + q * 256;
      const int vv = id & 31, cc = id >> 5;  // 16 chunks of 8 co
      const long long v = v0 + vv;
      uint16_t e[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (v < vend && co0 + cc * 8 < cout) {
        const u32x4 t = *(const u32x4*)(dy + v * gy.ldc + co0 + cc * 8);
        e[0] = t[0] & 0xffff; e[1] = t[0] >> 16; e[2] = t[1] & 0xffff; e[3] = t[1] >> 16;
        e[4] = t[2] & 0xffff; e[5] = t[2] >> 16; e[6] = t[3] & 0xffff; e[7] = t[3] >> 16;
      }
      for (int j = 0; j < 8; ++j) As[(cc * 8 + j) * LDK + vv] = e[j];
    }
    // B[k][vox]: 32 voxels x 64 k -> 256 chunks of 8 k, 1 per thread
    {
      const int vv = tid & 31, kc = tid >> 5;  // 8 chunks of 8 k
      const long long v = v0 + vv;
      const int k = k0c + kc * 8;
      const int tap = k / kin, c0 = k - tap * kin;
      uint16_t e[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (v < vend && tap < taps) {
        int n, d, h, w;
        unvox(gy, v, n, d, h, w);
        const int kd = tap / (ksize * ksize), kh = (tap / ksize) % ksize, kw = tap % ksize;
        const int sd = d * stride + kd - pad, sh = h * stride + kh - pad, sw = w * stride + kw - pad;
        if (sd >= 0 && sd < gx.d && sh >= 0 && sh < gx.h && sw >= 0 && sw < gx.w) {
          const u32x4 t = *(const u32x4*)(x + vox(gx, n, sd, sh, sw) * gx.ldc + c0);
          e[0] = t[0] & 0xffff; e[1] = t[0] >> 16; e[2] = t[1] & 0xffff; e[3] = t[1] >> 16;
          e[4] = t[2] & 0xffff; e[5] = t[2] >> 16; e[6] = t[3] & 0xffff; e[7] = t[3] >> 16;
        }
      }
      for (int j = 0; j < 8; ++j) Bs[(kc * 8 + j) * LDK + vv] = e[j];
    }
    __syncthreads();
    const int row = lane & 15, kg = (lane >> 4) * 8;
    bf16x8 a0 = *(const bf16x8*)(As + (wave * 32 + row) * LDK + kg);
    bf16x8 a1 = *(const bf16x8*)(As + (wave * 32 + 16 + row) * LDK + kg);
#pragma unroll
    for (int j = 0; j < BN / 16; ++j) {
      bf16x8 b = *(const bf16x8*)(Bs + (j * 16 + row) * LDK + kg);
      acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[0][j], 0, 0, 0);
      acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[1][j], 0, 0, 0);
    }
    __syncthreads();
  }
  for (int i = 0; i < 2; ++i)
    for (int r = 0; r < 4; ++r) {
      const int co = co0 + wave * 32 + i * 16 + (lane >> 4) * 4 + r;
      if (co >= cout) continue;
#pragma unroll
      for (int j = 0; j < BN / 16; ++j) {
        const int k = k0c + j * 16 + (lane & 15);
        if (k >= kpad) continue;
        const long long e = (long long)co * kpad + k;
        if (part)
          part[(long long)blockIdx.z * cout * kpad + e] = acc[i][j][r];
        else
          atomicAdd(dw + e, acc[i][j][r]);
      }
    }
}

// ------------------------------ fwd / bwd-data, stride 1, 3x3x3, row tiles
typedef __attribute__((address_space(3))) void lds_void;

// 16 bytes per lane from a buffer straight into LDS: lane l's bytes land at
// dst + 16 l (dst uniform), an offset past the range stores zeros.
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t rs, uint16_t* dst, unsigned voff, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, (int)voff, (int)soff, 0, 0);
}

// A barrier that every wave's LDS-direct loads end before: vmcnt(0), said
// outright, as the barrier alone orders LDS accesses and not these loads (the
// other counters at their no-wait values).
__device__ __forceinline__ void load_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();
}

// The stride-1 3x3x3 products.  A workgroup owns a TH x 16 tile of output
// voxels (rows h0.., columns w0.. of one plane) and 32 output channels; per
// source plane and 32-channel chunk it brings the input halo (TH + 2) x 18 x 32
// and the nine taps' weights into LDS by 16-byte buffer loads that write LDS
// directly (no staging registers, no ds_write), then multiplies.  Wave v owns R
// rows of 16 voxels.  What the tile is built around is LDS reads per MFMA:
//  * an operand of 16 voxels of halo row r serves the taps kh = 0, 1, 2 of
//    output rows r, r - 1 and r - 2 from registers, and the nine taps' weights
//    stay in registers for the whole stage: 3 (R + 2) voxel and 18 weight
//    reads for 18 R MFMAs (36 for 72 with R = 4; reading both operands tap by
//    tap takes 54);
//  * 39 KB of LDS and 122 VGPRs (R = 4) keep four workgroups per compute unit,
//    so one's loads run under the others' MFMAs and a stage needs no second
//    buffer (three workgroups, without the register limit: 258 against 237 us
//    on the first layer below).  Tiles of 8 rows per wave or 64 channels read
//    LDS less, leave two workgroups and measured slower.
// Every output sums its products in the order (plane kd, 32-channel chunk, kh,
// kw), so a layer's result does not depend on the tile.
// The weights are the MFMA's row operand, its row m of fragment j standing for
// channel 8 (m / 4) + 4 j + m % 4: a lane then ends with eight consecutive
// channels of one voxel, one 16-byte store (two 8-byte stores: forward 4 %,
// input gradient with its mask 7 % slower).  LDS cells are 64 bytes, unpadded
// as the direct loads want them; the 16-byte chunks of a cell are permuted by
// its column (by the channel / 8 for weights) so that the 8 lanes of a read
// cycle meet 8 different bank groups.
// MODE 1 (input gradient) runs the mirrored taps on the transposed weights.
// Channels in 8s: the part of a chunk past C loads zeros (TAIL).
// Measured on gfx950 at batch 8, us, forward / input gradient with its mask,
// against the halo-staged and tap-major kernels before: 128x64x64 32->32 370 / 477
// -> 236 / 272, 64->32 555 / 1047 -> 407 / 522; 64x32x32 64->64 146 / 163 -> 102 /
// 107, 128->64 forward 235 -> 192 (1210 TFLOP/s; a large library matrix product
// reaches 1280-1380 here).  The full-resolution layers are held by HBM (0.54 GB
// forward, 0.8 with the mask) beside the MFMAs, the rest by the matrix cores.
template <int MODE, int R, bool TAIL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) k_conv_rows(DArgs a) {
  constexpr int FN = 2, BN = 16 * FN;
  constexpr int TW = 16, TH = R * 4;            // output tile of the workgroup
  constexpr int HC = TW + 2, HR = TH + 2;       // its halo
  constexpr int CELLS = HR * HC;
  constexpr int NXI = (CELLS * 4 + 63) / 64;    // wave-wide 16-byte loads of the halo
  constexpr int NWI = 9 * BN * 4 / 64;          // ... of the weights
  constexpr int SX = (NXI + 3) / 4, SW = (NWI + 3) / 4;
  constexpr int TPI = 256 / (BN * 4);           // taps per round of weight loads
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[NXI * 512];
  __shared__ __attribute__((aligned(1024))) uint16_t Ws[NWI * 512];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gs = a.gs, go = a.go;
  const int ncols = go.c, C = a.C;
  // XCD-aware work index: neighbouring tiles and the column tiles of one
  // voxel tile share an XCD's L2
  const int total = (int)gridDim.x, id0 = (int)blockIdx.x, q8 = total / 8 * 8;
  int bx = id0 < q8 ? (id0 % 8) * (total / 8) + id0 / 8 : id0;
  const int nct = (ncols + BN - 1) / BN, nwb = (go.w + TW - 1) / TW, nhb = (go.h + TH - 1) / TH;
  const int n0 = bx % nct * BN;
  bx /= nct;
  const int w0 = bx % nwb * TW;
  bx /= nwb;
  const int h0 = bx % nhb * TH;
  bx /= nhb;
  const int d = bx % go.d, n = bx / go.d;

  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
  // load slots: 16-byte chunk (id & 3) of a cell holds channels
  // 8 (chunk ^ (column / 2 mod 4)) .. + 7 of the stage's 32
  unsigned xoff[SX];
  int xq[SX];
#pragma unroll
  for (int i = 0; i < SX; ++i) {
    const int id = (i * 4 + wave) * 64 + lane;
    const int cell = id >> 2, r = cell / HC, c = cell - r * HC;
    const int q = (id & 3) ^ ((c >> 1) & 3);
    const int hs = h0 - 1 + r, ws = w0 - 1 + c;
    const bool ok = cell < CELLS && hs >= 0 && hs < gs.h && ws >= 0 && ws < gs.w;
    xq[i] = q;
    xoff[i] = ok ? (unsigned)((hs * gs.w + ws) * gs.ldc + q * 8) * 2u : OOB;
  }
  unsigned woff;
  int wq;
  {
    const int rem = tid % (BN * 4), t = tid / (BN * 4);
    const int col = rem >> 2;
    wq = (rem & 3) ^ ((col >> 3) & 3);
    woff = n0 + col < ncols ? (unsigned)((n0 + col) * a.kstride + t * C + wq * 8) * 2u : OOB;
  }
  const int L = lane & 15, g = lane >> 4;
  const int hr0 = wave * R;
  // LDS bases of the operand reads: per column shift of the halo, and weights
  const uint16_t* xb[3];
#pragma unroll
  for (int ow = 0; ow < 3; ++ow)
    xb[ow] = Xs + (hr0 * HC + L + ow) * 32 + ((g ^ (((L + ow) >> 1) & 3)) * 8);
  const uint16_t* wb = Ws + ((L >> 2) * 8 + (L & 3)) * 32 + ((g ^ (L >> 2)) * 8);

  f32x4 acc[R][FN];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const unsigned plane = (unsigned)(gs.h * gs.w * gs.ldc) * 2u;
  for (int kd = 0; kd < 3; ++kd) {
    const int ds = MODE == 0 ? d + kd - 1 : d + 1 - kd;
    if (ds < 0 || ds >= gs.d) continue;  // the plane beyond the volume adds nothing
    const unsigned sp = (unsigned)(n * gs.d + ds) * plane;
    for (int c0 = 0; c0 < C; c0 += 32) {
      __syncthreads();  // the previous stage's readers are done
#pragma unroll
      for (int i = 0; i < SX; ++i)
        if (i * 4 + wave < NXI)
          lds_dma16(rs, Xs + (i * 4 + wave) * 512, !TAIL || c0 + xq[i] * 8 < C ? xoff[i] : OOB, sp + (unsigned)c0 * 2u);
#pragma unroll
      for (int i = 0; i < SW; ++i)
        if (i * 4 + wave < NWI)
          lds_dma16(rw, Ws + (i * 4 + wave) * 512, !TAIL || c0 + wq * 8 < C ? woff : OOB,
                    (unsigned)((kd * 9 + i * TPI) * C + c0) * 2u);
      load_barrier();
      bf16x8 wf[9][FN];
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int j = 0; j < FN; ++j) wf[t][j] = *(const bf16x8*)(wb + (t * BN + j * 4) * 32);
#pragma unroll
      for (int r_ = 0; r_ < R + 2; ++r_) {
        const int r = MODE == 0 ? r_ : R + 1 - r_;  // halo row
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
          const bf16x8 xf = *(const bf16x8*)(xb[MODE == 0 ? kw : 2 - kw] + r * HC * 32);
#pragma unroll
          for (int kh = 0; kh < 3; ++kh) {
            const int ro = MODE == 0 ? r - kh : r - 2 + kh;  // output row that tap (kh, kw) takes this one to
            if (ro < 0 || ro >= R) continue;
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[ro][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kh * 3 + kw][j], xf, acc[ro][j], 0, 0, 0);
          }
        }
      }
    }
  }
  // epilogue: the two accumulators hold channels 8 g .. + 3 and + 4 .. + 7 of
  // voxel column L of each row
  const int w = w0 + L, col = n0 + g * 8;
  if (w >= go.w || col >= ncols) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int h = h0 + hr0 + r;
    if (h >= go.h) break;
    const long long vo = (((long long)n * go.d + d) * go.h + h) * go.w + w;
    store8(a, vo, col, acc[r][0], acc[r][1]);
  }
}

// ----------------------- fwd / bwd-data, stride 1, 3x3x3, plane tiles, tap-major
// The stride-1 3x3x3 products of 64, 128 or 256 channels (NC chunks of 32)
// whose sums run tap by tap with the chunks inside.  Against the tap-major
// kernel, which gathers every operand from L1/L2 once per tap (about 10 TB/s
// in all) and waits on those loads in every K step, a workgroup brings the
// halo of one source plane, all chunks, into LDS once for its nine taps, and
// streams the taps' weights ([column][32 NC channels]) through two LDS buffers
// one tap ahead; both operands are LDS reads.  A tile is 4 R rows of 16 voxels
// and 32 WN columns: wave v takes R rows and 32 columns.  A 16-voxel operand
// is a row of 16 (WF = 16) or rows of 8 of two planes (WF = 8, the volumes 8
// wide, or off 16s).  Cell layout, weight rows and stores as in k_conv_rows.
// Bound by LDS reads (four for four MFMAs per chunk with R = 2) at full chips
// and by the chain of nine weight loads per plane at small ones.  Measured on
// gfx950, us, against the tap-major kernel: batch 1 16x8x8 256->256 67.6 ->
// 19.0, 32x16x16 128->128 41 -> 16.2 and 256->128 85 -> 26; batch 8 87 -> 56,
// 85 -> 64 and 155 -> 140 (831 TFLOP/s); input gradients alike (89 -> 58, 91 ->
// 65, 165 -> 130; 64x32x32 128->64 380 -> 251).  MODE 1 runs mirrored taps.
template <int MODE, int NC, int WF, int R, int WN>
__global__ void __launch_bounds__(256 * WN) k_conv_plane(DArgs a) {
  constexpr int FN = 2, BN = 16 * FN * WN;
  constexpr int NWV = 4 * WN;                   // waves: 4 row groups x WN column groups
  constexpr int DP = 16 / WF;                   // planes of a 16-voxel operand
  constexpr int TH = R * 4;
  constexpr int HC = WF + 2, HR = TH + 2;
  constexpr int CELLS = DP * HR * HC;
  constexpr int NXI = (CELLS * 4 + 63) / 64;    // wave-wide 16-byte loads of one chunk's halo
  constexpr int SX = (NXI + NWV - 1) / NWV;
  constexpr int SW = NC / 2;                    // ... of a tap's weights, per wave
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[NC][NXI * 512];
  __shared__ __attribute__((aligned(1024))) uint16_t Ws[2][NC * BN * 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gs = a.gs, go = a.go;
  const int ncols = go.c;
  constexpr int C = NC * 32;
  const int total = (int)gridDim.x, id0 = (int)blockIdx.x, q8 = total / 8 * 8;
  int bx = id0 < q8 ? (id0 % 8) * (total / 8) + id0 / 8 : id0;
  const int nct = (ncols + BN - 1) / BN, nwb = (go.w + WF - 1) / WF, nhb = (go.h + TH - 1) / TH,
            ndb = (go.d + DP - 1) / DP;
  const int n0 = bx % nct * BN;
  bx /= nct;
  const int w0 = bx % nwb * WF;
  bx /= nwb;
  const int h0 = bx % nhb * TH;
  bx /= nhb;
  const int d0 = bx % ndb * DP, n = bx / ndb;

  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
  unsigned xoff[SX];
  int xp[SX];
#pragma unroll
  for (int i = 0; i < SX; ++i) {
    const int id = (i * NWV + wave) * 64 + lane;
    const int cell = id >> 2, p = cell / (HR * HC), r = cell / HC % HR, c = cell % HC;
    const int q = (id & 3) ^ ((c >> 1) & 3);
    const int hs = h0 - 1 + r, ws = w0 - 1 + c;
    const bool ok = cell < CELLS && hs >= 0 && hs < gs.h && ws >= 0 && ws < gs.w;
    xp[i] = p;
    xoff[i] = ok ? (unsigned)(((p * gs.h + hs) * gs.w + ws) * gs.ldc + q * 8) * 2u : OOB;
  }
  unsigned woff[SW];
#pragma unroll
  for (int i = 0; i < SW; ++i) {
    const int id = (i * NWV + wave) * 64 + lane;
    const int ck = id / (BN * 4), rem = id % (BN * 4);
    const int col = rem >> 2, q = (rem & 3) ^ ((col >> 3) & 3);
    woff[i] = n0 + col < ncols ? (unsigned)((n0 + col) * a.kstride + ck * 32 + q * 8) * 2u : OOB;
  }
  auto load_w = [&](int t, int buf) {
#pragma unroll
    for (int i = 0; i < SW; ++i) lds_dma16(rw, Ws[buf] + (i * NWV + wave) * 512, woff[i], (unsigned)(t * C) * 2u);
  };
  const int L = lane & 15, g = lane >> 4;
  const int hr0 = wave / WN * R, nc0 = wave % WN * 32, vp = L / WF, vc = L % WF;
  int xb[3];
#pragma unroll
  for (int kw = 0; kw < 3; ++kw)
    xb[kw] = ((vp * HR + hr0) * HC + vc + kw) * 32 + ((g ^ (((vc + kw) >> 1) & 3)) * 8);
  const int wb = (nc0 + (L >> 2) * 8 + (L & 3)) * 32 + ((g ^ (L >> 2)) * 8);

  f32x4 acc[R][FN];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const unsigned plane = (unsigned)(gs.h * gs.w * gs.ldc) * 2u;
  for (int kd = 0; kd < 3; ++kd) {
    const int ds = MODE == 0 ? d0 + kd - 1 : d0 + 1 - kd;  // source plane of the tile's first one
    if (ds + DP <= 0 || ds >= gs.d) continue;
    const unsigned sp = (unsigned)(n * gs.d + ds) * plane;
    __syncthreads();  // the previous plane's readers are done
    load_w(kd * 9, 0);
#pragma unroll
    for (int i = 0; i < SX; ++i)
      if (i * NWV + wave < NXI) {
        const bool ok = ds + xp[i] >= 0 && ds + xp[i] < gs.d;
        // (a tile's first plane may lie before the volume: its offset is added per lane)
        const unsigned vo = ok && xoff[i] != OOB ? xoff[i] + sp : OOB;
#pragma unroll
        for (int k = 0; k < NC; ++k) lds_dma16(rs, Xs[k] + (i * NWV + wave) * 512, vo, (unsigned)k * 64u);
      }
    load_barrier();
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      if (t < 8) load_w(kd * 9 + t + 1, (t + 1) & 1);  // in flight while this tap runs
      const int kh = t / 3, kw = t % 3;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        bf16x8 wf[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) wf[j] = *(const bf16x8*)(&Ws[t & 1][wb + (k * BN + j * 4) * 32]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const bf16x8 xf = *(const bf16x8*)(&Xs[k][xb[MODE == 0 ? kw : 2 - kw] + (r + (MODE == 0 ? kh : 2 - kh)) * HC * 32]);
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf, acc[r][j], 0, 0, 0);
        }
      }
      load_barrier();  // this tap's weights are read, the next one's have arrived
    }
  }
  const int w = w0 + vc, d = d0 + vp, col = n0 + nc0 + g * 8;
  if (w >= go.w || d >= go.d || col >= ncols) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int h = h0 + hr0 + r;
    if (h >= go.h) break;
    const long long vo = (((long long)n * go.d + d) * go.h + h) * go.w + w;
    store8(a, vo, col, acc[r][0], acc[r][1]);
  }
}

// ------------------------------------- bwd-data, stride 2, 3x3x3, all parities
// The stride-2 input gradients of 32 or 64 channels (NC chunks).  An input
// voxel i = 2 j + p receives, per axis, from dy voxel j through tap 1 (p = 0), or
// from j + 1 through tap 0 and j through tap 2 (p = 1).  The tap-major kernel runs
// the eight parities as separate grids, each gathering dy and writing every
// other voxel of a line; here a workgroup owns 4 R rows of 16 dy voxels of one
// plane, i.e. their 2 x 8 R x 32 input voxels, and 32 channels: dy and its next
// plane, row and column come into LDS once, all chunks, and the weights pass
// through two LDS buffers in nine stages of three kw taps, grouped by the parity
// of plane and row.  Both parities along w are finished together, so a lane
// writes two neighbouring voxels.  Cells, weight rows and stores as in
// k_conv_rows; the order of the sums is the tap-major kernel's (kd, kh, kw,
// chunk), bit for bit.  Bound by HBM (the mask and the accumulated gradient).
// Measured on gfx950, with the mask: batch 8 128x64x64 32 <- 64 channels 479 us
// before, 178 now, adding to a gradient that is there 665 and 275; batch 4
// 100x60x52 32 <- 64 125 before, 63 now.
template <int NC, int R>
__global__ void __launch_bounds__(256) k_conv_up(DArgs a) {
  constexpr int TH = 4 * R, HC = 17, HR = TH + 1, CELLS = 2 * HR * HC;
  constexpr int NXI = (CELLS * 4 + 63) / 64, NWI = 6 * NC;  // wave-wide 16-byte loads: a chunk's halo, a stage's weights
  constexpr int SX = (NXI + 3) / 4, SW = (NWI + 3) / 4;
  constexpr int C = NC * 32;
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[NC][NXI * 512];
  __shared__ __attribute__((aligned(1024))) uint16_t Ws[2][NWI * 512];  // [kw][chunk][32 columns][32]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gs = a.gs, go = a.go;
  const int total = (int)gridDim.x, id0 = (int)blockIdx.x, q8 = total / 8 * 8;
  int bx = id0 < q8 ? (id0 % 8) * (total / 8) + id0 / 8 : id0;
  const int nct = (go.c + 31) / 32, nwb = (gs.w + 15) / 16, nhb = (gs.h + TH - 1) / TH;
  const int n0 = bx % nct * 32;
  bx /= nct;
  const int w0 = bx % nwb * 16;
  bx /= nwb;
  const int h0 = bx % nhb * TH;
  bx /= nhb;
  const int jd0 = bx % gs.d, n = bx / gs.d;
  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
  unsigned woff[SW];
#pragma unroll
  for (int i = 0; i < SW; ++i) {
    const int id = (i * 4 + wave) * 64 + lane;
    const int kw = id / (NC * 128), ck = id / 128 % NC, col = id % 128 >> 2, q = (id & 3) ^ ((col >> 3) & 3);
    woff[i] = n0 + col < go.c ? (unsigned)((n0 + col) * a.kstride + kw * C + ck * 32 + q * 8) * 2u : OOB;
  }
  // stage s: parities (pd, ph) of plane and row, and which of their one or two
  // taps along each (jd, jh)
  auto stage = [](int s, int& pd, int& ph, int& jd, int& jh) {
    constexpr int PD[9] = {0, 0, 0, 1, 1, 1, 1, 1, 1}, PH[9] = {0, 1, 1, 0, 0, 1, 1, 1, 1};
    constexpr int JD[9] = {0, 0, 0, 0, 1, 0, 0, 1, 1}, JH[9] = {0, 0, 1, 0, 0, 0, 1, 0, 1};
    pd = PD[s], ph = PH[s], jd = JD[s], jh = JH[s];
  };
  auto load_w = [&](int s) {
    int pd, ph, jd, jh;
    stage(s, pd, ph, jd, jh);
    const int kd = pd ? 2 * jd : 1, kh = ph ? 2 * jh : 1;
#pragma unroll
    for (int i = 0; i < SW; ++i)
      if (i * 4 + wave < NWI)
        lds_dma16(rw, Ws[s & 1] + (i * 4 + wave) * 512, woff[i], (unsigned)((kd * 3 + kh) * 3 * C) * 2u);
  };
  load_w(0);
#pragma unroll
  for (int i = 0; i < SX; ++i)
    if (i * 4 + wave < NXI) {
      const int id = (i * 4 + wave) * 64 + lane;
      const int cell = id >> 2, p = cell / (HR * HC), r = cell / HC % HR, c = cell % HC;
      const int q = (id & 3) ^ ((c >> 1) & 3);
      const bool ok = cell < CELLS && jd0 + p < gs.d && h0 + r < gs.h && w0 + c < gs.w;
      const unsigned vo =
          ok ? (unsigned)((((n * gs.d + jd0 + p) * gs.h + h0 + r) * gs.w + w0 + c) * gs.ldc + q * 8) * 2u : OOB;
#pragma unroll
      for (int k = 0; k < NC; ++k) lds_dma16(rs, Xs[k] + (i * 4 + wave) * 512, vo, (unsigned)k * 64u);
    }
  const int L = lane & 15, g = lane >> 4;
  int xb[2];
#pragma unroll
  for (int o = 0; o < 2; ++o) xb[o] = (wave * R * HC + L + o) * 32 + ((g ^ (((L + o) >> 1) & 3)) * 8);
  const int wb = ((L >> 2) * 8 + (L & 3)) * 32 + ((g ^ (L >> 2)) * 8);
  load_barrier();

  const int col = n0 + g * 8, w = 2 * (w0 + L);
  f32x4 acc[R][2][2];  // [row][parity along w][column fragment]
#pragma unroll
  for (int s = 0; s < 9; ++s) {
    int pd, ph, jd, jh;
    stage(s, pd, ph, jd, jh);
    if (s < 8) load_w(s + 1);  // in flight while this stage runs
    if (jd == 0 && jh == 0) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int o = 0; o < 2; ++o) acc[r][o][0] = acc[r][o][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int xo = ((pd - jd) * HR + ph - jh) * HC * 32;  // source plane and row
    // kw = 1 (even voxels, dy column j), 0 (odd, j + 1), 2 (odd, j)
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int kw = t == 0 ? 1 : (t == 1 ? 0 : 2), odd = t == 0 ? 0 : 1, o = t == 1 ? 1 : 0;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        bf16x8 wf[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) wf[j] = *(const bf16x8*)(&Ws[s & 1][wb + ((kw * NC + k) * 32 + j * 4) * 32]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const bf16x8 xf = *(const bf16x8*)(&Xs[k][xb[o] + xo + r * HC * 32]);
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[r][odd][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf, acc[r][odd][j], 0, 0, 0);
        }
      }
    }
    if (jd == pd && jh == ph) {  // the parity's last stage
      const int d = 2 * jd0 + pd;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int h = 2 * (h0 + wave * R + r) + ph;
#pragma unroll
        for (int o = 0; o < 2; ++o)
          if (d < go.d && h < go.h && w + o < go.w && col < go.c)
            store8(a, (((long long)n * go.d + d) * go.h + h) * go.w + w + o, col, acc[r][o][0], acc[r][o][1]);
      }
    }
    load_barrier();  // this stage's weights are read, the next one's have arrived
  }
}

// --------------------------------------------- fwd / bwd-data, 1x1x1 layers
// The pointwise products (either direction: rows = voxels, K = the gathered
// channels).  A wave takes 64 consecutive voxels (four 16-voxel operands) and
// 32 columns; the operands are direct 16-byte loads, whole lines of the
// channels-last rows, all of a chunk's issued before its MFMAs.  A wave's
// weights of the chunk come from L1.  No LDS: no value is used twice.  Bound by
// HBM.  Measured on gfx950 at 8 x 128x64x64: 32->8 forward 122 -> 69 us, its input
// gradient 233 -> 104 (against the tap-major and the general kernel).
__global__ void __launch_bounds__(256) k_conv_point(DArgs a) {
  constexpr unsigned OOB = 0x80000000u;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int L = lane & 15, g = lane >> 4;
  const Geo go = a.go;
  const int V = go.n * go.d * go.h * go.w;
  const int v0 = (blockIdx.x * 4 + wave) * 64 + L, n0 = blockIdx.y * 32;
  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
  unsigned xo[4], wo[2];
#pragma unroll
  for (int f = 0; f < 4; ++f) xo[f] = v0 + f * 16 < V ? (unsigned)((v0 + f * 16) * a.gs.ldc + g * 8) * 2u : OOB;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = n0 + (L >> 2) * 8 + j * 4 + (L & 3);  // weight rows as in k_conv_rows
    wo[j] = col < go.c ? (unsigned)(col * a.kstride + g * 8) * 2u : OOB;
  }
  f32x4 acc[4][2];
#pragma unroll
  for (int f = 0; f < 4; ++f) acc[f][0] = acc[f][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < a.C; c0 += 32) {
    const unsigned dead = c0 + g * 8 < a.C ? 0u : OOB;
    u32x4 x[4], w[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) w[j] = __builtin_amdgcn_raw_buffer_load_b128(rw, wo[j] | dead, c0 * 2, 0);
#pragma unroll
    for (int f = 0; f < 4; ++f) x[f] = __builtin_amdgcn_raw_buffer_load_b128(rs, xo[f] | dead, c0 * 2, 0);
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j]),
                                                            __builtin_bit_cast(bf16x8, x[f]), acc[f][j], 0, 0, 0);
  }
  const int col = n0 + g * 8;
  if (col >= go.c) return;
#pragma unroll
  for (int f = 0; f < 4; ++f)
    if (v0 + f * 16 < V) store8(a, v0 + f * 16, col, acc[f][0], acc[f][1]);
}

// -------------------------------------- forward, stride 1, 3x3x3, 8 channels
// The input layer.  K = tap * 8 + channel, four taps per MFMA (lane group g of
// step s: tap 4 s + g; the 28th is zeros), seven steps in all, whose weights a
// wave keeps in registers.  A workgroup owns 16 x 16 voxels of kPl planes and 32
// output channels: it brings the kPl + 2 source planes' halos into LDS (16-byte
// cells, LDS-direct loads) once; wave v takes rows 4 v .. 4 v + 3 of every plane.
// A voxel operand is one LDS read per lane, at the lane's own tap.  Bound by the
// stores of its 32 channels.  Measured on gfx950 at 8 x 128x64x64: 366 -> 108 us
// against the general kernel, which gathered every tap from memory.
__global__ void __launch_bounds__(256) k_conv_fwd_c8(DArgs a) {
  constexpr int kPl = 4, HC = 18, HR = 18, CELLS = (kPl + 2) * HR * HC;
  constexpr int NXI = (CELLS + 63) / 64, SX = (NXI + 3) / 4;
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[NXI * 512 + 8];  // the last cell: zeros
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gs = a.gs, go = a.go;
  const int total = (int)gridDim.x, id0 = (int)blockIdx.x, q8 = total / 8 * 8;
  int bx = id0 < q8 ? (id0 % 8) * (total / 8) + id0 / 8 : id0;
  const int nct = (go.c + 31) / 32, nwb = (go.w + 15) / 16, nhb = (go.h + 15) / 16, ndb = (go.d + kPl - 1) / kPl;
  const int n0 = bx % nct * 32;
  bx /= nct;
  const int w0 = bx % nwb * 16;
  bx /= nwb;
  const int h0 = bx % nhb * 16;
  bx /= nhb;
  const int d0 = bx % ndb * kPl, n = bx / ndb;
  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.src, a.src_bytes);
  const __amdgpu_buffer_rsrc_t rw = rsrc_of(a.wk, a.wk_bytes);
#pragma unroll
  for (int i = 0; i < SX; ++i)
    if (i * 4 + wave < NXI) {
      const int cell = (i * 4 + wave) * 64 + lane;
      const int p = cell / (HR * HC), r = cell / HC % HR, c = cell % HC;
      const int ds = d0 - 1 + p, hs = h0 - 1 + r, ws = w0 - 1 + c;
      const bool ok = cell < CELLS && ds >= 0 && ds < gs.d && hs >= 0 && hs < gs.h && ws >= 0 && ws < gs.w;
      lds_dma16(rs, Xs + (i * 4 + wave) * 512,
                ok ? (unsigned)((((n * gs.d + ds) * gs.h + hs) * gs.w + ws) * gs.ldc) * 2u : OOB, 0);
    }
  if (tid == 0) *(u32x4*)(Xs + NXI * 512) = u32x4{0u, 0u, 0u, 0u};
  const int L = lane & 15, g = lane >> 4;
  bf16x8 wf[7][2];
#pragma unroll
  for (int s = 0; s < 7; ++s)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + (L >> 2) * 8 + j * 4 + (L & 3);
      const unsigned wo = col < go.c ? (unsigned)(col * a.kstride + s * 32 + g * 8) * 2u : OOB;
      wf[s][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, wo, 0, 0));
    }
  int xo[7];  // cell of the lane's tap, relative to the output voxel's row and plane
#pragma unroll
  for (int s = 0; s < 7; ++s) {
    const int t = 4 * s + g;
    xo[s] = ((t / 9 * HR + t / 3 % 3) * HC + t % 3 + L) * 8;
  }
  const bool none = g == 3;  // tap 27 of the last step
  load_barrier();
  const int w = w0 + L, col = n0 + g * 8;
  for (int p = 0; p < kPl; ++p) {
    if (d0 + p >= go.d) break;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int h = h0 + wave * 4 + r;
      const int base = (p * HR + wave * 4 + r) * HC * 8;
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < 7; ++s) {
        const int at = s == 6 && none ? NXI * 512 : base + xo[s];
        const bf16x8 xf = *(const bf16x8*)(Xs + at);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][j], xf, acc[j], 0, 0, 0);
      }
      if (h < go.h && w < go.w && col < go.c)
        store8(a, (((long long)n * go.d + d0 + p) * go.h + h) * go.w + w, col, acc[0], acc[1]);
    }
  }
}

// ------------------------------------------------------- bwd-weight operands
struct WArgs {
  const uint16_t* x;
  Geo gx;
  unsigned x_bytes;
  const uint16_t* dy;
  Geo gy;
  unsigned dy_bytes;
  float* dw;
  float* db;            // bias gradient, or nullptr
  int kpad;
  int nhb, nwb;         // steps per column of rows / per row
  int steps, per_wg;    // total steps, steps per workgroup
  int nco, nci;         // output / input channel tiles
  float* part;          // the splits' sums [split][Cout][kpad], or nullptr: atomics into dw, db
  float* part_b;        // ... of the bias gradient [split][Cout]
};

// Where a workgroup's sums of dw go: their split's part, stored for k_wgrad_sum,
// or dw itself, added.
__device__ __forceinline__ float* dw_of(const WArgs& a, int split) {
  return a.part ? a.part + (long long)split * a.gy.c * a.kpad : a.dw;
}
template <bool ADD>
__device__ __forceinline__ void put(float* p, float v) {
  if constexpr (ADD)
    atomicAdd(p, v);
  else
    *p = v;
}

// The bias gradient of a split from NG partial sums per channel of a CH-channel
// tile (thread tid: group tid / CH, channel tid % CH), added up through LDS in a
// fixed order.  The caller's waves are past their last reads of `red`.
template <int CH, int NG>
__device__ __forceinline__ void put_db(const WArgs& a, int split, int co0, int tid, float v, float* red) {
  red[tid] = v;
  __syncthreads();
  if (tid < CH && co0 + tid < a.gy.c) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < NG; ++k) t += red[k * CH + tid];
    if (a.part_b)
      a.part_b[(long long)split * a.gy.c + co0 + tid] = t;
    else
      atomicAdd(a.db + co0 + tid, t);
  }
}

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

__device__ __forceinline__ bf16x8 tr_load8(const uint16_t* p, int off_lo, int off_hi) {
  const __attribute__((address_space(3))) uint16_t* q = (const __attribute__((address_space(3))) uint16_t*)p;
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(q + off_lo));
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(q + off_hi));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// ------------------------------------------------ bwd-weight, 3x3x3, row steps
// dw[co][tap*Cin + ci] += sum_v dy[v][co] * x[src(v, tap)][ci] for 3x3x3
// kernels, and (db given) db[co] += sum_v dy[v][co] from the dy tiles already
// in LDS, by the workgroups of kernel plane 0 and input-channel tile 0 (each
// dy tile once).  A workgroup owns one kernel plane kd, 32 input channels and
// BM output channels, i.e. a BM x (9 taps x 32) block of dw, and walks steps of
// RR rows of 32 voxels of dy (a row: 32 along w, or WP along w of 32 / WP planes,
// whichever pads the volume least).  Per step it brings the dy tile and the x
// halo of plane d S + kd - 1, the sources of all nine (kh, kw) taps, into LDS by
// 16-byte buffer loads that write LDS directly; both MFMA operands (voxels as K)
// are then transposing reads (ds_read_b64_tr_b16: a 16-lane group gives the
// addresses of four rows of four 16-bit values; lane l receives column l%16 of
// that 4 x 16 block).
//  * The dy rows stay in registers, and an x row read once per column shift kw
//    serves the three taps kh whose dy row it meets: 26 reads for 72 MFMAs of
//    a wave (tap by tap it takes 44; 40 for 36 with 32 output channels, whose
//    four waves now pair up on two halves of the rows and add up through LDS).
//  * Steps go along the depth first: the workgroups of the three kernel
//    planes, which run side by side on one XCD, then meet each x plane within
//    three steps, in their L2 (going along the rows first read x three times
//    from memory: 128x64x64 32->32 290 against 267 us at batch 8, 64->32 512
//    against 460).
//  * About 768 workgroups, one round (wgrad_splits).  Every one ends with BM x 288
//    values, stored as its split's part and added up in a fixed order by
//    k_wgrad_sum: against FP32 atomics into dw, of which the card takes about 95
//    G/s, the sums repeat bit for bit and are nearer the exact ones (batch 8
//    128x64x64 32->32: dw off by 4.7e-7 of its norm, 5.5e-7 before; db 6e-8, 9e-7
//    before), and small layers may be split further (batch 1 128x64x64 32->32 77
//    -> 49 us).
// Channels in 8s: the part of a tile past Cin or Cout loads zeros.
// Measured on gfx950 at batch 8, us with the sum and the bias, against the
// tap-by-tap kernel with atomics: 128x64x64 32->32 349 -> 242, 64->32 590 -> 495;
// 64x32x32 64->64 190 -> 114; 32x16x16 256->128 182 -> 121; 16x8x8 256->256 69 ->
// 45; stride 2 128x64x64 32->64 141 -> 126; batch 1 128x64x64 32->32 136 -> 50.
// Bound by HBM at full resolution, by LDS reads and MFMAs otherwise.
// (Waves per SIMD: four fit without spills but where the halo or its addresses
// take more registers; asked for four, 64 columns on rows of 32 spill.)
constexpr int wgrad_waves(int S, int BM, int WP) { return S == 2 || WP <= 8 ? 2 : (BM == 64 && WP == 32 ? 3 : 4); }
template <int S, int BM, int WP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(wgrad_waves(S, BM, WP))))
k_conv_wgrad_rows(WArgs a) {
  constexpr int KS = BM == 32 ? 2 : 1;             // waves that share a dw tile, each with RW of a step's rows
  constexpr int RW = S == 2 && BM == 32 ? 2 : 4;   // (eight rows of stride 2 would leave one workgroup per compute unit)
  constexpr int RR = RW * KS;
  constexpr int DP = 32 / WP;                      // planes of a 32-voxel row
  constexpr int HR = (RR - 1) * S + 3, HC = (WP - 1) * S + 3;
  constexpr int CELLS = DP * HR * HC;
  constexpr int NXI = (CELLS * 4 + 63) / 64, NAI = RR * BM / 16;  // wave-wide loads of x and dy
  constexpr int SX = (NXI + 3) / 4, SA = NAI / 4;
  constexpr unsigned OOB = 0x80000000u;
  constexpr int kX = NXI * 512, kA = NAI * 512;
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[kX + kA];
  uint16_t* const As = Xs + kX;                    // [BM / 32][RR * 32 voxels][32 channels]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gx = a.gx, gy = a.gy;
  // XCD-aware work index (see k_conv_rows): the weight tiles of one step range
  // read the same dy and x data and share an XCD's L2
  const int total = (int)gridDim.x, L8 = (int)blockIdx.x, q8 = total / 8 * 8;
  const int idx = L8 < q8 ? (L8 % 8) * (total / 8) + L8 / 8 : L8;
  const int ntiles = 3 * a.nci * a.nco;
  int by = idx % ntiles;
  const int split = idx / ntiles;
  const int co0 = by % a.nco * BM;
  by /= a.nco;
  const int ci0 = by % a.nci * 32;
  const int kd = by / a.nci;

  // load slots: dy chunk (id & 3) of voxel v of row r of channel half hf; x
  // chunk of halo cell (plane p, row, column), for S = 2 with the cell's two
  // 32-byte halves swapped by column so that the strided operand reads meet
  // different banks.  Packed as row | column << 8 | plane << 16.
  int adl[SA], apos[SA], xdl[SX], xpos[SX];
#pragma unroll
  for (int i = 0; i < SA; ++i) {
    const int id = (i * 4 + wave) * 64 + lane;
    const int v = (id >> 2) % (RR * 32), hf = (id >> 2) / (RR * 32), r = v / 32, c = v % WP, p = v % 32 / WP;
    const int ch = co0 + hf * 32 + (id & 3) * 8;
    apos[i] = ch < gy.c ? r | c << 8 | p << 16 : -1;
    adl[i] = (int)((((unsigned)p * gy.h + r) * gy.w + c) * gy.ldc + ch);  // (may wrap past the volume)
  }
#pragma unroll
  for (int i = 0; i < SX; ++i) {
    const int id = (i * 4 + wave) * 64 + lane;
    const int cell = id >> 2, p = cell / (HR * HC), r = cell / HC % HR, c = cell % HC;
    const int q = S == 1 ? id & 3 : (id & 3) ^ (((c >> 2) & 1) << 1);
    const int ch = ci0 + q * 8;
    xpos[i] = cell < CELLS && ch < gx.c ? r | c << 8 | p << 16 : -1;
    xdl[i] = (int)((((unsigned)p * S * gx.h + r) * gx.w + c) * gx.ldc + ch);
  }
  // operand reads: 16-lane group g covers voxels 8 g .. 8 g + 7 of a row, half
  // hh the voxels 8 g + 4 hh .. + 3; lane L addresses voxel L / 4, channels
  // 4 (L % 4) .. + 3 of its 16
  const int L = lane & 15, g = lane >> 4;
  const int jsub = wave & 1, rk = KS == 2 ? (wave >> 1) * RW : 0, cs = KS == 2 ? 0 : wave >> 1;
  int aoff[2], xoff[S == 1 ? 1 : 3][2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int v = 8 * g + 4 * hh + (L >> 2), c = v % WP, p = v / WP;
    aoff[hh] = (cs * (RR * 32) + rk * 32 + v) * 32 + (L & 3) * 4;
#pragma unroll
    for (int k = 0; k < (S == 1 ? 1 : 3); ++k) {
      const int cc = c * S + k;
      const int sub = S == 1 ? jsub : jsub ^ ((cc >> 2) & 1);
      xoff[k][hh] = ((p * HR + rk * S) * HC + cc) * 32 + sub * 16 + (L & 3) * 4;
    }
  }

  const __amdgpu_buffer_rsrc_t rx = rsrc_of(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t rd = rsrc_of(a.dy, a.dy_bytes);
  const int s_begin = split * a.per_wg;
  const int s_end = s_begin + a.per_wg < a.steps ? s_begin + a.per_wg : a.steps;
  const int ndb = (gy.d + DP - 1) / DP;
  int db = s_begin % ndb, pl = s_begin / ndb;
  int wb = pl % a.nwb, hb = pl / a.nwb % a.nhb, nn = pl / (a.nwb * a.nhb);

  constexpr int BG = 256 / BM;
  const bool do_bias = a.db != nullptr && kd == 0 && ci0 == 0;
  const int b_ch = tid % BM, b_v0 = tid / BM * (RR * 32 / BG);

  f32x4 acc[2][9];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  for (int st = s_begin; st < s_end; ++st) {
    const int d0 = db * DP, h0 = hb * RR, w0 = wb * WP;
    const int ab = ((nn * gy.d + d0) * gy.h + h0) * gy.w * gy.ldc + w0 * gy.ldc;
    const int zs = d0 * S + kd - 1, ys = h0 * S - 1, xs = w0 * S - 1;
    const int xb = ((nn * gx.d + zs) * gx.h + ys) * gx.w * gx.ldc + xs * gx.ldc;
    __syncthreads();  // the previous step's readers are done
#pragma unroll
    for (int i = 0; i < SA; ++i) {
      const int r = apos[i] & 255, c = apos[i] >> 8 & 255, p = apos[i] >> 16;
      const bool ok = apos[i] >= 0 && h0 + r < gy.h && w0 + c < gy.w && d0 + p < gy.d;
      lds_dma16(rd, As + (i * 4 + wave) * 512, ok ? (unsigned)(ab + adl[i]) * 2u : OOB, 0);
    }
#pragma unroll
    for (int i = 0; i < SX; ++i)
      if (i * 4 + wave < NXI) {
        const int r = xpos[i] & 255, c = xpos[i] >> 8 & 255, p = xpos[i] >> 16;
        const int z = zs + p * S;
        const bool ok = xpos[i] >= 0 && (unsigned)(ys + r) < (unsigned)gx.h && (unsigned)(xs + c) < (unsigned)gx.w &&
                        (unsigned)z < (unsigned)gx.d;
        lds_dma16(rx, Xs + (i * 4 + wave) * 512, ok ? (unsigned)(xb + xdl[i]) * 2u : OOB, 0);
      }
    ++db;
    const int c1 = db == ndb;
    db = c1 ? 0 : db;
    wb += c1;
    const int c2 = wb == a.nwb;
    wb = c2 ? 0 : wb;
    hb += c2;
    const int c3 = hb == a.nhb;
    hb = c3 ? 0 : hb;
    nn += c3;
    load_barrier();
    bf16x8 af[RW][2];
    // an x row serves every tap row kh whose dy row it meets
#pragma unroll
    for (int xr = 0; xr < (RW - 1) * S + 3; ++xr) {
      if (xr % S == 0 && xr / S < RW) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          af[xr / S][i] = tr_load8(As, aoff[0] + xr / S * 1024 + i * 16, aoff[1] + xr / S * 1024 + i * 16);
      }
#pragma unroll
      for (int kw = 0; kw < 3; ++kw) {
        const int to = xr * HC * 32 + (S == 1 ? kw * 32 : 0);
        const bf16x8 bfr = tr_load8(Xs, xoff[S == 1 ? 0 : kw][0] + to, xoff[S == 1 ? 0 : kw][1] + to);
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
          if (xr - kh < 0 || (xr - kh) % S != 0 || (xr - kh) / S >= RW) continue;
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i][kh * 3 + kw] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[(xr - kh) / S][i], bfr, acc[i][kh * 3 + kw], 0, 0, 0);
        }
      }
    }
    if (do_bias) {
      float t = 0.f;
#pragma unroll 8
      for (int j = 0; j < RR * 32 / BG; ++j)
        t += bf2f(As[((b_ch >> 5) * (RR * 32) + b_v0 + j) * 32 + (b_ch & 31)]);
      bsum += t;
    }
  }
  if constexpr (KS == 2) {
    // the second pair of waves hands its sums over through LDS
    __syncthreads();
    f32x4* red = (f32x4*)Xs + (wave & 1) * (18 * 64) + lane;
    static_assert(2 * 18 * 64 * 16 <= (kX + kA) * 2, "the sums fit");
    if (wave >= 2) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 9; ++t) red[(i * 9 + t) * 64] = acc[i][t];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[i][t] += red[(i * 9 + t) * 64];
    }
  }
  // lane holds D[4 g + q][L] of each tile: rows co, columns ci
  const int cin = gx.c, ci = ci0 + jsub * 16 + L;
  float* const dw = dw_of(a, split);
  auto finish = [&](auto add) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int co = co0 + (cs * 2 + i) * 16 + g * 4 + q;
        if (co >= gy.c) continue;
#pragma unroll
        for (int t = 0; t < 9; ++t)
          put<add.value>(dw + (unsigned)(co * a.kpad + (kd * 9 + t) * cin + ci), acc[i][t][q]);
      }
  };
  if ((KS == 1 || wave < 2) && ci < cin) {
    if (a.part)
      finish(std::false_type{});
    else
      finish(std::true_type{});
  }
  if (do_bias) {
    __syncthreads();  // the last readers of LDS are done
    put_db<BM, BG>(a, split, co0, tid, bsum, (float*)Xs);
  }
}

// --------------------------------- bwd-weight, 3x3x3, 8 input channels
// dw[co][tap*8 + ci] += sum_v dy[v][co] * x[src(v, tap)][ci] for the input
// layer (8 channels, stride 1): all 27 taps of a 32-output-channel tile in one
// workgroup, the 216 columns as 14 MFMA column tiles of two taps x 8 channels
// (the last holds tap 26 and zeros).  Steps are rows of 32 voxels as in
// k_conv_wgrad_rows; per step the dy tile [32 RR voxels][32 channels] and the x
// halo of all source planes (16-byte cells) come into LDS by direct loads.
// ds_read_b64_tr_b16 takes one address per lane, so each lane of an x operand
// points at the tap of its half of the tile's columns.  Wave v owns both
// 16-channel halves of dy and the column tiles v, v + 4, v + 8, v + 12: six reads
// for eight MFMAs of a row.  With db given the dy tiles are summed from LDS
// (each once per channel tile), one value per channel and workgroup.  Bound by LDS
// reads.  Measured on gfx950 at 8 x 128x64x64, 8->32: 121 us with the sum and the
// bias (384 with steps of one row staged through registers; 213 with eight
// atomics per channel and workgroup for the bias, which queued at 32 addresses).
template <int WP>
__global__ void __launch_bounds__(256) k_conv_wgrad_c8(WArgs a) {
  constexpr int RR = 8, DP = 32 / WP;
  constexpr int HR = RR + 2, HC = WP + 2, CELLS = (DP + 2) * HR * HC;
  constexpr int NXI = (CELLS + 63) / 64, NAI = RR * 2;  // wave-wide 16-byte loads of x and dy
  constexpr int SX = (NXI + 3) / 4, SA = NAI / 4;
  constexpr int ZERO = NXI * 512;                       // a cell of zeros (the missing 28th tap)
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t As[NAI * 512];
  __shared__ __attribute__((aligned(1024))) uint16_t Xs[NXI * 512 + 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gx = a.gx, gy = a.gy;
  // XCD-aware work index (see k_conv_wgrad_rows)
  const int total = (int)gridDim.x, L8 = (int)blockIdx.x, q8 = total / 8 * 8;
  const int idx = L8 < q8 ? (L8 % 8) * (total / 8) + L8 / 8 : L8;
  const int co0 = idx % a.nco * 32, split = idx / a.nco;
  if (tid == 0) *(u32x4*)(Xs + ZERO) = u32x4{0u, 0u, 0u, 0u};

  // load slots (row | column << 8 | plane << 16, -1: none)
  int adl[SA], apos[SA], xdl[SX], xpos[SX];
#pragma unroll
  for (int i = 0; i < SA; ++i) {
    const int id = (i * 4 + wave) * 64 + lane;
    const int v = id >> 2, r = v / 32, c = v % WP, p = v % 32 / WP, ch = co0 + (id & 3) * 8;
    apos[i] = ch < gy.c ? r | c << 8 | p << 16 : -1;
    adl[i] = ((p * gy.h + r) * gy.w + c) * gy.ldc + ch;
  }
#pragma unroll
  for (int i = 0; i < SX; ++i) {
    const int cell = (i * 4 + wave) * 64 + lane;
    const int p = cell / (HR * HC), r = cell / HC % HR, c = cell % HC;
    xpos[i] = cell < CELLS ? r | c << 8 | p << 16 : -1;
    xdl[i] = ((p * gx.h + r) * gx.w + c) * gx.ldc;
  }
  // operand reads (16-lane group g covers voxels 8 g .. 8 g + 7 of a row, half
  // hh the voxels 8 g + 4 hh .. + 3; lane L addresses voxel L / 4, columns
  // 4 (L % 4) .. + 3 of its 16)
  const int L = lane & 15, g = lane >> 4, cio = (L & 1) * 4;
  int aoff[2], xv[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int v = 8 * g + 4 * hh + (L >> 2);
    aoff[hh] = v * 32 + (L & 3) * 4;
    xv[hh] = (v / WP * HR * HC + v % WP) * 8 + cio;
  }
  int toff[4];  // the lane's tap of each column tile, -1: none
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int t = 2 * (wave + 4 * j) + ((L & 3) >> 1);
    toff[j] = t < 27 ? ((t / 9 * HR + t / 3 % 3) * HC + t % 3) * 8 : -1;
  }

  const __amdgpu_buffer_rsrc_t rx = rsrc_of(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t rd = rsrc_of(a.dy, a.dy_bytes);
  const int s_begin = split * a.per_wg;
  const int s_end = s_begin + a.per_wg < a.steps ? s_begin + a.per_wg : a.steps;
  const int ndb = (gy.d + DP - 1) / DP;
  int db = s_begin % ndb, pl = s_begin / ndb;
  int wb = pl % a.nwb, hb = pl / a.nwb % a.nhb, nn = pl / (a.nwb * a.nhb);

  const bool do_bias = a.db != nullptr;

  f32x4 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  for (int st = s_begin; st < s_end; ++st) {
    const int d0 = db * DP, h0 = hb * RR, w0 = wb * WP;
    const int ab = ((nn * gy.d + d0) * gy.h + h0) * gy.w * gy.ldc + w0 * gy.ldc;
    const int xb = ((nn * gx.d + d0 - 1) * gx.h + h0 - 1) * gx.w * gx.ldc + (w0 - 1) * gx.ldc;
    __syncthreads();  // the previous step's readers are done
#pragma unroll
    for (int i = 0; i < SA; ++i) {
      const int r = apos[i] & 255, c = apos[i] >> 8 & 255, p = apos[i] >> 16;
      const bool ok = apos[i] >= 0 && h0 + r < gy.h && w0 + c < gy.w && d0 + p < gy.d;
      lds_dma16(rd, As + (i * 4 + wave) * 512, ok ? (unsigned)(ab + adl[i]) * 2u : OOB, 0);
    }
#pragma unroll
    for (int i = 0; i < SX; ++i)
      if (i * 4 + wave < NXI) {
        const int r = xpos[i] & 255, c = xpos[i] >> 8 & 255, p = xpos[i] >> 16;
        const bool ok = xpos[i] >= 0 && (unsigned)(h0 - 1 + r) < (unsigned)gx.h &&
                        (unsigned)(w0 - 1 + c) < (unsigned)gx.w && (unsigned)(d0 - 1 + p) < (unsigned)gx.d;
        lds_dma16(rx, Xs + (i * 4 + wave) * 512, ok ? (unsigned)(xb + xdl[i]) * 2u : OOB, 0);
      }
    ++db;
    const int c1 = db == ndb;
    db = c1 ? 0 : db;
    wb += c1;
    const int c2 = wb == a.nwb;
    wb = c2 ? 0 : wb;
    hb += c2;
    const int c3 = hb == a.nhb;
    hb = c3 ? 0 : hb;
    nn += c3;
    load_barrier();
#pragma unroll
    for (int r = 0; r < RR; ++r) {
      bf16x8 af[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) af[i] = tr_load8(As, aoff[0] + r * 1024 + i * 16, aoff[1] + r * 1024 + i * 16);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j == 3 && wave >= 2) continue;  // 14 column tiles
        const int t = toff[j] + r * HC * 8;
        const bf16x8 bfr = tr_load8(Xs, toff[j] < 0 ? ZERO + cio : xv[0] + t, toff[j] < 0 ? ZERO + cio : xv[1] + t);
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr, acc[i][j], 0, 0, 0);
      }
    }
    if (do_bias) {
      float t = 0.f;
#pragma unroll 8
      for (int j = 0; j < RR * 4; ++j) t += bf2f(As[(tid / 32 * (RR * 4) + j) * 32 + tid % 32]);
      bsum += t;
    }
  }
  // lane holds D[4 g + q][L] of each tile: rows co, columns k
  float* const dw = dw_of(a, split);
  auto finish = [&](auto add) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int co = co0 + i * 16 + g * 4 + q;
        if (co >= gy.c) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int k = (wave + 4 * j) * 16 + L;
          if (k < 216) put<add.value>(dw + (unsigned)(co * a.kpad + k), acc[i][j][q]);
        }
      }
  };
  if (a.part)
    finish(std::false_type{});
  else
    finish(std::true_type{});
  if (do_bias) {
    __syncthreads();  // the last readers of LDS are done
    put_db<32, 8>(a, split, co0, tid, bsum, (float*)As);
  }
}

// ------------------------------------------------------- bwd-weight, 1x1x1
// dw[co][ci] += sum_v dy[v][co] * x[v][ci] and db[co] += sum_v dy[v][co]: a
// workgroup owns 32 output and 32 input channels and walks steps of 512
// voxels, both tiles brought into LDS by direct loads (64-byte cells, zeros
// past the channels); wave v multiplies voxels 64 v .. + 63, and the eight waves'
// sums meet in LDS.  Bound by HBM (the channels are read once per tile of the
// other side).  Measured on gfx950 at 8 x 128x64x64, 32->8, with the sum and the
// bias: 239 -> 78 us, against the general kernel, which transposes by hand, and a
// bias pass of its own (140 with the splits' values as atomics).
__global__ void __launch_bounds__(512) k_conv_wgrad_point(WArgs a) {
  constexpr unsigned OOB = 0x80000000u;
  __shared__ __attribute__((aligned(1024))) uint16_t As[512 * 32], Xs[512 * 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const Geo gx = a.gx, gy = a.gy;
  const int V = gy.n * gy.d * gy.h * gy.w;
  const int ntiles = a.nci * a.nco, split = blockIdx.x / ntiles, tile = blockIdx.x % ntiles;
  const int co0 = tile % a.nco * 32, ci0 = tile / a.nco * 32;
  const __amdgpu_buffer_rsrc_t rx = rsrc_of(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t rd = rsrc_of(a.dy, a.dy_bytes);
  const int q = (lane & 3) * 8;
  const bool aok = co0 + q < gy.c, xok = ci0 + q < gx.c;
  const int L = lane & 15, g = lane >> 4;
  int off[2];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) off[hh] = (wave * 64 + 8 * g + 4 * hh + (L >> 2)) * 32 + (L & 3) * 4;
  const bool do_bias = a.db != nullptr && ci0 == 0;
  const int s_begin = split * a.per_wg, s_end = s_begin + a.per_wg < a.steps ? s_begin + a.per_wg : a.steps;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  for (int st = s_begin; st < s_end; ++st) {
    __syncthreads();  // the previous step's readers are done
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int slot = i * 8 + wave, v = st * 512 + slot * 16 + (lane >> 2);
      lds_dma16(rd, As + slot * 512, aok && v < V ? (unsigned)(v * gy.ldc + co0 + q) * 2u : OOB, 0);
      lds_dma16(rx, Xs + slot * 512, xok && v < V ? (unsigned)(v * gx.ldc + ci0 + q) * 2u : OOB, 0);
    }
    load_barrier();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bf16x8 af[2], bx[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        af[i] = tr_load8(As, off[0] + c * 1024 + i * 16, off[1] + c * 1024 + i * 16);
        bx[i] = tr_load8(Xs, off[0] + c * 1024 + i * 16, off[1] + c * 1024 + i * 16);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bx[j], acc[i][j], 0, 0, 0);
    }
    if (do_bias) {
      float t = 0.f;
#pragma unroll 8
      for (int j = 0; j < 32; ++j) t += bf2f(As[(tid / 32 * 32 + j) * 32 + tid % 32]);
      bsum += t;
    }
  }
  float* T = (float*)Xs;  // [wave][32 co][32 ci]
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) T[(wave * 32 + i * 16 + g * 4 + k) * 32 + j * 16 + L] = acc[i][j][k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int e = k * 512 + tid, co = co0 + e / 32, ci = ci0 + e % 32;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) t += T[w * 1024 + e];
    if (co >= gy.c || ci >= gx.c) continue;
    float* const p = dw_of(a, split) + (unsigned)(co * a.kpad + ci);
    if (a.part)
      put<false>(p, t);
    else
      put<true>(p, t);
  }
  if (do_bias) put_db<32, 16>(a, split, co0, tid, bsum, (float*)As);  // (As is free since the sums met in Xs)
}

// dbias[co] += sum_v dy[v][co]: a thread sums 8 channels (one 16-byte load
// per voxel) over every (256 / groups)-th voxel of the workgroup's range; the
// partial sums meet in LDS and each channel takes one atomic per workgroup.
__global__ void __launch_bounds__(256) k_bias_grad(const uint16_t* __restrict__ dy, Geo gy, float* __restrict__ db,
                                                   float* __restrict__ part, long long vox_per_wg) {
  __shared__ float sums[256 * 8];
  const long long V = (long long)gy.n * gy.d * gy.h * gy.w;
  const long long vbeg = (long long)blockIdx.x * vox_per_wg;
  const long long vend = vbeg + vox_per_wg < V ? vbeg + vox_per_wg : V;
  const int groups = gy.c / 8;         // at most 256 (host check)
  const int vl = 256 / groups;         // voxel lanes
  const int tid = threadIdx.x, cg = tid % groups, vi = tid / groups;
  float s8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (vi < vl)
    for (long long v = vbeg + vi; v < vend; v += vl) {
      const u32x4 t = *(const u32x4*)(dy + v * gy.ldc + cg * 8);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s8[2 * j] += __uint_as_float(t[j] << 16);
        s8[2 * j + 1] += __uint_as_float(t[j] & 0xffff0000u);
      }
    }
#pragma unroll
  for (int j = 0; j < 8; ++j) sums[tid * 8 + j] = s8[j];
  __syncthreads();
  for (int c = tid; c < gy.c; c += 256) {
    const int g = c / 8, j = c % 8;
    float t = 0.f;
    for (int k = 0; k < vl; ++k) t += sums[(k * groups + g) * 8 + j];
    if (part)
      part[(long long)blockIdx.x * gy.c + c] = t;
    else
      atomicAdd(db + c, t);
  }
}

// dw[co][k] += the sum of its splits' parts, and db alike, in a fixed order
// and in FP64 (one rounding), so that a repeated gradient repeats bit for bit.
// Four neighbouring values per thread; where there are many splits the block's
// eight groups of 32 threads take every eighth part each and meet in LDS (few
// values and many parts would otherwise be one long chain of loads).  Bound by
// reading the parts once, from the memory-side cache for most layers.
struct WSum {
  const float *part, *part_b;
  float *dw, *db;
  int splits, splits_b;
  int cout, kpad, kuse;  // (the K padding of dw stays as it is)
};

template <int G>
__global__ void __launch_bounds__(256) k_wgrad_sum(WSum a) {
  constexpr int T = 256 / G;
  __shared__ double red[G > 1 ? G * T * 4 : 1];
  const int tid = threadIdx.x, g = tid / T;
  const long long nw = (long long)a.cout * a.kpad, q = ((long long)blockIdx.x * T + tid % T) * 4;
  const bool bias = q >= nw;
  const bool on = q < nw + (a.db ? a.cout : 0);
  const float* p = bias ? a.part_b + (q - nw) : a.part + q;
  const long long stride = bias ? a.cout : nw;
  const int n = !on ? 0 : (bias ? a.splits_b : a.splits);
  double t[4] = {0., 0., 0., 0.};
#pragma unroll 4
  for (int k = g; k < n; k += G) {
    const f32x4 v = *(const f32x4*)(p + k * stride);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] += (double)v[j];
  }
  if constexpr (G > 1) {
#pragma unroll
    for (int j = 0; j < 4; ++j) red[tid * 4 + j] = t[j];
    __syncthreads();
    if (g > 0) return;
#pragma unroll
    for (int k = 1; k < G; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) t[j] += red[(k * T + tid) * 4 + j];
  }
  if (!on) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (bias)
      a.db[q - nw + j] += (float)t[j];
    else if ((int)(q % a.kpad) + j < a.kuse)
      a.dw[q + j] += (float)t[j];
  }
}

// w_bf16[co][t*cin+ci] = w[co][t*cin+ci]; wt[ci][t*cout+co] = w[co][t*cin+ci]
__global__ void __launch_bounds__(256) k_weight_t(const float* __restrict__ w, int taps, int cin, int cout,
                                                  int kpad_f, int kpad_t, uint16_t* __restrict__ wb,
                                                  uint16_t* __restrict__ wt) {
  const long long nf = (long long)cout * kpad_f;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < nf; q += (long long)gridDim.x * blockDim.x) {
    const int co = (int)(q / kpad_f), k = (int)(q % kpad_f);
    wb[q] = f2bf(w[q]);
    if (k < taps * cin) {
      const int t = k / cin, ci = k % cin;
      wt[(long long)ci * kpad_t + (long long)t * cout + co] = f2bf(w[q]);
    }
  }
  // zero the K padding of wt
  const long long nt = (long long)cin * kpad_t;
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < nt; q += (long long)gridDim.x * blockDim.x)
    if ((int)(q % kpad_t) >= taps * cout) wt[q] = 0;
}

// Nearest-neighbour 2x upsampling and its adjoint.  A thread owns the 8
// channels (16 bytes) of one coarse voxel: one load and eight stores, or eight
// loads and one store; consecutive threads walk the channels, then w, so the
// two fine voxels of a pair along w are written (read) as whole lines.  One
// workgroup per 256 of a row's (w, channel group) pairs, rows by blockIdx.y
// (strided past the grid limit), so the row's coordinates are uniform.  Bound
// by HBM.  Measured on gfx950, batch 8, 64 channels to (from) 128x64x64, against
// one fine voxel's chunk (adjoint: one channel) per thread: upsampling 165 ->
// 109 us, adjoint 333 -> 112 us (5.4 TB/s).
__device__ __forceinline__ void coarse_row(const Geo& g, int row, int& n, int& d, int& h) {
  h = row % g.h;
  const int r = row / g.h;
  d = r % g.d;
  n = r / g.d;
}

__global__ void __launch_bounds__(256) k_up2(const uint16_t* __restrict__ x, Geo gx, uint16_t* __restrict__ y,
                                             Geo gy) {
  const int cv = gx.c / 8, q = blockIdx.x * 256 + threadIdx.x;
  if (q >= gx.w * cv) return;
  const int w = q / cv, c8 = (q - w * cv) * 8;
  const int rows = gx.n * gx.d * gx.h;
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    int n, d, h;
    coarse_row(gx, row, n, d, h);
    const u32x4 v = *(const u32x4*)(x + ((long long)row * gx.w + w) * gx.ldc + c8);
    uint16_t* o = y + vox(gy, n, 2 * d, 2 * h, 2 * w) * gy.ldc + c8;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      *(u32x4*)(o + (((long long)(j >> 2) * gy.h + ((j >> 1) & 1)) * gy.w + (j & 1)) * gy.ldc) = v;
  }
}

__global__ void __launch_bounds__(256) k_up2_bwd(const uint16_t* __restrict__ dy, Geo gy, uint16_t* __restrict__ dx,
                                                 Geo gx, int accumulate) {
  const int cv = gx.c / 8, q = blockIdx.x * 256 + threadIdx.x;
  if (q >= gx.w * cv) return;
  const int w = q / cv, c8 = (q - w * cv) * 8;
  const int rows = gx.n * gx.d * gx.h;
  for (int row = blockIdx.y; row < rows; row += gridDim.y) {
    int n, d, h;
    coarse_row(gx, row, n, d, h);
    const uint16_t* p = dy + vox(gy, n, 2 * d, 2 * h, 2 * w) * gy.ldc + c8;
    u32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = *(const u32x4*)(p + (((long long)(j >> 2) * gy.h + ((j >> 1) & 1)) * gy.w + (j & 1)) * gy.ldc);
    u32x4* o = (u32x4*)(dx + ((long long)row * gx.w + w) * gx.ldc + c8);
    u32x4 prev = u32x4{0u, 0u, 0u, 0u}, out;
    if (accumulate) prev = *o;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float lo = 0.f, hi = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        lo += __uint_as_float(v[j][k] << 16);
        hi += __uint_as_float(v[j][k] & 0xffff0000u);
      }
      if (accumulate) {
        lo += __uint_as_float(prev[k] << 16);
        hi += __uint_as_float(prev[k] & 0xffff0000u);
      }
      out[k] = (unsigned)f2bf(lo) | (unsigned)f2bf(hi) << 16;
    }
    *o = out;
  }
}

__global__ void __launch_bounds__(256) k_mse(const uint16_t* __restrict__ pred, Geo gp, const float* __restrict__ t,
                                             const uint8_t* __restrict__ wgt, int nch, float inv_count,
                                             uint16_t* __restrict__ dp, int dp_ldc, float* __restrict__ loss) {
  const long long V = (long long)gp.n * gp.d * gp.h * gp.w;
  float s = 0.f;
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
    const bool on = wgt == nullptr || wgt[v] != 0;
    for (int c = 0; c < gp.c; ++c) {
      float g = 0.f;
      if (on && c < nch) {
        const float d = bf2f(pred[v * gp.ldc + c]) - t[v * nch + c];
        s += d * d;
        g = 2.f * d * inv_count;
      }
      dp[v * dp_ldc + c] = f2bf(g);
    }
  }
  __shared__ float red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(loss, red[0] * inv_count);
}

__global__ void __launch_bounds__(256) k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, long long n, float lr, float b1, float b2,
                                              float eps, float c1, float c2) {
  for (long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (long long)gridDim.x * blockDim.x) {
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.f - b1) * gq;
    const float vq = b2 * v[q] + (1.f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    w[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
  }
}

__global__ void __launch_bounds__(256) k_sur_input(const uint8_t* __restrict__ solid, float gnorm, uint16_t* __restrict__ x,
                                                   Geo g) {
  const long long V = (long long)g.d * g.h * g.w;
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
    const int d = (int)(v / ((long long)g.h * g.w));
    const float zc = g.d > 1 ? 2.f * d / (g.d - 1) - 1.f : 0.f;
    uint16_t* o = x + v * g.ldc;
    o[0] = f2bf(solid[v] ? 1.f : 0.f);
    o[1] = f2bf(gnorm);
    o[2] = f2bf(1.f - zc * zc);
    for (int c = 3; c < g.c; ++c) o[c] = 0;
  }
}

__global__ void __launch_bounds__(256) k_sur_target(const double* __restrict__ rho, const double* __restrict__ u,
                                                    const uint8_t* __restrict__ solid, double rho0, double inv,
                                                    long long V, float* __restrict__ t, uint8_t* __restrict__ wgt) {
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
    const bool s = solid && solid[v];
    t[v * 4 + 0] = s ? 0.f : (float)(u[v] * inv);
    t[v * 4 + 1] = s ? 0.f : (float)(u[V + v] * inv);
    t[v * 4 + 2] = s ? 0.f : (float)(u[2 * V + v] * inv);
    t[v * 4 + 3] = s ? 0.f : (float)((rho[v] - rho0) * inv);
    wgt[v] = s ? 0 : 1;
  }
}

__global__ void __launch_bounds__(256) k_sur_fields(const uint16_t* __restrict__ p, Geo g, const uint8_t* __restrict__ solid,
                                                    double rho0, double mul, double* __restrict__ rho,
                                                    double* __restrict__ u) {
  const long long V = (long long)g.d * g.h * g.w;
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < V; v += (long long)gridDim.x * blockDim.x) {
    const bool s = solid && solid[v];
    const uint16_t* q = p + v * g.ldc;
    u[v] = s ? 0.0 : bf2f(q[0]) * mul;
    u[V + v] = s ? 0.0 : bf2f(q[1]) * mul;
    u[2 * V + v] = s ? 0.0 : bf2f(q[2]) * mul;
    rho[v] = s ? rho0 : rho0 + bf2f(q[3]) * mul;
  }
}

// --------------------------------------------------------------- helpers
Geo geo_of(const lbm_tensor5* t) { return Geo{t->n, t->d, t->h, t->w, t->c, t->ldc}; }

bool tensor_ok(const lbm_tensor5* t) {
  return t && t->ptr && t->n > 0 && t->d > 0 && t->h > 0 && t->w > 0 && t->c > 0 && (t->c % 8) == 0 &&
         (t->ldc % 8) == 0 && t->ldc >= t->c && (((uintptr_t)t->ptr) & 15) == 0;
}

constexpr long long kBiasVoxels = 2048;  // voxels of a workgroup of k_bias_grad

int outdim(int in, int stride) { return (in + stride - 1) / stride; }

// bytes spanned by a channels-last view (last voxel's last channel included)
long long view_bytes(const lbm_tensor5* t) {
  return (((long long)t->n * t->d * t->h * t->w - 1) * t->ldc + t->c) * 2;
}

// the tap-major kernels index in 32 bits and address through buffer resources
bool tap_fits(const lbm_tensor5* t) { return view_bytes(t) < (1ll << 31); }

template <int MODE, bool CLS, int FM, int FN>
void launch_tap(const DArgs& a, long long rows, int nz, hipStream_t s) {
  constexpr int BMW = 64 * FM, BN = 16 * FN;
  const dim3 g((unsigned)((rows + BMW - 1) / BMW), (unsigned)((a.go.c + BN - 1) / BN), (unsigned)nz);
  hipLaunchKernelGGL((k_conv_tap<MODE, CLS, FM, FN>), g, dim3(256), 0, s, a);
}

// tile shape by output columns: 32 -> 64 rows x 32 per wave, 64 -> 32 x 64,
// more -> 32 x 128 per column tile, or 32 x 64 where 128-column tiles would
// leave the chip short of workgroups (fewer than two per compute unit: the
// 16x8x8 layers of 256 channels)
template <int MODE, bool CLS>
void launch_tap_cols(const DArgs& a, long long rows, int nz, hipStream_t s) {
  const long long wide = (rows + 127) / 128 * ((a.go.c + 127) / 128) * nz;
  if (a.go.c <= 32)
    launch_tap<MODE, CLS, 4, 2>(a, rows, nz, s);
  else if (a.go.c <= 64 || wide < 512)
    launch_tap<MODE, CLS, 2, 4>(a, rows, nz, s);
  else
    launch_tap<MODE, CLS, 2, 8>(a, rows, nz, s);
}

// One shape of the plane kernel: its workgroups, and an estimate of its time in
// us: rounds of workgroups (as many per compute unit as LDS holds) times a
// round's measured time.
template <int MODE, int NC, int WF, int R, int WN>
struct PlaneTile {
  static constexpr int DP = 16 / WF;
  static constexpr int kLds = NC * ((DP * (4 * R + 2) * (WF + 2) * 4 + 63) / 64 * 1024 + 2 * 32 * WN * 64);
  static long long groups(const Geo& go) {
    return (long long)((go.w + WF - 1) / WF) * ((go.h + 4 * R - 1) / (4 * R)) * ((go.d + DP - 1) / DP) * go.n *
           ((go.c + 32 * WN - 1) / (32 * WN));
  }
  static double us(const Geo& go) {
    constexpr double small = NC == 8 ? 18.5 : (NC == 4 ? 16.0 : 12.0), mid = NC == 8 ? 23.3 : (NC == 4 ? 16.4 : 18.0),
                     big = NC == 8 ? 31.7 : (NC == 4 ? 28.0 : 18.0);
    const long long slots = 256 * (160 * 1024 / kLds);
    return (double)((groups(go) + slots - 1) / slots) * (R * WN == 1 ? small : (R * WN == 2 ? mid : big));
  }
  static void launch(const DArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((k_conv_plane<MODE, NC, WF, R, WN>), dim3((unsigned)groups(a.go)), dim3(256 * WN), 0, s, a);
  }
};

// The tap-major kernel's time alike: rounds of 512 workgroups, 0.75 us per K
// step of a 128 x 128 tile, half with 64 columns (launch_tap_cols).
double tap_us(const Geo& go, int ksize, int C) {
  const long long rows = ((long long)go.n * go.d * go.h * go.w + 127) / 128;
  const int steps = ksize * ksize * ksize * (C / 32);
  const long long wide = rows * ((go.c + 127) / 128);
  if (go.c > 64 && wide >= 512) return (double)((wide + 511) / 512) * 0.75 * steps;
  return (double)((rows * ((go.c + 63) / 64) + 511) / 512) * 0.37 * steps;
}

// The products that keep the tap-by-tap order of their sums (see pick_rows),
// for the channel counts the plane kernel holds in LDS: its fastest shape, or
// the tap-major kernel, whose result is the same, where that is the faster one
// (widths that fill the tiles badly: 42x37x19 at batch 4, 128->256, 312 against
// 366 us on plane tiles, its input gradient 335 against 468).
template <int NC>
int32_t pick_plane(const Geo& go) {
  const double cs = PlaneTile<0, NC, 8, 1, 1>::us(go), cm = PlaneTile<0, NC, 8, 2, 1>::us(go),
               cb = PlaneTile<0, NC, 16, 2, 2>::us(go);
  if (tap_us(go, 3, NC * 32) < std::min(cs, std::min(cm, cb))) return LBM_CONV_TAP;
  return cb < cm && cb < cs ? LBM_CONV_PLANE_BIG : (cm <= cs ? LBM_CONV_PLANE_MID : LBM_CONV_PLANE_SMALL);
}

template <int MODE, int NC>
void launch_plane(const DArgs& a, int32_t k, hipStream_t s) {
  if (k == LBM_CONV_PLANE_BIG)
    PlaneTile<MODE, NC, 16, 2, 2>::launch(a, s);
  else if (k == LBM_CONV_PLANE_MID)
    PlaneTile<MODE, NC, 8, 2, 1>::launch(a, s);
  else
    PlaneTile<MODE, NC, 8, 1, 1>::launch(a, s);
}

template <int NC, int R>
void launch_up_t(const DArgs& a, hipStream_t s) {
  const long long g = (long long)((a.gs.w + 15) / 16) * ((a.gs.h + 4 * R - 1) / (4 * R)) * a.gs.d * a.gs.n *
                      ((a.go.c + 31) / 32);
  hipLaunchKernelGGL((k_conv_up<NC, R>), dim3((unsigned)g), dim3(256), 0, s, a);
}

// Stride-2 input gradients of 32 or 64 channels, where the 16 x 8 tiles are at
// least half filled.  Below that the tap-major kernel's flat rows win (100x100x8
// 32 <- 64: 86 us against 64; 100x100x22, 0.6 filled: 90 against 172).  128
// channels take the LDS to one workgroup a CU: 80 us against 104 on 64x32x32
// 64 <- 128, but 621 against 549 on 40x40x64 256 <- 128.
bool up_fits(const Geo& gs) {
  const long long full = (long long)((gs.w + 15) / 16 * 16) * ((gs.h + 7) / 8 * 8);
  return (gs.c == 32 || gs.c == 64) && 2 * (long long)gs.w * gs.h >= full;
}

// 1x1x1 layers onto at most 32 channels, or with channels off 32s; onto more,
// the tap-major kernel's wider column tiles read the input fewer times (8 x
// 32x16x16 256->128: 25.9 against 28.2 us).
bool point_fits(int ksize, const Geo& src, const Geo& out) {
  return ksize == 1 && (out.c <= 32 || src.c % 32 != 0);
}

void launch_point(const DArgs& a, hipStream_t s) {
  const long long V = (long long)a.go.n * a.go.d * a.go.h * a.go.w;
  hipLaunchKernelGGL(k_conv_point, dim3((unsigned)((V + 255) / 256), (unsigned)((a.go.c + 31) / 32)), dim3(256), 0, s, a);
}

// Workgroups of the 8-channel forward, and of the row-tile kernel with R rows
// per wave.
long long c8_tiles(const Geo& go) {
  return (long long)((go.w + 15) / 16) * ((go.h + 15) / 16) * ((go.d + 3) / 4) * go.n * ((go.c + 31) / 32);
}

template <int R>
long long row_tiles(const Geo& go) {
  return (long long)((go.w + 15) / 16) * ((go.h + 4 * R - 1) / (4 * R)) * go.d * go.n * ((go.c + 31) / 32);
}

// Stride-1 3x3x3 products: 16 x 16 tiles, or 8 x 16 where the larger ones
// would leave compute units without a workgroup (batch 1, 32x16x16 128->128:
// 18.6 -> 16.7 us on 128 tiles) or pad the rows enough to lose what the
// smaller ones lose in operand reuse (1180 against 1000 TFLOP/s at 64x32x32
// 64->64).  Where even the small tiles are less than a quarter filled, and those
// of the 8-channel forward less than an eighth, the volume goes to the kernels
// that take voxels in any shape: the tap-major one, or, with channels off 32s,
// the general one (1 x 65536x1x1 40->48 forward 40 us there against 1150 on row
// tiles, 1 x 4096x4x4, an eighth filled, 48 against 85, 1 x 682x4x24, three
// eighths, 48 against 36; 8->32 forward at a sixteenth 13.7 against 17.5, at
// 3/16 14.0 against 13.0).  Products of 64, 128 or 256 channels off rows of whole
// 32s or onto more than 64 channels go to the plane kernel, whose sums run tap
// by tap over all chunks.  That line is one of rounding, not of speed: it is
// where a layer's sums have always changed their order, and results rounded
// otherwise would flip ReLU masks all through a trained network's passes (row
// tiles would take the input gradient of 32x16x16 256->128 at batch 8 from 116 to
// about 91 us).  So the order depends on whether the width is a multiple of 32.
template <int MODE>
int32_t pick_rows(const Geo& gs, const Geo& go) {
  const long long big = row_tiles<4>(go), small = row_tiles<2>(go);
  const long long vox = (long long)go.n * go.d * go.h * go.w, nct = (go.c + 31) / 32;
  const int C = gs.c;
  if (MODE == 0 && C == 8) return c8_tiles(go) * 1024 > 8 * vox * nct ? LBM_CONV_GENERAL : LBM_CONV_C8;
  if (go.w % 32 != 0 || go.c > 64) {
    if (C == 64) return pick_plane<2>(go);
    if (C == 128) return pick_plane<4>(go);
    if (C == 256) return pick_plane<8>(go);
  }
  if (small * 128 > 4 * vox * nct) return C % 32 == 0 ? LBM_CONV_TAP : LBM_CONV_GENERAL;
  return big >= 256 && big * 2 <= small * 1.22 ? LBM_CONV_ROWS4 : LBM_CONV_ROWS2;
}

// The kernel of a forward (MODE 0: gs = x, go = y) or input-gradient (gs = dy,
// go = dx) product.
template <int MODE>
int32_t pick_conv(const Geo& gs, const Geo& go, int ksize, int stride, bool fits) {
  if (!fits) return LBM_CONV_GENERAL;
  if (point_fits(ksize, gs, go)) return LBM_CONV_POINT;
  if (ksize == 3 && stride == 1) return pick_rows<MODE>(gs, go);
  if (gs.c % 32 != 0) return LBM_CONV_GENERAL;
  return MODE == 1 && stride == 2 && up_fits(gs) ? LBM_CONV_UP : LBM_CONV_TAP;
}

template <int MODE, int BN>
void launch_gemm(const DArgs& a, hipStream_t s) {
  const long long M = (long long)a.go.n * a.go.d * a.go.h * a.go.w;
  const dim3 g((unsigned)((M + BM - 1) / BM), (a.go.c + BN - 1) / BN);
  hipLaunchKernelGGL((k_conv_gemm<MODE, BN>), g, dim3(256), 0, s, a.src, a.gs, a.wk, a.kstride, a.bias, a.out, a.go,
                     a.act, a.act_ldc, a.ksize, a.stride, a.relu, a.accumulate, a.C);
}

template <int MODE>
void launch_conv(const DArgs& a, int32_t k, hipStream_t s) {
  const long long M = (long long)a.go.n * a.go.d * a.go.h * a.go.w;
  const bool tail = a.C % 32 != 0;
  const dim3 b(256);
  switch (k) {
    case LBM_CONV_GENERAL:
      if (a.go.c <= 16)
        launch_gemm<MODE, 16>(a, s);
      else if (a.go.c <= 32)
        launch_gemm<MODE, 32>(a, s);
      else
        launch_gemm<MODE, 64>(a, s);
      break;
    case LBM_CONV_POINT: launch_point(a, s); break;
    case LBM_CONV_C8:
      if constexpr (MODE == 0) hipLaunchKernelGGL(k_conv_fwd_c8, dim3((unsigned)c8_tiles(a.go)), b, 0, s, a);
      break;
    case LBM_CONV_ROWS2:
    case LBM_CONV_ROWS4: {
      const bool four = k == LBM_CONV_ROWS4;
      const dim3 g((unsigned)(four ? row_tiles<4>(a.go) : row_tiles<2>(a.go)));
      if (four && tail)
        hipLaunchKernelGGL((k_conv_rows<MODE, 4, true>), g, b, 0, s, a);
      else if (four)
        hipLaunchKernelGGL((k_conv_rows<MODE, 4, false>), g, b, 0, s, a);
      else if (tail)
        hipLaunchKernelGGL((k_conv_rows<MODE, 2, true>), g, b, 0, s, a);
      else
        hipLaunchKernelGGL((k_conv_rows<MODE, 2, false>), g, b, 0, s, a);
      break;
    }
    case LBM_CONV_PLANE_SMALL:
    case LBM_CONV_PLANE_MID:
    case LBM_CONV_PLANE_BIG:
      if (a.C == 64)
        launch_plane<MODE, 2>(a, k, s);
      else if (a.C == 128)
        launch_plane<MODE, 4>(a, k, s);
      else
        launch_plane<MODE, 8>(a, k, s);
      break;
    case LBM_CONV_UP:
      if constexpr (MODE == 1) {
        if (a.C == 32)
          launch_up_t<1, 2>(a, s);
        else
          launch_up_t<2, 2>(a, s);
      }
      break;
    default:
      if (MODE == 1 && a.stride == 2) {
        // rows of the largest parity class; smaller classes mask their tail
        const long long rows = (long long)a.go.n * ((a.go.d + 1) / 2) * ((a.go.h + 1) / 2) * ((a.go.w + 1) / 2);
        launch_tap_cols<MODE, MODE == 1>(a, rows, 8, s);
      } else {
        launch_tap_cols<MODE, false>(a, M, 1, s);
      }
  }
}

// Whether the kernels that index in 32 bits take the call.  A 1x1x1 layer in
// place, onto 33 to 64 channels off 32s, stays with the general kernel, which
// has them all in one workgroup: the pointwise kernel's second column tile
// would read what the first has written.
bool conv_fits(const lbm_tensor5* src, const lbm_tensor5* out, int ksize) {
  const int kpad = lbm_conv_kpad(ksize * ksize * ksize, src->c);
  const bool in_place = ksize == 1 && src->ptr == out->ptr && out->c > 32 && src->c % 32 != 0;
  return !in_place && tap_fits(src) && tap_fits(out) && (long long)out->c * kpad < (1ll << 30);
}

// How a weight gradient runs: its kernel and tile, its steps (kGeneral: voxels),
// how many of them a workgroup takes, and the workgroups that so share a tile.
struct WPlan {
  enum Kind { kRows, kC8, kPoint, kGeneral } kind = kGeneral;
  int bm = 0, wp = 0;        // kRows: output channels of a tile, voxels of a row along w (kC8 too)
  int nhb = 0, nwb = 0, nco = 0, nci = 0;
  long long steps = 0, tiles = 0, per_wg = 0;
  long long splits = 0, splits_b = 0;  // (of the bias gradient)
  long long floats(const Geo& gy, int kpad) const { return (splits * kpad + splits_b) * gy.c; }
};

// Voxels of a 32-voxel row along w: what pads the volume least, the longest of
// equals.  Rows under 8 long, whose halo has up to three cells a voxel, only
// where they save a third (64->64, 1 x 1024x64x1 34 us, 118 on rows of 8; 1 x
// 4096x4x4 31 against 42).
int row_voxels(const Geo& g, int shortest) {
  int best = 32;
  long long least = -1;
  for (int wp = 32; wp >= shortest; wp /= 2) {
    const int dp = 32 / wp;
    const long long p = (long long)((g.w + wp - 1) / wp) * wp * ((g.d + dp - 1) / dp) * dp;
    if (least < 0 || (wp < 8 ? 3 * p < 2 * least : p < least)) least = p, best = wp;
  }
  return best;
}

// Workgroups that share one tile of a weight gradient.  N of them cost a step's
// time (us) times steps / N plus N times the end of each, and N is where the two
// are equal, as long as one round (`slots` workgroups) holds them:
//  * with a workspace (parts) the end is a store of the tile's values and their
//    later sum, 8 bytes a value at about 4 TB/s;
//  * without, one atomic per value: the memory side takes the atomics of one
//    address one after the other, about 0.16 us each, and about 95 G/s in all.
//    (A 1x1x1 layer, 256 addresses, 85 us with 512 workgroups, 44 with 80; batch
//    1 128x64x64 32->32 129 us with 342, 76 with 90.)
// A sum of n products one after the other is off by about sqrt(n / 2) * 2^-24, so
// N also keeps the chains short (per_step products a step; V voxels, 32 a
// product): with parts, which are added in FP64, to 44 + V / 3200 products, as far
// as the parts stay under 128 MB, which the memory-side cache holds (4 x 42x37x19
// 128->256 269 us with 233 MB of them); with atomics, which go on in FP32, chain and
// adds together to 48 + V / 1536.
void wgrad_splits(WPlan& p, long long V, int per_step, long long values, long long slots, double step_us, bool parts) {
  const long long v32 = (V + 31) / 32, sum = p.steps * per_step;
  const double each = (double)(p.tiles * values) * (parts ? 2e-6 : 1.0 / 95000.0) + (parts ? 0.0 : 0.16);
  long long n = (long long)std::sqrt(step_us * (double)p.steps / each);
  n = std::max<long long>(1, std::min(slots / p.tiles, n));
  if (parts)
    n = std::max(n, std::min(v32 / (44 + v32 / 100), (32ll << 20) / (p.tiles * values)));
  else if (sum / n + n > 48 + v32 / 48)
    n = std::max(n, std::min(v32 / 48, 2048 / p.tiles));
  n = std::min(n, p.steps);
  p.per_wg = (p.steps + n - 1) / n;
  p.splits = p.splits_b = (p.steps + p.per_wg - 1) / p.per_wg;
}

template <int S, int BM, int WP>
void launch_wgrad_rows_t(const WArgs& a, unsigned grid, hipStream_t s) {
  hipLaunchKernelGGL((k_conv_wgrad_rows<S, BM, WP>), dim3(grid), dim3(256), 0, s, a);
}

template <int S, int BM>
void launch_wgrad_rows(const WArgs& a, int wp, unsigned grid, hipStream_t s) {
  switch (wp) {
    case 32: launch_wgrad_rows_t<S, BM, 32>(a, grid, s); break;
    case 16: launch_wgrad_rows_t<S, BM, 16>(a, grid, s); break;
    case 8: launch_wgrad_rows_t<S, BM, 8>(a, grid, s); break;
    case 4: launch_wgrad_rows_t<S, BM, 4>(a, grid, s); break;
    case 2: launch_wgrad_rows_t<S, BM, 2>(a, grid, s); break;
    default: launch_wgrad_rows_t<S, BM, 1>(a, grid, s); break;
  }
}

WPlan wgrad_plan(const lbm_tensor5* x, const lbm_tensor5* dy, int ksize, int stride, bool parts) {
  const Geo gx = geo_of(x), gy = geo_of(dy);
  const long long V = (long long)gy.n * gy.d * gy.h * gy.w;
  WPlan p;
  // (1x1x1: the general kernel's wider tiles read the channels of large layers
  // fewer times: 6 x 107x68x49 64->64 232 against 369 us; 8 x 32x16x16 256->128
  // 114 against 56)
  const long long tiles1 = (long long)((gx.c + 31) / 32) * ((gy.c + 31) / 32);
  const bool wide1 = ksize == 1 && tiles1 >= 4 && V * tiles1 > 3000000;
  // (a handful of stride-2 steps on channels off 32s: 6 x 4x13x6 24->64 8 us on
  // the general kernel against 12)
  const bool tiny = stride == 2 && gx.c % 32 != 0 && V < 4096;
  const int kpad = lbm_conv_kpad(ksize * ksize * ksize, gx.c);
  const long long gtiles = (long long)((gy.c + BM - 1) / BM) * ((kpad + 63) / 64);
  if (ksize == 3) {
    const bool c8 = stride == 1 && gx.c == 8;
    p.kind = c8 ? WPlan::kC8 : WPlan::kRows;
    // 32-channel output tiles where 64 would be half empty
    p.bm = c8 || (gy.c % 64 > 0 && gy.c % 64 <= 32) ? 32 : 64;
    p.wp = row_voxels(gy, c8 ? 8 : 1);
    const int rr = c8 || (stride == 1 && p.bm == 32) ? 8 : 4, dp = 32 / p.wp;
    p.nhb = (gy.h + rr - 1) / rr;
    p.nwb = (gy.w + p.wp - 1) / p.wp;
    p.steps = (long long)gy.n * ((gy.d + dp - 1) / dp) * p.nhb * p.nwb;
    p.nco = (gy.c + p.bm - 1) / p.bm;
    p.nci = c8 ? 1 : (gx.c + 31) / 32;
    p.tiles = (c8 ? 1ll : 3ll) * p.nci * p.nco;
  }
  // Volumes so narrow that the steps are mostly padding: the general kernel takes
  // its voxels in any shape, at 2.1 ns per chunk of 32 and tile, against 4.3 ns
  // per step and tile of 64 channels, 5.4 of 32 (12 on rows of one or two), 8 of
  // the 8-channel layer (1 x 65536x1x1 24->32 60 us against 80, 8->32 54 against 159;
  // 1 x 16384x2x2 24->32 61 against 50, 4096x4x4 8->32 about 55 against 32).
  const double step_ns = p.kind == WPlan::kC8 ? 8.0 : (p.bm == 64 ? 4.3 : (p.wp > 2 ? 5.4 : 12.0));
  const bool narrow =
      ksize == 3 && 2.1 * (double)((V + 31) / 32) * (double)gtiles < step_ns * (double)(p.steps * p.tiles);
  const bool fits = tap_fits(x) && tap_fits(dy) && V < (1ll << 31) && (long long)gy.c * kpad < (1ll << 30);
  if (!fits || narrow || wide1 || tiny) {
    p = WPlan{};
    p.kind = WPlan::kGeneral;
    p.nco = (gy.c + BM - 1) / BM;
    p.nci = (kpad + 63) / 64;
    p.tiles = (long long)p.nco * p.nci;
    // split the voxel range so that the grid holds about 2048 workgroups, 1024
    // where their sums are stored and read again
    const long long n = std::max<long long>(1, (parts ? 1024 : 2048) / p.tiles);
    p.per_wg = ((V + n - 1) / n + BK - 1) / BK * BK;
    p.splits = (V + p.per_wg - 1) / p.per_wg;
    p.splits_b = (V + kBiasVoxels - 1) / kBiasVoxels;
    return p;
  }
  if (ksize == 1) {
    p.kind = WPlan::kPoint;
    p.steps = (V + 511) / 512;  // steps of 512 voxels
    p.nco = (gy.c + 31) / 32;
    p.nci = (gx.c + 31) / 32;
    p.tiles = (long long)p.nco * p.nci;
    wgrad_splits(p, V, 2, 1024, 512, 1.0, parts);
    return p;
  }
  if (p.kind == WPlan::kC8)
    wgrad_splits(p, V, 8, 32 * 216, 512, 2.5, parts);
  else
    wgrad_splits(p, V, stride == 2 && p.bm == 32 ? 2 : 4, p.bm * 288, 768, 3.0, parts);
  return p;
}

// Floats of workspace that make the sums independent of the workgroups' order
// (none where every value has one workgroup anyway).
long long wgrad_floats(const WPlan& p, const Geo& gy, int kpad) {
  return p.splits > 1 || p.splits_b > 1 ? p.floats(gy, kpad) : 0;
}

void launch_wgrad(const WPlan& p, const lbm_tensor5* x, const lbm_tensor5* dy, float* dw, float* db, int ksize,
                  int stride, float* part, hipStream_t s) {
  WArgs a{};
  a.x = (const uint16_t*)x->ptr;
  a.gx = geo_of(x);
  a.dy = (const uint16_t*)dy->ptr;
  a.gy = geo_of(dy);
  a.dw = dw;
  a.db = db;
  a.kpad = lbm_conv_kpad(ksize * ksize * ksize, x->c);
  a.part = part;
  a.part_b = part && db ? part + p.splits * a.kpad * a.gy.c : nullptr;
  if (p.kind == WPlan::kGeneral) {
    const dim3 g(p.nco, p.nci, (unsigned)p.splits);
    hipLaunchKernelGGL(k_conv_wgrad, g, dim3(256), 0, s, a.x, a.gx, a.dy, a.gy, dw, part, a.kpad, x->c, ksize, stride,
                       p.per_wg);
    if (db)
      hipLaunchKernelGGL(k_bias_grad, dim3((unsigned)p.splits_b), dim3(256), 0, s, a.dy, a.gy, db, a.part_b,
                         kBiasVoxels);
  } else {
    a.x_bytes = (unsigned)view_bytes(x);
    a.dy_bytes = (unsigned)view_bytes(dy);
    a.nhb = p.nhb;
    a.nwb = p.nwb;
    a.nco = p.nco;
    a.nci = p.nci;
    a.steps = (int)p.steps;
    a.per_wg = (int)p.per_wg;
    const unsigned grid = (unsigned)(p.splits * p.tiles);
    if (p.kind == WPlan::kPoint)
      hipLaunchKernelGGL(k_conv_wgrad_point, dim3(grid), dim3(512), 0, s, a);
    else if (p.kind == WPlan::kC8 && p.wp == 32)
      hipLaunchKernelGGL(k_conv_wgrad_c8<32>, dim3(grid), dim3(256), 0, s, a);
    else if (p.kind == WPlan::kC8 && p.wp == 16)
      hipLaunchKernelGGL(k_conv_wgrad_c8<16>, dim3(grid), dim3(256), 0, s, a);
    else if (p.kind == WPlan::kC8)
      hipLaunchKernelGGL(k_conv_wgrad_c8<8>, dim3(grid), dim3(256), 0, s, a);
    else if (stride == 2 && p.bm == 32)
      launch_wgrad_rows<2, 32>(a, p.wp, grid, s);
    else if (stride == 2)
      launch_wgrad_rows<2, 64>(a, p.wp, grid, s);
    else if (p.bm == 32)
      launch_wgrad_rows<1, 32>(a, p.wp, grid, s);
    else
      launch_wgrad_rows<1, 64>(a, p.wp, grid, s);
  }
  if (!part) return;
  const WSum w{part, a.part_b, dw, db, (int)p.splits, (int)p.splits_b, a.gy.c, a.kpad, ksize * ksize * ksize * x->c};
  const long long q = ((long long)a.gy.c * a.kpad + a.gy.c) / 4;  // values in fours
  // (sixteen parts or more: eight groups a block, see the kernel)
  if (std::max(p.splits, p.splits_b) >= 16)
    hipLaunchKernelGGL(k_wgrad_sum<8>, dim3((unsigned)((q + 31) / 32)), dim3(256), 0, s, w);
  else
    hipLaunchKernelGGL(k_wgrad_sum<1>, dim3((unsigned)((q + 255) / 256)), dim3(256), 0, s, w);
}

// Rows (n, d, h) by y, (w, channel group) pairs by x.
dim3 grid_rows(const lbm_tensor5* t) {
  const long long rows = (long long)t->n * t->d * t->h;
  return dim3((unsigned)(((long long)t->w * (t->c / 8) + 255) / 256), (unsigned)std::min<long long>(rows, 65535));
}

int grid1(long long n) {
  long long g = (n + 255) / 256;
  if (g > 65536) g = 65536;
  return (int)(g < 1 ? 1 : g);
}

}  // namespace

extern "C" {

int32_t lbm_conv_kpad(int32_t taps, int32_t cin) { return ((taps * cin + 31) / 32) * 32; }

// Shapes of a convolution from x to y.
static bool conv_ok(const lbm_tensor5* x, const lbm_tensor5* y, int32_t ksize, int32_t stride) {
  if (!tensor_ok(x) || !tensor_ok(y) || (ksize != 1 && ksize != 3) || (stride != 1 && stride != 2) ||
      (ksize == 1 && stride != 1))
    return false;
  return y->n == x->n && y->d == outdim(x->d, stride) && y->h == outdim(x->h, stride) && y->w == outdim(x->w, stride);
}

lbm_status lbm_conv3d_fwd(const lbm_tensor5* x, const uint16_t* w, const float* bias, const lbm_tensor5* y,
                          int32_t ksize, int32_t stride, int32_t relu, void* stream) {
  if (!conv_ok(x, y, ksize, stride) || !w) return LBM_EINVAL;
  const int kpad = lbm_conv_kpad(ksize * ksize * ksize, x->c);
  const DArgs a{(const uint16_t*)x->ptr, geo_of(x), (unsigned)view_bytes(x), w, kpad,
                (unsigned)((long long)y->c * kpad * 2), bias, (uint16_t*)y->ptr, geo_of(y), nullptr, 0, ksize, stride,
                relu, 0, x->c};
  launch_conv<0>(a, pick_conv<0>(a.gs, a.go, ksize, stride, conv_fits(x, y, ksize)), (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_conv3d_bwd_data(const lbm_tensor5* dy, const uint16_t* w_t, const lbm_tensor5* dx,
                               const lbm_tensor5* act, int32_t ksize, int32_t stride, int32_t accumulate,
                               void* stream) {
  if (!conv_ok(dx, dy, ksize, stride) || !w_t) return LBM_EINVAL;
  if (act && (!tensor_ok(act) || act->n != dx->n || act->d != dx->d || act->h != dx->h || act->w != dx->w ||
              act->c < dx->c))
    return LBM_EINVAL;
  const int kpad = lbm_conv_kpad(ksize * ksize * ksize, dy->c);
  const DArgs a{(const uint16_t*)dy->ptr, geo_of(dy), (unsigned)view_bytes(dy), w_t, kpad,
                (unsigned)((long long)dx->c * kpad * 2), nullptr, (uint16_t*)dx->ptr, geo_of(dx),
                act ? (const uint16_t*)act->ptr : nullptr, act ? act->ldc : 0, ksize, stride, 0, accumulate, dy->c};
  launch_conv<1>(a, pick_conv<1>(a.gs, a.go, ksize, stride, conv_fits(dy, dx, ksize)), (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

int32_t lbm_conv3d_kernel(int32_t pass, const lbm_tensor5* x, const lbm_tensor5* y, int32_t ksize, int32_t stride) {
  if (!conv_ok(x, y, ksize, stride) || pass < 0 || pass > 2) return -1;
  if (pass == 0)
    return pick_conv<0>(geo_of(x), geo_of(y), ksize, stride, conv_fits(x, y, ksize));
  if (pass == 1)
    return pick_conv<1>(geo_of(y), geo_of(x), ksize, stride, conv_fits(y, x, ksize));
  const WPlan p = wgrad_plan(x, y, ksize, stride, true);
  switch (p.kind) {
    case WPlan::kRows: return p.bm == 32 ? LBM_WGRAD_ROWS32 : LBM_WGRAD_ROWS64;
    case WPlan::kC8: return LBM_WGRAD_C8;
    case WPlan::kPoint: return LBM_WGRAD_POINT;
    default: return LBM_WGRAD_GENERAL;
  }
}

lbm_status lbm_conv3d_bwd_weight(const lbm_tensor5* x, const lbm_tensor5* dy, float* dw, float* dbias,
                                 int32_t ksize, int32_t stride, void* stream) {
  if (!conv_ok(x, dy, ksize, stride) || !dw || (dbias && dy->c > 2048)) return LBM_EINVAL;
  launch_wgrad(wgrad_plan(x, dy, ksize, stride, false), x, dy, dw, dbias, ksize, stride, nullptr,
               (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

int64_t lbm_conv3d_bwd_weight_scratch(const lbm_tensor5* x, const lbm_tensor5* dy, int32_t ksize, int32_t stride) {
  if (!conv_ok(x, dy, ksize, stride)) return -1;
  return 4 * wgrad_floats(wgrad_plan(x, dy, ksize, stride, true), geo_of(dy),
                          lbm_conv_kpad(ksize * ksize * ksize, x->c));
}

lbm_status lbm_conv3d_bwd_weight_ordered(const lbm_tensor5* x, const lbm_tensor5* dy, float* dw, float* dbias,
                                         int32_t ksize, int32_t stride, void* scratch, int64_t scratch_bytes,
                                         void* stream) {
  if (!conv_ok(x, dy, ksize, stride) || !dw || (dbias && dy->c > 2048)) return LBM_EINVAL;
  const WPlan p = wgrad_plan(x, dy, ksize, stride, true);
  const int64_t need = 4 * wgrad_floats(p, geo_of(dy), lbm_conv_kpad(ksize * ksize * ksize, x->c));
  if (need > 0 && (!scratch || scratch_bytes < need || ((uintptr_t)scratch & 15))) return LBM_EINVAL;
  launch_wgrad(p, x, dy, dw, dbias, ksize, stride, need > 0 ? (float*)scratch : nullptr, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_conv3d_weight_t(const float* w_master, int32_t taps, int32_t cin, int32_t cout, uint16_t* w_bf16,
                               uint16_t* wt_bf16, void* stream) {
  if (!w_master || !w_bf16 || !wt_bf16 || (taps != 1 && taps != 27) || cin <= 0 || cout <= 0 || (cin % 8) ||
      (cout % 8))
    return LBM_EINVAL;
  const int kf = lbm_conv_kpad(taps, cin), kt = lbm_conv_kpad(taps, cout);
  const long long n = (long long)cout * kf > (long long)cin * kt ? (long long)cout * kf : (long long)cin * kt;
  hipLaunchKernelGGL(k_weight_t, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, w_master, taps, cin, cout, kf,
                     kt, w_bf16, wt_bf16);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_upsample2(const lbm_tensor5* x, const lbm_tensor5* y, void* stream) {
  if (!tensor_ok(x) || !tensor_ok(y) || y->n != x->n || y->c != x->c || y->d != 2 * x->d || y->h != 2 * x->h ||
      y->w != 2 * x->w)
    return LBM_EINVAL;
  hipLaunchKernelGGL(k_up2, grid_rows(x), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)x->ptr, geo_of(x),
                     (uint16_t*)y->ptr, geo_of(y));
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_upsample2_bwd(const lbm_tensor5* dy, const lbm_tensor5* dx, int32_t accumulate, void* stream) {
  if (!tensor_ok(dy) || !tensor_ok(dx) || dy->n != dx->n || dy->c != dx->c || dy->d != 2 * dx->d ||
      dy->h != 2 * dx->h || dy->w != 2 * dx->w)
    return LBM_EINVAL;
  hipLaunchKernelGGL(k_up2_bwd, grid_rows(dx), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)dy->ptr,
                     geo_of(dy), (uint16_t*)dx->ptr, geo_of(dx), accumulate);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_mse_loss(const lbm_tensor5* pred, const float* target, const uint8_t* weight, int32_t nch,
                        float inv_count, const lbm_tensor5* dpred, float* loss, void* stream) {
  if (!tensor_ok(pred) || !tensor_ok(dpred) || !target || !loss || nch <= 0 || nch > pred->c ||
      dpred->c != pred->c || dpred->n != pred->n || dpred->d != pred->d || dpred->h != pred->h || dpred->w != pred->w)
    return LBM_EINVAL;
  const long long V = (long long)pred->n * pred->d * pred->h * pred->w;
  int g = grid1(V);
  if (g > 2048) g = 2048;
  hipLaunchKernelGGL(k_mse, dim3(g), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)pred->ptr, geo_of(pred),
                     target, weight, nch, inv_count, (uint16_t*)dpred->ptr, dpred->ldc, loss);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_adam_step(float* w, const float* g, float* m, float* v, int64_t n, float lr, float beta1, float beta2,
                         float eps, int32_t t, void* stream) {
  if (!w || !g || !m || !v || n <= 0 || t < 1) return LBM_EINVAL;
  const float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3(grid1(n)), dim3(256), 0, (hipStream_t)stream, w, g, m, v, (long long)n, lr, beta1,
                     beta2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_surrogate_input(const uint8_t* solid, double gx, const lbm_tensor5* x, void* stream) {
  if (!solid || !tensor_ok(x) || x->c < 8 || x->n != 1 || !(gx > 0)) return LBM_EINVAL;
  const float gnorm = (float)((log10(gx) + 5.8) / 0.5);
  const long long V = (long long)x->d * x->h * x->w;
  hipLaunchKernelGGL(k_sur_input, dim3(grid1(V)), dim3(256), 0, (hipStream_t)stream, solid, gnorm,
                     (uint16_t*)x->ptr, geo_of(x));
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_surrogate_target(const double* rho, const double* u, const uint8_t* solid, double rho0, double gx,
                                double scale, int64_t voxels, float* target, uint8_t* weight, void* stream) {
  if (!rho || !u || !target || !weight || voxels <= 0 || !(gx > 0) || !(scale > 0)) return LBM_EINVAL;
  hipLaunchKernelGGL(k_sur_target, dim3(grid1(voxels)), dim3(256), 0, (hipStream_t)stream, rho, u, solid, rho0,
                     1.0 / (gx * scale), (long long)voxels, target, weight);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

lbm_status lbm_surrogate_fields(const lbm_tensor5* pred, const uint8_t* solid, double rho0, double gx, double scale,
                                double* rho, double* u, void* stream) {
  if (!tensor_ok(pred) || pred->n != 1 || !rho || !u || !(gx > 0) || !(scale > 0)) return LBM_EINVAL;
  const long long V = (long long)pred->d * pred->h * pred->w;
  hipLaunchKernelGGL(k_sur_fields, dim3(grid1(V)), dim3(256), 0, (hipStream_t)stream, (const uint16_t*)pred->ptr,
                     geo_of(pred), solid, rho0, gx * scale, rho, u);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

}  // extern "C"
