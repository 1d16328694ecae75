// Fusion network of the hybrid method on gfx950: every convolution is an
// implicit GEMM on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation; the residual stream stays FP32; weights keep FP32 masters and
// BF16 packed copies.
//
// Architecture (paper Sec. 4; trunk of 16 residual blocks):
//   h0  = ReLU(conv3x3 10->64 (HRLS rgb + albedo + normal + depth))   @HR
//   fl  = ReLU(conv3x3 3->64  (LRHS rgb))                              @LR
//   F0  = ReLU(conv1x1 [fl, unshuffle4(h0)] 1088->64)                 @LR
//   r   <- r + 0.1 conv3x3(ReLU(conv3x3(r))), 16 times, r_0 = F0      @LR
//   FDF = r_16 + F0
//   U   = ReLU(conv3x3 64->256 (FDF))                                  @LR
//   out = conv3x3 [shuffle4(U), h0] 80->3                              @HR
// The (un)shuffles are never materialised: they are folded into the input
// addressing of the convs that read them.  Channel conventions: unshuffle by r
// puts HR pixel (rY+i, rX+j) channel c at LR channel (i r + j) C + c; shuffle
// is its inverse.
//
// GEMM mapping: M = output pixels (NHWC raster order), N = output channels,
// K = taps x padded input channels.  A wave computes 32 pixels x (16 NT)
// channels: 2 x NT accumulator tiles of 16x16.  Per 32-wide K step, lane l
// loads the 8 consecutive input channels (one 16-byte load) of pixel l%16 of
// each row tile for K chunk l/16, and the matching 8 weights of output channel
// l%16 of each column tile.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "mrs_internal.hpp"
#include "devmath.hpp"
#include "cnn.hpp"

namespace mrs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Round to nearest even, NaN stays NaN (v_cvt_pk_bf16_f32): one value, and two
// in one word (a low).
__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ bf16x8 zero8() {
  uint4 z = make_uint4(0u, 0u, 0u, 0u);
  return __builtin_bit_cast(bf16x8, z);
}

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

// Offset (I, J) inside its r x r block of the HR pixel held by unshuffle slot
// q.  One stride-r unshuffle (dsf = 0): q = I r + J.  dsf stacked stride-2
// deshuffles (r = 2^dsf), the first consuming the low bits: base-4 digit k of
// q is 2 (bit k of I) + (bit k of J).
__device__ __forceinline__ void unshuffle_slot(int q, int r, int dsf, int& I, int& J) {
  if (dsf) {
    I = J = 0;
    for (int k = 0; k < dsf; ++k) {
      J |= ((q >> (2 * k)) & 1) << k;
      I |= ((q >> (2 * k + 1)) & 1) << k;
    }
  } else {
    I = q / r;
    J = q - I * r;
  }
}

// Address of channel c of the conv input at pixel (b, y, x) through the view
// (nullptr outside the image); channels c .. c+7 are contiguous there when c is
// a multiple of 8.
__device__ __forceinline__ const uint16_t* view_ptr(const ConvArgs& p, int b, int y, int x,
                                                    int c) {
  if (y < 0 || y >= p.H || x < 0 || x >= p.W) return nullptr;
  switch (p.mode) {
    case VIEW_PLAIN:
      return p.a + ((size_t)(b * p.H + y) * p.W + x) * p.ca + c;
    case VIEW_CONCAT_UNSHUFFLE:  // [a (LR, ca ch), unshuffle_r(b (HR, cb ch))]
      if (c < p.ca) {
        return p.a + ((size_t)(b * p.H + y) * p.W + x) * p.ca + c;
      } else {
        const int cc = c - p.ca;
        const int qq = cc / p.cb, ch = cc - qq * p.cb;
        int I, J;
        unshuffle_slot(qq, p.r, p.dsf, I, J);
        const int hy = y * p.r + I, hx = x * p.r + J;
        return p.b + ((size_t)(b * p.H * p.r + hy) * (p.W * p.r) + hx) * p.cb + ch;
      }
    default:  // VIEW_SHUFFLE_CONCAT: [shuffle_r(a (LR, ca = r^2 c0 ch)), b (HR, cb ch)]
      if (c < p.c0) {
        const int qq = (y % p.r) * p.r + (x % p.r);
        return p.a + ((size_t)(b * (p.H / p.r) + y / p.r) * (p.W / p.r) + x / p.r) * p.ca +
               qq * p.c0 + c;
      }
      return p.b + ((size_t)(b * p.H + y) * p.W + x) * p.cb + (c - p.c0);
  }
}

// 8 consecutive channels [c, c+8) of the conv input at pixel (b, y, x) through
// the view (zero outside the image).
__device__ __forceinline__ bf16x8 view_chunk(const ConvArgs& p, int b, int y, int x, int c) {
  const uint16_t* ptr = view_ptr(p, b, y, x, c);
  return ptr ? ld8(ptr) : zero8();
}

__device__ __forceinline__ bf16x8 load_chunk(const ConvArgs& p, int b, int y, int x, int tap,
                                             int c) {
  if (tap >= p.taps) return zero8();
  if (p.taps == 9) {
    y += tap / 3 - 1;
    x += tap % 3 - 1;
  }
  return view_chunk(p, b, y, x, c);
}

// Accumulates the 32 x (16 NT) output tile of one wave over the whole K.  SWAP: the
// weights are the MFMA's A operand, so that a lane holds 4 channels of one pixel
// (acc[r][j]: pixel 16 r + lane % 16, channels 16 j + 4 (lane / 16) ..) instead of 4
// pixels of one channel; bitwise the same sums.
template <int NT, bool SWAP = false>
__device__ __forceinline__ void conv_mainloop(const ConvArgs& p, int M, int m0, int n0, int lane,
                                              f32x4 (&acc)[2][NT]) {
  const int kq = lane >> 4, li = lane & 15;
  int pb[2], py[2], px[2];
  bool pv[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int m = m0 + r * 16 + li;
    pv[r] = m < M;
    const int mm = pv[r] ? m : 0;
    px[r] = mm % p.W;
    const int t = mm / p.W;
    py[r] = t % p.H;
    pb[r] = t / p.H;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int cpt = p.cin_p >> 3;  // 8-channel chunks per tap
  // packed row by row, or in fragment order: 16 rows x 32 K as 64 lanes x 8
  const uint16_t* wrow =
      p.w + (p.frag ? (size_t)n0 * p.kp + lane * 8 : (size_t)(n0 + li) * p.kp + kq * 8);
  const int wstep = p.frag ? 16 : 1;  // elements from one K index to the next, in steps of 32
  // Operands of K step ks; the next step's loads are issued before this step's
  // MFMAs so that their latency overlaps the matrix work.
  auto load_step = [&](int ks, bf16x8 (&A)[2], bf16x8 (&Bv)[NT]) {
    const int q = (ks >> 3) + kq;
    const int tap = q / cpt;
    const int c = (q - tap * cpt) << 3;
#pragma unroll
    for (int r = 0; r < 2; ++r) A[r] = pv[r] ? load_chunk(p, pb[r], py[r], px[r], tap, c) : zero8();
#pragma unroll
    for (int j = 0; j < NT; ++j) Bv[j] = ld8(wrow + (size_t)j * 16 * p.kp + ks * wstep);
  };
  bf16x8 A[2], Bv[NT];
  load_step(0, A, Bv);
  for (int ks = 0; ks < p.kp; ks += 32) {
    bf16x8 An[2], Bn[NT];
    if (ks + 32 < p.kp) load_step(ks + 32, An, Bn);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[r][j] = SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bv[j], A[r], acc[r][j], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[r], Bv[j], acc[r][j], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 2; ++r) A[r] = An[r];
#pragma unroll
    for (int j = 0; j < NT; ++j) Bv[j] = Bn[j];
  }
}

// Epilogue of a wave's 32 x (16 NT) tile: bias, ReLU, residuals, FP32 and/or
// BF16 stores.  m[r][v] is the output pixel of accumulator row v of row tile r
// (-1: outside the image).  Every load (bias, residuals) is issued before the
// first store: the output pointers may alias nothing, but the compiler cannot
// know that, and interleaving would serialise one memory latency per element.
// The epilogue's first inputs (bias and the first residual), which a kernel
// may load before its main loop so that their latency overlaps the MFMAs.
template <int NT>
struct EpiIn {
  float bias[NT];
  float res[2][NT][4];
};

template <int NT>
__device__ __forceinline__ void epi_load(const ConvArgs& p, const int64_t (&m)[2][4], int n0,
                                         int li, EpiIn<NT>& in) {
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int n = n0 + j * 16 + li;
    in.bias[j] = n < p.cout ? p.bias[n] : 0.0f;
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = n0 + j * 16 + li;
        in.res[r][j][v] = (p.res && m[r][v] >= 0 && n < p.cout)
                              ? p.res[(size_t)m[r][v] * p.cout + n] : 0.0f;
      }
}

template <int NT>
__device__ __forceinline__ void conv_epilogue(const ConvArgs& p, const f32x4 (&acc)[2][NT],
                                              const int64_t (&m)[2][4], int n0, int li,
                                              const EpiIn<NT>& in) {
  bool nv[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) nv[j] = n0 + j * 16 + li < p.cout;
  float y[2][NT][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float t = acc[r][j][v] + in.bias[j];
        y[r][j][v] = p.relu ? fmaxf(t, 0.0f) : t;
      }
  if (p.res) {
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[r][j][v] = in.res[r][j][v] + p.res_scale * y[r][j][v];
  }
  if (p.res2) {
    float rv[2][NT][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          rv[r][j][v] = (m[r][v] >= 0 && nv[j])
                            ? p.res2[(size_t)m[r][v] * p.cout + n0 + j * 16 + li] : 0.0f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[r][j][v] += rv[r][j][v];
  }
  if (p.res3) {
    float rv[2][NT][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          rv[r][j][v] = (m[r][v] >= 0 && nv[j])
                            ? p.res3[(size_t)m[r][v] * p.cout + n0 + j * 16 + li] : 0.0f;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[r][j][v] += rv[r][j][v];
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (m[r][v] < 0 || !nv[j]) continue;
        const int n = n0 + j * 16 + li;
        if (p.out_f) p.out_f[(size_t)m[r][v] * p.out_f_stride + n] = y[r][j][v];
        if (p.out_h) p.out_h[(size_t)m[r][v] * p.out_h_stride + n] = f2bf(y[r][j][v]);
      }
}

constexpr int C3_W = 16;  // tile width: one 16-pixel MFMA row tile

__device__ __forceinline__ bool pos_bf(uint16_t h) { return h != 0 && !(h & 0x8000u); }

// Fragment order of packed weights: 16-row tiles, each as K steps of 32, each as the 64
// lanes' 8 weights in the order of the MFMA's A operand (lane l: row l % 16, K
// 8 (l / 16) ..), so that a wave loads a step as one run of 1 KB.

// 3x3 convolution of 64-channel slices (cin_p a multiple of 64) with its weights
// held in registers.  A block owns a tile of 16 columns x WR R rows of one image
// and 16 WN output channels; wave (wr, wn) computes R rows x 16 channels.  The
// input tile with its halo is staged in LDS, 64 channels at a time; the 18 K
// steps' weights of a slice stay in the wave's registers and the wave sweeps the
// R + 2 input rows once: a row's operands are read from LDS for the outer two tap
// columns, shifted between lanes for the middle one, and feed the three output
// rows that use them (taps dy = 0, 1, 2).  That is 0.28 LDS reads per MFMA (R = 8);
// reading both operands for every product took 0.75 and made LDS bandwidth the
// bound.  The weights are the MFMA's A operand (rows = output channels), the
// pixels its B operand, so a lane ends up with 4 consecutive channels of one
// pixel and the epilogue moves 8 and 16 bytes at a time.  The next slice's
// weights are loaded as the last rows release the registers, and the next tile
// goes through registers into the other LDS buffer.  The weights are packed in
// fragment order: row-major ones cost 16 half-used lines a load
// and 7 us a launch.
// Every output sums its K in the order slice, tap, channel, whatever the plan.
// Measured (720p LR image, 64 / 128 / 256 input channels, one launch after the
// other): 8.6 / 11.7 / 24.0 us (with FP32 residual in and out), 494 / 725 / 708
// TFLOP/s; the 2-wave-per-SIMD MFMA time is 1.9 us for 64 channels, the LDS reads
// 1.1, a launch 2.5, the first loads 1.7, the stores 2.  As data gradients of the
// dense blocks (16384 pixels) 43-50 us by the direct conv, 5-8 now.
template <int R, int WR>
constexpr int rw_tile_px() {
  return (WR * R + 2) * (C3_W + 2);
}
// BF16 per tile pixel.  A wave's operand read takes 8 clocks at this pitch (16 without the
// padding; 5 with 16 of padding, which changes no conv's time: they wait on latency).
constexpr int RW_PITCH = 64 + 8;

// What the epilogue of a conv adds and where it stores: y = relu?(acc + bias),
// y = a1 + s1 y, y += a2, y += a3, zero where mask <= 0, to out_f (FP32) and
// out_h (BF16 of y out_h_scale).  Pointers are to channel 0 of the block's group
// of channels at pixel 0, with a stride in channels per pixel each.
struct RwEpi {
  const float *a1, *a2, *a3;
  const uint16_t* mask;
  float* out_f;
  uint16_t* out_h;
  int st1, st2, st3, stm, stf, sth;
  float s1, out_h_scale;
};

enum RwMode { RW_FWD = 0, RW_DG = 1 };

template <int MODE>
__device__ __forceinline__ RwEpi rw_epi(const ConvArgs& p, const BwdEpi& e, int n0) {
  RwEpi o;
  o.a1 = o.a2 = o.a3 = nullptr;
  o.mask = nullptr;
  o.out_f = nullptr;
  o.out_h = nullptr;
  o.st1 = o.st2 = o.st3 = o.stm = o.stf = o.sth = NET_FEAT;
  o.s1 = 1.0f;
  o.out_h_scale = 1.0f;
  if (MODE == RW_FWD) {
    o.a1 = p.res ? p.res + n0 : nullptr;
    o.a2 = p.res2 ? p.res2 + n0 : nullptr;
    o.a3 = p.res3 ? p.res3 + n0 : nullptr;
    o.st1 = o.st2 = o.st3 = p.cout;
    o.s1 = p.res_scale;
    o.out_f = p.out_f ? p.out_f + n0 : nullptr;
    o.stf = p.out_f_stride;
    o.out_h = p.out_h ? p.out_h + n0 : nullptr;
    o.sth = p.out_h_stride;
  } else if (e.mode == EPI_PLAIN) {
    o.a1 = e.add1 ? e.add1 + n0 : nullptr;
    o.a2 = e.add2 ? e.add2 + n0 : nullptr;
    o.mask = e.mask ? e.mask + n0 : nullptr;
    o.out_f = e.out_f ? e.out_f + n0 : nullptr;
    o.out_h = e.out_h ? e.out_h + n0 : nullptr;
    o.st1 = o.st2 = o.stm = o.stf = o.sth = e.stride;
    o.out_h_scale = e.out_h_scale;
  } else {  // EPI_DENSE: input slice n0 / 64 of a residual dense block
    const int sl = n0 >> 6, ch = n0 & 63;
    if (e.k == 1) {  // x_0 complete: the gradient of the block input
      o.a1 = e.ga + n0;
      o.st1 = RDG_DENSE;
      o.a2 = e.add1 ? e.add1 + ch : nullptr;
      o.a3 = e.add2 ? e.add2 + ch : nullptr;
      o.mask = e.mask0 ? e.dense + n0 : nullptr;
      o.stm = RDG_DENSE;
      o.out_f = e.out_f ? e.out_f + ch : nullptr;
      o.out_h = e.out_h + ch;
    } else if (sl == e.k - 1) {  // x_{k-1} complete: through its ReLU
      o.a1 = e.fusing ? nullptr : e.ga + n0;
      o.st1 = RDG_DENSE;
      o.mask = e.dense + n0;
      o.stm = RDG_DENSE;
      o.out_h = e.dy_next + ch;
    } else {  // a running slice gradient; the block's last conv starts it
      if (e.fusing) {
        o.a1 = sl == 0 ? e.ds + ch : nullptr;
      } else {
        o.a1 = e.ga + n0;
        o.st1 = RDG_DENSE;
      }
      o.out_f = e.ga + n0;
      o.stf = RDG_DENSE;
    }
  }
  return o;
}

// Buffer accesses: a uniform base, a 32-bit lane offset in bytes and a scalar
// offset in one instruction.  A lane whose offset is not below `bytes` loads
// zeros and stores nothing (the buffer's range check), so a lane outside the
// image gets the offset BUF_OUT and needs no branch; in-image offsets stay
// below 2^31 (18 rows of 256 FP32 channels: up to 116,508 pixels a row, which the
// launches check).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t BUF_OUT = 0x80000000u, BUF_MAX = 0x7fffffffu;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void* base, uint32_t bytes = BUF_MAX) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 buf_ld16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t s = 0) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)s, 0);
}
__device__ __forceinline__ u32x2 buf_ld8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
}
__device__ __forceinline__ void buf_st16(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, 0);
}
__device__ __forceinline__ void buf_st8(__amdgpu_buffer_rsrc_t r, uint32_t off, u32x2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)off, 0, 0);
}

// The operands of the middle tap column (pixel li + 1 in lane li) from those of
// the outer two (pixels li and li + 2): lanes 1..15 of a row take the next
// column's operand of the lane before, lane 0 this column's of the lane after.
__device__ __forceinline__ bf16x8 rw_middle(bf16x8 left, bf16x8 right) {
  const uint4 l = __builtin_bit_cast(uint4, left), r = __builtin_bit_cast(uint4, right);
  auto one = [](uint32_t a, uint32_t c) {
    const int first = __builtin_amdgcn_update_dpp(0, (int)a, 0x101, 0xf, 0xf, false);  // row_shl:1
    return (uint32_t)__builtin_amdgcn_update_dpp(first, (int)c, 0x111, 0xf, 0xf, false);  // row_shr:1
  };
  return __builtin_bit_cast(bf16x8,
                            make_uint4(one(l.x, r.x), one(l.y, r.y), one(l.z, r.z), one(l.w, r.w)));
}

// One wave's sweep over R + 2 rows of an LDS tile TW pixels wide (tp: this lane's
// operand at the first row): acc[r] gets rows r .. r + 2 through the weights W[dy],
// s = 2 dx + c / 32.  after_row(i) runs when input row i is done with.
template <int R, int TW, class F>
__device__ __forceinline__ void rw_sweep(const uint16_t* tp, bf16x8 (&W)[3][6], f32x4 (&acc)[R],
                                         F after_row) {
  bf16x8 P[6], Q[6];
  auto row_load = [&](int i, bf16x8(&o)[6]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      o[c] = ld8(tp + i * TW * RW_PITCH + c * 32);
      o[4 + c] = ld8(tp + (i * TW + 2) * RW_PITCH + c * 32);
    }
  };
  row_load(0, P);
#pragma unroll
  for (int i = 0; i < R + 2; ++i) {
    if (i + 1 < R + 2) row_load(i + 1, Q);
#pragma unroll
    for (int c = 0; c < 2; ++c) P[2 + c] = rw_middle(P[c], P[4 + c]);
#pragma unroll
    for (int s = 0; s < 6; ++s)
#pragma unroll
      for (int dy = 2; dy >= 0; --dy) {
        const int r = i - dy;
        if (r < 0 || r >= R) continue;
        acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[dy][s], P[s], acc[r], 0, 0, 0);
      }
    after_row(i);
#pragma unroll
    for (int s = 0; s < 6; ++s) P[s] = Q[s];
    // keep the LDS reads one row ahead: hoisted further they spill
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Weights of tap row dy of channel slice ch (64 channels) for the 16 output
// channels from n on.
__device__ __forceinline__ void rw_weights(const ConvArgs& p, int dy, int n, int ch, int lane,
                                           bf16x8 (&W)[6]) {
  const auto w = buf(p.w);
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    const int ks = (dy * 3 + (s >> 1)) * (p.cin_p >> 5) + ch * 2;
    W[s] = __builtin_bit_cast(bf16x8,
                              buf_ld16(w, lane * 16 + (s & 1) * 1024, n * p.kp * 2 + ks * 1024));
  }
}

// The part of a conv's output that one wave holds: R rows of 16 pixels from
// (x0, yo) of image b, lane (li, kq) with 4 channels from nw + 4 kq of pixel li.
template <int R>
struct RwOut {
  size_t mo;   // the wave's first pixel
  int W, nw, rows, li, kq;
  bool xin;
  __device__ __forceinline__ RwOut(const ConvArgs& p, int b, int yo, int x0, int nw_, int li_,
                                   int kq_)
      : W(p.W), nw(nw_), li(li_), kq(kq_) {
    rows = min(max(p.H - yo, 0), R);  // rows inside the image
    mo = ((size_t)b * p.H + min(yo, p.H - 1)) * p.W + x0;
    xin = x0 + li < p.W;
  }
  // a tensor of `stride` channels of `sz` bytes from the wave's first pixel and
  // channel on, ending with its last row in the image, and the lane's offset in it
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t tbuf(const void* base, int stride,
                                                         int sz) const {
    return buf((const char*)base + (mo * stride + nw) * sz, (uint32_t)(rows * W * stride) * sz);
  }
  __device__ __forceinline__ uint32_t off(int stride, int sz) const {
    return xin ? (uint32_t)(li * stride + kq * 4) * sz : BUF_OUT;
  }
  __device__ __forceinline__ void load(const float* a, int stride, f32x4 (&v)[R]) const {
    const auto t = tbuf(a, stride, 4);
    const uint32_t o = off(stride, 4);
#pragma unroll
    for (int r = 0; r < R; ++r)
      v[r] = __builtin_bit_cast(f32x4, buf_ld16(t, o + r * (W * stride * 4)));
  }
};

// The epilogue's first inputs, loaded ahead: the first tensor to add and the bias.
template <int R, int MODE>
__device__ __forceinline__ void rw_epi_load(const ConvArgs& p, const RwEpi& e, const RwOut<R>& o,
                                            int n0, f32x4 (&r1)[R], float (&bias)[4]) {
  if (e.a1) o.load(e.a1, e.st1, r1);
  if (MODE == RW_FWD) {
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[q] = p.bias[n0 + o.nw + o.kq * 4 + q];
  }
}

// Loads before stores: the outputs may alias the inputs for all the compiler knows.
template <int R, int MODE>
__device__ __forceinline__ void rw_epilogue(const ConvArgs& p, const RwEpi& e, const RwOut<R>& o,
                                            const f32x4 (&r1)[R], const float (&bias)[4],
                                            f32x4 (&acc)[R]) {
  if (MODE == RW_FWD) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[r][q] += bias[q];
    if (p.relu) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[r][q] = fmaxf(acc[r][q], 0.0f);
    }
  }
  if (e.a1) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[r][q] = r1[r][q] + e.s1 * acc[r][q];
  }
#pragma unroll 1
  for (int k = 0; k < 2; ++k) {
    const float* a = k ? e.a3 : e.a2;
    if (!a) continue;
    f32x4 v[R];
    o.load(a, k ? e.st3 : e.st2, v);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[r][q] += v[r][q];
  }
  if (MODE != RW_FWD && e.mask) {
    u32x2 mk[R];
    const auto t = o.tbuf(e.mask, e.stm, 2);
    const uint32_t lo = o.off(e.stm, 2);
#pragma unroll
    for (int r = 0; r < R; ++r) mk[r] = buf_ld8(t, lo + r * (o.W * e.stm * 2));
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (!pos_bf((uint16_t)(mk[r][q >> 1] >> (16 * (q & 1))))) acc[r][q] = 0.0f;
  }
  if (e.out_f) {
    const auto t = o.tbuf(e.out_f, e.stf, 4);
    const uint32_t lo = o.off(e.stf, 4);
#pragma unroll
    for (int r = 0; r < R; ++r)
      buf_st16(t, lo + r * (o.W * e.stf * 4), __builtin_bit_cast(u32x4, acc[r]));
  }
  if (e.out_h) {
    const auto t = o.tbuf(e.out_h, e.sth, 2);
    const uint32_t lo = o.off(e.sth, 2);
    const float sc = MODE == RW_DG ? e.out_h_scale : 1.0f;
#pragma unroll
    for (int r = 0; r < R; ++r)
      buf_st8(t, lo + r * (o.W * e.sth * 2), u32x2{f2bf2(acc[r][0] * sc, acc[r][1] * sc),
                                                   f2bf2(acc[r][2] * sc, acc[r][3] * sc)});
  }
}

template <int R, int WR, bool MULTI>
constexpr int rw_lds() {  // BF16 values of LDS that a block takes
  return (MULTI ? 2 : 1) * rw_tile_px<R, WR>() * RW_PITCH;
}

// Block (bx, by, bz) of the conv, with rw_lds() values of LDS from `lds` on.
template <int R, int WR, int WN, bool MULTI, int MODE>
__device__ __forceinline__ void conv3_rw_block(const ConvArgs& p, int cout_p, int nsplit,
                                               const BwdEpi& be, uint16_t* lds, int bx, int by,
                                               int bz) {
  constexpr int THREADS = 64 * WR * WN, TH = WR * R, TILE = rw_tile_px<R, WR>();
  constexpr int TCH = TILE * 8, CNT = (TCH + THREADS - 1) / THREADS;
  constexpr int BN = WN * 16;
  auto tile = reinterpret_cast<uint16_t(*)[TILE * RW_PITCH]>(lds);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, li = lane & 15;
  const int wr = wave % WR, wn = wave / WR;
  const int x0 = bx * C3_W, y0 = by * TH;
  const int b = bz / nsplit, part = bz - b * nsplit;
  const int nper = cout_p / nsplit;  // output channels of this block (a multiple of BN)
  const int nchunk = MULTI ? p.cin_p >> 6 : 1;
  // this thread's chunks (8 channels of a pixel) of the input tile: byte offsets
  // from the tile's first pixel inside the image (BUF_OUT: outside, zeros)
  const int vs = p.mode == VIEW_PLAIN ? 0 : 1;  // log2 of the view's shuffle
  const int yb = max(y0 - 1, 0) >> vs, xb = max(x0 - 1, 0) >> vs;
  const auto src = buf(p.a + (((size_t)b * (p.H >> vs) + yb) * (p.W >> vs) + xb) * p.ca);
  uint32_t off[CNT];
#pragma unroll
  for (int u = 0; u < CNT; ++u) {
    const int i = tid + u * THREADS, px = i >> 3;
    const int ty = px / (C3_W + 2), tx = px - ty * (C3_W + 2);
    const int y = y0 - 1 + ty, x = x0 - 1 + tx;
    int c = (i & 7) * 8;
    if (vs) c += (2 * (y & 1) + (x & 1)) * 64;  // shuffle: slot of the coarse pixel
    off[u] = i < TCH && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W
                 ? (uint32_t)((((y >> vs) - yb) * (p.W >> vs) + ((x >> vs) - xb)) * p.ca + c) * 2u
                 : BUF_OUT;
  }
  auto tile_load = [&](int cbase, u32x4(&v)[CNT]) {
#pragma unroll
    for (int u = 0; u < CNT; ++u) v[u] = buf_ld16(src, off[u], cbase * 2);
  };
  auto tile_store = [&](int which, const u32x4(&v)[CNT]) {
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int i = tid + u * THREADS;
      if (i < TCH)
        *reinterpret_cast<u32x4*>(&tile[which][(i >> 3) * RW_PITCH + (i & 7) * 8]) = v[u];
    }
  };
  bf16x8 W[3][6];
  const int nw = wn * 16;  // the wave's channels within a group of BN
  {
    u32x4 v[CNT];
    tile_load(0, v);
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) rw_weights(p, dy, part * nper + nw, 0, lane, W[dy]);
    tile_store(0, v);
  }
  __syncthreads();
  const int nstep = nper / BN * nchunk;
  f32x4 acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  const RwOut<R> out(p, b, y0 + wr * R, x0, nw, li, kq);
  int n0 = part * nper, ch = 0;
  for (int st = 0; st < nstep; ++st) {
    const bool lastch = !MULTI || ch == nchunk - 1;
    const bool more = st + 1 < nstep;
    const int ch1 = lastch ? 0 : ch + 1, n1 = lastch ? n0 + BN : n0;  // the next step's
    u32x4 v[CNT];
    if (MULTI && more) tile_load(ch1 * 64, v);
    // the epilogue's first inputs are on their way during the last slice
    const RwEpi e = rw_epi<MODE>(p, be, n0);
    f32x4 r1[R];
    float bias[4];
    if (lastch) rw_epi_load<R, MODE>(p, e, out, n0, r1, bias);
    rw_sweep<R, C3_W + 2>(
        &tile[MULTI ? st & 1 : 0][((wr * R) * (C3_W + 2) + li) * RW_PITCH + kq * 8], W, acc,
        [&](int i) {  // tap row i - R + 1 is done with: the next step's weights
          if (i >= R - 1 && more) rw_weights(p, i - (R - 1), n1 + nw, ch1, lane, W[i - (R - 1)]);
        });
    if (MULTI && more) {
      tile_store((st + 1) & 1, v);
      __syncthreads();
    }
    if (lastch) {
      rw_epilogue<R, MODE>(p, e, out, r1, bias, acc);
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    n0 = n1;
    ch = ch1;
  }
}

template <int R, int WR, int WN, bool MULTI, int MODE>
__global__ __launch_bounds__(64 * WR * WN) void k_conv3_rw(ConvArgs p, int cout_p, int nsplit,
                                                           BwdEpi be) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[rw_lds<R, WR, MULTI>()];
  conv3_rw_block<R, WR, WN, MULTI, MODE>(p, cout_p, nsplit, be, lds, blockIdx.x, blockIdx.y,
                                         blockIdx.z);
}

// Runs the conv on k_conv3_rw if it fits: 3x3 over cin_p = 64 n channels of a
// plain view, or the 64 channels of a shuffle by 2; no padding in K or in the
// output channels, and channel strides that the epilogue's vectors can take.
// The output channels are split over nsplit blocks per tile.
template <int R, int WR, int WN, int MODE>
bool conv3_rw_fits(const ConvArgs& a, int cout_p, int nsplit, const BwdEpi* be) {
  const bool multi = a.cin_p > 64;
  if (!a.frag || a.taps != 9 || (a.mode == VIEW_PLAIN && a.ca < a.cin_p) || a.cin_p % 64 || a.kp != 9 * a.cin_p ||
      (a.mode != VIEW_PLAIN && (multi || a.c0 != 64 || a.r != 2)) || a.cout != cout_p ||
      cout_p % (WN * 16 * nsplit))
    return false;
  // a tile's offsets fit 31 bits (images up to about 116,000 pixels wide)
  if ((int64_t)(WR * R + 2) * a.W * RDG_DENSE * 4 >= (int64_t)BUF_OUT) return false;
  if (MODE == RW_FWD && ((a.out_f && a.out_f_stride % 4) || (a.out_h && a.out_h_stride % 8)))
    return false;
  if (be && be->scale != 1.0f) return false;
  if (MODE == RW_DG &&
      (be->mode == EPI_PLAIN ? be->stride % 8 != 0 : be->mode != EPI_DENSE))
    return false;
  return true;
}
template <int R, int WR, int WN, int MODE>
bool try_conv3_rw(const ConvArgs& a, int cout_p, int nsplit, hipStream_t st, const BwdEpi* be) {
  if (!conv3_rw_fits<R, WR, WN, MODE>(a, cout_p, nsplit, be)) return false;
  const bool multi = a.cin_p > 64;
  BwdEpi e;
  if (be) e = *be;
  else std::memset(&e, 0, sizeof e);
  const dim3 grid((a.W + C3_W - 1) / C3_W, (a.H + WR * R - 1) / (WR * R), a.B * nsplit);
  if (multi)
    k_conv3_rw<R, WR, WN, true, MODE><<<grid, 64 * WR * WN, 0, st>>>(a, cout_p, nsplit, e);
  else
    k_conv3_rw<R, WR, WN, false, MODE><<<grid, 64 * WR * WN, 0, st>>>(a, cout_p, nsplit, e);
  return true;
}

// One residual block of the trunk in one launch: for a 16 x 16 output tile,
// y = res + res_scale convB(ReLU(convA(x))) (+ res2), convA and convB 3x3 convs
// of 64 channels, both as in k_conv3_rw (weights in registers, 8 waves of 8 or 9
// rows x 16 channels).  The block stages x with a halo of 2 and computes convA on
// the 18 x 18 pixels convB needs: 16 columns of them by the row sweep, the last
// two as pixel groups of 8 rows x 2 columns (19 M tiles in place of 16), whose
// MFMAs run between the sweep's.  ReLU(convA) goes to LDS as BF16 -- zero outside
// the image, which is convB's zero padding.  ConvB's weights are loaded as convA's
// last rows release the registers, the FP32 residual during convB.  The
// intermediate is rounded to BF16 as the two-conv path stores it and every output
// element sums its K in the same order, so the result is bitwise that of convA
// then convB as two launches, less one launch and the intermediate's round trip.
// Measured (720p LR image, 240 tiles): 27.0 -> 19.9 us a launch (with both operands
// of every MFMA read from LDS: 0.75 reads each); the MFMA time is 4.7 us.
constexpr int RB_T = 16;          // output tile
constexpr int RB_IN = RB_T + 4;   // input tile rows / columns (halo of both convs)
constexpr int RB_MID = RB_T + 2;  // convA outputs = convB's input tile
constexpr int RB_C = 64;          // channels in and out of both convs
constexpr int RB_KP = 9 * RB_C;
constexpr int RB_THREADS = 512;   // 8 waves: 2 halves of the rows x 4 channel tiles
constexpr int RB_RA = RB_MID / 2, RB_RB = RB_T / 2;  // rows per wave of convA and convB

__global__ __launch_bounds__(RB_THREADS) void k_res_block(ConvArgs pa, ConvArgs pb) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[RB_IN * RB_IN * RW_PITCH];
  __shared__ __attribute__((aligned(16))) uint16_t mid[RB_MID * RB_MID * RW_PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, li = lane & 15;
  const int wr = wave & 1, nw = (wave >> 1) * 16;
  const int x0 = blockIdx.x * RB_T, y0 = blockIdx.y * RB_T, b = blockIdx.z;
  constexpr int TCH = RB_IN * RB_IN * (RB_C / 8), CNT = (TCH + RB_THREADS - 1) / RB_THREADS;
  bf16x8 W[3][6];
  {
    const int yb = max(y0 - 2, 0), xb = max(x0 - 2, 0);
    const auto src = buf(pa.a + (((size_t)b * pa.H + yb) * pa.W + xb) * pa.ca);
    u32x4 v[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int i = tid + u * RB_THREADS, px = i >> 3;
      const int ty = px / RB_IN, tx = px - ty * RB_IN;
      const int y = y0 - 2 + ty, x = x0 - 2 + tx;
      v[u] = buf_ld16(src, i < TCH && (unsigned)y < (unsigned)pa.H && (unsigned)x < (unsigned)pa.W
                               ? (uint32_t)(((y - yb) * pa.W + (x - xb)) * pa.ca + (i & 7) * 8) * 2u
                               : BUF_OUT);
    }
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) rw_weights(pa, dy, nw, 0, lane, W[dy]);
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int i = tid + u * RB_THREADS;
      if (i < TCH) *reinterpret_cast<u32x4*>(tile + (i >> 3) * RW_PITCH + (i & 7) * 8) = v[u];
    }
  }
  float bias[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) bias[q] = pa.bias[nw + kq * 4 + q];
  __syncthreads();
  {
    // convA.  Columns 16 and 17: lane li holds pixel (er + li / 2, 16 + li % 2) of
    // group g; half wr takes rows 8 wr .. 8 wr + 7 (g = 0), half 1 also rows 16, 17
    f32x4 acc[RB_RA], ex[2];
#pragma unroll
    for (int r = 0; r < RB_RA; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    ex[0] = ex[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int er0 = 8 * wr + (li >> 1), er1 = RB_T + ((li >> 1) & 1), ec = RB_T + (li & 1);
    const uint16_t* e0 = tile + (er0 * RB_IN + ec) * RW_PITCH + kq * 8;
    const uint16_t* e1 = tile + (er1 * RB_IN + ec) * RW_PITCH + kq * 8;
    rw_sweep<RB_RA, RB_IN>(
        tile + (wr * RB_RA * RB_IN + li) * RW_PITCH + kq * 8, W, acc, [&](int i) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {  // K steps 2 i and 2 i + 1 of the last two columns
            const int t = (2 * i + h) / 2, c = h;  // tap, channel half
            if (t >= 9) continue;
            const int dy = t / 3, dx = t - dy * 3, o = (dy * RB_IN + dx) * RW_PITCH + c * 32;
            ex[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[dy][2 * dx + c], ld8(e0 + o), ex[0],
                                                            0, 0, 0);
            if (wr)
              ex[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[dy][2 * dx + c], ld8(e1 + o),
                                                              ex[1], 0, 0, 0);
          }
          if (i >= RB_RA - 1) rw_weights(pb, i - (RB_RA - 1), nw, 0, lane, W[i - (RB_RA - 1)]);
        });
    // ReLU(convA + bias) as BF16, zero outside the image
    auto put = [&](const f32x4& a, int iy, int ix) {
      const int y = y0 - 1 + iy, x = x0 - 1 + ix;
      const bool in = (unsigned)y < (unsigned)pa.H && (unsigned)x < (unsigned)pa.W;
      float v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = in ? fmaxf(a[q] + bias[q], 0.0f) : 0.0f;
      *reinterpret_cast<u32x2*>(mid + (iy * RB_MID + ix) * RW_PITCH + nw + kq * 4) =
          u32x2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
    };
#pragma unroll
    for (int r = 0; r < RB_RA; ++r) put(acc[r], wr * RB_RA + r, li);
    put(ex[0], er0, ec);
    if (wr && li < 4) put(ex[1], er1, ec);
  }
  __syncthreads();
  // convB on the 16 x 16 tile
  f32x4 acc[RB_RB], r1[RB_RB];
#pragma unroll
  for (int r = 0; r < RB_RB; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  BwdEpi none;
  const RwEpi e = rw_epi<RW_FWD>(pb, none, 0);
  const RwOut<RB_RB> out(pb, b, y0 + wr * RB_RB, x0, nw, li, kq);
  rw_epi_load<RB_RB, RW_FWD>(pb, e, out, 0, r1, bias);
  rw_sweep<RB_RB, RB_MID>(mid + (wr * RB_RB * RB_MID + li) * RW_PITCH + kq * 8, W, acc,
                          [](int) {});
  rw_epilogue<RB_RB, RW_FWD>(pb, e, out, r1, bias, acc);
}

// The 1x1 fuse conv [a, unshuffle(b)] -> 64 channels.  Its K is the LR image's 64
// channels and then 64 for each of the r^2 pixels of the HR block: reading the HR
// features once is what bounds it.  A block of 8 waves stages the weights of
// FU_KS K steps in LDS (48 KB, two blocks per CU); each wave owns 16 LR pixels x 64
// channels and has the operands of all these K steps in flight at once, straight
// from memory into registers (a K step is 32 channels of one HR pixel per LR
// pixel, so its place in the block is uniform).  K steps ascend, as in k_conv.
// Measured at 720p: 57 us as k_conv<4>, 32 here (51 MB read once: 11 us at the rate of a
// copy); 17 K steps a batch instead of 12 spill.
constexpr int FU_KS = 12, FU_WAVES = 8;

__global__ __launch_bounds__(64 * FU_WAVES, 4) void k_fuse(ConvArgs p) {
  __shared__ __attribute__((aligned(16))) uint16_t wts[FU_KS * 4 * 512];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, li = lane & 15;
  const int64_t M = (int64_t)p.B * p.H * p.W, m0 = ((int64_t)blockIdx.x * FU_WAVES + wave) * 16;
  const int ks_all = p.kp >> 5;
  // this lane's pixel and its operands' offsets from the wave's first pixel's
  const int64_t mf = m0 < M ? m0 : M - 1, m = m0 + li;
  const int64_t tf = mf / p.W, t = (m < M ? m : M - 1) / p.W;
  const int Xf = (int)(mf - tf * p.W), X = (int)((m < M ? m : M - 1) - t * p.W);
  const int wr = p.W * p.r;
  const auto fa = buf(p.a + mf * NET_FEAT);
  const auto fb = buf(p.b + (tf * p.r * wr + (int64_t)Xf * p.r) * NET_FEAT);
  const uint32_t oa = m < M ? (uint32_t)(li * NET_FEAT + kq * 8) * 2u : BUF_OUT;
  const uint32_t ob = m < M ? (uint32_t)(((int)(t - tf) * p.r * wr + (X - Xf) * p.r) * NET_FEAT +
                                         kq * 8) * 2u
                            : BUF_OUT;
  f32x4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const auto wb = buf(p.w);
  for (int k0 = 0; k0 < ks_all; k0 += FU_KS) {
    // weights [K step][16-channel tile][lane], packed as [tile][K step][lane]
    constexpr int WCH = FU_KS * 4 * 64, CNT = (WCH + 64 * FU_WAVES - 1) / (64 * FU_WAVES);
    u32x4 v[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int i = tid + u * 64 * FU_WAVES, ks = k0 + (i >> 8), j = (i >> 6) & 3;
      v[u] = buf_ld16(wb, i < WCH && ks < ks_all
                              ? (uint32_t)((j * ks_all + ks) * 64 + (i & 63)) * 16u
                              : BUF_OUT);
    }
    bf16x8 P[FU_KS];
#pragma unroll
    for (int u = 0; u < FU_KS; ++u) {
      const int ks = k0 + u;
      if (ks >= ks_all) continue;  // uniform
      if (ks < 2) {
        P[u] = __builtin_bit_cast(bf16x8, buf_ld16(fa, oa, ks * 64));
      } else {
        int I, J;
        unshuffle_slot((ks - 2) >> 1, p.r, p.dsf, I, J);
        P[u] = __builtin_bit_cast(
            bf16x8, buf_ld16(fb, ob, (uint32_t)((I * wr + J) * NET_FEAT + (ks & 1) * 32) * 2u));
      }
    }
    if (k0) __syncthreads();  // the previous steps' weights are no longer read
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      const int i = tid + u * 64 * FU_WAVES;
      if (i < WCH) *reinterpret_cast<u32x4*>(wts + (size_t)i * 8) = v[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < FU_KS; ++u) {
      if (k0 + u >= ks_all) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(wts + ((u * 4 + j) * 64 + lane) * 8),
                                                         P[u], acc[j], 0, 0, 0);
    }
  }
  if (m >= M) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = j * 16 + kq * 4;
    f32x4 y;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      y[q] = acc[j][q] + p.bias[n + q];
      y[q] = p.relu ? fmaxf(y[q], 0.0f) : y[q];
    }
    if (p.out_f) *reinterpret_cast<f32x4*>(p.out_f + (size_t)m * p.out_f_stride + n) = y;
    if (p.out_h)
      *reinterpret_cast<u32x2*>(p.out_h + (size_t)m * p.out_h_stride + n) =
          u32x2{f2bf2(y[0], y[1]), f2bf2(y[2], y[3])};
  }
}

bool try_fuse(const ConvArgs& a, int cout_p, hipStream_t st) {
  if (a.mode != VIEW_CONCAT_UNSHUFFLE || a.taps != 1 || !a.frag || cout_p != 64 || a.cout != 64 ||
      a.ca != NET_FEAT || a.cb != NET_FEAT || a.kp != NET_FEAT * (1 + a.r * a.r) || a.res ||
      (a.out_f && a.out_f_stride % 4) || (a.out_h && a.out_h_stride % 4) ||
      // offsets within two rows of HR blocks fit 31 bits
      (int64_t)2 * a.r * a.r * a.W * NET_FEAT * 2 >= (int64_t)BUF_OUT)
    return false;
  const int64_t M = (int64_t)a.B * a.H * a.W;
  k_fuse<<<(unsigned)((M + 16 * FU_WAVES - 1) / (16 * FU_WAVES)), 64 * FU_WAVES, 0, st>>>(a);
  return true;
}

// The reconstruction conv: 3x3 over [shuffle_r(a) (C0 channels), b (CB)] to 3
// channels in FP32.  A block of 4 waves stages the (16 + 2)^2 pixels of its tile in
// LDS (every load in flight at once), wave w computes rows 4 w .. 4 w + 3 with all
// weights in registers (only the 3 rows of the MFMA's A operand that hold output
// channels are read from memory).  Bound by reading its input (147 MB at 720p,
// 31 us at the rate of a copy).  K index tap (C0 + CB) + c: a K step may span taps.
// Measured at 720p: 79 -> 47 us (80 channels), 60 -> 37 (64).  Ten-odd dependent LDS reads
// and three blocks a CU lie between that and the floor.
template <int C0, int CB, int RS>
__global__ __launch_bounds__(256, 3) void k_rec(ConvArgs p) {
  constexpr int CIN = C0 + CB, KS = (9 * CIN + 31) / 32, TW = C3_W + 2, NPX = TW * TW;
  constexpr int PITCH = CIN % 32 == 0 ? CIN + 8 : CIN;  // 16-byte reads of 8 lanes hit all banks
  __shared__ __attribute__((aligned(16))) uint16_t tile[NPX * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kq = lane >> 4, li = lane & 15;
  const int x0 = blockIdx.x * C3_W, y0 = blockIdx.y * C3_W, b = blockIdx.z;
  // byte offsets from the tile's first pixel in the image (coarse pixel for a)
  const int yf = max(y0 - 1, 0), xf = max(x0 - 1, 0);
  const int hh = p.H / RS, ww = p.W / RS;
  const auto sa = buf(p.a + (((size_t)b * hh + yf / RS) * ww + xf / RS) * (C0 * RS * RS));
  const auto sb = buf(p.b + (((size_t)b * p.H + yf) * p.W + xf) * CB);
  constexpr int CA8 = C0 / 8, CB8 = CB / 8;
  constexpr int NA = (NPX * CA8 + 255) / 256, NB = (NPX * CB8 + 255) / 256;
  u32x4 va[NA], vb[NB > 0 ? NB : 1];
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int i = tid + u * 256, px = i / CA8, c = i - px * CA8;
    const int r = px / TW, y = y0 - 1 + r, x = x0 - 1 + px - r * TW;
    const bool in = px < NPX && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W;
    const int Y = y / RS, X = x / RS;
    va[u] = buf_ld16(sa, in ? (uint32_t)(((Y - yf / RS) * ww + X - xf / RS) * (C0 * RS * RS) +
                                         ((y - Y * RS) * RS + x - X * RS) * C0 + c * 8) * 2u
                            : BUF_OUT);
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int i = tid + u * 256, px = i / (CB8 > 0 ? CB8 : 1), c = i - px * CB8;
    const int r = px / TW, y = y0 - 1 + r, x = x0 - 1 + px - r * TW;
    const bool in = px < NPX && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W;
    vb[u] = buf_ld16(sb, in ? (uint32_t)(((y - yf) * p.W + x - xf) * CB + c * 8) * 2u : BUF_OUT);
  }
  bf16x8 Wt[KS];
  const auto wb = buf(p.w);
  const uint32_t wo = li < p.cout ? (uint32_t)(li * p.kp + kq * 8) * 2u : BUF_OUT;
#pragma unroll
  for (int s = 0; s < KS; ++s) Wt[s] = __builtin_bit_cast(bf16x8, buf_ld16(wb, wo, s * 64));
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int i = tid + u * 256, px = i / CA8, c = i - px * CA8;
    if (px < NPX) *reinterpret_cast<u32x4*>(tile + px * PITCH + c * 8) = va[u];
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int i = tid + u * 256, px = i / (CB8 > 0 ? CB8 : 1), c = i - px * CB8;
    if (px < NPX) *reinterpret_cast<u32x4*>(tile + px * PITCH + C0 + c * 8) = vb[u];
  }
  __syncthreads();
  f32x4 acc[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint16_t* tp = tile + ((4 * wave) * TW + li) * PITCH;
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = 32 * s + 8 * kq, tap = k / CIN, c = k - tap * CIN;
    const bool pad = 32 * (s + 1) > 9 * CIN && tap >= 9;  // the last K step's zero padding
    const int dy = tap / 3, dx = tap - dy * 3;
    const uint16_t* o = tp + (pad ? 0 : (dy * TW + dx) * PITCH + c);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bf16x8 P = ld8(o + r * TW * PITCH);
      if (pad) P = zero8();
      acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wt[s], P, acc[r], 0, 0, 0);
    }
  }
  const int x = x0 + li;
  if (kq == 0 && x < p.W) {  // rows 0 .. 2 of the result
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int y = y0 + 4 * wave + r;
      if (y >= p.H) continue;
      float* o = p.out_f + (((size_t)b * p.H + y) * p.W + x) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) o[c] = acc[r][c] + p.bias[c];
    }
  }
}

template <int C0, int CB, int RS>
bool try_rec(const ConvArgs& a, hipStream_t st) {
  if (a.mode != VIEW_SHUFFLE_CONCAT || a.taps != 9 || a.frag || a.cout != 3 || a.r != RS ||
      a.c0 != C0 || a.ca != C0 * RS * RS || a.cb != CB || a.cin_p != C0 + CB ||
      a.kp != (9 * a.cin_p + 31) / 32 * 32 || a.relu || a.res || a.res2 || a.out_h ||
      a.out_f_stride != 3 || (int64_t)(C3_W + 2) * a.W * 64 * 2 * RS >= (int64_t)BUF_OUT)
    return false;
  k_rec<C0, CB, RS><<<dim3((a.W + C3_W - 1) / C3_W, (a.H + C3_W - 1) / C3_W, a.B), 256, 0, st>>>(a);
  return true;
}

template <int NT>
__global__ __launch_bounds__(256) void k_conv(ConvArgs p) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int M = p.B * p.H * p.W;
  const int m0 = (blockIdx.x * 4 + wave) * 32;
  if (m0 >= M) return;
  const int n0 = blockIdx.y * (NT * 16);
  f32x4 acc[2][NT];
  conv_mainloop<NT>(p, M, m0, n0, lane, acc);
  const int kq = lane >> 4, li = lane & 15;
  int64_t m[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int mm = m0 + r * 16 + kq * 4 + v;
      m[r][v] = mm < M ? mm : -1;
    }
  EpiIn<NT> in;
  epi_load<NT>(p, m, n0, li, in);
  conv_epilogue<NT>(p, acc, m, n0, li, in);
}

// What the epilogue of k_dgrad does to 4 channels n .. n + 3 (n a multiple of 4, as are
// all strides and splits) of pixel m: the tensors to add, the mask, the outputs, with
// offsets in elements.
struct DgOut {
  const float *a1, *a2;
  const uint16_t* mask;
  float* out_f;
  uint16_t* out_h;
  float h_scale;
};

// b, y, x: pixel m's place in the conv's image.
template <int MODE>
__device__ __forceinline__ DgOut dg_out(const ConvArgs& p, const BwdEpi& e, int64_t m, int b,
                                        int y, int x, int n) {
  DgOut o{nullptr, nullptr, nullptr, nullptr, nullptr, 1.0f};
  if (MODE == EPI_PLAIN) {
    const int64_t i = m * e.stride + n;
    o.a1 = e.add1 ? e.add1 + i : nullptr;
    o.a2 = e.add2 ? e.add2 + i : nullptr;
    o.mask = e.mask ? e.mask + i : nullptr;
    o.out_f = e.out_f ? e.out_f + i : nullptr;
    o.out_h = e.out_h ? e.out_h + i : nullptr;
    o.h_scale = e.out_h_scale;
  } else if (MODE == EPI_REC_SPLIT) {  // this conv at HR; [shuffle(U) | h0]
    if (n < e.c_split) {
      const int Y = y / e.r, X = x / e.r, hh = p.H / e.r, ww = p.W / e.r;
      const int64_t i = ((int64_t)(b * hh + Y) * ww + X) * e.stride2 +
                        ((y - Y * e.r) * e.r + x - X * e.r) * e.c_split + n;
      o.mask = e.mask + i;
      o.out_h = e.out_h + i;
    } else {
      o.out_f = e.out_f + m * e.stride + (n - e.c_split);
    }
  } else if (MODE == EPI_FUSE_SPLIT) {  // this conv at LR; [fl | unshuffle(h0)]
    if (n < e.c_split) {
      const int64_t i = m * e.c_split + n;
      o.mask = e.mask + i;
      o.out_h = e.out_h + i;
    } else {
      const int cc = n - e.c_split, q = cc / e.stride, ch = cc - q * e.stride;
      int I, J;
      unshuffle_slot(q, e.r, e.dsf, I, J);
      const int64_t i =
          ((int64_t)(b * p.H * e.r + y * e.r + I) * (p.W * e.r) + x * e.r + J) * e.stride + ch;
      o.a1 = e.add1 ? e.add1 + i : nullptr;
      o.mask = e.mask2 + i;
      o.out_h = e.out_h2 + i;
    }
  } else {  // EPI_DENSE: input slices 0 .. k-1 of a residual dense block
    const int sl = n >> 6, ch = n & 63;
    const int64_t gi = m * RDG_DENSE + n, i64 = m * NET_FEAT + ch;
    if (e.k == 1) {  // x_0 complete: the gradient of the block input (a third sum: add2)
      o.a1 = e.ga + gi;
      o.a2 = e.add1 ? e.add1 + i64 : nullptr;
      o.mask = e.mask0 ? e.dense + gi : nullptr;
      o.out_f = e.out_f ? e.out_f + i64 : nullptr;
      o.out_h = e.out_h + i64;
    } else if (sl == e.k - 1) {  // x_{k-1} complete: through its ReLU
      o.a1 = e.fusing ? nullptr : e.ga + gi;
      o.mask = e.dense + gi;
      o.out_h = e.dy_next + i64;
    } else {
      o.a1 = !e.fusing ? e.ga + gi : sl == 0 ? e.ds + i64 : nullptr;
      o.out_f = e.ga + gi;
    }
  }
  return o;
}

// Data gradient of a conv: the same implicit GEMM over dY with the packed
// transposed, flipped weights; the epilogue applies the backward of what
// surrounds the conv (ReLU masks, residual sums, the (un)shuffle views).  Bound by the
// epilogue's traffic in the fuse and reconstruction convs that run here; a lane holds 4
// channels of a pixel, so that it moves 8 and 16 bytes at a time (2 and 4 with the
// operands' roles exchanged).  16 images of 128 x 128: fuse 113 -> 51 us (136 MB, 28 us
// at the rate of a copy), reconstruction 64 -> 34 (90 MB, 19 us); with 64 shuffled
// channels 90 -> 41 and 78 -> 30 us.
template <int NT, int MODE>
__device__ __forceinline__ void dgrad_block(const ConvArgs& p, const BwdEpi& e, int bx, int by) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int M = p.B * p.H * p.W;
  const int m0 = (bx * 4 + wave) * 32;
  if (m0 >= M) return;
  const int n0 = by * (NT * 16);
  f32x4 acc[2][NT];
  conv_mainloop<NT, true>(p, M, m0, n0, lane, acc);
  const int kq = lane >> 4, li = lane & 15;
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int m = m0 + r * 16 + li;
    if (m >= M) continue;
    const int x = m % p.W, t = m / p.W, y = t % p.H, b = t / p.H;
    DgOut o[NT];
    f32x4 v1[NT], v2[NT], v3[NT];
    u32x2 mk[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {  // loads before stores
      const int n = n0 + j * 16 + kq * 4;
      if (n >= p.cout) continue;
      o[j] = dg_out<MODE>(p, e, m, b, y, x, n);
      if (o[j].a1) v1[j] = *reinterpret_cast<const f32x4*>(o[j].a1);
      if (o[j].a2) v2[j] = *reinterpret_cast<const f32x4*>(o[j].a2);
      if (MODE == EPI_DENSE && e.k == 1 && e.add2)
        v3[j] = *reinterpret_cast<const f32x4*>(e.add2 + (int64_t)m * NET_FEAT + (n & 63));
      if (o[j].mask) mk[j] = *reinterpret_cast<const u32x2*>(o[j].mask);
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (n0 + j * 16 + kq * 4 >= p.cout) continue;
      f32x4 g = acc[r][j];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        g[q] *= e.scale;
        if (o[j].a1) g[q] += v1[j][q];
        if (o[j].a2) g[q] += v2[j][q];
        if (MODE == EPI_DENSE && e.k == 1 && e.add2) g[q] += v3[j][q];
        if (o[j].mask && !pos_bf((uint16_t)(mk[j][q >> 1] >> (16 * (q & 1))))) g[q] = 0.0f;
      }
      if (o[j].out_f) *reinterpret_cast<f32x4*>(o[j].out_f) = g;
      if (o[j].out_h)
        *reinterpret_cast<u32x2*>(o[j].out_h) =
            u32x2{f2bf2(g[0] * o[j].h_scale, g[1] * o[j].h_scale),
                  f2bf2(g[2] * o[j].h_scale, g[3] * o[j].h_scale)};
    }
  }
}

template <int NT, int MODE>
__global__ __launch_bounds__(256) void k_dgrad(ConvArgs p, BwdEpi e) {
  dgrad_block<NT, MODE>(p, e, blockIdx.x, blockIdx.y);
}

// Network input channels of one HRLS pixel: 16 BF16 values (log1p of clipped RGB,
// albedo, normal, log1p depth, 6 zeros; with the render layers instead of the
// depth: log1p of the clipped diffuse and glossy layers, log1p of the per-sample
// variance averaged over RGB, clamped to [0, 1e4]).
__device__ __forceinline__ float tone(float v) { return log1pf(fminf(fmaxf(v, 0.0f), 100.0f)); }

template <bool LAYERS>
struct HrPixel {  // loaded before any is used
  float rgb[3], aux[LAYERS ? 6 : 7], lay[LAYERS ? 6 : 1], sq[LAYERS ? 3 : 1];
  __device__ __forceinline__ void load(const InputArgs& p, int64_t i) {
#pragma unroll
    for (int c = 0; c < 3; ++c) rgb[c] = p.hr[3 * i + c];
#pragma unroll
    for (int c = 0; c < (LAYERS ? 6 : 7); ++c) aux[c] = p.aux[7 * i + c];
    if (LAYERS) {
#pragma unroll
      for (int c = 0; c < 6; ++c) lay[c] = p.layers[9 * i + 3 + c];
#pragma unroll
      for (int c = 0; c < 3; ++c) sq[c] = p.sumsq[3 * i + c];
    }
  }
  __device__ __forceinline__ void pack(const InputArgs& p, u32x4 (&o)[2]) const {
    float v[16];
    float var = 0.0f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      v[c] = tone(rgb[c]);
      if (LAYERS) var += sq[c] * p.inv_spp - rgb[c] * rgb[c];
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) v[3 + c] = aux[c];
    if (LAYERS) {
#pragma unroll
      for (int c = 0; c < 6; ++c) v[9 + c] = tone(lay[c]);
      v[15] = log1pf(fminf(fmaxf(var * (1.0f / 3.0f), 0.0f), 1.0e4f));
    } else {
      v[9] = log1pf(fmaxf(aux[LAYERS ? 0 : 6], 0.0f));
#pragma unroll
      for (int c = 10; c < 16; ++c) v[c] = 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
      o[k] = u32x4{f2bf2(v[8 * k], v[8 * k + 1]), f2bf2(v[8 * k + 2], v[8 * k + 3]),
                   f2bf2(v[8 * k + 4], v[8 * k + 5]), f2bf2(v[8 * k + 6], v[8 * k + 7])};
  }
};

// The two input convs and what precedes them in one launch: blocks 0 .. nhr - 1
// preprocess and convolve tiles of the HRLS image (16 channels), the others tiles
// of the LRHS image (log1p RGB and 5 zeros: 8 channels), each to 64 channels with
// bias and ReLU.  A block of 4 waves owns 32 x 16 pixels: the preprocessed tile with
// its zero halo goes to LDS (pitch 24 channels for 16: 16-byte reads of 8 lanes
// hit all banks), each wave computes 4 rows x 2 column tiles x 64 channels with
// all weights in registers (5 or 3 K steps; K index tap CIN + c, a K step spans 2
// or 4 taps).  Row i of M tile j holds channel 16 (i / 4) + 4 j + i % 4, so that
// a lane has 16 consecutive channels of a pixel: 16-byte stores.
// Writing the 64-channel result bounds it (118 MB at 720p, 25 us at the rate of
// a copy).  A preprocessing pass, then one conv launch per image, both operands
// of every MFMA from LDS, took 17 + 99 + 8 us; one launch takes 50.
// xh / xl: also store the preprocessed images (training reads them again).
constexpr int IN_W = 32, IN_H = 16, IN_TW = IN_W + 2, IN_PX = IN_TW * (IN_H + 2);
constexpr int IN_CNT = (IN_PX + 255) / 256;

template <int CIN>
__device__ __forceinline__ void input_conv(const uint16_t* tile, const uint16_t* w,
                                           const float* bias, uint16_t* out, int b, int H, int W,
                                           int x0, int y0) {
  constexpr int KS = (9 * CIN + 31) / 32, PITCH = CIN == 16 ? 24 : CIN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = lane >> 4, li = lane & 15;
  bf16x8 Wt[KS][4];
  const auto wb = buf(w);
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j)  // row li / 4 of 16 channels, 4 j + li % 4 within
      Wt[s][j] = __builtin_bit_cast(
          bf16x8, buf_ld16(wb, ((li >> 2) * KS * 64 + kq * 16 + 4 * j + (li & 3)) * 16 + s * 1024));
  float bs[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) bs[q] = bias[16 * kq + q];
  // offset of this lane's operand of K step s: tap (32 s + 8 kq) / CIN
  int to[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = 32 * s + 8 * kq, tap = min(k / CIN, 8), c = k & (CIN - 1);
    const int dy = tap / 3, dx = tap - dy * 3;
    to[s] = (dy * IN_TW + dx + li) * PITCH + c;
  }
  const bool pad = 32 * (KS - 1) + 8 * kq >= 9 * CIN;  // the last K step's zero padding
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int row = 4 * wave + (t >> 1), col = 16 * (t & 1);
    const uint16_t* tp = tile + (row * IN_TW + col) * PITCH;
    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bf16x8 P = ld8(tp + to[s]);
      if (s == KS - 1 && pad) P = zero8();
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wt[s][j], P, acc[j], 0, 0, 0);
    }
    const int y = y0 + row, x = x0 + col + li;
    if (y < H && x < W) {
      uint32_t h[8];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          h[2 * j + q] = f2bf2(fmaxf(acc[j][2 * q] + bs[4 * j + 2 * q], 0.0f),
                               fmaxf(acc[j][2 * q + 1] + bs[4 * j + 2 * q + 1], 0.0f));
      u32x4* o = reinterpret_cast<u32x4*>(out + (((size_t)b * H + y) * W + x) * NET_FEAT + 16 * kq);
      o[0] = u32x4{h[0], h[1], h[2], h[3]};
      o[1] = u32x4{h[4], h[5], h[6], h[7]};
    }
  }
}

template <bool LAYERS>
__global__ __launch_bounds__(256) void k_input(InputArgs p) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[IN_PX * 24];
  const bool hr = (int)blockIdx.x < p.nhr;
  const int W = hr ? p.W : p.w, H = hr ? p.H : p.h;
  const int tx = (W + IN_W - 1) / IN_W, ty = (H + IN_H - 1) / IN_H;
  int t = hr ? blockIdx.x : blockIdx.x - p.nhr;
  const int x0 = t % tx * IN_W;
  t /= tx;
  const int y0 = t % ty * IN_H, b = t / ty;
  int64_t at[IN_CNT];  // the pixel's index in its image batch, -1 outside
  bool own[IN_CNT];    // inside the block's own tile
#pragma unroll
  for (int u = 0; u < IN_CNT; ++u) {
    const int i = threadIdx.x + u * 256, r = i / IN_TW, c = i - r * IN_TW;
    const int y = y0 - 1 + r, x = x0 - 1 + c;
    const bool in = i < IN_PX && (unsigned)y < (unsigned)H && (unsigned)x < (unsigned)W;
    at[u] = in ? ((int64_t)b * H + y) * W + x : -1;
    own[u] = in && r >= 1 && r <= IN_H && c >= 1 && c <= IN_W;
  }
  if (hr) {
    HrPixel<LAYERS> px[IN_CNT];
#pragma unroll
    for (int u = 0; u < IN_CNT; ++u)
      if (at[u] >= 0) px[u].load(p, at[u]);
#pragma unroll
    for (int u = 0; u < IN_CNT; ++u) {
      const int i = threadIdx.x + u * 256;
      u32x4 o[2] = {u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}};
      if (at[u] >= 0) px[u].pack(p, o);
      if (i < IN_PX) {
        u32x4* d = reinterpret_cast<u32x4*>(tile + i * 24);
        d[0] = o[0];
        d[1] = o[1];
      }
      if (p.xh && own[u]) {
        u32x4* d = reinterpret_cast<u32x4*>(p.xh + 16 * at[u]);
        d[0] = o[0];
        d[1] = o[1];
      }
    }
    input_conv<16>(tile, p.wh, p.bh, p.h0, b, H, W, x0, y0);
  } else {
#pragma unroll
    for (int u = 0; u < IN_CNT; ++u) {
      const int i = threadIdx.x + u * 256;
      u32x4 o = u32x4{0, 0, 0, 0};
      if (at[u] >= 0) {
        const float* s = p.lr + 3 * at[u];
        o = u32x4{f2bf2(tone(s[0]), tone(s[1])), f2bf2(tone(s[2]), 0.0f), 0, 0};
      }
      if (i < IN_PX) *reinterpret_cast<u32x4*>(tile + i * 8) = o;
      if (p.xl && own[u]) *reinterpret_cast<u32x4*>(p.xl + 8 * at[u]) = o;
    }
    input_conv<8>(tile, p.wl, p.bl, p.fl, b, H, W, x0, y0);
  }
}

// One tile of k_pack_all: 16 rows x 32 channels (of the padded cinp) x all taps.  The
// master's weights of a row and consecutive channels (t = 0), or of a column and
// consecutive rows (t = 1), lie together: they are read in order into LDS and written in
// the order of the packed layout, 4 bytes a lane.
constexpr int PK_ROWS = 16, PK_COLS = 32;
template <int TAPS>
__device__ __forceinline__ void pack_tile(const PackJob& J, int tile, const float* __restrict__ w,
                                          uint16_t* __restrict__ out, float* lds) {
  const int nc = (J.cinp + PK_COLS - 1) / PK_COLS, rt = tile / nc, c0 = (tile - rt * nc) * PK_COLS;
  const int r0 = rt * PK_ROWS;
  // runs of consecutive weights in the master, and their pitch in LDS
  const int runs = J.t ? PK_COLS : PK_ROWS;
  const int len = (J.t ? PK_ROWS : PK_COLS) * TAPS, pitch = len + 1;
  const int run0 = J.t ? c0 : r0, in0 = J.t ? r0 : c0;  // first output / input channel
  const int have = min(len, (J.cin - in0) * TAPS);
  for (int u = threadIdx.x >> 6; u < runs; u += 4) {
    const int n = run0 + u;
    const float* src = w + ((size_t)n * J.cin + in0) * TAPS;
    const int m = n < J.cout ? have : 0;
    for (int k = threadIdx.x & 63; k < len; k += 64) lds[u * pitch + k] = k < m ? src[k] : 0.0f;
  }
  __syncthreads();
  // place of K index k (even) of row r0 + row
  const auto at = [&](int row, int k) {
    return J.frag ? (size_t)r0 * J.kp + (k >> 5) * 512 + (((k >> 3) & 3) * 16 + row) * 8 + (k & 7)
                  : (size_t)(r0 + row) * J.kp + k;
  };
  const int cols = min(PK_COLS, J.cinp - c0);
#pragma unroll
  for (int tap = 0; tap < TAPS; ++tap) {
    const int f = threadIdx.x;  // two channels of a row
    const int row = J.frag ? (f >> 2) & 15 : f >> 4;
    const int col = J.frag ? (f >> 6) * 8 + (f & 3) * 2 : (f & 15) * 2;
    if (col >= cols) continue;
    const float* v = lds + (J.t ? col * pitch + row * TAPS + TAPS - 1 - tap
                                : row * pitch + col * TAPS + tap);
    *reinterpret_cast<uint32_t*>(out + at(row, tap * J.cinp + c0 + col)) =
        f2bf2(v[0], v[J.t ? pitch : TAPS]);
  }
  if (c0 + PK_COLS >= J.cinp) {  // zeros from the last tap to kp
    const int pad = (J.kp - TAPS * J.cinp) / 2;
    for (int f = threadIdx.x; f < PK_ROWS * pad; f += 256) {
      const int row = f / pad, k = TAPS * J.cinp + 2 * (f - row * pad);
      *reinterpret_cast<uint32_t*>(out + at(row, k)) = 0u;
    }
  }
}

// BF16 weight packing of every layer in one launch (master layout
// [cout][cin][k][k]), a block per tile; tile i belongs to the last job whose begin is <= i.
// t = 0: wp[n][tap cin_p + c] = W[n][c][tap], the forward convs' B operand.
// t = 1: wt[c][tap' cinp_t + n] = W[n][c][taps - 1 - tap'], the data-gradient
// conv (flipped taps, input and output channels swapped).  Padding is zero.
// Forward layers of a multiple of 64 output channels (all but the reconstruction convs)
// are stored in fragment order, which k_conv3_rw, k_input and k_fuse read, and so are the
// transposed 3x3 layers of a multiple of 64 channels on both sides; the others row by row.
// Bound by memory, 6 bytes a weight and direction: 2.7 M and 11.8 M packed weights (16
// blocks, dense groups) 26 -> 13 us and 96 -> 24; a thread per weight read the master in
// steps of a kernel's taps.
__global__ __launch_bounds__(256) void k_pack_all(const float* __restrict__ wm,
                                                  const PackJob* __restrict__ jobs, int njobs,
                                                  uint16_t* __restrict__ packed,
                                                  uint16_t* __restrict__ packed_t) {
  __shared__ float lds[PK_COLS * (PK_ROWS * 9 + 1)];
  const int64_t i = blockIdx.x;
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (jobs[mid].begin <= i) lo = mid;
    else hi = mid - 1;
  }
  const PackJob J = jobs[lo];
  uint16_t* out = (J.t ? packed_t : packed) + J.out_off;
  const int tile = (int)(i - J.begin);
  if (J.ksz == 3) pack_tile<9>(J, tile, wm + J.w_off, out, lds);
  else pack_tile<1>(J, tile, wm + J.w_off, out, lds);
}

// He-uniform initialisation (fan-in), Philox4x32-10 with tag 2; biases 0.
__global__ __launch_bounds__(256) void k_init(float* __restrict__ dst, int64_t nw, int64_t nb,
                                              int64_t first, float bound, uint32_t k0,
                                              uint32_t k1) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nw) {
    const int64_t g = first + i;
    const uint4 r = philox4x32_10(make_uint4((uint32_t)g, (uint32_t)(g >> 32), 0u, 2u), k0, k1);
    dst[i] = (2.0f * unit24(r.x) - 1.0f) * bound;
  } else if (i < nw + nb) {
    dst[i] = 0.0f;
  }
}

// Weight gradient on the matrix cores, split over pixels: part[s][n][col] = sum
// over the pixels of split s of dY[p][n] X[p + off(tap)][c], col = tap cin_p + c
// (the packed K layout).  The pixel is the MFMA's K index: lane (i, kq) of a
// wave reads, for the pixels p0 + 8 kq + e (e < 8) of each 32-pixel step, RN
// channels of dY and QX columns of X with one load each, and re-packs the
// 16-bit halves into operands: dY operand c maps row i to channel n0 + RN i + c
// (RN = 1: channel n0 + i), X operand d maps column i to col0 + QX i + d.  No LDS
// staging and no barrier in the loop; the next step's loads are issued before
// this step's MFMAs.  The 4 waves of a workgroup take consecutive quarters of
// the split's pixels and their tiles are summed in LDS in wave order
// (deterministic).  The first column block also sums dY, the bias gradient.
// VIEW: how the lane finds X (WgView).
template <int W>
struct Dw {
  uint32_t v[W];
};

template <int W>
__device__ __forceinline__ Dw<W> ldw(const uint16_t* p) {
  Dw<W> r;
  if constexpr (W == 1) {
    r.v[0] = *reinterpret_cast<const uint32_t*>(p);
  } else if constexpr (W == 2) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    r.v[0] = u.x;
    r.v[1] = u.y;
  } else {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    r.v[0] = u.x;
    r.v[1] = u.y;
    r.v[2] = u.z;
    r.v[3] = u.w;
  }
  return r;
}

template <int W>
__device__ __forceinline__ Dw<W> zdw() {
  Dw<W> r;
#pragma unroll
  for (int k = 0; k < W; ++k) r.v[k] = 0u;
  return r;
}

// The 16-bit half at bit `sh` (0 or 16) of word u of pixels 2k and 2k+1, packed
// into one operand word (pixel 2k low).
__device__ __forceinline__ uint32_t pair16(uint32_t lo, uint32_t hi, int sh) {
  return ((lo >> sh) & 0xffffu) | ((hi >> sh) << 16);
}

// Input views of the weight gradient: a plain tensor or one shuffled by a power of two,
// with rows of a multiple of 8 pixels, so that the 8 pixels a lane takes share one image
// row and a shift or two give their places; any other view, pixel by pixel (view_ptr).
// Measured, view_ptr against shifts, 16 images of 128 x 128: reconstruction 93 / 52 us
// (80 channels), 85 / 40 (64), second upscaling step 147 / 117, fuse 32 / 22.
enum WgView { WG_ANY = 0, WG_PLAIN = 1, WG_POW2 = 2 };

// One channel's place in a view whose shuffle factor is a power of two: pixel (b, y, x)
// is at base + b sb + (y >> l) sy + (y & msk) sy2 + (x >> l) sx + (x & msk) sx2 (as
// view_ptr gives it).
struct LaneView {
  const uint16_t* base;
  int64_t sb, sy;
  int sy2, sx, sx2, l, msk;
  __device__ __forceinline__ const uint16_t* row(int b, int y) const {
    return base + b * sb + (y >> l) * sy + (y & msk) * sy2;
  }
  __device__ __forceinline__ int col(int x) const { return (x >> l) * sx + (x & msk) * sx2; }
};
__device__ __forceinline__ LaneView lane_view(const ConvArgs& p, int c) {
  LaneView v{p.a + c, 0, 0, 0, p.ca, 0, 0, 0};
  int rows = p.H, cols = p.W;
  if (p.mode == VIEW_CONCAT_UNSHUFFLE && c >= p.ca) {
    const int cc = c - p.ca, q = cc / p.cb;
    int I, J;
    unshuffle_slot(q, p.r, p.dsf, I, J);
    v.base = p.b + ((int64_t)I * p.W * p.r + J) * p.cb + (cc - q * p.cb);
    v.sx = p.r * p.cb;
    v.sy = (int64_t)p.W * p.r * p.r * p.cb;
    v.sb = p.H * v.sy;
    return v;
  }
  if (p.mode == VIEW_SHUFFLE_CONCAT) {
    if (c < p.c0) {
      v.l = 31 - __clz(p.r);
      v.msk = p.r - 1;
      v.sy2 = p.r * p.c0;
      v.sx2 = p.c0;
      rows >>= v.l;
      cols >>= v.l;
    } else {
      v.base = p.b + (c - p.c0);
      v.sx = p.cb;
    }
  }
  v.sy = (int64_t)cols * v.sx;
  v.sb = rows * v.sy;
  return v;
}

template <int RN, int QX>
constexpr int wgrad_lds() {  // floats of LDS that a block takes
  return 4 * 4 * RN * 16 * QX + 4 * 16 * RN;
}

// Block (bx, by, bz), with wgrad_lds() floats of LDS from `lds` on.
template <int RN, int QX, int VIEW>
__device__ __forceinline__ void wgrad_block(const WgradArgs& a, float* lds, int bx, int by, int bz) {
  constexpr int NN = 16 * RN, NC = 16 * QX;
  constexpr int YW = RN == 1 ? 1 : RN / 2, XW = QX / 2;  // dwords per pixel
  auto red = reinterpret_cast<float(*)[4 * RN * NC]>(lds);
  auto bred = reinterpret_cast<float(*)[NN]>(lds + 4 * 4 * RN * NC);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, kq = lane >> 4;
  const int col0 = bx * NC, n0 = by * NN;
  const ConvArgs& x = a.x;
  const int quarter = a.chunk >> 2;
  const int pw0 = bz * a.chunk + wave * quarter;
  const int pw1 = min(a.npix, pw0 + quarter);
  // this lane's X columns: QX channels cx.. of tap `tap` (one tap: cin_p % 8 == 0)
  const int colx = col0 + QX * i;
  const int tapx = colx / x.cin_p, cx = colx - tapx * x.cin_p;
  const bool xon = colx < x.kp && tapx < x.taps;
  const int ty = x.taps == 9 ? tapx / 3 - 1 : 0, tx = x.taps == 9 ? tapx % 3 - 1 : 0;
  // this lane's dY channels (RN = 1: the word holding channel n0 + i)
  const int ny = RN == 1 ? ((n0 + i) & ~1) : n0 + RN * i;
  const bool yon = (RN == 1 ? n0 + i : ny) < a.dy_stride;
  const int ysh = RN == 1 ? 16 * ((n0 + i) & 1) : 0;
  const bool bias_blk = bx == 0 && a.bpart;

  const LaneView xv = VIEW == WG_POW2 ? lane_view(x, xon ? cx : 0) : LaneView{};
  auto load_step = [&](int pk, Dw<YW>(&yd)[8], Dw<XW>(&xd)[8]) {
    const int pp0 = pk + 8 * kq;
    const uint16_t* yp = a.dy + (int64_t)pp0 * a.dy_stride + ny;
    if constexpr (VIEW != WG_ANY) {
      const bool gv = pp0 < pw1;  // W % 8 == 0: the 8 pixels are valid together
      const int t = pp0 / x.W, x0 = pp0 - t * x.W + tx, pb = t / x.H, y = t - pb * x.H + ty;
      const bool rowv = gv && xon && (unsigned)y < (unsigned)x.H;
      const uint16_t* xp = VIEW == WG_POW2
                               ? xv.row(pb, y)
                               : x.a + ((int64_t)pp0 + ty * x.W + tx) * x.ca + cx;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool in = rowv && (unsigned)(x0 + e) < (unsigned)x.W;
        xd[e] = in ? ldw<XW>(xp + (VIEW == WG_POW2 ? xv.col(x0 + e) : e * x.ca)) : zdw<XW>();
        yd[e] = (gv && yon) ? ldw<YW>(yp + (int64_t)e * a.dy_stride) : zdw<YW>();
      }
    } else {
      int px = pp0 % x.W;
      const int t = pp0 / x.W;
      int py = t % x.H, pb = t / x.H;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool v = pp0 + e < pw1;
        const uint16_t* q = (v && xon) ? view_ptr(x, pb, py + ty, px + tx, cx) : nullptr;
        xd[e] = q ? ldw<XW>(q) : zdw<XW>();
        yd[e] = (v && yon) ? ldw<YW>(yp + (int64_t)e * a.dy_stride) : zdw<YW>();
        ++px;
        const bool wrap = px == x.W;
        px = wrap ? 0 : px;
        py += wrap;
        const bool wrap2 = py == x.H;
        py = wrap2 ? 0 : py;
        pb += wrap2;
      }
    }
  };

  f32x4 acc[RN][QX];
#pragma unroll
  for (int c = 0; c < RN; ++c)
#pragma unroll
    for (int d = 0; d < QX; ++d) acc[c][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bs[RN];
#pragma unroll
  for (int c = 0; c < RN; ++c) bs[c] = 0.0f;

  Dw<YW> yd[8];
  Dw<XW> xd[8];
  if (pw0 < pw1) load_step(pw0, yd, xd);
  for (int pk = pw0; pk < pw1; pk += 32) {
    Dw<YW> yn[8];
    Dw<XW> xn[8];
    if (pk + 32 < pw1) load_step(pk + 32, yn, xn);
    bf16x8 A[RN], Bv[QX];
#pragma unroll
    for (int c = 0; c < RN; ++c) {
      const int u = RN == 1 ? 0 : c >> 1, sh = RN == 1 ? ysh : 16 * (c & 1);
      uint4 w;
      w.x = pair16(yd[0].v[u], yd[1].v[u], sh);
      w.y = pair16(yd[2].v[u], yd[3].v[u], sh);
      w.z = pair16(yd[4].v[u], yd[5].v[u], sh);
      w.w = pair16(yd[6].v[u], yd[7].v[u], sh);
      A[c] = __builtin_bit_cast(bf16x8, w);
      if (bias_blk) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bs[c] += __uint_as_float(((yd[e].v[u] >> sh) & 0xffffu) << 16);
      }
    }
#pragma unroll
    for (int d = 0; d < QX; ++d) {
      const int u = d >> 1, sh = 16 * (d & 1);
      uint4 w;
      w.x = pair16(xd[0].v[u], xd[1].v[u], sh);
      w.y = pair16(xd[2].v[u], xd[3].v[u], sh);
      w.z = pair16(xd[4].v[u], xd[5].v[u], sh);
      w.w = pair16(xd[6].v[u], xd[7].v[u], sh);
      Bv[d] = __builtin_bit_cast(bf16x8, w);
    }
#pragma unroll
    for (int c = 0; c < RN; ++c)
#pragma unroll
      for (int d = 0; d < QX; ++d)
        acc[c][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[c], Bv[d], acc[c][d], 0, 0, 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      yd[e] = yn[e];
      xd[e] = xn[e];
    }
  }
  if (bias_blk) {  // over kq (lanes 16 apart), then per wave into LDS
#pragma unroll
    for (int c = 0; c < RN; ++c) {
      bs[c] += __shfl_xor(bs[c], 16);
      bs[c] += __shfl_xor(bs[c], 32);
    }
    if (kq == 0) {
#pragma unroll
      for (int c = 0; c < RN; ++c) bred[wave][RN == 1 ? i : RN * i + c] = bs[c];
    }
  }
  // accumulator (c, d) of lane (j, g): rows 4g + v (channel n0 + RN row + c), column j
  // (col0 + QX j + d).  The four waves' tiles are added a quarter (one v) at a time:
  // 4 RN rows, 16 KB of LDS a block instead of 65, so that three blocks share a CU (168
  // registers; a training step of the dense groups 3.71 -> 3.64 ms).
  const int t = threadIdx.x;
  float* out = a.part + ((size_t)bz * a.cout_p + n0) * x.kp + col0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v) __syncthreads();
#pragma unroll
    for (int c = 0; c < RN; ++c) {
      float* row = red[wave] + (RN * kq + c) * NC + QX * i;
#pragma unroll
      for (int d4 = 0; d4 < QX; d4 += 4)
        *reinterpret_cast<float4*>(row + d4) =
            make_float4(acc[c][d4][v], acc[c][d4 + 1][v], acc[c][d4 + 2][v], acc[c][d4 + 3][v]);
    }
    __syncthreads();
    for (int f = t; f < RN * NC; f += 256) {
      const int rl = (4 * f) / NC, cl = (4 * f) % NC;
      if (col0 + cl >= x.kp) continue;
      const int nl = RN * (4 * (rl / RN) + v) + rl % RN;
      const float4 r0 = reinterpret_cast<const float4*>(red[0])[f];
      const float4 r1 = reinterpret_cast<const float4*>(red[1])[f];
      const float4 r2 = reinterpret_cast<const float4*>(red[2])[f];
      const float4 r3 = reinterpret_cast<const float4*>(red[3])[f];
      *reinterpret_cast<float4*>(out + (size_t)nl * x.kp + cl) =
          make_float4(((r0.x + r1.x) + r2.x) + r3.x, ((r0.y + r1.y) + r2.y) + r3.y,
                      ((r0.z + r1.z) + r2.z) + r3.z, ((r0.w + r1.w) + r2.w) + r3.w);
    }
  }
  if (bias_blk && t < NN && n0 + t < a.cout)
    a.bpart[(size_t)bz * a.cout + n0 + t] =
        ((bred[0][t] + bred[1][t]) + bred[2][t]) + bred[3][t];
}

// Sum of v[sp * stride] over the splits: eight independent partial sums
// (split sp into sum sp % 8), so that eight loads are in flight, then added in a
// fixed order.
__device__ __forceinline__ float sum_splits(const float* __restrict__ v, size_t stride,
                                            int splits) {
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int sp = 0;
  for (; sp + 8 <= splits; sp += 8) {
#pragma unroll
    for (int k = 0; k < 8; ++k) s[k] += v[(size_t)(sp + k) * stride];
  }
  for (int k = 0; sp < splits; ++sp, ++k) s[k] += v[(size_t)sp * stride];
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// Sum the split partials in order and scatter into the master gradient layout
// [cout][cin][k][k] followed by the bias.  Threads walk the packed layout
// [n][tap cin_p + c], so that the split partials are read coalesced.
__device__ __forceinline__ void grad_reduce_block(const ReduceArgs& a, int block) {
  const int64_t np = (int64_t)a.cout * a.kp;
  const int64_t i = (int64_t)block * 256 + threadIdx.x;
  if (i < np) {
    const int n = (int)(i / a.kp), col = (int)(i - (int64_t)n * a.kp);
    const int tap = col / a.cin_p, c = col - tap * a.cin_p;
    if (c >= a.cin || tap >= a.ksz * a.ksz) return;
    const int ky = tap / a.ksz, kx = tap - ky * a.ksz;
    a.g[((size_t)(n * a.cin + c) * a.ksz + ky) * a.ksz + kx] =
        sum_splits(a.part + i, (size_t)a.cout_p * a.kp, a.splits);
  } else if (i < np + a.cout) {
    const int n = (int)(i - np);
    a.g[(size_t)a.cout * a.cin * a.ksz * a.ksz + n] =
        sum_splits(a.bpart + n, (size_t)a.cout, a.splits);
  }
}
__global__ __launch_bounds__(256) void k_grad_reduce(ReduceArgs a) {
  grad_reduce_block(a, blockIdx.x);
}

// The blocks of a launch that are a weight gradient's: wx x wy x splits of them.
struct WgradGrid {
  WgradArgs w;
  int wx, wy, n;
};
template <int RN, int QX, int VIEW>
__device__ __forceinline__ void wgrad_block(const WgradGrid& g, float* lds, int i) {
  const int t = i / g.wx;
  wgrad_block<RN, QX, VIEW>(g.w, lds, i - t * g.wx, t % g.wy, t / g.wy);
}

// A weight gradient's partial sums, and the sum of an earlier layer's.
template <int RN, int QX, int VIEW>
__global__ __launch_bounds__(256, 3) void k_wgrad(WgradGrid g, ReduceArgs r) {
  __shared__ __attribute__((aligned(16))) float lds[wgrad_lds<RN, QX>()];
  const int i = blockIdx.x;
  if (i < g.n) wgrad_block<RN, QX, VIEW>(g, lds, i);
  else grad_reduce_block(r, i - g.n);
}

// k_layer_bwd for the layers whose data gradient is a direct conv through a view (the
// reconstruction, the later upscaling steps, the fuse conv): gx column blocks, nd in all.
// Measured (16 images of 128 x 128) against the launches one by one: fuse 63 against
// 51 + 22 + 5 us, reconstruction 82 against 34 + 52 (80 channels; both fill the chip),
// 60 against 30 + 40 (64), second upscaling step 178 against 78 + 117.
template <int MODE, int RN, int QX>
__global__ __launch_bounds__(256, 3) void k_layer_bwd_view(ConvArgs p, BwdEpi e, int gx, int nd,
                                                           WgradGrid g, ReduceArgs r) {
  __shared__ __attribute__((aligned(16))) float lds[wgrad_lds<RN, QX>()];
  int i = blockIdx.x;
  // the longer blocks first: a later upscaling step's data gradient sums K = 2304
  constexpr bool DG_FIRST = MODE == EPI_REC_SPLIT && RN == 4;
  const int wg0 = DG_FIRST ? nd : 0, dg0 = DG_FIRST ? 0 : g.n;
  if (i >= nd + g.n) {
    grad_reduce_block(r, i - nd - g.n);
  } else if ((unsigned)(i - wg0) < (unsigned)g.n) {
    wgrad_block<RN, QX, WG_POW2>(g, lds, i - wg0);
  } else {
    i -= dg0;
    const int t = i / gx;
    dgrad_block<4, MODE>(p, e, i - t * gx, t);
  }
}

// One layer of the backward pass in one launch: the data gradient (conv3_rw_block on
// 16 x 8 tiles), the weight gradient's partial sums, which need nothing of it, and the
// sum over the splits of the layer done before, whose partial sums lie in the other half
// of the scratch.  Each is bound by latency -- a few dependent steps per block and one
// to four blocks per CU -- so side by side they take little more than the longest.  The
// weight gradient's blocks, the longest, come first (a layer of 64 channels 15.1 -> 14.3
// us, of 256 31 -> 27.7).  Measured, one training step of 16 images of 128 x 128: 1.58 ->
// 1.30 ms (16 blocks: 24 -> 15 us a layer), 3.64 -> 3.19 ms (dense groups).
// Three blocks a CU leave 168 registers: 3 spilled with 64 channels, 16 with more, 24 in
// k_layer_bwd_view's 4 x 4 tiles; two blocks, without spills, take 4.39 against 4.37 ms for
// four steps of the 16-block network, 11.47 against 11.16 of the dense groups.
// The rule is the small plan's of k_conv3_rw (128 tiles).  The launch still pays above it:
// a step of images of 128 x 128 (4 tiles each) in separate launches on the large plan / in
// one launch on the small plan, 16 images 1451 / 992 us (dense groups 3656 / 2428), 32
// images 1928 / 1537 (4679 / 3802), 64 images 2832 / 2698 (6928 / 6650);
// mrs_tuning.conv_small_tiles moves the line.
template <bool MULTI>
__global__ __launch_bounds__(256, 3) void k_layer_bwd(ConvArgs p, int cout_p, int nsplit,
                                                      BwdEpi be, int gx, int gy, int nd,
                                                      WgradGrid g, ReduceArgs r) {
  constexpr int BYTES_D = 2 * rw_lds<4, 2, MULTI>(), BYTES_W = 4 * wgrad_lds<4, 4>();
  __shared__ __attribute__((aligned(16))) char lds[BYTES_D > BYTES_W ? BYTES_D : BYTES_W];
  int i = blockIdx.x;
  if (i < g.n) {
    wgrad_block<4, 4, WG_PLAIN>(g, reinterpret_cast<float*>(lds), i);
  } else if ((i -= g.n) < nd) {
    const int t = i / gx;
    conv3_rw_block<4, 2, 2, MULTI, RW_DG>(p, cout_p, nsplit, be, reinterpret_cast<uint16_t*>(lds),
                                          i - t * gx, t % gy, t / gy);
  } else {
    grad_reduce_block(r, i - nd);
  }
}

// Loss pieces (t clipped to [0, 100], d = y - t).  beta <= 0: L1, FP64 partial
// sums of |d| per block and the gradient sign(d) / N.  beta > 0: the robust loss
// of Sec. 4, partial sums of |d| / (beta + |d|) in FP64 and the gradient
// sign(d) beta / (beta + |d|)^2 / N.  sign(0) = 0; the gradient is stored as
// BF16 in an 8-channel padded tensor.
__global__ __launch_bounds__(256) void k_l1(const float* __restrict__ y,
                                            const float* __restrict__ tgt, int64_t npix,
                                            double inv_n, float beta, double* __restrict__ part,
                                            uint16_t* __restrict__ g8) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < npix;
       p += (int64_t)gridDim.x * 256) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    for (int c = 0; c < 3; ++c) {
      // targets are clipped to [0, 100] like the training data (fireflies, Sec. 3.2)
      const float d = y[3 * p + c] - fminf(fmaxf(tgt[3 * p + c], 0.0f), 100.0f);
      const double ad = fabs((double)d);
      const float gsgn = d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f);
      float gv;
      if (beta > 0.0f) {
        s += ad / ((double)beta + ad);
        const float den = beta + fabsf(d);
        gv = gsgn * (beta / (den * den)) * (float)inv_n;
      } else {
        s += ad;
        gv = gsgn * (float)inv_n;
      }
      const uint32_t h = f2bf(gv);
      w[c >> 1] |= h << (16 * (c & 1));
    }
    *reinterpret_cast<uint4*>(g8 + 8 * p) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void k_l1_final(const double* __restrict__ part, int nparts,
                                                  double inv_n, double* __restrict__ loss) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int b = threadIdx.x; b < nparts; b += 256) s += part[b];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if ((int)threadIdx.x < k) sh[threadIdx.x] += sh[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = sh[0] * inv_n;
}

// A caller-supplied output gradient (FP32 [P][3]) as BF16 in the 8-channel
// padded layout the backward pass reads.
__global__ __launch_bounds__(256) void k_grad_in(const float* __restrict__ gout, int64_t npix,
                                                 uint16_t* __restrict__ g8) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= npix) return;
  const uint32_t w0 = (uint32_t)f2bf(gout[3 * p]) | ((uint32_t)f2bf(gout[3 * p + 1]) << 16);
  const uint32_t w1 = (uint32_t)f2bf(gout[3 * p + 2]);
  *reinterpret_cast<uint4*>(g8 + 8 * p) = make_uint4(w0, w1, 0u, 0u);
}

// Plain SGD on the FP32 masters (the paper's optimiser): w -= lr g.
__global__ __launch_bounds__(256) void k_sgd(float* __restrict__ w, const float* __restrict__ g,
                                             int64_t n, float lr) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) w[i] -= lr * g[i];
}

// Adam (Kingma & Ba 2015, Algorithm 1) on the FP32 masters; c1 = 1 - b1^t,
// c2 = 1 - b2^t are the bias corrections of step t.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ w, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v,
                                              int64_t n, float lr, float b1, float b2, float eps,
                                              float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

namespace {
inline unsigned cdiv64(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }
}  // namespace

namespace {
std::atomic<int64_t> g_conv_launches[MRS_NUM_CONV_KINDS];
inline void count_conv(int kind) { g_conv_launches[kind].fetch_add(1, std::memory_order_relaxed); }
}  // namespace

void launch_dgrad(const ConvArgs& a, const BwdEpi& e, int cout_p, hipStream_t st) {
  // 3x3 data gradients of 64-channel slices: the same kernel and tile plans as
  // the forward convs
  const int64_t tiles = (int64_t)((a.W + 15) / 16) * ((a.H + 15) / 16) * a.B;
  if (tiles < conv_small_tiles() && try_conv3_rw<4, 2, 2, RW_DG>(a, cout_p, cout_p / 32, st, &e))
    return count_conv(8);
  if (try_conv3_rw<8, 2, 4, RW_DG>(a, cout_p, 1, st, &e)) return count_conv(9);
  const int64_t M = (int64_t)a.B * a.H * a.W;
  const unsigned gx = cdiv64(M, 128);
  const dim3 g4(gx, cout_p / 64), g1(gx, cout_p / 16);
  const auto run = [&](auto k4, auto k1) {
    if (cout_p >= 64) k4<<<g4, 256, 0, st>>>(a, e);
    else k1<<<g1, 256, 0, st>>>(a, e);
  };
  switch (e.mode) {
    case EPI_PLAIN: run(k_dgrad<4, EPI_PLAIN>, k_dgrad<1, EPI_PLAIN>); break;
    case EPI_REC_SPLIT: run(k_dgrad<4, EPI_REC_SPLIT>, k_dgrad<1, EPI_REC_SPLIT>); break;
    case EPI_FUSE_SPLIT: run(k_dgrad<4, EPI_FUSE_SPLIT>, k_dgrad<1, EPI_FUSE_SPLIT>); break;
    default: run(k_dgrad<4, EPI_DENSE>, k_dgrad<1, EPI_DENSE>);
  }
}

// Weight-gradient tile per workgroup: 64 x 64 (RN 4, QX 4) for 64 or more
// output channels, else 16 x 128 (RN 1, QX 8).
namespace {
inline int wgrad_nc(int cout_p) { return cout_p >= 64 ? 64 : 128; }
inline int wgrad_nn(int cout_p) { return cout_p >= 64 ? 64 : 16; }
}  // namespace

int wgrad_splits(int64_t npix, int kp, int cout_p, int& chunk) {
  // about 1024 workgroups over the tiles, at most 128 splits, and at least 4
  // steps of 32 pixels per wave (512 pixels per workgroup)
  const int64_t tiles = (int64_t)cdiv64(kp, wgrad_nc(cout_p)) * (cout_p / wgrad_nn(cout_p));
  const int64_t s = std::max<int64_t>(1, std::min<int64_t>(128, (1024 + tiles - 1) / tiles));
  const int64_t per = std::max<int64_t>(512, (npix + s - 1) / s);
  chunk = (int)((per + 127) / 128 * 128);
  return (int)std::max<int64_t>(1, (npix + chunk - 1) / chunk);
}

ReduceArgs reduce_args(const WgradArgs& w, int splits, const NetLayer& L, float* g) {
  return ReduceArgs{w.part, w.bpart, splits, L.cout, L.cin, L.k, L.cin_p, L.kp, L.cout_p, g};
}

namespace {
unsigned reduce_blocks(const ReduceArgs& r) {
  return r.part ? cdiv64((int64_t)r.cout * r.kp + r.cout, 256) : 0u;
}
WgradGrid wgrad_grid(const WgradArgs& w, int splits) {
  const int wx = (int)cdiv64(w.x.kp, wgrad_nc(w.cout_p)), wy = w.cout_p / wgrad_nn(w.cout_p);
  return WgradGrid{w, wx, wy, wx * wy * splits};
}
int wgrad_view(const ConvArgs& x) {
  return x.W % 8 ? WG_ANY
         : x.mode == VIEW_PLAIN ? WG_PLAIN
         : (x.r & (x.r - 1)) == 0 ? WG_POW2 : WG_ANY;
}
}  // namespace

void launch_grad_reduce(const ReduceArgs& r, hipStream_t st) {
  if (r.part) k_grad_reduce<<<reduce_blocks(r), 256, 0, st>>>(r);
}

void launch_wgrad(const WgradArgs& w, int splits, const ReduceArgs& r, hipStream_t st) {
  const WgradGrid g = wgrad_grid(w, splits);
  const auto run = [&](auto k44, auto k18) {
    (w.cout_p >= 64 ? k44 : k18)<<<g.n + reduce_blocks(r), 256, 0, st>>>(g, r);
  };
  switch (wgrad_view(w.x)) {
    case WG_PLAIN: run(k_wgrad<4, 4, WG_PLAIN>, k_wgrad<1, 8, WG_PLAIN>); break;
    case WG_POW2: run(k_wgrad<4, 4, WG_POW2>, k_wgrad<1, 8, WG_POW2>); break;
    default: run(k_wgrad<4, 4, WG_ANY>, k_wgrad<1, 8, WG_ANY>);
  }
}

bool launch_layer_bwd(const ConvArgs& a, const BwdEpi& e, int cout_p, const WgradArgs& w,
                      int splits, const ReduceArgs& r, hipStream_t st) {
  const int64_t tiles = (int64_t)((a.W + 15) / 16) * ((a.H + 15) / 16) * a.B;
  const int nsplit = cout_p / 32, view = wgrad_view(w.x);
  const WgradGrid g = wgrad_grid(w, splits);
  if (tiles < conv_small_tiles() && w.cout_p >= 64 && view == WG_PLAIN &&
      conv3_rw_fits<4, 2, 2, RW_DG>(a, cout_p, nsplit, &e)) {
    const int gx = (a.W + 15) / 16, gy = (a.H + 7) / 8, nd = gx * gy * a.B * nsplit;
    auto kern = a.cin_p > 64 ? k_layer_bwd<true> : k_layer_bwd<false>;
    kern<<<nd + g.n + reduce_blocks(r), 256, 0, st>>>(a, cout_p, nsplit, e, gx, gy, nd, g, r);
    count_conv(8);
    return true;
  }
  if (view == WG_POW2 && cout_p >= 64 &&
      (e.mode == EPI_REC_SPLIT || (e.mode == EPI_FUSE_SPLIT && w.cout_p >= 64))) {
    const int gx = (int)cdiv64((int64_t)a.B * a.H * a.W, 128), nd = gx * (cout_p / 64);
    auto kern = e.mode == EPI_FUSE_SPLIT ? k_layer_bwd_view<EPI_FUSE_SPLIT, 4, 4>
                : w.cout_p >= 64 ? k_layer_bwd_view<EPI_REC_SPLIT, 4, 4>
                                 : k_layer_bwd_view<EPI_REC_SPLIT, 1, 8>;
    kern<<<nd + g.n + reduce_blocks(r), 256, 0, st>>>(a, e, gx, nd, g, r);
    return true;
  }
  return false;
}

void launch_out_grad(const OutGrad& o, const float* y, int64_t npix, uint16_t* g8,
                     hipStream_t st) {
  if (o.tgt) {
    const double inv_n = 1.0 / (double)(3 * npix);
    k_l1<<<o.nparts, 256, 0, st>>>(y, o.tgt, npix, inv_n, o.beta, o.part, g8);
    k_l1_final<<<1, 256, 0, st>>>(o.part, o.nparts, inv_n, o.loss);
  } else {
    k_grad_in<<<cdiv64(npix, 256), 256, 0, st>>>(o.gout, npix, g8);
  }
}

void launch_sgd(float* w, const float* g, int64_t n, float lr, hipStream_t st) {
  k_sgd<<<cdiv64(n, 256), 256, 0, st>>>(w, g, n, lr);
}

void launch_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                 float b2, float eps, float c1, float c2, hipStream_t st) {
  k_adam<<<cdiv64(n, 256), 256, 0, st>>>(w, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

void conv_launch_counts(int64_t* out, bool reset) {
  for (int i = 0; i < MRS_NUM_CONV_KINDS; ++i)
    out[i] = reset ? g_conv_launches[i].exchange(0) : g_conv_launches[i].load();
}

bool launch_res_block(const ConvArgs& a, const ConvArgs& b, hipStream_t st) {
  const auto fits = [](const ConvArgs& p) {
    return p.mode == VIEW_PLAIN && p.taps == 9 && p.cin_p == RB_C && p.kp == RB_KP &&
           p.cout == RB_C && p.frag && (!p.out_f || p.out_f_stride % 4 == 0) &&
           (!p.out_h || p.out_h_stride % 8 == 0) &&
           (int64_t)RB_IN * p.W * std::max(p.ca, RDG_DENSE) * 4 < (int64_t)BUF_OUT;
  };
  if (!fits(a) || !fits(b) || a.ca < RB_C || !a.relu || a.B != b.B || a.H != b.H ||
      a.W != b.W)
    return false;
  k_res_block<<<dim3((a.W + RB_T - 1) / RB_T, (a.H + RB_T - 1) / RB_T, a.B), RB_THREADS, 0,
                st>>>(a, b);
  count_conv(10);
  return true;
}

// Tile plan of a 3x3 conv on k_conv3_rw: 16 x 16 tiles of 8 waves with 64 output
// channels at a time; when such tiles are fewer than mrs_tuning.conv_small_tiles
// (default 128: half of the 256 CUs), 16 x 8 tiles of 4 waves with the output
// channels split over blocks of 32 (two fit a CU at once).  Both plans sum every
// output in the same K order, so the choice changes speed only.  Measured, small
// against large plan, 64 / 128 / 256 input channels: 40 tiles 4.8 / 6.4 / 10.1
// against 7.7 / 10.7 / 19.7 us, 120 tiles 6.1 / 8.9 / 15.9 against 7.9 / 11.0 /
// 21.4, 160 tiles 7.1 / 13.2 / 23.2 against 8.0 / 11.2 / 22.5, 240 tiles (the 720p
// LR image) 10.3 / 16.6 / 29.7 against 8.5 / 11.8 / 24.2.
void launch_conv(const ConvArgs& a, int cout_p, hipStream_t st) {
  const int64_t tiles = (int64_t)((a.W + 15) / 16) * ((a.H + 15) / 16) * a.B;
  if (tiles < conv_small_tiles() &&
      try_conv3_rw<4, 2, 2, RW_FWD>(a, cout_p, cout_p / 32, st, nullptr))
    return count_conv(0);
  if (try_conv3_rw<8, 2, 4, RW_FWD>(a, cout_p, 1, st, nullptr)) return count_conv(1);
  if (try_rec<16, 64, 4>(a, st)) return count_conv(4);
  if (try_rec<64, 0, 2>(a, st)) return count_conv(5);
  if (try_fuse(a, cout_p, st)) return count_conv(6);
  const int64_t M = (int64_t)a.B * a.H * a.W;
  const unsigned gx = cdiv64(M, 128);
  if (cout_p >= 64) {
    k_conv<4><<<dim3(gx, cout_p / 64), 256, 0, st>>>(a);
    count_conv(6);
  } else {
    k_conv<1><<<dim3(gx, cout_p / 16), 256, 0, st>>>(a);
    count_conv(7);
  }
}

void launch_input(const mrs_net* net, int B, int H, int W, const float* hr, const float* aux,
                  const float* lr, uint16_t* xh, uint16_t* xl, uint16_t* h0, uint16_t* fl,
                  hipStream_t st) {
  const NetLayer &Lh = net->layers[0], &Ll = net->layers[1];
  const int s = arch_scale(net->arch);
  InputArgs a;
  a.hr = hr;
  a.aux = aux;
  a.lr = lr;
  a.layers = net->in_layers;
  a.sumsq = net->in_sumsq;
  a.inv_spp = net->in_spp ? 1.0f / (float)net->in_spp : 0.0f;
  a.H = H;
  a.W = W;
  a.h = H / s;
  a.w = W / s;
  a.wh = net->d_packed + Lh.pk_off;
  a.wl = net->d_packed + Ll.pk_off;
  a.bh = net->d_master + Lh.b_off;
  a.bl = net->d_master + Ll.b_off;
  a.xh = xh;
  a.xl = xl;
  a.h0 = h0;
  a.fl = fl;
  const auto tiles = [B](int h, int w) {
    return (int64_t)B * ((h + IN_H - 1) / IN_H) * ((w + IN_W - 1) / IN_W);
  };
  a.nhr = (int)tiles(H, W);
  const unsigned grid = (unsigned)(a.nhr + tiles(a.h, a.w));
  if (arch_has_layers(net->arch)) k_input<true><<<grid, 256, 0, st>>>(a);
  else k_input<false><<<grid, 256, 0, st>>>(a);
  count_conv(2);
  count_conv(3);
}

int64_t pack_tiles(const PackJob& j) {
  return (int64_t)((j.coutp + PK_ROWS - 1) / PK_ROWS) * ((j.cinp + PK_COLS - 1) / PK_COLS);
}

void launch_pack_all(const float* wm, const PackJob* jobs, int njobs, int64_t tiles,
                     uint16_t* packed, uint16_t* packed_t, hipStream_t st) {
  if (tiles > 0)
    k_pack_all<<<(unsigned)tiles, 256, 0, st>>>(wm, jobs, njobs, packed, packed_t);
}

void launch_init(float* dst, const NetLayer& L, uint64_t seed, hipStream_t st) {
  const int64_t nw = (int64_t)L.cout * L.cin * L.k * L.k;
  const float bound = (float)(std::sqrt(6.0 / (double)(L.cin * L.k * L.k)) * L.init_scale);
  k_init<<<cdiv64(nw + L.cout, 256), 256, 0, st>>>(dst, nw, L.cout, (int64_t)L.w_off, bound,
                                                   (uint32_t)seed, (uint32_t)(seed >> 32));
}

}  // namespace mrs
