// Forward and input-gradient 3x3x3 convolutions of the warm-start network on the
// bf16 matrix cores, operand fragments loaded straight from global memory.
//
// Both are out[v][m] = sum over taps j and channels c of w[m][tap_j][c] src[v + off_j][c]:
//   forward:            v an output voxel, centre s v, off = tap - 1;
//   gradient, stride 1: v an input voxel,  centre v,   off = 1 - tap;
//   gradient, stride 2: one problem per parity class of v: an even coordinate
//                       meets tap 1 only, an odd one taps 0 and 2, so a class has
//                       1, 2, 4 or 8 taps instead of 27 (of which the others are
//                       structural zeros: 7/8 of the general kernel's products).
// The weights are the A operand (rows m), 16 voxels the B operand, so a lane ends
// with four consecutive channels of one voxel and stores them at once.
//
// A lane's 8 k-values of B are 16 consecutive bytes of one voxel's channels, so a
// fragment is one buffer load per lane, with an out-of-range offset (which reads
// zero) where the tap leaves the grid: no im2col in LDS, no bounds branches, and a
// voxel's channels are read once per tap for all output channels.  The weights go
// through LDS in fragment order (lane l's 16 bytes at l), four k-steps at a
// time, double-buffered, shared by the block's four wavefronts.  Voxel fragments
// are loaded three steps ahead.
//
// The k order (tap outer, channel inner, 32 per instruction) and the instruction
// are those of k_conv_gemm, so both give the same bits; skipped taps are exact
// zeros there.
#include <algorithm>
#include <utility>

#include "cnn_internal.h"
#include "internal.h"

namespace lddmm_cnn {
namespace {

constexpr int kBlk = 256;          // 4 wavefronts
constexpr int KS = 4;              // k-steps of weights per LDS buffer
constexpr int RING = 4;            // voxel fragments in flight (steps)
static_assert(KS == RING, "one ring slot per unrolled step");

// How a k-step's 32 values map to (tap, channel), by the source's channel count C.
enum { KM_32 = 0, KM_16 = 1, KM_PAIR = 2 };   // C % 32 == 0; C == 16 (two taps); C even

struct Axis {                      // taps along one axis: k = k0 + j kd at offset o0 + j od
  int n, k0, kd, o0, od;
};

struct FragArgs {
  const u16* src;
  const u16* w;
  const float* bias;
  const u16* mask;
  const u16* add;
  void* out;
  uint32_t src_bytes;
  int C;                           // source channels
  int sd, sh, sw;                  // source extents
  int vd, vh, vw;                  // voxels enumerated per sample (a class's extents)
  lddmm::FastDiv dd, dh, dw;       // division by them
  int nvox;                        // over all samples
  int cs;                          // centre = cs * v
  int os, pz, py, px;              // output voxel = os * v + p
  int fd, fh, fw;                  // output extents
  Axis az, ay, ax;
  int M, K, steps;                 // rows, row length of w, k-steps
  uint32_t pmagic;                 // KM_PAIR: (k pmagic) >> 20 = k / C
  int relu, out_f32, add_stride, add_off, vec;
};

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 bld16(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ uint32_t bld4(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
constexpr uint32_t kOut = 0xfffffff0u;   // past every source (at most 0xffff0000 bytes)

struct Problem {                   // the eight parity classes of a strided gradient
  FragArgs c[8];
  int nblk[8];
};

// Bit j: tap j of the axis stays inside [0, n) around centre c.
__device__ __forceinline__ uint32_t axis_bits(const Axis& x, int c, int n) {
  uint32_t m = 0;
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (j < x.n && (unsigned)(c + x.o0 + j * x.od) < (unsigned)n) m |= 1u << j;
  return m;
}

// Two values as bf16, to nearest even: the hardware conversion, which equals f2bf for
// every one of the 2^32 floats.
__device__ __forceinline__ uint32_t pack_bf(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 p = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, p);
}

template <int KM, bool DGRAD, bool CLASS, int MT, int NT>
__device__ __forceinline__ void conv_frag(const FragArgs& a, int bx) {
  __shared__ u32x4 wl[2][KS * MT * 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * (MT * 16);
  const rsrc_t S = __builtin_amdgcn_make_buffer_rsrc((void*)a.src, (short)0, (int)a.src_bytes,
                                                     0x00020000);
  // this lane's voxel of each tile: centre's byte offset (with the lane's channel group) and
  // the taps that stay on the grid
  uint32_t base[NT], ok[NT];
  int vox[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int v = (bx * 4 + wave) * (NT * 16) + t * 16 + r16;
    const int q = (int)lddmm::fdiv(v, a.dw), x = v - q * a.vw;
    const int q2 = (int)lddmm::fdiv(q, a.dh), y = q - q2 * a.vh;
    const int b = (int)lddmm::fdiv(q2, a.dd), z = q2 - b * a.vd;
    const int cz = a.cs * z, cy = a.cs * y, cx = a.cs * x;
    base[t] = (uint32_t)((((b * a.sd + cz) * a.sh + cy) * a.sw + cx) * a.C) * 2u;
    vox[t] = v < a.nvox ? ((b * a.fd + a.os * z + a.pz) * a.fh + a.os * y + a.py) * a.fw +
                              a.os * x + a.px
                        : -1;
    // bit j = (jz ny + jy) nx + jx: the product of the axes' bits
    const uint32_t mx = axis_bits(a.ax, cx, a.sw), my = axis_bits(a.ay, cy, a.sh),
                   mz = axis_bits(a.az, cz, a.sd);
    const int nyx = a.ay.n * a.ax.n;
    const uint32_t row = (my & 1u ? mx : 0u) | (my & 2u ? mx << a.ax.n : 0u) |
                         (my & 4u ? mx << (2 * a.ax.n) : 0u);
    uint32_t m = (mz & 1u ? row : 0u) | (mz & 2u ? row << nyx : 0u) |
                 (mz & 4u ? row << (2 * nyx) : 0u);
    m = v < a.nvox ? m : 0u;
    ok[t] = m;
    if (KM == KM_32) base[t] += 16u * g;
    if (KM == KM_16) base[t] += 16u * (g & 1);
  }
  const int sy = a.sw * a.C * 2, sz = a.sh * sy, sx = a.C * 2;   // strides in bytes

  // ---- voxel fragments of step st into f
  int pj = 0, pc = 0, pjx = 0, pjy = 0, pjz = 0;   // KM_32: next step's tap and channel block
  int pst = 0;
  auto load_b = [&](u32x4 (&f)[NT]) {
    if (pst >= a.steps) return;
    if (KM == KM_32) {
      const uint32_t off = (uint32_t)((a.az.o0 + pjz * a.az.od) * sz +
                                      (a.ay.o0 + pjy * a.ay.od) * sy +
                                      (a.ax.o0 + pjx * a.ax.od) * sx + pc * 64);
      const uint32_t bit = 1u << pj;
#pragma unroll
      for (int t = 0; t < NT; ++t) f[t] = bld16(S, (ok[t] & bit) ? base[t] + off : kOut);
      if (++pc == a.C / 32) {
        pc = 0;
        ++pj;
        if (++pjx == a.ax.n) {
          pjx = 0;
          if (++pjy == a.ay.n) {
            pjy = 0;
            ++pjz;
          }
        }
      }
    } else if (KM == KM_16) {                      // 27 taps, two per step
      const int j = 2 * pst + (g >> 1);
      const int jz = (j * 57) >> 9, r = j - 9 * jz, jy = (r * 11) >> 5, jx = r - 3 * jy;
      const uint32_t off = (uint32_t)((a.az.o0 + jz * a.az.od) * sz +
                                      (a.ay.o0 + jy * a.ay.od) * sy +
                                      (a.ax.o0 + jx * a.ax.od) * sx);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        f[t] = bld16(S, (j < 27 && ((ok[t] >> j) & 1u)) ? base[t] + off : kOut);
    } else {                                       // pairs of channels, 27 taps
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t k = 32u * pst + 8u * g + 2u * i;
        const int j = (int)((k * a.pmagic) >> 20), c = (int)k - j * a.C;
        const int jz = (j * 57) >> 9, r = j - 9 * jz, jy = (r * 11) >> 5, jx = r - 3 * jy;
        const uint32_t off = (uint32_t)((a.az.o0 + jz * a.az.od) * sz +
                                        (a.ay.o0 + jy * a.ay.od) * sy +
                                        (a.ax.o0 + jx * a.ax.od) * sx + 2 * c);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          f[t][i] = bld4(S, (j < 27 && ((ok[t] >> j) & 1u)) ? base[t] + off : kOut);
      }
    }
    ++pst;
  };

  // ---- weight fragments of chunk ch: wave w stages fragments w, w + 4, ... of KS * MT
  constexpr int WF = KS * MT / 4;
  u32x4 wr[WF];
  auto load_w = [&](int ch) {
#pragma unroll
    for (int i = 0; i < WF; ++i) {
      const int fr = wave + 4 * i, st = ch * KS + fr / MT, row = m0 + (fr % MT) * 16 + r16;
      u32x4 v = {0u, 0u, 0u, 0u};
      if (CLASS) {                                 // the class's taps of the full row
        if (st < a.steps && row < a.M) {
          const int nb = a.C / 32, j = st / nb, cb = st - j * nb;
          const int nyx = a.ay.n * a.ax.n, jz = j / nyx, r = j - jz * nyx, jy = r / a.ax.n,
                    jx = r - jy * a.ax.n;
          const int tap = ((a.az.k0 + jz * a.az.kd) * 3 + a.ay.k0 + jy * a.ay.kd) * 3 + a.ax.k0 +
                          jx * a.ax.kd;
          v = *(const u32x4*)(a.w + (long)row * a.K + tap * a.C + cb * 32 + 8 * g);
        }
      } else if (KM != KM_PAIR) {
        const int k = st * 32 + 8 * g;
        if (k < a.K && row < a.M) v = *(const u32x4*)(a.w + (long)row * a.K + k);
      } else if (row < a.M) {
        const int k = st * 32 + 8 * g;
        const u16* p = a.w + (long)row * a.K + k;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t lo = k + 2 * e < a.K ? p[2 * e] : 0u;
          const uint32_t hi = k + 2 * e + 1 < a.K ? p[2 * e + 1] : 0u;
          v[e] = lo | hi << 16;
        }
      }
      wr[i] = v;
    }
  };
  auto put_w = [&](int buf) {
#pragma unroll
    for (int i = 0; i < WF; ++i) wl[buf][(wave + 4 * i) * 64 + lane] = wr[i];
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 ring[RING][NT];
  load_w(0);
#pragma unroll
  for (int q = 0; q < RING - 1; ++q) load_b(ring[q]);
  put_w(0);
  const int nch = (a.steps + KS - 1) / KS;
  for (int ch = 0; ch < nch; ++ch) {
    __syncthreads();                               // buffer ch & 1 is written, the other is free
    if (ch + 1 < nch) load_w(ch + 1);
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      load_b(ring[(q + RING - 1) % RING]);
      if (ch * KS + q >= a.steps) break;
      const u32x4* wq = &wl[ch & 1][q * MT * 64 + lane];
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const bf16x8 fa = __builtin_bit_cast(bf16x8, wq[i * 64]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fa, __builtin_bit_cast(bf16x8, ring[q][t]), acc[i][t], 0, 0, 0);
      }
    }
    if (ch + 1 < nch) put_w((ch + 1) & 1);
  }

  // ---- epilogue: lane holds channels col .. col + 3 of voxel vox[t]
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int col = m0 + 16 * i + 4 * g;
    if (col >= a.M) continue;
    const int nc = a.M - col < 4 ? a.M - col : 4;
    float bias[4] = {0.f, 0.f, 0.f, 0.f};
    if (!DGRAD && a.bias)
      for (int r = 0; r < nc; ++r) bias[r] = a.bias[col + r];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (vox[t] < 0) continue;
      const long o = (long)vox[t] * a.M + col;
      float v[4];
      if (!DGRAD) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = acc[i][t][r];
          if (a.bias) v[r] += bias[r];
          if (a.relu) v[r] = fmaxf(v[r], 0.f);
        }
      } else {
        u16 mk[4] = {0, 0, 0, 0}, ad[4] = {0, 0, 0, 0};
        const long oa = (long)vox[t] * a.add_stride + a.add_off + col;
        if (a.vec) {
          if (a.mask) *(uint2*)mk = *(const uint2*)(a.mask + o);
          if (a.add) *(uint2*)ad = *(const uint2*)(a.add + oa);
        } else {
          for (int r = 0; r < nc; ++r) {
            if (a.mask) mk[r] = a.mask[o + r];
            if (a.add) ad[r] = a.add[oa + r];
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = acc[i][t][r];
          if (a.mask && !(bf2f(mk[r]) > 0.f)) v[r] = 0.f;
          if (a.add) v[r] += bf2f(ad[r]);
        }
      }
      if (a.vec) {
        if (a.out_f32) {
          *(float4*)((float*)a.out + o) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          uint2 p;
          p.x = pack_bf(v[0], v[1]);
          p.y = pack_bf(v[2], v[3]);
          *(uint2*)((u16*)a.out + o) = p;
        }
      } else {
        for (int r = 0; r < nc; ++r) {
          if (a.out_f32)
            ((float*)a.out)[o + r] = v[r];
          else
            ((u16*)a.out)[o + r] = f2bf(v[r]);
        }
      }
    }
  }
}

// Blocks run on XCD b mod 8: block b of a multiple of 8 takes its XCD's contiguous
// eighth of the voxels, so the 27 taps of a block's voxels, and their neighbours',
// are read behind one L2 (dealt in order, every XCD's L2 fetched the whole source).
__device__ __forceinline__ int xcd_block(int b, int n) {
  return (b % lddmm::kXCD) * (n / lddmm::kXCD) + b / lddmm::kXCD;
}

inline int round_xcd(long long blocks) {
  return (int)((blocks + lddmm::kXCD - 1) / lddmm::kXCD * lddmm::kXCD);
}

template <int KM, bool DGRAD, int MT, int NT>
__global__ __launch_bounds__(kBlk) void k_conv_frag(FragArgs a) {
  conv_frag<KM, DGRAD, false, MT, NT>(a, xcd_block(blockIdx.x, gridDim.x));
}

// The parity classes of a strided input gradient, those with the most taps first.
template <int MT, int NT>
__global__ __launch_bounds__(kBlk) void k_conv_frag_classes(Problem p) {
  int c = 0, b = blockIdx.x;
  while (b >= p.nblk[c]) b -= p.nblk[c++];
  conv_frag<KM_32, true, true, MT, NT>(p.c[c], xcd_block(b, p.nblk[c]));
}

template <bool DGRAD, int MT, int NT>
void launch_km(int km, const FragArgs& a, hipStream_t s) {
  const dim3 grid(round_xcd((a.nvox + 64 * NT - 1) / (64 * NT)), (a.M + 16 * MT - 1) / (16 * MT));
  if (km == KM_32)
    hipLaunchKernelGGL((k_conv_frag<KM_32, DGRAD, MT, NT>), grid, dim3(kBlk), 0, s, a);
  else if (km == KM_16)
    hipLaunchKernelGGL((k_conv_frag<KM_16, DGRAD, MT, NT>), grid, dim3(kBlk), 0, s, a);
  else
    hipLaunchKernelGGL((k_conv_frag<KM_PAIR, DGRAD, MT, NT>), grid, dim3(kBlk), 0, s, a);
}

template <int MT, int NT>
void launch_classes(const Problem& p, hipStream_t s) {
  int n = 0;
  for (int c = 0; c < 8; ++c) n += p.nblk[c];
  const dim3 grid(n, (p.c[0].M + 16 * MT - 1) / (16 * MT));
  hipLaunchKernelGGL((k_conv_frag_classes<MT, NT>), grid, dim3(kBlk), 0, s, p);
}


// ---------------------------------------------------------------- source tile in LDS ----
// The same products with the source in LDS, for 32, 64, 128 or 192 source channels: a
// block owns a tile of TZ x 4 x 8 voxels (16 consecutive lanes = two rows of 8) and
// all channels of its halo, read once; the taps then only move an LDS offset.
// (The fragment kernel above reads each voxel's channels 27 times through L1, whose
// misses bounded it: 205 us for the decoder's 192 -> 64 at 8 x 24^3, 353 TFLOP/s.)
// A block's four wavefronts are WV groups of voxels x WM groups of rows.  The weights
// of two steps (128 consecutive bytes of every row) are loaded three chunks ahead,
// eight adjacent lanes to a row, and pass through a double buffer in LDS: a
// fragment's own layout, adjacent lanes in different rows, reads L2 at 15 B a clock
// and CU against 40-55 for whole lines (measured on 0.65 MB read by all blocks),
// and with it every variant of this kernel took 200 us.  The k loop is unrolled
// over the taps of a plane and the channel blocks, so every LDS offset in it is an
// immediate.
// A strided gradient runs its eight parity classes one after the other on one tile
// of dy, so the lines of dx and of the mask, which two classes share, are touched
// while they are in L2.
constexpr int HY = 4, HX = 8;      // rows and columns of a tile

enum { H_FWD = 0, H_DG1 = 1, H_DG2 = 2 };

struct HaloArgs {
  const u16* src;
  const u16* w;
  const float* bias;
  const u16* mask;
  const u16* add;
  void* out;
  uint32_t src_bytes, w_bytes;
  int sd, sh, sw;                  // source extents
  int vd, vh, vw;                  // voxels of a sample in tile space
  int fd, fh, fw;                  // output extents
  int ntx, nty, ntz, ntiles;       // tiles per sample, and over all samples
  int M;                           // rows (output channels)
  int relu, out_f32, add_stride, add_off, vec;
};

// Compile-time geometry of one variant.
template <int OP, int S, int NB, int RF>
struct HaloGeom {
  static constexpr int C = 32 * NB;
  static constexpr int SPAN = OP == H_DG2 ? 2 : 3;           // source coordinates a tap can reach
  static constexpr int LO = OP == H_DG2 ? 0 : -1;            // the first, from the centre
  static constexpr int CS = OP == H_FWD ? S : 1;             // centre = CS * voxel
  static constexpr int EY = CS * (HY - 1) + SPAN, EX = CS * (HX - 1) + SPAN;
  static constexpr int VU = C / 8 + 1;                       // 16-byte units per voxel, one of padding
  static constexpr int ez(int tz) { return CS * (tz - 1) + SPAN; }
  static constexpr int units(int tz) { return ez(tz) * EY * EX * VU; }
  // four planes (128 voxels) unless only two leave room for a second block on the CU, or fit
  static constexpr int lds(int tz) { return (units(tz) + 63) / 64 * 1024; }
  static constexpr int WL = RF * 4096;                       // two buffers of two steps of RF fragments
  static constexpr int MOST = 160 * 1024 - WL;
  static constexpr int TZ =
      lds(4) <= MOST / 2 ? 4 : (lds(2) <= MOST / 2 ? 2 : (lds(4) <= MOST ? 4 : 2));
  static constexpr bool fits = lds(TZ) <= MOST;
  static constexpr int EZ = ez(TZ), UNITS = units(TZ), TILE = lds(TZ), LDS = TILE + WL;
};

// Step u of a strided gradient's 27 NB: its class, tap and LDS offset.
struct ClassStep {
  int cls, tap, dz, dy, dx, cb;
  bool last;                       // of its class
};
template <int NB>
constexpr ClassStep class_step(int u) {
  int seen = 0;
  for (int c = 0; c < 8; ++c) {
    const int nz = 1 + (c >> 2), ny = 1 + ((c >> 1) & 1), nx = 1 + (c & 1);
    const int n = nz * ny * nx * NB;
    if (u < seen + n) {
      const int r = u - seen, cb = r % NB, j = r / NB;
      const int jx = j % nx, jy = (j / nx) % ny, jz = j / (nx * ny);
      // an odd coordinate: tap 0 at offset 1, tap 2 at offset 0; an even one: tap 1 at 0
      const int kz = nz == 2 ? 2 * jz : 1, ky = ny == 2 ? 2 * jy : 1, kx = nx == 2 ? 2 * jx : 1;
      return ClassStep{c, (kz * 3 + ky) * 3 + kx, nz == 2 ? 1 - jz : 0, ny == 2 ? 1 - jy : 0,
                       nx == 2 ? 1 - jx : 0, cb, r == n - 1};
    }
    seen += n;
  }
  return ClassStep{};
}

template <int... I, class F>
__device__ __forceinline__ void unroll_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unroll(F&& f) {
  unroll_impl(std::make_integer_sequence<int, N>{}, f);
}

template <bool DGRAD>
__device__ __forceinline__ void conv_store(const HaloArgs& a, const f32x4& acc, int vox, int col) {
  if (vox < 0 || col >= a.M) return;
  const int nc = a.M - col < 4 ? a.M - col : 4;
  const long o = (long)vox * a.M + col;
  float v[4] = {acc[0], acc[1], acc[2], acc[3]};
  if (!DGRAD) {
    if (a.bias) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < nc) v[r] += a.bias[col + r];
    }
    if (a.relu) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
    }
  } else {
    const long oa = (long)vox * a.add_stride + a.add_off + col;
    u16 mk[4] = {0, 0, 0, 0}, ad[4] = {0, 0, 0, 0};
    if (a.vec) {
      if (a.mask) *(uint2*)mk = *(const uint2*)(a.mask + o);
      if (a.add) *(uint2*)ad = *(const uint2*)(a.add + oa);
    } else {
      for (int r = 0; r < nc; ++r) {
        if (a.mask) mk[r] = a.mask[o + r];
        if (a.add) ad[r] = a.add[oa + r];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (a.mask && !(bf2f(mk[r]) > 0.f)) v[r] = 0.f;
      if (a.add) v[r] += bf2f(ad[r]);
    }
  }
  if (a.vec) {
    if (a.out_f32) {
      *(float4*)((float*)a.out + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
      uint2 p;
      p.x = pack_bf(v[0], v[1]);
      p.y = pack_bf(v[2], v[3]);
      *(uint2*)((u16*)a.out + o) = p;
    }
  } else {
    for (int r = 0; r < nc; ++r) {
      if (a.out_f32)
        ((float*)a.out)[o + r] = v[r];
      else
        ((u16*)a.out)[o + r] = f2bf(v[r]);
    }
  }
}

template <int OP, int S, int NB, int MT, int WM>
__global__ __launch_bounds__(kBlk) void k_conv_halo(HaloArgs a) {
  constexpr int RF = WM * MT;                                // row fragments of the block
  using G = HaloGeom<OP, S, NB, RF>;
  constexpr bool DG = OP != H_FWD;
  constexpr int WV = 4 / WM, NT = G::TZ * 2 / WV;            // tiles of 16 voxels per wavefront
  constexpr int K2 = 27 * G::C * 2;                          // bytes of a row of weights
  constexpr int STEPS = 27 * NB, CHUNKS = (STEPS + 1) / 2;   // two steps to a chunk
  constexpr int WU = (RF + 1) / 2;                           // 16-byte units per thread and chunk
  constexpr int AHEAD = 3;                                   // chunks of weights in registers
  extern __shared__ u32x4 tile[];                            // [EZ][EY][EX][VU], weight buffers
  u32x4* const wl = tile + G::TILE / 16;                     // [2][2 steps][RF][64]
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wv = wave % WV, wm = wave / WV;
  const int mb = blockIdx.y * (RF * 16), m0 = mb + wm * (MT * 16);
  int b = xcd_block(blockIdx.x, gridDim.x);
  if (b >= a.ntiles) return;
  const int x0 = (b % a.ntx) * HX;
  b /= a.ntx;
  const int y0 = (b % a.nty) * HY;
  b /= a.nty;
  const int z0 = (b % a.ntz) * G::TZ;
  b /= a.ntz;                                                // the sample

  // ---- weights: unit u of a chunk is row u / 8, step (u / 4) % 2, octet u % 4; it goes to the
  // fragment's lane of that row and octet, the row XORed with u % 8 so that a row's eight
  // units meet eight different bank groups
  const rsrc_t Wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, (short)0, (int)a.w_bytes,
                                                      0x00020000);
  uint32_t wsrc[WU];                                         // byte offset of the unit's row and octet
  int wdst[WU];                                              // LDS unit; -1: no unit (RF = 1)
  const int wp = threadIdx.x & 7, wh = wp >> 2;
#pragma unroll
  for (int i = 0; i < WU; ++i) {
    const int r = (threadIdx.x + i * kBlk) >> 3;             // row within the block's rows
    const int row = mb + r;                                  // rows past M repeat the last one
    wsrc[i] = (uint32_t)(row < a.M ? row : a.M - 1) * K2 + 16u * (wp & 3);
    wdst[i] = r < RF * 16 ? (wh * RF + (r >> 4)) * 64 + (wp & 3) * 16 + ((r & 15) ^ wp) : -1;
  }
  u32x4 wr[AHEAD][WU];
  // k0, k1: byte offsets in a row of the chunk's two steps
  auto load_w = [&](u32x4 (&f)[WU], int k0, int k1) {
    const uint32_t k = wh ? k1 : k0;
#pragma unroll
    for (int i = 0; i < WU; ++i)
      f[i] = __builtin_bit_cast(u32x4,
                                __builtin_amdgcn_raw_buffer_load_b128(Wr, wsrc[i] + k, 0, 0));
  };
  auto put_w = [&](const u32x4 (&f)[WU], int buf) {
#pragma unroll
    for (int i = 0; i < WU; ++i)
      if (RF > 1 || wdst[i] >= 0) wl[buf * (2 * RF * 64) + wdst[i]] = f[i];
  };
  // this lane's unit of fragment 0 of step 0, 1 of buffer 0
  const u32x4* wread[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) wread[h] = wl + (h * RF + wm * MT) * 64 + g * 16 + (r16 ^ (4 * h + g));

  // ---- source tile and halo straight into LDS: unit e of the tile to LDS unit e, units of
  // padding or outside the grid read as zero
  {
    const rsrc_t Sr = __builtin_amdgcn_make_buffer_rsrc((void*)a.src, (short)0, (int)a.src_bytes,
                                                        0x00020000);
    const int sz0 = G::CS * z0 + G::LO, sy0 = G::CS * y0 + G::LO, sx0 = G::CS * x0 + G::LO;
    for (int e0 = wave * 64; e0 < G::UNITS; e0 += kBlk) {
      const int e = e0 + lane;
      const int p = e / G::VU, c = e - p * G::VU;
      const int q = p / G::EX, x = p - q * G::EX, z = q / G::EY, y = q - z * G::EY;
      const int iz = sz0 + z, iy = sy0 + y, ix = sx0 + x;
      const bool in = c < G::C / 8 && e < G::UNITS && (unsigned)iz < (unsigned)a.sd &&
                      (unsigned)iy < (unsigned)a.sh && (unsigned)ix < (unsigned)a.sw;
      const uint32_t off =
          (uint32_t)(((b * a.sd + iz) * a.sh + iy) * a.sw + ix) * (uint32_t)(2 * G::C) + 16u * c;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          Sr, (__attribute__((address_space(3))) void*)(tile + e0), 16, in ? off : kOut, 0, 0, 0);
    }
  }

  // ---- this lane's voxels
  int vz[NT], vy[NT];
  const int vx = x0 + (r16 & 7);
  const char* base[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int q = wv * NT + t;                               // two tiles of 16 per plane
    const int lz = q >> 1, ly = (q & 1) * 2 + (r16 >> 3), lx = r16 & 7;
    vz[t] = z0 + lz;
    vy[t] = y0 + ly;
    base[t] = reinterpret_cast<const char*>(tile) +
              ((G::CS * lz * G::EY + G::CS * ly) * G::EX + G::CS * lx) * (G::VU * 16) + 16 * g;
  }
  auto load_v = [&](u32x4 (&f)[NT], int imm) {
#pragma unroll
    for (int t = 0; t < NT; ++t) f[t] = *reinterpret_cast<const u32x4*>(base[t] + imm);
  };
  f32x4 acc[MT][NT];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  u32x4 vf[4][NT], wf[4][MT];      // step u in slot u mod 4
  auto load_f = [&](u32x4 (&f)[MT], int h, int buf) {
#pragma unroll
    for (int i = 0; i < MT; ++i) f[i] = wread[h][buf * (2 * RF * 64) + i * 64];
  };
  auto products = [&](const u32x4 (&w)[MT], const u32x4 (&v)[NT]) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[i]),
                                                            __builtin_bit_cast(bf16x8, v[t]),
                                                            acc[i][t], 0, 0, 0);
  };
  auto store = [&](int os, int pz, int py, int px) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int oz = os * vz[t] + pz, oy = os * vy[t] + py, ox = os * vx + px;
      const int vox = oz < a.fd && oy < a.fh && ox < a.fw
                          ? ((b * a.fd + oz) * a.fh + oy) * a.fw + ox
                          : -1;
#pragma unroll
      for (int i = 0; i < MT; ++i) conv_store<DG>(a, acc[i][t], vox, m0 + 16 * i + 4 * g);
    }
  };
  constexpr int LX = G::VU * 16, LY = G::EX * LX, LZ = G::EY * LY;   // LDS bytes per voxel
  clear();
  // byte offset in a row of weights of step u (steps past the last: the last again)
  auto kof = [](int u) constexpr {
    u = u < STEPS ? u : STEPS - 1;
    if constexpr (OP == H_DG2) {
      const ClassStep s = class_step<NB>(u);
      return 2 * (s.tap * G::C + 32 * s.cb);
    } else {
      return 64 * u;
    }
  };
  // LDS offset of the voxels of step u; the gradient's offsets run backwards
  auto vof = [](int u) constexpr {
    u = u < STEPS ? u : STEPS - 1;
    if constexpr (OP == H_DG2) {
      const ClassStep s = class_step<NB>(u);
      return s.dz * LZ + s.dy * LY + s.dx * LX + s.cb * 64;
    } else {
      const int tap = u / NB, kz = tap / 9, ky = (tap / 3) % 3, kx = tap % 3;
      return (DG ? 2 - kz : kz) * LZ + (DG ? 2 - ky : ky) * LY + (DG ? 2 - kx : kx) * LX +
             (u % NB) * 64;
    }
  };
  unroll<AHEAD>([&](auto c) {
    constexpr int u = 2 * decltype(c)::value;
    load_w(wr[c], kof(u), kof(u + 1));
  });
  put_w(wr[0], 0);                                           // waits for every load before it too
  __builtin_amdgcn_s_waitcnt(0x0f70);                        // the tile's LDS writes (vmcnt 0)
  __syncthreads();
  load_v(vf[0], vof(0));
  load_v(vf[1], vof(1));
  // products of step u; a strided gradient's class is stored after its last
  auto finish = [&](auto uc) {
    constexpr int u = decltype(uc)::value;
    products(wf[u & 3], vf[u & 3]);
    if constexpr (OP == H_DG2) {
      constexpr ClassStep s = class_step<NB>(u);
      if constexpr (s.last) {
        store(2, s.cls >> 2, (s.cls >> 1) & 1, s.cls & 1);
        clear();
      }
    }
  };
  // Chunk c is steps 2c, 2c + 1.  After the barrier its weights are read and the next chunk's
  // written to the other buffer; the products of the step before the barrier and of its first
  // step then cover those reads, and the voxels of the next chunk are read under them.
  unroll<CHUNKS>([&](auto cc) {
    constexpr int c = decltype(cc)::value, a0 = 2 * c, a1 = 2 * c + 1;
    __syncthreads();
    load_f(wf[a0 & 3], 0, c & 1);
    load_f(wf[a1 & 3], 1, c & 1);
    if constexpr (c + 1 < CHUNKS) put_w(wr[(c + 1) % AHEAD], (c + 1) & 1);
    load_v(vf[(a0 + 2) & 3], vof(a0 + 2));
    if constexpr (c > 0) finish(std::integral_constant<int, a0 - 1>{});
    load_v(vf[(a1 + 2) & 3], vof(a1 + 2));
    finish(std::integral_constant<int, a0>{});
    if constexpr (c + AHEAD < CHUNKS) load_w(wr[c % AHEAD], kof(a0 + 2 * AHEAD), kof(a1 + 2 * AHEAD));
    __builtin_amdgcn_sched_barrier(0);
  });
  if constexpr (2 * CHUNKS - 1 < STEPS) finish(std::integral_constant<int, 2 * CHUNKS - 1>{});
  if constexpr (OP != H_DG2) store(1, 0, 0, 0);
}

// ---------------------------------------------------- two source channels, stride 1 ----
// The network's first layer.  A voxel's two channels are one 32-bit word, so a block stages the
// words of a P2X x P2Y x P2Z tile and its halo in LDS and a fragment is four reads at offsets
// that belong to the lane alone (the taps of its k-values), the tile's place an immediate; the 54
// weights of a row stay in two registers' worth of fragments.  Bound by its vector instructions
// (0.71 a cycle and CU at 8 x 96^3, where it writes 226 MB at 3.1 TB/s).  Read straight from memory (the fragment kernel: eight gathers of 4 B per
// lane for 16 voxels, each as dear to L1 as one of 16 B) 8 x 96^3 took 180 us and one 29:
// 70 and 15.5 now (93 and 19 with four planes to a block and stores of 8 B).
// k order and instruction as there, so the same bits.
constexpr int P2X = 32, P2Y = 4, P2Z = 8, P2W = P2X + 4;   // P2W: words of a staged row

__global__ __launch_bounds__(kBlk) void k_conv_two(HaloArgs a) {
  constexpr int SY = P2Y + 2, SZ = P2Z + 2, PLANE = SY * P2W;
  __shared__ uint32_t tile[SZ * PLANE];
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.y * 16;
  int b = xcd_block(blockIdx.x, gridDim.x);
  if (b >= a.ntiles) return;
  const int x0 = (b % a.ntx) * P2X;
  b /= a.ntx;
  const int y0 = (b % a.nty) * P2Y;
  b /= a.nty;
  const int z0 = (b % a.ntz) * P2Z;
  b /= a.ntz;                                                // the sample
  const rsrc_t Sr = __builtin_amdgcn_make_buffer_rsrc((void*)a.src, (short)0, (int)a.src_bytes,
                                                      0x00020000);
  constexpr int PER = (SZ * PLANE + kBlk - 1) / kBlk;
  uint32_t st[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = threadIdx.x + i * kBlk;
    const int q = e / P2W, x = e - q * P2W, z = q / SY, y = q - z * SY;
    const int iz = z0 - 1 + z, iy = y0 - 1 + y, ix = x0 - 1 + x;
    const bool in = e < SZ * PLANE && (unsigned)iz < (unsigned)a.sd &&
                    (unsigned)iy < (unsigned)a.sh && (unsigned)ix < (unsigned)a.sw;
    st[i] = bld4(Sr, in ? (uint32_t)(((b * a.sd + iz) * a.sh + iy) * a.sw + ix) * 4u : kOut);
  }
  // weights: k = 32 step + 8 g + e of row m0 + r16, zero past the row's 54
  bf16x8 wf[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (m0 + r16 < a.M) {
      const u16* p = a.w + (long)(m0 + r16) * 54;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = 32 * h + 8 * g + 2 * e;
        if (k < 54) v[e] = p[k] | (uint32_t)p[k + 1] << 16;
      }
    }
    wf[h] = __builtin_bit_cast(bf16x8, v);
  }
  // this lane's words of a fragment: tap j = 16 step + 4 g + i at its voxel; past the taps, zero
  int off[2][4];
  bool tap[4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = 16 * h + 4 * g + i, c = j < 27 ? j : 0;
      const int jz = c / 9, jy = (c / 3) % 3, jx = c % 3;
      off[h][i] = (wave + jz) * PLANE + jy * P2W + jx + r16;   // a wavefront takes one plane
      if (h == 1) tap[i] = j < 27;
    }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = threadIdx.x + i * kBlk;
    if (e < SZ * PLANE) tile[e] = st[i];
  }
  __syncthreads();
  // pairs of tiles along x: with 16 rows of bf16, rows of lanes exchanged between the two, so that
  // a lane stores eight channels of one voxel at once
  const bool wide = a.vec && !a.out_f32 && a.M % 16 == 0 && ((uintptr_t)a.out & 15) == 0;
  float bias[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (a.bias && m0 + 4 * g + r < a.M) bias[r] = a.bias[m0 + 4 * g + r];
  for (int z = wave; z < P2Z; z += 4) {
    const int oz = z0 + z;
    if (oz >= a.fd) break;
#pragma unroll
    for (int y = 0; y < P2Y; ++y) {
      const int oy = y0 + y;
      f32x4 acc[P2X / 16];
#pragma unroll
      for (int xh = 0; xh < P2X / 16; ++xh) {
        const uint32_t* p = tile + (z - wave) * PLANE + y * P2W + 16 * xh;
        u32x4 f[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f[0][i] = p[off[0][i]];
          const uint32_t v = p[off[1][i]];
          f[1][i] = tap[i] ? v : 0u;
        }
        acc[xh] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < 2; ++h)
          acc[xh] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              wf[h], __builtin_bit_cast(bf16x8, f[h]), acc[xh], 0, 0, 0);
      }
      const int row = ((b * a.fd + oz) * a.fh + oy) * a.fw;
      if (wide) {
        uint32_t w[2][2];
#pragma unroll
        for (int xh = 0; xh < 2; ++xh) {
          float v[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = acc[xh][r];
            if (a.bias) v[r] += bias[r];
            if (a.relu) v[r] = fmaxf(v[r], 0.f);
          }
          w[xh][0] = pack_bf(v[0], v[1]);
          w[xh][1] = pack_bf(v[2], v[3]);
        }
        // lane rows 0 .. 3 hold channels 4 g of both tiles; after the swap rows 0, 2 hold eight
        // channels of the first tile's voxel and rows 1, 3 of the second's
        const auto lo = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
        const u32x4 q = {lo[0], hi[0], lo[1], hi[1]};
        const int ox = x0 + 16 * (g & 1) + r16;
        if (oy < a.fh && ox < a.fw)
          *reinterpret_cast<u32x4*>((u16*)a.out + (long)(row + ox) * a.M + m0 + 8 * (g >> 1)) = q;
      } else {
#pragma unroll
        for (int xh = 0; xh < 2; ++xh) {
          const int ox = x0 + 16 * xh + r16;
          conv_store<false>(a, acc[xh], oy < a.fh && ox < a.fw ? row + ox : -1, m0 + 4 * g);
        }
      }
    }
  }
}

void launch_two(HaloArgs h, int samples, hipStream_t s) {
  h.ntx = (h.vw + P2X - 1) / P2X;
  h.nty = (h.vh + P2Y - 1) / P2Y;
  h.ntz = (h.vd + P2Z - 1) / P2Z;
  h.ntiles = h.ntx * h.nty * h.ntz * samples;
  hipLaunchKernelGGL(k_conv_two, dim3(round_xcd(h.ntiles), (h.M + 15) / 16), dim3(kBlk), 0, s, h);
}

template <int OP, int S, int NB, int MT, int WM>
void launch_halo_k(HaloArgs h, int samples, hipStream_t s) {
  using G = HaloGeom<OP, S, NB, MT * WM>;
  h.ntx = (h.vw + HX - 1) / HX;
  h.nty = (h.vh + HY - 1) / HY;
  h.ntz = (h.vd + G::TZ - 1) / G::TZ;
  h.ntiles = h.ntx * h.nty * h.ntz * samples;
  const dim3 grid(round_xcd(h.ntiles), (h.M + 16 * MT * WM - 1) / (16 * MT * WM));
  hipLaunchKernelGGL((k_conv_halo<OP, S, NB, MT, WM>), grid, dim3(kBlk), G::LDS, s, h);
}

template <int OP, int S, int NB, int MT, int WM>
bool try_halo(const HaloArgs& h, int samples, hipStream_t s) {
  if constexpr (!HaloGeom<OP, S, NB, MT * WM>::fits) {
    return false;
  } else {
    launch_halo_k<OP, S, NB, MT, WM>(h, samples, s);
    return true;
  }
}

// Blocks of a variant; 0: it has none.
template <int OP, int S, int NB, int MT, int WM>
long long halo_blocks(const HaloArgs& h, int samples) {
  using G = HaloGeom<OP, S, NB, MT * WM>;
  if (!G::fits) return 0;
  return (long long)((h.vw + HX - 1) / HX) * ((h.vh + HY - 1) / HY) * ((h.vd + G::TZ - 1) / G::TZ) *
         samples * ((h.M + 16 * MT * WM - 1) / (16 * MT * WM));
}

// Rows of a block: as many as there are up to 192, so that a tile is staged once for all; but
// while that leaves half of the 256 CUs without a block, half as many (the staging is repeated,
// the products, which take most of the time, are shared out).  One 96^3 sample through the
// network: 43 -> 32 us in the decoder, 21 -> 12 and 15 -> 11 in the deepest encoder and the head.
template <int OP, int S, int NB>
bool launch_halo_m(const HaloArgs& h, int samples, hipStream_t s) {
  constexpr int kFew = 128;
  if (h.M <= 16) return try_halo<OP, S, NB, 1, 1>(h, samples, s);
  if (h.M <= 32 || halo_blocks<OP, S, NB, 2, 2>(h, samples) <= kFew) {
    if (halo_blocks<OP, S, NB, 1, 2>(h, samples) <= kFew)
      return try_halo<OP, S, NB, 1, 1>(h, samples, s);
    return try_halo<OP, S, NB, 1, 2>(h, samples, s);
  }
  if (h.M <= 64) return try_halo<OP, S, NB, 2, 2>(h, samples, s);
  if constexpr (NB <= 2) {         // with more channels the blocks of 64 rows fill the CU's LDS
    if (h.M % 192 == 0 && halo_blocks<OP, S, NB, 6, 2>(h, samples) > kFew &&
        try_halo<OP, S, NB, 6, 2>(h, samples, s))
      return true;
    if (halo_blocks<OP, S, NB, 4, 2>(h, samples) > kFew && try_halo<OP, S, NB, 4, 2>(h, samples, s))
      return true;
  }
  return try_halo<OP, S, NB, 2, 2>(h, samples, s);
}

template <int OP, int S>
bool launch_halo_c(int c, const HaloArgs& h, int samples, hipStream_t s) {
  switch (c) {
    case 32: return launch_halo_m<OP, S, 1>(h, samples, s);
    case 64: return launch_halo_m<OP, S, 2>(h, samples, s);
    // a strided gradient's 108 unrolled steps and eight epilogues outgrow the instruction
    // cache (281 us for 64 <- 128 channels at 8 x 12^3, about 30 with fragments)
    case 128:
      if constexpr (OP != H_DG2) return launch_halo_m<OP, S, 4>(h, samples, s);
      return false;
    case 192:
      if constexpr (OP != H_DG2) return launch_halo_m<OP, S, 6>(h, samples, s);
      return false;
    default: return false;
  }
}

bool launch_halo(const FragArgs& f, bool dg, int stride, int samples, hipStream_t s) {
  HaloArgs h{};
  if (2LL * f.M * f.K > 0x7fffffffLL) return false;
  h.src = f.src;
  h.w = f.w;
  h.bias = f.bias;
  h.mask = f.mask;
  h.add = f.add;
  h.out = f.out;
  h.src_bytes = f.src_bytes;
  h.w_bytes = (uint32_t)(2LL * f.M * f.K);
  h.sd = f.sd;
  h.sh = f.sh;
  h.sw = f.sw;
  h.fd = f.fd;
  h.fh = f.fh;
  h.fw = f.fw;
  const bool cls = dg && stride == 2;
  h.vd = cls ? (f.fd + 1) / 2 : f.fd;            // an odd extent's last odd coordinate is not stored
  h.vh = cls ? (f.fh + 1) / 2 : f.fh;
  h.vw = cls ? (f.fw + 1) / 2 : f.fw;
  h.M = f.M;
  h.relu = f.relu;
  h.out_f32 = f.out_f32;
  h.add_stride = f.add_stride;
  h.add_off = f.add_off;
  h.vec = f.vec;
  if (f.C == 2) {
    if (dg || stride != 1) return false;
    launch_two(h, samples, s);
    return true;
  }
  if (cls) return launch_halo_c<H_DG2, 1>(f.C, h, samples, s);
  if (dg) return launch_halo_c<H_DG1, 1>(f.C, h, samples, s);
  return stride == 2 ? launch_halo_c<H_FWD, 2>(f.C, h, samples, s)
                     : launch_halo_c<H_FWD, 1>(f.C, h, samples, s);
}

}  // namespace

bool launch_conv_frag(int op, const ConvArgs& a, hipStream_t s) {
  FragArgs f{};
  const bool dg = op == OP_DGRAD;
  f.C = dg ? a.co : a.ci;
  f.sd = dg ? a.od : a.d;
  f.sh = dg ? a.oh : a.h;
  f.sw = dg ? a.ow : a.w;
  f.fd = dg ? a.d : a.od;
  f.fh = dg ? a.h : a.oh;
  f.fw = dg ? a.w : a.ow;
  const long long sb = 2LL * a.n * f.sd * f.sh * f.sw * f.C;
  if (sb > 0xffff0000LL || ((uintptr_t)a.x & 3)) return false;
  const int km = f.C % 32 == 0 ? KM_32 : (f.C == 16 ? KM_16 : (f.C % 2 == 0 ? KM_PAIR : -1));
  if (km < 0 || (dg && a.s == 2 && km != KM_32)) return false;
  if (km != KM_PAIR && ((uintptr_t)a.wb & 15)) return false;
  if (km == KM_PAIR) {
    f.pmagic = (1u << 20) / (uint32_t)f.C + 1;
    for (int k = 0; k < 27 * f.C + 192; ++k)       // the steps loaded ahead included
      if ((long long)k * f.pmagic > 0xffffffffLL || (int)((k * f.pmagic) >> 20) != k / f.C)
        return false;
  }
  f.src = a.x;
  f.w = a.wb;
  f.bias = a.bias;
  f.mask = a.mask;
  f.add = a.add;
  f.out = a.out;
  f.src_bytes = (uint32_t)sb;
  f.M = a.N;
  f.K = a.K;
  f.relu = a.relu;
  f.out_f32 = a.out_f32;
  f.add_stride = a.add_stride;
  f.add_off = a.add_off;
  // four channels of a voxel at once: when rows keep the alignment
  f.vec = f.M % 4 == 0 && ((uintptr_t)a.out & (a.out_f32 ? 15 : 7)) == 0 &&
          ((uintptr_t)a.mask & 7) == 0 &&
          (!a.add || (((uintptr_t)a.add & 7) == 0 && a.add_stride % 4 == 0 && a.add_off % 4 == 0));
  // The staged kernel loads 16 bytes a lane straight to LDS and wants them aligned, as the weight
  // gradient does; k_conv_two's words and the fragments' buffer loads need 4-byte alignment.
  const bool staged = f.C == 2 || (km == KM_32 && ((uintptr_t)a.x & 15) == 0);
  if (staged && launch_halo(f, dg, a.s, a.n, s)) return true;
  const int mt = f.M <= 16 ? 1 : (f.M <= 32 ? 2 : (f.M <= 64 ? 4 : (f.M % 96 == 0 ? 6 : 8)));
  if (dg && a.s == 2) {
    Problem p{};
    const int order[8] = {7, 3, 5, 6, 1, 2, 4, 0};
    const long nv = (long)a.n * a.d * a.h * a.w / 8;
    const int nt = nv >= 64L * 4 * 192 ? 4 : (nv >= 64L * 2 * 192 ? 2 : 1);
    for (int q = 0; q < 8; ++q) {
      const int c = order[q];
      FragArgs& e = p.c[q];
      e = f;
      e.pz = (c >> 2) & 1;
      e.py = (c >> 1) & 1;
      e.px = c & 1;
      auto axis = [](int par) { return par ? Axis{2, 0, 2, 1, -1} : Axis{1, 1, 0, 0, 0}; };
      e.az = axis(e.pz);
      e.ay = axis(e.py);
      e.ax = axis(e.px);
      e.cs = 1;
      e.os = 2;
      e.vd = (a.d - e.pz + 1) / 2;
      e.vh = (a.h - e.py + 1) / 2;
      e.vw = (a.w - e.px + 1) / 2;
      e.dd = lddmm::make_fastdiv(std::max(e.vd, 1));
      e.dh = lddmm::make_fastdiv(std::max(e.vh, 1));
      e.dw = lddmm::make_fastdiv(std::max(e.vw, 1));
      e.nvox = a.n * e.vd * e.vh * e.vw;
      e.steps = e.az.n * e.ay.n * e.ax.n * (f.C / 32);
      p.nblk[q] = round_xcd((e.nvox + 64 * nt - 1) / (64 * nt));
    }
#define LDDMM_CASE(MT)                      \
  if (mt == MT) {                           \
    if (nt == 4) launch_classes<MT, 4>(p, s); \
    else if (nt == 2) launch_classes<MT, 2>(p, s); \
    else launch_classes<MT, 1>(p, s);       \
  }
    LDDMM_CASE(1) LDDMM_CASE(2) LDDMM_CASE(4) LDDMM_CASE(6) LDDMM_CASE(8)
#undef LDDMM_CASE
    return true;
  }
  const Axis ax = dg ? Axis{3, 0, 1, 1, -1} : Axis{3, 0, 1, -1, 1};
  f.az = f.ay = f.ax = ax;
  f.cs = dg ? 1 : a.s;
  f.os = 1;
  f.vd = f.fd;
  f.vh = f.fh;
  f.vw = f.fw;
  f.dd = lddmm::make_fastdiv(f.vd);
  f.dh = lddmm::make_fastdiv(f.vh);
  f.dw = lddmm::make_fastdiv(f.vw);
  f.nvox = a.M;
  f.steps = (f.K + 31) / 32;
  const int nt = f.nvox >= 64 * 4 * 192 ? 4 : (f.nvox >= 64 * 2 * 192 ? 2 : 1);
#define LDDMM_CASE(MT)                                            \
  if (mt == MT) {                                                 \
    if (dg) {                                                     \
      if (nt == 4) launch_km<true, MT, 4>(km, f, s);              \
      else if (nt == 2) launch_km<true, MT, 2>(km, f, s);         \
      else launch_km<true, MT, 1>(km, f, s);                      \
    } else {                                                      \
      if (nt == 4) launch_km<false, MT, 4>(km, f, s);             \
      else if (nt == 2) launch_km<false, MT, 2>(km, f, s);        \
      else launch_km<false, MT, 1>(km, f, s);                     \
    }                                                             \
  }
  LDDMM_CASE(1) LDDMM_CASE(2) LDDMM_CASE(4) LDDMM_CASE(6) LDDMM_CASE(8)
#undef LDDMM_CASE
  return true;
}

}  // namespace lddmm_cnn
