// Weight and bias gradients of the warm-start network's 3x3x3 convolutions on the
// bf16 matrix cores:
//   dw[m][tap][c] = sum over output voxels o of dy[o][m] x[s o + tap - 1][c],
//   db[m] = sum over o of dy[o][m].
//
// The sum runs over voxels, so both operands are needed with the voxel as the fast
// index while memory has the channel there.  A block stages a chunk of 2 x 8 x 8
// output voxels of dy and the halo of x once in LDS (straight from memory, double
// buffered) and reads fragments with the transposing LDS load (16 lanes give the
// addresses of 4 voxels x 16 channels and receive 4 voxels of one channel each),
// so nothing is shuffled and a tap only moves an LDS offset.
// A block owns the rows of RB output channels and the columns of KZ planes of taps
// times CB input channels; its wavefronts are WM groups of rows x 4 / WM groups of
// voxels, each with all the block's columns, so one dy fragment serves 9 to 27
// column tiles.  Two input channels (the network's first layer): a column tile
// holds 8 neighbouring voxels x 2 channels of one (kz, ky), of which the 3 taps
// are used; its rows start on odd voxels too, where an 8-byte LDS load may not, so
// the tile is staged twice, one voxel apart.
// The bias gradient is one more column tile of ones.
// The voxels are split over blocks whose FP32 partial tiles are added in a fixed
// order: results are deterministic.
// Weight and bias gradient together, us, batch 8 of 96^3 (k_conv_gemm with its transposing
// 2-byte LDS stores, a bias pass of 27 to 1728 blocks and one-thread sums of the splits):
// enc0 2051 -> 138, enc1 442 -> 97, decoder 532 -> 167, head 259 -> 99.
#include <algorithm>

#include "cnn_internal.h"
#include "internal.h"

namespace lddmm_cnn {
namespace {

constexpr int kBlk = 256;          // 4 wavefronts
typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
constexpr uint32_t kOut = 0xfffffff0u;   // past every operand (at most 0xffff0000 bytes)

struct WgradArgs {
  const u16* dy;
  const u16* x;
  float* part;                     // [nsplit][M][27 ci], then [nsplit][M]
  uint32_t dy_bytes, x_bytes;
  int n, d, h, w, ci;              // input
  int od, oh, ow, M;               // output extents and channels
  int ncz, ncy, ncx, nchunks;      // chunks per sample, and over all samples
  int nsplit, per;                 // chunks per split
  int ncb;                         // channel blocks
  int nkz;                         // column blocks along kz: 3 / KZ
  int bias;
};

template <int CB, int S, int MT, int WM, int KZ>
struct WgradGeom {
  static constexpr bool C2 = CB == 2;
  static constexpr int RB = WM * MT * 16;                    // rows of a block
  static constexpr int PZ = KZ == 3 ? S + 3 : 2;             // x planes of a chunk
  static constexpr int EY = 7 * S + 3, EX = C2 ? 16 : 7 * S + 3;
  static constexpr int XS = C2 ? 4 : CB * 2 + 16;            // bytes per voxel of x, 16 of padding
  static constexpr int DS = RB * 2 + 16;                     // of dy
  static constexpr int XV = PZ * EY * EX;
  static constexpr int XB = C2 ? (XV * 4 + 255) / 256 * 256 : (XV * XS + 1023) / 1024 * 1024;
  static constexpr int DB = (128 * DS + 1023) / 1024 * 1024;
  static constexpr int STAGE = XB * (C2 ? 2 : 1) + DB;       // one buffer
  static constexpr int NTL = C2 ? 3 * KZ : KZ * 9 * CB / 16; // column tiles of 16
  static constexpr int RED = WM * MT * (NTL + 1) * 1024;     // one wavefront's tiles per row group
  // zeros as far as a fragment's taps of one plane reach from its first voxel (see RAGGED)
  static constexpr int ZEROS = (((C2 ? 2 * EX : 2 * EX + 2) * XS + (C2 ? 32 : CB * 2)) + 15) / 16 * 16;
  static constexpr int lds(bool ragged) {
    const int used = 2 * STAGE + (ragged ? ZEROS : 0);
    return used > RED ? used : RED;
  }
};

// 16 or 4 bytes per lane from offset `off` of the buffer to LDS, the wavefront's first lane at
// `at` and the others behind it.
__device__ __forceinline__ void to_lds16(rsrc_t d, char* at, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(d, (__attribute__((address_space(3))) void*)at, 16, off,
                                           0, 0, 0);
}
__device__ __forceinline__ void to_lds4(rsrc_t d, char* at, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(d, (__attribute__((address_space(3))) void*)at, 4, off,
                                           0, 0, 0);
}

// Whether a staged unit at place p (plane | row << 8 | column << 16) of a chunk at (z0, y0, x0)
// lies on the grid; p < 0: padding.
__device__ __forceinline__ bool inside(int p, int z0, int y0, int x0, int nz, int ny, int nx) {
  return p >= 0 && (unsigned)(z0 + (p & 255)) < (unsigned)nz &&
         (unsigned)(y0 + ((p >> 8) & 255)) < (unsigned)ny && (unsigned)(x0 + (p >> 16)) < (unsigned)nx;
}

// A fragment: 8 consecutive k (voxels) of this lane's row or column, from two transposing loads.
typedef __attribute__((address_space(3))) char* lds_p;

__device__ __forceinline__ bf16x8 frag(lds_p lo, lds_p hi) {
  typedef __attribute__((address_space(3))) s16x4* lds_t;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)lo);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)hi);
  const s16x8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  return __builtin_bit_cast(bf16x8, r);
}

// DYV: dy rows are whole 16-byte units (M a multiple of 8), else staged value by value.
// RAGGED: some chunk reaches past the output (an extent not a multiple of 2 x 8 x 8).
template <int CB, int S, int MT, int WM, int KZ, bool DYV, bool RAGGED>
__global__ __launch_bounds__(kBlk) void k_wgrad(WgradArgs a) {
  using G = WgradGeom<CB, S, MT, WM, KZ>;
  constexpr int WK = 4 / WM, KST = 4 / WK;                   // k-steps per wavefront and chunk
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int lane = threadIdx.x & 63, g = lane >> 4, r = (lane >> 2) & 3, q = lane & 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wk = wave / WM;
  int yb = blockIdx.y;
  const int kz0 = yb % a.nkz * KZ;
  yb /= a.nkz;
  const int c0 = yb % a.ncb * CB, m0 = yb / a.ncb * G::RB;
  const int split = blockIdx.x;
  const rsrc_t X = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, (short)0, (int)a.x_bytes,
                                                     0x00020000);
  const rsrc_t D = __builtin_amdgcn_make_buffer_rsrc((void*)a.dy, (short)0, (int)a.dy_bytes,
                                                     0x00020000);

  // Each thread stages the same units of every chunk: their byte offsets from the chunk's first
  // voxel and their places in it (plane | row << 8 | column << 16, negative for padding) are
  // worked out once.  Done anew per chunk, these divisions and 32-bit products took most of
  // the kernel's time (decoder at 8 x 24^3: 227 us).
  constexpr int XIT = G::C2 ? (G::XB / 4 + kBlk - 1) / kBlk : (G::XB / 16 + kBlk - 1) / kBlk;
  constexpr int DIT = (G::DB / 16 + kBlk - 1) / kBlk;
  constexpr int ZS = KZ == 3 ? 1 : S;                        // source planes between staged ones
  uint32_t xo[XIT], dof[DIT];
  int xp_[XIT], dp_[DIT];
#pragma unroll
  for (int i = 0; i < XIT; ++i) {
    constexpr int U = G::C2 ? 1 : G::XS / 16;
    const int e = threadIdx.x + i * kBlk, v = e / U, c = e - v * U;
    const int x = v % G::EX, p = v / G::EX, y = p % G::EY, z = p / G::EY;
    xo[i] = ((uint32_t)((z * ZS * a.h + y) * a.w + x) * (uint32_t)a.ci + 8 * c) * 2u;
    xp_[i] = v < G::XV && (G::C2 || c < U - 1) ? z * ZS | y << 8 | x << 16 : -1;
  }
#pragma unroll
  for (int i = 0; i < DIT; ++i) {
    constexpr int U = G::DS / 16;
    const int e = threadIdx.x + i * kBlk, v = e / U, c = e - v * U;
    const int z = v >> 6, y = (v >> 3) & 7, x = v & 7;
    dof[i] = ((uint32_t)((z * a.oh + y) * a.ow + x) * (uint32_t)a.M + m0 + 8 * c) * 2u;
    dp_[i] = v < 128 && c < U - 1 && m0 + 8 * c < a.M ? z | y << 8 | x << 16 : -1;
  }
  // chunk ch into buffer buf; returns its first voxel on the output
  struct Place {
    int z, y, x;
  };
  auto stage = [&](int ch, int buf) {
    char* base = lds + buf * G::STAGE;
    const int cx = ch % a.ncx, t = ch / a.ncx, cy = t % a.ncy, t2 = t / a.ncy, cz = t2 % a.ncz,
              b = t2 / a.ncz;
    const int z0 = cz * 2, y0 = cy * 8, x0 = cx * 8;
    const int sz0 = KZ == 3 ? S * z0 - 1 : S * z0 + kz0 - 1, sy0 = S * y0 - 1, sx0 = S * x0 - 1;
    // of the first staged voxel, which may lie outside: the sums below wrap back
    const uint32_t xbase =
        ((uint32_t)(((b * a.d + sz0) * a.h + sy0) * a.w + sx0) * (uint32_t)a.ci + c0) * 2u;
    if constexpr (G::C2) {
#pragma unroll
      for (int copy = 0; copy < 2; ++copy)
#pragma unroll
        for (int i = 0; i < XIT; ++i) {
          const int e0 = wave * 64 + i * kBlk;
          if (e0 >= G::XB / 4) break;
          const bool in = inside(xp_[i], sz0, sy0, sx0 + copy, a.d, a.h, a.w);
          to_lds4(X, base + copy * G::XB + e0 * 4, in ? xbase + 4u * copy + xo[i] : kOut);
        }
    } else {
#pragma unroll
      for (int i = 0; i < XIT; ++i) {
        const int e0 = wave * 64 + i * kBlk;
        if (e0 >= G::XB / 16) break;
        const bool in = inside(xp_[i], sz0, sy0, sx0, a.d, a.h, a.w);
        to_lds16(X, base + e0 * 16, in ? xbase + xo[i] : kOut);
      }
    }
    char* db = base + G::XB * (G::C2 ? 2 : 1);
    if constexpr (DYV) {
      const uint32_t dbase = (uint32_t)(((b * a.od + z0) * a.oh + y0) * a.ow + x0) * (uint32_t)a.M * 2u;
#pragma unroll
      for (int i = 0; i < DIT; ++i) {
        const int e0 = wave * 64 + i * kBlk;
        if (e0 >= G::DB / 16) break;
        const bool in = inside(dp_[i], z0, y0, x0, a.od, a.oh, a.ow);
        to_lds16(D, db + e0 * 16, in ? dbase + dof[i] : kOut);
      }
    } else {
      constexpr int H = G::RB / 2;                           // pairs of channels per voxel
#pragma unroll 8
      for (int e = threadIdx.x; e < 128 * H; e += kBlk) {
        const int v = e / H, m = m0 + 2 * (e - v * H);
        const int iz = z0 + (v >> 6), iy = y0 + ((v >> 3) & 7), ix = x0 + (v & 7);
        uint32_t val = 0;
        if (m < a.M && iz < a.od && iy < a.oh && ix < a.ow) {
          const u16* p = a.dy + (long)(((b * a.od + iz) * a.oh + iy) * a.ow + ix) * a.M + m;
          val = p[0] | (m + 1 < a.M ? (uint32_t)p[1] << 16 : 0u);
        }
        *reinterpret_cast<uint32_t*>(db + v * G::DS + 4 * (e - v * H)) = val;
      }
    }
    return Place{z0, y0, x0};
  };

  f32x4 acc[MT][G::NTL], accb[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < G::NTL; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  s16x8 one8;
#pragma unroll
  for (int e = 0; e < 8; ++e) one8[e] = 0x3f80;              // 1.0 in bf16
  const bf16x8 ones = __builtin_bit_cast(bf16x8, one8);
  const bool bias = a.bias && kz0 == 0 && c0 == 0;

  // k = 8 g + 4 h + r of a k-step is the voxel (plane, row 4 half + g, column 4 h + r).  Voxels of
  // a ragged chunk that lie past the output have zero dy, but their x may be real voxels of the
  // last plane, row or column, which would enter taps that do not use them as 0 * inf.  RAGGED
  // reads zeros in their place: a lane gives the addresses of one voxel of each half, so it points
  // them at a block of zeros.  The compiler then reads each fragment just before its products, so
  // the order is given: three fragments ahead.  Decoder at 4 x 23^3 93 us, as without the zeros;
  // 104 in the compiler's order, 110 with fragments masked after the read.
  char* const zeros = lds + 2 * G::STAGE;
  if constexpr (RAGGED)
    for (int i = threadIdx.x; i < G::ZEROS / 4; i += kBlk) reinterpret_cast<uint32_t*>(zeros)[i] = 0u;
  const int ch0 = split * a.per, ch1 = ch0 + a.per < a.nchunks ? ch0 + a.per : a.nchunks;
  Place next{};
  if (ch0 < ch1) next = stage(ch0, 0);
  for (int ch = ch0; ch < ch1; ++ch) {
    const int buf = (ch - ch0) & 1;
    __builtin_amdgcn_s_waitcnt(0x0f70);                      // this chunk's LDS writes (vmcnt 0)
    __syncthreads();
    const Place at = next;
    if (ch + 1 < ch1) next = stage(ch + 1, buf ^ 1);
    const char* xb = lds + buf * G::STAGE;
    const char* db = xb + G::XB * (G::C2 ? 2 : 1);
    const int planes = a.od - at.z, rows = a.oh - at.y, cols = a.ow - at.x;   // inside, or more
#pragma unroll
    for (int s = 0; s < KST; ++s) {
      const int ks = wk * KST + s, vz = ks >> 1, vy = (ks & 1) * 4 + g;
      const char* dp = db + ((vz * 8 + vy) * 8 + r) * G::DS + (wm * MT * 16 + 4 * q) * 2;
      // addresses of the lane's voxels of both halves (p, p + half) for each plane of taps
      lds_p lo[KZ], hi[KZ];
      auto voxels = [&](const char* p, int half, int plane) {
        const bool in = vz < planes && vy < rows;
#pragma unroll
        for (int k = 0; k < KZ; ++k) {
          lo[k] = (lds_p)(p + k * plane);
          hi[k] = lo[k] + half;
          if (RAGGED) {
            lo[k] = in && r < cols ? lo[k] : (lds_p)zeros + 8 * q;
            hi[k] = in && r + 4 < cols ? hi[k] : (lds_p)zeros + 8 * q;
          }
        }
      };
      bf16x8 fa[MT];
#pragma unroll
      for (int i = 0; i < MT; ++i) fa[i] = frag((lds_p)dp + i * 32, (lds_p)dp + 4 * G::DS + i * 32);
      if constexpr (G::C2) {
        // tile t: kz = t / 3, ky = t % 3; columns are voxels x - 1 .. x + 6, two channels each;
        // an odd start takes the copy that is one voxel ahead
        voxels(xb + (r & 1) * G::XB + ((vz * G::EY + vy) * G::EX + r - (r & 1)) * 4 + 8 * q, 16,
               G::EY * G::EX * 4);
#pragma unroll
        for (int t = 0; t < G::NTL; ++t) {
          const int off = t % 3 * G::EX * 4;
          const bf16x8 fb = frag(lo[t / 3] + off, hi[t / 3] + off);
#pragma unroll
          for (int i = 0; i < MT; ++i)
            acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb, acc[i][t], 0, 0, 0);
        }
      } else {
        constexpr int PT = CB / 16;                          // column tiles per tap
        constexpr int ZP = KZ == 3 ? S : 1;                  // staged planes between output planes
        voxels(xb + ((vz * ZP * G::EY + vy * S) * G::EX + r * S) * G::XS + 8 * q, 4 * S * G::XS,
               G::EY * G::EX * G::XS);
        auto tile = [&](int t) {
          const int tap = t / PT, kz = tap / 9, ky = tap / 3 % 3, kx = tap % 3;
          const int off = (ky * G::EX + kx) * G::XS + (t % PT) * 32;
          return frag(lo[kz] + off, hi[kz] + off);
        };
        constexpr int AHEAD = RAGGED ? 3 : 0;                // fragments read ahead (see RAGGED)
        bf16x8 fb[AHEAD + 1];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) fb[t] = tile(t);
#pragma unroll
        for (int t = 0; t < G::NTL; ++t) {
          if (t + AHEAD < G::NTL) fb[(t + AHEAD) % (AHEAD + 1)] = tile(t + AHEAD);
#pragma unroll
          for (int i = 0; i < MT; ++i)
            acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[t % (AHEAD + 1)],
                                                                acc[i][t], 0, 0, 0);
          if (RAGGED) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (bias) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
          accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], ones, accb[i], 0, 0, 0);
      }
    }
  }

  // ---- the voxel groups' tiles onto the first group's, one group after the other
  f32x4* red = reinterpret_cast<f32x4*>(lds) + wm * MT * (G::NTL + 1) * 64 + lane;
  for (int k = 1; k < WK; ++k) {
    __syncthreads();
    if (wk == k) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int t = 0; t < G::NTL; ++t) red[(i * (G::NTL + 1) + t) * 64] = acc[i][t];
        red[(i * (G::NTL + 1) + G::NTL) * 64] = accb[i];
      }
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int t = 0; t < G::NTL; ++t) acc[i][t] += red[(i * (G::NTL + 1) + t) * 64];
        accb[i] += red[(i * (G::NTL + 1) + G::NTL) * 64];
      }
    }
  }
  if (wk != 0) return;
  const long N = 27L * a.ci;
  const int col = lane & 15;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int row = m0 + (wm * MT + i) * 16 + 4 * g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (row + e >= a.M) continue;
      float* out = a.part + ((long)split * a.M + row + e) * N;
#pragma unroll
      for (int t = 0; t < G::NTL; ++t) {
        if constexpr (G::C2) {
          if (col < 6) out[((kz0 + t / 3) * 9 + t % 3 * 3) * 2 + col] = acc[i][t][e];
        } else {
          constexpr int PT = CB / 16;
          out[(long)(kz0 * 9 + t / PT) * a.ci + c0 + (t % PT) * 16 + col] = acc[i][t][e];
        }
      }
      if (bias && col == 0)
        a.part[(long)a.nsplit * a.M * N + (long)split * a.M + row + e] = accb[i][e];
    }
  }
}

// dw and db from the partial tiles: 64 neighbouring values per block, the splits dealt to four
// groups of 64 threads, each adding its own in order.
__global__ __launch_bounds__(kBlk) void k_wgrad_sum(const float* __restrict__ part, int nsplit,
                                                    long nw, int M, float* __restrict__ dw,
                                                    float* __restrict__ db) {
  __shared__ float red[4][64];
  const int l = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const long i = (long)blockIdx.x * 64 + l;
  const long total = nw + (db ? M : 0);
  const float* p = i < nw ? part + i : part + (long)nsplit * nw + (i - nw);
  const long stride = i < nw ? nw : M;
  float v = 0.f;
  if (i < total) {
#pragma unroll 8
    for (int s = grp; s < nsplit; s += 4) v += p[(long)s * stride];
  }
  red[grp][l] = v;
  __syncthreads();
  if (grp != 0 || i >= total) return;
  v = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
  if (i < nw)
    dw[i] = v;
  else
    db[i - nw] = v;
}

template <int CB, int S, int MT, int WM, int KZ>
int launch_one(WgradArgs a, long max_split, int target, hipStream_t s) {
  using G = WgradGeom<CB, S, MT, WM, KZ>;
  static_assert(G::lds(true) <= 160 * 1024, "fits the CU");
  a.nkz = 3 / KZ;
  a.ncb = a.ci / CB;
  const int ny = a.nkz * a.ncb * ((a.M + G::RB - 1) / G::RB);
  // Splits: a multiple of 8 where there are that many, so that the column blocks of a split run
  // on one XCD and read its chunks behind one L2; but not where that leaves splits without a
  // chunk and makes the others longer.  At most 7 are empty (they write zeros).
  auto chunks_per = [&](long n) { return (a.nchunks + n - 1) / n; };
  const long most = std::min<long>({std::max(1, target / ny), max_split, (long)a.nchunks});
  long ns = most > 8 ? most / 8 * 8 : most;
  if ((ns - 1) * chunks_per(ns) >= a.nchunks && chunks_per(most) < chunks_per(ns)) ns = most;
  a.per = (int)chunks_per(ns);
  const long busy = chunks_per(a.per);
  a.nsplit = (int)std::min(ns, busy > 8 ? (busy + 7) / 8 * 8 : busy);
  const dim3 grid(a.nsplit, ny);
  const bool ragged = a.od % 2 || a.oh % 8 || a.ow % 8;
  auto kernel = a.M % 8 == 0 ? (ragged ? k_wgrad<CB, S, MT, WM, KZ, true, true>
                                       : k_wgrad<CB, S, MT, WM, KZ, true, false>)
                             : (ragged ? k_wgrad<CB, S, MT, WM, KZ, false, true>
                                       : k_wgrad<CB, S, MT, WM, KZ, false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kBlk), G::lds(ragged), s, a);
  return a.nsplit;
}

}  // namespace

bool launch_wgrad(const ConvArgs& c, float* dw, float* db, float* part, size_t part_floats,
                  hipStream_t s) {
  WgradArgs a{};
  a.n = c.n;
  a.d = c.d;
  a.h = c.h;
  a.w = c.w;
  a.ci = c.ci;
  a.od = c.od;
  a.oh = c.oh;
  a.ow = c.ow;
  a.M = c.co;
  const long long xb = 2LL * c.n * c.d * c.h * c.w * c.ci;
  const long long yb = 2LL * c.n * c.od * c.oh * c.ow * c.co;
  if (xb > 0xffff0000LL || yb > 0xffff0000LL) return false;
  const bool c2 = c.ci == 2 && c.s == 1, c16 = c.ci % 16 == 0;
  if (!c2 && !c16) return false;
  if (((uintptr_t)c.x & (c2 ? 3 : 15)) || (c.co % 8 == 0 && ((uintptr_t)c.wb & 15))) return false;
  a.x = c.x;
  a.dy = c.wb;
  a.x_bytes = (uint32_t)xb;
  a.dy_bytes = (uint32_t)yb;
  a.part = part;
  a.bias = db != nullptr;
  a.ncz = (c.od + 1) / 2;
  a.ncy = (c.oh + 7) / 8;
  a.ncx = (c.ow + 7) / 8;
  const long long nch = (long long)c.n * a.ncz * a.ncy * a.ncx;
  if (nch > 0x3fffffff) return false;
  a.nchunks = (int)nch;
  const long nw = 27L * c.ci * c.co;
  const long most = (long)(part_floats / (size_t)(nw + c.co));
  if (most < 1) return false;
#define LDDMM_WGRAD(CB, S, KZ, TARGET)                                          \
  do {                                                                          \
    if (a.M <= 16) ns = launch_one<CB, S, 1, 1, KZ>(a, most, TARGET, s);             \
    else if (a.M <= 32) ns = launch_one<CB, S, 2, 1, KZ>(a, most, TARGET, s);        \
    else ns = launch_one<CB, S, 2, 2, KZ>(a, most, TARGET, s);                       \
  } while (0)
  int ns = 0;
  if (c2) {
    LDDMM_WGRAD(2, 1, 3, 2048);
  } else if (c.ci % 32 == 0) {
    if (c.s == 1) LDDMM_WGRAD(32, 1, 1, 512);
    else LDDMM_WGRAD(32, 2, 1, 256);
  } else if (c.s == 1) {
    LDDMM_WGRAD(16, 1, 3, 512);
  } else if (a.M <= 32) {
    if (a.M <= 16) ns = launch_one<16, 2, 1, 1, 3>(a, most, 256, s);
    else ns = launch_one<16, 2, 2, 1, 3>(a, most, 256, s);
  } else {
    ns = launch_one<16, 2, 2, 2, 1>(a, most, 512, s);
  }
#undef LDDMM_WGRAD
  const long total = nw + (db ? c.co : 0);
  hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)((total + 63) / 64)), dim3(kBlk), 0, s, part, ns, nw,
                     (int)c.co, dw, db);
  return true;
}

}  // namespace lddmm_cnn
