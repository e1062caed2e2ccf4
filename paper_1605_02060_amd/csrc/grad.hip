// Exact gradient of the discrete energy (reverse mode through the forward sweep).
//
// Forward sweep (Methods, Registration, semi-Lagrangian reading):
//   u_{j+1}(x) = -dt v_j(x) + S_clamp(u_j; y_j(x)),   y_j(x) = x - dt v_j(x)/h,
//   E = R(v) + (h^3/sigma^2) sum_c w_c sum_x (S_zero(J0c; x + u_T/h) - J1c)^2.
// Reverse sweep, with ubar_j = dE/du_j:
//   ubar_T  = (2 h^3/sigma^2) sum_c w_c r_c (1/h) grad_y S_zero(J0c; y)|_{y = x + u_T/h}
//   vbar_j  = -dt ubar_{j+1} - (dt/h) (d_y S_clamp(u_j; y_j))^T ubar_{j+1}
//   ubar_j  = S_clamp(.; y_j)^T ubar_{j+1}                       (adjoint of sampling)
//   dE/dv_j = vbar_j + 2 dt h^3 L(L v_j),   L = gamma - alpha Lap (periodic).
// The adjoint of sampling is evaluated as a gather: output voxel z sums the
// contributions of every source x whose clamped cell has z as a corner.  With
// |dt v/h| < Rr along every axis those sources satisfy |x - z| <= Rr, so the
// sum is over a (2 Rr + 1)^3 neighbourhood in a fixed order: deterministic.
#include "device.h"

namespace lddmm {

static inline unsigned grid_for(long long n) {
  long long b = (n + kBlock - 1) / kBlock;
  if (b > 65536) b = 65536;
  return (unsigned)(b < 1 ? 1 : b);
}

// ----------------------------------------------------------- d/dy of samplers

// Trilinear interpolant and its derivatives at a cell (corners loaded by caller).
struct TriD {
  float d[3];
};

__device__ __forceinline__ TriD tri_deriv(float v000, float v100, float v010, float v110,
                                          float v001, float v101, float v011, float v111,
                                          float fx, float fy, float fz) {
  const float gx = 1.f - fx, gy = 1.f - fy, gz = 1.f - fz;
  TriD t;
  t.d[0] = gy * gz * (v100 - v000) + fy * gz * (v110 - v010) + gy * fz * (v101 - v001) +
           fy * fz * (v111 - v011);
  t.d[1] = gx * gz * (v010 - v000) + fx * gz * (v110 - v100) + gx * fz * (v011 - v001) +
           fx * fz * (v111 - v101);
  t.d[2] = gx * gy * (v001 - v000) + fx * gy * (v101 - v100) + gx * fy * (v011 - v010) +
           fx * fy * (v111 - v110);
  return t;
}

__device__ __forceinline__ TriD tri_deriv_cell(rsrc_t r, const Cell& c) {
  return tri_deriv(bld(r, c.o[0]), bld(r, c.o[1]), bld(r, c.o[2]), bld(r, c.o[3]), bld(r, c.o[4]),
                   bld(r, c.o[5]), bld(r, c.o[6]), bld(r, c.o[7]), c.fx, c.fy, c.fz);
}

// Axis clamped?  (y outside [0, n-1]; the derivative along it is zero.)
__device__ __forceinline__ bool clamped(int i, float d, int n) {
  d = fminf(fmaxf(d, -(float)(n + 2)), (float)(n + 2));
  const float y = (float)i + d;
  return y < 0.f || y > (float)(n - 1);
}

// ------------------------------------------------------------------ kernels

constexpr int kSplatMaxR = 3;

// ubar_T = coef * sum_c w_c r_c (1/h) grad_y S_zero(J0c; x + u_T/h)
template <int NC>
__global__ __launch_bounds__(kBlock) void k_ubar_init(GradArgs a) {
  const Geom g = a.g;
  const long long N = g.n;
  const uint32_t n = (uint32_t)N;
  const rsrc_t U0 = rsrc(a.u, n), U1 = rsrc(a.u + N, n), U2 = rsrc(a.u + 2 * N, n);
  const rsrc_t O0 = rsrc(a.ub_out, n), O1 = rsrc(a.ub_out + N, n), O2 = rsrc(a.ub_out + 2 * N, n);
  rsrc_t T0[NC], RR[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    T0[c] = rsrc(a.J0 + (long long)a.ch[c] * N, n);
    RR[c] = rsrc(a.r + (long long)c * N, n);
  }
  const float ih = g.inv_h;
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    int x, y, z;
    vcoord(g, i, x, y, z);
    const Cell cz = make_cell_zero(g, x, y, z, bld(U0, i) * ih, bld(U1, i) * ih, bld(U2, i) * ih);
    float gx = 0.f, gy = 0.f, gz = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const TriD t = tri_deriv_cell(T0[c], cz);
      const float s = a.coef * a.wc[c] * bld(RR[c], i) * ih;
      gx += s * t.d[0];
      gy += s * t.d[1];
      gz += s * t.d[2];
    }
    bst(O0, i, gx);
    bst(O1, i, gy);
    bst(O2, i, gz);
  }
}

// w = L v_j (periodic 7-point Laplacian), and each block's largest |v_j| of any
// component, which bounds the splat's reach.  This pass reads v_j anyway, so the
// maximum costs no traffic: a pass of its own over v_j by one block took 2553 us
// at 128^3 (10 GB/s) and was 92 % of the whole gradient's time.  Every block
// stores its own maximum and k_coord_grad's first block reduces them: an atomic
// maximum on one address took this pass from 14 to 50 us with 8192 blocks and
// to 32 us with 1024.  NaN components are passed over, as fmaxf does.
constexpr unsigned kMaxParts = 2 * kPartMax;   // floats in one step's worth of min-det partials

__device__ __forceinline__ void Lv_body(const GradArgs& a, const float* v, uint32_t nblocks) {
  const Geom g = a.g;
  const long long N = g.n;
  const uint32_t n = (uint32_t)N;
  const float c2 = a.alpha * g.inv_h * g.inv_h;
  float m = 0.f;
  for (int c = 0; c < 3; ++c) {
    const rsrc_t V = rsrc(v + c * N, n), W = rsrc(a.w + c * N, n);
    for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += nblocks * kBlock) {
      int x, y, z;
      vcoord(g, i, x, y, z);
      const Nbr nb = periodic_nbr(g, i, x, y, z);
      const float v0 = bld(V, i);
      m = fmaxf(m, fabsf(v0));
      bst(W, i, a.gamma * v0 - c2 * lap7_b(V, nb, v0));
    }
  }
  __shared__ float red[kBlock / 64];
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_down(m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kBlock / 64; ++k) m = fmaxf(m, red[k]);
    a.vpart[blockIdx.x] = m;
  }
}

__global__ __launch_bounds__(kBlock) void k_Lv(GradArgs a) { Lv_body(a, a.v, gridDim.x); }

// Splat radius: floor(max_x max_axis |dt v_j / h|) + 1 (at least one source
// further than any displacement reaches).
__device__ __forceinline__ int splat_radius(const GradArgs& a) {
  const float d = *a.vmax * (a.dt * a.g.inv_h);
  return (int)floorf(fminf(d, 1e6f)) + 1;
}

// dE/dv_j = -dt ubar - (dt/h) (d_y S_clamp(u_j; y_j))^T ubar + reg * L w
__global__ __launch_bounds__(kBlock) void k_coord_grad(GradArgs a) {
  const Geom g = a.g;
  const long long N = g.n;
  const uint32_t n = (uint32_t)N;
  const rsrc_t V0 = rsrc(a.v, n), V1 = rsrc(a.v + N, n), V2 = rsrc(a.v + 2 * N, n);
  const rsrc_t U0 = rsrc(a.u, n), U1 = rsrc(a.u + N, n), U2 = rsrc(a.u + 2 * N, n);
  const rsrc_t B0 = rsrc(a.ub_in, n), B1 = rsrc(a.ub_in + N, n), B2 = rsrc(a.ub_in + 2 * N, n);
  const rsrc_t W0 = rsrc(a.w, n), W1 = rsrc(a.w + N, n), W2 = rsrc(a.w + 2 * N, n);
  const rsrc_t G0 = rsrc(a.grad, n), G1 = rsrc(a.grad + N, n), G2 = rsrc(a.grad + 2 * N, n);
  const float dt = a.dt, ih = g.inv_h;
  const float c2 = a.alpha * ih * ih;
  if (blockIdx.x == 0) {             // the step's largest |v_j| from k_Lv's blocks
    __shared__ float red[kBlock / 64];
    float m = 0.f;
#pragma unroll 8
    for (int k = threadIdx.x; k < a.nvpart; k += kBlock) m = fmaxf(m, a.vpart[k]);
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_down(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int k = 1; k < kBlock / 64; ++k) m = fmaxf(m, red[k]);
      *a.vmax = m;
    }
  }
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    int x, y, z;
    vcoord(g, i, x, y, z);
    const float dx = -dt * bld(V0, i) * ih, dy = -dt * bld(V1, i) * ih, dz = -dt * bld(V2, i) * ih;
    const Cell cl = make_cell_clamp(g, x, y, z, dx, dy, dz);
    const bool kx = clamped(x, dx, g.nx), ky = clamped(y, dy, g.ny), kz = clamped(z, dz, g.nz);
    const float b0 = bld(B0, i), b1 = bld(B1, i), b2 = bld(B2, i);
    // J[a][b] = d S(u_j[a]) / d y_b ; vbar_b = -dt ub_b - (dt/h) sum_a J[a][b] ub_a
    const TriD t0 = tri_deriv_cell(U0, cl), t1 = tri_deriv_cell(U1, cl), t2 = tri_deriv_cell(U2, cl);
    float vb[3];
    const float bb[3] = {b0, b1, b2};
    const bool kc[3] = {kx, ky, kz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float jt = kc[d] ? 0.f : (t0.d[d] * b0 + t1.d[d] * b1 + t2.d[d] * b2);
      vb[d] = -dt * bb[d] - dt * ih * jt;
    }
    const Nbr nb = periodic_nbr(g, i, x, y, z);
    const float w0 = bld(W0, i), w1 = bld(W1, i), w2 = bld(W2, i);
    bst(G0, i, vb[0] + a.reg * (a.gamma * w0 - c2 * lap7_b(W0, nb, w0)));
    bst(G1, i, vb[1] + a.reg * (a.gamma * w1 - c2 * lap7_b(W1, nb, w1)));
    bst(G2, i, vb[2] + a.reg * (a.gamma * w2 - c2 * lap7_b(W2, nb, w2)));
  }
}

// ubar_j(z) = sum over sources x with z a corner of x's clamped cell of weight * ubar_{j+1}(x)
//
// Reach 1 (|dt v_j / h| < 1 everywhere, the usual case): a block owns a kSX x kSY
// column of (x, y) and marches up a run of planes with a ring of three source
// planes (halo 1) in LDS.  A source's cell, fractions and ubar are worked out
// once per staged value instead of once per (output, source) pair, and of the
// 27 sources of an output only those offsets are visited that some source of
// the staged planes can reach: per axis a cell offset of 0 reaches outputs 0 and
// +1, one of -1 reaches -1 and 0, so where the displacement keeps its sign over
// the tile two of the three offsets per axis remain (8 sources of 27).  A skipped
// source contributes nothing and the visited ones keep their order, so the sums
// are those of the general body, which larger reaches run, to the rounding of an fma.  The general body
// spent its time on address and cell arithmetic (27 x about 30 instructions per
// output): 91.2 us at 128^3 against 54.9 us staged.
// Below kStagedVoxels it runs all reaches: its blocks then fill the chip at once, where the staged
// one's few march with one memory latency per plane (35 us a step at 32^3 against 13).  Whole call,
// T = 10, staged against general: 32^3 488 and 239 us, 64^3 554 and 363, 80^3 691 and 647,
// 96^3 839 and 920, 112^3 1171 and 1462.
constexpr long long kStagedVoxels = 655360;
constexpr int kSX = 64, kSY = 4;
constexpr int kSXH = kSX + 2, kSYH = kSY + 2;
constexpr int kSPlane = kSXH * kSYH;

struct SplatTiling {
  int ntx, nty, nrun, run;       // tiles along x, y; runs of `run` planes
};

// About 1024 blocks (four of 33 KB fit a CU, so 1024 are one round of the chip: 1216
// left a second round nearly empty), with runs of at least 6 planes (a run
// stages two planes more than it writes).
__host__ __device__ inline SplatTiling splat_tiling(const Geom& g) {
  SplatTiling t;
  t.ntx = (g.nx + kSX - 1) / kSX;
  t.nty = (g.ny + kSY - 1) / kSY;
  const int cols = t.ntx * t.nty;
  int want = 1024 / cols < 1 ? 1 : 1024 / cols;
  const int most = g.nz / 6 < 1 ? 1 : g.nz / 6;
  want = want > most ? most : want;
  t.run = (g.nz + want - 1) / want;
  t.nrun = (g.nz + t.run - 1) / t.run;
  return t;
}

// Cell minus source index per axis in one byte each (+ 8), so that one subtraction
// from an output's offset leaves the output's corner of the cell, ex | ey << 8 |
// ez << 16 (+ 8 each): bytes of 8 or 9 where the source reaches the output.
struct SplatPlane {
  float f[3][kSPlane];           // cell fractions, 0 outside the grid
  float b[3][kSPlane];           // ubar_{j+1}, 0 outside the grid
  uint32_t e[kSPlane];
};
constexpr uint32_t kByte8 = 0x080808u, kNoSource = 0x0c0c0cu;   // 4 past: reaches no output

// Sources at own + (oz, oy, ox) of the ring, ox in [XL, XL + NX): their sum onto the output.
template <bool UNIFORM, int NX>
__device__ __forceinline__ void splat_row(const SplatPlane& s, int at, int xl, uint32_t k,
                                          bool ey, bool ez, float& s0, float& s1, float& s2) {
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    const int i = at + xl + q;
    const float fx = s.f[0][i], fy = s.f[1][i], fz = s.f[2][i];
    if (UNIFORM) {               // two offsets per axis, the first the far corner of its cell
      const float w = (q == 0 ? fx : 1.f - fx) * (ey ? fy : 1.f - fy) * (ez ? fz : 1.f - fz);
      s0 += w * s.b[0][i];
      s1 += w * s.b[1][i];
      s2 += w * s.b[2][i];
    } else {
      const uint32_t d = k - (uint32_t)q - s.e[i] + kByte8;
      const float w = ((d & 1u) ? fx : 1.f - fx) * ((d & 0x100u) ? fy : 1.f - fy) *
                      ((d & 0x10000u) ? fz : 1.f - fz);
      const bool ok = (d & 0xfefefeu) == kByte8;
      const float c0 = w * s.b[0][i], c1 = w * s.b[1][i], c2 = w * s.b[2][i];
      s0 += ok ? c0 : 0.f;
      s1 += ok ? c1 : 0.f;
      s2 += ok ? c2 : 0.f;
    }
  }
}

__device__ __forceinline__ void splat_staged(const GradArgs& a, uint32_t block, uint32_t nblocks) {
  __shared__ SplatPlane ring[3];
  // of each row of plane p, in [p mod 4]: bit 2 axis: some offset of 0, bit 2 axis + 1: of -1
  // (any other, from a NaN: both)
  __shared__ int reach[4][kSYH];
  const Geom g = a.g;
  const uint32_t n = (uint32_t)g.n;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const uint32_t nxy = (uint32_t)(nx * ny);
  const rsrc_t V = rsrc(a.v, 3u * n), B = rsrc(a.ub_in, 3u * n);
  const rsrc_t O = rsrc(a.ub_out, 3u * n);
  const SplatTiling tl = splat_tiling(g);
  // contiguous runs of tiles per XCD (block b runs on XCD b mod 8; nblocks is a multiple of 8)
  const uint32_t l = (block % kXCD) * (nblocks / kXCD) + block / kXCD;
  const int cols = tl.ntx * tl.nty;
  const int r = (int)l / cols, col = (int)l % cols;
  if (r >= tl.nrun) return;
  const int x0 = (col % tl.ntx) * kSX, y0 = (col / tl.ntx) * kSY;
  const int z0 = r * tl.run, z1 = z0 + tl.run < nz ? z0 + tl.run : nz;
  const float dt = a.dt, ih = g.inv_h;
  // staged values of a thread: first its wavefront's row of 64 columns, then rows
  // 4 and 5 (wavefronts 0, 1) and the last two columns of every row (wavefront 2),
  // so that a row's reach is one ballot per bit
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  static_assert(kSX == 64 && kSY == 4 && kBlock == 256, "one wavefront per row");
  int row[2], colx[2], sx[2], sy[2], at[2];
  bool in[2], has[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool edge = q == 1 && wave == 2;
    row[q] = q == 0 ? wave : (edge ? lane >> 1 : 4 + wave);
    colx[q] = edge ? 64 + (lane & 1) : lane;
    has[q] = q == 0 || wave < 2 || (edge && lane < 2 * kSYH);
    sy[q] = y0 - 1 + row[q];
    sx[q] = x0 - 1 + colx[q];
    at[q] = row[q] * kSXH + colx[q];
    in[q] = has[q] && (unsigned)sx[q] < (unsigned)nx && (unsigned)sy[q] < (unsigned)ny;
  }
  float rv[2][3], rb[2][3];
  auto fetch = [&](int p) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool ok = in[q] && p >= 0 && p < nz;
      const uint32_t i = (uint32_t)p * nxy + (uint32_t)(sy[q] * nx + sx[q]);
#pragma unroll
      for (int c = 0; c < 3; ++c) {                          // out of range: reads 0
        rv[q][c] = bld(V, ok ? i + (uint32_t)c * n : kOutside);
        rb[q][c] = bld(B, ok ? i + (uint32_t)c * n : kOutside);
      }
    }
  };
  auto put = [&](int p) {
    SplatPlane& s = ring[(p + 3) % 3];
    if (threadIdx.x < kSYH) reach[(p + 5) & 3][threadIdx.x] = 0;        // of the plane after this one
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      int mine = 0;
      if (has[q]) {
        const int e = at[q];
        uint32_t off = kNoSource;
        s.b[0][e] = rb[q][0];
        s.b[1][e] = rb[q][1];
        s.b[2][e] = rb[q][2];
        if (in[q] && p >= 0 && p < nz) {
          int cx, cy, cz;
          cell_clamp(sx[q], -dt * rv[q][0] * ih, nx, cx, s.f[0][e]);
          cell_clamp(sy[q], -dt * rv[q][1] * ih, ny, cy, s.f[1][e]);
          cell_clamp(p, -dt * rv[q][2] * ih, nz, cz, s.f[2][e]);
          // offsets past +-4 (from NaN only) reach nothing either way
          const int dx = min(max(cx - sx[q], -4), 4), dy = min(max(cy - sy[q], -4), 4),
                    dz = min(max(cz - p, -4), 4);
          off = (uint32_t)(dx + 8) | (uint32_t)(dy + 8) << 8 | (uint32_t)(dz + 8) << 16;
          mine = (dx == 0 ? 1 : (dx == -1 ? 2 : 3)) | (dy == 0 ? 4 : (dy == -1 ? 8 : 12)) |
                 (dz == 0 ? 16 : (dz == -1 ? 32 : 48));
        } else {
          s.f[0][e] = s.f[1][e] = s.f[2][e] = 0.f;
        }
        s.e[e] = off;
      }
      if (q == 1 && wave == 2) {                              // one lane per value: two per row
        if (mine) atomicOr(&reach[(p + 4) & 3][row[q]], mine);
      } else if (q == 0 || wave < 2) {
        int any = 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) any |= __any(mine & (1 << k)) ? 1 << k : 0;
        if (lane == 0 && any) atomicOr(&reach[(p + 4) & 3][row[q]], any);
      }
    }
  };
  if (threadIdx.x < 4 * kSYH) reach[threadIdx.x / kSYH][threadIdx.x % kSYH] = 0;
  __syncthreads();
  fetch(z0 - 1);
  put(z0 - 1);
  fetch(z0);
  __syncthreads();
  put(z0);
  fetch(z0 + 1);
  const int tx = threadIdx.x % kSX, ty = threadIdx.x / kSX;
  const int x = x0 + tx, y = y0 + ty;
  const bool inside = x < nx && y < ny;
  const int own = (ty + 1) * kSXH + tx + 1;
  __syncthreads();
  for (int z = z0; z < z1; ++z) {
    put(z + 1);
    __syncthreads();
    if (z + 1 < z1) fetch(z + 2);
    if (inside) {
      float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int oz = -1; oz <= 1; ++oz) {
        const SplatPlane& s = ring[(z + oz + 3) % 3];
#pragma unroll
        for (int oy = -1; oy <= 1; ++oy) {
          // what this row of sources reaches (the same for the whole wavefront)
          const int fl = __builtin_amdgcn_readfirstlane(reach[(z + oz + 4) & 3][ty + 1 + oy]);
          if (fl == 0 || (oz == -1 && !(fl & 16)) || (oz == 1 && !(fl & 32)) ||
              (oy == -1 && !(fl & 4)) || (oy == 1 && !(fl & 8)))
            continue;
          const int i = own + oy * kSXH;
          const int xl = (fl & 1) ? -1 : 0;
          // the output's offset from the row's first source, + 8 per byte
          const uint32_t k = (uint32_t)(8 - xl) | (uint32_t)(8 - oy) << 8 | (uint32_t)(8 - oz) << 16;
          // one sign per axis (one bit of each pair set): both sources of the row reach the
          // output at known corners
          if ((fl & (fl >> 1) & 0x15) == 0)
            splat_row<true, 2>(s, i, xl, k, oy == ((fl & 4) ? -1 : 0), oz == ((fl & 16) ? -1 : 0),
                               s0, s1, s2);
          else if ((fl & 3) == 3)
            splat_row<false, 3>(s, i, xl, k, false, false, s0, s1, s2);
          else
            splat_row<false, 2>(s, i, xl, k, false, false, s0, s1, s2);
        }
      }
      const uint32_t i = (uint32_t)z * nxy + (uint32_t)(y * nx + x);
      bst(O, i, s0);
      bst(O, i + n, s1);
      bst(O, i + 2 * n, s2);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void k_splat_staged(GradArgs a) {
  if (splat_radius(a) == 1) splat_staged(a, blockIdx.x, gridDim.x);   // uniform over the grid
}

// Any reach: each output looks at every source within it.
__device__ __forceinline__ void splat_any(const GradArgs& a, uint32_t block, uint32_t nblocks) {
  const Geom g = a.g;
  const long long N = g.n;
  const uint32_t n = (uint32_t)N;
  int Rr = splat_radius(a);
  if (Rr == 1 && a.staged) return;
  const rsrc_t V0 = rsrc(a.v, n), V1 = rsrc(a.v + N, n), V2 = rsrc(a.v + 2 * N, n);
  const rsrc_t B0 = rsrc(a.ub_in, n), B1 = rsrc(a.ub_in + N, n), B2 = rsrc(a.ub_in + 2 * N, n);
  const rsrc_t O0 = rsrc(a.ub_out, n), O1 = rsrc(a.ub_out + N, n), O2 = rsrc(a.ub_out + 2 * N, n);
  if (Rr > kSplatMaxR) {
    if (block == 0 && threadIdx.x == 0) *a.overflow = 1;
    Rr = kSplatMaxR;
  }
  const float dt = a.dt, ih = g.inv_h;
  for (uint32_t i = block * kBlock + threadIdx.x; i < n; i += nblocks * kBlock) {
    int zx, zy, zz;
    vcoord(g, i, zx, zy, zz);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f;
    for (int oz = -Rr; oz <= Rr; ++oz) {
      const int sz = zz + oz;
      if (sz < 0 || sz >= g.nz) continue;
      for (int oy = -Rr; oy <= Rr; ++oy) {
        const int sy = zy + oy;
        if (sy < 0 || sy >= g.ny) continue;
        for (int ox = -Rr; ox <= Rr; ++ox) {
          const int sx = zx + ox;
          if (sx < 0 || sx >= g.nx) continue;
          const uint32_t src = vidx(g, sx, sy, sz);
          int cx, cy, cz;
          float fx, fy, fz;
          cell_clamp(sx, -dt * bld(V0, src) * ih, g.nx, cx, fx);
          cell_clamp(sy, -dt * bld(V1, src) * ih, g.ny, cy, fy);
          cell_clamp(sz, -dt * bld(V2, src) * ih, g.nz, cz, fz);
          const int ex = zx - cx, ey = zy - cy, ez = zz - cz;
          if ((unsigned)ex > 1u || (unsigned)ey > 1u || (unsigned)ez > 1u) continue;
          const float w = (ex ? fx : 1.f - fx) * (ey ? fy : 1.f - fy) * (ez ? fz : 1.f - fz);
          s0 += w * bld(B0, src);
          s1 += w * bld(B1, src);
          s2 += w * bld(B2, src);
        }
      }
    }
    bst(O0, i, s0);
    bst(O1, i, s1);
    bst(O2, i, s2);
  }
}

// The splat of a step where k_splat_staged does not run or finds a larger reach, and the L v
// pass of the step before it (v_prev, on the first a.nvpart blocks): neither needs the other, and
// where the splat returns at once its launch costs nothing.  The general body needs a grid and
// an occupancy of its own: in one kernel with the staged one (its few blocks, 33 KB of LDS) energy
// and gradient at T = 10 and 1.5 voxels a step took 1196 us at 32^3, 2195 at 64^3 and 5184 at
// 128^3; 458, 782 and 4562 now.
__global__ __launch_bounds__(kBlock) void k_splat_Lv(GradArgs a, const float* v_prev) {
  const uint32_t nlv = v_prev ? (uint32_t)a.nvpart : 0u;
  if (blockIdx.x < nlv)
    Lv_body(a, v_prev, nlv);
  else
    splat_any(a, blockIdx.x - nlv, gridDim.x - nlv);
}

// ------------------------------------------------------------ launchers

void launch_ubar_init(const GradArgs& a, hipStream_t s) {
  if (a.nch == 2)
    hipLaunchKernelGGL(k_ubar_init<2>, dim3(grid_for(a.g.n)), dim3(kBlock), 0, s, a);
  else
    hipLaunchKernelGGL(k_ubar_init<1>, dim3(grid_for(a.g.n)), dim3(kBlock), 0, s, a);
}

static unsigned Lv_blocks(const Geom& g) {
  const unsigned gb = grid_for(g.n);
  return gb < kMaxParts ? gb : kMaxParts;
}

void launch_Lv(const GradArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_Lv, dim3(Lv_blocks(a.g)), dim3(kBlock), 0, s, a);
}

// Blocks of the general splat: every wavefront slot of the chip (1024: 1.4 times as long at 128^3);
// where they return at once, 0.9 us a step.
constexpr unsigned kSplatBlocks = 2048;

void launch_grad_step(const GradArgs& a0, const float* v_prev, hipStream_t s) {
  GradArgs a = a0;
  const unsigned gb = grid_for(a.g.n);
  a.nvpart = (int)Lv_blocks(a.g);
  a.staged = a.g.n >= kStagedVoxels && 3 * a.g.n < (1LL << 30);   // byte offsets of 3 n floats
  hipLaunchKernelGGL(k_coord_grad, dim3(gb), dim3(kBlock), 0, s, a);
  if (a.staged) {
    const SplatTiling t = splat_tiling(a.g);
    const int tiles = (t.ntx * t.nty * t.nrun + kXCD - 1) / kXCD * kXCD;
    hipLaunchKernelGGL(k_splat_staged, dim3(tiles), dim3(kBlock), 0, s, a);
  }
  const unsigned sb = gb < kSplatBlocks ? gb : kSplatBlocks;
  hipLaunchKernelGGL(k_splat_Lv, dim3((v_prev ? a.nvpart : 0) + sb), dim3(kBlock), 0, s, a, v_prev);
}

}  // namespace lddmm
