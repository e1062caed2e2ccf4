// Mask generation (Methods, Mask Generation) and the surface metrics of the
// evaluation (Methods, Evaluation), on bit-packed masks.
//
// Layout: a mask is packed 32 voxels per word along x, rows of W = ceil(nx/32)
// words, word (wx, y, z) at (z ny + y) W + wx, bit b = voxel x = 32 wx + b;
// bits past nx are always 0.
//
// Morphology with a ball: the ball of physical radius r is the union, over the
// (dy, dz) with dy^2 + dz^2 <= (r/h)^2, of x-runs of half-width w(dy, dz) =
// max{dx : dx^2 + dy^2 + dz^2 <= (r/h)^2}.  Dilation of a word ORs, over those
// (dy, dz), the row (y+dy, z+dz) dilated along x by w (shifts of the word and
// its two neighbours); erosion ANDs the x-eroded rows.  Outside the grid is
// background for both.  One thread per output word: 32 voxels per thread, and
// the per-word work is independent of how many voxels the ball holds.
//
// Surface distances: S = mask voxels with a face neighbour outside the mask.
// The squared distance (in voxels, exact integers) from every voxel to the
// nearest voxel of the other surface is the separable minimum
//   d2(x, y, z) = min_z' [ min_y' [ g1(x, y', z') + (y - y')^2 ] + (z - z')^2 ],
//   g1(x, y, z) = min over surface voxels x' of row (y, z) of (x - x')^2,
// computed as: for a column of 32 x (one word) in a plane, the nearest set bit of every
// row from bit scans of the packed words, and the min along y from them, in one pass
// through LDS; then the min along z only at the voxels of the first surface, searched
// outward from the voxel and stopped once the squared offset alone reaches the best
// value found (exact).  The Hausdorff distance takes the largest d2 (atomicMax); the median
// counts every d2 in a histogram over the integers 0 .. max possible (counts in
// LDS for small d2, which hold nearly all of them), and one block finds the
// middle rank(s).  Distances are h sqrt(d2) in FP64.  Both masks, and both directions,
// share every launch.
#include <cfloat>
#include <cmath>

#include "internal.h"
#include "lddmm.h"
#include "lddmm_masks.h"

namespace lddmm {
namespace {

constexpr int kWaves = kBlock / 64;
constexpr int kMaxM = LDDMM_MORPH_MAX_RADIUS_VOXELS + 1;
constexpr int kTable = (2 * kMaxM + 1) * (2 * kMaxM + 1);
constexpr uint32_t kInf = 0x3FFFFFFFu;
constexpr int kLdsBins = 4096;          // squared distances counted in LDS first

struct MGrid {
  int nx, ny, nz, W;                    // W: words per row
  long long nwords;                     // W ny nz
  long long n;                          // nx ny nz
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

MGrid make_mgrid(const lddmm_grid* g) {
  MGrid m;
  m.nx = g->nx;
  m.ny = g->ny;
  m.nz = g->nz;
  m.W = (g->nx + 31) / 32;
  m.nwords = (long long)m.W * g->ny * g->nz;
  m.n = (long long)g->nx * g->ny * g->nz;
  return m;
}

inline long long grid_voxels(const lddmm_grid* g) {
  if (!g || g->nx < 1 || g->ny < 1 || g->nz < 1 || g->nx > LDDMM_MAX_DIM ||
      g->ny > LDDMM_MAX_DIM || g->nz > LDDMM_MAX_DIM || !(g->spacing > 0.0) ||
      !std::isfinite(g->spacing))
    return -1;
  return (long long)g->nx * g->ny * g->nz;
}

inline unsigned blocks_for(long long n) {
  long long b = (n + kBlock - 1) / kBlock;
  if (b > 65535) b = 65535;
  return (unsigned)(b < 1 ? 1 : b);
}

// ------------------------------------------------------------- packing ----

enum : int { SRC_MASK = 0, SRC_THRESHOLD = 1 };

// One wavefront per row, four rows per block: lanes read 64 consecutive voxels, a ballot
// packs them; up to kPackSegs segments are in flight at once.  Bound by reading the source
// (4 B per voxel).  blockIdx.y: which of two sources.
constexpr int kPackSegs = 5;

template <int KIND>
__global__ __launch_bounds__(kBlock) void k_pack(MGrid g, const float* __restrict__ src0,
                                                 const float* __restrict__ src1, float tau,
                                                 uint32_t* __restrict__ out0,
                                                 uint32_t* __restrict__ out1) {
  const float* __restrict__ src = blockIdx.y ? src1 : src0;
  const float level = KIND == SRC_THRESHOLD ? tau : 0.f;
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * kWaves + (threadIdx.x >> 6);   // y + ny z
  if (row >= (long long)g.ny * g.nz) return;
  const long long base = row * g.nx;
  uint32_t* dst = (blockIdx.y ? out1 : out0) + row * g.W;
  for (int s0 = 0; 64 * s0 < g.nx; s0 += kPackSegs) {
    float v[kPackSegs];
#pragma unroll
    for (int s = 0; s < kPackSegs; ++s) {                 // no branch: all loads go out first
      const int x = 64 * (s0 + s) + lane;
      v[s] = src[base + (x < g.nx ? x : g.nx - 1)];
    }
#pragma unroll
    for (int s = 0; s < kPackSegs; ++s) {
      const unsigned long long bits = __ballot(64 * (s0 + s) + lane < g.nx && v[s] > level);
      const int w = 2 * (s0 + s) + (lane & 1);
      if (lane < 2 && w < g.W) dst[w] = (uint32_t)(bits >> (32 * (lane & 1)));
    }
  }
}

// One wavefront per row.
__global__ __launch_bounds__(kBlock) void k_unpack(MGrid g, const uint32_t* __restrict__ in,
                                                   float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const long long row = (long long)blockIdx.x * kWaves + (threadIdx.x >> 6);
  if (row >= (long long)g.ny * g.nz) return;
  for (int x = lane; x < g.nx; x += 64)
    out[row * g.nx + x] = (in[row * g.W + (x >> 5)] >> (x & 31)) & 1u ? 1.f : 0.f;
}

// ---------------------------------------------------------- morphology ----

__device__ __forceinline__ uint32_t word_at(const uint32_t* __restrict__ a, const MGrid& g, int wx,
                                            long long rowbase) {
  return (wx >= 0 && wx < g.W) ? a[rowbase + wx] : 0u;
}

__device__ __forceinline__ uint32_t dilate_x(uint32_t prev, uint32_t cur, uint32_t next, int w) {
  uint32_t acc = cur;
  for (int s = 1; s <= w; ++s)
    acc |= (cur << s) | (prev >> (32 - s)) | (cur >> s) | (next << (32 - s));
  return acc;
}

__device__ __forceinline__ uint32_t erode_x(uint32_t prev, uint32_t cur, uint32_t next, int w) {
  uint32_t acc = cur;
  for (int s = 1; s <= w; ++s)
    acc &= ((cur << s) | (prev >> (32 - s))) & ((cur >> s) | (next << (32 - s)));
  return acc;
}

__device__ __forceinline__ uint32_t valid_bits(const MGrid& g, int wx) {
  const int rem = g.nx - 32 * wx;
  return rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
}

// One thread per output word; erosion or dilation with the ball of radius rho voxels, m =
// floor(rho).  Each block makes its own table of the half-widths w(dy, dz) (-1: no voxel
// of the ball in that row) with the definition's FP64 decision dx^2 + dy^2 + dz^2 <= (r/h)^2:
// a launch that made it for all cost 4 us a pass.  Bound by the latency of the words' loads:
// kMorphAhead rows are loaded before the first is used, and a word that its own row already
// decides (empty for an erosion, full for a dilation) looks at no other.  One row at a
// time took 18 us a pass at 264 x 160 x 228, radii 1 and 2.5: 8.6 an erosion, 10.4 a
// dilation now.
constexpr int kMorphAhead = 5;

template <bool DILATE>
__global__ __launch_bounds__(kBlock) void k_morph(MGrid g, const uint32_t* __restrict__ in,
                                                  uint32_t* __restrict__ out, double rho, int m) {
  __shared__ int8_t tab[kTable];
  const int side = 2 * m + 1;
  const double rr = rho * rho;
  for (int k = threadIdx.x; k < side * side; k += kBlock) {
    const int dy = k % side - m, dz = k / side - m;
    int w = -1;
    for (int dx = 0; dx <= m; ++dx)
      if ((double)(dx * dx + dy * dy + dz * dz) <= rr) w = dx;
    tab[k] = (int8_t)w;
  }
  __syncthreads();
  const int my = min(m, g.ny - 1), mz = min(m, g.nz - 1);  // rows further off lie outside for all
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < g.nwords;
       i += (long long)gridDim.x * kBlock) {
    const uint32_t row = (uint32_t)i / (uint32_t)g.W;      // fewer than 2^25 words
    const int wx = (int)((uint32_t)i - row * g.W);
    const int z = (int)(row / (uint32_t)g.ny), y = (int)(row - (uint32_t)z * g.ny);
    const uint32_t valid = valid_bits(g, wx), decided = DILATE ? valid : 0u;
    uint32_t acc = in[i];
    // the ball's rows (0, +-m) and (+-m, 0) hold a voxel: an erosion leaves none where one of them
    // lies outside the grid
    if (!DILATE && (z < m || z + m >= g.nz || y < m || y + m >= g.ny)) acc = 0u;
    for (int dz = -mz; dz <= mz && acc != decided; ++dz) {
      const int zz = z + dz;
      const bool zok = zz >= 0 && zz < g.nz;
      for (int dy0 = -my; dy0 <= my; dy0 += kMorphAhead) {
        int w[kMorphAhead];
        uint32_t p[kMorphAhead], c[kMorphAhead], n[kMorphAhead];
#pragma unroll
        for (int u = 0; u < kMorphAhead; ++u) {
          const int dy = dy0 + u, yy = y + dy;
          w[u] = dy <= my ? __builtin_amdgcn_readfirstlane(tab[(dz + m) * side + dy + m]) : -1;
          // rows outside the grid are background; their loads go to the word's own row
          const bool ok = w[u] >= 0 && zok && yy >= 0 && yy < g.ny;
          const uint32_t* rb = in + (ok ? ((long long)zz * g.ny + yy) * g.W + wx : i);
          const uint32_t pv = rb[wx > 0 ? -1 : 0], cv = rb[0], nv = rb[wx + 1 < g.W ? 1 : 0];
          p[u] = ok && wx > 0 ? pv : 0u;
          c[u] = ok ? cv : 0u;
          n[u] = ok && wx + 1 < g.W ? nv : 0u;
        }
#pragma unroll
        for (int u = 0; u < kMorphAhead; ++u) {
          if (w[u] < 0) continue;
          if (DILATE)
            acc |= dilate_x(p[u], c[u], n[u], w[u]);
          else
            acc &= erode_x(p[u], c[u], n[u], w[u]);
        }
      }
      if (DILATE) acc &= valid;
    }
    out[i] = acc & valid;
  }
}

// --------------------------------------------------------------- surfaces ----

// Surfaces of both masks (blockIdx.y) and the number of their voxels in counts[0..1]: few blocks,
// so that the counts' address sees few atomics.
__global__ __launch_bounds__(kBlock) void k_surface(MGrid g, const uint32_t* __restrict__ a0,
                                                    const uint32_t* __restrict__ a1,
                                                    uint32_t* __restrict__ s0,
                                                    uint32_t* __restrict__ s1,
                                                    unsigned* __restrict__ counts) {
  const uint32_t* __restrict__ a = blockIdx.y ? a1 : a0;
  uint32_t* __restrict__ s = blockIdx.y ? s1 : s0;
  unsigned cnt = 0;
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < g.nwords;
       i += (long long)gridDim.x * kBlock) {
    const uint32_t row = (uint32_t)i / (uint32_t)g.W;      // fewer than 2^25 words
    const int wx = (int)((uint32_t)i - row * g.W);
    const int z = (int)(row / (uint32_t)g.ny), y = (int)(row - (uint32_t)z * g.ny);
    const uint32_t c = a[i];
    const uint32_t p = word_at(a, g, wx - 1, row * g.W), n = word_at(a, g, wx + 1, row * g.W);
    uint32_t inner = c & ((c << 1) | (p >> 31)) & ((c >> 1) | (n << 31));
    inner &= y > 0 ? a[i - g.W] : 0u;
    inner &= y + 1 < g.ny ? a[i + g.W] : 0u;
    inner &= z > 0 ? a[i - (long long)g.W * g.ny] : 0u;
    inner &= z + 1 < g.nz ? a[i + (long long)g.W * g.ny] : 0u;
    const uint32_t out = c & ~inner;
    s[i] = out;
    cnt += __popc(out);
  }
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  __shared__ unsigned sw[kWaves];
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned t = 0;
    for (int w = 0; w < kWaves; ++w) t += sw[w];
    if (t) atomicAdd(&counts[blockIdx.y], t);
  }
}

// x and y passes of one plane's column of 32 x (one word per row), all rows in LDS:
// g2(x, y, z) = min over y' of g1(x, y', z) + (y - y')^2, g1 the squared distance along
// row y' to its nearest surface voxel (bit scans of the row's words).  The min along y
// looks at blocks of 8 rows, nearest first: a block whose smallest g1 plus the squared
// distance to its nearest row is no better than the best found is skipped, and the
// search ends when that distance alone is.  A thread does 8 rows of results at once, so a
// value read from LDS serves all of them, (y - y')^2 by differences.  (A min over all rows of a column, with g1
// written and read back, took 203 + 66 us a direction at 264 x 160 x 228; both directions take 68 us now.)
// blockIdx.y: the direction, 0: distances to S_B, 1: to S_A.
constexpr int kRowBlock = 8;

constexpr uint32_t kNone = 0x7FFFu;     // "no surface voxel in this row"; kNone^2 + 1023^2 < 2^31

// Distances along x are below LDDMM_MAX_DIM, so 16 bits hold them (80 KB at 1024 rows).
inline size_t edt_lds(int ny) {
  const size_t nb = (ny + kRowBlock - 1) / kRowBlock;
  return sizeof(uint16_t) * 32 * (kRowBlock + 1) * nb + (sizeof(uint32_t) + 2 * sizeof(int16_t)) * ny;
}

__global__ __launch_bounds__(kBlock) void k_edt_xy(MGrid g, const uint32_t* __restrict__ sA,
                                                   const uint32_t* __restrict__ sB,
                                                   uint32_t* __restrict__ gB,
                                                   uint32_t* __restrict__ gA) {
  extern __shared__ uint32_t lds[];
  const uint32_t* __restrict__ s = blockIdx.y ? sA : sB;
  uint32_t* __restrict__ g2 = blockIdx.y ? gA : gB;
  const int ny = g.ny, nb = (ny + kRowBlock - 1) / kRowBlock;
  uint32_t* const cur = lds;                              // [ny] the row's word
  uint16_t* const col = reinterpret_cast<uint16_t*>(cur + ny);   // [nb * kRowBlock][32] distance along x
  uint16_t* const bmin = col + nb * kRowBlock * 32;       // [nb][32] smallest of a block of rows
  int16_t* const left = reinterpret_cast<int16_t*>(bmin + nb * 32);  // [ny] nearest x left of the word
  int16_t* const right = left + ny;                       // [ny] and right of it, or -1
  const int z = blockIdx.x / g.W, wx = blockIdx.x % g.W;
  for (int y = threadIdx.x; y < ny; y += kBlock) {
    const uint32_t* sr = s + ((long long)z * ny + y) * g.W;
    cur[y] = sr[wx];
    int l = -1, r = -1;
    for (int w = wx - 1; w >= 0; --w)
      if (const uint32_t m = sr[w]) {
        l = 32 * w + 31 - __clz(m);
        break;
      }
    for (int w = wx + 1; w < g.W; ++w)
      if (const uint32_t m = sr[w]) {
        r = 32 * w + __ffs(m) - 1;
        break;
      }
    left[y] = (int16_t)l;
    right[y] = (int16_t)r;
  }
  __syncthreads();
  const int b = threadIdx.x & 31, x = 32 * wx + b;
  for (int k = threadIdx.x >> 5; k < nb; k += kBlock / 32) {
    uint32_t m = kNone;
    for (int y = k * kRowBlock; y < (k + 1) * kRowBlock; ++y) {
      if (y >= ny) {
        col[y * 32 + b] = (uint16_t)kNone;
        continue;
      }
      const uint32_t c = cur[y], lo = c & (b == 31 ? 0xFFFFFFFFu : ((2u << b) - 1u)),
                     hi = c & ~((1u << b) - 1u);
      const int l = lo ? 32 * wx + 31 - __clz(lo) : left[y];
      const int r = hi ? 32 * wx + __ffs(hi) - 1 : right[y];
      uint32_t d = kNone;
      if (l >= 0) d = (uint32_t)(x - l);
      if (r >= 0 && (uint32_t)(r - x) < d) d = (uint32_t)(r - x);
      col[y * 32 + b] = (uint16_t)d;
      m = d < m ? d : m;
    }
    bmin[k * 32 + b] = (uint16_t)m;
  }
  __syncthreads();
  if (x >= g.nx) return;
  uint32_t any = kNone;
  for (int k = 0; k < nb; ++k) {
    const uint32_t m = bmin[k * 32 + b];
    any = m < any ? m : any;
  }
  uint32_t* out = g2 + (long long)z * ny * g.nx + x;
  for (int yk = threadIdx.x >> 5; yk < nb; yk += kBlock / 32) {
    uint32_t best[kRowBlock];
#pragma unroll
    for (int j = 0; j < kRowBlock; ++j) best[j] = kInf;
    if (any < kNone) {
      auto rows = [&](int k) {
        uint32_t worst = 0u;
#pragma unroll
        for (int i = 0; i < kRowBlock; ++i) {
          const uint32_t d = col[(k * kRowBlock + i) * 32 + b];
          const int dy = (yk - k) * kRowBlock - i;        // from row y' to the first of the results
          uint32_t e = d * d + (uint32_t)(dy * dy), step = (uint32_t)(2 * dy + 1);
#pragma unroll
          for (int j = 0; j < kRowBlock; ++j) {
            best[j] = e < best[j] ? e : best[j];
            e += step;
            step += 2u;
          }
        }
#pragma unroll
        for (int j = 0; j < kRowBlock; ++j) worst = best[j] > worst ? best[j] : worst;
        return worst;
      };
      uint32_t worst = rows(yk);
      for (int k = 1;; ++k) {
        const int klo = yk - k, khi = yk + k, gap = k * kRowBlock - (kRowBlock - 1);
        const uint32_t gap2 = (uint32_t)(gap * gap);
        if ((klo < 0 && khi >= nb) || gap2 >= worst) break;
        if (klo >= 0) {
          const uint32_t m = bmin[klo * 32 + b];
          if (m * m + gap2 < worst) worst = rows(klo);
        }
        if (khi < nb) {
          const uint32_t m = bmin[khi * 32 + b];
          if (m * m + gap2 < worst) worst = rows(khi);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kRowBlock; ++j)
      if (yk * kRowBlock + j < ny) out[(long long)(yk * kRowBlock + j) * g.nx] = best[j];
  }
}

// z pass at the voxels of one surface (its set bits only): d2 = min_z' g2(x, y, z') + (z -
// z')^2, searched outward from z until (z - z')^2 >= d2; then the Hausdorff maximum and
// the histogram of d2.  A wavefront spreads the set bits of up to 64 words over its lanes
// (a thread that walked its own word's bits one after the other left most lanes idle; a grid of few
// words gives each wavefront fewer, down to kZFewest: both masks noise on 300 x 2 x 300, all calls
// together, 76 us with 64 words each),
// and each lane looks kZAhead planes each way ahead, so the search is not one memory
// latency per plane.  Few large blocks: every block adds its counts to the same few
// bins.  blockIdx.y: the direction, as above.
constexpr int kZAhead = 4;
constexpr int kZBlock = 1024, kZWaves = kZBlock / 64, kZBlocks = 128, kZFewest = 8;

inline int z_words(long long nwords) {
  int n = 64;
  while (n > kZFewest && nwords < (long long)n * kZWaves * kZBlocks) n /= 2;
  return n;
}

__global__ __launch_bounds__(kZBlock) void k_edt_z_collect(MGrid g, const uint32_t* __restrict__ sA,
                                                          const uint32_t* __restrict__ sB,
                                                          const uint32_t* __restrict__ gB,
                                                          const uint32_t* __restrict__ gA,
                                                          uint32_t* __restrict__ hist,
                                                          uint32_t nbins, int nw,
                                                          unsigned* __restrict__ scal) {
  __shared__ uint32_t lh[kLdsBins];
  __shared__ unsigned lmax, lcnt;
  __shared__ uint32_t words[kZWaves][64];
  __shared__ unsigned ends[kZWaves][64];                   // set bits of the wavefront's words 0 .. k
  const uint32_t* __restrict__ sa = blockIdx.y ? sB : sA;
  const uint32_t* __restrict__ g2 = blockIdx.y ? gA : gB;
  for (int k = threadIdx.x; k < kLdsBins; k += kZBlock) lh[k] = 0u;
  if (threadIdx.x == 0) {
    lmax = 0u;
    lcnt = 0u;
  }
  __syncthreads();
  const long long plane = (long long)g.nx * g.ny;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  unsigned my_max = 0u, my_cnt = 0u;
  for (long long w0 = ((long long)blockIdx.x * kZWaves + wv) * nw; w0 < g.nwords;
       w0 += (long long)gridDim.x * kZWaves * nw) {
    const uint32_t mine = lane < nw && w0 + lane < g.nwords ? sa[w0 + lane] : 0u;
    unsigned end = __popc(mine);
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned up = __shfl_up(end, o);
      if (lane >= o) end += up;
    }
    const unsigned total = __shfl(end, 63);
    if (!total) continue;
    words[wv][lane] = mine;
    ends[wv][lane] = end;
    // the wavefront's own LDS: no other wave reads it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (unsigned k = lane; k < total; k += 64) {
      int lo = 0, hi = 63;                                // first word with ends > k
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ends[wv][mid] > k)
          hi = mid;
        else
          lo = mid + 1;
      }
      uint32_t bits = words[wv][lo];
      for (unsigned n = k - (ends[wv][lo] - __popc(bits)); n > 0; --n) bits &= bits - 1u;
      const long long i = w0 + lo;
      const uint32_t row = (uint32_t)i / (uint32_t)g.W;    // fewer than 2^25 words
      const int x = 32 * (int)((uint32_t)i - row * g.W) + __ffs(bits) - 1;
      const int z = (int)(row / (uint32_t)g.ny), y = (int)(row - (uint32_t)z * g.ny);
      const uint32_t* p = g2 + (long long)z * plane + (long long)y * g.nx + x;
      uint32_t best = *p;
      for (int d0 = 1; (uint32_t)(d0 * d0) < best; d0 += kZAhead) {
        if (z - d0 < 0 && z + d0 >= g.nz) break;
        uint32_t a[kZAhead], c[kZAhead];
#pragma unroll
        for (int u = 0; u < kZAhead; ++u) {
          const int d = d0 + u;
          a[u] = z - d >= 0 ? p[-(long long)d * plane] : kInf;
          c[u] = z + d < g.nz ? p[(long long)d * plane] : kInf;
        }
#pragma unroll
        for (int u = 0; u < kZAhead; ++u) {
          const uint32_t m = a[u] < c[u] ? a[u] : c[u];
          const uint32_t e = m + (uint32_t)((d0 + u) * (d0 + u));
          best = e < best ? e : best;
        }
      }
      // the other surface is non-empty whenever the result is used, so best < kInf
      my_max = best > my_max ? best : my_max;
      ++my_cnt;
      if (best < (uint32_t)kLdsBins)
        atomicAdd(&lh[best], 1u);
      else if (best < nbins)
        atomicAdd(&hist[best], 1u);
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (my_cnt) {
    atomicMax(&lmax, my_max);
    atomicAdd(&lcnt, my_cnt);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kLdsBins && k < (int)nbins; k += kZBlock)
    if (lh[k]) atomicAdd(&hist[k], lh[k]);
  if (threadIdx.x == 0 && lcnt) {
    atomicMax(&scal[0], lmax);
    atomicAdd(&scal[1], lcnt);
  }
}

// Zeros in p[0..n) and q[0..m), m <= kBlock.
__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t* __restrict__ p, long long n,
                                                     unsigned* __restrict__ q, int m) {
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (long long)gridDim.x * kBlock)
    p[i] = 0u;
  if (blockIdx.x == 0 && (int)threadIdx.x < m) q[threadIdx.x] = 0u;
}

// Sums of the histogram in tiles of kBlock bins, one block per tile.
__global__ __launch_bounds__(kBlock) void k_tile_sums(const uint32_t* __restrict__ hist,
                                                      uint32_t nbins, uint32_t* __restrict__ tsum) {
  const uint32_t k = blockIdx.x * kBlock + threadIdx.x;
  uint32_t c = k < nbins ? hist[k] : 0u;
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  __shared__ uint32_t wsum[kWaves];
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int w = 0; w < kWaves; ++w) t += wsum[w];
    tsum[blockIdx.x] = t;
  }
}

// One block: Hausdorff distance and the median of the histogram of d2 over both
// directions; out = {d_H, d_M, |S_A|, |S_B|}.  The tile sums (in LDS) locate the
// tiles of the middle rank(s), whose bins are then read into LDS and scanned.
constexpr int kMaxTiles = 12800;        // >= (3 * 1023^2 + 1) / kBlock

__global__ __launch_bounds__(kBlock) void k_surface_final(const uint32_t* __restrict__ hist,
                                                          uint32_t nbins,
                                                          const uint32_t* __restrict__ tsum_g,
                                                          const unsigned* __restrict__ scal,
                                                          double h, double* __restrict__ out) {
#pragma clang fp contract(off)          // h sqrt(d2) is rounded before two of them are averaged
  __shared__ uint32_t tsum[kMaxTiles];
  __shared__ uint32_t bins[2][kBlock];
  __shared__ uint32_t tile[2];
  __shared__ unsigned long long before_tile[2];
  const unsigned na = scal[2], nb = scal[3];
  const unsigned long long m = (unsigned long long)scal[1];   // distances counted, both ways
  const uint32_t ntiles = (nbins + kBlock - 1) / kBlock;
  for (uint32_t t = threadIdx.x; t < ntiles; t += kBlock) tsum[t] = tsum_g[t];
  __syncthreads();
  const bool empty = na == 0 || nb == 0 || m == 0;
  // 0-based ranks of the middle value(s) in increasing d2 order
  const unsigned long long ranks[2] = {empty ? 0 : (m - 1) / 2, empty ? 0 : m / 2};
  if (threadIdx.x < 2) {
    unsigned long long before = 0;
    uint32_t t = 0;
    if (!empty)
      while (before + tsum[t] <= ranks[threadIdx.x]) before += tsum[t++];
    tile[threadIdx.x] = t;
    before_tile[threadIdx.x] = before;
  }
  __syncthreads();
  for (int q = 0; q < 2; ++q) {
    const uint32_t k = tile[q] * kBlock + threadIdx.x;
    bins[q][threadIdx.x] = k < nbins ? hist[k] : 0u;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  out[2] = (double)na;
  out[3] = (double)nb;
  if (empty) {
    out[0] = NAN;
    out[1] = NAN;
    return;
  }
  out[0] = h * sqrt((double)scal[0]);
  double v[2];
  for (int q = 0; q < 2; ++q) {
    unsigned long long before = before_tile[q];
    int j = 0;
    for (;; ++j) {
      before += bins[q][j];
      if (before > ranks[q]) break;
    }
    v[q] = h * sqrt((double)(tile[q] * kBlock + j));
  }
  out[1] = (m & 1ull) ? v[0] : (v[0] + v[1]) / 2.0;
}

__global__ __launch_bounds__(kBlock) void k_label_mask(const int32_t* __restrict__ L, long long n,
                                                       float* __restrict__ m) {
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (long long)gridDim.x * kBlock)
    m[i] = L[i] != 0 ? 1.f : 0.f;
}

inline unsigned pack_blocks(const MGrid& g) {
  return (unsigned)(((long long)g.ny * g.nz + kWaves - 1) / kWaves);
}

// ------------------------------------------------------------- workspace ----

struct MaskLayout {
  size_t a, b, g1, g2, hist, tsum, scal, total;
};

MaskLayout mask_layout(const MGrid& g, uint32_t nbins) {
  MaskLayout L;
  size_t o = 0;
  const size_t wb = align256(sizeof(uint32_t) * (size_t)g.nwords);
  L.a = o; o += wb;
  L.b = o; o += wb;
  L.g1 = o; o += align256(sizeof(uint32_t) * (size_t)g.n);
  L.g2 = o; o += align256(sizeof(uint32_t) * (size_t)g.n);
  L.hist = o; o += align256(sizeof(uint32_t) * (size_t)nbins);
  L.tsum = o; o += align256(sizeof(uint32_t) * (size_t)((nbins + kBlock - 1) / kBlock));
  L.scal = o; o += align256(sizeof(unsigned) * 8);
  L.total = o;
  return L;
}

uint32_t dist_bins(const MGrid& g) {
  const long long dx = g.nx - 1, dy = g.ny - 1, dz = g.nz - 1;
  return (uint32_t)(dx * dx + dy * dy + dz * dz + 1);
}

int launch_status() {
  return hipGetLastError() == hipSuccess ? LDDMM_OK : LDDMM_EHIP;
}

// One erosion or dilation of `in` into `out` with the ball of radius rho voxels.
void morph_pass(const MGrid& g, const uint32_t* in, uint32_t* out, double rho, int dilate,
                hipStream_t s) {
  const int m = (int)floor(rho);       // no offset beyond it has a square up to rho^2
  hipLaunchKernelGGL(dilate ? k_morph<true> : k_morph<false>, dim3(blocks_for(g.nwords)),
                     dim3(kBlock), 0, s, g, in, out, rho, m);
}

bool radius_ok(double radius, double h) {
  return radius >= 0.0 && std::isfinite(radius) &&
         radius / h < (double)(LDDMM_MORPH_MAX_RADIUS_VOXELS + 1);
}

}  // namespace
}  // namespace lddmm

using namespace lddmm;

extern "C" {

size_t lddmm_masks_workspace_size(const lddmm_grid* grid) {
  if (grid_voxels(grid) < 0) return 0;
  const MGrid g = make_mgrid(grid);
  return mask_layout(g, dist_bins(g)).total;
}

int lddmm_label_mask(const lddmm_grid* grid, const int32_t* labels, float* mask, void* stream) {
  if (grid_voxels(grid) < 0 || !labels || !mask) return LDDMM_EINVAL;
  const MGrid g = make_mgrid(grid);
  (void)hipGetLastError();   // clear an earlier error: the status returned is these launches'
  hipLaunchKernelGGL(k_label_mask, dim3(blocks_for(g.n)), dim3(kBlock), 0, (hipStream_t)stream,
                     labels, g.n, mask);
  return launch_status();
}

int lddmm_morphology(const lddmm_grid* grid, const float* mask, int32_t op, double radius,
                     float* out, void* workspace, size_t workspace_bytes, void* stream) {
  if (grid_voxels(grid) < 0 || !mask || !out || !workspace) return LDDMM_EINVAL;
  if (op < LDDMM_MORPH_ERODE || op > LDDMM_MORPH_CLOSE) return LDDMM_EINVAL;
  if (!radius_ok(radius, grid->spacing)) return LDDMM_EINVAL;
  if (workspace_bytes < lddmm_masks_workspace_size(grid)) return LDDMM_EINVAL;
  const MGrid g = make_mgrid(grid);
  const MaskLayout L = mask_layout(g, dist_bins(g));
  char* ws = static_cast<char*>(workspace);
  uint32_t* a = reinterpret_cast<uint32_t*>(ws + L.a);
  uint32_t* b = reinterpret_cast<uint32_t*>(ws + L.b);
  const double rho = radius / grid->spacing;
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();   // clear an earlier error: the status returned is these launches'
  {
    hipLaunchKernelGGL(k_pack<SRC_MASK>, dim3(pack_blocks(g)), dim3(kBlock), 0, s, g, mask, nullptr,
                       0.f, a, nullptr);
    if (op == LDDMM_MORPH_ERODE || op == LDDMM_MORPH_DILATE) {
      morph_pass(g, a, b, rho, op == LDDMM_MORPH_DILATE, s);
      hipLaunchKernelGGL(k_unpack, dim3(pack_blocks(g)), dim3(kBlock), 0, s, g, b, out);
    } else {
      const int first_dilates = op == LDDMM_MORPH_CLOSE;
      morph_pass(g, a, b, rho, first_dilates, s);
      morph_pass(g, b, a, rho, !first_dilates, s);
      hipLaunchKernelGGL(k_unpack, dim3(pack_blocks(g)), dim3(kBlock), 0, s, g, a, out);
    }
  }
  return launch_status();
}

int lddmm_target_mask(const lddmm_grid* grid, const float* image, float tau, double open_radius,
                      double close_radius, float* mask, void* workspace, size_t workspace_bytes,
                      void* stream) {
  if (grid_voxels(grid) < 0 || !image || !mask || !workspace) return LDDMM_EINVAL;
  if (!radius_ok(open_radius, grid->spacing) || !radius_ok(close_radius, grid->spacing))
    return LDDMM_EINVAL;
  if (workspace_bytes < lddmm_masks_workspace_size(grid)) return LDDMM_EINVAL;
  const MGrid g = make_mgrid(grid);
  const MaskLayout L = mask_layout(g, dist_bins(g));
  char* ws = static_cast<char*>(workspace);
  uint32_t* a = reinterpret_cast<uint32_t*>(ws + L.a);
  uint32_t* b = reinterpret_cast<uint32_t*>(ws + L.b);
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();   // clear an earlier error: the status returned is these launches'
  {
    hipLaunchKernelGGL(k_pack<SRC_THRESHOLD>, dim3(pack_blocks(g)), dim3(kBlock), 0, s, g, image,
                       nullptr, tau, a, nullptr);
    const double ro = open_radius / grid->spacing, rc = close_radius / grid->spacing;
    morph_pass(g, a, b, ro, 0, s);        // opening: erode, then dilate
    morph_pass(g, b, a, ro, 1, s);
    morph_pass(g, a, b, rc, 1, s);        // closing: dilate, then erode
    morph_pass(g, b, a, rc, 0, s);
    hipLaunchKernelGGL(k_unpack, dim3(pack_blocks(g)), dim3(kBlock), 0, s, g, a, mask);
  }
  return launch_status();
}

int lddmm_surface_distance(const lddmm_grid* grid, const float* mask_a, const float* mask_b,
                           double* out, void* workspace, size_t workspace_bytes, void* stream) {
  if (grid_voxels(grid) < 0 || !mask_a || !mask_b || !out || !workspace) return LDDMM_EINVAL;
  if (workspace_bytes < lddmm_masks_workspace_size(grid)) return LDDMM_EINVAL;
  const MGrid g = make_mgrid(grid);
  const uint32_t nbins = dist_bins(g);
  const MaskLayout L = mask_layout(g, nbins);
  char* ws = static_cast<char*>(workspace);
  uint32_t* a = reinterpret_cast<uint32_t*>(ws + L.a);
  uint32_t* b = reinterpret_cast<uint32_t*>(ws + L.b);
  uint32_t* g1 = reinterpret_cast<uint32_t*>(ws + L.g1);
  uint32_t* g2 = reinterpret_cast<uint32_t*>(ws + L.g2);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* tsum = reinterpret_cast<uint32_t*>(ws + L.tsum);
  unsigned* scal = reinterpret_cast<unsigned*>(ws + L.scal);
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();   // clear an earlier error: the status returned is these launches'
  {
    // the histogram and, behind its tile sums, the counters
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(nbins)), dim3(kBlock), 0, s, hist,
                       (long long)nbins, scal, 8);
    hipLaunchKernelGGL(k_pack<SRC_MASK>, dim3(pack_blocks(g), 2), dim3(kBlock), 0, s, g, mask_a,
                       mask_b, 0.f, g1, g2);               // free until the distances
    hipLaunchKernelGGL(k_surface, dim3(std::min(blocks_for(g.nwords), 256u), 2), dim3(kBlock), 0, s,
                       g, g1, g2, a, b, scal + 2);         // S_A in a, S_B in b
    {
      ProfScope ps(LDDMM_PROF_OTHER, g.n, s);              // the dominant kernel
      hipLaunchKernelGGL(k_edt_xy, dim3((unsigned)(g.nz * g.W), 2), dim3(kBlock), edt_lds(g.ny), s,
                         g, a, b, g1, g2);
    }
    hipLaunchKernelGGL(k_edt_z_collect, dim3(kZBlocks, 2), dim3(kZBlock), 0, s, g, a, b, g1, g2, hist,
                       nbins, z_words(g.nwords), scal);
    hipLaunchKernelGGL(k_tile_sums, dim3((nbins + kBlock - 1) / kBlock), dim3(kBlock), 0, s, hist,
                       nbins, tsum);
    hipLaunchKernelGGL(k_surface_final, dim3(1), dim3(kBlock), 0, s, hist, nbins, tsum, scal,
                       grid->spacing, out);
  }
  return launch_status();
}

}  // extern "C"
