// Source-to-target (M2L) cell by cell: the alternative to the single padded grid that the paper
// weighs and sets aside (Sec. 2.5). It computes the same sums as the (8 N_g)^3 route: every
// target node receives G(target node - source node) times each effective mass of its 189
// interaction-zone cubes (Sec. 2.1, Eq. 1).
//
// Each source cube's gridlet, zero padded to C^3 with C = 2 N_g, is transformed once per solve.
// For a target and one of its sources at cube offset d = source - target (|d|_inf in 2..3), the
// C^3 cyclic array whose entry u holds g(h |d N_g - u_c|), where u_c = u for u < N_g and
// u - C otherwise, convolved cyclically with the padded source gives the potential at the
// target's N_g^3 nodes in the corner [0, N_g)^3: every node offset d N_g + (p - q) of the pair,
// |p - q| < N_g per axis, lands on a distinct entry, so nothing wraps. The transforms of these
// arrays (one per offset and level, divided by C^3) are constant tables. The sum over sources is
// taken in frequency space, then one pruned inverse transform per target keeps the corner.
//
// The paper's operation count charges one padded transform per (target, source) pair; here a
// source's transform is shared by every target that sees it (up to 27 parents' blocks), so what
// remains per pair is the pointwise product, C^2 (N_g + 1) complex multiply-adds.
//
// Stored order of a spectrum's modes: kz fastest, then kx, then ky (mode k = (ky HC + kx) C + kz), so
// that the transforms' z passes handle whole runs. FP32 rows are interleaved (re, im); FP64 rows
// hold two real parts, then their two imaginary parts (16 bytes each), as the FP64 product kernel
// loads them.
//
// Kernels:
//   k_cells_forward   several source gridlets (cells of levels >= 2 and virtual cubes) per
//                     workgroup: half spectrum [kz < C][ky < C][kx <= N_g] by separable direct
//                     sums, one line per thread.
//   k_cells_accum_f32, k_cells_accum_f64
//                     the products on the matrix cores: for one mode, the 8 children's sums over
//                     the 216 block slots are a matrix product, child x slot (Green values, the
//                     same for every parent of a level) times slot x parent (spectra). One launch
//                     for all levels.
//   k_cells_inverse   several targets per workgroup: pruned inverse (z, then y, then the Hermitian
//                     x sum), the N_g^3 corner written as the target's gridlet potentials. The
//                     inverse runs in double whatever the plan's precision (it is a small part of
//                     the work); in FP32 plans the result is stored as its mean (double) plus the
//                     zero-mean gridlet, so that the large common value of a target's potentials
//                     does not cost the precision of their differences.
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "fft.h"
#include "hpm_internal.h"

#include <algorithm>

namespace hpm {

// EXT = 1: extended target gridlets (N_g + 2 nodes per axis, Sec. 2.5). Target-minus-source
// node offsets then span 2 N_g + 1 values per axis, and C = 2 N_g + 2 keeps them apart.
template <int NG, int EXT>
struct CellShape {
  static constexpr int C = 2 * NG + 2 * EXT;
  static constexpr int HC = C / 2 + 1;
  static constexpr int K = C * C * HC;      // modes, [ky][kx][kz]
  static constexpr int KP = (K + 15) / 16 * 16;  // stored row: K modes, then zeros
  static constexpr int M = NG * NG * NG;    // source gridlet
  static constexpr int NL = NG + 2 * EXT;   // target gridlet nodes per axis
  static constexpr int ML = NL * NL * NL;
  static constexpr int OFFS = 343;          // d in [-3, 3]^3, index (dx+3) + 7 (dy+3) + 49 (dz+3)
};

// place of mode k, part c (0 real, 1 imaginary), in a stored row of reals
template <typename T>
__host__ __device__ constexpr int mode_pos(int k, int c) {
  return sizeof(T) == 4 ? 2 * k + c : (k / 2) * 4 + c * 2 + k % 2;
}

template <typename T>
struct CellArgs {
  int first_cell;    // id of the first cell of level 2: sources and targets are indexed from it
  int nsources;      // cells of levels >= 2, then the virtual cubes (row nsources of the
                     // source spectra is zero)
  int ntargets;
  int first_parent;  // first row of the block table (cells of level 1)
  const int* child8;
  const int* blocks;
  const T* gridlet;
  T* local;
  const T* gcell;    // [level - 2][343][2 KP]
  T* sspec;          // [source - first_cell][2 KP]
  T* tspec;          // [target - first_cell][2 KP]
  double* m2l_mean;  // [cells]: mean of each target's result, FP32 plans
};

constexpr int kCellThreads = 256;

// Gridlets per workgroup of the forward and inverse transforms: as many as keep one column
// (ky, kx) per thread, which is the widest pass of either (3 at N_g = 6: 252 of 256 threads).
template <int NG, int EXT>
constexpr int cells_per_group() {
  using S = CellShape<NG, EXT>;
  constexpr int t = kCellThreads / (S::C * S::HC);
  return t > 16 ? 16 : t;
}

// out_k = sum_j v[j] w^{jk}, w = exp(SIGN 2 pi i / C), for the C outputs k < K of one line, in order,
// handed to put(k, value). Compile-time twiddles: no output waits on a chain of table loads.
template <typename T, int NG, int C, int K, bool REAL_IN, typename F>
__device__ __forceinline__ void line_dft(const cplx<T> (&v)[NG], F&& put) {
  static_for<0, K>([&](auto kc) {
    constexpr int k = decltype(kc)::value;
    cplx<T> acc = {T(0), T(0)};
    static_for<0, NG>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr T wr = T(cis_cos(long(j) * k, C)), wi = T(-cis_sin(long(j) * k, C));
      if constexpr (REAL_IN) {
        acc.re += v[j].re * wr;
        acc.im += v[j].re * wi;
      } else {
        acc = cadd(acc, cmul(v[j], cplx<T>{wr, wi}));
      }
    });
    put(kc, acc);
  });
}

// The kernel writes KP complex values for the N_g^3 it reads, so its floor is the write (2^24
// clustered particles, N_g = 4, FP32: 7.6 GB in 1.62 ms, 1.90 ms with a wave per source). The z pass
// keeps its outputs in registers until the whole workgroup has read the y pass's, then assembles
// the stored rows in the same LDS and copies them out 16 bytes per lane in order: every line is
// written whole, by one instruction.
template <typename T, int NG, int EXT>
__global__ __launch_bounds__(kCellThreads) void k_cells_forward(CellArgs<T> a) {
  using S = CellShape<NG, EXT>;
  constexpr int C = S::C, HC = S::HC, K = S::K, KP = S::KP, M = S::M;
  constexpr int PER = cells_per_group<NG, EXT>();
  constexpr int N1 = PER * NG * NG * HC, N2 = PER * NG * C * HC;  // complex values of the passes
  constexpr size_t work_bytes = (N1 + N2) * sizeof(cplx<T>) + PER * M * sizeof(T);
  constexpr size_t row_bytes = size_t(PER) * 2 * KP * sizeof(T);
  static_assert(PER * C * HC <= kCellThreads, "one column per thread in the z pass");
  __shared__ __align__(16) char s_mem[work_bytes > row_bytes ? work_bytes : row_bytes];
  cplx<T>* s_a1 = reinterpret_cast<cplx<T>*>(s_mem);  // [source][z][y][kx]
  cplx<T>* s_a2 = s_a1 + N1;                          // [source][z][ky][kx]
  T* s_g = reinterpret_cast<T*>(s_a2 + N2);
  T* s_row = reinterpret_cast<T*>(s_mem);             // [source][2 KP], after the z pass
  const int tid = threadIdx.x;
  const int src0 = blockIdx.x * PER;
  // sources of this workgroup: src0 .. src0 + cnt - 1; row nsources is the zero row that empty
  // block slots read
  const int cnt = min(PER, a.nsources - src0);
  if (src0 + PER > a.nsources) {
    T* zero = a.sspec + size_t(a.nsources) * 2 * KP;
    for (int e = tid; e < 2 * KP; e += kCellThreads) zero[e] = T(0);
  }
  if (cnt <= 0) return;
  const T* g = a.gridlet + size_t(a.first_cell + src0) * M;
  for (int e = tid; e < cnt * M; e += kCellThreads) s_g[e] = g[e];
  __syncthreads();
  // x: one real row (source, z, y) per thread, its half spectrum kx <= C/2
  for (int r = tid; r < cnt * NG * NG; r += kCellThreads) {
    cplx<T> v[NG];
#pragma unroll
    for (int x = 0; x < NG; ++x) v[x] = {s_g[r * NG + x], T(0)};
    line_dft<T, NG, C, HC, true>(v, [&](auto kc, cplx<T> o) { s_a1[r * HC + decltype(kc)::value] = o; });
  }
  __syncthreads();
  // y: one column (source, z, kx) per thread, all C values of ky
  for (int q = tid; q < cnt * NG * HC; q += kCellThreads) {
    const int z = q / HC, kx = q % HC;  // z: (source, z)
    cplx<T> v[NG];
#pragma unroll
    for (int y = 0; y < NG; ++y) v[y] = s_a1[(z * NG + y) * HC + kx];
    line_dft<T, NG, C, C, false>(
        v, [&](auto kc, cplx<T> o) { s_a2[(z * C + decltype(kc)::value) * HC + kx] = o; });
  }
  __syncthreads();
  // z: one column (source, ky, kx) per thread, all C values of kz
  const bool live = tid < cnt * C * HC;
  const int sl = tid / (C * HC), col = tid % (C * HC);
  cplx<T> out[C];
  if (live) {
    cplx<T> v[NG];
#pragma unroll
    for (int z = 0; z < NG; ++z) v[z] = s_a2[(sl * NG + z) * C * HC + col];
    line_dft<T, NG, C, C, false>(v, [&](auto kc, cplx<T> o) { out[decltype(kc)::value] = o; });
  }
  __syncthreads();  // the y pass's values are consumed
  if (live) {
    T* row = s_row + sl * 2 * KP;
#pragma unroll
    for (int kz = 0; kz < C; ++kz) {
      row[mode_pos<T>(col * C + kz, 0)] = out[kz].re;
      row[mode_pos<T>(col * C + kz, 1)] = out[kz].im;
    }
  }
  if constexpr (KP > K) {
    for (int e = tid; e < cnt * (KP - K); e += kCellThreads) {
      T* row = s_row + (e / (KP - K)) * 2 * KP;
      row[mode_pos<T>(K + e % (KP - K), 0)] = T(0);
      row[mode_pos<T>(K + e % (KP - K), 1)] = T(0);
    }
  }
  __syncthreads();
  constexpr int PIECES = 2 * KP * int(sizeof(T)) / 16;  // 16-byte pieces of a row
  const float4* from = reinterpret_cast<const float4*>(s_row);
  float4* to = reinterpret_cast<float4*>(a.sspec + size_t(src0) * 2 * KP);
  for (int e = tid; e < cnt * PIECES; e += kCellThreads) to[e] = from[e];
}

// ---------------------------------------------------------------------------------------------
// Products on the matrix cores. For one mode, child c's sum over the block slots s of its parent is
// T_c = sum_s G(d(c, s)) S_s (complex; G = 0 for the near offsets and d = slot - 2 - child per
// axis, so the Green values depend on (c, s) alone and serve every parent of the level). 189 of the
// 216 slots carry work, so 88% of the matrix work is wanted.
//
// A workgroup takes a tile of split parents of one level and a chunk of modes (32 in FP32, 8 in FP64),
// whose Green values it keeps in LDS (88 or 44 KB). Workgroups are persistent; work
// items are (chunk, tile) with the tiles of all levels fastest, one contiguous range of items per
// XCD, taken by its workgroups in turn: those in flight share a chunk and neighbouring parents,
// whose source rows overlap in the XCD's L2.
// ---------------------------------------------------------------------------------------------
// threads of a workgroup and its parents, 8 per wave (FINE: 4 per pair of waves, see the FP32 kernel);
// resident workgroups per CU (two waves per SIMD)
template <typename T, bool CENTRAL>
constexpr int kAccumThreads = sizeof(T) == 4 && !CENTRAL ? 512 : 256;
template <typename T, bool CENTRAL, bool FINE = false>
constexpr int kTileParents = kAccumThreads<T, CENTRAL> / (FINE ? 32 : 8);
template <typename T, bool CENTRAL>
constexpr int kAccumPerCU = 512 / kAccumThreads<T, CENTRAL>;
template <typename T>
constexpr int kChunkModes = sizeof(T) == 4 ? 32 : 8;

// FP32: up to this many items, half the CUs, the fine split is the faster one (evaluations of uniform
// and Plummer sets of 500 to 240,000 particles, us): 8 parents, N_g = 4, 84 -> 63 (one thread per
// (parent, mode) on the vector ALU: 63); 72 parents, 126 -> 81 (107); 32 parents in 128 items, N_g = 6,
// 193 -> 174; 584 in 100, 155 -> 143. Above it loses more often than it gains: 4680 in 148, 223 -> 234;
// 929 in 180, 255 -> 264; 1880 in 1024, 738 -> 880.
constexpr int kFineItems = 128;

struct TileTable {
  int ntiles;                       // tiles of all parent levels
  int first[kMaxLevelsHost + 1];    // first tile of parent level l (ntiles past the last)
  int pbeg[kMaxLevelsHost + 1];     // first list entry of parent level l
};

// The work items of this workgroup: it = begin; it < end; it += step. A few items per workgroup are
// taken in order, so that a chunk's Green values are staged once for consecutive tiles; many are
// taken in turn by the XCD's workgroups.
struct Items {
  int begin, end, step;
  __device__ __forceinline__ explicit Items(int total) {
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3, per = gridDim.x >> 3;
    const int first = int((int64_t(total) * xcd) / 8), last = int((int64_t(total) * (xcd + 1)) / 8);
    if (last - first <= 8 * per) {
      begin = first + int((int64_t(last - first) * j) / per);
      end = first + int((int64_t(last - first) * (j + 1)) / per);
      step = 1;
    } else {
      begin = first + j;
      end = last;
      step = per;
    }
  }
};

// of an item its chunk, its parents' level lp, its first list entry p0 and its number of parents pn
template <int TILE>
__device__ __forceinline__ void item_of(const TileTable& tt, int it, int& chunk, int& lp, int& p0,
                                        int& pn) {
  chunk = it / tt.ntiles;
  const int tile = it % tt.ntiles;
  lp = 1;
  while (lp + 1 < kMaxLevelsHost && tile >= tt.first[lp + 1]) ++lp;
  p0 = tt.pbeg[lp] + (tile - tt.first[lp]) * TILE;
  pn = min(TILE, tt.pbeg[lp + 1] - p0);
}

// staged offsets: all 7^3 (|d| <= 3), or for the central cubes the 5^3 with |d| <= 2
template <bool CENTRAL>
struct AccumShape {
  static constexpr int OW = CENTRAL ? 5 : 7, OR = OW / 2, NOFF = OW * OW * OW;
  static constexpr int B0 = CENTRAL ? 1 : 0, NB = CENTRAL ? 4 : 6;  // first block coordinate, count
};

// Each wave takes 8 of the tile's parents and all modes of the chunk, and steps through the slots. The
// spectra go from memory to the wave's own LDS rows in whole lines (consecutive lanes per line: a
// lane per parent and mode, the operand layout, costs the vector cache one access per lane, which
// bounded a version without the LDS rows at 40% matrix utilization). The steps are pipelined: while
// one's products run, later ones' loads are in flight, and in FP32 the next one's operands are read
// from LDS and the rows of the one after it written there (two buffers). No barrier in the loop, since a
// wave's LDS operations execute in order. LDS serves 16 lanes x 16 bytes per cycle from 64 banks;
// both operands' rows are swizzled in 16-byte pieces so that the 16 lanes of a pass read all banks
// once.
//
// Measured per evaluation, near zone in line, against one thread per (parent, mode) on the vector
// ALU, one launch per level: 2^24 clustered particles (N_g = 4, FP32) 21.1 -> 14.2 ms (68 TFLOP/s of
// matrix work; the matrix cores busy 43% of the time at 2.4 GHz, 58% of the cycles at the clock the chip
// then runs); 10^6 clustered, extended N_g = 6, FP32 3.73 -> 2.27 ms; 150,001
// Plummer, N_g = 6, FP64 0.96 -> 0.52 ms; the central cubes of 2^18 Plummer, N_g = 6, FP32
// 0.31 -> 0.20 ms. With every source row in L2 the 2^24 case takes 13.2 ms (measured on the version
// before the operand pipeline): what bounds it is issue beside the matrix instructions, two waves
// per SIMD, not memory.

// this wave's LDS writes before, its reads after (and the reverse), in program order
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The matrix instructions multiply every slot, the near ones by zero Green values, and zero times an
// infinite or NaN spectrum (an infinite mass, or one that overflows) is NaN. A child whose result is
// not finite is therefore summed again over its own zone alone, slot by slot in the same order, so
// that a source has no part in the far field of the targets near it, as on the padded grid. Only
// such results come here, behind a test of the finished sums.
template <typename T, int NG, int EXT, bool CENTRAL>
__device__ __forceinline__ cplx<T> zone_sum(const CellArgs<T>& a, int lp, int parent, int child, int mode) {
  using S = CellShape<NG, EXT>;
  constexpr int B0 = AccumShape<CENTRAL>::B0, NB = AccumShape<CENTRAL>::NB;
  const int cx = child & 1, cy = (child >> 1) & 1, cz = child >> 2;
  const int re = mode_pos<T>(mode, 0), im = mode_pos<T>(mode, 1);
  const T* G = a.gcell + size_t(lp - 1) * S::OFFS * 2 * S::KP;
  const int* ids = a.blocks + size_t(parent - a.first_parent) * 216;
  cplx<T> o = {T(0), T(0)};
#pragma unroll 1
  for (int s = 0; s < NB * NB * NB; ++s) {
    const int bx = B0 + s % NB, by = B0 + (s / NB) % NB, bz = B0 + s / (NB * NB);
    const int dx = bx - 2 - cx, dy = by - 2 - cy, dz = bz - 2 - cz;
    if (abs(dx) <= 1 && abs(dy) <= 1 && abs(dz) <= 1) continue;
    const int id = ids[bx + 6 * by + 36 * bz];
    const T* sv = a.sspec + size_t(id >= 0 ? id - a.first_cell : a.nsources) * 2 * S::KP;
    const T* gv = G + size_t((dx + 3) + 7 * (dy + 3) + 49 * (dz + 3)) * 2 * S::KP;
    const T gr = gv[re], gi = gv[im], sr = sv[re], si = sv[im];
    o.re = fma(gr, sr, o.re);
    o.re = fma(-gi, si, o.re);
    o.im = fma(gr, si, o.im);
    o.im = fma(gi, sr, o.im);
  }
  return o;
}

template <typename T>
__device__ __forceinline__ bool finite(T x) {
  return fabs(x) <= (sizeof(T) == 4 ? T(3.402823466e+38) : T(1.7976931348623157e308));
}

// FP32. v_mfma_f32_4x4x1: 16 blocks (modes) of 4 children times 4 parents, one slot per
// instruction. Each instruction is one fused multiply-add per result, so a result's terms are added
// in slot order, real products before cross terms: the FP32 rounding of the sums (which the
// interpolation amplifies at N_g = 6) is that of a plain loop over the slots.
//
// Lane l holds modes 2 (l / 4) and 2 (l / 4) + 1 of the chunk's 32 and, as an operand, child or parent
// l % 4 of a quad; 2 x 2 quads of (children, parents) with real and imaginary parts of two modes are
// 16 accumulators. A step is one slot; loads run one row of slots (fixed by, bz) ahead.
//
// FINE: a wave takes one quad of parents and one of children, a quarter of the products per slot, so
// that a tree with fewer tiles than CUs has a chain of 216 short steps instead of 216 long ones.
template <int NG, int EXT, bool CENTRAL = false, bool FINE = false>
__global__ __launch_bounds__((kAccumThreads<float, CENTRAL>), (kAccumPerCU<float, CENTRAL>)) void k_cells_accum_f32(CellArgs<float> a,
                                                                             TileTable tt,
                                                                             const int* plist) {
  using S = CellShape<NG, EXT>;
  using A = AccumShape<CENTRAL>;
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int KP = S::KP, KC = kChunkModes<float>, NCH = (KP + KC - 1) / KC;
  constexpr int OW = A::OW, OR = A::OR, NOFF = A::NOFF, B0 = A::B0, NB = A::NB;
  constexpr int NQ = FINE ? 1 : 2;                            // quads of a wave's parents, and of its children
  constexpr int TILE = kTileParents<float, CENTRAL, FINE>, WP = 4 * NQ;  // parents of a tile, of a wave
  constexpr int PC = KC / 2;                         // 16-byte pieces (mode pairs) of a row
  constexpr int NR = NB * NB;                        // rows of slots
  __shared__ f4 s_g[NOFF * PC];                      // [offset][pieces, swizzled]
  constexpr int NW = kAccumThreads<float, CENTRAL> / 64;
  __shared__ f4 s_b[NW][2 * WP * PC];                // per wave: [buffer][parent][pieces, swizzled]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mp = lane >> 2, i = lane & 3;            // mode pair, child or parent of a quad
  const int cx = i & 1, cy = i >> 1;
  // first child half of the wave, place of its parents in the tile
  const int cz0 = FINE ? wave & 1 : 0, wp0 = (FINE ? wave >> 1 : wave) * WP;
  // byte offsets into s_g of (child i of cz = cz0 + 1, this mode pair) at slot (0, 0, 0), for slots whose
  // bx and by have parities px and py
  int ga[2][2];
#pragma unroll
  for (int py = 0; py < 2; ++py)
#pragma unroll
    for (int px = 0; px < 2; ++px) {
      const int swz = ((1 - cx + px) & 1) | (((1 - cy + py) & 1) << 1);
      ga[py][px] = (((1 - cx) + OW * (1 - cy) - OW * OW * cz0) * PC + (mp ^ (swz << 2))) * 16;
    }
  const char* sg = reinterpret_cast<const char*>(s_g);
  const f4* sb = s_b[wave] + i * PC + (mp ^ (i << 2));  // parent i of either quad, this mode pair
  // as a loader: piece lane % 16 of the parents lane / 16 and 4 + lane / 16
  const int lpar = lane >> 4, lpiece = lane & 15;
  f4* sw = s_b[wave] + lpar * PC + (lpiece ^ (lpar << 2));

  const Items items(NCH * tt.ntiles);
  int staged = -1;
  for (int it = items.begin; it < items.end; it += items.step) {
    int chunk, lp, p0, pn;
    item_of<TILE>(tt, it, chunk, lp, p0, pn);
    // the last chunk may be half full: its absent pieces are read as the first one and not written
    const int pieces = min(PC, (KP - chunk * KC) / 2);
    if (staged != chunk * kMaxLevelsHost + lp) {  // workgroup-uniform
      staged = chunk * kMaxLevelsHost + lp;
      __syncthreads();  // the previous item's Green values are consumed
      // the children's level is lp + 1
      const float* G = a.gcell + size_t(lp - 1) * S::OFFS * 2 * KP + chunk * 2 * KC;
      for (int e = tid; e < NOFF * PC; e += kAccumThreads<float, CENTRAL>) {
        const int o = e / PC, j = e % PC;
        const int x = o % OW, y = (o / OW) % OW, z = o / (OW * OW);
        const int o343 = (x + 3 - OR) + 7 * (y + 3 - OR) + 49 * (z + 3 - OR);
        const int swz = (x & 1) | ((y & 1) << 1);
        s_g[o * PC + (j ^ (swz << 2))] =
            reinterpret_cast<const f4*>(G + size_t(o343) * 2 * KP)[j < pieces ? j : 0];
      }
      __syncthreads();
    }
    if (wp0 >= pn) continue;  // wave-uniform; the barriers above are workgroup-uniform
    // row ids: lane (parent lane / 8, bx lane % 8) holds one row of slots of its parent (the zero row
    // for an empty slot; any valid table row for an absent parent, whose ids are not used)
    const int ipar = wp0 + (lane >> 3);
    const bool have = ipar < pn && (lane >> 3) < WP;
    const int* ids = a.blocks + size_t(plist[p0 + min(ipar, pn - 1)] - a.first_parent) * 216 + B0 * 43 +
                     min(lane & 7, NB - 1);
    auto load_ids = [&](int row) {
      const int v = ids[6 * (row % NB) + 36 * (row / NB)];
      return have && v >= 0 ? v - a.first_cell : a.nsources;
    };
    const float* spec = a.sspec + chunk * 2 * KC + (lpiece < pieces ? lpiece : 0) * 4;
    f4 rows[NB][NQ];
    // spectrum rows of slot bx, both of the loader's parents, from a row of ids
    auto row_of = [&](int idv, int bx, int (&r)[NQ]) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) r[j] = __shfl(idv, (lpar + 4 * j) * 8 + bx, 64);
    };
    auto load_rows = [&](const int (&r)[NQ], f4 (&to)[NQ]) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) to[j] = *reinterpret_cast<const f4*>(spec + size_t(r[j]) * 2 * KP);
    };
    auto put_rows = [&](int buf, const f4 (&from)[NQ]) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) sw[(buf * WP + 4 * j) * PC] = from[j];
    };
    // Green values of slot bx of the row at gr (by of parity py), and this lane's two parents' spectra
    auto load_slot = [&](const char* gr, int py, int bx, f4 (&g)[NQ], f4 (&v)[NQ]) {
#pragma unroll
      for (int c = 0; c < NQ; ++c)
        g[c] = *reinterpret_cast<const f4*>(gr + ga[py][bx & 1] + (bx + OW * OW * (1 - c)) * (PC * 16));
#pragma unroll
      for (int p = 0; p < NQ; ++p) v[p] = sb[((bx & 1) * WP + 4 * p) * PC];
    };
    auto mac = [](float x, float y, f4 c) { return __builtin_amdgcn_mfma_f32_4x4x1f32(x, y, c, 0, 0, 0); };
    f4 re[2][NQ][NQ], im[2][NQ][NQ];  // [mode][cz - cz0][parent quad]
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int c = 0; c < NQ; ++c)
#pragma unroll
        for (int p = 0; p < NQ; ++p) re[m][c][p] = im[m][c][p] = f4{0.f, 0.f, 0.f, 0.f};
    // ids of the rows of slots after the current one (past the last: the last one's again)
    int id1 = load_ids(min(1, NR - 1)), id2 = load_ids(min(2, NR - 1));
    int r[NQ];
    {
      const int id0 = load_ids(0);
#pragma unroll
      for (int bx = 0; bx < NB; ++bx) {
        row_of(id0, bx, r);
        load_rows(r, rows[bx]);
      }
    }
    wave_lds_fence();
    put_rows(0, rows[0]);
    put_rows(1, rows[1]);
    wave_lds_fence();
    row_of(id1, 0, r);
    load_rows(r, rows[0]);
    row_of(id1, 1, r);
    load_rows(r, rows[1]);
    row_of(id1, 2, r);  // the next load's rows, ready before they are wanted
    f4 g[NQ], v[NQ], gn[NQ], vn[NQ];
    load_slot(sg, 0, 0, g, v);
    // rows of slots in pairs, by even and odd (NB is even)
    auto green_row = [&](int row) { return sg + (OW * (row % NB) + OW * OW * (row / NB)) * (PC * 16); };
#pragma unroll 1
    for (int row0 = 0; row0 < NR; row0 += 2) {
#pragma unroll
      for (int py = 0; py < 2; ++py) {
        const int row = row0 + py;
        const char* gr = green_row(row);
        const char* gr1 = green_row(min(row + 1, NR - 1));
        const int id3 = load_ids(min(row + 3, NR - 1));
#pragma unroll
        for (int bx = 0; bx < NB; ++bx) {
          // operands of the next slot (past the last one: of some slot, not used)
          if (bx + 1 < NB) load_slot(gr, py, bx + 1, gn, vn);
          else load_slot(gr1, py ^ 1, 0, gn, vn);
          wave_lds_fence();
          // rows of the slot after it, in the buffer whose operands are in registers; their
          // registers then take the rows one row of slots later
          constexpr int N = NB;
          const int k = (bx + 2) % N;
          put_rows(bx & 1, rows[k]);
          load_rows(r, rows[k]);
          wave_lds_fence();
          row_of(bx + 3 < N ? id1 : id2, (bx + 3) % N, r);
          __builtin_amdgcn_sched_barrier(0);
          // two rounds of 16 (FINE: 4) independent products
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int c = 0; c < NQ; ++c)
#pragma unroll
              for (int p = 0; p < NQ; ++p) {
                re[m][c][p] = mac(g[c][2 * m], v[p][2 * m], re[m][c][p]);
                im[m][c][p] = mac(g[c][2 * m], v[p][2 * m + 1], im[m][c][p]);
              }
          float ng[NQ][2];
#pragma unroll
          for (int c = 0; c < NQ; ++c) {
            ng[c][0] = -g[c][1];
            ng[c][1] = -g[c][3];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int c = 0; c < NQ; ++c)
#pragma unroll
              for (int p = 0; p < NQ; ++p) {
                re[m][c][p] = mac(ng[c][m], v[p][2 * m + 1], re[m][c][p]);
                im[m][c][p] = mac(g[c][2 * m + 1], v[p][2 * m], im[m][c][p]);
              }
#pragma unroll
          for (int c = 0; c < NQ; ++c) {
            g[c] = gn[c];
            v[c] = vn[c];
          }
        }
        id1 = id2;
        id2 = id3;
      }
    }
    // register r of lane l: child r of the quad, parent l % 4
    if (mp < pieces) {
      float* out = a.tspec + chunk * 2 * KC + mp * 4;
#pragma unroll
      for (int p = 0; p < NQ; ++p) {
        const int k = wp0 + p * 4 + i;
        const int* kids = a.child8 + size_t(plist[p0 + min(k, pn - 1)]) * 8;
#pragma unroll
        for (int c = 0; c < NQ; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int t = k < pn ? kids[4 * (cz0 + c) + r] : -1;
            if (t >= 0)
              *reinterpret_cast<f4*>(out + size_t(t - a.first_cell) * 2 * KP) =
                  f4{re[0][c][p][r], im[0][c][p][r], re[1][c][p][r], im[1][c][p][r]};
          }
      }
      // a source that is not finite shows in either part of every child, near or far: one part of
      // one child tells (a sum that overflows by itself is what it would be slot by slot)
      bool odd = false;
#pragma unroll
      for (int p = 0; p < NQ; ++p) odd = odd || !finite(re[0][0][p][0]) || !finite(re[1][0][p][0]);
      if (odd) {
#pragma unroll 1
        for (int e = 0; e < 4 * NQ * NQ; ++e) {
          const int k = wp0 + e / (4 * NQ) * 4 + i, child = 4 * cz0 + e % (4 * NQ);
          if (k >= pn) break;
          const int par = plist[p0 + k], t = a.child8[size_t(par) * 8 + child];
          if (t < 0) continue;
          f4* at = reinterpret_cast<f4*>(out + size_t(t - a.first_cell) * 2 * KP);
          const f4 v = *at;
          if (finite(v[0]) && finite(v[1]) && finite(v[2]) && finite(v[3])) continue;
          const cplx<float> lo = zone_sum<float, NG, EXT, CENTRAL>(a, lp, par, child, chunk * KC + 2 * mp);
          const cplx<float> hi = zone_sum<float, NG, EXT, CENTRAL>(a, lp, par, child, chunk * KC + 2 * mp + 1);
          *at = f4{lo.re, lo.im, hi.re, hi.im};
        }
      }
    }
  }
}

// FP64. v_mfma_f64_16x16x4: rows (child, part of G), columns (parent, part of S), 4 slots per
// instruction; the four real products Gr Sr, Gr Si, Gi Sr, Gi Si of 8 children and 8 parents, whose
// parts are combined once at the end. As operands, lane l is column (or row) l % 16 and slot l / 16 of
// a step of 2 x 2 slots (2u .. 2u + 1, 2v .. 2v + 1, bz), so every LDS address is a lane constant plus
// an immediate, and the swizzle of the Green values, by the parities of dx and dy, is a lane constant
// too. One LDS buffer per wave (a second one was no faster alone, 0.53 against 0.52 ms on 150,001
// Plummer particles, and left no room for the near-zone workgroups that run beside it).
template <int NG, int EXT, bool CENTRAL = false>
__global__ __launch_bounds__((kAccumThreads<double, CENTRAL>), (kAccumPerCU<double, CENTRAL>)) void k_cells_accum_f64(CellArgs<double> a,
                                                                              TileTable tt,
                                                                              const int* plist) {
  using S = CellShape<NG, EXT>;
  using A = AccumShape<CENTRAL>;
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef double d4 __attribute__((ext_vector_type(4)));
  constexpr int KP = S::KP, KC = kChunkModes<double>, NCH = KP / KC;  // KP is a multiple of 16
  constexpr int OW = A::OW, OR = A::OR, NOFF = A::NOFF, B0 = A::B0, NB = A::NB, NU = NB / 2;
  constexpr int TILE = kTileParents<double, CENTRAL>, WP = 8;  // parents of a tile, of a wave
  constexpr int PC = 8;                               // 16-byte pieces: 4 mode pairs x 2 parts
  __shared__ d2 s_g[NOFF * PC];                       // [offset][pieces, swizzled]
  __shared__ d2 s_b[TILE / WP][4 * WP * PC];          // per wave: [slot][parent][pieces, swizzled]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = lane & 15, q = lane >> 4;
  // as operand A: row n = (child, part of G). Register r of the accumulator holds row 4 r + q: with
  // the part in bit 2 of the row a lane gets both parts of children q and q + 4.
  const int achild = (n & 3) | ((n >> 3) << 2), apart = (n >> 2) & 1;
  const int cx = achild & 1, cy = (achild >> 1) & 1, cz = achild >> 2;
  const int ox = (q & 1) + 1 - cx, oy = (q >> 1) + 1 - cy, oz = 1 - cz;  // offset of slot (0, 0, 0)
  const int aswz = (ox & 1) * 2 + (oy & 1) * 4;
  const d2* ga = s_g + (ox + OW * oy + OW * OW * oz) * PC;
  // as operand B: column n = (parent, part of S)
  const int bpar = n >> 1, bpart = n & 1;
  const d2* sb = s_b[wave] + (q * WP + bpar) * PC;
  const int bswz = (bpar >> 1) << 1;
  // as a loader: piece lane % 8 of parent lane / 8, the 4 slots of the step in turn
  const int lpar = lane >> 3, lpiece = lane & 7;
  d2* sw = s_b[wave] + lpar * PC + (lpiece ^ ((lpar >> 1) << 1));

  const Items items(NCH * tt.ntiles);
  int staged = -1;
  for (int it = items.begin; it < items.end; it += items.step) {
    int chunk, lp, p0, pn;
    item_of<TILE>(tt, it, chunk, lp, p0, pn);
    if (staged != chunk * kMaxLevelsHost + lp) {  // workgroup-uniform
      staged = chunk * kMaxLevelsHost + lp;
      __syncthreads();  // the previous item's Green values are consumed
      // the children's level is lp + 1
      const double* G = a.gcell + size_t(lp - 1) * S::OFFS * 2 * KP + chunk * 2 * KC;
      for (int e = tid; e < NOFF * PC; e += kAccumThreads<double, CENTRAL>) {
        const int o = e / PC, j = e % PC;
        const int x = o % OW, y = (o / OW) % OW, z = o / (OW * OW);
        const int o343 = (x + 3 - OR) + 7 * (y + 3 - OR) + 49 * (z + 3 - OR);
        s_g[o * PC + (j ^ ((x & 1) * 2 + (y & 1) * 4))] =
            reinterpret_cast<const d2*>(G + size_t(o343) * 2 * KP)[j];
      }
      __syncthreads();
    }
    if (wave * WP >= pn) continue;  // wave-uniform; the barriers above are workgroup-uniform
    // row ids of the loader's parent (the zero row for an empty slot; any valid table row for an
    // absent parent, whose ids are not used): lane % 4 holds slot lane % 4 of a step
    const bool have = wave * WP + lpar < pn;
    const int* ids = a.blocks + size_t(plist[p0 + min(wave * WP + lpar, pn - 1)] - a.first_parent) * 216 +
                     B0 * 43 + (lane & 1) + 6 * ((lane >> 1) & 1);
    auto load_ids = [&](int u, int v, int bz) {
      const int r = ids[2 * u + 12 * v + 36 * bz];
      return have && r >= 0 ? r - a.first_cell : a.nsources;
    };
    const double* spec = a.sspec + chunk * 2 * KC + lpiece * 2;
    d2 rows[4];
    auto load_rows = [&](int idv, d2 (&to)[4]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int r = __shfl(idv, (lane & 60) + k, 64);
        to[k] = *reinterpret_cast<const d2*>(spec + size_t(r) * 2 * KP);
      }
    };
    d4 acc[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[m] = d4{0.0, 0.0, 0.0, 0.0};
    load_rows(load_ids(0, 0, 0), rows);
    int id_next = load_ids(1, 0, 0);
    for (int bz = 0; bz < NB; ++bz) {
#pragma unroll
      for (int st = 0; st < NU * NU; ++st) {
        const int u = st % NU, v = st / NU;
        wave_lds_fence();
#pragma unroll
        for (int k = 0; k < 4; ++k) sw[k * WP * PC] = rows[k];
        wave_lds_fence();
        if (st + 1 < NU * NU || bz + 1 < NB) {
          load_rows(id_next, rows);
          constexpr int NN = NU * NU;
          if (st + 2 < NN) id_next = load_ids((st + 2) % NU, (st + 2) / NU, bz);
          else if (bz + 1 < NB) id_next = load_ids((st + 2 - NN) % NU, (st + 2 - NN) / NU, bz + 1);
        }
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of this step's products
        const d2* gs = ga + (2 * u + 2 * OW * v + OW * OW * bz) * PC;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const d2 g = gs[(2 * w + apart) ^ aswz], b = sb[(2 * w + bpart) ^ bswz];
          acc[2 * w] = __builtin_amdgcn_mfma_f64_16x16x4f64(g.x, b.x, acc[2 * w], 0, 0, 0);
          acc[2 * w + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(g.y, b.y, acc[2 * w + 1], 0, 0, 0);
        }
      }
    }
    // D(c, Gr), D(c, Gi) of this column's part of S: the real part of T_c is D(Gr) of the real
    // column minus D(Gi) of the imaginary one, the imaginary part the sum of the other two
    const int k = wave * WP + bpar;
    const int par = plist[p0 + min(k, pn - 1)];
    const int* kids = a.child8 + size_t(par) * 8;
    double* out = a.tspec + chunk * 2 * KC + bpart * 2;
    d2 all = {0.0, 0.0};  // not finite where a value is not (or, harmlessly, the sum)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int t = k < pn ? kids[q + 4 * h] : -1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const double x0 = __shfl_xor(acc[2 * w][2 * h + 1], 1, 64);
        const double x1 = __shfl_xor(acc[2 * w + 1][2 * h + 1], 1, 64);
        const d2 o = bpart ? d2{acc[2 * w][2 * h] + x0, acc[2 * w + 1][2 * h] + x1}
                           : d2{acc[2 * w][2 * h] - x0, acc[2 * w + 1][2 * h] - x1};
        all += o;
        if (t >= 0) *reinterpret_cast<d2*>(out + size_t(t - a.first_cell) * 2 * KP + 4 * w) = o;
      }
    }
    if (k < pn && !finite(all.x + all.y)) {
#pragma unroll 1
      for (int e = 0; e < 8; ++e) {  // (child's half, mode pair)
        const int child = q + 4 * (e >> 2), w = e & 3, t = kids[child];
        if (t < 0) continue;
        d2* at = reinterpret_cast<d2*>(out + size_t(t - a.first_cell) * 2 * KP + 4 * w);
        const d2 v = *at;
        if (finite(v.x) && finite(v.y)) continue;
        const cplx<double> lo = zone_sum<double, NG, EXT, CENTRAL>(a, lp, par, child, chunk * KC + 2 * w);
        const cplx<double> hi = zone_sum<double, NG, EXT, CENTRAL>(a, lp, par, child, chunk * KC + 2 * w + 1);
        *at = bpart ? d2{lo.im, hi.im} : d2{lo.re, hi.re};
      }
    }
  }
}

// target node t (0 .. NL-1) of an axis sits at cyclic index t - EXT (mod C)
template <int C, int EXT>
__host__ __device__ constexpr int cyc(int t) { return t >= EXT ? t - EXT : t - EXT + C; }

// out_t = sum_k f[k] exp(+2 pi i k t' / C) at the NL target nodes t (t' = cyc(t)), handed to
// put(t, value); compile-time twiddles
template <int NL, int C, int EXT, typename F>
__device__ __forceinline__ void inverse_line(const cplx<double> (&f)[C], F&& put) {
  static_for<0, NL>([&](auto tc) {
    constexpr int t = cyc<C, EXT>(decltype(tc)::value);
    cplx<double> acc = f[0];
    static_for<1, C>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      constexpr double wr = cis_cos(long(k) * t, C), wi = cis_sin(long(k) * t, C);
      acc.re = fma(f[k].re, wr, acc.re);
      acc.re = fma(-f[k].im, wi, acc.re);
      acc.im = fma(f[k].re, wi, acc.im);
      acc.im = fma(f[k].im, wr, acc.im);
    });
    put(tc, acc);
  });
}

// ADD: the target already holds (mean, zero-mean gridlet) from the transform shared by its
// parent's children; this pass adds its own mean and zero-mean part to them (both precisions).
//
// Whole lines per thread, samples in registers and twiddles as immediates, instead of one output
// per thread with samples and twiddles from LDS (whose reads bounded it): 2^24 clustered particles,
// N_g = 4, FP32 2.88 -> 0.91 ms (4.5 GB read); 2^18 Plummer, N_g = 6 0.092 -> 0.035 ms.
template <typename T, int NG, int EXT, bool ADD = false>
__global__ __launch_bounds__(kCellThreads) void k_cells_inverse(CellArgs<T> a) {
  using S = CellShape<NG, EXT>;
  constexpr int C = S::C, HC = S::HC, KP = S::KP, NL = S::NL, M = S::ML;
  constexpr bool split = ADD || sizeof(T) == 4;
  constexpr int PER = cells_per_group<NG, EXT>();
  __shared__ cplx<double> s_b1[PER * NL * C * HC];   // [target][z][ky][kx]
  __shared__ cplx<double> s_b2[PER * NL * NL * HC];  // [target][z][y][kx]
  __shared__ double s_row[split ? PER * NL * NL : 1];
  const int tid = threadIdx.x;
  const int t0 = blockIdx.x * PER;
  const int cnt = min(PER, a.ntargets - t0);
  // z: one column (target, ky, kx) per thread, the NL target z values
  for (int q = tid; q < cnt * C * HC; q += kCellThreads) {
    const int tl = q / (C * HC), col = q % (C * HC);
    const T* row = a.tspec + size_t(t0 + tl) * 2 * KP;
    cplx<double> f[C];
    // C is even: whole mode pairs, 16 or 32 bytes, aligned
    typedef T t4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int j = 0; j < C / 2; ++j) {
      const t4 v = *reinterpret_cast<const t4*>(row + 2 * (col * C + 2 * j));
      f[2 * j] = {double(v[mode_pos<T>(0, 0)]), double(v[mode_pos<T>(0, 1)])};
      f[2 * j + 1] = {double(v[mode_pos<T>(1, 0)]), double(v[mode_pos<T>(1, 1)])};
    }
    inverse_line<NL, C, EXT>(f, [&](auto zc, cplx<double> o) {
      s_b1[(tl * NL + decltype(zc)::value) * C * HC + col] = o;
    });
  }
  __syncthreads();
  // y: one column (target, z, kx) per thread, the NL target y values
  for (int q = tid; q < cnt * NL * HC; q += kCellThreads) {
    const int z = q / HC, kx = q % HC;  // z: (target, z)
    cplx<double> f[C];
#pragma unroll
    for (int ky = 0; ky < C; ++ky) f[ky] = s_b1[(z * C + ky) * HC + kx];
    inverse_line<NL, C, EXT>(f, [&](auto yc, cplx<double> o) {
      s_b2[(z * NL + decltype(yc)::value) * HC + kx] = o;
    });
  }
  __syncthreads();
  // x: one row (target, z, y) per thread, the real part of the Hermitian sum over kx in
  // (-C/2, C/2]: the kx = 0 and kx = C/2 (Nyquist) terms once, the others twice
  const int g0 = a.first_cell + t0;
  constexpr int ROUNDS = (PER * NL * NL + kCellThreads - 1) / kCellThreads;
  double out[ROUNDS][NL];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int e = tid + r * kCellThreads;  // (target, z, y)
    if (e >= cnt * NL * NL) continue;
    cplx<double> f[HC];
#pragma unroll
    for (int kx = 0; kx < HC; ++kx) f[kx] = s_b2[e * HC + kx];
    double sum = 0.0;
    static_for<0, NL>([&](auto xc) {
      constexpr int X = cyc<C, EXT>(decltype(xc)::value);
      double acc = f[0].re;
      static_for<1, HC>([&](auto kc) {
        constexpr int kx = decltype(kc)::value;
        constexpr double w = kx == C / 2 ? 1.0 : 2.0;
        constexpr double wr = w * cis_cos(long(kx) * X, C), wi = w * cis_sin(long(kx) * X, C);
        acc = fma(f[kx].re, wr, acc);
        acc = fma(-f[kx].im, wi, acc);
      });
      out[r][decltype(xc)::value] = acc;
      sum += acc;
    });
    if constexpr (split) s_row[e] = sum;
    else {
#pragma unroll
      for (int x = 0; x < NL; ++x) a.local[size_t(g0) * M + size_t(e) * NL + x] = T(out[r][x]);
    }
  }
  if constexpr (split) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int e = tid + r * kCellThreads;
      if (e >= cnt * NL * NL) continue;
      const int tl = e / (NL * NL);
      double mean = 0.0;
      for (int k = 0; k < NL * NL; ++k) mean += s_row[tl * NL * NL + k];
      mean *= 1.0 / M;
      T* o = a.local + size_t(g0) * M + size_t(e) * NL;
#pragma unroll
      for (int x = 0; x < NL; ++x) {
        if constexpr (ADD) o[x] = T(double(o[x]) + (out[r][x] - mean));
        else o[x] = T(out[r][x] - mean);
      }
      if (e % (NL * NL) == 0) {
        if constexpr (ADD) a.m2l_mean[g0 + tl] += mean;
        else a.m2l_mean[g0 + tl] = mean;
      }
    }
  }
}

// tiles of at most "tile" split parents of one level
static TileTable tile_table(const Plan& p, int tile) {
  TileTable tt{};
  for (int lp = 1; lp <= kMaxLevelsHost; ++lp) {
    tt.first[lp] = tt.ntiles;
    tt.pbeg[lp] = p.cell_pbeg[std::min(lp, p.nlevels - 1)];
    if (lp + 1 < p.nlevels)
      tt.ntiles += (p.cell_pbeg[lp + 1] - p.cell_pbeg[lp] + tile - 1) / tile;
  }
  return tt;
}

// SHARED: the route with the transform shared by siblings (the central cubes here, the outer
// cubes by the per-parent kernel before the inverse adds to its result)
template <typename T, int NG, int EXT, bool SHARED = false>
static void cells_t(Plan& p, hipStream_t s, hipEvent_t fork) {
  using S = CellShape<NG, EXT>;
  static_assert(S::C <= kMaxCellC, "the Green table's kernel holds arrays of kMaxCellC per axis");
  p.m2l_split = SHARED || sizeof(T) == 4;
  p.m2l_mean_ff = false;  // this route's means are doubles
  if (p.nlevels <= 2) return;
  CellArgs<T> a;
  a.first_cell = p.level_off[2];
  const int ntargets = int(p.ncells) - a.first_cell;
  if (ntargets <= 0) return;
  a.nsources = ntargets + int(p.nvirt);
  a.ntargets = ntargets;
  a.first_parent = p.blocks_first;
  a.child8 = p.child8.as<int>();
  a.blocks = p.blocks.as<int>();
  a.gridlet = p.gridlet.as<T>();
  a.local = p.local.as<T>();
  a.gcell = p.tab.gcell.as<T>();
  a.sspec = p.cell_src.as<T>();
  a.tspec = p.cell_tgt.as<T>();
  a.m2l_mean = p.m2l_mean.as<double>();
  if (p.tab.gcell_levels < p.nlevels - 2) fail(HPM_ERR_DEVICE, "cell Green tables missing");
  if (p.cell_src.bytes < size_t(a.nsources + 1) * S::KP * sizeof(cplx<T>) ||
      p.cell_tgt.bytes < size_t(ntargets) * S::KP * sizeof(cplx<T>) ||
      p.local.bytes < size_t(p.ncells) * S::ML * sizeof(T))
    fail(HPM_ERR_DEVICE, "cell spectra buffers too small");
  constexpr int PER = cells_per_group<NG, EXT>();
  k_cells_forward<T, NG, EXT><<<a.nsources / PER + 1, kCellThreads, 0, s>>>(a);
  HPM_LAUNCH_CHECK();
  if (fork) HPM_HIP(hipEventRecord(fork, s));
  constexpr int64_t chunks = (S::KP + kChunkModes<T> - 1) / kChunkModes<T>;
  TileTable tt = tile_table(p, kTileParents<T, SHARED>);
  const bool fine = sizeof(T) == 4 && chunks * tt.ntiles <= kFineItems;
  if (fine) tt = tile_table(p, kTileParents<T, SHARED, sizeof(T) == 4>);
  if (tt.ntiles > 0) {
    const int64_t items = chunks * tt.ntiles;
    if (items > (int64_t(1) << 30)) fail(HPM_ERR_UNSUPPORTED, "too many cells for the cell-by-cell route");
    const int grid = int(std::min<int64_t>((items + 7) / 8 * 8, 256 * kAccumPerCU<T, SHARED>));
    if constexpr (sizeof(T) == 4) {
      if (fine)
        k_cells_accum_f32<NG, EXT, SHARED, true><<<grid, kAccumThreads<T, SHARED>, 0, s>>>(a, tt, p.cell_plist.as<int>());
      else
        k_cells_accum_f32<NG, EXT, SHARED><<<grid, kAccumThreads<T, SHARED>, 0, s>>>(a, tt, p.cell_plist.as<int>());
    } else
      k_cells_accum_f64<NG, EXT, SHARED><<<grid, kAccumThreads<T, SHARED>, 0, s>>>(a, tt, p.cell_plist.as<int>());
    HPM_LAUNCH_CHECK();
  }
  if constexpr (SHARED) launch_m2l_parents(p, s);
  k_cells_inverse<T, NG, EXT, SHARED><<<(ntargets + PER - 1) / PER, kCellThreads, 0, s>>>(a);
  HPM_LAUNCH_CHECK();
}

size_t cell_modes(int ng, int ext) {
  const size_t c = size_t(2 * ng + 2 * ext), k = c * c * (c / 2 + 1);
  return (k + 15) / 16 * 16;
}

// ---- list of split parents (cells of levels 1 .. L-2 with children), by level ----------------
// The list itself is written by the tree build; the start of each parent level in it is in the
// mailbox.
void read_cell_parents(Plan& p) {
  for (int l = 0; l <= kMaxLevelsHost; ++l) p.cell_pbeg[l] = 0;
  if (p.nlevels <= 2 || p.level_off[p.nlevels - 1] <= p.level_off[1]) return;
  for (int l = 1; l <= p.nlevels - 1; ++l) p.cell_pbeg[l] = p.hbox[Plan::kBoxCellLevels + l];
}

template <typename T>
static void cells_dispatch(Plan& p, hipStream_t s, hipEvent_t fork) {
  switch (p.ng * 2 + p.ext) {
    case 4: cells_t<T, 2, 0>(p, s, fork); break;
    case 5: cells_t<T, 2, 1>(p, s, fork); break;
    case 6: cells_t<T, 3, 0>(p, s, fork); break;
    case 7: cells_t<T, 3, 1>(p, s, fork); break;
    case 8: cells_t<T, 4, 0>(p, s, fork); break;
    case 9: cells_t<T, 4, 1>(p, s, fork); break;
    case 12: cells_t<T, 6, 0>(p, s, fork); break;
    case 13: cells_t<T, 6, 1>(p, s, fork); break;
    default: fail(HPM_ERR_UNSUPPORTED, "no cell-by-cell kernels for this gridlet");
  }
}

void launch_m2l_cells(Plan& p, hipStream_t s, hipEvent_t fork) {
  if (p.prec == HPM_F32) cells_dispatch<float>(p, s, fork);
  else cells_dispatch<double>(p, s, fork);
}

template <typename T>
static void shared_dispatch(Plan& p, hipStream_t s, hipEvent_t fork) {
  if (p.ext) fail(HPM_ERR_UNSUPPORTED, "the shared-transform route has no extended gridlet");
  switch (p.ng) {
    case 2: cells_t<T, 2, 0, true>(p, s, fork); break;
    case 3: cells_t<T, 3, 0, true>(p, s, fork); break;
    case 4: cells_t<T, 4, 0, true>(p, s, fork); break;
    case 6: cells_t<T, 6, 0, true>(p, s, fork); break;
    default: fail(HPM_ERR_UNSUPPORTED, "no shared-transform kernels for this gridlet");
  }
}

void launch_m2l_shared(Plan& p, hipStream_t s, hipEvent_t fork) {
  if (p.prec == HPM_F32) shared_dispatch<float>(p, s, fork);
  else shared_dispatch<double>(p, s, fork);
}

}  // namespace hpm
