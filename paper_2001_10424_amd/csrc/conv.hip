// Convolutions of the preconditioner network as implicit GEMMs on
// v_mfma_f32_16x16x32_bf16 (see conv.hpp).
//
// A block stages the input of a tile of points with its one-point halo in LDS
// once (zeros outside the grid), so a tap is an LDS read at a fixed offset
// instead of a gather from memory with its own address and bounds.  32 values
// of the GEMM's K dimension are two taps of 16 channels, four of 8 or eight
// of 4.
#include "conv.hpp"

#include <algorithm>
#include <type_traits>

namespace gkb {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

// tile of output points: rows of 32 points, 16 rows, whatever the grid (a grid
// two points wide is still no slower than single points gathered from memory,
// one point wide it is: 65536 x 1, 3 -> 8 -> 8 -> 2 channels 54 against 39 us)
template <int DIM>
struct CTile {
  static constexpr int TX = 32, TY = DIM == 3 ? 4 : 16, TZ = DIM == 3 ? 4 : 1;
  static constexpr int SX = TX + 2, SY = TY + 2, SZ = DIM == 3 ? TZ + 2 : 1;
  static constexpr int N = SX * SY * SZ;     // staged points
  static constexpr int TAPS = DIM == 3 ? 27 : 9;
};

// four values rounded to BF16 (to nearest even, the packed conversion of the
// hardware)
__device__ __forceinline__ s16x4 round4(f32x4 v) {
  return __builtin_bit_cast(s16x4, __builtin_convertvector(v, bf16x4));
}

struct TileAt {
  int x, y, z;  // origin
  long base;    // first point of the batch entry
};

template <int DIM>
__host__ __device__ inline long tile_count(const CnnGeom& g) {
  typedef CTile<DIM> C;
  return (long)((g.nx + C::TX - 1) / C::TX) * ((g.ny + C::TY - 1) / C::TY) *
         ((g.nz + C::TZ - 1) / C::TZ) * g.batch;
}

// The tiles of this block: first, first + step, .. < end.  Blocks with the same
// index mod 8 run on one XCD and get one range of consecutive tiles, so the
// halos that neighbours share come from that XCD's L2.  The grid is a multiple
// of 8 blocks.
struct TileRange {
  unsigned first, end, step;
};
__device__ __forceinline__ TileRange my_tiles(unsigned tiles) {
  const unsigned xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const unsigned lo = unsigned((unsigned long)tiles * xcd / 8),
                 hi = unsigned((unsigned long)tiles * (xcd + 1) / 8);
  return {lo + j, hi, gridDim.x >> 3};
}

template <int DIM>
__device__ __forceinline__ TileAt tile_at(const CnnGeom& g, unsigned t) {
  typedef CTile<DIM> C;
  const unsigned tx = (g.nx + C::TX - 1) / C::TX, ty = (g.ny + C::TY - 1) / C::TY,
                 tz = (g.nz + C::TZ - 1) / C::TZ;
  const unsigned a = t / tx, b = a / ty, c = b / tz;
  TileAt r;
  r.x = int(t - a * tx) * C::TX;
  r.y = int(a - b * ty) * C::TY;
  r.z = int(b - c * tz) * C::TZ;
  r.base = (long)c * g.nx * g.ny * g.nz;
  return r;
}

// CG channels of a point as loaded (BF16, or FP32 to be rounded): point q +
// row + x (q and row uniform)
template <int CG, bool F32>
struct Raw {
  s16x4 h[F32 ? 1 : CG / 4];
  f32x4 f[F32 ? CG / 4 : 1];
  __device__ __forceinline__ void load(const void* p, int c, long q, unsigned row, unsigned x) {
    if constexpr (!F32) {
      const s16x4* a = reinterpret_cast<const s16x4*>(static_cast<const uint16_t*>(p) + q * CG) +
                       (size_t)x * (CG / 4) + (size_t)row * (CG / 4);
#pragma unroll
      for (int e = 0; e < CG / 4; ++e) h[e] = a[e];
    } else {
      const float* a = static_cast<const float*>(p) + q * c;
      if (CG == 4 && c == 4 && (reinterpret_cast<uintptr_t>(p) & 15) == 0) {  // uniform
        f[0] = *(reinterpret_cast<const f32x4*>(a) + (size_t)x + (size_t)row);
        return;
      }
      a += ((size_t)x + row) * c;
#pragma unroll
      for (int e = 0; e < CG; ++e) f[e / 4][e % 4] = e < c ? a[e] : 0.f;
    }
  }
  __device__ __forceinline__ s16x4 get(int e) const {
    if constexpr (F32) return round4(f[e]);
    else return h[e];
  }
};

// Staging of a tile (with halo: HALO 1, without: 0) into sh[point][CG]: fetch
// issues a thread's loads, store writes them to LDS.  With the halo a wave
// takes whole rows of 34 points, so row, bounds and base are uniform and a
// lane's part of the address never changes; every load comes from inside the
// array (clamped) and a thread's loads are in flight together.  (Points dealt
// out to the threads one by one cost 50 vector instructions each for division,
// bounds and addresses.)
template <int DIM, int CG, bool F32, int HALO>
struct Stage {
  typedef CTile<DIM> C;
  static constexpr int SX = C::TX + 2 * HALO, SY = C::TY + 2 * HALO,
                       SZ = DIM == 3 ? C::TZ + 2 * HALO : 1;
  static constexpr int RPW = HALO ? 1 : 2;  // rows per wave and turn
  static constexpr int ROWS = SY * SZ, PER = (ROWS + 4 * RPW - 1) / (4 * RPW);
  static_assert(RPW * SX <= 64, "rows of a wave");
  Raw<CG, F32> r[PER];
  unsigned long rows;  // with the halo: bit l: row l of the box is in the grid
  unsigned in;         // the lane's x is; without: bit q: the point of turn q is
  __device__ __forceinline__ static int wave() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  }
  __device__ __forceinline__ void fetch(const CnnGeom& g, const TileAt& t, const void* p, int c) {
    const int lane = threadIdx.x & 63;
    const int lx = RPW == 1 ? lane : lane % SX, sub = RPW == 1 ? 0 : lane / SX;
    const int x = t.x + lx - HALO;
    const bool inx = lx < SX && unsigned(x) < unsigned(g.nx);
    const int xc = std::min(std::max(x, 0), g.nx - 1);
    // row `row` of the box: first point in the grid's array, and whether it
    // lies in the grid
    auto place = [&](int row, bool& on) {
      const int y = t.y + (DIM == 3 ? row % SY : row) - HALO,
                z = DIM == 3 ? t.z + row / SY - HALO : 0;
      on = row < ROWS && unsigned(y) < unsigned(g.ny) && unsigned(z) < unsigned(g.nz);
      const int yc = std::min(std::max(y, 0), g.ny - 1), zc = std::min(std::max(z, 0), g.nz - 1);
      return unsigned((zc * g.ny + yc) * g.nx);
    };
    in = inx ? 1u : 0u;
    if constexpr (RPW == 1) {
      // lane l places row l, and the wave takes its rows from the lanes: the
      // scalar unit, one instruction per cycle for the whole compute unit,
      // bounded the kernels when every wave placed its rows there (600
      // instructions per tile and wave: 30 us a layer at 128^3, 26 us like this)
      static_assert(ROWS <= 64, "a row per lane");
      bool on;
      const unsigned at = place(lane, on);
      rows = __ballot(on);
#pragma unroll
      for (int q = 0; q < PER; ++q)
        r[q].load(p, c, t.base, unsigned(__builtin_amdgcn_readlane(at, wave() + 4 * q)), xc);
    } else {
      in = 0;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        bool on;
        const unsigned at = place((wave() + 4 * q) * RPW + sub, on);
        r[q].load(p, c, t.base, 0u, at + xc);
        in |= (on && inx ? 1u : 0u) << q;
      }
    }
  }
  __device__ __forceinline__ void store(uint16_t* sh) const {
    const int lane = threadIdx.x & 63;
    const int lx = RPW == 1 ? lane : lane % SX, sub = RPW == 1 ? 0 : lane / SX;
    uint16_t* const d = sh + ((wave() * RPW + sub) * SX + lx) * CG;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (lx < SX && (wave() + 4 * q) * RPW + sub < ROWS)
#pragma unroll
        for (int e = 0; e < CG / 4; ++e) {
          const s16x4 v = r[q].get(e);
          const bool on = RPW == 1 ? in && ((rows >> (wave() + 4 * q)) & 1u) : (in >> q) & 1u;
          *reinterpret_cast<s16x4*>(d + 4 * q * RPW * SX * CG + 4 * e) = on ? v : s16x4{0, 0, 0, 0};
        }
    }
  }
};
template <int DIM, int CG, bool F32, int HALO>
__device__ __forceinline__ void stage(const CnnGeom& g, const TileAt& t, const void* p, int c,
                                      uint16_t* sh) {
  Stage<DIM, CG, F32, HALO> s;
  s.fetch(g, t, p, c);
  s.store(sh);
}

// output of four consecutive channels 4 c4 .. of point p (acc + bias)
template <int OUT>
__device__ __forceinline__ void put(f32x4 v, void* __restrict__ out, long p, int c4, int cout,
                                    int cgo, const uint16_t* __restrict__ mask) {
  if constexpr (OUT == kOutF32) {
    float* o = static_cast<float*>(out) + p * cout + 4 * c4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * c4 + e < cout) o[e] = v[e];
  } else if (4 * c4 < cgo) {
    // padded channels have weights, bias and mask 0
    s16x4 h;
    if (OUT == kOutReluBf16) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
      h = round4(v);
    } else {
      const s16x4 mk = *reinterpret_cast<const s16x4*>(mask + p * cgo + 4 * c4);
      h = round4(v);
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = mk[e] > 0 ? h[e] : short(0);  // sign bit: <= 0
    }
    *reinterpret_cast<s16x4*>(static_cast<uint16_t*>(out) + p * cgo + 4 * c4) = h;
  }
}

// LDS offset (in points of the halo box) of tap t seen from the point that
// the box stores at (x + 1, y + 1, z + 1)
template <int DIM>
__device__ __forceinline__ int tap_offset(int t) {
  typedef CTile<DIM> C;
  const int dx = t % 3, dy = (t / 3) % 3, dz = DIM == 3 ? t / 9 : 0;
  return (dz * C::SY + dy) * C::SX + dx;
}

// The A operand (rows = output channels) is the weights, kept in registers
// for the whole block; the B operand (columns = points) comes from LDS, 16
// bytes per lane and MFMA; a lane ends up with four consecutive channels of
// one point, an 8-byte store.
// (More than 8 output channels; k_conv_pair takes the others.)  Bound: LDS reads
// of the B operand, 1 KB per MFMA, and the staging in front of them; 512^2, 3
// -> 16 -> 16 -> 16 -> 2 channels: 44 us a forward call.
template <int DIM, int CG, bool F32, int OUT>
__global__ __launch_bounds__(kThreads) void k_conv(CnnGeom g, const void* __restrict__ in, int cin,
                                                   const uint16_t* __restrict__ w,
                                                   const float* __restrict__ bias,
                                                   void* __restrict__ out, int cout,
                                                   const uint16_t* __restrict__ mask,
                                                   const int* __restrict__ skip1,
                                                   const int* __restrict__ skip2,
                                                   unsigned first) {
  typedef CTile<DIM> C;
  if ((skip1 && *skip1) || (skip2 && *skip2)) return;
  constexpr int TPM = 32 / CG;                       // taps per MFMA
  constexpr int NM = (C::TAPS + TPM - 1) / TPM;      // MFMAs per 16 points
  __shared__ __align__(16) uint16_t sh[C::N * CG];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = lane & 15, kg = lane >> 4;
  const TileAt t = tile_at<DIM>(g, first + blockIdx.x);
  // the lane's eight K values of MFMA j: CG >= 8: tap t0, channels c0 ..;
  // CG = 4: taps t0 and t0 + 1
  s16x8 wr[NM];
  int off[NM], off1[NM];
#pragma unroll
  for (int j = 0; j < NM; ++j) {
    const int t0 = CG == 16 ? 2 * j + (kg >> 1) : (CG == 8 ? 4 * j + kg : 8 * j + 2 * kg);
    const int c0 = CG == 16 ? 8 * (kg & 1) : 0;
    s16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if constexpr (CG >= 8) {
      if (t0 < C::TAPS) v = *reinterpret_cast<const s16x8*>(w + t0 * 256 + m * 16 + c0);
      off[j] = t0 < C::TAPS ? tap_offset<DIM>(t0) * CG + c0 : -1;
      off1[j] = 0;
    } else {
      s16x4 a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
      if (t0 < C::TAPS) a = *reinterpret_cast<const s16x4*>(w + t0 * 256 + m * 16);
      if (t0 + 1 < C::TAPS) b = *reinterpret_cast<const s16x4*>(w + (t0 + 1) * 256 + m * 16);
      v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      off[j] = t0 < C::TAPS ? tap_offset<DIM>(t0) * CG : -1;
      off1[j] = t0 + 1 < C::TAPS ? tap_offset<DIM>(t0 + 1) * CG : -1;
    }
    wr[j] = v;
  }
  f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
  if (bias) b4 = *reinterpret_cast<const f32x4*>(bias + 4 * kg);
  const int cgo = chan_group(cout);
  stage<DIM, CG, F32, 1>(g, t, in, cin, sh);
  __syncthreads();
  // a wave takes one half of every second row of points
  const int wu = __builtin_amdgcn_readfirstlane(wv);
  const int lx = (wu & 1) * 16 + m, x = t.x + lx;
#pragma unroll 2
  for (int i = 0; i < C::TY * C::TZ / 2; ++i) {
    const int row = (wu >> 1) + 2 * i, ly = row % C::TY, lz = row / C::TY;
    const uint16_t* src = sh + ((lz * C::SY + ly) * C::SX + lx) * CG;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      s16x8 v;
      // only the last MFMA can run past the taps: those K values are 0
      if constexpr (CG >= 8) {
        v = *reinterpret_cast<const s16x8*>(src + (off[j] < 0 ? 0 : off[j]));
        if (j == NM - 1 && off[j] < 0) v = s16x8{0, 0, 0, 0, 0, 0, 0, 0};
      } else {
        s16x4 a = *reinterpret_cast<const s16x4*>(src + (off[j] < 0 ? 0 : off[j]));
        s16x4 b = *reinterpret_cast<const s16x4*>(src + (off1[j] < 0 ? 0 : off1[j]));
        if (j == NM - 1 && off[j] < 0) a = s16x4{0, 0, 0, 0};
        if (j == NM - 1 && off1[j] < 0) b = s16x4{0, 0, 0, 0};
        v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[j]),
                                                    __builtin_bit_cast(bf16x8, v), acc, 0, 0, 0);
    }
    // acc[e] = channel 4 kg + e of point m of the group
    const int y = t.y + ly, z = t.z + lz;  // uniform
    if (y >= g.ny || z >= g.nz) continue;
    const long p = t.base + ((long)z * g.ny + y) * g.nx + x;
    if (x < g.nx) put<OUT>(acc + b4, out, p, kg, cout, cgo, mask);
  }
}

// At most 8 output channels: the 16 rows of the A operand are the channels of
// two neighbouring points, (s, co) = (row / 8, row % 8), its K dimension the four
// taps dx = 0 .. 3 that the pair sees per tap row (dy, dz) (weight 0 where the
// point does not see the tap), and a column is a pair of points.  A row of 32
// points is one group: 9 MFMAs and LDS reads with 8 input channels where one
// point per column takes 14, and all offsets are compile-time ones plus the
// lane's.
// Infinities and NaNs must not reach a point that does not see them through a
// weight of 0: where a result is NaN the group is formed again, once per point
// of the pair, with the fourth tap zeroed.
// A block stays for several tiles (four blocks per CU): weights and set-up once,
// the next tile's loads in flight during the products.
// Bound: LDS reads, vector and scalar issue and MFMA take 2 to 3 us each of a
// tile's 5.5 us; 128^3, 4 -> 8 -> 8 -> 3 channels: 25 + 22 + 22 us, one point
// per column and one tile per block 34 + 31 + 29 us.
template <int DIM, int CG, bool F32, int OUT>
__global__ __launch_bounds__(kThreads, CG == 16 ? 2 : 4) void k_conv_pair(CnnGeom g, const void* __restrict__ in,
                                                        int cin, const uint16_t* __restrict__ w,
                                                        const float* __restrict__ bias,
                                                        void* __restrict__ out, int cout,
                                                        const uint16_t* __restrict__ mask,
                                                        const int* __restrict__ skip1,
                                                        const int* __restrict__ skip2) {
  typedef CTile<DIM> C;
  if ((skip1 && *skip1) || (skip2 && *skip2)) return;
  constexpr int R = C::TAPS / 3;  // tap rows
  constexpr int NM = CG == 4 ? (R + 1) / 2 : (CG == 8 ? R : 2 * R);
  __shared__ __align__(16) uint16_t sh[2][C::N * CG];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 15, kg = lane >> 4;
  const unsigned tiles = unsigned(tile_count<DIM>(g));
  const TileRange tr = my_tiles(tiles);
  if (tr.first >= tr.end) return;
  TileAt t = tile_at<DIM>(g, tr.first);
  Stage<DIM, CG, F32, 1> st;
  st.fetch(g, t, in, cin);
  // K values of the lane in MFMA j.  CG = 4: taps dx, dx + 1 of tap row 2 j +
  // (kg >> 1); CG = 8: tap kg of row j; CG = 16: half of the channels of tap
  // 2 (j & 1) + (kg >> 1) of row j >> 1
  auto tap_row = [&](int j) { return CG == 4 ? 2 * j + (kg >> 1) : (CG == 8 ? j : j >> 1); };
  auto tap_dx = [&](int j) { return CG == 4 ? 2 * (kg & 1) : (CG == 8 ? kg : 2 * (j & 1) + (kg >> 1)); };
  constexpr auto row_off = [](int r) { return ((r / 3) * C::SY + r % 3) * C::SX; };
  s16x8 wr[NM];
  {
    const int sft = m >> 3, co = m & 7;
    auto weight = [&](int r, int dx, int ch) {
      const int d = dx - sft;
      const bool on = r < R && unsigned(d) < 3u;
      return w + (on ? ((r * 3 + d) * 256 + co * 16 + ch) : 0);
    };
    auto seen = [&](int r, int dx) { return r < R && unsigned(dx - sft) < 3u; };
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      const int r = tap_row(j), dx = tap_dx(j), ch = CG == 16 ? 8 * (kg & 1) : 0;
      if constexpr (CG == 4) {
        s16x4 a = *reinterpret_cast<const s16x4*>(weight(r, dx, 0));
        s16x4 b = *reinterpret_cast<const s16x4*>(weight(r, dx + 1, 0));
        a = seen(r, dx) ? a : s16x4{0, 0, 0, 0};
        b = seen(r, dx + 1) ? b : s16x4{0, 0, 0, 0};
        wr[j] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      } else {
        const s16x8 a = *reinterpret_cast<const s16x8*>(weight(r, dx, ch));
        wr[j] = seen(r, dx) ? a : s16x8{0, 0, 0, 0, 0, 0, 0, 0};
      }
    }
  }
  const int c4 = kg & 1, px = 2 * m + (kg >> 1);  // the lane's channels and point
  f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
  if (bias) b4 = *reinterpret_cast<const f32x4*>(bias + 4 * c4);
  const int cgo = chan_group(cout);
  // drop: 0 none, 1 the tap that the first point of the pair does not see, 2
  // that of the second
  auto group = [&](const uint16_t* src, int drop) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      const int r = tap_row(j), dx = tap_dx(j);
      // the last tap row of CG = 4 is half empty: weights 0 on row 0
      const int ro = CG == 4 ? ((kg >> 1) ? row_off(2 * j + 1 < R ? 2 * j + 1 : 0) : row_off(2 * j))
                             : row_off(CG == 8 ? j : j >> 1);
      s16x8 v = *reinterpret_cast<const s16x8*>(src + (ro + dx) * CG + (CG == 16 ? 8 * (kg & 1) : 0));
      if (drop) {
        const int gone = drop == 1 ? 3 : 0;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (r >= R || dx + (CG == 4 ? e / 4 : 0) == gone) v[e] = 0;
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[j]),
                                                    __builtin_bit_cast(bf16x8, v), acc, 0, 0, 0);
    }
    return acc;
  };
  // the next tile's loads are in flight while this one is computed; its LDS
  // was last read before the barrier
  int buf = 0;
  for (unsigned tl = tr.first; tl < tr.end; tl += tr.step, buf ^= 1) {
    st.store(sh[buf]);
    __syncthreads();
    const TileAt cur = t;
    if (tl + tr.step < tr.end) {
      t = tile_at<DIM>(g, tl + tr.step);
      st.fetch(g, t, in, cin);
    }
#pragma unroll 1
    for (int i = 0; i < C::TY * C::TZ / 4; ++i) {
      const int ly = DIM == 3 ? wv : wv + 4 * i, lz = DIM == 3 ? i : 0;
      static_assert(DIM == 2 || (C::TY == 4 && C::TZ == 4), "a wave per row of a plane");
      const uint16_t* src = sh[buf] + ((lz * C::SY + ly) * C::SX + 2 * m) * CG;
      f32x4 acc = group(src, 0);
      const float sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
      if (__any(!(sum == sum))) {
        // (reads LDS again: its values are not kept for this path)
        asm volatile("" ::: "memory");
        const f32x4 a = group(src, 1);
        asm volatile("" ::: "memory");
        const f32x4 b = group(src, 2);
        acc = kg < 2 ? a : b;
      }
      const int x = cur.x + px, y = cur.y + ly, z = cur.z + lz;  // y, z uniform
      if (y >= g.ny || z >= g.nz) continue;
      const long p = cur.base + ((long)z * g.ny + y) * g.nx + x;
      if (x < g.nx) put<OUT>(acc + b4, out, p, c4, cout, cgo, mask);
    }
  }
}

// four consecutive 16-bit values along the first index of a matrix stored
// with rows of 16-bit elements in LDS: the 16 lanes of a quarter wave give the
// 8-byte pieces of four rows, lane i piece i % 4 of row i / 4, and lane i gets
// column i of the four rows
__device__ __forceinline__ s16x4 lds_transposed(const uint16_t* a) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(const_cast<uint16_t*>(a)));
}

// Weight gradient: a GEMM over points.  The rows of an accumulator tile are
// (tap, ci) pairs (one tap of 16 input channels, two of 8 or four of 4), its
// columns the output channels, its K dimension 32 points of a row.  Both
// operands need consecutive points per lane while LDS holds points by
// channels, which the transposing LDS read resolves; a tap is an offset of
// whole points, so it stays aligned.  One more tile with a row of ones gives
// the bias gradient.  A block sums several tiles of points and writes one set
// of FP32 partials; k_wgrad_reduce adds the sets in a fixed order.
// CUT: tiles can reach past the grid.  The points there have dz = 0, but their
// taps see activations inside it, and 0 times an infinity is no 0: where a
// block's sums hold a NaN it forms them again without those points (their rows
// left out, zeros read in a row).  Leaving them out at once, by a mask or by the
// address, cost 3 to 4 us a layer at 62^3 x 2 points.
// 64^3 x 2 points: 15 us for 8 x 8 channels and 14 us for 4 x 8; 235 and 142
// us with single BF16 values gathered from memory.
template <int DIM, int CG>
constexpr int wgrad_tiles() { return (CTile<DIM>::TAPS * CG + 15) / 16; }

template <int DIM, int CG, int CGZ, bool FA, bool FZ, bool CUT>
__global__ __launch_bounds__(kThreads) void k_wgrad(CnnGeom g, const void* __restrict__ act, int ca,
                                                    const void* __restrict__ dz, int cz,
                                                    float* __restrict__ part) {
  typedef CTile<DIM> C;
  constexpr int NT = wgrad_tiles<DIM, CG>(), TPT = 16 / CG;  // taps per tile
  constexpr int NZ = C::TX * C::TY * C::TZ;
  constexpr int NR = (NT + 1) * 256;
  // CUT: zeros as far as a point's taps reach
  constexpr int ZERO = CUT ? (((DIM == 3 ? 2 * C::SY : 0) + 2) * C::SX + 3) * CG : 0;
  constexpr int BYTES = (C::N * CG + NZ * CGZ + ZERO) * 2;
  __shared__ __align__(16) char raw[BYTES > NR * 4 ? BYTES : NR * 4];
  uint16_t* sa = reinterpret_cast<uint16_t*>(raw);
  uint16_t* sz = sa + C::N * CG;
  uint16_t* zero = sz + NZ * CGZ;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = lane & 15, kg = lane >> 4;
  const int piece = i & 3, row = i >> 2;
  // LDS offset of the lane's piece of tile t, relative to its point
  int off[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int tap = std::min(t * TPT + (CG == 16 ? 0 : (CG == 8 ? piece >> 1 : piece)), C::TAPS - 1);
    const int ch = CG == 16 ? 4 * piece : (CG == 8 ? 4 * (piece & 1) : 0);
    off[t] = tap_offset<DIM>(tap) * CG + ch;
  }
  const int zch = 4 * (piece % (CGZ / 4));  // columns beyond the group are not used
  f32x4 acc[NT + 1];
  s16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = short(0x3F80);
  const unsigned tiles = unsigned(tile_count<DIM>(g));
  // the block's tiles; cut: points past the grid take no part
  auto sweep = [&](auto cut) {
#pragma unroll
    for (int t = 0; t <= NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (unsigned tl = blockIdx.x; tl < tiles; tl += gridDim.x) {
      const TileAt t = tile_at<DIM>(g, tl);
      __syncthreads();  // the last tile's reads
      stage<DIM, CG, FA, 1>(g, t, act, ca, sa);
      stage<DIM, CGZ, FZ, 0>(g, t, dz, cz, sz);
      __syncthreads();
      for (int r = wv; r < C::TY * C::TZ; r += kThreads / 64) {
        const int ly = r % C::TY, lz = r / C::TY;
        if (cut && (t.y + ly >= g.ny || t.z + lz >= g.nz)) continue;  // uniform in the wave
        // K values of the lane: points 8 kg + 0 .. 7 of the row
        const int x = 8 * kg + row;
        const uint16_t* pz = sz + (r * C::TX + x) * CGZ + zch;
        const s16x4 z0 = lds_transposed(pz), z1 = lds_transposed(pz + 4 * CGZ);
        const s16x8 zv = __builtin_shufflevector(z0, z1, 0, 1, 2, 3, 4, 5, 6, 7);
        const uint16_t* pa = sa + ((lz * C::SY + ly) * C::SX + x) * CG;
        const uint16_t* pb = pa + 4 * CG;
        if constexpr (cut) {
          if (t.x + x >= g.nx) pa = zero;
          if (t.x + x + 4 >= g.nx) pb = zero;
        }
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          const s16x4 a0 = lds_transposed(pa + off[q]), a1 = lds_transposed(pb + off[q]);
          const s16x8 av = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av),
                                                           __builtin_bit_cast(bf16x8, zv), acc[q],
                                                           0, 0, 0);
        }
        acc[NT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones),
                                                          __builtin_bit_cast(bf16x8, zv), acc[NT],
                                                          0, 0, 0);
      }
    }
  };
  sweep(std::false_type{});
  if constexpr (CUT) {
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) sum += (acc[t][0] + acc[t][1]) + (acc[t][2] + acc[t][3]);
    if (__syncthreads_or(sum != sum)) {
      for (int e = threadIdx.x; e < ZERO; e += kThreads) zero[e] = 0;
      sweep(std::true_type{});
    }
  }
  // the waves add their tiles in a fixed order
  float* red = reinterpret_cast<float*>(raw);
  for (int w = 0; w < kThreads / 64; ++w) {
    __syncthreads();
    if (wv == w)
#pragma unroll
      for (int t = 0; t <= NT; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float* d = red + t * 256 + (4 * kg + q) * 16 + i;
          *d = w == 0 ? acc[t][q] : *d + acc[t][q];
        }
  }
  __syncthreads();
  float* dst = part + (size_t)blockIdx.x * NR;
  for (int e = threadIdx.x; e < NR; e += kThreads) dst[e] = red[e];
}

// Sum the block partials in a fixed order into the flat layer gradient
// W[tap][ci][co], b[co]: a block takes 16 consecutive partial entries, its 16
// thread groups sum the sets b = grp, grp + 16, ..., and the 16 group sums are
// added in order.  One launch for all layers of a network: a layer's sum is
// one dependent trip to memory of 4.7 us that leaves most of the chip idle;
// three together take 8.9 us.  Backward
// of three layers at 64^3 x 2 points: 146.7 -> 142.9 us (mean of three
// comparisons; 145.8-147.3 against 142.6-143.1).
constexpr int kRedOut = 16;
__global__ __launch_bounds__(kThreads) void k_wgrad_reduce(WgradSum ws, int taps) {
  int la = 0;
  while (la + 1 < ws.layers && int(blockIdx.x) >= ws.first[la + 1]) ++la;
  const WgradLayer& l = ws.l[la];
  const int nblk = ws.nblk, nt = l.nt, cg = l.cg, cin = l.cin, cout = l.cout;
  const float* __restrict__ part = l.part;
  float* __restrict__ flat = l.flat;
  const int o = threadIdx.x % kRedOut, grp = threadIdx.x / kRedOut;
  const int np = (nt + 1) * 256, e = (int(blockIdx.x) - ws.first[la]) * kRedOut + o;
  float s = 0.f;
#pragma unroll 8
  for (int b = grp; b < nblk; b += kThreads / kRedOut) s += part[(size_t)b * np + e];
  __shared__ float sh[kThreads];
  sh[threadIdx.x] = s;
  __syncthreads();
  if (grp != 0) return;
  float t = 0.f;
  for (int q = 0; q < kThreads / kRedOut; ++q) t += sh[q * kRedOut + o];
  // entry e: tile, row (tap, ci) of the tile, column co = o
  const int row = (e >> 4) & 15, tile = e >> 8;
  if (o >= cout) return;
  if (tile == nt) {
    if (row == 0) flat[taps * cin * cout + o] = t;
    return;
  }
  const int tap = tile * (16 / cg) + row / cg, ci = row % cg;
  if (tap < taps && ci < cin) flat[(tap * cin + ci) * cout + o] = t;
}

constexpr unsigned kPairBlocks = 1024;  // four per CU, which fit
constexpr unsigned kMaxBlocks = 1u << 23;  // a launch has less than 2^32 threads

template <int DIM, int CG, bool F32>
void launch_conv(hipStream_t s, const CnnGeom& g, const ConvIn& in, const uint16_t* w,
                 const float* bias, ConvOut mode, void* out, int cout, const uint16_t* mask,
                 const int* skip1, const int* skip2) {
  const unsigned tiles = unsigned(tile_count<DIM>(g));
  auto several = [&](auto kernel) {  // tiles per block
    const unsigned grid = std::min((tiles + 7) / 8 * 8, kPairBlocks);
    kernel<<<grid, kThreads, 0, s>>>(g, in.p, in.c, w, bias, out, cout, mask, skip1, skip2);
  };
  auto one = [&](auto kernel) {
    for (unsigned first = 0; first < tiles; first += kMaxBlocks)
      kernel<<<std::min(tiles - first, kMaxBlocks), kThreads, 0, s>>>(
          g, in.p, in.c, w, bias, out, cout, mask, skip1, skip2, first);
  };
  const bool pair = cout <= 8;
  switch (mode) {
    case kOutReluBf16:
      pair ? several(k_conv_pair<DIM, CG, F32, kOutReluBf16>)
           : one(k_conv<DIM, CG, F32, kOutReluBf16>);
      break;
    case kOutF32:
      pair ? several(k_conv_pair<DIM, CG, F32, kOutF32>) : one(k_conv<DIM, CG, F32, kOutF32>);
      break;
    case kOutMaskBf16:
      pair ? several(k_conv_pair<DIM, CG, F32, kOutMaskBf16>)
           : one(k_conv<DIM, CG, F32, kOutMaskBf16>);
      break;
  }
}

template <int DIM, bool F32>
void conv_cg(hipStream_t s, const CnnGeom& g, const ConvIn& in, const uint16_t* w,
             const float* bias, ConvOut mode, void* out, int cout, const uint16_t* mask,
             const int* skip1, const int* skip2) {
  const int cg = chan_group(in.c);
  if (cg == 4) launch_conv<DIM, 4, F32>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
  else if (cg == 8) launch_conv<DIM, 8, F32>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
  else launch_conv<DIM, 16, F32>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
}

template <int DIM, int CG, int CGZ, bool FA>
void wgrad_fz(hipStream_t s, const CnnGeom& g, const ConvIn& act, const ConvIn& dz, float* part,
              int nblk) {
  typedef CTile<DIM> C;
  const bool cut = g.nx % C::TX || g.ny % C::TY || g.nz % C::TZ;
  auto go = [&](auto kernel) {
    kernel<<<nblk, kThreads, 0, s>>>(g, act.p, act.c, dz.p, dz.c, part);
  };
  if (dz.f32) cut ? go(k_wgrad<DIM, CG, CGZ, FA, true, true>) : go(k_wgrad<DIM, CG, CGZ, FA, true, false>);
  else cut ? go(k_wgrad<DIM, CG, CGZ, FA, false, true>) : go(k_wgrad<DIM, CG, CGZ, FA, false, false>);
}

template <int DIM, int CG>
void wgrad_cg(hipStream_t s, const CnnGeom& g, const ConvIn& act, const ConvIn& dz, float* part,
              float* flat, WgradSum& sum) {
  const int nblk = wgrad_blocks(DIM, g), cz = chan_group(dz.c);
  // FP32 activations are the network's input only
  if (act.f32) {
    if (cz == 4) wgrad_fz<DIM, CG, 4, true>(s, g, act, dz, part, nblk);
    else if (cz == 8) wgrad_fz<DIM, CG, 8, true>(s, g, act, dz, part, nblk);
    else wgrad_fz<DIM, CG, 16, true>(s, g, act, dz, part, nblk);
  } else {
    if (cz == 4) wgrad_fz<DIM, CG, 4, false>(s, g, act, dz, part, nblk);
    else if (cz == 8) wgrad_fz<DIM, CG, 8, false>(s, g, act, dz, part, nblk);
    else wgrad_fz<DIM, CG, 16, false>(s, g, act, dz, part, nblk);
  }
  constexpr int nt = wgrad_tiles<DIM, CG>();
  sum.nblk = nblk;
  sum.l[sum.layers] = WgradLayer{part, flat, nt, CG, act.c, dz.c};
  sum.first[sum.layers + 1] = sum.first[sum.layers] + (nt + 1) * 256 / kRedOut;
  ++sum.layers;
}

template <int DIM>
void wgrad_dim(hipStream_t s, const CnnGeom& g, const ConvIn& act, const ConvIn& dz, float* part,
               float* flat, WgradSum& sum) {
  const int cg = chan_group(act.c);
  if (cg == 4) wgrad_cg<DIM, 4>(s, g, act, dz, part, flat, sum);
  else if (cg == 8) wgrad_cg<DIM, 8>(s, g, act, dz, part, flat, sum);
  else wgrad_cg<DIM, 16>(s, g, act, dz, part, flat, sum);
}

}  // namespace

void conv_layer(hipStream_t s, int dim, const CnnGeom& g, const ConvIn& in, const uint16_t* w,
                const float* bias, ConvOut mode, void* out, int cout, const uint16_t* mask,
                const int* skip1, const int* skip2) {
  if (dim == 2) {
    if (in.f32) conv_cg<2, true>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
    else conv_cg<2, false>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
  } else {
    if (in.f32) conv_cg<3, true>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
    else conv_cg<3, false>(s, g, in, w, bias, mode, out, cout, mask, skip1, skip2);
  }
}

// blocks of the weight gradient: two per CU (14-15 us a layer at 64^3 x 2; one
// per CU takes 16-18 us and saves nothing in the reduction, 4.7 us)
int wgrad_blocks(int dim, const CnnGeom& g) {
  const long tiles = dim == 2 ? tile_count<2>(g) : tile_count<3>(g);
  return int(std::min<long>(tiles, 512));
}

size_t wgrad_part_floats(int dim, const CnnGeom& g, int cin) {
  const int cg = chan_group(cin), taps = dim == 2 ? CTile<2>::TAPS : CTile<3>::TAPS;
  const int nt = (taps * cg + 15) / 16;
  return (size_t)wgrad_blocks(dim, g) * (nt + 1) * 256;
}

void wgrad_layer(hipStream_t s, int dim, const CnnGeom& g, const ConvIn& act, const ConvIn& dz,
                 float* part, float* flat, WgradSum& sum) {
  if (dim == 2) wgrad_dim<2>(s, g, act, dz, part, flat, sum);
  else wgrad_dim<3>(s, g, act, dz, part, flat, sum);
}

void wgrad_finish(hipStream_t s, int dim, const WgradSum& sum) {
  if (sum.layers == 0) return;
  k_wgrad_reduce<<<sum.first[sum.layers], kThreads, 0, s>>>(
      sum, dim == 2 ? CTile<2>::TAPS : CTile<3>::TAPS);
}

}  // namespace gkb
