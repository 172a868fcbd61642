// tiles_ahead.hip -- the tiled schedule (tiles.hip) with tiles of edge 16 or (2D)
// 32 or 64 at one bit per site in LDS, their decisions formed ahead.
//
// What a site draws does not depend on the state: whether it would accept as a
// member of each class that can refuse is one bit a class, the prefix byte
// against the class's threshold and, on a tie, the refinement draw.  So the
// waves of a workgroup first form those masks for the 2 H passes of H hits --
// every draw, with the ties of all passes in full waves -- and the passes
// themselves are left with the neighbours' words, the count of unsatisfied bonds
// and a select among the masks.  Forming them as the passes need them has the
// draws, the transpose and the round of tie draws in every pass's serial chain
// (1.9 us a hit where a tile has a SIMD to itself).
//
// A workgroup owns 64 words (one to sixteen tiles), a lane of its first wave a
// word of both colours in registers.  That wave runs the passes of one chunk of
// hits while the others form the next chunk's masks.  us a sweep of k = 100,
// forming them in the passes / here: 2D T = 16 L = 1024 378 / 80, L = 4096 586 /
// 473; T = 32 L = 1024 313 / 68, L = 4096 483 / 371; T = 64 L = 2048 346 / 113, L =
// 4096 471 / 375; 3D T = 16 L = 128 402 / 100, L = 256 629 / 548.  Vector issue
// bounds the large ones: 309 instructions a word and pass for 16-edge tiles (four
// Philox blocks 134, transpose 59, masks 32, ties 45, the pass 40), 206 of 236 us
// a launch at L = 4096.
#include "chunk.hpp"
#include "packed.hpp"

#include <algorithm>
#include <type_traits>

namespace smc {

namespace {

// Layout of a T x T tile (a plane of a 3D one): a tile row holds RB = T / 2 sites
// of a colour, so a word packs 32 / RB tile rows -- word i of a tile's colour
// holds rows NR i .. NR i + NR - 1 of the tile, site s of row r in bit RB r + s
// (bit 1 = spin -1).  Per colour, LDS holds the column [above, w0 .. w(NW - 1),
// below] (the boundary row above the tile in the top RB bits of `above`, the one
// below in the low bits of `below`), so the y neighbours of word i are funnel
// shifts of its column by RB; x neighbours are a shift by one within each row's
// bits, completed by the sites left and right of the rows (bits RB r and RB r +
// RB - 1), which the lane keeps.  Row r of a word has parity (c + r) & 1 (tiles
// start at even rows), a mask.  T = 16: a row's 8 prefix bytes are words 2 h0, 2
// h0 + 1 of its 16-site Philox block, so a word takes four blocks; else two.
template <uint32_t T>
struct RowTile {
  static constexpr uint32_t RB = T / 2;       // sites of a colour in a tile row
  static constexpr uint32_t NR = 32 / RB;     // tile rows of a word
  static constexpr uint32_t NW = T / NR;      // words of a colour in a plane of the tile
  static constexpr uint32_t Words = NW + 2;   // with the boundary rows
  static constexpr uint32_t First = T == 16 ? 0x01010101u : T == 32 ? 0x00010001u : 1u;  // bit 0 of each row
  static constexpr uint32_t Last = First << (RB - 1);
  // rows with the next site as x + 1 neighbour: those of odd c + y + z
  __device__ static __forceinline__ uint32_t ahead(uint32_t parity) {  // of the word's first row
    if (T == 64) return 0u - parity;
    const uint32_t odd = T == 16 ? 0xFF00FF00u : 0xFFFF0000u;
    return parity ? ~odd : odd;
  }
  __device__ static __forceinline__ uint32_t above(uint32_t before, uint32_t w) {
    return T == 64 ? before : __builtin_amdgcn_alignbit(w, before, 32u - RB);
  }
  __device__ static __forceinline__ uint32_t below(uint32_t w, uint32_t after) {
    return T == 64 ? after : __builtin_amdgcn_alignbit(after, w, RB);
  }
  // sign bits of a tile row's sites
  __device__ static __forceinline__ uint32_t bits(const int8_t* row) {
    uint32_t v = 0;
#pragma unroll
    for (uint32_t k = 0; k < RB / 8; ++k) {
      const uint2 q = *reinterpret_cast<const uint2*>(row + 8 * k);
      v |= (gather7(q.x) | (gather7(q.y) << 4)) << (8 * k);
    }
    return v;
  }
  // the prefix bytes of the word whose first site is j0, hit h; H0 (T = 16): the
  // half of the Philox blocks the wave's rows take, 2: some take either
  template <int H0>
  __device__ static __forceinline__ void prefix(const RngKey& key, uint32_t t, uint32_t c, uint32_t h,
                                                uint32_t j0, uint32_t R, uint32_t P[8]) {
    constexpr uint32_t Blocks = T == 16 ? 4 : 2;
#pragma unroll
    for (uint32_t r = 0; r < Blocks; ++r) {
      const uint32_t jr = T == 64 ? j0 + 16 * r : j0 + r * R;
      const Rand4 rb = philox(jr >> 4, t, key.replica, tag(c, kIsingPrefix) | (h << 8), key.k0, key.k1);
      if (T == 16) {
        const bool h0 = H0 == 2 ? ((jr >> 3) & 1u) != 0 : H0 == 1;
        P[2 * r] = h0 ? rb.w[2] : rb.w[0];
        P[2 * r + 1] = h0 ? rb.w[3] : rb.w[1];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) P[(4 * r + k) & 7u] = rb.w[k];
      }
    }
  }
  // a tile row's +-1 bytes from its bits
  __device__ static __forceinline__ void store(int8_t* row, uint32_t v) {
#pragma unroll
    for (uint32_t k = 0; k < RB / 8; ++k) {
      const uint32_t byte = (v >> (8 * k)) & 0xFFu;
      uint32_t q[2];
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const uint32_t spread = (((byte >> (4 * w)) & 0xFu) * 0x00204081u) & kOnes;
        q[w] = kOnes | (spread * 0xFEu);
      }
      *reinterpret_cast<uint2*>(row + 8 * k) = make_uint2(q[0], q[1]);
    }
  }
};

template <int D, uint32_t T>
struct Group {
  static constexpr uint32_t Lanes = (D == 3 ? T : 1u) * RowTile<T>::NW;  // words of a colour of a tile
  static constexpr uint32_t Tiles = 64u / Lanes;                         // of the workgroup
  static constexpr uint32_t CW = (D == 3 ? T + 2 : 1u) * RowTile<T>::Words;  // LDS words of a tile's colour
};

struct TileAheadArgs {
  Geom g;
  RngKey key;
  uint32_t th[7], frac[7];  // of the classes with a mask
  uint32_t invert;          // ~0: count satisfied bonds (Metropolis with J0 < 0)
  uint32_t hits, chunk;     // hits of a launch; hits whose masks are formed together
  uint32_t t, tc, ntiles;
  int8_t* s;
};

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t sel3(uint32_t m, uint32_t a, uint32_t b) {  // m ? a : b, bitwise
  return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}

}  // namespace

template <int D, uint32_t T, bool HB>
__global__ __launch_bounds__(768) void tile_ahead_kernel(const TileAheadArgs a) {
  using TL = RowTile<T>;
  using GR = Group<D, T>;
  constexpr uint32_t NC = HB ? 2 * D + 1 : D;  // classes with a mask
  extern __shared__ uint32_t lds[];
  const uint32_t tid = threadIdx.x, lane = __lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
  uint32_t* const state = lds;                // [Tiles][2][CW]
  const uint32_t buf_words = 2u * a.chunk * NC * 64u;  // masks of a chunk, twice
  uint32_t* const masks = state + GR::Tiles * 2u * GR::CW;
  uint32_t* const list = masks + 2u * buf_words + wave * 128u;
  const uint32_t L = (uint32_t)a.g.L, R = (uint32_t)a.g.R;
  const uint64_t Nh = (uint64_t)a.g.Nh;

  // ---- the lane's word (the same in every wave) ----
  const uint32_t gi = lane / GR::Lanes, li = lane % GR::Lanes, z = li / TL::NW, i = li % TL::NW;
  const uint32_t bt = blockIdx.x * GR::Tiles + gi;
  const bool valid = bt < a.ntiles;
  const uint32_t nt = L / T, half = nt / 2;
  const uint32_t bv = valid ? bt : 0u;
  const uint32_t tz = D == 3 ? bv / (nt * half) : 0u, rem = bv - tz * nt * half;
  const uint32_t ty = rem / half;
  const uint32_t tx = 2 * (rem - ty * half) + ((ty + tz + a.tc) & 1u);
  const uint32_t Zg = tz * T + z, Y = ty * T + TL::NR * i, x0 = tx * TL::RB;
  const uint32_t j0 = (Zg * L + Y) * R + x0;  // in-colour index of the word's first site
  uint32_t* const col = state + gi * 2u * GR::CW + (D == 3 ? (z + 1u) * TL::Words : 0u);  // colour 0

  // ---- stage ----
  uint32_t ow[2] = {0u, 0u}, lh[2] = {0u, 0u}, rh[2] = {0u, 0u};
  if (wave == 0u && valid) {
    const uint32_t xl = x0 == 0 ? R - 1 : x0 - 1, xr = x0 + TL::RB == R ? 0 : x0 + TL::RB;
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c) {
      auto rowp = [&](uint32_t zg, uint32_t y) -> const int8_t* {
        return a.s + c * Nh + ((uint64_t)zg * L + y) * R;
      };
      uint32_t* const cc = col + c * GR::CW;
#pragma unroll
      for (uint32_t r = 0; r < TL::NR; ++r) {
        const int8_t* row = rowp(Zg, Y + r);
        ow[c] |= TL::bits(row + x0) << (TL::RB * r);
        lh[c] |= (row[xl] < 0 ? 1u : 0u) << (TL::RB * r);
        rh[c] |= (row[xr] < 0 ? 1u << (TL::RB - 1) : 0u) << (TL::RB * r);
      }
      cc[1 + i] = ow[c];
      const uint32_t Y0 = ty * T;
      if (i == 0) cc[0] = TL::bits(rowp(Zg, Y0 == 0 ? L - 1 : Y0 - 1) + x0) << (32 - TL::RB);
      if (i == TL::NW - 1) cc[TL::NW + 1] = TL::bits(rowp(Zg, Y0 + T == L ? 0 : Y0 + T) + x0);
      if (D == 3 && (z == 0 || z == T - 1)) {
        const uint32_t zb = z == 0 ? (Zg == 0 ? L - 1 : Zg - 1) : (Zg + 1 == L ? 0 : Zg + 1);
        uint32_t wb = 0;
#pragma unroll
        for (uint32_t r = 0; r < TL::NR; ++r) wb |= TL::bits(rowp(zb, Y + r) + x0) << (TL::RB * r);
        state[gi * 2u * GR::CW + c * GR::CW + (z == 0 ? 0u : T + 1) * TL::Words + 1 + i] = wb;
      }
    }
  }

  // ---- masks of the passes k0, k0 + dk, ... of the hits h0 .. h0 + nh - 1 ----
  auto form_half = [&](auto H0, uint32_t h0, uint32_t nh, uint32_t* m, uint32_t k0,
                       uint32_t dk) __attribute__((always_inline)) {
    uint32_t n = 0u;  // tied sites in the wave's list
    auto draw = [&](uint32_t from) __attribute__((always_inline)) {
      wave_sync();
      const uint32_t e = from + lane < n ? list[from + lane] : 0u;
      const uint32_t who = e & 63u, b = (e >> 6) & 31u, q = (e >> 11) & 7u, k = e >> 14;
      const uint32_t jw = (uint32_t)__shfl((int)j0, (int)who);
      if (from + lane < n) {
        const Rand4 rr = philox(jw + b / TL::RB * R + b % TL::RB, a.t, a.key.replica,
                                tag(k & 1u, kIsingRefine) | ((h0 + (k >> 1)) << 8), a.key.k0, a.key.k1);
        uint32_t frac = a.frac[0];
#pragma unroll
        for (uint32_t p = 1; p < NC; ++p) frac = q == p ? a.frac[p] : frac;
        if ((rr.w[0] & 0xFFFFFFu) < frac) atomicOr(&m[(k * NC + q) * 64u + who], 1u << b);
      }
      n = from;
    };
#pragma unroll 1
    for (uint32_t k = k0; k < 2u * nh; k += dk) {
      uint32_t P[8], B[8];
      TL::template prefix<decltype(H0)::value>(a.key, a.t, k & 1u, h0 + (k >> 1), j0, R, P);
      prefix_planes(P, B);
#pragma unroll
      for (uint32_t q = 0; q < NC; ++q) {
        uint32_t lt = 0u, e = ~0u;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const uint32_t X = 0u - ((a.th[q] >> b) & 1u);  // wave-uniform
          lt = __builtin_amdgcn_bitop3_b32(B[b], X, lt, 0x8E);
          e = __builtin_amdgcn_bitop3_b32(B[b], X, e, 0x82);
        }
        m[(k * NC + q) * 64u + lane] = lt;
        // the class's tied sites to the wave's list, one a lane at a time
        if (!valid) e = 0u;
        const uint32_t id = (k << 14) | (q << 11) | lane;
#pragma unroll 1
        for (uint64_t more = __ballot(e != 0u); more; more = __ballot(e != 0u)) {
          if (e) {
            const uint32_t at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(more >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)more, 0u));
            list[at] = ((uint32_t)__builtin_ctz(e) << 6) | id;
            e &= e - 1u;
          }
          n += (uint32_t)__popcll(more);
          if (n >= 64u) draw(n - 64u);
        }
      }
    }
    draw(0u);
  };
  // T = 16: tiles of a row of them take the same half of the blocks, so a wave
  // within one draws only that half (16 of 310 instructions a word)
  const uint64_t odd = __ballot(((j0 >> 3) & 1u) != 0u), all = __ballot(true);
  auto form = [&](uint32_t h0, uint32_t nh, uint32_t* m, uint32_t k0, uint32_t dk) __attribute__((always_inline)) {
    if constexpr (T == 16) {
      if (odd == 0u) return form_half(std::integral_constant<int, 0>(), h0, nh, m, k0, dk);
      if (odd == all) return form_half(std::integral_constant<int, 1>(), h0, nh, m, k0, dk);
    }
    form_half(std::integral_constant<int, 2>(), h0, nh, m, k0, dk);
  };

  // ---- one pass of the first wave ----
  uint32_t A[2][NC];  // masks by colour, loaded a pass ahead
  auto fetch = [&](const uint32_t* m, uint32_t k, auto C) {
    constexpr uint32_t c = decltype(C)::value;
#pragma unroll
    for (uint32_t q = 0; q < NC; ++q) A[c][q] = m[(k * NC + q) * 64u + lane];
  };
  auto pass = [&](const uint32_t* m, uint32_t k, uint32_t last, auto C) {
    constexpr uint32_t c = decltype(C)::value;
    const uint32_t* const oth = col + (1 - c) * GR::CW;
    const uint32_t o = ow[c], ct = ow[1 - c];
    const uint32_t before = oth[i], after = oth[2 + i];
    uint32_t fz = 0u, bz = 0u;
    if (D == 3) {
      fz = oth[1 + (int)i - (int)TL::Words];
      bz = oth[1 + i + TL::Words];
    }
    if (k < last) fetch(m, k + 1u, std::integral_constant<uint32_t, 1u - c>());
    const uint32_t up = TL::above(before, ct), dn = TL::below(ct, after);
    const uint32_t next = ((ct >> 1) & ~TL::Last) | rh[1 - c];   // site + 1 in its row
    const uint32_t prev = ((ct << 1) & ~TL::First) | lh[1 - c];  // site - 1
    const uint32_t pm = TL::ahead((c + Y + Zg) & 1u);
    const uint32_t nxp = sel3(pm, next, ct), nxm = sel3(pm, ct, prev);
    // Metropolis: unsatisfied bonds (satisfied ones when J0 < 0); heat bath: up neighbours
    const uint32_t f = o ^ a.invert;
    const uint32_t u[6] = {HB ? ~nxp : f ^ nxp, HB ? ~nxm : f ^ nxm, HB ? ~dn : f ^ dn,
                           HB ? ~up : f ^ up,   HB ? ~bz : f ^ bz,   HB ? ~fz : f ^ fz};
    uint32_t k0, k1, k2;
    count_planes<D>(u, k0, k1, k2);
    const uint32_t* M = A[c];
    uint32_t nw;
    if constexpr (HB) {
      const uint32_t lo4 = sel3(k1, sel3(k0, M[3], M[2]), sel3(k0, M[1], M[0]));
      if constexpr (D == 2) nw = ~sel3(k2, M[4], lo4);
      else nw = ~sel3(k2, sel3(k1, M[6], sel3(k0, M[5], M[4])), lo4);
    } else if constexpr (D == 2) {
      nw = o ^ (k1 | k2 | sel3(k0, M[1], M[0]));  // classes 0 and 1 can refuse
    } else {
      nw = o ^ (k2 | (k1 & k0) | sel3(k1, M[2], sel3(k0, M[1], M[0])));
    }
    ow[c] = nw;
    col[c * GR::CW + 1 + i] = nw;
    wave_sync();
  };
  auto passes = [&](const uint32_t* m, uint32_t nh) {
    using C0 = std::integral_constant<uint32_t, 0>;
    using C1 = std::integral_constant<uint32_t, 1>;
    fetch(m, 0u, C0());
#pragma unroll 1
    for (uint32_t k = 0; k < 2u * nh; k += 2u) {
      pass(m, k, 2u * nh - 1u, C0());
      pass(m, k + 1u, 2u * nh - 1u, C1());
    }
  };

  // the first chunk's masks by all waves, the next ones' by all but the first
  uint32_t buf = 0u;
#pragma unroll 1
  for (uint32_t h = 0, hn = 0; h < a.hits;) {
    if ((wave != 0u || hn == 0u) && hn < a.hits)
      form(hn, min(a.chunk, a.hits - hn), masks + buf, hn == 0u ? wave : wave - 1u,
           hn == 0u ? waves : waves - 1u);
    if (hn != 0u) {
      if (wave == 0u) passes(masks + buf_words - buf, min(a.chunk, a.hits - h));
      h += a.chunk;
    }
    hn += a.chunk;
    buf = buf_words - buf;
    __syncthreads();
  }

  // ---- the tiles go back as +-1 bytes ----
  if (wave == 0u && valid) {
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c)
#pragma unroll
      for (uint32_t r = 0; r < TL::NR; ++r)
        TL::store(a.s + c * Nh + ((uint64_t)Zg * L + Y + r) * R + x0, ow[c] >> (TL::RB * r));
  }
}

bool tile_ahead_supported(const Geom& g, uint32_t T) {
  return (T == 16 || (g.d == 2 && (T == 32 || T == 64))) && (uint32_t)g.L % T == 0 &&
         ((uint32_t)g.L / T) % 2 == 0;
}

// Waves of a workgroup, 0: the kernels of tiles.hip, which form the masks in the
// passes, are faster.  More waves form masks faster and hold more SIMD slots of
// one workgroup's passes idle, and with few hits have nothing to do; with 64 words
// a workgroup, n workgroups in a launch (us a sweep of k = 100 by waves 4 / 8 / 12):
// Metropolis 2D T = 16 n = 128 126 / 86 / 81, n = 1013 294 / 265 / 268, n = 2048 483 /
// 471 / 502, n = 8192 1678 / 1816 / 1946; k = 4 n = 1013 26 / 30 / 33, n = 2048 37 / 40 / 47.
// The heat bath has 2 d + 1 classes with a mask each, which is more work than the
// compare of each site's own class in the pass (`in`): T = 16 n = 128 242 / 167 / 142,
// in 477; n = 512 317 / 232 / 212, in 486; n = 1013 435 / 412 / 410, in 491; n = 2048
// 739 / 736 / 773, in 710; 3D T = 16 n = 864 497 / 489 / 483, in 555; n = 2048 923 / 881 /
// 928, in 788.
// One wave of a workgroup stages and stores its tiles, where a 256-lane group in
// the passes does by four waves, in 3D with four tiles a row: with few hits and a
// full chip that is most of the time, and the masks ahead win from `least` hits on (us
// a sweep, in the passes / ahead): Metropolis 2D T = 16 n = 2048 k = 1 26 / 30, k = 2 33 /
// 31; n = 8192 k = 1 62 / 85, k = 3 89 / 93, k = 4 108 / 102; T = 32 n = 2048 k = 2 31 / 34, k =
// 4 41 / 40; T = 64 n = 4608 k = 3 64 / 71, k = 4 73 / 68; 3D T = 16 n = 2048 k = 1 42 / 106, k =
// 8 86 / 105, k = 12 112 / 107; n = 6912 k = 12 255 / 272, k = 16 322 / 316, k = 100 1746 / 1684;
// above, at any k in the passes (n = 10976 k = 16 465 / 485, k = 100 2604 / 2625; n = 16384 1211 /
// 1289 at k = 32, 3666 / 3852 at k = 100).
uint32_t tile_ahead_waves(const Geom& g, uint32_t T, bool heatbath, uint32_t hits) {
  if (!tile_ahead_supported(g, T)) return 0u;
  const uint64_t words = (uint64_t)g.Nh / 32 / 2;  // of the tiles of one colour
  const uint64_t n = (words + 63) / 64;
  if (n <= 512) return 12u;
  const uint32_t never = ~0u;
  uint32_t least;
  if (heatbath)
    least = n > 1700 ? never : g.d == 3 ? (n <= 896 ? 2 : 6) : T == 64 && n <= 1200 ? 1 : 2;
  else if (g.d == 3)
    least = n <= 1400 ? 2 : n <= 6000 ? 12 : n <= 9000 ? 16 : never;
  else if (T == 16)
    least = n <= 768 ? 1 : n <= 3500 ? 2 : n <= 7000 ? 3 : 4;
  else if (T == 32)
    least = n <= 768 ? 1 : n <= 1500 ? 2 : n <= 7000 ? 4 : 6;
  else
    least = n <= 1500 ? 1 : n <= 2300 ? 2 : n <= 3500 ? 3 : 4;
  if (hits < least) return 0u;
  if (heatbath) return n > 896 && (g.d == 3 || hits >= 8) ? 8u : hits < (g.d == 3 ? 32u : 8u) ? 4u : 12u;
  return n > 3072 || hits < (g.d == 3 && n <= 1400 ? 12u : 8u) ? 4u : 8u;
}

template <int D, uint32_t T>
static hipError_t launch_tile_ahead(const IsingLaunch& a, bool hb, uint32_t hits, int8_t* spins,
                                    uint32_t t, uint32_t tc, uint32_t waves, hipStream_t st) {
  using GR = Group<D, T>;
  TileAheadArgs x;
  x.g = a.g;
  x.key = a.key;
  // Metropolis: with J0 < 0 the classes that can refuse are those of many
  // unsatisfied bonds; counting satisfied ones instead makes them 0 .. d - 1
  uint32_t al0 = 0;
  for (int k = 0; k < D; ++k) al0 |= ((a.tab.al_lo >> (8 * k)) & 0xFFu) != 0xFFu ? 1u : 0u;
  const bool flip = !hb && al0 == 0u;
  x.invert = flip ? ~0u : 0u;
  const uint32_t nc = hb ? 2 * D + 1 : D;
  for (uint32_t q = 0; q < 7; ++q) x.th[q] = x.frac[q] = 0u;
  for (uint32_t q = 0; q < nc; ++q) {
    const uint32_t k = flip ? 2 * D - q : q;
    x.th[q] = ((k < 4 ? a.tab.th_lo : a.tab.th_hi) >> (8 * (k & 3))) & 0xFFu;
    x.frac[q] = a.tab.frac[k];
  }
  const uint32_t nt = (uint32_t)a.g.L / T;
  x.ntiles = (D == 3 ? nt * nt * nt : nt * nt) / 2;
  x.hits = hits;
  x.t = t;
  x.tc = tc;
  x.s = spins;
  const uint32_t groups = (x.ntiles + GR::Tiles - 1) / GR::Tiles;
  // eight hits' masks of two buffers: 16 KiB in 2D, 24 in 3D (heat bath: half
  // the hits, as many bytes)
  x.chunk = std::min(hits, hb ? 4u : 8u);
  const size_t lds = 4 * ((size_t)GR::Tiles * 2 * GR::CW + (size_t)4 * x.chunk * nc * 64u + waves * 128u);
  if (hb) hipLaunchKernelGGL((tile_ahead_kernel<D, T, true>), dim3(groups), dim3(64u * waves), lds, st, x);
  else hipLaunchKernelGGL((tile_ahead_kernel<D, T, false>), dim3(groups), dim3(64u * waves), lds, st, x);
  return hipGetLastError();
}

hipError_t launch_tile_ahead_pass(const IsingLaunch& a, bool heatbath, uint32_t T, uint32_t hits,
                                  int8_t* spins, uint32_t t, uint32_t tc, hipStream_t st, uint32_t waves) {
  if (a.g.d == 3) return launch_tile_ahead<3, 16>(a, heatbath, hits, spins, t, tc, waves, st);
  return T == 16 ? launch_tile_ahead<2, 16>(a, heatbath, hits, spins, t, tc, waves, st)
       : T == 32 ? launch_tile_ahead<2, 32>(a, heatbath, hits, spins, t, tc, waves, st)
                 : launch_tile_ahead<2, 64>(a, heatbath, hits, spins, t, tc, waves, st);
}

}  // namespace smc
