// batch.hip -- many independent Ising lattices of uneven size, temperature and
// disorder realisation in one persistent launch (the paper's trivial
// parallelism over disorder realisations on top of the checkerboard
// decomposition, Sec. 2).
//
// One workgroup owns one lattice: it stages both colour planes (L^d bytes,
// at most 64 KiB) in LDS, runs every sweep of the call there -- colour 0,
// barrier, colour 1, barrier -- and writes the planes back once, so HBM is
// touched only at the start and the end.  Couplings stay in global memory
// (they are re-read from L2 / Infinity Cache).  Lattice r uses replica r in
// the Philox counter, so each lattice reproduces the single-lattice chain
// with that replica bit for bit.  A lane walks groups of 16 consecutive
// same-colour sites (one Philox block of prefix bytes per group); the
// decision per site is the integer threshold test of the single-lattice
// kernels with its exact tie refinement.  Lattices whose plane rows are whole
// 4-site words (L/2 % 4 == 0) take the decision four sites per 32-bit op
// (rows of whole 2-site pairs, L/2 even, two sites per op):
// neighbour words from LDS (the in-row neighbours as the centre word shifted
// by one byte), unsatisfied-bond counts per byte, and the byte-wise threshold
// compare of the single-lattice kernels.  The index arithmetic of a word
// (its row, the periodic wraps of its neighbours) is formed once per call when
// each lane holds one group, and once per group when a group is a whole part
// of one plane row (L/2 % 16 == 0).  With MEASURE the workgroup also
// reduces E and M of its state from LDS after every `every` sweeps (record m
// of the call at obs[m * n_lattices + lattice]; with no sweeps, one record of
// the current state).
#include <algorithm>
#include <type_traits>

#include "chunk.hpp"
#include "packed.hpp"
#include "reduce.hpp"

namespace smc {

constexpr uint32_t kBatchTieSlots = 4;  // deferred ties per lane before a flush

// ---------------------------------------------------------------------------
// Packed path (any even edge whose words number at most two per lane): the
// lattice sits in LDS at one bit per site -- word w of colour c holds sites
// 32 w .. 32 w + 31 of that plane (the last word may be partly filled), the
// two colours' words side by side (byte 12 (w + 1) + 4 c, a zero pad pair at
// each end) -- with the signs of each site's 2d bonds as 2d words aligned with
// it (the -mu bonds by the gather of the -mu neighbours' spins, run on the
// coupling planes when the lattice is staged).  A lane owns words w = lane and
// w = lane + T of both colours for the whole call.  The neighbour words of the
// other colour come from funnel shifts of LDS words, with the row ends, the
// row parity and the periodic wraps as per-word masks: in-row x +- 1, y +- 1 a
// shift by R = L / 2 sites, z +- 1 a shift by L^2 / 2 sites (a whole word when
// L % 8 == 0).  Counts, the decision with its prefix bit planes and exact
// ties, and the random bytes per site are those of the packed single-lattice
// kernel, so every lattice keeps the chain of its replica bit for bit.
//
// A lattice of at most 64 words a colour (2D L <= 64, 3D L <= 16) is one
// wave's (WAVE): several share a workgroup (batch_split) and none waits at a
// barrier.  With a workgroup each, three of its four waves idled and held
// their registers: 2048 spin-glass samples of L = 8 .. 32, 100 sweeps recorded
// every 10: 957 -> 738 us, of which 85 us were the couplings' bit-by-bit
// staging.  Edges that are no multiple of four, and 2D, took the byte path:
// 512 samples, 100 sweeps: 3D L = 10 1103 -> 159 us, L = 30 5692 -> 579, 2D
// L = 100 1343 -> 262, L = 128 640 -> 273.
// ---------------------------------------------------------------------------
constexpr uint32_t kPackedBatchWordsPerLane = 2;
constexpr uint32_t kWaveWords = 64;  // words a colour of a lattice that one wave takes
constexpr uint32_t kTinyWords = 8;   // of a tiny one (batch_split)
// LDS strides of a word's spin pair (colour 0, colour 1, unused) and of its
// 4 d bond-sign words (+ one unused): an odd number of dwords, so that 32
// lanes reading consecutive words touch 32 different banks.
constexpr uint32_t kPkSpin = 12;
__host__ __device__ constexpr uint32_t pk_bond(int d) { return 16u * d + 4u; }

__host__ __device__ inline uint32_t batch_words(int d, uint32_t L) {
  return (L * L * (d == 3 ? L : 1u) / 2u + 31u) / 32u;
}

__host__ __device__ inline bool batch_packed_ok(int d, uint32_t L, uint32_t threads) {
  return (d == 2 || L <= 40u) && batch_words(d, L) <= kPackedBatchWordsPerLane * threads;
}

bool batch_lattice_wave(int d, uint32_t L) { return batch_words(d, L) <= kWaveWords; }

// LDS bytes of the packed path for `words` words a colour: the spin pairs with
// their pads and the aligned bond-sign words (+-1 couplings).  (A lane's tied
// words -- at most one per word it owns -- wait in registers until the end of
// the half-sweep.)
__host__ __device__ constexpr uint32_t batch_packed_lds_bytes(int d, uint32_t words, bool pm) {
  return (kPkSpin * (words + 2u) + 15u) / 16u * 16u + (pm ? (pk_bond(d) * words + 15u) / 16u * 16u : 0u);
}

template <int D>
struct PackedWord {  // per-call constants of one word of the lane
  uint32_t E, S, Pm0, Ymp, Ymm;  // row end / start, rows of colour-0 parity 1, y = L-1 / y = 0
  uint32_t Zmp, Zmm;             // sites at z = L-1 / z = 0 (used when z-planes split words)
  uint32_t ayp, aym;             // LDS byte addresses (colour 0) of the y wrap sources
  uint32_t azp, azm;             // z +- 1 sources (low words of the funnels); 2D: y +- 1
  uint32_t azpw, azmw;           // z wrap sources (z-planes that split words); 2D: the x wraps
  uint32_t a0;                   // LDS byte address of word w, colour 0
  uint32_t aj;                   // LDS byte address of its bond-sign words
  uint32_t ok;                   // its sites that exist (0: the lane has no such word)
};

// Funnel shifts of the wrap and z gathers (site offset mod 32).  LR = L^2/2
// sites per z-plane of one colour (2D: of the lattice); when LR % 32 == 0 the
// z neighbours are whole words (zs == 0).
struct PackedZ {
  uint32_t ysw, ysmw;     // y wraps: R - LR, LR - R
  uint32_t zs, zsw;       // +z: LR, LR (1 - L)
  uint32_t zsm, zsmw;     // -z: -LR, LR (L - 1)
};

// Neighbour words (+x, -x, +y, -y, +z, -z) of word `pw` of colour C from the
// other colour's words.  In 3D a row is at most 20 sites, so its wrap and the
// rows around it lie in the words beside the own one; in 2D they have sources
// of their own.
template <int D, uint32_t C>
__device__ __forceinline__ void packed_neighbours(const unsigned char* lds, const PackedWord<D>& pw,
                                                  uint32_t R, const PackedZ& pz, uint32_t nb[6]) {
  constexpr uint32_t O = 4u * (1u - C);  // the other colour's word in a pair
  auto ldw = [&](uint32_t a) -> uint32_t { return *reinterpret_cast<const uint32_t*>(lds + a); };
  auto fun = [&](uint32_t a, uint32_t sh) -> uint32_t {
    return __builtin_amdgcn_alignbit(ldw(a + kPkSpin + O), ldw(a + O), sh);
  };
  const uint32_t wp = ldw(pw.a0 - kPkSpin + O), wc = ldw(pw.a0 + O), wn = ldw(pw.a0 + kPkSpin + O);
  const uint32_t next = __builtin_amdgcn_alignbit(wn, wc, 1u);        // site + 1
  const uint32_t prev = __builtin_amdgcn_alignbit(wc, wp, 31u);       // site - 1
  // site - (R - 1): row start; site + (R - 1): row end
  const uint32_t wst = D == 3 ? __builtin_amdgcn_alignbit(wc, wp, 33u - R) : fun(pw.azpw, (1u - R) & 31u);
  const uint32_t wen = D == 3 ? __builtin_amdgcn_alignbit(wn, wc, R - 1u) : fun(pw.azmw, (R - 1u) & 31u);
  // row parity of colour C: p = 1 rows take x + 1 = in-row index + 1
  const uint32_t Pm = C == 0 ? pw.Pm0 : ~pw.Pm0;
  nb[0] = __builtin_amdgcn_bitop3_b32(Pm, __builtin_amdgcn_bitop3_b32(pw.E, wst, next, 0xCA), wc, 0xCA);
  nb[1] = __builtin_amdgcn_bitop3_b32(Pm, wc, __builtin_amdgcn_bitop3_b32(pw.S, wen, prev, 0xCA), 0xCA);
  const uint32_t yp = D == 3 ? __builtin_amdgcn_alignbit(wn, wc, R) : fun(pw.azp, R & 31u);
  nb[2] = __builtin_amdgcn_bitop3_b32(pw.Ymp, fun(pw.ayp, pz.ysw), yp, 0xCA);
  const uint32_t ym = D == 3 ? __builtin_amdgcn_alignbit(wc, wp, 32u - R) : fun(pw.azm, (0u - R) & 31u);
  nb[3] = __builtin_amdgcn_bitop3_b32(pw.Ymm, fun(pw.aym, pz.ysmw), ym, 0xCA);
  nb[4] = nb[5] = 0u;
  if constexpr (D == 3) {
    if (pz.zs == 0u) {  // z-planes hold whole words
      nb[4] = ldw(pw.azp + O);
      nb[5] = ldw(pw.azm + O);
    } else {
      nb[4] = __builtin_amdgcn_bitop3_b32(pw.Zmp, fun(pw.azpw, pz.zsw), fun(pw.azp, pz.zs), 0xCA);
      nb[5] = __builtin_amdgcn_bitop3_b32(pw.Zmm, fun(pw.azmw, pz.zsmw), fun(pw.azm, pz.zsm), 0xCA);
    }
  }
}

// Count planes of word `pw` of colour C: unsatisfied bonds (spin bits differ,
// xor the bond's sign bit).
template <int D, uint32_t C, bool PM>
__device__ __forceinline__ uint32_t packed_word_counts(const unsigned char* lds, const PackedWord<D>& pw,
                                                       uint32_t R, const PackedZ& pz, uint32_t& k0,
                                                       uint32_t& k1, uint32_t& k2) {
  const uint32_t o = *reinterpret_cast<const uint32_t*>(lds + pw.a0 + 4u * C);
  uint32_t nb[6];
  packed_neighbours<D, C>(lds, pw, R, pz, nb);
  uint32_t u[6];
#pragma unroll
  for (int m = 0; m < 2 * D; ++m) {
    const uint32_t js = PM ? *reinterpret_cast<const uint32_t*>(lds + pw.aj + 4u * (2u * m + C)) : 0u;
    u[m] = o ^ nb[m] ^ js;
  }
  count_planes<D>(u, k0, k1, k2);
  return o;
}

// WPL words a lane; WAVE: the lattice is the wave's, `lds` its part.
template <int D, bool PM, bool MEASURE, int WPL, bool WAVE>
__device__ __forceinline__ void batch_packed_lattice(unsigned char* lds, const BatchDesc* dp, uint32_t li,
                                     const RngKey& key0, int8_t* gs, const int8_t* gJ,
                                     uint32_t L, uint32_t R, uint32_t Nh, uint32_t replica,
                                     const TabRegs& tab, uint32_t t0, uint32_t n_sweeps,
                                     uint32_t every, uint32_t n_lattices, ObsOut* obs) {
  const uint32_t T = WAVE ? 64u : blockDim.x, q = WAVE ? __lane_id() : threadIdx.x;
  const uint32_t Wp = (Nh + 31u) / 32u, tail = 32u * Wp - Nh;
  const uint32_t LR = L * R;  // sites of a z-plane of one colour
  constexpr uint32_t SB = 0;
  const uint32_t JB = (kPkSpin * (Wp + 2u) + 15u) / 16u * 16u;
  const RngKey key{key0.k0, key0.k1, replica};
  auto sync = [&]() {
    if constexpr (WAVE) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  auto word_sites = [&](uint32_t w) -> uint32_t { return w + 1u == Wp ? 32u - tail : 32u; };
  // sign bits of a pair of int8 planes into the spin pairs
  auto stage = [&](const int8_t* planes) {
#pragma unroll 1
    for (uint32_t i = q; i < 2u * Wp; i += T) {
      const uint32_t c = i & 1u, w = i >> 1;
      *reinterpret_cast<uint32_t*>(lds + SB + kPkSpin * (w + 1u) + 4u * c) =
          load_signs(planes + (size_t)c * Nh + 32u * w, word_sites(w));
    }
  };
  if (q < 2u) {
    *reinterpret_cast<uint32_t*>(lds + SB + 4u * q) = 0u;
    *reinterpret_cast<uint32_t*>(lds + SB + kPkSpin * (Wp + 1u) + 4u * q) = 0u;
  }
  // funnel shifts of the wrap and z gathers
  PackedZ pz;
  pz.ysw = (R - LR) & 31u;
  pz.ysmw = (LR - R) & 31u;
  pz.zs = LR & 31u;
  pz.zsw = (uint32_t)((int32_t)LR * (1 - (int32_t)L)) & 31u;
  pz.zsm = (0u - LR) & 31u;
  pz.zsmw = (LR * (L - 1u)) & 31u;
  // the lane's words: row masks, wrap and z sources
  PackedWord<D> pw[WPL];
#pragma unroll
  for (uint32_t p = 0; p < (uint32_t)WPL; ++p) {
    const uint32_t w = q + p * T;
    PackedWord<D>& x = pw[p];
    const bool valid = w < Wp;
    const uint32_t wv = valid ? w : 0u, nv = word_sites(wv);
    x.ok = valid ? ~0u >> (32u - nv) : 0u;
    x.E = x.S = x.Pm0 = x.Ymp = x.Ymm = x.Zmp = x.Zmm = 0;
    const uint32_t j0 = 32u * wv;
    uint32_t r = j0 / R, jx = j0 - r * R;
    uint32_t z = D == 3 ? r / L : 0u, y = r - z * L;
#pragma unroll 1
    for (uint32_t b = 0; b < nv;) {  // the word's pieces of rows
      const uint32_t len = min(R - jx, 32u - b);
      const uint32_t seg = (len == 32u ? ~0u : (1u << len) - 1u) << b;
      if (jx + len == R) x.E |= 1u << (b + len - 1u);
      if (jx == 0u) x.S |= 1u << b;
      if ((y + z) & 1u) x.Pm0 |= seg;
      if (y + 1u == L) x.Ymp |= seg;
      if (y == 0u) x.Ymm |= seg;
      if (z + 1u == L) x.Zmp |= seg;
      if (z == 0u) x.Zmm |= seg;
      b += len;
      jx = 0u;
      ++y;
      if (D == 3 && y == L) {
        y = 0u;
        ++z;
      }
    }
    // Sources: bit i of a gather at site offset off is site 32 w + i + off,
    // from the funnel of words w + floor(off / 32) and the next; that low word
    // is clamped to the pads (-1 .. Wp - 1) where the word has no site that
    // uses the gather.  y wraps: rows y = L - 1 take off = R - LR, rows y = 0
    // off = LR - R; z (when z-planes split words): +-LR, and the wrapped
    // LR (1 - L) / LR (L - 1) for the last / first z-plane.
    auto lo = [&](int32_t off) -> uint32_t {  // LDS byte address of the clamped low word
      const int32_t i = (int32_t)wv + (off >> 5);
      return SB + kPkSpin * (uint32_t)((i < -1 ? -1 : (i > (int32_t)Wp - 1 ? (int32_t)Wp - 1 : i)) + 1);
    };
    const int32_t lr = (int32_t)LR, l = (int32_t)L, rr = (int32_t)R;
    x.ayp = lo(rr - lr);
    x.aym = lo(lr - rr);
    if constexpr (D == 2) {
      x.azp = lo(rr);
      x.azm = lo(-rr);
      x.azpw = lo(1 - rr);
      x.azmw = lo(rr - 1);
    } else if (pz.zs == 0u) {  // z-planes hold whole words: the z neighbours are words
      const uint32_t zw = LR / 32u;  // words per z-plane
      const uint32_t izp = wv + zw >= Wp ? wv + zw - Wp : wv + zw;
      const uint32_t izm = wv < zw ? wv + Wp - zw : wv - zw;
      x.azp = SB + kPkSpin * (izp + 1u);
      x.azm = SB + kPkSpin * (izm + 1u);
      x.azpw = x.azmw = SB;
    } else {
      x.azp = lo(lr);
      x.azpw = lo(lr * (1 - l));
      x.azm = lo(-lr);
      x.azmw = lo(lr * (l - 1));
    }
    x.a0 = SB + kPkSpin * (wv + 1u);
    x.aj = JB + pk_bond(D) * wv;
  }
  if (PM) {
    // J[mu] in the spin pairs: a word's +mu bonds are its own words, its -mu
    // bonds those of its -mu neighbours
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
      stage(gJ + (size_t)(2 * mu) * Nh);
      sync();
#pragma unroll
      for (uint32_t p = 0; p < (uint32_t)WPL; ++p) {
        if (!pw[p].ok) continue;
        uint32_t n0[6], n1[6];
        packed_neighbours<D, 0>(lds, pw[p], R, pz, n0);
        packed_neighbours<D, 1>(lds, pw[p], R, pz, n1);
        uint32_t* j = reinterpret_cast<uint32_t*>(lds + pw[p].aj) + 4 * mu;  // (2 (2 mu + s) + c)
        j[0] = *reinterpret_cast<const uint32_t*>(lds + pw[p].a0);
        j[1] = *reinterpret_cast<const uint32_t*>(lds + pw[p].a0 + 4u);
        j[2] = n0[2 * mu + 1];
        j[3] = n1[2 * mu + 1];
      }
      sync();
    }
  }
  stage(gs);
  // thresholds of this lattice: the fast decision when only classes k < d can
  // refuse (every class k >= d always accepts)
  bool fast = true;
#pragma unroll
  for (int k = D; k <= 2 * D; ++k) fast = fast && table_byte(tab.al_lo, tab.al_hi, k) == 0xFFu;
  FastTab ft = fast_tab<D>(tab);
  sync();

  // a word's exact ties wait in registers (tie mask and count planes) until
  // the lane's words of the colour are stored, then take their refinement
  // draws; a lane writes only its own words, so the fix-up is race-free
  auto resolve = [&](uint32_t c, uint32_t t, uint32_t w, uint32_t a, const uint4& en) {
    uint32_t m = en.x, flips = 0;
    while (m) {
      const uint32_t b = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t k = ((en.y >> b) & 1u) | (((en.z >> b) & 1u) << 1) | (((en.w >> b) & 1u) << 2);
      const Rand4 rr = philox(32u * w + b, t, replica, tag(c, kIsingRefine), key.k0, key.k1);
      if ((rr.w[0] & 0xFFFFFFu) < frac_sel(tab.fr, k)) flips |= 1u << b;
    }
    *reinterpret_cast<uint32_t*>(lds + a + 4u * c) ^= flips;
  };
  auto half = [&](auto cc, uint32_t t) {
    constexpr uint32_t C = decltype(cc)::value;
    uint4 tie[WPL];
#pragma unroll
    for (uint32_t p = 0; p < (uint32_t)WPL; ++p) {
      tie[p] = make_uint4(0u, 0u, 0u, 0u);
      if (!pw[p].ok) continue;
      uint32_t k0, k1, k2;
      const uint32_t o = packed_word_counts<D, C, PM>(lds, pw[p], R, pz, k0, k1, k2);
      const uint32_t w = q + p * T;
      uint32_t ties;
      const uint32_t flip = fast ? packed_decide_fast<D>(ft, key, t, C, w, k0, k1, k2, ties)
                                 : packed_decide<D>(tab, key, t, C, w, k0, k1, k2, ties);
      *reinterpret_cast<uint32_t*>(lds + pw[p].a0 + 4u * C) = o ^ flip;
      tie[p] = make_uint4(ties & pw[p].ok, k0, k1, k2);
    }
#pragma unroll
    for (uint32_t p = 0; p < (uint32_t)WPL; ++p)
      if (tie[p].x) resolve(C, t, q + p * T, pw[p].a0, tie[p]);
    sync();
  };
  auto measure = [&](uint32_t slot, int64_t sweep) {
    int64_t Esum = 0, Msum = 0;
#pragma unroll
    for (uint32_t p = 0; p < (uint32_t)WPL; ++p) {
      const uint32_t ok = pw[p].ok;
      if (!ok) continue;
      uint32_t k0, k1, k2;
      const uint32_t o1 = packed_word_counts<D, 1, PM>(lds, pw[p], R, pz, k0, k1, k2);
      const uint32_t o0 = *reinterpret_cast<const uint32_t*>(lds + pw[p].a0);
      const int32_t ks = __builtin_popcount(k0 & ok) + 2 * __builtin_popcount(k1 & ok) +
                         4 * __builtin_popcount(k2 & ok);
      const int32_t nv = __builtin_popcount(ok);
      Esum += 2 * (int64_t)ks - nv * 2 * D;
      Msum += 2 * nv - 2 * (int64_t)(__builtin_popcount(o1 & ok) + __builtin_popcount(o0 & ok));
    }
    __shared__ Partial part[1];
    if constexpr (WAVE) {
      Esum = wave_sum(Esum);
      Msum = wave_sum(Msum);
    } else {
      block_partial_int(Esum, Msum, part, 0);
    }
    if (q == 0) {
      if constexpr (!WAVE) {
        Esum = part[0].Ei;
        Msum = part[0].Mi;
      }
      ObsOut o;
      o.E_int = Esum;
      o.M_int = Msum;
      o.E = (double)Esum * dp->J0;
      o.M[0] = (double)Msum;
      o.M[1] = 0.0;
      o.M[2] = 0.0;
      o.absM = fabs((double)Msum);
      o.sweep = sweep;
      obs[(uint64_t)slot * n_lattices + li] = o;
    }
  };
  // records are counted down: a remainder a sweep is 30 instructions and scalar registers
  // that the loop lacks (us, 100 sweeps of 1024 lattices: 3D L = 12 185 / 177, L = 16 176 / 169)
  uint32_t slot = 0, left = every;
  for (uint32_t sw = 0; sw < n_sweeps; ++sw) {
    const uint32_t t = t0 + sw;
    half(std::integral_constant<uint32_t, 0>(), t);
    half(std::integral_constant<uint32_t, 1>(), t);
    if (MEASURE && --left == 0) {
      measure(slot++, (int64_t)t + 1);
      left = every;
    }
  }
  if (MEASURE && n_sweeps == 0) measure(0, (int64_t)t0);
  // the lane's words of both planes back as +-1 bytes
#pragma unroll
  for (uint32_t p = 0; p < (uint32_t)WPL; ++p) {
    if (!pw[p].ok) continue;
    const uint32_t w = q + p * T;
#pragma unroll 1
    for (uint32_t c = 0; c < 2u; ++c)
      store_signs(gs + (size_t)c * Nh + 32u * w,
                  *reinterpret_cast<const uint32_t*>(lds + pw[p].a0 + 4u * c), word_sites(w));
  }
}

// (`split` comes last: next to the counts that the sweeps' loop keeps it was loaded with
// them, and the loop then lacked scalar registers; see the records' count there)
template <int D, bool PM, bool MEASURE>
__global__ __launch_bounds__(1024) void batch_kernel(const BatchDesc* __restrict__ descs,
                                                    const uint32_t* __restrict__ order,
                                                    const RngKey key, int8_t* __restrict__ spins,
                                                    const int8_t* __restrict__ J,
                                                    const uint32_t t0, const uint32_t n_sweeps,
                                                    const uint32_t every, const uint32_t n_lattices,
                                                    ObsOut* __restrict__ obs,
                                                    const BatchSplit split) {
  extern __shared__ uint32_t lat_words[];  // [2][Nh] spins of this lattice
  int8_t* const lat = reinterpret_cast<int8_t*>(lat_words);
  // workgroups from n_single on: a lattice a wave of the first `per` (no wave waits
  // for another)
  const bool by_wave = blockIdx.x >= split.n_single;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t at = blockIdx.x;
  if (by_wave) {
    const uint32_t b = blockIdx.x - split.n_single;
    const bool full = b < split.g_full;
    const uint32_t per = full ? split.per_full : split.per_tiny;
    at = split.n_single + wave + (full ? b * per : split.g_full * split.per_full + (b - split.g_full) * per);
    if (wave >= per) return;
  }
  if (at >= n_lattices) return;
  const uint32_t li = __builtin_amdgcn_readfirstlane(order[at]);
  const BatchDesc* dp = descs + li;
  const uint32_t L = __builtin_amdgcn_readfirstlane(dp->L);
  const uint32_t R = __builtin_amdgcn_readfirstlane(dp->R);
  const uint32_t Nh = __builtin_amdgcn_readfirstlane(dp->Nh);
  FastDiv divR, divL;
  divR.d = R;
  divR.m = (uint32_t)__builtin_amdgcn_readfirstlane(dp->divR_m);
  divR.s = (uint32_t)__builtin_amdgcn_readfirstlane(dp->divR_s);
  divL.d = L;
  divL.m = (uint32_t)__builtin_amdgcn_readfirstlane(dp->divL_m);
  divL.s = (uint32_t)__builtin_amdgcn_readfirstlane(dp->divL_s);
  const uint32_t th_lo = __builtin_amdgcn_readfirstlane(dp->th_lo);
  const uint32_t th_hi = __builtin_amdgcn_readfirstlane(dp->th_hi);
  const uint32_t al_lo = __builtin_amdgcn_readfirstlane(dp->al_lo);
  const uint32_t al_hi = __builtin_amdgcn_readfirstlane(dp->al_hi);
  const uint32_t replica = __builtin_amdgcn_readfirstlane(dp->replica);
  const uint64_t soff = ((uint64_t)__builtin_amdgcn_readfirstlane(dp->spin_off_hi) << 32) |
                        __builtin_amdgcn_readfirstlane(dp->spin_off_lo);
  const uint64_t joff = ((uint64_t)__builtin_amdgcn_readfirstlane(dp->J_off_hi) << 32) |
                        __builtin_amdgcn_readfirstlane(dp->J_off_lo);
  int8_t* gs = spins + soff;
  const int8_t* gJ = J + joff;
  const uint32_t N = 2 * Nh;  // L^d, a multiple of 4 (L even)
  if (__builtin_amdgcn_readfirstlane(dp->packed) && batch_packed_ok(D, L, blockDim.x)) {
    TabRegs tab;
    tab.th_lo = th_lo;
    tab.th_hi = th_hi;
    tab.al_lo = al_lo;
    tab.al_hi = al_hi;
    tab.fr.f0 = __builtin_amdgcn_readfirstlane(dp->frac[0]);
    tab.fr.f1 = __builtin_amdgcn_readfirstlane(dp->frac[1]);
    tab.fr.f2 = __builtin_amdgcn_readfirstlane(dp->frac[2]);
    tab.fr.f3 = __builtin_amdgcn_readfirstlane(dp->frac[3]);
    tab.fr.f4 = __builtin_amdgcn_readfirstlane(dp->frac[4]);
    tab.fr.f5 = __builtin_amdgcn_readfirstlane(dp->frac[5]);
    tab.fr.f6 = __builtin_amdgcn_readfirstlane(dp->frac[6]);
    unsigned char* lds = reinterpret_cast<unsigned char*>(lat_words);
    if (by_wave)
      batch_packed_lattice<D, PM, MEASURE, 1, true>(lds + wave * batch_packed_lds_bytes(D, kWaveWords, PM), dp, li,
                                                    key, gs, gJ, L, R, Nh, replica, tab, t0, n_sweeps, every,
                                                    n_lattices, obs);
    else
      batch_packed_lattice<D, PM, MEASURE, kPackedBatchWordsPerLane, false>(lds, dp, li, key, gs, gJ, L, R, Nh,
                                                                            replica, tab, t0, n_sweeps, every,
                                                                            n_lattices, obs);
    return;
  }

  // Stage both planes into LDS as one byte per site: bit 0 = spin -1, bit
  // 1 + m = coupling of bond m negative (m = +x, -x, +y, -y, +z, -z), so the
  // sweep reads couplings from LDS together with the spins.
  // Row and plane strides (wave-uniform): neighbour rows are the own row's
  // offset plus or minus a stride, with the periodic wrap as a select.
  const uint32_t sYw = (L - 1) * R, sZ = L * R, sZw = (L - 1) * L * R;
  auto nbr = [&](uint32_t c, uint32_t j, uint32_t nbi[6]) {  // in-plane neighbour indices
    const uint32_t r = fdiv(j, divR);
    const uint32_t rowb = r * R;
    const uint32_t jx = j - rowb;
    const uint32_t z = D == 3 ? fdiv(r, divL) : 0u;
    const uint32_t y = r - z * L;
    const uint32_t p = (c + r + z) & 1u;  // (c + y + z) & 1 with L even
    nbi[0] = jx + p == R ? rowb : j + p;
    nbi[1] = jx + p == 0 ? rowb + R - 1 : j + p - 1;
    nbi[2] = y + 1 == L ? j - sYw : j + R;
    nbi[3] = y == 0 ? j + sYw : j - R;
    nbi[4] = nbi[5] = 0;
    if (D == 3) {
      nbi[4] = z + 1 == L ? j - sZw : j + sZ;
      nbi[5] = z == 0 ? j + sZw : j - sZ;
    }
  };
  for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) {
    const uint32_t c = i >= Nh ? 1u : 0u;
    const uint32_t j = i - c * Nh;
    uint32_t v = gs[i] < 0 ? 1u : 0u;
    if (PM) {
      uint32_t nbi[6];
      nbr(c, j, nbi);
      const int8_t* Jo = gJ + (uint64_t)c * Nh;        // J[mu][c] = gJ + (2 mu + c) Nh
      const int8_t* Jn = gJ + (uint64_t)(1 - c) * Nh;  // J[mu][1 - c]
#pragma unroll
      for (int mu = 0; mu < D; ++mu) {
        v |= (Jo[2 * (uint64_t)mu * Nh + j] < 0 ? 1u : 0u) << (1 + 2 * mu);
        v |= (Jn[2 * (uint64_t)mu * Nh + nbi[2 * mu + 1]] < 0 ? 1u : 0u) << (2 + 2 * mu);
      }
    }
    lat[i] = (int8_t)v;
  }
  __syncthreads();

  // One site: k = bonds with J s_i s_nb < 0 from the combined bytes.
  auto site_k = [&](const int8_t* own, const int8_t* oth, uint32_t c, uint32_t j,
                    uint32_t& o) -> uint32_t {
    uint32_t nbi[6];
    nbr(c, j, nbi);
    o = (uint8_t)own[j];
    uint32_t nm = 0;
#pragma unroll
    for (int m = 0; m < 2 * D; ++m) nm |= ((uint32_t)(uint8_t)oth[nbi[m]] & 1u) << m;
    const uint32_t om = (0u - (o & 1u)) & ((1u << (2 * D)) - 1u);
    return __builtin_popcount(nm ^ om ^ (PM ? (o >> 1) : 0u));
  };
  // Four sites j .. j + 3 of one plane row (j % 4 == 0, R % 4 == 0): new
  // word of the own plane, decided by prefix word P; ties (prefix byte equal
  // to the threshold byte of a refusable class) take the site's refinement
  // draw on the spot.
  auto ld = [&](const int8_t* base, uint32_t i) -> uint32_t {
    return *reinterpret_cast<const uint32_t*>(base + i);
  };
  // Unsatisfied bonds per byte of the own word W against its 2d neighbour
  // words: the spin bits differ, xor the bond's sign bit.
  auto count_bytes = [&](uint32_t W, const uint32_t nb[6]) -> uint32_t {
    uint32_t k = 0;
#pragma unroll
    for (int m = 0; m < 2 * D; ++m) {
      uint32_t u = W ^ nb[m];
      if (PM) u ^= W >> (1 + m);
      k += u & kOnes;
    }
    return k;
  };
  // Unsatisfied-bond counts (byte b: site j + b) of a WB-site word of plane c
  // (WB = 4: j % 4 == 0 and R % 4 == 0; WB = 2: j even and R even; the word
  // lies in one plane row).  The in-row neighbours are the centre word
  // shifted by one byte with the adjacent word's edge byte.
  auto counts = [&](auto wb, const int8_t* own, const int8_t* oth, uint32_t c, uint32_t j,
                    uint32_t& W) -> uint32_t {
    constexpr uint32_t WB = decltype(wb)::value;
    auto ldw = [&](const int8_t* base, uint32_t i) -> uint32_t {
      if constexpr (WB == 4) return *reinterpret_cast<const uint32_t*>(base + i);
      else return *reinterpret_cast<const uint16_t*>(base + i);
    };
    const uint32_t r = fdiv(j, divR);
    const uint32_t rowb = r * R;
    const uint32_t jx = j - rowb;
    const uint32_t z = D == 3 ? fdiv(r, divL) : 0u;
    const uint32_t y = r - z * L;
    const uint32_t p = (c + r + z) & 1u;  // (c + y + z) & 1 with L even
    W = ldw(own, j);
    const uint32_t C = ldw(oth, j);
    // p = 1: x+1 is the next word's first byte onwards; p = 0: x-1 ends with
    // the previous word's last byte
    const uint32_t Ej = p ? (jx + WB == R ? rowb : j + WB) : (jx == 0 ? rowb + R - WB : j - WB);
    const uint32_t E = ldw(oth, Ej);
    uint32_t S;
    if constexpr (WB == 4)
      S = p ? __builtin_amdgcn_alignbyte(E, C, 1) : __builtin_amdgcn_alignbyte(C, E, 3);
    else
      S = p ? ((C >> 8) | ((E & 0xFFu) << 8)) : (((C << 8) & 0xFF00u) | (E >> 8));
    uint32_t nb[6];
    nb[0] = p ? S : C;  // +x
    nb[1] = p ? C : S;  // -x
    nb[2] = ldw(oth, y + 1 == L ? j - sYw : j + R);
    nb[3] = ldw(oth, y == 0 ? j + sYw : j - R);
    if (D == 3) {
      nb[4] = ldw(oth, z + 1 == L ? j - sZw : j + sZ);
      nb[5] = ldw(oth, z == 0 ? j + sZw : j - sZ);
    }
    return count_bytes(W, nb);
  };
  // New word for prefix bytes P (byte b: site j + b); `tie` gets bit 7 of
  // each byte whose prefix equals the threshold byte of a refusable class
  // (left unflipped), `kout` the counts.  Only the low WB bytes of the
  // result are meaningful.
  auto decide = [&](auto wb, uint32_t W, uint32_t k, uint32_t P, uint32_t& tie) -> uint32_t {
    constexpr uint32_t WB = decltype(wb)::value;
    const uint32_t Th = __builtin_amdgcn_perm(th_hi, th_lo, k);
    const uint32_t Al = __builtin_amdgcn_perm(al_hi, al_lo, k);
    const uint32_t x = P ^ Th;
    const uint32_t dlow = (P | kHigh) - (Th & ~kHigh);
    const uint32_t ge = (x & P) | (~x & dlow);  // bit 7 of each byte: P >= Th
    const uint32_t rej = __builtin_amdgcn_perm(ge, ge << 8, 0x0B090A08u);
    const uint32_t zb = (x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu;
    tie = ~(zb | x | Al) & (WB == 4 ? kHigh : 0x8080u);
    return W ^ ((~rej | Al) & kOnes);
  };
  auto word = [&](auto wb, const int8_t* own, const int8_t* oth, uint32_t c, uint32_t j,
                  uint32_t P, uint32_t& tie, uint32_t& kout) -> uint32_t {
    uint32_t W;
    const uint32_t k = counts(wb, own, oth, c, j, W);
    kout = k;
    return decide(wb, W, k, P, tie);
  };
  using W4 = std::integral_constant<uint32_t, 4>;
  using W2 = std::integral_constant<uint32_t, 2>;
  // Ties wait in a per-lane LDS queue (entry (site << 3) | class, lane-major)
  // and are resolved by their refinement draws before the colour's barrier:
  // a lane alone writes the sites of its groups, so the late flip is
  // race-free, and a wave pays for the longest queue of its lanes once per
  // half-sweep instead of once per word.
  uint32_t* const tq = lat_words + (N + 15) / 16 * 4 + threadIdx.x;
  uint32_t nq = 0;
  auto flush = [&](int8_t* own, uint32_t c, uint32_t t) {
    for (uint32_t i = 0; i < nq; ++i) {
      const uint32_t e = tq[i * blockDim.x];
      const uint32_t js = e >> 3;
      const Rand4 rr = philox(js, t, replica, tag(c, kIsingRefine), key.k0, key.k1);
      if ((rr.w[0] & 0xFFFFFFu) < dp->frac[e & 7u]) own[js] ^= 1;
    }
    nq = 0;
  };
  const bool words = (R & 3u) == 0;
  const bool pairs = !words && (R & 1u) == 0;
  // E = sum over colour-1 sites of (unsatisfied - satisfied) bonds (each bond
  // once), M = sum of the spins of both colours; record `slot` of this call
  auto measure = [&](uint32_t slot, int64_t sweep) {
    int64_t Esum = 0, Msum = 0;
    if (words) {
      for (uint32_t j = 4 * threadIdx.x; j < Nh; j += 4 * blockDim.x) {
        uint32_t W;
        const uint32_t k = counts(W4{}, lat + Nh, lat, 1u, j, W);
        const uint32_t down = __builtin_popcount(W & kOnes) + __builtin_popcount(ld(lat, j) & kOnes);
        Esum += 2 * (int64_t)__builtin_amdgcn_sad_u8(k, 0u, 0u) - 4 * 2 * D;
        Msum += 8 - 2 * (int64_t)down;
      }
    } else if (pairs) {
      for (uint32_t j = 2 * threadIdx.x; j < Nh; j += 2 * blockDim.x) {
        uint32_t W;
        const uint32_t k = counts(W2{}, lat + Nh, lat, 1u, j, W);
        const uint32_t w0 = *reinterpret_cast<const uint16_t*>(lat + j);
        const uint32_t down = __builtin_popcount(W & kOnes) + __builtin_popcount(w0 & kOnes);
        Esum += 2 * (int64_t)__builtin_amdgcn_sad_u8(k, 0u, 0u) - 2 * 2 * D;
        Msum += 4 - 2 * (int64_t)down;
      }
    } else {
      for (uint32_t j = threadIdx.x; j < Nh; j += blockDim.x) {
        uint32_t o;
        const uint32_t k = site_k(lat + Nh, lat, 1u, j, o);
        Esum += 2 * (int64_t)k - 2 * D;
        Msum += (1 - 2 * (int32_t)(o & 1u)) + (1 - 2 * (int32_t)(lat[j] & 1));
      }
    }
    __shared__ Partial part[1];
    block_partial_int(Esum, Msum, part, 0);
    if (threadIdx.x == 0) {
      ObsOut o;
      o.E_int = part[0].Ei;
      o.M_int = part[0].Mi;
      o.E = (double)part[0].Ei * dp->J0;
      o.M[0] = (double)part[0].Mi;
      o.M[1] = 0.0;
      o.M[2] = 0.0;
      o.absM = fabs((double)part[0].Mi);
      o.sweep = sweep;
      obs[(uint64_t)slot * n_lattices + li] = o;
    }
  };
  const uint32_t ngroups = (Nh + 15) / 16;
  // One group per lane (a lattice with no more groups than lanes): the lane
  // sees the same four words in every half-sweep of the call, so their plane
  // indices and those of their neighbour words (periodic wraps included) are
  // formed once here.  Slot s holds word ws = (s + lane / 8) % 4 of the group
  // (the bank-spreading order of the general path); fpar bit s is the
  // word's (row + z) parity, fval bit s marks the words inside the plane.
  const bool fast = words && ngroups <= blockDim.x;
  uint32_t fj[4], fyp[4], fym[4], fzp[4], fzm[4], fe1[4], fe0[4];
  uint32_t fpar = 0, fval = 0;
  if (fast && threadIdx.x < ngroups) {
#pragma unroll
    for (uint32_t sl = 0; sl < 4; ++sl) {
      const uint32_t ws = (sl + (threadIdx.x >> 3)) & 3u;
      const uint32_t j = 16 * threadIdx.x + 4 * ws;
      const uint32_t jc = j < Nh ? j : 0u;  // words past the plane's end: never used
      fval |= (j < Nh ? 1u : 0u) << sl;
      const uint32_t r = fdiv(jc, divR);
      const uint32_t rowb = r * R;
      const uint32_t jx = jc - rowb;
      const uint32_t z = D == 3 ? fdiv(r, divL) : 0u;
      const uint32_t y = r - z * L;
      fpar |= ((r + z) & 1u) << sl;
      fj[sl] = jc;
      fe1[sl] = jx + 4 == R ? rowb : jc + 4;
      fe0[sl] = jx == 0 ? rowb + R - 4 : jc - 4;
      fyp[sl] = y + 1 == L ? jc - sYw : jc + R;
      fym[sl] = y == 0 ? jc + sYw : jc - R;
      fzp[sl] = fzm[sl] = 0;
      if (D == 3) {
        fzp[sl] = z + 1 == L ? jc - sZw : jc + sZ;
        fzm[sl] = z == 0 ? jc + sZw : jc - sZ;
      }
    }
  }
  for (uint32_t sw = 0; sw < n_sweeps; ++sw) {
    const uint32_t t = t0 + sw;
    for (uint32_t c = 0; c < 2; ++c) {
      int8_t* own = lat + c * Nh;
      const int8_t* oth = lat + (1 - c) * Nh;
      if (fast) {
        if (threadIdx.x < ngroups) {
          const uint32_t g = threadIdx.x;
          const Rand4 rp = philox(g, t, replica, tag(c, kIsingPrefix), key.k0, key.k1);
#pragma unroll
          for (uint32_t sl = 0; sl < 4; ++sl) {
            if ((fval >> sl) & 1u) {
              const uint32_t ws = (sl + (g >> 3)) & 3u;
              const uint32_t j = fj[sl];
              const uint32_t p = (c ^ (fpar >> sl)) & 1u;
              const uint32_t W = ld(own, j);
              const uint32_t C = ld(oth, j);
              const uint32_t E = ld(oth, p ? fe1[sl] : fe0[sl]);
              const uint32_t S = p ? __builtin_amdgcn_alignbyte(E, C, 1) : __builtin_amdgcn_alignbyte(C, E, 3);
              uint32_t nb[6];
              nb[0] = p ? S : C;  // +x
              nb[1] = p ? C : S;  // -x
              nb[2] = ld(oth, fyp[sl]);
              nb[3] = ld(oth, fym[sl]);
              nb[4] = nb[5] = 0;
              if (D == 3) {
                nb[4] = ld(oth, fzp[sl]);
                nb[5] = ld(oth, fzm[sl]);
              }
              const uint32_t k = count_bytes(W, nb);
              uint32_t tie;
              const uint32_t nw = decide(W4{}, W, k, word_of(rp.w, ws), tie);
              *reinterpret_cast<uint32_t*>(own + j) = nw;
              while (tie) {
                const uint32_t b = (uint32_t)__builtin_ctz(tie) >> 3;
                tie &= tie - 1;
                if (nq == kBatchTieSlots) flush(own, c, t);
                tq[nq * blockDim.x] = ((j + b) << 3) | ((k >> (8 * b)) & 7u);
                ++nq;
              }
            }
          }
        }
        flush(own, c, t);
        __syncthreads();
        continue;
      }
      if (words && (R & 15u) == 0) {
        // plane rows of whole groups: a group's four words share the row, its
        // parity and the periodic wraps of their y and z neighbours, formed
        // once per group
        for (uint32_t g = threadIdx.x; g < ngroups; g += blockDim.x) {
          const uint32_t j0 = 16 * g;
          const Rand4 rp = philox(g, t, replica, tag(c, kIsingPrefix), key.k0, key.k1);
          const uint32_t r = fdiv(j0, divR);
          const uint32_t rowb = r * R;
          const uint32_t jx0 = j0 - rowb;
          const uint32_t z = D == 3 ? fdiv(r, divL) : 0u;
          const uint32_t y = r - z * L;
          const uint32_t p = (c + r + z) & 1u;
          const uint32_t dyp = y + 1 == L ? 0u - sYw : R, dym = y == 0 ? sYw : 0u - R;
          const uint32_t dzp = z + 1 == L ? 0u - sZw : sZ, dzm = z == 0 ? sZw : 0u - sZ;
#pragma unroll
          for (uint32_t w = 0; w < 4; ++w) {
            const uint32_t ws = (w + (threadIdx.x >> 3)) & 3u;
            const uint32_t j = j0 + 4 * ws;
            const uint32_t jx = jx0 + 4 * ws;
            const uint32_t W = ld(own, j);
            const uint32_t C = ld(oth, j);
            const uint32_t E = ld(oth, p ? (jx + 4 == R ? rowb : j + 4) : (jx == 0 ? rowb + R - 4 : j - 4));
            const uint32_t S = p ? __builtin_amdgcn_alignbyte(E, C, 1) : __builtin_amdgcn_alignbyte(C, E, 3);
            uint32_t nb[6];
            nb[0] = p ? S : C;  // +x
            nb[1] = p ? C : S;  // -x
            nb[2] = ld(oth, j + dyp);
            nb[3] = ld(oth, j + dym);
            nb[4] = nb[5] = 0;
            if (D == 3) {
              nb[4] = ld(oth, j + dzp);
              nb[5] = ld(oth, j + dzm);
            }
            const uint32_t k = count_bytes(W, nb);
            uint32_t tie;
            const uint32_t nw = decide(W4{}, W, k, word_of(rp.w, ws), tie);
            *reinterpret_cast<uint32_t*>(own + j) = nw;
            while (tie) {
              const uint32_t b = (uint32_t)__builtin_ctz(tie) >> 3;
              tie &= tie - 1;
              if (nq == kBatchTieSlots) flush(own, c, t);
              tq[nq * blockDim.x] = ((j + b) << 3) | ((k >> (8 * b)) & 7u);
              ++nq;
            }
          }
        }
        flush(own, c, t);
        __syncthreads();
        continue;
      }
      if (words) {
        // Nh is a multiple of 4: a group holds nj / 4 whole words
        for (uint32_t g = threadIdx.x; g < ngroups; g += blockDim.x) {
          const uint32_t j0 = 16 * g;
          const Rand4 rp = philox(g, t, replica, tag(c, kIsingPrefix), key.k0, key.k1);
          const uint32_t nwords = Nh - j0 < 16 ? (Nh - j0) >> 2 : 4u;
#pragma unroll
          for (uint32_t w = 0; w < 4; ++w) {
            // lanes 8 apart start on different words of their groups: the
            // words of a step then fall in different LDS banks
            const uint32_t ws = (w + (threadIdx.x >> 3)) & 3u;
            if (ws < nwords) {
              const uint32_t j = j0 + 4 * ws;
              uint32_t tie, k;
              const uint32_t nw = word(W4{}, own, oth, c, j, word_of(rp.w, ws), tie, k);
              *reinterpret_cast<uint32_t*>(own + j) = nw;
              while (tie) {
                const uint32_t b = (uint32_t)__builtin_ctz(tie) >> 3;
                tie &= tie - 1;
                if (nq == kBatchTieSlots) flush(own, c, t);
                tq[nq * blockDim.x] = ((j + b) << 3) | ((k >> (8 * b)) & 7u);
                ++nq;
              }
            }
          }
        }
        flush(own, c, t);
        __syncthreads();
        continue;
      }
      if (pairs) {
        // Nh is even: a group holds nj / 2 whole pairs
        for (uint32_t g = threadIdx.x; g < ngroups; g += blockDim.x) {
          const uint32_t j0 = 16 * g;
          const Rand4 rp = philox(g, t, replica, tag(c, kIsingPrefix), key.k0, key.k1);
          const uint32_t npairs = Nh - j0 < 16 ? (Nh - j0) >> 1 : 8u;
          // not unrolled: the few lattices on this path must not raise the
          // register count of the whole kernel
#pragma unroll 1
          for (uint32_t w = 0; w < 8; ++w) {
            // lanes 8 apart start on different dwords of their groups
            const uint32_t ps = (w + 2 * ((threadIdx.x >> 3) & 3u)) & 7u;
            if (ps < npairs) {
              const uint32_t j = j0 + 2 * ps;
              const uint32_t P = word_of(rp.w, ps >> 1) >> (8 * (j & 2u));
              uint32_t tie, k;
              const uint32_t nw = word(W2{}, own, oth, c, j, P, tie, k);
              *reinterpret_cast<uint16_t*>(own + j) = (uint16_t)nw;
              while (tie) {
                const uint32_t b = (uint32_t)__builtin_ctz(tie) >> 3;
                tie &= tie - 1;
                if (nq == kBatchTieSlots) flush(own, c, t);
                tq[nq * blockDim.x] = ((j + b) << 3) | ((k >> (8 * b)) & 7u);
                ++nq;
              }
            }
          }
        }
        flush(own, c, t);
        __syncthreads();
        continue;
      }
      for (uint32_t g = threadIdx.x; g < ngroups; g += blockDim.x) {
        const uint32_t j0 = 16 * g;
        const Rand4 rp = philox(g, t, replica, tag(c, kIsingPrefix), key.k0, key.k1);
        const uint32_t nj = Nh - j0 < 16 ? Nh - j0 : 16u;
        auto one = [&](uint32_t jj, uint32_t word) {
          const uint32_t j = j0 + jj;
          uint32_t o;
          const uint32_t k = site_k(own, oth, c, j, o);
          const uint32_t P = (word >> (8 * (jj & 3))) & 0xFFu;
          const uint32_t Th = table_byte(th_lo, th_hi, k);
          bool accept = P < Th;
          if (P == Th) {
            const Rand4 rr = philox(j, t, replica, tag(c, kIsingRefine), key.k0, key.k1);
            accept = (rr.w[0] & 0xFFFFFFu) < dp->frac[k];  // rare: read from the table
          }
          if (accept) own[j] = (int8_t)(o ^ 1u);
        };
        // not unrolled: the few lattices on this path must not raise the
        // register count of the whole kernel
#pragma unroll 1
        for (uint32_t jj = 0; jj < nj; ++jj) one(jj, word_of(rp.w, jj >> 2));
      }
      __syncthreads();
    }
    // every thread reaches the barrier inside the block reduction after its
    // reads of the planes: none writes them again before all have read
    if (MEASURE && (sw + 1) % every == 0) measure((sw + 1) / every - 1, (int64_t)t + 1);
  }
  if (MEASURE && n_sweeps == 0) measure(0, (int64_t)t0);

  // write both planes back as +-1 bytes
  for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) gs[i] = (lat[i] & 1) ? (int8_t)-1 : (int8_t)1;

}

bool batch_lattice_packed(int d, uint32_t L, uint32_t threads) {
  return batch_packed_ok(d, L, threads);
}

size_t batch_lds_bytes(int d, bool pm, bool packed, const uint32_t* L, uint32_t n,
                       uint32_t threads, const BatchSplit& split) {
  const uint32_t per = std::max(split.per_full, split.per_tiny);
  size_t bytes = 0;
  for (uint32_t r = 0; r < n; ++r) {
    size_t need;
    if (packed && batch_lattice_wave(d, L[r])) {
      need = (size_t)per * batch_packed_lds_bytes(d, kWaveWords, pm);
    } else if (packed && batch_packed_ok(d, L[r], threads)) {
      need = batch_packed_lds_bytes(d, batch_words(d, L[r]), pm);
    } else {
      size_t N = 1;
      for (int k = 0; k < d; ++k) N *= L[r];
      need = (N + 15) / 16 * 16 + (size_t)threads * kBatchTieSlots * 4;
    }
    bytes = need > bytes ? need : bytes;
  }
  return bytes;
}

bool batch_lattice_tiny(int d, uint32_t L) { return batch_words(d, L) <= kTinyWords; }

// One-wave lattices of more than eight words run best four a workgroup at any count
// (2D L = 32, 20 sweeps, 1 / 2 / 4 a workgroup of 256 lanes: 16 lattices 37 / 49 / 32 us,
// 512 39 / 39 / 33; of 512 lanes 8 a workgroup 43 and 45), up to sixteen where 1024 lanes
// would not all run at once.  Tiny ones slow each other down beside each other while
// CUs are idle (3D L = 8: 16 lattices 35 / 48 / 57, 512 35 / 35 / 36): they fill the others'
// last workgroup, and the rest of them get a workgroup each as long as all run at once (16 waves
// a CU), or, in a batch of other lattices too, have a CU each (512 of 2D L = 8, 32: 95 us
// one a workgroup, 78 by fours).
BatchSplit batch_split(uint32_t n_single, uint32_t n_mid, uint32_t n_tiny, uint32_t threads) {
  const uint32_t waves = threads / 64u, room = 4096u / waves;
  const uint32_t most = n_single ? std::min(waves, 8u) : waves;
  auto fit = [&](uint32_t n, uint32_t used, uint32_t groups) -> uint32_t {  // the least per workgroup
    const uint32_t left = used < groups ? groups - used : 1u;
    return (n + left - 1u) / left;
  };
  BatchSplit s;
  s.n_single = n_single;
  s.per_full = std::min(most, std::max(4u, fit(n_mid, n_single, room)));
  s.g_full = (n_mid + s.per_full - 1u) / s.per_full;
  const uint32_t used = n_single + s.g_full, rest = n_mid + n_tiny - std::min(n_mid + n_tiny, s.g_full * s.per_full);
  s.per_tiny = used == 0 ? fit(rest, 0u, room) : std::min(std::max(4u, fit(rest, used, room)), fit(rest, used, 256u));
  s.per_tiny = std::max(1u, std::min(most, s.per_tiny));
  s.groups = used + (rest + s.per_tiny - 1u) / s.per_tiny;
  return s;
}

hipError_t launch_batch(const BatchLaunch& a, int8_t* spins, const int8_t* J, uint32_t t0,
                        uint32_t n_sweeps, uint32_t every, void* dev_obs, hipStream_t st) {
  const dim3 grid(a.split.groups), block(a.threads);
  const size_t lds = a.lds_bytes;
#define SMC_BK(DD, PMM, MM)                                                                      \
  hipLaunchKernelGGL((batch_kernel<DD, PMM, MM>), grid, block, lds, st, a.descs, a.order, a.key, \
                     spins, J, t0, n_sweeps, every, a.n_lattices, (ObsOut*)dev_obs, a.split)
  const bool m = dev_obs != nullptr;
  if (a.d == 2) {
    if (a.pm) { if (m) SMC_BK(2, true, true); else SMC_BK(2, true, false); }
    else { if (m) SMC_BK(2, false, true); else SMC_BK(2, false, false); }
  } else {
    if (a.pm) { if (m) SMC_BK(3, true, true); else SMC_BK(3, true, false); }
    else { if (m) SMC_BK(3, false, true); else SMC_BK(3, false, false); }
  }
#undef SMC_BK
  return hipGetLastError();
}

// Dynamic LDS beyond the default 64 KiB needs the kernels' attribute raised.
hipError_t batch_allow_lds(size_t bytes) {
  hipError_t e = hipSuccess;
#define SMC_BA(DD, PMM, MM)                                                                     \
  if (e == hipSuccess)                                                                          \
    e = allow_dynamic_lds((const void*)batch_kernel<DD, PMM, MM>, bytes)
  SMC_BA(2, true, true); SMC_BA(2, true, false); SMC_BA(2, false, true); SMC_BA(2, false, false);
  SMC_BA(3, true, true); SMC_BA(3, true, false); SMC_BA(3, false, true); SMC_BA(3, false, false);
#undef SMC_BA
  return e;
}

}  // namespace smc

namespace smc {

const void* batch_kernel_fn(int d, bool pm, bool measure) {
  if (d == 2) {
    if (pm) return measure ? (const void*)batch_kernel<2, true, true> : (const void*)batch_kernel<2, true, false>;
    return measure ? (const void*)batch_kernel<2, false, true> : (const void*)batch_kernel<2, false, false>;
  }
  if (pm) return measure ? (const void*)batch_kernel<3, true, true> : (const void*)batch_kernel<3, true, false>;
  return measure ? (const void*)batch_kernel<3, false, true> : (const void*)batch_kernel<3, false, false>;
}

}  // namespace smc
