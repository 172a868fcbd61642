// resident.hip -- many half-sweeps of one Ising lattice in one launch, its
// words held in LDS (uniform or +-1 couplings, Metropolis or heat bath).
//
// What bounds a small or middling lattice is not its arithmetic but the
// launches (about 4 us each, two a sweep) and the chain of dependent
// instructions inside a half-sweep (two Philox blocks, their transpose, the
// compare, the ties' refinement draws), which a lattice of a few hundred
// words cannot hide behind other waves.  Both go away here:
//  * a launch runs `steps` half-sweeps.  A workgroup owns a run of words of
//    both colours and stages it with a halo of rho words a step on each side
//    (rho: the furthest word a neighbour bit comes from); step k updates the
//    words still valid, so the halo is used up exactly at the end.  Owned
//    words go to another buffer, and no workgroup waits for another.  A small
//    lattice is one workgroup without a halo;
//  * the random part of a decision depends on the counter only: for each word
//    and step the masks "u32 < T[k]" of the refusable classes k, exact ties
//    included, are formed first, for all steps of a chunk at once with every
//    lane busy.  A step is then a few LDS reads, the bit-sliced count of the
//    neighbours and a select among the masks.
// Words are runs of 32 same-colour sites in plane order (as the packed
// kernels'), whether or not a row is a whole number of them: where it is
// (AL) a neighbour word is one LDS word, else a funnel of two with masks at
// the row ends.  The draws per site are those of every other kernel, so the
// chain is the same bit for bit.
#include "packed.hpp"
#include "reduce.hpp"

namespace smc {

namespace {

constexpr uint32_t kListBits = 12;  // local word index in a tie entry
// A wave's tie list: drained whenever it holds 64, and a push adds at most 64.
constexpr uint32_t kListWords = 128;
// Plane stride in LDS: local words -1 .. kMaxWords + 1.  A constant, so that
// the plane of a neighbour read is an immediate offset.
constexpr uint32_t kMaxWords = 2048, kPlane = kMaxWords + 4;

struct GatherAL {  // LDS byte addresses of a word's neighbours; rows of whole words
  uint32_t ctr, e0, e1, yp, ym, zp, zm;  // e0 / e1: the word on the side a row of colour 0 / 1 leaves
  uint32_t Pm0;    // all ones where colour 0's x + 1 neighbour is the next in-row site
};

struct GatherAny {  // rows that split words: low words of funnels, and masks
  uint32_t ctr, wst, wen, yp, ym, ypw, ymw, zp, zm, zpw, zmw;
  uint32_t E, S, Pm0;            // sites at row end / row start, rows of colour-0 parity 1
  uint32_t Ymp, Ymm, Zmp, Zmm;   // sites at y = L-1 / y = 0 / z = L-1 / z = 0
};

// The masks of one word: bit s of lt[q] set where site s's prefix byte is below
// th[q], and the sites `any` whose byte equals some class's (eq[q]).
template <int NC>
__device__ __forceinline__ uint32_t word_masks(const uint32_t th[NC], const RngKey& key, uint32_t t,
                                               uint32_t c, uint32_t gw, uint32_t lt[NC],
                                               uint32_t eq[NC]) {
  uint32_t B[8], any = 0u;
  word_prefix(key, t, c, gw, B);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    uint32_t l = 0u, e = ~0u;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint32_t X = 0u - ((th[q] >> b) & 1u);  // wave-uniform
      l = __builtin_amdgcn_bitop3_b32(B[b], X, l, 0x8E);
      e = __builtin_amdgcn_bitop3_b32(B[b], X, e, 0x82);
    }
    lt[q] = l;
    eq[q] = e;
    any |= e;
  }
  return any;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// f, or f - n where f >= n, twice: f mod n for f < 3 n.
__device__ __forceinline__ uint32_t mod3(uint32_t f, uint32_t n) {
  f = f >= n ? f - n : f;
  return f >= n ? f - n : f;
}

}  // namespace

template <int D, bool HB, bool PM, bool AL, int WPL>
__global__ __launch_bounds__(1024) void resident_kernel(const ResidentLaunch a) {
  constexpr int NC = HB ? 2 * D + 1 : D;  // classes with a mask
  extern __shared__ uint32_t lds[];
  const uint32_t T = blockDim.x, tid = threadIdx.x;
  const uint32_t Wl = a.own + 2u * a.halo;  // local words per colour
  const uint32_t w0 = blockIdx.x * a.own;
  const uint32_t own = min(a.own, a.Wp - w0);
  uint32_t* const sp = lds + 1;  // word l of colour c at sp[c kPlane + l]
  uint32_t* const masks = lds + 2u * kPlane;
  const uint32_t lane = __lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* const list = masks + NC * a.mask_words + wave * kListWords;
  // global word of local word 0
  const uint32_t base = (w0 + a.Wp * ((a.halo + a.Wp - 1u) / a.Wp) - a.halo) % a.Wp;
  const uint32_t L = (uint32_t)a.g.L, R = (uint32_t)a.g.R;
  const uint32_t Nh = (uint32_t)a.g.Nh;
  const uint32_t tail = a.Wp * 32u - Nh;  // bits of the last word past the plane
  const bool whole = a.halo == 0u;
  const uint32_t LR = L * R;

  auto word_of_local = [&](uint32_t l) -> uint32_t { return mod3(base + l, a.Wp); };
  auto valid_bits = [&](uint32_t gw) -> uint32_t { return gw + 1u == a.Wp ? ~0u >> tail : ~0u; };

  // ---- stage the words ----
#pragma unroll 1
  for (uint32_t i = tid; i < 2u * Wl; i += T) {
    const uint32_t c = i >= Wl ? 1u : 0u, l = i - c * Wl;
    const uint32_t gw = word_of_local(l);
    sp[c * kPlane + l] =
        a.src_bytes ? load_signs((const int8_t*)a.src + (uint64_t)c * Nh + 32u * (uint64_t)gw,
                                 gw + 1u == a.Wp ? 32u - tail : 32u)
                    : ((const uint32_t*)a.src)[c * a.Wp + gw];
  }
  // ---- the lane's neighbour addresses and bond signs ----
  using Gather = typename std::conditional<AL, GatherAL, GatherAny>::type;
  Gather gt[WPL];
  uint32_t jb[WPL][PM ? 4 * D : 1];
  uint32_t ow[WPL][2];  // the lane's words (copies of those in LDS)
  // Offsets in sites of the last axis' neighbours across the periodic
  // boundary: the whole plane back when it is local, else the next copy of
  // the plane, which starts after the last word's unused bits.
  const int32_t last = D == 2 ? (int32_t)R : (int32_t)LR;
  const int32_t wrapp = whole ? last - (int32_t)Nh : last + (int32_t)tail;
#pragma unroll
  for (int p = 0; p < WPL; ++p) {
    const uint32_t l = tid + (uint32_t)p * T;
    const uint32_t lv = l < Wl ? l : 0u;
    const uint32_t gw = word_of_local(lv);
    const uint32_t nv = gw + 1u == a.Wp ? 32u - tail : 32u;
    if (l < Wl) {
      if (PM) {
#pragma unroll
        for (int m = 0; m < 4 * D; ++m) jb[p][m] = a.bonds[(uint32_t)m * a.Wp + gw];
      }
    }
    Gather& x = gt[p];
    x.ctr = 4u * (lv + 1u);
    auto clampw = [&](int32_t i) -> uint32_t {  // words -1 .. Wl - 1 (the low word of a funnel)
      return 4u * (uint32_t)((i < -1 ? -1 : (i > (int32_t)Wl - 1 ? (int32_t)Wl - 1 : i)) + 1);
    };
    if constexpr (AL) {
      const uint32_t W = R >> 5;
      const uint32_t r = gw / W, q = gw - r * W;
      const uint32_t z = D == 3 ? r / L : 0u, y = r - z * L;
      const uint32_t odd = (y + z) & 1u;
      x.Pm0 = 0u - odd;
      const int32_t li = (int32_t)lv, Wi = (int32_t)W, col = (int32_t)((L - 1u) * W);
      const uint32_t nx = clampw(q + 1u == W ? li - Wi + 1 : li + 1);
      const uint32_t pv = clampw(q == 0u ? li + Wi - 1 : li - 1);
      x.e0 = odd ? nx : pv;
      x.e1 = odd ? pv : nx;
      const bool wy = D == 3 || whole;  // y closes on itself inside the local words
      x.yp = clampw(wy && y + 1u == L ? li - col : li + Wi);
      x.ym = clampw(wy && y == 0u ? li + col : li - Wi);
      if (D == 3) {
        const int32_t pl = (int32_t)(L * W), all = (int32_t)((L - 1u) * L * W);
        x.zp = clampw(whole && z + 1u == L ? li - all : li + pl);
        x.zm = clampw(whole && z == 0u ? li + all : li - pl);
      }
    } else {
      x.E = x.S = x.Pm0 = x.Ymp = x.Ymm = x.Zmp = x.Zmm = 0u;
      const uint32_t j0 = 32u * gw;
      uint32_t r = j0 / R, jx = j0 - r * R;
      uint32_t z = D == 3 ? r / L : 0u, y = r - z * L;
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
      auto at = [&](int32_t off) -> uint32_t { return clampw((int32_t)lv + (off >> 5)); };
      const int32_t Ri = (int32_t)R;
      x.wst = at(1 - Ri);
      x.wen = at(Ri - 1);
      x.yp = at(Ri);
      x.ym = at(-Ri);
      x.ypw = at(D == 2 ? wrapp : Ri - (int32_t)LR);
      x.ymw = at(D == 2 ? -wrapp : (int32_t)LR - Ri);
      if (D == 3) {
        x.zp = at(last);
        x.zm = at(-last);
        x.zpw = at(wrapp);
        x.zmw = at(-wrapp);
      }
    }
  }
  if (tid < 2u) {  // the pad words are read, never used
    lds[tid * kPlane] = 0u;
    sp[tid * kPlane + Wl] = 0u;
    sp[tid * kPlane + Wl + 1u] = 0u;
  }

  auto sel = [](uint32_t m, uint32_t u, uint32_t v) -> uint32_t {  // m ? u : v
    return __builtin_amdgcn_bitop3_b32(m, u, v, 0xCA);
  };
  // Neighbour words (+x, -x, +y, -y, +z, -z) of a word of colour c.
  auto neighbours = [&](const Gather& x, auto cc, uint32_t nb[6]) {
    constexpr uint32_t c = decltype(cc)::value;
    auto ld = [&](uint32_t at, uint32_t word = 0u) -> uint32_t {
      return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(lds) + at +
                                                4u * ((1u - c) * kPlane + word));
    };
    const uint32_t wc = ld(x.ctr);
    if constexpr (AL) {
      const uint32_t e = ld(c == 0u ? x.e0 : x.e1);
      const uint32_t Pm = c == 0u ? x.Pm0 : ~x.Pm0;
      nb[0] = sel(Pm, __builtin_amdgcn_alignbit(e, wc, 1u), wc);
      nb[1] = sel(Pm, wc, __builtin_amdgcn_alignbit(wc, e, 31u));
      nb[2] = ld(x.yp);
      nb[3] = ld(x.ym);
      if (D == 3) {
        nb[4] = ld(x.zp);
        nb[5] = ld(x.zm);
      }
    } else {
      auto fun = [&](uint32_t i, int32_t off) -> uint32_t {  // bit b: site 32 l + b + off
        return __builtin_amdgcn_alignbit(ld(i, 1u), ld(i), (uint32_t)off & 31u);
      };
      const int32_t Ri = (int32_t)R;
      const uint32_t wp = ld(x.ctr - 4u), wn = ld(x.ctr, 1u);
      const uint32_t next = __builtin_amdgcn_alignbit(wn, wc, 1u);
      const uint32_t prev = __builtin_amdgcn_alignbit(wc, wp, 31u);
      const uint32_t Pm = x.Pm0 ^ (0u - c);
      nb[0] = sel(Pm, sel(x.E, fun(x.wst, 1 - Ri), next), wc);
      nb[1] = sel(Pm, wc, sel(x.S, fun(x.wen, Ri - 1), prev));
      const int32_t wy = D == 2 ? wrapp : Ri - (int32_t)LR;
      nb[2] = sel(x.Ymp, fun(x.ypw, wy), fun(x.yp, Ri));
      nb[3] = sel(x.Ymm, fun(x.ymw, -wy), fun(x.ym, -Ri));
      if (D == 3) {
        nb[4] = sel(x.Zmp, fun(x.zpw, wrapp), fun(x.zp, last));
        nb[5] = sel(x.Zmm, fun(x.zmw, -wrapp), fun(x.zm, -last));
      }
    }
  };

  // words of step k of this launch: lo_k .. Wl - lo_k - 1, lo_k = rho (k + 1);
  // its masks start at first(k) - first(ka) of a chunk that begins at ka
  auto lo_of = [&](uint32_t k) -> uint32_t { return a.rho * (k + 1u); };
  auto first = [&](uint32_t k) -> uint32_t { return k * Wl - a.rho * k * (k + 1u); };
  uint32_t th[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) th[q] = a.th[q];
  // The refinement draw of a listed site: its bit joins the masks of the tied
  // classes whose threshold it is below.
  auto resolve = [&](uint32_t e, uint32_t ka, uint32_t f0) {
    const uint32_t l = e & ((1u << kListBits) - 1u), b = (e >> kListBits) & 31u;
    const uint32_t cls = (e >> (kListBits + 5u)) & 127u, kk = ka + (e >> (kListBits + 12u));
    const uint32_t h = a.step0 + kk, t = a.t0 + (h >> 1), c = h & 1u;
    const Rand4 rr = philox(32u * word_of_local(l) + b, t, a.key.replica, tag(c, kIsingRefine), a.key.k0, a.key.k1);
    const uint32_t at = first(kk) - f0 + l - lo_of(kk);
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (((cls >> q) & 1u) && (rr.w[0] & 0xFFFFFFu) < a.frac[q])
        atomicOr(&masks[(uint32_t)q * a.mask_words + at], 1u << b);
  };

  __syncthreads();
#pragma unroll
  for (int p = 0; p < WPL; ++p) {
    const uint32_t l = tid + (uint32_t)p * T;
    ow[p][0] = ow[p][1] = 0u;
    if (l < Wl) {
      ow[p][0] = sp[l];
      ow[p][1] = sp[kPlane + l];
    }
  }

  for (uint32_t ka = 0; ka < a.steps; ka += a.chunk) {
    const uint32_t kb = min(ka + a.chunk, a.steps);
    const uint32_t f0 = first(ka), M = first(kb) - f0;
    // ---- the masks of the chunk ----
    // Exact ties (a prefix byte equal to some class's threshold byte, 2^-8 a
    // class) go to the wave's own list, numbered by ballots: no atomic, and
    // no barrier before the wave draws their refinements.
    uint32_t nt = 0u;  // wave-uniform: entries of the list
    // the list's entries from `from` on, a lane each
    auto draw_ties = [&](uint32_t from) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (from + lane < nt) resolve(list[from + lane], ka, f0);
      nt = from;
    };
    // the lane's word: r-th of step k, whose words start at lo and number n
    uint32_t k = ka, r = tid, lo = lo_of(ka), n = Wl - 2u * lo;
    if (a.drawn) {  // made by draw_kernel: four words' loads in flight a lane
#pragma unroll 1
      for (uint32_t i0 = tid; i0 < M; i0 += 4u * T) {
        uint32_t v[4][NC];
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
          if (i0 + j * T < M) {
            while (r >= n) {
              r -= n;
              n -= 2u * a.rho;
              lo += a.rho;
              ++k;
            }
            const uint32_t* src = a.drawn + (uint64_t)(a.step0 + k) * a.Wp + word_of_local(lo + r);
#pragma unroll
            for (int q = 0; q < NC; ++q) v[j][q] = src[(uint64_t)q * a.drawn_stride];
            r += T;
          }
        }
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
          if (i0 + j * T < M) {
#pragma unroll
            for (int q = 0; q < NC; ++q) masks[(uint32_t)q * a.mask_words + i0 + j * T] = v[j][q];
          }
        }
      }
    } else
#pragma unroll 1
    for (uint32_t i0 = wave * 64u; i0 < M; i0 += T, r += T) {
      const uint32_t i = i0 + lane;
      uint32_t any = 0u, eq[NC], tie = 0u;
      if (i < M) {
        while (r >= n) {
          r -= n;
          n -= 2u * a.rho;
          lo += a.rho;
          ++k;
        }
        const uint32_t l = lo + r, gw = word_of_local(l);
        const uint32_t h = a.step0 + k, t = a.t0 + (h >> 1), c = h & 1u;
        uint32_t lt[NC];
        any = word_masks<NC>(th, a.key, t, c, gw, lt, eq);
#pragma unroll
        for (int q = 0; q < NC; ++q) masks[(uint32_t)q * a.mask_words + i] = lt[q];
        any &= valid_bits(gw);
        tie = ((k - ka) << (kListBits + 12u)) | l;
      }
#pragma unroll 1
      for (uint64_t more = __ballot(any != 0u); more; more = __ballot(any != 0u)) {
        if (any) {
          const uint32_t b = __builtin_ctz(any);
          any &= any - 1u;
          uint32_t cls = 0u;
#pragma unroll
          for (int q = 0; q < NC; ++q) cls |= ((eq[q] >> b) & 1u) << q;
          list[nt + lanes_below(more)] =
              tie | (cls << (kListBits + 5u)) | (b << kListBits);
        }
        nt += (uint32_t)__popcll(more);
        if (nt >= 64u) draw_ties(nt - 64u);  // a full wave of them
      }
    }
    draw_ties(0u);
    __syncthreads();
    // ---- the chunk's half-sweeps ----
    // A step reads its neighbour words and the next step's masks together.  A
    // wave none of whose words the step needs skips it; the other words a
    // step does not need may take any value: no later step reads them.
    uint32_t A[2][WPL][NC];  // by colour
    auto fetch = [&](uint32_t kk, auto cc) {
      constexpr uint32_t c = decltype(cc)::value;
      const uint32_t mb = first(kk) - f0 - lo_of(kk);
#pragma unroll
      for (int p = 0; p < WPL; ++p) {
        const uint32_t at = min(mb + tid + (uint32_t)p * T, a.mask_words - 1u);
#pragma unroll
        for (int q = 0; q < NC; ++q) A[c][p][q] = masks[(uint32_t)q * a.mask_words + at];
      }
    };
    const uint32_t w64 = wave * 64u;
    auto step = [&](uint32_t kk, auto cc) {
      constexpr uint32_t c = decltype(cc)::value;
      const uint32_t slo = lo_of(kk);
      bool used = false;
#pragma unroll
      for (int p = 0; p < WPL; ++p) {
        const uint32_t wl = w64 + (uint32_t)p * T;
        used = used || (wl + 64u > slo && wl + slo < Wl);
      }
      if (used) {
        uint32_t nb[WPL][6];
#pragma unroll
        for (int p = 0; p < WPL; ++p) neighbours(gt[p], cc, nb[p]);
        if (kk + 1u < kb) fetch(kk + 1u, std::integral_constant<uint32_t, 1u - c>());
#pragma unroll
        for (int p = 0; p < WPL; ++p) {
          const uint32_t l = tid + (uint32_t)p * T;
          uint32_t u[6];
          const uint32_t o = ow[p][c];
#pragma unroll
          for (int m = 0; m < 2 * D; ++m) {
            // Metropolis: unsatisfied bonds (satisfied ones when J0 < 0);
            // heat bath: up neighbours
            u[m] = HB ? ~nb[p][m] : o ^ nb[p][m] ^ a.invert;
            if (PM) u[m] ^= jb[p][c * 2 * D + m];
          }
          uint32_t k0, k1, k2;
          count_planes<D>(u, k0, k1, k2);
          const uint32_t* M = A[c][p];
          uint32_t nw;
          if constexpr (HB) {
            const uint32_t a01 = sel(k0, M[1], M[0]), a23 = sel(k0, M[3], M[2]);
            const uint32_t lo4 = sel(k1, a23, a01);
            if constexpr (D == 2) {
              nw = ~sel(k2, M[4], lo4);
            } else {
              nw = ~sel(k2, sel(k1, M[6], sel(k0, M[5], M[4])), lo4);
            }
          } else if constexpr (D == 2) {
            nw = o ^ (k1 | k2 | sel(k0, M[1], M[0]));
          } else {
            // classes 0, 1, 2 can refuse; 3 and above always accept
            nw = o ^ (k2 | (k1 & k0) | sel(k1, M[2], sel(k0, M[1], M[0])));
          }
          ow[p][c] = nw;
          if (l < Wl) sp[c * kPlane + l] = nw;
        }
      }
      __syncthreads();
    };
    using C0 = std::integral_constant<uint32_t, 0>;
    using C1 = std::integral_constant<uint32_t, 1>;
    uint32_t kk = ka;
    if ((a.step0 + kk) & 1u) {
      fetch(kk, C1());
      step(kk++, C1());
    } else {
      fetch(kk, C0());
    }
#pragma unroll 1
    while (kk < kb) {
      step(kk++, C0());
      if (kk < kb) step(kk++, C1());
    }
  }

  // ---- the owned words go back ----
  int64_t Esum = 0, Msum = 0;
  const bool measure = a.parts != nullptr || a.obs != nullptr;
#pragma unroll
  for (int p = 0; p < WPL; ++p) {
    const uint32_t l = tid + (uint32_t)p * T;
    if (l < a.halo || l >= a.halo + own) continue;
    const uint32_t gw = w0 + (l - a.halo);
    const uint32_t nv = gw + 1u == a.Wp ? 32u - tail : 32u;
#pragma unroll
    for (uint32_t c = 0; c < 2u; ++c) {
      const uint32_t v = ow[p][c];
      if (a.dst_bytes)
        store_signs((int8_t*)a.dst + (uint64_t)c * Nh + 32u * (uint64_t)gw, v, nv);
      else
        ((uint32_t*)a.dst)[c * a.Wp + gw] = v;
    }
    if (measure) {  // every bond has one colour-1 end
      const uint32_t ok = valid_bits(gw);
      const uint32_t o = ow[p][1], o0 = ow[p][0];
      uint32_t nb[6], u[6], k0, k1, k2;
      neighbours(gt[p], std::integral_constant<uint32_t, 1>(), nb);
#pragma unroll
      for (int m = 0; m < 2 * D; ++m) u[m] = o ^ nb[m] ^ (PM ? jb[p][2 * D + m] : 0u);
      count_planes<D>(u, k0, k1, k2);
      const int32_t ks = __builtin_popcount(k0 & ok) + 2 * __builtin_popcount(k1 & ok) +
                         4 * __builtin_popcount(k2 & ok);
      Esum += 2 * (int64_t)ks - (int64_t)nv * 2 * D;
      Msum += 2 * (int64_t)nv - 2 * (int64_t)(__builtin_popcount(o & ok) + __builtin_popcount(o0 & ok));
    }
  }
  if (!measure) return;
  if (gridDim.x > 1u) {
    block_partial_int(Esum, Msum, (Partial*)a.parts, blockIdx.x);
    return;
  }
  __shared__ Partial part[1];  // one workgroup: the record itself
  block_partial_int(Esum, Msum, part, 0);
  if (tid != 0) return;
  const int64_t E = part[0].Ei, M = part[0].Mi;
  ObsOut o;
  o.E_int = E;
  o.M_int = M;
  o.E = a.J0 * (double)E;
  o.M[0] = (double)M;
  o.M[1] = 0.0;
  o.M[2] = 0.0;
  o.absM = fabs((double)M);
  o.sweep = a.sweep;
  *(ObsOut*)a.obs = o;
}

// The masks of a call's half-sweeps, a word and step a lane, into memory: what
// the workgroups of resident_kernel would each form for their halo is formed
// once (a launch and a read of the masks against two to five times the draws).
// blockIdx.y is the step: its counter words are scalar.  The ties of the four
// waves share a round of draws.
template <int NC>
__global__ __launch_bounds__(256) void draw_kernel(const ResidentLaunch a, uint32_t* __restrict__ out) {
  __shared__ uint32_t mask[NC][256], list[4][256], count[4];
  const uint32_t tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
  const uint32_t gw = blockIdx.x * 256u + tid, k = blockIdx.y;
  const uint32_t t = a.t0 + (k >> 1), c = k & 1u;
  const uint32_t tail = a.Wp * 32u - (uint32_t)a.g.Nh;
  uint32_t th[NC], lt[NC], eq[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) th[q] = a.th[q];
  uint32_t any = word_masks<NC>(th, a.key, t, c, gw, lt, eq);
  if (gw + 1u >= a.Wp) any &= gw + 1u == a.Wp ? ~0u >> tail : 0u;
#pragma unroll
  for (int q = 0; q < NC; ++q) mask[q][tid] = lt[q];
  uint32_t nt = 0u;
#pragma unroll 1
  for (uint64_t more = __ballot(any != 0u); more && nt <= 192u; more = __ballot(any != 0u)) {
    if (any) {
      const uint32_t b = __builtin_ctz(any);
      any &= any - 1u;
      uint32_t cls = 0u;
#pragma unroll
      for (int q = 0; q < NC; ++q) cls |= ((eq[q] >> b) & 1u) << q;
      list[wave][nt + lanes_below(more)] = (cls << 13) | (b << 8) | tid;
    }
    nt += (uint32_t)__popcll(more);
  }
  if (lane == 0u) count[wave] = nt;
  __syncthreads();
  auto draw = [&](uint32_t b) -> uint32_t {
    return philox(32u * (blockIdx.x * 256u) + b, t, a.key.replica, tag(c, kIsingRefine), a.key.k0, a.key.k1).w[0] & 0xFFFFFFu;
  };
  const uint32_t n0 = count[0], n1 = n0 + count[1], n2 = n1 + count[2], n3 = n2 + count[3];
#pragma unroll 1
  for (uint32_t i = tid; i < n3; i += 256u) {
    const uint32_t w = (i >= n0 ? 1u : 0u) + (i >= n1 ? 1u : 0u) + (i >= n2 ? 1u : 0u);
    const uint32_t e = list[w][i - (w == 0u ? 0u : w == 1u ? n0 : w == 2u ? n1 : n2)];
    const uint32_t who = e & 255u, b = (e >> 8) & 31u, cls = e >> 13;
    const uint32_t u = draw(32u * who + b);
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (((cls >> q) & 1u) && u < a.frac[q]) atomicOr(&mask[q][who], 1u << b);
  }
#pragma unroll 1
  while (any) {  // more ties in the wave than its list holds: the lane's own
    const uint32_t b = __builtin_ctz(any);
    any &= any - 1u;
    const uint32_t u = draw(32u * tid + b);
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (((eq[q] >> b) & 1u) && u < a.frac[q]) atomicOr(&mask[q][tid], 1u << b);
  }
  __syncthreads();
  if (gw < a.Wp) {
#pragma unroll
    for (int q = 0; q < NC; ++q) out[(uint64_t)q * a.drawn_stride + (uint64_t)k * a.Wp + gw] = mask[q][tid];
  }
}

hipError_t launch_draws(const ResidentLaunch& a, bool heatbath, uint32_t steps, uint32_t* out,
                        hipStream_t st) {
  const dim3 grid((a.Wp + 255u) / 256u, steps), block(256);
  if (a.g.d == 2) {
    if (heatbath) hipLaunchKernelGGL(draw_kernel<5>, grid, block, 0, st, a, out);
    else hipLaunchKernelGGL(draw_kernel<2>, grid, block, 0, st, a, out);
  } else {
    if (heatbath) hipLaunchKernelGGL(draw_kernel<7>, grid, block, 0, st, a, out);
    else hipLaunchKernelGGL(draw_kernel<3>, grid, block, 0, st, a, out);
  }
  return hipGetLastError();
}

// The signs of every site's 2 d bonds as words aligned with the sites':
// out[(c 2d + m) Wp + w], m = +x, -x, +y, -y, ...  One lane a site; a wave's
// ballot is two words.
template <int D, bool BYTES>
__global__ __launch_bounds__(256) void bond_words_kernel(const Geom g, const FastDiv divR,
                                                         const FastDiv divL, const uint32_t Wp,
                                                         const void* __restrict__ J,
                                                         uint32_t* __restrict__ out) {
  const uint32_t j = blockIdx.x * 256u + threadIdx.x, c = blockIdx.y;
  const uint32_t L = (uint32_t)g.L, R = (uint32_t)g.R, Nh = (uint32_t)g.Nh;
  const bool in = j < Nh;
  const uint32_t jc = in ? j : 0u;
  const uint32_t r = fdiv(jc, divR), jx = jc - r * R;
  const uint32_t z = D == 3 ? fdiv(r, divL) : 0u, y = r - z * L;
  const uint32_t p = (c + y + z) & 1u;
  uint32_t im[3];
  im[0] = jx + p == 0u ? jc + R - 1u : jc + p - 1u;
  im[1] = y == 0u ? jc + (L - 1u) * R : jc - R;
  im[2] = z == 0u ? jc + (L - 1u) * L * R : jc - L * R;
  auto neg = [&](uint32_t plane, uint32_t i) -> bool {
    if (BYTES) return ((const int8_t*)J)[(uint64_t)plane * Nh + i] < 0;
    return (((const uint32_t*)J)[(uint64_t)plane * Wp + (i >> 5)] >> (i & 31u)) & 1u;
  };
  const uint32_t w = j >> 5;
#pragma unroll
  for (int mu = 0; mu < D; ++mu) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const uint64_t b = __ballot(in && (s == 0 ? neg(2u * mu + c, jc) : neg(2u * mu + 1u - c, im[mu])));
      if ((threadIdx.x & 31u) == 0u && w < Wp)
        out[(c * 2u * D + 2u * mu + s) * Wp + w] = (uint32_t)(threadIdx.x & 32u ? b >> 32 : b);
    }
  }
}

hipError_t launch_bond_words(const Geom& g, bool bytes, const void* J, uint32_t* out,
                             hipStream_t st) {
  const uint32_t Wp = (uint32_t)((g.Nh + 31) / 32);
  const dim3 grid((Wp * 32u + 255u) / 256u, 2), block(256);
  const FastDiv dR = make_fastdiv((uint32_t)g.R), dL = make_fastdiv((uint32_t)g.L);
#define SMC_BW(DD, BB) \
  hipLaunchKernelGGL((bond_words_kernel<DD, BB>), grid, block, 0, st, g, dR, dL, Wp, J, out)
  if (g.d == 2) { if (bytes) SMC_BW(2, true); else SMC_BW(2, false); }
  else { if (bytes) SMC_BW(3, true); else SMC_BW(3, false); }
#undef SMC_BW
  return hipGetLastError();
}

static size_t resident_lds_bytes(const ResidentLaunch& a, bool heatbath, uint32_t threads) {
  const uint32_t nc = (uint32_t)(heatbath ? 2 * a.g.d + 1 : a.g.d);
  return 4u * (2u * (size_t)kPlane + (size_t)nc * a.mask_words + (threads / 64u) * (size_t)kListWords);
}

template <int D, bool HB, bool PM, bool AL>
static hipError_t launch_resident_w(const ResidentLaunch& a, uint32_t threads, uint32_t groups,
                                    size_t lds, hipStream_t st) {
  const uint32_t Wl = a.own + 2u * a.halo;
  const void* fn = Wl <= threads ? (const void*)resident_kernel<D, HB, PM, AL, 1>
                                 : (const void*)resident_kernel<D, HB, PM, AL, 2>;
  const hipError_t e = lds > 65536 ? allow_dynamic_lds(fn, lds) : hipSuccess;
  if (e != hipSuccess) return e;
  if (Wl <= threads)
    hipLaunchKernelGGL((resident_kernel<D, HB, PM, AL, 1>), dim3(groups), dim3(threads), lds, st, a);
  else
    hipLaunchKernelGGL((resident_kernel<D, HB, PM, AL, 2>), dim3(groups), dim3(threads), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_resident(const ResidentLaunch& a, bool heatbath, uint32_t threads,
                           hipStream_t st) {
  const uint32_t groups = (a.Wp + a.own - 1u) / a.own;
  const size_t lds = resident_lds_bytes(a, heatbath, threads);
  const bool pm = a.bonds != nullptr, al = a.g.R % 32 == 0;
#define SMC_RS(DD, HH, PP) \
  (al ? launch_resident_w<DD, HH, PP, true>(a, threads, groups, lds, st) \
      : launch_resident_w<DD, HH, PP, false>(a, threads, groups, lds, st))
  if (a.g.d == 2) {
    if (heatbath) return pm ? SMC_RS(2, true, true) : SMC_RS(2, true, false);
    return pm ? SMC_RS(2, false, true) : SMC_RS(2, false, false);
  }
  if (heatbath) return pm ? SMC_RS(3, true, true) : SMC_RS(3, true, false);
  return pm ? SMC_RS(3, false, true) : SMC_RS(3, false, false);
#undef SMC_RS
}

}  // namespace smc
