// ising.hip -- checkerboard Metropolis half-sweeps for Ising spins (n = 1).
//
// One launch updates every site of one colour (Sec. 2 of the paper: all sites
// of a sublattice are independent given the other sublattice).  Decision per
// site (Eq. (2)): k = number of unsatisfied bonds (J_b s_i s_b < 0), dE =
// 4 J0 (d - k); accept iff class k is "always" (dE <= 0) or the site's 32-bit
// uniform u32 = prefix byte << 24 | refinement word is below the integer
// threshold T[k] = ceil(2^32 exp(-beta dE)).  The prefix byte decides unless
// it equals T[k] >> 24 (probability 2^-8), and only then is the refinement
// block drawn.
//
// Two kernels of the integer rules give bit-identical results (a third, below,
// has the real-valued rule of FP32 couplings):
//  * ising_site_kernel -- one site per thread, any even L;
//  * ising_chunk_kernel -- one 16-byte chunk (16 consecutive same-colour
//    sites of a plane row) per lane, L % 32 == 0, uniform or +-1 couplings.
//    Neighbour chunks are loaded as whole 16-byte vectors; the in-row
//    neighbour is the centre chunk shifted by one byte (v_alignbyte) with one
//    edge word from the adjacent chunk; unsatisfied-bond counts are formed
//    four sites per 32-bit op (SWAR on bit 1 of the +-1 bytes); the threshold
//    bytes come from a v_perm byte lookup; one Philox block supplies the 16
//    prefix bytes.
#include "chunk.hpp"
#include "reduce.hpp"

namespace smc {

FastDiv make_fastdiv(uint32_t d) {
  FastDiv f{d, 0u, 0u};
  if (d <= 1) return f;
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  const unsigned __int128 num = ((unsigned __int128)1 << 32) * (((uint64_t)1 << l) - d);
  f.m = (uint32_t)(num / d + 1);
  f.s = l - 1;
  return f;
}

// ---------------------------------------------------------------------------
// One site per thread.  MEASURE (colour 1, here and in the chunk kernel): the
// energy of the bonds of the updated sites and the magnetisation on the way,
// which spares a measured sweep a launch over the whole state (us a measured
// sweep, apart / on the way: 2D L = 288 heat bath 13.1 / 9.8, L = 1002 +-1 19.6 / 14.2,
// 3D L = 64 +-1 13.9 / 10.7, L = 160 18.5 / 12.6).
// ---------------------------------------------------------------------------
template <int D, int JK, bool MEASURE>
__global__ __launch_bounds__(256) void ising_site_kernel(const Geom g, const RngKey key,
                                                         const IsingTable tab,
                                                         const int8_t* __restrict__ J,
                                                         const FastDiv divR, const FastDiv divL,
                                                         int8_t* __restrict__ s,
                                                         const uint32_t t, const uint32_t c,
                                                         const int heatbath,
                                                         Partial* __restrict__ parts) {
  const uint32_t L = (uint32_t)g.L, R = (uint32_t)g.R;
  const int64_t Nh = g.Nh;
  const uint32_t j = blockIdx.x * 256u + threadIdx.x;
  int64_t Esum = 0, Msum = 0;
  if (j < (uint32_t)Nh) {
    int8_t* own = s + (int64_t)c * Nh;
    const int8_t* oth = s + (int64_t)(1 - c) * Nh;
    const uint32_t r = fdiv(j, divR), jx = j - r * R;
    const uint32_t z = D == 3 ? fdiv(r, divL) : 0u, y = r - z * L;
    const uint32_t p = (c + y + z) & 1u;
    uint32_t ip[3], im[3];
    ip[0] = jx + p == R ? j - jx : j + p;
    im[0] = jx + p == 0u ? j + R - 1u : j + p - 1u;
    ip[1] = y + 1u == L ? j - (L - 1u) * R : j + R;
    im[1] = y == 0u ? j + (L - 1u) * R : j - R;
    if (D == 3) {
      ip[2] = z + 1u == L ? j - (L - 1u) * L * R : j + L * R;
      im[2] = z == 0u ? j + (L - 1u) * L * R : j - L * R;
    }
    const int si = own[j];
    int kunsat = 0, field = 0;
#pragma unroll
    for (int mu = 0; mu < D; ++mu) {
      int sp = oth[ip[mu]], sm = oth[im[mu]];
      if (JK == 1) {
        sp *= J[((int64_t)mu * 2 + c) * Nh + j];
        sm *= J[((int64_t)mu * 2 + (1 - c)) * Nh + im[mu]];
      }
      kunsat += (si * sp < 0) + (si * sm < 0);
      field += sp + sm;
    }
    const uint32_t k = (uint32_t)kunsat;
    const Rand4 rp = philox(j >> 4, t, key.replica, tag(c, kIsingPrefix), key.k0, key.k1);
    const uint32_t P = (pick4(rp, (j >> 2) & 3u) >> (8 * (j & 3u))) & 0xFFu;
    // heat bath: class npos = neighbours with sign(J) s_nb = +1, new spin +1
    // iff u32 < T_hb; Metropolis: class k, the spin turns iff u32 < T
    const uint32_t cls = heatbath && si > 0 ? 2u * D - k : k;
    const uint32_t Th = table_byte(tab.th_lo, tab.th_hi, cls);
    bool below = P < Th || (!heatbath && table_byte(tab.al_lo, tab.al_hi, cls) != 0);
    if (!below && P == Th) {
      const Rand4 rr = philox(j, t, key.replica, tag(c, kIsingRefine), key.k0, key.k1);
      below = (rr.w[0] & 0xFFFFFFu) < frac_of(tab, cls);
    }
    const int nv = heatbath ? (below ? 1 : -1) : below ? -si : si;
    if (nv != si) own[j] = (int8_t)nv;
    if (MEASURE) {
      Esum = -(int64_t)nv * field;
      Msum = nv + (int)oth[j];
    }
  }
  if (MEASURE) block_partial_int(Esum, Msum, parts, blockIdx.x);
}

// ---------------------------------------------------------------------------
// FP32 couplings: V sites of a row per lane.  A half-sweep reads every
// coupling (4 N d bytes) for N / 2 sites, so with V = 4 they come in 16-byte
// loads, one Philox block serves the lane, and the row is found by two
// multiplications; V = 1 where rows are no multiple of four.  MEASURE
// (colour 1): energy and magnetisation of the result on the way.
// us a half-sweep, one site a lane by divisions / V = 1 / V = 4: 2D L = 1440
// 7.2 / 4.8 / 3.4, L = 2048 11.3 / 7.8 / 6.3 (33.5 MB of couplings: 5.3 TB/s),
// 3D L = 128 7.6 / 5.4 / 3.8; a measured sweep of 2D L = 1856 33.8 / 28.2 / 15.6.
// ---------------------------------------------------------------------------
template <int D, int V, bool MEASURE>
__global__ __launch_bounds__(256) void ising_real_kernel(const Geom g, const RngKey key,
                                                         const float* __restrict__ J,
                                                         const float beta, const FastDiv divR,
                                                         const FastDiv divL,
                                                         int8_t* __restrict__ s, const uint32_t t,
                                                         const uint32_t c, Partial* __restrict__ parts) {
  const uint32_t L = (uint32_t)g.L, R = (uint32_t)g.R;
  const int64_t Nh = g.Nh;
  const uint32_t gid = xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  Partial part{0, 0, 0.0, {0.0, 0.0, 0.0}};
  if (gid < (uint32_t)(Nh / V)) {
    int8_t* own = s + (int64_t)c * Nh;
    const int8_t* oth = s + (int64_t)(1 - c) * Nh;
    const uint32_t j = V * gid;
    const uint32_t r = fdiv(j, divR), jx = j - r * R;
    const uint32_t z = D == 3 ? fdiv(r, divL) : 0u, y = r - z * L;
    const bool p = ((c + y + z) & 1u) != 0u;
    // y and z neighbours; x: the row's sites j .. j + V - 1 and the one beyond
    // them (p: after, else before)
    uint32_t ip[3], im[3];
    ip[1] = y + 1u == L ? j - (L - 1u) * R : j + R;
    im[1] = y == 0u ? j + (L - 1u) * R : j - R;
    if (D == 3) {
      ip[2] = z + 1u == L ? j - (L - 1u) * L * R : j + L * R;
      im[2] = z == 0u ? j + (L - 1u) * L * R : j - L * R;
    }
    const uint32_t edge = p ? (jx + V == R ? j - jx : j + V) : (jx == 0u ? j + R - 1u : j - 1u);
    auto signs = [&](const int8_t* from, uint32_t at, int o[V]) {
      if (V == 4) {
        const char4 q = *reinterpret_cast<const char4*>(from + at);
        o[0] = q.x; o[V > 1 ? 1 : 0] = q.y; o[V > 2 ? 2 : 0] = q.z; o[V > 3 ? 3 : 0] = q.w;
      } else {
        o[0] = from[at];
      }
    };
    auto bonds = [&](int mu, uint32_t colour, uint32_t at, float o[V]) {
      const float* from = J + ((int64_t)mu * 2 + colour) * Nh;
      if (V == 4) {
        const float4 q = *reinterpret_cast<const float4*>(from + at);
        o[0] = q.x; o[V > 1 ? 1 : 0] = q.y; o[V > 2 ? 2 : 0] = q.z; o[V > 3 ? 3 : 0] = q.w;
      } else {
        o[0] = from[at];
      }
    };
    int si[V], ctr[V], sn[2 * D][V];
    float jb[2 * D][V];
    signs(own, j, si);
    signs(oth, j, ctr);
    const int es = oth[edge];
    bonds(0, c, j, jb[0]);
    float jc[V];
    // the -x bonds belong to the other colour's sites: p: the row's, else one back
    const float* Jx = J + (int64_t)(1 - c) * Nh;
    bonds(0, 1 - c, j, jc);
    const float je = Jx[edge];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      sn[0][v] = p ? (v + 1 < V ? ctr[(v + 1) % V] : es) : ctr[v];
      sn[1][v] = p ? ctr[v] : (v > 0 ? ctr[(v + V - 1) % V] : es);
      jb[1][v] = p ? jc[v] : (v > 0 ? jc[(v + V - 1) % V] : je);
    }
#pragma unroll
    for (int mu = 1; mu < D; ++mu) {
      signs(oth, ip[mu], sn[2 * mu]);
      signs(oth, im[mu], sn[2 * mu + 1]);
      bonds(mu, c, j, jb[2 * mu]);
      bonds(mu, 1 - c, im[mu], jb[2 * mu + 1]);
    }
    const Rand4 rnd = philox(j >> 2, t, key.replica, tag(c, kContinuous), key.k0, key.k1);
    const float bl2e = beta_log2e(beta);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      float h = 0.0f;
#pragma unroll
      for (int b = 0; b < 2 * D; ++b) h += jb[b][v] * (float)sn[b][v];
      const float dE = 2.0f * (float)si[v] * h;
      const uint32_t w = V == 4 ? rnd.w[v] : pick4(rnd, j & 3u);
      if (metropolis_fp32(dE, u01f(w), bl2e)) {
        si[v] = -si[v];
        own[j + v] = (int8_t)si[v];
      }
      if (MEASURE) {
#pragma unroll
        for (int b = 0; b < 2 * D; ++b) part.E -= (double)jb[b][v] * (double)(si[v] * sn[b][v]);
        part.Mi += si[v] + ctr[v];
      }
    }
  }
  if (MEASURE) block_partial(part, parts);
}

// ---------------------------------------------------------------------------
// 16 sites per lane.
// ---------------------------------------------------------------------------
template <int D, bool PM, bool MEASURE>
__global__ __launch_bounds__(256) void ising_chunk_kernel(const Geom g, const RngKey key,
                                                          const IsingTable tab,
                                                          const int8_t* __restrict__ J,
                                                          const FastDiv divQ, const FastDiv divL,
                                                          int8_t* __restrict__ s,
                                                          const uint32_t t, const uint32_t c,
                                                          Partial* __restrict__ parts) {
  const uint32_t gid = xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  int64_t Esum = 0, Msum = 0;
  if (gid < (uint32_t)(g.Nh >> 4)) {
    int64_t base;
    Chunk o, ctr;
    uint32_t kk[4];
    chunk_counts<D, PM>(g, s, J, divQ, divL, c, gid, base, o, ctr, kk);
    int8_t* own = s + (int64_t)c * g.Nh;
    // rare prefix ties on uphill moves are resolved exactly by the sites'
    // 24-bit refinement draws
    const Chunk n = update_chunk_now(tab_regs(tab), key, t, c, (uint32_t)base, o, kk);
    const uint32_t nw[4] = {n.w[0], n.w[1], n.w[2], n.w[3]};
    st16(own + base, nw);
    if (MEASURE) {
      uint32_t unsat = 0, down = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t turned = (((n.w[w] ^ o.w[w]) >> 1) & kOnes) * 0xFFu;
        unsat = __builtin_amdgcn_sad_u8(((2u * D * kOnes - kk[w]) & turned) | (kk[w] & ~turned), 0u, unsat);
        down = __builtin_amdgcn_sad_u8(n.w[w] & kBit1, 0u, down);
        down = __builtin_amdgcn_sad_u8(ctr.w[w] & kBit1, 0u, down);
      }
      // each site: s_i h_i = 2d - 2k; M: 32 sites, down counted twice (bit value 2)
      Esum = -(int64_t)(16 * 2 * D) + 2 * (int64_t)unsat;
      Msum = 32 - (int64_t)down;
    }
  }
  if (MEASURE) block_partial_int(Esum, Msum, parts, blockIdx.x);
}


// ---------------------------------------------------------------------------
// Streaming half-sweep (uniform couplings, L % 32 == 0).  Lane (band, q) owns
// chunk column q of plane rows band*H .. band*H + H - 1 (H divides L, so a
// band stays inside one z-plane) and walks down them, keeping the other
// colour's rows y-1, y, y+1 of its column in registers: per row it loads one
// new other-colour chunk, its own chunk (both one row ahead), one edge word,
// and in 3D the two z-neighbour chunks.  Bands of neighbouring rows fall in
// the same XCD (xcd_remap), so the band halo rows and the z-neighbour rows
// are L2 hits.
// ---------------------------------------------------------------------------
template <int D, bool MEASURE>
__global__ __launch_bounds__(256) void ising_stream_kernel(const Geom g, const RngKey key,
                                                           const IsingTable table,
                                                           const FastDiv divQ, const FastDiv divL,
                                                           const uint32_t H, const uint32_t nbands,
                                                           int8_t* __restrict__ s,
                                                           const uint32_t t, const uint32_t c,
                                                           Partial* __restrict__ parts) {
  __shared__ uint16_t tie_slots[kTieSlots * 256];
  const uint32_t tid = xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  const uint32_t band = fdiv(tid, divQ);
  int64_t Esum = 0, Msum = 0;
  if (band < nbands) {
    const uint32_t Q = divQ.d;
    const uint32_t q = tid - band * Q;
    const uint32_t L = (uint32_t)g.L;
    const uint32_t R = (uint32_t)g.R;
    const uint32_t r0 = band * H;
    uint32_t z = 0, y0 = r0;
    if (D == 3) {
      z = fdiv(r0, divL);
      y0 = r0 - z * L;
    }
    int8_t* own = s + (int64_t)c * g.Nh;
    const int8_t* oth = s + (int64_t)(1 - c) * g.Nh;
    const uint32_t col = 16 * q;
    const uint32_t zrow = L * z;  // row index of (y = 0, z)
    const uint32_t qn = q + 1 == Q ? 0u : q + 1, qp = q == 0 ? Q - 1 : q - 1;
    // the in-row neighbour chunk's edge word: next chunk's word 0 (parity 1)
    // or previous chunk's word 3 (parity 0); parity alternates with y
    const uint32_t pz = (c + z) & 1u;
    const uint32_t edge_even = pz ? 16 * qn : 16 * qp + 12;  // rows with y even
    const uint32_t edge_odd = pz ? 16 * qp + 12 : 16 * qn;
    auto roff = [&](uint32_t y) -> uint32_t {  // y in [0, 2L)
      return (zrow + (y >= L ? y - L : y)) * R;
    };
    uint32_t zm_row = 0, zp_row = 0;
    if (D == 3) {
      zm_row = L * (z == 0 ? L - 1 : z - 1);
      zp_row = L * (z + 1 == L ? 0 : z + 1);
    }
    auto zoff = [&](uint32_t zr, uint32_t y) -> uint32_t { return (zr + (y >= L ? y - L : y)) * R + col; };
    const TabRegs tab = tab_regs(table);
    TieQueue tq;
    tq.slot = tie_slots + threadIdx.x;
    tq.stride = 256;
    tq.n = 0;
    tq.base = roff(y0) + col;
    tq.R = R;
    tq.dE = 0;
    tq.dM = 0;

    // Software pipeline: slot y & 3 of Ro holds the other colour's row y,
    // slot y & 1 of Ow / Ed / Fz / Bz our own row y, its edge word and its
    // z-neighbours.  A load is issued only into a slot whose row is dead and
    // is consumed at least one full row later, so no wait stalls the stream.
    Chunk Ro[4], Ow[2], Fz[2], Bz[2];
    uint32_t Ed[2];
    const uint32_t ym1 = y0 == 0 ? L - 1 : y0 - 1;
    Ro[3] = ld16(oth + roff(ym1) + col);
    Ro[0] = ld16(oth + roff(y0) + col);
    Ro[1] = ld16(oth + roff(y0 + 1) + col);
    Ro[2] = ld16(oth + roff(y0 + 2) + col);
    Ow[0] = ld16(own + roff(y0) + col);
    Ow[1] = ld16(own + roff(y0 + 1) + col);
    Ed[0] = *reinterpret_cast<const uint32_t*>(oth + roff(y0) + edge_even);
    Ed[1] = *reinterpret_cast<const uint32_t*>(oth + roff(y0 + 1) + edge_odd);
    if (D == 3) {
      Fz[0] = ld16(oth + zoff(zm_row, y0));
      Fz[1] = ld16(oth + zoff(zm_row, y0 + 1));
      Bz[0] = ld16(oth + zoff(zp_row, y0));
      Bz[1] = ld16(oth + zoff(zp_row, y0 + 1));
    }
    for (uint32_t i = 0; i < H; i += 4) {
#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const uint32_t y = y0 + i + ph;  // y0 and i are multiples of 4: y & 3 == ph
        const uint32_t p = (pz + ph) & 1u;
        const Chunk& up = Ro[(ph + 3) & 3];
        const Chunk& ct = Ro[ph];
        const Chunk& dn = Ro[(ph + 1) & 3];
        const Chunk& o = Ow[ph & 1];
        const uint32_t e = Ed[ph & 1];
        const Chunk sh = p ? shift_next(ct, e) : shift_prev(ct, e);
        const uint32_t jbase = roff(y) + col;
        uint32_t kk[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t ow = o.w[w];
          uint32_t k2 = ((ow ^ ct.w[w]) & kBit1) + ((ow ^ sh.w[w]) & kBit1) +
                        ((ow ^ up.w[w]) & kBit1) + ((ow ^ dn.w[w]) & kBit1);
          if (D == 3) k2 += ((ow ^ Fz[ph & 1].w[w]) & kBit1) + ((ow ^ Bz[ph & 1].w[w]) & kBit1);
          kk[w] = k2 >> 1;
        }
        // rare exact ties are queued and resolved at the end of the band
        const Chunk nc = update_chunk_deferred<D>(tab, key, t, c, jbase, i + ph, o, kk, tq, own);
        uint32_t nw[4] = {nc.w[0], nc.w[1], nc.w[2], nc.w[3]};
        st16(own + jbase, nw);
        if (MEASURE) {
          // colour 1 after its update: every bond has one colour-1 end, and the
          // colour-0 chunk at the same position covers each colour-0 site once
          uint32_t kn[4];
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            uint32_t k2 = ((nw[w] ^ ct.w[w]) & kBit1) + ((nw[w] ^ sh.w[w]) & kBit1) +
                          ((nw[w] ^ up.w[w]) & kBit1) + ((nw[w] ^ dn.w[w]) & kBit1);
            if (D == 3)
              k2 += ((nw[w] ^ Fz[ph & 1].w[w]) & kBit1) + ((nw[w] ^ Bz[ph & 1].w[w]) & kBit1);
            kn[w] = k2 >> 1;
          }
          Chunk nc;
          nc.w[0] = nw[0]; nc.w[1] = nw[1]; nc.w[2] = nw[2]; nc.w[3] = nw[3];
          Esum += -(int64_t)(16 * 2 * D) + 2 * (int64_t)chunk_count_sum(kn);
          Msum += chunk_spin_sum(nc) + chunk_spin_sum(ct);
        }
        // refill the dead slots: other row y + 3, own row y + 2 with its edge
        // word and z-neighbours (rows past the band are read, never used)
        Ro[(ph + 3) & 3] = ld16(oth + roff(y + 3) + col);
        Ow[ph & 1] = ld16(own + roff(y + 2) + col);
        Ed[ph & 1] = *reinterpret_cast<const uint32_t*>(oth + roff(y + 2) + ((ph & 1) ? edge_odd : edge_even));
        if (D == 3) {
          Fz[ph & 1] = ld16(oth + zoff(zm_row, y + 2));
          Bz[ph & 1] = ld16(oth + zoff(zp_row, y + 2));
        }
      }
    }
    // deferred ties: the site belongs to this lane's column of its own colour,
    // which no other lane of this launch touches
    tie_flush<D>(tq, tab, key, t, c, own);
    if (MEASURE) {
      Esum += tq.dE;
      Msum += tq.dM;
    }
  }
  if (MEASURE) block_partial_int(Esum, Msum, parts, blockIdx.x);
}

bool ising_chunk_supported(const Geom& g, int J_kind) {
  return J_kind != 2 && (g.L % 32) == 0;
}

// Four sites a lane wherever their loads are aligned, unless the one-site
// kernel is asked for by name.
template <int D>
static hipError_t launch_real(const IsingLaunch& a, int8_t* s, uint32_t t, uint32_t c, hipStream_t st,
                              void* partials = nullptr, int64_t* nparts = nullptr) {
  const bool four = a.variant != kVariantSite && a.g.R % 4 == 0 && ((uintptr_t)a.J & 15u) == 0u &&
                    ((uintptr_t)s & 3u) == 0u;
  const int64_t lanes = a.g.Nh / (four ? 4 : 1);
  const dim3 grid((unsigned)((lanes + 255) / 256));
  if (partials && nparts) *nparts = grid.x;
#define SMC_REAL(V, M)                                                                             \
  hipLaunchKernelGGL((ising_real_kernel<D, V, M>), grid, dim3(256), 0, st, a.g, a.key,             \
                     (const float*)a.J, a.beta, a.divR, a.divL, s, t, c, (Partial*)partials)
  if (four) { if (partials) SMC_REAL(4, true); else SMC_REAL(4, false); }
  else { if (partials) SMC_REAL(1, true); else SMC_REAL(1, false); }
#undef SMC_REAL
  return hipGetLastError();
}

template <int D>
static hipError_t launch_site(const IsingLaunch& a, int8_t* spins, uint32_t t, uint32_t c,
                              hipStream_t st, void* partials = nullptr, int64_t* nparts = nullptr) {
  if (a.J_kind == 2) return launch_real<D>(a, spins, t, c, st, partials, nparts);
  const dim3 grid((unsigned)((a.g.Nh + 255) / 256));
  if (partials && nparts) *nparts = grid.x;
#define SMC_SITE(JK, M)                                                                          \
  hipLaunchKernelGGL((ising_site_kernel<D, JK, M>), grid, dim3(256), 0, st, a.g, a.key, a.tab,   \
                     (const int8_t*)a.J, a.divR, a.divL, spins, t, c, a.heatbath, (Partial*)partials)
  if (a.J_kind == 0) { if (partials) SMC_SITE(0, true); else SMC_SITE(0, false); }
  else { if (partials) SMC_SITE(1, true); else SMC_SITE(1, false); }
#undef SMC_SITE
  return hipGetLastError();
}

template <int D>
static hipError_t launch_chunk(const IsingLaunch& a, int8_t* spins, uint32_t t, uint32_t c,
                               hipStream_t st, void* partials = nullptr, int64_t* nparts = nullptr) {
  const uint32_t nchunks = (uint32_t)(a.g.Nh >> 4);
  const dim3 grid((nchunks + 255) / 256);
  if (partials && nparts) *nparts = grid.x;
#define SMC_CHUNK(PM, M)                                                                         \
  hipLaunchKernelGGL((ising_chunk_kernel<D, PM, M>), grid, dim3(256), 0, st, a.g, a.key, a.tab,  \
                     (const int8_t*)a.J, a.divQ, a.divL, spins, t, c, (Partial*)partials)
  if (a.J_kind == 1) { if (partials) SMC_CHUNK(true, true); else SMC_CHUNK(true, false); }
  else { if (partials) SMC_CHUNK(false, true); else SMC_CHUNK(false, false); }
#undef SMC_CHUNK
  return hipGetLastError();
}

// Rows per band of the streaming kernel: the largest divisor of L up to 64
// that still gives at least `min_waves` waves.
uint32_t stream_rows_per_band(const Geom& g, uint32_t min_waves) {
  const uint32_t Q = (uint32_t)(g.R / 16);
  uint32_t best = 4;
  for (uint32_t H = 4; H <= 64; H *= 2) {  // the tie queue holds rows < 64
    if (g.L % H) break;
    const uint64_t waves = (uint64_t)Q * (uint64_t)(g.rows / H) / 64;
    if (waves >= min_waves) best = H;
  }
  return best;
}

template <int D>
static hipError_t launch_stream(const IsingLaunch& a, int8_t* spins, uint32_t t, uint32_t c,
                                hipStream_t st, void* partials = nullptr, int64_t* nparts = nullptr) {
  const uint32_t H = a.rows_per_band;
  const uint32_t nbands = (uint32_t)a.g.rows / H;
  const uint64_t threads = (uint64_t)nbands * a.divQ.d;
  const dim3 grid((unsigned)((threads + 255) / 256));
  if (partials) {
    hipLaunchKernelGGL((ising_stream_kernel<D, true>), grid, dim3(256), 0, st, a.g, a.key, a.tab,
                       a.divQ, a.divL, H, nbands, spins, t, c, (Partial*)partials);
    if (nparts) *nparts = grid.x;
  } else {
    hipLaunchKernelGGL((ising_stream_kernel<D, false>), grid, dim3(256), 0, st, a.g, a.key, a.tab,
                       a.divQ, a.divL, H, nbands, spins, t, c, (Partial*)nullptr);
  }
  return hipGetLastError();
}

int ising_variant_used(const IsingLaunch& a) {
  if (a.heatbath) return kVariantSite;  // the heat-bath rule runs on the site kernel
  int v = a.variant == kVariantFusedWave ? kVariantAuto : a.variant;
  const bool chunk_ok = ising_chunk_supported(a.g, a.J_kind);
  if (v == kVariantAuto) v = !chunk_ok ? kVariantSite : (a.J_kind == 0 ? kVariantStream : kVariantChunk);
  if (v == kVariantStream && !(chunk_ok && a.J_kind == 0 && a.rows_per_band >= 4 &&
                               a.rows_per_band % 4 == 0 && a.g.L % a.rows_per_band == 0))
    v = chunk_ok ? kVariantChunk : kVariantSite;
  if (v == kVariantChunk && !chunk_ok) v = kVariantSite;
  return v;
}

template <int D>
static hipError_t launch_half(const IsingLaunch& a, int8_t* spins, uint32_t t, uint32_t c, hipStream_t st,
                              void* partials = nullptr, int64_t* nparts = nullptr) {
  const int v = ising_variant_used(a);
  if (v == kVariantStream) return launch_stream<D>(a, spins, t, c, st, partials, nparts);
  if (v == kVariantChunk) return launch_chunk<D>(a, spins, t, c, st, partials, nparts);
  return launch_site<D>(a, spins, t, c, st, partials, nparts);
}

hipError_t launch_ising_half_sweep(const IsingLaunch& a, int8_t* spins, uint32_t t,
                                   uint32_t colour, hipStream_t st) {
  return a.g.d == 2 ? launch_half<2>(a, spins, t, colour, st) : launch_half<3>(a, spins, t, colour, st);
}

hipError_t ising_half_sweep_measured(const IsingLaunch& a, int8_t* spins, uint32_t t, void* partials,
                                     int64_t* nparts, hipStream_t st) {
  return a.g.d == 2 ? launch_half<2>(a, spins, t, 1u, st, partials, nparts)
                    : launch_half<3>(a, spins, t, 1u, st, partials, nparts);
}

}  // namespace smc
