// continuous.hip -- checkerboard Metropolis half-sweeps for XY (n = 2) and
// Heisenberg (n = 3) spins stored as FP32 unit vectors (Sec. 2: spins in
// single precision, aggregates in double).
//
// Proposal: XY rotates s by Delta = delta (2u - 1); Heisenberg picks a point
// uniformly on the spherical cap of half-angle theta_max around s (cos alpha
// = 1 - u (1 - cos theta_max), azimuth 2 pi u' in the frame e1 = normalised
// (e_k - s_k s) with k the component of smallest magnitude, e2 = s x e1).
// Acceptance (Eq. (2)): dE = -(s' - s) . h, accept iff dE <= 0 or
// u_acc < exp(-beta dE).  The random words come from Philox blocks keyed by
// (seed, t, replica, colour): XY block j>>1 words 2(j&1) (accept) and
// 2(j&1)+1 (proposal); Heisenberg block j words 0 (accept), 1, 2.  An XY
// thread updates the two sites of one block.
#include "chunk.hpp"
#include "reduce.hpp"
#include "spin_update.hpp"

namespace smc {

// One lane a Philox block: two sites of XY (j = 2 b, 2 b + 1, which an odd row
// length may put into two rows), one of Heisenberg.  Lanes run over the plane,
// not over its rows: a block of 256 lanes a row leaves most of them idle where
// L / 2 is not near a multiple of 256 (us a half-sweep, lanes of
// rows / of the plane: XY 3D L = 100 9.4 / 6.7, L = 138 19.4 / 13.8; Heisenberg
// 3D L = 90 7.9 / 5.0, L = 154 24.6 / 13.6).  What bounds it then is the address
// unit: 2 d + 1 loads a component and site.
//
// MEASURE (colour 1 only): the energy of the bonds of the updated sites and the
// magnetisation, as in the streaming kernel below; block sums go to
// parts[block].
template <int D, int N, int JK, bool FAST, bool MEASURE>
__global__ __launch_bounds__(256) void cont_site_kernel(
    const Geom g, const RngKey key, const void* __restrict__ J, const float J0, const float beta,
    const float param, const FastDiv divR, const FastDiv divL, float* __restrict__ s,
    const uint32_t t, const uint32_t c, const double J0d, Partial* __restrict__ parts) {
  constexpr int SPL = N == 2 ? 2 : 1;
  const uint32_t L = (uint32_t)g.L, R = (uint32_t)g.R;
  const int64_t Nh = g.Nh, Nfull = 2 * Nh;
  const uint32_t gid = xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  Partial part{0, 0, 0.0, {0.0, 0.0, 0.0}};
  if (gid < (uint32_t)(Nh / SPL)) {
    float* own = s + (int64_t)c * Nh;
    const float* oth = s + (int64_t)(1 - c) * Nh;
    uint32_t j = SPL * gid;
    uint32_t r = fdiv(j, divR);
    uint32_t jx = j - r * R;
    uint32_t z = D == 3 ? fdiv(r, divL) : 0u, y = r - z * L;
    const Rand4 rnd = philox(gid, t, key.replica, tag(c, kContinuous), key.k0, key.k1);
#pragma unroll
    for (int v = 0; v < SPL; ++v) {
      const uint32_t p = (c + y + z) & 1u;
      // x + 1 and x - 1: in-row indices jx + p and jx + p - 1 (periodic)
      uint32_t ip[3], im[3];
      ip[0] = jx + p == R ? j - jx : j + p;
      im[0] = jx + p == 0u ? j + R - 1u : j + p - 1u;
      ip[1] = y + 1u == L ? j - (L - 1u) * R : j + R;
      im[1] = y == 0u ? j + (L - 1u) * R : j - R;
      if (D == 3) {
        ip[2] = z + 1u == L ? j - (L - 1u) * L * R : j + L * R;
        im[2] = z == 0u ? j + (L - 1u) * L * R : j - L * R;
      }
      float nb[2 * D][N], sv[3] = {0.0f, 0.0f, 0.0f}, h[3] = {0.0f, 0.0f, 0.0f};
      float jb[2 * D];
#pragma unroll
      for (int mu = 0; mu < D; ++mu) {
        jb[2 * mu] = bond<JK>(J, J0, Nh, mu, c, j);
        jb[2 * mu + 1] = bond<JK>(J, J0, Nh, mu, 1 - c, im[mu]);
#pragma unroll
        for (int k = 0; k < N; ++k) {
          nb[2 * mu][k] = oth[k * Nfull + ip[mu]];
          nb[2 * mu + 1][k] = oth[k * Nfull + im[mu]];
        }
      }
#pragma unroll
      for (int k = 0; k < N; ++k) sv[k] = own[k * Nfull + j];
#pragma unroll
      for (int b = 0; b < 2 * D; ++b)
#pragma unroll
        for (int k = 0; k < N; ++k) h[k] += jb[b] * nb[b][k];
      bool accept;
      if (N == 2)
        accept = xy_update<FAST>(sv[0], sv[1], h, rnd.w[2 * v], rnd.w[2 * v + 1], beta,
                                 beta_log2e(beta), param);
      else
        accept = heis_update<FAST>(sv, h, rnd.w[0], rnd.w[1], rnd.w[2], beta, beta_log2e(beta), param);
      if (accept) {
#pragma unroll
        for (int k = 0; k < N; ++k) own[k * Nfull + j] = sv[k];
      }
      if (MEASURE) {
        double e = 0.0;
#pragma unroll
        for (int mu = 0; mu < D; ++mu) {
          double dp = 0.0, dm = 0.0;
#pragma unroll
          for (int k = 0; k < N; ++k) {
            dp += (double)sv[k] * (double)nb[2 * mu][k];
            dm += (double)sv[k] * (double)nb[2 * mu + 1][k];
          }
          double jp = J0d, jm = J0d;
          if (JK == 1) {
            const int8_t* Jb = (const int8_t*)J;
            jp = J0d * Jb[((int64_t)mu * 2 + 1) * Nh + j];
            jm = J0d * Jb[((int64_t)mu * 2 + 0) * Nh + im[mu]];
          } else if (JK == 2) {
            jp = (double)jb[2 * mu];
            jm = (double)jb[2 * mu + 1];
          }
          e -= jp * dp + jm * dm;
        }
        part.E += e;
#pragma unroll
        for (int k = 0; k < N; ++k) part.M[k] += (double)sv[k] + (double)oth[k * Nfull + j];
      }
      ++j;
      if (++jx == R) {
        jx = 0u;
        if (++y == L) {
          y = 0u;
          ++z;
        }
      }
    }
  }
  if (MEASURE) block_partial(part, parts);
}

// Streaming variant (the layout of the int8 streaming kernel with FP32
// components): a lane owns V consecutive in-row sites of one colour and walks
// a band of H plane rows at fixed z, keeping the other colour's rows y - 1,
// y, y + 1 (and the z-neighbour rows) in registers, so each row of either
// plane crosses HBM about once per half-sweep.  The x-neighbour beyond the
// lane's V sites (the "edge" element: the next group's first site for row
// parity 1, the previous group's last for parity 0) is one extra element per
// row and component.  Field order, random words and update arithmetic are
// those of the row kernels.  Requires R % V == 0, H % 4 == 0, L % H == 0.
// Plane accesses take a wave-uniform plane base and a 32-bit byte offset
// (planes below 4 GiB), which maps onto the scalar-base + vector-offset
// addressing of global loads and stores.
__device__ __forceinline__ const float* at(const float* base, uint32_t idx) {
  return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + (idx << 2));
}
__device__ __forceinline__ float* at(float* base, uint32_t idx) {
  return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + (idx << 2));
}
template <int V>
__device__ __forceinline__ void ldv(const float* base, uint32_t idx, float* o) {
  if (V == 4) {
    const float4 v = *reinterpret_cast<const float4*>(at(base, idx));
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  } else if (V == 1) {
    o[0] = *at(base, idx);
  } else {
    const float2 v = *reinterpret_cast<const float2*>(at(base, idx));
    o[0] = v.x; o[1] = v.y;
  }
}
template <int V>
__device__ __forceinline__ void stv(float* base, uint32_t idx, const float* o) {
  if (V == 4)
    *reinterpret_cast<float4*>(at(base, idx)) = make_float4(o[0], o[1], o[2], o[3]);
  else if (V == 1)
    *at(base, idx) = o[0];
  else
    *reinterpret_cast<float2*>(at(base, idx)) = make_float2(o[0], o[1]);
}

// MEASURE (colour 1 only): each lane also sums, in FP64, the energy of the
// bonds of its updated sites and the magnetisation of its sites plus the
// colour-0 sites at the same positions (the per-site formula of the
// measurement kernel); block sums go to parts[block].
// V sites per lane: XY 4 or 2 (a lane holds whole Philox blocks of two
// sites), Heisenberg 2 or 1.
template <int D, int N, int JK, bool FAST, bool MEASURE, int V>
__global__ __launch_bounds__(256) void cont_stream_kernel(
    const Geom g, const RngKey key, const void* __restrict__ J, const float J0, const float beta,
    const float param, const FastDiv divQ, const FastDiv divL, const uint32_t H,
    const uint32_t nbands, float* __restrict__ s, const uint32_t t, const uint32_t c,
    const double J0d, Partial* __restrict__ parts) {
  static_assert(N == 2 ? (V == 2 || V == 4) : (V == 1 || V == 2), "sites per lane");
  const float bl2e = beta_log2e(beta);
  const uint32_t tid = xcd_remap(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
  const uint32_t band = fdiv(tid, divQ);
  double Esum = 0.0, Msum[3] = {0.0, 0.0, 0.0};
  if (band < nbands) {
  const uint32_t Q = divQ.d;
  const uint32_t q = tid - band * Q;
  const uint32_t L = (uint32_t)g.L, R = (uint32_t)g.R;
  const uint32_t r0 = band * H;
  uint32_t z = 0, y0 = r0;
  if (D == 3) {
    z = fdiv(r0, divL);
    y0 = r0 - z * L;
  }
  const int64_t Nh = g.Nh, Nfull = 2 * Nh;
  float* own[N];
  const float* oth[N];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    own[m] = s + (int64_t)m * Nfull + (int64_t)c * Nh;
    oth[m] = s + (int64_t)m * Nfull + (int64_t)(1 - c) * Nh;
  }
  const uint32_t col = V * q;
  const uint32_t zrow = L * z;
  const uint32_t pz = (c + z) & 1u;  // row parity of y even
  const uint32_t e_next = q + 1 == Q ? 0u : col + V;
  const uint32_t e_prev = q == 0 ? R - 1 : col - 1;
  const uint32_t edge_even = pz ? e_next : e_prev;
  const uint32_t edge_odd = pz ? e_prev : e_next;
  auto roff = [&](uint32_t y) -> uint32_t { return (zrow + (y >= L ? y - L : y)) * R; };
  uint32_t zm_row = 0, zp_row = 0;
  if (D == 3) {
    zm_row = L * (z == 0 ? L - 1 : z - 1);
    zp_row = L * (z + 1 == L ? 0 : z + 1);
  }
  auto zoff = [&](uint32_t zr, uint32_t y) -> uint32_t {
    return (zr + (y >= L ? y - L : y)) * R + col;
  };
  // ring buffers as in the int8 streaming kernel: Ro[y & 3] other row y,
  // Ow / Ed / Fz / Bz [y & 1] own row y, its edge element, its z-neighbours
  float Ro[4][N][V], Ow[2][N][V], Ed[2][N], Fz[2][N][V], Bz[2][N][V];
  const uint32_t ym1 = y0 == 0 ? L - 1 : y0 - 1;
#pragma unroll
  for (int m = 0; m < N; ++m) {
    ldv<V>(oth[m], roff(ym1) + col, Ro[3][m]);
    ldv<V>(oth[m], roff(y0) + col, Ro[0][m]);
    ldv<V>(oth[m], roff(y0 + 1) + col, Ro[1][m]);
    ldv<V>(oth[m], roff(y0 + 2) + col, Ro[2][m]);
    ldv<V>(own[m], roff(y0) + col, Ow[0][m]);
    ldv<V>(own[m], roff(y0 + 1) + col, Ow[1][m]);
    Ed[0][m] = *at(oth[m], roff(y0) + edge_even);
    Ed[1][m] = *at(oth[m], roff(y0 + 1) + edge_odd);
    if (D == 3) {
      ldv<V>(oth[m], zoff(zm_row, y0), Fz[0][m]);
      ldv<V>(oth[m], zoff(zm_row, y0 + 1), Fz[1][m]);
      ldv<V>(oth[m], zoff(zp_row, y0), Bz[0][m]);
      ldv<V>(oth[m], zoff(zp_row, y0 + 1), Bz[1][m]);
    }
  }
  // 3D: plane offsets of the rows the loop touches, stepped by R per row (a
  // row past L - 1 wraps to row 0 of its z-plane) -- row y, y - 1, y + 2,
  // y + 3, and the z - 1 / z + 1 planes' rows y and y + 2 -- instead of a
  // multiply per row and stream (in 2D the running offsets cost more
  // registers than the multiplies cost issue slots)
  constexpr bool STEP = D == 3;
  const uint32_t zR = zrow * R, zmR = zm_row * R, zpR = zp_row * R;
  auto step = [&](uint32_t off, uint32_t yy, uint32_t base) -> uint32_t {
    return yy + 1 == L ? base : off + R;
  };
  uint32_t ry = roff(y0), rym = roff(ym1), ry2 = roff(y0 + 2), ry3 = roff(y0 + 3);
  uint32_t zm0 = zoff(zm_row, y0) - col, zm2 = zoff(zm_row, y0 + 2) - col;
  uint32_t zp2 = zoff(zp_row, y0 + 2) - col;
  for (uint32_t i = 0; i < H; i += 4) {
#pragma unroll
    for (int ph = 0; ph < 4; ++ph) {
      const uint32_t y = y0 + i + ph;  // y0 and i are multiples of 4
      const bool p = ((pz + (uint32_t)ph) & 1u) != 0;
      const uint32_t rowoff = STEP ? ry : roff(y);
      const uint32_t jrow = rowoff + col;
      const int up = (ph + 3) & 3, ct = ph, dn = (ph + 1) & 3, b = ph & 1;
      Rand4 rnd[N == 2 ? V / 2 : V];
#pragma unroll
      for (int k = 0; k < (N == 2 ? V / 2 : V); ++k)
        rnd[k] = philox(N == 2 ? (jrow >> 1) + k : jrow + k, t, key.replica, tag(c, kContinuous),
                        key.k0, key.k1);
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const uint32_t j = jrow + k;
        float h[3] = {0.0f, 0.0f, 0.0f};
        float jp = J0, jm = J0;
        // +x, -x
        if (JK != 0) {
          const uint32_t xm = p ? col + k : (k > 0 ? col + k - 1 : e_prev);
          jp = bond<JK>(J, J0, Nh, 0, c, j);
          jm = bond<JK>(J, J0, Nh, 0, 1 - c, rowoff + xm);
        }
#pragma unroll
        for (int m = 0; m < N; ++m) {
          const float vp = p ? (k + 1 < V ? Ro[ct][m][(k + 1) % V] : Ed[b][m]) : Ro[ct][m][k];
          h[m] += jp * vp;
        }
#pragma unroll
        for (int m = 0; m < N; ++m) {
          const float vm = p ? Ro[ct][m][k] : (k > 0 ? Ro[ct][m][(k + V - 1) % V] : Ed[b][m]);
          h[m] += jm * vm;
        }
        // +y, -y
        if (JK != 0) {
          jp = bond<JK>(J, J0, Nh, 1, c, j);
          jm = bond<JK>(J, J0, Nh, 1, 1 - c, (STEP ? rym : roff(y + L - 1)) + col + k);
        }
#pragma unroll
        for (int m = 0; m < N; ++m) h[m] += jp * Ro[dn][m][k];
#pragma unroll
        for (int m = 0; m < N; ++m) h[m] += jm * Ro[up][m][k];
        if (D == 3) {
          if (JK != 0) {
            jp = bond<JK>(J, J0, Nh, 2, c, j);
            jm = bond<JK>(J, J0, Nh, 2, 1 - c, zm0 + col + k);
          }
#pragma unroll
          for (int m = 0; m < N; ++m) h[m] += jp * Bz[b][m][k];
#pragma unroll
          for (int m = 0; m < N; ++m) h[m] += jm * Fz[b][m][k];
        }
        if (N == 2) {
          const Rand4& rw = rnd[k >> 1];
          xy_update<FAST>(Ow[b][0][k], Ow[b][1][k], h, (k & 1) ? rw.w[2] : rw.w[0],
                          (k & 1) ? rw.w[3] : rw.w[1], beta, bl2e, param);
        } else {
          float sv[3] = {Ow[b][0][k], Ow[b][1][k], Ow[b][2][k]};
          heis_update<FAST>(sv, h, rnd[k].w[0], rnd[k].w[1], rnd[k].w[2], beta, bl2e, param);
          Ow[b][0][k] = sv[0];
          Ow[b][1][k] = sv[1];
          Ow[b][2][k] = sv[2];
        }
      }
#pragma unroll
      for (int m = 0; m < N; ++m) stv<V>(own[m], jrow, Ow[b][m]);
      if (MEASURE) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
          const uint32_t j = jrow + k;
          double si[3] = {0.0, 0.0, 0.0};
#pragma unroll
          for (int m = 0; m < N; ++m) si[m] = (double)Ow[b][m][k];
          double e = 0.0;
#pragma unroll
          for (int mu = 0; mu < D; ++mu) {
            double dp = 0.0, dm = 0.0;
#pragma unroll
            for (int m = 0; m < N; ++m) {
              float vp, vm;
              if (mu == 0) {
                vp = p ? (k + 1 < V ? Ro[ct][m][(k + 1) % V] : Ed[b][m]) : Ro[ct][m][k];
                vm = p ? Ro[ct][m][k] : (k > 0 ? Ro[ct][m][(k + V - 1) % V] : Ed[b][m]);
              } else if (mu == 1) {
                vp = Ro[dn][m][k];
                vm = Ro[up][m][k];
              } else {
                vp = Bz[b][m][k];
                vm = Fz[b][m][k];
              }
              dp += si[m] * (double)vp;
              dm += si[m] * (double)vm;
            }
            double jp = J0d, jm = J0d;
            if (JK != 0) {
              uint32_t im;
              if (mu == 0) im = rowoff + (p ? col + k : (k > 0 ? col + k - 1 : e_prev));
              else if (mu == 1) im = (STEP ? rym : roff(y + L - 1)) + col + k;
              else im = zm0 + col + k;
              if (JK == 1) {
                const int8_t* Jb = (const int8_t*)J;
                jp = J0d * Jb[((int64_t)mu * 2 + 1) * Nh + j];
                jm = J0d * Jb[((int64_t)mu * 2 + 0) * Nh + im];
              } else {
                const float* Jf = (const float*)J;
                jp = Jf[((int64_t)mu * 2 + 1) * Nh + j];
                jm = Jf[((int64_t)mu * 2 + 0) * Nh + im];
              }
            }
            e -= jp * dp + jm * dm;
          }
          Esum += e;
#pragma unroll
          for (int m = 0; m < N; ++m) Msum[m] += si[m] + (double)Ro[ct][m][k];
        }
      }
      // refill the dead slots: other row y + 3, own row y + 2 with its edge
      // element and z-neighbours (rows past the band are read, never used)
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const uint32_t r3 = STEP ? ry3 : roff(y + 3), r2 = STEP ? ry2 : roff(y + 2);
        ldv<V>(oth[m], r3 + col, Ro[up][m]);
        ldv<V>(own[m], r2 + col, Ow[b][m]);
        Ed[b][m] = *at(oth[m], r2 + (b ? edge_odd : edge_even));
        if (D == 3) {
          ldv<V>(oth[m], zm2 + col, Fz[b][m]);
          ldv<V>(oth[m], zp2 + col, Bz[b][m]);
        }
      }
      rym = ry;
      ry = step(ry, y, zR);
      ry2 = ry3;
      ry3 = step(ry3, y + 3, zR);
      zm0 = step(zm0, y, zmR);
      zm2 = step(zm2, y + 2, zmR);
      zp2 = step(zp2, y + 2, zpR);
    }
  }
  }
  if (MEASURE) {
    Partial v{0, 0, Esum, {Msum[0], Msum[1], Msum[2]}};
    block_partial(v, parts);
  }
}

template <int D, int JK>
static hipError_t launch_cont_site(const ContLaunch& a, float* s, uint32_t t, uint32_t c,
                                   hipStream_t st, void* partials = nullptr,
                                   int64_t* nparts = nullptr) {
  const int64_t lanes = a.g.Nh / (a.n == 2 ? 2 : 1);
  const dim3 grid((unsigned)((lanes + 255) / 256));
  const float param = a.n == 2 ? a.delta : a.one_minus_cos_cap;
  if (partials && nparts) *nparts = grid.x;
#define SMC_CS(N, F, M)                                                                         \
  hipLaunchKernelGGL((cont_site_kernel<D, N, JK, F, M>), grid, dim3(256), 0, st, a.g, a.key, a.J, \
                     a.J0, a.beta, param, a.divR, a.divL, s, t, c, a.J0d, (Partial*)partials)
#define SMC_CSM(N)                                                                \
  do {                                                                            \
    if (partials) { if (a.fast_math) SMC_CS(N, true, true); else SMC_CS(N, false, true); } \
    else { if (a.fast_math) SMC_CS(N, true, false); else SMC_CS(N, false, false); }        \
  } while (0)
  if (a.n == 2) SMC_CSM(2); else SMC_CSM(3);
#undef SMC_CSM
#undef SMC_CS
  return hipGetLastError();
}

template <int D, int JK>
static hipError_t launch_cont_stream(const ContLaunch& a, float* s, uint32_t t, uint32_t c,
                                     hipStream_t st, void* partials = nullptr,
                                     int64_t* nparts = nullptr) {
  const uint32_t H = a.rows_per_band;
  const uint32_t nbands = (uint32_t)a.g.rows / H;
  const uint64_t threads = (uint64_t)nbands * a.divQ.d;
  const dim3 grid((unsigned)((threads + 255) / 256));
  const float param = a.n == 2 ? a.delta : a.one_minus_cos_cap;
  const bool meas = partials != nullptr;
  if (meas && nparts) *nparts = grid.x;
#define SMC_CS(N, F, M, V)                                                                         \
  hipLaunchKernelGGL((cont_stream_kernel<D, N, JK, F, M, V>), grid, dim3(256), 0, st, a.g, a.key,  \
                     a.J, a.J0, a.beta, param, a.divQ, a.divL, H, nbands, s, t, c, a.J0d,           \
                     (Partial*)partials)
#define SMC_CSV(N, V)                                                 \
  do {                                                                \
    if (meas) { if (a.fast_math) SMC_CS(N, true, true, V); else SMC_CS(N, false, true, V); } \
    else { if (a.fast_math) SMC_CS(N, true, false, V); else SMC_CS(N, false, false, V); }   \
  } while (0)
  if (a.n == 2) {
    if (a.sites_per_lane == 2) SMC_CSV(2, 2); else SMC_CSV(2, 4);
  } else {
    if (a.sites_per_lane == 1) SMC_CSV(3, 1); else SMC_CSV(3, 2);
  }
#undef SMC_CSV
#undef SMC_CS
  return hipGetLastError();
}

uint32_t cont_default_sites_per_lane(int n) { return n == 2 ? 4u : 2u; }

// The streaming kernel below some hundred thousand sites a colour leaves a SIMD few
// waves, each waiting on the loads that fill its ring: fewer sites a lane are
// more waves.  us a half-sweep: XY, 4 / 2 a lane: 2D L = 1000 5.8 / 5.0, 3D
// L = 64 5.7 / 4.6, L = 96 6.4 / 5.1, but 2D L = 2048 7.9 / 8.5, 3D L = 128
// 6.7 / 7.0; Heisenberg, 2 / 1 a lane at the best height: 3D L = 64 6.5 / 4.6,
// L = 128 9.4 / 8.3, L = 192 27.5 / 24.5, L = 256 52.9 / 50.3.  XY rows of an
// odd number of pairs take 2 where 4 do not divide them (2D L = 1500, else one
// site a lane: 11.9 / 7.4).
// With uniform or +-1 couplings 4 a lane are faster from 540000 sites a colour on in
// 3D, where a few more waves do not make up for the rows between the lanes (ten
// sweeps, 4 / 2 a lane: uniform L = 96 121 / 99, L = 104 128 / 131, L = 112 126 / 134, L = 120
// 135 / 144; +-1 L = 96 191 / 158, L = 104 200 / 220, L = 112 198 / 215), and from 950000 in
// 2D (uniform L = 1200 120 / 123, L = 1400 123 / 129, +-1 175 / 182; below, calls of sweeps run in
// bricks); FP32 couplings, a 16-byte load a bond and lane, stay with 2 (L = 112 236 / 224,
// 2D L = 1400 201 / 152).
uint32_t cont_sites_per_lane(const Geom& g, int n, int J_kind) {
  if (n == 3) return 1u;
  const int64_t least = J_kind == 2 ? 1 << 20 : g.d == 3 ? 540000 : 950000;
  return g.Nh >= least && g.R % 4 == 0 ? 4u : 2u;
}

// Smaller lattices still are done in less than the time of a launch by the
// one-site kernel, whose lanes wait on one round of loads.  us a half-sweep,
// one site / streaming: XY 2D L = 256 2.9 / 4.1, L = 512 3.1 / 4.2, L = 700 3.9 /
// 4.8, L = 1000 5.5 / 5.0; 3D L = 64 3.4 / 4.6, L = 96 6.5 / 5.1; Heisenberg 3D
// L = 64 3.1 / 4.6, L = 112 7.4 / 7.0, 2D L = 512 3.1 / 4.1, L = 1000 6.4 / 5.6.
bool cont_prefers_row(const Geom& g, int n) {
  return g.Nh < (n == 3 ? 250000 : g.d == 2 ? 350000 : 200000);
}

bool cont_sites_per_lane_ok(int n, uint32_t V) {
  return n == 2 ? (V == 2 || V == 4) : (V == 1 || V == 2);
}

bool cont_stream_supported(const Geom& g, uint32_t V, uint32_t H) {
  return V >= 1 && (uint32_t)g.R % V == 0 && H >= 4 && H % 4 == 0 && (uint32_t)g.L % H == 0 &&
         g.Nh < ((int64_t)1 << 30);  // 32-bit byte offsets within a plane
}

// Band height of the streaming kernel: the largest power of two up to 64 that
// divides L and still gives at least `min_waves` waves (1536: XY, H = 4 / 8 / 16 /
// 32, waves in brackets: 3D L = 192 18.3 (3456) / 15.8 (1728) / 18.2 / 33 us, L = 256
// 40.6 / 38.3 / 32.2 (2048) / 34.5 (1024); 2D L = 2600 16.1 (3300) / 14.8 (1650)).
uint32_t cont_rows_per_band(const Geom& g, uint32_t V, uint32_t min_waves) {
  const uint32_t Q = (uint32_t)g.R / V;
  uint32_t best = 4;
  // one site a lane (Heisenberg): taller bands lose more in waves than they
  // save in halo rows (3D L = 128, H = 4 / 8 / 16: 8.4 / 9.0 / 12.1 us, L = 256, H =
  // 4 / 8 / 16 / 32: 50 / 57 / 68 / 76), but for half as many partials where the
  // state is a few times the L2s (a measured sweep, H = 4 / 8: L = 144 32.3 / 30.0,
  // L = 160 41.0 / 38.7, L = 192 59.9 / 57.4)
  if (V == 1) return g.L % 8 == 0 && g.Nh >= 1400000 && g.Nh < 5000000 ? 8u : best;
  for (uint32_t H = 4; H <= 64; H *= 2) {
    if (g.L % H) break;
    const uint64_t waves = (uint64_t)Q * (uint64_t)(g.rows / H) / 64;
    if (waves >= min_waves) best = H;
  }
  return best;
}

int cont_variant_used(const ContLaunch& a) {
  if (a.variant == kContRow) return kContRow;
  return cont_stream_supported(a.g, a.sites_per_lane, a.rows_per_band) ? kContStream : kContRow;
}

template <int D>
static hipError_t launch_cont_d(const ContLaunch& a, float* s, uint32_t t, uint32_t c,
                                hipStream_t st) {
  const bool stream = cont_variant_used(a) == kContStream;
  switch (a.J_kind) {
    case 0: return stream ? launch_cont_stream<D, 0>(a, s, t, c, st) : launch_cont_site<D, 0>(a, s, t, c, st);
    case 1: return stream ? launch_cont_stream<D, 1>(a, s, t, c, st) : launch_cont_site<D, 1>(a, s, t, c, st);
    default: return stream ? launch_cont_stream<D, 2>(a, s, t, c, st) : launch_cont_site<D, 2>(a, s, t, c, st);
  }
}

hipError_t launch_cont_half_sweep(const ContLaunch& a, float* spins, uint32_t t, uint32_t colour,
                                  hipStream_t st) {
  return a.g.d == 2 ? launch_cont_d<2>(a, spins, t, colour, st)
                    : launch_cont_d<3>(a, spins, t, colour, st);
}

hipError_t cont_half_sweep_measured(const ContLaunch& a, float* spins, uint32_t t, void* partials,
                                    int64_t* nparts, hipStream_t st) {
  const bool stream = cont_variant_used(a) == kContStream;
#define SMC_CM(D, JK)                                                                     \
  (stream ? launch_cont_stream<D, JK>(a, spins, t, 1u, st, partials, nparts)              \
          : launch_cont_site<D, JK>(a, spins, t, 1u, st, partials, nparts))
  if (a.g.d == 2)
    return a.J_kind == 0 ? SMC_CM(2, 0) : a.J_kind == 1 ? SMC_CM(2, 1) : SMC_CM(2, 2);
    return a.J_kind == 0 ? SMC_CM(3, 0) : a.J_kind == 1 ? SMC_CM(3, 1) : SMC_CM(3, 2);
#undef SMC_CM
}

template <int N>
__global__ __launch_bounds__(256) void renorm_kernel(const int64_t Nfull, float* __restrict__ s) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= Nfull) return;
  float v[N];
  float q = 0.0f;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    v[k] = s[k * Nfull + i];
    q += v[k] * v[k];
  }
  const float inv = 1.0f / sqrtf(q);
#pragma unroll
  for (int k = 0; k < N; ++k) s[k * Nfull + i] = v[k] * inv;
}

hipError_t launch_renormalize(const Geom& g, int n, float* spins, hipStream_t st) {
  const int64_t Nfull = 2 * g.Nh;
  const dim3 grid((unsigned)((Nfull + 255) / 256));
  if (n == 2)
    hipLaunchKernelGGL(renorm_kernel<2>, grid, dim3(256), 0, st, Nfull, spins);
  else
    hipLaunchKernelGGL(renorm_kernel<3>, grid, dim3(256), 0, st, Nfull, spins);
  return hipGetLastError();
}

}  // namespace smc
