// march.hip -- two sweeps of a large 2D XY lattice in one pass over memory.
//
// A half-sweep in place moves 24 N bytes a sweep (both planes read, one written,
// twice) for 84 vector instructions a site: at L = 4096, where the state sits in
// the last-level cache, that is 402 MB a sweep at about 6 TB/s, 67 us, of which
// the instructions would take 36.  Here a wave marches down a band of rows with
// K = 4 half-sweeps in flight a row apart -- colour 0 of row r - 1, colour 1 of
// row r - 2, colour 0 of r - 3, colour 1 of r - 4 -- on rows it keeps in registers,
// so the state crosses memory once a pass (from one buffer to the other: rows
// around a band are read by its neighbours' waves too).
//
// A lane holds four in-row sites of both colours; the site beyond them is the
// next lane's (a DPP move).  A wave's first and last lane repeat their
// neighbours' work (a half-sweep spoils one site from the edge: four of them,
// one lane), and so do K - 1 - s rows above and below the band at half-sweep s.
// Field, draws and arithmetic are the streaming kernel's: the same bits.
//
// us for ten measured sweeps, half-sweeps in place / here: L = 4096 675 / 533, L =
// 3104 440 / 359, L = 3000 425 / 345, L = 8192 3125 / 1765 (from HBM); at L = 2048 the state sits in the L2s and the
// half-sweeps take 162, here 257.  Vector issue bounds it at two waves a SIMD: 84
// instructions a site, a seventh more for the edge lanes and a tenth for the rows
// around a band.
#include "chunk.hpp"
#include "kernels.hpp"
#include "reduce.hpp"
#include "spin_update.hpp"

#include <algorithm>
#include <type_traits>

namespace smc {

template <int K, bool MEASURE>
__global__ __launch_bounds__(64) void xy_march_kernel(const Geom g, const RngKey key, const float J0,
                                                      const float beta, const float delta,
                                                      const double J0d, const uint32_t segs,
                                                      const uint32_t bands, const float* __restrict__ src,
                                                      float* __restrict__ dst, const uint32_t t0,
                                                      Partial* __restrict__ parts) {
  constexpr int W = K + 2;  // rows in flight: r, r - 1, .., r - K - 1
  const int32_t L = g.L, R = g.R;
  const uint32_t Q = (uint32_t)R / 4u;
  const int64_t Nh = g.Nh, Nfull = 2 * Nh;
  const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t band = b / segs, seg = b - band * segs, lane = threadIdx.x;
  const uint32_t q0 = (uint32_t)((uint64_t)Q * seg / segs), q1 = (uint32_t)((uint64_t)Q * (seg + 1u) / segs);
  uint32_t q = q0 + lane + Q - 1u;  // lane 0: the group before the segment's first
  q = q >= Q ? q - Q : q;
  q = q >= Q ? q - Q : q;
  const bool own = lane >= 1u && lane <= q1 - q0;
  const uint32_t col = 4u * q;
  // rows y0 .. y1 - 1, both even
  const int32_t y0 = 2 * (int32_t)((uint64_t)(L / 2) * band / bands);
  const int32_t y1 = 2 * (int32_t)((uint64_t)(L / 2) * (band + 1u) / bands);
  const float bl2e = beta_log2e(beta);
  float s[2][W][2][4];  // [colour][rows back][component][site]
  float nx[2][2][4];    // the next row
  double Esum = 0.0, Msum[2] = {0.0, 0.0};
  auto offset = [&](int32_t r) -> uint32_t {
    const int32_t y = r < 0 ? r + L : r >= L ? r - L : r;
    return (uint32_t)y * (uint32_t)R + col;
  };
  auto load = [&](int32_t r) {
    const uint32_t o = offset(r);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const float4 v = *reinterpret_cast<const float4*>(src + m * Nfull + c * Nh + o);
        nx[c][m][0] = v.x; nx[c][m][1] = v.y; nx[c][m][2] = v.z; nx[c][m][3] = v.w;
      }
  };
  // row r arrives; half-sweep k of row r - 1 - k for all k; row r - K leaves
  auto row = [&](int32_t r, auto P) {
    constexpr bool p = !decltype(P)::value;  // (colour + row) odd, for every half-sweep
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
          for (int k = W - 1; k > 0; --k) s[c][k][m][v] = s[c][k - 1][m][v];
          s[c][0][m][v] = nx[c][m][v];
        }
    if (r + 1 < y1 + K) load(r + 1);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int32_t y = r - 1 - k;
      if (y >= y0 - (K - 1 - k) && y < y1 + (K - 1 - k)) {
        const int c = k & 1;
        float(&o)[2][4] = s[c][1 + k];
        const float(&ct)[2][4] = s[1 - c][1 + k];
        const float(&up)[2][4] = s[1 - c][2 + k];
        const float(&dn)[2][4] = s[1 - c][k];
        float e[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          // wave_shl / wave_shr by one lane: the next lane's first, the previous one's last
          const int x = __float_as_int(p ? ct[m][0] : ct[m][3]);
          e[m] = __int_as_float(p ? __builtin_amdgcn_update_dpp(x, x, 0x130, 0xF, 0xF, false)
                                  : __builtin_amdgcn_update_dpp(x, x, 0x138, 0xF, 0xF, false));
        }
        const uint32_t blk = offset(y) >> 1;
        Rand4 rnd[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          rnd[u] = philox(blk + u, t0 + (uint32_t)(k >> 1), key.replica, tag((uint32_t)c, kContinuous),
                          key.k0, key.k1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float h[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int m = 0; m < 2; ++m) h[m] += J0 * (p ? (v < 3 ? ct[m][(v + 1) & 3] : e[m]) : ct[m][v]);
#pragma unroll
          for (int m = 0; m < 2; ++m) h[m] += J0 * (p ? ct[m][v] : (v > 0 ? ct[m][(v + 3) & 3] : e[m]));
#pragma unroll
          for (int m = 0; m < 2; ++m) h[m] += J0 * dn[m][v];
#pragma unroll
          for (int m = 0; m < 2; ++m) h[m] += J0 * up[m][v];
          const Rand4& rw = rnd[v >> 1];
          xy_update<false>(o[0][v], o[1][v], h, (v & 1) ? rw.w[2] : rw.w[0], (v & 1) ? rw.w[3] : rw.w[1],
                           beta, bl2e, delta);
          if (MEASURE && k == K - 1 && own) {
            double dp = 0.0;
            double bonds[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int m = 0; m < 2; ++m) {
              const double sm = (double)o[m][v];
              bonds[0] += sm * (double)(p ? (v < 3 ? ct[m][(v + 1) & 3] : e[m]) : ct[m][v]);
              bonds[1] += sm * (double)(p ? ct[m][v] : (v > 0 ? ct[m][(v + 3) & 3] : e[m]));
              bonds[2] += sm * (double)dn[m][v];
              bonds[3] += sm * (double)up[m][v];
              Msum[m] += sm + (double)ct[m][v];
            }
            dp -= J0d * bonds[0] + J0d * bonds[1];
            dp -= J0d * bonds[2] + J0d * bonds[3];
            Esum += dp;
          }
        }
      }
    }
    const int32_t y = r - K;
    if (own && y >= y0 && y < y1) {
      const uint32_t o = offset(y);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int m = 0; m < 2; ++m)
          *reinterpret_cast<float4*>(dst + m * Nfull + c * Nh + o) =
              make_float4(s[c][K][m][0], s[c][K][m][1], s[c][K][m][2], s[c][K][m][3]);
    }
  };
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int k = 0; k < W; ++k)
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) s[c][k][m][v] = 0.0f;
  load(y0 - K);
#pragma unroll 1
  for (int32_t r = y0 - K; r < y1 + K; r += 2) {
    row(r, std::integral_constant<bool, false>());
    row(r + 1, std::integral_constant<bool, true>());
  }
  if (MEASURE) {
    Partial v{0, 0, Esum, {Msum[0], Msum[1], 0.0}};
    v = block_sum(v);
    if (lane == 0u) parts[blockIdx.x] = v;
  }
}

bool xy_march_supported(const Geom& g) {
  return g.d == 2 && g.R % 4 == 0 && g.R >= 256 && g.Nh < ((int64_t)1 << 30);
}

// Rows of a band for the least time of ten sweeps, or 0 where half-sweeps in
// place take less.  A wave's time goes with 4 H + 12 rows' half-sweeps and the
// waves of the fullest SIMD share it: 2.95 us for each (a wave alone waits on
// itself: 4).  Fits L = 3000 to 4096 and H = 8 to 64 within 6 %: L = 4096 H = 12 /
// 18 / 24 / 36 525 / 514 / 627 / 626.  In place a half-sweep takes 4.6 us + N /
// 0.6e6 from L = 2600 on (328 / 272; L = 2400 takes 244 in place and 7.7 us a half-sweep at L =
// 2048, where the L2s hold the state).
uint32_t xy_march_rows(const Geom& g) {
  if (!xy_march_supported(g) || g.Nh < 3000000) return 0u;
  const uint32_t segs = ((uint32_t)g.R / 4u + 61u) / 62u;
  double best = 0.95 * 20.0 * (4.6 + 2.0 * (double)g.Nh / 0.6e6);
  uint32_t rows = 0;
  for (uint32_t H = 6; H <= 256; H += 2) {
    const uint32_t bands = (uint32_t)g.L / H, tall = ((uint32_t)g.L / 2 + bands - 1) / bands * 2;
    const uint32_t waves = (segs * bands + 1023u) / 1024u;
    const double us = waves * (4.0 * tall + 12.0) * (waves == 1 ? 4.0 : 2.95);
    if (us < best) {
      best = us;
      rows = H;
    }
  }
  return rows;
}

hipError_t launch_xy_march(const ContLaunch& a, int sweeps, uint32_t rows, const float* src, float* dst,
                           uint32_t t0, void* partials, int64_t* nparts, hipStream_t st) {
  const uint32_t Q = (uint32_t)a.g.R / 4u, segs = (Q + 61u) / 62u;
  const uint32_t bands = std::max(1u, (uint32_t)a.g.L / rows);
  const dim3 grid(segs * bands), block(64);
  if (partials && nparts) *nparts = grid.x;
#define SMC_MARCH(K, M)                                                                           \
  hipLaunchKernelGGL((xy_march_kernel<K, M>), grid, block, 0, st, a.g, a.key, a.J0, a.beta, a.delta, \
                     a.J0d, segs, bands, src, dst, t0, (Partial*)partials)
  if (sweeps == 2) { if (partials) SMC_MARCH(4, true); else SMC_MARCH(4, false); }
  else { if (partials) SMC_MARCH(2, true); else SMC_MARCH(2, false); }
#undef SMC_MARCH
  return hipGetLastError();
}

}  // namespace smc
