// brick.hip -- several sweeps in one launch for lattices whose updates are real
// valued: Ising spins with FP32 couplings, XY and Heisenberg spins.
//
// A half-sweep of a small lattice costs a launch (3.5 - 4 us) for less than a
// microsecond of work.  Here a workgroup loads a brick of the lattice with a
// halo as deep as the half-sweeps it will run, keeps the spins in LDS, and
// steps through all of them with a barrier each; what it computes in the halo
// is thrown away (its neighbours compute the same from the same counters).  A
// lattice that fits one workgroup needs no halo and runs a whole call, its
// measurement included.
//
// A position is a pair of sites (0, j), (1, j): the two planes have the same
// layout, so a position's in-row index, row and neighbours serve both colours.
// A lane holds V consecutive positions of a row, their neighbours' LDS
// addresses and their 2 d couplings of both colours in registers, so a step
// reads spins only (LDS) and draws.  Sites whose neighbours the steps before
// have spoiled are left out: a site at distance e of the nearest cut face, in
// sites, is right after steps 0 .. e - 1.
//
// What bounds it: a step takes 0.35 - 0.9 us however small (one lane's draw,
// proposal and exponential in turn, and a barrier), the launch 2 us before the
// first; where a SIMD has three waves or more, their issue slots.  us a
// half-sweep, launches of single half-sweeps / bricks: FP32 couplings 2D L = 32
// 2.4 / 0.42 (one workgroup), L = 256 2.8 / 0.69 (four sweeps a launch, 256
// bricks of 8 x 16 positions), L = 1000 3.2 / 1.9, 3D L = 40 2.8 / 2.2; XY 2D
// L = 256 2.8 / 0.80; Heisenberg 3D L = 40 3.9 / 2.6.
// V = 1 leaves a SIMD the most waves and is fastest where a brick fits 1024
// lanes; V = 2 and 4 share a Philox block between sites and hold larger bricks
// (2D L = 1000, two sweeps a
// launch: 2.3 us with 2 in 16 x 32 bricks, 3.2 with 1 in 20 x 40).
//
// The arithmetic, the field's order and the random words are those of the
// one-site kernels, so the chain is the same bit for bit.
#include "chunk.hpp"
#include "kernels.hpp"
#include "reduce.hpp"
#include "spin_update.hpp"

namespace smc {

template <int D, int N, int JK, int V>
__global__ __launch_bounds__(1024) void brick_kernel(const BrickLaunch a) {
  extern __shared__ float sp[];  // [N][2][positions]
  const uint32_t L = (uint32_t)a.g.L, R = (uint32_t)a.g.R;
  const int64_t Nh = a.g.Nh, Nfull = 2 * Nh;
  const uint32_t K = a.steps;
  const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t bx = b % a.nb[0], byz = b / a.nb[0];
  const uint32_t by = D == 3 ? byz % a.nb[1] : byz, bz = D == 3 ? byz / a.nb[1] : 0u;
  // owned ranges (x in positions) and the local extents with the halos
  const bool wx = a.nb[0] == 1u, wy = a.nb[1] == 1u, wz = D == 2 || a.nb[2] == 1u;
  const uint32_t x0 = R / V * bx / a.nb[0] * V, nx = R / V * (bx + 1u) / a.nb[0] * V - x0;
  const uint32_t y0 = L * by / a.nb[1], ny = L * (by + 1u) / a.nb[1] - y0;
  const uint32_t z0 = D == 3 ? L * bz / a.nb[2] : 0u, nz = D == 3 ? L * (bz + 1u) / a.nb[2] - z0 : 1u;
  const uint32_t hx = wx ? 0u : a.halo_x, hy = wy ? 0u : K, hz = wz ? 0u : K;
  const uint32_t W = nx + 2u * hx, H = ny + 2u * hy, Z = nz + 2u * hz, P = W * H * Z;
  const uint32_t i = threadIdx.x * V;  // first position of the lane
  const bool in = i < P;
  const uint32_t row = i / W, lx = i - row * W;
  const uint32_t lz = D == 3 ? row / H : 0u, ly = row - lz * H;
  auto global = [](uint32_t l, uint32_t o, uint32_t h, uint32_t n) -> uint32_t {
    const uint32_t v = o + l + n - h;  // halos are at most the edge
    return v >= 2u * n ? v - 2u * n : v >= n ? v - n : v;
  };
  const uint32_t gx = global(lx, x0, hx, R), gy = global(ly, y0, hy, L);
  const uint32_t gz = D == 3 ? global(lz, z0, hz, L) : 0u;
  const uint32_t j = in ? (gz * L + gy) * R + gx : 0u;
  const uint32_t q = (gy + gz) & 1u;  // row parity of colour 0
  // LDS addresses of the neighbours; at a cut face the site itself (not used)
  const uint32_t oL = lx == 0u ? (wx ? i + W - 1u : i) : i - 1u;
  const uint32_t oR = lx + V >= W ? (wx ? i + V - W : i + V - 1u) : i + V;
  const uint32_t oym = ly == 0u ? (wy ? i + (H - 1u) * W : i) : i - W;
  const uint32_t oyp = ly + 1u == H ? (wy ? i - (H - 1u) * W : i) : i + W;
  uint32_t ozm = i, ozp = i;
  if (D == 3) {
    ozm = lz == 0u ? (wz ? i + (Z - 1u) * H * W : i) : i - H * W;
    ozp = lz + 1u == Z ? (wz ? i - (Z - 1u) * H * W : i) : i + H * W;
  }
  uint32_t e = in ? ~0u : 0u;  // (no cut face: right after every step of a call)
  if (in && !wx) e = min(e, 2u * min(lx + V, W - lx) - 1u);  // of its innermost site
  if (in && !wy) e = min(e, min(ly, H - 1u - ly));
  if (in && !wz) e = min(e, min(lz, Z - 1u - lz));

  // ---- spins to LDS, couplings to registers ----
  float jr[2][V][2 * D];
  if (in) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int m = 0; m < N; ++m)
#pragma unroll
        for (int v = 0; v < V; ++v)
          sp[(2 * m + c) * P + i + v] =
              N == 1 ? (float)((const int8_t*)a.src)[(uint32_t)c * Nh + j + v]
                     : ((const float*)a.src)[m * Nfull + c * Nh + j + v];
      if (JK != 0) {
        const bool p = ((q + (uint32_t)c) & 1u) != 0u;
        const uint32_t jym = gy == 0u ? j + (L - 1u) * R : j - R;
        const uint32_t jzm = gz == 0u ? j + (L - 1u) * L * R : j - L * R;
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const uint32_t xm = p ? j + v : v > 0 ? j + v - 1u : gx == 0u ? j + R - 1u : j - 1u;
#pragma unroll
          for (int mu = 0; mu < D; ++mu) {
            // +-1 couplings without J0: the field and the energy scale them in
            // FP32 and FP64
            jr[c][v][2 * mu] = bond<JK>(a.J, 1.0f, Nh, mu, c, j + v);
            jr[c][v][2 * mu + 1] =
                bond<JK>(a.J, 1.0f, Nh, mu, 1 - c, mu == 0 ? xm : mu == 1 ? jym + v : jzm + v);
          }
        }
      }
    }
  }
  __syncthreads();

  // value k of the 2 D neighbours of position i + v, colour c, component m
  auto nbr = [&](int c, int v, int m, int k) -> float {
    const float* o = sp + (2 * m + 1 - c) * P;
    const bool p = ((q + (uint32_t)c) & 1u) != 0u;
    switch (k) {
      case 0: return o[p ? (v + 1 < V ? i + v + 1u : oR) : i + v];
      case 1: return o[p ? i + v : (v > 0 ? i + v - 1u : oL)];
      case 2: return o[oyp + v];
      case 3: return o[oym + v];
      case 4: return o[ozp + v];
      default: return o[ozm + v];
    }
  };
  const float bl2e = beta_log2e(a.beta);
  auto step = [&](auto C, uint32_t k, uint32_t t) {
    constexpr int c = decltype(C)::value;
    if (k < e) {
      constexpr int kDraws = N == 3 ? V : N == 2 && V > 2 ? V / 2 : 1;
      Rand4 rnd[kDraws];
#pragma unroll
      for (int r = 0; r < kDraws; ++r)
        rnd[r] = philox(N == 3 ? j + r : N == 2 ? (j >> 1) + r : j >> 2, t, a.key.replica,
                        tag(c, kContinuous), a.key.k0, a.key.k1);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        float h[3] = {0.0f, 0.0f, 0.0f}, s[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int m = 0; m < N; ++m) s[m] = sp[(2 * m + c) * P + i + v];
#pragma unroll
        for (int b2 = 0; b2 < 2 * D; ++b2) {
          const float jb = JK == 0 ? a.J0 : JK == 1 ? a.J0 * jr[c][v][b2] : jr[c][v][b2];
#pragma unroll
          for (int m = 0; m < N; ++m) h[m] += jb * nbr(c, v, m, b2);
        }
        bool accept;
        if (N == 1) {
          const float dE = 2.0f * s[0] * h[0];
          const uint32_t w = V == 4 ? rnd[0].w[v] : pick4(rnd[0], (j + v) & 3u);
          accept = metropolis_fp32(dE, u01f(w), bl2e);
          s[0] = -s[0];
        } else if (N == 2) {
          const Rand4& rw = rnd[V > 2 ? v >> 1 : 0];
          const bool odd = V == 1 ? (j & 1u) != 0u : (v & 1) != 0;
          accept = xy_update<false>(s[0], s[1], h, odd ? rw.w[2] : rw.w[0], odd ? rw.w[3] : rw.w[1],
                                    a.beta, bl2e, a.param);
        } else {
          const Rand4& rw = rnd[N == 3 ? v : 0];
          accept = heis_update<false>(s, h, rw.w[0], rw.w[1], rw.w[2], a.beta, bl2e, a.param);
        }
        if (accept) {
#pragma unroll
          for (int m = 0; m < N; ++m) sp[(2 * m + c) * P + i + v] = s[m];
        }
      }
    }
    __syncthreads();
  };
#pragma unroll 1
  for (uint32_t k = 0; k < K; k += 2u) {
    step(std::integral_constant<int, 0>(), k, a.t0 + (k >> 1));
    step(std::integral_constant<int, 1>(), k + 1u, a.t0 + (k >> 1));
  }

  // ---- the owned positions go back ----
  const bool own = in && lx - hx < nx && ly - hy < ny && lz - hz < nz;
  const bool measure = a.parts != nullptr || a.obs != nullptr;
  Partial part{0, 0, 0.0, {0.0, 0.0, 0.0}};
  if (own) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int m = 0; m < N; ++m)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const float s = sp[(2 * m + c) * P + i + v];
          if (N == 1) ((int8_t*)a.dst)[(uint32_t)c * Nh + j + v] = (int8_t)s;
          else ((float*)a.dst)[m * Nfull + c * Nh + j + v] = s;
        }
    if (measure) {  // every bond has one colour-1 end
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double s[3] = {0.0, 0.0, 0.0}, en = 0.0;
#pragma unroll
        for (int m = 0; m < N; ++m) s[m] = (double)sp[(2 * m + 1) * P + i + v];
#pragma unroll
        for (int mu = 0; mu < D; ++mu) {
          double dp = 0.0, dm = 0.0;
#pragma unroll
          for (int m = 0; m < N; ++m) {
            dp += s[m] * (double)nbr(1, v, m, 2 * mu);
            dm += s[m] * (double)nbr(1, v, m, 2 * mu + 1);
          }
          double jp = a.J0d, jm = a.J0d;
          if (JK != 0) {
            jp = (double)jr[1][v][2 * mu] * (JK == 1 ? a.J0d : 1.0);
            jm = (double)jr[1][v][2 * mu + 1] * (JK == 1 ? a.J0d : 1.0);
          }
          en -= jp * dp + jm * dm;
        }
        part.E += en;
        if (N == 1) part.Mi += (int64_t)(s[0] + (double)sp[i + v]);
        else
#pragma unroll
          for (int m = 0; m < N; ++m) part.M[m] += s[m] + (double)sp[2 * m * P + i + v];
      }
    }
  }
  if (!measure) return;
  part = block_sum(part);
  if (threadIdx.x != 0u) return;
  if (a.parts) ((Partial*)a.parts)[blockIdx.x] = part;
  else write_obs(part, N == 1, false, a.J0d, a.sweep, (ObsOut*)a.obs);
}

size_t brick_lds_bytes(int n, uint32_t positions) { return (size_t)n * 2 * 4 * positions; }

template <int D, int N, int JK>
static hipError_t launch_brick_v(const BrickLaunch& a, hipStream_t st) {
  const dim3 grid(a.nb[0] * a.nb[1] * (D == 3 ? a.nb[2] : 1u));
  const dim3 block((a.positions / a.V + 63u) / 64u * 64u);
  const size_t lds = brick_lds_bytes(N, a.positions);
  switch (a.V) {
    case 1: hipLaunchKernelGGL((brick_kernel<D, N, JK, 1>), grid, block, lds, st, a); break;
    case 2: hipLaunchKernelGGL((brick_kernel<D, N, JK, 2>), grid, block, lds, st, a); break;
    default: hipLaunchKernelGGL((brick_kernel<D, N, JK, 4>), grid, block, lds, st, a); break;
  }
  return hipGetLastError();
}

template <int D>
static hipError_t launch_brick_d(const BrickLaunch& a, hipStream_t st) {
  if (a.n == 1) return launch_brick_v<D, 1, 2>(a, st);
  switch (a.n * 3 + a.J_kind) {
    case 6: return launch_brick_v<D, 2, 0>(a, st);
    case 7: return launch_brick_v<D, 2, 1>(a, st);
    case 8: return launch_brick_v<D, 2, 2>(a, st);
    case 9: return launch_brick_v<D, 3, 0>(a, st);
    case 10: return launch_brick_v<D, 3, 1>(a, st);
    default: return launch_brick_v<D, 3, 2>(a, st);
  }
}

hipError_t launch_brick(const BrickLaunch& a, hipStream_t st) {
  return a.g.d == 2 ? launch_brick_d<2>(a, st) : launch_brick_d<3>(a, st);
}

}  // namespace smc
