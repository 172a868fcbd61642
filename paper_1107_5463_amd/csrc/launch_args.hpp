// launch_args.hpp -- the argument structures the libsmc kernels receive
// (internal).  Kept apart from the launchers' declarations (kernels.hpp): a
// kernel's code depends on these layouts, not on the host-side function list.
#pragma once

#include <stdint.h>

#include "device.hpp"

namespace smc {

struct RngKey {
  uint32_t k0, k1;   // seed low / high word
  uint32_t replica;  // counter word 2
};

// Exact unsigned 32-bit division by a runtime constant (Granlund-Montgomery):
// q = (hi + ((n - hi) >> 1)) >> (l - 1) with hi = umulhi(m, n).
struct FastDiv {
  uint32_t d, m, s;
};

enum IsingVariant { kVariantAuto = 0, kVariantSite = 1, kVariantChunk = 2, kVariantStream = 3,
                    kVariantFusedWave = 4 };  // fused schedule: wave-segment kernel (no barriers)

struct IsingLaunch {
  Geom g;
  RngKey key;
  IsingTable tab;    // integer thresholds (uniform and +-1 couplings)
  int J_kind;        // 0 uniform, 1 +-1 int8, 2 FP32
  const void* J;     // [d][2][N/2] or null
  float beta;        // FP32 couplings only
  int variant;       // IsingVariant
  uint32_t rows_per_band;  // streaming kernel: rows walked by one lane (divides L)
  int heatbath;      // rule: 0 Metropolis, 1 heat bath (table holds p_+ thresholds)
  int packed_ties;   // bit-packed kernels' exact ties: 0 resolved by the workgroup, 1 by each
                     // lane, 2 by the workgroup's fallback (tied words numbered per wave;
                     // the tile kernels: each lane)
  FastDiv divQ;      // chunks per plane row
  FastDiv divL;      // edge length
  FastDiv divR;      // plane row length
};

// Several half-sweeps of one Ising lattice with its words in LDS (resident.hip).
struct ResidentLaunch {
  Geom g;
  RngKey key;
  uint32_t th[7];      // threshold byte T >> 24 of each class with a mask
  uint32_t frac[7];    // T & 0xFFFFFF (2^24: accepts on every draw)
  uint32_t invert;     // ~0: count satisfied bonds (Metropolis with J0 < 0)
  uint32_t Wp;         // 32-site words of a colour plane
  uint32_t t0;         // sweep counter of step 0 of the call
  uint32_t step0;      // first half-sweep of this launch (of the call); its parity is the colour
  uint32_t steps;      // half-sweeps of this launch
  uint32_t own;        // words of a colour a workgroup owns
  uint32_t rho;        // words of halo a half-sweep uses up (0: the whole lattice is local)
  uint32_t halo;       // rho * steps
  uint32_t chunk;      // half-sweeps whose masks are formed together
  uint32_t mask_words; // capacity of a class's masks
  uint32_t src_bytes, dst_bytes;  // 1: int8 planes, 0: words
  const void* src;
  void* dst;
  const uint32_t* bonds;  // bond-sign words (+-1 couplings) or null
  const uint32_t* drawn;  // masks of the call's steps from memory, or null: formed in the kernel;
  uint64_t drawn_stride;  // class q's of step k at q drawn_stride + k Wp
  void* parts;         // reduction partials of the final state (several workgroups), or null
  void* obs;           // its record (one workgroup), or null
  double J0;
  int64_t sweep;
};

struct ContLaunch {
  Geom g;
  int n;             // 2 or 3
  RngKey key;
  int J_kind;
  float J0;
  const void* J;
  float beta;
  float delta;       // XY max angle
  float one_minus_cos_cap;  // Heisenberg 1 - cos(theta_max)
  int fast_math;
  int variant;              // ContVariant
  uint32_t rows_per_band;   // streaming kernel band height
  uint32_t sites_per_lane;  // streaming kernel: XY 4 or 2, Heisenberg 2 or 1
  FastDiv divQ;             // lanes per plane row (R / sites per lane)
  FastDiv divL;             // edge length
  FastDiv divR;             // plane row length
  double J0d;               // uniform coupling in FP64 (fused measurement)
};

// Several sweeps of one lattice of real-valued updates (FP32 couplings, or XY
// and Heisenberg spins) with bricks of it in LDS (brick.hip).
struct BrickLaunch {
  Geom g;
  int n;               // spin components
  RngKey key;
  int J_kind;
  const void* J;
  float J0, beta;
  float param;         // XY max angle, Heisenberg 1 - cos(theta_max)
  double J0d;
  uint32_t V;          // positions of a row a lane holds
  uint32_t nb[3];      // bricks along x, y, z; 1: the whole edge, no halo
  uint32_t halo_x;     // halo in positions (pairs of sites) along x, a multiple of V
  uint32_t steps;      // half-sweeps of the launch (whole sweeps): the halo in sites along y, z
  uint32_t positions;  // the largest brick with its halo
  uint32_t t0;         // sweep counter of the launch's first
  const void* src;     // FP32 components, or int8 signs (n = 1)
  void* dst;           // src itself with one brick only
  void* parts;         // reduction partials of the final state (several bricks), or null
  void* obs;           // its record (one brick), or null
  int64_t sweep;
};

enum ContVariant { kContAuto = 0, kContRow = 1, kContStream = 2 };

// One lattice of a batch (device table, written by the host runtime).
struct BatchDesc {
  uint32_t L, R, Nh, replica;
  uint32_t divR_m, divR_s, divL_m, divL_s;  // FastDiv constants for R and L
  uint32_t th_lo, th_hi;                    // threshold bytes (always-accept classes: 0xFF)
  uint32_t spin_off_lo, spin_off_hi;        // byte offset of its [2][Nh] spins
  uint32_t J_off_lo, J_off_hi;              // byte offset of its [d][2][Nh] couplings
  uint32_t frac[7];                         // refinement fractions (2^24: always)
  uint32_t al_lo, al_hi;                    // byte k = 0xFF if class k always accepts
  uint32_t packed;                          // 1: may take the packed path (one bit per site)
  double J0;
};

// Workgroups of a batch, in its order: n_single lattices one each, per_full (a wave
// each) in each of the next g_full, per_tiny in the others.
struct BatchSplit {
  uint32_t n_single, g_full, per_full, per_tiny, groups;
};

struct BatchLaunch {
  int d;
  bool pm;                 // +-1 couplings (else uniform)
  uint32_t n_lattices;
  BatchSplit split;
  uint32_t threads;        // workgroup size
  size_t max_sites;        // the largest L^d
  size_t lds_bytes;        // dynamic LDS of a workgroup (batch_lds_bytes)
  const BatchDesc* descs;  // device
  const uint32_t* order;   // device: workgroup -> lattice
  RngKey key;              // replica is taken from each descriptor
};

struct MeasureLaunch {
  Geom g;
  int n;
  int J_kind;
  const void* J;
  double J0;
  int64_t sweep;  // sweep counter of the measured state
};

// Independent chains of one small Ising lattice with shared FP32 couplings.
struct ChainsLaunch {
  Geom g;
  RngKey key;        // key.replica = replica of chain 0
  const float* J;    // [d][2][Nh]
  float beta;
  uint32_t n_chains;
  FastDiv divR, divL;  // plane row length L/2, edge L
  const int8_t* start; // covariance replay from these spins, which stay as they are (sums
                       // overwritten), or null: from the chains' own, which move (sums added to)
  int pair_kernel;     // one pair of sites per lane, state in registers (N/4 <= 1024)
  int multi_kernel;    // larger ones: two or three pairs per lane
};

}  // namespace smc
