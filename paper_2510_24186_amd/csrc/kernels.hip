// HIP kernels of the docking hot path for gfx950 and their launchers.
//
//  map_kernel     receptor grid maps (one thread per node, the atoms near its
//                 brick of nodes collected in LDS, terms and sums in FP64)
//  score_kernel   E and dE/dq of caller-supplied poses
//  sample_kernel  Metropolis MC + local refinement; one LPP-lane group per
//                 trajectory, trajectory state in registers for a whole
//                 chunk of MC steps; plain (one launch per ligand) or
//                 persistent (device work queue over ragged-packed items)
//  best_kernel    per ligand: bitonic sort of the trajectories' best
//                 energies, greedy RMSD clustering, top N
//  rank_kernel    screening rank across ligands: blocks of 2,048 scores
//                 sorted (two keys a thread, exchanged by shuffles and through
//                 LDS) and cut to the k smallest, pass by pass
#include <float.h>
#include <math.h>

#include <algorithm>

#include "dock_device.h"
#include "dock_kernels.h"

namespace dock {

// ================================================================ maps

// ((dx*dx + dy*dy) + dz*dz) with every operation rounded separately.  The
// default contraction would fuse a product into the following sum (one
// rounding fewer), which moves d2 by an ulp and flips cutoff decisions that
// sit on the boundary.
__device__ __forceinline__ float d2_rounded(float dx, float dy, float dz) {
#pragma clang fp contract(off)
  const float xx = dx * dx, yy = dy * dy, zz = dz * dz;
  return (xx + yy) + zz;
}

// One thread per node, a workgroup per brick of 8 x 8 x 4 nodes.  The
// receptor atoms that can be inside the largest cutoff of some node of the
// brick are first collected in LDS, in their order (the test takes the
// brick's nearest point with the node's own rounding: each difference,
// product and sum is no larger than any node's, so no atom is lost), so a
// node tests about 1.5 times the atoms it needs instead of the whole
// receptor.  Bound by FP64 VALU: a square root and per radius class (three
// for the eight ligand types) one exponential per atom inside the cutoff,
// two for the Vina terms; the clash, contact and hydrogen-bond terms are
// evaluated where a node is near enough, once per class.  Every sum takes
// its terms in atom order.  2,000 atoms, 64^3 nodes, TRIDS with per-term
// maps: 2.54 -> 0.26 ms against testing every atom at every node and
// evaluating each type's terms (same bits).
constexpr int kBrickX = 8, kBrickY = 8, kBrickZ = 4, kMapList = 512, kXcds = 8;

template <int K, bool ROWS>
__global__ void __launch_bounds__(256) map_kernel(MapArgs a) {
  constexpr bool TRIDS = K == 3;
  __shared__ float4 list[kMapList];
  __shared__ int wave_n[4];
  __shared__ double s_rs[kTypes][kRadClasses];   // radius sums
  __shared__ float s_dc2[kTypes][kRadClasses];   // FP32 squared clash distances without a hydrogen bond
  __shared__ uint32_t s_hb[kTypes];              // bit t: ligand type t and this receptor type hydrogen-bond
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid < kTypes) {
    uint32_t hb = 0;
#pragma unroll
    for (int t = 0; t < kTypes; ++t) hb |= (a.tab[t * kTypes + tid].flags & 1u) << t;
    s_hb[tid] = hb;
#pragma unroll
    for (int c = 0; c < kRadClasses; ++c) {
      const TypePair& tp = a.tab[kRadType[c] * kTypes + tid];
      s_rs[tid][c] = tp.rsum64;
      s_dc2[tid][c] = tp.rsum * tp.rsum;
    }
  }
  const int nx = a.grid.dims[0], ny = a.grid.dims[1], nz = a.grid.dims[2];
  const int nbx = (nx + kBrickX - 1) / kBrickX, nby = (ny + kBrickY - 1) / kBrickY;
  int b = blockIdx.x;
  if (ROWS) {  // see launch_map_build
    b = (b / kXcds / nbx * kXcds + b % kXcds) * nbx + b / kXcds % nbx;
    if (b >= nbx * nby * ((nz + kBrickZ - 1) / kBrickZ)) return;
  }
  const int x0 = (b % nbx) * kBrickX, y0 = (b / nbx % nby) * kBrickY, z0 = (b / (nbx * nby)) * kBrickZ;
  const int ix = x0 + tid % kBrickX, iy = y0 + tid / kBrickX % kBrickY, iz = z0 + wv;
  const bool live = ix < nx && iy < ny && iz < nz;
  // node coordinate: FP64 origin + spacing * index, rounded once to FP32
  auto coord = [&](int axis, int i) { return float(double(a.grid.origin[axis]) + double(a.grid.spacing) * i); };
  const float px = coord(0, ix), py = coord(1, iy), pz = coord(2, iz);
  const float lox = coord(0, x0), hix = coord(0, min(x0 + kBrickX, nx) - 1);
  const float loy = coord(1, y0), hiy = coord(1, min(y0 + kBrickY, ny) - 1);
  const float loz = coord(2, z0), hiz = coord(2, min(z0 + kBrickZ, nz) - 1);
  const float cmax2 = TRIDS ? 100.0f : 64.0f;
  // sums per class: a0, a1, a2 by radius class (TRIDS: a0 E_long; Vina: gauss1,
  // gauss2, repulsion), clash by role class, hydrogen bonds by type 3 .. 6,
  // hydrophobic contacts of types 0 and 7
  double a0[kRadClasses] = {}, a1[kRadClasses] = {}, a2[kRadClasses] = {}, clash[kRoleClasses] = {}, hbond[4] = {},
         hyd[2] = {};
  auto add_atoms = [&](int n) {
    for (int j = 0; j < n; ++j) {
      const float4 rj = list[j];
      // FP32 squared distance in a fixed order, each product and sum rounded
      // on its own: the inside-cutoff decisions depend on these exact bits
      const float d2 = d2_rounded(px - rj.x, py - rj.y, pz - rj.z);
      if (!(d2 < cmax2)) continue;
      const double ex = double(px) - double(rj.x), ey = double(py) - double(rj.y),
                   ez = double(pz) - double(rj.z);
      const double d = sqrt(ex * ex + ey * ey + ez * ez);
      const int tr = __builtin_amdgcn_readfirstlane(__float_as_int(rj.w)) & 0xff;  // the same for all lanes
      const uint32_t hbm = s_hb[tr];
      if (TRIDS) {
#pragma unroll
        for (int c = 0; c < kRadClasses; ++c) {
          const double s = d - s_rs[tr][c] - 3.0;
          a0[c] += -exp(-0.25 * s * s);
        }
        // largest clash distance and hydrogen-bond cutoff: 3.8 A
        if (d2 < 3.81f * 3.81f) {
          const double dd = fmax(d, 0.1);
          double cl[kRadClasses], clh = 0.0, eh = 0.0;
#pragma unroll
          for (int c = 0; c < kRadClasses; ++c)
            cl[c] = d2 < s_dc2[tr][c] ? -log(dd / s_rs[tr][c]) : 0.0;
          if (hbm) {
            const float c26 = float(2.6);
            if (d2 < c26 * c26) clh = -log(dd / 2.6);
            if (d2 < 3.4f * 3.4f) {
              const double t = d - 2.88;
              eh = -exp(-t * t / 0.18);
            }
          }
#pragma unroll
          for (int c = 0; c < kRoleClasses; ++c) clash[c] += (hbm >> kRoleType[c]) & 1u ? clh : cl[kRoleRad[c]];
#pragma unroll
          for (int t = 3; t <= 6; ++t)
            if ((hbm >> t) & 1u) hbond[t - 3] += eh;
        }
      } else {
        double s[kRadClasses];
#pragma unroll
        for (int c = 0; c < kRadClasses; ++c) {
          s[c] = d - s_rs[tr][c];
          a0[c] += exp(-4.0 * s[c] * s[c]);
          const double t = s[c] - 3.0;
          a1[c] += exp(-0.25 * t * t);
          a2[c] += s[c] < 0.0 ? s[c] * s[c] : 0.0;
        }
        auto contact = [](double x) { return x < 0.5 ? 1.0 : (x < 1.5 ? 1.5 - x : 0.0); };
        auto bond = [](double x) { return x < -0.7 ? 1.0 : (x < 0.0 ? -x / 0.7 : 0.0); };
        if (tr == 0 || tr == 7) {
          hyd[0] += contact(s[kRadClass[0]]);
          hyd[1] += contact(s[kRadClass[7]]);
        }
        if (hbm && d2 < 3.81f * 3.81f) {
#pragma unroll
          for (int t = 3; t <= 6; ++t)
            if ((hbm >> t) & 1u) hbond[t - 3] += bond(s[kRadClass[t]]);
        }
      }
    }
  };
  int n = 0;
  for (int base = 0; base < a.n_rec; base += 256) {
    float4 rj = make_float4(0.f, 0.f, 0.f, 0.f);
    bool near = false;
    if (base + tid < a.n_rec) {
      rj = a.rec[base + tid];
      const float dx = fmaxf(fmaxf(lox - rj.x, rj.x - hix), 0.f), dy = fmaxf(fmaxf(loy - rj.y, rj.y - hiy), 0.f),
                  dz = fmaxf(fmaxf(loz - rj.z, rj.z - hiz), 0.f);
      near = d2_rounded(dx, dy, dz) < cmax2;
    }
    const unsigned long long m = __builtin_amdgcn_ballot_w64(near);
    if (lane == 0) wave_n[wv] = __popcll(m);
    __syncthreads();
    int at = n;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      at += k < wv ? wave_n[k] : 0;
      n += wave_n[k];
    }
    if (near) list[at + __popcll(m & ((1ull << lane) - 1ull))] = rj;
    __syncthreads();
    // the list takes up to one more chunk
    if (n > kMapList - 256 || base + 256 >= a.n_rec) {
      if (live) add_atoms(n);
      n = 0;
      __syncthreads();
    }
  }
  if (!live) return;
  const long long total = (long long)nx * ny * nz, node = ((long long)iz * ny + iy) * nx + ix;
#pragma unroll
  for (int t = 0; t < kTypes; ++t) {
    double acc[K];
    acc[0] = a0[kRadClass[t]];
    if (TRIDS) {
      acc[1] = clash[kRoleClass[t]];
      acc[2] = t >= 3 && t <= 6 ? hbond[(t - 3) & 3] : 0.0;
    } else {
      acc[1] = a1[kRadClass[t]];
      acc[2] = a2[kRadClass[t]];
      acc[K - 2] = t == 0 ? hyd[0] : (t == 7 ? hyd[1] : 0.0);
      acc[K - 1] = t >= 3 && t <= 6 ? hbond[(t - 3) & 3] : 0.0;
    }
    double m = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      m += double(a.w[k]) * acc[k];
      if (a.G) a.G[((long long)t * K + k) * total + node] = float(acc[k]);
    }
    a.M[(long long)t * total + node] = float(m);
  }
}

// Bricks write 32-byte parts of a line, four bricks along x share it, and blocks
// go round the eight XCDs: their L2s then write the parts back one by one.  On
// large grids a row of bricks stays on one XCD; on small ones that leaves the
// XCDs uneven work (88^3 nodes, 1,210 atoms, Vina terms: 3 % slower by rows).
// TRIDS with per-term maps, 800 atoms, us brick by brick and row by row: 96^3
// nodes 420 and 430, 112^3 474 and 455, 128^3 735 and 483, 192^3 786 and 568 (five
// atoms 1,010 and 271).
hipError_t launch_map_build(const MapArgs& a, hipStream_t s) {
  const auto bricks = [](int n, int b) { return unsigned((n + b - 1) / b); };
  const unsigned nbx = bricks(a.grid.dims[0], kBrickX),
                 rows = bricks(a.grid.dims[1], kBrickY) * bricks(a.grid.dims[2], kBrickZ);
  const bool by_rows = rows >= 384;
  const unsigned blocks = nbx * (by_rows ? (rows + kXcds - 1) / kXcds * kXcds : rows);
  if (a.n_terms == 3 && by_rows)
    hipLaunchKernelGGL((map_kernel<3, true>), dim3(blocks), dim3(256), 0, s, a);
  else if (a.n_terms == 3)
    hipLaunchKernelGGL((map_kernel<3, false>), dim3(blocks), dim3(256), 0, s, a);
  else if (by_rows)
    hipLaunchKernelGGL((map_kernel<5, true>), dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((map_kernel<5, false>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ================================================================ map adjoint

// Bricks of 8 x 4 x 2 nodes, one per wavefront.
constexpr int kAdjX = 8, kAdjY = 4, kAdjZ = 2;

// mask[b]: the nodes of brick b, bit x + 8 y + 32 z, where some lambda is not
// zero (one wave per brick).
__global__ void __launch_bounds__(256) map_adjoint_mask_kernel(const float* __restrict__ lam, int nx, int ny, int nz,
                                                               int nbx, int nby, long long n_bricks,
                                                               unsigned long long* __restrict__ mask) {
  const long long b = (long long)blockIdx.x * 4 + threadIdx.x / 64;
  if (b >= n_bricks) return;
  const int lane = threadIdx.x & 63;
  const int ix = int(b % nbx) * kAdjX + lane % kAdjX, iy = int(b / nbx % nby) * kAdjY + lane / kAdjX % kAdjY,
            iz = int(b / ((long long)nbx * nby)) * kAdjZ + lane / (kAdjX * kAdjY);
  bool any = false;
  if (ix < nx && iy < ny && iz < nz) {
    const long long nodes = (long long)nx * ny * nz, node = ((long long)iz * ny + iy) * nx + ix;
#pragma unroll
    for (int q = 0; q < 3 * kTypes; ++q) any |= lam[q * nodes + node] != 0.f;
  }
  const unsigned long long m = __builtin_amdgcn_ballot_w64(any);
  if (lane == 0) mask[b] = m;
}

DK_INLINE double wave_sum(double v) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k);
  return v;
}

// One workgroup per receptor atom over the bricks around it: a wave tests 64
// bricks at a time (inside the cutoff at their nearest point, and with a
// nonzero lambda where masks are given: the lambda of a set of docked poses
// is zero in most of a pocket), then the nodes of each hit (the same FP32
// cutoff decisions as map_kernel), and queues the numbers of those that count
// in LDS; 64 queued nodes are taken at a time, one per lane.  The chain rule
// in FP64: per node one exponential for each of the three radius classes of
// the ligand types, the short-range terms where the node is near.  Bound by
// those exponentials (256 poses' lambda, 2,000 atoms, 64^3 nodes: 2.69 ms
// with every node of the box and every type's exponential, 0.48 ms with every
// node of a brick that holds a nonzero lambda, of which three in ten counted,
// now 0.28 ms).  dL/dr is written once per atom in a fixed order (no atomics);
// dL/dtheta takes 13 atomic adds per atom.
__global__ void __launch_bounds__(256) map_adjoint_kernel(MapAdjArgs a) {
  __shared__ double red[4][3 + kMapTheta];
  __shared__ uint32_t queue[4][128];  // per wave, a ring: ix | iy << 10 | iz << 20 (dims <= 1024)
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = blockIdx.x;
  const float4 ri = a.rec[i];
  const int u = __builtin_amdgcn_readfirstlane(__float_as_int(ri.w)) & 0xff;
  const int nx = a.grid.dims[0], ny = a.grid.dims[1], nz = a.grid.dims[2];
  const long long nodes = (long long)nx * ny * nz;
  const int nbx = (nx + kAdjX - 1) / kAdjX, nby = (ny + kAdjY - 1) / kAdjY;
  // bricks that hold a node of the box around the cutoff sphere
  int lo[3], cnt[3];
  const float rr[3] = {ri.x, ri.y, ri.z};
  const int bs[3] = {kAdjX, kAdjY, kAdjZ};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double o = a.grid.origin[c], h = a.grid.spacing;
    const int n = a.grid.dims[c];
    const double first = floor((double(rr[c]) - 10.0 - o) / h) - 1.0, last = ceil((double(rr[c]) + 10.0 - o) / h) + 1.0;
    const int l = int(fmin(fmax(first, 0.0), double(n))), g = int(fmin(fmax(last, -1.0), double(n - 1)));
    lo[c] = l / bs[c];
    cnt[c] = g >= l ? g / bs[c] - lo[c] + 1 : 0;
  }
  const long long nb = (long long)cnt[0] * cnt[1] * cnt[2];
  double rs[kRadClasses];
  float dc2[kRadClasses];
  uint32_t hbm = 0;
#pragma unroll
  for (int c = 0; c < kRadClasses; ++c) {
    const TypePair& tp = a.tab[kRadType[c] * kTypes + u];
    rs[c] = tp.rsum64;
    dc2[c] = tp.rsum * tp.rsum;
  }
#pragma unroll
  for (int t = 0; t < kTypes; ++t) hbm |= (a.tab[t * kTypes + u].flags & 1u) << t;
  auto coord = [&](int axis, int k) { return float(double(a.grid.origin[axis]) + double(a.grid.spacing) * k); };
  constexpr double kSigL2 = 2.0, kSigL3 = 2.0 * 1.4142135623730951;  // sigma_long^2, ^3 (2 sigma^2 = 4)
  constexpr double kSigH2 = 0.09, kSigH3 = 0.027;
  // dL/dr; per ligand type sum of lambda g x / sigma^2 (E_long) and of
  // lambda / d_clash (pairs without a hydrogen bond); the other constants
  double dr[3] = {}, rl[kTypes] = {}, rc[kTypes] = {}, sig_l = 0.0, mu_h = 0.0, sig_h = 0.0, dc_h = 0.0;
  auto take_node = [&](uint32_t code) {
    const int ix = code & 1023u, iy = (code >> 10) & 1023u, iz = code >> 20;
    const float px = coord(0, ix), py = coord(1, iy), pz = coord(2, iz);
    const float d2 = d2_rounded(px - ri.x, py - ri.y, pz - ri.z);
    const double ex = double(ri.x) - double(px), ey = double(ri.y) - double(py), ez = double(ri.z) - double(pz);
    const double d = sqrt(ex * ex + ey * ey + ez * ez);
    const float* lt = a.lam + ((long long)iz * ny + iy) * nx + ix;
    double gx[kRadClasses], l0c[kRadClasses] = {};
#pragma unroll
    for (int c = 0; c < kRadClasses; ++c) {
      const double x = d - rs[c] - 3.0;
      gx[c] = exp(-0.25 * x * x) * x * (1.0 / kSigL2);
    }
#pragma unroll
    for (int t = 0; t < kTypes; ++t) {
      const double l0 = lt[(long long)(3 * t) * nodes];
      rl[t] += l0 * gx[kRadClass[t]];
      l0c[kRadClass[t]] += l0;
    }
    double dphi = 0.0;
#pragma unroll
    for (int c = 0; c < kRadClasses; ++c) {
      const double w = l0c[c] * gx[c];
      dphi += w;
      sig_l += w * (d - rs[c] - 3.0) * (kSigL2 / kSigL3);
    }
    // largest clash distance and hydrogen-bond cutoff: 3.8 A
    if (d2 < 3.81f * 3.81f) {
      const double inv_d = 1.0 / d;
      const float c26 = float(2.6);
#pragma unroll
      for (int t = 0; t < kTypes; ++t) {
        const bool hb = (hbm >> t) & 1u;
        if (hb ? d2 < c26 * c26 : d2 < dc2[kRadClass[t]]) {
          const double l1 = lt[(long long)(3 * t + 1) * nodes];
          dphi -= d > 0.1 ? l1 * inv_d : 0.0;  // flat below (a lambda may be infinite)
          if (hb)
            dc_h += l1 / 2.6;
          else
            rc[t] += l1 / rs[kRadClass[t]];
        }
      }
      if (hbm && d2 < 3.4f * 3.4f) {
        const double x = d - 2.88, g = exp(-x * x / 0.18) * x / kSigH2;
#pragma unroll
        for (int t = 0; t < kTypes; ++t) {
          if (!((hbm >> t) & 1u)) continue;
          const double c = double(lt[(long long)(3 * t + 2) * nodes]) * g;
          dphi += c;
          mu_h -= c;
          sig_h -= c * x * (kSigH2 / kSigH3);
        }
      }
    }
    if (d > 0.0) {
      const double f = dphi / d;
      dr[0] += f * ex;
      dr[1] += f * ey;
      dr[2] += f * ez;
    }
  };
  int head = 0, queued = 0;  // of the wave's ring
  for (long long base = 64 * wv; base < nb; base += 256) {
    const long long q = base + lane;
    unsigned long long nz_mask = 0;  // nodes of this lane's brick to test
    int bx = 0, by = 0, bz = 0;
    if (q < nb) {
      bx = lo[0] + int(q % cnt[0]);
      by = lo[1] + int(q / cnt[0] % cnt[1]);
      bz = lo[2] + int(q / ((long long)cnt[0] * cnt[1]));
      // the brick's nearest point, rounded as its nodes are: no node is nearer
      auto gap = [&](int axis, int b, float p, int n) {
        const int k0 = b * bs[axis], k1 = min(k0 + bs[axis], n) - 1;
        return fmaxf(fmaxf(coord(axis, k0) - p, p - coord(axis, k1)), 0.f);
      };
      if (d2_rounded(gap(0, bx, ri.x, nx), gap(1, by, ri.y, ny), gap(2, bz, ri.z, nz)) < 100.0f)
        nz_mask = a.mask ? a.mask[((long long)bz * nby + by) * nbx + bx] : ~0ull;
    }
    unsigned long long m = __builtin_amdgcn_ballot_w64(nz_mask != 0);
    while (m) {
      const int l = __builtin_ctzll(m);
      m &= m - 1;
      const unsigned long long nm = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane(int(nz_mask >> 32), l) << 32 |
                                    (uint32_t)__builtin_amdgcn_readlane(int(nz_mask), l);
      const int ix = __builtin_amdgcn_readlane(bx, l) * kAdjX + lane % kAdjX,
                iy = __builtin_amdgcn_readlane(by, l) * kAdjY + lane / kAdjX % kAdjY,
                iz = __builtin_amdgcn_readlane(bz, l) * kAdjZ + lane / (kAdjX * kAdjY);
      const bool in = (nm >> lane & 1) && ix < nx && iy < ny && iz < nz &&
                      d2_rounded(coord(0, ix) - ri.x, coord(1, iy) - ri.y, coord(2, iz) - ri.z) < 100.0f;
      const unsigned long long im = __builtin_amdgcn_ballot_w64(in);
      if (in)
        queue[wv][(head + queued + __popcll(im & ((1ull << lane) - 1))) & 127] =
            uint32_t(ix) | uint32_t(iy) << 10 | uint32_t(iz) << 20;
      queued += __popcll(im);
      if (queued >= 64) {
        wave_sync();
        take_node(queue[wv][(head + lane) & 127]);
        head = (head + 64) & 127;
        queued -= 64;
        wave_sync();
      }
    }
  }
  wave_sync();
  if (lane < queued) take_node(queue[wv][(head + lane) & 127]);
  // sums over the workgroup; theta = (mu_long, sigma_long, mu_hb, sigma_hb,
  // d_clash_hb, R_0 .. R_7), both types of a pair taking its radius terms
  double all[3 + kMapTheta];
  double mu_l = 0.0, ru = 0.0;
#pragma unroll
  for (int t = 0; t < kTypes; ++t) {
    mu_l -= rl[t];
    ru += rc[t] - rl[t];
    all[3 + 5 + t] = rc[t] - rl[t];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) all[k] = dr[k];
  all[3] = mu_l;
  all[4] = -sig_l;
  all[5] = mu_h;
  all[6] = sig_h;
  all[7] = dc_h;
#pragma unroll
  for (int t = 0; t < kTypes; ++t) all[3 + 5 + t] += t == u ? ru : 0.0;
#pragma unroll
  for (int k = 0; k < 3 + kMapTheta; ++k) {
    const double v = wave_sum(all[k]);
    if (lane == 0) red[wv][k] = v;
  }
  __syncthreads();
  if (tid < 3 + kMapTheta) {
    const double v = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
    if (tid < 3) {
      if (a.dLdxyz) a.dLdxyz[3 * i + tid] += float(v);
    } else if (a.dLdtheta && v != 0.0) {
      atomicAdd(&a.dLdtheta[tid - 3], v);
    }
  }
}

long long map_adjoint_bricks(const GridDev& g) {
  const auto bricks = [](int n, int b) { return (long long)((n + b - 1) / b); };
  return bricks(g.dims[0], kAdjX) * bricks(g.dims[1], kAdjY) * bricks(g.dims[2], kAdjZ);
}

hipError_t launch_map_adjoint(const MapAdjArgs& a, hipStream_t s) {
  if (a.n_rec <= 0) return hipSuccess;
  if (a.mask) {
    const long long n = map_adjoint_bricks(a.grid);
    const int nbx = (a.grid.dims[0] + kAdjX - 1) / kAdjX, nby = (a.grid.dims[1] + kAdjY - 1) / kAdjY;
    hipLaunchKernelGGL(map_adjoint_mask_kernel, dim3(unsigned((n + 3) / 4)), dim3(256), 0, s, a.lam, a.grid.dims[0],
                       a.grid.dims[1], a.grid.dims[2], nbx, nby, n, a.mask);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(map_adjoint_kernel, dim3(a.n_rec), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ================================================================ slabs

template <int LPP, int APL>
DK_INLINE GroupSlab make_slab(unsigned char* base) {
  constexpr int NA = LPP * APL;
  GroupSlab S;
  S.xs = reinterpret_cast<float4*>(base);
  S.fx = reinterpret_cast<double*>(base + 16 * NA);
  S.fy = S.fx + NA;
  S.fz = S.fy + NA;
  S.fb = reinterpret_cast<float4*>(S.fx);
  S.l2 = nullptr;
  return S;
}
// coordinates (16 B per atom), then the larger of three FP64 force arrays
// (24 B per atom) and the force entries of the pass layout (2 * lanes + 1
// float4)
constexpr size_t slab_bytes(int lpp, int apl) {
  return size_t(lpp) * apl * 16 +
         (size_t(lpp) * apl * 24 > size_t(lpp) * 32 + 16 ? size_t(lpp) * apl * 24 : size_t(lpp) * 32 + 16);
}
// staged pair entries (8 bytes each), padded so the float4 slab that follows
// is aligned (sampler)
constexpr size_t pair_bytes(int max_pairs) { return (size_t(max_pairs) * 8 + 15) / 16 * 16; }

size_t group_lds_bytes(int lpp, int apl, int max_pairs) {
  return size_t(64 / lpp) * (pair_bytes(max_pairs) + slab_bytes(lpp, apl));
}

size_t sample_lds_bytes(int lpp, int apl, int block, int max_pairs) {
  const int gpb = block / lpp;
  return pair_bytes(max_pairs) + size_t(gpb) * slab_bytes(lpp, apl) + 16;
}

// E_MDN parameters of one ligand when the term is active for its pocket.
DK_INLINE MdnArg mdn_for(const LigandArrays& A, const LigDev& lg, const PocketDev& pk) {
  MdnArg m{nullptr, 0, 0};
  if (A.mdn && pk.mdn_res > 0 && pk.mdn_w != 0.f && A.mdn_res == pk.mdn_res) {
    m.par = A.mdn + size_t(lg.atom_off) * A.mdn_res * A.mdn_k;
    m.n_res = A.mdn_res;
    m.k = A.mdn_k;
  }
  return m;
}

// ================================================================ score

// A wavefront takes `chunk` consecutive poses and evaluates as many at a time
// as their ligands' lane configurations allow: four in 16-lane groups, two in
// 32-lane groups, else one (one atom per lane up to 64 atoms).  Pair records
// are read from global memory: a wave's LDS is its slabs alone, so the
// registers and not the LDS set how many waves a CU holds (three per SIMD:
// four spill 42 registers and ran 130 us where three take 109).  32,768 poses
// of 256 ligands of 10-60 atoms: 370 us with records staged per group and
// every pose in the lane configuration of the largest ligand, 109 us so.
struct WaveForm {
  int lanes, poses;  // lanes per pose (16, 32, 64; 128: 64 lanes, two atoms each), poses taken
};
// form of the poses from `at` on; cfg: per lane, the lane configuration of
// pose `lane` of the chunk (16, 32, 64, 128; 0 past the chunk's end)
DK_INLINE WaveForm next_form(int cfg, int at, int chunk) {
  const int c = __builtin_amdgcn_readlane(cfg, at);
  if (c > 32) return WaveForm{c, 1};
  const unsigned long long le32 = __builtin_amdgcn_ballot_w64(cfg <= 32), le16 = __builtin_amdgcn_ballot_w64(cfg <= 16);
  if (chunk - at >= 4 && ((le16 >> at) & 15u) == 15u) return WaveForm{16, 4};
  if (chunk - at >= 2 && ((le32 >> at) & 3u) == 3u) return WaveForm{32, 2};
  return WaveForm{64, 1};
}
// lane configuration of a ligand with one atom per lane up to 64 atoms
DK_INLINE int lane_config(const LigDev* g) {
  if (g->n_atoms > 64) return 128;
  const int need = max(g->n_atoms, max(g->n_dof, g->n_frags));
  return need <= 16 ? 16 : (need <= 32 ? 32 : 64);
}
// slabs of the forms: 4 of 16 lanes, 2 of 32, 1 of 64
constexpr size_t wave_slab_bytes(int lanes) {
  return lanes == 128 ? slab_bytes(64, 2)
                      : std::max({4 * slab_bytes(16, 1), 2 * slab_bytes(32, 1), slab_bytes(64, 1)});
}
constexpr size_t kClashBytes = sizeof(float) * kClashTable;
size_t wave_lds_bytes(int lanes) { return wave_slab_bytes(lanes) + 4 * kClashBytes; }

// The log2(d_clash) table of a pass layout into the group's LDS.
template <int LPP>
DK_INLINE void stage_clash_table(const LigDev& lg, const PairRec* pairs, float* l2, int r) {
  if (lg.n_pass > 0 && r < kClashTable) {
    const size_t at = 2 * size_t(lg.n_prec) + (lg.pass_apl * lg.pull_cap == 8 ? size_t(lg.n_prec) / 2 : 0);
    l2[r] = ldg(reinterpret_cast<const float*>(pairs + at) + r);
  }
}

template <int LPP, int APL, int MODE>
DK_INLINE void score_poses(const ScoreArgs& a, long long first, unsigned char* smem, unsigned char* tables) {
  const int grp = threadIdx.x / LPP, r = threadIdx.x % LPP;
  const long long pose = first + grp;
  if (pose >= a.n_poses) return;
  const int lig = a.pose_lig[pose];
  if (lig < 0 || lig >= a.n_ligands) {
    if (r == 0) a.E[pose] = __int_as_float(0x7fc00000);
    return;
  }
  GroupSlab S = make_slab<LPP, APL>(smem + size_t(grp) * slab_bytes(LPP, APL));
  S.l2 = reinterpret_cast<float*>(tables + grp * kClashBytes);
  // the alternative (one atom per lane up to 64 atoms) pair layouts
  LigDev lg = a.L.ligs[lig];
  use_alt_layout(lg);
  const PocketDev pk = a.pockets[lg.pocket];
  LaneLig<APL> L;
  load_lane_lig<LPP, APL>(L, lg, a.L.ligs + lig, a.L.atoms, a.L.frags, a.L.tors, pk, r);
  const PairRec* pairs = a.L.pairs + lg.pair_off;
  stage_clash_table<LPP>(lg, pairs, S.l2, r);
  wave_sync();
  const float q = r < lg.n_dof ? a.q[pose * a.q_stride + r] : 0.f;
  float xo[APL][3], go[APL][3];
  const EvalOut o =
      eval_pose<LPP, APL, kWantBoth, true, MODE, true>(L, q, pk, pairs, S, r, xo, go, mdn_for(a.L, lg, pk));
  if (r == 0) a.E[pose] = o.E;
  if (a.dEdq && r < lg.n_dof) a.dEdq[pose * a.q_stride + r] = o.g;
  if (a.xyz) {
#pragma unroll
    for (int s = 0; s < APL; ++s) {
      const int atom = APL * r + s;
      if (atom < lg.n_atoms) {
        float* dst = a.xyz + pose * a.xyz_stride + 3 * L.aorig[s];
        dst[0] = xo[s][0];
        dst[1] = xo[s][1];
        dst[2] = xo[s][2];
      }
    }
  }
}

// SMALL: every ligand of the handle takes 16 lanes, so a wavefront always takes
// four poses of one form, with the registers of that form alone (10- and 14-atom
// ligands, 8,192 poses: kernel 15.8 us in the general form, 9.3 so; 65,536 51.3 and
// 40.1).
template <int MODE, bool SMALL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(SMALL ? 4 : 3))) score_kernel(ScoreArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* tables = smem + a.slab_bytes;
  const long long base = (long long)blockIdx.x * a.chunk;
  if (SMALL) {
    score_poses<16, 1, MODE>(a, base, smem, tables);
    return;
  }
  const int n = int(min((long long)a.chunk, a.n_poses - base));
  int cfg = 0;
  if (int(threadIdx.x) < n) {
    const int lig = a.pose_lig[base + threadIdx.x];
    if (lig >= 0 && lig < a.n_ligands) cfg = lane_config(a.L.ligs + lig);
  }
  for (int at = 0; at < n;) {
    const WaveForm f = next_form(cfg, at, n);
    if (f.lanes == 16)
      score_poses<16, 1, MODE>(a, base + at, smem, tables);
    else if (f.lanes == 32)
      score_poses<32, 1, MODE>(a, base + at, smem, tables);
    else if (f.lanes == 64)
      score_poses<64, 1, MODE>(a, base + at, smem, tables);
    else
      score_poses<64, 2, MODE>(a, base + at, smem, tables);
    wave_sync();
    at += f.poses;
  }
}

// Poses per wavefront, for a handle whose widest ligand takes `lanes` (16, 32,
// 64; 128: two atoms per lane): one while the waves of one pose each are few,
// then two, then four where small ligands can share a wave.  Score kernel, us
// with one and two poses a wave: ligands of 20 and 30 atoms, 2,048 poses 10.9 and
// 11.4, 4,096 19.5 and 12.2; 10-60 atoms, 4,096 poses 28.2 and 29.2.
int wave_chunk(long long n_poses, int lanes) {
  if (lanes == 16) return 4;
  return n_poses <= (lanes == 32 ? 2048 : 4096) ? 1 : (n_poses <= 8192 ? 2 : 4);
}

hipError_t launch_score(ScoreArgs a, int lanes, int mode, hipStream_t s) {
  if (a.n_poses <= 0) return hipSuccess;
  a.chunk = wave_chunk(a.n_poses, lanes);
  a.slab_bytes = unsigned(wave_slab_bytes(lanes));
  const unsigned blocks = unsigned((a.n_poses + a.chunk - 1) / a.chunk);
  const size_t lds = wave_lds_bytes(lanes);
  const bool small = lanes == 16;
#define X(M, SM)                                                                      \
  if (mode == M && small == SM) {                                                     \
    hipLaunchKernelGGL((score_kernel<M, SM>), dim3(blocks), dim3(64), lds, s, a);     \
    return hipGetLastError();                                                         \
  }
  X(kModeGrid, false) X(kModeGrid, true) X(kModeDirect, false) X(kModeDirect, true)
  X(kModeGridMdn, false) X(kModeGridMdn, true)
#undef X
  return hipErrorInvalidValue;
}

// ================================================================ differentiable form

// Fixed-point scale of a pocket's sums: 2^(62 - e) with 2^e >= B = n_poses *
// max_p(|dLdE_p| N_p) * max_k |w_k|, a bound on any node's |dL/dG| (an atom's
// eight corner weights are non-negative and sum to one); 0 where B is not
// finite.  Maxima do not depend on the order of evaluation.
DK_INLINE double fixed_scale(const TermsArgs& a, int pi, int K) {
  float mw = 0.f;
  for (int k = 0; k < K; ++k) {
    const float v = fabsf(a.w[pi * K + k]);
    mw = fmaxf(mw, v <= FLT_MAX ? v : INFINITY);
  }
  const double B = double(a.n_poses) * double(__uint_as_float(a.bound[pi])) * double(mw);
  if (!(B <= DBL_MAX)) return 0.0;
  if (!(B > 0.0)) return 1.0;
  int ex = 0;
  (void)frexp(B, &ex);
  return ldexp(1.0, 62 - ex);
}

template <int LPP, int APL, int K, bool XIN, bool ADJ>
DK_INLINE void terms_poses(const TermsArgs& a, long long first, unsigned char* smem) {
  const int grp = threadIdx.x / LPP, r = threadIdx.x % LPP;
  const long long pose = first + grp;
  if (pose >= a.n_poses) return;
  const GroupSlab S = make_slab<LPP, APL>(smem + size_t(grp) * slab_bytes(LPP, APL));
  const int lig = a.pose_lig[pose];
  if (lig < 0 || lig >= a.n_ligands) {
    if (r == 0 && a.E) a.E[pose] = __int_as_float(0x7fc00000);
    if (r == 0 && a.w_pocket) a.w_pocket[pose] = -1;
    return;
  }
  LigDev lg = a.L.ligs[lig];
  use_alt_layout(lg);
  const int pi = lg.pocket;
  const PocketDev pk = a.pockets[pi];
  LaneLig<APL> L;
  load_lane_lig<LPP, APL>(L, lg, a.L.ligs + lig, a.L.atoms, a.L.frags, a.L.tors, pk, r);
  float w[K];
#pragma unroll
  for (int k = 0; k < K; ++k) w[k] = a.w[pi * K + k];
  float q = 0.f;
  float x[APL][3], g[APL][3], ek[K];
  Rigid rg{};
  if (XIN) {
#pragma unroll
    for (int s = 0; s < APL; ++s) {
      const int atom = APL * r + s;
      const float* src = a.xyz + pose * a.xyz_stride + 3 * L.aorig[s];
      x[s][0] = atom < lg.n_atoms ? src[0] : 0.f;
      x[s][1] = atom < lg.n_atoms ? src[1] : 0.f;
      x[s][2] = atom < lg.n_atoms ? src[2] : 0.f;
    }
  } else {
    q = r < lg.n_dof ? a.q[pose * a.q_stride + r] : 0.f;
  }
  const float E = eval_terms<LPP, APL, K, XIN, ADJ>(L, q, x, g, rg, a.G[pi], pk.grid, w, a.L.pairs + lg.pair_off, S,
                                                    r, ek);
  if (r == 0 && a.E) a.E[pose] = E;
  if (!ADJ) return;
  const float dLdE = a.dLdE[pose];
  if (a.dLdx) {
#pragma unroll
    for (int s = 0; s < APL; ++s) {
      const int atom = APL * r + s;
      if (atom < lg.n_atoms) {
        float* d = a.dLdx + pose * a.xyz_stride + 3 * L.aorig[s];
        d[0] += dLdE * g[s][0];
        d[1] += dLdE * g[s][1];
        d[2] += dLdE * g[s][2];
      }
    }
  }
  if (!XIN && a.dLdq) {
    const float gq = chain_rule<LPP, APL>(L, rg, x, g, S, r);
    if (r < lg.n_dof) a.dLdq[pose * a.q_stride + r] += dLdE * gq;
  }
  // atomics last: loads after them would wait for them
  if (r == 0 && a.w_pose) {
#pragma unroll
    for (int k = 0; k < K; ++k) a.w_pose[pose * K + k] = dLdE * ek[k];
    a.w_pocket[pose] = pi;
  } else if (r == 0 && a.dLdw) {
#pragma unroll
    for (int k = 0; k < K; ++k) atomicAdd(&a.dLdw[pi * K + k], dLdE * ek[k]);
  }
  if (a.dLdG[pi]) {
    Scatter sc;
    const size_t at = size_t(a.unit_off[pi]) * kSumUnit;
    // (float sums are multiplied by w_k afterwards, where the sum is not zero:
    // a weight that is not finite has to meet every contribution, zeros too)
    bool finite_w = true;
#pragma unroll
    for (int k = 0; k < K; ++k) finite_w &= fabsf(w[k]) <= FLT_MAX;
    if (!a.sum || (!a.fixed && !finite_w)) {
      sc.direct = a.dLdG[pi];
    } else if (a.fixed) {
      sc.fixed = static_cast<unsigned long long*>(a.sum) + at * K;
      sc.scale = fixed_scale(a, pi, K);
    } else {
      sc.sum = static_cast<float*>(a.sum) + at;
    }
    scatter_terms<APL, K>(L, x, pk.grid, w, r, dLdE, sc);
  }
}

// The general adjoint holds two waves per SIMD without spills (at three it spills
// 18 to 28 registers: 8,192 poses of 10-60 atoms, TRIDS, sums 229 us the call, two
// 219), the others four.  The gathers from the per-term maps and the scatter's
// lines, both beyond L2, bound them.
template <int K, bool XIN, bool ADJ, bool SMALL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(ADJ && !SMALL ? 2 : 4))) terms_kernel(TermsArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const long long base = (long long)blockIdx.x * a.chunk;
  if (SMALL) {  // as in score_kernel
    terms_poses<16, 1, K, XIN, ADJ>(a, base, smem);
    return;
  }
  const int n = int(min((long long)a.chunk, a.n_poses - base));
  int cfg = 0;
  if (int(threadIdx.x) < n) {
    const int lig = a.pose_lig[base + threadIdx.x];
    if (lig >= 0 && lig < a.n_ligands) cfg = lane_config(a.L.ligs + lig);
  }
  for (int at = 0; at < n;) {
    const WaveForm f = next_form(cfg, at, n);
    if (f.lanes == 16)
      terms_poses<16, 1, K, XIN, ADJ>(a, base + at, smem);
    else if (f.lanes == 32)
      terms_poses<32, 1, K, XIN, ADJ>(a, base + at, smem);
    else if (f.lanes == 64)
      terms_poses<64, 1, K, XIN, ADJ>(a, base + at, smem);
    else
      terms_poses<64, 2, K, XIN, ADJ>(a, base + at, smem);
    wave_sync();
    at += f.poses;
  }
}

hipError_t launch_terms(TermsArgs a, int lanes, int K, hipStream_t s) {
  if (a.n_poses <= 0) return hipSuccess;
  a.chunk = wave_chunk(a.n_poses, lanes);
  const unsigned blocks = unsigned((a.n_poses + a.chunk - 1) / a.chunk);
  const size_t lds = wave_slab_bytes(lanes);
  const bool xin = a.xyz != nullptr, adj = a.dLdE != nullptr, small = lanes == 16;
#define X(KK, XI, AD, SM)                                                                          \
  if (K == KK && xin == XI && adj == AD && small == SM) {                                          \
    hipLaunchKernelGGL((terms_kernel<KK, XI, AD, SM>), dim3(blocks), dim3(64), lds, s, a);         \
    return hipGetLastError();                                                                      \
  }
#define Y(KK, XI) X(KK, XI, false, false) X(KK, XI, false, true) X(KK, XI, true, false) X(KK, XI, true, true)
  Y(3, false) Y(3, true) Y(5, false) Y(5, true)
#undef Y
#undef X
  return hipErrorInvalidValue;
}

// ================================================================ deterministic adjoint

// Marks the units of S that the poses' atoms reach, and takes the bound of
// the fixed-point scale along: a pose per group, its forward kinematics only.
template <int LPP, int APL, bool XIN>
DK_INLINE void mark_poses(const TermsArgs& a, long long first, unsigned char* smem) {
  const int grp = threadIdx.x / LPP, r = threadIdx.x % LPP;
  const long long pose = first + grp;
  if (pose >= a.n_poses) return;
  const int lig = a.pose_lig[pose];
  if (lig < 0 || lig >= a.n_ligands) return;
  const GroupSlab S = make_slab<LPP, APL>(smem + size_t(grp) * slab_bytes(LPP, APL));
  const LigDev lg = a.L.ligs[lig];
  const int pi = lg.pocket;
  if (!a.dLdG[pi]) return;
  if (r == 0 && a.fixed) {
    float v = fabsf(a.dLdE[pose]) * float(lg.n_atoms);
    if (!(v <= FLT_MAX)) v = INFINITY;  // NaN counts as unbounded
    // by slots: atomics on one address take their turns
    atomicMax(&a.bound[kMaxDiffPockets + pi * kBoundSlots + int(pose) % kBoundSlots], __float_as_uint(v));
  }
  const PocketDev pk = a.pockets[pi];
  LaneLig<APL> L;
  load_lane_lig<LPP, APL>(L, lg, a.L.ligs + lig, a.L.atoms, a.L.frags, a.L.tors, pk, r);
  float x[APL][3], reach = 0.f;
  Rigid rg{};
  if (XIN) {
#pragma unroll
    for (int s = 0; s < APL; ++s) {
      const float* src = a.xyz + pose * a.xyz_stride + 3 * L.aorig[s];
#pragma unroll
      for (int c = 0; c < 3; ++c) x[s][c] = APL * r + s < lg.n_atoms ? src[c] : 0.f;
    }
  } else {
    const float q = r < lg.n_dof ? a.q[pose * a.q_stride + r] : 0.f;
    rg = fk_place<LPP, APL>(L, q, r, x, S.xs);
#pragma unroll
    for (int c = 0; c < 3; ++c) reach = fmaxf(reach, fabsf(L.fxb[c]));
#pragma unroll
    for (int s = 0; s < APL; ++s) reach = fmaxf(fmaxf(reach, fabsf(L.ax[s])), fmaxf(fabsf(L.ay[s]), fabsf(L.az[s])));
#pragma unroll
    for (int k = LPP / 2; k > 0; k >>= 1) reach = fmaxf(reach, __shfl_xor(reach, k));
  }
  const float T[3] = {rg.Tx, rg.Ty, rg.Tz};
  const SumGrid sg = sum_grid(pk.grid);
#pragma unroll
  for (int s = 0; s < APL; ++s) {
    float err[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) err[c] = XIN ? 0.f : fk_spread(x[s][c], T[c], reach);
    if (APL * r + s < lg.n_atoms) mark_units(a.flag + a.unit_off[pi], sg, pk.grid, L.atype[s], x[s], err);
  }
}

template <bool XIN>
__global__ void __launch_bounds__(64) adj_mark_kernel(TermsArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const long long base = (long long)blockIdx.x * a.chunk;
  const int n = int(min((long long)a.chunk, a.n_poses - base));
  int cfg = 0;
  if (int(threadIdx.x) < n) {
    const int lig = a.pose_lig[base + threadIdx.x];
    if (lig >= 0 && lig < a.n_ligands) cfg = lane_config(a.L.ligs + lig);
  }
  for (int at = 0; at < n;) {
    const WaveForm f = next_form(cfg, at, n);
    if (f.lanes == 16)
      mark_poses<16, 1, XIN>(a, base + at, smem);
    else if (f.lanes == 32)
      mark_poses<32, 1, XIN>(a, base + at, smem);
    else if (f.lanes == 64)
      mark_poses<64, 1, XIN>(a, base + at, smem);
    else
      mark_poses<64, 2, XIN>(a, base + at, smem);
    wave_sync();
    at += f.poses;
  }
}

hipError_t launch_adj_mark(TermsArgs a, int lanes, hipStream_t s) {
  if (a.n_poses <= 0) return hipSuccess;
  a.chunk = wave_chunk(a.n_poses, lanes);
  const unsigned blocks = unsigned((a.n_poses + a.chunk - 1) / a.chunk);
  const size_t lds = wave_slab_bytes(lanes);
  if (a.xyz)
    hipLaunchKernelGGL(adj_mark_kernel<true>, dim3(blocks), dim3(64), lds, s, a);
  else
    hipLaunchKernelGGL(adj_mark_kernel<false>, dim3(blocks), dim3(64), lds, s, a);
  return hipGetLastError();
}

long long adj_units(const GridDev& g) { return (long long)kTypes * sum_grid(g).nb; }

// Calls f(unit, entry) for every marked unit of [u0, u1) (all of them where
// all(unit) says so), each with 16 lanes: a wave looks at 32 flags, then takes
// the marked ones four at a time.
constexpr int kFlagsPerWave = 32;
template <class All, class F>
DK_INLINE void for_marked_units(const unsigned char* flag, long long u0, long long u1, All&& all, F&& f) {
  const int lane = threadIdx.x & 63, grp = lane / kSumUnit;
  const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / 64,
                  n_waves = (long long)gridDim.x * blockDim.x / 64;
  for (long long base = u0 + kFlagsPerWave * wave; base < u1; base += kFlagsPerWave * n_waves) {
    const long long u = base + lane;
    uint32_t m = uint32_t(
        __builtin_amdgcn_ballot_w64(lane < kFlagsPerWave && u < u1 && (flag[u] != 0 || all(u))));
    while (m) {
      uint32_t mine = m;  // the grp-th lowest set bit
      for (int k = 0; k < grp; ++k) mine &= mine - 1;
      if (mine) f(base + __builtin_ctz(mine), lane % kSumUnit);
#pragma unroll
      for (int k = 0; k < 64 / kSumUnit; ++k) m &= m - 1;
    }
  }
}
static unsigned unit_blocks(long long units) {
  return unsigned(std::min<long long>((units + 4 * kFlagsPerWave - 1) / (4 * kFlagsPerWave), 32768));
}

// Also takes each pocket's largest bound over its slots (see mark_poses).
// fixed: bricks of 64-bit sums per unit (0: one of floats)
__global__ void __launch_bounds__(256) adj_clear_kernel(const unsigned char* flag, void* sum, int fixed, long long units,
                                                        unsigned* bound) {
  if (blockIdx.x == 0 && threadIdx.x < kMaxDiffPockets) {
    unsigned v = 0;
    for (int k = 0; k < kBoundSlots; ++k) v = max(v, bound[kMaxDiffPockets + threadIdx.x * kBoundSlots + k]);
    bound[threadIdx.x] = v;
  }
  for_marked_units(flag, 0, units, [](long long) { return false; },
                   [&](long long u, int at) {
                     if (!fixed) static_cast<float*>(sum)[u * kSumUnit + at] = 0.f;
                     for (int k = 0; k < fixed; ++k)
                       static_cast<unsigned long long*>(sum)[(u * fixed + k) * kSumUnit + at] = 0ull;
                   });
}

hipError_t launch_adj_clear(const TermsArgs& a, hipStream_t s) {
  const long long units = a.unit_off[a.n_pockets];
  if (units <= 0) return hipSuccess;
  hipLaunchKernelGGL(adj_clear_kernel, dim3(unit_blocks(units)), dim3(256), 0, s, a.flag, a.sum, a.fixed, units, a.bound);
  return hipGetLastError();
}

struct ExpandArgs {
  TermsArgs t;
  GridDev grids[kMaxDiffPockets];
};

// dL/dG[t][k] += the term's sum, or w_k S[t]: 16 lanes per marked unit, which
// reads its part of the sums once and reads and writes its part of dL/dG
// once.  Float sums are added atomically, as float contributions are in calls
// without sums: calls on several streams may add to one buffer.  Where the
// fixed-point scale says a bound was not finite, every entry of the pocket
// becomes NaN.
template <int K>
__global__ void __launch_bounds__(256) adj_expand_kernel(ExpandArgs e, long long u0, long long u1) {
  const TermsArgs& a = e.t;
  __shared__ double scale[kMaxDiffPockets];
  if (int(threadIdx.x) < a.n_pockets) scale[threadIdx.x] = a.fixed ? fixed_scale(a, threadIdx.x, K) : 1.0;
  __syncthreads();
  auto pocket_of = [&](long long u) {
    int p = 0;
    while (u >= a.unit_off[p + 1]) ++p;
    return p;
  };
  for_marked_units(a.flag, u0, u1, [&](long long u) { return scale[pocket_of(u)] == 0.0; },
                   [&](long long u, int at) {
                     const int p = pocket_of(u);
                     const GridDev& g = e.grids[p];
                     const SumGrid sg = sum_grid(g);
                     const int ub = int(u - a.unit_off[p]), t = ub / sg.nb, b = ub % sg.nb;
                     const int ix = b % sg.nbx * kSumX + at % kSumX, iy = b / sg.nbx % sg.nby * kSumY + at / kSumX % kSumY,
                               iz = b / (sg.nbx * sg.nby) * kSumZ + at / (kSumX * kSumY);
                     if (ix >= g.dims[0] || iy >= g.dims[1] || iz >= g.dims[2]) return;
                     const size_t nodes = size_t(g.dims[0]) * g.dims[1] * g.dims[2];
                     float* dst = a.dLdG[p] + size_t(t) * K * nodes + (size_t(iz) * g.dims[1] + iy) * g.dims[0] + ix;
                     const double sc = scale[p];
                     if (sc == 0.0) {
#pragma unroll
                       for (int k = 0; k < K; ++k) dst[k * nodes] += __int_as_float(0x7fc00000);
                     } else if (a.fixed) {
                       long long v[K];
#pragma unroll
                       for (int k = 0; k < K; ++k)
                         v[k] = static_cast<const long long*>(a.sum)[(u * K + k) * kSumUnit + at];
                       const double inv = 1.0 / sc;
#pragma unroll
                       for (int k = 0; k < K; ++k)
                         if (v[k] != 0) dst[k * nodes] += float(double(v[k]) * inv);
                     } else {
                       const float v = static_cast<const float*>(a.sum)[u * kSumUnit + at];
                       if (v == 0.f) return;  // no atom reaches the node
#pragma unroll
                       for (int k = 0; k < K; ++k) atomicAdd(dst + k * nodes, a.w[p * K + k] * v);
                     }
                   });
}

hipError_t launch_adj_expand(const TermsArgs& a, const GridDev* grids, int K, long long u0, long long u1, hipStream_t s) {
  if (u1 <= u0) return hipSuccess;
  ExpandArgs e;
  e.t = a;
  for (int p = 0; p < a.n_pockets; ++p) e.grids[p] = grids[p];
  if (K == 3)
    hipLaunchKernelGGL(adj_expand_kernel<3>, dim3(unit_blocks(u1 - u0)), dim3(256), 0, s, e, u0, u1);
  else
    hipLaunchKernelGGL(adj_expand_kernel<5>, dim3(unit_blocks(u1 - u0)), dim3(256), 0, s, e, u0, u1);
  return hipGetLastError();
}

// One workgroup per (pocket, term): thread t sums poses t, t + 1024, ... in
// order, then a fixed tree over the workgroup; added atomically, so that calls
// on several streams may add to one dL/dw.
__global__ void __launch_bounds__(1024) adj_wreduce_kernel(const float* __restrict__ w_pose,
                                                           const int* __restrict__ w_pocket, long long n_poses,
                                                           int K, float* dLdw) {
  __shared__ float red[1024];
  const int pi = blockIdx.x / K, k = blockIdx.x % K;
  float acc = 0.f;
#pragma unroll 4
  for (long long p = threadIdx.x; p < n_poses; p += 1024) {
    const float v = w_pose[p * K + k];
    if (w_pocket[p] == pi) acc += v;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(dLdw + pi * K + k, red[0]);
}

hipError_t launch_adj_wreduce(const float* w_pose, const int* w_pocket, long long n_poses, int n_pockets, int K,
                              float* dLdw, hipStream_t s) {
  if (n_pockets * K <= 0) return hipSuccess;
  hipLaunchKernelGGL(adj_wreduce_kernel, dim3(unsigned(n_pockets * K)), dim3(1024), 0, s, w_pose, w_pocket,
                     n_poses, K, dLdw);
  return hipGetLastError();
}

// ================================================================ sampler

template <int APL>
DK_INLINE float wrap_clamp(float q, int r, const LaneLig<APL>& L) {
  if (r < 3) return fminf(fmaxf(q, L.lo), L.hi);
  return wrap_angle(q);
}

// FULL: line search and logged trajectories, where every evaluation gives E
// and the gradient.  Otherwise the first-order rules use the energy of a
// step's last evaluation only and no gradient there, so the n_local
// evaluations before it compute the gradient alone and that one (like the
// initial pose's) the energy alone.  With the slot records cut to one read
// per pass, 256 ligands of 10-60 atoms x 128 trajectories x 100 steps went
// from 46.8 to 43.0 ms, 2,048 ligands of 10-70 atoms in 16 pockets x 64 x 30
// from 83.2 to 65.1 ms (the kernel is bound by VALU issue, then LDS).
// The FULL kernel has one evaluation site for its first-order rules and its line
// search: with one for each it spilled 264 bytes a lane (two atoms per lane), now
// 176, and 512 ligands of 10-60 atoms x 64 x 3 line-searched steps took 6.62 ms,
// now 5.66 (logged Adam steps: 2.12 and 1.82).
template <int LPP, int APL, int MODE, bool FULL>
DK_INLINE void run_traj(const SampleArgs& a, LaneLig<APL>& L, const PocketDev& pk, const MdnArg& mdn,
                        const PairRec* pairs,
                        const GroupSlab& S, int lig, int traj, int r) {
  const size_t ti = size_t(lig) * a.n_traj + traj;
  const uint32_t k0 = uint32_t(lig), k1 = uint32_t(a.step_base[1]);
  const bool dof = r < L.n_dof;
  const int qs = a.q_stride;
  int nev = a.n_evals[ti];
  float* trow = nullptr;
  if (FULL && a.trace && lig % a.trace_stride == 0 && traj < a.trace_traj)
    trow = a.trace + (size_t(lig / a.trace_stride) * a.trace_traj + traj) * size_t(a.trace_cap) * (2 * qs + 1);
  auto record = [&](float qv, float gv, float Ev) {
    if (trow && nev < a.trace_cap) {
      float* row = trow + size_t(nev) * (2 * qs + 1);
      if (r < qs) {
        row[r] = dof ? qv : 0.f;
        row[qs + r] = dof ? gv : 0.f;
      }
      if (r == 0) row[2 * qs] = Ev;
    }
    ++nev;
  };
  if (a.init) {
    const uint4 w = philox4x32_10(make_uint4(uint32_t(traj), 0u, 0u, uint32_t(r >> 2)), k0, k1);
    const float q = dof ? L.lo + (L.hi - L.lo) * u01(pick4(w, r & 3)) : 0.f;
    const EvalOut o =
        eval_pose<LPP, APL, FULL ? kWantBoth : kWantE, false, MODE>(L, q, pk, pairs, S, r, nullptr, nullptr, mdn);
    record(q, o.g, o.E);
    if (dof) {
      a.q_cur[ti * qs + r] = q;
      a.q_best[ti * qs + r] = q;
    }
    if (r == 0) {
      a.E_cur[ti] = o.E;
      a.E_best[ti] = o.E;
      a.n_evals[ti] = nev;
    }
    return;
  }
  float q = dof ? a.q_cur[ti * qs + r] : 0.f;
  float qb = dof ? a.q_best[ti * qs + r] : 0.f;
  float Ecur = a.E_cur[ti], Ebest = a.E_best[ti];
  const int base = *a.step_base + a.step_off;
  for (int s = base + 1; s <= base + a.step_count; ++s) {
    const uint4 w = philox4x32_10(make_uint4(uint32_t(traj), uint32_t(s), 1u, 0u), k0, k1);
    const int j = int(__umulhi(w.x, uint32_t(L.n_dof)));
    float qn = q;
    if (r == j) qn = L.lo + (L.hi - L.lo) * u01(w.y);
    float E = 0.f;
    // first-order update of qn from the gradient g (Adam by default; the Table
    // S5 alternatives otherwise)
    float m = 0.f, v = 0.f, b1t = 1.f, b2t = 1.f;
    auto update = [&](float g) {
      // square roots and quotients on the hardware units (about 1 ulp;
      // the IEEE-exact sequences cost ~12 instructions each)
      float step;
      if (a.local_opt == DOCK_LOCAL_SGD) {
        step = a.lr * g;
      } else if (a.local_opt == DOCK_LOCAL_RMSPROP) {
        v = a.rms_alpha * v + (1.f - a.rms_alpha) * g * g;
        step = a.lr * g * rcp_hw(sqrt_hw(v) + a.eps);
      } else if (a.local_opt == DOCK_LOCAL_ADAGRAD) {
        v += g * g;
        step = a.lr * g * rcp_hw(sqrt_hw(v) + a.eps);
      } else {
        if (a.local_opt == DOCK_LOCAL_ADAMW) qn *= 1.f - a.lr * a.weight_decay;
        m = a.b1 * m + (1.f - a.b1) * g;
        v = a.b2 * v + (1.f - a.b2) * g * g;
        b1t *= a.b1;
        b2t *= a.b2;
        const float mh = m * rcp_hw(1.f - b1t), vh = v * rcp_hw(1.f - b2t);
        step = a.lr * mh * rcp_hw(sqrt_hw(vh) + a.eps);
      }
      if (dof) qn = wrap_clamp(qn - step, r, L);
    };
    if (!FULL) {
      for (int t = 0; t < a.n_local; ++t) {
        update(eval_pose<LPP, APL, kWantG, false, MODE>(L, qn, pk, pairs, S, r, nullptr, nullptr, mdn).g);
        ++nev;
      }
      E = eval_pose<LPP, APL, kWantE, false, MODE>(L, qn, pk, pairs, S, r, nullptr, nullptr, mdn).E;
      ++nev;
    } else {
      // one evaluation site for both rules.  First order: n_local gradient
      // evaluations with an update after each, then the energy of the refined
      // pose.  Armijo line search as a loop over trial poses: the first call
      // scores the perturbed pose; each search tries alpha = 1, 1/2, ...,
      // 2^-10 along -g/|g|; a failed search ends the refinement (m, v, b1t:
      // its gradient, direction and slope)
      const bool line = a.local_opt == DOCK_LOCAL_LINESEARCH;
      float qtry = qn, alpha = 1.f;
      int done_steps = -1, halvings = 0;
      for (;;) {
        const EvalOut o = eval_pose<LPP, APL, kWantBoth, false, MODE>(L, qtry, pk, pairs, S, r, nullptr, nullptr, mdn);
        record(qtry, o.g, o.E);
        if (!line) {
          E = o.E;
          if (++done_steps == a.n_local) break;
          update(o.g);
          qtry = qn;
          continue;
        }
        if (done_steps < 0 || o.E <= E + 1e-4f * alpha * b1t) {
          qn = qtry;
          E = o.E;
          m = o.g;
          ++done_steps;
        } else {
          if (++halvings > 10) break;
          alpha *= 0.5f;
          qtry = dof ? wrap_clamp(qn + alpha * v, r, L) : 0.f;
          continue;
        }
        if (done_steps >= a.n_local) break;
        const float gn = sqrtf(group_sum<LPP>(dof ? m * m : 0.f));
        if (!(gn > 0.f)) break;
        v = dof ? -m / gn : 0.f;
        b1t = -gn;
        alpha = 1.f;
        halvings = 0;
        qtry = dof ? wrap_clamp(qn + v, r, L) : 0.f;
      }
    }
    const float u = u01(w.z);
    const bool acc = u < expf(-a.mc_beta * (E - Ecur));
    if (acc) {
      q = qn;
      Ecur = E;
    }
    if (E < Ebest) {
      qb = qn;
      Ebest = E;
    }
  }
  if (dof) {
    a.q_cur[ti * qs + r] = q;
    a.q_best[ti * qs + r] = qb;
  }
  if (r == 0) {
    a.E_cur[ti] = Ecur;
    a.E_best[ti] = Ebest;
    a.n_evals[ti] = nev;
  }
}

// A pointer that is the same in every lane, in scalar registers.
template <class T>
DK_INLINE T* wave_uniform(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v)))),
                 hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32))));
  return reinterpret_cast<T*>(uint64_t(hi) << 32 | lo);
}

// Three waves per SIMD (168 VGPRs).  With two atoms per lane the step loop
// needs more and spills a few registers to scratch (served from L2, outside
// the pair-pass loop); two waves per SIMD without spills measured slower.
template <int LPP, int APL, int BLOCK, int MODE, bool FULL>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(3))) sample_kernel(SampleArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int GPB = BLOCK / LPP;
  const int grp = threadIdx.x / LPP, r = threadIdx.x % LPP;
  PairRec* sp = reinterpret_cast<PairRec*>(smem);
  unsigned char* slabs = smem + pair_bytes(a.max_pairs);
  const GroupSlab S = make_slab<LPP, APL>(slabs + size_t(grp) * slab_bytes(LPP, APL));
  int* s_item = reinterpret_cast<int*>(slabs + size_t(GPB) * slab_bytes(LPP, APL));
  int taken = 0;
  // persistent: partitions in turn from the block's own (b mod n_part); a
  // partition is left for good once its counter passes its size, so every
  // block exits after at most n_part empty pops
  const int home = a.queue ? int(blockIdx.x % unsigned(a.n_part)) : 0;
  int tried = 0;
  for (;;) {
    if (threadIdx.x == 0) {
      int it = a.n_items;
      if (a.queue) {
        while (tried < a.n_part) {
          int q = home + tried;
          if (q >= a.n_part) q -= a.n_part;
          const int lo = a.part_off[q], n = a.part_off[q + 1] - lo;
          const int k = n > 0 ? atomicAdd(a.queue + q, 1) : n;
          if (k < n) {
            it = lo + k;
            break;
          }
          ++tried;
        }
      } else {
        it = taken == 0 ? int(blockIdx.x) : a.n_items;
      }
      *s_item = it;
    }
    __syncthreads();
    const int item = *s_item;
    __syncthreads();
    if (item >= a.n_items) break;
    ++taken;
    const int2 wi = a.items[item];
    const int lig = wi.x;
    // one atom per lane: the alternative layout (the primary one for every
    // ligand not laid out with two atoms per lane)
    LigDev lg = a.L.ligs[lig];
    if (APL == 1) use_alt_layout(lg);
    for (int p = threadIdx.x; p < lg.n_stage; p += BLOCK) sp[p] = a.L.pairs[lg.pair_off + p];
    __syncthreads();
    const int traj = wi.y + grp;
    if (traj < a.n_traj) {
      PocketDev pk = a.pockets[lg.pocket];
      MdnArg mdn = mdn_for(a.L, lg, pk);
      if (MODE == kModeGridMdn) {
        // a workgroup has one ligand: the residue loops' pointers go to scalar
        // registers (in vector registers they were spilled, and read from
        // scratch for every residue: 512 ligands x 64 x 3 steps, line search
        // 46.9 ms so and 40.1 now, Adam 12.4 and 11.1)
        pk.mcell_start = wave_uniform(pk.mcell_start);
        pk.mcell_res = wave_uniform(pk.mcell_res);
        pk.res_range = wave_uniform(pk.res_range);
        pk.res_xyz = wave_uniform(pk.res_xyz);
        mdn.par = wave_uniform(mdn.par);
      }
      LaneLig<APL> L;
      load_lane_lig<LPP, APL>(L, lg, a.L.ligs + lig, a.L.atoms, a.L.frags, a.L.tors, pk, r);
      run_traj<LPP, APL, MODE, FULL>(a, L, pk, mdn, sp, S, lig, traj, r);
    }
    __syncthreads();
  }
}

// Runs that log trajectories or search along a line evaluate E and the
// gradient every time.
static bool full_evals(int local_opt, bool trace) { return trace || local_opt == DOCK_LOCAL_LINESEARCH; }

template <int LPP, int APL, int BLOCK, int MODE>
static hipError_t launch_sample_t(const SampleArgs& a, int grid, hipStream_t s) {
  const size_t lds = sample_lds_bytes(LPP, APL, BLOCK, a.max_pairs);
  if (full_evals(a.local_opt, a.trace != nullptr))
    hipLaunchKernelGGL((sample_kernel<LPP, APL, BLOCK, MODE, true>), dim3(grid), dim3(BLOCK), lds, s, a);
  else
    hipLaunchKernelGGL((sample_kernel<LPP, APL, BLOCK, MODE, false>), dim3(grid), dim3(BLOCK), lds, s, a);
  return hipGetLastError();
}

#define DOCK_SAMPLE_CASES(X)                                                                      \
  X(16, 1, 64) X(32, 1, 64) X(64, 1, 64) X(32, 2, 64) X(64, 2, 64) X(16, 1, 128) X(32, 1, 128)    \
      X(64, 1, 128) X(32, 2, 128) X(64, 2, 128) X(16, 1, 256) X(32, 1, 256) X(64, 1, 256)          \
          X(32, 2, 256) X(64, 2, 256)

hipError_t launch_sample(const SampleArgs& a, int lpp, int apl, int grid, int block, int mode,
                         hipStream_t s) {
  if (grid <= 0) return hipSuccess;
#define X(L, A, B)                                                                     \
  if (lpp == L && apl == A && block == B) {                                            \
    if (mode == kModeDirect) return launch_sample_t<L, A, B, kModeDirect>(a, grid, s); \
    if (mode == kModeGridMdn) return launch_sample_t<L, A, B, kModeGridMdn>(a, grid, s); \
    return launch_sample_t<L, A, B, kModeGrid>(a, grid, s);                            \
  }
  DOCK_SAMPLE_CASES(X)
#undef X
  return hipErrorInvalidValue;
}

template <int L, int A, int B, bool FULL>
static int blocks_per_cu(int mode, size_t lds) {
  int n = 0;
  hipError_t e;
  if (mode == kModeDirect)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sample_kernel<L, A, B, kModeDirect, FULL>, B, lds);
  else if (mode == kModeGridMdn)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sample_kernel<L, A, B, kModeGridMdn, FULL>, B, lds);
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sample_kernel<L, A, B, kModeGrid, FULL>, B, lds);
  if (e != hipSuccess) n = 1;
  return n > 0 ? n : 1;
}

int sample_max_blocks_per_cu(int lpp, int apl, int block, int mode, int local_opt, bool trace, size_t lds) {
  const bool full = full_evals(local_opt, trace);
#define X(L, A, B)                              \
  if (lpp == L && apl == A && block == B)       \
    return full ? blocks_per_cu<L, A, B, true>(mode, lds) : blocks_per_cu<L, A, B, false>(mode, lds);
  DOCK_SAMPLE_CASES(X)
#undef X
  return 1;
}

// ================================================================ best poses

// Sort key of (value, index): the value's bits mapped to an unsigned key that
// sorts like the float (-0.0 as +0.0, every NaN after +inf), the index
// breaking ties.
DK_INLINE unsigned long long rank_key(float v, int idx) {
  uint32_t u = __float_as_uint(v);
  if (v != v) u = 0xffffffffu;
  else if (u == 0x80000000u) u = 0u;
  if (u != 0xffffffffu) u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (static_cast<unsigned long long>(u) << 32) | static_cast<uint32_t>(idx);
}

// rank_key of a candidate, from which its energy comes back bit for bit (the
// lowest bit marks -0.0): a caller may let the outputs take the place of the
// energies, which are not read again once they are sorted.
DK_INLINE unsigned long long best_key(float e, int idx) {
  return rank_key(e, int(uint32_t(idx) << 1 | (__float_as_uint(e) == 0x80000000u ? 1u : 0u)));
}
DK_INLINE float best_energy(unsigned long long key) {
  const uint32_t u = uint32_t(key >> 32);
  return __uint_as_float((key & 1u) ? 0x80000000u : ((u & 0x80000000u) ? u ^ 0x80000000u : ~u));
}

// RMSD^2 sum of the lane's atoms against a pose in LDS.
template <int APL>
DK_INLINE float sq_diff(const float (&x)[APL][3], const float4* y, int n_atoms, int r) {
  float acc = 0.f;
#pragma unroll
  for (int s = 0; s < APL; ++s) {
    const int atom = APL * r + s;
    if (atom < n_atoms) {
      const float4 v = y[atom];
      const float dx = x[s][0] - v.x, dy = x[s][1] - v.y, dz = x[s][2] - v.z;
      acc += dx * dx + dy * dy + dz * dz;
    }
  }
  return acc;
}

// A workgroup per ligand: the candidates' keys sorted in LDS, then W at a
// time (one per wave) placed, compared with the kept poses and, in order,
// with those of the same turn that were kept.  Bound by the latency of a
// turn's placement and comparisons, which four waves share where ligands are
// few (one ligand with 1,024 candidates: 134 -> 27 us, the sort included);
// LDS is sized by the handle's largest ligand (4,096 ligands x 64 candidates:
// 157 -> 122 us).
template <int W>
__global__ void __launch_bounds__(64 * W) best_kernel(BestArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int LPP = 64, APL = 2;
  __shared__ int s_kept[W];
  const int lig = blockIdx.x, tid = threadIdx.x, r = tid & 63, wv = tid >> 6;
  unsigned long long* key = reinterpret_cast<unsigned long long*>(smem);
  float4* kept = reinterpret_cast<float4*>(smem + (size_t(a.t_pad) * 8 + 15) / 16 * 16);  // [top_n][max_atoms]
  float4* cand = kept + size_t(a.top_n) * a.max_atoms;                                     // [W][max_atoms], W > 1
  const LigDev lg = a.L.ligs[lig];
  PocketDev none;
  none.preset = DOCK_PRESET_TRIDS;
  none.n_terms = 0;
  LaneLig<APL> L;
  load_lane_lig<LPP, APL>(L, lg, a.L.ligs + lig, a.L.atoms, a.L.frags, a.L.tors, none, r);
  const int T = a.n_traj;
  const unsigned long long inf_key = rank_key(INFINITY, 0);
  for (int i = tid; i < a.t_pad; i += 64 * W) {
    float e = i < T ? a.E_best[size_t(lig) * T + i] : INFINITY;
    if (!(e < INFINITY)) e = INFINITY;  // NaN and +inf rank last
    key[i] = best_key(e, i < T ? i : 0x7fffffff);
  }
  auto sync = [] {
    if (W > 1)
      __syncthreads();
    else
      wave_sync();
  };
  sync();
  for (int k = 2; k <= a.t_pad; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int p = tid; p < a.t_pad / 2; p += 64 * W) {
        const int lo = 2 * p - (p & (j - 1)), hi = lo + j;
        const unsigned long long kl = key[lo], kh = key[hi];
        if ((kl > kh) == ((lo & k) == 0)) {
          key[lo] = kh;
          key[hi] = kl;
        }
      }
      sync();
    }
  }
  int n_kept = 0;
  const float inv_n = 1.0f / float(lg.n_atoms);
  auto near = [&](float acc) { return sqrtf(group_sum<64>(acc) * inv_n) < a.rmsd_cut; };
  // this wave's candidate of the next turn: read ahead of the comparisons
  auto cand_of = [&](int c) { return c < T && key[c] < inf_key ? int(uint32_t(key[c]) >> 1) : -1; };
  auto q_of = [&](int t) {
    return t >= 0 && r < lg.n_dof ? a.q_best[(size_t(lig) * T + t) * a.q_stride + r] : 0.f;
  };
  int t = cand_of(wv);
  float q = q_of(t);
  for (int c = 0; c < T && n_kept < a.top_n && key[c] < inf_key; c += W) {
    const int t_next = cand_of(c + W + wv);
    const float q_next = q_of(t_next);
    float x[APL][3];
    fk_place_shfl<LPP, APL>(L, q, r, x);
    bool dup = t < 0;
    int k = 0;
    for (; k + 4 <= n_kept && !dup; k += 4) {
      // four at a time: their sums and square roots overlap
      float acc[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] = sq_diff<APL>(x, kept + size_t(k + m) * a.max_atoms, lg.n_atoms, r);
#pragma unroll
      for (int m = 0; m < 4; ++m) dup |= near(acc[m]);
    }
    for (; k < n_kept && !dup; ++k) dup = near(sq_diff<APL>(x, kept + size_t(k) * a.max_atoms, lg.n_atoms, r));
    if (W > 1) {
#pragma unroll
      for (int s = 0; s < APL; ++s)
        if (APL * r + s < lg.n_atoms) cand[wv * a.max_atoms + APL * r + s] = make_float4(x[s][0], x[s][1], x[s][2], 0.f);
      if (r == 0) s_kept[wv] = !dup;
      __syncthreads();
      // in order: a candidate is compared with those of this turn that stay
      for (int m = 0; m + 1 < W; ++m) {
        const bool stays = s_kept[m];
        if (stays && wv > m && !dup) {
          dup = near(sq_diff<APL>(x, cand + m * a.max_atoms, lg.n_atoms, r));
          if (dup && r == 0) s_kept[wv] = 0;
        }
        __syncthreads();
      }
    }
    // slots in order, up to top_n
    int slot = n_kept;
    if (W > 1) {
      int total = n_kept;
#pragma unroll
      for (int m = 0; m < W; ++m) {
        slot += m < wv && s_kept[m];
        total += s_kept[m];
      }
      n_kept = min(total, a.top_n);
    } else if (!dup) {
      ++n_kept;
    }
    if (!dup && slot < a.top_n) {
      const size_t o = size_t(lig) * a.top_n + slot;
#pragma unroll
      for (int s = 0; s < APL; ++s) {
        const int atom = APL * r + s;
        if (atom < lg.n_atoms) {
          kept[size_t(slot) * a.max_atoms + atom] = make_float4(x[s][0], x[s][1], x[s][2], 0.f);
          if (a.xyz_out) {
            float* dst = a.xyz_out + o * a.xyz_stride + 3 * L.aorig[s];
            dst[0] = x[s][0];
            dst[1] = x[s][1];
            dst[2] = x[s][2];
          }
        }
      }
      if (r == 0) {
        const float E = best_energy(key[c + wv]);
        if (a.E_out) a.E_out[o] = E;
        if (a.E_screen) a.E_screen[o] = E / (1.0f + a.w_tor * float(lg.n_tors));
        if (a.idx_out) a.idx_out[o] = t;
      }
      if (a.q_out && r < a.q_stride) a.q_out[o * a.q_stride + r] = r < lg.n_dof ? q : 0.f;
    }
    sync();
    t = t_next;
    q = q_next;
  }
  if (wv > 0) return;
  for (int k = n_kept; k < a.top_n; ++k) {
    const size_t o = size_t(lig) * a.top_n + k;
    if (r == 0) {
      if (a.E_out) a.E_out[o] = INFINITY;
      if (a.E_screen) a.E_screen[o] = INFINITY;
      if (a.idx_out) a.idx_out[o] = -1;
    }
    if (a.q_out && r < a.q_stride) a.q_out[o * a.q_stride + r] = 0.f;
  }
  if (r == 0 && a.n_out) a.n_out[lig] = n_kept;
}

hipError_t launch_best(const BestArgs& a, hipStream_t s) {
  if (a.n_ligands <= 0) return hipSuccess;
  auto lds = [&](int waves) {
    return (size_t(a.t_pad) * 8 + 15) / 16 * 16 + size_t(a.top_n + (waves > 1 ? waves : 0)) * a.max_atoms * 16;
  };
  // Four waves per ligand share a turn's placement and comparisons, one wave
  // spends less on a workgroup and stops at its first kept pose.  So four where
  // there are several poses to keep and a CU holds few ligands (by their number
  // and by the LDS): a turn's waves then overlap what the ligands alone leave
  // idle.  Or a long sort, where few ligands wait for it.  Far-apart candidates,
  // us with one wave and with four: 64 candidates, best 8: 512 ligands 27.3 and
  // 14.7, 2,048 32.0 and 30.0, 4,096 47.0 and 50.3; best 24 of 4,096 (six
  // ligands a CU by their LDS) 332 and 167; best 1 of 1,024 8.3 and 11.9, of
  // 4,096 11.0 and 30.9; 256 candidates, best 1: 512 ligands 14.0 and 13.3,
  // 2,048 16.1 and 25.3.  (No more poses are kept than there are candidates.)
  // Best 8 of 4,096 ligands x 64 candidates of which many are near each other,
  // with its rank: 174 and 168 us the calls; 16,384 x 16: 220 and 246.
  constexpr int kCus = 256;
  const int resident = int(std::min<size_t>((size_t(a.n_ligands) + kCus - 1) / kCus, 160 * 1024 / lds(1)));
  const int keep = std::min(a.top_n, a.n_traj);
  const bool four = keep >= std::max(4, resident) || (keep >= 8 && a.n_ligands <= 16 * kCus) ||
                    (keep >= 2 && resident <= 1) || (a.n_traj >= 256 && resident <= 2);
  if (four && lds(4) <= 64 * 1024)
    hipLaunchKernelGGL(best_kernel<4>, dim3(a.n_ligands), dim3(256), lds(4), s, a);
  else
    hipLaunchKernelGGL(best_kernel<1>, dim3(a.n_ligands), dim3(64), lds(1), s, a);
  return hipGetLastError();
}

// ================================================================ screening rank

// A workgroup sorts a block of 2,048 keys, two per thread (elements 2 t and
// 2 t + 1).  Exchanges within a thread's pair are free and those within a
// wave are shuffles, so only distances of 128 and more, 10 of the 66 steps, go
// through LDS with a barrier (2,048 scores: 46 us with every step in LDS on 256
// threads and the values carried along, 15 so).
__global__ void __launch_bounds__(kRankBlock / 2) rank_kernel(RankArgs a) {
  __shared__ unsigned long long key[kRankBlock];
  const long long base = (long long)blockIdx.x * kRankBlock;
  const int tid = threadIdx.x;
  unsigned long long k2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const long long e = base + 2 * tid + h;
    k2[h] = ~0ull;
    if (e < a.n) {
      const float v = a.idx ? a.score[e] : a.score[e * a.stride];
      const int id = a.idx ? a.idx[e] : int(e);
      // an empty slot of an earlier pass (index -1) stays empty
      if (id >= 0) k2[h] = rank_key(v, id);
    }
  }
  auto order = [](unsigned long long& lo, unsigned long long& hi, bool up) {
    if ((lo > hi) == up) {
      const unsigned long long t = lo;
      lo = hi;
      hi = t;
    }
  };
  for (int size = 2; size <= kRankBlock; size <<= 1) {
    const bool up = ((2 * tid) & size) == 0;
    for (int stride = size >> 1; stride > 64; stride >>= 1) {
      // through LDS: thread t takes the pair (lo, lo + stride)
      key[2 * tid] = k2[0];
      key[2 * tid + 1] = k2[1];
      __syncthreads();
      const int lo = 2 * tid - (tid & (stride - 1));
      unsigned long long x = key[lo], y = key[lo + stride];
      order(x, y, (lo & size) == 0);
      key[lo] = x;
      key[lo + stride] = y;
      __syncthreads();
      k2[0] = key[2 * tid];
      k2[1] = key[2 * tid + 1];
      __syncthreads();
    }
    for (int stride = size >> 1 > 64 ? 64 : size >> 1; stride > 1; stride >>= 1) {
      // partner thread t ^ (stride / 2) holds elements 2 t + h +- stride
      const bool low = (tid & (stride / 2)) == 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const unsigned long long o = __shfl_xor(k2[h], stride / 2);
        const bool take = (k2[h] > o) == (low == up);
        if (take && k2[h] != o) k2[h] = o;
      }
    }
    order(k2[0], k2[1], up);
  }
  // values from the ligands' scores, read before any is written (a caller may
  // rank in place)
  const int keep = a.k < kRankBlock ? a.k : kRankBlock;
  float v2[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    v2[h] = __int_as_float(0x7f800000);
    if (2 * tid + h < keep && k2[h] != ~0ull) v2[h] = a.all[(long long)(uint32_t(k2[h])) * a.stride_all];
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = 2 * tid + h;
    if (t >= keep) continue;
    a.out_score[(long long)blockIdx.x * keep + t] = v2[h];
    a.out_idx[(long long)blockIdx.x * keep + t] = k2[h] == ~0ull ? -1 : int(uint32_t(k2[h]));
  }
}

hipError_t launch_rank(const RankArgs& a, hipStream_t s) {
  const long long nb = (a.n + kRankBlock - 1) / kRankBlock;
  const unsigned blocks = unsigned(nb > 0 ? nb : 1);
  hipLaunchKernelGGL(rank_kernel, dim3(blocks), dim3(kRankBlock / 2), 0, s, a);
  return hipGetLastError();
}

// ================================================================ Philox dump

__global__ void philox_kernel(const uint4* ctr, uint32_t k0, uint32_t k1, long long n, uint4* out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = philox4x32_10(ctr[i], k0, k1);
}

hipError_t launch_philox(const uint32_t* ctr, uint32_t k0, uint32_t k1, long long n, uint32_t* out,
                         hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(philox_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const uint4*>(ctr), k0, k1, n, reinterpret_cast<uint4*>(out));
  return hipGetLastError();
}

// ================================================================ small helpers

__global__ void fill_int_kernel(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void add_int_kernel(int* p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p += v;
}

hipError_t launch_fill_int(int* p, int n, int v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_int_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}
__global__ void fill_u32_kernel(uint32_t* p, long long n, uint32_t v) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x)
    p[i] = v;
}
hipError_t launch_fill_u32(uint32_t* p, long long n, uint32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const long long blocks = std::min<long long>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(unsigned(blocks)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}
hipError_t launch_add_int(int* p, int v, hipStream_t s) {
  hipLaunchKernelGGL(add_int_kernel, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

}  // namespace dock
