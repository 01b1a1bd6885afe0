// Kernel argument blocks and launchers (host <-> device interface of libdock).
#pragma once

#include "dock_internal.h"

namespace dock {

struct PairRec;

struct LigandArrays {
  const LigDev* ligs;
  const float4* atoms;   // DFS order; w = bits(type | frag << 8 | caller index << 16)
  const FragDev* frags;
  const TorsDev* tors;
  const PairRec* pairs;
  // E_MDN mixture parameters, float4 (pi, mu, log2(e) / (2 sigma^2),
  // 1 / sigma^2) per [atom (DFS, global)][residue][gaussian]; null if none
  const float4* mdn;
  int mdn_res, mdn_k;
};

struct ScoreArgs {
  LigandArrays L;
  const PocketDev* pockets;
  int n_ligands, n_pockets;
  long long n_poses;
  const int* pose_lig;
  const float* q;
  int q_stride;
  float* E;
  float* dEdq;
  float* xyz;
  int xyz_stride;
  int chunk;            // poses per wavefront
  unsigned slab_bytes;  // LDS of a wavefront's slabs
};

constexpr int kMaxDiffPockets = 16;
constexpr int kBoundSlots = 32;
constexpr int kBoundWords = kMaxDiffPockets * (1 + kBoundSlots);

struct TermsArgs {
  LigandArrays L;
  const PocketDev* pockets;  // grid geometry per pocket
  int n_ligands, n_pockets;
  long long n_poses;
  const int* pose_lig;
  const float* q;            // pose DOFs (coordinates mode: null)
  int q_stride;
  const float* xyz;          // world coordinates, caller atom order (DOF mode: null)
  int xyz_stride;
  const float* G[kMaxDiffPockets];   // per-term maps per pocket
  const float* w;                    // device [n_pockets * K]
  float* E;
  const float* dLdE;                 // null: forward only
  float* dLdG[kMaxDiffPockets];
  float* dLdw;
  float* dLdq;
  float* dLdx;
  int chunk;                         // poses per wavefront
  // dL/dG through per-pocket sums (null: float atomics into dLdG): flags of
  // the units, the sums (floats, one brick per unit; or, when fixed = K, 64-bit
  // fixed point, K bricks per unit), the first unit of each pocket (no units:
  // no dL/dG wanted), and for the fixed-point scale the largest |dLdE| * atoms
  // of a pocket's poses (FP32 bits): bound[pocket], after launch_adj_clear,
  // from kBoundSlots slots per pocket behind
  unsigned char* flag;
  void* sum;
  int fixed;
  long long unit_off[kMaxDiffPockets + 1];
  unsigned* bound;
  // dL/dw in a fixed order (null: float atomics): per-pose contributions
  // w_pose [n_poses * K] and the pose's pocket w_pocket [n_poses] (-1: invalid
  // ligand), reduced afterwards
  float* w_pose;
  int* w_pocket;
};

// The passes around launch_terms when a.sum is set: units marked (flag and
// bound cleared by the caller), the marked units' sums cleared, and after
// launch_terms the units [u0, u1) added to dLdG.
hipError_t launch_adj_mark(TermsArgs a, int lanes, hipStream_t s);
hipError_t launch_adj_clear(const TermsArgs& a, hipStream_t s);
hipError_t launch_adj_expand(const TermsArgs& a, const GridDev* grids, int K, long long u0, long long u1, hipStream_t s);
// units of a pocket
long long adj_units(const GridDev& g);
// dLdw[pi * K + k] += sum over poses p with w_pocket[p] == pi of w_pose[p * K + k],
// in a fixed order
hipError_t launch_adj_wreduce(const float* w_pose, const int* w_pocket, long long n_poses, int n_pockets, int K,
                              float* dLdw, hipStream_t s);

struct SampleArgs {
  LigandArrays L;
  const PocketDev* pockets;
  const int2* items;      // (ligand, first trajectory)
  int n_items;
  int* queue;             // persistent work counters (one per partition), or null:
                          // item = blockIdx.x
  const int* part_off;    // n_part + 1 item bounds of the partitions
  int n_part;             // block b takes partition b mod n_part first, then the others
  const int* step_base;   // device: [0] MC steps already taken, [1] the seed
  int step_off;           // this launch covers steps base+off+1 .. base+off+count
  int step_count;
  int init;               // draw initial poses and score them instead of stepping
  int n_traj, q_stride;
  int n_local, local_opt;
  float lr, b1, b2, eps, mc_beta, rms_alpha, weight_decay;
  float* q_cur;
  float* E_cur;
  float* q_best;
  float* E_best;
  int* n_evals;
  float* trace;
  int trace_cap;
  int trace_stride, trace_traj;  // logged: ligands l % stride == 0, trajectories < trace_traj
  int max_pairs;
};

struct BestArgs {
  LigandArrays L;
  int n_ligands, n_traj, q_stride;
  const float* E_best;
  const float* q_best;
  int top_n;
  float rmsd_cut, w_tor;
  float* E_out;
  float* E_screen;
  float* q_out;
  int* idx_out;
  float* xyz_out;
  int xyz_stride;
  int* n_out;
  int t_pad, max_atoms;  // candidates padded to a power of two; largest ligand of the handle
};

struct MapArgs {
  const float4* rec;  // xyz, w = bits(type)
  int n_rec;
  GridDev grid;
  int preset, n_terms;
  float w[kMaxTerms];
  TypePair tab[kTypes * kTypes];
  float* G;  // [8][K][nodes] or null
  float* M;  // [8][nodes]
};

// Adjoint of the TRIDS map build: dL/d(receptor xyz) and dL/dtheta for
// theta = (mu_long, sigma_long, mu_hb, sigma_hb, d_clash_hb, R_0..R_7).
constexpr int kMapTheta = 5 + kTypes;
struct MapAdjArgs {
  const float4* rec;   // xyz, w = bits(type), caller order
  int n_rec;
  GridDev grid;
  TypePair tab[kTypes * kTypes];
  const float* lam;    // dL/dG [8][3][nodes]
  float* dLdxyz;       // [n_rec * 3], +=
  double* dLdtheta;    // [kMapTheta], +=
  unsigned long long* mask;  // scratch, a bit per node in words of one brick (map_adjoint_bricks), or
                             // null: every node counts as holding a nonzero lambda
};
long long map_adjoint_bricks(const GridDev& g);
hipError_t launch_map_adjoint(const MapAdjArgs& a, hipStream_t s);

// LDS bytes a sampler block of `block` threads needs.
size_t sample_lds_bytes(int lpp, int apl, int block, int max_pairs);
// LDS of the groups of one wavefront with their pair records.
size_t group_lds_bytes(int lpp, int apl, int max_pairs);

hipError_t launch_map_build(const MapArgs& a, hipStream_t s);
// mode: 0 grid maps, 1 direct pair sums, 2 grid maps + E_MDN
// (lanes: of the handle's widest ligand, 16, 32 or 64; 128 where one has more
// than 64 atoms, two a lane)
hipError_t launch_score(ScoreArgs a, int lanes, int mode, hipStream_t s);
hipError_t launch_sample(const SampleArgs& a, int lpp, int apl, int grid, int block, int mode,
                         hipStream_t s);
hipError_t launch_best(const BestArgs& a, hipStream_t s);

// Screening rank: one pass reduces every block of kRankBlock (score, index)
// entries to its k smallest.
constexpr int kRankBlock = 2048;
struct RankArgs {
  const float* score;  // first pass: strided ligand scores; later: packed
  const int* idx;      // null on the first pass (index = position)
  long long n;
  int stride;
  int k;
  const float* all;    // the ligands' scores (ligand i at all[i * stride_all]): what an output value is read from
  int stride_all;
  float* out_score;
  int* out_idx;
};
hipError_t launch_rank(const RankArgs& a, hipStream_t s);
hipError_t launch_terms(TermsArgs a, int lanes, int K, hipStream_t s);
hipError_t launch_philox(const uint32_t* ctr, uint32_t k0, uint32_t k1, long long n, uint32_t* out,
                         hipStream_t s);
hipError_t launch_fill_int(int* p, int n, int v, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, long long n, uint32_t v, hipStream_t s);
hipError_t launch_add_int(int* p, int v, hipStream_t s);
int sample_max_blocks_per_cu(int lpp, int apl, int block, int mode, int local_opt, bool trace, size_t lds);

}  // namespace dock
