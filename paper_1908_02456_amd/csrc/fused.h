// Fused single-pass Taylor-4 step (face form with a local boundary operator,
// Dirichlet and periodic boxes).  Declarations shared with the C ABI.
#pragma once

#include <string>
#include <vector>

#include "abc_internal.h"

// true when the fused kernel covers the parameters; otherwise *why says why
bool fused_supported(const abc_params& p, std::string* why);
// the same for the one-pass sweep (all four stages in one launch)
bool fused4_supported(const abc_params& p, std::string* why);
// first order in the face form with a non-local operator (window > 0): the
// one-pass sweep runs without the condition plus the boundary-shell rounds
bool fused_shell_case(const abc_params& p);

// allocate/prepare whatever the fused path needs beyond the staged scratch
abc_status fused_prepare(const abc_params& p, abc_launch& L, std::vector<void*>* allocs, size_t* bytes,
                         std::string& err);

hipError_t launch_step_fused(const abc_launch& L, const abc_scratch& S, void* psi, double2* aux, const void* V,
                             int n_steps, hipStream_t st, abc_timer* tm = nullptr);

// Tile depth (planes) of the two-stage kernels for boxes launched together
// (`count` of each), at most `limit`; limits are 4, 8 or 16, the largest one
// an order allows in a box of nz planes being fused_max_limit.
struct FusedBox {
  int nx, ny, nz, count;
};
int fused_max_limit(int order, int nz);
int fused_pick_depth(int order, int limit, const std::vector<FusedBox>& boxes);
// planes per tile of the launches of a step on L's path, `orbitals` per launch
int fused_tile_depth(const abc_launch& L, int orbitals);

// Batched two-stage launch over boxes sharing (order, precision, tile depth).
// fused_batch_build writes 2 descriptor sets (one per launch of a step) into
// `host` (fused_batch_desc_bytes(nbox) bytes) and returns the total tile
// count; once they are in device memory at `dev`, launch_batch_fused runs n
// steps as 2 launches per step over the concatenated tiles of all boxes.
struct FusedMember {
  const abc_launch* L;
  const abc_scratch* S;
  void* psi;
  double2* aux;
  const void* V;
};
size_t fused_batch_desc_bytes(int nbox);
int fused_batch_build(const std::vector<FusedMember>& m, void* host);
hipError_t launch_batch_fused(const std::vector<FusedMember>& m, int tz, const void* dev, int total, int n,
                              hipStream_t st, abc_timer* tm);

// Orbital batches (and the mean field) on the fused path: the orbitals are
// transposed once per call from [point][orbital] to one array per orbital,
// stepped as boxes of a descriptor-driven launch sharing one potential (the
// mean field rebuilt from the current state before every step), and
// transposed back.  All buffers below are owned by the context.
struct OrbitalBatch {
  abc_launch L1;                   // the launch of one orbital (batch 1 geometry)
  int B = 0;                       // orbitals
  int tz = 8;
  void* soa[2] = {nullptr, nullptr};     // psi arrays [B][npts]: the state, and its other buffer
  double2* soa_f[2] = {nullptr, nullptr};  // aux arrays [B][nface], the same
  void* veff = nullptr;            // V + mean field (psi's real type), or null
  // descriptors of the two-stage launches, one set per step-count parity
  // (alike: a step ends where it began), built on first use for a given
  // potential buffer and reused after that (so a warmed-up step issues no copy
  // and can be captured in a graph)
  void* desc_host = nullptr;       // pinned staging, two sets
  void* desc_dev = nullptr;        // two sets
  const void* desc_V[2] = {nullptr, nullptr};
  bool desc_ok[2] = {false, false};
  int desc_total = 0;
  hipEvent_t copied = nullptr;
  bool pending = false;
  std::vector<abc_scratch> S;      // per-orbital scratch views into soa / soa_f
};
hipError_t launch_step_orbitals(OrbitalBatch& ob, void* psi, double2* aux, const void* V, int n_steps,
                                hipStream_t st, abc_timer* tm);
