// The sparse LU in nested-dissection order (rr_nd.hip): plan and launches.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace rr {

struct OpDesc;

// One front of the elimination tree: a separator line of grid nodes (or a
// leaf block of them), whose p unknowns are eliminated, and the q unknowns of
// the separators around its block.  P and Q are p and q rounded up to 16 (the
// MFMA block edge); padding carries the identity in A and zeros elsewhere.
// Rows number the unknowns, separators first: the solves' workspaces hold
// only those.
struct NdFront {
  int p, q, P, Q;
  int row;             // its unknowns' first row
  int bor;             // its border's first entry in the border tables
  int childA, childB;  // fronts of the two halves, -1 for a leaf
  int baseA, baseB;    // the separator's first position in the halves' borders
  int urow;            // first row of its update in the level's update arena
  int side[5];         // border offsets: left, right, low, high, end
  int across;          // a leaf's nodes along y
  int64_t a, b12, f21;  // offsets in one shift's factors (a leaf keeps A alone)
  int64_t s;           // offset of its Schur complement in the level's arena
  int64_t t;           // offset of its temporaries (P > kNdTile only)
  // the halves' Q, s and urow, so that a kernel reads one front
  int QA, QB, uA, uB;
  int64_t sA, sB;
};
constexpr int kNdTile = 64;       // product tile edge, and the widest one-launch inverse
// Fronts up to this P take their sweep down in one workgroup; wider ones 16
// rows a workgroup, whose waves then share the border instead of one wave
// walking all of it (P = 64, Q = 376: 48 / 79 us forward / adjoint a level for
// one shift against 20 / 28; level by level about equal for 16).
constexpr int kNdDownP = 32;
// From kNdLeafApart narrow leaves (all shifts') on, the factor launches leaves up
// to kNdLeafP apart from the wider ones, whose FP64 tile takes 75 KB of LDS:
// three workgroups a CU then, not two.  At 512 x 256 4001 of 4096 leaves have 48
// rows; 16 shifts, the factor 31.9 -> 30.8 ms FP64, 21.6 -> 20.4 FP32; with 977
// (256 x 128, one shift) the second launch costs 20 us more than it gives.
constexpr int kNdLeafP = 48, kNdLeafApart = 3072;
constexpr int kNdLeafNodes = 32;  // blocks of at most this many nodes are leaves

struct NdTask { int front, i, j, kind; };
struct NdSpan { int first = 0, count = 0; };  // a range of the task list

struct NdLevel {  // fronts at one depth of the tree
  NdSpan leaf;       // one task a leaf, those of P <= kNdLeafP first:
  NdSpan leafs[2];   // the two widths apart, for the factor
  NdSpan small;      // one task a front with halves, P <= kNdTile
  NdSpan assemble;   // P > kNdTile: tiles of A, T12 and F21
  std::vector<NdSpan> panel, update;  // per pivot tile
  NdSpan border;     // tiles of B12
  NdSpan schur;      // tiles of S, every front with halves
  NdSpan gather, rowsP, rowsQ;  // solves, P > kNdTile: 64 rows; 16 rows of P; of Q
  NdSpan down;       // solves, down: one task a front with halves, P <= kNdDownP
  NdSpan rowsX;      // ... and 16 rows of the wider ones
  int maxP = 0, maxQ = 0;  // over the small fronts
  int downP = 0;           // largest P of the fronts in `down`
  int largeP = 0;          // largest P of the fronts past kNdTile
  int leafP = 0;           // largest P of the leaves
  int front = 0;           // the level's first front
};

struct NdPlan {
  int nx = 0, ny = 0;
  std::vector<NdFront> fronts;  // by depth, the root first
  std::vector<NdLevel> levels;  // [depth]
  std::vector<NdTask> tasks;
  std::vector<int> pdof;   // row -> unknown, -1: padding
  // border entry -> 2 * (position in a half's border) + half, -1: none; a
  // leaf's: the position of its one neighbour among the leaf's unknowns
  std::vector<int> bmap;
  std::vector<int> grow;   // border entry -> row (padding: the zero row)
  int64_t nfronts = 0;
  int64_t rows = 0;        // rows of the separators; row `rows` of the workspaces is zero
  int64_t allrows = 0;     // with the leaves'
  int64_t border = 0;
  int64_t factor = 0;      // complex elements of one shift: factors,
  int64_t schur[2] = {};   // Schur arenas of even and odd depths,
  int64_t temp = 0;        // temporaries of the largest level
  int64_t urows[2] = {};   // rows of the update arenas
  int64_t ntasks = 0;
};
// the counts and sizes alone (nfronts and below), from the distinct blocks
void nd_sizes(int nx, int ny, NdPlan* plan);
// the whole plan
void nd_make_plan(int nx, int ny, NdPlan* plan);

struct NdDevice {  // device pointers of a handle
  NdFront* fronts = nullptr;
  NdTask* tasks = nullptr;
  int *pdof = nullptr, *bmap = nullptr, *grow = nullptr;
  void* factor = nullptr;
  void* schur[2] = {};
  void* temp = nullptr;
  void *w = nullptr, *z = nullptr;  // n_omega * (rows + 1) * k: separators' right-hand
                                    // sides, then solutions; A b1 or b1
  void* u[2] = {};                  // n_omega * urows * k: updates
};

hipError_t nd_prepare();
hipError_t launch_nd_factor(const OpDesc& op, const NdPlan& pl, const NdDevice& d,
                            const double* omega, int n_omega, bool fp32, uint32_t* status,
                            hipStream_t s);
// X = M^-1 Bm (M^-H Bm) for columns [c0, c0 + k) of blocks with ktot columns
// per shift, k <= 32; Bm's blocks are bstride complex elements apart (0:
// shared) and may be X's.  io32 (FP32 factors only): Bm and X are FP32.
hipError_t launch_nd_solve(const OpDesc& op, const NdPlan& pl, const NdDevice& d, int64_t n,
                           int n_omega, int k, int c0, int ktot, bool fp32, bool io32, int adjoint,
                           const void* Bm, int64_t bstride, void* X, hipStream_t s,
                           const uint32_t* skip = nullptr);

}  // namespace rr
