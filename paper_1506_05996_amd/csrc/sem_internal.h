// Internal state of a sem_mesh handle, shared by the host set-up (sem_setup.cpp)
// and the device side (sem_device.hip).  Not part of the public ABI.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/sem.h"

namespace sem {

// Status carrier for internal code: never crosses the C ABI as an exception.
struct Error {
  int status;
  std::string msg;
};

void set_error(const std::string& msg);

// --- entity records ---------------------------------------------------------
// Each element has 27 node classes: class c = cx + 3 cy + 9 cz with
// cx = 0 (i = 0), 1 (0 < i < N), 2 (i = N), likewise cy, cz.  Class 13 is the
// element interior, the 8 corner classes are vertices, 12 are edges and 6 faces.
// For every class the global id of local node (i,j,k) is affine:
//     gid = gbase + ai*i + aj*j + ak*k,
// and so is its slot in the shared-node work array w (faces: 2 slots per face
// node, edges and vertices: one slot per incident element):
//     wid = wbase + ai*i + aj*j + ak*k.
// Record layout (int32 x4): gbase, packed coefficients (three signed 10-bit
// fields), wbase, flags.
constexpr int kRecInts = 4;  // kernels read a record as one int4
constexpr int kClasses = 27;
constexpr int kInteriorClass = 13;
constexpr int kFlagOwned = 1;     // this element holds the first local copy of the node
constexpr int kFlagInterior = 2;  // interior node: written straight to the global vector
constexpr int kFlagMaskedInterior = 4;  // (interior record) some interior node of the element is Dirichlet

inline int32_t pack_coef(int ai, int aj, int ak) {
  return (ai & 0x3FF) | ((aj & 0x3FF) << 10) | ((ak & 0x3FF) << 20);
}

// records of the patch tables (see build_patch_records): this bit of the packed strides marks NULL
constexpr int32_t kPatchNull = 1 << 30;
constexpr int kPatchRecordsFrom = 5;  // orders from here use the records on the device

// Coarse solve by nested dissection.  The free-vertex graph of each connected
// component is split recursively by separators (one BFS level across the
// longest extent); the separators and the final small parts are the nodes of
// a forest, of which runs of consecutive heights are then merged into single
// nodes (see merge_heights).  Nodes are numbered in post-order, and each node's
// own vertices form one contiguous range of coarse indices.  A node t holds its
// own vertices I and the boundary B: the vertices of its ancestors coupled to
// its subtree once the subtree is eliminated.  After elimination of the
// subtree, the front [F_II F_IB; F_BI F_BB] gives S = F_II and W = F_BI S^-1.
//
// Rows of the sweeps: node t owns the row slots roff .. roff + s + b - 1 (its
// own vertices, then its boundary).  The values that a row starts from sit side
// by side in the contribution vector, row slot g holding entries
// rs_off[g] .. rs_off[g + 1]: for an own row the negated coarse residual at its
// vertex, then one entry per child whose boundary holds the vertex; for a
// boundary row the children's entries alone.  A child writes entry k of its
// contribution straight to its parent's slot cdst[coff + k].  The residual
// comes in parts, one per element at the vertex: they are the first entries of
// a leaf's row, and of a higher row sit in a slot of their own (slots past the
// row slots), whose sum the lowest launch writes to the row's first entry.
struct FrontNode {
  int64_t off;     // first coarse index of the node's own vertices
  int64_t fwd;     // offset of [S^-1 ; W] in the forward pool: (s + b) rows of s, row stride lds
  int64_t bwd;     // offset of W^T in the backward pool: s rows of b, row stride ldb
  int64_t bidx;    // offset of the boundary list (ascending coarse indices) in fb_idx
  int64_t coff;    // offset of the node's contribution slots in cdst
  int64_t roff;    // first row slot
  int32_t s;       // own vertices
  int32_t b;       // boundary vertices
  int32_t lds, ldb;  // row strides: s and b rounded up to even, so that rows are 16-byte aligned
  int32_t parent;  // -1 for a root
  int32_t height;  // 0 for a leaf, else 1 + the largest height of its children
};

inline int32_t even_up(int32_t v) { return (v + 1) & ~1; }

// one workgroup of a coarse sweep: rows row .. row + 4 RW - 1 of one node
struct CoarseTile {
  int64_t mat;   // the node's matrix in the forward or backward pool
  int32_t ld;    // row stride
  int32_t len;   // row length: s forward, b backward
  int32_t row;   // first row
  int32_t rows;  // rows of the node: s + b forward, s backward
  int32_t s;     // own vertices
  int32_t off;   // first coarse index
  int32_t src;   // forward: first row slot; backward: offset of the boundary list
  int32_t coff;  // forward: offset of the contribution slots
  int32_t root;  // no boundary: the forward rows are the solution
  int32_t pad;
};

// Rows per wave of a sweep launch over `rows` rows of at most `len` entries.
// Every workgroup stages its node's vector for its own rows, so more rows per
// wave save staging, as long as enough waves are left to keep the chip's loads
// in flight: at least 1,024 forward, where an entry of the vector is a sum of
// several loads, and 2,048 backward, where it is one (24^3: 42.8 us with 1,024
// and 2,048, 48 us with 4,096 for both; 56^3 488 against 498 us).  Rows of up to
// 128 entries are one 16-byte load per lane, so eight of them fit the registers
// that four longer rows take.
inline int32_t coarse_rows_per_wave(int64_t rows, int64_t len, bool forward) {
  const int64_t waves = forward ? 1024 : 2048;
  const int32_t most = len <= 128 ? 8 : 4;
  int32_t rw = 1;
  while (rw < most && rows >= waves * rw * 2) rw *= 2;
  return rw;
}

// one launch of a sweep: tiles [first, first + count) with rw rows per wave
struct CoarseLaunch {
  int64_t first, count;
  int32_t rw;
  int32_t wide;  // rows beyond 128 entries
};

struct HostTables {
  int N = 0, n1 = 0, np = 0;  // order, N+1, N+3
  int64_t E = 0, n_global = 0, n_local = 0;
  int64_t V = 0, n_edges = 0, n_faces = 0;
  int64_t base_e = 0, base_f = 0, base_i = 0;  // first global id of edges, faces, interiors

  // reference data
  std::vector<double> t, rho, D;  // D[i*(N+1)+j] = phi_j'(t_i)
  std::vector<double> S, lam;     // fast-diagonalisation basis by parity (packed, [(N+3)/2 rows][N+3] + middle row), eigenvalues [N+3]

  // numbering and gather
  std::vector<int32_t> rec;              // [E][27][4]
  std::vector<uint8_t> dir;              // [n_global] 1 = Dirichlet
  std::vector<int32_t> vinc_off;         // [V+1]   vertex incidences (slot = index)
  std::vector<int32_t> einc_off;         // [n_edges+1]
  std::vector<uint8_t> fcount;           // [n_faces] 1 or 2 hexahedra
  int64_t wedge_off = 0, wvert_off = 0, w_size = 0;
  std::vector<int32_t> owner;            // [n_global] local index of the first copy

  // faces and patches
  std::vector<int32_t> face_nbr;         // [E][6][2] (element, local face) or -1
  std::vector<int32_t> ip;               // [E][(N+3)^3] global id or -1
  // the nx = (N+3)^3 - (N+1)^3 patch slots outside the element: their ordinal
  // (xord[slot] >= 0, grouped by face plane, edge line and corner; inside:
  // -(local index) - 1; the device derives the slot of an ordinal in closed
  // form) and, per patch, where each
  // lands in the consumer layout [E][nx] of the element that holds it:
  // 6 face planes [(N+1)^2] at one layer in from that face (in-plane index
  // x_lo + (N+1) x_hi over the other two axes in increasing order), 12 edge
  // lines [N+1] at one layer in from both faces of the edge (edge id
  // 4 axis + side_lo + 2 side_hi, position along the axis), 8 corner points
  // (id = side_x + 2 side_y + 4 side_z); -1 where the slot is NULL
  int64_t nx = 0;
  std::vector<int32_t> xord;             // [(N+3)^3]
  std::vector<int32_t> xdest;            // [E][nx]

  // geometry
  std::vector<double> G;     // [E][6][(N+1)^3]
  std::vector<double> X8;    // [E][8][3] vertex coordinates in tensor corner order
  std::vector<double> mass;  // [E][(N+1)^3]
  std::vector<double> mN;    // [n_global]
  std::vector<double> xN;    // [n_global][3]
  std::vector<double> h;     // [E][3]
  std::vector<int32_t> order;  // element traversal order: Morton order of the centroids

  // coarse space (order-1 operator on the free vertices, nested-dissection order)
  std::vector<int32_t> cidx;             // [V] coarse index or -1 (Dirichlet vertex)
  int64_t nc = 0;                        // number of free vertices
  std::vector<int32_t> ac_off, ac_col;   // CSR of A_c in coarse order
  std::vector<double> ac_val;
  std::vector<FrontNode> fnodes;         // post-order
  std::vector<std::vector<int32_t>> fchildren;  // children of each node, ascending
  std::vector<int32_t> fb_idx;           // boundary lists
  std::vector<int32_t> cvert;            // [nc] vertex of each coarse index
  std::vector<int32_t> pslot;            // [nc] slot of the element parts of each coarse index
  std::vector<int32_t> rs_off;           // [slots + 1]: entries of each slot
  std::vector<int32_t> pre_slot, pre_row;  // part slots of the higher rows, and those rows
  std::vector<int32_t> part_dst;         // [E][8]: entry of an element's part of the residual, -1 at Dirichlet vertices
  std::vector<int32_t> cdst;             // [sum of b]: entry each contribution goes to
  int64_t fwd_size = 0, bwd_size = 0;    // entries of the pools, padding included
  int64_t fwd_entries = 0, bwd_entries = 0;  // without padding
  int64_t c_size = 0;                    // entries of the contribution vector
  int64_t ustack_size = 0;               // largest sum of pending update matrices (set-up)
  int32_t max_front = 0;                 // largest s + b
  std::vector<CoarseTile> tiles;         // of all launches
  std::vector<CoarseLaunch> fwd_launch, bwd_launch;  // in the order they run
  std::vector<double> corner_K;          // [E][8][8] order-1 element stiffness matrices
  std::vector<double> corner_M;          // [E][8] order-1 element mass (|J| at the corners, diagonal)
  std::vector<int64_t> coarse_vid;       // [E][8] global id of each element's corner vertices

  // coefficients of the model problem c u - div(kappa grad u) = s: constants,
  // or one value per element (kap_e, c_e non-empty; kappa, cmass are then NaN)
  double kappa = 1.0, cmass = 0.0;
  std::vector<double> kap_e, c_e;
};

// aggregation AMG hierarchy of the coarse system (sem_amg.cpp); level 0 holds
// the free vertices in ascending vertex id
struct AmgLevel {
  int64_t n = 0;
  std::vector<int32_t> off, col;  // CSR, columns ascending
  std::vector<double> val, diag;
  std::vector<int32_t> agg;       // [n] aggregate (row of the next level); empty on the coarsest
  std::vector<int32_t> moff, mem; // members of each aggregate, ascending
};

struct AmgHierarchy {
  std::vector<AmgLevel> levels;
  std::vector<double> coarse_inv;  // dense inverse of the coarsest matrix, row-major
  std::vector<int32_t> nd_of;      // level-0 unknown -> coarse (nested-dissection) index
};

void build_amg(const HostTables& T, AmgHierarchy& H);

// host set-up entry points (sem_setup.cpp)
void build_reference(HostTables& T, int N);
void build_numbering(HostTables& T, const int64_t* hex, int64_t n_hex, int64_t n_vtx);
void build_geometry(HostTables& T, const double* vtx, const int64_t* hex);
void build_patches(HostTables& T, const int64_t* hex);
void build_patch_records(const HostTables& T, std::vector<int32_t>& pidx, std::vector<int32_t>& pdst);
void build_coarse_matrices(HostTables& T, const double* vtx, const int64_t* hex);
void build_coarse_tree(HostTables& T, int leaf_max = 0);
void assemble_coarse_matrix(HostTables& T);
void boundary_face_mass(const HostTables& T, const int64_t* faces, int64_t n_faces, double* ws);
void export_l2g(const HostTables& T, int32_t* l2g);
void update_interior_mask_flags(HostTables& T);
int64_t gid_of(const HostTables& T, int64_t e, int i, int j, int k);

}  // namespace sem
