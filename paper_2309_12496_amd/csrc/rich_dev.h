// Device-side data layout of librich (shared by the host scene builder and the kernels).
//
// HBM layout of a scene:
//   nodes  : Node4[]  128 B each, all BVH4s (top level first, then one BVH per
//            instance), depth-first so that a parent and its children are near.
//   lane_nodes : LaneNode[]  64 B each, the same nodes for a lane's own walk.
//   tris   : Tri[]    64 B each, grouped by leaf, vertices in the local frame of
//            their instance, unit normals computed in FP64 on the host.
//   inst   : Instance[] world<->local transforms of mesh instances.
//   caps, rects, mats, detector tables: a few KB, read through the scalar cache.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rich {

constexpr uint32_t kStreamTag = 0x52494348u;   // fourth Philox counter word ("RICH")
constexpr int kStackDepth = 32;                // traversal stack entries
// A wave's stacks in LDS are rows of 64 words, lane l's entry d being word
// 64 d + l (the lanes of a row sit in distinct banks at any mix of depths, and
// consecutive entries are a fixed 256 B apart).  With the wave phase there are
// kLdsRows rows and the kStackDepth references the wave still has to walk
// together; a lane's entries beyond the rows, which few rays ever need, go to
// private memory (5 KB of LDS per wave instead of 9 lets a fifth wave per SIMD
// run).  A lane then has kPending entries more than kStackDepth: as many as
// the wave phase may leave on its stack before it walks on its own.
constexpr int kStackRow = 64;
constexpr int kPending = 4;
constexpr int kLaneRows = kStackDepth + kPending;
constexpr int kLdsRows = 20;
// The wave phase parts at a node with two children met when fewer than one in
// kWaveShare of the wave's rays meet them.
constexpr int kWaveShare = 4;
constexpr int kMaxTable = 32;
constexpr int kFates = 7;                      // photon fates, RICH_N_FATES

// BVH4 child reference encoding.
constexpr uint32_t kEmpty = 0xFFFFFFFFu;       // no child
constexpr uint32_t kLeafBit = 0x80000000u;     // leaf or instance
constexpr uint32_t kInstBit = 0x40000000u;     // with kLeafBit: instance reference
constexpr uint32_t kExitMarker = 0xFFFFFFFEu;  // stack entry: return to the world frame
constexpr uint32_t kLeafMaxTris = 8;
// Scene size limits: traversal addresses triangles (64 B) and nodes (128 B)
// with 32-bit byte offsets from the array bases.
constexpr int64_t kMaxTriangles = int64_t(1) << 26;   // exclusive
constexpr int64_t kMaxNodes = int64_t(1) << 25;       // exclusive
// leaf: kLeafBit | (count-1) << 27 | first   (first < 2^27, count 1..8)
// instance: kLeafBit | kInstBit | index
__host__ __device__ inline uint32_t make_leaf(uint32_t first, uint32_t count) {
    return kLeafBit | ((count - 1u) << 27) | first;
}
__host__ __device__ inline uint32_t make_inst(uint32_t idx) { return kLeafBit | kInstBit | idx; }

struct alignas(128) Node4 {
    float lox[4], hix[4], loy[4], hiy[4], loz[4], hiz[4];
    uint32_t child[4];
    uint32_t leaves;     // bit c: child c is a leaf (triangles)
    uint32_t order;      // 3 bits for each pair of children (01 02 03 12 13 23): the axis along
                         // which they lie furthest apart, and 4 if the second is on its positive side
    uint32_t pad[2];
};
static_assert(sizeof(Node4) == 128, "Node4 must be 128 bytes");

// The same node for a lane's own walk: its children's boxes on a grid of 256
// steps a side over their union, rounded outwards (plane q of axis a lies at
// org[a] + q step[a]).  A lane fetches four 16-byte words instead of Node4's
// seven: the vector cache's return path was 83 % busy and the vector units 47,
// now 77 and 68 (1e6 unsorted photons on 210,082 triangles 280 -> 249 us; 4,096
// tracks there 737 -> 700, and on 2,009,708 triangles 2,290 -> 2,080).  An
// empty slot is an inverted box with the first child's reference.
struct alignas(64) LaneNode {
    float org[3], step[3];
    uint32_t lox, hix, loy, hiy, loz, hiz;   // byte c: child c
    uint32_t child[4];
};
static_assert(sizeof(LaneNode) == 64, "LaneNode must be 64 bytes");

// Triangle record: v0.xyz + global triangle index, v1.xyz + material, v2.xyz, normal.xyz + sheet.
struct alignas(16) Tri {
    float v0[3];
    uint32_t index;
    float v1[3];
    uint32_t material;
    float v2[3];
    uint32_t pad0;
    float n[3];
    uint32_t sheet;      // 1 + index into DevScene::sheets, 0: none
};
static_assert(sizeof(Tri) == 64, "Tri must be 64 bytes");

// A mirror surface that a photon it has just reflected cannot meet again: its
// triangles are the facets of one concave sphere or one plane (the proof the
// builder checks is at sheet_rule).  Its subtree's nodes are contiguous, and
// the query after such a reflection leaves them out: without that it walks
// down to the facet it starts on, whose boxes all hold its origin (1e7 photons
// on 210,082 triangles: 16.4 nodes and 5.6 triangle tests per photon instead
// of 23.9 and 7.4, 1.57 -> 1.27 ms).
struct alignas(16) Sheet {
    uint32_t node_lo, node_n;   // nodes of its subtree
    float min_cos;              // holds for directions with d . (hit facet's normal) >= min_cos
    float rule;                 // min_cos where the rule is proved (see kSheetSlack)
};
// A moving segment's sheet is left out while the segment is scaled by no more
// than this and its box reaches no further than this times the scene's extent.
// Beyond, min_cos is 2.
constexpr float kSheetSlack = 1.1f;

// Mesh instance: local = m * (world - org); world normal = rot * local normal.
struct alignas(16) Instance {
    float m[9];
    float org[3];
    float rot[9];
    float scale;
    uint32_t root;       // root node of this instance's BVH
    int32_t segment;     // -1: fixed
    float lo[3], hi[3];  // world AABB at the current parameters
    float loc_lo[3], loc_hi[3];  // local AABB
    float drx[9];        // d rot / d tilt_x (for the adjoint)
    float dry[9];        // d rot / d tilt_y
    float inv_r0;        // 1 / nominal radius of the segment (0 for fixed meshes)
    float pad;
};

// Analytic spherical cap at the current parameters.
struct alignas(16) CapDev {
    float C[3];
    float R;
    float axis[3];       // unit pivot -> centre
    int32_t segment;
    float O[3];
    int32_t material;
    float A[3];
    float a_lo;
    float B[3];
    float a_hi;
    float lo[3];         // world AABB of the cap
    float b_lo;
    float hi[3];
    float b_hi;
    float dCdtx[3];      // derivatives of C for the adjoint
    float pad0;
    float dCdty[3];
    float pad1;
};

struct alignas(16) RectDev {
    float c[3];
    int32_t material;
    float n[3];
    float hu;
    float u[3];
    float hv;
    float v[3];
    float pad;
};

// Piecewise-linear table: nodes x, values y, slope s[j] = (y[j+1]-y[j])/(x[j+1]-x[j]) (FP64 on the host).
struct MatDev {
    int32_t kind;
    int32_t n;
    float x[kMaxTable];
    float y[kMaxTable];
    float s[kMaxTable];
};

struct DetDev {
    float c[3], n[3], u[3], v[3];
    float hu, hv;            // geometric half sizes
    float pitch;
    float act_hu, act_hv;    // half sizes of the pixel grid
    int32_t nx, ny;
    int32_t n_qe;
    float inv_pitch;
    float qe_x[kMaxTable];
    float qe_y[kMaxTable];
    float qe_s[kMaxTable];
};

// FP64 master data used by the parameter update kernel.
struct SegDev {
    double pivot[3], u0[3], e1[3], e2[3];
    double r0;
};

struct CapStatic {
    int32_t segment, material;
    double O[3], A[3], B[3];
    double bounds[4];
};

// Everything a propagation kernel reads, passed by value.
struct DevScene {
    const CapDev *caps;
    const RectDev *rects;
    const MatDev *mats;
    const Node4 *nodes;
    const LaneNode *lane_nodes;
    const Tri *tris;
    const Instance *inst;
    const Sheet *sheets;
    const DetDev *det;
    unsigned int *status;
    int32_t n_caps, n_rects, n_mats, n_inst;
    int32_t has_mesh, has_box;
    uint32_t top_root;
    int32_t max_bounces;
    float t_min;
    uint32_t prim_det, prim_box, prim_tri;   // global primitive numbering
    float box_lo[3], box_hi[3];
    int32_t n_seg;
    float sheet_reach;   // longest flight to a sheet for which its rule holds (mm)
};

// Photon source as seen by the kernels.
struct DevSource {
    int32_t kind;        // 0 track, 1 batch, 2 explicit
    // track: emission origin, direction frame, cone, spectrum (precomputed on the host in FP64)
    float P0[3], T[3], E1[3], E2[3];
    float length, cos_t, sin_t;
    float inv_lmin, inv_span;   // 1/lambda_min and 1/lambda_min - 1/lambda_max
    // batch
    const float *tracks;        // rich_track[] as 8 floats
    const uint64_t *offsets;
    int32_t n_tracks;
    // batch processing order (null: id order): the tracks in the order their
    // photons are processed, and the exclusive scan of their counts in that
    // order ([n_tracks + 1]); photon ids, hence results, do not change
    const int32_t *order;
    const uint64_t *order_off;
    double n_radiator;
    // explicit
    const float *ex_o, *ex_d, *ex_l;
    // pre-propagation efficiency filter (0 materials and prefilter = 0: off)
    int32_t prefilter;
    int32_t pf_n;
    int32_t pf_mats[4];
    // radiator dispersion (n_disp = 0: constant index): nodes, n - 1 and the
    // segment slopes dn/dlambda; the largest index over the band (FP64 host)
    int32_t n_disp;
    float disp_x[kMaxTable], disp_m[kMaxTable], disp_s[kMaxTable];
    double disp_nmax;
    float ng_const;     // group index without a table
    float beta;         // track: particle velocity / c
};

constexpr uint32_t kDispBlock = 0x7FFFFFFEu;   // wavelength retries use blocks kDispBlock - k
constexpr int kDispMaxTries = 64;
constexpr float kInvC = 1.0f / 299.792458f;    // ns per mm in vacuum

constexpr uint32_t kPrefilterBlock = 0x7FFFFFFFu;   // Philox block of the pre-filter draw

struct DevOutputs {
    uint8_t *fate;
    int32_t *pixel;
    float *hit_xyz;
    float *hit_uv;
    uint32_t *histogram;
    unsigned long long *fate_counts;
    void *hit_list;             // rich_hit[]
    unsigned long long *hit_count;
    uint64_t hit_capacity;
    float *hit_time;
};

}  // namespace rich
