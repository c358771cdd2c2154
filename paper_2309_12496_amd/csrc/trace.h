// Device functions of the photon path: random stream, generation, closest hit,
// interaction.  Shared by the forward, batch and adjoint kernels.
//
// Precision: FP32 throughout, except the Cherenkov cone constants of batch
// tracks (1/(n beta) and its sine, FP64 to avoid cancellation in 1 - cos^2)
// and the rare watertight-test fallback on exactly-zero edge functions.
#pragma once

#include "rich_dev.h"

namespace rich {

// ---------------------------------------------------------------- vectors

struct V3 {
    float x, y, z;
};
__device__ __forceinline__ V3 v3(float x, float y, float z) { return V3{x, y, z}; }
__device__ __forceinline__ V3 ld3(const float *p) { return V3{p[0], p[1], p[2]}; }
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return V3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return V3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(float s, V3 a) { return V3{s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ float dot(V3 a, V3 b) { return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z)); }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
    return V3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ __forceinline__ V3 fma3(float s, V3 a, V3 b) {  // s*a + b
    return V3{fmaf(s, a.x, b.x), fmaf(s, a.y, b.y), fmaf(s, a.z, b.z)};
}
__device__ __forceinline__ V3 mat3(const float *m, V3 v) {  // row-major 3x3 times v
    return V3{fmaf(m[0], v.x, fmaf(m[1], v.y, m[2] * v.z)), fmaf(m[3], v.x, fmaf(m[4], v.y, m[5] * v.z)),
              fmaf(m[6], v.x, fmaf(m[7], v.y, m[8] * v.z))};
}
__device__ __forceinline__ float comp(V3 a, int k) { return k == 0 ? a.x : (k == 1 ? a.y : a.z); }

// Scene data (caps, rects, detector, materials and their tables) is never
// written while a propagation kernel runs: the prepare kernel updates it in an
// earlier launch.  Reading it through the constant address space tells the
// compiler so, and reads at wave-uniform addresses (the loops over analytic
// primitives and table nodes) become one scalar load per wave instead of one
// vector load per lane.  Without it, any output store earlier in the kernel
// keeps the compiler from proving the data unchanged.
#define RICH_CONST __attribute__((address_space(4)))

// The kernels' scene and source are their first two arguments, read from the
// argument segment where they are used.  Held in scalar registers from the
// start, as the compiler prefers, they and the detector's fields overflowed
// the 102 there are: 324 were kept in lanes of vector registers and read back
// one by one inside the bounce loop.  fresh() hides where a pointer comes from,
// so that what is read through it is read after this point.
using SceneRef = const RICH_CONST DevScene &;
using SourceRef = const RICH_CONST DevSource &;
template <class T>
__device__ __forceinline__ const RICH_CONST T *fresh(const RICH_CONST T *p) {
    asm volatile("" : "+s"(p));
    return p;
}
template <class T>
__device__ __forceinline__ const RICH_CONST T &fresh(const RICH_CONST T &x) {
    return *fresh(&x);
}
// Kernel argument of type T at byte offset `at` of the argument segment.
template <class T>
__device__ __forceinline__ const RICH_CONST T &kernel_arg(size_t at) {
    return *(const RICH_CONST T *)((const RICH_CONST char *)__builtin_amdgcn_kernarg_segment_ptr() + at);
}
constexpr size_t arg_after(size_t end, size_t align) { return (end + align - 1) / align * align; }
constexpr size_t kSourceArg = arg_after(sizeof(DevScene), alignof(DevSource));
constexpr size_t kThirdArg = kSourceArg + sizeof(DevSource);   // what follows them (8-byte aligned)
static_assert(kThirdArg % 8 == 0, "argument layout");
__device__ __forceinline__ SceneRef scene_arg() { return kernel_arg<DevScene>(0); }
__device__ __forceinline__ SourceRef source_arg() { return kernel_arg<DevSource>(kSourceArg); }

// Work counters of the measurement build (compiled with -DRICH_WORK_COUNTERS;
// the product library has none of this).  Each counts one unit of work per
// active lane: a traced photon, a Philox block (of which the regrouping's
// second draw of block 0 for its sort key is also counted apart), a
// closest-hit query (ray set-up and the detector plane), a cap's bounding-box
// test and its sphere test, a rectangle, the analytic box, a BVH4 node whose
// four child boxes are tested, a leaf, a triangle test, an entry into a mesh
// instance's frame (and apart those that rotate and scale the ray), a
// reflection, a detector hit; in the adjoint, a counted photon's pass back
// through the detector plane and each reflection it sweeps back through (cap
// or facet).  Lanes of a wave are summed with one atomic per counter and wave;
// a second word in the counter's line counts the waves that did the unit, so
// lanes / (64 x waves) is the unit's SIMD efficiency.
enum WorkUnit {
    kWorkPhotons, kWorkPhilox, kWorkSortKeys, kWorkQueries, kWorkCapBoxes, kWorkCaps, kWorkRects, kWorkBoxes,
    kWorkNodes, kWorkLeaves, kWorkTris, kWorkInstances, kWorkMovingInstances, kWorkReflections, kWorkDetections,
    kWorkBackDetector, kWorkBackCaps, kWorkBackFacets, kWorkBackPlanes,
    kWorkWaveNodes, kWorkWaveLeaves, kWorkWaveTris, kWorkUnits
};
#ifdef RICH_WORK_COUNTERS
static __device__ unsigned long long rich_work[16 * kWorkUnits];   // one 128-byte line per counter
__device__ __forceinline__ void work(int unit) {
    const unsigned long long m = __ballot(1);
    if (__lane_id() == __ffsll((long long)m) - 1) {
        atomicAdd(&rich_work[16 * unit], (unsigned long long)__popcll(m));
        atomicAdd(&rich_work[16 * unit + 1], 1ull);
    }
}
#else
__device__ __forceinline__ void work(int) {}
#endif
template <class T>
__device__ __forceinline__ const RICH_CONST T &cref(const T &x) {
    return *(const RICH_CONST T *)&x;
}
typedef float Float4 __attribute__((ext_vector_type(4)));
typedef uint32_t Uint8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ V3 ld3(const RICH_CONST float *p) { return V3{p[0], p[1], p[2]}; }

// ---------------------------------------------------------------- Philox4x32-10

// Counter-based generator of Salmon et al. (SC'11): ten rounds of two 32x32->64
// multiplies whose halves are cross-mixed with the other words and the key;
// the key advances by the Weyl constants (golden ratio, sqrt 3) each round.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t p0 = (uint64_t)0xD2511F53u * c.x;   // one 32x32->64 multiply gives both halves
        uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ __forceinline__ uint4 photon_block(uint64_t seed, uint64_t g, uint32_t blk) {
    work(kWorkPhilox);
    return philox4x32_10(make_uint4((uint32_t)g, (uint32_t)(g >> 32), blk, kStreamTag), (uint32_t)seed,
                         (uint32_t)(seed >> 32));
}

// top 24 bits as a float in [0,1): exact
__device__ __forceinline__ float u24(uint32_t x) { return (float)(x >> 8) * 5.9604644775390625e-8f; }

// Hardware reciprocal (1 ulp).  Used on the geometric path where a few ulps
// are far below the tolerance; the IEEE division sequence costs ~10 instructions.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// ---------------------------------------------------------------- tables

// Piecewise-linear table with per-segment slopes, clamped outside its range.
// The loop bound and the node addresses are uniform, so the nodes arrive
// through scalar loads and each lane only selects.
template <class P>   // const float * or const RICH_CONST float *
__device__ __forceinline__ float lerp_table(int n, P x, P y, P sl, float l) {
    float v = l <= x[0] ? y[0] : y[n - 1];
    for (int j = 0; j + 1 < n; ++j) {
        float xa = x[j];
        if (l >= xa && l < x[j + 1]) v = fmaf(sl[j], l - xa, y[j]);
    }
    return v;
}

// ---------------------------------------------------------------- generation

struct Photon {
    V3 o, d;
    float lambda;
    float u_qe;
    float t0;       // emission time after the track start (ns)
    float ng_c;     // group index / c (ns per mm)
};

// n(lambda) - 1 and the table slope dn/dlambda at l (slope 0 outside the
// table).  The interval's index is the count of the nodes up to l, two vector
// operations a node (a value taken or not at every interval took seven), and
// its three numbers are then read by each lane from the argument segment
// (2e7 photons, 17 nodes, with the acceptance's divisions gone: 908 -> 801 us).
__device__ __forceinline__ float disp_lookup(SourceRef src, float l, float &slope) {
    const int n = src.n_disp;
    int j = -1;
    for (int k = 0; k < n; ++k) j += l >= src.disp_x[k] ? 1 : 0;
    const bool in = j >= 0 && j < n - 1;
    if (!in) j = l <= src.disp_x[0] ? 0 : n - 1;
    const float m = src.disp_m[j], s = src.disp_s[j], xa = src.disp_x[j];
    slope = in ? s : 0.0f;
    return in ? fmaf(s, l - xa, m) : m;
}

__device__ __forceinline__ int find_track(const uint64_t *off, int n_tracks, uint64_t g) {
    int lo = 0, hi = n_tracks;  // last k with off[k] <= g
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= g) lo = mid; else hi = mid;
    }
    return lo;
}

// Track of photon g when the wave's photons mostly share one: a scalar
// binary search (constant address space, wave-uniform index) for the wave's
// first active photon; lanes outside that track's id range try the next two
// tracks (a wave of consecutive ids that crosses a boundary) and search on
// their own only beyond them.
__device__ __forceinline__ int find_track_wave(const uint64_t *off, int n_tracks, uint64_t g) {
    const RICH_CONST uint64_t *oc = (const RICH_CONST uint64_t *)off;
    const uint64_t g0 = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(g >> 32)) << 32) |
                        __builtin_amdgcn_readfirstlane((uint32_t)g);
    int lo = 0, hi = n_tracks;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (oc[mid] <= g0) lo = mid; else hi = mid;
    }
    if (g >= oc[lo] && g < oc[lo + 1]) return lo;
    if (g >= oc[lo + 1]) {
        for (int k = lo + 1; k < lo + 3 && k < n_tracks; ++k)
            if (g < off[k + 1]) return k;
    }
    return find_track(off, n_tracks, g);
}

// Orthonormal basis (b1, b2) around unit n, after Duff et al., JCGT 2017.
__device__ __forceinline__ void basis(V3 n, V3 &b1, V3 &b2) {
    float sgn = copysignf(1.0f, n.z);
    float a = -1.0f / (sgn + n.z);
    float b = n.x * n.y * a;
    b1 = V3{1.0f + sgn * n.x * n.x * a, sgn * b, -sgn * n.x};
    b2 = V3{b, sgn + n.y * n.y * a, -n.y};
}

// wave_track: the wave's photons come from consecutive ids (forward and batch
// kernels), so most lanes share the first lane's track; the adjoint's queued
// photons do not, and search per lane.  track >= 0: the caller knows the
// photon's track (batch processing order) and no search is made.
__device__ __forceinline__ Photon make_photon(SourceRef src, uint64_t seed, uint64_t g, uint64_t i,
                                              bool wave_track = true, int track = -1) {
    uint4 w = photon_block(seed, g, 0);
    Photon ph;
    ph.u_qe = u24(w.w);
    if (src.kind == 2) {
        ph.o = ld3(src.ex_o + 3 * i);
        ph.d = ld3(src.ex_d + 3 * i);
        ph.lambda = src.ex_l[i];
        ph.t0 = 0.0f;
        float slope = 0.0f, m = src.n_disp > 0 ? disp_lookup(src, ph.lambda, slope) : 0.0f;
        ph.ng_c = (src.n_disp > 0 ? 1.0f + fmaf(-ph.lambda, slope, m) : src.ng_const) * kInvC;
        return ph;
    }
    V3 P0, T, E1, E2;
    float L, ct, st, beta;
    if (src.kind == 1) {
        int k = track >= 0 ? track
                           : (wave_track ? find_track_wave(src.offsets, src.n_tracks, g)
                                         : find_track(src.offsets, src.n_tracks, g));
        const float4 *tr = reinterpret_cast<const float4 *>(src.tracks) + 2 * k;
        float4 a = tr[0], b = tr[1];
        P0 = V3{a.x, a.y, a.z};
        T = V3{a.w, b.x, b.y};
        T = rsqrtf(dot(T, T)) * T;
        L = b.z;
        beta = b.w;
        double c = 1.0 / (src.n_radiator * (double)b.w);
        ct = (float)c;
        st = (float)sqrt((1.0 - c) * (1.0 + c));
        basis(T, E1, E2);
    } else {
        P0 = ld3(src.P0);
        T = ld3(src.T);
        E1 = ld3(src.E1);
        E2 = ld3(src.E2);
        L = src.length;
        ct = src.cos_t;
        st = src.sin_t;
        beta = src.beta;
    }
    ph.lambda = rcp(fmaf(-u24(w.y), src.inv_span, src.inv_lmin));
    ph.ng_c = src.ng_const * kInvC;
    if (src.n_disp > 0) {
        // Frank-Tamm spectrum with dispersion: accept the 1/lambda^2 draw with
        // probability w(lambda)/w_max, else draw again from the next block.
        // w = 1 - 1/x with x = (beta n)^2 (zero below threshold), so u < w/w_max
        // is u (x_max - 1) x < (x - 1) x_max: no division.  FP64: n - 1 is
        // small, so the cone and the acceptance need more than FP32 carries in n.
        const double b2 = (double)beta;
        const double xmax = b2 * b2 * src.disp_nmax * src.disp_nmax;
        float slope = 0.0f, m = 0.0f;
        for (int k = 0; k < kDispMaxTries; ++k) {
            uint4 r = photon_block(seed, g, kDispBlock - (uint32_t)k);
            if (k > 0) ph.lambda = rcp(fmaf(-u24(r.y), src.inv_span, src.inv_lmin));
            m = disp_lookup(src, ph.lambda, slope);
            const double nb = (1.0 + (double)m) * b2, x = nb * nb;
            if (x > 1.0 && (double)u24(r.x) * (xmax - 1.0) * x < (x - 1.0) * xmax) break;
        }
        // the cone at the photon's own index
        double c = 1.0 / ((1.0 + (double)m) * b2);
        ct = (float)c;
        st = (float)sqrt((1.0 - c) * (1.0 + c));
        ph.ng_c = (1.0f + fmaf(-ph.lambda, slope, m)) * kInvC;
    }
    float sp, cp;
    sincospif(2.0f * u24(w.x), &sp, &cp);
    V3 d = fma3(ct, T, st * fma3(cp, E1, sp * E2));
    ph.d = rsqrtf(dot(d, d)) * d;
    const float s = u24(w.z) * L;
    ph.o = fma3(s, T, P0);
    ph.t0 = s / beta * kInvC;
    return ph;
}

// ---------------------------------------------------------------- ray state

struct Ray {
    V3 o, d;          // current frame (world or instance-local)
    V3 inv;           // 1/d with zeros nudged away
    V3 oi;            // o * inv
};

constexpr float kFarScale = 1.0000004f;

__device__ __forceinline__ float safe_inv(float x) {
    return rcp(fabsf(x) > 1e-30f ? x : copysignf(1e-30f, x));
}

__device__ __forceinline__ void ray_setup(Ray &r, V3 o, V3 d) {
    r.o = o;
    r.d = d;
    r.inv = V3{safe_inv(d.x), safe_inv(d.y), safe_inv(d.z)};
    r.oi = V3{o.x * r.inv.x, o.y * r.inv.y, o.z * r.inv.z};
}

// Watertight permutation and shear of a direction (Woop, Benthin, Wald).
struct Shear {
    int kx, ky, kz;
    float sx, sy, sz;
};
__device__ __forceinline__ Shear make_shear(V3 d) {
    Shear w;
    float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
    w.kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    w.kx = w.kz == 2 ? 0 : w.kz + 1;
    w.ky = w.kx == 2 ? 0 : w.kx + 1;
    float dz = comp(d, w.kz);
    if (dz < 0.0f) { int t = w.kx; w.kx = w.ky; w.ky = t; }
    w.sz = rcp(dz);
    w.sx = comp(d, w.kx) * w.sz;
    w.sy = comp(d, w.ky) * w.sz;
    return w;
}

// Slab test of an AABB with the robust far-distance scaling of Ize (JCGT 2013).
// Returns INFINITY on a miss, else a visiting-order key: the entry distance,
// or, when the ray starts inside the box, the exit distance (an enclosure
// that contains the origin is then visited after the surfaces in front of it,
// whose hits cull most of it).
__device__ __forceinline__ float slab_entry(const Ray &r, float lx, float ly, float lz, float hx, float hy, float hz,
                                            float tmax) {
    float t0x = fmaf(lx, r.inv.x, -r.oi.x), t1x = fmaf(hx, r.inv.x, -r.oi.x);
    float t0y = fmaf(ly, r.inv.y, -r.oi.y), t1y = fmaf(hy, r.inv.y, -r.oi.y);
    float t0z = fmaf(lz, r.inv.z, -r.oi.z), t1z = fmaf(hz, r.inv.z, -r.oi.z);
    float tn = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), 0.0f));
    float tf = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fmaxf(t0z, t1z)) * 1.0000004f;
    tf = fminf(tf, tmax);
    return tn <= tf ? (tn > 0.0f ? tn : tf) : INFINITY;
}

// ---------------------------------------------------------------- closest hit

struct Hit {
    float t;
    uint32_t prim;   // global primitive id (ties: lower wins)
    uint32_t tri;    // triangle slot (meshes)
    int32_t inst;    // instance of the triangle
    int32_t root;    // sphere root taken (caps)
};

__device__ __forceinline__ bool better(float t, uint32_t prim, const Hit &h) {
    return t < h.t || (t == h.t && prim < h.prim);
}

// Sphere cap with the cancellation-free discriminant of Haines et al.
// (Ray Tracing Gems, ch. 7): disc = R^2 - |f - (f.d) d|^2, roots q and c/q.
__device__ __forceinline__ bool hit_cap(const RICH_CONST CapDev &cp, V3 o, V3 d, float tmin, float &t_out, int &root) {
    V3 C = ld3(cp.C);
    V3 f = o - C;
    float b = dot(f, d);
    V3 fp = fma3(-b, d, f);
    float R = cp.R;
    float disc = fmaf(R, R, -dot(fp, fp));
    if (!(disc >= 0.0f)) return false;
    float sq = sqrtf(disc);
    float c = fmaf(-R, R, dot(f, f));
    float q = -(b + copysignf(sq, b));
    if (q == 0.0f) return false;
    float r0 = c * rcp(q), r1 = q;
    float ta = fminf(r0, r1), tb = fmaxf(r0, r1);
    V3 ax = ld3(cp.axis), O = ld3(cp.O), A = ld3(cp.A), B = ld3(cp.B);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        float t = k == 0 ? ta : tb;
        if (!(t > tmin)) continue;
        V3 P = fma3(t, d, o);
        if (dot(P - C, ax) >= 0.0f) continue;
        V3 PO = P - O;
        float a = dot(PO, A), bb = dot(PO, B);
        if (a >= cp.a_lo && a < cp.a_hi && bb >= cp.b_lo && bb < cp.b_hi) {
            t_out = t;
            root = k;
            return true;
        }
    }
    return false;
}

__device__ __forceinline__ bool hit_plane_rect(V3 c, V3 n, V3 U, V3 W, float hu, float hv, V3 o, V3 d, float tmin,
                                               float &t_out) {
    float dn = dot(d, n);
    if (dn == 0.0f) return false;
    V3 co = c - o;
    float t = dot(co, n) * rcp(dn);
    if (!(t > tmin)) return false;
    V3 Pc = fma3(t, d, o - c);
    float u = dot(Pc, U), v = dot(Pc, W);
    if (fabsf(u) <= hu && fabsf(v) <= hv) {
        t_out = t;
        return true;
    }
    return false;
}

// Box surface through the ray's inverse direction: entry or exit, whichever is first beyond tmin.
__device__ __forceinline__ bool hit_box(const RICH_CONST float *lo, const RICH_CONST float *hi, const Ray &r, float tmin, float &t_out) {
    float t0x = fmaf(lo[0], r.inv.x, -r.oi.x), t1x = fmaf(hi[0], r.inv.x, -r.oi.x);
    float t0y = fmaf(lo[1], r.inv.y, -r.oi.y), t1y = fmaf(hi[1], r.inv.y, -r.oi.y);
    float t0z = fmaf(lo[2], r.inv.z, -r.oi.z), t1z = fmaf(hi[2], r.inv.z, -r.oi.z);
    float tn = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fminf(t0z, t1z));
    float tf = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fmaxf(t0z, t1z));
    if (tn > tf) return false;
    if (tn > tmin) { t_out = tn; return true; }
    if (tf > tmin) { t_out = tf; return true; }
    return false;
}

// Watertight ray/triangle test (Woop, Benthin, Wald, JCGT 2013), two-sided.
// A, B, C are the vertices relative to the ray's origin, components in the
// order of the shear (kx, ky, kz).  Each edge function is two rounded products
// and one difference, never contracted into an FMA: only then does a
// triangle's edge function equal the exact negative of its neighbour's for
// their shared edge, so a ray through that edge cannot be rejected by both.
__device__ __forceinline__ bool hit_tri(V3 A, V3 B, V3 C, float sx, float sy, float sz, float tmin, float &t_out) {
#pragma clang fp contract(off)
    float Ax = fmaf(-sx, A.z, A.x), Ay = fmaf(-sy, A.z, A.y);
    float Bx = fmaf(-sx, B.z, B.x), By = fmaf(-sy, B.z, B.y);
    float Cx = fmaf(-sx, C.z, C.x), Cy = fmaf(-sy, C.z, C.y);
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    if (U == 0.0f || V == 0.0f || W == 0.0f) {
        U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
        V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
        W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
    }
    if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return false;
    float det = U + V + W;
    if (det == 0.0f) return false;
    float T = fmaf(U, sz * A.z, fmaf(V, sz * B.z, W * (sz * C.z)));
    float t = T * rcp(det);
    if (!(t > tmin)) return false;
    t_out = t;
    return true;
}

// Re-origin the ray at o (same direction): only the origin terms change.
__device__ __forceinline__ void set_origin(Ray &r, V3 o) {
    r.o = o;
    r.oi = V3{o.x * r.inv.x, o.y * r.inv.y, o.z * r.inv.z};
}

// What a kernel's queries are built for: no meshes; meshes, each lane walking
// the tree on its own; meshes, with the wave phase (photons in an order that
// gives a wave neighbouring rays); meshes, each lane on its own, with the
// wave phase's short stacks in LDS and a fifth wave per SIMD (photon arrays, in
// the order given or sorted by direction: 1e6 in the order given 249 -> 233 us;
// photons of one source sorted by azimuth gain nothing from it).
enum TraceKind { kAnalytic = 0, kMeshLane = 1, kMeshWave = 2, kMeshLoose = 3 };
// LDS words of a wave's stacks.
constexpr int stack_words(TraceKind kind) {
    return kind == kAnalytic   ? 0
           : kind == kMeshLane ? kStackDepth * kStackRow
                               : kLdsRows * kStackRow + (kind == kMeshWave ? kStackDepth : 0);
}

// This lane's traversal stack in a block's LDS (layout at kStackRow).
template <TraceKind kTrace>
__device__ __forceinline__ uint32_t *lane_stack(uint32_t *lds) {
    return lds + (threadIdx.x >> 6) * stack_words(kTrace) + (threadIdx.x & 63);
}

// Nodes a query leaves out: the sheet its ray has just been reflected by.
struct Skip {
    uint32_t lo = 0, n = 0;
    __device__ __forceinline__ bool holds(uint32_t node) const { return node - lo < n; }
};

__device__ __forceinline__ uint32_t first_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint32_t lane_value(float x, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane);
}
typedef unsigned long long Mask;   // lanes of a wave

// Bit k set where the k-th mask is not zero: eight scalar instructions (left
// to itself the compiler takes one of the four through a vector register).
__device__ __forceinline__ uint32_t nonzero4(Mask m0, Mask m1, Mask m2, Mask m3) {
    uint32_t r;
    asm("s_cmp_lg_u64 %4, 0\n\t"
        "s_cselect_b32 %0, 1, 0\n\t"
        "s_cmp_lg_u64 %3, 0\n\t"
        "s_addc_u32 %0, %0, %0\n\t"
        "s_cmp_lg_u64 %2, 0\n\t"
        "s_addc_u32 %0, %0, %0\n\t"
        "s_cmp_lg_u64 %1, 0\n\t"
        "s_addc_u32 %0, %0, %0"
        : "=&s"(r)
        : "s"(m0), "s"(m1), "s"(m2), "s"(m3)
        : "scc");
    return r;
}

// What the rays of a wave have in common in the current frame: where a node
// keeps its near and far planes for the signs of their direction (byte
// offsets), the signs (bit a: component a is not negative) and the axis they
// run along most.
struct WaveRays {
    uint32_t nx, fx, ny, fy, nz, fz;
    uint32_t signs;
    int axis;
};

// True when every active lane's ray has the same signs and dominant axis.
__device__ __forceinline__ bool wave_rays(const Ray &r, WaveRays &w) {
    const Mask all = __ballot(1);
    const Mask x = __ballot(r.inv.x >= 0.0f), y = __ballot(r.inv.y >= 0.0f), z = __ballot(r.inv.z >= 0.0f);
    const float ax = fabsf(r.d.x), ay = fabsf(r.d.y), az = fabsf(r.d.z);
    const int axis = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
    w.axis = (int)first_lane((uint32_t)axis);
    w.nx = x ? 0u : 16u;
    w.fx = 16u - w.nx;
    w.ny = y ? 32u : 48u;
    w.fy = 80u - w.ny;
    w.nz = z ? 64u : 80u;
    w.fz = 144u - w.nz;
    w.signs = (x ? 1u : 0u) | (y ? 2u : 0u) | (z ? 4u : 0u);
    return (x == 0ull || x == all) && (y == 0ull || y == all) && (z == 0ull || z == all) &&
           __ballot(axis == w.axis) == all;
}

// Tests the triangles of a leaf, the same for the whole wave, by the lanes of
// `m`: hit_tri and the best-hit update without branches.
__device__ __forceinline__ void wave_leaf(SceneRef S, const Ray &r, int axis, uint32_t ref, Mask m, int inst,
                                          Hit &h) {
#pragma clang fp contract(off)
    if (!__builtin_amdgcn_inverse_ballot_w64(m)) return;
    work(kWorkWaveLeaves);
    const RICH_CONST char *const tris = (const RICH_CONST char *)S.tris;
    // components in the cyclic order that ends with the dominant axis; the
    // shear's swap of the first two for a negative axis only flips the signs
    // of all edge functions
    const bool a0 = axis == 0, a2 = axis == 2;
    auto one = [&](float x, float y, float z) {
        const float yz = a0 ? y : z;
        return a2 ? x : yz;
    };
    auto turn = [&](float x, float y, float z) { return V3{one(x, y, z), one(y, z, x), one(z, x, y)}; };
    const V3 d = turn(r.d.x, r.d.y, r.d.z), o = turn(r.o.x, r.o.y, r.o.z);
    const float sz = rcp(d.z), sx = d.x * sz, sy = d.y * sz;
    const uint32_t first = ref & 0x07FFFFFFu, end = first + ((ref >> 27) & 7u) + 1u;
    const uint32_t prim_tri = S.prim_tri;
    const float tmin = S.t_min;
    for (uint32_t t = first; t < end; ++t) {
        work(kWorkWaveTris);
        const Float4 a = *(const RICH_CONST Float4 *)(tris + (t << 6));
        const Float4 b = *(const RICH_CONST Float4 *)(tris + ((t << 6) + 16u));
        const Float4 c = *(const RICH_CONST Float4 *)(tris + ((t << 6) + 32u));
        const V3 A = turn(a.x, a.y, a.z) - o, B = turn(b.x, b.y, b.z) - o, C = turn(c.x, c.y, c.z) - o;
        const float Ax = fmaf(-sx, A.z, A.x), Ay = fmaf(-sy, A.z, A.y);
        const float Bx = fmaf(-sx, B.z, B.x), By = fmaf(-sy, B.z, B.y);
        const float Cx = fmaf(-sx, C.z, C.x), Cy = fmaf(-sy, C.z, C.y);
        float U = Cx * By - Cy * Bx, V = Ax * Cy - Ay * Cx, W = Bx * Ay - By * Ax;
        const bool zero = fminf(fminf(fabsf(U), fabsf(V)), fabsf(W)) == 0.0f;
        if (__ballot(zero)) {
            if (zero) {
                U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
                V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
                W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
            }
        }
        const float det = U + V + W;
        const float T = fmaf(U, sz * A.z, fmaf(V, sz * B.z, W * (sz * C.z)));
        const float th = T * rcp(det);
        const uint32_t prim = prim_tri + __float_as_uint(a.w);
        const float least = fminf(fminf(U, V), W), most = fmaxf(fmaxf(U, V), W);
        const bool hit = !((least < 0.0f) & (most > 0.0f)) & (det != 0.0f) & (th > tmin) &
                         ((th < h.t) | ((th == h.t) & (prim < h.prim)));
        h.t = hit ? th : h.t;
        h.prim = hit ? prim : h.prim;
        h.tri = hit ? t : h.tri;
        h.inst = hit ? inst : h.inst;
    }
}

// Rounding of a lane's plane distances: inv and the two roundings of
// (org - o) * inv are relative to the distance plus the plane's own offset in
// its node; the builder's margin covers the latter (see write_lane_axis), and
// this the former for a near and a far plane of different axes (10 x 2^-24).
constexpr float kLaneFarScale = 1.000001f;

// Lane phase: this lane works through its own stack, from entry sp down.
// r, inst: the frame the entries were met in, left as they were.  kRows: the
// LDS rows of its stack, of kAll entries.
template <int kRows, int kAll>
__device__ __forceinline__ void lane_walk(SceneRef S, const V3 ow, const V3 dw, Ray &r, int inst, int sp, Hit &h,
                                          uint32_t *stk, Skip skip) {
    bool moved = false;   // current frame rotated/scaled (a parametrised segment)
    constexpr int kEnd = kAll * kStackRow, kLds = kRows * kStackRow;
    const float tmin = S.t_min;
    uint32_t deep[kAll > kRows ? kAll - kRows : 1];   // entries beyond the LDS rows
    auto push = [&](uint32_t x) {
        if (kAll == kRows || sp < kLds) stk[sp] = x;
        else deep[(sp - kLds) / kStackRow] = x;
        sp += kStackRow;
    };
    auto top = [&]() -> uint32_t {
        sp -= kStackRow;
        return kAll == kRows || sp < kLds ? stk[sp] : deep[(sp - kLds) / kStackRow];
    };
    uint32_t ref = top();
    while (true) {
        if (!(ref & kLeafBit)) {
            if (skip.holds(ref)) {
                if (sp == 0) break;
                ref = top();
                continue;
            }
            work(kWorkNodes);
            // 32-bit byte offsets from the uniform base keep the address
            // arithmetic scalar
            const float4 *nb = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(S.lane_nodes) + (ref << 6));
            const float4 q0 = nb[0], q1 = nb[1];
            const uint4 q2 = *reinterpret_cast<const uint4 *>(nb + 2), ch = *reinterpret_cast<const uint4 *>(nb + 3);
            // near/far planes per axis follow the direction signs
            const bool px = r.inv.x >= 0.0f, py = r.inv.y >= 0.0f, pz = r.inv.z >= 0.0f;
            const uint32_t lox = __float_as_uint(q1.z), hix = __float_as_uint(q1.w);
            const uint32_t nx = px ? lox : hix, fx = px ? hix : lox;
            const uint32_t ny = py ? q2.x : q2.y, fy = py ? q2.y : q2.x;
            const uint32_t nz = pz ? q2.z : q2.w, fz = pz ? q2.w : q2.z;
            const float sx = q0.w * r.inv.x, sy = q1.x * r.inv.y, sz = q1.y * r.inv.z;
            const float bx = (q0.x - r.o.x) * r.inv.x, by = (q0.y - r.o.y) * r.inv.y, bz = (q0.z - r.o.z) * r.inv.z;
            const float tmax = h.t;
            auto key = [&](int c) -> uint32_t {
                auto q = [&](uint32_t planes) { return (float)((planes >> (8 * c)) & 255u); };
                const float tn = fmaxf(fmaxf(fmaf(q(nx), sx, bx), fmaf(q(ny), sy, by)), fmaf(q(nz), sz, bz));
                float tf = fminf(fminf(fmaf(q(fx), sx, bx), fmaf(q(fy), sy, by)), fmaf(q(fz), sz, bz));
                tf = fminf(tf * kLaneFarScale, tmax);
                return __float_as_uint(tn > tf ? INFINITY : (tn > 0.0f ? tn : tf));   // (tn may be no number)
            };
            // keys: distance bits with the child slot in the two lowest mantissa bits
            // (non-negative floats order like unsigned integers; a miss is +inf,
            // or negative for a box behind the origin)
            uint32_t k0 = (key(0) & ~3u) | 0u;
            uint32_t k1 = (key(1) & ~3u) | 1u;
            uint32_t k2 = (key(2) & ~3u) | 2u;
            uint32_t k3 = (key(3) & ~3u) | 3u;
            // 4-element sorting network, branch-free
            uint32_t t;
            t = min(k0, k1); k1 = max(k0, k1); k0 = t;
            t = min(k2, k3); k3 = max(k2, k3); k2 = t;
            t = min(k0, k2); k2 = max(k0, k2); k0 = t;
            t = min(k1, k3); k3 = max(k1, k3); k1 = t;
            t = min(k1, k2); k2 = max(k1, k2); k1 = t;
            const uint32_t kMiss = 0x7F800000u;   // +inf
            if (k0 >= kMiss) {
                if (sp == 0) break;
                ref = top();
                continue;
            }
            // child of a key by its slot bits, with selects only
            auto pick = [&](uint32_t k) -> uint32_t {
                const uint32_t lo = (k & 1u) ? ch.y : ch.x;
                const uint32_t hi = (k & 1u) ? ch.w : ch.z;
                return (k & 2u) ? hi : lo;
            };
            // the hit children after the nearest go on the stack, farthest
            // deepest; the keys are sorted, so k3 hit implies k2 and k1 hit
            uint32_t p2 = k2 < kMiss, p3 = k3 < kMiss;
            int need = (k1 < kMiss) + (int)p2 + (int)p3;
            if (sp + need * kStackRow > kLds) {
                if (sp + need * kStackRow > kEnd) {
                    atomicOr(S.status, 2u);  // RICH_FLAG_STACK_OVERFLOW: the farthest are dropped
                    need = (kEnd - sp) / kStackRow;
                }
                if (need >= 3) push(pick(k3));
                if (need >= 2) push(pick(k2));
                if (need >= 1) push(pick(k1));
            } else if (need > 0) {
                // the entries land in slots 0..need-1 above the top: a write to
                // a slot that a later write also takes is overwritten by it
                stk[sp] = pick(k3);
                stk[sp + (int)p3 * kStackRow] = pick(k2);
                stk[sp + (int)(p2 + p3) * kStackRow] = pick(k1);
                sp += need * kStackRow;
            }
            ref = pick(k0);
            continue;
        }
        if (ref == kExitMarker) {
            if (moved) ray_setup(r, ow, dw);
            else set_origin(r, ow);
            inst = -1;
            moved = false;
        } else if (ref & kInstBit) {
            int k = (int)(ref & ~(kLeafBit | kInstBit));
            const Instance &in = S.inst[k];
            if (sp == kEnd) {
                atomicOr(S.status, 2u);
            } else if (!skip.holds(in.root)) {
                push(kExitMarker);
                work(kWorkInstances);
                if (in.segment < 0) {
                    set_origin(r, ow - ld3(in.org));   // fixed instances only translate
                } else {
                    work(kWorkMovingInstances);
                    ray_setup(r, mat3(in.m, ow - ld3(in.org)), mat3(in.m, dw));
                    moved = true;
                }
                inst = k;
                ref = in.root;
                continue;
            }
        } else {
            uint32_t first = ref & 0x07FFFFFFu;
            uint32_t cnt = ((ref >> 27) & 7u) + 1u;
            work(kWorkLeaves);
            const Shear sh = make_shear(r.d);
            auto vert = [&](const float4 &v) {
                const V3 q = V3{v.x, v.y, v.z} - r.o;
                return V3{comp(q, sh.kx), comp(q, sh.ky), comp(q, sh.kz)};
            };
            for (uint32_t q = first; q < first + cnt; ++q) {
                work(kWorkTris);
                const char *tb = reinterpret_cast<const char *>(S.tris) + (q << 6);
                float4 a = *reinterpret_cast<const float4 *>(tb);
                float4 b = *reinterpret_cast<const float4 *>(tb + 16);
                float4 c = *reinterpret_cast<const float4 *>(tb + 32);
                float t;
                if (hit_tri(vert(a), vert(b), vert(c), sh.sx, sh.sy, sh.sz, tmin, t)) {
                    uint32_t prim = S.prim_tri + __float_as_uint(a.w);
                    if (better(t, prim, h)) {
                        h.t = t;
                        h.prim = prim;
                        h.tri = q;
                        h.inst = inst;
                    }
                }
            }
        }
        if (sp == 0) break;
        ref = top();
    }
}

// Closest triangle along (ow, dw) with t < h.t, through the two-level BVH4.
//
// Wave phase (kMeshWave).  A wave's photons leave in neighbouring directions, so
// its rays share most of their way down the tree.  While they do, the wave
// walks it together: a node is read once, through the scalar cache (the
// return path of 7 x 16 bytes for each lane was 95 % busy), one stack in LDS
// holds the wave's references, a child costs 12 vector operations to test and
// none to sort or pick, and a leaf is tested at once by the lanes that meet
// its box.  A node below which the rays part (three or four children met, or
// two with fewer than one in kWaveShare of the rays left) goes onto the stacks
// of the lanes that meet it.
// Lane phase.  Every lane works through its own stack.  It runs when three
// quarters of the lanes have something there, before the wave changes frames,
// and at the end; so near surfaces still cut off far ones.  Rays of different
// signs or dominant axes go straight to it.
// The order of visits never changes the result: the closest hit is exact and
// ties go to the lower primitive.
// 1e7 photons from a point on 210,082 triangles: 20 nodes and 8 triangles per
// 64 photons, 2,790 vector and 2,540 scalar instructions; 1.29 -> 1.03 ms.
// Bound by instruction issue and its stalls (vector units 65 % busy, five
// waves per SIMD), no longer by the vector-memory return path.
//
// stk is this lane's stack (lane_stack); sp is the word offset of its next
// free entry, depth x kStackRow.
template <TraceKind kTrace>
__device__ __forceinline__ void traverse(SceneRef S, const Ray &world, Hit &h, uint32_t *stk, Skip skip) {
    const V3 ow = world.o, dw = world.d;
    Ray r = world;
    int inst = -1;
    if constexpr (kTrace != kMeshWave) {
        stk[0] = S.top_root;
        lane_walk<kTrace == kMeshLane ? kStackDepth : kLdsRows, kStackDepth>(S, ow, dw, r, inst, kStackRow, h, stk, skip);
        return;
    }
    uint32_t *const ustk = stk + kLdsRows * kStackRow - (threadIdx.x & 63);
    const int active = (int)__popcll(__ballot(1));
    const uint32_t skip_lo = first_lane(skip.lo);    // what all lanes leave out
    const uint32_t skip_n = __ballot(skip.lo != skip_lo || skip.n != first_lane(skip.n)) ? 0u : first_lane(skip.n);
    constexpr uint32_t kNone = kExitMarker;
    uint32_t next = S.top_root;   // what the wave visits next (kNone: the next entry of its stack)
    int usp = 0, base = 0;        // its stack, and where the current frame's entries begin
    int sp = 0;                   // this lane's stack
    bool pending = false;         // lanes have entries on theirs
    WaveRays w;
    if (!wave_rays(r, w)) {
        stk[0] = next;
        sp = kStackRow;
        pending = true;
        next = kNone;
    }
    while (true) {
        // walk nodes of the current frame together
        while (true) {
            if (next == kNone) {
                if (usp == base || (pending && 4 * (int)__popcll(__ballot(sp > 0)) >= 3 * active)) break;
                next = first_lane(ustk[--usp]);
            }
            if (next & kLeafBit) break;
            const uint32_t at = next << 7;
            const bool left_out = next - skip_lo < skip_n;
            next = kNone;
            if (!left_out) {
                work(kWorkWaveNodes);
                const RICH_CONST char *const nodes = (const RICH_CONST char *)S.nodes;
                auto plane = [&](uint32_t side) { return *(const RICH_CONST Float4 *)(nodes + (at + side)); };
                const Float4 nx = plane(w.nx), fx = plane(w.fx), ny = plane(w.ny), fy = plane(w.fy),
                             nz = plane(w.nz), fz = plane(w.fz);
                const Uint8 ch = *(const RICH_CONST Uint8 *)(nodes + (at + 96u));   // children, leaves, order
                auto meets = [&](int c) -> Mask {
                    const float tn = fmaxf(fmaxf(fmaf(nx[c], r.inv.x, -r.oi.x), fmaf(ny[c], r.inv.y, -r.oi.y)),
                                           fmaxf(fmaf(nz[c], r.inv.z, -r.oi.z), 0.0f));
                    const float tf = fminf(fminf(fmaf(fx[c], r.inv.x, -r.oi.x), fmaf(fy[c], r.inv.y, -r.oi.y)),
                                           fmaf(fz[c], r.inv.z, -r.oi.z));
                    return __ballot(tn <= fminf(tf * kFarScale, h.t));
                };
                const Mask m0 = meets(0), m1 = meets(1), m2 = meets(2), m3 = meets(3);
                uint32_t met = nonzero4(m0, m1, m2, m3);
                const uint32_t more = met & (met - 1u);   // without its lowest child
                // in registers by now, so that no second wait follows the branch
                asm volatile("" ::"s"(ch));
                if (more != 0u && ((more & (more - 1u)) != 0u ||
                                   kWaveShare * (int)__popcll(m0 | m1 | m2 | m3) < active)) {
                    // the rays part here
                    if (__builtin_amdgcn_inverse_ballot_w64(m0 | m1 | m2 | m3)) {
                        stk[sp] = at >> 7;
                        sp += kStackRow;
                    }
                    pending = true;
                    if (__ballot(sp >= kPending * kStackRow)) break;
                } else {
                    auto child = [&](uint32_t set) {   // of the lowest bit
                        return (set & 1u) ? ch[0] : ((set & 2u) ? ch[1] : ((set & 4u) ? ch[2] : ch[3]));
                    };
                    uint32_t leaves = met & ch[4];
                    met ^= leaves;
                    while (leaves) {
                        const Mask who = (leaves & 1u) ? m0 : ((leaves & 2u) ? m1 : ((leaves & 4u) ? m2 : m3));
                        wave_leaf(S, r, w.axis, child(leaves), who, inst, h);
                        leaves &= leaves - 1u;
                    }
                    if (met) {
                        next = child(met);
                        const uint32_t other = met & (met - 1u);
                        if (other) {
                            // two: which lies first along the rays (Node4::order)
                            const uint32_t pair = (uint32_t)(0x5042003100000ull >> (4u * met)) & 15u;
                            const uint32_t o3 = ch[5] >> (3u * pair);
                            uint32_t far = child(other);
                            if ((((w.signs >> (o3 & 3u)) ^ (o3 >> 2)) & 1u) != 0u) {
                                const uint32_t t = far;
                                far = next;
                                next = t;
                            }
                            if (usp == kStackDepth) atomicOr(S.status, 2u);  // stack overflow: the far one is dropped
                            else ustk[usp++] = far;
                        }
                    }
                }
            }
        }
        if (pending) {
            if (sp > 0) lane_walk<kLdsRows, kLaneRows>(S, ow, dw, r, inst, sp, h, stk, skip);
            sp = 0;
            pending = false;
        }
        if (next == kNone) {
            if (usp > base) continue;
            if (inst < 0) break;
            // the end of an instance
            set_origin(r, ow);
            inst = -1;
            base = 0;
            continue;
        }
        if (!(next & kLeafBit)) continue;
        // an instance
        const int k = (int)(next & ~(kLeafBit | kInstBit));
        next = kNone;
        const RICH_CONST Instance &in = cref(S.inst[k]);
        if (in.root - skip_lo < skip_n) continue;
        if (in.segment >= 0) {
            // a moving segment: each lane that meets its box enters on its own
            if (slab_entry(r, in.lo[0], in.lo[1], in.lo[2], in.hi[0], in.hi[1], in.hi[2], h.t) < INFINITY) {
                stk[0] = make_inst((uint32_t)k);
                sp = kStackRow;
            }
            pending = true;
            continue;
        }
        work(kWorkInstances);
        set_origin(r, ow - ld3(in.org));   // fixed instances only translate
        inst = k;
        base = usp;
        next = in.root;
    }
}

template <TraceKind kTrace>
__device__ __forceinline__ void closest_hit(SceneRef S, V3 o, V3 d, Hit &h, uint32_t *stk, Skip skip) {
    const RICH_CONST DetDev &det = cref(*S.det);
    h.t = INFINITY;
    h.prim = 0xFFFFFFFFu;
    h.tri = 0;
    h.inst = -1;
    h.root = 0;
    const float tmin = S.t_min;
    Ray r;
    ray_setup(r, o, d);
    float t;
    for (int i = 0; i < S.n_caps; ++i) {
        const RICH_CONST CapDev &cp = cref(S.caps[i]);
        work(kWorkCapBoxes);
        if (slab_entry(r, cp.lo[0], cp.lo[1], cp.lo[2], cp.hi[0], cp.hi[1], cp.hi[2], h.t) == INFINITY) continue;
        work(kWorkCaps);
        int root;
        if (hit_cap(cp, o, d, tmin, t, root) && better(t, (uint32_t)i, h)) {
            h.t = t;
            h.prim = (uint32_t)i;
            h.root = root;
        }
    }
    for (int i = 0; i < S.n_rects; ++i) {
        const RICH_CONST RectDev &rc = cref(S.rects[i]);
        work(kWorkRects);
        if (hit_plane_rect(ld3(rc.c), ld3(rc.n), ld3(rc.u), ld3(rc.v), rc.hu, rc.hv, o, d, tmin, t) &&
            better(t, (uint32_t)(S.n_caps + i), h)) {
            h.t = t;
            h.prim = (uint32_t)(S.n_caps + i);
        }
    }
    if (hit_plane_rect(ld3(det.c), ld3(det.n), ld3(det.u), ld3(det.v), det.hu, det.hv, o, d, tmin, t) &&
        better(t, S.prim_det, h)) {
        h.t = t;
        h.prim = S.prim_det;
    }
    if (S.has_box) work(kWorkBoxes);
    if (S.has_box && hit_box(S.box_lo, S.box_hi, r, tmin, t) && better(t, S.prim_box, h)) {
        h.t = t;
        h.prim = S.prim_box;
    }
    if constexpr (kTrace != kAnalytic) traverse<kTrace>(fresh(S), r, h, stk, skip);
}

// Reflectivity of material `mat` at `lambda`.  The loop over materials is
// uniform so every table is read through scalar loads; lanes select their own.
__device__ __forceinline__ float reflectivity(SceneRef S, int mat, float lambda) {
    float v = 0.0f;
    for (int m = 0; m < S.n_mats; ++m) {
        const RICH_CONST MatDev &M = cref(S.mats[m]);
        if (M.kind != 0) continue;
        float r = lerp_table(M.n, M.x, M.y, M.s, lambda);
        v = (mat == m) ? r : v;
    }
    return v;
}

// ---------------------------------------------------------------- interaction

constexpr int kDetected = 0, kQeRejected = 1, kAbsorbedMirror = 2, kAbsorbed = 3, kEscaped = 4, kMaxBounces = 5;

struct PathEnd {
    int fate;
    int pixel;
    V3 P;
    float u, v;
    float time;     // arrival time at the detector hit (ns)
};

// Receives every reflection and the detector hit; the forward kernels ignore them.
struct NoRecord {
    __device__ __forceinline__ void reflect(int b, const Hit &h, V3 o, V3 d, V3 P, V3 n) {}
    __device__ __forceinline__ void detect(int b, V3 o, V3 d, float t) {}
};

// sheet: 1 + the index of the sheet the hit facet belongs to, or 0.
__device__ __forceinline__ V3 surface_normal(SceneRef S, const Hit &h, V3 P, int &mat, uint32_t &sheet) {
    sheet = 0;
    if (h.prim < (uint32_t)S.n_caps) {
        const CapDev &cp = S.caps[h.prim];
        mat = cp.material;
        return rcp(cp.R) * (ld3(cp.C) - P);
    }
    if (h.prim < S.prim_det) {
        const RectDev &rc = S.rects[h.prim - S.n_caps];
        mat = rc.material;
        return ld3(rc.n);
    }
    const Tri &tr = S.tris[h.tri];
    mat = (int)tr.material;
    sheet = tr.sheet;
    V3 n = ld3(tr.n);
    if (h.inst >= 0 && S.inst[h.inst].segment >= 0) n = mat3(S.inst[h.inst].rot, n);
    return n;
}

constexpr int kPrefiltered = 6;

// Pre-propagation efficiency filter: keep the photon with probability
// QE(lambda) * prod_k refl_k(lambda), as one accept-reject per photon.
__device__ __forceinline__ bool prefilter_keep(SceneRef S, SourceRef src, const Photon &ph, uint64_t seed,
                                               uint64_t g) {
    const RICH_CONST DetDev &det = cref(*S.det);
    float p = lerp_table(det.n_qe, det.qe_x, det.qe_y, det.qe_s, ph.lambda);
    for (int k = 0; k < src.pf_n; ++k) p *= reflectivity(S, src.pf_mats[k], ph.lambda);
    return u24(photon_block(seed, g, kPrefilterBlock).x) < p;
}

// Trace one photon.  With kEfficiencies false
// (photons kept by the pre-filter) mirrors always reflect and the detector
// always detects.  Kernels are built for each combination, so that none holds
// the code and registers of the others.
template <TraceKind kTrace, bool kEfficiencies, class Rec>
__device__ __forceinline__ void propagate(SceneRef scene, const Photon &ph, uint64_t seed, uint64_t g, uint32_t *stk,
                                          PathEnd &end, Rec &rec) {
    V3 o = ph.o, d = ph.d;
    end.fate = kMaxBounces;
    end.pixel = -1;
    // a track below the Cherenkov threshold has no cone (NaN direction): no light
    if (!(fabsf(d.x) <= 1.0f && fabsf(d.y) <= 1.0f && fabsf(d.z) <= 1.0f)) {
        end.fate = kEscaped;
        return;
    }
    uint4 blk = make_uint4(0, 0, 0, 0);
    int have = -1;
    float clock = ph.t0;        // time at the start of the current segment (ns)
    Skip skip;
    work(kWorkPhotons);
    for (int b = 0; b < scene.max_bounces; ++b) {
        Hit h;
        work(kWorkQueries);
        closest_hit<kTrace>(fresh(scene), o, d, h, stk, skip);
        SceneRef S = fresh(scene);
        const RICH_CONST DetDev &det = cref(*S.det);
        if (h.prim == 0xFFFFFFFFu) {
            end.fate = kEscaped;
            break;
        }
        if (h.prim == S.prim_det) {
            if (dot(d, ld3(det.n)) >= 0.0f) {
                end.fate = kAbsorbed;
                break;
            }
            V3 Pc = fma3(h.t, d, o - ld3(det.c));
            float u = dot(Pc, ld3(det.u)), v = dot(Pc, ld3(det.v));
            float fi = floorf((u + det.act_hu) * det.inv_pitch), fj = floorf((v + det.act_hv) * det.inv_pitch);
            if (!(fi >= 0.0f && fi < (float)det.nx && fj >= 0.0f && fj < (float)det.ny)) {  // NaN-safe
                end.fate = kAbsorbed;
                break;
            }
            end.pixel = (int)fj * det.nx + (int)fi;
            end.P = fma3(h.t, d, o);
            end.u = u;
            end.v = v;
            end.time = fmaf(h.t, ph.ng_c, clock);
            work(kWorkDetections);
            rec.detect(b, o, d, h.t);
            if constexpr (kEfficiencies) {
                float qe = lerp_table(det.n_qe, det.qe_x, det.qe_y, det.qe_s, ph.lambda);
                end.fate = ph.u_qe < qe ? kDetected : kQeRejected;
            } else {
                end.fate = kDetected;
            }
            break;
        }
        if (h.prim == S.prim_box) {
            end.fate = kAbsorbed;
            break;
        }
        V3 P = fma3(h.t, d, o);
        int mat;
        uint32_t sheet;
        V3 n = surface_normal(S, h, P, mat, sheet);
        if (S.mats[mat].kind != 0 || dot(d, n) >= 0.0f) {
            end.fate = kAbsorbed;
            break;
        }
        if constexpr (kEfficiencies) {
            int bid = 1 + (b >> 2);
            if (have != bid) {
                blk = photon_block(seed, g, (uint32_t)bid);
                have = bid;
            }
            int w = b & 3;
            uint32_t word = w == 0 ? blk.x : (w == 1 ? blk.y : (w == 2 ? blk.z : blk.w));
            float refl = reflectivity(S, mat, ph.lambda);
            if (u24(word) >= refl) {
                end.fate = kAbsorbedMirror;
                break;
            }
        }
        work(kWorkReflections);
        rec.reflect(b, h, o, d, P, n);
        clock = fmaf(h.t, ph.ng_c, clock);
        skip = Skip{};
        if (sheet != 0u && h.t <= S.sheet_reach) {
            const Sheet sh = S.sheets[sheet - 1u];
            if (-dot(d, n) >= sh.min_cos) skip = Skip{sh.node_lo, sh.node_n};
        }
        V3 dr = fma3(-2.0f * dot(d, n), n, d);
        d = rsqrtf(dot(dr, dr)) * dr;
        o = P;
    }
}

}  // namespace rich
