// librich kernels for gfx950: parameter refresh, forward propagation (one
// photon per lane), the persistent batch kernel, and small helpers.
#include <hip/hip_runtime.h>

#include <atomic>

#include "kernels.h"
#include "trace.h"

namespace rich {

// ---------------------------------------------------------------- parameters (FP64)

namespace {

struct D3 {
    double x, y, z;
};
__device__ inline D3 dload(const double *p) { return D3{p[0], p[1], p[2]}; }
__device__ inline D3 dadd(D3 a, D3 b) { return D3{a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ inline D3 dsub(D3 a, D3 b) { return D3{a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline D3 dmul(D3 a, double s) { return D3{a.x * s, a.y * s, a.z * s}; }
__device__ inline double ddot(D3 a, D3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline D3 dcross(D3 a, D3 b) {
    return D3{a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
// rotation of v about unit axis k by angle th (Rodrigues)
__device__ inline D3 drot(D3 k, double th, D3 v) {
    double c = cos(th), s = sin(th);
    return dadd(dadd(dmul(v, c), dmul(dcross(k, v), s)), dmul(k, ddot(k, v) * (1.0 - c)));
}
__device__ inline void store3(float *p, D3 v) {
    p[0] = (float)v.x;
    p[1] = (float)v.y;
    p[2] = (float)v.z;
}

}  // namespace

// One axis of a node for a lane's own walk.  The grid spans the children's
// boxes widened by 2^-20 of the largest coordinate, and each plane is at least
// 2^-21 of it outside the box: more than the walk's rounding of a plane's
// offset in the node (three operations of 2^-24 of at most twice that).  An axis
// along which a child reaches beyond FP32 has no number for its planes, so
// that the walk takes no notice of it.
__device__ void write_lane_axis(const Node4 &n, LaneNode &out, int a) {
    const float *lo_of = a == 0 ? n.lox : (a == 1 ? n.loy : n.loz), *hi_of = a == 0 ? n.hix : (a == 1 ? n.hiy : n.hiz);
    double lo = 1e300, hi = -1e300;
    uint32_t first = kEmpty;
    // a box that is no number (parameters out of range) is never met, like an empty slot
    auto has_box = [&](int c) { return n.child[c] != kEmpty && lo_of[c] <= hi_of[c]; };
    bool open = false;
    for (int c = 3; c >= 0; --c) {
        if (n.child[c] != kEmpty) first = n.child[c];
        if (!has_box(c)) continue;
        open = open || isinf(lo_of[c]) || isinf(hi_of[c]);
        lo = fmin(lo, (double)lo_of[c]);
        hi = fmax(hi, (double)hi_of[c]);
    }
    const double slack = fmax(fabs(lo), fabs(hi)) * 0x1p-21;
    float org = (float)(lo - 2.0 * slack);
    float step = (float)((hi + 2.0 * slack - (double)org) * (1.000001 / 255.0));
    if (lo > hi) org = INFINITY, step = 0.0f;   // no box: the node's planes lie nowhere
    if (open) org = NAN, step = 0.0f;
    const double inv = 1.0 / (double)step;
    uint32_t qlo = 0, qhi = 0;
    for (int c = 0; c < 4; ++c) {
        int l = 255, h = 0;
        if (has_box(c)) {
            l = 0, h = 255;
            if (step > 0.0f) {
                const double want_l = (double)lo_of[c] - slack - org, want_h = (double)hi_of[c] + slack - org;
                l = (int)fmin(fmax(floor(want_l * inv), 0.0), 255.0);
                h = (int)fmin(fmax(ceil(want_h * inv), 0.0), 255.0);
                if (l > 0 && l * (double)step > want_l) --l;
                if (h < 255 && h * (double)step < want_h) ++h;
            }
        }
        qlo |= (uint32_t)l << (8 * c);
        qhi |= (uint32_t)h << (8 * c);
    }
    out.org[a] = org;
    out.step[a] = step;
    uint32_t *const q = &out.lox + 2 * a;
    q[0] = qlo;
    q[1] = qhi;
    if (a == 0)
        for (int c = 0; c < 4; ++c) out.child[c] = n.child[c] != kEmpty ? n.child[c] : first;
}

// Every node's (or the top level's) form for a lane's own walk.
__global__ __launch_bounds__(256) void lane_nodes_kernel(const Node4 *nodes, LaneNode *out, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        for (int a = 0; a < 3; ++a) write_lane_axis(nodes[i], out[i], a);
}

// One thread per cap and per instance; then the sheets' rules are switched and
// the top level's boxes refitted.
__global__ void prepare_kernel(PrepareArgs a) {
    int tid = threadIdx.x;
    for (int i = tid; i < a.n_caps; i += blockDim.x) {
        const CapStatic &cs = a.caps_static[i];
        const SegDev &sg = a.segs[cs.segment];
        const float *p = a.params + 6 * cs.segment;
        double tx = p[0], ty = p[1], R = p[2];
        D3 e1 = dload(sg.e1), e2 = dload(sg.e2), u0 = dload(sg.u0);
        D3 r1 = drot(e1, tx, u0);
        D3 ax = drot(e2, ty, r1);
        D3 C = dadd(dadd(dload(sg.pivot), D3{p[3], p[4], p[5]}), dmul(ax, R));
        CapDev &cd = a.caps[i];
        store3(cd.C, C);
        cd.R = (float)R;
        store3(cd.axis, ax);
        cd.segment = cs.segment;
        store3(cd.O, dload(cs.O));
        cd.material = cs.material;
        store3(cd.A, dload(cs.A));
        store3(cd.B, dload(cs.B));
        cd.a_lo = (float)cs.bounds[0];
        cd.a_hi = (float)cs.bounds[1];
        cd.b_lo = (float)cs.bounds[2];
        cd.b_hi = (float)cs.bounds[3];
        store3(cd.dCdtx, dmul(drot(e2, ty, dcross(e1, r1)), R));
        store3(cd.dCdty, dmul(dcross(e2, ax), R));
        // box of the cap: the cell prism over the sphere heights reached inside the cell
        D3 O = dload(cs.O), A = dload(cs.A), B = dload(cs.B);
        D3 W = dcross(A, B);
        D3 CO = dsub(C, O);
        double ca = ddot(CO, A), cb = ddot(CO, B), cw = ddot(CO, W);
        double sgn = ddot(ax, W) > 0 ? -1.0 : 1.0;   // pivot side of the centre along W
        double qa = fmin(fmax(ca, cs.bounds[0]), cs.bounds[1]) - ca;
        double qb = fmin(fmax(cb, cs.bounds[2]), cs.bounds[3]) - cb;
        double rmin2 = qa * qa + qb * qb;
        double fa = fmax(fabs(cs.bounds[0] - ca), fabs(cs.bounds[1] - ca));
        double fb = fmax(fabs(cs.bounds[2] - cb), fabs(cs.bounds[3] - cb));
        double rmax2 = fa * fa + fb * fb;
        double h0 = cw + sgn * sqrt(fmax(0.0, R * R - rmax2));
        double h1 = cw + sgn * sqrt(fmax(0.0, R * R - rmin2));
        double hlo = fmin(h0, h1), hhi = fmax(h0, h1);
        double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
        for (int c = 0; c < 8; ++c) {
            double aa = cs.bounds[(c & 1) ? 1 : 0], bb = cs.bounds[(c & 2) ? 3 : 2], hh = (c & 4) ? hhi : hlo;
            D3 P = dadd(dadd(dadd(O, dmul(A, aa)), dmul(B, bb)), dmul(W, hh));
            double q[3] = {P.x, P.y, P.z};
            for (int k = 0; k < 3; ++k) {
                lo[k] = fmin(lo[k], q[k]);
                hi[k] = fmax(hi[k], q[k]);
            }
        }
        for (int k = 0; k < 3; ++k) {
            double pad = 1e-2 + 1e-6 * fmax(fabs(lo[k]), fabs(hi[k]));
            cd.lo[k] = (float)(lo[k] - pad);
            cd.hi[k] = (float)(hi[k] + pad);
        }
    }
    for (int j = tid; j < a.n_inst; j += blockDim.x) {
        Instance &in = a.inst[j];
        if (in.segment < 0) continue;
        const SegDev &sg = a.segs[in.segment];
        const float *p = a.params + 6 * in.segment;
        double tx = p[0], ty = p[1], R = p[2];
        double s = R / sg.r0;
        D3 e1 = dload(sg.e1), e2 = dload(sg.e2);
        D3 cols[3], dcx[3], dcy[3];
        for (int c = 0; c < 3; ++c) {
            D3 ej = D3{c == 0 ? 1.0 : 0.0, c == 1 ? 1.0 : 0.0, c == 2 ? 1.0 : 0.0};
            D3 r1 = drot(e1, tx, ej);
            cols[c] = drot(e2, ty, r1);
            dcx[c] = drot(e2, ty, dcross(e1, r1));
            dcy[c] = dcross(e2, cols[c]);
        }
        for (int r = 0; r < 3; ++r)
            for (int c = 0; c < 3; ++c) {
                double rc = r == 0 ? cols[c].x : (r == 1 ? cols[c].y : cols[c].z);
                in.rot[3 * r + c] = (float)rc;
                in.m[3 * c + r] = (float)(rc / s);   // (1/s) Rot^T
                in.drx[3 * r + c] = (float)(r == 0 ? dcx[c].x : (r == 1 ? dcx[c].y : dcx[c].z));
                in.dry[3 * r + c] = (float)(r == 0 ? dcy[c].x : (r == 1 ? dcy[c].y : dcy[c].z));
            }
        D3 org = dadd(dload(sg.pivot), D3{p[3], p[4], p[5]});
        store3(in.org, org);
        in.scale = (float)s;
        in.inv_r0 = (float)(1.0 / sg.r0);
        double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
        for (int c = 0; c < 8; ++c) {
            D3 l = D3{(c & 1) ? in.loc_hi[0] : in.loc_lo[0], (c & 2) ? in.loc_hi[1] : in.loc_lo[1],
                      (c & 4) ? in.loc_hi[2] : in.loc_lo[2]};
            D3 w = dadd(org, dmul(dadd(dadd(dmul(cols[0], l.x), dmul(cols[1], l.y)), dmul(cols[2], l.z)), s));
            double q[3] = {w.x, w.y, w.z};
            for (int k = 0; k < 3; ++k) {
                lo[k] = fmin(lo[k], q[k]);
                hi[k] = fmax(hi[k], q[k]);
            }
        }
        for (int k = 0; k < 3; ++k) {
            double pad = 1e-2 + 1e-6 * fmax(fabs(lo[k]), fabs(hi[k]));
            in.lo[k] = (float)(lo[k] - pad);
            in.hi[k] = (float)(hi[k] + pad);
        }
    }
    __syncthreads();
    for (int k = tid; k < a.n_sheets; k += blockDim.x) {
        const Instance &in = a.inst[a.sheet_inst[k]];
        bool holds = true;
        if (in.segment >= 0) {
            holds = in.scale > 0.0f && in.scale <= kSheetSlack;
            for (int q = 0; q < 3; ++q)
                holds = holds && fabsf(in.lo[q]) <= kSheetSlack * a.extent && fabsf(in.hi[q]) <= kSheetSlack * a.extent;
        }
        a.sheets[k].min_cos = holds ? a.sheets[k].rule : 2.0f;
    }
    // Refit: each child's box from what it holds, all at once, until none
    // changes, which takes a pass per level (one thread going through the nodes
    // from the back took 23 us on 33 instances, this 8).
    for (bool changed = true; changed;) {
        changed = false;
        for (int i0 = 0; i0 < 4 * a.n_top; i0 += blockDim.x) {
            const int i = (i0 + tid) / 4, k = (i0 + tid) % 4;
            const uint32_t c = i < a.n_top ? a.nodes[i].child[k] : kEmpty;
            float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
            if (c == kEmpty) {
            } else if (c & kLeafBit) {
                const Instance &in = a.inst[c & ~(kLeafBit | kInstBit)];
                for (int q = 0; q < 3; ++q) {
                    lo[q] = in.lo[q];
                    hi[q] = in.hi[q];
                }
            } else {
                const Node4 &ch = a.nodes[c];
                for (int m = 0; m < 4; ++m) {
                    if (ch.child[m] == kEmpty) continue;
                    lo[0] = fminf(lo[0], ch.lox[m]);
                    lo[1] = fminf(lo[1], ch.loy[m]);
                    lo[2] = fminf(lo[2], ch.loz[m]);
                    hi[0] = fmaxf(hi[0], ch.hix[m]);
                    hi[1] = fmaxf(hi[1], ch.hiy[m]);
                    hi[2] = fmaxf(hi[2], ch.hiz[m]);
                }
            }
            __syncthreads();   // all read before any is written
            if (c != kEmpty) {
                Node4 &nd = a.nodes[i];
                auto set = [&](float &x, float y) {
                    changed |= __float_as_uint(x) != __float_as_uint(y);
                    x = y;
                };
                set(nd.lox[k], lo[0]);
                set(nd.loy[k], lo[1]);
                set(nd.loz[k], lo[2]);
                set(nd.hix[k], hi[0]);
                set(nd.hiy[k], hi[1]);
                set(nd.hiz[k], hi[2]);
            }
            __syncthreads();
        }
        changed = __syncthreads_or(changed);
    }
    for (int i = tid; i < 3 * a.n_top; i += blockDim.x) write_lane_axis(a.nodes[i / 3], a.lane_nodes[i / 3], i % 3);
}

hipError_t launch_prepare(const PrepareArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(prepare_kernel, dim3(1), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.n_nodes == 0) return e;
    hipLaunchKernelGGL(lane_nodes_kernel, dim3((a.n_nodes + 255) / 256), dim3(256), 0, st, a.nodes, a.lane_nodes,
                       a.n_nodes);
    return hipGetLastError();
}

// Graph-safe zeroing of small counters (no memset node in captured graphs).
__global__ void fill_u64_kernel(unsigned long long *p, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

hipError_t launch_fill_u64(unsigned long long *p, int n, hipStream_t st) {
    hipLaunchKernelGGL(fill_u64_kernel, dim3((n + 63) / 64), dim3(64), 0, st, p, n);
    return hipGetLastError();
}

// Two ranges of 32-bit words, a word a thread: 173 KB and 56 bytes take 1.7 us,
// a launch for each or one launch of a block a range 3.4.
__global__ __launch_bounds__(256) void clear_words_kernel(uint32_t *a, uint64_t n_a, uint32_t *b, uint64_t n_b) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_a) a[i] = 0u;
    else if (i - n_a < n_b) b[i - n_a] = 0u;
}

hipError_t launch_clear_words(uint32_t *a, uint64_t n_a, uint32_t *b, uint64_t n_b, hipStream_t st) {
    const uint64_t blocks = (n_a + n_b + 255) / 256;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, n_a, b, n_b);
    return hipGetLastError();
}

// ---------------------------------------------------------------- per-photon body

using OutputsRef = const RICH_CONST DevOutputs &;
__device__ __forceinline__ OutputsRef outputs_arg() { return kernel_arg<DevOutputs>(kThirdArg); }

// Per-photon output store.  kStream: a non-temporal store, which L2 keeps
// for a short time only, so that a large batch's gigabytes of outputs do
// not push the scene out of L2 (the batch kernel; the forward kernel writes
// each line in several passes and keeps them in L2 to merge).
template <bool kStream, class T>
__device__ __forceinline__ void put(T *p, T v) {
    if constexpr (kStream) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Trace photon g (output slot i), write its results and return its fate (-1
// for inactive lanes).  Every lane of the wave must call this together: the
// hit list uses wave-wide ballots.
// kTrace, kPrefilter: what the kernel is built for (see propagate).  kStream:
// the outputs stream past L2 (batches).  rejected: the pre-filter's decision
// for this photon is already known to be a rejection (the forward sort took
// it), so it is neither generated nor tested again.
template <TraceKind kTrace, bool kPrefilter, bool kStream>
__device__ __forceinline__ int photon_job(SceneRef S, SourceRef src, OutputsRef outputs, bool active, uint64_t i,
                                          uint64_t g, uint64_t seed, uint32_t *stk, int track = -1,
                                          bool rejected = false) {
    PathEnd end;
    end.fate = -1;
    end.pixel = -1;
    if (active) {
        if (kPrefilter && rejected) {
            end.fate = kPrefiltered;
        } else {
            Photon ph = make_photon(fresh(src), seed, g, i, true, track);
            NoRecord rec;
            if (!kPrefilter || prefilter_keep(fresh(S), fresh(src), ph, seed, g)) {
                propagate<kTrace, !kPrefilter>(S, ph, seed, g, stk, end, rec);
            } else {
                end.fate = kPrefiltered;
            }
        }
    }
    OutputsRef out = fresh(outputs);
    if (active) {
        bool on_det = end.fate == kDetected || end.fate == kQeRejected;
        const float nan = __builtin_nanf("");
        if (out.fate) put<kStream>(out.fate + i, (uint8_t)end.fate);
        if (out.pixel) put<kStream>(out.pixel + i, on_det ? end.pixel : -1);
        if (out.hit_xyz) {
            float *p = out.hit_xyz + 3 * i;
            put<kStream>(p, on_det ? end.P.x : nan);
            put<kStream>(p + 1, on_det ? end.P.y : nan);
            put<kStream>(p + 2, on_det ? end.P.z : nan);
        }
        if (out.hit_uv) {
            float *p = out.hit_uv + 2 * i;
            put<kStream>(p, on_det ? end.u : nan);
            put<kStream>(p + 1, on_det ? end.v : nan);
        }
        if (out.hit_time) put<kStream>(out.hit_time + i, on_det ? end.time : nan);
        if (out.histogram && end.fate == kDetected) atomicAdd(out.histogram + end.pixel, 1u);
    }
    if (out.hit_list) {
        const int lane = __lane_id();
        unsigned long long m = __ballot(end.fate == kDetected);
        if (m) {
            int leader = __ffsll((long long)m) - 1;
            unsigned long long base = 0;
            if (lane == leader) base = atomicAdd(out.hit_count, (unsigned long long)__popcll(m));
            uint32_t lo = __shfl((uint32_t)base, leader), hi = __shfl((uint32_t)(base >> 32), leader);
            base = ((unsigned long long)hi << 32) | lo;
            if (end.fate == kDetected) {
                unsigned long long slot = base + __popcll(m & ((1ull << lane) - 1ull));
                if (slot < out.hit_capacity) {
                    char *rec = reinterpret_cast<char *>(out.hit_list) + 24 * slot;
                    *reinterpret_cast<uint64_t *>(rec) = g;
                    *reinterpret_cast<int32_t *>(rec + 8) = end.pixel;
                    float *xyz = reinterpret_cast<float *>(rec + 12);
                    xyz[0] = end.P.x;
                    xyz[1] = end.P.y;
                    xyz[2] = end.P.z;
                } else {
                    atomicOr(S.status, 1u);  // RICH_FLAG_HITLIST_OVERFLOW
                }
            }
        }
    }
    return end.fate;
}

// Per-wave fate tally: ballots give wave-uniform counts, so no atomics here.
__device__ __forceinline__ void tally_wave(uint32_t cnt[kFates], int fate) {
#pragma unroll
    for (int f = 0; f < kFates; ++f)
        cnt[f] += (uint32_t)__builtin_amdgcn_readfirstlane((int)__popcll(__ballot(fate == f)));
}

// Add the waves' tallies, summed over the block in LDS, to the caller's fate
// counters (if any): at most kFates additions a block, which nothing waits
// for.  Gathered in slots that the last block to finish folded, each block had
// to order its additions before its arrival (__threadfence, which on eight
// XCDs writes a whole L2 back): 1e6 photons 125 -> 60 us in the analytic
// geometry, 188 -> 159 on 210,082 triangles, 300,000 there 103 -> 76, 1,000
// 12.6 -> 11.1.  Called by every thread.
__device__ __forceinline__ void flush_tally(OutputsRef out, const uint32_t cnt[kFates], uint32_t *lds_cnt) {
    const int lane = __lane_id(), wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    if (lane == 0)
        for (int f = 0; f < kFates; ++f) lds_cnt[kFates * wave + f] = cnt[f];
    __syncthreads();
    if (wave != 0 || lane >= kFates || !out.fate_counts) return;
    unsigned long long sum = 0;
    for (int w = 0; w < waves; ++w) sum += lds_cnt[kFates * w + lane];
    if (sum) atomicAdd(out.fate_counts + lane, sum);
}

// ---------------------------------------------------------------- forward: sorted order or grid-stride

constexpr int kForwardBlock = 256;

// Regrouping bin of photon g among `bins` bins: its cone azimuth's uniform
// (word 0 of its first Philox block) in bins 0..bins-2, and the last bin
// for photons the pre-filter rejects (so kept photons fill waves densely).
// With s_bits, the azimuth in bins / 2^s_bits steps and within each the
// emission point (word 2) in 2^s_bits.
template <bool kPrefilter>
__device__ __forceinline__ uint32_t regroup_bin(SceneRef S, SourceRef src, uint64_t seed, uint64_t g, uint32_t bins,
                                                int s_bits = 0) {
    const uint32_t top = bins - 1u;
    work(kWorkSortKeys);
    const uint4 w = photon_block(seed, g, 0);
    if (kPrefilter && src.n_disp == 0 && src.kind != 2) {
        // the wavelength alone decides (with dispersion or explicit photons
        // the rejected ones are not set apart)
        Photon ph;
        ph.lambda = rcp(fmaf(-u24(w.y), src.inv_span, src.inv_lmin));
        if (!prefilter_keep(S, src, ph, seed, g)) return top;
    }
    if (src.kind == 2) return 0u;
    uint32_t b = (uint32_t)(((uint64_t)w.x * bins) >> 32);
    if (s_bits > 0) {
        // the emission point within the azimuth bin, to and fro
        const uint32_t steps = 1u << s_bits, az = b >> s_bits, q = w.z >> (32 - s_bits);
        b = (az << s_bits) | ((az & 1u) ? steps - 1u - q : q);
    }
    return b < top ? b : top - 1u;
}

// Photon id of processing position v of a batch: v itself in id order, else
// the photon v - order_off[k] of the k-th track in processing order, whose
// index goes to `track` (-1 when unknown: make_photon then searches).  When n
// is not the tracks' photon total the order is not used (ids beyond it are
// drawn from the last track, as in id order).
__device__ __forceinline__ uint64_t batch_photon_id(SourceRef src, uint64_t v, uint64_t n, int &track) {
    track = -1;
    if (!src.order) return v;
    const RICH_CONST uint64_t *oo = (const RICH_CONST uint64_t *)src.order_off;
    if (oo[src.n_tracks] != n || v >= n) return v;
    const int k = find_track_wave(src.order_off, src.n_tracks, v);
    const int t = src.order[k];
    const uint64_t g = src.offsets[t] + (v - oo[k]);
    if (g >= n) return v;   // offsets that do not rise (bad input) never send a write out of range
    track = t;
    return g;
}

// Photons of a forward launch are traced in an order sorted by cone azimuth
// within windows of kWindow ids: sort_photons_kernel counting-sorts each
// window by the azimuth's uniform (word 0 of the photon's first Philox block;
// the photons the pre-filter rejects last) into kBins bins, and the trace
// kernel's waves then take 64 neighbours in that order, whose rays meet the
// same parts of the scene.  Every photon keeps its id and random numbers and
// writes its outputs at its id; only the lane that traces it changes.  Wider
// windows give each wave closer directions but keep fewer CUs sorting: large
// launches sort windows of 32,768 ids, or if pre-filtered (their trace is
// short) of 8192; smaller ones, bound by the latency of what they do in turn,
// windows of 1024 (limits and times at launch_forward).
template <int kWindow, int kBins, int kThreads>
struct SortShape {
    static constexpr int window = kWindow, bins = kBins, threads = kThreads;
    static_assert(kWindow % kThreads == 0 && kBins % kThreads == 0 && kWindow <= 65536 &&
                      kSortedChunk % kWindow == 0 && kSortedChunk <= (uint64_t(1) << 31) && kThreads % 64 == 0 &&
                      kThreads >= kBatchCounters,   // one block zeroes every claim counter
                  "sort shape");
};
using WideSort = SortShape<32768, 2048, 1024>;
using NarrowSort = SortShape<8192, 1024, 512>;
using SmallSort = SortShape<1024, 512, 512>;
using BatchSort = SortShape<4096, 1024, 1024>;
constexpr uint64_t kWideMin = uint64_t(1) << 18;   // photons from which wide windows are sorted

// The photons' bins by themselves, where sorted's windows will go.  Drawing
// them (Philox) is most of the sort, and with fewer windows than CUs the rest
// of the chip would watch: such launches of wide windows draw them in a launch
// of its own.  210,082 triangles: 300,000 photons 121 -> 111 us, 2e6 280 ->
// 272, 4e6 the same.
__global__ __launch_bounds__(256) void sort_bins_kernel(DevScene, DevSource, uint64_t n, uint64_t first, uint64_t seed,
                                                        uint32_t *sorted, uint32_t bins, int s_bits) {
    SceneRef S = scene_arg();
    SourceRef src = source_arg();
    const uint64_t l = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (l < n) sorted[l] = regroup_bin<false>(S, src, seed, first + l, bins, s_bits);
}

// Bin of the photon at position v of a batch: its azimuth in a quarter of the
// bins, the quarter by its track's place after first_place, that of the
// window's first position (a window of long tracks holds one track or two, so
// the place is found by steps from there: with a binary search for each photon
// the sort of 1e7 took 114 us, with this 53).  in_order: the processing
// order holds (see batch_photon_id).
__device__ __forceinline__ uint32_t batch_bin(SourceRef src, uint64_t seed, uint64_t v, int first_place, bool in_order,
                                              uint64_t total, uint32_t bins) {
    const uint64_t *off = in_order ? src.order_off : src.offsets;
    int place = first_place;
    for (int k = 0; k < 3; ++k) place += place + 1 < src.n_tracks && v >= off[place + 1] ? 1 : 0;
    const int quarter = place - first_place;
    uint64_t g = v;
    if (in_order) {
        if (quarter == 3) place = find_track(off, src.n_tracks, v);
        const int t = src.order[place];
        g = src.offsets[t] + (v - off[place]);
        if (g >= total) g = v;
    }
    work(kWorkSortKeys);
    const uint32_t az = (uint32_t)(((uint64_t)photon_block(seed, g, 0).x * (bins / 4)) >> 32);
    return (uint32_t)quarter * (bins / 4) + az;
}

// The octahedral map of the unit sphere onto [-1, 1]^2 (the lower hemisphere
// folded outwards).
__device__ __forceinline__ void direction_map(float x, float y, float z, float &u, float &v) {
    const float s = fabsf(x) + fabsf(y) + fabsf(z);
    u = s > 0.0f ? x / s : 0.0f;
    v = s > 0.0f ? y / s : 0.0f;
    if (z < 0.0f) {
        const float fu = (1.0f - fabsf(v)) * copysignf(1.0f, u), fv = (1.0f - fabsf(u)) * copysignf(1.0f, v);
        u = fu;
        v = fv;
    }
}

// The bits of x (at most 8) at the even places.
__device__ __forceinline__ uint32_t spread_bits(uint32_t x) {
    x = (x | x << 4) & 0x0F0Fu;
    x = (x | x << 2) & 0x3333u;
    return (x | x << 1) & 0x5555u;
}

// Bins of a window of photon arrays, from their packed direction maps (16 bits
// each way) in key[]: a grid over the window's own range of directions, in
// Morton order.  Every thread of the block calls it.
template <int kBins, int kPer>
__device__ __forceinline__ void array_bins(uint32_t (&key)[kPer], uint32_t m, uint32_t threads, uint32_t *range) {
    const int lane = threadIdx.x & 63;
    uint32_t lo_u = 0xFFFFu, hi_u = 0, lo_v = 0xFFFFu, hi_v = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if ((uint32_t)j * threads + threadIdx.x >= m) continue;
        lo_u = min(lo_u, key[j] & 0xFFFFu);
        hi_u = max(hi_u, key[j] & 0xFFFFu);
        lo_v = min(lo_v, key[j] >> 16);
        hi_v = max(hi_v, key[j] >> 16);
    }
    for (int d = 1; d < 64; d <<= 1) {
        lo_u = min(lo_u, (uint32_t)__shfl_xor((int)lo_u, d));
        hi_u = max(hi_u, (uint32_t)__shfl_xor((int)hi_u, d));
        lo_v = min(lo_v, (uint32_t)__shfl_xor((int)lo_v, d));
        hi_v = max(hi_v, (uint32_t)__shfl_xor((int)hi_v, d));
    }
    if (lane == 0) {
        atomicMin(range + 0, lo_u);
        atomicMax(range + 1, hi_u);
        atomicMin(range + 2, lo_v);
        atomicMax(range + 3, hi_v);
    }
    __syncthreads();
    constexpr int bits = __builtin_ctz(kBins), u_bits = (bits + 1) / 2, v_bits = bits / 2;
    const uint32_t u0 = range[0], v0 = range[2];
    const float su = (float)(1 << u_bits) / (float)(range[1] - u0 + 1u), sv = (float)(1 << v_bits) / (float)(range[3] - v0 + 1u);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t iu = min((uint32_t)((float)((key[j] & 0xFFFFu) - u0) * su), (1u << u_bits) - 1u);
        const uint32_t iv = min((uint32_t)((float)((key[j] >> 16) - v0) * sv), (1u << v_bits) - 1u);
        key[j] = spread_bits(iu) | spread_bits(iv) << 1;
    }
}

// kBatch: the positions first.. of a batch of `total` photons.  kArrays: photon
// arrays, by direction.
template <class Shape, bool kPrefilter, bool kBinned, bool kBatch = false, bool kArrays = false>
__global__ __launch_bounds__(Shape::threads) __attribute__((amdgpu_waves_per_eu(8))) void sort_photons_kernel(
    DevScene, DevSource, uint64_t n, uint64_t first, uint64_t seed, uint32_t *sorted, unsigned long long *counter,
    int s_bits, uint64_t total) {
    SceneRef S = scene_arg();
    SourceRef src = source_arg();
    constexpr int kSortWindow = Shape::window, kSortBins = Shape::bins, kSortThreads = Shape::threads;
    __shared__ uint32_t bins[kSortBins];
    // the trace kernel's claim counters start at zero (it runs next on the stream)
    if (blockIdx.x == 0 && threadIdx.x < kBatchCounters) counter[threadIdx.x] = 0;
    __shared__ uint16_t slot[kSortWindow];
    __shared__ uint32_t wave_sum[kSortThreads / 64];
    constexpr int per = kSortWindow / kSortThreads;
    const uint64_t w0 = (uint64_t)blockIdx.x * kSortWindow;
    const uint32_t m = (uint32_t)(n - w0 < (uint64_t)kSortWindow ? n - w0 : (uint64_t)kSortWindow);
    for (int q = threadIdx.x; q < kSortBins; q += kSortThreads) bins[q] = 0;
    __shared__ uint32_t range[kArrays ? 4 : 1];
    if (kArrays && threadIdx.x < 4) range[threadIdx.x] = threadIdx.x & 1 ? 0u : 0xFFFFu;
    __syncthreads();
    const bool in_order = kBatch && src.order && src.order_off[src.n_tracks] == total;
    const int first_place =
        kBatch ? find_track_wave(in_order ? src.order_off : src.offsets, src.n_tracks, first + w0) : 0;
    // bin and rank within the bin (16 bits each) of this thread's photons
    uint32_t key[per];
    if (kBinned) {
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const uint32_t l = (uint32_t)(j * kSortThreads) + threadIdx.x;
            key[j] = l < m ? sorted[w0 + l] : 0u;
        }
    }
    if constexpr (kArrays) {
#pragma unroll
        for (int j = 0; j < per; ++j) {
            const uint32_t l = (uint32_t)(j * kSortThreads) + threadIdx.x;
            key[j] = 0u;
            if (l < m) {
                const V3 d = ld3(src.ex_d + 3 * (w0 + l));
                float u, v;
                direction_map(d.x, d.y, d.z, u, v);
                const uint32_t iu = (uint32_t)fminf(fmaxf(fmaf(u, 32767.0f, 32767.5f), 0.0f), 65535.0f);
                const uint32_t iv = (uint32_t)fminf(fmaxf(fmaf(v, 32767.0f, 32767.5f), 0.0f), 65535.0f);
                key[j] = iu | iv << 16;
            }
        }
        array_bins<kSortBins>(key, m, kSortThreads, range);
    }
#pragma unroll
    for (int j = 0; j < per; ++j) {
        const uint32_t l = (uint32_t)(j * kSortThreads) + threadIdx.x;
        if (l < m) {
            const uint32_t b =
                kBatch    ? batch_bin(src, seed, first + w0 + l, first_place, in_order, total, kSortBins)
                : kBinned || kArrays ? key[j]
                          : regroup_bin<kPrefilter>(S, src, seed, first + w0 + l, kSortBins, s_bits);
            uint32_t rank = 0;
            // most photons of a pre-filtered window share the last bin: one
            // addition a wave (30,000 photons 50 -> 47 us; windows of more photons
            // per thread have no registers to spare for it)
            constexpr bool kCountTop = kPrefilter && per <= 4;
            if (kCountTop) {
                const unsigned long long m = __ballot(b == kSortBins - 1);
                if (b == kSortBins - 1) {
                    const int leader = __ffsll((long long)m) - 1;
                    if ((int)(threadIdx.x & 63) == leader) rank = atomicAdd(bins + b, (uint32_t)__popcll(m));
                    rank = (uint32_t)__builtin_amdgcn_readlane((int)rank, leader) +
                           (uint32_t)__popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
                }
            }
            if (!kCountTop || b != kSortBins - 1) rank = atomicAdd(bins + b, 1u);
            key[j] = b | (rank << 16);
        }
    }
    __syncthreads();
    // exclusive scan of the bin counts: per thread, then per wave, then across waves
    constexpr int bpt = kSortBins / kSortThreads;
    uint32_t c[bpt], sum = 0;
#pragma unroll
    for (int q = 0; q < bpt; ++q) {
        c[q] = bins[bpt * threadIdx.x + q];
        sum += c[q];
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = sum;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
    for (int q = 0; q < bpt; ++q) {
        bins[bpt * threadIdx.x + q] = run;
        run += c[q];
    }
    __syncthreads();
    // the thread's photons again: kept from above they would cost 64 registers
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
#pragma unroll
    for (int j = 0; j < per; ++j) {
        const uint32_t l = (uint32_t)(j * kSortThreads) + tid;
        if (l < m) slot[bins[key[j] & 0xFFFFu] + (key[j] >> 16)] = (uint16_t)l;
    }
    // photons the pre-filter rejects fill the window's last bin (when the
    // wavelength alone decides): their sorted entries carry the top bit, and
    // the trace writes their fate without generating them again
    const uint32_t rejected_from = kPrefilter && src.n_disp == 0 && src.kind != 2 ? bins[kSortBins - 1] : m;
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < m; q += kSortThreads)
        sorted[w0 + q] = (uint32_t)(w0 + slot[q]) | (q >= rejected_from ? 0x80000000u : 0u);
}

// How a forward launch hands photons to lanes: a grid-stride loop over the
// ids (small analytic launches and photon arrays: no extra launch before it),
// or waves claiming 64 positions at a time, of the sorted order (meshed scenes,
// pre-filter), of the ids themselves (large analytic launches) or of the
// sorted processing order of a batch.
enum ForwardMode { kGridStride = 0, kSortedClaims = 1, kIdClaims = 2, kBatchClaims = 3 };

// Scenes without meshes need neither the traversal's registers nor its stacks:
// 63-74 vector registers and six or seven waves per SIMD instead of 99 and
// four.  With meshes the kernel is held to 128 registers for four, or where
// the stacks in LDS are short to 96 for five.
template <TraceKind kTrace, bool kPrefilter, ForwardMode kMode>
__global__ __launch_bounds__(kForwardBlock) __attribute__((amdgpu_waves_per_eu(kTrace >= kMeshWave ? 5 : 4))) void
forward_kernel(DevScene, DevSource, DevOutputs, uint64_t n, uint64_t first, uint64_t seed, const uint32_t *sorted,
               unsigned long long *counter, uint64_t total) {
    extern __shared__ uint32_t lds_stack[];
    SceneRef S = scene_arg();
    SourceRef src = source_arg();
    OutputsRef out = outputs_arg();
    uint32_t cnt[kFates] = {0, 0, 0, 0, 0, 0, 0};
    auto job = [&](bool active, uint64_t i, bool rejected) {
        const int fate = photon_job<kTrace, kPrefilter, false>(S, src, out, active, i, first + i, seed,
                                                              lane_stack<kTrace>(lds_stack), -1, rejected);
        if (out.fate_counts) tally_wave(cnt, fate);
    };
    if (kMode == kBatchClaims && first == 0 && blockIdx.x == 0 && threadIdx.x == 0 &&
        src.offsets[src.n_tracks] != total)
        atomicOr(S.status, 8u);   // RICH_FLAG_BATCH_SIZE: n is not the photon total of the tracks
    if constexpr (kMode == kGridStride) {
        const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
        for (uint64_t base = (uint64_t)blockIdx.x * blockDim.x; base < n; base += stride)
            job(base + threadIdx.x < n, base + threadIdx.x, false);
    } else {
        // The positions are split into one contiguous range per XCD
        // (workgroups are dealt to the eight XCDs round robin), so that an
        // XCD's photons in flight are neighbours in the sorted order and
        // their outputs lie in few windows.  Each wave claims the next 64
        // positions of its XCD's range from that range's counter (its own
        // cache line), so the waves of a CU trace neighbouring directions at
        // once, a wave that drew cheap photons takes more, and the XCD's
        // waves finish together.
        const uint32_t parts = gridDim.x >= 8 ? 8u : 1u;
        const uint32_t x = blockIdx.x % parts;
        const uint64_t span = (n + (uint64_t)parts * 64 - 1) / ((uint64_t)parts * 64) * 64;
        const uint64_t lo = (uint64_t)x * span, hi = lo + span < n ? lo + span : n;
        unsigned long long *ctr = counter + kCounterStride * x;
        const int lane = threadIdx.x & 63;
        while (true) {
            unsigned long long c = 0;
            if (lane == 0) c = atomicAdd(ctr, 64ull);
            const uint32_t c_lo = __shfl((uint32_t)c, 0), c_hi = __shfl((uint32_t)(c >> 32), 0);
            const uint64_t k = lo + (((uint64_t)c_hi << 32) | c_lo) + (uint64_t)lane;
            if (k - lane >= hi) break;
            const bool active = k < hi;
            if constexpr (kMode == kIdClaims) {
                job(active, k, false);
            } else if constexpr (kMode == kBatchClaims) {
                int track = -1;
                const uint64_t g = active ? batch_photon_id(src, first + sorted[k], total, track) : 0;
                const int fate = photon_job<kTrace, kPrefilter, false>(S, src, out, active, g, g, seed,
                                                                      lane_stack<kTrace>(lds_stack), track);
                if (out.fate_counts) tally_wave(cnt, fate);
            } else {
                // entries with the top bit set are photons the sort already
                // saw the pre-filter reject
                const uint32_t e = active ? sorted[k] : 0u;
                job(active, e & 0x7FFFFFFFu, (e >> 31) != 0u);
            }
        }
    }
    if (out.fate_counts) flush_tally(out, cnt, lds_stack + kForwardBlock / 64 * stack_words(kTrace));
}

// Photon arrays on meshes of at least this many are sorted by direction, if
// there is an order buffer: in windows of 4096 over a grid of the window's own
// directions.  Arrays of 64 tracks in emission order, 210,082 triangles: 5e5
// photons 126 -> 118 us, 1e6 205 -> 179, 4e6 725 -> 554 (262,144: 75 / 80);
// random directions 1e6 241 -> 219, 4e6 897 -> 732.  Windows of 8192 measured
// the same, of 32,768 (too few for the chip) 205 at 1e6.
bool arrays_sorted(const DevScene &S, const DevSource &src, uint64_t n) {
    return S.has_mesh && src.kind == 2 && !src.prefilter && n >= uint64_t(1) << 19;
}

bool forward_sorted(const DevScene &S, const DevSource &src) {
    return (S.has_mesh && src.kind != 2) || src.prefilter;
}

// Unsorted launches of at least this many photons claim their ids (after a
// fill launch that zeroes the counters); smaller ones are launch bound, or
// short of photons to share out: analytic 3e6 146 / 145 us, 8e6 424 -> 354.
constexpr uint64_t kIdClaimsMin = uint64_t(1) << 22;

// Steps of the emission point in the sort's bins (as a power of two): a track
// of length L shifts a photon's path sideways by up to L sin(theta), its
// azimuth by up to 2 pi D sin(theta) at the surfaces a distance D away (taken
// as the scene's extent), and a wave's photons are closest together when a bin
// is as long as it is wide.
static int s_bits(const DevSource &src, const DevScene &S, int bins) {
    const float extent = S.sheet_reach;
    if (src.kind != 0 || !(src.length > 0.0f) || !(extent > 0.0f)) return 0;
    int bits = 0;
    while (bits < 5 && 6.2831853f * extent * (float)(1 << (2 * bits)) < (float)bins * src.length) ++bits;
    return bits;
}

// Whether a sorted launch's rays are close enough together for the wave phase
// to pay (see traverse): 64 neighbours of a full window of 32,768 sorted
// photons from one point or a short track, or with many windows in flight
// from a long one.  Lane phase against wave phase, microseconds, 210,082 and
// 2,009,708 triangles: point 300,000 photons 80 / 75 and 109 / 104, 1e6
// 168 / 141 and 225 / 207, 4e6 521 / 417 and 704 / 602; 1 m track 600,000
// 118 / 127 and 183 / 161, 1e6 170 / 173 and 262 / 223, 4e6 565 / 550 and
// 845 / 691; pre-filtered launches (one photon in nine is traced) were up to
// 20 % slower with it.
static bool wave_walk(const DevSource &src, const DevScene &S, uint64_t n) {
    if (src.kind != 0 || src.prefilter || n < kWideMin) return false;
    return s_bits(src, S, WideSort::bins) <= 2 || n >= uint64_t(1) << 20;
}

hipError_t launch_forward(const DevScene &S, const DevSource &src, const DevOutputs &out, uint64_t n, uint64_t first,
                          uint64_t seed, int n_cu, uint32_t *sorted, unsigned long long *counter, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const bool arrays = sorted && arrays_sorted(S, src, n);
    const bool sort = forward_sorted(S, src) || arrays;
    if (!counter || (sort && !sorted)) return hipErrorInvalidValue;
    const TraceKind kind =
        !S.has_mesh ? kAnalytic : (!sort || arrays ? kMeshLoose : (wave_walk(src, S, n) ? kMeshWave : kMeshLane));
    const size_t lds = (size_t)(kForwardBlock / 64) * (stack_words(kind) + kFates) * sizeof(uint32_t);
    // One block per resident slot (registers and LDS decide how many fit on
    // a CU: the runtime's occupancy query), each looping over its photons; a
    // grid of more blocks runs in waves of blocks, and a partial last wave
    // leaves most CUs idle.  The grid-stride form takes two blocks per slot,
    // which measured faster there.  A claiming grid is a multiple of the
    // eight XCDs, each XCD's blocks claiming from its own counter: the next
    // one above the photons' blocks, so that no wave of a small launch has a
    // second pass (20,000 photons on 80 blocks 69 -> 50 us against 72).
    using Kernel = void (*)(DevScene, DevSource, DevOutputs, uint64_t, uint64_t, uint64_t, const uint32_t *,
                            unsigned long long *, uint64_t);
    static const Kernel kernels[4][2][3] = {
        {{forward_kernel<kAnalytic, false, kGridStride>, nullptr, forward_kernel<kAnalytic, false, kIdClaims>},
         {nullptr, forward_kernel<kAnalytic, true, kSortedClaims>, nullptr}},
        {{nullptr, forward_kernel<kMeshLane, false, kSortedClaims>, nullptr},
         {nullptr, forward_kernel<kMeshLane, true, kSortedClaims>, nullptr}},
        {{nullptr, forward_kernel<kMeshWave, false, kSortedClaims>, nullptr}, {nullptr, nullptr, nullptr}},
        {{forward_kernel<kMeshLoose, false, kGridStride>, forward_kernel<kMeshLoose, false, kSortedClaims>,
          forward_kernel<kMeshLoose, false, kIdClaims>},
         {nullptr, nullptr, nullptr}}};
    static std::atomic<int> resident[4][2][3];   // blocks of each that a CU holds (0: not asked yet)
    const int pre = src.prefilter ? 1 : 0;
    // sorted launches go in chunks of at most kSortedChunk photons (the order
    // buffer's size); the outputs of a chunk start at its first photon
    const uint64_t step = sort ? kSortedChunk : n;
    for (uint64_t off = 0; off < n; off += step) {
        const uint64_t m = n - off < step ? n - off : step;
        const int mode = sort ? kSortedClaims : (m >= kIdClaimsMin ? kIdClaims : kGridStride);
        const Kernel kernel = kernels[kind][pre][mode];
        int per_cu = resident[kind][pre][mode].load(std::memory_order_relaxed);
        if (per_cu == 0) {
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kernel, kForwardBlock, lds) !=
                    hipSuccess ||
                per_cu < 1)
                per_cu = 4;
            resident[kind][pre][mode].store(per_cu, std::memory_order_relaxed);
        }
        DevSource cs = src;
        if (cs.kind == 2) {
            cs.ex_o += 3 * off;
            cs.ex_d += 3 * off;
            cs.ex_l += off;
        }
        DevOutputs o = out;   // every per-photon output is optional
        if (o.fate) o.fate += off;
        if (o.pixel) o.pixel += off;
        if (o.hit_xyz) o.hit_xyz += 3 * off;
        if (o.hit_uv) o.hit_uv += 2 * off;
        if (o.hit_time) o.hit_time += off;
        const uint64_t cap = (uint64_t)(n_cu > 0 ? n_cu : 256) * (uint64_t)per_cu * (mode == kGridStride ? 2u : 1u);
        uint64_t blocks = (m + kForwardBlock - 1) / kForwardBlock;
        if (mode != kGridStride && blocks >= 8) blocks = (blocks + 7) / 8 * 8;
        if (blocks > cap) blocks = cap;
        if (mode != kGridStride && blocks >= 8) blocks -= blocks % 8;
        hipError_t e = hipSuccess;
        if (mode == kSortedClaims) {
            // the sort also zeroes the claim counters
            auto launch = [&](auto shape, auto prefilter, auto binned, auto arrays) {
                using Shape = decltype(shape);
                hipLaunchKernelGGL((sort_photons_kernel<Shape, decltype(prefilter)::value, decltype(binned)::value,
                                                        false, decltype(arrays)::value>),
                                   dim3((unsigned)((m + Shape::window - 1) / Shape::window)), dim3(Shape::threads), 0,
                                   st, S, cs, m, first + off, seed, sorted, counter, s_bits(src, S, Shape::bins), n);
            };
            using Yes = std::true_type;
            using No = std::false_type;
            // Windows of 1024 against 32,768, 210,082 and 2,009,708 triangles: 20,011
            // photons 36 / 44 us and 59 / 76, 200,000 56 / 63 and 85 / 97, 300,000
            // 72 / 77 and 114 / 108.  Pre-filtered, against 8192: 30,000 photons
            // 40 / 44 and 63 / 68, 3e6 168 / 179 and 206 / 212, 1e7 444 / 441 and
            // 508 / 487.
            if (arrays) {
                launch(BatchSort(), No(), No(), Yes());
            } else if (src.prefilter) {
                if (m < uint64_t(1) << 22) launch(SmallSort(), Yes(), No(), No());
                else launch(NarrowSort(), Yes(), No(), No());
            } else if (m < kWideMin) {
                launch(SmallSort(), No(), No(), No());
            } else if ((m + WideSort::window - 1) / WideSort::window < (uint64_t)(n_cu > 0 ? n_cu : 256)) {
                hipLaunchKernelGGL(sort_bins_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, S, src, m,
                                   first + off, seed, sorted, (uint32_t)WideSort::bins, s_bits(src, S, WideSort::bins));
                launch(WideSort(), No(), Yes(), No());
            } else {
                launch(WideSort(), No(), No(), No());
            }
            e = hipGetLastError();
        } else if (mode == kIdClaims) {
            e = launch_fill_u64(counter, kBatchCounters, st);
        }
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kForwardBlock), lds, st, S, cs, o, m, first + off,
                           seed, (const uint32_t *)sorted, counter, n);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// Large batches of long tracks: the positions of the processing order (or the
// ids, of batches that have none) sorted by track and azimuth in windows of
// 4096, then traced with the wave phase.  Against the batch kernel, which
// regroups 256 photons at a time, on 210,082 and 2,009,708 triangles: 2,048
// tracks of 5,000 photons 1,409 -> 1,200 and 2,038 -> 1,485 us, 4,096 of 1,000
// 662 -> 576 and 907 -> 740, 2,500 of 900 385 -> 377 and 531 -> 478 (4,200 of
// 520 382 / 416 and 516 / 534); in id order 300 of 5,000 261 -> 236 and 371 ->
// 294, 250 of 2,100 121 / 121 and 165 -> 148 (80 of 3,000 72 / 87 and 98 / 110).
bool batch_sorted(const DevScene &S, const DevSource &src, uint64_t n) {
    if (!S.has_mesh || src.prefilter) return false;
    const uint64_t tracks = (uint64_t)src.n_tracks;
    return src.order ? n >= tracks * 768 : n >= tracks * 2048 && n >= uint64_t(1) << 19;
}

hipError_t launch_batch_sorted(const DevScene &S, const DevSource &src, const DevOutputs &out, uint64_t n,
                               uint64_t seed, int n_cu, uint32_t *sorted, unsigned long long *counter, hipStream_t st) {
    const auto kernel = forward_kernel<kMeshWave, false, kBatchClaims>;
    const size_t lds = (size_t)(kForwardBlock / 64) * (stack_words(kMeshWave) + kFates) * sizeof(uint32_t);
    static std::atomic<int> resident{0};
    int per_cu = resident.load(std::memory_order_relaxed);
    if (per_cu == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kernel, kForwardBlock, lds) !=
                hipSuccess ||
            per_cu < 1)
            per_cu = 4;
        resident.store(per_cu, std::memory_order_relaxed);
    }
    const unsigned blocks = (unsigned)((n_cu > 0 ? n_cu : 256) * per_cu) / 8 * 8;
    for (uint64_t off = 0; off < n; off += kSortedChunk) {
        const uint64_t m = n - off < kSortedChunk ? n - off : kSortedChunk;
        hipLaunchKernelGGL((sort_photons_kernel<BatchSort, false, false, true>),
                           dim3((unsigned)((m + BatchSort::window - 1) / BatchSort::window)), dim3(BatchSort::threads), 0,
                           st, S, src, m, off, seed, sorted, counter, 0, n);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kForwardBlock), lds, st, S, src, out, m, off, seed,
                           (const uint32_t *)sorted, counter, n);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- batch: processing order

constexpr int kOrderCellBits = 7;                        // cells per axis: 128
constexpr int kOrderCells = 1 << (2 * kOrderCellBits);   // 16384

// Cell of a direction: a 128 x 128 grid over its map, cells numbered in Morton
// order so that neighbouring numbers are neighbouring directions.
__device__ __forceinline__ uint32_t direction_cell(float x, float y, float z) {
    float u, v;
    direction_map(x, y, z, u, v);
    const int n = 1 << kOrderCellBits;
    const uint32_t iu = (uint32_t)min(max((int)((u + 1.0f) * 0.5f * n), 0), n - 1);
    const uint32_t iv = (uint32_t)min(max((int)((v + 1.0f) * 0.5f * n), 0), n - 1);
    uint32_t m = 0;
    for (int b = 0; b < kOrderCellBits; ++b) m |= (((iu >> b) & 1u) << (2 * b)) | (((iv >> b) & 1u) << (2 * b + 1));
    return m;
}

__global__ void order_cells_kernel(const float *tracks, int n_tracks, uint32_t *hist, uint32_t *cell_of) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tracks) return;
    const float4 *tr = reinterpret_cast<const float4 *>(tracks) + 2 * t;
    const float4 a = tr[0], b = tr[1];
    const uint32_t c = direction_cell(a.w, b.x, b.y);
    cell_of[t] = c;
    atomicAdd(hist + c, 1u);
}

// In place: counts per cell -> first position of each cell (one block).
__global__ __launch_bounds__(1024) void order_scan_cells_kernel(uint32_t *hist) {
    __shared__ uint32_t part[1024];
    constexpr int per = kOrderCells / 1024;
    const int t = threadIdx.x;
    uint32_t v[per], sum = 0;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        v[j] = hist[t * per + j];
        sum += v[j];
    }
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint32_t y = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += y;
        __syncthreads();
    }
    uint32_t run = part[t] - sum;
#pragma unroll
    for (int j = 0; j < per; ++j) {
        hist[t * per + j] = run;
        run += v[j];
    }
}

// Track t takes the next position of its cell (order within a cell is that of
// the atomics: it does not change any photon's result), and position pos goes
// to partition pos mod parts: order[] lists partition 0's tracks, then 1's, ...
// Each position's photon count goes beside it, into order_off (scanned next).
__global__ void order_scatter_kernel(const uint32_t *cell_of, const uint64_t *offsets, uint32_t *cursor,
                                     int n_tracks, int parts, int32_t *order, uint64_t *order_count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tracks) return;
    const uint32_t pos = atomicAdd(cursor + cell_of[t], 1u);
    const uint32_t c = pos % (uint32_t)parts, per = (uint32_t)n_tracks / (uint32_t)parts;
    const uint32_t rem = (uint32_t)n_tracks % (uint32_t)parts;
    const uint32_t q = c * per + min(c, rem) + pos / (uint32_t)parts;
    order[q] = t;
    order_count[q] = offsets[t + 1] - offsets[t];
}

// In place: photon counts by position -> photons of the tracks before each
// position, order_off[n_tracks] = the total (one block).
__global__ __launch_bounds__(1024) void order_offsets_kernel(int n_tracks, uint64_t *order_off) {
    __shared__ unsigned long long part[1024];
    const int t = threadIdx.x;
    const int per = (n_tracks + 1023) / 1024;
    const int lo = min(t * per, n_tracks), hi = min(lo + per, n_tracks);
    unsigned long long sum = 0;
#pragma unroll 8
    for (int q = lo; q < hi; ++q) sum += order_off[q];   // unrolled: the loads overlap
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        unsigned long long y = t >= off ? part[t - off] : 0ull;
        __syncthreads();
        part[t] += y;
        __syncthreads();
    }
    unsigned long long run = part[t] - sum;
#pragma unroll 8
    for (int q = lo; q < hi; ++q) {
        const unsigned long long c = order_off[q];
        order_off[q] = run;
        run += c;
    }
    if (t == 1023) order_off[n_tracks] = part[1023];
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t order_buffer_bytes(int n_tracks) {
    return align256((size_t)kOrderCells * 4) + align256((size_t)n_tracks * 4) + align256((size_t)n_tracks * 4) +
           ((size_t)n_tracks + 1) * 8;
}

void set_order(DevSource &src, void *buffer) {
    const int T = src.n_tracks;
    char *b = static_cast<char *>(buffer);
    src.order = reinterpret_cast<const int32_t *>(b + align256((size_t)kOrderCells * 4) + align256((size_t)T * 4));
    src.order_off =
        reinterpret_cast<const uint64_t *>(b + align256((size_t)kOrderCells * 4) + 2 * align256((size_t)T * 4));
}

hipError_t launch_order(const DevSource &src, int n_parts, void *buffer, hipStream_t st) {
    const int T = src.n_tracks;
    char *b = static_cast<char *>(buffer);
    uint32_t *hist = reinterpret_cast<uint32_t *>(b);
    uint32_t *cell_of = reinterpret_cast<uint32_t *>(b + align256((size_t)kOrderCells * 4));
    int32_t *order = const_cast<int32_t *>(src.order);
    uint64_t *order_off = const_cast<uint64_t *>(src.order_off);
    hipError_t e = launch_fill_u64(reinterpret_cast<unsigned long long *>(hist), kOrderCells / 2, st);
    if (e != hipSuccess) return e;
    const int blocks = (T + 255) / 256;
    hipLaunchKernelGGL(order_cells_kernel, dim3(blocks), dim3(256), 0, st, src.tracks, T, hist, cell_of);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(order_scan_cells_kernel, dim3(1), dim3(1024), 0, st, hist);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(order_scatter_kernel, dim3(blocks), dim3(256), 0, st, (const uint32_t *)cell_of, src.offsets,
                       hist, T, n_parts, order, order_off);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(order_offsets_kernel, dim3(1), dim3(1024), 0, st, T, order_off);
    return hipGetLastError();
}

// ---------------------------------------------------------------- batch: persistent, dynamic chunks

// Each wave repeatedly claims `chunk` consecutive photon ids from a global
// counter and traces them 64 at a time until the ids run out.  Every wave
// leaves the loop when a claim starts at or beyond n.
constexpr int kWaveGroup = 256;   // photons a batch wave regroups by cone azimuth
// a wave's regrouping buffer: 64 bins, then the positions in regrouped order (bytes)
constexpr int kRegroupWords = 64 + kWaveGroup / 4;

// Held to 128 VGPRs for 4 waves per SIMD.
template <bool kMesh, bool kPrefilter>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void batch_kernel(
    DevScene, DevSource, DevOutputs, uint64_t n, uint64_t seed, unsigned long long *counter, unsigned long long *next,
    int chunk, int whole_batch, uint64_t part, int n_parts) {
    extern __shared__ uint32_t lds_stack[];
    SceneRef S = scene_arg();
    SourceRef src = source_arg();
    OutputsRef out = outputs_arg();
    const int lane = __lane_id();
    constexpr TraceKind kTrace = kMesh ? kMeshLane : kAnalytic;
    uint32_t *stk = lane_stack<kTrace>(lds_stack);
    const int wave = threadIdx.x >> 6;
    uint32_t *wbins = lds_stack + (blockDim.x / 64) * (stack_words(kTrace) + kFates) + (size_t)wave * kRegroupWords;
    uint8_t *wperm = reinterpret_cast<uint8_t *>(wbins + 64);
    uint32_t cnt[kFates] = {0, 0, 0, 0, 0, 0, 0};
    if (whole_batch && blockIdx.x == 0 && threadIdx.x == 0 && src.offsets[src.n_tracks] != n)
        atomicOr(S.status, 8u);  // RICH_FLAG_BATCH_SIZE: n is not the photon total of the tracks
    if (next && blockIdx.x == 0 && threadIdx.x < kBatchParts) next[kCounterStride * threadIdx.x] = 0ull;
    // The processing positions 0..n-1 (photon ids, or with a processing order
    // its positions) are cut into n_parts contiguous partitions of `part`
    // positions (a multiple of the chunk); block b claims chunks of partition
    // b mod n_parts from that partition's own counter.  Blocks are dispatched
    // to the 8 XCDs round robin, so with 8 partitions each XCD works through
    // its own run of tracks and its L2 holds their geometry only.
    const int xp = (int)(blockIdx.x % (unsigned)n_parts);
    unsigned long long *ctr = counter + kCounterStride * xp;
    const uint64_t p_lo = (uint64_t)xp * part;
    const uint64_t p_hi = min(p_lo + part, n);
    while (true) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(ctr, (unsigned long long)chunk);
        uint32_t lo = __shfl((uint32_t)base, 0), hi = __shfl((uint32_t)(base >> 32), 0);
        base = p_lo + (((unsigned long long)hi << 32) | lo);
        if (base >= p_hi) break;
        // With meshes (or the pre-filter), each kWaveGroup-photon slice of the
        // chunk is regrouped by cone azimuth (64 bins of the azimuth's
        // uniform; pre-filter rejects last) in this wave's own LDS region, so
        // that each 64-photon pass traces neighbouring directions.  Only
        // chunks made of whole slices are regrouped: a partial slice would
        // reach into the next claim.  A wave's LDS operations complete in
        // order; the fences keep the compiler from moving them across phases.
        const bool regroup = (kMesh || kPrefilter) && chunk % kWaveGroup == 0;
        const int group = regroup ? kWaveGroup : 64;
        for (int k = 0; k < chunk; k += group) {
            if (regroup) {
                constexpr int per = kWaveGroup / 64;
                wbins[lane] = 0;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                uint32_t bin[per], rank[per];
                for (int j = 0; j < per; ++j) {
                    const uint64_t v = base + (uint64_t)(k + j * 64 + lane);
                    int tk = -1;
                    const uint64_t g = v < n ? batch_photon_id(src, v, n, tk) : v;
                    bin[j] = v < n ? regroup_bin<kPrefilter>(S, src, seed, g, 64u) : 63u;
                    rank[j] = atomicAdd(wbins + bin[j], 1u);
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                const uint32_t c = wbins[lane];
                uint32_t incl = c;
                for (int d = 1; d < 64; d <<= 1) {
                    uint32_t v = __shfl_up(incl, d);
                    if (lane >= d) incl += v;
                }
                wbins[lane] = incl - c;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                for (int j = 0; j < per; ++j)
                    wperm[min(wbins[bin[j]] + rank[j], (uint32_t)kWaveGroup - 1u)] = (uint8_t)(j * 64 + lane);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            }
            for (int j = 0; j < group; j += 64) {
                const uint32_t off = regroup ? (uint32_t)wperm[j + lane] : (uint32_t)(j + lane);
                const uint64_t v = base + (uint64_t)k + off;
                int tk = -1;
                const uint64_t g = v < n ? batch_photon_id(src, v, n, tk) : v;
                const int fate = photon_job<kTrace, kPrefilter, true>(S, src, out, v < n, g, g, seed, stk, tk);
                if (out.fate_counts) tally_wave(cnt, fate);
            }
            if (regroup) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
    }
    if (out.fate_counts) flush_tally(out, cnt, lds_stack + (blockDim.x / 64) * stack_words(kTrace));
}

// Dynamic LDS of the batch kernel: per-lane stacks, per-wave fate tallies,
// per-wave regrouping buffers.
size_t batch_lds_bytes(int block, bool mesh) {
    return (size_t)(block / 64) * (stack_words(mesh ? kMeshLane : kAnalytic) + kFates + kRegroupWords) * sizeof(uint32_t);
}

int batch_parts(int grid) { return (grid >= kBatchParts && grid % kBatchParts == 0) ? kBatchParts : 1; }

hipError_t launch_batch(const DevScene &S, const DevSource &src, const DevOutputs &out, uint64_t n, uint64_t seed,
                        unsigned long long *counter, unsigned long long *next, int block, int chunk, int grid,
                        bool whole_batch, hipStream_t st) {
    size_t lds = batch_lds_bytes(block, S.has_mesh != 0);
    const int n_parts = batch_parts(grid);
    const uint64_t per = (n + n_parts - 1) / n_parts;
    const uint64_t part = (per + chunk - 1) / chunk * chunk;
    static const auto kernels = {batch_kernel<false, false>, batch_kernel<false, true>, batch_kernel<true, false>,
                                 batch_kernel<true, true>};
    const auto kernel = kernels.begin()[(S.has_mesh ? 2 : 0) + (src.prefilter ? 1 : 0)];
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), lds, st, S, src, out, n, seed, counter, next, chunk,
                       whole_batch ? 1 : 0, part, n_parts);
    return hipGetLastError();
}

}  // namespace rich

#ifdef RICH_WORK_COUNTERS
// Measurement build only: copy the forward and batch kernels' work counters
// to the host (WorkUnit order: kWorkUnits lane counts, then kWorkUnits wave
// counts), then zero them when reset is set.  Synchronises the current device.
extern "C" int rich_work_counters(unsigned long long *out, int reset) {
    unsigned long long raw[16 * rich::kWorkUnits];
    if (hipDeviceSynchronize() != hipSuccess) return -3;
    if (hipMemcpyFromSymbol(raw, HIP_SYMBOL(rich::rich_work), sizeof raw) != hipSuccess) return -3;
    for (int u = 0; u < rich::kWorkUnits; ++u) {
        out[u] = raw[16 * u];
        out[rich::kWorkUnits + u] = raw[16 * u + 1];
    }
    if (reset) {
        unsigned long long zero[16 * rich::kWorkUnits] = {};
        if (hipMemcpyToSymbol(HIP_SYMBOL(rich::rich_work), zero, sizeof zero) != hipSuccess) return -3;
    }
    return 0;
}
#endif
