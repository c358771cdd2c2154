// Binned-SAH BVH builder: a binary tree built in FP64 over triangle centroids,
// collapsed into 4-wide nodes whose children are the (up to) four largest
// descendants, stored depth-first with FP32 boxes rounded outward.
#include "bvh_build.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <limits>
#include <map>
#include <thread>
#include <tuple>

namespace rich {

namespace {

constexpr int kBins = 32;
constexpr uint32_t kLeafSize = 4;      // largest leaf
constexpr uint32_t kAlwaysLeaf = 1;    // nodes of this many triangles or fewer are leaves
// Surface-area cost of testing a node against that of one triangle: a range
// of up to kLeafSize triangles becomes a leaf when testing them all costs no
// more than the node plus the children the split would make.
constexpr double kNodeCost = 1.0;
// A group of an instance with several meshes gets its own subtree when its
// box has at least this fraction of the instance box's surface area.
constexpr double kLargeGroupArea = 0.1;
// Sheets that share a subtree with other triangles get subtrees of their own,
// the largest by area first, up to this many.
constexpr int kMaxSheets = 8;
// Ranges of at least kParallelMin triangles in the top kParallelDepth levels
// of a subtree build their right half on a thread of its own.
constexpr int kParallelDepth = 3;
constexpr uint32_t kParallelMin = 16384;

struct BNode {
    BuildBox box;
    int left = -1, right = -1;
    uint32_t first = 0, count = 0;
};

BuildBox empty_box() {
    BuildBox b;
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = std::numeric_limits<double>::infinity();
        b.hi[a] = -std::numeric_limits<double>::infinity();
    }
    return b;
}

void grow(BuildBox &b, const double *p) {
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = std::min(b.lo[a], p[a]);
        b.hi[a] = std::max(b.hi[a], p[a]);
    }
}

void grow(BuildBox &b, const BuildBox &o) {
    for (int a = 0; a < 3; ++a) {
        b.lo[a] = std::min(b.lo[a], o.lo[a]);
        b.hi[a] = std::max(b.hi[a], o.hi[a]);
    }
}

double area(const BuildBox &b) {
    double dx = b.hi[0] - b.lo[0], dy = b.hi[1] - b.lo[1], dz = b.hi[2] - b.lo[2];
    if (dx < 0 || dy < 0 || dz < 0) return 0.0;
    return 2.0 * (dx * dy + dy * dz + dz * dx);
}

double dot3(const double *a, const double *b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }

// Centre of the sphere closest to the members' vertices (linear least squares
// of |x|^2 = 2 C.x + k about `mid`, in units of `size`).  False: no sphere
// (a plane, a line or a point).
bool fit_centre(const std::vector<BuildTri> &tris, const std::vector<uint32_t> &members, const double mid[3],
                double size, double C[3]) {
    double A[4][5] = {};
    for (uint32_t i : members)
        for (int m = 0; m < 3; ++m) {
            double r[4] = {0, 0, 0, 1.0}, q = 0;
            for (int a = 0; a < 3; ++a) {
                r[a] = (tris[i].v[m][a] - mid[a]) / size;
                q += r[a] * r[a];
            }
            for (int a = 0; a < 4; ++a) {
                for (int b = a; b < 4; ++b) A[a][b] += r[a] * r[b];
                A[a][4] += r[a] * q;
            }
        }
    for (int a = 0; a < 4; ++a)
        for (int b = 0; b < a; ++b) A[a][b] = A[b][a];
    // elimination with column pivoting over the rows
    for (int c = 0; c < 4; ++c) {
        int p = c;
        for (int r = c + 1; r < 4; ++r)
            if (std::fabs(A[r][c]) > std::fabs(A[p][c])) p = r;
        if (!(std::fabs(A[p][c]) > 1e-14 * (double)members.size())) return false;
        for (int k = 0; k < 5; ++k) std::swap(A[c][k], A[p][k]);
        for (int r = 0; r < 4; ++r) {
            if (r == c) continue;
            const double f = A[r][c] / A[c][c];
            for (int k = c; k < 5; ++k) A[r][k] -= f * A[c][k];
        }
    }
    for (int a = 0; a < 3; ++a) C[a] = mid[a] + 0.5 * size * A[a][4] / A[a][a];
    return std::isfinite(C[0]) && std::isfinite(C[1]) && std::isfinite(C[2]);
}

// How far a reflection point as the device computes it can lie from its facet,
// and what the next query's tests add: in units u = 2^-24 (half an FP32 step
// of 1), T the flight, rho the vertices' distance from the frame's origin, W
// the point's from the world's, L the longest edge.
//   the ray's origin in the frame                rho + T
//   vertices relative to it                      T + L
//   the shear's reciprocal (2 u) moves point and ray alike along one axis,
//   and its two products                         3 T
//   t = sum(U z) / (U + V + W): four roundings of the terms, two of the sum,
//   two of its reciprocal, one of the product    9 (T + L)
//   o + t d in the world                         W
//   the next query: the same with T = 0          rho + 17 L
// and where the frame turns, three products and sums per component (a factor
// 3 sqrt 3) for the origin twice and for the direction: 6 (2 rho + T) + 6 T.
// The edge functions' own products, u L'^2 each of L' <= sqrt 3 L (the sheared
// edges), shift the point within its facet by 8 u L^3 / (area cos), which for
// slivers is more than all of these, and once more in the next query; cos is
// that of the angle to the normal, at least the rule's m.
double point_error(const SheetBudget &b, double rho, double longest) {
    const double t = b.reach;
    double units = 14.0 * t + 2.0 * rho + b.far + 27.0 * longest;
    if (b.moving) units += 12.0 * (rho + t);
    return std::ldexp(units, -24);
}

// Whether the members form a sheet, and the least d.n of a reflected
// direction d with the normal n of the facet it left for which the sheet
// cannot be met again.
//
// For any point C: a facet's plane lies n.(C - v) from C and every vertex at
// most R = max |v - C|, so every vertex, and every point of every facet, is at
// worst `behind` = R - min n.(C - v) behind the plane of another facet (the
// cap a facet cuts off its sphere: 4e-4 mm for 3.5 mm facets of an 8 m
// sphere; 0 for a plane, whose C is far away).  The photon starts within
// point_error of its facet, and the device's facets lie within `rounding` of
// the exact ones.  A direction with d.n >= m for every facet's n thus meets
// no facet beyond (behind + point_error + 2 rounding) / m, and hits nearer
// than t_min do not count.  All normals lie within alpha of their mean, so m
// for every facet follows from an angle of at most acos(m) - 2 alpha with the
// normal of one.  Of the factor 1.25, kSheetSlack is for segments that move:
// scaled by s, their facets reach s times as far behind each other.
bool sheet_rule(const std::vector<BuildTri> &tris, const std::vector<uint32_t> &members, const SheetBudget &budget,
                float *min_cos) {
    if (members.empty()) return false;
    double axis[3] = {0, 0, 0}, mid[3] = {0, 0, 0}, rounding2 = 0, rho2 = 0, edge2 = 0, sliver = 0;
    BuildBox box = empty_box();
    for (uint32_t i : members) {
        const BuildTri &t = tris[i];
        if (!t.mirror || !(dot3(t.n, t.n) > 0.5)) return false;   // (a triangle without area has no normal)
        for (int a = 0; a < 3; ++a) axis[a] += t.n[a];
        for (int m = 0; m < 3; ++m) {
            grow(box, t.v[m]);
            double e2 = 0;
            for (int a = 0; a < 3; ++a) {
                const double e = t.v[m][a] - (double)(float)t.v[m][a];
                e2 += e * e;
            }
            rounding2 = std::max(rounding2, e2);
            rho2 = std::max(rho2, dot3(t.v[m], t.v[m]));
        }
        double e[3][3], l2 = 0;
        for (int m = 0; m < 3; ++m) {
            for (int a = 0; a < 3; ++a) e[m][a] = t.v[(m + 1) % 3][a] - t.v[m][a];
            l2 = std::max(l2, dot3(e[m], e[m]));
        }
        const double c[3] = {e[0][1] * e[1][2] - e[0][2] * e[1][1], e[0][2] * e[1][0] - e[0][0] * e[1][2],
                             e[0][0] * e[1][1] - e[0][1] * e[1][0]};
        edge2 = std::max(edge2, l2);
        sliver = std::max(sliver, std::ldexp(8.0, -24) * l2 * std::sqrt(l2) / (0.5 * std::sqrt(dot3(c, c))));
    }
    double len = std::sqrt(dot3(axis, axis)), size = 0, cos_alpha = 1.0;
    if (!(len > 0)) return false;
    for (int a = 0; a < 3; ++a) {
        axis[a] /= len;
        mid[a] = 0.5 * (box.lo[a] + box.hi[a]);
        size = std::max(size, box.hi[a] - box.lo[a]);
    }
    if (!(size > 0)) return false;
    for (uint32_t i : members) cos_alpha = std::min(cos_alpha, dot3(tris[i].n, axis));
    const double alpha = std::acos(std::max(-1.0, std::min(1.0, cos_alpha)));
    double centre[2][3];
    int n_centres = 1;
    for (int a = 0; a < 3; ++a) centre[0][a] = mid[a] + 1e6 * size * axis[a];
    if (fit_centre(tris, members, mid, size, centre[1])) n_centres = 2;
    double behind = std::numeric_limits<double>::infinity();
    for (int k = 0; k < n_centres; ++k) {
        double r2 = 0, p = std::numeric_limits<double>::infinity();
        for (uint32_t i : members) {
            const BuildTri &t = tris[i];
            for (int m = 0; m < 3; ++m) {
                const double q[3] = {centre[k][0] - t.v[m][0], centre[k][1] - t.v[m][1], centre[k][2] - t.v[m][2]};
                r2 = std::max(r2, dot3(q, q));
                p = std::min(p, dot3(t.n, q));
            }
        }
        behind = std::min(behind, std::sqrt(r2) - p);
    }
    const double off = std::max(behind, 0.0) + point_error(budget, std::sqrt(rho2), std::sqrt(edge2)) +
                       2.0 * std::sqrt(rounding2);
    const double m = 1.25 * (off + 2.0 * sliver / (1.25 * off / budget.t_min)) / budget.t_min;
    if (!(m < 1.0)) return false;
    const double angle = std::acos(m) - 2.0 * alpha;
    if (!(angle > 0.05)) return false;
    *min_cos = (float)std::min(1.0, std::cos(angle) + 1e-4);
    return true;
}

// A sheet found by the builder: its triangles' positions in Builder::idx.
struct SheetSpan {
    uint32_t first, count;
    float min_cos;
};

struct Builder {
    std::vector<BuildTri> &tris;
    const SheetBudget &budget;
    std::vector<BuildBox> tbox;
    std::vector<double> cen;  // [n][3]
    std::vector<uint32_t> idx;
    std::vector<BNode> bn;
    std::vector<SheetSpan> spans;

    Builder(std::vector<BuildTri> &t, const SheetBudget &b) : tris(t), budget(b) {
        size_t n = t.size();
        tbox.resize(n);
        cen.resize(3 * n);
        idx.resize(n);
        for (size_t i = 0; i < n; ++i) {
            BuildBox b = empty_box();
            for (int m = 0; m < 3; ++m) grow(b, t[i].v[m]);
            tbox[i] = b;
            for (int a = 0; a < 3; ++a) cen[3 * i + a] = 0.5 * (b.lo[a] + b.hi[a]);
            idx[i] = (uint32_t)i;
        }
    }

    // Given groups: an instance that holds several meshes gets one subtree per
    // large group (a plane whose box has at least kLargeGroupArea of the
    // instance box's surface area, such as an enclosure's wall), and one
    // subtree over all the other triangles, so that the SAH never mixes a thin
    // enclosure wall into a mirror's boxes.  Nodes whose box holds the ray's
    // origin cannot be culled; with the walls as the only separate subtrees
    // the fewest such nodes stand above them.  Within the other triangles'
    // subtree each sheet has one of its own (so that its nodes are contiguous).
    // Returns the root, or -1 unless every triangle has a group and two or
    // more subtrees result.
    int build_grouped() {
        std::map<int, int> dense;
        std::vector<int> grp(tris.size());
        for (size_t i = 0; i < tris.size(); ++i) {
            if (tris[i].group < 0) return -1;
            grp[i] = dense.emplace(tris[i].group, (int)dense.size()).first->second;
        }
        const int ng = (int)dense.size();
        std::vector<BuildBox> gbox(ng, empty_box());
        std::vector<std::vector<uint32_t>> members(ng);
        BuildBox all = empty_box();
        for (size_t i = 0; i < tris.size(); ++i) {
            grow(gbox[grp[i]], tbox[i]);
            grow(all, tbox[i]);
            members[grp[i]].push_back((uint32_t)i);
        }
        // parts: the large groups, then the sheets among the others, then the rest of them
        std::vector<int> part(ng, -1);
        int n_large = 0, n_parts = 0;
        for (int g = 0; g < ng; ++g)
            if (area(gbox[g]) >= kLargeGroupArea * area(all)) part[g] = n_large++;
        n_parts = n_large;
        std::vector<int> by_area;
        for (int g = 0; g < ng; ++g)
            if (part[g] < 0) by_area.push_back(g);
        std::stable_sort(by_area.begin(), by_area.end(), [&](int a, int b) { return area(gbox[a]) > area(gbox[b]); });
        std::vector<float> min_cos;
        for (int g : by_area) {
            float c;
            if ((int)min_cos.size() < kMaxSheets && sheet_rule(tris, members[g], budget, &c)) {
                part[g] = n_parts++;
                min_cos.push_back(c);
            }
        }
        bool rest = false;
        for (int g = 0; g < ng; ++g)
            if (part[g] < 0) {
                part[g] = n_parts;
                rest = true;
            }
        if (rest) ++n_parts;
        if (n_parts < 2) return -1;
        for (auto &v : grp) v = part[v];
        return chain_groups(grp, n_parts, n_large, min_cos);
    }

    // Planar grouping: a mesh made of a few planes (an enclosure's walls) gets
    // one subtree per plane, the planes chained under the root so that the
    // BVH4 root holds thin per-wall boxes rather than half-box boxes that
    // contain every ray starting inside.  Returns the root, or -1 if the mesh
    // is not a union of 2..64 planes.
    int build_planar() {
        std::vector<int> grp;
        int ng = plane_groups(tris, 64, grp);
        if (ng < 2) return -1;
        return chain_groups(grp, ng, ng, {});
    }

    // Subtrees of the groups: those from n_chain on joined into one, then this
    // and the others, largest first, chained under the root.  min_cos: of the
    // groups from n_chain on that are sheets.
    int chain_groups(const std::vector<int> &grp, int ng, int n_chain, const std::vector<float> &min_cos) {
        std::vector<uint32_t> gcount(ng, 0);
        for (int g : grp) ++gcount[g];
        std::vector<int> order(ng);
        for (int g = 0; g < ng; ++g) order[g] = g;
        std::sort(order.begin(), order.end(), [&](int a, int b) { return gcount[a] > gcount[b] || (gcount[a] == gcount[b] && a < b); });
        std::vector<int> rank(ng), pos_of(ng);
        for (int r = 0; r < ng; ++r) pos_of[order[r]] = rank[order[r]] = r;
        std::stable_sort(idx.begin(), idx.end(), [&](uint32_t a, uint32_t b) { return rank[grp[a]] < rank[grp[b]]; });
        std::vector<uint32_t> start(ng + 1, 0);
        for (int r = 0; r < ng; ++r) start[r + 1] = start[r] + gcount[order[r]];
        // the groups' subtrees are independent: built on host threads into
        // their own node lists, then appended in group order with their
        // indices rebased (the same tree as building them in turn)
        std::vector<std::vector<BNode>> local(ng);
        std::vector<int> root(ng);
        parallel_for((size_t)ng, std::min(16u, std::max(1u, std::thread::hardware_concurrency())), [&](size_t r) {
            root[r] = build_into(local[r], start[r], start[r + 1] - start[r]);
        });
        for (int r = 0; r < ng; ++r) {
            const int base = (int)bn.size();
            for (BNode b : local[r]) {
                if (b.left >= 0) {
                    b.left += base;
                    b.right += base;
                }
                bn.push_back(b);
            }
            root[r] += base;
        }
        for (size_t k = 0; k < min_cos.size(); ++k) {
            const int r = pos_of[n_chain + (int)k];
            spans.push_back({start[r], start[r + 1] - start[r], min_cos[k]});
        }
        std::vector<int> links;   // subtrees to chain, the joined one among them by its triangle count
        std::vector<int> joined;
        for (int r = 0; r < ng; ++r) (order[r] < n_chain ? links : joined).push_back(root[r]);
        if (!joined.empty()) links.push_back(join(joined));
        std::stable_sort(links.begin(), links.end(), [&](int a, int b) { return bn[a].count > bn[b].count; });
        int top = links.back();
        for (size_t k = links.size() - 1; k-- > 0;) top = pair(links[k], top);
        return top;
    }

    int pair(int l, int r) {
        const int me = (int)bn.size();
        bn.emplace_back();
        BuildBox box = bn[l].box;
        grow(box, bn[r].box);
        bn[me].box = box;
        bn[me].first = std::min(bn[l].first, bn[r].first);
        bn[me].count = bn[l].count + bn[r].count;
        bn[me].left = l;
        bn[me].right = r;
        return me;
    }

    // One tree over a few subtrees: splits by their boxes' centres along the
    // axis and at the place of the least surface-area cost.
    int join(std::vector<int> roots) {
        if (roots.size() == 1) return roots[0];
        double best = std::numeric_limits<double>::infinity();
        std::vector<int> left, right;
        for (int a = 0; a < 3; ++a) {
            std::stable_sort(roots.begin(), roots.end(), [&](int x, int y) {
                return bn[x].box.lo[a] + bn[x].box.hi[a] < bn[y].box.lo[a] + bn[y].box.hi[a];
            });
            for (size_t k = 1; k < roots.size(); ++k) {
                double cost = 0;
                for (int side = 0; side < 2; ++side) {
                    BuildBox box = empty_box();
                    double count = 0;
                    for (size_t q = side ? k : 0; q < (side ? roots.size() : k); ++q) {
                        grow(box, bn[roots[q]].box);
                        count += bn[roots[q]].count;
                    }
                    cost += area(box) * count;
                }
                if (cost < best || left.empty()) {   // (areas overflow from coordinates of 1e154 on)
                    best = cost;
                    left.assign(roots.begin(), roots.begin() + (long)k);
                    right.assign(roots.begin() + (long)k, roots.end());
                }
            }
        }
        const int l = join(left), r = join(right);
        return pair(l, r);
    }

    int build(uint32_t first, uint32_t count) { return build_into(bn, first, count); }

    // Binary SAH subtree over idx[first, first + count), appended to `out`
    // (child indices are positions in `out`).  The right halves of the top
    // kParallelDepth splits of large ranges are built on host threads of
    // their own and appended after the left ones: the same tree, so the same
    // emitted arrays, as building them in turn.
    int build_into(std::vector<BNode> &out, uint32_t first, uint32_t count, int depth = 0) {
        int me = (int)out.size();
        out.emplace_back();
        BuildBox box = empty_box(), cb = empty_box();
        for (uint32_t q = first; q < first + count; ++q) {
            grow(box, tbox[idx[q]]);
            grow(cb, &cen[3 * idx[q]]);
        }
        out[me].box = box;
        out[me].first = first;
        out[me].count = count;
        if (count <= kAlwaysLeaf) return me;

        // binned SAH over the centroid bounds
        double best_cost = std::numeric_limits<double>::infinity();
        int best_axis = -1, best_split = -1;
        for (int a = 0; a < 3; ++a) {
            double ext = cb.hi[a] - cb.lo[a];
            if (!(ext > 0)) continue;
            double scale = kBins / ext;
            BuildBox bb[kBins];
            uint32_t bc[kBins] = {};
            for (int k = 0; k < kBins; ++k) bb[k] = empty_box();
            for (uint32_t q = first; q < first + count; ++q) {
                int k = std::min(kBins - 1, (int)((cen[3 * idx[q] + a] - cb.lo[a]) * scale));
                ++bc[k];
                grow(bb[k], tbox[idx[q]]);
            }
            double right_area[kBins];
            uint32_t right_cnt[kBins];
            BuildBox acc = empty_box();
            uint32_t cnt = 0;
            for (int k = kBins - 1; k > 0; --k) {
                grow(acc, bb[k]);
                cnt += bc[k];
                right_area[k] = area(acc);
                right_cnt[k] = cnt;
            }
            acc = empty_box();
            cnt = 0;
            for (int k = 0; k < kBins - 1; ++k) {
                grow(acc, bb[k]);
                cnt += bc[k];
                if (cnt == 0 || right_cnt[k + 1] == 0) continue;
                double cost = area(acc) * cnt + right_area[k + 1] * right_cnt[k + 1];
                if (cost < best_cost) {
                    best_cost = cost;
                    best_axis = a;
                    best_split = k + 1;
                }
            }
        }
        if (count <= kLeafSize && (best_axis < 0 || area(box) * count <= kNodeCost * area(box) + best_cost)) return me;
        uint32_t mid;
        if (best_axis >= 0) {
            double ext = cb.hi[best_axis] - cb.lo[best_axis];
            double scale = kBins / ext;
            auto it = std::partition(idx.begin() + first, idx.begin() + first + count, [&](uint32_t i) {
                int k = std::min(kBins - 1, (int)((cen[3 * i + best_axis] - cb.lo[best_axis]) * scale));
                return k < best_split;
            });
            mid = (uint32_t)(it - idx.begin());
        } else {
            mid = first + count / 2;  // all centroids coincide: split the index range
        }
        if (mid == first || mid == first + count) mid = first + count / 2;
        int l, r;
        if (depth < kParallelDepth && count >= kParallelMin) {
            std::vector<BNode> right;
            int r_local = -1;
            parallel_for(2, 2, [&](size_t half) {
                if (half == 0) l = build_into(out, first, mid - first, depth + 1);
                else r_local = build_into(right, mid, first + count - mid, depth + 1);
            });
            const int base = (int)out.size();
            for (BNode b : right) {
                if (b.left >= 0) {
                    b.left += base;
                    b.right += base;
                }
                out.push_back(b);
            }
            r = r_local + base;
        } else {
            l = build_into(out, first, mid - first, depth + 1);
            r = build_into(out, mid, first + count - mid, depth + 1);
        }
        out[me].left = l;
        out[me].right = r;
        return me;
    }
};

void set_child_box(Node4 &nd, int k, const BuildBox &b) {
    nd.lox[k] = lower_f32(b.lo[0]);
    nd.loy[k] = lower_f32(b.lo[1]);
    nd.loz[k] = lower_f32(b.lo[2]);
    nd.hix[k] = upper_f32(b.hi[0]);
    nd.hiy[k] = upper_f32(b.hi[1]);
    nd.hiz[k] = upper_f32(b.hi[2]);
}

void clear_node(Node4 &nd) {
    for (int k = 0; k < 4; ++k) {
        nd.lox[k] = nd.loy[k] = nd.loz[k] = std::numeric_limits<float>::infinity();
        nd.hix[k] = nd.hiy[k] = nd.hiz[k] = -std::numeric_limits<float>::infinity();
        nd.child[k] = kEmpty;
    }
    nd.leaves = nd.order = nd.pad[0] = nd.pad[1] = 0;
}

// Node4::order of a node whose children's boxes are set: for each pair the
// axis of the widest gap between their boxes (or least overlap).
void set_order(Node4 &nd) {
    const float *lo[3] = {nd.lox, nd.loy, nd.loz}, *hi[3] = {nd.hix, nd.hiy, nd.hiz};
    int shift = 0;
    nd.order = 0;
    for (int i = 0; i < 4; ++i)
        for (int j = i + 1; j < 4; ++j, shift += 3) {
            if (nd.child[i] == kEmpty || nd.child[j] == kEmpty) continue;
            uint32_t best = 0;
            float gap = -std::numeric_limits<float>::infinity();
            for (uint32_t a = 0; a < 3; ++a) {
                const float up = lo[a][j] - hi[a][i], down = lo[a][i] - hi[a][j];
                if (std::max(up, down) > gap) {
                    gap = std::max(up, down);
                    best = a | (up > down ? 4u : 0u);
                }
            }
            nd.order |= best << shift;
        }
}

// Pick up to four descendants of a binary node: repeatedly open the largest internal one.
std::vector<int> gather4(const std::vector<BNode> &bn, int root) {
    std::vector<int> kids;
    if (bn[root].left < 0) {
        kids.push_back(root);
        return kids;
    }
    kids = {bn[root].left, bn[root].right};
    while (kids.size() < 4) {
        int pick = -1;
        double best = -1;
        for (size_t k = 0; k < kids.size(); ++k) {
            const BNode &c = bn[kids[k]];
            if (c.left >= 0 && area(c.box) > best) {
                best = area(c.box);
                pick = (int)k;
            }
        }
        if (pick < 0) break;
        int c = kids[pick];
        kids.erase(kids.begin() + pick);
        kids.push_back(bn[c].left);
        kids.push_back(bn[c].right);
    }
    return kids;
}

struct Emitter {
    const std::vector<BNode> &bn;
    const std::vector<uint32_t> &idx;
    const std::vector<BuildTri> &tris;
    std::vector<Node4> &nodes;
    std::vector<Tri> &out;
    const std::vector<SheetSpan> &spans;
    std::vector<Sheet> &sheets;   // one per span, in order
    size_t sheet_base = 0;        // sheets.size() before them
    int max_depth = 0;

    bool bad_leaf = false;   // a leaf the reference encoding cannot hold

    // The span that holds a node's triangles, or -1.
    int span_of(const BNode &b) const {
        for (size_t k = 0; k < spans.size(); ++k)
            if (b.first >= spans[k].first && b.first + b.count <= spans[k].first + spans[k].count) return (int)k;
        return -1;
    }

    uint32_t leaf_ref(const BNode &b) {
        if (b.count == 0 || b.count > kLeafMaxTris) bad_leaf = true;
        uint32_t first = (uint32_t)out.size();
        const int span = span_of(b);
        const uint32_t sheet = span < 0 ? 0u : 1u + (uint32_t)(sheet_base + (size_t)span);
        for (uint32_t q = b.first; q < b.first + b.count; ++q) {
            const BuildTri &t = tris[idx[q]];
            Tri r;
            for (int a = 0; a < 3; ++a) {
                r.v0[a] = (float)t.v[0][a];
                r.v1[a] = (float)t.v[1][a];
                r.v2[a] = (float)t.v[2][a];
                r.n[a] = (float)t.n[a];
            }
            r.index = t.index;
            r.material = t.material;
            r.pad0 = 0;
            r.sheet = sheet;
            out.push_back(r);
        }
        return make_leaf(first, b.count);
    }

    uint32_t emit(int root, int depth) {
        max_depth = std::max(max_depth, depth);
        uint32_t me = (uint32_t)nodes.size();
        nodes.emplace_back();
        clear_node(nodes[me]);
        const int span = span_of(bn[root]);
        if (span >= 0) {
            // depth-first emission in triangle order: the span's nodes follow each other
            Sheet &sh = sheets[sheet_base + (size_t)span];
            if (sh.node_n == 0) sh.node_lo = me;
            sh.node_n = me - sh.node_lo + 1;
        }
        std::vector<int> kids = gather4(bn, root);
        std::stable_sort(kids.begin(), kids.end(), [&](int a, int b) { return bn[a].first < bn[b].first; });
        for (size_t k = 0; k < kids.size(); ++k) {
            const BNode &c = bn[kids[k]];
            uint32_t ref = (c.left < 0) ? leaf_ref(c) : emit(kids[k], depth + 1);
            Node4 &nd = nodes[me];
            set_child_box(nd, (int)k, c.box);
            nd.child[k] = ref;
            if (c.left < 0) nd.leaves |= 1u << k;
        }
        set_order(nodes[me]);
        return me;
    }
};

}  // namespace

bool PlaneKey::operator<(const PlaneKey &o) const {
    return std::tie(nx, ny, nz, off) < std::tie(o.nx, o.ny, o.nz, o.off);
}

PlaneKey plane_key(const BuildTri &t) {
    double off = t.n[0] * t.v[0][0] + t.n[1] * t.v[0][1] + t.n[2] * t.v[0][2];
    return {std::llround(t.n[0] * 1e6), std::llround(t.n[1] * 1e6), std::llround(t.n[2] * 1e6), std::llround(off * 1e3)};
}

int plane_groups(const std::vector<BuildTri> &tris, int max_groups, std::vector<int> &grp) {
    std::map<PlaneKey, int> key_to_group;
    grp.resize(tris.size());
    for (size_t i = 0; i < tris.size(); ++i) {
        auto it = key_to_group.find(plane_key(tris[i]));
        if (it == key_to_group.end()) {
            if ((int)key_to_group.size() >= max_groups) return -1;
            it = key_to_group.emplace(plane_key(tris[i]), (int)key_to_group.size()).first;
        }
        grp[i] = it->second;
    }
    return (int)key_to_group.size();
}

float lower_f32(double x) {
    double pad = 1e-3 + 1e-6 * std::fabs(x);
    float f = (float)(x - pad);
    while ((double)f > x - pad) f = std::nextafter(f, -std::numeric_limits<float>::infinity());
    return f;
}

float upper_f32(double x) {
    double pad = 1e-3 + 1e-6 * std::fabs(x);
    float f = (float)(x + pad);
    while ((double)f < x + pad) f = std::nextafter(f, std::numeric_limits<float>::infinity());
    return f;
}

uint32_t build_mesh_bvh4(std::vector<BuildTri> &tris, std::vector<Node4> &nodes, std::vector<Tri> &out, int *depth,
                         BuildBox *bounds, const SheetBudget &budget, std::vector<Sheet> &sheets) {
    Builder b(tris, budget);
    b.bn.reserve(2 * tris.size() / kLeafSize + 2);
    int top = b.build_grouped();
    if (top < 0) {
        float c;
        if (sheet_rule(tris, b.idx, budget, &c)) b.spans.push_back({0, (uint32_t)tris.size(), c});
        top = b.build_planar();
    }
    if (top < 0) top = b.build(0, (uint32_t)tris.size());
    if (bounds) *bounds = b.bn[top].box;
    Emitter e{b.bn, b.idx, tris, nodes, out, b.spans, sheets, sheets.size()};
    for (const SheetSpan &sp : b.spans) sheets.push_back({0, 0, sp.min_cos, sp.min_cos});
    uint32_t root = e.emit(top, 1);
    if (depth) *depth = e.max_depth;
    return e.bad_leaf ? kEmpty : root;
}

uint32_t build_top_bvh4(const std::vector<BuildBox> &boxes, std::vector<Node4> &nodes, int *depth) {
    // binary median splits over instance boxes (largest extent first), one instance per leaf
    std::vector<BuildTri> pseudo(boxes.size());
    for (size_t i = 0; i < boxes.size(); ++i) {
        for (int a = 0; a < 3; ++a) {
            pseudo[i].v[0][a] = boxes[i].lo[a];
            pseudo[i].v[1][a] = boxes[i].hi[a];
            pseudo[i].v[2][a] = boxes[i].lo[a];
            pseudo[i].n[a] = 0;
        }
        pseudo[i].index = (uint32_t)i;
        pseudo[i].material = 0;
    }
    // one instance per leaf: build with leaf size 1 by splitting until single
    struct TopBuilder {
        std::vector<BuildTri> &t;
        std::vector<uint32_t> idx;
        std::vector<BNode> bn;
        int build(uint32_t first, uint32_t count, const std::vector<BuildBox> &bx) {
            int me = (int)bn.size();
            bn.emplace_back();
            BuildBox box = empty_box();
            for (uint32_t q = first; q < first + count; ++q) grow(box, bx[idx[q]]);
            bn[me].box = box;
            bn[me].first = first;
            bn[me].count = count;
            if (count == 1) return me;
            int axis = 0;
            double ext[3];
            for (int a = 0; a < 3; ++a) ext[a] = box.hi[a] - box.lo[a];
            if (ext[1] > ext[axis]) axis = 1;
            if (ext[2] > ext[axis]) axis = 2;
            std::sort(idx.begin() + first, idx.begin() + first + count, [&](uint32_t a, uint32_t b) {
                double ca = bx[a].lo[axis] + bx[a].hi[axis], cb = bx[b].lo[axis] + bx[b].hi[axis];
                return ca < cb || (ca == cb && a < b);
            });
            uint32_t mid = first + count / 2;
            int l = build(first, mid - first, bx);
            int r = build(mid, first + count - mid, bx);
            bn[me].left = l;
            bn[me].right = r;
            return me;
        }
    } tb{pseudo, {}, {}};
    // An instance whose box has at least kLargeGroupArea of the scene box's
    // area (the fixed meshes of an enclosure, which hold every ray origin)
    // hangs from the root itself: a node above it would hold the origin too
    // and be visited by every query.  Up to three such instances, the rest
    // in a median-split tree beside them.
    BuildBox all = empty_box();
    for (const auto &b : boxes) grow(all, b);
    std::vector<uint32_t> large, rest;
    for (size_t i = 0; i < boxes.size(); ++i)
        (area(boxes[i]) >= kLargeGroupArea * area(all) ? large : rest).push_back((uint32_t)i);
    int top;
    if (!large.empty() && large.size() <= 3 && !rest.empty()) {
        tb.idx = large;
        tb.idx.insert(tb.idx.end(), rest.begin(), rest.end());
        const uint32_t nl = (uint32_t)large.size();
        top = tb.build(nl, (uint32_t)rest.size(), boxes);
        for (int k = (int)nl - 1; k >= 0; --k) {
            const int leaf = tb.build((uint32_t)k, 1, boxes);
            const int me = (int)tb.bn.size();
            tb.bn.emplace_back();
            BuildBox box = tb.bn[leaf].box;
            grow(box, tb.bn[top].box);
            tb.bn[me].box = box;
            tb.bn[me].first = (uint32_t)k;
            tb.bn[me].count = (uint32_t)boxes.size() - (uint32_t)k;
            tb.bn[me].left = leaf;
            tb.bn[me].right = top;
            top = me;
        }
    } else {
        tb.idx.resize(boxes.size());
        for (size_t i = 0; i < boxes.size(); ++i) tb.idx[i] = (uint32_t)i;
        top = tb.build(0, (uint32_t)boxes.size(), boxes);
    }

    int maxd = 0;
    std::vector<Node4> &nd = nodes;
    struct TopEmit {
        const std::vector<BNode> &bn;
        const std::vector<uint32_t> &idx;
        std::vector<Node4> &nodes;
        int &maxd;
        uint32_t emit(int root, int depth) {
            maxd = std::max(maxd, depth);
            uint32_t me = (uint32_t)nodes.size();
            nodes.emplace_back();
            clear_node(nodes[me]);
            std::vector<int> kids;
            if (bn[root].left < 0) kids.push_back(root);
            else kids = gather4(bn, root);
            for (size_t k = 0; k < kids.size(); ++k) {
                const BNode &c = bn[kids[k]];
                uint32_t ref = (c.left < 0) ? make_inst(idx[c.first]) : emit(kids[k], depth + 1);
                set_child_box(nodes[me], (int)k, c.box);
                nodes[me].child[k] = ref;
            }
            set_order(nodes[me]);
            return me;
        }
    } te{tb.bn, tb.idx, nd, maxd};
    uint32_t root = te.emit(top, 1);
    if (depth) *depth = maxd;
    return root;
}

}  // namespace rich
