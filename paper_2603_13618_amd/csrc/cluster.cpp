// cluster.cpp -- Berger-Rigoutsos clustering of tagged tiles into
// rectangular patches (the paper's regridding step 2, Sec. II.B.2), host C++.
//
// Input: the number of tagged cells of every ts x ts tile of an nx x ny grid
// (the device's tile counts).  A box is the tight bounding box of the tagged
// tiles inside it; it is accepted when its efficiency (tagged cells / cells)
// reaches eff, otherwise cut:
//   1. at a hole of the column or row signature (a tile column / row with no
//      tag), cutting just before it; the hole nearest the middle of its axis
//      (smallest |2k + 1 - n|), x before y, then the lower index;
//   2. else at an inflection of a signature: between tiles k-1 and k where
//      its discrete Laplacian changes strict sign; the largest jump of the
//      Laplacian, then nearest the middle (smallest |2k - n|), x before y,
//      then the lower index;
//   3. else halfway along the longer axis (x on a tie).
// Every cut leaves at least min_tiles tiles on both sides; a box with no
// admissible cut is accepted as it is.  The low part of a cut is clustered
// first, so the output order is depth-first.
//
// Signatures of a box are differences of two rows of prefix-sum tables (counts
// summed over the tile rows below and over the tile columns to the left), so
// each costs O(box side), not O(box area), and reads memory in order.
#include <cstdint>
#include <cstdlib>
#include <vector>

#include "lks.h"

namespace {

struct Grid {
    int tx, ty, ts, nx, ny;
    std::vector<int64_t> below;    // below[j][i]: sum of counts[0 .. j-1][i], ty+1 rows of tx
    std::vector<int64_t> left;     // left[i][j]: sum of counts[j][0 .. i-1], tx+1 rows of ty

    int64_t cells(int lo, int hi, int n) const
    {
        const int64_t end = (int64_t)hi * ts < n ? (int64_t)hi * ts : n;
        return end - (int64_t)lo * ts;
    }
};

struct Cut {
    bool found = false;
    int axis = 0, k = 0;
};

// signature along an axis: x = per tile column of the box, y = per tile row
void signatures(const Grid& g, int i0, int j0, int i1, int j1, std::vector<int64_t>& sx,
                std::vector<int64_t>& sy)
{
    sx.resize(i1 - i0);
    sy.resize(j1 - j0);
    const int64_t* b0 = &g.below[(size_t)j0 * g.tx + i0];
    const int64_t* b1 = &g.below[(size_t)j1 * g.tx + i0];
    for (int i = 0; i < i1 - i0; ++i) sx[i] = b1[i] - b0[i];
    const int64_t* l0 = &g.left[(size_t)i0 * g.ty + j0];
    const int64_t* l1 = &g.left[(size_t)i1 * g.ty + j0];
    for (int j = 0; j < j1 - j0; ++j) sy[j] = l1[j] - l0[j];
}

struct Signature {
    const int64_t* s;
    int n;
};

Cut find_cut(const Signature& sx, const Signature& sy, int min_tiles)
{
    const Signature* sig[2] = {&sx, &sy};
    Cut best;
    // 1. holes: outwards from the middle of each axis, the lower index of a
    // pair first, so the first hole found is the axis's nearest
    int bdist = 0;
    for (int axis = 0; axis < 2; ++axis) {
        const int64_t* s = sig[axis]->s;
        const int n = sig[axis]->n;
        for (int dist = (n + 1) % 2; dist < n; dist += 2) {     // |2k + 1 - n|
            if (best.found && dist >= bdist) break;
            const int lo = (n - 1 - dist) / 2, hi = (n - 1 + dist) / 2;
            const int k = lo >= min_tiles && n - lo >= min_tiles && s[lo] == 0   ? lo
                          : hi >= min_tiles && n - hi >= min_tiles && s[hi] == 0 ? hi
                                                                                  : -1;
            if (k < 0) continue;
            best.found = true;
            best.axis = axis;
            best.k = k;
            bdist = dist;
            break;
        }
    }
    if (best.found) return best;
    // 2. inflections
    int64_t bjump = 0;
    int bmid = 0;
    for (int axis = 0; axis < 2; ++axis) {
        const int64_t* s = sig[axis]->s;
        const int n = sig[axis]->n;
        if (n < 4) continue;
        const int k0 = min_tiles > 2 ? min_tiles : 2, k1 = n - (min_tiles > 2 ? min_tiles : 2);
        if (k0 > k1) continue;
        int64_t lap_a = s[k0] - 2 * s[k0 - 1] + s[k0 - 2];             // at tile k - 1
        for (int k = k0; k <= k1; ++k) {
            const int64_t lap_b = s[k + 1] - 2 * s[k] + s[k - 1];      // at tile k
            const int64_t jump = lap_b > lap_a ? lap_b - lap_a : lap_a - lap_b;
            const bool cross = (lap_a < 0 && lap_b > 0) || (lap_a > 0 && lap_b < 0);
            lap_a = lap_b;
            if (!cross || (best.found && jump < bjump)) continue;
            const int mid = std::abs(2 * k - n);
            if (best.found && jump == bjump && mid >= bmid) continue;
            best.found = true;
            best.axis = axis;
            best.k = k;
            bjump = jump;
            bmid = mid;
        }
    }
    if (best.found) return best;
    // 3. bisection of the longer axis
    const int nx = sx.n, ny = sy.n;
    const int axis = nx >= ny ? 0 : 1;
    const int n = axis == 0 ? nx : ny;
    if (n / 2 >= min_tiles && n - n / 2 >= min_tiles) {
        best.found = true;
        best.axis = axis;
        best.k = n / 2;
    }
    return best;
}

struct Work {
    int i0, j0, i1, j1;
};

} // namespace

extern "C" lks_status lks_cluster(const int32_t* counts, int32_t nx, int32_t ny, int32_t ts, double eff,
                                  int32_t min_tiles, lks_box* boxes, int32_t max_boxes, int32_t* nboxes)
{
    if (!counts || !nboxes || nx < 1 || ny < 1 || ts < 1 || min_tiles < 1 || max_boxes < 0 ||
        (max_boxes > 0 && !boxes) || !(eff >= 0.0 && eff <= 1.0))
        return LKS_EINVAL;
    Grid g;
    g.ts = ts;
    g.nx = nx;
    g.ny = ny;
    g.tx = (nx + ts - 1) / ts;
    g.ty = (ny + ts - 1) / ts;
    g.below.resize((size_t)(g.ty + 1) * g.tx);
    g.left.resize((size_t)(g.tx + 1) * g.ty);
    for (int i = 0; i < g.tx; ++i) g.below[i] = 0;
    for (int j = 0; j < g.ty; ++j) {
        const int32_t* c = &counts[(size_t)j * g.tx];
        const int64_t* from = &g.below[(size_t)j * g.tx];
        int64_t* to = &g.below[(size_t)(j + 1) * g.tx];
        int32_t bad = 0;
        for (int i = 0; i < g.tx; ++i) {
            bad |= c[i];
            to[i] = from[i] + c[i];
        }
        if (bad < 0) return LKS_EINVAL;             // some count is negative
        int64_t sum = 0;
        g.left[j] = 0;
        for (int i = 0; i < g.tx; ++i) g.left[(size_t)(i + 1) * g.ty + j] = sum += c[i];
    }

    int32_t n = 0;
    std::vector<Work> stack;          // depth-first, low part of every cut first
    stack.push_back({0, 0, g.tx, g.ty});
    std::vector<int64_t> sx, sy;
    while (!stack.empty()) {
        Work w = stack.back();
        stack.pop_back();
        // tight bounding box of the tagged tiles
        signatures(g, w.i0, w.j0, w.i1, w.j1, sx, sy);
        int a = 0, b = (int)sx.size() - 1;
        while (a <= b && sx[a] == 0) ++a;
        if (a > b) continue;                        // no tag in this box
        while (sx[b] == 0) --b;
        int c = 0, d = (int)sy.size() - 1;
        while (sy[c] == 0) ++c;
        while (sy[d] == 0) --d;
        const int i0 = w.i0 + a, i1 = w.i0 + b + 1, j0 = w.j0 + c, j1 = w.j0 + d + 1;
        // its own signatures: no tag lies in the tiles cut off, so the others'
        // values stand
        const Signature bx = {sx.data() + a, b - a + 1}, by = {sy.data() + c, d - c + 1};
        int64_t tagged = 0;
        for (int i = 0; i < bx.n; ++i) tagged += bx.s[i];
        const int64_t area = g.cells(i0, i1, nx) * g.cells(j0, j1, ny);
        Cut cut;
        if (!((double)tagged >= eff * (double)area)) cut = find_cut(bx, by, min_tiles);
        if (!cut.found) {
            if (n < max_boxes) {
                lks_box& o = boxes[n];
                o.x0 = i0 * ts;
                o.y0 = j0 * ts;
                o.x1 = (int64_t)i1 * ts < nx ? i1 * ts : nx;
                o.y1 = (int64_t)j1 * ts < ny ? j1 * ts : ny;
            }
            ++n;
            continue;
        }
        // push the high part first so the low part is taken next
        if (cut.axis == 0) {
            stack.push_back({i0 + cut.k, j0, i1, j1});
            stack.push_back({i0, j0, i0 + cut.k, j1});
        } else {
            stack.push_back({i0, j0 + cut.k, i1, j1});
            stack.push_back({i0, j0, i1, j0 + cut.k});
        }
    }
    *nboxes = n;
    return n <= max_boxes ? LKS_OK : LKS_EINVAL;
}
