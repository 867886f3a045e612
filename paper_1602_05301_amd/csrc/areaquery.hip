// Area queries (Sec. 5) and target association through them (Sec. 6.1).
//
// An area query returns the leaves meeting a closed square C_r(c).  It first
// descends from the root along the boxes holding c while the box radius is
// at least 2r, stopping at the first box b with |b|/2 < r <= |b| or where no
// child holds c: the guiding box.  Its peers (Sec. 5 definition: adjacent,
// at least as large, and finest such) cover the 3 x 3 block of cells of b's
// level around it, which holds C_r(c) because c lies in b and r <= |b|.
// The leaves below the peers are then tested against the square.
//
// Peers are found per cell of that block: the finest box of level <= l(b)
// holding the cell.  The tree leaves out children without points, so the
// descent to a cell can stop at a box that has children but none on the
// cell's side; that quadrant holds no leaf (an area query skips it) and is
// kept as a region of its own for association lists.  No peer is then an
// ancestor of another, so every leaf is visited at most once.
#include "areaquery.hpp"

#include <cmath>

namespace qbx {
namespace {

// DFS stack: at most 9 peers, then at most 3 pending siblings per level below
// them.  A lane's entries are kAqThreads apart in LDS, and what a workgroup
// takes follows the tree's depth: with room for 31 levels (32 KiB) five waves
// fit a CU, and a million disk tests on a tree of 8192 points took 589 us, where
// scratch memory had taken 409; now 314.
// One wave a workgroup: a few thousand queries then reach every CU.
constexpr int kAqThreads = 64;
// Relative margin of the subtree pruning test, so that rounding in the
// stored box centres never cuts off a leaf that meets the square.
constexpr double kAqSlack = 1e-12;

__device__ __forceinline__ double aq_rad(const AQTree &t, int l) { return ldexp(t.R0, -l); }

// The closed box of centre (mx, my) and radius rb meets C_r(c).
__device__ __forceinline__ bool aq_meets(double mx, double my, double rb, double cx, double cy, double r)
{
    double lim = r + rb;
    return fabs(mx - cx) <= lim && fabs(my - cy) <= lim;
}

__device__ __forceinline__ bool aq_may_meet(double mx, double my, double rb, double cx, double cy, double r)
{
    double lim = (r + rb) * (1.0 + kAqSlack);
    return fabs(mx - cx) <= lim && fabs(my - cy) <= lim;
}

// A box as the traversal needs it, in one round of loads.
struct AqBox {
    double x, y, r;
    int leaf;
    int4 child;
};

__device__ __forceinline__ AqBox aq_box(const AQTree &t, int b)
{
    return AqBox{t.bcx[b], t.bcy[b], aq_rad(t, t.blev[b]), t.leaf[b], reinterpret_cast<const int4 *>(t.child4)[b]};
}

__device__ __forceinline__ int aq_child(const int4 &c, int q) { return q == 0 ? c.x : q == 1 ? c.y : q == 2 ? c.z : c.w; }

struct Guide {
    int l, ix, iy;        // level and integer position of the box at that level
};

__device__ Guide aq_guide(const AQTree &t, double cx, double cy, double r)
{
    Guide gd{0, 0, 0};
    AqBox bx = aq_box(t, 0);
    // a centre outside the root square: the root guides, so all its leaves
    // are examined (the paper takes c in the root)
    if (!(fabs(cx - bx.x) <= t.R0 && fabs(cy - bx.y) <= t.R0)) return gd;
    // r > |b0| stops at the root as well: descending could only shrink b
    while (!(r > 0.5 * aq_rad(t, gd.l)) && !bx.leaf) {
        int qx = cx >= bx.x, qy = cy >= bx.y;
        int c = aq_child(bx.child, qx + 2 * qy);
        if (c < 0) break;
        gd.ix = 2 * gd.ix + qx;
        gd.iy = 2 * gd.iy + qy;
        ++gd.l;
        bx = aq_box(t, c);
    }
    return gd;
}

// Calls emit(key, b) for every leaf b meeting C_r(c) (key 5b + 4) and, with
// regions, emit(key, -1) for every empty quadrant (key 5b + q) meeting it.
// A query is a chain of dependent loads, one lane each, so what counts is the
// rounds of them: the nine peers descend together (one round a level, where
// one after the other took nine), a box is one round, and the stack is LDS
// (stack[kAqThreads * i], this lane's entries), not scratch memory.
// 8192 squares of panel size on a star's tree, from one descent after the other
// with a scratch stack and 256 lanes a workgroup: area query 30.6 to 17.4 us,
// region lists 44 to 23, disk tests 50.5 to 28.
template <class F>
__device__ __forceinline__ void aq_visit(const AQTree &t, double cx, double cy, double r, bool regions, int *stack,
                                         int *err, F emit)
{
    Guide gd = aq_guide(t, cx, cy, r);
    int sp = 0;
    int n = 1 << gd.l;
    int pb[9], stop[9];       // box reached; quadrant where the descent ended early, or -1
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        int jx = gd.ix + i % 3 - 1, jy = gd.iy + i / 3 - 1;
        pb[i] = jx < 0 || jy < 0 || jx >= n || jy >= n ? -1 : 0;
        stop[i] = -1;
    }
    for (int sh = gd.l - 1; sh >= 0; --sh) {
        int c[9], q[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            q[i] = (((gd.ix + i % 3 - 1) >> sh) & 1) | ((((gd.iy + i / 3 - 1) >> sh) & 1) << 1);
            c[i] = t.child4[4 * max(pb[i], 0) + q[i]];
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            bool on = pb[i] >= 0 && stop[i] < 0;
            if (on && c[i] < 0) stop[i] = q[i];
            else if (on) pb[i] = c[i];
        }
    }
    int key[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        // ended early below a box with children: that empty quadrant; at a
        // leaf: the coarser leaf
        bool quad = pb[i] >= 0 && stop[i] >= 0 && !t.leaf[max(pb[i], 0)];
        key[i] = pb[i] < 0 ? -1 : kAqKeysPerBox * pb[i] + (quad ? stop[i] : 4);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        bool dup = key[i] < 0;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if (k < i) dup |= key[k] == key[i];
        if (dup) continue;
        int q = key[i] - kAqKeysPerBox * pb[i];
        if (q == 4) {
            stack[kAqThreads * sp++] = pb[i];
        } else if (regions) {
            double h = 0.5 * aq_rad(t, t.blev[pb[i]]);
            if (aq_may_meet(t.bcx[pb[i]] + ((q & 1) ? h : -h), t.bcy[pb[i]] + ((q & 2) ? h : -h), h, cx, cy, r))
                emit(key[i], -1);
        }
    }
    while (sp > 0) {
        int b = stack[kAqThreads * --sp];
        AqBox bx = aq_box(t, b);
        if (bx.leaf) {
            if (regions ? aq_may_meet(bx.x, bx.y, bx.r, cx, cy, r) : aq_meets(bx.x, bx.y, bx.r, cx, cy, r))
                emit(kAqKeysPerBox * b + 4, b);
            continue;
        }
        if (!aq_may_meet(bx.x, bx.y, bx.r, cx, cy, r)) continue;
        double h = 0.5 * bx.r;
        for (int q = 3; q >= 0; --q) {
            int c = aq_child(bx.child, q);
            if (c >= 0) {
                if (sp == t.stack) {           // cannot happen by the bound above; reported, not dropped silently
                    atomicOr(err, 1);
                    return;
                }
                stack[kAqThreads * sp++] = c;
            } else if (regions && aq_may_meet(bx.x + ((q & 1) ? h : -h), bx.y + ((q & 2) ? h : -h), h, cx, cy, r)) {
                emit(kAqKeysPerBox * b + q, -1);
            }
        }
    }
}

__global__ void __launch_bounds__(kAqThreads) k_area_query(AQTree t, int64_t n, const double *qx, const double *qy, const double *qr,
                             int32_t *cnt, const int64_t *start, int32_t *list, int *err)
{
    extern __shared__ int stack[];
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double r = qr[i];
    int32_t c = 0;
    if (r >= 0.0) {                             // negative or NaN radius: empty square
        int32_t *dst = list ? list + start[i] : nullptr;
        aq_visit(t, qx[i], qy[i], r, false, stack + threadIdx.x, err, [&](int, int b) {
            if (dst) dst[c] = b;
            ++c;
        });
    }
    if (!list) cnt[i] = c;
}

__global__ void __launch_bounds__(kAqThreads) k_region_lists(AQTree t, int64_t n, const double *x, const double *y, const double *rad,
                               double scale, int32_t *kcnt, const int64_t *kstart, int32_t *kcur,
                               int32_t *list, int *err)
{
    extern __shared__ int stack[];
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double r = rad[i] * scale;
    if (!(r >= 0.0)) return;
    aq_visit(t, x[i], y[i], r, true, stack + threadIdx.x, err, [&](int key, int) {
        if (!list) atomicAdd(&kcnt[key], 1);
        else list[kstart[key] + atomicAdd(&kcur[key], 1)] = (int32_t)i;
    });
}

// A point of the disk lies in the square and so in a leaf meeting it.  The
// leaves are taken with the widened test (the traversal's region mode, whose
// empty quadrants hold no points and are skipped), so that rounding in the
// stored box centres cannot drop a point on a leaf's edge; the point test
// itself is exact.
__global__ void __launch_bounds__(kAqThreads) k_points_near(AQTree t, int64_t n, const double *qx, const double *qy, const double *qr,
                              const int *pbeg, const int *pend, const double *px, const double *py,
                              int32_t *hit, int *err)
{
    extern __shared__ int stack[];
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x = qx[i], y = qy[i], r = qr[i];
    int32_t h = 0;
    if (r >= 0.0) {
        double r2 = r * r;
        aq_visit(t, x, y, r, true, stack + threadIdx.x, err, [&](int, int b) {
            if (b < 0) return;
            // four points' loads go out together
            constexpr int U = 4;
            int k1 = pend[b];
            for (int k0 = pbeg[b]; k0 < k1 && !h; k0 += U) {
                double dx[U], dy[U];
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    int k = min(k0 + i, k1 - 1);
                    dx[i] = px[k] - x;
                    dy[i] = py[k] - y;
                }
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (dx[i] * dx[i] + dy[i] * dy[i] <= r2) h = 1;
            }
        });
    }
    hit[i] = h;
}

// Region (key) holding the point clamped to the root square.  A square
// about a point of the root that holds the target holds the clamped point
// too, so the region's list has every candidate of the target.
__device__ int aq_region_of(const AQTree &t, double x, double y)
{
    x = fmin(fmax(x, t.bcx[0] - t.R0), t.bcx[0] + t.R0);
    y = fmin(fmax(y, t.bcy[0] - t.R0), t.bcy[0] + t.R0);
    int b = 0;
    for (AqBox bx = aq_box(t, 0); !bx.leaf; bx = aq_box(t, b)) {
        int q = (x >= bx.x) | ((y >= bx.y) << 1);
        int c = aq_child(bx.child, q);
        if (c < 0) return kAqKeysPerBox * b + q;
        b = c;
    }
    return kAqKeysPerBox * b + 4;
}

__global__ void k_associate(AQTree t, AQAssoc a, int64_t n, const double *tx, const double *ty, int32_t *out,
                            unsigned long long *nfail)
{
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    double x = tx[m], y = ty[m];
    int key = aq_region_of(t, x, y);
    // the host planner's rule, with its roundings (no contraction here)
    int best = -1;
    double bestd = 0.0;
    // four candidates' loads go out together
    constexpr int U = 4;
    int64_t e1 = a.cstart[key + 1];
    for (int64_t e0 = a.cstart[key]; e0 < e1; e0 += U) {
        int k[U], u[U];
        double px[U], py[U], pr[U];
#pragma unroll
        for (int i = 0; i < U; ++i) k[i] = a.clist[min(e0 + i, e1 - 1)];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            px[i] = a.cx[k[i]];
            py[i] = a.cy[k[i]];
            pr[i] = a.cr[k[i]];
            u[i] = a.ctr_user[k[i]];
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            // (past the end the last candidate is met again: no change)
            double dx = x - px[i], dy = y - py[i];
            double d2 = dx * dx + dy * dy;
            double lim = pr[i] * (1.0 + a.ea);
            if (d2 <= lim * lim && (best < 0 || d2 < bestd || (d2 == bestd && u[i] < best))) {
                best = u[i];
                bestd = d2;
            }
        }
    }
    out[m] = best;
    if (best >= 0) return;
    bool near = false;
    for (int64_t e = a.sstart[key]; e < a.sstart[key + 1]; ++e) {
        int j = a.slist[e];
        double dx = x - a.sx[j], dy = y - a.sy[j];
        double q = 0.25 * a.sh[j];
        if (dx * dx + dy * dy <= q * q) near = true;
    }
    if (near) atomicAdd(nfail, 1ull);
}

// Exclusive scan of n counts into start[0..n] (start[n], and *total, the sum):
// a block's counts, the blocks, then the counts within each block.
constexpr int kScanItems = 8, kScanThreads = 256, kScanBlock = kScanItems * kScanThreads;

__global__ void __launch_bounds__(kScanThreads) k_scan_sums(int64_t n, const int32_t *cnt, int64_t *bsum)
{
    __shared__ int64_t part[kScanThreads];
    int64_t i0 = (int64_t)blockIdx.x * kScanBlock, s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = i0 + k * kScanThreads + threadIdx.x;
        if (i < n) s += cnt[i];
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = kScanThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = part[0];
}

// Inclusive scan of one value per thread of a block.
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t *part)
{
    part[threadIdx.x] = v;
    __syncthreads();
    for (int h = 1; h < kScanThreads; h <<= 1) {
        int64_t add = (int)threadIdx.x >= h ? part[threadIdx.x - h] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    return part[threadIdx.x];
}

__global__ void __launch_bounds__(kScanThreads) k_scan_blocks(int64_t nb, int64_t *bsum, int64_t *last, int64_t *total)
{
    __shared__ int64_t part[kScanThreads];
    int64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        int64_t b = b0 + threadIdx.x, v = b < nb ? bsum[b] : 0;
        int64_t inc = block_scan(v, part);
        if (b < nb) bsum[b] = carry + inc - v;
        carry += part[kScanThreads - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) *last = *total = carry;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_write(int64_t n, const int32_t *cnt, const int64_t *bsum, int64_t *start)
{
    __shared__ int64_t part[kScanThreads];
    int64_t i0 = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems, s = 0;
    int32_t c[kScanItems];
    for (int k = 0; k < kScanItems; ++k) {
        c[k] = i0 + k < n ? cnt[i0 + k] : 0;
        s += c[k];
    }
    int64_t at = bsum[blockIdx.x] + block_scan(s, part) - s;
    for (int k = 0; k < kScanItems; ++k) {
        if (i0 + k < n) start[i0 + k] = at;
        at += c[k];
    }
}

size_t aq_lds_bytes(const AQTree &t) { return sizeof(int) * kAqThreads * (size_t)t.stack; }

unsigned aq_blocks(int64_t n) { return (unsigned)((n + kAqThreads - 1) / kAqThreads); }

}  // namespace

size_t scan_scratch(int64_t n) { return sizeof(int64_t) * (size_t)((n + kScanBlock - 1) / kScanBlock + 1); }

hipError_t launch_scan(int64_t n, const int32_t *cnt, int64_t *start, int64_t *total, void *scratch, hipStream_t s)
{
    int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    int64_t *bsum = static_cast<int64_t *>(scratch);
    if (nb > 0) k_scan_sums<<<(unsigned)nb, kScanThreads, 0, s>>>(n, cnt, bsum);
    k_scan_blocks<<<1, kScanThreads, 0, s>>>(nb, bsum, start + n, total);
    if (nb > 0) k_scan_write<<<(unsigned)nb, kScanThreads, 0, s>>>(n, cnt, bsum, start);
    return hipGetLastError();
}

hipError_t launch_area_query(const AQTree &t, int64_t n, const double *qx, const double *qy,
                             const double *qr, int32_t *cnt, const int64_t *start, int32_t *list,
                             int *err, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_area_query<<<aq_blocks(n), kAqThreads, aq_lds_bytes(t), s>>>(t, n, qx, qy, qr, cnt, start, list, err);
    return hipGetLastError();
}

hipError_t launch_region_lists(const AQTree &t, int64_t n, const double *x, const double *y,
                               const double *rad, double scale, int32_t *kcnt,
                               const int64_t *kstart, int32_t *kcur, int32_t *list, int *err,
                               hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_region_lists<<<aq_blocks(n), kAqThreads, aq_lds_bytes(t), s>>>(t, n, x, y, rad, scale, kcnt, kstart, kcur, list, err);
    return hipGetLastError();
}

hipError_t launch_points_near(const AQTree &t, int64_t n, const double *qx, const double *qy,
                              const double *qr, const int *pbeg, const int *pend, const double *px,
                              const double *py, int32_t *hit, int *err, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_points_near<<<aq_blocks(n), kAqThreads, aq_lds_bytes(t), s>>>(t, n, qx, qy, qr, pbeg, pend, px, py, hit, err);
    return hipGetLastError();
}

hipError_t launch_associate(const AQTree &t, const AQAssoc &a, int64_t n, const double *tx,
                            const double *ty, int32_t *out, unsigned long long *nfail,
                            hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_associate<<<aq_blocks(n), kAqThreads, 0, s>>>(t, a, n, tx, ty, out, nfail);
    return hipGetLastError();
}

}  // namespace qbx
