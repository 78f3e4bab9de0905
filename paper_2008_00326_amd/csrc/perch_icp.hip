// gfx950 kernels for the steps around pose scoring: ICP refinement of
// candidate poses (Sec. IV-A "Parallel M2M GICP"; point-to-point, as in the
// 3-DoF experiments of Sec. VI-A) and 6-DoF pose proposals (Sec. V-B).
// Geometry in binary64 without FMA contraction (built with
// -ffp-contract=off), as the oracle computes it.

#include "perch_device.h"

namespace perch {

// ------------------------------------------------------------------ ICP refinement

// Per-iteration ICP sums over the matched pairs (q, c): n, q (3), c (3),
// q q^T (9, row-major), q c^T (9, row-major).
constexpr int kIcpSums = 25;
// GICP: 21 upper entries of the 6x6 Gauss-Newton matrix, then 6 of its
// right-hand side, in 64-bit fixed point (times 1024, rounded).
constexpr int kGicpSums = 27;
constexpr int kRedSums = 28;

// Sum of a lane value over the wave (exact 64-bit integers; every lane
// active), in DPP adds: within rows of 16, then across the rows into lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ long long dpp_add64(long long x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((unsigned long long)x >> 32), CTRL, ROWS, 0xF, false);
    return x + (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}

// Collects wave-wide sums, sum j in lane j.
struct WaveSums {
    int lane, lo, hi;
    __device__ __forceinline__ explicit WaveSums(int l) : lane(l), lo(0), hi(0) {}
    __device__ __forceinline__ void set(int j, long long x)
    {
        x = dpp_add64<0x111, 0xF>(x);      // row_shr 1, 2, 4, 8: lane 15 of each row holds the row's sum
        x = dpp_add64<0x112, 0xF>(x);
        x = dpp_add64<0x114, 0xF>(x);
        x = dpp_add64<0x118, 0xF>(x);
        x = dpp_add64<0x142, 0xA>(x);      // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
        x = dpp_add64<0x143, 0xC>(x);
        const int tl = __builtin_amdgcn_readlane((int)(uint32_t)x, 63);
        const int th = __builtin_amdgcn_readlane((int)(uint32_t)((unsigned long long)x >> 32), 63);
        lo = lane == j ? tl : lo;
        hi = lane == j ? th : hi;
    }
    __device__ __forceinline__ long long value() const
    {
        return (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
    }
};

// The ICP target in tiles of 4x4 pixels, 16 lanes each: the tile's points
// side by side as (X, Y, Z, -), Z = kNoPoint where there is none that can
// match (label volumes: off the label), and their box (1/16 mm), {lo, -} and
// {hi, -}, lo > hi without a point.  With the label folded in here the search
// needs no second, dependent load where a nearer point turns up.  Also zeroes
// the cursor.
__global__ __launch_bounds__(256) void icp_target_kernel(IcpArgs a)
{
    const SceneDev &s = a.s;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.cursor[0] = 0;
    const int tiles_x = (s.W + kIcpTile - 1) / kIcpTile, tiles_y = (s.H + kIcpTile - 1) / kIcpTile;
    const int t = blockIdx.x * 16 + (threadIdx.x >> 4), lane = threadIdx.x & 15;
    const int i = (t % tiles_x) * kIcpTile + (lane & 3), j = (t / tiles_x) * kIcpTile + (lane >> 2);
    const bool label_mode = (s.flags & (3u << 4)) == (2u << 4);
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-(1 << 30), -(1 << 30), -(1 << 30)};
    int4 o = make_int4(0, 0, kNoPoint, 0);
    if (i < s.W && j < s.H) {
        const int pix = j * s.W + i;
        o = gld(s.opt + pix);
        if (o.z != kNoPoint && (!(label_mode && s.labels) || gld(s.labels + pix) == a.label)) {
            lo[0] = hi[0] = o.x;
            lo[1] = hi[1] = o.y;
            lo[2] = hi[2] = o.z;
        } else {
            o.z = kNoPoint;
        }
    }
    if (t < tiles_x * tiles_y) a.target[16 * (size_t)t + lane] = o;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        for (int off = 8; off > 0; off >>= 1) {
            lo[c] = min(lo[c], __shfl_xor(lo[c], off));
            hi[c] = max(hi[c], __shfl_xor(hi[c], off));
        }
    if (lane == 0 && t < tiles_x * tiles_y) {
        a.boxes[2 * t] = make_int4(lo[0], lo[1], lo[2], 0);
        a.boxes[2 * t + 1] = make_int4(hi[0], hi[1], hi[2], 0);
    }
}

// Per tile, the box of the 4x4 tiles from it on (16x16 pixels, clipped to the
// image), after the tiles' own: one test then rules out sixteen.
__global__ __launch_bounds__(256) void icp_target_wide_kernel(IcpArgs a)
{
    const int tiles_x = (a.s.W + kIcpTile - 1) / kIcpTile, tiles_y = (a.s.H + kIcpTile - 1) / kIcpTile;
    const int t = blockIdx.x * 256 + threadIdx.x, n = tiles_x * tiles_y;
    if (t >= n) return;
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    int4 lo = make_int4(1 << 30, 1 << 30, 1 << 30, 0), hi = make_int4(-(1 << 30), -(1 << 30), -(1 << 30), 0);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        // past the edge: the last tile again
        const int u = min(ty + (k >> 2), tiles_y - 1) * tiles_x + min(tx + (k & 3), tiles_x - 1);
        const int4 l = gld(a.boxes + 2 * u), h = gld(a.boxes + 2 * u + 1);
        lo = make_int4(min(lo.x, l.x), min(lo.y, l.y), min(lo.z, l.z), 0);
        hi = make_int4(max(hi.x, h.x), max(hi.y, h.y), max(hi.z, h.z), 0);
    }
    a.boxes[2 * (n + t)] = lo;
    a.boxes[2 * (n + t) + 1] = hi;
}

// v of lane K of the quad, for the whole quad.
template <int K>
__device__ __forceinline__ int quad_lane(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, K * 0x55, 0xF, 0xF, false);    // quad_perm [K, K, K, K]
}
// Least value over the four lanes of a quad.
__device__ __forceinline__ int quad_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));    // quad_perm [1, 0, 3, 2]
    return min(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false)); // quad_perm [2, 3, 0, 1]
}

// 1 / x for whole x >= 1: v_rcp_f64 and one Newton step, within a relative
// 2^-48 (over 1 .. 65,536: 2^-24.4 before the step, 2^-48.8 after), far inside
// the pixel of margin of what it bounds.
__device__ __forceinline__ double icp_rcp(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    return y * (2.0 - x * y);
}

// Pixels [w[0], w[2]] x [w[1], w[3]], inside `box`, that hold every observed
// point within r of q (1/16 mm); false when there are none.  An observed
// point at depth d (mm) with |Xq - qx| <= r has rint(kx[i] d) in
// [qx - r, qx + r], so kx[i] d lies within half a unit of that range, for d
// in [(qz - r) / 16, (qz + r) / 16]; one pixel of margin on each side, far
// above the rounding.  The quad's lane `sub` computes w[sub], the upper
// bounds as the negated lower bounds of the mirrored axis.
__device__ __forceinline__ bool icp_window(const SceneDev &s, int4 q, int r, const int *box, int sub, int w[4])
{
    const int dlo = q.z - r <= 16 ? 1 : (q.z - r + 15) >> 4;
    const int dhi = min(65534, (q.z + r) >> 4);
    if (q.z + r < 16 || dlo > dhi) return false;
    const double ilo = icp_rcp((double)dlo), ihi = icp_rcp((double)dhi);
    const bool row = sub & 1, up = sub & 2;
    const double f16 = (double)(row ? s.fy : s.fx) / 16.0, c = (double)(row ? s.cy : s.cx);
    const int qv = row ? q.y : q.x;
    const double e = (double)((up ? -qv : qv) - r) - 0.5;
    const double v = (up ? -c : c) + f16 * fmin(e * ilo, e * ihi);
    const int g = (int)floor(fmax(fmin(v, 1e8), -1e8)) - 1;
    const int bound = up ? min(-g, row ? box[3] : box[2]) : max(g, row ? box[1] : box[0]);
    w[0] = quad_lane<0>(bound);
    w[1] = quad_lane<1>(bound);
    w[2] = quad_lane<2>(bound);
    w[3] = quad_lane<3>(bound);
    return w[0] <= w[2] && w[1] <= w[3];
}

// Box of target points.
struct IcpBox {
    int3 lo, hi;
};
__device__ __forceinline__ IcpBox icp_box(const int4 *boxes, int t)
{
    return IcpBox{opt_at(boxes, (uint32_t)(2 * t)), opt_at(boxes, (uint32_t)(2 * t + 1))};
}

// Nearest observed point of q (1/16 mm) within rq, ties to the lower pixel
// index, or -1; in label mode only pixels carrying the label count.  Four
// lanes (a quad, `sub` 0..3) per point, every value but the lane's own tiles
// alike in all four.  A first guess (`seed`, the match of the previous
// update, else the pixel q projects to) bounds the distance, and with it the
// window of pixels that can hold a nearer point: a surface point's nearest
// neighbour lies a few mm away where rq is 20 mm.  The window's 4x4 tiles go
// by their boxes of target points, the nearest first and only while one comes
// as near as the best; sixteen tiles through one wider box before, so that a
// point with no match within rq costs a few box tests.
//
// What bounds it is VALU issue, the search's own integer work; with one lane
// per point it was the rate of distinct cache lines (every load of a scan
// touched 64), where a quad reads 64 contiguous bytes per load.
__device__ __forceinline__ int icp_nn(const IcpArgs &a, int4 q, int seed, int sub)
{
    const SceneDev &s = a.s;
    if (q.z + a.rq < 16 || a.box[0] > a.box[2] || a.box[1] > a.box[3]) return -1;
    const uint32_t cap = (uint32_t)a.rq2 + 1;
    // the best so far: squared distance and pixel; nothing yet: above rq^2
    int bd2 = a.rq2 + 1, bpix = -1;
    auto d2_of = [&](int3 o) { return capped_d2(o.x - q.x, o.y - q.y, o.z - q.z, cap); };
    const int tiles_x = (s.W + kIcpTile - 1) / kIcpTile;
    if (seed >= 0) {
        bd2 = d2_of(opt_at(s.opt, (uint32_t)seed));
        bpix = seed;
    } else if (q.z > 0) {
        const float iz = 1.0f / (float)q.z;
        const float u = s.cx + s.fx * (float)q.x * iz, v = s.cy + s.fy * (float)q.y * iz;
        const int i = (int)fmaxf(fminf(rintf(u), (float)a.box[2]), (float)a.box[0]);
        const int j = (int)fmaxf(fminf(rintf(v), (float)a.box[3]), (float)a.box[1]);
        const int t = (j / kIcpTile) * tiles_x + i / kIcpTile;
        bd2 = d2_of(opt_at(a.target, (uint32_t)(16 * t + kIcpTile * (j % kIcpTile) + i % kIcpTile)));
        bpix = j * s.W + i;
    }
    // every point at least as near as the best lies within r: r^2 >= its d2
    int r = a.rq;
    if (bd2 <= a.rq2) r = min(a.rq, (int)sqrtf((float)bd2) + 1);
    int w[4];
    if (icp_window(s, q, r, a.box, sub, w)) {
        const int tx0 = w[0] / kIcpTile, ty0 = w[1] / kIcpTile, tx1 = w[2] / kIcpTile, ty1 = w[3] / kIcpTile;
        const int n_tiles = tiles_x * ((s.H + kIcpTile - 1) / kIcpTile);
        // blocks of 4x4 wide boxes, each of 4x4 tiles: the quad's lane `sub`
        // holds column `sub` of either, as keys (box distance << 4 | index)
        constexpr int kNone = 0x7FFFFFFF;
        for (int by = ty0; by <= ty1; by += 16)
            for (int bx = tx0; bx <= tx1; bx += 16) {
                int wide[4], tile[4];
                auto test = [&](int first, int x, int y0, int step, int key[4]) {
                    IcpBox box[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        box[k] = icp_box(a.boxes, first + min(y0 + step * k, ty1) * tiles_x + min(x, tx1));
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const IcpBox &b = box[k];
                        const int d2 = capped_d2(max(max(b.lo.x - q.x, q.x - b.hi.x), 0),
                                                 max(max(b.lo.y - q.y, q.y - b.hi.y), 0),
                                                 max(max(b.lo.z - q.z, q.z - b.hi.z), 0), cap);
                        key[k] = x <= tx1 && y0 + step * k <= ty1 ? (d2 << 4) | (4 * k + sub) : kNone;
                    }
                };
                // the quad's nearest key of those left, taken out; false when
                // none comes as near as the best (of points within rq: a box
                // or point at the cap is out of reach)
                auto next = [&](int key[4], int &got) {
                    got = quad_min(min(min(key[0], key[1]), min(key[2], key[3])));
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (key[k] == got) key[k] = kNone;
                    return (got >> 4) <= min(bd2, a.rq2);
                };
                int c, f;
                test(n_tiles, bx + 4 * sub, by, 4, wide);
                while (next(wide, c)) {
                    const int cx = bx + 4 * (c & 3), cy = by + (c & 12);
                    test(0, cx + sub, cy, 1, tile);
                    while (next(tile, f)) {
                        const int tx = cx + (f & 3), ty = cy + ((f >> 2) & 3);
                        int3 o[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            o[k] = opt_at(a.target, (uint32_t)(16 * (ty * tiles_x + tx) + 4 * k + sub));
                        // lane `sub` reads column `sub`: the key's low bits count the tile's pixels row by row
                        int m = kNone;
#pragma unroll
                        for (int k = 0; k < 4; ++k) m = min(m, (d2_of(o[k]) << 4) | (4 * k + sub));
                        m = quad_min(m);
                        const int pix = (kIcpTile * ty + ((m >> 2) & 3)) * s.W + kIcpTile * tx + (m & 3);
                        if ((m >> 4) < bd2 || ((m >> 4) == bd2 && pix < bpix)) {
                            bd2 = m >> 4;
                            bpix = pix;
                        }
                    }
                }
            }
    }
    return bd2 <= a.rq2 ? bpix : -1;
}

// One ICP update from the sums (n, q, c, q q^T, q c^T): the increment about
// the source centroid mq composed into (A, b), b in 1/16 mm.  3-DoF: the
// planar Procrustes rotation about the unit axis u and the centroid moved
// within the plane normal to u; 6-DoF: a Gauss-Newton step of the
// linearised rotation, (tr(S) I - S) w' = w, mapped to a rotation by the
// unit quaternion (1, w'/2) and the centroid moved onto mc.  Every step
// uses + - * / and sqrt only, left to right.  Returns 1 when the 6-DoF
// system is singular (nothing changes).
__device__ __noinline__ int icp_update(const long long *z, int dof, const double u[3], double *A, double *b)
{
    const double n = (double)z[0];
    double mq[3], mc[3], S[3][3], H[3][3];
    for (int a = 0; a < 3; ++a) {
        mq[a] = (double)z[1 + a] / n;
        mc[a] = (double)z[4 + a] / n;
    }
    for (int a = 0; a < 3; ++a)
        for (int c = 0; c < 3; ++c) {
            S[a][c] = (double)z[7 + 3 * a + c] - ((double)z[1 + a] * (double)z[1 + c]) / n;
            H[a][c] = (double)z[16 + 3 * a + c] - ((double)z[1 + a] * (double)z[4 + c]) / n;
        }
    const double w[3] = {H[1][2] - H[2][1], H[2][0] - H[0][2], H[0][1] - H[1][0]};
    double R[3][3], mp[3];
    if (dof == 3) {
        double Hu[3];
        for (int a = 0; a < 3; ++a) Hu[a] = (H[a][0] * u[0] + H[a][1] * u[1]) + H[a][2] * u[2];
        const double uHu = (u[0] * Hu[0] + u[1] * Hu[1]) + u[2] * Hu[2];
        const double Ap = ((H[0][0] + H[1][1]) + H[2][2]) - uHu;
        const double B = (u[0] * w[0] + u[1] * w[1]) + u[2] * w[2];
        const double h = sqrt(Ap * Ap + B * B);
        double co = 1.0, si = 0.0;
        if (h > 0.0) {
            co = Ap / h;
            si = B / h;
        }
        const double Kx[3][3] = {{0.0, -u[2], u[1]}, {u[2], 0.0, -u[0]}, {-u[1], u[0], 0.0}};
        for (int a = 0; a < 3; ++a)
            for (int c = 0; c < 3; ++c) R[a][c] = ((a == c ? co : 0.0) + si * Kx[a][c]) + ((1.0 - co) * u[a]) * u[c];
        const double d[3] = {mc[0] - mq[0], mc[1] - mq[1], mc[2] - mq[2]};
        const double ud = (u[0] * d[0] + u[1] * d[1]) + u[2] * d[2];
        for (int a = 0; a < 3; ++a) mp[a] = mq[a] + (d[a] - ud * u[a]);
    } else {
        const double tr = (S[0][0] + S[1][1]) + S[2][2];
        double M[3][3];
        for (int a = 0; a < 3; ++a)
            for (int c = 0; c < 3; ++c) M[a][c] = (a == c ? tr : 0.0) - S[a][c];
        double adj[3][3];
        adj[0][0] = M[1][1] * M[2][2] - M[1][2] * M[2][1];
        adj[0][1] = M[0][2] * M[2][1] - M[0][1] * M[2][2];
        adj[0][2] = M[0][1] * M[1][2] - M[0][2] * M[1][1];
        adj[1][0] = M[1][2] * M[2][0] - M[1][0] * M[2][2];
        adj[1][1] = M[0][0] * M[2][2] - M[0][2] * M[2][0];
        adj[1][2] = M[0][2] * M[1][0] - M[0][0] * M[1][2];
        adj[2][0] = M[1][0] * M[2][1] - M[1][1] * M[2][0];
        adj[2][1] = M[0][1] * M[2][0] - M[0][0] * M[2][1];
        adj[2][2] = M[0][0] * M[1][1] - M[0][1] * M[1][0];
        const double det = (M[0][0] * adj[0][0] + M[0][1] * adj[1][0]) + M[0][2] * adj[2][0];
        if (!(det > 0.0)) return 1;
        double h[3];
        for (int a = 0; a < 3; ++a) h[a] = (((adj[a][0] * w[0] + adj[a][1] * w[1]) + adj[a][2] * w[2]) / det) / 2.0;
        const double r = sqrt(1.0 + ((h[0] * h[0] + h[1] * h[1]) + h[2] * h[2]));
        const double qw = 1.0 / r, qx = h[0] / r, qy = h[1] / r, qz = h[2] / r;
        R[0][0] = 1.0 - 2.0 * (qy * qy + qz * qz);
        R[0][1] = 2.0 * (qx * qy - qz * qw);
        R[0][2] = 2.0 * (qx * qz + qy * qw);
        R[1][0] = 2.0 * (qx * qy + qz * qw);
        R[1][1] = 1.0 - 2.0 * (qx * qx + qz * qz);
        R[1][2] = 2.0 * (qy * qz - qx * qw);
        R[2][0] = 2.0 * (qx * qz - qy * qw);
        R[2][1] = 2.0 * (qy * qz + qx * qw);
        R[2][2] = 1.0 - 2.0 * (qx * qx + qy * qy);
        for (int a = 0; a < 3; ++a) mp[a] = mc[a];
    }
    double An[9], bn[3];
    const double e[3] = {b[0] - mq[0], b[1] - mq[1], b[2] - mq[2]};
    for (int a = 0; a < 3; ++a) {
        for (int c = 0; c < 3; ++c) An[3 * a + c] = (R[a][0] * A[c] + R[a][1] * A[3 + c]) + R[a][2] * A[6 + c];
        bn[a] = ((R[a][0] * e[0] + R[a][1] * e[1]) + R[a][2] * e[2]) + mp[a];
    }
    for (int k = 0; k < 9; ++k) A[k] = An[k];
    for (int k = 0; k < 3; ++k) b[k] = bn[k];
    return 0;
}

// ------------------------------------------------------------------ GICP

// int4 arrays per work-group slot: source points, mapped points (with the
// match), and for GICP the source normals.
__host__ __device__ constexpr int gicp_slots(int method) { return method == 1 ? 3 : 2; }

// Integer normal direction of the point at pixel (i, j) of a depth image
// (depth(i', j') in mm, 0 = none): the cross product of the differences of
// the 1/16 mm points of the row and column neighbours, when all four exist
// inside the image, lie within `gap` mm of the pixel's depth and differ by
// at most 2^14 units per axis; 0 when there is none.
template <class Depth>
__device__ int pixel_normal(const SceneDev &s, int i, int j, int gap, Depth depth, int c[3])
{
    if (i < 1 || j < 1 || i > s.W - 2 || j > s.H - 2) return 0;
    const int d = depth(i, j);
    const int ni[4] = {i - 1, i + 1, i, i}, nj[4] = {j, j, j - 1, j + 1};
    int p[4][3];
    for (int k = 0; k < 4; ++k) {
        const int dn = depth(ni[k], nj[k]);
        if (d == 0 || dn == 0 || dn - d > gap || d - dn > gap) return 0;
        p[k][0] = (int)rint(gld(s.kx + ni[k]) * (double)dn);
        p[k][1] = (int)rint(gld(s.ky + nj[k]) * (double)dn);
        p[k][2] = 16 * dn;
    }
    int ex[3], ey[3];
    for (int a = 0; a < 3; ++a) {
        ex[a] = p[1][a] - p[0][a];
        ey[a] = p[3][a] - p[2][a];
        if (ex[a] > 16384 || ex[a] < -16384 || ey[a] > 16384 || ey[a] < -16384) return 0;
    }
    c[0] = ex[1] * ey[2] - ex[2] * ey[1];
    c[1] = ex[2] * ey[0] - ex[0] * ey[2];
    c[2] = ex[0] * ey[1] - ex[1] * ey[0];
    return c[0] != 0 || c[1] != 0 || c[2] != 0;
}

__device__ __forceinline__ void unit_of(const int c[3], double n[3])
{
    const double x = (double)c[0], y = (double)c[1], z = (double)c[2];
    const double l = sqrt((x * x + y * y) + z * z);
    n[0] = x / l;
    n[1] = y / l;
    n[2] = z / l;
}

// The kGicpSums terms of one match q -> c per lane, summed over the wave
// (lanes without a match, `has` false, add nothing): with the plane covariances
// I - (1 - 1/1024) n n^T of the source normal turned by A and of the target
// normal (I without one), M = (C_a + C_b)^-1 by the adjugate, K = -[q - mu]x
// and e = c - q, the Gauss-Newton matrix [[K^T M K, K^T M], [M K, M]] (upper
// entries row by row) and right-hand side [K^T M e; M e], times 1024, rounded.
__device__ __forceinline__ void gicp_terms(bool has, int4 q, int3 c, const long long mu[3], int has_a, const double na[3],
                                           int has_b, const double nb[3], const double *A, WaveSums &w)
{
    const double eps = 1.0 / 1024.0;
    double ra[3] = {0.0, 0.0, 0.0};
    if (has_a)
        for (int r = 0; r < 3; ++r) ra[r] = (A[3 * r] * na[0] + A[3 * r + 1] * na[1]) + A[3 * r + 2] * na[2];
    const double ka = has_a ? 1.0 - eps : 0.0, kb = has_b ? 1.0 - eps : 0.0;
    double S[3][3];
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) {
            const double sa = (r == k ? 1.0 : 0.0) - ka * (ra[r] * ra[k]);
            const double sb = (r == k ? 1.0 : 0.0) - kb * (nb[r] * nb[k]);
            S[r][k] = sa + sb;
        }
    double adj[3][3];
    adj[0][0] = S[1][1] * S[2][2] - S[1][2] * S[2][1];
    adj[0][1] = S[0][2] * S[2][1] - S[0][1] * S[2][2];
    adj[0][2] = S[0][1] * S[1][2] - S[0][2] * S[1][1];
    adj[1][0] = S[1][2] * S[2][0] - S[1][0] * S[2][2];
    adj[1][1] = S[0][0] * S[2][2] - S[0][2] * S[2][0];
    adj[1][2] = S[0][2] * S[1][0] - S[0][0] * S[1][2];
    adj[2][0] = S[1][0] * S[2][1] - S[1][1] * S[2][0];
    adj[2][1] = S[0][1] * S[2][0] - S[0][0] * S[2][1];
    adj[2][2] = S[0][0] * S[1][1] - S[0][1] * S[1][0];
    const double det = (S[0][0] * adj[0][0] + S[0][1] * adj[1][0]) + S[0][2] * adj[2][0];
    double M[3][3];
    for (int r = 0; r < 3; ++r)
        for (int k = 0; k < 3; ++k) M[r][k] = adj[r][k] / det;
    const double x = (double)((long long)q.x - mu[0]), y = (double)((long long)q.y - mu[1]),
                 z = (double)((long long)q.z - mu[2]);
    const double Kq[3][3] = {{0.0, z, -y}, {-z, 0.0, x}, {y, -x, 0.0}};
    const double e[3] = {(double)(c.x - q.x), (double)(c.y - q.y), (double)(c.z - q.z)};
    double MK[3][3], Me[3];
    for (int r = 0; r < 3; ++r) {
        for (int k = 0; k < 3; ++k) MK[r][k] = (M[r][0] * Kq[0][k] + M[r][1] * Kq[1][k]) + M[r][2] * Kq[2][k];
        Me[r] = (M[r][0] * e[0] + M[r][1] * e[1]) + M[r][2] * e[2];
    }
    int j = 0;
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int k = r; k < 6; ++k) {
            double v;
            if (r < 3 && k < 3) v = (Kq[0][r] * MK[0][k] + Kq[1][r] * MK[1][k]) + Kq[2][r] * MK[2][k];
            else if (r < 3) v = MK[k - 3][r];
            else v = M[r - 3][k - 3];
            w.set(j++, has ? (long long)rint(v * 1024.0) : 0);
        }
#pragma unroll
    for (int r = 0; r < 3; ++r)
        w.set(j++, has ? (long long)rint(((Kq[0][r] * Me[0] + Kq[1][r] * Me[1]) + Kq[2][r] * Me[2]) * 1024.0) : 0);
#pragma unroll
    for (int r = 0; r < 3; ++r) w.set(j++, has ? (long long)rint(Me[r] * 1024.0) : 0);
}

// The GICP update from the fixed-point sums: H w = g by Cholesky (a pivot
// <= 0 returns 1, nothing changes), the rotation the unit quaternion
// (1, w/2) normalised, and (A, b) <- (Rc A, Rc (b - mu) + mu + t).
__device__ __noinline__ int gicp_update(const long long *z, const long long mu[3], double *A, double *b)
{
    double Hm[6][6], g[6];
    int t = 0;
    for (int r = 0; r < 6; ++r)
        for (int k = r; k < 6; ++k) {
            Hm[r][k] = (double)z[t++] / 1024.0;
            Hm[k][r] = Hm[r][k];
        }
    for (int r = 0; r < 6; ++r) g[r] = (double)z[t++] / 1024.0;
    double L[6][6];
    for (int r = 0; r < 6; ++r)
        for (int k = 0; k < 6; ++k) L[r][k] = 0.0;
    for (int jj = 0; jj < 6; ++jj) {
        double sjj = Hm[jj][jj];
        for (int k = 0; k < jj; ++k) sjj = sjj - L[jj][k] * L[jj][k];
        if (!(sjj > 0.0)) return 1;
        L[jj][jj] = sqrt(sjj);
        for (int i = jj + 1; i < 6; ++i) {
            double sij = Hm[i][jj];
            for (int k = 0; k < jj; ++k) sij = sij - L[i][k] * L[jj][k];
            L[i][jj] = sij / L[jj][jj];
        }
    }
    double yv[6], xv[6];
    for (int i = 0; i < 6; ++i) {
        double v = g[i];
        for (int k = 0; k < i; ++k) v = v - L[i][k] * yv[k];
        yv[i] = v / L[i][i];
    }
    for (int i = 5; i >= 0; --i) {
        double v = yv[i];
        for (int k = i + 1; k < 6; ++k) v = v - L[k][i] * xv[k];
        xv[i] = v / L[i][i];
    }
    const double h[3] = {xv[0] / 2.0, xv[1] / 2.0, xv[2] / 2.0};
    const double r = sqrt(1.0 + ((h[0] * h[0] + h[1] * h[1]) + h[2] * h[2]));
    const double qw = 1.0 / r, qx = h[0] / r, qy = h[1] / r, qz = h[2] / r;
    double R[3][3];
    R[0][0] = 1.0 - 2.0 * (qy * qy + qz * qz);
    R[0][1] = 2.0 * (qx * qy - qz * qw);
    R[0][2] = 2.0 * (qx * qz + qy * qw);
    R[1][0] = 2.0 * (qx * qy + qz * qw);
    R[1][1] = 1.0 - 2.0 * (qx * qx + qz * qz);
    R[1][2] = 2.0 * (qy * qz - qx * qw);
    R[2][0] = 2.0 * (qx * qz - qy * qw);
    R[2][1] = 2.0 * (qy * qz + qx * qw);
    R[2][2] = 1.0 - 2.0 * (qx * qx + qy * qy);
    double An[9], bn[3];
    const double m[3] = {(double)mu[0], (double)mu[1], (double)mu[2]};
    const double e[3] = {b[0] - m[0], b[1] - m[1], b[2] - m[2]};
    for (int a = 0; a < 3; ++a) {
        for (int c = 0; c < 3; ++c) An[3 * a + c] = (R[a][0] * A[c] + R[a][1] * A[3 + c]) + R[a][2] * A[6 + c];
        bn[a] = (((R[a][0] * e[0] + R[a][1] * e[1]) + R[a][2] * e[2]) + m[a]) + xv[3 + a];
    }
    for (int k = 0; k < 9; ++k) A[k] = An[k];
    for (int k = 0; k < 3; ++k) b[k] = bn[k];
    return 0;
}

// ICP refinement (Sec. IV-A "Parallel M2M GICP"; point-to-point): one pose
// per work-group at a time, taken through a cursor.  The pose is rendered
// into the work-group's device tile, its rendered points (R minus C on the
// ICP stride grid) collected, then each iteration maps them by the current
// transform (rounded to 1/16 mm), stops when no mapped point moved, matches
// each to its nearest observed point within rho (four lanes per point), sums
// the pairs exactly in int64 and updates the transform on one thread.
// Measured (640x480, rho 20 mm, ten updates, about 900 source points): 1,600
// 3-DoF poses against a label 25.2 -> 2.6 ms, 128 GICP poses of a 20k-triangle
// mesh 12.6 -> 0.9 ms; before, a wave scanned the whole window of each point
// and computed each GICP term set once per match.  Of a pose's time now: the
// search 70 %, the sums 18 %, the raster 5 %.  Full launches issue vector
// instructions at 0.61-0.63 of the card's rate; 32 (GICP 42) of the 128
// registers' worth is spilled, raster, normals, search and sums sharing them.
template <int BLOCK, bool GICP>
__global__ __launch_bounds__(BLOCK, 4) void icp_kernel(IcpArgs a)
{
    constexpr int NW = BLOCK / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SceneDev &s = a.s;
    const MeshDev &m = a.m;
    extern __shared__ uint32_t icp_lds[];
    __shared__ int s_pose, s_n, s_box[4], s_changed, s_stop;
    __shared__ long long s_red[NW][kRedSums], s_tot[kRedSums];
    __shared__ double s_A[9], s_b[3], s_u[3];
    __shared__ long long s_mu[3];
    uint32_t *tile = a.tiles + (size_t)blockIdx.x * s.W * s.H;
    int4 *src = a.pts + (size_t)blockIdx.x * (gicp_slots(a.method)) * a.pts_cap;
    int4 *qb = src + a.pts_cap;
    int4 *nrm = qb + a.pts_cap;            // GICP: integer source normals (x, y, z, has)
    constexpr bool gicp = GICP;
    const int gap = a.rq >> 4;
    const bool mark = (s.flags & 2u) != 0;
    const bool label_mode = (s.flags & (3u << 4)) == (2u << 4);
    // Poses come through the cursor.  The loop is rotated by hand so that
    // its condition is a wave-uniform value (readfirstlane of the LDS copy)
    // and no branch on the thread index heads it; every exit from the
    // iteration loop below tests a readfirstlane value too.
    if (tid == 0) s_pose = atomicAdd(a.cursor, 1);
    __syncthreads();
    for (int p = __builtin_amdgcn_readfirstlane(s_pose); p < a.n;) {
        float P[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) P[k] = a.poses[12 * (size_t)p + k];
        if (tid == 0) {
            double umin, umax, vmin, vmax, zmin, zmax;
            int x0 = 0, y0 = 0, w = 0, h = 0;
            project_box(P, m.lo, m.hi, 0.0, s, &umin, &umax, &vmin, &vmax, &zmin, &zmax);
            if (zmin >= 100.0) {
                clip_box(umin, umax, vmin, vmax, s.W, s.H, &x0, &y0, &w, &h);
                // Nothing in reach: every rendered point lies on a pixel of the
                // tile at depth >= zmin - 1/2 (depths are rounded to whole mm),
                // and a match lies within rho + 1/4 mm of it (points are rounded
                // to 1/16 mm), so its pixel is within
                // f (rho + 1/4) sqrt(1 + t^2) / (zmin - 1/2 - rho - 1/4) of the
                // tile (t the tile's largest ray slope), plus one.  When that
                // grown tile misses the target box, no point can match: the
                // pose comes back unchanged, as the iteration would return it.
                const double rp = (double)a.rq / 16.0 + 0.25;
                const double zn = zmin - 0.5;
                if (w > 0 && zn - rp > 1.0) {
                    const double tx = fmax(fabs((double)x0 - (double)s.cx), fabs((double)(x0 + w - 1) - (double)s.cx)) / (double)s.fx;
                    const double ty = fmax(fabs((double)y0 - (double)s.cy), fabs((double)(y0 + h - 1) - (double)s.cy)) / (double)s.fy;
                    const double du = (double)s.fx * rp * sqrt(1.0 + tx * tx) / (zn - rp) + 1.0;
                    const double dv = (double)s.fy * rp * sqrt(1.0 + ty * ty) / (zn - rp) + 1.0;
                    if ((double)(x0 + w - 1) + du < (double)a.box[0] || (double)x0 - du > (double)a.box[2]
                        || (double)(y0 + h - 1) + dv < (double)a.box[1] || (double)y0 - dv > (double)a.box[3])
                        w = h = 0;
                }
            } else if (!(zmax < 99.999)) {
                w = s.W;
                h = s.H;
            }
            s_box[0] = x0;
            s_box[1] = y0;
            s_box[2] = w;
            s_box[3] = h;
            s_n = 0;
            const double v[3] = {(double)P[2], (double)P[6], (double)P[10]};
            const double nv = sqrt((v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]);
            for (int c = 0; c < 3; ++c) s_u[c] = v[c] / nv;
            for (int k = 0; k < 9; ++k) s_A[k] = (k % 4 == 0) ? 1.0 : 0.0;
            s_b[0] = s_b[1] = s_b[2] = 0.0;
        }
        __syncthreads();
        const int tx0 = s_box[0], ty0 = s_box[1], tw = s_box[2], th = s_box[3];
        const int tpx = tw * th;
        // the tile in LDS when it fits (then, with room to spare, every
        // vertex projected once for the pose), else in device memory
        const bool in_lds = tpx <= a.lds_words;
        const int tile_q = (tpx + 3) & ~3;
        const int4 *vcache = nullptr;
        if (in_lds) {
            for (int k = tid; k < tpx; k += BLOCK) icp_lds[k] = kEmptyKey;
            if (tpx > 0 && 4 * m.nv <= a.lds_words - tile_q) {
                int4 *vc = reinterpret_cast<int4 *>(icp_lds + tile_q);
                for (int v = tid; v < m.nv; v += BLOCK) vc[v] = pack_vtx(project_vertex(P, gld(m.verts + v), s));
                vcache = vc;
            }
        } else {
            for (int k = tid; k < tpx; k += BLOCK) tst<true>(tile + k, kEmptyKey);
        }
        __syncthreads();
        if (tpx > 0)
            for (int t0 = 0; t0 < m.nt; t0 += BLOCK)
                if (t0 + tid < m.nt) {
                    if (in_lds) raster_triangle<false>(s, m, P, t0 + tid, tx0, ty0, tw, th, icp_lds, vcache);
                    else raster_triangle<true>(s, m, P, t0 + tid, tx0, ty0, tw, th, tile);
                }
        __syncthreads();
        for (int k = tid; k < tpx; k += BLOCK) {
            const uint32_t key = in_lds ? icp_lds[k] : tld<true>(tile + k);
            if (key == kEmptyKey) continue;
            const int ty = k / tw, tx = k - ty * tw;
            const int i = tx0 + tx, j = ty0 + ty, d = (int)(key >> 16);
            if (i % a.stride != 0 || j % a.stride != 0) continue;
            const int pix = j * s.W + i;
            if (mark) {
                const int dob = gld(s.depth + pix);
                if (dob > 0 && 16 * dob + s.dq < 16 * d && (!(label_mode && s.labels) || s.labels[pix] != a.label))
                    continue;
            }
            const int slot = atomicAdd(&s_n, 1);
            src[slot] = make_int4((int)rint(gld(s.kx + i) * (double)d), (int)rint(gld(s.ky + j) * (double)d), 16 * d, 0);
            if (gicp) {
                // the render's own neighbours (any rendered pixel, on or off the stride grid)
                auto rdepth = [&](int ii, int jj) -> int {
                    if (ii < tx0 || jj < ty0 || ii >= tx0 + tw || jj >= ty0 + th) return 0;
                    const int kk = (jj - ty0) * tw + (ii - tx0);
                    const uint32_t kv = in_lds ? icp_lds[kk] : tld<true>(tile + kk);
                    return kv == kEmptyKey ? 0 : (int)(kv >> 16);
                };
                int c[3];
                const int has = pixel_normal(s, i, j, gap, rdepth, c);
                nrm[slot] = has ? make_int4(c[0], c[1], c[2], 1) : make_int4(0, 0, 0, 0);
            }
        }
        __syncthreads();
        const int ns = __builtin_amdgcn_readfirstlane(s_n);
        int iters = 0, matched = 0;
        for (int it = 0; it < a.iterations; ++it) {
            if (tid == 0) s_changed = 0;
            __syncthreads();
            bool ch = false;
            for (int t = tid; t < ns; t += BLOCK) {
                const int4 sp = src[t];
                int qv[3];
                for (int c = 0; c < 3; ++c) {
                    // beyond 2^28 units (16 km) nothing can match; the clamp keeps the search in int range
                    const double v = rint(((s_A[3 * c] * (double)sp.x + s_A[3 * c + 1] * (double)sp.y)
                                           + s_A[3 * c + 2] * (double)sp.z) + s_b[c]);
                    qv[c] = (int)fmax(fmin(v, 268435456.0), -268435456.0);
                }
                int4 q = make_int4(qv[0], qv[1], qv[2], -1);
                if (it == 0) {
                    ch = true;
                } else {
                    const int4 o = qb[t];
                    ch |= o.x != q.x || o.y != q.y || o.z != q.z;
                    q.w = o.w;
                }
                qb[t] = q;
            }
            if (ch) s_changed = 1;
            __syncthreads();
            if (!__builtin_amdgcn_readfirstlane(s_changed)) break;
            for (int t = tid >> 2; t < ns; t += BLOCK / 4) {
                const int4 q = qb[t];
                // the match: also the next iteration's first guess, and read by GICP's second pass
                const int nn = icp_nn(a, q, q.w, lane & 3);
                if ((lane & 3) == 0) qb[t].w = nn;
            }
            __syncthreads();
            // the pairs' sums, 64 points at a time: sum j in lane j
            long long acc = 0;
            for (int t0 = wave * 64; t0 < ns; t0 += BLOCK) {
                const int t = t0 + lane;
                int4 q = make_int4(0, 0, 0, -1);
                if (t < ns) q = qb[t];
                const bool has = q.w >= 0;
                const int qv[3] = {has ? q.x : 0, has ? q.y : 0, has ? q.z : 0};
                WaveSums w(lane);
                w.set(0, has);
#pragma unroll
                for (int k = 0; k < 3; ++k) w.set(1 + k, qv[k]);
                if (!gicp) {     // GICP takes the matches' centre only
                    const int3 c = opt_at(s.opt, (uint32_t)max(q.w, 0));
                    const int cv[3] = {has ? c.x : 0, has ? c.y : 0, has ? c.z : 0};
#pragma unroll
                    for (int k = 0; k < 3; ++k) w.set(4 + k, cv[k]);
#pragma unroll
                    for (int k = 0; k < 9; ++k) {
                        if (k / 3 <= k % 3) w.set(7 + k, (long long)qv[k / 3] * (long long)qv[k % 3]);
                        w.set(16 + k, (long long)qv[k / 3] * (long long)cv[k % 3]);
                    }
                }
                acc += w.value();
            }
            if (lane < kIcpSums) s_red[wave][lane] = acc;
            __syncthreads();
            if (tid < kIcpSums) {
                // q q^T is symmetric: its lower entries come from the upper ones
                const int up = tid == 10 ? 8 : (tid == 13 ? 9 : (tid == 14 ? 12 : tid));
                long long z = 0;
                for (int v = 0; v < NW; ++v) z += s_red[v][up];
                s_tot[tid] = z;
            }
            __syncthreads();
            if (tid == 0) {
                int stop = 0;
                matched = (int)s_tot[0];
                if (s_tot[0] < a.min_points) stop = 1;
                else if (gicp) {
                    // the centre of the matched points, rounded: exact integer sums
                    for (int c = 0; c < 3; ++c) s_mu[c] = (long long)rint((double)s_tot[1 + c] / (double)s_tot[0]);
                } else if (icp_update(s_tot, a.dof, s_u, s_A, s_b)) {
                    stop = 1;
                } else {
                    iters = it + 1;
                }
                s_stop = stop;
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(s_stop)) break;
            if (gicp) {
                // second pass: the Gauss-Newton terms of every match, one
                // match per lane
                const long long mu[3] = {s_mu[0], s_mu[1], s_mu[2]};
                acc = 0;
                for (int t0 = wave * 64; t0 < ns; t0 += BLOCK) {
                    const int t = t0 + lane;
                    int4 q = make_int4(0, 0, 0, -1), cs = make_int4(0, 0, 0, 0);
                    if (t < ns) {
                        q = qb[t];
                        cs = nrm[t];
                    }
                    const bool has = q.w >= 0;
                    const int nn = max(q.w, 0);
                    const int3 c = opt_at(s.opt, (uint32_t)nn);
                    double na[3] = {0.0, 0.0, 0.0}, nb[3] = {0.0, 0.0, 0.0};
                    const int csv[3] = {cs.x, cs.y, cs.z};
                    if (cs.w) unit_of(csv, na);
                    const int pj = nn / s.W, pi = nn - pj * s.W;
                    auto odepth = [&](int ii, int jj) -> int { return gld(s.depth + jj * s.W + ii); };
                    int cb[3];
                    const int has_b = pixel_normal(s, pi, pj, gap, odepth, cb);
                    if (has_b) unit_of(cb, nb);
                    WaveSums w(lane);
                    gicp_terms(has, q, c, mu, cs.w, na, has_b, nb, s_A, w);
                    acc += w.value();
                }
                if (lane < kGicpSums) s_red[wave][lane] = acc;
                __syncthreads();
                if (tid < kGicpSums) {
                    long long z = 0;
                    for (int v = 0; v < NW; ++v) z += s_red[v][tid];
                    s_tot[tid] = z;
                }
                __syncthreads();
                if (tid == 0) {
                    const int stop = gicp_update(s_tot, mu, s_A, s_b);
                    if (!stop) iters = it + 1;
                    s_stop = stop;
                }
                __syncthreads();
                if (__builtin_amdgcn_readfirstlane(s_stop)) break;
            }
        }
        if (tid == 0) {
            float *out = a.refined + 12 * (size_t)p;
            const float *P = a.poses + 12 * (size_t)p;     // read again: not held through the iterations
            for (int r = 0; r < 3; ++r) {
                for (int c = 0; c < 3; ++c)
                    out[4 * r + c] = (float)((s_A[3 * r] * (double)P[c] + s_A[3 * r + 1] * (double)P[4 + c])
                                             + s_A[3 * r + 2] * (double)P[8 + c]);
                const double t = ((s_A[3 * r] * (16.0 * (double)P[3]) + s_A[3 * r + 1] * (16.0 * (double)P[7]))
                                  + s_A[3 * r + 2] * (16.0 * (double)P[11])) + s_b[r];
                out[4 * r + 3] = (float)(t / 16.0);
            }
            if (a.iters) a.iters[p] = iters;
            if (a.matched) a.matched[p] = matched;
            s_pose = atomicAdd(a.cursor, 1);
        }
        __syncthreads();
        p = __builtin_amdgcn_readfirstlane(s_pose);
    }
}

// ------------------------------------------------------------------ pose proposals

// 6-DoF pose proposals (Sec. V-B "Pose Proposal Generation"): pose p is
// viewpoint i, in-plane angle k and depth t, p = (i N + k) T + t.  Viewpoint
// i of M on the Fibonacci lattice, z_i = 1 - (2 i + 1) / M at longitude
// i pi (3 - sqrt 5): the camera sits in direction v_i from the object, so
// the rotation takes v_i to the camera's -z axis (rows b1, b2, b3 with
// b3 = -v_i and b1 along z_obj x b3, or y_obj x b3 near the poles), then
// turns by 2 pi k / N about the optical axis.  The translation puts the
// object's centre (its mesh's AABB centre c) on the ray through the label
// box centre at depth z_t: t = z_t ray - R c.
__global__ void proposal_kernel(ProposalArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n) return;
    const int t = p % a.T, k = (p / a.T) % a.N, i = p / (a.T * a.N);
    const double pi = 3.14159265358979323846;
    const double vz = 1.0 - (double)(2 * i + 1) / (double)a.M;
    const double r = sqrt(fmax(0.0, 1.0 - vz * vz));
    const double phi = (double)i * (pi * (3.0 - sqrt(5.0)));
    const double v[3] = {r * cos(phi), r * sin(phi), vz};
    const double b3[3] = {-v[0], -v[1], -v[2]};
    const double up[3] = {0.0, fabs(vz) > 0.999 ? 1.0 : 0.0, fabs(vz) > 0.999 ? 0.0 : 1.0};
    double b1[3] = {up[1] * b3[2] - up[2] * b3[1], up[2] * b3[0] - up[0] * b3[2], up[0] * b3[1] - up[1] * b3[0]};
    const double nb = sqrt((b1[0] * b1[0] + b1[1] * b1[1]) + b1[2] * b1[2]);
    for (int c = 0; c < 3; ++c) b1[c] = b1[c] / nb;
    const double b2[3] = {b3[1] * b1[2] - b3[2] * b1[1], b3[2] * b1[0] - b3[0] * b1[2], b3[0] * b1[1] - b3[1] * b1[0]};
    const double th = 2.0 * pi * (double)k / (double)a.N;
    const double co = cos(th), si = sin(th);
    const double z = a.zmin + (double)t * a.step;
    float *o = a.out + 12 * (size_t)p;
    for (int c = 0; c < 3; ++c) {
        o[c] = (float)(co * b1[c] - si * b2[c]);
        o[4 + c] = (float)(si * b1[c] + co * b2[c]);
        o[8 + c] = (float)b3[c];
    }
    const double ray[3] = {z * ((a.uc - (double)a.cx) / (double)a.fx), z * ((a.vc - (double)a.cy) / (double)a.fy), z};
    for (int r = 0; r < 3; ++r) {
        const double R0 = r == 0 ? co * b1[0] - si * b2[0] : (r == 1 ? si * b1[0] + co * b2[0] : b3[0]);
        const double R1 = r == 0 ? co * b1[1] - si * b2[1] : (r == 1 ? si * b1[1] + co * b2[1] : b3[1]);
        const double R2 = r == 0 ? co * b1[2] - si * b2[2] : (r == 1 ? si * b1[2] + co * b2[2] : b3[2]);
        o[4 * r + 3] = (float)(ray[r] - ((R0 * a.centre[0] + R1 * a.centre[1]) + R2 * a.centre[2]));
    }
}

// ------------------------------------------------------------------ launchers

hipError_t launch_proposals(const ProposalArgs &a, hipStream_t st)
{
    if (a.n > 0) proposal_kernel<<<(a.n + 255) / 256, 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_icp(const IcpArgs &a, int block, int grid, hipStream_t st)
{
    const int tiles = (int)icp_tiles(a.s.W, a.s.H);
    icp_target_kernel<<<(tiles + 15) / 16, 256, 0, st>>>(a);
    icp_target_wide_kernel<<<(tiles + 255) / 256, 256, 0, st>>>(a);
    const size_t lds = (size_t)a.lds_words * 4;
    if (block == 512) {
        if (a.method == 1) icp_kernel<512, true><<<grid, 512, lds, st>>>(a);
        else icp_kernel<512, false><<<grid, 512, lds, st>>>(a);
    } else {
        if (a.method == 1) icp_kernel<1024, true><<<grid, 1024, lds, st>>>(a);
        else icp_kernel<1024, false><<<grid, 1024, lds, st>>>(a);
    }
    return hipGetLastError();
}

hipError_t prepare_icp_kernel(int lds_per_group, int lds_words[2])
{
    lds_words[0] = lds_words[1] = 0;
    const void *ks[2][2] = {{(const void *)icp_kernel<512, false>, (const void *)icp_kernel<512, true>},
                            {(const void *)icp_kernel<1024, false>, (const void *)icp_kernel<1024, true>}};
    for (int b = 0; b < 2; ++b) {
        const int share = b == 0 ? lds_per_group / 2 : lds_per_group;
        int st = 0;
        for (const void *f : ks[b]) {
            hipFuncAttributes at{};
            if (hipError_t e = hipFuncGetAttributes(&at, f)) return e;
            st = max(st, (int)at.sharedSizeBytes);
        }
        for (const void *f : ks[b])
            if (hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, share - st)) return e;
        lds_words[b] = (share - st) / 4;
    }
    return hipSuccess;
}

}  // namespace perch
