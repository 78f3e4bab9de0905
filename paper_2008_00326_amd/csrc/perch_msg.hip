// gfx950 kernels of the Monotone Scene Generation tree, the sequential search
// of the original PERCH that the variant 2.0-B of PERCH 2.0 keeps (Sec. III-B
// and its tree figure, Sec. VI-A).  A state's render lives in HBM as a few
// full-image planes; every successor of a state (one object in each of its
// candidate poses) is scored by one persistent launch:
//   1. rasterize the successor into a tile (LDS when it fits);
//   2. it is not monotone if it is nearer than the state's render on any
//      pixel both draw; its own points dR are its pixels the state leaves
//      empty, on the stride grid, less occluders (Eq. 3);
//   3. J_r of dR from the scene's nearest-neighbour table, with the colour
//      test of Eq. 4;
//   4. J_o over the observed points inside V(O) and outside every placed
//      object's volume: the nearest point of the composed render is the
//      nearer of the state's (kept per observed pixel with the state) and
//      the successor's own (searched in the tile), then Eq. 4.

#include "perch_device.h"

#include <math.h>

#include <algorithm>

namespace perch {

// ------------------------------------------------------------------ state images

__global__ __launch_bounds__(256) void msg_clear_kernel(SceneDev s, MsgState st)
{
    const int N = s.W * s.H;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < N; k += gridDim.x * 256) {
        st.depth[k] = 0;
        st.pts[k] = 0;
        if (st.rgb) st.rgb[k] = 0;
        st.cov[k] = 0;
        st.near[k] = ~0ULL;
    }
}

constexpr int kNoBox = -(1 << 30);

// The kernels below append one object to each of up to kMsgAdds states
// (blockIdx.y).
__global__ __launch_bounds__(256) void msg_keys_kernel(MsgAddArgs a)
{
    const int N = a.s.W * a.s.H;
    uint32_t *keys = a.add[blockIdx.y].keys;
    if (a.first && blockIdx.x == 0 && threadIdx.x < 4) a.add[blockIdx.y].box[threadIdx.x] = kNoBox;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < N; k += gridDim.x * 256) keys[k] = kEmptyKey;
}

// One thread per triangle over the whole image.
__global__ __launch_bounds__(256) void msg_raster_kernel(MsgAddArgs a)
{
    const MsgAdd &o = a.add[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= o.m.nt) return;
    float P[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) P[k] = o.pose[k];
    raster_triangle<true>(a.s, o.m, P, t, 0, 0, a.s.W, a.s.H, o.keys);
}

// Append the rendered object to the state: pixels the state leaves empty
// take its depth and colour, and become points of R \ C on the stride grid
// unless the observed depth marks them as occluded (Eq. 3, the object's own
// label exempt); a pixel where it is nearer than the state flags the state
// as not monotone.  Observed points inside its volume become covered, and a
// series' box grows to hold the new points.
__global__ __launch_bounds__(256) void msg_compose_kernel(MsgAddArgs a)
{
    const SceneDev &s = a.s;
    const MsgAdd &ad = a.add[blockIdx.y];
    const int N = s.W * s.H;
    const bool mark = (s.flags & 2u) != 0;
    const bool label_mode = (s.flags & (3u << 4)) == (2u << 4);
    const bool cyl = (s.flags & (3u << 4)) == (1u << 4);
    const double dl = (double)s.delta;
    float P[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) P[k] = ad.pose[k];
    __shared__ int s_box[4];
    if (threadIdx.x < 4) s_box[threadIdx.x] = kNoBox;
    int b[4] = {kNoBox, kNoBox, kNoBox, kNoBox};
    for (int k = blockIdx.x * 256 + threadIdx.x; k < N; k += gridDim.x * 256) {
        const int j = k / s.W, i = k - j * s.W;
        const uint32_t key = ad.keys[k];
        if (key != kEmptyKey) {
            const int d = (int)(key >> 16);
            const int sd = ad.st.depth[k];
            if (sd > 0) {
                if (d < sd) atomicOr(a.flag, 1);
            } else {
                ad.st.depth[k] = (uint16_t)d;
                if (ad.st.rgb) ad.st.rgb[k] = triangle_colour(s, ad.m, P, (int)(key & 0xFFFFu), i, j);
                bool pt = i % s.stride == 0 && j % s.stride == 0;
                if (pt && mark) {
                    const int dob = s.depth[k];
                    if (dob > 0 && 16 * dob + s.dq < 16 * d && (!(label_mode && s.labels) || s.labels[k] != ad.label))
                        pt = false;
                }
                ad.st.pts[k] = pt ? (uint16_t)d : (uint16_t)0;
                if (pt) {
                    b[0] = max(b[0], -i);
                    b[1] = max(b[1], -j);
                    b[2] = max(b[2], i);
                    b[3] = max(b[3], j);
                }
            }
        }
        const int4 o = s.opt[k];
        if (o.z != kNoPoint && !ad.st.cov[k]) {
            const bool in = label_mode ? (s.labels && s.labels[k] == ad.label)
                                       : in_volume(ad.m, P, o.x, o.y, o.z >> 4, dl, cyl);
            if (in) ad.st.cov[k] = 1;
        }
    }
    if (a.first && a.last) return;                 // a single object: its projected box will do
    if (!__syncthreads_or(b[2] >= 0)) return;      // no new point in this work-group's pixels
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        for (int o = 1; o < 64; o <<= 1) b[c] = max(b[c], __shfl_xor(b[c], o));
        if ((threadIdx.x & 63) == 0) atomicMax(&s_box[c], b[c]);
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 4 && s_box[c] > __hip_atomic_load(ad.box + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(ad.box + c, s_box[c]);
}

// Per observed pixel, the nearest point of the state's R \ C within delta:
// min (squared distance << 32 | pixel), ~0 when none.  Only the objects
// appended since the last time have new points, in the box that compose keeps
// of a series' points or in a single object's projected box (a tree search's
// children, where the box's reduction costs 6 % of an exhaustive search):
// pixels beyond it grown by the scene's neighbour windows keep what they have.
// One pass for a series of objects, on as many work-groups as the image fills
// (640x480, all of msg_expand with a state of one object and of 32: small
// objects 0.20 and 0.69 ms, objects of the image's size at delta 30 mm 3.0 and
// 3.5 ms; with a pass for each object over its projected box, on at most 256
// work-groups, 0.20 and 2.2, 6.2 and 52 ms).
__global__ __launch_bounds__(256) void msg_near_kernel(MsgAddArgs a)
{
    const SceneDev &s = a.s;
    const MsgAdd &ad = a.add[blockIdx.y];
    const MsgState st = ad.st;
    int x0, y0, x1, y1;
    if (a.first && a.last) {
        float P[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) P[k] = ad.pose[k];
        double umin, umax, vmin, vmax, zmin, zmax;
        project_box_wave(P, ad.m.lo, ad.m.hi, 0.0, s, threadIdx.x & 63, &umin, &umax, &vmin, &vmax, &zmin, &zmax);
        int bw = s.W, bh = s.H;
        x0 = y0 = 0;
        if (zmin >= 100.0) clip_box(umin, umax, vmin, vmax, s.W, s.H, &x0, &y0, &bw, &bh);
        else if (zmax < 99.999) bw = bh = 0;
        if (bw == 0 || bh == 0) return;
        x1 = x0 + bw - 1;
        y1 = y0 + bh - 1;
    } else {
        x0 = -ad.box[0];
        y0 = -ad.box[1];
        x1 = ad.box[2];
        y1 = ad.box[3];
        if (x1 < 0) return;
    }
    x0 = max(x0 - s.wtx, 0);
    y0 = max(y0 - s.wty, 0);
    x1 = min(x1 + s.wtx, s.W - 1);
    y1 = min(y1 + s.wty, s.H - 1);
    const int w = x1 - x0 + 1, n = w * (y1 - y0 + 1);
    const float dlw = s.delta + 0.25f, winv = 1.0f / (float)w;
    for (int q = blockIdx.x * 256 + threadIdx.x; q < n; q += gridDim.x * 256) {
        const int r = window_row(q, w, winv), j = y0 + r, i = x0 + q - r * w, k = j * s.W + i;
        const int3 o = opt_at(s.opt, (uint32_t)k);
        if (o.z == kNoPoint) continue;
        const float iz = window_inv(o.z >> 4, dlw);
        const int wu = window_half(gld(s.ax + i), iz, s.W), wv = window_half(gld(s.ay + j), iz, s.H);
        const int i0 = max(i - wu, 0), i1 = min(i + wu, s.W - 1);
        const int j0 = max(j - wv, 0), j1 = min(j + wv, s.H - 1);
        unsigned long long best = gld(st.near + k);
        for (int jj = j0; jj <= j1; ++jj)
            for (int ii = i0; ii <= i1; ii += 4) {
                int d[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) d[u] = gld(st.pts + (jj * s.W + min(ii + u, i1)));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    // a point of the same depth range only: the others are beyond delta
                    if (d[u] == 0 || abs(16 * d[u] - o.z) > s.dq) continue;
                    const int c = min(ii + u, i1);
                    const double dx = rint(gld(s.kx + c) * (double)d[u]) - (double)o.x;
                    const double dy = rint(gld(s.ky + jj) * (double)d[u]) - (double)o.y;
                    const int d2 = capped_d2((int)dx, (int)dy, 16 * d[u] - o.z, (uint32_t)s.dq2 + 1);
                    const unsigned long long v = ((unsigned long long)(uint32_t)d2 << 32) | (uint32_t)(jj * s.W + c);
                    if (d2 <= s.dq2 && v < best) best = v;
                }
            }
        st.near[k] = best;
    }
}

// ------------------------------------------------------------------ successors

__global__ void msg_zero_kernel(int *cursor)
{
    if (threadIdx.x == 0) cursor[0] = 0;
}

constexpr int kMsgBlock = 1024;

// One work-group per successor, taken through a cursor over the launch's
// items.  Its four parts: raster; one pass over the tile (monotone test,
// dR \ C, J_r table lookup); one pass over the V region; and, from per-wave
// queues so that every lane has a point, the colour tests and the search for
// the nearest rendered point of each charged observed point.
//
// That search was nine tenths of the kernel as a scan of each point's whole
// window (15x15 pixels at delta 10 mm) in 64-bit arithmetic.  Now the
// state's nearest point and the rendered points around the pixel itself bound
// it first, the window shrinks to what can still be nearer, and its 4x4 pixel tiles are
// skipped by their depth ranges; the tile's back-projection factors come from
// LDS.  All successors of a level go in one launch.  Three objects of 400
// candidates, beam 4, 640x480 RGB: 21.8 ms in 15 launches -> 3.3 ms in 3; what
// is left is spread over the parts (raster 14 %, its set-up 11 %, J_r 30 %,
// J_o 35 %), each a chain of loads at 16 waves per compute unit (waiting 65 % of
// their time, issue 0.53 of the card's rate; 19 registers spilled).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void msg_kernel(MsgArgs a)
{
    constexpr int NW = BLOCK / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SceneDev &s = a.s;
    extern __shared__ __align__(16) uint32_t msg_lds[];
    __shared__ int s_pose, s_bad, s_cnt[4];
    __shared__ int s_queue[NW][128];
    int *const q = s_queue[wave];
    uint32_t *gtile = a.tiles + (size_t)blockIdx.x * s.W * s.H;
    const bool rgb = (s.flags & 1u) != 0;
    const bool mark = (s.flags & 2u) != 0;
    const bool label_mode = (s.flags & (3u << 4)) == (2u << 4);
    const bool cyl = (s.flags & (3u << 4)) == (1u << 4);
    const double dl = (double)s.delta;
    // Poses come through the cursor; the loop is rotated by hand so that its
    // condition is a wave-uniform value and no branch on the thread index
    // heads it: with a divergent `if (tid == 0)` fetch at the top, the
    // compiler may send thread 0 alone round an outer loop to fetch the next
    // pose while the other lanes wait for it at the barrier, which they then
    // pass without it.
    if (tid == 0) s_pose = atomicAdd(a.cursor, 1);
    __syncthreads();
    for (int p = __builtin_amdgcn_readfirstlane(s_pose); p < a.n;) {
        // the item holding successor p: the last one with first <= p
        int lo = 0, hi = a.n_items - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.items[mid].first <= p) lo = mid;
            else hi = mid - 1;
        }
        const MsgItem &w = a.items[lo];
        const MeshDev &m = w.m;
        const int local = p - w.first;
        float P[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) P[k] = w.poses[12 * (size_t)local + k];
        int tx0 = 0, ty0 = 0, tw = 0, th = 0, rx0 = 0, ry0 = 0, rw = 0, rh = 0;
        {
            double umin, umax, vmin, vmax, zmin, zmax;
            project_box_wave(P, m.lo, m.hi, 0.0, s, lane, &umin, &umax, &vmin, &vmax, &zmin, &zmax);
            if (zmin >= 100.0) {
                clip_box(umin, umax, vmin, vmax, s.W, s.H, &tx0, &ty0, &tw, &th);
            } else if (!(zmax < 99.999)) {
                tw = s.W;
                th = s.H;
            }
            // every observed pixel that may lie in V(O): the label's box, or
            // the projection of the grown box when it lies wholly in front of
            // the camera, else the whole image
            if (label_mode) {
                rx0 = w.vbox[0];
                ry0 = w.vbox[1];
                rw = w.vbox[2];
                rh = w.vbox[3];
            } else {
                project_box_wave(P, m.lo, m.hi, dl, s, lane, &umin, &umax, &vmin, &vmax, &zmin, &zmax);
                if (zmin > 0.0) {
                    clip_box(umin, umax, vmin, vmax, s.W, s.H, &rx0, &ry0, &rw, &rh);
                } else {
                    rw = s.W;
                    rh = s.H;
                }
            }
            tx0 = __builtin_amdgcn_readfirstlane(tx0);
            ty0 = __builtin_amdgcn_readfirstlane(ty0);
            tw = __builtin_amdgcn_readfirstlane(tw);
            th = __builtin_amdgcn_readfirstlane(th);
            rx0 = __builtin_amdgcn_readfirstlane(rx0);
            ry0 = __builtin_amdgcn_readfirstlane(ry0);
            rw = __builtin_amdgcn_readfirstlane(rw);
            rh = __builtin_amdgcn_readfirstlane(rh);
        }
        if (tid < 4) s_cnt[tid] = 0;
        if (tid == 4) s_bad = 0;
        const int tpx = tw * th;
        const bool in_lds = tpx <= a.lds_words;
        const int tile_q = (tpx + 3) & ~3;
        const int4 *vcache = nullptr;
        if (in_lds) {
            for (int k = tid; k < tpx; k += BLOCK) msg_lds[k] = kEmptyKey;
            if (tpx > 0 && 4 * m.nv <= a.lds_words - tile_q) {
                int4 *vc = reinterpret_cast<int4 *>(msg_lds + tile_q);
                for (int v = tid; v < m.nv; v += BLOCK) vc[v] = pack_vtx(project_vertex(P, gld(m.verts + v), s));
                vcache = vc;
            }
        } else {
            for (int k = tid; k < tpx; k += BLOCK) tst<true>(gtile + k, kEmptyKey);
        }
        __syncthreads();
        if (tpx > 0)
            for (int t0 = 0; t0 < m.nt; t0 += BLOCK)
                if (t0 + tid < m.nt) {
                    if (in_lds) raster_triangle<false>(s, m, P, t0 + tid, tx0, ty0, tw, th, msg_lds, vcache);
                    else raster_triangle<true>(s, m, P, t0 + tid, tx0, ty0, tw, th, gtile);
                }
        __syncthreads();
        auto tkey = [&](int k) { return in_lds ? msg_lds[k] : tld<true>(gtile + k); };
        // row of tile index k: an LDS tile holds fewer than 2^16 pixels,
        // where (k + 1/2) / tw in binary32 truncates to the exact quotient
        const float tinv = 1.0f / (float)max(tw, 1);
        auto trow = [&](int k) { return in_lds ? (int)(((float)k + 0.5f) * tinv) : k / max(tw, 1); };
        auto table_nn = [&](int2 tr, int d) {
            const int e = d - (tr.y & 0xFFFF);
            const bool ok = e >= 0 && e < (int)((uint32_t)tr.y >> 16);
            const int nn = gld(s.tnn + (uint32_t)(ok ? tr.x + e : 0));
            return ok ? nn : -1;
        };
        const bool hashed = (s.flags & kHashFlag) != 0;
        auto point_nn = [&](int i, int j, int d) {
            if (hashed) return hash_nn(s, (int)rint(gld(s.kx + i) * (double)d), (int)rint(gld(s.ky + j) * (double)d), 16 * d);
            return table_nn(gld(s.thdr + (uint32_t)(j * s.W + i)), d);
        };

        // monotonicity, dR \ C (the tile keeps only its pixels) and J_r;
        // the points to colour-test are queued and tested 64 at a time
        int cr = 0, cn = 0, qc = 0;
        bool bad = false;
        auto flush_r = [&](int n) {
            wave_lds_sync();
            bool out = false;
            if (lane < n) {
                const int k = q[lane];
                const uint32_t key = tkey(k);
                const int ty = trow(k), i = tx0 + k - ty * tw, j = ty0 + ty;
                const int nn = max(point_nn(i, j, (int)(key >> 16)), 0);
                out = ciede2000(srgb_to_lab(triangle_colour(s, m, P, (int)(key & 0xFFFFu), i, j)), gld(s.olab + nn)) > s.tau;
            }
            cr += wave_popc(out);
        };
        auto push = [&](bool need, int v, auto &&flush) {
            const unsigned long long mq = __ballot(need);
            if (need) q[qc + lane_rank(mq)] = v;
            qc += __popcll(mq);
            if (qc >= 64) {
                flush(64);
                wave_lds_sync();
                if (64 + lane < qc) q[lane] = q[64 + lane];     // the overflow moves to the front
                qc -= 64;
            }
        };
        // two chunks a turn, their loads issued first (every lane loads, at a clamped pixel)
        for (int k0 = wave * 64; k0 < tpx; k0 += 2 * BLOCK) {
            uint32_t key[2];
            int ii[2], jj[2], sd[2], dob[2];
            int2 tr[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = k0 + u * BLOCK + lane, kc = min(k, tpx - 1);
                key[u] = k < tpx ? tkey(kc) : kEmptyKey;
                const int ty = trow(kc);
                ii[u] = tx0 + kc - ty * tw;
                jj[u] = ty0 + ty;
                const uint32_t pix = (uint32_t)(jj[u] * s.W + ii[u]);
                sd[u] = gld(w.st.depth + pix);
                dob[u] = mark ? (int)gld(s.depth + pix) : 0;
                tr[u] = hashed ? make_int2(0, 0) : gld(s.thdr + pix);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (k0 + u * BLOCK >= tpx) break;
                const int k = k0 + u * BLOCK + lane, d = (int)(key[u] >> 16), i = ii[u], j = jj[u];
                const bool has = key[u] != kEmptyKey;
                bad |= has && sd[u] > 0 && d < sd[u];
                bool keep = has && sd[u] == 0 && (s.stride == 1 || (i % s.stride == 0 && j % s.stride == 0));
                if (keep && dob[u] > 0 && 16 * dob[u] + s.dq < 16 * d
                    && (!(label_mode && s.labels) || gld(s.labels + j * s.W + i) != w.label))
                    keep = false;
                if (has && !keep) {
                    if (in_lds) msg_lds[k] = kEmptyKey;
                    else tst<true>(gtile + k, kEmptyKey);
                }
                int nn = -1;
                if (hashed) {
                    if (keep) nn = point_nn(i, j, d);
                } else {
                    nn = table_nn(tr[u], d);
                }
                cn += wave_popc(keep);
                cr += wave_popc(keep && nn < 0);
                if (rgb) push(keep && nn >= 0, k, flush_r);
            }
        }
        if (qc > 0) flush_r(qc);
        if (wave_popc(bad) && lane == 0) s_bad = 1;
        if (lane == 0) {
            atomicAdd(&s_cnt[0], cr);
            atomicAdd(&s_cnt[2], cn);
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(s_bad)) {
            // beyond the LDS tile: back-projection factors of its columns and
            // rows, and the depth range of each of its 4x4 pixel tiles
            // (least | greatest << 16; 65535 | 0 without a point)
            const int bw = (tw + 3) >> 2, bh = (th + 3) >> 2;
            const bool fast = in_lds && tile_q + 2 * (tw + th) + bw * bh <= a.lds_words;
            double *kxs = reinterpret_cast<double *>(msg_lds + tile_q), *kys = kxs + tw;
            uint32_t *range = msg_lds + tile_q + 2 * (tw + th);
            if (fast) {
                for (int k = tid; k < tw + th; k += BLOCK) kxs[k] = k < tw ? gld(s.kx + tx0 + k) : gld(s.ky + ty0 + k - tw);
                for (int t = tid; t < bw * bh; t += BLOCK) {
                    const int by = t / bw, bx = t - by * bw;
                    uint32_t dmin = 65535, dmax = 0;
                    for (int k = 0; k < 16; ++k) {
                        const uint32_t key = msg_lds[min(4 * by + (k >> 2), th - 1) * tw + min(4 * bx + (k & 3), tw - 1)];
                        if (key == kEmptyKey) continue;
                        dmin = min(dmin, key >> 16);
                        dmax = max(dmax, key >> 16);
                    }
                    range[t] = dmin | (dmax << 16);
                }
                __syncthreads();
            }
            // J_o over the observed points of V(O) outside every placed volume
            const int rpx = rw * rh;
            int co = 0, cq = 0;
            const float dlw = s.delta + 0.25f;
            auto flush_o = [&](int n) {
                wave_lds_sync();
                bool out = false;
                if (lane < n) {
                    const int pix = q[lane];
                    const int3 o = opt_at(s.opt, (uint32_t)pix);
                    const unsigned long long near = gld(w.st.near + pix);
                    const int j = pix / s.W, i = pix - j * s.W;
                    // squared distance and pixel of the nearest point so far; nothing yet: above dq^2
                    int bd2 = near == ~0ULL ? s.dq2 + 1 : (int)(near >> 32);
                    int bpix = near == ~0ULL ? -1 : (int)(near & 0xFFFFFFFFu);
                    const double ox = (double)o.x, oy = (double)o.y;
                    auto take = [&](uint32_t key, double kx, double ky, int u) {
                        const int d = (int)(key >> 16);
                        const int d2 = capped_d2((int)(rint(kx * (double)d) - ox), (int)(rint(ky * (double)d) - oy),
                                                 16 * d - o.z, (uint32_t)s.dq2 + 1);
                        if (key != kEmptyKey && (d2 < bd2 || (d2 == bd2 && u < bpix))) {
                            bd2 = d2;
                            bpix = u;
                        }
                    };
                    auto scan = [&](int lx, int ly) {     // the 4x4 tile at (lx, ly), clamped to the LDS tile
#pragma unroll
                        for (int y = 0; y < 4; ++y) {
                            const int yy = min(ly + y, th - 1);
                            const double ky = kys[yy];
                            const int u = (ty0 + yy) * s.W + tx0;
#pragma unroll
                            for (int x = 0; x < 4; ++x) {
                                const int xx = min(lx + x, tw - 1);
                                take(msg_lds[yy * tw + xx], kxs[xx], ky, u + xx);
                            }
                        }
                    };
                    // without the colour term any point within delta will do
                    if (tpx > 0 && (rgb || bd2 > s.dq2)) {
                        if (fast) {
                            nearest_rendered(s, o, i, j, tx0, ty0, tw, th, !rgb, bd2, [&](int b) { return range[b]; },
                                             [&](int b) { scan(4 * (b % bw), 4 * (b / bw)); });
                        } else {
                            const float iz = window_inv(o.z >> 4, dlw);
                            const int wu = window_half(gld(s.ax + i), iz, s.W), wv = window_half(gld(s.ay + j), iz, s.H);
                            for (int jj = max(j - wv, ty0); jj <= min(j + wv, ty0 + th - 1); ++jj)
                                for (int ii = max(i - wu, tx0); ii <= min(i + wu, tx0 + tw - 1); ++ii)
                                    take(tkey((jj - ty0) * tw + (ii - tx0)), gld(s.kx + ii), gld(s.ky + jj), jj * s.W + ii);
                        }
                    }
                    out = bd2 > s.dq2;
                    if (!out && rgb) {
                        // the nearest point is the state's or the successor's own
                        uint32_t c;
                        if (gld(w.st.pts + bpix) > 0) {
                            c = gld(w.st.rgb + bpix);
                        } else {
                            const int uj = bpix / s.W, ui = bpix - uj * s.W;
                            const uint32_t key = tkey((uj - ty0) * tw + (ui - tx0));
                            c = triangle_colour(s, m, P, (int)(key & 0xFFFFu), ui, uj);
                        }
                        out = ciede2000(gld(s.olab + pix), srgb_to_lab(c)) > s.tau;
                    }
                }
                co += wave_popc(out);
            };
            qc = 0;
            const float rinv = 1.0f / (float)max(rw, 1);
            for (int k0 = wave * 64; k0 < rpx; k0 += 2 * BLOCK) {
                int pix[2], cov[2], lab[2];
                int3 o[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int kc = min(k0 + u * BLOCK + lane, rpx - 1);
                    const int ry = window_row(kc, rw, rinv);
                    pix[u] = (ry0 + ry) * s.W + rx0 + kc - ry * rw;
                    o[u] = opt_at(s.opt, (uint32_t)pix[u]);
                    cov[u] = gld(w.st.cov + pix[u]);
                    lab[u] = label_mode && s.labels ? gld(s.labels + pix[u]) : ~w.label;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (k0 + u * BLOCK >= rpx) break;
                    bool in = k0 + u * BLOCK + lane < rpx && o[u].z != kNoPoint && !cov[u];
                    if (in) in = label_mode ? lab[u] == w.label : in_volume(m, P, o[u].x, o[u].y, o[u].z >> 4, dl, cyl);
                    cq += wave_popc(in);
                    push(in, pix[u], flush_o);
                }
            }
            if (qc > 0) flush_o(qc);
            if (lane == 0) {
                atomicAdd(&s_cnt[1], co);
                atomicAdd(&s_cnt[3], cq);
            }
        }
        __syncthreads();
        if (tid == 0) {
            const bool ok = !s_bad;
            w.valid[local] = ok;
            w.jr[local] = ok ? s_cnt[0] : 0;
            w.jo[local] = ok ? s_cnt[1] : 0;
            if (w.nr) w.nr[local] = ok ? s_cnt[2] : 0;
            if (w.nq) w.nq[local] = ok ? s_cnt[3] : 0;
            s_pose = atomicAdd(a.cursor, 1);
        }
        __syncthreads();
        p = __builtin_amdgcn_readfirstlane(s_pose);
    }
}

// ------------------------------------------------------------------ launches

hipError_t upload_msg_colour_table(const float *lin256)
{
    return hipMemcpyToSymbol(HIP_SYMBOL(c_lin), lin256, 256 * sizeof(float));
}

static int pixel_grid(int N)
{
    return std::max(1, std::min((N + 255) / 256, 4096));
}

hipError_t msg_state_clear(const SceneDev &s, const MsgState &st, hipStream_t stream)
{
    msg_clear_kernel<<<pixel_grid(s.W * s.H), 256, 0, stream>>>(s, st);
    return hipGetLastError();
}

hipError_t msg_state_add(const MsgAddArgs &a, hipStream_t stream)
{
    if (a.n < 1 || a.n > kMsgAdds) return hipErrorInvalidValue;
    int nt = 1;
    for (int k = 0; k < a.n; ++k) nt = std::max(nt, a.add[k].m.nt);
    const dim3 px(pixel_grid(a.s.W * a.s.H), a.n);
    msg_keys_kernel<<<px, 256, 0, stream>>>(a);
    msg_raster_kernel<<<dim3((nt + 255) / 256, a.n), 256, 0, stream>>>(a);
    msg_compose_kernel<<<px, 256, 0, stream>>>(a);
    // many states at once share the device: fewer work-groups of each, most of which a small box leaves empty
    if (a.last) msg_near_kernel<<<dim3(a.n > 1 ? std::min(px.x, 512u) : px.x, a.n), 256, 0, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_msg(const MsgArgs &a, int grid, hipStream_t stream)
{
    msg_zero_kernel<<<1, 1, 0, stream>>>(a.cursor);
    msg_kernel<kMsgBlock><<<grid, kMsgBlock, (size_t)a.lds_words * 4, stream>>>(a);
    return hipGetLastError();
}

hipError_t prepare_msg_kernel(int lds_per_group, int *lds_words)
{
    const void *f = (const void *)msg_kernel<kMsgBlock>;
    hipFuncAttributes at{};
    hipError_t e = hipFuncGetAttributes(&at, f);
    if (e != hipSuccess) return e;
    const int dyn = lds_per_group - (int)at.sharedSizeBytes;
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    *lds_words = e == hipSuccess ? dyn / 4 : 0;
    return e;
}

}  // namespace perch
