// Ray-cast backend of the Gigapixel renderer for gfx950 (MI355X): the
// paper's renderer can rasterise or ray-trace the same scene (App. A,
// "High-Throughput Batched Rendering"); this kernel casts one primary ray per
// pixel sample and keeps, per pixel, the largest key in the raster's order
// (1/z bits, class, inverted primitive index, colour), so both backends
// resolve alike.
//
// Per-sample arithmetic (binary32, every fused operation an fmaf, correctly
// rounded division and square root):
//   ray      offsets a = i + 0.5 - cx, b = cy - (j + 0.5); world direction
//            d = (fmaf(a, fy, f fx), fmaf(a, -fx, f fy), b) from the camera at
//            (px, py, h) with forward (fx, fy); a hit at parameter s has
//            planar depth z = s f, kept in [z_near, z_far]
//   boxes    the ray in the box frame, o = (fmaf(ox, c, oy s), fmaf(oy, c,
//            -(ox s)), h), e = (fmaf(dx, c, dy s), fmaf(dy, c, -(dx s)), b)
//            with (ox, oy) = camera - box centre and (c, s) the heading
//            cosines, against the slabs [-L/2, L/2] x [-W/2, W/2] x [0, H]:
//            the entry is the largest per-axis entry (first axis on ties),
//            its face the side entered; a hit needs entry <= exit
//   roads    a downward ray meets z = 0 at s = -h / b, point (fmaf(s, dx, px),
//            fmaf(s, dy, py)); a strip holds it when its four edge cross
//            products fmaf(ex, wy, -(ey wx)) share one strict sign
//   lights   the raster's sphere test in camera space
//
// The tests are dealt by primitive, not by pixel: every ray starts at the
// camera, so a strip can only hold the ground points of the samples inside its
// image.  Per (strip, row) the columns that the strip can reach are computed
// with a margin (the slab of depths around the row's against the strip's
// edges, no projection and no clipping), and those it holds for certain; the
// exact test runs only for the samples between.  Boxes likewise by the
// rectangle of their (near-clipped) image: where the hit of a side is certain
// only its division is left.  Lights are tested inside their rectangle.
// One workgroup per view.  Strips are culled by bins and one by one into the
// view's ring (gp_view.h).  In rgb-only renders of scenes with one road
// colour (COV) strips leave coverage bits, the rows without boxes are written
// like the raster's; in the others they leave 32-bit key words in bands of rows
// (the strips of a row's sample have one depth: the largest word wins), and the
// road work is done again for each band.  64-bit keys are kept for box rows only,
// in bands of LDS.
//
// Bound by VALU issue.  One MI355X: 2,048 views at 128 x 128 (32 agents, 2,000
// strips) 110 us (1,100 us with the tests dealt by pixel; 218 us before the
// certain runs of boxes and strips were taken without the full test), 16 scenes
// of 8..64 agents, four cameras at 210 x 126, lit, with depth and ids 390 us
// (474 us with 64-bit keys of strips too, 2,400 us by pixel).
#include "gp_view.h"

namespace gp {

namespace {

constexpr int kRcPiece = 8;               // samples of one lane's certain box hits
constexpr int kRcTests = 4;               // samples of one lane's exact tests
constexpr int kRcNarrow = 12;             // items of fewer columns are tested whole
static_assert(kRcTests <= 16, "a piece's coverage bits fit the 32-bit pair below");

struct RcLayout {
    size_t cnt, bits, faces, sbins, sring, waves, pal, keys, road, total;
    int krows, region;
};

// LDS of one view: the band of 64-bit keys takes memory that is free by then, with
// COV that from sbins on behind the pattern table, without it that of the ring and
// the staging; the band of road keys (without COV) has its own
__host__ __device__ inline RcLayout rc_layout(int W, int H, const RcCfg &c)
{
    RcLayout l;
    l.road = 0;
    size_t o = 0;
    l.cnt = o; o = align16(o + 4 * R_NCNT);
    l.faces = o; o = align16(o + sizeof(FaceRec) * (size_t)c.bcap);
    l.bits = o;
    if (c.cover) o = align16(o + 8 * (((size_t)W * (size_t)(H - first_road_row(H)) + 63) / 64 + 1));
    l.pal = o;
    if (!c.cover) o = align16(o + 4 * 256);
    l.sbins = o; o = align16(o + 4 * (size_t)c.bins_cap);
    l.sring = o; o = align16(o + 4 * (size_t)kSharedRing);
    l.waves = o; o = align16(o + (size_t)kWaveBytes * (size_t)c.waves);
    const size_t band = 8 * (size_t)W * (size_t)c.band_rows;
    if (c.cover) {
        l.keys = l.sbins + kPatBytes;
        const size_t least = align16(l.keys + band);
        o = o > least ? o : least;
        l.region = (int)(o - l.keys);
    } else {
        // box keys in the memory of the ring and the staging, road keys behind them
        l.keys = l.sring;
        const size_t least = align16(l.keys + 8 * (size_t)W);
        o = o > least ? o : least;
        l.region = (int)(o - l.keys);
        l.road = o; o = align16(o + band / 2);
    }
    l.krows = l.region / (8 * W) > 0 ? l.region / (8 * W) : 1;
    l.total = o;
    return l;
}

// A staged strip (48 bytes): its world corners, its rows j0 | j1 << 16, key
// word (class 0) and margin
struct RcStrip {
    float x0, y0, x1, y1, x2, y2, x3, y3;
    int32_t rows;
    uint32_t keylo;
    float m;
    int32_t pad;
};
static_assert(sizeof(RcStrip) == 48, "staged strip size");

// What a row of samples sees of the ground: the ray parameter s = -h / b and
// the planar depth z = s f (the per-sample arithmetic's own values), and
// whether the depth is kept.
struct RcRow {
    float b, sp, z;
    bool ok;
};

__device__ __forceinline__ RcRow rc_row(const Cam &c, int j)
{
    RcRow r;
    r.b = c.cy - ((float)j + 0.5f);
    r.sp = -c.h / r.b;
    r.z = r.sp * c.f;
    r.ok = (r.b < 0.0f) & (r.z >= c.zn) & (r.z <= c.zf);
    return r;
}

// Camera-space depth of the ground seen by a sample at planar depth z is s2 z
// and its x is s2 s a, with s2 = fx^2 + fy^2 (1 for unit camera directions).
__device__ __forceinline__ float rc_scale2(const Cam &c) { return fmaf(c.fx, c.fx, c.fy * c.fy); }

// Rows [r0, r1) whose ground depth can lie within [zmin, zmax] (camera depth,
// margins included by the caller): j + 0.5 - cy = h f s2 / z; the slack covers
// the reciprocal's and the product's rounding (relative, 2^-20 of up to 1,024
// rows, doubled).
__device__ __forceinline__ bool rc_rows(const Cam &c, float hfs, float zmin, float zmax, int r0, int r1, int &j0, int &j1)
{
    if (!(zmax > 0.0f)) return false;
    const float lo = fmaf(hfs, __builtin_amdgcn_rcpf(zmax), c.cy) - 0.51f;
    float hi = (float)(r1 - 1);
    if (zmin > 0.0f) hi = fminf(hi, fmaf(hfs, __builtin_amdgcn_rcpf(zmin), c.cy) - 0.49f);
    j0 = max(r0, (int)fminf(ceilf(lo), (float)r1));
    j1 = (int)floorf(fmaxf(hi, -1.0f));
    return j0 <= j1;
}

// Margin in metres that dominates the rounding of the exact test: the ground
// point, its differences to the corners and the cross products are off by less
// than 2^-21 of the coordinates and distances in play.
__device__ __forceinline__ float rc_margin(const Cam &c, const float *x, const float *z)
{
    float r = fabsf(c.px) + fabsf(c.py);
#pragma unroll
    for (int k = 0; k < 4; ++k) r += fabsf(x[k]) + fabsf(z[k]);
    return fmaf(r, 0x1p-18f, 1e-4f);
}

// Conservative cull of a strip (or of a bin's box) with camera-space corners
// x, z against rows [r0, r1): the depths and the sides of the frustum that its
// ground points can lie in.
__device__ __forceinline__ bool rc_outside(const Cam &c, float hfs, const float *x, const float *z, int r0, int r1,
                                           int &j0, int &j1, float &m)
{
    m = rc_margin(c, x, z);
    bool l = true, r = true;
    float zmin = INFINITY, zmax = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float mk = 1e-3f * (fabsf(x[k]) + fabsf(z[k])) + m;
        r = r & (x[k] - c.t_right * z[k] > mk);
        l = l & (-x[k] - c.t_left * z[k] > mk);
        zmin = fminf(zmin, z[k]);
        zmax = fmaxf(zmax, z[k]);
    }
    return l | r | !rc_rows(c, hfs, zmin - m, zmax + m, r0, r1, j0, j1);
}

__device__ __forceinline__ void rc_corners(const Cam &c, const float4 &q0, const float4 &q1, float *x, float *z)
{
    ground_xz(c, q0.x, q0.y, x[0], z[0]);
    ground_xz(c, q0.z, q0.w, x[1], z[1]);
    ground_xz(c, q1.x, q1.y, x[2], z[2]);
    ground_xz(c, q1.z, q1.w, x[3], z[3]);
}

// Columns of row j whose samples the strip can hold: its extent in x over the
// depths within m of the row's, edge by edge.  (A point with four cross
// products of one strict sign lies inside the closed polygon, so between edge
// crossings of the row, also when the quad is not convex.)
__device__ __forceinline__ bool rc_columns(const Cam &c, const RcStrip &t, const RcRow &row, float s2, int &xl, int &xr)
{
    float x[4], z[4];
    rc_corners(c, make_float4(t.x0, t.y0, t.x1, t.y1), make_float4(t.x2, t.y2, t.x3, t.y3), x, z);
    const float zr = row.z * s2, m = fmaf(zr, 0x1p-18f, t.m);
    const float zlo = zr - m, zhi = zr + m;
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int k1 = (k + 1) & 3;
        const bool up = z[k] <= z[k1];
        const float za = up ? z[k] : z[k1], zb = up ? z[k1] : z[k], xa = up ? x[k] : x[k1], xb = up ? x[k1] : x[k];
        const float d = zb - za, inv = __builtin_amdgcn_rcpf(d);
        // an edge along the row counts whole
        const bool steep = d > m;
        const float t0 = steep ? fminf(fmaxf((zlo - za) * inv, 0.0f), 1.0f) : 0.0f;
        const float t1 = steep ? fminf(fmaxf((zhi - za) * inv, 0.0f), 1.0f) : 1.0f;
        const float e0 = fmaf(t0, xb - xa, xa), e1 = fmaf(t1, xb - xa, xa);
        const bool in = (zb >= zlo) & (za <= zhi);
        lo = in ? fminf(lo, fminf(e0, e1)) : lo;
        hi = in ? fmaxf(hi, fmaxf(e0, e1)) : hi;
    }
    const float ia = __builtin_amdgcn_rcpf(row.sp * s2);            // columns per metre
    const float al = fmaf(lo - m, ia, c.cx) - 0.52f, ar = fmaf(hi + m, ia, c.cx) - 0.48f;
    const float Wf = (float)c.W;
    xl = (int)ceilf(fminf(fmaxf(al, 0.0f), Wf));
    xr = (int)floorf(fminf(fmaxf(ar, -1.0f), Wf - 1.0f));
    return lo <= hi && xl <= xr;
}

// Columns [xl, xr] of a row cut down to those whose samples the strip holds
// for certain: along a row each cross product is affine in the column, and
// beyond the margin (in metres from each edge) its sign is the exact test's.
__device__ __forceinline__ void rc_inside(const Cam &c, const RcStrip &t, const RcRow &row, int &xl, int &xr)
{
    const float qx[4] = {t.x0, t.x1, t.x2, t.x3}, qy[4] = {t.y0, t.y1, t.y2, t.y3};
    // ground point of column offset a relative to the camera: P + a D
    const float Px = row.z * c.fx, Py = row.z * c.fy, Dx = row.sp * c.fy, Dy = -(row.sp * c.fx);
    const float area = (qx[2] - qx[0]) * (qy[3] - qy[1]) - (qy[2] - qy[0]) * (qx[3] - qx[1]);
    const float m = fmaf(row.z, 0x1p-18f, t.m);
    float al = -INFINITY, ar = INFINITY;
    bool ok = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float ux = qx[(e + 1) & 3] - qx[e], uy = qy[(e + 1) & 3] - qy[e];
        const float ex = area < 0.0f ? -ux : ux, ey = area < 0.0f ? -uy : uy;
        const float C = ex * (Py + (c.py - qy[e])) - ey * (Px + (c.px - qx[e])) - m * (fabsf(ex) + fabsf(ey));
        const float G = ex * Dy - ey * Dx;
        const float r = -C * __builtin_amdgcn_rcpf(G);
        al = G > 0.0f ? fmaxf(al, r) : al;
        ar = G < 0.0f ? fminf(ar, r) : ar;
        ok = ok & ((G != 0.0f) | (C > 0.0f));
    }
    const int l = max(xl, (int)ceilf(fminf(fmaxf(al + c.cx - 0.48f, -1.0f), 2048.0f)));
    const int r = min(xr, (int)floorf(fminf(fmaxf(ar + c.cx - 0.52f, -2.0f), 2048.0f)));
    xl = l;
    xr = ok ? r : -1;
}

// One set-up job: the n ring strips from a staged, their (strip, row) items on
// rows [b0, b1) dealt to the lanes by a prefix over row counts, the items'
// columns cut into pieces, dealt again: without COV the certain ones of up to 16
// samples, the others of up to kRcTests, with the exact test run per sample.  Without COV the strips' key words are folded into the
// band of road keys (from row band0): every strip lies in one plane, so the
// largest key word of a row's sample names the strip it shows.
template <bool COV>
__device__ __forceinline__ void rc_strips(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L,
                                          lptr<RcStrip> st, lptr<uint32_t> road, float hfs, float s2, int a, int n, int b0,
                                          int b1, int band0)
{
    const int ln = (int)lane_id(), W = cam.W;
    wave_lds_order();
    int rows = 0;
    if (ln < n) {
        const int g = L.sring[a + ln];
        const float4 q0 = s.roads[2 * g], q1 = s.roads[2 * g + 1];
        float x[4], z[4];
        rc_corners(cam, q0, q1, x, z);
        int j0, j1;
        RcStrip t;
        if (!rc_outside(cam, hfs, x, z, b0, b1, j0, j1, t.m)) rows = j1 - j0 + 1;
        t.x0 = q0.x; t.y0 = q0.y; t.x1 = q0.z; t.y1 = q0.w; t.x2 = q1.x; t.y2 = q1.y; t.x3 = q1.z; t.y3 = q1.w;
        t.rows = j0 | (j1 << 16);
        t.keylo = COV ? 0u : key_low(0u, 6 * (sc.n_agents + sc.n_static) + s.road_index[g], s.road_color[g]);
        t.pad = 0;
        lds_store(st + ln, t);
    }
    const int incl = wave_incl_scan(rows);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int excl = incl - rows;
    wave_lds_order();
    for (int g0 = 0; g0 < total; g0 += 64) {
        const int gi = g0 + ln;
        const int o = owner_of(incl, gi);
        const int ex = __shfl(excl, o);
        int xl = 0, xr = -1, yl = W, yr = -1, j = 0;
        if (gi < total) {
            const RcStrip t = lds_load(st + o);
            j = (t.rows & 0xFFFF) + (gi - ex);
            const RcRow row = rc_row(cam, j);
            if (!(row.ok && rc_columns(cam, t, row, s2, xl, xr))) { xl = 0; xr = -1; }
            if (xr - xl >= kRcNarrow) {
                yl = xl;
                yr = xr;
                rc_inside(cam, t, row, yl, yr);
            }
            if (yl > yr) {                                  // no certain column: all lie left of xr + 1
                yl = xr + 1;
                yr = xr;
            }
            if (COV && yl <= yr) or_span(L.bits, (j - L.hr0) * W + yl, (j - L.hr0) * W + yr);
        }
        if (!COV) {
            // the certain columns' keys
            const int nc = yl <= yr ? (yr - yl + 16) >> 4 : 0;
            const int inc2 = wave_incl_scan(nc);
            const int npt = __builtin_amdgcn_readlane(inc2, 63);
            const int ex2 = inc2 - nc;
            for (int p0 = 0; p0 < npt; p0 += 64) {
                const int pi = p0 + ln;
                const int o2 = owner_of(inc2, pi);
                const int k = pi - __shfl(ex2, o2);
                const int syl = __shfl(yl, o2), syr = __shfl(yr, o2), sj = __shfl(j, o2), so = __shfl(o, o2);
                if (pi >= npt) continue;
                const int i0 = syl + 16 * k, i1 = min(i0 + 15, syr);
                const uint32_t key = ((lptr<const uint32_t>)(st + so))[9];
                lptr<uint32_t> kp = road + (sj - band0) * W;
                for (int i = i0; i <= i1; ++i) lds_max32(kp + i, key);
            }
        }
        const int nl = (yl - xl + kRcTests - 1) / kRcTests;
        const int np = xl <= xr ? nl + (xr - yr + kRcTests - 1) / kRcTests : 0;
        const int inc2 = wave_incl_scan(np);
        const int npt = __builtin_amdgcn_readlane(inc2, 63);
        const int ex2 = inc2 - np;
        const int x2 = xl | (xr << 16), y2 = yl | (yr << 16);
        for (int p0 = 0; p0 < npt; p0 += 64) {
            const int pi = p0 + ln;
            const int o2 = owner_of(inc2, pi);
            const int k = pi - __shfl(ex2, o2);
            const int sx = __shfl(x2, o2), sy = __shfl(y2, o2), sj = __shfl(j, o2), so = __shfl(o, o2);
            if (pi >= npt) continue;
            const int sxl = sx & 0xFFFF, sxr = sx >> 16, syl = sy & 0xFFFF, syr = sy >> 16;
            const int snl = (syl - sxl + kRcTests - 1) / kRcTests;
            const int i0 = k < snl ? sxl + kRcTests * k : syr + 1 + kRcTests * (k - snl);
            const int i1 = min(i0 + kRcTests, k < snl ? syl : sxr + 1) - 1;
            const RcStrip t = lds_load(st + so);
            const RcRow row = rc_row(cam, sj);
            const float qx[4] = {t.x0, t.x1, t.x2, t.x3}, qy[4] = {t.y0, t.y1, t.y2, t.y3};
            float ex4[4], ey4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ex4[e] = qx[(e + 1) & 3] - qx[e];
                ey4[e] = qy[(e + 1) & 3] - qy[e];
            }
            uint32_t in = 0u;
            for (int i = i0; i <= i1; ++i) {
                const float av = ((float)i + 0.5f) - cam.cx;
                const float dx = fmaf(av, cam.fy, cam.f * cam.fx), dy = fmaf(av, -cam.fx, cam.f * cam.fy);
                const float x = fmaf(row.sp, dx, cam.px), y = fmaf(row.sp, dy, cam.py);
                bool pos = true, neg = true;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float c = fmaf(ex4[e], y - qy[e], -(ey4[e] * (x - qx[e])));
                    pos = pos & (c > 0.0f);
                    neg = neg & (c < 0.0f);
                }
                in |= (uint32_t)(pos | neg) << (i - i0);
            }
            if (in == 0u) continue;
            if (COV) {
                const int b = (sj - L.hr0) * W + i0;
                const unsigned long long m = (unsigned long long)in << (b & 31);
                lptr<uint32_t> w = (lptr<uint32_t>)L.bits + (b >> 5);
                lds_or32(w, (uint32_t)m);
                if ((uint32_t)(m >> 32)) lds_or32(w + 1, (uint32_t)(m >> 32));
            } else {
                lptr<uint32_t> kp = road + (sj - band0) * W + i0;
                for (; in != 0u; in &= in - 1u) lds_max32(kp + (__ffs((int)in) - 1), t.keylo);
            }
        }
    }
    wave_lds_order();
}

// store entry t of the list, named by its key word's low byte
__device__ __forceinline__ void list_entry(const RgbLds &L, bool has, int t, FaceRec f)
{
    f.keylo |= (uint32_t)t & 0xFFu;
    if (has) lds_store(L.faces + t, f);
}

// Colour of a winning box or light key: of its list entry's side, or (the list
// was filled in chunks) from the scene.
__device__ __forceinline__ uint32_t rc_color(const DevSim &s, const SceneRec &sc, const RgbLds &L, bool chunked, uint32_t keylo)
{
    const int prim = (kMaxPrims - 1) - (int)((keylo >> 8) & (uint32_t)(kMaxPrims - 1));
    const int nbox = sc.n_agents + sc.n_static;
    const int face = prim < 6 * nbox ? prim % 6 : 4;
    if (chunked) return streamed_rgb<true>(s, sc, keylo);
    const int word = face >= 4 ? 14 : ((face & 1) ? 10 : 9);
    return ((lptr<const uint32_t>)(L.faces + (keylo & 0xFFu)))[word];
}

// Box unit: boxes [u0, u0 + n) of the scene (n <= 64) against the view: an
// entry holds the box (centre, heading cosines, half sizes, height) and the
// pixel rectangle that every sample whose ray can hit it lies in: the hull of
// the images of its footprint's corners, clipped just before the near plane,
// at the ground and at its top (a pixel of margin for rounding).
__device__ __forceinline__ void rc_boxes(const DevSim &s, const SceneRec &sc, const Cam &cam, int ego, const RgbLds &L,
                                         float s2, int u0, int n)
{
    const int ln = (int)lane_id();
    const int u = u0 + ln;
    bool keep = false;
    FaceRec f = {};
    if (ln < n && u < sc.n_agents + sc.n_static && u != ego) {
        const int g = box_slot(sc, u);
        const float4 st = s.state[g], dm = s.dims[g];
        const float2 cs = s.cs[g];
        const float ox = st.x - cam.px, oy = st.y - cam.py;
        const float ax = 0.5f * dm.x * cs.x, ay = 0.5f * dm.x * cs.y, bx = -(0.5f * dm.y * cs.y), by = 0.5f * dm.y * cs.x;
        float x[4], z[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float sa = k == 0 || k == 1 ? 1.0f : -1.0f, sb = k == 0 || k == 3 ? -1.0f : 1.0f;
            const float wx = ox + sa * ax + sb * bx, wy = oy + sa * ay + sb * by;
            z[k] = fmaf(wx, cam.fx, wy * cam.fy);
            x[k] = fmaf(wx, cam.fy, -(wy * cam.fx));
        }
        // hits lie at planar depth >= z_near, camera depth >= s2 z_near
        const float zc = 0.99f * (cam.zn * s2);
        const float vt = (dm.z - cam.h) * cam.f * s2, vg = -cam.h * cam.f * s2;
        float umin = INFINITY, umax = -INFINITY, vmin = INFINITY, vmax = -INFINITY, zmin = INFINITY;
        auto point = [&](float px, float pz) {
            const float iz = 1.0f / pz;
            const float uu = fmaf(cam.f * px, iz, cam.cx);
            umin = fminf(umin, uu);
            umax = fmaxf(umax, uu);
            const float v0 = fmaf(-vg, iz, cam.cy), v1 = fmaf(-vt, iz, cam.cy);
            vmin = fminf(vmin, fminf(v0, v1));
            vmax = fmaxf(vmax, fmaxf(v0, v1));
        };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int k1 = (k + 1) & 3;
            zmin = fminf(zmin, z[k]);
            if (z[k] >= zc) point(x[k], z[k]);
            if ((z[k] >= zc) != (z[k1] >= zc)) point(fmaf((zc - z[k]) / (z[k1] - z[k]), x[k1] - x[k], x[k]), zc);
        }
        const float Wf = (float)cam.W, Hf = (float)cam.H;
        int i0 = max(0, (int)fminf(fmaxf(floorf(umin - 0.5f) - 1.0f, -1.0f), Wf));
        int i1 = min(cam.W - 1, (int)fminf(fmaxf(ceilf(umax - 0.5f) + 1.0f, -1.0f), Wf));
        int j0 = max(0, (int)fminf(fmaxf(floorf(vmin - 0.5f) - 1.0f, -1.0f), Hf));
        int j1 = min(cam.H - 1, (int)fminf(fmaxf(ceilf(vmax - 0.5f) + 1.0f, -1.0f), Hf));
        keep = (umin <= umax) & !(zmin > 1.01f * (cam.zf * s2)) & (i0 <= i1) & (j0 <= j1);
        // A negative size turns a box inside out (its exit comes before its entry:
        // no hit), and where a corner is 100 km off or no number at all neither a
        // crossing of the near plane nor the runs of rc_certain are to be relied on:
        // such boxes take the slab test of every sample, of the whole image where
        // they reach behind the near plane
        const float far = fabsf(ox) + fabsf(oy) + fabsf(ax) + fabsf(ay) + fabsf(bx) + fabsf(by);
        const bool plain = (dm.x >= 0.0f) & (dm.y >= 0.0f) & (dm.z >= 0.0f) & (dm.z < 1e5f) & (far < 1e5f);
        if (!plain & (zmin < zc)) {
            i0 = j0 = 0;
            i1 = cam.W - 1;
            j1 = cam.H - 1;
            keep = true;
        }
        f.X0 = __float_as_int(st.x); f.Y0 = __float_as_int(st.y);
        f.X1 = __float_as_int(cs.x); f.Y1 = __float_as_int(cs.y);
        f.X2 = __float_as_int(0.5f * dm.x); f.Y2 = __float_as_int(0.5f * dm.y);
        f.X3 = i0; f.Y3 = i1;
        f.A = dm.z;
        // colours of the sides facing the camera: across the length, across the
        // width, the top
        const float px = cam.px - st.x, py = cam.py - st.y;
        const bool front = fmaf(px, cs.x, py * cs.y) > 0.0f, left = fmaf(py, cs.x, -(px * cs.y)) > 0.0f;
        const uint32_t c = s.box_rgb[g];
        f.B = __uint_as_float(s.shade ? lit_face(s, sc, c, u, front ? 0 : 2) : c);
        f.C = __uint_as_float(s.shade ? lit_face(s, sc, c, u, left ? 1 : 3) : c);
        f.rgb = s.shade ? lit_face(s, sc, c, u, 4) : c;
        f.keylo = key_low(1u, 6 * u, 0u);
        f.j0 = (int16_t)j0; f.j1 = (int16_t)j1;
        f.nv = 1;
        f.huge = !plain;
    }
    const unsigned long long bm = __ballot(keep);
    int nbt = 0;
    const int at = box_reserve(L, true, nbt, __popcll(bm));
    list_entry(L, keep && at >= 0, at + lanes_below(bm), f);
    int bmin = keep ? (int)f.j0 : 0x7FFFFFFF, bmax = keep ? (int)f.j1 : -1;
    box_rows(L, bmin, bmax);
}

// Traffic lights [u0, u0 + 64): light_pass's entries.
__device__ __forceinline__ void rc_lights(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, int u0)
{
    const int u = u0 + (int)lane_id();
    bool keep = false;
    FaceRec f = {};
    if (u < sc.n_signals) {
        const float4 q = s.signals[sc.signal_base + u];
        const V3 c = to_cam(cam, q.x - cam.px, q.y - cam.py, q.z);
        int i0, i1, j0, j1;
        keep = signal_bounds(cam, c, q.w, i0, i1, j0, j1);
        f.X0 = __float_as_int(c.x); f.Y0 = __float_as_int(c.y); f.X1 = __float_as_int(c.z);
        f.Y1 = __float_as_int(q.w * q.w); f.X2 = __float_as_int(cam.f * c.z);
        f.X3 = i0; f.Y3 = i1;
        f.j0 = (int16_t)j0; f.j1 = (int16_t)j1;
        f.keylo = key_low(1u, 6 * (sc.n_agents + sc.n_static) + sc.n_roads + u, 0u);
        f.rgb = signal_rgb(s, sc, u);
    }
    const unsigned long long bm = __ballot(keep);
    int nbt = 0;
    const int at = box_reserve(L, true, nbt, __popcll(bm));
    list_entry(L, keep && at >= 0, at + lanes_below(bm), f);
    box_rows(L, keep ? (int)f.j0 : 0x7FFFFFFF, keep ? (int)f.j1 : -1);
}

// the key of the box entry's hit at the sample offsets a, b, or 0
__device__ __forceinline__ unsigned long long rc_box_key(const Cam &cam, const float *o, const float *half, float cb,
                                                         float sb, float Hb, uint32_t keylo, float a, float b)
{
    const float dx = fmaf(a, cam.fy, cam.f * cam.fx), dy = fmaf(a, -cam.fx, cam.f * cam.fy);
    const float e0 = fmaf(dx, cb, dy * sb), e1 = fmaf(dy, cb, -(dx * sb)), e2 = b;
    float t_in = -INFINITY, t_out = INFINITY;
    int face = -1;
    // the slab lo .. hi of an axis: entry and exit, the side entered (flo for a
    // positive direction, fhi for a negative one)
    auto axis = [&](float e, float p, float lo, float hi, int flo, int fhi) {
        float en, lv;
        int fk;
        if (e != 0.0f) {
            const bool up = e > 0.0f;
            en = ((up ? lo : hi) - p) / e;
            lv = ((up ? hi : lo) - p) / e;
            fk = up ? flo : fhi;
        } else {
            const bool in = lo < p && p < hi;
            en = in ? -INFINITY : INFINITY;
            lv = in ? INFINITY : -INFINITY;
            fk = -1;
        }
        if (en > t_in) {
            t_in = en;
            face = fk;
        }
        t_out = fminf(t_out, lv);
    };
    axis(e0, o[0], -half[0], half[0], 2, 0);
    axis(e1, o[1], -half[1], half[1], 3, 1);
    axis(e2, cam.h, 0.0f, Hb, 5, 4);
    if (!((t_in <= t_out) & (t_in > 0.0f) & (t_in < INFINITY))) return 0ull;
    const float z = t_in * cam.f;
    if (!((z >= cam.zn) & (z <= cam.zf))) return 0ull;
    return ((unsigned long long)__float_as_uint(1.0f / z) << 32) | (keylo - ((uint32_t)face << 8));
}

// The columns of row offset b on which a box's hit is certain, by the side
// entered: segs[] holds up to three disjoint runs l << 16 | r << 2 | axis in
// column order (unused ones last, l = W).  Along a row the ray's direction in
// the box frame is affine in the column offset a, e_k = A_k + B_k a, so the hit
// at t = N / e_k of the side facing the camera on axis k lies inside the other
// two slabs, and within [z_near, z_far], where seven affine functions of a are
// positive.  The margin (2^-16 of the distances in play) dominates the rounding
// of the exact test, so on these columns that test takes this side and
// accepts the hit: only its division is left to do.  (Boxes of finite sizes that
// are not negative: else the runs need be neither right nor disjoint.)
__device__ __forceinline__ void rc_certain(const Cam &cam, const FaceRec &f, float b, int xl, int xr, int *segs)
{
    const float cb = __int_as_float(f.X1), sb = __int_as_float(f.Y1);
    const float ox = cam.px - __int_as_float(f.X0), oy = cam.py - __int_as_float(f.Y0);
    const float p[3] = {fmaf(ox, cb, oy * sb), fmaf(oy, cb, -(ox * sb)), cam.h};
    const float lo[3] = {-__int_as_float(f.X2), -__int_as_float(f.Y2), 0.0f};
    const float hi[3] = {-lo[0], -lo[1], f.A};
    const float ca = cam.fx * cb + cam.fy * sb, sa = cam.fy * cb - cam.fx * sb;     // forward in the box frame
    const float A[3] = {cam.f * ca, cam.f * sa, b}, B[3] = {sa, -ca, 0.0f};
    const float mu = fmaf(fabsf(ox) + fabsf(oy) + cam.h + hi[0] + hi[1] + hi[2], 0x1p-16f, 1e-5f);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        segs[k] = (cam.W << 16) | (int)((uint32_t)(cam.W - 1) << 2);
        // the side facing the camera, and the direction's sign towards it
        const bool above = p[k] > hi[k], below = p[k] < lo[k];
        const float sg = above ? -1.0f : 1.0f;
        const float M = above ? p[k] - hi[k] : lo[k] - p[k];
        const float E0 = sg * A[k], E1 = sg * B[k];
        float al = -INFINITY, ar = INFINITY;
        bool ok = above | below;
        auto positive = [&](float F0, float F1) {            // F0 + F1 a > 0
            const float r = -F0 * __builtin_amdgcn_rcpf(F1);
            al = F1 > 0.0f ? fmaxf(al, r) : al;
            ar = F1 < 0.0f ? fminf(ar, r) : ar;
            ok = ok & ((F1 != 0.0f) | (F0 > 0.0f));
        };
        positive(E0 - 1e-6f * cam.f, E1);
        positive(M * cam.f - 1.0001f * (cam.zn * E0), -1.0001f * (cam.zn * E1));
        positive(0.9999f * (cam.zf * E0) - M * cam.f, 0.9999f * (cam.zf * E1));
#pragma unroll
        for (int q = 1; q < 3; ++q) {
            const int m = (k + q) % 3;
            const float u = hi[m] - mu - p[m], v = p[m] - lo[m] - mu;
            positive(fmaf(u, E0, -(M * A[m])), fmaf(u, E1, -(M * B[m])));
            positive(fmaf(v, E0, M * A[m]), fmaf(v, E1, M * B[m]));
        }
        // whole columns, 2% of a column inside
        const int l = max(xl, (int)ceilf(fminf(fmaxf(al + cam.cx - 0.48f, -1.0f), 2048.0f)));
        const int r = min(xr, (int)floorf(fminf(fmaxf(ar + cam.cx - 0.52f, -2.0f), 2048.0f)));
        if (ok & (l <= r)) segs[k] = (l << 16) | (r << 2) | k;
    }
    // column order
    const int s01 = min(segs[0], segs[1]), l01 = max(segs[0], segs[1]);
    segs[0] = min(s01, segs[2]);
    const int t = max(s01, segs[2]);
    segs[1] = min(l01, t);
    segs[2] = max(l01, t);
}

// Fragments of the list's n entries in rows [b0, b1) folded into the key band.
// The (entry, row) items are dealt to the lanes; an item's columns are the
// certain runs above and what is left between them, cut into pieces that are
// dealt again: certain pieces take one division a sample for the hit, the
// others the full test.  Passes of 64 items are shared out over the wavefronts;
// where there are fewer passes than wavefronts, several set up the same pass and
// share its pieces (one box near the camera can hold most of a view's samples).
__device__ __forceinline__ void rc_band(const RgbLds &L, const Cam &cam, int n, int b0, int b1, int wv, int nwv)
{
    const int ln = (int)lane_id(), W = cam.W;
    int pass = 0;
    for (int t0 = 0; t0 < n; t0 += 64) {
        const int t = t0 + ln;
        int c = 0, first = 0;
        if (t < n) {
            const int32_t jj = ((lptr<const int32_t>)(L.faces + t))[12];
            first = max((int)(int16_t)(jj & 0xFFFF), b0);
            c = max(0, min(jj >> 16, b1 - 1) - first + 1);
        }
        const int incl = wave_incl_scan(c);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int excl = incl - c;
        // a pass of 64 items goes to one of the groups of gsz wavefronts
        const int gsz = max(1, nwv / max(1, (total + 63) >> 6)), groups = nwv / gsz, mine = wv / gsz, wi = wv - mine * gsz;
        for (int g0 = 0; g0 < total; g0 += 64, ++pass) {
            if (pass % groups != mine) continue;
            const int gi = g0 + ln;
            const int o = owner_of(incl, gi);
            const int j = __shfl(first, o) + (gi - __shfl(excl, o));
            int xl = 0, xr = -1;
            const int none = (W << 16) | ((W - 1) << 2);
            int segs[3] = {none, none, none};
            int nq = 0, nu = 0;
            if (gi < total) {
                const FaceRec f = lds_load(L.faces + t0 + o);
                xl = f.X3;
                xr = f.Y3;
                if (f.nv != 0 && f.huge == 0) rc_certain(cam, f, cam.cy - ((float)j + 0.5f), xl, xr, segs);
                int at = xl;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int l = segs[k] >> 16, r = (segs[k] >> 2) & 0x3FFF;
                    if (l > r) continue;
                    nq += (r - l + kRcPiece) / kRcPiece;
                    nu += (l - at + kRcTests - 1) / kRcTests;
                    at = r + 1;
                }
                nu += (xr - at + kRcTests) / kRcTests;
            }
            // ---- certain pieces
            {
                const int inc2 = wave_incl_scan(nq);
                const int npt = __builtin_amdgcn_readlane(inc2, 63);
                const int ex2 = inc2 - nq;
                for (int p0 = 64 * wi; p0 < npt; p0 += 64 * gsz) {
                    const int pi = p0 + ln;
                    const int o2 = owner_of(inc2, pi);
                    int k = pi - __shfl(ex2, o2);
                    const int sj = __shfl(j, o2), so = t0 + __shfl(o, o2);
                    const int g[3] = {__shfl(segs[0], o2), __shfl(segs[1], o2), __shfl(segs[2], o2)};
                    if (pi >= npt) continue;
                    int i0 = 0, i1 = -1, axis = 0;
                    bool found = false;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const int l = g[q] >> 16, r = (g[q] >> 2) & 0x3FFF;
                        const int np = l <= r ? (r - l + kRcPiece) / kRcPiece : 0;
                        if (!found && k < np) {
                            i0 = l + kRcPiece * k;
                            i1 = min(i0 + kRcPiece - 1, r);
                            axis = g[q] & 3;
                            found = true;
                        }
                        k -= np;
                    }
                    const float b = cam.cy - ((float)sj + 0.5f);
                    lptr<unsigned long long> kp = L.work + (sj - b0) * W;
                    const FaceRec f = lds_load(L.faces + so);
                    const float cb = __int_as_float(f.X1), sb = __int_as_float(f.Y1);
                    const float ox = cam.px - __int_as_float(f.X0), oy = cam.py - __int_as_float(f.Y0);
                    const float pk = axis == 0 ? fmaf(ox, cb, oy * sb) : (axis == 1 ? fmaf(oy, cb, -(ox * sb)) : cam.h);
                    const float hk = axis == 0 ? __int_as_float(f.X2) : (axis == 1 ? __int_as_float(f.Y2) : f.A);
                    const bool above = pk > 0.0f;            // the camera is beyond the side hk (else beyond -hk)
                    const float num = (above ? hk : -hk) - pk;
                    const int face = axis == 2 ? 4 : (axis == 0 ? (above ? 0 : 2) : (above ? 1 : 3));
                    const uint32_t keylo = f.keylo - ((uint32_t)face << 8);
                    const float s1 = axis == 0 ? sb : -sb;
                    for (int i = i0; i <= i1; ++i) {
                        const float a = ((float)i + 0.5f) - cam.cx;
                        const float dx = fmaf(a, cam.fy, cam.f * cam.fx), dy = fmaf(a, -cam.fx, cam.f * cam.fy);
                        float e = axis == 0 ? fmaf(dx, cb, dy * s1) : fmaf(dy, cb, dx * s1);
                        e = axis == 2 ? b : e;
                        const float z = (num / e) * cam.f;
                        lds_max64(kp + i, ((unsigned long long)__float_as_uint(1.0f / z) << 32) | keylo);
                    }
                }
            }
            // ---- the rest
            const int inc2 = wave_incl_scan(nu);
            const int npt = __builtin_amdgcn_readlane(inc2, 63);
            const int ex2 = inc2 - nu;
            for (int p0 = 64 * wi; p0 < npt; p0 += 64 * gsz) {
                const int pi = p0 + ln;
                const int o2 = owner_of(inc2, pi);
                int k = pi - __shfl(ex2, o2);
                const int sj = __shfl(j, o2), so = t0 + __shfl(o, o2);
                const int sxl = __shfl(xl, o2), sxr = __shfl(xr, o2);
                const int g[3] = {__shfl(segs[0], o2), __shfl(segs[1], o2), __shfl(segs[2], o2)};
                if (pi >= npt) continue;
                int i0 = 0, i1 = -1, at = sxl;
                bool found = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    // the gap before run q, or after the last one
                    const int l = q < 3 ? g[q < 3 ? q : 0] >> 16 : sxr + 1, r = q < 3 ? (g[q < 3 ? q : 0] >> 2) & 0x3FFF : sxr;
                    if (q < 3 && l > r) continue;
                    const int np = (l - at + kRcTests - 1) / kRcTests;
                    if (!found && k < np) {
                        i0 = at + kRcTests * k;
                        i1 = min(i0 + kRcTests, l) - 1;
                        found = true;
                    }
                    k -= np;
                    at = r + 1;
                }
                const float b = cam.cy - ((float)sj + 0.5f);
                lptr<unsigned long long> kp = L.work + (sj - b0) * W;
                const FaceRec f = lds_load(L.faces + so);
                if (f.nv == 0) {
                    for (int i = i0; i <= i1; ++i) {
                        const float invz = light_invz(L, cam, so, ((float)i + 0.5f) - cam.cx, b);
                        if (invz > 0.0f) lds_max64(kp + i, ((unsigned long long)__float_as_uint(invz) << 32) | f.keylo);
                    }
                    continue;
                }
                const float cb = __int_as_float(f.X1), sb = __int_as_float(f.Y1);
                const float ox = cam.px - __int_as_float(f.X0), oy = cam.py - __int_as_float(f.Y0);
                const float og[2] = {fmaf(ox, cb, oy * sb), fmaf(oy, cb, -(ox * sb))};
                const float half[2] = {__int_as_float(f.X2), __int_as_float(f.Y2)};
                for (int i = i0; i <= i1; ++i) {
                    const unsigned long long key = rc_box_key(cam, og, half, cb, sb, f.A, f.keylo, ((float)i + 0.5f) - cam.cx, b);
                    if (key != 0ull) lds_max64(kp + i, key);
                }
            }
        }
    }
}

// Bins [s0, s1) of the scene whose strips some row below the horizon can see, into
// the view's list (R_NSB counts them all, also those that it cannot hold).
__device__ __forceinline__ void rc_cull(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, float hfs, int H,
                                        int s0, int s1, int wv, int B)
{
    for (int b0 = s0 + 64 * wv; b0 < s1; b0 += B) {
        const int b = b0 + (int)lane_id();
        bool keep = false;
        int rec = 0;
        if (b < s1) {
            const RoadBin bn = s.bins[sc.bin_base + b];
            float x[4], z[4], m;
            int j0, j1;
            rc_corners(cam, make_float4(bn.xmin, bn.ymin, bn.xmax, bn.ymin), make_float4(bn.xmax, bn.ymax, bn.xmin, bn.ymax),
                       x, z);
            keep = !rc_outside(cam, hfs, x, z, L.hr0, H, j0, j1, m);
            rec = bn.start * 128 + bn.count;
        }
        const unsigned long long bm = __ballot(keep);
        if (bm == 0ull) continue;
        int at = 0;
        if (lane_id() == 0) at = lds_add(L.cnt + R_NSB, __popcll(bm));
        at = __builtin_amdgcn_readlane(at, 0) + lanes_below(bm);
        if (keep && at < L.bins) L.sbins[at] = rec;
    }
}

// SEG: the scene may have more bins than the list holds (instances of their own:
// the segments' state spills 35 scalar registers more, 3% of a render of the others)
template <bool COV, bool SEG>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_raycast(DevSim s, RenderOut o, RcCfg c,
                                                                                         int view_begin)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int B = (int)blockDim.x, K = B >> 6, tid = (int)threadIdx.x, wv = tid >> 6;
    const int W = s.width, H = s.height;
    const RcLayout l = rc_layout(W, H, c);
    RgbLds L;
    L.cnt = (lptr<int32_t>)(smem + l.cnt);
    L.bits = (lptr<unsigned long long>)(smem + l.bits);
    L.faces = (lptr<FaceRec>)(smem + l.faces);
    L.sbins = (lptr<int32_t>)(smem + l.sbins);
    L.cq = nullptr;
    L.sring = (lptr<int32_t>)(smem + l.sring);
    L.waves = (lptr<unsigned char>)(smem + l.waves);
    L.pat = (lptr<gp_v4i>)(smem + l.sbins);
    L.work = (lptr<unsigned long long>)(smem + l.keys);
    L.bcap = c.bcap;
    L.krows = l.krows;
    L.hr0 = first_road_row(H);
    L.batch = kBatch;
    L.ring = kSharedRing;
    L.bins = c.bins_cap;
    L.nrec = 0;
    L.nmw = 0;
    L.region = l.region;
    lptr<uint32_t> pal = (lptr<uint32_t>)(smem + l.pal), road = (lptr<uint32_t>)(smem + l.road);

    const ViewInit vi = view_init(s.vorder + view_begin + (int)blockIdx.x);
    const int view = vi.view, ego = vi.ego;
    const SceneRec &sc = vi.sc;
    const Cam cam = make_cam(s, sc, ego, vi.cam);
    const float s2 = uniform_f(rc_scale2(cam));
    const float hfs = uniform_f(cam.h * cam.f * s2);

    if (COV) {
        const int nbits = ((W * (H - L.hr0) + 63) >> 6) + 1;
        for (int p = tid; p < nbits; p += B) L.bits[p] = 0ull;
    } else {
        road_palette(s, pal);
    }
    if (tid < R_NCNT) L.cnt[tid] = tid == R_BMIN ? 0x7FFFFFFF : (tid == R_BMAX ? -1 : 0);
    __syncthreads();

    // ---- bins of the scene whose strips some row can see
    // (with segments: below; called through rc_cull this loop costs a few spilled
    // registers more, 1.5% of a render with labels)
    for (int b0 = 64 * wv; !SEG && b0 < sc.n_bins; b0 += B) {
        const int b = b0 + (int)lane_id();
        bool keep = false;
        int rec = 0;
        if (b < sc.n_bins) {
            const RoadBin bn = s.bins[sc.bin_base + b];
            float x[4], z[4], m;
            int j0, j1;
            rc_corners(cam, make_float4(bn.xmin, bn.ymin, bn.xmax, bn.ymin), make_float4(bn.xmax, bn.ymax, bn.xmin, bn.ymax),
                       x, z);
            keep = !rc_outside(cam, hfs, x, z, L.hr0, H, j0, j1, m);
            rec = bn.start * 128 + bn.count;
        }
        const unsigned long long bm = __ballot(keep);
        if (bm == 0ull) continue;
        int at = 0;
        if (lane_id() == 0) at = lds_add(L.cnt + R_NSB, __popcll(bm));
        at = __builtin_amdgcn_readlane(at, 0) + lanes_below(bm);
        if (keep) L.sbins[at] = rec;
    }
    __syncthreads();
    const int nsb = L.cnt[R_NSB];
    lptr<RcStrip> st = (lptr<RcStrip>)(L.waves + (size_t)wv * kWaveBytes);

    // The list holds every box and light of the scene, or (chunked) is filled and
    // folded in chunks of candidates per band.
    const int nbox = sc.n_agents + sc.n_static, ncand = nbox + sc.n_signals;
    const bool chunked = ncand > c.bcap;
    const int ub = K >= 8 ? 16 : 64;
    const int nbu = (nbox + ub - 1) / ub, nlu = (sc.n_signals + 63) / 64;
    auto box_job = [&](int u) {
        if (u < nbu) rc_boxes(s, sc, cam, ego, L, s2, ub * u, ub);
        else rc_lights(s, sc, cam, L, 64 * (u - nbu));
    };
    // the strips on rows [b0, b1) and the jobs before them; SEG: where more bins
    // survive than the list holds, the scene's bins in segments that it does hold
    // (what strips leave is OR-ed or folded, so their order is free).  Ends with a
    // barrier.
    bool listed = false, over = false;           // (SEG) the list holds the survivors; there are more
    auto roads = [&](int jobs, int b0, int b1) {
        auto test = [&](bool live, const float4 &q0, const float4 &q1) -> bool {
            float x[4], z[4], m;
            int j0, j1;
            rc_corners(cam, q0, q1, x, z);
            return live && !rc_outside(cam, hfs, x, z, b0, b1, j0, j1, m);
        };
        auto strips = [&](int a, int n) { rc_strips<COV>(s, sc, cam, L, st, road, hfs, s2, a, n, b0, b1, b0); };
        if constexpr (!SEG) {
            road_work(s, sc, L, b0 < b1 ? nsb : 0, jobs, test, box_job, strips);
        } else {
            for (int s0 = 0;;) {
                if (!listed) {
                    __syncthreads();             // the counters are read
                    if (tid == 0) L.cnt[R_NSB] = L.cnt[R_RING] = L.cnt[R_JOB] = 0;
                    __syncthreads();
                    rc_cull(s, sc, cam, L, hfs, H, s0, over ? min(s0 + L.bins, sc.n_bins) : sc.n_bins, wv, B);
                    __syncthreads();
                    const bool fits = L.cnt[R_NSB] <= L.bins;
                    listed = fits & !over;
                    if (!fits) {
                        over = true;
                        continue;
                    }
                }
                road_work(s, sc, L, b0 < b1 ? L.cnt[R_NSB] : 0, jobs, test, box_job, strips);
                jobs = 0;
                s0 += L.bins;
                if (!over || s0 >= sc.n_bins) return;
            }
        }
    };
    // the entries of rows [b0, b1) folded into the (cleared) key band; ends with a barrier
    auto boxes = [&](int b0, int b1) {
        if (!chunked) {
            rc_band(L, cam, L.cnt[R_NBT], b0, b1, wv, K);
            __syncthreads();
            return;
        }
        for (int c0 = 0; c0 < nbox; c0 += c.bcap) {
            if (tid == 0) L.cnt[R_NBT] = 0;
            __syncthreads();
            for (int u = c0 + 64 * wv; u < min(nbox, c0 + c.bcap); u += B)
                rc_boxes(s, sc, cam, ego, L, s2, u, min(64, c0 + c.bcap - u));
            __syncthreads();
            rc_band(L, cam, L.cnt[R_NBT], b0, b1, wv, K);
            __syncthreads();
        }
        for (int c0 = 0; c0 < sc.n_signals; c0 += 64) {
            if (tid == 0) L.cnt[R_NBT] = 0;
            __syncthreads();
            if (wv == 0) rc_lights(s, sc, cam, L, c0);
            __syncthreads();
            rc_band(L, cam, L.cnt[R_NBT], b0, b1, wv, K);
            __syncthreads();
        }
    };
    auto clear = [&](int npix) {
        for (int p = tid; p < npix; p += B) L.work[p] = 0ull;
    };
    if (COV) {
        roads(chunked ? 0 : nbu + nlu, L.hr0, H);
        uint8_t *img = o.rgb + 3 * ((int64_t)view * W * H);
        int kr0 = H, kr1 = H;
        if (chunked) {
            kr0 = 0;
        } else if (L.cnt[R_NBT] > 0) {
            kr0 = L.cnt[R_BMIN];
            kr1 = L.cnt[R_BMAX] + 1;
        }
        const uint32_t bg_rgb = s.bg_rgb;
        const uint32_t road_rgb = s.shade ? shade_rgb(s.road_rgb, shade_level(s, 0.0f, 0.0f, 4)) : s.road_rgb;
        build_patterns(L, road_rgb, bg_rgb);
        clear((min(kr0 + L.krows, kr1) - kr0) * W);
        __syncthreads();
        write_rows(L, img, road_rgb, bg_rgb, W, 0, kr0);
        write_rows(L, img, road_rgb, bg_rgb, W, kr1, H);
        for (int b0 = kr0; b0 < kr1; b0 += L.krows) {
            const int b1 = min(b0 + L.krows, kr1);
            if (b0 != kr0) {
                __syncthreads();
                clear((b1 - b0) * W);
                __syncthreads();
            }
            boxes(b0, b1);
            resolve_band(
                L, W,
                [&](int j) {
                    const RcRow r = rc_row(cam, j);
                    return r.ok ? 1.0f / r.z : 0.0f;
                },
                [&](uint32_t keylo) { return rc_color(s, sc, L, chunked, keylo); }, L.work, img, road_rgb, bg_rgb, b0, b1);
        }
        return;
    }
    const int64_t view_px = (int64_t)view * H * W;
    auto rz = [&](int j) {
        const RcRow r = rc_row(cam, j);
        return r.ok ? 1.0f / r.z : 0.0f;
    };
    auto color = [&](uint32_t keylo) { return rc_color(s, sc, L, chunked, keylo); };
    const lptr<const uint32_t> cpal = (lptr<const uint32_t>)pal, croad = (lptr<const uint32_t>)road;
    const lptr<const unsigned long long> none = (lptr<const unsigned long long>)nullptr;
    int kr0 = H, kr1 = H;                        // rows that boxes and lights reach
    // bands of the rows below the horizon; the rows above go with the first
    for (int b0 = L.hr0;; b0 += c.band_rows) {
        const bool first = b0 == L.hr0;
        const int b1 = min(b0 + c.band_rows, H);
        if (!first) __syncthreads();             // the last band's keys are read
        for (int p = tid; p < (b1 - b0) * W; p += B) road[p] = 0u;
        if (!first && tid == 0) L.cnt[R_RING] = L.cnt[R_JOB] = 0;
        __syncthreads();
        roads(first && !chunked ? nbu + nlu : 0, b0, b1);
        if (first) {
            if (chunked) {
                kr0 = 0;
            } else if (L.cnt[R_NBT] > 0) {
                kr0 = L.cnt[R_BMIN];
                kr1 = L.cnt[R_BMAX] + 1;
            }
        }
        const int r0 = first ? 0 : b0;
        const int k0 = min(max(kr0, r0), b1), k1 = min(max(kr1, k0), b1);      // this band's box rows
        resolve_rows(s, cpal, rz, color, W, L.hr0, croad, b0, none, o, view_px, r0, k0);
        resolve_rows(s, cpal, rz, color, W, L.hr0, croad, b0, none, o, view_px, k1, b1);
        for (int c0 = k0; c0 < k1; c0 += L.krows) {
            const int c1 = min(c0 + L.krows, k1);
            __syncthreads();
            clear((c1 - c0) * W);
            __syncthreads();
            boxes(c0, c1);
            resolve_rows(s, cpal, rz, color, W, L.hr0, croad, b0, (lptr<const unsigned long long>)L.work, o, view_px, c0, c1);
        }
        if (b1 >= H) break;
    }
}

}  // namespace

size_t raycast_lds_bytes(int width, int height, const RcCfg &c) { return rc_layout(width, height, c).total; }

hipError_t launch_raycast(const DevSim &s, const RenderOut &o, const RcCfg &c, int view_begin, int n_views, hipStream_t st)
{
    if (n_views <= 0) return hipSuccess;
    if (c.waves < 1 || c.waves > 16 || c.band_rows < 1 || c.bcap < 64 || c.bcap % 64 != 0 || (c.cover && s.width < 16))
        return hipErrorInvalidValue;
    const size_t lds = raycast_lds_bytes(s.width, s.height, c);
    const dim3 block(64 * c.waves);
    const auto kernel = c.cover ? (c.seg ? k_raycast<true, true> : k_raycast<true, false>)
                                : (c.seg ? k_raycast<false, true> : k_raycast<false, false>);
    hipLaunchKernelGGL(kernel, dim3(n_views), block, lds, st, s, o, c, view_begin);
    return hipGetLastError();
}

}  // namespace gp
