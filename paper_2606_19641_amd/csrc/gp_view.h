// Device code of the renderers that split one view's work over the wavefronts
// of a workgroup through LDS work counters (the rgb raster, the general raster
// and the ray caster): LDS layout, culling of bins and strips, set-up of road
// primitives and box lists, and the writing of rows.
#pragma once

#include "gp_device.h"
#include "gp_geom.h"

namespace gp {

namespace {

constexpr int kSharedRing = 768;   // strips passed by the cheap test, one ring per view (road slot indices)
constexpr int kBatch = 64;      // road primitives (quads, triangles) a wavefront stages for one span pass, strips
                                // of one set-up job at most (one quad each; the rest are queued), and entries
                                // of its queue: strips waiting for the clipper (from the front) or for their fan
                                // triangles (from the back)
constexpr int kSmallBatch = 32, kSmallRing = 256;    // the same, and the ring, in a crowded view
__host__ __device__ constexpr int wave_bytes(int batch) { return batch * (48 + 4); }
constexpr int kWaveBytes = wave_bytes(kBatch);
static_assert(kWaveBytes % 16 == 0 && wave_bytes(kSmallBatch) % 16 == 0, "wave regions stay 16-byte aligned");
static_assert(sizeof(Prim) == 48, "staged primitive size");

// LDS counters
enum { R_NSB = 0, R_NBT, R_BOVF, R_BMIN, R_BMAX, R_RING, R_JOB, R_NSV, R_AT, R_NCNT = 12 };
constexpr int kBoxClip = 64;     // box faces waiting for the clipper (one setup pass)
constexpr int kBoxRecs = 64;     // boxes of one view kept in LDS after their culling, at most

// A box that may be seen by the view: what its faces are built from.  (Box
// units that culled 16 boxes each and read the survivors' state again took 7,000
// cycles apiece, 40% of the set-up of scenes with 128 agents.)
struct BoxRec {
    float x, y, c, s;            // centre, cosine and sine of the heading
    float dx, dy, dz;            // size
    int32_t j;                   // box of the scene
};
static_assert(sizeof(BoxRec) == 32, "BoxRec layout");

struct RgbLds {
    lptr<int32_t> cnt;               // [R_NCNT]
    lptr<unsigned long long> bits;   // road coverage: bit (j - hr0) * W + i is sample i of row j >= hr0
    lptr<FaceRec> faces;             // [bcap] the view's box faces
    lptr<int32_t> sbins;             // [bins_cap] surviving bins: start * 128 + count
    lptr<BoxRec> recs;               // [nrec] the boxes that survived their culling
    lptr<int32_t> cq;                // [kBoxClip] box faces to clip (record * 8 + face)
    lptr<int32_t> sring;             // [ring] strips that passed the cheap test (this round)
    lptr<unsigned char> waves;       // K regions of wave_bytes(batch)
    // after the units the memory behind the listed faces is free again: the pattern table, then masks and
    // spans or keys
    lptr<gp_v4i> pat;                // [3][64] the 16 bytes at byte phase p of a run of six pixels, by its coverage bits
    lptr<unsigned long long> work;   // masks and spans, or rows of 64-bit keys
    int bcap, krows;
    int batch, ring;                 // primitives a wavefront stages, strips the ring holds
    int bins;                        // surviving bins the list holds
    int nrec;                        // boxes the records hold
    int hr0;                         // first image row below the horizon
    int nmw;                         // 64-bit words of a face mask
    int region;                      // bytes from work to the end
    int tail;                        // bytes from faces to the end
};

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// byte offsets of the LDS sections (shared by the carve and the size query)
struct RgbLayout {
    size_t cnt, bits, recs, sbins, faces, sring, waves, total;
};

constexpr int kPatBytes = 3 * 64 * 16;

// the resolve's memory behind the listed faces: the pattern table, and a row of
// keys or a row of masks and spans of up to 256 faces
__host__ __device__ inline int resolve_bytes(int W) { return kPatBytes + 8 * W + 1280; }

// rows that can show road: below the principal point (the road's 1/z there is
// positive only where (j + 0.5) - H / 2 is)
__host__ __device__ inline int first_road_row(int H) { return (H + 1) >> 1; }

__host__ __device__ inline RgbLayout rgb_layout(int W, int H, const RgbCfg &c)
{
    RgbLayout l;
    // whole words of the flat coverage bits, and one more for reads across a word end
    const size_t nbw = ((size_t)W * (size_t)(H - first_road_row(H)) + 63) / 64 + 1;
    size_t o = 0;
    l.cnt = o; o = align16(o + 4 * R_NCNT);
    l.bits = o; o = align16(o + 8 * nbw);
    l.recs = o; o = align16(o + sizeof(BoxRec) * (size_t)c.recs);
    l.sbins = o; o = align16(o + 4 * (size_t)c.bins_cap);
    l.faces = o; o = align16(o + sizeof(FaceRec) * (size_t)c.bcap);
    const size_t least = align16(o + (size_t)resolve_bytes(W));
    l.sring = o; o = align16(o + 4 * (size_t)kSharedRing);
    l.waves = o; o = align16(o + (size_t)kWaveBytes * (size_t)c.waves);
    o = o > least ? o : least;
    l.total = o;
    return l;
}

// ------------------------------------------------------------ per-wave state

struct WaveSt {
    lptr<Prim> tris;         // [batch] road primitives
    lptr<int32_t> clipq;     // [batch] road slots (global): nclip for the clipper at the front,
                             // nfan for their two fan triangles at the back
    int nclip, nfan;         // queued strips
    int batch;
};

__device__ __forceinline__ WaveSt wave_state(const RgbLds &L, int wv)
{
    lptr<unsigned char> base = L.waves + (size_t)wv * wave_bytes(L.batch);
    WaveSt ws;
    ws.tris = (lptr<Prim>)base;
    ws.clipq = (lptr<int32_t>)(base + L.batch * 48);
    ws.nclip = 0;
    ws.nfan = 0;
    ws.batch = L.batch;
    return ws;
}

// A view that may list more faces (three a box) than its list holds gives it
// memory of its ring, as much as it needs down to kSmallRing, and of the staging.
// STAGING: of the staging first, in the general raster, whose bands set up their
// strips in small jobs anyway (depth and ids of crowds of 50 boxes, ring / staging
// first, us: four wavefronts 205 / 184, eight 138 / 137 and at 352 x 352 1,230 /
// 1,200, sixteen 99 / 92).  The rgb raster's rounds are larger: ring first (two to
// four wavefronts 234 / 234, 96 / 96, a batch of eight rollouts 86.5 / 87, eight 72.5
// / 73, at 352 x 352 364 / 373).  Before the first wave_state.
template <bool STAGING>
__device__ __forceinline__ void grow_list(RgbLds &L, int most, int K, int W)
{
    int lack = (min(most, 256) - L.bcap) * (int)sizeof(FaceRec);
    if (STAGING) {
        L.batch = kSmallBatch;
        lack -= K * (wave_bytes(kBatch) - wave_bytes(kSmallBatch));
    }
    if (lack > 0) {
        L.ring = max(kSmallRing, kSharedRing - 64 * ((lack + 255) >> 8));
        lack -= 4 * (kSharedRing - L.ring);
    }
    if (lack > 0) L.batch = kSmallBatch;
    const int tail = 4 * L.ring + K * wave_bytes(L.batch);
    L.bcap = max(L.bcap, min(256, (L.tail - max(tail, resolve_bytes(W))) / (int)sizeof(FaceRec)));
    L.sring = (lptr<int32_t>)((lptr<unsigned char>)L.faces + L.tail - tail);
    L.waves = (lptr<unsigned char>)(L.sring + L.ring);
}

// The memory behind the list's n faces for the resolve (the ring and the
// wavefronts' staging are idle by then); after the pattern table's use its
// place holds the streaming pass's clip queue.
__device__ __forceinline__ void free_region(RgbLds &L, int n, int W)
{
    lptr<unsigned char> p = (lptr<unsigned char>)(L.faces + n);
    L.pat = (lptr<gp_v4i>)p;
    L.cq = (lptr<int32_t>)p;
    L.work = (lptr<unsigned long long>)(p + kPatBytes);
    L.region = L.tail - n * (int)sizeof(FaceRec) - kPatBytes;
    L.krows = max(1, L.region / (8 * W));
    L.nmw = max(1, (n + 63) >> 6);
}

// OR the coverage bits [b0, b1] into their words
__device__ __forceinline__ void or_span(lptr<unsigned long long> bits, int b0, int b1)
{
    const int w0 = b0 >> 6, w1 = b1 >> 6;
    for (int w = w0; w <= w1; ++w) {
        const int lo = (w == w0) ? (b0 & 63) : 0;
        const int hi = (w == w1) ? (b1 & 63) : 63;
        const unsigned long long m = (~0ull >> (63 - hi)) & (~0ull << lo);
        lds_or64(bits + w, m);
    }
}

// the coverage bits from b on (at least 32 of them), bit 0 first
__device__ __forceinline__ uint32_t bits_at(const RgbLds &L, int b)
{
    lptr<const uint32_t> w = (lptr<const uint32_t>)L.bits + (b >> 5);
    return __builtin_amdgcn_alignbit(w[1], w[0], b & 31);
}

// Rasterise the n (<= 64) staged road primitives into the coverage bitmask.
// Their (primitive, row) items are dealt to the lanes by a prefix over row
// counts; per item the exact span of covered samples is OR-ed into the coverage
// words.  Every primitive has a row, so the first items of the primitives that
// start within a pass of 64 items are distinct: a bit for each, OR-ed over the
// wavefront, tells a lane its item's primitive by counting (owner_of's search
// takes about fifteen instructions and seven cross-lane reads more).
__device__ __forceinline__ void road_spans(const RgbLds &L, const Cam &cam, const WaveSt &ws, int n)
{
    const int ln = (int)lane_id();
    wave_lds_order();
    int c = 0;
    if (ln < n) {
        const int32_t jj = ((lptr<const int32_t>)(ws.tris + ln))[8];     // j0 | j1 << 16
        c = (jj >> 16) - (int)(int16_t)(jj & 0xFFFF) + 1;
    }
    const int incl = wave_incl_scan(c);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int excl = incl - c;
    for (int g0 = 0; g0 < total; g0 += 64) {
        const int gi = g0 + ln, at = excl - g0;
        const bool starts = (ln < n) & ((uint32_t)at < 64u);
        const unsigned long long m = wave_or64(starts ? 1ull << (at & 63) : 0ull);
        const int before = __popcll(__ballot((ln < n) & (at < 0)));
        const int o = before + lanes_below(m) + (int)((m >> ln) & 1ull) - 1;
        const int ex = __shfl(excl, o);
        if (gi < total) {
            const Prim pr = lds_load(ws.tris + o);
            const int j = pr.j0 + (gi - ex);
            int xl, xr;
            // (the row test holds for every row with road unless 1/z underflows)
            const float rz = fmaf(cam.road.B, ((float)j + 0.5f) - cam.cy, cam.road.C);
            const int b = (j - L.hr0) * cam.W;
            if ((b >= 0) & (rz > 0.0f) & prim_span(pr, j, cam.W, xl, xr)) or_span(L.bits, b + xl, b + xr);
        }
    }
    wave_lds_order();
}

// Fragments of the n staged road primitives in rows [b0, b1) folded into the
// band of road keys (first row band0): (primitive, row) items dealt to the lanes,
// their exact spans cut into pieces of up to 16 samples, dealt again.  Every
// strip lies in one plane, so 1/z is the row's and the strip that a sample shows
// is the one with the largest key word: the band holds key words only.
__device__ __forceinline__ void road_fold(const RgbLds &L, lptr<uint32_t> road, const Cam &cam, const WaveSt &ws, int n, int b0,
                                          int b1, int band0)
{
    const int ln = (int)lane_id(), W = cam.W;
    wave_lds_order();
    int c = 0, first = 0;
    if (ln < n) {
        const int32_t jj = ((lptr<const int32_t>)(ws.tris + ln))[8];     // j0 | j1 << 16
        first = max((int)(int16_t)(jj & 0xFFFF), b0);
        c = max(0, min(jj >> 16, b1 - 1) - first + 1);
    }
    const int incl = wave_incl_scan(c);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int excl = incl - c;
    for (int g0 = 0; g0 < total; g0 += 64) {
        const int gi = g0 + ln;
        const int o = owner_of(incl, gi);
        const int j = __shfl(first, o) + (gi - __shfl(excl, o));
        int xl = 0, xr = -1, key = 0;
        if (gi < total) {
            const Prim pr = lds_load(ws.tris + o);
            key = pr.pad0;
            const float rz = fmaf(cam.road.B, ((float)j + 0.5f) - cam.cy, cam.road.C);
            if (!((rz > 0.0f) & prim_span(pr, j, W, xl, xr))) { xl = 0; xr = -1; }
        }
        const int np = (xr - xl + 16) >> 4;
        const int inc2 = wave_incl_scan(np);
        const int npt = __builtin_amdgcn_readlane(inc2, 63);
        const int ex2 = inc2 - np;
        const int x2 = xl | (xr << 16);
        for (int p0 = 0; p0 < npt; p0 += 64) {
            const int pi = p0 + ln;
            const int o2 = owner_of(inc2, pi);
            const int k = pi - __shfl(ex2, o2);
            const int sx = __shfl(x2, o2), sj = __shfl(j, o2), sk = __shfl(key, o2);
            if (pi >= npt) continue;
            const int i0 = (sx & 0xFFFF) + 16 * k, i1 = min(i0 + 15, sx >> 16);
            lptr<uint32_t> row = road + (sj - band0) * W;
            for (int i = i0; i <= i1; ++i) lds_max32(row + i, (uint32_t)sk);
        }
    }
    wave_lds_order();
}

// the key word of the strip in road slot g (global)
__device__ __forceinline__ int road_key(const DevSim &s, const SceneRec &sc, int g)
{
    return (int)key_low(0u, 6 * (sc.n_agents + sc.n_static) + s.road_index[g], s.road_color[g]);
}

// Stage the triangles held by the lanes (v) behind the n staged ones; returns
// how many are staged then.
__device__ __forceinline__ int stage_tris(const WaveSt &ws, int n, bool v, const Prim &t)
{
    const unsigned long long b = __ballot(v);
    if (v) lds_store(ws.tris + n + lanes_below(b), t);
    return n + __popcll(b);
}

// Clip up to four queued strips (the last ones of the queue), one per 16-lane
// segment; stages their fan triangles behind the n staged primitives and
// returns how many are staged then, or -1 (the strips stay queued) where they
// do not fit.  They always fit an empty stage.
template <bool KEY>
__device__ __forceinline__ int road_clip(const DevSim &s, const SceneRec &sc, const Cam &cam, WaveSt &ws, int n)
{
    const int m = min(ws.nclip, min(4, ws.batch / kMaxTrisPerCand));
    const int seg = (int)lane_id() >> 4;
    const bool live = seg < m;
    Poly P = {};
    int key = 0;
    if (live) {
        const int g = ws.clipq[ws.nclip - m + seg];
        road_corners(s, cam, g, P.v);
        if (KEY) key = road_key(s, sc, g);
    }
    P.n = dir_to_cam(cam, 0.0f, 0.0f, 1.0f);
    P.one_sided = false;
    P.keylo = 0u;
    TriRec t;
    const bool ok = clip_seg<false>(cam, P, live, 0, cam.H, t);
    if (n + __popcll(__ballot(ok)) > ws.batch) return -1;
    ws.nclip -= m;
    Prim p = prim_of(t.g);
    p.pad0 = key;
    return stage_tris(ws, n, ok, p);
}

// The two fan triangles of up to batch / 2 queued strips (the last ones queued
// at the back of the queue); stages them behind the n staged primitives and
// returns how many are staged then.  Their corners
// and snap are computed again, as the set-up computed them.
template <bool KEY>
__device__ __forceinline__ int road_fan(const DevSim &s, const SceneRec &sc, const Cam &cam, WaveSt &ws, int n)
{
    const int m = min(ws.nfan, ws.batch / 2);
    const int ln = (int)lane_id();
    Prim p0 = {}, p1 = {};
    bool v0 = false, v1 = false;
    if (ln < m) {
        const int g = ws.clipq[ws.batch - ws.nfan + ln];
        V3 v[4];
        road_corners(s, cam, g, v);
        int32_t X[4], Y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) snap(cam, v[k], X[k], Y[k]);
        TriGeo t0, t1;
        v0 = make_tri(cam, false, X[0], Y[0], X[1], Y[1], X[2], Y[2], 0, cam.H, t0);
        v1 = make_tri(cam, false, X[0], Y[0], X[2], Y[2], X[3], Y[3], 0, cam.H, t1);
        if (v0) p0 = prim_of(t0);
        if (v1) p1 = prim_of(t1);
        if (KEY) p0.pad0 = p1.pad0 = road_key(s, sc, g);
    }
    ws.nfan -= m;
    n = stage_tris(ws, n, v0, p0);
    return stage_tris(ws, n, v1, p1);
}

// Full setup of the n (<= batch) strips ring[a .. a + n): clip test,
// snap, and the quad of the strips whose quad covers exactly what their two
// fan triangles cover (staged; returns how many); strips that need the
// clipper join the front of the wave's queue, strips that need their fan
// triangles its back (both empty when a job starts).
template <bool KEY>
__device__ __forceinline__ int road_setup(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, WaveSt &ws,
                                          int a, int n)
{
    const int ln = (int)lane_id();
    wave_lds_order();
    const bool live = ln < n;
    int g = 0;
    V3 v[4] = {};
    if (live) {
        g = L.sring[a + ln];
        road_corners(s, cam, g, v);
    }
    const bool clip = live && needs_clip(cam, v);
    const unsigned long long cb = __ballot(clip);
    if (clip) ws.clipq[ws.nclip + lanes_below(cb)] = g;
    ws.nclip += __popcll(cb);
    Prim p0 = {};
    bool v0 = false, fan = false;
    if (live && !clip) {
        int32_t X[4], Y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) snap(cam, v[k], X[k], Y[k]);
        // one quad where it covers exactly what the two fan triangles cover
        const int qs = make_quad(cam, false, X, Y, 0, cam.H, p0);
        v0 = qs > 0;
        fan = qs < 0;
        if (KEY) p0.pad0 = road_key(s, sc, g);
    }
    const unsigned long long fb = __ballot(fan);
    if (fan) ws.clipq[ws.batch - 1 - (ws.nfan + lanes_below(fb))] = g;
    ws.nfan += __popcll(fb);
    return stage_tris(ws, 0, v0, p0);
}

// One set-up job: the n ring strips from a set up and their primitives
// rasterised (spans(n): the n staged ones): the quads, with the triangles of
// the strips that need the clipper (four at a time) and of those that need
// their fan triangles where they fit behind them, else in passes of their own
// (four strips cut by one plane have sixteen triangles at most).  KEY: a staged primitive carries its
// strip's key word in pad0.
template <bool KEY, class Spans>
__device__ __forceinline__ void setup_job(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, WaveSt &ws,
                                          int a, int n, Spans spans)
{
    int staged = road_setup<KEY>(s, sc, cam, L, ws, a, n);
    for (;;) {
        while (ws.nclip > 0 && (staged == 0 || staged + 16 <= ws.batch)) {
            const int t = road_clip<KEY>(s, sc, cam, ws, staged);
            if (t < 0) break;
            staged = t;
        }
        if (ws.nfan > 0 && staged + 2 * min(ws.nfan, ws.batch / 2) <= ws.batch) staged = road_fan<KEY>(s, sc, cam, ws, staged);
        if (staged > 0) spans(staged);
        else if (ws.nclip + ws.nfan == 0) break;
        staged = 0;
    }
}

// The survivors of one unit's strips (pass; slot g) appended to the view's
// ring (a round has no more units than the ring takes 64 strips of).
__device__ __forceinline__ void ring_append(const RgbLds &L, bool pass, int g)
{
    const unsigned long long bm = __ballot(pass);
    if (bm == 0ull) return;
    int base = 0;
    if (lane_id() == 0) base = lds_add(L.cnt + R_RING, __popcll(bm));
    base = __builtin_amdgcn_readlane(base, 0);
    if (pass) L.sring[base + lanes_below(bm)] = g;
}

// strip data of unit u (lane l: strip l % 16 of surviving bin 4 u + l / 16)
__device__ __forceinline__ bool load_unit(const DevSim &s, const SceneRec &sc, const RgbLds &L, int nsb, int u,
                                          int &g, float4 &q0, float4 &q1)
{
    const int ln = (int)lane_id();
    const int bi = 4 * u + (ln >> 4), k = ln & 15;
    bool live = false;
    if (u >= 0 && bi < nsb) {
        const int pk = L.sbins[bi];
        live = k < (pk & 127);
        if (live) {
            g = sc.road_base + (pk >> 7) + k;
            q0 = s.roads[2 * g];
            q1 = s.roads[2 * g + 1];
        }
    }
    return live;
}

// The road work of a view (and, as its first jobs, the box and light units),
// shared by the wavefronts in rounds of two steps.  B1: the road units (four
// surviving bins each), as many as the ring has 64 entries for, in turn:
// test(live, q0, q1) is the cheap test of the unit's strips, whose survivors
// join the view's ring.  B2: the jobs, dealt through an LDS counter -- in the
// first round box(u) for u < box_jobs (their lists are needed only by the
// resolve, so a long box unit overlaps the other wavefronts' road jobs), then
// road(a, n) for up to batch ring strips at a time.  R_RING and R_JOB are zero
// at the start (published by a barrier); ends with a barrier.
// (The units were dealt through LDS counters too, with ring entries reserved:
// four dependent LDS operations before a unit's loads, and units cost the same.)
template <class Test, class Box, class Road>
__device__ __forceinline__ void road_work(const DevSim &s, const SceneRec &sc, const RgbLds &L, int nsb, int box_jobs,
                                          Test test, Box box, Road road)
{
    const int ln = (int)lane_id(), K = (int)blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n_units = (nsb + 3) / 4, per = L.ring / 64;
    for (int u0 = 0;; u0 += per) {
        // B1, the next unit's strips loaded while the current one is tested
        const int u1 = min(u0 + per, n_units);
        float4 q0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), q1 = q0;
        int gq = 0;
        bool live = u0 + wv < u1 && load_unit(s, sc, L, nsb, u0 + wv, gq, q0, q1);
        for (int u = u0 + wv; u < u1; u += K) {
            float4 n0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), n1 = n0;
            int gn = 0;
            const bool nlive = u + K < u1 && load_unit(s, sc, L, nsb, u + K, gn, n0, n1);
            ring_append(L, test(live, q0, q1), gq);
            q0 = n0;
            q1 = n1;
            gq = gn;
            live = nlive;
        }
        __syncthreads();
        const int nring = L.cnt[R_RING];
        const bool more = u1 < n_units;
        // the ring cut into jobs of at most batch strips, as many as a
        // multiple of the wavefronts, of equal size: a job's set-up takes about
        // the same time for any number of strips up to a wavefront's width.
        const int njobs = (max(K, (nring + L.batch - 1) / L.batch) + K - 1) / K * K;
        const int jsz = (nring + njobs - 1) / njobs;
        // B2
        for (;;) {
            int j = 0;
            if (ln == 0) j = lds_add(L.cnt + R_JOB, 1);
            j = __builtin_amdgcn_readlane(j, 0) - box_jobs;
            if (j < 0) {
                box(j + box_jobs);
                continue;
            }
            const int a = j * jsz;
            if (a >= nring) break;
            road(a, min(jsz, nring - a));
        }
        __syncthreads();
        box_jobs = 0;
        if (!more) return;
        if (threadIdx.x == 0) L.cnt[R_RING] = L.cnt[R_JOB] = 0;
        __syncthreads();
    }
}

// ------------------------------------------------------------ boxes

// Reserve n entries of the box list: at the wave's own count nbt (shared
// false: the overflow path's private list), or through the view's LDS
// counter (shared: several wavefronts append); returns the first entry, or
// -1 (marking the view overflowed when shared) if they would not fit.
__device__ __forceinline__ int box_reserve(const RgbLds &L, bool shared, int &nbt, int n)
{
    if (!shared) {
        if (nbt + n > L.bcap) return -1;
        const int at = nbt;
        nbt += n;
        return at;
    }
    int at = 0;
    if (lane_id() == 0 && n > 0) at = lds_add(L.cnt + R_NBT, n);
    at = __builtin_amdgcn_readlane(at, 0);
    if (at + n > L.bcap) {
        if (lane_id() == 0) L.cnt[R_BOVF] = 1;
        return -1;
    }
    return at;
}

// the colour of face f of a box, lit where the sim has a light
template <bool AP>
__device__ __forceinline__ uint32_t rec_rgb(const DevSim &s, const SceneRec &sc, const BoxRec &b, int f)
{
    const uint32_t c = s.box_rgb[box_slot(sc, b.j)];
    return AP && s.shade ? lit_heading(s, c, make_float2(b.c, b.s), f) : c;
}

// the colour of traffic light g's state (never lit)
__device__ __forceinline__ uint32_t signal_rgb(const DevSim &s, const SceneRec &sc, int g)
{
    const int c = s.signal_color[sc.signal_base + g];
    return (uint32_t)s.palette[3 * c] | ((uint32_t)s.palette[3 * c + 1] << 8) | ((uint32_t)s.palette[3 * c + 2] << 16);
}

// Traffic lights [g0, g0 + 64) of the scene into the view's list: an entry
// holds the sphere test's terms (centre, squared radius, f zc) and the pixel
// rectangle its image lies in (columns X3 .. Y3); nv = 0 tells it from a face.
__device__ __forceinline__ bool light_pass(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, int g0,
                                           bool shared, int &nbt, int &bmin, int &bmax)
{
    const int g = g0 + (int)lane_id();
    bool keep = false;
    FaceRec f = {};
    if (g < sc.n_signals) {
        const float4 q = s.signals[sc.signal_base + g];
        const V3 c = to_cam(cam, q.x - cam.px, q.y - cam.py, q.z);
        int i0, i1, j0, j1;
        keep = signal_bounds(cam, c, q.w, i0, i1, j0, j1);
        if (keep) {
            f.X0 = __float_as_int(c.x); f.Y0 = __float_as_int(c.y); f.X1 = __float_as_int(c.z);
            f.Y1 = __float_as_int(q.w * q.w); f.X2 = __float_as_int(cam.f * c.z);
            f.X3 = i0; f.Y3 = i1;
            f.j0 = (int16_t)j0; f.j1 = (int16_t)j1;
            f.keylo = key_low(1u, 6 * (sc.n_agents + sc.n_static) + sc.n_roads + g, 0u);
            f.rgb = signal_rgb(s, sc, g);
        }
    }
    const unsigned long long bm = __ballot(keep);
    const int at = box_reserve(L, shared, nbt, __popcll(bm));
    if (at < 0) return false;
    if (keep) {
        const int t = at + lanes_below(bm);
        f.keylo |= (uint32_t)t;
        lds_store(L.faces + t, f);
        bmin = min(bmin, (int)f.j0);
        bmax = max(bmax, (int)f.j1);
    }
    return true;
}

// face f of the box in a record; the key word without its low byte
__device__ __forceinline__ void rec_face(const Cam &cam, const BoxRec &b, int f, Poly &P)
{
    face_corners(cam, b.x, b.y, b.c, b.s, b.dx, b.dy, b.dz, f, P);
    P.keylo = key_low(1u, 6 * b.j + f, 0u);
}

// One setup pass over the faces of box records [r0, r0 + n) (n <= 10): fast
// faces and the triangles of clipped faces (clip queue cq) that have a sample row
// in [y0, y1) are appended to the box list (box_reserve), the low byte of each key
// word naming the entry; returns false as soon as they would not fit (the list is
// then incomplete).
// One record never overflows a private list of 64 (its six faces have at most
// 10 triangles each).
template <bool AP>
__device__ __forceinline__ bool box_pass(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, int r0, int n,
                                         int y0, int y1, lptr<int32_t> cq, bool shared, int &nbt, int &bmin, int &bmax)
{
    const int ln = (int)lane_id();
    const bool live = ln < 6 * n;
    const int r = r0 + ln / 6, f = ln % 6;
    Poly Pf;
    FaceRec f0, f1;
    bool v0 = false, v1 = false, clip = false;
    if (live) {
        const BoxRec b = lds_load(L.recs + r);
        rec_face(cam, b, f, Pf);
        fast_face(cam, Pf, rec_rgb<AP>(s, sc, b, f), y0, y1, f0, v0, f1, v1, clip);
    }
    const unsigned long long b0 = __ballot(v0), b1 = __ballot(v1), bc = __ballot(clip);
    const int n0 = __popcll(b0), nf = n0 + __popcll(b1), ncl = __popcll(bc);
    const int at = box_reserve(L, shared, nbt, nf);
    if (at < 0) return false;
    if (v0) {
        const int t = at + lanes_below(b0);
        f0.keylo = (f0.keylo & ~0xFFu) | (uint32_t)t;
        lds_store(L.faces + t, f0);
        bmin = min(bmin, (int)f0.j0);
        bmax = max(bmax, (int)f0.j1);
    }
    if (v1) {
        const int t = at + n0 + lanes_below(b1);
        f1.keylo = (f1.keylo & ~0xFFu) | (uint32_t)t;
        lds_store(L.faces + t, f1);
        bmin = min(bmin, (int)f1.j0);
        bmax = max(bmax, (int)f1.j1);
    }
    if (clip) cq[lanes_below(bc)] = r * 8 + f;
    wave_lds_order();
    // the clipped faces, four per wavefront
    for (int q0 = 0; q0 < ncl; q0 += 4) {
        const int q = q0 + (ln >> 4);
        const bool lv = q < ncl;
        Poly Q = {};
        uint32_t rgb = 0u;
        if (lv) {
            const int code = cq[q];
            const BoxRec b = lds_load(L.recs + (code >> 3));
            rec_face(cam, b, code & 7, Q);
            rgb = rec_rgb<AP>(s, sc, b, code & 7);
        }
        TriRec t;
        const bool ok = clip_seg<true>(cam, Q, lv, y0, y1, t);
        const unsigned long long bo = __ballot(ok);
        const int ato = box_reserve(L, shared, nbt, __popcll(bo));
        if (ato < 0) return false;
        if (ok) {
            const int e = ato + lanes_below(bo);
            t.keylo = (t.keylo & ~0xFFu) | (uint32_t)e;
            lds_store(L.faces + e, face_of(t, rgb));
            bmin = min(bmin, (int)t.g.j0);
            bmax = max(bmax, (int)t.g.j1);
        }
    }
    return true;
}

// the rows bmin .. bmax that the lanes' entries reach added to the view's box rows
__device__ __forceinline__ void box_rows(const RgbLds &L, int bmin, int bmax)
{
    bmin = wave_min(bmin);
    bmax = wave_max(bmax);
    if (lane_id() == 0 && bmax >= 0) {
        lds_min(L.cnt + R_BMIN, bmin);
        lds_max(L.cnt + R_BMAX, bmax);
    }
}

// Light unit k: traffic lights [64 k, 64 (k + 1)) of the scene.
__device__ __forceinline__ void do_lights(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, int k)
{
    int nbt = 0, bmin = 0x7FFFFFFF, bmax = -1;
    if (light_pass(s, sc, cam, L, 64 * k, true, nbt, bmin, bmax)) box_rows(L, bmin, bmax);
}

// A lane's bin and box of a culling pass: bin b of the scene's [0, n_bins), box
// b of [0, nbox) but the ego.  The loads need no camera: the first pass's are
// under way while the camera is computed.
struct CullIn {
    RoadBin bn;
    float4 st, dm;
    float2 cs, act;
    int b;
    bool bin, box, moved;
};

template <bool STEP>
__device__ __forceinline__ CullIn cull_load(const DevSim &s, const SceneRec &sc, int ego, int b0, int n_bins, int nbox)
{
    CullIn c = {};
    c.b = b0 + (int)lane_id();
    c.bin = c.b < n_bins;
    c.box = c.b < nbox && c.b != ego;
    if (c.bin) c.bn = s.bins[sc.bin_base + c.b];
    if (c.box) {
        const int ga = box_slot(sc, c.b);
        c.dm = s.dims[ga];
        c.st = s.state[ga];
        c.cs = s.cs[ga];
        if (STEP && s.act && ga < s.n_agents) {
            c.act = s.act[ga];
            c.moved = s.halted[ga] == 0;
        }
    }
    return c;
}

// Bins (frustum, road depth limit and row-gap test) and boxes loaded from b0
// on, against the view: the survivors join the view's bin list and box records
// (R_NSB and R_NSV count them all, also those that the lists cannot hold).
template <bool STEP>
__device__ __forceinline__ void cull_pass(const DevSim &s, const Cam &cam, const RgbLds &L, const CullIn &c, int b0, int n_bins,
                                          int nbox)
{
    const RoadBin &bn = c.bn;
    const float4 dm = c.dm;
    float4 st = c.st;
    float2 cs = c.cs;
    const bool bin = c.bin, box = c.box;
    const int b = c.b;
    if (STEP && s.act && b0 < nbox) {
        float4 n;
        float2 t;
        (void)bicycle(s.dt, st, dm.x, c.act.x, c.act.y, n, t);
        st.x = c.moved ? n.x : st.x;
        st.y = c.moved ? n.y : st.y;
        cs.x = c.moved ? t.x : cs.x;
        cs.y = c.moved ? t.y : cs.y;
    }
    bool kbin = false, kbox = false;
    if (b0 < n_bins) {
        float x[4], z[4];
        ground_xz(cam, bn.xmin, bn.ymin, x[0], z[0]);
        ground_xz(cam, bn.xmax, bn.ymin, x[1], z[1]);
        ground_xz(cam, bn.xmax, bn.ymax, x[2], z[2]);
        ground_xz(cam, bn.xmin, bn.ymax, x[3], z[3]);
        kbin = bin & !road_culled<true>(cam, x, z, 0, cam.H);
    }
    if (b0 < nbox) kbox = box & !box_outside_at(cam, st, dm);
    // the counters of both lists are advanced together
    const unsigned long long mbin = __ballot(kbin), mbox = __ballot(kbox);
    int abin = 0, abox = 0;
    if (lane_id() == 0) {
        if (mbin != 0ull) abin = lds_add(L.cnt + R_NSB, __popcll(mbin));
        if (mbox != 0ull) abox = lds_add(L.cnt + R_NSV, __popcll(mbox));
    }
    abin = __builtin_amdgcn_readlane(abin, 0) + lanes_below(mbin);
    abox = __builtin_amdgcn_readlane(abox, 0) + lanes_below(mbox);
    if (kbin && abin < L.bins) L.sbins[abin] = bn.start * 128 + bn.count;
    if (kbox && abox < L.nrec) lds_store(L.recs + abox, BoxRec{st.x, st.y, cs.x, cs.y, dm.x, dm.y, dm.z, b});
}

// The culling of a whole scene, shared by the wavefronts; in holds the loads of
// this wavefront's first pass.
template <bool STEP>
__device__ __forceinline__ void cull_all(const DevSim &s, const SceneRec &sc, const Cam &cam, int ego, const RgbLds &L, CullIn &in,
                                         int wv, int B)
{
    const int nbox = sc.n_agents + sc.n_static, n = max(sc.n_bins, nbox);
    for (int b0 = 64 * wv; b0 < n; b0 += B) {
        // the next pass's loads are under way while this one is tested
        CullIn next = {};
        if (b0 + B < n) next = cull_load<STEP>(s, sc, ego, b0 + B, sc.n_bins, nbox);
        cull_pass<STEP>(s, cam, L, in, b0, sc.n_bins, nbox);
        in = next;
    }
}

// records a box unit sets up: ten fill a pass's lanes with their six faces;
// workgroups of many wavefronts take smaller units, so that clipped faces are
// spread over them
__device__ __forceinline__ int box_unit(int K) { return K >= 8 ? 4 : 10; }

// Box unit k: the faces of records [unit k, unit (k + 1)) into the view's box
// list (shared by the wavefronts; its row range kept with LDS min / max).
// scr: 64 ints of the wavefront's staging (the clip queue).
template <bool AP>
__device__ __forceinline__ void do_boxes(const DevSim &s, const SceneRec &sc, const Cam &cam, const RgbLds &L, int k, int unit,
                                         int n_recs, lptr<int32_t> scr)
{
    int nbt = 0, bmin = 0x7FFFFFFF, bmax = -1;
    if (box_pass<AP>(s, sc, cam, L, unit * k, min(unit, n_recs - unit * k), 0, cam.H, scr, true, nbt, bmin, bmax))
        box_rows(L, bmin, bmax);
}

typedef float f4v __attribute__((ext_vector_type(4)));

// the samples of row j that entry e may show: a face's exact span, or the
// columns of a light's rectangle
template <bool AP>
__device__ __forceinline__ bool entry_span(const Prim &e, int j, int W, int &xl, int &xr)
{
    if (AP && e.nv == 0) {
        xl = e.X3;
        xr = e.Y3;
        return true;
    }
    return prim_span(e, j, W, xl, xr);
}

// Box keys as doubles: a key's high word, the bits of a positive 1/z, is below
// 0x7ff00000, so keys order like the positive doubles of the same bits, and one
// v_max_f64 keeps the larger of two.  (fmax would quiet its operands first.)
__device__ __forceinline__ double key_max(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// 1/z of the light entry at t for the sample offsets a, b (0: not shown)
__device__ __forceinline__ float light_invz(const RgbLds &L, const Cam &cam, int t, float a, float b)
{
    const lptr<const f4v> e = (lptr<const f4v>)(L.faces + t);
    const f4v p = e[0];
    return signal_invz(cam, p.x, p.y, p.z, p.w, e[1].x, a, b);
}

// Fragments of the list's n entries in rows [b0, b1) folded into the key band
// by wavefronts wv of nwv (passes of many items shared out, of few their
// pieces).  The (entry, row) items are dealt to the lanes by a prefix
// over row counts; each lane computes its item's exact span; the spans are cut
// into pieces of up to 16 samples, which are dealt to the lanes by a prefix
// over piece counts, and each lane folds its piece's samples into the band
// with LDS atomic max.
template <bool AP>
__device__ __forceinline__ void box_band(const RgbLds &L, const Cam &cam, lptr<unsigned long long> keys, int n, int b0,
                                         int b1, int wv, int nwv)
{
    const int ln = (int)lane_id();
    const int W = cam.W;
    int pass = 0;
    for (int t0 = 0; t0 < n; t0 += 64) {
        const int t = t0 + ln;
        int c = 0;
        if (t < n) {
            const int32_t jj = ((lptr<const int32_t>)(L.faces + t))[12];
            const int j0 = max((int)(int16_t)(jj & 0xFFFF), b0), j1 = min(jj >> 16, b1 - 1);
            c = max(0, j1 - j0 + 1);
        }
        const int incl = wave_incl_scan(c);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int excl = incl - c;
        const bool split = total <= 128 * nwv;
        for (int g0 = 0; g0 < total; g0 += 64, ++pass) {
            if (!split && pass % nwv != wv) continue;
            const int gi = g0 + ln;
            const int o = owner_of(incl, gi);
            const int ex = __shfl(excl, o);
            int xl = 0, xr = -1, j = 0, light = 0;
            if (gi < total) {
                const Prim pr = lds_face_prim((lptr<const FaceRec>)(L.faces + t0 + o));
                j = max((int)pr.j0, b0) + (gi - ex);
                if (!entry_span<AP>(pr, j, W, xl, xr)) { xl = 0; xr = -1; }
                light = AP && pr.nv == 0;
            }
            const int te = (t0 + o) | (light << 16);
            const int np = (xr - xl + 16) >> 4;            // pieces of up to 16 samples (0 if empty)
            const int inc2 = wave_incl_scan(np);
            const int npt = __builtin_amdgcn_readlane(inc2, 63);
            const int ex2 = inc2 - np;
            for (int p0 = split ? 64 * wv : 0; p0 < npt; p0 += split ? 64 * nwv : 64) {
                const int pi = p0 + ln;
                const int o2 = owner_of(inc2, pi);
                const int k = pi - __shfl(ex2, o2);
                const int sxl = __shfl(xl, o2), sxr = __shfl(xr, o2), sj = __shfl(j, o2), st = __shfl(te, o2);
                if (pi >= npt) continue;
                const f4v pk = ((lptr<const f4v>)(L.faces + (st & 0xFFFF)))[2];      // A B C keylo
                const int i0 = sxl + 16 * k, i1 = min(i0 + 15, sxr);
                const float dv = ((float)sj + 0.5f) - cam.cy, bdv = fmaf(pk.y, dv, pk.z);
                lptr<unsigned long long> row = keys + (size_t)(sj - b0) * W;
                for (int i = i0; i <= i1; ++i) {
                    const float du = ((float)i + 0.5f) - cam.cx;
                    float invz = fmaf(pk.x, du, bdv);
                    if (AP && (st >> 16)) invz = light_invz(L, cam, st & 0xFFFF, du, -dv);
                    if (invz > 0.0f) lds_max64(row + i, ((unsigned long long)__float_as_uint(invz) << 32) | __float_as_uint(pk.w));
                }
            }
        }
    }
}

// ------------------------------------------------------------ box rows by group masks
//
// The box rows [c0, c1) without a key band: the exact span of every (box
// face, row) item is computed once and stored, and every group of 16 samples
// of a row gets a mask of the faces whose span meets it.  The resolve then
// walks, for its 16 samples, the faces of its group's mask and keeps the
// largest key of each sample in registers.  The G = ceil(W / 16) groups of a
// row start at samples 0, 16, ...; where W is not a multiple of 16 the last
// one starts at W - 16 and shares samples with the one before (both compute
// and store the same pixels).  Memory (L.work): the masks M[c1 - c0][G][nmw],
// then the spans S[t][c1 - c0].
__host__ __device__ inline int mask_rows_fit(int region, int n, int W, int nmw)
{
    // rows per chunk so that the masks and a span of every face in every row fit
    return region / (8 * nmw * ((W + 15) / 16) + 4 * n);
}

template <bool AP>
__device__ __forceinline__ void box_spans(const RgbLds &L, const Cam &cam, int n, int c0, int c1, int wv, int nwv)
{
    const int ln = (int)lane_id();
    const int R = c1 - c0, G = (cam.W + 15) >> 4, nmw = L.nmw;
    lptr<unsigned long long> M = L.work;
    lptr<int32_t> S = (lptr<int32_t>)(M + nmw * G * R);
    int pass = 0;
    for (int t0 = 0; t0 < n; t0 += 64) {
        const int t = t0 + ln;
        int c = 0;
        if (t < n) {
            const int32_t jj = ((lptr<const int32_t>)(L.faces + t))[12];
            const int j0c = max((int)(int16_t)(jj & 0xFFFF), c0);
            c = max(0, min(jj >> 16, c1 - 1) - j0c + 1);
        }
        const int incl = wave_incl_scan(c);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        const int excl = incl - c;
        for (int g0 = 0; g0 < total; g0 += 64, ++pass) {
            if (pass % nwv != wv) continue;
            const int gi = g0 + ln;
            const int o = owner_of(incl, gi);
            const int ex = __shfl(excl, o);
            if (gi < total) {
                const int tt = t0 + o;
                const Prim pr = lds_face_prim((lptr<const FaceRec>)(L.faces + tt));
                const int j = max((int)pr.j0, c0) + (gi - ex);
                int xl, xr;
                if (entry_span<AP>(pr, j, cam.W, xl, xr)) {
                    // bit 31 marks a light's columns and faces of no finite plane
                    S[tt * R + (j - c0)] = xl | (xr << 16) | (((AP && pr.nv == 0) || pr.pad1 != 0) ? (int)0x80000000 : 0);
                    lptr<unsigned long long> mrow = M + nmw * G * (j - c0) + (tt >> 6);
                    const unsigned long long bit = 1ull << (tt & 63);
                    const int gl = xr >= cam.W - 16 ? G - 1 : xr >> 4;
                    for (int g = xl >> 4; g <= gl; ++g) lds_or64(mrow + nmw * g, bit);
                }
            }
        }
    }
}

// rows [c0, c1) from the group masks and spans: 16 samples (48 bytes) per
// task; tasks alternate over the view's wavefronts in blocks of 32 lanes so
// that a few box rows still keep every wavefront busy
template <bool AP>
__device__ __forceinline__ void resolve_masks(const RgbLds &L, const Cam &cam, uint8_t *img, uint32_t road_rgb,
                                              uint32_t bg_rgb, int c0, int c1, int wv, int nwv)
{
    const int R = c1 - c0, G = (cam.W + 15) >> 4, nmw = L.nmw;
    lptr<const unsigned long long> M = (lptr<const unsigned long long>)L.work;
    lptr<const int32_t> S = (lptr<const int32_t>)(M + nmw * G * R);
    const int W = cam.W;
    const int n = R * G;
    const int ln = (int)lane_id();
    const int half = ln >> 5, sub = ln & 31;
    for (int blk = 2 * wv + half; 32 * blk < n; blk += 2 * nwv) {
        const int task = 32 * blk + sub;
        if (task >= n) continue;
        const int r = task / G, g = task - r * G, i = min(g << 4, W - 16), j = c0 + r;
        const float dv = ((float)j + 0.5f) - cam.cy;
        const float rz = fmaf(cam.road.B, dv, cam.road.C);
        const uint32_t bits = j >= L.hr0 ? bits_at(L, (j - L.hr0) * W + i) : 0u;
        const uint32_t rzb = __float_as_uint(rz);
        // sample offsets ((float)(i + m) + 0.5f) - cx are small exact values: du0 + m
        const float du0 = ((float)i + 0.5f) - cam.cx;
        double best[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) best[m] = 0.0;
        for (int w = 0; w < nmw; ++w) {
            unsigned long long mk = M[nmw * (G * r + g) + w];
            while (mk != 0ull) {
                const int t = 64 * w + (__ffsll((long long)mk) - 1);
                mk &= mk - 1ull;
                // span and plane read together (both depend on t only)
                const int sp = S[t * R + r];
                const f4v pk = ((lptr<const f4v>)(L.faces + t))[2];   // A B C keylo
                // the span's samples within this group as a bit mask
                const int lo = max((sp & 0xFFFF) - i, 0), hi = min(((sp >> 16) & 0x7FFF) - i, 15);
                const uint32_t in = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
                const float bdv = fmaf(pk.y, dv, pk.z);
                const uint32_t keylo = __float_as_uint(pk.w);
                if (sp < 0) {
                    // a light: few samples, each with its own sphere test; or a
                    // face whose 1/z may be no number: with the test spelt out
                    const bool light = AP && ((lptr<const int32_t>)(L.faces + t))[15] == 0;
#pragma unroll
                    for (int m = 0; m < 16; ++m) {
                        if (!((in >> m) & 1u)) continue;
                        const float invz = light ? light_invz(L, cam, t, du0 + (float)m, -dv) : fmaf(pk.x, du0 + (float)m, bdv);
                        if (invz > 0.0f) best[m] = key_max(best[m], __hiloint2double(__float_as_int(invz), (int)keylo));
                    }
                    continue;
                }
                // outside the span the sign bit is set: such keys, like those of
                // negative 1/z, lose to any other
                const uint32_t out = ~in;
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    const uint32_t hw = __float_as_uint(fmaf(pk.x, du0 + (float)m, bdv)) | ((out << (31 - m)) & 0x80000000u);
                    best[m] = key_max(best[m], __hiloint2double((int)hw, (int)keylo));
                }
            }
        }
        uint32_t c[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const uint32_t kh = (uint32_t)__double2hiint(best[m]), kl = (uint32_t)__double2loint(best[m]);
            const bool road = (bits >> m) & 1u;
            const bool box = (kh != 0u) & (!road | (kh >= rzb));          // (1/z of zero counts as no key)
            // the key's low byte names the list entry (entry 0 without a key: read, not used)
            const uint32_t boxc = ((lptr<const uint32_t>)(L.faces + (kl & 0xFFu)))[14];
            c[m] = box ? boxc : (road ? road_rgb : bg_rgb);
        }
        store16(img + 3 * ((int64_t)j * W + i), c);
    }
}

// ------------------------------------------------------------ resolve

typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// The rows that no box fragment touches are written as one run of bytes, in
// 16-byte pieces at 16-byte aligned addresses whatever the width and the
// image's address: piece q holds the bytes o .. o + 15 of the image, o = 16 q -
// a (a: the image's address mod 1024), which lie in the six pixels from f =
// o / 3 on, at phase o mod 3 of their run.  A store instruction writes one
// aligned KB (64 pieces), whole cache lines but at the run's ends; the
// wavefronts take turns.  A kernel that only writes images, one per workgroup,
// reaches 5.5..6.1 TB/s so, 3.6 TB/s where the KBs of 128 threads start within a
// cache line (images of 328,104 bytes), 3.9 TB/s where a lane writes 16 pixels
// as three pieces 48 bytes apart; a plain fill of the same memory reaches 6.9.
// Blocks of 3 to 30 KB per wavefront in turn are no faster than single KBs.

// byte b of a pixel's colour at channel c
__device__ __forceinline__ uint8_t channel(uint32_t rgb, int c) { return (uint8_t)(rgb >> (8 * c)); }

// The pieces of bytes [b0, b1) of an image: pieces [q0, q1) whole, in chunks of
// 64; chunks [f0, f1) are whole too.  This wavefront takes chunks c0, c0 + step, ...
struct Run {
    gp_v4i *out;         // piece 0
    int a, q0, q1, f0, f1, c0, step;
};

__device__ __forceinline__ Run run_of(uint8_t *img, int b0, int b1)
{
    Run r;
    r.a = (int)(reinterpret_cast<uintptr_t>(img) & 1023);
    r.out = reinterpret_cast<gp_v4i *>(img - r.a);
    r.q0 = (b0 + r.a + 15) >> 4;
    r.q1 = (b1 + r.a) >> 4;
    r.f0 = (r.q0 + 63) >> 6;
    r.f1 = max(r.q1 >> 6, r.f0);
    const int K = (int)blockDim.x >> 6, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    r.step = K;
    r.c0 = r.f0 + w;
    return r;
}

// the whole piece of the run's first or last, partial chunk that this lane
// writes, or -1: by the first wavefront, the last chunk by the last one
__device__ __forceinline__ int run_end_piece(const Run &r, bool last)
{
    const int K = (int)blockDim.x >> 6, w = (int)threadIdx.x >> 6, ln = (int)lane_id();
    if (w != (last ? K - 1 : 0)) return -1;
    const int q = last ? 64 * r.f1 + ln : 64 * (r.f0 - 1) + ln;
    return q >= r.q0 && q < (last ? r.q1 : min(r.q1, 64 * r.f0)) ? q : -1;
}

// the byte offset of a partial piece at the run's ends that this thread writes, or -1
__device__ __forceinline__ int run_end_byte(const Run &r, int b0, int b1)
{
    const int tid = (int)threadIdx.x;
    const int head = min(16 * r.q0 - r.a, b1) - b0, tail = b1 - max(16 * r.q1 - r.a, b0);
    if (tid < head) return b0 + tid;
    if (tid >= 32 && tid < 32 + tail && r.q0 <= r.q1) return b1 - tail + tid - 32;
    return -1;
}

// bytes [b0, b1) of the background (the sky)
__device__ __forceinline__ void write_sky(uint8_t *img, uint32_t bg, int b0, int b1)
{
    if (b0 >= b1) return;
    const Run r = run_of(img, b0, b1);
    const int ln = (int)lane_id();
    const uint32_t w[3] = {bg | (bg << 24), (bg >> 8) | (bg << 16), (bg >> 16) | (bg << 8)};
    auto piece = [&](int ph) -> gp_v4i {
        return gp_v4i{(int)__builtin_amdgcn_alignbyte(w[1], w[0], ph), (int)__builtin_amdgcn_alignbyte(w[2], w[1], ph),
                      (int)__builtin_amdgcn_alignbyte(w[0], w[2], ph), (int)__builtin_amdgcn_alignbyte(w[1], w[0], ph)};
    };
    auto phase = [&](int q) -> int { return (16 * q - r.a + 3072) % 3; };
    // a lane's pieces are 64 step apart: their phases repeat after three
    const gp_v4i v0 = piece(phase(64 * r.c0 + ln)), v1 = piece(phase(64 * (r.c0 + r.step) + ln)),
                 v2 = piece(phase(64 * (r.c0 + 2 * r.step) + ln));
    int c = r.c0;
    gp_v4i *p = r.out + (size_t)64 * c + ln;
    const size_t st = (size_t)64 * r.step;
    for (; c + 2 * r.step < r.f1; c += 3 * r.step, p += 3 * st) {
        p[0] = v0;
        p[st] = v1;
        p[2 * st] = v2;
    }
    if (c < r.f1) p[0] = v0;
    if (c + r.step < r.f1) p[st] = v1;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int q = run_end_piece(r, t != 0);
        if (q >= 0) r.out[q] = piece(phase(q));
    }
    const int o = run_end_byte(r, b0, b1);
    if (o >= 0) img[o] = channel(bg, o % 3);
}

// the pattern table: entry (p, b) holds the 16 bytes at phase p of the run of
// six pixels that are road where bit k of b is set and background elsewhere
__device__ __forceinline__ void build_patterns(const RgbLds &L, uint32_t road, uint32_t bg)
{
    for (int e = (int)threadIdx.x; e < 3 * 64; e += (int)blockDim.x) {
        const int ph = e >> 6;
        uint32_t c[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) c[k] = (e >> k) & 1 ? road : bg;
        const uint32_t w[5] = {c[0] | (c[1] << 24), (c[1] >> 8) | (c[2] << 16), (c[2] >> 16) | (c[3] << 8),
                               c[4] | (c[5] << 24), c[5] >> 8};
        gp_v4i v;
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = (int)__builtin_amdgcn_alignbyte(w[d + 1], w[d], ph);
        L.pat[e] = v;
    }
}

// bytes [b0, b1) of rows below the horizon, road or background by the coverage bits
__device__ __forceinline__ void write_road(const RgbLds &L, uint8_t *img, uint32_t road, uint32_t bg, int W, int b0,
                                           int b1)
{
    if (b0 >= b1) return;
    const Run r = run_of(img, b0, b1);
    const int ln = (int)lane_id();
    const int f0 = L.hr0 * W;            // pixel of coverage bit 0
    // the coverage bit of the first pixel of piece q, and its phase
    auto pixel = [&](int q, int &ph) -> int {
        const uint32_t o = (uint32_t)(16 * q - r.a), f = o / 3u;
        ph = (int)(o - 3u * f);
        return (int)f - f0;
    };
    // three of a lane's pieces are 1,024 step pixels, whole words of coverage:
    // word addresses advance, shifts and phases stay
    const lptr<const uint32_t> bits = (lptr<const uint32_t>)L.bits;
    lptr<const uint32_t> wd[3];
    lptr<const gp_v4i> tab[3];
    int sh[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int ph;
        const int f = pixel(64 * (r.c0 + k * r.step) + ln, ph);
        wd[k] = bits + (f >> 5);
        sh[k] = f & 31;
        tab[k] = (lptr<const gp_v4i>)L.pat + (ph << 6);
    }
    int c = r.c0, at = 0;
    gp_v4i *p = r.out + (size_t)64 * c + ln;
    const size_t st = (size_t)64 * r.step;
    for (; c + 2 * r.step < r.f1; c += 3 * r.step, p += 3 * st, at += 32 * r.step) {
        gp_v4i v[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = tab[k][__builtin_amdgcn_alignbit(wd[k][at + 1], wd[k][at], sh[k]) & 63u];
        p[0] = v[0];
        p[st] = v[1];
        p[2 * st] = v[2];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (c + k * r.step < r.f1) p[k * st] = tab[k][__builtin_amdgcn_alignbit(wd[k][at + 1], wd[k][at], sh[k]) & 63u];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int q = run_end_piece(r, t != 0);
        if (q >= 0) {
            int ph;
            const int f = pixel(q, ph);
            r.out[q] = L.pat[(ph << 6) | (int)(bits_at(L, f) & 63u)];
        }
    }
    const int o = run_end_byte(r, b0, b1);
    if (o >= 0) {
        const int f = o / 3;
        img[o] = channel(bits_at(L, f - f0) & 1u ? road : bg, o - 3 * f);
    }
}

// rows [r0, r1) that no box fragment touches: sky above the horizon, road or
// background below it
__device__ __forceinline__ void write_rows(const RgbLds &L, uint8_t *img, uint32_t road, uint32_t bg, int W, int r0, int r1)
{
    write_sky(img, bg, 3 * W * r0, 3 * W * min(r1, L.hr0));
    write_road(L, img, road, bg, W, 3 * W * max(r0, L.hr0), 3 * W * r1);
}

// Rows [b0, b1) of the key band: a box fragment wins where its 1/z is not below
// the road's (agents rank above roads on equal depth); otherwise road or
// background by the coverage bit.  rz(j): the road's 1/z in row j; color(w): the
// colour of a box or light key with low word w.
template <class Rz, class Color>
__device__ __forceinline__ void resolve_band(const RgbLds &L, int W, Rz rz, Color color, lptr<unsigned long long> keys,
                                             uint8_t *img, uint32_t road_rgb, uint32_t bg_rgb, int b0, int b1)
{
    const int gpr = (W + 15) >> 4;
    const int n = (b1 - b0) * gpr;
    for (int task = (int)threadIdx.x; task < n; task += (int)blockDim.x) {
        const int r = task / gpr, i = min((task - r * gpr) << 4, W - 16), j = b0 + r;
        const uint32_t bits = j >= L.hr0 ? bits_at(L, (j - L.hr0) * W + i) : 0u;
        const uint32_t rzb = __float_as_uint(rz(j));
        lptr<unsigned long long> kp = keys + (size_t)r * W + i;
        uint32_t c[16];
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            const unsigned long long kb = kp[m];
            const bool road = (bits >> m) & 1u;
            const bool box = (kb != 0ull) & (!road | ((uint32_t)(kb >> 32) >= rzb));
            c[m] = road ? road_rgb : bg_rgb;
            if (box) c[m] = color((uint32_t)kb);
        }
        store16(img + 3 * ((int64_t)j * W + i), c);
    }
}

// the palette as the roads show it (lit where the sim has a light) into LDS
__device__ __forceinline__ void road_palette(const DevSim &s, lptr<uint32_t> pal)
{
    const uint32_t q = s.shade ? shade_level(s, 0.0f, 0.0f, 4) : 255u;
    for (int p = (int)threadIdx.x; p < 256; p += (int)blockDim.x) {
        const uint32_t c = (uint32_t)s.palette[3 * p] | ((uint32_t)s.palette[3 * p + 1] << 8) | ((uint32_t)s.palette[3 * p + 2] << 16);
        pal[p] = s.shade ? shade_rgb(c, q) : c;
    }
}

// Four pixels from px on: colours c (byte 3 ignored), depths d, ids.
__device__ __forceinline__ void store4(const RenderOut &o, int64_t px, const uint32_t (&c)[4], const uint32_t (&d)[4],
                                       const uint32_t (&id)[4])
{
    struct __attribute__((packed, aligned(1))) P3 { uint32_t x, y, z; };
    struct __attribute__((packed, aligned(4))) P4 { uint32_t x, y, z, w; };
    *reinterpret_cast<P3 *>(o.rgb + 3 * px) = P3{(c[0] & 0xFFFFFFu) | (c[1] << 24), ((c[1] >> 8) & 0xFFFFu) | (c[2] << 16),
                                                 ((c[2] >> 16) & 0xFFu) | (c[3] << 8)};
    if (o.depth) *reinterpret_cast<P4 *>(o.depth + px) = P4{d[0], d[1], d[2], d[3]};
    if (o.primid) *reinterpret_cast<P4 *>(o.primid + px) = P4{id[0], id[1], id[2], id[3]};
}

// What four pixels from px on show by their keys: colour and optional depth and
// primitive id.  Road keys hold their palette index in the low byte; color(w) is
// the colour of a box or light key with low word w.  Writes 12 bytes of colour,
// 16 of depth and 16 of ids (n < 4: the first n pixels).
template <class Color>
__device__ __forceinline__ void show4(const DevSim &s, lptr<const uint32_t> pal, Color color, const RenderOut &o,
                                      const unsigned long long (&keys)[4], int64_t px, int n)
{
    uint32_t c[4], d[4], id[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned long long key = keys[k];
        const int prim = (kMaxPrims - 1) - (int)(((uint32_t)key >> 8) & (uint32_t)(kMaxPrims - 1));
        const bool box = ((uint32_t)key >> 31) != 0u;          // the class bit: boxes and lights
        c[k] = pal[box ? 0u : ((uint32_t)key & 0xFFu)];
        if (key == 0ull) c[k] = s.bg_rgb;
        if (box) c[k] = color((uint32_t)key);
        id[k] = key != 0ull ? (uint32_t)prim : 0xFFFFFFFFu;
        d[k] = 0x7F800000u;
        if (o.depth && key != 0ull) d[k] = __float_as_uint(1.0f / __uint_as_float((uint32_t)(key >> 32)));
    }
    if (n == 4) {
        store4(o, px, c, d, id);
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k >= n) continue;
        for (int ch = 0; ch < 3; ++ch) o.rgb[3 * (px + k) + ch] = channel(c[k], ch);
        if (o.depth) o.depth[px + k] = __uint_as_float(d[k]);
        if (o.primid) o.primid[px + k] = (int32_t)id[k];
    }
}

// Rows [r0, r1) that no box reaches, from the band of road keys (first row
// band0); four pixels of one row per lane, the last four of a row sharing some
// with those before them where W is no multiple of four (W >= 4).  rz(j): the
// road's 1/z in row j.  Most rows of a view: a lane's pixels take one division
// and no choice between boxes (2,048 views at 128 x 128 with depth and ids 119 us;
// 135 with a 64-bit key resolved per pixel).
template <class Rz>
__device__ __forceinline__ void resolve_roads(const DevSim &s, lptr<const uint32_t> pal, Rz rz, int W, int hr0,
                                              lptr<const uint32_t> road, int band0, const RenderOut &o, int64_t view_px, int r0,
                                              int r1)
{
    const int G = (W + 3) >> 2, B = (int)blockDim.x, dr = B / G, dg = B - dr * G;
    int r = r0 + (int)threadIdx.x / G, g = (int)threadIdx.x % G;
    while (r < r1) {
        const int i = min(4 * g, W - 4);
        uint32_t c[4], d[4], id[4], w[4] = {0u, 0u, 0u, 0u};
        uint32_t depth = 0x7F800000u;
        if (r >= hr0) {
            lptr<const uint32_t> p = road + (r - band0) * W + i;
#pragma unroll
            for (int k = 0; k < 4; ++k) w[k] = p[k];
            if (o.depth) depth = __float_as_uint(1.0f / rz(r));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool has = w[k] != 0u;
            c[k] = has ? pal[w[k] & 0xFFu] : s.bg_rgb;
            d[k] = has ? depth : 0x7F800000u;
            id[k] = has ? (uint32_t)(kMaxPrims - 1) - ((w[k] >> 8) & (uint32_t)(kMaxPrims - 1)) : 0xFFFFFFFFu;
        }
        store4(o, view_px + (int64_t)r * W + i, c, d, id);
        r += dr;
        g += dg;
        if (g >= G) {
            g -= G;
            ++r;
        }
    }
}

// Rows [r0, r1) from the band of road keys (first row band0; only its rows
// show road) and, where keys is set, the 64-bit box keys of the same rows; four
// pixels per lane.  rz(j): the road's 1/z in row j.
template <class Rz, class Color>
__device__ __forceinline__ void resolve_rows(const DevSim &s, lptr<const uint32_t> pal, Rz rz, Color color, int W, int hr0,
                                             lptr<const uint32_t> road, int band0, lptr<const unsigned long long> keys,
                                             const RenderOut &o, int64_t view_px, int r0, int r1)
{
    if (!keys && W >= 4) {
        resolve_roads(s, pal, rz, W, hr0, road, band0, o, view_px, r0, r1);
        return;
    }
    const int npix = (r1 - r0) * W;
    for (int p = 4 * (int)threadIdx.x; p < npix; p += 4 * (int)blockDim.x) {
        const int n = min(4, npix - p);
        int j = r0 + p / W, i = p - (j - r0) * W;
        unsigned long long k4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            k4[k] = 0ull;
            if (k < n) {
                if (keys) k4[k] = keys[p + k];
                if (j >= hr0) {
                    const uint32_t w = road[(j - band0) * W + i];
                    const unsigned long long rk = ((unsigned long long)__float_as_uint(rz(j)) << 32) | w;
                    if (w != 0u && rk > k4[k]) k4[k] = rk;
                }
            }
            if (++i == W) {
                i = 0;
                ++j;
            }
        }
        show4(s, pal, color, o, k4, view_px + (int64_t)r0 * W + p, n);
    }
}

// The fragments of every box and light in rows [b0, b1) folded into the key
// band, for views with more boxes than the records or entries than the list
// hold: as many boxes at a time are culled as there are records, the wavefronts
// (twelve clip queues fit the idle pattern table) list their faces in these rows,
// every wavefront folds them; records whose faces overflow the list are listed by
// the first wavefront, as many at a time as fit (ends with a barrier).  With the
// first wavefront listing everything, all rows of it in every band, depth and ids of
// 2,160 views 128 x 128 among 90 crowded boxes took 820 us, now 553, of 1,800 among
// 300 3,120, now 1,585 (the banded kernel 691 and 2,037).
template <bool AP, bool STEP>
__device__ __forceinline__ void stream_entries(const DevSim &s, const SceneRec &sc, const Cam &cam, int ego, const RgbLds &L,
                                               lptr<unsigned long long> keys, int b0, int b1, int wv, int K)
{
    const int nbox = sc.n_agents + sc.n_static;
    for (int j0 = 0; j0 < nbox; j0 += L.nrec) {
        if (threadIdx.x == 0) L.cnt[R_NSV] = L.cnt[R_AT] = L.cnt[R_NBT] = L.cnt[R_BOVF] = 0;
        __syncthreads();
        if (wv == 0) {
            const int j1 = min(j0 + L.nrec, nbox);
            cull_pass<STEP>(s, cam, L, cull_load<STEP>(s, sc, ego, j0, 0, j1), j0, 0, j1);
        }
        __syncthreads();
        const int ns = L.cnt[R_NSV];
        // all of them at once by all wavefronts
        const int kw = min(K, kPatBytes / (4 * kBoxClip)), unit = min(10, (ns + kw - 1) / kw);
        bool shared = true;
        for (int q = 0; q < ns;) {
            int bmn = 0, bmx = 0;
            if (shared) {
                for (int r = unit * wv; wv < kw && r < ns; r += unit * kw) {
                    int n = 0;
                    wave_lds_order();
                    if (!box_pass<AP>(s, sc, cam, L, r, min(unit, ns - r), b0, b1, L.cq + kBoxClip * wv, true, n, bmn, bmx)) break;
                }
            } else if (wv == 0) {
                int n = 0, step = 10;
                while (q < ns) {
                    int m = n;
                    wave_lds_order();
                    if (box_pass<AP>(s, sc, cam, L, q, min(step, ns - q), b0, b1, L.cq, false, m, bmn, bmx)) {
                        n = m;
                        q += min(step, ns - q);
                    } else if (n > 0 || step == 1) {
                        break;
                    } else {
                        step = 1;      // clipped faces: one record always fits an empty list
                    }
                }
                if (lane_id() == 0) {
                    L.cnt[R_NBT] = n;
                    L.cnt[R_AT] = q;
                }
            }
            __syncthreads();
            if (shared && L.cnt[R_BOVF] != 0) {
                shared = false;
                __syncthreads();       // the list is read by none
                continue;
            }
            q = shared ? ns : L.cnt[R_AT];
            box_band<AP>(L, cam, keys, L.cnt[R_NBT], b0, b1, wv, K);
            __syncthreads();
        }
    }
    for (int g0 = 0; AP && g0 < sc.n_signals; g0 += 64) {
        if (wv == 0) {
            int n = 0, bmn = 0, bmx = 0;
            (void)light_pass(s, sc, cam, L, g0, false, n, bmn, bmx);
            if (lane_id() == 0) L.cnt[R_NBT] = n;
        }
        __syncthreads();
        box_band<AP>(L, cam, keys, L.cnt[R_NBT], b0, b1, wv, K);
        __syncthreads();
    }
}

// Colour of a streamed box or light key: from its primitive (the list's
// entries are gone).
template <bool AP>
__device__ __forceinline__ uint32_t streamed_rgb(const DevSim &s, const SceneRec &sc, uint32_t keylo)
{
    const int prim = (kMaxPrims - 1) - (int)((keylo >> 8) & (uint32_t)(kMaxPrims - 1));
    const int nbox = sc.n_agents + sc.n_static;
    if (!AP || prim < 6 * nbox) {
        const int slot = box_slot(sc, prim / 6);
        const uint32_t c = s.box_rgb[slot];
        if (!AP || !s.shade) return c;
        float4 st;
        float2 cs;
        box_pose(s, slot, s.dims[slot], st, cs);
        return lit_heading(s, c, cs, prim % 6);
    }
    return signal_rgb(s, sc, prim - 6 * nbox - sc.n_roads);
}

// Rows [kr0, kr1) of a view whose box list overflowed, through bands of
// 64-bit keys (the whole workgroup; the region from the surviving-bin list on
// is free).  wv: this wavefront among the workgroup's.
template <bool AP>
__device__ __forceinline__ void key_band_rows(const DevSim &s, const SceneRec &sc, const Cam &cam, int ego, const RgbLds &L,
                                              uint8_t *img, uint32_t road_rgb, uint32_t bg_rgb, int kr0, int kr1, int wv)
{
    const int W = cam.W;
    lptr<unsigned long long> keys = L.work;
    for (int b0 = kr0; b0 < kr1; b0 += L.krows) {
        const int b1 = min(b0 + L.krows, kr1);
        __syncthreads();
        for (int p = (int)threadIdx.x; p < (b1 - b0) * W; p += (int)blockDim.x) keys[p] = 0ull;
        __syncthreads();
        stream_entries<AP, true>(s, sc, cam, ego, L, keys, b0, b1, wv, (int)blockDim.x >> 6);
        __syncthreads();
        resolve_band(
            L, W, [&](int j) { return fmaf(cam.road.B, ((float)j + 0.5f) - cam.cy, cam.road.C); },
            [&](uint32_t keylo) { return streamed_rgb<AP>(s, sc, keylo); },
            keys, img, road_rgb, bg_rgb, b0, b1);
    }
}

// ------------------------------------------------------------ per view

// Issue priority of the view's wavefronts (0..3) against the other views'
// on the same SIMDs.  Every view of a launch is resident at once, so the
// launch lasts as long as its slowest view: a view with much work left
// raises its priority and the views with little fill the gaps.  Only the
// instruction issue order changes, never a result.
__device__ __forceinline__ void view_priority(int p)
{
    p = __builtin_amdgcn_readfirstlane(p);
    if (p >= 3) __builtin_amdgcn_s_setprio(3);
    else if (p == 2) __builtin_amdgcn_s_setprio(2);
    else if (p == 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

}  // namespace

}  // namespace gp
