// General raster of the Gigapixel hot path for gfx950 (MI355X): the ego-centric
// render (Sec. 3.1 O_pixel) with depth and primitive ids, and of sims whose
// road strips have several colours; with the directional light and traffic
// lights where the sim has them.  Same clip, snap, fill rule and winner order
// as the other rasterisers.
//
// One workgroup per view, its work divided as in the wave-split rgb raster
// (gp_view.h): bins, strips that pass the cheap test in a ring, set-up jobs, box
// and light units into the view's list.  Here every fragment counts, so the
// image goes in bands of rows whose 64-bit keys lie in LDS: per band the strips
// that reach its rows are set up, their exact spans cut into pieces of 16
// samples that fold the strip's key (its 1/z is the row's) with LDS atomic max,
// then the list's entries likewise; a lane resolves four pixels and writes 12
// bytes of colour, 16 of depth and 16 of ids.
//
// Bound by the keys' folding and the three output streams.  One MI355X, 2,048
// views at 128 x 128 with depth and ids: 180 us (the banded kernel, which sets up
// every strip of a surviving bin and writes single bytes, 282 us).
#include "gp_view.h"

namespace gp {

namespace {

struct FullLayout {
    size_t cnt, faces, recs, cq, pal, sbins, sring, waves, keys, total;
};

__host__ __device__ inline FullLayout full_layout(int W, const FullCfg &c)
{
    FullLayout l;
    size_t o = 0;
    l.cnt = o; o = align16(o + 4 * R_NCNT);
    l.faces = o; o = align16(o + sizeof(FaceRec) * (size_t)c.bcap);
    l.recs = o; o = align16(o + sizeof(BoxRec) * (size_t)c.recs);
    l.cq = o; o = align16(o + 4 * (size_t)kBoxClip);
    l.pal = o; o = align16(o + 4 * 256);
    l.sbins = o; o = align16(o + 4 * (size_t)c.bins_cap);
    l.sring = o; o = align16(o + 4 * (size_t)kSharedRing);
    l.waves = o; o = align16(o + (size_t)kWaveBytes * (size_t)c.waves);
    l.keys = o; o = align16(o + 8 * (size_t)W * (size_t)c.band_rows);
    l.total = o;
    return l;
}

// One workgroup per view: view view_begin + blockIdx.x (ordered 0), or
// order[blockIdx.x].
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_render_full(DevSim s, RenderOut o, FullCfg c,
                                                                                             int ordered, int view_begin)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int B = (int)blockDim.x, K = B >> 6, tid = (int)threadIdx.x, wv = tid >> 6;
    const int W = s.width, H = s.height;
    const FullLayout l = full_layout(W, c);
    RgbLds L = {};
    L.cnt = (lptr<int32_t>)(smem + l.cnt);
    L.faces = (lptr<FaceRec>)(smem + l.faces);
    L.recs = (lptr<BoxRec>)(smem + l.recs);
    L.cq = (lptr<int32_t>)(smem + l.cq);
    L.sbins = (lptr<int32_t>)(smem + l.sbins);
    L.sring = (lptr<int32_t>)(smem + l.sring);
    L.waves = (lptr<unsigned char>)(smem + l.waves);
    L.work = (lptr<unsigned long long>)(smem + l.keys);
    L.bcap = c.bcap;
    L.batch = kBatch;
    L.ring = kSharedRing;
    L.bins = c.bins_cap;
    L.nrec = c.recs;
    L.krows = c.band_rows;
    L.hr0 = first_road_row(H);
    lptr<uint32_t> pal = (lptr<uint32_t>)(smem + l.pal);

    const ViewInit vi = view_init(ordered ? s.vorder + blockIdx.x : s.vinit + view_begin + (int)blockIdx.x);
    const int view = vi.view, ego = vi.ego;
    const SceneRec &sc = vi.sc;
    const int nbox = sc.n_agents + sc.n_static;
    CullIn in = cull_load<false>(s, sc, ego, 64 * wv, sc.n_bins, nbox);
    const Cam cam = make_cam(s, sc, ego, vi.cam);
    for (int p = tid; p < 256; p += B)
        pal[p] = (uint32_t)s.palette[3 * p] | ((uint32_t)s.palette[3 * p + 1] << 8) | ((uint32_t)s.palette[3 * p + 2] << 16);
    if (tid < R_NCNT) L.cnt[tid] = tid == R_BMIN ? 0x7FFFFFFF : (tid == R_BMAX ? -1 : 0);
    __syncthreads();
    cull_all<false>(s, sc, cam, ego, L, in, wv, B);
    __syncthreads();
    const int nsb = L.cnt[R_NSB], nsv = L.cnt[R_NSV];
    const int ubox = box_unit(K);
    const int nbu = nsv <= L.nrec ? (nsv + ubox - 1) / ubox : 0, nlu = (sc.n_signals + 63) / 64;
    WaveSt ws = wave_state(L, wv);
    for (int b0 = 0; b0 < H; b0 += L.krows) {
        const int b1 = min(b0 + L.krows, H);
        const int r0 = max(b0, L.hr0), r1 = max(b1, L.hr0);        // rows that can show road
        if (b0 > 0) __syncthreads();                               // the last band's keys are read
        for (int p = tid; p < (b1 - b0) * W; p += B) L.work[p] = 0ull;
        if (b0 > 0 && tid == 0) L.cnt[R_RING] = L.cnt[R_JOB] = 0;
        __syncthreads();
        // the first band's road work lists the boxes and lights too
        if (b0 == 0 || r0 < r1)
            (void)road_work(
                s, sc, L, r0 < r1 ? nsb : 0, b0 == 0 ? nbu + nlu : 0, false,
                [&](bool live, const float4 &q0, const float4 &q1) -> bool {
                    float x[4], z[4];
                    ground_xz(cam, q0.x, q0.y, x[0], z[0]);
                    ground_xz(cam, q0.z, q0.w, x[1], z[1]);
                    ground_xz(cam, q1.x, q1.y, x[2], z[2]);
                    ground_xz(cam, q1.z, q1.w, x[3], z[3]);
                    return live && !road_culled<false>(cam, x, z, r0, r1);
                },
                [&](int u) {
                    if (u >= nbu) do_lights(s, sc, cam, L, u - nbu);
                    else do_boxes<true>(s, sc, cam, L, u, ubox, nsv, (lptr<int32_t>)ws.tris);   // the staging is free here
                },
                [&](int a, int n) {
                    setup_job<true>(s, sc, cam, L, ws, a, n, [&](int t) { road_fold(L, cam, ws, t, r0, r1, b0); });
                });
        const bool ovf = L.cnt[R_BOVF] != 0 || nsv > L.nrec;
        if (!ovf) box_band<true>(L, cam, L.work, L.cnt[R_NBT], b0, b1, wv, K);
        else stream_entries<true, false>(s, sc, cam, ego, L, L.work, b0, b1, wv, K);
        __syncthreads();
        resolve_full(
            s, (lptr<const uint32_t>)pal,
            [&](uint32_t keylo) -> uint32_t {
                if (ovf) return streamed_rgb<true>(s, sc, keylo);
                return ((lptr<const uint32_t>)(L.faces + (keylo & 0xFFu)))[14];
            },
            (lptr<const unsigned long long>)L.work, o, ((int64_t)view * H + b0) * W, (b1 - b0) * W);
    }
}

}  // namespace

size_t full_lds_bytes(int width, const FullCfg &c) { return full_layout(width, c).total; }

hipError_t launch_render_full(const DevSim &s, const RenderOut &o, const FullCfg &c, int ordered, int view_begin, int grid,
                              hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    if (c.waves < 1 || c.waves > 16 || c.band_rows < 1 || c.bcap < 64 || c.bcap > 256 || c.recs < 1 || c.recs > 64 || c.bins_cap < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_render_full, dim3(grid), dim3(64 * c.waves), full_lds_bytes(s.width, c), st, s, o, c, ordered,
                       view_begin);
    return hipGetLastError();
}

}  // namespace gp
