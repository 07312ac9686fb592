// Wave-split rgb raster of the Gigapixel hot path for gfx950 (MI355X).
//
// The rgb-only ego-centric render (Sec. 3.1 O_pixel; App. A "High-Throughput
// Batched Rendering": one world per ego agent, all views in one batched
// launch) for sims whose road strips share one colour and renders that need
// neither depth nor primitive ids.  Its results are bit-identical to the
// banded kernel (k_render) and to the plain definition: the same clip, snap,
// fill rule and winner order, only organised for throughput.
//
// One workgroup of K wavefronts (1..16) renders one view of any size from 16
// samples a row on, with up to 10 KB of LDS per wavefront where the image leaves
// room for it (about 19 KB at 128 x 128 and two wavefronts):
//   A  cull    the scene's road culling bins are tested against the view
//              (frustum, road depth limit and the row-gap test below) and its
//              boxes against the frustum; the surviving bins are listed in
//              LDS, the surviving boxes with what their faces are built from.
//   B  units   the waves share the work units.  A road unit is four surviving
//              bins (64 strip slots).  A strip first
//              meets a cheap test that can only reject strips covering no
//              sample: the frustum, the road depth limit, and the row-gap test
//              (every vertex a strip's clip can produce lies at camera height
//              -h, so its snapped row coordinate is a non-increasing function
//              of its depth; a strip whose depth range maps between two sample
//              rows covers none).  Survivors join the view's ring.  Then the
//              jobs: box units (face set-up and clipping of ten boxes into the
//              view's box list, a face as one quad where it covers what its triangles
//              cover) and set-up jobs of up to 64 ring strips (clip test, snap,
//              a quad or the two fan triangles, the clipper four strips per
//              wavefront); per (primitive, row) the exact span of covered
//              samples is OR-ed into the view's road coverage bits, which run
//              on from row to row over the rows below the horizon.
//   C  resolve rows no box face touches are written as one run of 16-byte
//              pieces (1 KB per store instruction): the sky from three constant
//              pieces, road rows from a table of the 64 patterns of six pixels
//              at the three byte phases.  Box rows go in chunks: the span of
//              every (face, row) once, masks of the faces per group of 16
//              samples, each lane folding the 64-bit keys of its 16 samples in
//              registers and writing 48 bytes.
//
// What bounds it: an image is a write stream, but at 128 x 128 the launch lasts as
// long as its views' chains of loads and LDS round trips (a wavefront waits for
// half of its time) and its slowest views; scenes of up to 128 agents are bound by
// VALU issue (84% busy), images from 434 x 252 on mostly by their stores.  Step +
// render on one MI355X, before the wave-split raster took a size / now: 2,048 views
// at 128 x 128 74 / 45 us (2.2 TB/s), 8,192 views at 210 x 126 480 / 177 us (3.7
// TB/s), at 434 x 252 1,505 / 553 us (4.9 TB/s), 4,096 views at 512 x 512 2,140 / 655
// us (4.9 TB/s), 64 scenes of 4..128 agents with three cameras at 128 x 128 2,730 /
// 265 us.
//
// Every float operation is written out (fmaf for fused operations) and the
// file is compiled with -ffp-contract=off, correctly rounded division and
// IEEE denormals.

#include "gp_full.h"      // the general raster, compiled here too
#include "gp_view.h"

namespace gp {

namespace {

// A render that steps the agents first (s.act): every view computes the states
// after the step of the boxes it culls by itself, and the state arrays are
// advanced in place by the last view of a scene to have read them: views count
// themselves in once their reads are done (the barrier before has every
// wavefront past them), and the one that completes the count steps the scene's
// agents and clears it.  A step kernel of its own before the render costs 5 us
// of start and drain: step + render of 2,048 views at 128 x 128 60.0 us, so 52.3
// us when this was built.
__device__ __forceinline__ int view_arrives(const DevSim &s, int scene)
{
    int n = 0;
    if (s.act && threadIdx.x == 0)
        n = (int)__hip_atomic_fetch_add(s.scene_done + (size_t)scene * kDoneStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return n;
}

// by the first wavefront: arrived is lane 0's view_arrives
__device__ __forceinline__ void step_scene(const DevSim &s, const SceneRec &sc, int scene, int arrived)
{
    if (!s.act || threadIdx.x >= 64) return;
    if (__builtin_amdgcn_readlane(arrived, 0) != sc.n_agents * s.n_cams - 1) return;
    for (int a = (int)lane_id(); a < sc.n_agents; a += 64) step_agent(s, s.act, sc.agent_base + a);
    if (threadIdx.x == 0) __hip_atomic_store(s.scene_done + (size_t)scene * kDoneStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// AP: the sim has a light or traffic lights (instances of their own, so that
// they add nothing to the plain ones).  Lit streets used to take the general
// kernel, which folds every road strip's keys with 64-bit LDS atomics and
// writes single bytes: 2,048 views at 128 x 128 with 16 obstacles and 12 lights
// a scene 326 us, here 56 us.  cam_index: the view's camera in s.cam_dir (0 in a
// batch's copy of the sim's record, which holds the view's direction only).
template <bool AP>
__device__ __forceinline__ void render_view_rgb(const DevSim &s, uint8_t *rgb, RgbLds L, const ViewInit &vi, int cam_index)
{
    const int B = (int)blockDim.x, K = B >> 6;
    const int tid = (int)threadIdx.x, wv = tid >> 6;
    const int view = vi.view, scene = vi.scene, ego = vi.ego;
    const SceneRec &sc = vi.sc;
    const int nbox = sc.n_agents + sc.n_static;
    CullIn in = cull_load<true>(s, sc, ego, 64 * wv, sc.n_bins, nbox);
    const Cam cam = make_cam<true>(s, sc, ego, cam_index);
    const int W = cam.W, H = cam.H;

    const int nbits = ((W * (H - L.hr0) + 63) >> 6) + 1;
    for (int p = tid; p < nbits; p += B) L.bits[p] = 0ull;
    const int nlu = AP ? (sc.n_signals + 63) / 64 : 0;
    if (tid < R_NCNT) L.cnt[tid] = tid == R_BMIN ? 0x7FFFFFFF : (tid == R_BMAX ? -1 : 0);
    __syncthreads();

    // ---- A: road culling bins and boxes
    cull_all<true>(s, sc, cam, ego, L, in, wv, B);
    __syncthreads();

    // ---- B: the road and box units (set-up and clipping of the faces into the
    // box list)
    const int nsb = L.cnt[R_NSB], nsv = L.cnt[R_NSV];
    const int ubox = box_unit(K);
    const int nbu = nsv <= L.nrec ? (nsv + ubox - 1) / ubox : 0;
    // road work ahead grows with the surviving bins (a mean view keeps about a dozen)
    const int prio_b = nsb >= 24 ? 2 : (nsb >= 16 ? 1 : 0);
    view_priority(prio_b);
    const int most = 3 * nsv + (AP ? sc.n_signals : 0);
    if (most > L.bcap && nsv <= L.nrec) grow_list<false>(L, most, K, W);
    WaveSt ws = wave_state(L, wv);
    // more surviving bins than the list holds: the scene's bins in segments that
    // it does hold
    const bool over = nsb > L.bins;
    for (int s0 = 0;;) {
        if (over) {
            __syncthreads();                       // the counters are read
            if (tid == 0) L.cnt[R_NSB] = L.cnt[R_RING] = L.cnt[R_JOB] = 0;
            __syncthreads();
            const int s1 = min(s0 + L.bins, sc.n_bins);
            for (int b0 = s0 + 64 * wv; b0 < s1; b0 += B) cull_pass<false>(s, cam, L, cull_load<false>(s, sc, ego, b0, s1, 0), b0, s1, 0);
            __syncthreads();
        }
        road_work(
            s, sc, L, over ? L.cnt[R_NSB] : nsb, s0 == 0 ? nbu + nlu : 0,
            [&](bool live, const float4 &q0, const float4 &q1) -> bool {
                float x[4], z[4];
                ground_xz(cam, q0.x, q0.y, x[0], z[0]);
                ground_xz(cam, q0.z, q0.w, x[1], z[1]);
                ground_xz(cam, q1.x, q1.y, x[2], z[2]);
                ground_xz(cam, q1.z, q1.w, x[3], z[3]);
                return live && !road_culled<false>(cam, x, z, 0, cam.H);
            },
            [&](int u) {
                if (AP && u >= nbu) do_lights(s, sc, cam, L, u - nbu);
                else do_boxes<AP>(s, sc, cam, L, u, ubox, nsv, (lptr<int32_t>)ws.tris);   // the staging is free here
            },
            [&](int a, int n) {
                setup_job<false>(s, sc, cam, L, ws, a, n, [&](int t) { road_spans(L, cam, ws, t); });
            });
        s0 += L.bins;
        if (!over || s0 >= sc.n_bins) break;
    }

    // ---- C: resolve
    uint8_t *img = rgb + 3 * ((int64_t)view * W * H);
    const int nbt = L.cnt[R_NBT];
    const bool ovf = L.cnt[R_BOVF] != 0 || nsv > L.nrec;
    int kr0 = H, kr1 = H;          // rows that need the key band
    if (ovf) {
        kr0 = 0;
    } else if (nbt > 0) {
        kr0 = L.cnt[R_BMIN];
        kr1 = L.cnt[R_BMAX] + 1;
    }
    // the box rows are the costly part of the resolve (a mean view has about a dozen)
    view_priority(max(prio_b, kr1 - kr0 >= 64 ? 3 : (kr1 - kr0 >= 32 ? 2 : 0)));
    const uint32_t bg_rgb = s.bg_rgb;
    const uint32_t road_rgb = AP && s.shade ? shade_rgb(s.road_rgb, shade_level(s, 0.0f, 0.0f, 4)) : s.road_rgb;
    free_region(L, ovf ? L.bcap : nbt, W);
    // every state this view needs is read, unless its boxes are streamed
    const int arrived = ovf ? 0 : view_arrives(s, scene);
    const int mrows = max(1, mask_rows_fit(L.region, nbt, W, L.nmw));
    // the pattern table, and the masks of the first chunk of box rows, in
    // chunks of rows whose items fit; the rows without boxes go with the first
    // chunk's spans
    const bool masks = !ovf && kr0 < kr1;
    int c1 = min(kr0 + mrows, kr1);
    build_patterns(L, road_rgb, bg_rgb);
    const int G = (W + 15) >> 4;
    if (masks)
        for (int p = tid; p < L.nmw * G * (c1 - kr0); p += B) L.work[p] = 0ull;
    __syncthreads();
    if (!ovf) step_scene(s, sc, scene, arrived);
    write_rows(L, img, road_rgb, bg_rgb, W, 0, kr0);
    write_rows(L, img, road_rgb, bg_rgb, W, kr1, H);
    if (masks) {
        for (int c0 = kr0;;) {
            box_spans<AP>(L, cam, nbt, c0, c1, wv, K);
            __syncthreads();
            resolve_masks<AP>(L, cam, img, road_rgb, bg_rgb, c0, c1, wv, K);
            if (c1 == kr1) return;
            c0 = c1;
            c1 = min(c0 + mrows, kr1);
            __syncthreads();
            for (int p = tid; p < L.nmw * G * (c1 - c0); p += B) L.work[p] = 0ull;
            __syncthreads();
        }
    }
    if (ovf) {
        key_band_rows<AP>(s, sc, cam, ego, L, img, road_rgb, bg_rgb, kr0, kr1, wv);
        __syncthreads();
        step_scene(s, sc, scene, view_arrives(s, scene));
    }
}

__device__ __forceinline__ void carve_rgb(unsigned char *smem, RgbLds &L, int W, int H, const RgbCfg &c)
{
    const RgbLayout l = rgb_layout(W, H, c);
    L.cnt = (lptr<int32_t>)(smem + l.cnt);
    L.bits = (lptr<unsigned long long>)(smem + l.bits);
    L.faces = (lptr<FaceRec>)(smem + l.faces);
    L.recs = (lptr<BoxRec>)(smem + l.recs);
    L.sbins = (lptr<int32_t>)(smem + l.sbins);
    L.sring = (lptr<int32_t>)(smem + l.sring);
    L.waves = (lptr<unsigned char>)(smem + l.waves);
    L.hr0 = first_road_row(H);
    L.bcap = c.bcap;
    L.bins = c.bins_cap;
    L.nrec = c.recs;
    L.tail = (int)(l.total - l.faces);
    L.batch = kBatch;
    L.ring = kSharedRing;
}

// One workgroup per view: view view_begin + blockIdx.x (ordered 0), or
// order[blockIdx.x].
template <bool AP>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_render_rgb(DevSim s, RenderOut o, RgbCfg c,
                                                                                            int ordered, int view_begin)
{
    extern __shared__ __align__(16) unsigned char smem[];
    RgbLds L;
    carve_rgb(smem, L, s.width, s.height, c);
    const ViewInit vi = view_init(ordered ? s.vorder + blockIdx.x : s.vinit + view_begin + (int)blockIdx.x);
    render_view_rgb<AP>(s, o.rgb, L, vi, vi.cam);
}

// Batched render over several sims (serving): workgroup b renders item b, a
// (sim, view) pair.  The sim's record is copied out of the table with its
// view's camera only: a copy indexed by camera would live in scratch memory,
// and a record read in place would be loaded again after every store.  Eight
// scenes of 8..128 agents at 128 x 128: 60 us per batch, 142 us in the banded
// queue kernel.
template <bool AP>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_render_rgb_multi(
    const SimEntry *__restrict__ tab, const int2 *__restrict__ items, RgbCfg c)
{
    extern __shared__ __align__(16) unsigned char smem[];
    typedef const __attribute__((address_space(4))) SimEntry *ctab;     // constant address space: scalar loads
    const int sim = __builtin_amdgcn_readfirstlane(items[blockIdx.x].x);
    const int view = __builtin_amdgcn_readfirstlane(items[blockIdx.x].y);
    ctab e = (ctab)tab + sim;
    DevSim s;
    s.scenes = e->s.scenes;
    s.camk.cx = e->s.camk.cx;
    s.camk.cy = e->s.camk.cy;
    s.camk.F256 = e->s.camk.F256;
    s.camk.CX256 = e->s.camk.CX256;
    s.camk.CY256 = e->s.camk.CY256;
    s.camk.G = e->s.camk.G;
    s.camk.t_left = e->s.camk.t_left;
    s.camk.t_right = e->s.camk.t_right;
    s.camk.t_top = e->s.camk.t_top;
    s.camk.t_bottom = e->s.camk.t_bottom;
    s.camk.road_b = e->s.camk.road_b;
    s.state = e->s.state;
    s.cs = e->s.cs;
    s.dims = e->s.dims;
    s.agent_color = e->s.agent_color;
    s.roads = e->s.roads;
    s.road_index = e->s.road_index;
    s.road_color = e->s.road_color;
    s.bins = e->s.bins;
    s.palette = e->s.palette;
    s.width = e->s.width;
    s.height = e->s.height;
    s.box_rgb = e->s.box_rgb;
    s.road_rgb = e->s.road_rgb;
    s.bg_rgb = e->s.bg_rgb;
    s.road_zmax = e->s.road_zmax;
    s.signals = e->s.signals;
    s.signal_color = e->s.signal_color;
    s.act = e->s.act;
    s.scene_done = e->s.scene_done;
    s.halted = e->s.halted;
    s.dt = e->s.dt;
    s.n_agents = e->s.n_agents;
    s.n_cams = e->s.n_cams;
    s.focal = e->s.focal;
    s.cam_height = e->s.cam_height;
    s.z_near = e->s.z_near;
    s.z_far = e->s.z_far;
#pragma unroll
    for (int k = 0; k < 4; ++k) s.light[k] = e->s.light[k];
    s.shade = e->s.shade;
    const ViewInit vi = view_init(e->s.vinit + view);
    s.cam_dir[0][0] = e->s.cam_dir[vi.cam][0];
    s.cam_dir[0][1] = e->s.cam_dir[vi.cam][1];
    RgbLds L;
    carve_rgb(smem, L, s.width, s.height, c);
    render_view_rgb<AP>(s, e->o.rgb, L, vi, 0);
}

}  // namespace

size_t rgb_lds_bytes(int width, int height, const RgbCfg &c) { return rgb_layout(width, height, c).total; }

hipError_t launch_render_rgb(const DevSim &s, const RenderOut &o, const RgbCfg &c, int ordered, int view_begin,
                             int grid, hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    if (c.waves < 1 || c.waves > 16 || s.width < 16 || c.bcap < 64 || c.bcap > 256 || c.recs < 1 || c.recs > 64) return hipErrorInvalidValue;
    const size_t lds = rgb_lds_bytes(s.width, s.height, c);
    const dim3 block(64 * c.waves);
    if (c.appear) hipLaunchKernelGGL(k_render_rgb<true>, dim3(grid), block, lds, st, s, o, c, ordered, view_begin);
    else hipLaunchKernelGGL(k_render_rgb<false>, dim3(grid), block, lds, st, s, o, c, ordered, view_begin);
    return hipGetLastError();
}

hipError_t launch_render_rgb_multi(const SimEntry *tab, const int2 *items, int n_items, const RgbCfg &c, int width,
                                   int height, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    if (c.waves < 1 || c.waves > 16 || width < 16 || c.bcap < 64 || c.bcap > 256 || c.recs < 1 || c.recs > 64) return hipErrorInvalidValue;
    const size_t lds = rgb_lds_bytes(width, height, c);
    const dim3 block(64 * c.waves);
    if (c.appear) hipLaunchKernelGGL(k_render_rgb_multi<true>, dim3(n_items), block, lds, st, tab, items, c);
    else hipLaunchKernelGGL(k_render_rgb_multi<false>, dim3(n_items), block, lds, st, tab, items, c);
    return hipGetLastError();
}

}  // namespace gp
