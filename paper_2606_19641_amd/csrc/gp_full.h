// General raster of the Gigapixel hot path for gfx950 (MI355X): the ego-centric
// render (Sec. 3.1 O_pixel) with depth and primitive ids, and of sims whose
// road strips have several colours; with the directional light and traffic
// lights where the sim has them.  Same clip, snap, fill rule and winner order
// as the other rasterisers.
//
// One workgroup per view, its work divided as in the wave-split rgb raster
// (gp_view.h): bins, strips that pass the cheap test in a ring, set-up jobs, box
// and light units into the view's list.  Here it matters which strip a sample
// shows, but every strip lies in one plane: in a row they all have the same 1/z,
// and the largest 32-bit key word wins.  So the rows below the horizon go in bands
// of road key words in LDS: per band the strips that reach its rows are set up,
// their exact spans cut into pieces of 16 samples that fold the strip's word with
// LDS atomic max.  Box rows then take the group masks and spans of the rgb raster
// and fold 64-bit keys in registers, eight samples per lane; in the other rows a
// lane resolves four pixels from the road words alone.  A lane writes 12 bytes of
// colour, 16 of depth and 16 of ids per four pixels.
//
// Bound by the road words' folding and the three output streams.  One MI355X,
// 2,048 views at 128 x 128 with depth and ids: 119 us (with 64-bit keys of every
// fragment in bands half as high 171, in the banded kernel, which sets up every
// strip of a surviving bin and writes single bytes, 282).
#pragma once

#include "gp_view.h"

namespace gp {

namespace {

struct FullLayout {
    size_t cnt, recs, pal, sbins, faces, sring, waves, road, total;
};

__host__ __device__ inline FullLayout full_layout(int W, const FullCfg &c)
{
    FullLayout l;
    size_t o = 0;
    l.cnt = o; o = align16(o + 4 * R_NCNT);
    l.recs = o; o = align16(o + sizeof(BoxRec) * (size_t)c.recs);
    l.pal = o; o = align16(o + 4 * 256);
    l.sbins = o; o = align16(o + 4 * (size_t)c.bins_cap);
    l.faces = o; o = align16(o + sizeof(FaceRec) * (size_t)c.bcap);
    const size_t least = align16(o + (size_t)resolve_bytes(W));
    l.sring = o; o = align16(o + 4 * (size_t)kSharedRing);
    l.waves = o; o = align16(o + (size_t)kWaveBytes * (size_t)c.waves);
    o = o > least ? o : least;
    l.road = o; o = align16(o + 4 * (size_t)W * (size_t)c.band_rows);
    l.total = o;
    return l;
}

// Rows [c0, c1) from the road keys and the box faces' group masks and spans, as
// in the rgb raster's resolve_masks, but eight samples per task: with sixteen
// the keys and what is written of them do not fit the registers.
template <class Color>
__device__ __forceinline__ void resolve_box_rows(const DevSim &s, lptr<const uint32_t> pal, Color color, const RgbLds &L,
                                                 const Cam &cam, lptr<const uint32_t> road, int band0, const RenderOut &o,
                                                 int64_t view_px, int c0, int c1)
{
    const int W = cam.W, R = c1 - c0, G = (W + 15) >> 4, n = 2 * R * G, nmw = L.nmw;
    lptr<const unsigned long long> M = (lptr<const unsigned long long>)L.work;
    lptr<const int32_t> S = (lptr<const int32_t>)(M + nmw * G * R);
    for (int task = (int)threadIdx.x; task < n; task += (int)blockDim.x) {
        const int r = task / (2 * G), h = task - 2 * r * G, g = h >> 1, i = min(g << 4, W - 16) + 8 * (h & 1), j = c0 + r;
        const float dv = ((float)j + 0.5f) - cam.cy;
        // sample offsets ((float)(i + m) + 0.5f) - cx are small exact values: du0 + m
        const float du0 = ((float)i + 0.5f) - cam.cx;
        const int rzb = __float_as_int(fmaf(cam.road.B, dv, cam.road.C));
        double best[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const uint32_t w = j >= L.hr0 ? road[(j - band0) * W + i + m] : 0u;
            best[m] = __hiloint2double(w != 0u ? rzb : 0, (int)w);
        }
        for (int w = 0; w < nmw; ++w) {
            unsigned long long mk = M[nmw * (G * r + g) + w];
            while (mk != 0ull) {
                const int t = 64 * w + (__ffsll((long long)mk) - 1);
                mk &= mk - 1ull;
                const int sp = S[t * R + r];
                const f4v pk = ((lptr<const f4v>)(L.faces + t))[2];   // A B C keylo
                const int lo = max((sp & 0xFFFF) - i, 0), hi = min(((sp >> 16) & 0x7FFF) - i, 7);
                if (lo > hi) continue;
                const uint32_t in = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
                const float bdv = fmaf(pk.y, dv, pk.z);
                const uint32_t keylo = __float_as_uint(pk.w);
                if (sp < 0) {
                    const bool light = ((lptr<const int32_t>)(L.faces + t))[15] == 0;
#pragma unroll
                    for (int m = 0; m < 8; ++m) {
                        if (!((in >> m) & 1u)) continue;
                        const float invz = light ? light_invz(L, cam, t, du0 + (float)m, -dv) : fmaf(pk.x, du0 + (float)m, bdv);
                        if (invz > 0.0f) best[m] = key_max(best[m], __hiloint2double(__float_as_int(invz), (int)keylo));
                    }
                    continue;
                }
                const uint32_t out = ~in;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const uint32_t hw = __float_as_uint(fmaf(pk.x, du0 + (float)m, bdv)) | ((out << (31 - m)) & 0x80000000u);
                    best[m] = key_max(best[m], __hiloint2double((int)hw, (int)keylo));
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            unsigned long long k4[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                k4[k] = (unsigned long long)__double_as_longlong(best[4 * q + k]);
                if (k4[k] >> 32 == 0ull) k4[k] = 0ull;               // 1/z of zero counts as no key
            }
            show4(s, pal, color, o, k4, view_px + (int64_t)j * W + i + 4 * q, 4);
        }
    }
}

// One workgroup per view: view view_begin + blockIdx.x (ordered 0), or the
// view of workgroup blockIdx.x.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_render_full(DevSim s, RenderOut o, FullCfg c,
                                                                                             int ordered, int view_begin)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int B = (int)blockDim.x, K = B >> 6, tid = (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = s.width, H = s.height;
    const FullLayout l = full_layout(W, c);
    RgbLds L = {};
    L.cnt = (lptr<int32_t>)(smem + l.cnt);
    L.recs = (lptr<BoxRec>)(smem + l.recs);
    L.faces = (lptr<FaceRec>)(smem + l.faces);
    L.sbins = (lptr<int32_t>)(smem + l.sbins);
    L.sring = (lptr<int32_t>)(smem + l.sring);
    L.waves = (lptr<unsigned char>)(smem + l.waves);
    L.bcap = c.bcap;
    L.batch = kBatch;
    L.ring = kSharedRing;
    L.bins = c.bins_cap;
    L.nrec = c.recs;
    L.tail = (int)(l.road - l.faces);
    L.hr0 = first_road_row(H);
    lptr<uint32_t> pal = (lptr<uint32_t>)(smem + l.pal), road = (lptr<uint32_t>)(smem + l.road);

    const ViewInit vi = view_init(ordered ? s.vorder + blockIdx.x : s.vinit + view_begin + (int)blockIdx.x);
    const int view = vi.view, ego = vi.ego;
    const SceneRec &sc = vi.sc;
    const int nbox = sc.n_agents + sc.n_static;
    CullIn in = cull_load<false>(s, sc, ego, 64 * wv, sc.n_bins, nbox);
    const Cam cam = make_cam(s, sc, ego, vi.cam);
    road_palette(s, pal);
    if (tid < R_NCNT) L.cnt[tid] = tid == R_BMIN ? 0x7FFFFFFF : (tid == R_BMAX ? -1 : 0);
    __syncthreads();
    cull_all<false>(s, sc, cam, ego, L, in, wv, B);
    __syncthreads();
    const int nsb = L.cnt[R_NSB], nsv = L.cnt[R_NSV];
    const int ubox = box_unit(K);
    const int nbu = nsv <= L.nrec ? (nsv + ubox - 1) / ubox : 0, nlu = (sc.n_signals + 63) / 64;
    const int most = 3 * nsv + sc.n_signals;
    if (most > L.bcap && nsv <= L.nrec) grow_list<true>(L, most, K, W);
    WaveSt ws = wave_state(L, wv);
    const int64_t view_px = (int64_t)view * H * W;
    int nbt = 0, kr0 = H, kr1 = H;               // listed entries, the rows that they reach
    bool ovf = false;
    auto color = [&](uint32_t keylo) -> uint32_t {
        if (ovf) return streamed_rgb<true>(s, sc, keylo);
        return ((lptr<const uint32_t>)(L.faces + (keylo & 0xFFu)))[14];
    };
    auto rz = [&](int j) { return fmaf(cam.road.B, ((float)j + 0.5f) - cam.cy, cam.road.C); };
    // Bands of the rows below the horizon; the rows above go with the first
    for (int b0 = L.hr0;; b0 += c.band_rows) {
        const bool first = b0 == L.hr0;
        const int b1 = min(b0 + c.band_rows, H);
        if (!first) __syncthreads();                               // the last band's keys are read
        for (int p = tid; p < (b1 - b0) * W; p += B) road[p] = 0u;
        if (!first && tid == 0) L.cnt[R_RING] = L.cnt[R_JOB] = 0;
        __syncthreads();
        // the first band's road work lists the boxes and lights too
        road_work(
            s, sc, L, b0 < b1 ? nsb : 0, first ? nbu + nlu : 0,
            [&](bool live, const float4 &q0, const float4 &q1) -> bool {
                float x[4], z[4];
                ground_xz(cam, q0.x, q0.y, x[0], z[0]);
                ground_xz(cam, q0.z, q0.w, x[1], z[1]);
                ground_xz(cam, q1.x, q1.y, x[2], z[2]);
                ground_xz(cam, q1.z, q1.w, x[3], z[3]);
                return live && !road_culled<false>(cam, x, z, b0, b1);
            },
            [&](int u) {
                if (u >= nbu) do_lights(s, sc, cam, L, u - nbu);
                else do_boxes<true>(s, sc, cam, L, u, ubox, nsv, (lptr<int32_t>)ws.tris);   // the staging is free here
            },
            [&](int a, int n) {
                setup_job<true>(s, sc, cam, L, ws, a, n, [&](int t) { road_fold(L, road, cam, ws, t, b0, b1, b0); });
            });
        if (first) {
            nbt = L.cnt[R_NBT];
            ovf = L.cnt[R_BOVF] != 0 || nsv > L.nrec;
            if (ovf) {
                kr0 = 0;
            } else if (nbt > 0) {
                kr0 = L.cnt[R_BMIN];
                kr1 = L.cnt[R_BMAX] + 1;
            }
            // streamed entries: a shorter list leaves more rows to a band of keys (300
            // crowded boxes 2,080 us; with 192 entries 1,755, with 128 1,583)
            if (ovf) L.bcap = min(L.bcap, 128);
            free_region(L, ovf ? L.bcap : nbt, W);
        }
        const int r0 = first ? 0 : b0;
        const int k0 = min(max(kr0, r0), b1), k1 = min(max(kr1, k0), b1);      // this band's box rows
        const lptr<const unsigned long long> none = (lptr<const unsigned long long>)nullptr;
        resolve_rows(s, (lptr<const uint32_t>)pal, rz, color, W, L.hr0, (lptr<const uint32_t>)road, b0, none, o, view_px, r0, k0);
        resolve_rows(s, (lptr<const uint32_t>)pal, rz, color, W, L.hr0, (lptr<const uint32_t>)road, b0, none, o, view_px, k1, b1);
        if (ovf) {
            // box keys of a few rows at a time
            for (int c0 = k0; c0 < k1; c0 += L.krows) {
                const int c1 = min(c0 + L.krows, k1);
                __syncthreads();
                for (int p = tid; p < (c1 - c0) * W; p += B) L.work[p] = 0ull;
                __syncthreads();
                stream_entries<true, false>(s, sc, cam, ego, L, L.work, c0, c1, wv, K);
                __syncthreads();
                resolve_rows(s, (lptr<const uint32_t>)pal, rz, color, W, L.hr0, (lptr<const uint32_t>)road, b0,
                             (lptr<const unsigned long long>)L.work, o, view_px, c0, c1);
            }
        } else {
            const int mrows = max(1, mask_rows_fit(L.region, nbt, W, L.nmw)), G = (W + 15) >> 4;
            for (int c0 = k0; c0 < k1; c0 += mrows) {
                const int c1 = min(c0 + mrows, k1);
                __syncthreads();
                for (int p = tid; p < L.nmw * G * (c1 - c0); p += B) L.work[p] = 0ull;
                __syncthreads();
                box_spans<true>(L, cam, nbt, c0, c1, wv, K);
                __syncthreads();
                resolve_box_rows(s, (lptr<const uint32_t>)pal, color, L, cam, (lptr<const uint32_t>)road, b0, o, view_px, c0, c1);
            }
        }
        if (b1 >= H) break;
    }
}

}  // namespace

size_t full_lds_bytes(int width, const FullCfg &c) { return full_layout(width, c).total; }

hipError_t launch_render_full(const DevSim &s, const RenderOut &o, const FullCfg &c, int ordered, int view_begin, int grid,
                              hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    if (c.waves < 1 || c.waves > 16 || s.width < 16 || c.band_rows < 1 || c.bcap < 64 || c.bcap > 256 || c.recs < 1 || c.recs > 64 || c.bins_cap < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_render_full, dim3(grid), dim3(64 * c.waves), full_lds_bytes(s.width, c), st, s, o, c, ordered,
                       view_begin);
    return hipGetLastError();
}

}  // namespace gp
