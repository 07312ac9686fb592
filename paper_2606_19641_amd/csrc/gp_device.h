// Device-side data layout shared by the kernels and the host runtime of the
// Gigapixel hot path.  Everything here describes memory inside the caller's
// workspace; no pointer is owned by the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gp {

constexpr int kMaxCams = 4;
constexpr int kBinQuads = 16;            // road strips per culling bin
constexpr int kMaxPrims = 1 << 23;       // primitives per scene (key packs 23 bits)
constexpr int kQueues = 8;               // work-queue segments, one per XCD of the MI355X
// Spacing of the queue's counters in 32-bit words: one counter per 256 bytes.
// Device-scope atomics on one cache line serialise (about 12 ns each on the
// MI355X), on distinct lines they proceed in parallel.
constexpr int kCtrStride = 64;

// Spacing of the scenes' view counters, a cache line each, for the same reason.
constexpr int kDoneStride = 32;

// Per-scene record.
struct SceneRec {
    int32_t agent_base, n_agents;   // agents [agent_base, agent_base + n_agents)
    int32_t road_base, n_roads;     // road slots [road_base, road_base + n_roads)
    int32_t view_base;              // first view of the scene
    int32_t bin_base, n_bins;       // culling bins [bin_base, bin_base + n_bins)
    int32_t static_base, n_static;  // static obstacles: box slots [static_base, static_base + n_static)
    int32_t signal_base, n_signals; // traffic lights [signal_base, signal_base + n_signals)
};

// Box b of a scene (the agents, then the static obstacles) -> its slot in the
// box arrays (state, cs, dims, agent_color): every agent first, then every
// static obstacle.
__host__ __device__ inline int box_slot(const SceneRec &sc, int b)
{
    return b < sc.n_agents ? sc.agent_base + b : sc.static_base + (b - sc.n_agents);
}

// One view: scene index and (ego agent local index, camera index).
struct ViewRec {
    int32_t scene;
    int32_t ego_cam;   // ego * 4 + cam
};

// All that a view's workgroup needs to start, in one cache line's half: read by
// scalar loads it saves the two dependent loads of view and scene record.
struct alignas(64) ViewInit {
    int32_t view, scene, ego, cam;
    SceneRec sc;
    int32_t pad;
};
static_assert(sizeof(ViewInit) == 64, "ViewInit layout");

// Camera constants of every view of a sim, computed once on the host with the
// operations written at their fields (binary32, round to nearest).
struct CamConst {
    float cx, cy;                             // 0.5 W, 0.5 H
    float F256, CX256, CY256, G;              // 256 f, 256 cx, 256 cy, 2^28 / F256
    float t_left, t_right, t_top, t_bottom;   // cx / f, (W - cx) / f, cy / f, (H - cy) / f
    float road_b;                             // -1 / (f (0 - cam_height)): the road plane's B; its A and C are zeros
};

// Road culling bin: bounding box of up to kBinQuads consecutive road slots.
struct RoadBin {
    float xmin, ymin, xmax, ymax;
    int32_t start, count;           // slot range, relative to the scene's road_base
    int32_t pad0, pad1;
};

// Everything a kernel needs, passed by value.
struct DevSim {
    const SceneRec *scenes;
    const ViewRec *views;
    const ViewInit *vinit;    // [V] by view
    const ViewInit *vorder;   // [V] in the order of order[]
    CamConst camk;
    float4 *state;            // [A + S] x, y, psi, v: the A agents, then the S static obstacles (v = 0)
    float2 *cs;               // [A + S] cos psi, sin psi
    const float4 *dims;       // [A + S] L, W, H, 0
    const uint8_t *agent_color;   // [A + S]
    const float4 *roads;      // [R][2] corners of road slot r: (x0 y0 x1 y1) (x2 y2 x3 y3)
    const int32_t *road_index;// [R] index of road slot r in its scene's input order
    const uint8_t *road_color;// [R] colour of road slot r
    const RoadBin *bins;
    const uint8_t *palette;   // [256*3]
    const int32_t *queue;     // [V] view order for the persistent schedule, kQueues segments
    const int32_t *order;     // [V] view of workgroup b when every view has a workgroup: consecutive
                              // workgroups (which go to the XCDs in turn) take the segments in turn
    uint32_t *counter;        // [(kQueues + 2) * kCtrStride] segment heads, finished workgroups,
                              // exhausted segment mask, kCtrStride words apart (all zero
                              // between launches)
    int32_t qseg[kQueues + 1];// segment q of the queue is [qseg[q], qseg[q + 1])
    int32_t n_scenes, n_agents, n_views;
    int32_t n_boxes;          // A + S
    int32_t width, height, n_cams;
    int32_t road_color_uniform;   // 1 if every road strip has the colour road_color0
    int32_t road_color0;
    const uint32_t *box_rgb;  // [A + S] palette colour of each box (byte 0 red)
    uint32_t road_rgb, bg_rgb;    // colours of road_color0 and of the background
    float road_zmax;          // no pixel sample sees the road plane beyond this depth
    // a render that steps the agents first (the rgb raster only; else act is null)
    const float2 *act;        // [A] actions (accel, steer)
    uint32_t *scene_done;     // [n_scenes * kDoneStride] views of each scene that have read its agents' states
                              // in this launch (zero between launches)
    uint8_t *halted;          // [A] 1 once the agent committed an infraction (frozen in place)
    uint8_t *infr;            // [A] infractions found by the last check (bit 0 collision, 1 off-road)
    float4 *actu;             // [A] jerk actuators: a_lon, a_lat, steering angle, 0
    const float4 *signals;    // [G] traffic lights: x, y, z (centre), radius
    uint8_t *signal_color;    // [G] palette index of each light's state
    float cam_dir[kMaxCams][2];
    float focal, cam_height, z_near, z_far, dt;
    float light[4];           // unit direction towards the light (world frame), ambient
    int32_t shade;            // 1: faces lit by the directional light
};

struct RenderOut {
    uint8_t *rgb;
    float *depth;
    int32_t *primid;
};

// One sim of a batched (serving) launch.
struct SimEntry {
    DevSim s;
    RenderOut o;
    const float2 *act;        // the sim's actions [n_agents] (accel, steer)
    const void *pad;
};

struct LaunchCfg {
    int band_rows;
    int batch_tris;
    int block_threads;
};

// Settings of the wave-split rgb raster (gp_raster.hip).
struct RgbCfg {
    int waves;        // wavefronts per view: 1..16
    int bcap;         // box faces and lights one view's list holds: 64..256
    int recs;         // boxes one view's records hold: 1..64
    int bins_cap;     // surviving culling bins one view's list holds (more are taken in segments): multiple of 64
                      // where it is below the bins of the largest scene
    int appear;       // 1: the instances with the directional light and traffic lights
};

// Settings of the general raster (gp_full.h).
struct FullCfg {
    int waves;        // wavefronts per view: 1..16
    int bcap;         // box faces and lights one view's list holds: 64..256
    int recs;         // boxes one view's records hold: 1..64
    int bins_cap;     // culling bins of the largest scene
    int band_rows;    // rows of the band of road keys
};

// Settings of the ray caster (gp_raycast.hip).
struct RcCfg {
    int waves;        // wavefronts per view: 1..16
    int bcap;         // boxes and lights the LDS list holds, a multiple of 64
    int bins_cap;     // surviving culling bins one view's list holds: every bin of the largest scene, or (seg) fewer
    int band_rows;    // rows of the key band (cover: at least), else of the band of road keys
    int cover;        // 1: roads as coverage bits
    int seg;          // 1: the scene's bins are taken in segments where more survive than the list holds
};

// Buffers of the chip-wide rgb raster (gp_chip.hip), all inside the
// workspace.  The coverage words and the counters are zero between renders.
enum { CHIP_NITEMS = 0, CHIP_NCTL = 8 };
struct ChipBufs {
    unsigned long long *cov;  // [V][H][nw] road coverage: bit i of word w of a row is sample 64 w + i
    int32_t *sbins;           // [V][bins_stride] surviving culling bins: start * 128 + count
    int4 *vinfo;              // [V] surviving bins, box triangles (-1: the list overflowed), box rows min, max
    void *btri;               // [V][btri_cap] the view's box triangles (TriRec)
    int4 *rinfo;              // [V] road triangles appended (may pass rtri_cap), coverage words used, 0, 0
    void *rtri;               // [V][rtri_cap] the view's road triangles (TriGeo)
    int32_t *rrows;           // [V][rtri_cap] their sample rows j0 | j1 << 16
    uint2 *items;             // road work items (view, unit of four surviving bins)
    uint32_t *ctl;            // [CHIP_NCTL] road item count (the others unused)
    int32_t bins_stride, btri_cap, rtri_cap, nw, rows_per_item, items_per_view;
};

// Host-side launch helpers (defined in gp_kernels.hip and gp_raster.hip).
hipError_t launch_step(const DevSim &s, const float *actions, int agent_begin, int agent_count,
                       hipStream_t st);
// The direct step of every agent as a graph kernel node: added to g when exec
// is null (the node returned in *node), else the arguments of *node in the
// instantiated graph exec replaced (a new action buffer, no re-capture).
hipError_t step_graph_node(hipGraph_t g, hipGraphExec_t exec, hipGraphNode_t *node, const DevSim &s,
                           const float *actions);
// clear_halted = 1 also clears the halted flags and the jerk actuators
hipError_t launch_cs(const DevSim &s, int clear_halted, hipStream_t st);
// agent states from device memory src [A][4] (4-byte aligned), a new episode
hipError_t launch_set_state(const DevSim &s, const float *src, hipStream_t st);
// dst's dynamic state from src's (same scenes, same device)
hipError_t launch_fork(const DevSim &dst, const DevSim &src, int n_signals, hipStream_t st);
// jerk-actuated step of every agent; actions [A] uint8 indices 0..11
hipError_t launch_step_jerk(const DevSim &s, const uint8_t *actions, hipStream_t st);
// infraction check of every agent; flags_out (optional) [A] gets bit 0
// collision, bit 1 off-road, bit 2 halted after the check
hipError_t launch_infractions(const DevSim &s, int max_agents, uint8_t *flags_out, hipStream_t st);
// kind 1: rgb-only kernel for a uniform road colour; 0: general kernel;
// 2: general kernel with traffic lights
hipError_t launch_render(const DevSim &s, const RenderOut &o, const LaunchCfg &c, int kind,
                         int persistent, int view_begin, int grid, hipStream_t st);
size_t render_lds_bytes(const DevSim &s, const LaunchCfg &c, int fast);
size_t render_lds_bytes(int width, int height, const LaunchCfg &c, int fast);
// ray-cast backend (gp_raycast.hip): one workgroup per view order[view_begin ..
// view_begin + n_views); c.cover: rgb only, one road colour, width >= 16
hipError_t launch_raycast(const DevSim &s, const RenderOut &o, const RcCfg &c, int view_begin, int n_views, hipStream_t st);
size_t raycast_lds_bytes(int width, int height, const RcCfg &c);
// general raster (gp_full.h): any outputs, road colours, light and traffic
// lights, width >= 16; workgroup b renders view order[b] (ordered) or view_begin + b
hipError_t launch_render_full(const DevSim &s, const RenderOut &o, const FullCfg &c, int ordered, int view_begin, int grid,
                              hipStream_t st);
size_t full_lds_bytes(int width, const FullCfg &c);
// wave-split rgb raster (gp_raster.hip) for uniform road colours, no depth /
// primitive id and width >= 16: workgroup b renders view order[b] (ordered) or
// view_begin + b
hipError_t launch_render_rgb(const DevSim &s, const RenderOut &o, const RgbCfg &c, int ordered, int view_begin,
                             int grid, hipStream_t st);
// the same over the (sim, view) items of a batch, every sim with width x height images
hipError_t launch_render_rgb_multi(const SimEntry *tab, const int2 *items, int n_items, const RgbCfg &c, int width,
                                   int height, hipStream_t st);
size_t rgb_lds_bytes(int width, int height, const RgbCfg &c);
constexpr int kFaceBytes = 64;            // LDS of one list entry
// chip-wide rgb raster (gp_chip.hip), same conditions as the wave-split one
// plus 64 <= width <= 1024: the setup pass over views [view_begin,
// view_begin + n_views) (mode 0) or every view in order[] (mode 1), the road
// pass on road_grid workgroups, the resolve pass on a workgroup per group of
// sixteen tiles of a view
hipError_t launch_render_chip(const DevSim &s, const RenderOut &o, const ChipBufs &cb, int mode, int view_begin,
                              int n_views, int road_grid, hipStream_t st);
// zero the chip-wide raster's counters and the first cov_words coverage words
hipError_t launch_chip_clear(const ChipBufs &cb, size_t cov_words, hipStream_t st);
// batched (serving) launches over a device table of sims
hipError_t launch_step_multi(const SimEntry *tab, int n_sims, int max_agents, hipStream_t st);
hipError_t launch_render_multi(const SimEntry *tab, const int2 *items, int n_items, uint32_t *ctl,
                               const LaunchCfg &c, int kind, int width, int height, int grid, hipStream_t st);

}  // namespace gp
