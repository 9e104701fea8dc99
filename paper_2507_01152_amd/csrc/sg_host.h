// Host-side state of the library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <memory>
#include <string>
#include <vector>

#include "sg_internal.h"
#include "sonosim.h"

namespace sg {

struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
    DevBuf() = default;
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    ~DevBuf();
    hipError_t ensure(size_t bytes);   // grow-only; synchronises the device before a regrow
};

// Pinned staging of uploads (launch parameters, poses): kStagingSlots parts of one allocation, taken in turn, so a
// call waits for the upload of kStagingSlots calls ago, not for the previous one.
constexpr int kStagingSlots = 4;
struct PinnedRing {
    void* p = nullptr;
    size_t cap = 0;                           // bytes of a slot
    hipEvent_t ev[kStagingSlots] = {};        // recorded after the last upload from each slot
    int at = 0;                               // the slot last taken
    PinnedRing() = default;
    PinnedRing(const PinnedRing&) = delete;
    PinnedRing& operator=(const PinnedRing&) = delete;
    ~PinnedRing();
    hipError_t acquire(size_t bytes, void** slot);   // the next slot, grown if need be (waits for its previous upload)
    hipError_t uploaded(hipStream_t s);              // to be called when the slot's upload is enqueued
};

struct HostVolume {
    VolDev dev{};
    uint8_t* bricks = nullptr;   // library-owned bricked label map (dev.labels); freed on release
    int32_t max_label = 0;
    bool live = false;
};

struct LaunchShape {
    int spw = 1;      // scanlines per wave in a ray item
    int tx = 64;      // PSF tile width (scanlines); tiles are 64 rows high
    int chunks = 1;   // env chunks: the PSF kernel of chunk k runs beside the ray kernel of chunk k + 1
};
constexpr int kMaxChunks = 4;

struct Plan {
    int32_t n_envs = 0;                // internal envs: one per image plane
    int32_t n_user = 0;                // caller envs (poses, volumes, probes, offsets)
    std::vector<int32_t> vol_ids;
    std::vector<sg_probe> probes;
    std::vector<int64_t> out_offsets;
    std::vector<EnvDev> envs;          // static parts
    std::vector<float> pool;
    std::vector<int> order;            // envs, longest scanlines first
    int64_t n_pixels = 0;
    int64_t n_scr = 0;                 // field-scratch elements per field (padded scanlines)
    int max_rax = 0, max_rlat = 0;
    int multiscale = 0;                // some env's volume has several noise scales
    int any_ct = 0;                    // some env's volume has a CT
    LaunchShape shape;
    int grid_ray = 0, grid_psf = 0, grid_psf_last = 0;   // (last: the last chunk's PSF kernel runs alone)
    DevBuf d_envs, d_pool, d_rays, d_tiles, d_poses, d_queue, fields;
    int32_t n_rays = 0, n_tiles = 0;
    // per chunk: ranges of the ray and PSF work lists (one queue each)
    int32_t ray_off[kMaxChunks] = {}, ray_cnt[kMaxChunks] = {}, tile_off[kMaxChunks] = {}, tile_cnt[kMaxChunks] = {};
    hipStream_t aux = nullptr;                      // second stream of the chunked pipeline
    hipEvent_t ev_ray[kMaxChunks] = {}, ev_join = nullptr;
    ~Plan();
};

}  // namespace sg

namespace sg {
struct Surrogate;   // surrogate.cpp
struct SurrogateDeleter {
    void operator()(Surrogate* p) const;
};
struct Recon;       // recon.hip
struct ReconDeleter {
    void operator()(Recon* p) const;
};
}  // namespace sg

struct sg_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int n_cu = 256;
    std::string arch;
    std::vector<sg::HostVolume> vols;
    bool vols_dirty = true;
    sg::DevBuf d_vols;
    sg::DevBuf table;
    sg::DevBuf pair_rt;   // (r, t) per label pair, when n_labels <= kPairLabels
    sg::DevBuf q_lut;     // quantised normal of the multi-scale gate (kNoiseQ int32, units of 2^-20)
    sg::DevBuf ms_thr;    // multi-scale gate thresholds, [SG_MAX_LABELS_DEV][kMaxNoiseScales] int32
    int32_t n_labels = 0;
    sg::DevBuf scan, params, fields, queue;
    sg::PinnedRing staging;
    std::map<int32_t, std::unique_ptr<sg::Plan>> plans;
    int32_t next_plan = 1;
    std::map<int32_t, std::unique_ptr<sg::Surrogate, sg::SurrogateDeleter>> surrogates;
    int32_t next_surr = 1;
    std::map<int32_t, std::unique_ptr<sg::Recon, sg::ReconDeleter>> recons;
    int32_t next_recon = 1;
    sg::DevBuf op_wt, op_parts;   // workspaces of the conv op entry points
};

namespace sg {

sg_status fail(sg_status code, const char* fmt, ...);
sg_status hip_fail(hipError_t e, const char* what);
constexpr int kPsfTapsMax = 2 * kMaxPsfRadius + 1;
int psf_taps_into(double sigma, float* out);   // no allocation
sg_status check_probe(const sg_probe& p, int idx);
// static parameters of plane `plane` of caller env idx (frame at out_off + plane * W * H)
sg_status fill_env_static(const sg_probe& p, int32_t vol, int idx, int plane, int64_t out_off, int64_t scr_off,
                          std::vector<float>& pool, EnvDev& e);
// the same without allocation: taps appended to pool[*pool_used ..) within pool_cap floats
// (SG_ERANGE when full), e.kax / e.klat as offsets into pool
sg_status fill_env_static_into(const sg_probe& p, int32_t vol, int idx, int plane, int64_t out_off, int64_t scr_off,
                               float* pool, int64_t pool_cap, int64_t* pool_used, EnvDev& e);
int probe_planes(const sg_probe& p);                 // image planes of a probe (>= 1)
double plane_elevation(const sg_probe& p, int j);   // elevation b of plane j, mm
void build_items(const std::vector<EnvDev>& envs, const std::vector<int>& order, int spw, int tx,
                 std::vector<ItemRay>& rays, std::vector<ItemPsf>& tiles);
// what the planes of a call or plan come to
struct Extent {
    int64_t scanlines = 0, tiles64 = 0, tiles32 = 0;   // PSF tiles of 64 and of 32 scanlines
    void add(int W, int H)
    {
        scanlines += W;
        tiles64 += (int64_t)((W + 63) / 64) * ((H + 63) / 64);
        tiles32 += (int64_t)((W + 31) / 32) * ((H + 63) / 64);
    }
};
// PSF tile width: 64 scanlines, which stage the smallest halo, from one frame (PSF kernel 7.8 against 8.3 us with 32) to
// 256 of 128 x 256 (34 against 39 us), unless 32 come out ahead by more than the halo costs:
//  * tiles that all fit at once, each on a compute unit of its own, with a radius past 16, where the tap loop's length
//    counts (one frame of 200 x 200, radius 24: 17.2 and 16.4 us);
//  * more tiles than fit at once, by the rounds of resident blocks (8 waves of a 64-wide block, 4 of a 32-wide one; a
//    round with more waves on a unit takes longer, 3 % each measured): frames of 32 scanlines and fewer, where half of
//    the waves of a 64-wide block have no column (256 of 24 x 256: 16.6 and 15.0 us), radii that leave one block of 64 on a
//    unit but three of 32 (256 of 256 x 256, radius 16: 180 and 140 us), widths that fill 32s better (256 of
//    200 x 200, radius 24: 220 and 194 us).  Within 10 % of each other it stays at 64 (256 of 128 x 200, radius 20: 106
//    and 105 us; 256 of 65 x 256: 30.6 and 31.5 us).
template <class Resident>   // resident(width): blocks that fit on the GPU at once
inline int psf_tile(const Extent& x, int max_rlat, int n_cu, Resident resident)
{
    const int resident64 = resident(64);
    if (resident64 < 1) return 32;
    if (max_rlat > 16 && x.tiles32 <= n_cu) return 32;
    if (x.tiles64 <= resident64) return 64;
    auto cost = [&](int64_t tiles, int at_once, int waves) {
        const double rounds = (double)tiles / at_once;
        return (rounds < 1.0 ? 1.0 : rounds) * (1.0 + 0.03 * ((double)waves * at_once / n_cu - 8.0));
    };
    return cost(x.tiles32, resident(32), 4) < 0.9 * cost(x.tiles64, resident64, 8) ? 32 : 64;
}
// launch shape of a call, and of a plan before it is tuned.  Fewer scanlines
// per ray item spread a small call over the GPU (64 frames of 128 x 256: 31, 33, 39 us of ray kernel with 4, 8,
// 16), more save item changes once every resident block (about six per compute unit) has several items (256
// volumetric probes, 12,800 items of 4: 62, 49, 47 us).
inline LaunchShape default_shape(const Extent& x, int max_rlat, int n_cu)
{
    const int64_t items = x.scanlines / kRayWaves, resident = 6 * (int64_t)n_cu;
    LaunchShape s;
    s.spw = items <= 2 * resident ? 1 : (items <= 6 * resident ? 2 : 4);
    s.tx = psf_tile(x, max_rlat, n_cu, [&](int tx) { return psf_grid(tx, max_rlat, n_cu); });
    return s;
}
sg_status sync_volumes(sg_ctx* c);
// entry point without allocation (noalloc.hip): its device scratch and limits
constexpr size_t kNoAllocBytes = SG_NOALLOC_SCRATCH_BYTES;
constexpr int kNoAllocMaxPlanes = SG_NOALLOC_MAX_PLANES;
hipError_t noalloc_init(int device);   // with `device` current; once per device (later calls return at once)

struct StageInfo {
    int tile_x = 64;
    int max_pixels = 0;
};
sg_status stage_physics(sg_ctx* c, int32_t n, const int32_t* vol_ids, const sg_probe* probes, const double* poses,
                        float* out, const int64_t* out_offsets, const sg_debug_planes* dbg, PhysArgs& a,
                        StageInfo& info);
sg_status launch_physics(sg_ctx* c, const PhysArgs& a, const StageInfo& info);
// enqueue the upload of `bytes` host bytes (host may be reused on return) to the device buffer dst
// (16-byte aligned, room for bytes rounded up to 16)
sg_status upload(sg_ctx* c, void* dst, const void* host, size_t bytes, const char* what);
sg_status check_envs(sg_ctx* c, int32_t n, const int32_t* vol_ids, const sg_probe* probes);
void surrogate_release_all(sg_ctx* c);
void recon_release_all(sg_ctx* c);

}  // namespace sg
