// integrate_frame: normals from a 5x5 plane fit, the viewing-angle filter,
// and the running weighted average of SDF and gradient, Eq. (1)-(3) of
// Gradient-SDF (Sec. 3.1, 3.2), driven by depth pixels as in the Sec. 5.3
// setup.
//
// Two kernels (the frame path runs the first together with allocation, as
// k_alloc_normals).
//  1. k_pixel_normals: one work-group per 16x16 pixel tile with its 2-pixel
//     halo staged in LDS; every pixel gets its world-frame normal and depth
//     (float4), or zeros when it fails the window or the angle test.
//  2. k_fuse_blocks: the blocks touched by the frame (the allocation step
//     counts the pixels that touch each), whole or in parts, taken by
//     work-groups that stay for the launch.  A work-group projects the
//     block's box into the image, walks its share of the pixels of that
//     rectangle, clips each pixel's ray to the box to find the few band
//     samples that can land inside, evaluates exactly those samples with the
//     binary32 band rule, and adds w d, w n_w and w into a 512-voxel
//     accumulator in LDS.  Each voxel the frame changed is then written once,
//     by one work-group (the last one done, where a block has parts), so no
//     atomics touch the map and every touched voxel costs one read and one
//     write of its record.
//
// FP32 storage keeps, per voxel, float4 {sum w d, g_x, g_y, g_z} and W:
// psi = (sum w d) / W is Eq. (1)-(2) unrolled over all observations and g
// is Eq. (3) exactly, so the write is an addition.  16-bit storage keeps
// {psi/T, gbar} (gbar = g / W, bounded) and applies Eq. (1)-(3) with the
// frame's sums before rounding once.  The gradient-free storage keeps
// {sum w d} and W only: the same distance sums as FP32 storage, without
// the three gradient sums (Eq. (3)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include <climits>

#include "gsdf_alloc.hpp"
#include "gsdf_common.hpp"
#include "gsdf_fixed.hpp"
#include "gsdf_host.hpp"

namespace gsdf {

constexpr int kTile = 16;
constexpr int kHalo = 2;
constexpr int kTileH = kTile + 2 * kHalo;
constexpr int kFuseBlock = 256;
constexpr int kFuseChunk = 1536;   // box pixels scanned per pass (LDS queue capacity)
constexpr int kScanBatch = 2;      // box pixels a thread of the scan looks at together
constexpr int kTeamGroups = 128;   // work-groups of a team: four a CU over the eight teams
constexpr int kClasses = 4;        // order of a team's pieces: parts of split blocks, then whole ones, long to short
constexpr int kPiecePixels = 1024;   // shortest part of a split block, in pixels whose band meets the block
constexpr int kSortBins = 32;      // queue entries are sorted by their number of band samples, 32 or more alike
constexpr float kBoxMargin = 1e-4f;  // metres; far above binary32 rounding of coordinates

struct FuseConsts {
    BandConsts band;
    float fxf, fyf, rcx, rcy;     // float32 intrinsics for the normal fit
    double fx_d, fy_d, ifx_d, ify_d, cx_d, cy_d;
    float zmin, zmax;
    float eps, cos_min;
    float inv_span;   // 1 / (T - eps), the slope of the linear weight
    double inv_vs_d, vs_d;
    float vs_f, T_f;
    float inv_df;   // 1 / band sample spacing
    int W, H;
    double magic;        // 1.5 * 2^(52-f): fixed-point grid of the per-frame voxel sums
    double fix_inv;      // 2^-f
};

// w(d) = 1 for d <= eps, (T - d) / (T - eps) for eps < d < T, 0 for d >= T,
// written as the clamp of the middle piece (the same function, no branches)
__device__ inline float linear_weight(float d, float T, float inv_span) {
    return fminf(1.0f, fmaxf(0.0f, (T - d) * inv_span));
}

// ---------------------------------------------------------------------------
// 1. Normals
// ---------------------------------------------------------------------------
// Tile (tu, tv) of 16x16 pixels; every thread of the 256-thread work-group
// must call it (it synchronises); tile and itile are kTileH x (kTileH + 1)
// floats of LDS (depths and their reciprocals, each computed once per tile).
__device__ inline void normals_tile(const float* __restrict__ depth, const FuseConsts& fc,
                                    const double* __restrict__ Twc, float4* __restrict__ pix, int tu, int tv,
                                    float (*tile)[kTileH + 1], float (*itile)[kTileH + 1]) {
    const int tx = threadIdx.x & (kTile - 1);
    const int ty = threadIdx.x / kTile;
    const int u0 = tu * kTile - kHalo;
    const int v0 = tv * kTile - kHalo;
    for (int i = threadIdx.x; i < kTileH * kTileH; i += blockDim.x) {
        const int ly = i / kTileH, lx = i % kTileH;
        const int uu = u0 + lx, vv = v0 + ly;
        float d = 0.0f;
        if (uu >= 0 && uu < fc.W && vv >= 0 && vv < fc.H) d = depth[(size_t)vv * fc.W + uu];
        tile[ly][lx] = d;
        itile[ly][lx] = d > 0.0f ? 1.0f / d : 0.0f;
    }
    __syncthreads();

    const int u = tu * kTile + tx;
    const int v = tv * kTile + ty;
    if (u >= fc.W || v >= fc.H) return;  // no barrier follows
    float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
    const float Dc = tile[ty + kHalo][tx + kHalo];
    if (u >= kHalo && v >= kHalo && u < fc.W - kHalo && v < fc.H - kHalo &&
        depth_ok(Dc, fc.zmin, fc.zmax)) {
        // least-squares plane 1/z = a . [x/z, y/z, 1] on the 5x5 window.
        // Over the symmetric window the design (1, du, dv) is orthogonal, so
        // the fit has a closed form in the centred inverse depths
        // 1/D_i - 1/D_c = (D_c - D_i) (1/D_c) (1/D_i), whose numerators are
        // exact (no cancellation; the reciprocals come from the tile).
        const float iDc = itile[ty + kHalo][tx + kHalo];
        float s0 = 0.0f, sa = 0.0f, sb = 0.0f;
        bool ok = true;
#pragma unroll
        for (int dv = -kHalo; dv <= kHalo; ++dv) {
#pragma unroll
            for (int du = -kHalo; du <= kHalo; ++du) {
                const float Di = tile[ty + kHalo + dv][tx + kHalo + du];
                ok = ok && depth_ok(Di, fc.zmin, fc.zmax) && (fabsf(Di - Dc) <= fc.band.Tf);
                const float dy = (Dc - Di) * iDc * itile[ty + kHalo + dv][tx + kHalo + du];
                s0 += dy;
                sa += (float)du * dy;
                sb += (float)dv * dy;
            }
        }
        if (ok) {
            const float h = iDc + s0 * (1.0f / 25.0f);
            const float alpha = sa * (1.0f / 50.0f);   // sum du^2 = 50 over the window
            const float beta = sb * (1.0f / 50.0f);
            const float ax = alpha * fc.fxf;
            const float ay = beta * fc.fyf;
            const float az = h - alpha * ((float)u - fc.rcx) - beta * ((float)v - fc.rcy);
            const float na = sqrtf(ax * ax + ay * ay + az * az);
            const float rx = ((float)u - fc.rcx) * fc.band.ifx;
            const float ry = ((float)v - fc.rcy) * fc.band.ify;
            const float ina = 1.0f / na;
            const float cosang = h * ina * __frsqrt_rn(rx * rx + ry * ry + 1.0f);
            if (cosang >= fc.cos_min) {
                // a . ray = h > 0: the normal faces away from the camera
                const float n0 = ax * ina, n1 = ay * ina, n2 = az * ina;
                float nw[3];
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    nw[i] = (float)Twc[4 * i] * n0 + (float)Twc[4 * i + 1] * n1 + (float)Twc[4 * i + 2] * n2;
                out = make_float4(nw[0], nw[1], nw[2], Dc);
            }
        }
    }
    pix[(size_t)v * fc.W + u] = out;
}

__global__ __launch_bounds__(256) void k_pixel_normals(const float* __restrict__ depth, FuseConsts fc,
                                                       const double* __restrict__ Twc,
                                                       float4* __restrict__ pix) {
    __shared__ float tile[kTileH][kTileH + 1];
    __shared__ float itile[kTileH][kTileH + 1];
    normals_tile(depth, fc, Twc, pix, blockIdx.x, blockIdx.y, tile, itile);
}

// The frame path's allocation and normals in one launch: both work on the
// same 16x16 tiles of the same depth image and pose and are independent of
// each other (allocation never reads a normal).  Work-groups with z = 0, which
// are dispatched first, take a tile's allocation, those with z = 1 its
// normals: the allocation's waits (its set in LDS, the table's entries) pass
// beside the normals' arithmetic.
__global__ __launch_bounds__(256) void k_alloc_normals(MapView M, const float* __restrict__ depth, FuseConsts fc,
                                                       const double* __restrict__ Twc, float4* __restrict__ pix,
                                                       int32_t* status) {
    __shared__ unsigned long long s_keys[kAllocSet];
    __shared__ int s_px[kAllocSet];
    __shared__ unsigned long long red[4];
    __shared__ float tile[kTileH][kTileH + 1];
    __shared__ float itile[kTileH][kTileH + 1];
    if (blockIdx.z == 0)
        allocate_tile<false>(M, depth, fc.W, fc.H, fc.zmin, fc.zmax, fc.band, Twc, status, blockIdx.x, blockIdx.y, s_keys,
                      s_px, red);
    else
        normals_tile(depth, fc, Twc, pix, blockIdx.x, blockIdx.y, tile, itile);
}

// ---------------------------------------------------------------------------
// 2. Per-block gather
// ---------------------------------------------------------------------------
struct BlockBox {
    int u0, u1, v0, v1;       // inclusive pixel rectangle (u1 < u0: empty)
    float lo[3], hi[3];       // box relative to the camera centre, with margin
    float zmin, zmax;         // camera-frame depth range of the box corners
    float inv_bw;             // 1 / rectangle width
};

// Sum over aligned groups of 16 lanes (every lane gets it).
__device__ inline unsigned long long row_sum(unsigned long long w) {
    const auto add = [&](auto move) {
        w += (unsigned long long)__double_as_longlong(move(__longlong_as_double((long long)w)));
    };
    add([](double v) { return lane_move<0xB1>(v); });
    add([](double v) { return lane_move<0x4E>(v); });
    add([](double v) { return lane_move<0x141>(v); });
    add([](double v) { return lane_move<0x140>(v); });
    return w;
}

// Called by lanes 0..7 of wave 0 together, one box corner each (on one
// lane the eight projections are a long dependent float64 chain); lane 0
// writes the result.
__device__ inline void block_box(const FuseConsts& fc, const double* __restrict__ T, int bx, int by, int bz,
                                 BlockBox* B) {
    const double t[3] = {T[3], T[7], T[11]};
    const int b[3] = {bx, by, bz};
    double lo[3], hi[3], mag = 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lo[i] = fc.vs_d * (8.0 * b[i] - 0.5);
        hi[i] = fc.vs_d * (8.0 * b[i] + 7.5);
        mag = fmax(mag, fmax(fabs(lo[i]), fabs(hi[i])) + fabs(t[i]));
    }
    // the margin stays far above the binary32 rounding of sample positions
    // (a few ulps of the coordinate magnitude)
    const double margin = kBoxMargin + 4e-6 * mag;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lo[i] -= margin;
        hi[i] += margin;
    }
    // corner c of the box: its camera-frame point and pixel; the extremes
    // over the 8 corners by moves within the 8 lanes
    double umin, umax, vmin, vmax, zlo, zhi;
    bool behind;
    {
        const int c = threadIdx.x & 7;
        const double X[3] = {(c & 1) ? hi[0] : lo[0], (c & 2) ? hi[1] : lo[1], (c & 4) ? hi[2] : lo[2]};
        double pc[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
            pc[j] = T[j] * (X[0] - t[0]) + T[4 + j] * (X[1] - t[1]) + T[8 + j] * (X[2] - t[2]);
        // reciprocal (hardware estimate and one Newton step) instead of two
        // divisions: the rectangle is widened by a pixel on each side anyway
        // (a corner behind the camera gives a meaningless value here, and
        // the whole image is used then)
        double iz = __builtin_amdgcn_rcp(pc[2]);
        iz = fma(iz, fma(-pc[2], iz, 1.0), iz);
        const double u = fc.fx_d * pc[0] * iz + fc.cx_d;
        const double v = fc.fy_d * pc[1] * iz + fc.cy_d;
        umin = umax = u;
        vmin = vmax = v;
        zlo = zhi = pc[2];
        behind = pc[2] <= 1e-6;
        const auto extremes = [&](auto move) {
            umin = fmin(umin, move(umin));
            umax = fmax(umax, move(umax));
            vmin = fmin(vmin, move(vmin));
            vmax = fmax(vmax, move(vmax));
            zlo = fmin(zlo, move(zlo));
            zhi = fmax(zhi, move(zhi));
        };
        extremes([](double x) { return lane_move<0xB1>(x); });    // lane ^ 1
        extremes([](double x) { return lane_move<0x4E>(x); });    // lane ^ 2
        extremes([](double x) { return lane_move<0x141>(x); });   // the other four of 8
        behind = __any(behind);
    }
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        B->lo[i] = (float)(lo[i] - t[i]);
        B->hi[i] = (float)(hi[i] - t[i]);
    }
    B->zmin = (float)zlo;
    B->zmax = (float)zhi;
    if (behind) {
        B->u0 = 0;
        B->u1 = fc.W - 1;
        B->v0 = 0;
        B->v1 = fc.H - 1;
        B->inv_bw = 1.0f / (float)fc.W;
        return;
    }
    // clamp in double before converting: far-off projections stay in range
    B->u0 = (int)fmin(fmax(0.0, floor(umin) - 1.0), (double)fc.W);
    B->u1 = (int)fmax(fmin((double)(fc.W - 1), ceil(umax) + 1.0), -1.0);
    B->v0 = (int)fmin(fmax(0.0, floor(vmin) - 1.0), (double)fc.H);
    B->v1 = (int)fmax(fmin((double)(fc.H - 1), ceil(vmax) + 1.0), -1.0);
    B->inv_bw = B->u1 >= B->u0 ? 1.0f / (float)(B->u1 - B->u0 + 1) : 0.0f;
}

// Per-frame voxel sums are fixed point with f fraction bits (magic_term,
// gsdf_fixed.hpp); f is chosen on the host so that the largest possible sum
// fits (see fix_bits).

__device__ inline float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ inline void store_agent(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long load_agent(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One piece of work of a fusion work-group: a whole block (n = 1) or part
// `part` of n of a split block, whose buffers start at `base`.
struct FuseItem {
    int slot;   // -1: none left
    int part, n, base;
    int bx, by, bz;
};

// What a block stands for whose band meets `pixels` pixels, at 1 / inv_target
// of them to a piece: its class (0: split into parts; then whole blocks above
// a half, above a quarter of the target, and the rest) and its pieces.
__device__ inline int piece_count(int pixels, float inv_target, int* cls) {
    const float share = (float)pixels * inv_target;
    *cls = share > 1.0f ? 0 : (share > 0.5f ? 1 : (share > 0.25f ? 2 : 3));
    return pixels <= 0 ? 0 : (share > 1.0f ? (int)fminf(ceilf(share), (float)kMaxParts) : 1);
}

// The team's t-th piece (all lanes of a wave; uniform result).  A member's
// start, every piece and every queue wait for short sums across lanes: by
// register moves instead of shuffles (LDS round trips), allocation, normals
// and fusion take 41.7 us instead of 43.9 at 213x157, 85.1 instead of 86.6 at
// 640x480, 188.9 instead of 190.8 at 1280x720.  pre[c][i]:
// pieces of class c in the spans before span i; a span is `chunks` of the
// team's chunks of 64 slots.
__device__ inline FuseItem find_item(const MapView& M, int team, int chunks, float inv_target, const int (*pre)[65],
                                     int t) {
    FuseItem it;
    it.slot = -1;
    it.part = it.base = it.bx = it.by = it.bz = 0;
    it.n = 1;
    const int lane = threadIdx.x & 63;
    int cls = 0;
    for (; cls < kClasses && t >= pre[cls][64]; ++cls) t -= pre[cls][64];
    if (cls == kClasses) return it;
    const int rank = t;
    const int span = __ffsll((long long)__ballot(pre[cls][lane] <= t && t < pre[cls][lane + 1])) - 1;
    t -= pre[cls][span];
#pragma unroll 1
    for (int j = span * chunks;; ++j) {   // the counted pieces are there: the loop ends in the span
        const int slot = (j * kFuseTeams + team) * 64 + lane;
        int own;
        const int pieces = piece_count(M.touched[slot], inv_target, &own);
        const int w = own == cls ? pieces : 0;
        int incl = w;
        if (cls == 0) {
            incl = wave_scan(w);
        } else {
            const unsigned long long m = __ballot(w != 0);
            incl = __popcll(m & (~0ull >> (63 - lane)));
        }
        const int all = __builtin_amdgcn_readlane(incl, 63);
        if (t >= all) {
            t -= all;
            continue;
        }
        const int src = __ffsll((long long)__ballot(t < incl)) - 1;
        it.slot = __builtin_amdgcn_readlane(slot, src);
        if (cls == 0) {
            it.n = __builtin_amdgcn_readlane(w, src);
            it.part = t - (__builtin_amdgcn_readlane(incl, src) - it.n);
            it.base = rank - it.part;
        }
        unpack_key(M.block_keys[it.slot], &it.bx, &it.by, &it.bz);
        return it;
    }
}

// Fusion of the touched blocks.  kFuseTeams x kTeamGroups work-groups stay
// for the whole launch; a team's members take its pieces by ticket, the
// longest first.  Wave 0 finds the next piece and its box before it joins the
// current one, whose steps the waves take in turn, so the chain of dependent
// loads (ticket, counts, key) and the box are off the others' path.  The last
// member to find nothing clears the team's counts and counters: every member
// has read them by then.
//
// What bounds it: a piece of 360 queue entries takes 17 us with four
// work-groups on a CU, about half of it waiting (pixel loads, queue, barriers,
// voxel loads) and half VALU issue, which is why pieces are many, even and
// started longest first.  One work-group per block in slot order, dispatched by
// the hardware, spent 4.3 us of its 20 on loading what it needs and on its
// counters and 3 us on each slot without work, and where surfaces are near
// the camera a few blocks ran long after the rest.  Event times, three views
// each: 640x480 FP32 139 / 79 / 87 -> 75 / 66 / 67 us; 1280x720 BF16
// 238 / 185 / 199 -> 153 / 149 / 148 us.  Small frames gain the least (the 5 us
// in which the members count the team's pieces show there), and lose where
// parts are short: a part stores, waits for and adds 20 KB of sums.  With
// kPiecePixels of 256, 512, 1024, 2048 the frame call takes 43.5, 36.7, 36.3,
// 37.0 us at 160x120 and 42.6, 40.8, 36.6, 38.0 at 213x157 without gradients
// (38.4 and 43.1 with one work-group to a block), and with a plane at 0.45 m
// 77, 68, 62, 70 at 160x120 and 60, 62, 54, 62 at 213x157 (127 and 183); from
// 640x480 on the four are alike, as a member's share is larger.  Sorting the queue by the number of samples:
// 640x480 137 / 90 / 98 -> 110 / 80 / 89 us before the pieces were even.
template <int STORAGE>
__global__ __launch_bounds__(kFuseBlock, 4) void k_fuse_blocks(MapView M, const float4* __restrict__ pix,
                                                              FuseConsts fc, const double* __restrict__ Twc,
                                                              unsigned long long* __restrict__ parts,
                                                              int32_t* status) {
    // per-voxel sums of the frame in fixed point (see magic_term), indexed
    // lx + 8 ly + 64 lz (the pool's Morton order is applied at the write):
    // integer additions are associative, so the sums (and the map) do not
    // depend on the order in which the work-group's threads add their updates
    constexpr bool kGrad = STORAGE != GSDF_NOGRAD_FP32;
    __shared__ unsigned long long aS[kBlockVoxels];
    __shared__ unsigned long long aG[kGrad ? 3 : 1][kGrad ? kBlockVoxels : 1];
    __shared__ unsigned long long aW[kBlockVoxels];
    __shared__ BlockBox s_box[2];
    __shared__ FuseItem s_item[2];
    __shared__ uint32_t q_pix[kFuseChunk];
    __shared__ uint32_t q_k[kFuseChunk];
    __shared__ uint16_t q_order[kFuseChunk];   // entries, the most band samples first
    __shared__ int q_count[3];   // entries; steps of the scan and rows of the update phase that waves have taken
    __shared__ int s_bin[kSortBins];
    __shared__ int s_last, s_done;
    __shared__ double s_c[18];
    __shared__ int s_pre[kClasses][65];
    __shared__ int s_sum[kFuseBlock / 64];

    if (!pose_finite(Twc)) {   // nothing is fused at a non-finite pose
        if (blockIdx.x == 0 && threadIdx.x == 0) raise_status(status, GSDF_EINVAL);
        return;
    }
    const int team = blockIdx.x % kFuseTeams;
    int32_t* ticket = &M.counters[kTeamTicket + team * 16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the team's pieces per span of chunks: 16 threads take a chunk, four
    // slots each.  The first chunks' counts are loaded before the number of
    // blocks is known (unused slots count nothing)
    constexpr int kPerStep = kFuseBlock / 16;   // chunks taken together
    const int my_chunk = threadIdx.x >> 4, my_sub = threadIdx.x & 15;
    const auto counts_of = [&](int j) {
        return *reinterpret_cast<const int4*>(M.touched + (j * kFuseTeams + team) * 64 + my_sub * 4);
    };
    int4 ahead = make_int4(0, 0, 0, 0);
    if ((my_chunk + 1) * 64 * kFuseTeams <= (int)touched_slots(M.max_blocks)) ahead = counts_of(my_chunk);
    int n_blocks = M.counters[kNumBlocks];
    n_blocks = n_blocks < M.max_blocks ? n_blocks : M.max_blocks;
    const int team_chunks = (n_blocks + 64 * kFuseTeams - 1) / (64 * kFuseTeams);
    const int chunks = (team_chunks + 63) / 64;
    for (int c = threadIdx.x; c < kBlockVoxels; c += kFuseBlock) {
        aS[c] = aW[c] = 0ull;
        if constexpr (kGrad) aG[0][c] = aG[1][c] = aG[2][c] = 0ull;
    }
    for (int i = threadIdx.x; i < kClasses * 65; i += kFuseBlock) (&s_pre[0][0])[i] = 0;
    // pixels to a piece: the share of a member, so that a frame whose blocks
    // are few or uneven still fills the chip
    // (a sum that wrapped, above some fifty megapixels, gives other pieces and
    // the same result)
    int sum = ahead.x + ahead.y + ahead.z + ahead.w;
#pragma unroll 1
    for (int j = my_chunk + kPerStep; j < team_chunks; j += kPerStep) {
        const int4 v = counts_of(j);
        sum += v.x + v.y + v.z + v.w;
    }
    sum = wave_scan(sum);
    if (lane == 63) s_sum[wave] = sum;
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int w = 0; w < kFuseBlock / 64; ++w) sum += s_sum[w];
    const float inv_target = 1.0f / fmaxf((float)kPiecePixels, (float)sum * (1.0f / kTeamGroups));
#pragma unroll 1
    for (int j = my_chunk; j < team_chunks; j += kPerStep) {
        const int4 v = j == my_chunk ? ahead : counts_of(j);
        const int px[4] = {v.x, v.y, v.z, v.w};
        unsigned long long w = 0;   // 16 bits a class (at most 512 pieces a chunk)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int cls;
            const int pieces = piece_count(px[k], inv_target, &cls);
            w += (unsigned long long)pieces << (16 * cls);
        }
        w = row_sum(w);
        if (my_sub < kClasses) atomicAdd(&s_pre[my_sub][j / chunks + 1], (int)((w >> (16 * my_sub)) & 0xffffu));
    }
    // what the set-up of a queue entry takes in float64: kept in LDS, since
    // the scalar registers do not hold it beside the loops' own constants
    if (threadIdx.x < 12) s_c[threadIdx.x] = Twc[threadIdx.x];
    if (threadIdx.x == 12) {
        s_c[12] = fc.cx_d;
        s_c[13] = fc.ifx_d;
        s_c[14] = fc.cy_d;
        s_c[15] = fc.ify_d;
        s_c[16] = fc.inv_vs_d;
        s_c[17] = fc.vs_d;
    }
    unsigned long long neg_magic = 0ull - double_bits(fc.magic);
    asm("" : "+s"(neg_magic));
    BandRule br = make_band_rule(Twc, fc.band.ifx, fc.band.ify, fc.band.cxf, fc.band.cyf,
                                 fc.band.invvs, fc.band.Tf, fc.band.Df, fc.band.nsamples);
    // the float pose in scalar registers (a conversion leaves it in vector
    // registers, of which the sample loop has none to spare)
#pragma unroll
    for (int i = 0; i < 9; ++i) br.R[i] = uniform(br.R[i]);
#pragma unroll
    for (int i = 0; i < 3; ++i) br.t[i] = uniform(br.t[i]);
    float inv_span = fc.inv_span;
    asm("" : "+v"(inv_span));   // held, not loaded in the sample loop
    unsigned my_updates = 0, my_visits = 0, my_voxels = 0, my_blocks = 0;
    __syncthreads();
    static_assert(kClasses <= kFuseBlock / 64, "a wave sums a class");
    if (wave < kClasses) {
        s_pre[wave][lane + 1] = wave_scan(s_pre[wave][lane + 1]);
    }
    if (wave == 0) {
        if (lane < 3) q_count[lane] = 0;
        if (lane < kSortBins) s_bin[lane] = 0;
        if (lane == 0) s_item[0].slot = -2;   // nothing yet: the first round only finds the first piece
    }
    __syncthreads();
    for (int cur = 0;; cur ^= 1) {
        const FuseItem item = s_item[cur];
        if (item.slot == -1) break;
        if (wave == 0) {
            // the next piece and its box: a member's first piece goes by its
            // number (128 tickets at once take 5.6 us on one address)
            int t = blockIdx.x / kFuseTeams;
            if (item.slot != -2 && lane == 0)
                t = kTeamGroups + __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const FuseItem next = find_item(M, team, chunks, inv_target, s_pre, __builtin_amdgcn_readfirstlane(t));
            if (lane == 0) {
                s_item[cur ^ 1] = next;
                // nothing left: this member has read the counts it needs
                if (next.slot < 0)
                    s_done = __hip_atomic_fetch_add(&M.counters[kTeamDone + team * 16], 1, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
            }
            if (next.slot >= 0 && lane < 8) block_box(fc, Twc, next.bx, next.by, next.bz, &s_box[cur ^ 1]);
        }
        if (item.slot == -2) {
            __syncthreads();
            continue;
        }
        const BlockBox& box = s_box[cur];
        const int slot = item.slot, bx = item.bx, by = item.by, bz = item.bz;
        // without room for its partial sums a split block's first part takes
        // all of it
        const bool room = parts && item.base + item.n <= kTeamBuffers;
        const int n_parts = room ? item.n : 1;
        const int part = item.part;
        const int bw = box.u1 - box.u0 + 1;
        const int bh = box.v1 - box.v0 + 1;
        const int box_px = (bw > 0 && bh > 0) ? bw * bh : 0;
        const int px0 = part < n_parts ? (int)((int64_t)box_px * part / n_parts) : 0;   // this part's pixels of the box
        const int px1 = part < n_parts ? (int)((int64_t)box_px * (part + 1) / n_parts) : 0;
        const float inv_bw = box.inv_bw;
        // the depth band [D - T, D + T] must reach the box's depth range
        const float zreach_lo = box.zmin - fc.band.Tf - fc.band.Df;
        const float zreach_hi = box.zmax + fc.band.Tf + fc.band.Df;
        const float last = (float)(fc.band.nsamples - 1);
        const float inv_df = fc.inv_df;

        // The box is gathered in chunks of kFuseChunk pixels, each in two
        // phases.  Scan: every thread tests pixels of the chunk against the
        // block (depth reach, ray/box slab, band samples inside) and the
        // survivors go to an LDS queue with their sample range.  Fuse: the
        // queue is worked densely, so the sample loop and the LDS atomics run
        // with most lanes busy (a thread-per-pixel loop over the box leaves
        // three lanes in four idle).
#pragma unroll 1
        for (int c0 = px0; c0 < px1; c0 += kFuseChunk) {
            const int cn = min(kFuseChunk, px1 - c0);
            if (c0 > px0) {   // the first chunk finds them cleared
                if (threadIdx.x < 3) q_count[threadIdx.x] = 0;
                if (threadIdx.x < kSortBins) s_bin[threadIdx.x] = 0;
                __syncthreads();
            }
            // kScanBatch pixels a thread, their loads in flight together
            for (;;) {
                int step = 0;
                if (lane == 0) step = atomicAdd(&q_count[1], 1);
                const int p0 = __builtin_amdgcn_readfirstlane(step) * (64 * kScanBatch);
                if (p0 >= cn) break;
                uint32_t uv[kScanBatch], kk[kScanBatch];
                float Dp[kScanBatch];
#pragma unroll
                for (int j = 0; j < kScanBatch; ++j) {
                    const int p = p0 + j * 64 + lane;
                    const int q = c0 + p;
                    // row and column without an integer division (q < 2^24 is exact)
                    int row = (int)(((float)q + 0.5f) * inv_bw);
                    int col = q - row * bw;
                    if (col < 0) {
                        --row;
                        col += bw;
                    } else if (col >= bw) {
                        ++row;
                        col -= bw;
                    }
                    const int u = box.u0 + col, v = box.v0 + row;
                    uv[j] = ((uint32_t)v << 16) | (uint32_t)u;   // u, v < 2^16
                    Dp[j] = p < cn ? pix[(size_t)v * fc.W + u].w : 0.0f;
                }
                unsigned long long sel[kScanBatch];   // lanes whose pixel is kept
                int total = 0;
#pragma unroll
                for (int j = 0; j < kScanBatch; ++j) {
                    const float D = Dp[j];
                    bool keep = D > 0.0f && D >= zreach_lo && D <= zreach_hi;
                    int k0 = 0, k1 = -1;
                    if (keep) {
                        ++my_visits;
                        // clip the pixel's ray z * (R ray) to the block's box (the
                        // box's margin absorbs the approximate reciprocals)
                        const float xr = pixel_xr(br, (int)(uv[j] & 0xffffu));
                        const float yr = pixel_yr(br, (int)(uv[j] >> 16));
                        float zin = 0.0f, zout = 3.0e38f;
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            const float dir = br.R[3 * i] * xr + br.R[3 * i + 1] * yr + br.R[3 * i + 2];
                            if (fabsf(dir) < 1e-20f) {
                                if (box.lo[i] > 0.0f || box.hi[i] < 0.0f) zout = -1.0f;
                            } else {
                                const float id = __builtin_amdgcn_rcpf(dir);
                                const float a = box.lo[i] * id, b = box.hi[i] * id;
                                zin = fmaxf(zin, fminf(a, b));
                                zout = fminf(zout, fmaxf(a, b));
                            }
                        }
                        // samples inside the box widened by kBoxMargin: no other
                        // sample can land in a voxel of this block (binary32
                        // rounding of a sample's position is far below the
                        // margin), so the run structure of the consecutive-repeat
                        // rule inside the block is the same as over the whole band
                        const float zb0 = D - fc.band.Tf;  // first band sample
                        keep = zin <= zout;
                        if (keep) {
                            k0 = (int)fmaxf(0.0f, ceilf(fminf((zin - zb0) * inv_df, last + 1.0f)));
                            k1 = (int)fminf(last, floorf(fmaxf((zout - zb0) * inv_df, -1.0f)));
                            keep = k0 <= k1;
                        }
                    }
                    kk[j] = (uint32_t)(k0 | (k1 << 16));
                    sel[j] = __ballot(keep);
                    total += __popcll(sel[j]);
                }
                // compaction into the queue, one reservation a wave
                int base = 0;
                if (lane == 0) base = atomicAdd(&q_count[0], total);
                base = __builtin_amdgcn_readfirstlane(base);
                const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
                for (int j = 0; j < kScanBatch; ++j) {
                    if ((sel[j] >> lane) & 1ull) {
                        const int e = base + __popcll(sel[j] & below);
                        q_pix[e] = uv[j];
                        q_k[e] = kk[j];
                    }
                    base += __popcll(sel[j]);
                }
            }
            __syncthreads();
            // Sort the entries by their number of samples, the longest
            // first, so that a wave's sample loop runs entries of one length
            // (in two classes, up to 8 samples and longer, half of its lanes
            // idled: 84 against 47 steps of the loop per block at 640x480).
            // The lanes of a wave take entries n/64 apart (different rows of
            // the box), so lanes that follow each other in a bin, whose LDS
            // atomics share an instruction, rarely hit the same voxel.
            const int nq = q_count[0];
            const int apart = (nq + 63) / 64;
            int bin_rank[kFuseChunk / kFuseBlock];
#pragma unroll
            for (int j = 0; j < kFuseChunk / kFuseBlock; ++j) {
                const int i = lane * apart + wave + j * (kFuseBlock / 64);
                bin_rank[j] = -1;
                if (wave + j * (kFuseBlock / 64) < apart && i < nq) {
                    const uint32_t k = q_k[i];
                    const int bin = kSortBins - min((int)(k >> 16) - (int)(k & 0xffffu) + 1, kSortBins);
                    bin_rank[j] = (bin << 16) | atomicAdd(&s_bin[bin], 1);
                }
            }
            __syncthreads();
            {
                int start = lane < kSortBins ? s_bin[lane] : 0;   // exclusive sums, in every wave
                const int own = start;
                start = wave_scan(start) - own;
#pragma unroll
                for (int j = 0; j < kFuseChunk / kFuseBlock; ++j) {
                    const int to = __shfl(start, (bin_rank[j] >> 16) & (kSortBins - 1)) + (bin_rank[j] & 0xffff);
                    if (bin_rank[j] >= 0) q_order[to] = (uint16_t)(lane * apart + wave + j * (kFuseBlock / 64));
                }
            }
            __syncthreads();
            for (;;) {
                int row = 0;
                if (lane == 0) row = atomicAdd(&q_count[2], 1);
                row = __builtin_amdgcn_readfirstlane(row);
                if (row >= apart) break;
                if (row * 64 + lane >= nq) continue;
                const int e = q_order[row * 64 + lane];
                const uint32_t uv = q_pix[e];
                int k0 = (int)(q_k[e] & 0xffffu);
                const int k1 = (int)(q_k[e] >> 16);
                const int v = (int)(uv >> 16);
                const int u = (int)(uv & 0xffffu);
                const float4 px = pix[(size_t)v * fc.W + u];
                const float D = px.w;
                const float xr = pixel_xr(br, u);
                const float yr = pixel_yr(br, v);
                // observed point as an offset from a nearby voxel: formed in
                // float64 for FP32 storage; camera-relative float32 for 16-bit
                // storage (q - v_s m_c = R x + t_r, |t_r| < v_s).  The
                // constants are read from LDS here, at an offset the
                // compiler cannot see through (it would keep all of them in
                // registers over the sample loop).
                int at = 0;
                asm("" : "+v"(at));
                const double* C = s_c + at;
                int mref[3];
                float prel[3];
                if (STORAGE == GSDF_FP32 || STORAGE == GSDF_NOGRAD_FP32) {
                    const double Dd = (double)D;
                    const double x0 = Dd * (((double)u - C[12]) * C[13]);
                    const double x1 = Dd * (((double)v - C[14]) * C[15]);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const double q = C[4 * i] * x0 + C[4 * i + 1] * x1 + C[4 * i + 2] * Dd + C[4 * i + 3];
                        mref[i] = (int)floor(q * C[16] + 0.5);
                        prel[i] = (float)(q - C[17] * (double)mref[i]);
                    }
                } else {
                    const float x0 = D * (((float)u - fc.rcx) / fc.fxf);
                    const float x1 = D * (((float)v - fc.rcy) / fc.fyf);
                    const float ivsf = (float)C[16];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const int mc = (int)floor(C[4 * i + 3] * C[16] + 0.5);
                        const float trf = (float)(C[4 * i + 3] - C[17] * (double)mc);
                        const float qc = br.R[3 * i] * x0 + br.R[3 * i + 1] * x1 + br.R[3 * i + 2] * D + trf;
                        const int dm = (int)floorf(qc * ivsf + 0.5f);
                        mref[i] = mc + dm;
                        prel[i] = qc - fc.vs_f * (float)dm;
                    }
                }
                const double n0 = (double)px.x, n1 = (double)px.y, n2 = (double)px.z;
                // samples at or behind the camera (only where D <= T) do not
                // count; z grows with k
                const float z0 = sub_rn(D, br.Tf);
                if (!(z0 > 0.0f)) {
#pragma unroll 1
                    while (k0 <= k1 && !(add_rn(z0, mul_rn((float)k0, br.Df)) > 0.0f)) ++k0;
                }
                float kf = (float)k0;
                int prev = INT_MAX;
#pragma unroll 1
                for (int k = k0; k <= k1; ++k, kf += 1.0f) {
                    // the sample's voxel (band_sample's rule), relative to the
                    // block's first; within the entry's range of samples it
                    // lies at most a voxel or two outside the block
                    int m[3], c[3];
                    const float z = add_rn(z0, mul_rn(kf, br.Df));
                    const float X = mul_rn(z, xr), Y = mul_rn(z, yr);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const float q = add_rn(add_rn(add_rn(mul_rn(br.R[3 * i], X), mul_rn(br.R[3 * i + 1], Y)),
                                                      mul_rn(br.R[3 * i + 2], z)),
                                               br.t[i]);
                        m[i] = floor_int(add_rn(mul_rn(q, br.invvs), 0.5f));
                    }
                    c[0] = m[0] - 8 * bx;
                    c[1] = m[1] - 8 * by;
                    c[2] = m[2] - 8 * bz;
                    const int packed = c[0] + (c[1] << 10) + (c[2] << 20);
                    const bool take = packed != prev && (unsigned)(c[0] | c[1] | c[2]) < 8u;
                    prev = packed;
                    if (!take) continue;
                    float off[3];
#pragma unroll
                    for (int i = 0; i < 3; ++i) off[i] = fc.vs_f * (float)(m[i] - mref[i]) - prel[i];
                    float d = px.x * off[0] + px.y * off[1] + px.z * off[2];
                    d = __builtin_amdgcn_fmed3f(d, -fc.T_f, fc.T_f);
                    const float w = linear_weight(d, fc.T_f, inv_span);
                    if (!(w > 0.0f)) continue;
                    const int at_c = (((c[2] << 3) | c[1]) << 3) | c[0];
                    const double wd = (double)w;
                    atomicAdd(&aS[at_c], magic_term(fma(wd, (double)d, fc.magic), neg_magic));
                    if constexpr (kGrad) {
                        atomicAdd(&aG[0][at_c], magic_term(fma(wd, n0, fc.magic), neg_magic));
                        atomicAdd(&aG[1][at_c], magic_term(fma(wd, n1, fc.magic), neg_magic));
                        atomicAdd(&aG[2][at_c], magic_term(fma(wd, n2, fc.magic), neg_magic));
                    }
                    atomicAdd(&aW[at_c], magic_term(wd + fc.magic, neg_magic));
                    ++my_updates;
                }
            }
            __syncthreads();
        }

        bool write = part < n_parts;
        if (n_parts > 1) {
            // the part's sums (integers, so the order in which parts are
            // added does not matter) to its buffer; the last part to finish
            // adds the others' and writes the block.  Device-scope stores
            // that have completed before the ticket, device-scope loads
            // after it (parts run on any XCD).
            constexpr int kArr = kGrad ? 5 : 2;
            constexpr size_t kBuf = (size_t)kArr * kBlockVoxels;
            unsigned long long* first = parts + (size_t)(team * kTeamBuffers + item.base) * kBuf;
            unsigned long long* mine = first + part * kBuf;
            for (int c = threadIdx.x; c < kBlockVoxels; c += kFuseBlock) {
                store_agent(&mine[c], aS[c]);
                store_agent(&mine[kBlockVoxels + c], aW[c]);
                if constexpr (kGrad) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) store_agent(&mine[(2 + i) * kBlockVoxels + c], aG[i][c]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // the stores stay above
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            int32_t* done = &M.split_done[team * kTeamBuffers + item.base];
            if (threadIdx.x == 0)
                s_last = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_parts - 1;
            __syncthreads();
            write = s_last != 0;
#pragma unroll 1
            for (int q = 0; write && q < n_parts; ++q) {
                if (q == part) continue;
                const unsigned long long* other = first + q * kBuf;
#pragma unroll
                for (int c = threadIdx.x; c < kBlockVoxels; c += kFuseBlock) {
                    aS[c] += load_agent(&other[c]);
                    aW[c] += load_agent(&other[kBlockVoxels + c]);
                    if constexpr (kGrad) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) aG[i][c] += load_agent(&other[(2 + i) * kBlockVoxels + c]);
                    }
                }
            }
            if (write && threadIdx.x == 0) __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (write && threadIdx.x == 0) ++my_blocks;

        // write the voxels this frame changed: this work-group owns the block.
        // A thread reads all of its voxels before it writes any, so their
        // loads are in flight together.
        constexpr int kPerThread = kBlockVoxels / kFuseBlock;
        static_assert(kBlockVoxels % kFuseBlock == 0, "every thread writes the same number of voxels");
        float sw[kPerThread], sS[kPerThread], sG[kPerThread][3], Wold[kPerThread], d1[kPerThread];
        int64_t vi[kPerThread];
        bool on[kPerThread];
        float4 r32[kPerThread];
        ushort4 r16[kPerThread];
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int c = threadIdx.x + j * kFuseBlock;
            // every element is set in every round (one left as it was would
            // hold its registers over the whole piece)
            sS[j] = sG[j][0] = sG[j][1] = sG[j][2] = Wold[j] = d1[j] = 0.0f;
            vi[j] = 0;
            r32[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            r16[j] = make_ushort4(0, 0, 0, 0);
            sw[j] = from_fixed(aW[c], fc.fix_inv);
            on[j] = write && sw[j] > 0.0f;
            if (!on[j]) continue;
            sS[j] = from_fixed(aS[c], fc.fix_inv);
            vi[j] = (int64_t)slot * kBlockVoxels + morton9(c & 7, (c >> 3) & 7, c >> 6);
            if constexpr (kGrad) {
#pragma unroll
                for (int i = 0; i < 3; ++i) sG[j][i] = from_fixed(aG[i][c], fc.fix_inv);
            }
            if constexpr (!kGrad)
                d1[j] = reinterpret_cast<const float*>(M.vox)[vi[j]];
            else if (STORAGE == GSDF_FP32)
                r32[j] = reinterpret_cast<const float4*>(M.vox)[vi[j]];
            else
                r16[j] = reinterpret_cast<const ushort4*>(M.vox)[vi[j]];
            Wold[j] = M.weight[vi[j]];
        }
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            if (!on[j]) continue;
            ++my_voxels;
            if constexpr (!kGrad) {
                reinterpret_cast<float*>(M.vox)[vi[j]] = d1[j] + sS[j];
                M.weight[vi[j]] = Wold[j] + sw[j];
                continue;
            }
            if (STORAGE == GSDF_FP32) {
                float4 r = r32[j];
                r.x += sS[j];
                r.y += sG[j][0];
                r.z += sG[j][1];
                r.w += sG[j][2];
                reinterpret_cast<float4*>(M.vox)[vi[j]] = r;
                M.weight[vi[j]] = Wold[j] + sw[j];
            } else {
                const ushort4 p = r16[j];
                const float Wn = Wold[j] + sw[j];
                const float psi = (Wold[j] * unpack16(p.x, STORAGE) * M.truncation + sS[j]) / Wn;
                const float g0 = (Wold[j] * unpack16(p.y, STORAGE) + sG[j][0]) / Wn;
                const float g1 = (Wold[j] * unpack16(p.z, STORAGE) + sG[j][1]) / Wn;
                const float g2 = (Wold[j] * unpack16(p.w, STORAGE) + sG[j][2]) / Wn;
                reinterpret_cast<ushort4*>(M.vox)[vi[j]] =
                    make_ushort4(pack16(psi / M.truncation, STORAGE), pack16(g0, STORAGE), pack16(g1, STORAGE),
                                 pack16(g2, STORAGE));
                M.weight[vi[j]] = Wn;
            }
        }
        // the sums and counters back to zero for the next piece
        if (threadIdx.x < 3) q_count[threadIdx.x] = 0;
        if (threadIdx.x < kSortBins) s_bin[threadIdx.x] = 0;
        for (int c = threadIdx.x; c < kBlockVoxels; c += kFuseBlock) {
            aS[c] = aW[c] = 0ull;
            if constexpr (kGrad) aG[0][c] = aG[1][c] = aG[2][c] = 0ull;
        }
        __syncthreads();
    }

    // the last member to find nothing clears the team's counts and counters
    if (s_done == kTeamGroups - 1) {
#pragma unroll 1
        for (int j = wave; j < team_chunks; j += kFuseBlock / 64)
            M.touched[(j * kFuseTeams + team) * 64 + lane] = 0;
        if (threadIdx.x == 0) {
            if (team == 0) M.counters[kPending] = 0;   // (no other member reads it)
            __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&M.counters[kTeamDone + team * 16], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // work counters: one striped atomic per wave and counter
    const unsigned long long sums[3] = {wave_sum_u64(my_updates), wave_sum_u64(my_visits), wave_sum_u64(my_voxels)};
    if (lane == 0) {
        add_stat(M, kStatUpdates, sums[0]);
        add_stat(M, kStatPixelVisits, sums[1]);
        add_stat(M, kStatFusedVoxels, sums[2]);
        add_stat(M, kStatFusedBlocks, my_blocks);
    }
}

// Fraction bits of the fixed-point voxel sums.  A pixel's band meets a voxel
// at most once and contributes |w d| <= T, |w n| <= 1, w <= 1.  A term must
// stay below 2^51 units (magic_term), and a frame's sum, bounded by
// max(1, T) times the pixels whose rays can cross the voxel (its footprint,
// at most (f v_s sqrt(3) / z + 2)^2 pixels at the nearest depth
// z = max(zmin - T, v_s) a voxel of the band can have), below 2^62.
inline int fix_bits(const gsdf_camera& cam, double vs, double T) {
    const double z = std::max((double)cam.zmin - T, vs);
    const double side = std::max(cam.fx, cam.fy) * vs * std::sqrt(3.0) / z + 2.0;
    const double term = std::max(1.0, T);
    const int f = (int)std::floor(std::min(62.0 - std::log2(side * side * term), 50.0 - std::log2(term)));
    return std::max(24, f);
}

inline FuseConsts fuse_consts(const gsdf_map& map, const gsdf_camera& cam, const gsdf_fuse_params& p) {
    FuseConsts fc;
    fc.band = band_consts(cam, map.desc.voxel_size, map.desc.truncation);
    fc.fxf = (float)cam.fx;
    fc.fyf = (float)cam.fy;
    fc.rcx = (float)cam.cx;
    fc.rcy = (float)cam.cy;
    fc.fx_d = cam.fx;
    fc.fy_d = cam.fy;
    fc.ifx_d = 1.0 / cam.fx;
    fc.ify_d = 1.0 / cam.fy;
    fc.cx_d = cam.cx;
    fc.cy_d = cam.cy;
    fc.zmin = cam.zmin;
    fc.zmax = cam.zmax;
    fc.eps = p.eps_weight;
    fc.inv_span = (float)(1.0 / (map.desc.truncation - (double)p.eps_weight));
    fc.cos_min = p.cos_max_angle;
    fc.inv_vs_d = 1.0 / map.desc.voxel_size;
    fc.vs_d = map.desc.voxel_size;
    fc.vs_f = (float)map.desc.voxel_size;
    fc.T_f = (float)map.desc.truncation;
    fc.inv_df = (float)(2.0 / map.desc.voxel_size);
    fc.W = cam.width;
    fc.H = cam.height;
    const int f = fix_bits(cam, map.desc.voxel_size, map.desc.truncation);
    fc.magic = magic_of(f);
    fc.fix_inv = std::ldexp(1.0, -f);
    return fc;
}

// Scratch of the fusion calls: {n_w, D} per pixel, then the partial sums of
// the parts of split blocks (40 MiB whatever the camera: the most parts that a
// frame can have).  A caller that brings the pixels' share alone has every
// block fused whole.
inline size_t pix_bytes(const gsdf_camera& cam) { return align256((size_t)cam.width * cam.height * sizeof(float4)); }
constexpr size_t kPartsBytes =
    (size_t)kFuseTeams * kTeamBuffers * 5 * kBlockVoxels * sizeof(unsigned long long);

inline void launch_fuse_blocks(const gsdf_map& map, const gsdf_camera& cam, hipStream_t s, const MapView& M,
                               void* scratch, size_t scratch_bytes, const FuseConsts& fc, const double* Twc,
                               int32_t* status) {
    const float4* pix = (const float4*)scratch;
    unsigned long long* parts = scratch_bytes >= pix_bytes(cam) + kPartsBytes
                                    ? (unsigned long long*)((char*)scratch + pix_bytes(cam))
                                    : nullptr;
    const dim3 grid(kFuseTeams * kTeamGroups);
    switch (map.desc.storage) {
        case GSDF_FP32: k_fuse_blocks<GSDF_FP32><<<grid, kFuseBlock, 0, s>>>(M, pix, fc, Twc, parts, status); break;
        case GSDF_BF16: k_fuse_blocks<GSDF_BF16><<<grid, kFuseBlock, 0, s>>>(M, pix, fc, Twc, parts, status); break;
        case GSDF_FP16: k_fuse_blocks<GSDF_FP16><<<grid, kFuseBlock, 0, s>>>(M, pix, fc, Twc, parts, status); break;
        default: k_fuse_blocks<GSDF_NOGRAD_FP32><<<grid, kFuseBlock, 0, s>>>(M, pix, fc, Twc, parts, status); break;
    }
}

}  // namespace gsdf

using namespace gsdf;

extern "C" size_t gsdf_integrate_scratch_bytes(const gsdf_camera* cam) {
    if (!valid_cam(cam)) return 0;
    return pix_bytes(*cam) + kPartsBytes;
}

extern "C" int gsdf_integrate_frame(gsdf_map* map, const float* depth_dev, const gsdf_camera* cam,
                                    const double* T_wc_dev, const gsdf_fuse_params* params,
                                    void* scratch_dev, size_t scratch_bytes, int32_t* status_dev,
                                    void* stream) {
    if (!valid_map(map) || !depth_dev || !valid_cam(cam) || !T_wc_dev || !params || !scratch_dev)
        return GSDF_EINVAL;
    if (!(params->eps_weight < map->desc.truncation)) return GSDF_EINVAL;
    if (scratch_bytes < pix_bytes(*cam)) return GSDF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const FuseConsts fc = fuse_consts(*map, *cam, *params);
    const MapView M = make_view(*map);
    float4* pix = (float4*)scratch_dev;
    {
        TimedLaunch t(map->timer, GSDF_K_NORMALS, s);
        dim3 grid(ceil_div(cam->width, kTile), ceil_div(cam->height, kTile));
        k_pixel_normals<<<grid, 256, 0, s>>>(depth_dev, fc, T_wc_dev, pix);
    }
    {
        TimedLaunch t(map->timer, GSDF_K_INTEGRATE, s);
        launch_fuse_blocks(*map, *cam, s, M, scratch_dev, scratch_bytes, fc, T_wc_dev, status_dev);
    }
    return launch_status();
}

extern "C" int gsdf_fuse_frame(gsdf_map* map, const float* depth_dev, const gsdf_camera* cam,
                               const double* T_wc_dev, const gsdf_fuse_params* params, void* scratch_dev,
                               size_t scratch_bytes, int32_t* status_dev, void* stream) {
    if (!valid_map(map) || !depth_dev || !valid_cam(cam) || !T_wc_dev || !params || !scratch_dev)
        return GSDF_EINVAL;
    if (!(params->eps_weight < map->desc.truncation)) return GSDF_EINVAL;
    if (scratch_bytes < pix_bytes(*cam)) return GSDF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const FuseConsts fc = fuse_consts(*map, *cam, *params);
    const MapView M = make_view(*map);
    float4* pix = (float4*)scratch_dev;
    {
        TimedLaunch t(map->timer, GSDF_K_ALLOC_NORMALS, s);
        dim3 grid(ceil_div(cam->width, kTile), ceil_div(cam->height, kTile), 2);
        k_alloc_normals<<<grid, 256, 0, s>>>(M, depth_dev, fc, T_wc_dev, pix, status_dev);
    }
    {
        TimedLaunch t(map->timer, GSDF_K_INTEGRATE, s);
        launch_fuse_blocks(*map, *cam, s, M, scratch_dev, scratch_bytes, fc, T_wc_dev, status_dev);
    }
    return launch_status();
}
