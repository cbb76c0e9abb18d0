// Differentiable form of the tracking energy over keyframes.
//
// Loss of keyframe i (Sec. 4.1 Eq. (5) with the Huber penalty of Sec. 5.1):
//   L_i = sum_k rho_delta(r_ik),  r = psi_j + gh_j . (q - v_j),
//   q = T_i x_k,  T_i = exp(xi_i^) T0_i,  j = nearest voxel of q (Eq. (14)),
// gh_j = g_j / |g_j|.  Per-voxel parameters are {psi_j, g_j} (float4 in the
// map's slot order, voxel c of a block at its Morton index); the map's W
// only marks a voxel as observed.
//
// The adjoint recomputes every residual from the depth and the pose (no
// per-pixel Jacobian is stored):
//   dL/dpsi_j += sum_k s rho'(r_k),
//   dL/dg_j   += (I - gh gh^T) / |g_j| sum_k s rho'(r_k) (q_k - v_j),
//   dL/dxi_i   = Jl(xi_i)^T sum_k s rho'(r_ik) [gh; q x gh],
// with s the upstream gradient of L_i and k over the pixels whose voxel is j
// (the projection (I - gh gh^T) / |g_j| is the same for every pixel of a
// voxel, so it is applied once to the voxel's sum).
//
// The loss is a pixel-parallel pass.  The adjoint gathers instead of
// scattering.  A pixel-parallel pass over 32x32 pixel tiles finds each
// pixel's voxel, adds the pixel's loss and pose terms into its keyframe's
// sums (fixed-order float64 reductions), and groups the tile's pixels by map
// block: each tile writes its pixels' ids block by block into its own part
// of a list and one record (block, count) per block it touches.  A scan of
// the per-block record counts and a scatter of the records give each block
// the runs of the list that hold its pixels.  Then one work-group owns a
// map block, walks its runs and adds the pixels' terms into the block's 512
// voxel sums in LDS, and writes each voxel once.  No two work-groups write
// the same voxel, so nothing is added to global memory atomically except
// integer counts, and the voxel sums are 64-bit fixed point (an integer sum
// does not depend on the order of its terms, and the order of the runs
// does vary), so the gradients are the same bits on every run.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>

#include "gsdf.h"
#include "gsdf_common.hpp"
#include "gsdf_finish.hpp"
#include "gsdf_fixed.hpp"
#include "gsdf_host.hpp"
#include "gsdf_se3.hpp"

namespace gsdf {

constexpr int kAdjBlock = 256;
constexpr int kAdjPart = 8;         // doubles per work-group partial: loss, 6 pose sums, count
constexpr int kAdjMaxGroups = 512;  // work-groups per keyframe of the pixel passes
constexpr int kAdjTile = 32;        // the pixel passes take 32x32 pixel tiles, four pixels a thread
constexpr int kScanTile = 4096;     // block counts per work-group of the offset scan
constexpr int kScanBlock = 1024;    // threads of the offset scan
constexpr int kTilePx = kAdjTile * kAdjTile;
constexpr int kCountBits = 10;      // of a record's count less one; the place above (below 2^31 / kTilePx)
static_assert(kTilePx == 1 << kCountBits, "a record's two numbers");
constexpr int kGatherBatch = 2;     // list entries a lane of the gather loads at a time
constexpr int kLookup = 2;          // pixels a thread of the pixel passes looks up together
// Pixels to a piece of the gather: a 2048th of the pixels of all keyframes (two
// pieces for each of the chip's resident work-groups), at least kMinPiece.  A
// block with more than twice that is gathered in parts.
constexpr int kGatherShare = 2048;
constexpr int kMinPiece = 1024;

struct AdjArgs {
    int32_t W, H, groups, freeze;
    double fx, fy, ifx, ify, cx, cy;
    float zmin, zmax, delta, pad;
    double vs, inv_vs;
    int64_t param_blocks;   // rows of the parameter buffer (slots beyond are unobserved)
};

// Scratch of the keyframe calls: per-work-group partials of the keyframe
// sums, the keyframe poses exp(xi^) T0, two words of bounds (the reach of a
// frozen association as float64 bits, max |s_i|), and the pixel lists:
// per tile (K x tiles of them) 1024 list entries (pixel of the tile, depth) and up
// to 1024 records (block; its count of pixels and the record's place among
// the block's), the records' count per tile, the runs (start, count) sorted
// by block, and per block its tally (runs in the low word, pixels in the
// high: one atomic counts both) and first run, with the per-tile sums of the
// scan.  Then what the gather needs to
// take a block in parts.
struct AdjScratch {
    size_t partials, poses, bounds, list, recs, nrec, runs, tally, run_off, tiles, total;
    // the gather's pieces (a caller whose scratch ends at `total` has every
    // block gathered whole)
    size_t tile_sums, items, done, buffers, split_total;
    int32_t piece, n_buffers;   // pixels to a piece; partial-sum buffers
};
constexpr size_t kBufferBytes = (size_t)4 * kBlockVoxels * sizeof(unsigned long long);

inline int64_t adj_tiles(int32_t W, int32_t H) {
    return (int64_t)((W + kAdjTile - 1) / kAdjTile) * ((H + kAdjTile - 1) / kAdjTile);
}

inline AdjScratch adj_scratch(int32_t K, int64_t tiles, int64_t param_blocks) {
    AdjScratch L;
    size_t o = 0;
    const size_t regions = (size_t)K * (size_t)tiles;
    const size_t n = regions * kTilePx;
    const size_t nb = (size_t)(param_blocks > 0 ? param_blocks : 1);
    L.partials = o;  o = align256(o + (size_t)K * kAdjMaxGroups * kAdjPart * sizeof(double));
    L.poses = o;     o = align256(o + (size_t)K * 12 * sizeof(double));
    L.bounds = o;    o = align256(o + 2 * sizeof(double));
    L.list = o;      o = align256(o + n * sizeof(uint2));
    L.recs = o;      o = align256(o + n * sizeof(int2));
    L.nrec = o;      o = align256(o + regions * sizeof(int32_t));
    L.runs = o;      o = align256(o + n * sizeof(int2));
    L.tally = o;     o = align256(align256(o + nb * sizeof(int32_t)) + nb * sizeof(int32_t));
    L.run_off = o;   o = align256(o + nb * sizeof(int32_t));
    o = align256(o + nb * sizeof(int32_t));   // not used; keeps the sizes that callers have
    L.tiles = o;     o = align256(o + ((nb + kScanTile - 1) / kScanTile) * sizeof(int32_t));
    L.total = o;
    const int64_t piece = (int64_t)(n / kGatherShare);
    L.piece = (int32_t)(piece > kMinPiece ? piece : kMinPiece);
    // blocks above two pieces: at most n / (2 piece) of them, with n / piece
    // whole pieces between them and one more each (and room for the rounding
    // of the quotients)
    L.n_buffers = (int32_t)(2 * (int64_t)n / (int64_t)L.piece + 2);
    L.tile_sums = o; o = align256(o + ((nb + kScanTile - 1) / kScanTile) * 2 * sizeof(int32_t));
    L.items = o;     o = align256(o + (nb + (size_t)L.n_buffers + 1) * sizeof(int4));
    L.done = o;      o = align256(o + nb * sizeof(int32_t));
    L.buffers = o;   o = align256(o + (size_t)L.n_buffers * kBufferBytes);
    L.split_total = o;
    return L;
}

// World point q = R x + t of pixel (u, v) with depth D, x = D [(u-cx)/fx,
// (v-cy)/fy, 1], in float64 with every multiply-add written out, so that
// the loss pass and the adjoint form the same bits.
__device__ inline void pixel_point(const AdjArgs& a, const double R[9], const double t[3], float D, int u, int v,
                                   double q[3]) {
    const double Dd = (double)D;
    const double x0 = Dd * (((double)u - a.cx) * a.ifx);
    const double x1 = Dd * (((double)v - a.cy) * a.ify);
#pragma unroll
    for (int r = 0; r < 3; ++r) q[r] = fma(R[3 * r], x0, fma(R[3 * r + 1], x1, fma(R[3 * r + 2], Dd, t[r])));
}

// The voxel, and its coordinates still in float64 (the same numbers where
// they fit the block keys' range).
__device__ inline void nearest_voxel(const AdjArgs& a, const double q[3], int m[3], double near[3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        near[r] = floor(fma(q[r], a.inv_vs, 0.5));
        m[r] = (int)near[r];
    }
}

// Voxel, offsets and parameters of one pixel.
struct PixelTerm {
    float D, psi, gh[3], inv_ng, dq[3], q[3];
};

// Pool slot of a block key whose first probe, at h, held neither the key
// nor the empty key: linear probing from h + 1 (an empty entry ends it).
__device__ inline int32_t hash_probe_rest(const MapView& M, uint64_t key, uint64_t h) {
    for (uint64_t probe = 1; probe <= M.mask; ++probe) {
        h = (h + 1) & M.mask;
        const uint4 e = *reinterpret_cast<const uint4*>(&M.hash[h]);
        const uint64_t k = (uint64_t)e.x | ((uint64_t)e.y << 32);
        if (k == key) return (int32_t)e.z;
        if (k == kEmptyKey) return -1;
    }
    return -1;
}

// The voxel terms of NP pixels of one thread, stage by stage, every load of
// a stage issued for all NP pixels before any is used: the depth (and the
// frozen voxel when READ_ASSOC), then the point q = T x and its nearest
// voxel (Eq. (14)) with the block's first hash probe, then the rest of the
// probe (rarely needed), then the voxel's weight and parameters.  ok[j]:
// the pixel has a usable voxel (valid depth, block present below
// param_blocks, W > 0, g != 0); then slot[j], m[j] (voxel coordinates) and
// P[j] hold it.  look[j]: the pixel reached the hash lookup (valid depth
// and, when READ_ASSOC, an associated voxel).  With READ_ASSOC, *reach
// takes the largest per-axis distance of a point outside its frozen
// voxel's cell.
template <int NP, bool READ_ASSOC>
__device__ inline void lookup_batch(const MapView& M, const AdjArgs& a, const double R[9], const double t[3],
                                    const float4* __restrict__ params, const float* __restrict__ dimg,
                                    const int32_t* __restrict__ aimg, const int (&u)[NP], const int (&v)[NP],
                                    const bool (&in)[NP], bool (&ok)[NP], bool (&look)[NP], int32_t (&slot)[NP],
                                    int (&m)[NP][3], PixelTerm (&P)[NP], double* reach) {
    float D[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int i = v[j] * a.W + u[j];   // a pixel of the image when in[j]
        D[j] = in[j] ? dimg[i] : 0.0f;
        if (READ_ASSOC && in[j]) {
            const int32_t* as = aimg + 3 * (size_t)i;
            m[j][0] = as[0];
            m[j][1] = as[1];
            m[j][2] = as[2];
        }
    }
    uint64_t key[NP], h[NP];
    uint4 e[NP];
    bool probe[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        probe[j] = false;
        look[j] = in[j] && depth_ok(D[j], a.zmin, a.zmax);
        if (READ_ASSOC) look[j] = look[j] && m[j][0] != INT_MIN;
        if (!look[j]) continue;
        P[j].D = D[j];
        double q[3], near[3];
        pixel_point(a, R, t, D[j], u[j], v[j], q);
        if (READ_ASSOC) {
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                near[r] = (double)m[j][r];
                *reach = fmax(*reach, fabs(q[r] - a.vs * near[r]) - 0.5 * a.vs);
            }
        } else {
            nearest_voxel(a, q, m[j], near);
        }
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            P[j].q[r] = (float)q[r];
            P[j].dq[r] = (float)(q[r] - a.vs * near[r]);
        }
        const int bx = block_of(m[j][0]), by = block_of(m[j][1]), bz = block_of(m[j][2]);
        probe[j] = key_in_range(bx, by, bz);
        if (!probe[j]) continue;
        key[j] = pack_key(bx, by, bz);
        h[j] = block_hash(bx, by, bz) & M.mask;
        e[j] = *reinterpret_cast<const uint4*>(&M.hash[h[j]]);
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        slot[j] = -1;
        if (!look[j] || !probe[j]) continue;
        const uint64_t k = (uint64_t)e[j].x | ((uint64_t)e[j].y << 32);
        if (k == key[j])
            slot[j] = (int32_t)e[j].z;
        else if (k != kEmptyKey)
            slot[j] = hash_probe_rest(M, key[j], h[j]);
    }
    float Wv[NP];
    float4 pr[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        ok[j] = slot[j] >= 0 && (int64_t)slot[j] < a.param_blocks;
        if (!ok[j]) continue;
        const int64_t vi = (int64_t)slot[j] * kBlockVoxels + morton9(m[j][0] & 7, m[j][1] & 7, m[j][2] & 7);
        Wv[j] = M.weight[vi];
        pr[j] = params[vi];
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        if (!ok[j]) continue;
        const float n2 = pr[j].y * pr[j].y + pr[j].z * pr[j].z + pr[j].w * pr[j].w;
        ok[j] = Wv[j] > 0.0f && n2 > 0.0f;
        if (!ok[j]) continue;
        P[j].inv_ng = 1.0f / sqrtf(n2);
        P[j].psi = pr[j].x;
        P[j].gh[0] = pr[j].y * P[j].inv_ng;
        P[j].gh[1] = pr[j].z * P[j].inv_ng;
        P[j].gh[2] = pr[j].w * P[j].inv_ng;
    }
}

// Residual terms of one pixel: Huber loss, s rho'(r) and the Jacobian row
// [gh; q x gh] of a left increment of the keyframe pose.
struct ResidualTerms {
    float rho, rp, J[6];
};

__device__ inline ResidualTerms residual_terms(const PixelTerm& P, float delta, float s) {
    ResidualTerms o;
    const float r = P.psi + P.gh[0] * P.dq[0] + P.gh[1] * P.dq[1] + P.gh[2] * P.dq[2];
    const float ar = fabsf(r);
    const bool quad = ar <= delta;
    o.rho = quad ? 0.5f * r * r : delta * (ar - 0.5f * delta);
    o.rp = s * (quad ? r : copysignf(delta, r));   // s rho'(r)
    o.J[0] = P.gh[0];
    o.J[1] = P.gh[1];
    o.J[2] = P.gh[2];
    o.J[3] = P.q[1] * P.gh[2] - P.q[2] * P.gh[1];
    o.J[4] = P.q[2] * P.gh[0] - P.q[0] * P.gh[2];
    o.J[5] = P.q[0] * P.gh[1] - P.q[1] * P.gh[0];
    return o;
}

// Work-group sum of kAdjPart values per thread, in float64 (across lanes,
// then one value per wave in a fixed order); the totals land in out[] of
// threads 0 .. kAdjPart-1 (out[k] in thread k).
template <typename T>
__device__ inline double block_sum_part(const T acc[kAdjPart], double (*s_red)[kAdjBlock / 64]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double d[kAdjPart];
#pragma unroll
    for (int k = 0; k < kAdjPart; ++k) d[k] = (double)acc[k];
    static_assert(kAdjPart == 8, "wave_sum8");
    const double y = wave_sum8(d, lane);
    if ((lane & 7) == 0) s_red[wave_sum8_value(lane)][wave] = y;
    __syncthreads();
    double x = 0.0;
    if (threadIdx.x < kAdjPart)
        for (int w = 0; w < kAdjBlock / 64; ++w) x += s_red[threadIdx.x][w];
    __syncthreads();
    return x;
}

// The loss pass.  Grid (groups, K): a work-group takes 32x32 pixel tiles of
// keyframe blockIdx.y (four pixels a thread, looked up together) and
// writes its partial sums (loss, the six pose sums unused here, the count
// of pixels used); FREEZE reads each pixel's voxel from the association
// buffer, else with an association buffer it records each pixel's voxel
// (INT32_MIN for a pixel without a usable voxel).
template <bool FREEZE>
__global__ __launch_bounds__(kAdjBlock) void k_keyframe_loss(MapView M, AdjArgs a, const float* __restrict__ depth,
                                                             const double* __restrict__ poses,
                                                             const float4* __restrict__ params,
                                                             int32_t* __restrict__ assoc,
                                                             double* __restrict__ partials) {
    __shared__ double s_red[kAdjPart][kAdjBlock / 64];
    constexpr int kPer = kTilePx / kAdjBlock;
    // work-group (x, k) in XCD-aware order: neighbouring tiles share an L2
    const int lin = band_rank(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int kf = lin / gridDim.x, grp = lin - kf * gridDim.x;
    double R[9], t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j) R[3 * i + j] = poses[12 * kf + 4 * i + j];
        t[i] = poses[12 * kf + 4 * i + 3];
    }
    const int N = a.W * a.H;
    const float* dimg = depth + (size_t)kf * N;
    int32_t* aimg = assoc ? assoc + (size_t)kf * N * 3 : nullptr;
    float acc[kAdjPart];
#pragma unroll
    for (int k = 0; k < kAdjPart; ++k) acc[k] = 0.0f;
    double reach = 0.0;
    const int tiles_x = (a.W + kAdjTile - 1) / kAdjTile;
    const int ntiles = tiles_x * ((a.H + kAdjTile - 1) / kAdjTile);
    for (int tile = grp; tile < ntiles; tile += a.groups) {
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
#pragma unroll
        for (int g = 0; g < kPer; g += kLookup) {
            int u[kLookup], v[kLookup];
            bool in[kLookup], ok[kLookup], look[kLookup];
            int32_t slot[kLookup];
            int m[kLookup][3];
            PixelTerm P[kLookup];
#pragma unroll
            for (int j = 0; j < kLookup; ++j) {
                const int px = threadIdx.x + (g + j) * kAdjBlock;
                u[j] = tx * kAdjTile + (px % kAdjTile);
                v[j] = ty * kAdjTile + px / kAdjTile;
                in[j] = u[j] < a.W && v[j] < a.H;
            }
            lookup_batch<kLookup, FREEZE>(M, a, R, t, params, dimg, aimg, u, v, in, ok, look, slot, m, P, &reach);
#pragma unroll
            for (int j = 0; j < kLookup; ++j) {
                if (ok[j]) {
                    acc[0] += residual_terms(P[j], a.delta, 0.0f).rho;
                    acc[7] += 1.0f;
                }
                if (!FREEZE && aimg && in[j]) {
                    int32_t* as = aimg + 3 * ((size_t)v[j] * a.W + u[j]);
                    as[0] = ok[j] ? m[j][0] : INT_MIN;
                    as[1] = ok[j] ? m[j][1] : INT_MIN;
                    as[2] = ok[j] ? m[j][2] : INT_MIN;
                }
            }
        }
    }
    const double x = block_sum_part(acc, s_red);
    if (threadIdx.x < kAdjPart) partials[((size_t)kf * a.groups + grp) * kAdjPart + threadIdx.x] = x;
}

// Keyframe poses exp(xi^) T0 (float64), and for the adjoint the cleared
// per-block counters and reach word.  One thread per keyframe and per block.
__global__ void k_adj_setup(int32_t K, const double* __restrict__ T0, const double* __restrict__ xi,
                            double* __restrict__ poses, int64_t nb, unsigned long long* __restrict__ tally,
                            int32_t* __restrict__ done, unsigned long long* __restrict__ reach) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < K) {
        double pose[12];
        for (int j = 0; j < 12; ++j) pose[j] = T0[12 * i + j];
        se3_apply_left(xi + 6 * i, pose);
        for (int j = 0; j < 12; ++j) poses[12 * i + j] = pose[j];
    }
    if (i < nb) {
        tally[i] = 0ull;
        if (done) done[i] = 0;
    }
    if (i == 0 && reach) *reach = 0ull;
}

// Exclusive work-group prefix sums of two int32 per thread (all threads of
// WAVES waves): a wave scan, the wave totals in LDS (s_w: 2 WAVES words).  The
// totals land in *tot_a, *tot_b.
template <int WAVES = 4>
__device__ inline void block_scan2(int32_t a, int32_t b, int32_t* ex_a, int32_t* ex_b, int32_t* tot_a,
                                   int32_t* tot_b, int32_t* s_w) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t ia = wave_scan(a), ib = wave_scan(b);
    __syncthreads();   // s_w may still be read by a previous call
    if (lane == 63) {
        s_w[wave] = ia;
        s_w[WAVES + wave] = ib;
    }
    __syncthreads();
    int32_t pa = 0, pb = 0, ta = 0, tb = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) {
            pa += s_w[w];
            pb += s_w[WAVES + w];
        }
        ta += s_w[w];
        tb += s_w[WAVES + w];
    }
    *ex_a = pa + ia - a;
    *ex_b = pb + ib - b;
    *tot_a = ta;
    *tot_b = tb;
}

// The adjoint's pixel pass.  Grid (groups, K), 32x32 tiles as the loss
// pass; tile t of keyframe k is region r = k tiles + t.  Per pixel: its
// voxel (nearest, or frozen), and when the voxel is usable (block present
// below param_blocks, W > 0, g != 0) its loss, pose terms s rho' [g^; q x g^]
// and count into this work-group's partial of its keyframe.  The tile's
// usable pixels are grouped by block in LDS (an open-addressing table of
// 1024 entries, so it never fills; one LDS atomic add gives a pixel its
// rank in its block); a scan of the entries' counts places each block's
// pixels (place in the tile and depth) in a run of the region's 1024 list
// entries, and the region gets one record per block (its count, and its place
// among the block's records, which the atomic that tallies the block
// returned), in run order, and nrec[r] records.  With a
// frozen association the pass also finds how far (per axis, metres) the
// points lie outside the cells of their frozen voxels, as the bits of a
// non-negative float64 (whose integer order is its numeric order); that
// bounds the offsets q - v of the voxel sums.
//
// A pixel without a finite offset is not listed: a fixed-point term of a NaN
// or an infinity would be an arbitrary integer in the sums of a voxel that
// other keyframes share.  So a keyframe whose pose is not finite (a NaN twist)
// lists nothing and reaches nowhere, and its own loss and pose sums alone are
// NaN.  At a finite pose the nearest voxel lies within half a voxel of the
// point; only a frozen one can be out of float32's range.
//
// Bound by instruction issue (300 vector and 180 scalar instructions a
// wave of pixels at the start of this form, the vector units 70 % busy; the
// LDS table's atomics are not it: one per block and wave instead of one per
// pixel changed nothing).  The sums across lanes and the scans by register
// moves instead of shuffles, the voxel kept in float64 and the shorter hash
// and Morton code: 30 keyframes of 640x480 122 -> 82 us, 88 with the records'
// places (which take 11 us from k_adj_runs), 92 with the check of the pose.
// 95 registers hold five waves to a SIMD; the frozen form takes four.
template <bool FREEZE>
__global__ __launch_bounds__(kAdjBlock, FREEZE ? 4 : 5) void k_adj_pixels(MapView M, AdjArgs a, const float* __restrict__ depth,
                                                          const double* __restrict__ poses,
                                                          const float4* __restrict__ params,
                                                          const float* __restrict__ gscale,
                                                          const int32_t* __restrict__ assoc,
                                                          uint2* __restrict__ list, int2* __restrict__ recs,
                                                          int32_t* __restrict__ nrec,
                                                          unsigned long long* __restrict__ tally,
                                                          unsigned long long* __restrict__ reach,
                                                          double* __restrict__ partials) {
    __shared__ double s_red[kAdjPart][kAdjBlock / 64];
    __shared__ double s_max[kAdjBlock / 64];
    __shared__ int32_t s_key[kTilePx];
    __shared__ int32_t s_cnt[kTilePx];
    __shared__ int32_t s_w[8];
    constexpr int kPer = kTilePx / kAdjBlock;   // pixels (and table entries) a thread takes: 4
    // work-group (x, k) in XCD-aware order: neighbouring tiles share an L2
    const int lin = band_rank(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int kf = lin / gridDim.x, grp = lin - kf * gridDim.x;
    double R[9], t[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int c = 0; c < 3; ++c) R[3 * r + c] = poses[12 * kf + 4 * r + c];
        t[r] = poses[12 * kf + 4 * r + 3];
    }
    const float s = gscale[kf];
    // uniform over the work-group; no branches, the lookups need not wait
    bool finite = true;
#pragma unroll
    for (int r = 0; r < 9; ++r) finite &= isfinite(R[r]);
#pragma unroll
    for (int r = 0; r < 3; ++r) finite &= isfinite(t[r]);
    const int N = a.W * a.H;
    const float* dimg = depth + (size_t)kf * N;
    const int32_t* aimg = FREEZE ? assoc + (size_t)kf * N * 3 : nullptr;
    float acc[kAdjPart];   // a thread's (at most four pixels per tile) sums; float64 across threads
#pragma unroll
    for (int k = 0; k < kAdjPart; ++k) acc[k] = 0.0f;
    double e = 0.0;
    const int tiles_x = (a.W + kAdjTile - 1) / kAdjTile;
    const int ntiles = tiles_x * ((a.H + kAdjTile - 1) / kAdjTile);
    for (int tile = grp; tile < ntiles; tile += a.groups) {
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        const int64_t region = (int64_t)kf * ntiles + tile;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            s_key[threadIdx.x + k * kAdjBlock] = -1;
            s_cnt[threadIdx.x + k * kAdjBlock] = 0;
        }
        __syncthreads();
        int32_t ent[kPer], rank[kPer];
        uint32_t pid[kPer];
        float dep[kPer];
#pragma unroll
        for (int g = 0; g < kPer; g += kLookup) {
            int u[kLookup], v[kLookup];
            bool in[kLookup], ok[kLookup], look[kLookup];
            int32_t slot[kLookup];
            int m[kLookup][3];
            PixelTerm P[kLookup];
#pragma unroll
            for (int j = 0; j < kLookup; ++j) {
                const int px = threadIdx.x + (g + j) * kAdjBlock;
                u[j] = tx * kAdjTile + (px % kAdjTile);
                v[j] = ty * kAdjTile + px / kAdjTile;
                in[j] = u[j] < a.W && v[j] < a.H;
            }
            lookup_batch<kLookup, FREEZE>(M, a, R, t, params, dimg, aimg, u, v, in, ok, look, slot, m, P, &e);
#pragma unroll
            for (int j = 0; j < kLookup; ++j) {
                ent[g + j] = -1;
                rank[g + j] = 0;
                pid[g + j] = threadIdx.x + (g + j) * kAdjBlock;
                dep[g + j] = P[j].D;
                if (!ok[j]) continue;
                const ResidualTerms rt = residual_terms(P[j], a.delta, s);
                acc[0] += rt.rho;
#pragma unroll
                for (int k = 0; k < 6; ++k) acc[1 + k] += rt.rp * rt.J[k];
                acc[7] += 1.0f;
                if (!finite) continue;
                if (FREEZE && !(isfinite(P[j].dq[0]) && isfinite(P[j].dq[1]) && isfinite(P[j].dq[2]))) continue;
                // the block's entry in the tile's table (at most 1024 keys: a
                // free or matching entry is always found)
                const int32_t sl = slot[j];
                uint32_t h = ((uint32_t)sl * 2654435761u) >> 22;
                for (;;) {
                    const int32_t old = atomicCAS(&s_key[h], -1, sl);
                    if (old == -1 || old == sl) break;
                    h = (h + 1) & (kTilePx - 1);
                }
                ent[g + j] = (int32_t)h;
                rank[g + j] = atomicAdd(&s_cnt[h], 1);
            }
        }
        __syncthreads();
        // runs: exclusive scan of the entries' counts (thread t owns entries
        // kPer t .. kPer t + kPer - 1), records in the same order
        int32_t c[kPer], own = 0, used = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            c[k] = s_cnt[kPer * threadIdx.x + k];
            own += c[k];
            used += c[k] > 0 ? 1 : 0;
        }
        // (both counts end at most at 1024: one scan of 16 bits each)
        int32_t both, none, tot, tot_none;
        block_scan2(own | (used << 16), 0, &both, &none, &tot, &tot_none, s_w);
        int32_t run = both & 0xffff, rec = both >> 16;
        const int32_t tot_rec = tot >> 16;
        __syncthreads();   // every count is read before s_cnt turns into offsets
        const int64_t base = region * kTilePx;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            s_cnt[kPer * threadIdx.x + k] = run;
            if (c[k] > 0) {
                const int32_t sl = s_key[kPer * threadIdx.x + k];
                const unsigned nth = (unsigned)atomicAdd(&tally[sl], ((unsigned long long)c[k] << 32) | 1ull);
                recs[base + rec] = make_int2(sl, (int)((nth << kCountBits) | (unsigned)(c[k] - 1)));
                ++rec;
            }
            run += c[k];
        }
        if (threadIdx.x == 0) nrec[region] = tot_rec;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (ent[j] >= 0)
                list[base + s_cnt[ent[j]] + rank[j]] = make_uint2(pid[j], __float_as_uint(dep[j]));
        __syncthreads();   // the table is cleared for the next tile
    }
    const double x = block_sum_part(acc, s_red);
    if (threadIdx.x < kAdjPart) partials[((size_t)kf * a.groups + grp) * kAdjPart + threadIdx.x] = x;
    if (!FREEZE || !finite) return;
    for (int off = 32; off > 0; off >>= 1) e = fmax(e, __shfl_xor(e, off));
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        double y = 0.0;
        for (int w = 0; w < kAdjBlock / 64; ++w) y = fmax(y, s_max[w]);
        atomicMax(reach, (unsigned long long)__double_as_longlong(y));
    }
}

// Work-group sum of one int32 per thread (all threads of WAVES waves), in
// every thread.
template <int WAVES>
__device__ inline int32_t block_sum_i32(int32_t x, int32_t* s_w) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
    __syncthreads();
    int32_t t = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) t += s_w[w];
    return t;
}

// Parts in which a block of n pixels in `runs` runs is gathered.
__device__ inline int32_t gather_parts(int32_t n, int32_t runs, int32_t piece, float inv_piece) {
    if (piece == 0 || n <= 2 * piece) return 1;
    const int32_t p = (int32_t)((float)n * inv_piece) + 1;
    return p < runs ? p : runs;
}

// Sums over each tile of kScanTile blocks: run counts, and with pieces the
// blocks that have pixels and the parts of those that are split.
__global__ __launch_bounds__(256) void k_adj_tile_sums(int64_t nb, const uint2* __restrict__ tally, int32_t piece,
                                                       int32_t* __restrict__ tiles, int32_t* __restrict__ piece_tiles) {
    __shared__ int32_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    int32_t x = 0, blocks = 0, parts = 0;
    for (int k = threadIdx.x; k < kScanTile; k += 256)
        if (base + k < nb) {
            const uint2 b = tally[base + k];
            const int32_t r = (int32_t)b.x;
            x += r;
            if (piece && r > 0) {
                const int32_t p = gather_parts((int32_t)b.y, r, piece, 1.0f / (float)piece);
                if (p > 1)
                    parts += p;
                else
                    ++blocks;
            }
        }
    x = block_sum_i32<4>(x, s_w);
    if (threadIdx.x == 0) tiles[blockIdx.x] = x;
    if (!piece) return;
    blocks = block_sum_i32<4>(blocks, s_w);
    parts = block_sum_i32<4>(parts, s_w);
    if (threadIdx.x == 0) {
        piece_tiles[2 * blockIdx.x] = blocks;
        piece_tiles[2 * blockIdx.x + 1] = parts;
    }
}

// First run of each block (exclusive prefix sums of the run counts), one
// work-group per tile: the sum of the earlier tiles, then a scan of the
// tile (four consecutive counts a thread).  With pieces also the list of the
// gather's items {slot, part, parts, first buffer}: at 1 + i the i-th part of
// a split block (buffer i), then from 1 + (all parts) on the whole blocks
// that have pixels; item 0 holds {all parts, whole blocks} (each written by
// the tile that knows it).  Work-group 0 also writes max_i |s_i|.
__global__ __launch_bounds__(kScanBlock) void k_adj_offsets(int64_t nb, const uint2* __restrict__ tally,
                                                     const int32_t* __restrict__ tiles,
                                                     int32_t* __restrict__ offsets, int32_t K,
                                                     const float* __restrict__ gscale, double* __restrict__ bounds,
                                                     int32_t piece, const int32_t* __restrict__ piece_tiles,
                                                     int4* __restrict__ items) {
    constexpr int kWaves = kScanBlock / 64, kPer = kScanTile / kScanBlock;
    __shared__ int32_t s_w[2 * kWaves];
    int32_t before = 0, before_blocks = 0, before_parts = 0, all_parts = 0;
    if (tiles) {   // null for a single tile
        for (int g = threadIdx.x; g < (int)blockIdx.x; g += kScanBlock) before += tiles[g];
        before = block_sum_i32<kWaves>(before, s_w);
        if (piece) {
            for (int g = threadIdx.x; g < (int)gridDim.x; g += kScanBlock) {
                if (g < (int)blockIdx.x) {
                    before_blocks += piece_tiles[2 * g];
                    before_parts += piece_tiles[2 * g + 1];
                }
                all_parts += piece_tiles[2 * g + 1];
            }
            before_blocks = block_sum_i32<kWaves>(before_blocks, s_w);
            before_parts = block_sum_i32<kWaves>(before_parts, s_w);
            all_parts = block_sum_i32<kWaves>(all_parts, s_w);
        }
    }
    const int64_t i0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kPer;
    int32_t c[kPer], n[kPer];
    int32_t own = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const uint2 b = i0 + k < nb ? tally[i0 + k] : make_uint2(0u, 0u);
        c[k] = (int32_t)b.x;
        n[k] = (int32_t)b.y;
        own += c[k];
    }
    int32_t run, unused, tot, tot2;
    block_scan2<kWaves>(own, 0, &run, &unused, &tot, &tot2, s_w);
    run += before;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (i0 + k < nb) offsets[i0 + k] = run;
        run += c[k];
    }
    if (piece) {
        int32_t p[kPer], blocks = 0, parts = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            p[k] = c[k] > 0 ? gather_parts(n[k], c[k], piece, 1.0f / (float)piece) : 0;
            if (p[k] > 1)
                parts += p[k];
            else
                blocks += p[k];
        }
        int32_t at_block, at_part, tot_blocks, tot_parts;
        block_scan2<kWaves>(blocks, parts, &at_block, &at_part, &tot_blocks, &tot_parts, s_w);
        at_block += before_blocks;
        at_part += before_parts;
        if (!tiles) all_parts = tot_parts;
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
            items[0] = make_int4(all_parts, before_blocks + tot_blocks, 0, 0);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (p[k] == 1) items[1 + all_parts + at_block++] = make_int4((int)(i0 + k), 0, 1, 0);
            if (p[k] > 1) {
                // (there are buffers for every part that the sizes allow)
                for (int j = 0; j < p[k]; ++j)
                    items[1 + at_part + j] = make_int4((int)(i0 + k), j, p[k], at_part);
                at_part += p[k];
            }
        }
    }
    if (blockIdx.x != 0) return;
    float smax = 0.0f;
    for (int k = threadIdx.x; k < K; k += kScanBlock) smax = fmaxf(smax, fabsf(gscale[k]));
    for (int off = 32; off > 0; off >>= 1) smax = fmaxf(smax, __shfl_xor(smax, off));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = __float_as_int(smax);   // non-negative: integer order
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t b = s_w[0];
        for (int w = 1; w < kWaves; ++w) b = s_w[w] > b ? s_w[w] : b;
        bounds[1] = (double)__int_as_float(b);
    }
}

// Each region's records into their blocks' run lists: one wave per region
// (four a work-group); a record's run starts in the region's list at the
// sum of the counts of the records before it; its place among its block's
// runs came with the block's count of runs.  (Taken here from a second counter
// for each block, the blocks that many tiles see made this 16.5 us at 30
// keyframes of 640x480, one atomic after the other.)
__global__ __launch_bounds__(256) void k_adj_runs(int64_t regions, const int32_t* __restrict__ nrec,
                                                  const int2* __restrict__ recs, const int32_t* __restrict__ run_off,
                                                  int2* __restrict__ runs) {
    const int64_t region = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (region >= regions) return;   // the whole wave
    const int32_t n = nrec[region];
    int32_t start = 0;
    for (int k0 = 0; k0 < n; k0 += 64) {   // uniform over the wave
        const int k = k0 + lane;
        const int2 r = k < n ? recs[region * kTilePx + k] : make_int2(0, 0);
        const int32_t count = k < n ? (r.y & (kTilePx - 1)) + 1 : 0;
        const int32_t incl = wave_scan(count);
        if (k < n)
            runs[run_off[r.x] + (int32_t)((uint32_t)r.y >> kCountBits)] =
                make_int2((int32_t)(region * kTilePx) + start + incl - count, count);
        start += __shfl(incl, 63);
    }
}

// Largest f with bound 2^f < 2^top (bound = m 2^e, 1 <= m < 2: f = top-1-e),
// kept where 2^-f and the terms' grid are normal float64 numbers.
__device__ inline int fix_scale(double bound, int top) {
    if (!(bound > 0.0)) return 62;
    const int e = ilogb(bound);
    return e > 900 ? -900 : (e < -900 ? 900 : top - 1 - e);
}

__device__ inline void store_agent(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned long long load_agent(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The adjoint's voxel sums, one work-group per map block or part of one (a
// share of its runs).  The waves take runs in turn; a run lies in one tile of
// one keyframe, so its pose and the tile's corner are the same for the whole
// wave.  A lane takes entries l, l + 64, ... of the run (kGatherBatch of them
// with their loads in flight together), recomputes each pixel's point, voxel
// and residual from the block's parameters in LDS, and adds s rho' and
// s rho' (q - v) into its voxel's sums in LDS.  Then each voxel's gradient is
// formed from its sums and added to dparams by the one thread that owns the
// voxel; of a block in parts, by the last part to finish, which adds the
// others' sums from their buffers.
//
// The sums are 64-bit fixed point (magic_term), so neither the order of the
// runs nor the parts change a bit.  With n the pixels of the block and
// s_max = max_i |s_i|, a term |s rho'| <= s_max delta and |q - v| per axis is
// at most v_s / 2 + reach + margin (reach: of a frozen association); the
// scales f_p and f_q keep a term below 2^51 and n terms below 2^62.
//
// Bound by VALU issue and the blocks' unevenness: blocks near the cameras hold
// many times the pixels of others, and one work-group for each ran long after
// the rest had finished: at
// 640x480 10 keyframes 79 -> 49 us, 30 keyframes 212 -> 100 us (kernel trace);
// with the gradients normalised once a voxel instead of once a pixel, 46 and
// 87 us.
template <bool FREEZE>
__global__ __launch_bounds__(kAdjBlock) void k_backward_gather(MapView M, AdjArgs a, int32_t ntiles, int32_t tiles_x,
                                                               const double* __restrict__ poses,
                                                               const float4* __restrict__ params,
                                                               const float* __restrict__ gscale,
                                                               const int32_t* __restrict__ assoc,
                                                               const uint2* __restrict__ list,
                                                               const int2* __restrict__ runs,
                                                               const uint2* __restrict__ tally,
                                                               const int32_t* __restrict__ run_off,
                                                               const double* __restrict__ bounds,
                                                               const int4* __restrict__ items,
                                                               int32_t* __restrict__ done,
                                                               unsigned long long* __restrict__ buffers,
                                                               float* __restrict__ dparams) {
    __shared__ unsigned long long sP[kBlockVoxels];
    __shared__ unsigned long long sQ[3][kBlockVoxels];
    // {psi, g^} in the map's (Morton) order, normalised once a voxel; psi = NaN
    // without a gradient (never a listed pixel's voxel: the pixel pass checked
    // it)
    __shared__ float4 s_par[kBlockVoxels];
    __shared__ int s_last;
    int4 item = make_int4((int)blockIdx.x, 0, 1, 0);
    if (items) {
        const int4 all = items[0];
        if ((int)blockIdx.x >= all.x + all.y) return;
        item = items[1 + blockIdx.x];
    }
    const int64_t slot = item.x;
    const uint2 counted = tally[slot];
    const int32_t n = (int32_t)counted.y, nruns = (int32_t)counted.x;
    if (n == 0) return;
    const int32_t roff = run_off[slot];
    const int32_t r0 = (int32_t)((int64_t)nruns * item.y / item.z), r1 = (int32_t)((int64_t)nruns * (item.y + 1) / item.z);
    for (int c = threadIdx.x; c < kBlockVoxels; c += kAdjBlock) {
        sP[c] = 0ull;
        sQ[0][c] = sQ[1][c] = sQ[2][c] = 0ull;
        const float4 pv = params[slot * kBlockVoxels + c];
        const float n2 = pv.y * pv.y + pv.z * pv.z + pv.w * pv.w;
        const float inv_ng = 1.0f / sqrtf(n2);
        s_par[c] = n2 > 0.0f ? make_float4(pv.x, pv.y * inv_ng, pv.z * inv_ng, pv.w * inv_ng)
                             : make_float4(__builtin_nanf(""), 0.0f, 0.0f, 0.0f);
    }
    const double rmax =
        FREEZE ? __longlong_as_double((long long)reinterpret_cast<const unsigned long long*>(bounds)[0]) : 0.0;
    const double margin = 1e-6 * (1.0 + fabs(a.vs) * 1e3);
    const double term_p = bounds[1] * (double)a.delta, term_q = term_p * (0.5 * a.vs + rmax + margin);
    const int fp = min(fix_scale(term_p, 51), fix_scale(term_p * (double)n, 62));
    const int fq = min(fix_scale(term_q, 51), fix_scale(term_q * (double)n, 62));
    const double mp = magic_of(fp), mq = magic_of(fq);
    const unsigned long long np = 0ull - double_bits(mp), nq = 0ull - double_bits(mq);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int r = r0 + (int)(threadIdx.x >> 6); r < r1; r += kAdjBlock / 64) {
        // uniform over the wave
        const int2 rn = runs[roff + r];
        const int start = __builtin_amdgcn_readfirstlane(rn.x), count = __builtin_amdgcn_readfirstlane(rn.y);
        const int region = start / kTilePx;
        const int kf = region / ntiles, tile = region - kf * ntiles;
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        double R[9], t[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int c = 0; c < 3; ++c) R[3 * i + c] = poses[12 * kf + 4 * i + c];
            t[i] = poses[12 * kf + 4 * i + 3];
        }
        const float s = gscale[kf];
        for (int j0 = lane; j0 - lane < count; j0 += 64 * kGatherBatch) {
            uint2 le[kGatherBatch];
            bool live[kGatherBatch];
            int m[kGatherBatch][3];
#pragma unroll
            for (int b = 0; b < kGatherBatch; ++b) {
                live[b] = j0 + 64 * b < count;
                le[b] = live[b] ? list[start + j0 + 64 * b] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int b = 0; b < kGatherBatch; ++b) {
                const int u = tx * kAdjTile + (int)(le[b].x % kAdjTile), v = ty * kAdjTile + (int)(le[b].x / kAdjTile);
                if (FREEZE && live[b]) {
                    const int32_t* as = assoc + ((size_t)kf * a.W * a.H + (size_t)v * a.W + u) * 3;
                    m[b][0] = as[0];
                    m[b][1] = as[1];
                    m[b][2] = as[2];
                }
            }
#pragma unroll
            for (int b = 0; b < kGatherBatch; ++b) {
                if (!live[b]) continue;
                const int u = tx * kAdjTile + (int)(le[b].x % kAdjTile), v = ty * kAdjTile + (int)(le[b].x / kAdjTile);
                double q[3], near[3];
                pixel_point(a, R, t, __uint_as_float(le[b].y), u, v, q);
                if (!FREEZE) nearest_voxel(a, q, m[b], near);
                PixelTerm P;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    P.dq[k] = (float)(q[k] - a.vs * (FREEZE ? (double)m[b][k] : near[k]));
                const float4 pv = s_par[morton9(m[b][0] & 7, m[b][1] & 7, m[b][2] & 7)];
                P.psi = pv.x;
                P.gh[0] = pv.y;
                P.gh[1] = pv.z;
                P.gh[2] = pv.w;
                P.q[0] = P.q[1] = P.q[2] = 0.0f;   // (the pose rows are not used here)
                float rp = residual_terms(P, a.delta, s).rp;
                rp = rp == rp ? rp : 0.0f;   // a NaN (of the upstream gradient) adds nothing
                const int c = (m[b][0] & 7) | ((m[b][1] & 7) << 3) | ((m[b][2] & 7) << 6);
                const double w = (double)rp;
                atomicAdd(&sP[c], magic_term(w + mp, np));
#pragma unroll
                for (int k = 0; k < 3; ++k) atomicAdd(&sQ[k][c], magic_term(fma(w, (double)P.dq[k], mq), nq));
            }
        }
    }
    __syncthreads();
    if (item.z > 1) {
        // device-scope stores that have completed before the ticket,
        // device-scope loads after it
        unsigned long long* mine = buffers + (size_t)(item.w + item.y) * 4 * kBlockVoxels;
        for (int c = threadIdx.x; c < kBlockVoxels; c += kAdjBlock) {
            store_agent(&mine[c], sP[c]);
#pragma unroll
            for (int k = 0; k < 3; ++k) store_agent(&mine[(1 + k) * kBlockVoxels + c], sQ[k][c]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");   // the stores stay above
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0)
            s_last = __hip_atomic_fetch_add(&done[slot], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == item.z - 1;
        __syncthreads();
        if (!s_last) return;
#pragma unroll 1
        for (int o = 0; o < item.z; ++o) {
            if (o == item.y) continue;
            const unsigned long long* other = buffers + (size_t)(item.w + o) * 4 * kBlockVoxels;
            for (int c = threadIdx.x; c < kBlockVoxels; c += kAdjBlock) {
                sP[c] += load_agent(&other[c]);
#pragma unroll
                for (int k = 0; k < 3; ++k) sQ[k][c] += load_agent(&other[(1 + k) * kBlockVoxels + c]);
            }
        }
    }
    // ---- each voxel's gradient from its sums, added once by its owner
    const double ip = ldexp(1.0, -fp), iq = ldexp(1.0, -fq);
    for (int c = threadIdx.x; c < kBlockVoxels; c += kAdjBlock) {
        const unsigned long long p0 = sP[c], q0 = sQ[0][c], q1 = sQ[1][c], q2 = sQ[2][c];
        if ((p0 | q0 | q1 | q2) == 0ull) continue;
        const int mo = morton9(c & 7, (c >> 3) & 7, c >> 6);
        const int64_t vi = slot * kBlockVoxels + mo;
        const float4 p = params[vi];
        const float inv_ng = 1.0f / sqrtf(p.y * p.y + p.z * p.z + p.w * p.w);
        const float gh[3] = {p.y * inv_ng, p.z * inv_ng, p.w * inv_ng};
        const float S[3] = {(float)((double)(long long)q0 * iq), (float)((double)(long long)q1 * iq),
                            (float)((double)(long long)q2 * iq)};
        const float gS = gh[0] * S[0] + gh[1] * S[1] + gh[2] * S[2];
        float4 d = reinterpret_cast<float4*>(dparams)[vi];
        d.x += (float)((double)(long long)p0 * ip);
        d.y += inv_ng * (S[0] - gh[0] * gS);
        d.z += inv_ng * (S[1] - gh[1] * gS);
        d.w += inv_ng * (S[2] - gh[2] * gS);
        reinterpret_cast<float4*>(dparams)[vi] = d;
    }
}

__global__ void k_export_params(MapView M, int storage, int64_t rows, float4* __restrict__ out) {
    const int32_t nb = M.counters[kNumBlocks] < M.max_blocks ? M.counters[kNumBlocks] : M.max_blocks;
    const int64_t n = (rows < (int64_t)nb ? rows : (int64_t)nb) * kBlockVoxels;
    for (int64_t vi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; vi < rows * kBlockVoxels;
         vi += (int64_t)gridDim.x * blockDim.x) {
        float4 p = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (vi < n) {
            const float Wv = M.weight[vi];
            if (storage == GSDF_FP32) {
                const float4 r = reinterpret_cast<const float4*>(M.vox)[vi];
                p = make_float4(Wv > 0.0f ? r.x / Wv : 0.0f, r.y, r.z, r.w);
            } else {
                const ushort4 r = reinterpret_cast<const ushort4*>(M.vox)[vi];
                p = make_float4(unpack16(r.x, storage) * M.truncation, unpack16(r.y, storage),
                                unpack16(r.z, storage), unpack16(r.w, storage));
            }
        }
        out[vi] = p;
    }
}

__global__ void k_import_params(MapView M, int storage, int64_t rows, const float4* __restrict__ in) {
    const int32_t nb = M.counters[kNumBlocks] < M.max_blocks ? M.counters[kNumBlocks] : M.max_blocks;
    const int64_t n = (rows < (int64_t)nb ? rows : (int64_t)nb) * kBlockVoxels;
    for (int64_t vi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; vi < n; vi += (int64_t)gridDim.x * blockDim.x) {
        const float Wv = M.weight[vi];
        if (!(Wv > 0.0f)) continue;   // unobserved voxels keep their (zero) record
        const float4 p = in[vi];
        if (storage == GSDF_FP32) {
            reinterpret_cast<float4*>(M.vox)[vi] = make_float4(p.x * Wv, p.y, p.z, p.w);
        } else {
            reinterpret_cast<ushort4*>(M.vox)[vi] =
                make_ushort4(pack16(p.x / M.truncation, storage), pack16(p.y, storage), pack16(p.z, storage),
                             pack16(p.w, storage));
        }
    }
}

__global__ void k_compose_poses(int32_t K, const double* __restrict__ T0, const double* __restrict__ xi,
                                double* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= K) return;
    double pose[12];
    for (int j = 0; j < 12; ++j) pose[j] = T0[12 * i + j];
    se3_apply_left(xi + 6 * i, pose);
    for (int j = 0; j < 12; ++j) out[12 * i + j] = pose[j];
}

inline int adj_groups(const gsdf_camera& cam) {
    const int n = ceil_div(cam.width, kAdjTile) * ceil_div(cam.height, kAdjTile);
    return n < kAdjMaxGroups ? n : kAdjMaxGroups;
}

inline AdjArgs adj_args(const gsdf_map& map, const gsdf_camera& cam, float delta, int32_t freeze,
                        int64_t param_blocks) {
    AdjArgs a;
    a.W = cam.width;
    a.H = cam.height;
    a.groups = adj_groups(cam);
    a.freeze = freeze;
    a.fx = cam.fx;
    a.fy = cam.fy;
    a.ifx = 1.0 / cam.fx;
    a.ify = 1.0 / cam.fy;
    a.cx = cam.cx;
    a.cy = cam.cy;
    a.zmin = cam.zmin;
    a.zmax = cam.zmax;
    a.delta = delta;
    a.pad = 0.0f;
    a.vs = map.desc.voxel_size;
    a.inv_vs = 1.0 / map.desc.voxel_size;
    a.param_blocks = param_blocks;
    return a;
}

}  // namespace gsdf

using namespace gsdf;

extern "C" {

size_t gsdf_keyframe_scratch_bytes(const gsdf_camera* cam, int32_t n_keyframes, int64_t param_blocks) {
    if (!valid_cam(cam) || n_keyframes <= 0 || n_keyframes > 65535 || param_blocks < 0) return 0;
    const int64_t tiles = adj_tiles(cam->width, cam->height);
    if ((int64_t)n_keyframes * tiles * kTilePx > (int64_t)INT32_MAX) return 0;   // list entries are int32
    return adj_scratch(n_keyframes, tiles, param_blocks).split_total;
}

static int keyframe_common(const gsdf_map* map, const float* depth_dev, int32_t K, const gsdf_camera* cam,
                           const double* T0_dev, const double* xi_dev, const float* params_dev,
                           int64_t param_blocks, float huber_delta, void* scratch, size_t scratch_bytes) {
    if (!valid_map(map) || !valid_cam(cam) || K <= 0 || K > 65535 || !depth_dev || !T0_dev || !xi_dev ||
        !params_dev || param_blocks < 0 || param_blocks > map->desc.max_blocks || !(huber_delta > 0.0f) || !scratch)
        return GSDF_EINVAL;
    if (gsdf_keyframe_scratch_bytes(cam, K, param_blocks) == 0 ||
        scratch_bytes < adj_scratch(K, adj_tiles(cam->width, cam->height), param_blocks).total)
        return GSDF_EINVAL;
    if (!has_gradients(map)) return GSDF_EINVAL;
    return GSDF_OK;
}

int gsdf_keyframe_loss(const gsdf_map* map, const float* depth_dev, int32_t n_keyframes, const gsdf_camera* cam,
                       const double* T0_dev, const double* xi_dev, const float* params_dev, int64_t param_blocks,
                       float huber_delta, int32_t* assoc_dev, int32_t freeze, double* loss_dev, double* count_dev,
                       void* scratch, size_t scratch_bytes, void* stream) {
    int rc = keyframe_common(map, depth_dev, n_keyframes, cam, T0_dev, xi_dev, params_dev, param_blocks,
                             huber_delta, scratch, scratch_bytes);
    if (rc != GSDF_OK) return rc;
    if (!loss_dev || (freeze && !assoc_dev)) return GSDF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const AdjArgs a = adj_args(*map, *cam, huber_delta, freeze, param_blocks);
    const AdjScratch L = adj_scratch(n_keyframes, adj_tiles(cam->width, cam->height), param_blocks);
    char* base = (char*)scratch;
    double* partials = (double*)(base + L.partials);
    double* poses = (double*)(base + L.poses);
    k_adj_setup<<<ceil_div(n_keyframes, 64), 64, 0, s>>>(n_keyframes, T0_dev, xi_dev, poses, 0, nullptr,
                                                        nullptr, nullptr);
    {
        TimedLaunch tl(map->timer, GSDF_K_LOSS, s);
        const dim3 grid(a.groups, n_keyframes);
        const float4* P = reinterpret_cast<const float4*>(params_dev);
        if (freeze)
            k_keyframe_loss<true><<<grid, kAdjBlock, 0, s>>>(make_view(*map), a, depth_dev, poses, P, assoc_dev,
                                                             partials);
        else
            k_keyframe_loss<false><<<grid, kAdjBlock, 0, s>>>(make_view(*map), a, depth_dev, poses, P, assoc_dev,
                                                              partials);
    }
    k_keyframe_finish<kAdjMaxGroups><<<n_keyframes, kAdjMaxGroups, 0, s>>>(a.groups, xi_dev, partials, loss_dev, nullptr, count_dev);
    return launch_status();
}

int gsdf_backward(const gsdf_map* map, const float* depth_dev, int32_t n_keyframes,
                  const gsdf_camera* cam, const double* T0_dev, const double* xi_dev, const float* params_dev,
                  int64_t param_blocks, float huber_delta, int32_t* assoc_dev, int32_t freeze,
                  const float* grad_loss_dev, float* dparams_dev, double* dxi_dev, double* loss_dev, void* scratch,
                  size_t scratch_bytes, void* stream) {
    int rc = keyframe_common(map, depth_dev, n_keyframes, cam, T0_dev, xi_dev, params_dev, param_blocks,
                             huber_delta, scratch, scratch_bytes);
    if (rc != GSDF_OK) return rc;
    if (!grad_loss_dev || !dparams_dev || !dxi_dev || (freeze && !assoc_dev)) return GSDF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int K = n_keyframes;
    const int64_t ntiles = adj_tiles(cam->width, cam->height);
    const AdjArgs a = adj_args(*map, *cam, huber_delta, freeze, param_blocks);
    const AdjScratch L = adj_scratch(K, ntiles, param_blocks);
    char* base = (char*)scratch;
    double* partials = (double*)(base + L.partials);
    double* poses = (double*)(base + L.poses);
    double* bounds = (double*)(base + L.bounds);
    unsigned long long* reach = (unsigned long long*)bounds;
    uint2* list = (uint2*)(base + L.list);
    int2* recs = (int2*)(base + L.recs);
    int32_t* nrec = (int32_t*)(base + L.nrec);
    int2* runs = (int2*)(base + L.runs);
    unsigned long long* tally = (unsigned long long*)(base + L.tally);
    const uint2* tallied = (const uint2*)tally;
    int32_t* run_off = (int32_t*)(base + L.run_off);
    int32_t* tiles = (int32_t*)(base + L.tiles);
    const MapView M = make_view(*map);
    const float4* P = reinterpret_cast<const float4*>(params_dev);
    const int64_t nb = param_blocks;
    const int nscan = (int)ceil_div(nb, (int64_t)kScanTile);
    // room for the gather's pieces: else every block whole
    const bool split = scratch_bytes >= L.split_total;
    const int32_t piece = split ? L.piece : 0;
    int32_t* piece_tiles = (int32_t*)(base + L.tile_sums);
    int4* items = split ? (int4*)(base + L.items) : nullptr;
    int32_t* done = split ? (int32_t*)(base + L.done) : nullptr;
    unsigned long long* buffers = split ? (unsigned long long*)(base + L.buffers) : nullptr;
    const int64_t groups = split ? nb + L.n_buffers : nb;
    const int32_t tiles_x = (cam->width + kAdjTile - 1) / kAdjTile;
    const int64_t setup_n = nb > K ? nb : K;
    const dim3 pgrid(a.groups, K);
    {
        TimedLaunch tl(map->timer, GSDF_K_BACKWARD, s);
        k_adj_setup<<<(unsigned)ceil_div(setup_n, (int64_t)256), 256, 0, s>>>(K, T0_dev, xi_dev, poses, nb, tally, done,
                                                                           reach);
        if (freeze)
            k_adj_pixels<true><<<pgrid, kAdjBlock, 0, s>>>(M, a, depth_dev, poses, P, grad_loss_dev, assoc_dev, list,
                                                           recs, nrec, tally, reach, partials);
        else
            k_adj_pixels<false><<<pgrid, kAdjBlock, 0, s>>>(M, a, depth_dev, poses, P, grad_loss_dev, nullptr, list,
                                                            recs, nrec, tally, reach, partials);
        if (nb > 0) {
            if (nscan > 1) k_adj_tile_sums<<<nscan, 256, 0, s>>>(nb, tallied, piece, tiles, piece_tiles);
            k_adj_offsets<<<nscan, kScanBlock, 0, s>>>(nb, tallied, nscan > 1 ? tiles : nullptr, run_off, K,
                                                       grad_loss_dev, bounds, piece, piece_tiles, items);
            const int64_t regions = (int64_t)K * ntiles;
            k_adj_runs<<<(unsigned)ceil_div(regions, (int64_t)4), 256, 0, s>>>(regions, nrec, recs, run_off, runs);
            if (freeze)
                k_backward_gather<true><<<(unsigned)groups, kAdjBlock, 0, s>>>(
                    M, a, (int32_t)ntiles, tiles_x, poses, P, grad_loss_dev, assoc_dev, list, runs, tallied,
                    run_off, bounds, items, done, buffers, dparams_dev);
            else
                k_backward_gather<false><<<(unsigned)groups, kAdjBlock, 0, s>>>(
                    M, a, (int32_t)ntiles, tiles_x, poses, P, grad_loss_dev, nullptr, list, runs, tallied,
                    run_off, bounds, items, done, buffers, dparams_dev);
        }
        k_keyframe_finish<kAdjMaxGroups><<<K, kAdjMaxGroups, 0, s>>>(a.groups, xi_dev, partials, loss_dev, dxi_dev, nullptr);
    }
    return launch_status();
}

int gsdf_export_params(const gsdf_map* map, float* params_dev, int64_t param_blocks, void* stream) {
    if (!valid_map(map) || !params_dev || param_blocks < 0 || param_blocks > map->desc.max_blocks ||
        !has_gradients(map))
        return GSDF_EINVAL;
    if (param_blocks == 0) return GSDF_OK;
    k_export_params<<<2048, 256, 0, (hipStream_t)stream>>>(make_view(*map), map->desc.storage, param_blocks,
                                                           reinterpret_cast<float4*>(params_dev));
    return launch_status();
}

int gsdf_import_params(gsdf_map* map, const float* params_dev, int64_t param_blocks, void* stream) {
    if (!valid_map(map) || !params_dev || param_blocks < 0 || param_blocks > map->desc.max_blocks ||
        !has_gradients(map))
        return GSDF_EINVAL;
    if (param_blocks == 0) return GSDF_OK;
    k_import_params<<<2048, 256, 0, (hipStream_t)stream>>>(make_view(*map), map->desc.storage, param_blocks,
                                                           reinterpret_cast<const float4*>(params_dev));
    return launch_status();
}

int gsdf_compose_poses(int32_t n, const double* T0_dev, const double* xi_dev, double* T_out_dev, void* stream) {
    if (n < 0 || (n > 0 && (!T0_dev || !xi_dev || !T_out_dev))) return GSDF_EINVAL;
    if (n == 0) return GSDF_OK;
    k_compose_poses<<<ceil_div(n, 64), 64, 0, (hipStream_t)stream>>>(n, T0_dev, xi_dev, T_out_dev);
    return launch_status();
}

int gsdf_voxel_order(int32_t order_out[512]) {
    if (!order_out) return GSDF_EINVAL;
    for (int c = 0; c < kBlockVoxels; ++c) order_out[c] = morton9(c & 7, (c >> 3) & 7, c >> 6);
    return GSDF_OK;
}

}  // extern "C"
