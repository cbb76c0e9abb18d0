// Oriented point cloud from the map (Sec. 4.3).
//
// Every observed voxel whose surface point lies inside its cell
// (|psi_j gh_jk| <= v_s/2 for each axis k) gives the point v_j - psi_j gh_j
// with normal -gh_j (gh points into the solid, so -gh faces free space).
// Upsampled (level 1): each voxel is split into 2x2x2 subvoxels with centres
// s = v_j + (v_s/4)(+-1, +-1, +-1); the Taylor expansion of the distance,
// psi(s) = psi_j + gh_j . (s - v_j), decides (|psi(s) gh_jk| <= v_s/4) and
// places the point s - psi(s) gh_j.  Selection is decided in float64 from the
// stored values; points and normals are written as float32.
//
// Three passes give a deterministic order (block slot, then voxel
// lx + 8 ly + 64 lz, then subvoxel sx + 2 sy + 4 sz): per-block counts, an
// exclusive scan over the blocks, and the write at the scanned offsets.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "gsdf.h"
#include "gsdf_common.hpp"
#include "gsdf_host.hpp"

namespace gsdf {

constexpr int kSurfBlock = 256;

// Stored distance and unit gradient of voxel vi; false when unobserved, and
// for a distance beyond kFar voxels, which no surfel comes from: the largest
// |gh_k| is at least 1/sqrt(3), so |psi gh_k| <= v_s/2 needs |psi| <= 0.8661
// v_s, and a subvoxel's |psi(s) gh_k| <= v_s/4 needs |psi(s)| <= 0.4331 v_s,
// whose psi(s) lies within 0.4331 v_s of psi.  Most voxels of a block are
// further off, and the square root and the three divisions in float64 are
// what the voxel costs.
constexpr double kFar = 0.875;

__device__ inline bool stored_voxel(const MapView& M, int storage, int64_t vi, double* psi, double gh[3]) {
    float p, g[3];
    if (!(load_voxel(M, storage, vi, &p, g) > 0.0f)) return false;
    if (fabs((double)p) > kFar * M.voxel_size_d) return false;
    const double ng = sqrt((double)g[0] * g[0] + (double)g[1] * g[1] + (double)g[2] * g[2]);
    if (!(ng > 0.0)) return false;
    for (int k = 0; k < 3; ++k) gh[k] = g[k] / ng;
    *psi = p;
    return true;
}

// Surfels of voxel c = lx + 8 ly + 64 lz of block `slot`: bit mask of the
// subvoxels taking part (bit 0 for level 0).
__device__ inline unsigned voxel_surfels(const MapView& M, int storage, int level, int64_t slot, int c, double* psi,
                                         double gh[3]) {
    const int64_t vi = slot * kBlockVoxels + morton9(c & 7, (c >> 3) & 7, c >> 6);
    if (!stored_voxel(M, storage, vi, psi, gh)) return 0u;
    const double vs = M.voxel_size_d;
    if (level == 0) {
        bool in = true;
        for (int k = 0; k < 3; ++k) in = in && fabs(*psi * gh[k]) <= 0.5 * vs;
        return in ? 1u : 0u;
    }
    unsigned mask = 0u;
    for (int sub = 0; sub < 8; ++sub) {
        double ps = *psi;
        for (int k = 0; k < 3; ++k) ps += gh[k] * (((sub >> k) & 1) ? 0.25 * vs : -0.25 * vs);
        bool in = true;
        for (int k = 0; k < 3; ++k) in = in && fabs(ps * gh[k]) <= 0.25 * vs;
        if (in) mask |= 1u << sub;
    }
    return mask;
}

// Block-wide exclusive scan of one int per thread (256 threads).
__device__ inline int block_exclusive_scan(int x, int* total, int* s_warp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int incl = wave_scan(x);
    if (lane == 63) s_warp[wave] = incl;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += s_warp[w];
    *total = s_warp[0] + s_warp[1] + s_warp[2] + s_warp[3];
    __syncthreads();
    return base + incl - x;
}

// PASS 0: count per block; PASS 1: write at offsets[slot].  The write pass
// lists a block's surfels (voxel and subvoxel, in order) in LDS beside their
// voxels' distance and gradient, then takes one surfel to a lane: the stores
// of a wave are consecutive, and no lane waits for another's subvoxels.  (A
// voxel to a lane, its subvoxels one after the other with ten scattered
// stores each: 21 us at the 640x480 map's upsampled cloud, this 13; counting
// without kFar 10, with it 9.)
template <int PASS>
__global__ __launch_bounds__(kSurfBlock) void k_surfels(MapView M, int storage, int level, int32_t* __restrict__ counts,
                                                        const int64_t* __restrict__ offsets, int64_t capacity,
                                                        float* __restrict__ points, float* __restrict__ normals,
                                                        int32_t* __restrict__ ids) {
    __shared__ int s_warp[4];
    __shared__ double s_vox[4][PASS == 1 ? kBlockVoxels : 1];              // psi, gh
    __shared__ unsigned short s_list[PASS == 1 ? 8 * kBlockVoxels : 1];   // voxel | subvoxel << 9
    const int32_t nb = M.counters[kNumBlocks] < M.max_blocks ? M.counters[kNumBlocks] : M.max_blocks;
    const bool wide = (reinterpret_cast<uintptr_t>(ids) & 15) == 0;   // else only int32's alignment
    for (int64_t slot = blockIdx.x; slot < nb; slot += gridDim.x) {
        int block_total = 0;
        // two voxels per thread, in voxel order lx + 8 ly + 64 lz
        for (int half = 0; half < 2; ++half) {
            const int c = half * kSurfBlock + threadIdx.x;
            double psi, gh[3];
            unsigned mask = voxel_surfels(M, storage, level, slot, c, &psi, gh);
            int total;
            int at = block_total + block_exclusive_scan(__popc(mask), &total, s_warp);
            if (PASS == 1 && mask) {
                s_vox[0][c] = psi;
                for (int k = 0; k < 3; ++k) s_vox[1 + k][c] = gh[k];
                for (; mask; mask &= mask - 1) s_list[at++] = (unsigned short)(c | ((__ffs((int)mask) - 1) << 9));
            }
            block_total += total;
        }
        if (PASS == 0) {
            if (threadIdx.x == 0) counts[slot] = block_total;
            continue;
        }
        __syncthreads();
        const int64_t base = offsets[slot];
        int b[3];
        unpack_key(M.block_keys[slot], &b[0], &b[1], &b[2]);
        for (int i = threadIdx.x; i < block_total; i += kSurfBlock) {
            const int64_t o = base + i;
            if (o >= capacity) break;
            const int c = s_list[i] & (kBlockVoxels - 1), sub = s_list[i] >> 9;
            const int id[3] = {8 * b[0] + (c & 7), 8 * b[1] + ((c >> 3) & 7), 8 * b[2] + (c >> 6)};
            double gh[3], s[3], ps = s_vox[0][c];
            for (int a = 0; a < 3; ++a) {
                gh[a] = s_vox[1 + a][c];
                s[a] = M.voxel_size_d * id[a];
            }
            if (level == 1) {
                for (int a = 0; a < 3; ++a) {
                    const double d = ((sub >> a) & 1) ? 0.25 * M.voxel_size_d : -0.25 * M.voxel_size_d;
                    s[a] += d;
                    ps += gh[a] * d;
                }
            }
            for (int a = 0; a < 3; ++a) {
                points[3 * o + a] = (float)(s[a] - ps * gh[a]);
                normals[3 * o + a] = (float)(-gh[a]);
            }
            if (wide) {
                reinterpret_cast<int4*>(ids)[o] = make_int4(id[0], id[1], id[2], sub);
            } else {
                for (int a = 0; a < 3; ++a) ids[4 * o + a] = id[a];
                ids[4 * o + 3] = sub;
            }
        }
        __syncthreads();   // the list is the next block's
    }
}

// Exclusive scan of the per-block counts (one work-group) and the total.
__global__ __launch_bounds__(1024) void k_surfel_scan(MapView M, const int32_t* __restrict__ counts,
                                                      int64_t* __restrict__ offsets, int64_t* __restrict__ total) {
    __shared__ int64_t s_part[1024];
    const int32_t nb = M.counters[kNumBlocks] < M.max_blocks ? M.counters[kNumBlocks] : M.max_blocks;
    const int per = (nb + 1023) / 1024;
    const int64_t lo = (int64_t)threadIdx.x * per;
    int64_t sum = 0;
    for (int64_t i = lo; i < lo + per && i < nb; ++i) sum += counts[i];
    s_part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int64_t y = threadIdx.x >= off ? s_part[threadIdx.x - off] : 0;
        __syncthreads();
        s_part[threadIdx.x] += y;
        __syncthreads();
    }
    int64_t run = s_part[threadIdx.x] - sum;
    for (int64_t i = lo; i < lo + per && i < nb; ++i) {
        offsets[i] = run;
        run += counts[i];
    }
    if (threadIdx.x == 1023) *total = s_part[1023];
}

}  // namespace gsdf

using namespace gsdf;

extern "C" {

size_t gsdf_surfel_scratch_bytes(const gsdf_map* map) {
    if (!valid_map(map)) return 0;
    return (size_t)map->desc.max_blocks * (sizeof(int32_t) + sizeof(int64_t)) + 256;
}

int gsdf_extract_surfels(const gsdf_map* map, int32_t level, float* points_dev, float* normals_dev, int32_t* ids_dev,
                         int64_t capacity, int64_t* count_dev, void* scratch_dev, size_t scratch_bytes, void* stream) {
    if (!valid_map(map) || !has_gradients(map) || (level != 0 && level != 1) || capacity < 0 || !count_dev ||
        !scratch_dev ||
        scratch_bytes < gsdf_surfel_scratch_bytes(map) ||
        (capacity > 0 && (!points_dev || !normals_dev || !ids_dev)))
        return GSDF_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const MapView M = make_view(*map);
    int64_t* offsets = (int64_t*)scratch_dev;
    int32_t* counts = (int32_t*)((char*)scratch_dev + (size_t)map->desc.max_blocks * sizeof(int64_t));
    const unsigned grid = 2048;
    k_surfels<0><<<grid, kSurfBlock, 0, s>>>(M, map->desc.storage, level, counts, nullptr, 0, nullptr, nullptr,
                                             nullptr);
    k_surfel_scan<<<1, 1024, 0, s>>>(M, counts, offsets, count_dev);
    if (capacity > 0)
        k_surfels<1><<<grid, kSurfBlock, 0, s>>>(M, map->desc.storage, level, counts, offsets, capacity, points_dev,
                                                 normals_dev, ids_dev);
    return launch_status();
}

}  // extern "C"
