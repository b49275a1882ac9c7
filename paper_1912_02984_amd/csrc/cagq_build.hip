// Voxelization and the occupied-voxel index (Appendix D, CAGQ general
// procedure, step 1; Sec. 3.2 "voxelize the input space ... map each point to
// a voxel index ... store up to n_v points in each voxel").
//
// Design (gfx950): the set O_v of non-empty voxels is an occupancy bitmap
// with one bit per grid voxel; a voxel's slot is its rank (popcount of the
// bits before it), which is a minimal, order-preserving hash of the linear
// voxel id to a compact slot. Points mark a byte per voxel with plain stores
// (no atomics); two kernels pack the bytes into bitmap words and rank them;
// counts come from one atomic per point,
// offsets from a look-back scan over the slots. Per-voxel lists hold
// the n_v lowest point indices in ascending order, independent of the
// arrival order the atomics produce: small voxels rank each point against
// the voxel's bucket, large voxels are reduced by a wavefront bitonic
// selection.
#include "cagq_internal.h"

namespace cagq {

namespace {

struct GridArgs {
    float o[3];
    float s[3];
    int32_t D[3];
};

GridArgs grid_args(const cagq_grid_desc& d) {
    GridArgs g;
    for (int a = 0; a < 3; ++a) {
        g.o[a] = d.origin[a];
        g.s[a] = d.voxel_size[a];
        g.D[a] = d.dims[a];
    }
    return g;
}

__global__ void k_clear(uint4* __restrict__ p, size_t n16) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// One lane per point: linear voxel id, occupancy byte.
__global__ __launch_bounds__(256) void k_mark(const float* __restrict__ P, int32_t N, int32_t BN,
                                              GridArgs g, int64_t W, uint32_t* __restrict__ pt_lin,
                                              uint8_t* __restrict__ bytemap, int* __restrict__ status) {
    int32_t gid = (int32_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (gid >= BN) return;
    int32_t b = gid / N;
    const float* p = P + (size_t)gid * 3;
    float c[3] = {p[0], p[1], p[2]};
    uint32_t gg[3];
    bool bad = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!isfinite(c[a])) {
            bad = true;
            gg[a] = 0;
        } else {
            gg[a] = (uint32_t)axis_index(c[a], g.o[a], g.s[a], g.D[a]);
        }
    }
    uint32_t lin = gg[0] + (uint32_t)g.D[0] * (gg[1] + (uint32_t)g.D[1] * gg[2]);
    pt_lin[gid] = lin;
    // every point of a voxel stores the same byte: no atomic is needed
    bytemap[(size_t)b * W * 64 + lin] = 1;
    if (bad) raise_error(status, CAGQ_ERR_NONFINITE_INPUT);
}

// 64 occupancy bytes (each 0 or 1) to one occupancy word: byte j -> bit j.
// Multiplying 4 such bytes by 0x01020408 moves byte k to bit 24 + k with no
// other term reaching bits 24..31.
__device__ __forceinline__ uint64_t pack_bytes(const uint4* __restrict__ p) {
    uint64_t r = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 v = p[q];
        const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) r |= (uint64_t)((a[k] * 0x01020408u) >> 24) << (16 * q + 4 * k);
    }
    return r;
}

// Occupancy words from the bytes, one word per thread, and the occupied voxels
// of each tile of kRankTile words and (device atomics on zeroed words, one per
// tile) of each group of kRankGroup tiles. With k_rank this replaces a
// look-back scan, whose tiles numbered themselves by tickets from one address:
// at about 20 ns a ticket the 1296 tiles of a 2^20-point sweep (802 x 802 x 33
// voxels) took 30 us, and 27 us with four words a thread, where a lane then
// lists four words' voxels in series; the two kernels take half (the sweep's
// layer: 236 -> 226 us).
__global__ __launch_bounds__(kScanThreads) void k_pack(const uint8_t* __restrict__ bytemap,
                                                       uint64_t* __restrict__ bitmap, int64_t W, int64_t tiles_w,
                                                       uint32_t* __restrict__ tile_cnt,
                                                       uint32_t* __restrict__ group_cnt) {
    __shared__ uint32_t s_wave[kScanThreads / kWave];
    const int32_t b = (int32_t)(blockIdx.x / tiles_w);
    const int64_t tile = (int64_t)(blockIdx.x % tiles_w);
    const int64_t w = tile * kRankTile + threadIdx.x;
    uint64_t word = 0;
    if (w < W) {
        word = pack_bytes(reinterpret_cast<const uint4*>(bytemap + (size_t)b * W * 64) + (size_t)w * 4);
        bitmap[(size_t)b * W + w] = word;
    }
    const uint32_t n = wave_sum_u32((uint32_t)__popcll(word));
    if (lane_id() == 0) s_wave[threadIdx.x / kWave] = n;
    lds_barrier();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
#pragma unroll
        for (int i = 0; i < kScanThreads / kWave; ++i) t += s_wave[i];
        tile_cnt[(size_t)b * tiles_w + tile] = t;
        if (t) atomicAdd(&group_cnt[(size_t)b * (tiles_w / kRankGroup + 1) + tile / kRankGroup], t);
    }
}

// Ranks of the occupancy words: word_rank[w] = occupied voxels before word w,
// from the groups and the tiles before this one. Also lists every occupied
// voxel's linear id at its slot and clears its count.
__global__ __launch_bounds__(kScanThreads) void k_rank(
    const uint64_t* __restrict__ bitmap, int64_t W, int64_t tiles_w, int32_t N,
    const uint32_t* __restrict__ tile_cnt, const uint32_t* __restrict__ group_cnt, uint32_t* __restrict__ word_rank,
    uint32_t* __restrict__ vox_lin, uint32_t* __restrict__ vox_count, int32_t* __restrict__ nvox) {
    __shared__ uint64_t s_wave[kScanThreads / kWave];
    const int32_t b = (int32_t)(blockIdx.x / tiles_w);
    const int64_t tile = (int64_t)(blockIdx.x % tiles_w);
    const int64_t w = tile * kRankTile + threadIdx.x;
    uint64_t m = w < W ? bitmap[(size_t)b * W + w] : 0ull;
    const int64_t g = tile / kRankGroup;
    const uint32_t* gc = group_cnt + (size_t)b * (tiles_w / kRankGroup + 1);
    uint32_t before = 0;
    for (int64_t i = threadIdx.x; i < g; i += kScanThreads) before += gc[i];
    const int64_t t0 = g * kRankGroup;
    if (threadIdx.x < tile - t0) before += tile_cnt[(size_t)b * tiles_w + t0 + threadIdx.x];
    // both sums in one scan: occupied voxels before the tile << 32 | of the tile
    uint64_t total;
    const uint64_t mine = ((uint64_t)before << 32) | (uint32_t)__popcll(m);
    const uint64_t excl = block_excl_scan(mine, s_wave, &total);
    uint32_t r = (uint32_t)(total >> 32) + (uint32_t)excl;
    if (tile == tiles_w - 1 && threadIdx.x == 0) nvox[b] = (int32_t)((uint32_t)(total >> 32) + (uint32_t)total);
    if (w >= W) return;
    word_rank[(size_t)b * W + w] = r;
    uint32_t* vl = vox_lin + (size_t)b * N;
    uint32_t* vc = vox_count + (size_t)b * N;
    for (; m; m &= m - 1, ++r) {
        vl[r] = (uint32_t)(w * 64 + __ffsll((unsigned long long)m) - 1);
        vc[r] = 0u;
    }
}

// One lane per point: slot (rank of its voxel) and arrival position.
__global__ __launch_bounds__(256) void k_count(int32_t BN, int32_t N, int64_t W,
                                               const uint64_t* __restrict__ bitmap,
                                               const uint32_t* __restrict__ word_rank,
                                               uint32_t* __restrict__ pt_slot, uint32_t* __restrict__ pt_pos,
                                               uint32_t* __restrict__ vox_count) {
    const int32_t gid = (int32_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const bool active = gid < BN;  // a prefix of the wave
    const int32_t b = active ? gid / N : 0;
    const uint32_t lin = active ? pt_slot[gid] : 0u;
    const uint32_t slot = active ? (uint32_t)slot_of(bitmap + (size_t)b * W, word_rank + (size_t)b * W, lin) : 0u;
    // Adjacent lanes with the same voxel (runs of one voxel's points, as in
    // a scan-ordered cloud) take their arrival positions with one atomic per
    // run: the positions within a voxel are a permutation either way.
    const size_t gs = (size_t)b * N + slot;
    const int lane = lane_id();
    const uint64_t prev = shfl_up64((uint64_t)gs, 1);
    const bool head = active && (lane == 0 || prev != (uint64_t)gs);
    const uint64_t heads = __ballot(head);
    const uint32_t n_act = (uint32_t)__popcll(__ballot(active));
    const uint64_t upto = lane == kWave - 1 ? ~0ull : ((2ull << lane) - 1);  // lanes <= this one
    const int h = active ? 63 - __clzll(heads & upto) : lane;  // the head of this lane's run
    uint32_t pos0 = 0;
    if (head) {
        const uint64_t next = heads & ~upto;
        const uint32_t end = next ? (uint32_t)(__ffsll((unsigned long long)next) - 1) : n_act;
        pos0 = atomicAdd(&vox_count[gs], end - (uint32_t)lane);
    }
    pos0 = (uint32_t)__shfl((int)pos0, h, kWave);
    if (!active) return;
    pt_slot[gid] = slot;
    pt_pos[gid] = pos0 + (uint32_t)(lane - h);
}

// Offsets: vox_off = exclusive prefix of min(count, n_v), full_off = exclusive
// prefix of count, over the slots [0, nvox[b]) of each cloud; entry nvox[b]
// holds the totals. Both are scanned at once, packed as (full << 31) | stored.
__global__ __launch_bounds__(kScanThreads) void k_offsets(
    int32_t B, int32_t N, int64_t tiles_s, uint32_t n_v, const int32_t* __restrict__ nvox,
    const uint32_t* __restrict__ vox_count, uint32_t* __restrict__ vox_off, uint32_t* __restrict__ full_off,
    uint64_t* __restrict__ desc_s, int* __restrict__ status, uint32_t* __restrict__ big, int64_t big_cap) {
    __shared__ uint32_t s_ticket;
    __shared__ uint64_t s_wave[kScanThreads / kWave];
    __shared__ uint64_t s_prefix;
    int32_t b;
    int64_t tile;
    if (!slot_tile(B, tiles_s, kScanTile, nvox, (unsigned*)&status[kStTicketOff], &s_ticket, b, tile)) return;
    const int64_t nv = nvox[b];
    const int64_t s0 = tile * kScanTile + (int64_t)threadIdx.x * kScanItems;
    const uint32_t* vc = vox_count + (size_t)b * N;
    uint32_t cnt[kScanItems];
    uint64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t s = s0 + i;
        cnt[i] = s < nv ? vc[s] : 0u;
        uint32_t st = cnt[i] < n_v ? cnt[i] : n_v;
        sum += ((uint64_t)cnt[i] << 31) | st;
        if (cnt[i] > kBigVoxel) {
            uint32_t k = atomicAdd((unsigned*)&status[kStBigCount], 1u);
            if ((int64_t)k < big_cap) big[k] = (uint32_t)((size_t)b * N + s);
        }
    }
    uint64_t total;
    uint64_t excl = block_excl_scan(sum, s_wave, &total);
    uint64_t run = tile_lookback(desc_s + (size_t)b * tiles_s, tile, total, &s_prefix) + excl;
    uint32_t* vo = vox_off + (size_t)b * (N + 1);
    uint32_t* fo = full_off + (size_t)b * (N + 1);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t s = s0 + i;
        if (s > nv) break;
        vo[s] = (uint32_t)(run & 0x7FFFFFFFu);
        fo[s] = (uint32_t)(run >> 31);
        if (s < nv) {
            uint32_t st = cnt[i] < n_v ? cnt[i] : n_v;
            run += ((uint64_t)cnt[i] << 31) | st;
        }
    }
    // the slot nvox sits in the next tile when nvox is a multiple of the tile size
    if (threadIdx.x == 0 && nv == (tile + 1) * kScanTile) {
        uint64_t end = s_prefix + total;
        vo[nv] = (uint32_t)(end & 0x7FFFFFFFu);
        fo[nv] = (uint32_t)(end >> 31);
    }
}

// One lane per point: its index into the bucket of its slot.
__global__ __launch_bounds__(256) void k_scatter(int32_t BN, int32_t N, const uint32_t* __restrict__ pt_slot,
                                                 const uint32_t* __restrict__ pt_pos,
                                                 const uint32_t* __restrict__ full_off,
                                                 uint32_t* __restrict__ bucket) {
    int32_t gid = (int32_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (gid >= BN) return;
    int32_t b = gid / N;
    uint32_t slot = pt_slot[gid];
    bucket[(size_t)b * N + full_off[(size_t)b * (N + 1) + slot] + pt_pos[gid]] = (uint32_t)(gid - b * N);
}

// Stored lists. Blocks [0, big_blocks): one wave per voxel of more than
// kBigVoxel points -- the n_v smallest indices by bitonic selection in 64-key
// chunks; first, since these waves are the longest. The others: one lane per
// point of a smaller voxel -- its rank among the voxel's indices places it,
// eight of them loaded at a time. 2^20-point sweep (3633 larger voxels of up to
// 438 points) with 64-bit keys, permutes and these waves last: 42 us; the layer
// 227 -> 215 us.
__global__ __launch_bounds__(256) void k_finalize(
    const float* __restrict__ P, int32_t BN, int32_t N, uint32_t n_v, int32_t big_blocks,
    const uint32_t* __restrict__ pt_slot, const uint32_t* __restrict__ vox_count,
    const uint32_t* __restrict__ vox_off, const uint32_t* __restrict__ full_off,
    const uint32_t* __restrict__ bucket, const uint32_t* __restrict__ big, int64_t big_cap,
    const int* __restrict__ status, uint32_t* __restrict__ pt_list, float4* __restrict__ pt4) {
    if ((int32_t)blockIdx.x >= big_blocks) {
        int32_t gid = (int32_t)xcd_block(blockIdx.x - big_blocks, gridDim.x - big_blocks) * blockDim.x + threadIdx.x;
        if (gid >= BN) return;
        int32_t b = gid / N;
        uint32_t i = (uint32_t)(gid - b * N);
        uint32_t slot = pt_slot[gid];
        size_t sg = (size_t)b * N + slot;
        uint32_t cnt = vox_count[sg];
        if (cnt > kBigVoxel) return;
        const uint32_t* bk = bucket + (size_t)b * N + full_off[(size_t)b * (N + 1) + slot];
        uint32_t rank = 0;
        for (uint32_t j = 0; j < cnt; j += 8) {
            uint32_t x[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) x[u] = bk[j + u < cnt ? j + u : j];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) rank += j + u < cnt && x[u] < i ? 1u : 0u;
        }
        if (rank < n_v) {
            size_t dst = (size_t)b * N + vox_off[(size_t)b * (N + 1) + slot] + rank;
            const float* p = P + (size_t)gid * 3;
            pt_list[dst] = i;
            pt4[dst] = make_float4(p[0], p[1], p[2], __uint_as_float(i));
        }
        return;
    }
    const int lane = lane_id();
    const int32_t nbig = (int64_t)status[kStBigCount] < big_cap ? status[kStBigCount] : (int32_t)big_cap;
    const int32_t wpb = blockDim.x / kWave;
    const int32_t nwaves = big_blocks * wpb;
    for (int32_t v = (int32_t)blockIdx.x * wpb + threadIdx.x / kWave; v < nbig; v += nwaves) {
        uint32_t g = big[v];
        int32_t b = (int32_t)(g / (uint32_t)N);
        uint32_t s = g - (uint32_t)b * N;
        uint32_t cnt = vox_count[g];
        const uint32_t* bk = bucket + (size_t)b * N + full_off[(size_t)b * (N + 1) + s];
        uint32_t best = ~0u, kth = ~0u;
        uint32_t k_n = (uint32_t)lane < cnt ? bk[lane] : ~0u;  // loaded a chunk ahead
        for (uint32_t c0 = 0; c0 < cnt; c0 += kWave) {
            uint32_t k = k_n;
            k_n = (c0 + kWave + lane < cnt) ? bk[c0 + kWave + lane] : ~0u;
            // an index above the n_v-th lowest so far is never kept; a chunk
            // left without any is not sorted
            k = k < kth ? k : ~0u;
            if (c0 != 0 && !__ballot(k != ~0u)) continue;
            k = wave_sort32(k);
            best = c0 == 0 ? k : wave_merge_low32(best, k);
            kth = (uint32_t)__shfl((int)best, (int)n_v - 1, kWave);
        }
        if ((uint32_t)lane < n_v) {
            const uint32_t i = best;
            size_t dst = (size_t)b * N + vox_off[(size_t)b * (N + 1) + s] + lane;
            const float* p = P + ((size_t)b * N + i) * 3;
            pt_list[dst] = i;
            pt4[dst] = make_float4(p[0], p[1], p[2], __uint_as_float(i));
        }
    }
}

// ---- larger clouds: sort the points into bricks, then build each brick.
// A brick is a run of consecutive linear voxel ids (2^wshift occupancy words,
// at most kBrickW: brick_wshift) of one cloud; the batch holds B * Q of them. The points are grouped
// by brick with a counting sort: a histogram per tile of points (one row per
// tile), a scan of each brick's column and of the bricks' totals (by each
// scatter tile itself, or by a launch of its own when a tile would read too
// many entries), a scatter that carries each point's coordinates and index. Then two
// passes over the bricks, a wave per brick (a workgroup for the largest):
// one counts each brick's points per voxel in LDS, which gives its occupancy
// words and its occupied and stored totals; the other sums the totals of the
// cloud's earlier bricks, ranks its occupied voxels by popcount, and places
// the n_v lowest point indices of every voxel. Every output is written once, the work is
// proportional to the points and the occupied voxels, and no global atomic
// is taken per point.
constexpr int kSortT = 1024;                    // threads per sort tile
constexpr int kSortIPT = kSortTile / kSortT;    // points per thread
constexpr int kHGroup = 64;                     // bricks per block of the column scan
constexpr int kBrickIPT = kBrickCap / kBrickT;  // points per thread of a part
constexpr int kLoadIPT = 8;                     // of them, loaded together
constexpr int kWaveIPT = kWavePts / kWave;      // points per lane of a wave's brick
constexpr int kBrickWaves = kBrickT / kWave;    // bricks per block
static_assert(kBrickW <= kWave, "a brick's occupancy words are scanned by one wave");
static_assert(kBrickIPT % kLoadIPT == 0 && kBrickCap < 65536, "a part is loaded in whole steps");
static_assert(kSortTile <= kBrickCap, "a tile's points of one brick fit in one part");
static_assert(kWavePts < kBrickCap && kBrickV % kBrickT == 0, "brick sizes");

// Linear voxel id of a point; `bad` is set for a non-finite coordinate (its
// axis index is then 0).
__device__ __forceinline__ uint32_t voxel_lin(float x, float y, float z, const GridArgs& g, bool& bad) {
    const float c[3] = {x, y, z};
    uint32_t gg[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!isfinite(c[a])) {
            bad = true;
            gg[a] = 0;
        } else {
            gg[a] = (uint32_t)axis_index(c[a], g.o[a], g.s[a], g.D[a]);
        }
    }
    return gg[0] + (uint32_t)g.D[0] * (gg[1] + (uint32_t)g.D[1] * gg[2]);
}

// Row t of the histogram: points of tile t in each brick of the batch (with
// `own`, only the entries of the bricks of the clouds the tile holds points
// of, which are the only ones read then). The blocks also zero the control
// words [clr, clr + n16) (status, tickets, descriptors) that the later
// kernels use.
__global__ __launch_bounds__(kSortT) void k_bhist(const float* __restrict__ P, int32_t N, int32_t BN, GridArgs g,
                                                  int32_t Q, int32_t BQ, int32_t vshift, int32_t T, bool own,
                                                  uint32_t* __restrict__ hist, uint4* __restrict__ clr, int64_t n16) {
    __shared__ uint32_t s_h[kMaxBricks];
    const int tid = threadIdx.x;
    const int32_t t = (int32_t)blockIdx.x;
    const int32_t p0 = t * kSortTile, p1 = p0 + kSortTile < BN ? p0 + kSortTile : BN;
    const int32_t e0 = own ? (p0 / N) * Q : 0, e1 = own ? ((p1 - 1) / N + 1) * Q : BQ;
    for (int32_t i = e0 + tid; i < e1; i += kSortT) s_h[i] = 0u;
    for (int64_t i = (int64_t)t * kSortT + tid; i < n16; i += (int64_t)T * kSortT) clr[i] = make_uint4(0u, 0u, 0u, 0u);
    // the points' coordinates first, all loads in flight together (a load
    // under the bounds test would be waited for before the next is issued)
    float c[kSortIPT][3];
#pragma unroll
    for (int k = 0; k < kSortIPT; ++k) {
        const int32_t gid = p0 + k * kSortT + tid;
        const float* p = P + (size_t)(gid < BN ? gid : 0) * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) c[k][a] = p[a];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < kSortIPT; ++k) {
        const int32_t gid = p0 + k * kSortT + tid;
        if (gid >= BN) break;
        bool bad = false;
        const uint32_t lin = voxel_lin(c[k][0], c[k][1], c[k][2], g, bad);
        atomicAdd(&s_h[(gid / N) * Q + (int32_t)(lin >> vshift)], 1u);
    }
    lds_barrier();
    uint32_t* row = hist + (size_t)t * BQ;
    for (int32_t i = e0 + tid; i < e1; i += kSortT) row[i] = s_h[i];
}

// The work items of the brick passes: a part of a brick of more than
// kWavePts points, for one block.
struct BrickItem {
    uint32_t g;   // the brick
    uint32_t p0;  // the part's first sorted position
    uint32_t n;   // (part << 12) | (its points - 1)
    int32_t hb;   // the heavy brick it is a part of, -1: the whole brick is one part
};

struct BrickLists {
    BrickItem* item;
    uint32_t* hfirst;  // per heavy brick: the count row of its first part
    uint32_t* hparts;  //                  its parts
    uint32_t* pcnt;    // the count rows, nvx (voxels per brick) entries each
    uint32_t nvx;
    int* status;
};

// Lists a brick of more than kWavePts points (brick g at sorted position
// `start`, `tot` points, those of tile t being hist[t * BQ + g], tiles
// [tf, tl]): one item for at most kBrickCap points, otherwise (heavy) parts of
// whole tiles, as many as fit in kBrickCap points. Tiles follow the points'
// order, so every point of an earlier part has a lower index than those of a
// later one, and a point's rank among its voxel's is the voxel's points in
// the earlier parts plus its rank within its own. Every lane of the wave
// calls it; one atomic per wave lists its bricks of one part.
__device__ __forceinline__ void list_big(const BrickLists& o, bool valid, uint32_t g, uint32_t start, uint32_t tot,
                                         const uint32_t* __restrict__ hist, int32_t BQ, int32_t tf, int32_t tl) {
    const bool one = valid && tot > (uint32_t)kWavePts && tot <= (uint32_t)kBrickCap;
    const uint64_t m = __ballot(one);
    if (m) {
        const int first = __ffsll((unsigned long long)m) - 1;
        uint32_t base = 0;
        if (lane_id() == first) base = (uint32_t)atomicAdd(&o.status[kStItems], __popcll(m));
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, first);
        if (one) o.item[base + (uint32_t)__popcll(m & ((1ull << lane_id()) - 1))] = BrickItem{g, start, tot - 1, -1};
    }
    if (!valid || tot <= (uint32_t)kBrickCap) return;
    // count rows for as many parts as there can be (two in a row hold more than
    // kBrickCap points), which keep the parts until their number is known, so
    // that one walk over the column lists them
    const int32_t hb = atomicAdd(&o.status[kStHeavy], 1);
    const uint32_t row = (uint32_t)atomicAdd(&o.status[kStRows], (int)(2ull * tot / kBrickCap) + 1);
    uint32_t* keep = o.pcnt + (size_t)row * o.nvx;
    constexpr int kU = 16;  // column entries in flight
    uint32_t parts = 0, p0 = start, acc = 0;
    auto put = [&]() {
        keep[(size_t)parts * o.nvx] = p0;
        keep[(size_t)parts * o.nvx + 1] = acc;
        ++parts;
    };
    for (int32_t t0 = tf; t0 <= tl; t0 += kU) {
        uint32_t x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = hist[(size_t)(t0 + u <= tl ? t0 + u : tl) * BQ + g];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t v = t0 + u <= tl ? x[u] : 0u;
            if (acc + v > (uint32_t)kBrickCap) {
                put();
                p0 += acc;
                acc = 0;
            }
            acc += v;
        }
    }
    put();
    const uint32_t e = (uint32_t)atomicAdd(&o.status[kStItems], (int)parts);
    o.hfirst[hb] = row;
    o.hparts[hb] = parts;
    for (uint32_t i = 0; i < parts; ++i)
        o.item[e + i] = BrickItem{g, keep[(size_t)i * o.nvx], (i << 12) | (keep[(size_t)i * o.nvx + 1] - 1), hb};
}

// Sorted positions and work items: bstart[g] = points of the bricks before g
// (bricks in cloud-major order), and entry (t, g) of the histogram becomes
// the first position of tile t's points in brick g. A block takes kHGroup
// bricks (one per lane) and splits the tiles over its waves; the blocks'
// totals are chained by a look-back.
__global__ __launch_bounds__(kScanThreads) void k_hscan(uint32_t* hist, int32_t N, int32_t Q, int32_t BQ,
                                                        int32_t T, uint32_t* __restrict__ bstart, BrickLists lists,
                                                        uint64_t* __restrict__ desc, int* __restrict__ status) {
    constexpr int kW = kScanThreads / kWave;
    __shared__ uint32_t s_ticket;
    __shared__ uint32_t s_part[kW][kHGroup];
    __shared__ uint32_t s_bex[kHGroup];
    __shared__ uint64_t s_prefix;
    if (threadIdx.x == 0) s_ticket = atomicAdd((unsigned*)&status[kStTicketHist], 1u);
    __syncthreads();
    const int32_t grp = (int32_t)s_ticket;
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int32_t g = grp * kHGroup + lane;
    const bool valid = g < BQ;
    const int32_t tc = (T + kW - 1) / kW;
    const int32_t t0 = wv * tc, t1 = t0 + tc < T ? t0 + tc : T;
    // the column's first kHKeep entries stay in registers for the rewrite
    constexpr int kHKeep = 16;
    uint32_t col[kHKeep];
    uint32_t sum = 0;
    if (valid) {
#pragma unroll
        for (int j = 0; j < kHKeep; ++j) {
            col[j] = t0 + j < t1 ? hist[(size_t)(t0 + j) * BQ + g] : 0u;
            sum += col[j];
        }
        for (int32_t t = t0 + kHKeep; t < t1; ++t) sum += hist[(size_t)t * BQ + g];
    }
    s_part[wv][lane] = sum;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
        const uint32_t x = s_part[w][lane];
        pre += w < wv ? x : 0u;
        tot += x;
    }
    uint64_t gtot = 0;
    if (wv == 0) {
        const uint32_t x = valid ? tot : 0u;
        const uint32_t incl = wave_incl_scan<uint32_t>(x);
        s_bex[lane] = incl - x;
        gtot = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    }
    const uint64_t P0 = tile_lookback(desc, grp, gtot, &s_prefix);
    const uint32_t base = (uint32_t)P0 + s_bex[lane];
    if (wv == 0) {
        if (valid) bstart[g] = base;
        const int64_t b = valid ? g / Q : 0;
        list_big(lists, valid, (uint32_t)g, base, tot, hist, BQ, (int32_t)(b * N / kSortTile),
                 (int32_t)(((b + 1) * N - 1) / kSortTile));
    }
    __syncthreads();  // the columns are read above and rewritten below
    if (!valid) return;
    uint32_t run = base + pre;
#pragma unroll
    for (int j = 0; j < kHKeep; ++j) {
        if (t0 + j < t1) hist[(size_t)(t0 + j) * BQ + g] = run;
        run += col[j];
    }
    for (int32_t t = t0 + kHKeep; t < t1; ++t) {
        const size_t e = (size_t)t * BQ + g;
        const uint32_t x = hist[e];
        hist[e] = run;
        run += x;
    }
}

// Exclusive scan of one value per thread of a kSortT block; *total receives
// the block sum. Every thread of the block calls it.
__device__ __forceinline__ uint32_t sort_excl_scan(uint32_t v, uint32_t* s_wave, uint32_t* total) {
    const uint32_t incl = wave_incl_scan<uint32_t>(v);
    const int wv = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) s_wave[wv] = incl;
    lds_barrier();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kSortT / kWave; ++i) {
        const uint32_t x = s_wave[i];
        off += i < wv ? x : 0u;
        tot += x;
    }
    lds_barrier();
    *total = tot;
    return off + incl - v;
}

// Column sums of the histogram for brick `col` over the tiles [tf, tl]: the
// brick's points (tot) and those in the tiles before t (pre), kU loads in
// flight per thread.
template <int kU>
__device__ __forceinline__ void brick_column(const uint32_t* __restrict__ hist, int32_t BQ, size_t col, int32_t tf,
                                             int32_t tl, int32_t t, uint32_t& tot, uint32_t& pre) {
    tot = pre = 0;
    for (int32_t t0 = tf; t0 <= tl; t0 += kU) {
        uint32_t x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = hist[(size_t)(t0 + u <= tl ? t0 + u : tl) * BQ + col];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t v = t0 + u <= tl ? x[u] : 0u;
            tot += v;
            pre += t0 + u < t ? v : 0u;
        }
    }
}

// The first sorted position of tile t's points in each brick of the clouds
// it holds points of, into s_o (indexed by brick): per brick, the column of
// the histogram over the cloud's tiles gives the points of the tiles before
// t and the brick's total, and an exclusive scan of the totals over the
// cloud's bricks (clouds hold N sorted positions each) gives the brick's
// first position.
__device__ __forceinline__ void tile_columns(int32_t t, int32_t N, int32_t BN, int32_t Q, int32_t BQ,
                                             const uint32_t* __restrict__ hist, uint32_t* s_o, uint32_t* s_wave) {
    const int32_t p0 = t * kSortTile, p1 = p0 + kSortTile < BN ? p0 + kSortTile : BN;
    for (int32_t b = p0 / N; b <= (p1 - 1) / N; ++b) {
        const int32_t tf = (int32_t)((int64_t)b * N / kSortTile);
        const int32_t tl = (int32_t)((((int64_t)b + 1) * N - 1) / kSortTile);
        uint32_t carry = (uint32_t)b * (uint32_t)N;
        for (int32_t q0 = 0; q0 < Q; q0 += kSortT) {
            const int32_t q = q0 + (int32_t)threadIdx.x;
            uint32_t tot, pre;
            // (32: all of a cloud's, up to 126976 points)
            brick_column<32>(hist, BQ, (size_t)b * Q + (q < Q ? q : 0), tf, tl, t, tot, pre);
            if (q >= Q) tot = 0;
            uint32_t sum;
            const uint32_t start = carry + sort_excl_scan(tot, s_wave, &sum);
            carry += sum;
            if (q < Q) s_o[b * Q + q] = start + pre;
        }
    }
}

// Cloud b's bricks: their first sorted positions (bstart), and the list of
// those of more than kWavePts points. It runs beside the tiles' blocks and ends
// before them; with 16 column loads in flight, not the tiles' 32, it fits in
// their registers.
__device__ __forceinline__ void cloud_columns(int32_t b, int32_t N, int32_t Q, int32_t BQ,
                                              const uint32_t* __restrict__ hist, uint32_t* s_wave,
                                              uint32_t* __restrict__ bstart, const BrickLists& lists) {
    const int32_t tf = (int32_t)((int64_t)b * N / kSortTile);
    const int32_t tl = (int32_t)((((int64_t)b + 1) * N - 1) / kSortTile);
    uint32_t carry = (uint32_t)b * (uint32_t)N;
    for (int32_t q0 = 0; q0 < Q; q0 += kSortT) {
        const int32_t q = q0 + (int32_t)threadIdx.x, gg = b * Q + q;
        uint32_t tot, pre;
        brick_column<16>(hist, BQ, (size_t)b * Q + (q < Q ? q : 0), tf, tl, tf, tot, pre);
        if (q >= Q) tot = 0;
        uint32_t sum;
        const uint32_t start = carry + sort_excl_scan(tot, s_wave, &sum);
        carry += sum;
        if (q < Q) bstart[gg] = start;
        list_big(lists, q < Q, (uint32_t)gg, start, tot, hist, BQ, tf, tl);
    }
}

// A sorted point's index and its voxel within the brick: both in one word for
// clouds of at most kPackN points (svox null), else the voxel in svox.
constexpr int32_t kPackN = 1 << kPackBits;
static_assert(kBrickV <= 1 << (32 - kPackBits), "a voxel fits beside the index");

// One lane per point: (x, y, z, index and voxel within the brick) at the next
// free position of its brick within the tile's range. With SCAN the tile finds its ranges from the
// histogram columns itself (tile_columns), and one more block per cloud, before
// the tiles', writes the bricks' starts and lists the larger ones
// (cloud_columns); otherwise k_hscan has done so and rewritten row t of the
// histogram into the ranges. Bound by the tile's chain of columns, scan, LDS
// atomics and stores. With the listing in each cloud's first tile and a second
// store per point (its voxel) the launch took 10.2 us for one cloud of 20000
// points, 11.4 for two of 81920 and 55.5 for one of 2^20, now 8.7, 9.7 and 43;
// either alone cost nearly as much as both. Computing the voxels again in the
// passes over the bricks instead costs those 1 to 6 us more.
template <bool SCAN>
__global__ __launch_bounds__(kSortT) void k_bscatter(const float* __restrict__ P, int32_t N, int32_t BN, GridArgs g,
                                                     int32_t Q, int32_t BQ, int32_t vshift, int32_t clouds,
                                                     const uint32_t* __restrict__ hist,
                                                     float4* __restrict__ sorted, uint16_t* __restrict__ svox,
                                                     uint32_t* __restrict__ bstart, BrickLists lists,
                                                     int* __restrict__ status) {
    __shared__ uint32_t s_o[kMaxBricks];
    __shared__ uint32_t s_wave[kSortT / kWave];
    const int tid = threadIdx.x;
    const int32_t t = (int32_t)blockIdx.x - clouds;
    if constexpr (SCAN) {
        if (__builtin_expect(t < 0, 0)) {
            cloud_columns((int32_t)blockIdx.x, N, Q, BQ, hist, s_wave, bstart, lists);
            return;
        }
    }
    // the points' coordinates first, all loads in flight together
    float c[kSortIPT][3];
#pragma unroll
    for (int k = 0; k < kSortIPT; ++k) {
        const int32_t gid = t * kSortTile + k * kSortT + tid;
        const float* p = P + (size_t)(gid < BN ? gid : 0) * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) c[k][a] = p[a];
    }
    if constexpr (SCAN) {
        tile_columns(t, N, BN, Q, BQ, hist, s_o, s_wave);
    } else {
        const uint32_t* row = hist + (size_t)t * BQ;
        for (int32_t i = tid; i < BQ; i += kSortT) s_o[i] = row[i];
    }
    lds_barrier();
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kSortIPT; ++k) {
        const int32_t gid = t * kSortTile + k * kSortT + tid;
        if (gid >= BN) break;
        const float x = c[k][0], y = c[k][1], z = c[k][2];
        const uint32_t lin = voxel_lin(x, y, z, g, bad);
        const int32_t b = gid / N;
        const uint32_t pos = atomicAdd(&s_o[b * Q + (int32_t)(lin >> vshift)], 1u);
        const uint32_t v = lin & ((1u << vshift) - 1), i = (uint32_t)(gid - b * N);
        sorted[pos] = make_float4(x, y, z, __uint_as_float(svox ? i : i | v << kPackBits));
        if (svox) svox[pos] = (uint16_t)v;
    }
    if (bad) raise_error(status, CAGQ_ERR_NONFINITE_INPUT);
}

struct BrickArgs {
    const float* P;
    int32_t N, BN, Q, BQ;
    int32_t wshift;      // log2 of the occupancy words per brick
    int32_t groups;      // blocks that take kBrickWaves bricks each
    int32_t items_max;   // the blocks before them take an item each
    int64_t W;
    uint32_t n_v;
    const uint32_t* bstart;
    const BrickItem* item;
    const uint32_t* hfirst;
    const uint32_t* hparts;
    const float4* sorted;
    const uint16_t* svox;  // null: packed with the points' indices
    uint64_t* bitmap;
    uint32_t* word_rank;
    uint32_t* vox_lin;
    uint32_t* vox_count;
    int32_t* nvox;
    uint32_t* vox_off;
    uint32_t* pt_list;
    float4* pt4;
    uint64_t* agg;      // per brick: occupied voxels << 31 | stored points
    uint32_t* pcnt;     // count rows: per part of a heavy brick and voxel, the part's points, then
                        // the brick's points in the parts before it
    uint32_t* htot;     // per heavy brick and voxel: the points
    uint32_t* hso;      // per heavy brick and voxel: exclusive prefix of min(points, n_v)
    uint32_t* hdone;    // per heavy brick: its parts that have counted their points
    const int* status;

    __device__ __forceinline__ int32_t words() const { return 1 << wshift; }
    __device__ __forceinline__ uint32_t voxels() const { return 64u << wshift; }
};

// Occupancy words of a brick and their exclusive ranks.
struct WordLds {
    uint64_t word[kBrickW];
    uint32_t wocc[kBrickW];
};

__device__ __forceinline__ uint32_t brick_rank(const WordLds& s, uint32_t v) {
    return s.wocc[v >> 6] + (uint32_t)__popcll(s.word[v >> 6] & ((1ull << (v & 63)) - 1));
}

// Puts a brick's occupancy words (lane l holds word l, 0 from the brick's
// word count on) and their exclusive ranks into LDS; called by one wave. The
// words' lane also gets its rank.
__device__ __forceinline__ uint32_t brick_put_words(WordLds& s, uint64_t word) {
    const int lane = lane_id();
    const uint32_t o = (uint32_t)__popcll(word);
    const uint32_t ex = wave_incl_scan<uint32_t>(o) - o;
    if (lane < kBrickW) {
        s.word[lane] = word;
        s.wocc[lane] = ex;
    }
    return ex;
}

// The waves of a brick group's lists exchange data through LDS among the
// lanes of one wave only.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive scan of one value per thread over a brick block; the waves meet
// at an LDS-only barrier (their global stores are not waited for).
__device__ __forceinline__ uint64_t brick_excl_scan(uint64_t v, uint64_t* s_wave, uint64_t* total) {
    const uint64_t incl = wave_incl_scan<uint64_t>(v);
    const int wv = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) s_wave[wv] = incl;
    lds_barrier();
    uint64_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kBrickWaves; ++i) {
        const uint64_t x = s_wave[i];
        off += i < wv ? x : 0ull;
        tot += x;
    }
    *total = tot;
    return off + incl - v;
}

// One brick: its cloud, its place in the cloud, its sorted range.
struct Brick {
    int32_t g, b, q;
    uint32_t start, cnt;
};

__device__ __forceinline__ Brick brick_at(const BrickArgs& a, int32_t g) {
    Brick k;
    k.g = g;
    k.b = g / a.Q;
    k.q = g - k.b * a.Q;
    k.start = a.bstart[g];
    k.cnt = (g + 1 < a.BQ ? a.bstart[g + 1] : (uint32_t)a.BN) - k.start;
    return k;
}

// Voxels (within their brick) of IPT points of the sorted range [p0, p0 + n),
// `stride` apart from `first` on: every point's load first, so that they are
// in flight together (a load used under its bounds test would be waited for
// before the next). n is at least 1: a lane past the end loads the first one.
template <int IPT>
__device__ __forceinline__ void brick_voxels(const BrickArgs& a, uint32_t p0, uint32_t n, uint32_t first,
                                             uint32_t stride, uint32_t (&v)[IPT]) {
    if (a.svox) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t i = first + j * stride;
            v[j] = a.svox[p0 + (i < n ? i : 0u)];
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = first + j * stride;
        v[j] = __float_as_uint(a.sorted[p0 + (i < n ? i : 0u)].w);
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) v[j] >>= kPackBits;
}

// The points and their voxels, in the same way.
template <int IPT>
__device__ __forceinline__ void brick_points(const BrickArgs& a, uint32_t p0, uint32_t n, uint32_t first,
                                             uint32_t stride, float (&x)[IPT], float (&y)[IPT], float (&z)[IPT],
                                             uint32_t (&idx)[IPT], uint32_t (&v)[IPT]) {
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t i = first + j * stride;
        const float4 e = a.sorted[p0 + (i < n ? i : 0u)];
        x[j] = e.x;
        y[j] = e.y;
        z[j] = e.z;
        idx[j] = __float_as_uint(e.w);
    }
    if (a.svox) {
        brick_voxels<IPT>(a, p0, n, first, stride, v);
        return;
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        v[j] = idx[j] >> kPackBits;
        idx[j] &= (uint32_t)kPackN - 1;
    }
}

// A block's item, decoded.
struct BrickPart {
    Brick k;
    uint32_t p0, n, part;
    int32_t hb;
};

// The item of this block, or false past the last one.
__device__ __forceinline__ bool brick_part_at(const BrickArgs& a, BrickPart& p) {
    if (blockIdx.x >= (uint32_t)a.status[kStItems]) return false;
    const BrickItem it = a.item[blockIdx.x];
    p.k = brick_at(a, (int32_t)it.g);
    p.p0 = it.p0;
    p.n = (it.n & 0xFFFu) + 1;
    p.part = it.n >> 12;
    p.hb = it.hb;
    return true;
}

struct CountLds {
    union {
        uint32_t cnt2[kBrickWaves][kBrickV / 2];  // points per voxel of a wave's brick, two 16-bit counts a
                                                  // word (a block's part uses the first row)
        uint32_t tot[kBrickV];                    // a heavy brick's points per voxel
    };
    uint64_t wave[kBrickWaves];
    uint32_t ticket;
};

// Counts a point of voxel v.
__device__ __forceinline__ void count_voxel(uint32_t* cnt2, uint32_t v) {
    atomicAdd(&cnt2[v >> 1], (v & 1u) ? 0x10000u : 1u);
}

// Pass 1 over the bricks: per brick its occupancy words (final) and its
// aggregate (occupied voxels, stored points), from the points counted per
// voxel in LDS: one ballot over 64 counts is an occupancy word. The blocks
// after the first items_max take kBrickWaves bricks, `groups` apart
// (neighbouring bricks, alike in size, go to different blocks), and count
// those of at most kWavePts points by one wave each, without a barrier: most
// bricks of an indoor scene hold under 100 points, and a wave's chain of loads
// and LDS steps is no longer than a block's, so that every brick's wave is
// resident at once. The blocks before them take a larger brick, or a part of
// a heavy one, each; the last part of a heavy brick to finish turns the
// parts' count rows into the counts before each part and sums them.
__global__ __launch_bounds__(kBrickT) void k_brick_count(BrickArgs a) {
    __shared__ CountLds s;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const int32_t nw = a.words();
    // from the brick's counts, cnt(v): its occupancy words and its stored
    // points; called by one wave
    auto finish = [&](auto cnt, const Brick& k) {
        uint64_t mine = 0;
        uint32_t st = 0, occ = 0;
        for (int32_t j = 0; j < nw; ++j) {
            const uint32_t c = cnt(j * kWave + lane);
            const uint64_t bal = __ballot(c != 0);
            mine = lane == j ? bal : mine;
            occ += (uint32_t)__popcll(bal);
            st += c < a.n_v ? c : a.n_v;
        }
        st = wave_sum_u32(st);
        if (lane < nw && (int64_t)k.q * nw + lane < a.W) a.bitmap[(size_t)k.b * a.W + (size_t)k.q * nw + lane] = mine;
        if (lane == 0) a.agg[k.g] = ((uint64_t)occ << 31) | st;
    };
    if (blockIdx.x >= (uint32_t)a.items_max) {
        const int32_t g = (int32_t)blockIdx.x - a.items_max + wv * a.groups;
        if (g >= a.BQ) return;
        const Brick k = brick_at(a, g);
        if (k.cnt > (uint32_t)kWavePts) return;
        uint32_t* cnt2 = s.cnt2[wv];
        uint4* c4 = reinterpret_cast<uint4*>(cnt2);
        for (int32_t j = lane; j < nw * 8; j += kWave) c4[j] = make_uint4(0u, 0u, 0u, 0u);
        wave_lds_order();
        if (k.cnt) {
            uint32_t v[kWaveIPT];
            brick_voxels<kWaveIPT>(a, k.start, k.cnt, (uint32_t)lane, kWave, v);
#pragma unroll
            for (int j = 0; j < kWaveIPT; ++j)
                if ((uint32_t)(lane + j * kWave) < k.cnt) count_voxel(cnt2, v[j]);
        }
        wave_lds_order();
        finish([&](int32_t x) { return (uint32_t)reinterpret_cast<const uint16_t*>(cnt2)[x]; }, k);
        return;
    }
    BrickPart p;
    if (!brick_part_at(a, p)) return;
    uint32_t* cnt2 = s.cnt2[0];
    const uint16_t* cnt = reinterpret_cast<const uint16_t*>(cnt2);
    const uint32_t nvx = a.voxels();
    for (uint32_t j = tid; j < nvx / 2; j += kBrickT) cnt2[j] = 0u;
    lds_barrier();
#pragma unroll
    for (int h = 0; h < kBrickIPT; h += kLoadIPT) {
        if ((uint32_t)(h * kBrickT) < p.n) {
            uint32_t v[kLoadIPT];
            brick_voxels<kLoadIPT>(a, p.p0, p.n, (uint32_t)(tid + h * kBrickT), kBrickT, v);
#pragma unroll
            for (int j = 0; j < kLoadIPT; ++j)
                if ((uint32_t)(tid + (h + j) * kBrickT) < p.n) count_voxel(cnt2, v[j]);
        }
    }
    lds_barrier();
    if (p.hb < 0) {
        if (wv == 0) finish([&](int32_t x) { return (uint32_t)cnt[x]; }, p.k);
        return;
    }
    const uint32_t parts = a.hparts[p.hb];
    uint32_t* row = a.pcnt + (size_t)a.hfirst[p.hb] * nvx;
    for (uint32_t j = tid; j < nvx; j += kBrickT) row[(size_t)p.part * nvx + j] = cnt[j];
    __threadfence();
    __syncthreads();
    if (tid == 0) s.ticket = atomicAdd(&a.hdone[p.hb], 1u);
    __syncthreads();
    if (s.ticket != parts - 1) return;
    __threadfence();
    for (uint32_t j = tid; j < nvx; j += kBrickT) {
        uint32_t run = 0;
        for (uint32_t i = 0; i < parts; ++i) {
            const uint32_t x = row[(size_t)i * nvx + j];
            row[(size_t)i * nvx + j] = run;
            run += x;
        }
        s.tot[j] = run;
        a.htot[(size_t)p.hb * nvx + j] = run;
    }
    lds_barrier();
    if (wv == 0) finish([&](int32_t x) { return s.tot[x]; }, p.k);
    const uint32_t per = (nvx + kBrickT - 1) / kBrickT, x0 = (uint32_t)tid * per;  // nvx is a power of two
    uint64_t sum = 0;
    for (uint32_t x = x0; x < x0 + per && x < nvx; ++x) sum += s.tot[x] < a.n_v ? s.tot[x] : a.n_v;
    uint64_t total;
    uint32_t pos = (uint32_t)brick_excl_scan(sum, s.wave, &total);
    for (uint32_t x = x0; x < x0 + per && x < nvx; ++x) {
        a.hso[(size_t)p.hb * nvx + x] = pos;
        pos += s.tot[x] < a.n_v ? s.tot[x] : a.n_v;
    }
}

// The lists of one wave's brick, and of a block's.
struct WaveLists {
    WordLds w;
    uint32_t va[kWavePts + 1];  // per occupied voxel: count, then (stored prefix << 16 | point prefix)
    uint32_t idx[kWavePts];     // point indices grouped by voxel (arrival order)
    uint16_t vox[kWavePts];     // the occupied voxels
};

struct BlockLists {
    WordLds w;
    uint64_t bigm[kBrickW];     // bit r: occupied voxel r holds more than kBigVoxel points
    uint32_t va[kBrickV + 1];
    uint32_t idx[kBrickCap];
    uint16_t vox[kBrickV];
    uint64_t wave[kBrickWaves];
};

union BuildLds {
    WaveLists wl[kBrickWaves];
    BlockLists bl;
};

// A voxel of c > kBigVoxel points at p (LDS): one wave writes its `keep`
// lowest indices and their points to the stored positions from dst on.
__device__ __forceinline__ void wave_big_voxel(const BrickArgs& a, const uint32_t* p, uint32_t c, uint32_t keep,
                                               size_t pb, size_t dst) {
    const int lane = lane_id();
    uint32_t best = ~0u, kth = ~0u;
    for (uint32_t c0 = 0; c0 < c; c0 += kWave) {
        uint32_t key = (c0 + lane < c) ? p[c0 + lane] : ~0u;
        // an index above the keep-th lowest so far is never kept
        key = key < kth ? key : ~0u;
        if (c0 != 0 && !__ballot(key != ~0u)) continue;
        key = wave_sort32(key);
        best = c0 == 0 ? key : wave_merge_low32(best, key);
        kth = (uint32_t)__shfl((int)best, (int)keep - 1, kWave);
    }
    if ((uint32_t)lane < keep) {
        const uint32_t i = best;
        const float* q = a.P + (pb + i) * 3;
        a.pt_list[dst + lane] = i;
        a.pt4[dst + lane] = make_float4(q[0], q[1], q[2], __uint_as_float(i));
    }
}

// A brick of at most kWavePts points: slots, offsets and stored lists by one
// wave, in LDS, without a barrier. `word`: lane l's occupancy word.
__device__ __forceinline__ void brick_by_wave(const BrickArgs& a, WaveLists& s, const Brick& k, uint64_t pre,
                                              uint32_t n_occ, uint64_t word) {
    const int lane = lane_id();
    const uint32_t p_occ = (uint32_t)(pre >> 31), p_st = (uint32_t)(pre & 0x7FFFFFFFu);
    const int32_t nw = a.words();
    const uint32_t vbase = (uint32_t)k.q * a.voxels();
    const size_t pb = (size_t)k.b * a.N;
    // the points' loads go out first
    uint32_t v[kWaveIPT], idx[kWaveIPT];
    float x[kWaveIPT], y[kWaveIPT], z[kWaveIPT];
    if (k.cnt) {
        brick_points<kWaveIPT>(a, k.start, k.cnt, (uint32_t)lane, kWave, x, y, z, idx, v);
    }
    const uint32_t wr = brick_put_words(s.w, word);
    if (lane < nw && (int64_t)k.q * nw + lane < a.W)
        a.word_rank[(size_t)k.b * a.W + (size_t)k.q * nw + lane] = p_occ + wr;
    if (k.cnt == 0) return;
    for (uint32_t j = lane; j <= n_occ; j += kWave) s.va[j] = 0u;
    wave_lds_order();
    // voxel rank and arrival position of every point; the first arrival
    // names the voxel
#pragma unroll
    for (int j = 0; j < kWaveIPT; ++j) {
        if ((uint32_t)(lane + j * kWave) < k.cnt) {
            const uint32_t r = brick_rank(s.w, v[j]);
            const uint32_t pos = atomicAdd(&s.va[r], 1u);
            if (pos == 0) s.vox[r] = (uint16_t)v[j];
            v[j] = (r << 16) | pos;
        }
    }
    wave_lds_order();
    // exclusive prefixes of (count, stored), packed as stored << 16 | count,
    // and the slots' own outputs, 64 occupied voxels at a time
    uint32_t run = 0;
    uint64_t big[kWaveIPT];  // voxels of more than kBigVoxel points
#pragma unroll
    for (int j = 0; j < kWaveIPT; ++j) {
        big[j] = 0;
        if ((uint32_t)(j * kWave) >= n_occ) continue;
        const uint32_t r = (uint32_t)(j * kWave + lane);
        const uint32_t c = r < n_occ ? s.va[r] : 0u;
        const uint32_t both = ((c < a.n_v ? c : a.n_v) << 16) | c;
        const uint32_t incl = wave_incl_sum_u32(both);
        const uint32_t ex = run + incl - both;
        run += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        big[j] = __ballot(c > kBigVoxel);
        if (r < n_occ) {
            s.va[r] = ex;
            const size_t slot = pb + p_occ + r;
            a.vox_lin[slot] = vbase + s.vox[r];
            a.vox_count[slot] = c;
            a.vox_off[slot + k.b] = p_st + (ex >> 16);
        }
    }
    if (lane == 0) s.va[n_occ] = run;
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < kWaveIPT; ++j)
        if ((uint32_t)(lane + j * kWave) < k.cnt) s.idx[(s.va[v[j] >> 16] & 0xFFFFu) + (v[j] & 0xFFFFu)] = idx[j];
    wave_lds_order();
    // stored lists: a point of a voxel of at most kBigVoxel points by its rank
#pragma unroll
    for (int j = 0; j < kWaveIPT; ++j) {
        uint32_t c = 0, f0 = 0, rank = 0, o = 0;
        if ((uint32_t)(lane + j * kWave) < k.cnt) {
            const uint32_t r = v[j] >> 16;
            o = s.va[r];
            f0 = o & 0xFFFFu;
            c = (s.va[r + 1] & 0xFFFFu) - f0;
        }
        if (c <= kBigVoxel) {
            for (uint32_t i = 0; i < c; ++i) rank += s.idx[f0 + i] < idx[j] ? 1u : 0u;
            if (c && rank < a.n_v) {
                const size_t dst = pb + p_st + (o >> 16) + rank;
                a.pt_list[dst] = idx[j];
                a.pt4[dst] = make_float4(x[j], y[j], z[j], __uint_as_float(idx[j]));
            }
        }
    }
    // larger voxels: the n_v smallest indices by bitonic selection
#pragma unroll
    for (int j = 0; j < kWaveIPT; ++j) {
        for (uint64_t m = big[j]; m; m &= m - 1) {
            const uint32_t r = (uint32_t)(j * kWave + __ffsll((unsigned long long)m) - 1);
            const uint32_t o = s.va[r], f0 = o & 0xFFFFu, c = (s.va[r + 1] & 0xFFFFu) - f0;
            wave_big_voxel(a, s.idx + f0, c, a.n_v, pb, pb + p_st + (o >> 16));
        }
    }
}

// A larger brick, or a part of a heavy one: the same by a block. A heavy
// brick's slots come from its totals, written by its first part, and its
// points rank after those of their voxel in the parts before.
__device__ __forceinline__ void brick_by_block(const BrickArgs& a, BlockLists& s, const BrickPart& p, uint64_t pre,
                                               uint32_t n_occ, uint64_t word) {
    const Brick& k = p.k;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const uint32_t p_occ = (uint32_t)(pre >> 31), p_st = (uint32_t)(pre & 0x7FFFFFFFu);
    const int32_t nw = a.words();
    const uint32_t nvx = a.voxels(), vbase = (uint32_t)k.q * nvx;
    const size_t pb = (size_t)k.b * a.N;
    const bool heavy = p.hb >= 0;
    const uint32_t* before = heavy ? a.pcnt + (size_t)(a.hfirst[p.hb] + p.part) * nvx : nullptr;
    const uint32_t* so = heavy ? a.hso + (size_t)p.hb * nvx : nullptr;
    uint32_t* va = s.va;  // n_occ + 1 entries
    // the points' loads go out first
    uint32_t v[kBrickIPT], idx[kBrickIPT];
    float x[kBrickIPT], y[kBrickIPT], z[kBrickIPT];
    brick_points<kBrickIPT>(a, p.p0, p.n, (uint32_t)tid, kBrickT, x, y, z, idx, v);
    if (wv == 0) {
        const uint32_t wr = brick_put_words(s.w, word);
        if (p.part == 0 && lane < nw && (int64_t)k.q * nw + lane < a.W)
            a.word_rank[(size_t)k.b * a.W + (size_t)k.q * nw + lane] = p_occ + wr;
    }
    if (tid < kBrickW) s.bigm[tid] = 0ull;
    for (uint32_t j = tid; j <= n_occ; j += kBrickT) va[j] = 0u;
    lds_barrier();
    // voxel rank and arrival position of every point; the first arrival names
    // the voxel
#pragma unroll
    for (int j = 0; j < kBrickIPT; ++j) {
        if ((uint32_t)(tid + j * kBrickT) < p.n) {
            const uint32_t r = brick_rank(s.w, v[j]);
            const uint32_t pos = atomicAdd(&va[r], 1u);
            if (pos == 0) s.vox[r] = (uint16_t)v[j];
            v[j] = (r << 16) | pos;
        }
    }
    lds_barrier();
    // exclusive prefixes of (count, stored) over the occupied voxels, packed
    // as stored << 16 | count (both at most kBrickCap)
    const uint32_t per = (n_occ + kBrickT - 1) / kBrickT;
    const uint32_t r0 = (uint32_t)tid * per;
    uint32_t sum = 0;
    for (uint32_t j = 0; j < per; ++j) {
        if (r0 + j >= n_occ) break;
        const uint32_t c = va[r0 + j];
        sum += ((c < a.n_v ? c : a.n_v) << 16) | c;
    }
    uint64_t total;
    uint32_t run = (uint32_t)brick_excl_scan(sum, s.wave, &total);
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t rr = r0 + j;
        if (rr >= n_occ) break;
        const uint32_t c = va[rr];
        va[rr] = run;
        if (c > kBigVoxel) atomicOr(reinterpret_cast<unsigned long long*>(&s.bigm[rr >> 6]), 1ull << (rr & 63));
        run += ((c < a.n_v ? c : a.n_v) << 16) | c;
    }
    if (tid == 0) va[n_occ] = p.n;
    lds_barrier();
    // the points grouped by voxel, and the slots' own outputs
#pragma unroll
    for (int j = 0; j < kBrickIPT; ++j)
        if ((uint32_t)(tid + j * kBrickT) < p.n) s.idx[(va[v[j] >> 16] & 0xFFFFu) + (v[j] & 0xFFFFu)] = idx[j];
    if (!heavy) {
        for (uint32_t r = tid; r < n_occ; r += kBrickT) {
            const uint32_t o = va[r];
            const size_t slot = pb + p_occ + r;
            a.vox_lin[slot] = vbase + s.vox[r];
            a.vox_count[slot] = (va[r + 1] & 0xFFFFu) - (o & 0xFFFFu);
            a.vox_off[slot + k.b] = p_st + (o >> 16);
        }
    } else if (p.part == 0) {
        for (uint32_t u = tid; u < nvx; u += kBrickT) {
            const uint32_t c = a.htot[(size_t)p.hb * nvx + u];
            if (!c) continue;
            const size_t slot = pb + p_occ + brick_rank(s.w, u);
            a.vox_lin[slot] = vbase + u;
            a.vox_count[slot] = c;
            a.vox_off[slot + k.b] = p_st + so[u];
        }
    }
    lds_barrier();
    // stored lists: a point of a voxel of at most kBigVoxel points (of this
    // part) by its rank
#pragma unroll
    for (int j = 0; j < kBrickIPT; ++j) {
        uint32_t r = 0, c = 0, f0 = 0, rank = 0, at0 = 0;
        if ((uint32_t)(tid + j * kBrickT) < p.n) {
            r = v[j] >> 16;
            at0 = va[r];
            f0 = at0 & 0xFFFFu;
            c = (va[r + 1] & 0xFFFFu) - f0;
            at0 >>= 16;
        }
        if (c <= kBigVoxel) {
            for (uint32_t i = 0; i < c; ++i) rank += s.idx[f0 + i] < idx[j] ? 1u : 0u;
            if (heavy && c) {
                rank += before[s.vox[r]];
                at0 = so[s.vox[r]];
            }
            if (c && rank < a.n_v) {
                const size_t dst = pb + p_st + at0 + rank;
                a.pt_list[dst] = idx[j];
                a.pt4[dst] = make_float4(x[j], y[j], z[j], __uint_as_float(idx[j]));
            }
        }
    }
    // larger voxels: one wave each
    for (int j = wv; j < kBrickW; j += kBrickWaves) {
        for (uint64_t m = s.bigm[j]; m; m &= m - 1) {
            const uint32_t r = (uint32_t)j * kWave + (uint32_t)(__ffsll((unsigned long long)m) - 1);
            const uint32_t o = va[r], f0 = o & 0xFFFFu, c = (va[r + 1] & 0xFFFFu) - f0;
            const uint32_t bf = heavy ? before[s.vox[r]] : 0u, at0 = heavy ? so[s.vox[r]] : o >> 16;
            if (bf < a.n_v) wave_big_voxel(a, s.idx + f0, c, a.n_v - bf, pb, pb + p_st + at0 + bf);
        }
    }
}

// The aggregate of the cloud's bricks before brick q (every one is final),
// in every lane of the wave; the loads go out together, 16 per lane.
__device__ __forceinline__ uint64_t brick_prefix(const uint64_t* ag, int32_t q) {
    const int lane = lane_id();
    uint64_t pre = 0;
    for (int32_t j0 = 0; j0 < q; j0 += 16 * kWave) {
        uint64_t x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int32_t j = j0 + u * kWave + lane;
            x[u] = j < q ? ag[j] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) pre += x[u];
    }
    return wave_sum<uint64_t>(pre);
}

// Pass 2 over the bricks: slots, offsets and stored lists, split over the
// blocks as in pass 1: a wave per brick of at most kWavePts points (no barrier
// at all), a block per item. Bound by the chain of loads and LDS steps of its
// largest bricks, not by bandwidth. Measured, first layer of four indoor
// scenes (81920 points each, 0.05 voxels): 46 -> 15 us against a block per
// brick of up to 2048 points, whose heavy bricks were finished by the last of
// their parts alone (and 13 -> 8 us for pass 1); one such scene on 0.1 voxels,
// ten heavy bricks: 153 -> 10 us. Waves that took up to 512 points, with the
// larger bricks after them in the same blocks, measured 54 us.
__global__ __launch_bounds__(kBrickT) void k_brick(BrickArgs a) {
    __shared__ BuildLds s;
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int32_t nw = a.words();
    auto load_word = [&](int32_t b, int32_t q) {
        const bool in = lane < nw && (int64_t)q * nw + lane < a.W;
        return in ? a.bitmap[(size_t)b * a.W + (size_t)q * nw + lane] : 0ull;
    };
    if (blockIdx.x < (uint32_t)a.items_max) {
        BrickPart p;
        if (!brick_part_at(a, p)) return;
        const uint64_t* ag = a.agg + (size_t)p.k.b * a.Q;
        const uint64_t word = load_word(p.k.b, p.k.q);
        const uint32_t n_occ = (uint32_t)(ag[p.k.q] >> 31);
        brick_by_block(a, s.bl, p, brick_prefix(ag, p.k.q), n_occ, word);
        return;
    }
    const int32_t g = (int32_t)blockIdx.x - a.items_max + wv * a.groups;
    if (g >= a.BQ) return;
    const Brick k = brick_at(a, g);
    const bool last = k.q == a.Q - 1;
    if (k.cnt > (uint32_t)kWavePts && !last) return;
    const uint64_t* ag = a.agg + (size_t)k.b * a.Q;
    const uint64_t word = load_word(k.b, k.q);
    const uint64_t my = ag[k.q];
    const uint64_t pre = brick_prefix(ag, k.q);
    if (last && lane == 0) {
        const uint64_t all = pre + my;
        a.nvox[k.b] = (int32_t)(all >> 31);
        a.vox_off[(size_t)k.b * (a.N + 1) + (all >> 31)] = (uint32_t)(all & 0x7FFFFFFFu);
    }
    if (k.cnt <= (uint32_t)kWavePts) brick_by_wave(a, s.wl[wv], k, pre, (uint32_t)(my >> 31), word);
}

// ---- small clouds: the whole build in one workgroup per cloud.
// For clouds of at most kSmallN points whose grid has at most kSmallW
// occupancy words, every step above runs in one 1024-thread workgroup with
// the bitmap, the ranks, the counts and offsets and the buckets in LDS, so
// the seven launches (and their dependent round trips to memory) become one.
// The outputs are those of the steps above, bit for bit: the same bitmap,
// ranks, slots and linear ids, counts and offsets, and per voxel the n_v
// lowest point indices in ascending order (ranked against the voxel's
// bucket, or selected by a wave for voxels of more than kBigVoxel points).
// The threads exchange data through LDS only, so the barriers do not wait for
// the global stores of the steps before them.
constexpr int kSmallT = 1024;
constexpr int kSmallPts = 8;   // points per thread
constexpr int kSmallWd = 4;    // occupancy words per thread
constexpr int32_t kSmallN = kSmallT * kSmallPts;
constexpr int64_t kSmallW = kSmallT * kSmallWd;
constexpr int kSmallBig = kSmallN / (kBigVoxel + 1) + 1;  // voxels of more than kBigVoxel points

// Exclusive scan of one value per thread over the kSmallT threads.
__device__ __forceinline__ uint64_t small_excl_scan(uint64_t v, uint64_t* s_wave, uint64_t* total) {
    const uint64_t incl = wave_incl_scan<uint64_t>(v);
    const int wv = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) s_wave[wv] = incl;
    lds_barrier();
    uint64_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kSmallT / kWave; ++i) {
        const uint64_t x = s_wave[i];
        off += i < wv ? x : 0ull;
        tot += x;
    }
    *total = tot;
    lds_barrier();
    return off + incl - v;
}

size_t small_lds_bytes(int32_t N, int64_t W) { return (size_t)12 * W + (size_t)4 * (2 * (size_t)N + 1); }

__global__ __launch_bounds__(kSmallT) void k_build_small(
    const float* __restrict__ P, int32_t N, GridArgs g, int64_t W, uint32_t n_v, uint64_t* __restrict__ bitmap,
    uint32_t* __restrict__ word_rank, uint32_t* __restrict__ vox_lin, uint32_t* __restrict__ vox_count,
    int32_t* __restrict__ nvox, uint32_t* __restrict__ vox_off, uint32_t* __restrict__ pt_list,
    float4* __restrict__ pt4, int* __restrict__ status, int* __restrict__ berr, uint64_t* __restrict__ ctx_desc,
    int32_t ctx_tiles) {
    extern __shared__ __align__(16) unsigned char lds[];
    uint64_t* s_bm = reinterpret_cast<uint64_t*>(lds);   // [W] occupancy words
    uint32_t* s_wr = reinterpret_cast<uint32_t*>(s_bm + W);  // [W] ranks
    uint32_t* s_off = s_wr + W;  // [N + 1] counts, then (full offset << 16) | stored offset
    uint32_t* s_bk = s_off + N + 1;  // [N] point indices grouped by slot (arrival order)
    __shared__ uint64_t s_wave[kSmallT / kWave];
    __shared__ uint32_t s_big[kSmallBig];
    __shared__ uint32_t s_nbig, s_bad;
    const int32_t b = blockIdx.x;
    const int tid = threadIdx.x;
    const size_t pb = (size_t)b * N;

    // the status words start at zero for the kernels after this one (this
    // kernel writes none: its errors go to the cloud's own word), and so do
    // the descriptors of the context offsets
    if (b == 0 && tid < kStSlots) status[tid] = 0;
    for (int32_t i = b * kSmallT + tid; i < ctx_tiles; i += (int32_t)gridDim.x * kSmallT) ctx_desc[i] = 0ull;
    for (int64_t w = tid; w < W; w += kSmallT) s_bm[w] = 0ull;
    for (int32_t i = tid; i <= N; i += kSmallT) s_off[i] = 0u;
    if (tid == 0) {
        s_nbig = 0;
        s_bad = 0;
    }
    lds_barrier();

    // voxelize: linear id, occupancy bit (every point's coordinates are
    // loaded first, so that their loads are in flight together)
    float pc[kSmallPts][3];
#pragma unroll
    for (int k = 0; k < kSmallPts; ++k) {
        const int32_t i = tid + k * kSmallT;
        const float* p = P + (pb + (i < N ? i : 0)) * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) pc[k][a] = p[a];
    }
    uint32_t lin[kSmallPts];
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kSmallPts; ++k) {
        const int32_t i = tid + k * kSmallT;
        lin[k] = 0;
        if (i >= N) continue;
        uint32_t gg[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (!isfinite(pc[k][a])) {
                bad = true;
                gg[a] = 0;
            } else {
                gg[a] = (uint32_t)axis_index(pc[k][a], g.o[a], g.s[a], g.D[a]);
            }
        }
        lin[k] = gg[0] + (uint32_t)g.D[0] * (gg[1] + (uint32_t)g.D[1] * gg[2]);
        atomicOr(reinterpret_cast<unsigned long long*>(&s_bm[lin[k] >> 6]), 1ull << (lin[k] & 63));
    }
    if (bad) s_bad = 1;
    lds_barrier();
    if (tid == 0) berr[b] = s_bad ? CAGQ_ERR_NONFINITE_INPUT : 0;

    // ranks of the words
    uint64_t wd[kSmallWd];
    uint32_t cnt = 0;
#pragma unroll
    for (int j = 0; j < kSmallWd; ++j) {
        const int64_t w = (int64_t)tid * kSmallWd + j;
        wd[j] = w < W ? s_bm[w] : 0ull;
        cnt += (uint32_t)__popcll(wd[j]);
    }
    uint64_t total;
    uint32_t r = (uint32_t)small_excl_scan(cnt, s_wave, &total);
    const uint32_t nv = (uint32_t)total;
#pragma unroll
    for (int j = 0; j < kSmallWd; ++j) {
        const int64_t w = (int64_t)tid * kSmallWd + j;
        if (w >= W) break;
        s_wr[w] = r;
        bitmap[(size_t)b * W + w] = wd[j];
        word_rank[(size_t)b * W + w] = r;
        r += (uint32_t)__popcll(wd[j]);
    }
    if (tid == 0) nvox[b] = (int32_t)nv;
    lds_barrier();

    // slot and arrival position of every point, packed as slot << 16 | position;
    // the first arrival in a voxel puts its linear id at its slot of s_bk
    // (free until the buckets), for the coalesced writes after the offsets
    uint32_t sp[kSmallPts];
#pragma unroll
    for (int k = 0; k < kSmallPts; ++k) {
        const int32_t i = tid + k * kSmallT;
        sp[k] = 0;
        if (i >= N) continue;
        const uint32_t w = lin[k] >> 6;
        const uint32_t sl = s_wr[w] + (uint32_t)__popcll(s_bm[w] & ((1ull << (lin[k] & 63)) - 1));
        const uint32_t pos = atomicAdd(&s_off[sl], 1u);
        sp[k] = (sl << 16) | pos;
        if (pos == 0) s_bk[sl] = lin[k];
    }
    lds_barrier();

    // offsets: (full << 31) | stored, scanned over the slots [0, nv)
    uint32_t c8[kSmallPts];
    uint64_t sum = 0;
#pragma unroll
    for (int j = 0; j < kSmallPts; ++j) {
        const uint32_t sl = (uint32_t)tid * kSmallPts + j;
        c8[j] = sl < nv ? s_off[sl] : 0u;
        sum += ((uint64_t)c8[j] << 31) | (c8[j] < n_v ? c8[j] : n_v);
    }
    uint64_t run = small_excl_scan(sum, s_wave, &total);
    uint32_t* vo = vox_off + (size_t)b * (N + 1);
#pragma unroll
    for (int j = 0; j < kSmallPts; ++j) {
        const uint32_t sl = (uint32_t)tid * kSmallPts + j;
        if (sl >= nv) break;
        const uint32_t full = (uint32_t)(run >> 31), stored = (uint32_t)(run & 0x7FFFFFFFu);
        s_off[sl] = (full << 16) | stored;
        if (c8[j] > kBigVoxel) s_big[atomicAdd(&s_nbig, 1u)] = sl;
        run += ((uint64_t)c8[j] << 31) | (c8[j] < n_v ? c8[j] : n_v);
    }
    if (tid == 0) {
        vo[nv] = (uint32_t)(total & 0x7FFFFFFFu);
        s_off[nv] = ((uint32_t)(total >> 31) << 16) | (uint32_t)(total & 0x7FFFFFFFu);
    }
    lds_barrier();
    // offsets, counts and linear ids, each slot's from LDS: consecutive
    // threads store consecutive slots
    for (uint32_t sl = (uint32_t)tid; sl < nv; sl += kSmallT) {
        const uint32_t o0 = s_off[sl], o1 = s_off[sl + 1];
        vo[sl] = o0 & 0xFFFFu;
        vox_count[pb + sl] = (o1 >> 16) - (o0 >> 16);
        vox_lin[pb + sl] = s_bk[sl];
    }
    lds_barrier();  // s_bk is read above and filled below

    // buckets
#pragma unroll
    for (int k = 0; k < kSmallPts; ++k) {
        const int32_t i = tid + k * kSmallT;
        if (i < N) s_bk[(s_off[sp[k] >> 16] >> 16) + (sp[k] & 0xFFFFu)] = (uint32_t)i;
    }
    lds_barrier();

    // stored lists: a point of a voxel of at most kBigVoxel points by its rank
#pragma unroll
    for (int k = 0; k < kSmallPts; ++k) {
        const int32_t i = tid + k * kSmallT;
        if (i >= N) continue;
        const uint32_t o0 = s_off[sp[k] >> 16], o1 = s_off[(sp[k] >> 16) + 1];
        const uint32_t f0 = o0 >> 16, cnt_v = (o1 >> 16) - f0;
        if (cnt_v > kBigVoxel) continue;
        uint32_t rank = 0;
        for (uint32_t j = 0; j < cnt_v; ++j) rank += s_bk[f0 + j] < (uint32_t)i ? 1u : 0u;
        if (rank < n_v) {
            const size_t dst = pb + (o0 & 0xFFFFu) + rank;
            const float* p = P + (pb + i) * 3;
            pt_list[dst] = (uint32_t)i;
            pt4[dst] = make_float4(p[0], p[1], p[2], __uint_as_float((uint32_t)i));
        }
    }
    // larger voxels: one wave each, the n_v smallest indices by bitonic selection
    const int lane = lane_id();
    for (uint32_t v = (uint32_t)(tid / kWave); v < s_nbig; v += kSmallT / kWave) {
        const uint32_t sl = s_big[v];
        const uint32_t o0 = s_off[sl], f0 = o0 >> 16, cnt_v = (s_off[sl + 1] >> 16) - f0;
        uint32_t best = ~0u, kth = ~0u;
        for (uint32_t c0 = 0; c0 < cnt_v; c0 += kWave) {
            uint32_t key = (c0 + lane < cnt_v) ? s_bk[f0 + c0 + lane] : ~0u;
            // an index above the n_v-th lowest so far is never kept
            key = key < kth ? key : ~0u;
            if (c0 != 0 && !__ballot(key != ~0u)) continue;
            key = wave_sort32(key);
            best = c0 == 0 ? key : wave_merge_low32(best, key);
            kth = (uint32_t)__shfl((int)best, (int)n_v - 1, kWave);
        }
        if ((uint32_t)lane < n_v) {
            const uint32_t i = best;
            const size_t dst = pb + (o0 & 0xFFFFu) + lane;
            const float* p = P + (pb + i) * 3;
            pt_list[dst] = i;
            pt4[dst] = make_float4(p[0], p[1], p[2], __uint_as_float(i));
        }
    }
}

// Dynamic LDS a workgroup of k_build_small may take on the current device, or -1.
int64_t small_lds_avail() {
    static int64_t avail[64];  // per device, 0 until known
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
    if (avail[dev] == 0) {
        int max_sh = 0;
        hipFuncAttributes fa{};
        if (hipDeviceGetAttribute(&max_sh, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
            hipFuncGetAttributes(&fa, (const void*)k_build_small) != hipSuccess)
            return -1;
        avail[dev] = (int64_t)max_sh - (int64_t)fa.sharedSizeBytes;
    }
    return avail[dev];
}

}  // namespace

hipError_t launch_build(const float* points, const Layout& L, const cagq_grid_desc& d, void* ws,
                        hipStream_t s) {
    const int32_t B = L.B, N = L.N, BN = B * N;
    const GridArgs g = grid_args(d);
    int* status = at<int>(ws, L.status);
    if (N <= kSmallN && L.W <= kSmallW && (int64_t)small_lds_bytes(N, L.W) <= small_lds_avail()) {
        // no clearing launch: the build zeroes the status words itself and
        // writes each cloud's error code (the selection's histogram serves
        // clouds of at least 16384 points only, the scan descriptors and
        // occupancy bytes other builds)
        const size_t bytes = small_lds_bytes(N, L.W);
        hipError_t e = hipFuncSetAttribute((const void*)k_build_small, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)bytes);
        if (e != hipSuccess) return e;
        k_build_small<<<B, kSmallT, bytes, s>>>(points, N, g, L.W, (uint32_t)d.n_v, at<uint64_t>(ws, L.bitmap),
                                                at<uint32_t>(ws, L.word_rank), at<uint32_t>(ws, L.vox_lin),
                                                at<uint32_t>(ws, L.vox_count),
                                                at<int32_t>(ws, L.nvox), at<uint32_t>(ws, L.vox_off),
                                                at<uint32_t>(ws, L.pt_list), at<float4>(ws, L.pt4), status,
                                                at<int>(ws, L.berr), at<uint64_t>(ws, L.ctx_desc),
                                                (int32_t)L.ctx_tiles);
        return hipGetLastError();
    }
    if (L.bricks) {
        const int32_t BQ = B * L.Q;
        uint32_t* hist = at<uint32_t>(ws, L.hist);
        int* status_w = at<int>(ws, L.status);
        const BrickLists lists{at<BrickItem>(ws, L.item), at<uint32_t>(ws, L.hfirst), at<uint32_t>(ws, L.hparts),
                               at<uint32_t>(ws, L.pcnt), 64u << L.wshift, status_w};
        k_bhist<<<(unsigned)L.T, kSortT, 0, s>>>(points, N, BN, g, L.Q, BQ, L.wshift + 6, L.T, L.tile_scan, hist,
                                                 at<uint4>(ws, L.status), (int64_t)(L.clear_brick - L.status) / 16);
        if (!L.tile_scan)
            k_hscan<<<(unsigned)((BQ + kHGroup - 1) / kHGroup), kScanThreads, 0, s>>>(
                hist, N, L.Q, BQ, L.T, at<uint32_t>(ws, L.bstart), lists, at<uint64_t>(ws, L.desc_h), status_w);
        uint16_t* svox = N <= kPackN ? nullptr : at<uint16_t>(ws, L.svox);
        const int32_t clouds = L.tile_scan ? B : 0;  // blocks before the tiles' (see k_bscatter)
        (L.tile_scan ? k_bscatter<true> : k_bscatter<false>)<<<(unsigned)(L.T + clouds), kSortT, 0, s>>>(
            points, N, BN, g, L.Q, BQ, L.wshift + 6, clouds, hist, at<float4>(ws, L.sorted), svox,
            at<uint32_t>(ws, L.bstart), lists, status_w);
        BrickArgs a;
        a.P = points;
        a.N = N;
        a.BN = BN;
        a.Q = L.Q;
        a.BQ = BQ;
        a.wshift = L.wshift;
        a.groups = (BQ + kBrickWaves - 1) / kBrickWaves;
        a.W = L.W;
        a.n_v = (uint32_t)d.n_v;
        a.bstart = at<uint32_t>(ws, L.bstart);
        a.items_max = (int32_t)L.items_max;
        a.item = lists.item;
        a.hfirst = lists.hfirst;
        a.hparts = lists.hparts;
        a.sorted = at<float4>(ws, L.sorted);
        a.svox = svox;
        a.bitmap = at<uint64_t>(ws, L.bitmap);
        a.word_rank = at<uint32_t>(ws, L.word_rank);
        a.vox_lin = at<uint32_t>(ws, L.vox_lin);
        a.vox_count = at<uint32_t>(ws, L.vox_count);
        a.nvox = at<int32_t>(ws, L.nvox);
        a.vox_off = at<uint32_t>(ws, L.vox_off);
        a.pt_list = at<uint32_t>(ws, L.pt_list);
        a.pt4 = at<float4>(ws, L.pt4);
        a.agg = at<uint64_t>(ws, L.agg);
        a.pcnt = at<uint32_t>(ws, L.pcnt);
        a.hdone = at<uint32_t>(ws, L.hdone);
        a.htot = at<uint32_t>(ws, L.htot);
        a.hso = at<uint32_t>(ws, L.hso);
        a.status = status_w;
        k_brick_count<<<(unsigned)(a.items_max + a.groups), kBrickT, 0, s>>>(a);
        k_brick<<<(unsigned)(a.items_max + a.groups), kBrickT, 0, s>>>(a);
        return hipGetLastError();
    }
    size_t n16 = (L.clear_end - L.status) / 16;
    int cb = (int)((n16 + 255) / 256);
    if (cb > 4096) cb = 4096;
    k_clear<<<cb, 256, 0, s>>>(at<uint4>(ws, L.status), n16);
    const int pb = (BN + 255) / 256;
    k_mark<<<pb, 256, 0, s>>>(points, N, BN, g, L.W, at<uint32_t>(ws, L.pt_slot), at<uint8_t>(ws, L.bytemap),
                              status);
    uint32_t* tile_cnt = at<uint32_t>(ws, L.desc_w);
    uint32_t* group_cnt = tile_cnt + (size_t)B * L.tiles_w;
    k_pack<<<(unsigned)(B * L.tiles_w), kScanThreads, 0, s>>>(at<uint8_t>(ws, L.bytemap), at<uint64_t>(ws, L.bitmap),
                                                              L.W, L.tiles_w, tile_cnt, group_cnt);
    k_rank<<<(unsigned)(B * L.tiles_w), kScanThreads, 0, s>>>(
        at<uint64_t>(ws, L.bitmap), L.W, L.tiles_w, N, tile_cnt, group_cnt, at<uint32_t>(ws, L.word_rank),
        at<uint32_t>(ws, L.vox_lin), at<uint32_t>(ws, L.vox_count), at<int32_t>(ws, L.nvox));
    k_count<<<pb, 256, 0, s>>>(BN, N, L.W, at<uint64_t>(ws, L.bitmap), at<uint32_t>(ws, L.word_rank),
                               at<uint32_t>(ws, L.pt_slot), at<uint32_t>(ws, L.pt_pos),
                               at<uint32_t>(ws, L.vox_count));
    k_offsets<<<(unsigned)(B * L.tiles_s), kScanThreads, 0, s>>>(
        B, N, L.tiles_s, (uint32_t)d.n_v, at<int32_t>(ws, L.nvox), at<uint32_t>(ws, L.vox_count),
        at<uint32_t>(ws, L.vox_off), at<uint32_t>(ws, L.full_off), at<uint64_t>(ws, L.desc_s), status,
        at<uint32_t>(ws, L.big), L.big_cap);
    k_scatter<<<pb, 256, 0, s>>>(BN, N, at<uint32_t>(ws, L.pt_slot), at<uint32_t>(ws, L.pt_pos),
                                 at<uint32_t>(ws, L.full_off), at<uint32_t>(ws, L.bucket));
    int64_t bigb = (L.big_cap + 3) / 4;
    if (bigb > 1024) bigb = 1024;
    if (bigb < 1) bigb = 1;
    k_finalize<<<(unsigned)(pb + bigb), 256, 0, s>>>(
        points, BN, N, (uint32_t)d.n_v, (int32_t)bigb, at<uint32_t>(ws, L.pt_slot), at<uint32_t>(ws, L.vox_count),
        at<uint32_t>(ws, L.vox_off), at<uint32_t>(ws, L.full_off), at<uint32_t>(ws, L.bucket),
        at<uint32_t>(ws, L.big), L.big_cap, status, at<uint32_t>(ws, L.pt_list), at<float4>(ws, L.pt4));
    return hipGetLastError();
}

}  // namespace cagq
