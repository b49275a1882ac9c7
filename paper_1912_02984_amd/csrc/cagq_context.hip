// Context lists for grid context pooling (Sec. 3.3: the context feature of a
// group is pooled over all of its context points, which CAGQ has already
// associated with the center voxel). The context of center voxel v is the
// stored points of the occupied voxels of pi(v), voxels in ascending linear
// id, each voxel's stored points ascending; v itself need not be occupied.
//
// A row segment of the (2r+1)^3 block holds consecutive slots, and the
// stored points are grouped by slot, so the context of one grid row is one
// contiguous range of the stored list: the block is (2r+1)^2 ranges.
//   k_ctx_count      per center the context count c (range lengths from the
//                    offsets array), and a decoupled look-back scan over the
//                    batch that writes the CSR offsets;
//   k_ctx_fill       one group of 16 lanes per center copies its ranges.
#include "cagq_internal.h"

namespace cagq {

namespace {

constexpr int kFillG = 16;  // lanes per center in the fill
constexpr int kFillU = 4;   // entries a lane loads at once (one at a time: 10.1 us at 4 x 8192 centers, four: 8.1)
constexpr int kFillThreads = 256;

// Most centers of a launch with one center per thread (k_ctx_count): four take
// a thread's loads four times, which grow with the rows, and save three of four
// tiles' atomics. One / four: r = 1, 65536 centers 15.7 / 21.6 us, 98304 24.4 /
// 22.5, 2^20 192 / 124; r = 2, 100000 33 / 43; r = 3, 100000 49 / 73.
constexpr int64_t ctx_one(int rad) { return (int64_t)(2 + rad) << 15; }


// The grid, and the launch's divisions by multiply and shift (a division by a
// kernel argument, 64-bit ones above all, costs more instructions than the
// rest of a center's set-up).
struct CtxGrid {
    GridDims g;
    int64_t V;
    Magic d0, d01, mm;  // division by D_x, by D_x * D_y and by M

    __host__ CtxGrid(const cagq_grid_desc& d, int32_t M) {
        for (int a = 0; a < 3; ++a) g.D[a] = d.dims[a];
        V = (int64_t)d.dims[0] * d.dims[1] * d.dims[2];
        d0 = make_magic((uint32_t)d.dims[0]);
        d01 = make_magic((uint32_t)d.dims[0] * (uint32_t)d.dims[1]);
        mm = make_magic((uint32_t)M);
    }

    // Cloud and voxel coordinates of center j, or false when its lin is
    // outside the grid.
    __device__ __forceinline__ bool center(const int32_t* center_lin, int64_t j, int32_t& b, int32_t& x, int32_t& y,
                                           int32_t& z) const {
        const int32_t l = center_lin[j];
        b = (int32_t)udiv((uint32_t)j, mm);
        if (l < 0 || (int64_t)l >= V) return false;
        const uint32_t zq = udiv((uint32_t)l, d01);
        const uint32_t rem = (uint32_t)l - zq * (uint32_t)g.D[0] * (uint32_t)g.D[1];
        const uint32_t yq = udiv(rem, d0);
        x = (int32_t)(rem - yq * (uint32_t)g.D[0]), y = (int32_t)yq, z = (int32_t)zq;
        return true;
    }
};

// A thread takes `items` centers in a row, whose rows' loads go out together:
// one, or four (KEEP of them, their counts kept in registers), or more where
// there are more centers than the points' and kCtxTiles tiles' descriptors hold
// (then each is counted twice). The descriptors, the ticket and the count of
// tiles that have finished their look-back start at zero: every build clears
// them, and the last tile to finish clears them again for the next call, so
// that the call is one launch. Bound by its chain of loads (center, rows,
// offsets) and the look-back: 4 x 8192 centers, 0.05 voxels: 9 us in tiles of
// 256 centers, against 21 us in tiles of 1024 and 26 us with the launches that
// cleared and unflagged the descriptors in the offsets array. Every tile takes
// two atomics on one line, ~20 ns each, which bind from some 400 tiles on: four
// centers a thread then (ctx_one), 4 x 81920 centers 63 -> 49 us.
template <int RAD, int KEEP>
__global__ __launch_bounds__(kScanThreads) void k_ctx_count(int32_t N, int32_t M, int64_t total, int32_t items,
                                                            int64_t W, CtxGrid g,
                                                            const uint64_t* __restrict__ bitmap,
                                                            const uint32_t* __restrict__ word_rank,
                                                            const uint32_t* __restrict__ vox_off,
                                                            const int32_t* __restrict__ center_lin,
                                                            int64_t* __restrict__ off, uint64_t* __restrict__ desc,
                                                            int* __restrict__ status) {
    constexpr int S = 2 * RAD + 1;
    __shared__ uint32_t s_ticket, s_done;
    __shared__ uint64_t s_wave[kScanThreads / kWave];
    __shared__ uint64_t s_prefix;
    if (threadIdx.x == 0) s_ticket = atomicAdd((unsigned*)&status[kStTicketCtx], 1u);
    __syncthreads();
    const int64_t tile = s_ticket;
    const int64_t j0 = (tile * kScanThreads + (int64_t)threadIdx.x) * items;
    // context points of center j
    auto count = [&](int64_t j) {
        uint32_t c = 0;
        int32_t b, x, y, z;
        if (j >= total) return c;
        if (!g.center(center_lin, j, b, x, y, z)) {
            raise_error(status, CAGQ_ERR_CENTER_NOT_OCCUPIED);
            return c;
        }
        const uint64_t* bm = bitmap + (size_t)b * W;
        const uint32_t* wr = word_rank + (size_t)b * W;
        const uint32_t* vo = vox_off + (size_t)b * (N + 1);
        for (int pl = 0; pl < S; ++pl) {
            int32_t yy[S], zz[S];
            GridRow r[S];
            uint32_t lo[S], hi[S];
#pragma unroll
            for (int i = 0; i < S; ++i) {
                yy[i] = y + i - RAD;
                zz[i] = z + pl - RAD;
            }
            load_rows<S>(bm, wr, g.g, x, yy, zz, RAD, r);
#pragma unroll
            for (int i = 0; i < S; ++i) {
                lo[i] = vo[r[i].first];
                hi[i] = vo[r[i].first + (uint32_t)__popc(r[i].mask)];
            }
#pragma unroll
            for (int i = 0; i < S; ++i) c += hi[i] - lo[i];
        }
        return c;
    };
    uint64_t sum = 0;
    uint32_t kept[KEEP];
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        kept[i] = count(j0 + i);
        sum += kept[i];
    }
    for (int32_t i = KEEP; i < items; ++i) sum += count(j0 + i);
    uint64_t agg;
    const uint64_t excl = block_excl_scan(sum, s_wave, &agg);
    uint64_t run = tile_lookback(desc, tile, agg, &s_prefix) + excl;
    if (j0 == 0) off[0] = 0;
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        run += kept[i];
        if (j0 + i < total) off[j0 + i + 1] = (int64_t)run;
    }
    for (int32_t i = KEEP; i < items && j0 + i < total; ++i) {
        run += count(j0 + i);
        off[j0 + i + 1] = (int64_t)run;
    }
    // past the look-back (its barrier): this tile reads no descriptor any
    // more; thread 0, which stored its own, waits until that has arrived, so
    // that the last tile's zeros come after it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0) s_done = atomicAdd((unsigned*)&status[kStCtxDone], 1u);
    __syncthreads();
    if (s_done != gridDim.x - 1) return;
    for (uint32_t t = threadIdx.x; t < gridDim.x; t += kScanThreads) st_desc(desc + t, 0ull);
    if (threadIdx.x == 0) {
        status[kStTicketCtx] = 0;
        status[kStCtxDone] = 0;
    }
}

template <int RAD>
__global__ __launch_bounds__(kFillThreads) void k_ctx_fill(int32_t N, int32_t M, int64_t total, int64_t W,
                                                           CtxGrid g, const uint64_t* __restrict__ bitmap,
                                                           const uint32_t* __restrict__ word_rank,
                                                           const uint32_t* __restrict__ vox_off,
                                                           const uint32_t* __restrict__ pt_list,
                                                           const int32_t* __restrict__ center_lin,
                                                           const int64_t* __restrict__ off,
                                                           int32_t* __restrict__ ctx_idx, int64_t capacity,
                                                           int* __restrict__ status) {
    constexpr int S = 2 * RAD + 1;
    constexpr int GPB = kFillThreads / kFillG;
    __shared__ uint32_t s_pre[GPB][kFillG];
    __shared__ uint32_t s_st[GPB][kFillG];
    const int gb = threadIdx.x / kFillG, lg = threadIdx.x & (kFillG - 1);
    const int64_t j = (int64_t)xcd_block(blockIdx.x, gridDim.x) * GPB + gb;
    // whole groups leave together: the group steps below need every lane
    if (j >= total) return;
    int32_t b, x, y, z;
    if (!g.center(center_lin, j, b, x, y, z)) return;  // an empty context
    const uint64_t* bm = bitmap + (size_t)b * W;
    const uint32_t* wr = word_rank + (size_t)b * W;
    const uint32_t* vo = vox_off + (size_t)b * (N + 1);
    const uint32_t* pl = pt_list + (size_t)b * N;
    int64_t dst = off[j];
    bool over = false;
    for (int q0 = 0; q0 < S * S; q0 += kFillG) {
        const int q = q0 + lg;
        uint32_t st = 0, len = 0;
        if (q < S * S) {
            const GridRow r = load_row(bm, wr, g.g, x, y + q % S - RAD, z + q / S - RAD, RAD);
            st = vo[r.first];
            len = vo[r.first + (uint32_t)__popc(r.mask)] - st;
        }
        // inclusive scan of the range lengths across the group
        uint32_t incl = len;
#pragma unroll
        for (int d = 1; d < kFillG; d <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)incl, d, kFillG);
            if (lg >= d) incl += o;
        }
        s_pre[gb][lg] = incl - len;
        s_st[gb][lg] = st;
        const uint32_t tot = (uint32_t)__shfl((int)incl, kFillG - 1, kFillG);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // kFillU entries per lane at a time, their loads in flight together
        for (uint32_t e0 = (uint32_t)lg; e0 < tot; e0 += kFillU * kFillG) {
            uint32_t v[kFillU];
#pragma unroll
            for (int u = 0; u < kFillU; ++u) {
                const uint32_t e = e0 + u * kFillG < tot ? e0 + u * kFillG : e0;
                // the last range starting at or before e (empty ranges share starts)
                uint32_t lo = 0;
#pragma unroll
                for (int h = kFillG / 2; h > 0; h >>= 1)
                    if (s_pre[gb][lo + h] <= e) lo += h;
                v[u] = pl[s_st[gb][lo] + (e - s_pre[gb][lo])];
            }
#pragma unroll
            for (int u = 0; u < kFillU; ++u) {
                const uint32_t e = e0 + u * kFillG;
                const int64_t k = dst + (int64_t)e;
                if (e < tot && k < capacity) ctx_idx[k] = (int32_t)v[u];
                over = over || (e < tot && k >= capacity);
            }
        }
        dst += tot;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (over) raise_error(status, CAGQ_ERR_CAPACITY);
}

}  // namespace

hipError_t launch_context_offsets(const Layout& L, const cagq_grid_desc& d, void* ws, const int32_t* center_lin,
                                  int32_t M, int64_t* ctx_off, hipStream_t s) {
    const CtxGrid g(d, M);
    const int64_t total = (int64_t)L.B * M;
    int64_t items = (total + L.ctx_tiles * kScanThreads - 1) / (L.ctx_tiles * kScanThreads);
    const bool four = items > 1 || total > ctx_one(d.radius);
    if (four && items < 4) items = 4;
    const int64_t tiles = (total + items * kScanThreads - 1) / (items * kScanThreads);
    if (tiles > L.ctx_tiles) return hipErrorInvalidValue;  // unreachable by the choice of items
    auto go = [&](auto kern) {
        kern<<<(unsigned)tiles, kScanThreads, 0, s>>>(L.N, M, total, (int32_t)items, L.W, g,
                                                      at<uint64_t>(ws, L.bitmap), at<uint32_t>(ws, L.word_rank),
                                                      at<uint32_t>(ws, L.vox_off), center_lin, ctx_off,
                                                      at<uint64_t>(ws, L.ctx_desc), at<int>(ws, L.status));
    };
    if (d.radius == 1)
        four ? go(k_ctx_count<1, 4>) : go(k_ctx_count<1, 1>);
    else if (d.radius == 2)
        four ? go(k_ctx_count<2, 4>) : go(k_ctx_count<2, 1>);
    else
        four ? go(k_ctx_count<3, 4>) : go(k_ctx_count<3, 1>);
    return hipGetLastError();
}

hipError_t launch_context_list(const Layout& L, const cagq_grid_desc& d, void* ws, const int32_t* center_lin,
                               int32_t M, const int64_t* ctx_off, int32_t* ctx_idx, int64_t capacity,
                               hipStream_t s) {
    const CtxGrid g(d, M);
    const int64_t total = (int64_t)L.B * M;
    constexpr int GPB = kFillThreads / kFillG;
    const unsigned blocks = (unsigned)((total + GPB - 1) / GPB);
    auto go = [&](auto kern) {
        kern<<<blocks, kFillThreads, 0, s>>>(L.N, M, total, L.W, g, at<uint64_t>(ws, L.bitmap),
                                             at<uint32_t>(ws, L.word_rank), at<uint32_t>(ws, L.vox_off),
                                             at<uint32_t>(ws, L.pt_list), center_lin, ctx_off, ctx_idx, capacity,
                                             at<int>(ws, L.status));
    };
    if (d.radius == 1)
        go(k_ctx_fill<1>);
    else if (d.radius == 2)
        go(k_ctx_fill<2>);
    else
        go(k_ctx_fill<3>);
    return hipGetLastError();
}

}  // namespace cagq
