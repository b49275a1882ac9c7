// The comparison methods CAGQ is measured against (Sec. 4, the latency and
// coverage tables), and the occupied-space coverage metric. None of this is
// CAGQ itself:
//   Random Point Sampling   the M points of smallest key
//                           (hi32(h(seed, 4, b, i)) << 32) | i, in ascending
//                           index: one 1024-thread workgroup per cloud finds
//                           the bound by a 4-pass 8-bit radix select over the
//                           keys' top halves, then compacts in index order;
//   Farthest Point Sampling from point 0, each next center the point with the
//                           largest d^2 to its nearest chosen center (ties to
//                           the lowest index): one workgroup per cloud keeps
//                           every point's distance in registers and reduces
//                           (d^2, -index) to the next center; up to 16384
//                           points it holds the points too, in spatial runs
//                           that a far-off center skips;
//   Ball Query              the first K points in index order with
//                           d^2 < R^2 among all N: one wave per center scans
//                           64 points at a time and stops at K;
//   coverage                occupied voxels holding at least one node point,
//                           marked per slot (each point's slot is kept by
//                           the grid build), then counted per cloud.
// d^2 = (dx*dx + dy*dy) + dz*dz in fp32, each operation rounded.
#include "cagq_internal.h"

namespace cagq {

namespace {

constexpr int kSelThreads = 1024;

__device__ __forceinline__ float dist2(const float* a, float bx, float by, float bz) {
    const float dx = a[0] - bx, dy = a[1] - by, dz = a[2] - bz;
    const float xx = dx * dx, yy = dy * dy, zz = dz * dz;
    const float s = xx + yy;
    return s + zz;
}

// ------------------------------------------------------------------ RPS

__global__ __launch_bounds__(kSelThreads) void k_rps(int32_t N, int32_t M, uint64_t seed,
                                                     int32_t* __restrict__ center_idx) {
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_prefix, s_need;
    __shared__ uint32_t s_wave[kSelThreads / kWave];
    const int32_t b = blockIdx.x;
    const int tid = threadIdx.x;
    const uint64_t hb = sm64(sm64(seed ^ 4ull) ^ (uint64_t)b);
    // radix select of the bound T on the keys' top halves, most significant
    // digit first: `need` keys with top half equal to T are taken
    uint32_t prefix = 0, need = (uint32_t)M;
    for (int pass = 0; pass < 4; ++pass) {
        const int sh = 24 - 8 * pass;
        const uint32_t hmask = pass == 0 ? 0u : ~0u << (sh + 8);
        for (int i = tid; i < 256; i += kSelThreads) hist[i] = 0;
        __syncthreads();
        for (int32_t i = tid; i < N; i += kSelThreads) {
            const uint32_t k = (uint32_t)(sm64(hb ^ (uint64_t)i) >> 32);
            if ((k & hmask) == prefix) atomicAdd(&hist[(k >> sh) & 255u], 1u);
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t acc = 0, d = 0;
            while (acc + hist[d] < need) acc += hist[d++];
            s_prefix = prefix | (d << sh);
            s_need = need - acc;
        }
        __syncthreads();
        prefix = s_prefix;
        need = s_need;
        __syncthreads();
    }
    // ordered compaction: keys below T, and the first `need` equal to T
    uint32_t base = 0, eq_base = 0;
    int32_t* out = center_idx + (size_t)b * M;
    const int lane = lane_id(), wv = tid / kWave;
    for (int32_t i0 = 0; i0 < N; i0 += kSelThreads) {
        const int32_t i = i0 + tid;
        const uint32_t k = i < N ? (uint32_t)(sm64(hb ^ (uint64_t)i) >> 32) : ~0u;
        const bool eq = i < N && k == prefix;
        // rank of this equal key among the equal keys so far
        const uint64_t eb = __ballot(eq);
        if (lane == 0) s_wave[wv] = (uint32_t)__popcll(eb);
        __syncthreads();
        uint32_t eoff = eq_base, etot = 0;
        for (int w = 0; w < kSelThreads / kWave; ++w) {
            if (w < wv) eoff += s_wave[w];
            etot += s_wave[w];
        }
        eoff += (uint32_t)__popcll(eb & ((1ull << lane) - 1));
        __syncthreads();
        const bool take = i < N && (k < prefix || (eq && eoff < need));
        const uint64_t tb = __ballot(take);
        if (lane == 0) s_wave[wv] = (uint32_t)__popcll(tb);
        __syncthreads();
        uint32_t off = base, tot = 0;
        for (int w = 0; w < kSelThreads / kWave; ++w) {
            if (w < wv) off += s_wave[w];
            tot += s_wave[w];
        }
        off += (uint32_t)__popcll(tb & ((1ull << lane) - 1));
        if (take) out[off] = i;
        base += tot;
        eq_base += etot;
        __syncthreads();
    }
}

// ------------------------------------------------------------------ FPS

// Lane i reads lane i - N of its row, or the row broadcasts of DPP control C;
// lanes without a source keep their own value.
template <int C, int RM>
__device__ __forceinline__ float dpp_own(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), C, RM, 0xF, false));
}

// Minimum over the wave, in every lane.
__device__ __forceinline__ float wave_fmin(float v) {
    v = fminf(v, dpp_own<0x111, 0xF>(v));  // row_shr:1, 2, 4, 8
    v = fminf(v, dpp_own<0x112, 0xF>(v));
    v = fminf(v, dpp_own<0x114, 0xF>(v));
    v = fminf(v, dpp_own<0x118, 0xF>(v));
    v = fminf(v, dpp_own<0x142, 0xA>(v));  // row_bcast:15 into rows 1 and 3
    v = fminf(v, dpp_own<0x143, 0xC>(v));  // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), kWave - 1));
}

// Maximum and minimum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_umax(uint32_t m) {
    m = max(m, dpp_row_shr<1>(m));
    m = max(m, dpp_row_shr<2>(m));
    m = max(m, dpp_row_shr<4>(m));
    m = max(m, dpp_row_shr<8>(m));
    return max(max((uint32_t)__builtin_amdgcn_readlane((int)m, 15), (uint32_t)__builtin_amdgcn_readlane((int)m, 31)),
               max((uint32_t)__builtin_amdgcn_readlane((int)m, 47), (uint32_t)__builtin_amdgcn_readlane((int)m, 63)));
}

__device__ __forceinline__ uint32_t wave_umin(uint32_t v) { return ~wave_umax(~v); }

// One halving of run_reduce: of N values per lane the lane keeps half, by bit
// BIT of its lane id, and takes the partner's part of them (DPP control C, a
// permutation of the row's 16 lanes that flips that bit).
template <int N, int BIT, int C, typename F>
__device__ __forceinline__ void reduce_half(uint32_t (&u)[N], bool hi, F op, uint32_t (&r)[N / 2]) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const uint32_t keep = hi ? u[i + N / 2] : u[i], give = hi ? u[i] : u[i + N / 2];
        r[i] = op(keep, (uint32_t)__builtin_amdgcn_mov_dpp((int)give, C, 0xF, 0xF, true));
    }
}

template <int C, typename F>
__device__ __forceinline__ uint32_t reduce_dpp(uint32_t v, F op) {
    return op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, C, 0xF, 0xF, true));
}

// Reduces PER values per lane over the wave, all of them together: lane l gets
// the reduction of value l % PER. PER - 1 exchanges inside the rows of 16
// lanes and two between them, where a reduction of each value takes six and
// reads it back through the scalar unit.
template <int PER, typename F>
__device__ __forceinline__ uint32_t run_reduce(uint32_t (&u)[PER], F op) {
    static_assert(PER == 4 || PER == 8 || PER == 16, "runs per wave");
    const int lane = lane_id();
    uint32_t a[PER / 2], b[PER / 4], v;
    if constexpr (PER == 16) {
        uint32_t c[2], d[1];
        reduce_half<16, 3, 0x140>(u, lane & 8, op, a);  // row_mirror
        reduce_half<8, 2, 0x141>(a, lane & 4, op, b);   // row_half_mirror
        reduce_half<4, 1, 0x1B>(b, lane & 2, op, c);    // quad_perm 3,2,1,0
        reduce_half<2, 0, 0xB1>(c, lane & 1, op, d);    // quad_perm 1,0,3,2
        v = d[0];
    } else if constexpr (PER == 8) {
        uint32_t c[1];
        reduce_half<8, 2, 0x141>(u, lane & 4, op, a);
        reduce_half<4, 1, 0x1B>(a, lane & 2, op, b);
        reduce_half<2, 0, 0xB1>(b, lane & 1, op, c);
        v = reduce_dpp<0x128>(c[0], op);  // row_ror:8
    } else {
        reduce_half<4, 1, 0x1B>(u, lane & 2, op, a);
        reduce_half<2, 0, 0xB1>(a, lane & 1, op, b);
        v = reduce_dpp<0x128>(reduce_dpp<0x124>(b[0], op), op);  // row_ror:4, row_ror:8
    }
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op((uint32_t)p[0], (uint32_t)p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return op((uint32_t)q[0], (uint32_t)q[1]);
}

// Farthest Point Sampling of clouds of at most 1024 * PER points: one
// workgroup per cloud, every point's coordinates and distance in registers.
// The picks are a serial chain; what a pick costs is what its slowest wave
// does between two barriers. So that a pick touches few points, the
// workgroup first sorts its points by the Morton code of a 16^3 grid over
// their bounding box (a counting sort in LDS): register k of a wave then
// holds 64 neighbouring points (a run), whose bounding box and largest
// distance sit in the wave's lane k. A new center changes no distance of a
// run when its distance to the box is at least the run's largest distance.
// That holds exactly in fp32: the distance to the box is computed with the
// same operations in the same order as a point's, from per-axis gaps no
// larger than any point's, and every rounding is monotonic. Points that are
// not finite are left out of the boxes: their distance to any center is
// infinite or not a number, so they keep the infinity they start with, as
// does every point against a center that is not finite.
// Measured: 4 clouds of 8192 points, 1024 picks: 1.99 -> 1.00 ms (a pick re-reading
// and updating every point: 1.95 us, now 0.95).
// Runs of a wave that a pick updates one by one, each with its own reduction;
// when it reaches more, it updates every run, with one reduction for all of
// them (PER / 2 instead of PER / 4: 4 x 8192 points of a room, 1024 picks 1.02
// -> 1.08 ms). So that a cloud whose runs are no neighbours (one point far from
// the rest takes the whole of the sort's grid, or most points do not differ)
// costs a pick no more than k_fps does: 4 x 16384 points and an outlier, 2048
// picks: k_fps 6.0 ms, one by one 6.7, now 4.0; points that are not numbers 6.0,
// 9.3 and 1.5.
template <int PER>
constexpr int kFewRuns = PER / 4;

template <int PER>
__global__ __launch_bounds__(kSelThreads) void k_fps_runs(const float* __restrict__ points, int32_t N, int32_t M,
                                                          int32_t* __restrict__ center_idx) {
    constexpr int kW = kSelThreads / kWave;
    constexpr int kCells = 4096;
    static_assert(PER <= 16 && kW == 16, "a wave's runs, and the waves, fit in 16 lanes");
    __shared__ uint32_t s_cell[kCells];
    __shared__ uint16_t s_perm[kSelThreads * PER];
    __shared__ float s_box[6][kW];
    __shared__ uint32_t s_wave[kW];
    __shared__ uint64_t s_key[2][kW];
    __shared__ float4 s_xyz[2][kW];
    const int32_t b = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    constexpr int nt = kSelThreads, nw = kW;
    const float* P = points + (size_t)b * N * 3;
    int32_t* out = center_idx + (size_t)b * M;
    const float inf = __builtin_inff();

    // bounding box of the finite points
    float lo[3] = {inf, inf, inf}, hi[3] = {-inf, -inf, -inf};
    for (int32_t i = tid; i < N; i += nt) {
        const float c[3] = {P[(size_t)i * 3], P[(size_t)i * 3 + 1], P[(size_t)i * 3 + 2]};
        if (isfinite(c[0]) && isfinite(c[1]) && isfinite(c[2])) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = fminf(lo[a], c[a]);
                hi[a] = fmaxf(hi[a], c[a]);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_fmin(lo[a]);
        hi[a] = -wave_fmin(-hi[a]);
        if (lane == 0) {
            s_box[a][wv] = lo[a];
            s_box[3 + a][wv] = hi[a];
        }
    }
    for (int i = tid; i < kCells; i += nt) s_cell[i] = 0u;
    __syncthreads();
    float scale[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int w = 0; w < nw; ++w) {
            lo[a] = fminf(lo[a], s_box[a][w]);
            hi[a] = fmaxf(hi[a], s_box[3 + a][w]);
        }
        scale[a] = 16.0f / (hi[a] - lo[a]);  // a flat or empty box: not finite, cell 0
    }
    // the cell of a point (any cell will do for one that is not finite: the
    // order decides only how well the runs' boxes fit)
    auto cell_of = [&](int32_t i) {
        uint32_t m = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float t = (P[(size_t)i * 3 + a] - lo[a]) * scale[a];
            uint32_t q = t >= 0.0f && t < 16.0f ? (uint32_t)t : (t >= 16.0f ? 15u : 0u);
            q = (q | (q << 4)) & 0xC3u;
            q = (q | (q << 2)) & 0x249u;
            m |= q << a;
        }
        return m;
    };
    uint32_t cell[PER], pos[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int32_t i = tid + k * nt;
        cell[k] = pos[k] = 0;
        if (i < N) {
            cell[k] = cell_of(i);
            pos[k] = atomicAdd(&s_cell[cell[k]], 1u);
        }
    }
    __syncthreads();
    {   // exclusive scan of the cells, kCells / nt of them per thread
        const int per = kCells / nt;
        uint32_t sum = 0;
        for (int j = 0; j < per; ++j) sum += s_cell[tid * per + j];
        const uint32_t incl = wave_incl_scan<uint32_t>(sum);
        if (lane == kWave - 1) s_wave[wv] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (int w = 0; w < wv; ++w) run += s_wave[w];
        for (int j = 0; j < per; ++j) {
            const uint32_t c = s_cell[tid * per + j];
            s_cell[tid * per + j] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (tid + k * nt < N) s_perm[s_cell[cell[k]] + pos[k]] = (uint16_t)(tid + k * nt);
    __syncthreads();

    // this wave's points, PER runs of 64; a place past the end holds no
    // number, distance 0 and the index that loses every tie
    float x[PER], y[PER], z[PER], dm[PER];
    uint32_t id[PER];
    float bl[3] = {inf, inf, inf}, bh[3] = {-inf, -inf, -inf};  // lane k: the box of run k
    uint32_t rmax = 0;                                          // lane k: bits of run k's largest distance
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int32_t at = (wv * PER + k) * kWave + lane;
        const bool in = at < N;
        id[k] = in ? (uint32_t)s_perm[at] : 0xFFFFFFFFu;
        const float* p = P + (size_t)(in ? id[k] : 0u) * 3;
        x[k] = in ? p[0] : __builtin_nanf("");
        y[k] = p[1];
        z[k] = p[2];
        dm[k] = in ? inf : 0.0f;
        const bool any = __ballot(in) != 0;
        rmax = lane == k && any ? __float_as_uint(inf) : rmax;
    }
    const auto least = [](uint32_t p, uint32_t q) {
        return __float_as_uint(fminf(__uint_as_float(p), __uint_as_float(q)));
    };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        uint32_t l[PER], h[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const bool fin = isfinite(x[k]) && isfinite(y[k]) && isfinite(z[k]);  // false past the end
            const float c = a == 0 ? x[k] : a == 1 ? y[k] : z[k];
            l[k] = __float_as_uint(fin ? c : inf);
            h[k] = __float_as_uint(fin ? -c : inf);
        }
        bl[a] = __uint_as_float(run_reduce<PER>(l, least));
        bh[a] = -__uint_as_float(run_reduce<PER>(h, least));
    }

    // the wave's farthest point: key (bits(d^2) << 32) | ~index, coordinates
    uint64_t wkey = 0;
    float wx = 0.f, wy = 0.f, wz = 0.f;
    auto find_best = [&]() {
        uint32_t m = lane < PER ? rmax : 0u;
        m = max(m, dpp_row_shr<1>(m));
        m = max(m, dpp_row_shr<2>(m));
        m = max(m, dpp_row_shr<4>(m));
        m = max(m, dpp_row_shr<8>(m));
        const uint32_t wm = (uint32_t)__builtin_amdgcn_readlane((int)m, 15);
        const uint64_t runs = __ballot(lane < PER && rmax == wm);
        uint32_t ci = 0xFFFFFFFFu;
        float px = 0.f, py = 0.f, pz = 0.f;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if ((runs >> k) & 1ull) {
                const bool better = __float_as_uint(dm[k]) == wm && id[k] < ci;
                ci = better ? id[k] : ci;
                px = better ? x[k] : px;
                py = better ? y[k] : py;
                pz = better ? z[k] : pz;
            }
        }
        uint64_t who = __ballot(ci != 0xFFFFFFFFu);
        if (who & (who - 1)) {  // a tie between lanes: the lowest index
            who = __ballot(ci == wave_umin(ci));
        }
        if (!who) return;  // a wave without points keeps key 0
        const int l = __ffsll((unsigned long long)who) - 1;
        wkey = ((uint64_t)wm << 32) | (uint32_t)~(uint32_t)__builtin_amdgcn_readlane((int)ci, l);
        wx = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(px), l));
        wy = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(py), l));
        wz = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(pz), l));
    };
    find_best();

    uint32_t cur = 0;
    float cx = P[0], cy = P[1], cz = P[2];
    for (int32_t j = 0;; ++j) {
        if (tid == 0) out[j] = (int32_t)cur;
        if (j + 1 >= M) break;
        // the runs the center may change: a lane per run
        const float gx = fmaxf(fmaxf(bl[0] - cx, cx - bh[0]), 0.0f);
        const float gy = fmaxf(fmaxf(bl[1] - cy, cy - bh[1]), 0.0f);
        const float gz = fmaxf(fmaxf(bl[2] - cz, cz - bh[2]), 0.0f);
        const float gxx = gx * gx, gyy = gy * gy, gzz = gz * gz;
        const float gxy = gxx + gyy;
        const float gap = gxy + gzz;
        // (none when it is not finite)
        const bool fin = isfinite(cx) && isfinite(cy) && isfinite(cz);
        const uint64_t need = __ballot(fin && lane < PER && gap < __uint_as_float(rmax));
        if (need) {
            auto update = [&](int k) {
                const float dx = x[k] - cx, dy = y[k] - cy, dz = z[k] - cz;
                const float xx = dx * dx, yy = dy * dy, zz = dz * dz;
                const float sxy = xx + yy;
                const float d = sxy + zz;
                dm[k] = d < dm[k] ? d : dm[k];
                return __float_as_uint(dm[k]);  // distances order as their bits
            };
            if (__popcll(need) > kFewRuns<PER>) {
                uint32_t u[PER];
#pragma unroll
                for (int k = 0; k < PER; ++k) u[k] = update(k);
                rmax = run_reduce<PER>(u, [](uint32_t p, uint32_t q) { return max(p, q); });
            } else {
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    if ((need >> k) & 1ull) {
                        const uint32_t m = wave_umax(update(k));
                        rmax = lane == k ? m : rmax;
                    }
                }
            }
            find_best();
        }
        // the farthest of the waves' points; two buffers, so that one barrier
        // a pick is enough
        const int par = j & 1;
        if (lane == 0) {
            s_key[par][wv] = wkey;
            s_xyz[par][wv] = make_float4(wx, wy, wz, 0.f);
        }
        lds_barrier();
        const uint64_t key = lane < nw ? s_key[par][lane] : 0ull;
        const float4 c = s_xyz[par][lane < nw ? lane : 0];
        uint32_t m = (uint32_t)(key >> 32);
        m = max(m, dpp_row_shr<1>(m));
        m = max(m, dpp_row_shr<2>(m));
        m = max(m, dpp_row_shr<4>(m));
        m = max(m, dpp_row_shr<8>(m));
        const uint32_t top = (uint32_t)__builtin_amdgcn_readlane((int)m, 15);
        uint64_t who = __ballot(lane < nw && (uint32_t)(key >> 32) == top);
        if (who & (who - 1)) {
            uint32_t low = ((who >> lane) & 1ull) ? (uint32_t)key : 0u;
            uint32_t mx = low;
            mx = max(mx, dpp_row_shr<1>(mx));
            mx = max(mx, dpp_row_shr<2>(mx));
            mx = max(mx, dpp_row_shr<4>(mx));
            mx = max(mx, dpp_row_shr<8>(mx));
            mx = (uint32_t)__builtin_amdgcn_readlane((int)mx, 15);
            who = __ballot(((who >> lane) & 1ull) && (uint32_t)key == mx);
        }
        const int w = __ffsll((unsigned long long)who) - 1;
        cur = ~(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, w);
        cx = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c.x), w));
        cy = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c.y), w));
        cz = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(c.z), w));
    }
}

// Larger and smaller clouds, and few picks: every thread keeps PER distances
// in registers, and every pick reads the cloud again.
template <int PER>
__global__ __launch_bounds__(kSelThreads) void k_fps(const float* __restrict__ points, int32_t N, int32_t M,
                                                     int32_t* __restrict__ center_idx) {
    __shared__ uint64_t s_best[kSelThreads / kWave];
    __shared__ int32_t s_cur;
    const int32_t b = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
    const float* P = points + (size_t)b * N * 3;
    int32_t* out = center_idx + (size_t)b * M;
    float dmin[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) dmin[k] = __builtin_inff();
    // the cloud as a raw buffer: point tid + k * 1024 sits at the thread's
    // byte offset plus a constant, so no per-point address stays live
    // across the iterations (loads past the buffer's end read 0)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)P, (short)0, N * 12, 0x00020000);
    const int vo = tid * 12;
    int32_t cur = 0;
    for (int32_t j = 0; j < M; ++j) {
        if (tid == 0) out[j] = cur;
        const float cx = P[(size_t)cur * 3 + 0], cy = P[(size_t)cur * 3 + 1], cz = P[(size_t)cur * 3 + 2];
        // this thread's farthest point (its indices ascend with k, so a
        // strict comparison keeps the lowest index of a tie)
        float bd = -1.0f;
        int32_t bi = 0;
#pragma unroll
        for (int k0 = 0; k0 < PER; k0 += 4) {
#pragma unroll
            for (int k = k0; k < k0 + 4 && k < PER; ++k) {
                const int32_t i = tid + k * kSelThreads;
                // one 12-byte load per point
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, vo, k * kSelThreads * 12, 0);
                const float px = __uint_as_float(v[0]), py = __uint_as_float(v[1]), pz = __uint_as_float(v[2]);
                if (i < N) {
                    const float dx = px - cx, dy = py - cy, dz = pz - cz;
                    const float xx = dx * dx, yy = dy * dy, zz = dz * dz;
                    const float sxy = xx + yy;
                    const float d = sxy + zz;
                    dmin[k] = d < dmin[k] ? d : dmin[k];
                    if (dmin[k] > bd) {
                        bd = dmin[k];
                        bi = i;
                    }
                }
            }
            // a few points' loads in flight at a time keep the distances in
            // registers
            __builtin_amdgcn_sched_barrier(0);
        }
        // (bits(d^2) << 32) | ~i: the largest is the farthest point, ties to
        // the lowest index (d^2 >= 0, so its bits order as the value)
        uint64_t best = bd < 0.0f ? 0ull : ((uint64_t)__float_as_uint(bd) << 32) | (uint32_t)~(uint32_t)bi;
        best = wave_max64(best);
        if (lane == 0) s_best[wv] = best;
        __syncthreads();
        if (tid < kWave) {
            uint64_t v = tid < kSelThreads / kWave ? s_best[tid] : 0ull;
            v = wave_max64(v);
            if (tid == 0) s_cur = (int32_t)~(uint32_t)v;
        }
        __syncthreads();
        cur = s_cur;
    }
}

// ------------------------------------------------------------------ Ball Query

constexpr int kBallThreads = 256;

__global__ __launch_bounds__(kBallThreads) void k_ball(const float* __restrict__ points, int32_t N, int32_t M,
                                                       int32_t total, const int32_t* __restrict__ center_idx,
                                                       int32_t K, float r2, int32_t* __restrict__ node_idx,
                                                       int32_t* __restrict__ n_valid) {
    const int lane = lane_id();
    const int32_t cid = (int32_t)xcd_block(blockIdx.x, gridDim.x) * (kBallThreads / kWave) + threadIdx.x / kWave;
    if (cid >= total) return;  // whole waves leave together
    const int32_t b = cid / M;
    const float* P = points + (size_t)b * N * 3;
    int32_t* out = node_idx + (size_t)cid * K;
    const int32_t ci = center_idx[cid];
    int32_t n = 0, first = -1;
    if (ci >= 0 && ci < N) {
        const float cx = P[(size_t)ci * 3 + 0], cy = P[(size_t)ci * 3 + 1], cz = P[(size_t)ci * 3 + 2];
        for (int32_t i0 = 0; i0 < N && n < K; i0 += kWave) {
            const int32_t i = i0 + lane;
            const bool in = i < N && dist2(P + (size_t)i * 3, cx, cy, cz) < r2;
            const uint64_t bal = __ballot(in);
            const int32_t pos = n + (int32_t)__popcll(bal & ((1ull << lane) - 1));
            if (in && pos < K) out[pos] = i;
            if (bal && first < 0) first = i0 + (__ffsll((unsigned long long)bal) - 1);
            n += (int32_t)__popcll(bal);
        }
    }
    n = n < K ? n : K;
    for (int32_t k = n + lane; k < K; k += kWave) out[k] = first;  // -1 when nothing is inside
    if (lane == 0) n_valid[cid] = n;
}

// ------------------------------------------------------------------ coverage

__global__ void k_cov_clear(uint4* __restrict__ p, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

struct CovGrid {
    float o[3], s[3];
    int32_t D[3];
    int64_t W;
};

// Every valid node point stores 1 into the byte of its voxel's slot (the same
// value from every writer: no atomic needed). The slot comes from the point's
// coordinates by the voxelization rule and the occupancy words.
__global__ __launch_bounds__(256) void k_cov_mark(const float* __restrict__ P, int32_t N, int32_t M, int32_t K,
                                                  int64_t total, CovGrid g, const int32_t* __restrict__ node_idx,
                                                  const int32_t* __restrict__ n_valid,
                                                  const uint64_t* __restrict__ bitmap,
                                                  const uint32_t* __restrict__ word_rank, uint8_t* __restrict__ mark) {
    const int64_t t = (int64_t)xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int64_t cj = t / K;
    const int32_t k = (int32_t)(t - cj * K);
    if (k >= n_valid[cj]) return;
    const int32_t i = node_idx[t];
    if (i < 0 || i >= N) return;
    const int32_t b = (int32_t)(cj / M);
    const float* p = P + ((size_t)b * N + i) * 3;
    uint32_t gg[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float c = p[a];
        gg[a] = isfinite(c) ? (uint32_t)axis_index(c, g.o[a], g.s[a], g.D[a]) : 0u;
    }
    const uint32_t lin = gg[0] + (uint32_t)g.D[0] * (gg[1] + (uint32_t)g.D[1] * gg[2]);
    const int32_t slot = slot_of(bitmap + (size_t)b * g.W, word_rank + (size_t)b * g.W, lin);
    if (slot >= 0) mark[(size_t)b * N + slot] = 1;
}

__global__ __launch_bounds__(1024) void k_cov_count(int32_t N, const int32_t* __restrict__ nvox,
                                                    const uint8_t* __restrict__ mark, int32_t* __restrict__ covered) {
    __shared__ uint32_t s_wave[1024 / kWave];
    const int32_t b = blockIdx.x;
    const int32_t nv = nvox[b];
    const uint8_t* m = mark + (size_t)b * N;
    uint32_t c = 0;
    for (int32_t s = threadIdx.x; s < nv; s += blockDim.x) c += m[s];
    c = wave_sum<uint32_t>(c);
    if (lane_id() == 0) s_wave[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < 1024 / kWave; ++w) t += s_wave[w];
        covered[b] = (int32_t)t;
    }
}

}  // namespace

// Picks and points from which k_fps_runs is used: its sort and its runs' boxes
// cost about 20 us, and a pick over up to 2048 points gains little from it.
// 4 clouds, 48 picks: 2049 points 48 us by k_fps, 45 by k_fps_runs; 8193 points
// 96 and 78; 16384 points 143 and 100.
constexpr int32_t kRunsMinN = 2049;
constexpr int32_t kRunsMinM = 48;

hipError_t launch_sample_points(const float* points, int32_t B, int32_t N, int32_t M, int32_t mode, uint64_t seed,
                                int32_t* center_idx, hipStream_t s) {
    if (mode == 0) {
        k_rps<<<B, kSelThreads, 0, s>>>(N, M, seed, center_idx);
    } else {
        const int32_t per = (N + kSelThreads - 1) / kSelThreads;
        // points in registers, sorted into runs, up to 16384 of them (the
        // most a workgroup's registers hold)
        const bool runs = per <= 16 && N >= kRunsMinN && M >= kRunsMinM;
        if (runs && per <= 4)
            k_fps_runs<4><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else if (runs && per <= 8)
            k_fps_runs<8><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else if (runs)
            k_fps_runs<16><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else if (per <= 4)
            k_fps<4><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else if (per <= 16)
            k_fps<16><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else if (per <= 40)
            k_fps<40><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
        else
            k_fps<80><<<B, kSelThreads, 0, s>>>(points, N, M, center_idx);
    }
    return hipGetLastError();
}

hipError_t launch_ball_query(const float* points, int32_t B, int32_t N, const int32_t* center_idx, int32_t M,
                             int32_t K, float radius2, int32_t* node_idx, int32_t* n_valid, hipStream_t s) {
    const int32_t total = B * M;
    constexpr int WPB = kBallThreads / kWave;
    k_ball<<<(unsigned)((total + WPB - 1) / WPB), kBallThreads, 0, s>>>(points, N, M, total, center_idx, K, radius2,
                                                                        node_idx, n_valid);
    return hipGetLastError();
}

hipError_t launch_coverage(const Layout& L, const cagq_grid_desc& d, const float* points, void* ws,
                           const int32_t* node_idx, const int32_t* n_valid, int32_t M, int32_t K, int32_t* covered,
                           hipStream_t s) {
    const size_t BN = (size_t)L.B * L.N;
    uint8_t* mark = at<uint8_t>(ws, L.cov_mark);
    const size_t n16 = (BN + 15) / 16;
    k_cov_clear<<<(unsigned)((n16 + 255) / 256 < 2048 ? (n16 + 255) / 256 : 2048), 256, 0, s>>>(
        reinterpret_cast<uint4*>(mark), n16);
    const int64_t total = (int64_t)L.B * M * K;
    CovGrid g;
    for (int a = 0; a < 3; ++a) {
        g.o[a] = d.origin[a];
        g.s[a] = d.voxel_size[a];
        g.D[a] = d.dims[a];
    }
    g.W = L.W;
    k_cov_mark<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(points, L.N, M, K, total, g, node_idx, n_valid,
                                                               at<uint64_t>(ws, L.bitmap),
                                                               at<uint32_t>(ws, L.word_rank), mark);
    k_cov_count<<<L.B, 1024, 0, s>>>(L.N, at<int32_t>(ws, L.nvox), mark, covered);
    return hipGetLastError();
}

}  // namespace cagq
