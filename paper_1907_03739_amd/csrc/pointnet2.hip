// The PointNet++ primitives that PVCNN++ keeps around its PVConv layers
// (Section 5.2 "Models": PointNet++ extended with PVConv), as PointNet++
// defines them: iterative farthest point sampling and ball-query grouping
// (set abstraction), and inverse-distance interpolation over the three
// nearest neighbours (feature propagation). gfx950, wave64.
//
// Every choice of an index (the farthest point, ball membership, the three
// nearest neighbours) compares fp32 squared distances formed as
// fma(dz, dz, fma(dy, dy, dx * dx)), dx = x_j - x_c, with ties going to the
// lower index: the same choices on every run and in every launch
// configuration.
#include "pv_common.h"
#include "pv_wave.h"

namespace {

__device__ __forceinline__ float sqdist(float ax, float ay, float az, float bx, float by,
                                        float bz) {
#pragma clang fp contract(off)
    const float dx = ax - bx, dy = ay - by, dz = az - bz;
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

struct MaxU32 {
    __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};

// ---------------------------------------------------------------------------
// Farthest point sampling.
//
// The method takes npoint sequential steps, each an argmax over the cloud of
// the distance to the samples taken so far. A step is bound by the instructions
// of its serial chain (the maximum, the winner's coordinates), issued by few
// waves, and in a workgroup by its barrier and LDS round trips:
//
//  * pv_fps_wave_kernel (small clouds): one wave holds the whole cloud, NS
//    points a lane.
//  * pv_fps_step_kernel (few samples): a workgroup, a barrier per sample.
//  * pv_fps_batch_kernel: distances only decrease, so if C holds every point
//    whose distance exceeds T, then as long as the farthest point of C is
//    farther than T it is the farthest point of the cloud, whatever the other
//    points' distances have become. Each round the workgroup collects such a C
//    (at most kFpsCand points), one wave takes samples from C in registers, up
//    to 64 of them, until its farthest is no farther than T, and then the whole
//    cloud is updated with the round's samples at once. Rooms of 8192 points
//    take 1024 samples in about 50 rounds. The points are sorted along a
//    Morton curve first, so that a wave's 64 lanes hold a compact cluster, and
//    a cluster is updated only with the samples closer to its box than the
//    farthest point of the cloud (about 10 of 128 clusters a sample; with each
//    cluster's own farthest point 8.5, which does not pay for a reduction per
//    cluster). An update that is skipped cannot change a minimum, so the
//    samples are the method's own.
//
// Ties go to the lower index: every point of C carries its index. If more
// points than C holds are equally far (a lattice), C takes the lowest indices
// among them, T being the value just below theirs.
// ---------------------------------------------------------------------------
constexpr int kFpsCand = 128;       // candidates a round can hold: two a lane
constexpr int kFpsTarget = 48;      // and aims at: one a lane
constexpr int kFpsCells = 16 * 16 * 16;

__device__ __forceinline__ float readlane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
// A distance as its bits: distances are >= 0, so their bits order as their
// values. What is not a number has bits above infinity's as an unsigned value,
// of either sign (an infinite point's own distance is one), and so replaces
// nothing. "No point" is a distance of 0 that stays one: it is never beyond a
// threshold, and where 0 is the farthest, point 0 is the lowest index.
__device__ __forceinline__ int nearer(int d, float x, float y, float z, float sx, float sy,
                                      float sz) {
    return (int)min((uint32_t)d, __float_as_uint(sqdist(x, y, z, sx, sy, sz)));
}
constexpr int kFpsNoPoint = 0;
constexpr int kFpsUnset = 0x7f800000;  // +infinity

// The largest of the wave's distances (wave-uniform).
__device__ __forceinline__ int wave_farthest(int m) {
    return (int)wave_reduce((uint32_t)m, MaxU32{});
}

template <int NS>
__global__ __launch_bounds__(64) void pv_fps_wave_kernel(const float* __restrict__ xyz, int N,
                                                         int npoint, int32_t* __restrict__ idx,
                                                         float* __restrict__ new_xyz) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const float* p = xyz + (size_t)b * N * 3;
    float x[NS], y[NS], z[NS];
    int d[NS];
#pragma unroll
    for (int k = 0; k < NS; k++) {
        const int j = lane + k * 64;
        const float* q = p + (size_t)(j < N ? j : 0) * 3;
        x[k] = q[0];
        y[k] = q[1];
        z[k] = q[2];
        d[k] = j < N ? kFpsUnset : kFpsNoPoint;
    }
    float sx = p[0], sy = p[1], sz = p[2];
    int pick = 0;  // lane l: the l-th sample of 64
    for (int s = 0;;) {
        // the samples' indices gather in the lanes and are stored 64 at a time
        if ((s & 63) == 63 || s == npoint - 1) {
            const int at = (s & ~63) + lane;
            if (at <= s) {
                idx[(size_t)b * npoint + at] = pick;
                if (new_xyz) {
                    const float* q = p + (size_t)pick * 3;
                    float* o = new_xyz + ((size_t)b * npoint + at) * 3;
                    o[0] = q[0];
                    o[1] = q[1];
                    o[2] = q[2];
                }
            }
        }
        if (++s >= npoint) break;
        // each lane's farthest point, the lowest index among equals (a strictly
        // larger distance replaces), then the wave's
        d[0] = nearer(d[0], x[0], y[0], z[0], sx, sy, sz);
        int m = d[0], mk = 0;
#pragma unroll
        for (int k = 1; k < NS; k++) {
            d[k] = nearer(d[k], x[k], y[k], z[k], sx, sy, sz);
            const bool more = d[k] > m;
            m = more ? d[k] : m;
            mk = more ? k : mk;
        }
        const int top = wave_farthest(m);
        uint64_t hold = __ballot(m == top);
        if ((hold & (hold - 1ull)) != 0ull) {  // several lanes: the lowest index
            const uint32_t low = m == top ? 0xffffffffu - (uint32_t)(lane + mk * 64) : 0u;
            const uint32_t lowest = wave_reduce(low, MaxU32{});  // in every lane
            hold = __ballot(low == lowest);
        }
        const int l = __builtin_ctzll(hold);  // not empty: top is some lane's
        const int wk = __builtin_amdgcn_readlane(mk, l);
#pragma unroll
        for (int k = 0; k < NS; k++)
            if (wk == k) {
                sx = readlane_f(x[k], l);
                sy = readlane_f(y[k], l);
                sz = readlane_f(z[k], l);
            }
        pick = lane == (s & 63) ? l + wk * 64 : pick;
    }
}

// Samples from the candidates until none is farther than T; returns how many.
// Lane n gets the n-th sample's place among the candidates.
template <int NS>
__device__ __forceinline__ int fps_take(const float4* s_c, const int* s_ci, int count, int T,
                                        int most, int lane, int& pick) {
    float x[NS], y[NS], z[NS];
    int d[NS], j[NS];
#pragma unroll
    for (int k = 0; k < NS; k++) {
        const float4 v = s_c[lane + k * 64];
        x[k] = v.x;
        y[k] = v.y;
        z[k] = v.z;
        d[k] = lane + k * 64 < count ? __float_as_int(v.w) : kFpsNoPoint;
        j[k] = s_ci[lane + k * 64];
    }
    // ~45 instructions in one dependent chain, ~390 cycles a sample
    int n = 0;
    do {
        bool second = false;
        int m = d[0];
        if constexpr (NS == 2) {
            second = d[1] > d[0];
            m = max(d[0], d[1]);
        }
        const int top = wave_farthest(m);
        if (top <= T) break;
        uint64_t hold = __ballot(m == top);
        uint64_t many = hold & (hold - 1ull);
        if constexpr (NS == 2) many |= __ballot(m == top && d[0] == d[1]);
        if (__builtin_expect(many != 0ull, 0)) {  // equal distances: the lowest index
            uint32_t low = d[0] == top ? 0xffffffffu - (uint32_t)j[0] : 0u;
            if constexpr (NS == 2)
                low = max(low, d[1] == top ? 0xffffffffu - (uint32_t)j[1] : 0u);
            const uint32_t lowest = wave_reduce(low, MaxU32{});
            hold = __ballot(low == lowest);
            if constexpr (NS == 2)
                second = d[1] == top && 0xffffffffu - (uint32_t)j[1] == lowest;
        }
        const int l = __builtin_ctzll(hold);  // not empty: top is some lane's
        float sx = readlane_f(x[0], l), sy = readlane_f(y[0], l), sz = readlane_f(z[0], l);
        int at = l;
        if constexpr (NS == 2) {
            const bool up = (__ballot(second) >> l) & 1ull;
            const float ux = readlane_f(x[1], l), uy = readlane_f(y[1], l),
                        uz = readlane_f(z[1], l);
            sx = up ? ux : sx;
            sy = up ? uy : sy;
            sz = up ? uz : sz;
            at = up ? l + 64 : l;
        }
        pick = lane == n ? at : pick;
#pragma unroll
        for (int k = 0; k < NS; k++) d[k] = nearer(d[k], x[k], y[k], z[k], sx, sy, sz);
    } while (++n < most);
    return n;
}

// One workgroup of NT threads per cloud, step by step. Thread t keeps points t,
// t + NT, ... (PPT of them) and their distance to the samples taken so far in
// registers. Each step: update those distances with the last sample and take
// the thread's farthest point (the lowest index among equals: the thread's
// points come in index order and only a strictly larger distance replaces);
// then the wave's; then the workgroup's through one LDS slot per wave. TAB
// (clouds of up to kFpsTab points): the cloud's coordinates sit in an LDS
// table, and the winner's are read from it by index; otherwise each thread also
// carries its farthest point's coordinates and the winning lane writes them to
// its slot. The slots alternate between two buffers so that one barrier per
// step suffices: step s+2 writes the buffer step s read only after every wave
// has passed the barrier of step s+1, which follows those reads.
constexpr int kFpsTab = 8192;

template <int PPT, int NT, bool TAB>
__global__ __launch_bounds__(NT) void pv_fps_step_kernel(const float* __restrict__ xyz, int N,
                                                    int npoint, int32_t* __restrict__ idx,
                                                    float* __restrict__ new_xyz) {
    constexpr int NW = NT / 64;
    __shared__ float s_d[2][NW];
    __shared__ int s_j[2][NW];
    __shared__ float s_pt[2][NW][4];
    __shared__ float s_tab[TAB ? 3 * kFpsTab : 1];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float* p = xyz + (size_t)b * N * 3;
    float px[PPT], py[PPT], pz[PPT], dmin[PPT];
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int j = tid + k * NT;
        const bool ok = j < N;
        const float* q = p + (size_t)(ok ? j : 0) * 3;
        px[k] = q[0];
        py[k] = q[1];
        pz[k] = q[2];
        dmin[k] = ok ? INFINITY : -1.f;  // -1: never the farthest
        if (TAB && ok) {  // the table is only read for TAB
            s_tab[j] = px[k];
            s_tab[kFpsTab + j] = py[k];
            s_tab[2 * kFpsTab + j] = pz[k];
        }
    }
    float lx = p[0], ly = p[1], lz = p[2];
    int32_t* out = idx + (size_t)b * npoint;
    float* oxyz = new_xyz ? new_xyz + (size_t)b * npoint * 3 : nullptr;
    if (tid == 0) {
        out[0] = 0;
        if (oxyz) {
            oxyz[0] = lx;
            oxyz[1] = ly;
            oxyz[2] = lz;
        }
    }
    if (TAB) pv_lds_barrier();
    for (int s = 1; s < npoint; s++) {
        float bestd = -1.f, bx = 0.f, by = 0.f, bz = 0.f;
        int bestj = 0;
#pragma unroll
        for (int k = 0; k < PPT; k++) {
            dmin[k] = fminf(dmin[k], sqdist(px[k], py[k], pz[k], lx, ly, lz));
            const bool better = dmin[k] > bestd;  // strict: the lower index stays
            bestd = better ? dmin[k] : bestd;
            bestj = better ? tid + k * NT : bestj;
            if constexpr (!TAB) {
                bx = better ? px[k] : bx;
                by = better ? py[k] : by;
                bz = better ? pz[k] : bz;
            }
        }
        // the wave's farthest point: a maximum over the distances' bits
        // (distances are >= 0, so their bits order as their values), offset
        // by one so that 0 means "no point" (the reduction fills lanes it
        // leaves out with 0); then the lanes holding it by ballot
        const uint32_t key = bestd >= 0.f ? __float_as_uint(bestd) + 1u : 0u;
        const uint32_t wkey = wave_reduce(key, MaxU32{});
        const uint64_t hold = __ballot(key != 0u && key == wkey);
        int wj = 0x7fffffff;
        float wd = -1.f;
        if (hold != 0ull) {
            wd = __uint_as_float(wkey - 1u);
            if ((hold & (hold - 1ull)) == 0ull) {  // one lane
                wj = __builtin_amdgcn_readlane(bestj, __ffsll((long long)hold) - 1);
            } else {  // equal distances in several lanes: the lowest index
                const uint32_t jk = (hold >> lane) & 1ull ? 0xffffffffu - (uint32_t)bestj : 0u;
                wj = (int)(0xffffffffu - wave_reduce(jk, MaxU32{}));
            }
        }
        const int buf = s & 1;
        if (lane == 0) {
            s_d[buf][w] = wd;
            s_j[buf][w] = wj;
        }
        if constexpr (!TAB) {
            if (bestj == wj && wd >= 0.f) {  // the one lane that holds it
                s_pt[buf][w][0] = bx;
                s_pt[buf][w][1] = by;
                s_pt[buf][w][2] = bz;
            }
        }
        pv_lds_barrier();
        float best = s_d[buf][0];
        int bj = s_j[buf][0], bw = 0;
#pragma unroll
        for (int i = 1; i < NW; i++) {
            const float d = s_d[buf][i];
            const int j = s_j[buf][i];
            if (d > best || (d == best && j < bj)) {
                best = d;
                bj = j;
                bw = i;
            }
        }
        if constexpr (TAB) {
            lx = s_tab[bj];
            ly = s_tab[kFpsTab + bj];
            lz = s_tab[2 * kFpsTab + bj];
        } else {
            lx = s_pt[buf][bw][0];
            ly = s_pt[buf][bw][1];
            lz = s_pt[buf][bw][2];
        }
        if (tid == 0) {
            out[s] = bj;
            if (oxyz) {
                oxyz[(size_t)s * 3] = lx;
                oxyz[(size_t)s * 3 + 1] = ly;
                oxyz[(size_t)s * 3 + 2] = lz;
            }
        }
    }
}

// Order-preserving map of a float's bits to u32 (any finite value maps above 0).
__device__ __forceinline__ uint32_t f32_key(float v) {
    const uint32_t u = __float_as_uint(v);
    return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ __forceinline__ float f32_unkey(uint32_t k) {
    return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xffffffffu));
}
// Bits 0..3 of v spread to every third bit.
__device__ __forceinline__ uint32_t spread4(uint32_t v) {
    return (v & 1u) | ((v & 2u) << 2) | ((v & 4u) << 4) | ((v & 8u) << 6);
}

template <int PPT, int NT>
__global__ __launch_bounds__(NT) void pv_fps_batch_kernel(const float* __restrict__ xyz, int N,
                                                          int npoint, int32_t* __restrict__ idx,
                                                          float* __restrict__ new_xyz) {
    constexpr int NW = NT / 64;
    static_assert(PPT % 2 == 0 && NW <= 16 && PPT * NT <= 65536, "slot pairs, u16 indices");
    __shared__ uint32_t s_cell[kFpsCells];
    __shared__ uint16_t s_order[PPT * NT];
    __shared__ float4 s_cand[kFpsCand];
    __shared__ int s_cand_i[kFpsCand];
    __shared__ float4 s_pick[64];
    __shared__ float4 s_box[PPT * NW][2];  // a cluster's lower, upper corner
    __shared__ uint32_t s_red[NW][6];
    __shared__ int s_far[NW];
    __shared__ int s_count[3];
    __shared__ int s_npick;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float* p = xyz + (size_t)b * N * 3;

    // --- the cloud's box, then its points in Morton order of a 16^3 grid over
    // it (a counting sort; the order inside a cell does not matter)
    if (tid < 3) s_count[tid] = 0;
    float px[PPT], py[PPT], pz[PPT];
    for (int c = tid; c < kFpsCells; c += NT) s_cell[c] = 0u;
    uint32_t box[6] = {0u, 0u, 0u, 0u, 0u, 0u};  // keys of max(-x), .., max(x), ..
#pragma unroll 4
    for (int k = 0; k < PPT; k++) {
        const int j = tid + k * NT;
        const float* q = p + (size_t)(j < N ? j : 0) * 3;
        const float x = q[0], y = q[1], z = q[2];
        box[0] = max(box[0], f32_key(-x));
        box[1] = max(box[1], f32_key(-y));
        box[2] = max(box[2], f32_key(-z));
        box[3] = max(box[3], f32_key(x));
        box[4] = max(box[4], f32_key(y));
        box[5] = max(box[5], f32_key(z));
    }
#pragma unroll
    for (int a = 0; a < 6; a++) {
        const uint32_t m = wave_reduce(box[a], MaxU32{});
        if (lane == 0) s_red[w][a] = m;
    }
    pv_lds_barrier();
#pragma unroll
    for (int a = 0; a < 6; a++) {
        uint32_t m = s_red[0][a];
        for (int i = 1; i < NW; i++) m = max(m, s_red[i][a]);
        box[a] = m;
    }
    const float lox = -f32_unkey(box[0]), loy = -f32_unkey(box[1]), loz = -f32_unkey(box[2]);
    const float ext = fmaxf(fmaxf(f32_unkey(box[3]) - lox, f32_unkey(box[4]) - loy),
                            f32_unkey(box[5]) - loz);
    const float scale = 16.f / ext;
#pragma unroll
    for (int k = 0; k < PPT; k++) {  // read again rather than held: registers
        const int j = tid + k * NT;
        const float* q = p + (size_t)(j < N ? j : 0) * 3;
        px[k] = q[0];
        py[k] = q[1];
        pz[k] = q[2];
    }
    uint32_t place[PPT];  // cell << 16 | rank within it
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        // clamped, so that any coordinate falls in some cell (NaN: cell 0)
        const float fx = fminf(fmaxf((px[k] - lox) * scale, 0.f), 15.f);
        const float fy = fminf(fmaxf((py[k] - loy) * scale, 0.f), 15.f);
        const float fz = fminf(fmaxf((pz[k] - loz) * scale, 0.f), 15.f);
        const uint32_t c = spread4((uint32_t)fx) | (spread4((uint32_t)fy) << 1) |
                           (spread4((uint32_t)fz) << 2);
        place[k] = c << 16;
        if (tid + k * NT < N) place[k] += atomicAdd(&s_cell[c], 1u);
    }
    pv_lds_barrier();
    {
        constexpr int E = kFpsCells / NT;
        uint32_t v[E], sum = 0u;
#pragma unroll
        for (int e = 0; e < E; e++) {
            v[e] = s_cell[tid * E + e];
            sum += v[e];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = (uint32_t)__shfl_up((int)incl, off, 64);
            if (lane >= off) incl += o;
        }
        if (lane == 63) s_red[w][0] = incl;  // every wave has read its box
        pv_lds_barrier();
        uint32_t base = incl - sum;
        for (int i = 0; i < w; i++) base += s_red[i][0];
#pragma unroll
        for (int e = 0; e < E; e++) {
            s_cell[tid * E + e] = base;
            base += v[e];
        }
    }
    pv_lds_barrier();
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int j = tid + k * NT;
        if (j < N) s_order[s_cell[place[k] >> 16] + (place[k] & 0xffffu)] = (uint16_t)j;
    }
    pv_lds_barrier();

    // --- slot k of wave w: the 64 points of cluster k * NW + w (neighbouring
    // clusters in different waves)
    int d[PPT];
    const float fx0 = p[0], fy0 = p[1], fz0 = p[2];
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int pos = (k * NW + w) * 64 + lane;
        const float* q = p + (size_t)(pos < N ? s_order[pos] : 0) * 3;
        px[k] = q[0];
        py[k] = q[1];
        pz[k] = q[2];
    }
    int wfar = 0;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int c0 = (k * NW + w) * 64;  // wave-uniform
        d[k] = kFpsNoPoint;
        if (c0 >= N) continue;
        const bool ok = c0 + lane < N;
        if (ok) d[k] = nearer(kFpsUnset, px[k], py[k], pz[k], fx0, fy0, fz0);
        wfar = max(wfar, d[k]);
        auto least = [&](float v) {
            return -f32_unkey(wave_reduce(ok ? f32_key(-v) : 0u, MaxU32{}));
        };
        auto most = [&](float v) {
            return f32_unkey(wave_reduce(ok ? f32_key(v) : 0u, MaxU32{}));
        };
        const float4 lo = make_float4(least(px[k]), least(py[k]), least(pz[k]), 0.f);
        const float4 hi = make_float4(most(px[k]), most(py[k]), most(pz[k]), 0.f);
        if (lane == 0) {
            s_box[k * NW + w][0] = lo;
            s_box[k * NW + w][1] = hi;
        }
    }
    if (tid == 0) {
        idx[(size_t)b * npoint] = 0;
        if (new_xyz) {
            float* o = new_xyz + (size_t)b * npoint * 3;
            o[0] = fx0;
            o[1] = fy0;
            o[2] = fz0;
        }
    }

    // --- rounds
    float below = 0.1f;  // T = (1 - below) * the largest distance
    int turn = 0;        // s_count[turn] counts the current candidates
    for (int s = 1; s < npoint;) {
        wfar = wave_farthest(wfar);
        if (lane == 0) s_far[w] = wfar;
        pv_lds_barrier();
        int top = s_far[0];
#pragma unroll
        for (int i = 1; i < NW; i++) top = max(top, s_far[i]);
        top = __builtin_amdgcn_readfirstlane(top);
        if (top == 0) {  // every point coincides with a sample: the lowest index
            for (int t = s + tid; t < npoint; t += NT) {
                const size_t o = (size_t)b * npoint + t;
                idx[o] = 0;
                if (new_xyz) {
                    new_xyz[o * 3] = fx0;
                    new_xyz[o * 3 + 1] = fy0;
                    new_xyz[o * 3 + 2] = fz0;
                }
            }
            return;  // the whole workgroup: `top` is uniform
        }
        const float ftop = __int_as_float(top);
        // T >= 0, at most the value just below the largest distance
        int T = min(__float_as_int(ftop * (1.f - below)), top - 1);
        bool tie = T == top - 1;
        int jmax = N, jlo = -1, jhi = N - 1, count = 0;
        // Collect; with too many candidates raise T, and once T is just below
        // the largest distance halve the range of indices instead. Both end:
        // the first within 12 turns, and the count grows by at most one with
        // each index.
        for (int t = 0; t < 40; t++) {
            uint64_t in[PPT];
            int n = 0;
#pragma unroll
            for (int k = 0; k < PPT; k++) {
                bool c = d[k] > T;  // no point: 0
                if (jmax < N) c = c && s_order[(k * NW + w) * 64 + lane] <= jmax;
                in[k] = __ballot(c);
                n += __popcll(in[k]);
            }
            if (n > 0) {
                int base = 0;
                if (lane == 0) base = atomicAdd(&s_count[turn], n);
                base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
                for (int k = 0; k < PPT; k++) {
                    if (in[k] == 0ull) continue;
                    const int at = base + __popcll(in[k] & ((1ull << lane) - 1ull));
                    if (((in[k] >> lane) & 1ull) && at < kFpsCand) {
                        s_cand[at] = make_float4(px[k], py[k], pz[k], __int_as_float(d[k]));
                        s_cand_i[at] = s_order[(k * NW + w) * 64 + lane];
                    }
                    base += __popcll(in[k]);
                }
            }
            pv_lds_barrier();
            count = __builtin_amdgcn_readfirstlane(s_count[turn]);
            turn = turn == 2 ? 0 : turn + 1;
            // the count after the next: every wave read it before this barrier
            if (tid == 0) s_count[turn == 2 ? 0 : turn + 1] = 0;
            if (count > 0 && count <= kFpsCand) break;
            if (!tie) {
                below *= 0.35f;
                T = min(__float_as_int(ftop * (1.f - below)), top - 1);
                if (t >= 10) T = top - 1;
                tie = T == top - 1;
            } else {
                if (jmax == N) jmax = N - 1;
                if (count == 0) jlo = jmax;
                else jhi = jmax;
                jmax = (jlo + jhi) >> 1;
            }
        }
        count = min(count, kFpsCand);
        if (w == 0) {
            int pick = 0;
            const int most = min(64, npoint - s);
            const int n = count <= 64 ? fps_take<1>(s_cand, s_cand_i, count, T, most, lane, pick)
                                      : fps_take<2>(s_cand, s_cand_i, count, T, most, lane, pick);
            float4 v = s_cand[pick];
            v.w = __int_as_float(s_cand_i[pick]);
            s_pick[lane] = v;
            if (lane == 0) s_npick = n;
        }
        // aim at kFpsTarget candidates in the next round
        const float ratio = sqrtf((float)kFpsTarget / (float)max(count, 1));
        below = fminf(0.9f, fmaxf(1e-6f, below * fminf(2.f, fmaxf(0.5f, ratio))));
        pv_lds_barrier();
        const int np = __builtin_amdgcn_readfirstlane(s_npick);
        if (np == 0) return;  // cannot be: a candidate is farther than T
        if (w == NW - 1 && lane < np) {
            const float4 v = s_pick[lane];
            const size_t o = (size_t)b * npoint + s + lane;
            idx[o] = __float_as_int(v.w);
            if (new_xyz) {
                new_xyz[o * 3] = v.x;
                new_xyz[o * 3 + 1] = v.y;
                new_xyz[o * 3 + 2] = v.z;
            }
        }
        s += np;
        if (s >= npoint) return;
        // Update each cluster with the samples that can reach it: 32 samples
        // against two clusters at once, one in each half of the wave. The
        // distance to the box and the points' own distances are rounded apart:
        // a margin of 2e-5 (and an absolute one, for squares that underflow)
        // keeps every sample that could change a minimum, and so does an
        // overflow or what is not a number.
        const float reach = (ftop + 1e-36f) * (1.f + 2e-5f);
        for (int p0 = 0; p0 < np; p0 += 32) {
            const float4 pk = s_pick[p0 + (lane & 31)];
            const bool some = p0 + (lane & 31) < np;
#pragma unroll
            for (int k = 0; k < PPT / 2; k++) {
                // read the box here, not ahead of the loops (registers)
                asm volatile("" ::: "memory");
                const int c = (lane < 32 ? k : k + PPT / 2) * NW + w;
                const float4 lo = s_box[c][0], hi = s_box[c][1];
                const float ex = fmaxf(fmaxf(lo.x - pk.x, pk.x - hi.x), 0.f);
                const float ey = fmaxf(fmaxf(lo.y - pk.y, pk.y - hi.y), 0.f);
                const float ez = fmaxf(fmaxf(lo.z - pk.z, pk.z - hi.z), 0.f);
                const float e2 = ex * ex + ey * ey + ez * ez;
                const uint64_t near = __ballot(some && !(e2 >= reach && e2 <= 3e38f));
                auto pass = [&](int kk, uint32_t m) {
                    while (m != 0u) {
                        const int l = __ffs((int)m) - 1;
                        m &= m - 1u;
                        d[kk] = nearer(d[kk], px[kk], py[kk], pz[kk], readlane_f(pk.x, l),
                                       readlane_f(pk.y, l), readlane_f(pk.z, l));
                    }
                };
                pass(k, (uint32_t)near);
                pass(k + PPT / 2, (uint32_t)(near >> 32));
            }
        }
        wfar = 0;
#pragma unroll
        for (int k = 0; k < PPT; k++) wfar = max(wfar, d[k]);
    }
}

// ---------------------------------------------------------------------------
// Ball query, one wave per centre: the wave scans the cloud in index order,
// kU chunks of 64 points per round (their loads in flight together), and
// keeps the first nsample points inside the ball in that order (ballot, then
// each lane's rank among the lanes below it). All control is wave-uniform.
// ---------------------------------------------------------------------------
constexpr int kBallWaves = 4;
constexpr int kBallU = 4;

__global__ __launch_bounds__(kBallWaves * 64) void pv_ball_query_kernel(
    const float* __restrict__ xyz, int N, const float* __restrict__ centers, int M,
    int total, float r2, int nsample, int32_t* __restrict__ idx) {
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * kBallWaves + (threadIdx.x >> 6);
    if (q >= total) return;  // the whole wave
    const int b = q / M;
    const float* p = xyz + (size_t)b * N * 3;
    const float cx = centers[(size_t)q * 3], cy = centers[(size_t)q * 3 + 1],
                cz = centers[(size_t)q * 3 + 2];
    int32_t* out = idx + (size_t)q * nsample;
    const uint64_t below = (1ull << lane) - 1ull;
    int cnt = 0, first = -1;
    for (int base = 0; base < N && cnt < nsample; base += 64 * kBallU) {
        float x[kBallU], y[kBallU], z[kBallU];
#pragma unroll
        for (int u = 0; u < kBallU; u++) {
            const int j = min(base + u * 64 + lane, N - 1);
            x[u] = p[(size_t)j * 3];
            y[u] = p[(size_t)j * 3 + 1];
            z[u] = p[(size_t)j * 3 + 2];
        }
#pragma unroll
        for (int u = 0; u < kBallU; u++) {
            const int j = base + u * 64 + lane;
            const bool in = j < N && sqdist(x[u], y[u], z[u], cx, cy, cz) < r2;
            const uint64_t m = __ballot(in);
            if (m != 0ull) {
                const int pos = cnt + __popcll(m & below);
                if (in && pos < nsample) out[pos] = j;
                if (first < 0) first = base + u * 64 + __ffsll((long long)m) - 1;
                cnt += __popcll(m);
            }
        }
    }
    const int fill = first >= 0 ? first : 0;
    for (int k = min(cnt, nsample) + lane; k < nsample; k += 64) out[k] = fill;
}

// V values of a row as fp32, and back.
template <int V>
__device__ __forceinline__ void row_load(const float* p, float (&v)[V]) {
    if constexpr (V == 8) {
        const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
        v[0] = *p;
    }
}
template <int V>
__device__ __forceinline__ void row_load(const uint16_t* p, float (&v)[V]) {
    if constexpr (V == 8) {
        const uint4 a = *(const uint4*)p;
        const uint32_t u[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            v[2 * i] = __uint_as_float(u[i] << 16);
            v[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
        }
    } else {
        v[0] = pv_bf16_to_f32(*p);
    }
}
template <int V>
__device__ __forceinline__ void row_store(float* p, const float (&v)[V]) {
    if constexpr (V == 8) {
        *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
        *(float4*)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else {
        *p = v[0];
    }
}
template <int V>
__device__ __forceinline__ void row_store(uint16_t* p, const float (&v)[V]) {
    if constexpr (V == 8)
        *(uint4*)p = make_uint4(pv_pack_bf16x2(v[0], v[1]), pv_pack_bf16x2(v[2], v[3]),
                                pv_pack_bf16x2(v[4], v[5]), pv_pack_bf16x2(v[6], v[7]));
    else
        *p = pv_f32_to_bf16(v[0]);
}
// Rows of ld elements of `bytes` each start at 16-byte boundaries and hold
// whole groups of eight channels.
bool rows_vec8(const void* p, int ld, int C, bool bf16) {
    return C % 8 == 0 && pv_aligned16(p) && ((size_t)ld * (bf16 ? 2 : 4)) % 16 == 0;
}

// ---------------------------------------------------------------------------
// Grouping: row (q, k) of the output holds the neighbour j = idx[q][k]'s
// coordinates relative to centre q, then its C features. V output elements
// per thread, elements fastest. V = 8 (output rows at 16-byte boundaries):
// one index and one store for eight elements, read one by one (a row's
// features start three elements in, off any boundary): 131072 rows of 3 + 32
// bf16 16.9 us one by one, 11.3 with 8. A row's last piece is written element
// by element: what follows the row is not the kernel's.
// ---------------------------------------------------------------------------
template <typename FT, typename OT, int V>
__global__ __launch_bounds__(256) void pv_group_kernel(
    const float* __restrict__ xyz, const FT* __restrict__ feats, int feat_ld, int N, int C,
    const float* __restrict__ centers, int M, const int32_t* __restrict__ idx, int nsample,
    OT* __restrict__ out, int out_ld, size_t total) {
    const int W = 3 + C, G = (W + V - 1) / V;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total;
         e += (size_t)gridDim.x * 256) {
        const size_t row = e / G;
        const int c0 = (int)(e - row * G) * V;
        const size_t q = row / nsample;
        const size_t p = (size_t)(int)(q / M) * N + min(max(idx[row], 0), N - 1);
        float v[V];
#pragma unroll
        for (int t = 0; t < V; t++) {
            const int c = c0 + t;
            v[t] = 0.f;
            if (c < 3) {
                v[t] = xyz[p * 3 + c] - centers[q * 3 + c];
            } else if (c < W) {
                if constexpr (sizeof(FT) == 2) v[t] = pv_bf16_to_f32(feats[p * feat_ld + c - 3]);
                else v[t] = feats[p * feat_ld + c - 3];
            }
        }
        OT* o = out + row * out_ld + c0;
        if (c0 + V <= W) {
            row_store<V>(o, v);
        } else {
#pragma unroll
            for (int t = 0; t < V; t++)
                if (c0 + t < W) {
                    if constexpr (sizeof(OT) == 2) o[t] = pv_f32_to_bf16(v[t]);
                    else o[t] = v[t];
                }
        }
    }
}

// ---------------------------------------------------------------------------
// Three nearest neighbours: kNnLanes lanes per unknown point, each scanning
// every kNnLanes-th known point (the cloud's known points pass through LDS
// in tiles) and keeping its three nearest in (distance, index) order: a
// strictly smaller distance moves ahead, and the lane's candidates come in
// index order, so among equals the lower index stays in front. Bound by the
// instructions per candidate: one 16-byte LDS read, six for the distance, and
// eleven without a branch to keep the three (some lane of the wave takes nearly
// every candidate of the first hundreds, so a branch around the insertion was
// taken almost always: 35 instructions). 4 x 8192 points, 1024 known: 43 ->
// 23 us. The lanes' lists are then merged pairwise by shuffles in the same
// (distance, index) order. Then the normalised inverse-distance weights, in
// fp32.
// ---------------------------------------------------------------------------
constexpr int kNnThreads = 256;
constexpr int kNnLanes = 4;
constexpr int kNnPoints = kNnThreads / kNnLanes;  // unknown points per workgroup
constexpr int kNnTile = 1024;

struct Near3 {
    float d[3];
    int i[3];
};
// (d, i) lexicographic order
__device__ __forceinline__ bool nn_less(float da, int ia, float db, int ib) {
    return da < db || (da == db && ia < ib);
}
__device__ __forceinline__ void nn_insert(Near3& n, float d, int i) {
    if (nn_less(d, i, n.d[2], n.i[2])) {
        if (nn_less(d, i, n.d[1], n.i[1])) {
            n.d[2] = n.d[1];
            n.i[2] = n.i[1];
            if (nn_less(d, i, n.d[0], n.i[0])) {
                n.d[1] = n.d[0];
                n.i[1] = n.i[0];
                n.d[0] = d;
                n.i[0] = i;
            } else {
                n.d[1] = d;
                n.i[1] = i;
            }
        } else {
            n.d[2] = d;
            n.i[2] = i;
        }
    }
}

__global__ __launch_bounds__(kNnThreads) void pv_three_nn_kernel(
    const float* __restrict__ unknown, int n, const float* __restrict__ known, int m,
    int32_t* __restrict__ idx, float* __restrict__ weight) {
    __shared__ float4 s_k[kNnTile];
    const int b = blockIdx.y;
    const int q = threadIdx.x % kNnLanes;  // this lane's share of the candidates
    const int i = blockIdx.x * kNnPoints + threadIdx.x / kNnLanes;
    const bool active = i < n;
    const float* u = unknown + ((size_t)b * n + (active ? i : 0)) * 3;
    const float ux = u[0], uy = u[1], uz = u[2];
    const float* kp = known + (size_t)b * m * 3;
    Near3 nn{{INFINITY, INFINITY, INFINITY}, {0x7fffffff, 0x7fffffff, 0x7fffffff}};
    for (int t0 = 0; t0 < m; t0 += kNnTile) {
        const int cnt = min(kNnTile, m - t0);
        pv_lds_barrier();  // the previous tile's reads are done
        for (int e = threadIdx.x; e < cnt; e += kNnThreads) {
            const float* k = kp + (size_t)(t0 + e) * 3;
            s_k[e] = make_float4(k[0], k[1], k[2], 0.f);
        }
        pv_lds_barrier();
#pragma unroll 4
        for (int j = q; j < cnt; j += kNnLanes) {
            const float4 k = s_k[j];
            const float d = sqdist(k.x, k.y, k.z, ux, uy, uz);
            const bool c0 = d < nn.d[0], c1 = d < nn.d[1], c2 = d < nn.d[2];
            const int jj = t0 + j;
            nn.i[2] = c1 ? nn.i[1] : (c2 ? jj : nn.i[2]);
            nn.i[1] = c0 ? nn.i[0] : (c1 ? jj : nn.i[1]);
            nn.i[0] = c0 ? jj : nn.i[0];
            nn.d[2] = c1 ? nn.d[1] : (c2 ? d : nn.d[2]);
            nn.d[1] = c0 ? nn.d[0] : (c1 ? d : nn.d[1]);
            nn.d[0] = c0 ? d : nn.d[0];
        }
    }
    // merge with the other lanes of this point (xor 1, then xor 2)
#pragma unroll
    for (int off = 1; off < kNnLanes; off <<= 1) {
        float od[3];
        int oi[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            od[k] = __shfl_xor(nn.d[k], off, 64);
            oi[k] = __shfl_xor(nn.i[k], off, 64);
        }
#pragma unroll
        for (int k = 0; k < 3; k++) nn_insert(nn, od[k], oi[k]);
    }
    if (!active || q != 0) return;
    const float a0 = 1.f / (sqrtf(nn.d[0]) + 1e-8f), a1 = 1.f / (sqrtf(nn.d[1]) + 1e-8f),
                a2 = 1.f / (sqrtf(nn.d[2]) + 1e-8f);
    const float sum = (a0 + a1) + a2;
    const size_t o = ((size_t)b * n + i) * 3;
    idx[o] = nn.i[0];
    idx[o + 1] = nn.i[1];
    idx[o + 2] = nn.i[2];
    weight[o] = a0 / sum;
    weight[o + 1] = a1 / sum;
    weight[o + 2] = a2 / sum;
}

// ---------------------------------------------------------------------------
// Inverse-distance interpolation: out[b][i][c] = sum_k w[b][i][k] *
// feats[b][idx[b][i][k]][c], V consecutive channels per thread, channels
// fastest. V = 8 where C, the row strides and the alignments allow 16-byte
// loads (4 x 8192 points of 128 channels: 16.6 us one by one, 6.0 with 8) and
// that leaves threads enough.
// ---------------------------------------------------------------------------
template <typename FT, typename OT, int V>
__global__ __launch_bounds__(256) void pv_three_interpolate_kernel(
    const FT* __restrict__ feats, int feat_ld, int m, int C, const int32_t* __restrict__ idx,
    const float* __restrict__ weight, int n, OT* __restrict__ out, int out_ld, size_t total) {
    const int G = C / V;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total;
         e += (size_t)gridDim.x * 256) {
        const size_t row = e / G;  // (b, i)
        const int c = (int)(e - row * G) * V;
        const int b = (int)(row / n);
        float acc[V];
#pragma unroll
        for (int t = 0; t < V; t++) acc[t] = 0.f;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int j = min(max(idx[row * 3 + k], 0), m - 1);
            float f[V];
            row_load<V>(feats + ((size_t)b * m + j) * feat_ld + c, f);
            const float w = weight[row * 3 + k];
#pragma unroll
            for (int t = 0; t < V; t++) acc[t] += w * f[t];
        }
        row_store<V>(out + row * out_ld + c, acc);
    }
}

// ---------------------------------------------------------------------------
// Maximum over each group's S rows (a centre's neighbours after the shared
// MLP): out[g][c] = max_k x[g*S + k][c]. V consecutive channels per thread,
// channels fastest; exact, so the order of the comparisons does not matter.
// Eight rows are in flight a thread (4096 groups of 32 x 64 bf16: 6.2 us one
// row after the other, 3.2 so). V = 8 where that leaves threads enough.
// ---------------------------------------------------------------------------
template <typename XT, typename OT, int V>
__global__ __launch_bounds__(256) void pv_group_max_kernel(const XT* __restrict__ x, int x_ld,
                                                           int S, int C, OT* __restrict__ out,
                                                           int out_ld, size_t total) {
    const int G = C / V;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total;
         e += (size_t)gridDim.x * 256) {
        const size_t g = e / G;
        const int c = (int)(e - g * G) * V;
        const XT* r = x + g * S * (size_t)x_ld + c;
        float m[V];
#pragma unroll
        for (int t = 0; t < V; t++) m[t] = -INFINITY;
#pragma unroll 8
        for (int k = 0; k < S; k++) {
            float v[V];
            row_load<V>(r + (size_t)k * x_ld, v);
#pragma unroll
            for (int t = 0; t < V; t++) m[t] = fmaxf(m[t], v[t]);
        }
        row_store<V>(out + g * out_ld + c, m);
    }
}

unsigned grid_for(size_t total) {
    const size_t blocks = (total + 255) / 256;
    return (unsigned)(blocks < 65536 ? blocks : 65536);
}

}  // namespace

// N lies in the upper half of the doubling that holds it, up to 8192.
static bool fps_upper_half(int N) {
    int top = 1024;
    while (top < N) top *= 2;
    return top <= 8192 && N > top / 4 * 3;
}

pvconv_status pv_launch_fps(const float* xyz, int B, int N, int npoint, int32_t* idx,
                            float* new_xyz, hipStream_t s) {
    if (B == 0) return PVCONV_OK;
#define PV_FPS(NT, ...)                                                                  \
    hipLaunchKernelGGL((__VA_ARGS__), dim3(B), dim3(NT), 0, s, xyz, N, npoint, idx, new_xyz)
    if (N > kPvFpsMaxN) return PVCONV_ENOTSUP;
    if (N <= 64) PV_FPS(64, pv_fps_wave_kernel<1>);
    else if (N <= 128) PV_FPS(64, pv_fps_wave_kernel<2>);
    else if (N <= 256) PV_FPS(64, pv_fps_wave_kernel<4>);
    else if (N <= 512) PV_FPS(64, pv_fps_wave_kernel<8>);
    // The rounds cost a sort (~10 us) and yield one to three samples each at
    // first: up to 64 samples the plain steps are as fast or faster (us, four
    // clouds: 8192 -> 32 points 39 against 68, -> 64 points 72 against 84,
    // -> 1024 points 1080 against 365). A step costs what the cloud's size
    // rounded up to a power of two does, the rounds grow with the cloud: in the
    // upper half of each doubling up to 8192 points the steps hold to 72
    // samples (us, steps and rounds, four to 64 clouds: 1024 -> 65 38 and 41 to
    // 46, -> 80 46 and 43 to 52; 8192 -> 65 74 and 80 to 91, -> 80 90 and 84 to
    // 99; but 1025 -> 65 43 and 38, 4097 -> 80 88 and 79). Clouds of few
    // distinct points (one in eight) would cross at 130.
    else if (npoint <= (fps_upper_half(N) ? 72 : 64)) {
        if (N <= 1024) PV_FPS(256, pv_fps_step_kernel<4, 256, true>);
        else if (N <= 2048) PV_FPS(256, pv_fps_step_kernel<8, 256, true>);
        else if (N <= 4096) PV_FPS(256, pv_fps_step_kernel<16, 256, true>);
        else if (N <= kFpsTab) PV_FPS(256, pv_fps_step_kernel<32, 256, true>);
        else PV_FPS(1024, pv_fps_step_kernel<16, 1024, false>);
    }
    else if (N <= 1024) PV_FPS(256, pv_fps_batch_kernel<4, 256>);
    else if (N <= 2048) PV_FPS(512, pv_fps_batch_kernel<4, 512>);
    else if (N <= 4096) PV_FPS(1024, pv_fps_batch_kernel<4, 1024>);
    else if (N <= 8192) PV_FPS(1024, pv_fps_batch_kernel<8, 1024>);
    else PV_FPS(1024, pv_fps_batch_kernel<16, 1024>);
#undef PV_FPS
    return pv_launch_status();
}

pvconv_status pv_launch_ball_query(const float* xyz, int B, int N, const float* centers, int M,
                                   float radius, int nsample, int32_t* idx, hipStream_t s) {
    const int total = B * M;
    if (total == 0) return PVCONV_OK;
    const float r2 = radius * radius;
    hipLaunchKernelGGL(pv_ball_query_kernel, dim3((total + kBallWaves - 1) / kBallWaves),
                       dim3(kBallWaves * 64), 0, s, xyz, N, centers, M, total, r2, nsample, idx);
    return pv_launch_status();
}

pvconv_status pv_launch_group(const float* xyz, const void* feats, bool feat_bf16, int feat_ld,
                              int B, int N, int C, const float* centers, int M,
                              const int32_t* idx, int nsample, void* out, bool out_bf16,
                              int out_ld, hipStream_t s) {
    if ((size_t)B * M * nsample == 0) return PVCONV_OK;
    // Eight elements a thread from 24 channels on (narrower rows are mostly their
    // ragged last piece) and where that leaves threads enough (us, one by one
    // and by eight, bf16: 131072 rows of 3 + 5 5.2 and 5.8, + 16 10.0 and 10.1,
    // + 20 11.4 and 12.6, + 24 13.3 and 11.9, + 64 31 and 14.5; 512 rows of + 64
    // 2.6 and 3.4; 8192 rows of + 32 3.2 and 3.6, + 64 4.0 and 3.7; fp32 8192
    // rows of + 64 3.9 and 4.1, 32768 of + 24 5.2 and 5.1).
    const size_t values = (size_t)B * M * nsample * C;
    const bool vec = pv_aligned16(out) && ((size_t)out_ld * (out_bf16 ? 2 : 4)) % 16 == 0 &&
                     C >= 24 && values >= (out_bf16 ? 2u << 18 : 3u << 18);
    const size_t total = (size_t)B * M * nsample * (vec ? (3 + C + 7) / 8 : 3 + C);
#define PV_GROUP(FT, OT, V)                                                                  \
    hipLaunchKernelGGL((pv_group_kernel<FT, OT, V>), dim3(grid_for(total)), dim3(256), 0, s,    \
                       xyz, (const FT*)feats, feat_ld, N, C, centers, M, idx, nsample, (OT*)out, \
                       out_ld, total)
#define PV_GROUP_V(FT, OT)                                                                   \
    do {                                                                                     \
        if (vec) PV_GROUP(FT, OT, 8); else PV_GROUP(FT, OT, 1);                              \
    } while (0)
    if (feat_bf16 && out_bf16) PV_GROUP_V(uint16_t, uint16_t);
    else if (feat_bf16) PV_GROUP_V(uint16_t, float);
    else if (out_bf16) PV_GROUP_V(float, uint16_t);
    else PV_GROUP_V(float, float);
#undef PV_GROUP_V
#undef PV_GROUP
    return pv_launch_status();
}

pvconv_status pv_launch_three_nn(const float* unknown, int B, int n, const float* known, int m,
                                 int32_t* idx, float* weight, hipStream_t s) {
    if (B == 0 || n == 0) return PVCONV_OK;
    hipLaunchKernelGGL(pv_three_nn_kernel, dim3((n + kNnPoints - 1) / kNnPoints, B),
                       dim3(kNnThreads), 0, s, unknown, n, known, m, idx, weight);
    return pv_launch_status();
}

pvconv_status pv_launch_three_interpolate(const void* feats, bool feat_bf16, int feat_ld, int B,
                                          int m, int C, const int32_t* idx, const float* weight,
                                          int n, void* out, bool out_bf16, int out_ld,
                                          hipStream_t s) {
    if ((size_t)B * n * C == 0) return PVCONV_OK;
    // From 250000 outputs on: by eight that is half a wave a SIMD, and with fewer
    // the wide loads do not make up for the waves (us, one by one and by eight:
    // 4 x 256 points of 64 channels 2.31 and 2.41, of 128 2.36 and 2.45, of 256
    // 2.74 and 2.56; 500 of 512 2.73 and 2.60; 4 x 8192 of 8 2.75 and 2.76).
    const bool vec = rows_vec8(feats, feat_ld, C, feat_bf16) &&
                     rows_vec8(out, out_ld, C, out_bf16) && (size_t)B * n * C >= 250000;
    const size_t total = (size_t)B * n * (vec ? C / 8 : C);
#define PV_INTERP(FT, OT, V)                                                                \
    hipLaunchKernelGGL((pv_three_interpolate_kernel<FT, OT, V>), dim3(grid_for(total)),      \
                       dim3(256), 0, s, (const FT*)feats, feat_ld, m, C, idx, weight, n,     \
                       (OT*)out, out_ld, total)
#define PV_INTERP_V(FT, OT)                                                                 \
    do {                                                                                    \
        if (vec) PV_INTERP(FT, OT, 8); else PV_INTERP(FT, OT, 1);                           \
    } while (0)
    if (feat_bf16 && out_bf16) PV_INTERP_V(uint16_t, uint16_t);
    else if (feat_bf16) PV_INTERP_V(uint16_t, float);
    else if (out_bf16) PV_INTERP_V(float, uint16_t);
    else PV_INTERP_V(float, float);
#undef PV_INTERP_V
#undef PV_INTERP
    return pv_launch_status();
}

pvconv_status pv_launch_group_max(const void* x, bool x_bf16, int x_ld, int G, int S, int C,
                                  void* out, bool out_bf16, int out_ld, hipStream_t s) {
    if ((size_t)G * C == 0) return PVCONV_OK;
    // A thread walks S rows one group of loads after the other, so the threads
    // in flight set the time: eight channels a thread pay from 2^19 outputs on
    // (us, eight and one: bf16, 32 rows of 64, 4096 groups 3.4 and 3.2, 8192
    // 4.9 and 5.0; 8 rows of 32, 32768 groups 2.8 and 3.9; 2048 rows of 1024,
    // 4 groups 156 and 44), fp32 rows of as many bytes only up to 8 of them (8
    // rows of 32, 32768 groups 4.3 and 5.3; 32 of 128, 4096 13.6 and 11.2).
    const bool vec = rows_vec8(x, x_ld, C, x_bf16) && rows_vec8(out, out_ld, C, out_bf16) &&
                     (size_t)G * C >= (1u << 19) && (x_bf16 || S <= 8);
    const size_t total = (size_t)G * (vec ? C / 8 : C);
#define PV_GMAX(XT, OT, V)                                                                  \
    hipLaunchKernelGGL((pv_group_max_kernel<XT, OT, V>), dim3(grid_for(total)), dim3(256), 0, s, \
                       (const XT*)x, x_ld, S, C, (OT*)out, out_ld, total)
#define PV_GMAX_V(XT, OT)                                                                   \
    do {                                                                                    \
        if (vec) PV_GMAX(XT, OT, 8); else PV_GMAX(XT, OT, 1);                               \
    } while (0)
    if (x_bf16 && out_bf16) PV_GMAX_V(uint16_t, uint16_t);
    else if (x_bf16) PV_GMAX_V(uint16_t, float);
    else if (out_bf16) PV_GMAX_V(float, uint16_t);
    else PV_GMAX_V(float, float);
#undef PV_GMAX_V
#undef PV_GMAX
    return pv_launch_status();
}
