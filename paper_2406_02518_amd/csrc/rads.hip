// rads.hip -- radiodensity-aware dual sampling (Sec. 3.3) on the device: the
// interface points of the CT volume at the (min + max) / 2 level (Sec. 4.1),
// i.e. the vertices marching cubes places on voxel edges, and voxel centres
// drawn in proportion to radiodensity, plus the nearest-neighbour scales the
// Gaussians start from.
#include "internal.h"

#include <math.h>

#include <algorithm>
#include <type_traits>
#include <utility>

namespace ddgs {

namespace {

constexpr int kRadsBlock = 256;
constexpr int kRadsSeg = 1024;  // voxels per segment (one wave)
constexpr int kRadsRounds = kRadsSeg / kWave;

__device__ __forceinline__ bool below(float v, float iso) { return v < iso; }

__global__ __launch_bounds__(kRadsBlock) void minmax_kernel(const float *hu, int64_t n, float2 *part)
{
    __shared__ float smin[kRadsBlock], smax[kRadsBlock];
    float mn = INFINITY, mx = -INFINITY;
    for (int64_t i = (int64_t)blockIdx.x * kRadsBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kRadsBlock) {
        const float v = hu[i];
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
    }
    smin[threadIdx.x] = mn;
    smax[threadIdx.x] = mx;
    __syncthreads();
    for (int o = kRadsBlock / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            smin[threadIdx.x] = fminf(smin[threadIdx.x], smin[threadIdx.x + o]);
            smax[threadIdx.x] = fmaxf(smax[threadIdx.x], smax[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = make_float2(smin[0], smax[0]);
}

// mm = (min, max, level = (min + max) / 2)
__global__ __launch_bounds__(kRadsBlock) void minmax_final_kernel(const float2 *part, int nb, float *mm)
{
    __shared__ float smin[kRadsBlock], smax[kRadsBlock];
    float mn = INFINITY, mx = -INFINITY;
    for (int b = threadIdx.x; b < nb; b += kRadsBlock) {
        mn = fminf(mn, part[b].x);
        mx = fmaxf(mx, part[b].y);
    }
    smin[threadIdx.x] = mn;
    smax[threadIdx.x] = mx;
    __syncthreads();
    for (int o = kRadsBlock / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            smin[threadIdx.x] = fminf(smin[threadIdx.x], smin[threadIdx.x + o]);
            smax[threadIdx.x] = fmaxf(smax[threadIdx.x], smax[threadIdx.x + o]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        mm[0] = smin[0];
        mm[1] = smax[0];
        mm[2] = (smin[0] + smax[0]) * 0.5f;
    }
}

// 16-bit radiodensity weight: floor((hu - min) / (max - min) * 65535)
__device__ __forceinline__ uint32_t weight_of(float hu, float mn, float mx)
{
    if (!(mx > mn)) return 0u;
    return (uint32_t)floorf(((hu - mn) / (mx - mn)) * 65535.0f);
}

// The volume is cut into segments of kRadsSeg consecutive voxels, one wave
// each (64 voxels a round, lane = voxel, so every load is a coalesced row).
// One pass finds a segment's level crossings (the +x, +y, +z edges leaving
// its voxel centres; three bits per voxel are kept), sums its weights and
// keeps them as 16-bit words; a scan of the segment totals places crossings
// and draws, a second launch writes the points from the kept bits, and a draw
// searches the segments and then the words of one.  The pass over the volume
// is bound by VALU issue and HBM: per voxel 4 B read, 2.4 B written (the running
// sums per voxel this replaces moved 60 B: the eight launches from the counts
// to the points of a 256^3 volume took 324 us, these three take 59).
struct RadsVoxel {
    int x, y, z;
};
__device__ __forceinline__ RadsVoxel voxel_of(const RadsVol &v, uint32_t i)
{
    const uint32_t row = i / (uint32_t)v.nx, z = row / (uint32_t)v.ny;
    return RadsVoxel{(int)(i - row * (uint32_t)v.nx), (int)(row - z * (uint32_t)v.ny), (int)z};
}

// hu / d for d in [2^-60, 2^100], 0 <= hu <= d, given r = 1 / d rounded: two
// residual steps, of which the first leaves an error below one unit in the last
// place and the second rounds correctly (Markstein's theorem), so the quotient
// is the division's; a quotient small enough for a residual to underflow
// weighs nothing either way.  Five operations for the division's eleven.
__device__ __forceinline__ float quotient(float hu, float d, float r)
{
    float q = __fmul_rn(hu, r);
    q = __fmaf_rn(__fmaf_rn(-q, d, hu), r, q);
    return __fmaf_rn(__fmaf_rn(-q, d, hu), r, q);
}

// lane LANE of (lo, hi) = the (uniform) word b
template <int LANE>
__device__ __forceinline__ void keep_word(uint32_t &lo, uint32_t &hi, uint64_t b)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((uint32_t)b), "n"(LANE));
    asm("v_writelane_b32 %0, %1, %2" : "+v"(hi) : "s"((uint32_t)(b >> 32)), "n"(LANE));
}
template <class F, int... R>
__device__ __forceinline__ void each_round(F f, std::integer_sequence<int, R...>)
{
    (f(std::integral_constant<int, R>{}), ...);
}

// edge: per segment the crossing edges of its 16 rounds of 64 voxels, one word
// per round and axis (word 3 round + axis, bit = lane).  Bound by VALU issue:
// the words are formed from compare masks in scalar registers, and segments
// whose far ends all lie in the volume (all but the last plane's) read the four
// voxels of a lane at one offset from four scalar bases, without a test
// (256^3: 88 VALU instructions a round and 43 us with a branch per far end and
// a division per voxel, 31 instructions and 28 us).
__global__ __launch_bounds__(kRadsBlock) void seg_count_kernel(RadsVol v, uint32_t n, const float *mm, int64_t nseg,
                                                               uint16_t *w16, uint64_t *edge, uint32_t *scnt,
                                                               uint64_t *swt)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t seg = (int64_t)blockIdx.x * (kRadsBlock / kWave) + threadIdx.x / kWave;
    if (seg >= nseg) return;
    const float mn = mm[0], mx = mm[1], iso = mm[2];
    const float d = mx - mn, rd = 1.0f / d;
    uint32_t cnt = 0, wt = 0;  // (at most 3 and 65535 per voxel)
    uint64_t mine = 0;         // lane 3 round + axis keeps that word
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(seg * kRadsSeg));
    const RadsVoxel c0 = voxel_of(v, first + (uint32_t)lane), step64 = voxel_of(v, kWave);
    int x = c0.x, y = c0.y;
    const uint32_t plane = (uint32_t)v.nx * (uint32_t)v.ny;
    const uint32_t step[3] = {1u, (uint32_t)v.nx, plane};
    // kWave voxels on
    auto next = [&] {
        x += step64.x;
        const int cx = x >= v.nx ? 1 : 0;
        x -= cx ? v.nx : 0;
        y += step64.y + cx;
        y -= y >= v.ny ? v.ny : 0;
    };
    // (uniform over the wave)
    if (first + (uint32_t)kRadsSeg + plane <= n && d >= 0x1p-60f && d <= 0x1p100f) {
        const float *const p = v.hu + first, *const px = p + step[0], *const py = p + step[1], *const pz = p + step[2];
        uint16_t *const pw = w16 + first;
        uint32_t lo = 0, hi = 0;
        auto round = [&](auto rc) {
            constexpr int r = decltype(rc)::value;
            const uint32_t o = (uint32_t)(r * kWave + lane);
            const float a = p[o], fx = px[o], fy = py[o], fz = pz[o];
            const uint32_t w = (uint32_t)floorf(quotient(a - mn, d, rd) * 65535.0f);
            pw[o] = (uint16_t)w;
            wt += w;
            const uint64_t ba = __builtin_amdgcn_ballot_w64(below(a, iso));
            const uint64_t b0 = (__builtin_amdgcn_ballot_w64(below(fx, iso)) ^ ba) &
                                __builtin_amdgcn_ballot_w64(x < v.nx - 1);
            const uint64_t b1 = (__builtin_amdgcn_ballot_w64(below(fy, iso)) ^ ba) &
                                __builtin_amdgcn_ballot_w64(y < v.ny - 1);
            const uint64_t b2 = __builtin_amdgcn_ballot_w64(below(fz, iso)) ^ ba;
            cnt += (uint32_t)(__popcll(b0) + __popcll(b1) + __popcll(b2));
            keep_word<3 * r>(lo, hi, b0);
            keep_word<3 * r + 1>(lo, hi, b1);
            keep_word<3 * r + 2>(lo, hi, b2);
            next();
        };
        each_round(round, std::make_integer_sequence<int, kRadsRounds>{});
        mine = ((uint64_t)hi << 32) | lo;
    } else {
#pragma unroll 1
        for (int r = 0; r < kRadsRounds; ++r) {
            const uint32_t i = first + (uint32_t)(r * kWave + lane);
            const bool ok = i < n;
            const float a = ok ? v.hu[i] : 0.0f;
            const bool in[3] = {ok && x < v.nx - 1, ok && y < v.ny - 1, i + plane < n};
            const uint32_t w = ok ? weight_of(a, mn, mx) : 0u;
            w16[i] = (uint16_t)w;  // (zero up to the segment's end)
            wt += w;
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const float far_end = in[ax] ? v.hu[i + step[ax]] : a;
                const uint64_t b = __builtin_amdgcn_ballot_w64(below(far_end, iso) != below(a, iso));
                cnt += (uint32_t)__popcll(b);
                mine = lane == 3 * r + ax ? b : mine;
            }
            next();
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wt += (uint32_t)__shfl_xor((int)wt, o, kWave);
    if (lane < 3 * kRadsRounds) edge[seg * (3 * kRadsRounds) + lane] = mine;
    if (lane == 0) {
        scnt[seg] = cnt;
        swt[seg] = wt;
    }
}

// Exclusive scans of the segment totals in place, by one block; entry nseg of
// each receives the total, and the pinned host words both.  A wave takes 16
// rounds of 64 consecutive segments (coalesced loads, all in flight together;
// one thread per 16 segments instead took 46 us for 16384 of them).
constexpr int kSegScanBlock = 1024;
__global__ __launch_bounds__(kSegScanBlock) void seg_scan_kernel(uint32_t *scnt, uint64_t *swt, int64_t nseg,
                                                                 const float *mm, RadsTotals *host)
{
    constexpr int NW = kSegScanBlock / kWave, PER = 16;
    // (64 segments weigh at most 64 x 1024 x 65535 < 2^32)
    static_assert((uint64_t)kWave * kRadsSeg * 65535u <= 0xFFFFFFFFull, "a round's weight fits 32 bits");
    __shared__ uint64_t lc[NW], lw[NW];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint64_t cc = 0, cw = 0;  // totals of the passes before
    for (int64_t b0 = 0; b0 < nseg; b0 += kSegScanBlock * PER) {
        const int64_t b = b0 + (int64_t)w * (kWave * PER) + lane;
        uint32_t xc[PER], xw[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int64_t j = b + q * kWave;
            xc[q] = j < nseg ? scnt[j] : 0u;
            xw[q] = j < nseg ? (uint32_t)swt[j] : 0u;
        }
        // inclusive scan of every round, then the rounds' totals in order
        uint32_t ic[PER], iw[PER];
        uint64_t sc = 0, sw = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            ic[q] = wave_incl_scan(xc[q]);
            iw[q] = wave_incl_scan(xw[q]);
            sc += (uint32_t)__builtin_amdgcn_readlane((int)ic[q], kWave - 1);
            sw += (uint32_t)__builtin_amdgcn_readlane((int)iw[q], kWave - 1);
        }
        if (lane == 0) {
            lc[w] = sc;
            lw[w] = sw;
        }
        __syncthreads();
        uint64_t pc = cc, pw = cw;
        for (int q = 0; q < NW; ++q) {
            if (q < w) {
                pc += lc[q];
                pw += lw[q];
            }
            cc += lc[q];
            cw += lw[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int64_t j = b + q * kWave;
            if (j < nseg) {
                scnt[j] = (uint32_t)pc + ic[q] - xc[q];
                swt[j] = pw + (iw[q] - xw[q]);
            }
            pc += (uint32_t)__builtin_amdgcn_readlane((int)ic[q], kWave - 1);
            pw += (uint32_t)__builtin_amdgcn_readlane((int)iw[q], kWave - 1);
        }
    }
    if (threadIdx.x == 0) {
        scnt[nseg] = (uint32_t)cc;
        swt[nseg] = cw;
        host->crossings = cc;
        host->weight = cw;
        host->level = mm[2];
    }
}

// the crossing points, [3][M], in edge order (voxel, then axis): the volume is
// read only where the kept words have a bit.  A wave walks its rounds one after
// another, each a chain of loads, so a segment's 16 rounds go to the four waves
// of a workgroup (256^3 volume, 126k crossings: 28 us with a wave per segment,
// 20 us; 23 us with eight waves).
__global__ __launch_bounds__(kRadsBlock) void mc_emit_kernel(RadsVol v, const float *mm, int64_t nseg,
                                                             const uint64_t *edge, const uint32_t *scnt, float *pts,
                                                             int64_t M)
{
    constexpr int PART = 3 * kRadsRounds / (kRadsBlock / kWave);  // words per wave
    static_assert(PART % 3 == 0, "whole rounds");
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t seg = blockIdx.x;
    const int w0 = (int)(threadIdx.x / kWave) * PART;
    if (seg >= nseg) return;
    uint32_t base = scnt[seg];
    if (base == scnt[seg + 1]) return;
    const float iso = mm[2];
    const uint64_t mine = lane < 3 * kRadsRounds ? edge[seg * (3 * kRadsRounds) + lane] : 0ull;
    const uint32_t step[3] = {1u, (uint32_t)v.nx, (uint32_t)v.nx * (uint32_t)v.ny};
    // the crossings of the waves before
    const uint32_t inc = wave_incl_scan(lane < w0 ? (uint32_t)__popcll(mine) : 0u);
    base += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    uint64_t left = __builtin_amdgcn_ballot_w64(mine != 0ull && lane >= w0 && lane < w0 + PART);
    while (left) {
        const int r = __builtin_ctzll(left) / 3;
        left &= ~(7ull << (3 * r));
        uint32_t m = 0u, o = base;
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, 3 * r + ax);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), 3 * r + ax);
            m |= (((lane < 32 ? lo : hi) >> (lane & 31)) & 1u) << ax;
            o += __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
            base += (uint32_t)(__popc(lo) + __popc(hi));
        }
        if (m == 0u) continue;  // (no wave-wide step below)
        const uint32_t i = (uint32_t)(seg * kRadsSeg) + (uint32_t)(r * kWave + lane);
        const RadsVoxel c = voxel_of(v, i);
        const float a = v.hu[i];
#pragma unroll
        for (int ax = 0; ax < 3; ++ax) {
            if (!((m >> ax) & 1u)) continue;
            const float t = (iso - a) / (v.hu[i + step[ax]] - a);
            const float gx = (float)c.x + (ax == 0 ? t : 0.0f);
            const float gy = (float)c.y + (ax == 1 ? t : 0.0f);
            const float gz = (float)c.z + (ax == 2 ? t : 0.0f);
            pts[o] = v.ox + gx * v.sx;
            pts[M + o] = v.oy + gy * v.sy;
            pts[2 * M + o] = v.oz + gz * v.sz;
            ++o;
        }
    }
}

__global__ __launch_bounds__(kRadsBlock) void iota_kernel(uint32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kRadsBlock + threadIdx.x;
    if (i < n) p[i] = (uint32_t)i;
}

// out[:, j] = src[:, idx[j]] for the first n1 sorted crossings
__global__ __launch_bounds__(kRadsBlock) void gather_kernel(const float *src, int64_t M, const uint32_t *idx,
                                                            int64_t n1, float *out, int64_t N)
{
    const int64_t j = (int64_t)blockIdx.x * kRadsBlock + threadIdx.x;
    if (j >= n1) return;
    const uint32_t i = idx[j];
    out[j] = src[i];
    out[N + j] = src[M + i];
    out[2 * N + j] = src[2 * M + i];
}

// The n1 smallest of M keys, ties by index, without sorting all of them: a
// stable pass by the top bits of the keys' range (radix_top_pass) leaves buckets of
// a few hundred evenly spread keys, and one workgroup per bucket orders its own and
// writes their points; the buckets behind the n1-th key are left alone.  Five
// launches instead of the fifteen of a whole sort, each of which lasted a launch's
// few microseconds (126k keys, n1 = 15000, the call alone: random keys 102 -> 39 us;
// a permutation, which the 32-bit keys' own top bits left in one bucket, 93 -> 38, by
// those bits 1033).  In a bucket of up to kPickLds keys an entry's place is the number
// of smaller ones, counted over the bucket in LDS; a longer one (keys crowded in a
// part of their range) is sorted by its workgroup with up to three stable 8-bit
// passes through memory (fourth powers of even ones 255 us, 24th powers 757).
constexpr int kPickBlock = 512, kPickLds = 1024, kPickWaves = kPickBlock / kWave;
__global__ __launch_bounds__(kPickBlock) void pick_kernel(const uint32_t *tot, const uint2 *range, uint32_t *ka,
                                                          uint32_t *va, uint32_t *kb, uint32_t *vb, int64_t n1,
                                                          const float *src, int64_t M, float *out, int64_t N)
{
    static_assert(kPickBlock == 1 << kTopBits, "one thread per bucket total");
    __shared__ __align__(16) uint32_t key[kPickLds];
    __shared__ uint32_t wh[kPickWaves][256], cur[256], wl[kPickWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    uint32_t start = 0;
    {
        const uint32_t inc = wave_incl_scan(tid < (int)blockIdx.x ? tot[tid] : 0u);
        if (lane == kWave - 1) wl[w] = inc;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPickWaves; ++q) start += wl[q];
    }
    const int len = (int)tot[blockIdx.x];
    if (len == 0 || (int64_t)start >= n1) return;  // uniform over the block
    auto put = [&](int rank, uint32_t i) {
        const int64_t o = (int64_t)start + rank;
        if (o >= n1) return;
        out[o] = src[i];
        out[N + o] = src[M + i];
        out[2 * N + o] = src[2 * M + i];
    };
    ka += start;
    va += start;
    if (len <= kPickLds) {
        uint32_t k[kPickLds / kPickBlock], v[kPickLds / kPickBlock];
#pragma unroll
        for (int q = 0; q < kPickLds / kPickBlock; ++q) {
            const int j = tid + q * kPickBlock;
            k[q] = j < len ? ka[j] : 0xFFFFFFFFu;
            v[q] = j < len ? va[j] : 0u;
            key[j] = k[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kPickLds / kPickBlock; ++q) {
            const int j = tid + q * kPickBlock;
            // the keys in front of this wave's, its own, and those behind
            const int jw = w * kWave + q * kPickBlock;
            if (jw >= len) break;
            const uint32_t x = k[q];
            int r = 0;
            for (int p = 0; p < jw; p += 4) {
                const uint4 y = *reinterpret_cast<const uint4 *>(&key[p]);
                r += (y.x <= x) + (y.y <= x) + (y.z <= x) + (y.w <= x);
            }
#pragma unroll 4
            for (int p = jw; p < jw + kWave; ++p) r += key[p] < x || (key[p] == x && p < j);
            for (int p = jw + kWave; p < len; p += 4) {
                const uint4 y = *reinterpret_cast<const uint4 *>(&key[p]);
                r += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
            }
            if (j < len) put(r, v[q]);
        }
        return;
    }
    kb += start;
    vb += start;
    const int low_bits = top_digit(range).shift;  // those that the top pass left
    for (int shift = 0; shift < low_bits; shift += 8) {
        if (tid < 256) cur[tid] = 0u;
        __syncthreads();
        for (int j = tid; j < len; j += kPickBlock) atomicAdd(&cur[(ka[j] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t c = tid < 256 ? cur[tid] : 0u, inc = wave_incl_scan(c);
        if (lane == kWave - 1) wl[w] = inc;
        __syncthreads();
        uint32_t pre = inc - c;
        for (int q = 0; q < w; ++q) pre += wl[q];
        if (tid < 256) cur[tid] = pre;
        for (int c0 = 0; c0 < len; c0 += kPickBlock) {
            for (int q = tid; q < kPickWaves * 256; q += kPickBlock) wh[q / 256][q % 256] = 0u;
            __syncthreads();
            const int j = c0 + tid;
            const bool ok = j < len;
            const uint32_t kk = ok ? ka[j] : 0u, vv = ok ? va[j] : 0u, d = (kk >> shift) & 255u;
            uint64_t peers = __ballot(ok);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bal = __ballot(bit);
                peers &= bit ? bal : ~bal;
            }
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
            if (ok && below == 0u) wh[w][d] = (uint32_t)__popcll(peers);
            __syncthreads();
            if (tid < 256) {
                uint32_t run = cur[tid];
#pragma unroll
                for (int q = 0; q < kPickWaves; ++q) {
                    const uint32_t t = wh[q][tid];
                    wh[q][tid] = run;
                    run += t;
                }
                cur[tid] = run;
            }
            __syncthreads();
            if (ok) {
                const uint32_t o = wh[w][d] + below;
                kb[o] = kk;
                vb[o] = vv;
            }
            __syncthreads();
        }
        uint32_t *t = ka;
        ka = kb;
        kb = t;
        t = va;
        va = vb;
        vb = t;
    }
    for (int j = tid; j < len; j += kPickBlock) put(j, va[j]);
}

// draw j: the first voxel whose inclusive weight sum exceeds draws[j] (the
// last voxel if none does), one wave per draw: a 64-way search of the
// segments' running sums, then the segment's words, 16 consecutive ones per
// lane.
__device__ __forceinline__ void draw_voxel(const RadsVol &v, uint32_t n, int64_t nseg, const RadsBegin &a, int64_t j)
{
    const uint64_t *const swt = a.swt;
    const uint16_t *const w16 = a.w16;
    constexpr int PER = kRadsSeg / kWave;
    static_assert(PER == 16, "two 16-byte loads per lane");
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t r = a.draws[j];
    uint32_t pick = n - 1u;
    if (r < swt[nseg]) {
        // the segment: the last one whose running sum before it is at most r
        int64_t lo = 0, len = nseg;
        while (len > 1) {
            const int64_t step = (len + kWave - 1) / kWave, p = (int64_t)lane * step;
            const uint64_t b = __builtin_amdgcn_ballot_w64(p < len && swt[lo + p] <= r);
            const int k = 63 - __builtin_clzll(b | 1ull);
            lo += k * step;
            len = len - k * step < step ? len - k * step : step;
        }
        const uint32_t rel = (uint32_t)(r - swt[lo]);
        const uint4 *q = reinterpret_cast<const uint4 *>(w16 + lo * kRadsSeg + lane * PER);
        const uint4 q0 = q[0], q1 = q[1];
        const uint32_t word[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
        uint32_t sum = 0u;
#pragma unroll
        for (int t = 0; t < 8; ++t) sum += (word[t] & 0xFFFFu) + (word[t] >> 16);
        const uint32_t incl = wave_incl_scan(sum);
        // the first lane whose words pass rel, then its first such word
        const uint64_t over = __builtin_amdgcn_ballot_w64(incl > rel);
        const int who = __builtin_ctzll(over);
        uint32_t run = incl - sum, at = 0u;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            run += word[t] & 0xFFFFu;
            at += run <= rel ? 1u : 0u;
            run += word[t] >> 16;
            at += run <= rel ? 1u : 0u;
        }
        pick = (uint32_t)(lo * kRadsSeg) + (uint32_t)(who * PER) + (uint32_t)__shfl((int)at, who, kWave);
    }
    if (lane != 0) return;
    const RadsVoxel c = voxel_of(v, pick);
    float *const out = a.out + a.first + j;
    out[0] = v.ox + (float)c.x * v.sx;
    out[a.N] = v.oy + (float)c.y * v.sy;
    out[2 * a.N] = v.oz + (float)c.z * v.sz;
}

// least and largest of share `b` of the keys (a share past the end: its last key)
__device__ __forceinline__ void key_range(const RadsBegin &a, int b)
{
    __shared__ uint2 red[kRadsBlock / kWave];
    constexpr int U = 8;  // loads in flight
    const int64_t per = (a.M + kKeyRangeBlocks - 1) / kKeyRangeBlocks;
    const int64_t b0 = min(b * per, a.M - 1), b1 = min(b0 + per, a.M);
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += U * kRadsBlock) {
        uint32_t x[U];
#pragma unroll
        for (int q = 0; q < U; ++q) x[q] = a.keys[min(i + q * kRadsBlock, b1 - 1)];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            lo = min(lo, x[q]);
            hi = max(hi, x[q]);
        }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = make_uint2(lo, hi);
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kRadsBlock / kWave; ++w) {
        lo = min(lo, red[w].x);
        hi = max(hi, red[w].y);
    }
    a.range[b] = make_uint2(lo, hi);
}

// One launch for what a sampling begins with: n_range blocks find the keys' range,
// the next n_clear_blocks clear words, and the rest draw, one wave per draw.
__global__ __launch_bounds__(kRadsBlock) void begin_kernel(RadsVol v, uint32_t n, int64_t nseg, RadsBegin a, int n_range,
                                                           int n_clear_blocks)
{
    const int b = (int)blockIdx.x - n_range;
    if (b < 0) {
        key_range(a, (int)blockIdx.x);
    } else if (b < n_clear_blocks) {
        const int64_t j = (int64_t)b * kRadsBlock + threadIdx.x;
        if (j < a.n_clear) a.clear[j] = 0u;
    } else {
        const int64_t j = (int64_t)(b - n_clear_blocks) * (kRadsBlock / kWave) + threadIdx.x / kWave;
        if (j < a.n2) draw_voxel(v, n, nseg, a, j);
    }
}


// ---------------------------------------------------- nearest neighbours
// log sqrt(mean squared distance to the 3 nearest other points), exact.  The
// three smallest of the float32 squared distances do not depend on the order
// in which the other points are visited, so the paths below give the same
// result bit for bit.
//
// Up to kKnnBrute points one workgroup per point tests them all.  Beyond, the
// points are binned in a uniform grid over the volume (about four cells per
// point, stored cell by cell), and sixteen lanes per point walk the rows of cells
// around its own, ring by ring, until no cell left can hold a nearer point;
// a point that three rings do not settle goes to a list that workgroups of
// the brute-force kernel take afterwards, so points far from all others cost
// no long serial walk.  What bounds a query is the latency of its row starts
// and points (about 30 of them), against N of them in a serial loop per lane
// before: 25000 points of a 256^3 volume 1785 -> 50 us (all seven launches).
// kKnnBrute: a workgroup per point costs N^2 / 256 lane loads; at 4096 points
// that is 65k of them, 256 waves deep on the card, and about the 25 us of the
// grid's small launches.
constexpr int kKnnBrute = 4096;
constexpr int kKnnRings = 3;
constexpr int kKnnLanes = 16;
constexpr int kKnnFarBlocks = 1024;
constexpr int64_t kKnnMaxCells = (int64_t)1 << 22;

struct Near3 {
    float d0, d1, d2;  // ascending
    __device__ __forceinline__ void insert(float d)
    {
        // (NaN distances are never nearer)
        if (d < d2) {
            const bool l1 = d < d1, l0 = d < d0;
            d2 = l1 ? d1 : d;
            d1 = l0 ? d0 : (l1 ? d : d1);
            d0 = l0 ? d : d0;
        }
    }
};

__device__ __forceinline__ float dist2(float qx, float qy, float qz, float px, float py, float pz)
{
    const float dx = qx - px, dy = qy - py, dz = qz - pz;
    return dx * dx + dy * dy + dz * dz;
}

__device__ __forceinline__ void store_scale(const Near3 &b, int64_t N, int64_t i, float *ls)
{
    const int64_t kk = N - 1 < 3 ? N - 1 : 3;
    float mean = 0.0f;
    if (kk == 3) mean = (b.d0 + b.d1 + b.d2) / 3.0f;
    else if (kk == 2) mean = (b.d0 + b.d1) * 0.5f;
    else if (kk == 1) mean = b.d0;
    const float l = 0.5f * logf(fmaxf(mean, 1e-7f));
    ls[i] = l;
    ls[N + i] = l;
    ls[2 * N + i] = l;
}

// One workgroup per point at a time: points 0 .. N - 1, or the list[0 ..
// *n_list) of them.
__global__ __launch_bounds__(kRadsBlock) void knn_brute_kernel(const float *pts, int64_t N, const uint32_t *list,
                                                               const uint32_t *n_list, float *ls)
{
    __shared__ float sd[kRadsBlock / kWave][3];
    const int64_t cnt = list ? (int64_t)*n_list : N;
    for (int64_t q = blockIdx.x; q < cnt; q += gridDim.x) {
        const int64_t i = list ? (int64_t)list[q] : q;
        const float px = pts[i], py = pts[N + i], pz = pts[2 * N + i];
        Near3 b{INFINITY, INFINITY, INFINITY};
        for (int64_t j = threadIdx.x; j < N; j += kRadsBlock) {
            const float d = dist2(pts[j], pts[N + j], pts[2 * N + j], px, py, pz);
            if (j != i) b.insert(d);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float e0 = __shfl_xor(b.d0, o, kWave), e1 = __shfl_xor(b.d1, o, kWave),
                        e2 = __shfl_xor(b.d2, o, kWave);
            b.insert(e0);
            b.insert(e1);
            b.insert(e2);
        }
        if ((threadIdx.x & (kWave - 1)) == 0) {
            const int w = threadIdx.x / kWave;
            sd[w][0] = b.d0;
            sd[w][1] = b.d1;
            sd[w][2] = b.d2;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kRadsBlock / kWave; ++w)
                for (int t = 0; t < 3; ++t) b.insert(sd[w][t]);
            store_scale(b, N, i, ls);
        }
        __syncthreads();
    }
}

// Cell of a coordinate along axis a, clamped to the grid (NaN: cell 0).
__device__ __forceinline__ int grid_cell(const KnnGrid &g, int a, float p)
{
    const float t = (p - g.x0[a]) * g.inv[a];
    return (int)fminf(fmaxf(t, 0.0f), (float)(g.n[a] - 1));
}
__device__ __forceinline__ uint32_t grid_cell3(const KnnGrid &g, float x, float y, float z)
{
    return (uint32_t)((grid_cell(g, 2, z) * g.n[1] + grid_cell(g, 1, y)) * g.n[0] + grid_cell(g, 0, x));
}

__global__ __launch_bounds__(kRadsBlock) void knn_count_kernel(KnnGrid g, const float *pts, int64_t N, uint32_t *cnt)
{
    const int64_t i = (int64_t)blockIdx.x * kRadsBlock + threadIdx.x;
    if (i >= N) return;
    const uint32_t c = grid_cell3(g, pts[i], pts[N + i], pts[2 * N + i]);
    // lanes that share the first lane's cell (points drawn many times from
    // one voxel) add their number at once: increments of one address serialise
    const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
    const uint64_t same = __builtin_amdgcn_ballot_w64(c == c0);
    if (c != c0) atomicAdd(&cnt[c], 1u);
    else if (__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u)) == 0u)
        atomicAdd(&cnt[c], (uint32_t)__popcll(same));
}

// The points cell by cell (cur: the cells' starts, advanced; the order inside
// a cell does not matter), with their index.
__global__ __launch_bounds__(kRadsBlock) void knn_place_kernel(KnnGrid g, const float *pts, int64_t N, uint32_t *cur,
                                                               float4 *out)
{
    const int64_t i = (int64_t)blockIdx.x * kRadsBlock + threadIdx.x;
    if (i >= N) return;
    const float x = pts[i], y = pts[N + i], z = pts[2 * N + i];
    const uint32_t c = grid_cell3(g, x, y, z);
    const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
    const uint64_t same = __builtin_amdgcn_ballot_w64(c == c0);
    uint32_t p;
    if (c != c0) {
        p = atomicAdd(&cur[c], 1u);
    } else {
        const uint32_t rank =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        uint32_t base = 0;
        if (rank == 0u) base = atomicAdd(&cur[c], (uint32_t)__popcll(same));
        p = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + rank;
    }
    out[p] = make_float4(x, y, z, __uint_as_float((uint32_t)i));
}

// (cur holds the cells' ends by now: cell c's points are [end(c - 1), end(c)))
// kKnnLanes lanes per point share the rows of a ring, then merge what they
// found: a lane per point walked its ~9 rows one after the other (109 us at
// 25000 points, against 27 us).
__global__ __launch_bounds__(kRadsBlock) void knn_query_kernel(KnnGrid g, const float4 *sp, int64_t N,
                                                               const uint32_t *end, float *ls, uint32_t *list,
                                                               uint32_t *n_list)
{
    const int64_t t = ((int64_t)blockIdx.x * kRadsBlock + threadIdx.x) / kKnnLanes;
    const int sub = threadIdx.x % kKnnLanes;
    if (t >= N) return;  // (whole groups)
    const float4 p = sp[t];
    const int cx = grid_cell(g, 0, p.x), cy = grid_cell(g, 1, p.y), cz = grid_cell(g, 2, p.z);
    Near3 b{INFINITY, INFINITY, INFINITY};
    auto run = [&](int z, int y, int xa, int xb) {
        xa = max(xa, 0);
        xb = min(xb, g.n[0] - 1);
        if (xa > xb) return;
        const int row = (z * g.n[1] + y) * g.n[0];
        const uint32_t e = end[row + xb];
        for (uint32_t q = row + xa > 0 ? end[row + xa - 1] : 0u; q < e; ++q) {
            const float4 o = sp[q];
            const float d = dist2(o.x, o.y, o.z, p.x, p.y, p.z);
            if ((int64_t)q != t) b.insert(d);
            if (b.d2 == 0.0f) return;  // three points at this place
        }
    };
    bool done = false;
    for (int r = 1; r <= kKnnRings && !done; ++r) {
        const int side = 2 * r + 1;
        for (int k = sub; k < side * side; k += kKnnLanes) {
            const int dz = k / side - r, dy = k % side - r, z = cz + dz, y = cy + dy;
            if (z < 0 || z >= g.n[2] || y < 0 || y >= g.n[1]) continue;
            if (r == 1 || abs(dz) == r || abs(dy) == r) {
                run(z, y, cx - r, cx + r);
            } else {
                if (cx - r >= 0) run(z, y, cx - r, cx - r);
                if (cx + r < g.n[0]) run(z, y, cx + r, cx + r);
            }
        }
        // the group's three nearest so far (the lanes' finds are disjoint,
        // so only lane 0 keeps the merged ones for the next ring)
        Near3 m = b;
#pragma unroll
        for (int o = kKnnLanes / 2; o > 0; o >>= 1) {
            const float e0 = __shfl_xor(m.d0, o, kWave), e1 = __shfl_xor(m.d1, o, kWave),
                        e2 = __shfl_xor(m.d2, o, kWave);
            m.insert(e0);
            m.insert(e1);
            m.insert(e2);
        }
        b = sub == 0 ? m : Near3{INFINITY, INFINITY, INFINITY};
        // every point left lies beyond a face of the cells walked that is
        // not the grid's own; slack covers the rounding of the cell index
        const float pc[3] = {p.x, p.y, p.z};
        const int cc[3] = {cx, cy, cz};
        float lb = INFINITY;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (cc[a] - r > 0) lb = fminf(lb, pc[a] - (g.x0[a] + (float)(cc[a] - r) * g.h[a]) - g.slack[a]);
            if (cc[a] + r < g.n[a] - 1)
                lb = fminf(lb, (g.x0[a] + (float)(cc[a] + r + 1) * g.h[a]) - pc[a] - g.slack[a]);
        }
        done = lb == INFINITY || (lb > 0.0f && m.d2 <= lb * lb * 0.9999f) || m.d2 == 0.0f;
    }
    if (sub != 0) return;
    const uint32_t i = __float_as_uint(p.w);
    if (done) store_scale(b, N, (int64_t)i, ls);
    else list[atomicAdd(n_list, 1u)] = i;
}

int64_t blocks(int64_t n, int per) { return (n + per - 1) / per; }

}  // namespace

int64_t rads_minmax_blocks(int64_t n, int num_cu) { return std::max<int64_t>(1, std::min<int64_t>(blocks(n, kRadsBlock), (int64_t)num_cu * 8)); }
size_t rads_edge_words(int64_t n) { return (size_t)rads_segments(n) * 3 * kRadsRounds; }
int64_t rads_segments(int64_t n) { return blocks(n, kRadsSeg); }
size_t rads_weight_words(int64_t n) { return (size_t)rads_segments(n) * kRadsSeg; }

hipError_t launch_rads_level(const RadsVol &v, float2 *part, int64_t nb, float *mm, hipStream_t s)
{
    const int64_t n = (int64_t)v.nx * v.ny * v.nz;
    minmax_kernel<<<(unsigned)nb, kRadsBlock, 0, s>>>(v.hu, n, part);
    minmax_final_kernel<<<1, kRadsBlock, 0, s>>>(part, (int)nb, mm);
    return hipGetLastError();
}

hipError_t launch_rads_segments(const RadsVol &v, const float *mm, uint16_t *w16, uint64_t *edge, uint32_t *scnt,
                                uint64_t *swt, RadsTotals *host, hipStream_t s)
{
    const int64_t n = (int64_t)v.nx * v.ny * v.nz, nseg = rads_segments(n);
    seg_count_kernel<<<(unsigned)blocks(nseg, kRadsBlock / kWave), kRadsBlock, 0, s>>>(v, (uint32_t)n, mm, nseg, w16,
                                                                                        edge, scnt, swt);
    seg_scan_kernel<<<1, kSegScanBlock, 0, s>>>(scnt, swt, nseg, mm, host);
    return hipGetLastError();
}

hipError_t launch_mc_emit(const RadsVol &v, const float *mm, const uint64_t *edge, const uint32_t *scnt, float *pts,
                          int64_t M, hipStream_t s)
{
    const int64_t n = (int64_t)v.nx * v.ny * v.nz, nseg = rads_segments(n);
    if (M == 0) return hipSuccess;
    mc_emit_kernel<<<(unsigned)nseg, kRadsBlock, 0, s>>>(v, mm, nseg, edge, scnt, pts, M);
    return hipGetLastError();
}

hipError_t launch_iota(uint32_t *p, int64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    iota_kernel<<<(unsigned)blocks(n, kRadsBlock), kRadsBlock, 0, s>>>(p, n);
    return hipGetLastError();
}

hipError_t launch_rads_gather(const float *src, int64_t M, const uint32_t *idx, int64_t n1, float *out, int64_t N,
                              hipStream_t s)
{
    if (n1 == 0) return hipSuccess;
    gather_kernel<<<(unsigned)blocks(n1, kRadsBlock), kRadsBlock, 0, s>>>(src, M, idx, n1, out, N);
    return hipGetLastError();
}

hipError_t launch_rads_pick(const uint32_t *tot, const uint2 *range, uint32_t *ka, uint32_t *va, uint32_t *kb,
                            uint32_t *vb, int64_t n1, const float *src, int64_t M, float *out, int64_t N, hipStream_t s)
{
    if (n1 == 0 || M == 0) return hipSuccess;
    if (M > kPickMax) return hipErrorInvalidValue;
    pick_kernel<<<1 << kTopBits, kPickBlock, 0, s>>>(tot, range, ka, va, kb, vb, n1, src, M, out, N);
    return hipGetLastError();
}

hipError_t launch_rads_begin(const RadsVol &v, const RadsBegin &b, hipStream_t s)
{
    const int64_t n = (int64_t)v.nx * v.ny * v.nz;
    if (b.range && b.M <= 0) return hipErrorInvalidValue;
    const int64_t n_range = b.range ? kKeyRangeBlocks : 0, n_clear = b.clear ? blocks(b.n_clear, kRadsBlock) : 0;
    const int64_t grid = n_range + n_clear + blocks(b.n2, kRadsBlock / kWave);
    if (grid == 0) return hipSuccess;
    begin_kernel<<<(unsigned)grid, kRadsBlock, 0, s>>>(v, (uint32_t)n, rads_segments(n), b, (int)n_range, (int)n_clear);
    return hipGetLastError();
}

bool knn_uses_grid(int64_t N) { return N > kKnnBrute; }

// Cubic cells over the box of the voxel centres, about four per point (axes
// thinner than a cell get one).
KnnGrid knn_grid(const RadsVol &v, int64_t N)
{
    KnnGrid g{};
    const double L[3] = {(double)(v.nx - 1) * v.sx, (double)(v.ny - 1) * v.sy, (double)(v.nz - 1) * v.sz};
    const float o[3] = {v.ox, v.oy, v.oz};
    const double target = std::min<double>(4.0 * (double)N, (double)kKnnMaxCells);
    bool on[3] = {L[0] > 0.0, L[1] > 0.0, L[2] > 0.0};
    double h = 0.0;
    for (int it = 0; it < 3; ++it) {
        double prod = 1.0;
        int dims = 0;
        for (int a = 0; a < 3; ++a)
            if (on[a]) {
                prod *= L[a];
                ++dims;
            }
        if (dims == 0) break;
        h = pow(prod / target, 1.0 / dims);
        for (int a = 0; a < 3; ++a) on[a] = on[a] && L[a] >= h;
    }
    double cells = 1.0;
    for (int a = 0; a < 3; ++a) {
        // (the running product keeps the cell count at most kKnnMaxCells)
        const double room = std::floor((double)kKnnMaxCells / cells);
        g.n[a] = on[a] && h > 0.0 ? (int)std::max(1.0, std::min(std::floor(L[a] / h), room)) : 1;
        cells *= g.n[a];
        const double ha = std::max(L[a], 1e-30) / g.n[a];
        g.x0[a] = o[a];
        g.h[a] = (float)ha;
        g.inv[a] = g.n[a] > 1 ? (float)(1.0 / ha) : 0.0f;
        g.slack[a] = (float)(8e-7 * (std::fabs((double)o[a]) + std::fabs((double)o[a] + L[a]) + L[a]));
    }
    return g;
}

hipError_t launch_knn_brute(const float *pts, int64_t N, float *ls, hipStream_t s)
{
    if (N == 0) return hipSuccess;
    knn_brute_kernel<<<(unsigned)N, kRadsBlock, 0, s>>>(pts, N, nullptr, nullptr, ls);
    return hipGetLastError();
}

hipError_t launch_knn_count(const KnnGrid &g, const float *pts, int64_t N, uint32_t *cnt, hipStream_t s)
{
    knn_count_kernel<<<(unsigned)blocks(N, kRadsBlock), kRadsBlock, 0, s>>>(g, pts, N, cnt);
    return hipGetLastError();
}

hipError_t launch_knn_grid(const KnnGrid &g, const float *pts, int64_t N, uint32_t *cur, float4 *sorted,
                           uint32_t *list, uint32_t *n_list, float *ls, hipStream_t s)
{
    knn_place_kernel<<<(unsigned)blocks(N, kRadsBlock), kRadsBlock, 0, s>>>(g, pts, N, cur, sorted);
    knn_query_kernel<<<(unsigned)blocks(N, kRadsBlock / kKnnLanes), kRadsBlock, 0, s>>>(g, sorted, N, cur, ls, list,
                                                                                        n_list);
    // (what the rings left open; a fixed grid, most of it idle)
    knn_brute_kernel<<<kKnnFarBlocks, kRadsBlock, 0, s>>>(pts, N, list, n_list, ls);
    return hipGetLastError();
}

}  // namespace ddgs
