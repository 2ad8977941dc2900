// raster.hip -- per-tile compositing of Eq. 1 on gfx950 and its backward.
//
// Work items.  A work item is a (tile, depth chunk) pair: the tile's
// depth-ordered list is cut into chunks of `split` entries (split = 0: one
// item per tile).  Chunking bounds the serial walk of any one workgroup, so
// tiles with very long lists no longer set the kernel's critical path, and
// the 256 CUs get thousands of similar-sized items.  Eq. 1 is a left fold
// of the "over" operator (C, T) o (C', T') = (C + T C', T T'), which is
// associative, so chunk results are merged exactly in depth order by a
// small merge kernel (which also stores, for every chunk, the (C, T) in
// front of it for the backward).  With split = 0 the image is bit-identical
// for every tile shape; with chunks it differs only by rounding.
//
// Inside an item one workgroup owns the tile and one lane owns one pixel.
// The item's entries are staged in LDS in batches (one 32-byte record per
// entry) and read back as wave-wide broadcasts.  The per-pair arithmetic is
// written with explicit round-to-nearest intrinsics so that the forward and
// the backward (which recomputes the transmittance instead of storing it)
// take bit-identical decisions.
//
// Backward: the tail S_j = sum_{m>j} c_m s_m T_m is the saved pixel value
// minus the running sum.  Per-pair image-plane gradients are summed over the
// wave (through LDS for chunked items, with DPP row operations for unchunked
// ones), over the waves of the workgroup in LDS in a fixed order,
// and written once per tile entry into its own slot (the pair's first slot plus the tile's row-major
// place in the pair's rectangle) -- no float atomics, so the gradients are
// run-to-run deterministic.
#include "internal.h"

namespace ddgs {

namespace {

// The falloff exponent.  The conic is staged in LDS pre-multiplied by
// kExpScale = -log2(e) / 2 (A00 k, 2 A01 k, A11 k), so that
// e = dx (A00' dx + B' dy) + A11' dy dy -- five rounded operations, the same
// in the forward and the backward -- is -d2 / 2 in base-2 units: the falloff
// exp(-d2 / 2) is v_exp_f32(e), and the cut-off d2 <= kappa^2 becomes
// e >= kappa^2 k (both sides scaled by the same negative factor).
constexpr float kExpScale = -0.7213475108146667f;  // 0xBF38AA3B, -log2(e) / 2
__device__ __forceinline__ float falloff_exponent(float dx, float dy, float A00, float B, float A11)
{
    const float u = __fmaf_rn(B, dy, __fmul_rn(A00, dx));
    return __fmaf_rn(dx, u, __fmul_rn(__fmul_rn(A11, dy), dy));
}
// The staged conic of a record: (mx, my, A00 k, 2 A01 k) and (A11 k, alpha, c, .)
__device__ __forceinline__ void scale_conic(float4 &r0, float4 &r1)
{
    r0.z = __fmul_rn(r0.z, kExpScale);
    r0.w = __fmul_rn(2.0f * r0.w, kExpScale);
    r1.x = __fmul_rn(r1.x, kExpScale);
}
// Cut-off value of a lane: kappa^2 k (< 0) while it composites, +infinity
// (which no exponent of a finite record reaches) once it has stopped or lies
// outside the image.
constexpr float kLaneOff = __builtin_huge_valf();

// min(s, sigma_max) for s = alpha G >= 0 as one v_med3_f32 (median of s,
// 0 and sigma_max), without the NaN canonicalisation fminf brings.
__device__ __forceinline__ float clamp_opacity(float s, float smax) { return __builtin_amdgcn_fmed3f(s, 0.0f, smax); }
// 1 - s for an unclamped s = alpha G, in one rounding (the same in the
// forward and every backward)
__device__ __forceinline__ float one_minus_alpha_g(float alpha, float G) { return __fmaf_rn(-alpha, G, 1.0f); }

// Wave-wide OR of a predicate as a lane mask (the compare mask itself).
__device__ __forceinline__ uint64_t wave_any_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }


__device__ __forceinline__ int view_of_tile(const ViewDev *views, int V, int tile)
{
    int lo = 0, hi = V - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_base <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct Item {
    int tile;
    uint32_t b, e;    // entry range [b, e) of the item
    int chunk;
};

// Resolves work item `it`; tile < 0 when `it` is past the last item.  The
// item is built in registers and returned whole (field-wise stores through
// a reference were kept in scratch memory by the compiler).
__device__ __forceinline__ Item resolve_item(const RasterArgs &a, int it)
{
    int tile = -1, chunk = 0;
    uint32_t b = 0, e = 0;
    if (it != 0x7FFFFFFF) {
        if (a.split == 0) {
            if (it < a.n_tiles) {
                const uint2 rg = a.ranges[it];
                tile = it;
                b = rg.x;
                e = rg.y;
            }
        } else if (it < (int)*a.n_items) {
            const uint2 q = a.items[it];
            const uint2 rg = a.ranges[q.x];
            tile = (int)q.x;
            chunk = (int)q.y;
            b = rg.x + q.y * (uint32_t)a.split;
            e = min(rg.y, b + (uint32_t)a.split);
        }
    }
    return Item{__builtin_amdgcn_readfirstlane(tile), (uint32_t)__builtin_amdgcn_readfirstlane((int)b),
                (uint32_t)__builtin_amdgcn_readfirstlane((int)e), __builtin_amdgcn_readfirstlane(chunk)};
}

// Item of block b when blocks map to items directly.  Workgroups are dealt
// to the eight XCDs in turn (block b to XCD b mod 8), and each XCD has its
// own L2: XCD x gets the x-th contiguous eighth of the n items, so that
// neighbouring tiles, which share most of their Gaussians, read those
// records through the same L2.  The grid is a multiple of 8 and at least n.
__device__ __forceinline__ int xcd_item(int b, int n)
{
    const int per = (n + 7) >> 3;
    const int k = b >> 3;
    return k < per ? (b & 7) * per + k : 0x7FFFFFFF;
}

// Next work item of this workgroup: the item of its block once, or
// (persistent mode) items taken from a shared counter until none are left.
__device__ __forceinline__ int next_item(const RasterArgs &a, int &iter, int *sh)
{
    if (!a.queue_counter) {
        const int n = a.split ? (int)*a.n_items : a.n_tiles;
        const int t = iter == 0 ? xcd_item((int)blockIdx.x, n) : 0x7FFFFFFF;
        ++iter;
        return t;
    }
    __syncthreads();
    if (threadIdx.x == 0) *sh = (int)atomicAdd(a.queue_counter, 1u);
    __syncthreads();
    const int k = *sh;
    ++iter;
    const int limit = a.split ? (int)*a.n_items : a.n_tiles;
    if (k >= limit) return 0x7FFFFFFF;
    return a.queue ? (int)a.queue[k] : k;
}

// Half-widths of a box around the mean that holds every pixel the cut-off test
// may pass, from the stored conic (kw: kappa, widened by 0.1 % for the rounding
// of the means, the half-widths and the box tests).  The ellipse's are kappa
// sqrt(A11 / det) and kappa sqrt(A00 / det) with det = A00 A11 - A01^2, which
// cancels for long thin footprints (by a relative 2^-24 A00 A11 / det: 6 % at
// 1000 x 0.5 pixels).  The test rounds d^T A d by at most 8 2^-24 (A00 dx^2 +
// 2 |A01 dx dy| + A11 dy^2), so what it passes lies in the ellipse of the form
// with A00 and A11 smaller and |A01| larger by that factor, whose determinant is
// at least det - 33 2^-24 A00 A11; with det's own rounding, 3e-6 A00 A11 are
// taken off.  Where nothing is left (footprints longer than about 1200 times
// their width, or products near the smallest float) the box has no bounds, and
// its tests are written so that a NaN passes them too.
__device__ __forceinline__ float2 cutoff_box(float kw, float A00, float A01, float A11)
{
    const float p = A00 * A11;
    const float det = __fmaf_rn(-A01, A01, p) - 3e-6f * p;
    // (v_rcp_f32 and v_sqrt_f32 are one ulp off, which the 0.1 % covers)
    const float idet = det > 1e-30f ? __builtin_amdgcn_rcpf(det) : INFINITY;
    return make_float2(kw * __builtin_amdgcn_sqrtf(A11 * idet), kw * __builtin_amdgcn_sqrtf(A00 * idet));
}
// the interval [x - h, x + h] reaches [lo, hi]
__device__ __forceinline__ bool box_reaches(float x, float h, float lo, float hi)
{
    return !(x - h > hi) & !(x + h < lo);
}

// SPLIT: work items are chunks (a.split > 0), so no per-pixel last index is
// kept; COUNT: pair counters on.
template <int TW, int TH, bool SPLIT, bool COUNT>
__global__ __launch_bounds__(TW *TH) void raster_fwd_kernel(RasterArgs a)
{
    constexpr int NT = TW * TH;
    __shared__ float4 s0[NT];
    __shared__ float4 s1[NT];
    __shared__ int sh_item;
    const int tid = threadIdx.x;
    const float k2s = __fmul_rn(a.o.kappa2, kExpScale), tmin = a.o.t_min;
    const float smax = a.o.sigma_max;
    int iter = 0;
    for (;;) {
        const int it = next_item(a, iter, &sh_item);
        const Item I = resolve_item(a, it);
        if (I.tile < 0) break;
        const int v = view_of_tile(a.views, a.V, I.tile);
        const ViewDev &V = a.views[v];
        const int lt = I.tile - V.tile_base;
        const int ty = lt / V.ntx, tx = lt - ty * V.ntx;
        const int px = tx * TW + tid % TW, py = ty * TH + tid / TW;
        const bool inside = px < V.W && py < V.H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        const size_t vbase = (size_t)v * a.n;
        float T = 1.0f, C = 0.0f;
        uint32_t last = I.b;
        uint32_t n_eval = 0, n_contrib = 0;
        // the cut-off test with the lane's state folded in (kLaneOff once the
        // lane has stopped or lies outside the image), so that a hit is one
        // compare and its wave ballot costs no vector instruction
        float k2e = inside ? k2s : kLaneOff;
        // one entry: when any lane hits, the whole wave runs it without
        // branches; lanes that miss keep their state.  CLAMP: some entry of
        // the batch has alpha > sigma_max / 2.  Otherwise alpha G stays below
        // sigma_max with a factor-two margin (G <= 1, up to the rounding of
        // its exponent) and the clamp min(alpha G, sigma_max) is the identity
        auto entry = [&](const float4 r0, const float4 r1, uint32_t pos, auto clamp_c) {
            constexpr bool CLAMP = decltype(clamp_c)::value;
            const float dx = __fsub_rn(fpx, r0.x), dy = __fsub_rn(fpy, r0.y);
            const float ex = falloff_exponent(dx, dy, r0.z, r0.w, r1.x);
            bool hit = ex >= k2e;
            if (wave_any_mask(hit) != 0ull) {
                // (an empty volatile asm keeps this a branch: the compiler would
                // otherwise turn the entry into selects, which run it, and
                // two more selects, even when no lane hits)
                asm volatile("");
                // lanes that miss run the same arithmetic with G = 0: s = 0,
                // 1 - s = 1, so C and T stay exactly as they are
                float G = hit ? __builtin_amdgcn_exp2f(ex) : 0.0f;
                float s = __fmul_rn(r1.y, G), om;
                if constexpr (CLAMP) {
                    s = clamp_opacity(s, smax);
                    om = __fsub_rn(1.0f, s);
                } else {
                    om = one_minus_alpha_g(r1.y, G);
                }
                if constexpr (!SPLIT) {
                    // early termination (t_min > 0 runs unsplit): the lane
                    // stops before this entry
                    if (tmin > 0.0f) {
                        const bool stop = hit & (__fmul_rn(T, om) < tmin);
                        k2e = stop ? kLaneOff : k2e;
                        hit = hit & !stop;
                        s = stop ? 0.0f : s;
                        om = stop ? 1.0f : om;
                    }
                }
                // C += c (s T); T *= 1 - s exactly as the backward recomputes it
                C = __fmaf_rn(r1.z, __fmul_rn(s, T), C);
                T = __fmul_rn(T, om);
                if constexpr (!SPLIT) last = hit ? pos + 1u : last;
                if constexpr (COUNT) n_contrib += hit ? 1u : 0u;
            }
        };
        // the batch's entries in order, four records read together (one LDS
        // address, immediate offsets)
        auto run_batch = [&](uint32_t b0, int cnt, auto clamp_c) {
            int q = 0;
            for (; q + 4 <= cnt; q += 4) {
                float4 r0[4], r1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    r0[u] = s0[q + u];
                    r1[u] = s1[q + u];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) entry(r0[u], r1[u], b0 + (uint32_t)(q + u), clamp_c);
            }
            for (; q < cnt; ++q) entry(s0[q], s1[q], b0 + (uint32_t)q, clamp_c);
        };
        for (uint32_t b0 = I.b; b0 < I.e; b0 += NT) {
            __syncthreads();
            const uint32_t j = b0 + tid;
            bool over = false;  // an opacity above sigma_max / 2 in this batch
            if (j < I.e) {
                const uint32_t gid = min(a.tval[j], (uint32_t)a.n - 1u);
                const size_t idx = vbase + gid;
                float4 r0 = a.rec[4 * idx], r1 = a.rec[4 * idx + 1];
                over = r1.y > 0.5f * smax;
                scale_conic(r0, r1);
                s0[tid] = r0;
                s1[tid] = r1;
            }
            const bool clamp = __syncthreads_or(over);
            const int cnt = (int)min((uint32_t)NT, I.e - b0);
            if (COUNT && k2e < 0.0f) n_eval += (uint32_t)cnt;
            if (clamp) run_batch(b0, cnt, std::true_type{});
            else run_batch(b0, cnt, std::false_type{});
            if (tmin > 0.0f && __syncthreads_and(k2e == kLaneOff)) break;
        }
        if constexpr (COUNT) {
            unsigned long long e = n_eval, c = n_contrib;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                e += __shfl_xor(e, o, kWave);
                c += __shfl_xor(c, o, kWave);
            }
            if ((tid & (kWave - 1)) == 0) {
                // 64 counter pairs, chosen by block, keep the atomics uncontended
                const int slot = (int)(blockIdx.x & 63u);
                atomicAdd(&a.pair_counts[2 * slot], e);
                atomicAdd(&a.pair_counts[2 * slot + 1], c);
            }
        }
        if constexpr (SPLIT) {
            a.part[(size_t)it * NT + tid] = make_float2(C, T);
        } else if (inside) {
            const size_t p = (size_t)V.pix_base + (size_t)py * V.W + px;
            a.img[p] = C;
            a.img_saved[p] = C;
            a.nlast[p] = last;
        }
    }
}

// Forward of chunked items with an entry list per 4 x 4 cell of the tile.  An
// entry's cut-off ellipse usually covers a part of the tile, and a wave that
// runs it on all its pixels spends most lanes on misses.  Here each wave owns
// an 8 x 8 part of the tile and lane l covers pixel (4 (q % 2) + r % 4,
// 4 (q / 2) + r / 4) of it (q = l / 16, r = l % 16), so that each 16-lane row
// covers one cell; each batch of entries is listed per cell whose pixel
// centres the ellipse's bounding box reaches (cutoff_box, which holds every
// pixel that the rounded per-pixel test passes), and the wave runs the longest of
// its four lists, the lanes of each cell taking their own list's entries in
// depth order (shorter lists are padded with a record that no pixel reaches).
// An entry left out of a cell's list misses all its pixels, where the update
// is an exact no-op, so the images and chunk results equal the unculled
// kernel's bit for bit.  The chunk results are stored by pixel (row-major in
// the tile), as the other kernels index them.
//
// Tiles of several waves stage a batch of one record per pixel together and
// every wave lists it for its own cells: at 500k Gaussians / 512^2 and 16 x 16
// tiles 86 us against 140 us for the unculled kernel (which runs every entry
// on all 256 pixels).
template <int TW, int TH>
__global__ __launch_bounds__(TW *TH) void raster_fwd_cells_kernel(RasterArgs a)
{
    constexpr int NT = TW * TH, NW = NT / kWave, NUL = NT;
    constexpr int CX = TW / 4, CY = TH / 4;  // cells per row and column of the tile
    // records by entry, s1 first: entry e's pair sits at byte 16 e (s1) and
    // 16 e + S0OFF (s0), so that one register with two immediate offsets
    // reads it; the lists hold these byte places
    constexpr uint32_t S0OFF = 16u * (NT + 1);
    __shared__ float4 s10[2 * (NT + 1)];
    float4 *const s1 = s10;
    float4 *const s0 = s10 + (NT + 1);
    // per cell: the byte places of its entries (rows four words apart in
    // bank, so that the four cells' reads of one step do not collide)
    __shared__ __align__(16) uint32_t ql[4 * NW][NT + 4];
    __shared__ uint32_t reach[NW > 1 ? NT : 1];  // cell columns (low bits) and rows an entry reaches
    __shared__ int sh_item;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = NW > 1 ? tid / kWave : 0;
    const int qd = lane >> 4, qr = lane & 15;
    // this wave's first cell, this lane's pixel of the tile
    const int wcx = 2 * (w % (TW / 8)), wcy = 2 * (w / (TW / 8));
    const int lx = 4 * (wcx + (qd & 1)) + (qr & 3), ly = 4 * (wcy + (qd >> 1)) + (qr >> 2);
    const float k2s = __fmul_rn(a.o.kappa2, kExpScale);
    const float smax = a.o.sigma_max;
    const float kw = a.o.kappa * 1.001f;
    if (tid == 0) {
        // the padding record: d^T A d = -(dx^2 + dy^2) ~ -2e36 < any cut-off
        s0[NUL] = make_float4(1e18f, 1e18f, -1.0f, 0.0f);
        s1[NUL] = make_float4(-1.0f, 0.0f, 0.0f, 0.0f);
    }
    const char *const srec = reinterpret_cast<const char *>(s10);
    int iter = 0;
    for (;;) {
        const int it = next_item(a, iter, &sh_item);
        const Item I = resolve_item(a, it);
        if (I.tile < 0) break;
        const int v = view_of_tile(a.views, a.V, I.tile);
        const ViewDev &V = a.views[v];
        const int lt = I.tile - V.tile_base;
        const int ty = lt / V.ntx, tx = lt - ty * V.ntx;
        const int px = tx * TW + lx, py = ty * TH + ly;
        const bool inside = px < V.W && py < V.H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        const float tx0 = (float)(tx * TW), ty0 = (float)(ty * TH);
        const size_t vbase = (size_t)v * a.n;
        float T = 1.0f, C = 0.0f;
        const float k2e = inside ? k2s : kLaneOff;
        auto entry = [&](const float4 r0, const float4 r1, auto clamp_c) {
            constexpr bool CLAMP = decltype(clamp_c)::value;
            const float dx = __fsub_rn(fpx, r0.x), dy = __fsub_rn(fpy, r0.y);
            const float ex = falloff_exponent(dx, dy, r0.z, r0.w, r1.x);
            const bool hit = ex >= k2e;
            if (wave_any_mask(hit) != 0ull) {
                asm volatile("");
                const float G = hit ? __builtin_amdgcn_exp2f(ex) : 0.0f;
                float s = __fmul_rn(r1.y, G), om;
                if constexpr (CLAMP) {
                    s = clamp_opacity(s, smax);
                    om = __fsub_rn(1.0f, s);
                } else {
                    om = one_minus_alpha_g(r1.y, G);
                }
                C = __fmaf_rn(r1.z, __fmul_rn(s, T), C);
                T = __fmul_rn(T, om);
            }
        };
        // the longest list in steps of four: four places of the lane's list,
        // then their records
        const uint32_t *const myl = &ql[4 * w + qd][0];
        auto run_lists = [&](int nmax, auto clamp_c) {
            for (int i0 = 0; i0 < nmax; i0 += 4) {
                const uint4 ev = *reinterpret_cast<const uint4 *>(myl + i0);
                const uint32_t e[4] = {ev.x, ev.y, ev.z, ev.w};
                float4 r0[4], r1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    r1[u] = *reinterpret_cast<const float4 *>(srec + e[u]);
                    r0[u] = *reinterpret_cast<const float4 *>(srec + e[u] + S0OFF);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) entry(r0[u], r1[u], clamp_c);
            }
        };
        for (uint32_t b0 = I.b; b0 < I.e; b0 += NT) {
            __syncthreads();
            const uint32_t j = b0 + tid;
            bool over = false;  // an opacity above sigma_max / 2 in this batch
            uint32_t rm = 0u;   // bit i: reaches cell column i; bit CX + i: cell row i
            if (j < I.e) {
                const uint32_t gid = min(a.tval[j], (uint32_t)a.n - 1u);
                const size_t idx = vbase + gid;
                float4 r0 = a.rec[4 * idx], r1 = a.rec[4 * idx + 1];
                over = r1.y > 0.5f * smax;
                // bounding box of the cut-off ellipse against the cells'
                // pixel-centre ranges [4 i + 0.5, 4 i + 3.5] of the tile
                const float2 h = cutoff_box(kw, r0.z, r0.w, r1.x);
                const float ux = r0.x - tx0, uy = r0.y - ty0;
#pragma unroll
                for (int i = 0; i < CX; ++i)
                    rm |= box_reaches(ux, h.x, 4.0f * i + 0.5f, 4.0f * i + 3.5f) ? 1u << i : 0u;
#pragma unroll
                for (int i = 0; i < CY; ++i)
                    rm |= box_reaches(uy, h.y, 4.0f * i + 0.5f, 4.0f * i + 3.5f) ? 1u << (CX + i) : 0u;
                scale_conic(r0, r1);
                s0[tid] = r0;
                s1[tid] = r1;
            }
            if constexpr (NW > 1) reach[tid] = rm;
            // lists: every place first holds the padding record, then each
            // cell's entries in batch order
#pragma unroll
            for (int h = 0; h < NW; ++h)
                reinterpret_cast<uint4 *>(&ql[4 * w + qd][4 * qr])[16 * h] =
                    make_uint4(16u * NUL, 16u * NUL, 16u * NUL, 16u * NUL);
            const bool clamp = __syncthreads_or(over);
            int len[4] = {0, 0, 0, 0};
#pragma unroll
            for (int h = 0; h < NW; ++h) {
                const uint32_t m = NW > 1 ? reach[h * kWave + lane] : rm;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t need = (1u << (wcx + (q & 1))) | (1u << (CX + wcy + (q >> 1)));
                    const bool in = (m & need) == need;
                    const uint64_t bal = wave_any_mask(in);
                    if (in) {
                        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                        ql[4 * w + q][len[q] + pos] = 16u * (uint32_t)(h * kWave + lane);
                    }
                    len[q] += (int)__popcll(bal);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int nmax = max(max(len[0], len[1]), max(len[2], len[3]));
            if (clamp) run_lists(nmax, std::true_type{});
            else run_lists(nmax, std::false_type{});
        }
        a.part[(size_t)it * NT + ly * TW + lx] = make_float2(C, T);
    }
}

// Split mode: folds each tile's chunk results in depth order with the over
// operator, writes the images, and replaces every chunk's (C, T) by the
// (C, T) accumulated in front of it (what the chunk's backward starts from).
// (several tiles per workgroup for the one-wave tiles, one per wave:
// fewer, larger workgroups)
template <int TW, int TH>
constexpr int merge_tiles_per_block() { return TW * TH >= 256 ? 1 : 256 / (TW * TH); }

template <int TW, int TH>
__global__ __launch_bounds__((TW * TH * merge_tiles_per_block<TW, TH>())) void merge_kernel(RasterArgs a)
{
    constexpr int NT = TW * TH;
    const int tile = blockIdx.x * merge_tiles_per_block<TW, TH>() + (int)threadIdx.x / NT;
    if (tile >= a.n_tiles) return;
    const int tid = threadIdx.x % NT;
    const int v = view_of_tile(a.views, a.V, tile);
    const ViewDev &V = a.views[v];
    const int lt = tile - V.tile_base;
    const int ty = lt / V.ntx, tx = lt - ty * V.ntx;
    const int px = tx * TW + tid % TW, py = ty * TH + tid / TW;
    const uint32_t base = a.item_base[tile], cnt = a.item_cnt[tile];
    const uint32_t last = a.ranges[tile].y;
    // items past the item capacity do not exist (overflowed step)
    const uint32_t mi = (uint32_t)a.max_items;
    const uint32_t kend = base < mi ? min(cnt, mi - base) : 0u;
    float2 *const pp = a.part + (size_t)base * NT + tid;
    float C = 0.0f, T = 1.0f;
    // four items' partials read together (each item's place then receives
    // the (C, T) in front of it)
    uint32_t k = 0;
    for (; k + 4u <= kend; k += 4u) {
        float2 ck[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ck[u] = pp[(size_t)(k + u) * NT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            pp[(size_t)(k + u) * NT] = make_float2(C, T);
            C = __fmaf_rn(T, ck[u].x, C);
            T = __fmul_rn(T, ck[u].y);
        }
    }
    for (; k < kend; ++k) {
        const float2 ck = pp[(size_t)k * NT];
        pp[(size_t)k * NT] = make_float2(C, T);
        C = __fmaf_rn(T, ck.x, C);
        T = __fmul_rn(T, ck.y);
    }
    if (px < V.W && py < V.H) {
        const size_t p = (size_t)V.pix_base + (size_t)py * V.W + px;
        a.img[p] = C;
        a.img_saved[p] = C;
        a.nlast[p] = last;
    }
}

// Backward of unchunked items (split 0, and t_min > 0, which a lane's stop
// needs): one workgroup per tile, every entry on all its pixels.
template <int TW, int TH>
__global__ __launch_bounds__(TW *TH) void raster_bwd_kernel(RasterArgs a)
{
    constexpr int NT = TW * TH;
    constexpr int NW = NT / kWave;
    constexpr int NA = NW > 1 ? NW : 1, NTA = NW > 1 ? NT : 1;
    // one array, s1 first: the paired 4-byte reads of alpha and c then reach
    // it with in-range immediate offsets from the same register as the
    // 16-byte reads of s0
    __shared__ float4 s10[2 * NT];
    float4 *const s1 = s10;
    float4 *const s0 = s10 + NT;
    __shared__ uint32_t se[NT];
    __shared__ __align__(16) float acc[NA][NTA][8];  // several waves: per-wave entry sums
    __shared__ uint32_t wmax[NW];
    __shared__ int sh_item;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    // entries per transposing sum, gradient terms per entry, entries staged
    // per batch (a whole number of groups), and this lane's (entry, term)
    // after the sum (lane 63 holds the pad)
    constexpr int kTerms = 7, EPG = kWave / kTerms;
    constexpr int BATCH = (NT / EPG) * EPG;
    static_assert(EPG * kTerms < kWave, "one pad value");
    const int l_entry = lane / kTerms, l_term = lane - l_entry * kTerms;
    const float k2s = __fmul_rn(a.o.kappa2, kExpScale), tmin = a.o.t_min;
    const float smax = a.o.sigma_max;
    float *slotf = reinterpret_cast<float *>(a.slot);
    int iter = 0;
    for (;;) {
        const int it = next_item(a, iter, &sh_item);
        const Item I = resolve_item(a, it);
        if (I.tile < 0) break;
        const int v = view_of_tile(a.views, a.V, I.tile);
        const ViewDev &V = a.views[v];
        const int lt = I.tile - V.tile_base;
        const int ty = lt / V.ntx, tx = lt - ty * V.ntx;
        const int px = tx * TW + tid % TW, py = ty * TH + tid / TW;
        const bool inside = px < V.W && py < V.H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        const size_t vbase = (size_t)v * a.n;
        float g = 0.0f, Cf = 0.0f, T = 1.0f;
        uint32_t lastp = I.b;
        if (inside) {
            const size_t p = (size_t)V.pix_base + (size_t)py * V.W + px;
            g = a.dL_dimg[p];
            Cf = a.img_saved[p];
            lastp = a.nlast[p];
        }
        // g times the tail S (the saved pixel value minus the colour
        // composited so far), kept up to date entry by entry
        float Sg = g * Cf;
        // end of the longest contributing prefix in the item
        uint32_t m = lastp;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, kWave));
        __syncthreads();
        if (lane == 0) wmax[w] = m;
        __syncthreads();
        uint32_t end = wmax[0];
#pragma unroll
        for (int q = 1; q < NW; ++q) end = max(end, wmax[q]);

        // the cut-off test with the lane's state folded in (kLaneOff once
        // stopped or outside the image): a hit is one compare, its ballot is free
        float k2e = inside ? k2s : kLaneOff;
        // the staged batch's entries in groups of EPG, CLAMP as in the forward
        // (without it every alpha of the batch is at most sigma_max / 2: s =
        // alpha G and no step is clamped)
        auto run_groups = [&](uint32_t b0, int cnt, auto clamp_c) {
            constexpr bool CLAMP = decltype(clamp_c)::value;
            // groups of EPG = 9 entries: their 7 gradient terms fill 63 of
            // the 64 values of one transposing wave sum (the last is a
            // zero pad); lane l ends with term l % 7 of entry l / 7
            for (int q0 = 0; q0 < cnt; q0 += EPG) {
                float gb[64];
                bool any = false;
                // the group's first entry index, held in one vector
                // register (an empty asm makes it opaque) so that the
                // entries' LDS reads use it with immediate offsets instead
                // of rebuilding an address for each entry
                int qv = q0;
                asm volatile("" : "+v"(qv));
#pragma unroll
                for (int qq = 0; qq < EPG; ++qq) {
                    float gv[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    const int q = q0 + qq;
                    if (q < cnt) {
                        const float4 r0 = s0[qv + qq];
                        const float4 r1 = s1[qv + qq];
                        const float dx = __fsub_rn(fpx, r0.x), dy = __fsub_rn(fpy, r0.y);
                        const float ex = falloff_exponent(dx, dy, r0.z, r0.w, r1.x);
                        bool hit = ex >= k2e;
                        hit = hit && (b0 + (uint32_t)q) < lastp;
                        // when any lane hits, the whole wave runs the entry:
                        // computed without branches, lanes that miss keep
                        // their state and contribute zeros
                        if (wave_any_mask(hit) != 0ull) {
                            // lanes that miss run the same arithmetic with
                            // G = 0: s = 0, 1 - s = 1, so the running colour
                            // and T stay exactly as they are and every term
                            // below is zero
                            float G = hit ? __builtin_amdgcn_exp2f(ex) : 0.0f;
                            float sraw = __fmul_rn(r1.y, G);
                            float s = sraw, om;
                            if constexpr (CLAMP) {
                                s = clamp_opacity(sraw, smax);
                                om = __fsub_rn(1.0f, s);
                            } else {
                                om = one_minus_alpha_g(r1.y, G);
                            }
                            if (tmin > 0.0f) {
                                const bool stop = hit & (__fmul_rn(T, om) < tmin);
                                k2e = stop ? kLaneOff : k2e;
                                hit = hit & !stop;
                                G = stop ? 0.0f : G;
                                sraw = stop ? 0.0f : sraw;
                                s = stop ? 0.0f : s;
                                om = stop ? 1.0f : om;
                            }
                            // dL/ds = g (c T - S / (1 - s)) with S the tail
                            // after this entry: g S is updated by -g c s T
                            const float c = r1.z;
                            const float sT = __fmul_rn(s, T);
                            const float gc = g * c;
                            Sg = __fmaf_rn(-gc, sT, Sg);
                            const float ds = __fmaf_rn(gc, T, -(Sg * __builtin_amdgcn_rcpf(om)));
                            // moments of dL/ds G about the mean; the conic and
                            // alpha factors are applied once per (view,
                            // Gaussian) in the projection backward
                            float gds = ds * G;
                            if constexpr (CLAMP) gds = (sraw > smax) ? 0.0f : gds;
                            const float m1x = gds * dx, m1y = gds * dy;
                            gv[0] = m1x;
                            gv[1] = m1y;
                            gv[2] = m1x * dx;
                            gv[3] = m1x * dy;
                            gv[4] = m1y * dy;
                            gv[5] = gds;
                            gv[6] = g * sT;
                            T = __fmul_rn(T, om);
                            any = true;
                        }
                    }
#pragma unroll
                    for (int c = 0; c < kTerms; ++c) gb[qq * kTerms + c] = gv[c];
                }
                gb[63] = 0.0f;
                float res = 0.0f;
                if (wave_any_mask(any) != 0ull) {
                    wave_transpose_sum64(gb);
                    res = gb[0];
                }
                const int q = q0 + l_entry;
                if (l_entry < EPG && q < cnt) {
                    if constexpr (NW == 1) {
                        const size_t e = se[q];
                        if (e < a.slot_cap) slotf[8 * e + l_term] = res;
                    } else {
                        acc[w][q][l_term] = res;
                    }
                }
            }
        };
        for (uint32_t b0 = I.b; b0 < I.e; b0 += BATCH) {
            const int cnt = (int)min((uint32_t)BATCH, I.e - b0);
            __syncthreads();
            const uint32_t j = b0 + tid;
            bool over = false;  // an opacity above sigma_max / 2 in this batch
            if (tid < BATCH && j < I.e) {
                const uint32_t gid = min(a.tval[j], (uint32_t)a.n - 1u);
                const size_t idx = vbase + gid;
                // one 64-byte line per pair: record, place in the slot
                // numbering, rectangle and tile mask
                float4 r0 = a.rec[4 * idx], r1 = a.rec[4 * idx + 1];
                const float4 r2 = a.rec[4 * idx + 2];
                const uint32_t place = __float_as_uint(r1.w);
                over = r1.y > 0.5f * smax;
                scale_conic(r0, r1);
                s0[tid] = r0;
                s1[tid] = r1;
                // the slot: the pair's first slot plus this tile's rank among
                // the pair's kept tiles (row-major in its rectangle)
                const uint32_t rx = __float_as_uint(r2.x), ry = __float_as_uint(r2.y);
                const int tx0 = rx & 0xFFFF, ty0 = rx >> 16, tx1 = ry & 0xFFFF, ty1 = ry >> 16;
                const uint32_t area = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
                const uint32_t at = (uint32_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0));
                se[tid] = first_slot(a.slot_bofs, a.slot_nblk, v, (int)gid, place) +
                          kept_rank(__float_as_uint(r2.z), area, at);
            }
            const bool clamp = __syncthreads_or(over);
            if (b0 < end && clamp) run_groups(b0, cnt, std::true_type{});
            else if (b0 < end) run_groups(b0, cnt, std::false_type{});
            if constexpr (NW > 1) {
                __syncthreads();
                if (tid < cnt) {
                    float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0;
                    if (b0 < end) {
#pragma unroll
                        for (int q = 0; q < NW; ++q) {
                            const float4 x0 = *reinterpret_cast<const float4 *>(&acc[q][tid][0]);
                            const float4 x1 = *reinterpret_cast<const float4 *>(&acc[q][tid][4]);
                            r0.x += x0.x; r0.y += x0.y; r0.z += x0.z; r0.w += x0.w;
                            r1.x += x1.x; r1.y += x1.y; r1.z += x1.z;
                        }
                    }
                    const size_t e = se[tid];
                    if (e < a.slot_cap) {
                        a.slot[2 * e] = r0;
                        a.slot[2 * e + 1] = r1;
                    }
                }
            } else {
                if (b0 >= end && tid < cnt) {
                    const size_t e = se[tid];
                    if (e < a.slot_cap) {
                        a.slot[2 * e] = make_float4(0.f, 0.f, 0.f, 0.f);
                        a.slot[2 * e + 1] = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                }
            }
        }
    }
}

// Backward of chunked items.  Each wave owns an 8 x 8 part of the tile, one
// lane per pixel, and runs the entries of its list (those whose cut-off box
// reaches the part; with 8 x 8 tiles every entry of the item) in two sweeps
// over eight at a time:
//
//   front to back: G, s and gT = g T (g = dL/dC of the pixel) of every entry,
//     the colour term g s T, and Sg = g times the tail S behind the eight;
//   back to front: with B = S / T = the colour seen behind entry j,
//     dL/ds_j = g T_j (c_j - B), then B <- c_j - (1 - s_j) (c_j - B).
// Only one division per eight entries is left (B behind the last, Sg /
// gT); per entry it was v_rcp_f32 (8.4 clocks per wave here, against 2.4 of a
// multiply) and three more operations.  Sg is a difference of colours of
// order g, so B = Sg / gT is only known to about eps / T; each step back
// multiplies that error by (1 - s) and gT_j = gT / prod (1 - s), so what
// reaches dL/ds_j is eps g / (1 - s_j), as with the division per entry.
//
// The seven per-entry sums over the pixels: q = dL/ds G (zero where a pixel
// misses an entry) goes to LDS for sixteen entries, and comes back with one
// lane per (entry, 4 x 4 quarter of the part), which forms the quarter's
// moments about its centre from its sixteen values in registers (43 additions
// and multiply-adds), shifts them to the entry's mean and adds the quarters
// over its lane row.  (About quarters, since a small Gaussian's moments lose
// bits in the shift from a distant centre.)  The same moments as a dense
// contraction on the matrix cores cost more: the monomials fill 6 of 8 columns
// of v_mfma_f32_4x4x1 (32 steps of about 10 clocks; 169 us) or 6 of 16 of
// v_mfma_f32_16x16x4 (525 clocks), matrix and vector instructions of a SIMD do
// not overlap on this part (measured), and float32 split into three bf16 terms
// spends on the split what the faster steps save (169 us).  The colour term is
// summed by a transposing butterfly over the wave.
//
// Tiles of several waves: the waves share the staged records, and every
// wave's sums go to LDS by entry, where the entry's lane adds the waves that
// ran it in a fixed order.
//
// Measured (500k Gaussians / 512^2, tile sides 16 and 8): 197 and 151 us; the
// general kernel above took 475 us at 16 x 16, a former one with a division
// per entry and v_mfma_f32_16x16x4 for 8 x 8 tiles 189 us.  Bound by VALU
// issue.
//
// Rounding, against 64 bits (2000 Gaussians / 64^2, geometric means of 32 models,
// relative L2 in 1e-6; the kernels before / this one).  16 x 16: opacity 1.02 /
// 1.05, mean 1.47 / 1.49, scale 1.35 / 1.38, rotation 1.88 / 1.90, pose 1.49 /
// 1.34; 8 x 8: 1.03 / 1.05, 1.52 / 1.49, 1.61 / 1.38, 2.12 / 1.90, 1.43 / 1.40.  So up
// to 3 % more in some groups, most of it the recurrence's, the rest the shift of
// the moments to the mean.
template <int TW, int TH>
__global__ __launch_bounds__(TW *TH) __attribute__((amdgpu_waves_per_eu(TW * TH == 64 ? 5 : 4))) void raster_bwd_parts_kernel(RasterArgs a)
{
    constexpr int NT = TW * TH, NW = NT / kWave, GRP = 16, SWEEP = 8, PX = TW / 8;
    constexpr bool MULTI = NW > 1;
    // entries per batch: with several waves 128 (their per-entry sums fill
    // LDS: four workgroups of 16 x 16 tiles per CU)
    constexpr int BATCH = MULTI ? 128 : NT;
    static_assert(BATCH <= NT, "one lane stages an entry");
    // records by entry, s1 first: entry e's pair sits at byte 16 e (s1) and
    // 16 e + S0OFF (s0); place BATCH holds a record no pixel reaches
    constexpr uint32_t S0OFF = 16u * (BATCH + 1);
    __shared__ float4 s10[2 * (BATCH + 1)];
    float4 *const s1 = s10;
    float4 *const s0 = s10 + (BATCH + 1);
    __shared__ uint32_t se[BATCH];
    // q by (entry of the group, pixel); rows padded so that the operand reads
    // fall in distinct banks
    constexpr int QROW = kWave + 4;
    __shared__ __align__(16) float aq[NW][GRP][QROW];
    // several waves: the byte places of a wave's entries, its sums by entry of
    // the batch, and the waves that run an entry (a bit each)
    __shared__ __align__(16) uint16_t list[MULTI ? NW : 1][MULTI ? BATCH + GRP : 1];
    __shared__ float acc_e[MULTI ? NW : 1][MULTI ? BATCH : 1][7];
    __shared__ uint8_t reach[MULTI ? BATCH : 1];
    __shared__ int sh_item;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = MULTI ? __builtin_amdgcn_readfirstlane(tid / kWave) : 0;
    const int wx = 8 * (w % PX), wy = 8 * (w / PX);  // the wave's part of the tile
    const float k2s = __fmul_rn(a.o.kappa2, kExpScale);
    const float smax = a.o.sigma_max;
    const float kw = a.o.kappa * 1.001f;
    const char *const srec = reinterpret_cast<const char *>(s10);
    if (tid == 0) {
        // d^T A d = -(dx^2 + dy^2) ~ -2e36, alpha = c = 0
        s0[BATCH] = make_float4(1e18f, 1e18f, -1.0f, 0.0f);
        s1[BATCH] = make_float4(-1.0f, 0.0f, 0.0f, 0.0f);
    }
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    int iter = 0;
    for (;;) {
        const int it = next_item(a, iter, &sh_item);
        const Item I = resolve_item(a, it);
        if (I.tile < 0) break;
        const int v = view_of_tile(a.views, a.V, I.tile);
        const ViewDev &V = a.views[v];
        const int lt = I.tile - V.tile_base;
        const int ty = lt / V.ntx, tx = lt - ty * V.ntx;
        // (lane 16 q + k: pixel k, row by row, of quarter q)
        const int lx = wx + 4 * ((lane >> 4) & 1) + (lane & 3), ly = wy + 4 * (lane >> 5) + ((lane >> 2) & 3);
        const int px = tx * TW + lx, py = ty * TH + ly;
        const bool inside = px < V.W && py < V.H;
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        // the monomials' origin
        const float cx = (float)(tx * TW + wx) + 4.0f, cy = (float)(ty * TH + wy) + 4.0f;
        const size_t vbase = (size_t)v * a.n;
        float g = 0.0f, Cf = 0.0f;
        if (inside) {
            const size_t p = (size_t)V.pix_base + (size_t)py * V.W + px;
            g = a.dL_dimg[p];
            Cf = a.img_saved[p];
        }
        // (C, T) in front of the chunk: g T and g times the tail S
        const float2 pre = a.part[(size_t)it * NT + ly * TW + lx];
        float gT = g * pre.y;
        float Sg = g * (Cf - pre.x);
        const float k2e = inside ? k2s : kLaneOff;
        // Sums of the group of entries at list place qp, whose q is in aq and
        // whose colour terms are in tsum (lane 4 e + .: entry e): lane (eg, qt,
        // j) = 16 eg + 4 qt + j takes quarter qt of entry 4 eg + j, shifts its
        // moments to the mean and adds the quarters over the lanes of its row;
        // the lane with qt = j stores.
        auto finalize = [&](int qp, int cnt, float tsum) {
            const int el = qp + 4 * (lane >> 4) + (lane & 3), qt = (lane >> 2) & 3;
            const float *const qrow = &aq[w][4 * (lane >> 4) + (lane & 3)][16 * qt];
            const float4 x0 = *reinterpret_cast<const float4 *>(qrow), x1 = *reinterpret_cast<const float4 *>(qrow + 4);
            const float4 x2 = *reinterpret_cast<const float4 *>(qrow + 8), x3 = *reinterpret_cast<const float4 *>(qrow + 12);
            const int e = MULTI ? (int)(list[w][el] / 16u) : el;
            const float4 r0 = s0[e];
            // raw moments of the quarter's 4 x 4 pixels about its centre, in half
            // pixels (X, Y = -3, -1, 1, 3): per pixel row the sums of q, q X and q
            // X^2, then over the rows
            float S[4], P[4], Q[4];
            auto row = [](const float4 x, float &s_, float &p_, float &q_) {
                const float o = x.x + x.w, i = x.y + x.z;
                s_ = o + i;
                p_ = __fmaf_rn(3.0f, x.w - x.x, x.z - x.y);
                q_ = __fmaf_rn(9.0f, o, i);
            };
            row(x0, S[0], P[0], Q[0]);
            row(x1, S[1], P[1], Q[1]);
            row(x2, S[2], P[2], Q[2]);
            row(x3, S[3], P[3], Q[3]);
            const float so = S[0] + S[3], si = S[1] + S[2];
            const float M0 = so + si, M1 = (P[0] + P[3]) + (P[1] + P[2]), M2 = __fmaf_rn(3.0f, S[3] - S[0], S[2] - S[1]);
            const float M3 = (Q[0] + Q[3]) + (Q[1] + Q[2]), M4 = __fmaf_rn(3.0f, P[3] - P[0], P[2] - P[1]);
            const float M5 = __fmaf_rn(9.0f, so, si);
            // moments about the mean: with X = U + (X - U), U the mean's offset
            // from the quarter's centre
            const float ux = 2.0f * (r0.x - (cx + ((qt & 1) ? 2.0f : -2.0f)));
            const float uy = 2.0f * (r0.y - (cy + ((qt & 2) ? 2.0f : -2.0f)));
            float m[6];
            m[0] = M1 - ux * M0;
            m[1] = M2 - uy * M0;
            m[2] = M3 - ux * (2.0f * M1 - ux * M0);
            m[3] = M4 - ux * M2 - uy * M1 + ux * uy * M0;
            m[4] = M5 - uy * (2.0f * M2 - uy * M0);
            m[5] = M0;
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                m[t] += dpp_move<0x128>(m[t]);  // row_ror:8
                m[t] += dpp_move<0x124>(m[t]);  // row_ror:4
            }
            m[0] *= 0.5f;  // (from half pixels)
            m[1] *= 0.5f;
            m[2] *= 0.25f;
            m[3] *= 0.25f;
            m[4] *= 0.25f;
            if (qt == (lane & 3) && el < cnt) {
                if constexpr (MULTI) {
                    float *const o = &acc_e[w][e][0];
                    o[0] = m[0]; o[1] = m[1]; o[2] = m[2]; o[3] = m[3]; o[4] = m[4]; o[5] = m[5]; o[6] = tsum;
                } else {
                    const size_t sl = se[e];
                    if (sl < a.slot_cap) {
                        a.slot[2 * sl] = make_float4(m[0], m[1], m[2], m[3]);
                        a.slot[2 * sl + 1] = make_float4(m[4], m[5], tsum, 0.0f);
                    }
                }
            }
            wave_sync();
        };
        // The wave's cnt entries in groups of 16 (a partial group ends in the
        // record no pixel reaches).  Branch-free: lanes that miss an entry run
        // the same arithmetic with G = 0, which leaves gT and the tail as they
        // are and makes q and g s T zero.
        auto run_groups = [&](int cnt, auto clamp_c) {
            constexpr bool CLAMP = decltype(clamp_c)::value;
            for (int q0 = 0; q0 < cnt; q0 += GRP) {
                float tv[GRP];
                // the group's first entry in one vector register (opaque to
                // the compiler), so that the record reads take immediate offsets
                int qv = q0;
                asm volatile("" : "+v"(qv));
#pragma unroll
                for (int h = 0; h < GRP; h += SWEEP) {
                    float ov[SWEEP], rv[SWEEP], cv[SWEEP];
#pragma unroll
                    for (int e2 = 0; e2 < SWEEP; e2 += 2) {
                        float4 R0[2], R1[2];
                        if constexpr (MULTI) {
                            const uint32_t pl = *reinterpret_cast<const uint32_t *>(&list[w][qv + h + e2]);
                            const uint32_t pa = pl & 0xFFFFu, pb = pl >> 16;
                            R1[0] = *reinterpret_cast<const float4 *>(srec + pa);
                            R0[0] = *reinterpret_cast<const float4 *>(srec + pa + S0OFF);
                            R1[1] = *reinterpret_cast<const float4 *>(srec + pb);
                            R0[1] = *reinterpret_cast<const float4 *>(srec + pb + S0OFF);
                        } else {
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                R0[u] = s0[qv + h + e2 + u];
                                R1[u] = s1[qv + h + e2 + u];
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int e = e2 + u;
                            const float4 r0 = R0[u], r1 = R1[u];
                            const float dx = __fsub_rn(fpx, r0.x), dy = __fsub_rn(fpy, r0.y);
                            const float ex = falloff_exponent(dx, dy, r0.z, r0.w, r1.x);
                            const bool hit = ex >= k2e;
                            const float G = hit ? __builtin_amdgcn_exp2f(ex) : 0.0f;
                            float r = gT * G, t, om;
                            if constexpr (CLAMP) {
                                const float sraw = __fmul_rn(r1.y, G), s = clamp_opacity(sraw, smax);
                                om = __fsub_rn(1.0f, s);
                                t = gT * s;
                                r = (sraw > smax) ? 0.0f : r;
                            } else {
                                om = one_minus_alpha_g(r1.y, G);
                                t = r1.y * r;
                            }
                            Sg = __fmaf_rn(-r1.z, t, Sg);
                            gT = gT * om;
                            tv[h + e] = t;
                            ov[e] = om;
                            rv[e] = r;
                            cv[e] = r1.z;
                        }
                    }
                    // the colour behind the sweep (0 where nothing of g T is
                    // left: its products with gT_j vanish then)
                    const float ig = fabsf(gT) > 1e-37f ? __builtin_amdgcn_rcpf(gT) : 0.0f;
                    float Bk = Sg * ig;
                    Bk = __fmaf_rn(__fmaf_rn(-Bk, gT, Sg), ig, Bk);  // (v_rcp_f32 alone is 1 ulp off)
                    Bk = __builtin_amdgcn_fmed3f(Bk, -1e30f, 1e30f);
#pragma unroll
                    for (int e = SWEEP - 1; e >= 0; --e) {
                        const float d = cv[e] - Bk;
                        Bk = __fmaf_rn(-ov[e], d, cv[e]);
                        aq[w][h + e][lane] = rv[e] * d;
                    }
                }
                const float tsum = wave_transpose_sum16(tv);
                wave_sync();
                finalize(q0, cnt, tsum);
            }
        };
        for (uint32_t b0 = I.b; b0 < I.e; b0 += BATCH) {
            const int cnt = (int)min((uint32_t)BATCH, I.e - b0);
            __syncthreads();
            const uint32_t j = b0 + tid;
            bool over = false;  // an opacity above sigma_max / 2 in this batch
            if (tid < BATCH && j < I.e) {
                const uint32_t gid = min(a.tval[j], (uint32_t)a.n - 1u);
                const size_t idx = vbase + gid;
                float4 r0 = a.rec[4 * idx], r1 = a.rec[4 * idx + 1];
                const float4 r2 = a.rec[4 * idx + 2];
                const uint32_t place = __float_as_uint(r1.w);
                over = r1.y > 0.5f * smax;
                if constexpr (MULTI) {
                    // the parts of the tile whose pixel centres the bounding
                    // box of the cut-off ellipse reaches (as in the forward)
                    const float2 h = cutoff_box(kw, r0.z, r0.w, r1.x);
                    const float ux = r0.x - (float)(tx * TW), uy = r0.y - (float)(ty * TH);
                    uint32_t m = 0u;
#pragma unroll
                    for (int q = 0; q < NW; ++q) {
                        const float ox = 8.0f * (q % PX), oy = 8.0f * (q / PX);
                        const bool in = box_reaches(ux, h.x, ox + 0.5f, ox + 7.5f) & box_reaches(uy, h.y, oy + 0.5f, oy + 7.5f);
                        m |= in ? 1u << q : 0u;
                    }
                    reach[tid] = (uint8_t)m;
                }
                scale_conic(r0, r1);
                s0[tid] = r0;
                s1[tid] = r1;
                // the slot: the pair's first slot plus this tile's rank among
                // the pair's kept tiles (row-major in its rectangle)
                const uint32_t rx = __float_as_uint(r2.x), ry = __float_as_uint(r2.y);
                const int tx0 = rx & 0xFFFF, ty0 = rx >> 16, tx1 = ry & 0xFFFF, ty1 = ry >> 16;
                const uint32_t area = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
                const uint32_t at = (uint32_t)((ty - ty0) * (tx1 - tx0 + 1) + (tx - tx0));
                se[tid] = first_slot(a.slot_bofs, a.slot_nblk, v, (int)gid, place) +
                          kept_rank(__float_as_uint(r2.z), area, at);
            } else if (tid < BATCH) {
                // places past the batch's entries: the record no pixel reaches
                if constexpr (MULTI) {
                    reach[tid] = 0u;
                } else {
                    s0[tid] = make_float4(1e18f, 1e18f, -1.0f, 0.0f);
                    s1[tid] = make_float4(-1.0f, 0.0f, 0.0f, 0.0f);
                }
            }
            const bool clamp = __syncthreads_or(over);
            int mine = cnt;  // entries this wave runs
            if constexpr (MULTI) {
                mine = 0;
#pragma unroll
                for (int h = 0; h < BATCH / kWave; ++h) {
                    const bool in = ((uint32_t)reach[h * kWave + lane] >> w) & 1u;
                    const uint64_t bal = wave_any_mask(in);
                    if (in) {
                        const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                        list[w][mine + pos] = (uint16_t)(16u * (uint32_t)(h * kWave + lane));
                    }
                    mine += (int)__popcll(bal);
                }
                if (lane < GRP) list[w][mine + lane] = (uint16_t)(16u * BATCH);
                wave_sync();
            }
            if (mine > 0) {
                if (clamp) run_groups(mine, std::true_type{});
                else run_groups(mine, std::false_type{});
            }
            if constexpr (MULTI) {
                __syncthreads();
                if (tid < cnt) {
                    const uint32_t m = reach[tid];
                    float r[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < NW; ++q) {
                        if ((m >> q) & 1u) {
#pragma unroll
                            for (int t = 0; t < 7; ++t) r[t] += acc_e[q][tid][t];
                        }
                    }
                    const size_t sl = se[tid];
                    if (sl < a.slot_cap) {
                        a.slot[2 * sl] = make_float4(r[0], r[1], r[2], r[3]);
                        a.slot[2 * sl + 1] = make_float4(r[4], r[5], r[6], 0.0f);
                    }
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void tile_cost_kernel(const uint2 *ranges, int n_tiles, uint32_t *keys,
                                                        uint32_t *vals, uint32_t *counter)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t == 0) *counter = 0;
    if (t >= n_tiles) return;
    const uint2 r = ranges[t];
    const uint32_t len = min(r.y - r.x, 0xFFFFFFu);
    keys[t] = 0xFFFFFFu - len;  // ascending sort -> longest first
    vals[t] = (uint32_t)t;
}

// grids of blocks mapped by xcd_item
inline int round_up8(int n) { return (n + 7) / 8 * 8; }

template <int TW, int TH>
hipError_t fwd_inst(const RasterArgs &a, int pb, hipStream_t s)
{
    const int grid = a.queue_counter ? pb : round_up8(a.split ? a.max_items : a.n_tiles);
    if (grid > 0) {
        const bool cnt = a.pair_counts != nullptr;
        if (a.split && cnt) raster_fwd_kernel<TW, TH, true, true><<<grid, TW * TH, 0, s>>>(a);
        else if (a.split) raster_fwd_cells_kernel<TW, TH><<<grid, TW * TH, 0, s>>>(a);
        else if (cnt) raster_fwd_kernel<TW, TH, false, true><<<grid, TW * TH, 0, s>>>(a);
        else raster_fwd_kernel<TW, TH, false, false><<<grid, TW * TH, 0, s>>>(a);
    }
    if (a.split && a.n_tiles > 0) {
        constexpr int MTB = merge_tiles_per_block<TW, TH>();
        merge_kernel<TW, TH><<<(a.n_tiles + MTB - 1) / MTB, TW * TH * MTB, 0, s>>>(a);
    }
    return hipGetLastError();
}

template <int TW, int TH>
hipError_t bwd_inst(const RasterArgs &a, int pb, hipStream_t s)
{
    const int grid = a.queue_counter ? pb : round_up8(a.split ? a.max_items : a.n_tiles);
    if (grid > 0) {
        if (a.split) raster_bwd_parts_kernel<TW, TH><<<grid, TW * TH, 0, s>>>(a);
        else raster_bwd_kernel<TW, TH><<<grid, TW * TH, 0, s>>>(a);
    }
    return hipGetLastError();
}

}  // namespace

bool raster_tile_supported(int tw, int th)
{
    return (tw == 16 && th == 16) || (tw == 8 && th == 8) || (tw == 16 && th == 8) || (tw == 32 && th == 8);
}

hipError_t launch_raster_fwd(const RasterArgs &a, int pb, hipStream_t s)
{
    const int tw = a.o.tile_w, th = a.o.tile_h;
    if (tw == 16 && th == 16) return fwd_inst<16, 16>(a, pb, s);
    if (tw == 8 && th == 8) return fwd_inst<8, 8>(a, pb, s);
    if (tw == 16 && th == 8) return fwd_inst<16, 8>(a, pb, s);
    if (tw == 32 && th == 8) return fwd_inst<32, 8>(a, pb, s);
    return hipErrorInvalidValue;
}

hipError_t launch_raster_bwd(const RasterArgs &a, int pb, hipStream_t s)
{
    const int tw = a.o.tile_w, th = a.o.tile_h;
    if (tw == 16 && th == 16) return bwd_inst<16, 16>(a, pb, s);
    if (tw == 8 && th == 8) return bwd_inst<8, 8>(a, pb, s);
    if (tw == 16 && th == 8) return bwd_inst<16, 8>(a, pb, s);
    if (tw == 32 && th == 8) return bwd_inst<32, 8>(a, pb, s);
    return hipErrorInvalidValue;
}

hipError_t launch_tile_cost_keys(const uint2 *ranges, int n_tiles, uint32_t *keys, uint32_t *vals,
                                 uint32_t *counter, hipStream_t s)
{
    tile_cost_kernel<<<(n_tiles + 255) / 256 + (n_tiles == 0), 256, 0, s>>>(ranges, n_tiles, keys, vals, counter);
    return hipGetLastError();
}

}  // namespace ddgs
