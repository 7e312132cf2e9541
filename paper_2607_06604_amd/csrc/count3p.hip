// count3p.hip - binned triangle counts through a paged label table (paper
// Sec. 2.2 hub-and-spoke enumeration, Sec. 3.1 sorted-list intersection).
//
// The enumeration is count3.hip's: a triangle {i < j < k} (labels) is found at
// hub i, spoke j in N+(i), third vertex k in N+(i) and N+(j). What differs is
// how "is k in N+(i), and in which bin" is answered. Labels follow cells, so
// a hub's forward row lies in a few short label intervals (the forward half
// of 27 cells: five runs of cells away from the faces). The hub's row is laid
// out as bytes, one per label of the pages (2^s consecutive labels) it
// touches, holding bin + 1 or 0; a page map of 256 words per hub turns a
// page number (modulo 256: the map covers at least the hub row's label
// range) into the page's LDS address, or that of the all-zero page. A
// candidate then costs two short LDS reads and no hash, key compare or probe
// chain: neighbouring lanes read neighbouring labels, so the byte reads share
// banks' words instead of scattering.
//
// A lane takes four consecutive entries of a spoke row with one 16-byte and
// one 4-byte load; S lanes make a step of 4 S entries. The hash walk is bound
// by vector instruction issue: 54 instructions per 64 candidates (24-bit
// hash, packed-key compare, linear-probe chains, rank arithmetic) are all of
// its 6.7 ms on the 1e6-point clustered count (5.1e9 candidates, 15 bins).
// Here it is 25, and vector issue (66%), LDS (65%, half of it bank conflicts
// of the counters' atomics) and the row loads share the 5.0 ms.
//
// Weighted sums. With lo <= hi the hub's and the spoke's weight magnitudes
// and r the third, the ascending product of the three is
// fl(fl(lo min(r, hi)) max(r, hi)) (products commute), and scaling by 2^s is
// exact, so the pair is ordered once per step and a hit costs a minimum, a
// maximum and two products. Its exact term t (an integer below 2^63) goes
// into two 64-bit LDS words by float64 additions alone: u = t + 1.5 2^72
// rounds t to a multiple of 2^20, which the bits of u hold as an integer
// above those of 1.5 2^72; the remainder t - (u - 1.5 2^72), at most 2^19 in
// magnitude, is exact, and adding 1.5 2^52 + 2^19 makes the low word of the
// sum's bits that remainder plus 2^19. The first counter word adds 2^42 (the
// hit count, from bit 42) and the biased remainder, the second the bits of u;
// the flush takes the biases off again, knowing the count. Two atomics where
// separate counts and sums take three. Fewer than 2^21 (signed terms: 2^20)
// increments per counter between flushes keep every field in range; before
// the candidates walked since the last look could reach that, the fullest
// counter is read, and the counters are flushed only if it comes near.
#include <cstdio>
#include <cstdlib>

#include "count3.h"

namespace gsn {
namespace {

constexpr uint32_t kNP = 256;            // page map entries per hub
constexpr uint32_t kMinShift = 6;        // pages of 64 to 2048 labels
constexpr uint32_t kMaxShift = 11;
constexpr uint32_t kPages = 2 * kNP * kMaxGroup;   // LDS address of the first page, behind the maps
static_assert(kPages == 1u << kMaxShift, "pages are aligned to their size");
constexpr int kLane = 4;                 // entries per lane
constexpr uint32_t kWaveSteps = 128;     // steps per fill of a wavefront's table

typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_a1 __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) const u32x4_a4 gbl_u32x4;
typedef __attribute__((address_space(1))) const u32_a1 gbl_u32u;
typedef __attribute__((address_space(1))) const double gbl_f64;
typedef __attribute__((address_space(3))) const uint8_t lds_u8;

constexpr int kMuLane = 2;         // triangles a lane takes at a time
constexpr uint32_t kMuBuf = 64 * kMuLane + 256;   // triangles of a wavefront: those left over and 4 x 64 new ones

// LDS layout of one work group (byte offsets): the page maps, then the pages
// (at kPages), so that a map and a page are aligned to their sizes.
struct LayoutP {
    uint32_t cnt, lut, step, mw, mperm, mj, buf, misc, total;
};

__host__ __device__ inline LayoutP layoutp(int block, uint32_t tbytes, int nconf, int nb, bool weighted,
                                           bool anchored, int mode, bool rows, bool mu = false) {
    LayoutP L{};
    uint32_t o = lds_align(kPages + tbytes, 16);
    L.cnt = o;    o = lds_align(o + (mode == kCube ? 4 * nb * nb * nb : (weighted ? 16 : 4) * nconf), 16);
    L.lut = o;    if (mode == kLut) o = lds_align(o + 2 * nb * nb * nb, 16);
    // the cube's fold counters share the step tables (idle during a flush)
    L.step = o;   o = lds_align(o + std::max(rows ? 0u : 8 * kWaveSteps * (uint32_t)(block / 64), mode == kCube ? 4u * nconf : 0u), 16);
    L.mw = o;     if (weighted && !rows) o = lds_align(o + 8 * block, 16);
    L.mperm = o;  if (anchored && !rows) o = lds_align(o + 4 * block, 16);
    L.mj = o;     if (mu) o = lds_align(o + 16 * (block + kMaxGroup), 16);
    L.buf = o;    if (mu) o = lds_align(o + 8 * kMuBuf * (uint32_t)(block / 64), 16);
    L.misc = o;   o = lds_align(o + 384, 16);
    // lanes without a candidate read (and ignore) up to 2 (24 * 24 + 256)
    // bytes past the counter table
    L.total = std::max(o, L.lut + 2u * nb * nb * nb + 2048u);
    return L;
}

// Counters into the 64-bit results (and their sum into the triangle total);
// the caller brackets it with barriers. WT: 0 unweighted, 1 positive terms
// below 2^63, 2 any terms.
template <int BLOCK, int WT, int MODE>
__device__ void flushp(const C3Args &a, const LayoutP &L, unsigned char *sm, unsigned long long *hout,
                       unsigned long long *tout) {
    uint32_t *hist = (uint32_t *)(sm + L.cnt);
    if (MODE == kCube) {
        uint32_t *fold = (uint32_t *)(sm + L.step);
        for (int b = threadIdx.x; b < a.nconf; b += BLOCK) fold[b] = 0;
        __syncthreads();
        const int n3 = a.nb * a.nb * a.nb;
        for (int t = threadIdx.x; t < n3; t += BLOCK) {
            const uint32_t v = hist[t];
            if (v) {
                hist[t] = 0;
                atomicAdd(&fold[a.cfg3[t]], v);
            }
        }
        __syncthreads();
        hist = fold;
    }
    unsigned long long sum = 0;
    // work groups that finish together start at different counters
    const int off = (int)((blockIdx.x * 97u) % (uint32_t)a.nconf);
    for (int t = threadIdx.x; t < a.nconf; t += BLOCK) {
        const int b = t + off < a.nconf ? t + off : t + off - a.nconf;
        if (WT) {
            unsigned long long *w = (unsigned long long *)(sm + L.cnt) + b;
            const unsigned long long A = w[0], n = A >> kCntShift;
            const unsigned long long B = w[a.nconf] - n * kRoundBits;
            if (n) {
                atomicAdd(&hout[b], n);
                sum += n;
                const __int128 hi = WT == 2 ? (__int128)(long long)B : (__int128)B;
                add128_words(&a.wsum[2 * b], (hi << kLowBits) + (__int128)(A & kLowMask) - ((__int128)n << (kLowBits - 1)));
                w[0] = 0;
                w[a.nconf] = 0;
            }
        } else {
            const uint32_t v = hist[b];
            if (v) {
                atomicAdd(&hout[b], (unsigned long long)v);
                hist[b] = 0;
                sum += v;
            }
        }
    }
    sum = wave_sum64(sum);
    if ((threadIdx.x & 63) == 0 && sum && tout) atomicAdd(tout, sum);
}

// A lane's value as a wavefront-uniform one.
__device__ __forceinline__ uint64_t lane_u64(uint64_t x, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double lane_f64(double x, int lane) {
    return __longlong_as_double((long long)lane_u64((uint64_t)__double_as_longlong(x), lane));
}

// What the walk over one step table reads.
struct WalkP {
    const uint2 *step;            // steps: row offset; entries | slot << 7 | bin << 17 | hub << 25
    gbl_u32 *srow;                // spoke rows, from the group's (32-bit offsets)
    gbl_u8 *sbrow;
    const double *mw, *hw;        // weights of the spokes (by slot) and of the group's hubs
    const uint32_t *mperm, *hp;   // their original indices
    gbl_f64 *w;
    const uint32_t *perm;
    unsigned long long *wsum;
    uint32_t cnt, cntb, xbase;    // LDS addresses: counters, (offset of) their second words, bins (0, -1, 0)
    uint32_t xmul, ymul;          // address steps of the spoke's and the hub entry's bin
    uint32_t shift, pmask;        // page size
    uint32_t slog;                // lanes per step (log2)
    double wmul;
    uint32_t anchor_lo, anchor_hi;
};

// A hit's exact term into counter ad: lo, hi the pair's ordered magnitudes
// (lo times 2^s), r the third weight, ng2 the pair's sign.
template <int WT>
__device__ __forceinline__ void add_term3(const WalkP &c, bool hit, uint32_t ad, double lo, double hi, bool ng2,
                                          double r) {
    const double rk = WT == 2 ? fabs(r) : r;
    double t = __dmul_rn(__dmul_rn(lo, min_f64(rk, hi)), max_f64(rk, hi));
    bool wide = false, ng = false;
    if (WT == 2) {
        ng = ng2 ^ (r < 0.0);
        wide = !narrow_term(t);
        if (ng) t = -t;
    }
    unsigned long long lw, hw;
    term_words(t, lw, hw);
    if (WT == 2 && wide) {   // only counted here: a zero term's words
        lw = (1ull << kCntShift) | (1ull << (kLowBits - 1));
        hw = kRoundBits;
    }
    if (hit) {
        __hip_atomic_fetch_add((lds_u64 *)(size_t)ad, lw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add((lds_u64 *)(size_t)(ad + c.cntb), hw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (WT == 2 && wide) add128_words(&c.wsum[2 * ((ad - c.cnt) >> 3)], wide_term(fabs(t), ng));
    }
}

// Steps [0, nsteps) of the wavefront's table: lane group g (2^slog lanes)
// takes steps g, g + G, ... (G groups), U per pass with their row loads issued
// together; lane s of a group takes entries 4 s .. 4 s + 3 of its step (a
// row's last lane may load up to three entries past its end: row slack or the
// next row, never counted).
// Everything up to the counters' atomics runs without a branch, so that the
// LDS reads of a pass's 4 U candidates are in flight together; a lane without
// a hit reads in bounds (any label has a page, at worst the zero page; the
// counter table has slack) and drops the value.
template <int WT, bool ANCHORED, int MODE, bool WIDE>
__device__ __forceinline__ void walkp(const WalkP &c, uint32_t nsteps) {
    constexpr int U = 2;
    constexpr int N = U * kLane;
    const uint32_t sub4 = (threadIdx.x & ((1u << c.slog) - 1u)) * kLane;
    const uint32_t per = 64u >> c.slog;
    const uint32_t first = (threadIdx.x & 63u) >> c.slog;
    const uint32_t pmap = (kNP - 1) << 1, psh = c.shift - 1;
    for (uint32_t base = 0; base < nsteps; base += U * per) {
        uint32_t kk[N], zb[U], xb[U], lim[U], ptb[U], meta[U];
        uint2 e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * per + first;
            e[u] = c.step[min(i, nsteps - 1)];
            if (i >= nsteps) e[u].y = 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            meta[u] = e[u].y;
            const uint32_t cnt = e[u].y & 127u;
            lim[u] = cnt > sub4 ? cnt - sub4 : 0u;
            const uint32_t pos = e[u].x + (lim[u] ? sub4 : 0u);
            u32x4_a4 k4;
            if (WIDE) k4 = *(gbl_u32x4 *)(c.srow + pos);
            else k4 = *(gbl_u32x4 *)((gbl_u8 *)c.srow + (pos << 2));
            zb[u] = *(gbl_u32u *)(c.sbrow + pos);
#pragma unroll
            for (int v = 0; v < kLane; ++v) kk[u * kLane + v] = k4[v];
            ptb[u] = (e[u].y >> 16) & (3u << 9);
            xb[u] = c.xbase + __umul24((e[u].y >> 17) & 255u, c.xmul);
        }
        // the page of every candidate, then its byte: bin of (hub, k) + 1
        uint32_t y[N];
#pragma unroll
        for (int q = 0; q < N; ++q) y[q] = *(lds_u16 *)(size_t)(((kk[q] >> psh) & pmap) | ptb[q / kLane]);
#pragma unroll
        for (int q = 0; q < N; ++q) y[q] = *(lds_u8 *)(size_t)((kk[q] & c.pmask) | y[q]);
        bool hit[N];
        uint32_t ad[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            hit[q] = y[q] != 0u && (uint32_t)(q % kLane) < lim[q / kLane];
            const uint32_t z = (zb[q / kLane] >> (8 * (q % kLane))) & 255u;
            ad[q] = xb[q / kLane] + __umul24(y[q], c.ymul) + (MODE == kCube ? z << 2 : z << 1);
        }
        if (MODE == kLut) {
#pragma unroll
            for (int q = 0; q < N; ++q) ad[q] = *(lds_u16 *)(size_t)ad[q];
#pragma unroll
            for (int q = 0; q < N; ++q) asm volatile("" : "+v"(ad[q]));   // (keeps the reads out of the branches)
        }
        double r[N];
        if (WT) {
#pragma unroll
            for (int q = 0; q < N; ++q) r[q] = *(gbl_f64 *)((gbl_u8 *)c.w + ((hit[q] ? kk[q] : 0u) << 3));
#pragma unroll
            for (int q = 0; q < N; ++q) asm volatile("" : "+v"(r[q]));   // (as above)
        }
        if (ANCHORED) {
            uint32_t pk[N];
#pragma unroll
            for (int q = 0; q < N; ++q) pk[q] = c.perm[hit[q] ? kk[q] : 0u];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t m2 = min(c.hp[(meta[u] >> 25) & 3u], c.mperm[(meta[u] >> 7) & 1023u]);
#pragma unroll
                for (int v = 0; v < kLane; ++v) {
                    const uint32_t m = min(m2, pk[u * kLane + v]);
                    hit[u * kLane + v] = hit[u * kLane + v] && m >= c.anchor_lo && m < c.anchor_hi;
                }
            }
        }
        if (!WT) {
#pragma unroll
            for (int q = 0; q < N; ++q) {
                if (hit[q])
                    __hip_atomic_fetch_add((lds_u32 *)(size_t)ad[q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            continue;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // the pair's weights in order, once per step
            const double wh = c.hw[(meta[u] >> 25) & 3u], ws = c.mw[(meta[u] >> 7) & 1023u];
            const bool ng2 = WT == 2 && ((wh < 0.0) ^ (ws < 0.0));
            const double ah = WT == 2 ? fabs(wh) : wh, as = WT == 2 ? fabs(ws) : ws;
            const double lo = __dmul_rn(min_f64(ah, as), c.wmul), hi = max_f64(ah, as);
#pragma unroll
            for (int v = 0; v < kLane; ++v)
                add_term3<WT>(c, hit[u * kLane + v], ad[u * kLane + v], lo, hi, ng2, r[u * kLane + v]);
        }
    }
}

// What the mu counts add: hits go through a buffer in LDS, so that their
// orientation is worked out on full wavefronts.
struct WalkMu {
    uint2 *buf;                   // third vertex; slot | hub << 10 | counters' LDS address << 16
    const float4 *mj;             // by slot: the spoke's separation from its hub over rmax; its label
    const int4 *q4, *mq;          // positions, by label; of the group's hubs
    const double *X, *Y, *Z;
    const uint32_t *perm;
    double L, half;
    float scale, eps;             // a position unit and 4.5 e (see eval_mu) over rmax
    int nmu;
    uint32_t i0;                  // the group's first hub
    uint32_t held;                // hits in the buffer
};

// The buffer's last n (at most 64 kMuLane) triangles. Whatever the order of the
// vertices, their plane is the same, so |nz| / |n| is first taken in float32
// from the separations u and v of j and k from the hub in units of rmax. Their
// components are off by e, twice the rounding of positions to 2^-32 of the
// box, and by 2 r of themselves (r = 2^-24; a common factor cancels), so with
// |.|1 for the sum of magnitudes each component of n is off by less than 5 r
// |u|1 |v|1 + e (|u|1 + |v|1) + r |n|, and nmu mu by less than 2.8 nmu / |n|
// times the first two and 6 nmu r for the rest. Where it comes within 1.6
// times that of a bin edge (some 1e-5 of the triangles) the bin is worked out
// in float64 from the coordinates in original-index order, as it is defined.
// Measured on 5e5 clustered points (2e9 triangles, 5 mu bins): 17.5 ms by the
// hash kernel with every bin in float64, 10.4 so, 9.5 with the hubs' positions
// in LDS and two triangles a lane, so that their gathers overlap. Bound by
// the walk's and this code's vector instructions (55% busy) at 16 wavefronts
// a CU, which the buffers' LDS allows.
__device__ __forceinline__ void eval_mu(WalkMu &m, uint32_t n) {
    const uint32_t lane = threadIdx.x & 63u;
    wave_lds_sync();
    m.held -= n;
    uint2 t[kMuLane];
    int4 qk[kMuLane];
#pragma unroll
    for (int s = 0; s < kMuLane; ++s) {
        t[s] = m.buf[m.held + min(64 * s + lane, n - 1)];
        qk[s] = m.q4[t[s].x];
    }
    const float fmu = (float)m.nmu;
#pragma unroll
    for (int s = 0; s < kMuLane; ++s) {
        const uint32_t hk = (t[s].y >> 10) & 3u;
        const int4 qi = m.mq[hk];
        const float4 u = m.mj[t[s].y & 1023u];
        const float vx = (float)(int)((uint32_t)qk[s].x - (uint32_t)qi.x) * m.scale,
                    vy = (float)(int)((uint32_t)qk[s].y - (uint32_t)qi.y) * m.scale,
                    vz = (float)(int)((uint32_t)qk[s].z - (uint32_t)qi.z) * m.scale;
        const float nx = fmaf(u.y, vz, -(u.z * vy)), ny = fmaf(u.z, vx, -(u.x * vz)), nz = fmaf(u.x, vy, -(u.y * vx));
        const float rs = __builtin_amdgcn_rsqf(fmaf(nx, nx, fmaf(ny, ny, nz * nz)));
        const float r = fabsf(nz) * rs * fmu, edge = rintf(r);
        const float ua = fabsf(u.x) + fabsf(u.y) + fabsf(u.z), va = fabsf(vx) + fabsf(vy) + fabsf(vz);
        const float margin = fmu * fmaf(rs, fmaf(24.0f * 0x1p-24f * ua, va, m.eps * (ua + va)), 10.0f * 0x1p-24f);
        uint32_t b = min((uint32_t)r, (uint32_t)m.nmu - 1u);
        const bool sure = margin < 0.25f && (fabsf(r - edge) > margin || edge < 0.5f || edge > fmu - 0.5f);
        if (64 * s + lane < n) {
            if (!sure) {
                const uint32_t i = m.i0 + hk, j = __float_as_uint(u.w), k = t[s].x;
                P3x v0{m.X[i], m.Y[i], m.Z[i], m.perm[i]}, v1{m.X[j], m.Y[j], m.Z[j], m.perm[j]},
                    v2{m.X[k], m.Y[k], m.Z[k], m.perm[k]};
                order3(v0, v1, v2);
                b = (uint32_t)mu_bin(min_image(v0.x, v1.x, m.L, m.half), min_image(v0.y, v1.y, m.L, m.half),
                                     min_image(v0.z, v1.z, m.L, m.half), min_image(v0.x, v2.x, m.L, m.half),
                                     min_image(v0.y, v2.y, m.L, m.half), min_image(v0.z, v2.z, m.L, m.half), m.nmu);
            }
            __hip_atomic_fetch_add((lds_u32 *)(size_t)((t[s].y >> 16) + 4 * b), 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    wave_lds_sync();
}

// walkp for mu counts (one step per lane group and pass).
__device__ __forceinline__ void walkp_mu(const WalkP &c, uint32_t nsteps, WalkMu &m) {
    const uint32_t sub4 = (threadIdx.x & ((1u << c.slog) - 1u)) * kLane;
    const uint32_t per = 64u >> c.slog;
    const uint32_t first = (threadIdx.x & 63u) >> c.slog;
    const uint32_t pmap = (kNP - 1) << 1, psh = c.shift - 1;
    auto load = [&](uint32_t base, uint32_t &meta, u32x4_a4 &k4, uint32_t &zb, uint32_t &lim) {
        const uint32_t i = base + first;
        const uint2 e = c.step[min(i, nsteps - 1)];
        const uint32_t cnt = i < nsteps ? e.y & 127u : 0u;
        meta = e.y;
        lim = cnt > sub4 ? cnt - sub4 : 0u;
        const uint32_t pos = e.x + (lim ? sub4 : 0u);
        k4 = *(gbl_u32x4 *)((gbl_u8 *)c.srow + (pos << 2));
        zb = *(gbl_u32u *)(c.sbrow + pos);
    };
    uint32_t meta, zb, lim;
    u32x4_a4 k4;
    load(0, meta, k4, zb, lim);
    for (uint32_t base = 0; base < nsteps; base += per) {
        uint32_t meta2, zb2, lim2;
        u32x4_a4 k42;
        load(base + per, meta2, k42, zb2, lim2);   // the next pass's rows
        const uint32_t ptb = (meta >> 16) & (3u << 9);
        const uint32_t xb = c.xbase + __umul24((meta >> 17) & 255u, c.xmul);
        const uint32_t sl = ((meta >> 7) & 1023u) | ((meta >> 25) & 3u) << 10;
        uint32_t y[kLane], ad[kLane];
#pragma unroll
        for (int v = 0; v < kLane; ++v) y[v] = *(lds_u16 *)(size_t)(((k4[v] >> psh) & pmap) | ptb);
#pragma unroll
        for (int v = 0; v < kLane; ++v) y[v] = *(lds_u8 *)(size_t)((k4[v] & c.pmask) | y[v]);
#pragma unroll
        for (int v = 0; v < kLane; ++v)
            ad[v] = *(lds_u16 *)(size_t)(xb + __umul24(y[v], c.ymul) + (((zb >> (8 * v)) & 255u) << 1));
#pragma unroll
        for (int v = 0; v < kLane; ++v) {
            const bool hit = y[v] != 0u && (uint32_t)v < lim;
            const uint64_t bal = __ballot(hit);
            if (hit) m.buf[m.held + lanes_below(bal)] = make_uint2(k4[v], sl | ad[v] << 16);
            m.held += (uint32_t)__popcll(bal);
        }
        while (m.held >= 64 * kMuLane) eval_mu(m, 64 * kMuLane);
        meta = meta2;
        zb = zb2;
        lim = lim2;
        k4 = k42;
    }
}

// Long rows: the whole wavefront takes one spoke row, 64 consecutive entries
// at a time, U blocks per pass; what belongs to the spoke sits in scalar
// registers. Consecutive lanes hold consecutive labels, so a block's byte
// reads touch a few neighbouring words. RANK (weighted or anchored counts):
// a page holds 16-bit entries, bin + 1 and the entry's rank among its row's
// entries in the page, and the map adds the rank of the page's first entry;
// the third vertex's weight (and original index) is then gathered from the
// group's packed copy of the hub row, where a block's hits lie side by side:
// from the label-ordered array a hit costs nearly a cache access of its own,
// which bounded the walk (one access per cycle and compute unit, 36 per
// block of candidates). The next pass's rows load behind this one's gathers.
// Measured on the 2.5e5-point BAO-scale weighted count (5.9e11 candidates,
// 1776 entries a row): 1216 ms by the hash walk, 747 by lane steps, 824 by
// this walk with label-ordered weights, 678 with hubs taken in label order
// over the whole device (the rows of one neighbourhood then stay in the
// memory-side cache; spread over eight slices they came from HBM at its 4
// TB/s), 637 with the loads ahead, 595 with constants held in vector
// registers: vector issue is 83% busy. FULL: every block is whole.
constexpr int kBlocks = 4;   // blocks per pass

// The row part of one pass: where it lies, and what its spoke brings.
struct RowPass {
    const gbl_u32 *row;
    const gbl_u8 *brow;
    uint32_t skip, left;   // entries before the row's first; skip + entries of the row from here on
};

// (a lane outside the row loads a neighbouring row or the slack)
__device__ __forceinline__ void load_blocks(const RowPass &p, uint32_t *kk, uint32_t *z) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int u = 0; u < kBlocks; ++u) {
        const uint32_t o = 64u * u < p.left ? 64u * u : 0u;
        kk[u] = (p.row + o)[lane];
        z[u] = (p.brow + o)[lane];
    }
}

template <int WT, bool ANCHORED, int MODE, bool FULL, class Next>
__device__ __forceinline__ void walk_blocks(const WalkP &c, const RowPass &p, const uint32_t *kk, const uint32_t *z,
                                            uint32_t ptb, uint32_t xb, double lo, double hi, bool ng2, uint32_t m2,
                                            Next &&next) {
    constexpr bool RANK = WT != 0 || ANCHORED;
    constexpr int U = kBlocks;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t pmap = (kNP - 1) << (RANK ? 2 : 1), psh = c.shift - (RANK ? 2 : 1);
    uint32_t pg[U], t[U], ad[U];
    bool hit[U];
    double r[U];
    uint32_t ym = c.ymul;
    asm("" : "+v"(ym));   // in vector registers: an instruction takes one scalar operand
    if (WT) asm("" : "+v"(hi));
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (FULL || 64u * u < p.left) {
            if (RANK) pg[u] = *(lds_u32 *)(size_t)((kk[u] >> psh) & pmap);
            else pg[u] = *(lds_u16 *)(size_t)(((kk[u] >> psh) & pmap) | ptb);
        }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (FULL || 64u * u < p.left) {
            if (RANK) t[u] = *(lds_u16 *)(size_t)((pg[u] & 0xFFFFu) + ((kk[u] & c.pmask) << 1));
            else t[u] = *(lds_u8 *)(size_t)((kk[u] & c.pmask) | pg[u]);
        }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        hit[u] = false;
        ad[u] = 0;
        if (FULL || 64u * u < p.left) {
            hit[u] = t[u] != 0u && (FULL ? u > 0 || lane >= p.skip : 64u * u + lane - p.skip < p.left - p.skip);
            const uint32_t y = RANK ? t[u] & 31u : t[u];
            ad[u] = (__umul24(y, ym) + xb) + (MODE == kCube ? z[u] << 2 : z[u] << 1);
            if (MODE == kLut) ad[u] = *(lds_u16 *)(size_t)ad[u];
            if (RANK) t[u] = (pg[u] >> 16) + (t[u] >> 5);   // position in the hub's row
        }
    }
    if (WT) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            asm("" : "=v"(r[u]));   // (any value: only hits use it)
            if (hit[u]) r[u] = *(gbl_f64 *)((gbl_u8 *)c.w + (t[u] << 3));
        }
    }
    uint32_t pk[U];
    if (ANCHORED) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pk[u] = 0;
            if (hit[u]) pk[u] = *(gbl_u32 *)((gbl_u8 *)c.perm + (t[u] << 2));
        }
    }
    next();   // the next pass's row loads, behind this one's gathers
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (FULL || 64u * u < p.left) {
            if (ANCHORED) {
                const uint32_t m = min(m2, pk[u]);
                hit[u] = hit[u] && m >= c.anchor_lo && m < c.anchor_hi;
            }
            if (WT) {
                add_term3<WT>(c, hit[u], ad[u], lo, hi, ng2, r[u]);
            } else {
                if (hit[u])
                    __hip_atomic_fetch_add((lds_u32 *)(size_t)ad[u], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
}

// A group of consecutive hubs whose rows lie in the table together.
struct GroupP {
    uint32_t hub, K;              // first hub (kEmptyKey: no more), hubs
    int g;                        // batched launch: catalogue
    uint32_t shift;               // page size (log2)
    uint64_t rb[kMaxGroup + 1];   // row bounds
    uint32_t first[kMaxGroup], last[kMaxGroup];   // a row's smallest and largest label
    double hw[kMaxGroup];         // weights, original indices, anchor marks
    uint32_t hp[kMaxGroup];
    uint8_t mk[kMaxGroup];
};
// Shared state of the work group (LDS).
struct SharedP {
    GroupP G[2];                  // the current group and the next
    HubCursor cursor, tcursor;    // claimed hubs and tiles
    unsigned long long acc;       // bound on the increments of any counter since the last flush
    uint32_t pages, next;         // pages taken; smallest label beyond the round
    uint32_t chunk, done;         // spoke chunks claimed; wavefronts out of chunks
    uint32_t need, top;           // a flush is due; the fullest counter
    uint32_t flushes, put_off;    // flushes in mid-count; those the fullest counter put off
};
static_assert(sizeof(SharedP) <= 384, "LayoutP::misc");

// Inclusive sum over the wavefront.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
#define GS_DPP_ADD(ctrl, rows) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false)
    GS_DPP_ADD(0x111, 0xf);   // row_shr:1, 2, 4, 8
    GS_DPP_ADD(0x112, 0xf);
    GS_DPP_ADD(0x114, 0xf);
    GS_DPP_ADD(0x118, 0xf);
    GS_DPP_ADD(0x142, 0xa);   // row_bcast:15, 31
    GS_DPP_ADD(0x143, 0xc);
#undef GS_DPP_ADD
    return x;
}

// One wavefront claims the next hubs and forms their group: up to kmax
// consecutive hubs whose rows (contiguous in the CSR) hold at most group_cap
// entries, and the page size with which 256 pages cover every row's labels.
template <int WT, bool ANCHORED, bool BATCH>
__device__ __forceinline__ void form_group(const C3Args &a, SharedP &S, GroupP &G, uint32_t smax) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t v0 = kEmptyKey, avail = 0;
    bool have = false;
    if (lane == 0) {
        if (a.inorder) {
            const uint32_t v = atomicAdd(a.queue, 1u), h1 = BATCH ? a.nvirt : a.h1 - a.h0;
            have = v < h1;
            S.cursor.cur = (BATCH ? 0u : a.h0) + v;
            S.cursor.end = S.cursor.cur + 1;
        } else if (a.tiles) {
            // the queues hand out tiles; a tile's hubs go in order
            have = S.cursor.cur < S.cursor.end;
            while (!have) {
                const uint32_t t = next_hub_in(a.queue, 0, a.ntiles, gridDim.x, S.tcursor, 1);
                if (t == kEmptyKey) break;
                S.cursor.cur = a.tiles[t];
                S.cursor.end = a.tiles[t + 1];
                have = S.cursor.cur < S.cursor.end;
            }
        } else {
            have = BATCH ? next_hub_run(a.queue, 0, a.nvirt, gridDim.x, S.cursor)
                         : next_hub_run(a.queue, a.h0, a.h1, gridDim.x, S.cursor);
        }
    }
    if (have) {
        v0 = S.cursor.cur;
        avail = S.cursor.end - S.cursor.cur;
    }
    v0 = __builtin_amdgcn_readfirstlane(v0);
    avail = __builtin_amdgcn_readfirstlane(avail);
    if (v0 == kEmptyKey) {
        if (lane == 0) G.hub = kEmptyKey;
        return;
    }
    const uint64_t *grp = a.rp;
    const uint32_t *gcol = a.hcol;
    uint64_t gbase = a.hbase;
    uint32_t i0 = v0;
    int g = 0;
    if (BATCH) {
        // a group stays inside one catalogue
        g = graph_of(a.gd, a.ngraph, v0);
        i0 = (uint32_t)(v0 - a.gd[g].v0);
        grp = a.gd[g].rp;
        gcol = a.gd[g].col;
        gbase = 0;
        avail = min(avail, a.gd[g].n - i0);
    }
    const uint32_t na = min(avail, (uint32_t)a.kmax);
    const uint64_t r = lane <= na ? grp[i0 + lane] : 0;
    const uint64_t rn = __shfl_down(r, 1, 64);
    const uint64_t span = uniform64(r);
    const bool fits = lane < na && (lane == 0 || rn - span <= a.group_cap);
    uint32_t K = max(1u, (uint32_t)__popcll(__ballot(fits)));
    uint32_t lo = 0, hi = 0;
    if (lane < K && rn > r) {
        lo = gcol[r - gbase];
        hi = gcol[rn - 1 - gbase];
    }
    uint32_t sh = kMinShift;
    while ((hi >> sh) - (lo >> sh) >= kNP) ++sh;
    uint32_t shm = sh;
#pragma unroll
    for (int o = 1; o < kMaxGroup; o <<= 1) shm = max(shm, (uint32_t)__shfl_xor(shm, o, 64));
    shm = __builtin_amdgcn_readfirstlane(shm);
    if (shm > smax) {   // alone, and in rounds of labels if even that does not cover its row
        K = 1;
        shm = min(smax, (uint32_t)__builtin_amdgcn_readfirstlane(sh));
    }
    if (lane <= K) G.rb[lane] = r;
    if (lane < K) {
        G.first[lane] = lo;
        G.last[lane] = hi;
        if (ANCHORED) G.hp[lane] = a.perm[i0 + lane];
        if (ANCHORED) G.mk[lane] = a.mark ? a.mark[i0 + lane] : 1;
        if (WT) G.hw[lane] = a.w[i0 + lane];
    }
    if (lane == 0) {
        G.hub = i0;
        G.K = K;
        G.g = g;
        G.shift = shm;
        S.cursor.cur += K;
    }
}

// The wavefronts of a work group share the hub table and the counters and are
// otherwise on their own: each claims chunks of spokes, cuts their rows into
// steps in a table of its own and walks them, so that a group of hubs costs
// four barriers however many steps it has. The first wavefront out of chunks
// forms the next group while the others finish.
template <int BLOCK, int WT, bool ANCHORED, bool BATCH, int MODE, bool WIDE, bool LONG, bool MU = false>
__global__ __launch_bounds__(BLOCK, (WT && BLOCK < 768) || MU ? 4 : 6) void k_count3p(C3Args a) {
    extern __shared__ __align__(16) unsigned char sm[];
    const LayoutP L = layoutp(BLOCK, a.tbytes, a.nconf, a.nb, WT != 0, ANCHORED, MODE, LONG, MU);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    if (lds_addr(sm) != 0) {   // map and page addresses start at LDS address 0
        if (tid == 0) atomicOr(a.err, 2u);
        return;
    }
    // offsets of spoke rows from the group's first: 64 bits cost a long row
    // nothing (2.5e5 points, BAO scale: 592 ms, as before), and its graph may
    // hold 2^32 entries (2e6 points, 7.2e9 entries: 4.81 s, against 9.21 by
    // the hash table, which took such graphs)
    using RowOfs = typename std::conditional<LONG, uint64_t, uint32_t>::type;
    constexpr bool RANK = LONG && (WT != 0 || ANCHORED);   // 16-bit page entries with ranks; lone hubs
    uint16_t *pt = (uint16_t *)sm;
    uint32_t *ptk = (uint32_t *)sm;   // RANK: page address | row position of its first entry << 16
    double *wrow = RANK && WT ? a.wrow + (size_t)blockIdx.x * a.maxdeg : nullptr;
    uint32_t *prow = RANK && ANCHORED ? a.prow + (size_t)blockIdx.x * a.maxdeg : nullptr;
    uint2 *step = (uint2 *)(sm + L.step) + wid * kWaveSteps;
    double *mw = (double *)(sm + L.mw);
    uint32_t *mperm = (uint32_t *)(sm + L.mperm);
    SharedP &S = *(SharedP *)(sm + L.misc);
    const uint32_t selog = (uint32_t)a.glog, SE = 1u << selog;
    const uint32_t smax = min(kMaxShift, 31u - (uint32_t)__clz(a.tbytes / (RANK ? 8 : 4)));   // at least four pages

    for (uint32_t t = tid; t < (L.lut - kPages) / 4; t += BLOCK) ((uint32_t *)(sm + kPages))[t] = 0;   // pages, counters
    if (MODE == kLut)
        for (int t = tid; t < a.nb * a.nb * a.nb; t += BLOCK)
            ((uint16_t *)(sm + L.lut))[t] = (uint16_t)(L.cnt + a.cfg3[t] * (WT ? 8u : MU ? 4u * a.nmu : 4u));
    if (tid == 0) {
        S.cursor = HubCursor();
        S.tcursor = HubCursor();
        S.acc = 0;
        S.need = 0;
        S.top = 0;
        S.flushes = 0;
        S.put_off = 0;
    }
    wave_lds_sync();
    if (wid == 0) form_group<WT, ANCHORED, BATCH>(a, S, S.G[0], smax);

    uint64_t probed = 0;  // candidates of this lane's spokes
    int cur = -1;
    const uint64_t *rp = a.rp;
    const uint32_t *hcol = a.hcol, *scol = a.scol;
    const uint8_t *hbinp = a.hbin, *sbinp = a.sbin;
    uint64_t hbase = a.hbase, sbase = a.sbase;
    uint32_t s0 = a.s0, s1 = a.s1;
    unsigned long long *hout = a.hist, *tout = a.ntri;

    WalkP c;
    c.step = step; c.mw = mw; c.mperm = mperm; c.w = (gbl_f64 *)(RANK ? wrow : a.w); c.perm = RANK ? prow : a.perm;
    c.wsum = a.wsum; c.slog = selog - 2; c.wmul = a.wmul;
    c.cnt = L.cnt; c.cntb = 8 * a.nconf;
    c.ymul = (MODE == kCube ? 4 : 2) * a.nb; c.xmul = c.ymul * a.nb;
    c.xbase = (MODE == kCube ? L.cnt : L.lut) - c.ymul;
    c.anchor_lo = a.anchor_lo; c.anchor_hi = a.anchor_hi;
    WalkMu m;
    float4 *mj = (float4 *)(sm + L.mj);
    if (MU)
        m = WalkMu{(uint2 *)(sm + L.buf) + wid * kMuBuf, mj, a.q4, (const int4 *)(mj + BLOCK), a.X, a.Y, a.Z, a.perm, a.L, a.half, a.qscale, 4.5f * a.qscale, a.nmu, 0, 0};
    uint32_t dirty = 0;   // page bytes in use

    for (uint32_t gi = 0;; gi ^= 1u) {
        __syncthreads();   // the group is formed, the last one walked
        const GroupP &G = S.G[gi];
        const uint32_t i0 = __builtin_amdgcn_readfirstlane(G.hub);
        if (i0 == kEmptyKey) break;
        const uint32_t K = __builtin_amdgcn_readfirstlane(G.K);
        if (BATCH) {
            const int g = __builtin_amdgcn_readfirstlane(G.g);
            if (g != cur) {
                // a new catalogue: hand the previous one its counts first
                if (cur >= 0) {
                    flushp<BLOCK, WT, MODE>(a, L, sm, hout, tout);
                    if (tid == 0) S.acc = 0;
                    __syncthreads();
                }
                cur = g;
                const GDesc &D = a.gd[g];
                rp = D.rp;
                hcol = scol = D.col;
                hbinp = sbinp = D.bin;
                hbase = sbase = 0;
                s0 = 0;
                s1 = D.n;
                hout = D.hist;
                tout = D.ntri;
            }
        }
        const uint32_t shift = __builtin_amdgcn_readfirstlane(G.shift), pmask = (1u << shift) - 1u;
        const uint32_t cap = (a.tbytes >> (shift + RANK)) - 1u;   // pages beside the zero page
        c.shift = shift;
        c.pmask = pmask;
        c.hw = G.hw;
        c.hp = G.hp;
        if (MU) {
            m.i0 = i0;
            if (tid < K) ((int4 *)(mj + BLOCK))[tid] = a.q4[i0 + tid];
        }
        // spokes of this tile have labels >= jlo; their rows are addressed
        // from rb = rp[jlo]
        const uint32_t jlo = max(i0 + 1, s0);
        const uint64_t rb = jlo >= s1 ? 0 : uniform64(jlo == i0 + 1 ? G.rb[1] : rp[jlo]);
        c.srow = (gbl_u32 *)uniform64((uint64_t)(scol + (rb - sbase)));
        c.sbrow = (gbl_u8 *)uniform64((uint64_t)(sbinp + (rb - sbase)));

        const uint32_t al = (uint32_t)(rb - sbase) & 15u;
        // the group's hubs [hb, hb + ks) together (all of them, unless their
        // pages do not fit)
        uint32_t ks = K;
        bool formed = false;   // the next group
        for (uint32_t hb = 0; hb < K;) {
            ks = min(ks, K - hb);
            const uint64_t rb0 = uniform64(G.rb[hb]);
            const uint32_t D = (uint32_t)(uniform64(G.rb[hb + ks]) - rb0);
            uint32_t ofs1 = kEmptyKey, ofs2 = kEmptyKey, ofs3 = kEmptyKey;
            if (ks > 1) ofs1 = (uint32_t)(uniform64(G.rb[hb + 1]) - rb0);
            if (ks > 2) ofs2 = (uint32_t)(uniform64(G.rb[hb + 2]) - rb0);
            if (ks > 3) ofs3 = (uint32_t)(uniform64(G.rb[hb + 3]) - rb0);
            const uint64_t beg = rb0 - hbase;
            const bool idle = D < 2 || jlo >= s1;
            const uint32_t csl = D > (uint32_t)BLOCK * 2 || a.maxdeg > 4096 ? 4 : 6;   // spokes per chunk (log2)
            const uint32_t nch = idle ? 0u : (D + (1u << csl) - 1) >> csl;
            uint32_t klo = __builtin_amdgcn_readfirstlane(G.first[hb]);   // a round's smallest label
            bool later = false, again = false;   // a round after the first (one hub); fewer hubs to take
            while (true) {
                // 1. clear the pages in use and the maps (every page the zero page)
                for (uint32_t t = tid; t < (dirty + 15) / 16; t += BLOCK) ((uint4 *)(sm + kPages))[t] = make_uint4(0, 0, 0, 0);
                for (uint32_t t = tid; t < kPages / 16; t += BLOCK) {
                    const uint32_t z = RANK ? kPages : kPages | (kPages << 16);
                    ((uint4 *)sm)[t] = make_uint4(z, z, z, z);
                }
                if (tid == 0) {
                    S.pages = 0;
                    S.next = kEmptyKey;
                    S.chunk = 0;
                    S.done = 0;
                }
                __syncthreads();
                // a round of a lone hub takes the labels from klo that one
                // table holds whatever pages they touch; else all of them
                uint32_t khi = kEmptyKey;
                if (later || (ks == 1 && (G.last[hb] >> shift) - (klo >> shift) >= kNP)) {
                    const uint64_t end = (uint64_t)((klo >> shift) + min(cap, kNP)) << shift;
                    if (end <= __builtin_amdgcn_readfirstlane(G.last[hb])) khi = (uint32_t)end - 1;
                }
                // 2. the first entry of a row in a page takes the page
                for (uint32_t e0 = 0; e0 < D; e0 += BLOCK) {
                    const uint32_t e = e0 + tid;
                    bool lead = false;
                    uint32_t k = 0, hk = 0;
                    if (e < D) {
                        k = hcol[beg + e];
                        hk = (e >= ofs1) + (e >= ofs2) + (e >= ofs3);
                        const uint32_t beg_e = hk == 0 ? 0u : hk == 1 ? ofs1 : hk == 2 ? ofs2 : ofs3;
                        lead = e == beg_e || (hcol[beg + e - 1] >> shift) != (k >> shift);
                        if (later && k >= klo && e > 0 && hcol[beg + e - 1] < klo) lead = true;
                        lead = lead && k >= klo * (uint32_t)(ks == 1) && k <= khi;
                    }
                    const uint64_t bal = __ballot(lead);
                    uint32_t at = 0;
                    if (lane == 0 && bal) at = atomicAdd(&S.pages, (uint32_t)__popcll(bal));
                    at = __builtin_amdgcn_readfirstlane(at) + lanes_below(bal);
                    if (lead && at < cap) {
                        const uint32_t p = (k >> shift) & (kNP - 1);
                        if (RANK) ptk[p] = (kPages + ((at + 1) << (shift + 1))) | (e << 16);
                        else pt[(hb + hk) * kNP + p] = (uint16_t)(kPages + ((at + 1) << shift));
                    }
                }
                __syncthreads();
                const uint32_t pages = __builtin_amdgcn_readfirstlane(S.pages);
                dirty = (min(pages, cap) + 1u) << (shift + RANK);
                if (pages > cap) {
                    // too many pages: half the hubs, or one in rounds
                    if (ks > 1) {
                        ks >>= 1;
                        again = true;
                        break;
                    }
                    later = true;
                    __syncthreads();
                    continue;
                }
                // 3. the rows' bytes
                for (uint32_t e = tid; e < D; e += BLOCK) {
                    const uint32_t k = hcol[beg + e];
                    const uint32_t yb = hbinp[beg + e];
                    const uint32_t hk = (e >= ofs1) + (e >= ofs2) + (e >= ofs3);
                    if (ks > 1 || (k >= klo && k <= khi)) {
                        const uint32_t p = (k >> shift) & (kNP - 1);
                        if (RANK) {
                            const uint32_t pg = ptk[p];
                            *(uint16_t *)(sm + (pg & 0xFFFFu) + 2 * (k & pmask)) = (uint16_t)((yb + 1u) | (e - (pg >> 16)) << 5);
                            if (WT) wrow[e] = a.w[k];
                            if (ANCHORED) prow[e] = a.perm[k];
                        } else {
                            sm[pt[(hb + hk) * kNP + p] | (k & pmask)] = (uint8_t)(yb + 1u);
                        }
                    } else if (k > khi) {
                        atomicMin(&S.next, k);
                    }
                }
                __syncthreads();
                // 4. the spokes, in chunks claimed by the wavefronts
                uint32_t pend = kEmptyKey;   // a chunk put off by a flush
                while (true) {
                    while (true) {
                        uint32_t ch = pend;
                        if (ch == kEmptyKey) {
                            if (lane == 0) ch = atomicAdd(&S.chunk, 1u);
                            ch = __builtin_amdgcn_readfirstlane(ch);
                        }
                        pend = kEmptyKey;
                        if (ch >= nch) break;
                        const uint32_t sidx = (ch << csl) + lane;
                        const uint32_t hk = (sidx >= ofs1) + (sidx >= ofs2) + (sidx >= ofs3);
                        const uint32_t next = hk == 0 ? ofs1 : hk == 1 ? ofs2 : hk == 2 ? ofs3 : kEmptyKey;
                        RowOfs st = 0;
                        uint32_t len = 0, x = 0, pj = 0;
                        double ws = 0.0;
                        // (the last entry of a row is no spoke)
                        if (lane < (1u << csl) && sidx + 1 < D && sidx + 1 != next) {
                            const uint32_t j = hcol[beg + sidx];
                            if (j >= s0 && j < s1 && j < khi) {
                                const uint64_t rk = rp[j];
                                x = hbinp[beg + sidx];
                                st = (RowOfs)(rk - rb);
                                len = (uint32_t)(rp[j + 1] - rk);
                                if (MU) {
                                    const int4 qj = a.q4[j], qi = m.mq[hb + hk];
                                    mj[tid] = make_float4((float)(int)((uint32_t)qj.x - (uint32_t)qi.x) * a.qscale,
                                                          (float)(int)((uint32_t)qj.y - (uint32_t)qi.y) * a.qscale,
                                                          (float)(int)((uint32_t)qj.z - (uint32_t)qi.z) * a.qscale,
                                                          __uint_as_float(j));
                                }
                                if (WT) {
                                    ws = a.w[j];
                                    if (!LONG) mw[tid] = ws;
                                }
                                if (ANCHORED) {
                                    pj = a.perm[j];
                                    if (!LONG) mperm[tid] = pj;
                                    // the smallest of three indices is at most that of the pair
                                    if (!G.mk[hb + hk] || min(G.hp[hb + hk], pj) < a.anchor_lo) len = 0;
                                }
                            }
                        }
                        if (len) {
                            // entries above the largest label of the hub's
                            // row (or outside the round) cannot match
                            const uint32_t top = min(G.last[hb + hk], khi);
                            if (c.srow[st + len - 1] > top) {
                                uint32_t lo = 0, hi = len - 1;  // first entry > top
                                while (lo < hi) {
                                    const uint32_t mid = (lo + hi) >> 1;
                                    if (c.srow[st + mid] <= top) lo = mid + 1;
                                    else hi = mid;
                                }
                                len = lo;
                            }
                            if (later && len) {
                                uint32_t lo = 0, hi = len;  // first entry >= klo
                                while (lo < hi) {
                                    const uint32_t mid = (lo + hi) >> 1;
                                    if (c.srow[st + mid] < klo) lo = mid + 1;
                                    else hi = mid;
                                }
                                st += lo;
                                len -= lo;
                            }
                        }
                        const uint32_t ns = (len + SE - 1) >> selog;
                        const uint32_t t1 = wave_incl_scan(ns), t0 = t1 - ns;
                        const uint32_t T = __builtin_amdgcn_readlane(t1, 63);
                        if (T == 0) continue;
                        // room for this many increments of any counter
                        unsigned long long before = 0;
                        if (lane == 0) before = atomicAdd(&S.acc, (unsigned long long)T << selog);
                        if (uniform64(before) + ((uint64_t)T << selog) >= a.flush_limit) {
                            if (lane == 0) {
                                atomicAdd(&S.acc, ~((unsigned long long)T << selog) + 1ull);
                                S.need = 1;
                            }
                            pend = ch;
                            break;
                        }
                        probed += len;
                        if (LONG) {
                            double lo = 0, hi = 0;   // the pair's weights in order (lo times 2^s)
                            uint32_t m2 = 0;
                            bool ng2 = false;
                            if (WT && len) {
                                const double wh = G.hw[hb + hk];
                                ng2 = (wh < 0.0) ^ (ws < 0.0);
                                lo = __dmul_rn(min_f64(fabs(wh), fabs(ws)), c.wmul);
                                hi = max_f64(fabs(wh), fabs(ws));
                            }
                            if (ANCHORED && len) m2 = min(G.hp[hb + hk], pj);
                            uint64_t live = __ballot(len != 0);
                            const uint64_t negs = __ballot(ng2);
                            int sl = __builtin_ctzll(live);
                            live &= live - 1;
                            // a spoke's row, from a 64-byte boundary of the labels
                            auto start = [&](int l) {
                                const uint64_t b = lane_u64(st, l);
                                const uint32_t skip = (al + (uint32_t)b) & 15u;
                                return RowPass{c.srow + b - skip, c.sbrow + b - skip, skip,
                                               skip + __builtin_amdgcn_readlane(len, l)};
                            };
                            RowPass p = start(sl);
                            uint32_t kk[kBlocks], z[kBlocks];
                            load_blocks(p, kk, z);
                            while (true) {
                                const uint32_t sx = __builtin_amdgcn_readlane(x | hk << 8, sl);
                                const double slo = lane_f64(lo, sl), shi = lane_f64(hi, sl);
                                const uint32_t sm2 = ANCHORED ? __builtin_amdgcn_readlane(m2, sl) : 0u;
                                const uint32_t ptb = (hb + (sx >> 8)) << 9, xb = c.xbase + (sx & 255u) * c.xmul;
                                const bool sng = (negs >> sl) & 1;
                                bool row_done = false;
                                while (!row_done) {
                                    // the pass after this one: further along the row, or the next spoke's
                                    RowPass q = p;
                                    row_done = p.left <= 64u * kBlocks;
                                    if (!row_done) {
                                        q.row += 64 * kBlocks;
                                        q.brow += 64 * kBlocks;
                                        q.left -= 64 * kBlocks;
                                        q.skip = 0;
                                    } else if (live) {
                                        q = start(__builtin_ctzll(live));
                                    }
                                    uint32_t nk[kBlocks], nz[kBlocks];
                                    auto next = [&]() { load_blocks(q, nk, nz); };
                                    if (p.left >= 64u * kBlocks)
                                        walk_blocks<WT, ANCHORED, MODE, true>(c, p, kk, z, ptb, xb, slo, shi, sng, sm2, next);
                                    else
                                        walk_blocks<WT, ANCHORED, MODE, false>(c, p, kk, z, ptb, xb, slo, shi, sng, sm2, next);
#pragma unroll
                                    for (int u = 0; u < kBlocks; ++u) {
                                        kk[u] = nk[u];
                                        z[u] = nz[u];
                                    }
                                    p = q;
                                }
                                if (!live) break;
                                sl = __builtin_ctzll(live);
                                live &= live - 1;
                            }
                            continue;
                        }
                        const uint32_t ey = (tid << 7) | (x << 17) | ((hb + hk) << 25);
                        for (uint32_t w0 = 0; w0 < T; w0 += kWaveSteps) {
                            const uint32_t lo = max(t0, w0), hi = min(t1, w0 + kWaveSteps);
                            for (uint32_t i = lo; i < hi; ++i) {
                                const uint32_t off = (i - t0) << selog;
                                step[i - w0] = make_uint2((uint32_t)st + off, ey | min(SE, len - off));
                            }
                            wave_lds_sync();
                            if (MU) walkp_mu(c, min(kWaveSteps, T - w0), m);
                            else walkp<WT, ANCHORED, MODE, WIDE>(c, min(kWaveSteps, T - w0));
                            wave_lds_sync();
                        }
                        if (MU && m.held) eval_mu(m, m.held);   // (the next chunk takes the slots)
                    }
                    if (!formed && hb + ks >= K) {
                        uint32_t d = 1;
                        if (lane == 0) d = atomicAdd(&S.done, 1u);
                        if (__builtin_amdgcn_readfirstlane(d) == 0)
                            form_group<WT, ANCHORED, BATCH>(a, S, S.G[gi ^ 1u], smax);
                        formed = true;
                    }
                    __syncthreads();
                    if (__builtin_amdgcn_readfirstlane(S.need) == 0) break;
                    // the walked candidates bound every counter; the fullest
                    // one is a better bound
                    unsigned long long now = a.flush_limit;
                    if (WT && a.look) {
                        uint32_t top = 0;
                        for (int b = tid; b < a.nconf; b += BLOCK)
                            top = max(top, (uint32_t)(((unsigned long long *)(sm + L.cnt))[b] >> kCntShift));
                        atomicMax(&S.top, top);
                        __syncthreads();
                        now = __builtin_amdgcn_readfirstlane(S.top);
                    }
                    const bool full = now >= a.flush_limit / 2;
                    if (full) {
                        flushp<BLOCK, WT, MODE>(a, L, sm, hout, tout);
                        now = 0;
                    }
                    __syncthreads();
                    if (tid == 0) {
                        ++*(full ? &S.flushes : &S.put_off);
                        S.acc = now;
                        S.need = 0;
                        S.top = 0;
                    }
                    __syncthreads();
                }
                const uint32_t nx = __builtin_amdgcn_readfirstlane(S.next);
                if (nx == kEmptyKey) break;
                __syncthreads();
                klo = nx;
                later = true;
            }
            if (!again) hb += ks;
            if (hb < K) __syncthreads();
        }
    }

    __syncthreads();
    flushp<BLOCK, WT, MODE>(a, L, sm, hout, tout);
    probed = wave_sum64(probed);
    if (lane == 0 && a.probes && probed) atomicAdd(a.probes, (unsigned long long)probed);
    if (tid == 0 && a.probes && (S.flushes | S.put_off))
        atomicAdd(a.probes + 1, S.flushes | (unsigned long long)S.put_off << 32);
}

template <int B, int WT, bool AN, bool BATCH, int MODE, bool WIDE, bool LONG, bool MU = false>
void launchp_k(Ctx &ctx, hipStream_t s, const C3Args &a, uint32_t lds) {
    const void *kern = reinterpret_cast<const void *>(&k_count3p<B, WT, AN, BATCH, MODE, WIDE, LONG, MU>);
    if (lds > 65536) GS_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0;
    GS_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_count3p<B, WT, AN, BATCH, MODE, WIDE, LONG, MU>, B, lds));
    if (per_cu < 1) fail(GS_EUNSUPPORTED, "count kernel does not fit a compute unit");
    uint32_t grid = (uint32_t)ctx.n_cu * (uint32_t)per_cu;
    grid = (grid + kNumQueues - 1) / kNumQueues * kNumQueues;
    // short work: at least about 40 hubs per work group, so that starting and
    // ending the groups does not outweigh the count (2e4 points: 135 us with
    // 512 groups, 195 us with the 1536 that fit the device)
    const uint64_t hubs = BATCH ? a.nvirt : a.h1 - a.h0;
    if (!LONG) grid = (uint32_t)std::min<uint64_t>(grid, std::max<uint64_t>(ctx.n_cu, hubs / 40) / kNumQueues * kNumQueues);
    if (LONG && (WT != 0 || AN) && grid > a.rowgroups) grid = a.rowgroups / kNumQueues * kNumQueues;
    if (const char *e = getenv("GS_PGRID")) grid = std::min<uint32_t>(grid, atoi(e));
    if (getenv("GS_PLAN_LOG")) fprintf(stderr, "count3p launch: %d groups per CU, grid %u\n", per_cu, grid);
    k_count3p<B, WT, AN, BATCH, MODE, WIDE, LONG, MU><<<dim3(grid), dim3(B), lds, s>>>(a);
    GS_HIP(hipGetLastError());
}

template <int B, bool WIDE, bool LONG>
void launchp_w(Ctx &ctx, hipStream_t s, const C3Args &a, const PlanP &P, int wt, bool an, bool batch) {
    const uint32_t lds = P.lds;
    if (batch && !WIDE) {
        if (P.mode == kCube) launchp_k<B, 0, false, true, kCube, false, LONG>(ctx, s, a, lds);
        else launchp_k<B, 0, false, true, kLut, false, LONG>(ctx, s, a, lds);
    } else if (wt == 0) {
        if (an) launchp_k<B, 0, true, false, kLut, WIDE, LONG>(ctx, s, a, lds);
        else if (P.mode == kCube) launchp_k<B, 0, false, false, kCube, WIDE, LONG>(ctx, s, a, lds);
        else launchp_k<B, 0, false, false, kLut, WIDE, LONG>(ctx, s, a, lds);
    } else if (wt == 1) {
        if (an) launchp_k<B, 1, true, false, kLut, WIDE, LONG>(ctx, s, a, lds);
        else launchp_k<B, 1, false, false, kLut, WIDE, LONG>(ctx, s, a, lds);
    } else {
        if (an) launchp_k<B, 2, true, false, kLut, WIDE, LONG>(ctx, s, a, lds);
        else launchp_k<B, 2, false, false, kLut, WIDE, LONG>(ctx, s, a, lds);
    }
}

// 32-bit row offsets in bytes (narrow) or entries (wide), or whole-wavefront
// rows, which take their base from scalar registers and serve either.
template <int B>
void launchp_b(Ctx &ctx, hipStream_t s, const C3Args &a, const PlanP &P, int wt, bool an, bool batch, bool wide) {
    if (P.glog >= 6) launchp_w<B, false, true>(ctx, s, a, P, wt, an, batch);
    else if (wide) launchp_w<B, true, false>(ctx, s, a, P, wt, an, batch);
    else launchp_w<B, false, false>(ctx, s, a, P, wt, an, batch);
}

int env_int(const char *name, int otherwise) {
    const char *e = getenv(name);
    return e ? atoi(e) : otherwise;
}

}  // namespace

namespace {
// Mean row from which the paged table counts faster than the hash walk, whose
// steps go down to one entry. Times as multiples of the hash walk's, uniform
// and clustered catalogues (8e5 points: uniform).
// Small counts are decided by their start: at 5 to 25 entries 0.72 to 0.79 on
// 18000 and 22000 points (weighted and anchored up to 1.05, from 18 bins on
// weighted 1.03 to 1.08 at 8 entries, 0.90 to 1.01 from 13 on), 0.74 to 0.87
// on 26000 and 32000 (weighted or anchored 0.78 to 1.03), 0.72 to 0.92 on
// 40000 (up to 1.08), but 1.03 to 1.19 on 60000 to 250000. Anchors leave few hubs to
// share that start: on 5000 points and more 1.01 to 1.14 at 2 entries, 0.75
// to 1.02 from 4 on, but where the rows are uneven up to 1.10 at 8 to 10
// (weighted 1.18 at 10, 1.10 at 12, 1.08 at 15); a few crowds among many
// sparse hubs keep the hash walk's tiles waiting (0.4 to 0.9 without them).
// Restricted counts have another kernel to beat (paged_pays in count3x.hip).
// Large counts: up to 17 bins 1.03 to 1.23 at 28 entries, 1.0 to 1.14 at 32,
// 0.90 at 34.5 (crowds of 50), 0.92 to 1.04 at 36; weighted with up to 12
// bins 0.80 to 1.0 at 30 to 32 on crowds, 0.99 to 1.09 on uniform points;
// anchored 1.35 at 28 and 1.18 at 36, 1.0 to 1.03 at 42, weighted 1.17 to
// 0.89 at 36 (0.9 at 35 to 40 where the rest is sparse). From 18 bins on the counters and
// their address table, which the hash walk has no more of, leave less room
// for work groups than shorter rows would fill: 20 bins 1.40 at 28, 1.12 at
// 55, 0.88 at 75; 18 bins weighted 1.61, 1.23 and 0.95 (plain 0.78 to 0.95
// from 32 on, anchored 1.40 at 33, 1.13 at 51); 24 bins 1.49, 1.33
// and 1.20 at 85 (0.87 at 110), weighted 0.94 at 28 (the hash walk then has
// one work group per CU), weighted and anchored 1.41 at 36, 0.94 at 75. On
// 60000 points 20 bins 1.07 at 45, 0.93 to 1.03 at 55, 24 bins 0.95 at 64.
// Batches: up to 18 bins 0.51 to 1.02 at 4 entries and more (2 to 32
// catalogues of 2000 to 120000 points); 20 to 24 bins the same below 50000
// points in all, beyond it 1.02 to 1.65 below 30 entries, 0.84 to 1.21 at 45,
// 0.81 to 1.01 at 60.
double least_row(const Shape3 &g) {
    if (g.batch) return g.nb <= 18 || g.batch < 50000 ? 0.0 : 60.0;
    if (g.restricted) return 28.0;
    const bool plain = !g.weighted && !g.anchored;
    const bool few = g.nb <= 17 || (g.nb == 18 && plain);   // bins
    if (g.n < (!few || g.anchored ? 24000u : g.weighted ? 32000u : 45000u)) {
        const double many = g.weighted && g.nb > 17 ? 12.0 : 0.0;
        const double deg = g.maxdeg, row = g.mean_row;
        if (!g.anchored || g.n < 5000 || (g.n < kTileHubs && deg > 6.0 * row)) return many;
        return std::max(many, deg <= 2.0 * row + 12.0 ? 3.0 : g.weighted ? 16.0 : 11.0);
    }
    if (few) return !g.anchored ? (g.weighted && g.nb <= 12 ? 29.0 : 34.0) : g.weighted ? 35.0 : 42.0;
    if (g.nb <= 22) return g.n < 100000 ? 52.0 : 70.0;
    if (g.weighted) return g.anchored ? 70.0 : 36.0;
    return g.n < 100000 ? 65.0 : g.anchored ? 100.0 : 110.0;
}
}  // namespace

bool planp(const Ctx &ctx, const Shape3 &g, const Tune3 &tune, PlanP &p) {
    if (env_int("GS_PAGED", 1) == 0 || tune.kernel == kHash3) return false;
    // overrides of the hash walk's schedule (tests) ask for the hash walk
    for (const char *e : {"GS_MODE3", "GS_PACK", "GS_BLOCK3", "GS_TMAX", "GS_TRUNC", "GS_GLOG"})
        if (getenv(e)) return false;
    const int nb = g.nb, nmu = g.nmu;
    const bool weighted = g.weighted, anchored = g.anchored;
    const uint32_t maxdeg = g.maxdeg;
    const double mean_row = g.mean_row;
    if (nb > kLutMaxBins || maxdeg > 16384 || g.n >= (1ull << 29)) return false;
    // a row's labels must be dense enough in its cells: about 6.4 labels per
    // entry when the cells are rmax wide
    if (13.5 * g.cell_points > 64.0 * (mean_row + 1.0)) return false;
    // (GS_PAGED, GS_PGLOG: any row, for tests)
    if (mean_row < least_row(g) && env_int("GS_PAGED", 0) == 0 && !getenv("GS_PGLOG")) return false;
    const int nconf = (int)n_configs(nb) * std::max(1, nmu);
    // steps of 16 or 32 entries (the latter 1.00 to 1.08 times the former's
    // time at 80 a row, 0.94 to 1.04 at 160, 0.80 to 1.03 at 200, 0.83 to 0.99
    // at 260; 2e4 to 4e5 points), whole-wavefront rows from 1000 entries on
    // (weighted, 5.5e4 points: 81 against 91 ms at 1318 a row, 37.3 against
    // 36.8 at 970, 25.5 against 19.9 at 606); only those have 64-bit offsets
    const bool far = g.max_rows >= kWideSpan;
    p.glog = mean_row >= 1000.0 ? 6 : mean_row >= 160.0 ? 5 : 4;
    if (tune.glog > 0 && !(far && tune.glog < 6)) p.glog = std::max(4, std::min(6, tune.glog));
    p.glog = env_int("GS_PGLOG", p.glog);
    if (nmu || (g.row_room == 0 && (weighted || anchored))) p.glog = std::min(p.glog, 5);
    if (far && p.glog < 6) return false;
    p.kmax = tune.group > 0 ? std::min(tune.group, kMaxGroup) : kMaxGroup;
    p.kmax = p.glog >= 6 ? 1 : std::max(1, std::min(p.kmax, env_int("GS_GROUP", p.kmax)));
    p.inorder = env_int("GS_PORDER", p.glog >= 6) != 0;
    int best = -1;
    auto search = [&](int block, int only) {   // (-1: any)
        for (int blk : {256, 512, 768}) {
            if (blk == 768 && (!weighted || anchored || p.glog < 6)) continue;
            if (block > 0 && blk != block) continue;
            if (getenv("GS_PBLOCK") && blk != env_int("GS_PBLOCK", 256)) continue;
            for (int mode : {kCube, kLut}) {
                if (mode == kCube && (weighted || anchored || nmu || nb > kCubeMaxBins || only == kLut)) continue;
                if (mode == kLut && only == kCube && !weighted && !anchored && !nmu && nb <= kCubeMaxBins) continue;
                if (getenv("GS_PMODE") && !nmu && mode != env_int("GS_PMODE", 0) && !weighted && !anchored) continue;
                const uint32_t fixed = layoutp(blk, 0, nconf, nb, weighted, anchored, mode, p.glog >= 6, nmu != 0).total;
                // pages: about 8 bytes per entry of the rows a group holds
                const double rows = p.glog >= 6 ? mean_row : std::max(mean_row, std::min<double>(p.kmax * mean_row, 2.0 * blk));
                const double per = p.glog >= 6 && (weighted || anchored) ? 2.0 : 1.0;   // bytes per label
                const uint32_t least = (uint32_t)(per * 8.0 * rows) + 2048u;
                const uint32_t most = std::max(least, (uint32_t)(per * 10.0 * std::max<double>(maxdeg, rows)) + 4096u);
                // the counter table holds 16-bit LDS addresses of the (first) counter words
                const uint32_t below = 65536u - kPages - 1024u - (mode == kCube ? 0u : (weighted ? 8u : 4u) * (uint32_t)nconf);
                if (4ull * nconf + kPages + 4096 >= 65536) continue;
                const int cap_waves = (weighted && blk < 768) || nmu ? 16 : 24;
                for (int gr = cap_waves * 64 / blk; gr >= 1; --gr) {
                    const int room = (ctx.max_lds / gr) / 1280 * 1280 - (int)fixed;
                    if (room < 1024 || (gr > 1 && (uint32_t)room < least)) continue;
                    const int waves = gr * blk / 64;
                    // on a tie the smaller group, but the larger where hubs are few
                    // and long, so that the last ones end sooner: 512 threads take
                    // 0.57 to 0.99 of the time of 256 at 200 to 460 entries on 9000
                    // to 32000 points, which the hash walk beat by up to 1.13, 0.97
                    // to 1.14 at 60 to 100; 0.6 to 0.7 at 500 to 1000 on 15000, but
                    // 1.14 on 150000 (weighted, 8 bins)
                    if (waves > best || (waves == best && mean_row >= 200.0 && p.glog < 6 && g.n < 128ull * ctx.n_cu)) {
                        best = waves;
                        p.block = blk;
                        p.mode = mode;
                        p.tbytes = std::min<uint32_t>(std::min<uint32_t>((uint32_t)room, most), below) / 1024 * 1024;
                        if (const char *e = getenv("GS_PTAB")) p.tbytes = std::max(1024, std::min(atoi(e), std::min(room, (int)below))) / 1024 * 1024;
                        p.lds = layoutp(blk, p.tbytes, nconf, nb, weighted, anchored, mode, p.glog >= 6, nmu != 0).total;
                    }
                    break;
                }
            }
        }
    };
    search(tune.block, tune.mode);
    if (best < 0) search(-1, -1);
    if (best < 0) return false;
    p.rowgroups = 0;
    p.rows = 0;
    if (p.glog >= 6 && (weighted || anchored)) {
        // packed hub rows, one per work group that can be resident; without
        // the device memory for them, steps of 32 entries
        p.rowgroups = (uint32_t)((size_t)ctx.n_cu * std::max<size_t>(1, std::min<size_t>(ctx.max_lds / p.lds, 2048 / p.block)) + kNumQueues);
        p.rows = (uint64_t)p.rowgroups * maxdeg * (8 * weighted + 4 * anchored);
        if (p.rows > g.row_room) {
            Shape3 h = g;
            h.row_room = 0;
            return planp(ctx, h, tune, p);
        }
    }
    if (getenv("GS_PLAN_LOG"))
        fprintf(stderr, "count3p plan: maxdeg %u mean_row %.1f block %d glog %d mode %d group %d table %u lds %u waves/CU %d\n",
                maxdeg, mean_row, p.block, p.glog, p.mode, p.kmax, p.tbytes, p.lds, best);
    return true;
}

void launchp(Ctx &ctx, hipStream_t s, const C3Args &a0, const PlanP &P, bool weighted, bool anchored, bool batch,
             bool wide, DevBuf &rows) {
    C3Args a = a0;
    a.glog = P.glog;
    a.mode = P.mode;
    a.kmax = P.kmax;
    a.group_cap = 2ull * P.block;
    if (P.rows) {
        if (rows.bytes < P.rows) rows.alloc(P.rows, ctx.pool);
        a.wrow = rows.as<double>();
        a.prow = (uint32_t *)(a.wrow + (weighted ? (size_t)P.rowgroups * a.maxdeg : 0));
        a.rowgroups = P.rowgroups;
    }
    a.tbytes = P.tbytes;
    a.inorder = P.inorder;
    const int wt = !weighted ? 0 : a.wgen ? 2 : 1;
    // fields of the weighted counters (see the head of this file)
    if (wt) a.flush_limit = std::min<uint64_t>(a.flush_limit, wt == 1 ? 1ull << 21 : 1ull << 20);
    a.look = env_int("GS_FLUSH_LOOK", 1);   // (0: always flush, for tests)
    // a chunk of spokes fits half the limit
    const uint64_t chunk = (a.maxdeg > 4096 ? 16ull : 64ull) * ((uint64_t)a.maxdeg + (1ull << P.glog));
    a.flush_limit = std::max<uint64_t>(a.flush_limit, 2 * chunk + 2);
    if (a.nmu) {
        if (P.block == 512) launchp_k<512, 0, false, false, kLut, false, false, true>(ctx, s, a, P.lds);
        else launchp_k<256, 0, false, false, kLut, false, false, true>(ctx, s, a, P.lds);
    } else if (P.block == 768) {   // weighted, unanchored, long rows
        if (wt == 1) launchp_k<768, 1, false, false, kLut, false, true>(ctx, s, a, P.lds);
        else launchp_k<768, 2, false, false, kLut, false, true>(ctx, s, a, P.lds);
    } else if (P.block == 512) {
        launchp_b<512>(ctx, s, a, P, wt, anchored, batch, wide);
    } else {
        launchp_b<256>(ctx, s, a, P, wt, anchored, batch, wide);
    }
}

}  // namespace gsn
