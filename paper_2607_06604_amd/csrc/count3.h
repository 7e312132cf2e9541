// count3.h - what the two triangle-count kernels (hash table: count3.hip,
// paged table: count3p.hip) and their launch code share.
#pragma once

#include "kern_util.h"

namespace gsn {

// One catalogue of a batched launch: its forward CSR, its first virtual hub
// index and where its counts go.
struct GDesc {
    const uint64_t *rp;
    const uint32_t *col;
    const uint8_t *bin;
    uint64_t v0;              // virtual hub index of label 0
    uint32_t n;
    uint32_t pad;
    unsigned long long *hist; // nconf
    unsigned long long *ntri; // 1
};

struct C3Args {
    const GDesc *gd;        // batched launch: ngraph descriptors (else null)
    int ngraph;
    uint32_t nvirt;         // batched launch: total hubs over all catalogues
    const uint64_t *rp;
    const uint32_t *hcol;   // hub rows (entry e of row i at rp[i] - hbase + e)
    const uint8_t *hbin;
    const uint32_t *scol;   // spoke rows (row j at rp[j] - sbase)
    const uint8_t *sbin;
    uint64_t hbase, sbase;
    uint32_t h0, h1, s0, s1;
    const double *w;        // label-ordered weights (weighted)
    const uint32_t *perm;   // label -> original index (anchored)
    const uint8_t *mark;    // anchored: hubs that can own an anchored triangle (nullable)
    int nb, nconf, log2h;
    int trunc;              // cut spoke rows at the hub row's largest label
    int packed;             // hash entries hold (bin << 24 | label): labels < 2^24 - 1
    int glog;               // entries per step = 2^glog
    int mode;               // hit counter addressing: kRank, kLut or kCube
    int kmax;               // hubs per group (1..kMaxGroup)
    int yshift;             // packed hash entries: bin << yshift | hub << 24 | label
    uint64_t group_cap;     // rows of a group (beyond the first hub) fit this many entries
    uint32_t maxdeg;
    uint32_t tmax;          // steps per table fill
    uint32_t tcap;          // table entries: tmax + padding of one pass
    int inorder;            // paged table: hubs handed out one at a time in label order, device-wide
    uint32_t tbytes;        // paged table: bytes of its pages (the zero page among them)
    double *wrow;           // paged table, long rows: packed weights and original indices of a
    uint32_t *prow;         // work group's hub row, maxdeg entries each
    uint32_t rowgroups;     // work groups they serve
    uint32_t anchor_lo, anchor_hi;
    double wmul;            // 2^wscale
    int wgen;               // some weight is negative or some term may reach 2^63
    uint64_t flush_limit;   // flush LDS counters before this many increments
    int look;               // paged table: unless the fullest one shows that there is room (weighted)
    uint32_t *queue;        // kQueueWords words
    unsigned long long *hist;   // nconf
    unsigned long long *wsum;   // 2*nconf (lo, hi)
    unsigned long long *ntri;   // 1
    unsigned long long *probes; // candidates probed (nullable); then, paged table, flushes in mid-count
                                // (low half) and those the fullest counter put off
    uint32_t *err;          // bit 1: LDS addressing
    uint64_t wspan;         // WIDE: entries a segment of spoke rows may span from its first row
    const uint16_t *cfg3;   // kLut / kCube: configuration index of ordered triple (x*nb + y)*nb + z
    int nmu;                // mu counts (else 0): counters per configuration
    const int4 *q4;         // their positions in units of the box / 2^32 (wrapping)
    float qscale;           // such a unit over rmax
    const double *X, *Y, *Z;
    double L, half;
    const uint32_t *tiles;  // hub tiles of about equal cost: tile t = [tiles[t], tiles[t+1]) (or null)
    uint32_t ntiles;
};

// 32-bit offsets of spoke rows from a hub's first: bytes below 2^30 entries,
// entries below 2^32.
constexpr uint64_t kNarrowSpan = 1ull << 30;
constexpr uint64_t kWideSpan = 1ull << 32;
constexpr int kLutMaxBins = 24;          // nb^3 u16 table up to 27 KB
constexpr int kCubeMaxBins = 16;         // nb^3 u32 counters up to 16 KB
constexpr int kMaxGroup = 4;             // hubs per group: two bits in a step entry

// How a hit finds its counter: the configuration index from the rank tables
// (kRank), an nb^3 table of counter addresses (kLut), or no index at all --
// one LDS counter per ordered bin triple (x, y, z), folded into
// configurations when the counters are flushed (kCube, unweighted only).
enum { kRank = 0, kLut = 1, kCube = 2 };

// Paged counts of fewer hubs leave out the tile plan where it does not pay.
constexpr uint32_t kTileHubs = 12288;

// The schedule of a paged-table count (count3p.hip).
struct PlanP {
    int block = 256;
    int glog = 4;          // entries per step = 2^glog (4 to 6)
    int mode = kLut;
    int kmax = kMaxGroup;  // hubs per group at most
    bool inorder = false;  // hubs go out one at a time in label order, not by tiles
    uint32_t tbytes = 0;   // bytes of the label table's pages
    uint32_t lds = 0;
    uint32_t rowgroups = 0;  // work groups with a packed hub row (long weighted or anchored rows)
    uint64_t rows = 0;       // and the device bytes of those rows
};

// What a schedule depends on.
struct Shape3 {
    uint32_t maxdeg = 0;
    int nb = 0;
    bool weighted = false, anchored = false;
    uint64_t n = 0;          // points (the largest catalogue of a batch)
    double mean_row = 0;     // forward entries per point
    double cell_points = 0;  // points per cell of the build's grid
    uint64_t max_rows = 0;   // entries that the spoke rows of one launch span
    int nmu = 0;             // mu bins (else 0)
    bool restricted = false; // for an equilateral or mu count
    uint64_t batch = 0;      // points of all catalogues of a batch (else 0)
    uint64_t row_room = ~0ull;   // device bytes left for packed hub rows
};

// The schedule for a graph of that shape, or false where the paged table does
// not serve (then the hash table does). A tuned value that this count cannot
// take (768 threads with anchors, say) gives way to the built-in choice.
bool planp(const Ctx &ctx, const Shape3 &g, const Tune3 &tune, PlanP &p);
// rows: device memory the launch may need (taken on first use; held by the
// caller until the launch has completed).
void launchp(Ctx &ctx, hipStream_t s, const C3Args &a, const PlanP &P, bool weighted, bool anchored, bool batch,
             bool wide, DevBuf &rows);

// Catalogue of virtual hub v: the last descriptor with v0 <= v.
__device__ __forceinline__ int graph_of(const GDesc *gd, int ng, uint32_t v) {
    int lo = 0, hi = ng;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (gd[mid].v0 <= v) lo = mid;
        else hi = mid;
    }
    return lo;
}

// mu bin of the triangle with (minimum-image) edge vectors u = p0->p1 and
// v = p0->p2.
__device__ __forceinline__ int mu_bin(double ux, double uy, double uz, double vx, double vy, double vz, int nmu) {
    const double nx = __dsub_rn(__dmul_rn(uy, vz), __dmul_rn(uz, vy));
    const double ny = __dsub_rn(__dmul_rn(uz, vx), __dmul_rn(ux, vz));
    const double nz = __dsub_rn(__dmul_rn(ux, vy), __dmul_rn(uy, vx));
    const double s = __dadd_rn(__dadd_rn(__dmul_rn(nx, nx), __dmul_rn(ny, ny)), __dmul_rn(nz, nz));
    const double t = __dmul_rn(__dmul_rn(nz, nz), (double)(nmu * nmu));
    int m = 0;
    if (s > 0.0)
        for (int k = 1; k < nmu; ++k) m += t >= __dmul_rn((double)(k * k), s);
    return m;
}

// A vertex: absolute coordinates and original index.
struct P3x {
    double x, y, z;
    uint32_t o;
};

__device__ __forceinline__ void swapx(P3x &a, P3x &b) {
    const P3x t = a;
    a = b;
    b = t;
}

// Sort three vertices by original index.
__device__ __forceinline__ void order3(P3x &a, P3x &b, P3x &c) {
    if (a.o > b.o) swapx(a, b);
    if (b.o > c.o) swapx(b, c);
    if (a.o > b.o) swapx(a, b);
}

__device__ __forceinline__ unsigned long long wave_sum64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace gsn
