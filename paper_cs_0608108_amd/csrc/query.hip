// Neighbourhood query kernels for gfx950 (wave64).
//
// Per query:
//   setup   (one thread per query, setup_kernel) home cell = q >> F, sub-cell
//           class = the top s bits of q's position inside its cell along y
//           and z (Section III.A: the position inside the cell selects a
//           specialised table), the method, and the class table's prefix end
//           from the radius index (Section II.A: one lookup tells where to
//           stop in the sorted table), stored as a 64-byte descriptor.
//   walk    the class table lists x-rows of cells (oy, oz) sorted by their
//           minimum distance, centre to edge; 64 rows per step, one per lane.
//           A lane solves the exact test of Eq. 1 for its row's contiguous
//           run of cells, wraps cyclic axes or clips to the region (Section
//           II.B), and turns the run into one range of objects (two when it
//           wraps), since objects are sorted by packed ZYX cell.
//   scan    the objects of the rows are spread over the lanes: a DPP prefix
//           sum of per-lane counts, an LDS map of where each lane's range
//           starts and a DPP max-scan give every slot its owner, so a wave
//           tests 64 candidates per step whatever the cell loads.  One
//           16-byte load fetches a candidate's coordinates and id.
//   output  count pass: hits per row (K-NN: min(K, hits within the cap),
//           stopping once K are found); with workspace to spare it also
//           sorts each radius row by (dist^2, id) and keeps it (the stash),
//           and the write pass only copies the kept rows into place.  Rows
//           not kept are walked again by the write pass.  Long radius rows
//           take one block each.  K-NN rows not kept go to the top-M
//           kernel, which keeps the M best (in registers for M <= 64),
//           shrinks the bound to the M-th distance once M are held and
//           stops at the first row whose key exceeds it (Section II.A, K
//           nearest).
// The count pass can also take radius queries in groups of several per
// wavefront, so that short rows and small radii fill whole steps, and
// all-agents queries of one radius by tiles of space, their pairs on the
// matrix cores.  Queries
// whose radius exceeds the tables' cap or the cyclic limit, or whose centre
// is outside the region, and every query of the cube method, scan the
// bin-lattice bounding cube instead (Section I; Section III.B).  With the
// per-query choice each query takes the sphere, the cube or the lattice's
// non-empty cell list, whichever the comparison of their cells (Section
// III.B, III.C) or of their estimated work finds smallest; a list entry is
// one more kind of row.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "sphidx_internal.h"

namespace {

constexpr uint32_t kMaxId = 0xFFFFFFFFu;
constexpr uint64_t kMaxD2 = ~0ull;
// Walk kinds: sphere rows only, cube rows only, either (chosen per query),
// or the paper's cell tables (cube rows for the queries they do not serve).
constexpr int kSphere = 0, kCube = 1, kEither = 2, kPaper = 3;

// ---------------------------------------------------------------------------
// Wave primitives

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t base = 0u) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}
// This lane's bit of a wave mask, as a predicate.
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ uint32_t bperm(uint32_t v, uint32_t lane) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(lane << 2), (int)v);
}
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
    return ((uint64_t)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v);
}
__device__ __forceinline__ uint32_t lane_val(uint32_t v, uint32_t l) { return __builtin_amdgcn_readlane(v, l); }
// LDS ordering point for one wavefront: its LDS operations execute in order;
// this keeps the compiler from moving them across the point.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL, int ROWS, bool BOUND>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, BOUND);
}

// Inclusive prefix sum over the 64 lanes: shifts by 1, 2, 4, 8 inside each
// row of 16 lanes, then row 0's total into row 1 and row 2's into row 3
// (row_bcast:15), then rows 0-1's total into rows 2-3 (row_bcast:31).
__device__ __forceinline__ uint32_t scan_add(uint32_t v) {
    v += dpp<0x111, 0xF, true>(v);
    v += dpp<0x112, 0xF, true>(v);
    v += dpp<0x114, 0xF, true>(v);
    v += dpp<0x118, 0xF, true>(v);
    v += dpp<0x142, 0xA, false>(v);
    v += dpp<0x143, 0xC, false>(v);
    return v;
}

__device__ __forceinline__ uint32_t scan_max(uint32_t v) {
    v = max(v, dpp<0x111, 0xF, true>(v));
    v = max(v, dpp<0x112, 0xF, true>(v));
    v = max(v, dpp<0x114, 0xF, true>(v));
    v = max(v, dpp<0x118, 0xF, true>(v));
    v = max(v, dpp<0x142, 0xA, false>(v));
    v = max(v, dpp<0x143, 0xC, false>(v));
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return lane_val(scan_add(v), 63); }

__device__ __forceinline__ bool key_less(uint64_t da, uint32_t ia, uint64_t db, uint32_t ib) {
    return da < db || (da == db && ia < ib);
}

// Sort one (d2, id) key per lane ascending over the 64 lanes (bitonic).
__device__ __forceinline__ void wave_sort64(uint64_t& d, uint32_t& id) {
    const uint32_t l = lane_id();
#pragma unroll
    for (uint32_t k = 2; k <= 64; k <<= 1) {
#pragma unroll
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            uint32_t plo = __shfl_xor((uint32_t)d, j);
            uint32_t phi = __shfl_xor((uint32_t)(d >> 32), j);
            uint32_t pid = __shfl_xor(id, j);
            uint64_t pd = ((uint64_t)phi << 32) | plo;
            bool want_min = ((l & j) == 0) == ((l & k) == 0);
            bool take = want_min ? key_less(pd, pid, d, id) : key_less(d, id, pd, pid);
            if (take) {
                d = pd;
                id = pid;
            }
        }
    }
}

// Sort a bitonic sequence of one (d2, id) key per lane ascending.
__device__ __forceinline__ void wave_bitonic_clean64(uint64_t& d, uint32_t& id) {
    const uint32_t l = lane_id();
#pragma unroll
    for (uint32_t j = 32; j > 0; j >>= 1) {
        uint32_t plo = __shfl_xor((uint32_t)d, j);
        uint32_t phi = __shfl_xor((uint32_t)(d >> 32), j);
        uint32_t pid = __shfl_xor(id, j);
        uint64_t pd = ((uint64_t)phi << 32) | plo;
        bool take = (l & j) == 0 ? key_less(pd, pid, d, id) : key_less(d, id, pd, pid);
        if (take) {
            d = pd;
            id = pid;
        }
    }
}

__device__ __forceinline__ uint64_t lane_val64(uint64_t v, uint32_t l) {
    return ((uint64_t)lane_val((uint32_t)(v >> 32), l) << 32) | lane_val((uint32_t)v, l);
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, uint32_t src) {
    return ((uint64_t)__shfl((uint32_t)(v >> 32), src) << 32) | (uint32_t)__shfl((uint32_t)v, src);
}

// Exact quotient (a < 2^31, 1 <= b < 2^31) from a double reciprocal and one
// correction step.
__device__ __forceinline__ uint32_t exact_div(uint32_t a, uint32_t b, double inv_b) {
    uint32_t q = (uint32_t)((double)a * inv_b);
    if ((uint64_t)q * b > a) --q;
    if ((uint64_t)(q + 1) * b <= a) ++q;
    return q;
}

__device__ __forceinline__ uint64_t sq(uint32_t g) { return (uint64_t)g * (uint64_t)g; }


// ---------------------------------------------------------------------------
// Query descriptors

// F_LIST: the query walks the non-empty cell list (neither F_SPHERE nor
// F_LIST: the bounding cube).
// F_KBOUND: a K-NN row whose count pass found K objects within the radius
// stored in descriptor word 12 (an upper bound of its K-th distance; sphere
// walks only, which leave that word unused).  F_LONG: a radius row expected
// to be longer than a wavefront's buffer, counted and kept one block per row.
// F_WINDOW: a radius row that the block kernel of the write pass left to the
// windowed top-M kernel.  F_ALONE: a K-NN row of a grouped count that the setup
// listed for the one-query-per-wave kernel.
enum : uint32_t {
    F_VALID = 1u, F_KNN = 2u, F_SPHERE = 4u, F_OUTSIDE = 8u, F_LIST = 16u, F_KBOUND = 32u, F_LONG = 64u,
    F_WINDOW = 128u, F_ALONE = 256u
};

struct Query {
    uint32_t q[3];  // normalised centre
    uint32_t row;   // output row
    uint32_t r;     // radius, or the K-NN cap
    uint32_t k;
    uint32_t flags;
    uint32_t tb;    // sphere: first entry of the class table
    uint32_t tend;  // sphere: prefix length
    uint32_t ncube; // cube: cells of the bounding cube
    uint32_t nn[3]; // cube: cells per axis (cell list: 0, its length, 1)
    int32_t lo[3];  // cube: first cell per axis
    uint32_t self;  // sorted position excluded (EXCLUDE_SELF, all agents) or ~0
    uint32_t kbr;   // F_KBOUND: a radius holding K objects
    uint32_t c[3];  // home cell
    uint32_t f[3];  // position inside the home cell
    uint32_t up[3]; // e - f: distance to the next cell up
    uint32_t dn[3]; // f + 1: distance to the last position of the cell below
    uint64_t r2;
};

__device__ __forceinline__ uint32_t pack_cell(const LatArgs& L, uint32_t x, uint32_t y, uint32_t z) {
    return (z << (L.lg[0] + L.lg[1])) | (y << L.lg[0]) | x;
}

// Zero counter words [begin, end), by one block; the count pass also writes the
// stash header (hdr != NULL: six words), inside the cleared range, after every
// clear.  Counters sit SPHIDX_QSTRIDE words apart and only those words are
// read: the others are left as they are.
__device__ void clear_counters(uint32_t* c, uint32_t begin, uint32_t end, uint32_t* hdr, uint4 hv, uint32_t tiles) {
    for (uint32_t i = begin + threadIdx.x * SPHIDX_QSTRIDE; i < end; i += blockDim.x * SPHIDX_QSTRIDE) c[i] = 0u;
    if (!hdr) return;
    __syncthreads();
    if (threadIdx.x == 0) {
        hdr[kHdrMode] = hv.x;
        hdr[kHdrElems] = hv.y;
        hdr[kHdrHasD2] = hv.z;
        hdr[kHdrD2Off] = hv.w;
        hdr[kHdrTiles] = tiles;
        hdr[kHdrSparse] = 0u;
    }
}

// `dense` > 0: whether half of 1,024 objects, of every part of the lattice, have
// fewer than `dense` other objects per cell in the 33 cells along x around their
// own (kGroupSampled; the header's sparse word).
__global__ void clear_counters_kernel(uint32_t* c, uint32_t begin, uint32_t end, uint32_t* hdr, uint4 hv,
                                      uint32_t tiles, LatArgs L, float dense) {
    __shared__ uint32_t votes;
    if (threadIdx.x == 0) votes = 0u;
    clear_counters(c, begin, end, hdr, hv, tiles);
    if (!(dense > 0.0f)) return;
    __syncthreads();
    const uint32_t in = L.cs[L.ncells], per = 1024u / blockDim.x;  // objects of the region
    for (uint32_t j = 0; j < per && in > 0u; ++j) {
        const uint4 P = L.pts[(uint32_t)(((uint64_t)(threadIdx.x * per + j) * in) >> 10)];
        const uint32_t cx = P.x >> L.F, nx = 1u << L.lg[0];
        const uint32_t below = min(cx, 16u), above = min(nx - 1u - cx, 16u);
        const uint32_t home = pack_cell(L, cx, P.y >> L.F, P.z >> L.F);
        const uint32_t others = L.cs[home + above + 1u] - L.cs[home - below] - 1u;
        if ((float)others < dense * (float)(below + above + 1u)) atomicAdd(&votes, 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0 && votes > 512u) hdr[kHdrSparse] = 1u;
}

// Whether the sample left a batch that could go in groups to one query per
// wavefront.
__device__ __forceinline__ bool left_sparse(const QArgs& A) {
    return A.group == kGroupSampled && uni(A.stash_hdr[kHdrSparse]) != 0u;
}

// One thread per query: centre, radius, K, method and walk extent.
// K-NN first search radius in the grouped count: the radius of the ball
// expected to hold knn_target(K) objects at the density around the home cell.
// For small K that is 1.2^3 K (about 1.7K): smaller leaves more rows short of
// K (searched again), larger overflows more hit buffers; on clustered K = 16
// the step took 5.93, 5.29, 5.23, 5.24, 5.34, 5.53, 6.50 and 8.45 ms at radius
// factors 1.1, 1.15, 1.18, 1.2, 1.22, 1.25, 1.35 and 1.5 (home cell density,
// cells in counting-sort order); with cells in x order and the three-cell
// density, 3.98, 3.82 and 4.30 ms at 1.15, 1.2 and 1.3.  For large K the count
// inside a ball varies relatively less (about sqrt(K)), so K + 3 sqrt(K) + 3
// is enough, and a row of K up to half the hit buffer fits it.
__host__ __device__ inline float knn_target(float k) {
    const float a = 1.728f * k, b = k + 3.0f * __builtin_sqrtf(k) + 3.0f;
    return a < b ? a : b;
}

// Pairs of the grouped count's hit buffer (eighths of sort_cap).
constexpr uint32_t kHitEighths = 8;
__host__ __device__ constexpr uint32_t group_hitcap(uint32_t cap) { return cap * kHitEighths / 8; }

// Every query; with the tile kernel, the objects outside the region only (a
// row that kernel does not keep is set up where it is walked, tile_query).
// With `counters` (a launch of one block) the block first clears the counters
// and writes the stash header, as clear_counters_kernel.
template <int METHOD>
__global__ __launch_bounds__(1024) void setup_kernel(LatArgs L, TabArgs T, QArgs A, uint32_t* counters, uint4 hv) {
    if (counters) {
        clear_counters(counters, 0u, SPHIDX_COUNTER_WORDS, A.stash_hdr, hv, A.tiles);
        __threadfence();
        __syncthreads();
    }
    const uint32_t first = A.tiles ? L.cs[L.ncells] : 0u, stride = gridDim.x * blockDim.x;
    for (uint32_t i = first + blockIdx.x * blockDim.x + threadIdx.x; uni(i) < A.Q; i += stride) {
    bool range_bad = false, fallback = false, to_list = false, longrow = false, alone = false;
    if (i < A.Q) {
        uint32_t q[3], row, r, k;
        bool valid = true;
        if (A.qx == nullptr) {
            const uint4 P = L.pts[i];
            q[0] = P.x;
            q[1] = P.y;
            q[2] = P.z;
            row = P.w;
            // objects left out by the build (clipped coordinate >= 2^30) sit
            // after the outside cell; their rows stay empty
            valid = i < L.cs[L.ncells + 1];
        } else {
            q[0] = A.qx[i];
            q[1] = A.qy[i];
            q[2] = A.qz[i];
            row = i;
            for (int a = 0; a < 3; ++a) {
                if ((L.cyc >> a) & 1u)
                    q[a] &= (1u << (L.lg[a] + L.F)) - 1u;
                else if (q[a] >= (1u << 30))
                    valid = false;
            }
            range_bad = !valid;
        }
        r = A.rad ? A.rad[row] : A.rad_u;
        k = A.kk ? A.kk[row] : A.k_u;
        const bool knn = A.mode == SPHIDX_MODE_KNN || (A.mode == SPHIDX_MODE_MIXED && k > 0);
        if (knn && k == 0) valid = false;
        const uint32_t e = 1u << L.F;
        bool inside = true, cyc_ok = true, outside = false;
        uint32_t ncube = 1, nn[3] = {0, 0, 0};
        uint64_t nfull = 1;  // the cube's cells before clipping to the region
        int32_t lo3[3] = {0, 0, 0};
        for (int a = 0; a < 3; ++a) {
            const uint32_t La = 1u << L.lg[a];
            int64_t lo = ((int64_t)q[a] - (int64_t)r) >> L.F;
            int64_t hi = ((int64_t)q[a] + (int64_t)r) >> L.F;
            nfull *= (uint64_t)min(hi - lo + 1, ((L.cyc >> a) & 1u) ? (int64_t)La : hi - lo + 1);
            if ((L.cyc >> a) & 1u) {
                // the sphere walk needs ceil(r/e) <= L/2 - 1 (no offset repeats a cell)
                if (La < 4 || (uint64_t)r > (uint64_t)(La / 2 - 1) * e) cyc_ok = false;
                if (hi - lo + 1 >= (int64_t)La) {
                    lo = 0;
                    hi = La - 1;
                }
            } else {
                if (q[a] >= (La << L.F)) inside = false;
                if (hi >= (int64_t)La) outside = true;
                if (lo < 0) lo = 0;
                if (hi > (int64_t)La - 1) hi = (int64_t)La - 1;
            }
            lo3[a] = (int32_t)lo;
            nn[a] = hi >= lo ? (uint32_t)(hi - lo + 1) : 0u;
            ncube *= nn[a];
        }
        // the tables serve centres inside the region, radii up to their cap
        // and, on cyclic axes, up to the limit where no offset repeats a cell
        const bool tables = METHOD == kSphere || METHOD == kPaper;
        const bool usable = tables && inside && cyc_ok && r <= T.rmax;
        bool sphere = usable, list = false;
        const uint32_t j = (uint32_t)(((uint64_t)r + (1u << T.rshift) - 1u) >> T.rshift);
        if (A.select == 2u) {
            sphere = false;
            list = true;
        } else if (A.select == 1u && valid) {
            // Section III.B/C: the walk with the fewest cells among the sphere
            // table's prefix, the bounding cube clipped to the region and the
            // non-empty cell list; the weight scales the sphere's count against
            // the cube's, and below the reversal distances the sphere is left
            // out (Appendix).  K-NN queries choose only between the sphere and
            // the cube (Section IV.B).
            // Model 1 (this design's reading of the weighting, for a row
            // walk): each walk's lane work, rows visited plus objects tested,
            // the latter as the mean objects per cell times the cells read.
            if (knn) {
                sphere = sphere && r >= A.knn_rev;
            } else {
                sphere = sphere && r >= A.rev;
                const uint64_t load = A.model ? min(((uint64_t)L.n << 8) / L.ncells, (uint64_t)1 << 24) : 0u;
                uint64_t ws = 0, tested = ncube;
                const uint64_t wc = A.model ? (uint64_t)nn[1] * nn[2] * 256u + load * ncube : ncube;
                uint64_t chosen = wc;
                if (sphere) {
                    const uint32_t cls3 = ((q[0] & (e - 1u)) >> (L.F - T.s)) |
                                          (((q[1] & (e - 1u)) >> (L.F - T.s)) << T.s) |
                                          (((q[2] & (e - 1u)) >> (L.F - T.s)) << (2u * T.s));
                    const uint64_t vs = T.vcount[(size_t)cls3 * T.nr + j];
                    if (A.model) {
                        // every table row takes a lane; objects are read only
                        // in the region: the sphere's cells scaled by the
                        // part of its bounding cube inside the region
                        const uint32_t rcls = cls3 >> T.s;
                        tested = vs * ncube / nfull;
                        ws = (uint64_t)T.rindex[(size_t)rcls * T.nr + j] * 256u + load * tested;
                    } else {
                        ws = vs;
                    }
                    sphere = (unsigned __int128)ws * A.weight <= (unsigned __int128)wc * 256u;
                    if (sphere) chosen = ws;
                }
                if (L.ncl) {
                    const uint64_t nl = *L.ncl;
                    // the list tests the objects of the cells the sphere meets
                    // (with the sphere left out: the cube's)
                    const uint64_t wl = A.model ? nl * 256u + load * tested : nl;
                    if (wl < chosen) {
                        sphere = false;
                        list = true;
                    }
                }
            }
        }
        fallback = valid && tables && !usable;
        // (chosen per query: the main kernels take every walk themselves)
        to_list = valid && tables && !sphere && A.select != 1u && !A.merged;
        // a radius row of the main kernels expected (at the lattice's mean
        // density) to pass 5/4 of a wavefront's row buffer: with the stash
        // and the block kernel, one block counts, orders and keeps it in a
        // single walk instead of a count walk and a write walk
        // (not with per-query statistics, which that kernel does not keep)
        if (valid && !knn && !to_list && !(A.merged && !sphere) && A.stash && A.long_waves > 1 && !A.stats) {
            const float rc = (float)r / (float)e;
            const float expect = 4.18879f * rc * rc * rc * ((float)L.n / (float)L.ncells);
            longrow = expect > 1.25f * (float)A.sort_cap;
        }
        // a K-NN row of the sphere tables that the groups never take (K past
        // half their buffer): straight onto the last list of a grouped count,
        // in the queries' order (262,144 rows of K = 200 through both grouped
        // rounds' lists took 9.18 ms, 0.78 of it to pass them on; one query per
        // wavefront 8.04, this way 8.48)
        alone = METHOD != kPaper && A.group && valid && knn && sphere && k > group_hitcap(A.sort_cap) / 2u &&
                !left_sparse(A);
        uint32_t tb = 0, tend = 0, kb = 0, kend = 0;
        if (METHOD == kPaper && sphere && valid) {
            // the paper's tables (Section III.A): with d = r / e, the unshaved
            // table below floor(d)^2, then, up to floor(d^2), the table chosen
            // by the six flags [frac(d) < zeta] (zeta: e - f up, f down);
            // tb = the specialised part's first entry, ncube = the unshaved
            // entries before it, tend = all entries
            const uint32_t D0 = r >> L.F, fu = r & (e - 1u);
            uint32_t tsel = 0;
            for (int a = 0; a < 3; ++a) {
                const uint32_t f = q[a] & (e - 1u);
                if (fu < e - f) tsel |= 1u << (2 * a);
                if (fu < f) tsel |= 1u << (2 * a + 1);
            }
            const uint32_t lo2 = D0 * D0;
            const uint32_t b2max = (uint32_t)(((uint64_t)r * r) >> (2 * L.F));
            const uint32_t* base_lo = T.p_lo + (size_t)64 * T.p_nb2;
            const uint32_t* spec_lo = T.p_lo + (size_t)tsel * T.p_nb2;
            const uint32_t nbase = base_lo[lo2] - base_lo[0];
            tb = spec_lo[lo2];
            tend = nbase + (spec_lo[b2max + 1] - tb);
            ncube = nbase;
        } else if (sphere && valid) {
            // row tables are specialised on the (y, z) sub-cell position
            const uint32_t cls = ((q[1] & (e - 1u)) >> (L.F - T.s)) | (((q[2] & (e - 1u)) >> (L.F - T.s)) << T.s);
            tb = T.cstart[cls];
            tend = T.rindex[(size_t)cls * T.nr + j];
            if (knn) {
                // K-NN: a first search radius expected to hold knn_target(K)
                // objects at the density of the home cell and its two
                // neighbours along x (one contiguous range of counts; the
                // lattice mean as a floor), and its table prefix; the grouped
                // count searches it as a radius row and keeps the first K
                // when it holds K.  (The home cell alone sent 3.4 % of the
                // clustered K = 16 rows to the one-query-per-wave kernel,
                // the three cells 2.0 %: 4.04 -> 3.82 ms per step.)
                const uint32_t home = pack_cell(L, q[0] >> L.F, q[1] >> L.F, q[2] >> L.F);
                const uint32_t hl = home > 0u ? home - 1u : 0u, hr = min(home + 2u, L.ncells);
                const float dens =
                    fmaxf((float)L.n / (float)L.ncells, (float)(L.cs[hr] - L.cs[hl]) / (float)(hr - hl));
                const float rho = (float)e * cbrtf(0.2387f * knn_target((float)k) / fmaxf(dens, 1e-6f));
                kb = rho >= (float)r ? r : max(1u, (uint32_t)rho);
                const uint32_t jb = (uint32_t)(((uint64_t)kb + (1u << T.rshift) - 1u) >> T.rshift);
                kend = T.rindex[(size_t)cls * T.nr + jb];
            }
        }
        if (list) {
            // the walk takes nn[1] * nn[2] entries: the whole list
            nn[0] = 0u;
            nn[1] = *L.ncl;
            nn[2] = 1u;
            lo3[0] = lo3[1] = lo3[2] = 0;
        }
        if (A.method_out)
            A.method_out[row] = !valid ? 0xFFFFFFFFu
                                       : sphere ? SPHIDX_METHOD_SPHERE : list ? SPHIDX_METHOD_LIST : SPHIDX_METHOD_CUBE;
        const uint32_t flags = (valid ? F_VALID : 0u) | (knn ? F_KNN : 0u) | (sphere ? F_SPHERE : 0u) |
                               (outside ? F_OUTSIDE : 0u) | (list ? F_LIST : 0u) | (longrow ? F_LONG : 0u) |
                               (alone ? F_ALONE : 0u);
        uint4* d = A.desc + 4 * (size_t)i;
        d[0] = make_uint4(q[0], q[1], q[2], row);
        d[1] = make_uint4(r, k, flags, tb);
        // (sphere K-NN queries walk no cube: its fields carry the first radius)
        const bool kfirst = METHOD != kPaper && sphere && valid && knn;
        d[2] = make_uint4(tend, kfirst ? kb : ncube, kfirst ? kend : nn[0], nn[1]);
        d[3] = make_uint4((uint32_t)lo3[0], (uint32_t)lo3[1], (uint32_t)lo3[2], nn[2]);
    }
    // queries for the fallback list's kernels (bounding cube or cell list):
    // one atomic per wavefront, the wavefront's queries in order
    const uint64_t lm = __ballot(to_list);
    if (lm) {
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(A.fb_count, (uint32_t)__popcll(lm));
        base = uni(base);
        if (to_list) A.fbq[base + lanes_below(lm)] = i;
    }
    const uint64_t gm = __ballot(longrow);
    if (gm) {
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(A.lq_count, (uint32_t)__popcll(gm));
        base = uni(base);
        if (longrow) A.lq[base + lanes_below(gm)] = i;
    }
    const uint64_t km = __ballot(alone);
    if (km) {
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(A.long_count, (uint32_t)__popcll(km));
        base = uni(base);
        if (alone) A.longq[base + lanes_below(km)] = i;
    }
    if (__ballot(range_bad) && lane_id() == 0) atomicOr(L.status, SPHIDX_FLAG_RANGE);
    if (__ballot(fallback) && lane_id() == 0) atomicOr(L.status, SPHIDX_FLAG_FALLBACK);
    }
}

// Descriptors are read through the scalar cache (the address is uniform and
// the array was written by an earlier kernel).
typedef __attribute__((address_space(4))) const uint32_t const_u32;

__device__ __forceinline__ Query load_query(const LatArgs& L, const QArgs& A, uint32_t qi) {
    Query s;
    const const_u32* d = (const const_u32*)(A.desc + 4 * (size_t)uni(qi));
    s.q[0] = d[0];
    s.q[1] = d[1];
    s.q[2] = d[2];
    s.row = d[3];
    s.r = d[4];
    s.k = d[5];
    s.flags = d[6];
    s.tb = d[7];
    s.tend = d[8];
    s.ncube = d[9];
    if (!(s.flags & F_SPHERE)) {
        s.nn[0] = d[10];
        s.nn[1] = d[11];
        s.nn[2] = d[15];
        s.lo[0] = (int32_t)d[12];
        s.lo[1] = (int32_t)d[13];
        s.lo[2] = (int32_t)d[14];
    }
    s.kbr = (s.flags & F_KBOUND) ? d[12] : 0u;
    s.self = (A.qx == nullptr && (A.flags & SPHIDX_EXCLUDE_SELF)) ? qi : kMaxId;
    const uint32_t e = 1u << L.F;
    for (int a = 0; a < 3; ++a) {
        s.c[a] = s.q[a] >> L.F;
        s.f[a] = s.q[a] & (e - 1u);
        s.up[a] = e - s.f[a];
        s.dn[a] = s.f[a] + 1u;
    }
    s.r2 = (uint64_t)s.r * (uint64_t)s.r;
    return s;
}

// The query of sorted position qi, an object of the region, after a count pass
// by tiles (one radius, on the sphere tables): what setup_kernel would have
// made of it.
__device__ __forceinline__ Query tile_query(const LatArgs& L, const TabArgs& T, const QArgs& A, uint32_t qi) {
    Query s;
    const const_u32* P = (const const_u32*)(L.pts + uni(qi));
    s.row = P[3];
    s.r = A.rad_u;
    s.r2 = (uint64_t)s.r * (uint64_t)s.r;
    s.k = s.ncube = s.kbr = 0u;
    s.flags = F_VALID | F_SPHERE;
    const uint32_t e = 1u << L.F;
    for (int a = 0; a < 3; ++a) {
        s.q[a] = P[a];
        s.c[a] = s.q[a] >> L.F;
        s.f[a] = s.q[a] & (e - 1u);
        s.up[a] = e - s.f[a];
        s.dn[a] = s.f[a] + 1u;
        if (!((L.cyc >> a) & 1u) && ((s.q[a] + s.r) >> L.F) >= (1u << L.lg[a])) s.flags |= F_OUTSIDE;
    }
    const uint32_t cls = (s.f[1] >> (L.F - T.s)) | ((s.f[2] >> (L.F - T.s)) << T.s);
    s.tb = T.cstart[cls];
    s.tend = T.rindex[(size_t)cls * T.nr + ((s.r + (1u << T.rshift) - 1u) >> T.rshift)];
    s.self = (A.flags & SPHIDX_EXCLUDE_SELF) ? qi : kMaxId;
    return s;
}

// Cells of the bounding cube of query s (in-region cells only), for stats.
__device__ __forceinline__ uint32_t cube_cells(const LatArgs& L, const Query& s) {
    uint32_t n = 1;
    for (int a = 0; a < 3; ++a) {
        const int64_t La = (int64_t)1 << L.lg[a];
        int64_t lo = ((int64_t)s.q[a] - (int64_t)s.r) >> L.F;
        int64_t hi = ((int64_t)s.q[a] + (int64_t)s.r) >> L.F;
        if ((L.cyc >> a) & 1u) {
            if (hi - lo + 1 >= La) {
                lo = 0;
                hi = La - 1;
            }
        } else {
            if (lo < 0) lo = 0;
            if (hi > La - 1) hi = La - 1;
        }
        n *= hi >= lo ? (uint32_t)(hi - lo + 1) : 0u;
    }
    return n;
}

// Row j of the class table that starts at tb ((y, z) class cls): from the
// staged copy when it holds it, else from device memory.
template <bool TLDS>
__device__ __forceinline__ uint32_t row_word(const TabArgs& T, const uint32_t* tab_lds, uint32_t tb, uint32_t cls,
                                             uint32_t j) {
    if (TLDS) {
        if (T.lds_chunk == 0) return tab_lds[tb + j];
        if (j < T.lds_chunk) return tab_lds[cls * T.lds_chunk + j];
    }
    return T.rows[tb + j];
}

// (y, z) sub-cell class of a query (the row table it walks).
__device__ __forceinline__ uint32_t row_class(const LatArgs& L, const TabArgs& T, const uint32_t* f) {
    return (f[1] >> (L.F - T.s)) | ((f[2] >> (L.F - T.s)) << T.s);
}

// ---------------------------------------------------------------------------
// Rows of the walk

// Per lane, one x-row of cells: up to two object ranges to test (two when
// the run of cells wraps around a cyclic x axis), a range of objects in cells
// wholly inside the sphere (counted without reading them), and the number
// of cells of the row the sphere meets.
struct RowRef {
    uint32_t st0, cnt0, st1, cnt1;
    uint32_t ist, icnt;
    uint32_t kept;
    bool plain;  // one range (st1, cnt1): the run neither wraps nor has a wholly-inside part
};

// Per-axis distance from a position f inside the home cell to the farthest
// position of the cell at offset o along that axis.
__device__ __forceinline__ uint32_t axis_far(int o, uint32_t f, uint32_t F) {
    const uint32_t e = 1u << F;
    if (o > 0) return (((uint32_t)o + 1u) << F) - 1u - f;
    if (o < 0) return f + ((uint32_t)(-o) << F);
    return max(f, e - 1u - f);
}

// s^2 for s < 2^24: two 24-bit multiplies (low and high word) instead of a
// 64-bit multiply-add.
__device__ __forceinline__ uint64_t sq24(uint32_t s) {
    const uint32_t t = s & 0xFFFFFFu;
    return (uint64_t)t * t;
}

// floor(sqrt(v)) for v < 2^62.
// Below 2^41 (roots below 2^20.5): v in single precision (the high word is
// exact, the low word and the sum round once each: relative error at most
// 1.5 x 2^-24) and the hardware square root (within 1 ulp) give the root to
// within 0.25, so its truncation is the floor or one either side of it; two
// exact steps with 24-bit products settle it.
// Above: the hardware reciprocal square root in double precision (relative
// error about 2^-23) and one Newton step give the root to about 2^-45
// relative, well within one unit below 2^31; exact integer steps settle the
// floor.  (v = 0 takes the first branch.)
__device__ __forceinline__ uint32_t isqrt64(uint64_t v) {
    const uint32_t hi = (uint32_t)(v >> 32);
    uint32_t s;
    if (hi < (1u << 9)) {
        const float fv = __builtin_fmaf((float)hi, 4294967296.0f, (float)(uint32_t)v);
        s = (uint32_t)__builtin_amdgcn_sqrtf(fv);
        if (sq24(s) > v) --s;
        if (sq24(s + 1u) <= v) ++s;
    } else {
        const double d = (double)v;
        const double y = __builtin_amdgcn_rsq(d);
        double x = d * y;
        x = __builtin_fma(x, __builtin_fma(-x, 0.5 * y, 0.5), x);
        s = (uint32_t)x;
        if ((uint64_t)s * s > v) --s;
        if ((uint64_t)s * s > v) --s;
        if ((uint64_t)(s + 1u) * (s + 1u) <= v) ++s;
    }
    return s;
}

// Turn an unwrapped x-run [a, b] of the row starting at cell `base` (and its
// wholly-inside part [ia, ib], empty when ia > ib) into object ranges.  On a
// cyclic axis the run (shorter than the axis) may cross the world edge once:
// it is then two pieces and is tested whole; on a clipped axis it is clamped
// to the region.  Lanes with `live` false get empty ranges (their loads read
// the row start, always a valid index).
__device__ __forceinline__ RowRef row_ranges(const LatArgs& L, uint32_t base, int a, int b, int ia, int ib,
                                             bool live) {
    const int Lx = 1 << L.lg[0];
    int p0, p1, p2, p3;
    bool has_int = ia <= ib;
    bool wrap = false;
    if (L.cyc & 1u) {
        const bool lo_out = a < 0, hi_out = b >= Lx;
        wrap = lo_out || hi_out;
        // pieces in memory order when wrapped: [0, e0) then [s1, Lx)
        const int e0 = lo_out ? b + 1 : b - Lx + 1;
        const int s1 = lo_out ? a + Lx : a;
        ia = max(ia, a);
        ib = min(ib, b);
        has_int = has_int && !wrap && ia <= ib;
        p0 = wrap ? 0 : a;
        p1 = wrap ? e0 : (has_int ? ia : a);
        p2 = wrap ? s1 : (has_int ? ib + 1 : a);
        p3 = wrap ? Lx : b + 1;
    } else {
        a = max(a, 0);
        b = min(b, Lx - 1);
        live = live && a <= b;
        ia = max(ia, a);
        ib = min(ib, b);
        has_int = has_int && ia <= ib;
        p0 = a;
        p1 = has_int ? ia : a;
        p2 = has_int ? ib + 1 : a;
        p3 = b + 1;
    }
    if (!live) p0 = p1 = p2 = p3 = 0;
    const uint32_t* row = L.cs + base;
    // a plain run is one range [p0, p3): its middle bounds are needed only
    // when it wraps or has a wholly-inside part
    const uint32_t v0 = row[p0], v3 = row[p3];
    uint32_t v1 = v0, v2 = v0;
    if (wrap || has_int) {
        v1 = row[p1];
        v2 = row[p2];
    }
    RowRef r;
    r.st0 = v0;
    r.cnt0 = v1 - v0;
    r.st1 = v2;
    r.cnt1 = v3 - v2;
    r.ist = v1;
    r.icnt = has_int ? v2 - v1 : 0u;
    r.kept = (uint32_t)(wrap ? (p1 - p0) + (p3 - p2) : (p3 - p0));
    r.plain = !wrap && !has_int;
    return r;
}

// Cells in x order (objects inside each cell by x, cells of a row in x
// order): the objects of a plain run have increasing x, and those within the
// sphere's x-slab [lo_t, hi_t] on this row are one sub-range, found by
// two binary searches on x (interleaved, so that their loads overlap).  Only
// for rows with many objects, where the searches cost less than testing the
// objects outside the slab.
constexpr uint32_t kNarrowMin = 24;

__device__ __forceinline__ void narrow_x(const LatArgs& L, RowRef& r, uint32_t lo_t, uint32_t hi_t) {
    const uint32_t* xs = (const uint32_t*)L.pts;  // x of sorted position p at xs[4 p]
    uint32_t a = r.st1, na = r.cnt1, b = r.st1, nb = r.cnt1;
    while (na | nb) {
        if (na) {
            const uint32_t h = na >> 1;
            if (xs[4 * (a + h)] < lo_t) {
                a += h + 1;
                na -= h + 1;
            } else {
                na = h;
            }
        }
        if (nb) {
            const uint32_t h = nb >> 1;
            if (xs[4 * (b + h)] <= hi_t) {
                b += h + 1;
                nb -= h + 1;
            } else {
                nb = h;
            }
        }
    }
    r.st1 = a;
    r.cnt1 = b - a;
}

// Squared distance along one axis from the query to the nearest position of
// the cell at offset o: 0 for o = 0, else (|o| - 1) cells plus the distance
// to the shared face (up = e - f above, dn = f + 1 below).  A lower bound
// only (the callers keep a cell or a row when it is within the bound, and
// test its objects exactly): a distance of 2^24 units or more is taken as
// 2^24 - 1, so that the square takes 24-bit products.
__device__ __forceinline__ uint64_t axis_gap2(int o, uint32_t up, uint32_t dn, uint32_t F) {
    const uint32_t ao = (uint32_t)(o < 0 ? -o : o);
    const uint32_t g = o == 0 ? 0u : ((ao - 1u) << F) + (o > 0 ? up : dn);
    return sq24(min(g, 0xFFFFFFu));
}

// Row (oy, oz) of the sphere table: the cells it meets are those whose
// x-gap satisfies gx^2 <= bound^2 - gy^2 - gz^2 -- the exact test of Eq. 1
// solved for x, one contiguous run; the wholly-inside cells solve the same
// with the far distances (Section III.A, last paragraph).
__device__ __forceinline__ RowRef sphere_row(const LatArgs& L, const Query& s, uint32_t w, bool has, uint64_t bound2,
                                             bool interior) {
    const int oy = ((int)(w << 16)) >> 16, oz = ((int)w) >> 16;
    const uint32_t Ly = 1u << L.lg[1], Lz = 1u << L.lg[2];
    uint32_t ty = (uint32_t)((int)s.c[1] + oy), tz = (uint32_t)((int)s.c[2] + oz);
    bool live = has;
    if (L.cyc & 2u)
        ty &= Ly - 1u;
    else
        live = live && ty < Ly;
    if (L.cyc & 4u)
        tz &= Lz - 1u;
    else
        live = live && tz < Lz;
    const uint64_t gyz = axis_gap2(oy, s.up[1], s.dn[1], L.F) + axis_gap2(oz, s.up[2], s.dn[2], L.F);
    live = live && gyz <= bound2;
    const uint32_t X = isqrt64(live ? bound2 - gyz : 0u);
    const uint32_t fx = s.f[0];
    const int npos = (int)((X + fx) >> L.F);
    const int nneg = X > fx ? (int)((X - fx - 1u) >> L.F) + 1 : 0;
    int ia = 1, ib = 0;
    if (interior) {
        const uint32_t hy = axis_far(oy, s.f[1], L.F), hz = axis_far(oz, s.f[2], L.F);
        const uint64_t hyz = sq(hy) + sq(hz);
        const uint32_t Xi = isqrt64(hyz <= s.r2 ? s.r2 - hyz : 0u);
        if (hyz <= s.r2 && Xi >= fx && Xi + fx + 1u >= (1u << L.F)) {
            ib = (int)s.c[0] + (int)((Xi + fx + 1u) >> L.F) - 1;
            ia = (int)s.c[0] - (int)((Xi - fx) >> L.F);
        }
    }
    if (!live) {
        ty = 0;
        tz = 0;
    }
    const uint32_t base = (tz << (L.lg[0] + L.lg[1])) | (ty << L.lg[0]);
    RowRef rr = row_ranges(L, base, (int)s.c[0] - nneg, (int)s.c[0] + npos, ia, ib, live);
    if (L.xsorted && rr.plain && rr.cnt1 >= kNarrowMin && *L.xsorted)
        narrow_x(L, rr, s.q[0] > X ? s.q[0] - X : 0u, s.q[0] + X);
    return rr;
}

// Row e of the bounding cube (no test: the bin-lattice scans every cell).
__device__ __forceinline__ RowRef cube_row(const LatArgs& L, const Query& s, uint32_t e, bool has, double inv_ny) {
    if (!has) e = 0;
    const uint32_t iz = exact_div(e, s.nn[1], inv_ny);
    const uint32_t iy = e - iz * s.nn[1];
    uint32_t ty = (uint32_t)(s.lo[1] + (int32_t)iy), tz = (uint32_t)(s.lo[2] + (int32_t)iz);
    if (L.cyc & 2u) ty &= (1u << L.lg[1]) - 1u;
    if (L.cyc & 4u) tz &= (1u << L.lg[2]) - 1u;
    if (!has) {
        // lanes without a row read the first row (always a valid index)
        ty = 0u;
        tz = 0u;
    }
    const uint32_t base = (tz << (L.lg[0] + L.lg[1])) | (ty << L.lg[0]);
    return row_ranges(L, base, s.lo[0], s.lo[0] + (int)s.nn[0] - 1, 1, 0, has);
}

// Entry `ent` of the non-empty cell list (Section III.B): the cell's objects
// are one range, kept when the cell's nearest position is within the radius
// -- the rejection of cells that are too far, instead of the sphere's
// rejection of empty cells.  On a cyclic axis the cell's offset is taken to
// the nearest image, o in [-L/2, L/2); at o = -L/2 the image at +L/2 is as
// many cells away, and the nearer face of the two counts.
__device__ __forceinline__ RowRef list_row(const LatArgs& L, const Query& s, uint32_t ent, bool has, uint64_t bound2) {
    // lanes without an entry read entry 0 (the closing entry of an empty
    // list), always present
    const uint2 c = L.cells[has ? ent : 0u];
    const uint32_t end = L.cells[has ? ent + 1u : 0u].y;
    const uint32_t cc[3] = {c.x & ((1u << L.lg[0]) - 1u), (c.x >> L.lg[0]) & ((1u << L.lg[1]) - 1u),
                            c.x >> (L.lg[0] + L.lg[1])};
    uint64_t g2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int o = (int)cc[a] - (int)s.c[a];
        uint32_t up = s.up[a], dn = s.dn[a];
        if ((L.cyc >> a) & 1u) {
            const int La = 1 << L.lg[a];
            o = ((o + La / 2) & (La - 1)) - La / 2;
            if (La >= 2 && o == -(La / 2)) dn = min(up, dn);
        }
        g2 += axis_gap2(o, up, dn, L.F);
    }
    const bool keep = has && g2 <= bound2;
    RowRef r;
    r.st0 = c.y;
    r.cnt0 = keep ? end - c.y : 0u;
    r.st1 = c.y;
    r.cnt1 = 0u;
    r.ist = c.y;
    r.icnt = 0u;
    r.kept = keep ? 1u : 0u;
    r.plain = false;
    return r;
}

// Entry `ent` of the paper's tables (Section III.A), one cell: the unshaved
// table's entries below floor(d)^2 come first (ent < s.ncube), then the
// query's specialised table from s.tb.  Cells with b e >= thr -- b at or
// above d - 1 when thr = (r - e)^2 -- take the run-time test of Eq. 1 with
// the paper's per-axis distances (b_o cells plus the distance to the face,
// e - f up and f down); objects of the kept cell are then tested one by one.
__device__ __forceinline__ RowRef paper_row(const LatArgs& L, const TabArgs& T, const Query& s, uint32_t ent,
                                            bool has, uint64_t bound2, uint64_t thr2) {
    const uint32_t idx = ent < s.ncube ? T.p_lo[(size_t)64 * T.p_nb2] + ent : s.tb + (ent - s.ncube);
    const uint32_t w = has ? T.p_off[idx] : 0u;
    const uint64_t b2e = has ? (uint64_t)T.p_b2[idx] << (2 * L.F) : 0ull;
    const int o[3] = {((int)(w << 22)) >> 22, ((int)(w << 12)) >> 22, ((int)(w << 2)) >> 22};
    const uint32_t e = 1u << L.F;
    bool live = has;
    uint32_t t[3];
    uint64_t g2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const uint32_t La = 1u << L.lg[a];
        uint32_t v = (uint32_t)((int)s.c[a] + o[a]);
        if ((L.cyc >> a) & 1u)
            v &= La - 1u;
        else
            live = live && v < La;
        t[a] = v;
        const uint32_t ao = (uint32_t)(o[a] < 0 ? -o[a] : o[a]);
        const uint64_t g = o[a] == 0 ? 0ull : ((uint64_t)(ao - 1u) << L.F) + (o[a] > 0 ? e - s.f[a] : s.f[a]);
        g2 += g * g;
    }
    if (b2e >= thr2 && g2 > bound2) live = false;
    if (!live) t[0] = t[1] = t[2] = 0u;
    const uint32_t cell = pack_cell(L, t[0], t[1], t[2]);
    const uint32_t st = L.cs[cell];
    RowRef r;
    r.st0 = st;
    r.cnt0 = live ? L.cs[cell + 1] - st : 0u;
    r.st1 = st;
    r.cnt1 = 0u;
    r.ist = st;
    r.icnt = 0u;
    r.kept = live ? 1u : 0u;
    r.plain = false;
    return r;
}

// Minimum-image squared distance of an object to the centre: on a cyclic
// axis ((p - q + W/2) mod W) - W/2; on a clipped axis plain p - q (both below
// 2^30, so the difference fits an int).
struct AxisWrap {
    uint32_t half[3];
    uint32_t mask[3];
};

__device__ __forceinline__ AxisWrap axis_wrap(const LatArgs& L) {
    AxisWrap w;
    for (int a = 0; a < 3; ++a) {
        if ((L.cyc >> a) & 1u) {
            const uint32_t W = 1u << (L.lg[a] + L.F);
            w.half[a] = W >> 1;
            w.mask[a] = W - 1u;
        } else {
            w.half[a] = 0u;
            w.mask[a] = 0xFFFFFFFFu;
        }
    }
    return w;
}

__device__ __forceinline__ uint64_t obj_dist2(const AxisWrap& w, const Query& s, const uint4& P) {
    const uint32_t pv[3] = {P.x, P.y, P.z};
    uint64_t d2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int32_t dd = (int32_t)(((pv[a] - s.q[a]) + w.half[a]) & w.mask[a]) - (int32_t)w.half[a];
        d2 += (uint64_t)((int64_t)dd * dd);
    }
    return d2;
}

// ---------------------------------------------------------------------------
// Candidate distribution: each lane holds two object ranges [st0, st0+cnt0)
// and [st1, st1+cnt1); every object becomes one slot, 64 slots per step.
// visit(active, position, record) returns true to stop (uniformly).

template <typename V>
__device__ __forceinline__ bool for_candidates(const LatArgs& L, uint32_t st0, uint32_t cnt0, uint32_t st1,
                                               uint32_t cnt1, uint32_t* own, uint32_t& total_out, V&& visit) {
    const uint32_t lane = lane_id();
    const uint32_t tl = cnt0 + cnt1;
    const uint32_t incl = scan_add(tl);
    const uint32_t total = lane_val(incl, 63);
    total_out += total;
    if (total == 0) return false;
    const uint32_t excl = incl - tl;
    const uint32_t smx0 = st0 - excl;
    const uint32_t bnd = excl + cnt0;
    const uint32_t smx1 = st1 - bnd;
    // slot cb + lane: mark where each lane's range starts inside the step's
    // 64 slots, then a max-scan hands every slot to the lane that owns it (a
    // step past the end marks nothing: lane 0 stands in)
    auto locate = [&](uint32_t cb, uint32_t& p) -> bool {
        wave_sync();
        own[lane] = 0;
        wave_sync();
        if (tl > 0 && excl < cb + 64 && incl > cb) own[excl > cb ? excl - cb : 0] = lane + 1;
        wave_sync();
        const uint32_t o = max(scan_max(own[lane]), 1u) - 1u;
        const uint32_t g = cb + lane;
        const uint32_t b = bperm(bnd, o);
        const uint32_t p0 = bperm(smx0, o) + g;
        const uint32_t p1 = bperm(smx1, o) + g;
        p = g < b ? p0 : p1;
        return g < total;
    };
    // two register sets taken in turn: the step after the one being visited
    // is already loading (lanes past the end load record 0, present whenever
    // a candidate is, and visit nothing)
    uint32_t pa = 0, pb = 0;
    bool aa = locate(0, pa), ab = false;
    uint4 PA = L.pts[aa ? pa : 0u], PB = PA;
    for (uint32_t cb = 0; cb < total; cb += 128) {
        ab = locate(cb + 64, pb);
        PB = L.pts[ab ? pb : 0u];
        if (visit(aa, pa, PA)) return true;
        if (cb + 64 >= total) break;
        aa = locate(cb + 128, pa);
        PA = L.pts[aa ? pa : 0u];
        if (visit(ab, pb, PB)) return true;
    }
    return false;
}

// Walk the query's rows: sphere-table rows or bounding-cube rows, 64 per
// step, one per lane.  When objects outside the region may be within r, the
// outside cell (Section II.B: every such object lives in one cell) is a
// leading pseudo-row of the first step.  on_step(row) returns true to stop.
// bound2_now() is re-read before every step (top-M shrinks it); KEY_STOP
// enables the cut-off on sorted row keys; `interior` marks the cells wholly
// inside the sphere (count pass).
// The steps of 64 entries a wavefront takes start at `first` and follow
// every `stride` entries (a block of W waves walks one row with first =
// 64 w, stride = 64 W; a lone wave takes them all).
template <int METHOD, bool TLDS, bool KEY_STOP, typename B, typename S>
__device__ __forceinline__ void walk(const LatArgs& L, const TabArgs& T, const uint32_t* tab_lds, const Query& s,
                                     bool interior, uint32_t& walked, B&& bound2_now, S&& on_step,
                                     uint32_t first = 0, uint32_t stride = 64) {
    const uint32_t lane = lane_id();
    const uint32_t pre = (s.flags & F_OUTSIDE) ? 1u : 0u;
    const bool sphere = METHOD == kSphere || ((METHOD == kEither || METHOD == kPaper) && (s.flags & F_SPHERE));
    const uint32_t nent = sphere ? s.tend : s.nn[1] * s.nn[2];
    const uint32_t total = nent + pre;
    const uint32_t rcls = TLDS ? row_class(L, T, s.f) : 0u;
    // entry index of this lane's row in the current step (pseudo-row: ~0)
    uint32_t ent = lane - pre + first;
    uint32_t nxt = 0;
    if (METHOD != kPaper && sphere && ent < nent) nxt = row_word<TLDS>(T, tab_lds, s.tb, rcls, ent);
    const double inv_ny = (!sphere && s.nn[1]) ? 1.0 / (double)s.nn[1] : 0.0;
    for (uint32_t base = first; base < total; base += stride, ent += stride) {
        const bool is_out = pre && base == 0 && lane == 0;
        RowRef r;
        if (METHOD == kPaper && sphere) {
            const uint64_t bound2 = bound2_now();
            // entries are sorted by b^2, and b e is below every cell's
            // distance: once b^2 e^2 exceeds the bound nothing further can
            // hold anything closer
            if (KEY_STOP && base > 0) {
                const uint32_t j = base - pre;
                const uint32_t idx = j < s.ncube ? T.p_lo[(size_t)64 * T.p_nb2] + j : s.tb + (j - s.ncube);
                if (((uint64_t)uni(T.p_b2[idx]) << (2 * L.F)) > bound2) break;
            }
            // the run-time test from b >= d - 1 on (every cell when d < 1)
            const uint32_t e = 1u << L.F;
            const uint32_t rt = uni(isqrt64(bound2));
            const uint64_t thr2 = rt > e ? sq(rt - e) : 0ull;
            r = paper_row(L, T, s, ent, ent < nent, bound2, thr2);
        } else if (METHOD == kSphere || (METHOD == kEither && sphere)) {
            const uint64_t bound2 = bound2_now();
            // rows are sorted by key: once the key exceeds the bound no
            // further row can hold anything closer (the first row's key is 0)
            if (KEY_STOP && base > 0 && uni64((uint64_t)T.rkey[s.tb + base - pre]) > bound2) break;
            const uint32_t w = nxt;
            if (ent + stride < nent) nxt = row_word<TLDS>(T, tab_lds, s.tb, rcls, ent + stride);
            r = sphere_row(L, s, w, ent < nent, bound2, interior);
        } else if (s.flags & F_LIST) {
            r = list_row(L, s, ent, ent < nent, bound2_now());
        } else {
            r = cube_row(L, s, ent, ent < nent, inv_ny);
        }
        if (is_out) {
            r.st0 = L.cs[L.ncells];
            r.cnt0 = L.cs[L.ncells + 1] - r.st0;
            r.cnt1 = 0u;
            r.icnt = 0u;
            r.kept = 0u;
        }
        walked += min(64u, total - base) - (base == 0 ? pre : 0u);
        if (on_step(r)) return;
    }
}

// ---------------------------------------------------------------------------
// Query scheduling: plain (each wave owns a fixed slice of `tile` queries,
// XCD-aware block order) or persistent (per-XCD work queues).

// Persistent grabs shrink with the work: about two per resident wave, at
// least `tmin` and at most A.tile (64 for the lists), so that a short batch
// or list of heavy queries is shared out instead of landing on a few waves,
// and a long one does not pay an atomic per query.
template <typename F>
__device__ __forceinline__ void for_each_range(uint32_t Q, const QArgs& A, uint32_t* queues, F&& f,
                                               uint32_t tmin = 1u) {
    if (Q == 0) return;
    const uint32_t lane = lane_id();
    const uint32_t wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t tmax = A.list ? 64u : A.tile;
    const uint32_t tile =
        A.persistent ? max(tmin, min(tmax, (uint32_t)((uint64_t)Q / ((uint64_t)gridDim.x * nw * 2u)))) : A.tile;
    // plain: consecutive block ids go round-robin over the 8 XCDs; give each
    // XCD a contiguous range of slices so neighbouring queries share its L2.
    // persistent: SPHIDX_NQUEUE queues, each over a contiguous range of
    // queries and served by blocks of one XCD (several queues per XCD, so
    // that fewer waves share each counter); a wave drains its own queue, then
    // looks at all the others at once and moves to the first with work left,
    // and stops when none has any.  Queues only drain, so every wave stops.
    uint32_t x = blockIdx.x % (A.persistent ? SPHIDX_NQUEUE : SPHIDX_NXCD);
    bool first = true;
    for (;;) {
        uint32_t b = 0, e = 0;
        if (!A.persistent) {
            if (!first) break;
            const uint32_t G = gridDim.x, bi = blockIdx.x;
            const uint32_t full = G / SPHIDX_NXCD, rem = G % SPHIDX_NXCD;
            const uint32_t lb = x * full + min(x, rem) + bi / SPHIDX_NXCD;
            const uint64_t q0 = ((uint64_t)lb * nw + wave) * tile;
            b = (uint32_t)min(q0, (uint64_t)Q);
            e = (uint32_t)min(q0 + tile, (uint64_t)Q);
        } else {
            const uint32_t qs = (uint32_t)(((uint64_t)x * Q) / SPHIDX_NQUEUE);
            const uint32_t qe = (uint32_t)(((uint64_t)(x + 1) * Q) / SPHIDX_NQUEUE);
            uint32_t* qc = queues + x * SPHIDX_QSTRIDE;
            uint32_t t = 0;
            if (lane == 0) {
                // an exhausted queue is skipped with a plain read, not an atomic
                t = __hip_atomic_load(qc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((uint64_t)qs + t < qe) t = atomicAdd(qc, tile);
            }
            t = uni(t);
            if ((uint64_t)qs + t >= qe) {
                // lane l reads queue x + 1 + l
                bool left = false;
                if (lane + 1u < SPHIDX_NQUEUE) {
                    const uint32_t y = (x + 1u + lane) % SPHIDX_NQUEUE;
                    const uint32_t ys = (uint32_t)(((uint64_t)y * Q) / SPHIDX_NQUEUE);
                    const uint32_t ye = (uint32_t)(((uint64_t)(y + 1) * Q) / SPHIDX_NQUEUE);
                    const uint32_t ty =
                        __hip_atomic_load(queues + y * SPHIDX_QSTRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    left = (uint64_t)ys + ty < ye;
                }
                const uint64_t m = __ballot(left);
                if (m == 0) break;
                x = (x + 1u + (uint32_t)__builtin_ctzll(m)) % SPHIDX_NQUEUE;
                continue;
            }
            b = qs + t;
            e = (uint32_t)min((uint64_t)qe, (uint64_t)qs + t + tile);
        }
        first = false;
        if (b < e) f(b, e);
    }
}

template <typename F>
__device__ __forceinline__ void for_each_query(uint32_t Q, const QArgs& A, uint32_t* queues, F&& f) {
    for_each_range(Q, A, queues, [&](uint32_t b, uint32_t e) {
        for (uint32_t qi = b; qi < e; ++qi) f(qi);
    });
}

// Stage the row table in LDS (shared by the block's waves): the whole table,
// or, in chunks, the first lds_chunk rows of every (y, z) class -- the rows
// nearest the centre, which every query of the class walks first.
template <bool TLDS>
__device__ __forceinline__ const uint32_t* stage_table(const TabArgs& T, char* smem) {
    if (!TLDS) return nullptr;
    uint32_t* t = (uint32_t*)smem;
    if (T.lds_chunk == 0) {
        for (uint32_t i = threadIdx.x; i < T.total; i += blockDim.x) t[i] = T.rows[i];
    } else {
        const uint32_t n = T.nrcls * T.lds_chunk;
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
            const uint32_t c = i / T.lds_chunk, j = i - c * T.lds_chunk;
            const uint32_t b = T.cstart[c];
            t[i] = b + j < T.cstart[c + 1] ? T.rows[b + j] : 0u;
        }
    }
    __syncthreads();
    return t;
}

template <bool TLDS>
__device__ __forceinline__ size_t table_lds_bytes(const TabArgs& T) {
    if (!TLDS) return 0;
    const size_t words = T.lds_chunk ? (size_t)T.nrcls * T.lds_chunk : (size_t)T.total;
    return (words * 4 + 15) & ~(size_t)15;
}



// ---------------------------------------------------------------------------
// Ordering a row by (dist^2, id) in LDS.

__device__ __forceinline__ void store_sorted(const QArgs& A, const uint64_t* td, const uint32_t* ti, uint32_t n,
                                             int64_t dst) {
    for (uint32_t t = lane_id(); t < n; t += 64) {
        A.out_ids[dst + t] = ti[t];
        if (A.out_d2) A.out_d2[dst + t] = (int64_t)td[t];
    }
}

// Sort the n <= cap pairs (td, ti) of one row by (dist^2, id) and store them
// at dst.  Every pair has dist^2 <= r2, so the bucket
// floor(n * dist^2 / r2) (float arithmetic: monotone in dist^2) never puts a
// larger distance in an earlier bucket; a histogram, its prefix sum and a
// scatter order the buckets, and each pair's place inside its bucket (about
// one pair per bucket) is the number of smaller pairs there.
__device__ __forceinline__ uint32_t sort_bucket(uint64_t d2, float scale, uint32_t n) {
    return min((uint32_t)((float)d2 * scale), n - 1u);
}

__device__ void bucket_sort_store(const uint64_t* td, const uint32_t* ti, uint64_t* sd, uint32_t* si, uint32_t* hist,
                                  uint32_t n, uint64_t r2, uint32_t* dst_ids, int64_t* dst_d2) {
    const uint32_t lane = lane_id();
    if (n == 0) return;
    const float scale = r2 > 0 ? (float)n / (float)r2 : 0.0f;
    for (uint32_t t = lane; t < n; t += 64) hist[t] = 0u;
    wave_sync();
    uint32_t slot[4];  // n <= 256 = 4 pairs per lane
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t t = lane + 64u * k;
        if (t < n) slot[k] = atomicAdd(&hist[sort_bucket(td[t], scale, n)], 1u);
    }
    wave_sync();
    // exclusive prefix over the buckets, each lane owning a run of them
    const uint32_t per = (n + 63u) >> 6;
    const uint32_t b0 = lane * per;
    uint32_t sum = 0;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) sum += hist[b0 + k];
    uint32_t run = scan_add(sum) - sum;
    wave_sync();
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) {
            const uint32_t c = hist[b0 + k];
            hist[b0 + k] = run;
            run += c;
        }
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t t = lane + 64u * k;
        if (t < n) {
            const uint32_t dst = hist[sort_bucket(td[t], scale, n)] + slot[k];
            sd[dst] = td[t];
            si[dst] = ti[t];
        }
    }
    wave_sync();
    for (uint32_t t = lane; t < n; t += 64) {
        const uint64_t d = sd[t];
        const uint32_t id = si[t];
        const uint32_t b = sort_bucket(d, scale, n);
        const uint32_t lo = hist[b], hi = b + 1 < n ? hist[b + 1] : n;
        uint32_t rank = lo;
        for (uint32_t j = lo; j < hi; ++j) rank += key_less(sd[j], si[j], d, id) ? 1u : 0u;
        dst_ids[rank] = id;
        if (dst_d2) dst_d2[rank] = (int64_t)d;
    }
}

// ---------------------------------------------------------------------------
// Top-M searches in registers

// First bound of a top-M search: the radius expected to hold `target`
// objects (K-NN rows: the density around the centre, the home cell's count
// with the lattice mean as a floor; radius rows of `rowlen`: the row's own
// mean density over its ball), never above the cap; the whole cap for the
// bounding cube and the cell list, which are scanned whole anyway.  A search
// grows it and starts again whenever fewer than M lie within it.
__device__ __forceinline__ uint64_t first_bound(const LatArgs& L, const Query& s, uint32_t target, uint32_t rowlen) {
    if (!(s.flags & F_SPHERE)) return s.r2;
    const float e = (float)(1u << L.F);
    float rho;
    if (s.flags & F_KBOUND) return min(s.r2, sq(s.kbr));
    if (s.flags & F_KNN) {
        const uint32_t home = pack_cell(L, s.c[0], s.c[1], s.c[2]);
        const float dens = fmaxf((float)L.n / (float)(L.ncells ? L.ncells : 1u), (float)(L.cs[home + 1] - L.cs[home]));
        rho = 1.25f * e * cbrtf(0.2387f * (float)target / fmaxf(dens, 1e-6f));
    } else {
        rho = 1.1f * (float)s.r * cbrtf((float)target / (float)rowlen);
    }
    return rho >= (float)s.r ? s.r2 : min(s.r2, (uint64_t)((double)rho * (double)rho));
}

// The M <= 64 nearest pairs (dist^2, id) of query s above the pair (ld, li)
// when has_lower, within the cap: lane i ends with the i-th in (rd, ri), and
// the count found, min(M, pairs within the cap), is returned.  The bound
// starts at B, shrinks to the M-th distance once M are held (Section II.A,
// K nearest) and, when fewer than M lie within it, grows by half and the
// walk starts again.  A few new pairs are inserted one by one (place = pairs
// ahead of it, the rest move up one lane); a large batch is sorted and
// merged (the 64 smallest of list and batch, as a bitonic sequence, then
// sorted).
template <int METHOD, bool TLDS>
__device__ __forceinline__ uint32_t topm_registers(const LatArgs& L, const TabArgs& T, const uint32_t* tab_lds,
                                                   const Query& s, const AxisWrap& aw, uint32_t* own, uint32_t M,
                                                   uint64_t B, bool has_lower, uint64_t ld, uint32_t li, uint64_t& rd,
                                                   uint32_t& ri, uint32_t* stat = nullptr) {
    const uint32_t lane = lane_id();
    rd = kMaxD2;
    ri = kMaxId;
    uint64_t kd = kMaxD2;
    uint32_t kid = kMaxId, held = 0, cand2 = 0, walked2 = 0, kept2 = 0;
    auto visit_r = [&](bool act, uint32_t p, const uint4& P) -> bool {
        const uint64_t d2 = obj_dist2(aw, s, P);
        const uint32_t id = P.w;
        bool cv = act && d2 <= B && p != s.self;
        if (cv && has_lower) cv = key_less(ld, li, d2, id);
        if (cv && held >= M) cv = key_less(d2, id, kd, kid);
        uint64_t qm = __ballot(cv);
        if (qm == 0) return false;
        const uint32_t nb = (uint32_t)__popcll(qm);
        if (nb > 6) {
            uint64_t cd = cv ? d2 : kMaxD2;
            uint32_t ci = cv ? id : kMaxId;
            wave_sort64(cd, ci);
            const uint64_t xd = shfl64(cd, 63u - lane);
            const uint32_t xi = __shfl(ci, 63u - lane);
            if (key_less(xd, xi, rd, ri)) {
                rd = xd;
                ri = xi;
            }
            wave_bitonic_clean64(rd, ri);
            held = min(held + nb, 64u);
        } else {
            while (qm) {
                const uint32_t j = (uint32_t)__builtin_ctzll(qm);
                qm &= qm - 1ull;
                const uint64_t nd = lane_val64(d2, j);
                const uint32_t ni = lane_val(id, j);
                if (held >= M && !key_less(nd, ni, kd, kid)) continue;
                const uint32_t pos = (uint32_t)__popcll(__ballot(key_less(rd, ri, nd, ni)));
                const uint32_t below = lane ? lane - 1u : 0u;
                const uint64_t sd = shfl64(rd, below);
                const uint32_t si = __shfl(ri, below);
                if (lane > pos) {
                    rd = sd;
                    ri = si;
                } else if (lane == pos) {
                    rd = nd;
                    ri = ni;
                }
                held = min(held + 1u, 64u);
                if (held >= M) {
                    kd = lane_val64(rd, M - 1u);
                    kid = lane_val(ri, M - 1u);
                }
            }
        }
        if (held >= M) {
            kd = lane_val64(rd, M - 1u);
            kid = lane_val(ri, M - 1u);
        }
        return false;
    };
    for (;;) {
        walk<METHOD, TLDS, true>(L, T, tab_lds, s, false, walked2, [&]() { return held >= M ? kd : B; },
                                 [&](const RowRef& r) -> bool {
            kept2 += r.kept;
            return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand2, visit_r);
        });
        if (held >= M || B >= s.r2) break;
        B = min(s.r2, B + B + (B >> 2) + 1u);  // radius x1.5
        held = 0;
        rd = kMaxD2;
        ri = kMaxId;
        kd = kMaxD2;
        kid = kMaxId;
    }
    if (stat) {
        // per-query statistics, every walk of the search included
        const uint32_t k2 = wave_sum(kept2);
        if (lane == 0) {
            stat[0] += walked2;
            stat[1] += k2;
            stat[2] += cand2;
        }
    }
    return min(held, M);
}

// ---------------------------------------------------------------------------
// Pass 0: row sizes

// A row that the count pass could not keep: on the big list when it is one for
// the block-per-row and top-M kernels (K-NN rows, radius rows longer than a
// wavefront's buffer), else on the walk list of the write kernel.  (One lane.
// A wavefront that only passes such rows on costs as much as one that walks a
// short row: 10,000 of them on the walk list took the write kernel 127 us.
// The fallback list's rows stay on the walk list: its write kernel passes on
// what it does not keep.)
__device__ __forceinline__ void list_row_again(const QArgs& A, uint32_t qi, bool big) {
    if (big)
        A.bigq[atomicAdd(A.big_count, 1u)] = qi;
    else
        A.walkq[atomicAdd(A.walk_count, 1u)] = qi;
}

// Queue sets of the work counters.
constexpr int kQCount = 0, kQWrite = 1, kQTopm = 2, kQFbCount = 3, kQFbWrite = 4, kQWalk = 5, kQExtra = 6;
// the count pass's last list (rows the second grouped round left) takes the
// fallback write set, which only the write pass uses and clears
constexpr int kQExtra2 = kQFbWrite;
// Longest radius row the block-per-row kernel orders in LDS (12 bytes per pair).
constexpr uint32_t kLongCap = 3072;

__device__ __forceinline__ uint32_t* queue_set(const QArgs& A, int set) {
    return A.queues + (size_t)set * SPHIDX_NQUEUE * SPHIDX_QSTRIDE;
}

// Rows of at most 64 pairs whose key fits one 64-bit word: with id < 2^idbits
// and dist^2 < 2^(64 - idbits), (dist^2 << idbits) | id orders exactly as
// (dist^2, id) and is unique, so a pair's place is the number of smaller
// keys.  One pair per lane; the keys are read back as LDS broadcasts.
__device__ void sort_small_store(const uint64_t* td, const uint32_t* ti, uint64_t* ck, uint32_t n, uint32_t idbits,
                                 uint32_t* dst_ids, int64_t* dst_d2) {
    const uint32_t lane = lane_id();
    uint64_t d = 0, k = ~0ull;
    uint32_t id = 0;
    if (lane < n) {
        d = td[lane];
        id = ti[lane];
        k = (d << idbits) | id;
    }
    ck[lane] = k;  // lanes past n: the largest key, padding for the paired reads
    wave_sync();
    uint32_t rank = 0;
    for (uint32_t j = 0; j < n; j += 2) {
        const ulonglong2 p = *(const ulonglong2*)(ck + j);
        rank += (p.x < k ? 1u : 0u) + (p.y < k ? 1u : 0u);
    }
    if (lane < n) {
        dst_ids[rank] = id;
        if (dst_d2) dst_d2[rank] = (int64_t)d;
    }
    wave_sync();
}

// Order the n <= cap pairs of one row by (dist^2, id) and store them at dst.
__device__ __forceinline__ void sort_row_store(const uint64_t* td, const uint32_t* ti, uint64_t* sd, uint32_t* si,
                                               uint32_t* hist, uint32_t n, uint64_t r2, uint32_t idbits,
                                               uint32_t* dst_ids, int64_t* dst_d2) {
    const uint32_t r2bits = r2 ? 64u - (uint32_t)__builtin_clzll(r2) : 0u;
    if (n <= 64 && r2bits + idbits <= 64)
        sort_small_store(td, ti, sd, n, idbits, dst_ids, dst_d2);
    else
        bucket_sort_store(td, ti, sd, si, hist, n, r2, dst_ids, dst_d2);
}

// FROM_LIST: a query list (the sphere method's fallback queries, scanned with
// the bounding cube).  STASH: radius rows of at most sort_cap hits are also
// collected, sorted and kept in the workspace's stash, so that the write pass
// only copies them into place; other rows go to the walk list.  KSTASH (with
// STASH): K-NN rows of K <= 64 are searched here, top-K in registers, and
// kept the same way, so that no later pass walks them again.
template <int METHOD, bool TLDS, bool FROM_LIST, bool STASH, bool KSTASH>
__global__ __launch_bounds__(256) void count_kernel(LatArgs L, TabArgs T, QArgs A) {
    extern __shared__ __align__(16) char smem[];
    if (KSTASH && !FROM_LIST && A.group == kGroupSampled && !left_sparse(A)) return;  // taken in groups
    const uint32_t* tab_lds = stage_table<TLDS>(T, smem);
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t cap = A.sort_cap;
    char* wb = smem + table_lds_bytes<TLDS>(T) + (size_t)wave * (STASH ? (size_t)cap * 28 + 256 : 256);
    uint64_t* td = (uint64_t*)wb;
    uint64_t* sd = td + cap;
    uint32_t* ti = (uint32_t*)(sd + cap);
    uint32_t* si = ti + cap;
    uint32_t* hist = si + cap;
    uint32_t* own = STASH ? hist + cap : (uint32_t*)wb;
    const AxisWrap aw = axis_wrap(L);
    const uint32_t lane = lane_id();
    const uint32_t nq = FROM_LIST ? uni(*A.list_count) : A.Q;
    // this wave's stash chunk [cur, lim) in its region; `dry` once the
    // region is used up
    const uint32_t region = blockIdx.x % SPHIDX_NREGION;
    uint32_t cur = 0, lim = 0;
    bool dry = false;
    const uint32_t idbits = L.n > 1 ? 32u - (uint32_t)__builtin_clz(L.n - 1u) : 0u;  // ids are below n
    // room for n more stash elements in this wave's chunk, grabbing a new
    // chunk of the region when needed; false once the region is used up
    auto stash_room = [&](uint32_t n) -> bool {
        if (cur + n <= lim) return true;
        if (dry) return false;
        const uint32_t grab = max(A.stash_chunk, n);
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(A.stash_ctr + region * SPHIDX_QSTRIDE, grab);
        t = uni(t);
        if ((uint64_t)t + grab <= A.stash_region) {
            cur = region * A.stash_region + t;
            lim = cur + grab;
            return true;
        }
        dry = true;
        return false;
    };
    for_each_query(nq, A, queue_set(A, FROM_LIST ? (int)A.list_set : kQCount), [&](uint32_t ti_) {
        const uint32_t qi = FROM_LIST ? uni(A.list[ti_]) : ti_;
        const Query s = load_query(L, A, qi);
        if ((METHOD == kSphere || METHOD == kPaper) && (s.flags & F_VALID) && !(s.flags & F_SPHERE))
            return;  // fallback list
        if (!FROM_LIST && (s.flags & F_LONG)) return;  // counted one block per row
        const bool knn = s.flags & F_KNN;
        if (KSTASH && knn && (s.flags & F_VALID) && s.k <= 64u) {
            // the row itself: lane i ends with the i-th nearest
            uint64_t rd;
            uint32_t ri;
            uint32_t* stp = A.stats ? A.stats + 4 * (size_t)s.row : nullptr;
            const uint32_t got = topm_registers<METHOD, TLDS>(L, T, tab_lds, s, aw, own, s.k,
                                                               first_bound(L, s, s.k, 0u), false, 0ull, 0u, rd, ri,
                                                               stp);
            if (stp) {
                const uint32_t nc = cube_cells(L, s);
                if (lane == 0) stp[3] = nc;
            }
            if (lane == 0) A.row_ptr[s.row] = (int64_t)got;
            uint32_t off = 0u;  // empty rows: nothing to copy
            if (got > 0) {
                if (stash_room(got)) {
                    if (lane < got) {
                        A.stash_ids[cur + lane] = ri;
                        if (A.stash_d2) A.stash_d2[cur + lane] = (int64_t)rd;
                    }
                    off = cur;
                    cur += got;
                } else {
                    off = kMaxId;
                    if (lane == 0) list_row_again(A, qi, !(FROM_LIST && METHOD == kCube));
                }
            }
            if (lane == 0) A.soff[s.row] = off;
            return;
        }
        uint32_t hits = 0, inner = 0, kept = 0, cand = 0, walked = 0;
        uint64_t dmax = 0;  // K-NN: the largest dist^2 among the hits so far
        bool self_inner = false;
        auto visit = [&](bool act, uint32_t p, const uint4& P) -> bool {
            const uint64_t d2 = obj_dist2(aw, s, P);
            const bool hit = act && d2 <= s.r2 && p != s.self;
            if (knn && hit) dmax = max(dmax, d2);
            const uint64_t hm = __ballot(hit);
            if (STASH && hit) {
                const uint32_t slot = hits + lanes_below(hm);
                if (slot < cap) {
                    td[slot] = d2;
                    ti[slot] = P.w;
                }
            }
            hits += (uint32_t)__popcll(hm);
            return knn && hits >= s.k;
        };
        auto on_row = [&](const RowRef& r) -> bool {
            kept += r.kept;
            // cells wholly inside: counted without reading objects; note when
            // the excluded own object was among them
            if (r.icnt && s.self - r.ist < r.icnt) self_inner = true;
            inner += r.icnt;
            return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand, visit);
        };
        if (s.flags & F_VALID) {
            walk<METHOD, TLDS, false>(L, T, tab_lds, s, !STASH && !knn && A.interior, walked,
                                      [&]() { return s.r2; }, on_row);
            uint32_t total = hits + wave_sum(inner);
            if (__ballot(self_inner) != 0) total -= 1;
            if (knn && (s.flags & F_SPHERE) && total >= s.k) {
                // the walk found K objects within the largest of their
                // distances: that radius (rounded up) bounds the K-th
                // distance, and the write pass's top-K starts from it
                const uint32_t rb = (uint32_t)min((double)s.r, ceil(sqrt((double)dmax)) + 1.0);
                const uint32_t rbm = lane_val(scan_max(rb), 63);
                if (lane == 0) {
                    uint32_t* dw = (uint32_t*)(A.desc + 4 * (size_t)qi);
                    dw[12] = rbm;
                    dw[6] = s.flags | F_KBOUND;
                }
            }
            if (knn && total > s.k) total = s.k;
            hits = total;
        }
        if (lane == 0) A.row_ptr[s.row] = (int64_t)hits;
        if (STASH) {
            uint32_t off = 0u;  // empty rows: nothing to copy
            if ((s.flags & F_VALID) && hits > 0) {
                const bool ok = !knn && hits <= cap && stash_room(hits);
                if (ok) {
                    wave_sync();
                    sort_row_store(td, ti, sd, si, hist, hits, s.r2, idbits, A.stash_ids + cur,
                                   A.stash_d2 ? A.stash_d2 + cur : nullptr);
                    wave_sync();
                    off = cur;
                    cur += hits;
                } else {
                    off = kMaxId;
                    if (lane == 0) list_row_again(A, qi, (knn || hits > cap) && !(FROM_LIST && METHOD == kCube));
                }
            }
            if (lane == 0) A.soff[s.row] = off;
        }
        if (A.stats) {
            const uint32_t kept_all = wave_sum(kept);
            const uint32_t ncube = (s.flags & F_VALID) ? cube_cells(L, s) : 0u;
            if (lane == 0) {
                // (added to: a grouped count may have walked the query first)
                uint32_t* stp = A.stats + 4 * (size_t)s.row;
                stp[0] += walked;
                stp[1] += kept_all;
                stp[2] += cand;
                stp[3] = ncube;
            }
        }
    });
}

// ---------------------------------------------------------------------------
// Pass 0, radius queries in groups: a wavefront takes kGroup consecutive
// queries and spreads all their table rows over its lanes, 64 rows per
// step, and all their candidate objects, 64 per step, so that short rows
// and small radii fill whole steps.  Hits of the group are collected as
// one 64-bit key (query slot, dist^2, id) each, and one bucket sort orders
// the group's rows together; with the stash they are kept in one chunk.
// K-NN queries (the KNN variant) take part as radius rows at their first
// search radius and keep the first K.  Queries it does not take (K-NN of
// large K or off the sphere tables, keys that would not fit 64 bits, rows
// short of K inside the first radius) go to the extra list for the
// one-query-per-wave kernel.  The list-driven K-NN variant is the second
// round over that list: a K-NN row short of K inside its first radius is
// searched again in groups at the larger radius the first round wrote into
// its descriptor from the count it saw (the cap at most); what that round
// does not take goes on to the one-query-per-wave kernel.

constexpr uint32_t kGroup = 8, kGroupBits = 3;
// hit buffer keys and rows per group, in eighths of sort_cap
constexpr uint32_t kRowEighths = 6;
constexpr uint32_t kMaxHitCap = 256 * kHitEighths / 8;
// The group's hit buffer holds sort_cap keys, and a group ends before its
// rows would exceed 3/4 of sort_cap.  When the hits overflow the buffer the
// group keeps its leading queries whose hits fit (hits arrive query by
// query), and the next group starts at the first query left out and walks
// it again; the wave's row budget shrinks to what fitted and grows back by
// an eighth per group that fits, so that dense regions do not repeat the
// waste.  Only a query whose own hits exceed the buffer is left to the
// write pass.  A smaller buffer buys occupancy (LDS) at the price of more
// overflows.  On the uneven-radius workload (1 M queries, ms per step):
// 2 x sort_cap keys, an overflowing group left whole to the write pass,
// 1.154; 1.5 x 1.092, 1.25 x 1.062; keeping the leading queries, 1.25 x
// 1.028, 1 x 1.006 (0.988 within 80 VGPRs), 7/8 x 1.039; rows up to 7/8 of
// sort_cap at 1 x, 1.004.
// A K-NN slot counts for its expected hits, 9/8 knn_target(K), where its rows
// are more: rows stand for hits only at about one object per cell, and on a
// sparse cloud a claim of eight queries broke into groups of six and two, the
// short one almost as long as the other (98,765 points at 0.38 per cell, K =
// 10: count pass 0.263 -> 0.249 ms).  Radius slots count for their rows: by
// their ball at the lattice's mean density, the uneven-radius workload's
// count pass took 0.691 ms instead of 0.675.
//
// Bound by instruction issue (some 2,000 vector instructions per group of
// eight, spread over row geometry, candidates and the ordering) and, at six
// waves per SIMD, by waiting.  A candidate finds its row by counting the bits
// below its lane, two instructions where a max-scan over marks took ten, and
// the keys and their buckets stay in registers from the first pass of the
// ordering to the rank.  Count pass, ms, before and after these: 4,194,304
// clustered points, K = 16, 2.62 -> 2.58; 1,048,576 uneven radii 0.683 ->
// 0.666; 1,869,073 uniform points, K = 1, 0.406 -> 0.400.  The distance in
// doubles (as in the tiles) saves nine issue slots per step but needs nine
// more registers than there are: 2.57 against 2.53 and 0.692 against 0.676 in
// the same build; noting slot ends by scalar code, only where the slot
// changes, was no faster, and slower where runs are short.

// Per-wave LDS of the grouped kernel: slot data (kGroup x 80 B), 32 words of
// per-slot counters, the 64-word owner map, then (stash) the hit keys in
// arrival order, the same by bucket, and the bucket counts, or (no stash)
// sort_cap 16-byte row records.
__host__ __device__ constexpr uint32_t group_rows(uint32_t cap) { return cap * kRowEighths / 8; }
// rows per chunk of the walk (at most 256): their 16-byte records
// fill the bucket buffer and the bucket counts, both free until the sort
__host__ __device__ constexpr uint32_t group_chunk(uint32_t cap) {
    return group_hitcap(cap) * 12 / 16 < 256u ? group_hitcap(cap) * 12 / 16 : 256u;
}
// 64-row layers of the largest chunk (sort_cap 256)
constexpr uint32_t kLayers = (group_chunk(256) + 63) / 64;
__host__ __device__ constexpr size_t group_lds_per_wave(bool stash, uint32_t cap) {
    return 640 + 128 + 256 + (stash ? (size_t)group_hitcap(cap) * 20 : (size_t)group_chunk(cap) * 16);
}

// dist^2 field of a group hit key (slot | dist^2 | id)
__device__ __forceinline__ uint64_t key_d2(uint64_t k, uint32_t idbits, uint32_t d2bits) {
    return (k >> idbits) & ((1ull << d2bits) - 1ull);
}

// At most 80 VGPRs, so that six waves share each SIMD (the LDS of a
// sort_cap 256 hit buffer allows as many).
// KNN: K-NN queries of the batch are searched in the groups too (a radius
// batch takes the variant without that code).
template <int METHOD, bool TLDS, bool STASH, bool FROM_LIST, bool KNN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void group_count_kernel(LatArgs L,
                                                                                                 TabArgs T,
                                                                                                 QArgs A) {
    extern __shared__ __align__(16) char smem[];
    if (KNN && !FROM_LIST && left_sparse(A)) return;
    const uint32_t* tab_lds = stage_table<TLDS>(T, smem);
    const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
    const uint32_t hitcap = group_hitcap(A.sort_cap), grows = group_rows(A.sort_cap);  // hitcap <= kMaxHitCap
    uint32_t rlim = grows;  // rows per group (shrinks where hits overflow the buffer)
    char* wb = smem + table_lds_bytes<TLDS>(T) + (size_t)wave * group_lds_per_wave(STASH, A.sort_cap);
    uint4* qp = (uint4*)wb;                    // five records of kGroup slots each (slot s of record k
                                               // at qp[k * kGroup + s]): centre + table start, r^2 + self + rows,
                                               // cube extent, flags + row, W/2 - centre + self
    uint32_t* cnt = (uint32_t*)(wb + 640);     // [0, 8) hits, [8, 16) row start, [16, 24) hits,
    uint32_t* qst = cnt + 8;                   // [24, 32) bucket scale (float)
    uint32_t* qn = cnt + 16;
    float* qsc = (float*)(cnt + 24);
    uint32_t* own = cnt + 32;                  // 64: owner map
    uint64_t* hb = (uint64_t*)(own + 64);      // hitcap keys in arrival order
    uint64_t* hs = hb + hitcap;                // hitcap keys by bucket
    uint32_t* hh = (uint32_t*)(hs + hitcap);   // hitcap bucket counts, then starts
    // sort_cap row records of the chunk being walked (in the stash case the
    // bucket buffer, free until the sort)
    uint4* rinfo = STASH ? (uint4*)hs : (uint4*)(own + 64);
    const AxisWrap aw = axis_wrap(L);
    const uint32_t idbits = L.n > 1 ? 32u - (uint32_t)__builtin_clz(L.n - 1u) : 0u;
    const uint32_t d2bits = 64u - kGroupBits - idbits;
    const uint64_t idmask = idbits ? (~0ull >> (64u - idbits)) : 0ull;
    const uint32_t region = blockIdx.x % SPHIDX_NREGION;
    uint32_t cur = 0, lim = 0;
    bool dry = false;
    const uint32_t nq = FROM_LIST ? uni(*A.list_count) : A.Q;
    for_each_range(nq, A, queue_set(A, FROM_LIST ? (int)A.list_set : kQCount), [&](uint32_t b, uint32_t e) {
        for (uint32_t g0 = b, ng = 0; g0 < e; g0 += ng) {
            const uint32_t cand = min(kGroup, e - g0);
            // ---- slots: lane l < cand looks at query g0 + l (of the list);
            // the group keeps the leading slots whose rows fit rlim (at
            // least one)
            const uint32_t qi = FROM_LIST ? (lane < cand ? A.list[g0 + lane] : 0u) : g0 + lane;
            uint32_t rows = 0, row = 0;
            bool mine = false, extra = false, invalid = false, knn = false;
            uint4 d0 = make_uint4(0, 0, 0, 0), d1 = d0, d2 = d0, d3 = d0;
            if (lane < cand) {
                d0 = A.desc[4 * (size_t)qi];
                d1 = A.desc[4 * (size_t)qi + 1];
                d2 = A.desc[4 * (size_t)qi + 2];
                d3 = A.desc[4 * (size_t)qi + 3];
                row = d0.w;
                const uint32_t flags = d1.z;
                const uint64_t r2 = (uint64_t)d1.x * d1.x;
                const uint32_t r2bits = r2 ? 64u - (uint32_t)__builtin_clzll(r2) : 0u;
                const bool valid = flags & F_VALID, sph = flags & F_SPHERE;
                if (!valid) {
                    invalid = true;
                } else if (KNN && FROM_LIST && !((flags & F_KNN) && sph)) {
                    // the second round takes sphere-table K-NN rows only;
                    // everything else on its list goes on
                    extra = true;
                } else if (METHOD == kSphere && !sph) {
                    // counted by the fallback list's kernel
                } else if (KNN && !FROM_LIST && (flags & F_ALONE)) {
                    // listed by the setup for the one-query-per-wave kernel
                } else if (KNN && (flags & F_KNN)) {
                    // K-NN (sphere tables, K up to half the buffer):
                    // a radius row at the first search radius d2.y, the
                    // table prefix d2.z; its first K are the K nearest when
                    // it holds K (Section II.A: beyond the radius every
                    // object is farther)
                    const uint64_t b2 = (uint64_t)d2.y * d2.y;
                    const uint32_t b2bits = b2 ? 64u - (uint32_t)__builtin_clzll(b2) : 0u;
                    if (!sph || (flags & F_LIST) || b2bits > d2bits) {
                        extra = true;
                    } else {
                        mine = true;
                        knn = true;
                        rows = d2.z + ((flags & F_OUTSIDE) ? 1u : 0u);
                    }
                } else if (flags & F_LONG) {
                    // counted one block per row
                } else if ((flags & (F_KNN | F_LIST)) || r2bits > d2bits) {
                    extra = true;
                } else {
                    mine = true;
                    rows = (sph ? d2.x : d2.w * d3.w) + ((flags & F_OUTSIDE) ? 1u : 0u);
                }
            }
            {
                // a K-NN slot counts for its rows or for the hits it is
                // expected to bring, whichever is less (see kRowEighths)
                const uint32_t load =
                    KNN && knn ? min(rows, (uint32_t)(1.125f * knn_target((float)d1.y)) + 1u) : rows;
                const uint32_t pre_incl = scan_add(load);
                const uint64_t fits = __ballot(lane < cand && pre_incl <= rlim);
                ng = max(1u, (uint32_t)__popcll(fits));
                if (lane < kGroup) qst[lane] = pre_incl;  // (free until the sort)
            }
            if (lane >= ng) {
                rows = 0;
                mine = extra = invalid = knn = false;
            }
            if (mine) {
                const uint64_t r2 = (KNN && knn) ? (uint64_t)d2.y * d2.y : (uint64_t)d1.x * d1.x;
                const uint32_t self = (A.qx == nullptr && (A.flags & SPHIDX_EXCLUDE_SELF)) ? qi : kMaxId;
                uint4* p = qp + lane;
                p[0] = make_uint4(d0.x, d0.y, d0.z, d1.w);
                p[kGroup] = make_uint4((uint32_t)r2, (uint32_t)(r2 >> 32), self, rows);
                // (a K-NN slot walks no cube: K and whether its search radius
                // covers the cap take the cube fields)
                p[2 * kGroup] = make_uint4(d3.x, d3.y, d3.z, (KNN && knn) ? d1.y : d2.z);
                p[3 * kGroup] = make_uint4(d2.w, (KNN && knn) ? (d2.y >= d1.x ? 1u : 0u) : d3.w, d1.z, row);
                // the candidate test's form of the centre: the minimum-image
                // offset is ((p + (W/2 - c)) mod W) - W/2
                p[4 * kGroup] = make_uint4(aw.half[0] - d0.x, aw.half[1] - d0.y, aw.half[2] - d0.z, self);
            }
            if (lane < kGroup) cnt[lane] = 0u;
            wave_sync();
            const uint32_t incl = scan_add(rows);
            const uint32_t R = lane_val(incl, 63);
            const uint32_t excl = incl - rows;
            uint32_t hcount = 0;
            // The group's rows go in chunks of sort_cap (at most kLayers x 64)
            // rows: first every row of the chunk, 64 per layer, one per lane,
            // gives its object ranges, numbered by a prefix over the chunk and
            // kept in LDS; then the chunk's candidates, 64 per step, in one
            // stream, with the next step's records loaded while this step's
            // are tested.
            const uint32_t CH = group_chunk(A.sort_cap);  // <= kLayers x 64
            // (a walk whose hits overflow the buffer ends there: only the slots
            // that fit are kept, and in a crowded place one or two of eight
            // do; 1,048,576 agents in 64 clusters, r = 1 cell, count pass with
            // walks to the end 1.98 ms, this way 1.43)
            bool full = false;
            for (uint32_t rb = 0; rb < R && !(STASH && full); rb += CH) {
                const uint32_t clen = min(CH, R - rb);
                uint32_t cex[kLayers];  // where the lane's rows start in the stream (~0: no candidates)
#pragma unroll
                for (uint32_t k = 0; k < kLayers; ++k) cex[k] = ~0u;
                uint32_t carry = 0, kept_rows = 0;
                for (uint32_t k = 0; k * 64u < clen; ++k) {
                    // ---- this lane's row: owner slot and entry
                    const uint32_t base = rb + k * 64u;
                    own[lane] = 0;
                    wave_sync();
                    if (rows > 0 && excl < base + 64 && incl > base) own[excl > base ? excl - base : 0] = lane + 1;
                    wave_sync();
                    const bool act = k * 64u + lane < clen;
                    const uint32_t fr = base + lane;
                    const uint32_t gmax = scan_max(own[lane]);
                    const uint32_t gs = act ? gmax - 1u : 0u;
                    const uint32_t ent = fr - bperm(excl, gs);
                    const uint4* p = qp + gs;
                    const uint4 pa = p[0], pb = p[kGroup], pc = p[2 * kGroup], pd = p[3 * kGroup];
                    Query sq;
                    sq.q[0] = pa.x;
                    sq.q[1] = pa.y;
                    sq.q[2] = pa.z;
                    sq.tb = pa.w;
                    sq.r2 = (uint64_t)pb.x | ((uint64_t)pb.y << 32);
                    sq.self = pb.z;
                    sq.lo[0] = (int32_t)pc.x;
                    sq.lo[1] = (int32_t)pc.y;
                    sq.lo[2] = (int32_t)pc.z;
                    sq.nn[0] = pc.w;
                    sq.nn[1] = pd.x;
                    sq.nn[2] = pd.y;
                    sq.flags = pd.z;
                    const uint32_t e1 = 1u << L.F;
                    for (int a = 0; a < 3; ++a) {
                        sq.c[a] = sq.q[a] >> L.F;
                        sq.f[a] = sq.q[a] & (e1 - 1u);
                        sq.up[a] = e1 - sq.f[a];
                        sq.dn[a] = sq.f[a] + 1u;
                    }
                    const bool is_out = act && (sq.flags & F_OUTSIDE) && ent + 1u == pb.w;
                    const bool sph = METHOD == kSphere || (METHOD == kEither && (sq.flags & F_SPHERE));
                    const bool live = act && !is_out;
                    RowRef r;
                    if (sph) {
                        const uint32_t w =
                            live ? row_word<TLDS>(T, tab_lds, sq.tb, TLDS ? row_class(L, T, sq.f) : 0u, ent) : 0u;
                        r = sphere_row(L, sq, w, live, sq.r2, false);
                    } else {
                        const double inv_ny = sq.nn[1] ? 1.0 / (double)sq.nn[1] : 0.0;
                        r = cube_row(L, sq, live ? ent : 0u, live, inv_ny);
                    }
                    if (is_out) {
                        // every object outside the region lives in one cell (Section II.B)
                        r.st0 = L.cs[L.ncells];
                        r.cnt0 = L.cs[L.ncells + 1] - r.st0;
                        r.cnt1 = 0u;
                    }
                    if (A.stats && live) {
                        // per-query statistics, the outside cell's pseudo-row
                        // left out (rows walked again are counted again)
                        uint32_t* stp = A.stats + 4 * (size_t)pd.w;
                        atomicAdd(stp, 1u);
                        atomicAdd(stp + 1, r.kept);
                    }
                    const uint32_t tl = act ? r.cnt0 + r.cnt1 : 0u;
                    const uint32_t ci = scan_add(tl);
                    const uint32_t ce = carry + ci - tl;
                    // per row with candidates, in order: position bases of its
                    // two ranges, the slot where the second starts, and the
                    // query slot
                    const uint64_t full = __builtin_amdgcn_ballot_w64(tl > 0u);
                    if (tl > 0u)
                        rinfo[lanes_below(full, kept_rows)] =
                            make_uint4(r.st0 - ce, ce + r.cnt0, r.st1 - (ce + r.cnt0), gs);
                    kept_rows += (uint32_t)__popcll(full);
#pragma unroll
                    for (uint32_t j = 0; j < kLayers; ++j) cex[j] = j == k && tl > 0u ? ce : cex[j];
                    carry += lane_val(ci, 63);
                }
                const uint32_t CT = carry;
                // ---- owner row of each of the 64 slots from cb: every row
                // marks the slot where it starts, in a window of four steps
                // (256 slots, one byte each in the owner map's words); a
                // slot's row is the number of marks up to its own, counted on
                // from the rows before.  Steps are located in order, each
                // once.  (One bit per slot, for 2,048 slots at a time, needs
                // no read per step, but rows of a candidate or two meet in
                // one word's atomics: 4 % slower on a K = 1 cloud.)
                uint32_t before = 0;
                auto locate = [&](uint32_t cb, uint32_t& pos, uint32_t& sl) {
                    const uint32_t wb = cb & ~255u;
                    uint8_t* own8 = (uint8_t*)own;
                    if (cb == wb) {
                        wave_sync();
                        own[lane] = 0;
                        wave_sync();
#pragma unroll
                        for (uint32_t k = 0; k < kLayers; ++k)
                            if (cex[k] - wb < 256u) own8[cex[k] - wb] = 1u;
                        wave_sync();
                    }
                    const uint64_t mk = __builtin_amdgcn_ballot_w64(own8[cb - wb + lane] != 0);
                    const uint4 ri = rinfo[lanes_below(mk >> 1, before + (uint32_t)(mk & 1u) - 1u)];
                    before += (uint32_t)__popcll(mk);
                    const uint32_t g = cb + lane;
                    // (slots past the end: the last row's, held inside the array)
                    pos = min((g < ri.y ? ri.x : ri.z) + g, L.n - 1u);
                    sl = ri.w;
                };
                auto test = [&](const uint4& P, uint32_t pos, uint32_t sl, uint32_t cb) {
                    const uint4 ch = qp[4 * kGroup + sl];
                    const uint2 cr = *(const uint2*)(qp + kGroup + sl);
                    const uint32_t pv[3] = {P.x, P.y, P.z}, hv[3] = {ch.x, ch.y, ch.z};
                    uint64_t d2 = 0;
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        const int32_t dd = (int32_t)((pv[a] + hv[a]) & aw.mask[a]) - (int32_t)aw.half[a];
                        d2 += (uint64_t)((int64_t)dd * dd);
                    }
                    const uint64_t in = CT - cb >= 64u ? ~0ull : (1ull << (CT - cb)) - 1ull;
                    const uint64_t H = in & __builtin_amdgcn_ballot_w64(d2 <= ((uint64_t)cr.x | ((uint64_t)cr.y << 32))) &
                                       __builtin_amdgcn_ballot_w64(pos != ch.w);
                    if (A.stats && lane_in(in)) atomicAdd(A.stats + 4 * (size_t)qp[3 * kGroup + sl].w + 2, 1u);
                    const uint32_t hp = lanes_below(H, hcount);
                    // hits per slot: a slot's candidates take contiguous lanes
                    // and its hits arrive in order, so the last lane of its
                    // run in a step records the group's hit count so far
                    // (lanes past the end belong to the last row's slot)
                    const uint32_t nsl = bperm(sl, (lane + 1u) & 63u);
                    if (lane == 63u || nsl != sl) cnt[sl] = hp + (lane_in(H) ? 1u : 0u);
                    if (STASH && lane_in(H) && hp < hitcap) {
                        const uint64_t k = d2 << idbits;
                        hb[hp] = ((uint64_t)((sl << (32u - kGroupBits)) | (uint32_t)(k >> 32)) << 32) |
                                 ((uint32_t)k | P.w);
                    }
                    hcount += (uint32_t)__popcll(H);
                };
                // whether the walk can stop: the buffer is full, and slot 0 has
                // been walked whole (the next step's first candidate, in slot
                // `next`, is past it), so the slots that fit have too
                auto over = [&](uint32_t next) -> bool {
                    if (STASH && hcount > hitcap && uni(next) > 0u) full = true;
                    return STASH && full;
                };
                if (CT > 0) {
                    // two register sets taken in turn: the step after the one
                    // under test is already loading (the one past the end,
                    // located once per chunk, reads a record and tests nothing)
                    uint32_t pa = 0, sa = 0, pb = 0, sb = 0;
                    locate(0, pa, sa);
                    uint4 PA = L.pts[pa], PB = PA;
                    for (uint32_t cb = 0; cb < CT; cb += 128) {
                        locate(cb + 64, pb, sb);
                        PB = L.pts[pb];
                        test(PA, pa, sa, cb);
                        if (cb + 64 >= CT || over(sb)) break;
                        locate(cb + 128, pa, sa);
                        PA = L.pts[pa];
                        test(PB, pb, sb, cb + 64);
                        if (over(sa)) break;
                    }
                }
                wave_sync();
            }
            // ---- row sizes: each slot's hits end where its last run left
            // the count (a slot without candidates left none: the max-scan
            // carries the previous slot's end)
            const uint32_t hend = scan_max(lane < kGroup ? cnt[lane] : 0u);
            const uint32_t hbeg = bperm(hend, (lane + 63u) & 63u);
            uint32_t nq = mine ? hend - (lane ? hbeg : 0u) : 0u;
            uint32_t total = hcount;
            if (STASH && hcount > hitcap && ng > 1) {
                // the hit buffer overflowed: keep the leading slots whose hits
                // fit (hits arrive slot by slot, so theirs are the buffer's
                // first keys); the next group starts at the first slot left
                // out and walks it again
                const uint32_t hi = scan_add(nq);
                ng = max(1u, (uint32_t)__popcll(__ballot(lane < ng && hi <= hitcap)));
                if (lane >= ng) {
                    mine = extra = invalid = knn = false;
                    nq = 0u;
                }
                total = lane_val(hi, ng - 1u);
                // later groups of this wave take no more rows than fitted
                // here, and grow back by an eighth per group that fits
                rlim = max(1u, uni(qst[ng - 1u]));
            } else if (STASH) {
                rlim = min(grows, rlim + max(1u, grows / 8u));
            }
            // K-NN rows: the first K, or every object when the search radius
            // covers the cap; a row with fewer than K inside a smaller radius
            // is searched again by the one-query-per-wave kernel
            uint32_t nrow = nq;
            if (KNN && knn) {
                const uint32_t kk = qp[2 * kGroup + lane].w;
                if (nq >= kk) {
                    nrow = kk;
                } else if (qp[3 * kGroup + lane].y == 0u) {
                    mine = false;
                    extra = true;
                    if (!FROM_LIST) {
                        // for the second round: the radius expected to hold
                        // knn_target(K) at the density the first ball showed
                        // (grown by 1.15 to 2 times, the cap at most), and its
                        // table prefix from the radius index of the row class
                        const float sc =
                            fminf(2.0f, fmaxf(1.15f, cbrtf(knn_target((float)kk) / fmaxf((float)nq, 0.5f))));
                        const uint32_t kb = (uint32_t)min((uint64_t)d1.x, (uint64_t)((float)d2.y * sc) + 1u);
                        const uint32_t e1 = 1u << L.F, sh = L.F - T.s;
                        const uint32_t cls = ((d0.y & (e1 - 1u)) >> sh) | (((d0.z & (e1 - 1u)) >> sh) << T.s);
                        const uint32_t jb = (uint32_t)(((uint64_t)kb + (1u << T.rshift) - 1u) >> T.rshift);
                        A.desc[4 * (size_t)qi + 2] = make_uint4(d2.x, kb, T.rindex[(size_t)cls * T.nr + jb], d2.w);
                    }
                }
            }
            if (invalid) {
                A.row_ptr[row] = 0;
                if (STASH) A.soff[row] = 0u;
            }
            {
                // the queries left to the one-query-per-wave kernel
                const uint64_t xm = __ballot(extra);
                uint32_t xb = 0;
                if (xm != 0 && lane == 0) xb = atomicAdd(A.xq_count, (uint32_t)__popcll(xm));
                xb = uni(xb);
                if (extra) A.xq[xb + lanes_below(xm)] = qi;
            }
            if (mine) A.row_ptr[row] = (int64_t)nrow;
            if (STASH) {
                // pairs kept per slot: a K-NN row keeps its first K, so the
                // stash takes those only (K-NN variant); a radius row, all
                const uint32_t ko = KNN ? (mine ? nrow : 0u) : nq;
                const uint32_t kincl = scan_add(ko);
                const uint32_t qo0 = kincl - ko;
                const uint32_t tout = KNN ? lane_val(kincl, 63) : total;
                bool ok = total <= hitcap;
                if (ok && tout > 0 && cur + tout > lim) {
                    ok = false;
                    if (!dry) {
                        const uint32_t grab = max(A.stash_chunk, tout);
                        uint32_t t = 0;
                        if (lane == 0) t = atomicAdd(A.stash_ctr + region * SPHIDX_QSTRIDE, grab);
                        t = uni(t);
                        if ((uint64_t)t + grab <= A.stash_region) {
                            cur = region * A.stash_region + t;
                            lim = cur + grab;
                            ok = true;
                        } else {
                            dry = true;
                        }
                    }
                }
                const uint32_t qs0 = scan_add(nq) - nq;
                if (ok && tout > 0) {
                    // every hit's dist^2 is at most its slot's r^2: shifted
                    // right by gsh, the largest r^2 of the group fits 24 bits,
                    // so a bucket needs one 32-bit conversion
                    uint64_t r2 = 0;
                    if (lane < kGroup) {
                        const uint4 pb = qp[kGroup + lane];
                        r2 = nq > 0 ? (uint64_t)pb.x | ((uint64_t)pb.y << 32) : 0ull;
                    }
                    const uint32_t rbits = lane_val(scan_max(r2 ? 64u - (uint32_t)__builtin_clzll(r2) : 0u), 63);
                    const uint32_t gsh = rbits > 24u ? rbits - 24u : 0u;
                    const uint32_t dsh = idbits + gsh, dmask = (1u << (rbits - gsh)) - 1u;
                    if (lane < kGroup) {
                        qst[lane] = qs0;
                        qn[lane] = nq;
                        qsc[lane] = r2 > 0 ? (float)nq / (float)((uint32_t)(r2 >> gsh) + 1u) : 0.0f;
                        // (the owner map is free until the next group)
                        own[lane] = qo0;
                        own[kGroup + lane] = ko;
                    }
                    for (uint32_t t = lane; t < total; t += 64) hh[t] = 0u;
                    wave_sync();
                    // bucket of a key: its slot's rows start + about
                    // n * d^2 / r^2, below n, never smaller for a larger d^2
                    auto bucket = [&](uint64_t k) -> uint32_t {
                        const uint32_t sl = (uint32_t)(k >> (64u - kGroupBits));
                        const uint32_t d = (uint32_t)(k >> dsh) & dmask;
                        const uint32_t bi = min((uint32_t)((float)d * qsc[sl]), qn[sl] - 1u);
                        return qst[sl] + bi;
                    };
                    uint32_t slot[(kMaxHitCap + 63) / 64], bk[(kMaxHitCap + 63) / 64];
                    uint64_t kv[(kMaxHitCap + 63) / 64];
#pragma unroll
                    for (uint32_t k = 0; k < (kMaxHitCap + 63) / 64; ++k) {
                        const uint32_t t = lane + 64u * k;
                        bk[k] = 0u;
                        if (t < total) {
                            kv[k] = hb[t];
                            bk[k] = bucket(kv[k]);
                            slot[k] = atomicAdd(&hh[bk[k]], 1u);
                        }
                    }
                    wave_sync();
                    const uint32_t per = (total + 63u) >> 6;
                    const uint32_t bb = lane * per;
                    uint32_t sum = 0;
                    for (uint32_t k = 0; k < per; ++k)
                        if (bb + k < total) sum += hh[bb + k];
                    uint32_t run = scan_add(sum) - sum;
                    wave_sync();
                    for (uint32_t k = 0; k < per; ++k)
                        if (bb + k < total) {
                            const uint32_t c = hh[bb + k];
                            hh[bb + k] = run;
                            run += c;
                        }
                    wave_sync();
#pragma unroll
                    for (uint32_t k = 0; k < (kMaxHitCap + 63) / 64; ++k) {
                        const uint32_t t = lane + 64u * k;
                        if (t < total) hs[hh[bk[k]] + slot[k]] = kv[k];
                    }
                    wave_sync();
#pragma unroll
                    for (uint32_t k = 0; k < (kMaxHitCap + 63) / 64; ++k) {
                        const uint32_t t = lane + 64u * k;
                        if (t >= total) continue;
                        const uint64_t key = kv[k];
                        const uint32_t bi = bk[k];
                        const uint32_t lo = hh[bi], hi = bi + 1 < total ? hh[bi + 1] : total;
                        uint32_t rank = lo;
                        for (uint32_t j = lo; j < hi; ++j) rank += hs[j] < key ? 1u : 0u;
                        uint32_t o = cur + rank;
                        bool keep = true;
                        if (KNN) {
                            // its rank inside its slot's row, kept when below K
                            const uint32_t sl = (uint32_t)(key >> (64u - kGroupBits));
                            const uint32_t wr = rank - qst[sl];
                            keep = wr < own[kGroup + sl];
                            o = cur + own[sl] + wr;
                        }
                        if (keep) {
                            A.stash_ids[o] = (uint32_t)(key & idmask);
                            if (A.stash_d2) A.stash_d2[o] = (int64_t)key_d2(key, idbits, d2bits);
                        }
                    }
                    wave_sync();
                    if (mine) A.soff[row] = cur + (KNN ? qo0 : qs0);
                    cur += tout;
                } else {
                    // not kept: the write pass walks these rows again
                    const bool walk_again = mine && nq > 0;
                    if (mine) A.soff[row] = walk_again ? kMaxId : 0u;
                    if (walk_again) list_row_again(A, qi, ((KNN && knn) || nq > A.sort_cap) && !(FROM_LIST && METHOD == kCube));
                }
            }
            wave_sync();
        }
    }, kGroup);
}

// ---------------------------------------------------------------------------
// Pass 0, all-agents queries of one radius by tiles of space: a wavefront
// takes up to 16 queries that lie close together, reads the candidates of all
// of them once, and tests every pair on the matrix cores.
//
// Queries are ordered for this by strips: a strip is 2^wy x 2^wz rows of
// cells along x, cut into chunks of 2^cl columns; a chunk's queries, column
// by column, go to work items (tile_items_kernel) and, inside an item, to
// groups of up to 16.  A group's candidates are the objects within the radius
// of the box around its queries: one lane per x-row of cells solves the row's
// run, the runs' objects are spread over the lanes, and those within reach of
// the box go to a ring in LDS as coordinates relative to the group's first
// query.
//
// 64 candidates at a time leave the ring, one per lane, as x, y, z and
// x^2 + y^2 + z^2 in double precision; eight lane-row swaps turn them into the
// operands of four v_mfma_f64_16x16x4.  With the queries' [-2x, -2y, -2z, 1]
// as rows and the accumulator starting at 2^52 + slot 2^d + |q|^2, every
// element is 2^52 + slot 2^d + dist^2: all operands and sums are integers
// below 2^53, so the result is exact whatever the order of the sum, its low 52
// bits are the integer (slot, dist^2), and a hit is one comparison with
// 2^52 + slot 2^d + r^2.  Hits go to LDS as 64-bit keys (slot, dist^2, id);
// one bucket sort, its keys held in registers and put in place, orders the
// group's rows.
//
// Bound by instruction issue (VALU 68 % busy on the 8.4 M-agent timestep, the
// rest waits on LDS at the 12 wavefronts a CU holds) and by what crosses the L2
// (13.5 GB, three quarters of a copy's rate).  Against a row walk per
// query (group_count_kernel) a query pays a sixteenth of its group's rows and
// candidate loads, and a pair a comparison instead of an address search, three
// wrapped differences and three products; in exchange it is tested against
// the whole group's candidates (about 310 for 57 hits at r = 3 cells and 0.5
// objects per cell, instead of 109).  There: 171 VALU instructions per query
// instead of 371, count kernel 5.60 -> 3.61 ms.  With the ring holding
// doubles, hits placed one by one, ranks from loops over each key's bucket and
// the descriptors read it took 6.0 ms; 128-register variants spill (5.3 ms),
// groups of 8 queries took the same time at twice the rows.

// queries per group, pairs of its hit buffer, rows per chunk of the walk,
// candidates of the ring (a power of two, at least 63 + 64), cells per strip
// chunk, queries per work item
constexpr uint32_t kTileMinQ = 1024;  // the smallest batch by tiles
constexpr uint32_t kTileQ = 16, kTileHits = 960, kTileRows = 88, kTileRing = 128;
constexpr uint32_t kTileCellLayers = 4, kTileCells = 64 * kTileCellLayers;
constexpr uint32_t kTileBuckets = 64;  // sort buckets per query slot
constexpr uint32_t kTileNear = 8;      // places a key can be from its rank in bucket order without the slow path
// LDS of a block (one wavefront): hit keys and a spare one; then ring, row
// records and owner marks, all free once the tests are done, when the sort's
// bucket counts take their place.  (kTileHits / 64 odd: a lane's run of keys
// then starts in another bank than its neighbours'.)
constexpr uint32_t kTileScratch = 4112;
constexpr uint32_t kTileLds = (kTileHits + 2) * 8 + kTileScratch;
static_assert(kTileScratch >= (kTileQ * kTileBuckets + 1) * 4, "the bucket counts fit the walk's buffers");
static_assert(kTileScratch >= kTileRing * 16 + kTileRows * 12 + 256, "the walk's buffers fit");
static_assert(kTileRows <= 254, "owner marks hold a row + 1 in one byte");

constexpr uint32_t kTileLayers = (kTileRows + 63) / 64;

struct TileArgs {
    uint32_t cl, wy, wz;    // log2 of a chunk's columns and of a strip's rows in y and z
    uint32_t nchunks;
    uint32_t part;          // queries per work item (a multiple of kTileQ)
    uint32_t mean;          // queries per chunk
    uint32_t d2bits;        // bits of dist^2 in a key: those of the largest r^2
};

typedef double dbl4 __attribute__((ext_vector_type(4)));

// First cell of row `row` of a chunk.
__device__ __forceinline__ uint32_t tile_cell(const LatArgs& L, const TileArgs& TA, uint32_t chunk, uint32_t row,
                                              uint32_t col) {
    const uint32_t lx = L.lg[0] - TA.cl, ly = L.lg[1] - TA.wy;
    const uint32_t cx = chunk & ((1u << lx) - 1u), sy = (chunk >> lx) & ((1u << ly) - 1u), sz = chunk >> (lx + ly);
    const uint32_t y = (sy << TA.wy) + (row & ((1u << TA.wy) - 1u)), z = (sz << TA.wz) + (row >> TA.wy);
    return pack_cell(L, (cx << TA.cl) + col, y, z);
}

// Queries per work item of a chunk of T queries: a multiple of kTileQ, fewer in
// chunks of half as many again as the mean (their rows are as much longer, and
// one wavefront would be left with an item for long after the others: 1,048,576
// agents in 1,024 clusters, r = 3 cells, count pass 4.5 ms, this way 2.8), at
// most 1,024 items per chunk.
__device__ __forceinline__ uint32_t tile_part(const TileArgs& TA, uint32_t T) {
    const uint32_t least = (T + 1023u) >> 10;
    const uint32_t part = T > TA.mean + TA.mean / 2u ? (uint32_t)((uint64_t)TA.part * TA.mean / T) : TA.part;
    return (max(max(part, least), 1u) + kTileQ - 1u) & ~(kTileQ - 1u);
}

// One thread per chunk: its work items, chunk | part << 22.  The objects left out
// by the build, after every cell, get empty rows here.
__global__ __launch_bounds__(256) void tile_items_kernel(LatArgs L, QArgs A, TileArgs TA, uint32_t* items,
                                                         uint32_t* count) {
    const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t i = L.cs[L.ncells + 1] + c; i < L.n; i += gridDim.x * blockDim.x) {
        const uint32_t row = L.pts[i].w;
        A.row_ptr[row] = 0;
        if (A.stash) A.soff[row] = 0u;
    }
    uint32_t T = 0;
    if (c < TA.nchunks) {
        for (uint32_t row = 0; row < (1u << (TA.wy + TA.wz)); ++row) {
            const uint32_t cell = tile_cell(L, TA, c, row, 0u);
            T += L.cs[cell + (1u << TA.cl)] - L.cs[cell];
        }
    }
    const uint32_t part = tile_part(TA, T), n = (T + part - 1u) / part;
    const uint32_t incl = scan_add(n), total = lane_val(incl, 63);
    uint32_t base = 0;
    if (total > 0 && lane_id() == 0) base = atomicAdd(count, total);
    base = uni(base) + incl - n;
    for (uint32_t k = 0; k < n; ++k) items[base + k] = c | (k << 22);
}

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
// Minimum and maximum over the 16 lanes of a DPP row (rotations).
__device__ __forceinline__ int row_min(int v) {
    v = min(v, dpp_i<0x128>(v));
    v = min(v, dpp_i<0x124>(v));
    v = min(v, dpp_i<0x122>(v));
    return min(v, dpp_i<0x121>(v));
}
__device__ __forceinline__ int row_max(int v) {
    v = max(v, dpp_i<0x128>(v));
    v = max(v, dpp_i<0x124>(v));
    v = max(v, dpp_i<0x122>(v));
    return max(v, dpp_i<0x121>(v));
}
__device__ __forceinline__ uint32_t row_sum(uint32_t v) {
    v += (uint32_t)dpp_i<0x128>((int)v);
    v += (uint32_t)dpp_i<0x124>((int)v);
    v += (uint32_t)dpp_i<0x122>((int)v);
    return v + (uint32_t)dpp_i<0x121>((int)v);
}

// Rows 2, 3 of a's 16-lane rows change places with rows 0, 1 of b; rows 1, 3
// of a with rows 0, 2 of b.
__device__ __forceinline__ void swap_rows32(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap_rows16(uint32_t& a, uint32_t& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
__device__ __forceinline__ void swap_rows32(double& a, double& b) {
    uint32_t ah = (uint32_t)__double2hiint(a), al = (uint32_t)__double2loint(a);
    uint32_t bh = (uint32_t)__double2hiint(b), bl = (uint32_t)__double2loint(b);
    swap_rows32(ah, bh);
    swap_rows32(al, bl);
    a = __hiloint2double((int)ah, (int)al);
    b = __hiloint2double((int)bh, (int)bl);
}
__device__ __forceinline__ void swap_rows16(double& a, double& b) {
    uint32_t ah = (uint32_t)__double2hiint(a), al = (uint32_t)__double2loint(a);
    uint32_t bh = (uint32_t)__double2hiint(b), bl = (uint32_t)__double2loint(b);
    swap_rows16(ah, bh);
    swap_rows16(al, bl);
    a = __hiloint2double((int)ah, (int)al);
    b = __hiloint2double((int)bh, (int)bl);
}

// The next lane's value (lane 63: all ones).
__device__ __forceinline__ uint64_t next_lane(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)v, 0x130, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)(uint32_t)(v >> 32), 0x130, 0xF, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}

// STASH: rows are sorted and kept; else counted only.  EXCL: an object's own
// entry is left out.
template <bool STASH, bool EXCL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void tile_count_kernel(LatArgs L, QArgs A,
                                                                                                 TileArgs TA) {
    extern __shared__ __align__(16) char smem[];
    uint32_t lane = lane_id();
    uint64_t* hb = (uint64_t*)smem;
    char* sc = smem + (kTileHits + 2) * 8;
    uint4* ring = (uint4*)sc;                            // kTileRing candidates: x, y, z relative, id
    uint2* rpos = (uint2*)(sc + kTileRing * 16);         // kTileRows: position bases of a row's two ranges,
    uint32_t* rbnd = (uint32_t*)(rpos + kTileRows);      // and the candidate slot where the second starts
    uint32_t* own = rbnd + kTileRows;                    // 64
    uint32_t* hh = (uint32_t*)sc;                        // the sort's bucket counts
    ulonglong2* slotd = (ulonglong2*)hb;                 // per slot: accumulator start, threshold (before the tests)
    const AxisWrap aw = axis_wrap(L);
    const uint32_t d2b = TA.d2bits, sh = 60u - d2b;      // key: slot (4 bits) | dist^2 (d2b) | id (sh)
    const uint32_t region = blockIdx.x % SPHIDX_NREGION;
    const uint32_t F = L.F, E1 = (1u << F) - 1u;
    const int R = (int)A.rad_u;
    // conservative single-precision reach (a candidate set only: every pair is
    // tested exactly)
    const float R2f = (float)R * (float)R * 1.000002f + 1.0f;
    // bucket of a key in its slot: floor(64 v / (v_max + 1)), v the top 24 bits
    // of dist^2: monotone in dist^2
    const float scale = (float)kTileBuckets / ((float)((((uint64_t)A.rad_u * A.rad_u) << sh) >> 36) + 1.0f);
    uint32_t cur = 0, lim = 0;
    bool dry = false;
    uint32_t nlim = kTileQ;  // queries per group (fewer where hits overflow the buffer)
    const uint32_t ncell = 1u << (TA.cl + TA.wy + TA.wz);
    const uint32_t rowmask = (1u << (TA.wy + TA.wz)) - 1u;
    for_each_range(uni(*A.item_count), A, queue_set(A, kQCount), [&](uint32_t ib, uint32_t ie) {
        for (uint32_t it = ib; it < ie; ++it) {
            const uint32_t item = uni(A.longq[it]);
            const uint32_t chunk = item & 0x3FFFFFu, part = item >> 22;
            // ---- the chunk's cells, column by column, four per lane: the
            // ranks of their queries and the position of rank 0
            uint32_t cex[kTileCellLayers], cin[kTileCellLayers], cst[kTileCellLayers], total_q = 0;
#pragma unroll
            for (uint32_t k = 0; k < kTileCellLayers; ++k) {
                const uint32_t c = k * 64u + lane;
                cin[k] = cst[k] = 0;
                if (c < ncell) {
                    const uint32_t cell = tile_cell(L, TA, chunk, c & rowmask, c >> (TA.wy + TA.wz));
                    cst[k] = L.cs[cell];
                    cin[k] = L.cs[cell + 1u] - cst[k];
                }
            }
#pragma unroll
            for (uint32_t k = 0; k < kTileCellLayers; ++k) {
                const uint32_t n = cin[k];
                cin[k] = total_q + scan_add(n);
                cex[k] = cin[k] - n;
                cst[k] -= cex[k];
                total_q = lane_val(cin[k], 63);
            }
            const uint32_t per = tile_part(TA, total_q);
            const uint32_t rend = min(total_q, (part + 1u) * per);
            uint32_t r0 = part * per, ng = 0;
            // ---- the group from rank r0 (groups of equal size): lane l takes
            // its query l mod 16 (the last one's record past the end); a cell
            // leaves its position base at its first rank in the group, and
            // every rank takes the last one before it
            uint32_t pos = 0;
            auto group = [&]() -> uint4 {
                const uint32_t slot = lane & 15u;
                ng = (rend - r0 + nlim - 1u) / nlim;
                ng = (rend - r0 + ng - 1u) / ng;
                wave_sync();
                if (lane < 16u) own[lane] = 0u;
                wave_sync();
#pragma unroll
                for (uint32_t k = 0; k < kTileCellLayers; ++k)
                    if (cin[k] > cex[k] && cex[k] < r0 + ng && cin[k] > r0) {
                        const uint32_t w = cex[k] > r0 ? cex[k] - r0 : 0u;
                        own[w] = w + 1u;
                        own[16u + w] = cst[k];
                    }
                wave_sync();
                uint32_t first = own[slot];
                first = max(first, (uint32_t)dpp_i<0x111>((int)first));
                first = max(first, (uint32_t)dpp_i<0x112>((int)first));
                first = max(first, (uint32_t)dpp_i<0x114>((int)first));
                first = max(first, (uint32_t)dpp_i<0x118>((int)first));
                pos = own[15u + max(first, 1u)] + r0 + min(slot, ng - 1u);
                wave_sync();
                return L.pts[pos];
            };
            uint4 Q = make_uint4(0, 0, 0, 0);
            if (r0 < rend) Q = group();
            while (r0 < rend) {
                // (what follows from the lane is made again for each group: kept
                // over all of them it would not fit the registers)
                asm volatile("" : "+v"(lane));
                const uint32_t slot = lane & 15u, quad = lane >> 4;
                const bool mine = slot < ng;
                const uint32_t row = Q.w, qpos = pos;
                uint32_t hcount = 0;  // hits of the group
                // ---- the box around the queries, relative to the first
                const uint32_t o[3] = {uni(Q.x), uni(Q.y), uni(Q.z)};
                const uint32_t qv[3] = {Q.x, Q.y, Q.z};
                int q3[3], lo[3], hi[3];
                bool outside = false;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    // (slots past the end repeat the last query)
                    q3[a] = (int)(((qv[a] - o[a]) + aw.half[a]) & aw.mask[a]) - (int)aw.half[a];
                    lo[a] = (int)uni((uint32_t)row_min(q3[a]));
                    hi[a] = (int)uni((uint32_t)row_max(q3[a]));
                    outside = outside || (!((L.cyc >> a) & 1u) && (((int)o[a] + hi[a] + R) >> (F + L.lg[a])) != 0);
                }
                const double qx = q3[0], qy = q3[1], qz = q3[2];
                const double bias = (double)((uint64_t)slot << d2b) + 4503599627370496.0;
                const double cq = __builtin_fma(qx, qx, __builtin_fma(qy, qy, __builtin_fma(qz, qz, bias)));
                const double tq = mine ? __builtin_fma((double)R, (double)R, bias) : 0.0;
                const double fa = quad == 0u ? -2.0 * qx : quad == 1u ? -2.0 * qy : quad == 2u ? -2.0 * qz : 1.0;
                // accumulator starts and thresholds of this lane's four rows,
                // slots quad + 4 i
                if (lane < kTileQ)
                    slotd[lane] = make_ulonglong2((uint64_t)__double_as_longlong(cq), (uint64_t)__double_as_longlong(tq));
                wave_sync();
                dbl4 C, thr;
                uint32_t selfp[4] = {kMaxId, kMaxId, kMaxId, kMaxId};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const ulonglong2 w = slotd[quad + 4u * i];
                    C[i] = __longlong_as_double((long long)w.x);
                    thr[i] = __longlong_as_double((long long)w.y);
                    if (EXCL) selfp[i] = bperm(row, quad + 4u * i);
                }
                wave_sync();
                uint32_t cnt[4] = {0u, 0u, 0u, 0u};
                uint32_t head = 0, fill = 0;  // ring: first pending entry, entries pending
                // 64 pending candidates, one per lane (nb of them; the rest
                // padding that is never within a radius): their four operand
                // rows are transposed between the lanes' 16-lane rows, so that
                // tile t's operand holds component k of candidate 16 t + column
                // in row k
                auto batch = [&](uint32_t nb) {
                    wave_sync();
                    const uint4 P = ring[(head + lane) & (kTileRing - 1u)];
                    wave_sync();
                    const double x = (double)(int)P.x, y = (double)(int)P.y, z = (double)(int)P.z;
                    double b[4] = {x, y, z, __builtin_fma(x, x, __builtin_fma(y, y, z * z))};
                    if (lane >= nb) b[3] = 1.0e30;
                    swap_rows32(b[0], b[2]);
                    swap_rows32(b[1], b[3]);
                    swap_rows16(b[0], b[1]);
                    swap_rows16(b[2], b[3]);
                    uint32_t id[4] = {P.w, 0, P.w, 0};
                    swap_rows32(id[0], id[2]);
                    id[1] = id[0];
                    id[3] = id[2];
                    swap_rows16(id[0], id[1]);
                    swap_rows16(id[2], id[3]);
                    dbl4 D[4];
                    bool H[16];
#pragma unroll
                    for (int j = 0; j < 4; ++j) D[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa, b[j], C, 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            H[4 * j + i] = D[j][i] <= thr[i];
                            if (EXCL) H[4 * j + i] = H[4 * j + i] && id[j] != selfp[i];
                        }
                    if (!STASH) {
#pragma unroll
                        for (int j = 0; j < 16; ++j) cnt[j & 3] += H[j] ? 1u : 0u;
                    } else {
                        // every lane writes its own hits, from its place in the
                        // prefix of their numbers (past the buffer: counted only)
                        uint32_t mc = 0;
#pragma unroll
                        for (int j = 0; j < 16; ++j) mc += H[j] ? 1u : 0u;
                        const uint32_t incl = scan_add(mc);
                        const uint32_t n = lane_val(incl, 63);
                        uint64_t* w = hb + (hcount + incl - mc);
                        if (hcount + n <= kTileHits) {
#pragma unroll
                            for (int j = 0; j < 16; ++j)
                                if (__builtin_expect(H[j], 1)) {
                                    *w = ((uint64_t)__double_as_longlong(D[j >> 2][j & 3]) << sh) | id[j >> 2];
                                    ++w;
                                }
                        }
                        hcount += n;
                    }
                    head = (head + 64u) & (kTileRing - 1u);
                };
                asm volatile("" : "+v"(lane));
                // ---- rows of cells within reach of the box, in chunks
                const int ax[3] = {(int)o[0], (int)o[1], (int)o[2]};
                int Y0 = (ax[1] + lo[1] - R) >> F, Y1 = (ax[1] + hi[1] + R) >> F;
                int Z0 = (ax[2] + lo[2] - R) >> F, Z1 = (ax[2] + hi[2] + R) >> F;
                if (!(L.cyc & 2u)) {
                    Y0 = max(Y0, 0);
                    Y1 = min(Y1, (1 << L.lg[1]) - 1);
                }
                if (!(L.cyc & 4u)) {
                    Z0 = max(Z0, 0);
                    Z1 = min(Z1, (1 << L.lg[2]) - 1);
                }
                const uint32_t ny = (uint32_t)(Y1 - Y0 + 1), nz = (uint32_t)(Z1 - Z0 + 1);
                const uint32_t NR = ny * nz + (outside ? 1u : 0u);
                const float inv_ny = 1.0f / (float)ny;
                for (uint32_t rb = 0; rb < NR; rb += kTileRows) {
                    const uint32_t clen = min(kTileRows, NR - rb);
                    uint32_t rex[kTileLayers], rin[kTileLayers];
                    uint32_t carry = 0;
#pragma unroll
                    for (uint32_t k = 0; k < kTileLayers; ++k) {
                        rex[k] = rin[k] = 0u;
                        if (k * 64u < clen) {
                            const uint32_t e = rb + k * 64u + lane;
                            const bool act = k * 64u + lane < clen;
                            const bool is_out = outside && e + 1u == NR;
                            bool live = act && !is_out;
                            const uint32_t iz = (uint32_t)(((float)e + 0.5f) * inv_ny);
                            const int ty = Y0 + (int)(e - iz * ny), tz = Z0 + (int)iz;
                            const int ylo = ty << F, zlo = tz << F;
                            const int gy = max(0, max(ylo - (ax[1] + hi[1]), ax[1] + lo[1] - ylo - (int)E1));
                            const int gz = max(0, max(zlo - (ax[2] + hi[2]), ax[2] + lo[2] - zlo - (int)E1));
                            const float g2 = (float)gy * (float)gy + (float)gz * (float)gz;
                            live = live && g2 <= R2f;
                            const int X = live ? (int)__builtin_amdgcn_sqrtf(R2f - g2) + 2 : 0;
                            uint32_t uy = (uint32_t)ty, uz = (uint32_t)tz;
                            if (L.cyc & 2u) uy &= (1u << L.lg[1]) - 1u;
                            if (L.cyc & 4u) uz &= (1u << L.lg[2]) - 1u;
                            if (!live) uy = uz = 0u;
                            const int xl = ax[0] + lo[0] - X, xh = ax[0] + hi[0] + X;
                            RowRef r = row_ranges(L, pack_cell(L, 0u, uy, uz), xl >> F, xh >> F, 1, 0, live);
                            if (L.xsorted && r.plain && r.cnt1 >= kNarrowMin && *L.xsorted)
                                narrow_x(L, r, (uint32_t)max(xl, 0), (uint32_t)xh);
                            if (is_out && act) {
                                r.st0 = L.cs[L.ncells];
                                r.cnt0 = L.cs[L.ncells + 1] - r.st0;
                                r.cnt1 = 0u;
                            }
                            const uint32_t tl = act ? r.cnt0 + r.cnt1 : 0u;
                            const uint32_t ci = scan_add(tl);
                            const uint32_t ce = carry + ci - tl;
                            if (act) {
                                rpos[k * 64u + lane] = make_uint2(r.st0 - ce, r.st1 - (ce + r.cnt0));
                                rbnd[k * 64u + lane] = ce + r.cnt0;
                            }
                            rex[k] = ce;
                            rin[k] = ce + tl;
                            carry += lane_val(ci, 63);
                        }
                    }
                    const uint32_t CT = carry;
                    // owner row of each candidate slot, as in group_count_kernel
                    uint8_t* own8 = (uint8_t*)own;
                    uint32_t wcarry = 0;
                    auto locate = [&](uint32_t cb) -> uint32_t {
                        const uint32_t w0 = cb & ~255u, wo = cb - w0;
                        if (wo == 0) {
                            wave_sync();
                            own[lane] = 0;
                            wave_sync();
#pragma unroll
                            for (uint32_t k = 0; k < kTileLayers; ++k)
                                if (rin[k] > rex[k] && rex[k] < w0 + 256u && rin[k] > w0)
                                    own8[rex[k] > w0 ? rex[k] - w0 : 0] = (uint8_t)(k * 64u + lane + 1u);
                            wave_sync();
                            wcarry = 0;
                        }
                        const uint32_t m = max(scan_max((uint32_t)own8[wo + lane]), wcarry);
                        wcarry = lane_val(m, 63);
                        const uint32_t o1 = max(m, 1u) - 1u;
                        const uint2 rp = rpos[o1];
                        const uint32_t g = cb + lane;
                        // (record 0 past the end)
                        return g < CT ? (g < rbnd[o1] ? rp.x : rp.y) + g : 0u;
                    };
                    if (CT > 0) {
                        // the next step's records load while this step's are
                        // staged (lanes past the end load record 0)
                        uint4 P = L.pts[locate(0)];
                        for (uint32_t cb = 0; cb < CT; cb += 64) {
                            const uint4 P1 = L.pts[locate(cb + 64)];
                            // candidates within reach of the box into the ring
                            const uint32_t pv[3] = {P.x, P.y, P.z};
                            int p3[3];
                            float g2 = 0.0f;
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                p3[a] = (int)(((pv[a] - o[a]) + aw.half[a]) & aw.mask[a]) - (int)aw.half[a];
                                const float g = (float)(p3[a] - min(max(p3[a], lo[a]), hi[a]));
                                g2 = __builtin_fmaf(g, g, g2);
                            }
                            uint64_t M = __ballot(g2 <= R2f);
                            if (CT - cb < 64u) M &= (1ull << (CT - cb)) - 1ull;
                            const uint32_t at = lanes_below(M, head + fill) & (kTileRing - 1u);
                            if (lane_in(M)) ring[at] = make_uint4((uint32_t)p3[0], (uint32_t)p3[1], (uint32_t)p3[2], P.w);
                            fill += (uint32_t)__popcll(M);
                            if (fill >= 64u) {
                                batch(64u);
                                fill -= 64u;
                            }
                            P = P1;
                        }
                    }
                    wave_sync();
                }
                if (fill > 0) batch(fill);
                uint32_t nq = 0;
                if (!STASH) {
                    // slot s = quad' + 4 i was counted by the lanes of quad'
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t v = bperm(row_sum(cnt[i]), (slot & 3u) << 4);
                        nq = (slot >> 2) == (uint32_t)i ? v : nq;
                    }
                    if (mine && lane < kTileQ) A.row_ptr[row] = (int64_t)nq;
                    r0 += ng;
                    if (r0 < rend) Q = group();
                    continue;
                }
                const uint32_t total = hcount;
                if (total > kTileHits && ng > 1u) {
                    // too many hits: the group again with as many queries as are
                    // expected to fit
                    nlim = max(1u, min(ng - 1u, (uint32_t)((uint64_t)ng * (kTileHits - kTileHits / 8u) / total)));
                    Q = group();
                    continue;
                }
                const bool fits = total <= kTileHits;
                if (nlim < kTileQ && total + total / ng + kTileHits / 16u <= kTileHits) ++nlim;
                const uint32_t n0 = ng;  // (the group's queries)
                r0 += ng;
                // the next group's queries load during the sort
                uint4 Qn = make_uint4(0, 0, 0, 0);
                if (r0 < rend) Qn = group();
                // ---- sort (in registers and in place): bucket counts, which
                // also give the slots' hits
                asm volatile("" : "+v"(lane));
                constexpr uint32_t kTileSteps = kTileHits / 64;
                uint64_t key[kTileSteps];
                uint32_t bs[kTileSteps];  // bucket | place in bucket << 16
                uint32_t qs0 = 0, near = 0;  // near: keys of the fullest bucket
                if (fits) {
                    uint4* h4 = (uint4*)hh;
                    for (uint32_t t = lane; t < kTileQ * kTileBuckets / 4; t += 64) h4[t] = make_uint4(0, 0, 0, 0);
                    wave_sync();
#pragma unroll
                    for (uint32_t k0 = 0; k0 < kTileSteps; k0 += 4) {
                        // (lanes past the end count into a spare bucket)
                        if (k0 * 64u < total) {
#pragma unroll
                            for (uint32_t k = k0; k < k0 + 4 && k < kTileSteps; ++k) key[k] = hb[k * 64u + lane];
#pragma unroll
                            for (uint32_t k = k0; k < k0 + 4 && k < kTileSteps; ++k) {
                                const uint32_t kh = (uint32_t)(key[k] >> 32);
                                const float v = (float)((kh >> 4) & 0xFFFFFFu);
                                const uint32_t b =
                                    ((kh >> 28) * kTileBuckets) + min((uint32_t)(v * scale), kTileBuckets - 1u);
                                bs[k] = k * 64u + lane < total ? b : kTileQ * kTileBuckets;
                            }
#pragma unroll
                            for (uint32_t k = k0; k < k0 + 4 && k < kTileSteps; ++k)
                                bs[k] |= atomicAdd(&hh[bs[k]], 1u) << 16;
                        }
                    }
                    wave_sync();
                    constexpr int kPer = kTileQ * kTileBuckets / 64;
                    uint32_t v[kPer], sum = 0, most = 0;
#pragma unroll
                    for (int k = 0; k < kPer / 4; ++k) {
                        const uint4 w = h4[lane * (kPer / 4) + k];
                        v[4 * k] = w.x;
                        v[4 * k + 1] = w.y;
                        v[4 * k + 2] = w.z;
                        v[4 * k + 3] = w.w;
                        sum += w.x + w.y + w.z + w.w;
                        most = max(max(most, max(w.x, w.y)), max(w.z, w.w));
                    }
                    near = lane_val(scan_max(most), 63);
                    uint32_t run = scan_add(sum) - sum;
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const uint32_t n = v[k];
                        v[k] = run;
                        run += n;
                    }
#pragma unroll
                    for (int k = 0; k < kPer / 4; ++k)
                        h4[lane * (kPer / 4) + k] = make_uint4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
                    if (lane == 0) hh[kTileQ * kTileBuckets] = total;
                    wave_sync();
                    qs0 = hh[slot * kTileBuckets];
                    nq = hh[(slot + 1u) * kTileBuckets] - qs0;
                } else {
                    // a row longer than the buffer, alone in its group
                    nq = total;
                }
                // ---- row sizes (lanes 0 .. n0 - 1 hold the slots) and room in
                // the stash
                const bool write = lane < n0;
                if (write) A.row_ptr[row] = (int64_t)nq;
                // the first `split` pairs, rows that end inside the wave's
                // chunk, go there, the rest to a new one: a group's pairs are
                // often as many as a chunk holds, and dropping what is left of
                // it would leave a stash of the size that keeps every row half
                // empty (1,048,576 agents in 128^3, count and write: r = 2.5
                // 0.625 -> 0.500 ms, r = 3 0.75 -> 0.69)
                uint32_t split = total, next_at = 0, kept = fits ? total : 0u;
                if (kept > 0 && cur + total > lim) {
                    const uint32_t end = qs0 + nq;
                    split = lane_val(scan_max(slot < n0 && end <= lim - cur ? end : 0u), 63);
                    kept = split;
                    if (!dry) {
                        const uint32_t grab = max(A.stash_chunk, total - split);
                        uint32_t t = 0;
                        if (lane == 0) t = atomicAdd(A.stash_ctr + region * SPHIDX_QSTRIDE, grab);
                        t = uni(t);
                        if ((uint64_t)t + grab <= A.stash_region) {
                            next_at = region * A.stash_region + t;
                            lim = next_at + grab;
                            kept = total;
                        } else {
                            dry = true;
                        }
                    }
                }
                auto place = [&](uint32_t t) -> uint32_t { return t < split ? cur + t : next_at + (t - split); };
                const bool keep = nq > 0 && qs0 + nq <= kept;
                if (kept > 0) {
                    // keys to their buckets; the keys are all in registers, so
                    // the buffer is written in place
#pragma unroll
                    for (uint32_t k0 = 0; k0 < kTileSteps; k0 += 4) {
                        if (k0 * 64u < total) {
                            uint32_t to[4];
#pragma unroll
                            for (uint32_t k = k0; k < k0 + 4 && k < kTileSteps; ++k)
                                to[k - k0] = hh[bs[k] & 0xFFFFu] + (bs[k] >> 16);
#pragma unroll
                            for (uint32_t k = k0; k < k0 + 4 && k < kTileSteps; ++k)
                                hb[k * 64u + lane < total ? to[k - k0] : kTileHits] = key[k];
                        }
                    }
                    asm volatile("" : "+v"(lane));
                    // (past the last key: nothing smaller)
                    for (uint32_t t = total + lane; t < kTileHits; t += 64) hb[t] = ~0ull;
                    wave_sync();
                    // In bucket order a key is out of place only among its
                    // bucket's keys: its rank is its place, plus the smaller
                    // keys after it, less the larger ones before it, none
                    // further away than the fullest bucket is long.
                    const uint32_t idm = sh >= 32u ? ~0u : (1u << sh) - 1u;
                    if (near <= kTileNear + 1u) {
                        // lane l takes kTileSteps keys in a row: pairs inside a
                        // lane are compared in registers, those across with the
                        // first keys of the next lane
                        uint64_t next[kTileNear];
                        uint32_t rk[kTileSteps];
#pragma unroll
                        for (uint32_t k = 0; k < kTileSteps; ++k) {
                            key[k] = hb[lane * kTileSteps + k];
                            rk[k] = lane * kTileSteps + k;
                        }
#pragma unroll
                        for (uint32_t k = 0; k < kTileNear; ++k)
                            if (k + 1u < near) next[k] = next_lane(key[k]);
                        // (one add or subtract with the comparison's mask as
                        // carry each; plain code, as the compiler keeps the wait
                        // states between the two, which it does not for inline
                        // assembly.  Leaving the loop by a break keeps it
                        // rolled, the keys in indexed registers: the 8.4
                        // M-agent timestep 7.65 ms instead of 5.11)
#pragma unroll
                        for (uint32_t d = 1; d <= kTileNear; ++d) {
                            if (d < near)
#pragma unroll
                            for (uint32_t k = 0; k < kTileSteps; ++k) {
                                const bool in = k + d < kTileSteps;
                                const bool less = (in ? key[k + d] : next[k + d - kTileSteps]) < key[k];
                                rk[k] += less ? 1u : 0u;
                                if (in)
                                    rk[k + d] -= less ? 1u : 0u;
                                else
                                    rk[k + d - kTileSteps] -= lane_in(__ballot(less) << 1) ? 1u : 0u;
                            }
                        }
                        wave_sync();
#pragma unroll
                        for (uint32_t k = 0; k < kTileSteps; ++k) hb[rk[k]] = key[k];
                        wave_sync();
                        for (uint32_t t = lane; t < kept; t += 64) {
                            const uint64_t kv = hb[t];
                            const uint32_t at = place(t);
                            A.stash_ids[at] = (uint32_t)kv & idm;
                            if (A.stash_d2) A.stash_d2[at] = (int64_t)((kv << 4) >> (64u - d2b));
                        }
                    } else {
                        for (uint32_t t = lane; t < total; t += 64) {
                            const uint64_t kv = hb[t];
                            uint32_t rk = t;
                            for (uint32_t d = 1; d < near; ++d) {
                                if (t + d < total && hb[t + d] < kv) ++rk;
                                if (d <= t && hb[t - d] > kv) --rk;
                            }
                            if (rk >= kept) continue;
                            const uint32_t at = place(rk);
                            A.stash_ids[at] = (uint32_t)kv & idm;
                            if (A.stash_d2) A.stash_d2[at] = (int64_t)((kv << 4) >> (64u - d2b));
                        }
                    }
                }
                // rows not kept are walked again by the write pass (no
                // descriptor yet: the write kernel makes it and passes a long
                // row on)
                if (write) A.soff[row] = keep ? place(qs0) : nq > 0 ? kMaxId : 0u;
                if (write && nq > 0 && !keep) list_row_again(A, qpos, false);
                cur = kept > split ? next_at + (total - split) : cur + min(split, kept);
                wave_sync();
                Q = Qn;
            }
        }
    });
}

// ---------------------------------------------------------------------------
// Pass 1, radius rows that fit the LDS buffer: collect, sort, store.

// TILES: the walk list may hold rows of tiles, which have no descriptor
// (tile_query); the kernel then has a copy of the row's code for each source.
// One query from either source was held in vector registers, 77 instead of 52,
// and a kernel with both costs short-lived waves more to start, so only the
// persistent schedule takes it in one launch, and only where the count pass can
// have used tiles (A.tiles).  The plain schedule takes the kernel without, which
// leaves such a walk list to a second launch (A.tiles 2).  Rows without a stash,
// write pass, ms, one query from either source and now: 1,048,576 uneven radii
// 1.07 -> 0.97; r = 3 cells 1.25 -> 1.11, plain launch 1.32 -> 1.22.
template <int METHOD, bool TLDS, bool FROM_LIST, bool TILES>
__global__ __launch_bounds__(256) void write_kernel(LatArgs L, TabArgs T, QArgs A) {
    extern __shared__ __align__(16) char smem[];
    const uint32_t* tab_lds = stage_table<TLDS>(T, smem);
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t cap = A.sort_cap;
    char* wb = smem + table_lds_bytes<TLDS>(T) + (size_t)wave * ((size_t)cap * 28 + 256);
    uint64_t* td = (uint64_t*)wb;
    uint64_t* sd = td + cap;
    uint32_t* ti = (uint32_t*)(sd + cap);
    uint32_t* si = ti + cap;
    uint32_t* hist = si + cap;
    uint32_t* own = hist + cap;
    if (A.row_ptr[A.Q] > A.capacity) {
        if (threadIdx.x == 0) atomicOr(L.status, SPHIDX_FLAG_CAPACITY);
        return;
    }
    const AxisWrap aw = axis_wrap(L);
    const uint32_t lane = lane_id();
    // after a stashing count pass only the rows it did not keep are walked:
    // the main launch takes the walk list, the list launch skips kept rows
    const bool stashed = A.stash_hdr[kHdrMode] != 0u;
    const bool from_walk = !FROM_LIST && stashed;
    const bool of_tiles = !FROM_LIST && A.tiles && from_walk && uni(A.stash_hdr[kHdrTiles]) != 0u;
    if (TILES ? A.tiles == 2u && !of_tiles : of_tiles) return;
    const uint32_t tiled = TILES && of_tiles ? uni(L.cs[L.ncells]) : 0u;  // rows of tiles: positions below, in the region
    const uint32_t idbits = L.n > 1 ? 32u - (uint32_t)__builtin_clz(L.n - 1u) : 0u;  // ids are below n
    const uint32_t nq = FROM_LIST ? uni(*A.list_count) : (from_walk ? uni(*A.walk_count) : A.Q);
    auto write_row = [&](const Query& s, uint32_t qi, auto from_tile) __attribute__((always_inline)) {
        constexpr bool bare = decltype(from_tile)::value;
        if (FROM_LIST && stashed && uni(A.soff[s.row]) != kMaxId) return;  // copied by the gather kernel
        if ((METHOD == kSphere || METHOD == kPaper) && (s.flags & F_VALID) && !(s.flags & F_SPHERE))
            return;  // fallback list
        const int64_t rb = A.row_ptr[s.row];
        const uint32_t rowlen = (uint32_t)(A.row_ptr[s.row + 1] - rb);
        if (rowlen == 0 || !(s.flags & F_VALID)) return;
        if ((s.flags & F_KNN) || rowlen > cap) {
            // handled by the block and top-M kernels
            if (lane == 0) {
                if (bare) {
                    uint4* d = A.desc + 4 * (size_t)qi;
                    d[0] = make_uint4(s.q[0], s.q[1], s.q[2], s.row);
                    d[1] = make_uint4(s.r, 0u, s.flags, s.tb);
                    d[2] = make_uint4(s.tend, 0u, 0u, 0u);
                    d[3] = make_uint4(0u, 0u, 0u, 0u);
                }
                A.longq[atomicAdd(A.long_count, 1u)] = qi;
            }
            return;
        }
        uint32_t n = 0, cand = 0, walked = 0;
        auto visit = [&](bool act, uint32_t p, const uint4& P) -> bool {
            const uint64_t d2 = obj_dist2(aw, s, P);
            const bool hit = act && d2 <= s.r2 && p != s.self;
            const uint64_t hm = __ballot(hit);
            if (hit) {
                const uint32_t slot = n + lanes_below(hm);
                if (slot < cap) {
                    td[slot] = d2;
                    ti[slot] = P.w;
                }
            }
            n += (uint32_t)__popcll(hm);
            return false;
        };
        walk<METHOD, TLDS, false>(L, T, tab_lds, s, false, walked, [&]() { return s.r2; },
                                         [&](const RowRef& r) -> bool {
            return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand, visit);
        });
        wave_sync();
        sort_row_store(td, ti, sd, si, hist, min(n, rowlen), s.r2, idbits, A.out_ids + rb,
                       A.out_d2 ? A.out_d2 + rb : nullptr);
        wave_sync();
    };
    for_each_query(nq, A, queue_set(A, FROM_LIST ? (int)A.list_set : (from_walk ? kQWalk : kQWrite)),
                   [&](uint32_t ti_) {
        const uint32_t qi = FROM_LIST ? uni(A.list[ti_]) : (from_walk ? uni(A.walkq[ti_]) : ti_);
        if constexpr (TILES) {
            if (qi < tiled) {
                write_row(tile_query(L, T, A, qi), qi, std::true_type());
                return;
            }
        }
        write_row(load_query(L, A, qi), qi, std::false_type());
    });
}

// ---------------------------------------------------------------------------
// Pass 1, K-NN rows and long radius rows: sorted top-M in LDS with the
// shrinking bound, in windows of at most `cap` entries (each window takes
// the M smallest pairs above the previous window's last one).

template <int METHOD, bool TLDS, bool FROM_LIST>
__global__ __launch_bounds__(256) void topm_kernel(LatArgs L, TabArgs T, QArgs A) {
    extern __shared__ __align__(16) char smem[];
    const uint32_t* tab_lds = stage_table<TLDS>(T, smem);
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t cap = A.sort_cap;
    char* wb = smem + table_lds_bytes<TLDS>(T) + (size_t)wave * ((size_t)cap * 24 + 64 * 12 + 256);
    uint64_t* tdA = (uint64_t*)wb;
    uint64_t* tdB = tdA + cap;
    uint64_t* bd = tdB + cap;
    uint32_t* tiA = (uint32_t*)(bd + 64);
    uint32_t* tiB = tiA + cap;
    uint32_t* bi = tiB + cap;
    uint32_t* own = bi + 64;
    if (A.row_ptr[A.Q] > A.capacity) {
        if (threadIdx.x == 0) atomicOr(L.status, SPHIDX_FLAG_CAPACITY);
        return;
    }
    const AxisWrap aw = axis_wrap(L);
    const uint32_t lane = lane_id();
    // every query, unless a stashing count pass kept rows and the copy placed
    // them: then only the rows it could not keep, which it listed on the walk
    // list (when this call asks for dist^2 and the stash holds none, the copy
    // placed nothing and every row is searched)
    const bool from_walk = !FROM_LIST && A.stash_hdr[kHdrMode] != 0u && !(A.out_d2 && A.stash_hdr[kHdrHasD2] == 0u);
    // (FROM_LIST: the count pass's big list, then the write kernel's long rows)
    const uint32_t nbig = FROM_LIST || from_walk ? uni(*A.big_count) : 0u;
    const uint32_t* rest = FROM_LIST ? A.list : A.walkq;
    const uint32_t nq = FROM_LIST ? nbig + uni(*A.list_count) : from_walk ? nbig + uni(*A.walk_count) : A.Q;
    for_each_query(nq, A, queue_set(A, kQTopm), [&](uint32_t ti_) {
        const uint32_t qi =
            ti_ < nbig ? uni(A.bigq[ti_]) : FROM_LIST || from_walk ? uni(rest[ti_ - nbig]) : ti_;
        const Query s = load_query(L, A, qi);
        if (!FROM_LIST && !(s.flags & F_KNN)) return;
        const int64_t rb = A.row_ptr[s.row];
        const uint32_t rowlen = (uint32_t)(A.row_ptr[s.row + 1] - rb);
        if (rowlen == 0 || !(s.flags & F_VALID)) return;
        // long radius rows the block-per-row kernel takes
        if (FROM_LIST && A.long_waves > 1 && !(s.flags & (F_KNN | F_WINDOW))) return;
        uint64_t* td = tdA;
        uint64_t* ud = tdB;
        uint32_t* tix = tiA;
        uint32_t* uix = tiB;
        bool has_lower = false;
        uint64_t ld = 0;
        uint32_t li = 0;
        uint32_t written = 0;
        while (written < rowlen) {
            const uint32_t M = min(cap, rowlen - written);
            const uint32_t target = written + M;
            uint64_t B = first_bound(L, s, target, rowlen);
            if (M <= 64) {
                // ---- a window of at most 64 in registers
                uint64_t rd;
                uint32_t ri;
                const uint32_t got = topm_registers<METHOD, TLDS>(L, T, tab_lds, s, aw, own, M, B, has_lower, ld, li,
                                                                   rd, ri);
                if (lane < got) {
                    A.out_ids[rb + written + lane] = ri;
                    if (A.out_d2) A.out_d2[rb + written + lane] = (int64_t)rd;
                }
                if (got == 0) break;
                has_lower = true;
                ld = lane_val64(rd, got - 1u);
                li = lane_val(ri, got - 1u);
                written += got;
                continue;
            }
            uint32_t m = 0;
            uint64_t bdd = kMaxD2;
            uint32_t bii = kMaxId;
            uint32_t cand = 0, walked = 0;
            auto visit = [&](bool act, uint32_t p, const uint4& P) -> bool {
                const uint64_t d2 = obj_dist2(aw, s, P);
                const uint32_t id = P.w;
                bool cv = act && d2 <= B && p != s.self;
                if (cv && has_lower) cv = key_less(ld, li, d2, id);
                if (cv && m == M) cv = key_less(d2, id, bdd, bii);
                const uint64_t bm = __ballot(cv);
                if (bm == 0) return false;
                const uint32_t nb = (uint32_t)__popcll(bm);
                uint64_t cd = cv ? d2 : kMaxD2;
                uint32_t ci = cv ? id : kMaxId;
                wave_sort64(cd, ci);
                bd[lane] = cd;
                bi[lane] = ci;
                wave_sync();
                const uint32_t nm = min(M, m + nb);
                // merge: an element's place = own index + elements of the
                // other sorted list that are smaller (ids are unique)
                for (uint32_t t = lane; t < m; t += 64) {
                    const uint64_t xd = td[t];
                    const uint32_t xi = tix[t];
                    uint32_t lo = 0, hi = nb;
                    while (lo < hi) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (key_less(bd[mid], bi[mid], xd, xi))
                            lo = mid + 1;
                        else
                            hi = mid;
                    }
                    if (t + lo < nm) {
                        ud[t + lo] = xd;
                        uix[t + lo] = xi;
                    }
                }
                if (lane < nb) {
                    uint32_t lo = 0, hi = m;
                    while (lo < hi) {
                        const uint32_t mid = (lo + hi) >> 1;
                        if (key_less(td[mid], tix[mid], cd, ci))
                            lo = mid + 1;
                        else
                            hi = mid;
                    }
                    if (lane + lo < nm) {
                        ud[lane + lo] = cd;
                        uix[lane + lo] = ci;
                    }
                }
                wave_sync();
                uint64_t* sd = td;
                td = ud;
                ud = sd;
                uint32_t* si = tix;
                tix = uix;
                uix = si;
                m = nm;
                if (m == M) {
                    bdd = uni64(td[M - 1]);
                    bii = uni(tix[M - 1]);
                }
                return false;
            };
            // every object within B is visited and nothing beyond B is kept,
            // so M kept means they are the M nearest above the lower bound
            for (;;) {
                walk<METHOD, TLDS, true>(L, T, tab_lds, s, false, walked, [&]() { return m == M ? bdd : B; },
                                                [&](const RowRef& r) -> bool {
                    return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand, visit);
                });
                if (m == M || B >= s.r2) break;
                B = min(s.r2, B + B + (B >> 2) + 1u);  // radius x1.5
                m = 0;
                bdd = kMaxD2;
                bii = kMaxId;
            }
            wave_sync();
            const uint32_t got = min(m, M);
            store_sorted(A, td, tix, got, rb + written);
            if (got == 0) break;
            has_lower = true;
            ld = uni64(td[got - 1]);
            li = uni(tix[got - 1]);
            written += got;
            wave_sync();
        }
    });
}

// ---------------------------------------------------------------------------
// Both passes, radius rows longer than a wavefront's LDS row buffer: one block
// of W waves per row.  Wave w walks the row's table entries in 64-entry steps
// w, w + W, ..., tests their candidates and appends its hits to a block-wide
// LDS buffer (one LDS atomic per wave step).  The block then orders the row by
// (dist^2, id) with one bucket sort (block_sort_store) and stores it; the
// write pass orders a row past the buffer's kLongCap pairs by shells of
// distance (shell_row).  The top-M kernel takes such rows only where many of
// their objects lie at one distance (F_WINDOW), and all of them where one
// wavefront per row is asked for.

// Exclusive scan over the block of one value per thread; `wsum` holds one
// word per wavefront.
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* wsum) {
    const uint32_t wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t incl = scan_add(v);
    if (lane_id() == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t off = 0;
    for (uint32_t w = 0; w < nw; ++w) off += w < wave ? wsum[w] : 0u;
    __syncthreads();
    return off + incl - v;
}

// Order the block's n <= kLongCap pairs by (dist^2, id) and store them at dst;
// kb holds their distances above base, at most span.  One counting sort over
// about n buckets (floor(n v / (v_max + 1)) of v = the top 24 bits of the
// distance: monotone), the pairs held in registers and put in place, then each
// one's rank from its place and the pairs near it (as the tile kernel's).
// A pair is one key, distance << idbits | id, and `side` holds the bucket
// counts; WIDE, where a distance leaves no room for an id: kb holds the
// distances, `side` the ids, and the counts take kb's place while the pairs are
// in registers (three barriers more, the same LDS).  kb[-kNearPad .. n + kNearPad)
// is the block's.
constexpr uint32_t kNearPad = 8;

template <int W, bool WIDE>
__device__ void block_sort_store(uint64_t* kb, uint32_t* side, uint32_t* ctl, uint32_t n, uint64_t span,
                                 uint32_t idbits, uint32_t* dst_ids, int64_t* dst_d2, uint64_t base = 0) {
    constexpr uint32_t nt = 64u * W, kPer = kLongCap / nt;
    const uint32_t tid = threadIdx.x;
    const uint32_t sbits = span ? 64u - (uint32_t)__builtin_clzll(span) : 0u;
    const uint32_t low = WIDE ? 0u : idbits;
    const uint32_t vs = min(sbits > 24u ? sbits - 24u : 0u, 63u - low);
    const float scale = (float)n / ((float)(span >> vs) + 1.0f);
    uint32_t* hist = WIDE ? (uint32_t*)kb : side;
    uint64_t key[kPer];
    uint32_t bs[kPer];  // bucket | place in bucket << 16
    if (WIDE) {
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k) {
            const uint32_t t = tid + k * nt;
            if (k * nt < n && t < n) key[k] = kb[t];
        }
        __syncthreads();
    }
    for (uint32_t t = tid; t < n; t += nt) hist[t] = 0u;
    if (tid == 0) ctl[3] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t t = tid + k * nt;
        if (k * nt < n && t < n) {
            if (!WIDE) key[k] = kb[t];
            const uint32_t b = min((uint32_t)((float)(uint32_t)(key[k] >> (low + vs)) * scale), n - 1u);
            bs[k] = b | (atomicAdd(&hist[b], 1u) << 16);
        }
    }
    __syncthreads();
    // bucket starts: each thread owns a run of buckets
    {
        const uint32_t per = (n + nt - 1u) / nt, b0 = tid * per;
        uint32_t sum = 0, most = 0;
        for (uint32_t k = 0; k < per; ++k)
            if (b0 + k < n) {
                sum += hist[b0 + k];
                most = max(most, hist[b0 + k]);
            }
        most = lane_val(scan_max(most), 63);
        if ((tid & 63u) == 0) atomicMax(&ctl[3], most);
        uint32_t run = block_scan_excl(sum, ctl + 4);
        for (uint32_t k = 0; k < per; ++k)
            if (b0 + k < n) {
                const uint32_t c = hist[b0 + k];
                hist[b0 + k] = run;
                run += c;
            }
    }
    __syncthreads();
    if (WIDE) {
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k)
            if (k * nt < n && tid + k * nt < n) bs[k] = hist[bs[k] & 0xFFFFu] + (bs[k] >> 16);
        __syncthreads();
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (k * nt < n && tid + k * nt < n) {
            const uint32_t to = WIDE ? bs[k] : hist[bs[k] & 0xFFFFu] + (bs[k] >> 16);
            kb[to] = key[k];
            // (the ids follow, in the keys' registers)
            if (WIDE) key[k] = side[tid + k * nt];
        }
    if (WIDE) {
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < kPer; ++k)
            if (k * nt < n && tid + k * nt < n) side[bs[k]] = (uint32_t)key[k];
    }
    if (!WIDE && tid < kNearPad) {
        // nothing before the first key is larger, nothing after the last smaller
        kb[(int)tid - (int)kNearPad] = 0ull;
        kb[n + tid] = ~0ull;
    }
    __syncthreads();
    const uint32_t near = ctl[3];  // pairs of the fullest bucket
    const uint64_t idm = (1ull << idbits) - 1ull;
    for (uint32_t t = tid; t < n; t += nt) {
        const uint64_t kv = kb[t];
        const uint32_t iv = WIDE ? side[t] : (uint32_t)(kv & idm);
        uint32_t rk = t;
        if (WIDE) {
            for (uint32_t d = 1; d < near; ++d) {
                if (t + d < n && key_less(kb[t + d], side[t + d], kv, iv)) ++rk;
                if (d <= t && key_less(kv, iv, kb[t - d], side[t - d])) --rk;
            }
        } else if (near <= kNearPad + 1u) {
            for (int d = 1; d < (int)near; ++d)
                rk += (kb[(int)t + d] < kv ? 1u : 0u) - (kb[(int)t - d] > kv ? 1u : 0u);
        } else {
            for (uint32_t d = 1; d < near; ++d) {
                if (t + d < n && kb[t + d] < kv) ++rk;
                if (d <= t && kb[t - d] > kv) --rk;
            }
        }
        dst_ids[rk] = iv;
        if (dst_d2) dst_d2[rk] = (int64_t)((kv >> low) + base);
    }
}

// A radius row of more than kLongCap pairs, by one block in two walks (write
// pass): the first counts its hits per distance bucket (dist^2 >> sh, sh such
// that r^2 falls below kShellBuckets), the second writes each hit's sorted
// position into the row's own output, grouped by bucket; then runs of buckets
// of at most kShellCap pairs (shells, centre to edge) are read back into LDS,
// their objects' distances computed again, ordered by the block sort and
// stored in place.  The row needs no memory but its output.  Returns false,
// with nothing written, when one bucket alone holds more than kShellCap pairs
// (many objects at one distance): such a row is left to the windowed kernel.
// What bounds it is the walk's and the block sort's instruction issue and LDS
// traffic.  Before, every such row took one window of sort_cap pairs after
// another on one wavefront, each window walking the whole row again: 512 rows
// of about 20,000 pairs (20 objects per cell, 7 cells, clipped 32^3) took
// 103 ms in all; now 0.59 ms.
// Keys (block_sort_store) hold a shell's distances from its first bucket's on,
// so they pack far beyond a whole row's; WIDE where so few buckets pack that
// shells would be cut by them and not by their pairs (shells_wide): 512 rows of
// 12,500 pairs at r = 32 cells, 256 buckets to a key, 0.56 ms, wide 0.60.
constexpr uint32_t kShellCap = 2304, kShellBuckets = 2048;

// log2 of the distances per bucket.
__device__ __forceinline__ uint32_t shell_shift(uint64_t r2) {
    const uint32_t rbits = r2 ? 64u - (uint32_t)__builtin_clzll(r2) : 0u;
    return rbits > 11u ? rbits - 11u : 0u;  // kShellBuckets = 2^11
}
// Buckets whose distances, from the first's on, pack with an id (0: not one's).
__device__ __forceinline__ uint32_t shell_buckets(uint64_t r2, uint32_t idbits) {
    const uint32_t used = shell_shift(r2) + idbits;
    return used > 64u ? 0u : 64u - used >= 11u ? kShellBuckets : 1u << (64u - used);
}
__device__ __forceinline__ bool shells_wide(uint64_t r2, uint32_t idbits, uint32_t rowlen) {
    const uint32_t b = shell_buckets(r2, idbits);
    return b == 0u || (b < kShellBuckets && (uint64_t)(kShellBuckets / b) * kShellCap > 2ull * rowlen);
}

template <int METHOD, int W, bool WIDE>
__device__ bool shell_row(const LatArgs& L, const TabArgs& T, const QArgs& A, const AxisWrap& aw, const Query& s,
                          int64_t rb, uint32_t rowlen, uint32_t idbits, uint64_t* kb, uint32_t* side, uint32_t* bkt,
                          uint32_t* own, uint32_t* ctl) {
    const uint32_t tid = threadIdx.x, nt = blockDim.x, wave = tid >> 6, nw = nt >> 6;
    const uint32_t sh = shell_shift(s.r2);
    const uint32_t most_b = WIDE ? kShellBuckets : shell_buckets(s.r2, idbits);
    uint32_t cand = 0, walked = 0;
    auto walk_row = [&](auto&& visit) {
        walk<METHOD, false, false>(L, T, nullptr, s, false, walked, [&]() { return s.r2; },
                                   [&](const RowRef& r) -> bool {
            return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand, visit);
        }, 64u * wave, 64u * nw);
    };
    for (uint32_t t = tid; t < kShellBuckets; t += nt) bkt[t] = 0u;
    if (tid == 0) ctl[3] = 0u;
    __syncthreads();
    walk_row([&](bool act, uint32_t p, const uint4& P) -> bool {
        const uint64_t d2 = obj_dist2(aw, s, P);
        if (act && d2 <= s.r2 && p != s.self) atomicAdd(&bkt[(uint32_t)(d2 >> sh)], 1u);
        return false;
    });
    __syncthreads();
    {
        // bucket starts, each thread owning a run of buckets
        const uint32_t per = kShellBuckets / nt, b0 = tid * per;
        uint32_t sum = 0, most = 0;
        for (uint32_t k = 0; k < per; ++k) {
            sum += bkt[b0 + k];
            most = max(most, bkt[b0 + k]);
        }
        if (most > kShellCap) ctl[3] = 1u;
        uint32_t run = block_scan_excl(sum, ctl + 4);
        for (uint32_t k = 0; k < per; ++k) {
            const uint32_t c = bkt[b0 + k];
            bkt[b0 + k] = run;
            run += c;
        }
    }
    __syncthreads();
    if (ctl[3]) return false;
    uint32_t* pos = A.out_ids + rb;
    walk_row([&](bool act, uint32_t p, const uint4& P) -> bool {
        const uint64_t d2 = obj_dist2(aw, s, P);
        if (act && d2 <= s.r2 && p != s.self) {
            const uint32_t t = atomicAdd(&bkt[(uint32_t)(d2 >> sh)], 1u);
            if (t < rowlen) pos[t] = p;
        }
        return false;
    });
    // (the block's own stores, seen by all of it after the barrier; each
    // bucket's cursor now ends at the next one's start)
    __syncthreads();
    for (uint32_t b = 0, t0 = 0; t0 < rowlen;) {
        // the shell: buckets b .. e - 1, as many as fit
        uint32_t lo = b + 1u, hi = min(kShellBuckets, b + most_b);  // the least e, the most
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1u) >> 1;
            if (bkt[mid - 1u] - t0 <= kShellCap)
                lo = mid;
            else
                hi = mid - 1u;
        }
        const uint32_t e = lo, n = min(bkt[e - 1u], rowlen) - t0;
        const uint64_t base = (uint64_t)b << sh;
        const uint64_t span = min(s.r2, ((uint64_t)e << sh) - 1ull) - base;
        for (uint32_t t = tid; t < n; t += nt) {
            const uint4 P = L.pts[pos[t0 + t]];
            const uint64_t d2 = obj_dist2(aw, s, P) - base;
            kb[t] = WIDE ? d2 : (d2 << idbits) | P.w;
            if (WIDE) side[t] = P.w;
        }
        __syncthreads();
        if (n > 0)
            block_sort_store<W, WIDE>(kb, side, ctl, n, span, idbits, A.out_ids + rb + t0,
                                      A.out_d2 ? A.out_d2 + rb + t0 : nullptr, base);
        __syncthreads();
        t0 += n;
        b = e;
        if (e >= kShellBuckets) break;
    }
    return true;
}

// COUNT: the count pass's form.  The rows come from the list of rows the
// setup expected to be long; the block counts the row, writes its size and,
// when it holds at most kLongCap pairs and the stash has room, orders it into
// the stash (one allocation per row) for the write pass to copy; otherwise
// the row goes on the big or the walk list like any row the count pass did not
// keep.  The write pass's form takes the big list and the long-row list.
// A row's hits are kept as keys dist^2 << idbits | id, or, where r^2 leaves no
// room for an id in 64 bits (16 fractional bits: past r = 16 cells at 16.7 M
// objects), as distances with the ids beside them, in the same LDS: counted
// only, and walked thrice more by the write pass, 8,192 such rows of about
// 3,100 pairs (16.7 M objects, r = 20 cells) took 2.18 ms and of 2,090 (33 M,
// r = 14) 1.27 ms; kept, 1.47 and 0.48 ms.
// A row is a chain of barriers with little work between them, so rows in flight
// are what counts: 12 bytes of LDS per pair (keys, bucket counts) let four
// blocks share a CU, where pairs with an index each, 20 bytes, let two: 16,400
// rows of about 1,100 pairs (a service's batch of 65,536) 528 -> 475 us.
// (Registers for the blocks that the LDS leaves room for: four per CU are W
// wavefronts per SIMD.)
template <int METHOD, bool COUNT, int W>
__global__ __launch_bounds__(64 * W, COUNT || W < 8 ? W : 6) void long_kernel(LatArgs L, TabArgs T, QArgs A) {
    extern __shared__ __align__(16) char smem[];
    uint64_t* kb = (uint64_t*)smem + kNearPad;        // hits in arrival order
    uint32_t* side = (uint32_t*)(kb + kLongCap + kNearPad);  // bucket counts, or the hits' ids
    uint32_t* ctl = side + kLongCap;  // [0] hits so far, [1] list entry taken, [2] stash offset, [3] fullest bucket,
                                      // [4, 12) wave sums
    const uint32_t wave = threadIdx.x >> 6, nw = W, lane = lane_id();
    uint32_t* own = ctl + 16 + wave * 64;
    static_assert(kShellCap * 12 + kShellBuckets * 4 <= kLongCap * 12, "a shell's buffers fit the row's");
    if (!COUNT && A.row_ptr[A.Q] > A.capacity) return;  // (the write kernel sets the flag)
    const uint32_t nbig = COUNT ? 0u : uni(*A.big_count);
    const uint32_t nq = nbig + uni(*A.list_count);
    if (nq == 0) return;
    const AxisWrap aw = axis_wrap(L);
    const uint32_t idbits = L.n > 1 ? 32u - (uint32_t)__builtin_clz(L.n - 1u) : 1u;
    uint32_t* qc = queue_set(A, (int)A.list_set);
    const uint32_t region = blockIdx.x % SPHIDX_NREGION;
    for (;;) {
        if (threadIdx.x == 0) {
            ctl[1] = atomicAdd(qc, 1u);
            ctl[0] = 0u;
        }
        __syncthreads();
        const uint32_t t = uni(ctl[1]);
        if (t >= nq) break;
        const uint32_t qi = uni(t < nbig ? A.bigq[t] : A.list[t - nbig]);
        const Query s = load_query(L, A, qi);
        int64_t rb = 0;
        uint32_t rowlen = kLongCap;
        if (!COUNT) {
            rb = A.row_ptr[s.row];
            rowlen = (uint32_t)(A.row_ptr[s.row + 1] - rb);
        }
        // the same for every wave of the block
        const bool mine = (s.flags & F_VALID) && !(s.flags & (F_KNN | F_WINDOW)) && rowlen > 0;
        const bool wide = (s.r2 >> (64u - idbits)) != 0;
        if (mine && rowlen <= kLongCap) {
            uint32_t cand = 0, walked = 0;
            auto visit = [&](bool act, uint32_t p, const uint4& P) -> bool {
                const uint64_t d2 = obj_dist2(aw, s, P);
                const bool hit = act && d2 <= s.r2 && p != s.self;
                const uint64_t hm = __ballot(hit);
                if (hm) {
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(&ctl[0], (uint32_t)__popcll(hm));
                    base = uni(base);
                    const uint32_t slot = lanes_below(hm, base);
                    if (hit && slot < kLongCap) {
                        kb[slot] = wide ? d2 : (d2 << idbits) | P.w;
                        if (wide) side[slot] = P.w;
                    }
                }
                return false;
            };
            walk<METHOD, false, false>(L, T, nullptr, s, false, walked, [&]() { return s.r2; },
                                       [&](const RowRef& r) -> bool {
                return for_candidates(L, r.st0, r.cnt0, r.st1, r.cnt1, own, cand, visit);
            }, 64u * wave, 64u * nw);
        }
        __syncthreads();
        if (COUNT) {
            const uint32_t n = (s.flags & F_VALID) ? ctl[0] : 0u;
            if (threadIdx.x == 0) {
                A.row_ptr[s.row] = (int64_t)n;
                uint32_t off = 0u;  // empty rows: nothing to copy
                if (n > 0) {
                    off = kMaxId;
                    if (n <= kLongCap && A.stash) {
                        const uint32_t c = atomicAdd(A.stash_ctr + region * SPHIDX_QSTRIDE, n);
                        if ((uint64_t)c + n <= A.stash_region) off = region * A.stash_region + c;
                    }
                    if (off == kMaxId) list_row_again(A, qi, n > A.sort_cap);
                }
                A.soff[s.row] = off;
                ctl[2] = off;
            }
            __syncthreads();
            const uint32_t off = ctl[2];
            if (n > 0 && off != kMaxId) {
                int64_t* d2 = A.stash_d2 ? A.stash_d2 + off : nullptr;
                if (wide)
                    block_sort_store<W, true>(kb, side, ctl, n, s.r2, idbits, A.stash_ids + off, d2);
                else
                    block_sort_store<W, false>(kb, side, ctl, n, s.r2, idbits, A.stash_ids + off, d2);
            }
        } else if (mine) {
            if (rowlen <= kLongCap) {
                const uint32_t n = min(ctl[0], rowlen);
                int64_t* d2 = A.out_d2 ? A.out_d2 + rb : nullptr;
                if (wide)
                    block_sort_store<W, true>(kb, side, ctl, n, s.r2, idbits, A.out_ids + rb, d2);
                else
                    block_sort_store<W, false>(kb, side, ctl, n, s.r2, idbits, A.out_ids + rb, d2);
            } else {
                uint32_t* bkt = (uint32_t*)(kb + kShellCap + kNearPad);
                uint32_t* sd = bkt + kShellBuckets;
                const bool done =
                    shells_wide(s.r2, idbits, rowlen)
                        ? shell_row<METHOD, W, true>(L, T, A, aw, s, rb, rowlen, idbits, kb, sd, bkt, own, ctl)
                        : shell_row<METHOD, W, false>(L, T, A, aw, s, rb, rowlen, idbits, kb, sd, bkt, own, ctl);
                if (!done && threadIdx.x == 0)
                    ((uint32_t*)(A.desc + 4 * (size_t)qi))[6] = s.flags | F_WINDOW;
            }
        }
        __syncthreads();
    }
}

// Pass 1 with the stash: copy each kept row into place.  A wavefront takes
// `rows` (at most 64) consecutive output rows and reads each one's stash offset
// (kept per output row) and its place from row_ptr.  Their objects are numbered
// in row order (a prefix sum), and each lane copies every 64th of them: its row
// is the last whose first number is at most the object's, found by a binary
// search over the starts kept in LDS (read-only, so steps need no barrier and
// four are in flight).  The writes are then one sequential stream per wavefront
// and each stash row is one contiguous read; rows come out of the count pass in
// lattice order, which is not the output's order for all-agents queries, and
// writing rows scattered over the output costs more than reading them scattered.
// With few rows a group is shared by `splits` wavefronts, which take its
// 256-object blocks in turn (the host's rule: copy_shape).
// Rows the count pass could not keep are left to the write kernel (offset ~0).
// When the write wants dist^2 and the stash lacks it, every kept row is walked
// again instead, and the walk list takes query slots: then the wavefront takes
// consecutive query slots and finds each one's output row (a group's first
// wavefront lists them, the others have nothing to do).
// First of the write pass, its first block also clears that pass's counters:
// the write-side queue sets and the long-row list; the descriptors, the
// fallback and walk lists, the stash header and the stash counters stay as the
// count pass left them.
__global__ __launch_bounds__(256) void gather_kernel(QArgs A, const uint4* pts, uint32_t* status, uint32_t rows,
                                                     uint32_t splits) {
    __shared__ uint32_t starts_all[4 * 64];
    if (blockIdx.x == 0)
        clear_counters(A.queues, SPHIDX_NQUEUE * SPHIDX_QSTRIDE, (SPHIDX_NQSETS * SPHIDX_NQUEUE + 1u) * SPHIDX_QSTRIDE,
                       nullptr, make_uint4(0, 0, 0, 0), 0u);
    const uint32_t* hdr = A.stash_hdr;
    if (hdr[kHdrMode] == 0u) return;
    if (A.row_ptr[A.Q] > A.capacity) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(status, SPHIDX_FLAG_CAPACITY);
        return;
    }
    const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
    uint32_t* starts = starts_all + wave * 64;
    const uint32_t w = blockIdx.x * (blockDim.x >> 6) + wave;
    const uint32_t grp = w / splits, part = w - grp * splits;
    const uint64_t q0 = (uint64_t)grp * rows;
    if (q0 >= A.Q) return;
    const uint32_t* s_ids = (const uint32_t*)A.stash_base;
    const bool has_d2 = hdr[kHdrHasD2] != 0u;
    const int64_t* s_d2 = (const int64_t*)(A.stash_base + hdr[kHdrD2Off] * (size_t)256);
    // walk again (dist^2 wanted, not stashed): by query slot; else by output row
    const bool again = A.out_d2 && !has_d2;
    if (again && part != 0u) return;
    const uint64_t qi = q0 + lane;
    uint32_t len = 0, src = 0;
    int64_t dst = 0;
    if (lane < rows && qi < A.Q) {
        // the output row: the object's id for all-agents queries (their
        // processing order is the sorted order), else the query index
        const uint32_t row = (again && A.qx == nullptr) ? pts[qi].w : (uint32_t)qi;
        src = A.soff[row];
        if (src != kMaxId) {
            dst = A.row_ptr[row];
            len = (uint32_t)(A.row_ptr[row + 1] - dst);
            if (len > 0 && again) {
                // the stash holds no dist^2 for this row: it is walked again,
                // by the main write kernel (from the walk list) or, for a row
                // off the sphere tables, by the list kernels, which walk rows
                // whose offset says "not kept"; marked so once, a later write
                // does not list it again
                A.soff[row] = kMaxId;
                A.walkq[atomicAdd(A.walk_count, 1u)] = (uint32_t)qi;
                len = 0;
            }
        }
    }
    const uint32_t incl = scan_add(len);
    const uint32_t total = lane_val(incl, 63);
    const uint32_t excl = incl - len;
    starts[lane] = excl;
    wave_sync();
    // object g of query o is at stash sbase[o] + g and output dbase[o] + g
    const uint32_t sbase = src - excl;
    const uint64_t dbase = (uint64_t)(dst - (int64_t)excl);
    const bool want_d2 = A.out_d2 != nullptr;
    constexpr uint32_t kSteps = 4;
    for (uint32_t cb = 64u * kSteps * part; cb < total; cb += 64u * kSteps * splits) {
        uint32_t v[kSteps];
        int64_t d2[kSteps], dp[kSteps];
#pragma unroll
        for (uint32_t k = 0; k < kSteps; ++k) {
            const uint32_t g = cb + 64u * k + lane;
            // the last query whose first object number is <= g (a query with
            // an empty row shares its start with the next, which wins)
            uint32_t o = 0;
#pragma unroll
            for (uint32_t step = 32; step; step >>= 1)
                if (starts[o + step] <= g) o += step;
            const uint32_t sp = bperm(sbase, o) + g;
            dp[k] = (int64_t)(((uint64_t)bperm((uint32_t)(dbase >> 32), o) << 32) | bperm((uint32_t)dbase, o)) + g;
            v[k] = 0u;
            d2[k] = 0;
            if (g < total) {
                v[k] = s_ids[sp];
                if (want_d2) d2[k] = s_d2[sp];
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kSteps; ++k) {
            if (cb + 64u * k + lane < total) {
                A.out_ids[dp[k]] = v[k];
                if (want_d2) A.out_d2[dp[k]] = d2[k];
            }
        }
    }
}

// Rows per wavefront and wavefronts per group of rows of the stash copy.  A
// wavefront's objects go in dependent rounds of 256 (a load latency each), so
// what matters is that one wavefront's rounds stay few while the chip holds
// every wavefront at once: kCopyWaves of them (32 per CU), from one row each,
// shared by up to 8 wavefronts, for a service's small batch (rows of up to
// thousands of pairs) to 64 rows each for an all-objects step.  With 64 rows
// per wavefront whatever the batch, the copy of 214 mixed rows took 130 us on
// four wavefronts and that of 65,536 rows (20 M pairs) 219 us; by this rule
// the batch of 214 went from 279 to 138 us in all and that of 65,536 from
// 1,410 to 1,261 (1,406, 1,330, 1,285, 1,261, 1,260, 1,260 us at 1, 2, 4, 8,
// 16 and 32 K wavefronts).
constexpr uint32_t kCopyWaves = 8192;
struct CopyShape {
    uint32_t rows, splits;
};
CopyShape copy_shape(uint32_t Q) {
    CopyShape c{1u, 1u};
    while (c.rows < 64u && (uint64_t)Q > (uint64_t)kCopyWaves * c.rows) c.rows *= 2u;
    while (c.splits < 8u && (uint64_t)Q * c.splits * 2u <= kCopyWaves) c.splits *= 2u;
    return c;
}

// Wavefronts (blocks) of the tile kernel that the chip holds.
uint32_t tile_blocks() { return (uint32_t)device_cu_count() * std::min(12u, 160u * 1024u / kTileLds); }

// Whether the count pass takes the tile kernel, and its strips and chunks:
// all-agents queries of one radius on the sphere tables, in groups, whose keys
// fit.  The line lies at rows of 12 to 160 expected pairs, and again from nine
// tenths of the grouped kernel's buffer (sort_cap) up to the length from which
// one block counts a row: count + write in ms, grouped against tiles, cyclic
// 64^3 and 128^3: 2 pairs 0.311 / 0.310 (1 M queries) but 0.076 / 0.080 (33 K,
// one launch more); 12 pairs 0.423 / 0.369; 33 pairs 0.691 / 0.522; 57 pairs
// 0.203 / 0.177; 134 pairs 2.11 / 1.76; 179 pairs 0.457 / 0.507; 226 pairs
// 1.88 / 2.11 (groups of four queries waste the matrix rows); 250 pairs
// 7.41 / 2.48 and 289 pairs 1.33 / 0.40 (the grouped kernel leaves rows past
// its buffer to the write pass); 349 pairs 2.21 / 2.70.
bool tile_plan(const LatArgs& L, const TabArgs& T, const QArgs& q, TileArgs& TA) {
    if (!q.group || q.qx || q.rad || q.mode != SPHIDX_MODE_RADIUS || q.stats || q.select || q.method_out || !T.has ||
        T.paper || q.Q < kTileMinQ)
        return false;
    const uint32_t rm = q.rad_u;
    if (rm > T.rmax) return false;
    auto bits = [](uint64_t v) { return v ? 64u - (uint32_t)__builtin_clzll(v) : 0u; };
    TA.d2bits = std::max(1u, bits((uint64_t)rm * rm));
    if (4u + TA.d2bits + bits(L.n > 1 ? L.n - 1u : 0u) > 64u) return false;
    const uint64_t E = 1ull << L.F, reach = (rm + E - 1) >> L.F;
    const double load = (double)L.n / (double)L.ncells, rc = (double)rm / (double)E;
    const double hits = load * 4.18879 * rc * rc * rc;
    if (hits < 12.0 || hits > 320.0 || (hits > 160.0 && hits < 0.9 * q.sort_cap)) return false;
    // strips about as wide as the side of the cube that holds a group
    const double side = std::cbrt((double)kTileQ / load);
    TA.wy = side >= 2.5 ? 2u : side >= 1.4 ? 1u : 0u;
    TA.wz = side >= 3.5 ? 2u : side >= 1.7 ? 1u : 0u;
    TA.cl = 31u - (uint32_t)__builtin_clz(kTileCells) - TA.wy - TA.wz;
    uint32_t* w[3] = {&TA.cl, &TA.wy, &TA.wz};
    for (int a = 0; a < 3; ++a) {
        *w[a] = std::min(*w[a], L.lg[a]);
        // no candidate row or run repeats a cell, no difference leaves its
        // image, and offsets stay below 2^23
        auto ok = [&]() {
            const uint64_t c = 1ull << *w[a];
            if (((c + reach + 2) << L.F) > (1ull << 23)) return false;
            return !((L.cyc >> a) & 1u) || 2 * (c + reach + 1) <= (1ull << L.lg[a]);
        };
        while (*w[a] > 0 && !ok()) --*w[a];
        if (!ok()) return false;
    }
    TA.nchunks = L.ncells >> (TA.cl + TA.wy + TA.wz);
    TA.part = std::min(256u, std::max(kTileQ, q.Q / (tile_blocks() * 4u) / kTileQ * kTileQ));
    TA.mean = q.Q / TA.nchunks;
    return TA.nchunks <= (1u << 22);
}

hipError_t launch_tiles(const LatArgs& L, const QArgs& q, const TileArgs& TA, hipStream_t st) {
    tile_items_kernel<<<(TA.nchunks + 255) / 256, 256, 0, st>>>(L, q, TA, q.longq, q.item_count);
    LatArgs l = L;
    QArgs a = q;
    a.tile = 1;  // work items per queue grab
    TileArgs ta = TA;
    void* args[] = {&l, &a, &ta};
    const bool excl = (q.flags & SPHIDX_EXCLUDE_SELF) != 0;
    return hipLaunchKernel(
        q.stash ? (excl ? (const void*)tile_count_kernel<true, true> : (const void*)tile_count_kernel<true, false>)
                : (excl ? (const void*)tile_count_kernel<false, true> : (const void*)tile_count_kernel<false, false>),
        dim3(tile_blocks()), dim3(64), args, kTileLds, st);
}

hipError_t launch_copy(const QArgs& q, const LatArgs& L, hipStream_t st) {
    const CopyShape c = copy_shape(q.Q);
    const uint64_t waves = (((uint64_t)q.Q + c.rows - 1) / c.rows) * c.splits;
    gather_kernel<<<(uint32_t)((waves + 3) / 4), 256, 0, st>>>(q, L.pts, L.status, c.rows, c.splits);
    return hipGetLastError();
}

// Kernel choice by variant: cube, sphere, sphere with the row table in LDS;
// SPHIDX_PICKP adds variant 3, the paper's cell tables, SPHIDX_PICKS is for the
// sphere's two variants alone.
#define SPHIDX_PICK(KERNEL, variant, SPH, ...)                                     \
    ((variant) == 0 ? (const void*)KERNEL<kCube, false __VA_ARGS__>                \
     : (variant) == 1 ? (const void*)KERNEL<SPH, false __VA_ARGS__>                \
                      : (const void*)KERNEL<SPH, true __VA_ARGS__>)
#define SPHIDX_PICKS(KERNEL, variant, SPH, ...) \
    ((variant) == 1 ? (const void*)KERNEL<SPH, false __VA_ARGS__> : (const void*)KERNEL<SPH, true __VA_ARGS__>)
#define SPHIDX_PICKP(KERNEL, variant, SPH, ...) \
    ((variant) == 3 ? (const void*)KERNEL<kPaper, false __VA_ARGS__> : SPHIDX_PICK(KERNEL, variant, SPH, __VA_ARGS__))

// The block-per-row kernel by its waves.
#define SPHIDX_LONG(METHOD, COUNT, w)                        \
    ((w) == 2   ? (const void*)long_kernel<METHOD, COUNT, 2> \
     : (w) == 4 ? (const void*)long_kernel<METHOD, COUNT, 4> \
                : (const void*)long_kernel<METHOD, COUNT, 8>)

// Small batches, where launches and not work are what a call costs: up to
// kSmallSetup queries one block clears the counters and sets up every query,
// and up to kMergedQ the main kernels walk the fallback queries too, instead of
// a list and a launch of their own in each pass; no launch has many more
// wavefronts than queries (2,048 empty blocks take 4 us to come and go).
constexpr uint32_t kSmallSetup = 1024, kMergedQ = 8192;

hipError_t launch_ptr(const void* fn, uint32_t nq, const QArgs& q, uint32_t waves, uint32_t bpc, size_t shmem,
                      hipStream_t st, const LatArgs& L, const TabArgs& T) {
    uint32_t blocks;
    if (q.persistent) {
        // a wavefront for each query of each queue, so that none waits behind
        // another (list-driven: at most every query; `nq` is 0 there)
        const uint32_t per = (q.Q + SPHIDX_NQUEUE - 1u) / SPHIDX_NQUEUE;
        blocks = std::min((uint32_t)device_cu_count() * bpc, SPHIDX_NQUEUE * ((per + waves - 1u) / waves));
    } else {
        const uint64_t per = (uint64_t)waves * q.tile;
        blocks = (uint32_t)((nq + per - 1) / per);
        if (blocks == 0) blocks = 1;
    }
    LatArgs l = L;
    TabArgs t = T;
    QArgs a = q;
    void* args[] = {&l, &t, &a};
    return hipLaunchKernel(fn, dim3(blocks), dim3(waves * 64), args, shmem, st);
}

}  // namespace

int device_cu_count() {
    static int cached = 0;
    if (cached) return cached;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    cached = cus;
    return cus;
}

size_t long_lds_bytes(uint32_t waves) {
    return (size_t)(kLongCap + 2 * kNearPad) * 8 + (size_t)kLongCap * 4 + 64 + (size_t)waves * 256;
}

// LDS bytes per block: pass 0 count (3 with the stash), 1 write, 2 top-M,
// 4 grouped count (5 with the stash).
size_t query_lds_bytes(int pass, uint32_t cap, uint32_t waves, size_t table_bytes) {
    size_t per = 256;
    if (pass == 1 || pass == 3) per = (size_t)cap * 28 + 256;
    if (pass == 2) per = (size_t)cap * 24 + 64 * 12 + 256;
    if (pass == 4 || pass == 5) per = group_lds_per_wave(pass == 5, cap);
    return table_bytes + per * waves;
}

const char* count_kernel_name(const LatArgs& L, const TabArgs& T, const QArgs& q) {
    TileArgs TA;
    if (tile_plan(L, T, q, TA)) return "tile_count_kernel";
    return q.group == kGroupAll       ? "group_count_kernel"
           : q.group == kGroupSampled ? "group_count_kernel or count_kernel"
                                      : "count_kernel";
}

hipError_t launch_query_pass(int pass, const LatArgs& L, const TabArgs& T, const QArgs& q_in,
                             uint32_t waves_per_block, uint32_t blocks_per_cu, hipStream_t st,
                             hipEvent_t ev_begin, hipEvent_t ev_end) {
    QArgs q = q_in;
    TileArgs TA;
    const bool tiles = pass == 0 && tile_plan(L, T, q, TA);
    // rows kept by the tile kernel need no descriptor (without the stash the
    // write pass walks every row)
    q.tiles = tiles && q.stash ? 1u : 0u;
    if (q.tiles) q.stash_chunk = stash_chunk(q.stash_region, tile_blocks(), q.sort_cap);
    q.merged = !tiles && T.has && !T.paper && q.select == 0u && q.Q <= kMergedQ ? 1u : 0u;
    // optional timing events around the pass's main kernel(s)
    auto mark = [st](hipEvent_t ev) { return ev ? hipEventRecord(ev, st) : hipSuccess; };
    const size_t tb = tab_lds_bytes(T);
    const int variant = !T.has ? 0 : T.paper ? 3 : (T.lds ? 2 : 1);
    hipError_t e;
    // one block per long radius row (count pass: the rows the setup listed;
    // write pass: rows longer than a wavefront's buffer)
    auto launch_long = [&](bool count, const QArgs& qa) -> hipError_t {
        const uint32_t lw = qa.long_waves;
        const void* lf = count ? (variant == 0   ? SPHIDX_LONG(kCube, true, lw)
                                  : variant == 3 ? SPHIDX_LONG(kPaper, true, lw)
                                                 : SPHIDX_LONG(kEither, true, lw))
                               : (variant == 0   ? SPHIDX_LONG(kCube, false, lw)
                                  : variant == 3 ? SPHIDX_LONG(kPaper, false, lw)
                                                 : SPHIDX_LONG(kEither, false, lw));
        const size_t lds = long_lds_bytes(qa.long_waves);
        const uint32_t per_cu = (uint32_t)std::max<size_t>(1, (160u * 1024u) / lds);
        LatArgs l = L;
        TabArgs t = T;
        QArgs a = qa;
        void* args[] = {&l, &t, &a};
        return hipLaunchKernel(lf, dim3(std::min((uint32_t)device_cu_count() * per_cu, qa.Q)), dim3(64u * qa.long_waves),
                               args, lds, st);
    };
    // whether the setup can have listed rows for it: a radius at the tables'
    // cap (per-query radii) or the batch's radius, at the lattice's mean
    // density, expected above 5/4 of the row buffer (the setup's test, with a
    // margin for its single precision)
    auto long_rows_possible = [&]() -> bool {
        if (!q.stash || q.long_waves <= 1 || q.mode == SPHIDX_MODE_KNN || q.stats || L.ncells == 0) return false;
        if (q.rad && (!T.has || q.select == 1u)) return true;
        const double rc = (double)(q.rad ? T.rmax : q.rad_u) / (double)(1u << L.F);
        return 4.18879 * rc * rc * rc * ((double)L.n / (double)L.ncells) > 0.98 * 1.25 * (double)q.sort_cap;
    };
    if (pass == 0) {
        // every counter cleared, the stash header for the write pass, and the
        // per-query descriptors (for the sphere method, the fallback list too);
        // with the tile kernel, of the objects outside the region only (none on
        // cyclic axes)
        const uint4 hv = make_uint4(q.stash, q.stash ? q.stash_region * SPHIDX_NREGION : 0u, q.stash_d2 ? 1u : 0u,
                                    q.stash_d2 ? (uint32_t)(((char*)q.stash_d2 - q.stash_base) / 256) : 0u);
        const bool setup = q.Q > 0 && !(q.tiles && L.cyc == 7u), one = setup && q.Q <= kSmallSetup;
        if (!one)
            clear_counters_kernel<<<1, 256, 0, st>>>(q.queues, 0u, SPHIDX_COUNTER_WORDS, q.stash_hdr, hv, q.tiles, L,
                                                     q.group == kGroupSampled ? q.group_dense : 0.0f);
        if (setup) {
            const uint32_t threads = one ? std::max(256u, (q.Q + 63u) & ~63u) : 256u;
            const uint32_t blocks = one ? 1u : q.tiles ? std::min((q.Q + 255u) / 256u, 512u) : (q.Q + 255u) / 256u;
            uint32_t* counters = one ? q.queues : nullptr;
            if (variant == 0)
                setup_kernel<kCube><<<blocks, threads, 0, st>>>(L, T, q, counters, hv);
            else if (variant == 3)
                setup_kernel<kPaper><<<blocks, threads, 0, st>>>(L, T, q, counters, hv);
            else
                setup_kernel<kSphere><<<blocks, threads, 0, st>>>(L, T, q, counters, hv);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (q.Q == 0) return hipSuccess;
    const uint32_t w = waves_per_block, b = blocks_per_cu;
    // per-query choice: the main kernels walk the sphere, the cube or the
    // cell list per query (grouping them apart would split the groups); small
    // batches take their fallback queries in the same way
    const bool either = q.merged || (variant != 0 && q.select == 1u);
    QArgs ql = q;  // list-driven launches: persistent, grabs sized from the list
    ql.persistent = 1;
    // the count pass's long rows: the setup's list, with the walk-list queue
    // set (the write pass's, cleared when it starts)
    auto long_list = [&]() {
        QArgs a = ql;
        a.list = q.lq;
        a.list_count = q.lq_count;
        a.list_set = kQWalk;
        return a;
    };
    if (pass == 0) {
        const int lp = q.stash ? 3 : 0;
        // K-NN rows searched and kept by the count pass
        const bool ks = q.stash && q.mode != SPHIDX_MODE_RADIUS;
        if ((e = mark(ev_begin)) != hipSuccess) return e;
        if (q.group) {
            // radius queries in groups: all queries (those of the tables),
            // then the fallback list's (bounding cube); the rest through the
            // extra list, one query per wavefront
            const size_t gl = query_lds_bytes(q.stash ? 5 : 4, q.sort_cap, w, tb);
            const bool gk = q.mode != SPHIDX_MODE_RADIUS;  // K-NN queries in the batch
            if (tiles)
                e = launch_tiles(L, q, TA, st);
            else if (q.stash)
                e = launch_ptr(gk ? (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , true, false, true)
                                            : SPHIDX_PICK(group_count_kernel, variant, kSphere, , true, false, true))
                                  : (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , true, false, false)
                                            : SPHIDX_PICK(group_count_kernel, variant, kSphere, , true, false, false)),
                               q.Q, q, w, b, gl, st, L, T);
            else
                e = launch_ptr(gk ? (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , false, false, true)
                                            : SPHIDX_PICK(group_count_kernel, variant, kSphere, , false, false, true))
                                  : (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , false, false, false)
                                            : SPHIDX_PICK(group_count_kernel, variant, kSphere, , false, false, false)),
                               q.Q, q, w, b, gl, st, L, T);
            // (one of the two finds nothing to do)
            if (e == hipSuccess && q.group == kGroupSampled)
                e = launch_ptr(SPHIDX_PICKS(count_kernel, variant, kSphere, , false, true, true), q.Q, q, w, b,
                               query_lds_bytes(lp, q.sort_cap, w, tb), st, L, T);
            if (e == hipSuccess) e = mark(ev_end);
            if (e != hipSuccess) return e;
            if (long_rows_possible() && (e = launch_long(true, long_list())) != hipSuccess) return e;
            if (variant != 0 && !either && !(q.tiles && L.cyc == 7u)) {
                QArgs qg = ql;
                qg.list = q.fbq;
                qg.list_count = q.fb_count;
                qg.list_set = kQFbCount;
                const size_t gl0 = query_lds_bytes(q.stash ? 5 : 4, q.sort_cap, w, 0);
                e = launch_ptr(q.stash ? (const void*)group_count_kernel<kCube, false, true, true, false>
                                       : (const void*)group_count_kernel<kCube, false, false, true, false>,
                               0, qg, w, b, gl0, st, L, T);
                if (e != hipSuccess) return e;
            }
            // (the tile kernel leaves no radius query to the extra list)
            if (tiles && !gk) return hipSuccess;
            ql.list = q.xq;
            ql.list_count = q.xq_count;
            ql.list_set = kQExtra;
            if (gk && variant != 0) {
                // K-NN rows short of K inside their first radius: a second
                // grouped round at a larger radius; what it leaves goes on
                // the long-row list (free until the write pass) to the
                // one-query-per-wave kernel
                QArgs qr = ql;
                qr.xq = q.longq;
                qr.xq_count = q.long_count;
                e = launch_ptr(q.stash ? (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , true, true, true)
                                                 : SPHIDX_PICK(group_count_kernel, variant, kSphere, , true, true, true))
                                       : (either ? SPHIDX_PICK(group_count_kernel, variant, kEither, , false, true, true)
                                                 : SPHIDX_PICK(group_count_kernel, variant, kSphere, , false, true, true)),
                               0, qr, w, b, gl, st, L, T);
                if (e != hipSuccess) return e;
                ql.list = q.longq;
                ql.list_count = q.long_count;
                ql.list_set = kQExtra2;
            }
            if (ks)
                return launch_ptr(SPHIDX_PICK(count_kernel, variant, kEither, , true, true, true), 0, ql, w, b,
                                  query_lds_bytes(lp, q.sort_cap, w, tb), st, L, T);
            if (q.stash)
                return launch_ptr(SPHIDX_PICK(count_kernel, variant, kEither, , true, true, false), 0, ql, w, b,
                                  query_lds_bytes(lp, q.sort_cap, w, tb), st, L, T);
            return launch_ptr(SPHIDX_PICK(count_kernel, variant, kEither, , true, false, false), 0, ql, w, b,
                              query_lds_bytes(lp, q.sort_cap, w, tb), st, L, T);
        }
        const void* fn;
        if (ks)
            fn = either ? SPHIDX_PICK(count_kernel, variant, kEither, , false, true, true)
                        : SPHIDX_PICKP(count_kernel, variant, kSphere, , false, true, true);
        else if (q.stash)
            fn = either ? SPHIDX_PICK(count_kernel, variant, kEither, , false, true, false)
                        : SPHIDX_PICKP(count_kernel, variant, kSphere, , false, true, false);
        else
            fn = either ? SPHIDX_PICK(count_kernel, variant, kEither, , false, false, false)
                        : SPHIDX_PICKP(count_kernel, variant, kSphere, , false, false, false);
        e = launch_ptr(fn, q.Q, q, w, b, query_lds_bytes(lp, q.sort_cap, w, tb), st, L, T);
        if (e == hipSuccess) e = mark(ev_end);
        if (e != hipSuccess) return e;
        if (long_rows_possible() && (e = launch_long(true, long_list())) != hipSuccess) return e;
        if (variant == 0 || either) return hipSuccess;
        ql.list = q.fbq;
        ql.list_count = q.fb_count;
        ql.list_set = kQFbCount;
        return launch_ptr(ks        ? (const void*)count_kernel<kCube, false, true, true, true>
                          : q.stash ? (const void*)count_kernel<kCube, false, true, true, false>
                                    : (const void*)count_kernel<kCube, false, true, false, false>,
                          0, ql, w, b, query_lds_bytes(lp, q.sort_cap, w, 0), st, L, T);
    }
    const size_t sh1 = query_lds_bytes(1, q.sort_cap, w, tb);
    const size_t sh2 = query_lds_bytes(2, q.sort_cap, w, tb);
    if (q.mode != SPHIDX_MODE_KNN) {
        if ((e = mark(ev_begin)) != hipSuccess) return e;
        // rows kept by a stashing count pass (does nothing otherwise)
        if ((e = launch_copy(q, L, st)) != hipSuccess) return e;
        // the count pass may have used tiles (by what both passes must share:
        // its launch may have differed from this one)
        QArgs qw = q;
        qw.tiles = T.has && !T.paper && q.select == 0u && !q.qx && !q.rad && q.mode == SPHIDX_MODE_RADIUS &&
                           q.Q >= kTileMinQ
                       ? 1u
                       : 0u;
        auto with_tiles = [&]() {
            return launch_ptr(either ? SPHIDX_PICKS(write_kernel, variant, kEither, , false, true)
                                     : SPHIDX_PICKS(write_kernel, variant, kSphere, , false, true),
                              q.Q, qw, w, b, sh1, st, L, T);
        };
        if (qw.tiles && q.persistent)
            e = with_tiles();
        else
            e = launch_ptr(either ? SPHIDX_PICK(write_kernel, variant, kEither, , false, false)
                                  : SPHIDX_PICKP(write_kernel, variant, kSphere, , false, false),
                           q.Q, qw, w, b, sh1, st, L, T);
        if (e == hipSuccess && qw.tiles && !q.persistent) {
            // (resident waves from the walk list's queues, which the copy has
            // cleared: a grid of a wave per query took 65 us to find nothing)
            qw.persistent = 1u;
            qw.tile = 64u;
            qw.tiles = 2u;
            e = with_tiles();
        }
        if (e == hipSuccess) e = mark(ev_end);
        if (e != hipSuccess) return e;
        if (variant != 0 && !either) {
            ql.list = q.fbq;
            ql.list_count = q.fb_count;
            ql.list_set = kQFbWrite;
            e = launch_ptr((const void*)write_kernel<kCube, false, true, false>, 0, ql, w, b,
                           query_lds_bytes(1, q.sort_cap, w, 0), st, L, T);
            if (e != hipSuccess) return e;
        }
        // K-NN rows of a mixed batch and long radius rows, from the list:
        // radius rows one block per row, the others (and radius rows whose
        // pairs crowd at one distance) one wavefront per row
        ql.list = q.longq;
        ql.list_count = q.long_count;
        if (q.long_waves > 1) {
            ql.list_set = kQExtra;
            if ((e = launch_long(false, ql)) != hipSuccess) return e;
        }
        ql.list_set = kQTopm;
        return launch_ptr(SPHIDX_PICKP(topm_kernel, variant, kEither, , true), 0, ql, w, b, sh2, st, L, T);
    }
    if ((e = mark(ev_begin)) != hipSuccess) return e;
    // rows kept by the count pass (does nothing otherwise), then the rest
    if ((e = launch_copy(q, L, st)) != hipSuccess) return e;
    e = launch_ptr(SPHIDX_PICKP(topm_kernel, variant, kEither, , false), q.Q, q, w, b, sh2, st, L, T);
    return e == hipSuccess ? mark(ev_end) : e;
}
