// Evaluation passes of the lattice FMM on gfx950 (Section 8.2), for a forest of instances.
//
// Expansions are stored box-major: box g owns kRankPad consecutive FP64 coefficients in Q
// (outgoing, q-hat) and U (incoming, u-hat).
//
//   P2M   q^tau   = T_ofs^tau q(J^tau)                 one wave per leaf, lanes = skeleton index
//   M2M   q^tau   = sum_c T_ofo^(c) q^child_c          FP64 MFMA box-matrix kernel
//   M2L   u^tau   = sum_{sigma in L_int} T_ifo^d q^sigma   FP64 MFMA box-matrix kernel
//   L2L   u^child += T_ofo^(c)T u^tau                  FP64 MFMA box-matrix kernel
//   L2P + near field + un-permutation                  one wave per leaf, lanes = targets x slices
#include "kernels.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <stdexcept>

namespace lfmm {

namespace {

constexpr int kBlock = 256;
constexpr int kBf16Block = 512;   // bf16 M2L: eight waves per 128-box tile
constexpr int kWaves = kBlock / 64;
// Levels of at most this many 64-box tiles run M2M and L2L on the fine-grained kernels, which
// spread one tile over twelve blocks (measured: M2M gains up to 64 tiles, L2L up to 256).
constexpr int32_t kFineM2mTiles = 64;
constexpr int32_t kFineL2lTiles = 256;
// M2L by tiles of 128 boxes, weighted by how full their interaction lists are (m2l_weighted): the
// 16-box kernels up to the first three counts, then, in FP64, blocks of 64 boxes while all blocks of all
// (unweighted) tiles run at once (two a tile, three a compute unit), then of 128.  Measured (16-box / 64-box / 128-box
// kernel, us), uniform points: 120 tiles 53 / 58 / 84, 152 tiles 76 / 82 / 85, 222 tiles 97 / 85 / 87, 353 tiles
// 140 / 111 / 134, 418 tiles 165 / 159 / 136, 485 tiles 182 / 156 / 137, 677 tiles 244 / 211 / 193; clusters, 244 tiles
// 99 / 85 / 87; a curve, 303 tiles 66 / 108 / 133; FP32 mixed 353 tiles 300 / - / 336, 418 tiles 369 / - / 345, clusters,
// 661 tiles 551 / - / 482; bf16 120 tiles 61 / - / 76, 152 tiles 78 / - / 77, clusters, 244 tiles 104 / - / 72, a curve,
// 303 tiles 73 / - / 82.
constexpr int32_t kFineM2lTiles = 160, kFineM2lMixedTiles = 384, kFineM2lBf16Tiles = 144, kHalfM2lTiles = 384;
constexpr double kPi = 3.14159265358979323846;
constexpr double kEulerGamma = 0.57721566490153286061;

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef double double2_t __attribute__((ext_vector_type(2)));
typedef int int2_t __attribute__((ext_vector_type(2)));
typedef int int4_t __attribute__((ext_vector_type(4)));

// Interaction-list slot k of a box in child position c lies at offset slot c_dslot[c][k]
// of the 7 x 7 offset grid; the order matches the list builder (dy outer, dx inner).
struct DSlots { int s[4][kNumInteractions]; };
__constant__ DSlots c_dslot;

__device__ inline uint32_t compact_bits(uint64_t x) {
    x &= 0x5555555555555555ull;
    x = (x | (x >> 1)) & 0x3333333333333333ull;
    x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
    x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
    x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
    return uint32_t(x);
}

// Far-field expansion of phi (eq. (3.1) for the 5-point operator, true Euler constant;
// coefficients of the context's operator in *e); (a, b) != 0
__device__ inline double phi_expansion_dev(double a, double b, const PhiFar* e) {
    const double r2 = a * a + b * b;
    const double ir2 = 1.0 / r2;
    const double c2 = (a * a - b * b) * ir2;   // cos 2 theta
    const double c4 = 2.0 * c2 * c2 - 1.0, c8 = 2.0 * c4 * c4 - 1.0, c12 = 2.0 * c4 * c8 - c4;
    const double lead = -(0.5 * log(r2) + e->C) * (1.0 / (2.0 * kPi));
    const double t1 = e->c[0][0] + e->c[0][1] * c4;
    const double t2 = e->c[1][0] + e->c[1][1] * c4 + e->c[1][2] * c8;
    const double t3 = e->c[2][0] + e->c[2][1] * c4 + e->c[2][2] * c8 + e->c[2][3] * c12;
    return lead + ir2 * (t1 + ir2 * (t2 + ir2 * t3));
}

// phi at offset (a, b), a, b >= 0: the device octant table (quadrature values inside radius
// 128, the expansion evaluated once between 128 and kPhiDeviceRadius), the expansion outside
__device__ inline double phi_oct(int a, int b, const double* oct, const PhiFar* far) {
    const int hi = max(a, b), lo = min(a, b);
    if (hi <= kPhiDeviceRadius) return oct[hi * (hi + 1) / 2 + lo];
    return phi_expansion_dev(double(hi), double(lo), far);
}

// Octant entries with r0 < hi <= r1 (index hi (hi + 1) / 2 + lo) set to the expansion, so
// that lookups replace the logarithm and division of the expansion for offsets up to r1.
__global__ void k_phi_extend(double* oct, int r0, int r1, const PhiFar* far) {
    const int64_t i0 = int64_t(r0 + 1) * (r0 + 2) / 2, i1 = int64_t(r1 + 1) * (r1 + 2) / 2;
    const int64_t i = i0 + int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= i1) return;
    int64_t hi = int64_t((sqrt(8.0 * double(i) + 1.0) - 1.0) * 0.5);
    while (hi * (hi + 1) / 2 > i) --hi;
    while ((hi + 1) * (hi + 2) / 2 <= i) ++hi;
    const int64_t lo = i - hi * (hi + 1) / 2;
    oct[i] = phi_expansion_dev(double(hi), double(lo), far);
}

inline unsigned grid_for(int64_t n, int per_block = kBlock) {
    const int64_t g = (n + per_block - 1) / per_block;
    return unsigned(g < 1 ? 1 : g);
}

__device__ inline int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Load of sorted point s of an instance with arrays e: in the caller's order, that of the
// instance-local index perm_local[s] = j; with sorted loads, of index s itself (coalesced); zero for a
// point that is a target only.  Also stored at fs[s] for the near field: P2M visits every point once.
__device__ inline double load_f(const ExecPtrs& e, int32_t j, int32_t s) {
    return j < e.nsrc ? e.f[e.sorted != 0 ? s : j] : 0.0;
}

// P2M with the dense-model operator (Remark 8.2): q-hat[p] = sum_j T[loc(j)][p] f_j; one
// wave per leaf, lane p < P accumulating entry p.  The leaf's points are loaded once, one
// per lane (coalesced), and handed to all lanes by shuffles, so the only memory reads in the
// loop are the operator rows, whose addresses are known in advance and can be in flight
// together.  Each entry is one sum over the leaf's points in order, as in k_p2m_lds: which of
// the two kernels a launch takes depends on the plan (its number of leaves), so a leaf must
// get the same bits from both for an instance alone and in a forest to agree.
template <int P>
__global__ __launch_bounds__(kBlock) void k_p2m(int32_t leaf0, int32_t leaf1, const int32_t* box_pt0,
                                                 const int32_t* box_pt1, const uint64_t* box_key, int64_t side,
                                                 const int2* pts, const ExecPtrs* tab, ExecPtrs single,
                                                 const int32_t* perm_local, const int32_t* box_inst,
                                                 double* fs, const double* leafT, double* Q) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int32_t g = leaf0 + int32_t(blockIdx.x) * kWaves + wave;
    if (g >= leaf1) return;
    const ExecPtrs e = tab ? tab[box_inst[g]] : single;
    const int32_t p0 = box_pt0[g], p1 = box_pt1[g];
    const uint64_t key = box_key[g];
    const int32_t cx = int32_t(compact_bits(key) * side), cy = int32_t(compact_bits(key >> 1) * side);
    const int l = lane < P ? lane : 0;
    double a = 0.0;
    for (int32_t c0 = p0; c0 < p1; c0 += 64) {
        const int32_t j = c0 + lane;
        int32_t loc = 0;   // lanes past the leaf's points carry a zero load at cell 0
        double f = 0.0;
        if (j < p1) {
            const int2 q = pts[j];
            loc = int32_t(int64_t(q.x - cx) + side * int64_t(q.y - cy));
            f = load_f(e, perm_local[j], j);
            fs[j] = f;
        }
        const int cnt = min(64, p1 - c0);
        for (int k = 0; k < cnt; k += 8) {   // k + 7 < 64: the tail reads the zero-load lanes
            // the eight rows are loaded together; the sum takes them in point order
            double t[8], fk[8];
            #pragma unroll
            for (int u = 0; u < 8; ++u) {
                t[u] = leafT[int64_t(__shfl(loc, k + u, 64)) * P + l];
                fk[u] = __shfl(f, k + u, 64);
            }
            #pragma unroll
            for (int u = 0; u < 8; ++u) a += t[u] * fk[u];
        }
    }
    if (lane < P) Q[size_t(g) * P + lane] = a;
}

// P2M with the leaf operator staged in LDS (leaf sides whose T_ofs fits: side^2 P doubles):
// persistent blocks of kP2mThreads copy T_ofs once, then each wave takes 8 leaves at a time,
// one per 8-lane group, eight points of each at a time (a chunk); lane l of a group accumulates entries
// 2 l + 16 r and 2 l + 16 r + 1 of Q-hat over the leaf's points, which the group loads one per lane and
// hands round by shuffles.  A group past the others' point counts adds zero loads at cell 0.
// What bounds it is the chain box -> points and order -> loads -> rows, a few dependent trips to
// memory per chunk: the points and their order are loaded two chunks ahead and the loads one, across
// leaves, and the boxes two steps ahead (16,384 leaves of 15 points, side 16: 20.4 -> 16.9 us; 8.9e6
// points in 512 trees 338 -> 273; 2e6 in 64 clusters, side 128, 183 -> 153).  From 1e6 points on the rows
// bound it: 384 bytes a point, from LDS, or from L2 and beyond (5 TB/s).
constexpr int kP2mThreads = 1024, kP2mFreeThreads = 512;   // with and without the staged operator
constexpr int kP2mGroup = 8;                   // lanes per leaf
constexpr int kP2mLeaves = 64 / kP2mGroup;     // leaves per wave and step
// A wave per leaf (k_p2m) for plans of at most this many leaves, whose waves all run at once: a leaf's
// points, loads and rows then take one trip to memory each, not one a chunk.  Measured (k_p2m / grouped,
// us): side 8, 15 points a leaf, 1,024 leaves 6.6 / 13.2, 4,096 9.6 / 14.7, 16,384 20.0 / 16.1; side 32, 25 points,
// 1,024 leaves 7.2 / 17.5, 4,096 11.4 / 17.5, 16,384 26.3 / 21.9.
constexpr int32_t kP2mWaveLeaves = 8192;
// With more leaves, too, where T_ofs does not fit LDS (the rows then come from L2 either way) and the leaves hold more
// than kP2mSparsePoints on average, up to kP2mWideLeaves leaves, and with any number if they are uneven: the eight
// leaves of a group take as long as its fullest.  The fullest leaf of a plan holds up to N_leaf points, so that an
// average below kP2mUneven of it tells clusters (0.03 to 0.10) from uniform points and curves (0.2 to 0.5).  Measured
// (k_p2m / grouped, us), clusters: side 32, 5.7 points a leaf of N_leaf 64, 123,691 leaves 71 / 46; side 64, 16 of 200,
// 42,811 leaves 45 / 71; side 128, 51 of 500, 13,673 leaves 56 / 155, 66,168 leaves 169 / 280; uniform points: side 32, 10
// of 64, 19,598 leaves 19 / 16; side 64, 14 of 64, 44,100 leaves 36 / 27; 102 of 256, 9,801 leaves 49 / 60; 40 of 200,
// 24,649 leaves 48 / 45; side 128, 162 of 500, 24,649 leaves 196 / 167; a curve, side 32, 32 of 64, 14,999 leaves
// 22.6 / 19.3.  (In LDS the grouped kernel is the faster from 15,625 leaves on at any density: 64 points a leaf
// 29 / 45, 256 90 / 145.)
constexpr double kP2mUneven = 0.15;
constexpr int32_t kP2mWideLeaves = 12288;
constexpr double kP2mSparsePoints = 12.0;

// STAGED false: the same for leaves whose T_ofs is too large for LDS: the operator rows come from global
// memory (L2-resident), eight lanes reading one 384-byte row together.
template <int P, bool STAGED>
__global__ __launch_bounds__(STAGED ? kP2mThreads : kP2mFreeThreads) void k_p2m_lds(int32_t leaf0, int32_t leaf1, const int32_t* box_pt0,
                                                        const int32_t* box_pt1, int64_t side,
                                                        const int2* pts, const ExecPtrs* tab, ExecPtrs single,
                                                        const int32_t* perm_local, const int32_t* box_inst,
                                                        double* fs, const double* leafT, double* Q) {
    constexpr int W = (STAGED ? kP2mThreads : kP2mFreeThreads) / 64;
    constexpr int R = P / (2 * kP2mGroup);   // pairs of entries per lane
    static_assert(P % (2 * kP2mGroup) == 0, "entries split evenly over a group");
    extern __shared__ __align__(16) double sT_lds[];
    const int ncell = int(side * side), sd = int(side);
    const int wave = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63, l = lane % kP2mGroup;
    const int grp = lane / kP2mGroup;
    const int32_t nleaf = leaf1 - leaf0;
    const int32_t stride = int32_t(gridDim.x) * W * kP2mLeaves;
    struct Box {
        int32_t p0, npt, inst;
    };
    auto box = [&](int32_t q) {   // of this lane's leaf at step q
        Box b = {0, 0, 0};
        if (q + grp < nleaf) {
            const int32_t g = leaf0 + q + grp;
            b.p0 = box_pt0[g];
            b.npt = box_pt1[g] - b.p0;
            if (tab) b.inst = box_inst[g];
        }
        return b;
    };
    // the chunk whose points are loaded next: chunk c of step q, its boxes, and the next step's
    int32_t q = (int32_t(blockIdx.x) * W + wave) * kP2mLeaves, c = 0, most = 0;
    Box cur = box(q), nxt = box(q + stride);
    ExecPtrs e = single;
    auto open = [&]() {   // step q's leaves
        if (tab) e = tab[cur.inst];
        most = cur.npt;
        #pragma unroll
        for (int o = kP2mGroup; o < 64; o <<= 1) most = max(most, __shfl_xor(most, o, 64));
        most = uniform(most);
    };
    struct Chunk {
        int32_t s, perm, q, pts;   // this lane's point (-1: none) and its place; step; points per leaf; pts < 0: none
        int2 xy;
        bool last;
        const double* f;
        int32_t nsrc, sorted;
    };
    auto fetch = [&]() {
        Chunk k;
        k.pts = -1;
        k.s = -1;
        k.q = q;
        k.perm = 0;
        k.xy = make_int2(0, 0);
        k.last = true;
        k.f = e.f;
        k.nsrc = e.nsrc;
        k.sorted = e.sorted;
        if (q >= nleaf) return k;
        if (c + l < cur.npt) {
            k.s = cur.p0 + c + l;
            k.xy = pts[k.s];
            k.perm = perm_local[k.s];
        }
        k.pts = min(most - c, kP2mGroup);
        c += kP2mGroup;
        if (c >= most) {
            q += stride;
            c = 0;
            cur = nxt;
            nxt = box(q + stride);
            if (q < nleaf) open();
        } else {
            k.last = false;
        }
        return k;
    };
    open();
    Chunk ahead = fetch();
    if (STAGED) {
        const double2* src = reinterpret_cast<const double2*>(leafT);
        double2* dst = reinterpret_cast<double2*>(sT_lds);
        for (int i = int(threadIdx.x); i < ncell * P / 2; i += kP2mThreads) dst[i] = src[i];
    }
    const double2_t* sT = reinterpret_cast<const double2_t*>(STAGED ? sT_lds : leafT);
    // the chunk whose loads are in flight
    int32_t n_s, n_q, n_pts, n_loc;
    bool n_last;
    double n_f;
    auto gather = [&](const Chunk& k) {
        n_s = k.s;
        n_q = k.q;
        n_pts = k.pts;
        n_last = k.last;
        n_loc = 0;
        n_f = 0.0;
        if (k.s >= 0) {
            n_loc = (k.xy.x & (sd - 1)) + sd * (k.xy.y & (sd - 1));   // the cell of its leaf: sides are powers of two
            if (k.perm < k.nsrc) n_f = k.f[k.sorted != 0 ? k.s : k.perm];
        }
    };
    gather(ahead);
    ahead = fetch();
    __syncthreads();
    double2_t a[R];
    #pragma unroll
    for (int r = 0; r < R; ++r) a[r] = double2_t{0.0, 0.0};
    while (n_pts >= 0) {   // uniform
        const int32_t loc = n_loc, npt = n_pts, cq = n_q;
        const double f = n_f;
        const bool last = n_last;
        if (n_s >= 0) fs[n_s] = f;
        gather(ahead);
        ahead = fetch();
        asm volatile("" ::: "memory");   // these loads go out here
        #pragma unroll
        for (int k = 0; k < kP2mGroup; ++k) {
            if (k >= npt) break;         // uniform
            const int src = (lane & ~(kP2mGroup - 1)) | k;
            const double2_t* row = sT + __shfl(loc, src, 64) * (P / 2) + l;
            const double fk = __shfl(f, src, 64);
            #pragma unroll
            for (int r = 0; r < R; ++r) a[r] += row[kP2mGroup * r] * fk;
        }
        if (last) {
            if (cq + grp < nleaf) {
                double2_t* out = reinterpret_cast<double2_t*>(Q + size_t(leaf0 + cq + grp) * P) + l;
                #pragma unroll
                for (int r = 0; r < R; ++r) out[kP2mGroup * r] = a[r];
            }
            #pragma unroll
            for (int r = 0; r < R; ++r) a[r] = double2_t{0.0, 0.0};
        }
    }
}

// XCD-aware tile order: blocks are dispatched round-robin over the 8 XCDs (block b runs on
// XCD b % 8), so block b walks the b % 8-th contiguous eighth of the tile list; spatially
// close tiles, which share source expansions, then meet in the same L2.
__device__ inline int32_t xcd_tile(int32_t b, int32_t G, int32_t step, int32_t ntiles) {
    const int32_t x = b & 7, local = b >> 3, per = (G + 7 - x) >> 3;   // blocks on XCD x
    const int32_t chunk = (ntiles + 7) >> 3;
    const int32_t t = x * chunk + local + step * per;
    return (t < min(ntiles, (x + 1) * chunk)) ? t : -1;
}

// Box-matrix passes on the FP64 matrix cores: for a tile of up to 64 target boxes that share
// their operators, out[box] (+)= sum over slots k of A_k in[src_k(box)] with 48 x 48 A_k:
//   M2M (step 2): 4 children, A_k = T_ofo^(k) at the tile's height, in = out = Q;
//   L2L (step 4): the parent, A = T_ofo^(c)T at the parent's height, in = out = U, added.
// Wave w of the block owns boxes 16 w .. 16 w + 15 (the 16 columns of its products) and runs
// every slot, so no partial sums cross waves.  Operators are stored in fragment order (lane
// l's operands of one instruction next to lane l+1's), staged once per block in LDS with
// coalesced loads, double-buffered, and read by all four waves; the next slot's operator and
// source expansion are loaded into registers while the current slot's instructions run, and
// the list entry behind the expansion read one slot before that.  One barrier per slot: the
// buffer a slot writes was last read two slots earlier, before the previous slot's barrier.
// Absent sources (empty list slots, lanes past the tile) read the all-zero row `zrow`.
//
// FP64: 16x16x4 instruction, step kk of row block m takes column g * 12 + kk in lane group
// g = lane / 16; element i of lane (g, n) is row 16 m + g + 4 i, column n.

// Pointers into global memory by address space, so that loads through them are global (not
// flat) loads: flat loads also count as LDS operations, and waiting for the LDS reads of a
// slot would then wait for the next slot's prefetch too.
template <class T>
using gptr = const __attribute__((address_space(1))) T*;
template <class T>
__device__ inline gptr<T> global(const T* p) {
    return (gptr<T>)(p);   // generic to global address space
}

// read-only data that every lane of a wave reads at the same address: constant address
// space, so that uniform reads become scalar loads
template <class T>
using cptr = const __attribute__((address_space(4))) T*;
template <class T>
__device__ inline cptr<T> as_const(const T* p) {
    return (cptr<T>)(p);   // generic to constant address space
}

template <int MODE>
__device__ inline void boxmat_tiles(const BoxTile* tiles, int32_t ntiles, const int32_t* box_list,
                                    const int32_t* src_tab, const OpsPtrs* ops, const double* in, int32_t zrow,
                                    double* out, const int8_t* role = nullptr) {
    constexpr int P = kRankPad, MT = P / 16, KQ = P / 4, NJ = KQ / 2;
    static_assert(MODE == kModeM2M || MODE == kModeL2L, "M2L has a kernel of its own");
    constexpr int NS = (MODE == kModeM2M) ? 4 : 1;
    constexpr int SW = NS;   // source table width
    constexpr int A2 = P * P / 2;                      // double2_t per operator: 4.5 per thread
    static_assert(A2 == 4 * kBlock + kBlock / 2, "staging below assumes P = 48");
    static_assert(MT == 3, "three row blocks");
    __shared__ double2_t sA[2][A2];
    __shared__ int s_dsl[4];   // operator of each slot of the tile
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int32_t G = int32_t(gridDim.x);
    const double2_t z2 = {0.0, 0.0};
    for (int32_t step = 0;; ++step) {
        const int32_t t = uniform(xcd_tile(int32_t(blockIdx.x), G, step, ntiles));
        if (t < 0) break;                                  // uniform over the block
        const int32_t count = uniform(tiles[t].count);
        if (count == 0) continue;
        const int32_t start = uniform(tiles[t].start), height = uniform(tiles[t].height);
        const int32_t cls = uniform(tiles[t].cls), opi = uniform(tiles[t].ops);
        const int col = 16 * wave + n;
        const int32_t box = (col < count) ? (box_list ? box_list[start + col] : start + col) : -1;
        const gptr<int32_t> srcs = global(src_tab + size_t(box >= 0 ? box : 0) * SW);
        const double* base = (MODE == kModeM2M) ? ops[opi].ofo_rm : ops[opi].ofo_cm;
        const gptr<double2_t> Ah = global(reinterpret_cast<const double2_t*>(base));
        const gptr<double> Xg = global(in) + g * KQ;
        if (tid < NS) s_dsl[tid] = (MODE == kModeM2M) ? height * 4 + tid : (height + 1) * 4 + cls;
        __syncthreads();
        const int* dsl = s_dsl;
        // slot 0 operands
        int32_t src = (box >= 0) ? srcs[0] : -1;
        src = src < 0 ? zrow : src;
        const gptr<double2_t> qs = reinterpret_cast<gptr<double2_t>>(Xg + size_t(src) * P);
        double2_t rb0 = qs[0], rb1 = qs[1], rb2 = qs[2], rb3 = qs[3], rb4 = qs[4], rb5 = qs[5];
        int32_t src_next = (box >= 0 && NS > 1) ? srcs[1] : -1;
        const gptr<double2_t> Ak = Ah + size_t(dsl[0]) * A2;
        int32_t dsl_next = NS > 1 ? dsl[1] : 0;   // operator of the next slot, read a slot ahead
        double2_t ra0 = Ak[tid], ra1 = Ak[tid + kBlock], ra2 = Ak[tid + 2 * kBlock], ra3 = Ak[tid + 3 * kBlock];
        double2_t ra4 = (tid < kBlock / 2) ? Ak[tid + 4 * kBlock] : z2;
        double4_t acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = acc0, acc2 = acc0;
        // M2M and L2L sum their contraction as four partial products added in order, the same
        // arithmetic as the fine-grained kernels below, so that a box's result does not depend
        // on which kernel its level runs on.
        double4_t run0 = acc0, run1 = acc0, run2 = acc0;
        auto fold = [&](bool first) {
            const double4_t z4 = {0.0, 0.0, 0.0, 0.0};
            if (first) {
                run0 = acc0;
                run1 = acc1;
                run2 = acc2;
            } else {
                run0 += acc0;
                run1 += acc1;
                run2 += acc2;
            }
            acc0 = z4;
            acc1 = z4;
            acc2 = z4;
        };
        for (int k = 0; k < NS; ++k) {
            double2_t* buf = sA[k & 1];
            buf[tid] = ra0;
            buf[tid + kBlock] = ra1;
            buf[tid + 2 * kBlock] = ra2;
            buf[tid + 3 * kBlock] = ra3;
            if (tid < kBlock / 2) buf[tid + 4 * kBlock] = ra4;
            const double2_t b[NJ] = {rb0, rb1, rb2, rb3, rb4, rb5};
            __syncthreads();
            if (k + 1 < NS) {
                // expansions first: their address waits only for the list entry read a slot ago
                const int32_t sn = src_next < 0 ? zrow : src_next;
                const gptr<double2_t> qn = reinterpret_cast<gptr<double2_t>>(Xg + size_t(sn) * P);
                rb0 = qn[0];
                rb1 = qn[1];
                rb2 = qn[2];
                rb3 = qn[3];
                rb4 = qn[4];
                rb5 = qn[5];
                src_next = (box >= 0 && k + 2 < NS) ? srcs[k + 2] : -1;
                const gptr<double2_t> An = Ah + size_t(uniform(dsl_next)) * A2;
                ra0 = An[tid];
                ra1 = An[tid + kBlock];
                ra2 = An[tid + 2 * kBlock];
                ra3 = An[tid + 3 * kBlock];
                if (tid < kBlock / 2) ra4 = An[tid + 4 * kBlock];
                dsl_next = (k + 2 < NS) ? dsl[k + 2] : 0;
            }
            // every wave runs the products (a wave past the tile's boxes multiplies the zero
            // row): no branch around them, so the accumulators stay in place between slots
            {
                #pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const double2_t a0 = buf[(0 * NJ + j) * 64 + lane];
                    const double2_t a1 = buf[(1 * NJ + j) * 64 + lane];
                    const double2_t a2 = buf[(2 * NJ + j) * 64 + lane];
                    #pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        if (MODE == kModeL2L && (2 * j + e) % 3 == 0 && j + e > 0) {
                            fold(2 * j + e == 3);   // step 3 c starts the c-th partial sum
                        }
                        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(e ? a0.y : a0.x, e ? b[j].y : b[j].x, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(e ? a1.y : a1.x, e ? b[j].y : b[j].x, acc1, 0, 0, 0);
                        acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(e ? a2.y : a2.x, e ? b[j].y : b[j].x, acc2, 0, 0, 0);
                    }
                }
            }
            if (MODE == kModeM2M) fold(k == 0);   // one partial sum per child slot
        }
        if (MODE == kModeL2L) fold(false);
        acc0 = run0;
        acc1 = run1;
        acc2 = run2;
        if (box >= 0) {
            double* ob = out + size_t(box) * P;
            // a pruned box of the adaptive tree has no M2L result: it takes its parent's alone
            const bool add = MODE == kModeL2L && !(role != nullptr && role[box] == kRolePruned);
            #pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (add) {
                    ob[g + 4 * i] += acc0[i];
                    ob[16 + g + 4 * i] += acc1[i];
                    ob[32 + g + 4 * i] += acc2[i];
                } else {
                    ob[g + 4 * i] = acc0[i];
                    ob[16 + g + 4 * i] = acc1[i];
                    ob[32 + g + 4 * i] = acc2[i];
                }
            }
        }
        __syncthreads();   // the next tile's first slot rewrites a buffer read above
    }
}

// M2L (Section 8.2 step 3) on the FP64 matrix cores for tiles of up to 128 target boxes that
// share their 27 operators (same operator set, height and child position).  Wave w owns the two
// 16-box column blocks of boxes 32 w .. 32 w + 31, so each operator staged in LDS (once per slot
// and block, double-buffered, one barrier per slot) feeds 72 matrix instructions per wave: the
// staging and the barrier cost half as much per product as with one column block, and a launch
// of the 1e6-point plan fits the device in one round of blocks.  The tile's interaction lists
// are copied into LDS when the tile starts, so the slot loop issues no dependent global loads:
// within a slot the wave runs its two column blocks one after the other, and the source
// expansion of the next (slot, column block) pair is loaded from global memory while the
// current pair's products run (its list entry read from LDS one pair earlier).  Absent sources
// (empty list slots, boxes past the tile) read the zero row.
// 16x16x4 FP64 instruction: step kk of row block m takes column g * 12 + kk in lane group
// g = lane / 16; element i of lane (g, n) is row 16 m + g + 4 i, column n.
// NC = 1: a block takes half a tile, one column block per wave, for plans of fewer tiles than the
// device has room for (a block then lasts half as long: 128,000 uniform points 81 -> 53 us).
template <int NC>
__global__ __launch_bounds__(kBlock, 3) void k_m2l(const BoxTile* tiles, const int32_t* ntiles_dev,
                                                    const int32_t* box_list, const int32_t* il27, const OpsPtrs* ops,
                                                    const double* Q, int32_t zrow, double* U) {
    constexpr int NB = 64 * NC, NH = kM2LTile / NB;   // boxes a block takes of a tile, and such parts
    const int32_t ntiles = uniform(*ntiles_dev) * NH;
    constexpr int P = kRankPad, KQ = P / 4, NJ = KQ / 2, NS = kNumInteractions;
    constexpr int A2 = P * P / 2;                      // double2_t per operator: 4.5 per thread
    static_assert(A2 == 4 * kBlock + kBlock / 2, "staging below assumes P = 48");
    __shared__ double2_t sA[2][A2];
    __shared__ int32_t s_src[NB * NS];     // source box of (tile column, slot), zrow if none
    __shared__ int32_t s_box[NB];
    __shared__ int s_dsl[NS];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int32_t G = int32_t(gridDim.x);
    const double2_t z2 = {0.0, 0.0};
    for (int32_t step = 0;; ++step) {
        const int32_t part = uniform(xcd_tile(int32_t(blockIdx.x), G, step, ntiles));
        if (part < 0) break;                               // uniform over the block
        const int32_t t = part / NH, first = (part % NH) * NB;
        const int32_t count = uniform(tiles[t].count) - first;
        if (count <= 0) continue;
        const int32_t start = uniform(tiles[t].start) + first, height = uniform(tiles[t].height);
        const int32_t cls = uniform(tiles[t].cls), opi = uniform(tiles[t].ops);
        if (tid < NS) s_dsl[tid] = height * kNumIfoSlots + c_dslot.s[cls][tid];
        if (tid < NB) s_box[tid] = (tid < count) ? box_list[start + tid] : -1;
        __syncthreads();
        for (int i = tid; i < NB * NS; i += kBlock) {
            const int b = i / NS;
            const int32_t box = s_box[b];
            const int32_t src = box >= 0 ? il27[size_t(box) * NS + (i - b * NS)] : -1;
            s_src[i] = src < 0 ? zrow : src;
        }
        const gptr<double2_t> Ah = global(reinterpret_cast<const double2_t*>(ops[opi].ifo));
        const gptr<double> Xg = global(Q) + g * KQ;
        const int col0 = 16 * NC * wave + n;
        const int32_t box0 = s_box[col0], box1 = NC == 2 ? s_box[col0 + 16] : -1;
        __syncthreads();
        const int* dsl = s_dsl;
        const int32_t* src0 = s_src + col0 * NS;          // this lane's two columns' lists
        const int32_t* src1 = NC == 2 ? src0 + 16 * NS : src0 + 1;
        auto load_q = [&](int32_t src, double2_t (&r)[NJ]) {
            const gptr<double2_t> q = reinterpret_cast<gptr<double2_t>>(Xg + size_t(src) * P);
            #pragma unroll
            for (int j = 0; j < NJ; ++j) r[j] = q[j];
        };
        double2_t bq[NJ], nq[NJ];
        load_q(src0[0], nq);                               // pair (slot 0, block 0)
        int32_t idx_next = src1[0];                        // pair (slot 0, block 1)
        const gptr<double2_t> A0 = Ah + size_t(dsl[0]) * A2;
        int32_t dsl_next = dsl[1];
        double2_t ra0 = A0[tid], ra1 = A0[tid + kBlock], ra2 = A0[tid + 2 * kBlock], ra3 = A0[tid + 3 * kBlock];
        double2_t ra4 = (tid < kBlock / 2) ? A0[tid + 4 * kBlock] : z2;
        double4_t acc[NC][3];
        #pragma unroll
        for (int c = 0; c < NC; ++c)
            #pragma unroll
            for (int m = 0; m < 3; ++m) acc[c][m] = double4_t{0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < NS; ++k) {
            double2_t* buf = sA[k & 1];
            buf[tid] = ra0;
            buf[tid + kBlock] = ra1;
            buf[tid + 2 * kBlock] = ra2;
            buf[tid + 3 * kBlock] = ra3;
            if (tid < kBlock / 2) buf[tid + 4 * kBlock] = ra4;
            __syncthreads();
            if (k + 1 < NS) {   // the next slot's operator, into registers
                const gptr<double2_t> An = Ah + size_t(uniform(dsl_next)) * A2;
                ra0 = An[tid];
                ra1 = An[tid + kBlock];
                ra2 = An[tid + 2 * kBlock];
                ra3 = An[tid + 3 * kBlock];
                if (tid < kBlock / 2) ra4 = An[tid + 4 * kBlock];
                dsl_next = (k + 2 < NS) ? dsl[k + 2] : 0;
            }
            // the slot's products at raised issue priority, the staging and barrier at the normal
            // one, so that a wave keeps the matrix pipe through its run of products (measured 1-3 %
            // faster here; the same in the bf16 kernel measured 19 % slower)
            __builtin_amdgcn_s_setprio(1);
            #pragma unroll
            for (int c = 0; c < NC; ++c) {
                // each pass reads its operator fragments from LDS anew: holding the first pass's
                // fragments in registers for the second would cost 72 VGPRs (a third of them)
                asm volatile("" ::: "memory");
                #pragma unroll
                for (int j = 0; j < NJ; ++j) bq[j] = nq[j];
                // the next pair: (k, block 1) after block 0, (k + 1, block 0) after block 1
                if (NC == 1) {
                    if (k + 1 < NS) load_q(idx_next, nq);
                    idx_next = k + 2 < NS ? src0[k + 2] : zrow;
                } else if (c == 0 || k + 1 < NS) {
                    load_q(idx_next, nq);
                    idx_next = (c == 0) ? (k + 1 < NS ? src0[k + 1] : zrow) : src1[k + 1];
                }
                #pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const double2_t a0 = buf[(0 * NJ + j) * 64 + lane];
                    const double2_t a1 = buf[(1 * NJ + j) * 64 + lane];
                    const double2_t a2 = buf[(2 * NJ + j) * 64 + lane];
                    acc[c][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.x, bq[j].x, acc[c][0], 0, 0, 0);
                    acc[c][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.x, bq[j].x, acc[c][1], 0, 0, 0);
                    acc[c][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2.x, bq[j].x, acc[c][2], 0, 0, 0);
                    acc[c][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.y, bq[j].y, acc[c][0], 0, 0, 0);
                    acc[c][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.y, bq[j].y, acc[c][1], 0, 0, 0);
                    acc[c][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2.y, bq[j].y, acc[c][2], 0, 0, 0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
        }
        #pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int32_t box = c ? box1 : box0;
            if (box >= 0) {
                double* ob = U + size_t(box) * P;
                // plain stores: streaming (non-temporal) ones were measured to leave the time
                // unchanged and to send these 8-byte pieces to memory uncombined (2.4x the
                // written bytes)
                #pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ob[g + 4 * i] = acc[c][0][i];
                    ob[16 + g + 4 * i] = acc[c][1][i];
                    ob[32 + g + 4 * i] = acc[c][2][i];
                }
            }
        }
        __syncthreads();   // the next tile rewrites the staging buffers and lists read above
    }
}

__global__ __launch_bounds__(kBlock) void k_m2m(const BoxTile* tiles, int32_t ntiles, const int32_t* box_child,
                                                 const OpsPtrs* ops, double* Q, int32_t zrow) {
    boxmat_tiles<kModeM2M>(tiles, ntiles, nullptr, box_child, ops, Q, zrow, Q);
}

__global__ __launch_bounds__(kBlock) void k_l2l(const BoxTile* tiles, int32_t ntiles, const int32_t* box_list,
                                                 const int32_t* box_parent, const OpsPtrs* ops, double* U,
                                                 int32_t zrow, const int8_t* role) {
    boxmat_tiles<kModeL2L>(tiles, ntiles, box_list, box_parent, ops, U, zrow, U, role);
}

// Box-matrix passes for levels with few boxes (M2M and L2L).  The kernels above run a 64-box
// tile on one block whose waves each run every slot, so a level of a handful of tiles lasts a
// whole sequence of dependent products on one SIMD.  Here block (t, q, m) computes rows
// 16 m .. 16 m + 15 of boxes 16 q .. 16 q + 15 of tile t, and its four waves split the
// contraction: in M2M wave w applies the operator of child slot w; in L2L wave w takes steps
// 3 w .. 3 w + 2 of the twelve 16x16x4 steps of the parent's operator.  The four partial
// products meet in LDS in a fixed order, and wave w writes element w of every lane's four.
// Operator fragments are read straight from the fragment-ordered table (the rows of one row
// block are contiguous there), without LDS staging.
template <int MODE>
__device__ inline void boxmat_fine(const BoxTile* tiles, const int32_t* box_list, const int32_t* src_tab,
                                   const OpsPtrs* ops, const double* in, int32_t zrow, double* out,
                                   const int8_t* role = nullptr) {
    constexpr int P = kRankPad, KQ = P / 4, NJ = KQ / 2, A2 = P * P / 2;
    static_assert(MODE == kModeM2M || MODE == kModeL2L, "fine mode serves M2M and L2L");
    __shared__ double red[4][4][64];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int32_t b = int32_t(blockIdx.x);
    const int m = b % 3, q = (b / 3) & 3;
    const int32_t t = b / 12;
    const int32_t count = uniform(tiles[t].count);
    if (16 * q >= count) return;                       // uniform over the block, before any barrier
    const int32_t start = uniform(tiles[t].start), height = uniform(tiles[t].height);
    const int32_t cls = uniform(tiles[t].cls), opi = uniform(tiles[t].ops);
    const int col = 16 * q + n;
    const int32_t box = (col < count) ? (MODE == kModeL2L ? box_list[start + col] : start + col) : -1;
    int32_t src = -1;
    if (box >= 0) src = (MODE == kModeM2M) ? src_tab[size_t(box) * 4 + wave] : src_tab[box];
    src = src < 0 ? zrow : src;
    const gptr<double> xs = global(in) + size_t(src) * P + g * KQ;
    const bool add = MODE == kModeL2L && box >= 0 && !(role != nullptr && role[box] == kRolePruned);
    const double old = add ? out[size_t(box) * P + 16 * m + g + 4 * wave] : 0.0;
    const double4_t zero4 = {0.0, 0.0, 0.0, 0.0};
    double4_t acc = zero4;
    if (MODE == kModeM2M) {
        const gptr<double2_t> A = global(reinterpret_cast<const double2_t*>(ops[opi].ofo_rm)) +
                                  size_t(height * 4 + wave) * A2 + size_t(m * NJ) * 64 + lane;
        const gptr<double2_t> xb = reinterpret_cast<gptr<double2_t>>(xs);
        double2_t a[NJ], x[NJ];
        #pragma unroll
        for (int j = 0; j < NJ; ++j) {
            x[j] = xb[j];
            a[j] = A[j * 64];
        }
        #pragma unroll
        for (int j = 0; j < NJ; ++j) {
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].x, x[j].x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].y, x[j].y, acc, 0, 0, 0);
        }
    } else {
        const gptr<double> A = global(ops[opi].ofo_cm) + size_t((height + 1) * 4 + cls) * (2 * A2) +
                               size_t(m * NJ) * 128 + 2 * lane;
        double a[3], x[3];
        #pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int s = 3 * wave + r, j = s >> 1, e = s & 1;   // step s = 2 j + e
            x[r] = xs[s];
            a[r] = A[j * 128 + e];
        }
        #pragma unroll
        for (int r = 0; r < 3; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], x[r], acc, 0, 0, 0);
    }
    #pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc[i];
    __syncthreads();
    const double v = ((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane];
    if (box >= 0) {
        out[size_t(box) * P + 16 * m + g + 4 * wave] = (MODE == kModeL2L) ? old + v : v;
    }
}

__global__ __launch_bounds__(kBlock) void k_m2m_fine(const BoxTile* tiles, const int32_t* box_child,
                                                      const OpsPtrs* ops, double* Q, int32_t zrow) {
    boxmat_fine<kModeM2M>(tiles, nullptr, box_child, ops, Q, zrow, Q);
}

__global__ __launch_bounds__(kBlock) void k_l2l_fine(const BoxTile* tiles, const int32_t* box_list,
                                                      const int32_t* box_parent, const OpsPtrs* ops, double* U,
                                                      int32_t zrow, const int8_t* role) {
    boxmat_fine<kModeL2L>(tiles, box_list, box_parent, ops, U, zrow, U, role);
}

// M2M and L2L over several levels in one launch, for the top of a tree, whose levels of few boxes each
// lasted a launch's 4.4 us with the kernels above: 2.4 us of it for the launch itself, then a chain of
// dependent loads, with the device nearly idle.  A block takes one box and all its descendants down to
// `depth` levels of boxes with children (depth <= kSubLevels; SubTree): level k of them is kept in LDS
// for the next, at most 4^k rows, so that a level costs its products and one or two barriers.  Twelve
// waves: wave w takes child position w % 4 and row block w / 4, as in the kernels above and with the same
// sums.  The children's indices and (L2L) their M2L results are loaded before the first product, a
// level's operators while the one before runs.  A level is bound by its matrix instructions, 1 us for
// up to 16 boxes: four levels of a curve's tree take 10.4 us (M2M) and 12.7 us (L2L), before 15 and 17.
constexpr int kSubThreads = 768, kSubRow = kRankPad + 2;
__device__ inline constexpr int sub_base(int k) { return k == 3 ? 0 : k == 2 ? 64 : k == 1 ? 80 : 84; }
constexpr int kSubRows = 85;
static_assert(kSubLevels == 4, "sub_base");

struct SubChildren {   // this lane's children, by level and unit of 16 boxes
    int32_t ch[3], ch3[4];
};
__device__ inline SubChildren sub_children(const SubTree& s, int depth, const int32_t* box_child, int c, int n) {
    SubChildren r;
    #pragma unroll
    for (int k = 0; k < 3; ++k)
        r.ch[k] = k < depth && n < s.count[k] ? box_child[size_t(s.first[k] + n) * 4 + c] : -1;
    #pragma unroll
    for (int q = 0; q < 4; ++q)
        r.ch3[q] = depth == 4 && 16 * q + n < s.count[3] ? box_child[size_t(s.first[3] + 16 * q + n) * 4 + c] : -1;
    return r;
}
__device__ inline SubTree sub_tree(const SubTree* subs) {
    const cptr<int32_t> p = as_const(reinterpret_cast<const int32_t*>(subs + blockIdx.x));
    SubTree s;
    #pragma unroll
    for (int k = 0; k < kSubLevels; ++k) {
        s.first[k] = p[k];
        s.count[k] = p[kSubLevels + k];
    }
    return s;
}

__global__ __launch_bounds__(kSubThreads, 3) void k_m2m_sub(const SubTree* subs, int depth, SubOps A,
                                                            const int32_t* box_child, double* Q, int32_t zrow) {
    constexpr int P = kRankPad, KQ = P / 4, NJ = KQ / 2, A2 = P * P / 2;
    __shared__ __align__(16) double qs[kSubRows][kSubRow];
    __shared__ double red[4][12][64];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4, c = wave & 3, m = wave >> 2;
    const SubTree s = sub_tree(subs);
    const SubChildren ch = sub_children(s, depth, box_child, c, n);
    auto load_a = [&](int k, double2_t (&a)[NJ]) {
        const gptr<double2_t> p = global(reinterpret_cast<const double2_t*>(A.A[k])) + size_t(c) * A2 + size_t(m * NJ) * 64 + lane;
        #pragma unroll
        for (int j = 0; j < NJ; ++j) a[j] = p[j * 64];
    };
    auto load_q = [&](int32_t child, double2_t (&x)[NJ]) {   // an expansion of an earlier kernel
        const gptr<double2_t> p = reinterpret_cast<gptr<double2_t>>(global(Q) + size_t(child < 0 ? zrow : child) * P + g * KQ);
        #pragma unroll
        for (int j = 0; j < NJ; ++j) x[j] = p[j];
    };
    double2_t a[NJ], an[NJ], x[2][NJ];
    load_a(depth - 1, a);
    if (depth == 4) {
        load_q(ch.ch3[0], x[0]);
        if (16 < s.count[3]) load_q(ch.ch3[1], x[1]);
    } else {
        load_q(depth == 3 ? ch.ch[2] : depth == 2 ? ch.ch[1] : ch.ch[0], x[0]);
    }
    #pragma unroll
    for (int k = kSubLevels - 1; k >= 0; --k) {
        if (k >= depth) continue;                          // uniform
        if (k < depth - 1) {
            #pragma unroll
            for (int j = 0; j < NJ; ++j) a[j] = an[j];
        }
        if (k > 0) load_a(k > 0 ? k - 1 : 0, an);          // the next level's
        asm volatile("" ::: "memory");
        #pragma unroll
        for (int q = 0; q < (k == 3 ? 4 : 1); ++q) {
            if (16 * q >= s.count[k]) continue;            // uniform
            if (k < depth - 1) {
                const int32_t child = ch.ch[k < 3 ? k : 0];
                const double2_t* p = reinterpret_cast<const double2_t*>(
                    &qs[sub_base(k + 1) + max(child - s.first[k < 3 ? k + 1 : 3], 0)][g * KQ]);
                #pragma unroll
                for (int j = 0; j < NJ; ++j) x[0][j] = child < 0 ? double2_t{0.0, 0.0} : p[j];
            }
            double4_t acc = {0.0, 0.0, 0.0, 0.0};
            #pragma unroll
            for (int j = 0; j < NJ; ++j) {
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].x, x[q & 1][j].x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j].y, x[q & 1][j].y, acc, 0, 0, 0);
            }
            if (k == 3 && q < 2 && 16 * (q + 2) < s.count[3]) load_q(ch.ch3[q < 2 ? q + 2 : 0], x[q & 1]);
            #pragma unroll
            for (int i = 0; i < 4; ++i) red[c][4 * m + i][lane] = acc[i];
            __syncthreads();
            // wave w writes element w of every lane's twelve
            const double v = ((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane];
            const int row = 16 * (wave >> 2) + g + 4 * (wave & 3), b = 16 * q + n;
            if (b < s.count[k]) {
                qs[sub_base(k) + b][row] = v;
                Q[size_t(s.first[k] + b) * P + row] = v;
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kSubThreads, 3) void k_l2l_sub(const SubTree* subs, int depth, SubOps A,
                                                            const int32_t* box_child, double* U, const int8_t* role) {
    constexpr int P = kRankPad, KQ = P / 4, NJ = KQ / 2, A2 = P * P / 2;
    __shared__ __align__(16) double us[kSubRows][kSubRow];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4, c = wave & 3, m = wave >> 2;
    const SubTree s = sub_tree(subs);
    const SubChildren ch = sub_children(s, depth, box_child, c, n);
    // Row 4 i + g of the row block is given row 12 g + 4 m + i of the operator, so that lane (g, n) ends up
    // with four consecutive elements of its child's expansion
    const int arow = 12 * (n & 3) + 4 * m + (n >> 2);
    auto load_a = [&](int k, double2_t (&a)[NJ]) {
        const gptr<double2_t> p = global(reinterpret_cast<const double2_t*>(A.A[k])) + size_t(c) * A2 +
                                  size_t(arow >> 4) * NJ * 64 + 16 * g + (arow & 15);
        #pragma unroll
        for (int j = 0; j < NJ; ++j) a[j] = p[j * 64];
    };
    // M2L's result; a pruned box of the adaptive tree has none: it takes its parent's alone
    auto load_old = [&](int32_t child, double2_t (&o)[2]) {
        const bool add = child >= 0 && !(role != nullptr && role[child] == kRolePruned);
        const double2_t* p = reinterpret_cast<const double2_t*>(U + size_t(add ? child : s.first[0]) * P + g * KQ + 4 * m);
        #pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double2_t v = p[j];
            o[j] = add ? v : double2_t{0.0, 0.0};
        }
    };
    double2_t a[NJ], an[NJ], x[NJ], old[3][2], old3[4][2];
    load_a(0, a);
    {
        const gptr<double2_t> p = reinterpret_cast<gptr<double2_t>>(global(static_cast<const double*>(U)) + size_t(s.first[0]) * P + g * KQ);
        #pragma unroll
        for (int j = 0; j < NJ; ++j) x[j] = p[j];
    }
    #pragma unroll
    for (int k = 0; k < 3; ++k)
        if (k < depth) load_old(ch.ch[k], old[k]);
    #pragma unroll
    for (int k = 0; k < kSubLevels; ++k) {
        if (k >= depth) continue;                          // uniform
        if (k > 0) {
            #pragma unroll
            for (int j = 0; j < NJ; ++j) a[j] = an[j];
        }
        if (k + 1 < depth) load_a(k < 3 ? k + 1 : 0, an);  // the next level's
        if (k == 2) {
            #pragma unroll
            for (int q = 0; q < 4; ++q)
                if (depth == 4 && 16 * q < s.count[3]) load_old(ch.ch3[q], old3[q]);
        }
        asm volatile("" ::: "memory");
        #pragma unroll
        for (int q = 0; q < (k == 3 ? 4 : 1); ++q) {
            if (16 * q >= s.count[k]) continue;            // uniform
            if (k > 0) {
                const double2_t* p = reinterpret_cast<const double2_t*>(&us[sub_base(k) + min(16 * q + n, s.count[k] - 1)][g * KQ]);
                #pragma unroll
                for (int j = 0; j < NJ; ++j) x[j] = p[j];
            }
            double4_t acc[4];
            #pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = double4_t{0.0, 0.0, 0.0, 0.0};
            #pragma unroll
            for (int t = 0; t < 3; ++t)                    // part r of the sum: steps 3 r .. 3 r + 2
                #pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = 3 * r + t;
                    acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(e & 1 ? a[e >> 1].y : a[e >> 1].x,
                                                                  e & 1 ? x[e >> 1].y : x[e >> 1].x, acc[r], 0, 0, 0);
                }
            const int32_t child = k == 3 ? ch.ch3[q] : ch.ch[k < 3 ? k : 0];
            if (child >= 0) {
                double2_t* out = reinterpret_cast<double2_t*>(U + size_t(child) * P + g * KQ + 4 * m);
                double2_t* row = reinterpret_cast<double2_t*>(
                    &us[k + 1 < depth ? sub_base(k + 1) + child - s.first[k < 3 ? k + 1 : 3] : 0][g * KQ + 4 * m]);
                #pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const double2_t o = k == 3 ? old3[q][j] : old[k < 3 ? k : 0][j];
                    const double2_t v = {o.x + (((acc[0][2 * j] + acc[1][2 * j]) + acc[2][2 * j]) + acc[3][2 * j]),
                                         o.y + (((acc[0][2 * j + 1] + acc[1][2 * j + 1]) + acc[2][2 * j + 1]) + acc[3][2 * j + 1])};
                    out[j] = v;
                    if (k + 1 < depth) row[j] = v;
                }
            }
        }
        __syncthreads();
    }
}

// Mixed-precision operands of the outgoing expansions, once per box: q-hat split into FP32
// hi + lo parts (hi = fl32(q), lo = fl32(q - hi), so that hi + lo equals q to about 2^-48) and
// its charge sum in FP64, for boxes [0, nrows) (the all-zero row included).
__global__ void k_split_q(const double* Q, int32_t nrows, float* Qh, float* Ql, double* qs) {
    constexpr int P = kRankPad;
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t box = t / 64;
    const int lane = int(t & 63);
    if (box >= nrows) return;   // uniform over the wave: a wave is one box
    const double q = lane < P ? Q[box * P + lane] : 0.0;
    const float hi = float(q);
    if (lane < P) {
        Qh[box * P + lane] = hi;
        Ql[box * P + lane] = float(q - double(hi));
    }
    double s = q;
    #pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) qs[box] = s;
}

// Mixed-precision M2L on the FP32 matrix cores, on the same 128-box tiles as k_m2l (each wave's
// two column blocks in two passes over the 27 slots) with the same staging.  Each
// operator is written T^d = c_d 1 1^T + R^d with c_d its mean entry: the constant part,
// which carries the large log|d| level of the kernel, is applied in FP64 as c_d times the
// source's charge sum; only the remainder R^d, several times smaller, goes through FP32.
// R^d and q-hat are split into FP32 hi + lo parts (q-hat once per box by k_split_q).  Each
// 4-term step of R_hi q_hi is an FP32 product of its own, converted and added to the FP64
// accumulators at once, so FP32 rounding acts on four terms at a time; the cross terms
// R_hi q_lo and R_lo q_hi (about 2^-24 of the main term) accumulate in two FP32 accumulators
// over the slot and are flushed once.  The FP32 instruction returns element i of lane (g, n)
// as row 4 g + i.
__global__ __launch_bounds__(kBlock) void k_m2l_mixed(const BoxTile* tiles, const int32_t* ntiles_p,
                                                       const int32_t* box_list, const int32_t* il27,
                                                       const OpsPtrs* ops, const float* Qh, const float* Ql,
                                                       const double* qs, int32_t zrow, double* U) {
    constexpr int P = kRankPad, MT = P / 16, KQ = P / 4, NJ4 = KQ / 4;
    constexpr int A4 = P * P / 4;                      // float4 per operator part: 2.25 per thread
    static_assert(A4 == 2 * kBlock + kBlock / 4, "staging below assumes P = 48");
    __shared__ float4_t sH[2][A4];
    __shared__ float4_t sL[2][A4];
    __shared__ int s_dsl[kNumInteractions];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const int32_t ntiles = uniform(*ntiles_p);
    const int32_t G = int32_t(gridDim.x);
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    for (int32_t step = 0;; ++step) {
        const int32_t t = uniform(xcd_tile(int32_t(blockIdx.x), G, step, ntiles));
        if (t < 0) break;
        const int32_t count = uniform(tiles[t].count);
        if (count == 0) continue;
        const int32_t start = uniform(tiles[t].start), height = uniform(tiles[t].height);
        const int32_t cls = uniform(tiles[t].cls), opi = uniform(tiles[t].ops);
        const int rk = ops[opi].rank[height];
        const size_t hbase = size_t(height) * kNumIfoSlots * A4;
        const gptr<float4_t> Hh = global(reinterpret_cast<const float4_t*>(ops[opi].ifo_hi)) + hbase;
        const gptr<float4_t> Lh = global(reinterpret_cast<const float4_t*>(ops[opi].ifo_lo)) + hbase;
        const gptr<double> mono = global(ops[opi].mono) + size_t(height) * kNumIfoSlots;
        // lane group g supplies rows 12 g .. 12 g + 11 of its column's q-hat
        const gptr<float4_t> QH = global(reinterpret_cast<const float4_t*>(Qh)) + 3 * g;
        const gptr<float4_t> QL = global(reinterpret_cast<const float4_t*>(Ql)) + 3 * g;
        const gptr<double> QS = global(qs);
        if (tid < kNumInteractions) s_dsl[tid] = c_dslot.s[cls][tid];
        __syncthreads();
        const int* dsl = s_dsl;
        // the wave's two 16-box column blocks (boxes 32 w .. 32 w + 31 of the tile), one pass each
        for (int cb = 0; cb < 2; ++cb) {
        const bool wave_on = 32 * wave + 16 * cb < count;
        const int col = 32 * wave + 16 * cb + n;
        const int32_t box = (col < count) ? box_list[start + col] : -1;
        const gptr<int32_t> il = global(il27 + size_t(box >= 0 ? box : 0) * kNumInteractions);
        int32_t src = (box >= 0) ? il[0] : -1;
        src = src < 0 ? zrow : src;
        float4_t h0 = QH[size_t(src) * 12], h1 = QH[size_t(src) * 12 + 1], h2 = QH[size_t(src) * 12 + 2];
        float4_t l0 = QL[size_t(src) * 12], l1 = QL[size_t(src) * 12 + 1], l2 = QL[size_t(src) * 12 + 2];
        double qsum = QS[src];
        int32_t src_next = (box >= 0) ? il[1] : -1;
        size_t off = size_t(dsl[0]) * A4;
        float4_t rh0 = Hh[off + tid], rh1 = Hh[off + tid + kBlock];
        float4_t rl0 = Lh[off + tid], rl1 = Lh[off + tid + kBlock];
        float4_t rh2 = (tid < kBlock / 4) ? Hh[off + tid + 2 * kBlock] : zero;
        float4_t rl2 = (tid < kBlock / 4) ? Lh[off + tid + 2 * kBlock] : zero;
        double4_t acc[MT];
        #pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = double4_t{0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < kNumInteractions; ++k) {
            const int bsel = k & 1;
            sH[bsel][tid] = rh0;
            sH[bsel][tid + kBlock] = rh1;
            sL[bsel][tid] = rl0;
            sL[bsel][tid + kBlock] = rl1;
            if (tid < kBlock / 4) {
                sH[bsel][tid + 2 * kBlock] = rh2;
                sL[bsel][tid + 2 * kBlock] = rl2;
            }
            const float4_t bh[NJ4] = {h0, h1, h2}, bl[NJ4] = {l0, l1, l2};
            const double cq = qsum;
            const int d = dsl[k];
            __syncthreads();
            if (k + 1 < kNumInteractions) {
                const int32_t sn = src_next < 0 ? zrow : src_next;
                h0 = QH[size_t(sn) * 12];
                h1 = QH[size_t(sn) * 12 + 1];
                h2 = QH[size_t(sn) * 12 + 2];
                l0 = QL[size_t(sn) * 12];
                l1 = QL[size_t(sn) * 12 + 1];
                l2 = QL[size_t(sn) * 12 + 2];
                qsum = QS[sn];
                src_next = (box >= 0 && k + 2 < kNumInteractions) ? il[k + 2] : -1;
                off = size_t(dsl[k + 1]) * A4;
                rh0 = Hh[off + tid];
                rh1 = Hh[off + tid + kBlock];
                rl0 = Lh[off + tid];
                rl1 = Lh[off + tid + kBlock];
                if (tid < kBlock / 4) {
                    rh2 = Hh[off + tid + 2 * kBlock];
                    rl2 = Lh[off + tid + 2 * kBlock];
                }
            }
            if (wave_on) {
                const double mq = mono[d] * cq;   // constant part of T^d times the charge sum
                #pragma unroll
                for (int m = 0; m < MT; ++m) {
                    #pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (16 * m + 4 * g + i < rk) acc[m][i] += mq;   // padded rows stay zero
                }
                #pragma unroll
                for (int m = 0; m < MT; ++m) {
                    float4_t c1 = zero, c2 = zero;
                    #pragma unroll
                    for (int j4 = 0; j4 < NJ4; ++j4) {
                        const float4_t ah = sH[bsel][(m * NJ4 + j4) * 64 + lane];
                        const float4_t al = sL[bsel][(m * NJ4 + j4) * 64 + lane];
                        #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float4_t p = __builtin_amdgcn_mfma_f32_16x16x4f32(ah[e], bh[j4][e], zero, 0, 0, 0);
                            c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ah[e], bl[j4][e], c1, 0, 0, 0);
                            c2 = __builtin_amdgcn_mfma_f32_16x16x4f32(al[e], bh[j4][e], c2, 0, 0, 0);
                            #pragma unroll
                            for (int i = 0; i < 4; ++i) acc[m][i] += double(p[i]);
                        }
                    }
                    #pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][i] += double(c1[i]) + double(c2[i]);
                }
            }
        }
        if (box >= 0) {
            double* ub = U + size_t(box) * P;
            #pragma unroll
            for (int m = 0; m < MT; ++m) {
                #pragma unroll
                for (int i = 0; i < 4; ++i) ub[16 * m + 4 * g + i] = acc[m][i];   // FP32 output layout
            }
        }
        __syncthreads();   // the next pass (or tile) rewrites the staging buffers
        }
    }
}

// bf16 mixed precision.  On gfx950 the bf16 matrix instructions run 32 times faster than the
// FP64 ones (16x16x32 in 16 cycles against 16x16x4 in 64), while FP32 runs only twice as fast,
// so that a split FP32 product (three instructions) cannot beat FP64.  Here q-hat and R^d
// (T^d less its constant part, applied in FP64 as for the FP32 form) are each split into three
// bf16 parts, x = x0 + x1 + x2 with x_k the rounded remainder of the parts before (about 24
// significant bits in all), and R q is formed from the six products R_a q_b with a + b <= 2:
// the dropped ones are below 2^-24 of the leading product.  bf16 x bf16 products are exact in
// FP32.  The six 48-term products are 36 (product, group of 8 columns) pieces, laid along the
// contraction of nine K = 32 instructions that sum into one FP32 accumulator, which is added
// to the FP64 accumulator once per interaction.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// bits of the bf16 nearest to x (through FP32, as the operators' host split) and their value
__device__ inline uint32_t bf16_bits(double x) {
    uint32_t u = __float_as_uint(float(x));
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ inline double bf16_val(uint32_t b) { return double(__uint_as_float(b << 16)); }

// q-hat in three bf16 parts (row of a box: part p holds entries p * 48 .. p * 48 + 47) and its
// FP64 charge sum, for boxes [0, nrows) (the all-zero row included); each remainder is exact.
// Eight lanes per box, lane g < 6 taking entries 8 g .. 8 g + 7 (one 64-byte read, one 16-byte
// write per part); the charge sum adds the six lanes' partial sums in a fixed order.
__global__ void k_split_q_bf16(const double* Q, int32_t nrows, uint16_t* Qb, double* qs) {
    constexpr int P = kRankPad;
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t box = t >> 3;
    const int g = int(t & 7);
    if (box >= nrows) return;   // uniform over each 8-lane group
    double part_sum = 0.0;
    if (g < P / 8) {
        const double2* src = reinterpret_cast<const double2*>(Q + box * P + 8 * g);
        double q[8];
        #pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double2 v = src[e];
            q[2 * e] = v.x;
            q[2 * e + 1] = v.y;
        }
        uint32_t bits[3][4];
        #pragma unroll
        for (int e = 0; e < 8; ++e) {
            part_sum += q[e];
            double r = q[e];
            #pragma unroll
            for (int part = 0; part < 3; ++part) {
                const uint32_t b = bf16_bits(r);
                r -= bf16_val(b);
                if (e & 1) bits[part][e >> 1] |= b << 16;
                else bits[part][e >> 1] = b;
            }
        }
        uint4* row = reinterpret_cast<uint4*>(Qb + box * (3 * P));
        #pragma unroll
        for (int part = 0; part < 3; ++part)
            row[part * (P / 8) + g] = make_uint4(bits[part][0], bits[part][1], bits[part][2], bits[part][3]);
    }
    part_sum += __shfl_xor(part_sum, 1, 64);
    part_sum += __shfl_xor(part_sum, 2, 64);
    part_sum += __shfl_xor(part_sum, 4, 64);
    if (g == 0) qs[box] = part_sum;
}

// M2L on the bf16 matrix cores, on the same 128-box tiles as k_m2l: eight waves per tile, wave w
// owning the 16-box column block w, four waves per SIMD.  (Two column blocks per wave would
// read each operator fragment from LDS once for two products, but its registers allow only
// two waves per SIMD, too few to hide the latencies of a slot that lasts a quarter of an FP64
// one; measured slower.)  The operator's three parts (13.5 KB) are staged in LDS once per slot
// and block.
//
// Contraction layout.  16x16x32 bf16 instruction: lane (g, n) supplies row n of the operator
// and column n of q-hat at contraction indices 8 g .. 8 g + 7 (one group of 8 columns of one
// part each); element i of its result is row 4 g + i, column n.  Lane group g owns column
// groups c = 3 (g & 1) + t, t = 0, 1, 2; in instruction j = 3 t + r it takes column group
// 3 (g & 1) + t of the product
//   g = 0, 1:  r = 0: R0 q0,  r = 1: R1 q0,  r = 2: R2 q0
//   g = 2, 3:  r = 0: R0 q1,  r = 1: R1 q1,  r = 2: R0 q2
// so every (product, column group) piece appears once, and a lane reads three groups of q-hat
// (g = 0, 1: q0) or six (g = 2, 3: q1 and q2) per source.
//
// Rounding.  The leading product R0 q0 sits in the instructions r = 0 (a third of it in each);
// each of them starts from zero and is added to the FP64 accumulator at once, so FP32 rounds
// partial sums of a third of the leading product only.  The r = 1, 2 instructions (at most
// 2^-8 of it) share one FP32 sum per interaction.  The constant part c_d times the source's
// charge sum is summed per column in FP64 and added once at the end.
//
// The next slot's q-hat groups are loaded into the registers of group t as soon as the
// current slot's instructions 3 t .. 3 t + 2 have read them.
__global__ __launch_bounds__(kBf16Block, 4) void k_m2l_bf16(const BoxTile* tiles, const int32_t* ntiles_dev,
                                                              const int32_t* box_list, const int32_t* il27,
                                                              const OpsPtrs* ops, const uint16_t* Qb,
                                                              const double* qs, int32_t zrow, double* U) {
    const int32_t ntiles = uniform(*ntiles_dev);
    constexpr int P = kRankPad, NS = kNumInteractions, NF = kBf16OpVecs, NT = kBf16Block;
    static_assert(kM2LTile == 16 * (kBf16Block / 64), "one column block per wave");
    constexpr int NST = (NF + NT - 1) / NT;     // staged groups per thread
    constexpr uint32_t QB = kBf16QVecs * 16;    // bytes of q-hat parts per box
    __shared__ u32x4_t sA[2][NF];
    __shared__ int32_t s_src[kM2LTile * NS];     // source box of (tile column, slot), zrow if none
    __shared__ int32_t s_box[kM2LTile];
    __shared__ int s_dsl[NS];
    __shared__ double s_mono[NS];
    const int tid = int(threadIdx.x), wave = tid >> 6, lane = tid & 63;
    const int n = lane & 15, g = lane >> 4;
    const bool q0_lanes = g < 2;                 // lane groups 0, 1: the three products with q0
    const int c0 = 3 * (g & 1);                  // first column group of the lane group
    const int32_t G = int32_t(gridDim.x);
    const u32x4_t z4 = {0u, 0u, 0u, 0u};
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    // operator fragment of instruction j = 3 t + r, row block m: group
    // pa * 288 + 96 m + 16 (c0 + t) + n with pa = r, except pa = 0 for r = 2 on lanes 2, 3
    const int abase = c0 * 16 + n;
    const int abase2 = abase + (q0_lanes ? 2 * 288 : 0);
    // q-hat groups of a source, byte offsets: lanes 0, 1 part 0, groups c0 .. c0 + 2 (twice, so
    // that instruction r = 2 reads the second copy on every lane); lanes 2, 3 part 1, then part 2
    const uint32_t qoff1 = uint32_t((q0_lanes ? 0 : 6) + c0) * 16u;
    const uint32_t qoff2 = uint32_t((q0_lanes ? 0 : 12) + c0) * 16u;
    const int col = 16 * wave + n;               // this lane's column of the tile
    for (int32_t step = 0;; ++step) {
        const int32_t t = uniform(xcd_tile(int32_t(blockIdx.x), G, step, ntiles));
        if (t < 0) break;                                  // uniform over the block
        const int32_t count = uniform(tiles[t].count);
        if (count == 0) continue;
        const int32_t start = uniform(tiles[t].start), height = uniform(tiles[t].height);
        const int32_t cls = uniform(tiles[t].cls), opi = uniform(tiles[t].ops);
        if (tid < NS) {
            const int d = height * kNumIfoSlots + c_dslot.s[cls][tid];
            s_dsl[tid] = d;
            s_mono[tid] = ops[opi].mono[d];
        }
        if (tid < kM2LTile) s_box[tid] = (tid < count) ? box_list[start + tid] : -1;
        __syncthreads();
        for (int i = tid; i < kM2LTile * NS; i += NT) {
            const int b = i / NS;
            const int32_t box = s_box[b];
            const int32_t src = box >= 0 ? il27[size_t(box) * NS + (i - b * NS)] : -1;
            s_src[i] = src < 0 ? zrow : src;
        }
        const int rk = uniform(ops[opi].rank[height]);
        const gptr<u32x4_t> Ah = global(reinterpret_cast<const u32x4_t*>(ops[opi].ifo_b));
        const gptr<double> QS = global(qs);
        const gptr<uint8_t> Xb = global(reinterpret_cast<const uint8_t*>(Qb));
        const int32_t box = s_box[col];
        __syncthreads();
        const int32_t* srcs = s_src + col * NS;
        // q-hat groups of the slot's source: [t] first part, [3 + t] the part that instruction
        // 3 t + 2 reads; sources addressed by 32-bit byte offsets from Qb
        u32x4_t bq[6];
        uint32_t qn = uint32_t(srcs[0]) * QB;
        double nsum = QS[srcs[0]];
        auto load_group = [&](int tt) {
            bq[tt] = *reinterpret_cast<gptr<u32x4_t>>(Xb + (qn + qoff1 + 16u * tt));
            bq[3 + tt] = *reinterpret_cast<gptr<u32x4_t>>(Xb + (qn + qoff2 + 16u * tt));
        };
        #pragma unroll
        for (int tt = 0; tt < 3; ++tt) load_group(tt);
        int32_t dsl_next = s_dsl[1];
        u32x4_t ra[NST];
        {
            const gptr<u32x4_t> A0 = Ah + size_t(s_dsl[0]) * NF;
            #pragma unroll
            for (int e = 0; e < NST; ++e) ra[e] = (e * NT + tid < NF) ? A0[e * NT + tid] : z4;
        }
        double4_t acc[3];
        #pragma unroll
        for (int m = 0; m < 3; ++m) acc[m] = double4_t{0.0, 0.0, 0.0, 0.0};
        double mono_acc = 0.0;
        for (int k = 0; k < NS; ++k) {
            u32x4_t* buf = sA[k & 1];
            #pragma unroll
            for (int e = 0; e < NST; ++e)
                if (e * NT + tid < NF) buf[e * NT + tid] = ra[e];
            mono_acc += s_mono[k] * nsum;   // constant part of T^d times the charge sum
            __syncthreads();
            if (k + 1 < NS) {   // the next slot's operator, into registers; its source
                const gptr<u32x4_t> An = Ah + size_t(uniform(dsl_next)) * NF;
                #pragma unroll
                for (int e = 0; e < NST; ++e)
                    if (e * NT + tid < NF) ra[e] = An[e * NT + tid];
                dsl_next = (k + 2 < NS) ? s_dsl[k + 2] : 0;
                const int32_t sn = srcs[k + 1];
                qn = uint32_t(sn) * QB;
                nsum = QS[sn];
            }
            asm volatile("" ::: "memory");
            float4_t small[3];
            #pragma unroll
            for (int tt = 0; tt < 3; ++tt) {
                #pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const int j = 3 * tt + r;
                    // three operator fragments in flight: more would cost the fourth wave per SIMD
                    asm volatile("" ::: "memory");
                    #pragma unroll
                    for (int m = 0; m < 3; ++m) {
                        const u32x4_t a =
                            (r == 2) ? buf[abase2 + 96 * m + 16 * tt] : buf[abase + r * 288 + 96 * m + 16 * tt];
                        // r = 2: q0 (lanes 0, 1) or q2 (lanes 2, 3); else the lane group's first part
                        const u32x4_t b = (r == 2) ? bq[3 + tt] : bq[tt];
                        const bf16x8_t av = __builtin_bit_cast(bf16x8_t, a), bv = __builtin_bit_cast(bf16x8_t, b);
                        if (r == 0) {
                            const float4_t p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, zero, 0, 0, 0);
                            #pragma unroll
                            for (int i = 0; i < 4; ++i) acc[m][i] += double(p[i]);
                        } else {
                            small[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, j == 1 ? zero : small[m], 0,
                                                                               0, 0);
                        }
                    }
                }
                if (k + 1 < NS) load_group(tt);   // group tt of the next slot's source
            }
            #pragma unroll
            for (int m = 0; m < 3; ++m)
                #pragma unroll
                for (int i = 0; i < 4; ++i) acc[m][i] += double(small[m][i]);
        }
        if (box >= 0) {
            double* ob = U + size_t(box) * P;
            #pragma unroll
            for (int m = 0; m < 3; ++m)
                #pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * m + 4 * g + i;
                    ob[row] = acc[m][i] + (row < rk ? mono_acc : 0.0);   // padded rows stay zero
                }
        }
        __syncthreads();   // the next tile rewrites the staging buffers and lists read above
    }
}

// M2L for plans of few tiles (all precisions).  On the 128-box tiles above a block runs 27 slots
// of 72 products per wave, so a plan of a handful of tiles lasts a whole tile's time (70-80 us) on a
// handful of compute units.  Here a block takes one 16-box column block of a tile, one row block per
// wave: the same products in the same order per result (bit-equal to the kernels above, which an
// instance alone and in a forest relies on), spread over 24 waves per tile.  Operator fragments go
// straight from the fragment-ordered tables to registers, the next slots' loads in flight; the
// source expansions are loaded once per block (consecutive lanes on consecutive bytes of a row: a
// fragment load spreads its lanes over 16 rows, and three waves of them saturated the texture
// addresser), written to LDS, one barrier per slot, and read from there as fragments.  Slots that no
// box of the column block has a source for are skipped: they would add zeros, and on curve-like
// point sets (the boundary of a box) they are most of the list.  What is left is the chain of 27 x 12
// dependent products (9.7 us) and about 10 us of dependent loads before it.  Phase times before / now:
// 1,000 uniform points 70 / 23 us (FP32 mixed 110 / 42, bf16 52 / 27), 64,000 points 80 / 35 us,
// 128,000 points on the boundary of a box 78 / 24 us.
constexpr int kFineCols = 16;
constexpr int kFineThreads = 64 * (kRankPad / 16);
constexpr int kFineDepth = 3;   // register sets of the slot pipeline (4: a wave less per SIMD, no faster)

// LDS of a fine block: interaction lists of its columns (absent sources as zrow), the slots any of
// them uses, and the staged expansions (NV 16-byte vectors a row, one more of padding).
template <int NV>
struct FineLds {
    int32_t src[kFineCols * kNumInteractions];
    uint32_t slots;
    u32x4_t rows[2][kFineCols * (NV + 1)];
};

// What a wave of the fine kernels needs of its tile; on false: nothing to do (uniform over the block).
struct FineTile {
    int32_t height, opi, box;   // box of this lane's column, -1 past the tile's end
    int dsl;                    // lane k < 27: operator index of slot k
    uint32_t slots;
    bool on;
};

template <int NV>
__device__ inline FineTile fine_tile(const BoxTile* tiles, const int32_t* ntiles_dev, const int32_t* box_list,
                                     const int32_t* il27, int32_t zrow, FineLds<NV>& s) {
    constexpr int NS = kNumInteractions, NB = kFineCols;
    FineTile f{};
    const int32_t b = int32_t(blockIdx.x), t = b / (kM2LTile / NB), q = b % (kM2LTile / NB);
    // the tile (inside its table whatever their number) and the number of tiles in one round trip
    const cptr<int4_t> tile = as_const(reinterpret_cast<const int4_t*>(tiles + t));
    const int4_t t0 = tile[0], t1 = tile[1];   // ops, height, cls, start; count
    const int32_t ntiles = as_const(ntiles_dev)[0];
    const int32_t cols = min(NB, t1.x - NB * q), start = t0.w + NB * q;
    if (t >= ntiles || cols <= 0) return f;
    const int tid = int(threadIdx.x), lane = tid & 63, n = lane & 15;
    if (tid == 0) s.slots = 0u;
    // every thread's list entries loaded together (a column past the tile reads the last one's)
    constexpr int NR = (NB * NS + kFineThreads - 1) / kFineThreads;
    int32_t src[NR];
    #pragma unroll
    for (int r = 0; r < NR; ++r) src[r] = box_list[start + min(min(tid + r * kFineThreads, NB * NS - 1) / NS, cols - 1)];
    f.box = box_list[start + min(n, cols - 1)];
    #pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int i = min(tid + r * kFineThreads, NB * NS - 1);
        src[r] = il27[size_t(src[r]) * NS + (i - i / NS * NS)];
    }
    f.on = true;
    f.height = t0.y;
    f.opi = t0.x;
    if (n >= cols) f.box = -1;
    f.dsl = f.height * kNumIfoSlots + (lane < NS ? c_dslot.s[t0.z][lane] : 0);
    __syncthreads();
    uint32_t mine = 0u;
    #pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int i = tid + r * kFineThreads, c = i / NS;
        if (c >= cols || src[r] < 0) src[r] = zrow;
        else mine |= 1u << (i - c * NS);
        if (i < NB * NS) s.src[i] = src[r];
    }
    if (mine) atomicOr(&s.slots, mine);
    __syncthreads();
    f.slots = uint32_t(uniform(int32_t(s.slots)));
    return f;
}

// The slots in order: frag(a, k) loads the operator fragments of slot k, row(src, v) names vector v of
// a source's expansion, use(a, b) runs the products with the staged row b of this lane's column.
// kFineDepth register sets in turn, reloaded right after their use (past the last slot with the last
// one again).  The buffer a slot writes was last read two slots earlier, before the previous barrier.
template <int NV, class Frag, class LoadFrag, class Row, class Use>
__device__ inline void fine_slots(uint32_t slots, FineLds<NV>& s, LoadFrag frag, Row row, Use use) {
    constexpr int NR = (kFineCols * NV + kFineThreads - 1) / kFineThreads;
    struct Set {
        Frag a;
        u32x4_t b[NR];
    };
    const int tid = int(threadIdx.x), n = tid & 15;
    int left = __popc(slots), k = 0, par = 0;
    if (left == 0) return;
    int rsrc[NR], rvec[NR], rlds[NR];   // list position, vector and place in LDS of this thread's loads
    #pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int i = min(tid + r * kFineThreads, kFineCols * NV - 1), c = i / NV;
        rsrc[r] = c * kNumInteractions;
        rvec[r] = i - c * NV;
        rlds[r] = c * (NV + 1) + rvec[r];
    }
    Set set[kFineDepth];
    auto fetch = [&](Set& t) {
        if (slots) {
            k = __ffs(int(slots)) - 1;
            slots &= slots - 1u;
        }
        #pragma unroll
        for (int r = 0; r < NR; ++r) t.b[r] = *row(size_t(s.src[rsrc[r] + k]), rvec[r]);
        frag(t.a, k);
        asm volatile("" ::: "memory");   // keeps the loads here, not sunk to their uses
    };
    #pragma unroll
    for (int d = 0; d < kFineDepth; ++d) fetch(set[d]);
    for (;;) {
        #pragma unroll
        for (int d = 0; d < kFineDepth; ++d) {
            u32x4_t* buf = s.rows[par];
            par ^= 1;
            #pragma unroll
            for (int r = 0; r < NR; ++r) buf[rlds[r]] = set[d].b[r];
            __syncthreads();
            use(set[d].a, buf + n * (NV + 1));
            if (--left == 0) return;
            fetch(set[d]);
        }
    }
}

__global__ __launch_bounds__(kFineThreads) void k_m2l_fine(const BoxTile* tiles, const int32_t* ntiles_dev,
                                                           const int32_t* box_list, const int32_t* il27,
                                                           const OpsPtrs* ops, const double* Q, int32_t zrow,
                                                           double* U) {
    constexpr int P = kRankPad, NJ = P / 8, A2 = P * P / 2, NV = P / 2;
    __shared__ FineLds<NV> lds;
    const FineTile f = fine_tile(tiles, ntiles_dev, box_list, il27, zrow, lds);
    if (!f.on) return;
    const int m = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63, g = lane >> 4;
    const gptr<double2_t> A = global(reinterpret_cast<const double2_t*>(ops[f.opi].ifo)) + size_t(m * NJ) * 64 + lane;
    const gptr<u32x4_t> X = global(reinterpret_cast<const u32x4_t*>(Q));
    struct Frag {
        double2_t a[NJ];
    };
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    fine_slots<NV, Frag>(
        f.slots, lds,
        [&](Frag& s, int k) {
            const gptr<double2_t> Ak = A + size_t(__builtin_amdgcn_readlane(f.dsl, k)) * A2;
            #pragma unroll
            for (int j = 0; j < NJ; ++j) s.a[j] = Ak[j * 64];
        },
        [&](size_t src, int v) { return X + src * NV + v; },
        [&](const Frag& s, const u32x4_t* b) {
            #pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const double2_t q = __builtin_bit_cast(double2_t, b[g * NJ + j]);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s.a[j].x, q.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s.a[j].y, q.y, acc, 0, 0, 0);
            }
        });
    if (f.box >= 0) {
        double* ob = U + size_t(f.box) * P + 16 * m + g;
        #pragma unroll
        for (int i = 0; i < 4; ++i) ob[4 * i] = acc[i];
    }
}

__global__ __launch_bounds__(kFineThreads) void k_m2l_mixed_fine(const BoxTile* tiles, const int32_t* ntiles_dev,
                                                                 const int32_t* box_list, const int32_t* il27,
                                                                 const OpsPtrs* ops, const float* Qh, const float* Ql,
                                                                 const double* qs, int32_t zrow, double* U) {
    constexpr int P = kRankPad, NJ4 = P / 16, A4 = P * P / 4, NH = P / 4, NV = 2 * NH;
    __shared__ FineLds<NV> lds;
    const FineTile f = fine_tile(tiles, ntiles_dev, box_list, il27, zrow, lds);
    if (!f.on) return;
    const int m = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63, n = lane & 15, g = lane >> 4;
    const gptr<float4_t> H = global(reinterpret_cast<const float4_t*>(ops[f.opi].ifo_hi)) + size_t(m * NJ4) * 64 + lane;
    const gptr<float4_t> L = global(reinterpret_cast<const float4_t*>(ops[f.opi].ifo_lo)) + size_t(m * NJ4) * 64 + lane;
    const gptr<u32x4_t> XH = global(reinterpret_cast<const u32x4_t*>(Qh)), XL = global(reinterpret_cast<const u32x4_t*>(Ql));
    const gptr<double> mono = global(ops[f.opi].mono), QS = global(qs);
    const int rk = uniform(ops[f.opi].rank[f.height]);
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    struct Frag {
        float4_t ah[NJ4], al[NJ4];
        double c, q;
    };
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    fine_slots<NV, Frag>(
        f.slots, lds,
        [&](Frag& s, int k) {
            const size_t d = size_t(__builtin_amdgcn_readlane(f.dsl, k));
            #pragma unroll
            for (int j = 0; j < NJ4; ++j) {
                s.ah[j] = H[d * A4 + j * 64];
                s.al[j] = L[d * A4 + j * 64];
            }
            s.c = mono[d];
            s.q = QS[size_t(lds.src[n * kNumInteractions + k])];
        },
        [&](size_t src, int v) { return v < NH ? XH + src * NH + v : XL + src * NH + (v - NH); },
        [&](const Frag& s, const u32x4_t* b) {
            const double mq = s.c * s.q;   // constant part of T^d times the charge sum
            #pragma unroll
            for (int i = 0; i < 4; ++i)
                if (16 * m + 4 * g + i < rk) acc[i] += mq;
            float4_t c1 = zero, c2 = zero;
            #pragma unroll
            for (int j = 0; j < NJ4; ++j) {
                const float4_t bh = __builtin_bit_cast(float4_t, b[g * NJ4 + j]);
                const float4_t bl = __builtin_bit_cast(float4_t, b[NH + g * NJ4 + j]);
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4_t p = __builtin_amdgcn_mfma_f32_16x16x4f32(s.ah[j][e], bh[e], zero, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(s.ah[j][e], bl[e], c1, 0, 0, 0);
                    c2 = __builtin_amdgcn_mfma_f32_16x16x4f32(s.al[j][e], bh[e], c2, 0, 0, 0);
                    #pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i] += double(p[i]);
                }
            }
            #pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += double(c1[i]) + double(c2[i]);
        });
    if (f.box >= 0) {
        double* ob = U + size_t(f.box) * P + 16 * m + 4 * g;
        #pragma unroll
        for (int i = 0; i < 4; ++i) ob[i] = acc[i];
    }
}

__global__ __launch_bounds__(kFineThreads) void k_m2l_bf16_fine(const BoxTile* tiles, const int32_t* ntiles_dev,
                                                                const int32_t* box_list, const int32_t* il27,
                                                                const OpsPtrs* ops, const uint16_t* Qb,
                                                                const double* qs, int32_t zrow, double* U) {
    constexpr int P = kRankPad, NF = kBf16OpVecs, NV = kBf16QVecs;
    __shared__ FineLds<NV> lds;
    const FineTile f = fine_tile(tiles, ntiles_dev, box_list, il27, zrow, lds);
    if (!f.on) return;
    const int m = int(threadIdx.x) >> 6, lane = int(threadIdx.x) & 63, n = lane & 15, g = lane >> 4;
    const bool q0_lanes = g < 2;                 // the contraction layout of k_m2l_bf16
    const int c0 = 3 * (g & 1);
    const gptr<u32x4_t> A = global(reinterpret_cast<const u32x4_t*>(ops[f.opi].ifo_b)) + c0 * 16 + n + 96 * m;
    const gptr<u32x4_t> X = global(reinterpret_cast<const u32x4_t*>(Qb));
    const int a2 = q0_lanes ? 2 * 288 : 0, b1 = c0 + (q0_lanes ? 0 : 6), b2 = c0 + (q0_lanes ? 0 : 12);
    const gptr<double> mono = global(ops[f.opi].mono), QS = global(qs);
    const int rk = uniform(ops[f.opi].rank[f.height]);
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    struct Frag {
        u32x4_t a[9];
        double c, q;
    };
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    double mono_acc = 0.0;
    fine_slots<NV, Frag>(
        f.slots, lds,
        [&](Frag& s, int k) {
            const size_t d = size_t(__builtin_amdgcn_readlane(f.dsl, k));
            const gptr<u32x4_t> Ak = A + d * NF;
            #pragma unroll
            for (int t = 0; t < 3; ++t) {
                s.a[3 * t] = Ak[16 * t];
                s.a[3 * t + 1] = Ak[288 + 16 * t];
                s.a[3 * t + 2] = Ak[a2 + 16 * t];
            }
            s.c = mono[d];
            s.q = QS[size_t(lds.src[n * kNumInteractions + k])];
        },
        [&](size_t src, int v) { return X + src * NV + v; },
        [&](const Frag& s, const u32x4_t* b) {
            mono_acc += s.c * s.q;
            float4_t small = zero;
            #pragma unroll
            for (int t = 0; t < 3; ++t)
                #pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const bf16x8_t av = __builtin_bit_cast(bf16x8_t, s.a[3 * t + r]);
                    const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, b[(r == 2 ? b2 : b1) + t]);
                    if (r == 0) {
                        const float4_t p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, zero, 0, 0, 0);
                        #pragma unroll
                        for (int i = 0; i < 4; ++i) acc[i] += double(p[i]);
                    } else {
                        small = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, small, 0, 0, 0);
                    }
                }
            #pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += double(small[i]);
        });
    if (f.box >= 0) {
        double* ob = U + size_t(f.box) * P;
        #pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 16 * m + 4 * g + i;
            ob[row] = acc[i] + (row < rk ? mono_acc : 0.0);   // padded rows stay zero
        }
    }
}

// Leaf pass: far field T_tfi u-hat with T_tfi = T_ofs^T (Section 7, symmetric kernel and
// targets = sources) plus the direct sum over the points of the leaf and its neighbours
// (Section 8.2 step 5), written back in the caller's point order.
//
// A wave takes one group: the (up to four) leaves of one parent box, whose targets are one
// contiguous run of Morton-ordered points, one target per lane.  The sources are the points
// of the union of the leaves' neighbourhoods (a 4 x 4 block of leaves at most), listed per
// group at plan time as point ranges with their leaf coordinates.  The wave walks those
// ranges in lockstep: range and source reads are uniform over the wave (scalar loads), and a
// lane adds a range's sources only if that leaf neighbours its own leaf (the group's own leaves
// are one range, near to every lane).
//   WINDOW (side <= 16): phi sits in a window table over all offsets in [-(2s-1), 2s-1]^2 and
//     each point carries the key K = 8 (y W + x) mod 2^32 (W = 4s - 1), so the byte offset of
//     phi(x_i - x_j) is K_i - K_j plus a constant: one subtraction per pair.
//   QUAD (side 32): a table over |dx|, |dy| < 64; a pair's address is two sums of absolute differences.
enum LeafMode { kWindow = 0, kQuad = 1 };
constexpr int kNearXcdChunk = 512;     // most groups per chunk of the near field's XCD-aware walk
constexpr int kQuadRow = 65;           // doubles a row of the quad table (odd: rows start on different banks)
constexpr int kNearTabMax = 64 * kQuadRow;   // doubles: the quad table (side 32); W^2 = 63^2 of the window (side 16)
// Block size: 512 threads share one table among eight waves and run persistently (each block builds
// its table once).
constexpr int kNearBlock = 512;

// |a - b| + c in one instruction (spelled out, the compiler rearranges it into five); b uniform
__device__ inline uint32_t sad(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_sad_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// L2P of up to 64 targets i0 .. i0 + 63 (lane t holds the cell `loc` of target i0 + t): the far field
// of this lane's target.  Leaf by leaf, eight targets at a time with eight lanes each, so that a load
// reads whole 128-byte lines of eight operator rows and one of the leaf's expansion.  With one target
// per lane the 24 loads of a row's pairs each touched about 27 lines (and 64 rows of the cell-major
// table), and the texture addresser's time on them, 46 us of the pass on 1e6 points, was its largest
// part (21 us now).  A target's sum: six terms per lane in order, then the eight lanes' by a tree.
// FEW (groups of at most 32 targets): all of the group's targets in turn, eight a step, each with its own leaf's
// expansion, so that leaves of one or two targets do not take a step of sixteen each (the pass on 1e6 points of
// N_leaf 4: 890 -> 628 us, on 7e5 in clusters of N_leaf 8 540 -> 382; with sixteen a step, 85 registers for 79 and a
// block less per compute unit, 917).  The same bits.
// sfar: 64 doubles of LDS of this wave.
template <int P, bool FEW>
__device__ inline double far_rows(int32_t leaf0, int32_t nleaf, const int32_t (&bnd)[5], int32_t i0, int32_t loc,
                                  const double* leafT, const double* U, double* sfar) {
    static_assert(P == 48, "three 128-byte lines a row");
    const int lane = int(threadIdx.x) & 63, g8 = lane >> 3, l = lane & 7;
    const gptr<double2_t> T = global(reinterpret_cast<const double2_t*>(leafT)) + l;
    const gptr<double2_t> X = global(reinterpret_cast<const double2_t*>(U)) + size_t(leaf0) * (P / 2) + l;
    auto dpp_add = [](double v, auto ctrl) -> double {
        const int2_t w = __builtin_bit_cast(int2_t, v);
        return v + __builtin_bit_cast(double, int2_t{__builtin_amdgcn_update_dpp(0, w.x, ctrl(), 0xf, 0xf, true),
                                                     __builtin_amdgcn_update_dpp(0, w.y, ctrl(), 0xf, 0xf, true)});
    };
    auto row = [&](int32_t t) -> size_t { return size_t(__shfl(loc, min(t, 63), 64)) * (P / 2); };
    auto tree = [&](double v) {                 // the other of the pair, the other pair of the four, the
        v = dpp_add(v, [] { return 0xB1; });    // other four (mirrored)
        v = dpp_add(v, [] { return 0x4E; });
        return dpp_add(v, [] { return 0x141; });
    };
    if (FEW) {
        const int32_t nt = min(bnd[4] - i0, 64);
        for (int32_t t = 0; t < nt; t += 8) {
            const int32_t ta = t + g8, i = min(i0 + ta, bnd[4] - 1);   // past the last target the last one's leaf
            const gptr<double2_t> u = X + size_t((i >= bnd[1]) + (i >= bnd[2]) + (i >= bnd[3])) * (P / 2);
            const size_t ra = row(ta);
            const double2_t x0 = T[ra], x1 = T[ra + 8], x2 = T[ra + 16], u0 = u[0], u1 = u[8], u2 = u[16];
            double a = x0.x * u0.x;
            a += x0.y * u0.y;
            a += x1.x * u1.x;
            a += x1.y * u1.y;
            a += x2.x * u2.x;
            a += x2.y * u2.y;
            a = tree(a);
            if (l == 0 && ta < nt) sfar[ta] = a;
        }
    } else {
        for (int c = 0; c < nleaf; ++c) {
            const int32_t b0 = c == 0 ? bnd[0] : c == 1 ? bnd[1] : c == 2 ? bnd[2] : bnd[3];
            const int32_t b1 = c == 0 ? bnd[1] : c == 1 ? bnd[2] : c == 2 ? bnd[3] : bnd[4];
            const int32_t t0 = max(b0 - i0, 0), t1 = min(b1 - i0, 64);   // its targets among the 64 (uniform)
            if (t0 >= t1) continue;
            const gptr<double2_t> u = X + size_t(c) * (P / 2);
            const double2_t u0 = u[0], u1 = u[8], u2 = u[16];
            for (int32_t t = t0; t < t1; t += 16) {
                const int32_t ta = t + g8, tb = t + 8 + g8;
                const size_t ra = row(ta), rb = row(tb);
                const double2_t x0 = T[ra], x1 = T[ra + 8], x2 = T[ra + 16], y0 = T[rb], y1 = T[rb + 8], y2 = T[rb + 16];
                double a = x0.x * u0.x, b = y0.x * u0.x;
                a += x0.y * u0.y;
                b += y0.y * u0.y;
                a += x1.x * u1.x;
                b += y1.x * u1.x;
                a += x1.y * u1.y;
                b += y1.y * u1.y;
                a += x2.x * u2.x;
                b += y2.x * u2.x;
                a += x2.y * u2.y;
                b += y2.y * u2.y;
                a = tree(a);
                b = tree(b);
                if (l == 0 && ta < t1) sfar[ta] = a;
                if (l == 1 && tb < t1) sfar[tb] = b;
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const double v = sfar[lane];   // lanes past the targets: unused
    __builtin_amdgcn_wave_barrier();
    return v;
}

// One group of leaves (see k_near).
//   SLICED = false (groups of more than 32 targets): one target per lane over the whole group,
//     sources read at wave-uniform addresses (scalar loads); a lane adds a range's sources only
//     if that range's leaf neighbours its own leaf.
//   SLICED = true (groups of at most 32 targets): leaf by leaf; the n targets of a leaf take T lanes each
//     (T = the power of two at or above n, at most 64) of S = 64 / T slices, slice s summing
//     every S-th source of each neighbouring range, and the slices are added by xor shuffles.
// The group's record and entries come in registers (word l of the record in lane l, entry e in lane
// e), loaded while the wave worked on the group before: read from memory when needed, they put three
// dependent round trips in front of every group and one in front of every range, half the pass's time.
template <int P, int MODE, bool SLICED>
__device__ inline void near_group(int32_t rec, int4 ent, int64_t side, int W, const double* tab, const char* tb,
                                  uint32_t kofs, const int2* pts,
                                  const uint32_t* pkey, const double* fs, const int32_t* perm_local,
                                  const ExecPtrs* tab_ptrs, ExecPtrs single, const double* U,
                                  const double* leafT, double* sfar, int far_on) {
    const int lane = threadIdx.x & 63;
    const cptr<uint32_t> SK = as_const(pkey);
    const cptr<double> SF = as_const(fs);
    const cptr<int2_t> SP = as_const(reinterpret_cast<const int2_t*>(pts));
    auto word = [&](int k) -> int32_t { return __builtin_amdgcn_readlane(rec, k); };   // of the NearGroup
    const int32_t leaf0 = word(0), nleaf = word(1), ne = word(2);
    const int32_t bnd[5] = {word(4), word(5), word(6), word(7), word(8)};
    const int32_t lx0 = word(9), ly0 = word(10), cposs = word(11);
    const int32_t t_end = bnd[4];
    const bool far = word(12) != 0 && far_on;
    const ExecPtrs eio = tab_ptrs ? tab_ptrs[word(3)] : single;
    double* u = eio.u;
    if (SLICED && far) {   // of all the group's targets, into sfar
        const int2 p = pts[min(bnd[0] + lane, t_end - 1)];
        far_rows<P, true>(leaf0, nleaf, bnd, bnd[0], (p.x & int32_t(side - 1)) + int32_t(side) * (p.y & int32_t(side - 1)), leafT,
                    U, sfar);
    }
    const bool sorted_out = eio.sorted != 0;   // u indexed by sorted point
    const int32_t tgt0 = eio.tgt0;   // first target index
    // passes: the whole group once (group mode) or each leaf in turn (sliced mode)
    for (int c0 = 0; c0 < (SLICED ? nleaf : 1); ++c0) {
        const int32_t p0 = SLICED ? bnd[c0] : bnd[0];
        const int32_t p1 = SLICED ? bnd[c0 + 1] : t_end;
        int T = 64;
        if (SLICED) {
            T = 1;
            while (T < p1 - p0 && T < 64) T <<= 1;
        }
        const int S = 64 / T, tl = lane & (T - 1), sl = lane / T;
        for (int32_t i0 = p0; i0 < p1; i0 += T) {
            const int32_t i = i0 + tl;
            const bool valid = i < p1;
            const int32_t ii = valid ? i : p0;
            // leaves past the last start at t_end, after every point
            const int c = SLICED ? c0 : (ii >= bnd[1]) + (ii >= bnd[2]) + (ii >= bnd[3]);
            const int cpos = (cposs >> (2 * c)) & 3;
            const int2 pi = pts[ii];
            // the window centre's byte offset is folded into the target's key once, so that a
            // pair costs one subtraction for its table address
            const uint32_t ki = (MODE == kWindow) ? pkey[ii] + kofs : 0u;
            const int32_t pout = perm_local[ii];
            // QUAD: byte offsets of the table relative to the lower-left corner of the 4 x 4 leaves
            const int32_t gx = (lx0 - 1) * int32_t(side), gy = (ly0 - 1) * int32_t(side);
            const uint32_t qx = uint32_t(pi.x - gx) * 8u, qy = uint32_t(pi.y - gy) * (8u * kQuadRow);
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
            auto phi_at = [&](uint32_t kj, int2_t pj) -> double {
                if (MODE == kWindow) return *reinterpret_cast<const double*>(tb + int32_t(ki - kj));
                if (MODE == kQuad && !SLICED)   // the source is uniform: its offset is scaled by scalar instructions
                    return *reinterpret_cast<const double*>(
                        tb + sad(qy, uint32_t(pj.y - gy) * (8u * kQuadRow), sad(qx, uint32_t(pj.x - gx) * 8u, 0u)));
                const int dx = abs(pi.x - pj.x), dy = abs(pi.y - pj.y);
                return tab[dy * kQuadRow + dx];
            };
            auto src_key = [&](int32_t j) -> uint32_t {
                if (MODE != kWindow) return 0u;
                return SLICED ? pkey[j] : SK[j];
            };
            auto src_pt = [&](int32_t j) -> int2_t {
                if (MODE == kWindow) return int2_t{0, 0};
                if (SLICED) {
                    const int2 p = pts[j];
                    return int2_t{p.x, p.y};
                }
                return SP[j];
            };
            auto src_f = [&](int32_t j) -> double { return SLICED ? fs[j] : SF[j]; };
            for (int e = 0; e < ne; ++e) {
                const int32_t e0 = __builtin_amdgcn_readlane(ent.x, e), e1 = __builtin_amdgcn_readlane(ent.y, e);
                const int32_t em = __builtin_amdgcn_readlane(ent.z, e);   // child positions near to the range
                if ((em >> cpos) & 1) {   // uniform when sliced
                    int32_t j = e0 + sl;
                    if (!SLICED)   // sixteen sources per step: few waits for their scalar loads
                        for (; j + 15 < e1; j += 16) {
                            #pragma unroll
                            for (int r = 0; r < 16; r += 4) {
                                a0 += phi_at(src_key(j + r), src_pt(j + r)) * src_f(j + r);
                                a1 += phi_at(src_key(j + r + 1), src_pt(j + r + 1)) * src_f(j + r + 1);
                                a2 += phi_at(src_key(j + r + 2), src_pt(j + r + 2)) * src_f(j + r + 2);
                                a3 += phi_at(src_key(j + r + 3), src_pt(j + r + 3)) * src_f(j + r + 3);
                            }
                        }
                    if (!SLICED)
                        for (; j + 7 < e1; j += 8) {
                            a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                            a1 += phi_at(src_key(j + 1), src_pt(j + 1)) * src_f(j + 1);
                            a2 += phi_at(src_key(j + 2), src_pt(j + 2)) * src_f(j + 2);
                            a3 += phi_at(src_key(j + 3), src_pt(j + 3)) * src_f(j + 3);
                            a0 += phi_at(src_key(j + 4), src_pt(j + 4)) * src_f(j + 4);
                            a1 += phi_at(src_key(j + 5), src_pt(j + 5)) * src_f(j + 5);
                            a2 += phi_at(src_key(j + 6), src_pt(j + 6)) * src_f(j + 6);
                            a3 += phi_at(src_key(j + 7), src_pt(j + 7)) * src_f(j + 7);
                        }
                    for (; j + 3 * S < e1; j += 4 * S) {
                        a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                        a1 += phi_at(src_key(j + S), src_pt(j + S)) * src_f(j + S);
                        a2 += phi_at(src_key(j + 2 * S), src_pt(j + 2 * S)) * src_f(j + 2 * S);
                        a3 += phi_at(src_key(j + 3 * S), src_pt(j + 3 * S)) * src_f(j + 3 * S);
                    }
                    if (!SLICED) {
                        // the last one to three sources with their loads issued together (one wait)
                        const int32_t rem = e1 - j;
                        if (rem == 3) {
                            a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                            a1 += phi_at(src_key(j + 1), src_pt(j + 1)) * src_f(j + 1);
                            a2 += phi_at(src_key(j + 2), src_pt(j + 2)) * src_f(j + 2);
                        } else if (rem == 2) {
                            a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                            a1 += phi_at(src_key(j + 1), src_pt(j + 1)) * src_f(j + 1);
                        } else if (rem == 1) {
                            a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                        }
                    } else {
                        for (; j < e1; j += S) a0 += phi_at(src_key(j), src_pt(j)) * src_f(j);
                    }
                }
            }
            double acc = (a0 + a1) + (a2 + a3);
            if (SLICED)
                for (int o = T; o < 64; o <<= 1) acc += __shfl_xor(acc, o, 64);
            // the far field last, as when k_l2p adds it
            if (far)
                acc += SLICED ? sfar[ii - bnd[0]]
                              : far_rows<P, false>(leaf0, nleaf, bnd, i0, (pi.x & int32_t(side - 1)) +
                                                int32_t(side) * (pi.y & int32_t(side - 1)), leafT, U, sfar);
            if (valid && sl == 0 && pout >= tgt0) u[sorted_out ? int64_t(ii) : int64_t(pout - tgt0)] = acc;
        }
    }
}

// Four waves per SIMD: six spill scalar registers (16-source steps hold 48 of them) and measured
// 115 against 93 us.
template <int P, int MODE>
__global__ __launch_bounds__(kNearBlock, 4) void k_near(
    int32_t q0, int32_t q1, const NearGroup* groups, const int4* ents, int64_t side, int W, const int2* pts,
    const uint32_t* pkey, const double* fs, const int32_t* perm_local, const ExecPtrs* tab_ptrs, ExecPtrs single,
    const double* U, const double* leafT, const double* phi_oct_tab, int far_on) {
    constexpr int kNearWaves = kNearBlock / 64;
    // fixed-size table (the quadrant table of side 32, or a window of sides up to 16), so that its base is a
    // compile-time constant and folds into the address of every read
    __shared__ double tab[kNearTabMax];
    __shared__ double sfar[kNearWaves][64];   // far fields of each wave's targets
    const int tid = threadIdx.x, wave = tid >> 6;
    {
        const int c = (MODE == kWindow) ? int(2 * side - 1) : 0, n = (MODE == kWindow) ? W * W : W * kQuadRow;
        const int row = (MODE == kWindow) ? W : kQuadRow;
        constexpr int kU = 9;   // loads in flight per thread: the whole table in one round
        for (int i0 = tid; i0 < n; i0 += kNearBlock * kU) {
            double v[kU];
            #pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int i = min(i0 + u * kNearBlock, n - 1);
                const int dy = abs(i / row - c), dx = abs(i - (i / row) * row - c);
                const int hi = max(dx, dy), lo = min(dx, dy);
                v[u] = phi_oct_tab[hi * (hi + 1) / 2 + lo];
            }
            #pragma unroll
            for (int u = 0; u < kU; ++u)
                if (i0 + u * kNearBlock < n) tab[i0 + u * kNearBlock] = v[u];
        }
        __syncthreads();
    }
    const int cw = (MODE == kWindow) ? int(2 * side - 1) : 0;
    const char* tb = reinterpret_cast<const char*>(tab);
    const uint32_t kofs = 8u * uint32_t(cw * W + cw);
    // XCD-aware walk of the group list: block b runs on XCD b % 8, and XCD x takes the chunks x,
    // x + 8, x + 16, ... of C consecutive (Morton-ordered) groups, so that most sources that
    // neighbouring groups share are read through one L2 (on 1e6 uniform points 5 % faster than the
    // plain walk; one contiguous eighth per XCD was 8 % faster there but leaves an XCD with all of a
    // dense region's work, which the same split made 1.1-1.8x slower in the clustered kernels).
    // The list is cut into a multiple of 8 chunks of at most kNearXcdChunk groups, so that every XCD
    // has the same share: with chunks of 512 groups whatever the list, a plan of 1,024 groups ran on
    // two XCDs (16,000 uniform points 161 -> 28 us, 16,000 in 1/40 of the cells 301 -> 78 us).
    // With fewer than 8 blocks, the plain walk.
    const int32_t G = int32_t(gridDim.x);
    int32_t x = 0, first = int32_t(blockIdx.x), nb = G, C = q1 - q0 + 1;
    if (G >= 8) {
        x = first & 7;
        first >>= 3;
        nb = (G + 7 - x) >> 3;   // blocks on XCD x
        const int32_t n = q1 - q0, chunks = (n + 8 * kNearXcdChunk - 1) / (8 * kNearXcdChunk) * 8;
        C = (n + chunks - 1) / chunks;
    }
    // word l of group q's record in lane l, its entry l in lane l (and again in the other rows of 16)
    static_assert(sizeof(NearGroup) == 64, "16 words");
    const int rl = tid & 15;
    int32_t l = first * kNearWaves + wave, rec = 0;
    int4 ent = make_int4(0, 0, 0, 0);
    auto group_at = [&](int32_t ll) -> int32_t { return q0 + (8 * (ll / C) + x) * C + ll % C; };   // increases with ll
    auto fetch = [&](int32_t q) {
        if (q < q1) {
            rec = reinterpret_cast<const int32_t*>(groups)[size_t(q) * 16 + rl];
            ent = ents[size_t(q) * kNearEntries + rl];   // entries past the group's last are not used
        }
    };
    int32_t q = group_at(l);
    fetch(q);
    while (q < q1) {
        const int32_t r = rec;
        const int4 en = ent;
        l += nb * kNearWaves;
        q = group_at(l);
        fetch(q);
        asm volatile("" ::: "memory");   // the next group's loads go out here
        const int32_t nt = __builtin_amdgcn_readlane(r, 8) - __builtin_amdgcn_readlane(r, 4);
        // group mode when half a wave or more is busy, leaf by leaf otherwise
        if (nt > 32)
            near_group<P, MODE, false>(r, en, side, W, tab, tb, kofs, pts, pkey, fs, perm_local, tab_ptrs, single, U,
                                       leafT, sfar[wave], far_on);
        else
            near_group<P, MODE, true>(r, en, side, W, tab, tb, kofs, pts, pkey, fs, perm_local, tab_ptrs, single, U,
                                      leafT, sfar[wave], far_on);
    }
}

// Load statistics for the input checks: per block, the sum, the sum of magnitudes and the
// number of non-finite entries of its slice of f (fixed slices and a fixed tree order, so
// the totals do not depend on timing); then one block adds the partials in block order.
constexpr int kStatBlocks = 256;
__global__ __launch_bounds__(kBlock) void k_load_stats_part(const double* f, int64_t n, double* part) {
    __shared__ double ss[kBlock], sa[kBlock], sn[kBlock];
    const int64_t per = (n + kStatBlocks - 1) / kStatBlocks;
    const int64_t i0 = int64_t(blockIdx.x) * per, i1 = min(n, i0 + per);
    double s = 0.0, a = 0.0, bad = 0.0;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kBlock) {
        const double v = f[i];
        if (isfinite(v)) {
            s += v;
            a += fabs(v);
        } else {
            bad += 1.0;
        }
    }
    ss[threadIdx.x] = s;
    sa[threadIdx.x] = a;
    sn[threadIdx.x] = bad;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if (int(threadIdx.x) < o) {
            ss[threadIdx.x] += ss[threadIdx.x + o];
            sa[threadIdx.x] += sa[threadIdx.x + o];
            sn[threadIdx.x] += sn[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x] = ss[0];
        part[3 * blockIdx.x + 1] = sa[0];
        part[3 * blockIdx.x + 2] = sn[0];
    }
}

// (the partials come to LDS together: read one after the other from memory they took 9 to 13 us)
__global__ __launch_bounds__(kBlock) void k_load_stats_final(const double* part, double* out) {
    __shared__ double p[3][kStatBlocks];
    for (int i = threadIdx.x; i < 3 * kStatBlocks; i += kBlock) p[i % 3][i / 3] = part[i];
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        #pragma unroll 32
        for (int b = 0; b < kStatBlocks; ++b) s += p[threadIdx.x][b];
        out[threadIdx.x] = s;
    }
}

// L2P alone, for groups whose pairs k_near adds up beside the passes before this one: adds the far field to
// u, a wave per group (same bits as k_near with L2P, which adds it last).  Bound by the launch and three
// dependent loads, 5 to 6 us for plans of up to some thousand groups.
template <int P>
__global__ __launch_bounds__(kBlock) void k_l2p(int32_t q0, int32_t q1, const NearGroup* groups, int32_t side,
                                                 const int2* pts, const int32_t* perm_local, const ExecPtrs* tab_ptrs,
                                                 ExecPtrs single, const double* U, const double* leafT) {
    __shared__ double sfar[kWaves][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int32_t q = q0 + int32_t(blockIdx.x) * kWaves + wave; q < q1; q += int32_t(gridDim.x) * kWaves) {
        const int32_t rec = reinterpret_cast<const int32_t*>(groups)[size_t(q) * 16 + (lane & 15)];
        auto word = [&](int k) -> int32_t { return __builtin_amdgcn_readlane(rec, k); };   // of the NearGroup
        if (word(12) == 0) continue;
        const int32_t bnd[5] = {word(4), word(5), word(6), word(7), word(8)};
        const ExecPtrs eio = tab_ptrs ? tab_ptrs[word(3)] : single;
        for (int32_t i0 = bnd[0]; i0 < bnd[4]; i0 += 64) {
            const int32_t i = min(i0 + lane, bnd[4] - 1);
            const int2 p = pts[i];
            const int32_t pout = perm_local[i];
            const bool on = i0 + lane < bnd[4] && pout >= eio.tgt0;
            double* u = eio.u + (eio.sorted ? int64_t(i) : int64_t(pout - eio.tgt0));
            const double old = on ? *u : 0.0;
            const int32_t loc = (p.x & (side - 1)) + side * (p.y & (side - 1));
            const double v = bnd[4] - bnd[0] <= 32 ? far_rows<P, true>(word(0), word(1), bnd, i0, loc, leafT, U, sfar[wave])
                                                   : far_rows<P, false>(word(0), word(1), bnd, i0, loc, leafT, U, sfar[wave]);
            if (on) *u = old + v;
        }
    }
}

// phi from radius kNearRadius on (PhiFast), the table below it (offsets below R): in LDS, both built by every block.
template <int R>
struct FastTab {
    static_assert(R >= kNearRadius && R % 2 == 0, "R");
    static constexpr int kRows = R, kRow = R + 1;   // doubles a row of the near table (odd)
    double near[R * kRow];
};

struct FastCoef {
    double a[14], log[5];
};

template <class Tab>
__device__ inline void load_near_tab(Tab& t, const double* phi_oct_tab, int tid, int nt) {
    for (int i = tid; i < Tab::kRows * Tab::kRow; i += nt) {
        const int dy = i / Tab::kRow, dx = i - dy * Tab::kRow;
        const int hi = max(dx, dy), lo = min(dx, dy);
        t.near[i] = phi_oct_tab[hi * (hi + 1) / 2 + lo];
    }
}

// uniform loads of the coefficients (scalar registers)
__device__ inline FastCoef fast_coef(const PhiFast* fast) {
    const cptr<double> p = as_const(reinterpret_cast<const double*>(fast));
    FastCoef c;
    #pragma unroll
    for (int k = 0; k < 14; ++k) c.a[k] = p[k];
    #pragma unroll
    for (int k = 0; k < 5; ++k) c.log[k] = p[14 + k];
    return c;
}

// an unsigned integer below 2^32 as a double plus 2^52 (differences of two are exact): no conversion
__device__ inline double biased(uint32_t v) { return __builtin_bit_cast(double, int2_t{int(v), 0x43300000}); }

// lead + the terms in 1 / r^2: z and v (see FarPhi) of r2, s = dx dy, lead = -(1/4pi) log(1/v) - C/2pi
// (and the exponent's share), ir2 = 1 / r2
__device__ inline double phi_terms(double z, double lead, double ir2, double s, const FastCoef& c) {
    double p = c.log[4];
    #pragma unroll
    for (int k = 3; k >= 0; --k) p = fma(p, z, c.log[k]);
    const double q = s * ir2, w = q * q;
    const double t1 = fma(c.a[1], w, c.a[0]);
    const double t2 = fma(fma(c.a[4], w, c.a[3]), w, c.a[2]);
    const double t3 = fma(fma(fma(c.a[8], w, c.a[7]), w, c.a[6]), w, c.a[5]);
    const double t4 = fma(fma(fma(fma(c.a[13], w, c.a[12]), w, c.a[11]), w, c.a[10]), w, c.a[9]);
    const double b = fma(fma(fma(t4, ir2, t3), ir2, t2), ir2, t1);
    return fma(b, ir2, fma(p, z, lead));
}

// phi at an offset below 2^8 in both coordinates (dx, dy exact): r2 in [2^11, 2^17) after clamping
template <class Tab>
__device__ inline double phi_fast_oct(double dx, double dy, uint32_t adx, uint32_t ady, const Tab& t,
                                      const double2_t* oct, const FastCoef& c) {
    constexpr double kMin = double(kNearRadius) * kNearRadius;
    const double r2 = fma(dx, dx, dy * dy), r = fmax(r2, kMin);
    // entry by exponent (modulo 8: 11 is 2 above a multiple) and the mantissa's first eight bits
    const uint32_t hi = uint32_t(__builtin_bit_cast(int2_t, r).y);
    const double2_t e = oct[int((hi >> 12) & 2047u) - 512];
    const double z = fma(r, e.x, -1.0);
    const double ir2 = e.x * fma(-z, fma(-z, 1.0 - z, 1.0), 1.0);   // |z| <= 2^-9: to 2^-36
    double ph = phi_terms(z, e.y, ir2, dx * dy, c);
    if (r2 < kMin) ph = t.near[ady * Tab::kRow + adx];
    return ph;
}

// phi at any offset (coordinates below 2^31)
template <class Tab>
__device__ inline double phi_fast_any(double dx, double dy, uint32_t adx, uint32_t ady, const Tab& t,
                                      const double2_t* mant, const FastCoef& c) {
    constexpr double kMin = double(kNearRadius) * kNearRadius;
    constexpr double kLn2 = -0.69314718055994530942 / (4.0 * kPi);
    const double r2 = fma(dx, dx, dy * dy), r = fmax(r2, kMin);
    const int2_t w = __builtin_bit_cast(int2_t, r);
    const double2_t e = mant[(uint32_t(w.y) >> 12) & 255u];
    const double m = __builtin_bit_cast(double, int2_t{w.x, int((uint32_t(w.y) & 0xfffffu) | 0x3ff00000u)});
    const double z = fma(m, e.x, -1.0);
    const double ex = double(int(uint32_t(w.y) >> 20) - 1023);
    const double scale = __builtin_bit_cast(double, int2_t{0, int(0x7fe00000u - (uint32_t(w.y) & 0x7ff00000u))});
    const double ir2 = e.x * fma(-z, fma(-z, 1.0 - z, 1.0), 1.0) * scale;
    double ph = phi_terms(z, fma(ex, kLn2, e.y), ir2, dx * dy, c);
    if (r2 < kMin) ph = t.near[ady * Tab::kRow + adx];
    return ph;
}

__device__ inline double bperm_d(int from4, int2_t v) {
    return __builtin_bit_cast(double, int2_t{__builtin_amdgcn_ds_bpermute(from4, v.x), __builtin_amdgcn_ds_bpermute(from4, v.y)});
}

// Lane t's entry among the lanes' consecutive ranges for list position base + t, t < C: lane e holds
// range e's start `beg` (ranges e < ne, none empty), e0 counts ranges that start before some earlier base
// and is moved on past the chunk.  A bit per start in the chunk, counted up to the lane.
template <int C>
__device__ inline int chunk_entry(int32_t beg, int32_t ne, int32_t base, int& e0) {
    while (e0 < ne && __builtin_amdgcn_readlane(beg, e0) <= base) ++e0;
    const int before = e0;
    uint64_t starts = 0;
    while (e0 < ne) {
        const int32_t b = __builtin_amdgcn_readlane(beg, e0) - base;
        if (b >= C) break;
        starts |= 1ull << b;
        ++e0;
    }
    const int lane = int(threadIdx.x) & 63;
    const uint64_t upto = starts & (~0ull >> (63 - lane));
    return before + __popcll(upto) - 1;
}

// A chunk's cnt sources, one per lane, added up for the lanes' targets: slice s of S takes sources s,
// s + S, ..., two at a time (two chains of dependent instructions); first = 4 s, and
// term(4 lane, a) = a + the term of that lane's source
template <class T>
__device__ inline double chunk_sum(int cnt, int S, int first, T term) {
    double a0 = 0.0, a1 = 0.0;
    int k = 0;
    for (; k + S < cnt; k += 2 * S) {
        a0 = term(4 * k + first, a0);
        a1 = term(4 * (k + S) + first, a1);
    }
    if (k < cnt) a0 = term(4 * k + first, a0);
    return a0 + a1;
}

// Slice sl's share of L2P for a lane's target: rows tl of the operator, uh of the expansion
template <int P>
__device__ inline double far_share(const double* tl, const double* uh, int sl, int S) {
    const double2_t* t2 = reinterpret_cast<const double2_t*>(tl);
    const double2_t* u2 = reinterpret_cast<const double2_t*>(uh);
    double a = 0.0;
    for (int p = sl; p < P / 2; p += 4 * S) {
        double2_t t[4], u[4];
        #pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = min(p + k * S, P / 2 - 1);
            t[k] = t2[q];
            u[k] = u2[q];
        }
        #pragma unroll
        for (int k = 0; k < 4; ++k)
            if (p + k * S < P / 2) a = fma(t[k].y, u[k].y, fma(t[k].x, u[k].x, a));
    }
    return a;
}

// The sums of a leaf's chunks are kept in four parts, chunk i in part i % 4, added as (0 + 1) + (2 + 3),
// so that one wave, or four with a part each, come to the same result.  One wave turns the parts
// round: the next chunk's part is always the first.
struct Parts {
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    __device__ void add(double v) {
        const double t = a[0] + v;
        a[0] = a[1];
        a[1] = a[2];
        a[2] = a[3];
        a[3] = t;
    }
    __device__ double sum(int chunks) {
        for (int r = chunks & 3; r != 0 && r < 4; ++r) {   // to part 0 first again
            const double t = a[0];
            a[0] = a[1];
            a[1] = a[2];
            a[2] = a[3];
            a[3] = t;
        }
        return (a[0] + a[1]) + (a[2] + a[3]);
    }
};

// x of every lane of a 16-lane row summed over the lanes up to it
__device__ inline int32_t row_inclusive_scan(int32_t x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    return x;
}

// Work item k of a persistent block, whose waves draw the k in increasing order from a counter in LDS:
// runs of 64 items go to the XCDs in turn (as blocks do), a run's items to the XCD's blocks in turn.
// The weights of clustered inputs' leaves differ by two orders and a wave takes only about 30: dealt
// out to the waves in a fixed order they left the CUs idle for 45 % of k_near_wide (1152 -> 830 us).
__device__ inline int32_t xcd_item(int32_t k) {
    const int32_t i = int32_t(blockIdx.x >> 3) + k * int32_t(gridDim.x >> 3);
    return ((i >> 6) * 8 + int32_t(blockIdx.x & 7)) * 64 + (i & 63);
}

// The wave's next k (uniform)
__device__ inline int32_t draw(int32_t* counter) {
    int32_t k = 0;
    if ((threadIdx.x & 63) == 0) k = atomicAdd(counter, 1);
    return __builtin_amdgcn_readfirstlane(k);
}

// A wave's lanes for n targets (1 .. 64): S = 64 / n slices of n lanes each; lanes past the last slice
// repeat it and are left out of the sums
struct Slices {
    int S, sl, t, raw;   // slices (uniform); this lane's slice, target, and slice before clamping
};
// (i + 1/2) / n lies 1/128 or more off every integer
__device__ inline int slice_count(int n) { return uniform(int(64.5f * __builtin_amdgcn_rcpf(float(n)))); }
__device__ inline Slices slices(int n, int lane) {
    const float inv = __builtin_amdgcn_rcpf(float(n));
    Slices r;
    r.S = slice_count(n);
    r.raw = int((float(lane) + 0.5f) * inv);
    r.t = lane - r.raw * n;
    r.sl = min(r.raw, r.S - 1);
    return r;
}
// Sum over the slices, to the lanes of slice 0
__device__ inline double sum_slices(double a, int n, int S, int raw) {
    for (int o = 1; o < S; o <<= 1) {
        const double v = __shfl(a, ((int(threadIdx.x) & 63) + o * n) & 63, 64);
        if (raw + o < S) a += v;
    }
    return a;
}

// Leaf pass for leaf sides 64 and 128.  Such leaves are the sparse ones of widely spread or
// clustered inputs: a group (the up to four leaves of one parent) holds a few dozen targets and its
// 4 x 4 block of source leaves a few hundred sources.  A wave takes one group, leaf by leaf; its
// record and entries were loaded a group ahead.  The ranges near to the leaf are read as one list, 60
// sources at a time, one per lane, the next 60 in flight.  The leaf's n targets take n lanes each of
// S = 64 / n slices, and slice s takes every S-th source from its lane by shuffles (60 rounded up to a
// multiple of any such S is at most 64).  phi is computed (PhiFast, about 42 instructions): random
// 8-byte gathers from the 4.2-MB table bound the pass at half an L2 request per cycle and compute unit,
// 3e11 pairs/s.  2e6 points in 64 clusters: 1097 -> 695 us.
// SPLIT: a block of four waves per leaf, a part of the chunks (see Parts) in each, for plans of few
// leaves, where a wave would work through a group's pairs alone (kSplitLeaves).
// Each target's sum depends on its group alone.
constexpr int kWideWaves = 8, kWideChunk = 60, kSplitWaves = 4;
// What a wave takes, by the number of units (child positions of the groups): a quarter of a leaf up to
// kSplitLeaves, a leaf up to kWaveLeaves, and up to kWaveLeavesFull where the groups hold 9/4 leaves or more on
// average, otherwise a group.  Measured (quarter / leaf / group; gathers from the table, us), on uniform points and
// clusters: 784 units 13 / 40 / 261; 83, 1.9e3 32 / 38 / 80; 88, 1.5e4 77 / 61 / 96; 108, 9.8e4
// 419 / 179 / 219; 254, 5.2e5 - / 762 / 695; 1097; on curves, whose groups hold two leaves: 984 units
// 22 / 19 / 53; 26, 3.9e3 44 / 26 / 33; 27, 2.5e4 198 / 88 / 72; 87.
constexpr int64_t kSplitLeaves = 2048, kWaveLeaves = 8192, kWaveLeavesFull = 196608;
// The same for adaptive leaves, a quarter or a leaf per wave, by their number and by the sources of one (the mean
// length of its U and W lists): a list of one or two chunks leaves most of four waves idle.  Measured (quarter / leaf,
// us): 59 sources, 1,569 leaves 21 / 22, 3,063 27 / 20, 18,295 102 / 50; 94 to 112 sources, 2,742 leaves 41 / 60, 5,393
// 63 / 83, 10,912 92 / 77, 21,389 120 / 55; 230 sources, 2,329 leaves 65 / 133, 9,677 102 / 113, 29,032 257 / 224; 320 to
// 360 sources, 3,577 leaves 189 / 335, 10,508 426 / 530, 22,276 401 / 444.
static int32_t split_adaptive(double sources) { return sources < 90.0 ? 2048 : sources < 150.0 ? 5632 : 16384; }

template <int P, bool SPLIT>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kWideWaves), SPLIT ? 3 : 4) void k_near_wide(
    int32_t q0, int32_t q1, const NearGroup* groups, const int4* ents, int64_t side, const int2* pts, const double* fs,
    const int32_t* perm_local, const ExecPtrs* tab_ptrs, ExecPtrs single, const double* U, const double* leafT,
    const double* phi_oct_tab, const PhiFast* fast, int by_leaf) {
    constexpr int W = SPLIT ? kSplitWaves : kWideWaves;
    __shared__ FastTab<kNearRadius> tab;
    __shared__ double2_t oct[kFarOctEntries];
    __shared__ double part[SPLIT ? kSplitWaves + 1 : 1][64];
    __shared__ int32_t next;
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6, rl = tid & 15;
    // by_leaf: leaf unit & 3 of group unit >> 2
    int32_t unit = SPLIT ? int32_t(blockIdx.x) : xcd_item(wave);
    int32_t q = q0 + (by_leaf ? unit >> 2 : unit), rec = 0;
    int4 ent = make_int4(0, 0, 0, 0);
    auto fetch = [&](int32_t g) {   // word l of group g's record in lane l, entry l in lane l (of each row)
        if (g < q1) {
            rec = reinterpret_cast<const int32_t*>(groups)[size_t(g) * 16 + rl];
            ent = ents[size_t(g) * kNearEntries + rl];
        }
    };
    fetch(q);
    {
        const double2_t* src = reinterpret_cast<const double2_t*>(&fast->oct[0][0]);
        for (int i = tid; i < kFarOctEntries; i += 64 * W) oct[i] = src[i];
        if (tid == 0) next = kWideWaves;
        load_near_tab(tab, phi_oct_tab, tid, 64 * W);
    }
    __syncthreads();
    const FastCoef coef = fast_coef(fast);
    const int32_t sd = int32_t(side);
    while (q < q1) {
        const int32_t r = rec, mine = unit & 3;
        const int4 en = ent;
        auto word = [&](int k) -> int32_t { return __builtin_amdgcn_readlane(r, k); };   // of the NearGroup
        unit = SPLIT ? unit + int32_t(gridDim.x) : xcd_item(draw(&next));
        q = q0 + (by_leaf ? unit >> 2 : unit);
        fetch(q);
        asm volatile("" ::: "memory");   // the next group's loads go out here
        const int32_t leaf0 = word(0), nleaf = word(1), ne = word(2), cposs = word(11);
        const int32_t gx = (word(9) - 1) * sd, gy = (word(10) - 1) * sd;   // corner of the 4 x 4 leaves
        const bool far = word(12) != 0;
        const ExecPtrs eio = tab_ptrs ? tab_ptrs[word(3)] : single;
        for (int c = by_leaf ? mine : 0; c < (by_leaf ? min(mine + 1, nleaf) : nleaf); ++c) {
            const int32_t t0 = word(4 + c), t_end = word(5 + c);
            // the ranges near to leaf c to the first lanes, in order
            const bool on = lane < 16 && lane < ne && ((en.z >> ((cposs >> (2 * c)) & 3)) & 1);
            const uint32_t m = uint32_t(__ballot(on));
            const int nr = __popc(m), below = __popc(m & ((1u << rl) - 1u));
            const int to = lane < 16 ? 4 * (on ? below : nr + rl - below) : 4 * lane;
            const int32_t start = __builtin_amdgcn_ds_permute(to, en.x);
            const int32_t len = __builtin_amdgcn_ds_permute(to, on ? en.y - en.x : 0);
            const int32_t end = row_inclusive_scan(len), beg = end - len, shift = start - beg;
            const int32_t ns = __builtin_amdgcn_readlane(end, 15), chunks = (ns + kWideChunk - 1) / kWideChunk;
            for (int32_t p0 = t0; p0 < t_end; p0 += 64) {
                const int32_t n = min(t_end - p0, 64);
                const Slices z = slices(n, lane);
                const int2 pi = pts[p0 + z.t];
                int e0 = 0;
                int2 pn = make_int2(0, 0);
                double fn = 0.0;
                auto load = [&](int32_t i) {   // chunk i: its source of this lane
                    const int32_t base = i * kWideChunk;
                    const int e = 4 * chunk_entry<kWideChunk>(beg, nr, base, e0);
                    const int32_t k = min(base + min(lane, kWideChunk - 1), ns - 1) + __builtin_amdgcn_ds_bpermute(e, shift);
                    pn = pts[k];
                    fn = fs[k];
                };
                const int32_t i0 = SPLIT ? wave : 0, step = SPLIT ? kSplitWaves : 1;
                if (i0 < chunks) load(i0);
                const int32_t pout = perm_local[p0 + z.t];
                double fa = 0.0;
                if (far && (!SPLIT || wave == kSplitWaves - 1))
                    fa = far_share<P>(leafT + size_t((pi.x & (sd - 1)) + sd * (pi.y & (sd - 1))) * P,   // its cell of the leaf
                                      U + size_t(leaf0 + c) * P, z.sl, z.S);
                const uint32_t tx = uint32_t(pi.x - gx), ty = uint32_t(pi.y - gy);
                const double xd = biased(tx), yd = biased(ty);
                Parts parts;
                for (int32_t i = i0; i < chunks; i += step) {
                    const int cnt = min(kWideChunk, ns - i * kWideChunk);
                    const int w = int(uint32_t(pn.x - gx) | (uint32_t(pn.y - gy) << 16));
                    const int2_t f = __builtin_bit_cast(int2_t, lane < cnt ? fn : 0.0);   // slots past the last: zero loads
                    if (i + step < chunks) load(i + step);
                    const double v = chunk_sum(cnt, z.S, 4 * z.sl, [&](int from, double a) -> double {
                        const uint32_t b = uint32_t(__builtin_amdgcn_ds_bpermute(from, w));
                        const double fk = bperm_d(from, f);
                        const uint32_t sx = b & 0xffffu, sy = b >> 16;
                        return fma(phi_fast_oct(xd - biased(sx), yd - biased(sy), uint32_t(abs(int(tx) - int(sx))),
                                                uint32_t(abs(int(ty) - int(sy))), tab, oct, coef), fk, a);
                    });
                    if (SPLIT) parts.a[0] += v;
                    else parts.add(v);
                }
                double acc;
                if (SPLIT) {
                    part[wave][lane] = parts.a[0];
                    if (wave == kSplitWaves - 1) part[kSplitWaves][lane] = fa;
                    __syncthreads();
                    acc = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) + part[4][lane];
                    __syncthreads();
                } else {
                    acc = parts.sum(chunks) + fa;
                }
                acc = sum_slices(acc, n, z.S, z.raw);
                if ((!SPLIT || wave == 0) && z.raw == 0 && pout >= eio.tgt0)
                    eio.u[eio.sorted ? int64_t(p0 + z.t) : int64_t(pout - eio.tgt0)] = acc;
            }
        }
    }
}

// ---- adaptive tree passes ----------------------------------------------------------------

__device__ inline double readlane_d(double v, int k) {
    const int2_t w = __builtin_bit_cast(int2_t, v);
    return __builtin_bit_cast(double, int2_t{__builtin_amdgcn_readlane(w.x, k), __builtin_amdgcn_readlane(w.y, k)});
}

// Lower-left corner of box g in its instance's root coordinates (root side 2^D).
__device__ inline int2 box_corner(const uint64_t* box_key, const int8_t* box_lev, int32_t g, int D) {
    const uint64_t k = box_key[g];
    const int sh = D - int(box_lev[g]);
    return make_int2(int32_t(compact_bits(k)) << sh, int32_t(compact_bits(k >> 1)) << sh);
}

// P2L (X lists): one wave per box tau, lane p for skeleton point p of tau; the points of each
// leaf of X(tau) are read 64 at a time (one coalesced load per lane) and broadcast lane by
// lane, every skeleton lane adding phi(y_p - x_j) f_j.  The sum joins tau's incoming
// expansion, which M2L wrote before and L2L reads after (the incoming skeleton is the
// outgoing one, T_ifi = T_ofo^T).
__global__ __launch_bounds__(kBlock) void k_p2l(int32_t nx, const int32_t* xitems, AdaptiveLists L,
                                                const int32_t* box_pt0, const int32_t* box_pt1,
                                                const uint64_t* box_key, const int8_t* box_lev,
                                                const int32_t* box_inst, const InstInfo* inst, const OpsPtrs* ops,
                                                const int2* pts, const double* fs, double* U,
                                                const double* phi_oct_tab, const PhiFar* phi_far) {
    constexpr int P = kRankPad;
    const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
    const int32_t q = int32_t(blockIdx.x) * kWaves + wave;
    if (q >= nx) return;
    const int32_t tau = uniform(xitems[q]);
    const int32_t k_inst = uniform(box_inst[tau]);
    const int D = uniform(inst[k_inst].D), Lf = uniform(inst[k_inst].L), opi = uniform(inst[k_inst].ops);
    const int h = Lf - int(box_lev[tau]);
    const int rank = uniform(ops[opi].rank[h]);
    const int2 c = box_corner(box_key, box_lev, tau, D);
    const bool on = lane < rank;
    int2 y = c;
    if (on) {
        const int32_t* sk = ops[opi].skel + (size_t(h) * P + lane) * 2;
        y = make_int2(c.x + sk[0], c.y + sk[1]);
    }
    double acc = 0.0;
    const int32_t e0 = uniform(L.off[2][tau]), e1 = uniform(L.off[2][tau + 1]);
    for (int32_t e = e0; e < e1; ++e) {
        const int32_t sg = uniform(L.ent[2][e]);
        const int32_t j0 = uniform(box_pt0[sg]), j1 = uniform(box_pt1[sg]);
        for (int32_t base = j0; base < j1; base += 64) {
            const int32_t j = base + lane;
            const bool ok = j < j1;
            const int2 pj = ok ? pts[j] : make_int2(0, 0);
            const double fj = ok ? fs[j] : 0.0;
            const int m = min(64, j1 - base);
            for (int k = 0; k < m; ++k) {
                const int32_t xk = __builtin_amdgcn_readlane(pj.x, k), yk = __builtin_amdgcn_readlane(pj.y, k);
                const double fk = readlane_d(fj, k);
                acc += phi_oct(abs(y.x - xk), abs(y.y - yk), phi_oct_tab, phi_far) * fk;
            }
        }
    }
    if (on && e1 > e0) U[size_t(tau) * P + lane] += acc;
}

// Near field of the adaptive leaves (Section 8.2 step 5 on the adaptive tree), one wave per
// leaf: the sources are the points of the U-list leaves and, for the W-list boxes, their skeleton
// points carrying their outgoing expansions (M2P: phi(x_i - y_p) q_p).  Lane e holds entry e of a batch
// of 64 list entries (start and length; the next leaf's record and first entries are loaded a leaf
// ahead), and the batch's sources are read as one list, 60 at a time, one per lane, the next 60 in
// flight.  The n targets take n lanes each of S = 64 / n slices; slice s takes every S-th source from
// its lane by shuffles.  phi is computed as in k_near_wide, for any offset: 2e6 clustered points
// 1842 -> 960 us (gathers from the 4.2-MB table, and a bisection over the entries for every source,
// before).  A chunk whose sources are all near to all of a leaf of side up to 64 takes phi from a table
// instead, in LDS for sides up to 32, the first 67 KB of the octant table for 64 (a third of the
// instructions; uniform points, N_leaf 64: 300,000 in leaves of side 16 and 32 278 -> 142 us, of side 64
// 379 -> 239, of which the gathers alone took 239 before).  L2P runs at each point's finest box (its incoming expansion holds those of the adaptive
// leaf relayed by L2L), then the caller-order write.
// SPLIT: as in k_near_wide, four waves per leaf.
constexpr int kAdWaves = 8, kAdChunk = kWideChunk;
// CLOSE: with those tables, for plans with leaves of such sides (the smallest side is at most kCloseSide); without,
// the larger table in LDS and the test cost 1 % of an execute on clusters (35,000 points, leaves of side 128 and more,
// 250 -> 253 us).
constexpr int kCloseOffsets = 64, kMidOffsets = 128;   // of either table
constexpr int kCloseSide = 64;

template <int P, bool SPLIT, bool CLOSE>
__global__ __launch_bounds__(64 * (SPLIT ? kSplitWaves : kAdWaves), SPLIT ? 3 : 4) void k_near_adaptive(
    int32_t nitems, const AdLeaf* recs, AdaptiveLists L, const int32_t* box_pt0, const int32_t* box_pt1,
    const uint64_t* box_key, const int8_t* box_lev, const InstInfo* inst, const OpsPtrs* ops, const int2* pts,
    const double* fs, const double* Q, const int32_t* pt_box, const double* U, const int32_t* perm_local,
    const ExecPtrs* tab_ptrs, ExecPtrs single, const uint8_t* far_inst, const double* phi_oct_tab,
    const PhiFast* fast) {
    constexpr int W = SPLIT ? kSplitWaves : kAdWaves;
    __shared__ FastTab<CLOSE ? kCloseOffsets : kNearRadius> tab;
    __shared__ double2_t mant[kFarMantEntries];
    __shared__ double part[SPLIT ? kSplitWaves + 1 : 1][64];
    __shared__ int32_t next;
    const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
    static_assert(sizeof(AdLeaf) == 32, "8 words");
    int32_t q = SPLIT ? int32_t(blockIdx.x) : xcd_item(wave);
    int32_t q1 = SPLIT ? q + int32_t(gridDim.x) : xcd_item(kAdWaves + wave);
    // word l of leaf i's record in lane l
    auto record = [&](int32_t i) -> int32_t {
        return i < nitems ? reinterpret_cast<const int32_t*>(recs)[size_t(i) * 8 + (lane & 7)] : 0;
    };
    // box of list entry eb + lane of a leaf (U entries, then W entries)
    auto entry = [&](int32_t u0, int32_t nu, int32_t w0, int32_t nw, int32_t eb) -> int32_t {
        const int32_t e = eb + lane;
        return e < nu ? L.ent[0][u0 + e] : e < nu + nw ? L.ent[1][w0 + e - nu] : -1;
    };
    int32_t rec = record(q), rec1 = record(q1);
    {
        const double2_t* src = reinterpret_cast<const double2_t*>(&fast->mant[0][0]);
        for (int i = tid; i < kFarMantEntries; i += 64 * W) mant[i] = src[i];
        if (tid == 0) next = 2 * kAdWaves;
        load_near_tab(tab, phi_oct_tab, tid, 64 * W);
    }
    __syncthreads();
    const FastCoef coef = fast_coef(fast);
    auto word = [](int32_t r, int k) -> int32_t { return __builtin_amdgcn_readlane(r, k); };
    int32_t sg = q < nitems ? entry(word(rec, 2), word(rec, 3), word(rec, 4), word(rec, 5), 0) : -1;
    while (q < nitems) {
        const int32_t t0 = word(rec, 0), t_end = word(rec, 1), u0 = word(rec, 2), nu = word(rec, 3), w0 = word(rec, 4);
        const int32_t nw = word(rec, 5), k_inst = word(rec, 6), sh = word(rec, 7), ne = nu + nw;
        const int32_t sg0 = sg;   // the first batch of entries
        // the next leaf's entries and the record after it
        q = q1;
        q1 = SPLIT ? q1 + int32_t(gridDim.x) : xcd_item(draw(&next));
        rec = rec1;
        if (q < nitems) sg = entry(word(rec, 2), word(rec, 3), word(rec, 4), word(rec, 5), 0);
        rec1 = record(q1);
        asm volatile("" ::: "memory");   // these loads go out here
        const InstInfo& I = inst[k_inst];
        const int D = uniform(I.D), Lf = uniform(I.L);
        const OpsPtrs& O = ops[uniform(I.ops)];
        const int32_t side0 = int32_t(O.side);
        const bool far = far_inst[k_inst] != 0;
        const ExecPtrs eio = tab_ptrs ? tab_ptrs[k_inst] : single;
        for (int32_t i0 = t0; i0 < t_end; i0 += 64) {
            const int32_t n = min(t_end - i0, 64);
            const Slices z = slices(n, lane);
            const int32_t ii = i0 + z.t;
            const int2 pi = pts[ii];
            const int32_t pout = perm_local[ii];
            const double xd = biased(uint32_t(pi.x)), yd = biased(uint32_t(pi.y));   // root coordinates: not negative
            // leaves of side up to 64: the sources at most `reach` off every point of the leaf in both
            // coordinates are those with x - near_x and y - near_y in [0, near_w]
            const int32_t top = (1 << min(sh, 6)) - 1, reach = (sh <= 5 ? kCloseOffsets : kMidOffsets) - 1, near_w = 2 * reach - top;
            const int32_t near_x = ((uniform(pi.x) >> sh) << sh) + top - reach, near_y = ((uniform(pi.y) >> sh) << sh) + top - reach;
            Parts parts;
            int32_t done = 0;   // chunks of the batches before
            for (int32_t eb = 0; eb < ne; eb += 64) {
                // this lane's entry: U (first point, length) or W (box, rank, height, corner)
                const int32_t d = eb == 0 ? sg0 : entry(u0, nu, w0, nw, eb);
                const bool is_w = eb + lane >= nu;
                int32_t a = 0, len = 0, hh = -1;
                int2 cc = make_int2(0, 0);
                if (d >= 0) {
                    if (!is_w) {
                        a = box_pt0[d];
                        len = box_pt1[d] - a;
                    } else {
                        hh = Lf - int(box_lev[d]);
                        len = O.rank[hh];
                        a = d;
                        cc = box_corner(box_key, box_lev, d, D);
                    }
                }
                int32_t end = len;
                #pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int32_t v = __shfl_up(end, o, 64);
                    if (lane >= o) end += v;
                }
                const int32_t beg = end - len, total = __builtin_amdgcn_readlane(end, 63);
                const int32_t m = min(64, ne - eb), chunks = (total + kAdChunk - 1) / kAdChunk;
                int e0 = 0;
                int2 pn = make_int2(0, 0);
                double fn = 0.0;
                auto load = [&](int32_t i) {   // chunk i: its source of this lane
                    const int32_t base = i * kAdChunk;
                    const int e = 4 * chunk_entry<kAdChunk>(beg, m, base, e0);
                    const int32_t k = min(base + min(lane, kAdChunk - 1), total - 1) - __builtin_amdgcn_ds_bpermute(e, beg);
                    const int32_t ae = __builtin_amdgcn_ds_bpermute(e, a), he = __builtin_amdgcn_ds_bpermute(e, hh);
                    if (eb + 64 <= nu || __ballot(he >= 0) == 0) {   // U entries alone
                        pn = pts[ae + k];
                        fn = fs[ae + k];
                    } else {
                        const int2 c = make_int2(__builtin_amdgcn_ds_bpermute(e, cc.x), __builtin_amdgcn_ds_bpermute(e, cc.y));
                        if (he < 0) {
                            pn = pts[ae + k];
                            fn = fs[ae + k];
                        } else {
                            const int32_t* sk = O.skel + (size_t(he) * P + k) * 2;
                            pn = make_int2(c.x + sk[0], c.y + sk[1]);
                            fn = Q[size_t(ae) * P + k];
                        }
                    }
                };
                const int32_t c0 = SPLIT ? (wave - done) & 3 : 0, step = SPLIT ? kSplitWaves : 1;
                if (c0 < chunks) load(c0);
                for (int32_t i = c0; i < chunks; i += step) {
                    const int sx = pn.x, sy = pn.y;
                    const int cnt = min(kAdChunk, total - i * kAdChunk);
                    const int2_t sf = __builtin_bit_cast(int2_t, lane < cnt ? fn : 0.0);   // slots past the last: zero loads
                    if (i + step < chunks) load(i + step);
                    double v;
                    const bool close = CLOSE && sh <= 6 && __ballot(uint32_t(sx) - uint32_t(near_x) > uint32_t(near_w) ||
                                                           uint32_t(sy) - uint32_t(near_y) > uint32_t(near_w)) == 0;
                    if (close && sh <= 5)
                        v = chunk_sum(cnt, z.S, 4 * z.sl, [&](int from, double acc) -> double {
                            const int x = __builtin_amdgcn_ds_bpermute(from, sx), y = __builtin_amdgcn_ds_bpermute(from, sy);
                            const double fk = bperm_d(from, sf);
                            return fma(tab.near[abs(pi.y - y) * tab.kRow + abs(pi.x - x)], fk, acc);
                        });
                    else if (close)
                        v = chunk_sum(cnt, z.S, 4 * z.sl, [&](int from, double acc) -> double {
                            const int x = __builtin_amdgcn_ds_bpermute(from, sx), y = __builtin_amdgcn_ds_bpermute(from, sy);
                            const double fk = bperm_d(from, sf);
                            const int dx = abs(pi.x - x), dy = abs(pi.y - y), hi = max(dx, dy);
                            return fma(global(phi_oct_tab)[uint32_t(__mul24(hi, hi + 1)) / 2u + uint32_t(min(dx, dy))], fk, acc);
                        });
                    else
                        v = chunk_sum(cnt, z.S, 4 * z.sl, [&](int from, double acc) -> double {
                            const int x = __builtin_amdgcn_ds_bpermute(from, sx), y = __builtin_amdgcn_ds_bpermute(from, sy);
                            const double fk = bperm_d(from, sf);
                            return fma(phi_fast_any(xd - biased(uint32_t(x)), yd - biased(uint32_t(y)), uint32_t(abs(pi.x - x)),
                                                    uint32_t(abs(pi.y - y)), tab, mant, coef), fk, acc);
                        });
                    if (SPLIT) parts.a[0] += v;
                    else parts.add(v);
                }
                done += chunks;
            }
            double fa = 0.0;
            if (far && (!SPLIT || wave == kSplitWaves - 1))
                fa = far_share<P>(O.leafT + (int64_t(pi.x & (side0 - 1)) + int64_t(side0) * int64_t(pi.y & (side0 - 1))) * P,
                                  U + size_t(pt_box[ii]) * P, z.sl, z.S);
            double acc;
            if (SPLIT) {
                part[wave][lane] = parts.a[0];
                if (wave == kSplitWaves - 1) part[kSplitWaves][lane] = fa;
                __syncthreads();
                acc = ((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane])) + part[4][lane];
                __syncthreads();
            } else {
                acc = parts.sum(done) + fa;
            }
            acc = sum_slices(acc, n, z.S, z.raw);
            if ((!SPLIT || wave == 0) && z.raw == 0 && pout >= eio.tgt0)
                eio.u[eio.sorted ? int64_t(ii) : int64_t(pout - eio.tgt0)] = acc;
        }
    }
}

// Brute-force sum over all sources for blocks of 256 targets; sources staged through LDS.
__global__ __launch_bounds__(kBlock) void k_direct(int64_t nt, const int2* txy, int64_t ns, const int2* sxy,
                                                    const double* f, const double* phi_oct, const PhiFar* far,
                                                    double* u) {
    __shared__ int2 sp[kBlock];
    __shared__ double sf[kBlock];
    const int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    const bool valid = t < nt;
    const int2 pt = valid ? txy[t] : make_int2(0, 0);
    double acc = 0.0;
    for (int64_t j0 = 0; j0 < ns; j0 += kBlock) {
        const int64_t j = j0 + threadIdx.x;
        if (j < ns) {
            sp[threadIdx.x] = sxy[j];
            sf[threadIdx.x] = f[j];
        }
        __syncthreads();
        const int cnt = int(min<int64_t>(kBlock, ns - j0));
        for (int k = 0; k < cnt; ++k) {
            int64_t dx = int64_t(pt.x) - sp[k].x, dy = int64_t(pt.y) - sp[k].y;
            dx = dx < 0 ? -dx : dx;
            dy = dy < 0 ? -dy : dy;
            const int64_t hi = dx > dy ? dx : dy, lo = dx > dy ? dy : dx;
            double ph;
            if (hi <= kPhiDeviceRadius) ph = phi_oct[hi * (hi + 1) / 2 + lo];
            else ph = phi_expansion_dev(double(hi), double(lo), far);
            acc += ph * sf[k];
        }
        __syncthreads();
    }
    if (valid) u[t] = acc;
}

}  // namespace

hipError_t upload_dslots() {
    DSlots ds{};
    for (int c = 0; c < 4; ++c) {
        const int cx = c & 1, cy = c >> 1;
        int k = 0;
        for (int dy = -2 - cy; dy <= 3 - cy; ++dy)
            for (int dx = -2 - cx; dx <= 3 - cx; ++dx) {
                if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1) continue;
                ds.s[c][k++] = (dy + 3) * 7 + (dx + 3);
            }
    }
    // synchronous copy, then read back: the table steers every M2L product
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(c_dslot), &ds, sizeof(ds), 0, hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    DSlots back{};
    e = hipMemcpyFromSymbol(&back, HIP_SYMBOL(c_dslot), sizeof(back), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    for (int c = 0; c < 4; ++c)
        for (int k = 0; k < kNumInteractions; ++k)
            if (back.s[c][k] != ds.s[c][k]) return hipErrorInvalidValue;
    return hipSuccess;
}

// Per device: compute units and the LDS a block may use (the staged P2M is set up to use it).
struct P2mDevice {
    int cus = 0, lds = 0;
};

P2mDevice p2m_device() {
    static P2mDevice dev[64];
    static std::once_flag once[64];
    int d = 0;
    if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= 64) return P2mDevice{};
    std::call_once(once[d], [&] {
        int cus = 0, lds = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, d) != hipSuccess ||
            hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, d) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&k_p2m_lds<kRankPad, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) {
            (void)hipGetLastError();
            return;   // the unstaged kernel serves every side
        }
        dev[d] = P2mDevice{cus, lds};
    });
    return dev[d];
}

// blocks of `threads` for `waves` work items of a wave each, as many as fit on the device at once
static unsigned persistent_grid(const void* fn, int threads, int64_t waves) {
    const int64_t want = (waves + threads / 64 - 1) / (threads / 64);
    const int cus = p2m_device().cus;
    int per = 0;
    int64_t g = std::min<int64_t>(want, 8192);
    if (cus > 0 && hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, threads, 0) == hipSuccess && per > 0)
        g = std::min<int64_t>(want, int64_t(cus) * per);
    else
        (void)hipGetLastError();
    return unsigned(std::max<int64_t>(g, 1));
}

void launch_p2m(int32_t leaf0, int32_t leaf1, const int32_t* box_pt0, const int32_t* box_pt1, const uint64_t* box_key,
                int64_t side, const int32_t* pts, const ExecPtrs* tab, const ExecPtrs& single,
                const int32_t* perm_local, const int32_t* box_inst, double* fs, const double* leafT, double* Q,
                double avg_pts, int32_t max_leaf, hipStream_t st) {
    const int32_t nleaf = leaf1 - leaf0;
    if (nleaf <= 0) return;
    const int2* p2 = reinterpret_cast<const int2*>(pts);
    const size_t lds = size_t(side * side) * kRankPad * sizeof(double);
    const P2mDevice dv = p2m_device();
    const bool staged = dv.cus > 0 && lds <= size_t(dv.lds);
    const bool full = !staged && avg_pts > kP2mSparsePoints &&
                        (nleaf <= kP2mWideLeaves || avg_pts < kP2mUneven * double(max_leaf));
    if (nleaf <= kP2mWaveLeaves || full) {
        hipLaunchKernelGGL(k_p2m<kRankPad>, dim3(grid_for(nleaf, kWaves)), dim3(kBlock), 0, st, leaf0, leaf1, box_pt0,
                           box_pt1, box_key, side, p2, tab, single, perm_local, box_inst, fs, leafT, Q);
        return;
    }
    if (staged) {
        const int64_t per_block = (kP2mThreads / 64) * kP2mLeaves;
        const int64_t grid = std::min<int64_t>((int64_t(nleaf) + per_block - 1) / per_block, dv.cus);
        hipLaunchKernelGGL((k_p2m_lds<kRankPad, true>), dim3(unsigned(grid)), dim3(kP2mThreads), lds, st, leaf0, leaf1,
                           box_pt0, box_pt1, side, p2, tab, single, perm_local, box_inst, fs, leafT, Q);
        return;
    }
    const unsigned grid = persistent_grid(reinterpret_cast<const void*>(&k_p2m_lds<kRankPad, false>), kP2mFreeThreads,
                                          (int64_t(nleaf) + kP2mLeaves - 1) / kP2mLeaves);
    hipLaunchKernelGGL((k_p2m_lds<kRankPad, false>), dim3(grid), dim3(kP2mFreeThreads), 0, st, leaf0, leaf1, box_pt0,
                       box_pt1, side, p2, tab, single, perm_local, box_inst, fs, leafT, Q);
}

void launch_m2m(const BoxTile* tiles, int32_t ntiles, const int32_t* box_child, const OpsPtrs* ops, double* Q,
                int32_t zrow, hipStream_t st) {
    if (ntiles <= 0) return;
    if (ntiles <= kFineM2mTiles) {
        hipLaunchKernelGGL(k_m2m_fine, dim3(unsigned(ntiles) * 12u), dim3(kBlock), 0, st, tiles, box_child, ops, Q,
                           zrow);
        return;
    }
    int64_t g = std::min<int64_t>(ntiles, 8192);
    g = std::max<int64_t>(8, (g + 7) / 8 * 8);
    hipLaunchKernelGGL(k_m2m, dim3(static_cast<unsigned>(g)), dim3(kBlock), 0, st, tiles, ntiles, box_child, ops, Q,
                       zrow);
}

void launch_l2l(const BoxTile* tiles, int32_t ntiles, const int32_t* box_list, const int32_t* box_parent,
                const OpsPtrs* ops, double* U, int32_t zrow, const int8_t* role, hipStream_t st) {
    if (ntiles <= 0) return;
    if (ntiles <= kFineL2lTiles) {
        hipLaunchKernelGGL(k_l2l_fine, dim3(unsigned(ntiles) * 12u), dim3(kBlock), 0, st, tiles, box_list, box_parent,
                           ops, U, zrow, role);
        return;
    }
    int64_t g = std::min<int64_t>(ntiles, 8192);
    g = std::max<int64_t>(8, (g + 7) / 8 * 8);
    hipLaunchKernelGGL(k_l2l, dim3(static_cast<unsigned>(g)), dim3(kBlock), 0, st, tiles, ntiles, box_list,
                       box_parent, ops, U, zrow, role);
}

void launch_m2m_sub(const SubTree* subs, int32_t n, int depth, const SubOps& A, const int32_t* box_child, double* Q,
                    int32_t zrow, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_m2m_sub, dim3(unsigned(n)), dim3(kSubThreads), 0, st, subs, depth, A, box_child, Q, zrow);
}

void launch_l2l_sub(const SubTree* subs, int32_t n, int depth, const SubOps& A, const int32_t* box_child, double* U,
                    const int8_t* role, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_l2l_sub, dim3(unsigned(n)), dim3(kSubThreads), 0, st, subs, depth, A, box_child, U, role);
}

// Tiles weighted by the share of the 27 slots that the 16-box kernels do not skip: those that any of 16 boxes has a
// source for.  Boxes with `children` children on average have (children / 4)^2 of the 27 each, but three children
// (clusters) already leave hardly a slot to no box of 16, and a curve's two leave about half of them.
static int32_t m2l_weighted(int32_t max_tiles, double children) {
    const double w = std::min(1.0, std::max(0.0, children) / 3.0);
    return int32_t(double(max_tiles) * w * w);
}

void launch_m2l(const BoxTile* tiles, const int32_t* ntiles_dev, int32_t max_tiles, double children,
                const int32_t* box_list, const int32_t* il27, const OpsPtrs* ops, const double* Q, int32_t zrow,
                double* U, hipStream_t st) {
    if (max_tiles <= 0) return;
    if (m2l_weighted(max_tiles, children) <= kFineM2lTiles) {
        hipLaunchKernelGGL(k_m2l_fine, dim3(unsigned(max_tiles) * (kM2LTile / kFineCols)), dim3(kFineThreads), 0, st,
                           tiles, ntiles_dev, box_list, il27, ops, Q, zrow, U);
        return;
    }
    const bool half = max_tiles <= kHalfM2lTiles;
    int64_t g = std::min<int64_t>(int64_t(max_tiles) * (half ? 2 : 1), 8192);
    g = std::max<int64_t>(8, (g + 7) / 8 * 8);
    hipLaunchKernelGGL(half ? k_m2l<1> : k_m2l<2>, dim3(static_cast<unsigned>(g)), dim3(kBlock), 0, st, tiles,
                       ntiles_dev, box_list, il27, ops, Q, zrow, U);
}

void launch_split_q(const double* Q, int32_t nrows, float* Qh, float* Ql, double* qs, hipStream_t st) {
    if (nrows <= 0) return;
    hipLaunchKernelGGL(k_split_q, dim3(grid_for(int64_t(nrows) * 64)), dim3(kBlock), 0, st, Q, nrows, Qh, Ql, qs);
}

void launch_m2l_mixed(const BoxTile* tiles, const int32_t* ntiles_dev, int32_t max_tiles, double children,
                      const int32_t* box_list, const int32_t* il27, const OpsPtrs* ops, const float* Qh, const float* Ql, const double* qs,
                      int32_t zrow, double* U, hipStream_t st) {
    if (max_tiles <= 0) return;
    if (m2l_weighted(max_tiles, children) <= kFineM2lMixedTiles) {
        hipLaunchKernelGGL(k_m2l_mixed_fine, dim3(unsigned(max_tiles) * (kM2LTile / kFineCols)), dim3(kFineThreads), 0, st, tiles,
                           ntiles_dev, box_list, il27, ops, Qh, Ql, qs, zrow, U);
        return;
    }
    int64_t g = std::min<int64_t>(max_tiles, 8192);
    g = std::max<int64_t>(8, (g + 7) / 8 * 8);
    hipLaunchKernelGGL(k_m2l_mixed, dim3(static_cast<unsigned>(g)), dim3(kBlock), 0, st, tiles, ntiles_dev, box_list,
                       il27, ops, Qh, Ql, qs, zrow, U);
}

void launch_split_q_bf16(const double* Q, int32_t nrows, uint16_t* Qb, double* qs, hipStream_t st) {
    if (nrows <= 0) return;
    hipLaunchKernelGGL(k_split_q_bf16, dim3(grid_for(int64_t(nrows) * 8)), dim3(kBlock), 0, st, Q, nrows, Qb, qs);
}

void launch_m2l_bf16(const BoxTile* tiles, const int32_t* ntiles_dev, int32_t max_tiles, double children,
                     const int32_t* box_list, const int32_t* il27, const OpsPtrs* ops, const uint16_t* Qb, const double* qs, int32_t zrow,
                     double* U, hipStream_t st) {
    if (max_tiles <= 0) return;
    if (m2l_weighted(max_tiles, children) <= kFineM2lBf16Tiles) {
        hipLaunchKernelGGL(k_m2l_bf16_fine, dim3(unsigned(max_tiles) * (kM2LTile / kFineCols)), dim3(kFineThreads), 0, st, tiles,
                           ntiles_dev, box_list, il27, ops, Qb, qs, zrow, U);
        return;
    }
    int64_t g = std::min<int64_t>(max_tiles, 8192);
    g = std::max<int64_t>(8, (g + 7) / 8 * 8);
    hipLaunchKernelGGL(k_m2l_bf16, dim3(static_cast<unsigned>(g)), dim3(kBf16Block), 0, st, tiles, ntiles_dev,
                       box_list, il27, ops, Qb, qs, zrow, U);
}

// the same in whole rounds of the XCDs, for xcd_item
static unsigned xcd_grid(const void* fn, int threads, int64_t waves) {
    return (persistent_grid(fn, threads, waves) + 7u) & ~7u;
}

void launch_near(int32_t q0, int32_t q1, const NearGroup* groups, const int4* ents, int64_t side, const int32_t* pts,
                 const uint32_t* pkey, const double* fs, const int32_t* perm_local, const ExecPtrs* tab,
                 const ExecPtrs& single, const double* U, const double* leafT, const double* phi_oct,
                 const PhiFast* fast, int32_t nleaf, int far_on, hipStream_t st) {
    if (q1 <= q0) return;
    if (!far_on && side > 32) throw std::logic_error("the kernel for wide leaves has no pass without L2P");
    const int2* p2 = reinterpret_cast<const int2*>(pts);
    if (side <= 16) {
        const int W = int(4 * side - 1);
        if (W * W > kNearTabMax) throw std::logic_error("near-field window table larger than its array");
        const unsigned g = persistent_grid(reinterpret_cast<const void*>(&k_near<kRankPad, kWindow>), kNearBlock, q1 - q0);
        hipLaunchKernelGGL((k_near<kRankPad, kWindow>), dim3(g), dim3(kNearBlock), 0, st, q0, q1, groups, ents, side, W,
                           p2, pkey, fs, perm_local, tab, single, U, leafT, phi_oct, far_on);
    } else if (side <= 32) {
        const int W = 64;   // rows: offsets of sides up to 32
        if (W * kQuadRow > kNearTabMax || 2 * side > W) throw std::logic_error("near-field quadrant table larger than its array");
        const unsigned g = persistent_grid(reinterpret_cast<const void*>(&k_near<kRankPad, kQuad>), kNearBlock, q1 - q0);
        hipLaunchKernelGGL((k_near<kRankPad, kQuad>), dim3(g), dim3(kNearBlock), 0, st, q0, q1, groups, ents, side, W, p2,
                           pkey, fs, perm_local, tab, single, U, leafT, phi_oct, far_on);
    } else {
        // near offsets are at most 2 side - 1, so that their squared length fits the octave table
        if (2 * side > 256) throw std::logic_error("leaf wider than the near-field table allows");
        const int64_t units = 4 * int64_t(q1 - q0);
        if (units <= kSplitLeaves) {
            const unsigned g = persistent_grid(reinterpret_cast<const void*>(&k_near_wide<kRankPad, true>),
                                               64 * kSplitWaves, units * kSplitWaves);
            hipLaunchKernelGGL((k_near_wide<kRankPad, true>), dim3(g), dim3(64 * kSplitWaves), 0, st, q0, q1, groups,
                               ents, side, p2, fs, perm_local, tab, single, U, leafT, phi_oct, fast, 1);
            return;
        }
        const int by_leaf = units <= kWaveLeaves || (units <= kWaveLeavesFull && 16 * int64_t(nleaf) >= 9 * units);
        const unsigned g = xcd_grid(reinterpret_cast<const void*>(&k_near_wide<kRankPad, false>), 64 * kWideWaves,
                                    by_leaf ? units : q1 - q0);
        hipLaunchKernelGGL((k_near_wide<kRankPad, false>), dim3(g), dim3(64 * kWideWaves), 0, st, q0, q1, groups, ents,
                           side, p2, fs, perm_local, tab, single, U, leafT, phi_oct, fast, by_leaf);
    }
}

void launch_l2p(int32_t q0, int32_t q1, const NearGroup* groups, int64_t side, const int32_t* pts,
                const int32_t* perm_local, const ExecPtrs* tab, const ExecPtrs& single, const double* U,
                const double* leafT, hipStream_t st) {
    if (q1 <= q0) return;
    const unsigned g = persistent_grid(reinterpret_cast<const void*>(&k_l2p<kRankPad>), kBlock, q1 - q0);
    hipLaunchKernelGGL(k_l2p<kRankPad>, dim3(g), dim3(kBlock), 0, st, q0, q1, groups, int32_t(side),
                       reinterpret_cast<const int2*>(pts), perm_local, tab, single, U, leafT);
}

size_t load_stats_scratch_bytes() { return size_t(kStatBlocks) * 3 * sizeof(double); }

void launch_load_stats(const double* f, int64_t n, double* scratch, double* out3, hipStream_t st) {
    hipLaunchKernelGGL(k_load_stats_part, dim3(kStatBlocks), dim3(kBlock), 0, st, f, n, scratch);
    hipLaunchKernelGGL(k_load_stats_final, dim3(1), dim3(kBlock), 0, st, scratch, out3);
}

void launch_phi_extend(double* oct, int r0, int r1, const PhiFar* far, hipStream_t st) {
    if (r1 <= r0) return;
    const int64_t n = int64_t(r1 + 1) * (r1 + 2) / 2 - int64_t(r0 + 1) * (r0 + 2) / 2;
    hipLaunchKernelGGL(k_phi_extend, dim3(grid_for(n)), dim3(kBlock), 0, st, oct, r0, r1, far);
}

void launch_p2l(int32_t nx, const int32_t* xitems, const AdaptiveLists& lists, const int32_t* box_pt0,
                const int32_t* box_pt1, const uint64_t* box_key, const int8_t* box_lev, const int32_t* box_inst,
                const InstInfo* inst, const OpsPtrs* ops, const int32_t* pts, const double* fs, double* U,
                const double* phi_oct, const PhiFar* phi_far, hipStream_t st) {
    if (nx <= 0) return;
    const unsigned g = unsigned((nx + kWaves - 1) / kWaves);
    hipLaunchKernelGGL(k_p2l, dim3(g), dim3(kBlock), 0, st, nx, xitems, lists, box_pt0, box_pt1, box_key, box_lev,
                       box_inst, inst, ops, reinterpret_cast<const int2*>(pts), fs, U, phi_oct, phi_far);
}

void launch_near_adaptive(int32_t nitems, const AdLeaf* recs, const AdaptiveLists& lists, const int32_t* box_pt0,
                          const int32_t* box_pt1, const uint64_t* box_key, const int8_t* box_lev,
                          const InstInfo* inst, const OpsPtrs* ops, const int32_t* pts,
                          const double* fs, const double* Q, const int32_t* pt_box, const double* U,
                          const int32_t* perm_local, const ExecPtrs* tab, const ExecPtrs& single,
                          const uint8_t* far_inst, const double* phi_oct, const PhiFast* fast, double sources, int64_t side,
                          hipStream_t st) {
    if (nitems <= 0) return;
    const int2* p2 = reinterpret_cast<const int2*>(pts);
    auto launch = [&](auto fn, unsigned g, int waves) {
        hipLaunchKernelGGL(fn, dim3(g), dim3(64 * waves), 0, st, nitems, recs, lists, box_pt0, box_pt1, box_key, box_lev,
                           inst, ops, p2, fs, Q, pt_box, U, perm_local, tab, single, far_inst, phi_oct, fast);
    };
    if (nitems <= split_adaptive(sources)) {
        auto fn = side <= kCloseSide ? &k_near_adaptive<kRankPad, true, true> : &k_near_adaptive<kRankPad, true, false>;
        launch(fn, persistent_grid(reinterpret_cast<const void*>(fn), 64 * kSplitWaves, int64_t(nitems) * kSplitWaves), kSplitWaves);
        return;
    }
    auto fn = side <= kCloseSide ? &k_near_adaptive<kRankPad, false, true> : &k_near_adaptive<kRankPad, false, false>;
    launch(fn, xcd_grid(reinterpret_cast<const void*>(fn), 64 * kAdWaves, nitems), kAdWaves);
}

void launch_direct(int64_t nt, const int32_t* txy, int64_t ns, const int32_t* sxy, const double* f,
                   const double* phi_oct, const PhiFar* far, double* u, hipStream_t st) {
    if (nt <= 0) return;
    hipLaunchKernelGGL(k_direct, dim3(grid_for(nt)), dim3(kBlock), 0, st, nt, reinterpret_cast<const int2*>(txy), ns,
                       reinterpret_cast<const int2*>(sxy), f, phi_oct, far, u);
}

}  // namespace lfmm
