// Ray tracing through the neighbour graph (Section 2.1, Fig. 2) and the
// device-wide scan that turns ray lengths into list offsets.
//
// From the current point a ray takes the forward neighbour (projection on the
// ray axis strictly beyond the current one) that lies closest to the axis,
// equal distances going to the smaller point id.  The
// geometry is IEEE FP64 in a fixed operation order, the fused multiply-adds
// written out and nothing else contracted (this file is compiled with
// -ffp-contract=off as well): Z = fma(R.z, d.z, fma(R.y, d.y, R.x d.x)),
// q = fma(-Z, d, R) per axis, D = fma(q.z, q.z, fma(q.y, q.y, q.x q.x)).  Every
// list is bit-identical to any other evaluation of the same rule.
//
// Data layout: each point has one row, a 32-byte head {x, y, z in FP64, id, the
// longest edge} followed by a 16-byte record per neighbour in ascending id:
// the edge to it in FP32 and where its own row lies.  Rows take whole units of
// 64 bytes, so the four lanes that walk a ray read a unit per load, the head
// and the first two records with the first, and a step reads one row (~280
// bytes on a Delaunay mesh) and nothing else; the rows of 50k points (~16 MB)
// stay in the Infinity Cache.
// The FP32 edges only rule candidates out: see k_trace.
#include "rt_internal.h"

#pragma clang fp contract(off)

namespace rt {

namespace {

constexpr int TRACE_BLOCK = 256;

// Rows are laid out in the order `lay` (a permutation of the points; NULL: point order):
// the row of point lay[q] is the q-th row in memory.  A row of `deg` neighbours takes
// row_units(deg) units of 64 bytes (its records start half a unit in), rounded up to whole
// units of 64 << sh.  A count that the low nb bits of a row code cannot hold is marked by all
// ones there; such a row has its degree in the code field of a blank first record.
__device__ inline bool row_counted(int64_t deg, int nb) { return (deg + 5) / 4 < ((int64_t)1 << nb) - 1; }
__device__ inline int64_t row_units(int64_t deg, int nb) { return (deg + (row_counted(deg, nb) ? 5 : 6)) / 4; }

__global__ __launch_bounds__(256) void k_layout_units(const int64_t* __restrict__ off, const int32_t* __restrict__ lay,
                                                       int64_t P, int sh, int nb, int32_t* __restrict__ units) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= P) return;
    const int64_t p = lay ? (int64_t)lay[q] : q;
    units[q] = (int32_t)((row_units(off[p + 1] - off[p], nb) + (1 << sh) - 1) >> sh);
}

// A record that no ray can take (NaN edge).
__device__ inline RowRec blank_rec(uint32_t code = 0) { return RowRec{NAN, 0.f, 0.f, code}; }

// The table starts with ROW_BLANK units of such records: what a lane of the walk reads in
// place of a record past its row's end.
constexpr int ROW_BLANK = 8;

__global__ void k_blank_rows(RowRec* __restrict__ recs, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) recs[i] = blank_rec();
}

// code[lay[q]] = the q-th row's start (`first` + scanned units) above nb bits of its units
__global__ __launch_bounds__(256) void k_layout_codes(const int64_t* __restrict__ start, const int64_t* __restrict__ off,
                                                       const int32_t* __restrict__ lay, int64_t P, int nb,
                                                       int64_t first, uint32_t* __restrict__ code) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= P) return;
    const int64_t p = lay ? (int64_t)lay[q] : q;
    const int64_t deg = off[p + 1] - off[p];
    const uint32_t u = row_counted(deg, nb) ? (uint32_t)row_units(deg, nb) : (1u << nb) - 1;
    code[p] = ((uint32_t)(first + start[q]) << nb) | u;
}

// Row of point p, BUILD_LANES lanes per point, each record placed by its rank in ascending
// id, or in ascending key[id] when a key is given (equal keys in list order).  The walk
// relies on that order: equal distances go to the earlier record.  The row's last unit is
// filled up with blank records.  The model has been checked, so every index is in range.
// axial: the edges along an axis, in AXIAL_COUNTERS parts (additions to one address go through one by one:
// 507 557 leaves of an octree 1.53 ms with a single one, 0.29 with none).
constexpr int BUILD_LANES = 16;

__global__ __launch_bounds__(256) void k_build_rows(const double* __restrict__ pos, int64_t P,
                                                     const int64_t* __restrict__ off,
                                                     const int32_t* __restrict__ idx, const int32_t* __restrict__ key,
                                                     const RowTab t, char* __restrict__ recs,
                                                     unsigned long long* __restrict__ axial) {
    const int64_t p = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / BUILD_LANES;
    if (p >= P) return;  // whole groups leave together
    const int sub = threadIdx.x & (BUILD_LANES - 1);
    const int64_t a = off[p];
    const int n = (int)(off[p + 1] - a);
    char* row = recs + t.offset(t.code[p]);
    const bool counted = row_counted(n, t.nb);
    RowRec* rec = (RowRec*)(row + sizeof(RowHead)) + (counted ? 0 : 1);
    const double x = pos[3 * p], y = pos[3 * p + 1], z = pos[3 * p + 2];
    double longest = 0.0;
    int along = 0;  // edges along an axis
    bool sorted = true;  // a row given in order is placed as it is: a point may have every other as its neighbour
    for (int j = sub; j + 1 < n; j += BUILD_LANES) {
        const int32_t k = idx[a + j], l = idx[a + j + 1];
        sorted = sorted && (key ? key[k] <= key[l] : k <= l);
    }
    const uint64_t group = (((uint64_t)1 << BUILD_LANES) - 1) << (threadIdx.x & 63 & ~(BUILD_LANES - 1));
    sorted = (__builtin_amdgcn_ballot_w64(!sorted) & group) == 0;
    for (int j = sub; j < n; j += BUILD_LANES) {
        const int32_t k = idx[a + j];
        const int32_t kk = key ? key[k] : k;
        int rank = sorted ? j : 0;
        for (int i = 0; i < n && !sorted; ++i) {
            const int32_t o = idx[a + i];
            const int32_t ok = key ? key[o] : o;
            rank += (ok < kk) || (ok == kk && i < j);
        }
        const double ex = (pos[3 * (int64_t)k] - x) * t.scale, ey = (pos[3 * (int64_t)k + 1] - y) * t.scale,
                     ez = (pos[3 * (int64_t)k + 2] - z) * t.scale;
        rec[rank] = RowRec{(float)ex, (float)ey, (float)ez, t.code[k]};
        const double l = sqrt(ex * ex + ey * ey + ez * ez);
        longest = l > longest ? l : longest;
        along += (ex == 0.0) + (ey == 0.0) + (ez == 0.0) == 2;
    }
    const int filled = (int)(4 * row_units(n, t.nb)) - (counted ? 2 : 3);  // records that fit after rec[0]
    for (int j = n + sub; j < filled; j += BUILD_LANES) rec[j] = blank_rec();
#pragma unroll
    for (int o = BUILD_LANES / 2; o > 0; o >>= 1) {
        const double l = __shfl_xor(longest, o, BUILD_LANES);
        longest = l > longest ? l : longest;
        along += __shfl_xor(along, o, BUILD_LANES);
    }
    if (sub == 0) {
        if (along) atomicAdd(axial + (blockIdx.x & (AXIAL_COUNTERS - 1)) * AXIAL_STRIDE, (unsigned long long)along);
        // never below the longest edge
        *(RowHead*)row = RowHead{x, y, z, (int32_t)p, (float)(longest * 1.000001)};
        if (!counted) rec[-1] = blank_rec((uint32_t)n);
    }
}

__global__ __launch_bounds__(256) void k_check_off(const int64_t* __restrict__ off, const int32_t* __restrict__ idx,
                                                    const double* __restrict__ pos, int64_t P, int64_t E,
                                                    int32_t* __restrict__ bad,
                                                    unsigned long long* __restrict__ reach) {
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    // the largest |coordinate|, as bits (non-negative doubles order as integers), one atomic per wave
    double far = 0.0;
    if (p < P)
        for (int i = 0; i < 3; ++i) far = fmax(far, fabs(pos[3 * p + i]));
    for (int o = 32; o > 0; o >>= 1) far = fmax(far, __shfl_xor(far, o, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(reach, (unsigned long long)__builtin_bit_cast(uint64_t, far));
    if (p >= P) return;
    int64_t a = off[p], b = off[p + 1];
    if (a > b || a < 0 || b > E || (p == 0 && a != 0) || (p == P - 1 && b != E)) {
        atomicOr(bad, 2);
        return;
    }
    for (int64_t e = a; e < b; ++e) {
        if (idx[e] < 0 || idx[e] >= P) atomicOr(bad, 1);
        if (idx[e] == p) atomicOr(bad, 4);
    }
    // |x| <= 1e150 keeps every squared distance of the walk finite
    for (int i = 0; i < 3; ++i)
        if (!(fabs(pos[3 * p + i]) <= 1e150)) atomicOr(bad, 8);
}

// GL lanes (4, 8 or 16) walk one ray.  At every step lane s takes candidates s,
// s+GL, ... of the current point's row, their loads issued together (UW per
// pass), and weighs them in FP32; the group combines its lanes in log2(GL) DPP
// stages (mirror within the row for 16 lanes, mirror within the half-row for 8
// or 16, then swap pairs, then swap neighbours).
//
// The choice is the FP64 rule's.  With p = R_c - Z_c d the current point's
// offset from the axis and e the edge to candidate k, in real arithmetic
//     Z_k - Z_c = s = e.d,     (offset of k from the axis) = p + e - s d,
// so FP32 values of s and D = |p + e|^2 - s^2 come from the 16-byte record
// alone, p (and the recorded Z) anew from the head's FP64 position at every
// step.  With u = 2^-24, E the row's longest edge, A = |p|_1 + E and Rm =
// |Z_c| + |p|_1 (at least |R_c|): rounding of e, d, p and of the chains moves s
// by at most 5.2 u E and D by 19 u A^2, and the FP64 rule's own rounding moves
// Z_k - Z_c by at most 2^-50 (Rm + E) and D_k by 2^-48 A Rm.  Hence
//     tol_s = 8 u A + 2^-48 Rm,   tol_D = 10 A tol_s  (at least 64 u A^2 + 2^-45 A Rm)
// plus floors for underflow (2^-120 for FP32's; on meshes of less than ~1e-140
// also the FP64 rule's own, whose D may vanish: there it always decides), with
// 2^-40 Rm added to A for edges near the resolution of the positions; edges are
// scaled by a power of two so that every coordinate is below 1 where FP32's
// range calls for it.  So a candidate with s < -tol_s is not forward, one with
// s > tol_s is, and D orders two candidates when their FP32 values are more
// than tol_D apart.  When the candidate of least D among those with s >= -tol_s
// has s > tol_s and is ahead of the second by more than tol_D, it is the FP64
// rule's choice; otherwise (about one step in 10^4 on irregular points, one in
// 20 on an octree: edges across the ray that end near the axis, and ties) the
// group evaluates the rule itself in FP64 over those that are left (exact_step).
// The lists are those of the FP64 rule, bit for bit.
//
// What bounds it: the L1's data path and VALU issue side by side, both full:
// the path returns data in 0.98 of the cycles on the cloud below, 0.97 on the grid
// and 0.98 on the octree (TD busy), and each SIMD issues one VALU instruction per 4
// cycles (~170 per step of a wave's 16 rays, 17 per candidate in FP32; the rule in
// FP64 takes ~20).  95 VGPRs, 5 waves per SIMD; 6 waves spill and are 3% slower.
// Branch-free loads matter: lanes past their
// row's end read blank records, and whether a wave takes a fifth or sixth
// piece is a scalar branch; loads under exec masks made the compiler wait for
// some before it issued the rest (7.9 ms).  50 000-point cloud, 96 pairs,
// 2.6e8 steps: 5.6 ms (46e9 steps/s), against 9.4 ms with every candidate's
// FP64 record (32 bytes) read and weighed; 26-neighbour grid, 5.0e8 steps: 10.0
// ms against 16.4; 50 000 leaves of an octree, 4.1e8 steps: 10.8 against 15.1,
// and bare lists of 20 000 of them at 24 pairs 3.5 against 4.25 (17.4 and 10.1
// where any edge across the ray, however far its end, sent the group to a rule
// that read its row again).  Where nearly every step is undecided and few waves
// hide the rounds to other rows' heads, it loses: lists of 512 points of a cubic
// lattice 105 us against 91, walks at 16 lanes 10% longer.
//
// List entries are buffered across the group and written in blocks of RUNL =
// max(GL, 8) entries aligned to absolute list positions (ids 32 or 64 bytes, Z
// 64 or 128 bytes at addresses that are multiples of those sizes), so the lists
// reach memory as whole aligned segments.  Lane s holds entries s*EPL ..
// s*EPL + EPL - 1 of a block (EPL = RUNL / GL, one or two), in a ring of two
// blocks.  Every RUNL steps -- the same step for every group of the wave, so
// the stores are issued once per wave -- each group stores the last block it
// has completed (exactly one completes per RUNL steps); the first block of a
// list is masked below its start, and when the ray ends the group stores what
// is left (at most the two ring blocks).
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline double make_f64(uint32_t lo, uint32_t hi) {
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

enum TraceMode { TRACE_COUNT = 0, TRACE_WRITE = 1, TRACE_PADDED = 2 };


// Every source lane of these permutations lies in the reading lane's own group
// (groups of 4, 8 or 16 lanes move through the loop together), so no lane
// reads a disabled one and the bound-control value is never used.
template <int CTRL>
__device__ inline int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ inline double dpp_d(double v) {
    int2 p = __builtin_bit_cast(int2, v);
    p.x = dpp_i<CTRL>(p.x);
    p.y = dpp_i<CTRL>(p.y);
    return __builtin_bit_cast(double, p);
}

constexpr int DPP_ROW_MIRROR = 0x140;   // lane i <-> 15-i within each 16 lanes
constexpr int DPP_HALF_MIRROR = 0x141;  // lane i <-> 7-i within each 8 lanes
constexpr int DPP_LANE0 = 0x00;         // quad_perm [0,0,0,0]
constexpr int DPP_LANE1 = 0x55;         // quad_perm [1,1,1,1]
constexpr int DPP_SWAP1 = 0xB1;         // quad_perm [1,0,3,2]
constexpr int DPP_SWAP2 = 0x4E;         // quad_perm [2,3,0,1]

template <int CTRL, typename T>
__device__ inline T dpp_t(T v) {  // a 32-bit value of another lane
    return __builtin_bit_cast(T, dpp_i<CTRL>(__builtin_bit_cast(int, v)));
}

// Reductions over the GL lanes of a group, the result in every lane of it.
template <int GL, typename T, typename F>
__device__ inline T group_reduce(T v, F f) {
    if (GL == 16) v = f(v, dpp_t<DPP_ROW_MIRROR>(v));
    if (GL >= 8) v = f(v, dpp_t<DPP_HALF_MIRROR>(v));
    v = f(v, dpp_t<DPP_SWAP2>(v));
    return f(v, dpp_t<DPP_SWAP1>(v));
}

// The stepping rule in FP64 over the row (candidate positions from their own heads): the
// lexicographic minimum of (D, place in the row) over the forward candidates; false if
// there is none.
template <int CTRL>
__device__ inline void exact_stage(double& D, int& i, uint32_t& code) {
    const double Do = dpp_d<CTRL>(D);
    const int io = dpp_i<CTRL>(i);
    const uint32_t co = (uint32_t)dpp_i<CTRL>((int)code);
    const bool take = Do < D || (Do == D && io < i);
    D = take ? Do : D;
    i = take ? io : i;
    code = take ? co : code;
}

// What the FP32 filter knows of a step: the current point's offset from the axis, the direction, the
// bounds on an edge's projection and a squared distance.
struct Filter {
    float px, py, pz, fx, fy, fz, tol_s, tol_D;
    // a candidate's projection from the current point and squared distance from the axis
    __device__ void eval(const f32x4 q, float& s, float& D) const {
        const float tx = px + q.x, ty = py + q.y, tz = pz + q.z;
        s = __builtin_fmaf(q.z, fz, __builtin_fmaf(q.y, fy, q.x * fx));
        D = __builtin_fmaf(-s, s, __builtin_fmaf(tz, tz, __builtin_fmaf(ty, ty, tx * tx)));
    }
};

// The rule over the candidates that the filter leaves.  The whole wave waits for its undecided groups, so the
// row's records are not read again: rec holds those of the first pass (cols per lane), and only the heads of
// the candidates left, mostly one or two in a group, are loaded, a round for each that a lane has.
// least: the least D of those surely forward where it is known (else infinite).
template <int GL, int UW>
__device__ inline bool exact_step(const RowTab t, const char* row, const f32x4 (&rec)[UW], int cols, int pieces,
                                  int sub, const Filter flt, float least, double ox, double oy, double oz, double dx,
                                  double dy, double dz, double Zc, uint32_t& code) {
    double D = __builtin_inf();
    int best = INT32_MAX;
    uint32_t c = 0;
    auto weigh = [&](int i, uint32_t ck) {
        const RowHead* h = (const RowHead*)(t.recs + t.offset(ck));
        const double Rx = h->x - ox, Ry = h->y - oy, Rz = h->z - oz;
        const double Zk = __builtin_fma(Rz, dz, __builtin_fma(Ry, dy, Rx * dx));
        const double qx = __builtin_fma(-Zk, dx, Rx), qy = __builtin_fma(-Zk, dy, Ry), qz = __builtin_fma(-Zk, dz, Rz);
        const double Dk = __builtin_fma(qz, qz, __builtin_fma(qy, qy, qx * qx));
        if (Zk > Zc && Dk < D) {  // ascending places within the lane: the first of equal D stays
            D = Dk;
            best = i;
            c = ck;
        }
    };
    float fs, fD, fDk[UW], sure = __builtin_inff();
#pragma unroll
    for (int k = 0; k < UW; ++k)
        if (k < cols) {
            flt.eval(rec[k], fs, fD);
            fDk[k] = fs >= -flt.tol_s ? fD : NAN;
            sure = fs > flt.tol_s && fD < sure ? fD : sure;
        }
    if (!(least < __builtin_inff())) {
        for (int i = sub + UW * GL; i < pieces; i += GL) {
            flt.eval(*(const f32x4*)(row + (int64_t)i * 16), fs, fD);
            sure = fs > flt.tol_s && fD < sure ? fD : sure;
        }
        least = group_reduce<GL>(sure, [](float a, float o) { return o < a ? o : a; });
    }
    const float lim_D = least + flt.tol_D;
    uint32_t left = 0;
#pragma unroll
    for (int k = 0; k < UW; ++k)
        if (k < cols) left |= (fDk[k] <= lim_D ? 1u : 0u) << k;
    while (left) {
        const int k = __builtin_ctz(left);
        left &= left - 1;
        float ck = rec[0].w;
#pragma unroll
        for (int j = 1; j < UW; ++j) ck = j == k ? (float)rec[j].w : ck;
        weigh(sub + k * GL, __builtin_bit_cast(uint32_t, ck));
    }
    for (int i = sub + UW * GL; i < pieces; i += GL) {
        const f32x4 q = *(const f32x4*)(row + (int64_t)i * 16);
        flt.eval(q, fs, fD);
        if (fs >= -flt.tol_s && fD <= lim_D) weigh(i, __builtin_bit_cast(uint32_t, (float)q.w));
    }
    if (GL == 16) exact_stage<DPP_ROW_MIRROR>(D, best, c);
    if (GL >= 8) exact_stage<DPP_HALF_MIRROR>(D, best, c);
    exact_stage<DPP_SWAP2>(D, best, c);
    exact_stage<DPP_SWAP1>(D, best, c);
    code = c;
    return best != INT32_MAX;
}

// Work order.  Without `order`, ray L is slot L (origin-major), but with TILE > 1
// the origins are taken TILE at a time, direction-major among them: the rays of
// a wave then share their direction.  With `order`
// (a permutation of origin positions, spatially sorted) ray L is direction
// L / n_origins of origin order[L % n_origins]: concurrent waves walk nearby
// origins in the same direction and share most of the rows they read.  With
// `ray_order` (n_rays origin positions, from k_length_order) ray L is direction
// L / n_origins of origin ray_order[L]: the same windows of nearby origins,
// their rays taken in order of length.  Register bounds by lanes per ray: 8 lanes
// at 6 waves per SIMD, 16 at 7 (graded cloud of 30k points 1.90 -> 1.79 and 2.82
// -> 2.65 ms).  Blocks are renumbered so that each XCD
// (own L2) takes runs of 16 consecutive blocks, the XCDs' runs side by side
// (xcd_block, XCD_RUN_WALK).
template <int MODE, int GL, bool FAR, int TILE>
__global__ __launch_bounds__(TRACE_BLOCK, GL == 4 ? 5 : GL == 8 ? 6 : 7) void k_trace(
    const double* __restrict__ pos, const RowTab t, int64_t P, const int32_t* __restrict__ origins, int64_t n_origins,
    int64_t R, const double* __restrict__ dirs, int per_origin, int32_t* __restrict__ lens,
    const int64_t* __restrict__ ray_off, int32_t* __restrict__ ids, double* __restrict__ Zout, int64_t capacity,
    int32_t* __restrict__ err, const int32_t* __restrict__ order, const int32_t* __restrict__ ray_order, int n_xcd) {
    static_assert(GL == 4 || GL == 8 || GL == 16, "4, 8 or 16 lanes per ray");
    // 16-byte pieces of a row per lane per pass (4 lanes: 22 neighbours; 5 and 7 pieces 2% and
    // 40% slower), and those of them that nearly every row has
    constexpr int UW = GL == 4 ? 6 : 32 / GL, U0 = GL == 4 ? 3 : 1;
    static_assert((UW - 1) * GL * 16 + 16 <= ROW_BLANK * 64, "blank records");
    constexpr int RUNL = GL >= 8 ? GL : 8;                              // entries per stored block
    constexpr int EPL = RUNL / GL;                                      // entries per lane per block
    constexpr int RING = 2 * RUNL, RSTR = RING + 2;                     // the ring's entries, and its stride
    constexpr int RAYS = TRACE_BLOCK / GL;
    __shared__ __attribute__((aligned(16))) double ring_z[MODE == TRACE_COUNT ? 2 : RAYS * RSTR];
    __shared__ __attribute__((aligned(16))) int32_t ring_i[MODE == TRACE_COUNT ? 2 : RAYS * RSTR];
    const int sub = threadIdx.x & (GL - 1);
    double* const rz = ring_z + (MODE == TRACE_COUNT ? 0 : (threadIdx.x / GL) * RSTR);
    int32_t* const ri = ring_i + (MODE == TRACE_COUNT ? 0 : (threadIdx.x / GL) * RSTR);
    const int64_t two_r = 2 * R;
    const int64_t n_rays = n_origins * two_r;
    const int64_t nb = (n_rays * GL + blockDim.x - 1) / blockDim.x;  // logical blocks
    for (int64_t blk = xcd_block(blockIdx.x, gridDim.x, n_xcd, XCD_RUN_WALK); blk < nb; blk += gridDim.x) {
    const int64_t L = (blk * (int64_t)blockDim.x + threadIdx.x) / GL;
    if (L >= n_rays) continue;  // whole groups leave together
    int64_t oi, rr;
    if (ray_order) {
        rr = L / n_origins;
        oi = ray_order[L];
    } else if (order) {
        const int64_t dslot = L / n_origins;
        oi = order[L - dslot * n_origins];
        rr = dslot;
    } else {
        oi = L / two_r;
        rr = L - oi * two_r;
        if (TILE > 1) {
            const int64_t o0 = oi / TILE * TILE, j = L - o0 * two_r;
            const int64_t m = n_origins - o0 < TILE ? n_origins - o0 : TILE;
            rr = j / m;
            oi = o0 + (j - rr * m);
        }
    }
    const int64_t ray = oi * two_r + rr;
    const int64_t r = rr >> 1;
    const int64_t o = origins ? (int64_t)origins[oi] : oi;
    if (o < 0 || o >= P) {  // invalid origin id: empty ray, error latched
        if (sub == 0) {
            if (MODE != TRACE_WRITE) lens[ray] = 0;
            if (MODE != TRACE_COUNT) atomicOr(err, ERRBIT_ORIGIN);
        }
        continue;
    }
    const double* dv = dirs + 3 * ((per_origin ? oi * R : 0) + r);
    double dx = dv[0], dy = dv[1], dz = dv[2];
    if (rr & 1) {
        dx = -dx;
        dy = -dy;
        dz = -dz;
    }
    const double ox = pos[3 * o], oy = pos[3 * o + 1], oz = pos[3 * o + 2];
    int64_t base = 0;
    int32_t room = 0;
    if (MODE == TRACE_WRITE) {
        base = ray_off[ray];
        int64_t rm = ray_off[ray + 1] - base;
        if (base + rm > capacity) rm = capacity - base;
        room = (int32_t)(rm < 0 ? 0 : rm);
    } else if (MODE == TRACE_PADDED) {
        base = ray * capacity;  // capacity = slots per ray
        room = (int32_t)capacity;
    }
    const float fx = (float)dx, fy = (float)dy, fz = (float)dz;
    uint32_t code = t.code[o];
    int32_t n = 0;                                 // list entries so far
    int32_t slot = (int32_t)(base - 1) & (RING - 1);  // the current point's place in the ring
    // the group's entries of the block starting at position S; positions outside the list
    // (before base, from hi on) are left out
    auto store_block = [&](int64_t S, int64_t hi) {
        const int64_t q = S + sub * EPL;
        const int k = (int)q & (RING - 1);
        if (EPL > 1 && q >= base && q + EPL <= hi) {
            *(int2*)(ids + q) = *(const int2*)(ri + k);
            *(double2*)(Zout + q) = *(const double2*)(rz + k);
        } else {
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                if (q + e >= base && q + e < hi) {
                    ids[q + e] = ri[k + e];
                    Zout[q + e] = rz[k + e];
                }
        }
    };
    for (int32_t count = 0;; ++count) {
        const int32_t step = __builtin_amdgcn_readfirstlane(count);  // the same in every active lane
        // the row, UW pieces of 16 bytes a lane (past the row's end: blank records); the first
        // two pieces are the head
        const char* row = t.recs + (FAR ? t.offset(code) : (uint64_t)(uint32_t)t.offset(code));
        int pieces = 4 * t.units(code);
        if (__builtin_amdgcn_ballot_w64(t.more(code)))
            if (t.more(code)) pieces = (int)((((const RowRec*)row)[2].code + 6) / 4 * 4);
        const int lim = pieces - sub;
        const uint64_t at0 = (FAR ? t.offset(code) : (uint64_t)(uint32_t)t.offset(code)) + (uint32_t)sub * 16;
        f32x4 rec[UW];
        int cols = U0;  // pieces a lane of the wave's longest row
#pragma unroll
        for (int i = 0; i < UW; ++i) {
            const bool has = (GL == 4 && i == 0) || i * GL < lim;  // every row has four pieces
            if (i < U0 || __builtin_amdgcn_ballot_w64(has)) {
                const uint64_t at = has ? at0 : 0;
                rec[i] = *(const f32x4*)(t.recs + (FAR ? at : (uint64_t)(uint32_t)at) + i * GL * 16);
                if (i >= U0) cols = i + 1;
            }
        }
        cols = __builtin_amdgcn_readfirstlane(cols);
        // the head, from the group's first two lanes (one quad each) or loaded again
        const u32x4 w0 = __builtin_bit_cast(u32x4, rec[0]);
        u32x4 hxy, hzi;
        if (GL == 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                hxy[k] = (uint32_t)dpp_i<DPP_LANE0>((int)w0[k]);
                hzi[k] = (uint32_t)dpp_i<DPP_LANE1>((int)w0[k]);
            }
        } else {
            hxy = *(const u32x4*)row;
            hzi = *(const u32x4*)(row + 16);
        }
        if (sub < 2) rec[0].x = NAN;
        // the current point: its exact projection and offset from the axis
        const double Rx = make_f64(hxy[0], hxy[1]) - ox, Ry = make_f64(hxy[2], hxy[3]) - oy,
                     Rz = make_f64(hzi[0], hzi[1]) - oz;
        const double Z = __builtin_fma(Rz, dz, __builtin_fma(Ry, dy, Rx * dx));
        n = step;
        if (MODE != TRACE_COUNT) {  // record it (the origin's place, before the list, is never stored)
            if (sub == 0) {
                ri[slot] = (int32_t)hzi[2];
                rz[slot] = Z;
            }
            slot = (slot + 1) & (RING - 1);
            if (step > 0 && (step & (RUNL - 1)) == 0) {  // the step of the wave's stores: the last block completed
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const int64_t end = base + step;
                store_block((end & ~(int64_t)(RUNL - 1)) - RUNL, end < base + room ? end : base + room);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (step > room) break;  // past its slot
            }
        }
        if (step >= (int32_t)P) break;  // Z grows at every step, so no ray is longer
        double qx = __builtin_fma(-Z, dx, Rx), qy = __builtin_fma(-Z, dy, Ry), qz = __builtin_fma(-Z, dz, Rz), Zs = Z;
        if (t.scale != 1.0) {
            qx *= t.scale;
            qy *= t.scale;
            qz *= t.scale;
            Zs *= t.scale;
        }
        const float px = (float)qx, py = (float)qy, pz = (float)qz;
        const float E = __builtin_bit_cast(float, (uint32_t)hzi[3]);
        const float P1 = fabsf(px) + fabsf(py) + fabsf(pz);
        const float Rm = fabsf((float)Zs) + P1, A = __builtin_fmaf(Rm, 0x1p-40f, P1 + E);
        const float tol_s = __builtin_fmaf(A, 0x1p-21f, __builtin_fmaf(Rm, 0x1p-48f, t.floor_s));
        const float tol_D = __builtin_fmaf(10.f * A, tol_s, t.floor_D);
        const float inf = __builtin_inff();
        // the lane's two least D among the candidates that may be forward, the first's row code and projection
        float D1 = inf, D2 = inf, s1 = 0.f;
        uint32_t best = 0;
        auto weigh = [&](const f32x4 q) {
            const float tx = px + q.x, ty = py + q.y, tz = pz + q.z;
            const float s = __builtin_fmaf(q.z, fz, __builtin_fmaf(q.y, fy, q.x * fx));
            const float T = __builtin_fmaf(tz, tz, __builtin_fmaf(ty, ty, tx * tx));
            const float D = s >= -tol_s ? __builtin_fmaf(-s, s, T) : inf;
            D2 = __builtin_amdgcn_fmed3f(D1, D2, D);
            const bool first = D < D1;
            D1 = first ? D : D1;
            s1 = first ? s : s1;
            best = first ? __builtin_bit_cast(uint32_t, (float)q.w) : best;
        };
#pragma unroll
        for (int i = 0; i < UW; ++i)
            if (i < U0 || i < cols) weigh(rec[i]);
        if (__builtin_amdgcn_ballot_w64(UW * GL < lim))
            for (int i = UW * GL; i < lim; i += GL)  // rows longer than one pass
                weigh(*(const f32x4*)(row + (int64_t)(sub + i) * 16));
        const float least = group_reduce<GL>(D1, [](float a, float o) { return o < a ? o : a; });
        if (least == inf) break;  // none may be forward: the ray leaves the model
        const float lim_D = least + tol_D;
        // candidates that may be the rule's choice, and (above 16 bits) those of them not surely forward: one
        // that is surely forward is known to be it
        const bool mine = D1 <= lim_D;
        const int rivals = group_reduce<GL>((mine ? (s1 > tol_s ? 1 : 0x10001) : 0) + (D2 <= lim_D ? 2 : 0),
                                            [](int a, int o) { return a + o; });
        code = group_reduce<GL>(mine ? best : 0u, [](uint32_t a, uint32_t o) { return a > o ? a : o; });
        const Filter flt = {px, py, pz, fx, fy, fz, tol_s, tol_D};
        if (__builtin_expect(rivals != 1, 0) &&
            !exact_step<GL, UW>(t, row, rec, cols, pieces, sub, flt, rivals < 0x10000 ? least : inf, ox, oy, oz, dx, dy, dz, Z, code))
            break;
    }
    if (MODE != TRACE_COUNT) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // a ray longer than its slot is cut there; one shorter than its slot leaves entries
        // unwritten: the offsets do not match this walk
        if (sub == 0 && (n > room || (MODE == TRACE_WRITE && n < room))) atomicOr(err, ERRBIT_CAPACITY);
        // what is left: at most the two ring blocks after the last stored one
        const int64_t done = base + (n & ~(RUNL - 1));  // the list's end at the last stores
        int64_t S = n >= RUNL ? (done & ~(int64_t)(RUNL - 1)) : (base & ~(int64_t)(RUNL - 1));
        if (n > room) n = room;
        for (int k = 0; k < 2; ++k, S += RUNL)
            if (S < base + n) store_block(S, base + n);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (MODE != TRACE_WRITE && sub == 0) lens[ray] = n;
    }
}

// Padded slots (ray * cap) -> compacted lists at ray_off.  Eight lanes per ray.
__global__ __launch_bounds__(256) void k_compact(const int32_t* __restrict__ pids, const double* __restrict__ pZ,
                                                  int64_t cap, const int64_t* __restrict__ ray_off, int64_t n_rays,
                                                  int32_t* __restrict__ ids, double* __restrict__ Z) {
    const int sub = threadIdx.x & 7;
    const int64_t nb = (n_rays * 8 + blockDim.x - 1) / blockDim.x;
    for (int64_t blk = blockIdx.x; blk < nb; blk += gridDim.x) {
        const int64_t ray = (blk * (int64_t)blockDim.x + threadIdx.x) >> 3;
        if (ray >= n_rays) continue;
        const int64_t b = ray_off[ray], n = ray_off[ray + 1] - b;
        const int64_t src = ray * cap;
        for (int64_t j = sub; j < n && j < cap; j += 8) {
            ids[b + j] = pids[src + j];
            Z[b + j] = pZ[src + j];
        }
    }
}


// ---------------------------------------------------------------- scan
// Exclusive scan of int32 lengths into int64 offsets, off[n] = total.
// Pass 1: per-tile sums; pass 2: one block scans the tile sums; pass 3: each
// tile scans itself and adds its tile offset.
constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int64_t SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t* sh, int64_t* total) {
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int d = 1; d < SCAN_BLOCK; d <<= 1) {
        int64_t add = (t >= d) ? sh[t - d] : 0;
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    int64_t incl = sh[t];
    *total = sh[SCAN_BLOCK - 1];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_tiles(const int32_t* __restrict__ in, int64_t n,
                                                            int64_t* __restrict__ tile_sum) {
    __shared__ int64_t sh[SCAN_BLOCK];
    const int64_t t0 = blockIdx.x * SCAN_TILE;
    int64_t s = 0;
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = t0 + (int64_t)i * SCAN_BLOCK + threadIdx.x;
        if (k < n) s += in[k];
    }
    int64_t tot;
    block_exclusive_scan(s, sh, &tot);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_sums(int64_t* __restrict__ tile_sum, int64_t n_tiles,
                                                           int64_t* __restrict__ out, int64_t n) {
    __shared__ int64_t sh[SCAN_BLOCK];
    int64_t carry = 0;
    for (int64_t b = 0; b < n_tiles; b += SCAN_BLOCK) {
        int64_t k = b + threadIdx.x;
        int64_t v = k < n_tiles ? tile_sum[k] : 0;
        int64_t tot;
        int64_t ex = block_exclusive_scan(v, sh, &tot);
        if (k < n_tiles) tile_sum[k] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) out[n] = carry;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_apply(const int32_t* __restrict__ in, int64_t n,
                                                            const int64_t* __restrict__ tile_off,
                                                            int64_t* __restrict__ out) {
    __shared__ int64_t sh[SCAN_BLOCK];
    // each thread owns SCAN_ITEMS consecutive elements of the tile
    const int64_t t0 = blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = t0 + i;
        v[i] = k < n ? in[k] : 0;
        s += v[i];
    }
    int64_t tot;
    int64_t run = tile_off[blockIdx.x] + block_exclusive_scan(s, sh, &tot);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int64_t k = t0 + i;
        if (k < n) out[k] = run;
        run += v[i];
    }
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

inline int64_t blocks_for(int64_t n, int b) { return (n + b - 1) / b; }

}  // namespace

hipError_t launch_check_model(const rt_model* m, int32_t* bad, uint64_t* reach, hipStream_t s) {
    hipLaunchKernelGGL(k_check_off, dim3((unsigned)blocks_for(m->P, 256)), dim3(256), 0, s, m->off, m->idx, m->pos, m->P,
                       m->E, bad, (unsigned long long*)reach);
    return hipGetLastError();
}

static size_t al256(size_t v) { return (v + 255) / 256 * 256; }

// Row addresses are 32-bit codes: the start in units of 64 << sh bytes above nb bits for the
// number of units.  28 bits of start and units of 64 bytes reach 17 GB of rows, far beyond
// any model measured; larger models give up the four bits (every row holds its degree) and
// take units of 128 bytes, which reach every model the ABI accepts.
size_t plan_rows(RowTab& t, int64_t P, int64_t E, int layout) {
    const int64_t units = ROW_BLANK + 2 * P + E / 4;  // of 64 bytes, at most
    const bool wide = layout == ROWS_WIDE || units >= (int64_t)1 << 28;
    t.nb = wide ? 0 : 4;
    t.sh = wide ? 1 : 0;
    return (size_t)(units + (wide ? P : 0)) * 64;
}

size_t build_rows_workspace(int64_t P) {
    return AXIAL_BYTES + al256(sizeof(int32_t) * (size_t)P) + al256(sizeof(int64_t) * (size_t)(P + 1)) + al256(scan_workspace(P));
}

hipError_t launch_build_rows(const rt_model* m, const int32_t* key, const int32_t* lay, void* ws, hipStream_t s) {
    int32_t* units = (int32_t*)((char*)ws + AXIAL_BYTES);
    int64_t* start = (int64_t*)((char*)units + al256(sizeof(int32_t) * (size_t)m->P));
    void* scan_ws = (char*)start + al256(sizeof(int64_t) * (size_t)(m->P + 1));
    const unsigned g = (unsigned)blocks_for(m->P, 256);
    hipLaunchKernelGGL(k_layout_units, dim3(g), dim3(256), 0, s, m->off, lay, m->P, m->tab.sh, m->tab.nb,
                       units);
    hipError_t e = launch_scan(units, m->P, start, scan_ws, s);
    if (e == hipSuccess) e = launch_fill_i32((int32_t*)ws, AXIAL_BYTES / sizeof(int32_t), 0, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_layout_codes, dim3(g), dim3(256), 0, s, start, m->off, lay, m->P, m->tab.nb,
                       (int64_t)(ROW_BLANK >> m->tab.sh), m->codes);
    hipLaunchKernelGGL(k_blank_rows, dim3(1), dim3(ROW_BLANK * 4), 0, s, (RowRec*)m->recs, ROW_BLANK * 4);
    hipLaunchKernelGGL(k_build_rows, dim3((unsigned)blocks_for(m->P * BUILD_LANES, 256)), dim3(256), 0, s, m->pos, m->P,
                       m->off, m->idx, key, m->tab, m->recs, (unsigned long long*)ws);
    return hipGetLastError();
}

template <int MODE>
static hipError_t trace_launch(const rt_model* m, const int32_t* origins, int64_t n_origins, int64_t R,
                               const double* dirs, int per_origin, int32_t* lens, const int64_t* ray_off,
                               int32_t* ids, double* Z, int64_t capacity, const int32_t* order,
                               const int32_t* ray_order, int gl, hipStream_t s) {
    const int64_t n = n_origins * 2 * R;
    if (n == 0) return hipSuccess;
    if (gl != 8 && gl != 16) gl = 4;  // 0 and other values: the default, 4 lanes
    if (m->far) gl = 4;
    int32_t* ew = MODE == TRACE_COUNT ? nullptr : error_word();
    const dim3 grid(capped_blocks(blocks_for(n * gl, TRACE_BLOCK)));
#define RT_TRACE(GL_, FAR_, TILE_)                                                                                    \
    hipLaunchKernelGGL((k_trace<MODE, GL_, FAR_, TILE_>), grid, dim3(TRACE_BLOCK), 0, s, m->pos, m->tab, m->P, origins, \
                       n_origins, R, dirs, per_origin, lens, ray_off, ids, Z, capacity, ew, order, ray_order, num_xcds())
    // Bare lists over lattices: undecided steps depend on the direction first, so waves of 16 directions from
    // one origin meet one at almost every step (ms, tiles of 1 and 16 origins: face-connected cubes of 55k
    // points, 24 pairs 8.5 and 5.9, 26-neighbour grid 8.4 and 6.0, octree 4.2 and 3.5).  Irregular points have
    // next to none, and near an origin its own rays share rows (log-spaced wind 3.4 and 3.8, disc 36.6 and 39.6).
    if (m->far) RT_TRACE(4, true, 1);
    else if (gl == 16) RT_TRACE(16, false, 1);
    else if (gl == 8) RT_TRACE(8, false, 1);
    else if (m->lattice && !order && !ray_order && !per_origin) RT_TRACE(4, false, MODE == TRACE_PADDED ? 1 : 16);
    else RT_TRACE(4, false, 1);
#undef RT_TRACE
    return hipGetLastError();
}

hipError_t launch_trace_count(const rt_model* m, const int32_t* origins, int64_t n_origins, int64_t R,
                              const double* dirs, int per_origin, int32_t* lens, hipStream_t s,
                              const int32_t* order, int gl) {
    return trace_launch<TRACE_COUNT>(m, origins, n_origins, R, dirs, per_origin, lens, nullptr, nullptr, nullptr, 0,
                                     order, nullptr, gl, s);
}

hipError_t launch_trace_write(const rt_model* m, const int32_t* origins, int64_t n_origins, int64_t R,
                              const double* dirs, int per_origin, const int64_t* ray_off, int32_t* ids,
                              double* Z, int64_t capacity, hipStream_t s, const int32_t* order, int gl,
                              const int32_t* ray_order) {
    return trace_launch<TRACE_WRITE>(m, origins, n_origins, R, dirs, per_origin, nullptr, ray_off, ids, Z, capacity,
                                     order, ray_order, gl, s);
}

hipError_t launch_trace_padded(const rt_model* m, const int32_t* origins, int64_t n_origins, int64_t R,
                               const double* dirs, int per_origin, int32_t* lens, int32_t* pids, double* pZ,
                               int64_t cap, hipStream_t s, const int32_t* order, int gl) {
    return trace_launch<TRACE_PADDED>(m, origins, n_origins, R, dirs, per_origin, lens, nullptr, pids, pZ, cap, order,
                                      nullptr, gl, s);
}

// For every direction slot d, the windows of LEN_WINDOW consecutive positions
// of `order` re-sorted by the length of their ray d (ties keep the given order;
// a bitonic sort of 32-bit keys (length << 8 | position in window) in LDS).
// out[d * n_o + k] is an origin position.  Rays walked by one wave then end at
// nearly the same step instead of the wave running until its longest ray ends,
// while each window stays a compact group of nearby origins.
constexpr int LEN_WINDOW = 64;

__global__ __launch_bounds__(LEN_WINDOW) void k_length_order(const int32_t* __restrict__ lens,
                                                             const int32_t* __restrict__ order, int64_t n_o,
                                                             int64_t two_r, int32_t* __restrict__ out) {
    __shared__ uint32_t sk[LEN_WINDOW];
    __shared__ int32_t so[LEN_WINDOW];
    const int t = threadIdx.x;
    const int64_t n_win = (n_o + LEN_WINDOW - 1) / LEN_WINDOW;
    for (int64_t w = blockIdx.x; w < n_win * two_r; w += gridDim.x) {
        const int64_t d = w / n_win;
        const int64_t k = (w - d * n_win) * LEN_WINDOW + t;
        uint32_t key = 0xFFFFFFFFu;  // past the end: sorts last
        int32_t oi = 0;
        if (k < n_o) {
            oi = order[k];
            const int32_t len = lens[(int64_t)oi * two_r + d];
            const uint32_t lc = len <= 0 ? 0u : (len >= 0xFFFFFE ? 0xFFFFFEu : (uint32_t)len);
            key = (lc << 8) | (uint32_t)t;
        }
        sk[t] = key;
        so[t] = oi;
        __syncthreads();
        for (int size = 2; size <= LEN_WINDOW; size <<= 1)
            for (int j = size >> 1; j > 0; j >>= 1) {
                const int u = t ^ j;
                if (u > t) {
                    const uint32_t a = sk[t], b = sk[u];
                    if ((a > b) == ((t & size) == 0)) {
                        sk[t] = b;
                        sk[u] = a;
                        const int32_t x = so[t];
                        so[t] = so[u];
                        so[u] = x;
                    }
                }
                __syncthreads();
            }
        if (k < n_o) out[d * n_o + k] = so[t];
        __syncthreads();  // the next window reuses the tables
    }
}

hipError_t launch_length_order(const int32_t* lens, const int32_t* order, int64_t n_origins, int64_t R,
                               int32_t* out, hipStream_t s) {
    const int64_t n_win = (n_origins + LEN_WINDOW - 1) / LEN_WINDOW;
    if (n_win == 0 || R == 0) return hipSuccess;
    hipLaunchKernelGGL(k_length_order, dim3(capped_blocks(n_win * 2 * R)), dim3(LEN_WINDOW), 0, s, lens, order,
                       n_origins, 2 * R, out);
    return hipGetLastError();
}

hipError_t launch_compact(const int32_t* pids, const double* pZ, int64_t cap, const int64_t* ray_off, int64_t n_rays,
                          int32_t* ids, double* Z, hipStream_t s) {
    if (n_rays == 0) return hipSuccess;
    hipLaunchKernelGGL(k_compact, dim3(capped_blocks(blocks_for(n_rays * 8, 256))), dim3(256), 0, s, pids, pZ, cap, ray_off, n_rays,
                       ids, Z);
    return hipGetLastError();
}

size_t scan_workspace(int64_t n) {
    int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    return (size_t)(tiles > 0 ? tiles : 1) * sizeof(int64_t);
}

hipError_t launch_scan(const int32_t* lens, int64_t n, int64_t* off, void* ws, hipStream_t s) {
    int64_t tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    int64_t* tile_sum = (int64_t*)ws;
    if (tiles > 0)
        hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, lens, n, tile_sum);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(SCAN_BLOCK), 0, s, tile_sum, tiles, off, n);
    if (tiles > 0)
        hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)tiles), dim3(SCAN_BLOCK), 0, s, lens, n, tile_sum, off);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(capped_blocks(blocks_for(n, 256))), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

}  // namespace rt
