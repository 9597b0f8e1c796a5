// polymer.hip -- multicanonical single-monomer shift moves of many
// bead-spring homopolymers (gfx950).
//
// Model (arXiv:1312.2213, Eq. 7): Lennard-Jones between beads |i-j| >= 2,
// cut at r_c and shifted to zero there, plus FENE bonds
// -(K/2) R^2 ln(1 - ((r - r0)/R)^2) between neighbours along the chain.
// A sweep moves beads 0..N-1 in order; bead i of chain c in sweep g draws
// Philox(c, g, i, SWEEP): words 0..2 give the displacement
// ((w >> 8) 2^-24 - 1/2) * step per axis (float), word 3 the acceptance.
//
// Mapping: one chain per wavefront, lane j holds bead j (and for 64 < N <= 128
// also bead j + 64).  At the start of a sweep lane j computes bead j's
// proposal and the FENE energies of its new bonds (the backward one for both
// outcomes of the previous bead's move), and from them what each neighbour's
// move will change in its own bond.  Moves are then taken two at a time: every
// lane computes its pair terms new - old of both in FP64 (the bonded partners
// take the precomputed changes), and the three sums that the outcomes can
// ask for (the first move; the second after a rejection and after an
// acceptance of the first) are taken together by a fixed binary tree (lane k
// += lane k + s for s = 32, 16, ..., 1) built from lane swaps and DPP moves,
// so that each sum is the same number on every run.  The acceptance
// thresholds T[b][b'] of the three bin changes are one load from the B x B
// matrix.
//
// With the paper's move set (moves = 1) each sweep continues with a
// spherical rotation of every bead (an inner bead about the line through its
// neighbours, an end bead about a coordinate axis through its neighbour,
// both by the quaternion (tau, axis) with tau symmetric about zero: only +,
// -, *, / in FP64, so the proposal is bit-identical everywhere) and one
// double bridging (two bonds swapped for two new ones, the beads between
// renumbered in reverse by one lane permute); rotations go in pairs like
// shifts, the second planned for the likelier outcome of the first.
#include <utility>

#include "muca_internal.h"
#include "philox.h"

namespace muca {

struct PolyParams {
    double lj_eps4;     // 4 eps
    double sig2;        // sigma^2
    double rc2;         // r_c^2
    double lj_shift;    // 4 eps ((sigma/r_c)^12 - (sigma/r_c)^6)
    double fene_pref;   // (K/2) R^2, evaluated as ((0.5 K) R) R
    double fene_r0, fene_R;
    double x_lo, x_hi, scale; // bins: floor((E - x_lo) * scale) on [x_lo, x_hi)
};

// 4 eps ((sigma^2/r2)^6 - (sigma^2/r2)^3) - shift inside the cutoff.  The
// quotient is the correctly rounded one: Newton steps on the reciprocal, then
// the quotient corrected by its exact remainder.  The compiler's division
// scales its operands first, against exponents near the ends of the range; a
// squared distance of two floats is 0 or between 2^-298 and 2^258, and where
// sigma^2 takes the quotient itself to an end, the powers below are 0 or not
// finite either way.
//
// Two at once, step by step: one's latency covers the other's.
__device__ __forceinline__ void lj_energy2(const PolyParams &p, double ra, double rb, double &ua, double &ub)
{
    double ya = __builtin_amdgcn_rcp(ra), yb = __builtin_amdgcn_rcp(rb);
    double ea = __builtin_fma(-ra, ya, 1.0), eb = __builtin_fma(-rb, yb, 1.0);
    ya = __builtin_fma(ya, ea, ya), yb = __builtin_fma(yb, eb, yb);
    ea = __builtin_fma(-ra, ya, 1.0), eb = __builtin_fma(-rb, yb, 1.0);
    ya = __builtin_fma(ya, ea, ya), yb = __builtin_fma(yb, eb, yb);
    const double qa = p.sig2 * ya, qb = p.sig2 * yb;
    ea = __builtin_fma(-ra, qa, p.sig2), eb = __builtin_fma(-rb, qb, p.sig2);
    const double sa = __builtin_fma(ea, ya, qa), sb = __builtin_fma(eb, yb, qb);
    double ta = sa * sa, tb = sb * sb;
    ta = ta * sa, tb = tb * sb;
    ua = p.lj_eps4 * (ta * ta - ta) - p.lj_shift;
    ub = p.lj_eps4 * (tb * tb - tb) - p.lj_shift;
    ua = ra < p.rc2 ? ua : 0.0;
    ub = rb < p.rc2 ? ub : 0.0;
}

__device__ __forceinline__ double lj_energy(const PolyParams &p, double r2)
{
    double u, v;
    lj_energy2(p, r2, r2, u, v);
    return u;
}

// FENE energy; sets *broken when the bond leaves (r0 - R, r0 + R)
__device__ __forceinline__ double fene_energy(const PolyParams &p, double r2, bool *broken)
{
    const double r = __builtin_sqrt(r2);
    const double t = (r - p.fene_r0) / p.fene_R;
    const double arg = 1.0 - t * t;
    if (!(arg > 0.0)) {
        *broken = true;
        return 0.0;
    }
    return -p.fene_pref * log(arg);
}

__device__ __forceinline__ double dist2(float ax, float ay, float az, float bx, float by, float bz)
{
    const double dx = (double)ax - (double)bx;
    const double dy = (double)ay - (double)by;
    const double dz = (double)az - (double)bz;
    return dx * dx + dy * dy + dz * dz;
}

// The same squared distance with both positions already in FP64 (a float
// converts to double exactly).
__device__ __forceinline__ double dist2d(double ax, double ay, double az, double bx, double by, double bz)
{
    const double dx = ax - bx;
    const double dy = ay - by;
    const double dz = az - bz;
    return dx * dx + dy * dy + dz * dz;
}

// (x, y, z) = (nx, ny, nz) in the lanes of m; every lane of the wave is active.
// Each output is written before the next input is read: none may share a register.
__device__ __forceinline__ void set_bead(uint64_t m, double &x, double &y, double &z, double nx, double ny, double nz)
{
    asm volatile("s_mov_b64 exec, %3\n\t"
        "v_mov_b64 %0, %4\n\t"
        "v_mov_b64 %1, %5\n\t"
        "v_mov_b64 %2, %6\n\t"
        "s_mov_b64 exec, -1"
        : "+&v"(x), "+&v"(y), "+&v"(z)
        : "s"(m), "v"(nx), "v"(ny), "v"(nz));
}

__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ float readlane_f32(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Lane k receives lane k + S (S = 32, 16, ..., 1) for every lane k < S; the
// other lanes receive values that are never read.  S = 32 and 16 cross rows
// of 16 lanes: v_permlane32_swap / v_permlane16_swap (the second result holds
// rows 2-3 / odd rows moved down); S <= 8 stays inside a row: DPP row_shl.
template <int S>
__device__ __forceinline__ uint32_t from_lane_above_u32(uint32_t v)
{
    if constexpr (S == 32)
        return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    else if constexpr (S == 16)
        return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
    else
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + S, 0xF, 0xF, true); // row_shl:S
}

template <int S>
__device__ __forceinline__ double from_lane_above(double v)
{
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = from_lane_above_u32<S>((uint32_t)u);
    const uint32_t hi = from_lane_above_u32<S>((uint32_t)(u >> 32));
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// One level of the tree across rows (S = 32 or 16) in place: the swap moves
// rows 2-3 (S = 32) or the odd rows (S = 16) of its first operand into the
// second, whose own values are never read, and leaves the lanes below S of
// the first operand as they were; the sum is valid in the lanes below S.
template <int S>
__device__ __forceinline__ double tree_level_swap(double t)
{
    const uint64_t u = __double_as_longlong(t);
    uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    uint32_t junk_lo, junk_hi;
    asm("" : "=v"(junk_lo), "=v"(junk_hi));
    uint32_t plo, phi;
    if constexpr (S == 32) {
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, junk_lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, junk_hi, false, false);
        lo = rl[0], plo = rl[1], hi = rh[0], phi = rh[1];
    } else {
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, junk_lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, junk_hi, false, false);
        lo = rl[0], plo = rl[1], hi = rh[0], phi = rh[1];
    }
    return __longlong_as_double(((uint64_t)hi << 32) | lo) + __longlong_as_double(((uint64_t)phi << 32) | plo);
}

// Exchange between two registers: rows 2-3 of a with rows 0-1 of b (S = 32),
// or the odd rows of a with the even rows of b (S = 16); their sum after.
template <int S>
__device__ __forceinline__ double swap_sum(double a, double b)
{
    const uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
    uint32_t al, ah, bl, bh;
    if constexpr (S == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
        al = l[0], bl = l[1], ah = h[0], bh = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
        al = l[0], bl = l[1], ah = h[0], bh = h[1];
    }
    return __longlong_as_double(((uint64_t)ah << 32) | al) + __longlong_as_double(((uint64_t)bh << 32) | bl);
}

// The fixed summation tree over 64 slots (slot k += slot k + s for
// s = 32, 16, ..., 1) of three values at once: level 32 of a and b fills the two
// halves of one register, level 16 the four rows; the sums of a, b and c end
// in lanes 0, 32 and 16.
__device__ __forceinline__ double tree_sum3(double a, double b, double c)
{
    double t = swap_sum<16>(swap_sum<32>(a, b), tree_level_swap<32>(c));
    t = t + from_lane_above<8>(t);
    t = t + from_lane_above<4>(t);
    t = t + from_lane_above<2>(t);
    t = t + from_lane_above<1>(t);
    return t;
}

// v_cvt_i32_f64: truncates, saturates, and takes NaN to 0
__device__ __forceinline__ int cvt_i32(double v)
{
    int r;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ int32_t energy_bin(const PolyParams &p, double E, int32_t nb)
{
    if (!(E >= p.x_lo) || !(E < p.x_hi))
        return -1;
    const double f = floor((E - p.x_lo) * p.scale);
    if (f < 0.0 || f >= (double)nb)
        return -1;
    return (int32_t)f;
}

// Value of lane `src` of the wave (once per sweep).
__device__ __forceinline__ float from_lane(float v, int src)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src * 4, __float_as_int(v)));
}

__device__ __forceinline__ uint32_t from_lane_u32(uint32_t v, int src)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute(src * 4, (int)v);
}

__device__ __forceinline__ double from_lane_f64(double v, int src)
{
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = from_lane_u32((uint32_t)u, src), hi = from_lane_u32((uint32_t)(u >> 32), src);
    return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// Rotation parameter of a 24-bit word: u = (k - (2^23 - 1/2)) / 2^23 in
// (-1, 1), tau = u / (1 - |u|); the mirrored word gives -tau.
__device__ __forceinline__ double rot_tau(uint32_t w)
{
    const double u = ((double)(w >> 8) - 8388607.5) / 8388608.0;
    return u / (1.0 - __builtin_fabs(u));
}

// v' = R v for the quaternion (w, a) (not normalised): |q|^2 R applied to v,
// divided by |q|^2; every product and sum in the order written.
__device__ __forceinline__ void quat_rotate(double w, double x, double y, double z, double vx, double vy, double vz,
                                            double &ox, double &oy, double &oz)
{
    const double ww = w * w, xx = x * x, yy = y * y, zz = z * z;
    const double n2 = ((ww + xx) + yy) + zz;
    const double m00 = ((ww + xx) - yy) - zz, m11 = ((ww - xx) + yy) - zz, m22 = ((ww - xx) - yy) + zz;
    const double m01 = 2.0 * (x * y - w * z), m02 = 2.0 * (x * z + w * y);
    const double m10 = 2.0 * (x * y + w * z), m12 = 2.0 * (y * z - w * x);
    const double m20 = 2.0 * (x * z - w * y), m21 = 2.0 * (y * z + w * x);
    ox = ((m00 * vx + m01 * vy) + m02 * vz) / n2;
    oy = ((m10 * vx + m11 * vy) + m12 * vz) / n2;
    oz = ((m20 * vx + m21 * vy) + m22 * vz) / n2;
}

// Pair-term cache (CACHE): the Lennard-Jones energy of every pair (a, b),
// a < b, of the wave's chain at the current positions, in LDS at slot
// f(a) + b with f(a) = a N - a (a + 1) / 2 - a - 1 (the upper triangle row
// by row).  A value depends only on the two positions and the pair's
// squared distance is the same number whichever bead is the moving one, so
// a cached term equals a recomputed one bit for bit.
__host__ __device__ inline int pair_row(int a, int N) { return a * N - a * (a + 1) / 2 - a - 1; }
__host__ __device__ inline int pair_slots(int N) { return N * (N - 1) / 2; }

typedef __attribute__((address_space(3))) const double lds_f64;
typedef __attribute__((address_space(3))) double lds_f64_out;

// A bead as every lane reads it (one LDS broadcast instead of a lane read per
// word): its proposal while shifts run and, without the cache, where it is.
struct alignas(16) BeadRecord {
    double x, y, z;
    uint32_t w, pad; // acceptance word
};

// A planned rotation: where it puts the bead, its acceptance word (all ones:
// a bond breaks, nothing to try) and the energies of the bead's two new bonds
// (to the bead before it, to the one after).
struct alignas(16) RotateRecord {
    float x, y, z;
    uint32_t w;
    double f[2];
};

// Rotations are planned for kPlanBeads beads and up to kPlanRuns - 1 accepted
// ones before each of them (see the kernel).
constexpr int kPlanBeads = 16, kPlanRuns = 4;

__host__ __device__ inline size_t hist_bytes(int n_bins) { return (size_t)((n_bins + 3) & ~3) * 4u; }
// LDS of one chain: [pair terms, or where its beads are | records or plan].
__host__ __device__ inline size_t chain_cache_bytes(int N) { return (size_t)((pair_slots(N) + 2) & ~1) * 8u; }
__host__ __device__ inline size_t chain_lds(int N, bool cache, bool moves)
{
    const size_t beads = (size_t)N * sizeof(BeadRecord), plan = kPlanBeads * kPlanRuns * sizeof(RotateRecord);
    return (cache ? chain_cache_bytes(N) : beads) + (moves && beads < plan ? plan : beads);
}

__device__ __forceinline__ bool lane_bit(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// Bound by instruction issue and, with one wavefront per SIMD, by the latency
// of one serial chain of FP64 operations: squared distance, quotient, pair
// term, six-level tree sum, bin, threshold load, decision.  So what a sweep
// knows beforehand is taken out of the moves (proposals and words are one LDS
// broadcast, bond changes wait in the lanes that add them, lanes of a move
// are scalar masks shifted along the chain, cache addresses are stepped), and
// two moves share the chain: their pair terms overlap, and tree, bins,
// thresholds and decisions are paid once.  82 vector instructions a shift,
// the sweep's own shared out (counted at N = 40, 4096 chains: vector unit
// busy 77 % of the cycles), where single moves took 96 and lane reads, masks
// from comparisons and 64-bit addresses 142.  Moves/s, with those / single moves / pairs:
//   N = 40, 4096 chains, shifts    3.1e9 / 4.4e9 / 4.6e9    full set  1.5e9 / 2.5e9 / 2.6e9
//   N = 40,  512 chains, shifts    9.3e8 / 1.1e9 / 1.4e9
//   N = 80, 4096 chains, shifts    1.9e9 / 2.7e9 / 2.6e9    full set  1.15e9 / 1.8e9 / 1.9e9
//   N = 80,  512 chains                                     full set  4.3e8 / 6.3e8 / 6.8e8
//   N = 100, 512 chains, shifts    6.6e8 / 7.9e8 / 9.4e8
// (N = 80, 4096 chains, without the cache: 143 registers leave three
// wavefronts per SIMD, 121 left four; held to 128 it spills and gains nothing.)
//
// One chain per wavefront.  Lane j holds bead j and, with TWO (64 < N <= 128),
// bead j + 64 (register set 1).  A pair sum slot is lane j's term plus, with
// TWO, the term of bead j + 64.  MOVES: the paper's full move set (a
// separate variant, so the shift-only kernel carries none of its registers).
// CACHE: a shift or rotation reads the old pair term from the cache instead
// of recomputing it, and an accepted move writes the new ones; an accepted
// double bridging renumbers beads and refills the cache.
template <bool TWO, bool MOVES, bool CACHE>
__global__ __launch_bounds__(256) void polymer_sweeps(PolymerArgs a, PolyParams p)
{
    extern __shared__ __align__(16) uint32_t lhist[];
    __shared__ unsigned long long accepted; // by the workgroup's chains
    if (threadIdx.x == 0)
        accepted = 0ull;
    for (int i = threadIdx.x; i < a.n_bins; i += blockDim.x)
        lhist[i] = 0u;
    __syncthreads();

    constexpr int NS = TWO ? 2 : 1; // beads per lane
    constexpr int SLOTS = 64 * NS;  // bead slots per chain in memory
    const int j = (int)(threadIdx.x & 63u);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = (int)(blockIdx.x * (blockDim.x >> 6)) + wave;
    const int N = a.n_beads;
    float4 *pos = a.pos + (size_t)c * SLOTS;
    double *bond = a.bond + (size_t)c * SLOTS;
    double xd[NS], yd[NS], zd[NS]; // positions (each a float, exactly)
    double ub[NS];                 // energy of bond (bead, bead + 1)
    uint64_t valid[NS];            // lanes that hold a bead
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int bd = j + 64 * s;
        const float4 v = bd < N ? pos[bd] : make_float4(0.f, 0.f, 0.f, 0.f);
        xd[s] = v.x, yd[s] = v.y, zd[s] = v.z;
        ub[s] = bd < N - 1 ? bond[bd] : 0.0;
        const int n = N - 64 * s;
        valid[s] = n >= 64 ? ~0ull : (1ull << n) - 1ull;
    }
    double E = readlane_f64(a.energy[c], 0);
    int32_t b = __builtin_amdgcn_readfirstlane(a.bins[c]);
    const uint32_t chain = (uint32_t)(a.chain0 + c);
    const uint32_t B = (uint32_t)a.n_bins;
    const int up_l = (j + 1) & 63, dn_l = (j + 63) & 63;
    uint64_t nacc = 0u; // accepted moves of the recorded sweeps (wave-uniform)

    uint8_t *mine = (uint8_t *)lhist + hist_bytes(a.n_bins) + (size_t)wave * chain_lds(N, CACHE, MOVES);
    double *cache = (double *)mine + 1; // CACHE (pair_row(0) + 0 is slot -1: read, never used)
    BeadRecord *was = (BeadRecord *)mine, *rec = (BeadRecord *)(mine + (CACHE ? chain_cache_bytes(N) : (size_t)N * sizeof(BeadRecord)));
    // lanes of one wave exchange data through LDS, whose accesses from one
    // wave complete in order: the fence only keeps the compiler from moving
    // them
    auto lds_fence = [] { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); };
    auto readlane_bead = [&](int k, double &px, double &py, double &pz) {
        const bool h = TWO && k >= 64;
        px = readlane_f64(h ? xd[NS - 1] : xd[0], k & 63);
        py = readlane_f64(h ? yd[NS - 1] : yd[0], k & 63);
        pz = readlane_f64(h ? zd[NS - 1] : zd[0], k & 63);
    };
    auto bond_of = [&](int k) { return readlane_f64((TWO && k >= 64) ? ub[NS - 1] : ub[0], k & 63); };
    // every pair term at the current positions
    auto fill_cache = [&]() {
        for (int k = 0; k + 2 < N; ++k) {
            double kx, ky, kz;
            readlane_bead(k, kx, ky, kz);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int bd = j + 64 * s;
                if (bd >= k + 2 && bd < N)
                    cache[pair_row(k, N) + bd] = lj_energy(p, dist2d(xd[s], yd[s], zd[s], kx, ky, kz));
            }
        }
        lds_fence();
    };
    if constexpr (CACHE)
        fill_cache();

    uint32_t row_at = 4u * B * (uint32_t)b; // byte offset of the present bin's thresholds (below 2^28)

    // Where a pass over the beads is: bead i, its lane, the lanes of the beads
    // up to it, and the LDS address of each lane's pair term with it (row i
    // of the triangle in lanes behind it, the lane's own row before).
    struct Place {
        int i;
        uint64_t me[NS], upto[NS];
        uint32_t at[NS];
    };
    auto start = [&]() {
        Place q;
        q.i = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            q.me[s] = q.upto[s] = s == 0 ? 1ull : 0ull;
            // lanes without a bead follow the last one
            q.at[s] = (uint32_t)(uintptr_t)(lds_f64 *)cache + 8u * (uint32_t)(min(j + 64 * s, N - 1) - 1);
        }
        return q;
    };
    auto next_lane = [](const uint64_t (&m)[NS], uint64_t (&r)[NS]) {
        if constexpr (TWO)
            r[NS - 1] = (m[NS - 1] << 1) | (m[0] >> 63);
        r[0] = m[0] << 1;
    };
    auto after = [&](const Place &q) {
        Place r;
        r.i = q.i + 1;
        next_lane(q.me, r.me);
        const uint32_t step = 8u * (uint32_t)(N - q.i - 2); // pair_row(i + 1) - pair_row(i)
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            r.upto[s] = q.upto[s] | r.me[s];
            r.at[s] = q.at[s] + (lane_bit(q.upto[s]) ? 8u : step);
        }
        return r;
    };
    struct Move {
        double x, y, z;
        uint32_t w;
    };
    constexpr uint64_t kA = 1ull, kB1 = 1ull << 16, kB0 = 1ull << 32;
    // Two moves at once, A of bead qa.i, then B of the next bead (at qb).  The
    // two are bonded, so B's pair terms do not depend on A's outcome: only
    // the change of the bond between them does (ddn0 if A is rejected, ddn1 if
    // accepted), and B's start.  The terms, summed over the lanes with the
    // bond changes in the lanes of the bonded partners (dup: the bond to the
    // bead after, ddn: to the bead before), are three sums: A, B after a
    // rejection, B after an acceptance; bin, threshold and decision of all
    // three are taken together, in lanes 0, 32 and 16.  can: the lanes of
    // those that may be accepted (no bond breaks, there is a bead).  Accepted
    // moves change positions, cached terms, E and b; acc_a, acc_b: which.
    auto attempt2 = [&](const Place &qa, const Place &qb, uint64_t can, const Move &A, const double (&dup_a)[NS],
                        const double (&ddn_a)[NS], const Move &Bm, const double (&dup_b)[NS],
                        const double (&ddn0)[NS], const double (&ddn1)[NS], uint32_t &acc_a, uint32_t &acc_b) {
        uint64_t mc[NS], mz[NS], pa[NS], pb[NS]; // the lanes after B's and before A's; the pair terms of A, B
        next_lane(qb.me, mc);
        mz[0] = qa.me[0] >> 1;
        if constexpr (TWO) {
            mz[0] |= qa.me[NS - 1] << 63;
            mz[NS - 1] = qa.me[NS - 1] >> 1;
        }
        double old_a[NS], old_b[NS];
        if constexpr (CACHE) {
            // the reads first, their latency covered by the new terms
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                old_a[s] = *(lds_f64 *)(uintptr_t)qa.at[s];
                old_b[s] = *(lds_f64 *)(uintptr_t)qb.at[s];
            }
            __builtin_amdgcn_sched_barrier(0);
        } else {
            const BeadRecord wa = was[qa.i], wb = was[min(qb.i, N - 1)];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                lj_energy2(p, dist2d(xd[s], yd[s], zd[s], wa.x, wa.y, wa.z), dist2d(xd[s], yd[s], zd[s], wb.x, wb.y, wb.z),
                           old_a[s], old_b[s]);
            }
        }
        double ta = 0.0, tb0 = 0.0, tb1 = 0.0;
        double la[NS], lb[NS]; // the new pair terms
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            pa[s] = valid[s] & ~(mz[s] | qa.me[s] | qb.me[s]);
            pb[s] = valid[s] & ~(qa.me[s] | qb.me[s] | mc[s]);
            lj_energy2(p, dist2d(xd[s], yd[s], zd[s], A.x, A.y, A.z), dist2d(xd[s], yd[s], zd[s], Bm.x, Bm.y, Bm.z), la[s],
                       lb[s]);
            double ea = lane_bit(pa[s]) ? la[s] - old_a[s] : 0.0;
            ea = lane_bit(qb.me[s]) ? dup_a[s] : ea;
            ea = lane_bit(mz[s]) ? ddn_a[s] : ea;
            double eb = lane_bit(pb[s]) ? lb[s] - old_b[s] : 0.0;
            eb = lane_bit(mc[s]) ? dup_b[s] : eb;
            const double eb0 = lane_bit(qa.me[s]) ? ddn0[s] : eb, eb1 = lane_bit(qa.me[s]) ? ddn1[s] : eb;
            ta = s == 0 ? ea : ta + ea;
            tb0 = s == 0 ? eb0 : tb0 + eb0;
            tb1 = s == 0 ? eb1 : tb1 + eb1;
        }
        const double t = tree_sum3(ta, tb0, tb1);
        const double Ea = E + readlane_f64(t, 0);
        const double En = (lane_bit(kB1) ? Ea : E) + t;
        const uint32_t bn = (uint32_t)cvt_i32((En - p.x_lo) * p.scale);
        // (inside the range the quotient is not negative: truncation is floor)
        const uint64_t ok = can & __builtin_amdgcn_ballot_w64(En >= p.x_lo) & __builtin_amdgcn_ballot_w64(En < p.x_hi) &
                            __builtin_amdgcn_ballot_w64(bn < B);
        const uint32_t row1 = 4u * B * min((uint32_t)__builtin_amdgcn_readlane((int)bn, 0), B - 1u);
        const uint32_t w = lane_bit(kA) ? A.w : Bm.w;
        // (one load for all lanes: those without a move read the first entry)
        const uint32_t entry = lane_bit(ok) ? (lane_bit(kB1) ? row1 : row_at) + 4u * bn : 0u;
        const uint32_t T = *(const uint32_t *)((const uint8_t *)a.thresholds + entry);
        const uint64_t acc = ok & __builtin_amdgcn_ballot_w64(w < T);
        acc_a = (uint32_t)acc & 1u;
        acc_b = (acc_a ? (uint32_t)acc >> 16 : (uint32_t)(acc >> 32)) & 1u;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            set_bead(acc_a ? qa.me[s] : 0ull, xd[s], yd[s], zd[s], A.x, A.y, A.z);
            set_bead(acc_b ? qb.me[s] : 0ull, xd[s], yd[s], zd[s], Bm.x, Bm.y, Bm.z);
            if constexpr (CACHE) {
                if (lane_bit(acc_a ? pa[s] : 0ull))
                    *(lds_f64_out *)(uintptr_t)qa.at[s] = la[s];
                if (lane_bit(acc_b ? pb[s] : 0ull))
                    *(lds_f64_out *)(uintptr_t)qb.at[s] = lb[s];
            }
        }
        if constexpr (CACHE)
            lds_fence();
        const int from = (int)((acc_a ? 16u : 32u) * acc_b);
        const uint32_t any = acc_a | acc_b;
        const double Et = readlane_f64(En, from);
        const int32_t bt = __builtin_amdgcn_readlane((int)bn, from);
        E = any ? Et : E;
        b = any ? bt : b;
        row_at = 4u * B * (uint32_t)b;
    };

    int trend = 0; // of the rotations' outcomes
    for (int s_ = 0; s_ < a.n_sweeps; ++s_) {
        const uint32_t g = a.g0 + (uint32_t)s_;
        float pnx[NS], pny[NS], pnz[NS];
        // Each bead's proposal: no earlier move of the sweep changes the bead.
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const Words4 w = philox4x32_10(chain, g, (uint32_t)(j + 64 * s), kTagSweep, a.k0, a.k1);
            pnx[s] = (float)xd[s] + ((float)(w.w[0] >> 8) * 5.9604644775390625e-08f - 0.5f) * a.step;
            pny[s] = (float)yd[s] + ((float)(w.w[1] >> 8) * 5.9604644775390625e-08f - 0.5f) * a.step;
            pnz[s] = (float)zd[s] + ((float)(w.w[2] >> 8) * 5.9604644775390625e-08f - 0.5f) * a.step;
            if (j + 64 * s < N) {
                // accept iff min(word, 2^32 - 2) < T
                rec[j + 64 * s] = BeadRecord{pnx[s], pny[s], pnz[s], min(w.w[3], 0xFFFFFFFEu), 0u};
                if constexpr (!CACHE)
                    was[j + 64 * s] = BeadRecord{xd[s], yd[s], zd[s], 0u, 0u};
            }
        }
        lds_fence();
        // The new bond energies of each bead's move, all known now: bead + 1
        // has not moved when the bead moves, and bead - 1 sits either where
        // the sweep found it (its move rejected) or at its proposal
        // (accepted).  Bonds whose stretch leaves the FENE domain break the
        // move: bits of brk_f (forward), brk_r, brk_a (backward).
        double f_fwd[NS], f_rej[NS], f_acc[NS];
        uint64_t brk_f[NS], brk_r[NS], brk_a[NS];
        {
            float rx[NS], ry[NS], rz[NS], lx[NS], ly[NS], lz[NS], qx[NS], qy[NS], qz[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float x = (float)xd[s], y = (float)yd[s], z = (float)zd[s];
                rx[s] = from_lane(x, up_l), ry[s] = from_lane(y, up_l), rz[s] = from_lane(z, up_l);
                lx[s] = from_lane(x, dn_l), ly[s] = from_lane(y, dn_l), lz[s] = from_lane(z, dn_l);
                qx[s] = from_lane(pnx[s], dn_l), qy[s] = from_lane(pny[s], dn_l), qz[s] = from_lane(pnz[s], dn_l);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int bd = j + 64 * s;
                // bead + 1 is in the next lane of the same set, or lane 0 of the next set
                const int rs = (j == 63) ? s + 1 : s;
                // bead - 1 is in the previous lane of the same set, or lane 63 of the previous set
                const int ls = (j == 0) ? s - 1 : s;
                f_fwd[s] = f_rej[s] = f_acc[s] = 0.0;
                bool bf = false, br = false, ba = false;
                if (bd + 1 < N && rs < NS) {
                    const float ax = rs == s ? rx[s] : rx[NS - 1], ay = rs == s ? ry[s] : ry[NS - 1],
                                az = rs == s ? rz[s] : rz[NS - 1];
                    f_fwd[s] = fene_energy(p, dist2(ax, ay, az, pnx[s], pny[s], pnz[s]), &bf);
                }
                if (bd >= 1 && bd < N && ls >= 0) {
                    const float ax = ls == s ? lx[s] : lx[0], ay = ls == s ? ly[s] : ly[0], az = ls == s ? lz[s] : lz[0];
                    const float bx = ls == s ? qx[s] : qx[0], by = ls == s ? qy[s] : qy[0], bz = ls == s ? qz[s] : qz[0];
                    f_rej[s] = fene_energy(p, dist2(ax, ay, az, pnx[s], pny[s], pnz[s]), &br);
                    f_acc[s] = fene_energy(p, dist2(bx, by, bz, pnx[s], pny[s], pnz[s]), &ba);
                }
                brk_f[s] = __builtin_amdgcn_ballot_w64(bf);
                brk_r[s] = __builtin_amdgcn_ballot_w64(br);
                brk_a[s] = __builtin_amdgcn_ballot_w64(ba);
            }
        }
        // What a neighbour's move changes in this lane's terms: when bead - 1
        // moves (bond (bead - 1, bead): its new energy minus the present
        // one), and when bead + 1 moves (bond (bead, bead + 1), whose present
        // energy depends on this bead's own move).
        double dup[NS], ddn_r[NS], ddn_a[NS], next_r[NS], next_a[NS];
        {
            double fwd_from[NS], rej_from[NS], acc_from[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                fwd_from[s] = from_lane_f64(f_fwd[s] - ub[s], dn_l);
                rej_from[s] = from_lane_f64(f_rej[s], up_l);
                acc_from[s] = from_lane_f64(f_acc[s], up_l);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                dup[s] = (TWO && s == 1 && j == 0) ? fwd_from[0] : fwd_from[s];
                next_r[s] = (TWO && s == 0 && j == 63) ? rej_from[NS - 1] : rej_from[s];
                next_a[s] = (TWO && s == 0 && j == 63) ? acc_from[NS - 1] : acc_from[s];
                ddn_r[s] = next_r[s] - ub[s];
                ddn_a[s] = next_a[s] - f_fwd[s];
            }
        }
        uint64_t done[NS]; // accepted beads
#pragma unroll
        for (int s = 0; s < NS; ++s)
            done[s] = 0ull;
        uint32_t prev_acc = 0u;
        auto shift2 = [&](Place &q, const Move &A, const Move &Bm) {
            const Place qb = after(q);
            uint64_t brk = 0ull, brk0 = 0ull, brk1 = 0ull; // no forward bond at the last bead, no backward one at the first: bits clear
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                brk |= q.me[s] & (brk_f[s] | (prev_acc ? brk_a[s] : brk_r[s]));
                brk0 |= qb.me[s] & (brk_f[s] | brk_r[s] | ~valid[s]);
                brk1 |= qb.me[s] & (brk_f[s] | brk_a[s] | ~valid[s]);
            }
            uint32_t acc_a = 0u, acc_b = 0u;
            if (!brk || !brk0) {
                double ddn[NS];
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    ddn[s] = prev_acc ? ddn_a[s] : ddn_r[s];
                attempt2(q, qb, (brk ? 0ull : kA) | (brk0 ? 0ull : kB0) | (brk1 ? 0ull : kB1), A, dup, ddn, Bm, dup, ddn_r,
                         ddn_a, acc_a, acc_b);
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    done[s] |= (acc_a ? q.me[s] : 0ull) | (acc_b ? qb.me[s] : 0ull);
            }
            prev_acc = acc_b;
            q = after(qb);
        };
        auto move_of = [&](int k) {
            const BeadRecord &r = rec[min(k, N - 1)];
            return Move{r.x, r.y, r.z, r.w};
        };
        Place q = start();
        Move a0 = move_of(0), b0 = move_of(1);
        for (;;) { // two pairs a turn, each read while the other is under way
            const Move a1 = move_of(q.i + 2), b1 = move_of(q.i + 3);
            shift2(q, a0, b0);
            if (q.i >= N)
                break;
            a0 = move_of(q.i + 2), b0 = move_of(q.i + 3);
            shift2(q, a1, b1);
            if (q.i >= N)
                break;
        }
        if (a.record) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                nacc += (uint64_t)__builtin_popcountll(done[s]);
        }
        // the bonds as the accepted moves left them
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint64_t after = (done[s] >> 1) | (TWO && s == 0 ? done[NS - 1] << 63 : 0ull); // bead + 1 accepted
            const double own = lane_bit(done[s]) ? f_fwd[s] : ub[s];
            const double both = lane_bit(done[s]) ? next_a[s] : next_r[s];
            ub[s] = lane_bit(after) ? both : own;
        }
        if constexpr (MOVES) {
            // Spherical rotations, beads 0..N-1 in order.  A proposal needs
            // the bead, the next one (which has not moved yet) and the one
            // before it, which is where the phase found it if its own
            // rotation was rejected, and else where that put it.  So the
            // proposals and bond energies of the next 16 beads are planned
            // at once, two lanes per bead (one bond each): plan[0] for the
            // case that the bead before was rejected, plan[k] for exactly k
            // accepted before, whose proposals are those of plan[k - 1].  A
            // plan ends with its beads or with the first four accepted in a
            // row; the next one starts from the positions then.  Three of
            // four rotations are accepted in earnest: a plan serves about
            // eight moves, and its FP64 chain of divisions, square root and
            // logarithm, which each move had to itself, is paid once (N = 80,
            // 512 chains: 5.4e8 -> 6.3e8 moves/s, moves one at a time).  Six or eight runs serve
            // little more and cost LDS (N = 40, 4096 chains, four, six and
            // eight: 2.48e9, 2.19e9, 2.19e9; N = 80, 512 chains: 6.31e8,
            // 6.51e8, 6.26e8).
            if constexpr (!CACHE) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (j + 64 * s < N)
                        was[j + 64 * s] = BeadRecord{xd[s], yd[s], zd[s], 0u, 0u};
            }
            RotateRecord *plan = (RotateRecord *)rec;
            const int slot = (j >> 1) & (kPlanBeads - 1);
            const bool right = lane_bit(0xAAAAAAAAAAAAAAAAull); // odd lanes: the bond to the bead after
            q = start();
            while (q.i < N) {
                const int i = q.i;
                const int bd = i + slot;
                auto at = [&](int k, double &x, double &y, double &z) {
                    float fx = from_lane((float)xd[0], k & 63), fy = from_lane((float)yd[0], k & 63),
                          fz = from_lane((float)zd[0], k & 63);
                    if constexpr (TWO) {
                        const float hx = from_lane((float)xd[NS - 1], k & 63), hy = from_lane((float)yd[NS - 1], k & 63),
                                    hz = from_lane((float)zd[NS - 1], k & 63);
                        fx = k >= 64 ? hx : fx, fy = k >= 64 ? hy : fy, fz = k >= 64 ? hz : fz;
                    }
                    x = fx, y = fy, z = fz;
                };
                double xi, yi, zi, lx, ly, lz, rx, ry, rz;
                at(bd, xi, yi, zi);
                at(bd - 1, lx, ly, lz);
                at(bd + 1, rx, ry, rz);
                const Words4 w = philox4x32_10(chain, g, (uint32_t)bd, kTagRotate, a.k0, a.k1);
                const double tau = rot_tau(w.w[0]);
                const uint32_t axis = (uint32_t)(((uint64_t)w.w[1] * 3u) >> 32);
                const bool first = bd == 0, inner = bd > 0 && bd < N - 1;
                const bool upper = lane_bit(0xFFFFFFFF00000000ull);
                const int dn2 = (j + 62) & 63; // a lane of the bead before
                const bool bonded = right ? bd + 1 < N : bd > 0;
                // the proposals, run by run, in every lane pair of the bead;
                // of two runs the lower half of the wave keeps the first, the
                // upper half the second
                float px[kPlanRuns / 2], py[kPlanRuns / 2], pz[kPlanRuns / 2];
                double fx[kPlanRuns / 2], fy[kPlanRuns / 2], fz[kPlanRuns / 2]; // the bonded neighbour
#pragma unroll
                for (int k = 0; k < kPlanRuns; ++k) {
                    // an inner bead: about the line through both neighbours;
                    // an end bead: about a coordinate axis through its neighbour
                    const double ax = inner ? rx - lx : (axis == 0u ? 1.0 : 0.0);
                    const double ay = inner ? ry - ly : (axis == 1u ? 1.0 : 0.0);
                    const double az = inner ? rz - lz : (axis == 2u ? 1.0 : 0.0);
                    const double cx = first ? rx : lx, cy = first ? ry : ly, cz = first ? rz : lz;
                    double ox, oy, oz;
                    quat_rotate(tau, ax, ay, az, xi - cx, yi - cy, zi - cz, ox, oy, oz);
                    const float nx = (float)(cx + ox), ny = (float)(cy + oy), nz = (float)(cz + oz);
                    const bool keep = (k & 1) == 0 || upper;
                    const int m = k / 2;
                    px[m] = keep ? nx : px[m], py[m] = keep ? ny : py[m], pz[m] = keep ? nz : pz[m];
                    fx[m] = keep ? (right ? rx : lx) : fx[m];
                    fy[m] = keep ? (right ? ry : ly) : fy[m];
                    fz[m] = keep ? (right ? rz : lz) : fz[m];
                    if (k + 1 < kPlanRuns)
                        lx = from_lane(nx, dn2), ly = from_lane(ny, dn2), lz = from_lane(nz, dn2);
                }
                // the bonds of all runs together
                lds_fence();
#pragma unroll
                for (int m = 0; m < kPlanRuns / 2; ++m) {
                    bool broken = false;
                    const double f = fene_energy(p, dist2d(fx[m], fy[m], fz[m], px[m], py[m], pz[m]), &broken);
                    const int out = broken && bonded ? 1 : 0;
                    const int other = __builtin_amdgcn_update_dpp(0, out, 0xB1, 0xF, 0xF, true); // quad_perm 1 0 3 2
                    RotateRecord *r = plan + (2 * m + (upper ? 1 : 0)) * kPlanBeads + slot;
                    if (!right)
                        r->x = px[m], r->y = py[m], r->z = pz[m], r->w = (out | other) ? 0xFFFFFFFFu : min(w.w[3], 0xFFFFFFFEu);
                    r->f[right ? 1 : 0] = f;
                }
                lds_fence();
                const int end = min(i + kPlanBeads, N);
                int run = 0;
                // Rotations in pairs as well, B's the one planned for the
                // likelier outcome of A: after the other outcome B is left
                // for the next turn.
                while (q.i < end && run < kPlanRuns) {
                    const RotateRecord ra = plan[run * kPlanBeads + q.i - i];
                    const bool guess = trend >= 0 && run + 1 < kPlanRuns;
                    const bool two = q.i + 1 < end;
                    const RotateRecord rb = plan[(guess ? run + 1 : 0) * kPlanBeads + (two ? q.i + 1 - i : 0)];
                    const Place qb = after(q);
                    const bool can_a = __builtin_amdgcn_readfirstlane((int)ra.w) != -1;
                    const bool can_b = two && __builtin_amdgcn_readfirstlane((int)rb.w) != -1;
                    uint32_t acc_a = 0u, acc_b = 0u;
                    if (can_a || (can_b && !guess)) {
                        const bool last_a = q.i + 1 == N, last_b = q.i + 2 >= N;
                        const double ua = bond_of(q.i), ub_ = bond_of(min(q.i + 1, N - 1));
                        double dup_a[NS], ddn_a2[NS], dup_b[NS], ddn0[NS], ddn1[NS];
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            dup_a[s] = last_a ? 0.0 : ra.f[1] - ua;
                            ddn_a2[s] = ra.f[0] - ub[s];
                            dup_b[s] = last_b ? 0.0 : rb.f[1] - ub_;
                            ddn0[s] = rb.f[0] - ua;
                            ddn1[s] = rb.f[0] - ra.f[1];
                        }
                        attempt2(q, qb, (can_a ? kA : 0ull) | (can_b ? (guess ? kB1 : kB0) : 0ull),
                                 Move{ra.x, ra.y, ra.z, ra.w}, dup_a, ddn_a2, Move{rb.x, rb.y, rb.z, rb.w}, dup_b, ddn0,
                                 ddn1, acc_a, acc_b);
                        nacc += a.record ? acc_a + acc_b : 0u;
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            uint64_t mz = q.me[s] >> 1;
                            if (TWO && s == 0)
                                mz |= q.me[NS - 1] << 63;
                            // bond i by A's forward bond, then by B's backward one
                            ub[s] = lane_bit(acc_a ? mz : 0ull) ? ra.f[0] : ub[s];
                            ub[s] = lane_bit(acc_a && !last_a ? q.me[s] : 0ull) ? ra.f[1] : ub[s];
                            ub[s] = lane_bit(acc_b ? q.me[s] : 0ull) ? rb.f[0] : ub[s];
                            ub[s] = lane_bit(acc_b && !last_b ? qb.me[s] : 0ull) ? rb.f[1] : ub[s];
                        }
                    }
                    trend = max(-4, min(3, trend + (acc_a ? 1 : -1)));
                    if (two && (acc_a != 0u) == guess) {
                        run = acc_b ? (acc_a ? run + 2 : 1) : 0;
                        q = after(qb);
                    } else {
                        run = acc_a ? run + 1 : 0;
                        q = qb;
                    }
                }
            }
            // one double bridging: bonds (bi, bi+1), (bj, bj+1) -> (bi, bj), (bi+1, bj+1)
            const Words4 w = philox4x32_10(chain, g, 0u, kTagBridge, a.k0, a.k1);
            int bi = (int)(((uint64_t)w.w[0] * (uint64_t)(N - 1)) >> 32);
            int bj = (int)(((uint64_t)w.w[1] * (uint64_t)(N - 1)) >> 32);
            if (bi > bj) {
                const int tmp = bi;
                bi = bj;
                bj = tmp;
            }
            if (N >= 4 && bj - bi >= 2) {
                double ix, iy, iz, kx, ky, kz, jx, jy, jz, mx, my, mz; // beads bi, bi+1, bj, bj+1
                readlane_bead(bi, ix, iy, iz);
                readlane_bead(bi + 1, kx, ky, kz);
                readlane_bead(bj, jx, jy, jz);
                readlane_bead(bj + 1, mx, my, mz);
                bool br = false;
                const double fij = fene_energy(p, dist2d(ix, iy, iz, jx, jy, jz), &br);
                const double fkl = fene_energy(p, dist2d(kx, ky, kz, mx, my, mz), &br);
                if (!br) {
                    const double fik = bond_of(bi), fjl = bond_of(bj);
                    const double lij = lj_energy(p, dist2d(ix, iy, iz, jx, jy, jz));
                    const double lkl = lj_energy(p, dist2d(kx, ky, kz, mx, my, mz));
                    const double lik = lj_energy(p, dist2d(ix, iy, iz, kx, ky, kz));
                    const double ljl = lj_energy(p, dist2d(jx, jy, jz, mx, my, mz));
                    const double dF = ((fij + fkl) - fik) - fjl;
                    const double dL = ((lik + ljl) - lij) - lkl;
                    const double En = E + (dF + dL);
                    const int32_t bn = energy_bin(p, En, a.n_bins);
                    if (bn >= 0 && min(w.w[3], 0xFFFFFFFEu) < a.thresholds[(size_t)b * B + (uint32_t)bn]) {
                        // beads bi+1 .. bj in reverse order; the bonds between them reversed
                        double nx[NS], ny[NS], nz[NS], nub[NS];
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            const int bd = j + 64 * s;
                            const int sx = (bd > bi && bd <= bj) ? bi + 1 + bj - bd : bd;
                            const int su = (bd > bi && bd < bj) ? bi + bj - bd : bd;
                            // (a position is a float, exactly)
                            float vx = from_lane((float)xd[0], sx & 63), vy = from_lane((float)yd[0], sx & 63),
                                  vz = from_lane((float)zd[0], sx & 63);
                            double u = from_lane_f64(ub[0], su & 63);
                            if constexpr (TWO) {
                                const float hx = from_lane((float)xd[NS - 1], sx & 63),
                                            hy = from_lane((float)yd[NS - 1], sx & 63),
                                            hz = from_lane((float)zd[NS - 1], sx & 63);
                                const double hu = from_lane_f64(ub[NS - 1], su & 63);
                                vx = sx >= 64 ? hx : vx, vy = sx >= 64 ? hy : vy, vz = sx >= 64 ? hz : vz;
                                u = su >= 64 ? hu : u;
                            }
                            nx[s] = vx, ny[s] = vy, nz[s] = vz;
                            nub[s] = bd == bi ? fij : (bd == bj ? fkl : u);
                        }
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            xd[s] = nx[s], yd[s] = ny[s], zd[s] = nz[s];
                            ub[s] = nub[s];
                        }
                        if constexpr (CACHE)
                            fill_cache(); // the pair terms under the new numbering
                        E = En;
                        b = __builtin_amdgcn_readfirstlane(bn);
                        row_at = 4u * B * (uint32_t)b;
                        nacc += a.record ? 1u : 0u;
                    }
                }
            }
        }
        if (a.record && c < a.n_chains && j == 0)
            atomicAdd(&lhist[b], 1u);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int bd = j + 64 * s;
        if (bd < N)
            pos[bd] = make_float4((float)xd[s], (float)yd[s], (float)zd[s], 0.f);
        if (bd < N - 1)
            bond[bd] = ub[s];
    }
    if (j == 0) {
        a.energy[c] = E;
        a.bins[c] = b;
        if (a.record && c < a.n_chains)
            atomicAdd(&accepted, (unsigned long long)nacc);
    }
    __syncthreads();
    // one atomic per workgroup on the run's one counter
    if (threadIdx.x == 0 && a.accepts && accepted)
        atomicAdd(a.accepts, accepted);
    for (int i = threadIdx.x; i < a.n_bins; i += blockDim.x) {
        const uint32_t v = lhist[i];
        if (v)
            atomicAdd(&a.hist[i], (unsigned long long)v);
    }
}

// One tile of the threshold matrix T[b][b'] = floor(2^32 e^D), D = lnW[b'] -
// lnW[b] (all ones for D >= 0 and from 2^32 - 1 on).  lnW is pinned host
// memory: a tile reads its rows' and columns' weights once.  The host's exp
// decides what the table holds; this one and the host's are within one unit
// in the last place of e^D each, so entries within eight units of an integer
// are listed for the host and all others are the host's.  Bound by FP64 issue
// (an exp per entry): the 2500 x 2500 matrix takes about 30 us, where sixteen
// host threads and the upload of 25 MB took 3.5 to 8 ms.
__global__ __launch_bounds__(1024) void polymer_table(const double *lnW, uint32_t *T, int B, uint32_t *unsure)
{
    __shared__ double wr[kTableRows], wc[kTableCols];
    __shared__ uint32_t count;
    const int r0 = (int)blockIdx.y * kTableRows, c0 = (int)blockIdx.x * kTableCols;
    const int rows = min(kTableRows, B - r0), cols = min(kTableCols, B - c0);
    uint32_t *list = unsure + (size_t)(blockIdx.y * gridDim.x + blockIdx.x) * (kTableUnsure + 1);
    const int tid = (int)threadIdx.x;
    if (tid < cols)
        wc[tid] = lnW[c0 + tid];
    else if (tid >= kTableCols && tid - kTableCols < rows)
        wr[tid - kTableCols] = lnW[r0 + tid - kTableCols];
    if (tid == 0)
        count = 0u;
    __syncthreads();
    const int c = tid % kTableCols;
    if (c < cols) {
        for (int r = tid / kTableCols; r < rows; r += 1024 / kTableCols) {
            const double D = wc[c] - wr[r];
            uint32_t t = D >= 0.0 ? 0xFFFFFFFFu : 0u;
            if (!(D >= 0.0) && !(D < -23.0)) { // D < -23: 2^32 e^D < 1
                const double v = exp(D) * 4294967296.0;
                t = v >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)v;
                const double n = rint(v);
                if (!(fabs(v - n) > v * 0x1p-49) && !(n == 0.0) && !(v >= 4294967295.5)) {
                    const uint32_t k = atomicAdd(&count, 1u);
                    if (k < (uint32_t)kTableUnsure)
                        list[1 + k] = (uint32_t)(r * kTableCols + c);
                }
            }
            T[(size_t)(r0 + r) * (size_t)B + (size_t)(c0 + c)] = t;
        }
    }
    __syncthreads();
    if (tid == 0)
        list[0] = count;
}

__global__ void patch_table(uint32_t *T, const uint32_t *pairs, int n)
{
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n)
        T[pairs[2 * i]] = pairs[2 * i + 1];
}

hipError_t launch_polymer_table(const double *lnW, uint32_t *T, int n_bins, uint32_t *unsure, hipStream_t s)
{
    const dim3 grid((unsigned)((n_bins + kTableCols - 1) / kTableCols), (unsigned)((n_bins + kTableRows - 1) / kTableRows));
    hipLaunchKernelGGL(polymer_table, grid, dim3(1024), 0, s, lnW, T, n_bins, unsure);
    return hipGetLastError();
}

hipError_t launch_patch_table(uint32_t *T, const uint32_t *pairs, int n, hipStream_t s)
{
    hipLaunchKernelGGL(patch_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, T, pairs, n);
    return hipGetLastError();
}

// The cache is used when a CU still holds two wavefronts per SIMD with it, or
// every workgroup of a small grid has its place at once.  Measured, moves/s
// with the cache and without (shifts | full set):
//   N = 50, 4096 chains (three workgroups per CU)   4.48e9 | 2.83e9   4.08e9 | 2.50e9   cache
//   N = 54, 4096 chains (two per CU)                4.19e9 | 2.64e9   4.11e9 | 2.56e9   cache
//   N = 64, 2048 chains (two per CU, all at once)   4.18e9 | 2.57e9   3.55e9 | 2.30e9   cache
//   N = 64, 2052 chains                             2.77e9 | 1.67e9   2.77e9 | 1.72e9   cache
//   N = 64, 4096 chains                             4.21e9 | 2.64e9   4.17e9 | 2.59e9   cache
//   N = 80, 1024 chains (one per CU, all at once)   1.91e9 | 1.35e9   1.83e9 | 1.30e9   cache
//   N = 80, 2048 chains                             1.88e9 | 1.35e9   2.34e9 | 1.67e9
static bool polymer_cache_fits(size_t lds, int chains_per_block, long blocks, int cus)
{
    const long room = (long)(160u * 1024u / (lds + 16u)); // 16: the workgroup's counter
    return room * chains_per_block >= 8 || (room >= 1 && room * cus >= blocks);
}

template <bool TWO, bool MOVES>
static hipError_t launch_polymer(const PolymerArgs &a, const PolyParams &p, int cus, hipStream_t s)
{
    const int n_c = a.chains_per_block;
    const dim3 grid((unsigned)(a.c_pad / n_c)), block((unsigned)(64 * n_c));
    const size_t cached = hist_bytes(a.n_bins) + (size_t)n_c * chain_lds(a.n_beads, true, MOVES);
    const size_t plain = hist_bytes(a.n_bins) + (size_t)n_c * chain_lds(a.n_beads, false, MOVES);
    const bool cache = polymer_cache_fits(cached, n_c, (long)grid.x, cus);
    const size_t lds = cache ? cached : plain;
    auto k = cache ? polymer_sweeps<TWO, MOVES, true> : polymer_sweeps<TWO, MOVES, false>;
    if (lds > 65536u) {
        hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess)
            return e;
    }
    hipLaunchKernelGGL(k, grid, block, lds, s, a, p);
    return hipGetLastError();
}

hipError_t launch_polymer_sweeps(const PolymerArgs &a, const PolymerConsts &k, hipStream_t s)
{
    PolyParams p;
    p.lj_eps4 = 4.0 * k.lj_eps;
    p.sig2 = k.lj_sigma * k.lj_sigma;
    p.rc2 = k.lj_rcut * k.lj_rcut;
    p.lj_shift = k.lj_shift;
    p.fene_pref = k.fene_pref;
    p.fene_r0 = k.fene_r0;
    p.fene_R = k.fene_R;
    p.x_lo = k.x_lo;
    p.x_hi = k.x_hi;
    p.scale = k.scale;
    if (a.chains_per_block < 1 || a.chains_per_block > 4 || a.c_pad % a.chains_per_block)
        return hipErrorInvalidValue;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (a.n_beads > 64)
        return a.moves ? launch_polymer<true, true>(a, p, cus, s) : launch_polymer<true, false>(a, p, cus, s);
    return a.moves ? launch_polymer<false, true>(a, p, cus, s) : launch_polymer<false, false>(a, p, cus, s);
}

} // namespace muca
