// lattice_tile.h -- Metropolis sweeps of one lattice chain per wavefront,
// a tile of up to 64 consecutive sites at a time (gfx950).
//
// A chain's attempts are a serial recurrence: an attempt's threshold depends
// on the chain's bin and on its neighbours, both of which earlier attempts
// change.  Visiting the sites one after another costs a compare, two selects
// and an LDS read per site on the critical path (80 cycles for Ising), and a
// few thousand chains do not fill the chip, so that path was the run time.
// Here lane i holds site i of a tile (R = 64 / L whole rows) and all attempts
// of the tile are decided together, as the fixed point of
//     outcomes -> bins (prefix sum over the lanes) -> thresholds -> outcomes.
// Starting from "nothing accepted", every pass decides all sites from the
// bins that the previous pass's outcomes give; the pass that reproduces its
// own input is the answer.  The first site's bin is always right, and a site
// is decided rightly once all sites before it are, so each pass extends the
// correct prefix by at least one site and the fixed point is unique: it is
// the serial result bit for bit, whatever the guesses were.  A wrong guess
// needs thresholds that differ between bins a few apart, which measured
// weights rarely do: 2.2 to 3.5 passes per tile on the weights of runs in
// progress, 10 with thresholds that jump by a factor e from bin to bin.
//
// The thresholds of a pass are read for every outcome of the neighbours that
// sit earlier in the tile (left, and up where a tile has several rows).  The
// outcomes are 64-bit masks on the scalar unit, where the dependence on those
// neighbours is followed a few links without further reads, and a lane's bin
// is counted from them (Ising, MUMA: bits below the lane; Potts, whose steps
// take nine values: a DPP scan).  The lattice never leaves the registers
// during a launch: lane t holds tile t as a 64-bit mask (Ising, MUMA), or
// lane i holds its site's colour of every tile, four per register (Potts).
//
// Bound, by SQ counters on weights of runs in progress.  Four wavefronts per
// SIMD: the vector unit is busy 63 to 75 % of the cycles and the scalar unit
// 55 % (Ising L = 64, 4096 chains: 68 vector, 59 scalar and 3 LDS
// instructions per tile of 64), the rest are waits between dependent
// instructions of all four.  Two: 59 % (Potts L = 48, 2048 chains: 118, 36 and
// 7 per tile of 48).  One or fewer: a tile is one chain of LDS reads, ballots
// and scalar operations.  Measured per iteration, before (16 lanes per chain,
// site by site) and after: Ising L = 64, 4096 chains, 400 sweeps 54.5 -> 17.6
// ms; Ising L = 32 int8, 1000 chains, 35 sweeps 1.69 -> 0.32 ms; MUMA L = 32
// with the joint histogram, 512 chains, 67 sweeps 2.85 -> 0.49 ms; Potts q = 8
// L = 48, 2048 chains, 362 sweeps 39.4 -> 10.9 ms; Potts q = 10 L = 64 (table
// in global memory), 1024 chains, 60 sweeps 14.4 -> 2.8 ms.
#pragma once
#include "lattice_impl.h"
#include "launch_rules.h"

namespace muca {

// Links of the chains of neighbours followed in one pass beyond the first.
// More save passes where weights are smooth, and cost scalar (Ising: vector)
// instructions in every pass where they are rough.  Cycles per site of a SIMD
// with four wavefronts, smooth weights / noise of 0.3 per bin: Ising L = 64
// two links 23.4 / 45.4, three 23.5 / 48.7; L = 16 one 39.3 / 46.0, two 37.6 /
// 46.9; MUMA L = 64 one 17.3 / 22.4, two 18.5 / 22.4; Potts L = 48 one 41.9 /
// 67.2, two 42.0 / 68.9.
template <int MODEL>
constexpr int kTileAhead = MODEL == kIsing ? 2 : 1;

template <int L>
struct Tile {
    static constexpr int R = L * L <= 64 ? L : 64 / L; // rows
    static constexpr int TS = R * L;                   // sites
    static constexpr int NT = L / R;                   // tiles of a lattice
    static constexpr bool kWhole = NT == 1;            // the tile is the lattice
    static constexpr uint64_t ones(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1ull; }
    static constexpr uint64_t column(int x)
    {
        uint64_t m = 0ull;
        for (int r = 0; r < R; ++r)
            m |= 1ull << (r * L + x);
        return m;
    }
    static constexpr uint64_t kAll = ones(TS), kFirst = column(0), kLast = column(L - 1);
    static_assert(L % R == 0 && (NT == 1 || NT % 4 == 0), "tiles come in whole Philox batches");
};

__device__ __forceinline__ bool lane_bit(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// v with lane `lane` set to x (the compiler has no builtin for this intrinsic):
// a tile's two words back to the lane that keeps them by one instruction each.
// A compare, copies and selects took five; cycles per site, 512 chains:
// Ising L = 64 13.2 -> 12.6, MUMA L = 32 11.2 -> 10.6.
extern "C" __device__ uint32_t write_lane(uint32_t x, uint32_t lane, uint32_t v) __asm("llvm.amdgcn.writelane.i32");

template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// v of lane i = first + the sum of v over the lanes below i.
__device__ __forceinline__ int32_t prefix_from(int32_t first, int32_t v)
{
    int32_t x = __builtin_amdgcn_update_dpp(first, v, 0x138, 0xF, 0xF, false); // wave_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);             // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);            // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);            // row_bcast:31
    return x;
}

// Words of four tiles from one Philox call per lane.  Lane 4 q + k has drawn
// call q of tile k; site 4 q + j of tile k takes word j of that call, so a
// tile's words are the columns of a 4 x 4 transpose within each quad (two
// exchange steps).
__device__ __forceinline__ void quad_transpose(uint32_t (&w)[4])
{
    const bool odd = lane_bit(0xAAAAAAAAAAAAAAAAull), high = lane_bit(0xCCCCCCCCCCCCCCCCull);
    uint32_t x[4], a[4];
    // the exchanges run on all lanes, the selects after them
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] = quad_perm<0xB1>(w[j]); // quad_perm [1,0,3,2]
    a[0] = odd ? x[1] : w[0];
    a[1] = odd ? w[1] : x[0];
    a[2] = odd ? x[3] : w[2];
    a[3] = odd ? w[3] : x[2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        x[j] = quad_perm<0x4E>(a[j]); // quad_perm [2,3,0,1]
    w[0] = high ? x[2] : a[0];
    w[2] = high ? a[2] : x[0];
    w[1] = high ? x[3] : a[1];
    w[3] = high ? a[3] : x[1];
}

// The lanes below this one whose bit is set in m, added to v.
__device__ __forceinline__ int32_t below(uint64_t m, int32_t v)
{
    return (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)v));
}

// v + (this lane's bit of m): one add with carry-in.  m comes from the scalar
// unit (a mask that a vector compare has just written would need two wait
// states).
__device__ __forceinline__ int32_t add_bit(int32_t v, uint64_t m)
{
    int32_t out;
    asm("v_addc_co_u32 %0, vcc, 0, %1, %2" : "=v"(out) : "v"(v), "s"(m) : "vcc");
    return out;
}

// ---------------------------------------------------------------------------
// Ising / MUMA
// ---------------------------------------------------------------------------
// The attempts of one tile: S its spins (bit set = +1), P and N the tiles
// above and below it, r each lane's acceptance word (accept iff r < T; lanes
// beyond the tile hold 2^32 - 1).  Returns the accepted sites; b becomes the
// bin after the tile.
template <int MODEL, int L, bool TLDS>
__device__ __forceinline__ uint64_t spin_tile(uint64_t S, uint64_t P, uint64_t N, uint32_t r, int32_t &b,
                                              int32_t n_bins, const uint32_t *T, int32_t tbase)
{
    using G = Tile<L>;
    constexpr int R = G::R, TS = G::TS, UP = TS - L;
    constexpr int COL = MODEL == kIsing ? 4 : 8, ROW = 4 * Cols<MODEL>::value; // bytes
    uint64_t Su, Sd;
    if constexpr (G::kWhole) {
        Su = (S << L) | (S >> UP);
        Sd = (S >> L) | (S << UP);
    } else if constexpr (R == 1) {
        Su = P;
        Sd = N;
    } else {
        Su = (S << L) | (P >> UP);
        Sd = (S >> L) | (N << UP);
    }
    const uint64_t Sl = ((S << 1) & ~G::kFirst) | ((S >> (L - 1)) & G::kFirst);
    const uint64_t Sr = ((S >> 1) & ~G::kLast) | ((S << (L - 1)) & G::kLast);
    // aligned with the left, up, right and down neighbours as the tile starts
    const uint64_t AL = ~(S ^ Sl), AU = ~(S ^ Su), AR = ~(S ^ Sr), AD = ~(S ^ Sd);
    // column of the aligned neighbours that earlier attempts of the tile do
    // not change
    int32_t col = TLDS ? tbase : 0;
    if constexpr (MODEL == kMuma)
        col += lane_bit(S) ? 4 : 0;
    const int32_t dr = lane_bit(AR) ? COL : 0, dd = lane_bit(AD) ? COL : 0;
    col += dr + dd;
    if constexpr (R == 1)
        col += lane_bit(AU) ? COL : 0;
    const int32_t col_wrap = col + COL - 2 * dr, wrap_d = COL - 2 * dd; // with the right neighbour flipped

    uint64_t F, A;           // accepted sites, and the outcomes at the bins that they give
    uint64_t l = AL, u = AU; // aligned left and up neighbours once the sites of F have flipped
    uint32_t t[3];           // thresholds by the number of those two
    auto read = [&](int32_t at) {
#pragma unroll
        for (int k = 0; k < (R == 1 ? 2 : 3); ++k)
            t[k] = TLDS ? ((lds_u32 *)(uintptr_t)(uint32_t)at)[k * (COL / 4)]
                        : ((const gu32 *)((uintptr_t)T + (uint32_t)at))[k * (COL / 4)];
    };
    auto flips = [&](uint64_t a) {
        if constexpr (R == 1) { // nothing shifts into site 0
            l = AL ^ (a << 1);
        } else {
            l = AL ^ ((a << 1) & ~G::kFirst);
            u = AU ^ (a << L);
        }
    };
    uint64_t C0 = 0ull, Q = 0ull; // R = 1: outcomes without an aligned left neighbour, and where one changes them
    auto decide = [&]() {
        if constexpr (R == 1) {
            C0 = ballot(r < t[0]);
            Q = C0 ^ ballot(r < t[1]);
        }
    };
    auto outcomes = [&]() -> uint64_t {
        if constexpr (R == 1) {
            return C0 ^ (Q & l);
        } else {
            const uint32_t t0 = lane_bit(l) ? t[1] : t[0], t1 = lane_bit(l) ? t[2] : t[1];
            return ballot(r < (lane_bit(u) ? t1 : t0));
        }
    };
    // a few links of the chains of neighbours at once; whatever is left is
    // found by the next pass
    auto ahead = [&](uint64_t a) {
#pragma unroll
        for (int k = 0; k < kTileAhead<MODEL>; ++k) {
            flips(a);
            a = outcomes();
        }
        flips(a);
        return a;
    };
    int32_t x, c;
    auto pass = [&]() {
        // bins that F gives.  A row's last site sees site 0 (its right
        // neighbour) as F left it, the last row of a whole lattice the first
        const uint64_t wr = (F << (L - 1)) & G::kLast, wd = G::kWhole ? F << UP : 0ull;
        c = lane_bit(wr) ? col_wrap : col;
        if constexpr (G::kWhole)
            c += lane_bit(wd) ? wrap_d : 0;
        if constexpr (MODEL == kMuma) // M grows where a -1 flips
            x = below(F & ~S, b) - below(F & S, 0);
        else // a flip with n aligned neighbours moves the bin by n - 2
            x = below(F & l, below(F & u, below(F & (AR ^ wr), below(F & (AD ^ wd), b)))) - 2 * below(F, 0);
        // a wrong guess may leave the table (the answer cannot): any row does
        read(__mul24((int32_t)min((uint32_t)x, (uint32_t)(n_bins - 1)), ROW) + c);
        decide();
        return outcomes();
    };
    read(b * ROW + col); // first every lane at the tile's first bin
    decide();
    F = ahead(outcomes());
    A = pass();
    while (A != F) {
        F = ahead(A);
        A = pass();
    }
    if constexpr (MODEL == kMuma) {
        b += __builtin_popcountll(F & ~S) - __builtin_popcountll(F & S);
    } else { // the last site's own step is behind its lane's bin
        int32_t n = add_bit((c >> 2) - ((TLDS ? tbase >> 2 : 0) + 2), l);
        if constexpr (R > 1)
            n = add_bit(n, u);
        b = __builtin_amdgcn_readlane(x + (lane_bit(F) ? n : 0), TS - 1);
    }
    return F;
}

// Tile t of a chain from storage, one lane per tile.
template <int L>
__device__ __forceinline__ uint64_t spin_load(const gu32 *base, size_t stride, int layout, int t)
{
    uint64_t m = 0ull;
#pragma unroll
    for (int r = 0; r < Tile<L>::R; ++r) {
        uint32_t row[Row1<L>::W];
        if (layout == kLayoutBit)
            load_row<L, kLayoutBit>(base, stride, t * Tile<L>::R + r, row);
        else
            load_row<L, kLayoutByte>(base, stride, t * Tile<L>::R + r, row);
        uint64_t v = row[0];
        if constexpr (Row1<L>::W > 1)
            v |= (uint64_t)row[1] << 32;
        m |= v << (r * L);
    }
    return m;
}

template <int L>
__device__ __forceinline__ void spin_store(gu32 *base, size_t stride, int layout, int t, uint64_t m)
{
#pragma unroll
    for (int r = 0; r < Tile<L>::R; ++r) {
        const uint64_t v = (m >> (r * L)) & Tile<L>::ones(L);
        uint32_t row[Row1<L>::W];
        row[0] = (uint32_t)v;
        if constexpr (Row1<L>::W > 1)
            row[1] = (uint32_t)(v >> 32);
        if (layout == kLayoutBit)
            store_row<L, kLayoutBit>(base, stride, t * Tile<L>::R + r, row);
        else
            store_row<L, kLayoutByte>(base, stride, t * Tile<L>::R + r, row);
    }
}

// What a wave carries from one launch segment to the next.
template <int MODEL, int L, bool TLDS>
struct SpinChain {
    using G = Tile<L>;
    uint32_t lo, hi; // lane t: tile t

    __device__ __forceinline__ void load(const LatticeArgs &a, int c, int lane)
    {
        uint64_t m = 0ull;
        if (lane < G::NT)
            m = spin_load<L>((const gu32 *)a.words + c, (size_t)a.c_pad, a.layout, lane);
        lo = (uint32_t)m;
        hi = (uint32_t)(m >> 32);
    }
    __device__ __forceinline__ void store(const LatticeArgs &a, int c, int lane) const
    {
        if (lane < G::NT)
            spin_store<L>((gu32 *)a.words + c, (size_t)a.c_pad, a.layout, lane, ((uint64_t)hi << 32) | lo);
    }
    __device__ __forceinline__ uint64_t tile(int t) const
    {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, t) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)lo, t);
    }
    __device__ __forceinline__ void set_tile(int t, uint64_t m)
    {
        if constexpr (G::kWhole) {
            lo = lane_bit(1ull) ? (uint32_t)m : lo;
            hi = lane_bit(1ull) ? (uint32_t)(m >> 32) : hi;
        } else {
            lo = write_lane((uint32_t)m, (uint32_t)t, lo);
            hi = write_lane((uint32_t)(m >> 32), (uint32_t)t, hi);
        }
    }

    // Unsatisfied bonds of the configuration (right and down bond of every
    // site, counted by the lane that holds its tile).
    __device__ __forceinline__ uint32_t unsatisfied(int lane) const
    {
        const uint64_t S = ((uint64_t)hi << 32) | lo;
        const int next = (lane + 1 < G::NT ? lane + 1 : 0) * 4;
        const uint64_t N = ((uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(next, (int)hi) << 32) |
                           (uint32_t)__builtin_amdgcn_ds_bpermute(next, (int)lo);
        const uint64_t Sr = ((S >> 1) & ~G::kLast) | ((S << (L - 1)) & G::kLast);
        uint64_t Sd = N;
        if constexpr (G::R > 1)
            Sd = (S >> L) | (N << (G::TS - L));
        int32_t n = __builtin_popcountll((S ^ Sr) & G::kAll) + __builtin_popcountll((S ^ Sd) & G::kAll);
        n = lane < G::NT ? n : 0;
        return (uint32_t)(__builtin_amdgcn_readlane(prefix_from(0, n), 63) + __builtin_amdgcn_readlane(n, 63));
    }

    // `n` sweeps from global sweep g; adds the accepted moves to nacc.
    template <class Count>
    __device__ __forceinline__ void sweeps(const LatticeArgs &a, uint32_t chain, uint32_t g, int n, int lane,
                                           const uint32_t *T, int32_t tbase, int32_t &b, uint32_t &nacc, Count count)
    {
        constexpr int NT = G::NT, CPT = G::TS / 4; // Philox calls per tile
        const uint32_t q = (uint32_t)lane >> 2, k = (uint32_t)lane & 3u;
        uint32_t w[4];
        // words of tiles t0 .. t0 + 3 (a whole-lattice tile: of four sweeps)
        auto draw = [&](uint32_t sweep, int t0) {
            const Words4 v = G::kWhole ? philox4x32_10(chain, sweep + k, q, kTagSweep, a.k0, a.k1)
                                       : philox4x32_10(chain, sweep, ((uint32_t)t0 + k) * (uint32_t)CPT + q, kTagSweep,
                                                       a.k0, a.k1);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = min(v.w[j], 0xFFFFFFFEu);
                if constexpr (G::TS < 64)
                    w[j] = lane < G::TS ? w[j] : 0xFFFFFFFFu;
            }
            quad_transpose(w);
        };
        if constexpr (G::kWhole) {
            uint64_t S = tile(0);
            for (int s = 0; s < n; s += 4) {
                draw(g + (uint32_t)s, 0);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    if (s + m >= n)
                        break;
                    const uint64_t F = spin_tile<MODEL, L, TLDS>(S, S, S, w[m], b, a.n_bins, T, tbase);
                    nacc += (uint32_t)__builtin_popcountll(F);
                    S ^= F;
                    if constexpr (MODEL == kMuma)
                        set_tile(0, S);
                    count(b);
                }
            }
            set_tile(0, S);
        } else {
            uint64_t P = tile(NT - 1), S = tile(0);
            for (int s = 0; s < n; ++s) {
                for (int t0 = 0; t0 < NT; t0 += 4) {
                    draw(g + (uint32_t)s, t0);
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int t = t0 + m;
                        const uint64_t N = tile(t + 1 < NT ? t + 1 : 0);
                        const uint64_t F = spin_tile<MODEL, L, TLDS>(S, P, N, w[m], b, a.n_bins, T, tbase);
                        nacc += (uint32_t)__builtin_popcountll(F);
                        P = S ^ F;
                        set_tile(t, P);
                        S = N;
                    }
                }
                count(b);
            }
        }
    }
};

// ---------------------------------------------------------------------------
// Potts
// ---------------------------------------------------------------------------
// e + (colour == old) - (colour == proposal): the change in unsatisfied bonds
// with one more neighbour counted.
__device__ __forceinline__ int32_t potts_add(int32_t e, uint32_t colour, uint32_t old, uint32_t nw)
{
    e += colour == old ? 1 : 0;
    e -= colour == nw ? 1 : 0;
    return e;
}

// Byte offset of the change dE in a bin's row.  Rows in global memory have
// nine columns, dE = -4..4; staged rows eight (dE = 0 always accepts and is
// not read), looked up by one byte permute with selector dE + 4: +4 selects
// the sign of byte 1, which is zero.
template <bool TLDS>
__device__ __forceinline__ int32_t potts_col(int32_t dE)
{
    if constexpr (TLDS)
        return (int32_t)__builtin_amdgcn_perm(0x18141000u, 0x0C08041Cu, (uint32_t)(dE + 0x0C0C0C04));
    return 4 * (dE + 4);
}

// The staged slot of a row's column c = dE + 4 (c = 4 has none).
__device__ __forceinline__ int potts_staged_slot(int c) { return c == 8 ? 0 : (c == 0 ? 7 : c - (c > 4 ? 1 : 0)); }

// The attempts of one tile.  cur, above, below: colours of this tile, of the
// tile above and of the tile below; (wp, r) proposal and acceptance words.
// Returns the accepted sites and each lane's proposed colour.
template <int L, bool TLDS>
__device__ __forceinline__ uint64_t potts_tile(uint32_t cur, uint32_t above, uint32_t below, uint32_t wp, uint32_t r,
                                               uint32_t q, int lane, int left_l, int right_l, int up_l, int down_l,
                                               int32_t &b, int32_t n_bins, const uint32_t *T, int32_t tbase,
                                               uint32_t &nw)
{
    using G = Tile<L>;
    constexpr int R = G::R, TS = G::TS, UP = TS - L;
    uint32_t p = cur + 1u + __umulhi(wp, q - 1u);
    p = min(p, p - q); // p - q wraps above p when p < q
    nw = p;
    const uint32_t both = cur | (p << 8); // (colour, proposal)
    const uint32_t lf = (uint32_t)__builtin_amdgcn_ds_bpermute(left_l, (int)both);
    const uint32_t rt = (uint32_t)__builtin_amdgcn_ds_bpermute(right_l, (int)both);
    uint32_t up = above, dn = below;
    if constexpr (R > 1) {
        uint32_t v = both;
        if constexpr (!G::kWhole)
            v = lane >= UP ? above | (above << 8) : both;
        up = (uint32_t)__builtin_amdgcn_ds_bpermute(up_l, (int)v);
        if constexpr (!G::kWhole)
            v = lane < L ? below | (below << 8) : both;
        dn = (uint32_t)__builtin_amdgcn_ds_bpermute(down_l, (int)v);
    }
    // dE by the attempts of the left and up neighbours earlier in this tile:
    // neither accepted, left, up, both.  A neighbour that the order visits
    // later, or that lies outside the tile, has one colour.
    constexpr int NV = R > 1 ? 4 : 2;
    int32_t e[4], c[4]; // and the byte offset of its column
    uint64_t Z[4];      // dE = 0
    {
        const bool col0 = lane_bit(G::kFirst);
        int32_t s = potts_add(0, dn & 0xFFu, cur, p);
        s = potts_add(s, rt & 0xFFu, cur, p);
        const int32_t s0 = potts_add(s, up & 0xFFu, cur, p);
        e[0] = potts_add(s0, lf & 0xFFu, cur, p);
        e[1] = potts_add(s0, (lf >> 8) & 0xFFu, cur, p);
        e[1] = col0 ? e[0] : e[1];
        if constexpr (R > 1) {
            const bool row0 = lane < L;
            int32_t s1 = potts_add(s, (up >> 8) & 0xFFu, cur, p);
            s1 = row0 ? s0 : s1;
            e[2] = potts_add(s1, lf & 0xFFu, cur, p);
            e[3] = potts_add(s1, (lf >> 8) & 0xFFu, cur, p);
            e[3] = col0 ? e[2] : e[3];
        }
    }
    auto columns = [&]() {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            c[v] = potts_col<TLDS>(e[v]);
            Z[v] = ballot(e[v] == 0) & G::kAll;
        }
    };
    columns();
    // A row's last site sees site 0 (its right neighbour) as the accepted
    // sites leave it, and the last row of a whole lattice the first one.
    uint64_t wrap_r = 0ull, wrap_d = 0ull;
    auto wraps = [&](uint64_t F) {
        const uint64_t wr = (F << (L - 1)) & G::kLast, wd = G::kWhole ? F << UP : 0ull;
        if (wr == wrap_r && wd == wrap_d)
            return;
        const uint32_t r_was = lane_bit(wrap_r) ? rt >> 8 : rt, r_now = lane_bit(wr) ? rt >> 8 : rt;
        int32_t d = potts_add(0, r_now & 0xFFu, cur, p) - potts_add(0, r_was & 0xFFu, cur, p);
        if constexpr (G::kWhole) {
            const uint32_t d_was = lane_bit(wrap_d) ? dn >> 8 : dn, d_now = lane_bit(wd) ? dn >> 8 : dn;
            d += potts_add(0, d_now & 0xFFu, cur, p) - potts_add(0, d_was & 0xFFu, cur, p);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v)
            e[v] += d;
        columns();
        wrap_r = wr;
        wrap_d = wd;
    };
    // Outcomes as the neighbours' outcomes enter them: B without an accepted
    // left (up) neighbour, toggled by DL (DU) where it was accepted, and by
    // DB more where both were.  Column 0 has one variant: no left neighbour
    // toggles it.
    uint64_t B, DL, DU = 0ull, DB = 0ull;
    auto decide = [&](int32_t row) {
        uint32_t t[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
            t[v] = load_t<TLDS>(T, row + c[v]);
        uint64_t C[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
            C[v] = ballot(r < t[v]) | Z[v];
        B = C[0];
        DL = C[0] ^ C[1];
        if constexpr (R > 1) {
            DU = C[0] ^ C[2];
            DB = DL ^ C[2] ^ C[3];
        }
    };
    auto outcomes = [&](uint64_t A) -> uint64_t {
        if constexpr (R == 1)
            return B ^ (DL & (A << 1));
        const uint64_t l = A << 1, u = A << (R > 1 ? L : 0);
        return B ^ (l & DL) ^ (u & (DU ^ (l & DB)));
    };
    auto ahead = [&](uint64_t A) {
#pragma unroll
        for (int k = 0; k < kTileAhead<kPotts>; ++k)
            A = outcomes(A);
        return A;
    };
    int32_t x, n;
    auto pass = [&](uint64_t F) {
        wraps(F);
        const bool la = lane_bit(F << 1);
        n = la ? e[1] : e[0];
        if constexpr (R > 1) {
            const int32_t m = la ? e[3] : e[2];
            n = lane_bit(F << L) ? m : n;
        }
        n = lane_bit(F) ? n : 0;
        x = prefix_from(b, n);
        // a wrong guess may leave the table (the answer cannot): any row does
        const int32_t xr = (int32_t)min((uint32_t)x, (uint32_t)(n_bins - 1));
        decide(TLDS ? tbase + 32 * xr : __mul24(xr, 36));
        return outcomes(F);
    };
    decide(TLDS ? tbase + 32 * b : 36 * b); // first every lane at the tile's first bin
    uint64_t F = ahead(B), A = pass(F);
    while (A != F) {
        F = ahead(A);
        A = pass(F);
    }
    b = __builtin_amdgcn_readlane(x, TS - 1) + __builtin_amdgcn_readlane(n, TS - 1);
    return F;
}

template <int L, bool TLDS>
struct PottsChain {
    using G = Tile<L>;
    static constexpr int NV = (G::NT + 3) / 4;
    uint32_t lat[NV]; // byte t % 4 of lat[t / 4]: this lane's site of tile t

    __device__ __forceinline__ void load(const LatticeArgs &a, int c, int lane)
    {
        const gu8 *base = (const gu8 *)((const gu32 *)a.words + c);
        const size_t stride = (size_t)a.c_pad * 4u;
#pragma unroll
        for (int v = 0; v < NV; ++v)
            lat[v] = 0u;
        if (lane < G::TS) {
#pragma unroll
            for (int t = 0; t < G::NT; ++t) {
                const int i = t * G::TS + lane; // site: word i / 4, byte i % 4
                lat[t / 4] |= (uint32_t)base[(size_t)(i >> 2) * stride + (size_t)(i & 3)] << (8 * (t % 4));
            }
        }
    }
    __device__ __forceinline__ void store(const LatticeArgs &a, int c, int lane) const
    {
        gu8 *base = (gu8 *)((gu32 *)a.words + c);
        const size_t stride = (size_t)a.c_pad * 4u;
        if (lane < G::TS) {
#pragma unroll
            for (int t = 0; t < G::NT; ++t) {
                const int i = t * G::TS + lane;
                base[(size_t)(i >> 2) * stride + (size_t)(i & 3)] = (uint8_t)(lat[t / 4] >> (8 * (t % 4)));
            }
        }
    }
    __device__ __forceinline__ uint32_t unsatisfied(int) const { return 0u; }

    template <class Count>
    __device__ __forceinline__ void sweeps(const LatticeArgs &a, uint32_t chain, uint32_t g, int n, int lane,
                                           const uint32_t *T, int32_t tbase, int32_t &b, uint32_t &nacc, Count count)
    {
        constexpr int NT = G::NT, TS = G::TS, CPT = TS / 2; // Philox calls per tile
        const uint32_t q = (uint32_t)a.q, pair = (uint32_t)lane >> 1, k = (uint32_t)lane & 1u;
        const bool odd = lane_bit(0xAAAAAAAAAAAAAAAAull);
        // byte addresses of the lanes that hold a site's neighbours
        const int col = lane % L;
        const int left_l = 4 * (col > 0 ? lane - 1 : lane + L - 1), right_l = 4 * (col < L - 1 ? lane + 1 : lane - L + 1);
        const int up_l = 4 * (lane >= L ? lane - L : lane + TS - L), down_l = 4 * (lane < TS - L ? lane + L : lane - TS + L);
        uint32_t w[4]; // (proposal, acceptance) words of two tiles
        // Lane 2 m + k draws call m of tile t0 + k (a whole-lattice tile: of
        // sweep + k); site 2 m + j of a tile takes words 2 j, 2 j + 1.
        auto draw = [&](uint32_t sweep, int t0) {
            const Words4 v = G::kWhole ? philox4x32_10(chain, sweep + k, pair, kTagSweep, a.k0, a.k1)
                                       : philox4x32_10(chain, sweep, ((uint32_t)t0 + k) * (uint32_t)CPT + pair,
                                                       kTagSweep, a.k0, a.k1);
            const uint32_t r0 = min(v.w[1], 0xFFFFFFFEu), r1 = min(v.w[3], 0xFFFFFFFEu);
            // the exchanges run on all lanes, the selects after them
            const uint32_t x0 = quad_perm<0xB1>(v.w[0]), x1 = quad_perm<0xB1>(r0), x2 = quad_perm<0xB1>(v.w[2]),
                           x3 = quad_perm<0xB1>(r1);
            w[0] = odd ? x2 : v.w[0];
            w[1] = odd ? x3 : r0;
            w[2] = odd ? v.w[2] : x0;
            w[3] = odd ? r1 : x1;
            if constexpr (TS < 64) {
                w[1] = lane < TS ? w[1] : 0xFFFFFFFFu;
                w[3] = lane < TS ? w[3] : 0xFFFFFFFFu;
            }
        };
        auto attempt = [&](uint32_t cur, uint32_t above, uint32_t below, int m) -> uint32_t {
            uint32_t nw;
            const uint64_t F = potts_tile<L, TLDS>(cur, above, below, w[2 * m], w[2 * m + 1], q, lane, left_l, right_l,
                                                   up_l, down_l, b, a.n_bins, T, tbase, nw);
            nacc += (uint32_t)__builtin_popcountll(F);
            return lane_bit(F) ? nw : cur;
        };
        if constexpr (G::kWhole) {
            for (int s = 0; s < n; s += 2) {
                draw(g + (uint32_t)s, 0);
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    if (s + m >= n)
                        break;
                    lat[0] = attempt(lat[0], lat[0], lat[0], m);
                    count(b);
                }
            }
        } else {
            uint32_t above = lat[NV - 1] >> 24;
            for (int s = 0; s < n; ++s) {
                for (int t0 = 0; t0 < NT; t0 += 4) {
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        if (m % 2 == 0)
                            draw(g + (uint32_t)s, t0 + m);
                        const uint32_t cur = (lat[0] >> (8 * m)) & 0xFFu;
                        const uint32_t below = m < 3 ? (lat[0] >> (8 * (m < 3 ? m + 1 : 0))) & 0xFFu : lat[1 % NV] & 0xFFu;
                        const uint32_t now = attempt(cur, above, below, m & 1);
                        lat[0] ^= (cur ^ now) << (8 * m);
                        above = now;
                    }
                    // the registers turn: lat[0] always holds the next four tiles
                    const uint32_t done = lat[0];
#pragma unroll
                    for (int v = 0; v + 1 < NV; ++v)
                        lat[v] = lat[v + 1];
                    lat[NV - 1] = done;
                }
                count(b);
            }
        }
    }
};

// Copies the threshold table to LDS, 16 bytes per load: short launches wait
// for it (82 KB for Ising L = 64, 147 KB for Potts L = 48).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 gu32x4;

template <int MODEL>
__device__ __forceinline__ void stage_table(const uint32_t *T_, int n_bins, uint32_t *smem)
{
    constexpr int NC = Cols<MODEL>::value;
    const gu32 *T = (const gu32 *)T_;
    const int n = n_bins * NC, n4 = n / 4, step = (int)blockDim.x;
#pragma unroll 8
    for (int i = threadIdx.x; i < n4; i += step) {
        const u32x4 v = ((const gu32x4 *)T_)[i];
        if constexpr (MODEL != kPotts) {
            *(u32x4 *)(smem + 4 * i) = v;
        } else {
            uint32_t row = __umulhi((uint32_t)(4 * i), 0x38E38E39u) >> 1; // 4 i / 9
            uint32_t col = (uint32_t)(4 * i) - 9u * row;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (col != 4u) // dE = 0 is not staged
                    smem[8u * row + (uint32_t)potts_staged_slot((int)col)] = v[k];
                col = col == 8u ? 0u : col + 1u;
                row += col == 0u ? 1u : 0u;
            }
        }
    }
    for (int i = 4 * n4 + (int)threadIdx.x; i < n; i += step) {
        if constexpr (MODEL != kPotts) {
            smem[i] = T[i];
        } else if (i % 9 != 4) {
            smem[8 * (i / 9) + potts_staged_slot(i % 9)] = T[i];
        }
    }
}

// The workgroup's accepted moves.  They reach the run's one counter by one
// atomic per workgroup: those of all wavefronts, which end together, took 13
// ns each on that address (4096 chains of Ising L = 8, 10 sweeps: 65 us, of
// which 53 us were these).
__device__ __forceinline__ uint32_t *block_accepts()
{
    __shared__ uint32_t n;
    return &n;
}

// ---------------------------------------------------------------------------
// One block: wave w runs chain c_first + w (w < n_c).  The threshold table is
// staged in LDS once for all of them (TLDS), the sweeps are counted in packed
// 16-bit LDS counters that are added to the global histogram before any of
// them can overflow.
// ---------------------------------------------------------------------------
template <int MODEL, int L, bool TLDS>
__device__ __forceinline__ void tile_block(const LatticeArgs &a, int c_first, int n_c, uint32_t *smem)
{
    constexpr int NC = Cols<MODEL>::value, NCL = MODEL == kPotts ? 8 : NC;
    uint32_t *lhist = TLDS ? smem + a.n_bins * NCL : smem;
    const int hw = lds_hist_words(a.n_bins);
    for (int i = threadIdx.x; i < hw; i += blockDim.x)
        lhist[i] = 0u;
    uint32_t *accepted = block_accepts();
    if (threadIdx.x == 0)
        *accepted = 0u;
    int32_t tbase = 0;
    if constexpr (TLDS) {
        stage_table<MODEL>(a.thresholds, a.n_bins, smem);
        tbase = (int32_t)(uint32_t)(uintptr_t)(lds_u32 *)smem;
    }
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63u), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = c_first + wave;
    const bool active = wave < n_c && c < a.n_chains;
    gu64 *blk = a.hist_blocks ? (gu64 *)a.hist_blocks + (size_t)(c_first / a.hist_block_chains) * (size_t)a.n_bins
                              : nullptr;
    using Chain = std::conditional_t<MODEL == kPotts, PottsChain<L, TLDS>, SpinChain<MODEL, L, TLDS>>;
    Chain ch;
    int32_t b = 0;
    if (active) {
        ch.load(a, c, lane);
        b = __builtin_amdgcn_readfirstlane(((const gi32 *)a.bins)[c]);
    }
    const int flush_every = kMaxBlockCount / n_c;
    for_segments(a.n_sweeps, flush_every, [&](int32_t s0, int32_t n) {
        if (active) {
            uint32_t nacc = 0u;
            ch.sweeps(a, (uint32_t)(a.chain0 + c), a.g0 + (uint32_t)s0, n, lane, a.thresholds, tbase, b, nacc,
                      [&](int32_t bb) {
                          if (!a.record)
                              return;
                          if (lane == 0)
                              atomicAdd(&lhist[bb >> 1], 1u << ((bb & 1) << 4));
                          if constexpr (MODEL == kMuma) {
                              if (a.em) { // E = -2N + 2 unsatisfied = -2N + 4 e, e <= N
                                  const uint32_t e = min(ch.unsatisfied(lane) >> 1, (uint32_t)(L * L));
                                  if (lane == 0)
                                      gadd((gu64 *)a.em + (size_t)e * (size_t)a.n_bins + (size_t)bb, 1ull);
                              }
                          }
                      });
            if (a.record && lane == 0) // at most 65535 sweeps of 4096 sites over the workgroup: below 2^32
                atomicAdd(accepted, nacc);
        }
        __syncthreads();
        flush_hist(lhist, hw, a.hist, blk);
        if (threadIdx.x == 0) {
            if (a.accepts && *accepted)
                gadd((gu64 *)a.accepts, (unsigned long long)*accepted);
            *accepted = 0u;
        }
        __syncthreads();
    });
    if (active) {
        ch.store(a, c, lane);
        if (lane == 0)
            ((gi32 *)a.bins)[c] = b;
    }
}

// 1024 threads: sixteen chains share one staged table, four wavefronts per
// SIMD where the table leaves room for one block per CU.
template <int MODEL, int L, bool TLDS>
__global__ __launch_bounds__(1024) void lattice_tiles(LatticeArgs a)
{
    extern __shared__ __align__(16) uint32_t smem[];
    tile_block<MODEL, L, TLDS>(a, (int)blockIdx.x * a.tile_chains, a.tile_chains, smem);
}

template <int MODEL, int L>
static hipError_t launch_tiles(const LatticeArgs &a, hipStream_t s)
{
    const int chains = a.tile_chains;
    if (chains < 1 || chains > 16)
        return hipErrorInvalidValue;
    // a large table is staged by sixteen wavefronts, however few carry chains
    const size_t table = a.table_in_lds ? (size_t)a.n_bins * lds_table_cols(MODEL) * 4u : 0u;
    const int waves = table > 16384u ? 16 : chains;
    const dim3 grid((unsigned)((a.n_chains + chains - 1) / chains)), block((unsigned)(64 * waves));
    size_t lds = (size_t)lds_hist_words(a.n_bins) * 4u;
    if (a.table_in_lds) {
        lds += (size_t)a.n_bins * lds_table_cols(MODEL) * 4u;
        if (lds > 65536u) {
            hipError_t e = hipFuncSetAttribute((const void *)lattice_tiles<MODEL, L, true>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess)
                return e;
        }
        hipLaunchKernelGGL((lattice_tiles<MODEL, L, true>), grid, block, lds, s, a);
    } else {
        hipLaunchKernelGGL((lattice_tiles<MODEL, L, false>), grid, block, lds, s, a);
    }
    return hipGetLastError();
}

// One wavefront per chain, a.tile_chains of them per block.
template <int MODEL>
static hipError_t launch_tile_model(int L, const LatticeArgs &a, hipStream_t s)
{
    switch (L) {
    case 4: return launch_tiles<MODEL, 4>(a, s);
    case 8: return launch_tiles<MODEL, 8>(a, s);
    case 16: return launch_tiles<MODEL, 16>(a, s);
    case 24: return launch_tiles<MODEL, 24>(a, s);
    case 32: return launch_tiles<MODEL, 32>(a, s);
    case 48: return launch_tiles<MODEL, 48>(a, s);
    case 64: return launch_tiles<MODEL, 64>(a, s);
    default: return hipErrorInvalidValue;
    }
}

} // namespace muca
