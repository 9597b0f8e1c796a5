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
// sit earlier in the tile (left, and up where a tile has several rows), so
// the outcomes are 64-bit masks on the scalar unit and the dependence on
// those neighbours is resolved there, without further reads.  The lattice
// never leaves the registers during a launch: lane t holds tile t as a
// 64-bit mask (Ising, MUMA), or lane i holds its site's colour of every tile,
// four per register (Potts).
//
// Bound: instruction issue with four wavefronts per SIMD, latency (LDS reads,
// the scalar chain) below that.  Measured per iteration, before (16 lanes per
// chain, site by site) and after: Ising L = 64, 4096 chains, 400 sweeps
// 54.4 -> 23.0 ms; Ising L = 32 int8, 1000 chains, 35 sweeps 1.69 -> 0.46 ms;
// MUMA L = 32 with the joint histogram, 512 chains, 67 sweeps 2.85 -> 0.69 ms;
// Potts q = 8 L = 48, 2048 chains, 362 sweeps 39.4 -> 12.7 ms; Potts q = 10
// L = 64 (table in global memory), 1024 chains, 60 sweeps 14.5 -> 3.5 ms.
#pragma once
#include "lattice_impl.h"

namespace muca {

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

// ---------------------------------------------------------------------------
// Ising / MUMA
// ---------------------------------------------------------------------------
// Thresholds T[bin][first + k + j * stride], j = 0..n-1, n = 2 or 3.
template <int MODEL, bool TLDS, int n>
__device__ __forceinline__ void spin_thresholds(const uint32_t *T, int32_t tbase, int32_t bin, int32_t col,
                                                uint32_t (&t)[3])
{
    constexpr int NC = Cols<MODEL>::value, ST = MODEL == kIsing ? 1 : 2;
    const int32_t at = bin * (4 * NC) + col;
    if constexpr (TLDS) {
        lds_u32 *p = (lds_u32 *)(uintptr_t)(uint32_t)(tbase + at);
#pragma unroll
        for (int j = 0; j < n; ++j)
            t[j] = p[j * ST];
    } else {
        const gu32 *p = (const gu32 *)((uintptr_t)T + (uint32_t)at);
#pragma unroll
        for (int j = 0; j < n; ++j)
            t[j] = p[j * ST];
    }
}

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
    const int32_t plus = MODEL == kMuma ? (lane_bit(S) ? 4 : 0) : 0;

    uint64_t F = 0ull;  // accepted, as the last pass found it
    int32_t x = b;      // this lane's bin if F is right
    int32_t end = b;    // the bin after the tile if F is right
    for (;;) {
        // neighbours that the inner resolution does not follow: a row's last
        // site sees site 0 (its right neighbour) as this pass's F left it,
        // and the last row of a whole lattice the first one
        const uint64_t ar = AR ^ ((F << (L - 1)) & G::kLast);
        const uint64_t ad = G::kWhole ? AD ^ (F << UP) : AD;
        int32_t k = (lane_bit(ar) ? 1 : 0) + (lane_bit(ad) ? 1 : 0);
        if constexpr (R == 1)
            k += lane_bit(AU) ? 1 : 0;
        if (F) {
            if constexpr (MODEL == kIsing) {
                int32_t n = k - 2 + (lane_bit(AL ^ ((F << 1) & ~G::kFirst)) ? 1 : 0);
                if constexpr (R > 1)
                    n += lane_bit(AU ^ (F << L)) ? 1 : 0;
                n = lane_bit(F) ? n : 0;
                x = prefix_from(b, n);
                end = __builtin_amdgcn_readlane(x, TS - 1) + __builtin_amdgcn_readlane(n, TS - 1);
            } else {
                const uint64_t up = F & ~S, dn = F & S; // M grows where a -1 flips
                x = (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(up >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)up, (uint32_t)b));
                x -= (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(dn >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)dn, 0u));
                end = b + __builtin_popcountll(up) - __builtin_popcountll(dn);
            }
            // a wrong guess may leave the table; the answer cannot
            x = min(max(x, 0), n_bins - 1);
        }
        uint32_t t[3];
        const int32_t col = MODEL == kIsing ? 4 * k : 8 * k + plus;
        spin_thresholds<MODEL, TLDS, (R == 1 ? 2 : 3)>(T, tbase, x, col, t);
        // outcome by the number of aligned neighbours among left (and up)
        const uint64_t C0 = ballot(r < t[0]), C1 = ballot(r < t[1]);
        uint64_t A = F, A0;
        if constexpr (R == 1) {
            const uint64_t Q = C0 ^ C1, B = C0 ^ (AL & Q), D = Q & ~G::kFirst;
            do {
                A0 = A;
                A = B ^ (D & (A << 1));
            } while (A != A0);
        } else {
            const uint64_t Q1 = C0 ^ C1, Q2 = C0 ^ ballot(r < t[2]);
            do {
                A0 = A;
                const uint64_t l = AL ^ ((A << 1) & ~G::kFirst), u = AU ^ (A << L);
                A = C0 ^ ((l ^ u) & Q1) ^ ((l & u) & Q2);
            } while (A != A0);
        }
        if (A == F)
            break;
        F = A;
    }
    b = end;
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
    __device__ __forceinline__ void set_tile(int lane, int t, uint64_t m)
    {
        lo = lane == t ? (uint32_t)m : lo;
        hi = lane == t ? (uint32_t)(m >> 32) : hi;
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
                        set_tile(lane, 0, S);
                    count(b);
                }
            }
            set_tile(lane, 0, S);
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
                        set_tile(lane, t, P);
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
// (colour == old) - (colour == proposal): a neighbour's share of the change
// in unsatisfied bonds.
__device__ __forceinline__ int32_t potts_share(uint32_t colour, uint32_t old, uint32_t nw)
{
    return (colour == old ? 1 : 0) - (colour == nw ? 1 : 0);
}

// Threshold of the change dE from bin x.  Staged rows hold eight columns,
// dE = -4..-1, 1..4 (dE = 0 always accepts and is not read); rows in global
// memory nine.
template <bool TLDS>
__device__ __forceinline__ int32_t potts_col(int32_t dE)
{
    return TLDS ? 4 * (dE + 4 - (dE > 0 ? 1 : 0)) : 4 * (dE + 4);
}

template <bool TLDS>
__device__ __forceinline__ uint32_t potts_threshold(const uint32_t *T, int32_t row, int32_t col)
{
    return load_t<TLDS>(T, row + col);
}

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
    // shares of the neighbours before and after their own attempts in this
    // tile; a neighbour that the order visits later, or that lies outside
    // the tile, has one share
    const bool col0 = lane_bit(G::kFirst), row0 = lane < L;
    const int32_t l0 = potts_share(lf & 0xFFu, cur, p);
    const int32_t l1 = col0 ? l0 : potts_share((lf >> 8) & 0xFFu, cur, p);
    const int32_t u0 = potts_share(up & 0xFFu, cur, p);
    int32_t u1 = u0;
    if constexpr (R > 1)
        u1 = row0 ? u0 : potts_share((up >> 8) & 0xFFu, cur, p);
    const int32_t r0 = potts_share(rt & 0xFFu, cur, p), r1 = potts_share((rt >> 8) & 0xFFu, cur, p);
    const int32_t d0 = potts_share(dn & 0xFFu, cur, p);
    const int32_t d1 = G::kWhole ? potts_share((dn >> 8) & 0xFFu, cur, p) : d0;

    uint64_t F = 0ull, wrap_r = 0ull, wrap_d = 0ull;
    int32_t x = b, end = b;
    int32_t e[4], c[4];    // dE and column by (left, up) accepted: 00, 10, 01, 11
    uint64_t Z[4];         // dE = 0
    constexpr int NV = R > 1 ? 4 : 2;
    auto variants = [&]() {
        const int32_t s = (lane_bit(wrap_r) ? r1 : r0) + (G::kWhole && lane_bit(wrap_d) ? d1 : d0);
        e[0] = s + l0 + u0;
        e[1] = s + l1 + u0;
        if constexpr (R > 1) {
            e[2] = s + l0 + u1;
            e[3] = s + l1 + u1;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            c[v] = potts_col<TLDS>(e[v]);
            Z[v] = ballot(e[v] == 0) & G::kAll;
        }
    };
    variants();
    for (;;) {
        if (F) {
            // a row's last site sees site 0 as this pass's F left it, and
            // the last row of a whole lattice the first one
            const uint64_t wr = (F << (L - 1)) & G::kLast, wd = G::kWhole ? F << UP : 0ull;
            if (wr != wrap_r || wd != wrap_d) {
                wrap_r = wr;
                wrap_d = wd;
                variants();
            }
            const bool la = lane_bit(F << 1);
            int32_t n = la ? e[1] : e[0];
            if constexpr (R > 1) {
                const int32_t m = la ? e[3] : e[2];
                n = lane_bit(F << L) ? m : n;
            }
            n = lane_bit(F) ? n : 0;
            x = prefix_from(b, n);
            end = __builtin_amdgcn_readlane(x, TS - 1) + __builtin_amdgcn_readlane(n, TS - 1);
            x = min(max(x, 0), n_bins - 1); // a wrong guess may leave the table; the answer cannot
        }
        const int32_t row = TLDS ? tbase + 32 * x : 36 * x;
        uint32_t t[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
            t[v] = potts_threshold<TLDS>(T, row, c[v]);
        uint64_t C[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
            C[v] = ballot(r < t[v]) | Z[v];
        uint64_t A = F, A0;
        if constexpr (R == 1) {
            const uint64_t D = C[0] ^ C[1]; // no bit in column 0: one variant there
            do {
                A0 = A;
                A = C[0] ^ (D & (A << 1));
            } while (A != A0);
        } else {
            const uint64_t D1 = C[0] ^ C[1], D2 = C[0] ^ C[2], D3 = D1 ^ C[2] ^ C[3];
            do {
                A0 = A;
                const uint64_t l = A << 1, u = A << L;
                A = C[0] ^ (l & D1) ^ (u & (D2 ^ (l & D3)));
            } while (A != A0);
        }
        if (A == F)
            break;
        F = A;
    }
    b = end;
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
    int32_t tbase = 0;
    if constexpr (TLDS) {
        for (int i = threadIdx.x; i < a.n_bins * NCL; i += blockDim.x) {
            int src = i;
            if constexpr (MODEL == kPotts) { // the dE = 0 column is not staged
                const int cc = i & 7;
                src = (i >> 3) * 9 + cc + (cc >= 4 ? 1 : 0);
            }
            smem[i] = ((const gu32 *)a.thresholds)[src];
        }
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
    for (int s0 = 0; s0 < a.n_sweeps; s0 += flush_every) {
        const int n = min(flush_every, a.n_sweeps - s0);
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
            if (a.record && a.accepts && lane == 0 && nacc)
                gadd((gu64 *)a.accepts, (unsigned long long)nacc);
        }
        __syncthreads();
        flush_hist(lhist, hw, a.hist, blk);
        __syncthreads();
    }
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
    extern __shared__ uint32_t smem[];
    const int n_c = (int)(blockDim.x >> 6);
    tile_block<MODEL, L, TLDS>(a, (int)blockIdx.x * n_c, n_c, smem);
}

template <int MODEL, int L>
static hipError_t launch_tiles(int chains, const LatticeArgs &a, hipStream_t s)
{
    if (chains < 1 || chains > 16)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((a.n_chains + chains - 1) / chains)), block((unsigned)(64 * chains));
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

// One wavefront per chain, `chains` of them per block.
template <int MODEL>
static hipError_t launch_tile_model(int L, int chains, const LatticeArgs &a, hipStream_t s)
{
    switch (L) {
    case 4: return launch_tiles<MODEL, 4>(chains, a, s);
    case 8: return launch_tiles<MODEL, 8>(chains, a, s);
    case 16: return launch_tiles<MODEL, 16>(chains, a, s);
    case 24: return launch_tiles<MODEL, 24>(chains, a, s);
    case 32: return launch_tiles<MODEL, 32>(chains, a, s);
    case 48: return launch_tiles<MODEL, 48>(chains, a, s);
    case 64: return launch_tiles<MODEL, 64>(chains, a, s);
    default: return hipErrorInvalidValue;
    }
}

} // namespace muca
