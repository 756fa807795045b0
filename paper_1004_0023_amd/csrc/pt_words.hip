// pt_words.hip -- sweeps of tiles of replicas whose shape the power-of-two kernels do not
// take, for both encodings: any slice count, any couplings (fields up to the library's
// bound), M = 1 and M = 2, and bit-packed instances the octet kernels do not take.
//
// A tile's replicas are held in LDS as words of four spins (one byte each) that one lane
// updates together:
//   slices (M >= 4)  word (q, p, i, g): slices 4g .. 4g + 3 of one parity of site i of
//                    replica q, which one Philox call serves; rows are padded to whole
//                    words, the padding stays 0 and is never flipped
//   replicas (M <= 2) word (Q, p, i): replicas 4Q .. 4Q + 3 at one slice of site i, four
//                    Philox calls (each attempt's draw is word 0 of its own call)
// The spins are expanded from either encoding when a tile is staged and packed again when it
// is written back, so the sweep itself is the same for both.
//
// Measured on MI355X, us per cycle of 10 sweeps and an exchange, the one-byte-at-a-time kernel
// or a launch per colour class -> word tiles, a launch per cycle -> many cycles a launch: 16
// lattices of 10^3 spins at M = 1, 32 replicas, 149 -> 32 -> 27; 8 instances of 201 spins at
// M = 100, 27 replicas, 262 -> 65 -> 54; 16 packed instances of 128 spins at M = 64 with
// couplings up to 3, 48 replicas, 760 -> 89 -> 82.
//
// Its operations are, per word, about 37 of Philox, 2 to 3 per neighbour, 5 for the table index
// and 4.5 per attempt for lookup, compare and merge (28 lane-operations an attempt in the packed
// batch above, 78 at M = 1).  What bounds it is not their number alone: the units that hold tiles
// issue VALU on 59 to 69 % of the slots in the packed batch and on 39 % at M = 1, and the waves
// wait the rest, since a class step is one pass of the workgroup and so a barrier, a chain of LDS
// trips and ten Philox rounds in series.  The time
// neighbours of every word come from one v_perm whose selector, fixed per thread, also does
// the wrap at the ends of a row, so slice counts that are not a multiple of eight cost
// nothing more.
//
// Table index (x (2F + 1) + f + F) 3 + tau, formed for the word's four spins at once:
//   narrow  F <= 20: in bytes (at most 245)
//   middle  F <= 63: x (2F + 1) + f + F in bytes (at most 253), the rest per attempt
//   wide    else:    in two pairs of 16-bit halves (at most 12,281)
#include <utility>

#include "pt_exchange.h"
#include "pt_internal.h"

#pragma clang fp contract(off)

namespace ptq {
namespace {

constexpr int kWave = 64;
constexpr int kWaitVmcnt0 = 0x0F70;                 // s_waitcnt: vector-memory count 0 only

template <int V>
struct IntC {
    static constexpr int value = V;
};

// Replicas per word, and words between the tile's units (replicas, or quads of replicas).
// The stride is padded so that it is congruent to a row's words modulo 64: the lanes of a
// wave run over (unit, group) with groups fastest, and the units then start on different
// banks.
__host__ __device__ __forceinline__ int words_rpw(const InstDesc &d) { return d.M <= 2 ? 4 : 1; }
__host__ __device__ __forceinline__ int words_row(const InstDesc &d) { return d.M <= 2 ? 1 : d.G4; }
__host__ __device__ __forceinline__ int words_units(const InstDesc &d, int P)
{
    return d.M <= 2 ? (P + 3) / 4 : P;
}
__host__ __device__ __forceinline__ int64_t words_stride(const InstDesc &d)
{
    const int64_t row = words_row(d);
    int64_t w = (int64_t)d.parities * d.N * row;
    if (row < 64) w += ((row - w) % 64 + 64) % 64;
    return w;
}

struct WordsOffsets {
    int64_t sp, ent, bias, csite, coff, tbl, red, end;
};

__host__ __device__ __forceinline__ WordsOffsets words_offsets(const InstDesc &d, int P)
{
    auto up = [](int64_t x) { return (x + 15) & ~(int64_t)15; };
    const int64_t units = words_units(d, P), reps = units * words_rpw(d);
    WordsOffsets o;
    o.sp = 0;
    o.ent = up(units * words_stride(d) * 4);
    o.bias = up(o.ent + (int64_t)d.N * d.D * 4);
    o.csite = up(o.bias + (int64_t)d.N * 4);
    o.coff = up(o.csite + (int64_t)d.N * 2);
    o.tbl = up(o.coff + (int64_t)(d.n_colors + 1) * 4);
    o.red = up(o.tbl + reps * d.tbl_words * 4);
    o.end = up(o.red + reps * 2 * 8 + 8);
    return o;
}

struct WordsLds {
    uint8_t *sp;
    const uint32_t *ent, *bias;
    const uint16_t *csite;
    const int32_t *coff;
    const uint32_t *tbl;
};

__device__ __forceinline__ uint32_t lds32(const uint8_t *base, uint32_t off)
{
    return *reinterpret_cast<const uint32_t *>(base + off);
}

// Division by a number fixed per launch, of dividends below 2^32 / d (here both are below
// the 2^16 words of LDS): one product instead of some twenty-five operations.
struct Div {
    uint32_t m;
    int d;
    __device__ __forceinline__ explicit Div(int d_) : m(0xFFFFFFFFu / (uint32_t)d_ + 1u), d(d_) {}
    __device__ __forceinline__ int operator()(int x) const { return d == 1 ? x : (int)__umulhi((uint32_t)x, m); }
};

// ------------------------------------------------------------------ one word

// Per launch, and per thread (its unit and group are fixed).
struct Args {
    uint32_t key0, key1, n;
    uint32_t plane, row;  // bytes of one parity of a unit, of a row
    uint32_t sel_x;       // v_perm selector: x -> x (2F + 1) (narrow, middle)
    uint32_t xstep;       // 2F + 1
    uint32_t ctr_site;    // Philox counter words per site (2 G4)
    int D, G4, tbl_words;
};

struct Lane {
    uint32_t base;        // byte of the lane's word in row 0, parity 0
    int32_t prev, next;   // bytes to the words before and after it in its row (cyclic)
    uint32_t sel0, sel1;  // selectors of the time neighbours of parity 0 and 1
    uint32_t valid;       // 1 in every byte that holds a spin
    uint32_t g;           // its group
    const uint32_t *tb;   // its (first) replica's table
};

// Weighted neighbour counts of a word's four spins: bytes (a0), or the even bytes' counts in
// the halves of a0 and the odd bytes' in those of a1 (wide).
template <int DT, int MODE>
__device__ __forceinline__ void field(const Args &a, const WordsLds &t, uint32_t at, int i, uint32_t &a0,
                                      uint32_t &a1)
{
    a0 = a1 = 0;
    auto add = [&](uint32_t e, uint32_t y) {
        const uint32_t w = __builtin_amdgcn_perm(0u, e, y);
        if constexpr (MODE == kWordsWide) {
            a0 += w & 0x00FF00FFu;
            a1 += (w >> 8) & 0x00FF00FFu;
        } else {
            a0 += w;
        }
    };
    if constexpr (DT > 0) {
        uint32_t e[DT], y[DT];
#pragma unroll
        for (int k = 0; k < DT; ++k) e[k] = t.ent[i * DT + k];
#pragma unroll
        for (int k = 0; k < DT; ++k) y[k] = lds32(t.sp, at + __umul24(e[k] >> 16, a.row));
#pragma unroll
        for (int k = 0; k < DT; ++k) add(e[k], y[k]);
    } else {
#pragma unroll 4
        for (int k = 0; k < a.D; ++k) {
            const uint32_t e = t.ent[i * a.D + k];
            add(e, lds32(t.sp, at + __umul24(e >> 16, a.row)));
        }
    }
}

// Table index of spin b of a word from its counts, spins X and time fields T.
template <int MODE>
struct Index {
    uint32_t i0, i1, T;
    __device__ __forceinline__ Index(const Args &a, uint32_t X, uint32_t a0, uint32_t a1, uint32_t T_,
                                     uint32_t bias)
        : i0(0), i1(0), T(T_)
    {
        if constexpr (MODE == kWordsWide) {
            const uint32_t v0 = __umul24(X & 0x00010001u, a.xstep) + (a0 << 1) + bias;
            const uint32_t v1 = __umul24((X >> 8) & 0x00010001u, a.xstep) + (a1 << 1) + bias;
            i0 = v0 + (v0 << 1) + (T & 0x00FF00FFu);
            i1 = v1 + (v1 << 1) + ((T >> 8) & 0x00FF00FFu);
        } else {
            i0 = __builtin_amdgcn_perm(0u, a.sel_x, X) + (a0 << 1) + bias;
            if constexpr (MODE == kWordsNarrow) i0 = i0 + (i0 << 1) + T;
        }
    }
    __device__ __forceinline__ uint32_t at(int b) const
    {
        if constexpr (MODE == kWordsWide)
            return ((b & 1 ? i1 : i0) >> (b & 2 ? 16 : 0)) & 0xFFFFu;
        else if constexpr (MODE == kWordsMiddle)
            return ((i0 >> (8 * b)) & 0xFFu) * 3u + ((T >> (8 * b)) & 0xFFu);
        else
            return (i0 >> (8 * b)) & 0xFFu;
    }
};

// The four attempts of the lane's word at site i, parity PAR.  RM: the word holds replicas;
// nr of them are in use (uniform), r[k] are their shared draws.
template <int DT, int PAR, int MODE, bool RM>
__device__ __forceinline__ void item(const Args &a, const WordsLds &t, const Lane &ln, const Draws *r,
                                     int nr, bool timed, int i)
{
    const uint32_t irow = __umul24((uint32_t)i, a.row);
    const uint32_t plane = ln.base + (uint32_t)PAR * a.plane;
    const uint32_t own = plane + irow, oth = ln.base + (uint32_t)(PAR ^ 1) * a.plane + irow;
    const uint32_t X = lds32(t.sp, own);
    uint32_t T;
    if constexpr (RM) {
        T = timed ? 2u * lds32(t.sp, oth) : 0x01010101u;  // M = 2: both neighbours are the other slice
    } else {
        const uint32_t W = lds32(t.sp, oth);
        const uint32_t Wx = lds32(t.sp, oth + (uint32_t)(PAR == 0 ? ln.prev : ln.next));
        T = __builtin_amdgcn_perm(W, Wx, PAR == 0 ? ln.sel0 : ln.sel1) + W;
    }
    uint32_t a0, a1;
    field<DT, MODE>(a, t, plane, i, a0, a1);
    const Index<MODE> idx(a, X, a0, a1, T, t.bias[i]);
    const SiteDraws s = site_draws(__umul24((uint32_t)i, a.ctr_site) + (uint32_t)(PAR * a.G4) + ln.g, a.n, a.key0, a.key1);
    uint32_t flip = 0;
    if constexpr (RM) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b < nr) {
                const uint32_t thr = ln.tb[b * a.tbl_words + idx.at(b)];
                flip |= (philox_draw<false>(r[b], s, a.key0, a.key1).w[0] <= thr ? 1u : 0u) << (8 * b);
            }
        }
    } else {
        const Words4 u = philox_draw<false>(r[0], s, a.key0, a.key1);
#pragma unroll
        for (int b = 0; b < 4; ++b) flip |= (u.w[b] <= ln.tb[idx.at(b)] ? 1u : 0u) << (8 * b);
    }
    *reinterpret_cast<uint32_t *>(t.sp + own) = X ^ (flip & ln.valid);
}

// ------------------------------------------------------------------ a tile

struct Tid {
    int s, rows;  // the thread's first site of a class, and the sites a pass covers
};

template <int DT, int MODE, bool RM>
__device__ __forceinline__ void sweeps(const SweepLaunch &L, const InstDesc &d, const Tile &tile,
                                       const WordsLds &t, const Args &a, const Lane &ln, const Tid &id,
                                       uint32_t c, uint64_t t0)
{
    constexpr int NR = RM ? 4 : 1;
    const int nr = min(tile.P, NR);
    const bool timed = d.M >= 2;
    const int nc = d.n_colors;
    auto draws = [&](Draws (&r)[NR], uint64_t tt) {
#pragma unroll
        for (int k = 0; k < NR; ++k) r[k] = draws_of((uint32_t)tt, c + (uint32_t)k, a.key0, a.key1);
    };
    auto cls = [&](auto par, const Draws (&r)[NR], int g) {
        const int s1 = t.coff[g + 1];
        for (int si = t.coff[g] + id.s; si < s1; si += id.rows)
            item<DT, decltype(par)::value, MODE, RM>(a, t, ln, r, nr, timed, t.csite[si]);
    };
    Draws ra[NR], rb[NR];
    if (!timed || nc < 2) {
        for (int sw = 0; sw < L.n_sweeps; ++sw) {
            draws(ra, t0 + (uint64_t)sw);
            for (int g = 0; g < nc; ++g) {
                cls(IntC<0>{}, ra, g);
                __syncthreads();
            }
            for (int g = 0; g < nc && timed; ++g) {
                cls(IntC<1>{}, ra, g);
                __syncthreads();
            }
        }
        return;
    }
    // class k of parity 0 with class k - 1 of parity 1 (from the previous sweep when k = 0):
    // they share no site, and each reads the other parity only at its own sites, so one
    // barrier closes both and every update reads what it reads in the plain order
    for (int sw = 0; sw <= L.n_sweeps; ++sw) {
        const bool tail = sw == L.n_sweeps;
        if (!tail) draws(ra, t0 + (uint64_t)sw);
        for (int k = 0; k < (tail ? 1 : nc); ++k) {
            if (k == 1)
                for (int j = 0; j < NR; ++j) rb[j] = ra[j];
            if (!tail) cls(IntC<0>{}, ra, k);
            if (k > 0 || sw > 0) cls(IntC<1>{}, rb, k > 0 ? k - 1 : nc - 1);
            __syncthreads();
        }
    }
}

// 2 E_cl and C of the tile's replicas, summed per replica in red[2 q], red[2 q + 1] (zeroed).
// 2E = sum_i s_i (f_i + h_i) with f + F from the weighted counts as in the sweep; sumJ comes
// from the entries (their two weight bytes sum to |J|).  A lane takes both parities of a
// word, so that a neighbour's entry is read once.
template <int MODE, bool RM>
__device__ __forceinline__ void energy(const InstDesc &d, const Tile &tile, const WordsLds &t, const Args &a,
                                       unsigned long long *red)
{
    const int row = words_row(d), units = words_units(d, tile.P), stride = (int)words_stride(d);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const int wpu = nw > units ? nw / units : 1, ngroups = nw / wpu;
    const int grp = wid / wpu, sub = wid - grp * wpu;
    const bool timed = d.M >= 2;
    const Div by_row(row);
    constexpr int NR = RM ? 4 : 1;
    for (int q = grp; q < units && grp < ngroups; q += ngroups) {
        // 32 bits hold a wave's sums: |2E| and |C| of a replica in LDS are below 2^30
        int e2[NR], cc[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) e2[k] = cc[k] = 0;
        const int items = d.N * row;
        for (int it = sub * kWave + lane; it < items; it += wpu * kWave) {
            const int i = RM ? it : by_row(it), g = RM ? 0 : it - i * row;
            const uint32_t base = 4u * (uint32_t)(q * stride + g), irow = __umul24((uint32_t)i, a.row);
            uint32_t X[2], a0[2] = {0u, 0u}, a1[2] = {0u, 0u}, sumJ = 0;
            X[0] = lds32(t.sp, base + irow);
            X[1] = timed ? lds32(t.sp, base + a.plane + irow) : 0u;
#pragma unroll 4
            for (int k = 0; k < a.D; ++k) {
                const uint32_t e = t.ent[i * a.D + k], at = base + __umul24(e >> 16, a.row);
                const uint32_t y[2] = {lds32(t.sp, at), lds32(t.sp, timed ? at + a.plane : at)};
                sumJ = __builtin_amdgcn_udot4(e, 0x00000101u, sumJ, false);
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const uint32_t w = __builtin_amdgcn_perm(0u, e, y[p]);
                    if constexpr (MODE == kWordsWide) {
                        a0[p] += w & 0x00FF00FFu;
                        a1[p] += (w >> 8) & 0x00FF00FFu;
                    } else {
                        a0[p] += w;
                    }
                }
            }
            const uint32_t bias = t.bias[i];
            const int b0 = (int)(bias & (MODE == kWordsWide ? 0xFFFFu : 0xFFu));
            const int hF = b0 + (int)sumJ - 2 * d.F;  // h - F
            const int left = RM ? 4 : d.Mh - 4 * g, nv = left < 4 ? left : 4;
            const uint32_t vm = 0x01010101u >> (8 * (4 - nv));
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if (p > 0 && !timed) break;
                if constexpr (!RM && MODE != kWordsWide) {
                    const uint32_t G = (a0[p] << 1) + bias;  // f + F of every spin
                    e2[0] += 2 * (int)__builtin_amdgcn_udot4(X[p], G, 0u, false) + 2 * hF * __popc(X[p]) -
                             (int)__builtin_amdgcn_udot4(vm, G, 0u, false) - nv * hF;
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        if (b >= nv) break;
                        const int cnt = MODE == kWordsWide ? (int)(((b & 1 ? a1[p] : a0[p]) >> (b & 2 ? 16 : 0)) & 0xFFFFu)
                                                           : (int)((a0[p] >> (8 * b)) & 0xFFu);
                        const int sgn = 2 * (int)((X[p] >> (8 * b)) & 1u) - 1;
                        e2[RM ? b : 0] += sgn * (2 * cnt + b0 + hF);
                    }
                }
            }
            if (timed) {
                // bonds (2m, 2m + 1) and (2m + 1, 2m + 2): parity 0 at the next slice
                if constexpr (RM) {
                    const uint32_t diff = X[0] ^ X[1];
#pragma unroll
                    for (int b = 0; b < 4; ++b) cc[b] += 2 - 4 * (int)((diff >> (8 * b)) & 1u);
                } else {
                    const int gn = g + 1 == row ? 0 : g + 1;
                    const uint32_t nx = __builtin_amdgcn_perm(
                        X[0], lds32(t.sp, 4u * (uint32_t)(q * stride + gn) + irow),
                        nv == 4 ? 0x00070605u : nv == 3 ? 0x0C000605u : nv == 2 ? 0x0C0C0005u : 0x0C0C0C00u);
                    cc[0] += 2 * nv - 2 * (__popc(X[0] ^ X[1]) + __popc(X[1] ^ nx));
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            int e = e2[k], c = cc[k];
#pragma unroll
            for (int o = kWave / 2; o > 0; o >>= 1) {
                e += __shfl_xor(e, o, kWave);
                c += __shfl_xor(c, o, kWave);
            }
            if (lane == 0) {
                atomicAdd(&red[2 * (NR * q + k)], (unsigned long long)(long long)e);
                atomicAdd(&red[2 * (NR * q + k) + 1], (unsigned long long)(long long)c);
            }
        }
    }
}

// ------------------------------------------------------------------ staging

__device__ __forceinline__ uint32_t spread4(uint32_t v) { return (v * 0x00204081u) & 0x01010101u; }

// A tile starts with half a dozen arrays to stage, each a trip to memory that no cache of
// this launch holds yet.  Every array's first K elements per thread are therefore loaded
// before any is stored (indexes past the end are clamped, so that no load is under a branch
// and waited for there); the rest follow K at a time.
template <int K, class Load>
struct Staged {
    decltype(std::declval<Load>()(0)) v[K];
    Load load;
    int count;
    __device__ __forceinline__ Staged(int n, Load f) : load(f), count(n)
    {
#pragma unroll
        for (int u = 0; u < K; ++u) v[u] = load(min((int)threadIdx.x + u * (int)blockDim.x, count - 1));
    }
    template <class Store>
    __device__ __forceinline__ void put(Store &&store)
    {
        const int nt = blockDim.x;
        for (int at = threadIdx.x;;) {
#pragma unroll
            for (int u = 0; u < K; ++u)
                if (at + u * nt < count) store(at + u * nt, v[u]);
            at += K * nt;
            if (at >= count) break;
#pragma unroll
            for (int u = 0; u < K; ++u) v[u] = load(min(at + u * nt, count - 1));
        }
    }
};

// The tile's replicas in the byte encoding, as LDS words: word x of all of them.
template <bool RM>
struct LoadBytes {
    const uint8_t *dev;
    int rep_bytes, G4, Mh, P;
    Div by_unit, by_row;  // words of a unit, of a row
    __device__ __forceinline__ uint32_t operator()(int x) const
    {
        const int q = by_unit(x), w = x - q * by_unit.d;
        if constexpr (RM) {
            // the four bytes are one position of four replicas (past the last one: its own)
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t y = dev[(int64_t)min(4 * q + b, P - 1) * rep_bytes + w];
                v |= (4 * q + b < P ? y : 0u) << (8 * b);
            }
            return v;
        } else {
            const uint32_t *rep = reinterpret_cast<const uint32_t *>(dev + (int64_t)q * rep_bytes);
            if ((Mh & 3) == 0) return rep[w];
            // a row of Mh bytes need not start at a word: two words joined, the padding cleared
            const int r = by_row(w), m = 4 * (w - r * G4), at = r * Mh + m, nv = min(Mh - m, 4);
            const uint32_t lo = rep[at >> 2], hi = rep[min((at >> 2) + 1, (rep_bytes >> 2) - 1)];
            return __builtin_amdgcn_alignbyte(hi, lo, (uint32_t)(at & 3)) & (0xFFFFFFFFu >> (8 * (4 - nv)));
        }
    }
};

// LDS words of byte-encoded replicas back to device memory.
template <bool RM>
__device__ __forceinline__ void store_bytes(const DevState &st, const InstDesc &d, const Tile &tile, const uint8_t *sp)
{
    uint8_t *dev = st.spins + d.spin_base + (int64_t)tile.c0 * d.rep_bytes;
    const int stride = (int)words_stride(d);
    if constexpr (RM) {
        const int pos = d.parities * d.N, units = words_units(d, tile.P);
        const Div by_unit(pos);
        for (int it = threadIdx.x; it < pos * units; it += blockDim.x) {
            const int Q = by_unit(it), x = it - Q * pos;
            const uint32_t v = reinterpret_cast<const uint32_t *>(sp)[Q * stride + x];
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (4 * Q + b < tile.P) dev[(int64_t)(4 * Q + b) * d.rep_bytes + x] = (uint8_t)(v >> (8 * b));
        }
        return;
    }
    const int words = (d.N * d.M + 3) >> 2;  // of a replica in device memory
    const int rows = 2 * d.N;
    const Div by_half(d.Mh);
    for (int q = 0; q < tile.P; ++q) {
        const uint8_t *l = sp + 4 * (int64_t)q * stride;
        uint32_t *g = reinterpret_cast<uint32_t *>(dev + (int64_t)q * d.rep_bytes);
        for (int w = threadIdx.x; w < words; w += blockDim.x) {
            if ((d.Mh & 3) == 0) {
                g[w] = reinterpret_cast<const uint32_t *>(l)[w];
                continue;
            }
            int rw = by_half(4 * w), m = 4 * w - rw * d.Mh;
            uint32_t v = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (rw < rows) v |= (uint32_t)l[rw * 4 * d.G4 + m] << (8 * b);
                if (++m == d.Mh) {
                    m = 0;
                    ++rw;
                }
            }
            g[w] = v;
        }
    }
}

// Bit-packed replicas (all within one word group): the words of a four-slice group are one
// 16-byte load for all the tile's replicas.
struct LoadBits {
    const uint4 *dev;
    __device__ __forceinline__ uint4 operator()(int x) const { return dev[x]; }
};

template <bool RM>
__device__ __forceinline__ void put_bits(const InstDesc &d, const Tile &tile, uint32_t *l, int x, const uint4 &v)
{
    const int stride = (int)words_stride(d), c = tile.c0 & 31;
    if constexpr (RM) {
        for (int Q = 0; 4 * Q < tile.P; ++Q) {
            const int nv = min(4, tile.P - 4 * Q);
            l[Q * stride + x] = spread4((v.x >> (c + 4 * Q)) & ((1u << nv) - 1u));
        }
    } else {
        for (int q = 0; q < tile.P; ++q) {
            const int sh = c + q;
            l[q * stride + x] = ((v.x >> sh) & 1u) | ((v.y >> sh) & 1u) << 8 | ((v.z >> sh) & 1u) << 16 |
                                ((v.w >> sh) & 1u) << 24;
        }
    }
}

// And back.  Other tiles hold other bits of the same words, so the bits that changed are
// flipped with atomic xors.
template <bool RM>
__device__ __forceinline__ void store_bits(const InstDesc &d, const Tile &tile, const uint32_t *l, uint32_t *dev,
                                           int x, const uint4 &v)
{
    const int stride = (int)words_stride(d), c = tile.c0 & 31;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    if constexpr (RM) {
        uint32_t now = 0, mask = 0;
        for (int Q = 0; 4 * Q < tile.P; ++Q) {
            const int sh = c + 4 * Q, nv = min(4, tile.P - 4 * Q);
            const uint32_t y = l[Q * stride + x];
            now |= ((y | (y >> 7) | (y >> 14) | (y >> 21)) & 0xFu) << sh;
            mask |= ((1u << nv) - 1u) << sh;
        }
        const uint32_t diff = (w[0] ^ now) & mask;
        if (diff) atomicXor(dev + 4 * (int64_t)x, diff);
    } else {
        uint32_t diff[4] = {0u, 0u, 0u, 0u};
        for (int q = 0; q < tile.P; ++q) {
            const uint32_t y = l[q * stride + x];
#pragma unroll
            for (int b = 0; b < 4; ++b) diff[b] |= (((y >> (8 * b)) ^ (w[b] >> (c + q))) & 1u) << (c + q);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (diff[b]) atomicXor(dev + 4 * (int64_t)x + b, diff[b]);
    }
}

// RM: replicas in a word (M <= 2).  COOP: L.cycles PT cycles with every tile resident, the
// arrays staged once and the exchange step in the launch (coop_cycle): 216 replicas of 201 x
// 100 spins took 65.3 us a cycle of 10 sweeps with a launch per cycle and take 54.0, 512 of
// 10^3 x 1 spins 32.1 and 26.6.  Its own instantiation, at four waves per SIMD: at eight the
// loop with the exchange step in it spills (62.4 us and 31.3 with the same tiles); the form for
// M <= 2 spills at four as well (148 registers).
template <bool RM, bool COOP>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(COOP ? 4 : 8))) sweep_words_kernel(SweepLaunch L)
{
    extern __shared__ __align__(16) char lds[];
    const DevState &st = L.st;
    const Tile tile = st.tiles[L.tile0 + blockIdx.x];
    const int n = tile.inst;
    const InstDesc d = st.inst[n];
    const WordsOffsets o = words_offsets(d, tile.P);
    uint8_t *sp = reinterpret_cast<uint8_t *>(lds);
    uint32_t *ent = reinterpret_cast<uint32_t *>(lds + o.ent), *bias = reinterpret_cast<uint32_t *>(lds + o.bias);
    uint16_t *csite = reinterpret_cast<uint16_t *>(lds + o.csite);
    int32_t *coff = reinterpret_cast<int32_t *>(lds + o.coff);
    uint32_t *tbl = reinterpret_cast<uint32_t *>(lds + o.tbl);
    unsigned long long *red = reinterpret_cast<unsigned long long *>(lds + o.red);
    const int tid = threadIdx.x, nt = blockDim.x;
    const bool packed = d.bp_row != 0;

    const int units = words_units(d, tile.P), pos = d.parities * d.N * words_row(d), stride = (int)words_stride(d);
    uint32_t *packed_dev = reinterpret_cast<uint32_t *>(st.spins + d.spin_base) +
                           (int64_t)(tile.c0 >> 5) * d.parities * d.N * d.bp_row;
    const LoadBits load_bits = {reinterpret_cast<const uint4 *>(packed_dev)};
    {
        auto table_at = [&](int k) {
            const int q = k / d.tbl_words;
            return d.tbl_base + (int64_t)st.rung_of[d.rep_base + tile.c0 + q] * d.tbl_words + (k - q * d.tbl_words);
        };
        const int n_tbl = tile.P * d.tbl_words;
        auto load_tbl = [&](int k) { return st.tbl[table_at(k)]; };
        // the first table addresses (which wait for the rungs) ahead of everything else
        Staged<2, decltype(load_tbl)> s_tbl(n_tbl, load_tbl);
        auto load_ent = [&](int e) { return st.ent[d.ent_base + e]; };
        Staged<2, decltype(load_ent)> s_ent(d.N * d.D, load_ent);
        auto load_bias = [&](int i) { return st.bias[d.site_base + i]; };
        Staged<1, decltype(load_bias)> s_bias(d.N, load_bias);
        auto load_site = [&](int i) { return st.csite[d.site_base + i]; };
        Staged<1, decltype(load_site)> s_site(d.N, load_site);
        auto load_cls = [&](int g) { return st.cls_off[d.cls_base + g]; };
        Staged<1, decltype(load_cls)> s_cls(d.n_colors + 1, load_cls);
        auto put_rest = [&]() __attribute__((always_inline)) {
            s_ent.put([&](int e, uint32_t v) { ent[e] = v; });
            s_bias.put([&](int i, uint32_t v) { bias[i] = v; });
            s_site.put([&](int i, uint16_t v) { csite[i] = v; });
            s_cls.put([&](int g, int32_t v) { coff[g] = v; });
            s_tbl.put([&](int k, uint32_t v) { tbl[k] = v; });
        };
        if (packed) {
            Staged<4, LoadBits> s_sp(pos, load_bits);
            put_rest();
            s_sp.put([&](int x, const uint4 &v) {
                put_bits<RM>(d, tile, reinterpret_cast<uint32_t *>(sp), x, v);
            });
        } else {
            const Div by_unit(pos), by_row(d.G4);
            const LoadBytes<RM> load = {st.spins + d.spin_base + (int64_t)tile.c0 * d.rep_bytes, d.rep_bytes,
                                        d.G4, d.Mh, tile.P, by_unit, by_row};
            Staged<RM ? 2 : 6, LoadBytes<RM>> s_sp(units * pos, load);
            put_rest();
            s_sp.put([&](int x, uint32_t v) {
                const int q = by_unit(x);
                reinterpret_cast<uint32_t *>(sp)[q * stride + x - q * pos] = v;
            });
        }
    }
    for (int k = tid; k < 2 * units * words_rpw(d); k += nt) red[k] = 0;
    uint64_t t0 = st.ctr[n].t;
    __syncthreads();

    const WordsLds t = {sp, ent, bias, csite, coff, tbl};
    Args a;
    a.key0 = L.key0;
    a.key1 = L.key1;
    a.n = (uint32_t)n;
    const int row = words_row(d);
    a.row = 4u * (uint32_t)row;
    a.plane = a.row * (uint32_t)d.N;
    a.xstep = (uint32_t)(2 * d.F + 1);
    a.sel_x = a.xstep << 8;
    a.ctr_site = 2u * (uint32_t)d.G4;
    a.D = d.D;
    a.G4 = d.G4;
    a.tbl_words = d.tbl_words;
    // lanes run over (unit, group), groups fastest; each keeps its own and strides over the
    // sites of a class, threads past the last whole row of lanes stay idle
    const int lanes = units * row;  // at most nt (the host's choice of P)
    Tid id;
    id.rows = nt / lanes;
    id.s = tid / lanes;
    const int r = tid - id.s * lanes;
    if (id.s >= id.rows) id.s = 1 << 30;
    const int unit = r / row, g = r - unit * row;
    Lane ln;
    ln.base = 4u * (uint32_t)(unit * (int)words_stride(d) + g);
    ln.g = (uint32_t)g;
    ln.prev = 4 * ((g == 0 ? row - 1 : g - 1) - g);
    ln.next = 4 * ((g + 1 == row ? 0 : g + 1) - g);
    ln.sel0 = 0x06050400u | (uint32_t)(g == 0 ? (d.Mh - 1) & 3 : 3);
    const int left = RM ? tile.P - 4 * unit : d.Mh - 4 * g, nv = left < 4 ? left : 4;
    // parity 1 in a row's last word: the wrapped spin follows the row's last one
    ln.sel1 = nv == 4 ? 0x00070605u : nv == 3 ? 0x0C000605u : nv == 2 ? 0x0C0C0005u : 0x0C0C0C00u;
    ln.valid = nv == 4 ? 0x01010101u : 0x01010101u >> (8 * (4 - nv));
    ln.tb = tbl + (RM ? 4 * unit : unit) * d.tbl_words;
    const uint32_t c = (uint32_t)(tile.c0 + (RM ? 4 * unit : unit));

    auto run = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        auto with = [&](auto dt) {
            constexpr int DT = MODE == kWordsWide ? 0 : decltype(dt)::value;
            sweeps<DT, MODE, RM>(L, d, tile, t, a, ln, id, c, t0);
        };
        switch (d.D) {
        case 3: with(IntC<3>{}); break;
        case 4: with(IntC<4>{}); break;
        case 5: with(IntC<5>{}); break;
        case 6: with(IntC<6>{}); break;
        case 7: with(IntC<7>{}); break;
        case 8: with(IntC<8>{}); break;
        default: with(IntC<0>{}); break;
        }
        energy<MODE, RM>(d, tile, t, a, red);
    };
    for (int cyc = 0;; ++cyc) {
        switch (d.words) {
        case kWordsNarrow: run(IntC<kWordsNarrow>{}); break;
        case kWordsMiddle: run(IntC<kWordsMiddle>{}); break;
        default: run(IntC<kWordsWide>{}); break;
        }
        __syncthreads();
        for (int q = tid; q < tile.P; q += nt) {
            // coherently for the whole device: the exchange step of this launch may read them
            __hip_atomic_store(&st.E[d.rep_base + tile.c0 + q], (int64_t)red[2 * q] / 2, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&st.C[d.rep_base + tile.c0 + q], (int64_t)red[2 * q + 1], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        if constexpr (!COOP) break;
        coop_cycle(st, n, tile.c0 == 0, cyc, L.cycles, L.swap_key0, L.swap_key1, L.t_add, L.wait_polls,
                   (uint32_t)L.wait_extra, kErrWait);
        if (cyc + 1 >= L.cycles) break;
        t0 += (uint64_t)L.t_add;
        for (int k = tid; k < tile.P * d.tbl_words; k += nt) {
            const int q = k / d.tbl_words, e = k - q * d.tbl_words;
            tbl[k] = st.tbl[d.tbl_base + (int64_t)coherent_rung(st, d.rep_base + tile.c0 + q) * d.tbl_words + e];
        }
        for (int k = tid; k < 2 * units * words_rpw(d); k += nt) red[k] = 0;
        __syncthreads();
    }
    if (packed) {
        Staged<4, LoadBits> s_sp(pos, load_bits);
        s_sp.put([&](int x, const uint4 &v) {
            store_bits<RM>(d, tile, reinterpret_cast<const uint32_t *>(sp), packed_dev, x, v);
        });
    } else {
        store_bytes<RM>(st, d, tile, sp);
    }
    if (!COOP && L.fuse_exchange) {
        // The tile that completes its instance runs the exchange step.  The step reads no
        // other tile's stores but E_cl and C, which are written and read coherently, so a
        // tile waits for those and counts itself; nothing waits on another workgroup.
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        uint32_t *flag = reinterpret_cast<uint32_t *>(red + 2 * units * words_rpw(d));
        if (tid == 0) {
            const uint32_t before = __hip_atomic_fetch_add(&st.icount[n], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t done = before + 1u == (uint32_t)st.itiles[n] ? 1u : 0u;
            if (done) __hip_atomic_store(&st.icount[n], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *flag = done;
        }
        __syncthreads();
        if (*flag) exchange_instance<true>(st, n, L.swap_key0, L.swap_key1, L.t_add);
    }
}

}  // namespace

int words_mode(int32_t F) { return F <= 20 ? kWordsNarrow : F <= 63 ? kWordsMiddle : kWordsWide; }

int32_t words_tile_lds_bytes(const InstDesc &d, int32_t P)
{
    const int64_t x = words_offsets(d, P).end;
    return (int32_t)(x > 0x7fffffff ? 0x7fffffff : x);
}

int32_t words_lanes(const InstDesc &d, int32_t P) { return words_units(d, P) * words_row(d); }

hipError_t words_kernels_set_lds(int32_t bytes)
{
    if (bytes <= 0) return hipSuccess;
    for (const void *fn : {reinterpret_cast<const void *>(&sweep_words_kernel<false, false>),
                           reinterpret_cast<const void *>(&sweep_words_kernel<true, false>),
                           reinterpret_cast<const void *>(&sweep_words_kernel<false, true>),
                           reinterpret_cast<const void *>(&sweep_words_kernel<true, true>)}) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t words_resident_per_cu(bool replicas, int32_t threads, int32_t lds_bytes, int32_t *per_cu)
{
    int v = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &v, replicas ? reinterpret_cast<const void *>(&sweep_words_kernel<true, true>)
                     : reinterpret_cast<const void *>(&sweep_words_kernel<false, true>), threads, lds_bytes);
    *per_cu = v;
    return e;
}

hipError_t launch_sweep_words(const SweepLaunch &L, bool replicas, hipStream_t s)
{
    if (L.n_tiles <= 0) return hipSuccess;
    const dim3 grid(L.n_tiles), block(L.block_threads);
    if (L.coop && replicas)
        hipLaunchKernelGGL((sweep_words_kernel<true, true>), grid, block, L.lds_bytes, s, L);
    else if (L.coop)
        hipLaunchKernelGGL((sweep_words_kernel<false, true>), grid, block, L.lds_bytes, s, L);
    else if (replicas)
        hipLaunchKernelGGL((sweep_words_kernel<true, false>), grid, block, L.lds_bytes, s, L);
    else
        hipLaunchKernelGGL((sweep_words_kernel<false, false>), grid, block, L.lds_bytes, s, L);
    return hipGetLastError();
}

}  // namespace ptq
