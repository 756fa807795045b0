// pt_host.hip -- host side of the C ABI declared in include/ptqmc.h.
//
// One context holds a batch of instances.  All state lives in one device workspace:
// an immutable region (instance descriptors, neighbour lists, colour blocks, threshold
// tables, pair constants, tiles) followed by the mutable state region (spins, energies,
// permutation, labels, swap statistics, accumulators, counters) that pt_save/pt_load
// copy as one block.  Every sweep and exchange runs on the device; the host only
// launches, so a PT cycle never crosses PCIe (unlike the per-cycle copies of the
// paper's Figure 6).
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <utility>
#include <string>
#include <vector>

#include "../../include/ptqmc.h"
#include "pt_internal.h"

using namespace ptq;

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(PT_EHIP, std::string(what) + ": " + hipGetErrorString(e) + " (hip error " +
                             std::to_string((int)e) + ")");
}

#define HIP_TRY(call)                                     \
    do {                                                  \
        hipError_t e__ = (call);                          \
        if (e__ != hipSuccess) return hip_fail(e__, #call); \
    } while (0)

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr uint32_t kMagic = 0x51505450u;  // checkpoint tag
constexpr uint32_t kVersion = 3;
constexpr int kMaxField = 1023;

// Host copy of everything that is uploaded once, plus the layout of the workspace.
struct Plan {
    std::vector<InstDesc> desc;
    std::vector<int32_t> adj, adj_off, cls_off, rep_inst;
    std::vector<int16_t> hfield;
    std::vector<uint16_t> csite;
    std::vector<uint32_t> ent, bias, tbl;
    std::vector<double> db, dK;
    std::vector<int32_t> n_adj;  // per instance
    int64_t total_reps = 0, total_pairs = 0, spin_bytes = 0;
    int64_t max_tiles = 0;  // tile slots: one per (replica, four-slice group) at most
    // bit-packed encoding: sweep blocks (n, item0) colour by colour with each colour's
    // (first block, blocks); position blocks (n, w, chunk, chunks); per word group
    // (first position block, blocks)
    int32_t encoding = PT_INT8;
    std::vector<int32_t> bp_sblk, bp_eblk, bp_wg;
    std::vector<std::pair<int32_t, int32_t>> bp_colour;
    int32_t bp_n_eblk = 0;
    // bit-packed encoding, octet kernels: 16-bit entries, field codes, per-rung tables and the
    // work list (tiles first, then slice blocks; kOctRec ints each)
    std::vector<uint16_t> oent;
    std::vector<uint8_t> ohinfo;
    std::vector<uint32_t> otbl;
    std::vector<int32_t> otiles;
    int32_t n_otile = 0, n_oblock = 0;         // whole-octet tiles, octet slice blocks
    // the whole-octet work queues: offsets of the 8 per-XCD queues (9 ints), then each
    // queue's list positions, largest octet first
    std::vector<int32_t> oqitems;
    // resident octet slice blocks: every ring of blocks in one run of the launch's map
    bool oblock_xcd = false;
    int32_t otile_lds = 0, oblock_lds = 0;     // their largest LDS need
    int32_t oblock_threads = 256;
    bool oblock_split = false;                 // slice blocks: two lanes per (site, group)
    int32_t oblock_res_lds = 0;                // slice blocks, resident layout
    int64_t orec_words = 0;                    // words of each boundary-record region
    bool bp_generic = false;                   // some packed instance runs the per-class kernel
    // per instance: octets of several degrees; whether any such slice block has a long sweep, or
    // is slower than the per-class kernel when launched per parity (make_plan)
    std::vector<char> irregular;
    bool long_blocks = false, slow_phases = false;
    bool words_alt = false;                    // every whole octet could run as word tiles
    // byte encoding: every instance could run as octets (lists, tables and entries as for the
    // packed one), which the tuner may choose instead of the byte tiles
    bool oct_alt = false;
    int64_t halo_words = 0; // one buffer of slice-block boundary records, at most
    uint64_t flips_per_sweep = 0;
    // byte offsets in the workspace
    size_t o_inst, o_adj, o_off, o_h, o_ent, o_bias, o_csite, o_cls, o_tbl, o_db, o_dK, o_tiles,
        o_repinst, o_halo, o_itiles, o_icount, o_icycle, o_dev, o_prog, o_err, o_bp_sblk, o_bp_eblk, o_bp_wg,
        o_bp_part, o_oent, o_ohinfo, o_otbl, o_otiles, o_orec, o_oprog, o_oqueue, o_oqitems,
        o_xseen;
    size_t o_state;  // start of the mutable region
    size_t o_spins, o_E, o_C, o_rung, o_label, o_rt, o_repof, o_sumE, o_sumC, o_sumE2,
        o_sumC2, o_nup, o_ndown, o_acc, o_att, o_ctr, o_sumCt;
    size_t state_bytes, total_bytes;
};

int validate(const pt_instance &in, int idx)
{
    auto bad = [&](const std::string &m) {
        return fail(PT_EINVAL, "instance " + std::to_string(idx) + ": " + m);
    };
    if (in.N < 1 || in.N > 65535) return bad("N must be in [1, 65535]");
    if (in.M < 1 || (in.M > 1 && (in.M % 2))) return bad("M must be 1 or even");
    if (in.M > 4096) return bad("M must be <= 4096");
    if (in.R < 2) return bad("R must be >= 2");
    if (in.n_edges < 0) return bad("n_edges < 0");
    if (in.n_colors < 1 || in.n_colors > 256) return bad("n_colors must be in [1, 256]");
    if (!in.h || !in.color || !in.rung_b || !in.rung_K) return bad("null array");
    if (in.n_edges > 0 && (!in.edge_i || !in.edge_j || !in.edge_J)) return bad("null edge array");
    for (int i = 0; i < in.N; ++i)
        if (in.color[i] >= in.n_colors) return bad("colour out of range");
    std::vector<int64_t> fsum(in.N);
    for (int i = 0; i < in.N; ++i) fsum[i] = std::abs((int)in.h[i]);
    std::vector<std::pair<int, int>> seen;
    seen.reserve(in.n_edges);
    for (int e = 0; e < in.n_edges; ++e) {
        const int i = in.edge_i[e], j = in.edge_j[e];
        if (i < 0 || j >= in.N || i >= j) return bad("edge " + std::to_string(e) + " needs 0 <= i < j < N");
        if (in.color[i] == in.color[j]) return bad("improper colouring at edge " + std::to_string(e));
        fsum[i] += std::abs((int)in.edge_J[e]);
        fsum[j] += std::abs((int)in.edge_J[e]);
        seen.emplace_back(i, j);
    }
    std::sort(seen.begin(), seen.end());
    if (std::adjacent_find(seen.begin(), seen.end()) != seen.end()) return bad("duplicate edge");
    for (int i = 0; i < in.N; ++i)
        if (fsum[i] > kMaxField) return bad("local field bound exceeds 1023");
    for (int r = 0; r < in.R; ++r) {
        if (!std::isfinite(in.rung_b[r])) return bad("non-finite b");
        if (in.M >= 2 && (!std::isfinite(in.rung_K[r]) || !(in.rung_K[r] > 0.0)))
            return bad("K must be finite and > 0 when M >= 2");
    }
    return PT_OK;
}

// Threshold table of one rung: [x][f + F][tau], x = (s + 1)/2, tau = t'/2 + 1.
void build_table(uint32_t *out, int F, int M, double b, double K)
{
    const double Keff = (M >= 2) ? K : 0.0;
    for (int x = 0; x < 2; ++x) {
        const int s = x ? 1 : -1;
        for (int f = -F; f <= F; ++f) {
            for (int tau = 0; tau < 3; ++tau) {
                const int tp = 2 * (tau - 1);
                const int64_t dE = -2 * (int64_t)s * f;
                const int64_t dC = -2 * (int64_t)s * tp;
                const double dS = b * (double)dE - Keff * (double)dC;
                out[(x * (2 * F + 1) + (f + F)) * 3 + tau] = threshold(dS);
            }
        }
    }
}

// Octet table of one rung (kOctTableWords words): entry n + 16 sigma + 64 hz holds thr(dS) for
// a = s f = 2 n - D - hz agreeing-minus-disagreeing inputs (hz: the table's half) and sigma agreeing time
// neighbours, i.e. dE = -2 a and dC = -4 (sigma - 1): the entry build_table holds for x = 1,
// f = a, tau = sigma, from the same operations.  Unused entries stay 0.
void build_oct_table(uint32_t *out, int D, double b, double K)
{
    for (int k = 0; k < kOctTableWords; ++k) out[k] = 0u;
    for (int hz = 0; hz < 2; ++hz)
        for (int sigma = 0; sigma < 3; ++sigma)
            for (int n = 0; n <= D + hz; ++n) {
                const int a = 2 * n - D - hz;
                const int64_t dE = -2 * (int64_t)a;
                const int64_t dC = -2 * (int64_t)(2 * (sigma - 1));
                const double dS = b * (double)dE - K * (double)dC;
                out[n + 16 * sigma + 64 * hz] = threshold(dS);
            }
}

bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

// LDS of one gfx950 workgroup; instances whose whole replicas exceed it run as slice blocks
constexpr int32_t kLdsPerWorkgroup = 163840;

// Compute units of a gfx950 device.
constexpr int64_t kMostCus = 256;

// Bit-packed encoding: position blocks per word group (at most this many; each block
// passes over 64 positions at a time).
constexpr int32_t kBpMaxChunks = 1024;
constexpr int32_t kBpThreadsHost = 256;

// Whether every ring of slice blocks ([first, end) positions, consecutive) lies within one
// run of the launches' map from workgroups to tiles (runs of nb / 8 positions, each on one
// XCD; the tail past 8 runs keeps its own indices and XCDs).
bool rings_in_runs(const std::vector<std::pair<int, int>> &rings, int nb)
{
    const int q = nb / 8;
    if (q == 0 || nb % 8 != 0) return false;
    for (const auto &r : rings)
        if (r.first / q != (r.second - 1) / q) return false;
    return true;
}

// Whether the launch shape is left to the tuner and no flag asks for a particular route.
bool free_shape(const pt_options &opt)
{
    return opt.tile_replicas == 0 && opt.tile_bytes == 0 && opt.block_threads == 0 &&
           !(opt.flags & (PT_FLAG_SLICE_BLOCKS | PT_FLAG_FOUR_SLICE_LANES | PT_FLAG_TWO_WORD_LANES |
                          PT_FLAG_NO_LATENCY_PATH | PT_FLAG_BLOCK_LAUNCH_PER_SWEEP | PT_FLAG_DEVICE_SCOPE_RECORDS |
                          PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT | PT_FLAG_TEST_XCD_MISMATCH |
                          PT_FLAG_INJECT_LAUNCH_OOR_ONCE));
}

// What a packed batch leaves to the launches per colour class although octets or word tiles
// could take it (make_plan).
struct PackedRoutes {
    bool irregular = true;                       // octets of several degrees run as octets
    int32_t merge_colors = 0, merge_parities = 0; // word tiles of at most so many classes do not
};

int lay_plan(const pt_instance *inst, int32_t n_inst, const pt_options &opt, const PackedRoutes &routes, Plan &P)
{
    const uint32_t flags = opt.flags;
    const int32_t encoding = opt.encoding;
    if (!inst || n_inst < 1) return fail(PT_EINVAL, "need at least one instance");
    if (encoding != PT_INT8 && encoding != PT_BITPACK32) return fail(PT_EINVAL, "unknown encoding");
    P = Plan();
    P.encoding = encoding;
    const bool bp = encoding == PT_BITPACK32;
    // octets of the batch, whichever kernel runs them
    int64_t octets = 0, replicas = 0;
    for (int n = 0; n < n_inst; ++n) {
        octets += (inst[n].R + 7) / 8;
        replicas += inst[n].R;
    }
    // A byte batch that might run as octets carries their tables (512 bytes a replica) beside its
    // own: up to 1 GiB of them, so that no batch outgrows the device for a route it need not take.
    P.oct_alt = !bp && free_shape(opt) && replicas * kOctTableWords * 4 <= (1ll << 30);
    int64_t rep = 0, pair = 0, adjb = 0, offb = 0, siteb = 0, entb = 0, clsb = 0, tblb = 0,
            spinb = 0, wgb = 0;
    for (int n = 0; n < n_inst; ++n) {
        int rc = validate(inst[n], n);
        if (rc) return rc;
        const pt_instance &in = inst[n];
        InstDesc d{};
        d.N = in.N;
        d.M = in.M;
        d.R = in.R;
        d.Mh = (in.M >= 2) ? in.M / 2 : 1;
        d.G4 = (d.Mh + 3) / 4;
        d.parities = (in.M >= 2) ? 2 : 1;
        d.n_colors = in.n_colors;
        // generic neighbour lists: (j & 0xFFFF) | (J << 16)
        std::vector<int32_t> deg(in.N + 1, 0);
        for (int e = 0; e < in.n_edges; ++e) {
            deg[in.edge_i[e] + 1]++;
            deg[in.edge_j[e] + 1]++;
        }
        int D = 0;
        for (int i = 0; i < in.N; ++i) D = std::max(D, deg[i + 1]);
        for (int i = 0; i < in.N; ++i) deg[i + 1] += deg[i];
        std::vector<int32_t> fill(in.N, 0), entries(2 * (size_t)in.n_edges);
        for (int e = 0; e < in.n_edges; ++e) {
            const int i = in.edge_i[e], j = in.edge_j[e];
            const int32_t J = in.edge_J[e];
            entries[deg[i] + fill[i]++] = (j & 0xFFFF) | (int32_t)((uint32_t)J << 16);
            entries[deg[j] + fill[j]++] = (i & 0xFFFF) | (int32_t)((uint32_t)J << 16);
        }
        int F = 0;
        std::vector<int> sumabs(in.N, 0);
        for (int i = 0; i < in.N; ++i) {
            for (int e = deg[i]; e < deg[i + 1]; ++e) sumabs[i] += std::abs(entries[e] >> 16);
            F = std::max(F, sumabs[i] + std::abs((int)in.h[i]));
        }
        d.F = F;
        d.D = std::max(D, 1);
        d.fast = (in.M >= 8 && in.M % 8 == 0 && is_pow2(in.M / 8) && F <= 20) ? 1 : 0;
        // whole-replica tiles address a neighbour row as j*Mh taken straight from the
        // entry; when that exceeds 16 bits the entry holds j and only slice blocks run
        int lgMh = 0;
        while ((1 << lgMh) < d.Mh) ++lgMh;
        d.ent_sh = ((int64_t)(in.N - 1) * d.Mh <= 65535) ? lgMh : 0;
        d.tbl_words = table_words(F);
        d.rep_bytes = (int32_t)align_up((size_t)in.N * in.M, 16);
        d.rep_base = (int32_t)rep;
        d.pair_base = (int32_t)pair;
        d.adj_base = (int32_t)adjb;
        d.off_base = (int32_t)offb;
        d.site_base = (int32_t)siteb;
        d.ent_base = (int32_t)entb;
        d.cls_base = (int32_t)clsb;
        d.tbl_base = (int32_t)tblb;
        d.spin_base = spinb;
        if (bp) {
            d.bp_W = (in.R + 31) / 32;
            d.bp_row = 4 * d.G4;
            d.bp_wg_base = (int32_t)wgb;
        }
        // sites of each colour, colour by colour
        std::vector<int32_t> cls(in.n_colors + 1, 0);
        for (int i = 0; i < in.N; ++i) cls[in.color[i] + 1]++;
        for (int g = 0; g < in.n_colors; ++g) cls[g + 1] += cls[g];
        std::vector<int32_t> cfill(in.n_colors, 0);
        std::vector<uint16_t> sites(in.N);
        for (int i = 0; i < in.N; ++i) sites[cls[in.color[i]] + cfill[in.color[i]]++] = (uint16_t)i;
        // bit-packed encoding: the octet kernels take +-1 couplings, |h| <= 1 and degrees
        // up to D <= 8 on the fast shapes (M a power-of-two multiple of 8).  Instances of
        // several degrees that do not fit them even as blocks of one group run elsewhere.
        bool regular = true;
        if ((bp || P.oct_alt) && d.fast && in.n_edges > 0 && in.N <= 32767) {
            bool ok = D <= 8;
            for (int e = 0; ok && e < in.n_edges; ++e) ok = std::abs((int)in.edge_J[e]) == 1;
            for (int i = 0; ok && i < in.N; ++i) {
                ok = std::abs((int)in.h[i]) <= 1;
                regular = regular && deg[i + 1] - deg[i] == D;
            }
            d.oct = ok && (regular || (routes.irregular && oct_lds_bytes(d, 1, kOctResident) <= kLdsPerWorkgroup)) ? 1 : 0;
        }
        P.irregular.push_back(d.oct && !regular);
        // word tiles: byte instances off the fast shapes and bit-packed ones the octet kernels
        // do not take (and, in batches with fewer octets than compute units, those they do:
        // the tuner decides), where padded neighbour rows and one replica fit a workgroup's
        // LDS (and, bit-packed, a row's lanes fit the smallest workgroup)
        P.oct_alt = P.oct_alt && d.oct;
        if ((bp ? (!d.oct || octets < kMostCus) && d.G4 <= 64 : !d.fast) &&
            (int64_t)in.N * d.D * 4 <= kLdsPerWorkgroup) {
            d.words = words_mode(F);
            if (words_tile_lds_bytes(d, 1) > kLdsPerWorkgroup) d.words = 0;
            // In a lone packed instance a tile's sweep is the whole time, and two launches a class
            // and sweep take less for the largest replicas of few classes: 512 sites, 256 slices
            // and two classes take 250 us a cycle as word tiles and 238 (2 replicas) or 275 (8 to
            // 32) per class; 300 sites without couplings and 400 slices 213 and 158 (8).
            const int few = d.n_colors == 1 ? 32 : d.n_colors == 2 ? 4 : 0;
            if (bp && n_inst == 1 && in.R <= few && (int64_t)in.N * in.M > 40000 * (d.n_colors + 1)) d.words = 0;
            if (bp && !d.oct && d.n_colors <= routes.merge_colors && d.parities <= routes.merge_parities) d.words = 0;
        }
        // fast-path rows: D entries per site, (j << ent_sh) << 16 | w1 << 8 | w0 with w0 / w1 the
        // contribution |J| [J < 0] / |J| [J > 0] of a neighbour whose spin byte is 0 / 1;
        // padding entries point at the site itself with weight 0.  When every |J| = 1, every
        // site has degree D and a one-replica tile would take more than half a compute
        // unit's LDS, the entries shrink to 16 bits (kEntXad16: j * Mh fits 15 bits), so
        // that two such tiles fit one unit.
        d.ent_mode = kEntPerm;
        if (d.fast && !d.words) {
            bool unit = true, regular = true;
            for (int e = 0; e < in.n_edges; ++e) unit = unit && std::abs((int)in.edge_J[e]) == 1;
            for (int i = 0; i < in.N; ++i) regular = regular && deg[i + 1] - deg[i] == d.D;
            int lg = 0;
            while ((1 << lg) < d.Mh) ++lg;
            if (unit && regular && in.n_edges > 0 && d.ent_sh == lg &&
                (int64_t)(in.N - 1) * d.Mh <= 32767 &&
                d.D >= 4 && d.G4 >= 2 &&
                !(flags & (PT_FLAG_SLICE_BLOCKS | PT_FLAG_FOUR_SLICE_LANES)) &&
                sweep_tile_lds_bytes(d, 2 * in.n_edges, 1) > kLdsPerWorkgroup / 2) {
                InstDesc d16 = d;
                d16.ent_mode = kEntXad16;
                if (sweep_tile_lds_bytes(d16, 2 * in.n_edges, 1) <= kLdsPerWorkgroup / 2)
                    d.ent_mode = kEntXad16;
            }
        }
        if (d.fast || d.words) {
            const int sh = d.words ? 0 : d.ent_sh;  // word tiles: the entry holds j itself
            std::vector<uint32_t> row;
            for (int i = 0; i < in.N; ++i) {
                int e = deg[i];
                for (int k = 0; k < d.D; ++k, ++e) {
                    uint32_t word = ((uint32_t)i << sh) << 16;
                    if (e < deg[i + 1]) {
                        const int j = entries[e] & 0xFFFF;
                        const int J = entries[e] >> 16;
                        const uint32_t w0 = (J < 0) ? (uint32_t)(-J) : 0u;
                        const uint32_t w1 = (J > 0) ? (uint32_t)J : 0u;
                        word = (d.ent_mode == kEntXad16)
                                   ? (((uint32_t)j << sh) | (J < 0 ? 0x8000u : 0u))
                                   : ((((uint32_t)j << sh) << 16) | (w1 << 8) | w0);
                    }
                    row.push_back(word);
                }
                // in every byte, or (wide table index of word tiles) in both halves
                const uint32_t b = (uint32_t)(in.h[i] - sumabs[i] + F);
                P.bias.push_back(d.words == kWordsWide ? b * 0x00010001u : (b & 0xFFu) * 0x01010101u);
            }
            if (d.ent_mode == kEntXad16) {
                for (size_t k = 0; k < row.size(); k += 2)
                    P.ent.push_back(row[k] | (k + 1 < row.size() ? row[k + 1] << 16 : 0u));
            } else {
                P.ent.insert(P.ent.end(), row.begin(), row.end());
            }
        } else {
            for (int i = 0; i < in.N; ++i) P.bias.push_back(0);
        }
        if (bp ? d.oct : P.oct_alt) {
            if (P.oent.size() > 0x7fffffff || P.otbl.size() > 0x7fffffff) {  // 32-bit bases
                if (bp) return fail(PT_EINVAL, "batch too large");
                P.oct_alt = false;
            }
        }
        if (bp ? d.oct : P.oct_alt) {
            // entries and field codes padded to 16 bytes per instance (the kernels copy them
            // in 16-byte pieces)
            d.oent_base = (int32_t)P.oent.size();
            // rows padded to D with the site itself, J > 0 (agrees with it) or J < 0 (does
            // not): with I inputs (couplings and a nonzero field) and T = D, or D + 1 where
            // that has I's parity, (T - I) / 2 agreeing ones make a = 2 n - T
            for (int i = 0; i < in.N; ++i) {
                for (int e = deg[i]; e < deg[i + 1]; ++e) {
                    const int j = entries[e] & 0xFFFF;
                    const int J = entries[e] >> 16;
                    P.oent.push_back((uint16_t)(j | (J < 0 ? 0x8000 : 0)));
                }
                const int di = deg[i + 1] - deg[i], inputs = di + (in.h[i] != 0 ? 1 : 0);
                const int agree = (D + ((D - inputs) & 1) - inputs) / 2;
                for (int k = 0; k < D - di; ++k) P.oent.push_back((uint16_t)(i | (k < agree ? 0 : 0x8000)));
            }
            P.oent.resize(align_up(P.oent.size(), 8), 0);
            // field codes: h < 0, h != 0, and whether T is D + 1 (the table's second half)
            d.opad = (int32_t)P.ohinfo.size();
            for (int i = 0; i < in.N; ++i) {
                const int inputs = deg[i + 1] - deg[i] + (in.h[i] != 0 ? 1 : 0);
                P.ohinfo.push_back((uint8_t)((in.h[i] < 0 ? 1 : 0) | (in.h[i] != 0 ? 2 : 0) |
                                             (((D - inputs) & 1) ? 4 : 0)));
            }
            P.ohinfo.resize(align_up(P.ohinfo.size(), 16), 0);
            d.otbl_base = (int32_t)P.otbl.size();
            P.otbl.resize(P.otbl.size() + (size_t)in.R * kOctTableWords);
            for (int r = 0; r < in.R; ++r)
                build_oct_table(P.otbl.data() + d.otbl_base + (size_t)r * kOctTableWords, D,
                                in.rung_b[r], in.rung_K[r]);
        }
        P.desc.push_back(d);
        P.adj.insert(P.adj.end(), entries.begin(), entries.end());
        P.adj_off.insert(P.adj_off.end(), deg.begin(), deg.end());
        for (int i = 0; i < in.N; ++i) P.hfield.push_back(in.h[i]);
        P.csite.insert(P.csite.end(), sites.begin(), sites.end());
        P.cls_off.insert(P.cls_off.end(), cls.begin(), cls.end());
        const size_t t0 = P.tbl.size();
        P.tbl.resize(t0 + (size_t)in.R * d.tbl_words);
        for (int r = 0; r < in.R; ++r)
            build_table(P.tbl.data() + t0 + (size_t)r * d.tbl_words, F, in.M, in.rung_b[r],
                        in.rung_K[r]);
        for (int r = 0; r + 1 < in.R; ++r) {
            P.db.push_back(in.rung_b[r] - in.rung_b[r + 1]);
            P.dK.push_back(in.M >= 2 ? in.rung_K[r] - in.rung_K[r + 1] : 0.0);
        }
        for (int c = 0; c < in.R; ++c) P.rep_inst.push_back(n);
        P.n_adj.push_back(2 * in.n_edges);
        // byte-encoding tiles and slice-block records (the bit-packed kernels use neither)
        if (P.encoding == PT_INT8) P.max_tiles += (int64_t)in.R * std::max(1, d.G4);
        else if (d.words) P.max_tiles += in.R;
        if (d.fast && P.encoding == PT_INT8) {
            // boundary records for slice blocks: three N-word rows per block, at most one
            // block per four-slice group, for every instance that may run as blocks
            const int lgMh_n = 31 - __builtin_clz((unsigned)d.Mh);
            const bool may_block = d.ent_sh != lgMh_n || (flags & PT_FLAG_SLICE_BLOCKS) ||
                                   sweep_tile_lds_bytes(d, 2 * in.n_edges, 1) > kLdsPerWorkgroup;
            if (may_block) P.halo_words += 3ll * in.N * in.R * std::max(1, d.G4);
        }
        P.flips_per_sweep += (uint64_t)in.R * in.N * in.M;
        rep += in.R;
        pair += in.R - 1;
        adjb += 2 * (int64_t)in.n_edges;
        offb += in.N + 1;
        siteb += in.N;
        entb += d.fast || d.words ? ent_words(in.N, d.D, d.ent_mode) : 0;
        clsb += in.n_colors + 1;
        tblb += (int64_t)in.R * d.tbl_words;
        spinb += bp ? (int64_t)d.bp_W * d.parities * in.N * d.bp_row * 4
                    : (int64_t)in.R * d.rep_bytes;
        wgb += d.bp_W;
        if (rep > (1 << 30) || tblb > (1ll << 31) || adjb > (1ll << 31) || entb > (1ll << 31))
            return fail(PT_EINVAL, "batch too large");
    }
    P.total_reps = rep;
    P.total_pairs = pair;
    P.spin_bytes = spinb;
    if (bp) {
        // A batch that also holds octet slice blocks keeps its other instances on the
        // per-class kernel: the blocks already take a clear and a resident launch per call.
        bool blocks_too = false;
        for (const auto &d : P.desc)
            blocks_too = blocks_too || (d.oct && oct_lds_bytes(d, d.G4, kOctTile) > kLdsPerWorkgroup / 2);
        for (auto &d : P.desc)
            if (blocks_too) d.words = 0;
        // sweep blocks: colour g of every instance that has it, 256 items per block
        int max_colors = 0;
        for (const auto &d : P.desc) max_colors = std::max(max_colors, d.n_colors);
        for (int g = 0; g < max_colors; ++g) {
            const int32_t first = (int32_t)(P.bp_sblk.size() / 2);
            for (int n = 0; n < n_inst; ++n) {
                const InstDesc &d = P.desc[n];
                if (g >= d.n_colors || d.oct || d.words) continue;
                const int64_t sg = P.cls_off[d.cls_base + g + 1] - P.cls_off[d.cls_base + g];
                const int64_t items = (int64_t)d.bp_W * sg * d.G4 * kBpSweepLanes;
                for (int64_t it = 0; it < items; it += kBpThreadsHost) {
                    P.bp_sblk.push_back(n);
                    P.bp_sblk.push_back((int32_t)it);
                }
                if (items > 0x7fffffff) return fail(PT_EINVAL, "batch too large");
            }
            P.bp_colour.emplace_back(first, (int32_t)(P.bp_sblk.size() / 2) - first);
        }
        // position blocks of every word group
        for (int n = 0; n < n_inst; ++n) {
            const InstDesc &d = P.desc[n];
            const int64_t Q = (int64_t)d.parities * d.N * d.G4;
            const int32_t chunks = (int32_t)std::min<int64_t>(kBpMaxChunks, std::max<int64_t>(1, (Q + 63) / 64));
            for (int w = 0; w < d.bp_W; ++w) {
                P.bp_wg.push_back((int32_t)(P.bp_eblk.size() / 4));
                P.bp_wg.push_back(chunks);
                for (int k = 0; k < chunks; ++k) {
                    P.bp_eblk.push_back(n);
                    P.bp_eblk.push_back(w);
                    P.bp_eblk.push_back(k);
                    P.bp_eblk.push_back(chunks);
                }
            }
        }
        P.bp_n_eblk = (int32_t)(P.bp_eblk.size() / 4);
        if (P.bp_sblk.size() / 2 > 0x7fffffff || P.bp_eblk.size() / 4 > 0x7fffffff)
            return fail(PT_EINVAL, "batch too large");
    }
    // Byte batches that could run as octets may: a cycle of 192 (512) instances of the uneven
    // batch takes 1182 (2998) us as byte tiles and 936 (2280) as octets.  Batches of fewer
    // octets than half the compute units are not offered the choice (at 136 octets the byte
    // tiles, several to an octet, fill the chip better: 210 us), and the tuner makes it; nor
    // are batches with byte slice blocks: with a launch per cycle those are as fast (one lattice
    // of 1024 x 256 spins: 178 us and 181, with correlations 194 and 199) or faster (two: 530 and
    // 711).  In launches of 64 cycles octet blocks take 138 us for the one lattice, which the few
    // cycles a shape is timed over do not show.
    bool any_block = false;
    for (const auto &d : P.desc)
        any_block = any_block || (d.oct && oct_lds_bytes(d, d.G4, kOctTile) > kLdsPerWorkgroup / 2);
    P.oct_alt = P.oct_alt && P.halo_words == 0 && (any_block || octets >= kMostCus / 2);
    if (bp || P.oct_alt) {
        // octet work: whole octets where one takes at most half a compute unit's LDS
        // (largest first), else slice blocks of ng groups, ng about 512 colour-class items
        // per launch and class
        std::vector<std::array<int32_t, kOctRec>> tiles, blocks;
        for (int n = 0; n < n_inst; ++n) {
            const InstDesc &d = P.desc[n];
            if (!d.oct) {
                P.bp_generic = P.bp_generic || !d.words;
                continue;
            }
            const bool whole = oct_lds_bytes(d, d.G4, kOctTile) <= kLdsPerWorkgroup / 2;
            int ng = d.G4;
            if (!whole) {
                ng = 1;
                while (2 * ng < d.G4 && (int64_t)2 * ng * d.N <= 512 * (int64_t)d.n_colors &&
                       oct_lds_bytes(d, 2 * ng, kOctResident) <= kLdsPerWorkgroup / 2)
                    ng *= 2;
                if (oct_lds_bytes(d, ng, kOctResident) > kLdsPerWorkgroup) {
                    if (bp)
                        return fail(PT_EINVAL, "instance " + std::to_string(n) +
                                                   ": an octet slice block does not fit in LDS");
                    P.oct_alt = false;
                }
                P.long_blocks = P.long_blocks || (P.irregular[n] && (int64_t)ng * d.N > 1400 * d.n_colors);
                P.slow_phases = P.slow_phases ||
                                (P.irregular[n] && (d.n_colors < 4 || (int64_t)ng * d.N > 500 * d.n_colors));
            }
            for (int w = 0; w < (d.R + 31) / 32; ++w)
                for (int o = 0; o < 4 && 32 * w + 8 * o < d.R; ++o) {
                    if (whole) {
                        tiles.push_back({n, w, o, 0, d.G4, 0, 0, 0});
                        P.otile_lds = std::max(P.otile_lds, oct_lds_bytes(d, d.G4, kOctTile) + kOctQueueLds);
                    } else {
                        // the octet's ring of blocks (at least two: ng < G4), consecutive in
                        // the list; neighbours and record offsets are filled in below
                        for (int g0 = 0; g0 < d.G4; g0 += ng) blocks.push_back({n, w, o, g0, ng, 0, 0, 0});
                        P.oblock_lds = std::max(P.oblock_lds, oct_lds_bytes(d, ng, kOctPhase));
                        P.oblock_res_lds = std::max(P.oblock_res_lds, oct_lds_bytes(d, ng, kOctResident));
                    }
                }
        }
        // Whole octets go out in one launch, largest first: the small ones, whose sweeps are
        // short chains of dependent colour classes, then run beside the large ones (launched
        // apart, a class of small octets took as long as one octet's chain).
        std::stable_sort(tiles.begin(), tiles.end(), [&](const std::array<int32_t, kOctRec> &a,
                                                         const std::array<int32_t, kOctRec> &b) {
            const InstDesc &da = P.desc[a[0]], &db = P.desc[b[0]];
            return (int64_t)da.N * da.M > (int64_t)db.N * db.M;
        });
        // The octets of one word group read the same 16-byte pieces of device memory and
        // write different bytes of them, so they should share an XCD's L2.  Workgroups go to
        // the XCDs round robin by index: the word groups (still largest first) are dealt to
        // per-XCD queues, each to the least loaded, and workgroup 8 s + x takes entry s of
        // queue x (the last rounds, where queue lengths differ, keep their order only).
        {
            constexpr int kXcds = 8;
            std::vector<std::vector<std::array<int32_t, kOctRec>>> q(kXcds);
            std::vector<int64_t> load(kXcds, 0);
            for (size_t k = 0; k < tiles.size();) {
                size_t e = k + 1;
                while (e < tiles.size() && tiles[e][0] == tiles[k][0] && tiles[e][1] == tiles[k][1]) ++e;
                const InstDesc &d = P.desc[tiles[k][0]];
                const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
                for (size_t j = k; j < e; ++j) q[x].push_back(tiles[j]);
                load[x] += (int64_t)d.N * d.M * (int64_t)(e - k);
                k = e;
            }
            std::vector<std::array<int32_t, kOctRec>> dealt;
            dealt.reserve(tiles.size());
            std::vector<std::vector<int32_t>> pos(kXcds);
            for (size_t r = 0; dealt.size() < tiles.size(); ++r)
                for (int x = 0; x < kXcds; ++x)
                    if (r < q[x].size()) {
                        pos[x].push_back((int32_t)dealt.size());
                        dealt.push_back(q[x][r]);
                    }
            tiles.swap(dealt);
            // the same queues for the work-queue launch, whose workgroups take positions
            // from their own XCD's queue
            P.oqitems.assign(kXcds + 1, 0);
            for (int x = 0; x < kXcds; ++x) P.oqitems[x + 1] = P.oqitems[x] + (int32_t)pos[x].size();
            for (int x = 0; x < kXcds; ++x) P.oqitems.insert(P.oqitems.end(), pos[x].begin(), pos[x].end());
        }
        // Resident slice blocks pass boundary records to their ring neighbours twice per
        // sweep.  When every ring lies in one run of the resident launch's workgroup-to-block
        // map (so on one XCD), the records pass through that XCD's L2 instead of
        // device-scope operations.
        const int base = (int)tiles.size();  // blocks follow the tiles in the list
        std::vector<int32_t> prev(blocks.size()), next(blocks.size());
        for (size_t k = 0; k < blocks.size(); ++k) {
            const auto &t = blocks[k];
            const int ring = P.desc[t[0]].G4 / t[4];   // blocks of the octet
            const int first = (int)k - t[3] / t[4];    // its block at group 0
            prev[k] = first + (t[3] / t[4] + ring - 1) % ring;
            next[k] = first + (t[3] / t[4] + 1) % ring;
        }
        {
            std::vector<std::pair<int, int>> rings;  // [first, end) in blocks
            const int nb = (int)blocks.size();
            for (int k = 0; k < nb;) {
                int e = k + 1;
                while (e < nb && blocks[e][0] == blocks[k][0] && blocks[e][1] == blocks[k][1] &&
                       blocks[e][2] == blocks[k][2])
                    ++e;
                rings.emplace_back(k, e);
                k = e;
            }
            P.oblock_xcd = rings_in_runs(rings, nb);
        }
        for (size_t k = 0; k < blocks.size(); ++k) {
            auto &t = blocks[k];
            t[5] = (int32_t)P.orec_words;
            t[6] = base + prev[k];
            t[7] = base + next[k];
            P.orec_words += P.desc[t[0]].N;
        }
        for (const auto &t : tiles) P.otiles.insert(P.otiles.end(), t.begin(), t.end());
        for (const auto &t : blocks) P.otiles.insert(P.otiles.end(), t.begin(), t.end());
        P.n_otile = (int32_t)tiles.size();
        P.n_oblock = (int32_t)blocks.size();
        P.words_alt = bp && P.n_otile > 0 && P.n_oblock == 0 && !P.bp_generic && !(flags & PT_FLAG_WORK_QUEUE);
        for (const auto &d : P.desc) P.words_alt = P.words_alt && d.words;
        // slice blocks: one pass over a colour class of the largest block, with two lanes per
        // (site, group) when a class has at most 512 of them
        int most = 1;
        for (const auto &t : blocks) {
            const InstDesc &d = P.desc[t[0]];
            most = std::max<int>(most, (int)std::min<int64_t>(1024, ((int64_t)d.N * t[4] + d.n_colors - 1) / d.n_colors));
        }
        P.oblock_split = most <= 512;
        if (P.oblock_split) most *= 2;
        P.oblock_threads = 64;
        while (P.oblock_threads < most && P.oblock_threads < 1024) P.oblock_threads *= 2;
        if (P.orec_words > 0x3fffffff) {
            if (bp) return fail(PT_EINVAL, "batch too large");
            P.oct_alt = false;
        }
        if (!bp && !P.oct_alt) P.n_otile = P.n_oblock = 0;
    }
    if (!bp && !P.oct_alt) {
        P.oent.clear();
        P.ohinfo.clear();
        P.otbl.clear();
        P.otiles.clear();
        P.orec_words = 0;
    }
    // layout
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + std::max<size_t>(bytes, 1), 256);
        return at;
    };
    P.o_inst = take(P.desc.size() * sizeof(InstDesc));
    P.o_adj = take(P.adj.size() * 4);
    P.o_off = take(P.adj_off.size() * 4);
    P.o_h = take(P.hfield.size() * 2);
    P.o_ent = take(P.ent.size() * 4);
    P.o_bias = take(P.bias.size() * 4);
    P.o_csite = take(P.csite.size() * 2);
    P.o_cls = take(P.cls_off.size() * 4);
    P.o_tbl = take(P.tbl.size() * 4);
    P.o_db = take(P.db.size() * 8);
    P.o_dK = take(P.dK.size() * 8);
    P.o_tiles = take((size_t)P.max_tiles * sizeof(Tile));
    P.o_repinst = take((size_t)rep * 4);
    P.o_halo = take((size_t)P.halo_words * 2 * 4);
    P.o_itiles = take((size_t)n_inst * 4);
    P.o_icount = take((size_t)n_inst * 4);  // zero in the uploaded image
    P.o_icycle = take((size_t)n_inst * 4);  // zero in the uploaded image
    P.o_dev = take(sizeof(DevState));
    P.o_prog = take((size_t)P.max_tiles * 4);
    P.o_err = take(4);                       // zero in the uploaded image
    P.o_bp_sblk = take(P.bp_sblk.size() * 4);
    P.o_bp_eblk = take(P.bp_eblk.size() * 4);
    P.o_bp_wg = take(P.bp_wg.size() * 4);
    P.o_bp_part = take((size_t)P.bp_n_eblk * 32 * 2 * 8);
    P.o_oent = take(P.oent.size() * 2);
    P.o_ohinfo = take(P.ohinfo.size());
    P.o_otbl = take(P.otbl.size() * 4);
    P.o_otiles = take(P.otiles.size() * 4);
    P.o_orec = take((size_t)P.orec_words * 2 * 4);
    P.o_oprog = take((size_t)(P.n_otile + P.n_oblock) * 2 * 4);
    P.o_oqueue = take(9 * 4);  // zero in the uploaded image
    P.o_oqitems = take(P.oqitems.size() * 4);
    P.o_xseen = take(2 * 4);
    P.o_state = o;
    P.o_spins = take((size_t)spinb);
    P.o_E = take((size_t)rep * 8);
    P.o_C = take((size_t)rep * 8);
    P.o_rung = take((size_t)rep * 4);
    P.o_label = take((size_t)rep * 4);
    P.o_rt = take((size_t)rep * 8);
    P.o_repof = take((size_t)rep * 4);
    P.o_sumE = take((size_t)rep * 8);
    P.o_sumC = take((size_t)rep * 8);
    P.o_sumE2 = take((size_t)rep * 8);
    P.o_sumC2 = take((size_t)rep * 8);
    P.o_sumCt = take((size_t)rep * PT_TAU_LAGS * 8);
    P.o_nup = take((size_t)rep * 8);
    P.o_ndown = take((size_t)rep * 8);
    P.o_acc = take((size_t)pair * 8);
    P.o_att = take((size_t)pair * 8);
    P.o_ctr = take((size_t)n_inst * sizeof(Counters));
    P.state_bytes = o - P.o_state;
    P.total_bytes = o;
    return PT_OK;
}

// The plan of a batch.  Packed instances that octets (of several degrees) or word tiles could take
// stay with the launches per colour class where those are faster, us a cycle of 10 sweeps:
//   - in a batch that needs those launches for another instance, whose launches the further items
//     share: beside 8000 sites (8 slices, couplings up to 3, 32 replicas: 278 alone) an open lattice
//     of 336 sites, 64 slices and 8 replicas takes 284 so and 514 as an octet of its own, 64 sites
//     with couplings up to 3 284 and 310 as word tiles.  Word tiles only while they are few spins
//     in all and bring no more classes (48 replicas of 128 x 64 spins in five classes: 660 and 342);
//   - octet slice blocks of several degrees with a long sweep and not enough of them: 16^3 sites
//     take 380 whatever the number of blocks, and per class 278 (4 blocks), 316 (32), 411 (64);
//     14^3 sites 275 and 280 to 361;
//   - those that are too many to be resident: 512 blocks of 9^3 to 16^3 sites take 611 to 2340
//     against 519 to 2106, but 1013 against 1392 for 1000 sites in four classes.
int make_plan(const pt_instance *inst, int32_t n_inst, const pt_options &opt, Plan &P)
{
    constexpr int kEnoughBlocks = 64;
    constexpr int64_t kMergeSpins = 4 << 20;  // some 40 us a cycle in launches that run anyway
    PackedRoutes routes;
    int rc = lay_plan(inst, n_inst, opt, routes, P);
    if (opt.encoding != PT_BITPACK32) return rc;
    auto per_class = [](const InstDesc &d) { return !d.oct && !d.words; };
    const bool any = std::find(P.irregular.begin(), P.irregular.end(), 1) != P.irregular.end();
    if (any && (rc || std::any_of(P.desc.begin(), P.desc.end(), per_class) ||
                (P.n_oblock > kMostCus ? P.slow_phases : P.long_blocks && P.n_oblock < kEnoughBlocks))) {
        routes.irregular = false;
        rc = lay_plan(inst, n_inst, opt, routes, P);
    }
    if (rc) return rc;
    for (const auto &d : P.desc)
        if (per_class(d)) {
            routes.merge_colors = std::max(routes.merge_colors, d.n_colors);
            routes.merge_parities = std::max(routes.merge_parities, d.parities);
        }
    int64_t spins = 0;
    for (const auto &d : P.desc)
        if (!d.oct && d.words && d.n_colors <= routes.merge_colors && d.parities <= routes.merge_parities)
            spins += (int64_t)d.bp_W * 32 * d.N * d.M;
    return spins > 0 && spins <= kMergeSpins ? lay_plan(inst, n_inst, opt, routes, P) : PT_OK;
}


struct CkptHeader {
    uint32_t magic, version;
    uint64_t state_bytes;
    uint64_t seed;
    int32_t n_inst, encoding;
    uint64_t flips_per_sweep;
};
static_assert(sizeof(CkptHeader) == 40, "checkpoint header layout is part of the ABI");

// A checkpoint for these instances and options: the header matches, and every value that
// the kernels use as an index is in range -- spin bytes in {0, 1} (they index threshold
// tables; any bit pattern is a valid bit-packed state), replica_of and rung_of inverse
// permutations of [0, R) per instance (they index energies and tables), labels in
// {NONE, UP, DOWN}.  Nothing is copied anywhere.
int check_checkpoint(const Plan &P, const pt_options &opt, int32_t n_inst, const void *buf,
                     size_t len)
{
    if (!buf) return fail(PT_EINVAL, "null checkpoint");
    if (len < sizeof(CkptHeader)) return fail(PT_ESTATE, "checkpoint too short");
    CkptHeader h;
    std::memcpy(&h, buf, sizeof h);
    if (h.magic != kMagic || h.version != kVersion) return fail(PT_ESTATE, "not a checkpoint");
    if (h.state_bytes != P.state_bytes || h.n_inst != n_inst || h.seed != opt.seed ||
        h.flips_per_sweep != P.flips_per_sweep || len != sizeof h + h.state_bytes)
        return fail(PT_ESTATE, "checkpoint belongs to different instances or options");
    if (h.encoding != opt.encoding)
        return fail(PT_ESTATE, "checkpoint was written under another spin encoding");
    const char *state = (const char *)buf + sizeof h;
    if (P.encoding == PT_INT8) {
        const uint8_t *sp = (const uint8_t *)(state + (P.o_spins - P.o_state));
        for (int64_t b = 0; b < P.spin_bytes; ++b)
            if (sp[b] > 1) return fail(PT_ESTATE, "checkpoint holds invalid spins");
    }
    auto i32_at = [&](size_t off, int64_t k) {
        int32_t v;
        std::memcpy(&v, state + (off - P.o_state) + 4 * k, 4);
        return v;
    };
    for (int32_t n = 0; n < n_inst; ++n) {
        const InstDesc &d = P.desc[n];
        for (int r = 0; r < d.R; ++r) {
            const int32_t c = i32_at(P.o_repof, d.rep_base + r);
            if (c < 0 || c >= d.R || i32_at(P.o_rung, d.rep_base + c) != r)
                return fail(PT_ESTATE, "checkpoint of instance " + std::to_string(n) +
                                           ": replica_of and rung_of are not inverse permutations");
        }
        for (int c = 0; c < d.R; ++c) {
            const int32_t lab = i32_at(P.o_label, d.rep_base + c);
            if (lab != PT_LABEL_NONE && lab != PT_LABEL_UP && lab != PT_LABEL_DOWN)
                return fail(PT_ESTATE, "checkpoint of instance " + std::to_string(n) +
                                           ": invalid round-trip label");
        }
    }
    return PT_OK;
}

}  // namespace

struct pt_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    char *ws = nullptr;
    bool own_ws = false;
    Plan plan;
    DevState st{};
    pt_options opt{};
    uint32_t key_flip0 = 0, key_flip1 = 0, key_swap0 = 0, key_swap1 = 0;
    // launch shape
    // fast-kernel tiles, then word tiles (slices, then replicas), generic ones, slice blocks
    std::vector<Tile> tiles;
    int n_fast_tiles = 0, n_words_tiles = 0, n_generic_tiles = 0, n_block_tiles = 0;
    int lds_block = 0;
    // resident slice blocks: compute-unit occupancy for (block threads, block LDS)
    std::pair<int, int> resident_key{-1, -1};
    int resident_per_cu = 0;
    int block_persistent = 0;   // the last slice-block call ran as one resident launch
    int lane_words = 2;         // whole-replica tiles: four-slice words per lane
    bool block_xcd = false;     // resident slice blocks: every replica's ring on one XCD
    bool lat = false;           // whole-replica tiles: the latency path
    bool oct_resident = false;  // octet slice blocks: one resident launch per call
    // Recovery when a resident launch's wait gave up: a device copy of the state region at
    // the last clean synchronisation, the calls queued since (kind, count: 0 pt_sweep,
    // 1 pt_exchange, 2 pt_run), whether resident launches are off since a recovery, and whether
    // a caller has captured a call.
    // (shadow is null where nothing can give up; shadow_mem is what was allocated for it.)
    char *shadow = nullptr, *shadow_mem = nullptr;
    std::vector<std::pair<int, int>> journal;
    bool replaying = false, resident_off = false, captured = false;
    int64_t recoveries = 0;
    uint32_t last_device_error = 0;  // the device error word of the last failed synchronisation
    // whole octets from the device work queue; the exchange fused into the octet that
    // completes an instance (every instance of the batch in whole octets)
    bool oct_queue = false, oct_fuse = false;
    // whole octets run as word tiles instead (the tuner's choice, Plan::words_alt)
    bool oct_as_words = false;
    // byte encoding: octets instead of the byte tiles (the tuner's choice, Plan::oct_alt)
    bool byte_octets = false;
    int coop_fits = -1;        // can_coop's answer for the tiles and block size in use (-1: not asked)
    int block_threads = 256;
    int tile_bytes = 0;        // target spin bytes per tile in use
    // self-tuning: candidate (tile bytes, threads) shapes timed on the first sweep launches
    bool tuning = false;
    struct Shape {
        int tile_bytes, threads;
        bool alt;            // oct_as_words or byte_octets
        int replicas;        // per tile; 0: from the tile bytes
        uint64_t tiles = 0;  // hash of the tile list, once built
    };
    std::vector<Shape> cand;
    std::vector<size_t> cand_order; // candidates still in the running, in the order they are tried
    std::vector<double> cand_ms;
    size_t cand_next = 0, tune_round = 0;
    int tune_done = 0, tune_most = 1;  // cycles timed so far; a launch's in the round under way
    hipEvent_t tune_ev[2] = {nullptr, nullptr};
    int lds_fast = 0, lds_words = 0, lds_generic = 0;
    int max_P = 1;
    int lds_limit = 65536;     // LDS one workgroup may use
    int cu_lds = 65536;        // LDS of one compute unit
    int cu_threads = 2048;     // resident threads of one compute unit
    int cus = 256;
    std::vector<int> tile_lds; // LDS bytes of every whole-replica tile (block tiles: 0)
    std::vector<int32_t> itiles;  // tiles per instance (host copy)
    int fallbacks = 0;
    bool inject_pending = false;
    // graph of whole cycles for pt_run
    hipGraphExec_t graph = nullptr;
    int graph_cycles = 0;
    // read-back: a pinned buffer for one instance's observables and the device error word,
    // and up to two of kSpinChunk bytes for spins (allocated on first use)
    char *obs_pin = nullptr;
    char *spin_pin = nullptr;
    size_t spin_pin_bytes = 0;
    hipEvent_t spin_ev[2] = {nullptr, nullptr};
    // timing
    std::vector<hipEvent_t> ev_pool;
    std::vector<std::pair<int, int>> sweep_ev, exch_ev;  // indices into ev_pool
    std::vector<int> sweep_ev_calls;  // sweep calls each sweep_ev pair covers
    size_t ev_used = 0;
    double sweep_ms = 0, exch_ms = 0;
    int64_t sweep_n = 0, exch_n = 0;
    // multi-cycle launches: how many were issued and the cycles they ran (always counted),
    // and their event time under PT_FLAG_TIMING (kept apart from the sweep calls)
    std::vector<std::pair<int, int>> multi_ev;
    double multi_ms = 0;
    int64_t multi_launches = 0, multi_cycles = 0;
};

namespace {

int n_inst_of(const pt_ctx *c) { return (int)c->plan.desc.size(); }

// Choose tiles: P replicas of one instance per workgroup, P limited by LDS (and a power of
// two on the fast path), sized so the batch yields a few workgroups per CU when it can
// (the paper's chain packing, Section 5, stops packing once multiprocessors would go
// idle).
int build_tiles(pt_ctx *c, int force_P, int tile_bytes)
{
    const Plan &P = c->plan;
    c->coop_fits = -1;
    // the tile list is uploaded from c->tiles: let any earlier upload finish first
    HIP_TRY(hipStreamSynchronize(c->stream));
    int64_t total_bytes = 0;
    for (const auto &d : P.desc) total_bytes += (int64_t)d.R * d.N * d.M;
    int64_t target_bytes = std::max<int64_t>(total_bytes / (2ll * c->cus), 4096);
    target_bytes = std::min<int64_t>(target_bytes, 64 * 1024);
    if (tile_bytes > 0) target_bytes = tile_bytes;
    c->tile_bytes = (int)target_bytes;
    const bool force_blocks = (c->opt.flags & PT_FLAG_SLICE_BLOCKS) != 0;
    std::vector<Tile> fast, words, generic, block;
    int lds_f = 0, lds_w = 0, lds_g = 0, lds_b = 0, maxP = 1;
    auto as_words = [&](const InstDesc &d) { return d.words && (!d.oct || c->oct_as_words); };
    int64_t words_reps = 0;
    for (const auto &d : P.desc) words_reps += as_words(d) ? d.R : 0;
    for (int n = 0; n < (int)P.desc.size(); ++n) {
        const InstDesc &d = P.desc[n];
        if (as_words(d) && words_lanes(d, 1) <= c->block_threads) {
            // Replicas per word tile: the target bytes, but as few as leave every compute
            // unit a tile (a tile's sweep is a chain of class steps, so a unit without one
            // idles for the whole call: 512 replicas of 10^3 spins at M = 1 take 33 us a cycle
            // in 256 tiles of 2 and 55 us in 64 tiles of 8; 768 packed replicas of 128 x 64
            // spins 95 us in 768 tiles and 204 us in 96); a lane per word of a site, half a
            // unit's LDS.
            int p = force_P > 0 ? force_P
                                : (int)std::min<int64_t>(target_bytes / ((int64_t)d.N * d.M),
                                                         words_reps / c->cus);
            p = std::max(1, std::min(p, d.R));
            auto fits = [&](int q, int lds) {
                return words_lanes(d, q) <= c->block_threads && words_tile_lds_bytes(d, q) <= lds;
            };
            while (p > 1 && !fits(p, force_P > 0 ? c->lds_limit : c->cu_lds / 2)) --p;
            if (fits(p, c->lds_limit)) {
                const int kind = d.M <= 2 ? kTileWordsR : kTileWords;
                // bit-packed tiles stay within a word group
                const int group = P.encoding == PT_BITPACK32 ? 32 : d.R;
                for (int c0 = 0; c0 < d.R;) {
                    const int q = std::min({p, d.R - c0, group - c0 % group});
                    words.push_back(Tile{n, c0, q, kind, 0, d.G4});
                    lds_w = std::max(lds_w, words_tile_lds_bytes(d, q));
                    maxP = std::max(maxP, q);
                    c0 += q;
                }
                continue;
            }
        }
        if (P.encoding == PT_BITPACK32) {
            if (!as_words(d)) continue;  // octets and the per-class kernel
            return fail(PT_EINVAL, "instance " + std::to_string(n) +
                                       ": a word tile needs more LDS than the device has");
        }
        int pmax = 0;
        for (int p = d.R; p >= 1; --p)
            if (sweep_tile_lds_bytes(d, P.n_adj[n], p) <= c->lds_limit &&
                (!d.fast || is_pow2(p))) {
                pmax = p;
                break;
            }
        const int lgMh_n = d.fast ? 31 - __builtin_clz((unsigned)d.Mh) : 0;
        const bool blocked = d.fast && (pmax < 1 || d.ent_sh != lgMh_n || (force_blocks && d.G4 >= 2));
        if (blocked && d.ent_mode == kEntXad16)
            return fail(PT_EINVAL, "instance " + std::to_string(n) +
                                       ": 16-bit neighbour entries need whole-replica tiles, "
                                       "but the device's LDS is smaller than the library assumes");
        if (blocked) {
            // slice blocks: ng four-slice groups per parity, halving until a block fits
            int ng = force_blocks ? std::max(1, d.G4 / 4) : d.G4;
            while (ng > 1 && ((int64_t)2 * d.N * 4 * (ng + 1) > std::max<int64_t>(target_bytes, 8 * d.N) ||
                              block_tile_lds_bytes(d, 1, ng) > c->lds_limit))
                ng /= 2;
            if (block_tile_lds_bytes(d, 1, ng) > c->lds_limit)
                return fail(PT_EINVAL, "instance " + std::to_string(n) +
                                           ": even one slice group does not fit in LDS");
            for (int c0 = 0; c0 < d.R; ++c0) {
                const int first = (int)block.size(), nb = d.G4 / ng;
                for (int k = 0; k < nb; ++k) {
                    // prev/next are indices within the block list here, made global below
                    block.push_back(Tile{n, c0, 1, kTileBlock, k * ng, ng, 0,
                                         first + (k + nb - 1) % nb, first + (k + 1) % nb});
                }
            }
            lds_b = std::max(lds_b, block_tile_lds_bytes(d, 1, ng));
            continue;
        }
        if (pmax < 1)
            return fail(PT_EINVAL, "instance " + std::to_string(n) +
                                       ": one replica does not fit in LDS (N*M too large)");
        int p = (int)std::max<int64_t>(1, target_bytes / ((int64_t)d.N * d.M));
        if (force_P > 0) p = force_P;
        p = std::max(1, std::min(p, pmax));
        if (d.fast)
            while (!is_pow2(p)) --p;
        // at most half a compute unit's LDS per tile where fewer replicas allow it, so that
        // two workgroups share a unit and the batch's tiles form one occupancy class
        if (force_P <= 0)
            while (p > 1 && sweep_tile_lds_bytes(d, P.n_adj[n], p) > c->cu_lds / 2)
                p = d.fast ? p / 2 : p - 1;
        for (int c0 = 0; c0 < d.R;) {
            int q = std::min(p, d.R - c0);
            if (d.fast)
                while (!is_pow2(q)) --q;
            Tile t{n, c0, q, d.fast ? kTileFast : kTileGeneric, 0, d.G4};
            (d.fast ? fast : generic).push_back(t);
            const int b = sweep_tile_lds_bytes(d, P.n_adj[n], q);
            (d.fast ? lds_f : lds_g) = std::max(d.fast ? lds_f : lds_g, b);
            maxP = std::max(maxP, q);
            c0 += q;
        }
    }
    // Tiles in order of decreasing LDS need, ties by decreasing work.  Launches then split
    // the list into occupancy classes (see launch_groups) and each class starts with its
    // largest tiles: the device dispatches workgroups roughly in order, so the longest work
    // starts earliest (the paper's "hardest chains first" work pool, Section 4).
    auto lds_of = [&](const Tile &t) {
        return t.kind == kTileWords || t.kind == kTileWordsR
                   ? words_tile_lds_bytes(P.desc[t.inst], t.P)
                   : sweep_tile_lds_bytes(P.desc[t.inst], P.n_adj[t.inst], t.P);
    };
    auto bigger = [&](const Tile &a, const Tile &b) {
        if (a.kind != b.kind) return a.kind < b.kind;
        const int la = lds_of(a), lb = lds_of(b);
        if (la != lb) return la > lb;
        const InstDesc &da = P.desc[a.inst], &db = P.desc[b.inst];
        return (int64_t)a.P * da.M * da.N > (int64_t)b.P * db.M * db.N;
    };
    std::stable_sort(fast.begin(), fast.end(), bigger);
    std::stable_sort(words.begin(), words.end(), bigger);
    std::stable_sort(generic.begin(), generic.end(), bigger);
    const size_t n_whole = fast.size() + words.size() + generic.size();
    if ((int64_t)(n_whole + block.size()) > P.max_tiles)
        return fail(PT_ESTATE, "internal: more tiles than reserved tile slots");
    // slice blocks: global neighbour indices and boundary-record offsets
    const int block0 = (int)n_whole;
    int64_t hb = 0;
    for (Tile &t : block) {
        t.prev += block0;
        t.next += block0;
        t.hb = (int32_t)hb;
        hb += 3ll * P.desc[t.inst].N;
    }
    if (hb > P.halo_words || hb > 0x7fffffff)
        return fail(PT_EINVAL, "slice blocks need more boundary records than were reserved "
                               "(the device's LDS is smaller than the library assumes)");
    // Resident slice blocks pass boundary records to the neighbouring blocks of their
    // replica every sweep: when every replica's ring of blocks lies in one run of the
    // launches' workgroup-to-tile map (so on one XCD), the records pass through that XCD's
    // L2 instead of device-scope operations.
    {
        std::vector<std::pair<int, int>> rings;
        const int nb = (int)block.size();
        for (int k = 0; k < nb;) {
            int e = k + 1;
            while (e < nb && block[e].inst == block[k].inst && block[e].c0 == block[k].c0) ++e;
            rings.emplace_back(k, e);
            k = e;
        }
        c->block_xcd = rings_in_runs(rings, nb);
    }
    c->tiles = fast;
    c->tiles.insert(c->tiles.end(), words.begin(), words.end());
    c->tiles.insert(c->tiles.end(), generic.begin(), generic.end());
    c->tiles.insert(c->tiles.end(), block.begin(), block.end());
    c->n_fast_tiles = (int)fast.size();
    c->n_words_tiles = (int)words.size();
    c->n_generic_tiles = (int)generic.size();
    c->tile_lds.assign(c->tiles.size(), 0);
    for (size_t k = 0; k < n_whole; ++k) c->tile_lds[k] = lds_of(c->tiles[k]);
    c->n_block_tiles = (int)block.size();
    c->lds_fast = lds_f;
    c->lds_words = lds_w;
    c->lds_generic = lds_g;
    c->lds_block = lds_b;
    c->max_P = maxP;
    HIP_TRY(hipMemcpyAsync(c->ws + P.o_tiles, c->tiles.data(), c->tiles.size() * sizeof(Tile),
                           hipMemcpyHostToDevice, c->stream));
    // tiles per instance: a PT cycle's exchange runs in the tile that completes the instance
    c->itiles.assign(P.desc.size(), 0);
    const bool octs = P.encoding == PT_BITPACK32 ? !c->oct_as_words : c->byte_octets;
    if (!c->byte_octets)
        for (const Tile &t : c->tiles) c->itiles[t.inst] += 1;
    for (int32_t k = 0; k < P.n_otile + P.n_oblock && octs; ++k) c->itiles[P.otiles[(size_t)k * kOctRec]] += 1;
    HIP_TRY(hipMemcpyAsync(c->ws + P.o_itiles, c->itiles.data(), c->itiles.size() * 4,
                           hipMemcpyHostToDevice, c->stream));
    HIP_TRY(sweep_kernels_set_lds(c->lds_fast, c->lds_generic, c->lds_block));
    HIP_TRY(words_kernels_set_lds(c->lds_words));
    // Whole-replica tiles: two four-slice words per lane, unless the batch's lanes of one
    // colour class at that width would not give every SIMD of the device one wave; then
    // the sweep is a chain of short, barely parallel class steps, and one word per lane
    // (twice the lanes, half the dependent work each) shortens every step (measured on
    // config 2, 2304 lanes per class: 3.6e10 attempts/s against 3.0e10).  Instances with
    // 16-bit neighbour entries are swept by the two-word instantiations only, so any such
    // instance keeps the batch at two words.
    int64_t lanes = 0;
    bool ent16 = false;
    for (int k = 0; k < c->n_fast_tiles; ++k) {
        const Tile &t = c->tiles[k];
        const InstDesc &d = P.desc[t.inst];
        ent16 = ent16 || d.ent_mode == kEntXad16;
        int64_t most = 0;
        for (int g = 0; g < d.n_colors; ++g)
            most = std::max<int64_t>(most, P.cls_off[d.cls_base + g + 1] - P.cls_off[d.cls_base + g]);
        lanes += (int64_t)t.P * most * std::max(1, d.G4 / 2);
    }
    c->lane_words = (c->opt.flags & PT_FLAG_FOUR_SLICE_LANES) ? 1
                    : ((c->opt.flags & PT_FLAG_TWO_WORD_LANES) || ent16) ? 2
                    : lanes < (int64_t)c->cus * 256 ? 1
                                                    : 2;
    // At most one whole-replica tile per compute unit: no other workgroup's waves overlap a
    // tile's class steps, so the kernel forms each thread's next item while the current one
    // is in flight (the tiles whose classes fit one pass of the workgroup).
    c->lat = !(c->opt.flags & PT_FLAG_NO_LATENCY_PATH) && c->n_fast_tiles > 0 &&
             c->n_fast_tiles <= c->cus;
    return PT_OK;
}

void drop_graph(pt_ctx *c)
{
    if (c->graph) (void)hipGraphExecDestroy(c->graph);
    c->graph = nullptr;
    c->graph_cycles = 0;
}

int event_pair(pt_ctx *c, int &a, int &b)
{
    while (c->ev_pool.size() < c->ev_used + 2) {
        hipEvent_t e;
        HIP_TRY(hipEventCreate(&e));
        c->ev_pool.push_back(e);
    }
    a = (int)c->ev_used++;
    b = (int)c->ev_used++;
    return PT_OK;
}

// Accumulate the elapsed times of recorded event pairs (synchronises).
int harvest_events(pt_ctx *c)
{
    if (c->ev_used == 0) return PT_OK;
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (size_t k = 0; k < c->sweep_ev.size(); ++k) {
        const auto &p = c->sweep_ev[k];
        float ms = 0;
        HIP_TRY(hipEventElapsedTime(&ms, c->ev_pool[p.first], c->ev_pool[p.second]));
        c->sweep_ms += ms;
        c->sweep_n += k < c->sweep_ev_calls.size() ? c->sweep_ev_calls[k] : 1;
    }
    for (auto &p : c->exch_ev) {
        float ms = 0;
        HIP_TRY(hipEventElapsedTime(&ms, c->ev_pool[p.first], c->ev_pool[p.second]));
        c->exch_ms += ms;
        c->exch_n++;
    }
    for (auto &p : c->multi_ev) {
        float ms = 0;
        HIP_TRY(hipEventElapsedTime(&ms, c->ev_pool[p.first], c->ev_pool[p.second]));
        c->multi_ms += ms;
    }
    c->sweep_ev.clear();
    c->sweep_ev_calls.clear();
    c->exch_ev.clear();
    c->multi_ev.clear();
    c->ev_used = 0;
    return PT_OK;
}

bool out_of_resources(hipError_t e)
{
    return e == hipErrorLaunchOutOfResources || e == hipErrorOutOfMemory ||
           e == hipErrorInvalidConfiguration;
}

// Launch n sweeps of every tile; on a resource failure halve the tile (and, at one
// replica per tile, the workgroup) and retry, as the paper's Figure 7 halves its chain
// packing when a launch runs out of registers.
// One launch of whole-replica tiles: a run of consecutive tiles of one kind that the
// compute units can hold `per_cu` at a time.
struct LaunchGroup {
    int kind, tile0, n_tiles, lds_bytes, per_cu;
};

// Workgroups of `lds` bytes a compute unit holds at once with the current block size.
int occupancy(const pt_ctx *c, int lds)
{
    const int by_threads = std::max(1, c->cu_threads / std::max(1, c->block_threads));
    const int by_lds = lds > 0 ? std::max(1, c->cu_lds / lds) : by_threads;
    return std::min(by_threads, by_lds);
}

// Split the (LDS-descending) tile lists into occupancy classes, one launch each, sized to
// the largest tile of the class.  A single launch would reserve the largest tile's LDS for
// every workgroup and hold small tiles to the occupancy of the largest.
std::vector<LaunchGroup> launch_groups(const pt_ctx *c)
{
    std::vector<LaunchGroup> out;
    auto add_range = [&](int kind, int begin, int end) {
        int t = begin;
        while (t < end) {
            const int k = occupancy(c, c->tile_lds[t]);
            int u = t + 1;
            while (u < end && occupancy(c, c->tile_lds[u]) == k) ++u;
            out.push_back(LaunchGroup{kind, t, u - t, c->tile_lds[t], k});
            t = u;
        }
    };
    add_range(kTileFast, 0, c->n_fast_tiles);
    const int w0 = c->n_fast_tiles, w1 = w0 + c->n_words_tiles;
    int wr = w0;  // first word tile of replicas
    while (wr < w1 && c->tiles[wr].kind == kTileWords) ++wr;
    add_range(kTileWords, w0, wr);
    add_range(kTileWordsR, wr, w1);
    add_range(kTileGeneric, w1, w1 + c->n_generic_tiles);
    return out;
}

// Whether the resident slice-block kernel can hold every block tile at once with the
// current block size: the grid must fit the compute units' occupancy, or the blocks that
// wait for their neighbours could wait for blocks that never start.
hipError_t blocks_resident(pt_ctx *c, bool &resident)
{
    resident = false;
    if ((c->opt.flags & PT_FLAG_BLOCK_LAUNCH_PER_SWEEP) || c->resident_off) return hipSuccess;
    if (c->resident_key != std::make_pair(c->block_threads, c->lds_block)) {
        int32_t per_cu = 0;
        const hipError_t e = block_resident_per_cu(c->block_threads, c->lds_block, &per_cu);
        if (e != hipSuccess) return e;
        c->resident_key = std::make_pair(c->block_threads, c->lds_block);
        c->resident_per_cu = per_cu;
    }
    resident = (int64_t)c->n_block_tiles <= (int64_t)c->resident_per_cu * c->cus;
    return hipSuccess;
}

int restore(pt_ctx *c);
int recover(pt_ctx *c);

// The state region copied to the shadow copy, the journal cleared (stream-ordered: the
// copy reads the state as the calls queued so far leave it).  Only where the device error word
// is known to be 0 or the whole state was just written.
hipError_t take_snapshot(pt_ctx *c)
{
    c->journal.clear();
    if (!c->shadow) return hipSuccess;
    return hipMemcpyAsync(c->shadow, c->ws + c->plan.o_state, c->plan.state_bytes,
                          hipMemcpyDeviceToDevice, c->stream);
}

// Whether the caller is capturing the context's stream.
bool capturing(const pt_ctx *c)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &status) != hipSuccess) (void)hipGetLastError();
    return status != hipStreamCaptureStatusNone;
}

// A call captured into a caller's graph does not run now, and its replays are not seen here: from
// then on the calls that ran since a synchronisation are not known, so none is noted, nothing is
// recovered (check_err), and there are no several cycles a launch (can_coop).  The graph holds
// the shape in use, whose tile list must stay as it is: tuning, which waits for the stream and
// so cannot be captured, ends there.
void journal_add(pt_ctx *c, int kind, int n)
{
    if (c->replaying || c->captured || !(c->shadow || c->tuning)) return;
    if (capturing(c)) {
        c->captured = true;
        c->tuning = false;
    } else if (c->shadow) {
        c->journal.emplace_back(kind, n);
    }
}

int check_err(pt_ctx *c, uint32_t err);

// The error word cleared, and the counts of tiles and cycles that a tile which gave up a wait
// may have left behind.
hipError_t clear_err(pt_ctx *c)
{
    const Plan &P = c->plan;
    const size_t n = P.desc.size() * 4;
    hipError_t e = hipMemsetAsync(c->ws + P.o_err, 0, 4, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws + P.o_icount, 0, n, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws + P.o_icycle, 0, n, c->stream);
    return e;
}

// Wait for the stream, then check the device error word (a resident slice-block launch
// that gave up a wait, an octet kernel that refused to run).  After a wait that gave up,
// the state is restored from the copy of the last clean synchronisation and the calls
// queued since are replayed with every slice block launched per sweep (or per parity),
// which gives the chain's state again; otherwise, and once a caller has captured a call, the
// call fails with PT_ESTATE (the word is cleared, and the chain state after such a launch is
// not the sampler's).  A clean synchronisation after new calls takes a new copy.
int sync_and_check(pt_ctx *c)
{
    uint32_t *err = reinterpret_cast<uint32_t *>(c->obs_pin);
    HIP_TRY(launch_gather_err(c->st, err, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return check_err(c, *err);
}

// The second half of sync_and_check, with the error word read by a launch that the stream
// has been waited for.
int check_err(pt_ctx *c, uint32_t err)
{
    if (err != 0) {
        c->last_device_error = err;
        HIP_TRY(clear_err(c));
        if (err & kErrLdsBase)
            return fail(PT_ESTATE, "an octet kernel found its dynamic LDS away from address 0 "
                                   "and did not run; the state is inconsistent");
        const bool known = c->shadow && !c->replaying;  // the state to restore
        if (known && c->captured && (err & (kErrWait | kErrPlace)))
            return fail(PT_ESTATE, "a resident launch gave up a wait, and replays of a caller's graph "
                                   "may have run since the last synchronisation; the state is inconsistent");
        if ((err & kErrPlace) && known) return recover(c);
        if (err & kErrPlace)
            return fail(PT_ESTATE, "the workgroups of a resident slice-block launch did not keep "
                                   "to round-robin XCDs; the state is inconsistent");
        if (err & kErrQueue)
            return fail(PT_ESTATE, "a whole-octet workgroup found every work queue empty; the "
                                   "state is inconsistent");
        if (known) return recover(c);
        return fail(PT_ESTATE, "a launch whose workgroups wait for each other gave up a wait; the "
                               "state is inconsistent");
    }
    if (!c->journal.empty() && !c->replaying) HIP_TRY(take_snapshot(c));
    return PT_OK;
}

// E_cl and C of replicas [rep_first, rep_first + n) from the spins in device memory (the
// bit-packed encoding recomputes every replica).
hipError_t energies_from_spins(pt_ctx *c, int rep_first, int n)
{
    if (c->plan.encoding == PT_BITPACK32)
        return launch_bp_energy(c->st, c->plan.bp_n_eblk, (int32_t)c->plan.total_reps, c->stream);
    return launch_energy(c->st, rep_first, n, c->stream);
}

// Whole octets from the device work queue: as many workgroups as the compute units hold at
// once for the current block size (at most one per octet).
// Resident byte slice blocks pass their records through the L2 of the XCD that holds their
// replica's ring.
bool block_ring_xcd(const pt_ctx *c)
{
    return c->block_xcd && c->n_block_tiles > 0 && !c->byte_octets && !c->resident_off &&
           !(c->opt.flags & (PT_FLAG_DEVICE_SCOPE_RECORDS | PT_FLAG_BLOCK_LAUNCH_PER_SWEEP));
}

// Resident octet slice blocks pass their records through the L2 of the XCD that holds
// their ring (the rings were placed one per XCD).
bool oct_ring_xcd(const pt_ctx *c)
{
    return c->oct_resident && c->plan.oblock_xcd &&
           !(c->opt.flags & PT_FLAG_DEVICE_SCOPE_RECORDS);
}

// Poll bound of the waits between the cycles of a launch.  An instance's tiles run unevenly
// where some share a unit and others do not, and they meet once a cycle: 66 octets of 2600 sites
// and 32 slices, 264 blocks on 256 units, take 65 us a sweep and 64 of them, a block a unit, 43;
// with 2000 sweeps a cycle the 66 gave up a bound of kCoopPolls alone (a poll takes some 0.6 us).
// A sweep's part grows with the classes, each a step of its own.  (Two contexts that each hold
// part of the chip wait for each other: the sooner they give up, the less that costs.)
int coop_polls(const pt_ctx *c)
{
    int64_t colors = 1;
    for (const auto &d : c->plan.desc) colors = std::max<int64_t>(colors, d.n_colors);
    return kCoopPolls + (int)std::min<int64_t>(c->opt.sweeps_per_exchange * (64 + 4 * colors), 1 << 30);
}

// Bit-packed encoding: n_sweeps sweeps as one launch per colour class (parity, colour) of
// every instance, then E_cl and C of every replica.
// cycles: PT cycles of a batch of resident octet blocks (can_coop), their exchange steps too.
int enqueue_bp_sweep(pt_ctx *c, int n_sweeps, bool fuse_exchange, int cycles = 0)
{
    const Plan &P = c->plan;
    const bool timing = (c->opt.flags & PT_FLAG_TIMING) != 0;
    int ea = -1, eb = -1;
    if (timing) {
        int rc = event_pair(c, ea, eb);
        if (rc) return rc;
        HIP_TRY(hipEventRecord(c->ev_pool[ea], c->stream));
    }
    // octets: whole octets in one launch for all sweeps of the call; slice blocks in one
    // resident launch, or else one launch per parity of every sweep, their E_cl and C
    // cleared first and summed by the resident launch or the last phase launch
    OctLaunch O{};
    O.st = c->st;
    O.key0 = c->key_flip0;
    O.key1 = c->key_flip1;
    O.n_sweeps = n_sweeps;
    if (P.n_otile > 0 && !c->oct_as_words) {
        O.tile0 = 0;
        O.n_tiles = P.n_otile;
        O.threads = c->block_threads;
        O.lds_bytes = P.otile_lds;
        O.queue = c->oct_queue ? 1 : 0;
        if (fuse_exchange) {
            O.fuse = 1;
            O.swap_key0 = c->key_swap0;
            O.swap_key1 = c->key_swap1;
            O.t_add = (uint32_t)n_sweeps;
        }
        const hipError_t e = launch_oct_tiles(O, c->stream);
        if (e != hipSuccess) return hip_fail(e, "octet tile launch");
        O.queue = O.fuse = 0;
    }
    if (c->n_words_tiles > 0) {
        SweepLaunch W{};
        W.st = c->st;
        W.key0 = c->key_flip0;
        W.key1 = c->key_flip1;
        W.n_sweeps = n_sweeps;
        W.block_threads = c->block_threads;
        W.fuse_exchange = fuse_exchange ? 1 : 0;
        W.swap_key0 = c->key_swap0;
        W.swap_key1 = c->key_swap1;
        W.t_add = (uint32_t)n_sweeps;
        for (const LaunchGroup &g : launch_groups(c)) {
            W.tile0 = g.tile0;
            W.n_tiles = g.n_tiles;
            W.lds_bytes = g.lds_bytes;
            const hipError_t e = launch_sweep(W, g.kind, c->stream);
            if (e != hipSuccess) return hip_fail(e, "word tile launch");
        }
    }
    if (P.n_oblock > 0) {
        O.tile0 = P.n_otile;
        O.n_tiles = P.n_oblock;
        O.threads = P.oblock_threads;
        O.lds_bytes = P.oblock_lds;
        O.split = P.oblock_split ? 1 : 0;
        hipError_t e = launch_oct_clear(O, c->stream);
        if (e != hipSuccess) return hip_fail(e, "octet clear launch");
        if (c->oct_resident) {
            O.lds_bytes = P.oblock_res_lds;
            O.rec_words = (int32_t)P.orec_words;
            O.xcd_local = !oct_ring_xcd(c) ? 0 : (c->opt.flags & PT_FLAG_TEST_XCD_MISMATCH) ? 2 : 1;
            O.cycles = cycles;
            O.cycle_polls = coop_polls(c);
            if (c->opt.flags & PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT) {
                O.wait_polls = O.cycle_polls = 16;
                O.wait_extra = 1 << 30;
            }
            O.dev = reinterpret_cast<const DevState *>(c->ws + P.o_dev);
            O.swap_key0 = c->key_swap0;
            O.swap_key1 = c->key_swap1;
            O.t_add = (uint32_t)n_sweeps;
            e = launch_oct_resident(O, c->stream);
            if (e != hipSuccess) return hip_fail(e, "octet resident launch");
        }
        for (int sw = 0; sw < n_sweeps && !c->oct_resident; ++sw)
            for (int p = 0; p < 2; ++p) {
                O.sweep_off = sw;
                O.p = p;
                O.last = (sw == n_sweeps - 1 && p == 1) ? 1 : 0;
                e = launch_oct_phase(O, c->stream);
                if (e != hipSuccess) return hip_fail(e, "octet slice-block launch");
            }
    }
    if (P.bp_generic) {
        int parities = 1;
        for (const auto &d : P.desc) parities = std::max(parities, d.parities);
        BpLaunch L{};
        L.st = c->st;
        L.key0 = c->key_flip0;
        L.key1 = c->key_flip1;
        for (int sw = 0; sw < n_sweeps; ++sw)
            for (int p = 0; p < parities; ++p)
                for (int g = 0; g < (int)P.bp_colour.size(); ++g) {
                    L.sweep_off = sw;
                    L.p = p;
                    L.g = g;
                    L.blk0 = P.bp_colour[g].first;
                    L.n_blocks = P.bp_colour[g].second;  // instances with one parity skip p = 1
                    if (L.n_blocks == 0) continue;
                    const hipError_t e = launch_bp_sweep(L, c->stream);
                    if (e != hipSuccess) return hip_fail(e, "bit-packed sweep launch");
                }
        // E_cl and C of every replica (the octets' are recomputed to the same values)
        const hipError_t e = energies_from_spins(c, 0, (int)P.total_reps);
        if (e != hipSuccess) return hip_fail(e, "bit-packed energy launch");
    }
    if (timing) {
        HIP_TRY(hipEventRecord(c->ev_pool[eb], c->stream));
        c->sweep_ev.emplace_back(ea, eb);
        c->sweep_ev_calls.push_back(1);
    }
    return PT_OK;
}

// n_sweeps sweeps of every tile; with fuse_exchange the tile that completes an instance
// then runs the instance's exchange step (a PT cycle in one set of launches).
// Every tile a fast whole-replica tile holding a whole instance (the condition for a
// launch of several PT cycles).
bool whole_instance_tiles(const pt_ctx *c)
{
    if (c->byte_octets || c->n_words_tiles != 0 || c->n_generic_tiles != 0 || c->n_block_tiles != 0 || c->n_fast_tiles != n_inst_of(c))
        return false;
    for (int k = 0; k < c->n_fast_tiles; ++k) {
        const Tile &t = c->tiles[k];
        const InstDesc &d = c->plan.desc[t.inst];
        // the multi-cycle kernel does not carry 16-bit neighbour entries
        if (t.c0 != 0 || t.P != d.R || d.ent_mode == kEntXad16) return false;
    }
    return true;
}

// Whether the whole-replica tiles sweep on the latency path with workgroups of `threads`:
// at most one tile per compute unit (no other workgroup overlaps a tile's class steps),
// and in some tile every step of the pipelined order (class k of parity 0 with class k - 1
// of parity 1) fits one pass of the workgroup, at least two classes and a degree of at
// most eight.  The kernel checks the per-tile condition again and sweeps the other tiles
// as usual.
bool latency_path(const pt_ctx *c, int threads)
{
    if (!c->lat || c->byte_octets) return false;
    bool any = false;
    for (int k = 0; k < c->n_fast_tiles && !any; ++k) {
        const Tile &t = c->tiles[k];
        const InstDesc &d = c->plan.desc[t.inst];
        if (d.n_colors < 2 || d.D < 1 || d.D > 8) continue;
        const int nw = (c->lane_words == 2 && d.G4 >= 2) ? 2 : 1;
        const int64_t lanes = (int64_t)t.P * (d.G4 / nw);  // per site
        if (lanes > threads) continue;
        const int32_t *off = c->plan.cls_off.data() + d.cls_base;
        int most = 0;
        for (int g = 0; g < d.n_colors; ++g) {
            const int gb = (g == 0 ? d.n_colors : g) - 1;
            most = std::max(most, off[g + 1] - off[g] + off[gb + 1] - off[gb]);
        }
        any = (int64_t)most * lanes <= threads;
    }
    return any;
}

// enqueue_sweep_once with cycles > 1 found the tiles no longer whole instances (after a
// launch-failure fallback): nothing was queued, run the cycles one by one.
constexpr int kCycleByCycle = 1;

int enqueue_sweep_once(pt_ctx *c, int n_sweeps, bool fuse_exchange, int cycles = 1)
{
    if (n_sweeps <= 0) return PT_OK;
    const bool timing = (c->opt.flags & PT_FLAG_TIMING) != 0;
    for (;;) {
        if (cycles > 1 && !whole_instance_tiles(c)) return kCycleByCycle;
        SweepLaunch L{};
        L.st = c->st;
        L.key0 = c->key_flip0;
        L.key1 = c->key_flip1;
        L.n_sweeps = n_sweeps;
        L.block_threads = c->block_threads;
        L.lane_words = c->lane_words;
        L.lat = latency_path(c, c->block_threads) ? 1 : 0;
        L.fuse_exchange = fuse_exchange ? 1 : 0;
        L.swap_key0 = c->key_swap0;
        L.swap_key1 = c->key_swap1;
        L.t_add = (uint32_t)n_sweeps;
        L.cycles = cycles;
        int ea = -1, eb = -1;
        if (timing) {
            int rc = event_pair(c, ea, eb);
            if (rc) return rc;
            HIP_TRY(hipEventRecord(c->ev_pool[ea], c->stream));
        }
        hipError_t e = hipSuccess;
        int queued = 0;  // launches of this call already queued
        if (c->inject_pending) {
            c->inject_pending = false;
            e = hipErrorLaunchOutOfResources;
        } else {
            for (const LaunchGroup &g : launch_groups(c)) {
                L.tile0 = g.tile0;
                L.n_tiles = g.n_tiles;
                L.lds_bytes = g.lds_bytes;
                e = launch_sweep(L, g.kind, c->stream);
                if (e != hipSuccess) break;
                ++queued;
            }
            // slice blocks: boundary records of the current state (and E_cl, C cleared),
            // then all sweeps in one launch when every block can be resident at once,
            // else one launch per sweep
            L.tile0 = c->n_fast_tiles + c->n_words_tiles + c->n_generic_tiles;
            L.n_tiles = c->n_block_tiles;
            L.lds_bytes = c->lds_block;
            if (e == hipSuccess && L.n_tiles > 0) {
                e = launch_block_prepare(L, c->stream);
                if (e == hipSuccess) ++queued;
            }
            if (e == hipSuccess && L.n_tiles > 0) {
                bool resident = false;
                e = blocks_resident(c, resident);
                c->block_persistent = resident ? 1 : 0;
                if (e == hipSuccess && resident) {
                    L.persist = 1;
                    L.xcd_local = !block_ring_xcd(c) ? 0
                                  : (c->opt.flags & PT_FLAG_TEST_XCD_MISMATCH) ? 2 : 1;
                    if (c->opt.flags & PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT) {
                        L.wait_polls = 16;
                        L.wait_extra = 1 << 30;
                    }
                    L.sweep_off = 0;
                    L.last = 1;
                    e = launch_sweep(L, kTileBlock, c->stream);
                    if (e == hipSuccess) ++queued;
                } else {
                    for (int sw = 0; sw < n_sweeps && e == hipSuccess; ++sw) {
                        L.sweep_off = sw;
                        L.last = (sw == n_sweeps - 1);
                        e = launch_sweep(L, kTileBlock, c->stream);
                        if (e == hipSuccess) ++queued;
                    }
                }
            }
        }
        if (e == hipSuccess) {
            if (timing) {
                HIP_TRY(hipEventRecord(c->ev_pool[eb], c->stream));
                if (cycles > 1) {
                    c->multi_ev.emplace_back(ea, eb);
                } else {
                    c->sweep_ev.emplace_back(ea, eb);
                    c->sweep_ev_calls.push_back(1);
                }
            }
            if (cycles > 1) {
                c->multi_launches += 1;
                c->multi_cycles += cycles;
            }
            return PT_OK;
        }
        if (timing) c->ev_used -= 2;
        if (!out_of_resources(e)) return hip_fail(e, "sweep launch");
        if (queued > 0)  // part of the call already runs: retrying would sweep it twice
            return fail(PT_ESTATE, std::string("a sweep launch failed after part of the call "
                                               "was queued; the state is inconsistent: ") +
                                       hipGetErrorString(e));
        (void)hipGetLastError();
        c->fallbacks++;
        drop_graph(c);
        if (c->max_P > 1) {
            int rc = build_tiles(c, std::max(1, c->max_P / 2), 0);
            if (rc) return rc;
        } else if (c->block_threads > 64) {
            c->block_threads /= 2;
            c->coop_fits = -1;
            if (c->n_words_tiles > 0) {  // a word tile needs a thread per lane of a site
                const int rc = build_tiles(c, 1, 0);
                if (rc) return rc;
            }
        } else {
            return fail(PT_ELAUNCH, std::string("sweep kernel cannot be launched: ") +
                                        hipGetErrorString(e));
        }
    }
}

// Batches of at most this many tiles run a PT cycle as one set of launches, the exchange
// step in the tile that completes each instance.  Every tile then waits for its stores and
// counts itself, which costs more than the separate exchange launch it saves once a call has
// hundreds of tiles; small batches are launch-latency bound and gain (measured a cycle, separate
// and fused: 1 tile +22 %, 32 tiles +4 %, 510 tiles 209.7 us and 217.3, 1155 tiles 454 and 475,
// 2303 tiles 782 and 826).
constexpr size_t kFuseMaxTiles = 64;

// Whether a PT cycle's exchange step runs in the sweep launches of the route in use.
bool can_fuse(const pt_ctx *c)
{
    if (c->plan.encoding == PT_BITPACK32 || c->byte_octets) return c->oct_fuse;
    // word tiles: whatever their number
    return c->tiles.size() <= kFuseMaxTiles || c->n_words_tiles == (int)c->tiles.size();
}

// Whether octet slice blocks are the whole batch on the route in use.
bool octet_blocks(const pt_ctx *c)
{
    const Plan &P = c->plan;
    return P.n_oblock > 0 && P.n_otile == 0 && !P.bp_generic &&
           (P.encoding == PT_BITPACK32 ? c->n_words_tiles == 0 : c->byte_octets);
}

// Whether pt_run may run several cycles per launch of tiles that wait for each other between
// cycles: every tile a word tile or, at most one per unit and on the latency path, a fast byte
// tile; a launch per kind, each resident as a whole.  Or every octet in resident slice blocks.  Not
// under PT_FLAG_TIMING, which times sweeps.
bool can_coop(pt_ctx *c)
{
    if (!c->shadow || c->resident_off || c->captured || c->inject_pending ||
        (c->opt.flags & (PT_FLAG_TAU_CORR | PT_FLAG_NO_GRAPH | PT_FLAG_TIMING)))
        return false;
    if (octet_blocks(c)) return c->oct_resident;
    if (c->byte_octets) return false;
    if (c->plan.encoding == PT_BITPACK32 && (!c->oct_fuse || (c->plan.n_otile > 0 && !c->oct_as_words)))
        return false;
    if (c->tiles.empty() || (int)c->tiles.size() != c->n_words_tiles + c->n_fast_tiles) return false;
    if (c->coop_fits < 0) {
        c->coop_fits = 1;
        for (int kind : {kTileFast, kTileWords, kTileWordsR}) {
            int64_t n = 0;
            int lds = 0;
            for (size_t k = 0; k < c->tiles.size(); ++k)
                if (c->tiles[k].kind == kind) {
                    ++n;
                    lds = std::max(lds, c->tile_lds[k]);
                }
            if (n == 0) continue;
            int32_t per_cu = 0;
            const hipError_t e = kind == kTileFast
                                     ? fast_resident_per_cu(c->block_threads, lds, &per_cu)
                                     : words_resident_per_cu(kind == kTileWordsR, c->block_threads, lds, &per_cu);
            if (e != hipSuccess) (void)hipGetLastError();
            if (e != hipSuccess || n > (int64_t)per_cu * c->cus || (kind == kTileFast && !latency_path(c, c->block_threads)))
                c->coop_fits = 0;
        }
    }
    return c->coop_fits > 0;
}

// Whether launches of the shape in use may wait for other workgroups (and so may give up).
bool waits(pt_ctx *c)
{
    return c->plan.halo_words > 0 ||
           (c->plan.n_oblock > 0 && (c->plan.encoding == PT_BITPACK32 || c->byte_octets)) ||
           (can_coop(c) && !whole_instance_tiles(c));
}

// `cycles` PT cycles in one launch per kind of tile (can_coop holds).
int enqueue_coop(pt_ctx *c, int cycles)
{
    if (octet_blocks(c)) {
        const int rc = enqueue_bp_sweep(c, c->opt.sweeps_per_exchange, false, cycles);
        if (rc) return rc;
        c->multi_launches += 1;
        c->multi_cycles += cycles;
        return PT_OK;
    }
    SweepLaunch L{};
    L.st = c->st;
    L.key0 = c->key_flip0;
    L.key1 = c->key_flip1;
    L.n_sweeps = c->opt.sweeps_per_exchange;
    L.block_threads = c->block_threads;
    L.lane_words = c->lane_words;
    L.lat = 1;
    L.fuse_exchange = 1;
    L.swap_key0 = c->key_swap0;
    L.swap_key1 = c->key_swap1;
    L.t_add = (uint32_t)L.n_sweeps;
    L.cycles = cycles;
    L.coop = 1;
    L.wait_polls = coop_polls(c);
    if (c->opt.flags & PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT) {
        L.wait_polls = 16;
        L.wait_extra = 1 << 30;
    }
    for (int at = 0; at < (int)c->tiles.size();) {
        L.tile0 = at;
        L.lds_bytes = 0;
        const int kind = c->tiles[at].kind;
        for (; at < (int)c->tiles.size() && c->tiles[at].kind == kind; ++at)
            L.lds_bytes = std::max(L.lds_bytes, c->tile_lds[at]);
        L.n_tiles = at - L.tile0;
        const hipError_t e = launch_sweep(L, kind, c->stream);
        if (e != hipSuccess) return hip_fail(e, "sweep launch of several cycles");
    }
    c->multi_launches += 1;
    c->multi_cycles += cycles;
    return PT_OK;
}

// Self-tuning: while candidates remain, each sweep launch uses the next candidate shape
// and is timed (synchronously) with its own events.  The candidates are run in
// kTuneRounds rounds, each keeping its best per-sweep time (one timing of a short call
// can be off by more than the gap between shapes), all but the fastest quarter only in the
// first two, and the fastest shape is kept.  Shapes with the same tiles are one candidate, and
// a shape that runs several cycles a launch is timed so from the second round on, over as many
// cycles as keep the whole tuning within kTuneCycles (320 replicas of 336 x 64 spins take 87.9 us
// a cycle in resident tiles of 2 and 101.7 in tiles of 1; over two cycles a launch the two timed
// alike).  With 13 shapes or more that is the third round only.
// Launch shape does not change the trajectory, so tuning costs only the slower
// candidates' extra time.
//
// A timed launch whose tiles wait for each other is checked before the next: the shape that
// wins may be one that never waits and keeps no copy to restore, and once a wait has been given
// up no tile waits, so such shapes would time too fast.  The copy is taken anew before the
// launch, so that only its own cycles are run again after it, and the round starts over with
// resident launches off.
constexpr size_t kTuneRounds = 3;
// Cycles that tuning takes at most when no wait is given up: three of each of the fifteen shapes
// of a byte batch, what it took before shapes ran several cycles a launch, so that a warm-up that
// was long enough is so still.
constexpr int kTuneCycles = 45;
// Candidates of the third round, of n in the second.
size_t tune_finalists(size_t n) { return std::min(n, std::max<size_t>(2, (n + 3) / 4)); }
// Cycles a launch of a candidate that runs several is timed over, with `left` of kTuneCycles for
// the rest of the tuning as the round begins.
int tune_cycles(const pt_ctx *c, int left)
{
    const int n = (int)c->cand_order.size();
    if (c->tune_round + 1 < kTuneRounds) left -= 2 * (int)tune_finalists(c->cand_order.size());
    return std::max(1, std::min({8, std::max(2, 24 / n), left / n}));
}
uint64_t tiles_hash(const pt_ctx *c)
{
    uint64_t h = 1469598103934665603ull;
    for (const Tile &t : c->tiles)
        for (const int32_t v : {t.inst, t.c0, t.P, t.kind, t.g0, t.ng}) h = (h ^ (uint32_t)v) * 1099511628211ull;
    return h;
}
// fused: ask for the exchange step too; set to whether the launches run it (the candidate's
// route decides).
// cycles: how many PT cycles are asked for (with fused); set to those the call ran.
int enqueue_sweep(pt_ctx *c, int n_sweeps, bool *fused = nullptr, int *cycles = nullptr)
{
    if (n_sweeps <= 0) return PT_OK;
    const bool bp = c->plan.encoding == PT_BITPACK32;
    auto sweep = [&]() {
        const bool fuse = fused && can_fuse(c);
        if (fused) *fused = fuse;
        return bp || c->byte_octets ? enqueue_bp_sweep(c, n_sweeps, fuse) : enqueue_sweep_once(c, n_sweeps, fuse);
    };
    const int ask = cycles ? *cycles : 1;
    if (cycles) *cycles = 1;
    if (!c->tuning) return sweep();
    auto use = [&](size_t k) -> int {
        const pt_ctx::Shape &s = c->cand[k];
        c->block_threads = s.threads;
        c->coop_fits = -1;
        (bp ? c->oct_as_words : c->byte_octets) = s.alt;
        if (bp && c->n_words_tiles == 0 && !c->plan.words_alt) return PT_OK;
        return build_tiles(c, s.replicas > 0 ? s.replicas : c->opt.tile_replicas, s.tile_bytes);
    };
    int rc = PT_OK;
    size_t k = 0;
    for (;;) {
        k = c->cand_order[c->cand_next];
        rc = use(k);
        if (rc) return rc;
        if (c->tune_round > 0) break;
        c->cand[k].tiles = tiles_hash(c);
        bool again = false;
        for (size_t j = 0; j < c->cand_next; ++j) {
            const pt_ctx::Shape &x = c->cand[c->cand_order[j]], &y = c->cand[k];
            again = again || (x.tiles == y.tiles && x.threads == y.threads && x.alt == y.alt);
        }
        if (!again) break;
        c->cand_order.erase(c->cand_order.begin() + (ptrdiff_t)c->cand_next);
        if (c->cand_next == c->cand_order.size()) {  // the first candidate again, in its next round
            c->cand_next = 0;
            c->tune_round = 1;
        }
    }
    const int fb = c->fallbacks;
    if (c->cand_next == 0) c->tune_most = tune_cycles(c, kTuneCycles - c->tune_done);
    const int most = c->tune_most;
    const int n_cyc = fused && c->tune_round > 0 && can_coop(c) && !whole_instance_tiles(c) ? std::min(ask, most) : 1;
    const bool waiting = c->shadow && !c->replaying &&
                         (n_cyc > 1 || (c->byte_octets && c->plan.n_oblock > 0 && c->oct_resident));
    if (waiting) {
        HIP_TRY(take_snapshot(c));
        c->journal.emplace_back(fused ? 2 : 0, fused ? ask : n_sweeps);  // the rest of this call
    }
    HIP_TRY(hipEventRecord(c->tune_ev[0], c->stream));
    if (n_cyc > 1) {
        *fused = true;
        *cycles = n_cyc;
        rc = enqueue_coop(c, n_cyc);
    } else {
        rc = sweep();
    }
    if (rc) return rc;
    HIP_TRY(hipEventRecord(c->tune_ev[1], c->stream));
    HIP_TRY(hipEventSynchronize(c->tune_ev[1]));
    if (waiting) {
        uint32_t *err = reinterpret_cast<uint32_t *>(c->obs_pin);
        HIP_TRY(launch_gather_err(c->st, err, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        if (*err & ~(kErrWait | kErrPlace)) return check_err(c, *err);
        if (*err != 0) {
            c->last_device_error = *err;
            if ((rc = restore(c))) return rc;
            c->recoveries += 1;
            c->cand_ms.assign(c->cand.size(), 1e30);
            c->cand_next = 0;
            c->tune_done = (int)c->tune_round * (int)c->cand_order.size();
            if (cycles) *cycles = ask;
            return enqueue_sweep(c, n_sweeps, fused, cycles);
        }
    }
    float ms = 0;
    HIP_TRY(hipEventElapsedTime(&ms, c->tune_ev[0], c->tune_ev[1]));
    const double t = (c->fallbacks == fb) ? (double)ms / ((double)n_sweeps * n_cyc) : 1e30;
    c->cand_ms[k] = std::min(c->cand_ms[k], t);
    c->tune_done += n_cyc;
    if (++c->cand_next < c->cand_order.size()) return PT_OK;
    c->cand_next = 0;
    std::stable_sort(c->cand_order.begin(), c->cand_order.end(),
                     [&](size_t x, size_t y) { return c->cand_ms[x] < c->cand_ms[y]; });
    if (++c->tune_round < kTuneRounds) {
        // (a process's first launch of a kernel loads its code, which spoils its first time)
        if (c->tune_round == 2)
            c->cand_order.resize(tune_finalists(c->cand_order.size()));
        return PT_OK;
    }
    c->tuning = false;
    rc = use(c->cand_order[0]);
    if (rc == PT_OK && c->shadow && !waits(c)) {
        // no launch whose tiles wait for each other after all, and those timed were checked:
        // nothing to recover from.  (The memory stays until pt_free: freeing it here would
        // wait for every stream of the device.)
        c->shadow = nullptr;
        c->journal.clear();
    }
    return rc;
}

int enqueue_exchange(pt_ctx *c, uint32_t t_add)
{
    const bool timing = (c->opt.flags & PT_FLAG_TIMING) != 0;
    int ea = -1, eb = -1;
    if (timing) {
        int rc = event_pair(c, ea, eb);
        if (rc) return rc;
        HIP_TRY(hipEventRecord(c->ev_pool[ea], c->stream));
    }
    hipError_t e = launch_exchange(c->st, n_inst_of(c), c->key_swap0, c->key_swap1, t_add,
                                   c->stream);
    if (e != hipSuccess) return hip_fail(e, "exchange launch");
    if (timing) {
        HIP_TRY(hipEventRecord(c->ev_pool[eb], c->stream));
        c->exch_ev.emplace_back(ea, eb);
    }
    return PT_OK;
}

static_assert(kTauLags == PT_TAU_LAGS, "device and ABI correlation lags differ");

// With PT_FLAG_TAU_CORR: after an exchange step, the imaginary-time correlations of
// every replica at its new rung.
int enqueue_tau_corr(pt_ctx *c)
{
    if (!(c->opt.flags & PT_FLAG_TAU_CORR)) return PT_OK;
    // workgroups per replica: about 8192 (parity, site, four-slice group) positions each,
    // for the largest replica of the batch
    int64_t most = 1;
    for (const auto &d : c->plan.desc) most = std::max<int64_t>(most, (int64_t)d.parities * d.N * d.G4);
    const int32_t chunks = (int32_t)std::min<int64_t>(64, (most + 8191) / 8192);
    const hipError_t e = launch_tau_corr(c->st, (int32_t)c->plan.total_reps, chunks, c->stream);
    if (e != hipSuccess) return hip_fail(e, "correlation launch");
    return PT_OK;
}

// cycles: as for enqueue_sweep.
int enqueue_cycle(pt_ctx *c, int *cycles = nullptr)
{
    const int k = c->opt.sweeps_per_exchange;
    bool fused = false;
    int rc = enqueue_sweep(c, k, &fused, cycles);
    if (rc == PT_OK && !fused) rc = enqueue_exchange(c, (uint32_t)k);
    if (rc) return rc;
    return enqueue_tau_corr(c);
}

// Instances of at most this many replicas are read back through the pinned buffer (164 bytes a
// replica, kept with the context, its offsets 32 bits), larger ones by a copy per array.  With the
// binding's Python 208 us by the buffer and 345 by copies at 16385 replicas, 906 and 797 at 65536.
constexpr int32_t kObsReplicas = 1 << 15;

// pt_observables by a copy per array.
int copy_observables(pt_ctx *c, int32_t inst, pt_obs *o)
{
    const Plan &P = c->plan;
    const InstDesc &d = P.desc[inst];
    const size_t R = (size_t)d.R, b = (size_t)d.rep_base, pb = (size_t)d.pair_base;
    const int rc = sync_and_check(c);
    if (rc) return rc;
    std::vector<int32_t> label;
    try {
        if (o->label) label.resize(R);
    } catch (...) {
        return fail(PT_ENOMEM, "host staging allocation failed");
    }
    Counters ctr{};
    const struct {
        void *dst;
        size_t off, bytes;
    } arrays[] = {
        {o->E_cl, P.o_E + 8 * b, 8 * R}, {o->C, P.o_C + 8 * b, 8 * R},
        {o->rung_of, P.o_rung + 4 * b, 4 * R}, {o->replica_of, P.o_repof + 4 * b, 4 * R},
        {o->acc, P.o_acc + 8 * pb, 8 * (R - 1)}, {o->att, P.o_att + 8 * pb, 8 * (R - 1)},
        {o->roundtrips, P.o_rt + 8 * b, 8 * R}, {label.data(), P.o_label + 4 * b, 4 * label.size()},
        {o->sumE, P.o_sumE + 8 * b, 8 * R}, {o->sumC, P.o_sumC + 8 * b, 8 * R},
        {o->sumE2, P.o_sumE2 + 8 * b, 8 * R}, {o->sumC2, P.o_sumC2 + 8 * b, 8 * R},
        {o->nup, P.o_nup + 8 * b, 8 * R}, {o->ndown, P.o_ndown + 8 * b, 8 * R},
        {o->sumCt, P.o_sumCt + 8 * PT_TAU_LAGS * b, 8 * PT_TAU_LAGS * R},
        {&ctr, P.o_ctr + sizeof(Counters) * (size_t)inst, sizeof(Counters)}};
    for (const auto &a : arrays)
        if (a.dst && a.bytes)
            HIP_TRY(hipMemcpyAsync(a.dst, c->ws + a.off, a.bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (size_t r = 0; r < label.size(); ++r) o->label[r] = (int8_t)label[r];
    o->t = ctr.t;
    o->e = ctr.e;
    o->n_acc = ctr.n_acc;
    return PT_OK;
}

int check_inst(pt_ctx *c, int32_t inst)
{
    if (!c) return fail(PT_EINVAL, "null context");
    if (inst < 0 || inst >= n_inst_of(c)) return fail(PT_EINVAL, "instance index out of range");
    return PT_OK;
}

}  // namespace

int ptq::report_error(int code, const char *msg) { return fail(code, msg); }

extern "C" {

int pt_workspace_bytes(const pt_instance *inst, int32_t n_inst, const pt_options *opt,
                       size_t *bytes)
{
    if (!bytes || !opt) return fail(PT_EINVAL, "null argument");
    Plan P;
    int rc = make_plan(inst, n_inst, *opt, P);
    if (rc) return rc;
    *bytes = P.total_bytes;
    return PT_OK;
}

int pt_init(pt_ctx **out, const pt_instance *inst, int32_t n_inst, const pt_options *opt,
            void *stream, void *workspace, size_t workspace_bytes)
{
    if (!out || !opt) return fail(PT_EINVAL, "null argument");
    *out = nullptr;
    if (opt->sweeps_per_exchange < 1) return fail(PT_EINVAL, "sweeps_per_exchange must be >= 1");
    if (opt->encoding != PT_INT8 && opt->encoding != PT_BITPACK32)
        return fail(PT_EINVAL, "unknown encoding");
    if (opt->encoding == PT_BITPACK32 && (opt->flags & PT_FLAG_TAU_CORR))
        return fail(PT_EINVAL, "PT_FLAG_TAU_CORR needs PT_INT8 spins");
    if (opt->block_threads < 0 || opt->block_threads > 1024 || (opt->block_threads % 64))
        return fail(PT_EINVAL, "block_threads must be a multiple of 64 in [64, 1024] or 0");
    if (opt->tile_replicas < 0 || opt->tile_bytes < 0)
        return fail(PT_EINVAL, "tile_replicas and tile_bytes must be >= 0");
    pt_ctx *c = new (std::nothrow) pt_ctx();
    if (!c) return fail(PT_ENOMEM, "host allocation failed");
    int rc = make_plan(inst, n_inst, *opt, c->plan);
    if (rc) {
        delete c;
        return rc;
    }
    const Plan &P = c->plan;
    c->opt = *opt;
    c->inject_pending = (opt->flags & PT_FLAG_INJECT_LAUNCH_OOR_ONCE) != 0;
    c->key_flip0 = (uint32_t)opt->seed;
    c->key_flip1 = (uint32_t)(opt->seed >> 32);
    c->key_swap0 = c->key_flip0;
    c->key_swap1 = c->key_flip1 ^ kDomainSwap;
    auto cleanup = [&](int code) {
        pt_free(c);
        return code;
    };
    hipError_t e = hipGetDevice(&c->device);
    if (e != hipSuccess) return cleanup(hip_fail(e, "hipGetDevice"));
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, c->device) ==
            hipSuccess && v > 0)
        c->lds_limit = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, c->device) ==
            hipSuccess && v > 0)
        c->cus = v;
    c->cu_lds = c->lds_limit;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, c->device) ==
            hipSuccess && v > 0)
        c->cu_lds = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxThreadsPerMultiProcessor, c->device) ==
            hipSuccess && v > 0)
        c->cu_threads = v;
    if (workspace) {
        if (workspace_bytes < P.total_bytes)
            return cleanup(fail(PT_ENOMEM, "workspace smaller than pt_workspace_bytes()"));
        if (((uintptr_t)workspace) % 256)
            return cleanup(fail(PT_EINVAL, "workspace must be 256-byte aligned"));
        c->ws = (char *)workspace;
    } else {
        e = hipMalloc((void **)&c->ws, P.total_bytes);
        if (e != hipSuccess) return cleanup(fail(PT_ENOMEM, "hipMalloc of the workspace failed"));
        c->own_ws = true;
    }
    if (stream) {
        c->stream = (hipStream_t)stream;
    } else {
        e = hipStreamCreate(&c->stream);
        if (e != hipSuccess) return cleanup(hip_fail(e, "hipStreamCreate"));
        c->own_stream = true;
    }
    char *w = c->ws;
    DevState &st = c->st;
    st.inst = (const InstDesc *)(w + P.o_inst);
    st.adj = (const int32_t *)(w + P.o_adj);
    st.adj_off = (const int32_t *)(w + P.o_off);
    st.hfield = (const int16_t *)(w + P.o_h);
    st.ent = (const uint32_t *)(w + P.o_ent);
    st.bias = (const uint32_t *)(w + P.o_bias);
    st.csite = (const uint16_t *)(w + P.o_csite);
    st.cls_off = (const int32_t *)(w + P.o_cls);
    st.tbl = (const uint32_t *)(w + P.o_tbl);
    st.db = (const double *)(w + P.o_db);
    st.dK = (const double *)(w + P.o_dK);
    st.tiles = (const Tile *)(w + P.o_tiles);
    st.spins = (uint8_t *)(w + P.o_spins);
    st.E = (int64_t *)(w + P.o_E);
    st.C = (int64_t *)(w + P.o_C);
    st.rung_of = (int32_t *)(w + P.o_rung);
    st.label = (int32_t *)(w + P.o_label);
    st.rt = (uint64_t *)(w + P.o_rt);
    st.replica_of = (int32_t *)(w + P.o_repof);
    st.sumE = (int64_t *)(w + P.o_sumE);
    st.sumC = (int64_t *)(w + P.o_sumC);
    st.sumE2 = (int64_t *)(w + P.o_sumE2);
    st.sumC2 = (int64_t *)(w + P.o_sumC2);
    st.sumCt = (int64_t *)(w + P.o_sumCt);
    st.nup = (uint64_t *)(w + P.o_nup);
    st.ndown = (uint64_t *)(w + P.o_ndown);
    st.acc = (uint64_t *)(w + P.o_acc);
    st.att = (uint64_t *)(w + P.o_att);
    st.ctr = (Counters *)(w + P.o_ctr);
    st.rep_inst = (const int32_t *)(w + P.o_repinst);
    st.halo = (uint32_t *)(w + P.o_halo);
    st.halo_words = P.halo_words;
    st.itiles = (const int32_t *)(w + P.o_itiles);
    st.icount = (uint32_t *)(w + P.o_icount);
    st.icycle = (uint32_t *)(w + P.o_icycle);
    st.prog = (int32_t *)(w + P.o_prog);
    st.err = (uint32_t *)(w + P.o_err);
    st.bp_sblk = (const int32_t *)(w + P.o_bp_sblk);
    st.bp_eblk = (const int32_t *)(w + P.o_bp_eblk);
    st.bp_wg = (const int32_t *)(w + P.o_bp_wg);
    st.bp_part = (int64_t *)(w + P.o_bp_part);
    st.oent = (const uint16_t *)(w + P.o_oent);
    st.ohinfo = (const uint8_t *)(w + P.o_ohinfo);
    st.otbl = (const uint32_t *)(w + P.o_otbl);
    st.otiles = (const int32_t *)(w + P.o_otiles);
    st.orec = (uint32_t *)(w + P.o_orec);
    st.oprog = (int32_t *)(w + P.o_oprog);
    st.oqueue = (int32_t *)(w + P.o_oqueue);
    st.oqitems = (const int32_t *)(w + P.o_oqitems);
    st.xseen = (uint32_t *)(w + P.o_xseen);

    // one host image of the whole workspace, uploaded in a single copy
    std::vector<char> img;
    try {
        img.assign(P.total_bytes, 0);
    } catch (...) {
        return cleanup(fail(PT_ENOMEM, "host staging allocation failed"));
    }
    auto put = [&](size_t off, const void *src, size_t bytes) {
        if (bytes) std::memcpy(img.data() + off, src, bytes);
    };
    put(P.o_inst, P.desc.data(), P.desc.size() * sizeof(InstDesc));
    put(P.o_adj, P.adj.data(), P.adj.size() * 4);
    put(P.o_off, P.adj_off.data(), P.adj_off.size() * 4);
    put(P.o_h, P.hfield.data(), P.hfield.size() * 2);
    put(P.o_ent, P.ent.data(), P.ent.size() * 4);
    put(P.o_bias, P.bias.data(), P.bias.size() * 4);
    put(P.o_csite, P.csite.data(), P.csite.size() * 2);
    put(P.o_cls, P.cls_off.data(), P.cls_off.size() * 4);
    put(P.o_tbl, P.tbl.data(), P.tbl.size() * 4);
    put(P.o_db, P.db.data(), P.db.size() * 8);
    put(P.o_dK, P.dK.data(), P.dK.size() * 8);
    put(P.o_repinst, P.rep_inst.data(), P.rep_inst.size() * 4);
    put(P.o_bp_sblk, P.bp_sblk.data(), P.bp_sblk.size() * 4);
    put(P.o_bp_eblk, P.bp_eblk.data(), P.bp_eblk.size() * 4);
    put(P.o_bp_wg, P.bp_wg.data(), P.bp_wg.size() * 4);
    put(P.o_oent, P.oent.data(), P.oent.size() * 2);
    put(P.o_ohinfo, P.ohinfo.data(), P.ohinfo.size());
    put(P.o_otbl, P.otbl.data(), P.otbl.size() * 4);
    put(P.o_otiles, P.otiles.data(), P.otiles.size() * 4);
    put(P.o_oqitems, P.oqitems.data(), P.oqitems.size() * 4);
    for (int n = 0; n < n_inst; ++n) {
        const InstDesc &d = P.desc[n];
        for (int r = 0; r < d.R; ++r) {
            ((int32_t *)(img.data() + P.o_rung))[d.rep_base + r] = r;
            ((int32_t *)(img.data() + P.o_repof))[d.rep_base + r] = r;
            ((int32_t *)(img.data() + P.o_label))[d.rep_base + r] = (r == 0) ? PT_LABEL_UP : PT_LABEL_NONE;
        }
    }
    std::memcpy(img.data() + P.o_dev, &st, sizeof st);
    e = hipMemcpyAsync(c->ws, img.data(), P.total_bytes, hipMemcpyHostToDevice, c->stream);
    if (e != hipSuccess) return cleanup(hip_fail(e, "upload"));
    if (P.encoding == PT_BITPACK32) {
        e = launch_bp_init(st, P.bp_n_eblk, c->key_flip0, c->key_flip1 ^ kDomainInit, c->stream);
        if (e != hipSuccess) return cleanup(hip_fail(e, "init launch"));
    } else {
        e = launch_init_spins(st, (int)P.total_reps, c->key_flip0,
                              c->key_flip1 ^ kDomainInit, c->stream);
        if (e != hipSuccess) return cleanup(hip_fail(e, "init launch"));
    }
    e = energies_from_spins(c, 0, (int)P.total_reps);
    if (e != hipSuccess) return cleanup(hip_fail(e, "energy launch"));
    c->block_threads = opt->block_threads > 0 ? opt->block_threads : 1024;
    if (P.encoding == PT_INT8) {
        rc = build_tiles(c, opt->tile_replicas, opt->tile_bytes);
        if (rc) return cleanup(rc);
    }
    bool oct_alt = P.oct_alt;
    if (P.n_otile > 0 || P.n_oblock > 0) {
        const bool fits = P.otile_lds <= c->lds_limit && P.oblock_lds <= c->lds_limit &&
                          P.oblock_res_lds <= c->lds_limit;
        if (!fits && P.encoding == PT_BITPACK32)
            return cleanup(fail(PT_EINVAL, "octet work needs more LDS than the device has"));
        oct_alt = oct_alt && fits;
        e = fits ? oct_kernels_set_lds(P.otile_lds, P.oblock_lds, P.oblock_res_lds) : hipSuccess;
        if (e != hipSuccess) return cleanup(hip_fail(e, "octet kernel LDS attribute"));
        // octet slice blocks run resident (one launch per call) when every block fits the
        // compute units at once: blocks wait for their neighbours, which must all have started
        if (fits && P.n_oblock > 0 && !(opt->flags & PT_FLAG_BLOCK_LAUNCH_PER_SWEEP)) {
            int32_t per_cu = 0;
            e = oct_resident_per_cu(P.oblock_threads, P.oblock_res_lds, &per_cu);
            if (e != hipSuccess) return cleanup(hip_fail(e, "octet occupancy query"));
            c->oct_resident = (int64_t)P.n_oblock <= (int64_t)per_cu * c->cus;
            oct_alt = oct_alt && c->oct_resident;
        }
    }
    if (P.encoding == PT_BITPACK32) {
        // whole octets in list order (or from the device work queues)
        c->oct_queue = P.n_otile > 0 && (opt->flags & PT_FLAG_WORK_QUEUE);
        c->block_threads = opt->block_threads > 0 ? opt->block_threads : 256;
        rc = build_tiles(c, opt->tile_replicas, opt->tile_bytes);
        if (rc) return cleanup(rc);
    }
    // the exchange step in the octet (or word tile) that completes an instance, when every
    // instance is in those
    c->oct_fuse = P.n_oblock == 0 && !P.bp_generic;
    int32_t most_R = 2;
    for (const auto &d : P.desc) most_R = std::max(most_R, std::min(d.R, kObsReplicas));
    e = hipHostMalloc((void **)&c->obs_pin, (size_t)ObsLayout(most_R).bytes, hipHostMallocDefault);
    if (e != hipSuccess) {
        c->obs_pin = nullptr;
        return cleanup(fail(PT_ENOMEM, "hipHostMalloc of the read-back buffer failed"));
    }
    const bool tune_int8 = P.encoding == PT_INT8 && opt->tile_replicas == 0 &&
                           opt->tile_bytes == 0 && opt->block_threads == 0;
    // packed: the workgroup size of the whole-octet and word-tile launches
    const bool tune_bp = P.encoding == PT_BITPACK32 && (P.n_otile > 0 || c->n_words_tiles > 0) &&
                         opt->block_threads == 0;
    if (tune_int8 || tune_bp) {
        if (tune_int8) {
            for (int tb : {8 * 1024, 16 * 1024, 32 * 1024, 64 * 1024, 128 * 1024})
                for (int th : {256, 512, 1024}) c->cand.push_back({tb, th, false, 0});
        } else {
            for (int th : {256, 512, 1024}) c->cand.push_back({opt->tile_bytes, th, false, 0});
        }
        if (tune_int8 && oct_alt)
            for (int th : {512, 1024}) {
                if (P.n_otile == 0 && th < 1024) continue;  // slice blocks have a size of their own
                c->cand.push_back({0, th, true, 0});
            }
        // Few octets leave most compute units idle, and a word tile can be as small as one
        // replica: try both.  40 octets of 336 x 64 spins take 255 us a cycle as octets and
        // 109 us as 320 word tiles; with an octet for every unit the octets' shared adder
        // tree wins (7.3e9 attempts/s a unit against about 3e9).
        if (tune_bp && P.words_alt)
            for (int th : {512, 1024}) c->cand.push_back({opt->tile_bytes, th, true, 0});
        // Packed word tiles that all fit the chip at once run many cycles a launch: about one
        // large tile a unit, with a number of replicas that divides a word group (320 replicas
        // of 336 x 64 spins: 87.9 us a cycle of 10 sweeps in 160 such tiles of 2 and 101.7 in
        // 320 of 1, too many to be resident; 768 of 128 x 64: 81.8 in tiles of 4, 89.2 before).
        if (tune_bp && opt->tile_replicas == 0 && opt->tile_bytes == 0) {
            int64_t reps = 0;
            for (const auto &d : P.desc) reps += d.words && (!d.oct || P.words_alt) ? d.R : 0;
            int p = 1;
            while (p < 32 && (int64_t)p * c->cus < reps) p *= 2;
            if (p > 1 && p <= 8) c->cand.push_back({0, 1024, P.words_alt, p});
        }
        c->cand_ms.assign(c->cand.size(), 1e30);
        for (size_t k = 0; k < c->cand.size(); ++k) c->cand_order.push_back(k);
        c->tuning = true;
        for (auto &ev : c->tune_ev) {
            e = hipEventCreate(&ev);
            if (e != hipSuccess) return cleanup(hip_fail(e, "hipEventCreate"));
        }
    }
    // A launch whose tiles wait for each other may give up a wait: keep a copy of the state to
    // restore.  Tiles of several cycles a launch hold all spins in LDS, so no larger batch needs
    // one for them, and without the memory for it they run a launch per cycle.
    const bool blocks = P.halo_words > 0 || P.n_oblock > 0;
    if (blocks || (!(opt->flags & (PT_FLAG_TAU_CORR | PT_FLAG_NO_GRAPH | PT_FLAG_TIMING)) &&
                   P.state_bytes <= (size_t)c->cus * (size_t)c->lds_limit)) {
        e = hipMalloc((void **)&c->shadow_mem, std::max<size_t>(P.state_bytes, 1));
        if (e != hipSuccess) {
            c->shadow_mem = nullptr;
            (void)hipGetLastError();
            if (blocks) return cleanup(hip_fail(e, "hipMalloc (state copy)"));
        }
        c->shadow = c->shadow_mem;
        if (c->shadow && !c->tuning && !waits(c)) {
            (void)hipFree(c->shadow_mem);
            c->shadow = c->shadow_mem = nullptr;
        }
        e = take_snapshot(c);
        if (e != hipSuccess) return cleanup(hip_fail(e, "state copy"));
    }
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return cleanup(hip_fail(e, "init synchronise"));
    *out = c;
    return PT_OK;
}

int pt_sweep(pt_ctx *c, int32_t n_sweeps)
{
    if (!c) return fail(PT_EINVAL, "null context");
    if (n_sweeps < 0) return fail(PT_EINVAL, "n_sweeps < 0");
    if (n_sweeps == 0) return PT_OK;
    journal_add(c, 0, n_sweeps);
    int rc = enqueue_sweep(c, n_sweeps);
    if (rc) return rc;
    hipError_t e = launch_advance(c->st, n_inst_of(c), (uint32_t)n_sweeps, c->stream);
    if (e != hipSuccess) return hip_fail(e, "advance launch");
    return PT_OK;
}

int pt_exchange(pt_ctx *c)
{
    if (!c) return fail(PT_EINVAL, "null context");
    journal_add(c, 1, 0);
    int rc = enqueue_exchange(c, 0);
    if (rc) return rc;
    return enqueue_tau_corr(c);
}

int pt_run(pt_ctx *c, int32_t n_cycles)
{
    if (!c) return fail(PT_EINVAL, "null context");
    if (n_cycles < 0) return fail(PT_EINVAL, "n_cycles < 0");
    if (n_cycles > 0) journal_add(c, 2, n_cycles);
    // Batches whose instances each fit one whole-replica tile run up to kLaunchCycles
    // cycles per launch, each workgroup doing its instance's exchange steps itself (no
    // launch per cycle, no graph).  Not with the correlations (a launch of their own per
    // exchange), while tuning, with a launch failure to inject, or under PT_FLAG_NO_GRAPH
    // (which asks for one set of launches per cycle).
    constexpr int kLaunchCycles = 1024;
    while (n_cycles > 0 && c->tuning) {
        int m = n_cycles;
        const int rc = enqueue_cycle(c, &m);
        if (rc) return rc;
        n_cycles -= m;
    }
    if (n_cycles > 1 && c->plan.encoding == PT_INT8 &&
        !(c->opt.flags & (PT_FLAG_TAU_CORR | PT_FLAG_NO_GRAPH)) &&
        !c->inject_pending && whole_instance_tiles(c)) {
        const int k = c->opt.sweeps_per_exchange;
        while (n_cycles > 0) {
            const int m = std::min(n_cycles, kLaunchCycles);
            const int rc = enqueue_sweep_once(c, k, true, m);
            if (rc == kCycleByCycle) break;
            if (rc) return rc;
            n_cycles -= m;
        }
        if (n_cycles == 0) return PT_OK;
    }
    // Batches of more tiles that are all resident do the same, the tiles waiting for each other
    // between cycles.
    if (n_cycles > 1 && can_coop(c)) {
        // (slice blocks count the sweeps of a launch in 32 bits)
        const int most = std::min(kLaunchCycles, std::max(1, (1 << 29) / c->opt.sweeps_per_exchange));
        for (; n_cycles > 0; n_cycles -= std::min(n_cycles, most)) {
            const int rc = enqueue_coop(c, std::min(n_cycles, most));
            if (rc) return rc;
        }
        return PT_OK;
    }
    const bool eager = (c->opt.flags & (PT_FLAG_NO_GRAPH | PT_FLAG_TIMING)) != 0 ||
                       c->inject_pending;
    if (eager) {
        for (int i = 0; i < n_cycles; ++i) {
            int rc = enqueue_cycle(c);
            if (rc) return rc;
        }
        return PT_OK;
    }
    // replay a captured graph of G cycles; the remainder runs eagerly
    const int G = 16;
    int done = 0;
    if (n_cycles >= G) {
        if (!c->graph) {
            hipGraph_t g = nullptr;
            HIP_TRY(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
            int rc = PT_OK;
            for (int i = 0; i < G && rc == PT_OK; ++i) rc = enqueue_cycle(c);
            hipError_t e = hipStreamEndCapture(c->stream, &g);
            if (rc) {
                if (g) (void)hipGraphDestroy(g);
                return rc;
            }
            if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
            e = hipGraphInstantiate(&c->graph, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            if (e != hipSuccess) {
                c->graph = nullptr;
                return hip_fail(e, "hipGraphInstantiate");
            }
            c->graph_cycles = G;
        }
        for (; done + G <= n_cycles; done += G) HIP_TRY(hipGraphLaunch(c->graph, c->stream));
    }
    for (; done < n_cycles; ++done) {
        int rc = enqueue_cycle(c);
        if (rc) return rc;
    }
    return PT_OK;
}

}  // extern "C"

namespace {

// After a resident launch gave up a wait: the state of the last copy again, with resident
// launches off from here on (and the captured graph, which holds them, dropped).
int restore(pt_ctx *c)
{
    HIP_TRY(clear_err(c));
    HIP_TRY(hipMemcpyAsync(c->ws + c->plan.o_state, c->shadow, c->plan.state_bytes,
                           hipMemcpyDeviceToDevice, c->stream));
    c->resident_off = true;
    c->oct_resident = false;
    drop_graph(c);
    return PT_OK;
}

// restore, then the calls queued since the copy was taken; the result is the chain's state.
int recover(pt_ctx *c)
{
    const int restored = restore(c);
    if (restored) return restored;
    const auto calls = c->journal;
    c->replaying = true;
    int rc = PT_OK;
    for (const auto &op : calls) {
        rc = op.first == 0 ? pt_sweep(c, op.second) : op.first == 1 ? pt_exchange(c) : pt_run(c, op.second);
        if (rc) break;
    }
    if (rc == PT_OK) rc = sync_and_check(c);
    c->replaying = false;
    if (rc) return rc;
    c->recoveries += 1;
    HIP_TRY(take_snapshot(c));
    return PT_OK;
}

}  // namespace

extern "C" {

int pt_sync(pt_ctx *c)
{
    if (!c) return fail(PT_EINVAL, "null context");
    return sync_and_check(c);
}

int pt_observables(pt_ctx *c, int32_t inst, pt_obs *o)
{
    int rc = check_inst(c, inst);
    if (rc) return rc;
    if (!o) return fail(PT_EINVAL, "null output");
    const InstDesc &d = c->plan.desc[inst];
    if (d.R > kObsReplicas) return copy_observables(c, inst, o);
    const ObsLayout L(d.R);
    const char *pin = c->obs_pin;
    uint32_t err = 0;
    for (int attempt = 0;; ++attempt) {
        HIP_TRY(launch_gather_obs(c->st, L, inst, d.rep_base, d.pair_base, c->obs_pin, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
        std::memcpy(&err, pin + L.err, 4);
        if (err == 0 || attempt > 0) break;
        // the recovery (or the failure) of a plain synchronisation, then what it left
        if ((rc = check_err(c, err))) return rc;
    }
    if ((rc = check_err(c, err))) return rc;
    auto get = [&](void *dst, int32_t at, int32_t bytes) {
        if (dst) std::memcpy(dst, pin + at, (size_t)bytes);
    };
    const int R = d.R;
    get(o->E_cl, L.E, 8 * R);
    get(o->C, L.C, 8 * R);
    get(o->rung_of, L.rung, 4 * R);
    get(o->replica_of, L.repof, 4 * R);
    get(o->acc, L.acc, 8 * (R - 1));
    get(o->att, L.att, 8 * (R - 1));
    get(o->roundtrips, L.rt, 8 * R);
    get(o->sumE, L.sumE, 8 * R);
    get(o->sumC, L.sumC, 8 * R);
    get(o->sumE2, L.sumE2, 8 * R);
    get(o->sumC2, L.sumC2, 8 * R);
    get(o->nup, L.nup, 8 * R);
    get(o->ndown, L.ndown, 8 * R);
    get(o->sumCt, L.sumCt, 8 * PT_TAU_LAGS * R);
    if (o->label) {
        const int32_t *label = reinterpret_cast<const int32_t *>(pin + L.label);
        for (int r = 0; r < R; ++r) o->label[r] = (int8_t)label[r];
    }
    Counters ctr{};
    get(&ctr, L.ctr, (int32_t)sizeof ctr);
    o->t = ctr.t;
    o->e = ctr.e;
    o->n_acc = ctr.n_acc;
    return PT_OK;
}

// Device layout of one replica: bytes x = (s + 1)/2 ordered [p][i][m], slice k = 2m + p.
// Bit-packed encoding: words of an instance, and the word that holds slot r at (k, i).
static inline int64_t bp_words(const InstDesc &d)
{
    return (int64_t)d.bp_W * d.parities * d.N * d.bp_row;
}
static inline size_t bp_pos(const InstDesc &d, int r, int k, int i)
{
    const int p = (d.M >= 2) ? (k & 1) : 0;
    const int m = (d.M >= 2) ? (k >> 1) : 0;
    return (((size_t)(r / 32) * d.parities + p) * d.N + i) * d.bp_row + m;
}

static inline size_t spin_pos(const InstDesc &d, int k, int i)
{
    const int p = (d.M >= 2) ? (k & 1) : 0;
    const int m = (d.M >= 2) ? (k >> 1) : 0;
    return (size_t)p * d.N * d.Mh + (size_t)i * d.Mh + m;
}

// The device writes the spins in the caller's order into two pinned buffers by turns, and the
// host copies one out while the other fills.
int pt_get_spins(pt_ctx *c, int32_t inst, int8_t *out)
{
    int rc = check_inst(c, inst);
    if (rc) return rc;
    if (!out) return fail(PT_EINVAL, "null output");
    const InstDesc &d = c->plan.desc[inst];
    // 2 MiB a buffer: a chunk's launch and wait (about 15 us) are a few percent of the time
    // the host takes to copy it out
    constexpr int64_t kSpinChunk = 2 << 20;
    const int64_t total = (int64_t)d.R * d.M * d.N;
    const int64_t chunk = std::min(total, kSpinChunk);
    const int64_t n = (total + chunk - 1) / chunk;
    const size_t stride = align_up((size_t)chunk, 256);
    const size_t need = stride * (n > 1 ? 2 : 1);
    if (c->spin_pin_bytes < need) {
        if (c->spin_pin) (void)hipHostFree(c->spin_pin);
        c->spin_pin = nullptr;
        c->spin_pin_bytes = 0;
        HIP_TRY(hipHostMalloc((void **)&c->spin_pin, need, hipHostMallocDefault));
        c->spin_pin_bytes = need;
    }
    for (auto &ev : c->spin_ev)
        if (!ev) HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    uint32_t *err = reinterpret_cast<uint32_t *>(c->obs_pin);
    auto issue = [&](int64_t j) -> int {
        const int64_t first = j * chunk;
        HIP_TRY(launch_gather_spins(c->st, c->plan.encoding == PT_BITPACK32, inst, first,
                                    (int32_t)std::min(chunk, total - first), c->spin_pin + (j & 1) * stride,
                                    err, c->stream));
        HIP_TRY(hipEventRecord(c->spin_ev[j & 1], c->stream));
        return PT_OK;
    };
    for (int attempt = 0;; ++attempt) {
        for (int64_t j = 0; j < std::min<int64_t>(n, 2); ++j)
            if ((rc = issue(j))) return rc;
        HIP_TRY(hipEventSynchronize(c->spin_ev[0]));
        if (*err == 0 || attempt > 0) break;
        // the recovery (or the failure) of a plain synchronisation, then the state it left
        if ((rc = sync_and_check(c))) return rc;
    }
    for (int64_t j = 0; j < n; ++j) {
        if (j > 0) HIP_TRY(hipEventSynchronize(c->spin_ev[j & 1]));
        const int64_t first = j * chunk;
        std::memcpy(out + first, c->spin_pin + (j & 1) * stride, (size_t)std::min(chunk, total - first));
        if (j + 2 < n && (rc = issue(j + 2))) return rc;
    }
    return check_err(c, *err);
}

int pt_set_spins(pt_ctx *c, int32_t inst, const int8_t *in)
{
    int rc = check_inst(c, inst);
    if (rc) return rc;
    if (!in) return fail(PT_EINVAL, "null input");
    const InstDesc &d = c->plan.desc[inst];
    for (size_t x = 0; x < (size_t)d.R * d.M * d.N; ++x)
        if (in[x] != 1 && in[x] != -1) return fail(PT_EINVAL, "spins must be +1 or -1");
    // the other instances' state must be the chain's before it becomes the copy a recovery
    // restores: a launch that gave up a wait is recovered from first
    if ((rc = sync_and_check(c))) return rc;
    if (c->plan.encoding == PT_BITPACK32) {
        std::vector<uint32_t> wb((size_t)bp_words(d), 0u);
        for (int r = 0; r < d.R; ++r)
            for (int k = 0; k < d.M; ++k)
                for (int i = 0; i < d.N; ++i)
                    if (in[((size_t)r * d.M + k) * d.N + i] == 1) wb[bp_pos(d, r, k, i)] |= 1u << (r & 31);
        HIP_TRY(hipMemcpyAsync(c->ws + c->plan.o_spins + d.spin_base, wb.data(), wb.size() * 4,
                               hipMemcpyHostToDevice, c->stream));
        // pageable source: the copy has been staged once the stream reaches this point
        HIP_TRY(hipStreamSynchronize(c->stream));
    } else {
        std::vector<uint8_t> buf((size_t)d.R * d.rep_bytes, 0);
        for (int r = 0; r < d.R; ++r)
            for (int k = 0; k < d.M; ++k)
                for (int i = 0; i < d.N; ++i)
                    buf[(size_t)r * d.rep_bytes + spin_pos(d, k, i)] =
                        (uint8_t)((in[((size_t)r * d.M + k) * d.N + i] + 1) / 2);
        HIP_TRY(hipMemcpyAsync(c->ws + c->plan.o_spins + d.spin_base, buf.data(), buf.size(),
                               hipMemcpyHostToDevice, c->stream));
        HIP_TRY(hipStreamSynchronize(c->stream));
    }
    hipError_t e = energies_from_spins(c, d.rep_base, d.R);
    if (e != hipSuccess) return hip_fail(e, "energy launch");
    HIP_TRY(take_snapshot(c));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return PT_OK;
}

int pt_save(pt_ctx *c, void *buf, size_t *len)
{
    if (!c || !len) return fail(PT_EINVAL, "null argument");
    const size_t need = sizeof(CkptHeader) + c->plan.state_bytes;
    if (!buf) {
        *len = need;
        return PT_OK;
    }
    if (*len < need) return fail(PT_EINVAL, "checkpoint buffer too small");
    CkptHeader h{kMagic, kVersion, c->plan.state_bytes, c->opt.seed, n_inst_of(c),
                 c->opt.encoding, c->plan.flips_per_sweep};
    // checked (and recovered) before the copy: what is written is the chain's state
    const int rc = sync_and_check(c);
    if (rc) return rc;
    std::memcpy(buf, &h, sizeof h);
    HIP_TRY(hipMemcpyAsync((char *)buf + sizeof h, c->ws + c->plan.o_state, c->plan.state_bytes,
                           hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    *len = need;
    return PT_OK;
}

int pt_load(pt_ctx *c, const void *buf, size_t len)
{
    if (!c || !buf) return fail(PT_EINVAL, "null argument");
    const int rc = check_checkpoint(c->plan, c->opt, n_inst_of(c), buf, len);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(c->ws + c->plan.o_state, (const char *)buf + sizeof(CkptHeader),
                           c->plan.state_bytes, hipMemcpyHostToDevice, c->stream));
    // the whole state is replaced: a wait that gave up before is of no account any more
    HIP_TRY(clear_err(c));
    HIP_TRY(take_snapshot(c));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return PT_OK;
}

int pt_checkpoint_validate(const pt_instance *inst, int32_t n_inst, const pt_options *opt,
                           const void *buf, size_t len, size_t *need)
{
    if (!opt) return fail(PT_EINVAL, "null options");
    Plan P;
    int rc = make_plan(inst, n_inst, *opt, P);
    if (rc) return rc;
    if (need) *need = sizeof(CkptHeader) + P.state_bytes;
    if (!buf) return PT_OK;
    return check_checkpoint(P, *opt, n_inst, buf, len);
}

int pt_get_info(pt_ctx *c, pt_info *o)
{
    if (!c || !o) return fail(PT_EINVAL, "null argument");
    int rc = harvest_events(c);
    if (rc) return rc;
    o->n_instances = n_inst_of(c);
    o->n_tiles = c->byte_octets ? 0 : (int)c->tiles.size();
    o->block_threads = c->block_threads;
    o->lds_bytes = c->byte_octets
                       ? std::max(c->plan.otile_lds, c->oct_resident ? c->plan.oblock_res_lds : c->plan.oblock_lds)
                       : std::max({c->lds_fast, c->lds_words, c->lds_generic, c->lds_block});
    o->max_tile_replicas = c->max_P;
    o->fallbacks = c->fallbacks;
    o->encoding = c->opt.encoding;
    o->device_cus = c->cus;
    o->tile_bytes = c->tile_bytes;
    o->tuned = c->tuning ? 0 : 1;
    o->flips_per_sweep = c->plan.flips_per_sweep;
    o->sweep_ms = c->sweep_ms;
    o->sweep_launches = c->sweep_n;
    o->exchange_ms = c->exch_ms;
    o->exchange_launches = c->exch_n;
    o->sweep_groups = c->byte_octets ? 0 : (int32_t)launch_groups(c).size();
    o->block_tiles = c->byte_octets ? 0 : c->n_block_tiles;
    o->block_resident = c->byte_octets ? 0 : c->block_persistent;
    o->class_launches = 0;
    const bool octs = c->plan.encoding == PT_BITPACK32 ? !c->oct_as_words : c->byte_octets;
    o->oct_tiles = octs ? c->plan.n_otile : 0;
    o->oct_blocks = octs ? c->plan.n_oblock : 0;
    o->oct_tile_launches = o->oct_tiles > 0 ? 1 : 0;
    o->oct_resident = octs && c->oct_resident ? 1 : 0;
    o->oct_queue = c->oct_queue ? 1 : 0;
    o->oct_fused = c->oct_fuse && o->oct_tiles > 0 ? 1 : 0;
    o->oct_ring_xcd = octs && oct_ring_xcd(c) ? 1 : 0;
    o->block_ring_xcd = block_ring_xcd(c) ? 1 : 0;
    o->recoveries = c->recoveries;
    o->last_device_error = c->last_device_error;
    o->lane_words = c->lane_words;
    o->latency_path = latency_path(c, c->block_threads) ? 1 : 0;
    o->ent16_instances = 0;
    for (const auto &d : c->plan.desc) o->ent16_instances += (d.fast && d.ent_mode == kEntXad16) ? 1 : 0;
    if (c->plan.encoding == PT_BITPACK32 && c->plan.bp_generic) {
        int parities = 1;
        for (const auto &d : c->plan.desc) parities = std::max(parities, d.parities);
        o->class_launches = parities * (int32_t)c->plan.bp_colour.size();
    }
    o->multi_launches = c->multi_launches;
    o->multi_cycles = c->multi_cycles;
    o->multi_ms = c->multi_ms;
    return PT_OK;
}

int pt_timing_enable(pt_ctx *c, int32_t on)
{
    if (!c) return fail(PT_EINVAL, "null context");
    int rc = harvest_events(c);
    if (rc) return rc;
    if (on)
        c->opt.flags |= PT_FLAG_TIMING;
    else
        c->opt.flags &= ~PT_FLAG_TIMING;
    return PT_OK;
}

int pt_timing_reset(pt_ctx *c)
{
    if (!c) return fail(PT_EINVAL, "null context");
    int rc = harvest_events(c);
    if (rc) return rc;
    c->sweep_ms = c->exch_ms = c->multi_ms = 0;
    c->sweep_n = c->exch_n = 0;
    return PT_OK;
}

void pt_free(pt_ctx *c)
{
    if (!c) return;
    if (c->stream) (void)hipStreamSynchronize(c->stream);
    drop_graph(c);
    if (c->shadow_mem) (void)hipFree(c->shadow_mem);
    if (c->obs_pin) (void)hipHostFree(c->obs_pin);
    if (c->spin_pin) (void)hipHostFree(c->spin_pin);
    for (auto e : c->spin_ev)
        if (e) (void)hipEventDestroy(e);
    for (auto e : c->ev_pool) (void)hipEventDestroy(e);
    for (auto e : c->tune_ev)
        if (e) (void)hipEventDestroy(e);
    if (c->own_ws && c->ws) (void)hipFree(c->ws);
    if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
    delete c;
}

const char *pt_strerror(int code)
{
    switch (code) {
    case PT_OK: return "ok";
    case PT_EINVAL: return "invalid argument";
    case PT_ENOMEM: return "out of memory";
    case PT_EHIP: return "HIP runtime error";
    case PT_ELAUNCH: return "kernel launch failed in every configuration";
    case PT_ESTATE: return "invalid state";
    default: return "unknown error";
    }
}

const char *pt_last_error(void) { return g_last_error.c_str(); }

uint32_t pt_threshold(double dS) { return threshold(dS); }

int pt_threshold_device(const double *dS, uint32_t *out, int32_t n, void *stream)
{
    if (n < 0 || (n > 0 && (!dS || !out))) return fail(PT_EINVAL, "bad argument");
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = launch_threshold_eval(dS, out, n, s);
    if (e != hipSuccess) return hip_fail(e, "threshold launch");
    HIP_TRY(hipStreamSynchronize(s));
    return PT_OK;
}

}  // extern "C"
