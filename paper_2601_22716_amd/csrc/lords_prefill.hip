// The large-M kernel's planner and launches (the kernel: lords_prefill_kernel.h).
#include <algorithm>
#include <numeric>
#include "lords_prefill.h"

namespace lords {

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
// Contraction length of the scales padded to 32 times 1, 2 or 4; six times, of which the A tile leaves LDS for 64 tokens
// only, with fp32 factors, whose ranks 43 .. 64 come to 129 .. 192 columns.
static int pf_ss(int contraction, bool f32fact)
{
    const int rp = (contraction + 31) / 32;
    return rp <= 1 ? 1 : rp <= 2 ? 2 : rp <= 4 ? 4 : rp <= 6 && f32fact ? 6 : 0;
}

static int pf_contraction(const MatmulProblem &p) { return p.f32fact ? 3 * p.r : p.r; }   // (fp32 factors: hi/lo parts)

// (the rows of a tile's X are addressed with 32-bit byte offsets from the tile's first: these rows, 256 at most, must stay below 4 GB)
bool prefill_fast_supported(const MatmulProblem &p)
{
    return pf_ss(pf_contraction(p), p.f32fact) != 0 && !(p.f32fact && p.tiled) && (size_t)p.K * 2 * (p.M < 256 ? p.M : 256) < ((size_t)1 << 32);
}

// Tile shape and the cut of the work.  Tile shapes: 256 tokens x 256 rows (8 waves of 32 rows x 256
// tokens), 256 x 128 (8 waves), and for at most 128 tokens 128 x 256 (8 waves side by side) and
// 128 x 128 (4 waves).  Padded ranks above 32 take 128-token tiles only in this kernel (their B operands
// need the registers, their A tile the LDS): 256 rows when that still gives every CU a tile, else 128;
// bf16 factors of padded rank 64 also 256 x 256 in lords_prefill_wide.hip.
//
// The work (output tiles x K tiles) is dealt to the CUs in equal contiguous runs of units, so that
// a tile count that is no multiple of the CU count costs no half-empty last round (448 tiles of the
// headline layer at 2048 tokens on 256 CUs: 56 K tiles per CU instead of 64).  A tile cut by a run
// boundary is summed from its parts in column order (see the kernel's epilogue); the parts travel as
// fp32 through `part`, one tile-sized buffer per workgroup.  Without that buffer (callers whose
// workspace is too small for it) every workgroup takes one whole tile.
struct PfPlan {
    int ss, wm, R, wn, mb, nt, mt;
    int per, wgs;          // units per workgroup, workgroups that get any
    size_t part_bytes;     // 0: whole tiles
    int meet;              // 0, or the parts of a tile that finish it together: 2, 4 or 8
    int walk;              // of these parts, how many one workgroup takes one after the other (1: none waits in memory for the next)
    double t;              // modelled time of a K tile, us
    double cost;           // ... and of the launch
};

constexpr int kPfCUs = 256;
// The estimates for 128-token tiles at padded rank 64 read about so much high (1.15 .. 1.3 of what 30 products took), those of the
// 256 x 256 tiles that they are compared with do not.  Of 78 drawn products (129 .. 8192 tokens, 256 .. 28672 rows, 32 .. 14336
// columns) for which the planner took the latter, they took 0.84 of the former's time in the middle, up to 0.96 for nine in ten, and
// longer for four, 1.04 and 1.07 at worst, those with one and two K tiles.
constexpr double kWideScale = 1.22;

// Whether every tile may be cut into `parts` that meet (see PfLayer::meet): one workgroup per CU at most.  (Not in
// lords_prefill_wide.hip, where it made no difference: two parts of 28672 x 8192, 2 bits, rank 64, 256 tokens 140 us either way.)
static bool pf_may_meet(long tiles, int parts, int ntiles_k, int R, int mb)
{
    return R != 4 && parts <= (mb < 8 ? 4 : 8) && ntiles_k >= 2 * parts && tiles * parts <= kPfCUs;
}

// Sums of a product in fp32, of blocks of 16 x 16 with tokens in them.
static double pf_live_mb(const MatmulProblem &p) { return (double)((p.M + 15) / 16 * 16) * ((p.N + 15) / 16 * 16) * sizeof(float) / 1048576.0; }

// What it takes beside the K tiles that `parts` of each of `tiles` tiles meet: parts travel at the rate above if all CUs are at it (to
// weigh one number of parts against another: the ratio of the times of 16 products of 32 to 2048 tokens to 0.06).
static double pf_meet_us(int parts, long tiles, double live_mb, int M)
{
    return (parts == 2 ? 7.5 : parts == 4 ? 8.0 : 10.0) + (parts - 1) * live_mb / (M <= 128 ? 3.0 : 2.5) * (tiles * parts) / kPfCUs;
}

static PfPlan pf_plan(const MatmulProblem &p, size_t avail, bool wide = true, bool meet = true)
{
    PfPlan d;
    d.ss = pf_ss(pf_contraction(p), p.f32fact);
    const int ntiles_k = (p.K + 127) / 128;
    // Candidates (tokens x rows of a tile) with the measured time of one K tile of one workgroup at
    // 4 bits and rank 32, all CUs busy, clocks settled:
    //   256 x 256, eight waves of 32 rows x 256 tokens each    3.45 us   (no weight is dequantised twice in a workgroup)
    //   256 x 128, eight waves of 32 rows x 128 tokens         2.4 us
    //   128 x 256, eight waves; 128 x 128, four waves          2.15 us, 1.75 us   (up to 128 tokens)
    // Padded ranks of 64 and 128 take the last two shapes at 1.4 and 2 times the cost.  With fp32 factors, whose A tile is split
    // on the way (65536 rows x 128 tokens, one round of 256 workgroups): 128 x 256 2.6 us (contraction up to 32) and 3.1 (64),
    // where bf16 factors take 2.5 and 2.8, so they are charged the same; 128 x 128 at 128 columns 3.15, charged 3.5.
    struct Cand { int wm, R, wn, mb; double t; };
    const double rank_cost = d.ss == 1 ? 1.0 : d.ss == 2 ? 1.4 : 2.0;      // (six times 32: a shape and a time of its own)
    const Cand small_rank[4] = {{1, 2, 8, 16, 3.45}, {2, 2, 4, 8, 2.4}, {1, 2, 8, 8, 2.15}, {1, 2, 4, 8, 1.75}};
    // fp32 factors (contraction 3 r) take them at any rank: the A tile of a 256-token tile has no registers to pass through.
    // bf16 factors of padded rank 64 have 256 x 256 tiles above 128 tokens in the other form of the kernel (lords_prefill_wide.hip):
    // 3.3 .. 3.6 us a K tile, which pays where there are tiles for most of the CUs: its parts are twice as large and cost
    // 27 us to hand over when a tile has two, 38 .. 47 when four, 50 when six (2-bit 28672 x 8192 at 256 tokens, whole / two / three
    // and more parts 214 / 142 / 148 us, 128-token tiles 177; 3-bit 11008 x 4096 at 333 tokens 115 / 91 / 85 against 66).
    const Cand large_rank[3] = {{1, 2, 8, 8, 2.15 * rank_cost}, {1, 2, 4, 8, 1.75 * rank_cost}, {1, 4, 4, 16, 3.55}};
    const Cand six[1] = {{1, 2, 4, 4, 3.0}};                 // (64 x 128, four waves: 3.3 us measured)
    const Cand *cands = d.ss == 1 ? small_rank : d.ss == 6 ? six : large_rank;
    const int ncands = d.ss == 1 ? 4 : d.ss == 6 ? 1 : d.ss == 2 && !p.f32fact && p.M > 128 && wide ? 3 : 2;
    double best = 1e30;
    d.wm = 1; d.R = 2; d.wn = 4; d.mb = d.ss == 6 ? 4 : 8; d.per = ntiles_k; d.part_bytes = 0; d.meet = 0; d.walk = 1; d.t = 0.0;
    for (int i = 0; i < ncands; ++i) {
        const Cand &c = cands[i];
        const int tokens = 16 * c.mb * c.wm, rows = 16 * c.R * c.wn;
        if (p.f32fact && d.ss == 4 && rows == 256) continue;     // (eight waves: 70 registers over, spilled)
        if (d.ss != 6 && (p.f32fact ? tokens != 128 : d.ss == 1 && (tokens == 128) != (p.M <= 128))) continue;
        const long tiles = (long)((p.N + rows - 1) / rows) * ((p.M + tokens - 1) / tokens);
        const long units = tiles * ntiles_k;
        const size_t tile_bytes = (size_t)tokens * rows * sizeof(float);
        // whole tiles, dealt by the hardware in rounds
        {
            const double cost = (double)((tiles + kPfCUs - 1) / kPfCUs) * ntiles_k * c.t * (c.R == 4 ? kWideScale : 1.0);
            if (cost < best) { best = cost; d.t = c.t; d.wm = c.wm; d.R = c.R; d.wn = c.wn; d.mb = c.mb; d.per = ntiles_k; d.part_bytes = 0; d.meet = 0; }
        }
        // equal runs of units over `wgs` workgroups.  Its price is the hand-over of the parts: measured
        // 4 us + 1 us per 1.2 MB of parts written when the runs are shorter than a tile (every part is
        // written and read at about the same time), half of that per MB when they are longer; and runs
        // that are out of step with each other walk their K tiles about 8 % slower than whole tiles
        // dealt in rounds do.
        if (tiles * sizeof(uint32_t) > kZeroBytes || units > (1L << 30)) continue;
        static const int kWgs[] = {256, 224, 192, 160, 128, 112, 96, 80, 64, 48, 32, 16, 8};
        auto consider = [&](int wgs) {
            const int per = (int)((units + wgs - 1) / wgs);
            if (per < 2 || (per % ntiles_k) == 0) return;                        // (the second: whole tiles again)
            const size_t bytes = (size_t)wgs * tile_bytes;
            if (bytes > avail) return;
            // parts that start inside a tile: run boundaries but those that fall on one between tiles
            const long bounds = (units - 1) / per, written = bounds - bounds / (ntiles_k / std::gcd(per, ntiles_k));
            const double full = p.M <= 64 && tokens == 128 ? 0.5 : 1.0;          // (half a tile travels)
            const double mb_written = (double)written * tile_bytes * full / 1048576.0;
            const int others = (ntiles_k - 2 + per) / per;                       // parts that the last of a tile's waits for, at most
            const double cost = c.R == 4 ? kWideScale * (per >= ntiles_k ? per * c.t * 1.08 + 25.0 : per * c.t + 20.0 + 7.0 * (ntiles_k % per ? others : ntiles_k / per - 1))
                              : per >= ntiles_k ? per * c.t * 1.08 + 4.0 + mb_written / 2.4
                                                : per * c.t + 4.0 + mb_written / 1.2;
            if (cost < best) { best = cost; d.t = c.t; d.wm = c.wm; d.R = c.R; d.wn = c.wn; d.mb = c.mb; d.per = per; d.part_bytes = bytes; d.meet = 0; }
        };
        for (int wgs : kWgs) consider(wgs);
        // Two, four or eight parts of every tile, which their workgroups finish together: 7 us + 1 us per 3 MB, of blocks with
        // tokens in them.  More parts only where they gain a tenth: beside other matrices (batched_plans) each part is a start, a store and
        // a load more.  Two / four parts, us: 1360 tokens of 1088 x 1088 23.1 / 22.7 alone, three of them 37.8 / 59; 1024 tokens of
        // 2048 x 2048 28.5 / 26.8, with two of 512 x 2048 30.8 / 41.9; 943 tokens of 1216 x 1216 21.9 / 20.2, three 28.0 / 41.6.  (At
        // 7.5 % three of 1216 x 1216 took four parts.)  Up to 128 tokens, whose parts are small, 3 % is enough (84 tokens of 7861 x 5152, four /
        // eight parts 34.6 / 31.6; q, k and v of 4096 + 1024 + 1024 x 4096 38 with either).
        const double live_mb = pf_live_mb(p);
        double cost = 1e30;
        int most = 0;
        for (size_t room : {~(size_t)0, avail}) {              // (room for the parts chosen is all that it takes to choose them)
            if (!meet || (most && most * tiles * tile_bytes <= avail)) break;
            double fewer = cost = 1e30;
            most = 0;
            for (int parts : {2, 4, 8}) {
                if (!pf_may_meet(tiles, parts, ntiles_k, c.R, c.mb) || parts * tiles * tile_bytes > room) continue;
                const double units = (ntiles_k + parts - 1) / parts * c.t, each = units + pf_meet_us(parts, tiles, live_mb, p.M);
                cost = std::min(cost, units + 7.0 + (parts - 1) * live_mb / 3.0);
                if (each > (p.M <= 128 ? 0.97 : 0.9) * fewer) continue;
                fewer = each;
                most = parts;
            }
        }
        if (cost < best) { best = cost; d.t = c.t; d.wm = c.wm; d.R = c.R; d.wn = c.wn; d.mb = c.mb; d.per = (ntiles_k + most - 1) / most; d.part_bytes = (size_t)tiles * most * tile_bytes; d.meet = most; }
    }
    const int tokens = 16 * d.mb * d.wm, rows = 16 * d.R * d.wn;
    d.nt = (p.N + rows - 1) / rows;
    d.mt = (p.M + tokens - 1) / tokens;
    const long units = (long)d.nt * d.mt * ntiles_k;
    d.wgs = d.meet ? d.nt * d.mt * d.meet : (int)((units + d.per - 1) / d.per);
    d.cost = best;
    return d;
}

size_t prefill_fast_workspace_bytes(const MatmulProblem &p, size_t limit)
{
    return pf_plan(p, limit).part_bytes;
}

size_t prefill_least_workspace_bytes(const MatmulProblem &p)
{
    size_t least = ~(size_t)0;
    for (bool wide : {true, false})
        for (bool meet : {true, false}) least = std::min(least, pf_plan(p, ~(size_t)0, wide, meet).part_bytes);
    return least;
}

PrefillCut prefill_cut(const MatmulProblem &p, size_t limit)
{
    const PfPlan d = pf_plan(p, limit);
    return PrefillCut{16 * d.mb * d.wm, 16 * d.R * d.wn, d.meet, d.walk};
}

bool prefill_wide_taken(const MatmulProblem &p, size_t limit) { return pf_plan(p, limit).R == 4; }

double prefill_fast_cost(const MatmulProblem &p) { return pf_plan(p, ~(size_t)0).cost; }

// The launch of the matrices in a.layer, all cut into tiles of the shape of `d`.
template <bool MULTI>
static hipError_t launch_pf(const PrefillArgsT<MULTI ? kMaxBatch : 1> &a, const PfPlan &d, int bits, bool f32fact, hipStream_t st)
{
    const dim3 grid(a.layer[a.L - 1].x0 + a.layer[a.L - 1].gx);
    if (d.R == 4) return launch_prefill_wide(a, grid, bits, st);
    const PfShape shape{d.ss, d.wm, d.wn, d.mb, f32fact};
    return bits == 2 ? launch_prefill_2bit(a, shape, grid, st) : bits == 3 ? launch_prefill_3bit(a, shape, grid, st) : launch_prefill_4bit(a, shape, grid, st);
}

template <class Args>
static void pf_common(Args &a, const MatmulProblem &p, const PfPlan &d, int polls)
{
    a.X = (const uint16_t *)p.X;
    a.codebook = p.codebook;
    a.M = p.M; a.K = p.K; a.r = pf_contraction(p); a.rf = p.r;
    a.y_f32 = p.f32out ? 1 : 0;
    a.row_bytes = p.K / 8 * p.bits;
    a.mt = d.mt;
    a.ntiles_k = (p.K + 127) / 128;
    a.tiled = p.tiled ? 1 : 0;
    a.polls = polls;
}

// Workgroups of a tile in parts; 0: tiles in runs, or whole and each by the workgroup of its number.
static int share(const PfPlan &d) { return d.meet / d.walk; }

static void pf_layer(PfLayer &ly, const MatmulProblem &p, const PfPlan &d, void *part, void *arrived, int x0, int xcd)
{
    ly.codes = (const uint8_t *)p.codes;
    ly.B = p.B;
    ly.A = p.A;
    ly.Y = p.Y;
    ly.gate = nullptr;
    ly.part = (float *)part;
    ly.arrived = (uint32_t *)arrived;
    ly.N = p.N;
    ly.nt = d.nt;
    ly.per = d.meet ? (p.K + 127) / 128 : d.per;
    ly.x0 = x0;
    ly.meet = share(d) == 8 ? 3 : share(d) / 2;
    ly.walk = d.walk == 8 ? 3 : d.walk / 2;
    const int at_once = 8 * std::max(share(d), 1);
    ly.gx = (d.wgs + at_once - 1) / at_once * at_once;
    ly.xcd = xcd;
}

// `part`: part_bytes bytes of scratch (what prefill_fast_workspace_bytes returned for a limit of at most
// part_bytes), `zeroed`: kZeroBytes of device memory, zero when handed over and left at zero.
hipError_t launch_prefill_fast(const MatmulProblem &p, void *part, size_t part_bytes, void *zeroed, hipStream_t st, const float *gate, int polls)
{
    const PfPlan d = pf_plan(p, (part && zeroed) ? part_bytes : 0);
    PrefillArgsT<1> a;
    pf_common(a, p, d, polls);
    a.L = 1;
    pf_layer(a.layer[0], p, d, part, zeroed, 0, 0);
    a.layer[0].gate = gate;
    return launch_pf<false>(a, d, p.bits, p.f32fact, st);
}

// ---- several matrices, the same activations ------------------------------------------------------------------
static bool same_shape(const PfPlan &a, const PfPlan &b) { return a.R == b.R && a.wm == b.wm && a.wn == b.wn && a.mb == b.mb; }

// The matrices' workgroups in order on the XCD that has most to do, each to the CU that is free first; the launches of other tile
// shapes behind it.  A workgroup's start and end (8 us), which a planner that weighs one tile shape against another can leave out, make
// several short rounds longer than one: of 250 calls of two to six matrices, measured / estimated lies within 0.72 .. 1.05 for nine in
// ten of each padded contraction (1.05 .. 1.3 at six times 32), 0.8 .. 1.8 without them.
constexpr double kPfStartEnd = 8.0;
static double batched_cost(const PfPlan *d, int L)
{
    constexpr int kXCDs = 8;
    bool done[kMaxBatch] = {};
    double us = 0;
    for (int l0 = 0; l0 < L; ++l0) {
        if (done[l0]) continue;
        long on[kXCDs][kMaxBatch] = {};
        double each[kMaxBatch], all[kXCDs] = {};
        int xcd = 0;
        for (int l = l0; l < L; ++l) {
            if (done[l] || !same_shape(d[l], d[l0])) continue;
            done[l] = true;
            each[l] = d[l].cost / ((d[l].wgs + kPfCUs - 1) / kPfCUs) + kPfStartEnd;
            const int tiles = d[l].nt * d[l].mt, most = (d[l].wgs + kXCDs - 1) / kXCDs;
            for (int x = 0; x < kXCDs; ++x) {
                on[x][l] = share(d[l]) ? (long)share(d[l]) * (tiles / kXCDs + (((x - xcd) & 7) < tiles % kXCDs ? 1 : 0)) : std::max(0, std::min(most, d[l].wgs - x * most));
                all[x] += on[x][l] * each[l];
            }
            if (share(d[l])) xcd = (xcd + tiles) & 7;
        }
        const int x = (int)(std::max_element(all, all + kXCDs) - all);
        struct Free { double at; long cus; } free[kMaxBatch + 1] = {{0.0, kPfCUs / kXCDs}};     // in order of time
        int n = 1;
        double end = 0;
        for (int l = l0; l < L; ++l) {
            for (long left = on[x][l]; left > 0;) {
                const Free next{free[0].at + each[l], std::min(left, free[0].cus)};
                left -= next.cus;
                free[0].cus -= next.cus;
                if (free[0].cus == 0) std::copy(free + 1, free + n--, free);
                int at = n++;
                for (; at > 0 && free[at - 1].at > next.at; --at) free[at] = free[at - 1];
                free[at] = next;
                end = std::max(end, next.at);
            }
        }
        us += end;
    }
    return us;
}

// A plan of whole tiles or of tiles in parts, on tiles of another shape and with several parts to a workgroup.  The cut of K, and
// with it every sum, stays.
static PfPlan recut(const PfPlan &d, const MatmulProblem &p, const PfPlan &shape, int walk)
{
    if (d.R == 4 || shape.R == 4 || (d.meet == 0 && d.part_bytes != 0)) return d;       // (runs: cut by the tiles' numbering)
    PfPlan e = d;
    e.wm = shape.wm; e.wn = shape.wn; e.mb = shape.mb; e.t = shape.t;
    const int tokens = 16 * e.mb * e.wm, rows = 16 * e.R * e.wn, ntiles_k = (p.K + 127) / 128;
    e.nt = (p.N + rows - 1) / rows;
    e.mt = (p.M + tokens - 1) / tokens;
    const int tiles = e.nt * e.mt;
    if (d.meet == 0) {
        e.wgs = tiles;
        e.cost = (double)((tiles + kPfCUs - 1) / kPfCUs) * ntiles_k * e.t;
        return e;
    }
    e.walk = std::min(walk, e.meet);
    e.wgs = tiles * share(e);
    e.part_bytes = (size_t)tiles * e.meet * tokens * rows * sizeof(float);
    const double mb = (e.meet - 1) * pf_live_mb(p);
    e.cost = (double)((e.wgs + kPfCUs - 1) / kPfCUs) * ((ntiles_k + share(e) - 1) / share(e) * e.t + (share(e) > 1 ? 7.0 : 0.0) + 2.0 * (e.walk - 1)) + mb / 3.0;
    return e;
}

// Each matrix's cut is the one that it has alone, which fixes its sums.  How many parts of a tile one workgroup takes, and the
// tiles' shape, are chosen for the launch, by the estimate: of 12 choices timed for each of 48 sets of three matrices, those it
// prefers were within 3 % of the fastest for all but one set (7 %).
static void batched_plans(const BatchedProblem &p, PfPlan (&d)[kMaxBatch])
{
    bool cut = false, one_shape = true;
    long wgs = 0;
    for (int l = 0; l < p.L; ++l) {
        d[l] = pf_plan(matrix_of(p, l), p.whole[l] ? 0 : ~(size_t)0);
        cut |= d[l].meet != 0;
        one_shape &= same_shape(d[l], d[0]);
        wgs += d[l].wgs;
    }
    if (p.L == 1 || !cut || (one_shape && wgs <= kPfCUs)) return;
    double best = batched_cost(d, p.L);
    PfPlan alone[kMaxBatch], e[kMaxBatch];
    std::copy(d, d + p.L, alone);
    for (int j = -1; j < p.L; ++j) {                           // tiles as alone, or as the j-th matrix has them
        if (j == 0 && one_shape) break;
        bool seen = false;
        for (int i = 0; i < j; ++i) seen |= same_shape(alone[i], alone[j]);
        if (seen) continue;
        auto take = [&](int l, int walk) { return j < 0 && walk == 1 ? alone[l] : recut(alone[l], matrix_of(p, l), j < 0 ? alone[l] : alone[j], walk); };
        int most = 1;
        for (int walk = 1; walk <= most; walk *= 2) {
            for (int l = 0; l < p.L; ++l) {
                most = std::max(most, alone[l].meet);
                e[l] = take(l, walk);
            }
            double cost = batched_cost(e, p.L);
            // ... one matrix more or less
            for (int l = p.L - 1; l >= 0; --l) {
                if (e[l].walk < 2) continue;
                const PfPlan now = e[l];
                e[l] = take(l, now.walk / 2);
                const double other = batched_cost(e, p.L);
                if (other < 0.97 * cost) cost = other;
                else e[l] = now;
            }
            // (Fewer workgroups only for a gain: CUs that idle raise the clock where the call is timed alone, but not among others that load
            // the chip.  q, k, v of 2048 tokens between gate/up pairs, one workgroup a part / two parts each 139 / 155 us; alone 126 / 126.)
            if (cost < 0.97 * best) { best = cost; std::copy(e, e + p.L, d); }
        }
    }
}

size_t prefill_batched_workspace_bytes(const BatchedProblem &p)
{
    PfPlan d[kMaxBatch];
    batched_plans(p, d);
    size_t sum = 0;
    for (int l = 0; l < p.L; ++l) sum += (d[l].part_bytes + 255) & ~(size_t)255;
    return sum;
}

bool prefill_batched_supported(const BatchedProblem &p)
{
    if (p.act || p.L < 1 || p.L > kMaxBatch) return false;
    for (int l = 0; l < p.L; ++l)
        if (!prefill_fast_supported(matrix_of(p, l))) return false;
    PfPlan d[kMaxBatch];
    batched_plans(p, d);
    size_t tiles = 0;
    for (int l = 0; l < p.L; ++l) {
        if (d[l].part_bytes) tiles += (size_t)d[l].nt * d[l].mt;
        if (d[l].wgs > (1 << 24)) return false;
    }
    return tiles * sizeof(uint32_t) <= kZeroBytes;
}

PrefillCut prefill_batched_cut(const BatchedProblem &p, int l)
{
    PfPlan d[kMaxBatch];
    batched_plans(p, d);
    return PrefillCut{16 * d[l].mb * d[l].wm, 16 * d[l].R * d[l].wn, d[l].meet, d[l].walk};
}

double prefill_batched_cost(const BatchedProblem &p)
{
    PfPlan d[kMaxBatch];
    batched_plans(p, d);
    return batched_cost(d, p.L);
}

// One launch per tile shape that the matrices' plans ask for (usually one).  Not all workgroups fit the chip at once.  In runs a
// workgroup waits for first parts of later ones, which wait for nothing and are dispatched as soon as any CU of the XCD is free; one
// whose tile meets waits for a while and then leaves its share to the others (lords_meet.h).
hipError_t launch_prefill_batched(const BatchedProblem &p, void *part, void *zeroed, hipStream_t st, int polls)
{
    PfPlan d[kMaxBatch];
    unsigned char *parts[kMaxBatch];
    uint32_t *arrived[kMaxBatch];
    unsigned char *next_part = (unsigned char *)part;
    uint32_t *next_arrived = (uint32_t *)zeroed;
    bool done[kMaxBatch] = {};
    batched_plans(p, d);
    for (int l = 0; l < p.L; ++l) {
        parts[l] = next_part;
        arrived[l] = next_arrived;
        next_part += (d[l].part_bytes + 255) & ~(size_t)255;
        if (d[l].part_bytes) next_arrived += (size_t)d[l].nt * d[l].mt;      // (whole tiles count no arrivals)
    }
    for (int l0 = 0; l0 < p.L; ++l0) {
        if (done[l0]) continue;
        PrefillArgsT<kMaxBatch> a;
        pf_common(a, matrix_of(p, l0), d[l0], polls);
        a.L = 0;
        int x0 = 0, xcd = 0;
        for (int l = l0; l < p.L; ++l) {
            if (done[l] || !same_shape(d[l], d[l0])) continue;
            pf_layer(a.layer[a.L], matrix_of(p, l), d[l], parts[l], arrived[l], x0, xcd);
            x0 += a.layer[a.L].gx;
            if (share(d[l])) xcd = (xcd + d[l].nt * d[l].mt) & 7;
            ++a.L;
            done[l] = true;
        }
        const hipError_t e = launch_pf<true>(a, d[l0], p.bits, p.f32fact, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lords
