// Exact assignment (Eq. 7-8, Table 1) by equilibrium prices and shortest augmenting paths.
//
// The dual of the transportation problem has one price per expert.  At given prices every token takes its k best
// experts by q - price; the right prices are those at which every expert is chosen by exactly as many tokens as it
// has places.  They are found from both sides at once:
//
//   price passes (k_price)   every token's k-th and (k+1)-th best value give, for each expert it takes, how far that
//                            expert's price may rise before the token leaves, and for each it does not take, how far
//                            the price has to fall before the token comes.  Histograms of these margins per expert
//                            (a few bins per octave) say by how much each price has to move for its own demand to
//                            meet its capacity; all prices move at once.  Displaced tokens spread over all the other
//                            experts, so the simultaneous step converges fast: the excess demand of a batch of 65536
//                            tokens over 128 experts goes 37000, 1200, 230, 110, 55, 40 tokens.  The first two
//                            passes of 131072 tokens and more look at 8192 of them only.
//   final pass               the tokens take their k best experts at the last prices, and every exchange that would
//                            cost less than a bound is listed: arc a -> b of token u, cost (q_ua - p_a) - (q_ub - p_b),
//                            never negative because the token holds its best experts.
//   k_price_finish           one workgroup moves the few tokens that are one too many along shortest paths in the graph of
//                            experts.  Paths of different branches of the shortest-path trees are disjoint, so many are
//                            taken per search, keeping the reduced costs non-negative.  When no excess is left the
//                            assignment is feasible, the potentials certify it, and the prices are exact.
//
// The list of arcs is complete below the bound; arcs left out stay non-negative if the potentials spread less than
// the bound, which is checked at the end.  If that fails, or no path is left, up to two more tries start from the prices
// reached with more arcs.  Whenever anything does not fit (values too wide for the packed keys, too many arcs, too much
// excess left) the result is thrown away and the auction of solver.hip solves the problem instead.
//
// What bounds it: the passes read the rewards once each (34 MB for 65536 tokens over 128 experts, 11 us a pass including the
// k-th best of every row, plus 6.0 us for the step between them, which one workgroup takes), the search is one serial chain of
// searches.  65536 tokens, 128 experts, top-8, capacity 1.0: 0.17 to 0.20 ms, of which five or six passes and their steps take 0.10,
// the last pass 0.02 and the search 0.05 to 0.08; 1.6 to 1.8 ms for the auction, whose 46 rounds each read the rewards as
// well.  16384 over 64 experts: 0.10 against 0.8 to 1.3 ms.
//
// Three forms of the problem, told apart by PriceArgs::mode:
//   demand = capacity   every expert ends full;
//   spare capacity      prices stay >= 0 and an expert with room left ends at price 0.  The spare places are counted as
//                       tokens without rewards: they sit at experts of price 0, and node Z (index E) of the graph passes
//                       them from expert to expert;
//   demand > capacity   the slots a token cannot fill are held by one more column (index E) of reward 0 that a token may
//                       hold several times and that has exactly as many places as there are slots too many.
// Everything is integer arithmetic with fixed tie rules: the result does not depend on the order of execution.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "host_words.h"
#include "price_loop.h"
#include "row_keys.h"

namespace maxscore {
namespace {

constexpr int kPThreads = 256;                    // ... of the final pass
constexpr int kQThreads = 512;                    // ... of a price pass
constexpr int kPStride = kPriceMaxE + 8;          // columns of the per-expert tables (E + 1 used)
// Copies of the histograms a pass adds to, at most one per chiplet.  The workgroup that reads them all waits for their bytes, so a pass
// of few workgroups makes do with fewer (a solve of 2000 tokens of 128 experts, 32 workgroups: 234 us with eight copies, 222 with four,
// 218 with two; 16384 of 64, 256 workgroups: 144, 151, 150), and counts that cannot reach 2^16 take 16 bits each, four to an addition:
// 65536 tokens of 128 experts 271 -> 242 us, 16384 of 256 324 -> 295, 10007 of 96 267 -> 240, none slower.
constexpr int kPCopies = 8;
constexpr int kPWgPerCopy = 32;
constexpr int kPArcs = 9216;                      // arcs the one-workgroup search holds in LDS
constexpr int kPBlocks = 4096;                    // blocks of rows of the final pass at most
constexpr int kPArcBuf = 16384;                   // arcs the final pass can list
constexpr int kBlockArcs = 512;                   // ... of one block, gathered in LDS
// ... in so many lists, which the blocks take in turn: a block reserves its places with one addition, and additions to one word are 11 ns
// apart (512 blocks of 16384 tokens of 64 experts: 12.6 -> 8.6 us for the last pass; of 65536 of 128 19.9 -> 18.0).  Few blocks share one list, which then
// has room for what a few of them find.
constexpr int kPLists = 8, kPListsFrom = 128;
constexpr int kFThreads = 1024, kUThreads = 1024;
constexpr int kFirstWindow = 1 << 22;             // margins of the first pass: up to four times a score of 1
constexpr int kSampleRows = 8192;
// A sample of one row in kSampleFrom and less.  What a sample leaves is its own noise: the first pass over all rows finds nearly as many
// tokens too many as the second one behind a full first one (16384 tokens of 64 experts: 1000), so that it has to save two passes to be worth
// it.  Without and with two passes over samples before the others, solves of 16384 to 32768 tokens take 0.84 to 0.86, to 65536 0.82 to
// 0.86, to 131072 0.79 to 0.94, to 185000 1.01, to 262144 1.06, beyond 1.16 to 1.19 of the time (230 batches to 8 to 256 experts).
constexpr int kSampleFrom = 16;
// (20 exchanges per expert 1.5 % slower, 16 0.4 %, 10 and 8 0.3 and 0.9 %, 600 solves.)  From the seventh pass on, and in another try, 16: of 540 batches with
// a twentieth to half of the rows nearly alike 5 take more than 1.25 times as long as with 16 throughout and a sixth or a third of a token per expert, and
// none goes to the auction that did not then; with 12 in these too it was 25, and four such auctions (3 to 5 times as long).
constexpr int kArcsPerExpert = 12, kLateArcsPerExpert = 16, kArcsWanted = 4500, kArcsMost = 5500;
constexpr int kMaxBound = (1 << 21) - 1;
constexpr int kAllArcs = 4000;                    // problems with this few exchanges in all are searched with all of them
// The passes end when five sixths of a token per expert are too many in all (in another try a sixth), and the step is taken all the same: what
// a step leaves is the noise of where the displaced tokens went, which the prices it ends at need not be looked at for.  Of 555 drawn batches
// (64 to 65536 tokens, 8 to 256 experts) solves took 0.915 of the time of passes that end at the prices they have looked at, with a third of a
// token per expert (a sixth beyond 128) and no expert with more than two; that rule with the step 0.975, half a token 0.926, two
// thirds 0.912, one 0.918, four thirds 0.936, two 0.968.  A search with more tokens to move takes more paths at a time.
// From the seventh pass on, which only rows that are nearly alike come to, a third of a token per expert: of 256 experts their searches are long
// (six such batches of 16384 tokens 1.17 of the time of before with five sixths throughout, 0.92 so; 40 others 0.97 and 0.95).
// Beyond 256 experts a third, and with more demand than room a sixth: a search has too many tokens to move there for the exchanges that it holds.  With five
// sixths 28 of 120 such solves of 512 went into a second try or to the auction, and they took 1.10 times as long as with that earlier rule (worst 12
// times); so 0.92 with spare room, 0.93 without, and 1.00 with less room than demand (1.10 with a third there).
constexpr int kEnough = 5, kLateEnough = 2, kRetryEnough = 1, kUsualPasses = 6;       // the first three are sixths of a token per expert ...
// Up to eight places per expert a third as well: five sixths of a token are a large part of all there are.  1308 solves of two to twelve places: 0.84 of the
// time of that rule, 25 beyond 1.25 (50 tokens to 8 of 128, three places each, 173 us, 268 with five sixths), else 0.86 and 52.
constexpr int kManyEnough = 2, kManyOverEnough = 1, kManyExperts = 256, kFewPlaces = 8;      // ... and the first two here
// With spare room most experts may have no price, and what is too many is too many at the others: from 97 experts on, up to the sixth pass,
// these alone count.  10007 to 65536 tokens of 128, 160 and 256 experts, a tenth to half more room than demand: 97 to 201 us, with all experts counted 175 to 460, as the search of a few that
// far from their capacity did not stand.  Of 252 solves 0.87 of the time of the earlier rule, none beyond 1.25; with five sixths of a token for every expert 0.90,
// nine beyond.  (Four thirds, of 144 solves: 0.88; two 0.88, five sixths 0.89.)  Up to 64 experts searches stand, and all counted is
// better (0.88, 0.90 and 0.92 at 64, 32 and 16; 0.89, 0.93 and 0.94 so), at 96 too (0.90, 0.92).
constexpr int kPricedFrom = 97, kPricedEnough = 8;
// A pass that finds no more than kSoon times as many is likely to be the last but one.  (305 solves against four times: 1.005 with three, 1.008 with two
// and six, 1.034 with one, 1.036 if the end is never enqueued ahead.)
constexpr int kSoon = 4;
// Steps are shortened by an eighth when few tokens are too many: experts that chase each other's last tokens settle sooner.  Of 500 drawn
// batches (64 to 65536 tokens, 8 to 256 experts) solves took 3.6 % longer with three eighths (6 % at 64 and 128 experts, 1 % at 8 and 16); with a sixth,
// a sixteenth or none within 1 % of an eighth; within 1 % the same with a twelfth and a twentieth.
constexpr int kDamp = 8;
constexpr int kSmallEntries = 1 << 16;            // rewards of a batch that one workgroup passes over by itself
constexpr int kSmallThreads = 4096;               // ... with this many lanes at work in all
constexpr int kSmallPasses = kPriceTryPasses;
// Where demand and capacity leave no room, rows that are nearly alike need more passes than others, and what more than eight tokens per expert
// have to be moved the search does not take on.  Whether they are needed shows two passes before the last, when the host decides (later it
// would cost every batch two empty launches).  16384 rows over 64 experts, top-8, half of them alike up to 0.1: 179 us in ten passes, a tenth
// alike up to 3e-2 222 us, with a quarter less room and a quarter of them alike 190 us; in six passes the auction took over, 1.2 to 6.8 ms.
constexpr int kFar = 4, kFarPasses = 4;
constexpr int kSampledPasses = 2, kTightPasses = 6, kSlackPasses = 18, kRetryPasses = 4;
static_assert(kPriceAhead <= kRetryPasses && kPriceAhead <= kTightPasses - 2, "passes that every solve has, before any is looked at");
static_assert(kSampledPasses + kSlackPasses <= kPriceTryPasses && kSampledPasses + kTightPasses + kFarPasses <= kPriceTryPasses, "the round cap of a call allows every pass");
constexpr int kPRowsMax = 128;                    // rows of a block of the final pass at most
// Pinned words of the calling thread.  Both carry the number of the solve, as passes that were begun and given up may still tell of theirs (in the
// same place only if another solve was begun and given up between them; words so lost are looked up in the solve's own state).
constexpr int kPriceWordDone = 0, kPriceWordPasses = 1;
// Bits of the passes' word: a pass found more than kFar tokens per expert to move; the last one found so few that the next one may end the passes;
// from kPriceSeqBit on the number of the solve.
constexpr int kPriceFarBit = 16, kPriceSoonBit = 17, kPriceSeqBit = 18, kPricePassMask = (1 << kPriceFarBit) - 1;
static_assert(kPriceSeqBit + kPriceSeqBits == 32, "the number of a solve fits above them");
enum { kModeTight = 0, kModeSlack = 1, kModeOver = 2 };

struct PriceMeta {
    int w;            // margins below this were binned by the pass
    int done;         // the prices need no further pass
    int bound;        // arcs cheaper than this are listed by the final pass
    int passes;       // price passes so far (the one that checks prices the caller has given is not counted)
    int excess;       // tokens too many in all, as the pass found them (a sample's count is scaled up)
    int far;          // 1: too far from the end when the passes were nearly used up; some more follow
    int together;     // spare capacity: the step that comes next moves the experts that have a price together
    int counted;      // experts by whose number the tokens too many are judged
    int stalled;      // ... passes so far that found few tokens less than the one before them
};

// Control words and tables inside the workspace (WorkspaceLayout::price_off).
struct PriceArea {
    int prices[kPStride];
    PriceMeta meta;                               // for the pass that comes next
    int loads[8][kPStride];                       // tokens per expert after the final pass, in eight partial counts
    int fail;
    int pad[7];
    long long t_start, t_pause, t_resume;         // device clock: the first kernel; the end of passes that were begun ahead, and the first one behind them (else both 0)
    PriceReport report;
    int arrived;                                  // workgroups of the call's last kernel
    // margins and holds, PriceArgs::copies times: (2 * nb + 1) rows of ES columns, filled by a pass (workgroup b adds to copy b
    // modulo their number), added up and cleared by the update behind it.  With one copy for all the additions took 25 us
    // (of 512 workgroups then): its lines travel from chiplet to chiplet with every addition.
    alignas(16) int hist[kPCopies][kPTableInts];
    unsigned long long arc[kPArcBuf];             // cost << 32 | from << 16 | to, in PriceArgs::lists equal parts
    int arc_tok[kPArcBuf];
    int n_arcs[kPLists][32];                      // arcs of each part (a line to itself)
};

struct PriceArgs {
    const int32_t *q;
    int32_t *assign;
    PriceArea *ar;
    int *blkcnt;                                  // pairs per (block of rows of the final pass, expert)
    long long *wg_sum;                            // sum of q over the block's pairs
    int T, E, k, C, mode;
    int rows, n_wg;                               // of the final pass
    int ib, nb, bshift;                           // bits of a column id in a packed key; bins per side; their width
    int es, quads;                                // columns of the histograms; 16-byte pieces of 32-bit counts of a copy
    int copies;                                   // ... their copies, a power of two ...
    int half;                                     // ... with counts of 16 bits (no copy's can reach 2^16), else of 32
    int retry;                                    // the search has failed at the prices or the bound before
    int arcs_wanted, arcs_late;                   // about so many exchanges are to lie under the bound; from the kUsualPasses-th pass on
    int lists;                                    // of arcs: one or kPLists
    int sampled;                                  // passes over a sample before the others
    int *host;                                    // pinned words
    int seq;                                      // number of the solve, not zero
    int look;                                     // the pass that tells whether more than the usual ones are needed, or -1
    int pause;                                    // the last pass that is begun ahead, or -1
    int resumes;                                  // the first launch behind these
};

// So many sixths of a token per expert too many end the passes at pass t.
__device__ __forceinline__ int enough_sixths(const PriceArgs &a, int t)
{
    if (a.retry) return kRetryEnough;
    if (a.E > kManyExperts) return a.mode == kModeOver ? kManyOverEnough : kManyEnough;
    if (a.C <= kFewPlaces) return kManyEnough;
    return t - a.sampled >= kUsualPasses ? kLateEnough : a.mode == kModeSlack && a.E >= kPricedFrom ? kPricedEnough : kEnough;
}

// Margins are binned relative to w0 = window / 2^9: linear up to w0, then two bins per octave (one beyond 256 experts).
__device__ __forceinline__ int bin_of(int m, int w0, int bshift)
{
    return (int)((__float_as_uint((float)(m + w0)) - __float_as_uint((float)w0)) >> bshift);
}
__device__ __forceinline__ int bin_edge(int b, int w0, int bshift)        // lowest margin of bin b
{
    const float f = __uint_as_float(__float_as_uint((float)w0) + ((unsigned)b << bshift));
    return (int)ceilf(f) - w0;
}
__device__ __forceinline__ int bin_w0(int w) { return (w >> 9) > 2 ? (w >> 9) : 2; }

__device__ __forceinline__ int wave_sum(int v)        // inclusive prefix sum over the lanes, the total in lane 63
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);    // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

__device__ __forceinline__ int wave_max(int v)        // over the lanes, uniform
{
    constexpr int low = -0x7fffffff - 1;
    int o;
    o = __builtin_amdgcn_update_dpp(low, v, 0x111, 0xf, 0xf, false); v = o > v ? o : v;
    o = __builtin_amdgcn_update_dpp(low, v, 0x112, 0xf, 0xf, false); v = o > v ? o : v;
    o = __builtin_amdgcn_update_dpp(low, v, 0x114, 0xf, 0xf, false); v = o > v ? o : v;
    o = __builtin_amdgcn_update_dpp(low, v, 0x118, 0xf, 0xf, false); v = o > v ? o : v;
    o = __builtin_amdgcn_update_dpp(low, v, 0x142, 0xa, 0xf, false); v = o > v ? o : v;
    o = __builtin_amdgcn_update_dpp(low, v, 0x143, 0xc, 0xf, false); v = o > v ? o : v;
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ unsigned row_mask(int row, int ib)      // equal values are ranked by column XOR a mask of the row
{
    return ((unsigned)row * 0x9E3779B1u) >> (32 - ib);
}

// New prices from the histograms of a pass: of s.was to s.now, with the margins in s_h; one workgroup.
//
// Demand = capacity: every expert's price is moved to where its own demand meets the capacity.  Demand > capacity: towards the mean demand
// one by one, and all together by the step that brings the mean to the capacity, whose margins are in column E of the histograms.
//
// Spare capacity: an expert's demand is taken to depend on how far its price moves beyond the level, the common move of the prices a token
// compares it with.  Its own margins say at which distance from the level it ends full; prices stay >= 0, and an expert that would have to
// fall below that ends with room, and with the tokens that its newcomers' margins (or those of its holds) give it at that distance.  The
// level is the one at which all demands add up to the tokens there are.  Moved one by one, the experts with too many tokens pushed them
// onto others that were as good as full, and so on: 10007 tokens of 96 experts and a tenth of spare capacity took nine passes (excess
// 25000, 14000, 8300, 4100, 1500, 350, 80, 35, 20), now six or seven (25000, 1200, 160, 65, 35, 20), each without the search for the exchanges
// of a common step (7.9 -> 6.0 us).  Solves of 250 batches with 2 to 100 % of spare capacity take 0.88 of the time (0.83 at 64 to 128
// experts, 0.92 to 0.95 at 16 and 32, 1.05 at 8).
//
// Rows that are nearly alike all move on to the same next expert, which no expert's own margins show: a step at the level reaches one expert
// further where many are needed.  Where the excess has not halved, the level's rises go twice as far and its falls half, and the next step is
// one of the other kind: the experts with a price move towards their mean demand one by one, and up together by what they have too many in all
// (of each row the margin of the lowest hold that has a price to the best alternative that has none), the others as far as their own margins
// say.  Neither kind gets there by itself.  Solves of 40 batches of 4096 to 65536 tokens to 16 to 256 experts, a twentieth to half of them
// alike up to 0.1 or 3e-2 and 2 to 50 % more room than demand, against these steps alone (most then go on to the auction): 0.52 with the
// level's alone, 0.39 in turn; a tenth of 16384 rows over 256 experts alike 1.83 and 0.80; a quarter of 32768 rows over 64 experts alike up
// to 3e-2, a quarter more room, 0.21 to 0.25 ms in 10 or 11 passes, 0.25 to 0.39 in 10 to 18, and 0.18 to 0.26 in 10 to 14.  Other
// batches hardly ever come to it: 50 solves within 1 %.
//
// Bound by latency, and by what the sixteen wavefronts do alike (four of them share a SIMD): sums are taken over the
// wavefronts that have experts only, and the bound of the arc list is worked out by the last one beside the columns.  The largest
// step is reduced by lane moves: an atomic maximum of all lanes on one word is compiled into a loop over the lanes (1.5 us).
struct StepLds {
    __attribute__((aligned(16))) int was[kPStride], now[kPStride];
    int cum[64];
    __attribute__((aligned(16))) int part[kPriceMaxE / 64][8];      // sums of the wavefronts that have experts
    float level[2][kUThreads / 64];                                 // demand beyond the tokens there are, at so many levels
    int maxd, ran_out, lam, bound, wide, reach;
};

__device__ __forceinline__ void step_clear(StepLds &s)
{
    if (threadIdx.x < 64) s.cum[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s.maxd = s.ran_out = s.lam = 0;
    }
}

__device__ __forceinline__ float wave_sum_f(float v)        // the total in lane 63
{
    auto add = [](float x, int y) { return x + __int_as_float(y); };
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xf, 0xf, true));
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xf, 0xf, true));
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xf, 0xf, true));
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));
    v = add(v, __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));
    return v;
}

// Behind step_clear and a barrier.  CUM: s.cum holds the sums of the bins already.  SPARE: there is spare capacity; the columns of s_h are
// summed up then.  TOGETHER: the step of the other kind.  (Three kinds of code, as the branches of the others cost every step: 0.4 to 0.5 us at
// 16, 64 and 128 experts those of spare capacity, and with that at 96 0.4 those of the other kind.)
template <bool CUM, bool SPARE, bool TOGETHER>
__device__ __forceinline__ PriceMeta price_step(const PriceArgs &a, int t, int nrows, const PriceMeta mt, int *s_h, StepLds &s)
{
    constexpr int NW = kUThreads / 64;
    static_assert(kPriceMaxE / 64 < NW - 2, "the last two wavefronts have no experts");
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int E = a.E, ES = a.es, nb = a.nb, nwe = (E + 63) >> 6;
    constexpr bool spare = SPARE, together = SPARE && TOGETHER, slack = SPARE && !TOGETHER;
    const bool over_all = !SPARE && a.mode == kModeOver;
    const bool sampled = nrows < a.T;
    const int w0 = bin_w0(mt.w), bs = a.bshift;
    const int Ct = sampled ? (int)(((long long)a.C * nrows + a.T / 2) / a.T) : a.C;
    const int *s_hn = s_h + 2 * nb * ES;
    const bool priced = spare && E >= kPricedFrom && !a.retry && t - a.sampled < kUsualPasses;
    if (wv < nwe) {
        const int ne = tid < E ? s_hn[tid] : 0, over = tid < E && ne > Ct ? ne - Ct : 0;
        const bool in = tid < E && (!spare || s.was[tid] > 0);
        const int sn = wave_sum(in ? ne : 0), sx = wave_sum(over), sd = wave_sum(in && ne < Ct ? Ct - ne : 0);
        const int sc = priced ? wave_sum(tid < E && (s.was[tid] > 0 || ne >= Ct) ? 1 : 0) : 0;
        if (lane == 63) *(int4 *)&s.part[wv][0] = make_int4(sn, sx, sd, sc);
        if (together) {
            const int ss = wave_sum(in ? 1 : 0), sz = wave_sum(in ? 0 : over);
            if (lane == 63) *(int2 *)&s.part[wv][4] = make_int2(ss, sz);
        }
    }
    // holds (0 .. nb-1) and newcomers (nb .. 2nb-1) per margin bin over all experts
    if constexpr (!CUM) {
        constexpr int NB = (2 * kPBins + NW - 1) / NW;
        int tot[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) tot[i] = 0;
        for (int e = lane; e < E; e += 64)
#pragma unroll
            for (int i = 0; i < NB; ++i) tot[i] += s_h[(wv + i * NW < 2 * nb ? wv + i * NW : 0) * ES + e];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            tot[i] = wave_sum(tot[i]);
            if (lane == 63 && wv + i * NW < 2 * nb) s.cum[wv + i * NW] = tot[i];
        }
    }
    __syncthreads();
    int sn = 0, sx = 0, sd = 0, sc = 0, ss = 0, sz = 0;      // sc: experts that have a price or are full; ss: whose price counts; sz: tokens too many at the others
    for (int x = 0; x < nwe; ++x) {
        const int4 p4 = *(const int4 *)&s.part[x][0];
        sn += p4.x;
        sx += p4.y;
        sd += p4.z;
        sc += p4.w;
        if (together) {
            const int2 p2 = *(const int2 *)&s.part[x][4];
            ss += p2.x;
            sz += p2.y;
        }
    }
    if (!together) ss = E;
    sx = sd > sx ? sd : sx;                                           // tokens too many or too few
    // enough: what is left is cheaper to move by the search
    const int excess = sampled ? (int)((long long)sx * a.T / nrows) : sx;
    const int counted = priced ? sc : E;
    const bool enough = !sampled && 6 * excess <= counted * enough_sixths(a, t);
    const bool moves = excess > 0 || sampled || a.retry;               // (another try may have to go on all the same)
    // the capacity, or the mean demand (of the experts together no less than the capacity: one of them that has room is at its own mean)
    int target = slack || ss == 0 ? Ct : (2 * sn + ss) / (2 * ss);
    if (together && target < Ct) target = Ct;
    if (moves && wv * 64 < E + (over_all ? 1 : 0)) {
        const int j = tid;
        const bool common = j == E;
        const int pj = j <= E ? s.was[j] : 0;
        const bool alone = together && pj == 0;              // (has no price: room is left there)
        int diff = 0;
        if (j < E + (over_all ? 1 : 0)) diff = common ? sn - Ct * E : s_hn[j] - (alone ? Ct : target);
        if (alone && diff < 0) diff = 0;
        const int side = diff < 0 ? 1 : 0, need = side ? -diff : diff;      // side 0: the price has to rise, side 1: to fall
        int most = 0;
        if (need != 0 || (slack && j < E)) {
            int prev = 0, b = 0, in_b = 0;                       // the first bin that reaches `need`, its count and the one before it
            for (int way = slack ? 0 : side; way <= (slack ? 1 : side); ++way) {
                int *col = s_h + way * nb * ES + j;
                int c[kPBins];                                   // (one branch for all: nb is kPBins or half of it)
#pragma unroll
                for (int x = 0; x < kPBins / 2; ++x) c[x] = col[x * ES];
#pragma unroll
                for (int x = kPBins / 2; x < kPBins; ++x) c[x] = 0;
                if (nb > kPBins / 2) {
#pragma unroll
                    for (int x = kPBins / 2; x < kPBins; ++x) c[x] = col[x * ES];
                }
#pragma unroll
                for (int x = 1; x < kPBins; ++x) c[x] += c[x - 1];
                if (way == side) {
#pragma unroll
                    for (int x = 0; x < kPBins; ++x) {
                        const bool less = c[x] < need;
                        b += less ? 1 : 0;
                        prev = less ? c[x] : prev;
                    }
                    if (b < nb) in_b = col[b * ES];
                }
                if (slack) {
#pragma unroll
                    for (int x = 0; x < kPBins / 2; ++x) col[x * ES] = c[x];
                    if (nb > kPBins / 2) {
#pragma unroll
                        for (int x = kPBins / 2; x < kPBins; ++x) col[x * ES] = c[x];
                    }
                }
            }
            b = b < nb ? b : nb;
            int d = mt.w;
            if (b < nb) {
                const int lo = bin_edge(b, w0, bs), hi = bin_edge(b + 1, w0, bs);
                d = lo + (int)((float)(hi - lo) * (float)(need - prev) * __builtin_amdgcn_rcpf((float)in_b) + 0.5f);
                d = d < lo ? lo : d > hi ? hi : d;
            }
            if (b == nb && (!slack || !side || pj > 0)) s.ran_out = 1;
            d = need == 0 ? 0 : d < 1 ? 1 : d;
            most = d;
            if (slack) s.now[j] = side ? -d : d;                 // distance from the level at which the expert ends full
            else if (common) s.lam = side ? -d : d;
            else s.now[j] = pj + (side ? -d : d);
        }
        if (!slack) {
            most = wave_max(most);           // (an atomic of every lane is compiled into a loop over the lanes)
            if (lane == 0 && most > 0) atomicMax(&s.maxd, most);
        }
    } else if (together && moves && wv == NW - 2) {
        // up together, by what those that have a price and those that are about to get one have too many
        const int need = sn - Ct * ss, x = lane < nb ? s_h[(2 * nb + 1) * ES + lane] : 0, cum = wave_sum(x);
        if (need > 0) {
            const unsigned long long far = __ballot(lane < nb && cum >= need + sz);
            int d = mt.w;
            if (far) {
                const int b = __ffsll((long long)far) - 1, lo = bin_edge(b, w0, bs), hi = bin_edge(b + 1, w0, bs);
                const int in_b = __builtin_amdgcn_readlane(x, b), before = __builtin_amdgcn_readlane(cum, b) - in_b;
                d = lo + (int)((float)(hi - lo) * (float)(need + sz - before) * __builtin_amdgcn_rcpf((float)in_b) + 0.5f);
                d = d < lo ? lo : d > hi ? hi : d;
            }
            if (lane == 0) {
                if (!far) s.ran_out = 1;
                s.lam = d < 1 ? 1 : d;
                atomicMax(&s.maxd, s.lam);
            }
        }
    } else if (wv == NW - 1) {
        // the bound of the arc list: about kArcsPerExpert exchanges per expert lie under it.  h holds and n newcomers make
        // h * n / rows of them if they are spread over all rows, and the larger of the two if every row has one of each.
        const float want = (float)(t - a.sampled < kUsualPasses ? a.arcs_wanted : a.arcs_late) * (float)nrows / (float)a.T;
        const float ch = (float)wave_sum(lane < nb ? s.cum[lane] : 0), cn = (float)wave_sum(lane < nb ? s.cum[nb + lane] : 0);
        const float cmin = fminf(fminf(ch, cn), (float)nrows), cum = cmin > 0.f ? ch * cn / cmin : 0.f;
        const unsigned long long fb = __ballot(lane < nb && cum >= want), fw = __ballot(lane < nb && cum >= 1.5f * want);
        int bound = mt.w;
        if (fb) {
            const int b = __ffsll((long long)fb) - 1, lo = bin_edge(b, w0, bs), hi = bin_edge(b + 1, w0, bs);
            const float c1 = __shfl(cum, b), c0 = b > 0 ? __shfl(cum, b - 1) : 0.f;
            bound = lo + (int)((float)(hi - lo) * (want - c0) / (c1 - c0));
        }
        if (lane == 0) {
            s.bound = bound;
            s.wide = fw ? bin_edge(__ffsll((long long)fw), w0, bs) : 4 * mt.w;
            s.reach = fb != 0;
        }
    }
    __syncthreads();
    float level = 0.f;
    if (slack && moves) {
        // sixteen levels at a time, one to a wavefront, the first ones closer to each other the closer to none: by how much the demands
        // add up to more than they do now
        float lo = -(float)mt.w, hi = (float)mt.w, flo = 0.f, fhi = 0.f;
        bool above = false, below = false;                       // flo, fhi are known
        for (int turn = 0; turn < 2; ++turn) {
            const float from = lo, span = hi - lo;
            auto level_of = [&](int x) {                         // of 0 .. NW + 1
                const float u = (float)x * (1.f / (NW + 1)), c = 2.f * u - 1.f;
                return turn == 0 ? (float)mt.w * c * c * c : from + span * u;
            };
            const float at = level_of(wv + 1);
            float f = 0.f;
            for (int e = lane; e < E; e += 64) {
                const float p = (float)s.was[e], own = (float)s.now[e];
                float n = (float)(Ct - s_hn[e]);                 // full
                if (at + own <= -p) {                            // at price 0: as far from the level as that leaves it
                    const float x = -p - at, m = fabsf(x);
                    const int *col = s_h + (x > 0.f ? 0 : nb) * ES + e;
                    const int mi = m < (float)mt.w ? (int)m : mt.w, b = bin_of(mi, w0, bs);
                    if (b >= nb) n = (float)col[(nb - 1) * ES];
                    else {
                        const float c0 = b > 0 ? (float)col[(b - 1) * ES] : 0.f, c1 = (float)col[b * ES];
                        const float e0 = (float)bin_edge(b, w0, bs), e1 = (float)bin_edge(b + 1, w0, bs);
                        n = c0 + (c1 - c0) * fmaxf(m - e0, 0.f) * __builtin_amdgcn_rcpf(e1 - e0);
                    }
                    n = x > 0.f ? -n : n;
                }
                f += n;
            }
            f = wave_sum_f(f);
            if (lane == 63) s.level[turn & 1][wv] = f;
            __syncthreads();
            const float y = s.level[turn & 1][lane & (NW - 1)];
            const unsigned many = (unsigned)__ballot(lane < NW && y >= 0.f);
            const int x = many ? __ffs((int)many) - 1 : NW;          // the first level with too many
            if (x < NW) {
                hi = level_of(x + 1);
                fhi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), x));
                below = true;
            }
            if (x > 0) {
                lo = level_of(x);
                flo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(y), x - 1));
                above = true;
            }
        }
        level = above && below ? lo + (hi - lo) * (flo < fhi ? -flo / (fhi - flo) : 0.5f) : below ? hi : lo;
        if (wv < nwe) {
            int dp = 0;
            if (tid < E) {
                const float x = level + (float)s.now[tid], p = (float)s.was[tid];
                dp = x <= -p ? -s.was[tid] : (int)rintf(x);
                s.now[tid] = s.was[tid] + dp;
            }
            const int most = wave_max(dp < 0 ? -dp : dp);
            if (lane == 0 && most > 0) atomicMax(&s.maxd, most);
        }
        __syncthreads();
    }
    PriceMeta m2 = mt;
    const int bound = s.bound;
    m2.bound = (long long)a.T * a.k * (E - a.k) <= kAllArcs ? kMaxBound : bound < 2 ? 2 : (bound > kMaxBound ? kMaxBound : bound);
    int w = s.maxd > s.wide ? s.maxd : s.wide;
    if (s.ran_out && w < 4 * mt.w) w = 4 * mt.w;
    m2.w = w < 16 ? 16 : (w < (1 << 26) ? w : (1 << 26));
    ++m2.passes;
    m2.excess = excess;
    m2.counted = counted;
    const bool listed = !a.retry || s.reach;             // another try needs more exchanges than the one before
    // stuck: it no longer shrinks (it ends up alternating by a few); with spare capacity the step of the other kind is to be tried first, unless
    // there are few left (16384 tokens, a tenth of them alike, to 8 of 256: a search of 137 tokens took longer than the passes it saved)
    const bool stalls = m2.excess <= E && m2.excess * 5 >= mt.excess * 4 && t >= 4;
    const bool stuck = stalls && (!spare || 4 * m2.excess <= E || (mt.stalled >= 1 && 2 * m2.excess <= E) || mt.stalled >= 4);
    m2.stalled += stalls ? 1 : 0;
    if (!sampled && (s.maxd == 0 || (listed && (enough || stuck)))) {
        m2.done = 1;
        m2.w = mt.w;
        if (m2.excess == 0) m2.bound = 2;                // nothing to move
    }
    if (m2.done && (!enough || m2.excess == 0 || s.maxd == 0)) {
        for (int e = tid; e < E; e += kUThreads) s.now[e] = s.was[e];
    } else {
        // (the first pass over all rows finds what the samples have left: nothing slow about that)
        const bool damp = !sampled && m2.excess <= E, slow = spare && t > a.sampled && 2ll * m2.excess > mt.excess;
        const int plim = (1 << (31 - a.ib)) - 1;
        for (int e = tid; e < E; e += kUThreads) {
            int dp = s.now[e] - s.was[e];
            dp = damp ? dp - dp / kDamp : !(slow && slack) ? dp : dp <= 0 ? dp / 2 : dp < (1 << 28) ? 2 * dp : dp;      // (a price has 31 bits)
            int pn = s.was[e] + dp + (over_all || (together && s.was[e] > 0) ? s.lam : 0);
            if (spare) pn = pn < 0 ? 0 : pn;
            s.now[e] = pn > plim ? plim : (pn < -plim ? -plim : pn);
        }
        if (slow && !m2.done) m2.together = !mt.together;
    }
    return m2;
}

// The sum of N copies of the histograms, which are cleared: up to M 16-byte pieces per thread, all on their way together.
template <int N, int M, bool HALF>
__device__ __forceinline__ void gather_copies(const PriceArgs &a, int *s_h, StepLds &s)
{
    constexpr int Q = HALF ? 2 : 1;                                   // quads of counts in a piece
    const int quads = a.quads, pieces = (quads + Q - 1) / Q;
    const float inv = __builtin_amdgcn_rcpf((float)(a.es / 4));       // (u + 1/2 quads are 1/2 from a row's edge: 1e-7 of 3000 is less)
    uint4 x[M][N];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = m * kUThreads + threadIdx.x;
#pragma unroll
        for (int r = 0; r < N; ++r) x[m][r] = i < pieces ? ((const uint4 *)a.ar->hist[r])[i] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int i = m * kUThreads + threadIdx.x;
        int4 y[Q];
#pragma unroll
        for (int h = 0; h < Q; ++h) y[h] = make_int4(0, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint4 z = x[m][r];
            if ((z.x | z.y | z.z | z.w) != 0) ((uint4 *)a.ar->hist[r])[i] = make_uint4(0, 0, 0, 0);
            if constexpr (HALF) {
                y[0].x += z.x & 0xffff; y[0].y += z.x >> 16; y[0].z += z.y & 0xffff; y[0].w += z.y >> 16;
                y[1].x += z.z & 0xffff; y[1].y += z.z >> 16; y[1].z += z.w & 0xffff; y[1].w += z.w >> 16;
            } else {
                y[0].x += z.x; y[0].y += z.y; y[0].z += z.z; y[0].w += z.w;
            }
        }
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            const int u = i * Q + h;
            if (u >= quads) continue;
            ((int4 *)s_h)[u] = y[h];
            // the sums of the bins on the way (the columns beyond the experts do not belong to them)
            const int row = (int)(((float)u + 0.5f) * inv), c = 4 * (u - row * (a.es / 4));
            const int sum = (c < a.E ? y[h].x : 0) + (c + 1 < a.E ? y[h].y : 0) + (c + 2 < a.E ? y[h].z : 0) + (c + 3 < a.E ? y[h].w : 0);
            if (row < 2 * a.nb && sum) atomicAdd(&s.cum[row], sum);
        }
    }
}
static_assert(kPTableInts % 4 == 0, "every copy starts on 16 bytes");
static_assert(2 * kPBins + 1 <= 64, "a sum per bin");
constexpr int price_pieces(bool half) { return (kPTableInts / (half ? 8 : 4) + kUThreads) / kUThreads; }      // per thread, at most

// One workgroup.  Half of it is the wait for the copies, which the pass's additions have left in memory; the rest two barriers' worth of
// sums and searches: 3.8 us at 16 experts, 5.0 at 64, 6.0 at 128, 8.0 at 256 (1.3 to 3.4 more with counts of 32 bits, and with the
// sums of the bins and the largest step taken behind the copies); with spare capacity 8.0 at 96, and 4.6 where the passes
// end.  As the first step of every workgroup of the next pass the same work took 10 to 20 us.
template <int N, int M, bool HALF, bool SPARE>
__global__ __launch_bounds__(kUThreads) void k_price_update(PriceArgs a, int t, int nrows)
{
    extern __shared__ __attribute__((aligned(16))) int s_h[];         // the sum of the copies
    __shared__ StepLds s;
    PriceArea *ar = a.ar;
    const int tid = threadIdx.x, E = a.E;
    // everything is requested before the state is looked at (the exit test then does not add a round trip)
    for (int e = tid; e < kPStride; e += kUThreads) s.was[e] = s.now[e] = e < E ? ar->prices[e] : 0;
    step_clear(s);
    __syncthreads();
    gather_copies<N, M, HALF>(a, s_h, s);
    const PriceMeta mt = ar->meta;
    if (mt.done) return;                 // (passes that find the prices done add nothing: the copies stay clear)
    __syncthreads();
    PriceMeta m2;
    if (SPARE && __builtin_expect(mt.together, 0)) m2 = price_step<true, SPARE, true>(a, t, nrows, mt, s_h, s);
    else m2 = price_step<true, SPARE, false>(a, t, nrows, mt, s_h, s);
    if (t == a.look) m2.far = m2.excess > kFar * E;
    for (int e = tid; e < E; e += kUThreads) ar->prices[e] = s.now[e];
    if (tid == 0) {
        ar->meta = m2;
        if (a.pause >= 0 && (t == a.pause || m2.done)) ar->t_pause = wall_clock64();
    }
}

// What the host is to know of the passes before pass t: the next launch tells it when it begins, as the step would have to wait a microsecond
// for the word to get there before it ends.
__device__ __forceinline__ void price_tell(const PriceArgs &a, const PriceMeta &mt, int t)
{
    if (mt.done) tell_host(a.host + kPriceWordDone, a.seq);
    else if (t > 0) {
        const bool soon = t > a.sampled && 6 * mt.excess <= kSoon * mt.counted * enough_sixths(a, t);
        tell_host(a.host + kPriceWordPasses, (int)((unsigned)t | (unsigned)mt.far << kPriceFarBit | (soon ? 1u : 0u) << kPriceSoonBit | (unsigned)a.seq << kPriceSeqBit));
    }
}

// The margins of rows r_first .. r_end - 1 of a pass (row i is token i * stride + shift), added to the histograms in
// s_hist; NT threads, G of them to a row.  nx holds this lane's part of its first row.
template <int G, int EPL, bool OS, bool TOGETHER, int NT>
__device__ __forceinline__ void price_rows(const PriceArgs &a, int W, int r_first, int r_end, int stride, int shift, int (&nx)[EPL],
                                           const int *s_p, int *s_hist)
{
    using RK = RowKeys<G, EPL>;
    constexpr int NG = NT / G;
    const int tid = threadIdx.x, E = a.E, k = a.k, ib = a.ib, nb = a.nb, ES = a.es, bs = a.bshift;
    const int lg = tid & (G - 1), grp = tid / G;
    const bool vec = (E & 3) == 0 && (((size_t)a.q) & 15) == 0;
    const int w0 = bin_w0(W);
    const int bias = 1 << (31 - ib);
    const unsigned cmask = (1u << ib) - 1;
    int pb[EPL];                                          // bias - price of this lane's columns
    unsigned priced = 0;                                  // TOGETHER: those with a price, and those beyond the experts
#pragma unroll
    for (int m = 0; m < EPL; ++m) {
        const int c = RK::col(m, lg);
        pb[m] = c < E ? bias - s_p[c] : 0;
        if (TOGETHER && pb[m] < bias) priced |= 1u << m;
    }
    const unsigned keyo = (unsigned)bias << ib;           // an unfilled slot: reward 0, price 0
    int *s_n = s_hist + 2 * nb * ES;
    for (int i0 = r_first + grp; i0 - grp < r_end; i0 += NG) {
        const bool live = i0 < r_end;
        const int row = (live ? i0 : r_end - 1) * stride + shift;
        int v[EPL];
#pragma unroll
        for (int m = 0; m < EPL; ++m) v[m] = nx[m];
        if (i0 - grp + NG < r_end) {
            int i = i0 + NG;
            i = i < r_end ? i : r_end - 1;
            RK::load(a.q + (size_t)(i * stride + shift) * E, E, vec, lg, nx);
        }
        const unsigned rot = row_mask(row, ib);
        unsigned key[EPL];
#pragma unroll
        for (int m = 0; m < EPL; ++m) {
            const int c = RK::col(m, lg);
            key[m] = c < E ? (((unsigned)(v[m] + pb[m])) << ib) | ((unsigned)c ^ rot) : 0u;
        }
        unsigned kth = RK::first(key), mine = kth;        // mine: the (lg + 1)-th best key
        for (int r = 1; r < k; ++r) {
            kth = RK::below(key, kth);
            mine = lg == r ? kth : mine;
        }
        const unsigned nxt = RK::below(key, kth);
        const bool slot = lg < k && live;
        // held: key >= thr; alt: the best a hold competes with; low: what a newcomer displaces
        unsigned thr = kth, alt = nxt, low = kth;
        bool near = (int)((kth - nxt) >> ib) < W;
        if (OS) {
            thr = kth > keyo ? kth : keyo + 1;
            low = kth > keyo ? kth : keyo;
            alt = nxt > keyo ? nxt : keyo;
            near = true;
        }
        const int mc = (int)((mine & cmask) ^ rot);
        if (slot && mine >= thr && mc < E) atomicAdd(&s_n[mc], 1);
        if (OS && slot) {
            // raising all prices together frees the slots in the order of their values, lowering fills the next best
            const bool real = mine > keyo;
            const int mg = (int)((real ? mine - keyo : keyo - mine) >> ib);
            if (mg < W) atomicAdd(&s_hist[((real ? 0 : nb) + bin_of(mg, w0, bs)) * ES + E], 1);
        }
        if (!near) continue;
        if (TOGETHER) {
            unsigned h = ~0u, f = 0u;                    // the lowest hold with a price, the best of the others without
            asm volatile("" : "+v"(priced));             // (else a condition of every column is kept in registers: 50 of them spilled)
#pragma unroll
            for (int m = 0; m < EPL; ++m) {
                const bool p = (priced >> m) & 1u, held = key[m] >= kth;
                h = p && held && key[m] < h ? key[m] : h;
                f = p || held || key[m] < f ? f : key[m];
            }
            h = group_min_u32<G>(h);
            f = ~group_min_u32<G>(~f);
            const int mg = (int)((h - f) >> ib);
            if (lg == 0 && live && h != ~0u && f != 0u && mg < W) atomicAdd(&s_hist[(2 * nb + 1) * ES + bin_of(mg, w0, bs)], 1);
        }
        if (live) {
#pragma unroll
            for (int m = 0; m < EPL; ++m) {
                const int c = RK::col(m, lg);
                const bool held = key[m] >= thr;
                const int mg = (int)((held ? key[m] - alt : low - key[m]) >> ib);
                if (mg < W && c < E) atomicAdd(&s_hist[((held ? 0 : nb) + bin_of(mg, w0, bs)) * ES + c], 1);
            }
        }
    }
}

// One price pass over `nrows` rows.  Bound by the atomics that add a workgroup's table to the sums: eight wavefronts share a
// table, one workgroup a compute unit, and four neighbouring counts of 16 bits (or two of 32) go in one 64-bit addition: mean over the
// passes 4.9 us at 16384 tokens of 64 experts, 10.2 at 256 experts and 11.0 at 65536 tokens of 128.  Two counts to an addition took
// 5.7, 13.0 and 13.0, one, with half as many wavefronts to a table, 10.6, 20.1 and 18.3; without any of the additions it would be 4.0,
// 6.2 and 7.1.
template <int G, int EPL, int MODE>
__global__ __launch_bounds__(kQThreads) void k_price(PriceArgs a, int t, int nrows, int stride, int shift, int rows_per_wg)
{
    using RK = RowKeys<G, EPL>;
    extern __shared__ __attribute__((aligned(16))) int s_hist[];      // (2 * nb + 1) x ES: margins of holds, of newcomers, holds
    __shared__ int s_p[kPStride];
    PriceArea *ar = a.ar;
    const int tid = threadIdx.x, lg = tid & (G - 1), grp = tid / G;
    const int E = a.E, nb = a.nb, ES = a.es;
    const bool vec = (E & 3) == 0 && (((size_t)a.q) & 15) == 0;
    const int r_first = blockIdx.x * rows_per_wg;
    int r_end = r_first + rows_per_wg;
    r_end = r_end < nrows ? r_end : nrows;
    // the first row is on its way while the prices are fetched
    int nx[EPL];
    {
        int i = r_first + grp;
        i = i < nrows ? i : nrows - 1;
        RK::load(a.q + (size_t)(i * stride + shift) * E, E, vec, lg, nx);
    }
    const PriceMeta mt = ar->meta;
    for (int e = tid; e < E; e += kQThreads) s_p[e] = ar->prices[e];
    if (blockIdx.x == 0 && tid == 0) {
        price_tell(a, mt, t);
        if (a.resumes) ar->t_resume = wall_clock64();
    }
    if (mt.done) return;
    const int hquads = a.quads;
    for (int i = tid; i < hquads; i += kQThreads) ((int4 *)s_hist)[i] = make_int4(0, 0, 0, 0);
    __syncthreads();
    // (the margins of the experts together in a loop of their own, behind the other one: a branch in that took 0.3 us of 5.7, 10007 rows of 96)
    if (MODE == kModeSlack && __builtin_expect(mt.together, 0)) price_rows<G, EPL, false, true, kQThreads>(a, mt.w, r_first, r_end, stride, shift, nx, s_p, s_hist);
    else price_rows<G, EPL, MODE == kModeOver, false, kQThreads>(a, mt.w, r_first, r_end, stride, shift, nx, s_p, s_hist);
    __syncthreads();
    int *hg = ar->hist[blockIdx.x & (a.copies - 1)];
    for (int i = tid; i < hquads; i += kQThreads) {
        const int4 x = ((int4 *)s_hist)[i];
        if (a.half) {
            const unsigned lo = (unsigned)x.x | ((unsigned)x.y << 16), hi = (unsigned)x.z | ((unsigned)x.w << 16);
            const unsigned long long four = lo | ((unsigned long long)hi << 32);
            if (four) atomicAdd((unsigned long long *)hg + i, four);
            continue;
        }
        unsigned long long *h64 = (unsigned long long *)(hg + 4 * i);
        if (x.x | x.y) atomicAdd(h64, (unsigned long long)(unsigned)x.x | ((unsigned long long)(unsigned)x.y << 32));
        if (x.z | x.w) atomicAdd(h64 + 1, (unsigned long long)(unsigned)x.z | ((unsigned long long)(unsigned)x.w << 32));
    }
}

// prices come in units of 1 / 2^sb
__device__ __forceinline__ int first_price(const int64_t *__restrict__ prices_in, int e, int E, int plim)
{
    int sb = 0;
    while ((1 << sb) < E + 1) ++sb;
    const long long p = prices_in && e < E ? prices_in[e] >> sb : 0;
    return p < 0 ? 0 : (p > plim ? plim : (int)p);
}
__device__ __forceinline__ PriceMeta first_meta(const PriceArea *ar, const int64_t *prices_in, int retry, int E)
{
    return PriceMeta{retry ? ar->meta.w : kFirstWindow, 0, 2, retry ? ar->meta.passes : prices_in ? -1 : 0, 0x7fffffff, 0, 0, E, 0};
}

// All passes of a small batch in one workgroup: a pass takes 4 to 11 us (64 tokens of 8 experts: two to four in 7 us; 256 of 64: 22)
// instead of two launches and their distance, none is launched in vain, and a batch that settles slowly may take more.
template <int G, int EPL, int MODE>
__global__ __launch_bounds__(kUThreads) void k_price_small(PriceArgs a, int n_pass, int plim, const int64_t *__restrict__ prices_in)
{
    using RK = RowKeys<G, EPL>;
    extern __shared__ __attribute__((aligned(16))) int s_hist[];
    __shared__ StepLds s;
    PriceArea *ar = a.ar;
    const int tid = threadIdx.x, lg = tid & (G - 1), grp = tid / G, E = a.E;
    const bool vec = (E & 3) == 0 && (((size_t)a.q) & 15) == 0;
    const int hquads = a.quads;
    PriceMeta mt = first_meta(ar, prices_in, a.retry, E);
    if (tid == 0 && !a.retry) {
        ar->t_start = wall_clock64();
        ar->t_pause = ar->t_resume = 0;
    }
    for (int e = tid; e < kPStride; e += kUThreads) s.was[e] = e >= E ? 0 : a.retry ? ar->prices[e] : first_price(prices_in, e, E, plim);
    for (int i = tid; i < 8 * kPStride; i += kUThreads) (&ar->loads[0][0])[i] = 0;
    for (int t = 0; t < n_pass && !mt.done; ++t) {
        int nx[EPL];
        RK::load(a.q + (size_t)(grp < a.T ? grp : a.T - 1) * E, E, vec, lg, nx);
        for (int i = tid; i < hquads; i += kUThreads) ((int4 *)s_hist)[i] = make_int4(0, 0, 0, 0);
        __syncthreads();
        if (MODE == kModeSlack && __builtin_expect(mt.together, 0)) price_rows<G, EPL, false, true, kUThreads>(a, mt.w, 0, a.T, 1, 0, nx, s.was, s_hist);
        else price_rows<G, EPL, MODE == kModeOver, false, kUThreads>(a, mt.w, 0, a.T, 1, 0, nx, s.was, s_hist);
        for (int e = tid; e < E; e += kUThreads) s.now[e] = s.was[e];
        step_clear(s);
        __syncthreads();
        mt = MODE == kModeSlack && mt.together ? price_step<false, MODE == kModeSlack, true>(a, t, a.T, mt, s_hist, s)
                                               : price_step<false, MODE == kModeSlack, false>(a, t, a.T, mt, s_hist, s);
        __syncthreads();
        for (int e = tid; e < E; e += kUThreads) s.was[e] = s.now[e];
    }
    for (int e = tid; e < E; e += kUThreads) ar->prices[e] = s.was[e];
    if (tid == 0) {
        ar->meta = mt;
        ar->fail = 0;
        if (a.pause >= 0) ar->t_pause = wall_clock64();
    }
    if (tid < kPLists) ar->n_arcs[tid][0] = 0;
}

// What the last pass does with a row; G lanes of a group each, s_p in LDS.
template <int G, int EPL, bool OS>
struct EndRow {
    using RK = RowKeys<G, EPL>;
    const int E, k, ib, lg, bias;
    const unsigned cmask, keyo;                                        // keyo: an unfilled slot: reward 0, price 0
    const int *s_p;
    int pb[EPL];
    bool bad = false;                                                  // something did not fit the packed keys

    __device__ __forceinline__ EndRow(const PriceArgs &a, const int *prices, int lane)
        : E(a.E), k(a.k), ib(a.ib), lg(lane), bias(1 << (31 - a.ib)), cmask((1u << a.ib) - 1), keyo(OS ? (unsigned)(1 << (31 - a.ib)) << a.ib : 0u), s_p(prices)
    {
#pragma unroll
        for (int m = 0; m < EPL; ++m) pb[m] = RK::col(m, lg) < E ? bias - s_p[RK::col(m, lg)] : 0;
    }
    __device__ __forceinline__ void make_keys(int row, const int (&v)[EPL], unsigned (&key)[EPL])
    {
        const unsigned rot = row_mask(row, ib);
#pragma unroll
        for (int m = 0; m < EPL; ++m) {
            const int c = RK::col(m, lg);
            const unsigned x = (unsigned)(v[m] + pb[m]);
            const bool wide = v[m] > (1 << 30) || v[m] < -(1 << 30) || x == 0u || (x >> (32 - ib)) != 0;
            if (c < E) bad |= wide;
            key[m] = c < E ? (x << ib) | ((unsigned)c ^ rot) : 0u;
        }
    }
    // The row's k best experts: assigned, counted, their rewards added to `sum`.  True if it has exchanges under the bound B; its holds are the keys
    // from `thr` on, `mine` that of slot lg, and `nxt` the best key below them.
    __device__ __forceinline__ bool choose(int32_t *assign, int row, bool live, const unsigned (&key)[EPL], int B, int *s_cnt, long long &sum, unsigned &thr,
                                           unsigned &mine, unsigned &nxt)
    {
        unsigned cur = RK::first(key), kth = cur, over = 0, under = 0;
        mine = 0;
        bool have_under = false;
        for (int r = 0; r < k; ++r) {
            if (r) cur = RK::below(key, cur);
            if (lg == r) mine = cur;
            if (OS) {
                if (cur > keyo) over = cur;
                else if (!have_under) {
                    under = cur;
                    have_under = true;
                }
            }
        }
        kth = cur;
        nxt = RK::below(key, cur);
        thr = kth;
        if (!live) return false;
        if (OS && !have_under) under = nxt;
        const bool real = lg < k && (!OS || mine > keyo);
        if (lg < k) {
            const int c = (int)((mine & cmask) ^ row_mask(row, ib));
            assign[(size_t)row * k + lg] = real ? c : -1;
            if (real) {
                if (c < E) atomicAdd(&s_cnt[c], 1);
                else bad = true;
                sum += (long long)(int)(mine >> ib) - bias + s_p[c < E ? c : 0];
            }
        }
        if (OS) {
            thr = kth > keyo ? kth : keyo + 1;
            const unsigned alt = under > keyo ? under : keyo;
            nxt = kth > keyo ? nxt : under;
            return (over != 0 && (int)((over - alt) >> ib) <= B) || (have_under && (int)((keyo - under) >> ib) <= B);
        }
        return k < E && (int)((kth >> ib) - (nxt >> ib)) < B;
    }
    // The row's exchanges under the bound, store(place, cost, from, to, row); places are counted in *s_narcs.  `cur` is the row's best key, next(r, x) the
    // one of slot r behind x, `nxt` the best below thr.
    template <class Next, class Store>
    __device__ __forceinline__ void list(int row, const unsigned (&key)[EPL], int B, unsigned thr, unsigned nxt, unsigned cur, const Next &next, int *s_narcs,
                                         const Store &store)
    {
        const int vo = (int)(keyo >> ib), vb = (int)(nxt >> ib);       // vb: the best expert the token does not hold (0: there is none)
        const unsigned rot = row_mask(row, ib);
        auto from_slot = [&](int va, int from) {           // to this lane's columns
            unsigned in = 0;
#pragma unroll
            for (int m = 0; m < EPL; ++m) in |= (RK::col(m, lg) < E && key[m] < thr && va - (int)(key[m] >> ib) < B ? 1u : 0u) << m;
            if (!in) return;
            int at = atomicAdd(s_narcs, __popc(in));
#pragma unroll
            for (int m = 0; m < EPL; ++m)
                if ((in >> m) & 1u) store(at++, va - (int)(key[m] >> ib), from, RK::col(m, lg), row);
        };
        int held = 0;
        for (int r = 0; r < k && cur >= thr; ++r) {
            const int va = (int)(cur >> ib), from = (int)((cur & cmask) ^ rot);
            ++held;
            if (va - vb < B) from_slot(va, from);
            if (OS && lg == 0 && va - vo < B) store(atomicAdd(s_narcs, 1), va - vo, from, E, row);
            if (r + 1 < k) cur = next(r + 1, cur);
        }
        if (OS && held < k) from_slot(vo, E);
    }
};

// The last pass: assignment, pairs per block and expert, sum of the rewards, and the arcs under the bound.  A row near a change is
// evaluated a second time for its arcs, which a block gathers in LDS: 18 us for 65536 tokens of 128 experts, 8.6 for 16384 of 64 (30 and
// 16 while the rows were evaluated three times, to count the arcs and to write them in the order of the rows).
template <int G, int EPL, bool OS>
__global__ __launch_bounds__(kPThreads) void k_price_assign(PriceArgs a, int if_done)          // if_done: nothing before that, a pass `if_done` will follow
{
    using RK = RowKeys<G, EPL>;
    constexpr int NG = kPThreads / G;
    __shared__ int s_p[kPStride], s_cnt[kPStride];
    __shared__ unsigned s_thr[kPRowsMax];
    __shared__ short s_queue[kPRowsMax];
    __shared__ unsigned long long s_arc[kBlockArcs];
    __shared__ int s_arc_tok[kBlockArcs];
    __shared__ int s_nq, s_narcs, s_base, s_bad;
    __shared__ long long s_sum[kPThreads / 64];
    PriceArea *ar = a.ar;
    const int tid = threadIdx.x, lane = tid & 63, lg = tid & (G - 1), grp = tid / G;
    const int E = a.E, w = blockIdx.x;
    const bool vec = (E & 3) == 0 && (((size_t)a.q) & 15) == 0;
    const int row0 = w * a.rows;
    int nr = a.T - row0;
    nr = nr < a.rows ? nr : a.rows;
    int nx[EPL];
    RK::load(a.q + (size_t)(row0 + (grp < nr ? grp : nr - 1)) * E, E, vec, lg, nx);
    for (int j = tid; j < kPStride; j += kPThreads) s_cnt[j] = 0;
    if (tid == 0) s_nq = s_narcs = s_bad = 0;
    for (int e = tid; e < E; e += kPThreads) s_p[e] = ar->prices[e];
    const int B = ar->meta.bound;
    if (a.resumes && w == 0 && tid == 0) ar->t_resume = wall_clock64();
    if (if_done) {
        const PriceMeta mt = ar->meta;
        if (w == 0 && tid == 0) price_tell(a, mt, if_done);
        if (!mt.done) return;
    }
    __syncthreads();
    EndRow<G, EPL, OS> er(a, s_p, lg);
    long long sum = 0;
    for (int l0 = grp; l0 - grp < nr; l0 += NG) {
        const bool live = l0 < nr;
        const int lr = live ? l0 : nr - 1;
        int v[EPL];
#pragma unroll
        for (int m = 0; m < EPL; ++m) v[m] = nx[m];
        if (l0 - grp + NG < nr) RK::load(a.q + (size_t)(row0 + (l0 + NG < nr ? l0 + NG : nr - 1)) * E, E, vec, lg, nx);
        unsigned key[EPL], thr, mine, nxt;
        er.make_keys(row0 + lr, v, key);
        if (er.choose(a.assign, row0 + lr, live, key, B, s_cnt, sum, thr, mine, nxt) && lg == 0) {
            s_thr[lr] = thr;
            s_queue[atomicAdd(&s_nq, 1)] = (short)lr;
        }
    }
    if (er.bad) s_bad = 1;
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned lo = __shfl_xor((unsigned)sum, off), hi = __shfl_xor((unsigned)((unsigned long long)sum >> 32), off);
        sum += (long long)(((unsigned long long)hi << 32) | lo);
    }
    if (lane == 0) s_sum[tid >> 6] = sum;
    __syncthreads();
    for (int e = tid; e < E; e += kPThreads) {
        const int c = s_cnt[e];
        a.blkcnt[(size_t)w * E + e] = c;
        if (c) atomicAdd(&ar->loads[w & 7][e], c);
    }
    if (tid == 0) {
        a.wg_sum[w] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        if (s_bad) ar->fail = 1;
    }
    if (s_bad) return;
    // arcs, gathered in LDS first (their order does not matter)
    const int list = w & (a.lists - 1), list_room = kPArcBuf / a.lists, list0 = list * list_room;
    int *n_list = ar->n_arcs[list];
    auto store = [&](int at, int cost, int from, int to, int row) {
        const unsigned long long r = ((unsigned long long)(unsigned)cost << 32) | (unsigned)((from << 16) | to);
        if (at < kBlockArcs) {
            s_arc[at] = r;
            s_arc_tok[at] = row;
        } else {                                           // (batches whose exchanges are all listed, in few blocks)
            const int pos = atomicAdd(n_list, 1);
            if ((unsigned)pos < (unsigned)list_room) {
                ar->arc[list0 + pos] = r;
                ar->arc_tok[list0 + pos] = row;
            }
        }
    };
    const int nq = s_nq;
    for (int i = grp; i < nq; i += NG) {
        const int lr = s_queue[i];
        int v[EPL];
        unsigned key[EPL];
        RK::load(a.q + (size_t)(row0 + lr) * E, E, vec, lg, v);
        er.make_keys(row0 + lr, v, key);
        const unsigned thr = s_thr[lr];
        er.list(row0 + lr, key, B, thr, RK::below(key, thr), RK::first(key), [&](int, unsigned x) { return RK::below(key, x); }, &s_narcs, store);
    }
    __syncthreads();
    const int n = s_narcs < kBlockArcs ? s_narcs : kBlockArcs;
    if (n == 0) return;
    if (tid == 0) s_base = atomicAdd(n_list, n);
    __syncthreads();
    for (int i = tid; i < n; i += kPThreads)
        if ((unsigned)(s_base + i) < (unsigned)list_room) {                      // (beyond: the search sees the count)
            ar->arc[list0 + s_base + i] = s_arc[i];
            ar->arc_tok[list0 + s_base + i] = s_arc_tok[i];
        }
}

// ---- the search ----

constexpr int kMovedSlots = 1024;     // at least half of them stay free
static_assert(kMovedSlots >= 2 * kPriceMaxE && (kMovedSlots & (kMovedSlots - 1)) == 0, "paths are disjoint: one arc into every node but the roots");

struct FinishLds {
    unsigned ft[kPArcs];              // from << 16 | to
    int tok[kPArcs];                  // -1: an arc of Z
    unsigned cost[kPArcs];            // reduced cost; kWInf: the arc is gone
    unsigned short near[kPArcs];      // arcs within the search's reach
    unsigned lab[kPStride];           // distance << 10 | hops
    unsigned pred[kPStride];          // last arc of the shortest path: its token + 1 (0: an arc of Z) << 10 | the node it comes from
    unsigned best[kPStride];          // of a branch: distance << 10 | target
    int p[kPStride], pi[kPStride], ex[kPStride], sl[kPStride], dd[kPStride];       // dd: what the last search added to pi
    unsigned mft[kPStride];           // path arcs ...
    int mtok[kPStride];               // ... and their tokens
    unsigned wkey[kPStride];          // paths offered by their branches: distance << 10 | target ...
    int wroot[kPStride];              // ... their root ...
    unsigned wtok[kPStride];          // ... the token that leaves or joins the root (+ 1) ...
    int wlen[kPStride];               // ... and their arcs, 0 if the root has no unit left for them
    unsigned moved[kMovedSlots];      // path arcs, hashed by their tokens: token << 10 | arc
    int chg[3], wsum[2][kFThreads / 64];
    int bad, bad_move, dmax, n_win, n_near[2], n_off, n_arcs, hit;       // bad: found while paths are chosen; bad_move: while tokens move
    long long dsum;
};

constexpr int kSpareBit = 1 << 16, kReachShift = 2, kManyArcs = 3 * kFThreads, kSearches = 8, kRelax = 4, kSearchRegs = 2;
constexpr unsigned kLabInf = ~0u, kPredNone = ~0u, kMovedNone = ~0u;
constexpr unsigned kWInf = 0x7fffffffu, kWMax = 1u << 21;  // distances from kWMax on are not followed
static_assert(sizeof(FinishLds) <= 160 * 1024, "one compute unit's LDS");
static_assert(kMaxBound < (int)kWMax, "every arc under the bound can be followed");
static_assert(kMaxTBits <= 21, "a token + 1 and a node fit the words of the shortest paths, none of which is kPredNone");
static_assert(kPriceMaxE < 1024 && kPStride <= 1024, "ten bits for a node, and for an arc of a search's paths");

// The last pass of a small batch (k_price_finish): lanes to a row, rows of a block of the counts, and counts at most.
constexpr int kEndLanes = 8, kEndBlock = kPThreads / kEndLanes;
// The search makes the last pass itself where that costs its one compute unit less than the launch it saves, up to eight rewards to a lane.  A layer
// around it, with a launch for the pass and without: 64 tokens of 8 experts 75.0 -> 70.4 us, of 64 to 8 102 -> 96.5, of 128 126 -> 112, 128 of 16 to 8
// 79.8 -> 73, of 64 to 4 97 -> 92, 500 of 8 to 2 89 -> 83.5, of 16 97.7 -> 94.9; but 400 of 24 to 4 92 -> 95, 128 of 128 to 8 129 -> 130, 256 of 64 to 8
// 113 -> 115, 512 of 64 133 -> 144.  With more demand than room and 65 to 128 experts the kernel spills 20 registers and is still no slower: assignment,
// gates and dispatch of 64 tokens of 128 to 8 of three places 297 -> 251 us, of 100 156 -> 140, 85 of 96 137 -> 133, 110 of 70 118.5 and 118.8.
constexpr int kEndEntries = 8 * kFThreads;
constexpr int kEndCounts = kEndEntries / kEndBlock + kEndLanes * 16;

// A move in the log: token, what it cost (nothing, if it gained), from, to.  Arcs of Z (no token) have Z at one end.
constexpr int kLogCostBits = 23;
__device__ __forceinline__ unsigned long long log_word(int u, int cost, int from, int to)
{
    const int c = cost < 0 ? 0 : cost < (1 << kLogCostBits) ? cost : (1 << kLogCostBits) - 1;
    return ((unsigned long long)(unsigned)(u < 0 ? 0 : u) << (20 + kLogCostBits)) | ((unsigned long long)(unsigned)c << 20) | (unsigned)(from << 10 | to);
}

__device__ __forceinline__ int wave_total(int v) { return __builtin_amdgcn_readlane(wave_sum(v), 63); }
__device__ __forceinline__ int moved_slot(int u) { return (u ^ (u >> 10)) & (kMovedSlots - 1); }

// One workgroup.  Bound by latency: about eight dependent steps between barriers per search, each a few LDS round trips, 6 to 9 us in all.
// What made it shorter (65536 tokens of 128 experts 154 -> 89 us, 10007 of 96 169 -> 96, 16384 of 256 242 -> 126, 16384 of 64 75 -> 43, 64
// of 8 17 -> 12): arcs in LDS and rolled loops instead of nine arcs of every thread in registers (14 KB of code instead of 32 to 40, which
// had to be fetched anew by every launch), only arcs within reach looked at, ties broken by token instead of by place in the list (so the
// list needs no order), a wavefront per offered path instead of a loop over all of them in every thread, and moved tokens hashed.  With
// 512 threads 330 instead of 302 us for a solve of 65536 tokens, with 256 387.
//
// A token that moves from a to b keeps its arcs: those of a become those of b, and what led to b leads to a.  Their reduced costs stay as
// they are, as the arc of the path has none left: the potentials of a and b make up for the difference in value.  So a search reads no
// row, and the list neither grows nor keeps arcs that are gone.  The moves are made at the end, where what the list then lacks of a moved
// token is checked.  With unfilled slots (OS) a token that gives one up may still have others, which its arcs do not say: there the arcs
// of moved tokens are listed anew, from their rows, in every search.  Rows read in every search against moves at the end, means of eight
// batches each: 65536 tokens of 128 experts 77 -> 61 us, 16384 of 256 155 -> 97, 10007 of 96 77 -> 47, 16384 of 64 52 -> 37, 4096 of 16 23
// -> 18, 64 of 8 18 -> 15.  (The prices the passes end at are others since; a single batch may go the other way.)
//
// SEPL > 0: a small batch, whose last pass this workgroup makes itself, eight lanes to a row and SEPL columns to a lane (kEndEntries).  Its arcs never
// leave LDS, and each row lists them from the keys that it has at hand: a queue of rows evaluated anew, as in k_price_assign, took 2 to 4 us more.
template <int TEPL, bool OS, int SEPL>
__global__ __launch_bounds__(kFThreads) void k_price_finish(PriceArgs a, int64_t *prices, int64_t *price_scale, int if_done)
{
    constexpr int NT = kFThreads, NW = NT / 64;
    constexpr int FIRST = 4;                     // arcs of every thread that are requested before their number is known
    static_assert(FIRST * NT <= kPArcBuf && kPArcs <= kPArcBuf, "inside the buffer; the moves fit where the arcs were");
    __shared__ FinishLds s;
    PriceArea *ar = a.ar;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int E = a.E, k = a.k, N = E + 1, mode = a.mode;
    const bool slack = !OS && mode == kModeSlack;
    const PriceMeta mt = ar->meta;
    if (a.resumes && tid == 0) ar->t_resume = wall_clock64();
    const int B = mt.bound, A0 = slack ? 2 * E : 0;
    int rounds = 0, augs = 0;
    bool ok = true, close = false;               // close: not solved, but near enough for another try
    int fail = 0;
    long long sum = 0;
    int *s_cnt = (int *)s.near;                  // SEPL: pairs per (block of rows, expert)
    if constexpr (SEPL > 0) {
        using RK = RowKeys<kEndLanes, SEPL>;
        constexpr int NG = NT / kEndLanes;
        static_assert(sizeof(int) * kEndCounts <= sizeof s.near, "the search lists arcs there later");
        const int lg = tid & (kEndLanes - 1), grp = tid / kEndLanes;
        const bool vec = (E & 3) == 0 && (((size_t)a.q) & 15) == 0;
        int nx[SEPL];
        RK::load(a.q + (size_t)(grp < a.T ? grp : a.T - 1) * E, E, vec, lg, nx);
        for (int i = tid; i < a.n_wg * E; i += NT) s_cnt[i] = 0;
        if (tid < N) {
            s.p[tid] = tid < E ? ar->prices[tid] : 0;
            s.pi[tid] = 0;
        }
        if (tid == 0) {
            s.bad = s.bad_move = s.n_near[0] = 0;
            s.dsum = 0;
            s.n_arcs = A0;
        }
        __syncthreads();
        EndRow<kEndLanes, SEPL, OS> er(a, s.p, lg);
        for (int l0 = grp; l0 - grp < a.T; l0 += NG) {
            const bool live = l0 < a.T;
            const int row = live ? l0 : a.T - 1;
            int v[SEPL];
#pragma unroll
            for (int m = 0; m < SEPL; ++m) v[m] = nx[m];
            if (l0 - grp + NG < a.T) RK::load(a.q + (size_t)(l0 + NG < a.T ? l0 + NG : a.T - 1) * E, E, vec, lg, nx);
            unsigned key[SEPL], thr, mine, nxt;
            er.make_keys(row, v, key);
            if (!er.choose(a.assign, row, live, key, B, s_cnt + row / kEndBlock * E, sum, thr, mine, nxt)) continue;
            er.list(row, key, B, thr, nxt, __shfl(mine, 0, kEndLanes), [&](int r, unsigned) { return __shfl(mine, r, kEndLanes); }, &s.n_arcs,
                    [&](int at, int cost, int from, int to, int u) {
                        if ((unsigned)at >= (unsigned)kPArcs) return;
                        s.ft[at] = (unsigned)((from << 16) | to);
                        s.cost[at] = (unsigned)cost;
                        s.tok[at] = u;
                    });
        }
        for (int i = tid; i < A0; i += NT) {
            s.ft[i] = i < E ? (i << 16) | E : (E << 16) | (i - E);
            s.cost[i] = 0;
            s.tok[i] = -1;
        }
        if (er.bad) s.bad = 1;
        __syncthreads();
        fail = s.bad;
        for (int i = tid; i < a.n_wg * E; i += NT) a.blkcnt[i] = s_cnt[i];
        __syncthreads();
        if (tid == 0) s.bad = 0;
        ok = fail == 0 && s.n_arcs <= kPArcs;
    }
    int tot;
    {
        int e0 = 0;
        auto balance = [&](int v, int n, int p) {        // of the expert that n tokens have taken
            const int sl = (slack && v < E && p == 0 && n < a.C) ? a.C - n : 0;
            s.sl[v] = sl;
            e0 = v < E ? n + sl - a.C : 0;
            s.ex[v] = e0;
        };
        if constexpr (SEPL > 0) {
            if (tid < N) {
                int n = 0;
                for (int w2 = 0; w2 < a.n_wg && tid < E; ++w2) n += s_cnt[w2 * E + tid];
                balance(tid, n, s.p[tid]);
            }
        } else {
            fail = ar->fail;
            const int n_list = lane < a.lists ? ar->n_arcs[lane][0] : 0;            // of list `lane`
            const bool many = a.lists > 1;
            const int per_list = many ? FIRST * NT / kPLists : FIRST * NT, list_room = many ? kPArcBuf / kPLists : kPArcBuf;
            static_assert(FIRST * NT / kPLists % 64 == 0, "a wavefront looks at one list at a time");
            const int *pg = ar->prices;
            unsigned long long arc0[FIRST];
            int tok0[FIRST];
#pragma unroll
            for (int j = 0; j < FIRST; ++j) {
                const int f = tid + j * NT, x = many ? __builtin_amdgcn_readfirstlane(f / (FIRST * NT / kPLists)) : 0, at = x * list_room + (f - x * per_list);
                arc0[j] = ar->arc[at];
                tok0[j] = ar->arc_tok[at];
            }
            if (if_done && !mt.done) return;
            const int n_upto = wave_sum(n_list), n_listed = __builtin_amdgcn_readlane(n_upto, 63);
            ok = fail == 0 && !__any((unsigned)n_list > (unsigned)list_room);
            if (A0 + n_listed > kPArcs) ok = false;
            if (tid == 0) {
                s.bad = s.bad_move = s.n_near[0] = 0;
                s.dsum = 0;
                s.n_arcs = A0 + n_listed;
            }
            for (int w2 = tid; w2 < a.n_wg; w2 += NT) sum += a.wg_sum[w2];
            if (tid < N) {
                const int v = tid;
                int n = 0;
                if (v < E)
                    for (int r = 0; r < 8; ++r) n += ar->loads[r][v];
                const int p = v < E ? pg[v] : 0;
                s.p[v] = p;
                s.pi[v] = 0;
                balance(v, n, p);
            }
            if (ok) {
                for (int i = tid; i < A0; i += NT) {
                    s.ft[i] = i < E ? (i << 16) | E : (E << 16) | (i - E);
                    s.cost[i] = 0;
                    s.tok[i] = -1;
                }
                auto keep = [&](int i, unsigned long long r, int t) {
                    s.ft[A0 + i] = (unsigned)r;
                    s.cost[A0 + i] = (unsigned)(r >> 32);
                    s.tok[A0 + i] = t;
                };
#pragma unroll
                for (int j = 0; j < FIRST; ++j) {
                    const int f = tid + j * NT, x = many ? __builtin_amdgcn_readfirstlane(f / (FIRST * NT / kPLists)) : 0, i = f - x * per_list;
                    const int n = __builtin_amdgcn_readlane(n_list, x);
                    if (i < n) keep(__builtin_amdgcn_readlane(n_upto, x) - n + i, arc0[j], tok0[j]);
                }
                if (__any(n_list > per_list))
                    for (int x = 0; x < a.lists; ++x) {
                        const int n = __builtin_amdgcn_readlane(n_list, x), first = __builtin_amdgcn_readlane(n_upto, x) - n;
                        for (int i = per_list + tid; i < n; i += NT) keep(first + i, ar->arc[x * list_room + i], ar->arc_tok[x * list_room + i]);
                    }
            }
        }
        const int t0 = wave_total(e0), q0 = wave_total(e0 > 0 ? e0 : 0);
        if (lane == 0) {
            s.wsum[0][wv] = t0;
            s.wsum[1][wv] = q0;
        }
        __syncthreads();
        tot = wave_total(lane < NW ? s.wsum[0][lane] : 0);
        const int pos = wave_total(lane < NW ? s.wsum[1][lane] : 0);
        if (tid == E) s.ex[E] = -tot;            // Z or the unfilled slots: supply and demand match overall (only this thread reads it first)
        const int most = pos > pos - tot ? pos : pos - tot;
        if (mode == kModeTight && tot != 0) ok = false;
        if (most > 8 * E + 64) ok = false;       // the prices are far from an equilibrium
        close = fail == 0 && most <= 2 * E + 64;
    }
    __syncthreads();
    // A token's slots and rewards, lane by lane.
    auto load_row = [&](int u, int &h, int (&qv)[TEPL]) {
        // (rows that an earlier search has changed were written by this workgroup)
        h = u >= 0 && lane < k ? __hip_atomic_load(&a.assign[(size_t)u * k + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : -2;
#pragma unroll
        for (int m = 0; m < TEPL; ++m) qv[m] = u >= 0 && lane + 64 * m < E ? a.q[(size_t)u * E + lane + 64 * m] : 0;
    };
    auto held_columns = [&](int h) {             // this lane's columns that the token holds
        unsigned held = 0;
        for (int sl = 0; sl < k; ++sl) {
            const int e = __builtin_amdgcn_readlane(h, sl);
            if (e >= 0 && (e & 63) == lane) held |= 1u << (e >> 6);
        }
        return held;
    };
    auto spread = [&] {                          // of the potentials
        int lo = -0x7fffffff, hi = -0x7fffffff;
        for (int v = lane; v < (OS ? N : E); v += 64) {
            const int x = s.pi[v];
            lo = -x > lo ? -x : lo;
            hi = x > hi ? x : hi;
        }
        return wave_max(hi) + wave_max(lo);
    };
    bool solved = false, forward = true;
    int n_old = 0;                               // arcs that were there when the last paths were taken
    int n_log = 0;                               // moves so far
    unsigned turn = 0;
    const int max_rounds = 8 * E + 128;
    for (; ok; ++rounds) {
        const int ev = tid < N ? s.ex[tid] : 0, n_arcs = s.n_arcs;
        const bool hub = OS && tid == E;
        const bool is_src = ev > 0 && (mode == kModeTight || tid < E), is_snk = ev < 0;
        // sources, sinks, and nodes out of balance: counted while the arcs are listed
        {
            const int c = wave_total((is_src ? 1 : 0) | (is_snk ? 1 << 10 : 0) | (ev != 0 ? 1 << 20 : 0));
            if (lane == 0) s.wsum[rounds & 1][wv] = c;
        }
        // Shortest paths from (backward: to) all roots, up to a reach that starts at a quarter of the bound (an eighth, if there are so many
        // arcs that a quarter of them is more than one to a lane: 16384 tokens of 256 experts 93 -> 83 us) and is doubled up to it until some
        // target lies within it; beyond the bound everything is looked at (doubled on and on, searches of very uneven experts took up
        // to 16 turns: 3000 tokens to 4 of 256, failed tries included, 1224 us, now 583).  Potentials that spread as far as the bound
        // hardly come together again: then, before a longer reach and after more searches than most solves need, this try ends (640 tokens
        // to 2 of 160, two such tries and the auction 2.9 -> 2.4 ms).  Only arcs shorter than the reach can be on such a path: they are
        // listed densely first, so that few arcs meet in a bank of LDS, whose look-ups bound the search.  Labels only fall, and where they
        // end does not depend on the order in which arcs are looked at; hops break ties of distance, so that the last arcs form trees.
        auto list_arcs = [&](unsigned reach, bool fresh, int *n_near) {          // fresh: reduced costs are those before the last paths
            auto near = [&](unsigned c, int i) {
                const bool in = c < reach;
                const unsigned long long bal = __ballot(in);
                if (bal) {
                    int at = 0;
                    if (lane == 0) at = atomicAdd(n_near, (int)__popcll(bal));
                    at = __builtin_amdgcn_readfirstlane(at);
                    if (in) s.near[__builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, (unsigned)at))] = (unsigned short)i;
                }
            };
            if (slack)
                for (int i = tid; i - lane < A0; i += NT) {      // a spare place may leave an expert that has one, and may enter any expert at its price
                    unsigned c = kWInf;
                    if (i < A0) {
                        const int v = i < E ? i : i - E, x = s.p[v] - s.pi[v] + s.pi[E];
                        c = i < E ? (s.sl[v] > 0 ? (unsigned)-x : kWInf) : (unsigned)x;
                        if (c != kWInf && (int)c < 0) s.bad = 1;
                        s.cost[i] = c;
                    }
                    near(c, i);
                }
            for (int i = A0 + tid; i - lane < n_arcs; i += NT) {
                unsigned c = i < n_arcs ? s.cost[i] : kWInf;
                if (fresh && i < n_old && c != kWInf) {
                    const unsigned f = s.ft[i];
                    const int u = s.tok[i], from = (int)(f >> 16), to = (int)(f & 0xffff);
                    int x = moved_slot(u);
                    unsigned o = s.moved[x];
                    c += (unsigned)(s.dd[from] - s.dd[to]);
                    if (o != kMovedNone) {
                        int nf = from, nt = to;
                        for (; o != kMovedNone; o = s.moved[x]) {
                            x = (x + 1) & (kMovedSlots - 1);
                            if ((int)(o >> 10) != u) continue;
                            if (OS) {
                                c = kWInf;                 // (a moved token has new arcs in the list)
                                break;
                            }
                            // (the places of a token that moves twice in a search are four different ones: two it held and two it did not)
                            const unsigned m = s.mft[o & 1023];
                            if (from == (int)(m >> 16)) nf = (int)(m & 0xffff);
                            if (to == (int)(m & 0xffff)) nt = (int)(m >> 16);
                        }
                        if (!OS && (nf != from || nt != to)) s.ft[i] = (unsigned)((nf << 16) | nt);
                    }
                    s.cost[i] = c;
                }
                near(c, i);
            }
            __syncthreads();
        };
        unsigned reach = (unsigned)B >> (n_arcs > kManyArcs ? kReachShift + 1 : kReachShift);
        reach = reach < 1 ? 1 : reach > kWMax ? kWMax : reach;
        list_arcs(reach, n_old > 0, &s.n_near[turn & 1]);
        const int n_all = wave_total(lane < NW ? s.wsum[rounds & 1][lane] : 0);
        if (n_all == 0) {
            solved = true;
            break;
        }
        if (rounds >= max_rounds || (rounds >= kSearches && spread() >= B)) break;
        const int n_src = n_all & 1023, n_snk = (n_all >> 10) & 1023;
        // Spare places, or unfilled slots: whatever is too many goes to the nearest place that lacks a token or has one to
        // spare (the trees grow backward from all of these), and what Z then has too many to the places that lack one.
        // Sent from expert to expert instead, nearly all paths would lead through Z, one at a time.  Otherwise the trees
        // grow from the side with fewer nodes: a tree ends a path at every node of the other side only once, but its root
        // can send as many paths as it has units.
        const bool spare_here = slack && tid < E && ev == 0 && s.sl[tid] > 0;
        const bool via_z = mode != kModeTight && n_src > 0;
        forward = mode == kModeTight ? n_src <= n_snk : !via_z;
        const bool is_root = via_z ? hub || spare_here || (is_snk && tid < E) : forward ? ev > 0 : is_snk;
        const bool is_target = via_z ? is_src : forward ? is_snk && tid < E + (mode == kModeTight) : is_src;
        unsigned limit = 0;
        bool settled = false, target = false;
        int nc = 0;
        auto turned = [&](unsigned f) { return forward ? f : __builtin_amdgcn_alignbit(f, f, 16); };     // tail << 16 | head
        for (;;) {
            limit = reach << 10;
            nc = s.n_near[turn & 1];
            ++turn;
            if (tid == 0) {
                s.lab[kPStride - 1] = kLabInf;
                s.n_off = s.dmax = s.n_win = s.hit = s.n_near[turn & 1] = 0;
            }
            if (tid < N) {
                s.lab[tid] = is_root ? 0u : kLabInf;
                s.pred[tid] = kPredNone;
                s.best[tid] = kLabInf;
            }
            if (tid < 3) s.chg[tid] = 0;
            // Each wavefront with arcs keeps them in registers, R to a lane; straight code, as taken branches cost more than the
            // look-ups.  (Spread over fewer wavefronts, several arcs to a lane, it took longer.)
            auto search = [&](auto regs) {
                constexpr int R = decltype(regs)::value;
                unsigned from[R], to[R], x[R], seen[R];
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    from[j] = to[j] = kPStride - 1;                      // a node whose label stays
                    x[j] = 0;
                    seen[j] = kLabInf;
                    const int y = tid + j * NT;
                    if (y < nc) {
                        const int i = s.near[y];
                        const unsigned f = turned(s.ft[i]);
                        from[j] = f >> 16;
                        to[j] = f & 0xffff;
                        x[j] = (s.cost[i] << 10) + 1;
                    }
                }
                __syncthreads();
                for (int it = 0; it < 4 * N; ++it) {
                    if (wv * 64 < nc) {
                        bool any = false;
                        // (no look at the head's label first: the round trip would be as long as the one behind it)
#pragma unroll
                        for (int again = 0; again < kRelax; ++again) {
                            unsigned la[R];
#pragma unroll
                            for (int j = 0; j < R; ++j) la[j] = __hip_atomic_load(&s.lab[from[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                            for (int j = 0; j < R; ++j) {
                                const bool fell = la[j] != seen[j];      // (a label that has fallen is below the limit)
                                seen[j] = la[j];
                                any |= fell;
                                if (fell && la[j] + x[j] < limit) atomicMin(&s.lab[to[j]], la[j] + x[j]);
                            }
                            if (R == kSearchRegs)
                                for (int y = tid + R * NT; y < nc; y += NT) {
                                    const int i = s.near[y];
                                    const unsigned f = turned(s.ft[i]), l = s.lab[f >> 16], c = l + (s.cost[i] << 10) + 1;
                                    if (l < limit && c < limit && c < s.lab[f & 0xffff]) {
                                        atomicMin(&s.lab[f & 0xffff], c);
                                        any = true;
                                    }
                                }
                        }
                        if (any) s.chg[it % 3] = 1;
                        if (tid == 0) s.chg[(it + 1) % 3] = 0;
                    }
                    __syncthreads();
                    if (!s.chg[it % 3]) return true;
                }
                return false;
            };
            if (nc <= NT) settled = search(std::integral_constant<int, 1>());
            else settled = search(std::integral_constant<int, kSearchRegs>());
            target = is_target && s.lab[tid] < limit;
            if (target) s.hit = 1;
            // last arcs of the paths (the lowest token wins, then the lowest node)
            for (int x = tid; x < nc; x += NT) {
                const int i = s.near[x];
                const unsigned f = turned(s.ft[i]), la = s.lab[f >> 16];
                if (la < limit && la + (s.cost[i] << 10) + 1 == s.lab[f & 0xffff])
                    atomicMin(&s.pred[f & 0xffff], ((unsigned)(s.tok[i] + 1) << 10) | (f >> 16));
            }
            __syncthreads();
            if (s.hit || !settled || reach >= kWMax) break;
            if (spread() >= B) {
                settled = false;
                break;
            }
            reach = reach >= (unsigned)B ? kWMax : 2 * reach < (unsigned)B ? 2 * reach : (unsigned)B;
            list_arcs(reach, false, &s.n_near[turn & 1]);
        }
        const unsigned lv = tid < N ? s.lab[tid] : kLabInf;
        const bool reached = lv < limit;
        const int dist = reached ? (int)(lv >> 10) : 0, hops = (int)(lv & 1023);
        // every branch of a root offers the path to its nearest target, a root takes as many as it has units
        int root = tid, branch = tid;
        const unsigned my_key = ((unsigned)dist << 10) | (unsigned)tid;
        if (target) {
            for (int i = 0; i < hops; ++i) {
                const unsigned l = s.pred[root];
                if (l == kPredNone) break;
                branch = root;
                root = (int)(l & 1023);
            }
            atomicMin(&s.best[branch], my_key);
        }
        __syncthreads();
        if (target && s.best[branch] == my_key) {
            const int i = atomicAdd(&s.n_off, 1);
            s.wkey[i] = my_key;
            s.wroot[i] = root;
            s.wtok[i] = s.pred[branch] >> 10;
        }
        for (int i = tid; i < kMovedSlots; i += NT) s.moved[i] = kMovedNone;
        __syncthreads();
        const int n_off = s.n_off;
        // (the i-th path offered belongs to wavefront i modulo their number)
        for (int i = wv; i < n_off; i += NW) {
            const unsigned key = s.wkey[i], tk = s.wtok[i];
            const int rt = s.wroot[i], er = s.ex[rt];
            int before = 0;
            bool clash = false;
            for (int c = lane; c - lane < n_off; c += 64) {
                const bool ahead = c < n_off && s.wkey[c] < key && s.wroot[c] == rt;
                before += __popcll(__ballot(ahead));
                clash |= __any(ahead && tk != 0 && s.wtok[c] == tk) != 0;       // (the token has one place at the root)
            }
            const int units = OS && via_z && rt == E ? 1 << 30 : er != 0 ? (er > 0 ? er : -er) : s.sl[rt];
            const bool win = !clash && before < units;
            if (lane == 0) {
                // (a root that has no token too many or too few gives a spare place)
                s.wlen[i] = win ? (int)(s.lab[key & 1023] & 1023) | (slack && via_z && er == 0 ? kSpareBit : 0) : 0;
                if (win) {
                    atomicMax(&s.dmax, (int)(key >> 10));
                    atomicAdd(&s.n_win, 1);
                }
            }
        }
        __syncthreads();
        int nm = 0;                              // path arcs in all
        {
            int mine = -1, at = 0, y = 0;
            for (int i0 = 0; i0 < n_off; i0 += 64) {
                const int len = i0 + lane < n_off ? s.wlen[i0 + lane] & (kSpareBit - 1) : 0;
                const int inc = wave_sum(len);
                for (int i = i0 + wv; i < i0 + 64 && i < n_off; i += NW, ++y) {
                    const int x = nm + __builtin_amdgcn_readlane(inc - len, i - i0);
                    if (lane == y) {
                        mine = i;
                        at = x;
                    }
                }
                nm += __builtin_amdgcn_readlane(inc, 63);
            }
            const int word = mine >= 0 ? s.wlen[mine] : 0, len = word & (kSpareBit - 1);
            if (len > 0 && nm <= kPStride && n_log + nm <= kPArcs) {        // (nm: always, the paths are disjoint)
                const int tgt = (int)(s.wkey[mine] & 1023), rt = s.wroot[mine];
                int x = tgt;
                for (int i = 0; i < len; ++i) {
                    const unsigned l = s.pred[x];
                    if (l == kPredNone) {
                        s.bad = 1;
                        break;
                    }
                    const int tail = (int)(l & 1023), from = forward ? tail : x, to = forward ? x : tail;
                    s.mft[at + i] = (unsigned)((from << 16) | to);
                    s.mtok[at + i] = (int)(l >> 10) - 1;
                    if (slack) {
                        if (from == E) atomicAdd(&s.sl[to], 1);          // a spare place comes to `to`
                        else if (to == E) atomicAdd(&s.sl[from], -1);    // a spare place leaves
                    }
                    x = tail;
                }
                const int src = forward ? rt : tgt, snk = forward ? tgt : rt;
                atomicAdd(&s.ex[src], -1);
                if (!(word & kSpareBit)) atomicAdd(&s.ex[snk], 1);
                else {
                    atomicAdd(&s.sl[snk], -1);
                    atomicAdd(&s.ex[E], 1);
                }
            }
        }
        if (tid < N) {
            // (no further than the paths taken: experts far from them keep their potentials close to the others)
            const int dm = s.dmax, d = reached && dist < dm ? dist : dm;
            s.dd[tid] = forward ? d : -d;
            s.pi[tid] += forward ? d : -d;
        }
        __syncthreads();
        if (s.n_win == 0 || s.bad || !settled || nm > kPStride || n_log + nm > kPArcs) break;         // no way to place what is left with these arcs
        augs += s.n_win;
        n_old = n_arcs;
        // the moves: a hash by token for the list, and for the end, with what each costs, where the arcs were
        if (tid < nm) {
            const int u = s.mtok[tid];
            const unsigned f = s.mft[tid];
            if (u >= 0)
                for (int y = moved_slot(u); atomicCAS(&s.moved[y], kMovedNone, (unsigned)(u << 10 | tid)) != kMovedNone;) y = (y + 1) & (kMovedSlots - 1);
            if (!OS) {
                const int from = (int)(f >> 16), to = (int)(f & 0xffff), cost = s.pi[to] - s.pi[from];
                if (u >= 0) sum += (long long)(s.p[to] - s.p[from]) - cost;        // (the arc has no reduced cost left)
                __hip_atomic_store(&ar->arc[n_log + tid], log_word(u, cost, from, to), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        n_log += OS ? 0 : nm;
        if constexpr (!OS) {
            __syncthreads();
            continue;
        }
        // OS: the tokens of the paths move, one per wavefront at a time, with the next one's row on its way.  The arcs a token
        // offers from where it is now replace its old ones in the list.
        int un = wv < nm ? s.mtok[wv] : -1, hn, qn[TEPL];
        load_row(un, hn, qn);
        for (int i = wv; i < nm; i += NW) {
            int u = un, h = hn, qv[TEPL];
#pragma unroll
            for (int m = 0; m < TEPL; ++m) qv[m] = qn[m];
            un = i + NW < nm ? s.mtok[i + NW] : -1;
            load_row(un, hn, qn);
            bool first = u >= 0;                                  // a token on two paths is taken once
            for (int x0 = 0; x0 < i && first; x0 += 64) first = !__any(x0 + lane < i && s.mtok[x0 + lane] == u);
            if (!first) continue;
            int *bcnt = a.blkcnt + (size_t)(u / a.rows) * E;
            for (int x0 = i & ~63; x0 < nm; x0 += 64) {
                unsigned long long same = __ballot(x0 + lane >= i && x0 + lane < nm && s.mtok[x0 + lane] == u);
                for (; same; same &= same - 1) {
                    const unsigned f = s.mft[x0 + __ffsll((long long)same) - 1];
                    const int from = __builtin_amdgcn_readfirstlane((int)(f >> 16));
                    const int to = __builtin_amdgcn_readfirstlane((int)(f & 0xffff));
                    const unsigned long long bf = __ballot(h == (from < E ? from : -1));
                    const unsigned long long bt = to < E ? __ballot(h == to) : 0ull;
                    if (bf == 0 || bt != 0) {          // (never: the arcs of a token are those of its row)
                        s.bad_move = 1;
                        continue;
                    }
                    if (lane == __ffsll((long long)bf) - 1) h = to < E ? to : -1;
                    int qt = 0, qf = 0;
#pragma unroll
                    for (int m = 0; m < TEPL; ++m) {
                        if (to < E && (to >> 6) == m) qt = __builtin_amdgcn_readlane(qv[m], to & 63);
                        if (from < E && (from >> 6) == m) qf = __builtin_amdgcn_readlane(qv[m], from & 63);
                    }
                    if (lane == 0) {
                        atomicAdd((unsigned long long *)&s.dsum, (unsigned long long)((long long)qt - qf));
                        if (from < E) atomicAdd(&bcnt[from], -1);
                        if (to < E) atomicAdd(&bcnt[to], 1);
                    }
                }
            }
            {                                          // empty slots go to the end of the row
                const unsigned long long be = __ballot(h == -1), br = __ballot(h >= 0);
                const int dst = h >= 0 ? __popcll(br & ((1ull << lane) - 1)) : __popcll(br) + __popcll(be & ((1ull << lane) - 1));
                if (lane < k) __hip_atomic_store(&a.assign[(size_t)u * k + dst], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            // Its exchanges: only slots near the best expert it does not hold have any under the bound.
            const unsigned heldm = held_columns(h);
            int v[TEPL], best = 0, vs = 0;     // vs: value of the expert in slot `lane`
#pragma unroll
            for (int m = 0; m < TEPL; ++m) {
                const int c = lane + 64 * m;
                v[m] = c < E ? qv[m] - s.p[c] : 0;
                const int x = __shfl(v[m], h & 63);
                vs = (h >> 6) == m ? x : vs;
                const bool free = c < E && !((heldm >> m) & 1u);
                if (!free) v[m] = -0x7fffffff;                    // (no exchange)
                best = v[m] > best ? v[m] : best;
            }
            best = wave_max(best);
            auto put = [&](int vh, int from) {
#pragma unroll
                for (int m = 0; m < TEPL; ++m) {
                    const bool in = v[m] != -0x7fffffff && vh - v[m] < B;
                    const unsigned long long bal = __ballot(in);
                    if (!bal) continue;
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&s.n_arcs, (int)__popcll(bal));
                    at = __builtin_amdgcn_readfirstlane(at) + __popcll(bal & ((1ull << lane) - 1));
                    if (in && at < kPArcs) {
                        const int to = lane + 64 * m, wn = vh - v[m] + s.pi[from] - s.pi[to];
                        if (wn < 0) s.bad_move = 1;
                        s.ft[at] = (unsigned)((from << 16) | to);
                        s.cost[at] = (unsigned)wn;
                        s.tok[at] = u;
                    }
                }
            };
            for (unsigned long long r = __ballot(lane < k && h >= 0 && vs - best < B); r; r &= r - 1) {
                const int sl = __ffsll((long long)r) - 1;
                const int e = __builtin_amdgcn_readlane(h, sl), vh = __builtin_amdgcn_readlane(vs, sl);
                put(vh, e);
                if (vh < B && lane == 0) {                  // ... for an unfilled slot
                    const int at = atomicAdd(&s.n_arcs, 1), wn = vh + s.pi[e] - s.pi[E];
                    if (at < kPArcs) {
                        if (wn < 0) s.bad_move = 1;
                        s.ft[at] = (unsigned)((e << 16) | E);
                        s.cost[at] = (unsigned)wn;
                        s.tok[at] = u;
                    }
                }
            }
            if (__any(lane < k && h == -1)) put(0, E);
        }
        __syncthreads();
        if (s.n_arcs > kPArcs || s.bad_move) break;
    }
    __syncthreads();
    // the arcs left out cost at least B: they stay non-negative if the potentials spread less than that
    const int apart = spread();
    int pmin = 0x7fffffff;
    for (int v = lane; v < E; v += 64) pmin = s.p[v] - s.pi[v] < pmin ? s.p[v] - s.pi[v] : pmin;
    pmin = -wave_max(-pmin);
    if (!OS && solved && apart < B && n_log > 0) {
        // The moves are made, one thread for all of a token.  An exchange of a token that has moved is in the list unless it costs the bound
        // less what the moves cost; where the potentials spread as far as that its row is looked at (as good as never): none of its
        // experts may be worth less than one that it does not hold.
        constexpr unsigned short none = 0xffff;
        static_assert(kPArcs < none, "a word of `near` links two moves");
        for (int i = tid; i < kMovedSlots; i += NT) s.moved[i] = kMovedNone;
        if (tid == 0) s.n_off = 0;
        for (int i = tid; i < n_log; i += NT) {
            const unsigned long long r = __hip_atomic_load(&ar->arc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const unsigned from = (unsigned)(r >> 10) & 1023, to = (unsigned)r & 1023;
            s.tok[i] = (int)from == E || (int)to == E ? -1 : (int)(r >> (20 + kLogCostBits));
            s.cost[i] = (unsigned)(r >> 20) & ((1u << kLogCostBits) - 1);
            s.ft[i] = from << 16 | to;
        }
        __syncthreads();
        for (int i = tid; i < n_log; i += NT) {
            const int u = s.tok[i];
            if (u < 0) continue;
            const unsigned o = atomicExch(&s.moved[moved_slot(u)], (unsigned)i);
            s.near[i] = o == kMovedNone ? none : (unsigned short)o;
        }
        __syncthreads();
        for (int i = tid; i < n_log; i += NT) {
            const int u = s.tok[i];
            bool first = u >= 0;
            unsigned head = kMovedNone;
            if (first) {
                head = s.moved[moved_slot(u)];
                for (unsigned o = head; o != none; o = s.near[o]) first = first && !(s.tok[o] == u && (int)o < i);
            }
            if (!first) continue;
            int *row = a.assign + (size_t)u * k, *bcnt = a.blkcnt + (size_t)(u / a.rows) * E;
            long long cost = 0;
            for (int at = i; at < n_log;) {
                const unsigned f = s.ft[at];
                const int from = (int)(f >> 16), to = (int)(f & 0xffff);
                cost += s.cost[at];
                int sl = -1;
#pragma unroll 8
                for (int x = 0; x < k; ++x)
                    if (__hip_atomic_load(row + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == from) sl = x;
                if (sl < 0) s.bad_move = 1;                  // (never: the arcs of a token are those of its row)
                else __hip_atomic_store(row + sl, to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                atomicAdd(&bcnt[from], -1);
                atomicAdd(&bcnt[to], 1);
                int then = n_log;
                for (unsigned o = head; o != none; o = s.near[o])
                    if (s.tok[o] == u && (int)o > at && (int)o < then) then = (int)o;
                at = then;
            }
            if (cost + apart >= B) {
                const int x = atomicAdd(&s.n_off, 1);
                if (x < kPStride) s.mtok[x] = u;
                else s.bad_move = 1;
            }
        }
        __syncthreads();
        const int n_far = s.n_off < kPStride ? s.n_off : kPStride;
        for (int i = wv; i < n_far; i += NW) {
            int h, qv[TEPL];
            load_row(s.mtok[i], h, qv);
            const unsigned held = held_columns(h);
            int least = 0x7fffffff, most = -0x7fffffff;
#pragma unroll
            for (int m = 0; m < TEPL; ++m) {
                const int c = lane + 64 * m;
                if (c >= E) continue;
                const int v = qv[m] - s.p[c] + s.pi[c];
                if ((held >> m) & 1u) least = v < least ? v : least;
                else most = v > most ? v : most;
            }
            if (wave_max(most) > -wave_max(-least) && lane == 0) s.bad_move = 1;
        }
        __syncthreads();
    }
    const bool certified = solved && apart < B && !s.bad_move;
    int sb = 0;
    while ((1 << sb) < E + 1) ++sb;
    if (certified && prices) {
        const int shift = slack ? -s.pi[E] : pmin;
        for (int e = tid; e < E; e += NT) prices[e] = (int64_t)(s.p[e] - s.pi[e] - shift) << sb;
    }
    // (one addition a wavefront: those of all lanes to one word are compiled into a loop over the lanes, 2 us)
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned x = __shfl_xor((unsigned)sum, off), y = __shfl_xor((unsigned)((unsigned long long)sum >> 32), off);
        sum += (long long)(((unsigned long long)y << 32) | x);
    }
    if (lane == 0 && sum) atomicAdd((unsigned long long *)&s.dsum, (unsigned long long)sum);
    __syncthreads();
    if (tid == 0) {
        if (certified && price_scale) *price_scale = (int64_t)1 << sb;
        ar->arrived = 0;
        PriceReport &r = ar->report;
        r.total = s.dsum;
        r.flow = OS ? E * a.C : a.T * k;
        r.passes = mt.passes;
        r.fin = certified ? 2 : close ? 1 : 3;
        r.paths = augs;
        r.t_end = wall_clock64();
        r.ticks = (r.t_end - ar->t_start) - (ar->t_resume - ar->t_pause);
    }
}

__global__ __launch_bounds__(kPThreads) void k_price_init(PriceArea *ar, int quads, int E, int plim,
                                                          const int64_t *__restrict__ prices_in, int retry)
{
    const int i0 = blockIdx.x * kPThreads + threadIdx.x, n = gridDim.x * kPThreads;
    for (int r = 0; r < kPCopies; ++r)
        for (int i = i0; i < quads; i += n) ((int4 *)ar->hist[r])[i] = make_int4(0, 0, 0, 0);
    for (int i = i0; i < 8 * kPStride; i += n) (&ar->loads[0][0])[i] = 0;
    for (int i = i0; i < kPLists; i += n) ar->n_arcs[i][0] = 0;
    for (int i = i0; i < kPStride && !retry; i += n) ar->prices[i] = first_price(prices_in, i, E, plim);
    if (i0 == 0) {
        ar->fail = 0;
        ar->meta = first_meta(ar, prices_in, retry, E);
        if (!retry) {
            ar->t_start = wall_clock64();
            ar->t_pause = ar->t_resume = 0;
        }
    }
}

}  // namespace

static_assert((sizeof(PriceArea) + 15) / 16 * 16 <= 864 * 1024, "the workspace holds the tables");

// Lanes per row (one per slot at least), columns per lane, rows per block of the final pass.
static bool price_shape(int T, int E, int k, int &G, int &EPL, int &rows, int &n_wg)
{
    if (E < 2 || E > kPriceMaxE || k > E) return false;
    G = 8;
    EPL = 1;
    while (G < k) G *= 2;
    while (G * 16 < E) G *= 2;
    while (G * EPL < E) EPL *= 2;
    rows = kPThreads / G;
    while (rows * 2 * k <= 1024 && rows * 2 <= kPRowsMax && (T + 2 * rows - 1) / (2 * rows) >= 512) rows *= 2;
    n_wg = (T + rows - 1) / rows;
    return rows * k <= 1024 && n_wg <= kPBlocks;
}

// Rows per workgroup of a price pass.
static int price_pass_rows(int nrows, int E, int k)
{
    int G, EPL, rows, n_wg;
    (void)price_shape(nrows, E, k, G, EPL, rows, n_wg);
    int rw = kQThreads / G;
    while (rw * 2 <= 128 && (nrows + 2 * rw - 1) / (2 * rw) >= 256) rw *= 2;
    return rw;
}

bool price_supported(int T, int E, int k)
{
    int G, EPL, rows, n_wg;
    return price_shape(T, E, k, G, EPL, rows, n_wg);
}

int32_t price_enqueue(const int32_t *q, int T, int E, int k, int C, const int64_t *prices_in, int retry, PricePart part, int32_t *assign, int64_t *prices,
                      int64_t *price_scale, char *ws, PriceGeometry *geom, hipStream_t s)
{
    int *words = nullptr, *words_dev = nullptr, seq = 0;
    const int32_t wrc = price_words(&words, &words_dev, &seq, part != kPriceRest);
    if (wrc) return wrc;
    volatile int *hw = words;
    if (part != kPriceRest) hw[kPriceWordDone] = hw[kPriceWordPasses] = 0;
    WorkspaceLayout L = workspace_layout(T, E, k);
    PriceArgs a;
    a.seq = seq;
    a.q = q;
    a.host = words_dev;
    a.assign = assign;
    a.ar = (PriceArea *)(ws + L.price_off);
    a.blkcnt = (int *)(ws + L.wcnt_off);
    a.wg_sum = (long long *)(ws + L.price_off + (sizeof(PriceArea) + 15) / 16 * 16);
    a.T = T;
    a.E = E;
    a.k = k;
    a.C = C;
    const long long spare = (long long)E * C - (long long)T * k;
    a.mode = spare == 0 ? kModeTight : spare > 0 ? kModeSlack : kModeOver;
    const int stride = T / kSampleRows;
    const int n_sampled = stride >= kSampleFrom && !prices_in && !retry ? kSampledPasses : 0;
    {
        const int rw = price_pass_rows(T, E, k), wgs = (T + rw - 1) / rw;
        a.copies = kPCopies;
        while (a.copies > 2 && a.copies * kPWgPerCopy > wgs) a.copies /= 2;
        // what one row adds to a count at most: one, or to that of the unfilled slots one a slot
        const long long each = a.mode == kModeOver ? k : 1;
        a.half = (wgs + a.copies - 1) / a.copies * (long long)rw * each < (1 << 16) ? 1 : 0;
    }
    a.arcs_wanted = std::min(kArcsPerExpert * E, kArcsWanted);
    a.retry = retry > 0 ? 1 : 0;
    a.arcs_late = std::min(kLateArcsPerExpert * E, kArcsWanted);
    if (retry) a.arcs_wanted = a.arcs_late = std::min((1 + retry) * a.arcs_late, kArcsMost);
    a.ib = 1;
    while ((1 << a.ib) < E) ++a.ib;
    a.nb = price_bins(E);
    a.bshift = E <= 256 ? 22 : 23;
    a.es = price_columns(E, a.mode != kModeOver);
    a.quads = price_table_ints(E, a.mode != kModeOver, a.mode == kModeSlack) / 4;

    int G, EPL, rows;
    if (!price_shape(T, E, k, G, EPL, rows, a.n_wg) || a.n_wg > L.max_wg) return MAXSCORE_ERR_SHAPE;
    a.rows = rows;
    a.lists = a.n_wg >= kPListsFrom ? kPLists : 1;
    a.sampled = n_sampled;
    a.look = a.mode != kModeSlack && !retry ? n_sampled + kTightPasses - 2 : -1;
    a.pause = part == kPriceBegin ? kPriceAhead - 1 : -1;
    a.resumes = part == kPriceRest ? 1 : 0;
    geom->report = &a.ar->report;
    geom->arrived = &a.ar->arrived;
    geom->rows = rows;
    geom->n_wg = a.n_wg;
    geom->ends_ahead = geom->ends_early = 0;

    int32_t mrc = MAXSCORE_OK;                    // (timing marks)
    auto mark = [&] { mrc = mrc ? mrc : solver_mark(s); };
    const bool os = a.mode == kModeOver;
    const size_t shm = sizeof(int4) * (size_t)a.quads;
    const int n_pass = n_sampled + (retry ? kRetryPasses : a.mode == kModeSlack ? kSlackPasses : kTightPasses);
    const bool small = (long long)T * G <= kSmallThreads && (long long)T * E <= kSmallEntries && shm + sizeof(StepLds) <= 64 * 1024;
    const int plim = (1 << (31 - a.ib)) - 1;
    geom->one_launch = small ? 1 : 0;
    const bool with_pass = small && G == kEndLanes && a.rows == kEndBlock && T * E <= kEndEntries;
#define MS_PG(GG, XX)                                                                                                     \
    do {                                                                                                                  \
        if (EPL == 1) XX(GG, 1);                                                                                          \
        else if (EPL == 2) XX(GG, 2);                                                                                     \
        else if (EPL == 4) XX(GG, 4);                                                                                     \
        else if (EPL == 8) XX(GG, 8);                                                                                     \
        else XX(GG, 16);                                                                                                  \
    } while (0)
#define MS_SHAPED(XX)            \
    do {                         \
        if (G == 8) MS_PG(8, XX); \
        else if (G == 16) MS_PG(16, XX); \
        else if (G == 32) MS_PG(32, XX); \
        else MS_PG(64, XX);      \
    } while (0)
    // a pass and its step
    auto enqueue_pass = [&](int t) {
        const int st = t < n_sampled ? stride : 1, nrows = st > 1 ? kSampleRows : T, shift = st > 1 ? t * (st / 2) : 0;
        const int rw = price_pass_rows(nrows, E, k), grid = (nrows + rw - 1) / rw;
        mark();
#define MS_P(GG, PP)                                                                                                      \
    do {                                                                                                                  \
        if (a.mode == kModeTight) hipLaunchKernelGGL((k_price<GG, PP, kModeTight>), dim3(grid), dim3(kQThreads), shm, s, a, t, nrows, st, shift, rw); \
        else if (os) hipLaunchKernelGGL((k_price<GG, PP, kModeOver>), dim3(grid), dim3(kQThreads), shm, s, a, t, nrows, st, shift, rw); \
        else hipLaunchKernelGGL((k_price<GG, PP, kModeSlack>), dim3(grid), dim3(kQThreads), shm, s, a, t, nrows, st, shift, rw); \
    } while (0)
        MS_SHAPED(MS_P);
#undef MS_P
        a.resumes = 0;
        mark();
#define MS_U(NN, SS)                                                                                                      \
    do {                                                                                                                  \
        if (!a.half) hipLaunchKernelGGL((k_price_update<NN, price_pieces(false), false, SS>), dim3(1), dim3(kUThreads), shm, s, a, t, nrows); \
        else if (a.quads <= 2 * kUThreads) hipLaunchKernelGGL((k_price_update<NN, 1, true, SS>), dim3(1), dim3(kUThreads), shm, s, a, t, nrows); \
        else hipLaunchKernelGGL((k_price_update<NN, price_pieces(true), true, SS>), dim3(1), dim3(kUThreads), shm, s, a, t, nrows); \
    } while (0)
#define MS_US(NN)                                  \
    do {                                           \
        if (a.mode == kModeSlack) MS_U(NN, true);  \
        else MS_U(NN, false);                      \
    } while (0)
        if (a.copies == 8) MS_US(8);
        else if (a.copies == 4) MS_US(4);
        else MS_US(2);
#undef MS_US
#undef MS_U
        mark();
    };
    // the last pass and the search; if_done: unless the passes turn out to go on with pass if_done
    auto enqueue_end = [&](int if_done) {
#define MS_P(GG, PP)                                                                                                      \
    do {                                                                                                                  \
        if (os) hipLaunchKernelGGL((k_price_assign<GG, PP, true>), dim3(a.n_wg), dim3(kPThreads), 0, s, a, if_done);      \
        else hipLaunchKernelGGL((k_price_assign<GG, PP, false>), dim3(a.n_wg), dim3(kPThreads), 0, s, a, if_done);        \
    } while (0)
        if (!with_pass) {
            MS_SHAPED(MS_P);
            a.resumes = 0;
        }
#undef MS_P
#define MS_F(PP, SS)                                                                                                      \
    do {                                                                                                                  \
        if (os) hipLaunchKernelGGL((k_price_finish<PP, true, SS>), dim3(1), dim3(kFThreads), 0, s, a, prices, price_scale, if_done);  \
        else hipLaunchKernelGGL((k_price_finish<PP, false, SS>), dim3(1), dim3(kFThreads), 0, s, a, prices, price_scale, if_done);    \
    } while (0)
        if (with_pass) {
            if (EPL == 1) MS_F(1, 1);
            else if (EPL == 2) MS_F(1, 2);
            else if (EPL == 4) MS_F(1, 4);
            else if (EPL == 8) MS_F(1, 8);
            else MS_F(2, 16);
        } else if (E <= 64) MS_F(1, 0);
        else if (E <= 128) MS_F(2, 0);
        else if (E <= 256) MS_F(4, 0);
        else MS_F(8, 0);
#undef MS_F
    };
    if (small) {
        if (part != kPriceRest) {
            mark();
#define MS_P(GG, PP)                                                                                                      \
    do {                                                                                                                  \
        if (a.mode == kModeTight) hipLaunchKernelGGL((k_price_small<GG, PP, kModeTight>), dim3(1), dim3(kUThreads), shm, s, a, kSmallPasses, plim, prices_in); \
        else if (os) hipLaunchKernelGGL((k_price_small<GG, PP, kModeOver>), dim3(1), dim3(kUThreads), shm, s, a, kSmallPasses, plim, prices_in); \
        else hipLaunchKernelGGL((k_price_small<GG, PP, kModeSlack>), dim3(1), dim3(kUThreads), shm, s, a, kSmallPasses, plim, prices_in); \
    } while (0)
            MS_SHAPED(MS_P);
#undef MS_P
            mark();
            mark();
        }
        if (part != kPriceBegin) enqueue_end(0);
        MS_HIP(hipGetLastError());
        return mrc;
    }
    if (part != kPriceRest) hipLaunchKernelGGL(k_price_init, dim3(64), dim3(kPThreads), 0, s, a.ar, a.quads, E, plim, prices_in, a.retry);
    struct Words {
        volatile int *hw;
        int seq;
        const PriceMeta *meta;
        hipStream_t s;
        PriceSeen told() const
        {
            const unsigned w = (unsigned)hw[kPriceWordPasses];
            const bool mine = (int)(w >> kPriceSeqBit) == seq;
            return {hw[kPriceWordDone] == seq, mine ? (int)(w & kPricePassMask) : 0, mine && (w >> kPriceFarBit & 1), mine && (w >> kPriceSoonBit & 1)};
        }
        int idle() const
        {
            const hipError_t e = hipStreamQuery(s);
            return e == hipErrorNotReady ? 0 : e == hipSuccess ? 1 : MAXSCORE_ERR_HIP;
        }
        int state(int t, PriceSeen *seen) const
        {
            PriceMeta m;
            MS_HIP(hipMemcpyAsync(&m, meta, sizeof(m), hipMemcpyDeviceToHost, s));
            MS_HIP(hipStreamSynchronize(s));
            *seen = {m.done != 0, t, m.far != 0, false};
            return MAXSCORE_OK;
        }
        void pause() const { __builtin_ia32_pause(); }
    };
    struct Queue {
        decltype(enqueue_pass) &pass;
        decltype(enqueue_end) &enqueue_end;
        Words words;
        PriceGeometry *geom;
        bool ahead = false;
        void end(int if_done)
        {
            enqueue_end(if_done);
            ahead = if_done > 0;
            geom->ends_ahead += ahead ? 1 : 0;
        }
        int seen(int t, PriceSeen *now)
        {
            const int rc = price_seen(words, t, now);
            geom->ends_early += ahead && !rc && !now->done ? 1 : 0;
            ahead = false;
            return rc;
        }
    } queue = {enqueue_pass, enqueue_end, {hw, seq, &a.ar->meta, s}, geom};
    const int32_t prc = price_passes(queue, n_pass, a.look, kFarPasses, part == kPriceBegin, part == kPriceRest);
#undef MS_SHAPED
#undef MS_PG
    MS_HIP(hipGetLastError());
    return prc ? prc : mrc;
}

}  // namespace maxscore
