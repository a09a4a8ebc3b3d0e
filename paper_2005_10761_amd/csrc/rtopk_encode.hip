// rtopk_encode: one node-side step of Algorithm 1 (error compensation, the
// rTop-k operator of Definition 3, residual write-back) as a chain of four to seven
// gfx950 kernels that stream the gradient and the residual exactly once
// (12d bytes). All cross-kernel state lives in the caller's workspace.
//
// The vector is cut into W short contiguous chunks. Every wavefront of the
// streaming kernel owns a piece of the candidate buffer S an eighth as long as the
// chunks it streams (one byte of workspace per element). It appends the entries
// it keeps, chunk after chunk and in index order, and stores for each chunk where
// its slice starts and how many entries it holds. A chunk's entries are therefore
// in index order without any cross-workgroup scan, ticket or fence, and a chunk that is
// dense in candidates takes the room that the wavefront's others leave. A chunk
// that would keep more than there is room for is
// marked; the later kernels read it from the residual buffer, which holds a by
// then. Later kernels walk S chunk by chunk; each of their
// wavefronts takes every U-th chunk, so that a region of the vector that is
// dense in candidates is shared by all wavefronts.
//
// Pipeline:
//   sample     a = g + m at up to 16384 jittered, stratified locations (4 elements
//              each); clears the control block
//   estimate   one workgroup: from the sample's order statistics, a lower
//              bound t_lo that the r-th largest magnitude exceeds and an upper
//              bound t_hi that it stays below, both with 4 doubled sigmas of margin;
//              [t_lo, t_hi] becomes the finely binned part of the histogram
//   fused      a = g + m, stored into the residual buffer (12d bytes, the
//              dominant kernel); entries with magnitude >= t_lo go into the
//              workgroup's own histogram row: up to 2048 linear bins over the
//              fine range and one bin for everything above it (every row also
//              carries the sums over groups of 64 bins). Their Philox keys are
//              computed in the shadow of the stream and compared with an
//              a-priori window [K_lo, K_hi] around the k-th smallest of r
//              uniform keys; an entry above the fine range whose key lies above
//              the window will not be sent, the others -> S with what the key said
//              (a vector of 3 to 4 M elements with few candidates: all of them -> S, unkeyed)
//   pick       one workgroup (short vectors: every classify workgroup for itself, as a rule):
//              the group sums of all rows -> the group that
//              holds the r-th largest magnitude; that group's bins of all
//              rows -> the bin that holds it (the deciding bin)
//   classify   entries of S above the deciding bin are certain members of
//              the top-r set: key below the window: certain winner (counted
//              per chunk), inside: copied to the short list M. Entries inside the deciding bin
//              are copied to the short list B and counted per chunk
//   finalize   one workgroup: exact r-th largest (magnitude, lower index
//              first) inside B -> (T, I*); members of B join the key lists;
//              exact (k - #certain)-th smallest (key, index) in M -> (K*, J*);
//              prefix sum of the winners per quad of chunks. When B overflowed because
//              the deciding bin is one long run of equal magnitudes (zeros,
//              signs, a few levels), the last member is the entry of a known
//              rank in index order and is located from the per-chunk counts.
//              When a short list overflowed otherwise or the key window
//              missed, the same quantities are found by radix selection over
//              S (exact; on all workgroups of the kernel's grid when the vector is
//              long, see grid_select96). Where members that were not to be sent
//              decide after all (the window missed high, the threshold lies above
//              the bracket), one pass over the vector puts them into S first
//   emit       entries of S that are members and winners -> the message in
//              index order, starting at the quad's prefix plus the winners of the quad's
//              earlier chunks; residual at the
//              sent positions <- a - a
// A short vector (counts_all) has no sample and no estimate: its magnitudes are all
// counted while they are added (count), and classify, once it has picked the
// deciding bin (and narrowed it, where it is crowded), makes S from the vector, which is still in the caches.
// Two special cases of Definition 3 take shortcuts: with k == r (top-k) no
// sampling key is ever computed, and with r == d (random-k) no magnitude is
// ever compared: the streaming kernel then keeps the elements whose key lies
// at or below the upper end of the a-priori window, and sample, estimate,
// and pick are not launched at all.
//
// Every kernel serves up to 16 independent vectors of equal sizes per launch
// (blockIdx.z is the member; rtopk_encode_batch), each with its own slice of
// the workspace and computed exactly as if it were alone.
//
// If the sample misleads the estimate so far that S holds fewer than r
// entries, the histogram shows it; pick then raises a flag and classify,
// finalize and emit walk the vector a itself instead of S (slow, exact).
//
// What the hardware punishes shaped this: a device-scope fence inside a
// kernel costs tens of microseconds once a few hundred workgroups execute
// one, atomics on a single address retire at about one per 12 ns, and
// atomics on one 64-byte line queue behind each other too. So on the ordinary
// path no kernel uses a fence, a ticket or a "last workgroup out" protocol and
// workgroups never wait for each other; histograms are accumulated in LDS and
// stored as plain rows; global atomics only go to per-chunk counters. Only the
// rare exact selection over all candidates lets the workgroups of one grid
// meet at barriers, and those have no device-scope fence (grid_barrier).
#include "rtopk_common.h"
#include "../../include/rtopk.h"
#include "../../include/rtopk_diag.h"

#include <math.h>
#include <cstddef>
#include <mutex>
#include <vector>

namespace rtopk {

constexpr u32 kMaxFineBins = 2048;            // linear bins over [t_lo, fine_hi]: 64 .. 2048, by r
constexpr u32 kCoarseBins = 64;               // one more group of bins, of which only the first is used:
                                              // everything above the linear bins
constexpr u32 kMaxBins = kMaxFineBins + kCoarseBins;
constexpr u32 kMaxFusedBlocks = 256;          // rows of per-workgroup histograms (one per compute unit)
constexpr u32 kCoarseSpan = 64;               // bins per group: every row also carries its group sums
constexpr u32 kMaxGroups = kMaxBins / kCoarseSpan;
static_assert(kMaxBins % kCoarseSpan == 0 && kCoarseSpan == 64, "one lane per bin of a group");

constexpr u32 kSampleLoc = 16384;             // sampled locations, 4 consecutive elements each
constexpr u32 kSampleThreads = 256;
constexpr u32 kEstThreads = 1024;
// A sample is the leading 15 bits of a magnitude (the estimate needs 12): the one workgroup of the
// estimate fetches cold lines at 0.4 a ns, and four bytes a sample were 2,048 of them.
constexpr u32 kSampleShift = 16, kBucketShift = 3;
constexpr u64 kShortVector = 1u << 22;
constexpr u32 kCountAnyR = 1024;              // a vector of up to this many chunks has no sample, whatever r (see counts_all)
constexpr u64 kHeavyTail = 1u << 14;          // (see make_geom)

constexpr u32 kChunkQuantum = 256;            // one wavefront iteration: 64 lanes x 4 elements
constexpr u32 kMinChunk = 4 * kChunkQuantum;  // short vectors: chunks of four iterations
constexpr u32 kTargetChunks = 32768;          // short chunks, dealt round-robin to the wavefronts
constexpr u32 kMaxUnits = 4096;               // wavefronts of classify / emit (per vector)
constexpr u32 kUnitChunks = kTargetChunks / kMaxUnits;   // chunks one of them walks, at most
// In a batch of many vectors the two walking kernels are bound by the
// instructions they issue, a good part of them per wavefront rather than per
// entry: half as many wavefronts then walk twice as many chunks each. With fewer
// vectors the longest wavefront decides (the one that holds a chunk of a hot
// layer). classify / emit with 4096 and 2048 wavefronts per vector, us: eight of
// 25.6 M elements 24.8 / 21.7 and 19.8 / 17.8; five of 11.2 M, r = 5%, 30.2 / 28.7 and
// 32.5 / 33.9; four of 2^28 105 / 501 and 102 / 524. Where the wavefronts are short (chunks of
// kMinChunk) and their chunks sparse, four members are many: five of 4.3 M, r = 0.4%, 12.0 / 9.3
// and 8.5 / 6.7. Whole calls of four to six members, 2048 against 4096 wavefronts: r = 0.5 to 2%
// of 3.4 to 4.3 M 0-9% faster (one layered vector of 4.15 M 1-7% slower), of 11.2 M 2-4%, of 25.6 M
// 0-2%; r = 5% 0-5% slower from 6 M on; 2.2 M and 3.1 M (hardly more chunks than wavefronts, some of
// which walk two) 11% slower to 5% faster, 50 M 0-3% slower.
constexpr u32 kBatchUnits = 2048;
constexpr u32 kBatchMembers = 7;              // ... from this many members per launch on,
constexpr u32 kSparseMembers = 4;             // ... or this many with few candidates and
constexpr u32 kSparseChunks = 3328;           // at least this many chunks (set_units)
constexpr u32 kUnitChunksMax = kTargetChunks / kBatchUnits;
constexpr u32 kWalkThreads = 256;             // fused / classify / emit workgroups: 4 wavefronts
constexpr u32 kWalkWaves = kWalkThreads / kWave;
constexpr u32 kMaxWalkBlocks = kMaxUnits / kWalkWaves;

// The numbers of candidates kept per chunk are stored unit by unit: the UC
// chunks u, u + U, u + 2U, ... that one walking wavefront takes lie next to
// each other, so it reads them as one 32- or 64-byte piece instead of UC
// separate cache lines.
__host__ __device__ inline u32 chunk_slot(u32 s, u32 U, u32 UC) { return (s % U) * UC + s / U; }
constexpr u32 kListCap = 128;                 // short-list slots per classify workgroup
// ... of the deciding bin's list of a counted vector: it goes on where else only lists too long for LDS are, M's
// keys of two lists
constexpr u32 kLongList = 3 * kListCap;
constexpr u32 kSliceDiv = 8;                  // S holds a kSliceDiv-th as many entries as there are elements
constexpr u32 kSliceFull = 1u << 31;          // (in a chunk's count) the chunk kept more than its slice could hold

// An entry of S: the binary32 pattern, and one word with the element's place in
// its chunk (18 bits), what its sampling key says (2 bits) and, for a key inside
// the a-priori window, where in the window it lies (12 bits). The streaming
// kernel computes the key of every candidate while it waits for memory, so the
// kernels that walk S compute almost none.
constexpr u32 kPlaceBits = 18, kPlaceMask = (1u << kPlaceBits) - 1u;
constexpr u32 kKeyAbove = 0u, kKeyBelow = 1u, kKeyInside = 2u;   // ... the window [K_lo, K_hi]
constexpr u32 kKeyUnknown = 3u;               // (entries read from the vector itself)
constexpr u32 kWindowBits = 12;
constexpr int kFinThreads = 1024;
constexpr u32 kFinWaves = kFinThreads / kWave;
constexpr u32 kSlabs = kTargetChunks / (16 * kFinThreads); // 16-byte groups of quad counters per thread
// Short lists that fit are selected in LDS (500 and 2,000 entries at r = 127,786, k = 25,558;
// 4,300 and 20,500 at 2^28, r = 5%, k = 1%): of B an entry's magnitude and index, of M one word with
// where in the window its key lies and its chunk. How long M gets is known beforehand: its mean and
// eight standard deviations (staged_keys) are what a call's finalize kernel claims LDS for, as far as
// there is any: 2^28 elements, k = 1% need 21,800 at r = 5 k, 23,100 at r = 10 k, 24,200 at r = d, which
// gets seven. With room for 20,992 whatever the call / now, us: k_finalize of four such vectors, r = 5 k,
// 35 / 36, r = d 89 / 31. Two streams whose exact selections meet, each with a vector of 11.2 M 304 / 293,
// of 66 M 750 / 728: a unit taken whole has no room for the other stream's kernels.
// What B needs is not known: about r / 3,000 at that length. At r = 5 k one vector in thirty has more than
// 4,608 entries (sixteen in a launch 53, but 100 to 126 in six launches of sixteen), at r = 10 k all do
// (6,800; 109 / 109): there is no room for them beside M, and B in the claimed part costs ordinary
// calls 0.3 to 0.8 us.
constexpr u32 kStageB = 4608, kStageM = 23936;
constexpr u32 kStageRun = 8192;               // keys of a run of equal magnitudes that are selected in LDS
constexpr u32 kChunkBits = 15;
static_assert(kTargetChunks == 1u << kChunkBits && kChunkBits + kWindowBits <= 32, "an entry of M is one word");
// A selection in the lists counts strings in bins by their leading bits, kWave groups of bins.
constexpr u32 kCutB = 1024, kCutM = 1u << kWindowBits;
// The winners per chunk are added up chunk by chunk only by emit; finalize goes by quads of them.
constexpr u32 kQuad = 4;
constexpr u32 kQuads = kTargetChunks / kQuad;

constexpr u32 kErrSelect = 2u;                // a selection found no element of the requested rank
constexpr u32 kErrCount = 4u;                 // the winners did not add up to k
constexpr u32 kErrBarrier = 8u;               // a workgroup gave up waiting for the others of its grid

// The exact fallback over ALL candidates (or over the vector itself) runs on
// kWideBlocks workgroups of the finalize kernel when the vector is long enough
// to be worth it; they exchange 256-bin histograms through the workspace and
// meet at a barrier between radix passes.
constexpr u32 kWideBlocks = 256;              // one per compute unit, shared by the members of a batch
constexpr u32 kWideMinChunks = 256;
constexpr u32 kWidePasses = 24;               // 8 (magnitude, index) + 12 (key, index) + slack; the last two
                                              // `found` slots hold the two selected strings
constexpr u32 kWideSpinLimit = 1u << 20;      // polls (about a microsecond each) before giving up
constexpr u32 kWideCheckInLimit = 1u << 14;   // ... while the workgroups gather for the first time
constexpr u32 kWideGo = 1u, kWideAbort = 2u;

struct WideScratch {
    u32 arrived;                              // workgroups that reached a barrier, over all barriers
    u32 decision;                             // 0, kWideGo (all are resident) or kWideAbort
    u32 pad[62];
    u32 hist[kWidePasses][256];
    u64 found[kWidePasses][2];                // the one string left under a resolved prefix
};

// Histogram geometry chosen by the estimate kernel.
struct Bins {
    u32 t_lo;           // candidates are the entries with magnitude pattern >= t_lo
    u32 fine_hi;        // last pattern of the linear bins
    u32 shift;          // log2 of the patterns per linear bin
    u32 nfine;          // number of linear bins
};

__device__ __forceinline__ u32 bin_of(const Bins &b, u32 m)
{
    return m <= b.fine_hi ? (m - b.t_lo) >> b.shift : b.nfine;
}

__device__ __forceinline__ void bin_range(const Bins &b, u32 bin, u32 *lo, u32 *hi)
{
    if (bin < b.nfine) {
        *lo = b.t_lo + (bin << b.shift);
        const u32 h = *lo + ((1u << b.shift) - 1u);
        *hi = h < b.fine_hi ? h : b.fine_hi;
    } else {
        // the one bin above the linear ones
        *lo = b.fine_hi + 1u;
        *hi = 0x7FFFFFFFu;
    }
}

struct EncodeCtl {
    u32 err;
    u32 path;           // 0: short lists; bit 0: some quantity came from selection over all
                        // candidates; bit 2: the threshold lies in a long run of equal magnitudes
    // written by k_estimate
    Bins bins;
    u32 n_samples;
    // written by k_pick
    u32 mode;           // bit 0: the estimate missed, S holds fewer than r entries: walk the vector itself;
                        // bit 1: the deciding bin lies above the bracket, where S only holds what may be sent
    u32 bd_lo, bd_hi;   // pattern range of the deciding bin
    u32 bd_bits;        // bit width of bd_hi - bd_lo
    u64 c_def;          // entries above bd_hi
    // written by k_classify
    u32 overflow;       // a short-list region of some classify workgroup was full
    u32 overflow_m;     // ... and it was a region of the key list M
    // Written by k_finalize, by workgroup 0 while others of the grid may only just start: none
    // of these may be a word that k_finalize reads. (A workgroup that starts late must decide
    // from the same words as the ones before it whether it stays for the selection over all
    // candidates; one that stays alone waits at check-in for workgroups that have left.)
    u32 emit_dense;     // r == d and the key window missed: k_emit walks the vector itself
    u32 T, I_star;      // last member of the top-r set in (magnitude desc, index asc) order
    u64 K_star;         // last winner in (key asc, index asc) order
    u32 J_star;
    u32 n_b, n_m;
    u32 W, U, UC;       // chunks and their share-out, for the host-side statistics
    u64 count_greater, ties;
    u32 how;            // kHow...: which lists of a counted vector decided (read by tests)
    u32 n_bin;          // (counted vectors, written by k_pick_counted) entries of the bin pick found, and kCrowds
};
static_assert(offsetof(EncodeCtl, how) == 128, "where the tests look");
constexpr u32 kHowRegisters = 1u, kHowNarrowed = 2u;

// (the error word is the first word of the workspace: callers may read it there)
static_assert(offsetof(EncodeCtl, err) == 0, "the error flags lead the control block");

// Geometry and sampling window: a pure function of (d, r, k), computed on the host.
struct Geom {
    u64 d, r, k;
    u32 C;              // elements per chunk (a power of two, at least 1024)
    u32 cap;            // entries of S per chunk (C / kSliceDiv)
    u32 W;              // chunks
    u32 each, over;     // of them per wavefront of the streaming kernel; its first `over` wavefronts stream one more
    u32 spread;         // neighbouring wavefronts (as the chunks are dealt out) are of different workgroups
    u32 U;              // wavefronts of classify / emit; wavefront u walks chunks u, u + U, ...
    u32 UC;             // ... at most this many of them (W <= U * UC)
    u32 G3;             // classify / emit workgroups
    u32 L;              // sampled locations
    u32 est_vecs;       // sampled locations per thread of the estimate kernel, a power of two
    u32 nfine;          // linear histogram bins
    u32 force_dense;    // diagnostics: make the estimate keep nothing, as if the sample had misled it (of a counted
                        // vector: as if the deciding bin's row had lost its slot)
    u32 force_abort;    // diagnostics: the workgroups of the wide selection decide "abort" at check-in
    u32 force_timeout;  // diagnostics: the barriers of the wide selection give up at their first poll
    u32 force_low;      // diagnostics: the bracket's upper end is put at its lower end, as if the sample
                        // had underestimated the r-th largest magnitude: it then lies above the linear bins
    u32 take_all;       // k == r: every member is sent, keys are never looked at
    u32 all_members;    // r == d: every coordinate is a member, magnitudes are never looked at
    u32 keyed;          // the streaming kernel keys the candidates (of a short vector only if they are many)
    u32 small;          // a counted vector whose short lists finalize keeps in registers, as a rule
    u32 k_nlz;          // leading zeros of K_hi - K_lo
    u32 stage_m;        // keys in the window that finalize has room for in LDS
    u64 K_lo, K_hi;     // key window
};

struct EncodeLayout {
    u64 ctl, wide, zero_bytes, partials, group_sums;
    u64 samples, seg, win_cnt, bd_cnt, quad_win, quad_base, blk_lists, blk_bmin, blk_bmax;
    u64 m_ent, b_ent;
    u64 dm_key, dm_idx, db_key, db_idx;
    u64 s_ent;
    u64 total;
};

// Room for the members whose key lies in the window, `mean` of them on average: with eight
// standard deviations on top, as far as LDS goes.
static u32 staged_keys(long double mean)
{
    const long double room = mean + 8.0L * sqrtl(mean) + 64.0L;
    return room < (long double)kStageM ? ((u32)room + 63u) / 64u * 64u : kStageM;
}

static Geom make_geom(u64 d, u64 r, u64 k)
{
    Geom g{};
    g.d = d; g.r = r; g.k = k;
    u64 per = (d + kTargetChunks - 1) / kTargetChunks;
    per = (per + kChunkQuantum - 1) / kChunkQuantum * kChunkQuantum;
    if (per < kMinChunk) per = kMinChunk;
    // A power of two: the bare streaming add over chunks of 1024, 2048, 4096, 8192
    // elements runs at 6.1, 6.0, 6.0, 5.8 TB/s (two rows in flight, 66 M to 2^28
    // elements), over 1280, 2304, 3328, 4352 at 5.4, 5.7, 5.9, 5.7.
    {
        u64 pow2 = kMinChunk;
        while (pow2 < per) pow2 *= 2;
        per = pow2;
    }
    g.C = (u32)per;
    g.cap = g.C / kSliceDiv;
    g.W = (u32)((d + per - 1) / per);
    g.U = g.W < kMaxUnits ? g.W : kMaxUnits;
    g.UC = kUnitChunks;
    g.G3 = (g.U + kWalkWaves - 1) / kWalkWaves;       // (the layout is sized for this many)
    // (Vectors that are counted have no sample, see counts_all.)
    // A wide bracket is enough for a short vector, whose few candidates cost the walking
    // kernels nothing, and the estimate's one workgroup is a good part of its time: 4-6
    // instead of 10 us with a quarter of the samples. With 80 samples in the top r the
    // bracket's upper end is the largest sample or two, and a heavy-tailed vector's deciding
    // bin holds r / 35 entries; from kHeavyTail on that costs finalize more than twice the
    // samples cost (as long as those are few: they cost every member of a batch). One call,
    // us, 80 / 160 / 320 samples, r = 1%: Student-t values 48.8 / 44.1 / 45.9 at 2^21 elements,
    // 63.5 / 54.5 / 55.5 at 3.5 M; values spread evenly over three decades 44.3 / 44.4 / 45.6 at
    // 2^21; sixteen layered vectors of 2 M, r = 5,046 134 / 155.
    u64 want = kSampleLoc;
    if (d < kShortVector) {
        want = kEstThreads;
        while (want < kSampleLoc && want * 4 * r < 80 * d) want *= 2;
        if (r >= kHeavyTail && want <= kSampleLoc / 4 && want * 4 * r < 160 * d) want *= 2;
    }
    g.L = (u32)want;
    g.est_vecs = (u32)want / kEstThreads;
    // Every workgroup of the streaming kernel stores its whole histogram: few
    // bins when r is small (the list B of the deciding bin then holds a few
    // hundred entries anyway), more when r is large.
    g.nfine = 256;
    while (g.nfine < kMaxFineBins && (u64)g.nfine * 256 < r) g.nfine *= 2;
    g.take_all = (k == r) ? 1u : 0u;
    g.all_members = (r == d) ? 1u : 0u;
    // The number of members with key below x * 2^64 is Binomial(r, x). The
    // window keeps 7 standard deviations plus a constant (for small k, where
    // the normal approximation is poor) on both sides of k; a miss is still
    // resolved exactly, only slowly.
    const long double two64 = 18446744073709551616.0L;
    const long double kk = (long double)k, rr = (long double)r;
    const long double slack = 7.0L * sqrtl(kk * (1.0L - kk / rr)) + 30.0L;
    const long double lo = (kk - slack) / rr, hi = (kk + slack) / rr;
    g.K_lo = lo <= 0.0L ? 0ull : (u64)(lo * two64);
    g.K_hi = hi >= 1.0L ? ~0ull : (u64)(hi * two64);
    if (g.K_hi < g.K_lo) g.K_hi = g.K_lo;
    const u64 width = g.K_hi - g.K_lo;
    g.k_nlz = width ? (u32)__builtin_clzll(width) : 63u;
    g.stage_m = g.take_all ? 0u : staged_keys((fminl(hi, 1.0L) - fmaxl(lo, 0.0L)) * rr);
    return g;
}

// the walking kernels' share-out for a launch that serves nb vectors (see kBatchUnits)
static void set_units(Geom &g, unsigned nb)
{
    const bool sparse = g.C == kMinChunk && g.W >= kSparseChunks && g.r * 32 <= g.d;
    const bool batch = nb >= kBatchMembers || (nb >= kSparseMembers && sparse);
    const u32 units = batch ? kBatchUnits : kMaxUnits;
    g.U = g.W < units ? g.W : units;
    g.UC = batch ? kUnitChunksMax : kUnitChunks;
    g.G3 = (g.U + kWalkWaves - 1) / kWalkWaves;
}

// The sample of a launch of nb vectors. One vector of up to kAloneElements elements, of which the top set is a small
// part, is sampled as a shorter one is: 160 samples in its top r bound the bracket well enough, and the estimate's one
// workgroup holds the whole call up. us, 65,536 samples / 160 in the top r: Student-t values, 4.3 M elements, r = 1%, 52.2 /
// 47.5, 8 M 59.9 / 55.3, 11.2 M 66.0 / 62.0; touched rows 61.2 / 58.0, 68.7 / 66.4, 77.5 / 75.2; layers 53.9 / 53.8, 58.7 / 57.1, 66.6 / 65.7; r = k
// of 11.2 M 65.1 / 62.7; uniform and nearly equal values, signs and layers of like magnitudes 4-17% faster too, but eight levels per
// unit, r = 3%, where the wider bracket reaches one level more, 121 / 136 at 11.2 M. Not longer ones (25.6 M touched rows, r = 1%, 102.4 / 103.9), nor larger top sets (layers of 11.2 M, r = 5%,
// 77.2 / 80.8), nor batches (four of 11.2 M 139.8 / 142.5, two of 5 M 66.0 / 66.5).
constexpr u64 kAloneElements = 1u << 24, kAloneShare = 32;
static void set_samples(Geom &g, unsigned nb)
{
    if (nb != 1u || g.d < kShortVector || g.d > kAloneElements || g.r * kAloneShare >= g.d) return;
    u64 want = 2 * kEstThreads;
    while (want < kSampleLoc && want * 4 * g.r < 160 * g.d) want *= 2;
    g.L = (u32)want;
    g.est_vecs = (u32)want / kEstThreads;
}

static EncodeLayout make_layout(const Geom &g)
{
    EncodeLayout L{};
    u64 o = 0;
    auto take = [&](u64 bytes) { u64 at = o; o = align_up(o + bytes, 256); return at; };
    L.ctl = take(sizeof(EncodeCtl));
    L.wide = take(sizeof(WideScratch));
    L.zero_bytes = o;                       // cleared at the start of every call
    L.partials = take((u64)kMaxFusedBlocks * kMaxBins * 4);
    L.group_sums = take((u64)kMaxFusedBlocks * kMaxGroups * 4);
    L.samples = take((u64)kSampleLoc * 8);
    L.seg = take((u64)kTargetChunks * 8);            // fixed size: its offset depends on nothing
    L.win_cnt = take((u64)kTargetChunks * 4);
    L.bd_cnt = take((u64)kTargetChunks * 4);
    L.quad_win = take((u64)kQuads * 4);
    L.quad_base = take((u64)kQuads * 4);
    L.blk_lists = take((u64)g.G3 * 8);
    L.blk_bmin = take((u64)g.G3 * 4);
    L.blk_bmax = take((u64)g.G3 * 4);
    const u64 slots = (u64)g.G3 * kListCap;
    L.m_ent = take(slots * 8);
    L.b_ent = take(slots * 8);
    static_assert(kListCap * 8 % 256 == 0 && kLongList <= 3 * kListCap, "B goes on without a gap");
    L.dm_key = take(2 * slots * 8);
    L.dm_idx = take(2 * slots * 4);
    L.db_key = take(slots * 8);
    L.db_idx = take(slots * 4);
    L.s_ent = take((u64)g.W * g.cap * 8);
    L.total = o;
    return L;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
// the same four floats at any address a float may have: the memory instructions of 16
// bytes only ask for 4-byte alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ u32 mag_of(u32 bits) { return bits & 0x7FFFFFFFu; }
__device__ __forceinline__ u32 popc64(u64 m) { return (u32)__popcll((unsigned long long)m); }

// ---------------------------------------------------------------------------
// workgroup-wide sums of one value per thread (thread order); the second
// level is a wavefront scan, not a serial loop: LDS round trips are slow
// ---------------------------------------------------------------------------
// exclusive prefix of v over the workgroup; the grand total is left in lds[waves]
__device__ __forceinline__ u32 block_exclusive_sum(u32 v, u32 *lds /* >= waves + 1 words */)
{
    const u32 lane = lane_id(), wave = threadIdx.x / kWave, nw = blockDim.x / kWave;
    const u32 inc = wave_inclusive_sum(v);
    if (lane == kWave - 1) lds[wave] = inc;
    lds_barrier();
    if (wave == 0) {
        const u32 x = lane < nw ? lds[lane] : 0u;
        const u32 xi = wave_inclusive_sum(x);
        if (lane < nw) lds[lane] = xi - x;
        if (lane == nw - 1) lds[nw] = xi;
    }
    lds_barrier();
    const u32 res = lds[wave] + inc - v;
    lds_barrier();
    return res;
}

// sum of v over the workgroup, in every thread (the sum must fit 32 bits)
__device__ __forceinline__ u32 block_sum(u32 v, u32 *lds /* >= waves words */)
{
    const u32 nw = blockDim.x / kWave;
    v = wave_sum(v);
    if (lane_id() == 0) lds[threadIdx.x / kWave] = v;
    lds_barrier();
    const u32 total = wave_sum(lane_id() < nw ? lds[lane_id()] : 0u);
    lds_barrier();
    return total;
}

// ---------------------------------------------------------------------------
// sample: magnitudes of a = g + m at g.L locations, one per stratum of the
// vector, at a hashed offset inside the stratum, four consecutive elements
// each. Also clears what later kernels accumulate into.
// ---------------------------------------------------------------------------
__device__ __forceinline__ u64 stratum_start(const Geom &g, u32 j)
{
    // strata of (almost) equal length, 64 elements or more: vectors of up to kCountAnyR chunks are counted
    static_assert((u64)kCountAnyR * kMinChunk >= 64u * (u64)kSampleLoc, "strata of 64 elements");
    return (g.d * (u64)j) >> (31 - __clz((int)g.L));        // (g.L is a power of two; d * j <= 2^46)
}

// A first element inside stratum [start, start + len). The offset depends on the
// stratum AND on (seed, step): a vector whose layout happens to mislead one set of offsets (a
// period close to the stratum length) does not mislead the next step's or another worker's.
// Which elements are sampled never changes the result, only the path.
__device__ __forceinline__ u64 sample_place(u32 j, u64 start, u64 len, const PhiloxSeed &seed)
{
    u32 hsh = (j + 1u) * 0x9E3779B1u;
    hsh ^= seed.seed_lo * 0x85EBCA77u + seed.step_lo * 0xC2B2AE3Du +
           (seed.seed_hi ^ seed.step_hi) * 0x27D4EB2Fu;
    hsh ^= hsh >> 15; hsh *= 0x85EBCA77u; hsh ^= hsh >> 13;
    hsh *= 0xC2B2AE3Du; hsh ^= hsh >> 16;
    // offset in [0, len - 4], scaled from the hash instead of a remainder
    return start + (u64)(((u64)hsh * (u64)(len - 3)) >> 32);
}

// the samples of location j, two to a word
__device__ __forceinline__ uint2 take_samples(const float *__restrict__ grad, const float *__restrict__ residual,
                                              const Geom &g, const PhiloxSeed &seed, u32 j)
{
    const u64 start = stratum_start(g, j), end = stratum_start(g, j + 1);
    // One 16-byte load per array, at whatever alignment the pointers have (word by word, a vector of
    // 11.2 M elements off 16 bytes took 6.8 us, now 4.8). The four elements may start up to
    // three before the stratum: it stays a spread-out sample.
    const u64 p = sample_place(j, start, end - start, seed) & ~3ull;
    const f32x4 gv = *reinterpret_cast<const f32x4u *>(grad + p);
    const f32x4 mv = *reinterpret_cast<const f32x4u *>(residual + p);
    u32 v[4];
#pragma unroll
    for (u32 e = 0; e < 4; ++e) v[e] = mag_of(__float_as_uint(gv[e] + mv[e])) >> kSampleShift;
    return make_uint2(v[0] | v[1] << 16, v[2] | v[3] << 16);
}

__device__ __forceinline__ void
sample_body(const float *__restrict__ grad, const float *__restrict__ residual, Geom g,
         PhiloxSeed seed, u32 *__restrict__ zero_base, u32 zero_words, u32 *__restrict__ samples)
{
    const u32 j = blockIdx.x * kSampleThreads + threadIdx.x;
    for (u32 i = j; i < zero_words; i += gridDim.x * kSampleThreads) zero_base[i] = 0u;
    if (j >= g.L) return;
    reinterpret_cast<uint2 *>(samples)[j] = take_samples(grad, residual, g, seed, j);
}

// ---------------------------------------------------------------------------
// estimate: order statistics of the sample -> histogram geometry.
// With n samples and p = r/d, the number of samples among the true top r is
// about Binomial(n, p); clusters of four that rise and fall together double
// the standard deviation at worst. t_lo is the lower edge of the 12-bit
// pattern bucket that holds the sample of rank np + 4 sd + 8 (so that at
// least r entries lie at or above t_lo), t_hi the upper edge of the bucket
// that holds the sample of rank np - 4 sd - 8 (fewer than r entries lie
// above it). Four of these doubled deviations are six to eight true ones; a
// miss (at worst 3 in 100,000 per side, were the clusters to rise and fall
// entirely together) costs 0.14 ms above the bracket and 0.35 ms below it at
// 25.6 M elements, 0.4 and 3.2 ms at 2^28, while six of them kept a
// fifth more candidates on every call (eight vectors of 25.6 M: classify 24.0
// instead of 17.8 us, emit 20.7 instead of 17.0).
// ---------------------------------------------------------------------------
// One wavefront: walking 4096 buckets (in LDS) downwards from the bucket
// `top` (nothing lies above it), 256 buckets at a time, find for each of
// NRANKS ranks the bucket b with #(buckets above b) < need <= #(buckets >= b).
// Stores b and the population above it; stores nothing for a rank that all
// buckets together do not reach. The samples that matter sit in the few
// buckets under the largest one: one or two steps instead of a walk over all.
template <int NRANKS>
__device__ __forceinline__ void wave_pick_from_top(const u32 *hist, u32 top, const u32 (&need)[NRANKS],
                                                   u32 *out_bin, u32 *out_before)
{
    const u32 lane = lane_id();
    u32 above = 0;
    bool pending[NRANKS];
#pragma unroll
    for (int k = 0; k < NRANKS; ++k) pending[k] = true;
    for (int hi = (int)(top | 255u); hi >= 0; hi -= 256) {
        u32 c[4];
        u32 mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) { c[q] = hist[hi - 4 * (int)lane - q]; mine += c[q]; }
        const u32 inc = wave_inclusive_sum(mine);
        const u32 before = above + inc - mine;
        bool any = false;
#pragma unroll
        for (int k = 0; k < NRANKS; ++k) {
            const bool here = pending[k] && before < need[k] && need[k] <= before + mine;
            if (here) {
                u32 run = before;
                bool done = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (!done && run + c[q] >= need[k]) {
                        out_bin[k] = (u32)(hi - 4 * (int)lane - q);
                        out_before[k] = run;
                        done = true;
                    }
                    run += c[q];
                }
            }
            if (__ballot(here) != 0ull) pending[k] = false;
            any = any || pending[k];
        }
        if (!any) break;
        above += (u32)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    }
}

template <u32 kVecs>      // locations (8 bytes, four samples) per thread
__device__ __forceinline__ void
estimate_body(const u32 *__restrict__ samples, Geom g, EncodeCtl *ctl)
{
    // One compute unit looks at 65,536 samples: the lines it fetches and the work per
    // sample are what this kernel costs, so the two passes over them are a handful of
    // instructions per location. A sample has 15 bits.
    __shared__ u32 h_max[4096];                           // buckets of the per-thread maxima
    __shared__ u32 h[4096];                               // buckets of the samples that matter
    __shared__ u32 bin_s[3], before_s[3], top_s;
    const u32 tid = threadIdx.x;
    const uint2 *s2 = reinterpret_cast<const uint2 *>(samples);
    uint2 v[kVecs];
#pragma unroll
    for (u32 q = 0; q < kVecs; ++q) v[q] = s2[q * kEstThreads + tid];
    for (u32 b = tid; b < 4096u; b += kEstThreads) { h[b] = 0u; h_max[b] = 0u; }
    if (tid < 3u) { bin_s[tid] = 0u; before_s[tid] = 0u; }
    if (tid == 0) top_s = 0u;
    auto smax = [](int a, int b) { return a > b ? a : b; };
    auto low = [](u32 w) { return (int)(short)(w & 0xFFFFu); };
    auto high = [](u32 w) { return (int)w >> 16; };
    int gmax[kVecs];                                      // largest of each location
    int tmax = 0;
#pragma unroll
    for (u32 q = 0; q < kVecs; ++q) {
        gmax[q] = smax(smax(low(v[q].x), high(v[q].x)), smax(low(v[q].y), high(v[q].y)));
        tmax = smax(tmax, gmax[q]);
    }
    const u32 n = 4u * g.L;
    lds_barrier();                                        // orders the clearing of the histograms

    const float p = (float)((double)g.r / (double)g.d);
    const float np = (float)n * p;
    const float sd = 2.0f * sqrtf(np * (1.0f - p));
    const float lo_rank = ceilf(np + 4.0f * sd + 8.0f), hi_rank = floorf(np - 4.0f * sd - 8.0f);
    const bool lo_all = lo_rank > (float)n;       // too few samples below the top: keep everything
    const u32 s_lo = lo_all ? n : (u32)lo_rank;
    const u32 s_hi = hi_rank < 1.0f ? 1u : (u32)hi_rank;

    // Only the top s_lo samples matter. At most s_lo - 1 threads hold a sample
    // above the s_lo-th largest one, so the s_lo-th largest of the per-thread
    // maxima is not above it: buckets below that maximum's bucket need no count.
    // (the bucket of the largest sample of all is where every walk starts)
    {
        const u32 wmax = wave_max_dpp((u32)tmax >> kBucketShift);
        if (lane_id() == 0 && wmax) atomicMax(&top_s, wmax);
    }
    // (Where the top holds more samples than there are threads, the same with the maxima of the
    // locations: every sample counted, five vectors of 11.2 M elements, r = 5%, took 11.4 us, now 9.3)
    u32 cut_bucket = 0;
    if (s_lo < g.L) {
        if (s_lo < kEstThreads) {
            atomicAdd(&h_max[(u32)tmax >> kBucketShift], 1u);
        } else {
#pragma unroll
            for (u32 q = 0; q < kVecs; ++q) atomicAdd(&h_max[(u32)gmax[q] >> kBucketShift], 1u);
        }
        lds_barrier();
        if (tid < kWave) {
            const u32 want_cut[1] = {s_lo};
            wave_pick_from_top<1>(h_max, top_s, want_cut, &bin_s[2], &before_s[2]);
        }
        lds_barrier();
        cut_bucket = bin_s[2];                     // (bucket 0 where all of them are zero)
    }
    const int cut = (int)(cut_bucket << kBucketShift);
    u32 nzero = 0;
    auto count = [&](int m) {
        if (m < cut) return;
        const u32 b = (u32)m >> kBucketShift;
        if (b == 0u) ++nzero;                     // zeros come in long runs: count them aside
        else atomicAdd(&h[b], 1u);
    };
#pragma unroll
    for (u32 q = 0; q < kVecs; ++q) {
        if (gmax[q] < cut) continue;               // nearly every location
        count(low(v[q].x)); count(high(v[q].x)); count(low(v[q].y)); count(high(v[q].y));
    }
    nzero = wave_sum(nzero);
    if (lane_id() == 0 && nzero) atomicAdd(&h[0], nzero);
    __syncthreads();
    if (tid < kWave) {
        const u32 want[2] = {s_lo, s_hi};
        wave_pick_from_top<2>(h, top_s, want, &bin_s[0], &before_s[0]);
    }
    __syncthreads();
    if (tid == 0) {
        u32 t_lo = lo_all ? 0u : (bin_s[0] << 19);
        u32 t_hi = (bin_s[1] << 19) | 0x7FFFFu;
        if (g.force_dense) t_lo = 0x7FFFFFFFu;
        if (g.force_low) t_hi = t_lo;
        if (t_hi < t_lo) t_hi = t_lo;
        u32 shift = 0;
        while (((t_hi - t_lo) >> shift) >= g.nfine) ++shift;
        const u64 top = (u64)t_lo + ((u64)g.nfine << shift) - 1ull;
        ctl->bins.t_lo = t_lo;
        ctl->bins.fine_hi = top > 0x7FFFFFFFull ? 0x7FFFFFFFu : (u32)top;
        ctl->bins.shift = shift;
        ctl->bins.nfine = g.nfine;
        ctl->n_samples = n;
    }
}

// ---------------------------------------------------------------------------
// One wavefront iteration of the streaming kernel covers 256 consecutive
// elements starting at `base`; a lane holds base + 4*lane + e (one 16-byte
// access per array). Kept entries are appended to the chunk's slice of S in index
// order.
// ---------------------------------------------------------------------------

__device__ __forceinline__ u64 elem_index(u64 base, int e) { return base + 4ull * lane_id() + (u64)e; }

// what the sampling key of element idx says, as the top 14 bits of an entry's first word
__device__ __forceinline__ u32 key_word(u32 idx, const Geom &g, const PhiloxSeed &seed)
{
    if (g.take_all) return kKeyBelow << 30;
    const u64 key = sample_key(idx, seed);
    if (key < g.K_lo) return kKeyBelow << 30;
    if (key > g.K_hi) return kKeyAbove << 30;
    return (kKeyInside << 30) | ((u32)(((key - g.K_lo) << g.k_nlz) >> (64 - kWindowBits)) << kPlaceBits);
}

// The candidates of the chunk a wavefront is streaming, in index order: they are
// gathered in a ring in LDS and leave it 64 at a time, so that the sampling keys are
// computed on full wavefronts and the slice of S is written in whole lines.
constexpr u32 kRing = 512;                    // a power of two >= 63 waiting + one row of 256
struct Ring {
    uint2 *buf;         // kRing entries owned by this wavefront: (place in the chunk, pattern)
    u32 head, pending;  // (head is reduced where it is used)
    u32 room;           // entries the chunk's slice may hold
    u32 out;            // entries of it so far (above room: it overflowed)

    __device__ __forceinline__ void append(const u32 (&bits)[4], const bool (&hit)[4], u32 place0)
    {
        const u64 b0 = __ballot(hit[0]), b1 = __ballot(hit[1]), b2 = __ballot(hit[2]),
                  b3 = __ballot(hit[3]);
        if ((b0 | b1 | b2 | b3) == 0ull) return;
        if (out > room) return;       // the slice overflowed: the chunk will be read from the vector itself
        const u64 below = lanes_below();
        const u32 at = head + pending;
        u32 p = at + popc64(b0 & below) + popc64(b1 & below) + popc64(b2 & below) + popc64(b3 & below);
#pragma unroll
        for (u32 e = 0; e < 4; ++e)
            if (hit[e]) { buf[p & (kRing - 1u)] = make_uint2(place0 + 4u * lane_id() + e, bits[e]); ++p; }
        pending += popc64(b0) + popc64(b1) + popc64(b2) + popc64(b3);
    }
    // straight to the slice, the keys left to be computed
    __device__ __forceinline__ void append_unkeyed(const u32 (&bits)[4], const bool (&hit)[4], u32 place0,
                                                   uint2 *__restrict__ my_ent)
    {
        const u64 b0 = __ballot(hit[0]), b1 = __ballot(hit[1]), b2 = __ballot(hit[2]),
                  b3 = __ballot(hit[3]);
        if ((b0 | b1 | b2 | b3) == 0ull) return;
        const u64 below = lanes_below();
        u32 p = out + popc64(b0 & below) + popc64(b1 & below) + popc64(b2 & below) + popc64(b3 & below);
#pragma unroll
        for (u32 e = 0; e < 4; ++e)
            if (hit[e]) {
                if (p < room) my_ent[p] = make_uint2((kKeyUnknown << 30) | (place0 + 4u * lane_id() + e), bits[e]);
                ++p;
            }
        out += popc64(b0) + popc64(b1) + popc64(b2) + popc64(b3);
    }
    // Up to 64 entries leave the ring. A candidate above the bracket is a certain member,
    // and one whose key lies above the window is certainly not sent: it is needed by
    // nobody and does not reach the slice (should the estimate or the window have missed,
    // finalize fills the slices again). In a layer that holds most of the top r, where nearly
    // all candidates lie above the bracket, four fifths of them go this way.
    __device__ __forceinline__ void take(u64 c0, const Geom &g, const PhiloxSeed &seed, u32 bracket_hi,
                                         uint2 *__restrict__ my_ent)
    {
        const u32 n = pending < (u32)kWave ? pending : (u32)kWave;
        wave_lds_fence();
        uint2 e = make_uint2(0u, 0u);
        bool stays = lane_id() < n;
        if (stays) {
            e = buf[(head + lane_id()) & (kRing - 1u)];
            e.x |= key_word((u32)c0 + e.x, g, seed);
            stays = mag_of(e.y) <= bracket_hi || (e.x >> 30) != kKeyAbove;
        }
        wave_lds_fence();
        const u64 mask = __ballot(stays);
        const u32 pos = out + popc64(mask & lanes_below());
        if (stays && pos < room) my_ent[pos] = e;
        head += n;
        pending -= n;
        out += popc64(mask);
    }
};

// ---------------------------------------------------------------------------
// fused: a = g + m -> residual buffer; candidates -> S and the histogram.
// Reads g and m once, writes a once: 12d bytes of HBM traffic. The grid is
// sized to what the device holds at once; wavefront v takes chunks v,
// v + #wavefronts, ... so that neighbouring wavefronts (deals_across says which those are)
// stream neighbouring 4 KB pieces of each array.
// ---------------------------------------------------------------------------
constexpr u32 kFusedThreads = 768;            // at most; a launch takes 4 to 12 wavefronts, see fused_waves
// kRows: rows of 256 elements a wavefront adds, stores and looks at together; the
// next ones are on their way meanwhile. One, but for short vectors, where a
// wavefront has a single chunk: two.
constexpr int kLongRows = 1, kShortRows = 2;
// kKeyed: the candidates are keyed, by way of a ring in LDS. A short vector's are few, as a
// rule, and a wavefront meets them at the end of its only chunk or two, where nothing hides the
// microsecond a key and the way through the ring take: they then go straight to S, and
// classify keys them, which waits for memory anyway (428,000 elements, r = 84: 6.3 instead of
// 7.1 us; 65,536, r = 13: the call 35.6 instead of 36.4). See keys_in_stream.

// kAll (r == d, the random-k operator): no magnitude decides anything. An
// element is kept when its sampling key lies at or below the upper end of the
// a-priori window (all of them when k == r as well); no histogram is made and
// the control block, which no earlier kernel has touched, is cleared here.
template <bool kAll, int kRows, bool kKeyed>
__device__ __forceinline__ void
fused_body(const float *__restrict__ grad, float *__restrict__ residual, Geom g, PhiloxSeed seed,
        EncodeCtl *__restrict__ ctl, u32 zero_words, u32 *__restrict__ partials,
        u32 *__restrict__ group_sums, uint2 *__restrict__ seg, uint2 *__restrict__ s_ent)
{
    __shared__ u32 h[kAll ? 1 : kMaxBins];
    extern __shared__ uint2 ring_s[];           // kRing entries per wavefront (and what the launch claims beyond), none if not keyed
    Bins bins{};
    u32 nbins = 0;
    if (kAll) {
        // (the control block and what follows it up to zero_words, at the workspace's start)
        if (blockIdx.x == 0)
            for (u32 i = threadIdx.x; i < zero_words; i += blockDim.x)
                reinterpret_cast<u32 *>(ctl)[i] = 0u;
    } else {
        bins = ctl->bins;
        nbins = bins.nfine + kCoarseBins;
        for (u32 b = threadIdx.x; b < nbins; b += blockDim.x) h[b] = 0u;
        __syncthreads();
    }

    const u32 n_waves = blockDim.x / kWave, wave_stride = gridDim.x * n_waves;
    u32 n_above = 0;        // this wavefront's candidates above the linear bins
    Ring ring{ring_s + threadIdx.x / kWave * kRing, 0u, 0u, 0u, 0u};
    const u32 bracket_hi = kAll ? 0x7FFFFFFFu : bins.fine_hi;
    u64 c0 = 0;             // the current chunk
    uint2 *my_ent = s_ent;
    auto keep = [&](const u32 (&bits)[4], const bool (&valid)[4], u32 place) {
        bool hit[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (kAll) {
                // (by the key's leading word: one of 2^32 candidates more, which classify leaves out)
                hit[e] = valid[e] &&
                         (g.take_all != 0u ||
                          (u32)(sample_key((u32)elem_index(c0 + place, e), seed) >> 32) <= (u32)(g.K_hi >> 32));
            } else {
                const u32 m = mag_of(bits[e]);
                hit[e] = valid[e] && m >= bins.t_lo;
                // candidates inside the bracket are counted bin by bin; the ones above it
                // (certain members, often most of the candidates and crowded in a few
                // exponents) only need their number: a popcount instead of LDS additions
                const bool fine = hit[e] && m <= bins.fine_hi;
                if (fine) atomicAdd(&h[(m - bins.t_lo) >> bins.shift], 1u);
                n_above += popc64(__ballot(hit[e] && !fine));
            }
        }
        if (kKeyed) {
            ring.append(bits, hit, place);
            while (ring.pending >= (u32)kWave) ring.take(c0, g, seed, bracket_hi, my_ent);
        } else {
            ring.append_unkeyed(bits, hit, place, my_ent);
        }
    };
    // This wavefront's part of S: the chunks it streams (w_first, w_first + wave_stride, ...) times
    // g.cap entries. A chunk may take what the ones before it have left and half of what the
    // ones after it are due (an ordinary chunk needs less than half): a layer that holds much of
    // the top r is dealt out over many wavefronts, a chunk or two each. With a slice of fixed size per
    // chunk a tenth of the chunks of layered vectors overflowed and were read again by
    // both walking kernels: classify / emit of five vectors of 11.2 M elements, r = 5%, 29.1 / 27.5
    // us, with shared room 16.1 / 17.6; of four of 66 M with a twentieth of the rows
    // touched 40.0 / 33.0 and 21.0 / 22.1. The stream pays for it, as it stores those entries: the five 115.7 ->
    // 118.2, the four 530 -> 541; 1% (53.9 -> 54.5 for one of 25.6 M) where hardly a chunk overflowed.
    const u32 w_first = g.spread != 0u ? threadIdx.x / kWave * gridDim.x + blockIdx.x
                                       : blockIdx.x * n_waves + threadIdx.x / kWave;
    u32 later, at;          // chunks still to come; where in S the next slice starts
    {
        later = g.each + (w_first < g.over ? 1u : 0u);
        at = (w_first * g.each + (w_first < g.over ? w_first : g.over)) * g.cap;
    }
    const u32 s_end = at + later * g.cap;
    auto open_chunk = [&](u32 w) {
        c0 = (u64)w * g.C;
        --later;
        my_ent = s_ent + at;
        ring.room = s_end - at - later * (g.cap / 2u);
        ring.out = 0u;
    };
    auto close_chunk = [&](u32 w) {
        if (kKeyed && ring.pending != 0u) ring.take(c0, g, seed, bracket_hi, my_ent);
        const bool full = ring.out > ring.room;
        if (lane_id() == 0) seg[chunk_slot(w, g.U, g.UC)] = make_uint2(ring.out | (full ? kSliceFull : 0u), at);
        if (!full) at += ring.out;
    };
    const bool all_valid[4] = {true, true, true, true};
    // Groups of kRows rows. Every element is read once and written once: both
    // the loads and the store carry the streaming hint. (Measured: the hint on the
    // residual's load AND store together shortens the kernel by 15%; either one
    // alone changes nothing.)
    constexpr u32 kGroup = kRows * kChunkQuantum;
    f32x4 gv[kRows], mv[kRows];
    auto load = [&](u64 base) {
        const f32x4u *gp = reinterpret_cast<const f32x4u *>(grad + base) + lane_id();
        const f32x4u *mp = reinterpret_cast<const f32x4u *>(residual + base) + lane_id();
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            gv[q] = __builtin_nontemporal_load(gp + q * kWave);
            mv[q] = __builtin_nontemporal_load(mp + q * kWave);
        }
    };
    // the sum of the group at `base`, which has been loaded, stored and handed on as patterns
    auto add = [&](u64 base, u32 (&bits)[kRows][4]) {
        f32x4u *mp = reinterpret_cast<f32x4u *>(residual + base) + lane_id();
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            const f32x4 a = gv[q] + mv[q];
            __builtin_nontemporal_store((f32x4u)a, mp + q * kWave);
            bits[q][0] = __float_as_uint(a.x); bits[q][1] = __float_as_uint(a.y);
            bits[q][2] = __float_as_uint(a.z); bits[q][3] = __float_as_uint(a.w);
        }
    };
    // The chunks that are whole: the next group is on its way while this one's
    // candidates are looked for.
    const u32 w_full = (u32)(g.d / g.C);
    u32 w = w_first;
    if (w < w_full) {
        open_chunk(w);
        u64 base = c0;
        load(base);
        for (;;) {
            u32 bits[kRows][4];
            add(base, bits);
            const u32 place = (u32)(base - c0);
            const bool last = place + kGroup >= g.C;
            const u32 w_next = last ? w + wave_stride : w;
            const u64 next = last ? (u64)w_next * g.C : base + kGroup;
            const bool more = w_next < w_full;
            if (more) load(next);
#pragma unroll
            for (int u = 0; u < kRows; ++u) keep(bits[u], all_valid, place + u * kChunkQuantum);
            if (last) {
                close_chunk(w);
                if (more) open_chunk(w_next);
            }
            if (!more) break;
            w = w_next;
            base = next;
        }
        while (w < w_full) w += wave_stride;
    }
    // The ragged end of the vector: one chunk, of some wavefront. It may be nearly C elements
    // long: its groups go the same way (read row by row without the next one on its way, it
    // held a call of 2^30 - 1 elements up by 3%, one of 3 * 2^30 - 1 by 6%).
    if (w == w_full && w < g.W) {
        open_chunk(w);
        u64 base = c0;
        bool more = base + kGroup <= g.d;
        if (more) load(base);
        while (more) {
            u32 bits[kRows][4];
            add(base, bits);
            const u32 place = (u32)(base - c0);
            base += kGroup;
            more = base + kGroup <= g.d;
            if (more) load(base);
#pragma unroll
            for (int u = 0; u < kRows; ++u) keep(bits[u], all_valid, place + u * kChunkQuantum);
        }
        for (; base < g.d; base += kChunkQuantum) {
            u32 bits[4];
            bool valid[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u64 i = elem_index(base, e);
                valid[e] = i < g.d;
                bits[e] = 0u;
                if (valid[e]) {
                    const float a = grad[i] + residual[i];
                    residual[i] = a;
                    bits[e] = __float_as_uint(a);
                }
            }
            keep(bits, valid, (u32)(base - c0));
        }
        close_chunk(w);
    }
    if (kAll) return;
    if (lane_id() == 0 && n_above != 0u) atomicAdd(&h[bins.nfine], n_above);
    __syncthreads();
    // The workgroup's histogram goes out as one dense row with plain stores:
    // device-wide atomics here, however few, slow the whole stream down. With
    // it go the sums over groups of kCoarseSpan bins: the pick kernel first adds
    // up those (a sixty-fourth of the data), finds the group that holds the
    // r-th largest magnitude and then only needs that group's bins of every row.
    u32 *row = partials + (u64)blockIdx.x * nbins;
    for (u32 b = threadIdx.x; b < nbins; b += blockDim.x) row[b] = h[b];
    const u32 ngroups = (nbins + kCoarseSpan - 1) / kCoarseSpan;
    for (u32 c = threadIdx.x / kWave; c < ngroups; c += n_waves) {
        const u32 b = c * kCoarseSpan + lane_id();
        const u32 sum = wave_sum(b < nbins ? h[b] : 0u);
        if (lane_id() == 0) group_sums[(u64)blockIdx.x * kMaxGroups + c] = sum;
    }
}

// ---------------------------------------------------------------------------
// The candidates as later kernels see them: chunk s holds count(s) entries
// (index, binary32 pattern), in index order. Normally that is the slice of S
// the fused kernel filled; in dense mode it is the chunk of a itself.
// ---------------------------------------------------------------------------
struct Candidates {
    const uint2 *__restrict__ seg;          // per chunk: entries in its slice of S (kSliceFull: too many), the slice's start
    const uint2 *__restrict__ s_ent;
    const float *__restrict__ a;
    u64 d;
    u32 C, U, UC;
    bool dense;         // every chunk is read from the vector (the estimate kept too little; r == d
                        // and the key window missed)

    __device__ __forceinline__ u32 length(u32 s) const
    {
        const u64 c0 = (u64)s * C;
        return (u32)(c0 + C < d ? C : d - c0);
    }
    // entries of chunk s, where in S they start, and whether they are the chunk's elements themselves:
    // a chunk that kept more than its slice holds is read from the vector (all
    // its elements then count as entries; what lies below the candidates'
    // lower bound is below every threshold the later kernels compare with)
    __device__ __forceinline__ u32 count(u32 s, u32 *start, bool *from_vector) const
    {
        const uint2 kept = dense ? make_uint2(kSliceFull, 0u) : seg[chunk_slot(s, U, UC)];
        *start = kept.y;
        *from_vector = (kept.x & kSliceFull) != 0u;
        return *from_vector ? length(s) : kept.x;
    }
    // entry j of chunk s, whose slice starts at `start`
    // (key: what the streaming kernel left of the sampling key, kKeyUnknown << 30 if nothing)
    __device__ __forceinline__ void entry(u32 s, u32 start, u32 j, bool from_vector, u32 *idx, u32 *bits, u32 *key) const
    {
        if (!from_vector) {
            const uint2 e = s_ent[start + j];
            *idx = s * C + (e.x & kPlaceMask);
            *bits = e.y;
            *key = e.x;
        } else {
            const u64 at = (u64)s * C + j;
            *idx = (u32)at;
            *bits = __float_as_uint(a[at]);
            *key = kKeyUnknown << 30;
        }
    }
};

// One wavefront walks chunks u, u + U, u + 2U, ... as one flat sequence: lane
// i first fetches the size of the i-th of them (there are at most
// kUnitChunksMax), a prefix sum turns flat positions into (chunk, entry) pairs,
// and every iteration of the walk hands 64 consecutive positions to the 64
// lanes; the entries of one chunk stay in index order. f(valid, i, index,
// pattern, first, p0) is called by all lanes in every iteration, so it may use
// wave-wide operations; (index, pattern) is the lane's entry, i the ordinal of
// its chunk among the wavefront's chunks, first the flat position of the
// chunk's first entry and p0 the flat position lane 0 holds.
// The same walk serves the slow exact paths of the finalize kernel, where a
// wavefront takes kWave consecutive chunks at a time (kChunks = kWave,
// stride 1).
template <u32 kChunks>
struct ChunkWalk {
    u32 u, stride, excl, inc, total;
    u32 shift;              // (in the chunk's lane) what turns flat positions into places in S
    u64 from_vector;        // bit i: the i-th chunk is read from the vector itself
    static constexpr u32 kRowQueueSize = 512; // a power of two >= 63 entries waiting + one row of 256

    // chunks first, first + step, ..., at most kChunks of them and only those below n_chunks
    __device__ __forceinline__ ChunkWalk(const Candidates &cand, u32 first, u32 step, u32 n_chunks)
    {
        static_assert(kChunks <= kWave && (kChunks & (kChunks - 1)) == 0, "one lane per chunk");
        const u32 lane = lane_id();
        u = first;
        stride = step;
        const u64 s = (u64)first + (u64)lane * step;
        bool fv = false;
        u32 start = 0u;
        u32 cnt = (lane < kChunks && s < n_chunks) ? cand.count((u32)s, &start, &fv) : 0u;
        from_vector = __ballot(fv);
        if (fv) cnt = 0u;           // not part of the flat sequence: see for_each_vector_row
        inc = wave_inclusive_sum(cnt);
        excl = inc - cnt;
        shift = start - excl;
        total = __shfl(inc, kWave - 1, kWave);
    }

    // flat position p -> ordinal of its chunk and the flat position of that chunk's first entry
    __device__ __forceinline__ void locate(u32 p, u32 *ordinal, u32 *first) const
    {
        // number of chunks that end at or before position p = ordinal of p's chunk
        u32 c = 0;
#pragma unroll
        for (u32 step = kChunks / 2; step > 0; step >>= 1) {
            const u32 end_of = __shfl(inc, c + step - 1, kWave);
            if (end_of <= p) c += step;
        }
        c &= kChunks - 1;
        *ordinal = c;
        *first = __shfl(excl, c, kWave);
    }

    // f(valid, i, index, pattern, key word, first, p0), see above; the entries of four
    // iterations are fetched together while that many are left
    template <class F>
    __device__ __forceinline__ void for_each(const Candidates &cand, F &&f) const
    {
        const u32 lane = lane_id();
        constexpr u32 kAhead = 4;
        u32 p0 = 0;
        for (; p0 + kAhead * kWave <= total; p0 += kAhead * kWave) {
            u32 c[kAhead], first[kAhead], idx[kAhead], bits[kAhead], key[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 p = p0 + q * kWave + lane;
                locate(p, &c[q], &first[q]);
                cand.entry(u + c[q] * stride, __shfl(shift, c[q], kWave), p, false, &idx[q], &bits[q], &key[q]);
            }
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) f(true, c[q], idx[q], bits[q], key[q], first[q], p0 + q * kWave);
        }
        for (; p0 < total; p0 += kWave) {
            const u32 p = p0 + lane;
            u32 c, first, idx = 0, bits = 0, key = 0;
            locate(p, &c, &first);
            const u32 to_s = __shfl(shift, c, kWave);
            if (p < total) cand.entry(u + c * stride, to_s, p, false, &idx, &bits, &key);
            f(p < total, c, idx, bits, key, first, p0);
        }
    }

    // Cursor over the rows of 256 elements of the wavefront's chunks that are read
    // from the vector itself (they kept more candidates than their slice of S
    // holds, or the whole vector is walked): lane l of a row holds the four
    // elements idx0 .. idx0 + 3, idx0 = row start + 4 l, loaded with one 16-byte
    // access where the vector's alignment allows.
    struct RowCursor {
        u64 rest;           // chunks still to come
        u64 c0;             // first element of the current chunk
        u32 i, len, r0;     // its ordinal among the wavefront's chunks, its length, the next row
        bool open;
    };
    __device__ __forceinline__ RowCursor rows() const { return RowCursor{from_vector, 0ull, 0u, 0u, 0u, false}; }
    // moves to the next chunk if the current one is used up; false when no chunk is left
    __device__ __forceinline__ bool next_chunk(const Candidates &cand, RowCursor &rc) const
    {
        if (rc.rest == 0ull) return false;
        rc.i = (u32)__ffsll((unsigned long long)rc.rest) - 1u;
        rc.rest &= rc.rest - 1ull;
        const u32 s = u + rc.i * stride;
        rc.c0 = (u64)s * cand.C;
        rc.len = cand.length(s);
        rc.r0 = 0;
        rc.open = true;
        return true;
    }
    // loads the current chunk's next row (the chunk must have one left)
    __device__ __forceinline__ void load_row(const Candidates &cand, RowCursor &rc, u32 *idx0,
                                             u32 (&bits)[4], bool (&valid)[4]) const
    {
        const u32 off = rc.r0 + 4u * lane_id();
        if (rc.r0 + kChunkQuantum <= rc.len) {
            const f32x4 v = *reinterpret_cast<const f32x4u *>(cand.a + rc.c0 + off);
            bits[0] = __float_as_uint(v.x); bits[1] = __float_as_uint(v.y);
            bits[2] = __float_as_uint(v.z); bits[3] = __float_as_uint(v.w);
#pragma unroll
            for (u32 e = 0; e < 4; ++e) valid[e] = true;
        } else {
#pragma unroll
            for (u32 e = 0; e < 4; ++e) {
                valid[e] = off + e < rc.len;
                bits[e] = valid[e] ? __float_as_uint(cand.a[rc.c0 + off + e]) : 0u;
            }
        }
        *idx0 = (u32)rc.c0 + off;
        rc.r0 += kChunkQuantum;
        if (rc.r0 >= rc.len) rc.open = false;
    }

    // g(i, idx0, patterns, valid) for every such row, all lanes together, rows of one
    // chunk in index order (rare paths: one row in flight)
    template <class G>
    __device__ __forceinline__ void for_each_vector_row(const Candidates &cand, G &&g) const
    {
        RowCursor rc = rows();
        for (;;) {
            if (!rc.open && !next_chunk(cand, rc)) break;
            u32 idx0, bits[4];
            bool valid[4];
            load_row(cand, rc, &idx0, bits, valid);
            g(rc.i, idx0, bits, valid);
        }
    }

    // The same chunks with the elements that keep(pattern) lets through gathered
    // first, so that the work per entry is done on full wavefronts: the survivors are
    // appended in index order to a ring in LDS (buf: kRowQueueSize entries owned by this
    // wavefront) and taken from its front 64 at a time; what is left of a chunk is taken
    // before the next chunk starts, so the ring only ever holds one chunk's entries.
    // f(valid, i, index, pattern) is called by all lanes together (from one place: its
    // code exists once), entries of one chunk in index order. Four rows of a chunk are
    // fetched together (one at a time, the trips to memory of the few wavefronts that
    // hold such a chunk were half of the walking kernels' time in a layered vector).
    template <class Keep, class F>
    __device__ __forceinline__ void for_each_vector_entry(const Candidates &cand, uint2 *buf,
                                                          Keep &&keep, F &&f) const
    {
        constexpr u32 kRows = 4;
        typedef u32 u32x16 __attribute__((ext_vector_type(4 * kRows)));
        const u32 lane = lane_id();
        const u64 below = lanes_below();
        u32 head = 0, pending = 0;
        for (u64 rest = from_vector; rest != 0ull; rest &= rest - 1ull) {
            const u32 i = (u32)__ffsll((unsigned long long)rest) - 1u;
            const u32 sc = u + i * stride;
            const u64 c0 = (u64)sc * cand.C;
            const u32 len = cand.length(sc);
            for (u32 r0 = 0; r0 < len || pending != 0u; r0 += kRows * kChunkQuantum) {
                u32x16 bits;
                if (r0 + kRows * kChunkQuantum <= len) {
#pragma unroll
                    for (u32 q = 0; q < kRows; ++q) {
                        const f32x4 v = *reinterpret_cast<const f32x4u *>(cand.a + c0 + r0 + q * kChunkQuantum + 4u * lane);
#pragma unroll
                        for (u32 e = 0; e < 4; ++e) bits[4 * q + e] = __float_as_uint(v[e]);
                    }
                } else {
#pragma unroll
                    for (u32 q = 0; q < kRows; ++q)
#pragma unroll
                        for (u32 e = 0; e < 4; ++e) {
                            const u32 at = r0 + q * kChunkQuantum + 4u * lane + e;
                            bits[4 * q + e] = at < len ? __float_as_uint(cand.a[c0 + at]) : 0u;
                        }
                }
#pragma unroll 1
                for (u32 q = 0; q <= kRows; ++q) {
                    const u32 place = r0 + q * kChunkQuantum + 4u * lane;
                    if (q < kRows) {
                        u64 b[4];
                        bool hit[4];
#pragma unroll
                        for (u32 e = 0; e < 4; ++e) {
                            hit[e] = place + e < len && keep(bits[4 * q + e]);
                            b[e] = __ballot(hit[e]);
                        }
                        if ((b[0] | b[1] | b[2] | b[3]) == 0ull) continue;
                        u32 p = head + pending + popc64(b[0] & below) + popc64(b[1] & below) +
                                popc64(b[2] & below) + popc64(b[3] & below);
#pragma unroll
                        for (u32 e = 0; e < 4; ++e)
                            if (hit[e]) {
                                buf[p & (kRowQueueSize - 1u)] = make_uint2((u32)c0 + place + e, bits[4 * q + e]);
                                ++p;
                            }
                        pending += popc64(b[0]) + popc64(b[1]) + popc64(b[2]) + popc64(b[3]);
                        wave_lds_fence();
                    }
                    // the chunk's end empties the ring
                    const bool flush = q == kRows && r0 + kRows * kChunkQuantum >= len;
                    while (pending >= (u32)kWave || (flush && pending != 0u)) {
                        const u32 take = pending < (u32)kWave ? pending : (u32)kWave;
                        const bool v = lane < take;
                        const uint2 e = v ? buf[(head + lane) & (kRowQueueSize - 1u)] : make_uint2(0u, 0u);
                        f(v, i, e.x, e.y);
                        head += take;
                        pending -= take;
                        wave_lds_fence();
                    }
                }
            }
        }
    }
};
constexpr u32 kRowQueue = 512;               // ring of one wavefront (ChunkWalk::kRowQueueSize entries)

using UnitWalk = ChunkWalk<kUnitChunksMax>;  // classify / emit: chunks u, u + U, u + 2U, ...

// per-element form of a row callback: f(valid, i, index, pattern) for the four
// elements of a lane, from one call site (the loop is kept rolled)
template <class F>
__device__ __forceinline__ auto each_of_row(F &&f)
{
    return [&f](u32 i, u32 idx0, const u32 (&bits)[4], const bool (&valid)[4]) {
#pragma unroll 1
        for (u32 e = 0; e < 4; ++e) {
            const u32 b = e == 0 ? bits[0] : e == 1 ? bits[1] : e == 2 ? bits[2] : bits[3];
            const bool v = e == 0 ? valid[0] : e == 1 ? valid[1] : e == 2 ? valid[2] : valid[3];
            f(v, i, idx0 + e, b);
        }
    };
}

// ---------------------------------------------------------------------------
// pick: one workgroup finds the bin that holds the r-th largest magnitude
// from the rows the streaming workgroups stored, in two rounds of loads:
// the group sums of all rows (which group holds it, and how many entries lie
// above that group), then that group's bins of all rows.
// ---------------------------------------------------------------------------
constexpr u32 kPickThreads = 1024;

// the deciding bin: its pattern range and the entries above it
struct Picked {
    u32 mode;           // see EncodeCtl
    u32 bd_lo, bd_hi;
    u64 c_def;
    u32 n_bin;
    __device__ __forceinline__ void store(EncodeCtl *ctl) const
    {
        ctl->mode = mode;
        ctl->bd_lo = bd_lo;
        ctl->bd_hi = bd_hi;
        ctl->bd_bits = bd_hi > bd_lo ? 32u - (u32)__clz(bd_hi - bd_lo) : 1u;
        ctl->c_def = c_def;
    }
};

// lane l holds the count of the l-th position from the top (0 beyond the
// last): the position p with #(above p) < need <= #(above p) + count(p), and
// #(above p); found is false when all positions together do not reach need
__device__ __forceinline__ void wave_pick_desc(u32 count, u64 need, u64 above_all, bool *found,
                                               u32 *pos, u64 *above)
{
    const u32 inc = wave_inclusive_sum(count);
    const u64 before = above_all + (inc - count);
    const u64 owner = __ballot(before < need && need <= before + count);
    *found = owner != 0ull;
    const int src = *found ? __ffsll((unsigned long long)owner) - 1 : 0;
    *pos = (u32)src;
    const u32 b_lo = (u32)__builtin_amdgcn_readlane((int)(u32)before, src);
    const u32 b_hi = (u32)__builtin_amdgcn_readlane((int)(u32)(before >> 32), src);
    *above = ((u64)b_hi << 32) | b_lo;
}

__device__ __forceinline__ Picked
pick_body(const u32 *__restrict__ partials, const u32 *__restrict__ group_sums, u32 n_rows, const Geom &g,
          const EncodeCtl *ctl)
{
    __shared__ u32 gtot[kMaxGroups];
    __shared__ u32 btot[kCoarseSpan];
    __shared__ u32 sel_group, sel_found;
    __shared__ u64 sel_above;
    __shared__ Picked picked;
    const Bins bins = ctl->bins;
    const u32 nbins = bins.nfine + kCoarseBins;
    const u32 ngroups = (nbins + kCoarseSpan - 1) / kCoarseSpan;
    const u32 tid = threadIdx.x, lane = lane_id();
    if (tid < kMaxGroups) gtot[tid] = 0u;
    if (tid < kCoarseSpan) btot[tid] = 0u;
    lds_barrier();
    // ---- the group sums of every row, four loads per thread in flight together
    //      (256 rows of 12 groups: one round)
    {
        constexpr u32 kAhead = 4;
        const u32 words = n_rows * ngroups;
        for (u32 i0 = tid; i0 < words; i0 += kAhead * kPickThreads) {
            u32 v[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 i = i0 + q * kPickThreads;
                v[q] = i < words ? group_sums[(u64)(i / ngroups) * kMaxGroups + i % ngroups] : 0u;
            }
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 i = i0 + q * kPickThreads;
                if (v[q]) atomicAdd(&gtot[i % ngroups], v[q]);
            }
        }
    }
    __syncthreads();
    if (tid < kWave) {
        // groups number at most 36: lane l looks at group ngroups - 1 - l
        static_assert(kMaxGroups <= kWave, "one lane per group");
        const u32 cnt = lane < ngroups ? gtot[ngroups - 1u - lane] : 0u;
        bool found;
        u32 pos;
        u64 above;
        wave_pick_desc(cnt, g.r, 0ull, &found, &pos, &above);
        if (lane == 0) {
            sel_found = found ? 1u : 0u;
            sel_group = found ? ngroups - 1u - pos : 0u;
            sel_above = above;
        }
    }
    lds_barrier();
    bool dense = sel_found == 0u;                  // all rows together hold fewer than r entries
    u32 bin_s = 0;
    u64 before_s = 0;
    if (!dense) {
        // ---- that group's bins of every row: 64 consecutive words per row, sixteen
        //      loads per thread in flight together (256 rows: one round)
        const u32 first_bin = sel_group * kCoarseSpan;
        constexpr u32 kAhead = 16;
        const u32 words = n_rows * kCoarseSpan;
        for (u32 i0 = tid; i0 < words; i0 += kAhead * kPickThreads) {
            u32 v[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 i = i0 + q * kPickThreads;
                const u32 b = first_bin + i % kCoarseSpan;
                v[q] = (i < words && b < nbins) ? partials[(u64)(i / kCoarseSpan) * nbins + b] : 0u;
            }
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 i = i0 + q * kPickThreads;
                if (v[q]) atomicAdd(&btot[i % kCoarseSpan], v[q]);
            }
        }
        __syncthreads();
        if (tid < kWave) {
            const u32 cnt = btot[kCoarseSpan - 1u - lane];     // bins past nbins stayed 0
            bool found;
            u32 pos;
            u64 above;
            wave_pick_desc(cnt, g.r, sel_above, &found, &pos, &above);
            bin_s = first_bin + (kCoarseSpan - 1u - pos);
            before_s = above;
            if (!found || bin_s >= nbins) dense = true;     // (the group's sum promised otherwise)
        }
    }
    if (tid == 0) {
        u32 bd_lo = 0, bd_hi = 0;
        if (!dense) bin_range(bins, bin_s, &bd_lo, &bd_hi);
        // above the bracket S only holds what may be sent (everything when k == r or nothing was
        // keyed): no short list can decide there
        const bool partial = !dense && bin_s >= bins.nfine && g.take_all == 0u && g.keyed != 0u;
        picked = Picked{(dense ? 1u : 0u) | (partial ? 2u : 0u), bd_lo, bd_hi, before_s, 0u};
    }
    lds_barrier();
    return picked;
}

// ---------------------------------------------------------------------------
// count: what a short vector has in the place of sample, estimate and fused. a = g + m ->
// residual buffer, and EVERY magnitude is counted by its leading 15 bits in the workgroup's histogram: no
// bracket is needed, and no candidates are kept: classify reads the vector again (a few MB, still
// in the caches) once the deciding bin is known. Two launches and their dependent trips less, for an LDS
// addition per element, which a short vector's stream (one chunk per wavefront, all its loads in
// flight at once) waits long enough for.
//
// A bin is a 128th of an octave wide; a group of kGroupBins bins is an octave. The row a workgroup
// stores: the sums of all 256 groups (two bytes each), and the bins of the groups it has anything
// in. Those lie in kRowSlots slots, group e in slot e mod kRowSlots: of groups that meet there the
// highest one that is not empty, the others are marked kNotStored in their sums (that takes magnitudes 64
// octaves apart in one workgroup; should one of those groups decide, classify narrows it as a crowded bin).
// Magnitudes in bin 0 (zeros, mostly, which come in long runs) are not counted: what the
// others do not account for lies there.
// ---------------------------------------------------------------------------
constexpr u32 kCountShift = 16, kCountBins = 1u << (31 - kCountShift);
constexpr u32 kGroupBins = 128, kCountGroups = kCountBins / kGroupBins;
constexpr u32 kRowSlots = 64, kNotStored = 0x8000u;
constexpr u32 kRowWords = kRowSlots * kGroupBins / 2;    // of a row's bins, two to a word
constexpr u32 kCountRows = 128;               // rows at most
constexpr u32 kCountChunks = 3072;            // chunks of a vector at most
constexpr u32 kCountThreads = 1024;           // at most
constexpr u32 kPartBits = 8;                  // (see narrow_bin)
static_assert((u64)kCountRows * kRowWords * 4 <= (u64)kMaxFusedBlocks * kMaxBins * 4, "the rows lie where the others would");
static_assert((u64)kCountRows * kCountGroups * 2 <= (u64)kSampleLoc * 8, "the sums lie where the samples would");
// chunks of a workgroup at most: one per wavefront, or one more for half of them
constexpr u32 kCountEach = kCountThreads / kWave * 3 / 2;
static_assert(kCountEach * kMinChunk < kNotStored && kCountEach * kCountRows >= kCountChunks, "sums leave the mark's bit free");

// every lane gets the sum over its row of 16 lanes
__device__ __forceinline__ u32 row_sum(u32 v)
{
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x128 /* row_ror:8 */, 0xF, 0xF, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, false);
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, false);
    return v;
}

constexpr u32 kChunkRows = kMinChunk / kChunkQuantum;

__device__ __forceinline__ void
count_body(const float *__restrict__ grad, float *__restrict__ residual, const Geom &g, u32 *__restrict__ zero_base,
           u32 zero_words, u32 *__restrict__ zero_groups, u32 group_words, u16 *__restrict__ sums, uint4 *__restrict__ rows)
{
    __shared__ uint4 h4[kCountBins / 8];
    u32 *const h = reinterpret_cast<u32 *>(h4);
    const u32 lane = lane_id(), wave = threadIdx.x / kWave, n_waves = blockDim.x / kWave;
    f32x4 gv[kChunkRows], mv[kChunkRows];
    auto load = [&](u64 c0) {
        const f32x4u *gp = reinterpret_cast<const f32x4u *>(grad + c0) + lane, *mp = reinterpret_cast<const f32x4u *>(residual + c0) + lane;
#pragma unroll
        for (u32 q = 0; q < kChunkRows; ++q) {
            gv[q] = __builtin_nontemporal_load(gp + q * kWave);
            mv[q] = mp[q * kWave];
        }
    };
    const u32 w_full = (u32)(g.d / kMinChunk), stride = gridDim.x * n_waves;
    u32 w = wave * gridDim.x + blockIdx.x;      // (a second round is a few wavefronts of every workgroup)
    if (w < w_full) load((u64)w * kMinChunk);
    for (u32 i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_words; i += gridDim.x * blockDim.x) zero_base[i] = 0u;
    for (u32 i = blockIdx.x * blockDim.x + threadIdx.x; i < group_words; i += gridDim.x * blockDim.x) zero_groups[i] = 0u;
    for (u32 i = threadIdx.x; i < kCountBins / 8; i += blockDim.x) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    lds_barrier();
    auto count = [&](float a) {
        const u32 b = mag_of(__float_as_uint(a)) >> kCountShift;
        if (b != 0u) atomicAdd(&h[b / 2u], 1u << (16u * (b & 1u)));
    };
    for (; w < w_full; w += stride) {
        f32x4u *mp = reinterpret_cast<f32x4u *>(residual + (u64)w * kMinChunk) + lane;
        f32x4 a[kChunkRows];
#pragma unroll
        for (u32 q = 0; q < kChunkRows; ++q) {
            a[q] = gv[q] + mv[q];
            mp[q * kWave] = a[q];
        }
        if (w + stride < w_full) load((u64)(w + stride) * kMinChunk);
#pragma unroll
        for (u32 q = 0; q < kChunkRows; ++q)
#pragma unroll
            for (u32 e = 0; e < 4; ++e) count(a[q][e]);
    }
    if (w == w_full)
        for (u64 i = (u64)w * kMinChunk + lane; i < g.d; i += kWave) {
            const float a = grad[i] + residual[i];
            residual[i] = a;
            count(a);
        }
    lds_barrier();
    // ---- the row: sixteen lanes per slot, the highest group first
    constexpr u32 kMeet = kCountGroups / kRowSlots;
    const u32 part = lane % 16u;
    u16 *my_sums = sums + blockIdx.x * kCountGroups;
    for (u32 slot = threadIdx.x / 16u; slot < kRowSlots; slot += blockDim.x / 16u) {
        uint4 c[kMeet];
#pragma unroll
        for (u32 x = 0; x < kMeet; ++x) c[x] = h4[(slot + x * kRowSlots) * (kGroupBins / 8u) + part];
        bool taken = false;
#pragma unroll
        for (u32 x = kMeet; x-- > 0;) {
            const u32 two = c[x].x + c[x].y + c[x].z + c[x].w;
            u32 sum = row_sum((two & 0xFFFFu) + (two >> 16));
            if (sum != 0u) {
                if (!taken) rows[((u64)blockIdx.x * kRowSlots + slot) * (kGroupBins / 8u) + part] = c[x];
                else sum |= kNotStored;
                taken = true;
            }
            if (part == 0u) my_sums[slot + x * kRowSlots] = (u16)sum;
        }
    }
}

// the deciding bin from those rows, by all threads of a workgroup (every thread gets the result; whether the
// bin's entries crowd in few places, *hot in LDS, after the next barrier)
typedef u16 u16x2 __attribute__((ext_vector_type(2)));
constexpr u32 kCrowds = 1u << 31;
template <u32 kThreads>
__device__ __forceinline__ Picked
pick_counted(const u16 *__restrict__ sums, const uint4 *__restrict__ rows, u32 n_rows, const Geom &g, u32 *hot)
{
    __shared__ u32 gtot[kCountGroups], btot[kGroupBins], lost_s;
    const u32 tid = threadIdx.x, lane = lane_id();
    for (u32 i = tid; i < kCountGroups; i += kThreads) gtot[i] = 0u;
    if (tid < kGroupBins) btot[tid] = 0u;
    if (tid == 0) { lost_s = 0u; *hot = 0u; }
    if (__builtin_expect(g.force_dense != 0u, 0)) return Picked{1u, 0u, 0u, 0ull, 0u};
    // ---- all rows' sums: a thread takes eight groups of every (kThreads / 32)-th row
    constexpr u32 kAt = kCountGroups / 8u, kOf = kGroupBins / 8u;
    constexpr u32 kAhead = kCountRows / (kThreads / kAt) < 8u ? kCountRows / (kThreads / kAt) : 8u;
    u32 sum[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    auto add_up = [&](const uint4 &v, u32 mask) {
        const u32 w[4] = {v.x & mask, v.y & mask, v.z & mask, v.w & mask};
#pragma unroll
        for (u32 c = 0; c < 4; ++c) { sum[2 * c] += w[c] & 0xFFFFu; sum[2 * c + 1] += w[c] >> 16; }
    };
    const uint4 *s4 = reinterpret_cast<const uint4 *>(sums);
    for (u32 r0 = tid / kAt; r0 < n_rows; r0 += kAhead * (kThreads / kAt)) {
        uint4 v[kAhead];
#pragma unroll
        for (u32 q = 0; q < kAhead; ++q) {
            const u32 row = r0 + q * (kThreads / kAt);
            v[q] = make_uint4(0u, 0u, 0u, 0u);
            if (row < n_rows) v[q] = s4[row * kAt + tid % kAt];
        }
#pragma unroll
        for (u32 q = 0; q < kAhead; ++q) add_up(v[q], 0x7FFF7FFFu);
    }
    lds_barrier();
#pragma unroll
    for (u32 c = 0; c < 8; ++c) if (sum[c]) atomicAdd(&gtot[tid % kAt * 8u + c], sum[c]);
    lds_barrier();
    // every wavefront finds the group for itself: lane l holds the l-th four groups from the top
    static_assert(kCountGroups == 4 * kWave && kGroupBins == 2 * kWave, "groups and bins per lane");
    u32 c4[4], four = 0;
#pragma unroll
    for (u32 q = 0; q < 4; ++q) { c4[q] = gtot[kCountGroups - 1u - 4u * lane - q]; four += c4[q]; }
    const u32 need = (u32)g.r;
    u32 inc = wave_inclusive_sum(four);
    u64 owner = __ballot(inc - four < need && need <= inc);
    if (owner == 0ull)       // the zeros decide
        return Picked{0u, 0u, (1u << kCountShift) - 1u, (u32)__builtin_amdgcn_readlane((int)inc, kWave - 1), 0u};
    u32 group = 0, above = inc - four;
#pragma unroll
    for (u32 q = 0; q < 3; ++q)
        if (group == q && above + c4[q] < need) { above += c4[q]; ++group; }
    int src = __ffsll((unsigned long long)owner) - 1;
    group = kCountGroups - 1u - 4u * (u32)src - (u32)__builtin_amdgcn_readlane((int)group, src);
    above = (u32)__builtin_amdgcn_readlane((int)above, src);
    // ---- that group's bins of the rows that have some
#pragma unroll
    for (u32 c = 0; c < 8; ++c) sum[c] = 0u;
    u16x2 most[4] = {};                    // of any row, in each of the eight bins
    u32 marks = 0;
    constexpr u32 kRounds = kCountRows / (kThreads / kOf);
    static_assert(kRounds <= 8u, "all rows in one round of loads");
    const u32 r0 = tid / kOf;
    {
        uint4 v[kRounds];
        u32 has[kRounds];
#pragma unroll
        for (u32 q = 0; q < kRounds; ++q) {
            const u32 row = r0 + q * (kThreads / kOf);
            v[q] = make_uint4(0u, 0u, 0u, 0u);
            has[q] = 0u;
            if (row < n_rows) {
                has[q] = sums[row * kCountGroups + group];
                v[q] = rows[((u64)row * kRowSlots + group % kRowSlots) * kOf + tid % kOf];
            }
        }
#pragma unroll
        for (u32 q = 0; q < kRounds; ++q) {
            if (q * (kThreads / kOf) >= n_rows) break;
            marks |= has[q] & kNotStored;
            const u32 mask = has[q] != 0u ? ~0u : 0u;
            add_up(v[q], mask);
            const u32 w[4] = {v[q].x & mask, v[q].y & mask, v[q].z & mask, v[q].w & mask};
#pragma unroll
            for (u32 c = 0; c < 4; ++c) most[c] = __builtin_elementwise_max(most[c], __builtin_bit_cast(u16x2, w[c]));
        }
    }
#pragma unroll
    for (u32 c = 0; c < 8; ++c) if (sum[c]) atomicAdd(&btot[tid % kOf * 8u + c], sum[c]);
    if (marks != 0u) lost_s = 1u;
    lds_barrier();
    if (__builtin_expect(lost_s != 0u, 0)) {
        // (the octave decides: classify narrows it, or the vector itself is walked)
        constexpr u32 kOctave = kGroupBins << kCountShift;
        *hot = 1u;
        return Picked{1u, group * kOctave, group * kOctave + (kOctave - 1u), above, gtot[group]};
    }
    const u32 b0 = btot[kGroupBins - 1u - 2u * lane], b1 = btot[kGroupBins - 2u - 2u * lane];
    inc = wave_inclusive_sum(b0 + b1);
    u32 before = above + inc - b0 - b1;
    owner = __ballot(before < need && need <= before + b0 + b1);
    src = owner != 0ull ? __ffsll((unsigned long long)owner) - 1 : 0;
    u32 bin = group * kGroupBins + kGroupBins - 1u - 2u * lane, in_bin = b0;
    if (before + b0 < need) { before += b0; --bin; in_bin = b1; }
    bin = (u32)__builtin_amdgcn_readlane((int)bin, src);
    before = (u32)__builtin_amdgcn_readlane((int)before, src);
    in_bin = (u32)__builtin_amdgcn_readlane((int)in_bin, src);
    // A classify workgroup's chunks are four rows' here, side by side: where it alone has more of the bin than
    // its list takes, one of them has more than a fourth of that. (A row is eight chunks or more, so spread entries may
    // look the same from 40 per classify workgroup on: up to 524,288 elements they are narrowed from there.)
    const u32 at = bin % kGroupBins;
    u32 mine = 0;
#pragma unroll
    for (u32 c = 0; c < 8; ++c) mine = at % 8u == c ? most[c / 2u][c % 2u] : mine;
    if (tid % kOf == at / 8u && in_bin > kLongList && mine > kLongList / kWalkWaves) *hot = 1u;
    return Picked{0u, bin << kCountShift, (bin << kCountShift) | ((1u << kCountShift) - 1u), before, in_bin};
}

// ---------------------------------------------------------------------------
// classify: walk S; certain members are keyed against the window, entries
// of the deciding bin go to the short list B. Of the deciding bin it also
// leaves the number of entries per chunk and the smallest and largest
// magnitude per workgroup: when the bin turns out to be one long run of equal
// magnitudes (a vector of zeros, of signs, of a few quantisation levels), the
// short list cannot hold it, but the last member is then simply the entry of
// a known rank in index order, which those counts locate.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void
classify_body(Geom g, PhiloxSeed seed, EncodeCtl *ctl, const float *__restrict__ a,
           const uint2 *__restrict__ seg, const uint2 *__restrict__ s_ent,
           u32 *__restrict__ win_cnt, u32 *__restrict__ bd_cnt, u32 *__restrict__ quad_win,
           uint2 *__restrict__ blk_lists, u32 *__restrict__ blk_bmin,
           u32 *__restrict__ blk_bmax, uint2 *__restrict__ m_ent, uint2 *__restrict__ b_ent)
{
    __shared__ u32 cnt_m, cnt_b, cnt_sure, bmin_s, bmax_s;
    __shared__ u32 per_chunk[kWalkWaves][kUnitChunksMax];
    __shared__ u32 per_chunk_b[kWalkWaves][kUnitChunksMax];
    __shared__ uint2 row_queue[kWalkWaves][kRowQueue];
    const u32 wave = threadIdx.x / kWave, lane = lane_id();
    const u32 u = blockIdx.x * kWalkWaves + wave;
    const bool undecided = ctl->mode != 0u;
    const u32 bd_lo = ctl->bd_lo, bd_hi = ctl->bd_hi;
    if (undecided) {
        if (threadIdx.x == 0) {
            blk_lists[blockIdx.x] = make_uint2(0u, 0u);
            blk_bmin[blockIdx.x] = 0xFFFFFFFFu; blk_bmax[blockIdx.x] = 0u;
        }
        return;
    }
    const Candidates cand{seg, s_ent, a, g.d, g.C, g.U, g.UC, false};
    const UnitWalk walk(cand, u < g.U ? u : g.W, g.U, g.W);
    if (threadIdx.x == 0) { cnt_m = 0u; cnt_b = 0u; cnt_sure = 0u; bmin_s = 0xFFFFFFFFu; bmax_s = 0u; }
    if (lane < kUnitChunksMax) { per_chunk[wave][lane] = 0u; per_chunk_b[wave][lane] = 0u; }
    __syncthreads();
    u32 lane_bmin = 0xFFFFFFFFu, lane_bmax = 0u;      // what this lane has already reported

    // entry p of this workgroup's short lists lives at [p][workgroup]: the
    // finalize kernel reads entry p of all workgroups with one coalesced load
    auto slot = [&](u32 p) { return (u64)p * g.G3 + blockIdx.x; };
    const u64 below = lanes_below();
    auto per_entry = [&](bool valid, u32 i, u32 idx, u32 bits, u32 key) {
        const u32 m = mag_of(bits);
        const bool member = valid && (g.all_members != 0u || m > bd_hi);
        const bool in_bin = valid && !member && m >= bd_lo;
        if (member) {
            if (key >> 30 == kKeyUnknown) key = key_word(idx, g, seed);
            const bool sure = key >> 30 == kKeyBelow;
            if (key >> 30 == kKeyInside) {
                const u32 p = atomicAdd(&cnt_m, 1u);
                if (p < kListCap) m_ent[slot(p)] = make_uint2((key >> kPlaceBits) & (kCutM - 1u), idx);
            }
            if (sure) atomicAdd(&per_chunk[wave][i], 1u);
        }
        if (in_bin) {
            // Entries of the deciding bin are few, or nearly all there is (a run of equal
            // magnitudes): the lanes that are here take their list slots with one addition.
            const u64 here = __ballot(true);
            u32 base = 0;
            if ((here & below) == 0ull) base = atomicAdd(&cnt_b, popc64(here));
            base = (u32)__builtin_amdgcn_readfirstlane((int)base);
            const u32 p = base + popc64(here & below);
            if (p < kListCap) b_ent[slot(p)] = make_uint2(m, idx);
            atomicAdd(&per_chunk_b[wave][i], 1u);
            if (m < lane_bmin) { lane_bmin = m; atomicMin(&bmin_s, m); }
            if (m > lane_bmax) { lane_bmax = m; atomicMax(&bmax_s, m); }
        }
    };
    walk.for_each(cand, [&](bool valid, u32 i, u32 idx, u32 bits, u32 key, u32, u32) {
        per_entry(valid, i, idx, bits, key);
    });
    if (__builtin_expect(walk.from_vector != 0ull, 0))
        walk.for_each_vector_entry(cand, row_queue[wave],
                                   [&](u32 bits) { return g.all_members != 0u || mag_of(bits) >= bd_lo; },
                                   [&](bool valid, u32 i, u32 idx, u32 bits) {
                                       per_entry(valid, i, idx, bits, kKeyUnknown << 30);
                                   });
    __builtin_amdgcn_wave_barrier();
    // certain winners, and entries of the deciding bin, of each of the wavefront's chunks
    u32 mine = 0;
    if (u < g.U && lane < g.UC) {
        const u32 s = u + lane * g.U;
        if (s < g.W) {
            mine = per_chunk[wave][lane];
            win_cnt[s] = mine;
            bd_cnt[s] = per_chunk_b[wave][lane];
        }
    }
    mine = wave_sum(mine);
    if (lane == 0 && mine) atomicAdd(&cnt_sure, mine);
    __syncthreads();
    // chunks u, u + 1, ... of the workgroup's wavefronts are neighbours: a quad in each round
    static_assert(kWalkWaves == kQuad, "the chunks of a round are a quad");
    if (threadIdx.x < g.UC && blockIdx.x * kQuad + threadIdx.x * g.U < g.W) {
        u32 sum = 0;
#pragma unroll
        for (u32 w = 0; w < kWalkWaves; ++w) sum += per_chunk[w][threadIdx.x];
        quad_win[blockIdx.x + threadIdx.x * (g.U / kQuad)] = sum;
    }
    if (threadIdx.x == 0) {
        const u32 in_m = cnt_m < kListCap ? cnt_m : kListCap, in_b = cnt_b < kListCap ? cnt_b : kListCap;
        blk_lists[blockIdx.x] = make_uint2(in_m | in_b << 16, cnt_sure);
        blk_bmin[blockIdx.x] = bmin_s;
        blk_bmax[blockIdx.x] = bmax_s;
        if (cnt_m > kListCap || cnt_b > kListCap) ctl->overflow = 1u;
        if (cnt_m > kListCap) ctl->overflow_m = 1u;
    }
}

// ---------------------------------------------------------------------------
// classify of a counted vector: every wavefront has one chunk of it, whose elements it has loaded
// before the deciding bin is known. What lies in the deciding bin or above it becomes the
// chunk's slice of S, keyed, and goes through the short lists and counters as in classify_body: from
// here on the call goes as any other. A crowded deciding bin is narrowed first.
// ---------------------------------------------------------------------------
struct ChunkRows {
    f32x4 v[kChunkRows];
    u32 len;                // elements of the chunk (0 beyond the vector)
    __device__ __forceinline__ ChunkRows(const float *__restrict__ a, u64 d, u32 s)
    {
        const u64 c0 = (u64)s * kMinChunk;
        len = c0 >= d ? 0u : d - c0 < kMinChunk ? (u32)(d - c0) : kMinChunk;
        const float *p = a + c0 + 4u * lane_id();
        if (len == kMinChunk) {
#pragma unroll
            for (u32 q = 0; q < kChunkRows; ++q) v[q] = *reinterpret_cast<const f32x4u *>(p + q * kChunkQuantum);
        } else {
#pragma unroll
            for (u32 q = 0; q < kChunkRows; ++q)
#pragma unroll
                for (u32 e = 0; e < 4; ++e) v[q][e] = q * kChunkQuantum + 4u * lane_id() + e < len ? p[q * kChunkQuantum + e] : 0.0f;
        }
    }
};

// until everything this wavefront has sent to memory is acknowledged
__device__ __forceinline__ void wait_own_memory()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// A bin of count is a 128th of an octave, whatever the values: of uniform ones the deciding bin may hold d / 256
// entries, of magnitudes that are nearly equal, or clipped with some noise on top, most of the vector, and no short list
// takes those. All workgroups know from the pick how many there are, and whether they crowd. From
// narrow_from on, or where they crowd, the workgroups count the bin's entries by their next 8 bits and go on with
// the one of 256 parts that decides. So they do with an octave whose bins some workgroup of count did not keep. Calls, us, with sample and bracket / counted, the bin as it is / narrowed, r = 1%:
// uniform values, 2 M elements 42.9 / 60.6 / 39.5, 3 M 45.4 / 76.7 / 47.1; 1 + 1% normal, 200,003 42.6 / 257 / 32.8, 2^20
// 46.9 / 83.3 / 38.6; clipped with noise of 1e-3, 200,003 42.8 / 3167 / 32.4, 2^20 70.9 / 124 / 39.2; one layer of 8192
// in 1..1.05, 200,003 45.0 / 390 / 38.5 (k = r / 40; with a tenth of r the layer's keys overflow M, by every path: 376 / 389 /
// 336); eight of 2^20, 1 + 5% normal 69.8 / 82.3 / 69.1. Where nothing
// narrows the call costs what it did (normal values, 2 M 34.3 / 34.4).
//
// For that they have to wait for each other (through device-scope atomics only, see grid_barrier). What bounds it is
// that additions to one line of memory take 35 ns each: so kPartGroup workgroups share counters and a count of
// arrivals, the last of them arrives for the group, and the last of all adds up the groups' counters, finds the
// part and leaves it in every group's word, which only that group polls. (One set of counters and one word for all: uniform
// values, 2^20 38.2, 2 M 50.8, 3 M 67.3; in groups 31.7, 37.9, 45.4; the look at whether the magnitudes are equal, which
// saves vectors of signs 2 to 15 us, costs the others 1.5.) A workgroup that has polled kNarrowPolls times in vain calls
// it off for all (one compare-and-swap stands): two grids of two streams, each holding half of the compute units, would
// otherwise wait for each other. Finalize then has the crowded bin.
struct PartGroup {
    u32 count[1u << kPartBits];
    u64 found;              // 0, kPartOff, or kPartFound and the part, its entries and the bin's entries above it
    u32 arrived;
    u32 pad[61];
};
constexpr u32 kPartGroup = 32, kPartGroups = kCountChunks / kWalkWaves / kPartGroup;
constexpr u64 kPartFound = 1ull, kPartOff = 2ull;
constexpr u32 kPartEntries = 22;             // bits
static_assert(kCountChunks * kMinChunk < 1u << kPartEntries && 2u + kPartBits + 2u * kPartEntries <= 64u, "a word holds it all");
// (the last one is for all groups; in the place of the group sums, which a counted vector has not)
static_assert((kPartGroups + 1u) * sizeof(PartGroup) <= (u64)kMaxFusedBlocks * kMaxGroups * 4, "room for the counters");
constexpr u32 kNarrowPolls = 1u << 9;        // (half a millisecond)
__host__ __device__ constexpr u32 part_groups(u32 G3) { return (G3 + kPartGroup - 1u) / kPartGroup; }

__device__ __forceinline__ Picked
narrow_bin(const ChunkRows &chunk, const Geom &g, const float *__restrict__ a, PartGroup *groups, const Picked &now)
{
    __shared__ u32 part[1u << kPartBits], last_s, looked_s, least_s, most_s;
    __shared__ u64 found_s;
    static_assert(kWalkThreads == 1u << kPartBits, "a counter per thread");
    constexpr u32 kMask = (1u << kPartBits) - 1u, kEntryMask = (1u << kPartEntries) - 1u;
    const u32 tid = threadIdx.x, lane = lane_id(), span = now.bd_hi - now.bd_lo;
    const u32 shift = 32u - kPartBits - (u32)__clz((int)span);
    // (where there is nothing narrower: the vector itself is walked if the bins were not kept)
    const Picked as_it_was = now.mode != 0u ? Picked{1u, 0u, 0u, 0ull, 0u} : now;
    const u32 n_groups = part_groups(gridDim.x), group = blockIdx.x / kPartGroup;
    PartGroup &mine = groups[group], &root = groups[n_groups];
    // (a look at 1,024 elements, the same ones by all workgroups; of a bin, which is crowded, so that there are four.
    // An octave may be narrowed in a vector of two.)
    const bool looks = now.mode == 0u && g.d >= 4u;
    f32x4 some = {};
    if (looks) some = *reinterpret_cast<const f32x4u *>(a + (u64)tid * (g.d - 4u) / (kWalkThreads - 1u));
    part[tid] = 0u;
    if (tid == 0u) { last_s = 0u; found_s = 0ull; looked_s = 0u; least_s = ~0u; most_s = 0u; }
    lds_barrier();
#pragma unroll
    for (u32 q = 0; q < kChunkRows; ++q)
#pragma unroll
        for (u32 e = 0; e < 4; ++e) {
            const u32 x = mag_of(__float_as_uint(chunk.v[q][e])) - now.bd_lo, at = x >> shift;
            const bool in = x <= span && q * kChunkQuantum + 4u * lane + e < chunk.len;
            const u64 here = __ballot(in);
            if (here == 0ull) continue;
            // (all of one part: one addition serves them)
            const int src = __ffsll((unsigned long long)here) - 1;
            const u32 first = (u32)__builtin_amdgcn_readlane((int)at, src);
            if (__ballot(in && at == first) == here) {
                if ((int)lane == src) atomicAdd(&part[first], popc64(here));
            } else if (in) {
                atomicAdd(&part[at], 1u);
            }
        }
    u32 looked = 0, least = ~0u, most = 0;
#pragma unroll
    for (u32 e = 0; e < 4; ++e) {
        const u32 m = mag_of(__float_as_uint(some[e]));
        if (m - now.bd_lo > span) continue;
        ++looked;
        least = m < least ? m : least;
        most = m > most ? m : most;
    }
    looked = wave_sum(looked);
    least = ~wave_max_dpp(~least);
    most = wave_max_dpp(most);
    if (lane == 0u) { atomicAdd(&looked_s, looked); atomicMin(&least_s, least); atomicMax(&most_s, most); }
    lds_barrier();
    // equal magnitudes (signs, a few levels): no part will be smaller
    if (looks && looked_s > 1u && least_s == most_s) return now;
    if (part[tid] != 0u) __hip_atomic_fetch_add(&mine.count[tid], part[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_own_memory();
    __syncthreads();
    if (tid == 0u) {
        const u32 of_group = gridDim.x - group * kPartGroup < kPartGroup ? gridDim.x - group * kPartGroup : kPartGroup;
        if (__hip_atomic_fetch_add(&mine.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == of_group)
            last_s = __hip_atomic_fetch_add(&root.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == n_groups ? 1u : 0u;
    }
    __syncthreads();
    // (by the first lanes of a workgroup: one word stands for all groups)
    auto decide = [&](u64 word) {
        u64 expected = 0ull;
        bool stands = false;
        if (tid == 0u)
            stands = __hip_atomic_compare_exchange_strong(&root.found, &expected, word, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
        if (__ballot(stands) != 0ull && lane < n_groups)
            __hip_atomic_store(&groups[lane].found, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    static_assert(kPartGroups <= (u32)kWave, "a lane per group");
    if (last_s != 0u) {
        constexpr u32 kAhead = 12;
        u32 sum = 0;
        for (u32 q0 = 0; q0 < n_groups; q0 += kAhead) {
            u32 c[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q)
                c[q] = __hip_atomic_load(&groups[q0 + q < n_groups ? q0 + q : 0u].count[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) sum += q0 + q < n_groups ? c[q] : 0u;
        }
        part[tid] = sum;
        __syncthreads();
        if (tid < (u32)kWave) {
            // lane l has the l-th four counters from the top
            u32 c[4], four = 0;
#pragma unroll
            for (u32 q = 0; q < 4; ++q) { c[q] = part[kMask - 4u * lane - q]; four += c[q]; }
            const u32 need = (u32)(g.r - now.c_def), inc = wave_inclusive_sum(four);
            const u64 owner = __ballot(inc - four < need && need <= inc);
            u32 at = 0, above = inc - four, here = c[0];
#pragma unroll
            for (u32 q = 0; q < 3; ++q)
                if (at == q && above + c[q] < need) { above += c[q]; ++at; here = c[q + 1u]; }
            const int src = owner != 0ull ? __ffsll((unsigned long long)owner) - 1 : 0;
            at = kMask - 4u * (u32)src - (u32)__builtin_amdgcn_readlane((int)at, src);
            above = (u32)__builtin_amdgcn_readlane((int)above, src);
            here = (u32)__builtin_amdgcn_readlane((int)here, src);
            // (the bin holds as many as are needed)
            decide(owner != 0ull ? kPartFound | (u64)at << 2 | (u64)here << (2u + kPartBits) | (u64)above << (2u + kPartBits + kPartEntries)
                                 : kPartOff);
        }
    }
    if (tid < (u32)kWave) {
        u64 word = 0ull;
        u32 polls = 0;
        while ((word = __hip_atomic_load(&mine.found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0ull) {
            __builtin_amdgcn_s_sleep(16);
            if (++polls == kNarrowPolls) decide(kPartOff);
            if (polls > kWideSpinLimit) { word = kPartOff; break; }      // (cannot happen: somebody decides)
        }
        if (tid == 0u) found_s = word;
    }
    __syncthreads();
    const u64 word = found_s;
    if ((word & kPartFound) == 0ull) return as_it_was;
    const u32 lo = now.bd_lo | ((u32)(word >> 2) & kMask) << shift;
    return Picked{0u, lo, lo | ((1u << shift) - 1u), now.c_def + ((u32)(word >> (2u + kPartBits + kPartEntries)) & kEntryMask),
                  (u32)(word >> (2u + kPartBits)) & kEntryMask};
}

// More entries of the bin than this, which only lists in memory would hold, are better off in the selections for lists that
// overflow where those run on many workgroups (1 - 1e-3 uniform, r = k = 1%, narrowed: 2^20, 16,000 entries, 132 in
// lists / 127, 2 M, 30,600, 200 / 137, 2.9 M, 44,000, 270 / 159).
constexpr u32 kMemoryEntries = 3u << 12;
__device__ __forceinline__ void
classify_counted(const ChunkRows &chunk, const Geom &g, const PhiloxSeed &seed, EncodeCtl *ctl, Picked now, const u32 &hot,
                 bool picked_here, u32 narrow_from, const float *__restrict__ a, PartGroup *groups, uint2 *__restrict__ seg,
                 uint2 *__restrict__ s_ent, u32 *__restrict__ win_cnt, u32 *__restrict__ bd_cnt,
                 u32 *__restrict__ quad_win, uint2 *__restrict__ blk_lists, u32 *__restrict__ blk_bmin,
                 u32 *__restrict__ blk_bmax, uint2 *__restrict__ m_ent, uint2 *__restrict__ b_ent)
{
    __shared__ u32 cnt_m, cnt_b, bmin_s, bmax_s, sure_s[kWalkWaves];
    __shared__ uint2 hits[kWalkWaves][kMinChunk];
    const u32 wave = threadIdx.x / kWave, lane = lane_id();
    const u32 s = blockIdx.x * kWalkWaves + wave;
    const u64 below = lanes_below();
    if (threadIdx.x == 0) { cnt_m = 0u; cnt_b = 0u; bmin_s = 0xFFFFFFFFu; bmax_s = 0u; }
    lds_barrier();
    const bool crowds = picked_here ? hot != 0u : (now.n_bin & kCrowds) != 0u;
    now.n_bin &= ~kCrowds;
    const bool narrows = narrow_from != 0u && (now.n_bin >= narrow_from || crowds);
    const u32 span = now.bd_hi - now.bd_lo;
    if (__builtin_expect(narrows, 0)) now = narrow_bin(chunk, g, a, groups, now);
    else if (now.mode != 0u) now = Picked{1u, 0u, 0u, 0ull, 0u};
    // The words of a kernel that picked are replaced by a narrower bin only: then all workgroups have arrived, and
    // nobody reads them any more. Otherwise one that starts late still may.
    const bool narrowed = narrows && now.mode == 0u && now.bd_hi - now.bd_lo < span;
    if ((picked_here || narrowed) && blockIdx.x == 0 && threadIdx.x == 0) now.store(ctl);
    // ---- the entries, in index order
    u32 n = 0;
    if (now.mode == 0u) {
#pragma unroll
        for (u32 q = 0; q < kChunkRows; ++q) {
            const u32 place = q * kChunkQuantum + 4u * lane;
            bool hit[4];
            u64 b[4];
#pragma unroll
            for (u32 e = 0; e < 4; ++e) {
                hit[e] = place + e < chunk.len && mag_of(__float_as_uint(chunk.v[q][e])) >= now.bd_lo;
                b[e] = __ballot(hit[e]);
            }
            if ((b[0] | b[1] | b[2] | b[3]) == 0ull) continue;
            u32 p = n + popc64(b[0] & below) + popc64(b[1] & below) + popc64(b[2] & below) + popc64(b[3] & below);
#pragma unroll
            for (u32 e = 0; e < 4; ++e)
                if (hit[e]) { hits[wave][p] = make_uint2(place + e, __float_as_uint(chunk.v[q][e])); ++p; }
            n += popc64(b[0]) + popc64(b[1]) + popc64(b[2]) + popc64(b[3]);
        }
    }
    wave_lds_fence();
    u32 kept = 0;           // entries of the slice (above g.cap: too many, the chunk will be read from the vector)
    // entry p of this workgroup's short lists lives at [p][workgroup]
    auto slot = [&](u32 p) { return (u64)p * g.G3 + blockIdx.x; };
    // places for the lanes that are here in a list of the workgroup: one addition
    auto places = [&](u32 *count, u64 here) {
        u32 base = 0;
        if ((here & below) == 0ull) base = atomicAdd(count, popc64(here));
        return (u32)__builtin_amdgcn_readfirstlane((int)base) + popc64(here & below);
    };
    // Where finalize has room for the whole bin, in LDS and in memory, a few workgroups may hold most of it (a layer of
    // like magnitudes).
    const u32 room = g.G3 * kListCap < kStageB ? g.G3 * kListCap : kStageB;
    const u32 cap_b = now.n_bin - 1u < room ? kLongList : kListCap;
    u32 sure = 0, in_bin = 0, lane_bmin = 0xFFFFFFFFu, lane_bmax = 0u;
    for (u32 j0 = 0; j0 < n; j0 += kWave) {
        const u32 j = j0 + lane;
        const bool valid = j < n;
        uint2 e = valid ? hits[wave][j] : make_uint2(0u, 0u);
        const u32 idx = s * kMinChunk + e.x, m = mag_of(e.y);
        const u32 key = key_word(idx, g, seed);
        const bool member = valid && m > now.bd_hi, here_b = valid && !member;
        // (as in Ring::take: of a vector whose members are many, those that will not be sent stay out)
        const bool stays = valid && (g.keyed == 0u || here_b || key >> 30 != kKeyAbove);
        const u64 mask = __ballot(stays);
        const u32 at = kept + popc64(mask & below);
        if (stays && at < g.cap) s_ent[s * g.cap + at] = make_uint2(key | e.x, e.y);
        kept += popc64(mask);
        sure += popc64(__ballot(member && key >> 30 == kKeyBelow));
        in_bin += popc64(__ballot(here_b));
        if (member && key >> 30 == kKeyInside) {
            const u32 p = places(&cnt_m, __ballot(true));
            if (p < kListCap) m_ent[slot(p)] = make_uint2((key >> kPlaceBits) & (kCutM - 1u), idx);
        }
        if (here_b) {
            const u32 p = places(&cnt_b, __ballot(true));
            // (finalize needs the key's word and, knowing the bin, half of the magnitude)
            if (p < cap_b) b_ent[slot(p)] = make_uint2((key & ~kPlaceMask) | (m & 0xFFFFu), idx);
            if (m < lane_bmin) { lane_bmin = m; atomicMin(&bmin_s, m); }
            if (m > lane_bmax) { lane_bmax = m; atomicMax(&bmax_s, m); }
        }
    }
    if (lane == 0) {
        sure_s[wave] = sure;
        if (s < g.W) {
            win_cnt[s] = sure;
            bd_cnt[s] = in_bin;
            seg[chunk_slot(s, g.U, g.UC)] = make_uint2(kept | (kept > g.cap ? kSliceFull : 0u), s * g.cap);
        }
    }
    lds_barrier();
    if (threadIdx.x == 0) {
        static_assert(kWalkWaves == kQuad, "the workgroup's chunks are a quad");
        const u32 of_quad = sure_s[0] + sure_s[1] + sure_s[2] + sure_s[3];
        quad_win[blockIdx.x] = of_quad;
        const u32 in_m = cnt_m < kListCap ? cnt_m : kListCap, in_b = cnt_b < cap_b ? cnt_b : cap_b;
        blk_lists[blockIdx.x] = make_uint2(in_m | in_b << 16, of_quad);
        blk_bmin[blockIdx.x] = bmin_s;
        blk_bmax[blockIdx.x] = bmax_s;
        if (cnt_m > kListCap || cnt_b > cap_b || (now.n_bin > kMemoryEntries && g.W >= kWideMinChunks)) ctl->overflow = 1u;
        if (cnt_m > kListCap) ctl->overflow_m = 1u;
    }
}

// ---------------------------------------------------------------------------
// Radix selection, most significant byte first, over distinct 96-bit strings
// hi:lo (hi 64 bits, lo 32 bits). for_each(f) calls f(hi, lo) for every
// element this thread is responsible for (the elements are split over the
// workgroup in a way that does not change between calls). Returns the
// rank-th smallest string (rank is 1-based). Bytes before first_byte are
// known to be zero in every string. *ok is cleared when fewer than `rank`
// strings exist. Two barriers per byte: the 256-bin histogram rotates through
// three buffers (the next one is cleared while the current one is filled),
// the first wavefront walks the bins and leaves the outcome in a fourth
// buffer for the others. The barriers
// order LDS only; for_each may read global memory but must not depend on
// global writes made by other threads since the last full barrier.
// ---------------------------------------------------------------------------
struct Pair96 {
    u64 hi;
    u32 lo;
};

__device__ __forceinline__ u32 pair_byte(u64 hi, u32 lo, int j /* 0 = most significant */)
{
    return j < 8 ? (u32)(hi >> (56 - 8 * j)) & 0xFFu : (lo >> (24 - 8 * (j - 8))) & 0xFFu;
}

__device__ __forceinline__ bool pair_matches(u64 hi, u32 lo, u64 phi, u32 plo, int nbytes)
{
    // do the first nbytes bytes of hi:lo equal those of phi:plo ?
    if (nbytes <= 0) return true;
    if (nbytes <= 8) return ((hi ^ phi) >> (64 - 8 * nbytes)) == 0ull;
    if (hi != phi) return false;
    return ((lo ^ plo) >> (32 - 8 * (nbytes - 8))) == 0u;
}

template <class ForEach>
__device__ __forceinline__ Pair96 block_select96(ForEach &&for_each, u64 rank, int first_byte,
                                                 u32 (*h)[256] /* 4 buffers */,
                                                 u64 *scratch /* 2 */, bool *ok)
{
    u64 phi = 0;
    u32 plo = 0;
    u64 need = rank;
    int j = first_byte;
    const u32 lane = lane_id();
    *ok = true;
    for (u32 b = threadIdx.x; b < 256u; b += blockDim.x) h[0][b] = 0u;
    lds_barrier();
    u32 cur = 0;
    for (; j < 12; ++j) {
        const u32 nxt = cur == 2u ? 0u : cur + 1u;
        for (u32 b = threadIdx.x; b < 256u; b += blockDim.x) h[nxt][b] = 0u;
        for_each([&](u64 hi, u32 lo) {
            if (pair_matches(hi, lo, phi, plo, j)) atomicAdd(&h[cur][pair_byte(hi, lo, j)], 1u);
        });
        lds_barrier();
        // the first wavefront walks the bins, lane l owning bins 4l .. 4l+3, and leaves
        // the outcome in the fourth buffer for the others (sixteen wavefronts walking
        // them side by side take twice as long as one walk and one more barrier)
        // (the strings number fewer than 2^32, so 32-bit counts do)
        if (threadIdx.x < kWave) {
            u32 c[4];
            u32 mine = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) { c[q] = h[cur][4 * lane + q]; mine += c[q]; }
            const u32 inc = wave_inclusive_sum(mine);
            u32 run = inc - mine;
            const bool mine_it = (u64)run < need && need <= (u64)inc;
            const u64 owner = __ballot(mine_it);
            if (owner == 0ull && lane == 0) h[3][3] = 0u;
            if (mine_it) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if ((u64)run < need && need <= (u64)run + c[q]) {
                        h[3][0] = 4 * lane + q;
                        h[3][1] = c[q];
                        h[3][2] = run;
                        h[3][3] = 1u;
                    }
                    run += c[q];
                }
            }
        }
        lds_barrier();
        if (h[3][3] == 0u) { *ok = false; return Pair96{0, 0}; }
        const u32 bin = h[3][0], in_bin = h[3][1], before = h[3][2];
        need -= before;
        if (j < 8) phi |= (u64)bin << (56 - 8 * j);
        else plo |= bin << (24 - 8 * (j - 8));
        cur = nxt;
        if (in_bin == 1u) { ++j; break; }
    }
    if (j < 12) {
        // exactly one string starts with the resolved bytes: fetch the rest of it
        for_each([&](u64 hi, u32 lo) {
            if (pair_matches(hi, lo, phi, plo, j)) { scratch[0] = hi; scratch[1] = lo; }
        });
        lds_barrier();
        phi = scratch[0];
        plo = (u32)scratch[1];
    }
    lds_barrier();
    return Pair96{phi, plo};
}

__device__ __forceinline__ bool pair_le(u64 hi, u32 lo, const Pair96 &p)
{
    return hi < p.hi || (hi == p.hi && lo <= p.lo);
}

// ---------------------------------------------------------------------------
// Selection among the short lists' strings: they have been counted in kWave * kPer bins
// (kPer a divisor of kWave) by their leading bits, and group by group of kPer bins. Every wavefront finds
// the bin of the rank-th string for itself (one group per lane, then one bin per lane: no barrier in
// between); the strings in that bin, a handful, are gathered, and every wavefront ranks them
// for itself, one per lane. (Byte by byte, as block_select96 goes, each byte takes two barriers of sixteen
// wavefronts and a walk over the bins, and the string left over one more round.)
// ---------------------------------------------------------------------------
template <u32 kPer, bool kTwoToAWord>
struct CutBins {
    u32 *bin, *group;       // counters in LDS
    __device__ __forceinline__ void add(u32 b) const
    {
        if (kTwoToAWord) atomicAdd(&bin[b / 2u], 1u << (16u * (b & 1u)));
        else atomicAdd(&bin[b], 1u);
        atomicAdd(&group[b / kPer], 1u);
    }
    __device__ __forceinline__ u32 in_bin(u32 b) const
    {
        return kTwoToAWord ? bin[b / 2u] >> (16u * (b & 1u)) & 0xFFFFu : bin[b];
    }
    // the bin that holds the rank-th string (1 <= rank <= strings added), the rank inside it and the strings in it
    __device__ __forceinline__ void find(u32 rank, u32 *at, u32 *rank_in, u32 *here) const
    {
        const u32 lane = lane_id();
        u32 c = group[lane], inc = wave_inclusive_sum(c);
        u64 owner = __ballot(inc - c < rank && rank <= inc);
        const int g0 = owner != 0ull ? __ffsll((unsigned long long)owner) - 1 : 0;
        rank -= (u32)__builtin_amdgcn_readlane((int)(inc - c), g0);
        c = lane < kPer ? in_bin((u32)g0 * kPer + lane) : 0u;
        inc = wave_inclusive_sum(c);
        owner = __ballot(inc - c < rank && rank <= inc);
        const int b0 = owner != 0ull ? __ffsll((unsigned long long)owner) - 1 : 0;
        *at = (u32)g0 * kPer + (u32)b0;
        *rank_in = rank - (u32)__builtin_amdgcn_readlane((int)(inc - c), b0);
        *here = (u32)__builtin_amdgcn_readlane((int)c, b0);
    }
};

// the rank-th (1-based) of n <= kWave distinct strings, one per lane; *up_to: the lane's
// string is it or comes before it
__device__ __forceinline__ Pair96 wave_rank(u64 hi, u32 lo, u32 n, u32 rank, bool *up_to)
{
    const u32 lane = lane_id();
    u32 smaller = 0;
#pragma unroll 1
    for (u32 j = 0; j < n; ++j) {
        const u32 h1 = (u32)__builtin_amdgcn_readlane((int)(u32)(hi >> 32), (int)j);
        const u32 h0 = (u32)__builtin_amdgcn_readlane((int)(u32)hi, (int)j);
        const u32 l = (u32)__builtin_amdgcn_readlane((int)lo, (int)j);
        const u64 h = ((u64)h1 << 32) | h0;
        smaller += (h < hi || (h == hi && l < lo)) ? 1u : 0u;
    }
    const u64 owner = __ballot(lane < n && smaller + 1u == rank);
    const int src = owner != 0ull ? __ffsll((unsigned long long)owner) - 1 : 0;
    *up_to = lane < n && smaller < rank;
    const u32 h1 = (u32)__builtin_amdgcn_readlane((int)(u32)(hi >> 32), src);
    const u32 h0 = (u32)__builtin_amdgcn_readlane((int)(u32)hi, src);
    return Pair96{((u64)h1 << 32) | h0, (u32)__builtin_amdgcn_readlane((int)lo, src)};
}

// ---------------------------------------------------------------------------
// The same selection spread over the workgroups of one grid (the finalize
// kernel's, at most kWideBlocks, which are resident together). Each workgroup
// histograms its share of the strings in LDS, adds its non-empty bins to the
// pass's 256-bin histogram in the workspace (device-scope atomics), and all
// meet at a barrier; every workgroup then reads the same totals and derives
// the same digit. The barrier is a counter that only grows; a workgroup that
// polls it kWideSpinLimit times in vain gives up, which ends the kernel with
// an error flag instead of a hang (the others give up in turn).
// ---------------------------------------------------------------------------
struct Wide {
    WideScratch *ws;
    u32 nblocks;
    u32 epoch;          // barriers passed
    u32 pass;           // histogram / fetch slots used
    bool alive;         // false once a barrier timed out
    u32 spin_limit;     // polls before a workgroup gives up at a barrier
};

// Everything the workgroups exchange goes through device-scope atomic
// operations (additions to the histograms, atomic stores of the few words
// workgroup 0 reads at the end, atomic loads on the reading side), which are
// carried out where all compute units see them. The barrier therefore only has
// to order them: every thread waits until its own operations are acknowledged
// before its workgroup checks in. (The wait is explicit: neither a workgroup-scope
// release nor the workgroup barrier waits for device memory, as the wavefronts of
// one workgroup share a cache.) A
// device-scope fence per thread, which writes back and invalidates the L2 of
// the XCD, made a barrier of 256 workgroups cost ~100 us.
__device__ __forceinline__ bool grid_barrier(Wide &w, u32 *lds_flag)
{
    if (!w.alive) return false;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    wait_own_memory();
    __syncthreads();
    ++w.epoch;
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&w.ws->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const u32 target = w.epoch * w.nblocks;
        u32 polls = 0;
        bool ok = true;
        while (__hip_atomic_load(&w.ws->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(32);
            if (++polls > w.spin_limit) { ok = false; break; }
        }
        *lds_flag = ok ? 1u : 0u;
    }
    __syncthreads();
    w.alive = *lds_flag != 0u;
    __syncthreads();
    return w.alive;
}

// What the selection over the grid settles: the first `bytes` bytes of the
// rank-th smallest string (the rest of hi:lo is zero). With bytes < 12 exactly
// ONE string starts with them, so "at or below the selected string" is the
// same as "at or below these bytes followed by ones" (bound()), and nobody has
// to go and fetch the rest before the next pass can start; is() recognises the
// selected string itself when a later pass comes across it.
struct Selected {
    u64 hi;
    u32 lo;
    int bytes;
    __device__ __forceinline__ Pair96 bound() const
    {
        if (bytes >= 12) return Pair96{hi, lo};
        if (bytes > 8) return Pair96{hi, lo | ((1u << (32 - 8 * (bytes - 8))) - 1u)};
        if (bytes == 8) return Pair96{hi, 0xFFFFFFFFu};
        return Pair96{hi | ((1ull << (64 - 8 * bytes)) - 1ull), 0xFFFFFFFFu};
    }
    __device__ __forceinline__ bool is(u64 shi, u32 slo) const { return pair_matches(shi, slo, hi, lo, bytes); }
};

// Before the first barrier the workgroups of the grid make sure that ALL of
// them are resident: every workgroup checks in; the last to arrive decides
// "go", a workgroup that has polled kWideCheckInLimit times in vain decides
// "abort" (compare-and-swap: one decision stands), and everybody waits for the
// decision. After "go" every workgroup is running, so the later barriers
// cannot wait for one that was never scheduled (two grids of two streams, each
// holding half of the compute units, would otherwise wait for each other until
// the poll limit). After "abort" nothing has been computed yet: the caller
// falls back to the selection by one workgroup. Counts as the first barrier.
__device__ __forceinline__ bool grid_check_in(Wide &w, u32 *lds_flag)
{
    __syncthreads();
    ++w.epoch;
    if (threadIdx.x == 0) {
        const u32 mine = __hip_atomic_fetch_add(&w.ws->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
        u32 expected = 0u;
        if (mine == w.nblocks)
            __hip_atomic_compare_exchange_strong(&w.ws->decision, &expected, kWideGo, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        u32 polls = 0, d = 0;
        while ((d = __hip_atomic_load(&w.ws->decision, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u) {
            __builtin_amdgcn_s_sleep(32);
            if (++polls == kWideCheckInLimit) {
                expected = 0u;
                __hip_atomic_compare_exchange_strong(&w.ws->decision, &expected, kWideAbort,
                                                     __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            }
            if (polls > kWideSpinLimit) { d = kWideAbort; break; }   // (cannot happen: somebody decides)
        }
        *lds_flag = d == kWideGo ? 1u : 0u;
    }
    __syncthreads();
    const bool go = *lds_flag != 0u;
    __syncthreads();
    return go;
}

// for_each(f) calls f(valid, hi, lo) for every string of this workgroup's
// share, ALL lanes of a wavefront together (valid says whether the lane holds
// one). *less_hi receives the number of strings whose high 64 bits are below
// the result's. h: 4 x 256 words of LDS.
template <class ForEach>
__device__ __forceinline__ Selected grid_select96(ForEach &&for_each, u64 rank, int first_byte, Wide &w,
                                                  u32 (*h)[256], u64 *less_hi, bool *ok)
{
    u64 phi = 0;
    u32 plo = 0;
    u64 need = rank;
    int j = first_byte;
    const u32 lane = lane_id();
    *ok = true;
    *less_hi = 0;
    for (; j < 12; ++j) {
        for (u32 b = threadIdx.x; b < 256u; b += blockDim.x) h[0][b] = 0u;
        lds_barrier();
        for_each([&](bool valid, u64 hi, u32 lo) {
            const bool on = valid && pair_matches(hi, lo, phi, plo, j);
            const u32 digit = pair_byte(hi, lo, j);
            // neighbouring strings often share the digit (runs of equal magnitudes): when all
            // of a wavefront's do, one addition serves them
            const u64 m = __ballot(on);
            if (m == 0ull) return;
            const int src = __ffsll((unsigned long long)m) - 1;
            const u32 first = (u32)__builtin_amdgcn_readlane((int)digit, src);
            if (__ballot(on && digit == first) == m) {
                if ((int)lane == src) atomicAdd(&h[0][first], popc64(m));
            } else if (on) {
                atomicAdd(&h[0][digit], 1u);
            }
        });
        lds_barrier();
        if (w.pass >= kWidePasses) { *ok = false; return Selected{0, 0, 12}; }
        u32 *gh = w.ws->hist[w.pass];
        for (u32 b = threadIdx.x; b < 256u; b += blockDim.x)
            if (h[0][b]) atomicAdd(&gh[b], h[0][b]);
        if (!grid_barrier(w, &h[3][4])) { *ok = false; return Selected{0, 0, 12}; }
        if (threadIdx.x < kWave) {
            u32 c[4];
            u32 mine = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = __hip_atomic_load(&gh[4 * lane + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                mine += c[q];
            }
            const u32 inc = wave_inclusive_sum(mine);
            u32 run = inc - mine;
            const bool mine_it = (u64)run < need && need <= (u64)inc;
            const u64 owner = __ballot(mine_it);
            if (owner == 0ull && lane == 0) h[3][3] = 0u;
            if (mine_it) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if ((u64)run < need && need <= (u64)run + c[q]) {
                        h[3][0] = 4 * lane + q;
                        h[3][1] = c[q];
                        h[3][2] = run;
                        h[3][3] = 1u;
                    }
                    run += c[q];
                }
            }
        }
        lds_barrier();
        ++w.pass;
        if (h[3][3] == 0u) { *ok = false; return Selected{0, 0, 12}; }
        const u32 bin = h[3][0], in_bin = h[3][1], before = h[3][2];
        lds_barrier();
        need -= before;
        if (j < 8) { phi |= (u64)bin << (56 - 8 * j); *less_hi += before; }
        else plo |= bin << (24 - 8 * (j - 8));
        if (in_bin == 1u) { ++j; break; }
    }
    return Selected{phi, plo, j};
}

// What finalize keeps in LDS. The short lists (see kStageB): counters of the two cuts (of M two to
// a word: M and the members of B that join it are fewer than 2^16), winners the lists add per quad
// (two to a word, at most a workgroup's lists), what shares a cut's bin. In their place, the keys of a run
// of equal magnitudes. Behind them, as much as the launch claims, M itself; elsewhere the run's indices or
// the winners per quad, and the histograms of the selections.
struct FinalizeLists {
    u32 bin_b[kCutB], bin_m[kCutM / 2], group_b[kWave], group_m[kWave], won[kQuads / 2];
    u32 b_x[kStageB], b_idx[kStageB];
    u32 cand[kWave], cand_idx[kWave], n_cand_b, n_cand_m;
};
constexpr u32 kRunWords = kStageRun + 4 * 256;
static_assert(kStageM + kStageB < 1u << 16, "two counters of M to a word");
static_assert(sizeof(FinalizeLists) >= 8 * kStageRun && sizeof(FinalizeLists) + 4 * kStageM + 1408 <= 160 * 1024,
              "the lists beside the kernel's other variables in one unit's LDS");
static u32 finalize_claim(const Geom &g) { return 4u * (g.stage_m > kRunWords ? g.stage_m : kRunWords); }

// ---------------------------------------------------------------------------
// The short lists of a counted vector of few classify workgroups, which leave a few entries each: all of them are
// fetched in the first round of loads, before it is known which places of the lists hold any, and stay in
// registers. What bounds finalize here is the chain of barriers and dependent steps; with sixteen wavefronts that all
// find the cuts and rank the candidates for themselves it was the issue of those instructions, four wavefronts
// to a SIMD, and the notes of where the entries are. Kernel, us: one vector of 200,003 elements 9.5 -> 6.8, of
// 2^20 10.2 -> 8.5.
// ---------------------------------------------------------------------------
constexpr u32 kSmallBlocks = 256;             // classify workgroups at most
constexpr u32 kOwn = 8;                       // entries of either list in a thread's registers
constexpr u32 kAtOnce = 8;                    // places of every workgroup's lists that are fetched before the counts are there
static_assert(kSmallBlocks <= (u32)kWave * 4u, "a classify workgroup is a quad of chunks: four per lane of one wavefront");

// Thread (row, col) of 2^(10 - c) x 2^c has kOwn entries of classify workgroup col. The lower half of the
// rows have the first ones; as a rule they are all there is, and the wavefronts of the upper half drop out.
struct OwnEntries {
    uint2 m[kOwn], b[kOwn];
    uint2 counts;               // as in blk_lists
    u32 cols, row, col, half, first;
    __device__ __forceinline__ OwnEntries(u32 G3, const uint2 *__restrict__ blk_lists, const uint2 *__restrict__ m_ent,
                                          const uint2 *__restrict__ b_ent)
    {
        constexpr u32 kThreadBits = 10;
        static_assert(kFinThreads == 1 << kThreadBits && kSmallBlocks <= kFinThreads / 2, "threads by columns and rows");
        cols = columns(G3);
        row = threadIdx.x >> cols;
        col = threadIdx.x & ((1u << cols) - 1u);
        half = kThreadBits - 1u - cols;                         // (the logarithm of half the rows)
        first = row >> half == 0u ? row : row + ((kOwn - 1u) << half);      // entries first, first + half the rows, ...
        counts = make_uint2(0u, 0u);
        if (col < G3) {
            counts = blk_lists[col];
#pragma unroll
            for (u32 q = 0; q < kOwn; ++q)
                if (place(q) < kAtOnce) {
                    m[q] = m_ent[place(q) * G3 + col];
                    b[q] = b_ent[place(q) * G3 + col];
                }
        }
    }
    __device__ __forceinline__ u32 place(u32 q) const { return first + (q << half); }
    // the other entries, once it is known that there are some: n of each workgroup's, `most` rounds of them
    __device__ __forceinline__ void fetch_rest(uint2 (&e)[kOwn], const uint2 *__restrict__ from, u32 G3, u32 n, u32 most)
    {
#pragma unroll
        for (u32 q = 0; q < kOwn; ++q) {
            if (q >= most) break;
            if (place(q) >= kAtOnce && place(q) < n) e[q] = from[place(q) * G3 + col];
        }
    }
    // (the rounds of this wavefront that hold any of n entries)
    __device__ __forceinline__ u32 rounds(u32 n) const
    {
        return wave_max_dpp(n > first ? (n - first + (1u << half) - 1u) >> half : 0u);
    }
    static __host__ __device__ __forceinline__ u32 columns(u32 G3)
    {
        u32 c = 4u;
        while (1u << c < G3) ++c;
        return c;
    }
    // places of either list of a classify workgroup that are in registers
    static __host__ __device__ __forceinline__ u32 deep(u32 cols) { return kOwn << (10u - cols); }
};

// False, with nothing changed that matters, where the lists cannot decide, have entries that are in no
// register, or many strings share a cut's bin.
__device__ __forceinline__ bool
finalize_small(const Geom &g, const PhiloxSeed &seed, EncodeCtl *ctl, FinalizeLists &ls, OwnEntries &own,
               u32 *__restrict__ win_cnt, const u32 *__restrict__ quad_win, const uint2 *__restrict__ m_ent,
               const uint2 *__restrict__ b_ent, u32 *__restrict__ quad_base)
{
    u32 (*part)[4] = reinterpret_cast<u32 (*)[4]>(ls.cand);     // (entries of M, of B, certain winners, whether more than fit) per wavefront
    static_assert(4 * kFinWaves <= kWave, "room for four words per wavefront");
    __shared__ u32 gt_s, sure_s, extra_s, done_s;
    const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const u32 chunk_shift = 31u - (u32)__clz((int)g.C);
    uint4 quads = make_uint4(0u, 0u, 0u, 0u);
    if (wave == 0 && 4u * lane * kQuad < g.W) quads = reinterpret_cast<const uint4 *>(quad_win)[lane];
    for (u32 i = tid; i < kCutM / 2u; i += kFinThreads) ls.bin_m[i] = 0u;
    if (tid < kCutB) ls.bin_b[tid] = 0u;
    if (tid < kSmallBlocks / 2u) ls.won[tid] = 0u;
    if (tid < (u32)kWave) { ls.group_b[tid] = 0u; ls.group_m[tid] = 0u; }
    if (tid == 0) { ls.n_cand_b = 0u; ls.n_cand_m = 0u; gt_s = 0u; sure_s = 0u; extra_s = 0u; done_s = 0u; }
    const u32 n_m = own.counts.x & 0xFFFFu, n_b = own.counts.x >> 16;
    if (wave < kSmallBlocks / kWave) {      // (row 0 is among these)
        const u32 deep = OwnEntries::deep(own.cols);
        const u64 more = __ballot(n_m > deep || n_b > deep), upper = __ballot(n_m > deep / 2u || n_b > deep / 2u);
        const u32 sum_m = wave_sum(own.row == 0u ? n_m : 0u), sum_b = wave_sum(own.row == 0u ? n_b : 0u),
                  sum_s = wave_sum(own.row == 0u ? own.counts.y : 0u);
        if (lane == 0) {
            part[wave][0] = sum_m;
            part[wave][1] = sum_b;
            part[wave][2] = sum_s;
            part[wave][3] = (more != 0ull ? 1u : 0u) | (upper != 0ull ? 2u : 0u);
        }
    }
    const u32 mode = ctl->mode, overflow = ctl->overflow, bd_hi = ctl->bd_hi, bd_bits = ctl->bd_bits;
    const u64 c_def = ctl->c_def;
    lds_barrier();
    u32 n_m0 = 0, n_bd = 0, sure_walk = 0, more = 0;
#pragma unroll
    for (u32 w = 0; w < kSmallBlocks / kWave; ++w) {
        n_m0 += part[w][0];
        n_bd += part[w][1];
        sure_walk += part[w][2];
        more |= part[w][3];
    }
    const u64 need2 = g.r - c_def;
    if (mode != 0u || overflow != 0u || (more & 1u) != 0u || c_def >= g.r || need2 > n_bd || n_bd > kStageB) return false;
    if (!g.take_all && (sure_walk >= g.k || sure_walk + n_m0 + need2 < g.k)) return false;     // (the window certainly missed)
    const bool works = wave < kFinWaves / 2u || (more & 2u) != 0u;
    // ---- count. An entry of B is the magnitude's low half (2^16 magnitudes to a bin) and the key's word.
    const u32 shift_b = bd_bits > 10u ? bd_bits - 10u : 0u;
    static_assert(kCutB == 1u << 10 && kCountShift == 16u, "bits of a bin of B");
    const CutBins<kCutB / kWave, false> cut_b{ls.bin_b, ls.group_b};
    const CutBins<kCutM / kWave, true> cut_m{ls.bin_m, ls.group_m};
    // (up to the last one that some lane holds)
    const u32 rounds_m = works ? own.rounds(n_m) : 0u, rounds_b = works ? own.rounds(n_b) : 0u;
    own.fetch_rest(own.m, m_ent, g.G3, n_m, rounds_m);
    own.fetch_rest(own.b, b_ent, g.G3, n_b, rounds_b);
    auto each_own = [&](u32 n, u32 most, auto &&f) {
#pragma unroll
        for (u32 q = 0; q < kOwn; ++q) {
            if (q >= most) break;
            if (own.place(q) < n) f(q);
        }
    };
    auto x_of = [&](u32 q) { return (bd_hi - own.b[q].x) & 0xFFFFu; };
    auto place_of = [&](u32 q) { return own.b[q].x >> kPlaceBits & (kCutM - 1u); };
    if (works) {
        each_own(n_m, rounds_m, [&](u32 q) { cut_m.add(own.m[q].x); });
        each_own(n_b, rounds_b, [&](u32 q) { cut_b.add(x_of(q) >> shift_b); });
    }
    lds_barrier();
    // ---- the cut in B
    u32 at = 0, rank = 0, here = 0;
    bool ok = works;
    if (works) {
        cut_b.find((u32)need2, &at, &rank, &here);
        ok = here <= (u32)kWave;
        if (ok)
            each_own(n_b, rounds_b, [&](u32 q) {
                if (x_of(q) >> shift_b == at) {
                    const u32 j = atomicAdd(&ls.n_cand_b, 1u);
                    ls.b_x[j] = x_of(q);
                    ls.b_idx[j] = own.b[q].y;
                }
            });
    }
    lds_barrier();
    // ---- members of the deciding bin: certain winners, or as good as entries of M
    Pair96 tb{0ull, 0u};
    bool up_to = false;
    u32 member = 0;             // bit q: own.b[q] is a member that may be sent
    if (ok) {
        tb = wave_rank(lane < here ? ls.b_x[lane] : 0u, lane < here ? ls.b_idx[lane] : 0u, here, rank, &up_to);
        u32 my_gt = 0, my_sure = 0, my_extra = 0;
        each_own(n_b, rounds_b, [&](u32 q) {
            const u32 says = own.b[q].x >> 30;
            if ((u64)x_of(q) < tb.hi) ++my_gt;
            if (!pair_le((u64)x_of(q), own.b[q].y, tb) || says == kKeyAbove) return;
            member |= 1u << q;
            if (says == kKeyBelow) ++my_sure;
            else { cut_m.add(place_of(q)); ++my_extra; }
        });
        static_assert(kOwn * kWave <= 1u << 10, "three sums, two to a word");
        const u32 sums = wave_sum(my_gt | my_sure << 16), extra = wave_sum(my_extra);
        if (lane == 0) {
            if (sums & 0xFFFFu) atomicAdd(&gt_s, sums & 0xFFFFu);
            if (sums >> 16) atomicAdd(&sure_s, sums >> 16);
            if (extra) atomicAdd(&extra_s, extra);
        }
    }
    lds_barrier();
    // ---- the cut in M
    auto won = [&](u32 sc) {
        const u32 x = sc / kQuad;
        atomicAdd(&ls.won[x / 2u], 1u << (16u * (x & 1u)));
        atomicAdd(&win_cnt[sc], 1u);
    };
    u32 n_mm = 0;
    if (ok) {
        n_mm = n_m0 + extra_s;
        const u32 c_klo = sure_walk + sure_s;
        at = 0;
        if (!g.take_all) {
            ok = c_klo < g.k && g.k - c_klo <= n_mm;
            if (ok) {
                cut_m.find((u32)g.k - c_klo, &at, &rank, &here);
                ok = here <= (u32)kWave;
            }
        }
        if (ok) {
            each_own(n_b, rounds_b, [&](u32 q) {
                if (!(member >> q & 1u)) return;
                if (own.b[q].x >> 30 == kKeyBelow || place_of(q) < at) won(own.b[q].y >> chunk_shift);
                else if (place_of(q) == at) ls.cand_idx[atomicAdd(&ls.n_cand_m, 1u)] = own.b[q].y;
            });
            each_own(n_m, rounds_m, [&](u32 q) {
                if (own.m[q].x < at) won(own.m[q].y >> chunk_shift);
                else if (own.m[q].x == at) ls.cand_idx[atomicAdd(&ls.n_cand_m, 1u)] = own.m[q].y;
            });
            if (tid == 0) done_s = 1u;
        }
    }
    lds_barrier();
    u64 K_star = ~0ull;
    u32 J_star = 0xFFFFFFFFu;
    if (ok && !g.take_all && wave == 0) {
        const u32 idx = lane < here ? ls.cand_idx[lane] : 0u;
        const Pair96 kb = wave_rank((sample_key(idx, seed) - g.K_lo) << g.k_nlz, idx, here, rank, &up_to);
        if (up_to) won(idx >> chunk_shift);
        K_star = (kb.hi >> g.k_nlz) + g.K_lo;
        J_star = kb.lo;
        wave_lds_fence();
    }
    if (done_s == 0u) return false;
    if (wave != 0u) return true;
    // ---- output offsets of the quads of chunks, and what emit needs
    const u32 w01 = ls.won[2u * lane], w23 = ls.won[2u * lane + 1u], x = 4u * lane;
    quads.x = x * kQuad < g.W ? quads.x + (w01 & 0xFFFFu) : 0u;
    quads.y = (x + 1u) * kQuad < g.W ? quads.y + (w01 >> 16) : 0u;
    quads.z = (x + 2u) * kQuad < g.W ? quads.z + (w23 & 0xFFFFu) : 0u;
    quads.w = (x + 3u) * kQuad < g.W ? quads.w + (w23 >> 16) : 0u;
    const u32 four = quads.x + quads.y + quads.z + quads.w, inc = wave_inclusive_sum(four);
    if (x * kQuad < g.W) {
        uint4 o;
        o.x = inc - four;
        o.y = o.x + quads.x;
        o.z = o.y + quads.y;
        o.w = o.z + quads.z;
        reinterpret_cast<uint4 *>(quad_base)[lane] = o;
    }
    if (lane == kWave - 1) {
        ctl->err = inc != (u32)g.k ? kErrCount : 0u;
        ctl->path = 0u;
        ctl->T = bd_hi - (u32)tb.hi;
        ctl->I_star = tb.lo;
        ctl->K_star = K_star;
        ctl->J_star = J_star;
        ctl->n_b = n_bd;
        ctl->n_m = n_mm;
        ctl->W = g.W;
        ctl->U = g.U;
        ctl->UC = g.UC;
        ctl->count_greater = c_def + gt_s;
        ctl->ties = g.r - (c_def + gt_s);
        ctl->how = kHowRegisters | (bd_bits < kCountShift ? kHowNarrowed : 0u);
    }
    return true;
}

// ---------------------------------------------------------------------------
// finalize: turns the short lists into the two cut points and the output
// offset of every chunk (workgroup 0; the others leave at once), or, when the
// counts left by classify show that the lists cannot decide and the vector is
// long, runs the exact selection over all candidates on all its workgroups.
// ---------------------------------------------------------------------------
template <bool kCounted>
__device__ __forceinline__ void
finalize_body(Geom g, PhiloxSeed seed, EncodeCtl *ctl, WideScratch *wide_ws,
           const float *__restrict__ a, uint2 *seg, uint2 *s_ent,
           u32 *win_cnt, const u32 *__restrict__ bd_cnt, const u32 *__restrict__ quad_win,
           const uint2 *__restrict__ blk_lists, const u32 *__restrict__ blk_bmin,
           const u32 *__restrict__ blk_bmax, const uint2 *__restrict__ m_ent,
           const uint2 *__restrict__ b_ent, u64 *dm_key,
           u32 *dm_idx, u64 *db_key, u32 *db_idx, u32 *__restrict__ quad_base)
{
    static_assert(kMaxWalkBlocks <= (u32)kFinThreads, "one thread per classify workgroup");
    __shared__ union { FinalizeLists lists; u64 run_key[kStageRun]; } lds;
    FinalizeLists &ls = lds.lists;
    u64 *const run_key = lds.run_key;
    extern __shared__ u32 list_m[];             // finalize_claim(g) bytes
    u32 *const run_idx = list_m;
    u32 (*h)[256] = reinterpret_cast<u32 (*)[256]>(list_m + kStageRun);
    __shared__ u32 scan32[3 * kFinWaves + 1];
    __shared__ u64 scratch[2];
    __shared__ u32 extra_m, sure_extra;
    __shared__ unsigned long long gt_extra;
    __shared__ u32 run_chunk, run_before, run_index, run_found;
    __shared__ u32 run_sure[kFinWaves][kUnitChunksMax];

    const u32 tid = threadIdx.x;
    const u32 wave = tid / kWave, lane = lane_id();
    // (These loads first: a wait for the control words before them is a trip more, 0.5 us.)
    const bool in_grid = tid < g.G3;
    uint2 counts = make_uint2(0u, 0u);
    if (kCounted && g.small != 0u && blockIdx.x == 0u) {
        // (should it not do, every thread of row 0 has its classify workgroup's counts)
        OwnEntries own(g.G3, blk_lists, m_ent, b_ent);
        if (__builtin_expect(finalize_small(g, seed, ctl, ls, own, win_cnt, quad_win, m_ent, b_ent, quad_base), 1)) return;
        if (in_grid) counts = own.counts;
        lds_barrier();
    } else if (in_grid) {
        counts = blk_lists[tid];
    }
    const u32 mode = ctl->mode;
    const bool dense = (mode & 1u) != 0u, partial = (mode & 2u) != 0u;
    const u32 bd_lo = ctl->bd_lo, bd_hi = ctl->bd_hi, bd_bits = ctl->bd_bits;
    const u64 c_def = ctl->c_def;
    Candidates cand{seg, s_ent, a, g.d, g.C, g.U, g.UC, dense};
    // Whether what the exact selections walk holds every member of the top-r set. Otherwise (S as
    // a keying stream left it) the members above the bracket whose key lies above the window are
    // missing.
    auto holds_all = [&] { return dense || g.take_all != 0u || g.keyed == 0u || g.all_members != 0u; };
    // Fills the slices of chunks first, first + step, ... again, from the vector and with every
    // element at or above the deciding bin: one pass over the vector (four rows of a chunk in
    // flight), after which S will do for all the passes of an exact selection and for emit. The
    // keys are left to be computed. (By one wavefront, which sees what it wrote itself.)
    // A chunk's slice goes back to its fixed place, over whatever slices the stream left there: this
    // may only run where nobody reads a slice of the stream's any more, that is after a barrier that
    // all readers have passed, and all chunks have to be refilled. Where some workgroups give up at a
    // barrier and others go on to refill, both layouts overlap: the call then ends with kErrBarrier (workgroup
    // 0 misses those that left at the next barrier, if it did not give up itself) and emit reads nothing.
    auto complete_slices = [&](u32 first, u32 step) {
        constexpr u32 kRows = 4;
        const u64 below = lanes_below();
        for (u32 sc = first; sc < g.W; sc += step) {
            const float *chunk = a + (u64)sc * g.C;
            const u32 len = cand.length(sc);
            const u32 start = sc * g.cap;
            uint2 *slice = s_ent + start;
            u32 kept = 0;
            for (u32 r0 = 0; r0 < len; r0 += kRows * kChunkQuantum) {
                u32 bits[kRows][4];
                if (r0 + kRows * kChunkQuantum <= len) {
                    const f32x4u *row = reinterpret_cast<const f32x4u *>(chunk + r0) + lane;
#pragma unroll
                    for (u32 q = 0; q < kRows; ++q) {
                        const f32x4 v = row[q * kWave];
#pragma unroll
                        for (u32 e = 0; e < 4; ++e) bits[q][e] = __float_as_uint(v[e]);
                    }
                } else {
#pragma unroll
                    for (u32 q = 0; q < kRows; ++q)
#pragma unroll
                        for (u32 e = 0; e < 4; ++e) {
                            const u32 at = r0 + q * kChunkQuantum + 4u * lane + e;
                            bits[q][e] = at < len ? __float_as_uint(chunk[at]) : 0u;
                        }
                }
#pragma unroll
                for (u32 q = 0; q < kRows; ++q) {
                    const u32 place = r0 + q * kChunkQuantum + 4u * lane;
                    bool hit[4];
                    u64 b[4];
#pragma unroll
                    for (u32 e = 0; e < 4; ++e) {
                        hit[e] = place + e < len && mag_of(bits[q][e]) >= bd_lo;
                        b[e] = __ballot(hit[e]);
                    }
                    u32 p = kept + popc64(b[0] & below) + popc64(b[1] & below) + popc64(b[2] & below) +
                            popc64(b[3] & below);
#pragma unroll
                    for (u32 e = 0; e < 4; ++e)
                        if (hit[e]) {
                            if (p < g.cap) slice[p] = make_uint2((kKeyUnknown << 30) | (place + e), bits[q][e]);
                            ++p;
                        }
                    kept += popc64(b[0]) + popc64(b[1]) + popc64(b[2]) + popc64(b[3]);
                }
            }
            if (lane == 0) seg[chunk_slot(sc, g.U, g.UC)] = make_uint2(kept | (kept > g.cap ? kSliceFull : 0u), start);
        }
        wait_own_memory();
    };
    // every candidate, split wavefront by chunk; f(index, pattern, chunk)
    auto each_s = [&](auto &&f) {
        // kWave consecutive chunks per wavefront at a time: their sizes in one round of
        // loads, then their entries as one flat sequence, four iterations fetched together
        for (u32 first = wave * kWave; first < g.W; first += kFinWaves * kWave) {
            const ChunkWalk<kWave> walk(cand, first, 1u, g.W);
            walk.for_each(cand, [&](bool valid, u32 i, u32 idx, u32 bits, u32, u32, u32) {
                if (valid) f(idx, bits, first + i);
            });
            auto of_row = [&](bool valid, u32 i, u32 idx, u32 bits) {
                if (valid) f(idx, bits, first + i);
            };
            walk.for_each_vector_row(cand, each_of_row(of_row));
        }
    };

    // ---- everything the short-list path needs has been fetched in one round ------
    const u32 vm = counts.x & 0xFFFFu, vb = counts.x >> 16, vs = counts.y;
    const bool overflow = ctl->overflow != 0u, overflow_m = ctl->overflow_m != 0u;
    if (tid == 0) { extra_m = 0u; sure_extra = 0u; gt_extra = 0ull; run_found = 0u; }
    // The three totals (every workgroup of the grid needs them to decide whether
    // it stays) and, from the same partial sums, where this thread's classify
    // workgroup's entries start in the two lists: one exchange, every wavefront
    // adds up the sixteen partial sums for itself.
    u32 n_m0, n_bd, em, eb;
    u64 sure_walk;
    {
        const u32 im = wave_inclusive_sum(vm), ib = wave_inclusive_sum(vb), wsure = wave_sum(vs);
        if (lane == kWave - 1) { scan32[wave] = im; scan32[kFinWaves + wave] = ib; scan32[2 * kFinWaves + wave] = wsure; }
        static_assert(kFinWaves <= kWave, "one lane per wavefront's partial sum");
        lds_barrier();
        const u32 pm = lane < kFinWaves ? scan32[lane] : 0u;
        const u32 pb = lane < kFinWaves ? scan32[kFinWaves + lane] : 0u;
        n_m0 = wave_sum(pm);
        n_bd = wave_sum(pb);
        sure_walk = wave_sum(lane < kFinWaves ? scan32[2 * kFinWaves + lane] : 0u);
        em = wave_sum(lane < wave ? pm : 0u) + im - vm;
        eb = wave_sum(lane < wave ? pb : 0u) + ib - vb;
        lds_barrier();
    }

    // the magnitude of an entry of B
    auto mag_in_b = [&](u32 x) { return kCounted ? bd_lo | (x & 0xFFFFu) : x; };
    const u64 need2 = g.r - c_def;
    u32 err = 0, path = 0;
    bool have_t = false, have_k = false, ok = true;
    u32 T = 0, I_star = 0, J_star = 0xFFFFFFFFu, n_mm = 0;
    u64 K_star = ~0ull, count_greater = 0;

    if (g.all_members) {
        // r == d: the "threshold" is the whole vector; only the key cut is found
        have_t = true;
        T = 0u;
        I_star = 0xFFFFFFFFu;
    }
    const bool lists = !dense && !partial && !overflow && (g.all_members || (c_def < g.r && need2 <= n_bd));
    // The list B overflowed but M did not, and every entry of the deciding bin has
    // the same magnitude: the last member is the need2-th of them in index order.
    bool tie_run = false;
    if (__builtin_expect(!dense && overflow && !overflow_m && !g.all_members && c_def < g.r, 0)) {
        const u32 vmin = in_grid ? blk_bmin[tid] : 0xFFFFFFFFu, vmax = in_grid ? blk_bmax[tid] : 0u;
        const u32 lo = wave_min(vmin), hi = wave_max(vmax);
        if (lane == 0) { scan32[wave] = lo; scan32[kFinWaves + wave] = hi; }
        lds_barrier();
        const u32 all_lo = wave_min(lane < kFinWaves ? scan32[lane] : 0xFFFFFFFFu);
        const u32 all_hi = wave_max(lane < kFinWaves ? scan32[kFinWaves + lane] : 0u);
        lds_barrier();
        tie_run = all_lo == all_hi;
        if (tie_run) T = all_lo;
    }
    // ---- many workgroups or one? Every workgroup of the grid decides alike,
    //      from what classify and pick left: the lists cannot give the
    //      threshold (the estimate kept too little; it lies above the bracket; the
    //      deciding bin crowded by several magnitudes), or the key window certainly missed.
    bool wide = false;
    if (gridDim.x > 1u) {
        const bool slow_t = !g.all_members && !lists && !tie_run;
        bool slow_k = false;
        if (!g.take_all && !tie_run) {
            const u64 from_b = (g.all_members || !lists) ? 0ull : (need2 < n_bd ? need2 : (u64)n_bd);
            slow_k = dense || overflow_m || (g.all_members && overflow) || sure_walk >= g.k ||
                     sure_walk + n_m0 + from_b < g.k;
        }
        wide = slow_t || slow_k;
        if (!wide && blockIdx.x != 0u) return;
    }
    if (__builtin_expect(wide, 0)) {
        // ---- exact selection over all candidates, on all workgroups of the grid
        Wide w{wide_ws, gridDim.x, 0u, 0u, true, kWideSpinLimit};
        if (g.force_abort != 0u || !grid_check_in(w, &h[3][4])) {
            // the grid's workgroups cannot be resident together right now (another
            // stream's grid holds compute units and waits as well): nothing has been
            // done yet, workgroup 0 runs the selection alone below
            if (blockIdx.x != 0u) return;
            wide = false;
        }
    }
    if (__builtin_expect(wide, 0)) {
        // (diagnostics: with no patience at all the barriers time out, the kernel ends
        // with the error flag set and every workgroup still leaves normally)
        Wide w{wide_ws, gridDim.x, 1u, 0u, true, g.force_timeout != 0u ? 0u : kWideSpinLimit};
        // r == d: S only holds the coordinates whose key the window admits, and every
        // coordinate is a member: the vector itself is walked, here and by the emit kernel
        if (g.all_members) cand.dense = true;
        bool whole = holds_all();
        const u32 n_waves = gridDim.x * kFinWaves;
        // f(valid, index, pattern) for every entry of this workgroup's chunks, all lanes
        // together; done(s) after the last entry of chunk s. Wavefront v of the grid takes
        // chunks v, v + n_waves, ...; a chunk read from the vector is streamed with
        // 16-byte loads, four rows in flight.
        auto wide_each = [&](auto &&f, auto &&done) {
            for (u32 sc = blockIdx.x * kFinWaves + wave; sc < g.W; sc += n_waves) {
                bool fv = false;
                u32 start = 0;
                const u32 n_e = cand.count(sc, &start, &fv);
                if (!fv) {
                    for (u32 j0 = 0; j0 < n_e; j0 += kWave) {
                        const u32 j = j0 + lane;
                        u32 idx = 0, bits = 0, key = 0;
                        if (j < n_e) cand.entry(sc, start, j, false, &idx, &bits, &key);
                        f(j < n_e, idx, bits);
                    }
                } else {
                    const u64 c0 = (u64)sc * g.C;
                    u32 j0 = 0;
                    for (; j0 + 4 * kChunkQuantum <= n_e; j0 += 4 * kChunkQuantum) {
                        const f32x4u *p4 = reinterpret_cast<const f32x4u *>(a + c0 + j0) + lane;
                        f32x4 v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = p4[q * kWave];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const u32 i0 = (u32)(c0 + j0) + (u32)q * kChunkQuantum + 4u * lane;
                            f(true, i0, __float_as_uint(v[q].x));
                            f(true, i0 + 1u, __float_as_uint(v[q].y));
                            f(true, i0 + 2u, __float_as_uint(v[q].z));
                            f(true, i0 + 3u, __float_as_uint(v[q].w));
                        }
                    }
                    for (; j0 < n_e; j0 += kWave) {
                        const u32 j = j0 + lane;
                        const u32 bits = j < n_e ? __float_as_uint(a[c0 + j]) : 0u;
                        f(j < n_e, (u32)(c0 + j), bits);
                    }
                }
                done(sc);
            }
        };
        auto nothing = [](u32) {};
        path = 1u | 8u;
        // where whoever comes across a selected string in a later pass leaves it whole
        u64 *found_t = w.ws->found[kWidePasses - 2], *found_k = w.ws->found[kWidePasses - 1];
        const bool in_bin_only = !g.all_members && !dense;
        auto complete = [&] {
            complete_slices(blockIdx.x * kFinWaves + wave, n_waves);     // the chunks wide_each gives this wavefront
            whole = true;
        };
        // (complete lists that show fewer than k members with a key the window admits)
        if (!whole && (partial || (lists && sure_walk + n_m0 + need2 < g.k))) complete();
        const u32 top = in_bin_only ? bd_hi : 0x7FFFFFFFu;
        Selected sel_t{0ull, 0u, 12}, sel_k{0ull, 0u, 12};
        Pair96 tbound{~0ull, 0xFFFFFFFFu}, kbound{~0ull, 0xFFFFFFFFu};
        if (!g.all_members) {
            // the r-th (magnitude desc, index asc): inside the deciding bin when pick found
            // one, over the whole vector when the estimate had kept too little
            auto each_mag = [&](auto &&f2) {
                wide_each([&](bool valid, u32 idx, u32 bits) {
                    const u32 m = mag_of(bits);
                    const bool on = valid && (!in_bin_only || (m >= bd_lo && m <= bd_hi));
                    f2(on, (u64)(top - (on ? m : top)), idx);
                }, nothing);
            };
            u64 less = 0;
            sel_t = grid_select96(each_mag, in_bin_only ? need2 : g.r,
                                  in_bin_only ? (64 - (int)bd_bits) / 8 : 4, w, h, &less, &ok);
            if (!ok) err |= kErrSelect;
            tbound = sel_t.bound();
            count_greater = (in_bin_only ? c_def : 0ull) + less;
        }
        // members: above the deciding bin, or at or below the selected string in
        // (magnitude desc, index asc) order
        auto is_member_w = [&](u32 idx, u32 bits) {
            if (g.all_members != 0u) return true;
            const u32 m = mag_of(bits);
            if (m > top) return true;
            if (in_bin_only && m < bd_lo) return false;
            return pair_le((u64)(top - m), idx, tbound);
        };
        if (!g.take_all && w.alive) {
            // Members whose key the window admits are all in S: where they number k or more
            // (a list overflowed, the window missed low) they decide; their number shows in
            // the first pass.
            auto each_key = [&](auto &&f2) {
                wide_each([&](bool valid, u32 idx, u32 bits) {
                    bool on = valid && is_member_w(idx, bits);
                    const u64 key = on ? sample_key(idx, seed) : 0ull;
                    on = on && (whole || key <= g.K_hi);
                    f2(on, key, idx);
                }, nothing);
            };
            bool ok_k = true;
            for (;;) {
                u64 less = 0;
                sel_k = grid_select96(each_key, g.k, 0, w, h, &less, &ok_k);
                if (ok_k || whole || !w.alive) break;
                complete();
            }
            if (!ok_k) err |= kErrSelect;
            kbound = sel_k.bound();
        }
        // winners per chunk (every chunk's counter is written: what classify left is
        // stale); the same pass leaves the two selected strings whole for workgroup 0
        if (w.alive) {
            u32 mine = 0;
            wide_each([&](bool valid, u32 idx, u32 bits) {
                if (!valid || !is_member_w(idx, bits)) return;
                const u32 m = mag_of(bits);
                if (sel_t.bytes < 12 && m <= top && sel_t.is((u64)(top - m), idx)) {
                    __hip_atomic_store(&found_t[0], (u64)(top - m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&found_t[1], (u64)idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (g.take_all != 0u) { ++mine; return; }
                const u64 key = sample_key(idx, seed);
                if (!pair_le(key, idx, kbound)) return;
                ++mine;
                if (sel_k.bytes < 12 && sel_k.is(key, idx)) {
                    __hip_atomic_store(&found_k[0], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&found_k[1], (u64)idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }, [&](u32 sc) {
                const u32 total = wave_sum(mine);
                if (lane == 0)
                    __hip_atomic_store(&win_cnt[sc], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                mine = 0;
            });
            grid_barrier(w, &h[3][4]);
        }
        if (w.alive && blockIdx.x == 0u) {
            Pair96 ts{sel_t.hi, sel_t.lo}, ks{sel_k.hi, sel_k.lo};
            if (sel_t.bytes < 12) {
                ts.hi = __hip_atomic_load(&found_t[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ts.lo = (u32)__hip_atomic_load(&found_t[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (sel_k.bytes < 12) {
                ks.hi = __hip_atomic_load(&found_k[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ks.lo = (u32)__hip_atomic_load(&found_k[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!g.all_members) { T = top - (u32)ts.hi; I_star = ts.lo; }
            if (!g.take_all) { K_star = ks.hi; J_star = ks.lo; }
        }
        if (!w.alive) err |= kErrBarrier;
        if (blockIdx.x != 0u) return;
        have_t = true;
        have_k = true;
        if (g.all_members && tid == 0) ctl->emit_dense = 1u;
    }

    // ---- the short lists decide, in LDS. What bounds this is latency: one workgroup's chain of trips
    //      to memory and barriers, and the few hundred cold lines that one compute unit fetches at
    //      0.4 a ns. So an entry of a list is 8 bytes (M: where in the window its key lies, not the key,
    //      which only the entries in the cut's own bin need), winners per chunk are read and added up by
    //      quads of chunks, and either cut is one pass over bins. Kernel, us, against lists of keys
    //      (16 and 12 bytes an entry, more than 8,192 keys in memory), a counter per chunk and a radix selection byte by
    //      byte: one vector of 200,003 elements 12.7 -> 10.0, of 2^20 14.0 -> 10.5, of 25.6 M 18.1 -> 12.8, top-k
    //      and random-k of 11.2 M 12.2 -> 8.5 and 17.2 -> 11.8, four of 2^28 (20,500 keys) 104 -> 35. (The loops
    //      that note an entry's place, where crowded chunks leave 128 entries to one thread, go four at a
    //      time: 65,536 elements with touched rows 12.4 -> 10.8, one at a time 12.8.)
    uint4 qw[kSlabs];
    auto load_quads = [&](auto &&load) {
#pragma unroll
        for (u32 q = 0; q < kSlabs; ++q) {
            const u32 x = 4u * (q * kFinThreads + tid);
            qw[q] = make_uint4(0u, 0u, 0u, 0u);
            if (x * kQuad < g.W) qw[q] = load(x);
        }
    };
    bool quick = false;         // what the lists add to the quads is in ls.won
    constexpr u32 kNotSent = 0xFFFFFFFFu, kSurelySent = 0xFFFFFFFEu;
    if (__builtin_expect(!wide && lists && n_bd <= kStageB && n_m0 <= g.stage_m, 1)) {
        const bool with_b = !g.all_members;
        for (u32 i = tid; i < kCutM / 2u; i += kFinThreads) ls.bin_m[i] = 0u;
        if (tid < kCutB) ls.bin_b[tid] = 0u;
        for (u32 i = tid; i < (g.W + 2u * kQuad - 1u) / (2u * kQuad) + 1u && i < kQuads / 2u; i += kFinThreads) ls.won[i] = 0u;
        if (tid < (u32)kWave) { ls.group_b[tid] = 0u; ls.group_m[tid] = 0u; }
        if (tid == 0) { ls.n_cand_b = 0u; ls.n_cand_m = 0u; }
        // Entry j of classify workgroup t lives at [j][t]. First every thread notes where the
        // entries of its workgroup are (a hot layer may sit in one workgroup's lists), then all fetch them.
#pragma unroll 4
        for (u32 j = 0; j < vb; ++j) ls.b_idx[eb + j] = j * g.G3 + tid;
#pragma unroll 4
        for (u32 j = 0; j < vm; ++j) list_m[em + j] = j * g.G3 + tid;
        lds_barrier();
        const CutBins<kCutB / kWave, false> cut_b{ls.bin_b, ls.group_b};
        const CutBins<kCutM / kWave, true> cut_m{ls.bin_m, ls.group_m};
        const u32 chunk_shift = 31u - (u32)__clz((int)g.C), shift_b = bd_bits > 10u ? bd_bits - 10u : 0u;
        static_assert(kCutB == 1u << 10, "bits of a bin of B");
        auto word_m = [&](u32 at, u32 idx) { return at << kChunkBits | idx >> chunk_shift; };
        constexpr u32 kAhead = 4;
#pragma unroll 1
        for (u32 p0 = tid; p0 < n_m0; p0 += kAhead * kFinThreads) {
            uint2 e[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 p = p0 + q * kFinThreads;
                e[q] = m_ent[p < n_m0 ? list_m[p] : 0u];
            }
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 p = p0 + q * kFinThreads;
                if (p < n_m0) { list_m[p] = word_m(e[q].x, e[q].y); cut_m.add(e[q].x); }
            }
        }
        if (with_b)
#pragma unroll 1
            for (u32 p = tid; p < n_bd; p += kFinThreads) {
                const uint2 e = b_ent[ls.b_idx[p]];
                const u32 x = bd_hi - mag_in_b(e.x);
                ls.b_x[p] = x;
                ls.b_idx[p] = e.y;
                cut_b.add(x >> shift_b);
            }
        load_quads([&](u32 x) { return reinterpret_cast<const uint4 *>(quad_win)[x / 4u]; });
        lds_barrier();
        // ---- exact threshold inside the deciding bin
        Pair96 tb{~0ull, 0xFFFFFFFFu};
        if (with_b) {
            u32 at, rank, here;
            cut_b.find((u32)need2, &at, &rank, &here);
            auto each_here = [&](auto &&f) {
#pragma unroll 1
                for (u32 p = tid; p < n_bd; p += kFinThreads)
                    if (ls.b_x[p] >> shift_b == at) f(p);
            };
            if (__builtin_expect(here <= (u32)kWave, 1)) {
                each_here([&](u32 p) { ls.cand[atomicAdd(&ls.n_cand_b, 1u)] = p; });
                lds_barrier();
                // (only the wavefronts that hold entries of B, and the first one, need the outcome: with all
                // sixteen ranking, four to a SIMD, the call waited for the issue of it)
                if (wave * (u32)kWave < n_bd || wave == 0u) {
                    const u32 p = lane < here ? ls.cand[lane] : 0u;
                    bool up_to;
                    tb = wave_rank(ls.b_x[p], ls.b_idx[p], here, rank, &up_to);
                }
                lds_barrier();                  // (the candidates of the key cut come next)
            } else {
                // many share it (a few levels): byte by byte, the bits that differ only (with
                // histograms in the place of the counters of B, which every wavefront has looked at)
                static_assert(kCutB >= 4 * 256, "histograms of block_select96");
                lds_barrier();
                const u64 low = (1ull << shift_b) - 1ull;
                const u32 idx_shift = g.d > 1ull ? (u32)__clz((int)(u32)(g.d - 1ull)) : 31u;
                tb = block_select96([&](auto &&f) {
                    each_here([&](u32 p) { f((u64)ls.b_x[p] & low, ls.b_idx[p] << idx_shift); });
                }, rank, (64 - (int)shift_b) / 8, reinterpret_cast<u32 (*)[256]>(ls.bin_b), scratch, &ok);
                if (!ok) err |= kErrSelect;
                tb = Pair96{(u64)at << shift_b | tb.hi, tb.lo >> idx_shift};
            }
            T = bd_hi - (u32)tb.hi;
            I_star = tb.lo;
            // ---- its members: a key decides between certain winner, one more entry of M, and nothing
            u32 my_gt = 0, my_sure = 0, my_extra = 0;
#pragma unroll 1
            for (u32 p = tid; p < n_bd; p += kFinThreads) {
                const u32 x = ls.b_x[p], idx = ls.b_idx[p];
                bool sure = pair_le((u64)x, idx, tb);
                my_gt += (u64)x < tb.hi ? 1u : 0u;
                u32 standing = kNotSent;
                if (sure && g.take_all == 0u) {
                    const u64 key = sample_key(idx, seed);
                    sure = key < g.K_lo;
                    if (!sure && key <= g.K_hi) {
                        standing = (u32)(((key - g.K_lo) << g.k_nlz) >> (64 - kWindowBits));
                        cut_m.add(standing);
                        ++my_extra;
                    }
                }
                if (sure) { standing = kSurelySent; ++my_sure; }
                ls.b_x[p] = standing;            // from here on: these two, or where in the window its key lies
            }
            my_extra = wave_sum(my_extra);
            if (lane == 0 && my_extra) atomicAdd(&extra_m, my_extra);
            my_gt = wave_sum(my_gt);
            my_sure = wave_sum(my_sure);
            if (lane == 0 && my_gt) atomicAdd(&gt_extra, (unsigned long long)my_gt);
            if (lane == 0 && my_sure) atomicAdd(&sure_extra, my_sure);
            lds_barrier();
        }
        have_t = true;
        count_greater = c_def + gt_extra;
        n_mm = n_m0 + extra_m;
        const u64 c_klo = sure_walk + sure_extra;
        u32 at = 0, rank = 0, here = 0;
        if (g.take_all) {
            quick = true;
        } else if (c_klo < g.k && g.k - c_klo <= n_mm) {
            cut_m.find((u32)(g.k - c_klo), &at, &rank, &here);
            quick = here <= (u32)kWave;         // (a 4096th of the window with more keys: as if the lists had not fitted)
        }
        if (__builtin_expect(quick, 1)) {
            // a winner of chunk sc: one more in its quad and (for emit) in the chunk
            auto won = [&](u32 sc) {
                const u32 x = sc / kQuad;
                atomicAdd(&ls.won[x / 2u], 1u << (16u * (x & 1u)));
                atomicAdd(&win_cnt[sc], 1u);
            };
            if (with_b)
#pragma unroll 1
                for (u32 p = tid; p < n_bd; p += kFinThreads) {
                    const u32 standing = ls.b_x[p], idx = ls.b_idx[p];
                    if (standing == kSurelySent || (standing != kNotSent && standing < at)) {
                        won(idx >> chunk_shift);
                    } else if (standing != kNotSent && standing == at) {
                        const u32 j = atomicAdd(&ls.n_cand_m, 1u);
                        ls.cand[j] = kNotSent;          // (not in M)
                        ls.cand_idx[j] = idx;
                    }
                }
            if (!g.take_all) {
#pragma unroll 1
                for (u32 p = tid; p < n_m0; p += kFinThreads) {
                    const u32 w = list_m[p];
                    if (w >> kChunkBits == at) ls.cand[atomicAdd(&ls.n_cand_m, 1u)] = p;
                    else if (w >> kChunkBits < at) won(w & ((1u << kChunkBits) - 1u));
                }
                lds_barrier();
                // the candidates' indices: whoever has the candidate's list fetches its entry again
#pragma unroll 1
                for (u32 j = 0; j < here; ++j) {
                    const u32 p = ls.cand[j];
                    if (p != kNotSent && p - em < vm) ls.cand_idx[j] = m_ent[(u64)(p - em) * g.G3 + tid].y;
                }
                lds_barrier();
                if (wave == 0u) {
                    const u32 idx = lane < here ? ls.cand_idx[lane] : 0u;
                    bool up_to;
                    const Pair96 kb = wave_rank((sample_key(idx, seed) - g.K_lo) << g.k_nlz, idx, here, rank, &up_to);
                    if (up_to) won(idx >> chunk_shift);
                    K_star = (kb.hi >> g.k_nlz) + g.K_lo;
                    J_star = kb.lo;
                }
            }
            have_k = true;
        } else {
            have_t = false;
            ok = true;
            lds_barrier();                      // (everybody has read the counts)
            if (tid == 0) { extra_m = 0u; sure_extra = 0u; gt_extra = 0ull; }
        }
        lds_barrier();
    }

    // The lists that do not fit LDS, and a run of equal magnitudes at the threshold: in memory.
    if (__builtin_expect(!wide && !quick && (lists || tie_run), 0)) {
        u64 *bk = db_key, *mk = dm_key;
        u32 *bi = db_idx, *mi = dm_idx;
        const u32 m_cap = 2u * g.G3 * kListCap;
        // as above: where the entries are, then the entries (M's keys are made here)
        if (lists) for (u32 j = 0; j < vb; ++j) bi[eb + j] = j * g.G3 + tid;
        for (u32 j = 0; j < vm; ++j) mi[em + j] = j * g.G3 + tid;
        __syncthreads();
        if (lists)
            for (u32 p = tid; p < n_bd; p += kFinThreads) {
                const uint2 e = b_ent[bi[p]];
                bk[p] = (u64)(bd_hi - mag_in_b(e.x));
                bi[p] = e.y;
            }
        if (kCounted) __syncthreads();          // (a long list of B reaches into where M's keys go)
        for (u32 p = tid; p < n_m0; p += kFinThreads) {
            const u32 idx = m_ent[mi[p]].y;
            mk[p] = (sample_key(idx, seed) - g.K_lo) << g.k_nlz;
            mi[p] = idx;
        }
        __syncthreads();
        auto each_b = [&](auto &&f) {
            for (u32 p = tid; p < n_bd; p += kFinThreads) f(bk[p], bi[p]);
        };
        Pair96 tb{0ull, 0u};
        if (__builtin_expect(tie_run, 0)) {
            // ---- the chunk that holds the need2-th entry of the run: thread t
            //      adds up the counts of chunks 32t .. 32t+31 ---------------------
            path = 4;
            constexpr u32 kPer = kTargetChunks / kFinThreads;
            static_assert(kPer % 4 == 0, "whole 16-byte groups of counters per thread");
            u32 mine = 0;
#pragma unroll
            for (u32 q = 0; q < kPer / 4; ++q) {
                const u32 s = tid * kPer + 4u * q;
                uint4 v = make_uint4(0u, 0u, 0u, 0u);
                if (s < g.W) v = reinterpret_cast<const uint4 *>(bd_cnt)[s / 4];
                mine += v.x + (s + 1 < g.W ? v.y : 0u) + (s + 2 < g.W ? v.z : 0u) +
                        (s + 3 < g.W ? v.w : 0u);
            }
            // (the entries of the bin number at most d < 2^32)
            const u32 before = block_exclusive_sum(mine, scan32);
            if ((u64)before < need2 && need2 <= (u64)before + mine) {
                run_chunk = tid * kPer;          // first of the kPer chunks that hold it
                run_before = before;
                run_found = 1u;
            }
            lds_barrier();
            if (wave == 0 && run_found != 0u) {
                // the counters of those chunks again, one per lane
                static_assert(kPer <= kWave, "one lane per counter");
                const u32 s0 = run_chunk, b0 = run_before;
                const u32 s = s0 + lane;
                const u32 c = (lane < kPer && s < g.W) ? bd_cnt[s] : 0u;
                const u32 inc = wave_inclusive_sum(c);
                if ((u64)b0 + (inc - c) < need2 && need2 <= (u64)b0 + inc) {
                    run_chunk = s;
                    run_before = b0 + (inc - c);
                }
            }
            lds_barrier();
            ok = run_found != 0u;
            if (ok) {
                // ---- the entry of that rank inside the chunk, 1024 entries a round
                const u32 sc = run_chunk;
                const u32 want = (u32)(need2 - run_before);      // 1-based, among the chunk's
                bool sc_vec = false;
                u32 start = 0;
                const u32 n_e = cand.count(sc, &start, &sc_vec);
                lds_barrier();
                if (tid == 0) run_found = 0u;
                u32 seen = 0;
                for (u32 j0 = 0; j0 < n_e && seen < want; j0 += kFinThreads) {
                    const u32 j = j0 + tid;
                    u32 idx = 0, bits = 0, key = 0;
                    if (j < n_e) cand.entry(sc, start, j, sc_vec, &idx, &bits, &key);
                    const u32 m = mag_of(bits);
                    const u32 flag = (j < n_e && m >= bd_lo && m <= bd_hi) ? 1u : 0u;
                    const u32 excl = block_exclusive_sum(flag, scan32);
                    const u32 round_total = scan32[kFinWaves];
                    if (flag && seen + excl + 1u == want) { run_index = idx; run_found = 1u; }
                    seen += round_total;
                    lds_barrier();
                }
                ok = run_found != 0u;
                I_star = run_index;
            }
            if (!ok) { T = 0; path = 0; }
        } else if (!g.all_members) {
            // ---- exact threshold inside the deciding bin --------------------
            tb = block_select96(each_b, need2, (64 - (int)bd_bits) / 8, h, scratch, &ok);
        }
        if (ok) {
            have_t = true;
            if (lists && !g.all_members) {
                T = bd_hi - (u32)tb.hi;
                I_star = tb.lo;
            }
            // ---- members of the deciding bin join the key lists; the atomics
            //      on the chunk counters are left in flight --------------------
            // join(idx, on_sure): idx is a member; its key decides between "certain
            // winner" (on_sure is called), the key list M, or nothing
            auto join = [&](u32 idx, auto &&on_sure) {
                if (g.take_all != 0u) { on_sure(); return; }
                const u64 key = sample_key(idx, seed);
                if (key < g.K_lo) {
                    on_sure();
                } else if (key <= g.K_hi) {
                    const u32 q = atomicAdd(&extra_m, 1u);
                    if (n_m0 + q < m_cap) {
                        mk[n_m0 + q] = (key - g.K_lo) << g.k_nlz;
                        mi[n_m0 + q] = idx;
                    }
                }
            };
            u32 my_gt = 0;
            if (__builtin_expect(lists, 1)) {
                each_b([&](u64 hi, u32 idx) {
                    if (hi < tb.hi) ++my_gt;
                    if (pair_le(hi, idx, tb))
                        join(idx, [&] { atomicAdd(&win_cnt[idx / g.C], 1u); atomicAdd(&sure_extra, 1u); });
                });
            } else {
                // the run's members: its entries up to index I*, all in chunks 0 .. run_chunk.
                // They may be many per chunk: certain winners are counted per chunk in LDS
                // and reach the chunk's counter as one addition.
                const u32 s_end = run_chunk + 1u;
                u32 my_sure = 0;
                for (u32 first = wave * kUnitChunksMax; first < s_end; first += kFinWaves * kUnitChunksMax) {
                    if (lane < kUnitChunksMax) run_sure[wave][lane] = 0u;
                    __builtin_amdgcn_wave_barrier();
                    const UnitWalk walk(cand, first, 1u, s_end);
                    auto run_member = [&](bool valid, u32 i, u32 idx, u32 bits) {
                        const u32 m = mag_of(bits);
                        if (valid && m >= bd_lo && m <= bd_hi && idx <= I_star)
                            join(idx, [&] { atomicAdd(&run_sure[wave][i], 1u); ++my_sure; });
                    };
                    walk.for_each(cand, [&](bool valid, u32 i, u32 idx, u32 bits, u32, u32, u32) {
                        run_member(valid, i, idx, bits);
                    });
                    walk.for_each_vector_row(cand, each_of_row(run_member));
                    __builtin_amdgcn_wave_barrier();
                    if (lane < kUnitChunksMax && first + lane < s_end && run_sure[wave][lane])
                        atomicAdd(&win_cnt[first + lane], run_sure[wave][lane]);
                    __builtin_amdgcn_wave_barrier();
                }
                my_sure = wave_sum(my_sure);
                if (lane == 0 && my_sure) atomicAdd(&sure_extra, my_sure);
            }
            if (my_gt) atomicAdd(&gt_extra, (unsigned long long)my_gt);
            __syncthreads();
            count_greater = c_def + gt_extra;
            n_mm = n_m0 + extra_m;
            if (n_mm <= kStageRun && n_mm <= m_cap) {
                // short after all: the selection below reads it several times, from LDS then
                for (u32 p = tid; p < n_mm; p += kFinThreads) { run_key[p] = mk[p]; run_idx[p] = mi[p]; }
                mk = run_key;
                mi = run_idx;
                lds_barrier();
            }
            const u64 c_klo = sure_walk + sure_extra;
            if (g.take_all) {
                have_k = true;
            } else if (n_mm <= m_cap && c_klo < g.k && g.k - c_klo <= n_mm) {
                auto each_m = [&](auto &&f) {
                    for (u32 p = tid; p < n_mm; p += kFinThreads) f(mk[p], mi[p]);
                };
                const Pair96 kb = block_select96(each_m, g.k - c_klo, 0, h, scratch, &ok);
                if (ok) {
                    have_k = true;
                    K_star = (kb.hi >> g.k_nlz) + g.K_lo;
                    J_star = kb.lo;
                    each_m([&](u64 key, u32 idx) {
                        if (pair_le(key, idx, kb)) atomicAdd(&win_cnt[idx / g.C], 1u);
                    });
                }
            }
        }
    }

    if (g.all_members && !have_k) {
        // r == d and a short list overflowed or the key window missed: as above
        cand.dense = true;
        if (tid == 0) ctl->emit_dense = 1u;
    }
    bool whole = holds_all();
    auto complete_alone = [&] {
        __syncthreads();
        complete_slices(wave, kFinWaves);
        __syncthreads();
        whole = true;
    };
    if (__builtin_expect(!have_t, 0)) {
        // ---- exact threshold by selection over all candidates: those of the deciding
        //      bin, or the whole vector when the estimate had kept too little ----------
        path |= 1u;
        if (partial && !whole) complete_alone();
        const u32 top = dense ? 0x7FFFFFFFu : bd_hi;
        auto each_mag = [&](auto &&f) {
            each_s([&](u32 idx, u32 bits, u32) {
                const u32 m = mag_of(bits);
                if (dense || (m >= bd_lo && m <= bd_hi)) f((u64)(top - m), idx);
            });
        };
        const Pair96 tb = block_select96(each_mag, dense ? g.r : need2, 4, h, scratch, &ok);
        if (!ok) err |= kErrSelect;
        T = top - (u32)tb.hi;
        I_star = tb.lo;
        u32 my_gt = 0;
        each_s([&](u32, u32 bits, u32) {
            const u32 m = mag_of(bits);
            if (m > T && m <= top) ++my_gt;
        });
        count_greater = (dense ? 0ull : c_def) + block_sum(my_gt, scan32);
    }
    auto is_member = [&](u32 idx, u32 bits) {
        const u32 m = mag_of(bits);
        return m > T || (m == T && idx <= I_star);
    };
    if (__builtin_expect(!have_k, 0)) {
        // ---- exact key cut and winners per chunk by selection over all candidates
        path |= 1u;
        __syncthreads();
        for (u32 s = tid; s < g.W; s += kFinThreads) win_cnt[s] = 0u;
        if (!g.take_all) {
            // (members whose key the window admits first, as above)
            auto each_key = [&](auto &&f) {
                each_s([&](u32 idx, u32 bits, u32) {
                    if (!is_member(idx, bits)) return;
                    const u64 key = sample_key(idx, seed);
                    if (whole || key <= g.K_hi) f(key, idx);
                });
            };
            Pair96 kb{0ull, 0u};
            for (;;) {
                kb = block_select96(each_key, g.k, 0, h, scratch, &ok);
                if (ok || whole) break;
                complete_alone();
            }
            if (!ok) err |= kErrSelect;
            K_star = kb.hi;
            J_star = kb.lo;
        } else {
            K_star = ~0ull;
            J_star = 0xFFFFFFFFu;
        }
        __syncthreads();
        const Pair96 kcut{K_star, J_star};
        each_s([&](u32 idx, u32 bits, u32 s) {
            if (is_member(idx, bits) &&
                (g.take_all || pair_le(sample_key(idx, seed), idx, kcut)))
                atomicAdd(&win_cnt[s], 1u);
        });
    }
    // (the lists' winners reach the chunks' counters meanwhile: nobody here reads those then)
    if (__builtin_expect(quick, 1)) lds_barrier(); else __syncthreads();

    // ---- output offset of every quad of chunks: thread t holds the winners of quads
    //      4*(1024*q + t) .. +3, q < kSlabs; prefix sums run slab after slab.
    if (__builtin_expect(quick, 1)) {
#pragma unroll
        for (u32 q = 0; q < kSlabs; ++q) {
            const u32 x = 4u * (q * kFinThreads + tid);
            if (x * kQuad >= g.W) continue;
            const u32 w01 = ls.won[x / 2u], w23 = ls.won[x / 2u + 1u];
            qw[q].x += w01 & 0xFFFFu;
            qw[q].y += w01 >> 16;
            qw[q].z += w23 & 0xFFFFu;
            qw[q].w += w23 >> 16;
        }
    } else {
        // From the chunks' counters: the workgroup's first read of them, after the barrier that
        // follows its atomics on them (wide: written by other workgroups of this grid, read where they
        // were written). A lane per counter, four lanes add up a quad and leave it in LDS, whose lists
        // nobody reads any more. (A lane per quad, whose loads fetch a line each: 155.7 us instead of
        // 151.4 after a missed key window at 25.6 M.)
        static_assert(kStageRun >= kQuads && kWave % kQuad == 0 && kQuad == 4, "room for the sums, whole quads per wavefront");
        u32 *sum = run_idx;
        constexpr u32 kAhead = 8;
        for (u32 s0 = 0; s0 < g.W; s0 += kAhead * kFinThreads) {
            u32 c[kAhead];
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 sc = s0 + q * kFinThreads + tid;
                c[q] = 0u;
                if (sc < g.W) c[q] = wide ? __hip_atomic_load(&win_cnt[sc], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : win_cnt[sc];
            }
#pragma unroll
            for (u32 q = 0; q < kAhead; ++q) {
                const u32 sc = s0 + q * kFinThreads + tid;
                u32 t = c[q] + __shfl_down(c[q], 1, kWave);
                t += __shfl_down(t, 2, kWave);
                if (lane % kQuad == 0u && sc < g.W) sum[sc / kQuad] = t;
            }
        }
        lds_barrier();
        load_quads([&](u32 x) { return make_uint4(sum[x], sum[x + 1u], sum[x + 2u], sum[x + 3u]); });
    }
    u32 s4[kSlabs], inc[kSlabs];
#pragma unroll
    for (u32 q = 0; q < kSlabs; ++q) {
        // (quads beyond the last chunk)
        const u32 x = 4u * (q * kFinThreads + tid);
        if ((x + 1u) * kQuad >= g.W) qw[q].y = 0u;
        if ((x + 2u) * kQuad >= g.W) qw[q].z = 0u;
        if ((x + 3u) * kQuad >= g.W) qw[q].w = 0u;
        s4[q] = qw[q].x + qw[q].y + qw[q].z + qw[q].w;
        inc[q] = wave_inclusive_sum(s4[q]);
    }
    static_assert(kSlabs * kFinWaves <= kWave, "one partial sum per lane");
    if (lane == kWave - 1) {
#pragma unroll
        for (u32 q = 0; q < kSlabs; ++q) scan32[q * kFinWaves + wave] = inc[q];
    }
    lds_barrier();
    const u32 part = lane < kSlabs * kFinWaves ? scan32[lane] : 0u;
    const u32 up_to_here = wave_inclusive_sum(part);
    const u64 total = (u32)__builtin_amdgcn_readlane((int)up_to_here, kWave - 1);
#pragma unroll
    for (u32 q = 0; q < kSlabs; ++q) {
        const u32 x = 4u * (q * kFinThreads + tid);
        const u32 before = (u32)__builtin_amdgcn_readlane((int)(up_to_here - part), (int)(q * kFinWaves + wave));
        if (x * kQuad < g.W) {
            uint4 o;
            o.x = before + inc[q] - s4[q];
            o.y = o.x + qw[q].x;
            o.z = o.y + qw[q].y;
            o.w = o.z + qw[q].z;
            reinterpret_cast<uint4 *>(quad_base)[x / 4u] = o;
        }
    }
    if (total != g.k) err |= kErrCount;
    if (tid == 0) {
        ctl->err = err;
        ctl->path = path;
        ctl->T = T;
        ctl->I_star = I_star;
        ctl->K_star = K_star;
        ctl->J_star = J_star;
        ctl->n_b = n_bd;
        ctl->n_m = n_mm;
        ctl->W = g.W;
        ctl->U = g.U;
        ctl->UC = g.UC;
        ctl->count_greater = count_greater;
        ctl->ties = g.r - count_greater;
        if (kCounted) ctl->how = !dense && bd_bits < kCountShift ? kHowNarrowed : 0u;
    }
}

// ---------------------------------------------------------------------------
// emit: members of the top-r set whose (key, index) is at or below the cut
// -> the message in index order; residual at the sent positions <- a - a.
// A winner's place is the output offset of its chunk plus the number of
// winners before it in the chunk; the latter is kept as the difference of two
// running totals over the wavefront's flat walk.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void
emit_body(Geom g, PhiloxSeed seed, const EncodeCtl *__restrict__ ctl,
       const uint2 *__restrict__ seg, const uint2 *__restrict__ s_ent,
       const u32 *__restrict__ win_cnt, const u32 *__restrict__ quad_base,
       u32 *__restrict__ out_idx, float *__restrict__ out_val, float *residual)
{
    __shared__ uint2 row_queue[kWalkWaves][kRowQueue];
    const u32 u = blockIdx.x * kWalkWaves + threadIdx.x / kWave;
    if (u >= g.U) return;
    const u32 lane = lane_id();
    const Candidates cand{seg, s_ent, residual, g.d, g.C, g.U, g.UC,
                          ((ctl->mode & 1u) | ctl->emit_dense) != 0u};
    // where the lane's chunk's winners go: after those of the quads before it and of the chunks before it
    // in its own quad. (Loaded by all lanes, those without a chunk the first quad's, before
    // anything that waits: behind a branch the two loads held the walk up for 0.1 to 0.5 us.)
    const u32 my_chunk = u + lane * g.U;
    const bool has_chunk = lane < g.UC && my_chunk < g.W;
    const u32 quad = has_chunk ? my_chunk / kQuad : 0u, in_quad = my_chunk % kQuad;
    const uint4 in_front = reinterpret_cast<const uint4 *>(win_cnt)[quad];
    const u32 of_quad = quad_base[quad];
    const u32 T = ctl->T, I_star = ctl->I_star, err = ctl->err;
    const Pair96 kcut{ctl->K_star, ctl->J_star};
    const UnitWalk walk(cand, u < g.U ? u : g.W, g.U, g.W);
    // A wait between workgroups of the selection that gave up: there are no cut points, and S may
    // be half refilled (see complete_slices), so that an entry need not lie inside its chunk.
    // (Looked at with what the first loads bring: a wait of its own at the start cost 0.5 us.)
    if ((err & kErrBarrier) != 0u) return;
    const u32 my_base = of_quad + (in_quad > 0u ? in_front.x : 0u) + (in_quad > 1u ? in_front.y : 0u) +
                        (in_quad > 2u ? in_front.z : 0u);
    const u64 below = lanes_below();
    u32 run = 0;          // winners at flat positions before this iteration
    u32 carry = 0;        // winners before the first entry of the chunk that runs into this iteration
    // With the cut inside the a-priori window the streaming kernel's word decides, but
    // for the few entries in the cut's own 4096th of the window.
    const bool in_window = g.take_all != 0u || (kcut.hi >= g.K_lo && kcut.hi <= g.K_hi);
    const u32 cut_at = (u32)(((kcut.hi - g.K_lo) << g.k_nlz) >> (64 - kWindowBits));
    auto wins = [&](bool valid, u32 idx, u32 bits, u32 key) {
        bool win = false;
        if (valid) {
            const u32 m = mag_of(bits);
            win = m > T || (m == T && idx <= I_star);
            if (win && !g.take_all) {
                const u32 says = key >> 30, at = (key >> kPlaceBits) & ((1u << kWindowBits) - 1u);
                if (__builtin_expect(!in_window || says == kKeyUnknown || (says == kKeyInside && at == cut_at), 0))
                    win = pair_le(sample_key(idx, seed), idx, kcut);
                else
                    win = says == kKeyBelow || (says == kKeyInside && at < cut_at);
            }
        }
        return win;
    };
    auto send = [&](u64 pos, u32 idx, u32 bits) {
        if (pos < g.k) {
            const float v = __uint_as_float(bits);
            out_idx[pos] = idx;
            out_val[pos] = v;
            // (a lone word in a line nobody reads again: the hint keeps it from displacing what
            // the walk still needs; eight vectors of 25.6 M elements 16.8 instead of 18.2 us)
            __builtin_nontemporal_store(v - v, residual + idx);
        }
    };
    walk.for_each(cand, [&](bool valid, u32 i, u32 idx, u32 bits, u32 key, u32 first, u32 p0) {
        const bool win = wins(valid, idx, bits, key);
        const u64 mask = __ballot(win);
        // winners before the first entry of this lane's chunk
        const u32 at_start =
            first >= p0 ? run + popc64(mask & ((1ull << (first - p0)) - 1ull)) : carry;
        const u32 base_c = __shfl(my_base, i, kWave);
        if (win) send((u64)base_c + (run + popc64(mask & below) - at_start), idx, bits);
        carry = __shfl(at_start, kWave - 1, kWave);
        run += popc64(mask);
    });
    // chunks read from the vector itself: what can be a member is gathered first,
    // then taken 64 at a time in index order; seen counts the chunk's winners so far
    u32 row_chunk = 0xFFFFFFFFu, seen = 0;
    if (__builtin_expect(walk.from_vector != 0ull, 0))
    walk.for_each_vector_entry(cand, row_queue[threadIdx.x / kWave],
                               [&](u32 bits) { return mag_of(bits) >= T; },
                               [&](bool valid, u32 i, u32 idx, u32 bits) {
        if (i != row_chunk) { row_chunk = i; seen = 0; }
        const bool win = wins(valid, idx, bits, kKeyUnknown << 30);
        const u64 mask = __ballot(win);
        if (mask == 0ull) return;
        const u32 base_c = __shfl(my_base, i, kWave);
        if (win) send((u64)base_c + seen + popc64(mask & below), idx, bits);
        seen += popc64(mask);
    });
}

// ---------------------------------------------------------------------------
// The kernels. One launch serves up to kMaxBatch independent vectors of the
// same sizes ("members": the workers of one node, or the tensors of one
// model): blockIdx.z is the member, and every member has its own workspace,
// ws_stride bytes after the previous one. Each member is computed exactly as
// if it were alone; batching only lets the short kernels of all members run
// side by side and the streaming kernel run on without draining in between.
// ---------------------------------------------------------------------------
constexpr u32 kMaxBatch = 16;

struct Batch {
    const float *grad[kMaxBatch];
    float *residual[kMaxBatch];
    u32 *out_idx[kMaxBatch];
    float *out_val[kMaxBatch];
    u32 seed_lo[kMaxBatch], seed_hi[kMaxBatch];
    u32 step_lo, step_hi;
    const u64 *step_dev;        // when not null, the step number is read from here instead
    char *ws;
    u64 ws_stride;
};

// what the workgroup's member works on
struct Member {
    const float *grad;
    float *residual;
    u32 *out_idx;
    float *out_val;
    PhiloxSeed seed;
    char *ws;
    __device__ __forceinline__ Member(const Batch &B)
    {
        const u32 i = blockIdx.z;
        grad = B.grad[i];
        residual = B.residual[i];
        out_idx = B.out_idx[i];
        out_val = B.out_val[i];
        u32 step_lo = B.step_lo, step_hi = B.step_hi;
        if (B.step_dev) {
            const u64 step = *B.step_dev;
            step_lo = (u32)step;
            step_hi = (u32)(step >> 32);
        }
        seed = PhiloxSeed{B.seed_lo[i], B.seed_hi[i], step_lo, step_hi};
        ws = B.ws + (u64)i * B.ws_stride;
    }
    template <class T>
    __device__ __forceinline__ T *at(u64 offset) const { return reinterpret_cast<T *>(ws + offset); }
};

__global__ void __launch_bounds__(kSampleThreads) k_sample(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    sample_body(m.grad, m.residual, g, m.seed, m.at<u32>(0), (u32)(L.zero_bytes / 4),
                m.at<u32>(L.samples));
}

template <u32 kVecs>
__global__ void __launch_bounds__(kEstThreads) k_estimate(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    estimate_body<kVecs>(m.at<u32>(L.samples), g, m.at<EncodeCtl>(L.ctl));
}

template <bool kAll, int kRows, bool kKeyed>
__global__ void __launch_bounds__(kFusedThreads) k_fused(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    fused_body<kAll, kRows, kKeyed>(m.grad, m.residual, g, m.seed, m.at<EncodeCtl>(L.ctl),
                            (u32)(L.zero_bytes / 4), m.at<u32>(L.partials), m.at<u32>(L.group_sums), m.at<uint2>(L.seg),
                            m.at<uint2>(L.s_ent));
}

__global__ void __launch_bounds__(kPickThreads) k_pick(Batch B, u32 n_rows, Geom g, EncodeLayout L)
{
    const Member m(B);
    EncodeCtl *ctl = m.at<EncodeCtl>(L.ctl);
    const Picked p = pick_body(m.at<u32>(L.partials), m.at<u32>(L.group_sums), n_rows, g, ctl);
    if (threadIdx.x == 0) p.store(ctl);
}

__global__ void __launch_bounds__(kWalkThreads) k_classify(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    classify_body(g, m.seed, m.at<EncodeCtl>(L.ctl), m.residual, m.at<uint2>(L.seg),
                  m.at<uint2>(L.s_ent), m.at<u32>(L.win_cnt), m.at<u32>(L.bd_cnt), m.at<u32>(L.quad_win),
                  m.at<uint2>(L.blk_lists), m.at<u32>(L.blk_bmin), m.at<u32>(L.blk_bmax),
                  m.at<uint2>(L.m_ent), m.at<uint2>(L.b_ent));
}

__global__ void __launch_bounds__(kCountThreads) k_count(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    const u32 group_words = (part_groups(g.G3) + 1u) * (u32)(sizeof(PartGroup) / 4u);
    count_body(m.grad, m.residual, g, m.at<u32>(0), (u32)(L.zero_bytes / 4), m.at<u32>(L.group_sums), group_words, m.at<u16>(L.samples), m.at<uint4>(L.partials));
}

__global__ void __launch_bounds__(kPickThreads) k_pick_counted(Batch B, u32 n_rows, Geom g, EncodeLayout L)
{
    const Member m(B);
    __shared__ u32 hot;
    Picked p = pick_counted<kPickThreads>(m.at<u16>(L.samples), m.at<uint4>(L.partials), n_rows, g, &hot);
    lds_barrier();
    if (hot != 0u) p.n_bin |= kCrowds;
    if (threadIdx.x == 0) {
        EncodeCtl *ctl = m.at<EncodeCtl>(L.ctl);
        p.store(ctl);
        ctl->n_bin = p.n_bin;
    }
}

template <bool kPick>
__global__ void __launch_bounds__(kWalkThreads) k_classify_counted(Batch B, u32 n_rows, u32 narrow_from, Geom g, EncodeLayout L)
{
    const Member m(B);
    EncodeCtl *ctl = m.at<EncodeCtl>(L.ctl);
    const ChunkRows chunk(m.residual, g.d, blockIdx.x * kWalkWaves + threadIdx.x / kWave);
    __shared__ u32 hot;
    Picked p{};
    if (kPick)
        p = pick_counted<kWalkThreads>(m.at<u16>(L.samples), m.at<uint4>(L.partials), n_rows, g, &hot);
    else
        p = Picked{ctl->mode, ctl->bd_lo, ctl->bd_hi, ctl->c_def, ctl->n_bin};
    classify_counted(chunk, g, m.seed, ctl, p, hot, kPick, narrow_from, m.residual, m.at<PartGroup>(L.group_sums), m.at<uint2>(L.seg), m.at<uint2>(L.s_ent), m.at<u32>(L.win_cnt),
                     m.at<u32>(L.bd_cnt), m.at<u32>(L.quad_win), m.at<uint2>(L.blk_lists), m.at<u32>(L.blk_bmin),
                     m.at<u32>(L.blk_bmax), m.at<uint2>(L.m_ent), m.at<uint2>(L.b_ent));
}

template <bool kCounted>
__global__ void __launch_bounds__(kFinThreads) k_finalize(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    finalize_body<kCounted>(g, m.seed, m.at<EncodeCtl>(L.ctl), m.at<WideScratch>(L.wide), m.residual,
                  m.at<uint2>(L.seg), m.at<uint2>(L.s_ent), m.at<u32>(L.win_cnt), m.at<u32>(L.bd_cnt),
                  m.at<u32>(L.quad_win), m.at<uint2>(L.blk_lists), m.at<u32>(L.blk_bmin), m.at<u32>(L.blk_bmax),
                  m.at<uint2>(L.m_ent), m.at<uint2>(L.b_ent), m.at<u64>(L.dm_key),
                  m.at<u32>(L.dm_idx), m.at<u64>(L.db_key), m.at<u32>(L.db_idx),
                  m.at<u32>(L.quad_base));
}

__global__ void __launch_bounds__(kWalkThreads) k_emit(Batch B, Geom g, EncodeLayout L)
{
    const Member m(B);
    emit_body(g, m.seed, m.at<EncodeCtl>(L.ctl), m.at<uint2>(L.seg), m.at<uint2>(L.s_ent),
              m.at<u32>(L.win_cnt), m.at<u32>(L.quad_base), m.out_idx, m.out_val, m.residual);
}

// ---------------------------------------------------------------------------
// Calibration (diagnostics): a = g + m into the residual buffer and nothing
// else, over the same chunks, with the same accesses, in the same order and
// on the same grid as the fused kernel: the speed of the bare read-read-write
// stream.
// ---------------------------------------------------------------------------
template <int kRows>
__global__ void __launch_bounds__(kFusedThreads)
k_stream_add(const float *__restrict__ grad, float *__restrict__ residual, u64 d, u32 C, u32 W)
{
    constexpr u32 kGroup = kRows * kChunkQuantum;
    const u32 n_waves = blockDim.x / kWave, wave_stride = gridDim.x * n_waves;
    f32x4 gv[kRows], mv[kRows];
    auto load = [&](u64 base) {
        const f32x4u *gp = reinterpret_cast<const f32x4u *>(grad + base) + lane_id();
        const f32x4u *mp = reinterpret_cast<const f32x4u *>(residual + base) + lane_id();
#pragma unroll
        for (int q = 0; q < kRows; ++q) {
            gv[q] = __builtin_nontemporal_load(gp + q * kWave);
            mv[q] = __builtin_nontemporal_load(mp + q * kWave);
        }
    };
    auto add = [&](u64 base, f32x4 (&a)[kRows]) {
#pragma unroll
        for (int q = 0; q < kRows; ++q) a[q] = gv[q] + mv[q];
        f32x4u *mp = reinterpret_cast<f32x4u *>(residual + base) + lane_id();
#pragma unroll
        for (int q = 0; q < kRows; ++q) __builtin_nontemporal_store((f32x4u)a[q], mp + q * kWave);
    };
    const u32 w_full = (u32)(d / C);
    u32 w = blockIdx.x * n_waves + threadIdx.x / kWave;
    if (w < w_full) {
        u64 c0 = (u64)w * C, base = c0;
        load(base);
        for (;;) {
            f32x4 a[kRows];
            add(base, a);
            const bool last = base - c0 + kGroup >= C;
            const u32 w_next = last ? w + wave_stride : w;
            const u64 next = last ? (u64)w_next * C : base + kGroup;
            if (w_next >= w_full) break;
            load(next);
            if (last) c0 = next;
            w = w_next;
            base = next;
        }
        while (w < w_full) w += wave_stride;
    }
    if (w == w_full && w < W) {
        u64 base = (u64)w * C;
        bool more = base + kGroup <= d;
        if (more) load(base);
        while (more) {
            f32x4 a[kRows];
            add(base, a);
            base += kGroup;
            more = base + kGroup <= d;
            if (more) load(base);
        }
        for (u64 i = base + lane_id(); i < d; i += kWave) residual[i] = grad[i] + residual[i];
    }
}

}  // namespace rtopk

// ===========================================================================
// C ABI
// ===========================================================================
using namespace rtopk;

static int check_sizes(uint64_t d, uint64_t r, uint64_t k)
{
    // domain of Definition 3, with 32-bit indices
    if (k < 1 || k > r || r > d || d > 0xFFFFFFFFull) return RTOPK_EINVAL;
    return RTOPK_OK;
}

extern "C" int rtopk_encode_workspace_bytes(uint64_t d, uint64_t r, uint64_t k, uint64_t *bytes)
{
    if (!bytes) return RTOPK_EINVAL;
    const int rc = check_sizes(d, r, k);
    if (rc) return rc;
    *bytes = make_layout(make_geom(d, r, k)).total;
    return RTOPK_OK;
}

namespace {
struct TraceRequest {
    int stage = 0;
    hipEvent_t begin = nullptr, end = nullptr;
};
thread_local TraceRequest g_trace;
thread_local unsigned g_force = 0;

// records the requested pair of events around one stage of the pipeline
struct StageScope {
    const TraceRequest &tr;
    hipStream_t stream;
    bool on;
    StageScope(const TraceRequest &t, int stage, hipStream_t s)
        : tr(t), stream(s), on(t.stage == stage)
    {
        if (on) (void)hipEventRecord(tr.begin, stream);
    }
    ~StageScope()
    {
        if (on) (void)hipEventRecord(tr.end, stream);
    }
};

// Workgroups of the streaming kernel: one per compute unit (all start
// together and share the chunks evenly, so none waits for a slot) of 4 to 12
// wavefronts (fused_shape), each with one row of 256 elements of both arrays on
// its way, two rows in a short vector. Two or three workgroups per unit stream
// no faster, leave three times the histogram rows to add up and less room for
// kernels of other streams.
// The count of units is looked up at the first call on the device.
constexpr int kMaxDevices = 64;
constexpr int kFusedBlocksPerCU = 1;
// A batched launch holds several times that grid (one grid per member). Left
// to itself the device then keeps three workgroups of different members on
// every compute unit, and the interleaved streams cost 8% (443 instead of
// 407 us for eight vectors of 25.6 M elements). Each workgroup therefore also
// claims more than half of the unit's 160 KB of LDS, most of which it does not use: one
// workgroup per unit at any time, members streamed one after the other. (Short vectors,
// whose workgroups only hold a chunk per wavefront, run side by side instead.)
constexpr unsigned kFusedLdsClaim = 96u * 1024u;
std::mutex g_device_mutex;
unsigned g_fused_grid[kMaxDevices], g_classify_grid[kMaxDevices];

template <class K>
bool allow_lds_claim(K kernel, unsigned bytes = kFusedLdsClaim)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}

// Wavefronts per workgroup of the streaming kernel, and its grid. A vector of up to 2048
// chunks is one chunk per wavefront. Above, short vectors are a few rounds of chunks (more
// wavefronts, fewer rounds), long ones stream best with least in flight. Measured (us, a
// launch with 8, 10, 12 wavefronts): five vectors of 11.2 M elements 131, 123, 116;
// eight of 25.6 M 419, 391, 399; four of 66 M 534, 524, 550; four of 134 M 1067, 1117,
// 1112; four of 2^28 2372, 2510, 2554. Whole calls for one vector: 3 M 54.6, 57.0, 53.1;
// 11.2 M 74.7, 72.6, 70.4; 40 M 140, 134.5, 142; 66 M 199, 194, 199; 100 M 276, 283, 281.5;
// 134 M 353, 364, 368. (What fits exactly is a saw-tooth in the number of chunks: 13 M runs 3%
// faster with 10, 134 M + 1 and 180 M 3% faster with 10 than with 8.)
// Between one round of 12 wavefronts (3072 chunks) and two of 8 (4096), a second round that is
// a third full or less costs more than the shape of the short vectors with two chunks per
// wavefront: one vector of 3.5 M 53.9 / 50.4 (r = d: 38.5 / 33.6), of 4 M 52.7 / 51.8, sixteen
// of 4 M 210.6 / 202.4, four of 4 M 88.9 / 91.1 (none of them keyed); just above 3072 chunks
// 47.3 / 49.3. A batch gains by that shape below 3072 chunks too, as its members run side by
// side: from kShortBatch chunks in all. k_fused of four vectors of 2.4 M 28.2 / 23.5; calls of
// sixteen of 2.2 M 7% faster, of four of 2.6 M 2-5%, of three 0-4% slower.
constexpr u32 kShortBatch = 9216;
struct FusedShape { unsigned threads, grid, lds; bool is_short; };
FusedShape fused_shape(u32 W, u64 d, unsigned nb, unsigned grid_limit)
{
    const bool is_short = W <= 2048u || (W > 3072u && W <= 4096u) || (W <= 3072u && nb * W >= kShortBatch);
    unsigned waves = W <= 512u ? 4u : is_short ? 8u : d < (1ull << 24) ? 12u : d <= (1ull << 26) ? 10u : 8u;
    unsigned grid = (W + waves - 1) / waves;
    return FusedShape{waves * (unsigned)kWave, grid > grid_limit ? grid_limit : grid,
                      is_short ? waves * kRing * (unsigned)sizeof(uint2) : kFusedLdsClaim, is_short};
}

// Whether the stream computes the candidates' keys (and leaves out what will not be sent).
// Those of a long vector always: they take the time in which the stream waits for memory. A
// short vector's stream has nothing to hide them behind, but where a launch's members have
// many, the classify and emit kernels do less for it. us, unkeyed / keyed: one vector of
// 300,007 elements, r = 1%, 34.7 / 36.7; eight of 2 M, r = 1% (160,000 in all), 81.3 / 79.3; five of
// 950,000, r = 5% (238,000), 53.3 / 51.6; sixteen of 2 M, r = 10%, 170 / 151; touched rows, four of
// a million, r = 5%, 54.3 / 50.6. Layered vectors, whose crowded chunks have no others of their wavefront to
// take room from, lose up to 2.5% by keys there (five of 950,000 56.1 / 57.4; four of 2 M, r = 10%, 75.6 / 77.3).
// From an eighth of the vector on every chunk overflows (sixteen of 2 M, r = 20%: 187.7 / 187.5). r == d,
// where the stream computes every element's key to know the candidates: one vector of 300,007 23.1 / 25.5, two of
// 3.5 M 44.5 / 44.9; eight of 2 M, k = 1%, 69.4 / 66.8, sixteen of 1 M 69.8 / 67.5.
// (Vectors that are counted go by the same rule: their classify kernel leaves out what a keying stream would. The
// figures of the shorter ones are those of streams that kept their candidates.)
constexpr u64 kKeyedMembers = 1u << 17, kKeyedElements = 1u << 23;
bool keys_in_stream(const Geom &g, bool is_short, unsigned nb)
{
    if (!is_short) return true;
    if (g.all_members) return nb * g.d >= kKeyedElements;
    return nb * g.r >= kKeyedMembers && g.r * kSliceDiv < g.d;
}

// How the chunks are dealt to the wavefronts: workgroup by workgroup (neighbouring wavefronts of one
// workgroup stream neighbouring chunks) or across the workgroups, so that the last, incomplete round of
// chunks is a few wavefronts of every compute unit and not all wavefronts of some. us, by workgroup /
// across: one vector of 11.2 M elements 67.0 / 66.2, of 21 M 90.8 / 88.6, of 25.6 M 97.8 / 95.5, of 40 M
// 131.0 / 128.7, of 66 M 183.7 / 182.6, but of 100 M 263.9 / 271.3 and of 180 M 452 / 457; a batch, which
// has no incomplete round but the last member's, loses locality: four of 11.2 M 140.4 / 144.0, eight of 5 M
// 136 / 146, four of 66 M 610 / 623, eight of 25.6 M 472 / 471. With r == d the keys are what a unit is busy with, in
// a batch too: one of 11.2 M 51.9 / 48.8, of 66 M 206.6 / 197.1, eight of 11.2 M 255.8 / 247.5; four of 6 M 90.2 / 90.7.
constexpr u64 kAcrossMax = 1u << 26, kAcrossKeyed = 1u << 23;
bool deals_across(const Geom &g, bool is_short, unsigned nb)
{
    if (is_short) return false;
    return g.all_members ? g.d >= kAcrossKeyed : nb == 1u && g.d <= kAcrossMax;
}

// Whether a vector's magnitudes are all counted (count_body): short vectors. Whole calls, us, by sample,
// estimate and candidates / counted: one vector of 65,536 elements 38.9 / 23.9, of 200,003 32.9 / 24.0, of
// 2^20 36.8 / 28.2, of 2 M, r = 0.5%, 44.7 / 35.8 (layered), of 3 M 45.8 / 38.9; four of 2 M 61.5 / 52.7,
// sixteen of 2^20 81.7 / 74.7, of 2 M 120 / 112, of 3 M 158 / 153. A bin is a 128th of an octave: of normal values at most
// 0.38% of all elements lie in one, 1 to 6% of the top r by where the threshold lies between two powers of two, which
// is a longer list for finalize than a bracket's bins leave. So r is limited where that costs more than the launches save.
// Normal values at eight scales, before / now from the least to the most favourable, without narrow_bin: 3.1 M, r = 32,000
// 1.10-1.15, 98,000 0.74-0.99; 3 M, r = 60,000 0.84-1.10; 2 M, r = 64,000
// 1.08-1.20, 130,000 0.80-1.17; 1.5 M, r = 64,000 1.10-1.16; 1.3 M, r = 200,000 0.95-1.16; 2^20, any r 1.17-1.25. Values
// with lighter tails have no such bound; their bins are narrowed (see there: from 2 M elements on they gain little, at 3 M
// uniform values lose 4%; a few levels of 2^20, r = 1%, lose 5%, uniform values eight at a time 2%). Above 3072 chunks the vector's second
// reading costs what the launches save, and hot chunks want the room that the stream's wavefronts share.
constexpr u32 kCountMid = 2048;               // chunks (kCountAnyR: with the sizes of the sample)
constexpr u64 kCountMidMembers = 1u << 16, kCountMembers = 1u << 15;
bool counts_all(const Geom &g)
{
    if (g.all_members || g.W > kCountChunks) return false;
    return g.W <= kCountAnyR || g.r <= (g.W <= kCountMid ? kCountMidMembers : kCountMembers);
}

// Workgroups of count: as many wavefronts as chunks, in few rows of bins (every workgroup that picks the deciding
// bin reads them all). us, 4 / 8 / 16 wavefronts: one vector of 200,003 27.4 / 26.7 / 27.3, of 524,288 30.3 / 29.5 /
// 30.7, eight of 524,288 45.3 / 41.3 / 40.0; 8 / 16: one of 2^20 30.1 / 30.0, four 42.5 / 39.5.
struct CountShape { unsigned threads, grid; };
CountShape count_shape(u32 W)
{
    const unsigned waves = W <= 512u ? 8u : kCountThreads / kWave, each = W <= kCountRows * waves ? waves : kCountEach;
    return CountShape{waves * (unsigned)kWave, (W + each - 1) / each};
}
// Whether the short lists are likely to be in reach of OwnEntries: eight times what a classify workgroup leaves on
// average, of the window's keys (most of stage_m) and of the deciding bin (a twentieth of the top r for
// normal values); a batch of many, which the slowest member holds up, only where next to every place is in reach. Calls, us, with
// the lists in LDS / in registers: one vector of 65,536 elements 23.6 / 20.8, of 200,003 24.4 / 21.7, layered,
// r = 2%, 30.1 / 28.4, of 524,288 25.8 / 24.6, of 2^20 28.0 / 25.9, layered 28.0 / 27.3, touched rows 27.7 / 28.4; eight of
// 200,003 29.0 / 28.1, of 2^20 49.9 / 50.5. Where the attempt fails (touched rows, whose keys are in few workgroups;
// lighter tails) it costs 0.7 to 1.7: 2^20, r = 2%, 33.0 / 34.6.
bool small_lists(const Geom &g, unsigned nb)
{
    if (g.G3 > kSmallBlocks || (nb > 2u && g.G3 > kSmallBlocks / 4u)) return false;
    const u64 room = (u64)OwnEntries::deep(OwnEntries::columns(g.G3)) * g.G3;
    return g.r / 20 * 8 <= room && (u64)g.stage_m * 8 <= room;
}

// The entries of the deciding bin from which on classify narrows it down wherever they are: more than finalize has room
// for (4,089 of 2^20 uniform values 34.1, narrowed 31.8, but eight at a time 62.8 and 68.1), or, of a vector of few classify
// workgroups, 96 to each, whose lists hold 384 (200,003 elements, 1,493 entries: 29.8, narrowed 30.0; 20,000 elements, 150
// entries 26.0, narrowed 29.7).
u32 narrows_from(u32 G3)
{
    const u32 spread = G3 * kListCap * 3u / 4u;
    return (spread < kStageB ? spread : kStageB) + 1u;
}

// Every classify workgroup picks for itself up to this many rows over all members, a kernel picks beyond. us, in
// classify / by a kernel: one of 200,003 (25 rows) 26.7 / 28.9, of 2^21 (128) 37.2 / 38.9; two of 2^21 44.0 / 43.6; four
// of 2^20 (64) 39.5 / 40.5, of 1.5 M (92) 50.9 / 47.8; eight of 524,288 (64) 41.3 / 41.5, of 2^20 55.1 / 52.6.
constexpr unsigned kPickRows = 256;

// workgroups of the streaming kernel in a launch at most, and workgroups of a counted vector's classify that the
// device holds at once
int fused_grid_limit(unsigned *out, unsigned *classify_out = nullptr)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return RTOPK_EHIP;
    std::lock_guard<std::mutex> lock(g_device_mutex);
    if (g_fused_grid[dev] == 0) {
        int cus = 0, fit_t = 0, fit_f = 0, fit_c = 0, fit_p = 0;
        if (!allow_lds_claim(k_fused<false, kLongRows, true>) || !allow_lds_claim(k_fused<false, kShortRows, true>) ||
            !allow_lds_claim(k_fused<true, kLongRows, true>) || !allow_lds_claim(k_stream_add<kLongRows>) ||
            !allow_lds_claim(k_finalize<false>, 4u * kStageM) || !allow_lds_claim(k_finalize<true>, 4u * kStageM))
            return RTOPK_EHIP;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit_t, k_fused<false, kShortRows, true>,
                                                         (int)kFusedThreads,
                                                         kFusedLdsClaim) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit_f, k_fused<true, kLongRows, true>,
                                                         (int)kFusedThreads,
                                                         kFusedLdsClaim) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit_c, k_classify_counted<false>, (int)kWalkThreads, 0) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit_p, k_classify_counted<true>, (int)kWalkThreads, 0) != hipSuccess)
            return RTOPK_EHIP;
        int per_cu = fit_t < fit_f ? fit_t : fit_f;
        per_cu = per_cu < kFusedBlocksPerCU ? per_cu : kFusedBlocksPerCU;
        if (cus < 1 || per_cu < 1) return RTOPK_EHIP;
        const unsigned grid = (unsigned)cus * (unsigned)per_cu;
        g_fused_grid[dev] = grid > kMaxFusedBlocks ? kMaxFusedBlocks : grid;
        g_classify_grid[dev] = (unsigned)cus * (unsigned)(fit_c < fit_p ? fit_c : fit_p);
    }
    *out = g_fused_grid[dev];
    if (classify_out) *classify_out = g_classify_grid[dev];
    return RTOPK_OK;
}
}  // namespace

extern "C" int rtopk_force_next_encode(unsigned flags)
{
    if (flags & ~(unsigned)(RTOPK_FORCE_ESTIMATE_MISS | RTOPK_FORCE_KEY_WINDOW_MISS |
                            RTOPK_FORCE_CHECK_IN_ABORT | RTOPK_FORCE_BRACKET_LOW |
                            RTOPK_FORCE_BARRIER_TIMEOUT))
        return RTOPK_EINVAL;
    g_force = flags;
    return RTOPK_OK;
}

extern "C" int rtopk_trace_next_encode(int stage, void *ev_begin, void *ev_end)
{
    if (stage != 0 && (!ev_begin || !ev_end)) return RTOPK_EINVAL;
    g_trace.stage = stage;
    g_trace.begin = (hipEvent_t)ev_begin;
    g_trace.end = (hipEvent_t)ev_end;
    return RTOPK_OK;
}

#define RTOPK_LAUNCH_CHECK()                              \
    do {                                                  \
        if (hipGetLastError() != hipSuccess) return RTOPK_EHIP; \
    } while (0)

static int encode_batch_impl(uint32_t n, const float *const *grad, float *const *residual,
                             uint64_t d, uint64_t r, uint64_t k, const uint64_t *seed,
                             uint64_t step, const uint64_t *step_dev, uint32_t *const *out_idx,
                             float *const *out_val, void *workspace, uint64_t workspace_bytes,
                             void *stream_v)
{
    if (n < 1 || !grad || !residual || !seed || !out_idx || !out_val) return RTOPK_EINVAL;
    const int rc = check_sizes(d, r, k);
    if (rc) return rc;
    for (uint32_t i = 0; i < n; ++i) {
        if (!grad[i] || !residual[i] || !out_idx[i] || !out_val[i]) return RTOPK_EINVAL;
        const uintptr_t g0 = (uintptr_t)grad[i], m0 = (uintptr_t)residual[i];
        if (g0 < m0 + d * 4 && m0 < g0 + d * 4) return RTOPK_EINVAL;
    }
    Geom g = make_geom(d, r, k);
    const EncodeLayout L = make_layout(g);
    if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes / n < L.total)
        return RTOPK_EWORKSPACE;
    const unsigned force = g_force;
    g_force = 0;
    // a forced estimate miss belongs to the general path; a forced window miss is
    // honoured on the r == d path too (it then walks the vector itself)
    if (force & RTOPK_FORCE_ESTIMATE_MISS) g.all_members = 0u;
    if (force & RTOPK_FORCE_ESTIMATE_MISS) g.force_dense = 1u;
    if (force & RTOPK_FORCE_CHECK_IN_ABORT) g.force_abort = 1u;
    if (force & RTOPK_FORCE_BRACKET_LOW) g.force_low = 1u;
    if (force & RTOPK_FORCE_BARRIER_TIMEOUT) g.force_timeout = 1u;
    if ((force & RTOPK_FORCE_KEY_WINDOW_MISS) && !g.take_all) {
        g.K_lo = g.K_hi = 0;       // a window that holds no key: the exact selection must run
        g.k_nlz = 63u;
    }
    // (a bracket that ends too low belongs to the path that has one, which vectors of up to kCountAnyR chunks never take)
    const bool force_bracket = (force & RTOPK_FORCE_BRACKET_LOW) != 0u && g.W > kCountAnyR;
    hipStream_t stream = (hipStream_t)stream_v;
    unsigned grid_limit = 0, classify_limit = 0;
    const int rc2 = fused_grid_limit(&grid_limit, &classify_limit);
    if (rc2) return rc2;
    const TraceRequest trace = g_trace;
    g_trace = TraceRequest{};
    StageScope whole(trace, RTOPK_STAGE_ALL, stream);

    for (uint32_t first = 0; first < n; first += kMaxBatch) {
        const unsigned nb = n - first < kMaxBatch ? n - first : kMaxBatch;
        Geom gg = g;                    // this launch group's share-out of the walking kernels
        set_units(gg, nb);
        set_samples(gg, nb);
        const FusedShape fs = fused_shape(g.W, g.d, nb, grid_limit);
        const unsigned fgrid = fs.grid;
        gg.keyed = keys_in_stream(gg, fs.is_short, nb) ? 1u : 0u;
        const u32 stream_waves = fgrid * (fs.threads / (unsigned)kWave);
        gg.each = g.W / stream_waves;
        gg.over = g.W % stream_waves;
        gg.spread = deals_across(gg, fs.is_short, nb) ? 1u : 0u;
        Batch B{};
        for (unsigned i = 0; i < nb; ++i) {
            B.grad[i] = grad[first + i];
            B.residual[i] = residual[first + i];
            B.out_idx[i] = out_idx[first + i];
            B.out_val[i] = out_val[first + i];
            B.seed_lo[i] = (u32)seed[first + i];
            B.seed_hi[i] = (u32)(seed[first + i] >> 32);
        }
        B.step_lo = (u32)step;
        B.step_hi = (u32)(step >> 32);
        B.step_dev = step_dev;
        B.ws = (char *)workspace + (u64)first * L.total;
        B.ws_stride = L.total;
        const dim3 fg(fgrid, 1, nb);
        const bool counts = !force_bracket && counts_all(gg);
        const CountShape cs = count_shape(gg.W);
        if (counts) set_units(gg, 1u);                  // a chunk per wavefront of the walking kernels
        gg.small = counts && small_lists(gg, nb) ? 1u : 0u;
        // (0: never)
        const u32 narrow_from = counts && gg.G3 <= classify_limit && gg.force_abort == 0u ? narrows_from(gg.G3) : 0u;
        if (counts) {
            { StageScope none(trace, RTOPK_STAGE_PREPARE, stream); }    // (nothing to prepare: the events are recorded all the same)
            StageScope sc(trace, RTOPK_STAGE_FUSED, stream);
            k_count<<<dim3(cs.grid, 1, nb), cs.threads, 0, stream>>>(B, gg, L);
            RTOPK_LAUNCH_CHECK();
        } else if (g.all_members) {
            // r == d (random-k): no estimate, no histogram, no threshold
            StageScope sc(trace, RTOPK_STAGE_FUSED, stream);
            if (fs.is_short && !gg.keyed)
                k_fused<true, kShortRows, false><<<fg, fs.threads, 0, stream>>>(B, gg, L);
            else if (fs.is_short)
                k_fused<true, kShortRows, true><<<fg, fs.threads, fs.lds, stream>>>(B, gg, L);
            else
                k_fused<true, kLongRows, true><<<fg, fs.threads, fs.lds, stream>>>(B, gg, L);
            RTOPK_LAUNCH_CHECK();
        } else {
            {
                StageScope sc(trace, RTOPK_STAGE_PREPARE, stream);
                const dim3 eg(1, 1, nb);
                static_assert(kSampleLoc == 16 * kEstThreads, "one kernel for each power of two");
                k_sample<<<dim3(gg.est_vecs * kEstThreads / kSampleThreads, 1, nb), kSampleThreads, 0, stream>>>(
                    B, gg, L);
                RTOPK_LAUNCH_CHECK();
                switch (gg.est_vecs) {
                case 1: k_estimate<1><<<eg, kEstThreads, 0, stream>>>(B, gg, L); break;
                case 2: k_estimate<2><<<eg, kEstThreads, 0, stream>>>(B, gg, L); break;
                case 4: k_estimate<4><<<eg, kEstThreads, 0, stream>>>(B, gg, L); break;
                case 8: k_estimate<8><<<eg, kEstThreads, 0, stream>>>(B, gg, L); break;
                default: k_estimate<16><<<eg, kEstThreads, 0, stream>>>(B, gg, L); break;
                }
                RTOPK_LAUNCH_CHECK();
            }
            {
                StageScope sc(trace, RTOPK_STAGE_FUSED, stream);
                if (fs.is_short && !gg.keyed)
                    k_fused<false, kShortRows, false><<<fg, fs.threads, 0, stream>>>(B, gg, L);
                else if (fs.is_short)
                    k_fused<false, kShortRows, true><<<fg, fs.threads, fs.lds, stream>>>(B, gg, L);
                else
                    k_fused<false, kLongRows, true><<<fg, fs.threads, fs.lds, stream>>>(B, gg, L);
                RTOPK_LAUNCH_CHECK();
            }
        }
        {
            StageScope sc(trace, RTOPK_STAGE_CLASSIFY, stream);
            const dim3 cg(gg.G3, 1, nb);
            const bool each_picks = nb * cs.grid <= kPickRows;
            if (counts && each_picks) {
                k_classify_counted<true><<<cg, kWalkThreads, 0, stream>>>(B, cs.grid, narrow_from, gg, L);
            } else if (counts) {
                k_pick_counted<<<dim3(1, 1, nb), kPickThreads, 0, stream>>>(B, cs.grid, gg, L);
                RTOPK_LAUNCH_CHECK();
                k_classify_counted<false><<<cg, kWalkThreads, 0, stream>>>(B, cs.grid, narrow_from, gg, L);
            } else {
                if (!g.all_members) {
                    k_pick<<<dim3(1, 1, nb), kPickThreads, 0, stream>>>(B, fgrid, gg, L);
                    RTOPK_LAUNCH_CHECK();
                }
                k_classify<<<cg, kWalkThreads, 0, stream>>>(B, gg, L);
            }
            RTOPK_LAUNCH_CHECK();
        }
        {
            StageScope sc(trace, RTOPK_STAGE_FINALIZE, stream);
            // long vectors: enough workgroups for the exact fallback over all candidates
            // (all but the first leave at once when the short lists decide)
            // (the kernel's workgroups are resident one per compute unit: a batch shares them)
            unsigned fin_grid = 1u;
            if (g.W >= kWideMinChunks) {
                fin_grid = 256u / nb;
                fin_grid = fin_grid > kWideBlocks ? kWideBlocks : (fin_grid < 16u ? 16u : fin_grid);
            }
            const dim3 ng(fin_grid, 1, nb);
            if (counts)
                k_finalize<true><<<ng, kFinThreads, finalize_claim(gg), stream>>>(B, gg, L);
            else
                k_finalize<false><<<ng, kFinThreads, finalize_claim(gg), stream>>>(B, gg, L);
            RTOPK_LAUNCH_CHECK();
        }
        {
            StageScope sc(trace, RTOPK_STAGE_EMIT, stream);
            k_emit<<<dim3(gg.G3, 1, nb), kWalkThreads, 0, stream>>>(B, gg, L);
            RTOPK_LAUNCH_CHECK();
        }
    }
    return RTOPK_OK;
}

extern "C" int rtopk_encode_batch(uint32_t n, const float *const *grad, float *const *residual,
                                  uint64_t d, uint64_t r, uint64_t k, const uint64_t *seed,
                                  uint64_t step, uint32_t *const *out_idx, float *const *out_val,
                                  void *workspace, uint64_t workspace_bytes, void *stream_v)
{
    return encode_batch_impl(n, grad, residual, d, r, k, seed, step, nullptr, out_idx, out_val,
                             workspace, workspace_bytes, stream_v);
}

extern "C" int rtopk_encode_batch_device_step(uint32_t n, const float *const *grad,
                                              float *const *residual, uint64_t d, uint64_t r,
                                              uint64_t k, const uint64_t *seed,
                                              const uint64_t *step_device,
                                              uint32_t *const *out_idx, float *const *out_val,
                                              void *workspace, uint64_t workspace_bytes,
                                              void *stream_v)
{
    if (!step_device || ((uintptr_t)step_device & 7u)) return RTOPK_EINVAL;
    return encode_batch_impl(n, grad, residual, d, r, k, seed, 0, step_device, out_idx, out_val,
                             workspace, workspace_bytes, stream_v);
}

extern "C" int rtopk_encode(const float *grad, float *residual, uint64_t d, uint64_t r,
                            uint64_t k, uint64_t seed, uint64_t step, uint32_t *out_idx,
                            float *out_val, void *workspace, uint64_t workspace_bytes,
                            void *stream_v)
{
    return rtopk_encode_batch(1, &grad, &residual, d, r, k, &seed, step, &out_idx, &out_val,
                              workspace, workspace_bytes, stream_v);
}

extern "C" int rtopk_diag_stream_add(const float *grad, float *residual, uint64_t d,
                                     void *stream_v)
{
    if (!grad || !residual || d < 1 || d > 0xFFFFFFFFull) return RTOPK_EINVAL;
    const uintptr_t g0 = (uintptr_t)grad, m0 = (uintptr_t)residual;
    if (((g0 | m0) & 15u) || (g0 < m0 + d * 4 && m0 < g0 + d * 4)) return RTOPK_EINVAL;
    const Geom g = make_geom(d, d, d);                     // the chunking only
    unsigned grid_limit = 0;
    const int rc = fused_grid_limit(&grid_limit);
    if (rc) return rc;
    const FusedShape fs = fused_shape(g.W, g.d, 1u, grid_limit);
    if (fs.is_short)
        k_stream_add<kShortRows><<<fs.grid, fs.threads, 0, (hipStream_t)stream_v>>>(grad, residual, d, g.C, g.W);
    else
        k_stream_add<kLongRows><<<fs.grid, fs.threads, fs.lds, (hipStream_t)stream_v>>>(grad, residual, d, g.C, g.W);
    RTOPK_LAUNCH_CHECK();
    return RTOPK_OK;
}

extern "C" int rtopk_encode_stats(const void *workspace, void *stream_v,
                                  rtopk_encode_stats_t *host_out)
{
    if (!workspace || !host_out) return RTOPK_EINVAL;
    hipStream_t stream = (hipStream_t)stream_v;
    if (hipStreamSynchronize(stream) != hipSuccess) return RTOPK_EHIP;
    EncodeCtl c;
    if (hipMemcpy(&c, workspace, sizeof c, hipMemcpyDeviceToHost) != hipSuccess)
        return RTOPK_EHIP;
    // candidates kept by the streaming kernel: the chunk sizes, added up here
    uint64_t superset = 0;
    if (c.W > 0 && c.W <= kTargetChunks && c.U > 0 && c.UC > 0 && (u64)c.U * c.UC <= kTargetChunks &&
        c.W <= c.U * c.UC) {
        const EncodeLayout L = make_layout(Geom{});   // the offset of seg is fixed
        std::vector<uint2> slices(kTargetChunks);
        if (hipMemcpy(slices.data(), (const char *)workspace + L.seg,
                      (size_t)kTargetChunks * sizeof(uint2), hipMemcpyDeviceToHost) != hipSuccess)
            return RTOPK_EHIP;
        for (u32 s2 = 0; s2 < c.W; ++s2) superset += slices[chunk_slot(s2, c.U, c.UC)].x & ~kSliceFull;
    }
    host_out->error_flags = c.err;
    host_out->path = c.path | (((c.mode & 1u) | c.emit_dense) != 0u ? 2u : 0u);
    host_out->threshold_bits = c.T;
    host_out->boundary_list_size = c.n_b;
    host_out->count_greater = c.count_greater;
    host_out->ties_taken = c.ties;
    host_out->superset_size = superset;
    host_out->key_list_size = c.n_m;
    return RTOPK_OK;
}
