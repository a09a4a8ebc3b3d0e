// rtopk_aggregate: the master step of Algorithm 1, ghat = (1/n) sum_i ghat_i,
// from n sorted sparse messages to one dense vector, in a single kernel.
//
// The output is cut into tiles of 2048 consecutive coordinates and every
// WAVEFRONT owns a run of consecutive tiles and an LDS copy of the tile it is
// working on; wavefronts never synchronise with each other. Lane w remembers
// how far the wavefront has come in worker w's ascending index list: where
// the wavefront's first tile starts in it is found once, by a search in which
// the 64 lanes probe several positions per worker at a time. For every tile
// and worker the wavefront then reads the next 64 (index, value) pairs of the
// message with one coalesced load (eight workers' loads in flight together),
// adds the pairs that fall below the tile's end into the LDS tile and moves
// the worker's position on by their number; when a slice fills all 64 lanes
// (the message is crowded in this tile: the top coordinates of one layer) the
// next eight groups of 64 are fetched together and added in order. No search
// is needed from tile to tile.
// Workers are taken in order 0, 1, ... and a wavefront's LDS accesses execute
// in program order, so the order of the binary32 additions is fixed: +0, then
// worker 0, 1, ... The tile is finally divided by n and written with 16-byte
// stores. HBM traffic: 4d bytes written + 8nk bytes read; no atomics, no
// sort, no workspace.
//
// rtopk_aggregate_update applies the master's next line, omega <- omega -
// eta * ghat, to the weights directly, so the dense ghat is never stored and
// only weights that some worker sent are read and written. It uses the same
// 2048-coordinate tiles with one wavefront per tile, but where a tile starts
// in each worker's list is not searched: a first kernel looks at every pair
// of neighbouring entries and, wherever the tile number changes, writes the
// entry's position into a [tile][worker] table for all tiles in between.
// The second kernel reads its tile's row and the next one, leaves at once if
// the tile is empty, and otherwise adds the entries into its LDS tile in
// worker order, then updates the weights at the non-zero positions. With up
// to 16 workers and up to 64 entries per worker in the tile, every entry
// stays in a register of one lane from the load to the store: the weight at
// its index is fetched while the LDS sums are formed, and the first entry to
// swap the finished sum out of LDS writes the new weight. Long vectors with
// sparse messages take one kernel instead (k_weights), whose workgroups form
// the sums in a hash table, whatever stretch of coordinates the entries span.
#include "rtopk_common.h"
#include "../../include/rtopk.h"

#include <mutex>

namespace rtopk {

constexpr int kAggThreads = 256;
constexpr int kAggWaves = kAggThreads / kWave;
constexpr int kAggTile = 2048;
constexpr int kAggAhead = 8;              // workers whose next pairs are fetched together
constexpr int kAggMore = 8;               // further slices of one crowded message fetched together
// Tiles per wavefront of the dense average: as many as give kAggMaxWaves wavefronts; where that is twice
// kAggRun or more and the workers are few, so that the search for the first tile is short, kAggRun. us, long
// runs / runs of four, evenly spread messages and messages clustered in forty places, k = 0.1%: two workers of 100 M
// 83.3 / 71.9 and 95.2 / 77.0, four 84.3 / 73.9 and 98.3 / 81.2, of 2^28 210 / 191 and 262 / 197 (k = 1%: 310 / 236
// and 363 / 276). Not with more workers: sixteen of 2^28, even messages, 238 / 283 (k = 0.01%); and not for runs of
// five: four workers of 40 M 28.0 / 31.1.
constexpr unsigned kAggMaxWaves = 4096;
constexpr u32 kAggRun = 4;
constexpr u32 kAggFewWorkers = 4;
// The sparse weight step takes k_weights (one kernel) where the vector is long and the
// messages are sparse: from kWeightsTiles tiles on, up to kWeightsWorkers workers and
// kWeightsPerTile entries per tile; k_tile_starts + k_update elsewhere. Measured (us,
// k_weights / the pair), messages crowded towards one end of the vector:
//   2^25, two and eight workers: 1 entry per tile 9 / 16, 14 / 22; 12: 11 / 27, 18 / 41;
//     100: 36 / 52, 42 / 135
//   2^26: 1: 9 / 26, 15 / 36; 12: 19 / 40, 24 / 73; 100: 65 / 67, 74 / 146
//   2^28: 1: 11 / 83, 16 / 111; 12: 56 / 106, 68 / 165; 50: 218 / 214, 236 / 258;
//     100: 347 / 334, 367 / 326
//   2^30: 1: 26 / 312, 31 / 427; 12: 274 / 490, 300 / 744.
// From 2^25 to 2^30, one to eight workers, 0.25 to 12 entries per tile, evenly spread,
// crowded, in stretches of their own or in a twentieth of the vector, k_weights is never the
// slower one; the line at 12 leaves out what it would still gain up to 50. Shorter vectors:
// five workers of 11.2 M coordinates, 10 per tile, 14.5 / 10.0; sixteen workers of 25.6 M (a
// table twice as large, half the workgroups) 51 / 36.
constexpr u64 kWeightsTiles = 1u << 14;
constexpr u32 kWeightsWorkers = 8;
constexpr u32 kWeightsPerTile = 12;
// Up to kWeightsFlat entries in all the workgroups learn how many entries they have (k_weights<true>) and are two per
// compute unit, up to kWeightsFew one: what they do to find their range is a good part of it, and they do it side
// by side. us, rounds of 256 per worker on four workgroups / now: layered messages, four and eight workers of 35 M,
// 0.3 entries per tile 10.5 / 8.0 and 13.4 / 9.5, 2 per tile 11.9 / 9.7 and 15.8 / 11.9, 6 per tile 14.8 / 12.5 and 17.5 / 15.3;
// of 66 M, 2 per tile 12.7 / 10.8 and 16.4 / 13.7. Above, where more is the weights' scattered lines, they lose what
// they look up twice: eight of 66 M, 6 per tile 25.5 / 27.7, four of 200 M, 12 per tile 67.0 / 70.6.
constexpr u64 kWeightsFew = 1u << 13, kWeightsFlat = 1u << 17;
constexpr u32 kPartsLog = 2;              // four workgroups per compute unit otherwise
// Tiles per wavefront of the momentum step: one, but with 17 to 64 workers two from
// kMomentumTwo tiles on and four from kMomentumFour on. The search for a wavefront's first tile
// has 64 lanes for n workers: up to sixteen it takes a few probes, with 33 it is a binary search of fifteen, and a run
// of tiles makes it once. (More than 64 workers are searched for every tile anyway.) us, runs of one / two / four,
// evenly spread messages, k = 0.1%: 33 workers of 20 M 95 / 86 / 87, of 25.6 M 117 / 116 / 124, of 33.5 M
// 145 / 134 / 139, of 66 M 268 / 242 / 232, of 2^28 1078 / 947 / 850, seventeen of 33.5 M 117 / 113 / 113, twenty of 2^28
// 836 / 780 / 734. The other side: sixteen of 25.6 M 84 / 88 / 94, of 66 M 193 / 192 / 186 (k = 0.01%: 181 / 186 /
// 183), 33 of 16.8 M 79 / 79 / 72, 65 of 66 M, k = 1%, 489 / 502 / 536. (Between 28 and
// 33.5 M, 4096 wavefronts of runs of four at two workgroups per unit come out exactly even: seventeen of 33.5 M 110.)
constexpr u32 kMomentumSearch = 16;
constexpr u64 kMomentumTwo = (1u << 13) + 1, kMomentumFour = (1u << 14) + 1;
constexpr unsigned kMomentumLdsClaim = 16u * 1024u;   // with the 32 KB of tiles: three workgroups per unit

__device__ __forceinline__ u32 popc_mask(u64 m) { return (u32)__popcll((unsigned long long)m); }

__device__ __forceinline__ u64 read_lane_u64(u64 v, int lane)
{
    const u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, lane);
    const u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

// For each of nw <= 64 workers (worker w0 + w <-> the group of P lanes
// starting at lane w * P, P = the largest power of two with nw * P <= 64): the
// first position in the worker's ascending index list whose entry is >= x.
// Every step the P lanes of a group probe P evenly spaced positions of the
// remaining range, which shrinks (P + 1)-fold. Returns the result of worker
// `lane` in lane `lane` (lanes >= nw: unspecified). The lanes of a group bring
// the range [lo, hi] of positions that is known to hold their worker's result.
// (kTwo: groups 2w and 2w + 1 belong to worker w, each with an x of its own.)
template <bool kTwo = false>
__device__ __forceinline__ u64 wave_lower_bounds(const u32 *__restrict__ idx, u32 w0, u32 nw, u64 k,
                                                 u64 x, u64 lo, u64 hi)
{
    const u32 lane = lane_id();
    u32 P = 1;
    while (2 * P * nw <= (u32)kWave) P *= 2;
    const u32 w = lane / P, p = lane % P;
    const bool live = w < nw;
    const u32 *wi = idx + (u64)(w0 + (live ? (kTwo ? w / 2u : w) : 0)) * k;
    if (!live) lo = hi;
    const float inv = 1.0f / (float)(P + 1);
    while (__any(hi > lo)) {
        // probe positions lo <= pos_0 <= pos_1 <= ... < hi, roughly evenly spaced (any
        // non-decreasing choice inside the range is valid; this one needs no division)
        const float len = (float)(hi - lo);
        auto probe_at = [&](u32 q) {
            const u64 t = lo + (u64)(len * ((float)(q + 1) * inv));
            return t < hi ? t : hi - 1;
        };
        const bool below = hi > lo && (u64)wi[probe_at(p)] < x;
        const u64 mask = __ballot(below);
        // sorted list: the group's probes below x form a prefix
        const u32 m = __popcll((mask >> (w * P)) & (P == 64 ? ~0ull : ((1ull << P) - 1ull)));
        if (hi > lo) {
            const u64 new_lo = m > 0 ? probe_at(m - 1) + 1 : lo;
            const u64 new_hi = m < P ? probe_at(m) : hi;
            lo = new_lo;
            hi = new_hi;
        }
    }
    // hand the result of worker w (held by all lanes of group w) to lane w
    const u32 lo_lo = __shfl((u32)lo, (int)((lane < nw ? lane : 0) * P), kWave);
    const u32 lo_hi = __shfl((u32)(lo >> 32), (int)((lane < nw ? lane : 0) * P), kWave);
    return ((u64)lo_hi << 32) | lo_lo;
}

// lane l gets lane l - 1's value, lane 0 gets `first` (by DPP: a shuffle goes through the LDS crossbar, and the
// master kernels look at the neighbour's index once per worker and tile, between dependent LDS accesses.
// k_update, five workers of 11.2 M, 17.0 -> 15.8 us; the average and the momentum step, bound by their streams, the same)
__device__ __forceinline__ u32 lane_left(u32 v, u32 first)
{
    return (u32)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
}

// What the momentum form of the kernel does with the average of a coordinate:
// u = scale * average, v <- fma(mu, v, u), w <- fma(neg_eta, v, w) with the
// rounded new velocity.
struct Momentum {
    float scale, mu, neg_eta;
    float *velocity;
};

// kMomentum == false: out[i] = average[i].
// kMomentum == true:  out is the weight vector w; see Momentum.
template <bool kMomentum>
__global__ void __launch_bounds__(kAggThreads)
k_aggregate(const u32 *__restrict__ idx, const float *__restrict__ val, u32 n, u64 k, u64 d,
            u64 tiles, u32 tiles_per_wave, float *__restrict__ out, Momentum mom)
{
    __shared__ float tile_s[kAggWaves][kAggTile];
    const u32 lane = lane_id(), wave = threadIdx.x / kWave;
    float *tile = tile_s[wave];
    const u64 gw = (u64)blockIdx.x * kAggWaves + wave;
    const u64 first_tile = gw * tiles_per_wave;
    const u64 last_tile = first_tile + tiles_per_wave < tiles ? first_tile + tiles_per_wave : tiles;
    if (first_tile >= last_tile) return;
    // one correctly rounded division per output; for n a power of two the
    // product with 1/n is the same number
    const float fn = (float)n;
    const bool n_pow2 = (n & (n - 1u)) == 0u;
    const float rn = 1.0f / fn;
    const bool out_vec =
        (((uintptr_t)out | (kMomentum ? (uintptr_t)mom.velocity : (uintptr_t)0)) & 15u) == 0;
    auto step = [&](float avg, float &v, float &w) {
        const float u = mom.scale * avg;
        v = fmaf(mom.mu, v, u);
        w = fmaf(mom.neg_eta, v, w);
    };
    const u32 groups = (n + kWave - 1) / kWave;    // workers are taken 64 at a time
    // lane w: where the current tile starts in the message of worker w (first group only;
    // with more than 64 workers the position is searched again for every tile)
    u64 pos0 = 0;
    if (groups == 1) pos0 = wave_lower_bounds(idx, 0, n, k, first_tile * kAggTile, 0, k);

    for (u64 t = first_tile; t < last_tile; ++t) {
        const u64 tile_base = t * kAggTile;
        const u64 tile_end = tile_base + kAggTile < d ? tile_base + kAggTile : d;
        for (int i = lane; i < kAggTile / 4; i += kWave)
            reinterpret_cast<float4 *>(tile)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

        for (u32 w0 = 0; w0 < n; w0 += kWave) {
            const u32 nw = n - w0 < (u32)kWave ? n - w0 : (u32)kWave;
            u64 lo = groups == 1 ? pos0 : wave_lower_bounds(idx, w0, nw, k, tile_base, 0, k);
            // ---- worker after worker: the next 64 pairs of its message in one
            //      coalesced load, those below the tile's end added into the tile;
            //      the loads of kAggAhead workers are in flight together --------
            for (u32 g0 = 0; g0 < nw; g0 += kAggAhead) {
                u64 from[kAggAhead];
                u32 ri[kAggAhead];
                float rv[kAggAhead];
#pragma unroll
                for (int q = 0; q < kAggAhead; ++q) {
                    const u32 w = g0 + q < nw ? g0 + q : nw - 1;
                    from[q] = read_lane_u64(lo, (int)w);
                    const u64 j = from[q] + lane;
                    const bool in = g0 + q < nw && j < k;
                    ri[q] = in ? idx[(u64)(w0 + w) * k + j] : 0xFFFFFFFFu;
                    rv[q] = in ? val[(u64)(w0 + w) * k + j] : 0.0f;
                }
#pragma unroll
                for (int q = 0; q < kAggAhead; ++q) {
                    if (g0 + q >= nw) break;
                    const u32 w = g0 + q;
                    const u32 *si = idx + (u64)(w0 + w) * k;
                    const float *sv = val + (u64)(w0 + w) * k;
                    u64 at = from[q];
                    // 64 pairs into the tile; returns how many of them lay inside it
                    auto add_slice = [&](u32 i, float v) -> u32 {
                        const bool inside = (u64)i < tile_end;     // 0xFFFFFFFF marks "no entry"
                        const u64 mask = __ballot(inside);         // a prefix of the lanes: sorted
                        // repeated indices inside one message (never produced by the
                        // encoder, but allowed) must be added in position order
                        const bool dup = inside && lane_left(i, 0xFFFFFFFFu) == i;
                        if (__ballot(dup) == 0ull) {
                            if (inside) tile[i - tile_base] += v;
                        } else {
                            for (u64 rest = mask; rest; rest &= rest - 1) {
                                const int src = __ffsll((unsigned long long)rest) - 1;
                                if ((int)lane == src) tile[i - tile_base] += v;
                            }
                        }
                        return popc_mask(mask);
                    };
                    u32 took = add_slice(ri[q], rv[q]);
                    at += took;
                    // The slice filled all 64 lanes: the message is crowded here (its
                    // entries cluster in a few tiles). The next kAggMore slices are
                    // fetched together and added in order up to the first that ends
                    // inside the tile.
                    while (took == (u32)kWave) {
                        u32 mi[kAggMore];
                        float mv[kAggMore];
#pragma unroll
                        for (int s2 = 0; s2 < kAggMore; ++s2) {
                            const u64 j = at + (u64)s2 * kWave + lane;
                            mi[s2] = j < k ? si[j] : 0xFFFFFFFFu;
                            mv[s2] = j < k ? sv[j] : 0.0f;
                        }
#pragma unroll
                        for (int s2 = 0; s2 < kAggMore; ++s2) {
                            if (took == (u32)kWave) {
                                took = add_slice(mi[s2], mv[s2]);
                                at += took;
                            }
                        }
                    }
                    // the new position of worker w goes back into lane w
                    if (lane == w) lo = at;
                }
            }
            if (groups == 1) pos0 = lo;
        }
        if (out_vec && tile_base + kAggTile <= d) {
            float4 *o4 = reinterpret_cast<float4 *>(out + tile_base);
            constexpr int kVecs = kAggTile / 4 / kWave;
            // weights and velocity are read once and written once, in place: both
            // carry the streaming hint (as in the encoder's streaming kernel, where
            // the hint on load and store together is worth 15%)
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            f32x4 vel[kMomentum ? kVecs : 1], wgt[kMomentum ? kVecs : 1];
            f32x4 *v4 = nullptr, *w4 = reinterpret_cast<f32x4 *>(o4);
            if (kMomentum) {
                v4 = reinterpret_cast<f32x4 *>(mom.velocity + tile_base);
#pragma unroll
                for (int q = 0; q < kVecs; ++q) {
                    vel[q] = __builtin_nontemporal_load(v4 + q * kWave + lane);
                    wgt[q] = __builtin_nontemporal_load(w4 + q * kWave + lane);
                }
            }
#pragma unroll
            for (int q = 0; q < kVecs; ++q) {
                const int i = q * kWave + lane;
                float4 v = reinterpret_cast<const float4 *>(tile)[i];
                if (n_pow2) { v.x *= rn; v.y *= rn; v.z *= rn; v.w *= rn; }
                else { v.x /= fn; v.y /= fn; v.z /= fn; v.w /= fn; }
                if (kMomentum) {
                    const int m = kMomentum ? q : 0;
                    const float avg[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float ve = vel[m][c], we = wgt[m][c];
                        step(avg[c], ve, we);
                        vel[m][c] = ve;
                        wgt[m][c] = we;
                    }
                    __builtin_nontemporal_store(vel[m], v4 + i);
                    __builtin_nontemporal_store(wgt[m], w4 + i);
                } else {
                    o4[i] = v;
                }
            }
        } else {
            for (u64 i = lane; tile_base + i < tile_end; i += kWave) {
                const float avg = tile[i] / fn;
                if (kMomentum) {
                    float v = mom.velocity[tile_base + i], w = out[tile_base + i];
                    step(avg, v, w);
                    mom.velocity[tile_base + i] = v;
                    out[tile_base + i] = w;
                } else {
                    out[tile_base + i] = avg;
                }
            }
        }
    }
}

// Bits that the wavefronts of a workgroup collect for each other: every thread
// gets the union of what the wavefronts put in (one barrier). Three words in
// turn: the one used after next is cleared once everybody has read it.
struct BitExchange {
    u32 *word;          // 3 words of LDS, zero before the first exchange
    u32 turn;
    __device__ __forceinline__ u32 operator()(u32 mine /* uniform over the wavefront */)
    {
        if (lane_id() == 0 && mine != 0u) atomicOr(&word[turn], mine);
        lds_barrier();
        const u32 all = (u32)__builtin_amdgcn_readfirstlane((int)word[turn]);
        const u32 next = turn == 2u ? 0u : turn + 1u;
        if (threadIdx.x == 0) word[next == 2u ? 0u : next + 1u] = 0u;
        turn = next;
        return all;
    }
};

// The coordinates [x0, x1) of one of the kAggThreads << parts_log workgroups, and where
// x0 (and, with kEnds, x1) starts in every worker's list (pos and end, LDS). Messages cluster (the top
// coordinates sit in a few layers), and no two workers' need cluster alike: so
// evenly spaced entries of EVERY worker, at most 255 in all, cut the coordinates
// into pieces, and each piece is cut into equal parts. A piece lies between two
// neighbouring samples of any worker: it holds at most an S-th of a
// message of which S entries were sampled. Where the samples lie in the message
// also narrows the search for x0 down. lds: 2 * kAggThreads words.
template <bool kEnds>
__device__ __forceinline__ bool weights_range(const u32 *__restrict__ idx, u32 n, u64 k, u64 d, u32 parts_log, u32 *lds,
                                              u64 *x0, u64 *x1, u64 *pos, u64 *end)
{
    // (a cut per thread, 2^parts_log workgroups between two cuts)
    const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const u32 per = (kAggThreads - 1) / n, cuts = per * n;      // samples of one worker, of all
    // position of worker v's sample s (staggered, or the samples of like messages would coincide)
    auto at = [&](u32 v, u32 s) { return (u64)(s * n + v + 1u) * k / (cuts + 1u); };
    const u32 w = tid / per, s = tid - w * per;
    u32 mine = 0xFFFFFFFFu;
    if (tid < cuts) mine = idx[w * k + at(w, s)];
    u32 *cut = lds, *sorted = lds + kAggThreads;
    cut[tid] = mine;
    lds_barrier();
    // samples of worker v that are below x (kLess) or at most x
    auto below = [&](u32 v, u64 x) {
        u32 lo = 0, hi = per;
        while (lo < hi) {
            const u32 mid = (lo + hi) / 2u;
            if ((u64)cut[v * per + mid] < x) lo = mid + 1u; else hi = mid;
        }
        return lo;
    };
    if (tid < cuts) {
        // place among all samples: ties in worker order
        u32 rank = s;
        for (u32 v = 0; v < n; ++v)
            if (v != w) rank += below(v, (u64)mine + (v < w ? 1u : 0u));
        sorted[rank] = mine;
    }
    lds_barrier();
    const u32 piece = blockIdx.x >> parts_log, part = blockIdx.x & ((1u << parts_log) - 1u);
    u64 lo = piece == 0u || piece > cuts ? 0ull : (u64)sorted[piece - 1u], hi = piece >= cuts ? d : (u64)sorted[piece];
    if (lo > d) lo = d;
    if (hi > d) hi = d;
    *x0 = lo + ((hi - lo) * part >> parts_log);
    *x1 = lo + ((hi - lo) * (part + 1u) >> parts_log);
    if (piece > cuts || lo >= hi || *x0 >= *x1) return false;
    // (with the ends, two searches per worker)
    constexpr u32 kSides = kEnds ? 2u : 1u;
    const u32 of_wave = (n + kAggWaves - 1) / kAggWaves, first = wave * of_wave;
    if (first < n) {
        const u32 here = kSides * (n - first < of_wave ? n - first : of_wave);
        u32 lanes = 1;
        while (2 * lanes * here <= (u32)kWave) lanes *= 2;
        const u32 of = lane / lanes < here ? lane / lanes : 0u, v = first + of / kSides;
        const u64 x = of % kSides == 0u ? *x0 : *x1;
        const u32 c = below(v, x);
        const u64 start = wave_lower_bounds<kEnds>(idx, first, here, k, x, c == 0u ? 0ull : at(v, c - 1u) + 1u,
                                                   c == per ? k : at(v, c));
        if (lane < here) (lane % kSides == 0u ? pos : end)[first + lane / kSides] = start;
    }
    lds_barrier();                                             // the words are the caller's again
    return true;
}

// ---------------------------------------------------------------------------
// weights: the sparse weight step for up to kWeightsWorkers workers:
// omega[i] = fma(neg_step, average[i], omega[i]) wherever the average of what
// the workers sent for i is not zero.
//
// A few MB are moved: what bounds it is the chain of dependent trips to
// memory (the search, the entries, the weights) and how many such chains one
// workgroup walks one after the other. So a workgroup takes ALL entries of its
// range at once, 256 per worker and round, whatever the coordinates between
// them: the sums are formed in a hash table in LDS (keyed by coordinate, at
// most half full) and not in a tile of coordinates. Every entry takes its slot;
// the one that finds the slot empty (the leader) has the weight fetched
// meanwhile and writes it. If no coordinate was sent twice, a leader's sum is its own value;
// otherwise the workers are added in order with a barrier in between.
// Four workers of 66 M coordinates (66,034 entries each): 19.3 us; the
// pair of kernels with a wavefront per tile of 2048 coordinates takes 4.8 + 33.8,
// as its 32,244 tiles walk the same chain in six rounds.
// ---------------------------------------------------------------------------
template <bool kFlat>
__global__ void __launch_bounds__(kAggThreads, 4)
k_weights(const u32 *__restrict__ idx, const float *__restrict__ val, u32 n, u64 k, u64 d, u32 few_parts_log,
          float neg_step, float *__restrict__ omega)
{
    const u32 parts_log = kFlat ? few_parts_log : kPartsLog;
    constexpr u32 kWindows = kWeightsWorkers;
    constexpr u32 kSlots = 2 * kWindows * kAggThreads;     // a power of two
    constexpr u32 kEmpty = 0xFFFFFFFFu;                    // never a coordinate
    __shared__ u32 key[kSlots];
    __shared__ float sum[kSlots];
    __shared__ u64 pos[kWindows], end[kWindows];
    __shared__ u32 word[3];
    __shared__ u32 bound_s;
    const u32 tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    u64 x0, x1;
    if (!weights_range<kFlat>(idx, n, k, d, parts_log, key, &x0, &x1, pos, end)) return;
    const float fn = (float)n;
    const bool n_pow2 = (n & (n - 1u)) == 0u;
    const float rn = 1.0f / fn;
    auto average = [&](float s) { return n_pow2 ? s * rn : s / fn; };
    if (tid < 3u) word[tid] = 0u;
    BitExchange exchange{word, 0u};
    if constexpr (kFlat) {
        // ---- the usual case: a few hundred entries, whoever sent them. Entry f of the range, worker after
        //      worker, is thread f % 256's (f / 256)-th; the table is four times as large as the entries need.
        u32 total = 0;
        u32 before[kWindows], from_here[kWindows];      // entries of the workers before; what turns f into a position
#pragma unroll
        for (u32 q = 0; q < kWindows; ++q) {
            before[q] = total;
            from_here[q] = 0u;
            if (q < n) {
                from_here[q] = (u32)pos[q] - total;
                total += (u32)(end[q] > pos[q] ? end[q] - pos[q] : 0ull);
            }
        }
        if (__builtin_expect(total <= kSlots / 2, 1)) {
            if (total == 0u) return;
            u32 log_slots = 9u;
            while (1u << log_slots < 4u * total && 1u << log_slots < kSlots) ++log_slots;
            const u32 slots = 1u << log_slots;
            constexpr u32 kMine = kSlots / 2 / kAggThreads;
            u32 e_i[kMine], e_w[kMine], slot[kMine];
            float e_v[kMine], w[kMine];
            u32 leader = 0, mine = 0, valid = 0;
            const u32 rounds = (total + kAggThreads - 1u) / kAggThreads;
#pragma unroll
            for (u32 i = 0; i < kMine; ++i) {
                if (i >= rounds) break;
                const u32 f = tid + i * kAggThreads;
                u32 of = 0, j = f + from_here[0];
#pragma unroll
                for (u32 q = 1; q < kWindows; ++q)
                    if (q < n && f >= before[q]) { of = q; j = f + from_here[q]; }
                e_w[i] = of;
                e_i[i] = kEmpty;
                if (f < total) {
                    e_i[i] = idx[of * k + j];
                    e_v[i] = val[of * k + j];
                    valid |= 1u << i;
                }
                // (a message that repeats an index: its entries are added position by position below. No encode
                // sends one; it costs 3-10% more than the rounds at once, eight of 34 M, 64 entries each, 20.9 / 23.1 us)
                u32 left = kEmpty;
                if (lane == 0u && f != 0u && f < total && j != 0u) left = idx[of * k + j - 1u];
                left = lane_left(e_i[i], left);
                const u32 of_left = lane_left(of, of);
                if (__ballot(f < total && left == e_i[i] && of_left == of) != 0ull) mine |= 2u;
            }
            for (u32 i = tid; i < slots; i += kAggThreads) { key[i] = kEmpty; sum[i] = 0.0f; }
            lds_barrier();
#pragma unroll
            for (u32 i = 0; i < kMine; ++i) {
                if (i >= rounds) break;
                const bool in = (valid >> i & 1u) != 0u && (u64)e_i[i] >= x0 && (u64)e_i[i] < x1;   // (a list that is not sorted: left out)
                if (!in) valid &= ~(1u << i);
                w[i] = in ? omega[e_i[i]] : 0.0f;
                if (in) {
                    slot[i] = (e_i[i] * 0x9E3779B1u) >> (32u - log_slots);
                    u32 was = atomicCAS(&key[slot[i]], kEmpty, e_i[i]);
                    while (was != kEmpty && was != e_i[i]) {
                        slot[i] = (slot[i] + 1u) & (slots - 1u);
                        was = atomicCAS(&key[slot[i]], kEmpty, e_i[i]);
                    }
                    if (was == kEmpty) leader |= 1u << i;
                }
                if (__ballot(in && (leader >> i & 1u) == 0u) != 0ull) mine |= 1u;
            }
            const u32 seen = exchange(mine);
            if ((seen & 2u) == 0u) {
                if ((seen & 1u) != 0u) {
                    // ---- coordinates sent by several workers: sums in worker order
                    for (u32 q = 0; q < n; ++q) {
#pragma unroll
                        for (u32 i = 0; i < kMine; ++i) {
                            if (i >= rounds) break;
                            if ((valid >> i & 1u) != 0u && e_w[i] == q) sum[slot[i]] += e_v[i];
                        }
                        lds_barrier();
                    }
                }
#pragma unroll
                for (u32 i = 0; i < kMine; ++i) {
                    if (i >= rounds) break;
                    if ((leader >> i & 1u) != 0u) {
                        const float avg = average((seen & 1u) != 0u ? sum[slot[i]] : 0.0f + e_v[i]);
                        if (avg != 0.0f) omega[e_i[i]] = fmaf(neg_step, avg, w[i]);
                    }
                }
                return;
            }
            lds_barrier();                              // (nobody reads the table any more)
        }
    }
    for (u32 i = tid; i < kSlots; i += kAggThreads) { key[i] = kEmpty; sum[i] = 0.0f; }
    lds_barrier();

    for (;;) {
        // ---- the next 256 entries of every worker --------------------------------
        u32 e_i[kWindows], left[kWindows];
        float e_v[kWindows];
        u32 bound = (u32)(x1 - 1);             // last coordinate of this round, at most
        bool cut = false;
#pragma unroll
        for (u32 q = 0; q < kWindows; ++q) {
            e_i[q] = left[q] = kEmpty;
            e_v[q] = 0.0f;
            if (q < n) {
                const u64 from = pos[q], j = from + tid;
                if (j < k) {
                    e_i[q] = idx[q * k + j];
                    e_v[q] = val[q * k + j];
                    if (lane == 0 && tid != 0u) left[q] = idx[q * k + j - 1];
                }
            }
        }
        // A round ends before the last entry of any window that has entries behind it (an
        // index may occur several times: what follows the window may belong to the same
        // coordinate), so that it holds every entry of its coordinates.
        if (tid == kAggThreads - 1) {
            u32 b = kEmpty;
#pragma unroll
            for (u32 q = 0; q < kWindows; ++q)
                if (q < n && pos[q] + kAggThreads < k && e_i[q] < b) b = e_i[q];
            bound_s = b;
        }
        lds_barrier();
        {
            const u32 b = bound_s;
            cut = b <= bound;
            if (cut) bound = b;
        }
        const u32 base = (u32)x0;
        // coordinates [x0, bound) of a round that was cut short, [x0, bound] otherwise
        const u32 span = bound - base + (cut ? 0u : 1u);
        auto inside = [&](u32 i) { return i - base < span && i != kEmpty; };
        float w[kWindows];
        u32 slot[kWindows];
        u32 leader = 0, mine = 0;
#pragma unroll
        for (u32 q = 0; q < kWindows; ++q) w[q] = inside(e_i[q]) ? omega[e_i[q]] : 0.0f;
        // bits: 1 some slot was taken by another entry already; 2 << q: worker q holds entries;
        // 2^17 a message repeats an index
#pragma unroll
        for (u32 q = 0; q < kWindows; ++q) {
            slot[q] = (e_i[q] * 0x9E3779B1u) >> (32 - __builtin_ctz(kSlots));
            const bool in = inside(e_i[q]);
            const u64 m = __ballot(in);
            if (m == 0ull) continue;
            mine |= 2u << q;
            if (__ballot(in && lane_left(e_i[q], left[q]) == e_i[q]) != 0ull) mine |= 1u << 17;
            if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long *>(&pos[q]), (unsigned long long)popc_mask(m));
            if (in) {
                u32 was = atomicCAS(&key[slot[q]], kEmpty, e_i[q]);
                while (was != kEmpty && was != e_i[q]) {
                    slot[q] = (slot[q] + 1u) & (kSlots - 1u);
                    was = atomicCAS(&key[slot[q]], kEmpty, e_i[q]);
                }
                if (was == kEmpty) leader |= 1u << q;
            }
            if (__ballot(in && ((leader >> q) & 1u) == 0u) != 0ull) mine |= 1u;
        }
        const u32 seen = exchange(mine);
        if ((seen & 1u) != 0u) {
            // ---- coordinates sent by several workers: sums in worker order -------------
#pragma unroll
            for (u32 q = 0; q < kWindows; ++q) {
                if (((seen >> (q + 1u)) & 1u) == 0u) continue;
                const bool in = inside(e_i[q]);
                if (__builtin_expect((seen >> 17) == 0u, 1)) {
                    if (in) sum[slot[q]] += e_v[q];
                    lds_barrier();
                } else {
                    // repeated indices inside one message: in position order, one wavefront
                    // after the other; the first entries of all runs of equal indices
                    // together, then the second ones, ...
                    const u32 before = lane_left(e_i[q], left[q]);
                    const u64 heads = __ballot(in && (lane == 0 || before != e_i[q]));
                    const u32 rank = in ? lane - (63u - (u32)__clzll(heads & (lanes_below() | (1ull << lane)))) : 0u;
                    const u32 most = wave_max(rank);
                    for (u32 wv = 0; wv < (u32)kAggWaves; ++wv) {
                        if (wave == wv)
                            for (u32 s = 0; s <= most; ++s) {
                                if (in && rank == s) sum[slot[q]] += e_v[q];
                                wave_lds_fence();
                            }
                        lds_barrier();
                    }
                }
            }
        }
#pragma unroll
        for (u32 q = 0; q < kWindows; ++q) {
            if (((leader >> q) & 1u) != 0u) {
                const float total = (seen & 1u) != 0u ? sum[slot[q]] : 0.0f + e_v[q];
                sum[slot[q]] = 0.0f;
                key[slot[q]] = kEmpty;
                const float avg = average(total);
                if (avg != 0.0f) omega[e_i[q]] = fmaf(neg_step, avg, w[q]);
            }
        }
        if (!cut) break;
        if (__builtin_expect(seen == 0u, 0)) {
            // Nothing lies below the bound: a window holds one coordinate only, the bound (an index
            // that occurs more than 255 times in one message). Its entries, worker after worker:
            // the workgroup fetches 256 at a time, one thread adds them up in position order.
            // (20,000 entries on one coordinate: 0.74 ms; 2.5 when that thread fetched them too, and
            // 1.5 on the pair of kernels.)
            float s = 0.0f;
            bool moved = false;
            for (u32 q = 0; q < n; ++q) {
                u32 c;
                do {
                    const u64 from = pos[q], j = from + tid;
                    const bool on = j < k && idx[q * k + j] == bound;
                    sum[tid] = on ? val[q * k + j] : 0.0f;
                    const u64 m = __ballot(on);
                    if (lane == 0) key[wave] = popc_mask(m);
                    lds_barrier();
                    c = 0;
                    for (u32 wv = 0; wv < (u32)kAggWaves; ++wv) c += key[wv];
                    moved = moved || c != 0u;
                    if (tid == 0) {
                        for (u32 t = 0; t < c; ++t) s += sum[t];
                        pos[q] = from + c;
                    }
                    lds_barrier();
                } while (c == (u32)kAggThreads);
            }
            sum[tid] = 0.0f;
            if (tid < (u32)kAggWaves) key[tid] = kEmpty;
            if (tid == 0) {
                const float avg = average(s);
                if (avg != 0.0f && bound >= base) omega[bound] = fmaf(neg_step, avg, omega[bound]);
                // (a list that is not sorted, a broken precondition: the loop ends all the same)
                if (!moved)
                    for (u32 q = 0; q < n; ++q) pos[q] += kAggThreads;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// tile_starts: start[t * n + w] = the first position in worker w's list whose
// index lies in tile t or later, for t = 0 .. tiles (the last row is k).
// Thread j of worker w compares the tiles of entries j - 1 and j (tile -1
// before the list, tile `tiles` after it) and fills the rows in between;
// since the list ascends, every row is written exactly once. A long run of
// empty tiles is filled by the whole wavefront. blockIdx.y is the worker.
// ---------------------------------------------------------------------------
constexpr int kStartThreads = 256;

__global__ void __launch_bounds__(kStartThreads)
k_tile_starts(const u32 *__restrict__ idx, u32 n, u64 k, u64 tiles, u32 *__restrict__ start)
{
    const u32 w = blockIdx.y;
    const u32 *wi = idx + (u64)w * k;
    const u64 j = (u64)blockIdx.x * kStartThreads + threadIdx.x;
    // rows (from, to] get the value j; an index past the last tile (a broken
    // precondition) is treated as the end of the list
    u64 from = 0, to = 0;
    if (j <= k) {
        const u64 t_prev = j > 0 ? (u64)wi[j - 1] / kAggTile + 1 : 0;   // first row to fill
        u64 t_cur = j < k ? (u64)wi[j] / kAggTile : tiles;
        if (t_cur > tiles) t_cur = tiles;
        from = t_prev;
        to = t_cur + 1;                                                  // one past the last row
        if (to < from) to = from;
    }
    const bool is_long = to - from > 8;
    if (!is_long)
        for (u64 t = from; t < to; ++t) start[t * n + w] = (u32)j;
    for (u64 rest = __ballot(is_long); rest; rest &= rest - 1) {
        const int src = __ffsll((unsigned long long)rest) - 1;
        const u64 a = read_lane_u64(from, src), b = read_lane_u64(to, src);
        const u32 v = (u32)read_lane_u64(j, src);
        for (u64 t = a + lane_id(); t < b; t += kWave) start[t * n + w] = v;
    }
}

// ---------------------------------------------------------------------------
// update: one wavefront per tile. omega[i] = fma(neg_step, average[i],
// omega[i]) wherever the average of what the workers sent for i is not zero.
// ---------------------------------------------------------------------------
constexpr u32 kDenseTileEntries = 512;     // from here on the whole tile is read and written
constexpr int kUpdateAhead = 16;           // workers whose entries are held in registers together

__global__ void __launch_bounds__(kAggThreads)
k_update(const u32 *__restrict__ idx, const float *__restrict__ val, u32 n, u64 k, u64 d,
         u64 tiles, const u32 *__restrict__ start, float neg_step, float *__restrict__ omega)
{
    __shared__ float tile_s[kAggWaves][kAggTile];
    const u32 lane = lane_id(), wave = threadIdx.x / kWave;
    float *tile = tile_s[wave];
    const u64 t = (u64)blockIdx.x * kAggWaves + wave;
    if (t >= tiles) return;
    const u64 tile_base = t * kAggTile;
    const u64 tile_end = tile_base + kAggTile < d ? tile_base + kAggTile : d;
    const float fn = (float)n;
    const bool n_pow2 = (n & (n - 1u)) == 0u;
    const float rn = 1.0f / fn;
    bool cleared = false;
    u32 entries = 0;
    // the average of a coordinate from its sum; a weight moves only where the
    // AVERAGE is not zero (a tiny sum may underflow in the division)
    auto average = [&](float sum) { return n_pow2 ? sum * rn : sum / fn; };
    auto step = [&](float avg, float w) { return fmaf(neg_step, avg, w); };

    // ---- few workers with at most 64 entries each in this tile (the usual
    //      case): every entry stays in a register of "its" lane. The weight at
    //      the entry's index is fetched while the sums are formed in LDS;
    //      afterwards every entry swaps a zero into its LDS word, and the one
    //      that gets the sum back (the first to arrive) writes the weight. ----
    if (n <= kUpdateAhead) {
        u32 lo = 0, cnt = 0;
        if (lane < n) {
            u64 a = start[t * n + lane], b = start[(t + 1) * n + lane];
            if (b > k) b = k;
            if (a > b) a = b;
            lo = (u32)a;
            cnt = (u32)(b - a);
        }
        if (__ballot(cnt != 0u) == 0ull) return;           // nobody sent anything in this tile
        if (__ballot(cnt > (u32)kWave) == 0ull) {
            for (int i = lane; i < kAggTile / 4; i += kWave)
                reinterpret_cast<float4 *>(tile)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            u32 ei[kUpdateAhead];
            float ev[kUpdateAhead], ew[kUpdateAhead];
            bool in[kUpdateAhead];
#pragma unroll
            for (int q = 0; q < kUpdateAhead; ++q) {
                in[q] = false;
                ei[q] = 0xFFFFFFFFu;
                ev[q] = 0.0f;
                if ((u32)q < n) {
                    const u32 from = (u32)__builtin_amdgcn_readlane((int)lo, q);
                    const u32 c = (u32)__builtin_amdgcn_readlane((int)cnt, q);
                    if (lane < c) {
                        ei[q] = idx[(u64)q * k + from + lane];
                        ev[q] = val[(u64)q * k + from + lane];
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kUpdateAhead; ++q) {
                // the range check keeps a list that is not sorted (a broken
                // precondition) inside the LDS tile
                in[q] = (u64)ei[q] >= tile_base && (u64)ei[q] < tile_end;
                ew[q] = in[q] ? omega[ei[q]] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < kUpdateAhead; ++q) {
                if ((u32)q < n) {
                    // repeated indices inside one message must be added in position order
                    const u32 mine = ei[q];
                    const float v = ev[q];
                    const bool inside = in[q];
                    const bool dup = inside && lane_left(mine, 0xFFFFFFFFu) == mine;
                    if (__ballot(dup) == 0ull) {
                        if (inside) tile[mine - tile_base] += v;
                    } else {
                        for (u64 rest = __ballot(inside); rest; rest &= rest - 1) {
                            const int src = __ffsll((unsigned long long)rest) - 1;
                            if ((int)lane == src) tile[mine - tile_base] += v;
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kUpdateAhead; ++q) {
                if ((u32)q < n && in[q]) {
                    const float avg = average(atomicExch(&tile[ei[q] - tile_base], 0.0f));
                    if (avg != 0.0f) omega[ei[q]] = step(avg, ew[q]);
                }
            }
            return;
        }
    }

    for (u32 w0 = 0; w0 < n; w0 += kWave) {
        const u32 nw = n - w0 < (u32)kWave ? n - w0 : (u32)kWave;
        // lane w: the part [lo, hi) of worker w0 + w's list that lies in this tile
        u64 lo = 0, hi = 0;
        if (lane < nw) {
            lo = start[t * n + w0 + lane];
            hi = start[(t + 1) * n + w0 + lane];
            if (hi > k) hi = k;
            if (lo > hi) lo = hi;
        }
        const u32 here = wave_sum((u32)(hi - lo));
        if (here == 0u) continue;
        if (!cleared) {
            for (int i = lane; i < kAggTile / 4; i += kWave)
                reinterpret_cast<float4 *>(tile)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            cleared = true;
        }
        entries += here;
        for (u32 g0 = 0; g0 < nw; g0 += kAggAhead) {
            u64 from[kAggAhead], to[kAggAhead];
            u32 ri[kAggAhead];
            float rv[kAggAhead];
#pragma unroll
            for (int q = 0; q < kAggAhead; ++q) {
                const u32 w = g0 + q < nw ? g0 + q : nw - 1;
                from[q] = read_lane_u64(lo, (int)w);
                to[q] = g0 + q < nw ? read_lane_u64(hi, (int)w) : from[q];
                const u64 j = from[q] + lane;
                const bool in = j < to[q];
                ri[q] = in ? idx[(u64)(w0 + w) * k + j] : 0xFFFFFFFFu;
                rv[q] = in ? val[(u64)(w0 + w) * k + j] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < kAggAhead; ++q) {
                if (g0 + q >= nw) break;
                const u32 *si = idx + (u64)(w0 + g0 + q) * k;
                const float *sv = val + (u64)(w0 + g0 + q) * k;
                u64 at = from[q];
                u32 i = ri[q];
                float v = rv[q];
                while (at < to[q]) {
                    // the table says these entries belong to the tile; the check keeps a
                    // list that is not sorted (a broken precondition) inside the LDS tile
                    const bool inside = at + lane < to[q] && (u64)i >= tile_base && (u64)i < tile_end;
                    // repeated indices inside one message must be added in position order
                    const bool dup = inside && lane_left(i, 0xFFFFFFFFu) == i;
                    if (__ballot(dup) == 0ull) {
                        if (inside) tile[i - tile_base] += v;
                    } else {
                        for (u64 rest = __ballot(inside); rest; rest &= rest - 1) {
                            const int src = __ffsll((unsigned long long)rest) - 1;
                            if ((int)lane == src) tile[i - tile_base] += v;
                        }
                    }
                    at += kWave;
                    if (at >= to[q]) break;
                    const u64 j = at + lane;
                    i = j < to[q] ? si[j] : 0xFFFFFFFFu;
                    v = j < to[q] ? sv[j] : 0.0f;
                }
            }
        }
    }
    if (!cleared) return;                               // nobody sent anything in this tile

    constexpr int kVecs = kAggTile / 4 / kWave;         // float4 per lane
    float4 s4[kVecs];                                   // the averages of this lane's coordinates
#pragma unroll
    for (int q = 0; q < kVecs; ++q) {
        const float4 t4 = reinterpret_cast<const float4 *>(tile)[q * kWave + lane];
        s4[q] = make_float4(average(t4.x), average(t4.y), average(t4.z), average(t4.w));
    }
    if (entries >= kDenseTileEntries && ((uintptr_t)omega & 15u) == 0 &&
        tile_base + kAggTile <= d) {
        float4 *o4 = reinterpret_cast<float4 *>(omega + tile_base);
        float4 w[kVecs];
#pragma unroll
        for (int q = 0; q < kVecs; ++q) w[q] = o4[q * kWave + lane];
#pragma unroll
        for (int q = 0; q < kVecs; ++q) {
            const float4 s = s4[q];
            if (s.x == 0.0f && s.y == 0.0f && s.z == 0.0f && s.w == 0.0f) continue;
            if (s.x != 0.0f) w[q].x = step(s.x, w[q].x);
            if (s.y != 0.0f) w[q].y = step(s.y, w[q].y);
            if (s.z != 0.0f) w[q].z = step(s.z, w[q].z);
            if (s.w != 0.0f) w[q].w = step(s.w, w[q].w);
            o4[q * kWave + lane] = w[q];
        }
    } else {
        // few entries: only the weights that move are read; all loads first
        float *o = omega + tile_base + 4 * lane;
        float w[kVecs][4];
#pragma unroll
        for (int q = 0; q < kVecs; ++q) {
            const float sv[4] = {s4[q].x, s4[q].y, s4[q].z, s4[q].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                w[q][c] = sv[c] != 0.0f ? o[q * 4 * kWave + c] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kVecs; ++q) {
            const float sv[4] = {s4[q].x, s4[q].y, s4[q].z, s4[q].w};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (sv[c] != 0.0f) o[q * 4 * kWave + c] = step(sv[c], w[q][c]);
        }
    }
}

#ifdef RTOPK_DEBUG_CHECKS
// ---------------------------------------------------------------------------
// Debug build only: the preconditions of the master entry points (every index
// below d, every worker's slice ascending) are checked on the device before
// the call's own kernels are enqueued. The check synchronises the stream, so
// it is kept out of the release build, where the conditions stay preconditions.
// ---------------------------------------------------------------------------
static __device__ u32 dbg_bad_entries;

__global__ void k_check_messages(const u32 *__restrict__ idx, u32 n, u64 k, u64 d, u32 *bad)
{
    const u64 total = (u64)n * k;
    u32 mine = 0;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (u64)gridDim.x * blockDim.x) {
        const u32 v = idx[i];
        if ((u64)v >= d) ++mine;
        else if (i % k != 0 && idx[i - 1] > v) ++mine;
    }
    if (mine) atomicAdd(bad, mine);
}
#endif

}  // namespace rtopk

using namespace rtopk;

// Release build: nothing. Debug build (RTOPK_DEBUG_CHECKS): RTOPK_EINVAL when a
// message breaks a precondition of the master entry points.
static int debug_check_messages(const uint32_t *idx, uint32_t n, uint64_t k, uint64_t d,
                                hipStream_t stream)
{
#ifdef RTOPK_DEBUG_CHECKS
    u32 *bad = nullptr;
    u32 host_bad = 0;
    if (hipGetSymbolAddress((void **)&bad, HIP_SYMBOL(dbg_bad_entries)) != hipSuccess ||
        hipMemcpyAsync(bad, &host_bad, sizeof host_bad, hipMemcpyHostToDevice, stream) != hipSuccess)
        return RTOPK_EHIP;
    k_check_messages<<<1024, 256, 0, stream>>>(idx, n, k, d, bad);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&host_bad, bad, sizeof host_bad, hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return RTOPK_EHIP;
    if (host_bad != 0) return RTOPK_EINVAL;
#else
    (void)idx; (void)n; (void)k; (void)d; (void)stream;
#endif
    return RTOPK_OK;
}

extern "C" int rtopk_aggregate_workspace_bytes(uint64_t d, uint32_t n, uint64_t k,
                                               uint64_t *bytes)
{
    if (!bytes || n < 1 || k < 1 || d < 1 || d > 0xFFFFFFFFull) return RTOPK_EINVAL;
    *bytes = 0;   // the single-kernel aggregator keeps everything in LDS
    return RTOPK_OK;
}

extern "C" int rtopk_aggregate(const uint32_t *idx, const float *val, uint32_t n, uint64_t k,
                               uint64_t d, float *out, void *workspace,
                               uint64_t workspace_bytes, void *stream_v)
{
    (void)workspace_bytes;
    if (!idx || !val || !out || n < 1 || k < 1 || d < 1 || d > 0xFFFFFFFFull)
        return RTOPK_EINVAL;
    if (workspace && ((uintptr_t)workspace & 255u)) return RTOPK_EWORKSPACE;
    hipStream_t stream = (hipStream_t)stream_v;
    if (const int rc = debug_check_messages(idx, n, k, d, stream)) return rc;
    const u64 tiles = (d + kAggTile - 1) / kAggTile;
    u64 run = (tiles + kAggMaxWaves - 1) / kAggMaxWaves;
    if (n <= kAggFewWorkers && run >= 2 * kAggRun) run = kAggRun;
    const u32 tiles_per_wave = (u32)run;
    const u64 waves = (tiles + tiles_per_wave - 1) / tiles_per_wave;
    const unsigned grid = (unsigned)((waves + kAggWaves - 1) / kAggWaves);
    k_aggregate<false><<<grid, kAggThreads, 0, stream>>>(idx, val, n, k, d, tiles, tiles_per_wave,
                                                         out, Momentum{});
    if (hipGetLastError() != hipSuccess) return RTOPK_EHIP;
    return RTOPK_OK;
}

extern "C" int rtopk_aggregate_update_momentum(const uint32_t *idx, const float *val, uint32_t n,
                                               uint64_t k, uint64_t d, float eta, float scale,
                                               float mu, float *omega, float *velocity,
                                               void *stream_v)
{
    if (!idx || !val || !omega || !velocity || n < 1 || k < 1 || d < 1 || d > 0xFFFFFFFFull)
        return RTOPK_EINVAL;
    {
        const uintptr_t w0 = (uintptr_t)omega, v0 = (uintptr_t)velocity;
        if (w0 < v0 + d * 4 && v0 < w0 + d * 4) return RTOPK_EINVAL;
    }
    hipStream_t stream = (hipStream_t)stream_v;
    if (const int rc = debug_check_messages(idx, n, k, d, stream)) return rc;
    const u64 tiles = (d + kAggTile - 1) / kAggTile;
    const bool runs = n > kMomentumSearch && n <= (u32)kWave;
    const u32 run = !runs ? 1u : tiles >= kMomentumFour ? 4u : tiles >= kMomentumTwo ? 2u : 1u;
    const u64 waves = (tiles + run - 1) / run;
    const unsigned grid = (unsigned)((waves + kAggWaves - 1) / kAggWaves);
    // This form streams 16 bytes per coordinate: few tiles per wavefront, in order, so that the
    // wavefronts that search and those that stream overlap, and three workgroups per
    // compute unit (each claims LDS it does not use). us, 4096 wavefronts of runs of tiles with two
    // workgroups per unit / one tile and two / three / five: eight workers of 25.6 M 80.9 / 76.7 / 74.4 / 75.6, sixteen, k = 1%,
    // 145 / 112 / 99 / 98; five of 11.2 M 45.3 / 39.2 / 38.8 / 38.9; eight of 100 M 357 / 275 / 269 / 274; two of
    // 200 M, k = 1%, 681 / 546 / 570 / 573; four of 66 M 200 / 182 / 185 / 184.
    k_aggregate<true><<<grid, kAggThreads, kMomentumLdsClaim, stream>>>(
        idx, val, n, k, d, tiles, run, omega, Momentum{scale, mu, -eta, velocity});
    if (hipGetLastError() != hipSuccess) return RTOPK_EHIP;
    return RTOPK_OK;
}

extern "C" int rtopk_aggregate_update_workspace_bytes(uint64_t d, uint32_t n, uint64_t k,
                                                      uint64_t *bytes)
{
    if (!bytes || n < 1 || k < 1 || k > 0xFFFFFFFFull || d < 1 || d > 0xFFFFFFFFull)
        return RTOPK_EINVAL;
    const u64 tiles = (d + kAggTile - 1) / kAggTile;
    *bytes = align_up((tiles + 1) * (u64)n * sizeof(u32), 256);
    return RTOPK_OK;
}

// the kernels of the fused update; `start` holds (tiles + 1) * n words
static int launch_update(const uint32_t *idx, const float *val, uint32_t n, uint64_t k, uint64_t d,
                         float eta, float scale, float *omega, u32 *start, hipStream_t stream)
{
    if (const int rc = debug_check_messages(idx, n, k, d, stream)) return rc;
    volatile float step = eta * scale;                  // one binary32 rounding, then negated
    if (n <= kWeightsWorkers && d / kAggTile >= kWeightsTiles && (u64)n * k <= d / kAggTile * kWeightsPerTile) {
        const u64 entries = (u64)n * k;
        const u32 parts_log = entries <= kWeightsFew ? 0u : entries <= kWeightsFlat ? 1u : kPartsLog;
        if (entries <= kWeightsFlat)
            k_weights<true><<<kAggThreads << parts_log, kAggThreads, 0, stream>>>(idx, val, n, k, d, parts_log, -step, omega);
        else
            k_weights<false><<<kAggThreads << parts_log, kAggThreads, 0, stream>>>(idx, val, n, k, d, parts_log, -step, omega);
        if (hipGetLastError() != hipSuccess) return RTOPK_EHIP;
        return RTOPK_OK;
    }
    const u64 tiles = (d + kAggTile - 1) / kAggTile;
    const dim3 sgrid((unsigned)((k + 1 + kStartThreads - 1) / kStartThreads), n);
    k_tile_starts<<<sgrid, kStartThreads, 0, stream>>>(idx, n, k, tiles, start);
    if (hipGetLastError() != hipSuccess) return RTOPK_EHIP;
    const unsigned grid = (unsigned)((tiles + kAggWaves - 1) / kAggWaves);
    k_update<<<grid, kAggThreads, 0, stream>>>(idx, val, n, k, d, tiles, start, -step, omega);
    if (hipGetLastError() != hipSuccess) return RTOPK_EHIP;
    return RTOPK_OK;
}

extern "C" int rtopk_aggregate_update(const uint32_t *idx, const float *val, uint32_t n,
                                      uint64_t k, uint64_t d, float eta, float scale,
                                      float *omega, void *workspace, uint64_t workspace_bytes,
                                      void *stream_v)
{
    uint64_t need = 0;
    if (!idx || !val || !omega || rtopk_aggregate_update_workspace_bytes(d, n, k, &need) != RTOPK_OK)
        return RTOPK_EINVAL;
    if (n > 65535u) return RTOPK_EINVAL;                // workers are a grid dimension
    if (!workspace || ((uintptr_t)workspace & 255u) || workspace_bytes < need)
        return RTOPK_EWORKSPACE;
    return launch_update(idx, val, n, k, d, eta, scale, omega, static_cast<u32 *>(workspace),
                         (hipStream_t)stream_v);
}

// ---------------------------------------------------------------------------
// rtopk_aggregate_update_static: the same two kernels with the tile-start
// table in a device array that is part of the library's code object, for
// callers that can neither allocate nor pass a workspace. Every device the
// library runs on holds its own copy of the array at its own address; the
// address is looked up once per device, with that device current, and kept.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[RTOPK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxScratchDevices];      // device address of `scratch`, per device

int static_scratch(void **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return RTOPK_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        // in host code the array's name is only a handle: the device address comes from here
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return RTOPK_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RTOPK_OK;
}
}  // namespace

extern "C" int rtopk_aggregate_update_static(const uint32_t *idx, const float *val, uint32_t n,
                                             uint64_t k, uint64_t d, float eta, float scale,
                                             float *omega, void *stream_v)
{
    uint64_t need = 0;
    if (!idx || !val || !omega || rtopk_aggregate_update_workspace_bytes(d, n, k, &need) != RTOPK_OK)
        return RTOPK_EINVAL;
    if (n > 65535u) return RTOPK_EINVAL;
    if (need > (uint64_t)RTOPK_STATIC_SCRATCH_BYTES) return RTOPK_ETOOLARGE;
    void *table = nullptr;
    const int rc = static_scratch(&table);
    if (rc) return rc;
    // k_tile_starts writes every word of the table that k_update reads, so
    // nothing of what the previous call left in the array has to be cleared
    return launch_update(idx, val, n, k, d, eta, scale, omega, static_cast<u32 *>(table),
                         (hipStream_t)stream_v);
}

extern "C" const char *rtopk_strerror(int code)
{
    switch (code) {
    case RTOPK_OK: return "ok";
    case RTOPK_EINVAL: return "invalid argument (null pointer, sizes outside 1 <= k <= r <= d < 2^32, n < 1, or grad overlaps residual)";
    case RTOPK_EWORKSPACE: return "workspace missing, not 256-byte aligned, or too small";
    case RTOPK_EHIP: return "a HIP call or kernel launch failed";
    case RTOPK_ETOOLARGE: return "sizes exceed the library's built-in scratch array (rtopk_aggregate_update_static needs 4 bytes per worker and per 2048 coordinates within RTOPK_STATIC_SCRATCH_BYTES); use the entry point that takes a workspace";
    default: return "unknown rtopk error code";
    }
}

extern "C" int rtopk_version(void) { return 200; }

// 1 when the library was built with RTOPK_DEBUG_CHECKS, else 0
extern "C" int rtopk_debug_checks(void)
{
#ifdef RTOPK_DEBUG_CHECKS
    return 1;
#else
    return 0;
#endif
}
