// Exact farthest point sampling and MDPS (Algorithms 1 and 2 of FastPoint, arXiv 2507.23480) by local decisions, for gfx950.
//
// The sequence of Alg. 1 is found without following it.  d_i is a point's squared distance to the samples found
// so far.  Say k comes before i when d_k > d_i, or d_k == d_i and k has the lower index.  Then
//
//   * i is a sample, found at distance d_i, as soon as no point that comes before it lies closer to it than d_i:
//     distances only fall, so whatever Alg. 1 takes before i comes before i now, and leaves d_i as it is;
//   * a sample k found at v_k lowers a point j to dist(j, k) exactly when dist(j, k) < min(d_j, v_k).  (If dist(j, k)
//     >= v_k, every distance is at most v_k <= dist(j, k) by the time Alg. 1 takes k.  If dist(j, k) < v_k and Alg. 1
//     took j before k, j would come before k now and k would have waited.)
//   * Alg. 1 takes the samples in the order (v descending, index ascending).
//
// So all points that are the first of their own neighbourhood are taken at once, wherever they lie, and the
// samples are put in sequence at the end (order_samples_kernel).  A round looks at the candidates, all points
// with d > tau; tau falls as the list has room.  To end with exactly n samples a candidate is only taken
// when the candidates that come before it leave room for it.
//
// One cloud is held by G workgroups for the whole call, points and distances in registers, in the order of a Hilbert
// curve.  Per round:
//   scan     every workgroup counts its points above four falling levels of tau and publishes the counts and the
//            points, the ones above the highest level first;
//   list     all workgroups read the counts, agree on the lowest level at which the list fits (the first level is the
//            last round's tau, whose list can only have got shorter), and fetch that list into LDS, with a box around
//            every 64 candidates (neighbours in the list are neighbours along the curve);
//   decide   each workgroup takes an equal share of the list, a wave per candidate, which is compared with the chunks
//            whose box it reaches; the decisions, one bit per candidate, go to the other workgroups;
//   fold     every wave folds the samples near the boxes of its points.
// Where the list does not help (many equal distances, infinities) one sample is taken by a plain arg-max.
//
// The threshold phase of Algorithm 2 runs in the same rounds (threshold_rounds): there a point comes before another by its
// key, and the radius is the level's.  MDPS takes two launches, for the prefix and for the rest: the thresholds need the
// prefix's curve in sequence.
//
// Bound: latency.  A round takes 11 us on 24 workgroups, 15 on 64, 17 on 245: three trips through memory (counts 2-4.7 us with the
// wait for the slowest workgroup, list 2-4.5, decisions 2-2.6), the rest of its parts 1-2 us each.  Rounds of exact FPS for the
// workloads below: 85, 56 and 40, against 436, 207 and 82 rounds of 256 candidates settled in sweeps before (94, 67 and 43 with
// lists that ended where half a workgroup had more than 191 points).
// us, before -> now: fps_exact_pruned million points -> 65536 5190 -> 1600, 4 x 120000 -> 16384 2750 -> 960, 8 x 24000 -> 6000
// 850 -> 525; mdps_sample_pruned in the scattered order with record 6250 -> 2080, 4530 -> 2320, 1070 -> 830.  (1024 threads; with
// 512 and twice the points per thread exact FPS took 10, 8 and 1 % longer.)  Comparing a candidate with the whole list instead
// of the chunks near it took 10-20 us a round.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "estimator.h"
#include "kernels.h"
#include "wave.h"

#pragma clang fp contract(off)

namespace fastpoint {
namespace {

constexpr int kT = kLocalThreads, kNW = kT / 64, kHW = kNW / 2;
constexpr int kList = kLocalList;           // candidates of a round
constexpr int kChunks = kList / 64;
constexpr int kOwn = kLocalOwn;             // candidates half a workgroup lists
constexpr int kWords = kLocalMaskWords;     // words of 32 decisions a workgroup publishes
constexpr int kUnit = 8;                    // the list is dealt out in units of 8 candidates for the decisions
constexpr int kLevels = 4;
constexpr int kSettle = 768;                // candidates settled in order (threshold_rounds)
constexpr int kSpans = kMaxGroup / 32;      // of 64 halves
constexpr int32_t kFull = 1 << 20;
static_assert(kLocalList == 4096 && kOwn < 1023, "a count has 12 bits, 64 of them at most kOwn + 1 each 16");
static_assert(kLevels == 4 && kSpans * kLevels == 32, "a lane per sum");
static_assert(kChunks == 64, "a lane per chunk");

struct Box {
    float lox, loy, loz, hix, hiy, hiz;
};

struct LocalShared {
    Box wbox[kNW][2];                       // boxes of a wave's points, before and behind the widest gap in their run
    float4 cand[kList];                     // x, y, z, index bits
    uint32_t dist[kList];                   // zero behind the last candidate, to the end of its chunk
    float box[7][kChunks];                  // per chunk of 64 candidates: lower corner, upper corner, largest distance
    uint64_t took[kChunks];                 // the round's samples, a bit per candidate
    unsigned long long cnt[2][2];           // per half, points above each level, 16 bits each (of this round and of the next)
    int32_t inc[2][2 * kMaxGroup];          // sums of the halves' counts inside 64 of them, two levels in a word
    int32_t tot[kSpans][kLevels];           // ... of all 64, kFull more where a half has more than it can list
    uint32_t acc[kList / 32];               // decisions on the candidates of this workgroup's part of the list
    int32_t fail;
    int32_t in_order;                       // follow_order: samples known to be in sequence
    Rec wrec[2][kNW];
    Rec win[2];
    uint64_t settled[kSettle / 64];         // settle_in_order: samples among 64 candidates that follow each other
};

// Threshold phase: where the thresholds are worked out, and the bookkeeping of the levels.
struct LevelShared {
    float ring[64];
    float thr_meas[FP_MAX_SEG], thr[FP_MAX_SEG];
    double terms[64], powb[FP_MAX_SEG];
    float mlp_val[32];
    double mlp_a[128], mlp_b[128];
    int32_t level_start[FP_MAX_SEG], level_exhausted[FP_MAX_SEG];
};

template <int P>
struct Held {
    float x[P], y[P], z[P], d[P];
    uint32_t oi[P];                         // index in the caller's cloud
    uint32_t key[P];                        // threshold phase: place in the scan order
    uint32_t bq_next, bq_room;              // recording: next entry of the wave's chunk, entries left in it
    bool bq_dead;                           // ... no chunk was left: nothing more is recorded for this cloud
    float ub;                               // largest distance among them
};

#ifdef FASTPOINT_PHASE_CLOCKS
__shared__ long long clk[16];               // tuning builds: ticks of thread 0 in the parts of a round, left behind the words of the decisions
__shared__ long long clk_at;
#define MARK(k) do { if (threadIdx.x == 0) { const long long now__ = wall_clock64(); clk[k] += now__ - clk_at; clk_at = now__; } } while (0)
#else
#define MARK(k) do { } while (0)
#endif

// Half a workgroup, its first or last kHW waves, holds 512 P records that follow each other; the halves of a workgroup lie half
// the cloud apart (space is filled unevenly, and a workgroup is as slow as its busiest waves).
struct Seat {
    int tid, lane, w, g, G, grp, c;
    int half;                               // half of the cloud's 2 G the wave belongs to: its place along the curve
};

// Evaluated like dist2 with the nearest box coordinate per axis: rounding is monotone, so no point of the box is closer.
__device__ __forceinline__ float sum_sq(float dx, float dy, float dz)
{
    float t = dx * dx;
    t = t + dy * dy;
    t = t + dz * dz;
    return t;
}
__device__ __forceinline__ float box_dist2(const Box& h, float cx, float cy, float cz)
{
    return sum_sq(fmaxf(fmaxf(h.lox - cx, cx - h.hix), 0.0f), fmaxf(fmaxf(h.loy - cy, cy - h.hiy), 0.0f),
                  fmaxf(fmaxf(h.loz - cz, cz - h.hiz), 0.0f));
}
__device__ __forceinline__ float box_box2(const Box& h, const Box& o)
{
    return sum_sq(fmaxf(fmaxf(h.lox - o.hix, o.lox - h.hix), 0.0f), fmaxf(fmaxf(h.loy - o.hiy, o.loy - h.hiy), 0.0f),
                  fmaxf(fmaxf(h.loz - o.hiz, o.loz - h.hiz), 0.0f));
}
// floats as integers of the same order
__device__ __forceinline__ uint32_t f2ord(float v)
{
    const uint32_t u = __float_as_uint(v);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float ord2f(uint32_t u)
{
    return __uint_as_float(u ^ ((u >> 31) != 0 ? 0x80000000u : 0xFFFFFFFFu));
}
// (a distance that is not a number is larger than any other as an integer: such a point keeps its distance)
template <int P>
__device__ __forceinline__ void fold(Held<P>& h, float cx, float cy, float cz, float v)
{
    if (v >= h.ub) {                        // uniform: no distance of the wave exceeds v
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint32_t t = __float_as_uint(dist2(cx, cy, cz, h.x[p], h.y[p], h.z[p]));
            h.d[p] = __uint_as_float(min(__float_as_uint(h.d[p]), t));
        }
    } else {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float t = dist2(cx, cy, cz, h.x[p], h.y[p], h.z[p]);
            const float m = __uint_as_float(min(__float_as_uint(h.d[p]), __float_as_uint(t)));
            h.d[p] = t < v ? m : h.d[p];
        }
    }
}

// The same for a sample whose ball reaches the wave: with the radius test of Section 4.2.  The hits of each block of 64 records
// become an entry of the cloud's list (kernels.h) under the sample's index; lane p hands on block p.  A wave fills a chunk
// of entries at a time and waits for the next one to be handed out.
template <int P>
__device__ __forceinline__ void fold_record(Held<P>& h, const Seat& me, const LocalArgs& a, float cx, float cy, float cz, float v,
                                            uint32_t idx)
{
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const float t = dist2(cx, cy, cz, h.x[p], h.y[p], h.z[p]);
        const float m = __uint_as_float(min(__float_as_uint(h.d[p]), __float_as_uint(t)));
        h.d[p] = t < v ? m : h.d[p];
        const uint64_t hits = __builtin_amdgcn_ballot_w64(t < a.bq_r2);
        set_lane(lo, me.lane, p, (uint32_t)hits);
        set_lane(hi, me.lane, p, (uint32_t)(hits >> 32));
    }
    const uint64_t some = __builtin_amdgcn_ballot_w64((lo | hi) != 0);
    if (some == 0 || h.bq_dead) return;     // uniform
    const uint32_t nchunks = (uint32_t)(a.bq_cap / kBqChunk);
    uint32_t* const fill = a.bq_fill + (int64_t)me.c * nchunks;
    const int total = (int)__builtin_popcountll(some), place = lanes_below(some);
    int done = 0;
    while (done < total) {
        if (h.bq_room == 0) {
            uint32_t ch = 0;
            if (me.lane == 0) ch = __hip_atomic_fetch_add(a.bq_cursor + me.c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ch = uni(ch);
            if (ch >= nchunks) {
                if (me.lane == 0) a.bq_ovf[me.c] = 1u;
                h.bq_dead = true;
                return;
            }
            h.bq_next = ch * (uint32_t)kBqChunk;
            h.bq_room = (uint32_t)kBqChunk;
        }
        const int take = total - done < (int)h.bq_room ? total - done : (int)h.bq_room;
        const int i = place - done;
        if (((some >> me.lane) & 1ull) != 0 && i >= 0 && i < take) {
            BqRaw e;
            e.mask = ((uint64_t)hi << 32) | lo;
            e.blk = (uint32_t)((me.half * kHW + (me.w & (kHW - 1))) * P + me.lane);
            e.q = idx;
            a.bq_raw[(int64_t)me.c * a.bq_cap + h.bq_next + (uint32_t)i] = e;
        }
        h.bq_next += (uint32_t)take;
        h.bq_room -= (uint32_t)take;
        done += take;
        if (h.bq_room == 0 && me.lane == 0) fill[h.bq_next / (uint32_t)kBqChunk - 1u] = (uint32_t)kBqChunk;
    }
}

template <int P>
__device__ __forceinline__ void refresh_bound(Held<P>& h)
{
    uint32_t m = __float_as_uint(h.d[0]);   // distances are >= +0: unsigned order
#pragma unroll
    for (int p = 1; p < P; ++p) m = max(m, __float_as_uint(h.d[p]));
    h.ub = __uint_as_float(wave_max_u32(m));
}

// Where a wave with points keeps its place in the record from one launch to the next.
__device__ __forceinline__ uint2& bq_place(const LocalArgs& a, const Seat& me, int P)
{
    return a.bq_at[(int64_t)me.c * ((a.N + 64 * P - 1) / (64 * P)) + me.half * kHW + (me.w & (kHW - 1))];
}

// Loads the wave's points and finds their boxes.  (Where the curve leaves a thin layer of occupied cells and comes back
// elsewhere, one box would span the cloud and the wave would fold every sample: 7000 to 10000 of 16384 instead of
// some 400 for one or two waves of a LiDAR sweep.)
template <int P, bool BQ, bool MDPS>
__device__ __forceinline__ void load_points(Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a)
{
    const float4* __restrict__ rec = a.sorted + (int64_t)me.c * a.N;
    const int base = (me.half * kHW + (me.w & (kHW - 1))) * P * 64;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int j = base + p * 64 + me.lane;
        h.x[p] = h.y[p] = h.z[p] = kPadCoord;
        h.oi[p] = kNoIdx;
        h.d[p] = 0.0f;
        if (j < a.N) {
            const float4 r = rec[j];
            h.x[p] = r.x;
            h.y[p] = r.y;
            h.z[p] = r.z;
            h.oi[p] = __float_as_uint(r.w);
            h.d[p] = MDPS ? a.dist[(int64_t)me.c * a.N + j] : __builtin_inff();
            if constexpr (BQ && !MDPS) a.bq_map[(int64_t)me.c * a.N + j] = (int32_t)h.oi[p];
        }
        if constexpr (MDPS)                 // place t of index j in the walk j = (t A) mod N, or the index itself
            h.key[p] = a.walk_inv != 0 && j < a.N ? (uint32_t)(((uint64_t)h.oi[p] * a.walk_inv) % (uint64_t)a.N) : h.oi[p];
    }
    h.bq_dead = false;
    h.bq_next = h.bq_room = 0;
    if constexpr (BQ && MDPS) {
        if (base < a.N) {                   // (a wave without points records nothing)
            const uint2 at = bq_place(a, me, P);
            h.bq_next = uni(at.x);
            h.bq_room = uni(at.y) & 0xFFu;
            h.bq_dead = (uni(at.y) >> 8) != 0;
        }
    }
    // the widest gap between two records that follow each other
    uint32_t gap = 0, at = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float nx = __shfl_down(h.x[p], 1), ny = __shfl_down(h.y[p], 1), nz = __shfl_down(h.z[p], 1);
        const int q = p + 1 < P ? p + 1 : p;
        if (me.lane == 63) {
            nx = rdlane_f(h.x[q], 0);
            ny = rdlane_f(h.y[q], 0);
            nz = rdlane_f(h.z[q], 0);
        }
        const int j = base + p * 64 + me.lane;
        const uint32_t t = __float_as_uint(dist2(h.x[p], h.y[p], h.z[p], nx, ny, nz));
        if (j + 1 < a.N && (me.lane < 63 || p + 1 < P) && t > gap) {
            gap = t;
            at = (uint32_t)(p * 64 + me.lane);
        }
    }
    const uint32_t widest = wave_max_u32(gap);
    const uint32_t cut = rdlane(at, first_lane(__builtin_amdgcn_ballot_w64(gap == widest)));
    uint32_t lo[2][3], hi[2][3];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            lo[s][k] = 0xFF800000u;
            hi[s][k] = 0x007FFFFFu;
        }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint32_t c[3] = {f2ord(h.x[p]), f2ord(h.y[p]), f2ord(h.z[p])};
        const bool in = base + p * 64 + me.lane < a.N, second = (uint32_t)(p * 64 + me.lane) > cut;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (in && !second) {
                lo[0][k] = min(lo[0][k], c[k]);
                hi[0][k] = max(hi[0][k], c[k]);
            }
            if (in && second) {
                lo[1][k] = min(lo[1][k], c[k]);
                hi[1][k] = max(hi[1][k], c[k]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        Box b;
        b.lox = ord2f(wave_min_u32(lo[e][0]));
        b.loy = ord2f(wave_min_u32(lo[e][1]));
        b.loz = ord2f(wave_min_u32(lo[e][2]));
        b.hix = ord2f(wave_max_u32(hi[e][0]));
        b.hiy = ord2f(wave_max_u32(hi[e][1]));
        b.hiz = ord2f(wave_max_u32(hi[e][2]));
        if (me.lane == 0) sh.wbox[me.w][e] = b;             // (read by this wave alone)
    }
}

// One iteration of Alg. 1 on up-to-date distances: arg-max over the cloud, lowest index among equals.
template <int P>
__device__ __forceinline__ Rec plain_pick(const Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a,
                                          uint32_t& it, uint32_t& seq)
{
    uint32_t bits = __float_as_uint(h.d[0]), boi = h.oi[0];
    float bx = h.x[0], by = h.y[0], bz = h.z[0];
#pragma unroll
    for (int p = 1; p < P; ++p) {
        const uint32_t v = __float_as_uint(h.d[p]);
        if (v > bits || (v == bits && h.oi[p] < boi)) {
            bits = v;
            boi = h.oi[p];
            bx = h.x[p];
            by = h.y[p];
            bz = h.z[p];
        }
    }
    Rec r;
    r.d = bits;
    r.idx = boi;
    r.x = bx;
    r.y = by;
    r.z = bz;
    r.fail = r.pad0 = r.pad1 = 0;
    r = reduce_recs(r, true);
    const int buf = (int)(it & 1u);
    ++it;
    if (me.lane == 0) sh.wrec[buf][me.w] = r;
    __syncthreads();
    r = reduce_recs(sh.wrec[buf][me.lane < kNW ? me.lane : 0], me.lane < kNW);
    if (me.G == 1) return r;
    ++seq;
    if (me.w == 0) {
        uint64_t* base = a.ll_pk + ((int64_t)(me.grp * 2 + (int)(seq & 1u)) * me.G) * kLlSlotWords;
        uint32_t v = r.d;
        v = me.lane == 1 ? r.idx : v;
        v = me.lane == 2 ? __float_as_uint(r.x) : v;
        v = me.lane == 3 ? __float_as_uint(r.y) : v;
        v = me.lane == 4 ? __float_as_uint(r.z) : v;
        if (me.lane < 5) ll_store(base + (int64_t)me.g * kLlSlotWords + me.lane, v, seq);
        Rec best = {};
        best.idx = kNoIdx;
        bool have = false;
        for (int t = me.lane; t < me.G; t += 64) {
            uint32_t val[5];
            if (!ll_wait<5>(base + (int64_t)t * kLlSlotWords, seq, val, a.wait_ticks)) {
                best.fail = 1;
            } else if (!have || val[0] > best.d || (val[0] == best.d && val[1] < best.idx)) {
                best.d = val[0];
                best.idx = val[1];
                best.x = __uint_as_float(val[2]);
                best.y = __uint_as_float(val[3]);
                best.z = __uint_as_float(val[4]);
            }
            have = true;
        }
        const Rec all = reduce_recs(best, have);
        if (me.lane == 0) sh.win[buf] = all;
    }
    __syncthreads();
    return sh.win[buf];
}

// A published candidate: three words with a stamp of 14 bits each around distance (31 bits, it is not negative),
// coordinates and index (21 bits).  The stamp is never 0 and does not come twice in the rounds up to the next one whose
// last bits (kWipe) are zero, in front of which the words are cleared.
constexpr int kCandWords3 = kLocalCandWords;
constexpr uint32_t kWipe = kLocalStampRounds - 1;
static_assert((kLocalStampRounds >> 1) < 1 << 14, "14 bits for a stamp");
static_assert(kMaxGroup * 8192 <= 1 << 21, "21 bits for an index");
constexpr int64_t kHalfWords = (int64_t)(kOwn + 1) * kCandWords3;
__device__ __forceinline__ uint64_t* half_list(const LocalArgs& a, const Seat& me, int par, int half)
{
    return a.ll_list + ((int64_t)(me.grp * 2 + par) * (2 * me.G) + half) * kHalfWords;
}
__device__ __forceinline__ void word_store(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cand_store(uint64_t* p, uint32_t stamp, float x, float y, float z, uint32_t idx, uint32_t d)
{
    const uint64_t st = (uint64_t)stamp << 50;
    const uint32_t yb = __float_as_uint(y);
    word_store(p, st | ((uint64_t)(idx & 0x7FFFFu) << 31) | d);
    word_store(p + 1, st | ((uint64_t)(yb >> 14) << 32) | __float_as_uint(x));
    word_store(p + 2, st | ((uint64_t)(yb & 0x3FFFu) << 34) | ((uint64_t)(idx >> 19) << 32) | __float_as_uint(z));
}
__device__ __forceinline__ bool cand_wait(const uint64_t* p, uint32_t stamp, uint64_t (&v)[kCandWords3], int64_t wait_ticks)
{
    int64_t t0 = 0;
    for (uint32_t spin = 0; (uint32_t)(v[0] >> 50) != stamp || (uint32_t)(v[1] >> 50) != stamp || (uint32_t)(v[2] >> 50) != stamp;
         ++spin) {
        if ((spin & 63u) == 63u || wait_ticks <= 0) {
            const int64_t now = (int64_t)wall_clock64();
            if (t0 == 0) t0 = now;
            else if (now - t0 > wait_ticks) return false;
        }
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int k = 0; k < kCandWords3; ++k) v[k] = ll_load(p + k);
    }
    return true;
}
// The counts of a half: a word with such a stamp around four of 12 bits each; waited for like ll_wait_close.
__device__ __forceinline__ bool hdr_wait(const uint64_t* p, uint32_t stamp, uint64_t& val, int64_t wait_ticks)
{
    constexpr int N = 4;
    uint64_t v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        v[k] = ll_load(p);
        if (k + 1 < N) __builtin_amdgcn_s_sleep(3);
    }
    int64_t t0 = 0;
    for (uint32_t spin = 0;; ++spin) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if ((uint32_t)(v[k] >> 50) == stamp) {
                val = v[k];
                return true;
            }
            v[k] = ll_load(p);
        }
        if ((spin & 15u) == 15u || wait_ticks <= 0) {
            const int64_t now = (int64_t)wall_clock64();
            if (t0 == 0) t0 = now;
            else if (now - t0 > wait_ticks) return false;
        }
    }
}
__device__ __forceinline__ float4 cand_unpack(const uint64_t (&v)[kCandWords3], uint32_t& d)
{
    d = (uint32_t)v[0] & 0x7FFFFFFFu;
    const uint32_t idx = ((uint32_t)(v[0] >> 31) & 0x7FFFFu) | (((uint32_t)(v[2] >> 32) & 3u) << 19);
    const uint32_t yb = (((uint32_t)(v[1] >> 32) & 0x3FFFFu) << 14) | ((uint32_t)(v[2] >> 34) & 0x3FFFu);
    return make_float4(__uint_as_float((uint32_t)v[1]), __uint_as_float(yb), __uint_as_float((uint32_t)v[2]), __uint_as_float(idx));
}

// Box and largest distance of a chunk, whose candidates the lanes of a wave hold.
// (Eight maxima over the wave at once: pairs of lanes share the eight values out, then groups of four lanes, so that
// each lane reduces two of them over its row of 16; 50 instructions instead of 95 for one after the other.)
__device__ __forceinline__ void chunk_box(LocalShared& sh, int chunk, int lane, const float4& c, uint32_t d, bool has)
{
    uint32_t v[8];
    v[0] = f2ord(c.x);
    v[1] = f2ord(c.y);
    v[2] = f2ord(c.z);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        v[4 + k] = has ? v[k] : 0u;
        v[k] = has ? ~v[k] : 0u;
    }
    v[3] = has ? d : 0u;
    v[7] = 0u;
    uint32_t r[4], q[2];
    const bool odd = (lane & 1) != 0, upper = (lane & 2) != 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t keep = odd ? v[4 + k] : v[k], give = odd ? v[k] : v[4 + k];
        r[k] = max(keep, dpp<0xB1>(give));              // quad_perm [1,0,3,2]
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t keep = upper ? r[2 + k] : r[k], give = upper ? r[k] : r[2 + k];
        q[k] = max(keep, dpp<0x4E>(give));              // quad_perm [2,3,0,1]
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        q[k] = max(q[k], dpp<0x124>(q[k]));             // row_ror:4
        q[k] = max(q[k], dpp<0x128>(q[k]));             // row_ror:8
        q[k] = max(q[k], (uint32_t)__shfl_xor((int)q[k], 16));
        q[k] = max(q[k], (uint32_t)__shfl_xor((int)q[k], 32));
    }
    if (lane < 4) {
        // lane 0: lower x, y; 2: lower z, distance; 1: upper x, y; 3: upper z
        const int first = (odd ? 4 : 0) + (upper ? 2 : 0);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = first + k;
            const float f = e < 3 ? ord2f(~q[k]) : (e == 3 ? __uint_as_float(q[k]) : ord2f(q[k]));
            if (e != 7) sh.box[e < 3 ? e : (e == 3 ? 6 : e - 1)][chunk] = f;
        }
    }
}
__device__ __forceinline__ Box box_of_chunk(const LocalShared& sh, int chunk)
{
    return Box{sh.box[0][chunk], sh.box[1][chunk], sh.box[2][chunk], sh.box[3][chunk], sh.box[4][chunk], sh.box[5][chunk]};
}

// A round's candidates.  Exact FPS: the points with d > level, the farther first, which are samples unless a point before
// them lies closer than their own distance.  Threshold phase (KEYED): the available points, d >= r2, with keys in front
// of a window's end, the lower key first, samples unless one before them lies closer than r2.  A candidate goes by
// its priority, the distance bits or kTopKey - key.
constexpr uint32_t kTopKey = 0x7FFFFFFFu;
struct Levels {
    float r2;                               // KEYED: the level's squared radius
    float d[kLevels];                       // four falling levels ...
    uint32_t end[kLevels];                  // ... or growing windows
};
template <bool KEYED, int P>
__device__ __forceinline__ bool listed(const Held<P>& h, const Levels& lv, int p, int j)
{
    if constexpr (KEYED) return h.d[p] >= lv.r2 && h.key[p] < lv.end[j];
    return h.d[p] > lv.d[j];
}

// Scan and list of a round.  Returns the length of the list (-1: a wait expired) and the level chosen.
template <int P, bool KEYED>
__device__ __forceinline__ int make_list(const Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a,
                                         uint32_t round, const Levels& lv, int aim, int& level)
{
    uint32_t c[kLevels] = {};
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(listed<KEYED>(h, lv, p, kLevels - 1));
        if (m != 0) {
            c[kLevels - 1] += __builtin_popcountll(m);
#pragma unroll
            for (int j = 0; j < kLevels - 1; ++j)
                c[j] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(listed<KEYED>(h, lv, p, j)));
        }
    }
    // where the wave's points lie among those of its half, in the order the waves get here (one workgroup for the cloud:
    // no halves)
    const int par = (int)(round & 1u), hf = me.G > 1 && me.w >= kHW ? 1 : 0;
    uint64_t before = 0;
    if (me.lane == 0 && c[kLevels - 1] != 0)
        before = atomicAdd(&sh.cnt[par][hf], (uint64_t)c[0] | ((uint64_t)c[1] << 16) | ((uint64_t)c[2] << 32) | ((uint64_t)c[3] << 48));
    __syncthreads();
    MARK(0);
    const uint64_t sum = uni64(sh.cnt[par][hf]);
    int tot[kLevels];
#pragma unroll
    for (int j = 0; j < kLevels; ++j) tot[j] = (int)((uint32_t)(sum >> (16 * j)) & 0xFFFFu);
    const int halves = 2 * me.G;
    uint64_t* const hdr = a.ll_hdr + (int64_t)(me.grp * 2 + par) * halves;
    const uint32_t stamp = ((round & kWipe) >> 1) + 1u;
    if (me.G > 1) {
        if (me.lane == 0 && (me.w & (kHW - 1)) == 0) {
            uint64_t v = (uint64_t)stamp << 50;
#pragma unroll
            for (int j = 0; j < kLevels; ++j) v |= (uint64_t)(uint32_t)(tot[j] <= kOwn ? tot[j] : kOwn + 1) << (12 * j);
            word_store(hdr + me.half, v);
        }
        level = kLevels - 1;
    } else {
        level = 0;
#pragma unroll
        for (int j = 1; j < kLevels; ++j) level = tot[j] <= aim ? j : level;
    }
    if (me.tid < kList / 32) sh.acc[me.tid] = 0;            // (last looked at before the barrier)
    if (me.tid < kChunks) sh.took[me.tid] = 0;
    if (me.tid < 2) sh.cnt[par ^ 1][me.tid] = 0;
    if (c[kLevels - 1] != 0) {
        // the points above level j lie behind those above level j - 1
        const uint64_t start = uni64((sum << 16) + before - (before << 16));
        uint32_t at[kLevels];
#pragma unroll
        for (int j = 0; j < kLevels; ++j) at[j] = (uint32_t)(start >> (16 * j)) & 0xFFFFu;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(listed<KEYED>(h, lv, p, kLevels - 1));
            if (m == 0) continue;
            const uint32_t prio = KEYED ? kTopKey - h.key[p] : __float_as_uint(h.d[p]);
            int pos = kList;
            uint64_t seen = 0;
#pragma unroll
            for (int j = 0; j < kLevels; ++j) {
                const uint64_t mj = (j == kLevels - 1 ? m : __builtin_amdgcn_ballot_w64(listed<KEYED>(h, lv, p, j))) & ~seen;
                seen |= mj;
                if (mj != 0 && j <= level) {
                    if (((mj >> me.lane) & 1ull) != 0) pos = (int)at[j] + lanes_below(mj);
                    at[j] += __builtin_popcountll(mj);
                }
            }
            if (me.G > 1) {
                if (pos < kOwn)
                    cand_store(half_list(a, me, par, me.half) + pos * kCandWords3, stamp, h.x[p], h.y[p], h.z[p], h.oi[p],
                               prio);
            } else if (pos < kList) {
                sh.cand[pos] = make_float4(h.x[p], h.y[p], h.z[p], __uint_as_float(h.oi[p]));
                sh.dist[pos] = prio;
            }
        }
    }
    MARK(1);
    int total;
    if (me.G == 1) {
        total = tot[0];
#pragma unroll
        for (int j = 1; j < kLevels; ++j) total = j == level ? tot[j] : total;
        if (me.tid < (-total & 63)) sh.dist[total + me.tid] = 0;
        __syncthreads();
        for (int k = me.w; 64 * k < total; k += kNW) {
            const int r = 64 * k + me.lane;
            chunk_box(sh, k, me.lane, sh.cand[r], sh.dist[r], r < total);
        }
    } else {
        const int spans = (halves + 63) >> 6;
        if (me.w < spans) {                                 // a wave takes 64 halves
            uint64_t v = 0;
            bool bad = false;
            if (me.tid < halves) bad = !hdr_wait(hdr + me.tid, stamp, v, a.wait_ticks);
            v = bad ? 0u : v;
            uint32_t n[kLevels];
#pragma unroll
            for (int j = 0; j < kLevels; ++j) n[j] = (uint32_t)(v >> (12 * j)) & 0xFFFu;
            int mine = 0;
#pragma unroll
            for (int k = 0; k < kLevels / 2; ++k) {
                const uint32_t s = (uint32_t)wave_incl_sum((int)(n[2 * k] | (n[2 * k + 1] << 16)), me.lane);
                sh.inc[k][me.tid] = (int32_t)s;
                const uint32_t all = rdlane(s, 63);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int full = __builtin_amdgcn_ballot_w64(n[2 * k + e] > (uint32_t)kOwn) != 0 ? kFull : 0;
                    mine = me.lane == 2 * k + e ? (int)((all >> (16 * e)) & 0xFFFFu) + full : mine;
                }
            }
            if (me.lane < kLevels) sh.tot[me.w][me.lane] = mine;
            if (__builtin_amdgcn_ballot_w64(bad) != 0 && me.lane == 0) sh.fail = 1;
        }
        __syncthreads();
        MARK(2);
        // lane 4 q + j: level j in the q-th 64 halves
        const int part = me.lane < kSpans * kLevels ? reinterpret_cast<const int32_t*>(sh.tot)[me.lane] : 0;
        int sum = part + (int)dpp<0x124>((uint32_t)part);   // row_ror:4
        sum += (int)dpp<0x128>((uint32_t)sum);              // row_ror:8
        sum += __shfl_xor(sum, 16);
        const uint64_t fits = __builtin_amdgcn_ballot_w64(sum <= aim) & ((1u << kLevels) - 2u);
        level = fits != 0 ? 63 - __builtin_clzll(fits) : 0;
        total = (int)rdlane((uint32_t)sum, level);
        const int shift = (level & 1) * 16;
        const int32_t* const inc = sh.inc[level >> 1];
        // candidates listed before each 64 halves
        int bases[kSpans];
        bases[0] = 0;
#pragma unroll
        for (int k = 1; k < kSpans; ++k)
            bases[k] = k < spans ? bases[k - 1] + (int)rdlane((uint32_t)part, kLevels * (k - 1) + level) : kList;
        if (uni(sh.fail) == 0) {
            constexpr int NE = 2;           // chunks a wave has under way at a time
            for (int k0 = me.w; 64 * k0 < total; k0 += NE * kNW) {
                uint64_t got[NE][kCandWords3];
                const uint64_t* src[NE];
#pragma unroll
                for (int u = 0; u < NE; ++u) {
                    const int r = 64 * (k0 + u * kNW) + me.lane;
                    src[u] = nullptr;
#pragma unroll
                    for (int e = 0; e < kCandWords3; ++e) got[u][e] = 0;
                    if (r < total) {
                        // the half that lists the r-th candidate: the first whose sum exceeds r
                        int q = 0, rr = r;
#pragma unroll
                        for (int k = 1; k < kSpans; ++k)
                            if (r >= bases[k]) {
                                q = k;
                                rr = r - bases[k];
                            }
                        int g = 0;
#pragma unroll
                        for (int s = 32; s > 0; s >>= 1)
                            if ((int)(((uint32_t)inc[64 * q + g + s - 1] >> shift) & 0xFFFFu) <= rr) g += s;
                        const int first = g > 0 ? (int)(((uint32_t)inc[64 * q + g - 1] >> shift) & 0xFFFFu) : 0;
                        src[u] = half_list(a, me, par, 64 * q + g) + (rr - first) * kCandWords3;
#pragma unroll
                        for (int e = 0; e < kCandWords3; ++e) got[u][e] = ll_load(src[u] + e);
                    }
                }
#pragma unroll
                for (int u = 0; u < NE; ++u) {
                    const int k = k0 + u * kNW, r = 64 * k + me.lane;
                    if (64 * k >= total) break;             // uniform
                    float4 c = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    uint32_t d = 0;
                    if (r < total) {
                        if (cand_wait(src[u], stamp, got[u], a.wait_ticks)) c = cand_unpack(got[u], d);
                        else sh.fail = 1;
                    }
                    sh.cand[r] = c;
                    sh.dist[r] = d;
                    chunk_box(sh, k, me.lane, c, d, r < total);
                }
            }
        }
    }
    __syncthreads();
    MARK(4);
    return uni(sh.fail) != 0 ? -1 : total;
}

// Decides this workgroup's part of the list and leaves the round's samples, of all workgroups, in sh.took.
// Returns their number, -1 if a wait expired.
template <bool KEYED>
__device__ __forceinline__ int decide(LocalShared& sh, const Seat& me, const LocalArgs& a, uint32_t round, int total,
                                      int room, float r2)
{
    const bool ranked = room < total;                   // uniform
    const int units = (total + kUnit - 1) / kUnit, chunks = (total + 63) >> 6;
    const int lo = (int)((uint32_t)(units * me.g) / (uint32_t)me.G) * kUnit;
    int hi = (int)((uint32_t)(units * (me.g + 1)) / (uint32_t)me.G) * kUnit;
    hi = hi < total ? hi : total;
    const int mine = me.lane < chunks ? me.lane : 0;    // lane l: chunk l
    const Box cb = box_of_chunk(sh, mine);
    const uint32_t far = me.lane < chunks ? __float_as_uint(sh.box[6][mine]) : 0u;
    for (int i = lo + me.w; i < hi; i += kNW) {
        const float4 mc = sh.cand[i];
        const uint32_t md = uni(sh.dist[i]), mi = __float_as_uint(mc.w);
        const uint32_t rad = KEYED ? __float_as_uint(r2) : md;
        uint64_t todo = __builtin_amdgcn_ballot_w64(far >= md && box_dist2(cb, mc.x, mc.y, mc.z) < __uint_as_float(rad));
        uint64_t blocked = 0;
        int k = i >> 6;                                 // its own chunk first
        while (true) {
            const float4 oc = sh.cand[64 * k + me.lane];
            const uint32_t od = sh.dist[64 * k + me.lane];
            const bool ahead = od > md || (od == md && __float_as_uint(oc.w) < mi);
            blocked = __builtin_amdgcn_ballot_w64(ahead && __float_as_uint(dist2(oc.x, oc.y, oc.z, mc.x, mc.y, mc.z)) < rad);
            todo &= ~(1ull << k);
            if (blocked != 0 || todo == 0) break;
            k = first_lane(todo);
        }
        int rank = 0;
        if (blocked == 0 && ranked) {
            for (uint64_t m = __builtin_amdgcn_ballot_w64(far >= md); m != 0; m &= m - 1) {
                const int r = 64 * first_lane(m) + me.lane;
                const uint32_t od = sh.dist[r];
                rank += __builtin_popcountll(
                    __builtin_amdgcn_ballot_w64(od > md || (od == md && __float_as_uint(sh.cand[r].w) < mi)));
            }
        }
        if (blocked == 0 && rank < room && me.lane == 0) atomicOr(&sh.acc[(i - lo) >> 5], 1u << ((i - lo) & 31));
    }
    __syncthreads();
    MARK(5);
    if (me.G > 1) {
        uint64_t* const msk = a.ll_mask + (int64_t)(me.grp * 2 + (int)(round & 1u)) * me.G * kWords;
        if (me.tid * 32 < hi - lo) ll_store(msk + (int64_t)me.g * kWords + me.tid, sh.acc[me.tid], round);
        const int words = ((units + me.G - 1) / me.G + 3) >> 2;             // the most a workgroup publishes
        const int g = me.tid >> a.own_shift;
        if (g < me.G) {
            const int from = (int)((uint32_t)(units * g) / (uint32_t)me.G);
            const int to = (int)((uint32_t)(units * (g + 1)) / (uint32_t)me.G);
            for (int q = me.tid & ((1 << a.own_shift) - 1); q < words; q += 1 << a.own_shift) {
                const int u0 = from + 4 * q;
                if (u0 >= to) break;
                uint32_t val = 0;
                if (!ll_wait_close(msk + (int64_t)g * kWords + q, round, val, a.wait_ticks)) sh.fail = 1;
                for (int u = 0; u < 4 && u0 + u < to; ++u)
                    reinterpret_cast<uint8_t*>(sh.took)[u0 + u] = (uint8_t)(val >> (8 * u));
            }
        }
    } else if (me.tid < 2 * kChunks) {
        reinterpret_cast<uint32_t*>(sh.took)[me.tid] = sh.acc[me.tid];
    }
    __syncthreads();
    MARK(6);
    if (uni(sh.fail) != 0) return -1;
    const int cnt = __builtin_popcountll(sh.took[me.lane]);
    return (int)rdlane((uint32_t)wave_incl_sum(cnt, me.lane), 63);
}

// The threshold phase where a sample waits for the one before it, which waits for the one before that (points whose keys follow a
// path or a scan line): such a list yields a sample per chain and round by local decisions, so all its candidates, kSettle at
// most, are settled at once in the order of their keys, by every workgroup for itself.  The waves take 64 of them each: a wave
// picks its first, drops those closer than R_l, picks the next and so on, and the waves behind it drop the ones
// closer than R_l to any of these.  Leaves the samples in sh.took and returns their number, `room` at most.
__device__ __forceinline__ int settle_in_order(LocalShared& sh, const Seat& me, int total, int room, float r2)
{
    const int chunks = (total + 63) >> 6;
    float4* const sorted = sh.cand + kList / 2;
    uint32_t d[kSettle / 64];               // (no two keys are the same)
#pragma unroll
    for (int k = 0; k < kSettle / 64; ++k) d[k] = k < chunks ? sh.dist[64 * k + me.lane] : 0u;
    for (int i = me.w; i < total; i += kNW) {
        const uint32_t md = uni(sh.dist[i]);
        int rank = 0;
#pragma unroll
        for (int k = 0; k < kSettle / 64; ++k) rank += __builtin_popcountll(__builtin_amdgcn_ballot_w64(d[k] > md));
        if (me.lane == 0) {
            const float4 c = sh.cand[i];
            sorted[rank] = make_float4(c.x, c.y, c.z, __int_as_float(i));
        }
    }
    __syncthreads();
    const int mine = 64 * me.w + me.lane;
    const float4 c = sorted[mine < total ? mine : 0];
    uint64_t open = __builtin_amdgcn_ballot_w64(mine < total);
    int got = 0;
    for (int k = 0; k < chunks; ++k) {
        if (me.w == k) {
            uint64_t samples = 0;
            for (int left = room - got; open != 0 && left > 0; --left) {
                const int s = first_lane(open);
                samples |= 1ull << s;
                open &= ~(1ull << s) &
                        ~__builtin_amdgcn_ballot_w64(dist2(rdlane_f(c.x, s), rdlane_f(c.y, s), rdlane_f(c.z, s), c.x, c.y, c.z) < r2);
            }
            if (me.lane == 0) sh.settled[k] = samples;
            if (((samples >> me.lane) & 1ull) != 0) {
                const int i = __float_as_int(c.w);
                atomicOr(reinterpret_cast<unsigned long long*>(&sh.took[i >> 6]), 1ull << (i & 63));
            }
        }
        __syncthreads();
        const uint64_t samples = uni64(sh.settled[k]);
        got += __builtin_popcountll(samples);
        if (me.w > k && open != 0) {
            for (uint64_t m = samples; m != 0; m &= m - 1) {
                const float4 o = sorted[64 * k + first_lane(m)];
                open &= ~__builtin_amdgcn_ballot_w64(dist2(o.x, o.y, o.z, c.x, c.y, c.z) < r2);
            }
        }
    }
    return got;
}

// Folds the round's samples into the wave's distances.
template <int P, bool BQ, bool KEYED>
__device__ __forceinline__ void fold_samples(Held<P>& h, const LocalShared& sh, const Seat& me, const LocalArgs& a, int total)
{
    const int chunks = (total + 63) >> 6, mine = me.lane < chunks ? me.lane : 0;
    const Box cb = box_of_chunk(sh, mine);
    float reach = KEYED ? h.ub : fminf(h.ub, sh.box[6][mine]);
    if constexpr (BQ) reach = fmaxf(reach, a.bq_r2);
    const Box a0 = sh.wbox[me.w][0], a1 = sh.wbox[me.w][1];
    const float bb = fminf(box_box2(a0, cb), box_box2(a1, cb));
    uint64_t todo = __builtin_amdgcn_ballot_w64(me.lane < chunks && sh.took[mine] != 0 && bb < reach);
    bool lowered = false;
    for (; todo != 0; todo &= todo - 1) {
        const int k = first_lane(todo);
        const float4 c = sh.cand[64 * k + me.lane];
        const float v = KEYED ? __builtin_inff() : __uint_as_float(sh.dist[64 * k + me.lane]);
        const float bd = fminf(box_dist2(a0, c.x, c.y, c.z), box_dist2(a1, c.x, c.y, c.z));
        const uint64_t took = uni64(sh.took[k]);
        uint64_t near = __builtin_amdgcn_ballot_w64(bd < fminf(h.ub, v)) & took;
        if constexpr (BQ) {
            uint64_t ball = __builtin_amdgcn_ballot_w64(bd < a.bq_r2) & took;
            near &= ~ball;
            lowered = lowered || ball != 0;
            for (; ball != 0; ball &= ball - 1) {
                const int l = first_lane(ball);
                fold_record<P>(h, me, a, rdlane_f(c.x, l), rdlane_f(c.y, l), rdlane_f(c.z, l), rdlane_f(v, l),
                               rdlane(__float_as_uint(c.w), l));
            }
        }
        lowered = lowered || near != 0;
        for (; near != 0; near &= near - 1) {
            const int l = first_lane(near);
            fold<P>(h, rdlane_f(c.x, l), rdlane_f(c.y, l), rdlane_f(c.z, l), rdlane_f(v, l));
        }
    }
    if (lowered) refresh_bound<P>(h);
}

// A sample found by itself.
template <int P, bool BQ>
__device__ __forceinline__ void fold_one(Held<P>& h, const LocalShared& sh, const Seat& me, const LocalArgs& a, float cx, float cy, float cz, float v,
                                         uint32_t idx)
{
    // (a coordinate that is not finite makes the bound one that is not: recorded by the exact test, or not at all)
    if (BQ && fminf(box_dist2(sh.wbox[me.w][0], cx, cy, cz), box_dist2(sh.wbox[me.w][1], cx, cy, cz)) < a.bq_r2) fold_record<P>(h, me, a, cx, cy, cz, v, idx);
    else fold<P>(h, cx, cy, cz, v);
    refresh_bound<P>(h);
}

// Clears the counts and candidates this workgroup has published; they are gone once the workgroups have met.
__device__ __forceinline__ void clear_lists(const LocalArgs& a, const Seat& me)
{
    for (int par = 0; par < 2; ++par) {
        uint64_t* own = half_list(a, me, par, me.half);
        for (int t = me.tid & (kT / 2 - 1); t < kHalfWords; t += kT / 2) word_store(own + t, 0ull);
        if ((me.tid & (kT / 2 - 1)) == 0) word_store(a.ll_hdr + (int64_t)(me.grp * 2 + par) * (2 * me.G) + me.half, 0ull);
    }
    __threadfence();
    __syncthreads();
}

// The stamps of published candidates start again: all workgroups meet when they are done with the last list, clear
// their words and meet once more.  False if a wait expired.  (The rounds go on without a gap: each of them clears the
// counters in LDS that the next one adds to.)
template <int P>
__device__ __forceinline__ bool renew_stamps(const Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a, uint32_t& it,
                                             uint32_t& seq)
{
    if (me.G == 1) return true;
    for (int k = 0; k < 2; ++k) {
        const Rec r = plain_pick<P>(h, sh, me, a, it, seq);
        if (uni(r.fail) != 0) return false;
        if (k == 0) clear_lists(a, me);
    }
    return true;
}

// Progress of one cloud; every field is uniform over all workgroups of the cloud.
struct Progress {
    int np;                 // samples found
    int rounds;
    float low;              // no sample of the run was found at a distance below
    uint32_t it, seq, round;
};

__device__ __forceinline__ uint64_t found_word(uint32_t prio, uint32_t idx)
{
    return ((uint64_t)(~prio & kTopKey) << 21) | idx;
}

// Notes the round's samples (one workgroup).
__device__ __forceinline__ void note_samples(const LocalShared& sh, const Seat& me, uint64_t* found, int np, int total)
{
    int at = np;
    for (int k = 0; 64 * k < total; ++k) {
        const uint64_t m = uni64(sh.took[k]);
        if (k % kNW == me.w && ((m >> me.lane) & 1ull) != 0)
            found[at + lanes_below(m)] = found_word(sh.dist[64 * k + me.lane], __float_as_uint(sh.cand[64 * k + me.lane].w));
        at += __builtin_popcountll(m);
    }
}

// Exact FPS up to `stop` samples.  Returns the status: 0, 2 if a wait expired.  (Fewer samples at status 0: every point lies
// on a sample, Alg. 1 takes index 0 from there on.)
template <int P, bool BQ>
__device__ __forceinline__ int exact_rounds(Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a, Progress& st,
                                            uint64_t* found, int stop)
{
    float tau = -1.0f;                      // every distance above it is in the next list; < 0: not known
    float step = 0.8f;                      // ratio of a round's levels
    int dry = 0, most_dry = 3;
    while (st.np < stop) {
        if ((st.round & kWipe) == kWipe && !renew_stamps<P>(h, sh, me, a, st.it, st.seq)) return 2;
        if (!(tau > 0.0f)) {
            const Rec r = plain_pick<P>(h, sh, me, a, st.it, st.seq);
            if (uni(r.fail) != 0) return 2;
            const float v = unif(__uint_as_float(r.d));
            ++st.rounds;
            if (v == 0.0f) {
                if (a.dist) {               // a prefix has all its samples
                    if (me.g == 0)
                        for (int t = st.np + me.tid; t < stop; t += kT) found[t] = found_word(0u, 0u);
                    st.np = stop;
                }
                return 0;
            }
            if (me.g == 0 && me.tid == 0) found[st.np] = found_word(r.d, r.idx);
            ++st.np;
            st.low = fminf(st.low, v);
            fold_one<P, BQ>(h, sh, me, a, unif(r.x), unif(r.y), unif(r.z), v, uni(r.idx));
            tau = v < __builtin_inff() ? v : -1.0f;
            dry = 0;
            continue;
        }
        ++st.round;
        ++st.rounds;
        Levels lv;
        lv.r2 = 0.0f;
        lv.d[0] = tau;
#pragma unroll
        for (int j = 1; j < kLevels; ++j) lv.d[j] = lv.d[j - 1] * step;
        int level;
        const int total = make_list<P, false>(h, sh, me, a, st.round, lv, a.aim, level);
        if (total < 0) return 2;
#pragma unroll
        for (int j = 1; j < kLevels; ++j) tau = j == level ? lv.d[j] : tau;
        if (level == kLevels - 1) step = fmaxf(step * step, 0.3f);
        else if (level == 0) step = sqrtf(step);
        else if (level == 1) step = sqrtf(sqrtf(step) * step);
        if (total == 0) {
            if (++dry >= most_dry) {
                tau = -1.0f;
                most_dry = 1;               // (until a list is of use again)
            }
            continue;
        }
        dry = 0;
        most_dry = 3;
        st.low = fminf(st.low, tau);
        const int got = decide<false>(sh, me, a, st.round, total, stop - st.np, 0.0f);
        if (got < 0) return 2;
        fold_samples<P, BQ, false>(h, sh, me, a, total);
        if ((int)(st.round % (uint32_t)me.G) == me.g) note_samples(sh, me, found, st.np, total);
        st.np += got;
        MARK(7);
    }
    return 0;
}

// The first thread of the cloud's first workgroup: where a run of samples begins.
__device__ __forceinline__ void begin_run(const LocalArgs& a, const Seat& me, int& runs, int at, uint32_t low)
{
    if (me.g == 0 && me.tid == 0 && runs < kLocalRuns) {
        a.cloud[me.c].begin[runs] = at;
        a.cloud[me.c].low[runs] = low;
    }
    ++runs;
}

// Threshold sampling (main loop of Alg. 2): the available points, d >= R_l^2, in the order of their keys.  Within a
// level the points with the lowest key of their neighbourhood are taken at once: a point that is not available never
// becomes so, and one that no available point with a lower key lies closer to than R_l stays available until its
// turn.  A round's list holds all available points in front of a window's end; the window grows as there is room.
// With CHAINS, a list that yields less than a sample in 64 candidates is tried in order (settle_in_order), and rounds stay with what
// yields more, looking at the other way again after 8, 16, ... of them.  ms by rounds of 256 candidates settled in order / by local
// decisions alone / now: path of 40000 points, 6000 samples 3.6 / 3.1 / 1.9, with a hundredth of them in the prefix 4.8 / 15.0 / 2.2,
// thresholds given 7.5 / 36.6 / 2.8; 104481 voxels of a room in rows, 5000 samples 2.5 / 3.2 / 2.1; 4 x 120000 points in rings, 16384 samples
// 4.9 / 2.19 / 2.04.  (Below a sample in 16 or 32 candidates: 2.36 and 2.20 in rings; 512 candidates in order: 2.7 for the voxels; 1024: 2.4.
// The scattered scan order has no chains, and its kernels are 3 % slower with this in them.)
// `seg`, the level (from 1), is left at nseg + 1 when the last one is exhausted.
template <int P, bool BQ, bool CHAINS>
__device__ __forceinline__ int threshold_rounds(Held<P>& h, LocalShared& sh, LevelShared& ls, const Seat& me, const LocalArgs& a,
                                                Progress& st, uint64_t* found, int& seg, int& runs)
{
    const int n = a.n;
    int level_end = 0;                      // first position the quota rule puts above the level: ceil(n l / nseg)
    uint32_t end = 0, len = 1;
    bool in_order = false;
    int hold = 0, span = 8, few = 0;        // rounds before the other way is tried again; what local decisions yielded last
    auto enter = [&]() {
        level_end = (int)(((int64_t)n * seg + a.nseg - 1) / a.nseg);
        if (me.tid == 0 && ls.level_start[seg - 1] < 0) ls.level_start[seg - 1] = st.np;
        begin_run(a, me, runs, st.np, ~0u);
        end = 0;
        len = (uint32_t)(a.N / 64 + 1);
        in_order = false;
        hold = 0;
        span = 8;
    };
    while (st.np < n) {
        if (st.np >= level_end) {
            while (st.np >= level_end) {
                ++seg;
                level_end = (int)(((int64_t)n * seg + a.nseg - 1) / a.nseg);
            }
            enter();
        }
        if ((st.round & kWipe) == kWipe && !renew_stamps<P>(h, sh, me, a, st.it, st.seq)) return 2;
        ++st.round;
        ++st.rounds;
        const int room = (level_end < n ? level_end : n) - st.np;
        Levels lv;
        lv.r2 = unif(ls.thr[seg - 1]);
        lv.end[0] = end;
#pragma unroll
        for (int j = 1; j < kLevels; ++j) {
            const uint64_t e = (uint64_t)end + ((uint64_t)len << (j - 1));
            lv.end[j] = e < (uint64_t)a.N ? (uint32_t)e : (uint32_t)a.N;
        }
        if (lv.end[2] == (uint32_t)a.N) lv.end[1] = end + ((uint32_t)a.N - end) / 2;
        int level;
        const int total = make_list<P, true>(h, sh, me, a, st.round, lv, CHAINS && in_order ? kSettle : a.aim, level);
        if (total < 0) return 2;
#pragma unroll
        for (int j = 1; j < kLevels; ++j) end = j == level ? lv.end[j] : end;
        if (level == kLevels - 1) len = len < 0x40000000u ? len * 2u : len;
        else if (level == 0) len = len / 4u + 1u;
        else if (level == 1) len = len / 2u + 1u;
        if (total == 0) {
            if (end < (uint32_t)a.N) continue;
            if (me.tid == 0) ls.level_exhausted[seg - 1] = 1;
            ++seg;
            if (seg > a.nseg) return 0;     // early termination
            enter();
            continue;
        }
        const int got = CHAINS && in_order && total <= kSettle ? settle_in_order(sh, me, total, room, lv.r2)
                                                               : decide<true>(sh, me, a, st.round, total, room, lv.r2);
        if (got < 0) return 2;
        fold_samples<P, BQ, true>(h, sh, me, a, total);
        if ((int)(st.round % (uint32_t)me.G) == me.g) note_samples(sh, me, found, st.np, total);
        st.np += got;
        if constexpr (CHAINS) {
            hold -= hold > 0 ? 1 : 0;
            if (in_order) {
                in_order = hold != 0;
                if (total > kSettle / 4 && got <= few) {        // no better
                    in_order = false;
                    hold = span;
                    span = min(2 * span, 256);
                }
            } else if (hold == 0 && total > 128 && 64 * got < total) {
                // the window starts again in front of the lowest key of the list, with half as many as are settled in order
                in_order = true;
                hold = span;
                span = min(2 * span, 256);
                few = got;
                const int chunk = me.lane < ((total + 63) >> 6) ? me.lane : 0;
                const uint32_t lowest = kTopKey - wave_max_u32(__float_as_uint(sh.box[6][chunk]));
                len = (uint32_t)((uint64_t)(end - lowest) * (kSettle / 2) / (uint32_t)total) + 1u;
                end = lowest;
            }
        }
        MARK(7);
    }
    return 0;
}

// Clouds in sampling order (the gathered samples of an earlier stage), whose samples are 0, 1, 2, ... again: what
// follow_order of sampler.hip does, on points in cell order.  A wave folds the points of the sequence that come near its
// boxes and looks at its largest distance in front of each; between two of them that stays, while the curve falls (which
// is checked), so the last of a stretch decides.  8 x 6000 gathered samples, 1500 of them: 280 -> 104 us.  Returns how many of the first points are the samples in sequence (1: not
// tried; 0: a wait expired); the distances are left anywhere.
__device__ __forceinline__ bool agree_in_order(LocalShared& sh, const Seat& me, const LocalArgs& a, uint32_t& round)
{
    __syncthreads();
    if (me.G == 1) return true;
    ++round;
    uint64_t* const hdr = a.ll_hdr + (int64_t)(me.grp * 2 + (int)(round & 1u)) * (2 * me.G);
    if (me.tid == 0) ll_store(hdr + me.g, (uint32_t)sh.in_order, round);
    __syncthreads();
    if (me.tid < me.G) {
        uint32_t val = 0;
        if (ll_wait_close(hdr + me.tid, round, val, a.wait_ticks)) atomicMin(&sh.in_order, (int)val);
        else sh.fail = 1;
    }
    __syncthreads();
    return uni(sh.fail) == 0;
}
constexpr int64_t kOrderWords = 4 * kHalfWords;             // per workgroup: most points the words hold
template <int P>
__device__ __forceinline__ int follow_order(Held<P>& h, LocalShared& sh, const Seat& me, const LocalArgs& a, uint32_t& round)
{
    const int n = a.n, N = a.N;
    const float* __restrict__ cloud = a.xyz + (int64_t)me.c * N * 3;
    if (n < 16 || n > kOrderWords * me.G || (round & kWipe) > kWipe - 32 || round >= 1u << 18) return 1;
    {
        // every workgroup looks at the same points
        const float x0 = cloud[0], y0 = cloud[1], z0 = cloud[2];
        const float d1 = dist2(x0, y0, z0, cloud[3], cloud[4], cloud[5]);
        const int64_t j = ((int64_t)me.tid * N) / kT;
        const float d = dist2(x0, y0, z0, cloud[3 * j], cloud[3 * j + 1], cloud[3 * j + 2]);
        if (__syncthreads_or(!(d <= d1) || !(d1 > 0.0f) || !(d1 < __builtin_inff()))) return 1;
    }
    if (me.tid == 0) sh.in_order = n;
    // Behind another cloud of the group the workgroups meet first: some may still be reading that one's last list and counts,
    // which the words and the agreement on them write over (a workgroup without a share of the decisions is
    // waited for by nobody).
    if (me.G == 1 || round == a.first_round) ++round;
    else if (!agree_in_order(sh, me, a, round)) return 0;
    const uint32_t stamp = round;
    uint64_t* const words = half_list(a, me, 0, 0);         // (a stamp of 32 bits is no stamp of a candidate's)
    float* const part = reinterpret_cast<float*>(sh.cand);
    const Box a0 = sh.wbox[me.w][0], a1 = sh.wbox[me.w][1];
    refresh_bound<P>(h);                                    // (0 for a wave without points)
    float last_v = __builtin_inff();
    int good = 0;                                           // points up to the last one this wave has folded
    int from = 0, upto = n < 64 ? n : 64;
    __syncthreads();
    while (true) {
        for (int b = (from >> 6) + me.g; 64 * b < upto; b += me.G) {
            const int k = 64 * b + me.lane, kk = k < N ? k : N - 1;
            const float kx = cloud[(int64_t)kk * 3], ky = cloud[(int64_t)kk * 3 + 1], kz = cloud[(int64_t)kk * 3 + 2];
            const int len = (64 / kNW) * (b + 1);
            uint32_t v = 0x7F800000u;
            for (int i0 = me.w * len; i0 < (me.w + 1) * len; i0 += 64 / kNW) {
                const int il = i0 + (me.lane & (64 / kNW - 1)), ij = il < N ? il : N - 1;
                const float px = cloud[(int64_t)ij * 3], py = cloud[(int64_t)ij * 3 + 1], pz = cloud[(int64_t)ij * 3 + 2];
#pragma unroll
                for (int u = 0; u < 64 / kNW; ++u) {
                    const uint32_t t = __float_as_uint(dist2(rdlane_f(px, u), rdlane_f(py, u), rdlane_f(pz, u), kx, ky, kz));
                    v = i0 + u < k && t < v ? t : v;
                }
            }
            part[me.tid] = __uint_as_float(v);
            __syncthreads();
            if (me.w == 0) {
#pragma unroll
                for (int w = 1; w < kNW; ++w) v = min(v, __float_as_uint(part[w * 64 + me.lane]));
                if (k >= from && k < upto) ll_store(words + k, v, stamp);
            }
            __syncthreads();
        }
        int bad = n;
        for (int c = from >> 6; 64 * c < upto && bad == n; ++c) {
            const int k = 64 * c + me.lane;
            const bool has = k >= from && k < upto;
            float kx = 0.0f, ky = 0.0f, kz = 0.0f, v = 0.0f;
            bool late = false;
            if (has) {
                uint32_t val = 0;
                late = !ll_wait_close(words + k, stamp, val, a.wait_ticks);
                v = __uint_as_float(val);
                kx = cloud[(int64_t)k * 3];
                ky = cloud[(int64_t)k * 3 + 1];
                kz = cloud[(int64_t)k * 3 + 2];
            }
            if (__builtin_amdgcn_ballot_w64(late) != 0) {
                if (me.lane == 0) sh.fail = 1;
                break;
            }
            float before = __shfl_up(v, 1);
            if (me.lane == 0 || k == from) before = last_v;
            const uint64_t rises = __builtin_amdgcn_ballot_w64(has && (!(v <= before) || !(v > 0.0f)));
            const int end = upto - 64 * c < 64 ? upto - 64 * c : 64;
            if (rises != 0) {
                bad = 64 * c + first_lane(rises);
                last_v = rdlane_f(before, first_lane(rises));
            } else {
                last_v = rdlane_f(v, end - 1);
            }
            const float bd = fminf(box_dist2(a0, kx, ky, kz), box_dist2(a1, kx, ky, kz));
            for (uint64_t near = __builtin_amdgcn_ballot_w64(has && bd < h.ub); near != 0; near &= near - 1) {
                const int s = first_lane(near);
                if (64 * c + s >= bad) break;
                if (h.ub > rdlane_f(v, s)) {
                    bad = good;
                    break;
                }
                fold<P>(h, rdlane_f(kx, s), rdlane_f(ky, s), rdlane_f(kz, s), __builtin_inff());
                refresh_bound<P>(h);
                good = 64 * c + s + 1;
            }
        }
        // up to where the curve falls the last value decides (a wave without points has no objection)
        if (h.ub > last_v) bad = min(bad, good);
        if (bad < n && me.lane == 0) atomicMin(&sh.in_order, bad);
        if (!agree_in_order(sh, me, a, round)) return 0;
        if (uni(sh.in_order) < upto || upto == n) break;
        from = upto;
        upto = n / 8 < upto ? n : 8 * upto;
        __syncthreads();                                    // (in_order has been read by all)
    }
    const int known = uni(sh.in_order);
    __syncthreads();
    return known > 1 ? known : 1;
}

// Folds the first `known` points, samples in sequence.
template <int P>
__device__ __forceinline__ void fold_order(Held<P>& h, const LocalShared& sh, const Seat& me, const LocalArgs& a, int known)
{
    const float* __restrict__ cloud = a.xyz + (int64_t)me.c * a.N * 3;
    const Box a0 = sh.wbox[me.w][0], a1 = sh.wbox[me.w][1];
    for (int k0 = 0; k0 < known; k0 += 64) {
        const int k = k0 + me.lane, kk = k < known ? k : 0;
        const float kx = cloud[(int64_t)kk * 3], ky = cloud[(int64_t)kk * 3 + 1], kz = cloud[(int64_t)kk * 3 + 2];
        const float bd = fminf(box_dist2(a0, kx, ky, kz), box_dist2(a1, kx, ky, kz));
        for (uint64_t near = __builtin_amdgcn_ballot_w64(k < known && bd < h.ub); near != 0; near &= near - 1) {
            const int s = first_lane(near);
            fold<P>(h, rdlane_f(kx, s), rdlane_f(ky, s), rdlane_f(kz, s), __builtin_inff());
        }
        refresh_bound<P>(h);
    }
}

// MDPS false: exact FPS up to a.stop samples; with a.dist, the prefix of Alg. 2, whose distances are kept there.  MDPS true:
// what follows the prefix -- thresholds, threshold sampling, exact FPS for what remains when the last level is exhausted.
// CHAINS: keys are indices, which may follow each other along the cloud.
template <int P, bool BQ, bool MDPS, bool CHAINS>
__device__ __forceinline__ void run_cloud(const LocalArgs& a, LocalShared& sh, LevelShared* ls, const Seat& me, Progress& st)
{
    const int n = a.n, N = a.N;
    uint64_t* const found = a.found + (int64_t)me.c * n;
    LocalCloud* const cl = a.cloud + me.c;
    const int start = uni(a.start_idx ? a.start_idx[me.c] : 0);
    const long long t0 = wall_clock64();
    long long t1 = t0, t2 = t0, t3 = t0;
    int status = MDPS ? uni(cl->status) : (start < 0 || start >= N ? 1 : 0);        // uniform over the group
    int runs = 0, et_index = n, prefix_ticks = 0;
    st.np = 1;
    st.rounds = 0;
    st.low = __builtin_inff();
    if constexpr (MDPS) {
        if (me.tid < FP_MAX_SEG) {
            ls->level_start[me.tid] = -1;
            ls->level_exhausted[me.tid] = 0;
            ls->thr[me.tid] = 0.0f;
        }
    }
    if (status == 0) {
        Held<P> h;
        load_points<P, BQ, MDPS>(h, sh, me, a);
        if (me.tid == 0) sh.fail = 0;
        if (me.tid < 4) sh.cnt[me.tid >> 1][me.tid & 1] = 0;
        if (me.tid < kSpans * kLevels) reinterpret_cast<int32_t*>(sh.tot)[me.tid] = 0;
        if constexpr (!MDPS) {
            int known = 1;
            // (Not with eight points per thread, clouds of 4097 to 8192 points that one workgroup holds: around this code their rounds
            // spill more, us without / with: 140 x 8000 -> 3000 uniform 1255 / 1403, rooms 1166 / 1298, rings 1338 / 1490.)
            constexpr bool FOLLOWS = !BQ && P < 8;
            if constexpr (FOLLOWS) {
                if (start == 0 && !a.dist) {
                    __syncthreads();                        // (fail)
                    known = follow_order<P>(h, sh, me, a, st.round);
                    if (known == 0) status = 2;
                    if (known > 1 && me.g == 0) {
                        const uint64_t* const words = half_list(a, me, 0, 0);
                        for (int k = 1 + me.tid; k < known; k += kT) found[k] = found_word((uint32_t)ll_load(words + k), (uint32_t)k);
                    }
                    if (known > 1) {
                        st.np = known;
                        st.low = __uint_as_float((uint32_t)ll_load(half_list(a, me, 0, 0) + known - 1));
                        // all have read the values: rounds and the next cloud write over them
                        if ((known < n || me.c + (int)gridDim.x / me.G < a.B) && !agree_in_order(sh, me, a, st.round)) status = 2;
                    }
#pragma unroll
                    for (int p = 0; p < P; ++p) h.d[p] = h.oi[p] != kNoIdx ? __builtin_inff() : 0.0f;
                }
            }
            const float* s = a.xyz + ((int64_t)me.c * N + start) * 3;
            h.ub = __builtin_inff();
            if (FOLLOWS && known > 1) {
                if (known < n) fold_order<P>(h, sh, me, a, known);
            } else {
                fold_one<P, BQ>(h, sh, me, a, s[0], s[1], s[2], __builtin_inff(), (uint32_t)start);
            }
        } else {
            refresh_bound<P>(h);
        }
        __syncthreads();
#ifdef FASTPOINT_PHASE_CLOCKS
        if (me.tid == 0) {
            for (int k = 0; k < 16; ++k) clk[k] = 0;
            clk_at = wall_clock64();
        }
#endif
        if constexpr (!MDPS) {
            begin_run(a, me, runs, 1, 0);
            if (status == 0) status = exact_rounds<P, BQ>(h, sh, me, a, st, found, a.stop);
            if (me.g == 0 && me.tid == 0) cl->low[0] = __float_as_uint(st.low);
        } else {
            st.np = uni(cl->count);
            st.rounds = uni(cl->rounds);
            prefix_ticks = uni(cl->ticks);
            int seg = 0;
            const float* curve = a.curve + (int64_t)me.c * n;
            if (me.tid < 64 && a.m - me.tid >= 1) ls->ring[(a.m - me.tid) & 63] = curve[a.m - me.tid];
            if (me.tid < FP_MAX_SEG) {
                const int b = me.tid < a.nseg ? boundary_index(n, a.nseg, me.tid + 1) : n;
                ls->thr_meas[me.tid] = b <= a.m ? curve[b] : 0.0f;
            }
            if (me.tid < 32) {
                const int64_t ik = ((int64_t)a.m * (me.tid + 1)) / 32;
                ls->mlp_val[me.tid] = curve[ik < 1 ? 1 : ik];
            }
            __syncthreads();
            predict_thresholds(a, *ls, me.tid);
            __syncthreads();
            t1 = wall_clock64();
            status = threshold_rounds<P, BQ, CHAINS>(h, sh, *ls, me, a, st, found, seg, runs);
            t2 = wall_clock64();
            if (status == 0 && st.np < n) {
                et_index = st.np;
                const int tail = runs;
                begin_run(a, me, runs, st.np, 0);
                st.low = __builtin_inff();
                status = exact_rounds<P, BQ>(h, sh, me, a, st, found, n);
                if (me.g == 0 && me.tid == 0) cl->low[tail] = __float_as_uint(st.low);
            }
            t3 = wall_clock64();
        }
        if constexpr (!MDPS)
            if (a.dist) {
                const int base = (me.half * kHW + (me.w & (kHW - 1))) * P * 64;
#pragma unroll
                for (int p = 0; p < P; ++p)
                    if (base + p * 64 + me.lane < N) a.dist[(int64_t)me.c * N + base + p * 64 + me.lane] = h.d[p];
            }
        if constexpr (BQ) {
            if (me.lane == 0) {
                if (!MDPS && a.dist && (me.half * kHW + (me.w & (kHW - 1))) * P * 64 < N)
                    bq_place(a, me, P) = make_uint2(h.bq_next, h.bq_room | (h.bq_dead ? 0x100u : 0u));
                if (h.bq_room != 0)
                    a.bq_fill[(int64_t)me.c * (a.bq_cap / kBqChunk) + h.bq_next / (uint32_t)kBqChunk] =
                        (uint32_t)kBqChunk - h.bq_room;
            }
        }
    }
#ifdef FASTPOINT_PHASE_CLOCKS
    if (me.tid == 0)
        for (int k = 0; k < 16; ++k)
            a.ll_mask[(int64_t)2 * kMaxGroup * kWords + blockIdx.x * 16 + k] = (uint64_t)clk[k];
#endif
    __syncthreads();
    if (me.g == 0 && me.tid == 0) {
        const int ticks = (int)(wall_clock64() - t0);
        cl->status = status;
        cl->count = st.np;
        cl->rounds = st.rounds;
        cl->ticks = ticks;
        cl->runs = runs;
        cl->begin[runs < kLocalRuns ? runs : kLocalRuns] = st.np;
        if (a.info && (MDPS || !a.dist)) {
            fp_mdps_info inf = {};
            if (status != 1) {
                inf.m = MDPS ? a.m : n - 1;
                inf.et_index = et_index;
                for (int l = 0; l < FP_MAX_SEG; ++l) {
                    inf.level_start[l] = MDPS ? ls->level_start[l] : -1;
                    if constexpr (MDPS) {
                        inf.level_exhausted[l] = ls->level_exhausted[l];
                        inf.thr2[l] = ls->thr[l];
                    }
                }
                inf.rounds = st.rounds;
                inf.phase_ticks[0] = MDPS ? prefix_ticks : ticks;
                if constexpr (MDPS) {
                    inf.phase_ticks[1] = (int32_t)(t1 - t0);
                    inf.phase_ticks[2] = (int32_t)(t2 - t1);
                    inf.phase_ticks[3] = (int32_t)(t3 - t2);
                }
            }
            inf.status = status;
            a.info[me.c] = inf;
        }
    }
    __syncthreads();
}

template <int P, bool BQ, bool MDPS, bool CHAINS>
__global__ __launch_bounds__(kT) void local_kernel(LocalArgs a)
{
    __shared__ LocalShared sh;
    __shared__ LevelShared ls[1];
    Seat me;
    me.tid = (int)threadIdx.x;
    me.lane = me.tid & 63;
    me.w = uni(me.tid >> 6);
    me.G = a.G;
    me.grp = (int)blockIdx.x / a.G;
    me.g = (int)blockIdx.x % a.G;
    me.half = me.g + (me.w >= kHW ? me.G : 0);
    const int ngroups = (int)gridDim.x / a.G;
    if constexpr (BQ && !MDPS) {
        // the header of the ball-query cache
        if (blockIdx.x == 0 && threadIdx.x == 0)
            *reinterpret_cast<BqHeader*>(a.bq_base) = bq_layout(a.B, a.N, a.n, a.bq_r2, a.bq_cap, 1);
    }
    Progress st;
    st.it = st.seq = 0;
    st.round = a.first_round;
    for (int c = me.grp; c < a.B; c += ngroups) {
        me.c = c;
        run_cloud<P, BQ, MDPS, CHAINS>(a, sh, ls, me, st);
    }
}

// ---- the samples in the sequence of Alg. 1: ascending keys (inverted distance bits, index).  The inverses of the
// distances are spread over 4096 ranges of equal width (the n-th of evenly spread samples is found at a distance that
// falls with 1 / n on surfaces, with n ** (-2 / 3) in space).  Every workgroup counts all keys by range (65536 keys are 0.5 MB, read
// by 32 workgroups), takes the ranges that begin in its share of the sequence, gathers their keys in LDS and
// places each among those of its range (a few dozen at most in the workloads; where one has more, all of them are sorted).
// A range of more keys than a share has places (equal distances, or a smallest distance so far below the others that
// these are all in the first range) is divided among the workgroups by place: each looks for the first and the last
// key of its share, twelve bits of the key at a time, and sorts those between.  Bound: the passes over the keys, two, or seven.
// fps_exact_pruned of 20000 points, all of them sampled, most of which are in one range: 0.85 ms; 23.9 ms where one workgroup
// compared all of them with each other.
constexpr int kOrderT = 1024;
constexpr int kRanges = 4096;                   // 2^12
constexpr int kShare = kOrderMost / 2;          // places of a workgroup at most
constexpr int kFewKeys = 128;                   // keys of a range up to which each is placed by comparing it with the others

// Puts the first `count` keys in order; `key` has room for the next power of two.
__device__ __forceinline__ void sort_keys(uint64_t* key, int count, int tid)
{
    int size = 64;
    while (size < count) size <<= 1;
    for (int t = count + tid; t < size; t += kOrderT) key[t] = ~0ull;
    for (int k = 2; k <= size; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int t = tid; t < size / 2; t += kOrderT) {
                const int lo = (t & ~(j - 1)) * 2 | (t & (j - 1)), hi = lo | j;
                const uint64_t u = key[lo], v = key[hi];
                if ((u > v) == ((lo & k) == 0)) {
                    key[lo] = v;
                    key[hi] = u;
                }
            }
        }
    __syncthreads();
}

__global__ __launch_bounds__(kOrderT) void order_samples_kernel(const uint64_t* __restrict__ found_all,
                                                                const LocalCloud* __restrict__ clouds,
                                                                const int32_t* __restrict__ start_idx, int N, int n, int Q,
                                                                bool fill, int32_t* __restrict__ out_idx,
                                                                float* __restrict__ out_mdc, int32_t* __restrict__ bq_idx,
                                                                int32_t* __restrict__ inv)
{
    __shared__ uint64_t key[kOrderMost];
    __shared__ int32_t first[kRanges + 1];              // counts, then keys in front of the range
    __shared__ int32_t next[kRanges];
    __shared__ int32_t sums[kOrderT / 64];
    __shared__ int32_t mine[4];
    __shared__ int32_t bin[2][3];                       // of the first and the last key looked for: digit, keys of it, keys in front
    __shared__ int32_t gathered;
    const int b = (int)blockIdx.y, q = (int)blockIdx.x, tid = (int)threadIdx.x, lane = tid & 63;
    const LocalCloud& cl = clouds[b];
    const int np = cl.count, runs = cl.runs;
    // again: a point that is a sample already (index 0, found at distance 0); the record has no row for it
    auto put = [&](int pos, uint32_t dbits, uint32_t i, bool again) {
        out_idx[(int64_t)b * n + pos] = (int32_t)i;
        if (out_mdc) out_mdc[(int64_t)b * n + pos] = __uint_as_float(dbits);
        if (bq_idx) bq_idx[(int64_t)b * n + pos] = again ? -1 : (int32_t)i;
        if (inv && !again) inv[(int64_t)b * N + i] = pos;
    };
    if (cl.status != 0) {
        if (fill)
            for (int t = q * kOrderT + tid; t < n; t += Q * kOrderT) {
                out_idx[(int64_t)b * n + t] = -1;
                if (bq_idx) bq_idx[(int64_t)b * n + t] = -1;               // no centre matches this cloud's record
            }
        return;
    }
    if (fill)
        for (int t = np + q * kOrderT + tid; t < n; t += Q * kOrderT) put(t, 0u, 0u, true);        // every point lies on a sample
    if (q == 0 && tid == 0) put(0, 0x7F800000u, start_idx ? (uint32_t)start_idx[b] : 0u, false);
    if (runs == 0 || np <= cl.begin[0]) return;                            // uniform
    const int all = cl.begin[0], len = np - all;
    const int s0 = all + (int)((int64_t)len * q / Q), s1 = all + (int)((int64_t)len * (q + 1) / Q);
    for (int run = 0; run < runs; ++run) {
        const int r_begin = cl.begin[run], m = cl.begin[run + 1] - r_begin;
        // this workgroup's share of the run's positions
        const int share0 = s0 > r_begin ? s0 - r_begin : 0, share1 = s1 - r_begin < m ? s1 - r_begin : m;
        if (share0 >= share1) continue;                                    // uniform
        const uint64_t* const keys = found_all + (int64_t)b * n + r_begin;
        const uint32_t bound = cl.low[run];
        const bool keyed = bound == ~0u;
        // 1 - f / 2 in place of 1 / (1 + f) inside a power of two: all in whole numbers, and falling with the distance
        const int low = (int)(bound >> 23);                                // exponent of the bound
        const int shift = N <= kRanges ? 0 : 32 - __builtin_clz((uint32_t)(N - 1) >> 12);
        auto range_of = [&](uint64_t k) {
            const uint32_t p = (uint32_t)(k >> 21);
            int r;
            if (keyed) {
                r = (int)(p >> shift);
            } else {
                const uint32_t v = ~p & kTopKey;
                const int o = (int)(v >> 23) - low;
                r = o < 12 ? (int)(((1u << 24) - (v & 0x7FFFFFu)) >> (12 + (o > 0 ? o : 0))) : 0;
            }
            return r < kRanges ? r : kRanges - 1;
        };
        auto emit = [&](int place, uint64_t k) {
            const uint32_t v = ~(uint32_t)(k >> 21) & kTopKey;
            put(r_begin + place, keyed ? 0u : v, (uint32_t)k & 0x1FFFFFu, !keyed && v == 0u);
        };
        __syncthreads();
        for (int t = tid; t < kRanges; t += kOrderT) {
            first[t] = 0;
            next[t] = 0;
        }
        __syncthreads();
        constexpr int U = 16;                                              // loads a thread has under way
        for (int t0 = tid; t0 < m; t0 += kOrderT * U) {
            uint64_t k[U];
#pragma unroll
            for (int u = 0; u < U; ++u) k[u] = t0 + u * kOrderT < m ? keys[t0 + u * kOrderT] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u * kOrderT < m) atomicAdd(&first[range_of(k[u])], 1);
        }
        __syncthreads();
        int c[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            c[u] = first[4 * tid + u];
            sum += c[u];
        }
        const int incl = wave_incl_sum(sum, lane);
        if (lane == 63) sums[tid >> 6] = incl;
        __syncthreads();
        int at = incl - sum;
        for (int w = 0; w < (tid >> 6); ++w) at += sums[w];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = 4 * tid + u;
            first[r] = at;
            // the ranges that hold the first and the last place of the share (one thread finds each)
            if (at <= share0 && share0 < at + c[u]) mine[0] = r;
            if (at < share1 && share1 <= at + c[u]) mine[1] = r;
            at += c[u];
        }
        if (tid == kOrderT - 1) first[kRanges] = at;
        __syncthreads();
        const int ra = uni(mine[0]), rb = uni(mine[1]);
        const int ra0 = uni(first[ra]), ra1 = uni(first[ra + 1]), rb0 = uni(first[rb]), rb1 = uni(first[rb + 1]);
        // the ranges that begin in the share, without the last one if that is longer than a share
        const int r0 = ra0 < share0 ? ra + 1 : ra, r1 = rb1 - rb0 > kShare ? rb : rb + 1;
        if (r0 < r1) {
            const int from = ra0 < share0 ? ra1 : ra0, count = (r1 == rb ? rb0 : rb1) - from;      // at most kOrderMost
            for (int t0 = tid; t0 < m; t0 += kOrderT * U) {
                uint64_t k[U];
#pragma unroll
                for (int u = 0; u < U; ++u) k[u] = t0 + u * kOrderT < m ? keys[t0 + u * kOrderT] : 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = range_of(k[u]);
                    if (t0 + u * kOrderT < m && r >= r0 && r < r1) key[first[r] - from + atomicAdd(&next[r], 1)] = k[u];
                }
            }
            bool many = false;                                             // (a range of keys has 512 of them at most)
            if (!keyed)
                for (int r = r0 + tid; r < r1; r += kOrderT) many = many || first[r + 1] - first[r] > kFewKeys;
            if (__syncthreads_or(many)) {
                sort_keys(key, count, tid);
                for (int t = tid; t < count; t += kOrderT) emit(from + t, key[t]);
            } else {
                for (int t = tid; t < count; t += kOrderT) {
                    const uint64_t k = key[t];
                    const int r = range_of(k), lo = first[r] - from, hi = first[r + 1] - from;
                    int place = first[r];
                    for (int e = lo; e < hi; ++e) place += key[e] < k || (key[e] == k && e < t) ? 1 : 0;
                    emit(place, k);
                }
            }
        }
        // the ranges longer than a share: at most the one it begins in and the one it ends in
        for (int part = 0; part < 2; ++part) {
            const int r = part == 0 ? ra : rb, begin = part == 0 ? ra0 : rb0, end = part == 0 ? ra1 : rb1;
            if (end - begin <= kShare || (part == 1 && ra == rb)) continue;                        // uniform
            const int g0 = begin > share0 ? begin : share0, g1 = end < share1 ? end : share1;
            uint64_t top[2] = {0, 0};                                      // the keys at places g0 and g1 - 1, as far as known
            int place[2] = {g0 - begin, g1 - 1 - begin}, equal[2] = {0, 0};
            for (int bit = 40; bit >= -8; bit -= 12) {
                const int down = bit > 0 ? bit : 0, digits = bit > 0 ? 12 : 12 + bit;
                const bool same = top[0] == top[1];
                __syncthreads();
                for (int t = tid; t < kRanges; t += kOrderT) {
                    first[t] = 0;
                    next[t] = 0;
                }
                __syncthreads();
                for (int t0 = tid; t0 < m; t0 += kOrderT * U) {
                    uint64_t k[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) k[u] = t0 + u * kOrderT < m ? keys[t0 + u * kOrderT] : 0;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool in = t0 + u * kOrderT < m && range_of(k[u]) == r;
                        const uint64_t above = k[u] >> (down + digits);
                        const int digit = (int)(k[u] >> down) & ((1 << digits) - 1);
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (e == 1 && same) break;
                            int32_t* const h = e == 0 ? first : next;
                            // (the lanes with the digit of the first of them together: equal distances share most of them)
                            const uint64_t who = __builtin_amdgcn_ballot_w64(in && above == top[e]);
                            if (who == 0) continue;
                            const int lead = first_lane(who), d0 = (int)rdlane((uint32_t)digit, lead);
                            const uint64_t alike = __builtin_amdgcn_ballot_w64(digit == d0) & who;
                            if (lane == lead) atomicAdd(&h[d0], (int)__builtin_popcountll(alike));
                            else if ((((who & ~alike) >> lane) & 1ull) != 0) atomicAdd(&h[digit], 1);
                        }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int32_t* const h = e == 1 && !same ? next : first;
                    int own = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) own += h[4 * tid + u];
                    const int upto = wave_incl_sum(own, lane);
                    if (lane == 63) sums[tid >> 6] = upto;
                    __syncthreads();
                    int before = upto - own;
                    for (int w = 0; w < (tid >> 6); ++w) before += sums[w];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int n_u = h[4 * tid + u];
                        if (before <= place[e] && place[e] < before + n_u) {
                            bin[e][0] = 4 * tid + u;
                            bin[e][1] = n_u;
                            bin[e][2] = before;
                        }
                        before += n_u;
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    top[e] = (top[e] << digits) | (uint64_t)(uint32_t)uni(bin[e][0]);
                    equal[e] = uni(bin[e][1]);
                    place[e] -= uni(bin[e][2]);
                }
            }
            // places g0 ... : the first key (again, where keys are equal), the keys between, the last key (again)
            const bool one = top[0] == top[1];
            const int inner0 = one ? g1 : g0 + equal[0] - place[0], inner1 = one ? g1 : g1 - 1 - place[1];
            for (int t = g0 + tid; t < inner0; t += kOrderT) emit(t, top[0]);
            for (int t = inner1 + tid; t < g1; t += kOrderT) emit(t, top[1]);
            if (inner0 < inner1) {                                         // uniform
                if (tid == 0) gathered = 0;
                __syncthreads();
                for (int t0 = tid; t0 < m; t0 += kOrderT * U) {
                    uint64_t k[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) k[u] = t0 + u * kOrderT < m ? keys[t0 + u * kOrderT] : 0;
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (t0 + u * kOrderT < m && k[u] > top[0] && k[u] < top[1]) key[atomicAdd(&gathered, 1)] = k[u];
                }
                __syncthreads();
                sort_keys(key, inner1 - inner0, tid);
                for (int t = tid; t < inner1 - inner0; t += kOrderT) emit(inner0 + t, key[t]);
            }
        }
    }
}

}  // namespace

template <int P, bool BQ>
static const void* pick_kernel(bool mdps, bool chains)
{
    if (!mdps) return reinterpret_cast<const void*>(&local_kernel<P, BQ, false, false>);
    return chains ? reinterpret_cast<const void*>(&local_kernel<P, BQ, true, true>)
                  : reinterpret_cast<const void*>(&local_kernel<P, BQ, true, false>);
}

const void* local_kernel_for(int points_per_thread, bool bq, bool mdps, bool chains)
{
    switch (points_per_thread) {
        case 1: return bq ? pick_kernel<1, true>(mdps, chains) : pick_kernel<1, false>(mdps, chains);
        case 2: return bq ? pick_kernel<2, true>(mdps, chains) : pick_kernel<2, false>(mdps, chains);
        case 4: return bq ? pick_kernel<4, true>(mdps, chains) : pick_kernel<4, false>(mdps, chains);
        case 8: return bq ? pick_kernel<8, true>(mdps, chains) : pick_kernel<8, false>(mdps, chains);
        default: return nullptr;
    }
}

hipError_t launch_order_samples(const uint64_t* found, const LocalCloud* cloud, const int32_t* start_idx, int B, int N, int n,
                                int most, bool fill, int32_t* out_idx, float* out_mdc, int32_t* bq_idx, int32_t* inv,
                                hipStream_t stream)
{
    const int Q = most <= kShare ? 1 : (most + kShare - 1) / kShare;
    hipLaunchKernelGGL(order_samples_kernel, dim3((unsigned)Q, (unsigned)B), dim3(kOrderT), 0, stream, found, cloud,
                       start_idx, N, n, Q, fill, out_idx, out_mdc, bq_idx, inv);
    return hipGetLastError();
}

}  // namespace fastpoint
