// Exact Top-k sparsifier with error feedback (Algorithm 1 with Top-k; the
// per-iteration optimum of Lemma 2).
//
// Keys are the 31-bit patterns of |p| (monotone in |p| for non-NaN values),
// ranked larger first and, on equal keys, lower index first.  Selection is a
// radix select (the paper notes radix select costs O(ceil(b/r) d), section 1)
// with a shortcut for error-feedback loops, where the k-th magnitude moves
// little from one iteration to the next.  Five launches, always all enqueued
// (work a call does not need returns at once):
//
//   reset  zero the control block and histograms (114,688 bytes); form the key
//          bracket [lo, hi] around the threshold predicted from the previous
//          calls on this workspace, as wide as their predictions were off
//          (kHalfMin .. kHalfMax keys either side).
//   pass1  p = e + lr*g written into e (12 B/element, streamed with the
//          non-temporal hint); LDS histogram of key bits 30..20; with a
//          bracket, keys above it go straight to the payload and keys inside
//          it to a candidate buffer (staged compaction) and into a histogram
//          of 1024 bins over the bracket.
//   step3  every workgroup first decides the path: the bracket path only
//          when the counts prove the k-th key lies inside the bracket
//          (#(key > hi) <= k <= #(key >= lo), every bracket key collected).
//          Bracket path: zero e at the pairs above the bracket, send the
//          candidates of the bins above the threshold's bin (e zeroed), list
//          those in it.  Radix path: select the top digit from the pass-1
//          histogram, then histogram bits 19..9 of the keys under it (a 4
//          B/element read of p).
//   step4  bracket path: one workgroup ranks the listed keys (key, then lower
//          index) and sends the last pairs.  Radix path: the threshold's bin is
//          now that of its bits 30..9; one read of p sends every larger key (e
//          zeroed) and lists the bin's (sends them too when all are kept).
//          Either path, when the bin holds more keys than the list: a
//          histogram of their low bits instead.
//   emit   radix path: one workgroup ranks the listed keys.  Either path,
//          without a list: the threshold follows from the last histogram and
//          one read of p sends the bin's kept keys, ties ranked in index
//          order: chunks of the vector are taken in order, and each adds up
//          the tie counts that the chunks before it have published.
//
// Selections made by every workgroup read the same histograms, so they agree;
// workgroup 0 records them in the control block.  Histograms are kept in
// kCopies copies (workgroup b adds to copy b mod kCopies: one address takes an
// atomic every 13 ns) and summed when read.
//
// The sweeps run over tiles that start on a 128-byte line of e, whatever e's
// and g's own alignment: the elements before the first line form a partial
// first tile.  g is read with 16-byte accesses at 4-byte alignment.
//
// Workspace (offsets 256-byte aligned): control block (256 B) | histograms |
// chunk states | candidates (int32 index, fp32 value) x ccap | list (the same)
// x lcap.
#include <stddef.h>

#include "device_common.hpp"
#include "launch.hpp"

namespace efs {

namespace {

constexpr int kBins1 = 2048;  // bits 30..20
constexpr int kBins2 = 2048;  // bits 19..9
constexpr int kLowBits = 9;
constexpr int kBins3 = 2048;  // low bits in the threshold's bin: at most 11
constexpr int kBinsB = 1024;  // the bracket
constexpr int kCopies = 4;
// The bracket reaches `half` keys below and above the predicted threshold:
// kHalfSlack times the last prediction's error, and at least three quarters
// of the previous reach, between kHalfMin and kHalfMax (2^20 keys are about
// 6..12 % in magnitude).  Where error feedback has settled the threshold
// moves by 1e-5 of itself a call, and a bracket of a fixed 2^20 keys holds
// more keys than the candidate buffer: every call then took the radix path
// (25.6e6 elements, 0.1 %: 190 us a step with its update, 84 so).
constexpr uint32_t kHalfMin = 1u << 12;
constexpr uint32_t kHalfMax = 1u << 20;
constexpr uint32_t kHalfStart = 1u << 19;
constexpr uint32_t kHalfSlack = 6;
// the extrapolated step is capped at kStepCap keys, or at kStepCapSteady
// when the step before went the same way and at least half as far
constexpr int64_t kStepCap = int64_t(1) << 18;
constexpr int64_t kStepCapSteady = int64_t(1) << 21;
constexpr uint32_t kHintMagic = 0x48494e55u;
constexpr int kStagePairs = 1024;
constexpr uint32_t kNoKey = 0xffffffffu;            // larger than every 31-bit key
// Pass 1 workgroups per CU: three, and from kPass1LongTiles tiles each (2.7e8
// elements) two, walking by XCD as the hard threshold does.  Measured with
// the bracket, three / two / two by XCD: 1.1e8 elements 239 / 254 / - us,
// 4e8 916 / 847 / 856, 1.2e9 2798 / 2647 / 2601 (four: 259 at 1.1e8).
constexpr int kPass1WorkgroupsPerCU = 3;
constexpr int kPass1LongWorkgroupsPerCU = 2;
constexpr uint32_t kPass1LongTiles = 128;
// The launches after pass 1 run 512-thread workgroups, two a CU: one of them
// ranks a list alone, so not 256 threads, and each ends its radix sweep with
// an atomic on one address, so not more of them.  Radix path at 25.6e6, step
// 3 + step 4: 57 us; three a CU 79, four 78, 1024 threads 56, two of those a
// CU 71; at 4e8: 676, 761, 697, 685, 697.
constexpr int kBig = 512;
constexpr int kBigWorkgroupsPerCU = 2;
constexpr int kBigWaves = kBig / kWave;
constexpr int kSpan = kBig * kVecPerThread * 4;     // elements a workgroup reads at a time
constexpr int kChunkSpans = 8;                      // spans per chunk of the ordered sweep
constexpr int kBigStage = 2048;
constexpr int kCandPer = 4;                         // candidates per thread at a time in step 3
// Keys of the threshold's bin ranked by one workgroup, at most (about 1 ns a
// key; the ordered sweep reads e twice, 3 ns for every 1000 elements).
constexpr int64_t kListMin = 16384, kListMax = int64_t(1) << 18;
constexpr int64_t kListPer = 512;                   // one for every kListPer elements between
constexpr uint32_t kRankDirect = 128;               // listed keys ranked against one another
constexpr uint32_t kRankTies = 512;                 // keys equal to the threshold, the same
constexpr int kRankKeep = 4;                        // listed keys a thread holds in registers

// How the kept keys of the threshold's bin are found: none is left to send,
// ranked from the list, or by the ordered sweep.
enum : uint32_t { kDone = 0, kList = 1, kSweep = 2 };

// Fields are written by workgroup 0 of one launch and read by later
// launches only, never by other workgroups of the launch that writes them
// (counters that workgroups add to apart).
struct TopkCtl {
    uint32_t p1, n1;      // radix path: top digit and the rank left under it (step 3)
    uint32_t base, bits;  // the threshold's bin: keys base .. base + 2^bits - 1
    uint32_t need, count, mode;   // keys to keep in it, keys in it, how they are found
    uint32_t pred, half;  // predicted threshold and reach of the bracket
    uint32_t fast;        // 1: bracket path
    uint32_t lo, hi;      // bracket of keys
    uint32_t shift;       // bracket bin of a key: (key - lo) >> shift
    uint32_t bracket_on;  // pass 1 collected the bracket
    uint32_t pad[2];
    unsigned long long emit;   // pass 1: pairs above the bracket (count in the low bits)
    unsigned long long cand;   // pass 1: bracket candidates
    unsigned long long emit2;  // pairs sent after pass 1
    unsigned long long listed; // listed keys
    uint32_t chunk_ticket;     // ordered sweep: chunks taken
    uint32_t last;             // threshold of the previous call (kNoKey if none)
    // Kept across calls (not cleared by reset): the thresholds of the last
    // three calls, each valid when its magic word is set, and the bracket's
    // next reach and its bound.
    uint32_t hint_key, hint_magic;
    uint32_t prev_key, prev_magic;
    uint32_t prev2_key, prev2_magic;
    uint32_t next_half, half_cap, half_magic;
};
static_assert(sizeof(TopkCtl) <= 256, "control block must fit its slot");
constexpr int kCtlClearWords = offsetof(TopkCtl, hint_key) / 4;
static_assert(offsetof(TopkCtl, hint_key) % 4 == 0, "control words are 32-bit");
static_assert(kCtlClearWords <= kBlock, "reset clears the control block with one workgroup");

constexpr size_t kCtlBytes = 256;
constexpr size_t kHistWords = size_t(kCopies) * (kBins1 + kBins2 + kBins3 + kBinsB);
constexpr size_t kHistBytes = sizeof(uint32_t) * kHistWords;
constexpr uint32_t kResetGrid = uint32_t(kHistWords / 4 / kBlock);
static_assert(size_t(kResetGrid) * kBlock * 4 == kHistWords, "one 16-byte store per thread clears the histograms");

size_t round256(size_t b) { return (b + 255) & ~size_t(255); }

struct Workspace {
    TopkCtl *ctl;
    uint32_t *hist1, *hist2, *hist3, *histb;   // kCopies copies each
    unsigned long long *chunk_state;
    int32_t *cand_idx;
    float *cand_val;
    int32_t *list_idx;
    float *list_val;
    uint32_t ccap, lcap;
};

// Candidate buffer size: the bracket around the k-th magnitude of an
// error-feedback vector holds several times k keys (about 8k measured on the
// segmented 25.6e6-element workload), so room for 16k.
int64_t candidate_capacity(int64_t d, int64_t k) {
    int64_t c = 16 * k;
    if (c < 262144) c = 262144;
    if (c > d) c = d;
    if (c < 1) c = 1;
    return c;
}

int64_t list_capacity(int64_t d) {
    const int64_t c = d / kListPer < kListMin ? kListMin : d / kListPer;
    return c < kListMax ? c : kListMax;
}

// At most one partial span more than d holds (see sweep_start).
int64_t max_chunks(int64_t d) { return d / (int64_t(kSpan) * kChunkSpans) + 2; }

Workspace carve(void *ws, int64_t d, int64_t k) {
    char *b = static_cast<char *>(ws);
    Workspace w;
    w.ctl = reinterpret_cast<TopkCtl *>(b);
    w.hist1 = reinterpret_cast<uint32_t *>(b + kCtlBytes);
    w.hist2 = w.hist1 + kCopies * kBins1;
    w.hist3 = w.hist2 + kCopies * kBins2;
    w.histb = w.hist3 + kCopies * kBins3;
    size_t off = kCtlBytes + round256(kHistBytes);
    w.chunk_state = reinterpret_cast<unsigned long long *>(b + off);
    off += round256(sizeof(unsigned long long) * size_t(max_chunks(d)));
    w.ccap = uint32_t(candidate_capacity(d, k));
    w.cand_idx = reinterpret_cast<int32_t *>(b + off);
    off += round256(sizeof(int32_t) * size_t(w.ccap));
    w.cand_val = reinterpret_cast<float *>(b + off);
    off += round256(sizeof(float) * size_t(w.ccap));
    w.lcap = uint32_t(list_capacity(d));
    w.list_idx = reinterpret_cast<int32_t *>(b + off);
    off += round256(sizeof(int32_t) * size_t(w.lcap));
    w.list_val = reinterpret_cast<float *>(b + off);
    return w;
}

// Inclusive sum of v over the lanes of the wave up to this one.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    return v;
}

// Called by every thread of a workgroup of kBig threads.  Bins are ranked
// from the top (kFromTop) or from the bottom; finds the bin where the running
// count first reaches `need` (1 <= need <= sum of bins) and writes {bin, count
// before the bin, count in the bin} to s_out ({0, 0, 0} if no bin
// qualifies).  A bin is the sum of kCount words `stride` apart.
template <int kBins, int kCount, bool kFromTop>
__device__ void select_bin(const uint32_t *hist, uint32_t need, uint32_t *s_scan,
                           uint32_t *s_out) {
    constexpr int kPer = (kBins + kBig - 1) / kBig;
    const int t = threadIdx.x;
    const int lane = t & (kWave - 1);
    const int wave = t / kWave;
    if (t < 3) s_out[t] = 0u;
    uint32_t c[kPer];
    uint32_t tot = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int r = t * kPer + i;
        c[i] = 0u;
        if (r < kBins) {
#pragma unroll
            for (int q = 0; q < kCount; ++q) c[i] += hist[q * kBins + (kFromTop ? kBins - 1 - r : r)];
        }
        tot += c[i];
    }
    const uint32_t incl_w = wave_inclusive_sum(tot);
    if (lane == kWave - 1) s_scan[wave] = incl_w;
    __syncthreads();
    uint32_t off = 0;
#pragma unroll
    for (int q = 0; q < kBigWaves; ++q) off += q < wave ? s_scan[q] : 0u;
    const uint32_t incl = off + incl_w;
    const uint32_t excl = incl - tot;
    if (excl < need && incl >= need) {
        uint32_t run = excl;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (run + c[i] >= need) {
                const int r = t * kPer + i;
                s_out[0] = uint32_t(kFromTop ? kBins - 1 - r : r);
                s_out[1] = run;
                s_out[2] = c[i];
                break;
            }
            run += c[i];
        }
    }
    __syncthreads();
}

// Zeroes the control block (except what is kept across calls) and the
// histograms, and forms the bracket around the threshold predicted from the
// last calls: the last threshold plus the last step in key space, the step
// capped at 2^18 keys, or at 2^21 during a steady drift; the last threshold
// alone when only one is known or the last two steps went opposite ways.
__global__ __launch_bounds__(kBlock) void topk_reset_kernel(Workspace ws) {
    const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    reinterpret_cast<f32x4 *>(ws.hist1)[blockIdx.x * kBlock + threadIdx.x] = z;
    if (blockIdx.x != 0) return;
    uint32_t *w = reinterpret_cast<uint32_t *>(ws.ctl);
    if (int(threadIdx.x) < kCtlClearWords) w[threadIdx.x] = 0u;
    __syncthreads();
    if (threadIdx.x != 0) return;
    TopkCtl *c = ws.ctl;
    c->last = kNoKey;
    if (c->hint_magic != kHintMagic) return;
    // the step since the previous call, capped so that the last threshold
    // stays inside a wide bracket, or further when the step before went the
    // same way and at least half as far: a steady drift of up to ~18 % in
    // |p| per call is then followed
    const int64_t h1 = int64_t(c->hint_key & 0x7fffffffu);
    int64_t pred = h1;
    if (c->prev_magic == kHintMagic) {
        const int64_t h0 = int64_t(c->prev_key & 0x7fffffffu);
        int64_t step = h1 - h0;
        int64_t cap = kStepCap;
        if (c->prev2_magic == kHintMagic) {
            const int64_t before = h0 - int64_t(c->prev2_key & 0x7fffffffu);
            const bool same_way = (step > 0 && before > 0) || (step < 0 && before < 0);
            const int64_t as = step < 0 ? -step : step;
            const int64_t ab = before < 0 ? -before : before;
            if (!same_way) cap = 0;   // steps to and fro: no drift to follow
            else if (2 * ab >= as) cap = kStepCapSteady;
        }
        step = step > cap ? cap : (step < -cap ? -cap : step);
        pred = h1 + step;
        if (pred < 0) pred = 0;
        if (pred > 0x7fffffff) pred = 0x7fffffff;
    }
    uint32_t half = kHalfStart;
    if (c->half_magic == kHintMagic) half = min(max(c->next_half, kHalfMin), kHalfMax);
    const uint32_t p = uint32_t(pred);
    const uint32_t lo = p > half ? p - half : 0u;
    const uint32_t span = 2u * half;
    c->pred = p;
    c->half = half;
    c->last = uint32_t(h1);
    c->lo = lo;
    c->hi = lo + (span - 1u);
    c->shift = 32u - uint32_t(__clz(int(span - 1u))) - 10u;   // span > 2^10
    c->bracket_on = 1u;
}
static_assert(2u * kHalfMin > uint32_t(kBinsB) && 2u * kHalfMax <= uint32_t(kBinsB) << 11,
              "a bracket bin holds 1 to 2^11 keys");

struct Pass1Shared {
    uint32_t h[kBins1];
    uint32_t coarse[kBinsB];
    uint32_t wave[2][kWaves];
    PairStageN<kStagePairs> above;   // keys above the bracket -> payload
    PairStageN<kStagePairs> inside;  // keys in the bracket -> candidates
};

// Appends this tile's `total` selected elements (bits of `mask`, this
// thread's from `pos` on) to a stage, flushing first when they might not fit;
// a tile with more than the stage holds is written straight out behind its
// own atomic.  Called by every thread of the workgroup; contains barriers.
template <int N>
__device__ __forceinline__ void stage_append(PairStageN<N> &st, uint32_t &fill, uint32_t mask,
                                             uint32_t pos, uint32_t total,
                                             const float (&v)[kVecPerThread][4], int64_t tile0,
                                             unsigned long long *word, uint64_t cap,
                                             int32_t *__restrict__ idx, float *__restrict__ val) {
    if (total == 0) return;
    const bool direct = total > uint32_t(N);
    if (direct || fill + total > uint32_t(N)) {
        stage_flush(st, fill, false, word, nullptr, cap, idx, val);
        fill = 0;
    }
    uint64_t o = fill + pos;
    if (direct) {
        if (threadIdx.x == 0) st.base = atomicAdd(word, (unsigned long long)total) & kCountMask;
        __syncthreads();
        o += st.base;
    }
    if (mask != 0u) {
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((mask >> (4 * j + c)) & 1u) {
                    const int32_t i = int32_t(tile0 + int64_t(j * kBlock + int(threadIdx.x)) * 4 + c);
                    if (direct) {
                        if (o < cap) {
                            idx[o] = i;
                            val[o] = v[j][c];
                        }
                    } else {
                        st.idx[o] = i;
                        st.val[o] = v[j][c];
                    }
                    ++o;
                }
            }
        }
    }
    if (direct)
        __syncthreads();
    else
        fill += total;
}

// The stage's pairs to the slots from its base on.
template <int N>
__device__ __forceinline__ void stage_write(const PairStageN<N> &st, uint32_t fill, uint64_t cap,
                                            int32_t *__restrict__ idx, float *__restrict__ val) {
    for (uint32_t j = threadIdx.x; j < fill; j += kBlock) {
        const uint64_t o = st.base + j;
        if (o < cap) {
            idx[o] = st.idx[j];
            val[o] = st.val[j];
        }
    }
}

__global__ __launch_bounds__(kBlock) void topk_pass1_kernel(const float *__restrict__ g,
                                                            float *__restrict__ e, int64_t d,
                                                            float lr, Sweep sw, bool by_xcd,
                                                            uint32_t k,
                                                            int32_t *__restrict__ idx,
                                                            float *__restrict__ val,
                                                            Workspace ws) {
    __shared__ Pass1Shared sh;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const bool bracket = ws.ctl->bracket_on != 0u;
    const uint32_t lo = ws.ctl->lo, hi = ws.ctl->hi, shift = ws.ctl->shift;
    for (int b = tid; b < kBins1; b += kBlock) sh.h[b] = 0u;
    for (int b = tid; b < kBinsB; b += kBlock) sh.coarse[b] = 0u;
    __syncthreads();
    uint32_t fill_above = 0, fill_inside = 0;
    int turn = 0;

    const TileWalk walk = tile_walk(sw.steps, by_xcd);
    for (uint32_t tile = walk.first; tile < walk.end; tile += walk.stride) {
        const int64_t tile0 = sw.first + int64_t(tile) * kTile;
        float p[kVecPerThread][4];
        uint32_t valid;
        if (tile0 >= 0 && tile0 + kTile <= d) {
            const f32x4u *g4 = reinterpret_cast<const f32x4u *>(g + tile0);
            f32x4 *e4 = reinterpret_cast<f32x4 *>(e + tile0);
            f32x4 gv[kVecPerThread], ev[kVecPerThread];
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
                gv[j] = __builtin_nontemporal_load(g4 + j * kBlock + tid);
                ev[j] = __builtin_nontemporal_load(e4 + j * kBlock + tid);
            }
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
                f32x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    o[c] = ef_accumulate(ev[j][c], lr, gv[j][c]);
                    p[j][c] = o[c];
                }
                __builtin_nontemporal_store(o, e4 + j * kBlock + tid);
            }
            valid = 0xffffu;
        } else {
            valid = 0;
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int64_t i = tile0 + int64_t(j * kBlock + tid) * 4 + c;
                    p[j][c] = 0.0f;
                    if (i >= 0 && i < d) {
                        p[j][c] = ef_accumulate(e[i], lr, g[i]);
                        e[i] = p[j][c];
                        valid |= 1u << (4 * j + c);
                    }
                }
            }
        }
        uint32_t m_above = 0, m_inside = 0;
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int b = 4 * j + c;
                const uint32_t key = magnitude_key(p[j][c]);
                if ((valid >> b) & 1u) {
                    atomicAdd(&sh.h[key >> 20], 1u);
                    m_above |= uint32_t(key > hi) << b;
                    m_inside |= uint32_t(key >= lo && key <= hi) << b;
                }
            }
        }
        if (!bracket) continue;
        // both prefix sums behind one barrier; the wave totals alternate
        // between two rows, so the next tile's are written while slower waves
        // still read these
        uint32_t tot_a, tot_i;
        uint32_t pos_a = wave_prefix_small(uint32_t(__popc(m_above)), tot_a);
        uint32_t pos_i = wave_prefix_small(uint32_t(__popc(m_inside)), tot_i);
        uint32_t *row = sh.wave[turn];
        turn ^= 1;
        if (lane == 0) row[wave] = tot_a | (tot_i << 16);
        __syncthreads();
        uint32_t off = 0, tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            off += w < wave ? row[w] : 0u;
            tot += row[w];
        }
        if (tot == 0u) continue;
        pos_a += off & 0xffffu;
        pos_i += off >> 16;
        if (m_inside != 0u) {
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if ((m_inside >> (4 * j + c)) & 1u)
                        atomicAdd(&sh.coarse[(magnitude_key(p[j][c]) - lo) >> shift], 1u);
        }
        stage_append(sh.above, fill_above, m_above, pos_a, tot & 0xffffu, p, tile0,
                     &ws.ctl->emit, k, idx, val);
        stage_append(sh.inside, fill_inside, m_inside, pos_i, tot >> 16, p, tile0,
                     &ws.ctl->cand, ws.ccap, ws.cand_idx, ws.cand_val);
    }
    __syncthreads();
    // the two stages' slots in one round trip, the histograms' adds under it
    if (tid == 0 && fill_above != 0u)
        sh.above.base = atomicAdd(&ws.ctl->emit, (unsigned long long)fill_above) & kCountMask;
    if (tid == kWave && fill_inside != 0u)
        sh.inside.base = atomicAdd(&ws.ctl->cand, (unsigned long long)fill_inside) & kCountMask;
    const uint32_t copy = blockIdx.x % kCopies;
    for (int b = tid; b < kBins1; b += kBlock)
        if (sh.h[b]) atomicAdd(ws.hist1 + copy * kBins1 + b, sh.h[b]);
    if (bracket)
        for (int b = tid; b < kBinsB; b += kBlock)
            if (sh.coarse[b]) atomicAdd(ws.histb + copy * kBinsB + b, sh.coarse[b]);
    __syncthreads();
    stage_write(sh.above, fill_above, k, idx, val);
    stage_write(sh.inside, fill_inside, ws.ccap, ws.cand_idx, ws.cand_val);
}

// The 16 values of a span for this thread of a kBig-thread workgroup (index
// s0 + (j * kBig + tid) * 4 + c).  Elements outside [0, d) read as zero and
// are cleared in `valid`.
__device__ __forceinline__ void load_span(const float *__restrict__ e, int64_t s0, int64_t d,
                                          float (&v)[kVecPerThread][4], uint32_t &valid) {
    const int tid = threadIdx.x;
    if (s0 >= 0 && s0 + kSpan <= d) {
        const f32x4 *s4 = reinterpret_cast<const f32x4 *>(e + s0);
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
            const f32x4 x = s4[j * kBig + tid];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[j][c] = x[c];
        }
        valid = 0xffffu;
    } else {
        valid = 0;
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t i = s0 + int64_t(j * kBig + tid) * 4 + c;
                v[j][c] = 0.0f;
                if (i >= 0 && i < d) {
                    v[j][c] = e[i];
                    valid |= 1u << (4 * j + c);
                }
            }
        }
    }
}

__device__ __forceinline__ int64_t span_elem(int64_t s0, int j, int c) {
    return s0 + int64_t(j * kBig + int(threadIdx.x)) * 4 + c;
}

// Exclusive prefixes over a kBig-thread workgroup of two per-thread counts
// (< 32, totals < 2^16), and the totals, the second of each in the upper half
// of its word.  One barrier; `rows` is two rows of kBigWaves words used in turn.
struct BigScan {
    uint32_t rows[2][kBigWaves];
};

__device__ __forceinline__ uint32_t big_prefix2(uint32_t c0, uint32_t c1, BigScan &s, int &turn,
                                                uint32_t &total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    uint32_t pre = 0u, wtot = 0u;
    if (__ballot((c0 | c1) != 0u) != 0ull) {
        uint32_t w0, w1;
        pre = wave_prefix_small(c0, w0);
        pre |= wave_prefix_small(c1, w1) << 16;
        wtot = w0 | (w1 << 16);
    }
    uint32_t *row = s.rows[turn];
    turn ^= 1;
    if (lane == 0) row[wave] = wtot;
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < kBigWaves; ++w) {
        pre += w < wave ? row[w] : 0u;
        tot += row[w];
    }
    total = tot;
    return pre;
}

__device__ __forceinline__ uint32_t big_prefix(uint32_t c, BigScan &s, int &turn,
                                               uint32_t &total) {
    return big_prefix2(c, 0u, s, turn, total);
}

// Pairs staged in LDS by a kBig-thread workgroup, flushed behind one atomic
// on `word` (only the count in it is used).
struct BigStage {
    int32_t idx[kBigStage];
    float val[kBigStage];
    unsigned long long base;
};

__device__ __forceinline__ void big_flush(BigStage &st, uint32_t &fill, unsigned long long *word,
                                          uint64_t cap, int32_t *__restrict__ idx,
                                          float *__restrict__ val) {
    __syncthreads();
    if (fill == 0u) return;
    if (threadIdx.x == 0) st.base = atomicAdd(word, (unsigned long long)fill);
    __syncthreads();
    const uint64_t base = st.base;
    for (uint32_t j = threadIdx.x; j < fill; j += kBig) {
        if (base + j < cap) {
            idx[base + j] = st.idx[j];
            val[base + j] = st.val[j];
        }
    }
    fill = 0u;
    __syncthreads();
}

// Appends the span's elements selected by `mask` (`total` of them, this
// thread's from `pos` on) to the stage (flushing it first when they might not
// fit).  More than it holds go out behind one atomic, staged one vector slot of
// the workgroup (kBigStage elements) at a time: written by each thread at its
// own `pos`, 16 elements apart from its neighbour's, they took a first call that
// keeps all of 1.1e8 elements 1569 us, 756 so.
static_assert(kBig * 4 <= kBigStage, "a vector slot of the workgroup fits the stage");

__device__ __forceinline__ void big_append(BigStage &st, uint32_t &fill, uint32_t mask,
                                           uint32_t pos, uint32_t total,
                                           const float (&v)[kVecPerThread][4], int64_t s0,
                                           unsigned long long *word, uint64_t cap,
                                           int32_t *__restrict__ idx, float *__restrict__ val,
                                           BigScan &scan, int &turn) {
    if (total == 0u) return;
    const bool direct = total > uint32_t(kBigStage);
    if (direct || fill + total > uint32_t(kBigStage)) big_flush(st, fill, word, cap, idx, val);
    if (direct) {
        if (threadIdx.x == 0) st.base = atomicAdd(word, (unsigned long long)total);
        uint32_t sent = 0u;
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
            const uint32_t mj = (mask >> (4 * j)) & 0xfu;
            uint32_t tj;
            uint32_t o = big_prefix(uint32_t(__popc(mj)), scan, turn, tj);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((mj >> c) & 1u) {
                    st.idx[o] = int32_t(span_elem(s0, j, c));
                    st.val[o] = v[j][c];
                    ++o;
                }
            }
            __syncthreads();
            const uint64_t base = st.base + sent;
            for (uint32_t q = threadIdx.x; q < tj; q += kBig) {
                if (base + q < cap) {
                    idx[base + q] = st.idx[q];
                    val[base + q] = st.val[q];
                }
            }
            sent += tj;   // the next slot is staged behind its prefix's barrier
        }
        __syncthreads();
        return;
    }
    uint32_t o = fill + pos;
#pragma unroll
    for (int j = 0; j < kVecPerThread; ++j) {
        if (((mask >> (4 * j)) & 0xfu) == 0u) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if ((mask >> (4 * j + c)) & 1u) {
                st.idx[o] = int32_t(span_elem(s0, j, c));
                st.val[o] = v[j][c];
                ++o;
            }
        }
    }
    fill += total;
}

__device__ __forceinline__ void clear_span(float *__restrict__ e, int64_t s0, uint32_t mask) {
#pragma unroll
    for (int j = 0; j < kVecPerThread; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if ((mask >> (4 * j + c)) & 1u) e[span_elem(s0, j, c)] = 0.0f;
}

// The threshold T of this call, kept with the two before it for the next
// call's prediction, and the next bracket's reach: kHalfSlack times this
// prediction's error, at least three quarters of this call's reach, within
// the bound.  A bracket that held more keys than the candidate buffer halves
// the bound; one that left three quarters of it free doubles it again.
// Workgroup 0, one thread.
__device__ __forceinline__ void keep_threshold(TopkCtl *c, uint32_t T, uint32_t ccap) {
    uint32_t half = kHalfStart, cap = kHalfMax;
    if (c->bracket_on != 0u) {
        if (c->half_magic == kHintMagic) cap = min(max(c->half_cap, kHalfMin), kHalfMax);
        const uint64_t inside = c->cand & kCountMask;
        if (inside > ccap) cap = max(c->half / 2u, kHalfMin);
        else if (inside * 4u < ccap) cap = min(cap * 2u, kHalfMax);
        const uint32_t err = T > c->pred ? T - c->pred : c->pred - T;
        const uint64_t want = uint64_t(err) * kHalfSlack;
        half = uint32_t(want < kHalfMax ? want : kHalfMax);
        half = max(half, c->half - c->half / 4u);
    }
    c->next_half = min(max(half, kHalfMin), cap);
    c->half_cap = cap;
    c->half_magic = kHintMagic;
    c->prev2_key = c->prev_key;
    c->prev2_magic = c->last != kNoKey ? c->prev_magic : 0u;
    c->prev_key = c->last;
    c->prev_magic = c->last != kNoKey ? kHintMagic : 0u;
    c->hint_key = T;
    c->hint_magic = kHintMagic;
}

struct SelectShared {
    uint32_t scan[kBigWaves];
    uint32_t sel[4];
};

struct RankShared {
    uint32_t hist[2048];
    uint2 item[kRankTies];   // (key, or the equal keys' bits of p; index)
    uint32_t T, cursor, ntie;
};

// One kBig-thread workgroup: of the n listed keys (n >= need >= 1; all within
// [base, base + 2^11)), the `need` first (larger key, then lower index) go to
// payload slots out0 .. out0 + need - 1 with e cleared at them.  Returns the
// threshold, the last of them.  Few keys are ranked against one another; more
// by a histogram of the key, and then the keys equal to the threshold, when
// only some of them are kept, against one another or, when they are many, by
// a radix select on the index (bits 30..20, 19..10, 9..0).  The first
// kRankKeep * kBig keys stay in registers; the others are read again for each
// pass.
template <typename F>
__device__ __forceinline__ void for_listed(const Workspace &ws, uint32_t n,
                                           const uint2 (&mine)[kRankKeep], F f) {
#pragma unroll
    for (int u = 0; u < kRankKeep; ++u)
        if (uint32_t(u) * kBig + threadIdx.x < n) f(mine[u].x, mine[u].y);
    for (uint32_t j = kRankKeep * kBig + threadIdx.x; j < n; j += kBig)
        f(__float_as_uint(ws.list_val[j]), uint32_t(ws.list_idx[j]));
}

__device__ uint32_t rank_list(const Workspace &ws, uint32_t n, uint32_t need, uint32_t base,
                              uint32_t out0, float *__restrict__ e, int32_t *__restrict__ idx,
                              float *__restrict__ val, SelectShared &ss, RankShared &rs) {
    const uint32_t tid = threadIdx.x;
    uint2 mine[kRankKeep];   // (bits of p, index)
#pragma unroll
    for (int u = 0; u < kRankKeep; ++u) {
        const uint32_t j = uint32_t(u) * kBig + tid;
        mine[u] = make_uint2(0u, 0u);
        if (j < n) mine[u] = make_uint2(__float_as_uint(ws.list_val[j]), uint32_t(ws.list_idx[j]));
    }
    auto send = [&](uint32_t slot, uint32_t bits, uint32_t i) {
        if (slot >= need) return;
        idx[out0 + slot] = int32_t(i);
        val[out0 + slot] = __uint_as_float(bits);
        e[i] = 0.0f;
    };
    if (n <= kRankDirect) {
        const uint32_t key = mine[0].x & 0x7fffffffu, i = mine[0].y;
        if (tid < n) rs.item[tid] = make_uint2(key, i);
        __syncthreads();
        if (tid < n) {
            uint32_t rank = 0u;
#pragma unroll 8
            for (uint32_t j = 0; j < n; ++j) {
                const uint2 o = rs.item[j];
                rank += (o.x > key || (o.x == key && o.y < i)) ? 1u : 0u;
            }
            send(rank, mine[0].x, i);
            if (rank == need - 1u) rs.T = key;
        }
        __syncthreads();
        return rs.T;
    }
    for (uint32_t b = tid; b < 2048u; b += kBig) rs.hist[b] = 0u;
    __syncthreads();
    for_listed(ws, n, mine, [&](uint32_t bits, uint32_t) {
        atomicAdd(&rs.hist[((bits & 0x7fffffffu) - base) & 2047u], 1u);
    });
    __syncthreads();
    select_bin<2048, 1, true>(rs.hist, need, ss.scan, ss.sel);
    const uint32_t T = base + ss.sel[0];
    const uint32_t above = ss.sel[1];
    const uint32_t m = need - above;
    const uint32_t ties = ss.sel[2];
    if (tid == 0) {
        rs.cursor = 0u;
        rs.ntie = 0u;
    }
    __syncthreads();
    if (m < ties && ties <= kRankTies) {
        for_listed(ws, n, mine, [&](uint32_t bits, uint32_t i) {
            const uint32_t key = bits & 0x7fffffffu;
            if (key > T) send(atomicAdd(&rs.cursor, 1u), bits, i);
            else if (key == T) rs.item[atomicAdd(&rs.ntie, 1u)] = make_uint2(bits, i);
        });
        __syncthreads();
        if (tid < ties) {
            const uint2 it = rs.item[tid];
            uint32_t rank = 0u;
#pragma unroll 8
            for (uint32_t j = 0; j < ties; ++j) rank += rs.item[j].y < it.y ? 1u : 0u;
            if (rank < m) send(above + rank, it.x, it.y);
        }
        return T;
    }
    uint32_t imax = 0xffffffffu;
    if (m < ties) {
        uint32_t prefix = 0, rem = m;
#pragma unroll 1
        for (int level = 0; level < 3; ++level) {
            const int shift = 20 - 10 * level;
            for (uint32_t b = tid; b < 2048u; b += kBig) rs.hist[b] = 0u;
            __syncthreads();
            for_listed(ws, n, mine, [&](uint32_t bits, uint32_t i) {
                if ((bits & 0x7fffffffu) != T) return;
                if (level > 0 && (i >> (shift + 10)) != prefix) return;
                atomicAdd(&rs.hist[(i >> shift) & (level == 0 ? 2047u : 1023u)], 1u);
            });
            __syncthreads();
            select_bin<2048, 1, false>(rs.hist, rem, ss.scan, ss.sel);
            prefix = (prefix << (level == 0 ? 11 : 10)) | ss.sel[0];
            rem -= ss.sel[1];
            __syncthreads();
        }
        imax = prefix;
    }
    for_listed(ws, n, mine, [&](uint32_t bits, uint32_t i) {
        const uint32_t key = bits & 0x7fffffffu;
        if (key > T || (key == T && i <= imax)) send(atomicAdd(&rs.cursor, 1u), bits, i);
    });
    return T;
}

// Step 3: path decision, then the bracket path's selection and emission or
// the radix path's second digit histogram.
__global__ __launch_bounds__(kBig) void topk_step3_kernel(float *__restrict__ e, int64_t d,
                                                          Sweep sw, uint32_t k,
                                                          int32_t *__restrict__ idx,
                                                          float *__restrict__ val,
                                                          Workspace ws) {
    __shared__ SelectShared ss;
    __shared__ uint32_t h[kBins2];
    __shared__ BigScan scan;
    __shared__ unsigned long long s_base[2][2];
    TopkCtl *c = ws.ctl;
    const int tid = threadIdx.x;
    const bool lead = blockIdx.x == 0 && tid == 0;
    const uint64_t above = c->emit & kCountMask;
    const uint64_t inside = c->cand & kCountMask;
    bool fast = c->bracket_on != 0u && above <= k && above + inside >= k && inside <= ws.ccap;
    const uint32_t need = fast ? k - uint32_t(above) : 0u;
    const uint32_t lo = c->lo, shift = c->shift;
    uint32_t da = 0u, needa = 0u, ca = 0u;
    if (need > 0u) {
        select_bin<kBinsB, kCopies, true>(ws.histb, need, ss.scan, ss.sel);
        da = ss.sel[0];
        needa = need - ss.sel[1];
        ca = ss.sel[2];
        __syncthreads();  // ss.sel is rewritten below
        // the ordered sweep finds the bin's keys in e, where the coordinates
        // cleared here would read as keys of the bin of zero: the radix path
        // clears those last
        fast = ca <= ws.lcap || lo + (da << shift) != 0u;
    }
    const uint32_t mode = need == 0u ? kDone : ca <= ws.lcap ? kList : kSweep;
    if (!fast) {
        // the pairs pass 1 sent are ignored: the radix path writes the whole
        // payload from slot 0 in the launches that follow
        select_bin<kBins1, kCopies, true>(ws.hist1, k, ss.scan, ss.sel);
        const uint32_t prefix = ss.sel[0];
        if (lead) {
            c->fast = 0u;
            c->p1 = prefix;
            c->n1 = k - ss.sel[1];
        }
        for (int b = tid; b < kBins2; b += kBig) h[b] = 0u;
        __syncthreads();
        for (uint32_t s = blockIdx.x; s < sw.steps; s += gridDim.x) {
            float v[kVecPerThread][4];
            uint32_t valid;
            load_span(e, sw.first + int64_t(s) * kSpan, d, v, valid);
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t key = magnitude_key(v[j][q]);
                    if (((valid >> (4 * j + q)) & 1u) && (key >> 20) == prefix)
                        atomicAdd(&h[(key >> kLowBits) & (kBins2 - 1)], 1u);
                }
            }
        }
        __syncthreads();
        uint32_t *out = ws.hist2 + (blockIdx.x % kCopies) * kBins2;
        for (int b = tid; b < kBins2; b += kBig)
            if (h[b]) atomicAdd(out + b, h[b]);
        return;
    }

    if (lead) {
        c->fast = 1u;
        c->base = lo + (da << shift);
        c->bits = shift;
        c->need = needa;
        c->count = ca;
        c->mode = mode;
    }
    // pairs pass 1 sent: zero their residuals (above <= k, so all were written)
    for (uint32_t j = blockIdx.x * kBig + tid; j < uint32_t(above); j += gridDim.x * kBig)
        e[idx[j]] = 0.0f;
    if (need == 0u) return;   // pass 1 sent exactly k pairs
    // candidates, kCandPer a thread at a time: one block-wide prefix and one
    // atomic each for the kept and the listed ones of a round
    const uint32_t n = uint32_t(inside);
    const uint32_t chunk = kCandPer * kBig;
    int turn = 0, round = 0;
    for (uint32_t base = blockIdx.x * chunk; base < n; base += gridDim.x * chunk, round ^= 1) {
        int32_t ci[kCandPer];
        float cv[kCandPer];
        uint32_t keep = 0, list = 0;
#pragma unroll
        for (int u = 0; u < kCandPer; ++u) {
            const uint32_t j = base + uint32_t(u * kBig + tid);
            ci[u] = 0;
            cv[u] = 0.0f;
            if (j < n) {
                ci[u] = ws.cand_idx[j];
                cv[u] = ws.cand_val[j];
                const uint32_t bin = (magnitude_key(cv[u]) - lo) >> shift;
                keep |= uint32_t(bin > da) << u;
                list |= uint32_t(bin == da && mode == kList) << u;
            }
        }
        uint32_t nk, nl;
        uint32_t both;
        const uint32_t pos = big_prefix2(uint32_t(__popc(keep)), uint32_t(__popc(list)), scan, turn, both);
        nk = both & 0xffffu;
        nl = both >> 16;
        if (nk == 0u && nl == 0u) continue;
        if (tid == 0 && nk != 0u) s_base[round][0] = atomicAdd(&c->emit2, (unsigned long long)nk);
        if (tid == kWave && nl != 0u) s_base[round][1] = atomicAdd(&c->listed, (unsigned long long)nl);
        __syncthreads();
        uint64_t ok = above + (nk != 0u ? s_base[round][0] : 0ull) + (pos & 0xffffu);
        uint64_t ol = (nl != 0u ? s_base[round][1] : 0ull) + (pos >> 16);
#pragma unroll
        for (int u = 0; u < kCandPer; ++u) {
            if ((keep >> u) & 1u) {
                if (ok < k) {
                    idx[ok] = ci[u];
                    val[ok] = cv[u];
                }
                e[ci[u]] = 0.0f;
                ++ok;
            }
            if ((list >> u) & 1u) {
                if (ol < ws.lcap) {
                    ws.list_idx[ol] = ci[u];
                    ws.list_val[ol] = cv[u];
                }
                ++ol;
            }
        }
    }
}

__device__ __forceinline__ uint32_t chunks_of(const Sweep &sw) {
    return (sw.steps + kChunkSpans - 1) / kChunkSpans;
}

// Adds a workgroup's histogram of low bits to the global one.
__device__ __forceinline__ void flush_low(const uint32_t *h, uint32_t *hist3) {
    uint32_t *out = hist3 + (blockIdx.x % kCopies) * kBins3;
    for (int b = threadIdx.x; b < kBins3; b += kBig)
        if (h[b]) atomicAdd(out + b, h[b]);
}

// Step 4: the bracket path's last pairs, or the radix path's sweep of p once
// bits 30..9 of the threshold are known.
__global__ __launch_bounds__(kBig) void topk_step4_kernel(float *__restrict__ e, int64_t d,
                                                          Sweep sw, uint32_t k,
                                                          int32_t *__restrict__ idx,
                                                          float *__restrict__ val,
                                                          Workspace ws) {
    __shared__ union {
        RankShared rank;
        struct {
            BigStage keep, list;
        } s;
    } sh;
    __shared__ uint32_t h[kBins3];
    __shared__ SelectShared ss;
    __shared__ BigScan scan;
    TopkCtl *c = ws.ctl;
    const int tid = threadIdx.x;
    const bool lead = blockIdx.x == 0 && tid == 0;
    for (int b = tid; b < kBins3; b += kBig) h[b] = 0u;
    if (c->fast != 0u) {
        const uint32_t mode = c->mode, base = c->base;
        if (mode == kDone) return;
        if (mode == kList) {
            if (blockIdx.x != 0) return;
            const uint32_t T = rank_list(ws, c->count, c->need, base, k - c->need, e, idx, val, ss,
                                         sh.rank);
            if (lead) keep_threshold(c, T, ws.ccap);
            return;
        }
        __syncthreads();
        const uint32_t n = uint32_t(c->cand & kCountMask), bits = c->bits;
        for (uint32_t j = blockIdx.x * kBig + tid; j < n; j += gridDim.x * kBig) {
            const uint32_t sub = magnitude_key(ws.cand_val[j]) - base;
            if ((sub >> bits) == 0u) atomicAdd(&h[sub], 1u);
        }
        for (uint32_t q = blockIdx.x * kBig + tid; q < chunks_of(sw); q += gridDim.x * kBig)
            ws.chunk_state[q] = 0ull;
        __syncthreads();
        flush_low(h, ws.hist3);
        return;
    }
    const uint32_t n1 = c->n1;
    select_bin<kBins2, kCopies, true>(ws.hist2, n1, ss.scan, ss.sel);
    const uint32_t p22 = (c->p1 << 11) | ss.sel[0];
    const uint32_t need2 = n1 - ss.sel[1];
    const uint32_t c2 = ss.sel[2];
    const uint32_t mode = need2 == c2 ? kDone : c2 <= ws.lcap ? kList : kSweep;
    if (lead) {
        c->base = p22 << kLowBits;
        c->bits = kLowBits;
        c->need = need2;
        c->count = c2;
        c->mode = mode;
        // the whole bin is kept: its lowest key serves as the threshold
        if (mode == kDone) keep_threshold(c, p22 << kLowBits, ws.ccap);
    }
    __syncthreads();
    // Without a list, the emission finds the bin's keys by reading e again,
    // where a cleared coordinate would read as one of them if p22 is the bin
    // of zero: it then clears the sent coordinates itself.
    const bool clear_now = mode != kSweep || p22 != 0u;
    uint32_t fill_keep = 0, fill_list = 0;
    int turn = 0;
    for (uint32_t s = blockIdx.x; s < sw.steps; s += gridDim.x) {
        const int64_t s0 = sw.first + int64_t(s) * kSpan;
        float v[kVecPerThread][4];
        uint32_t valid;
        load_span(e, s0, d, v, valid);
        uint32_t keep = 0, bin = 0;
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = 4 * j + q;
                const uint32_t key = magnitude_key(v[j][q]);
                const bool ok = (valid >> b) & 1u;
                const uint32_t up = key >> kLowBits;
                keep |= uint32_t(ok && (up > p22 || (up == p22 && mode == kDone))) << b;
                if (ok && up == p22 && mode != kDone) {
                    bin |= 1u << b;
                    if (mode == kSweep) atomicAdd(&h[key & ((1u << kLowBits) - 1u)], 1u);
                }
            }
        }
        if (mode != kList) bin = 0u;
        uint32_t total;
        const uint32_t pos =
            big_prefix2(uint32_t(__popc(keep)), uint32_t(__popc(bin)), scan, turn, total);
        big_append(sh.s.keep, fill_keep, keep, pos & 0xffffu, total & 0xffffu, v, s0, &c->emit2,
                   k, idx, val, scan, turn);
        if (clear_now) clear_span(e, s0, keep);
        big_append(sh.s.list, fill_list, bin, pos >> 16, total >> 16, v, s0, &c->listed, ws.lcap,
                   ws.list_idx, ws.list_val, scan, turn);
        if (mode == kSweep && tid == 0 && s % kChunkSpans == 0)
            ws.chunk_state[s / kChunkSpans] = 0ull;
    }
    big_flush(sh.s.keep, fill_keep, &c->emit2, k, idx, val);
    if (mode == kList)
        big_flush(sh.s.list, fill_list, &c->listed, ws.lcap, ws.list_idx, ws.list_val);
    if (mode == kSweep) {
        __syncthreads();
        flush_low(h, ws.hist3);
    }
}

constexpr unsigned long long kChunkSum = 1ull << 62;     // the chunk's own ties
constexpr unsigned long long kChunkPrefix = 2ull << 62;  // the ties up to and with the chunk
constexpr unsigned long long kChunkCount = kChunkSum - 1;

// Ties in the chunks before chunk q, whose own count is `mine`: publishes
// the chunk's count, then adds up the counts before it back to the last chunk
// whose prefix is known.  Chunks are taken in order and each publishes its
// count before it waits, so every chunk waited for is being worked on and
// every wait ends.  One thread.
__device__ uint32_t ties_before_chunk(unsigned long long *state, uint32_t q, uint32_t mine) {
    if (q == 0u) {
        __hip_atomic_store(&state[0], kChunkPrefix | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return 0u;
    }
    __hip_atomic_store(&state[q], kChunkSum | mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t before = 0u;
    for (uint32_t p = q; p-- > 0u;) {
        unsigned long long v;
        while ((v = __hip_atomic_load(&state[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0ull)
            __builtin_amdgcn_s_sleep(2);
        before += uint32_t(v & kChunkCount);
        if (v & kChunkPrefix) break;
    }
    __hip_atomic_store(&state[q], kChunkPrefix | (before + mine), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    return before;
}

// The last pairs.  Radix path with a list: one workgroup ranks it.  No list
// (most of its keys are then equal): the threshold from the last histogram,
// then a sweep that sends the bin's keys above it and the ties of index rank
// < m.
__global__ __launch_bounds__(kBig) void topk_emit_kernel(float *__restrict__ e, int64_t d,
                                                         Sweep sw, uint32_t k,
                                                         int32_t *__restrict__ idx,
                                                         float *__restrict__ val,
                                                         Workspace ws) {
    __shared__ union {
        RankShared rank;
        BigStage keep;
    } sh;
    __shared__ SelectShared ss;
    __shared__ BigScan scan;
    __shared__ uint32_t s_chunk, s_before;
    TopkCtl *c = ws.ctl;
    const int tid = threadIdx.x;
    const bool lead = blockIdx.x == 0 && tid == 0;
    const uint32_t mode = c->mode, base = c->base, bits = c->bits, need = c->need;
    if (mode == kDone || (c->fast != 0u && mode == kList)) return;
    if (mode == kList) {
        if (blockIdx.x != 0) return;
        const uint32_t T = rank_list(ws, c->count, need, base, k - need, e, idx, val, ss, sh.rank);
        if (lead) keep_threshold(c, T, ws.ccap);
        return;
    }
    select_bin<kBins3, kCopies, true>(ws.hist3, need, ss.scan, ss.sel);
    const uint32_t T = base + ss.sel[0];
    const uint32_t m = need - ss.sel[1];
    if (lead) keep_threshold(c, T, ws.ccap);
    // bracket path: after the pairs above the bracket; radix path: from slot 0
    const uint64_t sent = c->fast != 0u ? c->emit & kCountMask : 0ull;
    idx += sent;
    val += sent;
    const uint64_t cap = k - sent;
    const bool clear_above = base == 0u;   // step 4 left the sent coordinates
    const uint32_t nchunks = chunks_of(sw);
    uint32_t fill = 0;
    int turn = 0;
    for (;;) {
        __syncthreads();
        if (tid == 0) s_chunk = atomicAdd(&c->chunk_ticket, 1u);
        __syncthreads();
        const uint32_t q = s_chunk;
        if (q >= nchunks) break;
        const uint32_t s1 = min(sw.steps, (q + 1u) * kChunkSpans);
        uint32_t ties = 0u;
        for (uint32_t s = q * kChunkSpans; s < s1; ++s) {
            float v[kVecPerThread][4];
            uint32_t valid;
            load_span(e, sw.first + int64_t(s) * kSpan, d, v, valid);
            uint32_t tie = 0u;
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    tie |= uint32_t(((valid >> (4 * j + x)) & 1u) && magnitude_key(v[j][x]) == T)
                           << (4 * j + x);
            uint32_t total;
            big_prefix(uint32_t(__popc(tie)), scan, turn, total);
            ties += total;
        }
        if (tid == 0) s_before = ties_before_chunk(ws.chunk_state, q, ties);
        __syncthreads();
        uint32_t rank = s_before;
        for (uint32_t s = q * kChunkSpans; s < s1; ++s) {
            const int64_t s0 = sw.first + int64_t(s) * kSpan;
            float v[kVecPerThread][4];
            uint32_t valid;
            load_span(e, s0, d, v, valid);
            uint32_t keep = 0u, tie = 0u, above = 0u;
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int b = 4 * j + x;
                    const uint32_t key = magnitude_key(v[j][x]);
                    if (!((valid >> b) & 1u)) continue;
                    if (key >= base && ((key - base) >> bits) == 0u) {
                        keep |= uint32_t(key > T) << b;
                        tie |= uint32_t(key == T) << b;
                    } else if (clear_above) {
                        above |= 1u << b;   // above the bin of zero: already sent
                    }
                }
            }
            // rank of each tied element in index order: earlier spans, then
            // earlier vector slots j, lower threads, lower c in the thread
#pragma unroll
            for (int j = 0; j < kVecPerThread; ++j) {
                const uint32_t tj = (tie >> (4 * j)) & 0xfu;
                uint32_t slot_total;
                uint32_t r = rank + big_prefix(uint32_t(__popc(tj)), scan, turn, slot_total);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    if ((tj >> x) & 1u) {
                        keep |= uint32_t(r < m) << (4 * j + x);
                        ++r;
                    }
                }
                rank += slot_total;
            }
            uint32_t total;
            const uint32_t pos = big_prefix(uint32_t(__popc(keep)), scan, turn, total);
            big_append(sh.keep, fill, keep, pos, total, v, s0, &c->emit2, cap, idx, val, scan, turn);
            clear_span(e, s0, keep | above);
        }
    }
    big_flush(sh.keep, fill, &c->emit2, cap, idx, val);
}

}  // namespace

size_t topk_path_flag_offset() { return offsetof(TopkCtl, fast); }

size_t topk_workspace_size(int64_t d, int64_t k) {
    const size_t ccap = size_t(candidate_capacity(d, k)), lcap = size_t(list_capacity(d));
    return kCtlBytes + round256(kHistBytes) +
           round256(sizeof(unsigned long long) * size_t(max_chunks(d))) +
           round256(sizeof(int32_t) * ccap) + round256(sizeof(float) * ccap) +
           round256(sizeof(int32_t) * lcap) + round256(sizeof(float) * lcap);
}

hipError_t launch_topk(const float *g, float *e, int64_t d, float lr, int64_t k,
                       int32_t *idx, float *val, void *workspace, hipStream_t stream) {
    if (d == 0) return hipSuccess;
    const Workspace ws = carve(workspace, d, k);
    const uint32_t kk = uint32_t(k);
    const Sweep tiles = sweep_start(e, d, kTile), spans = sweep_start(e, d, kSpan);
    uint32_t pgrid = balanced_grid(tiles.steps, kPass1LongWorkgroupsPerCU);
    if (tiles.steps < kPass1LongTiles * pgrid)
        pgrid = balanced_grid(tiles.steps, kPass1WorkgroupsPerCU);
    const bool by_xcd = tiles.steps >= uint32_t(kXcdWalkMinTiles) * pgrid;
    const uint32_t grid = balanced_grid(spans.steps, kBigWorkgroupsPerCU);

    topk_reset_kernel<<<kResetGrid, kBlock, 0, stream>>>(ws);
    topk_pass1_kernel<<<pgrid, kBlock, 0, stream>>>(g, e, d, lr, tiles, by_xcd, kk, idx,
                                                       val, ws);
    if (k == 0) return hipGetLastError();
    topk_step3_kernel<<<grid, kBig, 0, stream>>>(e, d, spans, kk, idx, val, ws);
    topk_step4_kernel<<<grid, kBig, 0, stream>>>(e, d, spans, kk, idx, val, ws);
    topk_emit_kernel<<<grid, kBig, 0, stream>>>(e, d, spans, kk, idx, val, ws);
    return hipGetLastError();
}

}  // namespace efs
