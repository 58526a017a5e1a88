// Exact streaming selection of the n largest (key, index) pairs of a row by one workgroup.
//
// Candidates are pushed into an LDS buffer as 64-bit composites (order-preserving image of the float
// key in the high word, complemented index in the low word: a larger composite is a larger key or,
// for equal keys - -0 and +0 are equal -, a smaller index, so all composites of a row are distinct).  Only composites above the
// current threshold are pushed.  A compaction finds a lower bound of the n-th largest composite, makes it the
// new threshold and keeps the entries at or above it.  In the stream a buffer of up to 256 entries is searched bit by bit
// for the top 20 bits of the n-th key, by every wave for itself (nth_key); a handful of entries too many survive.  Fuller buffers
// go by radix passes, which stop after the top 16 bits unless more than kTopKeep entries share them.  Where many entries
// share the bits, and at the end of the row, the n-th composite is found exactly, by counting ranks or with all 8 radix passes.
// Nothing that belongs to the final top n is ever dropped: the threshold is a lower bound of the n-th largest of what has been seen.
// (4096 x 128,256, k = 50 and s = 16, T = 1: 500 us with rank counts, radix passes and a priming run over every entry of the first
// round; 420 with bits, with priming by a key per thread, with what the compactions decide in scalar registers, and with priorities
// by what is left of the row.)
//
// Capacity.  The caller works in epochs of a few stream rounds without any barrier.  A push that finds the
// buffer full raises `over` instead of storing its entry, and the caller then starts the row again in a careful
// mode: one wave and one round at a time, with a compaction check after each such step.  A step starts with
// fewer than kTopTrigger entries and adds at most 8 per thread of one wave, so in that mode kTopCapSmall =
// kTopTrigger + 64 * 8 slots always suffice, whatever the order of the data.  Small buffers are what lets five
// workgroups share a compute unit; selections of more than kTopSmallN entries push so much in an ordinary epoch
// that they get kTopCapMid, kTopCapBig or kTopCapOne slots instead (the kernels are instantiated for each).
#pragma once

#include "difr_device.hpp"
#include "selection_epochs.hpp"

namespace difr {

constexpr int kTopFresh = 16;      // a compaction is due after max(n, kTopFresh) pushes (measured: 8 to 64 within 1%)
constexpr int kTopSmallN = 64;     // largest n served with the small buffer
constexpr int kTopMaxN = 256;      // largest n supported
constexpr int kTopKeep = 256;      // a coarse compaction may leave up to this many entries
constexpr int kTopBits = 20;       // key bits at which a coarse compaction or the priming separates (nth_key)
constexpr int kTopTies = 8;        // more entries than this that share the n-th key's bits: what follows is exact

// float -> uint32 such that a < b  <=>  image(a) < image(b)  (-0 < +0; NaNs must be kept out by the caller)
__device__ __forceinline__ uint32_t float_order_bits(float f)
{
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float float_from_order_bits(uint32_t o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}
// (-0 and +0 are the same key - between them the index decides -, so -0 is read as +0: x + 0 does that)
__device__ __forceinline__ uint64_t top_composite(float key, int32_t index)
{
    return ((uint64_t)float_order_bits(key + 0.0f) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)index);
}
__device__ __forceinline__ float top_key(uint64_t c) { return float_from_order_bits((uint32_t)(c >> 32)); }
__device__ __forceinline__ int32_t top_index(uint64_t c) { return (int32_t)(0xFFFFFFFFu - (uint32_t)c); }

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | lo;
}

// LDS scratch shared by the selections of one workgroup (they never run at the same time).
struct TopScratch {
    int32_t hist[256];
    int32_t wave_sum[kWaves];
    int32_t sel_bin, sel_need, kept;
    uint64_t sel64;
    uint64_t tmp[kTopKeep];
};

// Key bits of the n-th largest of the entries whose top kTopBits key bits the lanes of this wave hold, PER to a lane (0: none), or
// 0 if there are fewer; `at_or_above`: how many have these bits or larger ones.  A search bit by bit, counting with ballots: every
// wave finds it by itself from the same values, without a barrier, in kTopBits * PER compares.  Without TIGHT the bits may be those of
// a smaller key that still lies above the next entry's (and any key at all if there are only n entries).
template <int PER, bool TIGHT = false>
__device__ __forceinline__ uint32_t nth_key(const uint32_t (&k)[PER], int n, int &at_or_above)
{
    uint32_t prefix = 0;
    auto count = [&](uint32_t least) {
        int c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) c += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(k[i] >= least));
        return c;
    };
    at_or_above = 0x7FFFFFFF;
    for (uint32_t bit = 1u << (kTopBits - 1); bit != 0u; bit >>= 1) {
        const int c = count(prefix | bit);
        if (c >= n) {
            prefix |= bit;
            at_or_above = c;
            if (!TIGHT && c == n) break;  // (the bits found separate exactly n from the others)
        }
    }
    return prefix;
}

struct TopN {
    uint64_t *buf;   // `cap` slots in LDS
    int cap;
    int32_t *count;  // in LDS
    int n;
    uint64_t theta;  // wave-uniform copy of the threshold: only composites above it are pushed
    int trigger;     // fill level at which the next compaction is due: max(n, kTopFresh) pushes after the last one, so
                     // that the threshold, which is also the bound of the stream's gates, stays fresh
    bool full;       // this thread's push took the buffer to the compaction trigger (combine over the workgroup
                     // with __syncthreads_or: reading the counter instead would race with the next round's pushes)
    bool over;       // a push of this thread found the buffer full: the row must be started again, carefully
    bool priming;    // see begin_prime()
    uint64_t prime_best;

    __device__ __forceinline__ void init(uint64_t *buf_, int32_t *count_, int n_, int cap_)
    {
        buf = buf_;
        cap = cap_;
        count = count_;
        n = n_;
        theta = n_ > 0 ? 0ull : ~0ull;  // nothing wanted: nothing is ever pushed
        trigger = n_ > kTopFresh ? n_ : kTopFresh;
        full = false;
        over = false;
        priming = false;
        prime_best = 0ull;
        if (threadIdx.x == 0) *count = 0;
    }

    __device__ __forceinline__ void new_epoch() { over = false; }

    // Priming.  While there is no threshold every entry of the first round is a candidate: 2048 pushes through
    // one counter and a compaction over all of them.  Instead the first round is run twice: the first time each
    // thread only remembers its best candidate; the n-th largest of those 256 is a valid lower bound of the
    // n-th largest overall (they are real entries), it becomes the threshold, and the second, ordinary run of
    // the round pushes only what lies above it.
    __device__ __forceinline__ void begin_prime()
    {
        priming = true;
        prime_best = 0ull;
    }
    // All 256 threads, after the priming run of the round; ends with a __syncthreads().  Returns true if a
    // threshold was found (the caller re-targets its gates either way and runs the round again).
    __device__ __forceinline__ bool end_prime(TopScratch &s)
    {
        priming = false;
        // (a small selection does not need all 256 candidates: the best of every 4 or 2 neighbouring lanes are real
        // entries too, and the n-th largest of 64 or 128 of them costs a fraction of the rank count over 256 to find -
        // it lies a few ranks lower, which lets a few more entries of the first round through.  Of equal - masked - entries, of which
        // the n-th candidate is the one with index 8 n group at most, 896 do for n = 28 and 56, with room for some others in 1024 slots.)
        const int group = n <= 28 ? 4 : (n <= 56 ? 2 : 1);
        if (group >= 2) {
            const uint64_t o = __shfl_xor(prime_best, 1, 64);
            if (o > prime_best) prime_best = o;
        }
        if (group >= 4) {
            const uint64_t o = __shfl_xor(prime_best, 2, 64);
            if (o > prime_best) prime_best = o;
        }
        if (prime_best != 0ull && ((int)threadIdx.x & (group - 1)) == 0) {
            const int32_t i = atomicAdd(count, 1);
            buf[i] = prime_best;  // at most one per thread
        }
        __syncthreads();
        const bool moved = compact(s, false);
        // the primed entries are dropped (they come again with the round itself); the n-th largest of them must
        // pass the push test then, so the threshold is put just below it
        if (threadIdx.x == 0) *count = 0;
        if (moved) theta -= 1ull;
        trigger = min(kTopTrigger, n > kTopFresh ? n : kTopFresh);
        full = false;
        __syncthreads();
        return moved;
    }

    // The same from one key per thread (float_order_bits of a real entry's key; 0: none) with one barrier instead of a compaction
    // and without running the round's entries through push(): publish_prime(), a __syncthreads(), read_prime().  `slots`: kBlock words.
    // read_prime() returns the threshold, or 0 if there are too few keys, if the n-th is a masked entry's, or if so many keys share its
    // bits (coarse logits; 256 bf16 keys around -10 share them by dozens) that it would let half as many entries again through, or - where
    // all keys are at or above it, which says nothing - if more than kTopTies do: then the priming run above finds one.  The next barrier
    // after it frees the slots.
    __device__ __forceinline__ int prime_group() const { return n <= 32 ? 4 : (n <= 100 ? 2 : 1); }
    // whether `lanes` keys can be enough (uniform)
    __device__ __forceinline__ bool can_prime(int lanes) const { return n * prime_group() <= lanes; }
    __device__ __forceinline__ void publish_prime(uint32_t key, uint32_t *slots) const
    {
        const int group = prime_group();
        if (group >= 2) key = max(key, (uint32_t)__shfl_xor((int)key, 1, 64));
        if (group >= 4) key = max(key, (uint32_t)__shfl_xor((int)key, 2, 64));
        if (((int)threadIdx.x & (group - 1)) == 0) slots[(int)threadIdx.x / group] = key >> (32 - kTopBits);
    }
    template <int PER>
    __device__ __forceinline__ uint64_t read_prime_of(const uint32_t *slots) const
    {
        uint32_t k[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) k[i] = slots[((int)threadIdx.x & 63) + 64 * i];
        int at_or_above, equal = 0;
        const uint32_t p = nth_key<PER, true>(k, n, at_or_above);
#pragma unroll
        for (int i = 0; i < PER; ++i) equal += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(k[i] == p));
        const bool coarse = at_or_above > n + max(kTopTies, n / 2) || (at_or_above == 64 * PER && equal > kTopTies);
        return p <= 0x007FFFFFu >> (32 - kTopBits) || coarse ? 0ull : (uint64_t)p << (64 - kTopBits);
    }
    __device__ __forceinline__ uint64_t read_prime(const uint32_t *slots) const
    {
        if (n <= 0) return ~0ull;
        const int group = prime_group();
        return group == 4 ? read_prime_of<1>(slots) : (group == 2 ? read_prime_of<2>(slots) : read_prime_of<4>(slots));
    }

    __device__ __forceinline__ void push(uint64_t c)
    {
        if (priming) {
            if (c > theta && c > prime_best) prime_best = c;
            return;
        }
        if (c > theta) {
            const int32_t i = atomicAdd(count, 1);
            if (i < cap)
                buf[i] = c;
            else
                over = true;  // no room: the entry is dropped and the row has to be started again
            if (i >= trigger - 1) full = true;
        }
    }

    // A coarse compaction of up to 64 * PER entries: every wave holds all of them and finds the threshold by itself; two barriers.  Returns
    // false, and has changed nothing, if too many entries share the threshold's bits.
    template <int PER>
    __device__ __forceinline__ bool compact_by_bits(int cnt)
    {
        const int lane = (int)threadIdx.x & 63;
        uint64_t c[PER];
        uint32_t k[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            c[i] = lane + 64 * i < cnt ? buf[lane + 64 * i] : 0ull;
            k[i] = (uint32_t)(c[i] >> (64 - kTopBits));
        }
        int kept;
        const uint32_t p = nth_key<PER>(k, n, kept);
        if (kept > n + kTopTies) return false;
        __syncthreads();
        if (threadIdx.x < 64) {
            int at = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const uint64_t m = __builtin_amdgcn_ballot_w64(k[i] >= p);
                if (k[i] >= p)
                    buf[at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = c[i];
                at += (int)__builtin_popcountll(m);
            }
            if (lane == 0) *count = kept;
        }
        theta = (uint64_t)p << (64 - kTopBits);
        trigger = min(kTopTrigger, kept + (n > kTopFresh ? n : kTopFresh));
        __syncthreads();
        return true;
    }

    // All 256 threads, after a barrier that follows the pushes.  If the buffer holds more than n entries,
    // raise the threshold to a lower bound of the n-th largest composite and keep only the entries at or
    // above it: exactly the n largest (coarse = false), or a few more (coarse = true): up to 256 entries are cut at the
    // resolution of the top kTopBits key bits, n + kTopTies of them at most staying, more at that of the top 16, at most kTopKeep
    // staying; where more share the bits the cut is exact.  Returns true if the threshold moved.  Ends with a __syncthreads().
    __device__ __forceinline__ bool compact(TopScratch &s, bool coarse = false)
    {
        const int tid = threadIdx.x;
        const int cnt = __builtin_amdgcn_readfirstlane(min(*count, cap));
        full = false;
        if (n <= 0) {  // nothing wanted: an impossible threshold
            __syncthreads();
            if (tid == 0) *count = 0;
            theta = ~0ull;
            __syncthreads();
            return true;
        }
        if (cnt <= n) {
            trigger = min(kTopTrigger, cnt + (n > kTopFresh ? n : kTopFresh));
            __syncthreads();
            return false;
        }
        if (coarse && cnt <= 2 * 64) {
            if (compact_by_bits<2>(cnt)) return true;
        } else if (coarse && cnt <= 4 * 64) {
            if (compact_by_bits<4>(cnt)) return true;
        }
        const bool by_rank = !coarse || cnt <= kBlock;
        if (by_rank && cnt <= kBlock) {
            // Few entries: every entry finds its rank by counting the entries above it (broadcast reads), the n
            // best move to the front in rank order and the n-th of them is the new, exact threshold.  Three
            // barriers instead of the dozen of the radix select below.
            const uint64_t mine = tid < cnt ? buf[tid] : 0ull;
            int r = 0;
            for (int i = 0; i < cnt; ++i) r += (int)(buf[i] > mine);
            if (tid < cnt && r == n - 1) s.sel64 = mine;
            __syncthreads();
            if (tid < cnt && r < n) buf[r] = mine;
            if (tid == 0) *count = n;
            theta = uniform64(s.sel64);
            trigger = min(kTopTrigger, n + (n > kTopFresh ? n : kTopFresh));
            __syncthreads();
            return true;
        }
        if (by_rank && cnt <= 2 * kBlock) {
            // the same with two entries per thread: one broadcast read serves both
            uint64_t mine0 = buf[tid], mine1 = tid + kBlock < cnt ? buf[tid + kBlock] : 0ull;
            int r0 = 0, r1 = 0;
            for (int i = 0; i < cnt; ++i) {
                const uint64_t c = buf[i];
                r0 += (int)(c > mine0);
                r1 += (int)(c > mine1);
            }
            if (r0 == n - 1) s.sel64 = mine0;
            if (tid + kBlock < cnt && r1 == n - 1) s.sel64 = mine1;
            __syncthreads();
            if (r0 < n) buf[r0] = mine0;
            if (tid + kBlock < cnt && r1 < n) buf[r1] = mine1;
            if (tid == 0) *count = n;
            theta = uniform64(s.sel64);
            trigger = min(kTopTrigger, n + (n > kTopFresh ? n : kTopFresh));
            __syncthreads();
            return true;
        }
        uint64_t prefix = 0ull, mask = 0ull;
        int need = n;        // rank of the wanted composite among the entries that match the prefix
        int at_or_above = cnt;  // entries at or above the prefix found so far (unset low bits zero)
        for (int pass = 7; pass >= 0; --pass) {
            if (coarse && pass < 6 && at_or_above <= kTopKeep) break;
            if (at_or_above == n) break;  // the prefix already separates exactly n entries from the rest
            const int shift = 8 * pass;
            s.hist[tid] = 0;
            __syncthreads();
            for (int i = tid; i < cnt; i += kBlock) {
                const uint64_t c = buf[i];
                if ((c & mask) == prefix) atomicAdd(&s.hist[(int)((c >> shift) & 255ull)], 1);
            }
            __syncthreads();
            // suffix sums over the 256 bins: thread b gets the number of matching entries in bins >= b
            int v = s.hist[tid];
            const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_down(v, off, 64);
                if (lane + off < 64) v += o;
            }
            if (lane == 0) s.wave_sum[wave] = v;
            __syncthreads();
            for (int w = wave + 1; w < kWaves; ++w) v += s.wave_sum[w];
            const int above = v - s.hist[tid];  // matching entries in bins > tid
            if (above < need && v >= need) {    // exactly one thread
                s.sel_bin = tid;
                s.sel_need = need - above;
                s.kept = (n - need) + v;
            }
            __syncthreads();
            prefix |= (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(s.sel_bin) << shift;
            mask |= 255ull << shift;
            need = __builtin_amdgcn_readfirstlane(s.sel_need);
            at_or_above = __builtin_amdgcn_readfirstlane(s.kept);
            __syncthreads();
        }
        // gather the survivors (at_or_above <= kTopKeep of them) and move them to the front
        if (tid == 0) s.kept = 0;
        __syncthreads();
        for (int i = tid; i < cnt; i += kBlock) {
            const uint64_t c = buf[i];
            if (c >= prefix) {
                const int j = atomicAdd(&s.kept, 1);
                if (j < kTopKeep) s.tmp[j] = c;
            }
        }
        __syncthreads();
        for (int i = tid; i < at_or_above; i += kBlock) buf[i] = s.tmp[i];
        if (tid == 0) *count = at_or_above;
        theta = prefix;
        trigger = min(kTopTrigger, at_or_above + (n > kTopFresh ? n : kTopFresh));
        __syncthreads();
        return true;
    }

    // All 256 threads: reduce to exactly the n largest, then order them.  Afterwards buf[0 .. m) holds them in
    // descending order, m = min(n, entries seen); returns m.  Each survivor finds its rank by counting the
    // survivors above it (m <= 256 broadcast reads, no barriers).
    __device__ __forceinline__ int finish_sorted(TopScratch &s)
    {
        const int tid = threadIdx.x;
        __syncthreads();
        const int cnt = __builtin_amdgcn_readfirstlane(min(*count, cap));
        compact(s, false);
        if (cnt > n && cnt <= 2 * kBlock) return n;  // (the n best were put in rank order)
        const int m = min(min(*count, cap), n);
        if (tid < m) {
            const uint64_t mine = buf[tid];
            int rank = 0;
            for (int i = 0; i < m; ++i) rank += (int)(buf[i] > mine);
            s.tmp[rank] = mine;
        }
        __syncthreads();
        if (tid < m) buf[tid] = s.tmp[tid];
        __syncthreads();
        return m;
    }
};

}  // namespace difr
