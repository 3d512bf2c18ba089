// region.hip -- theta join with region pruning on gfx950 (the paper's improved theta join).
//
// Section 4.2 cuts the |T| x |S| matrix into regions of join-key ranges, with the same range
// boundaries on both axes (quantiles, figure "classb"), and classifies each region from its
// ranges alone (figures "greena"/"greenb"/"greenc"): in a green region every pair satisfies the
// condition, in a white region none does, and only red regions need pair-by-pair evaluation
// (Algorithm 3).  Here the regions shrink to single R rows: with both sides sorted by column a,
// the S rows that satisfy op_a with one R row are one interval of S (two for !=), found by binary
// search.  Inside it every row is green for op_a, outside it white, and nothing is left red: a
// condition on column c is the only thing evaluated pair by pair, and only inside the interval.
//
//   1. setup:    value bins over a sample of both sides (gathered by one launch, binned by the
//                next), buckets (quantiles of the sample) made of whole bins, so both sides share
//                boundaries and bucket ids rise with the value; where a few bins hold most of the
//                sample, buckets between quantiles of the sorted sample instead;
//   2. sizes:    rows of each bucket; the last workgroup turns them into starts;
//   3. scatter:  rows (a, [c,] rid) into their buckets, tile by tile through LDS;
//   4. sort:     each bucket sorted by a in LDS, written as columns: both sides are sorted;
//   5. count:    each R row's interval and its matches, long intervals walked by the wave and wide
//                ones cut into shares; the last workgroup scans the counts;
//   6. write:    the pairs of each wave from the offset the count pass gave it.
// Sides that fit one workgroup's LDS skip 1 to 3.
//
// What bounds it: launches and dependent memory round trips up to 1M rows a side (every pass
// moves 8 to 32 MB, 2 to 8 us at the copy rate, and takes 4 to 29), from 4M on the LDS work of
// the sort and the partition's traffic.  Count pass of a band of w = 8 at 4M x 4M: sample and
// setup 22 us, sizes 24, scatter 58, sort 50, intervals and counts 55.  The former design put
// every R row of a bucket against every S row of its red span, in 26 launches: 1M x 1M with a
// condition on c 414 us of kernels, now 110; the count at 4M x 4M 1200, now 211.
#include "region.hpp"
#include "debug.hpp"

#include "prof.hpp"

namespace jl {

namespace {

constexpr int kBlk = 1024;        // threads of the partition and sort kernels
constexpr int kPer = 4;           // rows per thread
constexpr int kCap = kBlk * kPer; // rows of a scatter tile, and of one LDS sort
constexpr int kSortBlk = 512;     // threads of a sort: four workgroups share a CU
constexpr int kSortPer = kCap / kSortBlk;
constexpr int kMeanRows = 2048;   // a bucket's mean size, at most (while bits < kMaxBits)
constexpr int kMaxBits = 13;      // 2^13 buckets: 64 KB of LDS state beside the scatter's tile
constexpr int kMinBinBits = 10;   // at least one bin per thread of the setup workgroup
constexpr int kMaxBinBits = 14;   // 68 KB of LDS counters, padding included
constexpr uint32_t kHeavyBin = 32;  // a bin with more samples, and more than a bucket's: see setup_k
constexpr int kSubBits = 12;      // value bins of one LDS sort: about one row each
constexpr int kSub = 1 << kSubBits;
constexpr uint32_t kRankBin = 64; // rows of a bin ranked one against the other, at most
constexpr int kJoinBlk = 256;     // threads of the count and write kernels
constexpr int kJoinWaves = kJoinBlk / kWave;
constexpr int64_t kMaxBlocks = 4096;  // R blocks of the count pass
// Intervals up to this length are walked lane by lane: neighbouring rows' intervals start close
// together, so each step's loads are nearly consecutive.  Longer ones are walked by the whole
// wave: without a condition on c one R row at a time, with one by whichever of two ways has fewer
// steps (by_rows).
constexpr uint32_t kSerial = 32;

struct Hdr {
    uint64_t total;
    int32_t lo;      // smallest sampled value
    uint32_t shift;  // bin = (a - lo) >> shift, clamped to the outer bins
    uint32_t nbins;
    uint32_t search; // 0: lut[bin] is the bucket; 1: the buckets of a bin are told apart by splitters
};

// Words of the cleared area: sizes of R's and S's buckets, arrivals at S's buckets of more than
// kCap rows, then these counters.
constexpr int kCntExtra = 0;  // entries of the extra chunk list
constexpr int kCntHist = 32;  // workgroups that finished the bucket sizes (an arrival set each)
constexpr int kCntCount = kCntHist + kArrivalWords;  // workgroups that finished counting
constexpr int kCounters = kCntCount + kArrivalWords;

struct Cols {
    const int32_t *a, *c, *rid;
    int64_t n;
};

__device__ __forceinline__ uint32_t bin_of(int32_t a, const Hdr& h)
{
    const uint32_t d = a < h.lo ? 0u : (uint32_t)a - (uint32_t)h.lo;
    return min(d >> h.shift, h.nbins - 1);
}

__device__ __forceinline__ int32_t wave_min_i(int32_t v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
    return v;
}

__device__ __forceinline__ int32_t wave_max_i(int32_t v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
    return v;
}

// Smallest and largest value of a BLOCK-thread workgroup; red: 2 * BLOCK / 64 words of LDS.
template <int BLOCK>
__device__ __forceinline__ void block_range(int32_t& lo, int32_t& hi, int32_t* red)
{
    constexpr int W = BLOCK / kWave;
    lo = wave_min_i(lo);
    hi = wave_max_i(hi);
    if (lane_id() == 0) {
        red[threadIdx.x / kWave] = lo;
        red[W + threadIdx.x / kWave] = hi;
    }
    __syncthreads();
    for (int w = 0; w < W; ++w) {
        lo = min(lo, red[w]);
        hi = max(hi, red[W + w]);
    }
    __syncthreads();
}

// Bits to shift a value span so that it falls below 2^bits.
__device__ __forceinline__ uint32_t span_shift(uint32_t span, int bits)
{
    const int len = span ? 32 - __builtin_clz(span) : 0;
    return len > bits ? (uint32_t)(len - bits) : 0u;
}

// The bucket of value a: the number of splitters up to a.  With h.search, lut[bin] counts those below
// the bin, so only the splitters inside the bin are searched.
__device__ __forceinline__ uint32_t bucket_of(int32_t a, const Hdr& h, const uint16_t* lut,
                                              const int32_t* __restrict__ split)
{
    const uint32_t bin = bin_of(a, h);
    uint32_t b = lut[bin];
    if (h.search) {  // uniform
        uint32_t e = lut[bin + 1];
        while (b < e) {
            const uint32_t m = (b + e) / 2;
            if (split[m] <= a) b = m + 1;
            else e = m;
        }
    }
    return b;
}

// ----------------------------------------------------------------------------------- setup --
// Evenly spaced rows of R, then of S, as one array, and the counters cleared.  Many workgroups,
// so that the scattered reads overlap (one workgroup took 64 us for 16K rows a side).
__global__ __launch_bounds__(kBlk) void sample_k(Cols R, Cols S, uint32_t sR, uint32_t sS,
                                                 int32_t* __restrict__ sample, uint32_t* __restrict__ zero,
                                                 uint32_t zeroWords)
{
    const uint32_t i = blockIdx.x * kBlk + threadIdx.x;
    if (i < sR) sample[i] = R.a[i * (R.n / sR)];
    else if (i < sR + sS) sample[i] = S.a[(i - sR) * (S.n / sS)];
    for (uint32_t z = i; z < zeroWords; z += gridDim.x * kBlk) zero[z] = 0;
}

// A word of an LDS counter array of which each thread scans 2^PB consecutive ones: one word of
// padding after each thread's, so that a wave's lanes read different banks (2^14 counters without
// it: 16 reads of 64 lanes on 4 banks).
template <int PB>
__host__ __device__ constexpr uint32_t padded(uint32_t i)
{
    return i + (i >> PB);
}

// The samples a skewed column's splitters are chosen from: 16 a thread, sorted in registers, across
// lanes and, for the ten steps between waves, through LDS.
constexpr int kSplitPer = 16;
constexpr uint32_t kSplitSample = kBlk * kSplitPer;

template <int J>
__device__ __forceinline__ void sort_step(int32_t (&v)[kSplitPer], uint32_t k)
{
#pragma unroll
    for (int i = 0; i < kSplitPer; ++i)
        if (!(i & J)) {
            const bool up = ((threadIdx.x * kSplitPer + i) & k) == 0;
            const int32_t lo = min(v[i], v[i | J]), hi = max(v[i], v[i | J]);
            v[i] = up ? lo : hi;
            v[i | J] = up ? hi : lo;
        }
}

// A bitonic network; afterwards value i of thread t is number t * kSplitPer + i in order.
// lds: kSplitSample words.
__device__ void sort_sample(int32_t (&v)[kSplitPer], int32_t* lds)
{
    const uint32_t tid = threadIdx.x;
    for (uint32_t k = 2; k <= kSplitSample; k *= 2)
        for (uint32_t j = k / 2; j > 0; j /= 2) {
            if (j >= kSplitPer) {
                const uint32_t t = j / kSplitPer;  // the other thread of each pair: tid ^ t
                const bool low = ((tid & t) == 0) == ((tid * kSplitPer & k) == 0);
                int32_t o[kSplitPer];
                if (t >= (uint32_t)kWave) {
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < kSplitPer; ++i) lds[i * kBlk + tid] = v[i];
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < kSplitPer; ++i) o[i] = lds[i * kBlk + (tid ^ t)];
                } else {
#pragma unroll
                    for (int i = 0; i < kSplitPer; ++i) o[i] = __shfl_xor(v[i], (int)t);
                }
#pragma unroll
                for (int i = 0; i < kSplitPer; ++i) v[i] = low ? min(v[i], o[i]) : max(v[i], o[i]);
            } else if (j == 8) {
                sort_step<8>(v, k);
            } else if (j == 4) {
                sort_step<4>(v, k);
            } else if (j == 2) {
                sort_step<2>(v, k);
            } else {
                sort_step<1>(v, k);
            }
        }
    __syncthreads();
}

// One workgroup: bins over the sampled range, buckets of about equal sample counts.  Rows outside
// the sampled range fall into the outer bins, so an outlier does not stretch the bins.  A
// bucket's size follows its sample count, 32 rows (16 from 8192 buckets on): up to 16M rows it stays
// under kCap, twice the mean or more, but for a few in a million (16 samples: one or two of 2048
// buckets were larger, and merging the chunks of an S bucket ended 25 us after the other sorts, 52 us
// at 4M rows a side).
// That is so while a bin, the unit the buckets are made of, holds less than a bucket.  A bin with more
// samples than that (a column with most values in a sliver of its range, or a frequent value) has
// the buckets made of single values instead: between quantiles of a sorted sample, of 2 to 8 samples
// each, and a value that fills a bucket has one of its own, whose chunks are in order as they are.
// Left to the bins, one workgroup merged most of S: 1K x 4M rows, half of S one value, 75 ms.
__global__ __launch_bounds__(kBlk) void setup_k(const int32_t* __restrict__ sample, uint32_t m, int binBits,
                                                int bits, Hdr* __restrict__ h, uint16_t* __restrict__ lut,
                                                int32_t* __restrict__ split)
{
    extern __shared__ uint32_t bins[];
    __shared__ int32_t red[2 * kBlk / kWave];
    __shared__ uint32_t wsum[kBlk / kWave + 1];
    const int tid = threadIdx.x;
    const int nb = 1 << binBits;
    constexpr int kPad = kMaxBinBits - 10;  // 16 counters a thread at most
    for (int i = tid; i < (int)padded<kPad>(nb); i += kBlk) bins[i] = 0;
    constexpr int kBatch = 16;  // loads of a thread in flight together
    auto each = [&](auto f) {
        for (uint32_t i0 = 0; i0 < m; i0 += kBlk * kBatch) {
            int32_t a[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) a[k] = sample[min(i0 + k * kBlk + tid, m - 1)];
#pragma unroll
            for (int k = 0; k < kBatch; ++k)
                if (i0 + k * kBlk + tid < m) f(a[k]);
        }
    };
    int32_t lo = INT32_MAX, hi = INT32_MIN;
    each([&](int32_t a) {
        lo = min(lo, a);
        hi = max(hi, a);
    });
    block_range<kBlk>(lo, hi, red);
    Hdr hh{0, lo, span_shift((uint32_t)hi - (uint32_t)lo, binBits), (uint32_t)nb, 0};
    each([&](int32_t a) { atomicAdd(&bins[padded<kPad>(bin_of(a, hh))], 1u); });
    __syncthreads();
    const int per = nb / kBlk;
    uint32_t s = 0, most = 0, tot;
    for (int k = 0; k < per; ++k) {
        const uint32_t c = bins[padded<kPad>(tid * per + k)];
        s += c;
        most = max(most, c);
    }
    const uint32_t B = 1u << bits;
    hh.search = __syncthreads_or(most > max(m / B, kHeavyBin)) ? 1 : 0;
    if (tid == 0) *h = hh;
    if (!hh.search) {
        uint32_t run = block_excl_scan<kBlk>(s, wsum, &tot);
        const float scale = (float)B / (float)tot;  // rounded, but never falling as run rises
        for (int k = 0; k < per; ++k) {
            uint32_t& c = bins[padded<kPad>(tid * per + k)];
            const uint32_t b = (uint32_t)((float)run * scale);  // run <= tot <= 2^17: exact as a float
            run += c;
            c = min(b, B - 1);
        }
    } else {
        const uint32_t n = min(m, kSplitSample);
        int32_t v[kSplitPer];
#pragma unroll
        for (int i = 0; i < kSplitPer; ++i) {
            const uint32_t e = (uint32_t)i * kBlk + tid;
            v[i] = e < n ? sample[(uint32_t)((uint64_t)e * m / n)] : INT32_MAX;
        }
        int32_t* t = reinterpret_cast<int32_t*>(bins);
        sort_sample(v, t);
#pragma unroll
        for (int i = 0; i < kSplitPer; ++i) t[tid * kSplitPer + i] = v[i];
        __syncthreads();
        constexpr int kMine = (1 << kMaxBits) / kBlk;
        int32_t sp[kMine];  // splitters tid, tid + kBlk, ... of B - 1
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            const uint32_t i = (uint32_t)k * kBlk + tid;
            sp[k] = 0;
            if (i + 1 < B) {
                const int32_t q = t[(i + 1) * n >> bits];  // at most 2^13 * 2^14
                // a value of several quantiles: its own bucket, from the first to the next value
                const bool again = i > 0 && t[i * n >> bits] == q;
                sp[k] = again && q < INT32_MAX ? q + 1 : q;
                split[i] = sp[k];
            }
        }
        __syncthreads();
        for (int i = tid; i < (int)padded<kPad>(nb); i += kBlk) bins[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kMine; ++k)
            if ((uint32_t)k * kBlk + tid + 1 < B) atomicAdd(&bins[padded<kPad>(bin_of(sp[k], hh))], 1u);
        __syncthreads();
        s = 0;
        for (int k = 0; k < per; ++k) s += bins[padded<kPad>(tid * per + k)];
        uint32_t run = block_excl_scan<kBlk>(s, wsum, &tot);
        for (int k = 0; k < per; ++k) {
            uint32_t& c = bins[padded<kPad>(tid * per + k)];
            const uint32_t below = run;
            run += c;
            c = below;
        }
        if (tid == 0) lut[nb] = (uint16_t)(B - 1);
    }
    __syncthreads();
    for (int i = tid; i < nb / 2; i += kBlk)
        reinterpret_cast<uint32_t*>(lut)[i] = bins[padded<kPad>(2 * i)] | bins[padded<kPad>(2 * i + 1)] << 16;
}

// --------------------------------------------------------------------------- bucket sizes --
// Exclusive starts of a side's B buckets (base[0..B], cur: the scatter's cursors), and an entry
// of the extra chunk list for every chunk of kCap rows of a bucket past its first one.
__device__ void bucket_starts(const uint32_t* tot, uint32_t* base, uint32_t* cur, int B, uint32_t side,
                              uint2* extra, uint32_t* nextra, uint32_t* wsum)
{
    uint32_t carry = 0;
    for (int b0 = 0; b0 < B; b0 += kBlk) {
        const int b = b0 + (int)threadIdx.x;
        const uint32_t n = b < B ? tot[b] : 0u;
        uint32_t sum;
        const uint32_t at = carry + block_excl_scan<kBlk>(n, wsum, &sum);
        if (b < B) {
            base[b] = at;
            cur[b] = at;
            if (n > (uint32_t)kCap) {
                const uint32_t k = (n - 1) / kCap;
                const uint32_t x = atomicAdd(nextra, k);
                for (uint32_t j = 0; j < k; ++j) extra[x + j] = make_uint2(side << 31 | (uint32_t)b, j + 1);
            }
        }
        carry += sum;
    }
    if (threadIdx.x == 0) base[B] = carry;
}

struct Sides {
    Cols X[2];           // R, S
    uint32_t split;      // workgroups of R (S's follow)
    int64_t chunk;       // rows per workgroup
    const Hdr* h;
    const uint16_t* lut;
    const int32_t* splitters;
    int B;
    uint32_t* zero;      // [2B] sizes, [B] arrivals, counters
    uint32_t *base, *cur;  // [2][B + 1], [2][B]
    uint2* extra;
    uint16_t* id[2];     // each row's bucket
    void* part[2];       // bucketed rows: int4 (a, c, rid, 0) with a condition on c, else int2 (a, rid)
    int32_t *oa[2], *oc[2], *orid[2];  // sorted columns
};

// The bucket of every row is kept (16 bits a row) for the scatter.  The table of bins goes through
// LDS: a gather from the caches serves one line per clock and lane.
// LDS: cnt[B] | lut[nbins + 1] (16 bits)
__global__ __launch_bounds__(kBlk) void sizes_k(Sides s)
{
    extern __shared__ uint32_t cnt[];
    uint16_t* lut = reinterpret_cast<uint16_t*>(cnt + s.B);
    __shared__ uint32_t wsum[kBlk / kWave + 1];
    __shared__ uint32_t last;
    const int side = blockIdx.x >= s.split;
    const int64_t beg = (int64_t)(blockIdx.x - (side ? s.split : 0)) * s.chunk;
    const Cols X = s.X[side];
    const int64_t end = beg + s.chunk < X.n ? beg + s.chunk : X.n;
    for (int b = threadIdx.x; b < s.B; b += kBlk) cnt[b] = 0;
    const Hdr h = *s.h;
    for (uint32_t k = threadIdx.x; k <= h.nbins / 2; k += kBlk)
        reinterpret_cast<uint32_t*>(lut)[k] = reinterpret_cast<const uint32_t*>(s.lut)[k];
    __syncthreads();
    for (int64_t i0 = beg; i0 < end; i0 += kCap) {
        int32_t a[kPer];
        uint16_t b[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = i0 + q * kBlk + threadIdx.x;
            a[q] = X.a[i < end ? i : beg];
        }
#pragma unroll
        for (int q = 0; q < kPer; ++q) b[q] = (uint16_t)bucket_of(a[q], h, lut, s.splitters);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t i = i0 + q * kBlk + threadIdx.x;
            if (i < end) {
                s.id[side][i] = b[q];
                atomicAdd(&cnt[b[q]], 1u);
            }
        }
    }
    __syncthreads();
    uint32_t* tot = s.zero + side * s.B;
    for (int b = threadIdx.x; b < s.B; b += kBlk)
        if (cnt[b]) atomicAdd(&tot[b], cnt[b]);
    // Device-scope atomics act on memory beyond the XCD's L2, so a wave's additions are in place
    // once it has waited for them; a release fence would also write back the whole L2 (16 waves
    // of 512 workgroups doing that took 50 of the kernel's 70 us at 1M rows a side).
    drain();
    __syncthreads();
    uint32_t* counters = s.zero + 3 * s.B;
    if (threadIdx.x == 0) last = arrive_last(counters + kCntHist, blockIdx.x, gridDim.x);
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    for (int x = 0; x < 2; ++x)
        bucket_starts(s.zero + x * s.B, s.base + x * (s.B + 1), s.cur + x * s.B, s.B, (uint32_t)x, s.extra,
                      &counters[kCntExtra], wsum);
}

// --------------------------------------------------------------------------------- scatter --
// One tile of kCap rows: counted by bucket, given a place in every bucket by one atomic per
// bucket and tile, sorted by bucket in LDS and written in runs.  Rows of one bucket travel as one
// 16-byte (8-byte) record, so a run of two rows still fills a 32-byte sector.
// LDS: cnt[B] | dlt[B] | a[kCap] | rid[kCap] | [c[kCap]] | bucket[kCap] (16 bits)
template <bool HAS_C>
__global__ __launch_bounds__(kBlk) void scatter_rows_k(Sides s)
{
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ uint32_t wsum[kBlk / kWave + 1];
    uint32_t* cnt = lds;
    uint32_t* dlt = cnt + s.B;
    int32_t* ta = reinterpret_cast<int32_t*>(dlt + s.B);
    int32_t* tr = ta + kCap;
    int32_t* tc = tr + kCap;
    uint16_t* tb = reinterpret_cast<uint16_t*>(HAS_C ? tc + kCap : tc);
    const int tid = threadIdx.x;
    const int side = blockIdx.x >= s.split;
    const Cols X = s.X[side];
    const int64_t beg = (int64_t)(blockIdx.x - (side ? s.split : 0)) * kCap;
    const int n = (int)(X.n - beg < kCap ? X.n - beg : kCap);
    for (int b = tid; b < s.B; b += kBlk) cnt[b] = 0;
    int32_t a[kPer], c[kPer], r[kPer];
    uint32_t b[kPer], rank[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int e = q * kBlk + tid;
        const int64_t i = beg + (e < n ? e : 0);
        a[q] = X.a[i];
        if (HAS_C) c[q] = X.c[i];
        r[q] = X.rid ? X.rid[i] : (int32_t)i;
        b[q] = s.id[side][i];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (q * kBlk + tid < n) rank[q] = atomicAdd(&cnt[b[q]], 1u);
    __syncthreads();
    uint32_t* cur = s.cur + side * s.B;
    uint32_t carry = 0;
    for (int b0 = 0; b0 < s.B; b0 += kBlk) {
        const int k = b0 + tid;
        const uint32_t m = k < s.B ? cnt[k] : 0u;
        const uint32_t g = m ? atomicAdd(&cur[k], m) : 0u;
        uint32_t sum;
        const uint32_t at = carry + block_excl_scan<kBlk>(m, wsum, &sum);
        if (k < s.B) {
            cnt[k] = at;
            dlt[k] = g - at;
        }
        carry += sum;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (q * kBlk + tid < n) {
            const uint32_t p = cnt[b[q]] + rank[q];
            ta[p] = a[q];
            tr[p] = r[q];
            if (HAS_C) tc[p] = c[q];
            tb[p] = (uint16_t)b[q];
        }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = q * kBlk + tid;
        if (p < n) {
            const uint32_t at = dlt[tb[p]] + (uint32_t)p;
            if (HAS_C) static_cast<int4*>(s.part[side])[at] = make_int4(ta[p], tc[p], tr[p], 0);
            else static_cast<int2*>(s.part[side])[at] = make_int2(ta[p], tr[p]);
        }
    }
}

// ------------------------------------------------------------------------------------ sort --
struct Row {
    int32_t a, c, r;
};

template <bool HAS_C>
__device__ __forceinline__ Row part_row(const void* part, uint32_t i)
{
    if (HAS_C) {
        const int4 v = static_cast<const int4*>(part)[i];
        return Row{v.x, v.y, v.z};
    }
    const int2 v = static_cast<const int2*>(part)[i];
    return Row{v.x, 0, v.y};
}

// A bucket of more than kCap rows, its chunks of kCap rows sorted: merged pairwise by one
// workgroup, back and forth between the sorted columns and the bucketed rows (which nothing
// reads any more).  Each thread makes kSortPer consecutive rows of a merged run; where they start in
// its two halves is the usual binary search along the diagonal.
template <bool HAS_C>
__device__ void merge_chunks(const Sides& s, int side, uint32_t b0, uint32_t n)
{
    int32_t *oa = s.oa[side], *oc = s.oc[side], *orr = s.orid[side];
    void* part = s.part[side];
    // one value in every chunk (a value frequent enough to fill its own bucket): nothing to merge
    __shared__ uint32_t mixed;
    if (threadIdx.x == 0) mixed = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)threadIdx.x * kCap; i < n; i += (uint64_t)kSortBlk * kCap)
        if (oa[b0 + i] != oa[b0] || oa[b0 + min(i + kCap, (uint64_t)n) - 1] != oa[b0]) mixed = 1;
    __syncthreads();
    if (!mixed) return;
    bool cols = true;  // the rows are in the columns
    auto key = [&](uint32_t i) { return cols ? oa[b0 + i] : part_row<HAS_C>(part, b0 + i).a; };
    auto row = [&](uint32_t i) {
        if (cols) return Row{oa[b0 + i], HAS_C ? oc[b0 + i] : 0, orr[b0 + i]};
        return part_row<HAS_C>(part, b0 + i);
    };
    auto put = [&](uint32_t i, const Row& v) {
        if (cols) {
            if (HAS_C) static_cast<int4*>(part)[b0 + i] = make_int4(v.a, v.c, v.r, 0);
            else static_cast<int2*>(part)[b0 + i] = make_int2(v.a, v.r);
        } else {
            oa[b0 + i] = v.a;
            if (HAS_C) oc[b0 + i] = v.c;
            orr[b0 + i] = v.r;
        }
    };
    for (uint64_t w = kCap; w < n || !cols; w *= 2) {  // at the end the rows are in the columns
        for (uint64_t o = (uint64_t)threadIdx.x * kSortPer; o < n; o += (uint64_t)kSortBlk * kSortPer) {
            const uint32_t x0 = (uint32_t)(o / (2 * w) * (2 * w));  // run [x0, y0) with [y0, y1)
            const uint32_t y0 = (uint32_t)(x0 + w < n ? x0 + w : n);
            const uint32_t y1 = (uint32_t)(x0 + 2 * w < n ? x0 + 2 * w : n);
            const uint32_t d = (uint32_t)o - x0;
            uint32_t lo = d > y1 - y0 ? d - (y1 - y0) : 0u, hi = min(d, y0 - x0);
            while (lo < hi) {  // rows of the first half among the run's first d
                const uint32_t m = (lo + hi) / 2;
                if (key(x0 + m) <= key(y0 + d - 1 - m)) lo = m + 1;
                else hi = m;
            }
            uint32_t x = x0 + lo, y = y0 + d - lo;
            for (int q = 0; q < kSortPer && o + q < y1; ++q) {
                const bool first = y >= y1 || (x < y0 && key(x) <= key(y));
                put((uint32_t)o + q, row(first ? x : y));
                if (first) ++x;
                else ++y;
            }
        }
        cols = !cols;
        // the rows are read by this workgroup alone
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
}

// Ranks of a chunk's n rows by (a, position) from a bitonic network over LDS, 78 steps for kCap
// rows whatever their values.  key: kCap words of 8 bytes.
__device__ void bitonic_ranks(const Row (&v)[kSortPer], uint32_t n, uint64_t* key, uint32_t (&rank)[kSortPer])
{
    const uint32_t tid = threadIdx.x;
    const uint32_t N = n <= 1 ? 1u : 1u << (32 - __builtin_clz(n - 1));
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) {
        const uint32_t e = (uint32_t)(q * kSortBlk) + tid;
        if (e < N) key[e] = e < n ? (uint64_t)((uint32_t)v[q].a ^ 0x80000000u) << 32 | e : ~0ull;
    }
    for (uint32_t k = 2; k <= N; k *= 2)
        for (uint32_t j = k / 2; j > 0; j /= 2) {
            __syncthreads();
            for (uint32_t i = tid; i < N / 2; i += kSortBlk) {
                const uint32_t x = 2 * j * (i / j) + i % j, y = x + j;
                const uint64_t kx = key[x], ky = key[y];
                if ((kx > ky) == ((x & k) == 0)) {
                    key[x] = ky;
                    key[y] = kx;
                }
            }
        }
    __syncthreads();
    uint32_t e[kSortPer];
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) e[q] = q * kSortBlk + tid < n ? (uint32_t)key[q * kSortBlk + tid] : 0u;
    __syncthreads();
    uint32_t* at = reinterpret_cast<uint32_t*>(key);
#pragma unroll
    for (int q = 0; q < kSortPer; ++q)
        if (q * kSortBlk + tid < n) at[e[q]] = (uint32_t)(q * kSortBlk) + tid;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortPer; ++q)
        if (q * kSortBlk + tid < n) rank[q] = at[q * kSortBlk + tid];
    __syncthreads();
}

constexpr int kSubPad = 3;  // log2 of the bins a thread scans
static_assert(kSub == kSortBlk << kSubPad, "bins of a sort");
__device__ __forceinline__ uint32_t sub_at(uint32_t i) { return padded<kSubPad>(i); }
constexpr uint32_t kSubWords = padded<kSubPad>(kSub) + 1;

// One chunk of up to kCap rows of one bucket per workgroup, sorted by a: counted into kSub value
// bins of the chunk's own range (about one row each), placed by bin, and each row of S ranked
// against the rows of its bin (nothing to do when a bin holds one value; when some bin holds more
// than kRankBin rows, a frequent value among others, the chunk goes through a bitonic network
// instead, since ranking takes the square of that number).  R stays in the order
// of the bins: its rows only have to lie near each other.  direct: the input columns, one
// workgroup per side; else workgroup i < 2B takes bucket i's first chunk, the others the list of
// further chunks.
// (4M rows a side: 50 us, 79 with unpadded bins and buckets of 16 samples, a few of which were merged.)
// LDS: bins[kSub + 1] (padded) | one column of kCap rows, which stages a, then rid and c, into sorted order
template <bool HAS_C>
__global__ __launch_bounds__(kSortBlk) void sort_k(Sides s, int direct)
{
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ int32_t red[2 * kSortBlk / kWave];
    __shared__ uint32_t wsum[kSortBlk / kWave + 1];
    __shared__ uint32_t last, crowded;
    if (threadIdx.x == 0) crowded = 0;
    uint32_t* bin = lds;
    int32_t* ta = reinterpret_cast<int32_t*>(bin + kSubWords);
    const int tid = threadIdx.x;
    int side;
    uint32_t b0, at, n, total;  // the bucket's first row, the chunk's first row and rows, the bucket's rows
    int bucket = 0;
    if (direct) {
        side = blockIdx.x;
        b0 = at = 0;
        n = total = (uint32_t)s.X[side].n;
        if (side == 0)
            for (int i = tid; i < kCounters; i += kSortBlk) s.zero[3 * s.B + i] = 0;
    } else {
        uint32_t chunk = 0;
        if (blockIdx.x < 2 * (uint32_t)s.B) {
            side = blockIdx.x >= (uint32_t)s.B;
            bucket = (int)blockIdx.x - side * s.B;
        } else {
            const uint32_t x = blockIdx.x - 2 * (uint32_t)s.B;
            if (x >= s.zero[3 * s.B + kCntExtra]) return;
            const uint2 e = s.extra[x];
            side = (int)(e.x >> 31);
            bucket = (int)(e.x & 0x7FFFFFFFu);
            chunk = e.y;
        }
        const uint32_t* base = s.base + side * (s.B + 1);
        b0 = base[bucket];
        total = base[bucket + 1] - b0;
        at = b0 + chunk * kCap;
        n = min((uint32_t)kCap, total - chunk * kCap);
        if (total == 0) return;
    }
    Row v[kSortPer];
    uint32_t sub[kSortPer], rank[kSortPer];
    int32_t lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) {
        const uint32_t e = (uint32_t)(q * kSortBlk + tid);
        const uint32_t i = at + (e < n ? e : 0u);
        if (direct) {
            const Cols& X = s.X[side];
            v[q] = Row{X.a[i], HAS_C ? X.c[i] : 0, X.rid ? X.rid[i] : (int32_t)i};
        } else {
            v[q] = part_row<HAS_C>(s.part[side], i);
        }
    }
    for (int i = tid; i < (int)kSubWords; i += kSortBlk) bin[i] = 0;
#pragma unroll
    for (int q = 0; q < kSortPer; ++q) {
        lo = min(lo, v[q].a);
        hi = max(hi, v[q].a);
    }
    block_range<kSortBlk>(lo, hi, red);
    const uint32_t sh = span_shift((uint32_t)hi - (uint32_t)lo, kSubBits);
    if (lo == hi) {  // uniform: one value (all rows would be counted in one bin, one after the other)
#pragma unroll
        for (int q = 0; q < kSortPer; ++q) rank[q] = (uint32_t)(q * kSortBlk + tid);
    } else {
#pragma unroll
        for (int q = 0; q < kSortPer; ++q) {
            sub[q] = ((uint32_t)v[q].a - (uint32_t)lo) >> sh;
            if ((uint32_t)(q * kSortBlk + tid) < n) rank[q] = atomicAdd(&bin[sub_at(sub[q])], 1u);
        }
        __syncthreads();
        {
            constexpr int S = kSub / kSortBlk;
            uint32_t x[S], sum = 0, tot;
#pragma unroll
            for (int k = 0; k < S; ++k) {
                x[k] = bin[sub_at(tid * S + k)];
                sum += x[k];
                if (x[k] > kRankBin) crowded = 1;
            }
            uint32_t run = block_excl_scan<kSortBlk>(sum, wsum, &tot);
#pragma unroll
            for (int k = 0; k < S; ++k) {
                bin[sub_at(tid * S + k)] = run;
                run += x[k];
            }
            if (tid == 0) bin[sub_at(kSub)] = n;
        }
        __syncthreads();
        const bool exact = sh && side == 1;  // uniform: a bin spans several values, and S needs them in order
        if (exact && crowded) {
            bitonic_ranks(v, n, reinterpret_cast<uint64_t*>(lds), rank);
        } else {
#pragma unroll
            for (int q = 0; q < kSortPer; ++q)
                if ((uint32_t)(q * kSortBlk + tid) < n) {
                    rank[q] += bin[sub_at(sub[q])];
                    if (exact) ta[rank[q]] = v[q].a;
                }
            __syncthreads();
            if (exact) {
#pragma unroll
                for (int q = 0; q < kSortPer; ++q)
                    if ((uint32_t)(q * kSortBlk + tid) < n) {
                        const uint32_t p0 = bin[sub_at(sub[q])], p1 = bin[sub_at(sub[q] + 1)], mine = rank[q];
                        uint32_t less = 0;
                        for (uint32_t p = p0; p < p1; ++p)
                            less += ta[p] < v[q].a || (ta[p] == v[q].a && p < mine) ? 1u : 0u;
                        rank[q] = p0 + less;
                    }
                __syncthreads();
            }
        }
    }
    // A chunk of a bucket that is merged is read by another workgroup: its stores reach memory by
    // themselves, so its arrival needs no release fence, which would write back the XCD's whole L2
    // (1K x 40M, most buckets of two chunks: 12.3 ms, now 2.8).  R's chunks stay as they are.
    const bool merged = total > (uint32_t)kCap && side == 1;  // uniform
    auto store = [&](auto col, int32_t* out) {
#pragma unroll
        for (int q = 0; q < kSortPer; ++q)
            if ((uint32_t)(q * kSortBlk + tid) < n) ta[rank[q]] = col(v[q]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSortPer; ++q) {
            const uint32_t p = (uint32_t)(q * kSortBlk + tid);
            if (p >= n) continue;
            if (merged) __hip_atomic_store(&out[at + p], ta[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else out[at + p] = ta[p];
        }
        __syncthreads();
    };
    store([](const Row& x) { return x.a; }, s.oa[side]);
    store([](const Row& x) { return x.r; }, s.orid[side]);
    if (HAS_C) store([](const Row& x) { return x.c; }, s.oc[side]);
    if (!merged) return;
    // the last of the bucket's chunks to finish merges them
    drain();
    __syncthreads();
    if (tid == 0)
        last = atomicAdd(&s.zero[2 * s.B + bucket], 1u) == (total - 1) / kCap;
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    merge_chunks<HAS_C>(s, side, b0, total);
}

// ------------------------------------------------------------------------- count and write --
struct Join {
    const int32_t *Ra, *Rc, *Rr, *Sa, *Sc, *Sr;  // sorted columns
    uint32_t nR, nS;
    int op_a;
    int64_t w;
    uint32_t rows;  // R rows per unit (a multiple of kJoinBlk)
    uint32_t U;     // units
    int log_y;      // 2^log_y shares of an R block's work: unit u = R block u >> log_y, share the bits below
    int tiled;      // the shares are S tiles (else equal parts of every interval)
    int direct;     // S is one bucket
    const Hdr* h;
    const uint16_t* lut;
    const uint32_t* baseS;
    uint32_t *lo, *hi;   // each R row's interval
    uint64_t* counts;    // [U] counts, then offsets
    uint64_t* wave_off;  // [U][kJoinWaves] each wave's start inside its unit's range
    uint32_t* done;
    uint64_t* stamp_at;
    uint64_t stamp;
    uint64_t* dbg;
};

// The first position in sorted S whose value is >= x (UP: > x), x the same in the whole wave.
// Buckets rise with the value, so it lies in x's bucket (which takes a search of its own where bins
// hold several buckets: then all of S is searched); there 64 probes at a time cut the range by 64 (two
// dependent loads for 2048 rows, a binary search takes eleven).
template <bool UP>
__device__ __forceinline__ uint32_t wave_bound(const Join& g, const Hdr& h, int32_t x)
{
    uint32_t lo = 0, hi = g.nS;
    if (!g.direct && !h.search) {  // uniform
        const uint32_t b = uniform((uint32_t)g.lut[bin_of(x, h)]);
        lo = uniform(g.baseS[b]);
        hi = uniform(g.baseS[b + 1]);
    }
    while (lo < hi) {
        const uint32_t step = (hi - lo + kWave - 1) / kWave;
        const uint32_t at = lo + (lane_id() + 1) * step - 1;  // the last row of this lane's part
        const int32_t v = g.Sa[at < hi ? at : hi - 1];
        const uint32_t k = (uint32_t)__builtin_popcountll(ballot(at < hi && (UP ? v <= x : v < x)));
        lo += k * step;
        if (step == 1) return lo;
        // the bound lies in part k, or behind the last whole part
        hi = lo + step - 1 < hi ? lo + step - 1 : hi;
    }
    return lo;
}

constexpr uint32_t kWin = 512;  // S values a wave stages for the bounds of its 64 rows

// The first position >= x (UP: > x) of sorted v[0, n), from `first` on.
template <bool UP, typename P>
__device__ __forceinline__ uint32_t lane_bound(P v, uint32_t first, uint32_t n, int32_t x)
{
    uint32_t lo = first, hi = first + n;
    while (lo < hi) {
        const uint32_t m = lo + (hi - lo) / 2;
        const int32_t a = v[m];
        if (UP ? a <= x : a < x) lo = m + 1;
        else hi = m;
    }
    return lo;
}

// The S rows that satisfy op_a with this lane's value a: [lo, hi), or for != everything outside
// it; by the whole wave.  The bounds of neighbouring rows lie close together: the rows of S
// between the wave's smallest and largest one are staged in LDS (win, kWin values of the wave)
// and searched there; too many of them are searched where they are.
__device__ __forceinline__ void interval(const Join& g, const Hdr& h, int32_t a, bool valid, int32_t* win,
                                         uint32_t& lo, uint32_t& hi)
{
    const int64_t w = g.w;  // 0 but for BAND
    const int32_t x0 = (int32_t)max((int64_t)a - w, (int64_t)INT32_MIN);
    const int32_t x1 = (int32_t)min((int64_t)a + w, (int64_t)INT32_MAX);
    const uint32_t w0 = wave_bound<false>(g, h, uniform(wave_min_i(valid ? x0 : INT32_MAX)));
    const uint32_t w1 = wave_bound<true>(g, h, uniform(wave_max_i(valid ? x1 : INT32_MIN)));
    const uint32_t n = w1 > w0 ? w1 - w0 : 0u;
    const bool need_lo = g.op_a != JOIN_OP_GT && g.op_a != JOIN_OP_GE;
    const bool need_hi = g.op_a != JOIN_OP_LT && g.op_a != JOIN_OP_LE;
    const bool up_lo = g.op_a == JOIN_OP_LT, up_hi = g.op_a != JOIN_OP_GT;
    auto bounds = [&](auto v, uint32_t first) {
        lo = 0;
        hi = g.nS;
        if (need_lo) lo = w0 - first + (up_lo ? lane_bound<true>(v, first, n, x0) : lane_bound<false>(v, first, n, x0));
        if (need_hi) hi = w0 - first + (up_hi ? lane_bound<true>(v, first, n, x1) : lane_bound<false>(v, first, n, x1));
    };
    if (n <= kWin) {  // uniform
        for (uint32_t k = lane_id(); k < n; k += kWave) win[k] = g.Sa[w0 + k];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        bounds((const int32_t*)win, 0u);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        bounds(g.Sa, w0);
    }
}

template <int OP>
__device__ __forceinline__ bool holds_c(int32_t r, int32_t s)
{
    if constexpr (OP == JOIN_OP_EQ) return r == s;
    if constexpr (OP == JOIN_OP_NE) return r != s;
    if constexpr (OP == JOIN_OP_LT) return r < s;
    if constexpr (OP == JOIN_OP_LE) return r <= s;
    if constexpr (OP == JOIN_OP_GT) return r > s;
    if constexpr (OP == JOIN_OP_GE) return r >= s;
    return true;
}

__device__ __forceinline__ uint32_t wave_min_u(uint32_t v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o));
    return uniform(v);
}

__device__ __forceinline__ uint32_t wave_max_u(uint32_t v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
    return uniform(v);
}

// How a wave walks long intervals under a condition on c.  By S rows: from the first to the last S
// row of any interval, every lane comparing its own R row; best when the intervals overlap.  By R
// rows: each interval by 64 lanes, four rows' loads in flight; best when R is sparse, and the
// intervals leave gaps or overlap little (1K x 1M, w = 1000: intervals of 125 rows spread over 64K;
// count 3710 us by S rows, 85 by R rows).  A step by R rows has a load's latency for four of them and
// is taken for eight steps by S rows.
constexpr int kRowsAtOnce = 4;

__device__ __forceinline__ bool by_rows(uint32_t len, uint32_t span)
{
    return 8ull * wave_sum64((len + kWave - 1) / kWave) < span;
}

// By R rows: f(x, r, in, v) for kRowsAtOnce R rows at a time (x, r: theirs) and 64 S rows of each
// (v: the lane's, if it has one).
template <typename Load, typename F>
__device__ __forceinline__ void walk_by_rows(int32_t x, int32_t r, uint32_t l, uint32_t len, Load load, F f)
{
    for (int q0 = 0; q0 < kWave; q0 += kRowsAtOnce) {
        uint32_t first[kRowsAtOnce], n[kRowsAtOnce], longest = 0;
#pragma unroll
        for (int i = 0; i < kRowsAtOnce; ++i) {
            n[i] = (uint32_t)__builtin_amdgcn_readlane((int)len, q0 + i);
            first[i] = (uint32_t)__builtin_amdgcn_readlane((int)l, q0 + i);
            longest = max(longest, n[i]);
        }
        for (uint32_t k0 = 0; k0 < longest; k0 += kWave) {
            const uint32_t k = k0 + lane_id();
            decltype(load(0u)) v[kRowsAtOnce];
#pragma unroll
            for (int i = 0; i < kRowsAtOnce; ++i) v[i] = load(k < n[i] ? first[i] + k : 0u);
#pragma unroll
            for (int i = 0; i < kRowsAtOnce; ++i)
                f(__builtin_amdgcn_readlane(x, q0 + i), __builtin_amdgcn_readlane(r, q0 + i), k < n[i], v[i]);
        }
    }
}

// By S rows: f(j, v, k, covered) for the S rows [j0, j1) in turn, and some beyond j1; lane k's v is
// load(j), loaded 64 rows at a time, the next 64 in flight meanwhile.  covered: a constant, true where
// j lies in [i0, i1).  (By a scalar load for a row or eight rows, each waits for its own round trip:
// 1K x 1M, <, count 1320 us, 540 this way.)
template <typename Load, typename F>
__device__ __forceinline__ void walk_by_s(uint32_t j0, uint32_t j1, uint32_t i0, uint32_t i1, Load load, F f)
{
    constexpr uint32_t G = 8;
    auto next = load(min(j0 + lane_id(), j1 - 1));
    for (uint32_t j = j0; j < j1; j += kWave) {
        const auto v = next;
        if (j1 - j > (uint32_t)kWave) next = load(min(j + kWave + lane_id(), j1 - 1));
        const uint32_t n = min(j1 - j, (uint32_t)kWave);
        auto rows = [&](auto covered) {
            for (uint32_t k = 0; k < n; k += G)
#pragma unroll
                for (uint32_t q = 0; q < G; ++q) f(j + k + q, v, k + q, covered);
        };
        if (j >= i0 && j + kWave <= i1) rows(std::true_type{});  // uniform
        else rows(std::false_type{});
    }
}

// Matches of this lane's R row among the S rows [l, h) (l == h: none), by the whole wave; of long
// intervals walked by R rows, the lane's share of the wave's matches.
template <int OPC>
__device__ __forceinline__ uint64_t count_in(const Join& g, int32_t xc, uint32_t l, uint32_t h)
{
    if constexpr (OPC == JOIN_OP_NONE) return h - l;
    const uint32_t len = h - l;
    const uint32_t longest = wave_max_u(len);
    if (longest == 0) return 0;
    uint32_t n = 0;  // an interval holds fewer than 2^32 rows
    if (longest <= kSerial) {
        constexpr uint32_t G = 4;
        for (uint32_t i = 0; i < longest; i += G) {
            int32_t sc[G];
#pragma unroll
            for (uint32_t k = 0; k < G; ++k) sc[k] = g.Sc[i + k < len ? l + i + k : 0u];
#pragma unroll
            for (uint32_t k = 0; k < G; ++k) n += i + k < len && holds_c<OPC>(xc, sc[k]) ? 1u : 0u;
        }
        return n;
    }
    const uint32_t j0 = wave_min_u(len ? l : ~0u), j1 = wave_max_u(len ? h : 0u);
    if (by_rows(len, j1 - j0)) {  // uniform
        uint64_t m = 0;
        walk_by_rows(xc, 0, l, len, [&](uint32_t i) { return g.Sc[i]; },
                     [&](int32_t x, int32_t, bool in, int32_t sc) { m += in && holds_c<OPC>(x, sc) ? 1u : 0u; });
        return m;
    }
    // the S rows in all of the wave's intervals: there nothing but c is compared
    const uint32_t i0 = wave_max_u(len ? l : 0u), i1 = wave_min_u(len ? h : ~0u);
    uint32_t m = 0;
    walk_by_s(j0, j1, i0, i1, [&](uint32_t j) { return g.Sc[j]; }, [&](uint32_t j, int32_t v, uint32_t k, auto covered) {
        const int32_t sc = __builtin_amdgcn_readlane(v, k);
        if constexpr (decltype(covered)::value) m += holds_c<OPC>(xc, sc) ? 1u : 0u;
        else n += j - l < len && holds_c<OPC>(xc, sc) ? 1u : 0u;
    });
    return len ? n + m : n;
}

// The pairs of this lane's R row (row id rr) with the S rows [l, h) from slot `at` on; the wave's
// pairs follow each other, and `at` moves past them.  part / parts: this workgroup's share of
// long intervals without a condition on c.
template <int OPC>
__device__ __forceinline__ void write_in(const Join& g, int32_t xc, int32_t rr, uint32_t l, uint32_t h,
                                         uint64_t& at, int2* __restrict__ out, uint32_t part, uint32_t parts)
{
    const uint32_t len = h - l;
    const uint32_t longest = wave_max_u(len);
    if (longest == 0) return;
    auto emit_of = [&](bool match, int32_t rrid, int32_t srid) {
        const uint64_t m = ballot(match);
        if (match) out[at + mask_rank(m)] = make_int2(rrid, srid);
        at += (uint64_t)__builtin_popcountll(m);
    };
    auto emit = [&](bool match, int32_t srid) { emit_of(match, rr, srid); };
    if (longest <= kSerial) {
        if (OPC == JOIN_OP_NONE && part) {  // uniform: the first workgroup writes short intervals
            at += wave_sum64(len);
            return;
        }
        for (uint32_t i = 0; i < longest; ++i) {
            const bool in = i < len;
            const uint32_t j = in ? l + i : 0u;
            emit(in && (OPC == JOIN_OP_NONE || holds_c<OPC>(xc, g.Sc[j])), g.Sr[j]);
        }
        return;
    }
    if constexpr (OPC == JOIN_OP_NONE) {
        // row by row, each by the whole wave
        for (int q = 0; q < kWave; ++q) {
            const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)len, q);
            const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)l, q);
            const int32_t r = __builtin_amdgcn_readlane(rr, q);
            const uint32_t k1 = (uint32_t)((uint64_t)n * (part + 1) / parts);
            for (uint32_t k = (uint32_t)((uint64_t)n * part / parts) + lane_id(); k < k1; k += kWave)
                out[at + k] = make_int2(r, g.Sr[s0 + k]);
            at += n;
        }
    } else {
        const uint32_t j0 = wave_min_u(len ? l : ~0u), j1 = wave_max_u(len ? h : 0u);
        auto row_of = [&](uint32_t j) { return make_int2(g.Sc[j], g.Sr[j]); };
        if (by_rows(len, j1 - j0)) {  // uniform
            walk_by_rows(xc, rr, l, len, row_of,
                         [&](int32_t x, int32_t r, bool in, int2 s) { emit_of(in && holds_c<OPC>(x, s.x), r, s.y); });
            return;
        }
        walk_by_s(j0, j1, j1, j1, row_of, [&](uint32_t j, int2 v, uint32_t k, auto) {
            emit(j - l < len && holds_c<OPC>(xc, __builtin_amdgcn_readlane(v.x, k)), __builtin_amdgcn_readlane(v.y, k));
        });
    }
}

// Unit u: R rows [r0, r1) and share y of them.
__device__ __forceinline__ void unit_of(const Join& g, uint32_t u, uint32_t& r0, uint32_t& r1, uint32_t& y)
{
    const uint32_t rb = u >> g.log_y;
    y = u - (rb << g.log_y);
    r0 = rb * g.rows;
    r1 = g.nR - r0 < g.rows ? g.nR : r0 + g.rows;
}

// Share y of [0, n).
__device__ __forceinline__ uint32_t share_at(const Join& g, uint32_t n, uint32_t y)
{
    return (uint32_t)((uint64_t)n * y >> g.log_y);
}

// Share y of a row's intervals: f(first, last + 1).  != has the rows before and after its equal
// run, every other operator one interval.  The intervals of =, and of a band, lie where the row's value
// does, so a tile of S would hold few rows' (the shares are parts of the interval); the others'
// reach an end of S, and S rows are best shared by all rows of a wave (the shares are tiles).
template <typename F>
__device__ __forceinline__ void each_interval(const Join& g, uint32_t lo, uint32_t hi, uint32_t y, bool valid, F f)
{
    if (!g.tiled) {  // uniform
        const uint32_t n = valid ? hi - lo : 0u;
        const uint32_t a = share_at(g, n, y), b = share_at(g, n, y + 1);
        f(a < b ? lo + a : 0u, a < b ? lo + b : 0u);
        return;
    }
    const uint32_t t0 = share_at(g, g.nS, y), t1 = share_at(g, g.nS, y + 1);
    auto clip = [&](uint32_t a, uint32_t b) {
        const uint32_t l = max(a, t0), h = min(b, t1);
        const bool some = valid && l < h;
        f(some ? l : 0u, some ? h : 0u);
    };
    if (g.op_a == JOIN_OP_NE) {
        clip(0, lo);
        clip(hi, g.nS);
    } else {
        clip(lo, hi);
    }
}

// Count pass, and by the last workgroup to finish the exclusive scan of the units' counts, the
// total of which goes to *total and to the host's pinned word.
template <int OPC>
__global__ __launch_bounds__(kJoinBlk) void region_count_k(Join g, uint64_t* __restrict__ total, uint64_t* pub)
{
    __shared__ uint64_t wsum[kJoinWaves];
    __shared__ int32_t win[kJoinWaves][kWin];
    __shared__ uint32_t last;
    const int wv = uniform((int32_t)(threadIdx.x / kWave));
    const uint32_t u = blockIdx.x;
    if (u == 0 && threadIdx.x == 0) *g.stamp_at = g.stamp;  // for the write pass
    uint32_t r0, r1, y;
    unit_of(g, u, r0, r1, y);
    Hdr h{};
    if (!g.direct) h = *g.h;
    uint64_t n = 0;
    for (uint32_t i0 = r0; i0 < r1; i0 += kJoinBlk) {
        const uint32_t i = i0 + threadIdx.x;
        const bool valid = i < r1;
        uint32_t lo = 0, hi = 0;
        interval(g, h, g.Ra[valid ? i : r1 - 1], valid, win[wv], lo, hi);
        if (valid && y == 0) {
            g.lo[i] = lo;
            g.hi[i] = hi;
        }
        const int32_t xc = OPC != JOIN_OP_NONE && valid ? g.Rc[i] : 0;
        each_interval(g, lo, hi, y, valid,
                      [&](uint32_t a, uint32_t b) { n += count_in<OPC>(g, xc, a, b); });
    }
    const uint64_t wt = wave_sum64(n);
    if (lane_id() == 0) wsum[wv] = wt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t run = 0;
        for (int w = 0; w < kJoinWaves; ++w) {
            g.wave_off[(uint64_t)u * kJoinWaves + w] = run;
            run += wsum[w];
        }
        store_shared(&g.counts[u], run);
        drain();
        last = arrive_last(g.done, u, g.U);
    }
    __syncthreads();
    if (!last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    uint64_t carry = 0;
    for (uint32_t b0 = 0; b0 < g.U; b0 += kJoinBlk * 8) {
        uint64_t v[8], s = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t i = b0 + threadIdx.x * 8 + k;
            v[k] = i < g.U ? g.counts[i] : 0;
            s += v[k];
        }
        const uint64_t inc = wave_incl_scan64(s);
        if (lane_id() == kWave - 1) wsum[wv] = inc;
        __syncthreads();
        uint64_t run = carry + inc - s;
        for (int w = 0; w < kJoinWaves; ++w) {
            run += w < wv ? wsum[w] : 0;
            carry += wsum[w];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t i = b0 + threadIdx.x * 8 + k;
            if (i < g.U) g.counts[i] = run;
            run += v[k];
        }
    }
    if (threadIdx.x == 0) {
        *total = carry;
        if (pub) publish_total(pub, carry);
    }
}

template <int OPC>
__global__ __launch_bounds__(kJoinBlk) void region_write_k(Join g, const uint64_t* __restrict__ total,
                                                           int2* __restrict__ out, uint64_t cap, uint32_t parts)
{
    // an output too small for the exact count, or a plan other than the count pass's, receives
    // nothing
    if (*total > cap || *g.stamp_at != g.stamp) return;
    const int wv = uniform((int32_t)(threadIdx.x / kWave));
    const uint32_t u = blockIdx.x / parts, part = blockIdx.x - u * parts;
    uint32_t r0, r1, y;
    unit_of(g, u, r0, r1, y);
    uint64_t at = uniform(g.counts[u] + g.wave_off[(uint64_t)u * kJoinWaves + wv]);
#if JL_DEBUG
    const uint64_t at0 = at;
#endif
    for (uint32_t i0 = r0; i0 < r1; i0 += kJoinBlk) {
        const uint32_t i = i0 + threadIdx.x;
        const bool valid = i < r1;
        const uint32_t lo = valid ? g.lo[i] : 0u, hi = valid ? g.hi[i] : 0u;
        const int32_t xc = OPC != JOIN_OP_NONE && valid ? g.Rc[i] : 0;
        const int32_t rr = valid ? g.Rr[i] : 0;
        each_interval(g, lo, hi, y, valid,
                      [&](uint32_t a, uint32_t b) { write_in<OPC>(g, xc, rr, a, b, at, out, part, parts); });
    }
#if JL_DEBUG
    if (g.dbg && part == 0 && lane_id() == 0 && at > at0)
        atomicAdd(reinterpret_cast<unsigned long long*>(&g.dbg[u]), (unsigned long long)(at - at0));
#endif
}

using CountFn = void (*)(Join, uint64_t*, uint64_t*);
using WriteFn = void (*)(Join, const uint64_t*, int2*, uint64_t, uint32_t);

CountFn count_fn(int opc)
{
    switch (opc) {
    case JOIN_OP_NONE: return region_count_k<JOIN_OP_NONE>;
    case JOIN_OP_EQ: return region_count_k<JOIN_OP_EQ>;
    case JOIN_OP_NE: return region_count_k<JOIN_OP_NE>;
    case JOIN_OP_LT: return region_count_k<JOIN_OP_LT>;
    case JOIN_OP_LE: return region_count_k<JOIN_OP_LE>;
    case JOIN_OP_GT: return region_count_k<JOIN_OP_GT>;
    case JOIN_OP_GE: return region_count_k<JOIN_OP_GE>;
    default: return nullptr;
    }
}

WriteFn write_fn(int opc)
{
    switch (opc) {
    case JOIN_OP_NONE: return region_write_k<JOIN_OP_NONE>;
    case JOIN_OP_EQ: return region_write_k<JOIN_OP_EQ>;
    case JOIN_OP_NE: return region_write_k<JOIN_OP_NE>;
    case JOIN_OP_LT: return region_write_k<JOIN_OP_LT>;
    case JOIN_OP_LE: return region_write_k<JOIN_OP_LE>;
    case JOIN_OP_GT: return region_write_k<JOIN_OP_GT>;
    case JOIN_OP_GE: return region_write_k<JOIN_OP_GE>;
    default: return nullptr;
    }
}

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

size_t scatter_lds(int B, bool has_c) { return (size_t)B * 8 + (size_t)kCap * (has_c ? 14 : 10); }

constexpr size_t kSortLds = (size_t)kSubWords * 4 + (size_t)kCap * 4;

}  // namespace

RegionPlan region_plan(int64_t nR, int64_t nS, int op_a, int op_c, int num_cus, int64_t knob)
{
    RegionPlan pl{};
    const int64_t n = nR > nS ? nR : nS;
    const bool has_c = op_a == JOIN_OP_NONE || op_c != JOIN_OP_NONE;
    pl.direct = n <= kCap;
    while (!pl.direct && pl.bits < kMaxBits && (n >> pl.bits) > kMeanRows) ++pl.bits;
    pl.B = 1 << pl.bits;
    pl.binBits = pl.bits + 4 < kMinBinBits ? kMinBinBits : (pl.bits + 4 > kMaxBinBits ? kMaxBinBits : pl.bits + 4);
    pl.samples = (int64_t)16 * pl.B < 4096 ? 4096 : ((int64_t)16 * pl.B > 65536 ? 65536 : (int64_t)16 * pl.B);
    pl.rows = ceil_div(ceil_div(nR > 0 ? nR : 1, kMaxBlocks), kJoinBlk) * kJoinBlk;
    const int64_t blocks = nR > 0 && nS > 0 ? ceil_div(nR, pl.rows) : 0;
    // A condition on c inside intervals of a large share of S is the one thing that costs more
    // than the sort: it is cut into S tiles until there are waves for every SIMD.  The intervals of a
    // band or of equal values may be long as well (w, frequent values), and the R blocks few: cut into
    // parts until there is a unit for every CU (1K x 1M, w = 100,000: count 7460 us whole,
    // 114 in 64 parts).
    pl.tiled = op_a != JOIN_OP_EQ && op_a != JOIN_OP_BAND;
    pl.Y = 1;
    if (has_c)
        while (pl.Y < 64 && blocks * pl.Y < (int64_t)num_cus * (pl.tiled ? 8 : 1) && nS / (2 * pl.Y) >= 256) pl.Y *= 2;
    pl.U = blocks * pl.Y;
    size_t off = 256;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return o;
    };
    pl.zero_words = (size_t)3 * pl.B + kCounters;
    pl.off_zero = take(pl.zero_words * 4);
    pl.off_base = take((size_t)2 * (pl.B + 1) * 4);
    pl.off_cur = take((size_t)2 * pl.B * 4);
    pl.off_extra = take(pl.direct ? 0 : (size_t)(nR / kCap + nS / kCap + 2) * 8);
    pl.off_lut = take(pl.direct ? 0 : ((size_t)2 << pl.binBits) + 4);
    pl.off_split = take(pl.direct ? 0 : (size_t)pl.B * 4);
    pl.off_sample = take(pl.direct ? 0 : (size_t)pl.samples * 8);
    pl.off_id = take(pl.direct ? 0 : (size_t)(nR + nS) * 2);
    const size_t rec = pl.direct ? 0 : (has_c ? 16 : 8);
    pl.off_pR = take((size_t)nR * rec);
    pl.off_pS = take((size_t)nS * rec);
    pl.off_Ra = take((size_t)nR * 4);
    pl.off_Rr = take((size_t)nR * 4);
    pl.off_Rc = take(has_c ? (size_t)nR * 4 : 0);
    pl.off_Sa = take((size_t)nS * 4);
    pl.off_Sr = take((size_t)nS * 4);
    pl.off_Sc = take(has_c ? (size_t)nS * 4 : 0);
    pl.off_lo = take((size_t)nR * 4);
    pl.off_hi = take((size_t)nR * 4);
    pl.off_counts = take((size_t)(pl.U > 0 ? pl.U : 1) * 8);
    pl.off_wave = take((size_t)(pl.U > 0 ? pl.U : 1) * kJoinWaves * 8);
    pl.off_dbg = take(JL_DEBUG ? (size_t)(pl.U > 0 ? pl.U : 1) * 8 : 0);  // last (checking build)
    pl.bytes = off;
    pl.stamp = plan_stamp({JOIN_KIND_THETA_REGION, nR, nS, op_a, op_c, pl.direct, pl.bits, pl.rows, pl.U, pl.Y,
                           knob, (int64_t)pl.bytes});
    return pl;
}

static hipError_t region_attrs()
{
    static bool done = false;
    if (done) return hipSuccess;
    for (const void* f : {(const void*)setup_k, (const void*)sizes_k, (const void*)scatter_rows_k<true>,
                          (const void*)scatter_rows_k<false>, (const void*)sort_k<true>, (const void*)sort_k<false>}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 4096);
        if (e != hipSuccess) return e;
    }
    done = true;
    return hipSuccess;
}

static Join join_of(const RegionPlan& pl, const join_rel_t& R, const join_rel_t& S, const join_pred_t& p, char* ws)
{
    auto i32 = [&](size_t o) { return reinterpret_cast<const int32_t*>(ws + o); };
    Join g{};
    g.Ra = i32(pl.off_Ra);
    g.Rc = i32(pl.off_Rc);
    g.Rr = i32(pl.off_Rr);
    g.Sa = i32(pl.off_Sa);
    g.Sc = i32(pl.off_Sc);
    g.Sr = i32(pl.off_Sr);
    g.nR = (uint32_t)R.n;
    g.nS = (uint32_t)S.n;
    g.op_a = p.op_a;
    g.w = p.op_a == JOIN_OP_BAND ? (int64_t)p.w : 0;
    g.rows = (uint32_t)pl.rows;
    g.U = (uint32_t)pl.U;
    g.log_y = __builtin_ctz((unsigned)pl.Y);
    g.tiled = pl.tiled;
    g.direct = pl.direct;
    g.h = reinterpret_cast<const Hdr*>(ws);
    g.lut = reinterpret_cast<const uint16_t*>(ws + pl.off_lut);
    g.baseS = reinterpret_cast<const uint32_t*>(ws + pl.off_base) + pl.B + 1;
    g.lo = reinterpret_cast<uint32_t*>(ws + pl.off_lo);
    g.hi = reinterpret_cast<uint32_t*>(ws + pl.off_hi);
    g.counts = reinterpret_cast<uint64_t*>(ws + pl.off_counts);
    g.wave_off = reinterpret_cast<uint64_t*>(ws + pl.off_wave);
    g.done = reinterpret_cast<uint32_t*>(ws + pl.off_zero) + 3 * pl.B + kCntCount;
    g.stamp_at = reinterpret_cast<uint64_t*>(ws + kStampOffset);
    g.stamp = pl.stamp;
    g.dbg = JL_DEBUG ? reinterpret_cast<uint64_t*>(ws + pl.off_dbg) : nullptr;
    return g;
}

hipError_t region_count(const RegionPlan& pl, const join_rel_t& R, const join_rel_t& S,
                        const join_pred_t& p, char* ws, hipStream_t st, uint64_t* pub)
{
    hipError_t e = region_attrs();
    if (e != hipSuccess) return e;
    const bool has_c = p.op_c != JOIN_OP_NONE;
    auto i32 = [&](size_t o) { return reinterpret_cast<int32_t*>(ws + o); };
    Sides s{};
    s.X[0] = Cols{R.key, has_c ? R.key2 : nullptr, R.rid, R.n};
    s.X[1] = Cols{S.key, has_c ? S.key2 : nullptr, S.rid, S.n};
    s.h = reinterpret_cast<const Hdr*>(ws);
    s.lut = reinterpret_cast<const uint16_t*>(ws + pl.off_lut);
    s.splitters = reinterpret_cast<const int32_t*>(ws + pl.off_split);
    s.B = pl.B;
    s.zero = reinterpret_cast<uint32_t*>(ws + pl.off_zero);
    s.base = reinterpret_cast<uint32_t*>(ws + pl.off_base);
    s.cur = reinterpret_cast<uint32_t*>(ws + pl.off_cur);
    s.extra = reinterpret_cast<uint2*>(ws + pl.off_extra);
    s.id[0] = reinterpret_cast<uint16_t*>(ws + pl.off_id);
    s.id[1] = s.id[0] + R.n;
    s.part[0] = ws + pl.off_pR;
    s.part[1] = ws + pl.off_pS;
    s.oa[0] = i32(pl.off_Ra);
    s.oa[1] = i32(pl.off_Sa);
    s.oc[0] = i32(pl.off_Rc);
    s.oc[1] = i32(pl.off_Sc);
    s.orid[0] = i32(pl.off_Rr);
    s.orid[1] = i32(pl.off_Sr);
    if (!pl.direct) {
        {
            prof::Scope ps(st, "region.bucket");
            const uint32_t sR = (uint32_t)(R.n < pl.samples ? R.n : pl.samples);
            const uint32_t sS = (uint32_t)(S.n < pl.samples ? S.n : pl.samples);
            int32_t* sample = reinterpret_cast<int32_t*>(ws + pl.off_sample);
            sample_k<<<(unsigned)ceil_div(sR + sS, kBlk), kBlk, 0, st>>>(s.X[0], s.X[1], sR, sS, sample, s.zero,
                                                                       (uint32_t)pl.zero_words);
            const size_t words = padded<kMaxBinBits - 10>(1u << pl.binBits);
            setup_k<<<1, kBlk, 4 * (words > kSplitSample ? words : kSplitSample), st>>>(
                sample, sR + sS, pl.binBits, pl.bits, reinterpret_cast<Hdr*>(ws),
                reinterpret_cast<uint16_t*>(ws + pl.off_lut), reinterpret_cast<int32_t*>(ws + pl.off_split));
            // a workgroup per two CUs' worth of rows, whole tiles: its B counters are flushed once
            s.chunk = ceil_div(ceil_div(R.n + S.n, 512), kCap) * kCap;
            s.split = (uint32_t)ceil_div(R.n, s.chunk);
            sizes_k<<<(unsigned)(s.split + ceil_div(S.n, s.chunk)), kBlk, ((size_t)pl.B * 4) + ((size_t)2 << pl.binBits) + 4, st>>>(s);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        s.split = (uint32_t)ceil_div(R.n, kCap);
        const unsigned tiles = (unsigned)(s.split + ceil_div(S.n, kCap));
        prof::Scope ps(st, "region.partition");
        if (has_c) scatter_rows_k<true><<<tiles, kBlk, scatter_lds(pl.B, true), st>>>(s);
        else scatter_rows_k<false><<<tiles, kBlk, scatter_lds(pl.B, false), st>>>(s);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    {
        prof::Scope ps(st, "region.sort");
        const unsigned grid = pl.direct ? 2u : (unsigned)(2 * pl.B + R.n / kCap + S.n / kCap);
        if (has_c) sort_k<true><<<grid, kSortBlk, kSortLds, st>>>(s, pl.direct);
        else sort_k<false><<<grid, kSortBlk, kSortLds, st>>>(s, pl.direct);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    CountFn f = count_fn(p.op_c);
    if (!f) return hipErrorInvalidValue;
    prof::Scope ps(st, "region.count");
    hipLaunchKernelGGL(f, dim3((unsigned)pl.U), dim3(kJoinBlk), 0, st, join_of(pl, R, S, p, ws),
                       reinterpret_cast<uint64_t*>(ws), pub);
    return hipGetLastError();
}

hipError_t region_write(const RegionPlan& pl, const join_rel_t& R, const join_rel_t& S,
                        const join_pred_t& p, char* ws, int32_t* pairs, uint64_t cap,
                        hipStream_t st)
{
    WriteFn f = write_fn(p.op_c);
    if (!f) return hipErrorInvalidValue;
    // Long intervals without a condition on c are shared by several workgroups per R block when
    // the R blocks alone leave the chip idle: one for every 256 pairs a row, up to 64.
    uint32_t parts = 1;
    if (p.op_c == JOIN_OP_NONE)
        while (parts < 64 && pl.U * parts < 2048 && cap / (uint64_t)R.n >= (uint64_t)512 * parts) parts *= 2;
    prof::Scope ps(st, "region.write");
    hipLaunchKernelGGL(f, dim3((unsigned)pl.U * parts), dim3(kJoinBlk), 0, st, join_of(pl, R, S, p, ws),
                       reinterpret_cast<const uint64_t*>(ws), reinterpret_cast<int2*>(pairs), cap, parts);
    return hipGetLastError();
}

}  // namespace jl
