// Offline bias calibration on the GPU (Alg. 2 of the paper, "Greedy Bias
// Calibration"; App. A "Greedy threshold selection"), from given damage weights
// w [D][T] and proxy scores s [D][T].
//
// The printed algorithm is a loop over a priority queue: pop the neuron whose
// next eta samples cost least, advance its pointer, push its next cost, until
// enough (neuron, sample) pairs are dropped.  That order has a closed form: a
// neuron's steps leave the queue in the order of the RUNNING MAXIMUM of its step
// costs (a step cheaper than its predecessor is taken right after it), so the
// whole sequence is all steps sorted by (running-max cost, neuron, step).  Two
// kernels follow from it:
//   k_calib_sort   one block per neuron: the samples from the first positive weight
//                  on (in the order by score, ties by sample index) are sorted
//                  in LDS by buckets, the ones below only counted; step costs (fp32, left
//                  to right), their running maxima, and for every step the
//                  number of dropped samples and the threshold it would set;
//                  optionally the Kendall check of App. A.
//   k_select_*     the cost level at which the required number of pairs is first
//                  reached, by a radix select over the keys' bit patterns
//                  (four digit launches, integer atomics); then the steps at
//                  exactly that level are taken in neuron order, and b = -tau
//                  and the pointers written.
// Integer results equal the sequential algorithm's bit for bit.
#pragma once

#include "svdp_device.h"

namespace svdp {

constexpr int CAL_THREADS = 256;
constexpr int CAL_MAX_T = 4096;

// order-preserving map float -> uint32 (-0 and +0 coincide; inputs are not NaN)
__device__ __forceinline__ uint32_t ordered_bits(float v)
{
    uint32_t u = __float_as_uint(v == 0.f ? 0.f : v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t u)
{
    return __uint_as_float((u & 0x80000000u) ? u ^ 0x80000000u : ~u);
}

// Per-neuron tables written by k_calib_sort, MS = ceil(T / eta) steps at most:
//   key  [D][MS]     running maximum of the step costs, +inf beyond the neuron's last step
//   drop [D][MS + 1] number of samples with s <= tau after 0, 1, 2, ... steps
//   tauc [D][MS + 1] the threshold after 0, 1, 2, ... steps
//   k0   [D]         the starting pointer (1-based count)
//   drop0[D]         drop[.][0] once more, side by side (16 bits: T <= CAL_MAX_T)
// Only the part of the order that the algorithm walks is sorted: everything below the first sample
// with a positive weight (in the order by score, then sample index) is merely counted -- those
// samples have zero weight and are dropped from the start -- and the rest, the "tail", typically a
// tenth to a third of the samples of a sparse layer, is sorted by score, then sample index.
// Bound: the dependent phases of a block (barriers, LDS round trips, two trips to memory), not the 16 KB a neuron reads.
// A bitonic network takes 55 steps with a barrier each at 1024 keys.  Instead a sample's bucket is a linear function of its
// score between the tail's ends (monotone in fp32 too), a counting pass gives the buckets' places, and inside a bucket (one
// to three samples on the scores of a layer) a sample's rank is the number of smaller keys: the number of barriers does not
// depend on the length.  A bucket of more than CAL_BUCKET_MAX samples (many equal scores, an outlier that leaves everybody
// else in one bucket, an infinite score) sends the neuron to the network, whose 55 to 78 stages cost more than counting 256 keys
// of a bucket does: whole call at D = 11008, eta = 16, limit 32 with twice the buckets / 32 / 256 / network for every neuron,
// in us, T = 2048 and T = 4096:
//   Gaussian                                   168 / 165 / 167 / 640       432 / 385 / 385 / 1960
//   Student t, 4 degrees of freedom            231 / 287 / 191 / 643       626 / 958 / 472 / 1961
//   Gaussian, token scale log-normal (0.6)     231 / 392 / 184 / 647       540 / 1140 / 446 / 1959
//   one outlier at 20 times the spread         244 / 656 / 210 / 655       650 / 1897 / 527 / 1970
//   one outlier at 10 times the spread         180 / 235 / 183 / 652       482 / 584 / 447 / 1969
// Scores of a 90 %-sparse layer (139 us) with one huge outlier per neuron 362 us, on a grid of quarters 267, all equal 711.
// Measured at D = 11008, T = 2048, eta = 16: network 450 us, buckets 131 us (512 threads, 64-bit reductions), 117 us with
// the sorted tail in the keys' place (four blocks a compute unit instead of three), 91 us with 256 threads, reductions on
// the scores alone and the ranks taken by tail position (660 -> 370 vector instructions a wave, half the waves); with 512
// instead of 1024 buckets and a bucket's count and place in one word, so that eight blocks share a compute unit instead of
// six, from memory instead of the cache 101 -> 92 us (D = 18944, T = 4096, eta = 1, whole call: 2915 -> 2144).
// Scores and weights are read once and stay in registers, PER of each per thread (T <= PER * CAL_THREADS).
// Dynamic LDS: calib_sort_lds().
constexpr int CAL_BUCKET_MAX = 256;
// As many as eight blocks' local memory has room for.  For T <= 512 no more, because clearing and adding up 1024 shows there
// (0.5 to 1 us of 100); against 512 at T = 1000, D = 18944, outlier at 40 times the spread 249 -> 229 us, Student t, 3 degrees
// of freedom 222 -> 208.
template <int PER>
constexpr int cal_buckets() { return PER == 2 || PER == 8 ? 512 : 1024; }

// sort keys (n2 = T rounded up to a power of two), later the sorted tail (s, w) in their place; costs and their running
// maxima; buckets.  19.5 KB at T = 2048, eta = 16: eight blocks a compute unit, as many as it has wave slots for.
template <int PER>
size_t calib_sort_lds(int n2, int MS)
{
    return (size_t)n2 * 8 + (size_t)(MS + 1) * 8 + (size_t)cal_buckets<PER>() * 4;
}

template <int PER>
__global__ __launch_bounds__(CAL_THREADS) void k_calib_sort(const float *__restrict__ w, const float *__restrict__ s,
                                                            int T, int n2max, int eta, int MS,
                                                            float *__restrict__ key, int32_t *__restrict__ drop,
                                                            float *__restrict__ tauc, int32_t *__restrict__ k0_out,
                                                            uint16_t *__restrict__ drop0, float *__restrict__ kendall,
                                                            uint32_t *__restrict__ clear0, int n_clear0,
                                                            uint32_t *__restrict__ clear1, int32_t *__restrict__ clear2)
{
    constexpr int NBK = cal_buckets<PER>(), BPT = NBK / CAL_THREADS, WAVES = CAL_THREADS / 64;
    extern __shared__ unsigned long long smem64[];
    unsigned long long *sk = smem64;                               // [n2max] (score, sample) of the tail
    float *ss = reinterpret_cast<float *>(sk);                     // [n2max] scores of the tail, sorted
    float *ww = ss + n2max;                                        // [n2max] weights in that order
    float *cost = ww + n2max;                                      // [MS + 1]
    float *scan = cost + (MS + 1);                                 // [MS + 1]
    // [NBK] samples of a bucket, and from the scan on, in the upper half, samples in front of it (T <= CAL_MAX_T < 2^16)
    uint32_t *bucket = reinterpret_cast<uint32_t *>(scan + (MS + 1));
    __shared__ float lo_w[WAVES], hi_w[WAVES];
    __shared__ int wave_tot[WAVES], first_sh, big_sh, kd_total;
    __shared__ unsigned long long last_sh;
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *si = s + (size_t)i * T, *wi = w + (size_t)i * T;
    auto key_of = [&](float v, int t) { return ((unsigned long long)ordered_bits(v) << 32) | (unsigned)t; };

    // samples beyond the last: a score below all, no weight
    float sv[PER], wv[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int t = tid + q * CAL_THREADS;
        sv[q] = t < T ? si[t] : -__builtin_inff();
        wv[q] = t < T ? wi[t] : 0.f;
    }
    if (tid == 0) {
        first_sh = T;
        big_sh = 0;
        kd_total = 0;
        last_sh = 0ull;
    }
#pragma unroll
    for (int q = 0; q < BPT; ++q) bucket[tid + q * CAL_THREADS] = 0u;
    // the smallest score with a positive weight (+inf if there is none), the largest score
    float s_lo = __builtin_inff(), s_hi = -__builtin_inff();
    bool some = false;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        s_lo = wv[q] > 0.f ? fminf(s_lo, sv[q]) : s_lo;
        some = some || wv[q] > 0.f;
        s_hi = fmaxf(s_hi, sv[q]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s_lo = fminf(s_lo, __shfl_xor(s_lo, off));
        s_hi = fmaxf(s_hi, __shfl_xor(s_hi, off));
    }
    if (lane == 0) {
        lo_w[wave] = s_lo;
        hi_w[wave] = s_hi;
    }
    const bool any = __syncthreads_or(some ? 1 : 0) != 0;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
        s_lo = fminf(s_lo, lo_w[v]);
        s_hi = fmaxf(s_hi, hi_w[v]);
    }
    // where the tail begins among equal scores: the first sample with that score and a positive weight
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (wv[q] > 0.f && sv[q] == s_lo) atomicMin(&first_sh, tid + q * CAL_THREADS);
    __syncthreads();
    const int first = first_sh;
    // the tail: samples at or above the first positive one, into buckets; the rest is counted
    const float range = s_hi - s_lo, scale = range > 0.f && range <= 3.4e38f && NBK / range <= 3.4e38f ? NBK / range : 0.f;
    auto bucket_of = [&](float v) { return scale > 0.f ? max(0, min((int)((v - s_lo) * scale), NBK - 1)) : 0; };
    int pos[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int t = tid + q * CAL_THREADS;
        pos[q] = -1;
        if (any && t < T && (sv[q] > s_lo || (sv[q] == s_lo && t >= first))) pos[q] = (int)atomicAdd(&bucket[bucket_of(sv[q])], 1u);
    }
    __syncthreads();
    int ntail = 0;
    {
        uint32_t h[BPT], most = 0u;
        int sum = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            h[q] = bucket[tid * BPT + q];
            most = h[q] > most ? h[q] : most;
            sum += (int)h[q];
        }
        if (most > CAL_BUCKET_MAX) big_sh = 1;
        int inc = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        int before = inc - sum;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            if (v < wave) before += wave_tot[v];
            ntail += wave_tot[v];
        }
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            bucket[tid * BPT + q] = ((uint32_t)before << 16) | h[q];
            before += (int)h[q];
        }
    }
    const int nb = T - ntail;                                      // samples below the tail (T if no weight is positive)
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (pos[q] >= 0) sk[(bucket[bucket_of(sv[q])] >> 16) + pos[q]] = key_of(sv[q], tid + q * CAL_THREADS);
    __syncthreads();
    if (big_sh != 0) {
        int n2 = 1;
        while (n2 < ntail) n2 <<= 1;
        for (int t = ntail + tid; t < n2; t += CAL_THREADS) sk[t] = ~0ull;
        __syncthreads();
        for (int k = 2; k <= n2; k <<= 1) {
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int t = tid; t < n2; t += CAL_THREADS) {
                    const int p = t ^ j;
                    if (p > t) {
                        const unsigned long long a = sk[t], b = sk[p];
                        const bool up = (t & k) == 0;
                        if ((a > b) == up) {
                            sk[t] = b;
                            sk[p] = a;
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
    // tail sample p (by bucket, or sorted already): its score, weight and place; then the keys make room
    float tw[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int p = tid + q * CAL_THREADS;
        pos[q] = -1;
        if (p < ntail) {
            const unsigned long long k = sk[p];
            const int t = (int)(k & 0xffffffffu);
            tw[q] = wi[t];
            sv[q] = si[t];                                         // not from the key: -0 keeps its sign
            pos[q] = p;
            if (big_sh == 0) {
                const uint32_t bk = bucket[bucket_of(from_ordered_bits((uint32_t)(k >> 32)))];
                const int b0 = (int)(bk >> 16), b1 = b0 + (int)(bk & 0xffffu);
                int rank = b0;
                for (int e = b0; e < b1; ++e) rank += sk[e] < k ? 1 : 0;
                pos[q] = rank;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (pos[q] < 0) continue;
        ss[pos[q]] = sv[q];
        ww[pos[q]] = tw[q];
    }
    if (ntail == 0) {                                              // nothing ever active: the last sample in sorted order
        unsigned long long last = 0ull;
        for (int t = tid; t < T; t += CAL_THREADS) {
            const unsigned long long k = key_of(si[t], t);
            last = k > last ? k : last;
        }
        atomicMax(&last_sh, last);
    }
    __syncthreads();
    // sorted position q of the whole sample = tail position q - nb; the first positive weight is tail position 0
    const int k0 = ntail > 0 ? nb + 1 : T;                         // min{k : w_(k) > 0}, or T if there is none
    const int M = (T - k0 + eta - 1) / eta;                        // steps this neuron can take

    // step costs C(k + eta) - C(k), fp32 left to right; the last step may be short (the listing's padding)
    for (int j = tid; j < M; j += CAL_THREADS) {
        const int lo = k0 - nb + j * eta, hi = min(lo + eta, ntail);
        float c = 0.f;
        int p = lo;
        for (; p + 4 <= hi; p += 4) {                               // four reads on their way, added in order
            const float a0 = ww[p], a1 = ww[p + 1], a2 = ww[p + 2], a3 = ww[p + 3];
            c += a0;
            c += a1;
            c += a2;
            c += a3;
        }
        for (; p < hi; ++p) c += ww[p];
        cost[j] = c;
    }
    __syncthreads();
    // running maximum (inclusive): one wave, consecutive steps per lane, then across the lanes
    if (wave == 0) {
        const int per = (M + 63) >> 6, j0 = min(lane * per, M), j1 = min(j0 + per, M);
        float m = -__builtin_inff();
        for (int j = j0; j < j1; ++j) m = fmaxf(m, cost[j]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const float o = __shfl_up(m, off);
            if (lane >= off) m = fmaxf(m, o);
        }
        float run = __shfl_up(m, 1);
        if (lane == 0) run = -__builtin_inff();
        for (int j = j0; j < j1; ++j) {
            run = fmaxf(run, cost[j]);
            scan[j] = run > -__builtin_inff() ? run : cost[j];      // nothing but NaN so far stays that
        }
    }
    __syncthreads();
    for (int j = tid; j < MS; j += CAL_THREADS) key[(size_t)i * MS + j] = j < M ? scan[j] : __builtin_inff();
    // thresholds and dropped counts after j steps: k = min(k0 + j*eta, T), tau = s_(k), #{s <= tau};
    // every sample below the tail has a score <= tau
    for (int j = tid; j <= MS; j += CAL_THREADS) {
        int dj = 0;
        float tj = 0.f;
        if (j <= M) {
            if (ntail == 0) {                                       // nothing ever active: all dropped, tau = the last score
                tj = si[(int)(last_sh & 0xffffffffu)];
                dj = T;
            } else {
                const int k = min(k0 + j * eta, T) - nb;            // tail count, >= 1
                tj = ss[k - 1];
                int lo = k, hi = ntail;                             // first tail position whose score exceeds tau
                if (lo < hi && !(ss[lo] <= tj)) hi = lo;            // mostly the next one
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (ss[mid] <= tj) lo = mid + 1;
                    else hi = mid;
                }
                dj = nb + lo;
            }
        }
        drop[(size_t)i * (MS + 1) + j] = dj;
        tauc[(size_t)i * (MS + 1) + j] = tj;
        if (j == 0) drop0[i] = (uint16_t)dj;
    }
    if (tid == 0) k0_out[i] = k0;
    if (i == 0) {                                                  // what the selection counts in
        for (int q = tid; q < n_clear0; q += CAL_THREADS) clear0[q] = 0u;
        if (tid == 0) {
            *clear1 = 0u;
            if (clear2 != nullptr) *clear2 = 0;
        }
    }

    if (kendall != nullptr) {
        // App. A: non-overlapping eta-step sums over the whole sorted sample (zero below the tail),
        // discordant pairs m1 < m2
        const int MK = T / eta;
        __syncthreads();                                            // cost/scan are free again
        float *S = cost;                                            // MK <= MS entries
        for (int m = tid; m < MK; m += CAL_THREADS) {
            float c = 0.f;
            for (int q = max(m * eta, nb); q < (m + 1) * eta; ++q) c += ww[q - nb];
            S[m] = c;
        }
        __syncthreads();
        int kd = 0;
        for (int m1 = tid; m1 < MK; m1 += CAL_THREADS) {
            const float a = S[m1];
            for (int m2 = m1 + 1; m2 < MK; ++m2) kd += a > S[m2] ? 1 : 0;
        }
        if (kd) atomicAdd(&kd_total, kd);
        __syncthreads();
        if (tid == 0) kendall[i] = MK < 2 ? 1.f : (float)(1.0 - (double)kd_total / ((double)MK * (MK - 1)));
    }
}

// Block-wide sum of a 64-bit count (every thread gets the result).
__device__ __forceinline__ long long block_sum_i64(long long v, long long *red)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    long long t = 0;
    for (int q = 0; q < (int)blockDim.x / 64; ++q) t += red[q];
    return t;
}

// Number of steps of a neuron whose key is <= level (INCLUSIVE) or < level (keys are non-decreasing; +inf pads).
template <bool INCLUSIVE>
__device__ __forceinline__ int steps_below(const float *__restrict__ key_i, int MS, float level)
{
    int lo = 0, hi = MS;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const float v = key_i[mid];
        if (INCLUSIVE ? v <= level : v < level) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The cost level at which the required number of pairs is first reached is found by a radix
// select over the bit patterns of the (non-negative) keys, most significant digit first: the pairs a
// step adds (its gain) are summed per digit value among the steps that match the digits found so
// far, and the digit is where the running sum first covers what is still missing.  Integer atomics
// only, so the result does not depend on the order of arrival.
//
// A digit is one launch: every block works out the digit before from that one's counts (a wave, 256 counts) and adds its
// gains to the other of two count buffers; the block that is last to have read a buffer clears it for the next digit but
// one.  Bound: the launches.  With a launch for every choice of a digit and one for the start (11 launches behind the sort
// instead of 7), whole call: D = 1344, T = 1423, eta = 23 50.2 -> 38.0 us, D = 5312, T = 77, eta = 22 51.3 -> 43.8, D = 11008,
// T = 2048, eta = 16 159.8 -> 157.4 (working a digit out costs a counting launch 3 us of the 4.9 that it saves).
struct SelectState {
    long long missing;       // pairs still to be found among steps at or above the current prefix
    long long c0;            // pairs dropped before any step
    uint32_t prefix;         // digits of the level found so far
    int32_t reachable;       // 0: the start already meets the target, or all finite steps together do not
    int32_t at_start;        // 1: the start already meets the target (no step is taken)
};
constexpr int SEL_BINS = 256;
constexpr int SEL_STATES = 5;                  // the start, then the state behind each digit
constexpr uint32_t SEL_TOP = 0x7f7fffffu;      // largest finite float: keys above it are padding
// The states and the counter of the blocks that have read a buffer: what the workspace keeps for the selection.
struct SelectWork {
    SelectState state[SEL_STATES];
    uint32_t readers;
};

// The state behind the digit whose counts are given (all 64 lanes of a wave; lane l owns bins 4l .. 4l+3).
template <typename Bin>
__device__ __forceinline__ SelectState select_pick(const SelectState &in, const Bin *__restrict__ counts, int shift)
{
    SelectState out = in;
    const int lane = threadIdx.x & 63;
    long long h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = (long long)counts[4 * lane + q];
    const long long missing = in.missing;
    const long long mine = h[0] + h[1] + h[2] + h[3];
    long long inc = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const long long o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
    const long long before = inc - mine;
    const unsigned long long who = __ballot(before < missing && inc >= missing);      // at most one lane
    if (in.reachable == 0) return out;
    if (who == 0ull) {                          // only on the first digit: every finite step together falls short
        out.reachable = 0;
        return out;
    }
    long long run = before;
    int digit = 0;
    for (int q = 0; q < 4; ++q) {
        if (run + h[q] >= missing) {
            digit = 4 * lane + q;
            break;
        }
        run += h[q];
    }
    const int src = __ffsll(who) - 1;
    out.missing = __shfl(missing - run, src);   // still to be found among the steps with this digit
    out.prefix |= (uint32_t)__shfl(digit, src) << shift;
    return out;
}

__device__ __forceinline__ void select_add(long long *at, long long v)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(at), (unsigned long long)v);
}
__device__ __forceinline__ void select_add(uint32_t *at, long long v) { atomicAdd(at, (uint32_t)v); }

// counts[digit] += gain over the steps whose key matches the prefix above this digit.  A thread takes SEL_RUN steps in a
// row: a neuron's keys do not decrease, so they share few digits and most gains are added before they reach the (then
// contended) counters.
// FIRST: no digit is known.  Every block adds up drop0, 16 bits a neuron, while its first keys are on their way, and counts
// nothing where the start meets the target already (a level below the share of zero weights); the first one sets the start
// state and clears the other buffer.  Against one more block that adds up drop0 beside the counting, whole call in us, target
// met: D = 18944, T = 1000, eta = 1 241 -> 159, D = 12544, T = 214, eta = 2 77.6 -> 64.3, D = 18944, T = 64, eta = 1 97 -> 78; steps
// to take: D = 11008, T = 2048, eta = 16 148.2 -> 146.5, D = 6000, T = 800, eta = 1 142 -> 144.  (Every block a part of drop0, and no more
// counting once all parts show it: 179, 78 and 99, and 149 and 147 with steps to take.)
// Otherwise the digit before is worked out from `last` first, while the first keys are on their way.
constexpr int SEL_RUN = 8;
template <int SHIFT, int BITS, int LAST_SHIFT, typename Bin>
__global__ __launch_bounds__(256) void k_select_hist(const float *__restrict__ key, const int32_t *__restrict__ drop,
                                                     const uint16_t *__restrict__ drop0, int D, int MS, long long need,
                                                     int which, SelectWork *__restrict__ work, Bin *__restrict__ last,
                                                     Bin *__restrict__ counts)
{
    constexpr bool FIRST = LAST_SHIFT < 0;
    __shared__ Bin lh[SEL_BINS];
    __shared__ long long red[4];
    __shared__ SelectState now;
    __shared__ uint32_t arrived;
    const int tid = threadIdx.x;
    const int blocks = gridDim.x;
    const size_t total = (size_t)D * MS, stride = (size_t)blocks * 256 * SEL_RUN;
    size_t e0 = ((size_t)blockIdx.x * 256 + tid) * SEL_RUN;
    uint32_t kb[SEL_RUN];
    auto request = [&](size_t e) {
#pragma unroll
        for (int q = 0; q < SEL_RUN; ++q) kb[q] = e + q < total ? __float_as_uint(key[e + q]) : ~0u;
    };
    request(e0);                                // on their way while the digit before is worked out
    lh[tid] = 0;
    if (FIRST) {
        const uint4 *v = reinterpret_cast<const uint4 *>(drop0);
        const int nvec = D / 8;
        constexpr int AHEAD = 8;
        long long c0 = tid < D % 8 ? drop0[nvec * 8 + tid] : 0;
        for (int g0 = tid; g0 < nvec; g0 += 256 * AHEAD) {
            uint4 r[AHEAD];
            uint32_t sum = 0u;
#pragma unroll
            for (int q = 0; q < AHEAD; ++q) r[q] = g0 + q * 256 < nvec ? v[g0 + q * 256] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int q = 0; q < AHEAD; ++q)
                sum += (r[q].x & 0xffffu) + (r[q].x >> 16) + (r[q].y & 0xffffu) + (r[q].y >> 16) + (r[q].z & 0xffffu) +
                       (r[q].z >> 16) + (r[q].w & 0xffffu) + (r[q].w >> 16);
            c0 += sum;
        }
        c0 = block_sum_i64(c0, red);
        if (blockIdx.x == 0) {
            last[tid] = 0;                      // the buffer of the second digit
            if (tid == 0) {
                SelectState st;
                st.c0 = c0;
                st.missing = need - c0;
                st.prefix = 0u;
                st.reachable = c0 < need ? 1 : 0;
                st.at_start = c0 < need ? 0 : 1;
                work->state[0] = st;
            }
        }
        if (c0 >= need) return;                 // in every block
    }
    if (!FIRST && tid < 64) {
        const SelectState st = select_pick<Bin>(work->state[which], last, LAST_SHIFT);
        if (tid == 0) {
            now = st;
            if (blockIdx.x == 0) work->state[which + 1] = st;
        }
    }
    __syncthreads();
    const uint32_t prefix = FIRST ? 0u : now.prefix;
    if (!FIRST && now.reachable == 0) return;   // in every block
    uint32_t order = 0u;
    if (!FIRST && tid == 0) order = atomicAdd(&work->readers, 1u);
    int i0 = (int)(e0 / MS), j0 = (int)(e0 % MS);                     // neuron and step of e0
    const int di0 = (int)(stride / MS), dj0 = (int)(stride % MS);
    while (e0 < total) {
        int i = i0, j = j0;
        long long gain = 0;
        int digit = -1;
#pragma unroll
        for (int q = 0; q < SEL_RUN; ++q) {
            if (kb[q] <= SEL_TOP &&
                !(SHIFT + BITS < 31 && (kb[q] >> (SHIFT + BITS)) != (prefix >> (SHIFT + BITS)))) {
                const int dg = (int)((kb[q] >> SHIFT) & ((1u << BITS) - 1u));
                if (dg != digit) {
                    if (gain != 0) select_add(&lh[digit], gain);
                    gain = 0;
                    digit = dg;
                }
                const int32_t *di = drop + (size_t)i * (MS + 1);
                gain += (long long)di[j + 1] - di[j];
            }
            if (++j == MS) {
                j = 0;
                ++i;
            }
        }
        if (gain != 0) select_add(&lh[digit], gain);
        e0 += stride;
        i0 += di0;
        j0 += dj0;
        if (j0 >= MS) {
            j0 -= MS;
            ++i0;
        }
        if (e0 < total) request(e0);
    }
    if (!FIRST && tid == 0) arrived = order;
    __syncthreads();
    if (lh[tid] != 0) select_add(&counts[tid], (long long)lh[tid]);
    if (!FIRST && arrived == (uint32_t)blocks - 1u) {                 // every block has read `last`
        last[tid] = 0;
        if (tid == 0) work->readers = 0u;
    }
}

// The last digit.  One wave.
template <typename Bin>
__global__ __launch_bounds__(64) void k_select_last(SelectWork *__restrict__ work, const Bin *__restrict__ counts)
{
    const SelectState st = select_pick<Bin>(work->state[SEL_STATES - 2], counts, 0);
    if (threadIdx.x == 0) work->state[SEL_STATES - 1] = st;
}

// With the level known, per neuron: the number of its steps strictly below the level and up to it, and (reachable target)
// how many pairs the latter add; per block the sum of those.  A block has `chunk` neurons, a multiple of 256.
__global__ __launch_bounds__(256) void k_select_bounds(const float *__restrict__ key, const int32_t *__restrict__ drop, int D,
                                                       int MS, int chunk, const SelectState *__restrict__ st,
                                                       int32_t *__restrict__ lo_out, int32_t *__restrict__ up_out,
                                                       long long *__restrict__ block_gain)
{
    __shared__ long long red[4];
    const float lv = __uint_as_float(st->reachable != 0 ? st->prefix : SEL_TOP);
    long long gain = 0;
    for (int i = blockIdx.x * chunk + threadIdx.x; i < min(D, (int)(blockIdx.x + 1) * chunk); i += 256) {
        const float *ki = key + (size_t)i * MS;
        const int32_t *di = drop + (size_t)i * (MS + 1);
        const int lo = steps_below<false>(ki, MS, lv), up = steps_below<true>(ki, MS, lv);
        lo_out[i] = lo;
        up_out[i] = up;
        gain += (long long)di[up] - di[lo];
    }
    gain = block_sum_i64(gain, red);
    if (threadIdx.x == 0) block_gain[blockIdx.x] = gain;
}

// Steps strictly below the level are all taken; those at the level in neuron order until the
// missing pairs are found; writes b = -tau, the pointers and the number of steps.  Every block adds up the gains in front
// of its own 256 neurons, so that no block waits for another (in one block, neuron by neuron behind two dependent loads,
// this took 30 us at D = 11008).
__global__ __launch_bounds__(256) void k_select_finish(const int32_t *__restrict__ lo_in, const int32_t *__restrict__ up_in,
                                                       const int32_t *__restrict__ drop, const float *__restrict__ tauc,
                                                       const int32_t *__restrict__ k0, int D, int T, int eta, int MS,
                                                       int chunk, const SelectState *__restrict__ st,
                                                       const long long *__restrict__ block_gain, float *__restrict__ b,
                                                       int32_t *__restrict__ k_out, int32_t *__restrict__ steps)
{
    __shared__ long long red[4], wave_tot[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool at_start = st->at_start != 0, reachable = st->reachable != 0;
    const long long missing = st->missing;                          // among the steps at the level
    long long carried = 0;
    for (int q = tid; q < (int)blockIdx.x; q += 256) carried += block_gain[q];
    carried = block_sum_i64(carried, red);
    long long taken = 0;
    for (int i0 = blockIdx.x * chunk; i0 < min(D, (int)(blockIdx.x + 1) * chunk); i0 += 256) {
        const int i = i0 + tid;
        int lo = 0, up = 0;
        const int32_t *di = drop + (size_t)(i < D ? i : 0) * (MS + 1);
        long long gain = 0;
        if (i < D) {
            lo = lo_in[i];
            up = up_in[i];
            gain = (long long)di[up] - di[lo];
        }
        long long inc = gain;                                       // inclusive scan inside the wave, then over the waves
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        __syncthreads();                                            // the previous round's readers are done
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        long long before = carried;
        for (int q = 0; q < 4; ++q) {
            if (q < wave) before += wave_tot[q];
            carried += wave_tot[q];
        }
        const long long found = before + inc;                       // with this neuron's steps at the level
        long long c = found - gain;                                 // and without
        if (i < D) {
            int J;
            if (at_start) {
                J = 0;
            } else if (!reachable || found < missing) {
                J = up;                                             // unreachable target: every finite step
            } else {
                J = lo;
                while (c < missing) {                               // the neuron that reaches the target: its steps at
                    c += di[J + 1] - di[J];                         // the level, one at a time
                    ++J;
                }
            }
            taken += J;
            b[i] = -tauc[(size_t)i * (MS + 1) + J];
            if (k_out != nullptr) k_out[i] = min(k0[i] + J * eta, T);
        }
    }
    if (steps != nullptr) {
        taken = block_sum_i64(taken, red);
        if (tid == 0 && taken != 0) atomicAdd(steps, (int32_t)taken);
    }
}

}   // namespace svdp
