// The selection-variable steps of the pruning framework (paper, section 5.1) and the pattern assignment (sections
// 4.1, 5.1) as device kernels: one thread per 3x3 kernel, everything in registers, bound by HBM.  Declared in
// include/pconv_admm.h.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "pconv_admm.h"
#include "pconv_internal.h"

namespace pconv {

#define PCONV_HIP(call)                                  \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) {                          \
            pconv::set_hip_error(#call, (int)e_);        \
            return PCONV_EHIP;                           \
        }                                                \
    } while (0)

namespace {

constexpr int kThreads = 256;

int grid_for(long long n) {
    return (int)((n + kThreads - 1) / kThreads);
}

// One thread, one kernel's vectors.  KMAX is K rounded up to 4, 8, 16 or 32: the vector lives in registers, entries
// from K on are minus infinity, which sorts behind everything and adds nothing to any sum that is used.
// WHOLE: K == KMAX and all four buffers are 16-byte aligned, so a vector is KMAX/4 128-bit accesses.
typedef float float4v __attribute__((ext_vector_type(4)));
template <int KMAX, bool WHOLE>
__global__ __launch_bounds__(kThreads) void proximal_kernel(const float* __restrict__ z, const float* __restrict__ mu,
                                                            double rho, long long n, int K, float* __restrict__ u,
                                                            float* mu_out) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const float* zi = z + i * K;
    float zf[KMAX], mf[KMAX];
    if constexpr (WHOLE) {
#pragma unroll
        for (int q = 0; q < KMAX / 4; ++q) {
            const float4v a = reinterpret_cast<const float4v*>(zi)[q];
            const float4v b = mu ? reinterpret_cast<const float4v*>(mu + i * K)[q] : float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                zf[4 * q + e] = a[e];
                mf[4 * q + e] = b[e];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            zf[j] = j < K ? zi[j] : 0.f;
            mf[j] = (j < K && mu) ? mu[i * K + j] : 0.f;
        }
    }
    double zv[KMAX], mv[KMAX], d[KMAX], s[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        zv[j] = (double)zf[j];
        mv[j] = (double)mf[j];
        d[j] = j < K ? zv[j] + mv[j] / rho : -INFINITY;
        s[j] = d[j];
    }
    // breakpoints, largest first (an odd-even transposition network: KMAX rounds of compare-exchanges on registers)
#pragma unroll
    for (int round = 0; round < KMAX; ++round)
#pragma unroll
        for (int j = round & 1; j + 1 < KMAX; j += 2) {
            const double a = s[j], b = s[j + 1];
            const bool swap = b > a;
            s[j] = swap ? b : a;
            s[j + 1] = swap ? a : b;
        }
    // the root of 1^T [d - nu 1]_+ = 1: with exactly the m largest entries above it, nu = (their sum - 1) / m, and it
    // is the root if it lies in [s[m], s[m-1])
    double nu = 0.0, total = 0.0;
    bool found = false;
#pragma unroll
    for (int m = 1; m <= KMAX; ++m) {
        total += s[m - 1];
        const double cand = (total - 1.0) / (double)m;
        const double lower = (m < KMAX && m < K) ? s[m] : -INFINITY;
        if (!found && m <= K && cand < s[m - 1] && cand >= lower) {
            nu = cand;
            found = true;
        }
    }
    float uf[KMAX], nf[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        const double uj = fmax(d[j] - nu, 0.0);
        uf[j] = (float)uj;
        nf[j] = (float)(mv[j] + rho * (zv[j] - uj));
    }
    if constexpr (WHOLE) {
#pragma unroll
        for (int q = 0; q < KMAX / 4; ++q) {
            if (u) reinterpret_cast<float4v*>(u + i * K)[q] = float4v{uf[4 * q], uf[4 * q + 1], uf[4 * q + 2], uf[4 * q + 3]};
            if (mu_out)
                reinterpret_cast<float4v*>(mu_out + i * K)[q] = float4v{nf[4 * q], nf[4 * q + 1], nf[4 * q + 2], nf[4 * q + 3]};
        }
    } else {
#pragma unroll
        for (int j = 0; j < KMAX; ++j)
            if (j < K) {
                if (u) u[i * K + j] = uf[j];
                if (mu_out) mu_out[i * K + j] = nf[j];
            }
    }
}

__global__ __launch_bounds__(kThreads) void binarize_kernel(const float* __restrict__ z, long long n, int K,
                                                            int32_t* __restrict__ pid) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const float* zi = z + i * K;
    float best = zi[0];
    int arg = 0;
    for (int j = 1; j < K; ++j) {
        const float v = zi[j];
        if (v > best) {          // (strictly: ties stay with the lowest index)
            best = v;
            arg = j;
        }
    }
    pid[i] = arg;
}

// K a multiple of 4 up to 32 and z 16-byte aligned: the vector in KQ 128-bit loads, all issued before the first use
template <int KQ>
__global__ __launch_bounds__(kThreads) void binarize_vec_kernel(const float4v* __restrict__ z, long long n,
                                                                int32_t* __restrict__ pid) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    float4v v[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) v[q] = z[i * KQ + q];
    float best = v[0][0];
    int arg = 0;
#pragma unroll
    for (int q = 0; q < KQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (v[q][e] > best) {
                best = v[q][e];
                arg = 4 * q + e;
            }
    pid[i] = arg;
}

struct Library {
    uint16_t mask[126];
};

// The 256 kernels of a block are 256 x 9 consecutive weights: loaded as one coalesced run (16 bytes per lane and
// load, whatever the storage type), parked in LDS, and read back 9 per thread (a stride of 9 words or 4.5 words
// touches every bank once per 64 lanes' worth of accesses).  Loading 9 weights per thread straight from memory makes
// every wave-wide load touch 36 cache lines.
template <typename T>
__global__ __launch_bounds__(kThreads) void assign_kernel(const T* __restrict__ w, long long n, Library lib, int K,
                                                          int32_t* __restrict__ pid) {
    __shared__ __attribute__((aligned(16))) T tile[kThreads * 9];
    // (the masks once into LDS: indexed by the loop counter straight from the kernel arguments they come as one
    // memory load per pattern, each waited for)
    __shared__ uint32_t masks[126];
    if ((int)threadIdx.x < K) masks[threadIdx.x] = lib.mask[threadIdx.x];
    const long long first = (long long)blockIdx.x * kThreads;             // first kernel of the block
    const int count = (int)(n - first < kThreads ? n - first : kThreads);  // kernels of the block
    const T* src = w + first * 9;
    constexpr int PER = 16 / (int)sizeof(T);                               // elements per 16-byte piece
    const bool aligned = (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
    const int pieces = aligned ? count * 9 / PER : 0;
    for (int k = threadIdx.x; k < pieces; k += kThreads)
        reinterpret_cast<float4v*>(tile)[k] = reinterpret_cast<const float4v*>(src)[k];
    for (int k = pieces * PER + threadIdx.x; k < count * 9; k += kThreads) tile[k] = src[k];   // (tail, or all of it)
    __syncthreads();
    if ((int)threadIdx.x >= count) return;
    double sq[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const double v = (double)(float)tile[threadIdx.x * 9 + t];
        sq[t] = v * v;
    }
    double best = -1.0;
    int arg = 0;
    for (int j = 0; j < K; ++j) {
        // (the mask is the same for the whole wave: its bits become the factors 1.0 and 0.0 on the scalar unit, and a
        // tap is one fused multiply-add -- fma(sq, 1, e) is the rounded sum e + sq, fma(sq, 0, e) is e, so this is
        // the sum of the kept taps in ascending order, one rounding per kept tap, as the host entry computes it;
        // with a select per tap the kernel was bound by its own instructions at a third of the memory rate)
        const unsigned m = __builtin_amdgcn_readfirstlane(masks[j]);
        double e = 0.0;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const double bit = __builtin_bit_cast(double, (m >> t & 1u) ? 0x3FF0000000000000ull : 0ull);
            e = __builtin_fma(sq[t], bit, e);
        }
        if (e > best) {
            best = e;
            arg = j;
        }
    }
    pid[first + threadIdx.x] = arg;
}

// ---- connectivity selection: the k largest squared norms, equal ones by ascending index, without sorting anything.
//
// The squared norm of a pattern-pruned kernel is its key: a non-negative double's bit pattern orders like its value.
// Up to kSmallN kernels are one workgroup's work, keys in registers; up to kMidN one workgroup still ranks them, while
// many compute the keys.  More of them go through a radix selection: one
// pass computes the keys and counts their exponents, one counts the next 10 bits of the keys with the exponent of the
// k-th largest, one gathers the keys that share those 21 bits (a few hundred of 1.6 million), and its last workgroup
// finds the k-th largest among them; the last pass compares every key with it.  Every pass works out the position of
// the k-th largest from the counts of the passes before it, redundantly in each workgroup, so that nothing waits for
// anything but the end of the kernel before.  Where more keys share 21 bits than the list holds -- many equal norms:
// kernels pruned to zero already -- and are not all the same, three more counting passes of 14 bits settle the rest of the
// key; equal keys are ranked by index through counts per run of kernels.  Those passes return at once otherwise.
// 1.6 million fp32 kernels: 300 us with a 64-bit radix sort of (norm, index) pairs, whose eight passes move the pairs
// through memory and back; 55 us so, of which 15 read the weights (59 MB at the rate of a copy).
constexpr int kSelThreads = 1024;
constexpr long long kSmallN = 8 * kSelThreads;                 // up to 8 keys per thread: one workgroup's work
constexpr long long kMidN = 32 * kSelThreads;                  // ... and 32, with two registers a key
constexpr int kBins = 2048;                                    // exponents
constexpr int kBins1 = 1024;                                   // the 10 bits below
constexpr int kReplicas = 8;                                   // copies of the first counts: blocks share few exponents
constexpr int kSlowBits = 14, kSlowBins = 1 << kSlowBits;      // 42 bits below the first 21, in three passes
constexpr int kListCap = 4096;
// (128 workgroups read 13 MB of keys in 4 us, and their counts are half as many additions in memory as 256's)
constexpr int kPassGrid = 128;
constexpr int kRuns = 1024;                                    // runs of kernels whose equal keys are counted

struct SelectState {
    unsigned listed;                   // keys that share the first 21 bits with the k-th largest
    unsigned slow;                     // more of them than the list holds: 1, or 2 where they are all the same
    unsigned last_index;               // of the keys equal to `threshold`, those with at most this index are kept
    unsigned ties_kept;                // slow: how many of them
    unsigned exponent, exponent_rank;  // of the k-th largest, and its rank among the keys with that exponent
    unsigned arrived;                  // workgroups of the gathering pass that are done
    unsigned long long threshold;      // the k-th largest key
    unsigned long long prefix[3];      // slow: its leading bits before each of the three passes, and its rank among the keys with them
    unsigned prefix_rank[3];
    alignas(16) unsigned hist0[kReplicas][kBins];
    unsigned hist1[kBins1];
    union {
        unsigned run_ties[kRuns];
        // (before that) of each workgroup's keys that share the first 21 bits with the k-th largest: the largest, and the
        // largest complement
        unsigned long long ends[kPassGrid][2];
    };
    unsigned slow_hist[3][kSlowBins];  // (the second and third are zeroed where the passes that use them run)
    unsigned list_index[kListCap];
    unsigned long long list_key[kListCap];
};
// words that have to be zero before the first pass
constexpr unsigned kStateWords = (offsetof(SelectState, slow_hist) + sizeof(unsigned[kSlowBins])) / 4;

template <typename T>
__device__ __forceinline__ unsigned long long norm_key(const T* k9, unsigned m) {
    double e = 0.0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const double v = (double)(float)k9[t];
        if (m >> t & 1u) e = e + v * v;                       // (taps ascending, product and sum rounded separately)
    }
    return __builtin_bit_cast(unsigned long long, e) & 0x7FFFFFFFFFFFFFFFull;
}

// The sum over the workgroup's kSelThreads threads of what lane 0 of each wave passes.  `slots` are 32 words of LDS used
// alternately, so one barrier per call is enough.
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ unsigned block_total(unsigned wave_sum, uint4v* slots, unsigned& turn) {
    uint4v* s = slots + (turn & 1u) * 4;
    ++turn;
    if ((threadIdx.x & 63) == 0) reinterpret_cast<unsigned*>(s)[threadIdx.x >> 6] = wave_sum;
    __syncthreads();
    const uint4v t = (s[0] + s[1]) + (s[2] + s[3]);
    return (t.x + t.y) + (t.z + t.w);
}
// ... and, of the waves in front of the calling thread's own.
__device__ __forceinline__ unsigned block_total(unsigned wave_sum, uint4v* slots, unsigned& turn, unsigned* before) {
    const unsigned* s = reinterpret_cast<const unsigned*>(slots + (turn & 1u) * 4);
    const unsigned total = block_total(wave_sum, slots, turn);
    *before = 0;
#pragma unroll
    for (int q = 0; q < kSelThreads / 64; ++q) *before += q < (int)(threadIdx.x >> 6) ? s[q] : 0u;
    return total;
}

// The largest of the threads' `h` and of their `l` (of some values: the largest, and the largest complement -- not 0, a key
// is below 2^63 -- or 0 and 0 where a thread has none).  `ends` is 2 words of LDS that nothing else uses; the call begins
// and ends with a barrier.
__device__ __forceinline__ void block_ends(unsigned long long h, unsigned long long l, unsigned long long* ends,
                                           unsigned long long* high, unsigned long long* not_low) {
    if (threadIdx.x == 0) ends[0] = ends[1] = 0ull;
    __syncthreads();
    if (__any(l != 0ull)) {
        for (int d = 32; d > 0; d >>= 1) {
            const unsigned long long oh = __shfl_xor(h, d), ol = __shfl_xor(l, d);
            h = oh > h ? oh : h;
            l = ol > l ? ol : l;
        }
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&ends[0], h);
            atomicMax(&ends[1], l);
        }
    }
    __syncthreads();
    *high = ends[0];
    *not_low = ends[1];
    __syncthreads();
}

// Bits hi - 1 to lo of the largest value T such that at least k of the workgroup's values are >= T (each thread holds PER,
// those at and beyond its count are 0), whose bits above are in `t`, found bit by bit; true as soon as exactly k values are.
template <int PER, typename V>
__device__ __forceinline__ bool block_bits(const V (&v)[PER], V& t, int hi, int lo, unsigned k, uint4v* slots, unsigned& turn) {
    for (int b = hi - 1; b >= lo; --b) {
        const V cand = t | ((V)1 << b);
        unsigned c = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) c += (unsigned)__popcll(__ballot(v[j] >= cand));
        const unsigned total = block_total(c, slots, turn);
        if (total >= k) t = cand;
        if (total == k) return true;
    }
    return false;
}

// The k-th largest of the workgroup's keys, or a value below it and above the next, where they are alike above the lowest
// `bits` and `base` there.  Keys that differ are apart after a third of their bits; where they are not, it is looked at
// whether those that are left are all the same (kernels pruned to zero, weights of few values: 256 of them took 21 us bit
// by bit to the last).
template <int PER>
__device__ __forceinline__ unsigned long long block_kth(const unsigned long long (&v)[PER], unsigned long long base, int bits,
                                                        unsigned k, uint4v* slots, unsigned& turn, unsigned long long* ends) {
    constexpr int LOOK = 26;
    unsigned long long t = base;
    if (block_bits(v, t, bits, bits < LOOK ? 0 : LOOK, k, slots, turn) || bits <= LOOK) return t;
    unsigned long long high = 0, not_low = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (v[j] >> LOOK == t >> LOOK) {
            high = v[j] > high ? v[j] : high;
            not_low = ~v[j] > not_low ? ~v[j] : not_low;
        }
    block_ends(high, not_low, ends, &high, &not_low);
    if (high == ~not_low) return high;
    block_bits(v, t, LOOK, 0, k, slots, turn);
    return t;
}

template <typename T, int PER>
__global__ __launch_bounds__(kSelThreads) void select_small_kernel(const T* __restrict__ w, int n, Library lib, int K,
                                                                   const int32_t* __restrict__ pid, unsigned k,
                                                                   uint8_t* __restrict__ mask) {
    __shared__ uint32_t masks[126];
    __shared__ uint4v slots[8];
    __shared__ unsigned long long ends[2];
    if ((int)threadIdx.x < K) masks[threadIdx.x] = lib.mask[threadIdx.x];
    __syncthreads();
    // (keys of kernels that do not exist are 0 like those of kernels without weight, but come behind all of them)
    unsigned long long key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kSelThreads + (int)threadIdx.x;
        key[j] = 0;
        if (i < n) {
            const int32_t q = pid[i];
            key[j] = norm_key(w + (size_t)i * 9, masks[(q >= 0 && q < K) ? q : 0]);
        }
    }
    unsigned turn = 0;
    const unsigned long long t = block_kth(key, 0ull, 63, k, slots, turn, ends);
    unsigned above = 0, equal = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        above += (unsigned)__popcll(__ballot(key[j] > t));
        equal += (unsigned)__popcll(__ballot(j * kSelThreads + (int)threadIdx.x < n && key[j] == t));
    }
    above = block_total(above, slots, turn);
    equal = block_total(equal, slots, turn);
    unsigned left = k - above;                                // of the keys equal to t, the first so many by index
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kSelThreads + (int)threadIdx.x;
        const bool tie = i < n && key[j] == t;
        bool keep = key[j] > t || (tie && equal <= left);
        if (equal > left && left > 0) {                       // (uniform: more equal keys than places)
            const unsigned long long ties = __ballot(tie);
            const unsigned before_lane = (unsigned)__popcll(ties & ((1ull << (threadIdx.x & 63)) - 1ull));
            unsigned before_wave;
            const unsigned total = block_total((unsigned)__popcll(ties), slots, turn, &before_wave);
            keep = keep || (tie && before_wave + before_lane < left);
            equal -= total;
            left -= total < left ? total : left;
        }
        if (i < n) mask[i] = keep ? 1 : 0;
    }
}

__global__ __launch_bounds__(kThreads) void select_clear_kernel(unsigned* words) {
    const unsigned i = blockIdx.x * kThreads + threadIdx.x;
    if (i < kStateWords) words[i] = 0u;
}

__global__ __launch_bounds__(kThreads) void select_all_kernel(uint8_t* mask, long long n, uint8_t value) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) mask[i] = value;
}

// The weights of a block's kernels are loaded as one coalesced run and parked in LDS, as in assign_kernel.
template <typename T, bool COUNT>
__global__ __launch_bounds__(kThreads) void norm_key_kernel(const T* __restrict__ w, long long n, Library lib, int K,
                                                            const int32_t* __restrict__ pid,
                                                            unsigned long long* __restrict__ key, SelectState* st) {
    __shared__ __attribute__((aligned(16))) T tile[kThreads * 9];
    __shared__ uint32_t masks[126];
    __shared__ unsigned hist[COUNT ? kBins : 1];
    if ((int)threadIdx.x < K) masks[threadIdx.x] = lib.mask[threadIdx.x];
    if constexpr (COUNT)
        for (int b = threadIdx.x; b < kBins; b += kThreads) hist[b] = 0u;
    constexpr int PER = 16 / (int)sizeof(T);
    for (long long first = (long long)blockIdx.x * kThreads; first < n; first += (long long)gridDim.x * kThreads) {
        const int count = (int)(n - first < kThreads ? n - first : kThreads);
        const T* src = w + first * 9;
        const bool aligned = (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
        const int pieces = aligned ? count * 9 / PER : 0;
        const int32_t q = (int)threadIdx.x < count ? pid[first + threadIdx.x] : 0;
        __syncthreads();                                      // (the tile's readers of the round before are done)
        for (int i = threadIdx.x; i < pieces; i += kThreads)
            reinterpret_cast<float4v*>(tile)[i] = reinterpret_cast<const float4v*>(src)[i];
        for (int i = pieces * PER + threadIdx.x; i < count * 9; i += kThreads) tile[i] = src[i];
        __syncthreads();
        if ((int)threadIdx.x < count) {
            const unsigned long long e = norm_key(tile + threadIdx.x * 9, masks[(q >= 0 && q < K) ? q : 0]);
            key[first + threadIdx.x] = e;
            if constexpr (COUNT) atomicAdd(&hist[(unsigned)(e >> 52)], 1u);
        }
    }
    if constexpr (COUNT) {
        __syncthreads();
        for (int b = threadIdx.x; b < kBins; b += kThreads)
            if (hist[b]) atomicAdd(&st->hist0[blockIdx.x % kReplicas][b], hist[b]);
    }
}

// Where the k-th largest lies among `bins` counted digits: the digit, and its rank (from 1) among the keys with that
// digit.  All threads of a workgroup of kSelThreads; `scratch` is 18 words of LDS.
template <int BINS>
__device__ __forceinline__ void find_digit(const unsigned* __restrict__ hist, int replicas, unsigned k, unsigned* scratch,
                                           unsigned* digit, unsigned* rank) {
    constexpr int PER = BINS / kSelThreads;
    unsigned c[PER], sum = 0;                                 // largest digit first
    if constexpr (PER % 4 == 0) {                             // (one copy of the counts, 16 bytes at a time)
        const uint4v* const mine = reinterpret_cast<const uint4v*>(hist + BINS - ((int)threadIdx.x + 1) * PER);
#pragma unroll
        for (int j = 0; j < PER / 4; ++j) {
            const uint4v v = mine[PER / 4 - 1 - j];
            c[4 * j] = v.w;
            c[4 * j + 1] = v.z;
            c[4 * j + 2] = v.y;
            c[4 * j + 3] = v.x;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) sum += c[j];
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int b = BINS - 1 - ((int)threadIdx.x * PER + j);
            c[j] = 0;
            for (int r = 0; r < replicas; ++r) c[j] += hist[r * BINS + b];
            sum += c[j];
        }
    }
    unsigned incl = sum;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    __syncthreads();
    if (lane == 63) scratch[wave] = incl;
    if (threadIdx.x == 0) {
        scratch[16] = 0;
        scratch[17] = 1;
    }
    __syncthreads();
    unsigned before = incl - sum;
    for (int w = 0; w < wave; ++w) before += scratch[w];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (before < k && k <= before + c[j]) {
            scratch[16] = (unsigned)(BINS - 1 - ((int)threadIdx.x * PER + j));
            scratch[17] = k - before;
        }
        before += c[j];
    }
    __syncthreads();
    *digit = scratch[16];
    *rank = scratch[17];
    __syncthreads();
}

// A workgroup's keys, kAhead per thread in flight at a time.
constexpr int kAhead = 8;
struct Keys {
    unsigned long long e[kAhead];
};
__device__ __forceinline__ Keys keys_from(const unsigned long long* __restrict__ key, long long n, long long first) {
    Keys k;
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
        const long long i = first + j * kSelThreads + threadIdx.x;
        k.e[j] = i < n ? key[i] : 0ull;
    }
    return k;
}
// (the first of them, to be asked for ahead of what the pass has to find out before it can use them)
constexpr long long kKeyRun = (long long)kSelThreads * kAhead;
__device__ __forceinline__ Keys first_keys(const unsigned long long* __restrict__ key, long long n) {
    return keys_from(key, n, (long long)blockIdx.x * kKeyRun);
}
template <typename Fn>
__device__ __forceinline__ void for_keys(const Keys& ahead, const unsigned long long* __restrict__ key, long long n, Fn fn) {
    Keys k = ahead;
    for (long long first = (long long)blockIdx.x * kKeyRun; first < n;) {
        const unsigned long long* const e = k.e;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const long long i = first + j * kSelThreads + threadIdx.x;
            fn(e[j], i, i < n);
        }
        first += (long long)gridDim.x * kKeyRun;
        if (first < n) k = keys_from(key, n, first);
    }
}

// One count more for the digits of the lanes with a hit.  (Equal keys come by the thousand, and additions to one address
// one after the other: where a quarter of a wave agrees with its first lane, those add once.  With an addition each, 32768
// kernels of which four fifths are zero took 15 us here.)
__device__ __forceinline__ void add_digit(unsigned* hist, bool hit, unsigned digit) {
    const unsigned long long hits = __ballot(hit);
    if (!hits) return;
    const int leader = __ffsll((long long)hits) - 1;
    const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)digit, leader);
    const unsigned same = (unsigned)__popcll(__ballot(hit && digit == first));
    if (same < 16u) {
        if (hit) atomicAdd(&hist[digit], 1u);
    } else {
        const bool leads = (int)(threadIdx.x & 63) == leader;
        if (leads || (hit && digit != first)) atomicAdd(&hist[digit], leads ? same : 1u);
    }
}

__global__ __launch_bounds__(kSelThreads) void select_count_kernel(const unsigned long long* __restrict__ key, long long n,
                                                                   unsigned k, SelectState* st) {
    __shared__ unsigned hist[kBins1], scratch[18];
    const Keys ahead = first_keys(key, n);
    for (int b = threadIdx.x; b < kBins1; b += kSelThreads) hist[b] = 0u;
    unsigned exponent, rank;
    find_digit<kBins>(&st->hist0[0][0], kReplicas, k, scratch, &exponent, &rank);
    if (blockIdx.x == 0 && threadIdx.x == 0) {                // (for the passes behind this one)
        st->exponent = exponent;
        st->exponent_rank = rank;
    }
    for_keys(ahead, key, n, [&](unsigned long long e, long long, bool there) {
        add_digit(hist, there && (unsigned)(e >> 52) == exponent, (unsigned)(e >> 42) & (unsigned)(kBins1 - 1));
    });
    __syncthreads();
    for (int b = threadIdx.x; b < kBins1; b += kSelThreads)
        if (hist[b]) atomicAdd(&st->hist1[b], hist[b]);
}

// The k-th largest of the workgroup's keys, all of them at least `base` and alike above the lowest `bits`, and of those
// equal to it the index of the last to be kept, lowest index first (`late`: ~index, 0 where there is no key).
template <int PER>
__device__ __forceinline__ void block_rank(const unsigned long long (&key)[PER], unsigned (&late)[PER],
                                           unsigned long long base, int bits, unsigned k, uint4v* slots,
                                           unsigned long long* ends, unsigned long long* kth, unsigned* last_index) {
    unsigned turn = 0, above = 0;
    const unsigned long long t = block_kth(key, base, bits, k, slots, turn, ends);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        above += (unsigned)__popcll(__ballot(key[j] > t));
        if (key[j] != t) late[j] = 0u;
    }
    above = block_total(above, slots, turn);
    *kth = t;
    unsigned first_late = 0u;
    block_bits(late, first_late, 32, 0, k - above, slots, turn);
    *last_index = ~first_late;
}

// What the last workgroup of a pass reads of the others' work: stored and loaded at device scope (see the pass), like the
// partial sums of a channel split.
template <typename T>
__device__ __forceinline__ void put_for_all(T* to, T v) {
    __hip_atomic_store(to, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T get_of_all(const T* from) {
    return __hip_atomic_load(const_cast<T*>(from), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One workgroup: the k-th largest among the gathered keys, the rank-th of those with the first 21 bits `prefix`, equal ones
// by index.
__device__ __forceinline__ void finish_selection(SelectState* st, unsigned prefix, unsigned rank, uint4v* slots,
                                                 unsigned long long* ends) {
    const unsigned m = get_of_all(&st->listed);
    if (m > (unsigned)kListCap) {
        // (workgroups that found none have left zeros)
        unsigned long long high = 0, not_low = 0;
        if (threadIdx.x < kPassGrid) {
            high = get_of_all(&st->ends[threadIdx.x][0]);
            not_low = get_of_all(&st->ends[threadIdx.x][1]);
        }
        block_ends(high, not_low, ends, &high, &not_low);
        for (int i = threadIdx.x; i < 2 * kSlowBins; i += kSelThreads) (&st->slow_hist[1][0])[i] = 0u;
        if (threadIdx.x == 0) {
            if (high == ~not_low) {
                st->threshold = high;
                st->ties_kept = rank;
            }
            st->prefix[0] = prefix;
            st->prefix_rank[0] = rank;
            st->slow = high == ~not_low ? 2u : 1u;
        }
        return;
    }
    constexpr int PER = kListCap / kSelThreads;
    unsigned long long key[PER];
    unsigned late[PER];                                       // ~index: equal keys, lowest index first
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const unsigned at = (unsigned)j * kSelThreads + threadIdx.x;
        key[j] = at < m ? get_of_all(&st->list_key[at]) : 0ull;
        late[j] = at < m ? ~get_of_all(&st->list_index[at]) : 0u;
    }
    unsigned long long t;
    unsigned last;
    block_rank(key, late, (unsigned long long)prefix << 42, 42, rank, slots, ends, &t, &last);
    if (threadIdx.x == 0) {
        st->threshold = t;
        st->last_index = last;
    }
}

// Lists the keys that share the first 21 bits with the k-th largest, and counts the next 14 of them for the case that the
// list does not hold them; the workgroup that is done last ranks the list.  (As a launch of its own the ranking took 5 us,
// the counting pass 4.4 where there was nothing to count: the end of one kernel and the start of the next.)
__global__ __launch_bounds__(kSelThreads) void select_gather_kernel(const unsigned long long* __restrict__ key, long long n,
                                                                    SelectState* st) {
    __shared__ unsigned scratch[18], found, at0;
    __shared__ uint4v slots[8];
    __shared__ unsigned index[kSelThreads], hist[kSlowBins];
    __shared__ unsigned long long ends[2];
    if (threadIdx.x == 0) {
        found = 0u;
        ends[0] = ends[1] = 0ull;
    }
    const Keys ahead = first_keys(key, n);
    unsigned next, rank;
    unsigned long long high = 0, not_low = 0;
    find_digit<kBins1>(st->hist1, 1, st->exponent_rank, scratch, &next, &rank);
    const unsigned prefix = st->exponent << 10 | next;
    for_keys(ahead, key, n, [&](unsigned long long e, long long i, bool there) {
        const bool hit = there && (unsigned)(e >> 42) == prefix;
        const unsigned long long hits = __ballot(hit);
        if (!hits) return;
        // (one addition per wave: equal keys come by the thousand)
        const int leader = __ffsll((long long)hits) - 1, lane = threadIdx.x & 63;
        unsigned at = 0;
        if (lane == leader) at = atomicAdd(&found, (unsigned)__popcll(hits));
        at = (unsigned)__builtin_amdgcn_readlane((int)at, leader) + (unsigned)__popcll(hits & ((1ull << lane) - 1ull));
        if (hit) {
            if (at < (unsigned)kSelThreads) index[at] = (unsigned)i;
            high = e > high ? e : high;
            not_low = ~e > not_low ? ~e : not_low;
        }
    });
    if (__any(not_low != 0ull)) {
        for (int d = 32; d > 0; d >>= 1) {
            const unsigned long long oh = __shfl_xor(high, d), ol = __shfl_xor(not_low, d);
            high = oh > high ? oh : high;
            not_low = ol > not_low ? ol : not_low;
        }
        if ((threadIdx.x & 63) == 0) {
            atomicMax(&ends[0], high);
            atomicMax(&ends[1], not_low);
        }
    }
    __syncthreads();
    const unsigned m = found;
    auto digit = [](unsigned long long e) { return (unsigned)(e >> (42 - kSlowBits)) & (unsigned)(kSlowBins - 1); };
    if (m != 0) {                                             // (uniform)
        if (threadIdx.x < 2) put_for_all(&st->ends[blockIdx.x][threadIdx.x], ends[threadIdx.x]);
        // (more than a workgroup can hold: the list counts as overflown)
        if (threadIdx.x == 0) at0 = atomicAdd(&st->listed, m <= (unsigned)kSelThreads ? m : (unsigned)kListCap + 1u);
        if (m > (unsigned)kSelThreads && ends[0] != ~ends[1]) {
            for (int b = threadIdx.x; b < kSlowBins; b += kSelThreads) hist[b] = 0u;
            __syncthreads();
            for_keys(first_keys(key, n), key, n, [&](unsigned long long e, long long, bool there) {
                add_digit(hist, there && (unsigned)(e >> 42) == prefix, digit(e));
            });
            __syncthreads();
            for (int b = threadIdx.x; b < kSlowBins; b += kSelThreads)
                if (hist[b]) atomicAdd(&st->slow_hist[0][b], hist[b]);
        } else if (m > (unsigned)kSelThreads) {
            if (threadIdx.x == 0) atomicAdd(&st->slow_hist[0][digit(ends[0])], m);
        }
        __syncthreads();
        if (m <= (unsigned)kSelThreads && threadIdx.x < m) {
            const unsigned long long e = key[index[threadIdx.x]];
            const unsigned at = at0 + threadIdx.x;
            atomicAdd(&st->slow_hist[0][digit(e)], 1u);
            if (at < (unsigned)kListCap) {
                put_for_all(&st->list_key[at], e);
                put_for_all(&st->list_index[at], index[threadIdx.x]);
            }
        }
    }
    // (every wave waits until its stores and additions have reached the level at which all XCDs agree; then the workgroup
    // counts as done.  What the last one reads was never in its own caches)
    __builtin_amdgcn_s_waitcnt(0x0F70);                       // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0)
        at0 = __hip_atomic_fetch_add(&st->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1u ? 1u : 0u;
    __syncthreads();
    if (at0) finish_selection(st, prefix, rank, slots, ends);
}

// The index of the rank-th (from 1) of the PER * kSelThreads keys that is equal to t.  `counts` is PER * 16 words of LDS,
// `found` one.
template <int PER>
__device__ __forceinline__ unsigned nth_equal(const unsigned long long* __restrict__ key, int n, unsigned long long t,
                                              unsigned rank, unsigned* counts, unsigned* found) {
    constexpr int WAVES = kSelThreads / 64, EACH = PER * WAVES / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto equal = [&](int i) { return key[i < n ? i : n - 1] == t && i < n; };
#pragma unroll 4
    for (int j = 0; j < PER; ++j) {
        const unsigned c = (unsigned)__popcll(__ballot(equal(j * kSelThreads + (int)threadIdx.x)));
        if (lane == 0) counts[j * WAVES + wave] = c;
    }
    __syncthreads();
    unsigned c[EACH], sum = 0;                                // (every wave works this out for itself)
#pragma unroll
    for (int q = 0; q < EACH; ++q) sum += c[q] = counts[lane * EACH + q];
    unsigned incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    unsigned before = incl - sum, at = ~0u, left = 0;
#pragma unroll
    for (int q = 0; q < EACH; ++q) {
        if (before < rank && rank <= before + c[q]) {
            at = (unsigned)(lane * EACH + q);
            left = rank - before;
        }
        before += c[q];
    }
    const int lead = __ffsll((long long)__ballot(at != ~0u)) - 1;     // (one lane has it: there are `rank` of them)
    at = __shfl(at, lead);
    left = __shfl(left, lead);
    if ((int)(at % WAVES) == wave) {
        const int i = (int)(at / WAVES) * kSelThreads + (int)threadIdx.x;
        const bool hit = equal(i);
        const unsigned long long hits = __ballot(hit);
        if (hit && (unsigned)__popcll(hits & ((1ull << lane) - 1ull)) + 1u == left) *found = (unsigned)i;
    }
    __syncthreads();
    return *found;
}

// kSmallN < n <= kMidN: one workgroup ranks the keys that norm_key_kernel left, from registers.  Their leading 19 bits
// are counted as a distance from the largest key's -- 256 bins an octave over the 16 octaves below it, everything
// smaller in the last bin -- and only the keys that share the k-th largest's bin are ranked bit by bit.  Where those do
// not fit the list (norms that are equal or nearly so by the thousand), their own bits below what they share are
// counted, 12 at a time, until the rest fits or is all the same.  The radix selection's ten launches took 52 us of an
// iteration at 12607 fp16 kernels (46 us with a library's sort); two launches take 23 us.
template <int PER>
__global__ __launch_bounds__(kSelThreads) void select_mid_kernel(const unsigned long long* __restrict__ src, int n,
                                                                 unsigned k, uint8_t* __restrict__ mask) {
    constexpr int DIST = 4096, LIST = kListCap / kSelThreads, LOW = 44, REST = 32;
    __shared__ __attribute__((aligned(16))) unsigned hist[DIST];
    __shared__ unsigned scratch[18], wave_max[kSelThreads / 64], listed;
    __shared__ unsigned long long list_key[kListCap], ends[2];
    __shared__ unsigned list_late[kListCap];
    __shared__ uint4v slots[8];
    // (the places' numbers and which of them exist, worked out anew for each of the loops: kept from the first one on
    // they are 32 vector and 64 scalar registers, and the kernel spills.  A form that did gave wrong marks: the compiler
    // had put copies of the keys' registers at the end of a branch that some waves do not take, in front of the
    // instruction that brings those waves back)
    int thread = (int)threadIdx.x;
    auto anew = [&] { asm volatile("" : "+v"(thread), "+s"(n)); };
    // (places behind the last kernel hold 0, like kernels without weight; a row of places is loaded by all lanes or not at
    // all: behind a branch of its own each load would be waited for)
    unsigned long long key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kSelThreads + thread;
        key[j] = 0ull;
        if (j * kSelThreads < n) key[j] = src[i < n ? i : n - 1];
    }
    anew();
    const bool partial = thread >= (n & (kSelThreads - 1));      // of the lanes of the last row, if that is not full
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (n - j * kSelThreads < kSelThreads && n > j * kSelThreads) key[j] = partial ? 0ull : key[j];
    for (int b = threadIdx.x; b < DIST; b += kSelThreads) hist[b] = 0u;
    if (threadIdx.x == 0) listed = 0u;
    unsigned top = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) top = max(top, (unsigned)(key[j] >> REST));
    for (int d = 32; d > 0; d >>= 1) top = max(top, (unsigned)__shfl_xor(top, d));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = top;
    __syncthreads();
    for (int q = 0; q < kSelThreads / 64; ++q) top = max(top, wave_max[q]);
    const unsigned first = top >> (LOW - REST);               // (19 bits)
    auto bin = [&](unsigned e) {                              // larger keys, larger bins
        const unsigned d = first - (e >> (LOW - REST));
        return d < (unsigned)DIST ? (unsigned)DIST - 1u - d : 0u;
    };
    anew();
    bool crowd = false;                                       // (a look at every eighth: 2 us at 32768 if at each)
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j * kSelThreads >= n) continue;
        const unsigned b = bin((unsigned)(key[j] >> REST));
        if (j % 8 == 0) crowd = __popcll(__ballot(b == (unsigned)__builtin_amdgcn_readfirstlane((int)b))) >= 16;
        if (crowd) add_digit(hist, true, b);
        else atomicAdd(&hist[b], 1u);
    }
    __syncthreads();
    unsigned digit, rank;
    find_digit<DIST>(hist, 1, k, scratch, &digit, &rank);
    // the candidates are the keys in [low, high]; those above are kept
    bool fits = hist[digit] <= (unsigned)kListCap;
    unsigned long long low, high;
    int bits;                                                 // in which the candidates may differ
    if (digit == 0) {                                         // (the last bin: everything that far below the largest)
        low = 0ull;
        high = (unsigned long long)(first - (unsigned)DIST + 1u) << LOW | ((1ull << LOW) - 1ull);
        bits = 63;
    } else {
        low = (unsigned long long)(first - ((unsigned)DIST - 1u - digit)) << LOW;
        high = low | ((1ull << LOW) - 1ull);
        bits = LOW;
    }
    unsigned long long t = 0ull;
    unsigned last = 0u;
    anew();
    while (!fits) {                                           // (uniform; 12 bits less each time, at most six times)
        unsigned long long h = 0, l = 0;
#pragma unroll 8
        for (int j = 0; j < PER; ++j) {
            const int i = j * kSelThreads + thread;
            const unsigned long long e = src[i < n ? i : n - 1];
            if (i < n && e >= low && e <= high) {
                h = e > h ? e : h;
                l = ~e > l ? ~e : l;
            }
        }
        unsigned long long not_low;
        block_ends(h, l, ends, &high, &not_low);
        low = ~not_low;
        if (low == high) break;
        bits = 64 - __clzll(low ^ high);
        const int shift = bits > 12 ? bits - 12 : 0;
        for (int b = threadIdx.x; b < DIST; b += kSelThreads) hist[b] = 0u;
        __syncthreads();
#pragma unroll 8
        for (int j = 0; j < PER; ++j) {
            const int i = j * kSelThreads + thread;
            const unsigned long long e = src[i < n ? i : n - 1];
            add_digit(hist, i < n && e >= low && e <= high, (unsigned)(e >> shift) & (unsigned)(DIST - 1));
        }
        __syncthreads();
        find_digit<DIST>(hist, 1, rank, scratch, &digit, &rank);
        fits = hist[digit] <= (unsigned)kListCap;
        low = (low >> bits << bits) | (unsigned long long)digit << shift;
        high = low | ((1ull << shift) - 1ull);
        bits = shift;
        __syncthreads();
    }
    anew();
    if (fits) {                                               // (uniform)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = j * kSelThreads + thread;
            if (key[j] < low || key[j] > high || i >= n) continue;
            const unsigned at = atomicAdd(&listed, 1u);
            list_key[at] = key[j];
            list_late[at] = ~(unsigned)i;
        }
        __syncthreads();
        const unsigned m = listed;
        unsigned long long some[LIST];
        unsigned late[LIST];
#pragma unroll
        for (int j = 0; j < LIST; ++j) {
            const unsigned at = (unsigned)j * kSelThreads + threadIdx.x;
            some[j] = at < m ? list_key[at] : 0ull;
            late[j] = at < m ? list_late[at] : 0u;
        }
        block_rank(some, late, low, bits, rank, slots, ends, &t, &last);
    } else {
        t = high;
        last = nth_equal<PER>(src, n, t, rank, hist, scratch);
    }
    anew();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * kSelThreads + thread;
        if (i >= n) continue;
        const bool keep = key[j] > t || (key[j] == t && (unsigned)i <= last);
        mask[i] = keep ? 1 : 0;
    }
}

// The bits below the first 21, 14 at a time, where too many keys share those: what is known of the k-th largest after
// `passes` (1 to 3) counts of them, from what the pass before has left and its counts.
__device__ __forceinline__ unsigned long long slow_prefix(const SelectState* st, int passes, unsigned* scratch,
                                                          unsigned* rank) {
    unsigned digit;
    find_digit<kSlowBins>(st->slow_hist[passes - 1], 1, st->prefix_rank[passes - 1], scratch, &digit, rank);
    return st->prefix[passes - 1] << kSlowBits | digit;
}
__global__ __launch_bounds__(kSelThreads) void select_slow_kernel(const unsigned long long* __restrict__ key, long long n,
                                                                  int pass, SelectState* st) {
    if (st->slow != 1u) return;
    __shared__ unsigned hist[kSlowBins], scratch[18];
    for (int b = threadIdx.x; b < kSlowBins; b += kSelThreads) hist[b] = 0u;
    unsigned rank;
    const unsigned long long prefix = slow_prefix(st, pass, scratch, &rank);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->prefix[pass] = prefix;
        st->prefix_rank[pass] = rank;
    }
    const int top = 42 - kSlowBits * pass, low = top - kSlowBits;
    for_keys(first_keys(key, n), key, n, [&](unsigned long long e, long long, bool there) {
        add_digit(hist, there && (e >> top) == prefix, (unsigned)(e >> low) & (unsigned)(kSlowBins - 1));
    });
    __syncthreads();
    for (int b = threadIdx.x; b < kSlowBins; b += kSelThreads)
        if (hist[b]) atomicAdd(&st->slow_hist[pass][b], hist[b]);
}

// Runs of kernels: run r of kRuns is kernels r*run .. r*run + run - 1.
__host__ __device__ __forceinline__ long long run_length(long long n) {
    const long long per = (n + kRuns - 1) / kRuns;
    return (per + kSelThreads - 1) / kSelThreads * kSelThreads;
}
__global__ __launch_bounds__(kSelThreads) void select_ties_kernel(const unsigned long long* __restrict__ key, long long n,
                                                                  SelectState* st) {
    if (!st->slow) return;
    __shared__ unsigned scratch[18];
    __shared__ uint4v slots[8];
    unsigned rank, turn = 0;
    const bool known = st->slow == 2u;
    const unsigned long long t = known ? st->threshold : slow_prefix(st, 3, scratch, &rank);
    const long long run = run_length(n);
    for (int r = blockIdx.x; r < kRuns && (long long)r * run < n; r += gridDim.x) {
        const long long first = (long long)r * run;
        unsigned c = 0;
        for (long long i = first + threadIdx.x; i < first + run && i - threadIdx.x < n; i += kSelThreads)
            c += (unsigned)__popcll(__ballot(i < n && key[i] == t));
        c = block_total(c, slots, turn);
        if (threadIdx.x == 0) st->run_ties[r] = c;
    }
    if (threadIdx.x == 0 && blockIdx.x == 0 && !known) {
        st->threshold = t;
        st->ties_kept = rank;
    }
}

// VEC: four keys and one word of marks per thread and round (n a multiple of 4, aligned buffers)
template <bool VEC>
__global__ __launch_bounds__(kSelThreads) void mark_kept_kernel(const unsigned long long* __restrict__ key, long long n,
                                                                const SelectState* st, uint8_t* __restrict__ mask) {
    const unsigned long long t = st->threshold;
    if (!st->slow) {
        const unsigned last = st->last_index;
        auto kept = [&](unsigned long long e, long long i) { return e > t || (e == t && (unsigned)i <= last); };
        const long long at = (long long)blockIdx.x * kSelThreads + threadIdx.x, step = (long long)gridDim.x * kSelThreads;
        if constexpr (VEC) {
            typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
            for (long long i = at * 4; i < n; i += step * 4) {
                const u64x2 a = *reinterpret_cast<const u64x2*>(key + i), b = *reinterpret_cast<const u64x2*>(key + i + 2);
                unsigned m = kept(a.x, i) ? 1u : 0u;
                m |= kept(a.y, i + 1) ? 0x100u : 0u;
                m |= kept(b.x, i + 2) ? 0x10000u : 0u;
                m |= kept(b.y, i + 3) ? 0x1000000u : 0u;
                *reinterpret_cast<unsigned*>(mask + i) = m;
            }
        } else {
            for (long long i = at; i < n; i += step) mask[i] = kept(key[i], i) ? 1 : 0;
        }
        return;
    }
    __shared__ uint4v slots[8];
    unsigned turn = 0;
    const unsigned ties_kept = st->ties_kept;
    const long long run = run_length(n);
    for (int r = blockIdx.x; r < kRuns && (long long)r * run < n; r += gridDim.x) {
        unsigned before = 0;
        for (int q = threadIdx.x; q < r; q += kSelThreads) before += st->run_ties[q];
        for (int d = 32; d > 0; d >>= 1) before += __shfl_down(before, d);
        before = block_total(before, slots, turn);            // (a wave's lane 0 holds its sum)
        const long long first = (long long)r * run;
        for (long long i = first + threadIdx.x; i < first + run && i - threadIdx.x < n; i += kSelThreads) {
            const unsigned long long e = i < n ? key[i] : 0ull;
            const bool tie = i < n && e == t;
            const unsigned long long ties = __ballot(tie);
            unsigned before_wave;
            const unsigned total = block_total((unsigned)__popcll(ties), slots, turn, &before_wave);
            const unsigned rank = before + before_wave + (unsigned)__popcll(ties & ((1ull << (threadIdx.x & 63)) - 1ull));
            before += total;
            if (i < n) mask[i] = (e > t || (tie && rank < ties_kept)) ? 1 : 0;
        }
    }
}

size_t round256(size_t b) {
    return (b + 255) / 256 * 256;
}

}  // namespace
}  // namespace pconv

using namespace pconv;

extern "C" int pconv_select_connectivity_device(const void* w, int dtype, long long n, const uint16_t* lib, int K,
                                                const int32_t* pid, double keep, uint8_t* mask, void* workspace,
                                                size_t* workspace_bytes, void* stream) {
    if (!workspace_bytes || n < 0 || (dtype != PCONV_F32 && dtype != PCONV_F16)) return PCONV_EINVAL;
    if (n > 0x7FFFFFFFll) return PCONV_ESHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // workspace: the keys and the radix selection's state (counts, list)
    const size_t kb = round256((size_t)n * 8);
    const size_t need = n <= kSmallN ? 256 : n <= kMidN ? kb : kb + round256(sizeof(SelectState));
    if (!workspace) {
        *workspace_bytes = need;
        return PCONV_OK;
    }
    if (!w || !lib || !pid || !mask || !(keep >= 0.0 && keep <= 1.0)) return PCONV_EINVAL;
    if (K < 1 || K > 126) return PCONV_EPATTERN;
    Library l{};
    for (int j = 0; j < K; ++j) {
        if (lib[j] >= 512 || __builtin_popcount(lib[j]) != 4) return PCONV_EPATTERN;
        l.mask[j] = lib[j];
    }
    if (*workspace_bytes < need || reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return PCONV_ESCRATCH;
    if (n == 0) return PCONV_OK;
    long long kept = (long long)std::floor(keep * (double)n + 0.5);
    kept = kept < 0 ? 0 : (kept > n ? n : kept);
    const unsigned k = (unsigned)kept;
    const bool f32 = dtype == PCONV_F32;
    if (kept == 0 || kept == n) {                              // nothing to choose
        hipLaunchKernelGGL(select_all_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, mask, n, (uint8_t)(kept ? 1 : 0));
        PCONV_HIP(hipGetLastError());
        return PCONV_OK;
    }
    if (n <= kSmallN) {
#define PCONV_SELECT(T, PER)                                                                                             \
    hipLaunchKernelGGL((select_small_kernel<T, PER>), dim3(1), dim3(kSelThreads), 0, st, static_cast<const T*>(w), (int)n, l, \
                       K, pid, k, mask)
        if (n <= kSelThreads) {
            if (f32) PCONV_SELECT(float, 1); else PCONV_SELECT(_Float16, 1);
        } else if (n <= 4 * kSelThreads) {
            if (f32) PCONV_SELECT(float, 4); else PCONV_SELECT(_Float16, 4);
        } else {
            if (f32) PCONV_SELECT(float, 8); else PCONV_SELECT(_Float16, 8);
        }
#undef PCONV_SELECT
        PCONV_HIP(hipGetLastError());
        return PCONV_OK;
    }
    unsigned long long* key = static_cast<unsigned long long*>(workspace);
    // (each block counts the exponents of several runs of kernels before it adds them to the counts in memory)
    const dim3 norm_grid((unsigned)std::min<long long>(grid_for(n), 2048)), block(kThreads), sel(kSelThreads);
#define PCONV_NORMS(COUNT, STATE)                                                                                        \
    do {                                                                                                                 \
        if (f32)                                                                                                         \
            hipLaunchKernelGGL((norm_key_kernel<float, COUNT>), norm_grid, block, 0, st, static_cast<const float*>(w), n, l, \
                               K, pid, key, STATE);                                                                      \
        else                                                                                                             \
            hipLaunchKernelGGL((norm_key_kernel<_Float16, COUNT>), norm_grid, block, 0, st,                              \
                               static_cast<const _Float16*>(w), n, l, K, pid, key, STATE);                               \
    } while (0)
    if (n <= kMidN) {
        PCONV_NORMS(false, nullptr);
        if (n <= kMidN / 2)
            hipLaunchKernelGGL(select_mid_kernel<16>, dim3(1), sel, 0, st, key, (int)n, k, mask);
        else
            hipLaunchKernelGGL(select_mid_kernel<32>, dim3(1), sel, 0, st, key, (int)n, k, mask);
        PCONV_HIP(hipGetLastError());
        return PCONV_OK;
    }
    SelectState* state = reinterpret_cast<SelectState*>(static_cast<char*>(workspace) + kb);
    hipLaunchKernelGGL(select_clear_kernel, dim3((kStateWords + kThreads - 1) / kThreads), dim3(kThreads), 0, st,
                       reinterpret_cast<unsigned*>(state));
    PCONV_NORMS(true, state);
#undef PCONV_NORMS
    const dim3 pass_grid((unsigned)std::min<long long>((n + kAhead * kSelThreads - 1) / (kAhead * kSelThreads), kPassGrid));
    hipLaunchKernelGGL(select_count_kernel, pass_grid, sel, 0, st, key, n, k, state);
    hipLaunchKernelGGL(select_gather_kernel, pass_grid, sel, 0, st, key, n, state);
    for (int p = 1; p < 3; ++p) hipLaunchKernelGGL(select_slow_kernel, pass_grid, sel, 0, st, key, n, p, state);
    // (a run at a time where equal keys are ranked: one workgroup a run as far as they go)
    const dim3 run_grid((unsigned)std::min<long long>((n + kSelThreads - 1) / kSelThreads, kPassGrid));
    hipLaunchKernelGGL(select_ties_kernel, run_grid, sel, 0, st, key, n, state);
    if (n % 4 == 0 && reinterpret_cast<uintptr_t>(mask) % 4 == 0)
        hipLaunchKernelGGL(mark_kept_kernel<true>, run_grid, sel, 0, st, key, n, state, mask);
    else
        hipLaunchKernelGGL(mark_kept_kernel<false>, run_grid, sel, 0, st, key, n, state, mask);
    PCONV_HIP(hipGetLastError());
    return PCONV_OK;
}

extern "C" int pconv_admm_proximal(const float* z, const float* mu, float rho, long long n, int K, float* u,
                                   float* mu_out, void* stream) {
    if (!z || K < 1 || K > 32 || n < 0 || !(rho > 0.0f) || std::isinf(rho)) return PCONV_EINVAL;
    if (n == 0 || (!u && !mu_out)) return PCONV_OK;
    if (n > 0x7FFFFFFFll * kThreads) return PCONV_ESHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid(grid_for(n)), block(kThreads);
    const uintptr_t bits = reinterpret_cast<uintptr_t>(z) | reinterpret_cast<uintptr_t>(mu) | reinterpret_cast<uintptr_t>(u) |
                           reinterpret_cast<uintptr_t>(mu_out);
    const bool whole = (K == 4 || K == 8 || K == 16 || K == 32) && bits % 16 == 0;
#define PCONV_PROX(KM)                                                                                              \
    do {                                                                                                            \
        if (whole)                                                                                                  \
            hipLaunchKernelGGL((proximal_kernel<KM, true>), grid, block, 0, st, z, mu, (double)rho, n, K, u, mu_out);   \
        else                                                                                                        \
            hipLaunchKernelGGL((proximal_kernel<KM, false>), grid, block, 0, st, z, mu, (double)rho, n, K, u, mu_out);  \
    } while (0)
    if (K <= 4)
        PCONV_PROX(4);
    else if (K <= 8)
        PCONV_PROX(8);
    else if (K <= 16)
        PCONV_PROX(16);
    else
        PCONV_PROX(32);
#undef PCONV_PROX
    PCONV_HIP(hipGetLastError());
    return PCONV_OK;
}

extern "C" int pconv_admm_binarize(const float* z, long long n, int K, int32_t* pid, void* stream) {
    if (!z || !pid || K < 1 || K > 126 || n < 0) return PCONV_EINVAL;
    if (n == 0) return PCONV_OK;
    if (n > 0x7FFFFFFFll * kThreads) return PCONV_ESHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid(grid_for(n)), block(kThreads);
    const float4v* zq = reinterpret_cast<const float4v*>(z);
    const bool vec = K % 4 == 0 && K <= 32 && reinterpret_cast<uintptr_t>(z) % 16 == 0;
    switch (vec ? K / 4 : 0) {
        case 1: hipLaunchKernelGGL(binarize_vec_kernel<1>, grid, block, 0, st, zq, n, pid); break;
        case 2: hipLaunchKernelGGL(binarize_vec_kernel<2>, grid, block, 0, st, zq, n, pid); break;
        case 3: hipLaunchKernelGGL(binarize_vec_kernel<3>, grid, block, 0, st, zq, n, pid); break;
        case 4: hipLaunchKernelGGL(binarize_vec_kernel<4>, grid, block, 0, st, zq, n, pid); break;
        case 5: hipLaunchKernelGGL(binarize_vec_kernel<5>, grid, block, 0, st, zq, n, pid); break;
        case 6: hipLaunchKernelGGL(binarize_vec_kernel<6>, grid, block, 0, st, zq, n, pid); break;
        case 7: hipLaunchKernelGGL(binarize_vec_kernel<7>, grid, block, 0, st, zq, n, pid); break;
        case 8: hipLaunchKernelGGL(binarize_vec_kernel<8>, grid, block, 0, st, zq, n, pid); break;
        default: hipLaunchKernelGGL(binarize_kernel, grid, block, 0, st, z, n, K, pid);
    }
    PCONV_HIP(hipGetLastError());
    return PCONV_OK;
}

extern "C" int pconv_assign_patterns_device(const void* w, int dtype, long long n, const uint16_t* lib, int K,
                                            int32_t* pid, void* stream) {
    if (!w || !lib || !pid || n < 0 || (dtype != PCONV_F32 && dtype != PCONV_F16)) return PCONV_EINVAL;
    if (K < 1 || K > 126) return PCONV_EPATTERN;
    Library l{};
    for (int j = 0; j < K; ++j) {
        if (lib[j] >= 512 || __builtin_popcount(lib[j]) != 4) return PCONV_EPATTERN;
        l.mask[j] = lib[j];
    }
    if (n == 0) return PCONV_OK;
    if (n > 0x7FFFFFFFll * kThreads) return PCONV_ESHAPE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dtype == PCONV_F32)
        hipLaunchKernelGGL(assign_kernel<float>, dim3(grid_for(n)), dim3(kThreads), 0, st, static_cast<const float*>(w), n,
                           l, K, pid);
    else
        hipLaunchKernelGGL(assign_kernel<_Float16>, dim3(grid_for(n)), dim3(kThreads), 0, st,
                           static_cast<const _Float16*>(w), n, l, K, pid);
    PCONV_HIP(hipGetLastError());
    return PCONV_OK;
}
