// gfx950 kernels of the exact top-k comparator (the sorting-based sparsifier
// of Sec. 1 that keeps the k largest accumulated gradients; Sec. 2's error
// feedback supplies the values): a radix select of the k-th largest
// magnitude, the trim of the threshold step's output list, and the pick of
// the top k straight from the residual.  See topk_kernel.h.
#include "topk_kernel.h"

#include <type_traits>

#include "sparsify_kernel.h"

namespace micro {
namespace {

using f32x4 = float __attribute__((ext_vector_type(4)));
using f32x4_dword = float __attribute__((ext_vector_type(4), aligned(4)));  // loads need dword alignment only

constexpr int kWave = 64;

// Where a histogram pass reads its keys.
constexpr int kSrcVec4 = 0;       // acc = grad + residual, 16-byte groups
constexpr int kSrcScalar = 1;     // acc = grad + residual, one value per load
constexpr int kSrcList = 2;       // the values of the step's output list
constexpr int kSrcResVec4 = 3;    // the residual alone (it holds acc), 16-byte groups
constexpr int kSrcResScalar = 4;  // the residual alone, one value per load

__device__ __forceinline__ uint32_t key_of(float v) {
    return __float_as_uint(v) & 0x7FFFFFFFu;
}

// Inclusive sum over the workgroup of one value per thread, in thread order;
// *total receives the workgroup's sum.  Contains two barriers.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_inclusive_sum(uint32_t v, uint32_t* s_wave, uint32_t* total) {
    constexpr int WAVES = BLOCK / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(v, off, kWave);
        if (lane >= off) v += o;
    }
    if (lane == kWave - 1) s_wave[wave] = v;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint32_t t = s_wave[w];
        if (w < wave) before += t;
        sum += t;
    }
    *total = sum;
    __syncthreads();  // s_wave is free again
    return before + v;
}

// Sum of one binary64 per thread over the workgroup in a fixed order (a
// butterfly in each wavefront, then the wavefronts in order); valid in
// thread 0.  Contains one barrier.
template <int WAVES>
__device__ __forceinline__ double block_sum_f64(double v, double* s_part) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) s_part[threadIdx.x / kWave] = v;
    __syncthreads();
    double total = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < WAVES; ++w) total += s_part[w];
    return total;
}

// Pass `pass` of the radix select: a histogram of one digit (bits 30..20,
// 19..9 or 8..0) of the keys that match the digits fixed by the earlier
// passes; NaN keys are not counted.  The keys are those of
// acc = grad + residual over [start, end) (binary32 addition, as in the
// step), of the residual alone there, or of the output list's values.  Each
// workgroup counts in LDS, then adds its nonzero counters to the global ones.
template <int SRC>
__global__ __launch_bounds__(kTopkHistBlock) void topk_hist_kernel(TopkArgs a, uint32_t pass) {
    constexpr bool kGrad = SRC == kSrcVec4 || SRC == kSrcScalar;
    __shared__ uint32_t s_hist[kTopkBins];
    const uint32_t* state = a.words + kTopkBins;
    uint32_t prefix = 0, mask = 0;
    if (pass > 0) {
        if (state[kTopkStatus] != 0) return;  // uniform: nothing left to find
        prefix = state[kTopkPrefix];
        mask = state[kTopkMask];
    }
    const uint32_t shift = pass == 0 ? kTopkFirstShift : pass == 1 ? 9u : 0u;
    const uint32_t digit = pass == 2 ? 511u : 2047u;
    for (int b = threadIdx.x; b < kTopkBins; b += kTopkHistBlock) s_hist[b] = 0u;
    __syncthreads();
    auto count_key = [&](uint32_t key) {
        if (key <= kTopkKeyMax && (key & mask) == prefix) atomicAdd(&s_hist[(key >> shift) & digit], 1u);
    };
    // acc at partition index i
    auto at = [&](int64_t i) {
        if constexpr (kGrad)
            return a.grad[i] + a.residual[i];
        else
            return a.residual[i];
    };
    const int64_t gtid = static_cast<int64_t>(blockIdx.x) * kTopkHistBlock + threadIdx.x;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kTopkHistBlock;
    if constexpr (SRC == kSrcVec4 || SRC == kSrcResVec4) {
        // the 16-byte groups of the body, two per thread in flight; fewer
        // than four values before and after it
        const f32x4* r4 = reinterpret_cast<const f32x4*>(a.residual + a.body_first);
        const f32x4* g4 = kGrad ? reinterpret_cast<const f32x4*>(a.grad + a.body_first) : r4;
        const int64_t groups = (a.body_end - a.body_first) / 4;
        int64_t q = gtid;
        for (; q + stride < groups; q += 2 * stride) {
            f32x4 v0, v1;
            if constexpr (kGrad) {
                const f32x4 g0 = __builtin_nontemporal_load(g4 + q);
                const f32x4 g1 = __builtin_nontemporal_load(g4 + q + stride);
                v0 = g0 + __builtin_nontemporal_load(r4 + q);
                v1 = g1 + __builtin_nontemporal_load(r4 + q + stride);
            } else {
                v0 = __builtin_nontemporal_load(r4 + q);
                v1 = __builtin_nontemporal_load(r4 + q + stride);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v0[c]));
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v1[c]));
        }
        if (q < groups) {
            f32x4 v0;
            if constexpr (kGrad)
                v0 = __builtin_nontemporal_load(g4 + q) + __builtin_nontemporal_load(r4 + q);
            else
                v0 = __builtin_nontemporal_load(r4 + q);
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v0[c]));
        }
        if (gtid < a.body_first - a.start) count_key(key_of(at(a.start + gtid)));
        if (gtid < a.end - a.body_end) count_key(key_of(at(a.body_end + gtid)));
    } else if constexpr (SRC == kSrcScalar || SRC == kSrcResScalar) {
        for (int64_t i = a.start + gtid; i < a.end; i += stride) count_key(key_of(at(i)));
    } else {
        // the list's 16-byte groups, two per thread in flight (the list is
        // 4-byte aligned); fewer than four values before and after them
        const uintptr_t addr = reinterpret_cast<uintptr_t>(a.list);
        int64_t head = static_cast<int64_t>(((16u - (addr & 15u)) & 15u) / sizeof(float));
        if (head > a.list_n) head = a.list_n;
        const f32x4* l4 = reinterpret_cast<const f32x4*>(a.list + head);
        const int64_t groups = (a.list_n - head) / 4;
        int64_t q = gtid;
        for (; q + stride < groups; q += 2 * stride) {
            const f32x4 v0 = l4[q];
            const f32x4 v1 = l4[q + stride];
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v0[c]));
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v1[c]));
        }
        if (q < groups) {
            const f32x4 v0 = l4[q];
#pragma unroll
            for (int c = 0; c < 4; ++c) count_key(key_of(v0[c]));
        }
        const int64_t tail = head + groups * 4;
        if (gtid < head) count_key(key_of(a.list[gtid]));
        if (gtid < a.list_n - tail) count_key(key_of(a.list[tail + gtid]));
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kTopkBins; b += kTopkHistBlock) {
        const uint32_t c = s_hist[b];
        if (c != 0u) atomicAdd(&a.words[b], c);
    }
}

// The select after pass `pass`, one workgroup: finds the digit value whose
// counter holds the wanted key (counting from the largest digit down), fixes
// it in the prefix and leaves the counters zero for the next pass.  Pass 0
// also counts the keys that are not NaN, caps the wanted rank by that count
// and reports its bin to the host; after pass 2 the prefix is the k-th key
// itself and the result goes to the host words.
__global__ __launch_bounds__(kTopkSelectBlock) void topk_select_kernel(TopkArgs a, uint32_t pass) {
    constexpr int PER = kTopkBins / kTopkSelectBlock;
    __shared__ uint32_t s_wave[kTopkSelectBlock / kWave];
    uint32_t* state = a.words + kTopkBins;
    const int tid = threadIdx.x;
    if (pass > 0 && state[kTopkStatus] != 0) return;  // uniform
    const uint32_t bins = pass == 2 ? 512u : static_cast<uint32_t>(kTopkBins);
    const uint32_t per = bins / kTopkSelectBlock;  // 8, or 2 for the last digit
    const uint32_t shift = pass == 0 ? kTopkFirstShift : pass == 1 ? 9u : 0u;
    const uint32_t digit = bins - 1;
    // thread t holds digits bins-1-t*per down to bins-(t+1)*per: thread order
    // is decreasing digit order
    uint32_t c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = static_cast<uint32_t>(i) < per ? a.words[bins - 1 - (tid * per + i)] : 0u;
        mine += c[i];
    }
    uint32_t total;
    const uint32_t above_mine = block_inclusive_sum<kTopkSelectBlock>(mine, s_wave, &total) - mine;
    // every counter of this pass has been read (the sum's barriers): clear them
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (static_cast<uint32_t>(i) < per) a.words[bins - 1 - (tid * per + i)] = 0u;
    uint32_t remaining, prefix = 0, mask = 0, greater = 0;
    if (pass == 0) {
        remaining = total < a.k ? total : a.k;
        if (tid == 0) {
            state[kTopkValid] = total;
            state[kTopkStatus] = remaining == 0 ? 2u : 0u;
        }
        if (remaining == 0) {  // uniform: every value is NaN
            if (tid == 0) {
                a.host[4] = total;
                a.host[5] = 2;
            }
            return;
        }
    } else {
        remaining = state[kTopkRemaining];
        prefix = state[kTopkPrefix];
        mask = state[kTopkMask];
        greater = state[kTopkGreater];
    }
    if (above_mine < remaining && remaining <= above_mine + mine) {
        uint32_t above = above_mine;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (static_cast<uint32_t>(i) >= per) break;
            if (above + c[i] >= remaining) {
                const uint32_t d = bins - 1 - (tid * per + i);
                prefix |= d << shift;
                mask |= digit << shift;
                greater += above;
                remaining -= above;
                state[kTopkPrefix] = prefix;
                state[kTopkMask] = mask;
                state[kTopkGreater] = greater;
                state[kTopkRemaining] = remaining;
                if (pass == 2) {
                    state[kTopkEqual] = c[i];
                    state[kTopkStatus] = 1u;
                }
                if (pass == 0 || pass == 2) {
                    a.host[0] = prefix;
                    a.host[1] = greater;
                    a.host[2] = c[i];
                    a.host[3] = remaining;
                    a.host[4] = pass == 0 ? total : state[kTopkValid];
                    a.host[5] = pass == 0 ? 3 : 1;
                }
                break;
            }
            above += c[i];
        }
    }
}

// The trim's rule for an entry of the output list, given the k-th key `key`
// and the number `keep` of entries equal to it that stay: an entry with a
// lower key leaves; an entry equal to it leaves if `keep` equal entries come
// before it; every other entry moves left by the entries that left before it.
// The step set the residual of the listed values with a key at or above
// `zkey` to +0 and left acc in the others: a leaving entry of the former
// returns its value to the residual, a staying entry of the latter sets its
// residual to +0.

// One workgroup walks the list in chunks of kTopkTrimBlock * 4 entries, in
// order.  A chunk's entries are all read before any of its stores (the
// scans' barriers), and no store reaches beyond its entry's own position, so
// the later chunks still find their entries in place.
__global__ __launch_bounds__(kTopkTrimBlock) void topk_trim_kernel(int32_t* out_idx, float* out_val, float* residual,
                                                                   int64_t n, uint32_t zkey, const uint32_t* words,
                                                                   int64_t* host) {
    constexpr int PER = 4;
    constexpr int64_t CHUNK = static_cast<int64_t>(kTopkTrimBlock) * PER;
    constexpr int WAVES = kTopkTrimBlock / kWave;
    __shared__ uint32_t s_wave[WAVES];
    __shared__ double s_sq[WAVES];
    const uint32_t* state = words + kTopkBins;
    if (state[kTopkStatus] != 1u) return;  // uniform: no k-th key
    const uint32_t key = state[kTopkPrefix];
    const int64_t keep = state[kTopkRemaining];
    const int tid = threadIdx.x;
    int64_t ties_seen = 0, below_seen = 0;
    double sq = 0.0;
    for (int64_t base = 0; base < n; base += CHUNK) {  // uniform
        int32_t idx[PER];
        float val[PER];
        bool tie[PER], below[PER];
        uint32_t mine_t = 0, mine_b = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t pos = base + tid * PER + i;
            const bool live = pos < n;
            idx[i] = live ? out_idx[pos] : 0;
            val[i] = live ? out_val[pos] : 0.0f;
            tie[i] = live && key_of(val[i]) == key;
            below[i] = live && key_of(val[i]) < key;
            mine_t += tie[i] ? 1u : 0u;
            mine_b += below[i] ? 1u : 0u;
        }
        uint32_t chunk_t, chunk_b;
        const uint32_t incl_t = block_inclusive_sum<kTopkTrimBlock>(mine_t, s_wave, &chunk_t);
        const uint32_t incl_b = block_inclusive_sum<kTopkTrimBlock>(mine_b, s_wave, &chunk_b);
        int64_t rank = ties_seen + (incl_t - mine_t);
        int64_t lower = below_seen + (incl_b - mine_b);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t pos = base + tid * PER + i;
            if (pos >= n) break;
            const int64_t before_t = rank, before_b = lower;
            if (tie[i]) ++rank;
            if (below[i]) ++lower;
            if (below[i] || (tie[i] && before_t >= keep)) {
                if (key_of(val[i]) >= zkey) {
                    residual[idx[i]] = val[i];
                    sq += static_cast<double>(val[i]) * static_cast<double>(val[i]);
                }
            } else {
                if (key_of(val[i]) < zkey) residual[idx[i]] = 0.0f;
                const int64_t shift = before_b + (before_t > keep ? before_t - keep : 0);
                if (shift > 0) {
                    out_idx[pos - shift] = idx[i];
                    out_val[pos - shift] = val[i];
                }
            }
        }
        ties_seen += chunk_t;
        below_seen += chunk_b;
    }
    const double total = block_sum_f64<WAVES>(sq, s_sq);
    if (tid == 0) host[6] = static_cast<int64_t>(__double_as_longlong(total));
}

constexpr int kTrimBlock = 256;
constexpr int kTrimPer = kTopkTrimChunk / kTrimBlock;  // entries per thread, row j at j * kTrimBlock + thread
constexpr int kTrimWaves = kTrimBlock / kWave;

// Rows [J0, J0 + J) of a chunk whose first entry is v[base], of the entries
// before v[end] (end > 0): row j's entry at base + j * kTrimBlock + thread,
// or `pad` past end.  Every load is issued before any value is used (the
// index is clamped inside the array and the value replaced afterwards), so
// the loads of a thread overlap instead of each waiting for the last.
template <int J0, int J, class T>
__device__ __forceinline__ void load_rows(const T* v, int64_t base, int64_t end, T pad, T (&out)[J]) {
    const int64_t first = base + J0 * kTrimBlock + threadIdx.x;
    if (base + kTopkTrimChunk <= end) {  // uniform: a whole chunk
#pragma unroll
        for (int j = 0; j < J; ++j) out[j] = v[first + j * kTrimBlock];
    } else {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int64_t p = first + j * kTrimBlock;
            out[j] = v[p < end ? p : end - 1];
        }
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (first + j * kTrimBlock >= end) out[j] = pad;
    }
}

// Parallel trim, launch 1: per chunk of kTopkTrimChunk list entries, the
// entries equal to the k-th key (counts[chunk]) and below it
// (counts[chunks + chunk]).
__global__ __launch_bounds__(kTrimBlock) void topk_trim_count_kernel(const float* out_val, int64_t n,
                                                                     const uint32_t* words, uint32_t* counts,
                                                                     uint32_t chunks) {
    __shared__ uint32_t s_wave[kTrimWaves];
    const uint32_t* state = words + kTopkBins;
    if (state[kTopkStatus] != 1u) return;  // uniform
    const uint32_t key = state[kTopkPrefix];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTopkTrimChunk;
    float v[kTrimPer];
    load_rows<0>(out_val, base, n, __uint_as_float(0xFFFFFFFFu), v);  // padding: a NaN key, neither count
    uint32_t t = 0, b = 0;
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint32_t kv = key_of(v[j]);
        t += kv == key ? 1u : 0u;
        b += kv < key ? 1u : 0u;
    }
    uint32_t total_t, total_b;
    block_inclusive_sum<kTrimBlock>(t, s_wave, &total_t);
    block_inclusive_sum<kTrimBlock>(b, s_wave, &total_b);
    if (threadIdx.x == 0) {
        counts[blockIdx.x] = total_t;
        counts[chunks + blockIdx.x] = total_b;
    }
}

// Launch 2, one workgroup: both count arrays become exclusive prefix sums,
// kScanPer consecutive counts of each array a thread (all loaded before any
// is used), one workgroup scan per kTopkTrimBlock * kScanPer counts.
constexpr int kScanPer = 16;
__global__ __launch_bounds__(kTopkTrimBlock) void topk_trim_scan_kernel(uint32_t* counts, uint32_t chunks) {
    __shared__ uint32_t s_wave[kTopkTrimBlock / kWave];
    constexpr uint32_t SPAN = static_cast<uint32_t>(kTopkTrimBlock) * kScanPer;
    uint32_t* c0 = counts;
    uint32_t* c1 = counts + chunks;
    uint32_t carry0 = 0, carry1 = 0;
    for (uint32_t base = 0; base < chunks; base += SPAN) {  // uniform
        const uint32_t first = base + threadIdx.x * kScanPer;
        uint32_t v0[kScanPer], v1[kScanPer];
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) {
            const uint32_t j = first + i;
            v0[i] = j < chunks ? c0[j] : 0u;
            v1[i] = j < chunks ? c1[j] : 0u;
        }
        uint32_t sum0 = 0, sum1 = 0;
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) {
            sum0 += v0[i];
            sum1 += v1[i];
        }
        uint32_t total0, total1;
        uint32_t run0 = carry0 + block_inclusive_sum<kTopkTrimBlock>(sum0, s_wave, &total0) - sum0;
        uint32_t run1 = carry1 + block_inclusive_sum<kTopkTrimBlock>(sum1, s_wave, &total1) - sum1;
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) {
            const uint32_t j = first + i;
            if (j < chunks) {
                c0[j] = run0;
                c1[j] = run1;
            }
            run0 += v0[i];
            run1 += v1[i];
        }
        carry0 += total0;
        carry1 += total1;
    }
}

// Launch 3: each entry's counts of equal and lower entries before it (its
// chunk's prefixes, then rows in order and lanes in order inside the chunk)
// decide it: a dropped entry returns to the residual (at or above zkey), a
// kept one goes to temp at its position less the entries dropped before it
// (and below zkey sets its residual to +0).  partial[chunk] receives the
// binary64 sum of squares of the returned values.
__global__ __launch_bounds__(kTrimBlock) void topk_trim_scatter_kernel(const int32_t* out_idx, const float* out_val,
                                                                       float* residual, int64_t n, uint32_t zkey,
                                                                       const uint32_t* words,
                                                                       const uint32_t* counts, uint32_t chunks,
                                                                       uint2* temp, double* partial) {
    constexpr int ROWS = kTrimPer * kTrimWaves;
    static_assert(ROWS == kWave, "one (row, wavefront) count per lane of wavefront 0");
    __shared__ uint32_t s_t[ROWS], s_b[ROWS];
    __shared__ double s_sq[kTrimWaves];
    const uint32_t* state = words + kTopkBins;
    if (state[kTopkStatus] != 1u) return;  // uniform
    const uint32_t key = state[kTopkPrefix];
    const int64_t keep = state[kTopkRemaining];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kTopkTrimChunk;
    const uint64_t lower_lanes = lane ? (~0ull >> (kWave - lane)) : 0ull;
    // the chunk's prefixes, read before they are needed
    const int64_t chunk_t = counts[blockIdx.x], chunk_b = counts[chunks + blockIdx.x];
    uint32_t rank_t[kTrimPer], rank_b[kTrimPer];
    bool tie[kTrimPer], below[kTrimPer];
    {
        float v[kTrimPer];
        load_rows<0>(out_val, base, n, __uint_as_float(0xFFFFFFFFu), v);
#pragma unroll
        for (int j = 0; j < kTrimPer; ++j) {
            const uint32_t kv = key_of(v[j]);
            tie[j] = kv == key;
            below[j] = kv < key;
        }
    }
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint64_t mt = __ballot(tie[j]);
        const uint64_t mb = __ballot(below[j]);
        rank_t[j] = static_cast<uint32_t>(__popcll(mt & lower_lanes));
        rank_b[j] = static_cast<uint32_t>(__popcll(mb & lower_lanes));
        if (lane == 0) {
            s_t[j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mt));
            s_b[j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mb));
        }
    }
    __syncthreads();
    if (wave == 0) {  // exclusive prefixes of the (row, wavefront) counts, in list order
        uint32_t vt = s_t[lane], vb = s_b[lane];
        const uint32_t own_t = vt, own_b = vb;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t ot = __shfl_up(vt, off, kWave);
            const uint32_t ob = __shfl_up(vb, off, kWave);
            if (lane >= off) {
                vt += ot;
                vb += ob;
            }
        }
        s_t[lane] = vt - own_t;
        s_b[lane] = vb - own_b;
    }
    __syncthreads();
    double sq = 0.0;
    // two halves of the rows, each with its loads issued together
    auto place = [&](auto half) {
        constexpr int J0 = decltype(half)::value * (kTrimPer / 2);
        int32_t idx[kTrimPer / 2];
        float val[kTrimPer / 2];
        load_rows<J0>(out_idx, base, n, int32_t(0), idx);
        load_rows<J0>(out_val, base, n, 0.0f, val);
#pragma unroll
        for (int u = 0; u < kTrimPer / 2; ++u) {
            const int j = J0 + u;
            const int64_t p = base + j * kTrimBlock + threadIdx.x;
            if (p >= n) continue;
            const int64_t before_t = chunk_t + s_t[j * kTrimWaves + wave] + rank_t[j];
            const int64_t before_b = chunk_b + s_b[j * kTrimWaves + wave] + rank_b[j];
            if (below[j] || (tie[j] && before_t >= keep)) {
                if (key_of(val[u]) >= zkey) {
                    residual[idx[u]] = val[u];
                    sq += static_cast<double>(val[u]) * static_cast<double>(val[u]);
                }
            } else {
                if (key_of(val[u]) < zkey) residual[idx[u]] = 0.0f;
                const int64_t to = p - before_b - (before_t > keep ? before_t - keep : 0);
                temp[to] = make_uint2(static_cast<uint32_t>(idx[u]), __float_as_uint(val[u]));
            }
        }
    };
    place(std::integral_constant<int, 0>{});
    place(std::integral_constant<int, 1>{});
    const double total = block_sum_f64<kTrimWaves>(sq, s_sq);
    if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// Launch 4: temp[0, kept) back into the output lists; workgroup 0 also adds
// the chunks' partial sums in a fixed order into host[6].
__global__ __launch_bounds__(kTrimBlock) void topk_trim_copy_kernel(const uint2* temp, int64_t kept, int32_t* out_idx,
                                                                    float* out_val, const uint32_t* words,
                                                                    const double* partial, uint32_t chunks,
                                                                    int64_t* host) {
    __shared__ double s_sq[kTrimWaves];
    if (words[kTopkBins + kTopkStatus] != 1u) return;  // uniform
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kTrimBlock;
    for (int64_t p = static_cast<int64_t>(blockIdx.x) * kTrimBlock + threadIdx.x; p < kept; p += stride) {
        const uint2 e = temp[p];
        out_idx[p] = static_cast<int32_t>(e.x);
        out_val[p] = __uint_as_float(e.y);
    }
    if (blockIdx.x == 0) {  // uniform
        double sq = 0.0;
        for (uint32_t c = threadIdx.x; c < chunks; c += kTrimBlock) sq += partial[c];
        const double total = block_sum_f64<kTrimWaves>(sq, s_sq);
        if (threadIdx.x == 0) host[6] = static_cast<int64_t>(__double_as_longlong(total));
    }
}

// ---------------------------------------------------------------------------
// The hinted select (topk_kernel.h)
// ---------------------------------------------------------------------------

enum HintedState : int { kHintedStatus = 0, kHintedBin = 1, kHintedGreater = 2, kHintedRank = 3 };

__device__ __forceinline__ bool hinted_list_ok(const TopkHinted& a, int64_t n) {
    return n >= static_cast<int64_t>(a.k) && n <= a.max_list;
}

// Calls f(key) for the keys of list[0, n), two 16-byte groups per thread in
// flight (the list is 4-byte aligned; dword-aligned 16-byte loads).
template <class F>
__device__ __forceinline__ void for_each_key(const float* list, int64_t n, F f) {
    const int64_t gtid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    const f32x4_dword* l4 = reinterpret_cast<const f32x4_dword*>(list);
    const int64_t groups = n / 4;
    int64_t q = gtid;
    for (; q + stride < groups; q += 2 * stride) {
        const f32x4 v0 = l4[q];
        const f32x4 v1 = l4[q + stride];
#pragma unroll
        for (int c = 0; c < 4; ++c) f(key_of(v0[c]));
#pragma unroll
        for (int c = 0; c < 4; ++c) f(key_of(v1[c]));
    }
    if (q < groups) {
        const f32x4 v0 = l4[q];
#pragma unroll
        for (int c = 0; c < 4; ++c) f(key_of(v0[c]));
    }
    if (gtid < n - groups * 4) f(key_of(list[groups * 4 + gtid]));
}

// Launch 1.  Each wavefront counts in a copy of its own in LDS; the workgroup
// adds the nonzero sums to the global counters, so the pass is bound by
// workgroups times lines of nonzero bins and takes few of both (BERT-large
// rank 3's list 6.6 us).
__global__ __launch_bounds__(kTopkHistBlock) void topk_hinted_bins_kernel(TopkHinted a) {
    constexpr int WAVES = kTopkHistBlock / kWave;
    constexpr int BINS = kTopkWindowBins + 1;
    __shared__ uint32_t s_hist[WAVES][BINS];
    const int tid = threadIdx.x;
    for (int i = blockIdx.x * kTopkHistBlock + tid; i < kTopkHintedState - kTopkHintedFine;
         i += gridDim.x * kTopkHistBlock)
        a.words[kTopkHintedFine + i] = 0u;
    const int64_t n = a.count[0];
    if (!hinted_list_ok(a, n)) return;  // uniform
    for (int b = tid; b < WAVES * BINS; b += kTopkHistBlock) (&s_hist[0][0])[b] = 0u;
    __syncthreads();
    uint32_t* mine = s_hist[tid / kWave];
    for_each_key(a.out_val, n, [&](uint32_t key) {
        const uint32_t bin = (key - a.key_floor) >> kTopkFineBits;
        atomicAdd(&mine[bin < kTopkWindowBins ? bin : kTopkWindowBins], 1u);
    });
    __syncthreads();
    for (int b = tid; b < BINS; b += kTopkHistBlock) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) c += s_hist[w][b];
        if (c != 0u) atomicAdd(&a.words[kTopkHintedBins + b], c);
    }
}

// The entry of counters[0, COUNT * STRIDE), one every STRIDE words, holding
// the wanted one, counted from the highest entry down: *entry, *above (the sum
// of the entries above it) and *at (its own).  Every thread of a BLOCK-thread
// workgroup gets the result; none found (wanted above the sum) leaves *entry
// at COUNT.
template <int BLOCK, int COUNT, int STRIDE>
__device__ __forceinline__ void find_from_top(const uint32_t* counters, uint32_t wanted, uint32_t* s_wave,
                                              uint32_t* s_found, uint32_t* entry, uint32_t* above, uint32_t* at) {
    static_assert(COUNT <= BLOCK, "one counter a thread");
    const int tid = threadIdx.x;
    const uint32_t c = tid < COUNT ? counters[(COUNT - 1 - tid) * STRIDE] : 0u;
    if (tid == 0) s_found[0] = COUNT;
    uint32_t total;
    const uint32_t before = block_inclusive_sum<BLOCK>(c, s_wave, &total) - c;  // two barriers
    if (before < wanted && wanted <= before + c) {
        s_found[0] = COUNT - 1 - tid;
        s_found[1] = before;
        s_found[2] = c;
    }
    __syncthreads();
    *entry = s_found[0];
    *above = s_found[1];
    *at = s_found[2];
    __syncthreads();  // s_found is free again
}

// Launch 2.  Every workgroup finds the k-th key's bin from the same counters
// and counts that bin's keys (about a hundredth of the list) in LDS, then
// adds the nonzero counters to those in memory.  (Adding each key straight
// to memory, 30 us on BERT-large's list: scattered atomics, and the group
// counters' few lines.)
__global__ __launch_bounds__(kTopkKeysBlock) void topk_hinted_keys_kernel(TopkHinted a) {
    __shared__ uint32_t s_fine[kTopkFine];
    __shared__ uint32_t s_wave[kTopkKeysBlock / kWave];
    __shared__ uint32_t s_found[3];
    uint32_t* state = a.words + kTopkHintedState;
    const int tid = threadIdx.x;
    const int64_t n = a.count[0];
    const uint32_t over = a.words[kTopkHintedBins + kTopkWindowBins];
    const bool ok = hinted_list_ok(a, n) && over < a.k;  // uniform
    if (!ok) {
        if (blockIdx.x == 0 && tid == 0) state[kHintedStatus] = 4u;
        return;
    }
    for (int i = tid; i < kTopkFine; i += kTopkKeysBlock) s_fine[i] = 0u;
    uint32_t bin, above, in_bin;
    find_from_top<kTopkKeysBlock, kTopkWindowBins, 1>(a.words + kTopkHintedBins, a.k - over, s_wave, s_found, &bin,
                                                      &above, &in_bin);  // barriers: the counters are zero
    if (blockIdx.x == 0 && tid == 0) {
        state[kHintedStatus] = bin < kTopkWindowBins ? 1u : 4u;
        state[kHintedBin] = bin;
        state[kHintedGreater] = over + above;
        state[kHintedRank] = a.k - over - above;
    }
    if (bin >= kTopkWindowBins) return;  // uniform; the counters hold n >= k keys, so not reached
    for_each_key(a.out_val, n, [&](uint32_t key) {
        const uint32_t off = key - a.key_floor;
        if ((off >> kTopkFineBits) == bin) atomicAdd(&s_fine[off & (kTopkFine - 1)], 1u);
    });
    __syncthreads();
    for (int i = tid; i < kTopkFine; i += kTopkKeysBlock) {  // uniform trip count
        const uint32_t c = s_fine[i];
        if (__ballot(c != 0u) == 0) continue;  // uniform in the wavefront, which lies inside one group
        if (c != 0u) atomicAdd(&a.words[kTopkHintedFine + i], c);
        uint32_t sum = c;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
        if ((tid & (kWave - 1)) == 0)
            atomicAdd(&a.words[kTopkHintedGroups + (i >> kTopkGroupBits) * kTopkGroupStride], sum);
    }
}

// Exclusive prefix of item `item` by one wavefront (uniform): look-back over
// status words (count | flag | epoch, the layout of the step's kernels), four
// words per lane and round.  A word is published without waiting for later
// items, so the retries end.
__device__ __forceinline__ uint32_t hinted_lookback(const uint64_t* status, uint32_t item, uint32_t epoch, int lane) {
    constexpr int D = 4;
    uint32_t sum = 0;  // this lane's part
    int64_t top = static_cast<int64_t>(item) - 1;
    for (;;) {
        uint64_t w[D];
        uint32_t valid = 0, incl = 0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int64_t p = top - (lane * D + j);
            w[j] = p >= 0 ? __hip_atomic_load(&status[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                          : (static_cast<uint64_t>(epoch) << kEpochShift) | (2ull << 32);
        }
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const uint32_t flag = static_cast<uint32_t>(w[j] >> 32) & 3u;
            const bool v = (w[j] >> kEpochShift) == epoch && flag != 0;
            valid |= static_cast<uint32_t>(v) << j;
            incl |= static_cast<uint32_t>(v && flag == 2) << j;
        }
        const uint64_t inc_lanes = __ballot(incl != 0);
        const int first = inc_lanes ? __builtin_ctzll(inc_lanes) : kWave;
        const uint32_t need = lane < first ? (1u << D) - 1u : lane == first ? (2u << __builtin_ctz(incl)) - 1u : 0u;
        if (__ballot((need & ~valid) != 0) != 0) {
            __builtin_amdgcn_s_sleep(2);
            continue;
        }
#pragma unroll
        for (int j = 0; j < D; ++j)
            if ((need >> j) & 1u) sum += static_cast<uint32_t>(w[j]);
        if (inc_lanes) break;
        top -= kWave * D;
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    return sum;
}

// Launch 3, bound by the scattered residual stores and the look-back (BERT-large
// rank 3's list 11.8 us, where the four launches of the trim took 25.4 us and
// the gaps between them).  A chunk's entries are all in registers, index and value, before
// its counts are published (the wait and the barrier below), and a chunk
// stores only once the counts of every chunk before it are published, to
// positions no later than its own entries': so no store reaches an entry that
// has not been read, and the list is compacted in place.  Chunks are drawn from
// a ticket counter: waits are for lower chunks of the same launch only, whose
// workgroups drew theirs before and publish without waiting, whatever other
// launches hold the chip.  The draws cost BERT-large's 200 chunks 0.5 us (a
// step 124.5 us by workgroup index, 125.0 drawn) and 1,250 chunks 16 us (100M
// values, k = 5M: 299 and 315 us, 377 before the hinted select).
__global__ __launch_bounds__(kTrimBlock) void topk_hinted_trim_kernel(TopkHinted a) {
    constexpr int ROWS = kTrimPer * kTrimWaves;
    static_assert(ROWS == kWave, "one (row, wavefront) count per lane");
    __shared__ uint32_t s_wave[kTrimWaves], s_found[3];
    __shared__ uint32_t s_cnt[2][ROWS];  // greater, equal: counts, then exclusive prefixes
    __shared__ uint32_t s_before[2], s_item;
    const uint32_t* state = a.words + kTopkHintedState;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int64_t n = a.count[0];
    const bool ok = state[kHintedStatus] == 1u;  // uniform
    if (blockIdx.x == 0) {
        for (int b = tid; b < kTopkWindowBins + 1; b += kTrimBlock) a.words[kTopkHintedBins + b] = 0u;
        if (!ok && tid == 0) a.host[5] = 4;
    }
    if (!ok || static_cast<int64_t>(blockIdx.x) * kTopkTrimChunk >= n) return;  // uniform
    const uint32_t chunks = static_cast<uint32_t>((n + kTopkTrimChunk - 1) / kTopkTrimChunk);
    if (tid == 0) {
        const uint32_t drawn = atomicAdd(&a.words[kTopkHintedTicket], 1u);
        if (drawn == chunks - 1)  // every other workgroup has drawn its ticket
            __hip_atomic_store(&a.words[kTopkHintedTicket], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_item = drawn;
    }
    __syncthreads();
    const uint32_t chunk = __builtin_amdgcn_readfirstlane(s_item);
    if (chunk >= chunks) return;  // only reachable if the counter was not rearmed
    const int64_t base = static_cast<int64_t>(chunk) * kTopkTrimChunk;
    float val[kTrimPer];
    int32_t idx[kTrimPer];
    load_rows<0>(a.out_val, base, n, 0.0f, val);  // padding: below every key of the list
    load_rows<0>(a.out_idx, base, n, int32_t(0), idx);
    const uint32_t bin = state[kHintedBin], rank = state[kHintedRank];
    uint32_t group, group_above, in_group, fine, fine_above, equal;
    find_from_top<kTrimBlock, kTopkGroups, kTopkGroupStride>(a.words + kTopkHintedGroups, rank, s_wave, s_found, &group,
                                                             &group_above, &in_group);
    group = group < kTopkGroups ? group : kTopkGroups - 1;
    find_from_top<kTrimBlock, 1 << kTopkGroupBits, 1>(a.words + kTopkHintedFine + (group << kTopkGroupBits),
                                                      rank - group_above, s_wave, s_found, &fine, &fine_above, &equal);
    const uint32_t key = a.key_floor + (bin << kTopkFineBits) + (group << kTopkGroupBits) + fine;
    const uint32_t keep = rank - group_above - fine_above;
    if (blockIdx.x == 0 && tid == 0) {
        a.host[0] = key;
        a.host[1] = state[kHintedGreater] + group_above + fine_above;
        a.host[2] = equal;
        a.host[3] = keep;
        a.host[4] = n;
        a.host[5] = 1;
    }
    const uint64_t lower_lanes = lane ? (~0ull >> (kWave - lane)) : 0ull;
    uint32_t rank_g[kTrimPer], rank_t[kTrimPer];
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint32_t kv = key_of(val[j]);
        const uint64_t mg = __ballot(kv > key);
        const uint64_t mt = __ballot(kv == key);
        rank_g[j] = static_cast<uint32_t>(__popcll(mg & lower_lanes));
        rank_t[j] = static_cast<uint32_t>(__popcll(mt & lower_lanes));
        if (lane == 0) {
            s_cnt[0][j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mg));
            s_cnt[1][j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mt));
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vector-memory count 0: the chunk's indices have arrived too
    __syncthreads();
    if (wave < 2) {  // wavefront 0: the greater entries; 1: the equal ones
        uint64_t* status = a.status + wave * ((a.max_list + kTopkTrimChunk - 1) / kTopkTrimChunk);
        const uint64_t tag = static_cast<uint64_t>(a.epoch) << kEpochShift;
        const uint32_t own = s_cnt[wave][lane];
        uint32_t v = own;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t o = __shfl_up(v, off, kWave);
            if (lane >= off) v += o;
        }
        const uint32_t total = __shfl(v, kWave - 1, kWave);
        s_cnt[wave][lane] = v - own;
        uint64_t* word = status + chunk;
        if (lane == 0)
            __hip_atomic_store(word, tag | ((chunk == 0 ? 2ull : 1ull) << 32) | total, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        uint32_t before = 0;
        if (chunk != 0) {
            before = hinted_lookback(status, chunk, a.epoch, lane);
            if (lane == 0)
                __hip_atomic_store(word, tag | (2ull << 32) | (before + total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        if (lane == 0) s_before[wave] = before;
    }
    __syncthreads();
    const uint32_t before_g = s_before[0], before_t = s_before[1];
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const int64_t p = base + j * kTrimBlock + tid;
        if (p >= n) continue;
        const uint32_t kv = key_of(val[j]);
        const uint32_t g = before_g + s_cnt[0][j * kTrimWaves + wave] + rank_g[j];
        const uint32_t t = before_t + s_cnt[1][j * kTrimWaves + wave] + rank_t[j];
        if (kv > key || (kv == key && t < keep)) {
            if (kv < a.zero_key) a.residual[idx[j]] = 0.0f;
            const int64_t to = static_cast<int64_t>(g) + (t < keep ? t : keep);
            if (to != p) {
                a.out_idx[to] = idx[j];
                a.out_val[to] = val[j];
            }
        } else if (kv >= a.zero_key) {
            a.residual[idx[j]] = val[j];
        }
    }
}

// The hinted select and the trim by one workgroup.  A short list is bound by
// launches and by each launch's first loads: on ResNet-50 rank 0's list the
// three kernels above take 18 us and two launch gaps, this one 8.9 us (the step
// 52.2 us of wall time with them, 36.4 with this one and the closer bound that
// shortens the list).  Every entry is in registers, index and value, before the first
// store (the wait and the barriers between), so the list is compacted in place.
constexpr int kSmallBlock = 1024;
constexpr int kSmallPer = static_cast<int>(kTopkSmallList) / kSmallBlock;
__global__ __launch_bounds__(kSmallBlock) void topk_hinted_small_kernel(TopkHinted a) {
    constexpr int WAVES = kSmallBlock / kWave;
    constexpr int COUNTS = kSmallPer * WAVES;      // one (row, wavefront) count each
    constexpr int FINE_PER = kTopkFine / kSmallBlock;
    static_assert(COUNTS <= kSmallBlock, "one count a thread in the scan");
    static_assert(kTopkSmallList < (1 << 16), "two counts in one word");
    __shared__ uint32_t s_fine[kTopkFine];
    __shared__ uint32_t s_bins[kTopkWindowBins + 1];
    __shared__ uint32_t s_cnt[COUNTS];             // greater in the low half, equal in the high half
    __shared__ uint32_t s_wave[WAVES], s_found[3];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int64_t count = a.count[0];
    if (count < static_cast<int64_t>(a.k) || count > kTopkSmallList) {  // uniform
        if (tid == 0) a.host[5] = 4;
        return;
    }
    const int n = static_cast<int>(count);
    float val[kSmallPer];
    int32_t idx[kSmallPer];
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (j * kSmallBlock < n) {  // uniform
            const int p = j * kSmallBlock + tid;
            val[j] = a.out_val[p < n ? p : n - 1];
        }
    }
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (j * kSmallBlock < n) {  // uniform
            const int p = j * kSmallBlock + tid;
            idx[j] = a.out_idx[p < n ? p : n - 1];
        }
    }
    for (int i = tid; i < kTopkFine; i += kSmallBlock) s_fine[i] = 0u;
    for (int i = tid; i < kTopkWindowBins + 1; i += kSmallBlock) s_bins[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (j * kSmallBlock < n && j * kSmallBlock + tid < n) {
            const uint32_t bin = (key_of(val[j]) - a.key_floor) >> kTopkFineBits;
            atomicAdd(&s_bins[bin < kTopkWindowBins ? bin : kTopkWindowBins], 1u);
        }
    }
    __syncthreads();
    const uint32_t over = s_bins[kTopkWindowBins];
    if (over >= a.k) {  // uniform: the k-th key is above the bins
        if (tid == 0) a.host[5] = 4;
        return;
    }
    uint32_t bin, above, in_bin;
    find_from_top<kSmallBlock, kTopkWindowBins, 1>(s_bins, a.k - over, s_wave, s_found, &bin, &above, &in_bin);
    const uint32_t rank = a.k - over - above;
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (j * kSmallBlock < n && j * kSmallBlock + tid < n) {
            const uint32_t off = key_of(val[j]) - a.key_floor;
            if ((off >> kTopkFineBits) == bin) atomicAdd(&s_fine[off & (kTopkFine - 1)], 1u);
        }
    }
    __syncthreads();
    {  // the k-th key among the bin's counters, FINE_PER a thread, from the top
        const int top = kTopkFine - 1 - tid * FINE_PER;
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < FINE_PER; ++i) mine += s_fine[top - i];
        uint32_t total;
        uint32_t before = block_inclusive_sum<kSmallBlock>(mine, s_wave, &total) - mine;
        if (before < rank && rank <= before + mine) {
#pragma unroll 1
            for (int i = 0; i < FINE_PER; ++i) {
                const uint32_t c = s_fine[top - i];
                if (before + c >= rank) {
                    s_found[0] = top - i;
                    s_found[1] = before;
                    s_found[2] = c;
                    break;
                }
                before += c;
            }
        }
        __syncthreads();
    }
    const uint32_t key = a.key_floor + (bin << kTopkFineBits) + s_found[0];
    const uint32_t keep = rank - s_found[1];
    if (tid == 0) {
        a.host[0] = key;
        a.host[1] = over + above + s_found[1];
        a.host[2] = s_found[2];
        a.host[3] = keep;
        a.host[4] = n;
        a.host[5] = 1;
    }
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        uint32_t c = 0;
        if (j * kSmallBlock < n) {  // uniform
            const uint32_t kv = j * kSmallBlock + tid < n ? key_of(val[j]) : 0u;
            c = static_cast<uint32_t>(__popcll(__ballot(kv > key))) |
                static_cast<uint32_t>(__popcll(__ballot(kv == key))) << 16;
        }
        if (lane == 0) s_cnt[j * WAVES + wave] = c;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vector-memory count 0: the indices have arrived too
    __syncthreads();
    {
        const uint32_t own = tid < COUNTS ? s_cnt[tid] : 0u;
        uint32_t total;
        const uint32_t incl = block_inclusive_sum<kSmallBlock>(own, s_wave, &total);
        if (tid < COUNTS) s_cnt[tid] = incl - own;
    }
    __syncthreads();
    const uint64_t lower_lanes = lane ? (~0ull >> (kWave - lane)) : 0ull;
#pragma unroll
    for (int j = 0; j < kSmallPer; ++j) {
        if (j * kSmallBlock >= n) break;  // uniform
        const int p = j * kSmallBlock + tid;
        const uint32_t kv = p < n ? key_of(val[j]) : 0u;
        const uint64_t mg = __ballot(kv > key), mt = __ballot(kv == key);
        if (p >= n) continue;
        const uint32_t before = s_cnt[j * WAVES + wave];
        const uint32_t g = (before & 0xffffu) + static_cast<uint32_t>(__popcll(mg & lower_lanes));
        const uint32_t t = (before >> 16) + static_cast<uint32_t>(__popcll(mt & lower_lanes));
        if (kv > key || (kv == key && t < keep)) {
            if (kv < a.zero_key) a.residual[idx[j]] = 0.0f;
            const uint32_t to = g + (t < keep ? t : keep);
            if (to != static_cast<uint32_t>(p)) {
                a.out_idx[to] = idx[j];
                a.out_val[to] = val[j];
            }
        } else if (kv >= a.zero_key) {
            a.residual[idx[j]] = val[j];
        }
    }
}

// Writes the output list back into the residual (one entry a thread, grid
// stride); indices outside [start, end) are skipped.
__global__ __launch_bounds__(kTrimBlock) void topk_restore_kernel(const int32_t* out_idx, const float* out_val,
                                                                  int64_t n, float* residual, int64_t start,
                                                                  int64_t end) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kTrimBlock;
    for (int64_t p = static_cast<int64_t>(blockIdx.x) * kTrimBlock + threadIdx.x; p < n; p += stride) {
        const int64_t i = out_idx[p];
        if (i >= start && i < end) residual[i] = out_val[p];
    }
}

// What a pick takes: the values whose key is above `key`, and the first
// `keep` of those equal to it, NaN aside.  With `words` the key and keep are
// the last select's (nothing is taken without a k-th key); without, they are
// the fixed ones here.
struct PickRule {
    const uint32_t* words;
    uint32_t key;
    int64_t keep;
};

__device__ __forceinline__ bool pick_rule(const PickRule& r, uint32_t& key, int64_t& keep) {
    if (r.words) {
        const uint32_t* state = r.words + kTopkBins;
        if (state[kTopkStatus] != 1u) return false;
        key = state[kTopkPrefix];
        keep = state[kTopkRemaining];
    } else {
        key = r.key;
        keep = r.keep;
    }
    return true;
}

// The pick, launch 1: per chunk of kTopkTrimChunk values of [start, end) of
// the residual, the values equal to the k-th key (counts[chunk]) and above it,
// NaN aside (counts[chunks + chunk]).
__global__ __launch_bounds__(kTrimBlock) void topk_pick_count_kernel(const float* residual, int64_t start,
                                                                     int64_t end, PickRule rule,
                                                                     uint32_t* counts, uint32_t chunks) {
    __shared__ uint32_t s_wave[kTrimWaves];
    uint32_t key;
    int64_t keep;
    if (!pick_rule(rule, key, keep)) return;  // uniform
    const int64_t base = start + static_cast<int64_t>(blockIdx.x) * kTopkTrimChunk;
    float v[kTrimPer];
    load_rows<0>(residual, base, end, __uint_as_float(0xFFFFFFFFu), v);  // padding: a NaN key, neither count
    uint32_t t = 0, h = 0;
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint32_t kv = key_of(v[j]);
        t += kv == key ? 1u : 0u;
        h += kv > key && kv <= kTopkKeyMax ? 1u : 0u;
    }
    uint32_t total_t, total_h;
    block_inclusive_sum<kTrimBlock>(t, s_wave, &total_t);
    block_inclusive_sum<kTrimBlock>(h, s_wave, &total_h);
    if (threadIdx.x == 0) {
        counts[blockIdx.x] = total_t;
        counts[chunks + blockIdx.x] = total_h;
    }
}

// Launch 3 (launch 2 is the trim's scan): each value's counts of equal and
// higher values before it (its chunk's prefixes, then rows in order and lanes
// in order inside the chunk) decide it.  A value above the k-th key, or equal
// to it with fewer than `keep` equal ones before it, is picked: it goes to the
// output at the number of values picked before it, and its residual becomes
// +0.  The placement never reaches past end - start entries.
__global__ __launch_bounds__(kTrimBlock) void topk_pick_scatter_kernel(float* residual, int64_t start, int64_t end,
                                                                       PickRule rule,
                                                                       const uint32_t* counts, uint32_t chunks,
                                                                       int32_t* out_idx, float* out_val) {
    constexpr int ROWS = kTrimPer * kTrimWaves;
    static_assert(ROWS == kWave, "one (row, wavefront) count per lane of wavefront 0");
    __shared__ uint32_t s_t[ROWS], s_h[ROWS];
    uint32_t key;
    int64_t keep;
    if (!pick_rule(rule, key, keep)) return;  // uniform
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t base = start + static_cast<int64_t>(blockIdx.x) * kTopkTrimChunk;
    const uint64_t lower_lanes = lane ? (~0ull >> (kWave - lane)) : 0ull;
    const int64_t chunk_t = counts[blockIdx.x], chunk_h = counts[chunks + blockIdx.x];
    uint32_t rank_t[kTrimPer], rank_h[kTrimPer];
    bool tie[kTrimPer], high[kTrimPer];
    float val[kTrimPer];
    load_rows<0>(residual, base, end, __uint_as_float(0xFFFFFFFFu), val);  // padding: a NaN key
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint32_t kv = key_of(val[j]);
        tie[j] = kv == key;
        high[j] = kv > key && kv <= kTopkKeyMax;
    }
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const uint64_t mt = __ballot(tie[j]);
        const uint64_t mh = __ballot(high[j]);
        rank_t[j] = static_cast<uint32_t>(__popcll(mt & lower_lanes));
        rank_h[j] = static_cast<uint32_t>(__popcll(mh & lower_lanes));
        if (lane == 0) {
            s_t[j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mt));
            s_h[j * kTrimWaves + wave] = static_cast<uint32_t>(__popcll(mh));
        }
    }
    __syncthreads();
    if (wave == 0) {  // exclusive prefixes of the (row, wavefront) counts, in index order
        uint32_t vt = s_t[lane], vh = s_h[lane];
        const uint32_t own_t = vt, own_h = vh;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t ot = __shfl_up(vt, off, kWave);
            const uint32_t oh = __shfl_up(vh, off, kWave);
            if (lane >= off) {
                vt += ot;
                vh += oh;
            }
        }
        s_t[lane] = vt - own_t;
        s_h[lane] = vh - own_h;
    }
    __syncthreads();
    const int64_t cap = end - start;
#pragma unroll
    for (int j = 0; j < kTrimPer; ++j) {
        const int64_t p = base + j * kTrimBlock + threadIdx.x;
        if (p >= end) continue;
        const int64_t before_t = chunk_t + s_t[j * kTrimWaves + wave] + rank_t[j];
        const int64_t before_h = chunk_h + s_h[j * kTrimWaves + wave] + rank_h[j];
        if (high[j] || (tie[j] && before_t < keep)) {
            const int64_t to = before_h + (before_t < keep ? before_t : keep);
            if (to < cap) {
                out_idx[to] = static_cast<int32_t>(p);
                out_val[to] = val[j];
                residual[p] = 0.0f;
            }
        }
    }
}

bool range_args_ok(const TopkArgs& a, bool grad) {
    return (!grad || a.grad) && a.residual && a.words && a.host && a.blocks > 0 && a.end > a.start && a.k > 0 &&
           (!a.vec4 || (a.body_first >= a.start && a.body_end >= a.body_first && a.body_end <= a.end &&
                        (a.body_end - a.body_first) % 4 == 0 && a.body_first - a.start <= 3 &&
                        a.end - a.body_end <= 3));
}

void launch_pass(const TopkArgs& a, TopkSource src, uint32_t pass, hipStream_t stream) {
    const dim3 grid(a.blocks), block(kTopkHistBlock);
    switch (src) {
    case TopkSource::kAcc:
        if (a.vec4)
            hipLaunchKernelGGL(topk_hist_kernel<kSrcVec4>, grid, block, 0, stream, a, pass);
        else
            hipLaunchKernelGGL(topk_hist_kernel<kSrcScalar>, grid, block, 0, stream, a, pass);
        break;
    case TopkSource::kResidual:
        if (a.vec4)
            hipLaunchKernelGGL(topk_hist_kernel<kSrcResVec4>, grid, block, 0, stream, a, pass);
        else
            hipLaunchKernelGGL(topk_hist_kernel<kSrcResScalar>, grid, block, 0, stream, a, pass);
        break;
    case TopkSource::kList:
        hipLaunchKernelGGL(topk_hist_kernel<kSrcList>, grid, block, 0, stream, a, pass);
        break;
    }
    hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(kTopkSelectBlock), 0, stream, a, pass);
}

}  // namespace

hipError_t launch_topk_passes(const TopkArgs& a, TopkSource src, uint32_t first, uint32_t last, hipStream_t stream) {
    if (first > last || last > 2) return hipErrorInvalidValue;
    const bool ok = src == TopkSource::kList ? a.list && a.list_n >= 1 && a.k > 0 && a.words && a.host && a.blocks > 0
                                             : range_args_ok(a, src == TopkSource::kAcc);
    if (!ok) return hipErrorInvalidValue;
    for (uint32_t pass = first; pass <= last; ++pass) launch_pass(a, src, pass, stream);
    return hipGetLastError();
}

hipError_t launch_topk_trim(int32_t* out_idx, float* out_val, float* residual, int64_t n, int64_t kept,
                            uint32_t zero_key, const uint32_t* words, int64_t* host,
                            const TopkTrimScratch* scratch, hipStream_t stream) {
    if (!out_idx || !out_val || !residual || !words || !host || n <= 0 || kept < 1 || kept > n)
        return hipErrorInvalidValue;
    if (!scratch || !scratch->temp) {
        hipLaunchKernelGGL(topk_trim_kernel, dim3(1), dim3(kTopkTrimBlock), 0, stream, out_idx, out_val, residual, n,
                           zero_key, words, host);
        return hipGetLastError();
    }
    if (!scratch->counts || !scratch->partial) return hipErrorInvalidValue;
    const int64_t chunks = (n + kTopkTrimChunk - 1) / kTopkTrimChunk;
    if (chunks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const uint32_t nc = static_cast<uint32_t>(chunks);
    hipLaunchKernelGGL(topk_trim_count_kernel, dim3(nc), dim3(kTrimBlock), 0, stream, out_val, n, words,
                       scratch->counts, nc);
    hipLaunchKernelGGL(topk_trim_scan_kernel, dim3(1), dim3(kTopkTrimBlock), 0, stream, scratch->counts, nc);
    hipLaunchKernelGGL(topk_trim_scatter_kernel, dim3(nc), dim3(kTrimBlock), 0, stream, out_idx, out_val, residual,
                       n, zero_key, words, scratch->counts, nc, scratch->temp, scratch->partial);
    const uint32_t copy_blocks = nc < 2048u ? nc : 2048u;
    hipLaunchKernelGGL(topk_trim_copy_kernel, dim3(copy_blocks), dim3(kTrimBlock), 0, stream, scratch->temp, kept,
                       out_idx, out_val, words, scratch->partial, nc, host);
    return hipGetLastError();
}

hipError_t launch_topk_hinted(const TopkHinted& a, hipStream_t stream) {
    if (!a.count || !a.out_idx || !a.out_val || !a.residual || !a.words || !a.status || !a.host || a.k < 1 ||
        a.max_list < static_cast<int64_t>(a.k) || a.key_floor > kTopkKeyMax)
        return hipErrorInvalidValue;
    const int64_t chunks = (a.max_list + kTopkTrimChunk - 1) / kTopkTrimChunk;
    if (chunks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    // sixteen values a thread of a list of twice k entries, at most 512
    // workgroups of 256 threads and 256 of 1024
    const int64_t want = (2ll * a.k + 4095) / 4096;
    const uint32_t bins_blocks = static_cast<uint32_t>(want < 512 ? want : 512);
    const uint32_t keys_blocks = static_cast<uint32_t>(want < 256 ? want : 256);
    hipLaunchKernelGGL(topk_hinted_bins_kernel, dim3(bins_blocks), dim3(kTopkHistBlock), 0, stream, a);
    hipLaunchKernelGGL(topk_hinted_keys_kernel, dim3(keys_blocks), dim3(kTopkKeysBlock), 0, stream, a);
    hipLaunchKernelGGL(topk_hinted_trim_kernel, dim3(static_cast<uint32_t>(chunks)), dim3(kTrimBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_topk_hinted_small(const TopkHinted& a, hipStream_t stream) {
    if (!a.count || !a.out_idx || !a.out_val || !a.residual || !a.host || a.k < 1 || a.key_floor > kTopkKeyMax)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(topk_hinted_small_kernel, dim3(1), dim3(kSmallBlock), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_topk_restore(const int32_t* out_idx, const float* out_val, int64_t n, float* residual,
                               int64_t start, int64_t end, hipStream_t stream) {
    if (!out_idx || !out_val || !residual || n < 0 || start < 0 || end < start) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    const int64_t blocks = (n + kTrimBlock - 1) / kTrimBlock;
    hipLaunchKernelGGL(topk_restore_kernel, dim3(static_cast<uint32_t>(blocks < 2048 ? blocks : 2048)),
                       dim3(kTrimBlock), 0, stream, out_idx, out_val, n, residual, start, end);
    return hipGetLastError();
}

namespace {

hipError_t launch_pick(float* residual, int64_t start, int64_t end, int32_t* out_idx, float* out_val,
                       const PickRule& rule, uint32_t* counts, hipStream_t stream) {
    if (!residual || !out_idx || !out_val || !counts || start < 0 || end <= start) return hipErrorInvalidValue;
    const int64_t chunks = (end - start + kTopkTrimChunk - 1) / kTopkTrimChunk;
    if (chunks > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const uint32_t nc = static_cast<uint32_t>(chunks);
    hipLaunchKernelGGL(topk_pick_count_kernel, dim3(nc), dim3(kTrimBlock), 0, stream, residual, start, end, rule,
                       counts, nc);
    hipLaunchKernelGGL(topk_trim_scan_kernel, dim3(1), dim3(kTopkTrimBlock), 0, stream, counts, nc);
    hipLaunchKernelGGL(topk_pick_scatter_kernel, dim3(nc), dim3(kTrimBlock), 0, stream, residual, start, end, rule,
                       counts, nc, out_idx, out_val);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_topk_pick(float* residual, int64_t start, int64_t end, int32_t* out_idx, float* out_val,
                            const uint32_t* words, uint32_t* counts, hipStream_t stream) {
    if (!words) return hipErrorInvalidValue;
    return launch_pick(residual, start, end, out_idx, out_val, PickRule{words, 0u, 0}, counts, stream);
}

hipError_t launch_topk_extract(float* residual, int64_t start, int64_t end, uint32_t key_floor, int32_t* out_idx,
                               float* out_val, uint32_t* counts, hipStream_t stream) {
    if (key_floor > kTopkKeyMax) return hipErrorInvalidValue;
    // every key above the floor, and every one equal to it
    return launch_pick(residual, start, end, out_idx, out_val,
                       PickRule{nullptr, key_floor, static_cast<int64_t>(0x7FFFFFFFFFFFFFFFll)}, counts, stream);
}

}  // namespace micro
