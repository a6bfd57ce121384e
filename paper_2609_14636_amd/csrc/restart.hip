// restart.hip -- prefix-buffer restart pick of the weakest correct unit.
//
// Sec. 4.2 step 1: unit k is correct iff its value exceeds alpha (strictly),
// here also requiring its correctness-mask bit.  Step 2 and Eq. (6): K_max
// counts the correct units from the start of the record up to the first one
// that is not, and k* is the argmin of the values among those K_max units.  Step 3 and Algorithm 1: the next rollout reuses K0 = k* - 1
// turns (1-based) as context; a task without a usable prefix starts from 0.
// The record is the rollout's units up to and including its stop (Algorithm 1
// records the generated turns).  Ties go to the lowest index.
//
// A wave or a workgroup per rollout reads the record once, in chunks of two or eight units per
// thread (their loads in flight together): an integer min over its threads finds the chunk's first
// non-correct unit, the units before it join the lexicographic min of
// (value, index), and the first chunk that has one ends the search.  The pick is
// exact and deterministic.
#include <climits>

#include "common.hpp"

namespace stride {
namespace {

// Where the average rollout has at most 128 units, one wave takes each record of up to kWaveLength units
// (two of its chunks of 512) and kHelpers workgroups of the same launch the longer ones: 40,000 units
// before 1,500 rollouts of 3 took a wave 161 us and take a helper 24.5 (one workgroup of 256 for every
// rollout and two passes: 43.7).  A prime number of helpers, so that long rollouts at regular places are
// spread over them.
constexpr int64_t kWaveLength = 1024;
constexpr int kHelpers = 127;

struct RestartArgs {
    stride_layout L;
    DomainTable alpha;
    int32_t n_dom;
    int32_t unit;
    const void *values;
    const int32_t *stop_unit;
    const uint8_t *mask;
    int32_t *k_star;
    int32_t *k0;
    int32_t *k_max;
    uint32_t *flags;
};

// A rollout's record: its first unit and its length, -1 where the offsets or the domain are bad.
struct Record {
    int64_t first, len;
    double alpha;
};

// With `report`, a rollout without a record gets its results and flag here.
__device__ __forceinline__ Record record_of(const RestartArgs &a, int64_t r, bool report) {
    const int64_t T = a.L.n_turns;
    const int64_t t0 = a.L.rollout_turn_off[r], t1 = a.L.rollout_turn_off[r + 1];
    const int32_t d = a.L.domain ? a.L.domain[r] : 0, s = a.stop_unit ? a.stop_unit[r] : -1;
    bool bad_off = t0 < 0 || t1 > T || t1 < t0;
    int64_t first = 0, n = 0;
    if (!bad_off) {
        if (a.unit == STRIDE_UNIT_TURN) {
            first = t0;
            n = t1 - t0;
        } else {
            first = a.L.turn_tok_off[t0];
            n = a.L.turn_tok_off[t1] - first;
            bad_off = first < 0 || n < 0 || first + n > a.L.n_tokens;
        }
    }
    const bool bad_dom = d < 0 || d >= a.n_dom;
    if (bad_off || bad_dom) {
        if (report) {
            a.k_star[r] = -1;
            a.k0[r] = 0;
            if (a.k_max) a.k_max[r] = 0;
            raise_flag(a.flags, bad_off ? STRIDE_FLAG_BAD_OFFSETS : STRIDE_FLAG_BAD_DOMAIN);
        }
        return Record{0, -1, 0.0};
    }
    return Record{first, s >= 0 && (int64_t)s + 1 < n ? (int64_t)s + 1 : n, a.alpha.v[d]};
}

// One rollout by NT threads (tid their number), PU units each at a time; with more than one wave
// they meet at workgroup barriers.  K_max = first non-correct unit in [0, len), else len; k* = lowest
// index of the minimum over [0, K_max).
template <typename VT, int NT, int PU>
__device__ __forceinline__ void pick(const RestartArgs &a, int64_t r, const Record &rec, int tid,
                                     int64_t *s_min, double *s_val, int64_t *s_idx) {
    constexpr int kWaves = NT / kWave;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t first = rec.first, len = rec.len;
    const double alpha = rec.alpha;
    const VT *vals = static_cast<const VT *>(a.values);
    int64_t kmax = len;
    if (kWaves > 1) {
        if (tid == 0) *s_min = len;
        __syncthreads();
    }
    double best = __builtin_inf();
    int64_t bidx = LLONG_MAX;
    VT v[PU], v2[PU];
    uint8_t mk[PU], mk2[PU];
    auto fetch = [&](int64_t c, VT *x, uint8_t *m) __attribute__((always_inline)) {
        if (c >= len) return;
        // Past the record's end its last unit is read again, so that no load waits for a bound, and the mask
        // is looked for once for all: 64 records of 4,096 units with a mask 5.7 us (a branch for each load
        // 6.0, and 6.3 where the records are ragged), 500,000 before 10,000 of 2 314 (the mask looked for at
        // each load 494).
        const int last = len - c > NT * PU ? NT * PU - 1 : (int)(len - c) - 1;
        const VT *p = vals + first + c;
#pragma unroll
        for (int k = 0; k < PU; ++k) x[k] = p[k * NT + tid < last ? k * NT + tid : last];
#pragma unroll
        for (int k = 0; k < PU; ++k) m[k] = 1;
        if (a.mask) {
            const uint8_t *q = a.mask + first + c;
#pragma unroll
            for (int k = 0; k < PU; ++k) m[k] = q[k * NT + tid < last ? k * NT + tid : last];
        }
    };
    constexpr bool kAhead = NT > 256;  // the next chunk's values in flight while this one is looked at
    if (kAhead) fetch(0, v, mk);
    for (int64_t c = 0; c < len; c += (int64_t)NT * PU) {
        if (kAhead)
            fetch(c + (int64_t)NT * PU, v2, mk2);
        else
            fetch(c, v, mk);
        int64_t wrong = LLONG_MAX;
#pragma unroll
        for (int k = PU - 1; k >= 0; --k) {
            const int64_t u = c + (int64_t)k * NT + tid;
            if (u < len && !(mk[k] != 0 && (double)v[k] > alpha)) wrong = u;
        }
        if (kWaves == 1) {
#pragma unroll
            for (int o = kWave / 2; o > 0; o >>= 1) {
                const int64_t w = __shfl_xor(wrong, o, kWave);
                wrong = w < wrong ? w : wrong;
            }
            kmax = wrong < len ? wrong : len;
        } else {
            if (wrong != LLONG_MAX) atomicMin((unsigned long long *)s_min, (unsigned long long)wrong);
            __syncthreads();
            kmax = *s_min;
        }
#pragma unroll
        for (int k = 0; k < PU; ++k) {
            const int64_t u = c + (int64_t)k * NT + tid;
            // u increases, so the first hit per thread is its lowest index; the first unit
            // always counts, so values of +inf still give an index
            if (u < kmax && ((double)v[k] < best || bidx == LLONG_MAX)) {
                best = (double)v[k];
                bidx = u;
            }
        }
        if (kmax < len) break;
        if (kAhead) {
#pragma unroll
            for (int k = 0; k < PU; ++k) {
                v[k] = v2[k];
                mk[k] = mk2[k];
            }
        }
        if (kWaves > 1) __syncthreads();  // s_min is read by all before any updates it again
    }

#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double b2 = __shfl_xor(best, off, kWave);
        const int64_t i2 = __shfl_xor(bidx, off, kWave);
        if (b2 < best || (b2 == best && i2 < bidx)) {
            best = b2;
            bidx = i2;
        }
    }
    if (kWaves > 1) {
        if (lane == 0) {
            s_val[wave] = best;
            s_idx[wave] = bidx;
        }
        __syncthreads();
    }
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w) {
            if (s_val[w] < best || (s_val[w] == best && s_idx[w] < bidx)) {
                best = s_val[w];
                bidx = s_idx[w];
            }
        }
        const int32_t ks = kmax > 0 ? (int32_t)bidx : -1;
        a.k_star[r] = ks;
        a.k0[r] = ks > 0 ? ks : 0;
        if (a.k_max) a.k_max[r] = (int32_t)kmax;
    }
}

// NT threads per rollout, by the rollouts' average length: one wave of a 256-thread workgroup
// up to 128 units, a workgroup of 256 up to 1,024, of 512 above (which also has the next chunk's
// values in flight: 5.4 us against 5.0 where 256 threads need no second chunk).  Latency bounds
// the kernels (a chunk costs a round trip to memory and two barriers), and for many short rollouts
// the number of workgroups.  Measured against 256 threads for every rollout and two passes:
// 8 x 16,384 units 28.1 -> 9.9 us with a mask and 24.3 -> 9.5 without (graph replays, the whole record
// correct), 64 x 4,096 9.3 -> 5.7, 500 x 500 5.5 -> 4.5, 8 x 8 4.7 -> 3.6, 20,000 x 12 39.5 -> 10.7,
// 200,000 x 3 392 -> 83.  1,024 threads are ahead at 8 x 16,384 and 1.9 us behind where the first chunk ends
// the search.
//
// One wave per rollout, four to a workgroup, behind `helpers` workgroups that take the records of more
// than kWaveLength units, which the waves pass over: helper k looks at rollouts k, k + helpers, ...
template <typename VT>
__global__ __launch_bounds__(256) void restart_waves_kernel(RestartArgs a, int helpers) {
    constexpr int kWaves = 256 / kWave;
    __shared__ int64_t s_min, s_idx[kWaves];
    __shared__ double s_val[kWaves];
    __shared__ int32_t s_count;
    __shared__ int32_t s_long[256];
    const int64_t R = a.L.n_rollouts;
    const int tid = threadIdx.x;
    if (block_index<256>() >= helpers) {
        const int64_t r = (block_index<256>() - helpers) * kWaves +
                          __builtin_amdgcn_readfirstlane(tid / kWave);
        if (r >= R) return;
        const Record rec = record_of(a, r, tid % kWave == 0);
        if (rec.len < 0 || rec.len > kWaveLength) return;
        if (rec.len <= 2 * kWave)
            pick<VT, kWave, 2>(a, r, rec, tid % kWave, nullptr, nullptr, nullptr);
        else
            pick<VT, kWave, 8>(a, r, rec, tid % kWave, nullptr, nullptr, nullptr);
        return;
    }
    const int64_t step = (int64_t)helpers * 256;
    for (int64_t base = blockIdx.x; base < R; base += step) {
        if (tid == 0) s_count = 0;
        __syncthreads();
        const int64_t r = base + (int64_t)tid * helpers;
        if (r < R) {
            if (record_of(a, r, false).len > kWaveLength) s_long[atomicAdd(&s_count, 1)] = (int32_t)r;
        }
        __syncthreads();
        const int n = s_count;
        for (int i = 0; i < n; ++i) {
            int t = tid;
            asm volatile("" : "+v"(t));  // opaque: addresses formed once for all records cost registers
            const int64_t far = __builtin_amdgcn_readfirstlane(s_long[i]);
            pick<VT, 256, 8>(a, far, record_of(a, far, false), t, &s_min, s_val, s_idx);
            __syncthreads();  // the shared values are read by all before the next record's are written
        }
    }
}

template <typename VT, int NT>
__global__ __launch_bounds__(NT) void restart_block_kernel(RestartArgs a) {
    __shared__ int64_t s_min, s_idx[NT / kWave];
    __shared__ double s_val[NT / kWave];
    const int64_t r = block_index<NT>();
    if (r >= a.L.n_rollouts) return;
    const Record rec = record_of(a, r, threadIdx.x == 0);
    if (rec.len < 0) return;
    // half the chunk where it holds the record: 300 records of 250 units or of 1,024 5.2 -> 4.4 us
    if (NT == 256 && rec.len <= 4 * NT)
        pick<VT, NT, 4>(a, r, rec, threadIdx.x, &s_min, s_val, s_idx);
    else
        pick<VT, NT, 8>(a, r, rec, threadIdx.x, &s_min, s_val, s_idx);
}

template <typename VT>
void launch_restart_groups(const RestartArgs &a, int64_t R, int64_t n_units, hipStream_t stream) {
    const int64_t per = n_units / R;
    if (per <= 128) {
        // no record is longer than the call
        const int helpers = n_units <= kWaveLength ? 0 : (R < kHelpers ? (int)R : kHelpers);
        hipLaunchKernelGGL(restart_waves_kernel<VT>, grid_of((R + 3) / 4 + helpers, 256), dim3(256), 0, stream, a, helpers);
    } else if (per <= 1024)
        hipLaunchKernelGGL((restart_block_kernel<VT, 256>), grid_of(R, 256), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((restart_block_kernel<VT, 512>), grid_of(R, 512), dim3(512), 0, stream, a);
}

}  // namespace

hipError_t launch_restart(const stride_layout &L, int32_t unit, const void *values,
                          const int32_t *stop_unit, const DomainTable &alpha, int32_t n_dom,
                          const uint8_t *mask, int32_t *k_star, int32_t *k0, int32_t *k_max,
                          uint32_t *flags, hipStream_t stream) {
    if (L.n_rollouts == 0) return hipSuccess;
    RestartArgs a;
    a.L = L;
    a.alpha = alpha;
    a.n_dom = n_dom;
    a.unit = unit;
    a.values = values;
    a.stop_unit = stop_unit;
    a.mask = mask;
    a.k_star = k_star;
    a.k0 = k0;
    a.k_max = k_max;
    a.flags = flags;
    const int64_t n_units = unit == STRIDE_UNIT_TURN ? L.n_turns : L.n_tokens;
    const int64_t R = L.n_rollouts;
    if (unit == STRIDE_UNIT_TURN)
        launch_restart_groups<double>(a, R, n_units, stream);
    else
        launch_restart_groups<float>(a, R, n_units, stream);
    return hipGetLastError();
}

}  // namespace stride
