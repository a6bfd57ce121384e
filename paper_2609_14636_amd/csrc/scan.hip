// scan.hip -- the early-stop test: per-rollout cumulative sums and first crossing.
//
// Eq. (5) (Sec. 4.1): stop at the first unit K* whose cumulative value is
// strictly below lambda; with a reused prefix of K0 units the sum starts at
// unit K0 (Sec. 4.1, prefix-buffer synergy; Algorithm 1).  Units are turns
// (values = lbar_k, Eq. 4) or tokens (values = teacher log-probabilities, the
// single-turn variant of Sec. 5.5), so one rollout can hold tens of thousands
// of units.
//
// Single-pass segmented scan (Merrill and Garland, "Single-pass Parallel Prefix
// Scan with Decoupled Look-back", 2016), specialised for determinism:
//   1. A workgroup takes the next tile id from a counter (tiles start in id
//      order, so every tile waited on is already running: forward progress).
//   2. It loads 2048 units, zeroes those before K0, and scans them in double
//      (per-thread sequential, then a fixed shuffle tree, then waves in order),
//      with the segmented operator (f1,v1)+(f2,v2) = (f1|f2, f2 ? v2 : v1+v2).
//   3. It publishes its aggregate (value after its last rollout start, and
//      whether one occurs) in two self-contained words, before waiting on anything.
//   4. If its first unit continues a rollout, it looks back over predecessor
//      aggregates only, 64 at a time, added nearest first, until the tile holding
//      that rollout's start.  Inclusive prefixes are never used, so every sum is
//      associated in the same order on every run: cum is bit-reproducible.
//   5. The first crossing per rollout is an integer min, reduced in LDS and
//      then with one global atomicMin per rollout per tile.
// Calls of up to 2^19 units, 2^15 rollouts and 2^15 units for each on average need none of this: a group
// of threads takes each rollout, in one launch (stop_waves_kernel, stop_block_kernel).
// Waits are bounded: past the spin limit the tile gives up, raises
// STRIDE_FLAG_SPIN_LIMIT and writes NaN, so no wave can hang.
#include <atomic>
#include <climits>
#include <mutex>

#include "common.hpp"

namespace stride {
namespace {

constexpr int kSlots = 256;            // rollouts per tile held in LDS
// Units of the call and of its average rollout, and rollouts, up to which each gets a group of threads
// of its own (one launch) instead of the tiles' three launches.  The whole test, tiles -> groups:
// 8 x 8 units 17.7 -> 3.6 us, 2,000 x 12 24.2 -> 4.7, 64 x 4,096 25.6 -> 7.3, 2 x 30,000 23.4 -> 15.9.
// A group scans its rollout alone, where tiles spread it over the chip: one rollout of 172,000 units
// takes 61.6 us as a group and 20.4 as tiles, one of 516,000 196 and 29.5.  The host does not know the
// longest rollout, so the call's own limit bounds what one long rollout among short ones can cost:
// about 0.5 us for every 1,024 units (scan_long), 285 us at 500,000.  Short rollouts cost a workgroup
// for every four: 32,768 of 8 units take 14.9 us against the tiles' 31.9, 100,000 of 3 36.1 against
// 32.9, 200,000 of 2 77 against 35.7.
constexpr int64_t kRolloutUnits = 1 << 19;
constexpr int64_t kRolloutLength = 1 << 15;
constexpr int64_t kRolloutCount = 1 << 15;
// Where the average rollout has at most 128 units, one wave takes each of up to kWaveLength units, eight
// of its chunks, and kHelpers workgroups of the same launch the longer ones.  A wave walks 128 units a
// chunk: 40,000 units before 1,500 rollouts of 3 took it 96 us, a helper 23.7 (the tiles of before 26);
// 1,200 before 30 of 5 take 5.9 us either way.  A prime number of helpers, so that long rollouts at
// regular places are spread over them.
constexpr int64_t kWaveLength = 1024;
constexpr int kHelpers = 127;
constexpr uint32_t kSpinLimit = 1u << 22;

struct StopArgs {
    stride_layout L;
    DomainTable lambda;
    int32_t n_dom;
    int32_t unit;
    int64_t n_units;
    int64_t n_tiles;
    const void *values;
    const int32_t *start;
    const int64_t *unit_off;  // [R+1] in the workspace
    double *cum;
    int32_t *stop_unit;
    int64_t *retained;
    uint32_t *counter;
    TileDesc *desc;
    uint32_t *flags;
    // Test hook (the library built with STRIDE_SCAN_DELAY_HOOK only): tiles picked by a
    // seeded hash sleep a bounded time before publishing their aggregate, so successors
    // must wait on unpublished descriptors.  Zero in the product build.
    uint64_t delay_seed;
    uint32_t delay_one_in;
    uint32_t delay_sleeps;
    // Test hook, same build only: a look-back wait bound other than kSpinLimit (0: kSpinLimit),
    // so that the give-up path can be forced from the host.
    uint32_t spin_limit;
};

#ifdef STRIDE_SCAN_DELAY_HOOK
std::atomic<uint64_t> g_delay_seed{0};
std::atomic<uint32_t> g_delay_one_in{0};
std::atomic<uint32_t> g_delay_sleeps{0};
std::atomic<uint32_t> g_spin_limit{0};
#endif

struct Seg {
    uint32_t f;
    double v;
};

__device__ __forceinline__ Seg combine(Seg a, Seg b) {
    return Seg{a.f | b.f, b.f ? b.v : a.v + b.v};
}

__device__ __forceinline__ int64_t find_rollout(const int64_t *off, int64_t R, int64_t u) {
    // last r in [0, R) with off[r] <= u; -1 if none
    if (R == 0 || off[0] > u) return -1;
    int64_t lo = 0, hi = R;
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (off[mid] <= u) lo = mid; else hi = mid;
    }
    return lo;
}

// What the stop test writes for a rollout: stop_unit (sentinel -> -1), retained rows, bad domains.
// s: first crossing or INT_MAX; [first, first + n) its units.
__device__ __forceinline__ void finish_rollout(const StopArgs &a, int64_t r, int32_t s,
                                               int64_t first, int64_t n) {
    const int32_t d = a.L.domain ? a.L.domain[r] : 0;
    if (d < 0 || d >= a.n_dom) raise_flag(a.flags, STRIDE_FLAG_BAD_DOMAIN);
    if (s == INT_MAX) s = -1;
    a.stop_unit[r] = s;
    if (!a.retained) return;
    if (n < 0) n = 0;
    int64_t k0 = a.start ? (int64_t)a.start[r] : 0;
    k0 = k0 < 0 ? 0 : (k0 > n ? n : k0);
    int64_t end = (s >= 0) ? (int64_t)s + 1 : n;
    if (end < k0) end = k0;
    if (a.unit == STRIDE_UNIT_TOKEN) {
        a.retained[r] = end - k0;
    } else {
        const int64_t T = a.L.n_turns;
        int64_t t0 = first + k0, t1 = first + end;
        t0 = t0 > T ? T : t0;
        t1 = t1 > T ? T : t1;
        a.retained[r] = a.L.turn_tok_off[t1] - a.L.turn_tok_off[t0];
    }
}

// First unit of rollout i (i = R: the end of the last), from the layout; raises BAD_OFFSETS.
__device__ __forceinline__ int64_t first_unit(const StopArgs &a, int64_t i) {
    const int64_t R = a.L.n_rollouts, T = a.L.n_turns;
    int64_t t = a.L.rollout_turn_off[i];
    bool bad = t < 0 || t > T;
    if (i == 0 && t != 0) bad = true;
    if (i == R && t != T) bad = true;
    if (i < R && a.L.rollout_turn_off[i + 1] < t) bad = true;
    t = t < 0 ? 0 : (t > T ? T : t);
    if (bad) raise_flag(a.flags, STRIDE_FLAG_BAD_OFFSETS);
    return (a.unit == STRIDE_UNIT_TURN) ? t : a.L.turn_tok_off[t];
}

// unit_off, stop_unit sentinels, descriptor reset, tile counter reset.
__global__ __launch_bounds__(256) void stop_prep_kernel(StopArgs a, int64_t *unit_off) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= a.L.n_rollouts) unit_off[i] = first_unit(a, i);
    if (i < a.L.n_rollouts) a.stop_unit[i] = INT_MAX;
    if (i < a.n_tiles) a.desc[i] = TileDesc{0, 0};
    if (i == 0) *a.counter = 0;
}

// Tile descriptor: the aggregate's 64 bits in two words, each with its own tag (bit 0:
// published, bit 1: a rollout starts in the tile) in the low half.  Each word is valid by
// itself, so relaxed stores and loads suffice: no fence orders them, and none empties a cache.
__device__ __forceinline__ void publish(TileDesc *d, double value, uint32_t head) {
    const uint64_t v = (uint64_t)__double_as_longlong(value), tag = 1u | (head << 1);
    __hip_atomic_store(&d->hi, (v & 0xFFFFFFFF00000000ull) | tag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&d->lo, (v << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The carry into tile `tile` (called by its first wave): the aggregates of its predecessors,
// added nearest first down to the first one that holds a rollout's start.  The lanes read 64
// descriptors at once -- one round trip to memory where a walk takes one per tile -- and wait
// only for those up to the nearest start; the additions keep the walk's order.
__device__ __forceinline__ double look_back(const StopArgs &a, int64_t tile, int lane) {
#ifdef STRIDE_SCAN_DELAY_HOOK
    const uint32_t limit = a.spin_limit ? a.spin_limit : kSpinLimit;
#else
    constexpr uint32_t limit = kSpinLimit;
#endif
    double carry = 0.0;
    for (int64_t base = tile - 1; base >= 0; base -= kWave) {
        const int64_t p = base - lane;
        bool ready = p < 0;  // lanes past tile 0 hold nothing
        uint64_t hi = 0, lo = 0;
        uint32_t spins = 0;
        int need;
        bool found;
        for (;;) {
            if (!ready) {
                hi = __hip_atomic_load(&a.desc[p].hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lo = __hip_atomic_load(&a.desc[p].lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ready = (hi & 1) && (lo & 1);
            }
            const uint64_t done = __ballot(ready);
            const uint64_t heads = __ballot(ready && (hi & 2));
            found = heads != 0;
            need = found ? __builtin_ctzll(heads) + 1 : kWave;
            const uint64_t upto = need == kWave ? ~0ull : (1ull << need) - 1;
            if ((done & upto) == upto) break;
            if (++spins > limit) {
                if (lane == 0) raise_flag(a.flags, STRIDE_FLAG_SPIN_LIMIT);
                return __builtin_nan("");
            }
            __builtin_amdgcn_s_sleep(1);
        }
        const uint64_t v = (hi & 0xFFFFFFFF00000000ull) | (lo >> 32);
        const int n = base + 1 < need ? (int)(base + 1) : need;
        for (int i = 0; i < n; ++i) {
            const uint32_t vh = __builtin_amdgcn_readlane((uint32_t)(v >> 32), i);
            const uint32_t vl = __builtin_amdgcn_readlane((uint32_t)v, i);
            carry = __longlong_as_double((long long)(((uint64_t)vh << 32) | vl)) + carry;
        }
        if (found) break;
    }
    return carry;
}

// One workgroup per tile of kScanTile units, between stop_prep_kernel and stop_finish_kernel.
// Latency bounds it (a tile reads 8 or 16 KB): the offsets, K0 and thresholds of the tile's
// rollouts are fetched once into LDS (the first kSlots of them; rollouts past those come from
// memory), so the searches and the per-unit tests make no dependent global loads.
template <typename VT>
__global__ __launch_bounds__(kScanThreads) void stop_scan_kernel(StopArgs a) {
    constexpr int kCap = kSlots;
    __shared__ int64_t s_tile;
    __shared__ Seg s_wave[kScanThreads / kWave];
    __shared__ double s_carry;
    __shared__ int32_t s_first[kCap];
    __shared__ int64_t s_off[kCap + 1];
    __shared__ int64_t s_k0[kCap];
    __shared__ double s_lam[kCap];
    __shared__ int64_t s_r0;

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t R = a.L.n_rollouts;
    const VT *vals = static_cast<const VT *>(a.values);
    if (tid == 0) s_tile = (int64_t)atomicAdd(a.counter, 1u);
    __syncthreads();
    const int64_t tile = s_tile;
    const int64_t u0 = tile * kScanTile;
    const int64_t ubase = u0 + (int64_t)tid * kScanItems;
    VT in[kScanItems];
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) in[j] = ubase + j < a.n_units ? vals[ubase + j] : (VT)0;

    // ---- the tile's rollouts ----
    if (wave == 0) {  // last rollout with unit_off <= u0, 64 pivots at a time; -1 if none
        int64_t lo = -1;
        if (R > 0 && a.unit_off[0] <= u0) {
            lo = 0;
            for (int64_t hi = R; hi - lo > 1;) {
                const int64_t step = (hi - lo + kWave - 1) / kWave, i = lo + lane * step;
                const uint64_t le = __ballot(i < hi && a.unit_off[i] <= u0);
                lo += (63 - __builtin_clzll(le)) * step;  // lane 0's pivot is always <= u0
                hi = lo + step < hi ? lo + step : hi;
            }
        }
        if (lane == 0) s_r0 = lo;
    }
    __syncthreads();
    const int64_t r0 = s_r0, rb = r0 < 0 ? 0 : r0;  // rb: rollout of LDS entry 0
    for (int i = tid; i <= kCap; i += kScanThreads) s_off[i] = a.unit_off[rb + i < R ? rb + i : R];
    auto off = [&](int64_t r) -> int64_t {
        return r - rb <= kCap ? s_off[r - rb] : a.unit_off[r];
    };
    auto prefix = [&](int64_t r, int64_t n) -> int64_t {  // K0 of rollout r, clamped
        const int64_t k0 = a.start ? (int64_t)a.start[r] : 0;
        return k0 < 0 ? 0 : (k0 > n ? n : k0);
    };
    auto limit = [&](int64_t r) -> double {
        const int32_t d = a.L.domain ? a.L.domain[r] : 0;
        return (d >= 0 && d < a.n_dom) ? a.lambda.v[d] : __builtin_nan("");
    };
    __syncthreads();
    const int cnt = R - rb < kCap ? (int)(R - rb) : kCap;
    for (int i = tid; i < cnt; i += kScanThreads) {
        s_first[i] = INT_MAX;
        s_k0[i] = prefix(rb + i, s_off[i + 1] - s_off[i]);
        s_lam[i] = limit(rb + i);
    }
    __syncthreads();
    // last rollout that starts at or before this thread's first unit, -1 if none
    int64_t r = -1;
    if (cnt > 0 && s_off[0] <= ubase) {
        int lo = 0, hi = cnt;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_off[mid] <= ubase) lo = mid; else hi = mid;
        }
        r = rb + lo;
        if (lo == kCap - 1 && r + 1 < R) r += find_rollout(a.unit_off + r, R - r, ubase);
    }

    // ---- thread-local segmented scan ----
    double run[kScanItems];
    bool head[kScanItems];
    int64_t rr[kScanItems];
    Seg tagg{0u, 0.0};
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t u = ubase + j;
        double v = 0.0;
        bool h = false;
        int64_t rj = -1;  // rollout holding unit u, -1 if none (only with bad offsets)
        if (u < a.n_units) {
            // on to the last rollout that starts at or before u (from -1 on where the first starts late),
            // in steps that double, since most of the rollouts on the way can be empty
            if (r + 1 < R && off(r + 1) <= u) {
                int64_t next = R;
                ++r;
                for (int64_t step = 1; r + step < R; step <<= 1) {
                    if (off(r + step) > u) {
                        next = r + step;
                        break;
                    }
                    r += step;
                }
                while (next - r > 1) {
                    const int64_t mid = (r + next) >> 1;
                    if (off(mid) <= u) r = mid; else next = mid;
                }
            }
            const int64_t first = r >= 0 ? off(r) : 0, n = r >= 0 ? off(r + 1) - first : 0, local = u - first;
            if (local >= 0 && local < n) {
                const int64_t k0 = r - rb < kCap ? s_k0[r - rb] : prefix(r, n);
                h = (local == 0);
                if (local >= k0) v = (double)in[j];
                rj = r;
            }
        }
        rr[j] = rj;
        head[j] = h;
        tagg = combine(tagg, Seg{h, v});
        run[j] = tagg.v;
    }

    // ---- block-level exclusive scan of the thread aggregates ----
    Seg inc = tagg;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t f2 = __shfl_up(inc.f, o, kWave);
        const double v2 = __shfl_up(inc.v, o, kWave);
        if (lane >= o) inc = combine(Seg{f2, v2}, inc);
    }
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    Seg wpre{0u, 0.0};
    for (int w = 0; w < wave; ++w) wpre = combine(wpre, s_wave[w]);
    Seg excl;
    {
        const uint32_t f2 = __shfl_up(inc.f, 1, kWave);
        const double v2 = __shfl_up(inc.v, 1, kWave);
        excl = (lane == 0) ? wpre : combine(wpre, Seg{f2, v2});
    }

    // ---- publish the tile aggregate, then look back ----
    if (wave == 0) {
        if (lane == 0) {
            Seg total{0u, 0.0};
            for (int w = 0; w < kScanThreads / kWave; ++w) total = combine(total, s_wave[w]);
#ifdef STRIDE_SCAN_DELAY_HOOK
            if (a.delay_one_in) {
                // splitmix64 step (Steele, Lea and Flood 2014) of (seed, tile): picks the
                // tile and its sleep count
                uint64_t z = a.delay_seed + 0x9E3779B97F4A7C15ull * (uint64_t)(tile + 1);
                z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
                z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
                z ^= z >> 31;
                if ((z % a.delay_one_in) == 0) {
                    const uint32_t n = 1 + (uint32_t)((z >> 32) % a.delay_sleeps);
                    for (uint32_t i = 0; i < n; ++i) __builtin_amdgcn_s_sleep(127);
                }
            }
#endif
            publish(&a.desc[tile], total.v, total.f);
        }
        double c = 0.0;
        if (tile > 0 && r0 >= 0 && s_off[0] < u0) c = look_back(a, tile, lane);
        if (lane == 0) s_carry = c;
    }
    __syncthreads();
    const double carry = s_carry;

    // ---- cumulative values and first crossings ----
    bool seen = excl.f != 0, head_in_thread = false;
    int64_t last_r = -2;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        const int64_t u = ubase + j;
        if (u >= a.n_units) break;
        const int64_t rj = rr[j];
        seen |= head[j];
        head_in_thread |= head[j];
        double c;
        if (rj < 0) {
            c = __builtin_nan("");
        } else {
            // thread-local running sum restarted at a head inside this thread's items
            c = head_in_thread ? run[j] : excl.v + run[j];
            if (!seen) c += carry;
        }
        a.cum[u] = c;
        if (rj < 0 || rj == last_r) continue;
        const int64_t i = rj - rb, first = off(rj), local = u - first;
        const bool in_lds = i < kCap;
        const int64_t k0 = in_lds ? s_k0[i] : prefix(rj, off(rj + 1) - first);
        if (local >= k0 && c < (in_lds ? s_lam[i] : limit(rj))) {
            last_r = rj;  // later units of this rollout in this thread cannot be earlier
            if (in_lds)
                atomicMin(&s_first[i], (int32_t)local);
            else
                atomicMin(&a.stop_unit[rj], (int32_t)local);
        }
    }
    __syncthreads();
    for (int i = tid; i < cnt; i += kScanThreads)
        if (s_first[i] != INT_MAX) atomicMin(&a.stop_unit[rb + i], s_first[i]);
}

__global__ __launch_bounds__(256) void stop_finish_kernel(StopArgs a) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= a.L.n_rollouts) return;
    finish_rollout(a, r, a.stop_unit[r], a.unit_off[r], a.unit_off[r + 1] - a.unit_off[r]);
}

// x + the lane's source under a data-parallel-primitive move (0 where the move has no source).
template <int kCtrl, int kRows>
__device__ __forceinline__ double moved(double x) {
    const uint64_t v = (uint64_t)__double_as_longlong(x);
    const uint32_t l = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, kCtrl, kRows, 0xF, false);
    const uint32_t h = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), kCtrl, kRows, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)h << 32) | l));
}

// Inclusive sum over the wave: within rows of 16 lanes (row_shr 1, 2, 4, 8), then row ends into
// the next row (row_bcast 15) and the lower half's end into the upper half (row_bcast 31).
// These moves are vector instructions, where __shfl_up goes through the LDS unit.  With loads and
// stores of one unit each, it took 8.1 us for a chunk of 8,192 units; both changed, 3.0.
__device__ __forceinline__ double wave_scan(double x) {
    x += moved<0x111, 0xF>(x);
    x += moved<0x112, 0xF>(x);
    x += moved<0x114, 0xF>(x);
    x += moved<0x118, 0xF>(x);
    x += moved<0x142, 0xA>(x);
    x += moved<0x143, 0xC>(x);
    return x;
}

typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));

// The last lane's x, in scalar registers.
__device__ __forceinline__ double last_lane(double x) {
    const uint64_t v = (uint64_t)__double_as_longlong(x);
    const uint32_t h = __builtin_amdgcn_readlane((uint32_t)(v >> 32), kWave - 1);
    const uint32_t l = __builtin_amdgcn_readlane((uint32_t)v, kWave - 1);
    return __longlong_as_double((long long)(((uint64_t)h << 32) | l));
}

// Up to N consecutive elements from p on (p + j < end), as few loads as their number allows; the
// addresses have the element's own alignment only, which global loads of several words accept.
template <typename VT, int N, typename I>
__device__ __forceinline__ void load_items(const VT *vals, I u, I hi, VT *x) {
    constexpr int kPer = 16 / sizeof(VT) < N ? 16 / sizeof(VT) : N;
    typedef VT Vec __attribute__((ext_vector_type(kPer), aligned(sizeof(VT))));
    if (u + N <= hi) {
#pragma unroll
        for (int j = 0; j < N; j += kPer) {
            const Vec v = *reinterpret_cast<const Vec *>(vals + u + j);
#pragma unroll
            for (int i = 0; i < kPer; ++i) x[j + i] = v[i];
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = u + j < hi ? vals[u + j] : (VT)0;
    }
}

// A rollout as its group sees it: [lo, hi) its units inside [0, U), `from` the first one after K0.
struct Rollout {
    int64_t r, first, n, lo, from, hi;
    double lam;
};

__device__ __forceinline__ Rollout rollout_of(const StopArgs &a, int64_t r, bool report) {
    const int64_t R = a.L.n_rollouts, T = a.L.n_turns, U = a.n_units;
    const int64_t t0 = a.L.rollout_turn_off[r], t1 = a.L.rollout_turn_off[r + 1];
    const int32_t start = a.start ? a.start[r] : 0, d = a.L.domain ? a.L.domain[r] : 0;
    if (report && (t0 < 0 || t0 > T || (r == 0 && t0 != 0) || t1 < t0 || (r == R - 1 && t1 != T)))
        raise_flag(a.flags, STRIDE_FLAG_BAD_OFFSETS);
    int64_t first = t0 < 0 ? 0 : (t0 > T ? T : t0), last = t1 < 0 ? 0 : (t1 > T ? T : t1);
    if (a.unit == STRIDE_UNIT_TOKEN) {
        first = a.L.turn_tok_off[first];
        last = a.L.turn_tok_off[last];
    }
    Rollout o;
    o.r = r;
    o.first = first;
    o.n = last - first;
    int64_t k0 = start;
    k0 = k0 < 0 ? 0 : (k0 > o.n ? o.n : k0);
    o.lam = (d >= 0 && d < a.n_dom) ? a.lambda.v[d] : __builtin_nan("");
    // offsets that do not cover [0, U) or leave it (flagged where they are not the caller's own
    // row offsets): units in no rollout are NaN, and no access leaves [0, U)
    o.lo = first < 0 ? 0 : first;
    o.hi = last > U ? U : last;
    o.from = first + k0 < o.lo ? o.lo : first + k0;
    return o;
}

// NaN for the units before the first rollout's and past the last one's, 0 for those before K0; tid and
// NT: the number and count of the threads that share the rollout.
__device__ __forceinline__ void fill_outside(const StopArgs &a, const Rollout &o, int tid, int NT) {
    const int64_t U = a.n_units;
    if (o.r == 0)
        for (int64_t u = tid; u < o.first && u < U; u += NT) a.cum[u] = __builtin_nan("");
    if (o.r == a.L.n_rollouts - 1)
        for (int64_t u = (o.first + o.n < 0 ? 0 : o.first + o.n) + tid; u < U; u += NT)
            a.cum[u] = __builtin_nan("");
    for (int64_t u = o.lo + tid; u < o.from && u < o.hi; u += NT) a.cum[u] = 0.0;
}

// The lowest first crossing of a group's threads, and the rollout's results.
template <int NT>
__device__ __forceinline__ void finish_group(const StopArgs &a, const Rollout &o, int tid, int32_t best,
                                             int32_t *s_best) {
    constexpr int kWaves = NT / kWave;
#pragma unroll
    for (int q = kWave / 2; q > 0; q >>= 1) {
        const int32_t b = __shfl_xor(best, q, kWave);
        best = b < best ? b : best;
    }
    if (kWaves > 1) {
        if (tid % kWave == 0) s_best[tid / kWave] = best;
        __syncthreads();
        if (tid == 0)
            for (int w = 1; w < kWaves; ++w) best = s_best[w] < best ? s_best[w] : best;
    }
    if (tid == 0) finish_rollout(a, o.r, best, o.first, o.n);
}

// The whole test of one rollout by NT threads (tid their number), NI units each at a time.  The units
// run through a fixed scan (a thread's items in order, a tree over the lanes, waves in order, chunks
// in order), so cum is bit-reproducible; the next chunk's values are in flight while one is scanned.
// All NT threads call it together; with more than one wave they meet at workgroup barriers.
template <typename VT, int NT, int NI>
__device__ __forceinline__ void scan_rollout(const StopArgs &a, const Rollout &o, int tid,
                                             double (*s_sum)[NT / kWave], int32_t *s_best) {
    constexpr int kWaves = NT / kWave;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int64_t first = o.first, hi = o.hi, from = o.from;
    const VT *vals = static_cast<const VT *>(a.values);
    const double lam = o.lam;
    fill_outside(a, o, tid, NT);

    constexpr int64_t kChunk = (int64_t)NT * NI;
    double carry = 0.0;
    int32_t best = INT_MAX;
    VT in[NI];
    const int64_t mine = (int64_t)tid * NI;
    load_items<VT, NI>(vals, from + mine, hi, in);
    int buf = 0;
    for (int64_t base = from; base < hi; base += kChunk, buf ^= 1) {
        const int64_t u0 = base + mine;
        VT next[NI];
        load_items<VT, NI>(vals, u0 + kChunk, hi, next);
        double run[NI];
        run[0] = (double)in[0];
#pragma unroll
        for (int j = 1; j < NI; ++j) run[j] = run[j - 1] + (double)in[j];
        const double inc = wave_scan(run[NI - 1]);
        double pre = moved<0x138, 0xF>(inc), total;  // wave_shr 1: the lanes before this one
        if (kWaves == 1) {
            total = __shfl(inc, kWave - 1, kWave);
        } else {
            if (lane == kWave - 1) s_sum[buf][wave] = inc;
            __syncthreads();  // the other buffer's readers are done before it is written again
            double before = 0.0;
            total = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const double v = s_sum[buf][w];
                if (w == wave) before = total;
                total += v;
            }
            pre += before;
        }
        pre += carry;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            run[j] += pre;
            if (best == INT_MAX && u0 + j < hi && run[j] < lam) best = (int32_t)(u0 + j - first);
        }
        if (u0 + NI <= hi) {
#pragma unroll
            for (int j = 0; j < NI; j += 2)
                *reinterpret_cast<Pair *>(a.cum + u0 + j) = Pair{run[j], run[j + 1]};
        } else {
#pragma unroll
            for (int j = 0; j < NI; ++j)
                if (u0 + j < hi) a.cum[u0 + j] = run[j];
        }
        carry += total;
#pragma unroll
        for (int j = 0; j < NI; ++j) in[j] = next[j];
    }
    finish_group<NT>(a, o, tid, best, s_best);
}

// The same for a rollout long against its group, by NT threads.  Each wave has a stretch of the units: it
// sums its stretch, meets the others once for what precedes it, and scans the stretch by itself, kRows
// rows of 128 units at a time with the next kRows in flight, two units to a lane.  Latency bounds it, as
// it does scan_rollout with 256 threads, whose chunk of 1,024 units costs a trip to memory, one through
// LDS and a barrier in turn: 400,000 units 298 -> 211 us (turn means), 20,000 15.2 -> 13.7.  The stretches
// depend on the number of units alone, so cum is bit-reproducible here too.
constexpr int kRows = 2;
template <typename VT, int NT>
__device__ __forceinline__ void scan_long(const StopArgs &a, const Rollout &o, int tid, double *s_sum,
                                          int32_t *s_best) {
    constexpr int kWaves = NT / kWave;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    fill_outside(a, o, tid, NT);

    // 32-bit places from the first unit after K0 on: a call of groups has at most kRolloutUnits
    const VT *vals = static_cast<const VT *>(a.values) + o.from;
    double *cum = a.cum + o.from;
    const int n = o.hi > o.from ? (int)(o.hi - o.from) : 0, shift = (int)(o.from - o.first);
    constexpr int kRow = 2 * kWave, kStep = kRow * kRows;
    const int each = (n + kRow * kWaves - 1) / (kRow * kWaves) * kRow;
    const int begin = wave * each < n ? wave * each : n, end = begin + each < n ? begin + each : n;
    typedef VT Two __attribute__((ext_vector_type(2), aligned(sizeof(VT))));
    auto load = [&](int base, VT (*x)[2]) __attribute__((always_inline)) {
        if (base + kStep <= end) {
#pragma unroll
            for (int g = 0; g < kRows; ++g) {
                const Two v = *reinterpret_cast<const Two *>(vals + base + 2 * lane + g * kRow);
                x[g][0] = v[0];
                x[g][1] = v[1];
            }
        } else {
#pragma unroll
            for (int g = 0; g < kRows; ++g)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int u = base + 2 * lane + g * kRow + j;
                    x[g][j] = u < end ? vals[u] : (VT)0;
                }
        }
    };
    constexpr int kPer = 16 / sizeof(VT), kLoads = 6;
    typedef VT Vec __attribute__((ext_vector_type(kPer), aligned(sizeof(VT))));
    double sum[kPer] = {};
    int u = begin;
    for (; u + kLoads * kPer * kWave <= end; u += kLoads * kPer * kWave) {
        Vec v[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            v[i] = *reinterpret_cast<const Vec *>(vals + u + (i * kWave + lane) * kPer);
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
#pragma unroll
            for (int j = 0; j < kPer; ++j) sum[j] += (double)v[i][j];
    }
    for (u += lane; u < end; u += kWave) sum[0] += (double)vals[u];
#pragma unroll
    for (int j = 1; j < kPer; ++j) sum[0] += sum[j];
    const double mine = last_lane(wave_scan(sum[0]));
    if (lane == 0) s_sum[wave] = mine;
    __syncthreads();
    double carry = 0.0;
    for (int w = 0; w < wave; ++w) carry += s_sum[w];

    int32_t best = INT_MAX;
    auto step = [&](int base, const VT (*in)[2]) __attribute__((always_inline)) {
        double inc[kRows];
#pragma unroll
        for (int g = 0; g < kRows; ++g) inc[g] = wave_scan((double)in[g][0] + (double)in[g][1]);
#pragma unroll
        for (int g = 0; g < kRows; ++g) {
            const int u = base + 2 * lane + g * kRow;
            const double c0 = carry + moved<0x138, 0xF>(inc[g]) + (double)in[g][0], c1 = c0 + (double)in[g][1];
            carry += last_lane(inc[g]);
            if (best == INT_MAX && u < end && c0 < o.lam) best = u + shift;
            if (best == INT_MAX && u + 1 < end && c1 < o.lam) best = u + 1 + shift;
            if (u + 1 < end)
                *reinterpret_cast<Pair *>(cum + u) = Pair{c0, c1};
            else if (u < end)
                cum[u] = c0;
        }
    };
    VT x[2][kRows][2];
    load(begin, x[0]);
    load(begin + kStep, x[1]);
    for (int base = begin; base < end; base += 2 * kStep) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            step(base + h * kStep, x[h]);
            load(base + (h + 2) * kStep, x[h]);
        }
    }
    finish_group<NT>(a, o, tid, best, s_best);
}

// The whole test with a group of threads for each rollout: no tiles, no look-back, one launch.
// Latency bounds it: offsets, then values, K0 and domain together, then a chunk after the other.
// kRolloutUnits has what it measured.
//
// One wave per rollout, four to a workgroup, behind `helpers` workgroups that take the rollouts of more
// than kWaveLength units, which the waves pass over: helper k looks at rollouts k, k + helpers, ...
// 64 registers, so that eight waves fit a SIMD (with 85 it took 18.4 us for 32,768 rollouts of 8 units).
template <typename VT>
__global__ __launch_bounds__(256, 8) void stop_waves_kernel(StopArgs a, int helpers) {
    constexpr int kWaves = 256 / kWave;
    __shared__ double s_sum[kWaves];
    __shared__ int32_t s_best[kWaves], s_count;
    __shared__ int32_t s_long[256];
    const int64_t R = a.L.n_rollouts;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= helpers) {
        const int64_t r = (int64_t)((int)blockIdx.x - helpers) * kWaves +
                          __builtin_amdgcn_readfirstlane(tid / kWave);
        if (r >= R) return;
        const Rollout o = rollout_of(a, r, tid % kWave == 0);
        if (o.hi - o.lo <= kWaveLength)
            scan_rollout<VT, kWave, 2>(a, o, tid % kWave, nullptr, nullptr);
        return;
    }
    const int64_t step = (int64_t)helpers * 256;
    for (int64_t base = blockIdx.x; base < R; base += step) {
        if (tid == 0) s_count = 0;
        __syncthreads();
        const int64_t r = base + (int64_t)tid * helpers;
        if (tid < 256 && r < R) {
            const Rollout o = rollout_of(a, r, false);
            if (o.hi - o.lo > kWaveLength) s_long[atomicAdd(&s_count, 1)] = (int32_t)r;
        }
        __syncthreads();
        const int n = s_count;
        for (int i = 0; i < n; ++i) {
            int t = tid;
            asm volatile("" : "+v"(t));  // opaque: addresses formed once for all rollouts cost registers
            scan_long<VT, 256>(a, rollout_of(a, __builtin_amdgcn_readfirstlane(s_long[i]), false), t, s_sum, s_best);
            __syncthreads();  // the shared sums are read by all before the next rollout's are written
        }
    }
}

// A workgroup per rollout.
template <typename VT, int NT, int NI>
__global__ __launch_bounds__(NT) void stop_block_kernel(StopArgs a) {
    __shared__ double s_sum[2][NT / kWave];
    __shared__ int32_t s_best[NT / kWave];
    const Rollout o = rollout_of(a, blockIdx.x, threadIdx.x == 0);
    if (NT == 256 && o.hi - o.from > 8 * NT * NI)
        scan_long<VT, NT>(a, o, threadIdx.x, s_sum[0], s_best);
    else
        scan_rollout<VT, NT, NI>(a, o, threadIdx.x, s_sum, s_best);
}

template <typename VT>
static hipError_t launch_stop_rollouts(const StopArgs &a, int64_t per, hipStream_t stream) {
    const unsigned R = (unsigned)a.L.n_rollouts;
    // Threads by the rollouts' average length: enough for one chunk or two of it.
    if (per <= 128) {
        // no rollout is longer than the call
        const int helpers = a.n_units <= kWaveLength ? 0 : (R < kHelpers ? (int)R : kHelpers);
        hipLaunchKernelGGL(stop_waves_kernel<VT>, dim3((R + 3) / 4 + helpers), dim3(256), 0, stream, a, helpers);
    } else if (per <= 1024) {
        hipLaunchKernelGGL((stop_block_kernel<VT, 256, 4>), dim3(R), dim3(256), 0, stream, a);
    } else {
        hipLaunchKernelGGL((stop_block_kernel<VT, 1024, 8>), dim3(R), dim3(1024), 0, stream, a);
    }
    return hipGetLastError();
}

// Online form of the stop test (Algorithm 1's inner loop while a rollout is being
// generated): active rollout a = 0 .. n_active-1 (state slot rid[a]) receives new
// units [new_off[a], new_off[a+1]) with the given values; they are appended at
// local index state_units[slot] on.  One wavefront per active rollout scans them in
// 64-unit chunks (fixed shuffle tree in double) on top of the carried sum; the
// first crossing found (ballot, lowest lane) becomes stop_unit[slot].  A rollout
// that has already stopped ignores further units.
template <typename VT>
__global__ __launch_bounds__(256) void stop_step_kernel(int32_t n_active, const int32_t *rid,
                                                        const int64_t *new_off, const VT *values,
                                                        const int32_t *domain, DomainTable lambda,
                                                        int32_t n_dom, double *state_cum,
                                                        int32_t *state_units, int32_t *stop_unit,
                                                        uint32_t *flags) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t a = block_index<256>() * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (a >= n_active) return;
    const int32_t slot = rid[a];
    if (slot < 0) {
        if (lane == 0) raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    const int64_t b0 = new_off[a], b1 = new_off[a + 1];
    if (b1 < b0 || b0 < 0) {
        if (lane == 0) raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    const int32_t d = domain ? domain[slot] : 0;
    if (d < 0 || d >= n_dom) {
        if (lane == 0) raise_flag(flags, STRIDE_FLAG_BAD_DOMAIN);
        return;
    }
    const double lam = lambda.v[d];
    int32_t stop = stop_unit[slot];
    double carry = state_cum[slot];
    const int32_t u0 = state_units[slot];
    if (stop < 0) {
        for (int64_t c = b0; c < b1; c += kWave) {
            const int64_t i = c + lane;
            double v = (i < b1) ? (double)values[i] : 0.0;
            // inclusive scan of the chunk, fixed association
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const double t = __shfl_up(v, off, kWave);
                if (lane >= off) v += t;
            }
            const double cum = carry + v;
            const bool cross = (i < b1) && (cum < lam);
            const uint64_t hit = __ballot(cross);
            if (hit) {
                const int first = __builtin_ctzll(hit);
                stop = u0 + (int32_t)(c - b0) + first;
                carry = __shfl(cum, first, kWave);
                break;
            }
            const int last = (int)((b1 - c) < kWave ? (b1 - c) : kWave) - 1;
            carry = __shfl(cum, last, kWave);
        }
    }
    if (lane == 0) {
        state_cum[slot] = carry;
        state_units[slot] = u0 + (int32_t)(b1 - b0);
        stop_unit[slot] = stop;
    }
}

}  // namespace

hipError_t launch_stop_step(int32_t n_active, const int32_t *rid, const int64_t *new_off,
                            int32_t unit, const void *values, const int32_t *domain,
                            const DomainTable &lambda, int32_t n_dom, double *state_cum,
                            int32_t *state_units, int32_t *stop_unit, uint32_t *flags,
                            hipStream_t stream) {
    if (n_active == 0) return hipSuccess;
    const dim3 grid = grid_of(((int64_t)n_active + 3) / 4, 256);
    if (unit == STRIDE_UNIT_TURN)
        hipLaunchKernelGGL(stop_step_kernel<double>, grid, dim3(256), 0, stream, n_active,
                           rid, new_off, static_cast<const double *>(values), domain, lambda, n_dom,
                           state_cum, state_units, stop_unit, flags);
    else
        hipLaunchKernelGGL(stop_step_kernel<float>, grid, dim3(256), 0, stream, n_active,
                           rid, new_off, static_cast<const float *>(values), domain, lambda, n_dom,
                           state_cum, state_units, stop_unit, flags);
    return hipGetLastError();
}

hipError_t launch_stop(const stride_layout &L, int32_t unit, const void *values,
                       const DomainTable &lambda, int32_t n_dom, const int32_t *start,
                       double *cum, int32_t *stop_unit, int64_t *retained, uint32_t *flags,
                       void *ws, hipStream_t stream) {
    const int64_t n_units = (unit == STRIDE_UNIT_TURN) ? L.n_turns : L.n_tokens;
    const WsLayout w = ws_layout(L.n_rollouts, 0, n_units, 0);
    char *base = static_cast<char *>(ws);
    StopArgs a;
    a.L = L;
    a.lambda = lambda;
    a.n_dom = n_dom;
    a.unit = unit;
    a.n_units = n_units;
    a.n_tiles = (n_units + kScanTile - 1) / kScanTile;
    a.values = values;
    a.start = start;
    a.unit_off = reinterpret_cast<const int64_t *>(base + w.unit_off);
    a.cum = cum;
    a.stop_unit = stop_unit;
    a.retained = retained;
    a.counter = reinterpret_cast<uint32_t *>(base + w.counter);
    a.desc = reinterpret_cast<TileDesc *>(base + w.desc);
    a.flags = flags;
#ifdef STRIDE_SCAN_DELAY_HOOK
    a.delay_seed = g_delay_seed.load();
    a.delay_one_in = g_delay_one_in.load();
    a.delay_sleeps = g_delay_sleeps.load();
    a.spin_limit = g_spin_limit.load();
#else
    a.delay_seed = 0;
    a.delay_one_in = 0;
    a.delay_sleeps = 0;
    a.spin_limit = 0;
#endif

    const int64_t per = L.n_rollouts > 0 ? n_units / L.n_rollouts : 0;
    if (L.n_rollouts > 0 && L.n_rollouts <= kRolloutCount && n_units <= kRolloutUnits &&
        per <= kRolloutLength) {
        if (unit == STRIDE_UNIT_TURN)
            return launch_stop_rollouts<double>(a, per, stream);
        return launch_stop_rollouts<float>(a, per, stream);
    }
    const int64_t prep_n = (L.n_rollouts + 1 > a.n_tiles) ? L.n_rollouts + 1 : a.n_tiles;
    hipLaunchKernelGGL(stop_prep_kernel, dim3((unsigned)((prep_n + 255) / 256)), dim3(256), 0,
                       stream, a, reinterpret_cast<int64_t *>(base + w.unit_off));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.n_tiles > 0) {
        if (unit == STRIDE_UNIT_TURN)
            hipLaunchKernelGGL(stop_scan_kernel<double>, dim3((unsigned)a.n_tiles),
                               dim3(kScanThreads), 0, stream, a);
        else
            hipLaunchKernelGGL(stop_scan_kernel<float>, dim3((unsigned)a.n_tiles),
                               dim3(kScanThreads), 0, stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (L.n_rollouts > 0) {
        hipLaunchKernelGGL(stop_finish_kernel, dim3((unsigned)((L.n_rollouts + 255) / 256)),
                           dim3(256), 0, stream, a);
        e = hipGetLastError();
    }
    return e;
}

// ---- scratch of the allocation-free stop test ----
// A fixed device array, one copy per GPU, held until the process ends.  In host code
// `scratch` names a host-side stand-in, not a device address: the device address of each
// GPU's copy comes from hipGetSymbolAddress, looked up once per device with that device
// current, and only that address is handed to kernels.
static __device__ __align__(256) char scratch[STRIDE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;

hipError_t noalloc_scratch(void **ptr) {
    static std::atomic<void *> addr[kMaxDevices];
    static std::mutex mu;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *p = addr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> g(mu);
        p = addr[dev].load(std::memory_order_relaxed);
        if (!p) {
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            addr[dev].store(p, std::memory_order_release);
        }
    }
    *ptr = p;
    return hipSuccess;
}

}  // namespace stride

extern "C" stride_status stride_debug_scan_delay(uint64_t seed, uint32_t one_in, uint32_t sleeps) {
#ifdef STRIDE_SCAN_DELAY_HOOK
    if (one_in > 0 && (sleeps < 1 || sleeps > stride::kMaxDelaySleeps)) return STRIDE_ERR_INVALID_ARG;
    stride::g_delay_seed.store(seed);
    stride::g_delay_sleeps.store(sleeps);
    stride::g_delay_one_in.store(one_in);
    return STRIDE_OK;
#else
    (void)seed;
    (void)one_in;
    (void)sleeps;
    return STRIDE_ERR_UNSUPPORTED;
#endif
}

extern "C" stride_status stride_debug_scan_spin_limit(uint32_t limit) {
#ifdef STRIDE_SCAN_DELAY_HOOK
    stride::g_spin_limit.store(limit);
    return STRIDE_OK;
#else
    (void)limit;
    return STRIDE_ERR_UNSUPPORTED;
#endif
}
