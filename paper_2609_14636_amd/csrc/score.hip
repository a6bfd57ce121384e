// score.hip -- sampled-token log-probabilities of teacher and student rows.
//
// Eq. (1) (Sec. 3.1): log pi(y_t | y_<t) = x[y_t] - log sum_v exp(x[v]) over the
// row's V logits.  Each row is read exactly once from HBM.
//
// Design (gfx950, wave64): one wavefront, or 4, 8 or 16 wavefronts of a workgroup,
// per row (score_rows_kernel).  Lanes stream the row
// with 16-byte non-temporal loads (8 bf16 or 4 fp32 per load, consecutive
// lanes on consecutive 16-byte words, so one wave instruction moves 1 KiB,
// fully coalesced).  Each lane keeps a
// running (max m, sum s) in fp32 registers and rescales once per chunk of
// U loads, not once per element (online normaliser, Milakov and Gimelshein
// 2018).  Per element the work is: unpack (shift or mask), max, one fma into
// the exp2 argument, v_exp_f32, add.  The 64 lane states are merged with a
// fixed butterfly of cross-lane shuffles, so the result does not depend on
// timing.  The sampled logit is fetched with one scalar-sized load per row.
#include "common.hpp"

namespace stride {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;
constexpr uint8_t kBadDomain = 0xFF;
// Lowest reference point of a (max, sum) state: times log2(e) it is still finite in fp32.  A state that
// has seen only values below it (-inf, or a mask of the type's lowest value) has sum 0 and leaves no
// trace in the states that it is merged with; with the maximum itself as reference its sum would be
// infinite, and NaN after the merge.
constexpr float kLowestRef = -2.358e38f;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int DT>
struct Elem;
template <>
struct Elem<STRIDE_BF16> {
    static constexpr uint32_t kNegInf = 0xFF80FF80u;
    static constexpr int kPerVec = 8;
    static constexpr int kSize = 2;
};
template <>
struct Elem<STRIDE_F32> {
    static constexpr uint32_t kNegInf = 0xFF800000u;
    static constexpr int kPerVec = 4;
    static constexpr int kSize = 4;
};

template <int DT>
__device__ __forceinline__ void unpack(const u32x4 &v, float *x);

template <>
__device__ __forceinline__ void unpack<STRIDE_BF16>(const u32x4 &v, float *x) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(v[i] << 16);
        x[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
}

template <>
__device__ __forceinline__ void unpack<STRIDE_F32>(const u32x4 &v, float *x) {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(v[i]);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Fold n values into the lane's running (m, s0 + s1).  The reference point is
// the running maximum, at least kLowestRef, so that -inf - -inf never appears.
template <int N>
__device__ __forceinline__ void fold(float &m, float &s0, float &s1, const float *x) {
    float cm = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) cm = fmaxf(cm, x[i]);
    const float mn = fmaxf(m, cm);
    const float ref = fmaxf(mn, kLowestRef);
    const float scale = fast_exp2((m - ref) * kLog2e);
    s0 *= scale;
    s1 *= scale;
    const float mref = ref * kLog2e;
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        s0 += fast_exp2(__builtin_fmaf(x[i], kLog2e, -mref));
        if (i + 1 < N) s1 += fast_exp2(__builtin_fmaf(x[i + 1], kLog2e, -mref));
    }
    m = mn;
}

// Merge two (m, s) states.
__device__ __forceinline__ void merge(float &m, float &s, float m2, float s2) {
    const float mn = fmaxf(m, m2);
    const float ref = fmaxf(mn, kLowestRef);
    s = s * fast_exp2((m - ref) * kLog2e) + s2 * fast_exp2((m2 - ref) * kLog2e);
    m = mn;
}

struct ScoreArgs {
    PtrTable teachers;
    const void *student;
    const uint8_t *row_dom;
    const int32_t *ids;
    float *logp_t;
    float *logp_s;
    uint32_t *flags;
    int64_t n_rows;
    int64_t ld;
    int32_t vocab;
    int32_t n_teachers;
};

// Merge the 64 lane states of a wavefront with a fixed butterfly of cross-lane shuffles (every
// lane ends with the same result, so it does not depend on timing).
__device__ __forceinline__ void wave_merge(float &m, float &s) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float m2 = __shfl_xor(m, off, kWave);
        const float s2 = __shfl_xor(s, off, kWave);
        merge(m, s, m2, s2);
    }
}

template <int DT>
__device__ __forceinline__ float element(const u32x4 *p, int32_t i) {
    if (DT == STRIDE_BF16)
        return __uint_as_float((uint32_t)(reinterpret_cast<const uint16_t *>(p)[i]) << 16);
    return reinterpret_cast<const float *>(p)[i];
}

// The row's result from its (max, sum) and sampled logit: log pi(y) = x_y - m - log s, NaN and a
// flag for a non-finite row or a token id outside [0, V).
__device__ __forceinline__ void write_row(const ScoreArgs &a, int64_t row, int32_t y, float xy,
                                          float m, float s, float *out) {
    float r;
    uint32_t bad = 0;
    const bool finite = (m > -INFINITY) && (m < INFINITY) && (s > 0.0f) && (s < INFINITY);
    if (!finite) bad |= STRIDE_FLAG_NONFINITE;
    if (y < 0 || y >= a.vocab) bad |= STRIDE_FLAG_TOKEN_OOB;
    if (bad) {
        r = __builtin_nanf("");
        raise_flag(a.flags, bad);
    } else {
        // At most 0: the maximum's own term is 1 in exact arithmetic.  Here it is exp2 of the
        // rounding residual of m * log2(e) (the exponent argument is one fma against that
        // rounded product), which can sit a few 1e-7 below 1; the clamp removes only that
        // excess (-inf stays -inf).
        r = fminf((xy - m) - __builtin_amdgcn_logf(s) * kLn2, 0.0f);
    }
    out[row] = r;
}

// W wavefronts share a row, RW rows per workgroup, D chunks of U loads per wavefront: wavefront w
// folds the row's chunks w, w + W, ... with the next D - 1 in flight, and its share of the words
// after the last whole chunk, which it fetches first.  The wavefronts' (max, sum) states are
// merged in their order through LDS, so the result does not depend on timing (the forms differ
// in the order of rounding only).  HBM bounds it while there are rows for every CU.
// launch_score_rows has the choice of a form and what it measured.
template <int DT, int W, int RW, int U, int D>
__global__ __launch_bounds__(W *RW *kWave) void score_rows_kernel(ScoreArgs a) {
    static_assert(W == 1 || RW == 1, "wavefronts that share a row meet at a workgroup barrier");
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ float s_m[W], s_s[W], s_xy;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wave = W == 1 ? 0 : wid;
    const int64_t item = block_index<W * RW * kWave>() * RW + (W == 1 ? wid : 0);
    const bool two = a.student != nullptr;
    const int64_t n_items = two ? 2 * a.n_rows : a.n_rows;
    if (item >= n_items) return;  // W > 1: the whole workgroup, before any barrier
    const bool is_student = two && (item & 1);
    const int64_t row = two ? (item >> 1) : item;
    float *out = is_student ? a.logp_s : a.logp_t;

    const void *base;
    if (is_student) {
        base = a.student;
    } else {
        const int d = a.row_dom ? (int)a.row_dom[row] : 0;
        // row not covered by the layout or bad domain (already flagged); the same for all
        // wavefronts of the row, which leave before any barrier
        if (d >= a.n_teachers) {
            if (wave == 0 && lane == 0) out[row] = __builtin_nanf("");
            return;
        }
        base = a.teachers.p[d];
    }
    const u32x4 *p = reinterpret_cast<const u32x4 *>(static_cast<const char *>(base) +
                                                     row * a.ld * Elem<DT>::kSize);
    const int32_t y = a.ids[row];
    const int nvec = a.vocab / E;  // 16-byte words lying wholly inside [0, vocab)
    const int tail = a.vocab % E;
    constexpr int kStep = U * kWave;
    const int nfull = nvec / kStep;  // whole chunks
    const int mine = nfull > wave ? (nfull - wave + W - 1) / W : 0;

    float m = -INFINITY, s0 = 0.0f, s1 = 0.0f;
    auto load = [&](int i, u32x4 *v) __attribute__((always_inline)) {
        const u32x4 *q = p + (int64_t)(wave + i * W) * kStep + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(q + u * kWave);
    };
    auto use = [&](const u32x4 *v) __attribute__((always_inline)) {
        float x[U * E];
#pragma unroll
        for (int u = 0; u < U; ++u) unpack<DT>(v[u], x + u * E);
        fold<U * E>(m, s0, s1, x);
    };
    // words after the last whole chunk, every W-th block of 64 of them; -inf past the row
    constexpr int kRest = (U + W - 1) / W;
    u32x4 rest[kRest];
#pragma unroll
    for (int i = 0; i < kRest; ++i) {
        const int k = nfull * kStep + (i * W + wave) * kWave + lane;
        constexpr uint32_t n = Elem<DT>::kNegInf;
        rest[i] = u32x4{n, n, n, n};
        if (k < nvec) rest[i] = __builtin_nontemporal_load(p + k);
    }
    u32x4 v[D][U];
    if (D == 1) {
        for (int i = 0; i < mine; ++i) {
            load(i, v[0]);
            use(v[0]);
        }
    } else {
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < mine) load(d, v[d]);
        int i = 0;
        for (; i + 2 * D - 2 < mine; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load(i + d + D - 1, v[(d + D - 1) % D]);
                use(v[d]);
            }
        }
        // at most 2 D - 2 chunks left, the first D - 1 of them in flight
#pragma unroll
        for (int d = 0; d < 2 * D - 2; ++d) {
            if (i + d + D - 1 < mine) load(i + d + D - 1, v[(d + D - 1) % D]);
            if (i + d < mine) use(v[d % D]);
        }
    }
#pragma unroll
    for (int i = 0; i < kRest; ++i) {
        if (nfull * kStep + (i * W + wave) * kWave >= nvec) break;  // the same for the whole wavefront
        float x[E];
        unpack<DT>(rest[i], x);
        fold<E>(m, s0, s1, x);
    }
    if (tail && wave == 0 && lane == 0) {
        // The last word also holds ld - vocab padding elements: mask them out.
        float x[E];
        unpack<DT>(p[nvec], x);
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (j >= tail) x[j] = -INFINITY;
        fold<E>(m, s0, s1, x);
    }
    // The sampled logit is the last wavefront's: it has the fewest chunks, so the others' loads
    // cover this one (before the row it would hold up the wavefront until the token id is there).
    float xy = 0.0f;
    if (wave == W - 1 && y >= 0 && y < a.vocab) xy = element<DT>(p, y);
    float s = s0 + s1;
    wave_merge(m, s);
    if (W > 1) {
        if (lane == 0) {
            s_m[wave] = m;
            s_s[wave] = s;
            if (wave == W - 1) s_xy = xy;
        }
        __syncthreads();
        if (wave != 0) return;
        xy = s_xy;
#pragma unroll
        for (int w = 1; w < W; ++w) merge(m, s, s_m[w], s_s[w]);
    }
    if (lane == 0) write_row(a, row, y, xy, m, s, out);
}

// Exact reverse KL in the same pass: a token's wavefronts stream the teacher
// and the student row together.  With p_S(v) = exp(s_v - LSE_S),
//   KL(pi_S || pi_T) = sum_v p_S(v) (s_v - t_v) - LSE_S + LSE_T
//                    = A / Z_S - LSE_S + LSE_T,  A = sum_v exp(s_v - m_S) (s_v - t_v),
// and A rescales with the student's running maximum exactly like Z_S.
template <int N>
__device__ __forceinline__ void fold_pair(float &mt, float &zt, float &ms, float &zs, float &am,
                                          const float *t, const float *x) {
    float ct = t[0], cs = x[0];
#pragma unroll
    for (int i = 1; i < N; ++i) {
        ct = fmaxf(ct, t[i]);
        cs = fmaxf(cs, x[i]);
    }
    const float mtn = fmaxf(mt, ct), msn = fmaxf(ms, cs);
    const float rt = fmaxf(mtn, kLowestRef);
    const float rs = fmaxf(msn, kLowestRef);
    zt *= fast_exp2((mt - rt) * kLog2e);
    const float ss = fast_exp2((ms - rs) * kLog2e);
    zs *= ss;
    am *= ss;
    const float rtl = rt * kLog2e, rsl = rs * kLog2e;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        zt += fast_exp2(__builtin_fmaf(t[i], kLog2e, -rtl));
        const float e = fast_exp2(__builtin_fmaf(x[i], kLog2e, -rsl));
        zs += e;
        // an entry with no student mass adds nothing, even where t - s is infinite
        if (e > 0.0f) am = __builtin_fmaf(e, x[i] - t[i], am);
    }
    mt = mtn;
    ms = msn;
}

struct PairArgs {
    PtrTable teachers;
    const void *student;
    const uint8_t *row_dom;
    const int32_t *ids;
    float *logp_t;
    float *logp_s;
    float *kl_full;
    uint32_t *flags;
    int64_t n_rows;
    int64_t ld;
    int32_t vocab;
    int32_t n_teachers;
};

// Merge two (max, sum) states of the teacher row and two of the student row, with the
// student's A rescaled like its sum.
__device__ __forceinline__ void pair_merge(float &mt, float &zt, float &ms, float &zs, float &am,
                                           float mt2, float zt2, float ms2, float zs2, float am2) {
    merge(mt, zt, mt2, zt2);
    const float mn = fmaxf(ms, ms2);
    const float ref = fmaxf(mn, kLowestRef);
    const float f1 = fast_exp2((ms - ref) * kLog2e), f2 = fast_exp2((ms2 - ref) * kLog2e);
    zs = zs * f1 + zs2 * f2;
    am = am * f1 + am2 * f2;
    ms = mn;
}

// The 64 lane states of a wavefront merged by a fixed butterfly of cross-lane shuffles.
__device__ __forceinline__ void pair_wave_merge(float &mt, float &zt, float &ms, float &zs, float &am) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const float mt2 = __shfl_xor(mt, o, kWave), zt2 = __shfl_xor(zt, o, kWave);
        const float ms2 = __shfl_xor(ms, o, kWave), zs2 = __shfl_xor(zs, o, kWave);
        const float am2 = __shfl_xor(am, o, kWave);
        pair_merge(mt, zt, ms, zs, am, mt2, zt2, ms2, zs2, am2);
    }
}

// The token's exact KL and both sampled-token log-probabilities from the merged states and the
// sampled logits.
__device__ __forceinline__ void write_pair(const PairArgs &a, int64_t row, int32_t y, float xt,
                                           float xs, float mt, float zt, float ms, float zs,
                                           float am) {
    uint32_t bad = 0;
    const bool fin_t = (mt > -INFINITY) && (mt < INFINITY) && (zt > 0.0f) && (zt < INFINITY);
    const bool fin_s = (ms > -INFINITY) && (ms < INFINITY) && (zs > 0.0f) && (zs < INFINITY);
    if (!fin_t || !fin_s) bad |= STRIDE_FLAG_NONFINITE;
    const float lt = __builtin_amdgcn_logf(zt) * kLn2, ls = __builtin_amdgcn_logf(zs) * kLn2;
    // sum_v p_S (log p_S - log p_T) = A/Z_S - (m_S + log Z_S) + (m_T + log Z_T)
    // +inf when the teacher gives no mass where the student has some
    float kl = bad ? __builtin_nanf("") : (am / zs - (ms - mt)) - (ls - lt);
    if (!(kl == kl)) bad |= STRIDE_FLAG_NONFINITE;
    // KL >= 0 (Gibbs); when the two rows differ by a constant the fp32 terms cancel to a
    // rounding residue of either sign, and clamping only reduces that error (NaN stays NaN)
    if (kl < 0.0f) kl = 0.0f;
    a.kl_full[row] = kl;
    if (y < 0 || y >= a.vocab) bad |= STRIDE_FLAG_TOKEN_OOB;
    float rt, rs;
    if (bad & (STRIDE_FLAG_TOKEN_OOB | (fin_t && fin_s ? 0u : STRIDE_FLAG_NONFINITE))) {
        rt = rs = __builtin_nanf("");
    } else {
        rt = fminf((xt - mt) - lt, 0.0f);  // at most 0, as in score_rows_kernel
        rs = fminf((xs - ms) - ls, 0.0f);
    }
    if (bad) raise_flag(a.flags, bad);
    a.logp_t[row] = rt;
    a.logp_s[row] = rs;
}

// W wavefronts share a token's two rows, RW tokens per workgroup, D chunks of U loads of each row per
// wavefront, as in score_rows_kernel; the five-value states are merged in wavefront order.  The
// two exponentials and eleven other instructions per pair of entries keep the vector units busy
// for most of the time that HBM takes, so fewer wavefronts than for single rows pay.
template <int DT, int W, int RW, int U, int D>
__global__ __launch_bounds__(W *RW *kWave) void score_pairs_kernel(PairArgs a) {
    static_assert(W == 1 || RW == 1, "wavefronts that share a token meet at a workgroup barrier");
    constexpr int E = Elem<DT>::kPerVec;
    __shared__ float s_st[5][W], s_x[2];
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wave = W == 1 ? 0 : wid;
    const int64_t row = block_index<W * RW * kWave>() * RW + (W == 1 ? wid : 0);
    if (row >= a.n_rows) return;  // W > 1: the whole workgroup, before any barrier
    const int d = a.row_dom ? (int)a.row_dom[row] : 0;
    if (d >= a.n_teachers) {  // the same for the token's wavefronts: they leave before any barrier
        if (wave == 0 && lane == 0) {
            a.logp_t[row] = __builtin_nanf("");
            a.kl_full[row] = __builtin_nanf("");
            a.logp_s[row] = __builtin_nanf("");
        }
        return;
    }
    const size_t off = (size_t)row * a.ld * Elem<DT>::kSize;
    const u32x4 *pt = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.teachers.p[d]) + off);
    const u32x4 *ps = reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.student) + off);
    const int32_t y = a.ids[row];
    const int nvec = a.vocab / E;
    const int tail = a.vocab % E;
    constexpr int kStep = U * kWave;
    const int nfull = nvec / kStep;
    const int mine = nfull > wave ? (nfull - wave + W - 1) / W : 0;
    float mt = -INFINITY, zt = 0.0f, ms = -INFINITY, zs = 0.0f, am = 0.0f;
    struct Chunk {
        u32x4 t[U], s[U];
    };
    auto load = [&](int i, Chunk &v) __attribute__((always_inline)) {
        const int64_t k = (int64_t)(wave + i * W) * kStep + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v.t[u] = __builtin_nontemporal_load(pt + k + u * kWave);
            v.s[u] = __builtin_nontemporal_load(ps + k + u * kWave);
        }
    };
    auto use = [&](const Chunk &v) __attribute__((always_inline)) {
        float xt[U * E], xs[U * E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            unpack<DT>(v.t[u], xt + u * E);
            unpack<DT>(v.s[u], xs + u * E);
        }
        fold_pair<U * E>(mt, zt, ms, zs, am, xt, xs);
    };
    // words after the last whole chunk, every W-th block of 64 of them
    constexpr int kRest = (U + W - 1) / W;
    u32x4 rest_t[kRest], rest_s[kRest];
#pragma unroll
    for (int i = 0; i < kRest; ++i) {
        const int k = nfull * kStep + (i * W + wave) * kWave + lane;
        constexpr uint32_t n = Elem<DT>::kNegInf;
        rest_t[i] = rest_s[i] = u32x4{n, n, n, n};
        if (k < nvec) {
            rest_t[i] = __builtin_nontemporal_load(pt + k);
            rest_s[i] = __builtin_nontemporal_load(ps + k);
        }
    }
    Chunk v[D];
    if (D == 1) {
        for (int i = 0; i < mine; ++i) {
            load(i, v[0]);
            use(v[0]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < D - 1; ++q)
            if (q < mine) load(q, v[q]);
        int i = 0;
        for (; i + 2 * D - 2 < mine; i += D) {
#pragma unroll
            for (int q = 0; q < D; ++q) {
                load(i + q + D - 1, v[(q + D - 1) % D]);
                use(v[q]);
            }
        }
        // at most 2 D - 2 chunks left, the first D - 1 of them in flight
#pragma unroll
        for (int q = 0; q < 2 * D - 2; ++q) {
            if (i + q + D - 1 < mine) load(i + q + D - 1, v[(q + D - 1) % D]);
            if (i + q < mine) use(v[q % D]);
        }
    }
#pragma unroll
    for (int i = 0; i < kRest; ++i) {
        if (nfull * kStep + (i * W + wave) * kWave >= nvec) break;  // the same for the whole wavefront
        float xt[E], xs[E];
        unpack<DT>(rest_t[i], xt);
        unpack<DT>(rest_s[i], xs);
        fold_pair<E>(mt, zt, ms, zs, am, xt, xs);
    }
    if (tail && wave == 0 && lane == 0) {
        float xt[E], xs[E];
        unpack<DT>(pt[nvec], xt);
        unpack<DT>(ps[nvec], xs);
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (j >= tail) {
                xt[j] = -INFINITY;
                xs[j] = -INFINITY;
            }
        fold_pair<E>(mt, zt, ms, zs, am, xt, xs);
    }
    float yt = 0.0f, ys = 0.0f;  // the sampled logits: the last wavefront has the fewest chunks
    if (wave == W - 1 && y >= 0 && y < a.vocab) {
        yt = element<DT>(pt, y);
        ys = element<DT>(ps, y);
    }
    pair_wave_merge(mt, zt, ms, zs, am);
    if (W > 1) {
        if (lane == 0) {
            s_st[0][wave] = mt;
            s_st[1][wave] = zt;
            s_st[2][wave] = ms;
            s_st[3][wave] = zs;
            s_st[4][wave] = am;
            if (wave == W - 1) {
                s_x[0] = yt;
                s_x[1] = ys;
            }
        }
        __syncthreads();
        if (wave != 0) return;
        yt = s_x[0];
        ys = s_x[1];
#pragma unroll
        for (int w = 1; w < W; ++w)
            pair_merge(mt, zt, ms, zs, am, s_st[0][w], s_st[1][w], s_st[2][w], s_st[3][w], s_st[4][w]);
    }
    if (lane == 0) write_pair(a, row, y, yt, ys, mt, zt, ms, zs, am);
}

// Teacher index of every row: row -> turn (by offsets) -> rollout -> domain.
// Rows outside every turn, or whose rollout's domain is out of range, get
// kBadDomain and raise a flag, so the scoring kernel writes NaN for them.
__global__ __launch_bounds__(256) void row_domain_kernel(stride_layout L, int32_t n_teachers,
                                                         uint8_t *row_dom, uint32_t *flags) {
    const int64_t i = block_index<256>() * blockDim.x + threadIdx.x;
    if (i >= L.n_tokens) return;
    // last turn t with turn_tok_off[t] <= i
    int64_t lo = 0, hi = L.n_turns;  // answer in [0, T)
    if (L.n_turns == 0 || L.turn_tok_off[0] > i) {
        row_dom[i] = kBadDomain;
        raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (L.turn_tok_off[mid] <= i) lo = mid; else hi = mid;
    }
    const int64_t t = lo;
    if (i >= L.turn_tok_off[t + 1]) {
        row_dom[i] = kBadDomain;
        raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    int64_t rlo = 0, rhi = L.n_rollouts;
    if (L.n_rollouts == 0 || L.rollout_turn_off[0] > t) {
        row_dom[i] = kBadDomain;
        raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    while (rhi - rlo > 1) {
        const int64_t mid = (rlo + rhi) >> 1;
        if (L.rollout_turn_off[mid] <= t) rlo = mid; else rhi = mid;
    }
    if (t >= L.rollout_turn_off[rlo + 1]) {
        row_dom[i] = kBadDomain;
        raise_flag(flags, STRIDE_FLAG_BAD_OFFSETS);
        return;
    }
    const int32_t d = L.domain ? L.domain[rlo] : 0;
    if (d < 0 || d >= n_teachers) {
        row_dom[i] = kBadDomain;
        raise_flag(flags, STRIDE_FLAG_BAD_DOMAIN);
        return;
    }
    row_dom[i] = (uint8_t)d;
}

template <int DT, int W, int RW, int U, int D>
hipError_t launch_rows_form(const ScoreArgs &a, hipStream_t stream) {
    const int64_t items = a.student ? 2 * a.n_rows : a.n_rows;
    hipLaunchKernelGGL((score_rows_kernel<DT, W, RW, U, D>), grid_of((items + RW - 1) / RW, W * RW * kWave),
                       dim3(W * RW * kWave), 0, stream, a);
    return hipGetLastError();
}

// The form by the row's 16-byte words and the number of row items (teacher and student rows, called rows
// below).  More wavefronts per row read fewer rows at a time, and leave less of the chip idle at the end,
// but each needs words enough for its loads.  Teacher and student rows, bf16, one wavefront per row -> the form taken here:
//   words    8, 32,768 rows: 23.6 -> 21.2 us (28.4 with the folds of words that are not there)
//   words  125, 60,000 rows: 57.6 -> 36.1 us (U = 4 instead of 8; eight wavefronts 131)
//   words 1,000: 32 rows 6.2 -> 5.6 us, 512 rows 7.2 -> 6.1, 2,048 rows 15.2 -> 9.3 (four wavefronts; one
//                7.8, 9.0 and 10.2, but 26.0 against 27.3 at 8,192); words 300: 512 rows 6.2 -> 5.9 (one 6.6),
//                2,048 rows 10.5 -> 7.1 (four 7.7).  These and the next are graph replays with the turn mean
//   words 1,030: 80,000 rows 219 -> 217 us (U = 8 leaves two of four wavefronts without a chunk: 252)
//   words 2,000, 60,000 rows: 282 -> 274 us; 2,000 rows 13.8 -> 12.5
//   words 4,000, 60,000 rows: 561 -> 524 us; words 6,250, 32,768 rows: 480 -> 458
//   words 8,300: 128 rows 9.1 -> 9.0 us (three chunks of U = 4 in flight, the form of more rows, 10.1);
//                words 18,992: 512 rows 25.9 us either way (26.7), 8,192 rows 365 (357)
//   words 18,992, rows for half the CUs at most: 64 rows 12.4 us (sixteen wavefronts; eight 13.1, with three
//                chunks in flight 12.8), 128 rows 13.3 (13.4, 13.6), and 11.3 (11.9, 11.5) and 11.8 (12.9, 12.2)
//                where the last-level cache holds them; 160 rows 13.9 (13.8, 14.3).  Words 12,500, 64 rows
//                9.9 (10.4, 11.1), but 10,500 9.5 (9.3, 9.9), and fp32 18,992 11.3 (11.0, 11.3)
//   words 12,500, 80,000 rows: 2,368 -> 2,252 us (U = 8, one chunk at a time: 2,260)
//   words 18,992: 128 rows 58 -> 11 us, 8,192 rows 383 -> 362 (sixteen wavefronts 366),
//                 32,768 rows 1,444 -> 1,425 (eight 1,435), 174,554 rows 7,681 -> 7,637 (7,669),
//                 196,608 rows 9,052 -> 8,931, 262,144 rows 11,736 -> 11,719
// Sixteen wavefronts at 48,000 rows, alternating with one and with eight: 0.943 and 0.960 of one's time at
// 16,200 words, 0.948 and 0.960 at 17,200, 0.953 and 0.965 at 19,800, 0.956 and 0.975 at 20,800; but
// 0.966 and 0.959 at 12,000, 1.06 and 0.943 at 9,000.  These rows start on 128-byte lines.  Off them
// eight are ahead, 1.003 and 0.987 at 16,700 words, 1.001 and 0.979 at 19,300: two wavefronts then share a
// line at each chunk's edge, and may both read it.  fp32 rows hold half the arithmetic per word and leave
// registers for two such workgroups per CU: sixteen from 8,448 words on, on lines or off them (853 against
// 869 us at 12,500 words, 30,000 rows; 1.04 of one wavefront's time at 8,192 words, where eight take 1.00).
template <int DT>
hipError_t launch_rows(const ScoreArgs &a, hipStream_t stream) {
    const int words = a.vocab / Elem<DT>::kPerVec;
    const int64_t items = a.student ? 2 * a.n_rows : a.n_rows;
    if (words < 1024) {
        if (items <= (words < 512 ? 1024 : 2048)) return launch_rows_form<DT, 4, 1, 4, 1>(a, stream);
        return launch_rows_form<DT, 1, 8, 4, 1>(a, stream);
    }
    if (DT == STRIDE_BF16 && words < 1408) return launch_rows_form<DT, 4, 1, 4, 1>(a, stream);
    if (words < 3072) return launch_rows_form<DT, 4, 1, 8, 1>(a, stream);
    if (DT == STRIDE_BF16 && words >= 12288 && items <= 128) return launch_rows_form<DT, 16, 1, 8, 1>(a, stream);
    if (words < 8192 || items < 4096) return launch_rows_form<DT, 8, 1, 8, 1>(a, stream);
    const bool lines = a.ld * Elem<DT>::kSize % 128 == 0;
    if (items >= 16384 && (DT == STRIDE_F32 ? words >= 8448 : (lines && words >= 16384 && words < 24576)))
        return launch_rows_form<DT, 16, 1, 8, 1>(a, stream);
    return launch_rows_form<DT, 8, 1, 4, 3>(a, stream);
}

template <int DT, int W, int RW, int U, int D>
hipError_t launch_pairs_form(const PairArgs &a, hipStream_t stream) {
    hipLaunchKernelGGL((score_pairs_kernel<DT, W, RW, U, D>), grid_of((a.n_rows + RW - 1) / RW, W * RW * kWave),
                       dim3(W * RW * kWave), 0, stream, a);
    return hipGetLastError();
}

// The form by the row's 16-byte words and the number of tokens, as for single rows.  bf16, eight
// wavefronts with one chunk in flight for every length -> the form taken here:
//   words  125, 30,000 tokens: 199 -> 32 us; words 500: 299 -> 78
//   words 1,000: 16 tokens 7.4 -> 6.9 us, 256 tokens 8.1 -> 7.2, 1,024 tokens 14.7 -> 10.8 (four wavefronts;
//                one 10.1, 12.5 and 14.0, but 28.7 against 31.6 at 4,096); words 300: 512 tokens 8.7 -> 7.9
//                (one 8.4), 1,024 tokens 8.4 either way
//   words 1,500, 30,000 tokens: 383 -> 220 us
//   words 4,000: 256 tokens 10.9 -> 10.8 us (four wavefronts 11.9), 4,096 tokens 90 -> 89 (93), 40,000 801 -> 771
//                (790); words 3,100: 4,096 tokens 74 -> 69, but fp32 69.9 -> 69.4 with eight (four 70.2)
//   words 12,500, 5,000 tokens: 303 -> 298 us (four wavefronts 304)
//   words 18,992: 64 tokens 23 us either way (four 28), 16,384 tokens 1,434 -> 1,422, 60,000 tokens
//                 5,210 -> 5,165 (one wavefront per token 5,287)
template <int DT>
hipError_t launch_pairs(const PairArgs &a, hipStream_t stream) {
    const int words = a.vocab / Elem<DT>::kPerVec;
    if (words < 1024 && a.n_rows > (words < 256 ? 256 : 1024))
        return launch_pairs_form<DT, 1, 4, 2, 1>(a, stream);
    if (words < (DT == STRIDE_BF16 ? 3584 : 2560)) return launch_pairs_form<DT, 4, 1, 4, 1>(a, stream);
    if (a.n_rows >= 16384) return launch_pairs_form<DT, 4, 1, 4, 2>(a, stream);
    return launch_pairs_form<DT, 8, 1, 4, 1>(a, stream);
}

}  // namespace

hipError_t launch_score_pairs(int32_t dtype, const PtrTable &teachers, int32_t n_teachers,
                              const uint8_t *row_dom, const void *student, const int32_t *ids,
                              float *logp_t, float *logp_s, float *kl_full, int64_t n_rows,
                              int32_t vocab, int64_t ld, uint32_t *flags, hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    PairArgs a;
    a.teachers = teachers;
    a.student = student;
    a.row_dom = row_dom;
    a.ids = ids;
    a.logp_t = logp_t;
    a.logp_s = logp_s;
    a.kl_full = kl_full;
    a.flags = flags;
    a.n_rows = n_rows;
    a.ld = ld;
    a.vocab = vocab;
    a.n_teachers = n_teachers;
    if (dtype == STRIDE_BF16) return launch_pairs<STRIDE_BF16>(a, stream);
    return launch_pairs<STRIDE_F32>(a, stream);
}

hipError_t launch_row_domain(const stride_layout &L, int32_t n_teachers, uint8_t *row_dom,
                             uint32_t *flags, hipStream_t stream) {
    if (L.n_tokens == 0) return hipSuccess;
    const int64_t blocks = (L.n_tokens + 255) / 256;
    hipLaunchKernelGGL(row_domain_kernel, grid_of(blocks, 256), dim3(256), 0, stream, L,
                       n_teachers, row_dom, flags);
    return hipGetLastError();
}

hipError_t launch_score_rows(int32_t dtype, const PtrTable &teachers, int32_t n_teachers,
                             const uint8_t *row_dom, const void *student, const int32_t *ids,
                             float *logp_t, float *logp_s, int64_t n_rows, int32_t vocab,
                             int64_t ld, uint32_t *flags, hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    ScoreArgs a;
    a.teachers = teachers;
    a.student = student;
    a.row_dom = row_dom;
    a.ids = ids;
    a.logp_t = logp_t;
    a.logp_s = logp_s;
    a.flags = flags;
    a.n_rows = n_rows;
    a.ld = ld;
    a.vocab = vocab;
    a.n_teachers = n_teachers;
    if (dtype == STRIDE_BF16) return launch_rows<STRIDE_BF16>(a, stream);
    return launch_rows<STRIDE_F32>(a, stream);
}

}  // namespace stride
